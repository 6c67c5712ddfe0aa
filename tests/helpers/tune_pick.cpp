// Reads "candidates rounds incumbent" and the candidates' times; prints the choice.
#include <cstdio>

#include "asd_tune.h"

int main()
{
    size_t n, r, inc;
    while (std::scanf("%zu %zu %zu", &n, &r, &inc) == 3) {
        std::vector<std::vector<double>> t(n, std::vector<double>(r));
        for (auto &v : t)
            for (double &x : v)
                if (std::scanf("%lf", &x) != 1) return 1;
        std::printf("%zu\n", asd::tune_pick(t, inc));
    }
    return 0;
}

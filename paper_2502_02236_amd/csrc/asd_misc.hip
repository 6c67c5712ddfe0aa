// asd_misc.hip -- Philox export, step-counter and window bookkeeping,
// column freezing for window shifts, the FP64 reductions, and the window-end
// transfer to and from a coarse (micromagnetic) grid.
#include <algorithm>

#include "asd_device.h"
#include "asd_internal.h"
#include "asd.h"
#include "asd_pair.h"

namespace asd {

__global__ void k_philox_export(uint32_t k0, uint32_t k1, int rounds, const uint32_t *ctr,
                                uint32_t *out, int64_t n)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint4 c = reinterpret_cast<const uint4 *>(ctr)[i];
    Words4 w = philox4x32(rounds, k0, k1, c.x, c.y, c.z, c.w);
    reinterpret_cast<uint4 *>(out)[i] = make_uint4(w.w0, w.w1, w.w2, w.w3);
}

int launch_philox_export(uint64_t seed, int rounds, const uint32_t *ctr, uint32_t *out, int64_t n,
                         void *stream)
{
    if (n == 0) return 0;
    int64_t blocks = (n + 255) / 256;
    hipLaunchKernelGGL(k_philox_export, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream,
                       (uint32_t)seed, (uint32_t)(seed >> 32), rounds, ctr, out, n);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

__global__ void k_advance(int64_t *step_base, int64_t n)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) *step_base += n;
}

int launch_advance_step(int64_t *step_base, int64_t n, void *stream)
{
    hipLaunchKernelGGL(k_advance, dim3(1), dim3(64), 0, (hipStream_t)stream, step_base, n);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

struct I32x8 {
    int32_t v[8];
};

__global__ void k_set_i32(int32_t *dst, I32x8 vals, int n)
{
    int i = threadIdx.x;
    if (i < n) dst[i] = vals.v[i];
}

int launch_set_i32(int32_t *dst, const int32_t *vals, int n, void *stream)
{
    for (int off = 0; off < n; off += 8) {
        I32x8 v{};
        int m = n - off < 8 ? n - off : 8;
        for (int k = 0; k < m; ++k) v.v[k] = vals[off + k];
        hipLaunchKernelGGL(k_set_i32, dim3(1), dim3(64), 0, (hipStream_t)stream, dst + off, v, m);
    }
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// copy stored columns [x0, x0 + ncols) of one system from src to dst
template <typename T>
__global__ void k_copy_columns(T *dst, const T *src, int64_t ncs, int64_t base, int kind, int sx,
                               int ny, int nz, int x0, int ncols)
{
    int per_col = (kind == ASD_SC ? 1 : 2);
    int64_t m = (int64_t)ncols * ny * nz * per_col;
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= m) return;
    int s = (int)(t % per_col);
    int64_t r = t / per_col;
    int xc = (int)(r % ncols);
    int64_t yz = r / ncols;
    int64_t cell = (x0 + xc) + (int64_t)sx * yz;
    int64_t i = base + cell * per_col + s;
    for (int k = 0; k < 3; ++k) dst[k * ncs + i] = src[k * ncs + i];
}

int launch_copy_columns(int prec, void *dst, const void *src, int64_t ncs, const SysDev &d, int x0,
                        int ncols, void *stream)
{
    int per_col = (d.kind == ASD_SC ? 1 : 2);
    int64_t m = (int64_t)ncols * d.ny * d.nz * per_col;
    if (m == 0) return 0;
    unsigned blocks = (unsigned)((m + 255) / 256);
    if (prec == ASD_FP64)
        hipLaunchKernelGGL(k_copy_columns<double>, dim3(blocks), dim3(256), 0, (hipStream_t)stream,
                           (double *)dst, (const double *)src, ncs, d.base, d.kind, d.sx, d.ny, d.nz,
                           x0, ncols);
    else
        hipLaunchKernelGGL(k_copy_columns<float>, dim3(blocks), dim3(256), 0, (hipStream_t)stream,
                           (float *)dst, (const float *)src, ncs, d.base, d.kind, d.sx, d.ny, d.nz,
                           x0, ncols);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// The three component rows of n elements at src, src + ncs, src + 2 ncs to dst
// [3][n], in chunks of V (the widest the alignment of every row allows); one
// launch where three device copies cost three (about 5 us each on a lattice
// that fits the caches).
template <typename V>
__global__ __launch_bounds__(256) void k_copy_rows(V *__restrict__ dst, const V *__restrict__ src,
                                                   int64_t n, int64_t ncs)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const V *s = src + blockIdx.y * ncs;
    V *d = dst + blockIdx.y * n;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) d[i] = s[i];
}

int launch_copy_rows(void *dst, const void *src, size_t row_bytes, size_t stride_bytes, void *stream)
{
    if (row_bytes == 0) return 0;
    const uintptr_t al = (uintptr_t)dst | (uintptr_t)src | row_bytes | stride_bytes;
    hipStream_t st = (hipStream_t)stream;
    auto grid = [](size_t n) { return dim3((unsigned)std::min<size_t>((n + 255) / 256, 4096), 3); };
    if (al % 16 == 0) {
        const size_t n = row_bytes / 16;
        hipLaunchKernelGGL(k_copy_rows<uint4>, grid(n), dim3(256), 0, st, (uint4 *)dst,
                           (const uint4 *)src, (int64_t)n, (int64_t)(stride_bytes / 16));
    } else if (al % 4 == 0) {
        const size_t n = row_bytes / 4;
        hipLaunchKernelGGL(k_copy_rows<uint32_t>, grid(n), dim3(256), 0, st, (uint32_t *)dst,
                           (const uint32_t *)src, (int64_t)n, (int64_t)(stride_bytes / 4));
    } else {
        return -2;
    }
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <typename T>
__global__ void k_mask(T *buf, int64_t ncs, const uint16_t *label, int64_t base, int64_t n)
{
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    int64_t i = base + t;
    if (label[i] == kNoGrain) {
        buf[i] = 0;
        buf[ncs + i] = 0;
        buf[2 * ncs + i] = 0;
    }
}

int launch_mask_spins(int prec, void *buf, int64_t ncs, const uint16_t *label, const SysDev &d,
                      void *stream)
{
    if (d.n_stored == 0) return 0;
    unsigned blocks = (unsigned)((d.n_stored + 255) / 256);
    if (prec == ASD_FP64)
        hipLaunchKernelGGL(k_mask<double>, dim3(blocks), dim3(256), 0, (hipStream_t)stream,
                           (double *)buf, ncs, label, d.base, d.n_stored);
    else
        hipLaunchKernelGGL(k_mask<float>, dim3(blocks), dim3(256), 0, (hipStream_t)stream,
                           (float *)buf, ncs, label, d.base, d.n_stored);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// A field per coarse cell of a window mesh ncx x ncy x ncz (dst [3][ncell]
// in the handle precision) from the cells [off, off + ncx) along x of a
// wider mesh of src_nx cells (src [3][src_nx ncy ncz], FP64)
template <typename T>
__global__ void k_cells_from_mesh(T *dst, const double *src, int src_nx, int src_off, int ncx,
                                  int ncy, int ncz)
{
    const int64_t ncell = (int64_t)ncx * ncy * ncz;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= 3 * ncell) return;
    const int c = (int)(t / ncell);
    const int64_t q = t - c * ncell;
    const int i = (int)(q % ncx);
    const int64_t jk = q / ncx;
    dst[t] = (T)src[c * (int64_t)src_nx * ncy * ncz + (src_off + i) + (int64_t)src_nx * jk];
}

int launch_cells_from_mesh(int prec, void *dst, const double *src, int src_nx, int src_off, int ncx,
                           int ncy, int ncz, void *stream)
{
    const int64_t n = 3 * (int64_t)ncx * ncy * ncz;
    const int blocks = (int)((n + 255) / 256);
    if (prec == ASD_FP64)
        hipLaunchKernelGGL(k_cells_from_mesh<double>, dim3(blocks), dim3(256), 0, (hipStream_t)stream,
                           (double *)dst, src, src_nx, src_off, ncx, ncy, ncz);
    else
        hipLaunchKernelGGL(k_cells_from_mesh<float>, dim3(blocks), dim3(256), 0, (hipStream_t)stream,
                           (float *)dst, src, src_nx, src_off, ncx, ncy, ncz);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// ---------------------------------------------------------------- reductions
// Sum of N values per thread over a workgroup of B threads, into thread 0:
// lanes of a wavefront by shuffles, then the wavefronts in order.
constexpr int kSumBlock = 1024;

template <int B, int N>
__device__ __forceinline__ void block_sum(double (&v)[N])
{
    __shared__ double part[N][B / 64];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
#pragma unroll
        for (int k = 0; k < N; ++k) v[k] += __shfl_down(v[k], off);
    if ((threadIdx.x & 63) == 0)
        for (int k = 0; k < N; ++k) part[k][threadIdx.x >> 6] = v[k];
    __syncthreads();
    if (threadIdx.x == 0)
        for (int k = 0; k < N; ++k) {
            v[k] = part[k][0];
            for (int w = 1; w < B / 64; ++w) v[k] += part[k][w];
        }
}

__device__ __forceinline__ bool site_in_window(const SysDev &d, int org, int32_t local)
{
    if (!d.track) return true;
    const uint32_t cell = d.kind == ASD_SC ? (uint32_t)local : ((uint32_t)local >> 1);
    const int32_t X = (int32_t)(cell % (uint32_t)d.sx);
    return X >= org && X < org + d.nx;
}

// Spin sums of the grains, each grain's site list (ascending site index) cut
// into n_parts equal parts, one workgroup per part.  Each pass covers kRedUnroll
// * kRedBlock sites: thread t takes sites t, t + kRedBlock, ... (coalesced),
// loads them all (beyond the part its last site, for a site outside the window the
// system's first one: without branches between them all are in flight, 512 systems
// of 2816 sites 9.0 -> 6.7 us), then adds them in that order; the workgroup then sums
// its threads in a fixed tree.  The order depends only on the site list, so the
// FP64 result is the same in every run.  Bound by the latency of the gather
// (index, then spins): one workgroup per grain left most of the chip idle (40
// us for the 224 grains of a 400x200x33 window, 50 us for 32 isolated grains).
constexpr int kRedBlock = 256;
// sites per thread and pass (independent loads): a part of up to 2048 sites in one pass
constexpr int kRedUnroll = 8;

template <typename T>
__global__ __launch_bounds__(kRedBlock) void k_reduce_parts(RedArgs a)
{
    const int g = blockIdx.x / a.n_parts, part = blockIdx.x - g * a.n_parts;
    const int s = a.grain_sys[g];
    const SysDev d = a.sys[s];
    const int org = d.track ? a.origin[s] : 0;
    const T *S = (const T *)a.S;
    const int64_t ka = a.grain_ptr[g], kb = a.grain_ptr[g + 1];
    const int64_t len = (kb - ka + a.n_parts - 1) / a.n_parts;
    const int64_t k0 = min(ka + part * len, kb), k1 = min(k0 + len, kb);
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t base = k0; base < k1; base += (int64_t)kRedUnroll * kRedBlock) {
        int32_t loc[kRedUnroll];
        bool ok[kRedUnroll];
#pragma unroll
        for (int j = 0; j < kRedUnroll; ++j) {
            const int64_t k = base + threadIdx.x + (int64_t)j * kRedBlock;
            ok[j] = k < k1;
            loc[j] = a.grain_sites[ok[j] ? k : k1 - 1];
        }
        T v[kRedUnroll][3];
#pragma unroll
        for (int j = 0; j < kRedUnroll; ++j) {
            ok[j] = ok[j] && site_in_window(d, org, loc[j]);
            const int64_t i = d.base + (ok[j] ? loc[j] : 0);
            v[j][0] = S[i];
            v[j][1] = S[a.ncs + i];
            v[j][2] = S[2 * a.ncs + i];
        }
#pragma unroll
        for (int j = 0; j < kRedUnroll; ++j) {
            acc[0] += ok[j] ? (double)v[j][0] : 0.0;
            acc[1] += ok[j] ? (double)v[j][1] : 0.0;
            acc[2] += ok[j] ? (double)v[j][2] : 0.0;
            acc[3] += ok[j] ? 1.0 : 0.0;
        }
    }
    block_sum<kRedBlock>(acc);
    if (threadIdx.x == 0)
        for (int k = 0; k < 4; ++k) a.part[4 * (int64_t)blockIdx.x + k] = acc[k];
}

int launch_reduce_grains(const RedArgs &a, void *stream)
{
    if (a.n_grains == 0) return 0;
    const dim3 grid((unsigned)a.n_grains * (unsigned)a.n_parts);
    if (a.prec == ASD_FP64)
        hipLaunchKernelGGL(k_reduce_parts<double>, grid, dim3(kRedBlock), 0, (hipStream_t)stream, a);
    else
        hipLaunchKernelGGL(k_reduce_parts<float>, grid, dim3(kRedBlock), 0, (hipStream_t)stream, a);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// the sums t of system s; optional moment statistics of m = |M| / N: samples,
// sum m, sum m^2, sum m^4
__device__ __forceinline__ void system_out(const RedArgs &a, int s, const double (&t)[4], int moments,
                                           int reset)
{
    for (int k = 0; k < 4; ++k) a.sys_out[4 * (int64_t)s + k] = t[k];
    if (moments) {
        double *mo = a.moments + 5 * (int64_t)s;
        if (reset)
            for (int k = 0; k < 5; ++k) mo[k] = 0.0;
        double m = t[3] > 0.0 ? sqrt(t[0] * t[0] + t[1] * t[1] + t[2] * t[2]) / t[3] : 0.0;
        double m2 = m * m;
        mo[0] += 1.0;
        mo[1] += m;
        mo[2] += m2;
        mo[3] += m2 * m2;
    }
}

// One workgroup of B threads per system: every grain's sum from its parts in order
// (a thread per grain up to kPartsThread parts, a wavefront per grain beyond),
// then the system's from its grains in a fixed tree.  One thread walking the 224
// grains of a window took 28 us.  Systems whose grains one wavefront covers get no
// more than that (the same sums: the others would add zeros).
constexpr int kPartsThread = 16;

template <int B>
__global__ __launch_bounds__(B) void k_reduce_systems(RedArgs a, int moments, int reset)
{
    const int s = blockIdx.x;
    const int g0 = a.sys[s].grain_base, g1 = g0 + a.sys[s].n_grains, P = a.n_parts;
    const bool by_wave = P > kPartsThread;
    const int lane = threadIdx.x & 63;
    double t[4] = {0.0, 0.0, 0.0, 0.0};
    const int first = by_wave ? (int)(threadIdx.x >> 6) : (int)threadIdx.x;
    for (int g = g0 + first; g < g1; g += by_wave ? B / 64 : B) {
        const double *p = a.part + 4 * (int64_t)g * P;
        double v[4] = {0.0, 0.0, 0.0, 0.0};
        for (int q = by_wave ? lane : 0; q < P; q += by_wave ? 64 : 1)
            for (int k = 0; k < 4; ++k) v[k] += p[4 * q + k];
        if (by_wave) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1)
                for (int k = 0; k < 4; ++k) v[k] += __shfl_down(v[k], off);
            if (lane > 0) continue;
        }
        for (int k = 0; k < 4; ++k) {
            a.grain_out[4 * (int64_t)g + k] = v[k];
            t[k] += v[k];
        }
    }
    block_sum<B>(t);
    if (threadIdx.x == 0) system_out(a, s, t, moments, reset);
}

// a thread per system: batches of isolated grains (one grain each, of few parts).  A
// moment sample of 64 systems of 2816 sites takes 16.8 us with it, 4096 of 512 sites
// 30.6 (19.2 and 34.5 with a wavefront per system and branches between the loads)
__global__ __launch_bounds__(64) void k_reduce_isolated(RedArgs a, int moments, int reset)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= a.n_sys) return;
    double t[4] = {0.0, 0.0, 0.0, 0.0};
    if (a.sys[s].n_grains > 0) {
        const int64_t g = a.sys[s].grain_base;
        const double *p = a.part + 4 * g * a.n_parts;
        for (int q = 0; q < a.n_parts; ++q)
            for (int k = 0; k < 4; ++k) t[k] += p[4 * q + k];
        for (int k = 0; k < 4; ++k) a.grain_out[4 * g + k] = t[k];
    }
    system_out(a, s, t, moments, reset);
}

int launch_reduce_systems(const RedArgs &a, int moments, int reset, void *stream)
{
    if (a.n_sys == 0) return 0;
    const int threads = a.n_parts > kPartsThread ? 64 * a.max_grains : a.max_grains;
    if (a.max_grains <= 1 && a.n_parts <= kPartsThread)
        hipLaunchKernelGGL(k_reduce_isolated, dim3((a.n_sys + 63) / 64), dim3(64), 0, (hipStream_t)stream, a,
                           moments, reset);
    else if (threads <= 64)
        hipLaunchKernelGGL(k_reduce_systems<64>, dim3(a.n_sys), dim3(64), 0, (hipStream_t)stream, a, moments,
                           reset);
    else
        hipLaunchKernelGGL(k_reduce_systems<kSumBlock>, dim3(a.n_sys), dim3(kSumBlock), 0, (hipStream_t)stream,
                           a, moments, reset);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// The tiles' partial energies of a system, one workgroup per system: thread
// t adds tiles t, t + B, ... in order, then the workgroup its threads
// in a fixed tree (the same FP64 result every run).  One thread walking the
// tiles was a chain of dependent loads and adds: 1147 us for the 10 313 tiles
// of a 400x200x33 window, 13 us this way.
template <int B>
__global__ __launch_bounds__(B) void k_energy_finish(const double *partial, const SysDev *sys, double *out)
{
    const int s = blockIdx.x;
    const int b0 = sys[s].tile_base, b1 = b0 + sys[s].n_tiles;
    double t[3] = {0.0, 0.0, 0.0};
    for (int b = b0 + (int)threadIdx.x; b < b1; b += B)
        for (int k = 0; k < 3; ++k) t[k] += partial[3 * (int64_t)b + k];
    block_sum<B>(t);
    if (threadIdx.x == 0) {
        for (int k = 0; k < 3; ++k) out[4 * (int64_t)s + k] = t[k];
        out[4 * (int64_t)s + 3] = (t[0] + t[1]) + t[2];
    }
}

// a thread per system, batches of small systems: 4096 of 512 sites 91 us a call with a
// workgroup of 1024 threads each, 69 with a wavefront each, 65 so
__global__ __launch_bounds__(64) void k_energy_finish_few(const double *partial, const SysDev *sys,
                                                          int n_sys, double *out)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n_sys) return;
    const int b0 = sys[s].tile_base, b1 = b0 + sys[s].n_tiles;
    double t[3] = {0.0, 0.0, 0.0};
    for (int b = b0; b < b1; ++b)
        for (int k = 0; k < 3; ++k) t[k] += partial[3 * (int64_t)b + k];
    for (int k = 0; k < 3; ++k) out[4 * (int64_t)s + k] = t[k];
    out[4 * (int64_t)s + 3] = (t[0] + t[1]) + t[2];
}

int launch_energy_finish(const double *partial, const SysDev *sys, int n_sys, int max_tiles,
                         double *sys_out, void *stream)
{
    if (max_tiles <= 8)
        hipLaunchKernelGGL(k_energy_finish_few, dim3((n_sys + 63) / 64), dim3(64), 0, (hipStream_t)stream,
                           partial, sys, n_sys, sys_out);
    else if (max_tiles <= 64)  // one wavefront covers them: 512 systems of 2816 sites 50.5 -> 47.5 us a call
        hipLaunchKernelGGL(k_energy_finish<64>, dim3(n_sys), dim3(64), 0, (hipStream_t)stream, partial, sys,
                           sys_out);
    else
        hipLaunchKernelGGL(k_energy_finish<kSumBlock>, dim3(n_sys), dim3(kSumBlock), 0, (hipStream_t)stream,
                           partial, sys, sys_out);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// ---------------------------------------------------------------- transfer
// Eq. 6 read forwards (Sec. II).  A workgroup takes kCgX consecutive coarse
// cells (i, j) of one layer k, i fastest (neighbouring cells along x, or
// along y when the columns hold fewer than kCgX cells, as a strip of one
// coarse column does); thread (tx, tz) sums, for its cell, the lattice rows
// tz, tz + kCgZ, ... of the cell (rows numbered y fastest, each row's sites
// contiguous), then thread tz = 0 adds the kCgZ partial sums in order: the
// same FP64 result every run.  Non-magnetic sites hold S = 0, so only the
// count looks at the label and the loads of a row do not wait on it.
constexpr int kCgX = 32, kCgZ = 8;

// face (strips one coarse column wide): not the sums but their directions, as
// the x-face neighbours of a region (zero where a cell has no magnetic site)
template <typename T>
__device__ __forceinline__ void coarse_grain_block(const TransferArgs &a, int bx, int by,
                                                   double *face = nullptr)
{
    const int tx = threadIdx.x % kCgX, tz = threadIdx.x / kCgX;
    const int ij = bx * kCgX + tx;  // cell i + ncx j of layer k
    const bool live = ij < a.ncx * a.ncy;
    const int j = ij / a.ncx, i = ij - j * a.ncx, k = by;
    const int jk = j + a.ncy * k;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    if (live) {
        const int xb = a.x0 + i * a.cx, yb = j * a.cy, zb = k * a.cz;
        const int wx = min(a.cx, a.x0 + a.ncols - xb), wy = min(a.cy, a.d.ny - yb),
                  wz = min(a.cz, a.d.nz - zb);
        const T *S = (const T *)a.S[0];
        const int nq = a.per * wx;
        for (int r = tz; r < wy * wz; r += kCgZ) {
            const int zz = r / wy, yy = r - zz * wy;
            const int64_t row =
                a.d.base + a.per * ((int64_t)xb + (int64_t)a.d.sx *
                                                      ((yb + yy) + (int64_t)a.d.ny * (zb + zz)));
            for (int q = 0; q < nq; ++q) {
                const int64_t g = row + q;
                acc[0] += (double)S[g];
                acc[1] += (double)S[a.ncs + g];
                acc[2] += (double)S[2 * a.ncs + g];
                acc[3] += a.label[g] != kNoGrain ? 1.0 : 0.0;
            }
        }
    }
    __shared__ double red[4][kCgZ][kCgX];
    for (int m = 0; m < 4; ++m) red[m][tz][tx] = acc[m];
    __syncthreads();
    if (tz == 0 && live) {
        const int64_t c = i + (int64_t)a.ncx * jk;
        double t[4];
        for (int m = 0; m < 4; ++m) {
            t[m] = red[m][0][tx];
            for (int z = 1; z < kCgZ; ++z) t[m] += red[m][z][tx];
        }
        if (face) {
            const double r = sqrt((t[0] * t[0] + t[1] * t[1]) + t[2] * t[2]);
            for (int m = 0; m < 3; ++m) face[3 * c + m] = r > 0.0 ? t[m] / r : 0.0;
        } else {
            for (int m = 0; m < 4; ++m) a.out[4 * c + m] = t[m];
        }
    }
}

template <typename T>
__global__ __launch_bounds__(kCgX * kCgZ) void k_coarse_grain(TransferArgs a)
{
    coarse_grain_block<T>(a, blockIdx.x, blockIdx.y);
}

int launch_coarse_grain(const TransferArgs &a, void *stream)
{
    if (a.ncell == 0) return 0;
    const int ncz = a.ncell / (a.ncx * a.ncy);
    const dim3 grid((a.ncx * a.ncy + kCgX - 1) / kCgX, ncz);
    if (a.prec == ASD_FP64)
        hipLaunchKernelGGL(k_coarse_grain<double>, grid, dim3(kCgX * kCgZ), 0, (hipStream_t)stream,
                           a);
    else
        hipLaunchKernelGGL(k_coarse_grain<float>, grid, dim3(kCgX * kCgZ), 0, (hipStream_t)stream,
                           a);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Widest cone of the inverse transfer (Sec. II), as printed: (5 pi / 9)
// sqrt(1 - sqrt(1 + 6 (m - 1) / 5)) with m clamped to [1/6, 1].
__device__ __forceinline__ double cone_theta_max(double m)
{
    if (m > 1.0) m = 1.0;
    if (m < 1.0 / 6.0) m = 1.0 / 6.0;
    double t = 1.0 + (6.0 * (m - 1.0)) / 5.0;
    if (t < 0.0) t = 0.0;
    return 1.7453292519943295 * sqrt(1.0 - sqrt(t));
}

// Eq. 6 read backwards (Sec. II): each magnetic site of the columns takes a
// spin in the cone around its coarse cell's reduced magnetisation m: polar
// angle uniform on [0, theta_max] (the printed reading), or cos theta
// uniform on [2 m - 1, 1] (the cap reading, whose mean cos theta is m);
// azimuth uniform, measured in the orthonormal basis of Duff et al. (JCGT
// 2017) around the cell direction.  FP64 throughout; both spin buffers
// receive the result.
template <typename T>
__device__ __forceinline__ void cone_column_site(const TransferArgs &a, int64_t t,
                                                 const RegionFace *region = nullptr)
{
    const int64_t n = (int64_t)a.per * a.ncols * a.d.ny * a.d.nz;
    if (t >= n) return;
    const int s = (int)(t % a.per);
    int64_t r = t / a.per;
    const int xx = (int)(r % a.ncols);
    r /= a.ncols;
    const int y = (int)(r % a.d.ny), z = (int)(r / a.d.ny);
    const int64_t site = a.per * ((int64_t)(a.x0 + xx) + (int64_t)a.d.sx * (y + (int64_t)a.d.ny * z)) + s;
    const int64_t g = a.d.base + site;
    if (a.label[g] == kNoGrain) return;
    const int c = xx / a.cx + a.ncx * (y / a.cy + a.ncy * (z / a.cz));
    double mx, my, mz;
    if (region) {  // the region's cell beside coarse cell c
        const int64_t q = region->col + (int64_t)region->nx * c;
        mx = region->at(q, 0);
        my = region->at(q, 1);
        mz = region->at(q, 2);
    } else {
        mx = a.mcell[3 * (int64_t)c];
        my = a.mcell[3 * (int64_t)c + 1];
        mz = a.mcell[3 * (int64_t)c + 2];
    }
    const double m = sqrt((mx * mx + my * my) + mz * mz);
    double nx = 0.0, ny = 0.0, nz = 1.0;
    if (m > 0.0) {
        nx = mx / m;
        ny = my / m;
        nz = mz / m;
    }
    if (a.exact) {  // the coarse cell's direction itself
        T *S0 = (T *)a.S[0], *S1 = (T *)a.S[1];
        const T v[3] = {(T)nx, (T)ny, (T)nz};
        for (int k = 0; k < 3; ++k) {
            S0[k * a.ncs + g] = v[k];
            S1[k * a.ncs + g] = v[k];
        }
        return;
    }
    const Words4 w = philox4x32(a.rounds, a.k0, a.k1, (uint32_t)site, a.step, a.d.sys_id, 1u);
    const double TWO_M32 = 2.3283064365386962890625e-10;
    const double u1 = ((double)w.w0 + 0.5) * TWO_M32;
    const double u2 = (double)w.w1 * TWO_M32;
    double st, ct, sp, cp;
    if (a.cap) {
        const double mc = m > 1.0 ? 1.0 : m;
        ct = 1.0 - u1 * (2.0 - 2.0 * mc);
        st = sqrt((1.0 - ct) * (1.0 + ct));
    } else {
        const double th = u1 * cone_theta_max(m);
        f64::sincos2pi(th / 6.283185307179586, st, ct);
    }
    f64::sincos2pi(u2, sp, cp);
    const double sg = nz >= 0.0 ? 1.0 : -1.0;
    const double aa = -1.0 / (sg + nz);
    const double b = (nx * ny) * aa;
    const double b1x = 1.0 + ((sg * nx) * nx) * aa, b1y = sg * b, b1z = -sg * nx;
    const double b2x = b, b2y = sg + (ny * ny) * aa, b2z = -ny;
    const double ex = st * cp, ey = st * sp;
    double vx = (ex * b1x + ey * b2x) + ct * nx;
    double vy = (ex * b1y + ey * b2y) + ct * ny;
    double vz = (ex * b1z + ey * b2z) + ct * nz;
    const double nn = sqrt((vx * vx + vy * vy) + vz * vz);
    vx = vx / nn;
    vy = vy / nn;
    vz = vz / nn;
    for (int b2 = 0; b2 < 2; ++b2) {
        T *S = (T *)a.S[b2];
        S[g] = (T)vx;
        S[a.ncs + g] = (T)vy;
        S[2 * a.ncs + g] = (T)vz;
    }
}

template <typename T>
__global__ void k_cone_columns(TransferArgs a)
{
    cone_column_site<T>(a, (int64_t)blockIdx.x * blockDim.x + threadIdx.x);
}

// Everything that crosses the two x faces of a multiscale window before a coupled
// step, in one launch: the directions of the window's first and last coarse
// column into the regions' face neighbours, and the regions' boundary cells into
// the frozen columns just outside the window (exact directions).  All four read
// the state at the start of the step and write what the others do not read.
// Bound by the launches: as four kernels (sums, their directions, the regions'
// faces, the columns) these took 19 us of a step with its gaps.
template <typename T>
__global__ __launch_bounds__(kCgX * kCgZ) void k_window_faces(WindowFaces f)
{
    int b = blockIdx.x;
    const int cg = f.gx * f.layers;  // blocks per strip
    if (b < 2 * cg) {
        const int side = b < cg ? 0 : 1;
        b -= side * cg;
        const int k = b / f.gx;
        coarse_grain_block<T>(f.strip[side], b - k * f.gx, k, f.region[side].ghost);
        return;
    }
    b -= 2 * cg;
    const int side = b < f.col_blocks ? 0 : 1;
    b -= side * f.col_blocks;
    cone_column_site<T>(f.cols[side], (int64_t)b * blockDim.x + threadIdx.x, &f.region[side]);
}

int launch_window_faces(WindowFaces &f, void *stream)
{
    const TransferArgs &a = f.strip[0], &c = f.cols[0];
    if (a.ncx != 1 || f.strip[1].ncx != 1 || a.ncell != f.strip[1].ncell || a.prec != f.strip[1].prec)
        return -1;
    const int64_t n = (int64_t)c.per * c.ncols * c.d.ny * c.d.nz;
    const int threads = kCgX * kCgZ;
    f.gx = (a.ncy + kCgX - 1) / kCgX;
    f.layers = a.ncell / a.ncy;
    const int64_t cb = (n + threads - 1) / threads, grid = 2 * ((int64_t)f.gx * f.layers + cb);
    if (grid > INT32_MAX) return -1;
    f.col_blocks = (int)cb;
    if (a.prec == ASD_FP64)
        hipLaunchKernelGGL(k_window_faces<double>, dim3((unsigned)grid), dim3(threads), 0,
                           (hipStream_t)stream, f);
    else
        hipLaunchKernelGGL(k_window_faces<float>, dim3((unsigned)grid), dim3(threads), 0,
                           (hipStream_t)stream, f);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_cone_columns(const TransferArgs &a, void *stream)
{
    const int64_t n = (int64_t)a.per * a.ncols * a.d.ny * a.d.nz;
    if (n == 0) return 0;
    const int64_t blocks = (n + 255) / 256;
    if (a.prec == ASD_FP64)
        hipLaunchKernelGGL(k_cone_columns<double>, dim3((unsigned)blocks), dim3(256), 0,
                           (hipStream_t)stream, a);
    else
        hipLaunchKernelGGL(k_cone_columns<float>, dim3((unsigned)blocks), dim3(256), 0,
                           (hipStream_t)stream, a);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace asd

"""The one-launch RK4 step of a micromagnetic region against the oracle, at the
edges of its tiles and of the meshes it takes."""
import numpy as np
import pytest

from paper_2502_02236_amd import asd as A
from test_gpu_mm import SPOT, gpu, make_pair, random_m  # noqa: F401 (gpu: the module's fixture)

pytestmark = pytest.mark.gpu

STILL = dict(B=(0.1, 0.0, -0.8), T_amb=300.0)
LOCKED = dict(B=(0.0, 0.0, -0.8), spot=A.ASD_SPOT_LOCKED, x0=9e-9, y0=6e-9, **SPOT)


# one column short of a tile, a full one, one more; one plane and the most a
# tile takes (16), one more (a launch per stage); periodic axes shorter than the
# tile's surroundings; a mesh of many tiles
@pytest.mark.parametrize("n,per,drive", [
    ((4, 5, 16), (0, 0, 0), STILL), ((6, 11, 16), (1, 1, 1), LOCKED), ((7, 5, 17), (0, 0, 1), STILL),
    ((13, 6, 13), (0, 1, 0), LOCKED), ((9, 17, 10), (1, 0, 1), STILL), ((11, 10, 8), (0, 0, 0), LOCKED),
    ((2, 3, 8), (1, 1, 0), STILL), ((33, 15, 4), (1, 0, 0), LOCKED), ((27, 53, 2), (0, 0, 0), STILL),
    ((1, 1, 1), (1, 1, 1), STILL), ((160, 70, 3), (0, 1, 0), LOCKED),
], ids=lambda v: str(v).replace(" ", "") if isinstance(v, tuple) else None)
@pytest.mark.parametrize("steps,graph", [(1, 0), (2, 0), (7, 3), (8, 4)], ids=lambda v: str(v))
def test_one_launch_step_is_bit_identical(n, per, drive, steps, graph):
    g, o = make_pair(n, (1e-9, 1.1e-9, 2e-9), per, A.ASD_FP64, drive, graph_steps=graph)
    m = random_m(g.n, 11)
    g.set_m(m)
    for _ in range(2):
        g.step(steps)
    ref = o.rk4(m, 0, 2 * steps)
    got = g.get_m()
    assert np.array_equal(got, ref), float(np.max(np.abs(got - ref)))
    g.close()


def test_one_launch_step_couples_through_the_faces():
    """Neighbours across both x faces, one of them with empty cells."""
    n, steps = (13, 9, 5), 5
    g, o = make_pair(n, (1e-9, 1e-9, 2e-9), (0, 0, 0), A.ASD_FP64, STILL)
    torch = g.torch
    m = random_m(g.n, 4)
    g.set_m(m)
    for face in (0, 1):
        d = random_m(n[1] * n[2], 7 + face).T.copy()
        if face:
            d[::4] = 0.0
        vec = torch.as_tensor(d, device="cuda").contiguous()
        torch.cuda.synchronize()
        A._mm_check(A.lib().asd_mm_set_face(g.h, face, vec.data_ptr(), 3), g.h)
        g.stream.synchronize()
        r = np.sqrt((d[:, 0] * d[:, 0] + d[:, 1] * d[:, 1]) + d[:, 2] * d[:, 2])
        o.set_ghost(face, np.where(r[:, None] > 0, d / np.where(r > 0, r, 1.0)[:, None], 0.0))
    g.step(steps)
    assert np.array_equal(g.get_m(), o.rk4(m, 0, steps))
    g.close()

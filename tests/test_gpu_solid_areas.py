"""Masks of large solid areas: work-groups whose region is solid throughout leave
at once.  Every sweep against the FP64 oracle (relative L2 1e-12 in FP64; in FP32
1e-5 on fields, 1e-4 on derivatives), on fluid that begins and ends beside the
edges of segments and regions, with exact zeros on the solid nodes of buffers
that held NaN."""
import numpy as np
import pytest

from paper_1908_03876_amd import inputs as I
from tests.gpu_util import rel_l2
from tests.test_gpu_parity import TOL, _ragged, _torch_dtype
from tests.test_gpu_sweeps import SCHEMES, _directions, _oracle, _sweeps

pytestmark = pytest.mark.gpu

# (nx, ny): steps
SIZES = {(390, 331): 11, (130, 520): 6, (1100, 700): 5}


def _areas(nx, ny):
    """Solid but for a block that ends at column 127 or 128, a channel of one node
    along a row and one along a column, and the last nodes of a corner."""
    s = np.ones((ny, nx), np.uint8)
    s[ny // 3:ny // 3 + 41, 65:127 + nx % 2] = 0
    s[ny // 3 + 5, :] = 0
    s[:, 100] = 0
    s[-3:, -2:] = 0
    return s


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("periodic", [False, True])
@pytest.mark.parametrize("scheme", sorted(SCHEMES))
@pytest.mark.parametrize("size", sorted(SIZES), ids=lambda s: "x".join(map(str, s)))
def test_large_solid_areas(size, scheme, periodic, prec):
    source, species = SCHEMES[scheme]
    p = _ragged(size[0], *size, SIZES[size], periodic, True).copy(solid=_areas(*size))
    for a in (p.u0, p.v0, p.control, p.u_target):
        a[p.solid != 0] = 0.0
    if species == 3:
        p = I.with_repellent(p)
    elif source > 1:
        p = I.slow_reaction(p, 0.1).copy(source_term=source)
    print(f"case {size} {scheme} {periodic} {prec}", flush=True)
    dirs = _directions(p)
    ref = _oracle(p, dirs)
    ftol, gtol = TOL[prec]
    for ckpt in (-1, 2):
        got = _sweeps(p, _torch_dtype(prec), ckpt, dirs)
        for k, want in ref.items():
            assert rel_l2(got[k], want, p.fluid) <= (ftol if k in ("uN", "vN") else gtol), k
            assert (got[k][p.solid != 0] == 0.0).all(), k

"""Every sweep of a lattice (forward, AMRT with the initial sensitivities,
tangent, continuous adjoint) in every shape that a launch can take, against the
FP64 oracle: relative L2 1e-12 in FP64; in FP32 1e-5 on fields, 1e-4 on
derivatives.  Checkpointed at every step the same sweeps run in rows of nodes,
one step a launch, and give the same bits."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1908_03876_amd import inputs as I
from tests.gpu_util import rel_l2
from tests.test_gpu_parity import TOL, _ragged, _torch_dtype

pytestmark = pytest.mark.gpu

SCHEMES = {"first": (1, 2), "explicit": (2, 2), "implicit": (3, 2), "three": (1, 3)}
KINDS = {"periodic": (True, False), "masked": (False, True), "walls": (False, False)}
# (nx, ny): steps, and the regions of a store-all sweep by precision
SIZES = {(70, 45): (9, {"f32": (16, 16), "f64": (16, 16)}),
         (257, 7): (1, {"f32": (256, 1), "f64": (256, 1)}),
         (161, 160): (9, {"f32": (64, 16), "f64": (32, 16)}),
         (20, 2100): (5, {"f32": (32, 32), "f64": (32, 16)}),  # single steps in regions too
         (32768, 2): (4, {"f32": (256, 1), "f64": (256, 1)}),
         (32768, 7): (6, {"f32": (64, 16), "f64": (32, 16)}),
         (386, 390): (11, {"f32": (32, 32), "f64": (32, 16)})}


def _problem(size, steps, scheme, kind):
    source, species = SCHEMES[scheme]
    p = _ragged(size[0] * 1000 + size[1], *size, steps, *KINDS[kind])
    if species == 3:
        return I.with_repellent(p)
    return p if source == 1 else I.slow_reaction(p, 0.1).copy(source_term=source)


def _directions(p):
    rng = np.random.default_rng(8)
    return [s * rng.standard_normal((p.ny, p.nx)) * p.fluid for s in (1.0, 1.0, 1.0, 0.1, 0.1)]


def _sweeps(p, dtype, ckpt, dirs, shape=None):
    import torch
    from paper_1908_03876_amd import abi
    from paper_1908_03876_amd.solver import DeviceProblem, Tape
    dp = DeviceProblem(p, dtype=dtype)
    if shape is not None:
        s = abi.mrt_step_plan(dp.struct, p.nsteps, p.nsteps)
        if shape == (32, 32) and p.nspecies == 3:
            shape = (32, 16)
        if shape == (64, 16) and p.nspecies == 3:
            shape = (32, 16)
        assert (s.width, s.height) == shape
    tape = Tape(dp, ckpt)
    a, b, dc, du0, dv0 = (dp.field(d) for d in dirs)
    fields = (dp.u0, dp.v0, dp.control)
    uN, vN, au0, av0, duN, dvN = (torch.full_like(dp.u0, float("nan")) for _ in range(6))
    gacc = torch.full_like(dp.u0, float("nan"), dtype=torch.float64)
    abi.mrt_forward(dp.struct, tape.handle, *fields, None, uN, vN)
    abi.amrt_adjoint(dp.struct, tape.handle, *fields, a, b, gacc, au0, av0)
    abi.mrt_tlm(dp.struct, tape.handle, *fields, dc, du0, dv0, duN, dvN)
    out = {"uN": uN, "vN": vN, "g": gacc, "au0": au0, "av0": av0, "duN": duN, "dvN": dvN}
    out = {k: dp.host(t) for k, t in out.items()}
    if p.nspecies == 2 and p.source_term == 1:
        gacc.fill_(float("nan"))
        abi.mrt_cadjoint(dp.struct, tape.handle, *fields, a, gacc)
        out["cg"] = dp.host(gacc)
    tape.close()
    return out


def _oracle(p, dirs):
    a, b, dc, du0, dv0 = dirs
    f = O.forward(p)
    out = {"uN": f["uN"], "vN": f["vN"]}
    out["g"], out["au0"], out["av0"] = O.adjoint(p, a, b)
    out["duN"], out["dvN"] = O.tlm(p, dc=dc, du0=du0, dv0=dv0)
    if p.nspecies == 2 and p.source_term == 1:
        out["cg"] = O.cadjoint(p, a)
    return out


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("scheme", sorted(SCHEMES))
@pytest.mark.parametrize("size", sorted(SIZES), ids=lambda s: "x".join(map(str, s)))
def test_sweeps(size, scheme, kind, prec):
    steps, shapes = SIZES[size]
    p = _problem(size, steps, scheme, kind)
    print(f"case {size} {scheme} {kind} {prec}", flush=True)
    dirs = _directions(p)
    ref = _oracle(p, dirs)
    ftol, gtol = TOL[prec]
    got = _sweeps(p, _torch_dtype(prec), -1, dirs, shapes[prec])
    rows = _sweeps(p, _torch_dtype(prec), 1, dirs)
    for k, want in ref.items():
        assert rel_l2(got[k], want, p.fluid) <= (ftol if k in ("uN", "vN") else gtol), k
        assert np.array_equal(got[k], rows[k]), k
        if p.solid is not None:
            assert (got[k][p.solid != 0] == 0.0).all(), k

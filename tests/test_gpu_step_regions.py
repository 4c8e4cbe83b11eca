"""Several time steps per launch: lattice sizes at the edges of the regions
that a work-group owns, and step counts that leave uneven launches, against
the FP64 oracle (relative L2 1e-12 in FP64; 1e-5 on fields and 1e-4 on the
gradient in FP32)."""
import pytest

from oracle import oracle as O
from paper_1908_03876_amd import inputs as I
from tests.gpu_util import device_gradient, rel_l2
from tests.test_gpu_parity import TOL, _ragged, _torch_dtype

pytestmark = pytest.mark.gpu

# (nx, ny, steps): one region, its last column or row, one node more; lattices
# narrower or lower than a region; the widths that 64-, 32- and 16-node regions
# own with 4 to 9 steps; both sides of the lines between the plans
SIZES = [(6, 6, 5), (7, 13, 6), (16, 16, 9), (17, 5, 11), (3, 40, 4), (61, 2, 7),
         (160, 160, 11), (161, 160, 12), (54, 498, 7), (1200, 23, 6),
         (384, 384, 7), (386, 384, 9), (58 * 7, 390, 5), (26 * 15 + 1, 401, 4),
         (16 * 16, 16 * 16, 18), (16 * 16 + 1, 16 * 16, 9), (24 * 22 + 1, 24 * 23, 10),
         (24 * 30, 650, 10)]
KINDS = {"periodic": (True, False), "masked": (False, True), "walls": (False, False),
         "masked_periodic": (True, True)}


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("size", SIZES, ids=lambda s: "x".join(map(str, s)))
def test_regions_match_oracle(size, kind, prec):
    nx, ny, steps = size
    p = _ragged(nx * 1000 + ny, nx, ny, steps, *KINDS[kind])
    print(f"case {size} {kind} {prec}", flush=True)
    ref = O.cost_gradient(p)
    ftol, gtol = TOL[prec]
    f = p.fluid
    for ckpt in (-1, 3):
        r = device_gradient(p, _torch_dtype(prec), ckpt_every=ckpt)
        assert rel_l2(r["uN"], ref["uN"], f) <= ftol
        assert rel_l2(r["grad"], ref["grad"], f) <= gtol


@pytest.mark.parametrize("source,species", [(2, 2), (3, 2), (1, 3)])
@pytest.mark.parametrize("size", [(17, 5, 11), (161, 160, 12), (391, 401, 5)],
                         ids=lambda s: "x".join(map(str, s)))
def test_regions_of_the_other_schemes(size, source, species):
    nx, ny, steps = size
    p = _ragged(nx * 1000 + ny, nx, ny, steps, False, True)
    p = I.with_repellent(p) if species == 3 else I.slow_reaction(p, 0.1).copy(source_term=source)
    print(f"case {size} source {source} species {species}", flush=True)
    ref = O.cost_gradient(p)
    r = device_gradient(p, _torch_dtype("f64"), ckpt_every=4)
    assert rel_l2(r["uN"], ref["uN"], p.fluid) <= 1e-12
    assert rel_l2(r["grad"], ref["grad"], p.fluid) <= 1e-12


@pytest.mark.parametrize("source", [2, 3])
@pytest.mark.parametrize("size", [(256, 257, 9), (529, 552, 10)],
                         ids=lambda s: "x".join(map(str, s)))
def test_square_regions_of_the_other_schemes(size, source):
    nx, ny, steps = size
    p = I.slow_reaction(_ragged(nx * 1000 + ny, nx, ny, steps, False, True), 0.1).copy(
        source_term=source)
    print(f"case {size} source {source}", flush=True)
    ref = O.cost_gradient(p)
    ftol, gtol = TOL["f32"]
    r = device_gradient(p, _torch_dtype("f32"))
    assert rel_l2(r["uN"], ref["uN"], p.fluid) <= ftol
    assert rel_l2(r["grad"], ref["grad"], p.fluid) <= gtol


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("source,ckpt", [(2, 4), (2, -1), (1, 4)])
def test_initial_sensitivities_on_solid_blocks(source, ckpt, prec):
    """dJ/du0 and dJ/dv0 in buffers that held NaN: exact zeros on solid nodes,
    whole 64-node segments and frame rows of them included."""
    import torch
    from paper_1908_03876_amd import abi
    from paper_1908_03876_amd.solver import DeviceProblem, GradientIteration
    p = _ragged(77, 200, 23, 9, False, True)
    p.solid[[0, -1], :] = p.solid[5:12, 64:192] = 1
    for a in (p.u0, p.v0, p.control, p.u_target):
        a[p.solid != 0] = 0.0
    p = I.slow_reaction(p, 0.1).copy(source_term=source)
    print(f"source {source} ckpt {ckpt} {prec}", flush=True)
    seed = (O.forward(p)["uN"] - p.u_target) * p.fluid
    _, want_u0, want_v0 = O.adjoint(p, seed)
    dp = DeviceProblem(p, dtype=_torch_dtype(prec))
    it = GradientIteration(dp, ckpt_every=ckpt)
    it.gradient()
    it.gacc.fill_(float("nan"))
    au0, av0 = (torch.full_like(it.uN, float("nan")) for _ in range(2))
    abi.amrt_adjoint(dp.struct, it.tape.handle, dp.u0, dp.v0, dp.control, it.seed, None, it.gacc,
                     au0, av0)
    gtol = TOL[prec][1]
    for dev, want in ((au0, want_u0), (av0, want_v0)):
        dev = dp.host(dev)
        assert (dev[p.solid != 0] == 0.0).all()
        assert rel_l2(dev, want, p.fluid) <= gtol
    assert (dp.host(it.gacc)[p.solid != 0] == 0.0).all()
    it.close()


@pytest.mark.parametrize("steps", [2, 4, 7])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_sensitivities_over_the_seeds(steps, prec):
    """dJ/du0, dJ/dv0 (and, in FP64, the continuous adjoint's integral) written
    over the seeds of a sweep so short that one launch could take all of it: the
    bits of separate buffers."""
    from paper_1908_03876_amd import abi
    from paper_1908_03876_amd.solver import DeviceProblem, GradientIteration
    p = _ragged(78, 300, 333, steps, False, True)
    print(f"{steps} steps {prec}", flush=True)
    dp = DeviceProblem(p, dtype=_torch_dtype(prec))
    it = GradientIteration(dp)
    it.gradient()
    fields = (dp.u0, dp.v0, dp.control)
    su, sv = it.seed.clone(), dp.field(p.u0)
    au0, av0 = dp.empty_field(), dp.empty_field()
    abi.amrt_adjoint(dp.struct, it.tape.handle, *fields, su, sv, it.gacc, au0, av0)
    abi.amrt_adjoint(dp.struct, it.tape.handle, *fields, su, sv, it.gacc, su, sv)
    assert (dp.host(su) == dp.host(au0)).all() and (dp.host(sv) == dp.host(av0)).all()
    if prec == "f64":
        su = it.seed.clone()
        abi.mrt_cadjoint(dp.struct, it.tape.handle, *fields, it.seed, it.gacc)
        abi.mrt_cadjoint(dp.struct, it.tape.handle, *fields, su, su)
        assert (dp.host(su) == dp.host(it.gacc)).all()
    it.close()

"""Planes of more than 2^29 elements, where the byte offsets of the FP64 gradient
accumulator pass 4 GiB: a lattice of few nodes whose rows lie far apart gives
the bits that it gives with its rows close together."""
import pytest

from tests.test_gpu_parity import _ragged

pytestmark = pytest.mark.gpu


def _sweeps(p, dtype, ckpt, pitch, monkeypatch):
    import torch
    from paper_1908_03876_amd import abi, solver
    monkeypatch.setattr(solver, "padded_pitch", lambda nx, align=64: pitch)
    dp = solver.DeviceProblem(p, dtype=dtype)
    it = solver.GradientIteration(dp, ckpt_every=ckpt)
    out = {}
    try:
        if ckpt == 0:
            it.forward()
        else:
            it.gradient()
            out["gacc"], out["grad"] = dp.host(it.gacc), dp.host(it.grad)
            if p.nspecies == 2 and p.source_term == 1:
                abi.mrt_cadjoint(dp.struct, it.tape.handle, dp.u0, dp.v0, dp.control, it.seed,
                                 it.gacc)
                out["continuous"] = dp.host(it.gacc)
        out["uN"], out["vN"] = dp.host(it.uN), dp.host(it.vN)
    finally:
        it.close()
        del it, dp
        torch.cuda.empty_cache()
    return out


@pytest.mark.parametrize("nx,prec,ckpt", [(300, "f32", -1), (40, "f32", -1), (40, "f64", 0)])
def test_rows_far_apart(nx, prec, ckpt, monkeypatch):
    import torch
    ny, steps, pitch = 520, 4, 1 << 20
    elem = 4 if prec == "f32" else 8
    need = ny * pitch * (((72 + 3 * steps) if ckpt else 36) * elem + 8 + 8 * elem)
    if torch.cuda.mem_get_info()[0] < need + (4 << 30):
        pytest.skip("needs %d GB of device memory" % (need >> 30))
    p = _ragged(nx, nx, ny, steps, False, False)
    dtype = torch.float32 if prec == "f32" else torch.float64
    print(f"{nx} x {ny} {prec}", flush=True)
    near = _sweeps(p, dtype, ckpt, 512, monkeypatch)
    far = _sweeps(p, dtype, ckpt, pitch, monkeypatch)
    for k in near:
        assert (near[k] == far[k]).all(), k

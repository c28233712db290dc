"""Allen-Cahn launches on grids too small to fill the chip, whose z-chunks
are shorter than the largest (64, 32 or 256 planes, down to 4): fused and
limited runs bit-identical to one launch per step without them, and x_T bit
for bit and dx0 within 1e-12 (fp64) / 1e-5 (fp32) of the oracle. Depths sit on
both sides of whole chunks of 4, 8 and 16 planes.
"""
import numpy as np
import pytest

import oracle
import paper_2509_02197_amd as adst
from tests.gpu_util import NP_DTYPE, TOL, dev, gpu_vjp, rel, say

pytestmark = pytest.mark.gpu

AC, F64, F32 = adst.ADST_ALLENCAHN3D7, adst.ADST_F64, adst.ADST_F32


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    adst.lib()


@pytest.mark.parametrize("dtype,shape", [
    (F64, (4, 5, 7)), (F64, (5, 31, 65)), (F64, (9, 60, 130)), (F32, (17, 40, 61)),
    (F64, (33, 57, 121)), (F64, (40, 130, 250)), (F32, (70, 200, 190)), (F64, (131, 16, 64))])
@pytest.mark.parametrize("lim", [None, (-0.6, 0.7)])
def test_short_chunks(dtype, shape, lim):
    say(f"allen-cahn chunks dtype={dtype} shape={shape} lim={lim}")
    r = np.random.Generator(np.random.PCG64(61))
    inp = {"x0": r.uniform(-1.0, 1.0, shape).astype(NP_DTYPE[dtype]),
           "aux": r.standard_normal(shape).astype(NP_DTYPE[dtype])}
    T, budget = 11, 2 * inp["x0"].nbytes
    kw = dict(budget=budget, sched=adst.ADST_SCHED_BINOMIAL, lim=lim)
    a = gpu_vjp(AC, inp, T, adst.ADST_LOSS_DOT_W, **kw)
    b = gpu_vjp(AC, inp, T, adst.ADST_LOSS_DOT_W, flags=adst.ADST_NO_FUSE, **kw)
    assert np.array_equal(a["dx0"], b["dx0"]) and np.array_equal(a["xT"], b["xT"])
    dx0, _, xT, _ = oracle.vjp(AC, inp["x0"], steps=T, loss=adst.ADST_LOSS_DOT_W, aux=inp["aux"],
                               lim=lim)
    assert np.array_equal(a["xT"], xT)
    assert rel(a["dx0"], dx0) <= TOL[dtype]


def test_one_step_on_a_grid_of_four_workgroups_a_cu():
    """1024 tiles of 32 planes: f64 single steps keep them, f32 ones take 16."""
    r = np.random.Generator(np.random.PCG64(62))
    x = r.uniform(-1.0, 1.0, (33, 256, 1024))
    for a in (x[:32], x, x[:32].astype(np.float32)):
        for lim in (None, (-0.6, 0.7)):
            got = adst.forward(AC, dev(a), None, 1, lim=lim).cpu().numpy()
            assert np.array_equal(got, oracle.forward(AC, a, steps=1, lim=lim))

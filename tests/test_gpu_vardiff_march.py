"""The variable-coefficient register march (two forward steps a launch) at
the edges of its pieces, against one launch per step and the oracle, bit for
bit: strips of 248 (f32) or 124 (f64) columns, chunks of 6, 12, 24 and more
rows (a wide grid takes the longest), rows narrower than a block; and with
infinities and NaN.
"""
import numpy as np
import pytest

import oracle
import paper_2509_02197_amd as adst
from tests.gpu_util import NP_DTYPE, dev, gpu_vjp, say

pytestmark = pytest.mark.gpu

VD, F64, F32 = adst.ADST_VARDIFF2D9, adst.ADST_F64, adst.ADST_F32


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    adst.lib()


def draw(dtype, shape, seed):
    r = np.random.Generator(np.random.PCG64(seed))
    t = NP_DTYPE[dtype]
    return (r.uniform(0, 1, shape).astype(t), r.uniform(0.5, 1.5, shape).astype(t),
            r.standard_normal(shape).astype(t))


@pytest.mark.parametrize("dtype,shape", [
    (F64, (12, 123)), (F64, (13, 124)), (F64, (37, 125)), (F64, (100, 250)), (F64, (2, 373)),
    (F32, (61, 247)), (F32, (25, 248)), (F32, (90, 249)), (F32, (300, 2)), (F32, (1, 500)),
    (F32, (400, 5000))])
def test_two_steps(dtype, shape):
    say(f"vardiff march dtype={dtype} shape={shape}")
    x, K, aux = draw(dtype, shape, 91)
    for T in (2, 5):
        a = adst.forward(VD, dev(x), dev(K), T).cpu().numpy()
        assert np.array_equal(a, oracle.forward(VD, x, K=K, steps=T)), T
    kw = dict(budget=20 * x.nbytes, sched=adst.ADST_SCHED_STORE_ALL, want_dK=True)
    inp = {"x0": x, "K": K, "aux": aux}
    a = gpu_vjp(VD, inp, 9, adst.ADST_LOSS_SEED, **kw)
    b = gpu_vjp(VD, inp, 9, adst.ADST_LOSS_SEED, flags=adst.ADST_NO_FUSE, **kw)
    for k in ("dx0", "dK", "xT"):
        assert np.array_equal(a[k], b[k]), k


def test_values_that_are_not_finite():
    x, K, _ = draw(F64, (70, 260), 92)
    x[30, 100], x[0, 3], K[50, 259], x[69, 200] = np.nan, np.inf, np.inf, -np.inf
    a = adst.forward(VD, dev(x), dev(K), 2).cpu().numpy()
    b = adst.forward(VD, dev(x), dev(K), 2, flags=adst.ADST_NO_FUSE).cpu().numpy()
    assert np.array_equal(a, b, equal_nan=True)

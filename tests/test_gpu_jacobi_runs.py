"""Jacobi forward launches under the limiter, store-through runs and pairs of
adjoint steps that read state: several steps per launch, bit-identical to one
launch per step, x_T bit for bit and gradients (dL/dw among them) within 1e-12
(fp64) / 1e-5 (fp32) of the oracle. Step counts reach
every depth (2 to 6 steps, runs of 2 to 4 kept states); shapes sit around a
strip's columns (116 to 124, 240 to 248) and a chunk's rows (48, 12, 6).
"""
import numpy as np
import pytest

import oracle
import paper_2509_02197_amd as adst
from tests.gpu_util import NP_DTYPE, TOL, check_dw, dev, gpu_vjp, rel, say

pytestmark = pytest.mark.gpu

J, F64, F32 = adst.ADST_JACOBI2D5, adst.ADST_F64, adst.ADST_F32
LIM = (0.3, 0.7)
SHAPES = [(F64, (1, 1)), (F64, (3, 2)), (F64, (13, 120)), (F64, (61, 121)), (F64, (100, 367)),
          (F64, (1100, 1)), (F64, (1, 1030)), (F32, (400, 3)), (F32, (12, 245)), (F32, (110, 500)),
          (F32, (13, 760))]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    adst.lib()


@pytest.mark.parametrize("dtype,shape", SHAPES)
def test_limited_forward(dtype, shape):
    r = np.random.Generator(np.random.PCG64(81))
    x = r.uniform(0, 1, shape).astype(NP_DTYPE[dtype])
    for T in (2, 3, 4, 5, 6, 7, 14):
        say(f"jacobi limited forward dtype={dtype} shape={shape} T={T}")
        a = adst.forward(J, dev(x), None, T, lim=LIM).cpu().numpy()
        assert np.array_equal(a, oracle.forward(J, x, steps=T, lim=LIM)), T


def test_limited_forward_keeps_nan_and_clamps_infinities():
    r = np.random.Generator(np.random.PCG64(82))
    x = r.uniform(0, 1, (60, 130))
    x[20, 40], x[0, 5], x[33, 129], x[41, 90] = np.nan, np.inf, -np.inf, np.inf
    a = adst.forward(J, dev(x), None, 6, lim=LIM).cpu().numpy()
    b = adst.forward(J, dev(x), None, 6, lim=LIM, flags=adst.ADST_NO_FUSE).cpu().numpy()
    assert np.array_equal(a, b, equal_nan=True) and np.isnan(a).any()


@pytest.mark.parametrize("dtype,shape", SHAPES)
@pytest.mark.parametrize("name,opt", [("lim", {"lim": LIM}), ("dp", {"want_dparams": True})])
@pytest.mark.parametrize("T,slots,sched", [(9, 7, adst.ADST_SCHED_STORE_ALL),
                                           (23, 4, adst.ADST_SCHED_BINOMIAL),
                                           (17, 3, adst.ADST_SCHED_UNIFORM)])
def test_runs(dtype, shape, name, opt, T, slots, sched):
    say(f"jacobi runs dtype={dtype} shape={shape} {name} T={T} sched={sched}")
    r = np.random.Generator(np.random.PCG64(83))
    inp = {"x0": r.uniform(0, 1, shape).astype(NP_DTYPE[dtype]),
           "aux": r.standard_normal(shape).astype(NP_DTYPE[dtype])}
    kw = dict(budget=slots * inp["x0"].nbytes, sched=sched, **opt)
    a = gpu_vjp(J, inp, T, adst.ADST_LOSS_DOT_W, **kw)
    b = gpu_vjp(J, inp, T, adst.ADST_LOSS_DOT_W, flags=adst.ADST_NO_FUSE, **kw)
    assert a["info"]["fwd_kernels"] < b["info"]["fwd_kernels"] == b["info"]["fwd_steps_total"]
    # adjoint steps pair up: under the limiter in f32 on grids of more rows than
    # the two end chunks hold, with dL/dw in f32 only and where the last interior
    # strip of 248 columns ends before the last columns
    ny, nx = shape
    last = -(-nx // 248) - 2
    pairs = ((dtype == F64 or ny > 12) if name == "lim" else
             dtype == F32 and ny > 12 and last >= 1 and last * 248 + 252 <= nx - 2)
    assert (a["info"]["adj_kernels"] < T) == pairs and b["info"]["adj_kernels"] == T
    for key in ("dx0", "xT", "dparams"):
        if a[key] is not None:
            assert np.array_equal(a[key], b[key]), key
    dx0, _, xT, _, dp = oracle.vjp(J, inp["x0"], steps=T, loss=adst.ADST_LOSS_DOT_W,
                                   aux=inp["aux"], want_dp=True, lim=opt.get("lim"))
    assert np.array_equal(a["xT"], xT)
    assert rel(a["dx0"], dx0) <= TOL[dtype]
    if name == "dp":
        check_dw(J, inp, T, a["dparams"], dp, TOL[dtype])


@pytest.mark.parametrize("dtype,shape", [(F64, (700, 700)), (F64, (1400, 1403)),
                                         (F32, (2100, 2604))])
@pytest.mark.parametrize("opt", [{}, {"lim": LIM}, {"want_dparams": True}])
def test_chunk_lengths(dtype, shape, opt):
    """Interior chunks of 12, 24 and 48 rows: the bits of one launch per step."""
    r = np.random.Generator(np.random.PCG64(84))
    inp = {"x0": r.uniform(0, 1, shape).astype(NP_DTYPE[dtype]),
           "aux": r.standard_normal(shape).astype(NP_DTYPE[dtype])}
    kw = dict(budget=5 * inp["x0"].nbytes, sched=adst.ADST_SCHED_BINOMIAL, **opt)
    a = gpu_vjp(J, inp, 13, adst.ADST_LOSS_DOT_W, **kw)
    b = gpu_vjp(J, inp, 13, adst.ADST_LOSS_DOT_W, flags=adst.ADST_NO_FUSE, **kw)
    for key in ("dx0", "xT", "dparams"):
        if a[key] is not None:
            assert np.array_equal(a[key], b[key]), key

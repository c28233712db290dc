"""Rows that are no multiple of 16 bytes, and arrays that start between
16-byte boundaries: the 2-D kinds load and store 16-byte blocks at element
alignment, the block with a row's end from the row's last whole block.
x_T bit for bit, gradients within 1e-12 (fp64) / 1e-5 (fp32) of the oracle,
and every result the same bits as from aligned copies of the arrays.
"""
import numpy as np
import pytest

import oracle
import paper_2509_02197_amd as adst
from tests.gpu_util import NP_DTYPE, TOL, check_dw, rel, say

pytestmark = pytest.mark.gpu

J, VD = adst.ADST_JACOBI2D5, adst.ADST_VARDIFF2D9
F64, F32 = adst.ADST_F64, adst.ADST_F32


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    adst.lib()


def at_offset(a, off):
    """A copy of a on the device starting `off` elements into its buffer."""
    import torch
    if a is None:
        return None
    t = torch.full((a.size + off + 8,), float("nan"), dtype=torch.from_numpy(a).dtype,
                   device="cuda")
    v = t[off:off + a.size].view(a.shape)
    v.copy_(torch.from_numpy(a))
    return v


# rows of 1 to 3 values more than whole blocks, narrower than a block, one
# strip and several (124 or 248 columns, 240 to 256), the row's end in a
# strip's first and last blocks
SHAPES = [(F64, (40, 1)), (F64, (9, 125)), (F64, (70, 247)), (F64, (33, 501)), (F32, (30, 3)),
          (F32, (25, 5)), (F32, (61, 249)), (F32, (40, 254)), (F32, (90, 751)), (F32, (20, 1023)),
          # rows of whole blocks: aligned ones from the buffer's start, off the
          # 16-byte grid from its second element
          (F64, (33, 500)), (F64, (15, 2)), (F32, (40, 752)), (F32, (61, 248)), (F32, (12, 4))]
OPTS = [("plain", {}), ("dp", {"want_dparams": True}), ("lim", {"lim": (0.3, 0.7)})]


@pytest.mark.parametrize("dtype,shape", SHAPES)
@pytest.mark.parametrize("kind", [J, VD])
@pytest.mark.parametrize("name,opt", OPTS, ids=[o[0] for o in OPTS])
def test_rows_off_the_16_byte_grid(kind, dtype, shape, name, opt):
    say(f"unaligned kind={kind} dtype={dtype} shape={shape} {name}")
    r = np.random.Generator(np.random.PCG64(71))
    dt = NP_DTYPE[dtype]
    x = r.uniform(0, 1, shape).astype(dt)
    K = r.uniform(0.5, 1.5, shape).astype(dt) if kind == VD else None
    aux = r.standard_normal(shape).astype(dt)
    T, dK = 13, kind == VD
    outs = []
    for off in (0, 1):
        o = adst.vjp(kind, at_offset(x, off), at_offset(K, off), T, adst.ADST_LOSS_SEED,
                     at_offset(aux, off), 3 * x.nbytes, adst.ADST_SCHED_BINOMIAL, dK, **opt)
        outs.append({k: o[k].cpu().numpy() for k in ("dx0", "dK", "xT", "dparams")
                     if o[k] is not None})
    for k in outs[0]:
        assert np.array_equal(outs[0][k], outs[1][k]), k
    dx0, gK, xT, _, dp = oracle.vjp(kind, x, K=K, steps=T, loss=adst.ADST_LOSS_SEED, aux=aux,
                                    want_dK=dK, want_dp=True, lim=opt.get("lim"))
    assert np.array_equal(outs[0]["xT"], xT)
    assert rel(outs[0]["dx0"], dx0) <= TOL[dtype]
    if dK:
        assert rel(outs[0]["dK"], gK) <= TOL[dtype]
    if name == "dp":
        check_dw(kind, {"x0": x, "K": K, "aux": aux}, T, outs[0]["dparams"], dp, TOL[dtype])


@pytest.mark.parametrize("dtype,shape", [(F64, (2901, 2903)), (F64, (4101, 4103)),
                                         (F32, (4101, 4103)), (F32, (5801, 5803))])
def test_odd_rows_beyond_the_cache(dtype, shape):
    """States of 64 MiB and 128 MiB, from which the adjoints that read state
    take the non-temporal hint on odd rows: dL/dw asked for or not, steps fused
    or not, the same bits."""
    say(f"odd rows beyond the cache dtype={dtype} shape={shape}")
    import torch
    x = torch.rand(*shape, dtype=torch.float64 if dtype == F64 else torch.float32, device="cuda")
    aux = torch.randn_like(x)

    def run(**kw):
        return adst.vjp(J, x, None, 5, adst.ADST_LOSS_SEED, aux, 6 * x.nbytes,
                        adst.ADST_SCHED_STORE_ALL, **kw)
    plain, dp = run(), run(want_dparams=True)
    assert torch.equal(plain["dx0"], dp["dx0"])
    one = run(want_dparams=True, flags=adst.ADST_NO_FUSE)
    assert torch.equal(one["dparams"], dp["dparams"])
    a, b = run(lim=(0.3, 0.7)), run(lim=(0.3, 0.7), flags=adst.ADST_NO_FUSE)
    assert torch.equal(a["dx0"], b["dx0"]) and torch.equal(a["xT"], b["xT"])

"""The persistent launch of the in-place kind's sweeps (a workspace with
adst_sweep_workspace_bytes more than the plan's) against the oracle and
against the level launches (the plan's own workspace), bit for bit.

Shapes sit at the edges of the launch's pieces: strips of 128 (f64) or 256
(f32) columns that move one column per sweep, groups of 8 or 16 sweeps (four
or eight waves; the last grid has more than 256 workgroups of four, so takes
eight), 256 sweeps per launch, odd rows, grids without interior points.
"""
import numpy as np
import pytest

import oracle
import paper_2509_02197_amd as adst
from tests.gpu_util import NP_DTYPE, TOL, dev, rel, say

pytestmark = pytest.mark.gpu

GS = adst.ADST_GAUSSSEIDEL2D5
F64, F32 = adst.ADST_F64, adst.ADST_F32
SEED = adst.ADST_LOSS_SEED


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    adst.lib()


def run(dtype, x, aux, T, room, tail=None):
    """adst_vjp in a workspace of the plan's bytes and `room` more; `tail`
    (optional) is placed where the scratch would be and read as loss_aux."""
    import torch
    shape = x.shape
    prob = adst.make_problem(GS, dtype, (shape[1], shape[0], 1))
    need = adst.adst_plan(prob, T, 0, adst.ADST_SCHED_AUTO).workspace_bytes
    ws = torch.full((need + room,), 0x5a, dtype=torch.uint8, device="cuda")
    x0, g = dev(x), dev(aux)
    if tail is not None:
        g = ws[need:need + g.numel() * g.element_size()].view(g.dtype).view(shape)
        g.copy_(dev(tail))
    dx0, xT = torch.empty_like(x0), torch.empty_like(x0)
    L = torch.empty((), dtype=torch.float64, device="cuda")
    adst.adst_vjp(prob, x0, None, T, SEED, g, 0, adst.ADST_SCHED_AUTO, dx0, None, xT, L, None, ws,
                  need + room)
    torch.cuda.synchronize()
    return dx0.cpu().numpy(), xT.cpu().numpy(), float(L)


CASES = [(F64, (70, 127), 7), (F64, (9, 128), 8), (F64, (200, 129), 9), (F64, (100, 257), 16),
         (F64, (3, 300), 17), (F64, (64, 3), 33), (F64, (2, 130), 5), (F64, (40, 2), 5),
         (F64, (1, 1), 3), (F64, (90, 140), 258), (F32, (75, 255), 15), (F32, (33, 513), 31),
         (F32, (20, 259), 130), (F64, (21, 5001), 60)]


@pytest.mark.parametrize("dtype,shape,T", CASES)
def test_one_launch_gives_the_level_launches_bits(dtype, shape, T):
    say(f"gs pipe dtype={dtype} shape={shape} T={T}")
    r = np.random.Generator(np.random.PCG64(21))
    x = r.uniform(-1, 1, shape).astype(NP_DTYPE[dtype])
    aux = r.standard_normal(shape).astype(NP_DTYPE[dtype])
    prob = adst.make_problem(GS, dtype, (shape[1], shape[0], 1))
    room = adst.adst_sweep_workspace_bytes(prob, T)
    assert room > 0
    a, b = run(dtype, x, aux, T, room), run(dtype, x, aux, T, 0)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]) and a[2] == b[2]
    dx0, _, xT, L = oracle.vjp(GS, x, steps=T, loss=SEED, aux=aux)
    assert np.array_equal(a[1], xT)
    assert rel(a[0], dx0) <= TOL[dtype] and abs(a[2] - L) <= TOL[dtype] * np.abs(aux * xT).sum()


def test_values_that_are_not_finite():
    r = np.random.Generator(np.random.PCG64(22))
    x, aux = r.uniform(-1, 1, (90, 300)), r.standard_normal((90, 300))
    x[40, 140], x[0, 7], aux[60, 1], aux[89, 200] = np.inf, -np.inf, np.nan, np.inf
    prob = adst.make_problem(GS, F64, (300, 90, 1))
    a = run(F64, x, aux, 12, adst.adst_sweep_workspace_bytes(prob, 12))
    b = run(F64, x, aux, 12, 0)
    for k in range(2):
        assert np.array_equal(a[k], b[k], equal_nan=True)


def test_scratch_that_overlaps_an_array_is_not_used():
    """A larger ws_bytes whose part beyond the plan's holds loss_aux."""
    r = np.random.Generator(np.random.PCG64(23))
    x, aux = r.uniform(-1, 1, (50, 300)), r.standard_normal((50, 300))
    prob = adst.make_problem(GS, F64, (300, 50, 1))
    room = max(adst.adst_sweep_workspace_bytes(prob, 9), aux.nbytes)
    a, b = run(F64, x, aux, 9, room, tail=aux), run(F64, x, aux, 9, 0)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]) and a[2] == b[2]


def test_both_python_calls_on_another_stream():
    import torch
    r = np.random.Generator(np.random.PCG64(24))
    x = r.uniform(-1, 1, (150, 400))
    ref = oracle.forward(GS, x, steps=20)
    s = torch.cuda.Stream()
    t = dev(x)
    torch.cuda.synchronize()
    for stream in (s, s.cuda_stream):
        out = adst.vjp(GS, t, None, 20, budget_bytes=0, stream=stream)
        xT = adst.forward(GS, t, None, 20, stream=stream)
        s.synchronize()
        assert np.array_equal(out["xT"].cpu().numpy(), ref)
        assert np.array_equal(xT.cpu().numpy(), ref)

"""The persistent launch of the in-place kind's sweeps (calls with
adst_sweep_workspace_bytes of scratch) against the oracle and against the
level launches (calls without), bit for bit.

Shapes sit at the edges of the launch's pieces: strips of 128 (f64) or 256
(f32) columns that move one column per sweep, groups of 8 or 16 sweeps (four
or eight waves: EIGHT), 256 sweeps per launch, odd rows, grids without interior
points.
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


def run(dtype, x, aux, T, room):
    """adst_vjp_scratch with `room` bytes of scratch; without any, adst_vjp in
    a workspace larger than the plan's, whose tail it leaves alone."""
    import torch
    shape = x.shape
    prob = adst.make_problem(GS, dtype, (shape[1], shape[0], 1))
    need = adst.adst_plan(prob, T, 0, adst.ADST_SCHED_AUTO).workspace_bytes
    spare = room or adst.adst_sweep_workspace_bytes(prob, T)
    ws = torch.full((need + spare,), 0x5a, dtype=torch.uint8, device="cuda")
    scratch = torch.full((room,), 0x5a, dtype=torch.uint8, device="cuda") if room else None
    x0, g = dev(x), dev(aux)
    dx0, xT = torch.empty_like(x0), torch.empty_like(x0)
    L = torch.empty((), dtype=torch.float64, device="cuda")
    adst.adst_vjp(prob, x0, None, T, SEED, g, 0, adst.ADST_SCHED_AUTO, dx0, None, xT, L, None, ws,
                  need + spare, scratch=scratch, scratch_bytes=room)
    torch.cuda.synchronize()
    assert bool((ws[need:] == 0x5a).all())
    return dx0.cpu().numpy(), xT.cpu().numpy(), float(L)


CASES = [(F64, (70, 127), 7), (F64, (9, 128), 8), (F64, (200, 129), 9), (F64, (100, 257), 16),
         (F64, (3, 300), 17), (F64, (64, 3), 33), (F64, (2, 130), 5), (F64, (40, 2), 5),
         (F64, (1, 1), 3), (F64, (90, 140), 258), (F32, (75, 255), 15), (F32, (33, 513), 31),
         (F32, (20, 259), 130), (F64, (21, 5001), 60)]


# More than 256 workgroups of four waves would be at work at once, so eight
# waves are taken (twice the phases a group, and twice the halo): rows enough
# for the interior form, several strips and halo slots used more than once.
EIGHT = [(F64, (510, 1210), 250), (F32, (515, 2403), 250)]


@pytest.mark.parametrize("dtype,shape,T", CASES + EIGHT)
def test_one_launch_gives_the_level_launches_bits(dtype, shape, T):
    say(f"gs pipe dtype={dtype} shape={shape} T={T}")
    r = np.random.Generator(np.random.PCG64(21))
    x = r.uniform(-1, 1, shape).astype(NP_DTYPE[dtype])
    aux = r.standard_normal(shape).astype(NP_DTYPE[dtype])
    prob = adst.make_problem(GS, dtype, (shape[1], shape[0], 1))
    room = adst.adst_sweep_workspace_bytes(prob, T)
    assert room > 0
    if (dtype, shape, T) in EIGHT:  # four waves' halo: an eighth and a sixteenth of a state
        assert room > 1.5 * x.nbytes * (1 / 8 if dtype == F64 else 1 / 16)
    a, b = run(dtype, x, aux, T, room), run(dtype, x, aux, T, 0)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]) and a[2] == b[2]
    dx0, _, xT, L = oracle.vjp(GS, x, steps=T, loss=SEED, aux=aux)
    assert np.array_equal(a[1], xT)
    assert rel(a[0], dx0) <= TOL[dtype] and abs(a[2] - L) <= TOL[dtype] * np.abs(aux * xT).sum()


@pytest.mark.parametrize("dtype,shape,T,pipe", [
    (F32, (400, 600), 1, False), (F32, (400, 600), 4, True), (F32, (2000, 2100), 3, False),
    (F32, (2000, 2100), 7, True), (F32, (2000, 2101), 1, True), (F32, (3000, 40), 1, True),
    (F64, (30, 40), 1, False), (F64, (30, 41), 1, True), (F64, (30, 40), 2, True),
    (F64, (400, 600), 1, True)])
def test_short_forward_runs_take_the_faster_route(dtype, shape, T, pipe):
    """A forward run of up to six sweeps goes by levels where they are the
    faster (aligned rows only); the reverse sweeps stay one launch. The bits are the same."""
    r = np.random.Generator(np.random.PCG64(26))
    x = dev(r.uniform(-1, 1, shape).astype(NP_DTYPE[dtype]))
    a = adst.vjp(GS, x, None, T, flags=adst.ADST_TRACE)
    names = {k["name"] for k in adst.adst_trace_kernels() if k["name"].startswith("gs_")}
    assert names == {"gs_pipe<fwd>" if pipe else "gs_wave<fwd>", "gs_pipe<adj>"}
    b = adst.vjp(GS, x, None, T, scratch=False)
    for key in ("xT", "dx0", "loss"):
        assert np.array_equal(a[key].cpu().numpy(), b[key].cpu().numpy()), key
    assert np.array_equal(a["xT"].cpu().numpy(), oracle.forward(GS, x.cpu().numpy(), steps=T))


def test_values_that_are_not_finite():
    r = np.random.Generator(np.random.PCG64(22))
    x, aux = r.uniform(-1, 1, (90, 300)), r.standard_normal((90, 300))
    x[40, 140], x[0, 7], aux[60, 1], aux[89, 200] = np.inf, -np.inf, np.nan, np.inf
    prob = adst.make_problem(GS, F64, (300, 90, 1))
    a = run(F64, x, aux, 12, adst.adst_sweep_workspace_bytes(prob, 12))
    b = run(F64, x, aux, 12, 0)
    for k in range(2):
        assert np.array_equal(a[k], b[k], equal_nan=True)


def test_forward_leaves_a_workspace_it_does_not_need():
    """In this kind's forward call ws is not used at all, however large."""
    import torch
    r = np.random.Generator(np.random.PCG64(23))
    x = r.uniform(-1, 1, (50, 300))
    prob = adst.make_problem(GS, F64, (300, 50, 1))
    room = adst.adst_sweep_workspace_bytes(prob, 9)
    x0, ref = dev(x), oracle.forward(GS, x, steps=9)
    for scratch in (None, torch.full((room,), 0x5a, dtype=torch.uint8, device="cuda")):
        ws = torch.full((2 * room,), 0x5a, dtype=torch.uint8, device="cuda")
        xT = torch.empty_like(x0)
        adst.adst_forward(prob, x0, None, 9, xT, ws, ws.numel(), scratch=scratch,
                          scratch_bytes=0 if scratch is None else room)
        assert bool((ws == 0x5a).all())
        assert np.array_equal(xT.cpu().numpy(), ref)


def test_the_callers_workspace_and_scratch_are_the_ones_used():
    """A call takes no workspace of its own beside a given one, and beyond the
    outputs only the scratch, which the caller can give or decline."""
    import torch
    r = np.random.Generator(np.random.PCG64(25))
    x = dev(r.uniform(-1, 1, (300, 500)))
    T, budget, flags = 12, 10 * x.nbytes, adst.ADST_FORCE_TAPE
    prob = adst.make_problem(GS, F64, (500, 300, 1), flags=flags)
    extra = adst.adst_sweep_workspace_bytes(prob, T)
    need = adst.adst_plan(prob, T, budget, adst.ADST_SCHED_BINOMIAL).workspace_bytes
    assert need > 10 * x.nbytes > extra > 0
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    mine = torch.empty(extra, dtype=torch.uint8, device="cuda")
    ref = oracle.forward(GS, x.cpu().numpy(), steps=T)
    for scratch, used in ((None, extra), (mine, extra), (False, 0)):
        torch.cuda.synchronize()
        torch.cuda.reset_peak_memory_stats()
        before = torch.cuda.memory_stats()["requested_bytes.all.current"]
        out = adst.vjp(GS, x, None, T, budget_bytes=budget, sched=adst.ADST_SCHED_BINOMIAL,
                       flags=flags, ws=ws, scratch=scratch)
        torch.cuda.synchronize()
        taken = torch.cuda.memory_stats()["requested_bytes.all.peak"] - before
        assert out["ws"] is ws and out["scratch_bytes"] == used
        assert taken <= 2 * x.nbytes + (extra if scratch is None else 0) + 4096, taken
        assert np.array_equal(out["xT"].cpu().numpy(), ref)
        del out
        assert np.array_equal(adst.forward(GS, x, None, T, scratch=scratch).cpu().numpy(), ref)


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

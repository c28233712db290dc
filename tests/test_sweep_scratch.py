"""adst_sweep_workspace_bytes on the host: the scratch with which the in-place
kind's sweeps run as one persistent launch, 0 where that launch cannot run."""
import pytest

import paper_2509_02197_amd as adst

GS = adst.ADST_GAUSSSEIDEL2D5
F64, F32 = adst.ADST_F64, adst.ADST_F32


def scratch(dtype, nx, ny, T):
    return adst.adst_sweep_workspace_bytes(adst.make_problem(GS, dtype, (nx, ny, 1)), T)


@pytest.mark.parametrize("dtype", [F64, F32])
def test_extents_near_the_32_bit_limit_have_no_persistent_launch(dtype):
    for nx, ny in [(2**31 - 1, 1), (2**31 - 200, 1), (1, 2**31 - 1), (1, 2**31 - 200)]:
        for T in (1, 100, 1000):
            assert scratch(dtype, nx, ny, T) == 0, (nx, ny, T)


def test_launches_beyond_the_dispatch_grid_have_no_persistent_launch():
    """Strips of 128 (f64) or 256 (f32) columns, groups of 16 phases of 512
    work-items each: these would have 2^32 work-items or more."""
    for dtype, nx, ny, T in [(F64, 160_000_000, 3, 100), (F64, 80_000_000, 20, 255),
                             (F64, 700_000_000, 3, 100), (F32, 320_000_000, 3, 100),
                             (F32, 160_000_000, 10, 1000)]:
        assert scratch(dtype, nx, ny, T) == 0, (dtype, nx, ny, T)


def test_an_invalid_problem_gets_0_and_leaves_the_last_error():
    """Both after a call that failed and after one that succeeded."""
    good = adst.make_problem(GS, F64, (40, 30, 1))
    for steps, bad in [(5, (0, 30, 1)), (5, (40, 30, 2))]:
        adst.adst_plan(good, 5, 0, 0)
        assert adst.adst_sweep_workspace_bytes(adst.make_problem(GS, F64, bad), steps) == 0
        assert adst.adst_last_error() == ""
        with pytest.raises(adst.AdstError):
            adst.adst_plan(good, -1, 0, 0)
        error = adst.adst_last_error()
        assert "steps" in error
        assert adst.adst_sweep_workspace_bytes(adst.make_problem(GS, F64, bad), steps) == 0
        assert adst.adst_last_error() == error
    assert scratch(F64, 40, 30, 0) == 0 and scratch(F64, 40, 30, -1) == 0


def test_scratch_is_bounded_and_of_the_documented_size():
    """Never more than two states and 64 KiB (or 1 MiB); at most about a
    quarter of an f64 state and an eighth of an f32 one on wide grids, a state or less from 48
    columns on at 200 sweeps."""
    for dtype, isz in ((F64, 8), (F32, 4)):
        for nx in (1, 3, 4, 7, 8, 15, 16, 24, 48, 127, 129, 400, 5000, 100_000):
            for ny in (1, 3, 50, 5000, 20_000, 300_000):
                if nx * ny > 2**30:
                    continue
                state = nx * ny * isz
                for T in (1, 9, 100, 200, 255, 1000):
                    b = scratch(dtype, nx, ny, T)
                    assert b <= max(2 * state + (64 << 10), 1 << 20) + 128, (nx, ny, T)
                    if 48 <= nx <= 5000 and 48 <= ny <= 5000 and T <= 200:
                        assert 0 < b <= state + 4096, (nx, ny, T)
        assert scratch(dtype, 3, 1_000_000, 255) == 0
        for n in (4096, 20_000):
            share = scratch(dtype, n, n, 100) / (n * n * isz)
            assert 0 < share <= (0.28 if dtype == F64 else 0.14)


def test_wide_grids_of_few_rows_take_the_narrow_workgroup():
    """Few strips of a group are at work at a time there: the halo is that of
    four waves, an eighth of an f64 state, not of eight."""
    for nx, ny, T, eight in [(20_000, 64, 10, False), (5000, 48, 100, False),
                             (100_000, 300, 20, False), (4096, 4096, 100, True),
                             (5000, 3000, 100, True)]:
        share = scratch(F64, nx, ny, T) / (nx * ny * 8)
        assert (0.2 < share < 0.3) if eight else (0.1 < share < 0.2), (nx, ny, T)


def test_scratch_that_overlaps_an_array_is_refused():
    """Only the bytes that the sweeps would use count; with too little the
    scratch is not used, so another argument's error is what the call reports.
    The pointers are never dereferenced."""
    import torch
    if torch.cuda.device_count() > 0:
        pytest.skip("host-only argument checks")
    prob = adst.make_problem(GS, F64, (300, 50, 1))
    S, T = 300 * 50 * 8, 9
    need = adst.adst_sweep_workspace_bytes(prob, T)
    x0, aux, dx0, xT, L, ws, free = (0x10000000 * (i + 1) for i in range(7))

    def status(at, nbytes, **kw):
        a = dict(xT=xT, steps=T)
        a.update(kw)
        with pytest.raises(adst.AdstError) as e:
            adst.adst_vjp(prob, x0, None, a["steps"], adst.ADST_LOSS_SEED, aux, 0, 0, dx0, None,
                          a["xT"], L, None, ws, 1 << 20, 0, scratch=at, scratch_bytes=nbytes)
        return e.value.status, str(e.value)

    for name, at in (("x0", x0), ("loss_aux", aux), ("dx0", dx0), ("xT", xT), ("ws", ws)):
        for p in (at, at - need // 2):
            st, msg = status(p, need)
            assert st == adst.ADST_ERR_ARG and "scratch" in msg and name in msg
        if name in ("x0", "xT"):
            with pytest.raises(adst.AdstError, match="scratch"):
                adst.adst_forward(prob, x0, None, T, xT, None, 0, 0, scratch=at,
                                  scratch_bytes=need)
    # too little, or beside the arrays: the next error is the one reported
    for at, nbytes in ((x0, need // 2), (free, need)):
        st, msg = status(at, nbytes, xT=dx0)
        assert st == adst.ADST_ERR_ARG and "scratch" not in msg

"""Shared helpers of the GPU tests: move inputs to the device, run the
library through its C-ABI binding, bring results back, compare."""
import sys

import numpy as np

import oracle
import paper_2509_02197_amd as adst

NP_DTYPE = {adst.ADST_F64: np.float64, adst.ADST_F32: np.float32}
TOL = {adst.ADST_F64: 1e-12, adst.ADST_F32: 1e-5}


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def rel(a, b):
    a = np.asarray(a, dtype=np.float64)
    b = np.asarray(b, dtype=np.float64)
    nb = np.linalg.norm(b)
    return float(np.linalg.norm(a - b) / (nb if nb > 0 else 1.0))


def dev(a):
    import torch
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    import torch
    if t is None:
        return None
    if torch.is_tensor(t):
        return t.detach().cpu().numpy()
    return t


def gpu_vjp(kind, inp, steps, loss, budget=None, sched=adst.ADST_SCHED_AUTO, want_dK=False,
            flags=0, params=None, ws=None, keep_ws=False, want_xT=True, want_dparams=False,
            lim=None, scratch=None):
    import torch
    out = adst.vjp(kind, dev(inp["x0"]), dev(inp.get("K")), steps, loss, dev(inp.get("aux")),
                   budget, sched, want_dK, params, flags, ws=ws, want_xT=want_xT,
                   want_dparams=want_dparams, lim=lim, scratch=scratch)
    torch.cuda.synchronize()
    res = {k: host(v) for k, v in out.items() if k not in ("ws", "info")}
    res["loss"] = float(res["loss"])
    res["info"] = out["info"].as_dict()
    if keep_ws:
        res["ws"] = out["ws"]
    return res


def check_dw(kind, inp, steps, got, want, tol, lim=None):
    """dL/dp[0] of a 2-D kind against the oracle's, for L = <aux, x_T>. It is a
    sum over points and steps of g_t * dF/dp[0](x_{t-1}); each g_t is within a
    relative tol of the oracle's, as dx0 is, so the sum is within tol of the
    sum of the terms' magnitudes (the terms may cancel). The second constant
    is unused: 0."""
    x, p0 = inp["x0"].astype(np.float64), 0.2 if kind == adst.ADST_JACOBI2D5 else 0.1
    K, aux = inp.get("K"), inp["aux"].astype(np.float64)
    K = None if K is None else K.astype(np.float64)
    size = 0.0
    for t in range(1, steps + 1):
        raw = oracle.forward(kind, x, K=K, steps=1)
        nxt = raw if lim is None else oracle.forward(kind, x, K=K, steps=1, lim=lim)
        g = oracle.vjp(kind, nxt, K=K, steps=steps - t, loss=adst.ADST_LOSS_SEED, aux=aux,
                       lim=lim)[0]
        part = np.zeros_like(x)
        if kind == adst.ADST_JACOBI2D5:
            part[1:-1, 1:-1] = raw[1:-1, 1:-1] / p0
        else:
            part = (raw - x) / p0
        size += np.abs(g * part).sum()
        x = nxt
    assert abs(got[0] - want[0]) <= tol * size, (got[0], want[0], size)
    assert got[1] == want[1] == 0.0

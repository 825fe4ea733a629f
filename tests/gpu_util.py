"""Helpers for the -m gpu tests: move a seeded workload to the device, call the library,
and compare with the fp64 oracle.  (Not collected by pytest.)"""
import numpy as np


def rel_l2(x, ref):
    x = np.asarray(x, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    den = np.linalg.norm(ref)
    num = np.linalg.norm(x - ref)
    return num / den if den > 0 else num


# Bars of the parity tests.  "head": relative L2 error of O over one (b, h), and of S_L (the
# stated tolerance of the build: 1e-4 for fp32 inputs, 2e-2 for bf16 inputs with fp32 accumulation);
# it must hold for EVERY head, not only for all heads taken together.  "token": |o_t - ref_t| over
# the head's RMS token norm, for every single token, so that a few wrong tokens cannot hide in a long
# sequence.  "element": largest single error over the head's RMS element.  The last two follow from
# the arithmetic: a bf16 result carries 2^-9 per rounding (operands of every contraction and the
# stored O), the chain of a head accumulates a few of them, and the largest of d_v * L elements of
# roughly normal errors sits 5 to 6 deviations out.
# Measured over every case of the suite (all heads of the five full-size configurations included):
# bf16 head <= 4.9e-3, token <= 9.9e-3, element <= 3.8e-2; fp32 head <= 3.4e-7, token <= 5.2e-7,
# element <= 2.4e-6.  The head bars are the stated ones; the others leave a factor of about three
# (bf16) and twenty (fp32, whose cases are short) over what was seen.
BARS = {"f32": dict(head=1e-4, token=1e-5, element=5e-5),
        "bf16": dict(head=2e-2, token=3e-2, element=1.2e-1)}


def error_stats(err2, ref2, maxabs, dv):
    """err2, ref2 [N, L] (squared error / squared norm of every token's output), maxabs [N]
    -> dict(all, head, token, element), each the worst over heads (all: heads taken together)."""
    err2 = np.asarray(err2, dtype=np.float64)
    ref2 = np.asarray(ref2, dtype=np.float64)
    tiny = np.finfo(np.float64).tiny
    rms_tok = np.sqrt(np.maximum(ref2.mean(axis=1), tiny))
    return dict(all=float(np.sqrt(err2.sum() / max(ref2.sum(), tiny))),
                head=float(np.sqrt(err2.sum(axis=1) / np.maximum(ref2.sum(axis=1), tiny)).max()),
                token=float((np.sqrt(err2) / rms_tok[:, None]).max()),
                element=float((np.asarray(maxabs) / (rms_tok / np.sqrt(dv))).max()))


def output_stats(O, Oref):
    """The same statistics from full arrays [N, L, dv]."""
    O = np.asarray(O, dtype=np.float64)
    Oref = np.asarray(Oref, dtype=np.float64)
    d = O - Oref
    return error_stats((d * d).sum(-1), (Oref * Oref).sum(-1), np.abs(d).reshape(d.shape[0], -1).max(axis=1), O.shape[-1])


def assert_parity(st, eS_heads, dtype, what=""):
    """st from error_stats / output_stats, eS_heads the per-head relative L2 errors of S_L."""
    bar = BARS[dtype]
    worst_S = float(np.max(eS_heads)) if len(eS_heads) else 0.0
    print(f"        {what}relL2(O) all={st['all']:.3e} worst head={st['head']:.3e} worst token={st['token']:.3e} "
          f"worst element={st['element']:.3e}  relL2(S_L) worst head={worst_S:.3e}", flush=True)
    assert st["head"] <= bar["head"], (st, bar)
    assert st["token"] <= bar["token"], (st, bar)
    assert st["element"] <= bar["element"], (st, bar)
    assert worst_S <= bar["head"], (worst_S, bar)


def state_errors(SL, SLref):
    """Per-head relative L2 error of the final state, [N, dv, dk] each."""
    SL = np.asarray(SL, dtype=np.float64)
    SLref = np.asarray(SLref, dtype=np.float64)
    num = np.sqrt(((SL - SLref) ** 2).sum(axis=(1, 2)))
    den = np.sqrt((SLref ** 2).sum(axis=(1, 2)))
    return np.where(den > 0, num / np.where(den > 0, den, 1.0), num)


def to_device(w, inp, B=None, H=None):
    """numpy fp32 inputs with head axis N -> torch tensors shaped [B, H, ...] in the workload's dtype."""
    import torch
    B = w.B if B is None else B
    H = w.H if H is None else H
    tdt = torch.bfloat16 if w.dtype == "bf16" else torch.float32
    dev = torch.device("cuda:0")

    def up(a, dt):
        t = torch.from_numpy(np.ascontiguousarray(a)).to(dev)
        return t.reshape((B, H) + tuple(a.shape[1:])).to(dt).contiguous()

    out = {k: up(inp[k], tdt) for k in ("Q", "K", "V", "beta")}
    out["S0"] = None if inp["S0"] is None else up(inp["S0"], torch.float32)
    return out


def run_gpu(pf, w, dev, chunk=None):
    import torch
    O, SL = pf.delta_fwd(dev["Q"], dev["K"], dev["V"], dev["beta"], dev["S0"], chunk=chunk or w.chunk)
    torch.cuda.synchronize()
    return O.float().cpu().numpy(), SL.cpu().numpy()


def flat_heads(a):
    return a.reshape((-1,) + a.shape[2:])


def kernels_of(call):
    """Names of this library's kernels that call() launches, in order and with their parameter lists, as a profiler prints them
    (the bodies of the generic kernel differ in the type of the last parameter)."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    call()                                       # (a first call looks up devices and kernels)
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA], acc_events=True) as p:
        call()
        torch.cuda.synchronize()
    ran = sorted((e for e in p.events() if "pf::" in e.name), key=lambda e: e.time_range.start)
    return [e.name for e in ran]


# ---- decoding of the tiled operand arrays of pf_delta_chunk_flow (layouts: include/pf.h)
def _lane_grid():
    lane = np.arange(64)
    return lane & 15, lane >> 4          # r16, g


def untile_rows8(t, ntile, nk, relabel=False):
    """[ntile][nk][64][8] -> matrix [16*ntile, 32*nk]; element (lane, e) sits at row 16 i + r16 and
    column 32 k + 8 g + e (or, with relabel, 32 k + 4 g + e for e < 4 and 32 k + 16 + 4 g + e - 4)."""
    t = np.asarray(t).reshape(ntile, nk, 64, 8)
    r16, g = _lane_grid()
    out = np.full((16 * ntile, 32 * nk), np.nan)
    e = np.arange(8)
    for i in range(ntile):
        for k in range(nk):
            if relabel:
                col = 32 * k + np.where(e[None, :] < 4, 4 * g[:, None] + e[None, :], 16 + 4 * g[:, None] + e[None, :] - 4)
            else:
                col = 32 * k + 8 * g[:, None] + e[None, :]
            out[(16 * i + r16)[:, None], col] = t[i, k]
    return out


def untile_acc4(t, mt, dt):
    """[mt][dt][64][4] -> matrix [16*mt, 16*dt]; element (lane, e) at row 16 i + 4 g + e, column 16 j + r16."""
    t = np.asarray(t).reshape(mt, dt, 64, 4)
    r16, g = _lane_grid()
    out = np.full((16 * mt, 16 * dt), np.nan)
    e = np.arange(4)
    for i in range(mt):
        for j in range(dt):
            out[16 * i + 4 * g[:, None] + e[None, :], (16 * j + r16)[:, None]] = t[i, j]
    return out


def launches(call):
    """[name, grid, threads] of the kernels of this library that `call` launches, in order, out of a trace."""
    import json
    import os
    import re
    import tempfile
    import torch
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA], acc_events=True) as p:
        call()
        torch.cuda.synchronize()
    with tempfile.TemporaryDirectory() as where:
        p.export_chrome_trace(os.path.join(where, "trace.json"))
        with open(os.path.join(where, "trace.json")) as f:
            events = [e for e in json.load(f)["traceEvents"] if "pf::" in e.get("name", "") and "grid" in e.get("args", {})]
    return [[re.sub(r"^void ", "", re.match(r"[^(]*", e["name"]).group(0)), e["args"]["grid"][0], e["args"]["block"][0]]
            for e in sorted(events, key=lambda e: e["ts"])]

"""What a user of this library has it do, as sized cases: the chunked forward of the rank-r delta rule
(additive and product form, Euler and exact steps), the same forward for general low-rank drivers, and
the step-by-step use of both through the state (a few tokens in, the state carried on), in bf16 and in
fp32.  Everything goes through the public entry points of paper_2504_00492_amd.binding.

A case is a dict of plain values:
  form     "delta" (pf delta_fwd), "drivers" (general drivers A, Atil, B)
  dtype    "bf16" or "f32": element type of the sequence arrays (states are always fp32)
  B, H, L, d_k, d_v, r, chunk   as in include/pf.h
  s0       an initial state is handed in (a sequence that goes on from an earlier one)
  reflect  share of tokens whose betas are near-reflections, U(1.5, 2)
  product  the r sub-updates of a token are applied one after another
  exact    beta goes through pf_beta_exponential first (exact rank-1 steps)
"""
import math

import torch

from paper_2504_00492_amd import binding as pf

DTYPES = {"bf16": (torch.bfloat16, pf.PF_BF16, 2), "f32": (torch.float32, pf.PF_F32, 4)}


def _case(name, form, dtype, B, H, L, d_k, d_v, r, chunk, s0=False, reflect=0.0, product=False, exact=False):
    c = dict(form=form, dtype=dtype, B=B, H=H, L=L, d_k=d_k, d_v=d_v, r=r, chunk=chunk, s0=s0, reflect=reflect,
             product=product, exact=exact)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # configuration 0: one small fp32 head, the cost of a call
        _case("tiny fp32", "delta", "f32", 1, 1, 64, 16, 16, 1, 16),
        # one new token per sequence for 64 sequences of 16 heads: serving, state in and out
        _case("one token", "delta", "bf16", 64, 16, 1, 128, 128, 2, 64, s0=True),
        # configuration 1: the rank-1 rule at head width 64
        _case("rank 1, width 64", "delta", "bf16", 4, 8, 2048, 64, 64, 1, 64),
        # configuration 2: the ordinary training-like batch
        _case("rank 2", "delta", "bf16", 4, 16, 4096, 128, 128, 2, 64),
        # configuration 3, chunk 128: rank 4 from a given state
        _case("rank 4", "delta", "bf16", 2, 16, 8192, 128, 128, 4, 128, s0=True),
        # configuration 4: the long sequence with near-reflections, the largest case
        _case("long sequence", "delta", "bf16", 1, 32, 65536, 128, 128, 2, 128, reflect=0.1),
        # a prompt of odd length that continues an earlier one
        _case("ragged length", "delta", "bf16", 2, 16, 3001, 128, 128, 1, 64, s0=True),
        # few heads (a small model, or one shard of a large one) on a long sequence
        _case("few heads", "delta", "bf16", 1, 4, 32768, 128, 128, 2, 64),
        # product of exact rank-1 steps, values wider than keys
        _case("exact product steps", "delta", "bf16", 2, 12, 4096, 64, 128, 2, 64, product=True, exact=True),
        # configuration 1's shape in fp32
        _case("fp32, width 64", "delta", "f32", 4, 8, 2048, 64, 64, 1, 64),
        # general drivers at the width of configurations 2 to 4
        _case("drivers", "drivers", "bf16", 2, 16, 4096, 128, 128, 2, 64),
        # general drivers in fp32, odd length, d_k and d_v apart
        _case("drivers fp32", "drivers", "f32", 1, 8, 500, 32, 48, 2, 16, s0=True),
    ]


# the largest listed case, in state elements touched per rank: drawn cases stay below it
MOST_WORK = 32 * 65536 * 128 * 128 * 2
MOST_WORK_F32 = 32 * 2048 * 64 * 64 * 1


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _heads(rng, most):
    H = _log(rng, 1, min(most, 32))
    return max(1, _log(rng, 1, max(1, most // H))), H


def draw(rng):
    kind = rng.random()
    if kind < 0.12:
        # a few new tokens per sequence
        B, H = _log(rng, 4, 96), rng.choice([8, 12, 16, 24])
        d = rng.choice([64, 128])
        return _case(None, "delta", "bf16", B, H, rng.choice([1, 1, 2, 3, 5, 8]), d, d, rng.choice([1, 2, 4]), 64, s0=True,
                     product=rng.random() < 0.25)
    if kind < 0.32:
        # fp32: any width
        form = "delta" if rng.random() < 0.7 else "drivers"
        d_k = rng.choice([16, 24, 32, 48, 64, 96, 128])
        d_v = d_k if rng.random() < 0.7 else rng.choice([16, 32, 40, 64, 96, 128])
        r, (B, H) = rng.choice([1, 1, 2, 3, 4]), _heads(rng, 64)
        L = min(_log(rng, 16, 2048), max(1, MOST_WORK_F32 // (B * H * d_k * d_v * r)))
        return _case(None, form, "f32", B, H, L, d_k, d_v, r, rng.choice([16, 32, 64]), s0=rng.random() < 0.5,
                     reflect=0.1 if form == "delta" and rng.random() < 0.3 else 0.0,
                     product=form == "delta" and r > 1 and rng.random() < 0.3)
    # bf16: the widths that have matrix kernels, any length
    form = "delta" if rng.random() < 0.8 else "drivers"
    d_k = rng.choice([64, 128, 128])
    d_v = d_k if rng.random() < 0.7 else rng.choice([32, 48, 64, 96, 128, 192, 256])
    r, chunk, (B, H) = rng.choice([1, 2, 2, 4]), rng.choice([64, 128]), _heads(rng, 128)
    L = min(_log(rng, 48, 65536), 131072 // r, max(48, MOST_WORK // (B * H * max(d_k * d_v, 128 * 128) * r)))
    if rng.random() < 0.4:
        L = max(64, L // 64 * 64)
    product = form == "delta" and r > 1 and rng.random() < 0.3
    return _case(None, form, "bf16", B, H, L, d_k, d_v, r, chunk, s0=rng.random() < 0.5,
                 reflect=0.1 if form == "delta" and rng.random() < 0.3 else 0.0, product=product,
                 exact=form == "delta" and (product or r == 1) and rng.random() < 0.25)


def prepare(case, seed):
    tdt, dt, _ = DTYPES[case["dtype"]]
    B, H, L, d_k, d_v, r = (case[k] for k in ("B", "H", "L", "d_k", "d_v", "r"))
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev).manual_seed(int(seed))
    n = lambda *shape: torch.randn(shape, generator=gen, device=dev)
    u = lambda *shape: torch.rand(shape, generator=gen, device=dev)

    def unit(x):
        return x.div_(x.norm(dim=-1, keepdim=True))

    s = dict(case=case)
    s["Q"] = (n(B, H, L, d_k) / math.sqrt(d_k)).to(tdt)
    k = unit(n(B, H, L, r, d_k))
    beta = torch.sigmoid(n(B, H, L, r))
    if case["reflect"]:
        near = u(B, H, L, 1) < case["reflect"]
        beta = torch.where(near, 1.5 + 0.5 * u(B, H, L, r), beta)
    v = n(B, H, L, r, d_v) / math.sqrt(d_v)
    if case["form"] == "delta":
        s["K"], s["V"], s["beta"] = k.to(tdt), v.to(tdt), beta.to(tdt)
        if case["exact"]:
            s["beta_eff"] = torch.empty_like(s["beta"])
        need = pf.pf_delta_fwd_workspace_bytes(B, H, L, d_k, d_v, r, case["chunk"], dt)
    else:
        # near the delta form (so that the state stays bounded), A and B independent of each other
        s["A"] = (beta[..., None] * (k + 0.3 * unit(n(B, H, L, r, d_k)))).to(tdt)
        s["Bm"] = (-(k + 0.3 * unit(n(B, H, L, r, d_k)))).to(tdt)
        s["Atil"] = v.to(tdt)
        need = 0
        if dt == pf.PF_BF16:
            need = pf.pf_flow_fwd_mfma_workspace_bytes(B, H, L, d_k, d_v, r, case["chunk"], dt)
            s["O"] = torch.empty((B, H, L, d_v), dtype=tdt, device=dev)
            s["S_L"] = torch.empty((B, H, d_v, d_k), dtype=torch.float32, device=dev)
    s["S0"] = 0.1 * n(B, H, d_v, d_k) if case["s0"] else None
    s["workspace"] = torch.empty(need, dtype=torch.uint8, device=dev) if need else None
    s["need"] = need
    return s


def run(state):
    c = state["case"]
    if c["form"] == "delta":
        beta = state["beta"]
        if c["exact"]:
            st = pf.pf_beta_exponential(state["K"], beta, state["beta_eff"], c["B"], c["H"], c["L"], c["d_k"], c["r"],
                                        DTYPES[c["dtype"]][1])
            if st != pf.PF_OK:
                raise pf.PfError(st, "pf_beta_exponential")
            beta = state["beta_eff"]
        return pf.delta_fwd(state["Q"], state["K"], state["V"], beta, state["S0"], chunk=c["chunk"],
                            workspace=state["workspace"], product=c["product"])
    if c["dtype"] == "f32":
        return pf.flow_fwd(state["Q"], state["A"], state["Atil"], state["Bm"], state["S0"], chunk=c["chunk"])
    st = pf.pf_flow_fwd_mfma(state["Q"], state["A"], state["Atil"], state["Bm"], state["S0"], state["O"], state["S_L"],
                             c["B"], c["H"], c["L"], c["d_k"], c["d_v"], c["r"], c["chunk"], pf.PF_BF16,
                             state["workspace"], state["need"])
    if st != pf.PF_OK:
        raise pf.PfError(st, "pf_flow_fwd_mfma")
    return state["O"], state["S_L"]


def work(case):
    """Every input read once, every output written once; flops of the token-by-token recurrence (S k and the
    rank-1 update for each of the r columns, S q): no chunking does with fewer products of that size."""
    e = DTYPES[case["dtype"]][2]
    heads, L, d_k, d_v, r = case["B"] * case["H"], case["L"], case["d_k"], case["d_v"], case["r"]
    per_token = d_k + r * d_k + r * d_v + d_v + (r if case["form"] == "delta" else r * d_k)
    states = (1 + (1 if case["s0"] else 0)) * d_k * d_v * 4
    return {"bytes": heads * (L * per_token * e + states), "flops": heads * L * (4 * r + 2) * d_k * d_v}


def tolerance(case):
    # bf16: T, P, S, the solved values and O are each rounded to bf16 once on the way (2^-9 each); the
    # largest single element of a long sequence sits five to six deviations out
    return {"rel": 1e-2, "max": 0.12} if case["dtype"] == "bf16" else {"rel": 1e-5, "max": 4e-4}

"""The generic kernel's row shapes against the fp64 oracle: every width class of d_k at its edges (rows
padded in registers, rows that are not whole 16-byte pieces, rows longer than the registers hold), ranks
with and without a shape of their own, row tiles that d_v does not fill, more tokens than one staging."""
import numpy as np
import pytest

from paper_2504_00492_amd import synth
from gpu_util import rel_l2, to_device, flat_heads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("product", [False, True])
@pytest.mark.parametrize("dtype,dk,dv,r,L,chunk", [
    ("f32", 16, 16, 1, 130, 64), ("f32", 17, 5, 2, 70, 32), ("f32", 32, 33, 4, 41, 16), ("f32", 33, 16, 3, 29, 8),
    ("f32", 64, 64, 1, 200, 64), ("f32", 65, 20, 2, 33, 16), ("f32", 128, 70, 4, 40, 16), ("f32", 129, 8, 1, 20, 4),
    ("f32", 256, 12, 2, 21, 8), ("f32", 260, 6, 5, 9, 2), ("f32", 512, 10, 1, 19, 16), ("f32", 600, 7, 3, 11, 4),
    ("bf16", 24, 40, 2, 90, 32), ("bf16", 36, 24, 8, 17, 4), ("bf16", 128, 128, 2, 5, 64), ("bf16", 64, 64, 1, 1, 64),
    ("bf16", 100, 9, 6, 13, 2), ("bf16", 520, 3, 2, 10, 4),
])
def test_generic_row_shapes(oracle, dtype, dk, dv, r, L, chunk, product):
    import torch
    from paper_2504_00492_amd import binding as pf
    w = synth.Workload("rows", dtype, 1, 3, L, dk, dv, r, chunk, seed=17, s0_std=0.2, reflect_frac=0.05)
    print(f"[case] generic rows {dtype} d=({dk},{dv}) r={r} L={L} chunk={chunk} product={product}", flush=True)
    assert pf.pf_delta_fwd_workspace_bytes(1, 3, L, dk, dv, r, chunk, pf.PF_BF16 if dtype == "bf16" else pf.PF_F32) == 0
    inp = synth.make_inputs(w)
    dev = to_device(w, inp)
    O, SL = pf.delta_fwd(dev["Q"], dev["K"], dev["V"], dev["beta"], dev["S0"], chunk=chunk, product=product)
    torch.cuda.synchronize()
    ref = oracle.delta_product_fwd if product else oracle.delta_fwd
    Oref, SLref = ref(inp["Q"], inp["K"], inp["V"], inp["beta"], inp["S0"])
    assert rel_l2(flat_heads(O.float().cpu().numpy()), Oref) <= (5e-6 if dtype == "f32" else 4e-3)
    assert rel_l2(flat_heads(SL.cpu().numpy()), SLref) <= 5e-6


@pytest.mark.parametrize("dtype,dk,dv,r,L,chunk", [
    ("f32", 32, 48, 2, 75, 16), ("f32", 40, 9, 3, 30, 8), ("f32", 64, 64, 1, 90, 64), ("f32", 100, 33, 4, 26, 16),
    ("f32", 128, 20, 2, 40, 16), ("f32", 129, 8, 1, 20, 4), ("f32", 256, 12, 2, 21, 8), ("f32", 260, 6, 5, 9, 2),
    ("f32", 512, 10, 4, 12, 4), ("f32", 520, 3, 2, 10, 4), ("f32", 600, 7, 3, 11, 4),
    ("bf16", 24, 40, 2, 70, 32), ("bf16", 36, 24, 8, 17, 4), ("bf16", 192, 10, 3, 15, 4), ("bf16", 256, 12, 1, 30, 8),
    ("bf16", 514, 5, 6, 9, 2),
])
def test_generic_row_shapes_of_drivers(oracle, dtype, dk, dv, r, L, chunk):
    """The same row shapes for general drivers (near the delta form, A and B independent of each other)."""
    import torch
    from paper_2504_00492_amd import binding as pf
    N = 3
    rng = np.random.default_rng(1000 * dk + r)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    unit = lambda *s: (lambda x: x / np.linalg.norm(x, axis=-1, keepdims=True))(rng.standard_normal(s))
    k, beta = unit(N, L, r, dk), 1.0 / (1.0 + np.exp(-rng.standard_normal((N, L, r, 1))))
    up = lambda a: torch.from_numpy(a.astype(np.float32)).to("cuda:0").to(tdt)[None].contiguous()
    tq, tat = up(rng.standard_normal((N, L, dk)) / np.sqrt(dk)), up(rng.standard_normal((N, L, r, dv)) / np.sqrt(dv))
    ta, tb = up(beta * (k + 0.3 * unit(N, L, r, dk))), up(-(k + 0.3 * unit(N, L, r, dk)))
    S0 = (0.2 * rng.standard_normal((N, dv, dk))).astype(np.float32)
    print(f"[case] generic rows of drivers {dtype} d=({dk},{dv}) r={r} L={L} chunk={chunk}", flush=True)
    O, SL = pf.flow_fwd(tq, ta, tat, tb, torch.from_numpy(S0).to("cuda:0")[None].contiguous(), chunk=chunk)
    torch.cuda.synchronize()
    back = lambda t: t[0].float().cpu().numpy().astype(np.float64)
    for h in range(N):
        Oref, SLref = oracle.flow_head(back(ta)[h], back(tat)[h], back(tb)[h], back(tq)[h], S0[h].astype(np.float64))
        assert rel_l2(back(O)[h], Oref) <= (5e-6 if dtype == "f32" else 4e-3)
        assert rel_l2(back(SL)[h], SLref) <= 5e-6

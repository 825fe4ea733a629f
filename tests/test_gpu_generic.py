"""The generic kernel's row shapes against the fp64 oracle: every width class of d_k at its edges (rows
padded in registers, rows that are not whole 16-byte pieces, rows longer than the registers hold), ranks
with and without a shape of their own, row tiles that d_v does not fill, more tokens than one staging.
Few heads of up to 128 columns go 16 virtual tokens at a time instead; test_bodies has the heads that take the
rows, and checks which body ran."""
import numpy as np
import pytest

from paper_2504_00492_amd import synth
from gpu_util import flat_heads, kernels_of, rel_l2, to_device

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


ROWS, BLOCKS, FEW = "RowShape<", "BlockShape<", "FewTokens<"
# on 256 compute units; a comment names the line of the dispatch that a case sits at
BODIES = [
    # rows: each width and rank, whole 16-byte pieces and not, several stagings with a remainder
    ("delta", "f32", 1300, 133, 16, 16, 1, 32, ROWS), ("delta", "f32", 700, 67, 17, 20, 2, 16, ROWS), ("delta", "f32", 600, 50, 32, 32, 4, 16, ROWS),
    ("delta", "f32", 560, 61, 33, 20, 3, 16, ROWS), ("delta", "f32", 300, 90, 64, 64, 2, 64, ROWS), ("delta", "f32", 300, 45, 50, 64, 5, 8, ROWS),
    ("delta", "f32", 130, 70, 128, 128, 4, 16, ROWS), ("delta", "f32", 150, 41, 100, 96, 3, 16, ROWS), ("delta", "f32", 200, 60, 128, 70, 1, 64, ROWS),
    ("delta", "bf16", 700, 83, 24, 40, 2, 64, ROWS), ("delta", "bf16", 560, 40, 36, 24, 8, 64, ROWS), ("delta", "bf16", 300, 150, 40, 64, 2, 64, ROWS),
    ("delta", "bf16", 200, 77, 100, 72, 4, 64, ROWS), ("delta", "bf16", 180, 30, 128, 128, 2, 64, ROWS),
    ("product", "f32", 300, 40, 64, 64, 2, 64, ROWS), ("product", "f32", 700, 35, 16, 20, 4, 16, ROWS), ("product", "bf16", 600, 29, 64, 64, 4, 64, ROWS),
    ("drivers", "f32", 1300, 150, 16, 16, 1, 32, ROWS), ("drivers", "f32", 600, 67, 32, 24, 2, 16, ROWS), ("drivers", "f32", 300, 45, 64, 50, 3, 16, ROWS),
    ("drivers", "f32", 150, 43, 128, 96, 4, 16, ROWS), ("drivers", "f32", 160, 29, 100, 96, 5, 8, ROWS), ("drivers", "f32", 300, 90, 128, 64, 1, 64, ROWS),
    ("drivers", "bf16", 700, 83, 24, 40, 2, 64, ROWS), ("drivers", "bf16", 300, 61, 64, 64, 4, 64, ROWS), ("drivers", "bf16", 200, 37, 120, 64, 8, 64, ROWS),
    # r = 1, up to 32 columns: four rounds of workgroups, five
    ("delta", "f32", 1024, 110, 16, 16, 1, 32, BLOCKS), ("delta", "f32", 1025, 110, 16, 16, 1, 32, ROWS), ("drivers", "bf16", 1030, 105, 32, 16, 1, 64, ROWS),
    ("delta", "f32", 1025, 105, 36, 16, 1, 32, BLOCKS), ("delta", "bf16", 1025, 201, 20, 16, 1, 64, BLOCKS), ("delta", "bf16", 1025, 200, 20, 16, 1, 64, ROWS),
    # bf16 rows that are not whole pieces of four: rounds, columns, ranks, lengths
    ("delta", "bf16", 354, 143, 17, 17, 1, 64, ROWS), ("delta", "bf16", 350, 143, 17, 16, 1, 64, BLOCKS), ("delta", "bf16", 300, 350, 17, 16, 1, 64, ROWS),
    ("delta", "bf16", 300, 143, 65, 16, 1, 64, ROWS), ("delta", "bf16", 24, 63, 33, 33, 4, 64, ROWS), ("delta", "bf16", 24, 50, 33, 33, 4, 64, BLOCKS),
    ("delta", "bf16", 24, 63, 31, 31, 4, 64, BLOCKS), ("delta", "bf16", 350, 143, 16, 16, 1, 64, BLOCKS), ("delta", "f32", 354, 143, 17, 17, 1, 64, BLOCKS),
    ("delta", "bf16", 13, 14, 127, 127, 1, 64, ROWS), ("delta", "bf16", 14, 13, 50, 50, 2, 64, ROWS),
    # where a block would lose digits: fewer than 16 columns, few tokens of few columns
    ("delta", "bf16", 354, 143, 15, 17, 1, 64, ROWS), ("delta", "f32", 3, 300, 15, 16, 1, 32, ROWS), ("drivers", "f32", 3, 150, 8, 16, 2, 16, ROWS),
    ("delta", "f32", 3, 40, 16, 16, 1, 32, ROWS), ("delta", "f32", 3, 41, 16, 16, 1, 32, BLOCKS), ("delta", "f32", 3, 16, 24, 16, 1, 32, ROWS),
    ("delta", "f32", 3, 17, 24, 16, 1, 32, BLOCKS), ("drivers", "f32", 3, 20, 20, 16, 2, 16, ROWS), ("drivers", "f32", 3, 21, 20, 16, 2, 16, BLOCKS),
    ("delta", "bf16", 3, 16, 16, 16, 1, 64, ROWS), ("delta", "bf16", 3, 17, 16, 16, 1, 64, BLOCKS), ("delta", "bf16", 3, 13, 24, 16, 1, 64, BLOCKS),
    # one round, ranks 2 and 4
    ("delta", "bf16", 16, 14, 128, 128, 2, 64, ROWS), ("delta", "bf16", 16, 15, 128, 128, 2, 64, BLOCKS), ("delta", "f32", 16, 11, 128, 128, 2, 16, BLOCKS),
    # a few tokens: rank times width, wavefronts, rows that they fill
    ("delta", "bf16", 22, 1, 128, 128, 4, 64, FEW), ("delta", "bf16", 22, 2, 128, 128, 4, 64, ROWS), ("delta", "bf16", 38, 2, 128, 128, 4, 64, FEW),
    ("drivers", "bf16", 8, 1, 128, 128, 4, 64, ROWS), ("drivers", "bf16", 15, 2, 128, 128, 2, 64, ROWS), ("drivers", "bf16", 15, 2, 64, 64, 2, 64, FEW),
    ("drivers", "f32", 574, 8, 128, 20, 4, 16, ROWS), ("drivers", "f32", 508, 4, 128, 128, 4, 16, FEW), ("drivers", "f32", 1981, 1, 128, 8, 4, 16, ROWS),
    ("delta", "bf16", 1358, 7, 128, 1, 4, 64, ROWS), ("delta", "bf16", 1580, 2, 64, 1, 2, 64, FEW), ("delta", "bf16", 134, 6, 128, 100, 1, 64, ROWS),
]


@pytest.mark.parametrize("form,dtype,heads,L,dk,dv,r,chunk,body", BODIES)
def test_bodies(oracle, form, dtype, heads, L, dk, dv, r, chunk, body):
    """Which body of the generic kernel takes a call, and its results on some of the heads, the first and the last among them."""
    import torch
    from paper_2504_00492_amd import binding as pf
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the lines lie by rounds over 256 compute units")
    gen = torch.Generator(device="cuda:0").manual_seed(heads + 1000 * dk + L)
    n = lambda *s: torch.randn((1, heads) + s, generator=gen, device="cuda:0")
    unit = lambda x: x / x.norm(dim=-1, keepdim=True)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    q, k, v, beta = n(L, dk) / dk ** 0.5, unit(n(L, r, dk)), n(L, r, dv) / dv ** 0.5, torch.sigmoid(n(L, r)) / max(1.0, r / 4)
    S0 = 0.2 * n(dv, dk)
    print(f"[case] body {form} {dtype} heads={heads} d=({dk},{dv}) r={r} L={L} chunk={chunk}", flush=True)
    if form == "drivers":
        ins = [x.to(tdt).contiguous() for x in (q, beta[..., None] * (k + 0.3 * unit(n(L, r, dk))), v, -(k + 0.3 * unit(n(L, r, dk))))]
        call = lambda: pf.flow_fwd(*ins, S0, chunk=chunk)
        one = lambda i, h: oracle.flow_head(i[1][h], i[2][h], i[3][h], i[0][h], S0[0, h].double().cpu().numpy())
    else:
        ins = [x.to(tdt).contiguous() for x in (q, k, v, beta)]
        call = lambda: pf.delta_fwd(*ins, S0, chunk=chunk, product=form == "product")
        ref = oracle.delta_product_fwd if form == "product" else oracle.delta_fwd
        one = lambda i, h: [x[0] for x in ref(*(a[h:h + 1] for a in i), S0[0, h:h + 1].cpu().numpy())]
    name, = kernels_of(call)
    assert body in name, name
    O, SL = (x[0].double().cpu().numpy() for x in call())
    some = sorted({0, 1, heads // 3, heads // 2 + 1, heads - 1} & set(range(heads)))
    host = [x[0].float().cpu().numpy() for x in ins]
    for h in some:
        Oref, SLref = one([a.astype(np.float64) for a in host] if form == "drivers" else host, h)
        assert rel_l2(O[h], Oref) <= (5e-6 if dtype == "f32" else 4e-3)
        assert rel_l2(SL[h], SLref) <= 5e-6

"""Which kernels a call launches, by name, and that a name tells which code ran.  Tiles of 16 rows and blocks of 64 virtual
tokens take the chain in one wavefront: one tile to a workgroup up to one workgroup per compute unit, two beyond where d_v
allows, and the body of eight wavefronts (two workgroups a compute unit) where it does not (d_v = 16 mod 32)."""
import re
import subprocess

import numpy as np
import pytest

from paper_2504_00492_amd import synth
from test_abi_host import pf  # noqa: F401  (fixture: builds / loads the library)
from test_wait_states import _functions, _listings


def _names(pf, heads, L, dk, dv, r):  # noqa: F811
    return pf.pf_delta_fwd_describe(1, heads, L, dk, dv, r, 64, pf.PF_BF16)


def _scan(pf, heads, L, dk, dv, r):  # noqa: F811
    return next(n for n in _names(pf, heads, L, dk, dv, r) if n.startswith("pf::scan_kernel"))


def _cus():
    try:
        import torch
        if torch.cuda.is_available():
            return torch.cuda.get_device_properties(0).multi_processor_count
    except ImportError:
        pass
    return 256


@pytest.mark.parametrize("dk", [64, 128])
@pytest.mark.parametrize("dv", [48, 64, 112, 128])
def test_body_by_workgroups(pf, dk, dv):  # noqa: F811
    most = _cus() // (dv // 16)                  # heads that still give every workgroup a compute unit
    for r in (1, 2):
        shape = f"pf::scan_kernel<{dk}, 64, {64 // r}, 16, true, false"
        assert _scan(pf, most, 640, dk, dv, r) == shape + ">"
        if dv % 32:                              # no tiles of 32 rows: any number of heads
            assert _scan(pf, most + 1, 640, dk, dv, r) == shape + ", true>"
            assert _scan(pf, 20 * most, 640, dk, dv, r) == shape + ", true>"
        else:
            assert _scan(pf, most + 1, 640, dk, dv, r) == f"pf::scan_kernel<{dk}, 64, {64 // r}, 32, true, false, true>"
    assert _scan(pf, 20 * most, 640, dk, 64, 2) == f"pf::scan_kernel<{dk}, 64, 32, 32, true, false>"


@pytest.mark.parametrize("dk", [64, 128])
@pytest.mark.parametrize("dv", [48, 128])
def test_rank_4_in_halves_where_the_chain_serves_them(pf, dk, dv):  # noqa: F811
    halves, whole, most = f"pf::flow_kernel<{dk}, 64, 16, false>", f"pf::flow_kernel<{dk}, 128, 32, false>", _cus() // (dv // 16)
    assert _names(pf, most, 96, dk, dv, 4) == [halves, f"pf::scan_kernel<{dk}, 64, 16, 16, true, false>"]
    if dv % 32:
        assert _names(pf, most + 1, 96, dk, dv, 4) == [whole, f"pf::scan_kernel<{dk}, 128, 32, 16, true, false>"]
    else:
        assert _names(pf, most + 1, 96, dk, dv, 4) == [halves, f"pf::scan_kernel<{dk}, 64, 16, 32, true, false, true>"]
        assert _names(pf, 2 * most, 96, dk, dv, 4) == [whole, f"pf::scan_kernel<{dk}, 128, 32, 32, true, false>"]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("r", [1, 2, 4])
def test_segments_by_heads_and_blocks(pf, d, r):  # noqa: F811
    """A quarter of the compute units in use and 32 blocks to cut: four segments a head, cut once more from 32 blocks of 64
    virtual tokens a segment on; more heads or fewer blocks: none."""
    most, tokens = _cus() // 4 // (d // 16), 64 // r
    kinds = lambda heads, L: [re.sub(r"<.*, (\d+)(, true, false(, true)?)?>", r"<\1>", n) for n in _names(pf, heads, L, d, d, r)[1:]]
    maps = lambda rows: 2 * [f"pf::segment_maps_kernel<{rows}>"]
    assert [n for n in kinds(most, 8 * 32 * tokens) if "compose" not in n] == maps(32) + ["pf::scan_kernel<32>"]
    assert [n for n in kinds(most, 8 * 30 * tokens) if "compose" not in n] == maps(16) + ["pf::scan_kernel<16>"]
    assert kinds(most + 1, 8 * 32 * tokens) == ["pf::scan_kernel<16>"]
    block = max(tokens, 32)                      # (of 128 virtual tokens at rank 4: they are what is counted)
    assert len(kinds(most, 32 * block)) == 4 and len(kinds(most, 28 * block)) == 1


@pytest.mark.parametrize("dk,dv,line", [(128, 128, 5), (128, 64, 5), (64, 64, 16), (64, 128, 64), (64, 192, None)])
@pytest.mark.parametrize("r", [1, 2])
def test_more_than_a_round_of_two_tiles_by_blocks(pf, dk, dv, line, r):  # noqa: F811
    """One round: the chain whatever the length.  More: the chain from as many blocks on as pay for the rounds, else the split."""
    once, block = _cus() // (dv // 32), 64 // r
    chain, split = (f"pf::scan_kernel<{dk}, 64, {block}, 32, true, false{x}>" for x in ("", ", false"))
    if _cus() % (dv // 32) == 0:                 # (as many workgroups as compute units: no fewer, which is another form)
        assert _scan(pf, once, block, dk, dv, r) == chain and _scan(pf, once, 100 * block, dk, dv, r) == chain
    assert _scan(pf, once + 1, ((line or 500) - 1) * block, dk, dv, r) == split
    if line:
        assert _scan(pf, once + 1, line * block, dk, dv, r) == chain and _scan(pf, 10 * once, line * block + 1, dk, dv, r) == chain


# every branch of the dispatch: B * H, L, d_k, d_v, r, chunk
SHAPES = [(65, 96, 128, 128, 2, 64), (32, 2048, 64, 64, 1, 64), (64, 4096, 128, 128, 2, 64), (32, 3001, 128, 128, 1, 64), (33, 256, 128, 128, 2, 64),
          (65, 300, 64, 64, 1, 64), (100, 96, 64, 48, 2, 64), (32, 1024, 128, 128, 4, 128), (40, 96, 64, 128, 4, 64),
          (20, 160, 64, 48, 4, 64), (64, 96, 128, 128, 4, 64), (100, 96, 64, 48, 4, 64), (2, 2048, 128, 128, 1, 64),
          (8, 8192, 128, 128, 2, 64), (2, 2048, 64, 64, 4, 64), (8, 16384, 64, 64, 4, 64), (3, 40, 128, 128, 1, 64)]


def _kernels(library, tmp_path):
    """Names of the kernels in the library, without parameter lists, one for each kernel."""
    names = []
    for listing in _listings(tmp_path):
        mangled = [name for name, body, _ in _functions(listing)]
        plain = subprocess.run(["c++filt"], input="\n".join(mangled), capture_output=True, text=True, check=True).stdout.split("\n")
        names += [re.sub(r"^void ", "", re.match(r"[^(]*", n).group(0)) for n in plain if n]
    return names


def test_a_name_stands_for_one_kernel(pf, tmp_path):  # noqa: F811
    kernels = _kernels(pf, tmp_path)
    for heads, L, dk, dv, r, chunk in SHAPES:
        for name in pf.pf_delta_fwd_describe(1, heads, L, dk, dv, r, chunk, pf.PF_BF16):
            if not name.startswith("pf::generic_kernel"):
                assert kernels.count(name) == 1, (name, kernels.count(name))


@pytest.mark.gpu
def test_described_kernels_are_the_ones_that_run():
    """Against the names that a profiler prints, in the order of the launches."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    from paper_2504_00492_amd import binding as pf  # noqa: F811
    gen, dev = torch.Generator(device="cuda:0").manual_seed(3), "cuda:0"
    rand = lambda *s: 0.1 * torch.randn(s, generator=gen, device=dev)
    inputs = [(rand(1, h, L, dk).bfloat16(), rand(1, h, L, r, dk).bfloat16(), rand(1, h, L, r, dv).bfloat16(), rand(1, h, L, r).bfloat16(), chunk)
              for h, L, dk, dv, r, chunk in SHAPES]
    for q, k, v, b, chunk in inputs:             # (first calls look up devices and kernels)
        pf.delta_fwd(q, k, v, b, None, chunk=chunk)
    torch.cuda.synchronize()
    for shape, (q, k, v, b, chunk) in zip(SHAPES, inputs):
        with profile(activities=[ProfilerActivity.CUDA], acc_events=True) as p:
            pf.delta_fwd(q, k, v, b, None, chunk=chunk)
            torch.cuda.synchronize()
        ran = sorted((e for e in p.events() if "pf::" in e.name), key=lambda e: e.time_range.start)
        names = [re.sub(r"^void ", "", re.match(r"[^(]*", e.name).group(0)) for e in ran]
        h, L, dk, dv, r, chunk = shape
        assert names == pf.pf_delta_fwd_describe(1, h, L, dk, dv, r, chunk, pf.PF_BF16), shape


@pytest.mark.gpu
@pytest.mark.parametrize("heads,L,dk,dv,r", [(65, 64, 64, 64, 1), (100, 165, 64, 64, 2), (33, 96, 128, 128, 2),
                                             (60, 150, 128, 128, 1), (90, 101, 64, 48, 2), (40, 224, 128, 112, 2)])
def test_parity_beyond_the_compute_units(oracle, heads, L, dk, dv, r):
    import torch
    from gpu_util import assert_parity, flat_heads, output_stats, rel_l2, to_device
    from paper_2504_00492_amd import binding as pf  # noqa: F811
    w = synth.Workload("route", "bf16", 1, heads, L, dk, dv, r, 64, seed=heads, s0_std=0.2, reflect_frac=0.05)
    print(f"[case] scan beyond the compute units heads={heads} L={L} d=({dk},{dv}) r={r}", flush=True)
    assert _scan(pf, heads, L, dk, dv, r).endswith("32, true, false, true>" if dv % 32 == 0 else "16, true, false, true>")
    inp = synth.make_inputs(w)
    dev = to_device(w, inp)
    O, SL = pf.delta_fwd(dev["Q"], dev["K"], dev["V"], dev["beta"], dev["S0"], chunk=64)
    torch.cuda.synchronize()
    Oref, SLref = oracle.delta_fwd(inp["Q"], inp["K"], inp["V"], inp["beta"], inp["S0"])
    SLn, SLref = SL.cpu().numpy().reshape(heads, dv, dk), np.asarray(SLref).reshape(heads, dv, dk)
    assert_parity(output_stats(flat_heads(O.float().cpu().numpy()), Oref), [rel_l2(SLn[h], SLref[h]) for h in range(heads)], "bf16")


@pytest.mark.gpu
@pytest.mark.parametrize("drivers", [False, True])
@pytest.mark.parametrize("heads,dk,dv,r,L", [(88, 64, 48, 2, 70), (96, 64, 48, 2, 64), (97, 128, 48, 2, 64), (128, 64, 48, 2, 45), (136, 128, 48, 2, 40),
                                             (104, 128, 48, 4, 40), (112, 64, 48, 4, 64), (96, 128, 48, 1, 64),
                                             (136, 64, 64, 2, 70), (160, 64, 64, 2, 40), (168, 64, 64, 1, 64), (96, 128, 128, 2, 40), (104, 128, 128, 2, 64), (73, 128, 128, 2, 64),
                                             (176, 128, 64, 2, 40), (64, 128, 160, 2, 40), (72, 128, 128, 1, 70), (72, 128, 128, 4, 40), (80, 64, 128, 4, 64)])
def test_parity_of_both_orders_of_tiles(oracle, heads, dk, dv, r, L, drivers):
    """Workgroups of the split, with 16 rows and with 32, around the lines between the two orders of its tiles: as many as compute units
    and a few more, one and a quarter times and one and a half times as many, heads that are no multiple of eight."""
    import torch
    from gpu_util import assert_parity, flat_heads, output_stats, rel_l2, to_device
    from paper_2504_00492_amd import binding as pf  # noqa: F811
    w = synth.Workload("order", "bf16", 1, heads, L, dk, dv, r, 64, seed=heads + r, s0_std=0.2, reflect_frac=0.05)
    print(f"[case] order of tiles heads={heads} L={L} d=({dk},{dv}) r={r} drivers={drivers}", flush=True)
    inp = synth.make_inputs(w)
    dev = to_device(w, inp)
    if drivers:
        A, Bm = (dev["beta"][..., None] * dev["K"]).contiguous(), (-dev["K"]).contiguous()
        O, SL = torch.empty(1, heads, L, dv, dtype=torch.bfloat16, device="cuda:0"), torch.empty(1, heads, dv, dk, device="cuda:0")
        need = pf.pf_flow_fwd_mfma_workspace_bytes(1, heads, L, dk, dv, r, 64, pf.PF_BF16)
        ws = torch.empty(need, dtype=torch.uint8, device="cuda:0")
        assert pf.pf_flow_fwd_mfma(dev["Q"], A, dev["V"], Bm, dev["S0"], O, SL, 1, heads, L, dk, dv, r, 64, pf.PF_BF16, ws, need) == pf.PF_OK
        f = lambda x: flat_heads(x.float().cpu().numpy())
        heads_of = zip(f(A), f(dev["V"]), f(Bm), f(dev["Q"]), f(dev["S0"]))
        Oref, SLref = (np.stack(x) for x in zip(*(oracle.flow_head(*x) for x in heads_of)))
    else:
        O, SL = pf.delta_fwd(dev["Q"], dev["K"], dev["V"], dev["beta"], dev["S0"], chunk=64)
        Oref, SLref = oracle.delta_fwd(inp["Q"], inp["K"], inp["V"], inp["beta"], inp["S0"])
    torch.cuda.synchronize()
    SLn, SLref = SL.cpu().numpy().reshape(heads, dv, dk), np.asarray(SLref).reshape(heads, dv, dk)
    assert_parity(output_stats(flat_heads(O.float().cpu().numpy()), Oref), [rel_l2(SLn[h], SLref[h]) for h in range(heads)], "bf16")

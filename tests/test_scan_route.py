"""Which body of the scan a call takes at 16-row tiles and blocks of 64 virtual tokens: the chain in one wavefront up to
one workgroup per compute unit, the body of eight wavefronts (two workgroups a compute unit) beyond."""
import numpy as np
import pytest

from paper_2504_00492_amd import synth
from test_abi_host import pf  # noqa: F401  (fixture: builds / loads the library)


def _scan(pf, heads, L, dk, dv, r):  # noqa: F811
    return next(n for n in pf.pf_delta_fwd_describe(1, heads, L, dk, dv, r, 64, pf.PF_BF16) if n.startswith("pf::scan_kernel"))


@pytest.mark.parametrize("dk", [64, 128])
@pytest.mark.parametrize("dv", [48, 64, 112, 128])
def test_body_by_workgroups(pf, dk, dv):  # noqa: F811
    cus = 256
    try:
        import torch
        if torch.cuda.is_available():
            cus = torch.cuda.get_device_properties(0).multi_processor_count
    except ImportError:
        pass
    most = cus // (dv // 16)                     # heads that still give every workgroup a compute unit
    for r in (1, 2):
        shape = f"pf::scan_kernel<{dk}, 64, {64 // r}, 16, true, false"
        assert _scan(pf, most, 640, dk, dv, r) == shape + ">"
        assert _scan(pf, most + 1, 640, dk, dv, r) == shape + ", true>"
        if dv % 32:                              # no tiles of 32 rows: any number of heads
            assert _scan(pf, 20 * most, 640, dk, dv, r) == shape + ", true>"
    assert _scan(pf, 20 * most, 640, dk, 64, 2) == f"pf::scan_kernel<{dk}, 64, 32, 32, true, false>"


@pytest.mark.gpu
@pytest.mark.parametrize("heads,L,dk,dv,r", [(65, 64, 64, 64, 1), (100, 165, 64, 64, 2), (33, 96, 128, 128, 2),
                                             (60, 150, 128, 128, 1), (90, 101, 64, 48, 2), (40, 224, 128, 112, 2)])
def test_parity_beyond_the_compute_units(oracle, heads, L, dk, dv, r):
    import torch
    from gpu_util import assert_parity, flat_heads, output_stats, rel_l2, to_device
    from paper_2504_00492_amd import binding as pf  # noqa: F811
    w = synth.Workload("route", "bf16", 1, heads, L, dk, dv, r, 64, seed=heads, s0_std=0.2, reflect_frac=0.05)
    print(f"[case] scan beyond the compute units heads={heads} L={L} d=({dk},{dv}) r={r}", flush=True)
    assert _scan(pf, heads, L, dk, dv, r).endswith("16, true, false, true>")
    inp = synth.make_inputs(w)
    dev = to_device(w, inp)
    O, SL = pf.delta_fwd(dev["Q"], dev["K"], dev["V"], dev["beta"], dev["S0"], chunk=64)
    torch.cuda.synchronize()
    Oref, SLref = oracle.delta_fwd(inp["Q"], inp["K"], inp["V"], inp["beta"], inp["S0"])
    SLn, SLref = SL.cpu().numpy().reshape(heads, dv, dk), np.asarray(SLref).reshape(heads, dv, dk)
    assert_parity(output_stats(flat_heads(O.float().cpu().numpy()), Oref), [rel_l2(SLn[h], SLref[h]) for h in range(heads)], "bf16")

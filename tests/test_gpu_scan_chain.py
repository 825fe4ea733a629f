"""The scan of 16-row tiles with the whole chain in one wavefront, against the fp64 oracle: every remainder of the
helper waves' block groups and of the LDS ring, fewer blocks than the ring holds, a tail behind the blocks (odd
element offsets of beta between heads), both token-tile counts, and the segment-parallel form of d = 64."""
import numpy as np
import pytest

from paper_2504_00492_amd import synth
from gpu_util import assert_parity, flat_heads, output_stats, rel_l2, to_device

pytestmark = pytest.mark.gpu


def _check(oracle, heads, L, dk, dv, r, seed):
    import torch
    from paper_2504_00492_amd import binding as pf
    w = synth.Workload("chain", "bf16", 1, heads, L, dk, dv, r, 64, seed=seed, s0_std=0.2, reflect_frac=0.05)
    print(f"[case] scan chain heads={heads} L={L} d=({dk},{dv}) r={r}", flush=True)
    inp = synth.make_inputs(w)
    dev = to_device(w, inp)
    O, SL = pf.delta_fwd(dev["Q"], dev["K"], dev["V"], dev["beta"], dev["S0"], chunk=64)
    torch.cuda.synchronize()
    Oref, SLref = oracle.delta_fwd(inp["Q"], inp["K"], inp["V"], inp["beta"], inp["S0"])
    SLn = SL.cpu().numpy().reshape(heads, dv, dk)
    assert_parity(output_stats(flat_heads(O.float().cpu().numpy()), Oref),
                  [rel_l2(SLn[h], np.asarray(SLref).reshape(heads, dv, dk)[h]) for h in range(heads)], "bf16")
    return pf.pf_delta_fwd_describe(1, heads, L, dk, dv, r, 64, pf.PF_BF16)


@pytest.mark.parametrize("dk,dv", [(64, 64), (128, 128), (128, 48), (64, 112)])
@pytest.mark.parametrize("r", [1, 2])
@pytest.mark.parametrize("blocks,tail", [(1, 0), (2, 5), (3, 0), (4, 1), (5, 0), (6, 3), (7, 0), (13, 9)])
def test_block_counts(oracle, blocks, tail, r, dk, dv):
    block = 64 // r
    names = _check(oracle, 3, blocks * block + tail, dk, dv, r, 100 * blocks + tail)
    assert any(n.startswith(f"pf::scan_kernel<{dk}, 64, {block}, 16, true") for n in names)


@pytest.mark.parametrize("d,r,L", [(64, 1, 2048), (64, 2, 1536), (128, 1, 2304)])
def test_segments(oracle, d, r, L):
    names = _check(oracle, 2, L, d, d, r, 7)
    assert "pf::segment_compose_kernel" in names

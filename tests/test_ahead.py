"""What asks for the chain's lines ahead of time, without a GPU: csrc/pf_ahead.h in a host library of its own, and a model of the
wavefronts that go by it (touch_ahead in csrc/pf_chain.h)."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2504_00492_amd", "csrc")
RING = 6


@pytest.fixture(scope="session")
def ahead(tmp_path_factory):
    where = tmp_path_factory.mktemp("ahead")
    (where / "ahead.cpp").write_text('#include "pf_ahead.h"\nextern "C" {\n'
                                     "int window(int d) { return pf::ahead_window(d); }\n"
                                     "int lost() { return pf::kAheadLost; }\n"
                                     "int beyond(int b, int at, int window) { return pf::ahead_beyond(b, at, window); }\n"
                                     "int late(int b, int at) { return pf::ahead_late(b, at); }\n"
                                     "int workgroups(int c, int h, int d, int dv, int chunk, int n) { return pf::ahead_workgroups(c, h, d, dv, chunk, n); }\n"
                                     "int wavefront(int c, int h, int dv, int n, int p) { return pf::ahead_wavefront(c, h, dv, n, p); }\n}\n")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(where / "ahead.cpp"), "-o", str(where / "ahead.so")], check=True)
    return ctypes.CDLL(str(where / "ahead.so"))


def _asks(ahead, window, blocks, each, starts, cost, lost=None):
    """Blocks that a wavefront asks for, each with the block that it last saw the chain at and the one that the chain is at; `each`: time
    of a block of the chain, `cost`: of asking for one, `starts`: when the wavefront does, `lost`: when nobody has seen progress any more."""
    out, now, seen, at, looks = [], starts, 0, RING - window, 0
    for b in range(RING, blocks):
        while ahead.beyond(b, at, window):
            if seen >= 0 and seen < blocks - window:     # the first wavefront looks until the rest is within the window
                seen = ahead.lost() if lost is not None and now >= lost else min(int(now // each), blocks - 1)
            at, now, looks = seen, now + 0.1, looks + 1
            if at == ahead.lost():
                return out
            assert looks < 100 * blocks + 100, "the loop does not end"
        if not ahead.late(b, at):
            out.append((b, at, min(int(now // each), blocks - 1)))
            now += cost
    return out


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("blocks", [1, 6, 7, 17, 18, 19, 24, 128])
@pytest.mark.parametrize("cost", [0.01, 0.9, 1.5, 40.0])
def test_asks_for_blocks_between_the_chain_and_the_window(ahead, d, blocks, cost):
    window = ahead.window(d)
    asked = _asks(ahead, window, blocks, 1.0, 0.0, cost)
    assert [b for b, _, _ in asked] == sorted({b for b, _, _ in asked})
    assert all(at + 2 <= b <= at + window for b, at, _ in asked[1:])
    if cost < 1:                                         # it keeps up: every block that the chain does not ask for at once itself
        assert [b for b, _, _ in asked] == list(range(RING, blocks)) and all(is_at <= b for b, _, is_at in asked)
    # however slow it is, no more than a window behind the chain between two looks
    behind = [b for b, _, is_at in asked[1:] if b < is_at]
    assert len(behind) <= window * sum(1 for x, y in zip(asked, asked[1:]) if y[1] != x[1]) + window


@pytest.mark.parametrize("blocks", [24, 128, 2048])
def test_a_late_start_asks_for_what_is_left(ahead, blocks):
    window = ahead.window(64)
    assert len(_asks(ahead, window, blocks, 1.0, 10.0 * blocks, 0.5)) == 1
    assert len(_asks(ahead, window, blocks, 1.0, blocks - 4.0, 0.5)) <= 3


def test_nothing_more_once_the_chain_is_lost(ahead):
    window = ahead.window(64)
    assert len(_asks(ahead, window, 2048, 1.0, 0.0, 0.5, lost=100.0)) <= 100 + window
    assert len(_asks(ahead, window, 2048, 1.0, 50.0, 0.5, lost=50.0)) == 1


# compute units, heads, d, d_v, tokens of a block, blocks: workgroups that ask
@pytest.mark.parametrize("call,some", [((256, 24, 64, 64, 32, 128), 56), ((256, 32, 64, 64, 32, 128), 72), ((256, 40, 64, 64, 32, 128), 88),   # as many as are of use, all
                                       ((256, 24, 64, 128, 32, 128), 64), ((256, 20, 128, 128, 32, 128), 40), ((256, 24, 128, 128, 32, 128), 48),
                                       ((256, 55, 64, 64, 32, 128), 36), ((256, 56, 64, 64, 32, 128), 0),          # too much for each
                                       ((256, 28, 128, 128, 32, 128), 32), ((256, 29, 128, 128, 32, 128), 0),
                                       ((256, 24, 64, 64, 32, 24), 56), ((256, 24, 64, 64, 32, 23), 0),            # too few blocks
                                       ((256, 4, 128, 128, 64, 128), 8), ((256, 3, 128, 128, 64, 128), 0), ((256, 8, 64, 64, 64, 128), 24), ((256, 7, 64, 64, 64, 128), 0),   # too few workgroups
                                       ((256, 4, 128, 128, 32, 357), 8), ((256, 4, 128, 128, 32, 356), 0), ((256, 23, 64, 64, 32, 110), 48), ((256, 23, 64, 64, 32, 109), 0),   # few and small
                                       ((256, 16, 128, 128, 32, 128), 32), ((256, 12, 128, 128, 64, 128), 24),
                                       ((256, 20, 128, 128, 16, 256), 48), ((256, 16, 128, 128, 16, 256), 40), ((256, 15, 128, 128, 16, 256), 0),   # halves of rank 4
                                       ((256, 24, 64, 64, 16, 128), 48), ((256, 23, 64, 64, 16, 128), 0),
                                       ((256, 60, 128, 48, 64, 128), 76), ((256, 68, 128, 48, 64, 128), 0),        # L2
                                       ((256, 110, 64, 16, 32, 128), 146), ((256, 97, 64, 16, 64, 128), 0),
                                       ((256, 32, 128, 128, 64, 1000), 0), ((256, 300, 64, 64, 64, 1000), 0)])     # none idle
def test_who_asks(ahead, call, some):
    assert ahead.workgroups(*call) == some


# compute units, heads, d_v, blocks, P handed over
@pytest.mark.parametrize("call,asks", [((256, 32, 64, 16, 0), 1), ((256, 32, 64, 15, 0), 0), ((256, 31, 64, 16, 0), 0), ((256, 60, 48, 128, 0), 0),
                                       ((256, 60, 48, 128, 1), 0), ((256, 64, 64, 128, 1), 0), ((256, 32, 80, 128, 1), 1),
                                       ((256, 8, 128, 1, 1), 1), ((256, 7, 128, 128, 1), 0)])
def test_which_workgroups_ask_themselves(ahead, call, asks):
    assert ahead.wavefront(*call) == asks


def test_no_more_than_idle_compute_units_and_what_fits_their_l2(ahead):
    for cus in (64, 80, 256, 304):
        for d in (64, 128):
            for dv in (16, 32, 48, 64, 112, 128, 256):
                for heads in range(1, cus // (dv // 16) + 2):
                    works = heads * (dv // 16)
                    for chunk in (16, 32, 64):
                        some, lines = ahead.workgroups(cus, heads, d, dv, chunk, 500), heads * (d + chunk * d // 64 + dv + 48)
                        assert 0 <= some <= max(0, cus - works)
                        assert some < 8 + lines / (100 if d == 64 else 220 if chunk >= 32 else 150)
                        if some:
                            assert 8 * works >= (1 if chunk >= 32 else 3 if d == 64 else 4) * cus
                            assert chunk != 32 or 8 * works >= (3 if d == 64 else 4) * cus or lines * 500 * 128 >= 64 << 20
                            assert lines * 128 * ahead.window(d) <= 8 * (5 << 20) + 8 * 128 * ahead.window(d)

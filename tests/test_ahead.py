"""What asks for the chain's lines ahead of time, without a GPU: csrc/pf_ahead.h in a host library of its own, and a model of the
wavefronts that go by it (touch_ahead in csrc/pf_chain.h)."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2504_00492_amd", "csrc")
WAIT, STOP, LOST, RING = -1, -2, -1, 6


@pytest.fixture(scope="session")
def ahead(tmp_path_factory):
    where = tmp_path_factory.mktemp("ahead")
    (where / "ahead.cpp").write_text('#include "pf_ahead.h"\nextern "C" {\n'
                                     "int window(int d) { return pf::ahead_window(d); }\n"
                                     "int step(int b, int seen, int window) { return pf::ahead_step(b, seen, window); }\n}\n")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(where / "ahead.cpp"), "-o", str(where / "ahead.so")], check=True)
    return ctypes.CDLL(str(where / "ahead.so"))


def _asks(ahead, window, blocks, each, starts, cost, lost=None):
    """Blocks that a wavefront asks for, each with the block that the chain was seen at; `each`: time of a block of the chain,
    `cost`: of asking for one, `starts`: when the wavefront does, `lost`: when nobody has seen progress any more."""
    out, b, now, seen = [], RING, starts, 0
    for _ in range(100 * blocks + 100):
        if b >= blocks:
            return out
        if seen != LOST and seen < blocks - window:      # the first wavefront looks until the rest is within the window
            seen = LOST if lost is not None and now >= lost else min(int(now // each), blocks - 1)
        nxt = ahead.step(b, seen, window)
        if nxt == STOP:
            return out
        if nxt == WAIT:
            now += 0.1
        elif nxt != b:
            assert nxt > b
            b = nxt
        else:
            out.append((b, seen))
            b, now = b + 1, now + cost
    raise AssertionError("the loop does not end")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("blocks", [1, 6, 7, 17, 18, 19, 24, 128])
@pytest.mark.parametrize("cost", [0.01, 0.9, 1.5, 40.0])
def test_asks_for_blocks_between_the_chain_and_the_window(ahead, d, blocks, cost):
    window = ahead.window(d)
    asked = _asks(ahead, window, blocks, 1.0, 0.0, cost)
    assert [b for b, _ in asked] == sorted({b for b, _ in asked})
    assert all(seen + 2 <= b <= seen + window for b, seen in asked)
    if cost < 1:                                         # it keeps up: every block that the chain does not ask for at once itself
        assert [b for b, _ in asked] == list(range(RING, blocks))


@pytest.mark.parametrize("blocks", [24, 128, 2048])
def test_a_late_start_asks_for_what_is_left(ahead, blocks):
    window = ahead.window(64)
    assert _asks(ahead, window, blocks, 1.0, 10.0 * blocks, 0.5) == []
    assert len(_asks(ahead, window, blocks, 1.0, blocks - 4.0, 0.5)) <= 3


def test_nothing_more_once_the_chain_is_lost(ahead):
    window = ahead.window(64)
    assert len(_asks(ahead, window, 2048, 1.0, 0.0, 0.5, lost=100.0)) <= 100 + window
    assert _asks(ahead, window, 2048, 1.0, 50.0, 0.5, lost=50.0) == []

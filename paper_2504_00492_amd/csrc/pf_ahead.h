// Lines of the chain's later blocks that compute units which it leaves idle ask for ahead of time (touch_ahead, pf_chain.h): plain
// arithmetic, so that it can be looked at without a GPU.
#pragma once

namespace pf {

// Blocks ahead of the chain that may be asked for (touch_ahead says what other numbers cost).
constexpr int ahead_window(int d) { return d == 64 ? 18 : 14; }

// What a wavefront that has come to block b does next, with the chain last seen at block `seen`: b, to ask for block b now; a later
// block, to go on there, because the chain comes to b too soon; or one of
constexpr int kAheadWait = -1;                   // block b is beyond the window
constexpr int kAheadStop = -2;                   // nobody watches the chain any more
constexpr int kAheadLost = -1;                   // (`seen`, then)
// A wavefront that has fallen behind goes on in the middle of the window: two blocks ahead of the chain it is late again at once
// (24 heads x 4096 tokens, d = 64, d_v = 128, r = 2, inputs from HBM, all idle compute units: 73.5 us, in the middle 70.2).
constexpr int ahead_step(int b, int seen, int window)
{
    if (seen == kAheadLost) return kAheadStop;
    if (b > seen + window) return kAheadWait;
    return b < seen + 2 ? seen + window / 2 : b;
}

}  // namespace pf

// Lines of the chain's later blocks that somebody asks for ahead of time (pf_chain.h): workgroups on compute units that the chain
// leaves idle (touch_ahead), or at d = 128 a wavefront of each of its own.  Plain arithmetic, so that it can be looked at without a GPU.
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

// 128-byte lines of a block (64 virtual tokens) of one head: K, Q, V and the six tiles of T
constexpr int ahead_lines(int d, int dv, int chunk) { return d + chunk * d / 64 + dv + 8 * 6; }

// Workgroups of touch_ahead for the chain with tiles of 16 rows, one to a compute unit.  Such a workgroup has the chain's LDS and
// registers, so that the compute unit is not free for another stream: no more of them than half of those that the chain leaves idle,
// at d = 128 none where two such calls fit the chip side by side.  Whole forward, 4096 tokens, r = 2, inputs from HBM, us: one call after the other /
// a pair on two streams / a call of 6 heads x 1024 tokens, d = 64, on another stream, without, with half and with all:
//   d = 64, 24 heads               81 / 100 / 44    68 /  88 / 43    68 / 104 /  73
//           32                     87 / 111 / 45    71 / 104 / 45    71 / 115 /  77
//           40                     90 / 138 / 45    77 / 127 / 56    73 / 124 /  80
//           44                     94 / 143 / 46    88 / 152 / 57    78 / 132 /  85
//           24, d_v = 128          86 / 129 / 45    74 / 122 / 56    70 / 119 /  79
//           26, d_v = 128          89 / 138 / 46    89 / 142 / 91    76 / 132 /  83
//   d = 128, 16                   101 / 115 / 40    94 / 131 / 42    94 / 168 / 103
//            20                   105 / 151 / 41    98 / 149 / 52    98 / 174 / 107
//            24                   107 / 169 / 41    99 / 167 / 55    99 / 180 / 109
//            26                   111 / 188 / 42   113 / 203 / 127  102 / 187 / 113
// What one of them has to ask for during a block of the chain (0.5 us at d = 64, 0.75 at 128) bounds how few they may be: it has
// 128 lines on their way, some 225 a us from HBM, and the chain asks for a part itself.  Lines a block to each, and the gain: d = 64
// 204 (24 heads, d_v = 128) 14 %, 217 (13, d_v = 256) 5, 229 (44) 6 but 6 lost by the pair, 295 (26, d_v = 128) none; d = 128 153
// (20) 7 %, 276 (24) 8, 303 (13, d_v = 256, r = 1) 2, 334 (44, d_v = 64) 3 but 7 lost by the pair, 399 (26) -2.  Halves of rank 4 at
// d = 128: none (20 heads x 3000 145 / 145).  Fewer blocks: none (24 heads x 800 18.8 / 19.1).  And what lies in the window has to fit
// the XCDs' 4 MB of L2, which narrow d_v with many heads would not (140 heads, d_v = 16 122 / 127).
constexpr int ahead_workgroups(int cus, int heads, int d, int dv, int chunk, int blocks)
{
    const int works = heads * (dv / 16), some = (cus - works) / 2;
    if (blocks < 24 || (d == 64 ? 8 * works < 3 * cus : 2 * works <= cus || chunk < 32)) return 0;
    const long long lines = (long long)heads * ahead_lines(d, dv, chunk);
    return lines <= (d == 64 ? 205ll : 280ll) * some && lines / 8 * 128 * ahead_window(d) <= 4 << 20 ? some : 0;
}

// Whether the last wavefront of each workgroup of the chain with tiles of 16 rows at d = 128 asks for lines ahead of time, where no
// compute units do.  Not where a head has few tiles, so that the share of each is large, where workgroups are few, or blocks.
// P built in the chain, whole forward, 4096 tokens, r = 2, us, without / with: 64 heads, d_v = 32 130 / 147, 60 heads, d_v = 48
// 136 / 140; 32 heads, d_v = 64 117 / 112, d_v = 128 121 / 114; 12 heads x 700 32.5 / 33.1, 9 x 4096 from the last-level cache 87.2 / 87.3,
// 32 heads x 256 16.7 / 17.0.
// P handed over (the split entry points: more lines that it does not ask for), scan alone, inputs from HBM: 64 heads, d_v = 32 111 /
// 126, 60, d_v = 48 116 / 122, 32, d_v = 64 111.2 / 112.6, 32, d_v = 80 110.9 / 110.9, 32, d_v = 96 112 / 110, d_v = 128 112.5 / 108.6; 9 heads
// 104.9 / 100.8, 4 heads 79.5 / 79.8, 3, r = 1 57.2 / 59.2; 32 heads x 256 10.0 / 9.8.
constexpr bool ahead_wavefront(int cus, int heads, int dv, int blocks, bool handed_over)
{
    const int tiles = dv / 16, works = heads * tiles;
    return handed_over ? tiles >= 5 && works >= cus / 4 : tiles >= 4 && works >= cus / 2 && blocks >= 16;
}

}  // namespace pf

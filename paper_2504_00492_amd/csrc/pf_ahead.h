// Lines of the chain's later blocks that somebody asks for ahead of time (pf_chain.h): workgroups on compute units that the chain
// leaves idle (touch_ahead), or at d = 128 a wavefront of each of its own.  Plain arithmetic, so that it can be looked at without a GPU.
#pragma once

namespace pf {

// Blocks ahead of the chain that may be asked for (touch_ahead says what other numbers cost).
constexpr int ahead_window(int d) { return d == 64 ? 18 : 14; }

// A wavefront that has come to block b and last saw the chain at block `at` waits and looks again, or leaves block b out.
constexpr int kAheadLost = -0x40000000;          // (`at`: nobody watches the chain any more)
constexpr bool ahead_beyond(int b, int at, int window) { return b > at + window; }
constexpr bool ahead_late(int b, int at) { return b < at + 2; }

// 128-byte lines of a block (64 virtual tokens) of one head: K, Q, V and the six tiles of T
constexpr int ahead_lines(int d, int dv, int chunk) { return d + chunk * d / 64 + dv + 8 * 6; }

// Workgroups of touch_ahead for the chain with tiles of 16 rows, one to a compute unit.  Such a workgroup has the chain's LDS and
// registers, so that the compute unit is not free for another stream: no more of them than are of use.  Whole forward, 4096 tokens, r = 2, inputs from HBM, us: one call after the other / a pair on two
// streams / a call of 6 heads x 1024 tokens, d = 64, on another stream, without, as here, and with all idle compute units:
//   d = 64, 24 heads (56 of 160)             81 / 103 / 42     67 /  88 / 41     67 / 105 / 73
//           32 (72 of 128)                   87 / 109 / 44     71 / 108 / 42     71 / 117 / 77
//           40 (88 of 96)                    90 / 139 / 45     73 / 127 / 82     73 / 127 / 82
//           44 (all 80)                      94 / 145 / 46     77 / 132 / 86
//           24, d_v = 128 (all 64)           87 / 130 / 45     68 / 120 / 78
//           26, d_v = 128 (all 48)           90 / 139 / 46     75 / 133 / 86
//   d = 128, 16 (32 of 128)                 101 / 116 / 41     92 / 125 / 40     93 / 166 / 103
//            20 (40 of 96)                  105 / 149 / 41     97 / 147 / 40     97 / 174 / 108
//            24 (48 of 64)                  107 / 170 / 41     98 / 170 / 47     99 / 179 / 110
//            26 (all 48)                    112 / 188 / 42    101 / 185 / 115
//            28 (all 32)                    112 / 194 / 43    110 / 214 / 125
// How many are of use: 24 heads, d = 64 (4992 lines a block) 32 of them 69.0 us, 48 67.0, 160 66.9; 32 heads (6656) 32 77.9, 48 71.7, 64
// 70.8, 128 70.7; 20 heads, d = 128 (7360) 27 101, 32 96.7, 96 97.2.  So one for 100 lines or 220 of a block, in which a compute unit with 128
// lines on their way from HBM gets about as many (225 a us; 0.5 us at d = 64, 0.75 at 128), and eight at a time, one for each XCD.
// Halves of rank 4 take 0.6 us a block, one for 150 lines: 25 heads x 7263, d = 128 (56 of 56) 326 us, 40 of them 337, none 347.
// Where even all of them would have 350 lines each the gain ends: 54 heads, d = 64 (281) 101 / 169 / 48 without, 100 / 177 / 106 with; 28, d = 128
// (322) above.  Few blocks: 24 heads x 800, d = 64 18.8 / 19.1.
// Halves of rank 4, from HBM, without / with, one after the other, pairs: 16 heads x 8000, d = 128 327 / 324, 20 x 4096 303 / 296 (a pair),
// 24 x 3000 149 / 147, 262 / 289, 24 x 6000 275 / 264, 25 x 7263 347 / 326, 634 / 628, 40 x 3000, d_v = 64 169 / 158; 16 x 3000 140 / 142, 8 x 3001 137 /
// 139: from half of the compute units on (d = 64: three eighths).
// Rank 1 and 2 with fewer workgroups: from HBM the chain's own reads (Q among them since P is built there) hold it up as they do many; from an
// eighth of the compute units on.  At rank 2 it loses 1 % where the inputs lie in the 256 MB of the last-level cache: from 64 MB on, which
// hardly lie there whole.  3001 tokens, from the last-level cache ~ from HBM, without / with:
//   d = 128, r = 1   4 heads 52.0 ~ 58.3 / 49.9 ~ 51.0   12, d_v = 64 56.6 ~ 68.2 / 52.8 ~ 54.4   16, d_v = 32 55.1 ~ 65.1 / 53.3 ~ 54.8
//            r = 2   12 x 4096 87.6 ~ 102 / 88.6 ~ 90.9  8, d_v = 64 75.2 ~ 85.6 / 76.3 ~ 77.5    10 x 20001 467 ~ 482 / 405 ~ 408
//   d = 64,  r = 1   8 heads 35.7 ~ 42.4 / 34.7 ~ 35.2   16 38.7 ~ 48.4 / 36.8 ~ 37.5             10 x 20001 172 ~ 233 / 148 ~ 153
//            r = 2   8 heads 53.1 ~ 60.9 / 54.2 ~ 54.4   12 55.1 ~ 64.9 / 55.9 ~ 56.5
// and pairs on two streams, 4096 tokens, from HBM: d = 128 12 heads 125 / 115, r = 1 88 / 71, 8 heads 122 / 125, d = 64 12 heads 79 / 82, 16, r = 1 63 / 66.
// What lies in the window has to fit the XCDs' L2, 4 MB each, of which the chain has passed a part: to 5 MB.  From the last-level
// cache ~ from HBM, without / with: 60 heads, d = 128, d_v = 48, r = 1 (4.5 MB) 71 ~ 91 / 75 ~ 78; 110 heads, d = 64, d_v = 16, r = 2 (4.8)
// 96 ~ 103 / 93 ~ 97; 97 heads, r = 1 (5.1) 48 ~ 63 / 60 ~ 58; 130 heads, d = 128, d_v = 16, r = 1 (8.9) 103 ~ 112 / 124 ~ 122.
constexpr int ahead_workgroups(int cus, int heads, int d, int dv, int chunk, int blocks)
{
    const int works = heads * (dv / 16), idle = cus - works, full = d == 64 ? 100 : chunk < 32 ? 150 : 220;
    const long long lines = (long long)heads * ahead_lines(d, dv, chunk), need = (lines + 8 * full - 1) / (8 * full) * 8;
    const bool few = 8 * works < (d == 64 ? 3 : 4) * cus;
    if (blocks < 24 || 8 * works < cus || (few && (chunk < 32 || (chunk < 64 && lines * blocks * 128 < 64ll << 20)))) return 0;
    if (lines > 350ll * idle || lines / 8 * 128 * ahead_window(d) > 5 << 20) return 0;
    return need < idle ? (int)need : idle;
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

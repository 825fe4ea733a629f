// Body of the scan kernel for flow blocks of 64 virtual tokens (the delta rule): one wavefront runs the whole chain
// R -> U_eff -> S of 16 rows by itself, out of registers.  A workgroup has one tile of 16 rows or two (scan_chain, scan_two_tiles and
// scan_wide_chain in pf_scan.hip).
//
// With S^T as accumulator tiles (rows d_k, columns the 16 rows of S) every product of a block takes the result of
// the one before it as its B operand, and an accumulator tile is a B operand lane for lane (pf_common.h):
//     R     = beta (.) (V - K S^T)     A operand: rows of K             B: S^T (bf16 copy in registers)
//     U_eff = T R                      A operand: T tiles               B: R
//     S^T  += K^T U_eff                A operand: K^T, transposing read  B: U_eff
// so neither R, U_eff nor S passes through LDS on the chain, and the chain needs no barrier inside a block.  Row
// tiles of S^T are numbered so that lane group g of tiles 2 ks and 2 ks + 1 holds d_k = 32 ks + 8 g .. + 7: the
// joined pair then pairs with 16 consecutive bytes of a row of K.
//
// A workgroup has one such state wave per tile of 16 rows (one tile, or two) and helper waves.  Two of them (stagers) load K,
// the V tile and the T tiles of a later block straight into a ring of up to six LDS slots, two more (readers, where O is
// wanted; one where a block holds 16 tokens) compute the readout of the block before,
//     O^T = S Q^T + U_eff^T P^T,
// from the copies of S and U_eff that the state waves leave in LDS in operand form.  One barrier per block.
//
// The flow kernel of the same call hands over -T diag(beta), rounded once (FOLD): beta and its widening are gone from the
// state wave, and V enters as a product with -Id: 177 instructions a block at d = 128 where there were 235.  P is not handed
// over either: the readers hold Q of a block as operands and its K lies in the ring, so they build P of the block that the
// state is at, the same products in the same order.  The flow then reads K and beta and writes T (22 KB a block of d = 128,
// r = 2 instead of 33), the chain has 24 requests of 328 fewer.  Whole forward, us, P handed over / built: 32 heads x 65536,
// d = 128, r = 2 2068 / 1867 (flow 415 / 275, scan 1657 / 1595), 32 x 8192, r = 4 439 / 404, 24 x 4096, d = 64, d_v = 128, r = 2
// 98.9 / 89.4, 32 x 3001, r = 1 74.2 / 73.6 (its Q then comes from HBM in the scan).  The split entry points hand over T itself
// and P and take the form without either.
//
// What bounds it: the loads.  At d = 128 with the readout, 16 rows and 256 workgroups a block takes 0.78 us, because its 32 KB
// come in at 17 bytes a cycle (304 requests of 128 bytes, some 114 of them on their way); at d = 64 a block of
// 24 heads x 4096 tokens, d_v = 128, r = 2 takes 0.57 us.  A compute unit has at most about 128 L2 lines on their way: 12 bytes
// a cycle where they come from HBM, 20 from the last-level cache, 42 from L2: with every read from L2 a block takes 0.58 us.
// At d = 128 another wavefront (toucher) asks for lines ahead of time: 0.73 us.
//
// Two tiles to a workgroup (scan_two_tiles, scan_wide_chain and the segments) read K, Q, T, P once for 32 rows: a block takes
// hardly longer (0.98 us at d = 128, r = 2 and 256 workgroups; with every read from L2 0.75, which is LDS: some 165 KB a block).
// In rounds of one workgroup a compute unit it is ahead of the split of pf_scan.hip, two of which fit a compute unit, as well, since
// P is built here (64 heads x 4096 tokens, d = 128, r = 2: whole forward 181 us / 161; 128 heads 357 / 320).  Those calls take T
// itself: -T diag(beta) rounds a product that T R adds to exactly once more, 0.5 % further from 64 bits, and beta costs the
// state waves 1 % of the time.  Nor does V enter as a product with -Id there, so that O and S_L are the split's, bit for bit.
// With 128 virtual tokens a block the operands of one wave do not fit its registers: blocks of rank 4 run as two halves (32
// heads x 8192 tokens, r = 4 529 -> 436 us).
#pragma once
#include "pf_ahead.h"
#include "pf_common.h"
#include "pf_internal.h"
#include "pf_layout.h"

namespace pf {

// K lies in LDS without padding, its 16-byte units permuted within a row (position = unit ^ swizzle of the row) so
// that 16 rows at one unit (row operand) and 4 rows at 4 neighbouring units (transposing read) both touch
// distinct banks.  With rows padded by 16 bytes the transposing reads were four-way conflicts.
template <int D>
__device__ __forceinline__ int k_swizzle(int row)
{
    static_assert(D == 64 || D == 128, "16-byte units per row");
    return D == 128 ? ((row & 3) << 2) | ((row >> 2) & 3) : (((row >> 1) & 1) << 2) | ((row >> 2) & 3);
}

// PAIR (state only): two sets of TV rows of one segment, the rows of its state from zero with V and the rows of its
// propagator, from the identity, without: they have a zero tile in LDS for V (so that an infinity in V stays out of the
// propagator).  Both read the same K and T, which a workgroup loads once: with two tiles, a state wave per SIMD, a block
// takes 1.0 us where the two passes took 0.7 us each (4 heads x 32768 tokens, d = 128, r = 2: 2 x 44.8 us -> 2 x 35.7 for
// half of the blocks each); what bounds it is LDS, four waves reading 42 KB a block each.  Whole forward, us, passes one
// after the other / PAIR:
//   d = 128, r = 2   4 heads x 32768  180 / 163    8 x 65536  685 / 570    1 x 131072  224 / 205    8 x 8192  97 / 87
//   d = 64           16 x 65536, r = 2  645 / 542    2 x 65536, r = 1  84 / 72    8 x 2048, r = 1  33.0 / 28.7
template <int D, int N, int C, int TV, bool RO, bool PAIR = false>
struct ChainPlan {
    static constexpr int states = (PAIR ? 2 : 1) * (TV / 16), stagers = 2, readers = !RO ? 0 : (C >= 32 ? 2 : 1);   // wavefronts of each role
    static constexpr int touchers = RO && D == 128 && TV == 16 ? 1 : 0;
    static constexpr int threads = 64 * (states + readers + stagers + touchers);
    static constexpr int NT = t_tile_count(N / 16);    // T tiles of a block
    // one ring slot: K, V tile, T tiles, beta (32 bits each)
    static constexpr size_t oV = (size_t)N * D * 2;
    static constexpr size_t oT = oV + (size_t)N * TV * 2;
    static constexpr size_t oB = oT + (size_t)NT * 1024;
    static constexpr size_t slot = oB + (size_t)N * 4;
    static constexpr size_t szX = RO ? (size_t)states * (D / 32) * 1024 : 0;   // S of a block, operand tiles
    static constexpr size_t szU = RO ? (size_t)states * (N / 32) * 1024 : 0;   // U_eff of a block, operand tiles
    // two slots are being read (this block, and the rows and T of the next), the others are on their way from memory
    static constexpr size_t szZ = PAIR ? (size_t)N * TV * 2 : 0;
    static constexpr size_t szW = touchers ? 256 : 0;   // what the toucher's loads bring, for nobody
    static constexpr int fit = (int)((kMaxLdsBytes - 2 * (szX + szU) - szZ - szW) / slot);
    static constexpr int kRing = fit < 6 ? fit : 6;
    static constexpr size_t oX = kRing * slot;
    static constexpr size_t oU = oX + 2 * szX;
    static constexpr size_t oZ = oU + 2 * szU;
    static constexpr size_t oW = oZ + szZ;
    static constexpr size_t total = oW + szW;
    static_assert(!(PAIR && RO), "a propagator has no readout");
    static constexpr bool kServes = N == 64 && (TV == 16 || TV == 32) && kRing >= 4;
};

// 16 bytes (4; 2, widened to 32 bits) per lane from memory to LDS; the LDS address is the wavefront's, lane l
// writes behind lane l - 1.
__device__ __forceinline__ void load_lds16(const bf16 *src, char *dst)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                     (__attribute__((address_space(3))) void *)(uintptr_t)(uint32_t)(uintptr_t)dst, 16, 0, 0);
}
__device__ __forceinline__ void load_lds4(const char *src, char *dst)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                     (__attribute__((address_space(3))) void *)(uintptr_t)(uint32_t)(uintptr_t)dst, 4, 0, 0);
}
__device__ __forceinline__ void load_lds2(const bf16 *src, char *dst)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                     (__attribute__((address_space(3))) void *)(uintptr_t)(uint32_t)(uintptr_t)dst, 2, 0, 0);
}

// A workgroup beyond those of the chain, on a compute unit that they leave idle: asks for the lines of the blocks that the heads of
// its XCD come to next, four bytes a line that nobody waits for, so that the chain finds them in L2 (a compute unit's reads come
// back in order: its own wait for memory holds up the chain's, another's does not).  What bounds it: 128 lines on their way at a time.
// Its first wavefront looks how far the chain is, until the rest of it is within the window; nothing but time depends on that.  The
// others look there when they are through the window that they last saw (at every block, or going on in its middle once late, they are up
// to 10 % slower: 16 heads x 64967 tokens, d = 64, d_v = 192, r = 2 963 us, so 880), and leave out what the chain had come to then;
// once the first has seen no progress for some 3 ms, they leave.  Who waits for the first ends with it: it leaves when no block is
// beyond the window, or says that it has lost the chain.
// The window: what lies ahead of the chain has to fit an XCD's 4 MB of L2.  Whole forward, us, without / 8, 12, 18 and 24 blocks:
//   24 heads x 4096, d = 64, r = 2  77.4 / 74.5, 66.4, 65.1, 65.3     20 x 4096, d = 128, r = 2  104 / 99.8, 95.9, 96.4, 96.8
template <int D, int N, int C, int kRing>
__device__ __forceinline__ void touch_ahead(const bf16 *Q, const bf16 *K, const bf16 *V, const bf16 *Tt, unsigned *pace,
                                            unsigned works, unsigned tiles, int NC, int tail, int dv, char *smem)
{
    constexpr int R = N / C, NKT = N / 32, NT = t_tile_count(N / 16);
    constexpr int kWindow = ahead_window(D), kPatience = 4096;
    const unsigned x = blockIdx.x & 7, each = works >> 3, more = works & 7;
    const unsigned count = each + (x < more), first = x * each + (x < more ? x : more);
    const unsigned groups = (gridDim.x >> 3) + (x < (gridDim.x & 7)) - count, group = (blockIdx.x >> 3) - count;
    volatile int *const seen = reinterpret_cast<volatile int *>(smem + 256);   // (the loads write below)
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), waves = blockDim.x >> 6, lane = threadIdx.x & 63;
    if (threadIdx.x == 0) *seen = 0;
    __syncthreads();
    if (count == 0) return;
    if (wave == 0) {
        int last = 0;                                      // until the rest of the chain is within the window
        for (int idle = 0; last < NC - kWindow; ++idle) {
            if (idle == kPatience) {
                *seen = kAheadLost;
                return;
            }
            const int now = (int)__hip_atomic_load(pace, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (now > last) {
                last = now;
                idle = 0;
                *seen = last;
            }
            __builtin_amdgcn_s_sleep(4);
        }
        return;
    }
    constexpr int KL = N * D / 64, QL = C * D / 64, TL = 8 * NT;
    const unsigned h0 = first / tiles, heads = (first + count - 1) / tiles - h0 + 1;
    const int VL = N * dv / 64, lines = KL + QL + TL + VL;
    int at = kRing - kWindow;                              // (so that a workgroup that starts late looks after its first block)
    for (int b = kRing; b < NC; ++b) {
        while (ahead_beyond(b, at, kWindow)) {
            // (the plain read waits for all that is on its way to LDS first, which pays with the many lines of r = 1: 30 heads x 34581
            // tokens, d = 64, d_v = 96 319 us, else 330; with r = 2, 35 heads x 38963, d = 64 623, else 586, r = 4, 30 x 10624 310 / 297)
            if constexpr (C < 64) asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(at) : "v"((uint32_t)(uintptr_t)(smem + 256)) : "memory");
            else at = *seen;
            if (at == kAheadLost) {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                return;
            }
            if (ahead_beyond(b, at, kWindow)) __builtin_amdgcn_s_sleep(2);
        }
        if (ahead_late(b, at)) continue;
        for (unsigned i = ((wave - 1) * groups + group) * 64 + lane; i < heads * lines; i += (waves - 1) * groups * 64) {
            const size_t head = h0 + i / lines, cid = head * (size_t)NC + b, skew = head * (size_t)tail;
            int l = i % lines;
            const char *a;
            if (l < KL) a = reinterpret_cast<const char *>(K + cid * N * D + skew * R * D) + 128 * l;
            else if ((l -= KL) < VL) a = reinterpret_cast<const char *>(V + (cid * N + skew * R) * dv) + 128 * l;
            else if ((l -= VL) < QL) a = reinterpret_cast<const char *>(Q + cid * C * D + skew * D) + 128 * l;
            else {
                l -= QL;
                const int t = l >> 3, mt = t < 1 ? 0 : t < 2 ? 1 : t < 4 ? 2 : 3;
                a = reinterpret_cast<const char *>(Tt + cid * N * N + full_tile_offset(NKT, mt, t - t_tile_index(mt, 0))) + 128 * (l & 7);
            }
            load_lds4(a, smem);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // nothing is under way to LDS when the wave ends
}

// FOLD: Tt holds -T diag(beta) (launch_chunk_flow), so that the chain takes K S^T - V as it comes out of the products: no
// beta, no factor, and V goes in as a product with -Id.
// PAIR: `stride` blocks a chain, of which this call takes NC from `first` on.  The rows of the state are in and out at SL, those
// of the propagator at SP; from the first block on they start as zeros and as the identity.
// BUILD: P is built by the readers, else Pt holds it.
template <int D, int N, int C, int TV, bool RO, bool FOLD, bool PAIR = false, bool BUILD = FOLD>
__device__ __forceinline__ void chain_scan(const bf16 *Q, const bf16 *K, const bf16 *V, const bf16 *beta,
                                           const bf16 *Tt, const bf16 *Pt, const float *S0, bf16 *O, float *SL,
                                           int nchains, int NC, int tail, int dv, char *smem,
                                           float *SP = nullptr, int stride = 0, int first = 0)
{
    using Pl = ChainPlan<D, N, C, TV, RO, PAIR>;
    constexpr int NT = Pl::NT, kRing = Pl::kRing;
    constexpr int R = N / C, NKS = D / 32, NKT = N / 32, MT = N / 16, MD = D / 16, CT = C / 16;
    constexpr int NSS = Pl::states, NSt = Pl::stagers;
    // T itself and P built here: calls that the split of pf_scan.hip had.  R comes out in its order, V - K S^T with the sum of the
    // products first and the difference on the vector ALU: every bit of O and S_L is what the split gives.  (With -V in the first
    // product they were 1.2e-3 apart on 64 heads x 4096 tokens, d = 128, r = 2, with -V in the last as well; 159.6 us in each.)
    constexpr bool kVLast = BUILD && !FOLD;

    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63, r16 = lane & 15, g = lane >> 4;
    const unsigned tiles = (unsigned)dv / TV, works = (unsigned)nchains * tiles;
    // FOLD, one tile to a workgroup: how far the first workgroup of each XCD is, 32 words apart, is kept where P would be (written
    // to the XCD's L2, by the state wave, which has no other access to memory to wait for; by a reader, whose reads of Q then waited
    // for it, at every block of every workgroup and through to memory, 24 heads x 4096, d_v = 128 took 333 us instead of 73)
    constexpr bool kPaced = RO && FOLD && TV == 16;
    unsigned *const pace = kPaced ? reinterpret_cast<unsigned *>(const_cast<bf16 *>(Pt)) + 32 * (blockIdx.x & 7) : nullptr;
    if constexpr (kPaced) {
        // (behind the chain's code: in front of it a scan without such workgroups, 32 heads x 65536 tokens, d = 128, r = 2, took 7 us more)
        if (__builtin_expect(blockIdx.x >= works, 0))
            return touch_ahead<D, N, C, Pl::kRing>(Q, K, V, Tt, pace, works, tiles, NC, tail, dv, smem);
    }
    const bool paces = kPaced && blockIdx.x < 8 && gridDim.x > works;
    const unsigned work = xcd_consecutive(blockIdx.x, works);
    const int tile = work % tiles;                     // the tiles of a head: one XCD
    const size_t chain = work / tiles;
    const size_t c0 = PAIR ? chain * (size_t)stride + (size_t)first : chain * (size_t)NC;
    // `tail` tokens of every head belong to another kernel
    Q += chain * (size_t)tail * D;
    K += chain * (size_t)tail * R * D;
    V += chain * (size_t)tail * R * dv + tile * TV;
    beta += chain * (size_t)tail * R;
    bf16 *Xs = reinterpret_cast<bf16 *>(smem + Pl::oX), *Us = reinterpret_cast<bf16 *>(smem + Pl::oU);
    constexpr int XB = (int)(Pl::szX / 2), UB = (int)(Pl::szU / 2);   // elements of one buffer

    if (wave < NSS) {
        // -------------------------------------------------------------- state waves, 16 rows each
        __builtin_amdgcn_s_setprio(3);                 // the helpers of this SIMD fill what the chain leaves
        auto dk0 = [&](int mt) { return 32 * (mt >> 1) + 8 * g + 4 * (mt & 1); };
        const bool prop = PAIR && wave >= NSS / 2;         // rows of the propagator
        const int rowt = PAIR ? wave % (NSS / 2) : wave;   // 16 rows of the tile
        const int row = tile * TV + 16 * rowt + r16;
        const size_t srow = (size_t)row * D;
        float *const out = prop ? SP : SL;
        f32x4 sacc[MD];
#pragma unroll
        for (int mt = 0; mt < MD; ++mt) {
            sacc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
            if constexpr (PAIR) {
                if (first) sacc[mt] = *reinterpret_cast<const f32x4 *>(out + chain * (size_t)dv * D + srow + dk0(mt));
                else if (prop) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) sacc[mt][e] = dk0(mt) + e == row ? 1.0f : 0.0f;
                }
            } else if (S0) sacc[mt] = *reinterpret_cast<const f32x4 *>(S0 + chain * (size_t)dv * D + srow + dk0(mt));
        }
        // byte offsets in a slot: row operand of K by k-step, transposing read of K by pair of d_k tiles
        int kr0[NKS], kt0[NKS];
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
            kr0[ks] = r16 * D * 2 + ((4 * ks + g) ^ k_swizzle<D>(r16)) * 16;
            kt0[ks] = (4 * g + (r16 >> 2)) * D * 2 + ((4 * ks + (r16 & 3)) ^ k_swizzle<D>(4 * g + (r16 >> 2))) * 16;
        }
        const int vt0 = (int)(prop ? Pl::oZ : Pl::oV) + ((4 * g + (r16 >> 2)) * TV + 16 * rowt + 4 * (r16 & 3)) * 2;
        if constexpr (PAIR) {
            if (prop) {
#pragma unroll
                for (int i = 0; i < N / 16; ++i)           // the columns of V that this wave reads
                    *reinterpret_cast<u32x2 *>(smem + vt0 + 16 * i * TV * 2) = u32x2{0, 0};
            }
        }
        const int tt0 = (int)Pl::oT + lane * 16, bt0 = (int)Pl::oB + 16 * g;
        auto at8 = [&](int off) { return *reinterpret_cast<const bf16x8 *>(smem + off); };

        // Operands of a block are read from its slot ahead of their use: K^T during R, rows of K, V, beta and T of the
        // next block during the update of S.  The order below is the order of issue (kInOrder keeps the compiler from
        // gathering the reads behind the products): every LDS read and every conversion lies in the shadow of products.
        // Reads gathered at the end of a block cost 0.1 us a block.
#define kInOrder() __builtin_amdgcn_sched_barrier(0)
        constexpr int NM = NKT * MD;                   // products of R, and of the update
        static_assert(NM == MT * NKS && MT == 4, "one operand of K^T is read per product of R");
        bf16x8 aK[MT][NKS], tA[NT], aT[NKT][MD];
        bf16x4 vt[MT];
        u32x4 bt[FOLD ? 1 : MT];                       // bf16 in the low half
        f32x4 bw[FOLD ? 1 : MT];                       // beta, widened
        bf16x8 nI[2];                                  // -Id on the first, on the second half of a k-step
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 8; ++e) nI[h][e] = (bf16)(e / 4 == h && 4 * g + (e & 3) == r16 ? -1.0f : 0.0f);
        auto read_kt = [&](int base, int i) {
            const int kt = i / MD, mt = i % MD;
            const bf16 *p = reinterpret_cast<const bf16 *>(smem + base + kt0[mt >> 1] + 32 * kt * D * 2 + 8 * (mt & 1));
            aT[kt][mt] = join(lds_read_tr4(p), lds_read_tr4(p + 16 * D));
        };
        constexpr int kVB = FOLD ? MT : 2 * MT, kAhead = kVB + MT * NKS + NT, kPer = (kAhead + NM - 1) / NM;
        auto read_ahead = [&](int base, int i) {
            if (i < MT) vt[i] = lds_read_tr4(reinterpret_cast<const bf16 *>(smem + (prop ? 0 : base) + vt0 + 16 * i * TV * 2));
            else if (i < kVB) bt[FOLD ? 0 : i - MT] = *reinterpret_cast<const u32x4 *>(smem + base + bt0 + 64 * (i - MT));
            else if (i < kVB + MT * NKS) {
                const int mt = (i - kVB) / NKS, ks = (i - kVB) % NKS;
                aK[mt][ks] = at8(base + kr0[ks] + 16 * mt * D * 2);
            } else if (i < kAhead) tA[i - kVB - MT * NKS] = at8(base + tt0 + (i - kVB - MT * NKS) * 1024);
        };
        auto widen = [&](int mt) {
            if constexpr (FOLD) return;
            bw[mt] = __builtin_bit_cast(f32x4, bt[mt] << 16);
            asm volatile("" : "+v"(bw[mt]));               // here, not at the use
        };
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kAhead; ++i) read_ahead(0, i);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) widen(mt);

        int slot = 0;
#pragma unroll 1
        for (int ch = 0; ch < NC; ++ch) {
            const int base = slot * (int)Pl::slot;
            slot = slot == kRing - 1 ? 0 : slot + 1;
            const int ahead = slot * (int)Pl::slot;    // (after the last block: some slot, not used)
            bf16x8 bS[NKS], bR[NKT], bU[NKT];
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) bS[ks] = join(cvt4(sacc[2 * ks]), cvt4(sacc[2 * ks + 1]));
            kInOrder();
            // ---- R = beta (.) (V - K S^T), from K S^T - V (or K S^T: kVLast); the first pair of row tiles is finished inside the second
            f32x4 acc[MT], u[MT];
            auto epilogue = [&](int kt) {
                if constexpr (FOLD) bR[kt] = join(cvt4(acc[2 * kt]), cvt4(acc[2 * kt + 1]));
                else if constexpr (kVLast) {
                    auto row = [&](int mt) { return cvt4((__builtin_convertvector(vt[mt], f32x4) - acc[mt]) * bw[mt]); };
                    bR[kt] = join(row(2 * kt), row(2 * kt + 1));
                } else bR[kt] = join(cvt4(acc[2 * kt] * -bw[2 * kt]), cvt4(acc[2 * kt + 1] * -bw[2 * kt + 1]));
            };
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
                if constexpr (!kVLast) acc[mt] = mfma16(nI[mt & 1], join(vt[mt & ~1], vt[mt | 1]), acc[mt]);
            }
#pragma unroll
            for (int i = 0; i < NM; ++i) {
                const int mt = 2 * (i / (2 * NKS)) + (i & 1), ks = (i / 2) % NKS;
                acc[mt] = mfma16(aK[mt][ks], bS[ks], acc[mt]);
                read_kt(base, i);
                if constexpr (RO)
                    if (i < NKS) st8(&Xs[(ch & 1) * XB + (wave * NKS + i) * 512 + lane * 8], bS[i]);
                if (i == 2 * NKS + NKS - 1) epilogue(0);
                kInOrder();
            }
            // ---- U_eff = T R, lower block-triangular
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) u[mt] = mfma16(tA[t_tile_index(mt, 0)], bR[0], f32x4{0.f, 0.f, 0.f, 0.f});
            kInOrder();
            epilogue(1);
            kInOrder();
#pragma unroll
            for (int mt = 2; mt < MT; ++mt) u[mt] = mfma16(tA[t_tile_index(mt, 1)], bR[1], u[mt]);
            bU[0] = join(cvt4(u[0]), cvt4(u[1]));
            kInOrder();
            // ---- S^T += K^T U_eff
#pragma unroll
            for (int i = 0; i < NM; ++i) {
                const int kt = i / MD, mt = i % MD;
                if (i == MD) bU[1] = join(cvt4(u[2]), cvt4(u[3]));
                sacc[mt] = mfma16(aT[kt][mt], bU[kt], sacc[mt]);
                if constexpr (RO)
                    if (mt == 0) st8(&Us[(ch & 1) * UB + (wave * NKT + kt) * 512 + lane * 8], bU[kt]);
#pragma unroll
                for (int q = 0; q < kPer; ++q) read_ahead(ahead, kPer * i + q);
                if (kt == 1 && mt % (MD / MT) == 0) widen(mt / (MD / MT));
                kInOrder();
            }
            if constexpr (kPaced) {
                // (at d = 128 every fourth block: at every one 25 heads x 4000 tokens, r = 4 took 173 us instead of 170, 12 x 4096, r = 2 from the
                // last-level cache 89.5 instead of 88.6; at d = 64 24 x 4096, r = 2 66.5, with every fourth 66.7)
                if (paces && (D == 64 || ch % 4 == 0)) __hip_atomic_store(pace, (unsigned)ch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            __syncthreads();
        }
#undef kInOrder
        if (out) {
#pragma unroll
            for (int mt = 0; mt < MD; ++mt)
                *reinterpret_cast<f32x4 *>(out + chain * (size_t)dv * D + srow + dk0(mt)) = sacc[mt];
        }
        return;
    }

    // ------------------------------------------------------------------ helper waves
    // Blocks in groups of one per register set of the readers, without a branch inside: a branch around a load or store makes
    // every later wait assume the shorter queue.
    constexpr int kSets = BUILD ? 4 : 3;                              // blocks of Q (and P) on their way in register sets
    auto for_blocks = [&](auto f) {
        int ch = 0;
#pragma unroll 1
        for (; ch + kSets <= NC; ch += kSets) {
            f(ch, std::integral_constant<int, 0>{});
            f(ch + 1, std::integral_constant<int, 1>{});
            f(ch + 2, std::integral_constant<int, 2>{});
            if constexpr (kSets == 4) f(ch + 3, std::integral_constant<int, 3>{});
        }
        if (ch < NC) f(ch, std::integral_constant<int, 0>{});
        if (ch + 1 < NC) f(ch + 1, std::integral_constant<int, 1>{});
        if constexpr (kSets == 4) {
            if (ch + 2 < NC) f(ch + 2, std::integral_constant<int, 2>{});
        }
    };
    auto clamp = [&](int ch) { return c0 + (size_t)(ch < NC ? ch : NC - 1); };

    // A workgroup's wavefronts go round the four SIMDs: the readers, who have products of their own, come right behind the state
    // waves, and the stagers share what SIMDs are left to share.
    constexpr int NRd = Pl::readers;
    // The barrier alone, without the wait for every load that __syncthreads brings; to the compiler it does not touch
    // memory, so the fences keep the loads of a later block, which reuse a slot, behind it.
    auto barrier = [&] {
        LDS_FENCE();
        __builtin_amdgcn_s_barrier();
        LDS_FENCE();
    };
    if (Pl::touchers && wave >= NSS + NRd + NSt) {
        // The tiles of a head read the same lines at the same time, so that no more of them are on their way from memory than one
        // of them asks for.  Each asks for its share of a later block's lines of K, V and Q as well, four bytes a line that
        // nobody waits for: the block's own loads then find them in L2.  Scan, us, without / five to seven blocks ahead / fourteen:
        // 32 heads x 65536, r = 2 1606 / 1500 / 1616; 32 x 3001, r = 1 55.5 / 52.9 / 52.6; 32 x 8192, r = 4 340 / 336 / 348.
        // Only V and Q: 1633, 52.1, 347.  With two tiles to a workgroup (64 heads x 4096, r = 2 131 / 142) and at d = 64, where a
        // block is shorter than the wait for memory (32 x 2048, r = 1 19.1 / 20.0; 24 x 4096, d_v = 128 72.7 / 72), there is none.
        constexpr int kTouch = 7, KL = N * D / 64, QL = C * D / 64;
        const int ntiles = dv / TV, VL = N * dv / 64, lines = KL + QL + VL;
        auto touch = [&](int ch) {
            const size_t cid = c0 + (size_t)ch;
            const char *Kg = reinterpret_cast<const char *>(K + cid * (size_t)N * D);
            const char *Qg = reinterpret_cast<const char *>(Q + cid * (size_t)C * D);
            const char *Vg = reinterpret_cast<const char *>(V - tile * TV + cid * (size_t)N * dv);
            for (int first = tile; first < lines; first += 64 * ntiles) {
                const int i = first + lane * ntiles;
                if (i < lines)
                    load_lds4(i < KL ? Kg + 128 * i : i < KL + QL ? Qg + 128 * (i - KL) : Vg + 128 * (i - KL - QL), smem + Pl::oW);
            }
        };
        for (int b = kRing - 1; b < kTouch && b < NC; ++b) touch(b);   // (the stagers ask for those before)
        barrier();
#pragma unroll 1
        for (int ch = 0; ch < NC; ++ch) {
            if (ch + kTouch < NC) touch(ch + kTouch);
            barrier();
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // nothing is under way to LDS when the wave ends
        return;
    }
    if (wave >= NSS + NRd) {
        // The stagers' loads go straight to LDS.  Pieces of 64 x 16 bytes, dealt to the stagers one by one.
        const int H = wave - NSS - NRd;
        constexpr int VPR = D / 8, PPR = TV / 8;                     // 16-byte units per row of K, of the V tile
        constexpr int KQ = N * VPR / 64 / NSt, VQ = N * PPR / 64 / NSt, TQ = NT / NSt;
        constexpr int kLoads = KQ + VQ + TQ + (FOLD ? 0 : 1);                     // loads of a stager per block
        static_assert(N * VPR % (64 * NSt) == 0 && N * PPR % (64 * NSt) == 0 && NT % NSt == 0 && N == 64, "whole pieces");
        static_assert((kRing - 3) * kLoads < 64, "vmcnt");
        int ksrc[KQ], vsrc[VQ], tsrc[TQ];
#pragma unroll
        for (int q = 0; q < KQ; ++q) {
            const int v = (H + NSt * q) * 64 + lane, row = v / VPR;
            ksrc[q] = row * D + ((v % VPR) ^ k_swizzle<D>(row)) * 8;
        }
#pragma unroll
        for (int q = 0; q < VQ; ++q) {
            const int v = (H + NSt * q) * 64 + lane;
            vsrc[q] = (v / PPR) * dv + (v % PPR) * 8;
        }
#pragma unroll
        for (int q = 0; q < TQ; ++q) {                               // the tiles that exist, row by row
            int mt = 0;
            while (t_tile_index(mt + 1, 0) <= H + NSt * q) ++mt;
            tsrc[q] = (int)full_tile_offset(NKT, mt, H + NSt * q - t_tile_index(mt, 0)) + lane * 8;
        }
        auto fetch = [&](int ch, int slot) {                         // (beyond the last block: the last once more)
            const size_t cid = clamp(ch);
            char *d = smem + slot * (int)Pl::slot;
            const bf16 *Kg = K + cid * (size_t)N * D, *Vg = V + cid * (size_t)N * dv, *Tg = Tt + cid * (size_t)N * N;
#pragma unroll
            for (int q = 0; q < KQ; ++q) load_lds16(Kg + ksrc[q], d + (H + NSt * q) * 1024);
#pragma unroll
            for (int q = 0; q < VQ; ++q) load_lds16(Vg + vsrc[q], d + Pl::oV + (H + NSt * q) * 1024);
#pragma unroll
            for (int q = 0; q < TQ; ++q) load_lds16(Tg + tsrc[q], d + Pl::oT + (H + NSt * q) * 1024);
            if constexpr (!FOLD) load_lds2(beta + cid * (size_t)N + lane, d + Pl::oB);    // both stagers: the same values to the same place
        };
        // Loads return in order: all but the newest n blocks have landed.
        auto landed_but = [&](auto Nc) {
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(decltype(Nc)::value * kLoads) : "memory");
        };
        if (NC > 0) {
#pragma unroll
            for (int b = 0; b < kRing - 1; ++b) fetch(b, b);
            landed_but(std::integral_constant<int, kRing - 3>{});
        }
        barrier();
        int slot = kRing - 1;
        // During block ch: request block ch + kRing - 1 into the slot that block ch - 1 left; blocks up to ch + 2 have
        // landed at its end, because the state wave reads the rows of block ch + 2 during block ch + 1.
#pragma unroll 1
        for (int ch = 0; ch < NC; ++ch) {
            fetch(ch + kRing - 1, slot);
            slot = slot == kRing - 1 ? 0 : slot + 1;
            landed_but(std::integral_constant<int, kRing - 3>{});
            barrier();
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // nothing is under way to LDS when the wave ends
        return;
    }

    // readers: token tiles w and CT - 1 - w (of two tiles: w; of one: one reader), a block behind the state.  BUILD: P of the
    // block that the state is at is built from the rows of K in its slot and the Q in registers, else it comes from memory.
    auto reader = [&](auto Wc) {
        constexpr int W = decltype(Wc)::value, TN = CT < 2 ? 1 : CT / 2;
        constexpr auto tok_tile = [](int i) constexpr { return i == 0 ? W : CT - 1 - W; };
        bf16x8 bQ[kSets][TN][NKS], bP[BUILD ? 1 : kSets][TN][NKT];    // (P tiles above the causal mask do not exist)
        auto fetch = [&](int ch, auto Sc) {
            constexpr int S = decltype(Sc)::value;
            const size_t cid = clamp(ch);
#pragma unroll
            for (int i = 0; i < TN; ++i) {
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks)
                    bQ[S][i][ks] = ld8(Q + cid * (size_t)C * D + (16 * tok_tile(i) + r16) * D + 32 * ks + 8 * g);
#pragma unroll
                for (int kt = 0; kt < NKT; ++kt)
                    if (!BUILD && kt < p_ksteps(R, tok_tile(i)))
                        bP[BUILD ? 0 : S][i][kt] = ld8(Pt + cid * (size_t)C * N + full_tile_offset(NKT, tok_tile(i), kt) + lane * 8);
            }
        };
        int kr0[NKS];                                                // row operand of K by k-step (as the state waves')
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) kr0[ks] = r16 * D * 2 + ((4 * ks + g) ^ k_swizzle<D>(r16)) * 16;
        // P = Mbar (.) Q K^T of the block in `base`, from K Q^T: two accumulator tiles, one upon the other, are a tile of P
        auto build = [&](int base, auto Sc) {
            constexpr int S = decltype(Sc)::value;
            constexpr int last = TN > 1 && tok_tile(TN - 1) > tok_tile(0) ? tok_tile(TN - 1) : tok_tile(0);
            f32x4 p[TN][MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                if (16 * mt >= R * (16 * last + 16)) continue;       // later than the last of the tokens
                bf16x8 k[NKS];
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks) k[ks] = ld8(reinterpret_cast<const bf16 *>(smem + base + kr0[ks] + 16 * mt * D * 2));
#pragma unroll
                for (int i = 0; i < TN; ++i) {
                    const int tt = tok_tile(i);
                    if (16 * mt >= R * (16 * tt + 16)) continue;
                    p[i][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ks = 0; ks < NKS; ++ks) p[i][mt] = mfma16(k[ks], bQ[S][i][ks], p[i][mt]);
                    if (16 * mt + 15 >= R * 16 * tt) {               // readout mask, inclusive in time
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            p[i][mt][e] = (16 * mt + 4 * g + e) / R > 16 * tt + r16 ? 0.0f : p[i][mt][e];
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int kt = 0; kt < NKT; ++kt)
                    if (kt < p_ksteps(R, tok_tile(i))) {
                        const bool both = 16 * (2 * kt + 1) < R * (16 * tok_tile(i) + 16);
                        bP[0][i][kt] = join(cvt4(p[i][2 * kt]), both ? cvt4(p[i][2 * kt + 1]) : cvt4(f32x4{0.f, 0.f, 0.f, 0.f}));
                    }
        };
        auto sets = [&](auto f) {
            f(0, std::integral_constant<int, 0>{});
            f(1, std::integral_constant<int, 1>{});
            f(2, std::integral_constant<int, 2>{});
            if constexpr (kSets == 4) f(3, std::integral_constant<int, 3>{});
        };
        if (NC > 0) sets(fetch);
        __syncthreads();
        if constexpr (BUILD) {
            if (NC > 0) build(0, std::integral_constant<int, 0>{});
        }
        int slot = 0;
        for_blocks([&](int ch, auto Sc) {
            constexpr int S = decltype(Sc)::value;
            __syncthreads();
            slot = slot == kRing - 1 ? 0 : slot + 1;                 // of block ch + 1 (beyond the last block: not used)
            bf16 *Oc = O + chain * (size_t)tail * dv + ((c0 + ch) * (size_t)C + r16) * dv + tile * TV + 4 * g;
            const bf16 *X = Xs + (ch & 1) * XB + lane * 8, *U = Us + (ch & 1) * UB + lane * 8;
            f32x4 o[NSS][TN];
#pragma unroll
            for (int w = 0; w < NSS; ++w) {
                bf16x8 x[NKS], u[NKT];
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks) x[ks] = ld8(X + (w * NKS + ks) * 512);
#pragma unroll
                for (int kt = 0; kt < NKT; ++kt) u[kt] = ld8(U + (w * NKT + kt) * 512);
#pragma unroll
                for (int i = 0; i < TN; ++i) {
                    o[w][i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ks = 0; ks < NKS; ++ks) o[w][i] = mfma16(x[ks], bQ[S][i][ks], o[w][i]);
#pragma unroll
                    for (int kt = 0; kt < NKT; ++kt)
                        if (kt < p_ksteps(R, tok_tile(i))) o[w][i] = mfma16(u[kt], bP[BUILD ? 0 : S][i][kt], o[w][i]);
                }
            }
            LDS_FENCE();
            fetch(ch + kSets, Sc);
            LDS_FENCE();
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int w = 0; w < NSS; ++w) st4(Oc + (size_t)16 * tok_tile(i) * dv + 16 * w, cvt4(o[w][i]));
            LDS_FENCE();
            if constexpr (BUILD) build(slot * (int)Pl::slot, std::integral_constant<int, (S + 1) % kSets>{});
        });
    };
    if constexpr (RO) {
        if (NRd == 1 || wave == NSS) reader(std::integral_constant<int, 0>{});
        else if constexpr (NRd == 2) reader(std::integral_constant<int, 1>{});
    }
}

}  // namespace pf

// Body of the generic kernel for more than a few tokens of rows up to 128 wide: the recurrence 16 virtual tokens at a
// time in the form of Theorem 3.2, every product on the fp32 matrix instruction (v_mfma_f32_16x16x4_f32).
//
//   delta rule   R = beta (.) (V - K S^T),  U = T R,  S^T += K^T U,  O^T = S Q^T + U^T P^T,  T = (Id + M (.) diag(beta) K K^T)^{-1}
//   drivers      R = Atil + A S^T,          U = T R,  S^T += B^T U,  O^T = S Q^T + U^T P^T,  T = (Id - M (.) A B^T)^{-1}
//
// and P = Mbar (.) Q K^T (Q B^T), with the masks in time of the block's tokens (M: in virtual tokens for the product
// form).  A block holds 16 / r whole tokens; rows beyond them, and beyond the end of the sequence, are zero.
//
// The matrix instruction (lane l, r16 = l & 15, g = l >> 4) takes A[r16][slot g] and B[slot g][r16] and returns
// D[4 g + e][r16] in element e.  With slot g of step e standing for index 4 g + e of the contraction, element e of an
// accumulator tile is the B operand of step e (its transpose: the A operand), and four neighbouring floats of a row in
// LDS are the A operands of the four steps.  So S^T stays in accumulators for the whole sequence, and R, U go from one
// product to the next without moving between lanes.
//
// A workgroup owns 16 rows of S of one head.  State waves (one to four, a share of d_k each) run the chain; the one thing
// they exchange is their share of K S^T, through LDS, at the one barrier of a block.  Helper waves (eight where LDS holds
// a slot for each, else four) prepare a block each: inputs from memory to LDS, Gram, T by forward substitution on the
// vector ALU (the products of powers of a nilpotent matrix would lose digits where keys are nearly parallel), P; and they
// add up and store O.  A helper's work is cut into as many pieces as there are helpers, one per block of the chain, so
// that in every interval each of them is at another piece.
//
// Why 16: one tile of the instruction is the smallest block that feeds it, and the chain of dependent products of a
// block grows with the block.  What bounds it: that chain (about 1350 cycles a block of 16 at d_k = 64 with the helpers
// idle: R, the exchange, U, S, each behind the latency of the one before), and the helpers that share its SIMDs and LDS.
// Against the recurrence token by token (pf_generic.hip), fp32, us: 32 heads x 2048 tokens, d = 64, r = 1 492 -> 112;
// drivers of 8 heads x 500 tokens, d_k = 32, d_v = 48, r = 2 127 -> 45; 64 heads x 1000, d = 128, r = 1 335 -> 184;
// 4 heads x 700, d = 128, r = 3 464 -> 197; 1 head x 64, d = 16 17.5 -> 6.  Error against 64 bits (2-norm of O, S_L): the
// first of these 2.5e-7, 2.5e-7 -> 1.6e-7, 1.3e-7, because S is rounded once per block.  What a block adds, its sums, is kept
// down by trees and by U = R + (T - Id) R: 3 % of the time (43.0 -> 45.0 us for the second of these), and without it few tokens
// were further from 64 bits than token by token (block_pays in pf_generic.hip has what is left of that).
#pragma once
#include "pf_generic.h"
#include "pf_internal.h"

#include <type_traits>

namespace pf {

constexpr int kBlockVT = 16;          // virtual tokens of a block
constexpr int kBlockPitch = 20;       // row pitch of 16 x 16 tiles in LDS

// d_k padded to 16 DT columns
template <bool kDrivers, int DT>
struct BlockLds {
    static constexpr int D = 16 * DT, KP = D + 4, plane = kBlockVT * KP;
    static constexpr int NSW = DT <= 4 ? DT : (DT % 4 == 0 ? 4 : 3);   // state waves
    static constexpr int TPW = DT / NSW;                               // tiles of S^T per state wave
    static constexpr int oB = 0;                                       // rows of the update (K; drivers: B)
    static constexpr int oA = kDrivers ? plane : 0;                    // rows that multiply the state
    static constexpr int oQ = oA + plane;
    static constexpr int oV = oQ + plane;                              // V^T
    static constexpr int oT = oV + 16 * kBlockPitch;
    static constexpr int oP = oT + 16 * kBlockPitch;                   // operand form
    static constexpr int oBt = oP + 256;
    static constexpr int slot = oBt + 16;
    static constexpr int shares = 4 * NSW * 256;                       // of K S^T and of O^T, two blocks each
    // helper waves: eight where LDS has a slot for each of them and registers for three waves a SIMD suffice, else four
    // (d_k = 128: six helpers 234 us, four 207 for 4 heads x 700 tokens, r = 3; drivers of d_k up to 48: eight spill, 130 us
    // against 113 for 948 tokens, d_k = 48, d_v = 16 on two rounds of workgroups, 5 % in the middle of 169 shapes)
    static constexpr int NH = DT <= 4 && !(kDrivers && DT == 3) && 9 * slot + shares <= (int)(kMaxLdsBytes / 4) ? 8 : 4;
    static constexpr int slots = NH + 1;                               // one in use, the others being prepared
    static constexpr int oR = slots * slot;                            // shares of K S^T
    static constexpr int oO = oR + 2 * NSW * 256;                      // shares of O^T
    static constexpr size_t bytes = 4 * (size_t)(oR + shares);
    static constexpr int threads = 64 * (NSW + NH);
    static_assert(DT % NSW == 0 && bytes <= kMaxLdsBytes, "plan");
    // the eight steps of preparing a block, by the interval of a helper that they fall into
    static constexpr int first_step(int interval)
    {
        constexpr int four[5] = {0, 1, 3, 5, 8};
        return NH == 4 ? four[interval] : interval;
    }
};

// A sum of products in N sums that are added up at the end: rounded less often, and neighbours do not wait for each other.
template <int N>
struct Sums {
    f32x4 a[N];
    __device__ Sums()
    {
#pragma unroll
        for (int i = 0; i < N; ++i) a[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    __device__ void add(int step, float x, float y) { a[step % N] = mfma4(x, y, a[step % N]); }
    __device__ f32x4 total() const
    {
        if constexpr (N == 1) return a[0];
        else if constexpr (N == 2) return a[0] + a[1];
        else return (a[0] + a[1]) + (a[2] + a[3]);
    }
};

// Sixteen wait states between a product and a use of it behind a join of branches: the compiler (ROCm 7.2) counts the wait
// states of its result along one path to the join only, the one through the code that the other jumps over, and a copy of
// an accumulator there got the old upper half.  Products that cross a branch without it (os and ds, the branch for numbers
// that are not finite) have enough of them on both paths as built: tests/test_wait_states.py follows all paths of all kernels.
__device__ __forceinline__ void settle(f32x4 &v) { asm volatile("s_nop 7\n\ts_nop 7" : "+v"(v)); }

// four elements of a row as they lie in memory (read as a vector: a copy of the struct can stay a copy through scratch memory)
template <typename T> struct Raw4;
template <> struct Raw4<float> {
    f32x4 w;
    __device__ static Raw4 read(const float *p) { return {*reinterpret_cast<const f32x4 *>(p)}; }
    __device__ f32x4 widen() const { return w; }
    __device__ static Raw4 narrow(f32x4 v) { return {v}; }
};
template <> struct Raw4<uint16_t> {
    u32x2 w;
    __device__ static Raw4 read(const uint16_t *p) { return {*reinterpret_cast<const u32x2 *>(p)}; }
    __device__ f32x4 widen() const
    {
        return f32x4{__uint_as_float(w[0] << 16), __uint_as_float(w[0] & 0xffff0000u), __uint_as_float(w[1] << 16),
                     __uint_as_float(w[1] & 0xffff0000u)};
    }
    __device__ static Raw4 narrow(f32x4 v) { return {__builtin_bit_cast(u32x2, cvt4(v))}; }
};

// the first `have` of four elements at p, one by one, the others zero
template <typename T>
__device__ __forceinline__ f32x4 load4(const T *p, int have)
{
    f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (e < have) x[e] = as_f32(p[e]);
    return x;
}

__device__ __forceinline__ bool not_finite(float v) { return !(__builtin_fabsf(v) < __builtin_inff()); }

template <typename T, bool kDrivers, int DT>
__device__ __forceinline__ void generic_block(const GenericArgs<T> &a, int C, float *smem)
{
    using Ld = BlockLds<kDrivers, DT>;
    constexpr int NSW = Ld::NSW, NH = Ld::NH, TPW = Ld::TPW, KP = Ld::KP, TP = kBlockPitch;
    constexpr int NA = DT == 1 ? 4 : 2;   // (one tile of d_k: nothing else keeps the sums short)
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63, r16 = lane & 15, g = lane >> 4;
    // workgroups of one head are `heads` apart in blockIdx (one XCD's L2 when heads is a multiple of 8)
    const size_t head = blockIdx.x % (unsigned)a.heads;
    const int base = (int)(blockIdx.x / (unsigned)a.heads) * 16;
    const int L = a.L, dk = a.dk, dv = a.dv, r = a.r;
    const int NC = (L - a.t0 + C - 1) / C;
    auto f4 = [&](int off) -> f32x4 & { return *reinterpret_cast<f32x4 *>(smem + off); };
    auto first = [&](int b) { return a.t0 + b * C; };                            // first token of block b
    auto tokens = [&](int b) { const int m = L - first(b); return m < C ? m : C; };   // its tokens
    // the barrier without the wait for loads and stores to memory that __syncthreads brings
    auto barrier = [] {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        LDS_FENCE();
    };

    if (wave < NSW) {
        // ------------------------------------------------------------------ state waves
        __builtin_amdgcn_s_setprio(3);
        const int row = base + r16;
        const bool live = row < dv;
        f32x4 s[TPW];
#pragma unroll
        for (int q = 0; q < TPW; ++q) {
            const int x = 16 * (wave * TPW + q) + 4 * g;
            s[q] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (a.S0 && live) {
                const float *s0 = a.S0 + (head * (size_t)dv + row) * dk + x;
                if (dk % 4 != 0) s[q] = load4(s0, dk - x);
                else if (x < dk) s[q] = *reinterpret_cast<const f32x4 *>(s0);
            }
        }
        struct Operands {
            f32x4 kA[TPW], qB[TPW], kT[TPW], v, bt, t, p;
        };
        auto read_block = [&](int slot, Operands &to) {
            const int o = slot * Ld::slot;
#pragma unroll
            for (int q = 0; q < TPW; ++q) {
                const int x = 16 * (wave * TPW + q);
                to.kA[q] = f4(o + Ld::oA + r16 * KP + x + 4 * g);
                to.qB[q] = f4(o + Ld::oQ + r16 * KP + x + 4 * g);
#pragma unroll
                for (int e = 0; e < 4; ++e) to.kT[q][e] = smem[o + Ld::oB + (4 * g + e) * KP + x + r16];
            }
            to.v = f4(o + Ld::oV + r16 * TP + 4 * g);
            to.t = f4(o + Ld::oT + r16 * TP + 4 * g);
            to.p = f4(o + Ld::oP + lane * 4);
            if constexpr (!kDrivers) to.bt = f4(o + Ld::oBt + 4 * g);
        };
        f32x4 one;                                         // this lane's elements of Id
#pragma unroll
        for (int e = 0; e < 4; ++e) one[e] = 4 * g + e == r16 ? 1.f : 0.f;
        Operands even, odd;
        barrier();
        read_block(0, even);
        int slot = 0;
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
        auto block = [&](int c, const Operands &x, Operands &ahead) {
            const int buf = (c & 1) * NSW * 256;
            Sums<NA> w, u, os, op;
#pragma unroll
            for (int q = 0; q < TPW; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) w.add(e, x.kA[q][e], s[q][e]);
            // this wave's share of O of the block before, in the shadow of the products (the first block's is not used)
            f4(Ld::oO + (NSW * 256 - buf) + wave * 256 + lane * 4) = o;
            f4(Ld::oR + buf + wave * 256 + lane * 4) = w.total();
#pragma unroll
            for (int q = 0; q < TPW; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) os.add(e, s[q][e], x.qB[q][e]);
            barrier();
            f32x4 share[NSW], sum;
#pragma unroll
            for (int i = 0; i < NSW; ++i) share[i] = f4(Ld::oR + buf + i * 256 + lane * 4);
            LDS_FENCE();
            sum = share[0];
#pragma unroll
            for (int i = 1; i < NSW; ++i) sum += share[i];
            f32x4 R = kDrivers ? x.v + sum : x.bt * (x.v - sum);
            const int n = tokens(c) * r;
            if (n < kBlockVT) {                        // (rows of zeros times an infinite state are no numbers)
#pragma unroll
                for (int e = 0; e < 4; ++e) R[e] = 4 * g + e < n ? R[e] : 0.f;
            }
            slot = slot == Ld::slots - 1 ? 0 : slot + 1;
            read_block(slot, ahead);                       // (after the last block: some slot, not used)
            // U = R + (T - Id) R: R, the largest term, is rounded once, not at every step of a sum
            const f32x4 t = x.t - one;
#pragma unroll
            for (int e = 0; e < 4; ++e) u.add(e, t[e], R[e]);
            const f32x4 U = R + u.total();
            // the block's update is summed by itself: S is rounded once per block, not once per token
            Sums<DT == 1 ? 4 : 2> ds[TPW];
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int q = 0; q < TPW; ++q) ds[q].add(e, x.kT[q][e], U[e]);
            // An infinity or NaN of a token reaches that token and later ones only: zeros of T and P do not hide it from
            // the tokens before, so those are computed without it.
            f32x4 up = U;
            o = f32x4{0.f, 0.f, 0.f, 0.f};
            const bool bad = not_finite(((R[0] + R[1]) + (R[2] + R[3])) + ((U[0] + U[1]) + (U[2] + U[3])));
            if (__builtin_expect(__any(bad), 0)) {
                int jb = kBlockVT;
#pragma unroll
                for (int e = 3; e >= 0; --e)
                    if (not_finite(R[e])) {
                        jb = 4 * g + e;
                        R[e] = 0.f;
                    }
                up = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int e = 0; e < 4; ++e) up = mfma4(x.t[e], R[e], up);
                settle(up);
#pragma unroll
                for (int e = 3; e >= 0; --e)
                    if (not_finite(up[e]) && 4 * g + e < jb) jb = 4 * g + e;
                jb = min(jb, __shfl_xor(jb, 16));
                jb = min(jb, __shfl_xor(jb, 32));
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (4 * g + e >= jb) up[e] = 0.f;
                    if (__shfl(jb, 4 * g + e) < (r16 + 1) * r) o[e] = __builtin_nanf("");
                }
            }
            // this wave's share of the four steps of U^T P^T
#pragma unroll
            for (int m = 0; m < 4; m += NSW) {
                float uw = up[m], pw = x.p[m];
#pragma unroll
                for (int i = 1; i < NSW; ++i) {
                    uw = wave == i ? (m + i < 4 ? up[(m + i) & 3] : 0.f) : uw;
                    pw = wave == i ? (m + i < 4 ? x.p[(m + i) & 3] : 0.f) : pw;
                }
                op.add(m / NSW, uw, pw);
            }
#pragma unroll
            for (int q = 0; q < TPW; ++q) s[q] += ds[q].total();
            o += os.total() + op.total();
        };
#pragma unroll 1
        for (int c = 0; c < NC; c += 2) {
            block(c, even, odd);
            if (c + 1 < NC) block(c + 1, odd, even);
        }
        settle(o);
        f4(Ld::oO + ((NC - 1) & 1) * NSW * 256 + wave * 256 + lane * 4) = o;
        barrier();
        if (a.SL && live) {
#pragma unroll
            for (int q = 0; q < TPW; ++q) {
                const int x = 16 * (wave * TPW + q) + 4 * g;
                float *sl = a.SL + (head * (size_t)dv + row) * dk + x;
                if (dk % 4 == 0) {
                    if (x < dk) *reinterpret_cast<f32x4 *>(sl) = s[q];
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (x + e < dk) sl[e] = s[q][e];
                }
            }
        }
        return;
    }

    // ---------------------------------------------------------------------- helper waves
    const int h = wave - NSW;
    const T *Qh = a.Q + head * (size_t)L * dk;
    const T *Kh = a.K + head * (size_t)L * r * dk;
    const T *Ah = kDrivers ? a.beta + head * (size_t)L * r * dk : nullptr;
    const T *Vh = a.V + head * (size_t)L * r * dv;
    const T *bh = a.beta + head * (size_t)L * r;
    T *Oh = a.O + head * (size_t)L * dv;
    const bool kvec = dk % 4 == 0, vvec = dv % 4 == 0;
    constexpr int UPR = 4 * DT;                            // pieces of four elements per row
    // token of virtual token 4 g + e of this lane, and of virtual token r16 (itself in the product form)
    int tok4[4], mask4[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        tok4[e] = (4 * g + e) / r;
        mask4[e] = a.product ? 4 * g + e : tok4[e];
    }
    const int mask16 = a.product ? r16 : r16 / r;

    // A block's inputs are requested four blocks ahead, by loads without a branch around them (out of range: the block's
    // first element again), so that nothing waits for them before they are staged.  Rows that are not whole pieces of
    // four elements are read element by element when they are staged; the loads here then go to the start of the arrays.
    Raw4<T> rk[DT], ra[kDrivers ? DT : 1], rq[DT], rv;
    T rb{};
    int prow[DT], pcol[DT];                                // row, column of a piece; columns beyond d_k: row 16
    uint32_t poff[DT];                                     // its offset in elements
#pragma unroll
    for (int q = 0; q < DT; ++q) {
        const int i = (lane + 64 * q) / UPR;
        pcol[q] = 4 * ((lane + 64 * q) % UPR);
        prow[q] = pcol[q] < dk ? i : kBlockVT;
        poff[q] = (uint32_t)(i * dk + pcol[q]);
    }
    const int vrow = base + 4 * (lane & 3) < dv ? lane >> 2 : kBlockVT;
    const uint32_t voff = (uint32_t)((lane >> 2) * dv + base + 4 * (lane & 3));
    auto at = [](const T *p, uint32_t off) { return *reinterpret_cast<const Raw4<T> *>(reinterpret_cast<const char *>(p) + off * (uint32_t)sizeof(T)); };
    auto fetch = [&](int b) {
        const int m = tokens(b), n = m * r, nk = kvec ? n : 0, mk = kvec ? m : 0;
        const size_t t = first(b);
        const T *Kb = kvec ? Kh + t * r * dk : a.K, *Qb = kvec ? Qh + t * dk : a.K, *Ab = nullptr;
        if constexpr (kDrivers) Ab = kvec ? Ah + t * r * dk : a.K;
#pragma unroll
        for (int q = 0; q < DT; ++q) {
            const uint32_t ki = prow[q] < nk ? poff[q] : 0u, qi = prow[q] < mk ? poff[q] : 0u;
            rk[q] = at(Kb, ki);
            if constexpr (kDrivers) ra[q] = at(Ab, ki);
            rq[q] = at(Qb, qi);
        }
        rv = at(vvec ? Vh + t * r * dv : a.V, vrow < (vvec ? n : 0) ? voff : 0u);
        if constexpr (!kDrivers) rb = bh[t * r + (r16 < n ? r16 : 0)];
    };
    // Whole blocks leave the zeros alone that rows and columns beyond theirs were given once.
    auto stage = [&](int b, int o) {
        const int m = tokens(b), n = m * r;
        if (kvec && vvec && m == C && b >= Ld::slots) {
#pragma unroll
            for (int q = 0; q < DT; ++q) {
                const int to = o + ((lane + 64 * q) / UPR) * KP + pcol[q];
                auto put = [&](int rows, int plane, const Raw4<T> &x) {
                    if (64 % UPR == 0 && dk == Ld::D && (q + 1) * (64 / UPR) <= rows) f4(to + plane) = x.widen();
                    else if (prow[q] < rows) f4(to + plane) = x.widen();
                };
                put(n, Ld::oB, rk[q]);
                if constexpr (kDrivers) put(n, Ld::oA, ra[q]);
                put(m, Ld::oQ, rq[q]);
            }
            if (vrow < n) {
                const f32x4 w = rv.widen();
#pragma unroll
                for (int e = 0; e < 4; ++e) smem[o + Ld::oV + (4 * (lane & 3) + e) * TP + (lane >> 2)] = w[e];
            }
            if constexpr (!kDrivers)
                if (lane < n) smem[o + Ld::oBt + lane] = as_f32(rb);
            return;
        }
        const size_t t = first(b);
        const f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < DT; ++q) {
            const int i = (lane + 64 * q) / UPR, x = pcol[q];
            f32x4 wk = z, wa = z, wq = z;
            if (kvec) {
                wk = prow[q] < n ? rk[q].widen() : z;
                if constexpr (kDrivers) wa = prow[q] < n ? ra[q].widen() : z;
                wq = prow[q] < m ? rq[q].widen() : z;
            } else {
                wk = load4(Kh + (t * r + i) * dk + x, i < n ? dk - x : 0);
                if constexpr (kDrivers) wa = load4(Ah + (t * r + i) * dk + x, i < n ? dk - x : 0);
                wq = load4(Qh + (t + i) * dk + x, i < m ? dk - x : 0);
            }
            f4(o + Ld::oB + i * KP + x) = wk;
            if constexpr (kDrivers) f4(o + Ld::oA + i * KP + x) = wa;
            f4(o + Ld::oQ + i * KP + x) = wq;
        }
        const int i = lane >> 2, x = base + 4 * (lane & 3);
        f32x4 wv = z;
        if (vvec) wv = vrow < n ? rv.widen() : z;
        else wv = load4(Vh + (t * r + i) * dv + x, i < n ? dv - x : 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) smem[o + Ld::oV + (4 * (lane & 3) + e) * TP + i] = wv[e];
        if constexpr (!kDrivers)
            if (lane < 16) smem[o + Ld::oBt + lane] = lane < n ? as_f32(rb) : 0.f;
    };
    // x y^T over tiles Q0 .. Q1 - 1 of 16 columns: the products of a tile in two or four sums of their own, which meet in a tree.
    // (In two sums over all of d_k = 128, O of 16 tokens from a zero state was 1.6 times as far from 64 bits as the rows' body
    // has it, whose sums are trees as well.  One tile after the other instead of all products first: 35 heads x 290 tokens,
    // d_k = 128, r = 4 in the product form, 123 us, this 114, the two sums 111.)
    auto dots = [&](int ox, int oy, auto Q0c, auto Q1c) -> f32x4 {
        constexpr int Q0 = decltype(Q0c)::value, M = decltype(Q1c)::value - Q0, N = DT <= 2 ? 4 : 2;
        f32x4 x[M], y[M], sum[M * N];
#pragma unroll
        for (int q = 0; q < M; ++q) {
            x[q] = f4(ox + r16 * KP + 16 * (Q0 + q) + 4 * g);
            y[q] = f4(oy + r16 * KP + 16 * (Q0 + q) + 4 * g);
        }
        LDS_FENCE();
#pragma unroll
        for (int i = 0; i < M * N; ++i) sum[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int q = 0; q < M; ++q) sum[N * q + e % N] = mfma4(x[q][e], y[q][e], sum[N * q + e % N]);
#pragma unroll
        for (int n = M * N; n > 1; n = (n + 1) / 2)
#pragma unroll
            for (int i = 0; i < n / 2; ++i) sum[i] += sum[(n + 1) / 2 + i];
        return sum[0];
    };
    constexpr int H1 = (DT + 1) / 2;
    constexpr std::integral_constant<int, 0> kFirst{};
    constexpr std::integral_constant<int, H1> kHalf{};
    constexpr std::integral_constant<int, DT> kLast{};
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};                      // the first half of the columns, from one interval to the next
    auto half = [&](int ox, int oy) { acc = dots(ox, oy, kFirst, kHalf); };
    auto whole = [&](int ox, int oy) {
        if constexpr (H1 < DT) acc += dots(ox, oy, kHalf, kLast);
    };
    auto put_gram = [&](int o) {                           // the strictly lower part of the system matrix less the identity
        f32x4 b = {-1.f, -1.f, -1.f, -1.f};
        if constexpr (!kDrivers) b = f4(o + Ld::oBt + 4 * g);
#pragma unroll
        for (int e = 0; e < 4; ++e) smem[o + Ld::oT + (4 * g + e) * TP + r16] = mask16 < mask4[e] ? acc[e] * b[e] : 0.f;
    };
    // Rows I0 .. I1 - 1 of T, a column per lane; a row of T takes the place of the row of the system matrix that it was
    // the last to need.  Several rows are read at a time (one by one, each read would be waited for: 2.6 us a block) and
    // taken by columns, so that products do not wait for each other.  (Elements by v_readlane out of the accumulator
    // instead of rows out of LDS: 119 us against 105 for 32 heads x 2048 tokens, d_k = 64.)
    auto rows_of_t = [&](int o, float *t, auto I0c, auto I1c) {
        constexpr int I0 = decltype(I0c)::value, I1 = decltype(I1c)::value;
        f32x4 n[I1 - I0][kBlockVT / 4];
#pragma unroll
        for (int i = I0; i < I1; ++i)
#pragma unroll
            for (int j = 0; j < i; j += 4) n[i - I0][j / 4] = f4(o + Ld::oT + i * TP + j);
        LDS_FENCE();
#pragma unroll
        for (int i = I0; i < I1; ++i) t[i] = i == r16 ? 1.f : 0.f;
#pragma unroll
        for (int j = 0; j < I1 - 1; ++j)
#pragma unroll
            for (int i = j + 1 > I0 ? j + 1 : I0; i < I1; ++i) t[i] = fmaf(-n[i - I0][j / 4][j & 3], t[j], t[i]);
        if (g == 0) {
#pragma unroll
            for (int i = I0; i < I1; ++i) smem[o + Ld::oT + i * TP + r16] = t[i];
        }
    };
    auto substitute_upper = [&](int o) {                   // half of the products lie before row 11
        float t[kBlockVT];
        rows_of_t(o, t, std::integral_constant<int, 0>{}, std::integral_constant<int, 8>{});
        rows_of_t(o, t, std::integral_constant<int, 8>{}, std::integral_constant<int, 11>{});
    };
    auto substitute_lower = [&](int o) {
        float t[kBlockVT];
#pragma unroll
        for (int j = 0; j < 11; ++j) t[j] = smem[o + Ld::oT + j * TP + r16];
        rows_of_t(o, t, std::integral_constant<int, 11>{}, std::integral_constant<int, 14>{});
        rows_of_t(o, t, std::integral_constant<int, 14>{}, std::integral_constant<int, kBlockVT>{});
    };
    auto put_p = [&](int o) {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = tok4[e] <= r16 ? acc[e] : 0.f;
        f4(o + Ld::oP + lane * 4) = acc;
    };
    auto store_o = [&](int b) {
        const int buf = Ld::oO + (b & 1) * NSW * 256;
        f32x4 x = f4(buf + lane * 4);
#pragma unroll
        for (int i = 1; i < NSW; ++i) x += f4(buf + i * 256 + lane * 4);
        const int col = base + 4 * g;
        if (r16 >= tokens(b) || col >= dv) return;
        T *dst = Oh + (size_t)(first(b) + r16) * dv + col;
        if (vvec) {
            *reinterpret_cast<Raw4<T> *>(dst) = Raw4<T>::narrow(x);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (col + e < dv) dst[e] = from_f32<T>(x[e]);
        }
    };
    auto clamp = [&](int b) { return b < NC ? b : NC - 1; };
    fetch(clamp(h));
    if (h < NC) {
        const int o = h * Ld::slot;
        stage(h, o);
        half(o + Ld::oA, o + Ld::oB);                      // rows that multiply the state times rows of the update
        whole(o + Ld::oA, o + Ld::oB);
        put_gram(o);
        substitute_upper(o);
        substitute_lower(o);
        half(o + Ld::oB, o + Ld::oQ);
        whole(o + Ld::oB, o + Ld::oQ);
        put_p(o);
    }
    fetch(clamp(h + NH));
    barrier();
    // Interval c lies between the barriers of blocks c and c + 1.  Block b is prepared in intervals b - NH - 1 .. b - 2 (its
    // slot is that of block b - NH - 1, and its operands are read from interval b - 1 on).  Each interval one helper is at
    // the step that also stores O of the block before.
    int left = NC + 1, b = h + NH;
    constexpr int kStoreAt = 2;                            // (well before the next wait for loads, which waits for it too)
    int next = NH - h;                                     // the interval that comes next
    for (int i = 0; i < h && left > 0; ++i, --left, ++next) barrier();
    while (left > 0) {
        const bool have = b < NC;
        const int o = (b % Ld::slots) * Ld::slot;
        // (left by break, not around code: a join behind the loads would make them wait for a copy)
#define INTERVAL(I)                                                                          \
        if constexpr (I < NH) {                                                              \
            constexpr int s0 = Ld::first_step(I), s1 = Ld::first_step(I + 1);                \
            if (s0 <= kStoreAt && kStoreAt < s1 && b + I >= NH + 2) store_o(b + I - NH - 2); \
            if (s0 <= 0 && have) stage(b, o);                                                \
            if (s0 <= 1 && 1 < s1) fetch(clamp(b + NH));                                     \
            if (have) {                                                                      \
                if (s0 <= 1 && 1 < s1) half(o + Ld::oA, o + Ld::oB);                         \
                if (s0 <= 2 && 2 < s1) {                                                     \
                    whole(o + Ld::oA, o + Ld::oB);                                           \
                    put_gram(o);                                                             \
                }                                                                            \
                if (s0 <= 3 && 3 < s1) substitute_upper(o);                                  \
                if (s0 <= 4 && 4 < s1) substitute_lower(o);                                  \
                if (s0 <= 5 && 5 < s1) half(o + Ld::oB, o + Ld::oQ);                         \
                if (s0 <= 6 && 6 < s1) {                                                     \
                    whole(o + Ld::oB, o + Ld::oQ);                                           \
                    put_p(o);                                                                \
                }                                                                            \
            }                                                                                \
            barrier();                                                                       \
            next = I + 1;                                                                    \
            if (--left == 0) break;                                                          \
        }
        INTERVAL(0)
        INTERVAL(1)
        INTERVAL(2)
        INTERVAL(3)
        INTERVAL(4)
        INTERVAL(5)
        INTERVAL(6)
        INTERVAL(7)
#undef INTERVAL
        b += NH;
    }
    next %= NH;
    if (Ld::first_step(next) <= kStoreAt && kStoreAt < Ld::first_step(next + 1)) store_o(NC - 1);
}

}  // namespace pf

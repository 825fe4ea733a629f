// Body of the chunk-flow kernel for blocks of 64 virtual tokens: one wavefront per block, no barrier, and nothing but the
// inverse of the diagonal tiles through LDS.
//
// The rows of K of a block fit one wavefront's registers as MFMA operands, and the layout that serves them as rows of the
// Gram serves them as columns, so G and K Q^T come out of registers alone.  What follows is the block substitution of
// Proposition 3.3 on 16 x 16 tiles, run on the transposed system (Id + G)^T X = Id, X = T^T, from the last tile up:
//     X_js = T_jj^T ( - sum_{j < i <= s} G_ij^T X_is ),     X_ss = T_ss^T.
// An accumulator tile of G is, element for element, the A operand of its transpose for the fp32 instruction, and an
// accumulator tile of X the B operand of the next product (mfma4), so the substitution moves nothing between lanes
// either, and T is rounded to bf16 once, when it is stored: with G, X and T_jj rounded to bf16 as operands the flow took
// 1 us less on every shape below and the forward was 1 % further from 64 bits (O 4.54e-3 against 4.49e-3 before this
// body and 4.42e-3 now, 20 heads x 8192 tokens, d = 128, r = 2).  Two accumulator tiles of X, one upon the other, are a
// tile of T as the scan reads it (pf_layout.h).
// T_jj = (Id + G_jj)^{-1}: forward substitution in fp32 on the vector ALU, four tiles at a time, a column per lane;
// the rows of G_jj come in 16 reads and go round by DPP (as operands that all lanes read out of LDS, 40 reads of 16 bytes,
// 32 x 2944 below took 18.0 us: the chain of one block is all it has).
//
// What bounds it: HBM.  Where the scan builds P (pf_chain.h) it reads K and beta and writes T: 64 heads x 4096 tokens, d = 128, r = 2
// 187 MB in 37 us, 5.1 TB/s, 32 heads x 65536 1.49 GB in 275 us, 5.4 TB/s.  With P (and Q) 278 MB in 45 us, 2.2 GB in 433 us.
// The rows of the next block are asked for as soon as the block before has had its two sets of products, and
// eight wavefronts a compute unit at different steps keep the loads going (at d = 64 a third workgroup a compute unit
// would spill).  The workgroup of eight wavefronts per block that serves the larger blocks (pf_flow.hip) had work for
// two to four of them here and six barriers; flow alone, us, that body / this one with P, when it was built / without P:
//   64 heads x 4096, d = 128, r = 2    70.2 / 44.7 / 37      32 x 2048, d = 64, r = 1    11.2 / 7.9 / 6.4
//   32 x 65536, d = 128, r = 2          533 / 432 / 275      24 x 4096, d = 64, r = 2    26.1 / 13.6 / 10.6
//   4 x 32768, d = 128, r = 2          36.6 / 23.8 / 20.8    32 x 2944, d = 128, r = 1   18.1 / 14.9 / 11 (one block a wavefront)
#pragma once
#include "pf_common.h"
#include "pf_internal.h"
#include "pf_layout.h"

#include <type_traits>

namespace pf {

struct FlowWavePlan {
    static constexpr int waves = 4, threads = 64 * waves;
    static constexpr int NP = 20;                                      // row pitch of a tile in LDS
    static constexpr int floats = 4 * 16 * NP + 64;                    // of a wavefront: diagonal tiles, row factors
    static constexpr size_t lds = (size_t)waves * floats * 4;
};

// t[i] -= (n[i] of lane J of a row of 16 lanes) * y for M <= 8 rows: DPP row_newbcast inside the product (written as a move, the
// compiler keeps it one and hoists all of them into registers).  The compiler does not look for hazards inside: the s_nop gives
// the two wait states between a register written just before, for instance by a copy, and its use by DPP.
template <int J, int M>
__device__ __forceinline__ void minus_rows(const float *n, float *t, float y)
{
#define PF_L(k) "\n\tv_fmac_f32_dpp %[t" #k "], -%[n" #k "], %[y] row_newbcast:%c[j] row_mask:0xf bank_mask:0xf"
#define PF_T(k) [t##k] "+&v"(t[k])
#define PF_N(k) [n##k] "v"(n[k])
#define PF_Y [y] "v"(y), [j] "n"(J)
    static_assert(M >= 1 && M <= 8);
    if constexpr (M == 8) {
        asm("s_nop 1" PF_L(0) PF_L(1) PF_L(2) PF_L(3) PF_L(4) PF_L(5) PF_L(6) PF_L(7)
            : PF_T(0), PF_T(1), PF_T(2), PF_T(3), PF_T(4), PF_T(5), PF_T(6), PF_T(7)
            : PF_N(0), PF_N(1), PF_N(2), PF_N(3), PF_N(4), PF_N(5), PF_N(6), PF_N(7), PF_Y);
    } else if constexpr (M >= 4) {
        asm("s_nop 1" PF_L(0) PF_L(1) PF_L(2) PF_L(3)
            : PF_T(0), PF_T(1), PF_T(2), PF_T(3) : PF_N(0), PF_N(1), PF_N(2), PF_N(3), PF_Y);
        if constexpr (M > 4) minus_rows<J, M - 4>(n + 4, t + 4, y);
    } else if constexpr (M == 3) {
        asm("s_nop 1" PF_L(0) PF_L(1) PF_L(2) : PF_T(0), PF_T(1), PF_T(2) : PF_N(0), PF_N(1), PF_N(2), PF_Y);
    } else if constexpr (M == 2) {
        asm("s_nop 1" PF_L(0) PF_L(1) : PF_T(0), PF_T(1) : PF_N(0), PF_N(1), PF_Y);
    } else {
        asm("s_nop 1" PF_L(0) : PF_T(0) : PF_N(0), PF_Y);
    }
#undef PF_L
#undef PF_T
#undef PF_N
#undef PF_Y
}

// T = (Id + N)^{-1}, N strictly lower 16 x 16, by forward substitution: lane c of a row of 16 lanes holds element c of row i of N
// in n[i] and column c of T in t.  By columns, so that products do not wait for each other.
template <int J = 0>
__device__ __forceinline__ void substitute_rows(const float (&n)[16], float (&t)[16], int c)
{
    if constexpr (J == 0) {
#pragma unroll
        for (int i = 0; i < 16; ++i) t[i] = i == c ? 1.f : 0.f;
    }
    if constexpr (J < 15) {
        constexpr int M = 15 - J, B = M < 8 ? M : 8;
        if constexpr (M > 8) minus_rows<J, M - 8>(n + J + 1, t + J + 1, t[J]);
        minus_rows<J, B>(n + 16 - B, t + 16 - B, t[J]);
        substitute_rows<J + 1>(n, t, c);
    }
}

// FOLD: -T diag(beta) is handed over, rounded once, in the place of T.  PT: P too (pf_chain.h says who builds it else).
template <int D, int C, bool GEN, bool FOLD, bool PT>
__device__ __forceinline__ void flow_wave(const bf16 *__restrict__ Q, const bf16 *__restrict__ K, const bf16 *__restrict__ beta,
                                          bf16 *__restrict__ Tt, bf16 *__restrict__ Pt, int nchunks, int NC, int tail,
                                          int mask_shift, float *smem)
{
    static_assert(!GEN || (!FOLD && PT), "the delta rule's forms");
    constexpr int N = 64, R = N / C, NKS = D / 32, NKT = N / 32, MT = N / 16, CT = C / 16, NP = FlowWavePlan::NP;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63, r16 = lane & 15, g = lane >> 4;
    float *Ns = smem + wave * FlowWavePlan::floats, *bs = Ns + 4 * 16 * NP;
    constexpr auto tri = [](int i, int j) constexpr { return i * (i + 1) / 2 + j; };   // tiles on and below the diagonal

    bf16x8 aK[MT][NKS], aA[GEN ? MT : 1][NKS], bQ[PT ? CT : 1][NKS];
    bf16 breg = (bf16)0.0f;
    // A head holds NC whole blocks followed by `tail` tokens that another kernel takes: block c of the compact
    // numbering starts (c / NC) * tail tokens further on in Q, K, beta.
    auto fetch = [&](size_t c) {
        const size_t skew = tail ? (c / (size_t)NC) * (size_t)tail : (size_t)0;
        const bf16 *Kg = K + (c * N + skew * R) * D, *Qg = Q + (c * C + skew) * D;
        const uint32_t at = (uint32_t)(r16 * D + 8 * g);
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) {
                aK[m][ks] = ld8(Kg + at + 16 * m * D + 32 * ks);
                if constexpr (GEN) aA[m][ks] = ld8(beta + (c * N + skew * R) * D + at + 16 * m * D + 32 * ks);
            }
        if constexpr (PT) {
#pragma unroll
            for (int t = 0; t < CT; ++t)
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks) bQ[t][ks] = ld8(Qg + at + 16 * t * D + 32 * ks);
        }
        if constexpr (!GEN) breg = beta[c * N + skew * R + lane];
    };

    const unsigned blocks = (unsigned)nchunks, step = gridDim.x * FlowWavePlan::waves;
    // no more blocks than workgroups: one to each; else neighbours in a workgroup (dealt a grid apart, 24 heads x 4096 tokens,
    // d = 64, r = 2 took 15.6 us instead of 13.7)
    unsigned cid = blocks <= gridDim.x ? blockIdx.x + gridDim.x * wave : blockIdx.x * FlowWavePlan::waves + wave;
    if (cid >= blocks) return;                         // whole wavefronts; no barrier below
    fetch(cid);
#pragma unroll 1
    for (bool more = true; more; cid += step) {
        bf16 *Ttg = Tt + (size_t)cid * N * N, *Ptg = Pt + (size_t)cid * C * N;
        // ---- row factor of the system matrix: beta_i for the delta rule (G_ij = beta_i k_i . k_j); -1 for general
        // drivers (G_ij = -a_i . b_j)
        f32x4 b[MT];
        if constexpr (!GEN) {
            bs[lane] = (float)breg;
            LDS_FENCE();
#pragma unroll
            for (int i = 0; i < MT; ++i) b[i] = *reinterpret_cast<const f32x4 *>(&bs[16 * i + 4 * g]);
        } else {
#pragma unroll
            for (int i = 0; i < MT; ++i) b[i] = f32x4{-1.f, -1.f, -1.f, -1.f};
        }
        // ---- G, lower tiles
        f32x4 G[tri(MT, 0)];
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j <= i; ++j) {
                f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks) acc = mfma16(GEN ? aA[GEN ? i : 0][ks] : aK[i][ks], aK[j][ks], acc);
                G[tri(i, j)] = acc;
            }
        // ---- P = Mbar (.) Q K^T, from K Q^T
#pragma unroll
        for (int t = 0; t < (PT ? CT : 0); ++t)
#pragma unroll
            for (int kt = 0; kt < NKT; ++kt) {
                if (kt >= p_ksteps(R, t)) continue;
                f32x4 acc[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    acc[h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ks = 0; ks < NKS; ++ks) acc[h] = mfma16(aK[2 * kt + h][ks], bQ[t][ks], acc[h]);
#pragma unroll
                    for (int e = 0; e < 4; ++e)        // readout mask, inclusive in time
                        if (32 * kt + 16 * h + 15 >= R * 16 * t) acc[h][e] = (32 * kt + 16 * h + 4 * g + e) / R > 16 * t + r16 ? 0.0f : acc[h][e];
                }
                st8(Ptg + full_tile_offset(NKT, t, kt) + lane * 8, join(cvt4(acc[0]), cvt4(acc[1])));
            }
        // ---- the next block's inputs
        more = cid + step < blocks;
        if (more) fetch(cid + step);
        // ---- diagonal tiles to LDS, strictly lower in time; the others as operands of -G^T
        f32x4 nG[tri(MT, 0)];
#pragma unroll
        for (int i = 0; i < MT; ++i) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                // rows and columns compared by token, i.e. by virtual token >> log2(R); mask_shift = 0 compares
                // virtual tokens themselves (the r sub-updates of a token then see each other, one after another)
                const bool seen = (r16 >> mask_shift) < ((4 * g + e) >> mask_shift);
                Ns[(16 * i + 4 * g + e) * NP + r16] = seen ? G[tri(i, i)][e] * b[i][e] : 0.0f;
            }
#pragma unroll
            for (int j = 0; j < i; ++j) nG[tri(i, j)] = G[tri(i, j)] * -b[i];
        }
        // ---- T_jj: lane group g inverts tile g, a column per lane
        {
            float n[16], t[16];
            LDS_FENCE();
#pragma unroll
            for (int i = 1; i < 16; ++i) n[i] = Ns[(16 * g + i) * NP + r16];
            substitute_rows(n, t, r16);
#pragma unroll
            for (int i = 0; i < 16; ++i) Ns[(16 * g + i) * NP + r16] = t[i];
            LDS_FENCE();
        }
        // ---- X, column by column of tiles; handed over as it is, or as -T diag(beta)
        f32x4 sc[MT];
#pragma unroll
        for (int j = 0; j < MT; ++j) sc[j] = FOLD ? -b[j] : f32x4{1.f, 1.f, 1.f, 1.f};
        f32x4 Xd[MT];                                      // T_ss^T
        f32x4 To[MT];                                      // T_jj as operand of its transpose
#pragma unroll
        for (int s = 0; s < MT; ++s) {
            Xd[s] = *reinterpret_cast<const f32x4 *>(&Ns[(16 * s + r16) * NP + 4 * g]);
#pragma unroll
            for (int e = 0; e < 4; ++e) To[s][e] = Ns[(16 * s + 4 * g + e) * NP + r16];
        }
        LDS_FENCE();
#pragma unroll
        for (int s = 0; s < MT; ++s) {
            f32x4 X[MT];
            bf16x4 out[MT];                                // (as handed over)
            X[s] = Xd[s];
            out[s] = cvt4(Xd[s] * sc[s]);
#pragma unroll
            for (int j = s - 1; j >= 0; --j) {
                f32x4 acc = {0.f, 0.f, 0.f, 0.f}, x = acc;
#pragma unroll
                for (int i = j + 1; i <= s; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc = mfma4(nG[tri(i, j)][e], X[i][e], acc);
#pragma unroll
                for (int e = 0; e < 4; ++e) x = mfma4(To[j][e], acc[e], x);
                X[j] = x;
                out[j] = cvt4(x * sc[j]);
            }
#pragma unroll
            for (int kt = 0; 2 * kt <= s; ++kt) {
                bf16x4 z;
#pragma unroll
                for (int e = 0; e < 4; ++e) z[e] = (bf16)0.0f;
                st8(Ttg + full_tile_offset(NKT, s, kt) + lane * 8, join(out[2 * kt], 2 * kt + 1 <= s ? out[2 * kt + 1] : z));
            }
        }
    }
}

}  // namespace pf

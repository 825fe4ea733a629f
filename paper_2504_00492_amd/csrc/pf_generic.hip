// Generic path: the recurrence itself (Section 3.1 of ParallelFlow, arXiv 2504.00492) in fp32.  Serves PF_F32, every
// shape the MFMA path has no instance for (any d_k, d_v, r), sequences shorter than one flow block (the
// step-by-step use of the forward: a few tokens in, the state in and out) and the L % block tokens a flow block
// leaves over.  Two forms: rows of up to 128 columns with more than a few tokens go 16 virtual tokens at a time
// through the fp32 matrix instruction (pf_generic_block.h; block_pays says when), the rest token by token in vector
// arithmetic with the state in registers, below.
//
//   delta rule   u_j = beta_j (v_j - S k_j),   S += sum_j u_j k_j^T,   o = S q
//   drivers      u_j = atil_j + S a_j,         S += sum_j u_j b_j^T,   o = S q
//
// Rows of S are independent (the recurrence multiplies S from the right), so a wavefront owns 64 / LPR
// rows of one head, LPR lanes to a row, CS columns of it in each lane's registers, and nothing but
// inputs and outputs ever leaves the registers between tokens.  The sums over a row are a butterfly of
// LPR lanes in DPP moves.  k (a, b), q, v, beta of a block of tokens are staged in LDS as fp32 by the whole
// workgroup (one read from memory for all its rows) while the block before is computed; the readout of
// token t and the products S k of token t + 1 both see S_t, so their sums run side by side.
//
// Few tokens against a state that many wavefronts share out have a body of their own (generic_few; few_tokens says when).
//
// What bounds it: one wavefront per SIMD, token after token.  Ranks without a shape of their own take the u_j through
// LDS, one rank after the other, and rows too long for registers are read from memory at every use (32 heads x 512
// tokens, d_v = 32, fp32: d_k = 512, r = 2 0.37 ms, d_k = 520 4.14 ms).
#include "pf_internal.h"
#include "pf_common.h"
#include "pf_generic.h"
#include "pf_generic_block.h"

#include <type_traits>

namespace pf {

namespace {

// 16 bytes of elements as they lie in memory -> fp32 in LDS
__device__ __forceinline__ void put16(float *dst, u32x4 w, float)
{
    *reinterpret_cast<u32x4 *>(dst) = w;
}
__device__ __forceinline__ void put16(float *dst, u32x4 w, uint16_t)
{
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        f32x4 v;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            v[2 * i] = __uint_as_float(w[2 * h + i] << 16);
            v[2 * i + 1] = __uint_as_float(w[2 * h + i] & 0xffff0000u);
        }
        *reinterpret_cast<f32x4 *>(dst + 4 * h) = v;
    }
}

template <int CTRL> __device__ __forceinline__ float dpp_add(float v)
{
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
// sum over the LPR neighbouring lanes of a row, in every one of them (the same bits: each step adds the same two numbers)
template <int LPR> __device__ __forceinline__ float row_sum(float v)
{
    static_assert(LPR == 4 || LPR == 8 || LPR == 16 || LPR == 64, "lanes per row");
    v = dpp_add<0xB1>(v);                        // quad_perm [1 0 3 2]
    v = dpp_add<0x4E>(v);                        // quad_perm [2 3 0 1]
    if (LPR >= 8) v = dpp_add<0x141>(v);         // row_half_mirror
    if (LPR >= 16) v = dpp_add<0x140>(v);        // row_mirror
    if (LPR >= 64) {
        v += __shfl_xor(v, 16);
        v += __shfl_xor(v, 32);
    }
    return v;
}

constexpr int kPre = 6;      // 16-byte pieces of rows a thread carries for the next block of tokens
constexpr int kPreV = 4;     // values a thread carries for it

}  // namespace

// How one call is cut up: filled in by the host, uniform over the grid.
struct GenericPlan {
    int lpr, cs;        // lanes per row, columns per lane (cs = 0: state rows in LDS, see generic_long_rows)
    int waves;          // wavefronts per workgroup
    int tb;             // tokens staged at a time
    int prefetch;       // the next block's inputs fit the registers a thread carries
    int vpr;            // pieces per row (16 bytes each when vec, else one element each)
    int vec;            // rows are whole 16-byte pieces
    int tiles;          // workgroups per head
    size_t lds;
};

namespace {

// R: ranks held side by side (their products with the state all see the state before the token); R = 1
// with nsub > 1 is the product form (the sub-updates of a token one after another); R = 0 takes any r.
template <typename T, bool kDrivers, int LPR, int CS, int R>
__device__ __forceinline__ void generic_rows(const GenericArgs<T> &a, const GenericPlan &pl, float *smem)
{
    constexpr int VEC = 16 / sizeof(T), CV = CS / 4, DKP = LPR * CS, RPW = 64 / LPR;
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63, wave = tid >> 6;
    const int c = lane % LPR, rr = lane / LPR;
    const int rowsWG = pl.waves * RPW;
    // workgroups of one head are `heads` apart in blockIdx (one XCD's L2 when heads is a multiple of 8)
    const size_t head = blockIdx.x % (unsigned)a.heads;
    const int base = (int)(blockIdx.x / (unsigned)a.heads) * rowsWG;
    const int rowl = wave * RPW + rr, row = base + rowl;
    const bool live = row < a.dv;
    const int L = a.L, dk = a.dk, dv = a.dv, r = a.r, tb = pl.tb;
    const int nsub = R == 1 ? r : 1;                 // r == 1, or the product form
    const T *Qh = a.Q + head * (size_t)L * dk;
    const T *Kh = a.K + head * (size_t)L * r * dk;
    const T *Ah = kDrivers ? a.beta + head * (size_t)L * r * dk : Kh;   // rows that multiply the state
    const T *Vh = a.V + head * (size_t)L * r * dv;
    const T *bh = a.beta + head * (size_t)L * r;
    T *Oh = a.O + head * (size_t)L * dv;

    // LDS: rows that multiply the state, (drivers: rows of the update,) q; v; beta; o; u (R = 0)
    const int krows = tb * r, urow0 = kDrivers ? krows : 0, qrow0 = urow0 + krows, nrows = qrow0 + tb;
    float *rows = smem, *vs = rows + (size_t)nrows * DKP, *bs = vs + (size_t)krows * rowsWG;
    float *os = bs + (kDrivers ? 0 : krows), *us = os + (size_t)tb * rowsWG + (size_t)rowl * r;

    float S[CS];
    {
        const float *s0 = a.S0 ? a.S0 + (head * (size_t)dv + (live ? row : 0)) * dk : nullptr;
#pragma unroll
        for (int i = 0; i < CV; ++i) {
            const int x = 4 * (c + LPR * i);
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
            if (s0 && live) {
                if (dk % 4 == 0) {
                    if (x < dk) v = *reinterpret_cast<const f32x4 *>(s0 + x);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (x + e < dk) v[e] = s0[x + e];
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) S[4 * i + e] = v[e];
        }
    }
    // columns beyond d_k are staged as zeros, once
    if (dk < DKP)
        for (int i = tid; i < nrows * (DKP - dk); i += nthr) rows[(i / (DKP - dk)) * DKP + dk + i % (DKP - dk)] = 0.f;

    // source of staged row i of the block that starts at token t (rows beyond its `cl` tokens: its first row)
    auto row_src = [&](int i, int t, int cl) -> const T * {
        if (i >= qrow0) return Qh + (size_t)(t + (i - qrow0 < cl ? i - qrow0 : 0)) * dk;
        const bool second = kDrivers && i >= urow0;
        const int j = second ? i - urow0 : i;
        return (second ? Kh : Ah) + ((size_t)t * r + (j < cl * r ? j : 0)) * dk;
    };
    const int rpp = nthr / pl.vpr > 0 ? nthr / pl.vpr : 1;      // rows per pass of the workgroup
    const int pr0 = tid / pl.vpr, px = tid % pl.vpr;
    u32x4 pre[kPre];
    T prev[kPreV], preb{};
    auto fetch = [&](int t) {                                   // prefetch == 1: rows are whole pieces
        const int cl = L - t < tb ? L - t : tb;
#pragma unroll
        for (int q = 0; q < kPre; ++q) {
            const int i = pr0 + q * rpp;
            if (pr0 < rpp && i < nrows) pre[q] = *reinterpret_cast<const u32x4 *>(row_src(i, t, cl) + px * VEC);
        }
#pragma unroll
        for (int q = 0; q < kPreV; ++q) {
            const int i = tid + q * nthr;
            if (i < krows * rowsWG) {
                const int j = i / rowsWG, m = i % rowsWG;
                prev[q] = Vh[((size_t)t * r + (j < cl * r ? j : 0)) * dv + (base + m < dv ? base + m : 0)];
            }
        }
        if (!kDrivers && tid < krows) preb = bh[(size_t)t * r + (tid < cl * r ? tid : 0)];
    };
    auto stage = [&](int t) {
        if (pl.prefetch) {
#pragma unroll
            for (int q = 0; q < kPre; ++q) {
                const int i = pr0 + q * rpp;
                if (pr0 < rpp && i < nrows) put16(rows + (size_t)i * DKP + px * VEC, pre[q], T{});
            }
#pragma unroll
            for (int q = 0; q < kPreV; ++q) {
                const int i = tid + q * nthr;
                if (i < krows * rowsWG) vs[i] = as_f32(prev[q]);
            }
            if (!kDrivers && tid < krows) bs[tid] = as_f32(preb);
            return;
        }
        const int cl = L - t < tb ? L - t : tb;
        for (int i0 = 0; i0 < nrows; i0 += rpp)
            for (int x = px; x < pl.vpr; x += nthr) {
                const int i = i0 + pr0;
                if (pr0 >= rpp || i >= nrows) continue;
                const T *p = row_src(i, t, cl);
                if (pl.vec) put16(rows + (size_t)i * DKP + x * VEC, *reinterpret_cast<const u32x4 *>(p + x * VEC), T{});
                else rows[(size_t)i * DKP + x] = as_f32(p[x]);
            }
        for (int i = tid; i < cl * r * rowsWG; i += nthr) {
            const int j = i / rowsWG, m = i % rowsWG;
            vs[i] = base + m < dv ? as_f32(Vh[((size_t)t * r + j) * dv + base + m]) : 0.f;
        }
        if (!kDrivers)
            for (int i = tid; i < cl * r; i += nthr) bs[i] = as_f32(bh[(size_t)t * r + i]);
    };
    auto load_row = [&](int i, float (&x)[CS]) {
#pragma unroll
        for (int q = 0; q < CV; ++q) {
            const f32x4 v = *reinterpret_cast<const f32x4 *>(rows + (size_t)i * DKP + 4 * (c + LPR * q));
#pragma unroll
            for (int e = 0; e < 4; ++e) x[4 * q + e] = v[e];
        }
    };
    auto dot = [&](const float (&x)[CS]) {                      // two partial sums: half the dependent chain
        float s0 = S[0] * x[0], s1 = S[1] * x[1];
#pragma unroll
        for (int i = 2; i < CS; i += 2) {
            s0 = fmaf(S[i], x[i], s0);
            s1 = fmaf(S[i + 1], x[i + 1], s1);
        }
        return s0 + s1;
    };

    if (pl.prefetch && a.t0 < L) fetch(a.t0);
    for (int t0 = a.t0; t0 < L; t0 += tb) {
        const int cl = L - t0 < tb ? L - t0 : tb;
        stage(t0);
        __syncthreads();
        if (pl.prefetch) fetch(t0 + tb < L ? t0 + tb : t0);
        if constexpr (R > 0) {
            const int steps = cl * nsub;                        // R = 1: virtual tokens
            float kd[R][CS], w[R];
#pragma unroll
            for (int j = 0; j < R; ++j) {
                load_row(j, kd[j]);
                w[j] = row_sum<LPR>(dot(kd[j]));
            }
            int sub = 0, t = 0;
#pragma unroll 1
            for (int s = 0; s < steps; ++s) {
                const int nx = s + 1 < steps ? s + 1 : s;
                float kn[R][CS], ku[kDrivers ? R : 1][CS], q[CS], u[R];
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    if constexpr (kDrivers) load_row(urow0 + s * R + j, ku[j]);
                    load_row(nx * R + j, kn[j]);
                    const float v = vs[(s * R + j) * rowsWG + rowl];
                    u[j] = kDrivers ? v + w[j] : bs[s * R + j] * (v - w[j]);
                }
                const bool out = ++sub == nsub;
                if (out) {
                    load_row(qrow0 + t, q);
                    sub = 0;
                }
#pragma unroll
                for (int j = 0; j < R; ++j)
#pragma unroll
                    for (int i = 0; i < CS; ++i) S[i] = fmaf(u[j], kDrivers ? ku[kDrivers ? j : 0][i] : kd[j][i], S[i]);
                float o = out ? dot(q) : 0.f;
#pragma unroll
                for (int j = 0; j < R; ++j) w[j] = dot(kn[j]);
                if (out) {
                    o = row_sum<LPR>(o);
                    if (c == 0) os[t * rowsWG + rowl] = o;
                    ++t;
                }
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    w[j] = row_sum<LPR>(w[j]);
#pragma unroll
                    for (int i = 0; i < CS; ++i) kd[j][i] = kn[j][i];
                }
            }
        } else {
            for (int t = 0; t < cl; ++t) {
                float x[CS];
                for (int j = 0; j < r; ++j) {
                    load_row(t * r + j, x);
                    const float w = row_sum<LPR>(dot(x)), v = vs[(t * r + j) * rowsWG + rowl];
                    us[j] = kDrivers ? v + w : bs[t * r + j] * (v - w);   // every lane: read back by the one that wrote it
                }
                for (int j = 0; j < r; ++j) {
                    load_row(urow0 + t * r + j, x);
                    const float u = us[j];
#pragma unroll
                    for (int i = 0; i < CS; ++i) S[i] = fmaf(u, x[i], S[i]);
                }
                load_row(qrow0 + t, x);
                const float o = row_sum<LPR>(dot(x));
                if (c == 0) os[t * rowsWG + rowl] = o;
            }
        }
        __syncthreads();
        for (int i = tid; i < cl * rowsWG; i += nthr) {
            const int t = i / rowsWG, m = i % rowsWG;
            if (base + m < dv) Oh[(size_t)(t0 + t) * dv + base + m] = from_f32<T>(os[i]);
        }
    }
    if (a.SL && live) {
        float *sl = a.SL + (head * (size_t)dv + row) * dk;
#pragma unroll
        for (int i = 0; i < CV; ++i) {
            const int x = 4 * (c + LPR * i);
            if (dk % 4 == 0) {
                if (x < dk) *reinterpret_cast<f32x4 *>(sl + x) = f32x4{S[4 * i], S[4 * i + 1], S[4 * i + 2], S[4 * i + 3]};
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (x + e < dk) sl[x + e] = S[4 * i + e];
            }
        }
    }
}

// A few tokens: a wavefront owns kFewRows rows of S, 16 lanes to a row, and asks for all of them at once; k (a, b) and q of a
// token come straight from memory into the registers of the lanes that need them (every wavefront of a head reads the
// same ones, out of L2), one token ahead.  No LDS, no barrier, and 8 KB of S per wavefront in flight at d_k = 128, where
// the body above has 2 KB and waits for its staging in between.  Bounded by the state's
// traffic: 1024 heads x 1 token, d = 128, r = 2 are 134 MB in 24 us (5.6 TB/s; 42 us in the body above).
constexpr int kFewRows = 16;

template <typename T, bool kDrivers, int CS, int R>
__device__ __forceinline__ void generic_few(const GenericArgs<T> &a)
{
    constexpr int LPR = 16, CV = CS / 4, NG = kFewRows * LPR / 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c = lane % LPR, rr = lane / LPR;
    const size_t head = blockIdx.x % (unsigned)a.heads;
    const int base = ((int)(blockIdx.x / (unsigned)a.heads) * (int)(blockDim.x >> 6) + wave) * kFewRows;
    if (base >= a.dv) return;                                  // whole wavefronts; no barrier below
    const int L = a.L, dk = a.dk, dv = a.dv, r = a.r;
    const int nsub = R == 1 ? r : 1;                           // r == 1, or the product form
    const T *Qh = a.Q + head * (size_t)L * dk;
    const T *Kh = a.K + head * (size_t)L * r * dk;
    const T *Ah = kDrivers ? a.beta + head * (size_t)L * r * dk : Kh;
    const T *Vh = a.V + head * (size_t)L * r * dv;
    const T *bh = a.beta + head * (size_t)L * r;
    T *Oh = a.O + head * (size_t)L * dv;
    f32x4 S[NG][CV];
    int row[NG];
#pragma unroll
    for (int n = 0; n < NG; ++n) {
        row[n] = base + n * (64 / LPR) + rr;
        const float *s0 = a.S0 ? a.S0 + (head * (size_t)dv + (row[n] < dv ? row[n] : dv - 1)) * dk : nullptr;
#pragma unroll
        for (int i = 0; i < CV; ++i) {
            const int x = 4 * (c + LPR * i);
            S[n][i] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (s0 && x < dk) S[n][i] = *reinterpret_cast<const f32x4 *>(s0 + x);
        }
    }
    struct Token {
        Raw4<T> k[R][CV], u[kDrivers ? R : 1][CV], q[CV];
        T v[R][NG], b[R];
    };
    // virtual tokens s R .. s R + R - 1 (sub-update s % nsub of token s / nsub)
    auto fetch = [&](int s, Token &t) {
        const size_t v0 = (size_t)s * R;
#pragma unroll
        for (int j = 0; j < R; ++j) {
#pragma unroll
            for (int i = 0; i < CV; ++i) {
                const int x = 4 * (c + LPR * i), xx = x < dk ? x : 0;
                t.k[j][i] = Raw4<T>::read(Ah + (v0 + j) * dk + xx);
                if constexpr (kDrivers) t.u[j][i] = Raw4<T>::read(Kh + (v0 + j) * dk + xx);
            }
#pragma unroll
            for (int n = 0; n < NG; ++n) t.v[j][n] = Vh[(v0 + j) * dv + (row[n] < dv ? row[n] : dv - 1)];
            if constexpr (!kDrivers) t.b[j] = bh[v0 + j];
        }
#pragma unroll
        for (int i = 0; i < CV; ++i) {
            const int x = 4 * (c + LPR * i);
            t.q[i] = Raw4<T>::read(Qh + (size_t)(s / nsub) * dk + (x < dk ? x : 0));
        }
    };
    auto dot = [&](const f32x4 (&x)[CV], const f32x4 (&y)[CV]) {
        float s0 = 0.f, s1 = 0.f;
#pragma unroll
        for (int i = 0; i < CV; ++i) {
            s0 = fmaf(x[i][0], y[i][0], s0);
            s1 = fmaf(x[i][1], y[i][1], s1);
            s0 = fmaf(x[i][2], y[i][2], s0);
            s1 = fmaf(x[i][3], y[i][3], s1);
        }
        return row_sum<LPR>(s0 + s1);
    };
    // columns beyond d_k were read from column 0: zero in the rows of the token, as they are in S
    auto widen = [&](const Raw4<T> (&x)[CV], f32x4 (&y)[CV]) {
#pragma unroll
        for (int i = 0; i < CV; ++i) y[i] = 4 * (c + LPR * i) < dk ? x[i].widen() : f32x4{0.f, 0.f, 0.f, 0.f};
    };
    const int steps = L * nsub;
    auto step = [&](int s, const Token &t) {
        f32x4 k[R][CV], q[CV];
        float u[R][NG];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            widen(t.k[j], k[j]);
#pragma unroll
            for (int n = 0; n < NG; ++n) {
                const float w = dot(S[n], k[j]), v = as_f32(t.v[j][n]);
                u[j][n] = kDrivers ? v + w : as_f32(t.b[j]) * (v - w);
            }
        }
#pragma unroll
        for (int j = 0; j < R; ++j) {
            if constexpr (kDrivers) widen(t.u[j], k[j]);
#pragma unroll
            for (int n = 0; n < NG; ++n)
#pragma unroll
                for (int i = 0; i < CV; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e) S[n][i][e] = fmaf(u[j][n], k[j][i][e], S[n][i][e]);
        }
        if (nsub == 1 || (s + 1) % nsub == 0) {
            widen(t.q, q);
#pragma unroll
            for (int n = 0; n < NG; ++n) {
                const float o = dot(S[n], q);
                if (c == 0 && row[n] < dv) Oh[(size_t)(s / nsub) * dv + row[n]] = from_f32<T>(o);
            }
        }
    };
    Token even, odd;
    fetch(0, even);
    for (int s = 0; s < steps; s += 2) {
        fetch(s + 1 < steps ? s + 1 : s, odd);
        step(s, even);
        if (s + 1 >= steps) break;
        fetch(s + 2 < steps ? s + 2 : s + 1, even);
        step(s + 1, odd);
    }
    if (a.SL)
#pragma unroll
        for (int n = 0; n < NG; ++n)
#pragma unroll
            for (int i = 0; i < CV; ++i) {
                const int x = 4 * (c + LPR * i);
                if (row[n] < dv && x < dk) *reinterpret_cast<f32x4 *>(a.SL + (head * (size_t)dv + row[n]) * dk + x) = S[n][i];
            }
}

// Rows too long for registers (d_k > 512) or too many ranks for the staging plan: a wavefront per row, the
// row and the u_j of a token in LDS, operands straight from memory.
template <typename T, bool kDrivers>
__device__ __forceinline__ void generic_long_rows(const GenericArgs<T> &a, const GenericPlan &pl, float *smem)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const size_t head = blockIdx.x % (unsigned)a.heads;
    const int row = (int)(blockIdx.x / (unsigned)a.heads) * pl.waves + wave;
    if (row >= a.dv) return;                                   // whole wavefronts; no barrier below
    const int L = a.L, dk = a.dk, dv = a.dv, r = a.r, nsub = a.product ? r : 1, rs = a.product ? 1 : r;
    float *S = smem + (size_t)wave * (dk + r), *us = S + dk;
    auto sum = [&](const T *x) {
        float s = 0.f;
        for (int i = lane; i < dk; i += 64) s = fmaf(S[i], as_f32(x[i]), s);
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) s += __shfl_xor(s, m);
        return s;
    };
    for (int i = lane; i < dk; i += 64) S[i] = a.S0 ? a.S0[(head * (size_t)dv + row) * dk + i] : 0.f;
    for (int t = a.t0; t < L; ++t) {
        for (int sub = 0; sub < nsub; ++sub) {
            const size_t v0 = (head * (size_t)L + t) * r + (size_t)sub * rs;
            for (int j = 0; j < rs; ++j) {
                const float w = sum((kDrivers ? a.beta : a.K) + (v0 + j) * dk), v = as_f32(a.V[(v0 + j) * dv + row]);
                us[j] = kDrivers ? v + w : as_f32(a.beta[v0 + j]) * (v - w);   // every lane: read back by the one that wrote it
            }
            for (int j = 0; j < rs; ++j) {
                const float u = us[j];
                const T *k = a.K + (v0 + j) * dk;
                for (int i = lane; i < dk; i += 64) S[i] = fmaf(u, as_f32(k[i]), S[i]);
            }
        }
        const float o = sum(a.Q + (head * (size_t)L + t) * dk);
        if (lane == 0) a.O[(head * (size_t)L + t) * dv + row] = from_f32<T>(o);
    }
    if (a.SL)
        for (int i = lane; i < dk; i += 64) a.SL[(head * (size_t)dv + row) * dk + i] = S[i];
}

}  // namespace

// kDrivers == false: (K, V, beta) are keys, values, betas of the delta rule.
// kDrivers == true:  (K, V, beta) are (B, Atil, A) of the general recurrence (beta: [.., r, d_k]).
// One overload per row shape, told apart by its last parameter, so that each gets registers of its own.
template <int LPR, int CS, int R> struct RowShape {};
struct LongRows {};
template <int CS, int R> struct FewTokens {};     // 16 lanes to a row, CS columns a lane
template <int DT> struct BlockShape {};          // d_k padded to 16 DT (pf_generic_block.h)

#define PF_RANKS(X, LPR, CS) X(LPR, CS, 1) X(LPR, CS, 2) X(LPR, CS, 4) X(LPR, CS, 0)
#define PF_ROW_SHAPES(X) \
    PF_RANKS(X, 4, 4) PF_RANKS(X, 8, 4) PF_RANKS(X, 16, 4) PF_RANKS(X, 16, 8) PF_RANKS(X, 64, 4) PF_RANKS(X, 64, 8)

#define X(LPR, CS, R)                                                                                           \
    template <typename T, bool kDrivers>                                                                        \
    __global__ __launch_bounds__(256) void generic_kernel(GenericArgs<T> a, GenericPlan pl, RowShape<LPR, CS, R>) \
    {                                                                                                           \
        extern __shared__ __attribute__((aligned(16))) float gsmem[];                                           \
        generic_rows<T, kDrivers, LPR, CS, R>(a, pl, gsmem);                                                    \
    }
PF_ROW_SHAPES(X)
#undef X

#define PF_FEW_SHAPES(X) X(4, 1) X(4, 2) X(4, 4) X(8, 1) X(8, 2) X(8, 4)
#define X(CS, R)                                                                                       \
    template <typename T, bool kDrivers>                                                               \
    __global__ __launch_bounds__(256) void generic_kernel(GenericArgs<T> a, FewTokens<CS, R>)          \
    {                                                                                                  \
        generic_few<T, kDrivers, CS, R>(a);                                                            \
    }
PF_FEW_SHAPES(X)
#undef X

#define PF_BLOCK_SHAPES(X) X(1) X(2) X(3) X(4) X(6) X(8)
#define X(DT)                                                                                          \
    template <typename T, bool kDrivers>                                                               \
    __global__ __launch_bounds__((BlockLds<kDrivers, DT>::threads)) void generic_kernel(GenericArgs<T> a, int C, BlockShape<DT>) \
    {                                                                                                  \
        extern __shared__ __attribute__((aligned(16))) float gsmem[];                                  \
        generic_block<T, kDrivers, DT>(a, C, gsmem);                                                   \
    }
PF_BLOCK_SHAPES(X)
#undef X

template <typename T, bool kDrivers>
__global__ __launch_bounds__(256) void generic_kernel(GenericArgs<T> a, GenericPlan pl, LongRows)
{
    extern __shared__ __attribute__((aligned(16))) float gsmem[];
    generic_long_rows<T, kDrivers>(a, pl, gsmem);
}

namespace {

// Lanes and columns by d_k (the smallest padded row that holds it), tokens per staging block by what a
// thread can carry in registers for the next block, at most `chunk`, and by 64 KiB of LDS.
GenericPlan plan_generic(int dk, int dv, int r, int chunk, int tokens, bool drivers, int esize)
{
    GenericPlan p{};
    const int vec = 16 / esize;
    p.vec = dk % vec == 0;
    p.vpr = p.vec ? dk / vec : dk;
    if (dk <= 16) { p.lpr = 4; p.cs = 4; }
    else if (dk <= 32) { p.lpr = 8; p.cs = 4; }
    else if (dk <= 64) { p.lpr = 16; p.cs = 4; }
    else if (dk <= 128) { p.lpr = 16; p.cs = 8; }
    else if (dk <= 256) { p.lpr = 64; p.cs = 4; }
    else if (dk <= 512) { p.lpr = 64; p.cs = 8; }
    const int cap = chunk < tokens ? chunk : (tokens > 0 ? tokens : 1);
    if (p.cs) {
        const int rpw = 64 / p.lpr, dkp = p.lpr * p.cs;
        p.waves = (dv + rpw - 1) / rpw < 4 ? (dv + rpw - 1) / rpw : 4;
        const int nthr = 64 * p.waves, rows_wg = p.waves * rpw, rpp = nthr / p.vpr;
        auto lds = [&](int tb) {
            const size_t k = (size_t)tb * r;
            return 4 * ((k * (drivers ? 2 : 1) + tb) * dkp + k * rows_wg + (drivers ? 0 : k) + (size_t)tb * rows_wg +
                        (size_t)rows_wg * r);
        };
        auto carried = [&](int tb) {
            const size_t k = (size_t)tb * r, rows = k * (drivers ? 2 : 1) + tb;
            return p.vec && rpp > 0 && rows <= (size_t)kPre * rpp && k * rows_wg <= (size_t)kPreV * nthr && k <= (size_t)nthr;
        };
        int tb = cap;
        while (tb > 1 && !(carried(tb) && lds(tb) <= 65536)) tb = tb > 16 ? tb - tb / 4 : tb - 1;
        p.prefetch = carried(tb) && lds(tb) <= 65536;
        if (!p.prefetch) {
            tb = cap;
            while (tb > 1 && lds(tb) > 65536) tb = (tb + 1) / 2;
        }
        p.tb = tb;
        p.lds = lds(tb);
        p.tiles = (dv + rows_wg - 1) / rows_wg;
    }
    if (!p.cs || p.lds > kMaxLdsBytes) {
        p.cs = 0;
        const size_t per_wave = 4 * ((size_t)dk + r);
        p.waves = 4;
        while (p.waves > 1 && p.waves * per_wave > kMaxLdsBytes) p.waves /= 2;
        p.lds = p.waves * per_wave;
        p.tiles = (dv + p.waves - 1) / p.waves;
    }
    return p;
}

// Whether the body for a few tokens serves the call (steps: virtual tokens in the product form, else tokens).  It waits
// for every token's rows to come out of L2, which many wavefronts hide from each other and few do not.  The body above /
// this one, us, d = 128, r = 2, bf16:
//   1024 heads   1 token 42.0 / 24.1    4 50.6 / 32.0    8 65.2 / 46.2    12 82.5 / 61.4
//   128 heads    1 token  8.4 /  5.1    4 10.2 /  7.6    8 12.8 / 11.0    16, r = 1 12.9 / 16.1
//   8 heads      1 token  5.1 /  4.5    2  4.8 /  4.8    4  5.4 /  6.4     8  6.6 / 9.8
// and d = 64 (half the wavefronts): 1024 heads 1 token 17.4 / 7.3, 16 r = 1 30.0 / 26.4; 128 heads 4 5.6 / 5.5, 8 6.8 / 8.0.
// Rows that a token brings cost it registers and time (operands: 1 at r = 1, d_k up to 64; rank 4, drivers' two arrays and
// wider rows multiply it up to 16), and a wavefront with few of its 16 rows in use costs as much as a full one:
//   8 operands, 2 tokens: d = 128, r = 4, 22 heads 5.9 / 6.5, 32 6.0 / 6.7; drivers d = 128, r = 2, 15 heads 5.2 / 5.6
//   16: drivers, d = 128, r = 4, 8 heads, 1 token 5.1 / 5.6; fp32, d_v = 20, 574 heads, 8 tokens 28 / 37, d = 128, 508 heads, 4 48 / 37
//   bf16, r = 1, d = 128, d_v = 100, 134 heads, 6 tokens 9.2 / 10.3
//   d_v = 1 on 1358 heads, d_k = 128, r = 4, 7 tokens 11.7 / 23.3; d_v = 8, drivers, fp32, 1981 heads, 1 token 10.9 / 23.7
bool few_tokens(int heads, int dk, int dv, int ranks, int steps, bool drivers, int esize)
{
    if (dk <= 32 || dk > 128 || dk % 4 != 0 || steps < 1 || steps > 16) return false;
    const long long waves = (long long)heads * ((dv + kFewRows - 1) / kFewRows);
    const bool wide = dk > 64, filled = dv >= kFewRows;
    const int operands = ranks * (drivers ? 2 : 1) * (wide ? 2 : 1);
    if (steps <= 2) return operands < 8 || steps * operands <= 8 || (filled && waves >= 300);
    return filled && steps <= waves / (operands == 16 && esize == 4 ? 256 : (operands == 2 && wide && esize == 2 ? 160 : 128));
}

// Tiles of 16 columns that hold d_k, for the body that takes 16 virtual tokens at a time (0: no instance).
int block_tiles(int dk, int r)
{
    if (dk < 16 || dk > 128 || r > kBlockVT) return 0;    // (below: block_pays)
    const int dt = (dk + 15) / 16;
    return dt <= 4 ? dt : (dt <= 6 ? 6 : 8);
}

// Whether that body serves the call.  A workgroup costs it 5 to 7 us before the second block of tokens and a compute unit
// runs one at a time, while the rows' many wavefronts share one, and at r = 2 and 4 hold a token's products side by side (not in
// the product form, which is taken as r = 3: 64 heads x 29 tokens, r = 4, d = 128, 45.5 / 48.5).  fp32, us, rows / blocks at virtual tokens a head:
//                            12          24          48          96         192         384 (400: r = 1)
//   256 workgroups
//     d_k = 64, r = 1     6.9 / 6.0  10.0 / 6.7  15.2 / 7.4  26.3 / 10.3                 96.4 / 28.3
//     d_k = 128, r = 2    6.7 / 7.3   8.5 / 8.3  12.8 / 9.2  20.0 / 14.8  35.8 / 23.6
//     d_k = 64, r = 4                 6.7 / 6.6   9.0 / 7.3  14.4 / 9.9   23.1 / 15.9    41.6 / 26.5
//   512 workgroups
//     d_k = 64, r = 1     7.5 / 10.5 10.8 / 11.8 16.0 / 13.1 28.1 / 18.8                104.3 / 54.8
//     d_k = 64, r = 2     6.8 / 10.5  8.3 / 11.8 11.8 / 12.9 18.6 / 18.5  32.1 / 30.0
//     d_k = 64, r = 4                 7.9 / 11.7 10.6 / 13.1 16.9 / 18.4  27.3 / 29.9    49.9 / 51.1
//     d_k = 128, r = 2    7.9 / 13.2  9.9 / 15.1 15.1 / 17.1 23.9 / 27.5  42.5 / 45.0   (800: 156.4 / 156.2)
//   800 workgroups
//     d_k = 64, r = 1     9.2 / 19.3 13.8 / 22.1 20.8 / 24.5 36.0 / 35.3                 129 / 108
//     d_k = 128, r = 1   11.5 / 25.0 18.0 / 28.3 27.3 / 31.9 48.2 / 53.8                 175 / 165
//     d_k = 64, r = 2                10.3 / 21.8 16.7 / 24.6 25.4 / 35.0  44.8 / 57.7
// and r = 3 at 512: d_k = 64 72 tokens 19.3 / 17.5, d_k = 128 144 39.3 / 39.6; at 800, d_k = 64, 288 73.1 / 89.0.
// Rows of up to 32 columns cost the rows' body less, 8 or 16 of them to a wavefront: r = 1, bf16, chunk 64, four rounds of
// workgroups d = 16 0.68 to 0.98 of its time, d = 32 0.31 to 1.15; six and seven 0.66 to 1.59; 12 to 16 1.3 to 2.7 (fp32 the
// same: 1387 heads x 198 tokens, d_k = 16, d_v = 96 188 / 385).  The rows' body reads bf16 rows of no whole 16 bytes by elements: 698 heads
// (six rounds) x 473 tokens, d = 20, 172 / 141, 601 x 334 118 / 91.
// d_k that is no multiple of four is read element by element when it is staged, not requested ahead.  In bf16, beyond 16
// columns, that pays with one round of workgroups, with two only while the inputs stay in L2, and more of them not:
//   two rounds   d = 33, r = 1, 241 tokens 76 / 72, d = 31, 595 187 / 200, d = 17, 730 192 / 234, r = 2, 348 63 / 79,
//                d = 127, 148 109 / 133        ten   1275 heads x 413, d = 17 168 / 636
//   one, r = 4   d = 33, 140 tokens 29 / 16, d = 65, 980 236 / 255, d = 127, 676 258 / 275, 2092 816 / 901
// Where it would lose digits the rows' body stays, whatever the time.  A block sums a token's products more often (K S^T, T R, U^T P^T,
// K^T U), which rounding S once a block makes up for from some tokens or columns on.  fp32, distance from 64 bits, blocks / rows, O and
// S_L, the worse of delta rule, product form and drivers, with and without S_0, mean of 8 seeds and 16 heads:
//                 16 tokens      24             32             40             48             64             128
//   d_k = 12     1.17, 1.18    1.13, 1.02     1.13, 1.07     1.10, 0.99     1.10, 1.03     1.09, 1.01     1.07, 1.01
//   d_k = 16     1.11, 1.06    1.06, 0.95     1.05, 0.96     1.03, 0.89     1.02, 0.92     1.00, 0.91     0.96, 0.88
//   d_k = 20     1.10, 1.03    1.06, 0.93     1.03, 0.93     1.01, 0.87     0.99, 0.88     0.97, 0.86     0.92, 0.82
//   d_k = 24     1.04, 1.00    1.01, 0.89     0.99, 0.89     0.98, 0.83     0.96, 0.84     0.93, 0.81     0.87, 0.76
//   d_k = 64     1.01, 0.90    0.97, 0.81     0.94, 0.78     0.91, 0.73     0.88, 0.70     0.84, 0.66     0.73, 0.57
//   d_k = 96     1.01, 0.89    0.99, 0.80     0.97, 0.76     0.93, 0.71     0.91, 0.68     0.85, 0.63     0.74, 0.54
// (d_k = 8: 1.2 to 1.3 at any length.)  O in bf16 is rounded far above these; there S_L alone counts.
bool block_pays(long long workgroups, int dk, int ranks, long long virtual_tokens, int esize)
{
    if (virtual_tokens <= (dk < 24 ? (esize == 4 ? 40 : 16) : (esize == 4 ? 16 : 0))) return false;
    const long long cus = device_cu_count(), rounds = (workgroups + cus - 1) / cus;
    const bool together = ranks == 2 || ranks == 4, wide = dk > 64;
    if (esize == 2 && dk % 4 != 0 && dk > 16) {
        if (rounds == 1) return virtual_tokens > (together ? 28 : 16) && (ranks != 4 || dk <= 32 || virtual_tokens <= 200);
        return rounds == 2 && !together && !wide && virtual_tokens > 60 && virtual_tokens <= 200;
    }
    // (bf16: 16 heads x 12 tokens, d = 128, r = 2 8.3 / 8.8; drivers, d = 64, r = 4, 7 tokens 6.8 / 7.4)
    if (rounds == 1) return virtual_tokens > (together ? (esize == 2 && dk >= 64 && dk % 8 == 0 ? 28 : 20) : 12);
    if (ranks == 1) return virtual_tokens > (rounds == 2 ? 32 : (wide ? 250 : 100)) && (dk > 32 || rounds <= (esize == 2 && dk % 8 == 4 && virtual_tokens > 200 ? 6 : 4));
    if (rounds > 2 || ranks == 4) return false;
    return ranks == 2 ? !wide && virtual_tokens > 100 : virtual_tokens > (wide ? 150 : 60);
}

}  // namespace

// LDS of the chunk-wise form of Theorem 3.2 at these dimensions (S, K, W, U, Q, G, P in fp32).  No kernel
// here needs it, the recurrence above takes less at any chunk; it is the documented line of the interface
// between dimensions that are taken and refused, and of the chunk that pf_delta_fwd_block names.
size_t generic_lds_bytes(int dk, int dv, int r, int chunk)
{
    const size_t n = (size_t)chunk * r;
    return 4 * ((size_t)(dv + 2 * n + chunk) * (dk + 1) + n * (dv + 1) + (n + chunk) * (n + 1));
}

template <typename T, bool kDrivers>
static hipError_t launch_generic_instance(const void *Q, const void *K, const void *V, const void *beta,
                                          const float *S0, void *O, float *SL, int heads, int L, int dk, int dv,
                                          int r, int chunk, int t0, bool product, hipStream_t stream)
{
    const GenericArgs<T> a{(const T *)Q, (const T *)K, (const T *)V, (const T *)beta, S0, (T *)O, SL,
                           heads, L, dk, dv, r, t0, product ? 1 : 0};
    const int ranks = product ? 1 : r;
    bool taken = false;
    hipError_t done = hipSuccess;
    auto blocks = [&](auto dt) {
        using Ld = BlockLds<kDrivers, decltype(dt)::value>;
        using Shape = BlockShape<decltype(dt)::value>;
        const long long grid = (long long)heads * ((dv + 15) / 16);
        if (grid > 0x7fffffffLL || !block_pays(grid, dk, product && r > 1 ? 3 : r, (long long)(L - t0) * r, (int)sizeof(T))) return;
        taken = true;
        void (*kern)(GenericArgs<T>, int, Shape) = generic_kernel<T, kDrivers>;
        if (Ld::bytes > 65536) {
            static std::atomic<uint64_t> armed{0};
            done = arm_dynamic_lds(armed, reinterpret_cast<const void *>(kern), Ld::bytes);
            if (done != hipSuccess) return;
        }
        hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(Ld::threads), Ld::bytes, stream, a, kBlockVT / r, Shape{});
        done = hipGetLastError();
    };
    switch (block_tiles(dk, r)) {
#define X(N) case N: blocks(std::integral_constant<int, N>{}); break;
        PF_BLOCK_SHAPES(X)
#undef X
    default: break;
    }
    if (taken) return done;
    if (t0 == 0 && L <= 16 && few_tokens(heads, dk, dv, ranks, L * (r / ranks), kDrivers, (int)sizeof(T)) && (ranks == 1 || ranks == 2 || ranks == 4)) {
        const int per_wg = 4 * kFewRows, tiles = (dv + per_wg - 1) / per_wg;
        if ((long long)heads * tiles > 0x7fffffffLL) return hipErrorInvalidValue;
        auto launch = [&](auto shape) -> hipError_t {
            void (*kern)(GenericArgs<T>, decltype(shape)) = generic_kernel<T, kDrivers>;
            hipLaunchKernelGGL(kern, dim3((unsigned)heads * tiles), dim3(256), 0, stream, a, shape);
            return hipGetLastError();
        };
#define X(CS, R) \
        if ((dk > 64 ? 8 : 4) == CS && ranks == R) return launch(FewTokens<CS, R>{});
        PF_FEW_SHAPES(X)
#undef X
    }
    const GenericPlan pl = plan_generic(dk, dv, r, chunk, L - t0, kDrivers, (int)sizeof(T));
    if (pl.lds > kMaxLdsBytes || (long long)heads * pl.tiles > 0x7fffffffLL) return hipErrorInvalidValue;
    auto launch = [&](auto shape) -> hipError_t {
        void (*kern)(GenericArgs<T>, GenericPlan, decltype(shape)) = generic_kernel<T, kDrivers>;
        if (pl.lds > 65536) {
            // the opt-in is for the largest size any call may ask for, so that it is made once per device
            static std::atomic<uint64_t> armed{0};
            hipError_t e = arm_dynamic_lds(armed, reinterpret_cast<const void *>(kern), kMaxLdsBytes);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kern, dim3((unsigned)heads * pl.tiles), dim3(64 * pl.waves), pl.lds, stream, a, pl, shape);
        return hipGetLastError();
    };
    if (pl.cs == 0) return launch(LongRows{});
    const int rank_shape = ranks == 1 || ranks == 2 || ranks == 4 ? ranks : 0;
#define X(LPR, CS, R) \
    if (pl.lpr == LPR && pl.cs == CS && rank_shape == R) return launch(RowShape<LPR, CS, R>{});
    PF_ROW_SHAPES(X)
#undef X
    return hipErrorInvalidValue;
}

hipError_t launch_generic(const void *Q, const void *K, const void *V, const void *beta, const float *S0,
                          void *O, float *SL, int heads, int L, int dk, int dv, int r, int chunk,
                          bool is_bf16, hipStream_t stream, int t0, bool product)
{
    return is_bf16 ? launch_generic_instance<uint16_t, false>(Q, K, V, beta, S0, O, SL, heads, L, dk, dv, r, chunk, t0, product, stream)
                   : launch_generic_instance<float, false>(Q, K, V, beta, S0, O, SL, heads, L, dk, dv, r, chunk, t0, product, stream);
}

hipError_t launch_generic_drivers(const void *Q, const void *A, const void *Atil, const void *Bm, const float *S0,
                                  void *O, float *SL, int heads, int L, int dk, int dv, int r, int chunk,
                                  bool is_bf16, hipStream_t stream, int t0)
{
    return is_bf16 ? launch_generic_instance<uint16_t, true>(Q, Bm, Atil, A, S0, O, SL, heads, L, dk, dv, r, chunk, t0, false, stream)
                   : launch_generic_instance<float, true>(Q, Bm, Atil, A, S0, O, SL, heads, L, dk, dv, r, chunk, t0, false, stream);
}

}  // namespace pf

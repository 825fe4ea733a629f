// Segment-parallel form of the state scan: step 3 of Section 3 of ParallelFlow (arXiv
// 2504.00492) as an actual scan over segments of the sequence instead of one hand-over chain
// per head, for workloads with too few heads to fill the GPU.
//
// The map of a segment (a run of consecutive flow blocks) on the state is affine,
//     S_out = S_in P_seg + H_seg,        P_seg in R^{d_k x d_k},  H_seg in R^{d_v x d_k},
// with P_seg the ordered product of the segment's transitions (Proposition 2.1) and H_seg what
// the segment writes into a zero state; affine maps compose, (P1, H1) then (P2, H2) =
// (P1 P2, H1 P2 + H2).  Rows of the state evolve independently, so both come out of the
// chain of the scan kernel, side by side (ChainPlan, PAIR, in pf_chain.h): H_seg is its final state
// from S_0 = 0, and P_seg is its final state when the rows of the identity are fed in and V is zero.
// The kernel here is the composition over the segments of a head; a last pass of the scan kernel
// then runs every segment from its true incoming state.
#include "pf_internal.h"
#include "pf_common.h"

namespace pf {

// One workgroup owns ROWS rows of the state of one head (rows are independent) and walks the segments:
// S <- S P_s + H_s in fp32.  Thread (yg, x4) sums d / kComposeSplit values of y for 4 columns of every row; the
// kComposeSplit partial sums meet in LDS.  A thread's piece of P_{s+1} is in registers before segment s is
// summed: P does not depend on the state, so the chain over the segments never waits for memory.  What bounds it is
// that chain (products and two barriers per segment; 64 KB of P a segment at d = 128).  One column per thread with P read
// as it was needed took 273 us for 4 heads x 8 segments, d = 128.
// Two rows where that gives no more workgroups than compute units, else four: half the products a step of the chain, but the
// whole of P for each workgroup.  The same sums in the same order.  Whole forward, r = 2, us, four rows / two:
//   d = 128   1 head x 131072 tokens  208 / 195    1 x 16384  76.9 / 72.3    2 x 16384  76.7 / 74.4    4 x 8192  68.1 / 66.7
//             8 x 8192 (512 workgroups)  90.6 / 92.0         d = 64   2 x 32768  66.1 / 63.9
// (32 partial sums instead of 16: no faster than two rows where those serve, and another order.)
constexpr int kComposeSplit = 16;

template <int D, int ROWS>
__global__ __launch_bounds__(D / 4 * kComposeSplit) void segment_compose_kernel(
    const float *S0, const float *__restrict__ Pseg, const float *__restrict__ Hseg, float *__restrict__ Sin, float *SL, int G)
{
    constexpr int X4 = D / 4, NTHR = X4 * kComposeSplit, YN = D / kComposeSplit;
    static_assert(ROWS * D <= NTHR, "a thread per state element");
    __shared__ __attribute__((aligned(16))) float cur[ROWS][D], part[kComposeSplit][ROWS][D];
    const int tiles = D / ROWS;
    const size_t head = blockIdx.x / tiles;
    const int r0 = (blockIdx.x % tiles) * ROWS;
    const int tid = threadIdx.x, x = 4 * (tid % X4), yg = tid / X4;
    const bool own = tid < ROWS * D;           // the state element this thread adds up
    const int om = own ? tid / D : 0, ox = tid % D;
    const size_t oel = (size_t)(r0 + om) * D + ox;
    float s = own && S0 ? S0[head * (size_t)D * D + oel] : 0.0f;
    f32x4 p[YN];
    float h = 0.0f;
    auto fetch = [&](int g) {
        const size_t seg = (head * (size_t)G + g) * D * D;
#pragma unroll
        for (int i = 0; i < YN; ++i) p[i] = *reinterpret_cast<const f32x4 *>(Pseg + seg + (size_t)(yg * YN + i) * D + x);
        h = Hseg[seg + oel];
    };
    fetch(0);
    for (int g = 0; g < G; ++g) {
        if (own) {
            cur[om][ox] = s;
            Sin[(head * (size_t)G + g) * D * D + oel] = s;
        }
        s = h;
        __syncthreads();
        f32x4 acc[ROWS];
#pragma unroll
        for (int m = 0; m < ROWS; ++m) acc[m] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < YN; ++i)
#pragma unroll
            for (int m = 0; m < ROWS; ++m) {
                const float c = cur[m][yg * YN + i];
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[m][e] = fmaf(c, p[i][e], acc[m][e]);
            }
        fetch(g + 1 < G ? g + 1 : g);
#pragma unroll
        for (int m = 0; m < ROWS; ++m) *reinterpret_cast<f32x4 *>(&part[yg][m][x]) = acc[m];
        __syncthreads();
        if (own) {
#pragma unroll
            for (int q = 0; q < kComposeSplit; ++q) s += part[q][om][ox];
        }
    }
    if (SL && own) SL[head * (size_t)D * D + oel] = s;
}

int segment_compose_rows(int heads, int d) { return (long long)heads * (d / 2) <= (long long)device_cu_count() ? 2 : 4; }

hipError_t launch_segment_compose(const float *S0, const float *Pseg, const float *Hseg, float *Sin,
                                  float *SL, int heads, int G, int d, hipStream_t stream)
{
    const int rows = segment_compose_rows(heads, d);
#define X(D, ROWS)                                                                                                          \
    if (d == D && rows == ROWS) {                                                                                           \
        hipLaunchKernelGGL((segment_compose_kernel<D, ROWS>), dim3((unsigned)(heads * (D / ROWS))), dim3(D / 4 * kComposeSplit), \
                           0, stream, S0, Pseg, Hseg, Sin, SL, G);                                                          \
        return hipGetLastError();                                                                                           \
    }
    X(64, 2) X(64, 4) X(128, 2) X(128, 4)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace pf

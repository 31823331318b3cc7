// conv2 and conv3 forward in fp32 for many rows: every wave walks rows of its own, without a barrier.
//
// The tiled kernel (g32::k_fwd) stages both operands through LDS, and its waves spend a quarter of the time at the stages'
// barriers and on staging: the vector instructions of a SIMD do not run beside its fp32 matrix instructions, not even those
// of another wave (2.4 of the 64 cycles of a 32x32x2 each).  Here a layer's weights, 132 / 148 KB, lie in LDS once per
// workgroup, one workgroup per CU, and the other operand, 32 rows per wave, comes from memory straight into the registers
// that the matrix instruction reads, a stage (32 of the reduction, a cache line per row) ahead: a stage of both column
// halves takes 2048 cycles of the matrix pipe, which the two waves of a SIMD share, 1.7 us for a load.
// The work is dealt out in units of 32 rows x 32 columns, to every SIMD the same number (+ 1): conv2's 243,000 rows at a
// batch of 1000 are 7.4 row tiles per SIMD and took the time of eight, and are 14.8 units, which take that of 15.
// Products and sums are those of g32::k_fwd<64, 64> in its order: the same bits.
// Bound by the matrix pipe (243,000 x 64 x 512: 105 us at the 151 TFLOP/s that nothing but these instructions reaches).
// At a batch of 1000 conv2 142.6 -> 122.4 us, conv3 99.3 -> 90.2 (of its 3063 units two per pass come to a SIMD too many, 8 us),
// the step 964 -> 941; at 448 496 -> 480, at 160 228.5 -> 224.7.  The input gradients in this form (their weights turned on the way into LDS)
// are no faster where other streams' launches hold compute units: their share of the rows is fixed before they run.
#pragma once
#include "gemm_fp32.h"

namespace rows {
using g32::mfma;
constexpr int THREADS = 512;
typedef __attribute__((address_space(1))) const float *Global;
__device__ __forceinline__ v4f ld4(Global p) { return *reinterpret_cast<__attribute__((address_space(1))) const v4f *>(p); }

struct Seg {
    const float *x, *w, *bias;
    float *y;
    int M;
    int wg_begin, wgs;   // the segment's workgroups
    uint32_t xs;         // elements between consecutive samples of x
};
struct Args {
    Seg seg[3];
    int nseg;
};

// A column's weights in LDS: 16 bytes beyond a multiple of 256, so that the columns of a 16-byte read lie in different banks
template <class G> constexpr int ld() { return G::K + 4; }
template <class G> constexpr int lds_bytes() { return G::N * ld<G>() * 4; }

// NC column blocks from `block` on of one row tile.  row: this lane's row, as an offset, its first stage (a[0]) already
// requested; next: that of the row tile after it.
template <class G, int NC>
__device__ __forceinline__ void tile(const Seg &S, const float *bp, v4f (&a)[2][4], uint32_t row, uint32_t next, int m0, int block, int lane)
{
    constexpr int NST = G::K / 32, LD = ld<G>();
    static_assert(NST % 2 == 0, "stages");
    const int li = lane & 31, h = lane >> 5;
    float bias[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) bias[c] = S.bias[32 * (block + c) + li];
    bp += block * 32 * LD;
    v4f b[2][NC];   // eight of the reduction ahead
#pragma unroll
    for (int c = 0; c < NC; ++c) b[0][c] = g32::ld4(bp + c * 32 * LD);
    v16f acc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[c] = v16f{0};
    // (as a loop of two stages, with its addresses and copies, 132 against 125 us)
#pragma unroll
    for (int st = 0; st < NST; ++st) {
        const Global p = (Global)S.x + (st + 1 < NST ? row + (uint32_t)G::k_off(32 * (st + 1)) : next);
#pragma unroll
        for (int j = 0; j < 4; ++j) a[(st + 1) & 1][j] = ld4(p + 8 * j + 4 * h);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            const int k = 32 * st + 8 * kk;
            if (k + 8 < G::K)
#pragma unroll
                for (int c = 0; c < NC; ++c) b[(kk + 1) & 1][c] = g32::ld4(bp + c * 32 * LD + k + 8);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int c = 0; c < NC; ++c) acc[c] = mfma(a[st & 1][kk][t], b[kk & 1][c][t], acc[c]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    float *y = S.y + ((uint32_t)(m0 + 4 * h) * G::N + 32 * block + li);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        float v[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = fmaxf(acc[c][r] + bias[c], 0.f);
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (m0 + 32 <= S.M || m0 + 4 * h + 8 * (r / 4) + r % 4 < S.M) y[(8 * (r / 4) + r % 4) * G::N + 32 * c] = v[r];
    }
}

template <class G> __global__ __launch_bounds__(THREADS, 1) void k_fwd(Args A)
{
    constexpr int NC = G::N / 32, LD = ld<G>(), CH = G::N * (G::K / 4) / THREADS;
    static_assert(NC == 2 && CH * THREADS == G::N * (G::K / 4) && G::K % 64 == 0 && lds_bytes<G>() <= 160 * 1024, "shape");
    extern __shared__ __attribute__((aligned(16))) float lds_rows[];
    Seg S = A.seg[0];
    if (A.nseg > 1 && (int)blockIdx.x >= A.seg[1].wg_begin) S = A.seg[1];
    if (A.nseg > 2 && (int)blockIdx.x >= A.seg[2].wg_begin) S = A.seg[2];
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // a SIMD's units (waves w and w + 4 run on one SIMD), then this wave's half of them, parted between row tiles
    const uint32_t units = (uint32_t)((S.M + 31) / 32) * NC, simds = 4u * S.wgs, simd = 4u * (blockIdx.x - S.wg_begin) + (wave & 3);
    const int s0 = (int)(simd * units / simds), s1 = (int)((simd + 1) * units / simds);   // (below 2^13 x 2^10)
    const int mid = min(max((s0 + s1 + NC) / 2 / NC * NC, s0), s1);
    int u = wave < 4 ? s0 : mid;
    const int end = wave < 4 ? mid : s1;

    auto row_of = [&](int u) { return G::row_off((uint32_t)min(u / NC * 32 + li, S.M - 1), S.xs); };   // (no row: the last one's)
    uint32_t row = row_of(u);
    v4f a[2][4], w[CH];
#pragma unroll
    for (int j = 0; j < 4; ++j) a[0][j] = ld4((Global)S.x + row + 8 * j + 4 * h);
#pragma unroll
    for (int i = 0; i < CH; ++i) w[i] = g32::ld4(S.w + (tid + i * THREADS) * 4);
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        const int t = tid + i * THREADS;
        *reinterpret_cast<v4f *>(&lds_rows[t / (G::K / 4) * LD + t % (G::K / 4) * 4]) = w[i];
    }
    __syncthreads();
    const float *bp = lds_rows + li * LD + 4 * h;
    while (u < end) {
        const bool both = u % NC == 0 && u + NC <= end;
        const int un = u + (both ? NC : 1);
        const uint32_t next = row_of(un);
        if (both) tile<G, NC>(S, bp, a, row, next, u / NC * 32, 0, lane);
        else tile<G, 1>(S, bp, a, row, next, u / NC * 32, u % NC, lane);
        row = next;
        u = un;
    }
}
}  // namespace rows

// fp32 implicit-GEMM kernels on the CDNA4 matrix cores (v_mfma_f32_32x32x2_f32).
//
// Three kernel shapes cover the whole network (Section 3; the forward /
// backward / calculateGradient split of the paper's Layer class is kept as
// three kernel families):
//   k_fwd   : Y[m][n]  = sum_k  A(m,k) * W[n][k]            (conv1-3, fc1 forward)
//   dgrad   : dX[m][c] = sum_(tap,o) dY(m,tap,o) * W[o][tap][c]   (input gradients)
//   k_wgrad : dW[o][k] = sum_m  dY[m][o] * A(m,k)           (weight gradients)
// A(m,k) is the im2col view of a channel-last activation tensor, formed on the
// fly while staging tiles in LDS; it never exists in memory.
//
// MFMA 32x32x2 operand layout (64-lane wave, lane = 32*h + i):
//   a-operand: A[i][k=h]     b-operand: B[k=h][j=i]
//   result   : acc[r] = D[8*(r/4) + 4*h + r%4][i]
// The reduction order inside a tile is free as long as both operands agree, so
// a lane that reads LDS along k takes 4 consecutive k (one 128-bit read) and
// feeds them to 4 MFMAs: MFMA t pairs k = 4*h + t of both operands.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "net.h"

typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));

namespace g32 {

constexpr int BK = 32;      // reduction elements staged per iteration
constexpr int LDK = BK + 4; // LDS row stride of a k-contiguous tile (floats)

__device__ __forceinline__ v16f mfma(float a, float b, v16f c)
{
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// A barrier that orders LDS accesses only: global loads and stores issued before it stay in flight across it
// (__syncthreads() would wait for all of them first).  The wait is written with the builtin so that the compiler's own
// counting knows that every LDS operation of the wave has completed here (behind an inline-asm barrier it waits for all of
// them again); the fences keep it from moving LDS accesses across, which the two builtins alone do not forbid.
__device__ __forceinline__ void sync_lds()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ v4f ld4(const float *p) { return *reinterpret_cast<const v4f *>(p); }
// Four input elements as they lie in memory, and their conversion: a staging register holds the raw form,
// so that nothing waits for a load before the tile of the stage before has been multiplied
__device__ __forceinline__ v4f ld4raw(const float *p) { return *reinterpret_cast<const v4f *>(p); }
__device__ __forceinline__ uint32_t ld4raw(const uint8_t *p) { return *reinterpret_cast<const uint32_t *>(p); }
__device__ __forceinline__ v4f cvt4(v4f v) { return v; }
__device__ __forceinline__ v4f cvt4(uint32_t u)
{
    v4f r;
    r.x = (float)(u & 0xFFu);
    r.y = (float)((u >> 8) & 0xFFu);
    r.z = (float)((u >> 16) & 0xFFu);
    r.w = (float)(u >> 24);
    return r;
}
__device__ __forceinline__ v4f ld4(const uint8_t *p)
{
    uint32_t u = *reinterpret_cast<const uint32_t *>(p);
    v4f r;
    r.x = (float)(u & 0xFFu);
    r.y = (float)((u >> 8) & 0xFFu);
    r.z = (float)((u >> 16) & 0xFFu);
    r.w = (float)(u >> 24);
    return r;
}

// ---------------------------------------------------------------------------
// Forward geometries: row m = (sample, out_y, out_x); k = position inside the
// receptive field in the order the weights are stored.  row_off: elements from the input's start, at most
// 8192 rows of 3136 floats or 1024 samples of 35280 bytes, so 32 bits: a weight-gradient tile forms four of them
// per thread and stage, and signed divisions and 64-bit products cost as much as its matrix instructions.
// ---------------------------------------------------------------------------
struct GConv1 {  // 8x8 stride 4, uint8 CHW input, k = (c, p, q)
    using in_t = uint8_t;
    static constexpr int K = 256, N = 32, P = 400;
    static __device__ __forceinline__ uint32_t row_off(uint32_t m, uint32_t xs)
    {
        return m / 400 * xs + pos_off(m % 400);
    }
    static __device__ __forceinline__ uint32_t pos_off(uint32_t r) { return __umul24(__umul24(r, 205) >> 12, 4 * 84 - 20 * 4) + r * 4; }   // r / 20, r < 400
    static __device__ __forceinline__ int k_off(int k) { return (k >> 6) * 7056 + ((k >> 3) & 7) * 84 + (k & 7); }
};
struct GConv2 {  // 4x4 stride 2 over 20x20x32, k = (p, q, c)
    using in_t = float;
    static constexpr int K = 512, N = 64, P = 81;
    static __device__ __forceinline__ uint32_t row_off(uint32_t m, uint32_t xs)
    {
        return m / 81 * xs + pos_off(m % 81);
    }
    static __device__ __forceinline__ uint32_t pos_off(uint32_t r) { return __umul24(__umul24(r, 57) >> 9, (2 * 20 - 9 * 2) * 32) + r * 64; }   // r / 9, r < 81
    static __device__ __forceinline__ int k_off(int k) { return (k >> 7) * 640 + (k & 127); }
};
struct GConv3 {  // 3x3 stride 1 over 9x9x64, k = (p, q, c)
    using in_t = float;
    static constexpr int K = 576, N = 64, P = 49;
    static __device__ __forceinline__ uint32_t row_off(uint32_t m, uint32_t xs)
    {
        return m / 49 * xs + pos_off(m % 49);
    }
    static __device__ __forceinline__ uint32_t pos_off(uint32_t r) { return __umul24(__umul24(r, 37) >> 8, (9 - 7) * 64) + r * 64; }   // r / 7, r < 49
    static __device__ __forceinline__ int k_off(int k) { return (k / 192) * 576 + (k % 192); }
};
struct GFc1 {  // dense 3136 -> 512 on the flattened conv3 output
    using in_t = float;
    static constexpr int K = 3136, N = 512, P = 1;
    static __device__ __forceinline__ uint32_t row_off(uint32_t m, uint32_t xs) { return m * xs; }
    static __device__ __forceinline__ uint32_t pos_off(uint32_t) { return 0; }
    static __device__ __forceinline__ int k_off(int k) { return k; }
};

// One launch serves up to three independent (input, weights, output) row
// ranges: the online net on s, the online net on s' and the target net on s'.
struct FwdSeg {
    const void *x;      // input activations (uint8 for conv1, float otherwise)
    const float *w;     // [N][K]
    const float *bias;  // [N] or nullptr (raw partial sums, no activation)
    float *y;           // [M][N] (+ z*split_stride per reduction split)
    int M;              // rows
    int tile_begin;     // first blockIdx.x of this segment
    long xs;            // elements between consecutive samples of x
};
struct FwdArgs {
    FwdSeg seg[3];
    int nseg;
    int klen;           // reduction elements per blockIdx.z
    long split_stride;  // elements between the outputs of consecutive splits
    float scale;        // multiplies the accumulated sum (1/255 for conv1)
};

// KS > 1 cuts every staged reduction slab into KS slices of 32, one per group of waves: the
// workgroup then has KS times the threads, the same loads per thread and KS times the bytes in
// flight, and the reduction loop is KS times shorter.  The KS partial tiles are added through
// LDS at the end.  This is what the small-batch launches use: with few rows there are few
// tiles, and a long dependent chain of short stages per tile is pure latency.
template <int NWT, int KS>
__device__ __forceinline__ void reduce_slices(v16f &acc, float *red /*LDS, (KS-1)*NWT*1024 floats*/, int ks,
                                              int w2, int lane)
{
    if constexpr (KS > 1) {
        __syncthreads();  // every wave is done reading the staged tiles
        if (ks > 0) {
            float *dst = red + ((ks - 1) * NWT + w2) * 1024;
#pragma unroll
            for (int r = 0; r < 16; ++r) dst[r * 64 + lane] = acc[r];
        }
        __syncthreads();
        if (ks == 0) {
#pragma unroll
            for (int s = 0; s < KS - 1; ++s) {
                const float *src = red + (s * NWT + w2) * 1024;
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[r] += src[r * 64 + lane];
            }
        }
    }
}

template <class G, int BM, int BN, int KS = 1>
__global__ __launch_bounds__((BM / 32) * (BN / 32) * KS * 64) void k_fwd(FwdArgs A)
{
    constexpr int NWT = (BM / 32) * (BN / 32), T = NWT * KS * 64;
    constexpr int BKS = BK * KS, LD = BKS + 4, CPR = BKS / 4, RPP = T / CPR;
    constexpr int NA = BM * CPR / T, NB = BN * CPR / T;
    static_assert(NA * T == BM * CPR && NB * T == BN * CPR && G::K % BKS == 0, "tile/threads mismatch");
    static_assert((BM + BN) * LD >= (KS - 1) * NWT * 1024, "reduction scratch does not fit the tiles");
    // Without slices: two buffers and one barrier per stage, the loads two stages ahead (see wgrad_tile)
    constexpr int NBUF = KS == 1 ? 2 : 1, STAGE = (BM + BN) * LD;
    using in_t = typename G::in_t;
    __shared__ __attribute__((aligned(16))) float smem[NBUF * (BM + BN) * LD];
    float *As = smem, *Bs = smem + BM * LD;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // tile order: column tiles of one row tile together, reduction splits apart
    const int t = net::tile_of_workgroup();
    const int by = t % (int)gridDim.y, bx = (t / (int)gridDim.y) % (int)gridDim.x, bz = t / (int)(gridDim.y * gridDim.x);
    FwdSeg S = A.seg[0];
    if (A.nseg > 1 && bx >= A.seg[1].tile_begin) S = A.seg[1];
    if (A.nseg > 2 && bx >= A.seg[2].tile_begin) S = A.seg[2];
    const int m0 = (bx - S.tile_begin) * BM, n0 = by * BN;
    const int kbeg = bz * A.klen, kend = kbeg + A.klen;
    const in_t *x = static_cast<const in_t *>(S.x);

    const int lr = tid / CPR, kq = (tid % CPR) * 4;
    long aoff[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int m = m0 + lr + i * RPP;
        aoff[i] = G::row_off(m < S.M ? m : S.M - 1, S.xs);   // (rows past the last one are not stored)
    }
    v4f ra[NA], rb[NB];
    auto gload = [&](int k0) {
        const int ko = G::k_off(k0 + kq);
#pragma unroll
        for (int i = 0; i < NA; ++i) ra[i] = ld4(x + aoff[i] + ko);
#pragma unroll
        for (int i = 0; i < NB; ++i)
            rb[i] = ld4(S.w + (long)(n0 + lr + i * RPP) * G::K + k0 + kq);
    };
    auto sstore = [&](int at) {
#pragma unroll
        for (int i = 0; i < NA; ++i) *reinterpret_cast<v4f *>(&As[at + (lr + i * RPP) * LD + kq]) = ra[i];
#pragma unroll
        for (int i = 0; i < NB; ++i) *reinterpret_cast<v4f *>(&Bs[at + (lr + i * RPP) * LD + kq]) = rb[i];
    };

    const int ks = wave / NWT, w2 = wave % NWT;
    const int wm = w2 % (BM / 32), wn = w2 / (BM / 32);
    const int li = lane & 31, h = lane >> 5;
    const float *ap = &As[(wm * 32 + li) * LD + ks * BK + 4 * h];
    const float *bp = &Bs[(wn * 32 + li) * LD + ks * BK + 4 * h];
    v16f acc = {0};
    const int col = n0 + wn * 32 + li;
    const float bias = S.bias ? S.bias[col] : 0.f;   // requested here, used in the epilogue

    auto compute = [&](int at) {
#pragma unroll
        for (int kk = 0; kk < BK; kk += 8) {
            v4f a = ld4(ap + at + kk), b = ld4(bp + at + kk);
            acc = mfma(a.x, b.x, acc);
            acc = mfma(a.y, b.y, acc);
            acc = mfma(a.z, b.z, acc);
            acc = mfma(a.w, b.w, acc);
        }
    };
    gload(kbeg);
    sstore(0);
    if constexpr (NBUF == 2) {
        if (kbeg + BKS < kend) gload(kbeg + BKS);
        sync_lds();
        int at = 0;
        for (int k0 = kbeg; k0 < kend; k0 += BKS) {
            if (k0 + BKS < kend) {
                sstore(STAGE - at);
                if (k0 + 2 * BKS < kend) gload(k0 + 2 * BKS);
            }
            compute(at);
            sync_lds();
            at = STAGE - at;
        }
    } else {
        __syncthreads();
        for (int k0 = kbeg; k0 < kend; k0 += BKS) {
            const bool more = k0 + BKS < kend;
            if (more) gload(k0 + BKS);
            compute(0);
            __syncthreads();
            if (more) {
                sstore(0);
                __syncthreads();
            }
        }
    }
    reduce_slices<NWT, KS>(acc, smem, ks, w2, lane);
    if (ks != 0) return;

    // all values first, then the stores: a wait for the bias inside the bounds-checked branches would be
    // repeated in every branch, and since stores count as outstanding memory operations too, each store
    // would then wait for the one before it to be acknowledged
    float *y = S.y + (long)bz * A.split_stride;
    float v[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        v[r] = acc[r] * A.scale;
        if (S.bias) v[r] = fmaxf(v[r] + bias, 0.f);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        int m = m0 + wm * 32 + 8 * (r / 4) + 4 * h + (r % 4);
        if (m < S.M) y[(long)m * G::N + col] = v[r];
    }
}

// ---------------------------------------------------------------------------
// Input gradient.  For a stride-S convolution the input pixels fall into S*S
// parity classes (h mod S, w mod S); a pixel of class (a,b) only meets the
// kernel taps p = a + S*u, q = b + S*v, so each class is its own dense GEMM
// over (KH/S)*(KW/S) taps with no multiplications by structural zeros:
//   dX[n][S*h'+a][S*w'+b][c] = sum_{u,v,o} dY[n][h'-u][w'-v][o] * W[o][a+S*u][b+S*v][c]
// (out-of-range dY positions contribute 0).  The result is multiplied by the
// ReLU mask of the layer below (its stored output > 0).
// ---------------------------------------------------------------------------
template <int S_, int TH_, int TW_, int OH_, int OW_, int HP_, int WP_, int CO_, int CI_, int KH_,
          int KW_, int H_, int W_>
struct DGeom {
    static constexpr int S = S_, TH = TH_, TW = TW_, OH = OH_, OW = OW_, HP = HP_, WP = WP_,
                         CO = CO_, CI = CI_, KH = KH_, KW = KW_, H = H_, W = W_;
    static constexpr int K = TH * TW * CO;  // reduction length per class
    static constexpr int PP = HP * WP;      // rows per sample per class
};
using DConv2 = DGeom<2, 2, 2, 9, 9, 10, 10, 64, 32, 4, 4, 20, 20>;
using DConv3 = DGeom<1, 3, 3, 7, 7, 9, 9, 64, 64, 3, 3, 9, 9>;
using DFc1 = DGeom<1, 1, 1, 1, 1, 1, 1, 512, 3136, 1, 1, 1, 1>;

struct DgradArgs {
    const float *dy;    // [B][OH][OW][CO] gradient w.r.t. this layer's pre-activation
    const float *w;     // [CO][KH][KW][CI]
    const float *xact;  // [B][H][W][CI] this layer's input (ReLU output of the layer below)
    float *dx;          // [B][H][W][CI] gradient w.r.t. the pre-activation of the layer below
    int B;
};

// LDS floats of an input-gradient tile
template <int BM, int BN, int KS> constexpr int dgrad_lds() { return (KS == 1 ? 2 : 1) * (BM * (BK * KS + 4) + BK * KS * (BN + 4)); }

// Tile number t of a grid of (gx, gy, gz) tiles, computed by the first (BM/32)(BN/32) KS waves of
// the workgroup (a launch may hold wider workgroups: the waves beyond leave at once; a barrier
// counts only the waves that are still there).  Tile order: the parity classes of one row tile
// together, then the row tiles of one column tile.
// The whole reduction is requested before the first stage is staged where it is at most four stages long
// (every layer at the tile shapes of the small-batch step): the tile is then one round trip to memory, not
// one per stage; so are the stored activations the epilogue masks with (the ReLU of the layer below).
// KA > 1: the KA slices of the reduction as sums of the same waves, in the order KS = KA waves would have them: the same
// bits from a tile of KA times the rows, for many rows.
template <class D, int BM, int BN, int KS, int KA = 1>
__device__ __forceinline__ void dgrad_tile(const DgradArgs &A, int t, int gx, int gz, float *smem)
{
    constexpr int NWT = (BM / 32) * (BN / 32), T = NWT * KS * 64;
    constexpr int BKS = BK * KS, LD = BKS + 4, CPR = BKS / 4, RPP = T / CPR;
    constexpr int NA = BM * CPR / T;
    constexpr int LDB = BN + 4;            // LDS row stride of the [k][c] weight tile
    constexpr int BROWS = T / (BN / 4);    // weight-tile rows filled per pass
    constexpr int NBL = BKS / BROWS;
    static_assert(NA * T == BM * CPR && NBL * BROWS == BKS && D::K % BKS == 0 && D::CO % 4 == 0, "tile/threads mismatch");
    static_assert(BM * LD + BKS * LDB >= (KS - 1) * NWT * 1024, "reduction scratch does not fit the tiles");
    if ((int)threadIdx.x >= T) return;
    float *As = smem, *Bs = smem + BM * LD;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int bz = t % gz, bx = (t / gz) % gx, by = t / (gz * gx);
    const int m0 = bx * BM, n0 = by * BN;
    const int ca = bz / D::S, cb = bz % D::S;
    const int Mc = A.B * D::PP;

    const int lr = tid / CPR, kq = (tid % CPR) * 4;
    int rn[NA], rh[NA], rw[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        int m = m0 + lr + i * RPP;
        if (m < Mc) {
            rn[i] = m / D::PP;
            int r = m % D::PP;
            rh[i] = r / D::WP;
            rw[i] = r % D::WP;
        } else {
            rn[i] = -1; rh[i] = 0; rw[i] = 0;
        }
    }
    const int br = tid / (BN / 4), bc = (tid % (BN / 4)) * 4;
    constexpr int NST = D::K / BKS;             // reduction stages
    constexpr bool ALLPRE = NST <= 4;           // all of them in flight at once
    static_assert(KA == 1 || (KS == 1 && !ALLPRE && NST % KA == 0), "slices");
    constexpr int NREG = ALLPRE ? NST : 1;
    v4f ra[NREG][NA], rb[NREG][NBL];
    auto gload = [&](int k0, v4f (&qa)[NA], v4f (&qb)[NBL]) {
        {   // a staged slab may span several kernel taps: each thread derives the tap of its chunk
            const int k = k0 + kq, tap = k / D::CO, o = k % D::CO;
            const int u = tap / D::TW, v = tap % D::TW;
#pragma unroll
            for (int i = 0; i < NA; ++i) {
                int ii = rh[i] - u, jj = rw[i] - v;
                bool ok = rn[i] >= 0 && ii >= 0 && ii < D::OH && jj >= 0 && jj < D::OW;
                qa[i] = ok ? ld4(A.dy + ((long)(rn[i] * D::OH + ii) * D::OW + jj) * D::CO + o)
                           : v4f{0, 0, 0, 0};
            }
        }
#pragma unroll
        for (int i = 0; i < NBL; ++i) {
            const int k = k0 + br + i * BROWS, tap = k / D::CO, o = k % D::CO;
            const int p = ca + D::S * (tap / D::TW), q = cb + D::S * (tap % D::TW);
            qb[i] = ld4(A.w + ((long)(o * D::KH + p) * D::KW + q) * D::CI + n0 + bc);
        }
    };
    auto sstore = [&](const v4f (&qa)[NA], const v4f (&qb)[NBL], int at = 0) {
#pragma unroll
        for (int i = 0; i < NA; ++i) *reinterpret_cast<v4f *>(&As[at + (lr + i * RPP) * LD + kq]) = qa[i];
#pragma unroll
        for (int i = 0; i < NBL; ++i) *reinterpret_cast<v4f *>(&Bs[at + (br + i * BROWS) * LDB + bc]) = qb[i];
    };

    const int ks = wave / NWT, w2 = wave % NWT;
    const int wm = w2 % (BM / 32), wn = w2 / (BM / 32);
    const int li = lane & 31, h = lane >> 5;
    const float *ap = &As[(wm * 32 + li) * LD + ks * BK + 4 * h];
    const float *bp = &Bs[(ks * BK + 4 * h) * LDB + wn * 32 + li];
    v16f acc_s[KA];
#pragma unroll
    for (int i = 0; i < KA; ++i) acc_s[i] = v16f{0};
    v16f &acc = acc_s[0];
    auto compute = [&](v16f &acc, int at = 0) {
#pragma unroll
        for (int kk = 0; kk < BK; kk += 8) {
            v4f a = ld4(ap + at + kk);
            acc = mfma(a.x, bp[at + (kk + 0) * LDB], acc);
            acc = mfma(a.y, bp[at + (kk + 1) * LDB], acc);
            acc = mfma(a.z, bp[at + (kk + 2) * LDB], acc);
            acc = mfma(a.w, bp[at + (kk + 3) * LDB], acc);
        }
    };
    // where this lane's results go (-1: no such row), and the stored activations there
    const int col = n0 + wn * 32 + li;
    int off[16];
    float xm[16];
    // (the loads are unconditional, from a clamped address: a value chosen between a loaded one and a
    // constant would make the compiler wait for the load right here)
    auto epilogue_loads = [&]() {
        if (__builtin_amdgcn_readfirstlane(ks) != 0) return;   // only the waves of slice 0 write the tile
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int mg = m0 + wm * 32 + 8 * g + 4 * h;
            int n = mg / D::PP, rr = mg % D::PP;
            int ph = rr / D::WP, pw = rr % D::WP;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int r = 4 * g + j;
                const int o = ((n * D::H + D::S * ph + ca) * D::W + D::S * pw + cb) * D::CI + col;
                const bool valid = mg + j < Mc;
                off[r] = valid ? o : -1;
                xm[r] = A.xact[valid ? o : 0];
                if (++pw == D::WP) {
                    pw = 0;
                    if (++ph == D::HP) { ph = 0; ++n; }
                }
            }
        }
    };

    if constexpr (ALLPRE) {
#pragma unroll
        for (int st = 0; st < NST; ++st) gload(st * BKS, ra[st], rb[st]);
        epilogue_loads();
#pragma unroll
        for (int st = 0; st < NST; ++st) {
            if (st) __syncthreads();   // every wave has read the stage before
            sstore(ra[st], rb[st]);
            __syncthreads();
            compute(acc);
        }
    } else if constexpr (KS == 1) {   // two buffers: see wgrad_tile
        constexpr int STAGE = BM * LD + BKS * LDB;
        gload(0, ra[0], rb[0]);
        sstore(ra[0], rb[0]);
        gload(BKS, ra[0], rb[0]);
        epilogue_loads();
        sync_lds();
        int at = 0;
        for (int ka = 0; ka < D::K; ka += KA * BKS)
#pragma unroll
            for (int i = 0; i < KA; ++i) {   // stage i of KA: slice i
                const int k0 = ka + i * BKS;
                if (k0 + BKS < D::K) {
                    sstore(ra[0], rb[0], STAGE - at);
                    if (k0 + 2 * BKS < D::K) gload(k0 + 2 * BKS, ra[0], rb[0]);
                }
                compute(acc_s[i], at);
                sync_lds();
                at = STAGE - at;
            }
#pragma unroll
        for (int i = 1; i < KA; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] += acc_s[i][r];
    } else {
        gload(0, ra[0], rb[0]);
        epilogue_loads();
        sstore(ra[0], rb[0]);
        __syncthreads();
        for (int k0 = 0; k0 < D::K; k0 += BKS) {
            const bool more = k0 + BKS < D::K;
            if (more) gload(k0 + BKS, ra[0], rb[0]);
            compute(acc);
            __syncthreads();
            if (more) {
                sstore(ra[0], rb[0]);
                __syncthreads();
            }
        }
    }
    reduce_slices<NWT, KS>(acc, smem, ks, w2, lane);
    if (ks != 0) return;

#pragma unroll
    for (int r = 0; r < 16; ++r)
        if (off[r] >= 0) A.dx[off[r]] = xm[r] > 0.f ? acc[r] : 0.f;
}
// conv2's input gradient for many rows: the four parity classes read the same dY (class (a, b) at pixel (2h' + a, 2w' + b) the
// positions h' - u, w' - v), so a tile is 64 of the 10 x 10 grids' rows by all classes' 32 channels, a wave per class, and dY is
// staged once for the four.
// Bound by the fp32 matrix pipe and by the vector instructions beside which it stands still (less than half of dgrad_tile's per
// product).  Two buffers and items behind matrix instructions as in wgrad_deep, the next stage but one in registers (one more
// took 187 of them, two workgroups per compute unit).  The reduction is in the order of dgrad_tile's four slices, 32 each of two
// taps, then the sums: the same bits.
// At a batch of 1000, alone, 111 us in dgrad_tile's 64 x 32 with the slices as waves, now 76; the step 880 -> 850, at 600 579 -> 568,
// at 449 465 -> 447.
constexpr int DG2_BM = 64, DG2_LDB = 128 + 4, DG2_STAGE = DG2_BM * LDK + BK * DG2_LDB;
__device__ const float dg2_zeros[64] = {};   // dY outside the image
__global__ __launch_bounds__(256, 3) void k_conv2_dgrad(DgradArgs A)
{
    using D = DConv2;
    typedef __attribute__((address_space(1))) const float *Global;   // (a choice between two arrays would become a flat pointer)
    __shared__ __attribute__((aligned(16))) float smem[2 * DG2_STAGE];
    float *As = smem, *Bs = smem + DG2_BM * LDK;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), li = lane & 31, h = lane >> 5;
    const int m0 = net::tile_of_workgroup() * DG2_BM, M = A.B * D::PP;
    // this thread's pieces of a stage: rows ar and ar + 32 of dY, 16 bytes of each; rows br, br + 8, .. of the weights, 16 bytes of a class
    const int ar = tid >> 3, ap = (tid & 7) * 4, br = tid >> 5, bc = tid & 31;
    const int bcls = bc >> 3;
    int arow[2];
    uint32_t taps[2];   // bit tap: inside the image
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int m = min(m0 + ar + 32 * i, M - 1), n = m / D::PP, r = m % D::PP, ph = r / D::WP, pw = r % D::WP;
        taps[i] = 0;
#pragma unroll
        for (int t = 0; t < 4; ++t) taps[i] |= (uint32_t)((uint32_t)(ph - t / 2) < (uint32_t)D::OH && (uint32_t)(pw - t % 2) < (uint32_t)D::OW) << t;
        arow[i] = ((n * D::OH + ph) * D::OW + pw) * D::CO + ap;
    }
    const float *wp = A.w + ((br * D::KH + bcls / 2) * D::KW + bcls % 2) * D::CI + (bc & 7) * 4;
    struct Regs { v4f a[2], b[4]; } R;
    // stage i of eight: 32 of slice i / 2, from tap i / 4 (i even) or 2 + i / 4 (i odd)
    auto tap_of = [](int i) { return 2 * (i & 1) + i / 4; };
    auto o_of = [](int i) { return 32 * (i / 2 % 2); };
    constexpr int NP = 6;
    auto request = [&](Regs &q, int i, int j) {
        const int tap = tap_of(i), o = o_of(i), u = tap / 2, v = tap % 2;
        if (j < 2) {
            const Global p = (Global)A.dy + (arow[j & 1] - (u * D::OW + v) * D::CO + o), z = (Global)dg2_zeros + ap;
            q.a[j & 1] = *reinterpret_cast<__attribute__((address_space(1))) const v4f *>(taps[j & 1] >> tap & 1 ? p : z);
        } else q.b[(j - 2) & 3] = ld4(wp + ((o + 8 * (j - 2)) * D::KH * D::KW + 2 * u * D::KW + 2 * v) * D::CI);
    };
    auto put = [&](const Regs &q, int at, int j) {
        if (j < 2) *reinterpret_cast<v4f *>(&As[at + (ar + 32 * j) * LDK + ap]) = q.a[j & 1];
        else *reinterpret_cast<v4f *>(&Bs[at + (br + 8 * (j - 2)) * DG2_LDB + bc * 4]) = q.b[(j - 2) & 3];
    };
    // operands of half a stage: eight of the reduction twice
    struct Ops { v4f a[2][2]; float b[8]; } O[2];
    const float *ap0 = As + li * LDK + 4 * h, *bp0 = Bs + 4 * h * DG2_LDB + 32 * wave + li;
    auto get = [&](Ops &o, int at, int half, int j) {   // j: 0-3 dY, 4-11 weights
        if (j < 4) o.a[j >> 1 & 1][j & 1] = ld4(ap0 + at + 32 * (j >> 1) * LDK + 16 * half + 8 * (j & 1));
        else o.b[(j - 4) & 7] = bp0[at + (16 * half + 8 * ((j - 4) >> 2) + (j & 3)) * DG2_LDB];
    };
    v16f acc[2], sum[2];
    auto multiply = [&](const Ops &o, auto item) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < 8; ++t)
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                acc[r] = mfma(o.a[r][t >> 2][t & 3], o.b[t], acc[r]);
                item(2 * t + r);
                __builtin_amdgcn_sched_barrier(0);
            }
    };
    auto all = [&](auto item) {
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            item(j);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    all([&](int j) { request(R, 0, j); });
    all([&](int j) { put(R, 0, j); });
    all([&](int j) { request(R, 1, j); });
    sync_lds();
#pragma unroll
    for (int j = 0; j < 12; ++j) get(O[0], 0, 0, j);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int at = i & 1 ? DG2_STAGE : 0;
        if (i % 2 == 0) acc[0] = acc[1] = v16f{0};
        multiply(O[0], [&](int k) {
            if (k < 12) get(O[1], at, 1, k);
            if (i + 1 < 8 && k < NP) put(R, DG2_STAGE - at, k);
            if (i + 2 < 8 && k >= NP && k < 2 * NP) request(R, i + 2, k - NP);
        });
        if (i + 1 < 8) sync_lds();
        multiply(O[1], [&](int k) {
            if (i + 1 < 8 && k < 12) get(O[0], DG2_STAGE - at, 0, k);
        });
        if (i % 2 == 1)
#pragma unroll
            for (int r = 0; r < 2; ++r) sum[r] = i == 1 ? acc[r] : sum[r] + acc[r];
    }
    const int ca = wave >> 1, cb = wave & 1;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        int off[16];
        float xm[16];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int mg = m0 + 32 * r + 8 * g + 4 * h;
            int n = mg / D::PP, rr = mg % D::PP, ph = rr / D::WP, pw = rr % D::WP;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int o = ((n * D::H + 2 * ph + ca) * D::W + 2 * pw + cb) * D::CI + li;
                const bool valid = mg + j < M;
                off[4 * g + j] = valid ? o : -1;
                xm[4 * g + j] = A.xact[valid ? o : 0];
                if (++pw == D::WP) {
                    pw = 0;
                    if (++ph == D::HP) { ph = 0; ++n; }
                }
            }
        }
#pragma unroll
        for (int k = 0; k < 16; ++k)
            if (off[k] >= 0) A.dx[off[k]] = xm[k] > 0.f ? sum[r][k] : 0.f;
    }
}

// conv3's and fc1's input gradients for many rows: the sums and bits of dgrad_tile in tiles of 64 x 64, in the manner of
// k_conv2_dgrad, two stages (conv3: a tap) per turn of the loop.  At a batch of 1000, alone, conv3's
// 69 -> 56 us (the step 852 -> 843, at 480 480 -> 472, at 930 807 -> 793, at 650 597 -> 603), then fc1's 49 -> 39 from tiles of 32 x 64
// (844 -> 835, at 480 471 -> 462, at 650 605 -> 596, at 700 652 either way).  In the launches with the weight gradients too, a step
// of 129 200 -> 193, of 200 243 -> 234, of 256 300 -> 289, of 419 435 -> 416.
constexpr int DG3_LDB = 64 + 4, DG3_STAGE = 64 * LDK + BK * DG3_LDB;
static_assert(dgrad_lds<64, 64, 1>() == 2 * DG3_STAGE, "LDS");
template <class D>   // tile of gx row tiles by the column tiles, 256 threads
__device__ __forceinline__ void dgrad_deep(const DgradArgs &A, int tile, int gx, float *smem)
{
    constexpr int TAPS = D::TH * D::TW, TURNS = D::K / 64, WROW = D::KH * D::KW * D::CI;
    static_assert(D::S == 1 && D::H == D::HP && D::W == D::WP && D::CO % 64 == 0 && D::CI % 64 == 0, "shape");
    typedef __attribute__((address_space(1))) const float *Global;
    float *As = smem, *Bs = smem + 64 * LDK;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), li = lane & 31, h = lane >> 5;
    const int wm = wave & 1, wn = wave >> 1, m0 = tile % gx * 64, n0 = tile / gx * 64, M = A.B * D::PP;
    // this thread's pieces of a stage: rows ar and ar + 32 of dY, 16 bytes of each; rows br and br + 16 of the weights, 16 bytes
    const int ar = tid >> 3, ap = (tid & 7) * 4, br = tid >> 4, bc = (tid & 15) * 4;
    int arow[2];
    uint32_t taps[2];   // bit tap: inside the image
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int m = min(m0 + ar + 32 * i, M - 1), n = m / D::PP, r = m % D::PP, ph = r / D::WP, pw = r % D::WP;
        taps[i] = 0;
#pragma unroll
        for (int t = 0; t < TAPS; ++t) taps[i] |= (uint32_t)((uint32_t)(ph - t / D::TW) < (uint32_t)D::OH && (uint32_t)(pw - t % D::TW) < (uint32_t)D::OW) << t;
        arow[i] = ((n * D::OH + ph) * D::OW + pw) * D::CO + ap;
    }
    const float *wp = A.w + br * WROW + n0 + bc;
    struct Regs { v4f a[2], b[2]; } R;
    constexpr int NP = 4;
    auto request = [&](int turn, int half, int j) {
        const int tap = turn * 64 / D::CO, o = turn * 64 % D::CO + half;
        if (j < 2) {
            const Global p = (Global)A.dy + (arow[j & 1] + (o - (tap / D::TW * D::OW + tap % D::TW) * D::CO)), z = (Global)dg2_zeros + ap;
            R.a[j & 1] = *reinterpret_cast<__attribute__((address_space(1))) const v4f *>(TAPS == 1 || taps[j & 1] >> tap & 1 ? p : z);
        } else R.b[j & 1] = ld4(wp + ((o + 16 * (j & 1)) * WROW + tap * D::CI));
    };
    auto put = [&](int at, int j) {
        if (j < 2) *reinterpret_cast<v4f *>(&As[at + (ar + 32 * j) * LDK + ap]) = R.a[j & 1];
        else *reinterpret_cast<v4f *>(&Bs[at + (br + 16 * (j & 1)) * DG3_LDB + bc]) = R.b[j & 1];
    };
    struct Ops { v4f a[2]; float b[8]; } O[2];   // of half a stage
    const float *ap0 = As + (32 * wm + li) * LDK + 4 * h, *bp0 = Bs + 4 * h * DG3_LDB + 32 * wn + li;
    auto get = [&](Ops &o, int at, int half, int j) {   // j: 0-7 weights, and with 0 and 4 dY
        if (j % 4 == 0) o.a[j / 4] = ld4(ap0 + at + 16 * half + 2 * j);
        o.b[j] = bp0[at + (16 * half + 8 * (j / 4) + j % 4) * DG3_LDB];
    };
    v16f acc = {0};
    auto multiply = [&](const Ops &o, auto item) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            acc = mfma(o.a[t / 4][t % 4], o.b[t], acc);
            item(t);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto stage = [&](int at, int turn, int o) {   // (turn, o): of the stage after the next
        multiply(O[0], [&](int k) {
            get(O[1], at, 1, k);
            if (k < NP) put(DG3_STAGE - at, k);
            else request(turn, o, k - NP);
        });
        sync_lds();
        multiply(O[1], [&](int k) { get(O[0], DG3_STAGE - at, 0, k); });
    };
#pragma unroll
    for (int j = 0; j < NP; ++j) request(0, 0, j);
#pragma unroll
    for (int j = 0; j < NP; ++j) put(0, j);
#pragma unroll
    for (int j = 0; j < NP; ++j) request(0, 32, j);
    sync_lds();
#pragma unroll
    for (int j = 0; j < 8; ++j) get(O[0], 0, 0, j);
    for (int turn = 0; turn < TURNS; ++turn) {   // (behind the last turn: its own again, which nobody multiplies)
        const int next = min(turn + 1, TURNS - 1);
        stage(0, next, 0);
        stage(DG3_STAGE, next, 32);
    }
    int off[16];
    float xm[16];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int m = m0 + 32 * wm + 8 * g + 4 * h + j;   // (a row of the result is a pixel of the input)
            off[4 * g + j] = m < M ? m * D::CI + n0 + 32 * wn + li : -1;
            xm[4 * g + j] = A.xact[m < M ? m * D::CI + n0 + 32 * wn + li : 0];
        }
    }
#pragma unroll
    for (int k = 0; k < 16; ++k)
        if (off[k] >= 0) A.dx[off[k]] = xm[k] > 0.f ? acc[k] : 0.f;
}

template <class D> __global__ __launch_bounds__(256, 4) void k_dgrad_deep(DgradArgs A)   // grid: row tiles x column tiles
{
    __shared__ __attribute__((aligned(16))) float smem[2 * DG3_STAGE];
    dgrad_deep<D>(A, net::tile_of_workgroup(), gridDim.x, smem);
}

// ---------------------------------------------------------------------------
// Weight gradient: dW[o][k] = sum_m dY[m][o] * A(m,k), db[o] = sum_m dY[m][o].
// The reduction runs over all output positions of all samples; it is cut into
// blockIdx.z splits of consecutive rows, each writing its own partial result
// ([W..., b...] per split), which the optimizer kernel adds up in a fixed order
// (no floating-point atomics, so results are reproducible).
// ---------------------------------------------------------------------------
struct WgradArgs {
    const float *dy;   // [B*P][N]
    const void *x;     // layer input (uint8 for conv1)
    float *part;       // [splits][N*K + N]
    int B;
    int rps;           // reduction rows (output positions) per split, a multiple of 32
    long xs;           // elements between consecutive samples of x
    long part_stride;  // elements between consecutive splits
    float scale;       // multiplies dW (1/255 for conv1)
};

// LDS of a weight-gradient tile, two buffers of both operands, in floats
template <int BMO, int BNK> constexpr int wgrad_lds() { return 2 * BK * (BMO + 4 + BNK + 4); }

// One weight-gradient tile: output channels [by*BMO, +BMO) x im2col columns [bx*BNK, +BNK) over the
// rows of split bz, computed by the first T threads of the workgroup; Ys/Xs are the workgroup's LDS.
template <class G, int BMO, int BNK>
__device__ __forceinline__ void wgrad_tile(const WgradArgs &A, int bx, int by, int bz, float *lds)
{
    constexpr int T = (BMO / 32) * (BNK / 32) * 64;
    constexpr int LDY = BMO + 4, LDX = BNK + 4;
    constexpr int YR = T / (BMO / 4), XR = T / (BNK / 4);  // tile rows filled per pass
    constexpr int NY = (BK + YR - 1) / YR, NX = (BK + XR - 1) / XR;
    using in_t = typename G::in_t;
    if ((int)threadIdx.x >= T) return;   // a wider workgroup: the waves beyond the tile's leave at once
    constexpr int STAGE = BK * (LDY + LDX);   // floats of a buffer
    float *Ys = lds, *Xs = lds + BK * LDY;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int kc0 = bx * BNK, o0 = by * BMO;
    const int mbeg = bz * A.rps;
    const int mend = min(mbeg + A.rps, A.B * G::P);
    const in_t *x = static_cast<const in_t *>(A.x);

    const int yr = tid / (BMO / 4), yc = (tid % (BMO / 4)) * 4;
    const int xr = tid / (BNK / 4), xc = (tid % (BNK / 4)) * 4;
    const int xko = G::k_off(kc0 + xc);
    using raw_t = decltype(ld4raw(x));
    v4f ry[NY];
    raw_t rx[NX];
    int left = 0;   // rows of the loaded stage that exist
    auto gload = [&](int mb) {
        left = mend - mb;
#pragma unroll
        for (int i = 0; i < NY; ++i) ry[i] = ld4(A.dy + (uint32_t)min(mb + yr + i * YR, mend - 1) * (uint32_t)G::N + (uint32_t)(o0 + yc));
#pragma unroll
        for (int i = 0; i < NX; ++i) rx[i] = ld4raw(x + (G::row_off((uint32_t)min(mb + xr + i * XR, mend - 1), (uint32_t)A.xs) + (uint32_t)xko));
    };
    // (rows past the end: dY as zeros is enough, the input there is that of the last row)
    auto sstore = [&](int at) {
#pragma unroll
        for (int i = 0; i < NY; ++i) {
            const int r = yr + i * YR;
            if (r < BK) *reinterpret_cast<v4f *>(&Ys[at + r * LDY + yc]) = r < left ? ry[i] : v4f{0, 0, 0, 0};
        }
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const int r = xr + i * XR;
            if (r < BK) *reinterpret_cast<v4f *>(&Xs[at + r * LDX + xc]) = cvt4(rx[i]);
        }
    };

    const int wo = wave % (BMO / 32), wk = wave / (BMO / 32);
    const int li = lane & 31, h = lane >> 5;
    const float *yp = &Ys[(4 * h) * LDY + wo * 32 + li];
    const float *xp = &Xs[(4 * h) * LDX + wk * 32 + li];
    const bool do_bias = bx == 0 && wk == 0;
    v16f acc = {0};
    // The bias gradient as vector additions in the order of the matrix instruction (k, then k + 4): against a column of
    // ones it doubled the matrix work of the waves that hold it, and a launch of one round lasts as long as they do
    // (conv1's at a batch of 1000: 118 -> 87 us, conv2's 129 -> 110, the step 1030 -> 976; at 256 336 -> 318)
    const float *yb = &Ys[wo * 32 + li];
    float bsum = 0.f;

    // Two buffers, one barrier per stage: while a stage is multiplied the next one is stored and the one after it is on its
    // way.  With one buffer and two barriers every stage was a round trip to memory.
    if (mbeg < mend) {
        gload(mbeg);
        sstore(0);
        if (mbeg + BK < mend) gload(mbeg + BK);
    }
    sync_lds();
    int at = 0;
    for (int mb = mbeg; mb < mend; mb += BK) {
        if (mb + BK < mend) {
            sstore(STAGE - at);
            if (mb + 2 * BK < mend) gload(mb + 2 * BK);
        }
#pragma unroll
        for (int kk = 0; kk < BK; kk += 8) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                float a = yp[at + (kk + t) * LDY], b = xp[at + (kk + t) * LDX];
                acc = mfma(a, b, acc);
            }
        }
        if (do_bias) {   // uniform for the wave; beside its matrix instructions, which are still running
#pragma unroll
            for (int kk = 0; kk < BK; kk += 8)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    bsum += yb[at + (kk + t) * LDY];
                    bsum += yb[at + (kk + 4 + t) * LDY];
                }
        }
        sync_lds();
        at = STAGE - at;
    }

    float *part = A.part + (long)bz * A.part_stride;
    const int col = kc0 + wk * 32 + li;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        int o = o0 + wo * 32 + 8 * (r / 4) + 4 * h + (r % 4);
        part[(long)o * G::K + col] = acc[r] * A.scale;
    }
    if (do_bias && h == 0) part[(long)G::N * G::K + o0 + wo * 32 + li] = bsum;
}

// The same tile for launches of their own with many stages per tile.  wgrad_tile's waves wait where a stage's operands are read
// in front of its matrix instructions, and a sixth of a SIMD's time are vector instructions, beside which it runs no fp32 matrix
// instructions: mostly the divisions in the rows' addresses, which are carried along here.  At a batch of 1000, alone, conv1's
// 87 -> 73 us, conv2's 74 -> 56, conv3's 52 -> 41, fc1's 52 -> 42, the step 898 -> 884; conv1's at 256 23.7 -> 22.0, at 100 equal, at 65
// 9.9 -> 10.2.  In the small-batch launches beside an input gradient its longer code and the registers cost 1 to 3 us per launch.
template <class G, int BMO, int BNK>
__device__ __forceinline__ void wgrad_deep(const WgradArgs &A, int bx, int by, int bz, float *lds)
{
    constexpr int T = (BMO / 32) * (BNK / 32) * 64;
    constexpr int LDY = BMO + 4, LDX = BNK + 4;
    constexpr int YR = T / (BMO / 4), XR = T / (BNK / 4);  // tile rows filled per pass
    constexpr int NY = (BK + YR - 1) / YR, NX = (BK + XR - 1) / XR;
    using in_t = typename G::in_t;
    if ((int)threadIdx.x >= T) return;   // a wider workgroup: the waves beyond the tile's leave at once
    constexpr int STAGE = BK * (LDY + LDX);   // floats of a buffer
    float *Ys = lds, *Xs = lds + BK * LDY;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kc0 = bx * BNK, o0 = by * BMO;
    const int mbeg = bz * A.rps;
    const int mend = min(mbeg + A.rps, A.B * G::P);
    const in_t *x = static_cast<const in_t *>(A.x);

    const int yr = tid / (BMO / 4), yc = (tid % (BMO / 4)) * 4;
    const int xr = tid / (BNK / 4), xc = (tid % (BNK / 4)) * 4;
    using raw_t = decltype(ld4raw(x));
    // where this thread's pieces of the next stage to be requested lie (further rows lie at higher offsets); a stage is 32 rows,
    // at most one sample further
    const uint32_t ymax = (uint32_t)(mend - 1) * G::N + o0 + yc, xlast = G::row_off(mend - 1, (uint32_t)A.xs) + G::k_off(kc0 + xc);
    uint32_t yo[NY], xs0[NX];
    int xp[NX];
#pragma unroll
    for (int i = 0; i < NY; ++i) yo[i] = (uint32_t)(mbeg + yr + i * YR) * G::N + o0 + yc;
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        const int m = mbeg + xr + i * XR;
        xp[i] = m % G::P;
        xs0[i] = m / G::P * (uint32_t)A.xs + G::k_off(kc0 + xc);
    }
    const int n = mbeg < mend ? (mend - mbeg + BK - 1) / BK : 0;
    struct Regs { v4f y[NY]; raw_t x[NX]; } R[2];
    auto request = [&](Regs &q, int j) {   // piece j; rows past the end: the last one
        if (j < NY) {
            q.y[j < NY ? j : 0] = ld4(A.dy + min(yo[j < NY ? j : 0], ymax));
            yo[j < NY ? j : 0] += BK * G::N;
        } else {
            const int i = j - NY;
            q.x[i] = ld4raw(x + min(xs0[i] + G::pos_off(xp[i]), xlast));
            if constexpr (G::P == 1) xs0[i] += BK * (uint32_t)A.xs;
            else {
                const bool over = (xp[i] += BK) >= G::P;
                xp[i] -= over ? G::P : 0;
                xs0[i] += over ? (uint32_t)A.xs : 0u;
            }
        }
    };
    // (rows past the end: dY as zeros is enough)
    auto put = [&](const Regs &q, int at, int left, int j) {
        if (j < NY) {
            const int r = yr + j * YR;
            v4f v = q.y[j < NY ? j : 0];
            if (left < BK) v = r < left ? v : v4f{0, 0, 0, 0};
            if (YR * NY == BK || r < BK) *reinterpret_cast<v4f *>(&Ys[at + r * LDY + yc]) = v;
        } else {
            const int r = xr + (j - NY) * XR;
            if (XR * NX == BK || r < BK) *reinterpret_cast<v4f *>(&Xs[at + r * LDX + xc]) = cvt4(q.x[j - NY]);
        }
    };

    const int wo = wave % (BMO / 32), wk = wave / (BMO / 32);
    const int li = lane & 31, h = lane >> 5;
    const float *yp = &Ys[(4 * h) * LDY + wo * 32 + li];
    const float *xp0 = &Xs[(4 * h) * LDX + wk * 32 + li];
    const bool do_bias = bx == 0 && wk == 0;
    v16f acc = {0};
    const float *yb = &Ys[wo * 32 + li];   // the bias gradient: see wgrad_tile
    float bsum = 0.f;

    // Two buffers, one barrier per stage.  A stage is requested three stages ahead and lies in registers until its buffer is
    // free; the operands of sixteen rows are read ahead of their matrix instructions, and the barrier stands between the
    // stage's halves, so that those behind it are read beside the second.  A load or LDS access in front of a matrix
    // instruction of the same wave holds it up, so they stand one or two at a time behind the matrix instructions.
    struct Ops { float a[8], b[8]; } O[2];
    auto get = [&](Ops &o, int at, int half, int j) {   // row 8 (j / 4) + j % 4 of the half, and the one four further
        const int k = 16 * half + 8 * (j / 4) + j % 4;
        o.a[j] = yp[at + k * LDY];
        o.b[j] = xp0[at + k * LDX];
    };
    constexpr int NP = NY + NX;
    auto multiply = [&](const Ops &o, auto item) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            acc = mfma(o.a[j], o.b[j], acc);
            item(j);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // stage s, in the buffer `at`; q: stage s + 1, then on its way s + 3
    // (inner: neither the last stages nor what they need)
    auto stage = [&](auto inner, int s, int at, Regs &q) {
        constexpr bool I = decltype(inner)::value;
        const int left = mend - mbeg - (s + 1) * BK;
        multiply(O[0], [&](int j) {
            get(O[1], at, 1, j);
            if (I || s + 1 < n) {
#pragma unroll
                for (int i = 0; i < NP; ++i)
                    if (i * 4 / NP == j) put(q, STAGE - at, I ? BK : left, i);
            }
            if (I || s + 3 < n) {
#pragma unroll
                for (int i = 0; i < NP; ++i)
                    if (4 + i * 4 / NP == j) request(q, i);
            }
        });
        if (do_bias) {   // uniform for the wave
#pragma unroll
            for (int kk = 0; kk < BK; kk += 8)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    bsum += yb[at + (kk + t) * LDY];
                    bsum += yb[at + (kk + 4 + t) * LDY];
                }
        }
        sync_lds();
        if (I || s + 1 < n) multiply(O[1], [&](int j) { get(O[0], STAGE - at, 0, j); });
        else multiply(O[1], [](int) {});
    };
    if (n > 0) {
        auto all = [&](auto item) {   // (in this order: ahead of the loop another one would make its waits longer)
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                item(i);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        all([&](int i) { request(R[0], i); });
        if (n > 1) all([&](int i) { request(R[1], i); });
        all([&](int i) { put(R[0], 0, mend - mbeg, i); });
        if (n > 2) all([&](int i) { request(R[0], i); });
        sync_lds();
#pragma unroll
        for (int j = 0; j < 8; ++j) get(O[0], 0, 0, j);
        int s = 0;
        for (; s + 5 <= n; s += 2) {
            stage(std::true_type{}, s, 0, R[1]);
            stage(std::true_type{}, s + 1, STAGE, R[0]);
        }
        for (; s < n; s += 2) {
            stage(std::false_type{}, s, 0, R[1]);
            if (s + 1 < n) stage(std::false_type{}, s + 1, STAGE, R[0]);
        }
    }

    float *part = A.part + (long)bz * A.part_stride;
    const int col = kc0 + wk * 32 + li;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        int o = o0 + wo * 32 + 8 * (r / 4) + 4 * h + (r % 4);
        part[(long)o * G::K + col] = acc[r] * A.scale;
    }
    if (do_bias && h == 0) part[(long)G::N * G::K + o0 + wo * 32 + li] = bsum;
}

// tile number -> (bx, by, bz) of a grid (gx, gy, gz): with row splits (conv layers) all tiles of one
// split together; without (fc1) all output tiles of one input-column tile together
__device__ __forceinline__ void wgrad_tile_of(int t, int gx, int gy, int gz, int &bx, int &by, int &bz)
{
    if (gz > 1) {
        bx = t % gx; by = (t / gx) % gy; bz = t / (gx * gy);
    } else {
        by = t % gy; bx = t / gy; bz = 0;
    }
}

// DEEP: with many stages per tile (wgrad_deep)
template <class G, int BMO, int BNK, bool DEEP>
__global__ __launch_bounds__((BMO / 32) * (BNK / 32) * 64) void k_wgrad(WgradArgs A)
{
    __shared__ __attribute__((aligned(16))) float lds[wgrad_lds<BMO, BNK>()];
    int bx, by, bz;
    wgrad_tile_of(net::tile_of_workgroup(), gridDim.x, gridDim.y, gridDim.z, bx, by, bz);
    if constexpr (DEEP) wgrad_deep<G, BMO, BNK>(A, bx, by, bz, lds);
    else wgrad_tile<G, BMO, BNK>(A, bx, by, bz, lds);
}

}  // namespace g32

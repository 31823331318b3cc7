// bf16 implicit-GEMM kernels on the CDNA4 matrix cores
// (v_mfma_f32_32x32x16_bf16: bf16 operands, fp32 accumulation).
//
// Same three kernel families and the same geometries as gemm_fp32.h; what
// differs is the staging:
//   * a reduction stage is 64 elements (128 bytes per row), moved as 16-byte
//     chunks; conv1 converts its uint8 pixels to bf16 while staging (integers
//     up to 255 are exact in bf16);
//   * an operand whose reduction index is the SLOW index in memory (weights in
//     the input-gradient kernel, both operands of the weight-gradient kernel)
//     is staged as it lies in memory, [reduction][column], and read with the
//     LDS transpose load (ds_read_b64_tr_b16), which hands each lane four
//     consecutive reduction elements of its column: within a group of 16 lanes,
//     lane s addresses row s/4, columns 4*(s%4)..+3 of a 4x16 block and lane d
//     receives column d of that block.
//
// MFMA 32x32x16 operand layout (lane = 32*h + i): a-operand A[i][8h..8h+7],
// b-operand B[8h..8h+7][i], result acc[r] = D[8*(r/4) + 4*h + r%4][i].
//
// Kernels whose output is channel-last ([position][channel]) feed the WEIGHT
// fragment as the a-operand and the activation fragment as the b-operand, i.e.
// they compute the transposed tile: a lane then owns one output position and 4
// groups of 4 consecutive channels, which it stores as 8-byte pieces (instead of
// sixteen 2-byte stores at a 64-byte row stride).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <iterator>
#include <vector>

#include "gemm_fp32.h"
#include "kernels_misc.h"
#include "packed.h"
#include "sumtree.h"

namespace gbf {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef short v4s __attribute__((ext_vector_type(4)));
typedef uint16_t bf16_t;  // storage type

constexpr int BK = 64;       // reduction elements per stage
constexpr int LDK = BK + 8;  // LDS row stride (elements) of a k-contiguous tile: 144 bytes

__device__ __forceinline__ v16f mfma(v8bf a, v8bf b, v16f c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// v_mfma_f32_16x16x32_bf16 (lane = 16*g + i): a-operand A[i][8g..8g+7], b-operand B[8g..8g+7][i],
// result acc[j] = D[4g + j][i]
__device__ __forceinline__ v4f mfma16(v8bf a, v8bf b, v4f c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ bf16_t f2bf(float f)  // round to nearest even
{
    return __builtin_bit_cast(bf16_t, (__bf16)f);
}
// four floats -> four bf16 in 8 bytes
__device__ __forceinline__ uint2 pack4(float a, float b, float c, float d)
{
    typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
    v2bf lo = {(__bf16)a, (__bf16)b}, hi = {(__bf16)c, (__bf16)d};
    return uint2{__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)};
}
__device__ __forceinline__ float bf2f(bf16_t b) { return __uint_as_float((uint32_t)b << 16); }

// 8 consecutive reduction elements as one 16-byte value
__device__ __forceinline__ uint4 ld8(const bf16_t *p) { return *reinterpret_cast<const uint4 *>(p); }
__device__ __forceinline__ uint32_t pack2_u8(uint32_t lo, uint32_t hi)
{
    return (__float_as_uint((float)lo) >> 16) | (__float_as_uint((float)hi) & 0xFFFF0000u);
}
// 8 pixels in two words -> 8 bf16 (exact): the upper halves of the floats, merged pairwise by a byte permute
__device__ __forceinline__ uint4 cvt8_u8(uint32_t a, uint32_t b)
{
    auto pk = [](float lo, float hi) { return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u); };
    uint4 o;
    o.x = pk((float)(a & 0xFFu), (float)((a >> 8) & 0xFFu));
    o.y = pk((float)((a >> 16) & 0xFFu), (float)(a >> 24));
    o.z = pk((float)(b & 0xFFu), (float)((b >> 8) & 0xFFu));
    o.w = pk((float)((b >> 16) & 0xFFu), (float)(b >> 24));
    return o;
}
__device__ __forceinline__ uint4 ld8(const uint8_t *p)  // 8 pixels -> 8 bf16 (exact)
{
    uint32_t a = *reinterpret_cast<const uint32_t *>(p), b = *reinterpret_cast<const uint32_t *>(p + 4);
    uint4 r;
    r.x = pack2_u8(a & 0xFFu, (a >> 8) & 0xFFu);
    r.y = pack2_u8((a >> 16) & 0xFFu, a >> 24);
    r.z = pack2_u8(b & 0xFFu, (b >> 8) & 0xFFu);
    r.w = pack2_u8((b >> 16) & 0xFFu, b >> 24);
    return r;
}

using g32::sync_lds;

__device__ __forceinline__ v8bf frag_k(const bf16_t *p)  // 8 consecutive k of one row
{
    return *reinterpret_cast<const v8bf *>(p);
}
// 8 consecutive reduction rows of one column out of a [reduction][column] tile.
// p points at (row0 + s/4, col_block + 4*(s%4)) for this lane; ld = row stride.
__device__ __forceinline__ v8bf frag_tr(const bf16_t *p, int ld)
{
    typedef __attribute__((address_space(3))) v4s *lds_v4s;
    v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(p));
    v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(p + 4 * ld));
    typedef short v8s __attribute__((ext_vector_type(8)));
    v8s r = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    return __builtin_bit_cast(v8bf, r);
}

// A [reduction][COLS] tile for frag_tr, without padding.  The hardware serves such a read half a wave at a time (measured):
// four consecutive rows of one block of 32 columns, 64 bytes each.  The blocks of a row are permuted by the row's number so
// that those four lie in all 64 banks side by side.  (Rows padded by 16 bytes instead: 1.6 times the cycles per read
// with 64 columns, 3 times with 128.)  Rows four apart are permuted alike.
template <int COLS> struct TrTile {
    static_assert(COLS == 64 || COLS == 128 || COLS == 192, "two, four or six blocks");
    static __device__ __forceinline__ int block(int row, int blk) { return blk ^ (COLS == 128 ? row & 3 : (row >> 1) & 1); }
    static __device__ __forceinline__ int at(int row, int col) { return row * COLS + block(row, col >> 5) * 32 + (col & 31); }
};

using g32::GConv1;
using g32::GConv2;
using g32::GConv3;
using g32::GFc1;

template <class G> struct in_type { using t = bf16_t; };
template <> struct in_type<GConv1> { using t = uint8_t; };

// ---------------------------------------------------------------------------
struct FwdSeg {
    const void *x;      // uint8 (conv1) or bf16 activations
    const bf16_t *w;    // [N][K] bf16 copy of the weights
    const float *bias;  // [N] fp32 (master copy) or nullptr
    void *y;            // fp32 raw partial sums [M][N]
    int M;
    int tile_begin;
    long xs;
};
struct FwdArgs {
    FwdSeg seg[3];
    int nseg;
    long split_stride;
};

// fc1 for few rows: raw fp32 partial sums of FC1_SPLITS reduction splits (the head kernels add them), 32 rows x BN
// columns per workgroup, one wave per 32 columns.  A split is seven stages of 64, and with few rows there is about
// one workgroup per CU, so nothing hides a stage's way from memory but the other stages: all seven are
// requested at once (140 registers) and the launch is one round trip, then seven short stages out of two LDS
// buffers.  With one stage in flight ahead of the one in work it was a chain of seven trips: 11.4 us at 231 rows.
constexpr int FC1_SPLITS = 7;
// The tile of rows m0 .. + 31 (S.M in all), columns n0 .. + BN - 1 and split bz by T threads, of which the first BN / 32 waves
// multiply; put(m, n, v): the sums of row m, columns n .. n + 3.  Dynamic or static LDS `lds`: fc1_few_lds<BN> elements.
template <int BN> constexpr int fc1_few_lds() { return 2 * (32 + BN) * LDK; }
template <int BN, int T, class Put>
__device__ __forceinline__ void fc1_few_tile(const FwdSeg &S, int m0, int n0, int bz, bf16_t *lds, Put put)
{
    constexpr int BM = 32, NST = GFc1::K / FC1_SPLITS / BK, NA = BM * 8 / T, NB = BN * 8 / T;
    static_assert(NST * FC1_SPLITS * BK == GFc1::K && NA * T == BM * 8 && NB * T == BN * 8, "tile/threads mismatch");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, k0 = bz * (NST * BK);
    const bf16_t *x = static_cast<const bf16_t *>(S.x);
    const int lr = tid >> 3, kq = (tid & 7) * 8;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // a native vector: stays in registers
    u32x4 ra[NST][NA], rb[NST][NB];
    const bf16_t *pa[NA], *pb[NB];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        int m = m0 + lr + i * (T / 8);
        if (m > S.M - 1) m = S.M - 1;             // rows past the end repeat the last row; they are never stored
        pa[i] = x + (long)m * S.xs + k0 + kq;
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) pb[i] = S.w + (long)(n0 + lr + i * (T / 8)) * GFc1::K + k0 + kq;
#pragma unroll
    for (int st = 0; st < NST; ++st) {
#pragma unroll
        for (int i = 0; i < NA; ++i) ra[st][i] = *reinterpret_cast<const u32x4 *>(pa[i] + st * BK);
#pragma unroll
        for (int i = 0; i < NB; ++i) rb[st][i] = *reinterpret_cast<const u32x4 *>(pb[i] + st * BK);
    }
    __builtin_amdgcn_sched_barrier(0);
    const int li = lane & 31, h = lane >> 5;
    v16f acc = {0};
#pragma unroll
    for (int st = 0; st < NST; ++st) {
        bf16_t *as = lds + (st & 1) * (BM * LDK), *bs = lds + 2 * BM * LDK + (st & 1) * (BN * LDK);
#pragma unroll
        for (int i = 0; i < NA; ++i) *reinterpret_cast<u32x4 *>(&as[(lr + i * (T / 8)) * LDK + kq]) = ra[st][i];
#pragma unroll
        for (int i = 0; i < NB; ++i) *reinterpret_cast<u32x4 *>(&bs[(lr + i * (T / 8)) * LDK + kq]) = rb[st][i];
        sync_lds();   // the buffer is complete; every wave is past the stage before, which read the other one
        if (T > 2 * BN && wave >= BN / 32) continue;
        v8bf fa[4], fb[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            fa[k] = frag_k(as + li * LDK + 8 * h + 16 * k);
            fb[k] = frag_k(bs + (wave * 32 + li) * LDK + 8 * h + 16 * k);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) acc = mfma(fb[k], fa[k], acc);   // transposed tile
    }
    // acc[4g + j] = Y[row m = lane li][channel = 8g + 4h + j]
    const int m = m0 + li;
    if (m >= S.M || (T > 2 * BN && wave >= BN / 32)) return;
#pragma unroll
    for (int g = 0; g < 4; ++g) put(m, n0 + wave * 32 + 4 * h + 8 * g, v4f{acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]});
}
template <int BN>
__global__ __launch_bounds__(2 * BN) void k_fc1_fwd_few(FwdArgs A)
{
    __shared__ __attribute__((aligned(16))) bf16_t lds[fc1_few_lds<BN>()];
    // tile order: column tiles of one row tile together, reduction splits apart
    const int t = net::tile_of_workgroup();
    const int by = t % (int)gridDim.y, bx = (t / (int)gridDim.y) % (int)gridDim.x, bz = t / (int)(gridDim.y * gridDim.x);
    FwdSeg S = A.seg[0];
    if (A.nseg > 1 && bx >= A.seg[1].tile_begin) S = A.seg[1];
    if (A.nseg > 2 && bx >= A.seg[2].tile_begin) S = A.seg[2];
    float *y = static_cast<float *>(S.y) + (long)bz * A.split_stride;
    fc1_few_tile<BN, 2 * BN>(S, (bx - S.tile_begin) * 32, by * BN, bz, lds,
                             [&](int m, int n, v4f v) { *reinterpret_cast<v4f *>(y + (long)m * GFc1::N + n) = v; });
}

// bf16 acting on up to misc::FEW_ROWS observations: fc1 and the head in one launch (see misc::k_fc1_head_act for fp32).  The
// tiles of k_fc1_fwd_few, 32 columns wide so that 112 CUs share the weights, their sums published instead of stored, and
// the head by the workgroup that arrives last.  Every thread stages; one wave multiplies.
template <int ROWS>
__global__ __launch_bounds__(256, 1) void k_fc1_head_act(misc::Fc1HeadArgs A)
{
    __shared__ __attribute__((aligned(16))) bf16_t lds[fc1_few_lds<32>()];
    __shared__ misc::FewLds L;
    const int by = blockIdx.x % (GFc1::N / 32), bz = blockIdx.x / (GFc1::N / 32);
    const FwdSeg S{A.x, static_cast<const bf16_t *>(A.w), nullptr, nullptr, ROWS, 0, (long)net::A3};
    fc1_few_tile<32, 256>(S, 0, by * 32, bz, lds, [&](int m, int n, v4f v) {
#pragma unroll
        for (int j = 0; j < 4; ++j) misc::publish_word(A.h + (bz * ROWS + m) * net::HID + n + j, v[j]);
    });
    misc::words_acknowledged();
    if (!misc::few_last(A, L, GFc1::N / 32 * FC1_SPLITS)) return;
    misc::few_head<ROWS, FC1_SPLITS>(A, L);
}
inline void launch_fc1_head_act(const misc::Fc1HeadArgs &A, hipStream_t st)
{
    constexpr int TILES = GFc1::N / 32 * FC1_SPLITS;
    if (A.head.E == 1) k_fc1_head_act<1><<<TILES, 256, 0, st>>>(A);
    else k_fc1_head_act<misc::FEW_ROWS><<<TILES, 256, 0, st>>>(A);
}

// Dispatch-order number u of `total` workgroups -> tile number, die-aware as net::tile_of_workgroup
// (a launch that holds two problems numbers each of them by itself).
__device__ __forceinline__ int tile_of(int u, int total)
{
    const int die = u & 7, slot = u >> 3, q = total >> 3, r = total & 7;
    return die * q + (die < r ? die : r) + slot;
}

// ---------------------------------------------------------------------------
// fc1 forward for many rows (Section 3 fourth layer: 3136 -> 512): raw fp32 partial sums of a few
// reduction splits, which the head kernel adds up.
//
// 128 x 128 output tile per workgroup of four waves, 64 x 64 per wave (2 x 2 MFMA blocks, so every
// LDS fragment feeds two matrix instructions), reduction stages of 64 elements, four of them in LDS.
// A CU gets one workgroup (8192 rows have 256 tiles, fewer rows are split until there are about as
// many), so nothing hides a wave's waits but its own depth: stages go from memory straight to LDS,
// three to four ahead, and from LDS to registers one whole stage ahead, so that a stage's sixteen
// MFMAs have their operands from the start and the next stage's reads and requests lie between
// them.  One barrier per stage, none of whose operands are on their way through registers to LDS.
// A row's 128 bytes of a stage are eight 16-byte pieces; piece c of row r lies in place c ^ (r % 8),
// which puts the sixteen rows that a read takes in one pass into different banks without padding
// (a load that goes to LDS cannot pad).  The 49 stages are dealt out evenly to the splits.
// Rows of both operands have to start on a cache line, or every piece of a stage is two requests:
// with the weights half a line off, 8192 rows took 43 us however deep the pipeline was.
// Measured (8192 rows, one split, behind conv3): 43 us with two buffers filled through registers,
// 35 us now; 24 us of it with nothing fetched, 22 us with nothing multiplied.  1536 rows in four
// splits: 13.6 -> 12.0 us.  The requests between the MFMAs instead of in front of them: 34 -> 30 us alone.
// Tile order: the four column tiles of one row tile and split next to each other (they share the
// activations), row tiles of one split after each other (they share the weights).
// ---------------------------------------------------------------------------
namespace f1 {
constexpr int BM = 128, BN = 128;
constexpr int TILE = BM * BK;                    // elements of one operand tile in LDS
// NBUF: stages in LDS.  Four are 131,072 bytes: one workgroup per CU; two are what a workgroup gets without asking.
template <int NBUF> constexpr int lds_bytes() { return 2 * NBUF * TILE * 2; }
constexpr int STAGES = GFc1::K / BK;             // 49

struct Args {
    FwdSeg seg[3];      // tile_begin counts row tiles of BM rows; y = fp32 [M][512] of split 0
    int nseg;
    int nsplit;
    int tiles_m;        // row tiles of all segments
    long split_stride;  // elements between the partial sums of consecutive splits
};

// 16 bytes per lane from memory to LDS, lane l's to p + 8 l, past the registers.  In assembly, because the compiler
// would let every LDS read behind it wait for its arrival; `ready` waits for what a stage needs.
__device__ __forceinline__ void to_lds(const bf16_t *g, bf16_t *p)
{
    const uint32_t at = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)p);
    uint32_t m0;   // left as it was: the compiler may hold something in it, and it is no register to declare as clobbered
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, off\n\ts_mov_b32 m0, %0"
                 : "=&s"(m0) : "s"(at), "v"(g) : "memory");
}

template <int NBUF>
__global__ __launch_bounds__(256, 1) void k_fc1_fwd(Args A)
{
    static_assert(NBUF % 2 == 0 && NBUF <= 4, "register sets alternate by buffer; ready() counts");
    extern __shared__ __attribute__((aligned(16))) bf16_t lds[];   // [operand][buffer][row][BK], pieces in permuted places
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int t = tile_of(blockIdx.x, gridDim.x);
    const int by = t & 3, bx = (t >> 2) % A.tiles_m, bz = (t >> 2) / A.tiles_m;
    FwdSeg S = A.seg[0];
    if (A.nseg > 1 && bx >= A.seg[1].tile_begin) S = A.seg[1];
    if (A.nseg > 2 && bx >= A.seg[2].tile_begin) S = A.seg[2];
    const int m0 = (bx - S.tile_begin) * BM, n0 = by * BN;
    const int s0 = STAGES * bz / A.nsplit, n = STAGES * (bz + 1) / A.nsplit - s0;
    const bf16_t *x = static_cast<const bf16_t *>(S.x);

    // Instruction q of a wave fetches rows 8 (4 wave + q) .. + 7 of a tile: lane l row l / 8, and of that row the
    // 16-byte piece whose place in LDS lane l's is (fetch_piece).
    const int fr = wave * 32 + (lane >> 3), fk = ((lane & 7) ^ (lane >> 3)) * 8;
    const bf16_t *pa[4], *pb[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        int m = m0 + fr + 8 * q;
        if (m > S.M - 1) m = S.M - 1;             // rows past the end repeat the last row; they are never stored
        pa[q] = x + (long)m * S.xs + fk + s0 * BK;
        pb[q] = S.w + (long)(n0 + fr + 8 * q) * GFc1::K + fk + s0 * BK;
    }
    auto fetch_a = [&](int st, int buf, int q) { to_lds(pa[q] + st * BK, lds + buf * TILE + (wave * 4 + q) * 512); };
    auto fetch_b = [&](int st, int buf, int q) { to_lds(pb[q] + st * BK, lds + (NBUF + buf) * TILE + (wave * 4 + q) * 512); };
    const int wm = wave & 1, wn = wave >> 1;
    const int li = lane & 31, h = lane >> 5;
    v16f acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = v16f{0};
    struct Frag { v8bf a[2], b[2]; };             // the operands of one 16-deep step of the wave's 64 x 64
    const bf16_t *ap[4], *bp[4];                  // of step s; the piece's place again
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int at = ((2 * s + h) ^ (li & 7)) * 8;
        ap[s] = lds + (wm * 64 + li) * BK + at;
        bp[s] = lds + NBUF * TILE + (wn * 64 + li) * BK + at;
    }
    auto rd = [&](int buf, int s) {
        Frag F;
        F.a[0] = frag_k(ap[s] + buf * TILE); F.a[1] = frag_k(ap[s] + buf * TILE + 32 * BK);
        F.b[0] = frag_k(bp[s] + buf * TILE); F.b[1] = frag_k(bp[s] + buf * TILE + 32 * BK);
        return F;
    };
    // everything but the last `later` stages that were requested has arrived in LDS, and every wave is through with
    // its reads
    auto ready = [&](int later) {
        if (later >= 3) asm volatile("s_waitcnt vmcnt(24)" ::: "memory");
        else if (later == 2) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
        else if (later == 1) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        sync_lds();
    };

#pragma unroll
    for (int st = 0; st < NBUF; ++st)
        if (st < n)
#pragma unroll
            for (int q = 0; q < 4; ++q) { fetch_a(st, st, q); fetch_b(st, st, q); }
    ready((n < NBUF ? n : NBUF) - 1);                              // stage 0
    Frag F[2][4];
#pragma unroll
    for (int s = 0; s < 4; ++s) F[0][s] = rd(0, s);
    ready((n < NBUF ? n : NBUF) - 2);                              // stage 1, and buffer 0 is free
    // Stage i, whose operands are in registers: stage i + 1 goes from LDS to registers meanwhile and stage i + NBUF is
    // requested into the buffer that stage i was read from.
    auto stage = [&](int i, int buf) {
        Frag (&C)[4] = F[buf & 1], (&X)[4] = F[(buf & 1) ^ 1];
        const bool more = i + NBUF < n;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            X[s] = rd((buf + 1) % NBUF, s);
            __builtin_amdgcn_sched_barrier(0);
            acc[0][0] = mfma(C[s].b[0], C[s].a[0], acc[0][0]);   // transposed tile
            __builtin_amdgcn_sched_barrier(0);
            if (more) fetch_a(i + NBUF, buf, s);
            __builtin_amdgcn_sched_barrier(0);
            acc[0][1] = mfma(C[s].b[1], C[s].a[0], acc[0][1]);
            acc[1][0] = mfma(C[s].b[0], C[s].a[1], acc[1][0]);
            __builtin_amdgcn_sched_barrier(0);
            if (more) fetch_b(i + NBUF, buf, s);
            __builtin_amdgcn_sched_barrier(0);
            acc[1][1] = mfma(C[s].b[1], C[s].a[1], acc[1][1]);
            __builtin_amdgcn_sched_barrier(0);
        }
        ready(n - 3 - i < NBUF - 2 ? n - 3 - i : NBUF - 2);
    };
    for (int i = 0; i < n; i += NBUF)
#pragma unroll
        for (int j = 0; j < NBUF; ++j)
            if (i + j < n) stage(i + j, j);

    // acc[a][b][4g + j] = Y[row block a, lane li][column block b, 8g + 4h + j].  The tile leaves through LDS
    // (the operand buffers are no longer read: the loop ends on a barrier), so that it is written as whole
    // 512-byte rows, two per wave and instruction, instead of 32-byte pieces of 32 different rows.
    constexpr int LDO = NBUF == 4 ? BN + 4 : BN;  // fp32 row stride of the staged output tile
    static_assert(BM * LDO * 4 <= lds_bytes<NBUF>(), "the output tile is staged in the operand buffers");
    float *ot = reinterpret_cast<float *>(lds);
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *reinterpret_cast<v4f *>(&ot[((wm * 2 + a) * 32 + li) * LDO + (wn * 2 + b) * 32 + 8 * g + 4 * h]) =
                    v4f{acc[a][b][4 * g], acc[a][b][4 * g + 1], acc[a][b][4 * g + 2], acc[a][b][4 * g + 3]};
    sync_lds();
    float *y = static_cast<float *>(S.y) + (long)bz * A.split_stride;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int r = (tid >> 5) + 8 * i, cq = (tid & 31) * 4, m = m0 + r;
        if (m < S.M) *reinterpret_cast<v4f *>(y + (long)m * GFc1::N + n0 + cq) = *reinterpret_cast<const v4f *>(&ot[r * LDO + cq]);
    }
}
}  // namespace f1

// ---------------------------------------------------------------------------
using g32::DConv2;
using g32::DFc1;

struct DgradArgs {
    const bf16_t *dy;    // [B][OH][OW][CO]
    const bf16_t *w;     // [CO][KH][KW][CI] bf16 copy of the weights
    const bf16_t *xact;  // [B][H][W][CI] layer input (ReLU output of the layer below)
    bf16_t *dx;          // [B][H][W][CI]
    int B;
};

// DB: the LDS tiles are double-buffered, which leaves one barrier per reduction stage instead of two
// (for the layers whose stages are so short that the barriers dominate them), and a wave with a
// single output block alternates between two accumulators so that consecutive MFMAs do not wait
// for each other's result.
// LDS elements of an input-gradient tile
template <int BM, int BN, bool DB> constexpr int dgrad_lds() { return (DB ? 2 : 1) * (BM * LDK + BK * BN); }

// Tile number t of a (gx, gy, gz) grid of tiles; tile order: the parity classes of one row tile
// together, then the row tiles of one column tile.
template <class D, int BM, int BN, int WM, int WN, bool DB>
__device__ __forceinline__ void dgrad_tile(const DgradArgs &A, int t, int gx, int gz, bf16_t *lds)
{
    constexpr int WAVES_M = BM / (32 * WM), WAVES_N = BN / (32 * WN), T = WAVES_M * WAVES_N * 64;
    constexpr int NA = BM * 8 / T;
    constexpr int LDB = BN;              // row stride of the [k][c] weight tile
    constexpr int BCH = BN / 8;          // 16-byte chunks per weight-tile row
    constexpr int BROWS = T / BCH;       // rows filled per pass
    constexpr int NBL = (BK + BROWS - 1) / BROWS;
    static_assert(NA * T == BM * 8 && D::CO % BK == 0 && BROWS % 4 == 0, "tile/threads mismatch");
    constexpr int NBUF = DB ? 2 : 1;
    constexpr bool ACC2 = DB && WM * WN == 1;
    bf16_t(*As2)[BM * LDK] = reinterpret_cast<bf16_t(*)[BM * LDK]>(lds);
    bf16_t(*Bs2)[BK * LDB] = reinterpret_cast<bf16_t(*)[BK * LDB]>(lds + NBUF * BM * LDK);

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int bz = t % gz, bx = (t / gz) % gx, by = t / (gz * gx);
    const int m0 = bx * BM, n0 = by * BN;
    const int ca = bz / D::S, cb = bz % D::S;
    const int Mc = A.B * D::PP;

    const int lr = tid >> 3, kq = (tid & 7) * 8;
    int rn[NA], rh[NA], rw[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        int m = m0 + lr + i * (T / 8);
        if (m < Mc) {
            rn[i] = m / D::PP;
            int r = m % D::PP;
            rh[i] = r / D::WP;
            rw[i] = r % D::WP;
        } else {
            rn[i] = -1; rh[i] = 0; rw[i] = 0;
        }
    }
    const int br = tid / BCH, bc = (tid % BCH) * 8, bst = TrTile<BN>::at(br, bc);
    uint4 ra[NA], rb[NBL];
    auto gload = [&](int k0) {
        const int tap = k0 / D::CO, o0 = k0 % D::CO;
        const int u = tap / D::TW, v = tap % D::TW;
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            int ii = rh[i] - u, jj = rw[i] - v;
            bool ok = rn[i] >= 0 && ii >= 0 && ii < D::OH && jj >= 0 && jj < D::OW;
            ra[i] = ok ? ld8(A.dy + ((long)(rn[i] * D::OH + ii) * D::OW + jj) * D::CO + o0 + kq)
                       : uint4{0, 0, 0, 0};
        }
        const int p = ca + D::S * u, q = cb + D::S * v;
#pragma unroll
        for (int i = 0; i < NBL; ++i) {
            int r = br + i * BROWS;
            if (r < BK) rb[i] = ld8(A.w + ((long)((o0 + r) * D::KH + p) * D::KW + q) * D::CI + n0 + bc);
        }
    };
    auto sstore = [&](int buf) {
        bf16_t *As = As2[buf], *Bs = Bs2[buf];
#pragma unroll
        for (int i = 0; i < NA; ++i) *reinterpret_cast<uint4 *>(&As[(lr + i * (T / 8)) * LDK + kq]) = ra[i];
#pragma unroll
        for (int i = 0; i < NBL; ++i) {
            int r = br + i * BROWS;
            if (r < BK) *reinterpret_cast<uint4 *>(&Bs[i * BROWS * LDB + bst]) = rb[i];
        }
    };

    const int wm = wave % WAVES_M, wn = wave / WAVES_M;
    const int li = lane & 31, h = lane >> 5, s16 = lane & 15, half = (lane >> 4) & 1;
    const int apo = (wm * 32 * WM + li) * LDK + 8 * h;
    // transpose-read base: row 8h + s/4, column (wave block) + 16*half + 4*(s%4)
    int bpo[WN];
#pragma unroll
    for (int b = 0; b < WN; ++b) bpo[b] = TrTile<BN>::at(8 * h + (s16 >> 2), (wn * WN + b) * 32 + 16 * half + 4 * (s16 & 3));
    v16f acc[WM][WN];
#pragma unroll
    for (int a = 0; a < WM; ++a)
#pragma unroll
        for (int b = 0; b < WN; ++b) acc[a][b] = v16f{0};

    // where this lane's results go, and the stored activations there (the ReLU mask), requested
    // before the loop so the epilogue does not wait for them
    long obase[WM];
    uint2 xa[WM][WN][4];
#pragma unroll
    for (int a = 0; a < WM; ++a) {
        const int m = m0 + (wm * WM + a) * 32 + li;
        obase[a] = -1;
        if (m < Mc) {
            const int n = m / D::PP, rr = m % D::PP;
            const int hh = D::S * (rr / D::WP) + ca, ww = D::S * (rr % D::WP) + cb;
            obase[a] = ((long)(n * D::H + hh) * D::W + ww) * D::CI + n0 + wn * WN * 32 + 4 * h;
        }
        // (unconditional, from a clamped address: a value chosen between a loaded one and a constant would
        // be waited for right here, in front of the first stage's loads)
        const long ob = obase[a] >= 0 ? obase[a] : 0;
#pragma unroll
        for (int b = 0; b < WN; ++b)
#pragma unroll
            for (int g = 0; g < 4; ++g) xa[a][b][g] = *reinterpret_cast<const uint2 *>(A.xact + ob + b * 32 + 8 * g);
    }

    v16f acc2 = {0};   // second accumulator (ACC2 only)
    auto compute = [&](int buf) {
        const bf16_t *ap = As2[buf] + apo, *bp = Bs2[buf];
        // the fragments of a 16-deep step are requested before the matrix instructions of the step before it
        auto frags = [&](int kk, v8bf (&fa)[WM], v8bf (&fb)[WN]) {
#pragma unroll
            for (int a = 0; a < WM; ++a) fa[a] = frag_k(ap + a * 32 * LDK + kk);
#pragma unroll
            for (int b = 0; b < WN; ++b) fb[b] = frag_tr(bp + kk * LDB + bpo[b], LDB);
        };
        v8bf fa[WM], fb[WN], fan[WM], fbn[WN];
        frags(0, fa, fb);
#pragma unroll
        for (int kk = 0; kk < BK; kk += 16) {
            if (kk + 16 < BK) frags(kk + 16, fan, fbn);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int a = 0; a < WM; ++a)
#pragma unroll
                for (int b = 0; b < WN; ++b) {  // transposed tile
                    if (ACC2 && (kk & 16)) acc2 = mfma(fb[b], fa[a], acc2);
                    else acc[a][b] = mfma(fb[b], fa[a], acc[a][b]);
                }
            __builtin_amdgcn_sched_barrier(0);
            if (kk + 16 < BK) {
#pragma unroll
                for (int a = 0; a < WM; ++a) fa[a] = fan[a];
#pragma unroll
                for (int b = 0; b < WN; ++b) fb[b] = fbn[b];
            }
        }
    };
    gload(0);
    if constexpr (DB) {
        int s = 0;
        for (int k0 = 0; k0 < D::K; k0 += BK, s ^= 1) {
            sstore(s);
            if (k0 + BK < D::K) gload(k0 + BK);
            sync_lds();   // buffer s is complete; every wave is past the previous stage, which read buffer s^1
            compute(s);
        }
        if (ACC2) acc[0][0] += acc2;
    } else {
        sstore(0);
        __syncthreads();
        for (int k0 = 0; k0 < D::K; k0 += BK) {
            const bool more = k0 + BK < D::K;
            if (more) gload(k0 + BK);
            compute(0);
            __syncthreads();
            if (more) {
                sstore(0);
                __syncthreads();
            }
        }
    }

    // acc[a][b][4g + j] = dX[position m = block a, lane li][channel = block b, 8g + 4h + j]
#pragma unroll
    for (int a = 0; a < WM; ++a) {
        if (obase[a] < 0) continue;
#pragma unroll
        for (int b = 0; b < WN; ++b) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const uint2 x = xa[a][b][g];
                // ReLU mask of the layer below: its stored output is > 0
                const float v0 = (int16_t)(x.x & 0xFFFFu) > 0 ? acc[a][b][4 * g] : 0.f;
                const float v1 = (int16_t)(x.x >> 16) > 0 ? acc[a][b][4 * g + 1] : 0.f;
                const float v2 = (int16_t)(x.y & 0xFFFFu) > 0 ? acc[a][b][4 * g + 2] : 0.f;
                const float v3 = (int16_t)(x.y >> 16) > 0 ? acc[a][b][4 * g + 3] : 0.f;
                *reinterpret_cast<uint2 *>(A.dx + obase[a] + b * 32 + 8 * g) = pack4(v0, v1, v2, v3);
            }
        }
    }
}


// ---------------------------------------------------------------------------
struct WgradArgs {
    const bf16_t *dy;  // [B*P][N]
    const void *x;     // layer input: uint8 (conv1) or bf16
    float *part;       // [splits][N*K + N] fp32
    int B;
    int rps;           // reduction rows per split, a multiple of 64
    long xs;
    long part_stride;
    float scale;
};

// LDS elements of a weight-gradient tile
template <int BMO, int BNK, bool DB> constexpr int wgrad_lds() { return (DB ? 2 : 1) * BK * (BMO + BNK); }

// Tile number t of a (gx, gy, gz) grid of tiles; tile order: with row splits (conv layers) all
// tiles of one split together; without (fc1) all output tiles of one input-column tile together.
// DB: double-buffered LDS tiles (one barrier per reduction stage) and, for a wave with a single
// output block, two alternating accumulators, as in the input gradient.
template <class G, int BMO, int BNK, int WM, int WN, bool DB>
__device__ __forceinline__ void wgrad_tile(const WgradArgs &A, int t, int gx, int gy, int gz, bf16_t *lds)
{
    constexpr int WAVES_M = BMO / (32 * WM), WAVES_N = BNK / (32 * WN), T = WAVES_M * WAVES_N * 64;
    constexpr int LDY = BMO, LDX = BNK;
    constexpr int YCH = BMO / 8, XCH = BNK / 8;          // 16-byte chunks per tile row
    constexpr int YR = T / YCH;                          // rows filled per pass
    constexpr int NY = (BK + YR - 1) / YR;
    constexpr bool WHOLE = T % XCH == 0;                 // a pass fills whole rows of X: a thread has one column
    constexpr int XR = T / XCH, NX = WHOLE ? (BK + XR - 1) / XR : BK * XCH / T, NC = WHOLE ? 1 : NX;
    static_assert(YR % 4 == 0 && (WHOLE ? XR % 4 == 0 : BK * XCH % T == 0), "rows permuted alike");
    using in_t = typename in_type<G>::t;
    constexpr int NBUF = DB ? 2 : 1;
    constexpr bool ACC2 = DB && WM * WN <= 3;   // two alternating accumulators per output block
    bf16_t(*Ys2)[BK * LDY] = reinterpret_cast<bf16_t(*)[BK * LDY]>(lds);
    bf16_t(*Xs2)[BK * LDX] = reinterpret_cast<bf16_t(*)[BK * LDX]>(lds + NBUF * BK * LDY);

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int bx, by, bz;
    if (gz > 1) {
        bx = t % gx; by = (t / gx) % gy; bz = t / (gx * gy);
    } else {
        by = t % gy; bx = t / gy; bz = 0;
    }
    const int kc0 = bx * BNK, o0 = by * BMO;
    const int mbeg = bz * A.rps;
    const int mend = min(mbeg + A.rps, A.B * G::P);
    const in_t *x = static_cast<const in_t *>(A.x);

    const int yr = tid / YCH, yc = (tid % YCH) * 8;
    const int yst = TrTile<BMO>::at(yr, yc);
    int xr[NC], xko[NC], xst[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        const int q = tid + i * T, xc = (q % XCH) * 8;
        xr[i] = q / XCH;
        xko[i] = G::k_off(kc0 + xc);
        xst[i] = TrTile<BNK>::at(xr[i], xc);
    }
    uint4 ry[NY], rx[NX];
    auto gload = [&](int mb) {
#pragma unroll
        for (int i = 0; i < NY; ++i) {
            int r = yr + i * YR, m = mb + r;
            ry[i] = (r < BK && m < mend) ? ld8(A.dy + (long)m * G::N + o0 + yc) : uint4{0, 0, 0, 0};
        }
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            int r = WHOLE ? xr[0] + i * XR : xr[i % NC], m = mb + r;
            rx[i] = (r < BK && m < mend) ? ld8(x + G::row_off(m, A.xs) + xko[i % NC]) : uint4{0, 0, 0, 0};
        }
    };
    auto sstore = [&](int buf) {
        bf16_t *Ys = Ys2[buf], *Xs = Xs2[buf];
#pragma unroll
        for (int i = 0; i < NY; ++i) {
            int r = yr + i * YR;
            if (r < BK) *reinterpret_cast<uint4 *>(&Ys[i * YR * LDY + yst]) = ry[i];
        }
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            if (!WHOLE) *reinterpret_cast<uint4 *>(&Xs[xst[i % NC]]) = rx[i];
            else if (xr[0] + i * XR < BK) *reinterpret_cast<uint4 *>(&Xs[i * XR * LDX + xst[0]]) = rx[i];
        }
    };

    const int wo = wave % WAVES_M, wk = wave / WAVES_M;
    const int li = lane & 31, h = lane >> 5, s16 = lane & 15, half = (lane >> 4) & 1;
    const int trow = 8 * h + (s16 >> 2), tcol = 16 * half + 4 * (s16 & 3);
    int ypo[WM], xpo[WN];
#pragma unroll
    for (int a = 0; a < WM; ++a) ypo[a] = TrTile<BMO>::at(trow, (wo * WM + a) * 32 + tcol);
#pragma unroll
    for (int b = 0; b < WN; ++b) xpo[b] = TrTile<BNK>::at(trow, (wk * WN + b) * 32 + tcol);
    const bool do_bias = bx == 0 && wk == 0;
    v16f acc[WM][WN], accb[WM];
#pragma unroll
    for (int a = 0; a < WM; ++a) {
        accb[a] = v16f{0};
#pragma unroll
        for (int b = 0; b < WN; ++b) acc[a][b] = v16f{0};
    }
    v8bf ones;
#pragma unroll
    for (int e = 0; e < 8; ++e) ones[e] = (__bf16)1.0f;

    v16f acc2[WM][WN];   // second accumulators (ACC2 only)
#pragma unroll
    for (int a = 0; a < WM; ++a)
#pragma unroll
        for (int b = 0; b < WN; ++b) acc2[a][b] = v16f{0};
    auto compute = [&](int buf) {
        const bf16_t *yp = Ys2[buf], *xp = Xs2[buf];
        // the fragments of a 16-deep step are requested before the matrix instructions of the step before it
        auto frags = [&](int kk, v8bf (&fa)[WM], v8bf (&fb)[WN]) {
#pragma unroll
            for (int a = 0; a < WM; ++a) fa[a] = frag_tr(yp + kk * LDY + ypo[a], LDY);
#pragma unroll
            for (int b = 0; b < WN; ++b) fb[b] = frag_tr(xp + kk * LDX + xpo[b], LDX);
        };
        v8bf fa[WM], fb[WN], fan[WM], fbn[WN];
        frags(0, fa, fb);
#pragma unroll
        for (int kk = 0; kk < BK; kk += 16) {
            if (kk + 16 < BK) frags(kk + 16, fan, fbn);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int a = 0; a < WM; ++a) {
#pragma unroll
                for (int b = 0; b < WN; ++b) {
                    if (ACC2 && (kk & 16)) acc2[a][b] = mfma(fa[a], fb[b], acc2[a][b]);
                    else acc[a][b] = mfma(fa[a], fb[b], acc[a][b]);
                }
                if (do_bias) accb[a] = mfma(fa[a], ones, accb[a]);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (kk + 16 < BK) {
#pragma unroll
                for (int a = 0; a < WM; ++a) fa[a] = fan[a];
#pragma unroll
                for (int b = 0; b < WN; ++b) fb[b] = fbn[b];
            }
        }
    };
    if constexpr (DB) {
        if (mbeg < mend) gload(mbeg);
        int sb = 0;
        for (int mb = mbeg; mb < mend; mb += BK, sb ^= 1) {
            sstore(sb);
            if (mb + BK < mend) gload(mb + BK);
            sync_lds();   // buffer sb is complete; every wave is past the previous stage, which read buffer sb^1
            compute(sb);
        }
        if (ACC2) {
#pragma unroll
            for (int a = 0; a < WM; ++a)
#pragma unroll
                for (int b = 0; b < WN; ++b) acc[a][b] += acc2[a][b];
        }
    } else {
        if (mbeg < mend) {
            gload(mbeg);
            sstore(0);
        }
        __syncthreads();
        for (int mb = mbeg; mb < mend; mb += BK) {
            const bool more = mb + BK < mend;
            if (more) gload(mb + BK);
            compute(0);
            __syncthreads();
            if (more) {
                sstore(0);
                __syncthreads();
            }
        }
    }

    float *part = A.part + (long)bz * A.part_stride;
#pragma unroll
    for (int a = 0; a < WM; ++a) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            int o = o0 + (wo * WM + a) * 32 + 8 * (r / 4) + 4 * h + (r % 4);
#pragma unroll
            for (int b = 0; b < WN; ++b) {
                int col = kc0 + (wk * WN + b) * 32 + li;
                part[(long)o * G::K + col] = acc[a][b][r] * A.scale;
            }
            if (do_bias && li == 0) part[(long)G::N * G::K + o] = accb[a][r];
        }
    }
}

// The input gradient and the weight gradient of fc1 go into ONE launch of 64x64 tiles (both
// read the layer's dY and depend on nothing else that is computed in the backward pass): nd
// input-gradient tiles, then nw weight-gradient tiles.  (The conv layers' pairs: c3b and dps.)
struct PairGrid {
    int nd, dgx, dgz;        // input gradient: tiles, grid x and z
    int nw, wgx, wgy, wgz;   // weight gradient: tiles, grid
};

// ===========================================================================
// conv1 (8x8 stride 4 over the uint8 frame stack), specialised.
//
// The generic kernels gather conv1's im2col rows from global memory in 4/8-byte
// pieces at 84-byte strides, which is address-bound.  Here the 84x84 frames are
// read with 16-byte loads -- from a materialised state, or straight from the
// replay ring through the sampled slot (the frame-stack gather fused into the
// loader) -- converted to bf16 and kept in LDS, and every operand of the 8x8/4
// convolution is an LDS read at a computed address:
//   forward : one WAVE stages the 20 input rows under 4 output rows of the four
//             frames in LDS of its own and reads them as two-row "quads";
//             all of W (32x256 bf16) sits in registers (see k_conv1_fwd);
//   wgrad   : one WORKGROUP stages two whole frames of a sample; 8 consecutive
//             pixels of one im2col column are fetched with the LDS transpose
//             load, whose lanes each supply their own address.
// ===========================================================================
namespace c1 {
constexpr int FR = 84 * 84;       // elements per frame

struct Src {                      // where the four frames of sample n come from
    const uint8_t *x;             // explicit states [n][4][84][84] (idx == nullptr) or the ring
    long xs;                      // bytes between samples (explicit)
    const int32_t *idx;           // sampled slots (ring mode)
    long cap;                     // ring capacity
    int shift;                    // 0: frames i-3..i (s), 1: frames i-2..i+1 (s')
    int sub;                      // length of the sub-ring a window wraps in: the capacity (one stream),
                                  // or the share of one environment stream when the ring holds many
};

// First slot of the sub-ring that slot i lies in.
__device__ __forceinline__ long sub_ring_base(const Src &S, long i)
{
    return (long)S.sub == S.cap ? 0 : (long)((uint32_t)i / (uint32_t)S.sub) * S.sub;
}

// The sampled slot of sample n (ring mode; 0 otherwise).  Fetched one sample ahead of the frame
// loads that depend on it, so that the two memory latencies do not add up.
// The value stays in a vector register until it is used (frame_ptr makes it scalar): were it
// made scalar where it is loaded, the wave would wait for every outstanding load right there.
__device__ __forceinline__ int sample_slot(const Src &S, int n)
{
    int zero;
    asm volatile("v_mov_b32 %0, 0" : "=v"(zero));  // opaque, so the load below is a vector load
    return S.idx ? S.idx[n + zero] : 0;
}

__device__ __forceinline__ const uint8_t *frame_ptr(const Src &S, int n, int slot_n, int k)
{
    if (!S.idx) return S.x + (long)n * S.xs + (long)k * FR;
    long i = __builtin_amdgcn_readfirstlane(slot_n);
    i = i < 0 ? 0 : (i >= S.cap ? S.cap - 1 : i);
    const long base = sub_ring_base(S, i);
    long slot = i - base - 3 + k + S.shift;  // within [-3, sub+1]: one wrap at most (sub >= 5)
    if (slot < 0) slot += S.sub;
    if (slot >= S.sub) slot -= S.sub;
    return S.x + (base + slot) * FR;
}

// Staging of frames k0 .. k0+NF-1 of sample n as bf16 into xin[(k-k0)*FR ...], in two halves so
// that the global loads of the next sample can be in flight while the current one is computed:
// stage_load issues every 16-byte load of a thread, stage_store converts (16 pixels -> 16 bf16)
// and writes two 16-byte LDS stores per load.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // a native vector: stays in registers
template <int T, int NF> struct Staged {
    static constexpr int CH = FR / 16, TOT = NF * CH, NL = (TOT + T - 1) / T;
    u32x4 raw[NL];
};
template <int T, int NF>
__device__ __forceinline__ void stage_load(Staged<T, NF> &R, const Src &S, int n, int slot_n, int k0, int tid)
{
    using ST = Staged<T, NF>;
    // the (workgroup-uniform) frame addresses first, so that the slot lookup does not sit
    // between the frame loads and serialise them
    const uint8_t *f[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) f[k] = frame_ptr(S, n, slot_n, k0 + (k < NF ? k : 0));
#pragma unroll
    for (int i = 0; i < ST::NL; ++i) {
        int t = tid + i * T;
        if (t > ST::TOT - 1) t = ST::TOT - 1;   // the last pass repeats a piece rather than branching
        const int k = t / ST::CH;
        const uint8_t *fp = k == 0 ? f[0] : k == 1 ? f[1] : k == 2 ? f[2] : f[3];
        R.raw[i] = *reinterpret_cast<const u32x4 *>(fp + (t % ST::CH) * 16);
    }
}
// 16 pixels -> 16 bf16 -> two 16-byte LDS stores; consecutive lanes write consecutive 32 bytes
template <int T, int NF>
__device__ __forceinline__ void stage_store(bf16_t *xin, const Staged<T, NF> &R, int tid)
{
    using ST = Staged<T, NF>;
#pragma unroll
    for (int i = 0; i < ST::NL; ++i) {
        const int t = tid + i * T;
        if (t < ST::TOT) {
            const u32x4 r = R.raw[i];
            uint4 *d = reinterpret_cast<uint4 *>(xin + t * 16);  // frames are contiguous in xin: (t/CH)*FR + (t%CH)*16 == t*16
            d[0] = cvt8_u8(r.x, r.y);
            d[1] = cvt8_u8(r.z, r.w);
        }
    }
}

struct FwdSeg {
    Src src;
    const bf16_t *w;    // [32][256] bf16
    const float *bias;  // [32]
    bf16_t *y;          // [n][400][32]
    int n;              // samples
    int first;          // index of the segment's first sample in the launch-wide sample list
};
struct FwdArgs {
    FwdSeg seg[3];
    int nseg;
    int total;          // samples of all segments
    int draw;           // replay mode: the kernel draws sample g of every segment itself (draw g of `samp`);
                        // segment 0 publishes the draws
    misc::SampleArgs samp;
};

// Forward pass, one WAVE per unit of work and no workgroup barrier anywhere.
//
// A unit is a strip of 4 output rows of one sample: 80 output pixels = 16 lanes x 5 consecutive
// pixels of one output row.  Its receptive field, input rows 16s .. 16s+19 of the four frames
// (13,440 bytes as bf16), sits in a part of LDS that belongs to this wave alone, so staging,
// matrix instructions and stores of different waves never wait for each other.
//
// v_mfma_f32_16x16x32_bf16, weights as the a-operand (row r = channel 8*(r/4) + 4*hh + r%4 for
// channel half hh), pixels as the b-operand (column n = lane % 16: output row n/4 of the strip,
// pixels 5*(n%4) .. +4 of that row).  Reduction step (c, xh) covers frame c, all 8 kernel rows,
// kernel columns 4xh .. 4xh+3: lane group kg = lane/16 holds kernel rows 2kg and 2kg+1, four
// columns each.  With that split the operand of pixel j at step (c, xh) is the "quad"
//   q[c][j + xh] = { input row 2kg, columns 4(j+xh)..+3 ; input row 2kg+1, same columns },
// i.e. six quads per frame serve all five pixels and both column halves, each fetched by ONE
// two-address LDS read, and every input element is read from LDS 2.4 times instead of 4.
// The result of lane (n, g = lane/16) is channels 8g .. 8g+7 of its pixels: 16 bytes per store.
constexpr int SROWS = 20;               // input rows per strip
constexpr int STRIP = 4 * SROWS * 84;   // elements per strip (four frames)
constexpr int UNITS = 5;                // strips per sample
constexpr int CHUNKS = STRIP / 16;      // 16-byte pieces of a strip's pixels: 420
constexpr int MAX_DRAWS = 8;            // samples one wave may draw for itself

struct StripRaw { u32x4 raw[7]; };      // this lane's pieces lane, lane + 64, ... of a strip
struct StripOff { uint32_t off[7]; };   // their byte offsets within four frames that are contiguous in memory

// The pixels of strip `strip` of sample g.  Four frames of a ring sample are contiguous unless
// they straddle the end of the ring (or its start, for the first slots); explicit states always are.
__device__ __forceinline__ void strip_load(StripRaw &R, const Src &S, int g, int slot_g, int strip, int lane,
                                           const StripOff &O)
{
    const uint8_t *base;
    bool contig = true;
    long b = 0, rb = 0;                           // first frame's slot within its sub-ring; the sub-ring's first slot
    if (!S.idx) {
        base = S.x + (long)g * S.xs;
    } else {
        long i = __builtin_amdgcn_readfirstlane(slot_g);
        i = i < 0 ? 0 : (i >= S.cap ? S.cap - 1 : i);
        rb = sub_ring_base(S, i);
        b = i - rb - 3 + S.shift;                 // within [-3, sub - 2]
        contig = b >= 0 && b + 3 < S.sub;
        base = S.x + (rb + b) * FR;
    }
    if (contig) {   // one scalar base, per-lane offsets that never change
        base += strip * (16 * 84);
#pragma unroll
        for (int i = 0; i < 7; ++i)
            if (i < 6 || lane < CHUNKS - 384) R.raw[i] = *reinterpret_cast<const u32x4 *>(base + O.off[i]);
    } else {
#pragma unroll
        for (int i = 0; i < 7; ++i) {
            const int t = lane + 64 * i;
            if (t < CHUNKS) {
                long slot = b + t / (CHUNKS / 4);
                if (slot < 0) slot += S.sub;
                if (slot >= S.sub) slot -= S.sub;
                R.raw[i] = *reinterpret_cast<const u32x4 *>(S.x + (rb + slot) * FR + strip * (16 * 84) + (t % (CHUNKS / 4)) * 16);
            }
        }
    }
}
// 16 pixels -> 16 bf16 -> two 16-byte LDS stores; consecutive lanes write consecutive 32 bytes
__device__ __forceinline__ void strip_store(bf16_t *xs, const StripRaw &R, int lane)
{
#pragma unroll
    for (int i = 0; i < 7; ++i) {
        const int t = lane + 64 * i;
        if (t < CHUNKS) {
            const u32x4 r = R.raw[i];
            uint4 *d = reinterpret_cast<uint4 *>(xs + t * 16);
            d[0] = cvt8_u8(r.x, r.y);
            d[1] = cvt8_u8(r.z, r.w);
        }
    }
}

// Units [u0, u1) of one segment (unit = UNITS * sample + strip), processed by one wave.  Weights and
// bias stay in registers; the pixels of the next unit are loaded while the current one is computed,
// and the ring slot of the unit after that is already on its way.
//
// In draw mode the kernel has drawn the samples itself (see k_conv1_fwd) and `slots` holds them;
// otherwise the slots are read from S.src.idx, where a sampling kernel left them.
__device__ __forceinline__ void conv1_fwd_units(const FwdSeg &S, int u0, int u1, bf16_t *xs, const int *slots, int lane)
{
    const int n = lane & 15, kg = lane >> 4, oyl = n >> 2, q = n & 3;
    StripOff O;
#pragma unroll
    for (int i = 0; i < 7; ++i) {
        const int t = lane + 64 * i;
        O.off[i] = t < CHUNKS ? (t / (CHUNKS / 4)) * FR + (t % (CHUNKS / 4)) * 16 : 0;
    }
    StripRaw R;
    int g = u0 / UNITS, strip = u0 % UNITS;   // current unit
    int gn = g, sn = strip + 1;               // next unit
    if (sn == UNITS) { sn = 0; ++gn; }
    // draw mode: slots[] holds the slots of this wave's samples of this segment, first one at index 0
    const int gfirst = g;
    auto slot_of = [&](int gq) { return slots ? slots[gq - gfirst] : sample_slot(S.src, gq); };
    strip_load(R, S.src, g, slot_of(g), strip, lane, O);
    int slot_next = u0 + 1 < u1 ? slot_of(gn) : 0;
    v8bf wa[8][2];   // [2c + xh][channel half]
#pragma unroll
    for (int st = 0; st < 8; ++st)
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
            const int ch = 8 * (n >> 2) + 4 * hh + (n & 3);
            const bf16_t *p = S.w + ch * 256 + (st >> 1) * 64 + (2 * kg) * 8 + 4 * (st & 1);
            const uint2 lo = *reinterpret_cast<const uint2 *>(p), hi = *reinterpret_cast<const uint2 *>(p + 8);
            wa[st][hh] = __builtin_bit_cast(v8bf, uint4{lo.x, lo.y, hi.x, hi.y});
        }
    const v4f b0 = *reinterpret_cast<const v4f *>(S.bias + 8 * kg), b1 = *reinterpret_cast<const v4f *>(S.bias + 8 * kg + 4);
    // LDS byte address of this lane's first quad of frame 0; a frame is SROWS * 84 elements further
    const uint32_t px = (uint32_t)(uintptr_t)(xs + (4 * oyl + 2 * kg) * 84 + 20 * q);
    const uint32_t yoff = ((20 * oyl + 5 * q) * 32 + 8 * kg) * 2;   // bytes, within the unit's 80 output pixels
    for (int u = u0; u < u1; ++u) {
        strip_store(xs, R, lane);   // LDS operations of one wave complete in order: no wait needed around this
        if (u + 1 < u1) {
            strip_load(R, S.src, gn, slot_next, sn, lane, O);
            int g2 = gn;
            if (sn + 1 == UNITS) ++g2;
            if (u + 2 < u1) slot_next = slot_of(g2);
        }
        struct Quads { uint4 q[6]; };
        // The compiler would pair neighbouring columns of ONE row into a two-address read and then
        // shuffle registers; the pairing wanted here is the same columns of TWO rows (21 eight-byte
        // steps apart), which lands each quad in the four consecutive registers the MFMA reads.
        // These reads are invisible to the compiler's wait counting: the waits are written out.
        auto quads = [&](int c) {
            typedef uint32_t v4u __attribute__((ext_vector_type(4)));
            const uint32_t addr = px + c * (SROWS * 84 * 2);
            Quads Q;
#define C1_RD2(JJ) { v4u t; asm volatile("ds_read2_b64 %0, %1 offset0:%2 offset1:%3" : "=v"(t) : "v"(addr), "n"(JJ), "n"(JJ + 21)); Q.q[JJ] = uint4{t.x, t.y, t.z, t.w}; }
            C1_RD2(0) C1_RD2(1) C1_RD2(2) C1_RD2(3) C1_RD2(4) C1_RD2(5)
#undef C1_RD2
            return Q;
        };
        v4f acc[5][2];
#pragma unroll
        for (int j = 0; j < 5; ++j) acc[j][0] = acc[j][1] = v4f{0, 0, 0, 0};
        Quads cur = quads(0);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            Quads nxt = cur;
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // `cur` has arrived
            if (c < 3) nxt = quads(c + 1);                        // in flight during the 20 MFMAs below
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int xh = 0; xh < 2; ++xh)
#pragma unroll
                for (int j = 0; j < 5; ++j) {
                    const v8bf b = __builtin_bit_cast(v8bf, cur.q[j + xh]);
                    acc[j][0] = mfma16(wa[2 * c + xh][0], b, acc[j][0]);
                    acc[j][1] = mfma16(wa[2 * c + xh][1], b, acc[j][1]);
                }
            __builtin_amdgcn_sched_barrier(0);
            cur = nxt;
        }
        // bias, 1/255, ReLU, bf16; the 80 pixels of a unit are contiguous in y
        uint8_t *yb = reinterpret_cast<uint8_t *>(S.y) + ((long)g * 400 + 80 * strip) * 64;
        constexpr float sc = 1.0f / 255.0f;
#pragma unroll
        for (int j = 0; j < 5; ++j) {
            const v4f a0 = acc[j][0], a1 = acc[j][1];
            const uint2 lo = pack4(fmaxf(a0.x * sc + b0.x, 0.f), fmaxf(a0.y * sc + b0.y, 0.f),
                                   fmaxf(a0.z * sc + b0.z, 0.f), fmaxf(a0.w * sc + b0.w, 0.f));
            const uint2 hi = pack4(fmaxf(a1.x * sc + b1.x, 0.f), fmaxf(a1.y * sc + b1.y, 0.f),
                                   fmaxf(a1.z * sc + b1.z, 0.f), fmaxf(a1.w * sc + b1.w, 0.f));
            *reinterpret_cast<uint4 *>(yb + yoff + j * 64) = uint4{lo.x, lo.y, hi.x, hi.y};
        }
        g = gn; strip = sn;
        if (++sn == UNITS) { sn = 0; ++gn; }
    }
}

// Draw mode (replay: every segment has the same n samples, sample g of a segment is draw g).
// The wave walks the sum-tree (Eq.10) for the samples of its unit range [u0, u1) before it requests
// a pixel: two draws per walk, its range touches two samples as a rule and never more than
// MAX_DRAWS (the host sizes the grid accordingly).  slots[k] = slot of the k-th sample of the
// range; with `publish`, the wave that owns strip 0 of a sample of segment 0 writes the index, the
// raw importance weight and the transition data for the kernels that follow.
__device__ __forceinline__ void draw_slots(const misc::SampleArgs &P, int n, int u0, int u1, int *slots, int lane,
                                           bool publish)
{
    const int gs0 = u0 / UNITS, gs1 = (u1 - 1) / UNITS;   // launch-wide sample numbers
#pragma unroll 1
    for (int ga = gs0; ga <= gs1; ga += 2) {
        const int gb = ga + 1 <= gs1 ? ga + 1 : ga;
        const int jj[2] = {ga % n, gb % n};
        long sl[2];
        float leaf[2];
        const float total = misc::per_sample_walk<2>(P, jj, lane, sl, leaf);
        if (lane == 0) {
            slots[ga - gs0] = (int)sl[0];
            slots[gb - gs0] = (int)sl[1];
        }
        // lanes 0 and 1 publish one draw each
        if (lane == 0 && publish && ga < n && UNITS * ga >= u0) misc::per_sample_emit(P, ga, sl[0], total, leaf[0]);
        if (lane == 1 && publish && gb < n && gb != ga) misc::per_sample_emit(P, gb, sl[1], total, leaf[1]);
    }
}

// Wave w of the launch owns units [w*U/W, (w+1)*U/W) of the launch-wide list (segment after segment,
// U = UNITS * samples, W = 4 * gridDim.x).  Two workgroups of four waves fit one CU.
__global__ __launch_bounds__(256, 2) void k_conv1_fwd(FwdArgs A)
{
    __shared__ __attribute__((aligned(16))) bf16_t lds[4 * STRIP];
    __shared__ int slot_tab[4][MAX_DRAWS];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    bf16_t *xs = lds + wave * STRIP;
    const long nw = (long)gridDim.x * 4, wid = (long)blockIdx.x * 4 + wave, units = (long)A.total * UNITS;
    const int u0 = (int)(wid * units / nw), u1 = (int)((wid + 1) * units / nw);
    if (A.draw && u0 < u1) draw_slots(A.samp, A.seg[0].n, u0, u1, slot_tab[wave], lane, true);
    for (int s = 0; s < A.nseg; ++s) {
        FwdSeg S = A.seg[0];
        if (s == 1) S = A.seg[1];
        if (s == 2) S = A.seg[2];
        const int lo = max(u0, UNITS * S.first) - UNITS * S.first;
        const int hi = min(u1, UNITS * (S.first + S.n)) - UNITS * S.first;
        // the first sample of [lo, hi) is launch-wide sample S.first + lo / UNITS
        if (lo < hi) conv1_fwd_units(S, lo, hi, xs, A.draw ? slot_tab[wave] + (S.first + lo / UNITS - u0 / UNITS) : nullptr, lane);
    }
}

// ---------------------------------------------------------------------------
// The same forward pass in fp32 (v_mfma_f32_16x16x4_f32), for the training rows of large fp32 batches (see
// forward_trunk_f32 for when; everything else in fp32 goes through sp::k_conv123_fwd).
//
// Units and lanes as above (strip of 4 output rows, 16 lanes x 5 pixels), but the strip stays in
// LDS as the uint8 it is (6,720 bytes per wave, no conversion while staging): the MFMA takes one
// reduction element per lane and instruction, lane group kg supplies kernel row 4yq + kg, and a
// lane's six 4-byte words of that row (pixels 4jj .. 4jj+3 of its run) serve, byte by byte, the
// kernel columns of all five pixels: word jj is columns 0-3 of pixel jj and columns 4-7 of pixel
// jj-1.  One v_cvt_f32_ubyte per byte, 24 per 40 MFMAs.
// A wave holds the weights of 16 output channels (64 registers): waves work in pairs, one channel
// half each.  The first wave of a pair can copy its strip to a gathered stack (the weight-gradient kernel
// of this path reads a materialised state).
// ---------------------------------------------------------------------------
constexpr int RAWSTRIP = 4 * SROWS * 84;   // bytes of one strip as uint8
struct FwdSegF {
    Src src;
    const float *w;     // [32][256] fp32, k = (c, ky, kx)
    const float *bias;  // [32]
    float *y;           // [n][400][32]
    int n;
    int first;
    uint8_t *stack;     // [n][5][84][84] or nullptr: frames 0-3 of the stack are written
};
struct FwdArgsF {
    FwdSegF seg[3];
    int nseg;
    int total;
    int draw;
    misc::SampleArgs samp;
};

__device__ __forceinline__ v4f mfma4(float a, float b, v4f c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ void conv1_fwd_units_f32(const FwdSegF &S, int u0, int u1, int hh, uint8_t *xs, const int *slots, int lane)
{
    const int n = lane & 15, kg = lane >> 4, oyl = n >> 2, q = n & 3;
    StripOff O;
#pragma unroll
    for (int i = 0; i < 7; ++i) {
        const int t = lane + 64 * i;
        O.off[i] = t < CHUNKS ? (t / (CHUNKS / 4)) * FR + (t % (CHUNKS / 4)) * 16 : 0;
    }
    const int gfirst = u0 / UNITS;
    auto slot_of = [&](int gq) { return slots ? slots[gq - gfirst] : sample_slot(S.src, gq); };
    StripRaw R;
    strip_load(R, S.src, gfirst, slot_of(gfirst), u0 % UNITS, lane, O);
    int slot_next = u0 + 1 < u1 ? slot_of((u0 + 1) / UNITS) : 0;
    // weights: wa[8 cy + 4 xh + b] = W[16hh + n][frame cy / 2, kernel row 4 (cy % 2) + kg][4 xh + b]
    float wa[64];
#pragma unroll
    for (int cy = 0; cy < 8; ++cy) {
        const float *p = S.w + (16 * hh + n) * 256 + (cy >> 1) * 64 + (4 * (cy & 1) + kg) * 8;
        const v4f lo = *reinterpret_cast<const v4f *>(p), hi = *reinterpret_cast<const v4f *>(p + 4);
        wa[8 * cy + 0] = lo.x; wa[8 * cy + 1] = lo.y; wa[8 * cy + 2] = lo.z; wa[8 * cy + 3] = lo.w;
        wa[8 * cy + 4] = hi.x; wa[8 * cy + 5] = hi.y; wa[8 * cy + 6] = hi.z; wa[8 * cy + 7] = hi.w;
    }
    const v4f bias = *reinterpret_cast<const v4f *>(S.bias + 16 * hh + 4 * kg);
    const uint8_t *px = xs + (4 * oyl + kg) * 84 + 20 * q;
    for (int u = u0; u < u1; ++u) {
        const int g = u / UNITS, strip = u % UNITS;
#pragma unroll
        for (int i = 0; i < 7; ++i) {
            const int t = lane + 64 * i;
            if (t < CHUNKS) {
                *reinterpret_cast<u32x4 *>(xs + t * 16) = R.raw[i];
                // rows 16s .. 16s+15 of the frames are this strip's own (the last strip owns all 20)
                const int fr = t / (CHUNKS / 4), off = (t % (CHUNKS / 4)) * 16;
                if (hh == 0 && S.stack && (off < 16 * 84 || strip == UNITS - 1))
                    *reinterpret_cast<u32x4 *>(S.stack + ((long)g * 5 + fr) * FR + strip * (16 * 84) + off) = R.raw[i];
            }
        }
        if (u + 1 < u1) {
            strip_load(R, S.src, (u + 1) / UNITS, slot_next, (u + 1) % UNITS, lane, O);
            if (u + 2 < u1) slot_next = slot_of((u + 2) / UNITS);
        }
        v4f acc[5];
#pragma unroll
        for (int j = 0; j < 5; ++j) acc[j] = v4f{0, 0, 0, 0};
#pragma unroll
        for (int cy = 0; cy < 8; ++cy) {   // frame cy / 2, kernel rows 4 (cy % 2) + kg
            const uint8_t *p = px + (cy >> 1) * (SROWS * 84) + (cy & 1) * (4 * 84);
            uint32_t d[6];
#pragma unroll
            for (int jj = 0; jj < 6; ++jj) d[jj] = *reinterpret_cast<const uint32_t *>(p + 4 * jj);
            float f[6][4];
#pragma unroll
            for (int jj = 0; jj < 6; ++jj) {
                f[jj][0] = (float)(d[jj] & 0xFFu);
                f[jj][1] = (float)((d[jj] >> 8) & 0xFFu);
                f[jj][2] = (float)((d[jj] >> 16) & 0xFFu);
                f[jj][3] = (float)(d[jj] >> 24);
            }
#pragma unroll
            for (int xh = 0; xh < 2; ++xh)
#pragma unroll
                for (int b = 0; b < 4; ++b)
#pragma unroll
                    for (int j = 0; j < 5; ++j) acc[j] = mfma4(wa[8 * cy + 4 * xh + b], f[j + xh][b], acc[j]);
        }
        float *y = S.y + ((long)g * 400 + 20 * (4 * strip + oyl) + 5 * q) * 32 + 16 * hh + 4 * kg;
        constexpr float sc = 1.0f / 255.0f;
#pragma unroll
        for (int j = 0; j < 5; ++j) {
            v4f o;
            o.x = fmaxf(acc[j].x * sc + bias.x, 0.f);
            o.y = fmaxf(acc[j].y * sc + bias.y, 0.f);
            o.z = fmaxf(acc[j].z * sc + bias.z, 0.f);
            o.w = fmaxf(acc[j].w * sc + bias.w, 0.f);
            *reinterpret_cast<v4f *>(y + j * 32) = o;
        }
    }
}

// The four waves of a workgroup are two pairs, each with a unit range of its own.
__global__ __launch_bounds__(256, 2) void k_conv1_fwd_f32(FwdArgsF A)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[4 * RAWSTRIP];
    __shared__ int slot_tab[4][MAX_DRAWS];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long np = (long)gridDim.x * 2, pid = (long)blockIdx.x * 2 + (wave >> 1), units = (long)A.total * UNITS;
    const int u0 = (int)(pid * units / np), u1 = (int)((pid + 1) * units / np);
    if (A.draw && u0 < u1) draw_slots(A.samp, A.seg[0].n, u0, u1, slot_tab[wave], lane, (wave & 1) == 0);
    for (int s = 0; s < A.nseg; ++s) {
        FwdSegF S = A.seg[0];
        if (s == 1) S = A.seg[1];
        if (s == 2) S = A.seg[2];
        const int lo = max(u0, UNITS * S.first) - UNITS * S.first;
        const int hi = min(u1, UNITS * (S.first + S.n)) - UNITS * S.first;
        if (lo < hi)
            conv1_fwd_units_f32(S, lo, hi, wave & 1, lds + wave * RAWSTRIP,
                                A.draw ? slot_tab[wave] + (S.first + lo / UNITS - u0 / UNITS) : nullptr, lane);
    }
}

struct WgradArgs {
    Src src;
    const bf16_t *dy;  // [B][400][32]
    float *part;       // [nsplit][32*256 + 32]
    int B;
    int nsplit;        // = gridDim.x; workgroup z sums samples z, z+nsplit, ...
};

// Row stride (elements) of the staged dY tile.  No padding: an 8-byte transpose read is served half a wave at a time, here
// four rows of 64 bytes, which lie in all 64 banks side by side (with 40 the fourth row met the first).
constexpr int LDY1 = 32;

// grid (nsplit, 2): a workgroup takes one channel pair y (frames 2y, 2y+1 = im2col columns
// 128y .. 128y+127), so a workgroup stages half a state and two workgroups fit one CU.
constexpr int WG1_LDS = 2 * FR + 400 * LDY1;   // LDS elements of a workgroup
// tile = 2 * split + channel pair
__device__ __forceinline__ void conv1_wgrad_block(const WgradArgs &A, int tile, bf16_t *lds)
{
    bf16_t *xin = lds, *dys = lds + 2 * FR;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;  // wave = block of 32 im2col columns
    const int li = lane & 31, h = lane >> 5, s16 = lane & 15, half = (lane >> 4) & 1;
    // the two channel pairs of one sample split run next to each other: same dY, same ring slots
    const int cp = tile & 1, split = tile >> 1;
    typedef __attribute__((address_space(3))) v4s *lds_v4s;

    // this lane's share of the transpose loads: reduction row offset s/4 (+4 for the second
    // load), columns 16*half + 4*(s%4) .. +3 of the wave's 32-column block
    const int rsub = 8 * h + (s16 >> 2);
    const int kc = 32 * wave + 16 * half + 4 * (s16 & 3);       // column within the pair: (c, p, q0)
    const int xoff = (kc >> 6) * FR + ((kc >> 3) & 7) * 84 + (kc & 7);
    const bf16_t *yp = dys + rsub * LDY1 + 16 * half + 4 * (s16 & 3);
    const bf16_t *xw = xin + xoff + 4 * rsub;   // the window of output pixel rsub

    v16f acc = {0}, accb = {0};
    v8bf ones;
#pragma unroll
    for (int e = 0; e < 8; ++e) ones[e] = (__bf16)1.0f;
    const bool do_bias = cp == 0 && wave == 0;

    Staged<256, 2> R;
    uint4 ry[7];
    auto load_sample = [&](int n, int slot_n) {
        stage_load<256, 2>(R, A.src, n, slot_n, 2 * cp, tid);
        const bf16_t *dyn = A.dy + (long)n * (400 * 32);
#pragma unroll
        for (int i = 0; i < 7; ++i) {
            const int t = tid + i * 256;
            if (t < 1600) ry[i] = ld8(dyn + (t >> 2) * 32 + (t & 3) * 8);
        }
    };
    // the ring slot of a sample is fetched one sample ahead of the frame loads that need it
    if (split < A.B) load_sample(split, sample_slot(A.src, split));
    int slot_next = split + A.nsplit < A.B ? sample_slot(A.src, split + A.nsplit) : 0;
    for (int n = split; n < A.B; n += A.nsplit) {
        __syncthreads();  // the previous sample's tiles are no longer read
        stage_store<256, 2>(xin, R, tid);
#pragma unroll
        for (int i = 0; i < 7; ++i) {
            const int t = tid + i * 256;
            if (t < 1600) *reinterpret_cast<uint4 *>(dys + (t >> 2) * LDY1 + (t & 3) * 8) = ry[i];
        }
        __syncthreads();
        if (n + A.nsplit < A.B) {
            load_sample(n + A.nsplit, slot_next);  // in flight during the MFMA loop
            if (n + 2 * A.nsplit < A.B) slot_next = sample_slot(A.src, n + 2 * A.nsplit);
        }
        // the operands of step t + 1 are requested before the matrix instruction of step t
        auto operands = [&](int t, v8bf &fa, v8bf &fb) {   // 16 output pixels per step
            fa = frag_tr(yp + 16 * t * LDY1, LDY1);
            // pixel m = 16t + rsub (and m + 4) of the 20-wide output: its window starts at input row 4(m/20),
            // column 4(m%20).  16t = 20q + r with q, r known at compile time, so the lane only has to see
            // whether r + rsub runs over into the next row: no division
            const int q = (16 * t) / 20, r = (16 * t) % 20;
            const bf16_t *x0 = xw + (336 * q + 4 * r) + (rsub >= 20 - r ? 256 : 0);
            const bf16_t *x1 = xw + (336 * q + 4 * r + 16) + (rsub + 4 >= 20 - r ? 256 : 0);
            v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)x0);
            v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)x1);
            typedef short v8s __attribute__((ext_vector_type(8)));
            v8s xb = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
            fb = __builtin_bit_cast(v8bf, xb);
        };
        v8bf fa, fb, fan, fbn;
        operands(0, fa, fb);
#pragma unroll
        for (int t = 0; t < 25; ++t) {
            fan = fa; fbn = fb;
            if (t + 1 < 25) operands(t + 1, fan, fbn);
            __builtin_amdgcn_sched_barrier(0);
            acc = mfma(fa, fb, acc);
            if (do_bias) accb = mfma(fa, ones, accb);
            __builtin_amdgcn_sched_barrier(0);
            fa = fan; fb = fbn;
        }
    }

    float *part = A.part + (long)split * (32 * 256 + 32);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int o = 8 * (r / 4) + 4 * h + (r % 4);
        part[o * 256 + 128 * cp + 32 * wave + li] = acc[r] * (1.0f / 255.0f);
        if (do_bias && li == 0) part[32 * 256 + o] = accb[r];
    }
}
__global__ __launch_bounds__(256) void k_conv1_wgrad(WgradArgs A)
{
    __shared__ __attribute__((aligned(16))) bf16_t lds[WG1_LDS];
    conv1_wgrad_block(A, net::tile_of_workgroup(), lds);
}
}  // namespace c1

// ===========================================================================
// conv2 and conv3 forward, one sample per workgroup at a time ("ps" = per sample).
//
// The generic kernels above cut the batch into row tiles and walk the reduction in stages with
// two barriers each; for these two layers a stage holds a handful of MFMAs, so the walk is a
// chain of latencies.  Here a persistent workgroup of four waves keeps its share of the WEIGHTS in
// registers (32 output channels x the whole reduction per wave), copies one sample's input
// (25.6 KB / 10.4 KB) into LDS with one barrier per sample, double-buffered, and every b-operand
// is a single 16-byte LDS read at base + immediate offset: no index arithmetic in the loop.
//
// v_mfma_f32_16x16x32_bf16, weights as the a-operand (row r = channel 32hh + 8(r/4) + 4cb + r%4 for
// the wave's channel half hh and channel block cb), output positions as the b-operand columns; one
// reduction step is one kernel tap x 32 input channels, lane group kg = lane/16 takes 8 of them.
// Wave (ph, hh) owns half of the position blocks and half of the channels; the result of lane
// (n, g = lane/16) is channels 32hh + 8g .. +7 of its positions: 16 bytes per store.
//
// LDS layout of a sample: see Shape.  conv2's reads meet no bank conflicts; conv3's, pixels in raster order 144 bytes
// apart, meet some (1.6 M conflict cycles in a launch of 1536 samples), and a layout without them changed
// nothing (42 us at 8192 samples either way: the launch is bound by its bytes).
// ===========================================================================
namespace ps {
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // a native vector: stays in registers across barriers

struct Seg {
    const bf16_t *x;    // [n][positions in][channels in]
    const bf16_t *w;    // [64][K] bf16, K = (tap, channel)
    const float *bias;  // [64]
    bf16_t *y;          // [n][positions out][64]
    int n;              // samples
    int first;          // index of the segment's first sample in the launch-wide sample list
};
struct Args {
    Seg seg[3];
    int nseg;
    int total;
};

// G: layer geometry.  IN_PIX pixels of IN_CH channels in, OUT x OUT positions out, TAPS x TAPS
// kernel with stride STRIDE, IN_W pixels per input row.
struct G2 { static constexpr int IN_PIX = 400, IN_CH = 32, IN_W = 20, OUT = 9, TAPS = 4, STRIDE = 2; };
struct G3 { static constexpr int IN_PIX = 81, IN_CH = 64, IN_W = 9, OUT = 7, TAPS = 3, STRIDE = 1; };

template <class G> struct Shape {
    static constexpr int PB = G::IN_CH * 2;                        // bytes per pixel
    // LDS layout of a sample.  64 channels: 144 bytes per pixel.  32 channels (stride 2): the even columns of a pixel row,
    // then the odd ones, 64 bytes each, and 16 bytes more per row.  A 16-byte read is served sixteen lanes at a time,
    // lanes 0-3, 12-15 and 20-27 of a half wave, then the others (measured): positions 0-3 and 12-15 of a tile with
    // piece kg, 4-11 with piece kg + 1.  Over two rows of eight positions these sixteen lie in the sixteen different
    // 16-byte columns of LDS this way; with positions in order and 144 bytes for two pixels every second read of conv2's
    // took twice as long.
    static constexpr bool SPLIT = G::IN_CH == 32;
    static constexpr int GB = 144;
    static constexpr int RB = (G::IN_W * 4 + 1) * 16;
    static constexpr int SAMPLE = SPLIT ? (G::IN_PIX / G::IN_W) * RB : G::IN_PIX * GB;
    static constexpr int K = G::TAPS * G::TAPS * G::IN_CH;
    static constexpr int STEPS = K / 32;                           // reduction steps: 16 / 18
    static constexpr int SPT = G::IN_CH / 32;                      // steps per tap: 1 / 2
    static constexpr int WROW = K * 2 + 16;                        // LDS bytes per weight row in transit
    static constexpr int NPOS = G::OUT * G::OUT;                   // 81 / 49
    static constexpr int NBLK = (NPOS + 31) / 32;                  // tiles of positions per wave: 3 / 2
    static constexpr int CHUNKS = G::IN_PIX * PB / 16;             // 16-byte pieces of a sample: 1600 / 648
    static constexpr int NLD = (CHUNKS + 255) / 256;               // pieces per thread: 7 / 3
    static constexpr int WCH = 32 * K * 2 / 16 / 256;              // weight pieces per thread and half: 8 / 9
    static constexpr int LDS = 32 * WROW > 2 * SAMPLE ? 32 * WROW : 2 * SAMPLE;
    // LDS byte offset of 16-byte piece c of pixel q
    static __device__ __forceinline__ uint32_t at(int q, int c)
    {
        if constexpr (SPLIT) {
            const int y = q / G::IN_W, x = q % G::IN_W;
            return y * RB + ((x & 1) * (2 * G::IN_W) + (x >> 1) * 4 + c) * 16;
        } else return q * GB + c * 16;
    }
    // Position n of tile t; where there is none, one that another lane has as well.  9 x 9: four tiles of two rows of eight,
    // then the last row and the last column of eight, then the corner.
    static __device__ __forceinline__ int position(int t, int n)
    {
        if constexpr (SPLIT) {
            const int r = n >> 3, x = n & 7;
            return t < 4 ? (2 * t + r) * G::OUT + x : t > 4 ? NPOS - 1 : r ? x * G::OUT + 8 : 8 * G::OUT + x;
        } else return min(16 * t + n, NPOS - 1);
    }
};

template <class G> struct Raw { u32x4 r[Shape<G>::NLD]; };
template <class G>
__device__ __forceinline__ void load_sample(Raw<G> &R, const bf16_t *x, int tid)
{
    using S = Shape<G>;
    const u32x4 *p = reinterpret_cast<const u32x4 *>(x);
#pragma unroll
    for (int i = 0; i < S::NLD; ++i) { const int t = tid + 256 * i; R.r[i] = p[t < S::CHUNKS ? t : S::CHUNKS - 1]; }
}
template <class G>
__device__ __forceinline__ void store_sample(uint8_t *buf, const Raw<G> &R, int tid)
{
    using S = Shape<G>;
    constexpr int CPP = S::PB / 16;   // pieces per pixel
#pragma unroll
    for (int i = 0; i < S::NLD; ++i) {
        const int t = tid + 256 * i;
        if (t < S::CHUNKS) *reinterpret_cast<u32x4 *>(buf + S::at(t / CPP, t % CPP)) = R.r[i];
    }
}

// Samples [g0, g1) of one segment.
template <class G>
__device__ __forceinline__ void run(const Seg &S, int g0, int g1, uint8_t *lds, int tid)
{
    using H = Shape<G>;
    const int lane = tid & 63, n = lane & 15, kg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), ph = wave & 1, hh = wave >> 1;
    Raw<G> R;
    load_sample<G>(R, S.x + (long)g0 * (G::IN_PIX * G::IN_CH), tid);   // on its way while the weights are fetched
    // The workgroup fetches each half of the weight matrix once, coalesced, into LDS; the two waves
    // that own the half pick their fragments from there.
    v8bf wa[H::STEPS][2];
    for (int half = 0; half < 2; ++half) {
        const u32x4 *src = reinterpret_cast<const u32x4 *>(S.w + half * 32 * H::K);
        sync_lds();   // LDS is free (the previous segment's last sample has been read)
#pragma unroll
        for (int i = 0; i < H::WCH; ++i) {
            const int c = tid + 256 * i;   // row c / (K/8), piece c % (K/8)
            *reinterpret_cast<u32x4 *>(lds + (c / (H::K / 8)) * H::WROW + (c % (H::K / 8)) * 16) = src[c];
        }
        sync_lds();
        if (hh == half) {
#pragma unroll
            for (int st = 0; st < H::STEPS; ++st)
#pragma unroll
                for (int cb = 0; cb < 2; ++cb) {
                    const int chl = 8 * (n >> 2) + 4 * cb + (n & 3);
                    wa[st][cb] = __builtin_bit_cast(v8bf, *reinterpret_cast<const uint4 *>(lds + chl * H::WROW + st * 64 + kg * 16));
                }
        }
    }
    const v4f b0 = *reinterpret_cast<const v4f *>(S.bias + 32 * hh + 8 * kg);
    const v4f b1 = *reinterpret_cast<const v4f *>(S.bias + 32 * hh + 8 * kg + 4);
    // this lane's positions and the LDS offset of their first tap
    uint32_t base[H::NBLK];
    int pos[H::NBLK];
#pragma unroll
    for (int b = 0; b < H::NBLK; ++b) {
        const int p = pos[b] = H::position(H::NBLK * ph + b, n);
        base[b] = H::at(G::STRIDE * (G::IN_W * (p / G::OUT) + (p % G::OUT)), kg);
    }
    sync_lds();   // the weight rows have been read
    store_sample<G>(lds + (g0 & 1) * H::SAMPLE, R, tid);
    load_sample<G>(R, S.x + (long)min(g0 + 1, g1 - 1) * (G::IN_PIX * G::IN_CH), tid);
    for (int g = g0; g < g1; ++g) {
        sync_lds();   // buffer g&1 is complete; buffer (g+1)&1 is no longer read
        if (g + 1 < g1) store_sample<G>(lds + ((g + 1) & 1) * H::SAMPLE, R, tid);
        // the last loads repeat the last sample: redundant, never out of range
        load_sample<G>(R, S.x + (long)min(g + 2, g1 - 1) * (G::IN_PIX * G::IN_CH), tid);
        const uint8_t *buf = lds + (g & 1) * H::SAMPLE;
        v4f acc[H::NBLK][2];
#pragma unroll
        for (int b = 0; b < H::NBLK; ++b) acc[b][0] = acc[b][1] = v4f{0, 0, 0, 0};
        // byte offset of reduction step st: pixel (ky, kx) further, second half of its channels for odd
        // steps of the 64-channel layer
        auto step_off = [](int st) {
            const int tap = st / H::SPT, ky = tap / G::TAPS, kx = tap % G::TAPS;
            return (int)H::at(G::IN_W * ky + kx, 0) + (st % H::SPT) * 64;
        };
        // the operands of step st+1 are requested before the matrix instructions of step st
        uint4 cur[H::NBLK], nxt[H::NBLK];
#pragma unroll
        for (int b = 0; b < H::NBLK; ++b) cur[b] = *reinterpret_cast<const uint4 *>(buf + base[b] + step_off(0));
#pragma unroll
        for (int st = 0; st < H::STEPS; ++st) {
            if (st + 1 < H::STEPS) {
#pragma unroll
                for (int b = 0; b < H::NBLK; ++b) nxt[b] = *reinterpret_cast<const uint4 *>(buf + base[b] + step_off(st + 1));
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int b = 0; b < H::NBLK; ++b) {
                const v8bf bb = __builtin_bit_cast(v8bf, cur[b]);
                acc[b][0] = mfma16(wa[st][0], bb, acc[b][0]);
                acc[b][1] = mfma16(wa[st][1], bb, acc[b][1]);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int b = 0; b < H::NBLK; ++b) cur[b] = nxt[b];
        }
        bf16_t *y = S.y + (long)g * (H::NPOS * 64) + 32 * hh + 8 * kg;
#pragma unroll
        for (int b = 0; b < H::NBLK; ++b) {
            // unconditional: a lane without a position of its own has computed another lane's once more (from the same
            // operands) and stores the same bits there.  Without a branch
            // the compiler can count these stores, and the wait for the next sample's pixels, requested
            // before them, does not wait for their acknowledgement as well.
            const v4f a0 = acc[b][0], a1 = acc[b][1];
            const uint2 lo = pack4(fmaxf(a0.x + b0.x, 0.f), fmaxf(a0.y + b0.y, 0.f), fmaxf(a0.z + b0.z, 0.f), fmaxf(a0.w + b0.w, 0.f));
            const uint2 hi = pack4(fmaxf(a1.x + b1.x, 0.f), fmaxf(a1.y + b1.y, 0.f), fmaxf(a1.z + b1.z, 0.f), fmaxf(a1.w + b1.w, 0.f));
            *reinterpret_cast<uint4 *>(y + pos[b] * 64) = uint4{lo.x, lo.y, hi.x, hi.y};
        }
    }
}

// Workgroup b owns samples [b*total/G, (b+1)*total/G) of the launch-wide list; two workgroups fit one CU.
template <class G>
__global__ __launch_bounds__(256, 2) void k_conv_fwd_ps(Args A)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[Shape<G>::LDS];
    const int g0 = (int)((long)blockIdx.x * A.total / gridDim.x);
    const int g1 = (int)((long)(blockIdx.x + 1) * A.total / gridDim.x);
    for (int s = 0; s < A.nseg; ++s) {
        Seg S = A.seg[0];
        if (s == 1) S = A.seg[1];
        if (s == 2) S = A.seg[2];
        const int lo = max(g0, S.first) - S.first, hi = min(g1, S.first + S.n) - S.first;
        if (lo < hi) run<G>(S, lo, hi, lds, threadIdx.x);
    }
}
}  // namespace ps

// ===========================================================================
// conv1, conv2 and conv3 forward in ONE launch for many samples: of what lies between the pixels and conv3's output,
// only what a later kernel reads leaves the CU (the backward pass reads conv1's and conv2's of the training rows).
//
// A workgroup of eight waves owns a run of samples of one segment, and the layers are a pipeline of waves.  Waves 0-3 are
// PRODUCERS: each computes conv1 strips as c1::k_conv1_fwd does (the strip's pixels in LDS of its own, as
// bytes, and widened between the matrix instructions of the frame before; weights in registers, next
// strip's pixels in flight) and writes the 80 x 32 result into the sample's place in a ring of four LDS
// images, in the layout ps::run reads.  Waves 4 and 5 hold conv2's weights in registers, a channel half each,
// and compute the conv2 output of each sample out of the ring into a ring of two images; waves 6 and 7 hold conv3's
// and finish the sample out of those.  The waves hand over by counts in LDS: a consumer waits for the five strips (the two
// halves) of its sample, whoever writes for the two consumers of the sample that had the image before.
// What bounds it is the issue of the SIMDs: 268 matrix instructions of 16 cycles and about 600 vector instructions of 4
// per SIMD and sample, which hardly overlap.  conv2's waves have a third more matrix instructions per sample than conv3's
// (192, 144), so the producers beside them (a wave sits on SIMD number % 4) take fewer strips: first_strip, next_strip (three of
// fourteen; one of six 177 us for 8192 observations, two of ten or four of eighteen the same 173, seven of thirty 175).
// Against conv1 + conv2 in a launch of four producers and four conv2 waves and conv3 in one of its own, which wrote conv2's output and
// read it back: 8192 observations 189.1 -> 170.1 us per call, a step of 512 136.1 -> 130.3, the fleet's iteration (acting on
// 2048, a step of 256) 188.8 -> 174.4; the same bits.  Consumers at a higher wave priority: 182 us for 8192.
//
// Replay mode: the workgroup draws its samples first (Eq.10 walk, two draws per wave and walk, all
// eight waves); the workgroups of segment 0 publish the draws.  The consumers request their weights behind the slot table,
// while the producers compute the first strips: ahead of it those 136 KB per workgroup queue in front of the walk and of the
// first pixels (a given batch of 128 69.5 -> 70.9 us, acting on 1024 38.9 -> 40.5, steps that draw 118.3 against 119.3 at 512,
// 76.4 against 75.5 at 128, 181.0 against 180.1 at 1000).  Otherwise the slots (ring mode) are copied into LDS from where a sampling kernel left them.
// Workgroups are dealt out per segment, so none pays the start-up twice.
// ===========================================================================
namespace pipe {
using c1::Src;
using c1::STRIP;
using c1::UNITS;
using S2 = ps::Shape<ps::G2>;
using S3 = ps::Shape<ps::G3>;
using ps::u32x4;

struct Seg {
    Src src;
    const bf16_t *w1;   // [32][256]
    const float *b1;    // [32]
    bf16_t *y1;         // [n][400][32], or nullptr: conv1's output is not kept
    const bf16_t *w2;   // [64][512]
    const float *b2;    // [64]
    bf16_t *y2;         // [n][81][64], or nullptr
    const bf16_t *w3;   // [64][576]
    const float *b3;    // [64]
    bf16_t *y3;         // [n][49][64]
    int n;              // samples
};
struct Args {
    Seg seg[3];
    int nseg;
    int draw;           // replay mode: sample g of every segment is draw g of `samp`; segment 0 publishes
    misc::SampleArgs samp;
};

constexpr int NRING = 4, NRING2 = 2;                        // conv1's and conv2's images in LDS
constexpr int MAX_PER_WG = 32;                              // samples one workgroup may own (slot table)
constexpr int PRODUCERS = 4, CONSUMERS = 2;                 // waves of conv1; of conv2, and of conv3
constexpr int STRIPS_B = PRODUCERS * STRIP;                 // 26,880 bytes: one strip per producer wave, pixels as bytes
constexpr int RING_B = NRING * S2::SAMPLE;                  // 103,680 bytes
constexpr int RING2_B = NRING2 * S3::SAMPLE;                // 23,328 bytes
constexpr int COUNTS = 4;                                   // per sample: strips, reads, halves, reads of conv2's image
constexpr int LDS_BYTES = STRIPS_B + RING_B + RING2_B + MAX_PER_WG * 8 + 16 + COUNTS * MAX_PER_WG * 4;   // + slot table, leaf values, total, counts
static_assert(STRIP % 16 == 0 && S3::SAMPLE % 16 == 0 && LDS_BYTES <= 160 * 1024, "LDS layout");
// The hand-over, as functions that the kernel and the host-side check (schedule_is_safe, behind
// dqn_selftest_fused_conv_schedule) both call.  The strips of a run are dealt out in order, PERIOD at a time: waves 2, 3, 0, 1,
// 2, 3 and so on, so that 2 and 3 get four of fourteen and 0 and 1 three.  A producer counts its strips in per sample, a
// consumer the samples it has read, a conv2 wave also those it has stored.
constexpr int PERIOD = 14;
static_assert(PERIOD % PRODUCERS == 2, "waves 2 and 3 first and last");
__host__ __device__ constexpr int first_strip(int w) { return (w + 2) % PRODUCERS; }
__host__ __device__ constexpr int next_strip(int u)
{
    const int at = u % PERIOD;
    return u + (at + PRODUCERS < PERIOD ? PRODUCERS : at < PERIOD - 2 ? PRODUCERS + 2 : 2);
}
__host__ __device__ constexpr int sample_of_strip(int u) { return u / UNITS; }
__host__ __device__ constexpr int image_of_sample(int k) { return k % NRING; }
__host__ __device__ constexpr int image2_of_sample(int k) { return k % NRING2; }
// may sample k be read, with `strips` of its strips (`halves` of its channel halves) counted in?
__host__ __device__ constexpr bool complete(int strips) { return strips == UNITS; }
__host__ __device__ constexpr bool complete2(int halves) { return halves == CONSUMERS; }
// may sample k's image be written, with `reads` consumers done with the sample that had it before?
__host__ __device__ constexpr bool image_free(int k, int reads) { return k < NRING || reads == CONSUMERS; }
__host__ __device__ constexpr bool image2_free(int k, int reads) { return k < NRING2 || reads == CONSUMERS; }

// The host-side check of one hand-over: a search of all states that its waves can reach, in whatever order they take
// their steps.  A state is how far each wave has come, twice the steps it is through with and one more while it is in one: a
// writer that stores has passed its wait and has not counted its share in yet, and so a reader of a sample.
// What a wait lets through is held against the positions themselves: a sample is complete when it is read, nothing is
// stored where a sample lies that some reader has still to read, none of a later sample lies where one is read; and no
// state but the last leaves every wave waiting.  of[w]: the samples of writer w's steps, in order; a sample is `parts` steps.
// Returns 0 if safe, else a code naming the failure.  (Readers are alike: their positions stay sorted, the last of equals moves.)
template <class Complete, class Image, class Free>
int handover_is_safe(int ns, int parts, const std::vector<std::vector<int>> &of, int ring, Complete is_complete, Image image, Free is_free)
{
    constexpr int BITS = 8;
    const int W = (int)of.size(), WAVES = W + CONSUMERS;
    int at[64 / BITS];
    std::vector<std::vector<uint8_t>> through(W);   // [n][k]: steps for sample k among a writer's first n
    std::vector<int> steps(WAVES, ns);
    for (int w = 0; w < W; ++w) {
        steps[w] = (int)of[w].size();
        through[w].assign((steps[w] + 1) * ns, 0);
        for (int n = 1; n <= steps[w]; ++n) {
            for (int k = 0; k < ns; ++k) through[w][n * ns + k] = through[w][(n - 1) * ns + k];
            ++through[w][n * ns + of[w][n - 1]];
        }
    }
    for (int w = 0; w < WAVES; ++w)
        if (2 * steps[w] >= 1 << BITS || WAVES * BITS > 64) return 4;
    auto stored = [&](int k) {   // counted in
        int n = 0;
        for (int w = 0; w < W; ++w) n += through[w][at[w] / 2 * ns + k];
        return n;
    };
    auto reads = [&](int k) {
        int n = 0;
        for (int w = W; w < WAVES; ++w) n += at[w] / 2 > k;
        return n;
    };
    std::vector<uint64_t> now{0}, next, sum;   // each in ascending order
    std::vector<std::vector<uint64_t>> by(WAVES);
    while (!now.empty()) {
        for (auto &b : by) b.clear();
        for (const uint64_t v : now) {
            bool moved = false, done = true;
            int begun = -1;   // the latest sample of which something has been stored or is being stored
            for (int w = 0; w < WAVES; ++w) {
                at[w] = (int)(v >> (BITS * w)) & ((1 << BITS) - 1);
                done &= at[w] == 2 * steps[w];
                if (w < W && at[w]) begun = std::max(begun, of[w][(at[w] + 1) / 2 - 1]);
            }
            for (int w = 0; w < WAVES; ++w) {
                if (at[w] == 2 * steps[w]) continue;
                const int i = at[w] / 2, k = w < W ? of[w][i] : i;
                if (!(at[w] & 1)) {   // its wait
                    if (w < W) {
                        if (!is_free(k, k < ring ? 0 : reads(k - ring))) continue;
                        for (int j = at[W] / 2; j < k; ++j)   // samples that the last reader is not through with
                            if (image(j) == image(k)) return 3;
                    } else {
                        if (!is_complete(stored(k))) continue;
                        if (stored(k) != parts) return 2;
                        for (int j = k + 1; j <= begun; ++j)
                            if (image(j) == image(k)) return 2;
                    }
                }
                if (w < W || w == WAVES - 1 || at[w + 1] > at[w]) by[w].push_back(v + (1ull << (BITS * w)));
                moved = true;
            }
            if (!moved && !done) return 5;
        }
        next.clear();
        for (const auto &b : by) {
            sum.clear();
            std::set_union(next.begin(), next.end(), b.begin(), b.end(), std::back_inserter(sum));
            next.swap(sum);
        }
        now.swap(next);
    }
    return 0;
}
// A run of ns samples: the two hand-overs one by one.  A conv2 wave is a reader in the first and a writer in the second; either
// search covers its steps at any pace, so also its waits in the other; and its wait for an image of the second ends without
// any step of the first (conv3's waves wait for nothing but halves that conv2's have begun).  Every strip has one owner.
inline int schedule_is_safe(int ns)
{
    if (ns < 1 || ns > MAX_PER_WG) return 1;
    std::vector<std::vector<int>> strips(PRODUCERS), halves(CONSUMERS);
    std::vector<int> owners(UNITS * ns, 0);
    for (int w = 0; w < PRODUCERS; ++w)
        for (int u = first_strip(w); u < UNITS * ns; u = next_strip(u)) {
            strips[w].push_back(sample_of_strip(u));
            ++owners[u];
        }
    for (const int n : owners)
        if (n != 1) return 6;
    for (auto &h : halves)
        for (int k = 0; k < ns; ++k) h.push_back(k);
    if (const int e = handover_is_safe(ns, UNITS, strips, NRING, complete, image_of_sample, image_free)) return e;
    const int e = handover_is_safe(ns, CONSUMERS, halves, NRING2, complete2, image2_of_sample, image2_free);
    return e ? 10 + e : 0;
}

// The counts of a sample, in LDS: every operation of a wave is carried out there in the order in which it was issued, so
// a count that has been seen stands behind the stores (or reads) of the wave that raised it.
struct Counts { int *strips, *reads, *halves, *reads2; };
__device__ __forceinline__ int count_of(int *p)
{
    return __builtin_amdgcn_readfirstlane(__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
}
__device__ __forceinline__ void count_in(int *p, int lane)
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    if (lane == 0) __hip_atomic_fetch_add(p, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
template <class Ready> __device__ __forceinline__ void await(Ready ready)
{
    while (!ready()) __builtin_amdgcn_s_sleep(1);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A strip's pixels as they lie in memory, a frame's 105 pieces of 16 bytes in two loads, the second one's last 23 lanes
// with the frame's last piece: one scalar address per frame, wherever the frames of a sample are
struct Pixels { u32x4 r[8]; };
constexpr int PIECES = c1::SROWS * 84 / 16;
__device__ __forceinline__ void load_strip(Pixels &R, const Src &S, int g, int slot, int strip, int lane)
{
    const uint32_t o0 = lane * 16, o1 = min(lane + 64, PIECES - 1) * 16;
    const uint8_t *x = S.x + strip * (16 * 84);
    int i = 0, rb = 0;   // the slot, its sub-ring (slots are below 2^30)
    if (S.idx) {
        i = __builtin_amdgcn_readfirstlane(slot);
        i = i < 0 ? 0 : i >= (int)S.cap ? (int)S.cap - 1 : i;
        rb = (int)c1::sub_ring_base(S, i);
        i += S.shift - 3 - rb;
    } else x += (long)g * S.xs;
#pragma unroll
    for (int f = 0; f < 4; ++f) {
        int fr = i + f;   // one wrap at most (see c1::frame_ptr)
        if (S.idx) {
            if (fr < 0) fr += S.sub;
            if (fr >= S.sub) fr -= S.sub;
            fr += rb;
        }
        const uint8_t *p = x + (long)(uint32_t)fr * c1::FR;
        R.r[2 * f] = *reinterpret_cast<const u32x4 *>(p + o0);
        R.r[2 * f + 1] = *reinterpret_cast<const u32x4 *>(p + o1);
    }
}
__device__ __forceinline__ void store_strip(uint8_t *xs, const Pixels &R, int lane)
{
    const uint32_t o0 = lane * 16, o1 = min(lane + 64, PIECES - 1) * 16;
#pragma unroll
    for (int f = 0; f < 4; ++f) {
        *reinterpret_cast<u32x4 *>(xs + f * (PIECES * 16) + o0) = R.r[2 * f];
        *reinterpret_cast<u32x4 *>(xs + f * (PIECES * 16) + o1) = R.r[2 * f + 1];
    }
}

// bias, ReLU, bf16 of a position's eight channels
__device__ __forceinline__ uint4 finished(v4f a0, v4f a1, v4f b0, v4f b1)
{
    const uint2 lo = pack4(fmaxf(a0.x + b0.x, 0.f), fmaxf(a0.y + b0.y, 0.f), fmaxf(a0.z + b0.z, 0.f), fmaxf(a0.w + b0.w, 0.f));
    const uint2 hi = pack4(fmaxf(a1.x + b1.x, 0.f), fmaxf(a1.y + b1.y, 0.f), fmaxf(a1.z + b1.z, 0.f), fmaxf(a1.w + b1.w, 0.f));
    return uint4{lo.x, lo.y, hi.x, hi.y};
}
// A consumer wave's weights of channel half hh, straight into a-operand registers: row 8(n/4) + 4cb + n%4 of the half,
// reduction elements 32st + 8kg .. +7
template <class S> __device__ __forceinline__ void load_weights(v8bf (&wa)[S::STEPS][2], const bf16_t *w, int lane, int hh)
{
    const int n = lane & 15, kg = lane >> 4;
#pragma unroll
    for (int st = 0; st < S::STEPS; ++st)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            const int chl = 8 * (n >> 2) + 4 * cb + (n & 3);
            wa[st][cb] = __builtin_bit_cast(v8bf, *reinterpret_cast<const uint4 *>(w + (32 * hh + chl) * S::K + st * 32 + kg * 8));
        }
}
// The sums of NB tiles of 16 positions, this lane's operand of tile b and step st at at(b, st); the operands are requested two
// steps ahead of their matrix instructions
template <class S, int NB, class At>
__device__ __forceinline__ void multiply(v4f (&acc)[NB][2], const v8bf (&wa)[S::STEPS][2], At at)
{
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b][0] = acc[b][1] = v4f{0, 0, 0, 0};
    uint4 q[3][NB];
    auto request = [&](int st) {
#pragma unroll
        for (int b = 0; b < NB; ++b) q[st % 3][b] = *reinterpret_cast<const uint4 *>(at(b, st));
    };
    request(0);
    request(1);
#pragma unroll
    for (int st = 0; st < S::STEPS; ++st) {
        if (st + 2 < S::STEPS) request(st + 2);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const v8bf bb = __builtin_bit_cast(v8bf, q[st % 3][b]);
            acc[b][0] = mfma16(wa[st][0], bb, acc[b][0]);
            acc[b][1] = mfma16(wa[st][1], bb, acc[b][1]);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) asm volatile("" : "+v"(acc[b][0]), "+v"(acc[b][1]));   // (half of the products would sink below the caller's wait)
}

// samples [lo, hi) of segment S: conv2, channel half hh, three tiles of positions and then the other three (all six at once
// would take the registers of the weights)
__device__ __forceinline__ void run_conv2(const Seg &S, int lo, int hi, const uint8_t *ring, uint8_t *ring2, const v8bf (&wa)[16][2],
                                          const Counts &C, int lane, int hh)
{
    const int n = lane & 15, kg = lane >> 4;
    const int ns = hi - lo;
    const v4f b0 = *reinterpret_cast<const v4f *>(S.b2 + 32 * hh + 8 * kg);
    const v4f b1 = *reinterpret_cast<const v4f *>(S.b2 + 32 * hh + 8 * kg + 4);
    // the first four tiles lie two rows of positions apart, the others anywhere (Shape::position)
    uint32_t base[6];
    int pos[6];
#pragma unroll
    for (int t = 0; t < 6; ++t) {
        pos[t] = t > 0 && t < 4 ? pos[0] + 18 * t : S2::position(t, n);
        base[t] = t > 0 && t < 4 ? base[0] + t * 4 * S2::RB : S2::at(2 * (20 * (pos[t] / 9) + pos[t] % 9), kg);
    }
    for (int k = 0; k < ns; ++k) {
        await([&] { return complete(count_of(C.strips + k)); });
        const uint8_t *buf = ring + image_of_sample(k) * S2::SAMPLE;
        uint8_t *img = ring2 + image2_of_sample(k) * S3::SAMPLE + 64 * hh + 16 * kg;
        bf16_t *y = S.y2 ? S.y2 + (long)(lo + k) * (81 * 64) + 32 * hh + 8 * kg : nullptr;   // uniform
#pragma unroll
        for (int t0 = 0; t0 < 6; t0 += 3) {
            v4f acc[3][2];
            multiply<S2, 3>(acc, wa, [&](int b, int st) { return buf + base[t0 + b] + S2::at(20 * (st >> 2) + (st & 3), 0); });
            if (t0 == 0) await([&] { return image2_free(k, k < NRING2 ? 0 : count_of(C.reads2 + k - NRING2)); });
            else count_in(C.reads + k, lane);
#pragma unroll
            for (int b = 0; b < 3; ++b) {   // (lanes that share a position store the same bits)
                const uint4 v = finished(acc[b][0], acc[b][1], b0, b1);
                *reinterpret_cast<uint4 *>(img + S3::at(pos[t0 + b], 0)) = v;
                if (y) *reinterpret_cast<uint4 *>(y + pos[t0 + b] * 64) = v;
            }
        }
        count_in(C.halves + k, lane);
    }
}

// ... conv3, two tiles and two tiles
__device__ __forceinline__ void run_conv3(const Seg &S, int lo, int hi, const uint8_t *ring2, const v8bf (&wa)[18][2],
                                          const Counts &C, int lane, int hh)
{
    const int n = lane & 15, kg = lane >> 4;
    const int ns = hi - lo;
    const v4f b0 = *reinterpret_cast<const v4f *>(S.b3 + 32 * hh + 8 * kg);
    const v4f b1 = *reinterpret_cast<const v4f *>(S.b3 + 32 * hh + 8 * kg + 4);
    uint32_t base[4];
    int pos[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const int p = pos[b] = S3::position(b, n);
        base[b] = S3::at(9 * (p / 7) + (p % 7), kg);
    }
    for (int k = 0; k < ns; ++k) {
        await([&] { return complete2(count_of(C.halves + k)); });
        const uint8_t *buf = ring2 + image2_of_sample(k) * S3::SAMPLE;
        bf16_t *y = S.y3 + (long)(lo + k) * (49 * 64) + 32 * hh + 8 * kg;
#pragma unroll
        for (int t = 0; t < 4; t += 2) {
            v4f acc[2][2];
            multiply<S3, 2>(acc, wa, [&](int b, int st) { return buf + base[t + b] + S3::at(9 * (st / 6) + (st >> 1) % 3, 0) + (st & 1) * 64; });
            if (t) count_in(C.reads2 + k, lane);
#pragma unroll
            for (int b = 0; b < 2; ++b) *reinterpret_cast<uint4 *>(y + pos[t + b] * 64) = finished(acc[b][0], acc[b][1], b0, b1);
        }
    }
}

// samples [lo, hi) of segment S, producer wave w: its strips of the run's list.
// R holds the pixels of the first (requested by the caller); slots: the run's ring slots (ring mode).
__device__ __forceinline__ void run_producer(const Seg &S, int lo, int hi, uint8_t *xs, uint8_t *ring, const int *slots,
                                             const Counts &C, Pixels &R, int lane, int w)
{
    const int n = lane & 15, kg = lane >> 4, oyl = n >> 2, q = n & 3;
    const int nstrips = UNITS * (hi - lo);
    // where this lane's pixels 5 q + j of a strip's image row go, two columns apart for every second j
    const int even = S2::at(20 * oyl + 5 * q, kg), odd = S2::at(20 * oyl + 5 * q + 1, kg);
    const uint32_t yoff = ((20 * oyl + 5 * q) * 32 + 8 * kg) * 2;   // ... and in memory
    v8bf wa[8][2];   // [2c + xh][channel half], as in c1::conv1_fwd_units
#pragma unroll
    for (int st = 0; st < 8; ++st)
#pragma unroll
        for (int h2 = 0; h2 < 2; ++h2) {
            const int ch = 8 * (n >> 2) + 4 * h2 + (n & 3);
            const bf16_t *p = S.w1 + ch * 256 + (st >> 1) * 64 + (2 * kg) * 8 + 4 * (st & 1);
            const uint2 l2 = *reinterpret_cast<const uint2 *>(p), hi2 = *reinterpret_cast<const uint2 *>(p + 8);
            wa[st][h2] = __builtin_bit_cast(v8bf, uint4{l2.x, l2.y, hi2.x, hi2.y});
        }
    const v4f b0 = *reinterpret_cast<const v4f *>(S.b1 + 8 * kg), b1 = *reinterpret_cast<const v4f *>(S.b1 + 8 * kg + 4);
    const uint32_t px = (uint32_t)(uintptr_t)(xs + (4 * oyl + 2 * kg) * 84 + 20 * q);
    auto slot_of = [&](int u) { return S.src.idx && u < nstrips ? slots[sample_of_strip(u)] : 0; };
    int slot = slot_of(next_strip(first_strip(w)));
    for (int u = first_strip(w), un; u < nstrips; u = un) {
        const int k = sample_of_strip(u), strip = u % UNITS;
        store_strip(xs, R, lane);            // (LDS operations of one wave complete in order)
        asm volatile("" ::: "memory");       // ... and the reads below are not ordered behind stores by the compiler
        un = next_strip(u);
        if (un < nstrips) load_strip(R, S.src, lo + un / UNITS, slot, un % UNITS, lane);
        slot = slot_of(next_strip(un));
        // a frame's six quads of pixels (see c1::conv1_fwd_units), two rows each, requested two frames ahead
        typedef uint32_t v2u __attribute__((ext_vector_type(2)));
        struct Bytes { v2u q[6]; };
        struct Quads { uint4 q[6]; };
        auto request = [&](int c) {
            const uint32_t addr = px + c * (c1::SROWS * 84);
            Bytes Q;
#define PIPE_RD2(JJ) asm volatile("ds_read2_b32 %0, %1 offset0:%2 offset1:%3" : "=v"(Q.q[JJ]) : "v"(addr), "n"(JJ), "n"(JJ + 21));
            PIPE_RD2(0) PIPE_RD2(1) PIPE_RD2(2) PIPE_RD2(3) PIPE_RD2(4) PIPE_RD2(5)
#undef PIPE_RD2
            return Q;
        };
        auto arrived = [&](Bytes &Q, bool more) {   // more: the six reads of another frame behind these
            if (more) asm volatile("s_waitcnt lgkmcnt(6)" : "+v"(Q.q[0]), "+v"(Q.q[1]), "+v"(Q.q[2]), "+v"(Q.q[3]), "+v"(Q.q[4]), "+v"(Q.q[5])::"memory");
            else asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(Q.q[0]), "+v"(Q.q[1]), "+v"(Q.q[2]), "+v"(Q.q[3]), "+v"(Q.q[4]), "+v"(Q.q[5])::"memory");
        };
        auto widened = [&](const Bytes &Q) {
            Quads W;
#pragma unroll
            for (int j = 0; j < 6; ++j) W.q[j] = cvt8_u8(Q.q[j].x, Q.q[j].y);
            return W;
        };
        v4f acc[5][2];
#pragma unroll
        for (int j = 0; j < 5; ++j) acc[j][0] = acc[j][1] = v4f{0, 0, 0, 0};
        Bytes r0 = request(0), r1 = request(1);
        arrived(r0, true);
        Quads cur = widened(r0), nxt;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            Bytes &rn = c & 1 ? r0 : r1;   // frame c + 1
            if (c < 2) (c & 1 ? r1 : r0) = request(c + 2);
            if (c < 3) arrived(rn, c < 2);
            __builtin_amdgcn_sched_barrier(0);
            if (c < 3) nxt = widened(rn);   // between the matrix instructions
#pragma unroll
            for (int xh = 0; xh < 2; ++xh)
#pragma unroll
                for (int j = 0; j < 5; ++j) {
                    const v8bf b = __builtin_bit_cast(v8bf, cur.q[j + xh]);
                    acc[j][0] = mfma16(wa[2 * c + xh][0], b, acc[j][0]);
                    acc[j][1] = mfma16(wa[2 * c + xh][1], b, acc[j][1]);
                }
            if (c < 3) {
#pragma unroll
                for (int g = 0; g < 20; ++g) {
                    __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x2, 4, 0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            cur = nxt;
        }
#pragma unroll
        for (int j = 0; j < 5; ++j) asm volatile("" : "+v"(acc[j][0]), "+v"(acc[j][1]));   // (half of the products would sink below the wait)
        await([&] { return image_free(k, k < NRING ? 0 : count_of(C.reads + k - NRING)); });
        // bias, 1/255, ReLU, bf16: into the sample's image in the ring and, where kept, to memory
        uint8_t *img = ring + image_of_sample(k) * S2::SAMPLE + strip * (4 * S2::RB);
        uint8_t *yb = S.y1 ? reinterpret_cast<uint8_t *>(S.y1) + ((long)(lo + k) * 400 + 80 * strip) * 64 : nullptr;   // uniform
        constexpr float sc = 1.0f / 255.0f;
#pragma unroll
        for (int j = 0; j < 5; ++j) {
            const v4f a0 = acc[j][0], a1 = acc[j][1];
            const uint2 l2 = pack4(fmaxf(a0.x * sc + b0.x, 0.f), fmaxf(a0.y * sc + b0.y, 0.f),
                                   fmaxf(a0.z * sc + b0.z, 0.f), fmaxf(a0.w * sc + b0.w, 0.f));
            const uint2 h2 = pack4(fmaxf(a1.x * sc + b1.x, 0.f), fmaxf(a1.y * sc + b1.y, 0.f),
                                   fmaxf(a1.z * sc + b1.z, 0.f), fmaxf(a1.w * sc + b1.w, 0.f));
            const uint4 v = uint4{l2.x, l2.y, h2.x, h2.y};
            *reinterpret_cast<uint4 *>(img + (j & 1 ? odd : even) + (j >> 1) * 64) = v;
            if (yb) *reinterpret_cast<uint4 *>(yb + yoff + j * 64) = v;
        }
        count_in(C.strips + k, lane);
    }
}

// Segment t owns workgroups [G t / nseg, G (t+1) / nseg); each of them an even share of its samples.
// The host sizes the grid so that no share exceeds MAX_PER_WG.  Dynamic LDS: LDS_BYTES.
__global__ __launch_bounds__(512) void k_conv_fwd_pipe(Args A)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    int s = 0, w0 = 0, w1 = 1;
    for (int t = 0; t < A.nseg; ++t) {
        const int a = (int)((long)gridDim.x * t / A.nseg), b = (int)((long)gridDim.x * (t + 1) / A.nseg);
        if ((int)blockIdx.x >= a && (int)blockIdx.x < b) { s = t; w0 = a; w1 = b; }
    }
    Seg S = A.seg[0];
    if (s == 1) S = A.seg[1];
    if (s == 2) S = A.seg[2];
    const int lo = (int)((long)((int)blockIdx.x - w0) * S.n / (w1 - w0));
    const int hi = (int)((long)((int)blockIdx.x - w0 + 1) * S.n / (w1 - w0));
    if (lo >= hi) return;   // the whole workgroup
    const int ns = hi - lo;
    uint8_t *ring = lds + STRIPS_B, *ring2 = ring + RING_B;
    int *slots = reinterpret_cast<int *>(ring2 + RING2_B);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    float *leafv = reinterpret_cast<float *>(slots + MAX_PER_WG);   // [MAX_PER_WG] leaf values, then the total
    int *const counts = reinterpret_cast<int *>(leafv + MAX_PER_WG + 4);
    const Counts C{counts, counts + MAX_PER_WG, counts + 2 * MAX_PER_WG, counts + 3 * MAX_PER_WG};
    if (tid < COUNTS * MAX_PER_WG) counts[tid] = 0;

    // The slots of the run: drawn here, two per wave and walk, or copied from the index list.  Nothing but
    // the slot stands between a draw and the first pixel request, so the walk leaves the leaf's value and
    // the total in LDS, and what is published per draw (publish_draws) is written after the barrier by a
    // wave that has nothing else to do yet.
    auto fill_slots = [&]() {
        if (!S.src.idx) return;
        if (A.draw) {
#pragma unroll 1
            for (int k = 2 * wave; k < ns; k += 16) {
                const int kb = k + 1 < ns ? k + 1 : k;
                const int jj[2] = {lo + k, lo + kb};
                long sl[2];
                float leaf[2];
                const float total = misc::per_sample_walk<2>(A.samp, jj, lane, sl, leaf);
                if (lane == 0) {
                    slots[k] = (int)sl[0];
                    slots[kb] = (int)sl[1];
                    leafv[k] = leaf[0];
                    leafv[kb] = leaf[1];
                    if (k == 0) leafv[MAX_PER_WG] = total;
                }
            }
        } else {
            for (int k = tid; k < ns; k += 512) slots[k] = S.src.idx[lo + k];
        }
    };
    // index, raw importance weight and transition data of the segment-0 draws, one draw per lane
    auto publish_draws = [&]() {
        if (S.src.idx && A.draw && s == 0 && lane < ns)
            misc::per_sample_emit(A.samp, lo + lane, slots[lane], leafv[MAX_PER_WG], leafv[lane]);
    };

    fill_slots();
    sync_lds();   // the slot table is complete, the counts are zero
    if (wave >= PRODUCERS + CONSUMERS) {
        v8bf wa[S3::STEPS][2];
        load_weights<S3>(wa, S.w3, lane, wave & 1);
        if (wave == PRODUCERS + CONSUMERS) publish_draws();   // (the first image is long in coming)
        run_conv3(S, lo, hi, ring2, wa, C, lane, wave & 1);
    } else if (wave >= PRODUCERS) {
        v8bf wa[S2::STEPS][2];
        load_weights<S2>(wa, S.w2, lane, wave & 1);
        run_conv2(S, lo, hi, ring, ring2, wa, C, lane, wave & 1);
    } else {
        Pixels R;
        const int u = first_strip(wave);
        if (u < UNITS * ns) load_strip(R, S.src, lo + sample_of_strip(u), S.src.idx ? slots[sample_of_strip(u)] : 0, u % UNITS, lane);
        run_producer(S, lo, hi, lds + wave * STRIP, ring, slots, C, R, lane, wave);
    }
}
}  // namespace pipe

// ===========================================================================
// conv1, conv2 and conv3 forward in one launch (bf16), for as many samples as the launch-bound sizes have.
//
// A unit is the part of a sample that yields R3 of conv3's seven output rows (see sp::k_conv123_fwd, the fp32
// form of this kernel: same units, same phases).  One workgroup of eight waves takes a unit through all
// three layers in LDS, phase by phase, every wave in the same phase; the weights stay in registers (200),
// from the packed copy.  A workgroup has one unit (one that took several whole samples spilled 37 registers beside the next
// one's pixels: conv launch of a step at 77 14.9 us against 12.9).  The images are laid out for the lanes
// that LDS serves together (Geo; at 77 12.9 -> 11.8).  16x16x32 instructions, transposed tiles:
//   conv1   wave = every eighth tile of 16 pixels, all 32 channels: a pixel fragment serves two products
//   conv2/3 wave = 16 channels, half of the tiles: the sum over the taps stays in one wave
// pipe::k_conv_fwd_pipe overlaps the layers of different samples and is faster per sample once it runs, but its first
// sample takes longer: a layer is the work of two or four waves there (fused_few in api.hip has both sides).
// ===========================================================================
namespace c123 {
struct Seg {
    c1::Src src;
    const bf16_t *w;              // packed conv weights (packed.h)
    const float *b1, *b2, *b3;
    bf16_t *y1, *y2;              // for the backward pass, or nullptr
    bf16_t *y3;
    int n;
    int first;                    // first unit of the segment
};
struct Args {
    Seg seg[3];
    int nseg;
    int draw;
    misc::SampleArgs samp;
    unsigned *clear;              // the arrival counters of a later launch, set to 0 here, or nullptr
};
template <int R3> struct Geo {
    static constexpr int PARTS = (7 + R3 - 1) / R3;
    static constexpr int R2 = R3 + 2, R1 = 2 * R3 + 6, PR = 4 * R1 + 4;
    static constexpr int M1 = R1 * 20, M2 = R2 * 9, M3 = R3 * 7;
    static constexpr int T1 = (M1 + 15) / 16, T2 = (M2 + 31) / 32, T3 = (M3 + 31) / 32;   // tiles of conv1; of conv2 / conv3 per wave
    static constexpr int CH = PR * 84 / 16, NPX = (4 * CH + 511) / 512;
    // conv1's and conv2's images, laid out and read as the samples of ps::Shape are: sixteen lanes, sixteen columns of LDS.
    // Bytes per pixel and row
    static constexpr int PXB = 4 * PR * 84 * 2, P1 = 64, B1 = (20 * 4 + 1) * 16, P2 = 144, B2 = 96 * 16;
    static constexpr int I1B = R1 * B1, I2B = R2 * B2;
    // position n of tile t, in y * 9 + x and y * 7 + x; where there is none, one that another lane has as well
    static __device__ __forceinline__ int position2(int t, int n)
    {
        constexpr int PAIRS = R2 / 2;
        const int r = n >> 3, x = n & 7;
        if (t < PAIRS) return (2 * t + r) * 9 + x;                     // two rows of eight
        if (t > PAIRS) return (R2 - 1) * 9 + 8;
        if (R2 % 2 == 0) return min(n, R2 - 1) * 9 + 8;                // the last column
        return r ? min(x, R2 - 1) * 9 + 8 : (R2 - 1) * 9 + x;          // the last row and the last column
    }
    static __device__ __forceinline__ int position3(int t, int n) { return min(2 * t + (n >> 3), R3 - 1) * 7 + min(n & 7, 6); }
    static constexpr int TAB = (4 + 160) * 4;   // slot, leaf value, total; biases
    static constexpr int LDS = PXB + I1B + I2B + TAB;
    static_assert(PR * 84 % 16 == 0, "LDS layout");
};

// Workgroup u takes unit u of the grid's
template <int R3>
__global__ __launch_bounds__(512, 1) void k_conv123_fwd(Args A)
{
    using G = Geo<R3>;
    typedef const __attribute__((address_space(4))) Args *ArgsPtr;      // the segments, indexed at run time
    const ArgsPtr AP = (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
#define C123_SEG(s) (AP->seg[s])
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    bf16_t *px = reinterpret_cast<bf16_t *>(lds);
    uint8_t *img1 = lds + G::PXB, *img2 = img1 + G::I1B;
    int *slot_at = reinterpret_cast<int *>(img2 + G::I2B);
    float *leafv = reinterpret_cast<float *>(slot_at + 1);   // the leaf's value, then the total
    float *bias = leafv + 3;                                 // conv1 [32], conv2 [64], conv3 [64]
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ct = wave & 3, mh = wave >> 2;
    int tid = threadIdx.x, lane = tid & 63;
    if (A.clear && blockIdx.x == 0) misc::few_clear(A.clear, tid);
    const int u = (int)blockIdx.x, si = (A.nseg > 1 && u >= A.seg[1].first) + (A.nseg > 2 && u >= A.seg[2].first);
    u32x4 raw[G::NPX];
    auto load_px = [&](int slot) {
        const int ul = u - C123_SEG(si).first, g = ul / G::PARTS, part = ul % G::PARTS;
        const int row0 = part * R3 < 7 - R3 ? part * R3 : 7 - R3;
        const uint8_t *f[4];
        const c1::Src src{C123_SEG(si).src.x, C123_SEG(si).src.xs, C123_SEG(si).src.idx, C123_SEG(si).src.cap, C123_SEG(si).src.shift, C123_SEG(si).src.sub};
        if (src.idx) {   // (tested once: with a test per frame acting on one took 0.2 us longer)
#pragma unroll
            for (int k = 0; k < 4; ++k) f[k] = c1::frame_ptr(src, g, slot, k) + row0 * (8 * 84);
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) f[k] = src.x + (long)g * src.xs + (long)(k * c1::FR + row0 * (8 * 84));
        }
#pragma unroll
        for (int i = 0; i < G::NPX; ++i) {
            int t = tid + 512 * i;
            if (t > 4 * G::CH - 1) t = 4 * G::CH - 1;
            const int k = t / G::CH;
            const uint8_t *fp = k == 0 ? f[0] : k == 1 ? f[1] : k == 2 ? f[2] : f[3];
            raw[i] = *reinterpret_cast<const u32x4 *>(fp + (t - k * G::CH) * 16);
        }
    };
    const bool ring = A.seg[0].src.idx != nullptr;
    v8bf w1[8][2], w2[16], w3[18];
    {
        const v8bf *p = reinterpret_cast<const v8bf *>(C123_SEG(si).w) + lane;
#pragma unroll
        for (int k = 0; k < 8; ++k) { w1[k][0] = p[k * 64]; w1[k][1] = p[(8 + k) * 64]; }
        const v8bf *p2 = p + sp::B_W2 / 8 + ct * 16 * 64, *p3 = p + sp::B_W3 / 8 + ct * 18 * 64;
#pragma unroll
        for (int k = 0; k < 16; ++k) w2[k] = p2[k * 64];
#pragma unroll
        for (int k = 0; k < 18; ++k) w3[k] = p3[k * 64];
    }
    if (ring) {
        if (wave == 0) {
            const int j[1] = {u / G::PARTS % A.seg[0].n};
            if (A.draw) {
                long sl[1];
                float leaf[1];
                const float total = misc::per_sample_walk<1>(A.samp, j, lane, sl, leaf);
                if (lane == 0) {
                    *slot_at = (int)sl[0];
                    leafv[0] = leaf[0];
                    leafv[1] = total;
                }
            } else if (lane == 0) *slot_at = A.seg[0].src.idx[j[0]];
        }
        sync_lds();
    }
    load_px(ring ? *slot_at : 0);
    if (A.draw && wave == 7 && lane == 0 && u < A.seg[0].n * G::PARTS && u % G::PARTS == 0)
        misc::per_sample_emit(A.samp, u / G::PARTS, *slot_at, leafv[1], leafv[0]);

    asm volatile("" : "+v"(tid));   // opaque: no lane address of a later phase is formed further up
    lane = tid & 63;
    const int n16 = lane & 15, kg = lane >> 4;
    if (tid < 160) bias[tid] = tid < 32 ? C123_SEG(si).b1[tid] : tid < 96 ? C123_SEG(si).b2[tid - 32] : C123_SEG(si).b3[tid - 96];
    // (load_px's once more; formed ahead of the weights' requests they delay those, acting on one 0.2 us)
    const int ul = u - C123_SEG(si).first, g = ul / G::PARTS, part = ul % G::PARTS;
    const int row0 = part * R3 < 7 - R3 ? part * R3 : 7 - R3;
    const int rowp = part == 0 ? -32 : (part - 1) * R3;   // first conv3 row of the part before this one
#pragma unroll
    for (int i = 0; i < G::NPX; ++i) {
        const int t = tid + 512 * i;
        if (t < 4 * G::CH) {
            uint4 *d = reinterpret_cast<uint4 *>(px + t * 16);
            d[0] = cvt8_u8(raw[i].x, raw[i].y);
            d[1] = cvt8_u8(raw[i].z, raw[i].w);
        }
    }
    bf16_t *const y1 = C123_SEG(si).y1, *const y2 = C123_SEG(si).y2;
    sync_lds();

    // ---- conv1
#pragma unroll 1
    for (int t = wave; t < G::T1; t += 8) {
        const int m = 16 * t + n16, mc = m < G::M1 ? m : G::M1 - 1;
        const int y = mc / 20, x = mc - 20 * y;
        // A step takes four columns (4 xh ..) of the kernel rows 2 kg, 2 kg + 1 of a frame, as in pipe::run_producer: the same
        // sums in the same order, so both launches leave the same bits.  Two-address reads put such a pair into
        // four consecutive registers; they are invisible to the compiler's wait counting.
        typedef uint32_t v4u __attribute__((ext_vector_type(4)));
        const uint32_t addr = (uint32_t)(uintptr_t)(px + (4 * y + 2 * kg) * 84 + 4 * x);
        auto pixels = [&](int f, v4u &q0, v4u &q1) {
            const uint32_t af = addr + f * (G::PR * 84 * 2);
            asm volatile("ds_read2_b64 %0, %1 offset0:0 offset1:21" : "=v"(q0) : "v"(af));
            asm volatile("ds_read2_b64 %0, %1 offset0:1 offset1:22" : "=v"(q1) : "v"(af));
        };
        v4f a0 = {0, 0, 0, 0}, a1 = {0, 0, 0, 0};
        v4u q[2][2];
        pixels(0, q[0][0], q[0][1]);
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            v4u(&c)[2] = q[f & 1], (&nx)[2] = q[(f & 1) ^ 1];
            if (f < 3) {
                pixels(f + 1, nx[0], nx[1]);
                asm volatile("s_waitcnt lgkmcnt(2)" : "+v"(c[0]), "+v"(c[1]));
            } else {
                asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(c[0]), "+v"(c[1]));
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int xh = 0; xh < 2; ++xh) {
                a0 = mfma16(w1[2 * f + xh][0], __builtin_bit_cast(v8bf, c[xh]), a0);
                a1 = mfma16(w1[2 * f + xh][1], __builtin_bit_cast(v8bf, c[xh]), a1);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        const v4f b1a = *reinterpret_cast<const v4f *>(bias + 8 * kg), b1b = *reinterpret_cast<const v4f *>(bias + 8 * kg + 4);
        constexpr float sc = 1.0f / 255.0f;
        v4f v0, v1;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            v0[r] = fmaxf(a0[r] * sc + b1a[r], 0.f);
            v1[r] = fmaxf(a1[r] * sc + b1b[r], 0.f);
        }
        if (m < G::M1) {
            const uint2 lo = pack4(v0.x, v0.y, v0.z, v0.w), hi = pack4(v1.x, v1.y, v1.z, v1.w);
            const uint4 o = {lo.x, lo.y, hi.x, hi.y};
            *reinterpret_cast<uint4 *>(img1 + y * G::B1 + ((x & 1) * 10 + (x >> 1)) * G::P1 + kg * 16) = o;
            if (y1 && 2 * row0 + y >= 2 * rowp + G::R1)
                *reinterpret_cast<uint4 *>(y1 + (long)g * net::A1 + ((2 * row0 + y) * 20 + x) * 32 + 8 * kg) = o;
        }
    }
    sync_lds();
    // ---- conv2: tiles T2 mh .. of 16 positions, channels 16 ct ..
    {
        constexpr int T = G::T2;
        const uint8_t *pa[T];
        int pos[T];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int m = pos[t] = G::position2(T * mh + t, n16), y = m / 9, x = m - 9 * y;
            pa[t] = img1 + 2 * y * G::B1 + x * G::P1 + kg * 16;
        }
        v4f acc[T];
#pragma unroll
        for (int t = 0; t < T; ++t) acc[t] = v4f{0, 0, 0, 0};
        v8bf f[2][T];
        auto rd = [&](int s) {   // kernel row s / 4, column s % 4
#pragma unroll
            for (int t = 0; t < T; ++t)
                f[s & 1][t] = *reinterpret_cast<const v8bf *>(pa[t] + (s >> 2) * G::B1 + ((s & 1) * 10 + ((s >> 1) & 1)) * G::P1);
        };
        rd(0);
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            if (s < 15) rd(s + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < T; ++t) acc[t] = mfma16(w2[s], f[s & 1][t], acc[t]);
            __builtin_amdgcn_sched_barrier(0);
        }
        const v4f b2 = *reinterpret_cast<const v4f *>(bias + 32 + 16 * ct + 4 * kg);
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int m = pos[t], y = m / 9, x = m - 9 * y;
            v4f v;
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = fmaxf(acc[t][r] + b2[r], 0.f);
            const uint2 o = pack4(v.x, v.y, v.z, v.w);   // (lanes that share a position store the same bits)
            *reinterpret_cast<uint2 *>(img2 + y * G::B2 + x * G::P2 + ct * 32 + kg * 8) = o;
            if (y2 && row0 + y >= rowp + G::R2)
                *reinterpret_cast<uint2 *>(y2 + (long)g * net::A2 + (row0 * 9 + m) * 64 + 16 * ct + 4 * kg) = o;
        }
    }
    sync_lds();
    // ---- conv3
    {
        constexpr int T = G::T3;
        const uint8_t *pa[T];
        int pos[T];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int m = pos[t] = G::position3(T * mh + t, n16), y = m / 7, x = m - 7 * y;
            pa[t] = img2 + y * G::B2 + x * G::P2 + kg * 16;
        }
        v4f acc[T];
#pragma unroll
        for (int t = 0; t < T; ++t) acc[t] = v4f{0, 0, 0, 0};
        v8bf f[2][T];
        auto rd = [&](int s) {   // tap s / 2, channel half s % 2
#pragma unroll
            for (int t = 0; t < T; ++t)
                f[s & 1][t] = *reinterpret_cast<const v8bf *>(pa[t] + (s / 6) * G::B2 + ((s / 2) % 3) * G::P2 + (s & 1) * 64);
        };
        rd(0);
#pragma unroll
        for (int s = 0; s < 18; ++s) {
            if (s < 17) rd(s + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < T; ++t) acc[t] = mfma16(w3[s], f[s & 1][t], acc[t]);
            __builtin_amdgcn_sched_barrier(0);
        }
        const v4f b3 = *reinterpret_cast<const v4f *>(bias + 96 + 16 * ct + 4 * kg);
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int m = pos[t], y = m / 7;
            v4f v;
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = fmaxf(acc[t][r] + b3[r], 0.f);
            if (row0 + y >= rowp + R3)
                *reinterpret_cast<uint2 *>(C123_SEG(si).y3 + (long)g * net::A3 + (row0 * 7 + m) * 64 + 16 * ct + 4 * kg) = pack4(v.x, v.y, v.z, v.w);
        }
    }
#undef C123_SEG
}
}  // namespace c123

// ===========================================================================
// Input gradient of conv2, one sample per workgroup (Section 2.1 network, backward pass of the
// Section 2.2 loss).  dX[pixel][ci] = sum over taps and co of dY[position][co] W[co][tap][ci]:
// the reduction runs over (tap, co), so the weights are needed with co as the reduction index and
// ci as the block row.  They are fetched once per workgroup in their natural [co][tap][ci] layout,
// passed through LDS in two halves of 32 output channels, and read back with the transposing LDS
// load (ds_read_tr16_b64) straight into a-operand registers, where they stay for all samples.
//
// A sample's dY image sits in LDS (160 bytes per pixel, PIX and ROW below) inside a border of zeros (written
// once), so taps that fall outside the image read zeros: no bounds test, and every b-operand is a
// single 16-byte read at a per-lane base + immediate offset.  The next sample's dY is in flight
// while the current one is multiplied.  The ReLU mask is the stored activation at the result's
// own place (16 bytes per lane per block, prefetched); the lane's 8 results are 8 consecutive
// channels, stored as 16 bytes.
//
// The kernel is 4x4 with stride 2, so the 20x20 input pixels fall into four stride-parity classes
// (y%2, x%2); a pixel of class (py, px) is reached by the four taps (py + 2ty, px + 2tx) only.
// Wave = class: 100 pixels = 7 position blocks, 4 taps x 64 co = 8 reduction steps, 64 weight
// registers.  (c3b is this scheme for the 3x3 stride-1 layer, in 144 weight registers.)
// ===========================================================================
namespace dps {
using ps::u32x4;
// The 9x9 image inside a border of one zero pixel: LDS bytes per pixel (128 + 32) and per row, and the ten by ten pixels of a
// parity class in tiles of sixteen.  As in ps::Shape: over two rows of eight pixels the sixteen lanes that are served
// together read from the sixteen different 16-byte columns of LDS (pixels in order at a pitch of 144: nearly every
// read took twice as long).
constexpr int PIX = 160, ROW = 11 * PIX + 32;
constexpr int IMG = 11 * ROW;
static_assert(ROW % 256 == 0, "rows of whole LDS lines");
struct Place { int y, x; };
// pixel n of tile b: five tiles of two rows of eight, then the last two columns; pixels that do not exist repeat another
__device__ __forceinline__ Place place_of(int b, int n)
{
    if (b < 5) return Place{2 * b + (n >> 3), n & 7};
    return Place{b == 5 ? n >> 1 : 8 + ((n >> 1) & 1), 8 + (n & 1)};
}

struct Args {
    const bf16_t *dy;    // [B][positions out][64]
    const bf16_t *w;     // [64][taps][channels in]
    const bf16_t *xact;  // [B][pixels in][channels in], the layer input after ReLU
    bf16_t *dx;          // [B][pixels in][channels in]
    int B;
};

// a-operand of v_mfma_f32_16x16x32_bf16 out of a [reduction][column] tile in LDS: lane 16kg + s gets
// reduction rows 8kg .. 8kg+7 of block row s.  The 16 block rows are four runs of four consecutive
// tile columns; colbyte is the byte offset of the run that block row s belongs to.
__device__ __forceinline__ v8bf frag_tr16(const uint8_t *tile, int pitch, int lane, int colbyte)
{
    typedef __attribute__((address_space(3))) v4s *lds_v4s;
    typedef short v8s __attribute__((ext_vector_type(8)));
    const int s = lane & 15, kg = lane >> 4;
    const uint8_t *p = tile + (8 * kg + (s >> 2)) * pitch + colbyte;
    const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(p));
    const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(p + 4 * pitch));
    const v8s r = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    return __builtin_bit_cast(v8bf, r);
}

// 8 results of a lane through the ReLU mask (activation bits > 0 as a signed 16-bit test) to 16 bytes
__device__ __forceinline__ uint4 masked8(const uint4 m, const v4f a0, const v4f a1)
{
    auto keep = [](uint32_t w2, int hi, float v) { return (int16_t)(hi ? (w2 >> 16) : (w2 & 0xFFFFu)) > 0 ? v : 0.f; };
    const uint2 lo = pack4(keep(m.x, 0, a0.x), keep(m.x, 1, a0.y), keep(m.y, 0, a0.z), keep(m.y, 1, a0.w));
    const uint2 hi = pack4(keep(m.z, 0, a1.x), keep(m.z, 1, a1.y), keep(m.w, 0, a1.z), keep(m.w, 1, a1.w));
    return uint4{lo.x, lo.y, hi.x, hi.y};
}

constexpr int W2PITCH = 512 * 2 + 16;   // LDS bytes per conv2 weight row in transit (one co: 16 taps x 32 ci)

// dy [B][81][64], w [64][4][4][32], xact and dx [B][400][32]; workgroup `bid` of `nblocks`
__device__ __forceinline__ void conv2_dgrad_ps_body(const Args &A, int bid, int nblocks, uint8_t *lds)
{
    uint8_t *img = lds, *wt = lds + IMG;
    const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, kg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), py = wave >> 1, px = wave & 1;
    const int g0 = (int)((long)bid * A.B / nblocks), g1 = (int)((long)(bid + 1) * A.B / nblocks);
    if (g0 >= g1) return;
    // a sample's dY is 648 pieces of 16 bytes; the first sample's is on its way while the weights pass through
    u32x4 r0, r1, r2;
    auto load_dy = [&](int g) {
        const u32x4 *p = reinterpret_cast<const u32x4 *>(A.dy + (long)g * (81 * 64));
        r0 = p[tid]; r1 = p[tid + 256]; r2 = p[tid < 136 ? tid + 512 : 647];
    };
    load_dy(g0);
    for (int i = tid; i < IMG / 16; i += 256) *reinterpret_cast<u32x4 *>(img + i * 16) = u32x4{0, 0, 0, 0};
    // wa[2 tap + co half][ci block], tap = 2ty + tx = kernel element (py + 2ty, px + 2tx); block row s of ci
    // block cb is input channel 8(s/4) + 4cb + s%4, so a lane's 8 results are 8 consecutive channels
    v8bf wa[8][2];
    for (int half = 0; half < 2; ++half) {
        const u32x4 *src = reinterpret_cast<const u32x4 *>(A.w + half * 32 * 512);
        sync_lds();
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int c = tid + 256 * i;   // row (co) c / 64, 16-byte piece c % 64
            *reinterpret_cast<u32x4 *>(wt + (c >> 6) * W2PITCH + (c & 63) * 16) = src[c];
        }
        sync_lds();
#pragma unroll
        for (int tap = 0; tap < 4; ++tap)
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                const int ky = py + 2 * (tap >> 1), kx = px + 2 * (tap & 1);
                const int col = (ky * 4 + kx) * 32 + 8 * (n & 3) + 4 * cb;
                wa[2 * tap + half][cb] = frag_tr16(wt, W2PITCH, lane, col * 2);
            }
    }
    // pixel (2a + py, 2b + px) takes dY positions (a - ty, b - tx); image pixel (a - ty + 1, b - tx + 1) holds them.
    // base = the (ty, tx) = (1, 1) corner, i.e. image pixel (a, b)
    uint32_t base[7];
    int pix[7];   // its pixel
#pragma unroll
    for (int b = 0; b < 7; ++b) {
        const Place P = place_of(b, n);
        base[b] = P.y * ROW + P.x * PIX + kg * 16;
        pix[b] = (2 * P.y + py) * 20 + 2 * P.x + px;
    }
    for (int g = g0; g < g1; ++g) {
        sync_lds();   // the previous sample's image (and, the first time, the weights in transit) has been read
#define DPS_ST(I, V) { const int t = tid + 256 * I; const int q = t >> 3; *reinterpret_cast<u32x4 *>(img + (q / 9 + 1) * ROW + (q % 9 + 1) * PIX + (t & 7) * 16) = V; }
        DPS_ST(0, r0) DPS_ST(1, r1)
        if (tid < 136) DPS_ST(2, r2)
#undef DPS_ST
        if (g + 1 < g1) load_dy(g + 1);
        const long obase = (long)g * (400 * 32) + 8 * kg;
        uint4 mk[7];
#pragma unroll
        for (int b = 0; b < 7; ++b) mk[b] = *reinterpret_cast<const uint4 *>(A.xact + obase + pix[b] * 32);
        sync_lds();
#pragma unroll
        for (int b = 0; b < 7; ++b) {
            v4f acc0 = {0, 0, 0, 0}, acc1 = {0, 0, 0, 0};
#pragma unroll
            for (int st = 0; st < 8; ++st) {
                const int tap = st >> 1, ty = tap >> 1, tx = tap & 1;
                const int off = (1 - ty) * ROW + (1 - tx) * PIX + (st & 1) * 64;
                const v8bf bb = __builtin_bit_cast(v8bf, *reinterpret_cast<const uint4 *>(img + base[b] + off));
                acc0 = mfma16(wa[st][0], bb, acc0);
                acc1 = mfma16(wa[st][1], bb, acc1);
            }
            // (lanes that share a pixel store the same bits)
            *reinterpret_cast<uint4 *>(A.dx + obase + pix[b] * 32) = masked8(mk[b], acc0, acc1);
        }
    }
}
constexpr int PS_LDS = IMG + 32 * W2PITCH;   // bytes

// conv2's input gradient AND conv1's weight gradient of a sample in one workgroup (Section 2.1 network,
// backward pass of the Section 2.2 loss): conv1's dY is needed by nothing but conv1's weight gradient,
// sample by sample, so the workgroup that forms it keeps it in LDS, in the layout the weight gradient
// stages it in, and goes on to the weight gradient of the same sample (c1::conv1_wgrad_block's loop,
// both channel pairs one after the other, the frames read from the ring or the explicit states).  conv1's dY is never written to
// memory, and the launch of conv1's weight gradient, with its hand-over, is gone.  Workgroup b takes samples b, b + nblocks, ... and
// writes ONE partial of conv1's weight gradient: the same samples in the same order as split b of
// c1::k_conv1_wgrad with nblocks splits, so the partials have the same bits.
struct FusedArgs {
    Args d;           // dx is not used
    c1::Src src;      // where the frames of sample n come from
    float *part1;     // [nblocks][32*256 + 32]
    const uint16_t *w2;  // conv2's weights in the order of sp::packed_conv2_back_at
};
constexpr int FUSED_DYS = 400 * c1::LDY1 * 2;             // 25,600 bytes: conv1's dY as the weight gradient reads it
constexpr int FUSED_XIN = 2 * c1::FR * 2;                 // 28,224 bytes: two frames as bf16
constexpr int FUSED_LDS = FUSED_DYS + FUSED_XIN + IMG;    // 73,536 bytes

__device__ __forceinline__ void conv2_dgrad_conv1_wgrad_body(const FusedArgs &F, int bid, int nblocks, uint8_t *lds)
{
    using c1::FR;
    using c1::LDY1;
    const Args &A = F.d;
    bf16_t *dys = reinterpret_cast<bf16_t *>(lds), *xin = reinterpret_cast<bf16_t *>(lds + FUSED_DYS);
    uint8_t *img = lds + FUSED_DYS + FUSED_XIN;
    const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, kg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), py = wave >> 1, px = wave & 1;
    if (bid >= A.B) return;
    u32x4 r0, r1, r2;
    auto load_dy = [&](int g) {
        const u32x4 *p = reinterpret_cast<const u32x4 *>(A.dy + (long)g * (81 * 64));
        r0 = p[tid]; r1 = p[tid + 256]; r2 = p[tid < 136 ? tid + 512 : 647];
    };
    load_dy(bid);
    int slot_n = c1::sample_slot(F.src, bid);
    const bf16_t *const xg0 = A.xact + 8 * kg;
    for (int i = tid; i < IMG / 16; i += 256) *reinterpret_cast<u32x4 *>(img + i * 16) = u32x4{0, 0, 0, 0};
    // conv2's weights, wa[2 tap + co half][ci block] as in conv2_dgrad_ps_body, from a copy in the order of the operands
    v8bf wa[8][2];
#pragma unroll
    for (int st = 0; st < 8; ++st)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
            wa[st][cb] = __builtin_bit_cast(v8bf, *reinterpret_cast<const uint4 *>(F.w2 + (((2 * py + px) * 8 + st) * 2 + cb) * sp::FRAG + lane * 8));
    // this lane's place of tile b in the wave's parity class: its dY corner in the image; its pixel
    auto base_of = [&](int b) { const Place P = place_of(b, n); return (uint32_t)(P.y * ROW + P.x * PIX + kg * 16); };
    auto pixel_of = [&](int b) { const Place P = place_of(b, n); return (2 * P.y + py) * 20 + 2 * P.x + px; };
    // conv1's weight gradient: this lane's share as in c1::conv1_wgrad_block (wave = block of 32 im2col columns)
    typedef __attribute__((address_space(3))) v4s *lds_v4s;
    const int li = lane & 31, h = lane >> 5, s16 = lane & 15, half = (lane >> 4) & 1;
    const int rsub = 8 * h + (s16 >> 2);
    const int kc = 32 * wave + 16 * half + 4 * (s16 & 3);
    const int xoff = (kc >> 6) * FR + ((kc >> 3) & 7) * 84 + (kc & 7);
    const bf16_t *yp = dys + rsub * LDY1 + 16 * half + 4 * (s16 & 3);
    const bf16_t *xw = xin + xoff + 4 * rsub;   // the window of output pixel rsub
    v16f acc[2] = {v16f{0}, v16f{0}}, accb = {0};
    v8bf ones;
#pragma unroll
    for (int e = 0; e < 8; ++e) ones[e] = (__bf16)1.0f;
    c1::Staged<256, 2> R, R2;   // the frames of the two channel pairs
    // A sample's dY, frames and first two ReLU masks are on their way while the sample before is computed, its slot one sample longer
    // (with the weights in the order of the operands, not 64 bytes at a time: a step of 512 124 -> 121 us, of 1000 190 -> 185, of 77
    // 58.4 -> 57.9; eight waves with all four frames in LDS, one workgroup per CU: 77 57.4, 256 91.1 against 89, 512 128 against 121)
    uint4 mk0 = *reinterpret_cast<const uint4 *>(xg0 + (long)bid * (400 * 32) + pixel_of(0) * 32);
    uint4 mk1 = *reinterpret_cast<const uint4 *>(xg0 + (long)bid * (400 * 32) + pixel_of(1) * 32);
    c1::stage_load<256, 2>(R, F.src, bid, slot_n, 0, tid);
    c1::stage_load<256, 2>(R2, F.src, bid, slot_n, 2, tid);
    slot_n = bid + nblocks < A.B ? c1::sample_slot(F.src, bid + nblocks) : 0;

    for (int g = bid; g < A.B; g += nblocks) {
        sync_lds();   // the previous sample's image, dY tile and frames have been read (the first time: the image is cleared)
#define DPS_ST(I, V) { const int t = tid + 256 * I; const int q = t >> 3; *reinterpret_cast<u32x4 *>(img + (q / 9 + 1) * ROW + (q % 9 + 1) * PIX + (t & 7) * 16) = V; }
        DPS_ST(0, r0) DPS_ST(1, r1)
        if (tid < 136) DPS_ST(2, r2)
#undef DPS_ST
        const int gn = g + nblocks;
        if (gn < A.B) load_dy(gn);
        const int slot_nn = gn + nblocks < A.B ? c1::sample_slot(F.src, gn + nblocks) : 0;
        const bf16_t *xg = xg0 + (long)g * (400 * 32), *xgn = gn < A.B ? xg0 + (long)gn * (400 * 32) : xg;
        sync_lds();
        // the operands are requested three reduction steps ahead (into the next blocks): a step's two matrix instructions
        // are a quarter of what a read takes
        constexpr int AHEAD = 3;
        auto operand = [&](int i) {   // step i % 8 of block i / 8
            const int b = i >> 3, st = i & 7, tap = st >> 1, ty = tap >> 1, tx = tap & 1;
            const int off = (1 - ty) * ROW + (1 - tx) * PIX + (st & 1) * 64;
            return *reinterpret_cast<const uint4 *>(img + base_of(b) + off);
        };
        uint4 q[AHEAD + 1];
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) q[i] = operand(i);
#pragma unroll
        for (int b = 0; b < 7; ++b) {
            const uint4 mk = mk0;
            mk0 = mk1;
            // ReLU masks two blocks ahead of their use (all seven at once would cost 28 registers)
            mk1 = *reinterpret_cast<const uint4 *>((b + 2 < 7 ? xg : xgn) + pixel_of((b + 2) % 7) * 32);
            v4f acc0 = {0, 0, 0, 0}, acc1 = {0, 0, 0, 0};
#pragma unroll
            for (int st = 0; st < 8; ++st) {
                const int i = 8 * b + st;
                if (i + AHEAD < 56) q[(i + AHEAD) % (AHEAD + 1)] = operand(i + AHEAD);
                __builtin_amdgcn_sched_barrier(0);
                const v8bf bb = __builtin_bit_cast(v8bf, q[i % (AHEAD + 1)]);
                acc0 = mfma16(wa[st][0], bb, acc0);
                acc1 = mfma16(wa[st][1], bb, acc1);
                __builtin_amdgcn_sched_barrier(0);
            }
            *reinterpret_cast<uint4 *>(dys + pixel_of(b) * LDY1 + 8 * kg) = masked8(mk, acc0, acc1);
        }
#pragma unroll
        for (int cp = 0; cp < 2; ++cp) {
            if (cp == 1) sync_lds();   // the first pair's frames have been read
            c1::stage_store<256, 2>(xin, cp == 0 ? R : R2, tid);
            if (gn < A.B) c1::stage_load<256, 2>(cp == 0 ? R : R2, F.src, gn, slot_n, 2 * cp, tid);
            sync_lds();   // the dY tile and the pair's frames are complete
            const bool do_bias = cp == 0 && wave == 0;
            // the operands are requested two steps ahead
            constexpr int AHEAD = 2;
            auto operands = [&](int t, v8bf &fa, v8bf &fb) {   // 16 output pixels per step
                fa = frag_tr(yp + 16 * t * LDY1, LDY1);
                // see c1::conv1_wgrad_block: no division
                const int q = (16 * t) / 20, r = (16 * t) % 20;
                const bf16_t *x0 = xw + (336 * q + 4 * r) + (rsub >= 20 - r ? 256 : 0);
                const bf16_t *x1 = xw + (336 * q + 4 * r + 16) + (rsub + 4 >= 20 - r ? 256 : 0);
                v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)x0);
                v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)x1);
                typedef short v8s __attribute__((ext_vector_type(8)));
                v8s xb = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
                fb = __builtin_bit_cast(v8bf, xb);
            };
            v8bf fa[AHEAD + 1], fb[AHEAD + 1];
#pragma unroll
            for (int t = 0; t < AHEAD; ++t) operands(t, fa[t], fb[t]);
#pragma unroll
            for (int t = 0; t < 25; ++t) {
                constexpr int N = AHEAD + 1;
                if (t + AHEAD < 25) operands(t + AHEAD, fa[(t + AHEAD) % N], fb[(t + AHEAD) % N]);
                __builtin_amdgcn_sched_barrier(0);
                acc[cp] = mfma(fa[t % N], fb[t % N], acc[cp]);
                if (do_bias) accb = mfma(fa[t % N], ones, accb);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        slot_n = slot_nn;
    }

    float *part = F.part1 + (long)bid * (32 * 256 + 32);
#pragma unroll
    for (int cp = 0; cp < 2; ++cp)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int o = 8 * (r / 4) + 4 * h + (r % 4);
            part[o * 256 + 128 * cp + 32 * wave + li] = acc[cp][r] * (1.0f / 255.0f);
            if (cp == 0 && wave == 0 && li == 0) part[32 * 256 + o] = accb[r];
        }
}
}  // namespace dps

// ===========================================================================
// conv3's input gradient (3x3 stride 1, 7x7x64 -> 9x9x64), a sample's dY inside a border of two zero pixels in LDS, the weights in
// registers (from a copy in the order of the operands, packed.h).  In 64 x 64 im2col tiles every dY was fetched once per
// tap, in nine dependent stages of 0.8 us.
// 32x32x16 instructions, the steps of sixteen output channels by turns into two sums, as in dgrad_tile: the same bits as its
// tiles.  A lane of the result holds sixteen channels of a pixel.
// A pixel is 144 bytes and a row 1808, so that position p lies 144 p bytes (mod 256) from the first: the sixteen positions that are
// served together read from the sixteen different 16-byte columns of LDS.
// In its launch conv3's weight gradient has become tiles of a whole kernel row (64 x 192; 64 x 64 before), which read dY a third
// as often.  A step of 512 131.2 -> 124 us, of 77 60.7 -> 59, of 256 96.2 -> 90 with these two; what bounds the launch is the chain
// of a tile's ten stages and of a workgroup's samples: both gradients are 2 us of matrix instructions spread over all CUs.
// (16x16x32 instructions, and the weight gradient out of whole samples in LDS, each in an order of its own, were 3 us faster at 512.
// In the old order, sixteen rows wherever a sample ends, the latter is a chain of LDS reads: 8 us slower.)
// ===========================================================================
namespace c3b {
using ps::u32x4;
constexpr int OUT = 49 * 64, IN = 81 * 64, YPIECES = OUT / 8;
constexpr int PIX = 144, ROW = 11 * PIX + 224, IMG = 11 * ROW;   // bytes
static_assert(ROW % 256 == 9 * PIX % 256, "banks");
constexpr int LDS = 2 * IMG;                                     // 39,776 bytes

struct Args {
    const bf16_t *dy;    // [B][7][7][64]
    const bf16_t *x;     // [B][9][9][64], conv2's output after ReLU
    const uint16_t *w;   // the weights in the order of sp::packed_conv3_back_at
    bf16_t *dx;          // [B][9][9][64]
    int B;
    int nd;              // workgroups
};

// Samples [bid * B / nd, (bid + 1) * B / nd), two at a time.  Wave (ph, hh): channels 32 hh .. + 31 of half of the six tiles of 32
// pixels that two samples have.
__device__ __forceinline__ void dgrad_body(const Args &A, int bid, uint8_t *lds)
{
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), ph = wave & 1, hh = wave >> 1;
    const int g0 = (int)((long)bid * A.B / A.nd), g1 = (int)((long)(bid + 1) * A.B / A.nd);
    if (g0 >= g1) return;
    u32x4 r[2][2];
    auto load_dy = [&](int g) {   // samples g and g + 1; the last loads repeat the last sample
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const u32x4 *p = reinterpret_cast<const u32x4 *>(A.dy + (long)min(g + s, g1 - 1) * OUT);
            r[s][0] = p[tid];
            r[s][1] = p[tid < YPIECES - 256 ? tid + 256 : YPIECES - 1];
        }
    };
    load_dy(g0);
    v8bf wa[36];   // step 4 tap + sixteenth of dY's channels
#pragma unroll
    for (int st = 0; st < 36; ++st) wa[st] = __builtin_bit_cast(v8bf, *reinterpret_cast<const uint4 *>(A.w + (hh * 36 + st) * sp::FRAG + lane * 8));
    for (int i = tid; i < LDS / 16; i += 256) *reinterpret_cast<u32x4 *>(lds + i * 16) = u32x4{0, 0, 0, 0};
    for (int g = g0; g < g1; g += 2) {
        sync_lds();   // the images have been read (the first time: are cleared)
        auto put = [&](int s, int t, u32x4 v) {
            const int q = t >> 3;
            *reinterpret_cast<u32x4 *>(lds + s * IMG + (q / 7 + 2) * ROW + (q % 7 + 2) * PIX + (t & 7) * 16) = v;
        };
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            put(s, tid, r[s][0]);
            if (tid < YPIECES - 256) put(s, tid + 256, r[s][1]);
        }
        load_dy(min(g + 2, g1 - 1));
        sync_lds();
        // pixel (y, x) takes dY position (y - p, x - q) for tap (p, q): image pixel (y - p + 2, x - q + 2)
        auto tile = [&](int s, int t) {
            const int pos = min(32 * t + li, 80);   // (past the last pixel: the last one once more, the same bits)
            const uint8_t *b = lds + s * IMG + pos / 9 * ROW + pos % 9 * PIX + h * 16;
            const long o = (long)(g + s) * IN + pos * 64 + 32 * hh + 16 * h;
            uint4 mk[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) mk[k] = *reinterpret_cast<const uint4 *>(A.x + o + 8 * k);
            auto operand = [&](int st) {
                const int tap = st >> 2;
                return *reinterpret_cast<const uint4 *>(b + (2 - tap / 3) * ROW + (2 - tap % 3) * PIX + (st & 3) * 32);
            };
            constexpr int N = 5;   // four steps ahead
            uint4 q[N];
#pragma unroll
            for (int st = 0; st < N - 1; ++st) q[st] = operand(st);
            v16f acc[2] = {v16f{0}, v16f{0}};
#pragma unroll
            for (int st = 0; st < 36; ++st) {
                if (st + N - 1 < 36) q[(st + N - 1) % N] = operand(st + N - 1);
                __builtin_amdgcn_sched_barrier(0);
                acc[st & 1] = mfma(wa[st], __builtin_bit_cast(v8bf, q[st % N]), acc[st & 1]);
                __builtin_amdgcn_sched_barrier(0);
            }
            acc[0] += acc[1];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const v4f a0 = {acc[0][8 * k], acc[0][8 * k + 1], acc[0][8 * k + 2], acc[0][8 * k + 3]};
                const v4f a1 = {acc[0][8 * k + 4], acc[0][8 * k + 5], acc[0][8 * k + 6], acc[0][8 * k + 7]};
                *reinterpret_cast<uint4 *>(A.dx + o + 8 * k) = dps::masked8(mk[k], a0, a1);
            }
        };
        // tiles 0 and 1 of the first sample and 0 of the second; 2 of the first, 1 and 2 of the second
#pragma unroll 1
        for (int k = 0; k < 3; ++k) {
            const int s = ph == 0 ? k == 2 : k > 0, t = ph == 0 ? (k == 2 ? 0 : k) : (k == 0 ? 2 : k);
            if (g + s < g1) tile(s, t);
        }
    }
}
}  // namespace c3b
}  // namespace gbf

// fp32 layers on the bf16 matrix cores, without giving up fp32 accuracy.
//
// A float is the sum of three bf16 numbers: x0 = bf16(x), x1 = bf16(x - x0), x2 = bf16(x - x0 - x1).
// Round-to-nearest leaves 8 significant bits to each, 24 in all, so the sum is x itself: nothing of an
// operand is dropped.  A product x*w is then nine products of bf16 numbers, each exact in the fp32
// accumulator of the matrix instruction.  The three smallest, x1*w2, x2*w1 and x2*w2, are left out: x1 is at most 2^-8
// of x and w2 at most 2^-17 of w, so together they reach 2^-24 of |x*w|, what rounding one product to fp32 may cost;
// over random operands their rms is 2^-27.5.  Pixels are bytes and exact in ONE bf16 number, so conv1 needs three
// products and drops none.
// The leading products x0*w0 are summed apart from the others, which are below 2^-7 of them (Acc2): the matrix
// instruction's additions do not round to nearest but leave errors of one sign, up to a unit in the last place of the
// sum, and an instruction of small products into a large sum costs as many of them as one of large products.
// Measured against fp64, conv2 and conv3 alone through the library's calls, for 3, 60, 200 and 600 observations (the
// geometries below): inputs after a ReLU, random 24-bit values, error over sum |x*w|, rms over the outputs in 1e-8
//   weights                              uniform    normal     a fifth nonzero   positive
//   this form                            0.4-0.5    0.4-0.6    0.8-1.1           4.2-5.4
//   the six products in one sum          0.8-1.3    0.8-1.4    1.5-2.4           5.2-8.2
//   v_mfma_f32 in the layers' launches   1.3-2.4    1.2-2.8    1.5-3.1           7.7-30
// In one sum the errors have a mean of -0.05 to -0.4 (positive weights: down to -1.1), in the other two none that stands
// out from the noise.
// Cost per 32 reduction elements of a 16 x 16 tile: six bf16 instructions of 16 cycles against eight
// fp32 ones of 32: 96 against 256 cycles of the matrix pipe.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "gemm_bf16.h"
#include "gemm_fp32.h"
#include "net.h"
#include "packed.h"
#include "sumtree.h"

namespace sp {

using gbf::bf16_t;
using gbf::mfma;
using gbf::mfma16;
using gbf::pack4;
using gbf::sync_lds;
using gbf::v8bf;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_a8 __attribute__((ext_vector_type(4), aligned(8)));

// The three bf16 parts of four floats
struct Split4 { uint2 p[3]; };
__device__ __forceinline__ v4f unpack4(uint2 u)
{
    return v4f{__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xFFFF0000u), __uint_as_float(u.y << 16),
               __uint_as_float(u.y & 0xFFFF0000u)};
}
__device__ __forceinline__ Split4 split4(v4f v)
{
    // (opaque: otherwise the compiler rounds the low value of each pair once more by itself to unpack it)
    auto opaque = [](uint2 u) { asm("" : "+v"(u.x), "+v"(u.y)); return u; };
    Split4 s;
    s.p[0] = opaque(pack4(v.x, v.y, v.z, v.w));
    v4f r = v - unpack4(s.p[0]);
    s.p[1] = opaque(pack4(r.x, r.y, r.z, r.w));
    r = r - unpack4(s.p[1]);
    s.p[2] = pack4(r.x, r.y, r.z, r.w);
    return s;
}
__device__ __forceinline__ void split8(v8bf (&f)[3], v4f a, v4f b)
{
    const Split4 s = split4(a), t = split4(b);
#pragma unroll
    for (int q = 0; q < 3; ++q) f[q] = __builtin_bit_cast(v8bf, u32x4{s.p[q].x, s.p[q].y, t.p[q].x, t.p[q].y});
}
// The six products of a 32 x 32 x 16 step, the leading ones in a sum of their own, to which the caller adds the rest once
// at the end.  In a gradient, which is a sum of tens of thousands of such results that cancel, the one-sided errors of a
// single sum would add up (conv1's weight gradient at a batch of 42 with everything in one sum: 8.2e-7 of its norm off
// fp64, in the plain fp32 chain 3.8e-7).
struct Acc2 { v16f hi, lo; };
// ... added.  An infinity splits into itself and NaNs: its sum of leading products is what the fp32 chain gives (infinite, or
// NaN where infinities cancel or meet a zero), the sum of the others NaN, which the median turns into a finite number.
// (Finite values above 3.39e38, which round to an infinite bf16, count as infinities.)
__device__ __forceinline__ float joined(float hi, float lo) { return hi + __builtin_amdgcn_fmed3f(lo, -__FLT_MAX__, __FLT_MAX__); }
__device__ __forceinline__ v16f joined(v16f hi, v16f lo)
{
    v16f s;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = joined(hi[r], lo[r]);
    return s;
}
__device__ __forceinline__ void mfma6(const v8bf (&a)[3], const v8bf (&b)[3], Acc2 &c)
{
    c.lo = mfma(a[2], b[0], c.lo);
    c.hi = mfma(a[0], b[0], c.hi);
    c.lo = mfma(a[0], b[2], c.lo);
    c.lo = mfma(a[1], b[1], c.lo);
    c.lo = mfma(a[1], b[0], c.lo);
    c.lo = mfma(a[0], b[1], c.lo);
}
// ... where b is exact in one part
__device__ __forceinline__ void mfma3(const v8bf (&a)[3], v8bf b, v16f &hi, v16f &lo)
{
    lo = mfma(a[2], b, lo);
    hi = mfma(a[0], b, hi);
    lo = mfma(a[1], b, lo);
}
// Sums of a's rows (bias gradients), in every column
struct RowSum {
    v8bf ones;
    Acc2 acc;
    __device__ __forceinline__ RowSum() : acc{v16f{0}, v16f{0}}
    {
#pragma unroll
        for (int e = 0; e < 8; ++e) ones[e] = (__bf16)1.0f;
    }
    __device__ __forceinline__ void add(const v8bf (&a)[3]) { mfma3(a, ones, acc.hi, acc.lo); }
    __device__ __forceinline__ float row(int r) const { return joined(acc.hi[r], acc.lo[r]); }
};

// ---------------------------------------------------------------------------
// conv1, conv2 and conv3 forward in ONE launch.  A unit is the part of a sample that yields R3 of the seven
// output rows of conv3 (R3 = 7: the whole sample): it needs R3 + 2 rows of conv2 and 2 R3 + 6 rows of conv1.
// One workgroup of eight waves works on a unit at a time and keeps everything between the pixels
// and conv3's output in LDS.
//   pixels    read from the ring (or the states) and staged as bf16 (exact)
//   conv1     16x16x32: wave = (channel half, every fourth tile of 16 pixels), the wave's weights in registers
//   conv2/3   32x32x16: wave = (channel half, quarter of the reduction), every weight
//             is read once per unit by one wave; the four partial tiles meet in LDS, each wave
//             finishing a quarter of the channels (bias, ReLU, split)
// The weights are the caller's fp32 parameters and are split here.  310 KB per network do not fit a CU beside the images,
// so they stream from the L2s: conv2's are requested before conv1 starts, conv3's take the registers conv2's leave step by
// step, and conv1's of the next unit those of conv3's; so do the next unit's pixels.  Four lanes load 64 bytes of a row
// together; conv1's weights are split on their way into LDS, where four waves read them, a step of conv2's and conv3's
// passes through 2 KB of LDS of its wave's own to the lanes that multiply it.  Its parts are formed between the matrix
// instructions of the step before.  Acting on one observation took 21.5 us (17.2 since, HALF below and k_fc1_head_act); with loads by the lanes that multiply
// (16 bytes of 64 rows per instruction) 24.7, with the parts formed in front of the matrix instructions 22.8, with parts
// kept in memory beside the parameters 20.1, but then a write to the parameters went unseen.
// R3 = 7 is the least work (no row twice); with few samples smaller parts spread a sample over
// several CUs, recomputing the rows that neighbouring parts share: R3 = 4 costs 1.3 times the conv1 and 1.2 times
// the conv2 work, R3 = 1 2.8 and 2.3 times.
// Image layout: a pixel's 32 (64) channels of part 0, then part 1, then part 2, at a pitch of an odd
// number of 16-byte units, so that the pixels of an output row hit different banks; conv1's image holds
// the even columns of a row before the odd ones (conv2 has stride 2).
// In draw mode the workgroup draws its units' transitions (two per wave and walk) before the first pixel;
// the workgroups that own part 0 of segment 0 publish the draws.
// ---------------------------------------------------------------------------
struct Seg {
    gbf::c1::Src src;
    const float *theta;          // the network's parameters
    float *y3;
    int n;
    int first;                   // first unit of the segment
};
struct Args {
    Seg seg[3];
    int nseg;
    int units;                   // of all segments
    int draw;                    // the samples are drawn from the ring here (every segment has the same n), or are states
    misc::SampleArgs samp;
    unsigned *clear;             // the arrival counters of a later launch, set to 0 here, or nullptr
};
constexpr int MAX_UNITS = 96;    // units of one workgroup at most
constexpr int TURN = 2048;       // bytes of LDS in which a wave hands a step's weights to the lanes that multiply them

template <int R3> struct Geo {
    static constexpr int PARTS = (7 + R3 - 1) / R3;
    static constexpr int R2 = R3 + 2, R1 = 2 * R3 + 6, PR = 4 * R1 + 4;   // rows of conv2, conv1, pixels
    static constexpr int M1 = R1 * 20, M2 = R2 * 9, M3 = R3 * 7;
    static constexpr int T1 = (M1 + 15) / 16, T2 = (M2 + 31) / 32, T3 = (M3 + 31) / 32;
    static constexpr int CH = PR * 84 / 16, NPX = (4 * CH + 511) / 512;   // 16-byte pieces per frame, per thread
    static constexpr int PXB = 4 * PR * 84 * 2;   // pixels; later conv2's image
    static constexpr int P1 = 208, P2 = 400;      // pixel pitch of the images in bytes
    static constexpr int W1B = 2 * 8 * 3 * 1024;  // conv1's weights, in the image's place until conv1 begins
    static constexpr int I1B = M1 * P1 > W1B ? M1 * P1 : W1B;   // conv1's image; later the partial tiles
    static constexpr int TAB = (2 * MAX_UNITS + 4 + 160) * 4;   // slots, leaf values, total; biases
    static constexpr int LDS = PXB + I1B + TAB + 8 * TURN;
    static_assert(PR * 84 % 16 == 0 && TAB % 16 == 0 && M2 * P2 <= PXB && 24 * T2 * 1024 <= I1B && 24 * T3 * 1024 <= I1B, "LDS layout");
};

// The sums of a wave: leading products and the others, of its NA turns
template <int NA, int T> __device__ __forceinline__ void close_sums(const Acc2 (&acc)[NA][T], v16f (&sum)[T])
{
#pragma unroll
    for (int t = 0; t < T; ++t) {
        v16f hi = acc[0][t].hi, lo = acc[0][t].lo;
        if constexpr (NA == 2) { hi += acc[1][t].hi; lo += acc[1][t].lo; }
        sum[t] = joined(hi, lo);
    }
}

// The partial tiles of the four waves of a channel half: wave kq ends up with rows 8 kq + 4 h + 0..3 of the half
// (accumulator registers 4 kq .. 4 kq + 3), summed in the order own, then the others ascending.
template <int T>
__device__ __forceinline__ void reduce_quarters(const v16f (&acc)[T], v4f (&own)[T], v4f *scratch, int kq, int ch, int lane)
{
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        if (g == kq) {
#pragma unroll
            for (int t = 0; t < T; ++t) own[t] = v4f{acc[t][4 * g], acc[t][4 * g + 1], acc[t][4 * g + 2], acc[t][4 * g + 3]};
        } else {
            v4f *d = scratch + (((g * 3 + (kq < g ? kq : kq - 1)) * 2 + ch) * T) * 64 + lane;
#pragma unroll
            for (int t = 0; t < T; ++t) d[t * 64] = v4f{acc[t][4 * g], acc[t][4 * g + 1], acc[t][4 * g + 2], acc[t][4 * g + 3]};
        }
    }
    sync_lds();
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int t = 0; t < T; ++t) own[t] += scratch[(((kq * 3 + j) * 2 + ch) * T + t) * 64 + lane];
}

// Workgroup bid of G0; the kernel's arguments begin with A.  MANY: it takes one unit after the other; otherwise just one
// (whole samples with a workgroup each: 129 observations 38.2 -> 36.7 us per call, 256 40.7 -> 38.7, a step at 128 191 -> 189).
// HALF (one unit): workgroups 2 b and 2 b + 1 share unit b, the second one finishing the upper half of conv3's channels.
// conv3, bound by its matrix instructions (an output row fills 7 of a tile's 32 columns), is then the work of four waves,
// one per SIMD, and half of its weights stay away; conv1 and conv2 are computed twice, on compute units that would be
// idle.  Acting on one observation 17.9 -> 17.2 us per call, on 3 to 18 0.6 us less each; the same bits.
template <int R3, bool MANY, bool HALF = false>
__device__ __forceinline__ void conv123_body(const Args &A, const int bid, const int G0, uint8_t *lds)
{
    static_assert(!(MANY && HALF), "one unit");
    // The segments are indexed at run time; through the by-value structure that would be a copy in scratch
    // memory, or a select over three times fifteen scalars.  The arguments themselves lie in constant memory.
    typedef const __attribute__((address_space(4))) Args *ArgsPtr;
    const ArgsPtr AP = (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
#define SP_SEG(s) (AP->seg[s])
    using G = Geo<R3>;
    uint8_t *pxb = lds, *img1 = lds + G::PXB;
    bf16_t *px = reinterpret_cast<bf16_t *>(pxb);
    uint8_t *img2 = pxb;
    v4f *scratch = reinterpret_cast<v4f *>(img1);
    int *slots = reinterpret_cast<int *>(lds + G::PXB + G::I1B);
    float *leafv = reinterpret_cast<float *>(slots + MAX_UNITS);   // [MAX_UNITS], then the total
    float *bias = leafv + MAX_UNITS + 4;                           // conv1 [32], conv2 [64], conv3 [64]
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nt = wave & 1, tg = wave >> 1;      // conv1
    const int ch = wave & 1, kq = wave >> 1;      // conv2, conv3
    const int ch3 = HALF ? bid & 1 : ch, kq3 = HALF ? wave & 3 : kq;
    const bool on3 = !HALF || wave < 4;           // has a share of conv3
    int tid = threadIdx.x, lane = tid & 63;
    const int nu = MANY ? (A.units - bid + G0 - 1) / G0 : 1;   // units of this workgroup (>= 1)
    if (A.clear && bid == 0) misc::few_clear(A.clear, tid);

    auto seg_of = [&](int u) { return (A.nseg > 1 && u >= A.seg[1].first) + (A.nseg > 2 && u >= A.seg[2].first); };
    v8bf w1[8][3];
    // this wave's eighth of conv1's weights (channel half wave / 4, steps 2 (wave % 4) ..), on their way to LDS
    v4f w1s[4];
    auto load_w1 = [&](const float *theta) {
        const float *p = theta + net::C1W + (16 * (wave >> 2) + (lane >> 2)) * 256 + 64 * (wave & 3) + 4 * (lane & 3);
#pragma unroll
        for (int q = 0; q < 4; ++q) w1s[q] = *reinterpret_cast<const v4f *>(p + 16 * q);
    };
    // four waves want the same half of them: through LDS they are fetched, and split, once per workgroup
    auto store_w1 = [&] {
#pragma unroll
        for (int q = 0; q < 4; ++q) {   // 16 of a row's 64 elements: half of step q / 2, lane group 2 (q % 2) + piece / 2
            uint8_t *d = img1 + ((2 * wave + (q >> 1)) * 3) * 1024 + ((lane >> 2) + 16 * (2 * (q & 1) + ((lane >> 1) & 1))) * 16 + 8 * (lane & 1);
            const Split4 f = split4(w1s[q]);
#pragma unroll
            for (int pl = 0; pl < 3; ++pl) *reinterpret_cast<uint2 *>(d + pl * 1024) = f.p[pl];
        }
    };
    auto read_w1 = [&] {
        const v8bf *p = reinterpret_cast<const v8bf *>(img1) + nt * 24 * 64 + lane;
#pragma unroll
        for (int s = 0; s < 8; ++s)
#pragma unroll
            for (int q = 0; q < 3; ++q) w1[s][q] = p[(s * 3 + q) * 64];
    };
    u32x4 raw[G::NPX];
    auto load_px = [&](const uint8_t *x, long xs, int shift, int first, int u, int slot) {
        const int ul = u - first, g = ul / G::PARTS, part = ul % G::PARTS;
        const int row0 = part * R3 < 7 - R3 ? part * R3 : 7 - R3;
        const uint8_t *f[4];
        // (the segments' slot lists, ring and sub-rings are one and the same)
        const gbf::c1::Src src{x, xs, A.seg[0].src.idx, A.seg[0].src.cap, shift, A.seg[0].src.sub};
#pragma unroll
        for (int k = 0; k < 4; ++k) f[k] = gbf::c1::frame_ptr(src, g, slot, k) + row0 * (8 * 84);
#pragma unroll
        for (int i = 0; i < G::NPX; ++i) {
            int t = tid + 512 * i;
            if (t > 4 * G::CH - 1) t = 4 * G::CH - 1;
            const int k = t / G::CH;
            const uint8_t *fp = k == 0 ? f[0] : k == 1 ? f[1] : k == 2 ? f[2] : f[3];
            raw[i] = *reinterpret_cast<const u32x4 *>(fp + (t - k * G::CH) * 16);
        }
    };

    int u = HALF ? bid >> 1 : bid;
    int si = seg_of(u);
    // (scalar loads: a select over the three segments' arguments became a table in scratch memory)
    const uint8_t *x0 = SP_SEG(si).src.x;
    const long xs0 = SP_SEG(si).src.xs;
    const int shift0 = SP_SEG(si).src.shift, first0 = SP_SEG(si).first;
    // The first pixels before the weights, which are twenty times as many bytes, where they are known; drawing
    // comes first otherwise, with the weights on their way
    if (!A.draw) load_px(x0, xs0, shift0, first0, u, 0);
    load_w1(SP_SEG(si).theta);
    if (A.draw) {
#pragma unroll 1
        for (int k = 2 * wave; k < nu; k += 16) {
            const int kb = k + 1 < nu ? k + 1 : k;
            // (draw j of a segment is its sample j)
            const int ga = (u + k * G0) / G::PARTS, gb = (u + kb * G0) / G::PARTS, n = A.seg[0].n;
            const int jj[2] = {ga % n, gb % n};
            long sl[2];
            float leaf[2];
            const float total = misc::per_sample_walk<2>(A.samp, jj, lane, sl, leaf);
            if (lane == 0) {
                slots[k] = (int)sl[0];
                slots[kb] = (int)sl[1];
                leafv[k] = leaf[0];
                leafv[kb] = leaf[1];
                if (k == 0) leafv[MAX_UNITS] = total;
            }
        }
        sync_lds();   // the slot table is complete
        load_px(x0, xs0, shift0, first0, u, slots[0]);
    }
    if (A.draw && wave == 7)   // index, raw importance weight and transition data of the segment-0 draws
        for (int k = lane; k < nu; k += 64) {
            const int uk = u + k * G0;
            if (uk < A.seg[0].n * G::PARTS && uk % G::PARTS == 0)
                misc::per_sample_emit(A.samp, uk / G::PARTS, slots[k], leafv[MAX_UNITS], leafv[k]);
        }

    for (int k = 0; k < nu; ++k) {
        // opaque, so that the lane addresses of all phases are formed where they are used and do not occupy
        // registers throughout the loop
        asm volatile("" : "+v"(tid));
        lane = tid & 63;
        const int n16 = lane & 15, kg = lane >> 4, i32 = lane & 31, h = lane >> 5;
        const int ul = u - SP_SEG(si).first, g = ul / G::PARTS, part = ul % G::PARTS;
        const int row0 = part * R3 < 7 - R3 ? part * R3 : 7 - R3;
        const float *const theta = SP_SEG(si).theta;
        const int rowp = part == 0 ? -32 : (part - 1) * R3;   // first conv3 row of the part before this one (none: far above)
        // a wave may still be in the last phase of the unit before, which reads that unit's biases: with units of two
        // networks in one workgroup they are others
        if (MANY && k > 0) sync_lds();
        if (tid < 160) bias[tid] = theta[tid < 32 ? net::C1B + tid : tid < 96 ? net::C2B + tid - 32 : net::C3B + tid - 96];
        // pixels -> LDS
#pragma unroll
        for (int i = 0; i < G::NPX; ++i) {
            const int t = tid + 512 * i;
            if (t < 4 * G::CH) {
                uint4 *d = reinterpret_cast<uint4 *>(px + t * 16);
                d[0] = gbf::cvt8_u8(raw[i].x, raw[i].y);
                d[1] = gbf::cvt8_u8(raw[i].z, raw[i].w);
            }
        }
        store_w1();
        sync_lds();
        read_w1();
        sync_lds();   // the weights' place is conv1's image from here on
        v4f w2[8][2], w3[9][2];
        const float *p2 = theta + net::C2W + (32 * ch + (lane >> 2)) * 512 + 128 * kq + 4 * (lane & 3);
        const float *p3 = theta + net::C3W + (32 * ch3 + (lane >> 2)) * 576 + 144 * kq3 + 4 * (lane & 3);
        auto load_w3 = [&](int s) {
            if (!on3) return;
#pragma unroll
            for (int q = 0; q < 2; ++q) w3[s][q] = *reinterpret_cast<const v4f *>(p3 + 16 * s + 16 * 576 * q);
        };
        // the weights of a step as they were loaded (row 16 q + lane / 4, piece lane % 4 of four) -> eight of row i32, from
        // 8 h on; the pieces of a row lie permuted by row / 4, so that the lanes that read together meet all banks
        uint8_t *const tw = lds + G::PXB + G::I1B + G::TAB + wave * TURN;
        v4f wr[2];
        auto turn = [&](const v4f (&w)[2]) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int q = 0; q < 2; ++q) *reinterpret_cast<v4f *>(tw + (16 * q + (lane >> 2)) * 64 + (((lane & 3) ^ (lane >> 4)) * 16)) = w[q];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // (LDS operations of a wave complete in order)
#pragma unroll
            for (int q = 0; q < 2; ++q) wr[q] = *reinterpret_cast<const v4f *>(tw + i32 * 64 + (((2 * h + q) ^ ((lane >> 2) & 3)) * 16));
        };
        const int co = 32 * ch + 8 * kq + 4 * h;    // the four channels this lane finishes in conv2, in conv3
        const int co3 = 32 * ch3 + 8 * kq3 + 4 * h;
        __builtin_amdgcn_sched_barrier(0);

        // ---- conv1
        auto conv1_tile = [&](int t) {
            const int m = 16 * t + n16, mc = m < G::M1 ? m : G::M1 - 1;
            const int y = mc / 20, x = mc - 20 * y;
            const bf16_t *p = px + (4 * y + kg) * 84 + 4 * x;
            auto pixels = [&](int s) {   // frame s / 2, kernel rows 4 (s % 2) + kg
                return __builtin_bit_cast(v8bf, *reinterpret_cast<const u32x4_a8 *>(p + (s >> 1) * (G::PR * 84) + (s & 1) * (4 * 84)));
            };
            v4f hi = {0, 0, 0, 0}, lo0 = {0, 0, 0, 0}, lo1 = {0, 0, 0, 0};
            v8bf b0 = pixels(0), b1 = pixels(1);
#pragma unroll
            for (int s = 0; s < 8; s += 2) {
                const v8bf c0 = b0, c1 = b1;
                if (s < 6) { b0 = pixels(s + 2); b1 = pixels(s + 3); }
                __builtin_amdgcn_sched_barrier(0);
                lo0 = mfma16(w1[s][2], c0, lo0);
                lo1 = mfma16(w1[s + 1][2], c1, lo1);
                hi = mfma16(w1[s][0], c0, hi);
                lo0 = mfma16(w1[s][1], c0, lo0);
                lo1 = mfma16(w1[s + 1][1], c1, lo1);
                hi = mfma16(w1[s + 1][0], c1, hi);
                __builtin_amdgcn_sched_barrier(0);
            }
            constexpr float sc = 1.0f / 255.0f;
            const v4f bias1 = *reinterpret_cast<const v4f *>(bias + 16 * nt + 4 * kg);
            v4f v;
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = fmaxf(joined(hi[r], lo0[r] + lo1[r]) * sc + bias1[r], 0.f);
            if (m < G::M1) {
                const Split4 q = split4(v);
                uint8_t *d = img1 + (y * 20 + (x & 1) * 10 + (x >> 1)) * G::P1 + (16 * nt + 4 * kg) * 2;
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) *reinterpret_cast<uint2 *>(d + pl * 64) = q.p[pl];
            }
        };
        auto load_w2 = [&] {
#pragma unroll
            for (int s = 0; s < 8; ++s)
#pragma unroll
                for (int q = 0; q < 2; ++q) w2[s][q] = *reinterpret_cast<const v4f *>(p2 + 16 * s + 16 * 512 * q);
        };
        // the parts of the next step's weights, formed between the six matrix instructions in front of them
        auto split_next = [&](v8bf (&f)[3]) {
            split8(f, wr[0], wr[1]);
#pragma unroll
            for (int q = 0; q < 6; ++q) {
                __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x2, 8, 0);
            }
        };
        // conv2's first weights: behind the first tile where in front of it they would hold up conv1's own
        if constexpr (MANY) load_w2();
        __builtin_amdgcn_sched_barrier(0);
        conv1_tile(tg);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (!MANY) load_w2();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll 1
        for (int t = tg + 4; t < G::T1; t += 4) conv1_tile(t);
        sync_lds();

        // ---- conv2: kernel row kq
        {
            constexpr int T = G::T2, NA = T == 1 ? 2 : 1;
            const uint8_t *pa[T];
#pragma unroll
            for (int t = 0; t < T; ++t) {
                int m = 32 * t + i32;
                if (m > G::M2 - 1) m = G::M2 - 1;
                const int y = m / 9, x = m - 9 * y;
                pa[t] = img1 + ((2 * y + kq) * 20 + x) * G::P1 + h * 16;
            }
            Acc2 acc[NA][T];
#pragma unroll
            for (int a = 0; a < NA; ++a)
#pragma unroll
                for (int t = 0; t < T; ++t) acc[a][t] = Acc2{v16f{0}, v16f{0}};
            v8bf b[3], nb[3], wp[2][3];
            auto load_b = [&](int i) {
                const int s = i / T, t = i % T, off = (((s >> 1) & 1) * 10 + (s >> 2)) * G::P1 + (s & 1) * 32;
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) nb[pl] = *reinterpret_cast<const v8bf *>(pa[t] + off + pl * 64);
            };
            turn(w2[0]);
            load_b(0);
            split8(wp[0], wr[0], wr[1]);
            turn(w2[1]);
#pragma unroll
            for (int i = 0; i < 8 * T; ++i) {   // the operands of a product are requested before the one before it
                const int s = i / T, t = i % T;
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) b[pl] = nb[pl];
                if (i + 1 < 8 * T) load_b(i + 1);
                if (t == 0 && s > 0) load_w3(s - 1);  // conv3's weights into the registers of step s - 1
                __builtin_amdgcn_sched_barrier(0);
                mfma6(wp[s & 1], b, acc[s % NA][t]);
                if (t == T - 1 && s < 7) split_next(wp[(s + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
                if (t == T - 1 && s < 6) turn(w2[s + 2]);
            }
            load_w3(7);
            load_w3(8);
            v16f sum[T];
            close_sums(acc, sum);
            sync_lds();   // every wave has read conv1's image
            v4f own[T];
            reduce_quarters<T>(sum, own, scratch, kq, ch, lane);
            const v4f bias2 = *reinterpret_cast<const v4f *>(bias + 32 + co);
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const int m = 32 * t + i32;
                v4f v;
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = fmaxf(own[t][r] + bias2[r], 0.f);
                if (m < G::M2) {
                    const Split4 q = split4(v);
                    uint8_t *d = img2 + m * G::P2 + co * 2;
#pragma unroll
                    for (int pl = 0; pl < 3; ++pl) *reinterpret_cast<uint2 *>(d + pl * 128) = q.p[pl];
                }
            }
        }
        // the next unit's pixels
        // (behind the last unit: its own once more, so that the registers are written on every path and do not
        // have to keep their old contents until here)
        const int kn = k + 1 < nu ? k + 1 : k, un = bid + kn * G0, sn = seg_of(un);
        if constexpr (MANY) load_w1(SP_SEG(sn).theta);
        if constexpr (MANY) load_px(SP_SEG(sn).src.x, SP_SEG(sn).src.xs, SP_SEG(sn).src.shift, SP_SEG(sn).first, un, A.draw ? slots[kn] : 0);
        sync_lds();

        // ---- conv3: steps 9 kq .. 9 kq + 8 of 36
        if (!on3) sync_lds();   // the barrier of reduce_quarters
        else {
            constexpr int T = G::T3, NA = T == 1 ? 2 : 1;
            const uint8_t *pa[T];
#pragma unroll
            for (int t = 0; t < T; ++t) {
                int m = 32 * t + i32;
                if (m > G::M3 - 1) m = G::M3 - 1;
                const int y = m / 7, x = m - 7 * y;
                pa[t] = img2 + (y * 9 + x) * G::P2 + h * 16;
            }
            Acc2 acc[NA][T];
#pragma unroll
            for (int a = 0; a < NA; ++a)
#pragma unroll
                for (int t = 0; t < T; ++t) acc[a][t] = Acc2{v16f{0}, v16f{0}};
            v8bf b[3], nb[3], wp[2][3];
            auto load_b = [&](int i) {
                const int s = i / T, t = i % T, sg = 9 * kq3 + s, tap = sg >> 2;
                const int off = ((tap / 3) * 9 + tap % 3) * G::P2 + (sg & 3) * 32;
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) nb[pl] = *reinterpret_cast<const v8bf *>(pa[t] + off + pl * 128);
            };
            turn(w3[0]);
            load_b(0);
            split8(wp[0], wr[0], wr[1]);
            turn(w3[1]);
#pragma unroll
            for (int i = 0; i < 9 * T; ++i) {
                const int s = i / T, t = i % T;
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) b[pl] = nb[pl];
                if (i + 1 < 9 * T) load_b(i + 1);
                __builtin_amdgcn_sched_barrier(0);
                mfma6(wp[s & 1], b, acc[s % NA][t]);
                if (t == T - 1 && s < 8) split_next(wp[(s + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
                if (t == T - 1 && s < 7) turn(w3[s + 2]);
            }
            v16f sum[T];
            close_sums(acc, sum);
            v4f own[T];
            reduce_quarters<T>(sum, own, scratch, kq3, ch3, lane);
            const v4f bias3 = *reinterpret_cast<const v4f *>(bias + 96 + co3);
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const int m = 32 * t + i32, y = m / 7;
                v4f v;
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = fmaxf(own[t][r] + bias3[r], 0.f);
                if (m < G::M3 && row0 + y >= rowp + R3)
                    *reinterpret_cast<v4f *>(SP_SEG(si).y3 + (long)g * net::A3 + (row0 * 7 + m) * 64 + co3) = v;
            }
        }
        if (!MANY) break;
        si = sn;
        u += G0;
    }
#undef SP_SEG
}

template <int R3, bool MANY, bool HALF = false>
__global__ __launch_bounds__(512, 1) void k_conv123_fwd(Args A)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    conv123_body<R3, MANY, HALF>(A, (int)blockIdx.x, (int)gridDim.x, lds);
}

// ---------------------------------------------------------------------------
// The same three layers of the pass on s of a training step, in the order of summation that the layers' own launches
// have (gbf::c1::k_conv1_fwd_f32, g32::k_fwd): its stored activations are what the backward pass takes its ReLU
// decisions on, and a decision on a pre-activation that is zero to within the rounding of its sum falls by the
// order of that sum.  In the split form one batch of 32 in thirty had a decision fall the other way and its gradient
// 1e-4 to 7e-2 of its norm off; in this order the activations are those launches' bit for bit.
// Beside the passes over s' (conv123_body) in one launch: a unit, R3 rows of conv3's output, has a compute unit to itself,
// and with R3 = 2 it takes about as long as theirs: 24 us alone, 27 beside 64 samples of s' (20 us).  Bound by the fp32
// matrix pipe (16x16x4: 32 cycles for 1024 products, 31,200 cycles for R3 = 2) and the round trips between the layers.  Of
// the first form's 32 us, 5 were weights that all waves asked for at once: conv1's now go through LDS, conv2's are
// requested behind the first tile, conv3's three at a time beside conv2's steps.  16-wide tiles waste a quarter of conv2's
// and an eighth of conv3's work where 32-wide ones waste almost half.
//   conv1   wave = (channel half, every fourth tile of 16 positions); the pixels lie in LDS as floats
//   conv2   wave = (channel half, kernel column), rows in order; then the four columns' sums in order
//   conv3   twelve tiles (16 channels, every third 32 of the reduction) over eight waves, three sums in order
// A 32x32x2 instruction of those launches adds products k and k + 4 of eight; the four of a 16x16x4 one are therefore
// k = 0, 4, 1, 5, then 2, 6, 3, 7: the images hold sixteen channels in that order (a lane's share is 16 bytes), the
// weights, sixteen natural bytes per lane, are brought into it by exchanging halves of registers.
// ---------------------------------------------------------------------------
struct NatArgs {
    gbf::c1::Src src;
    const float *w1, *b1, *w2, *b2, *w3, *b3;
    float *y1, *y2, *y3;
    int halves;   // conv1 sums frames 0-1 and 2-3 apart
};
struct StepArgs {
    Args split;   // the passes over s'
    NatArgs nat;
    int nat_blocks;
};
template <int R3> struct NatGeo {
    static constexpr int PARTS = (7 + R3 - 1) / R3;
    static constexpr int R2 = R3 + 2, R1 = 2 * R3 + 6, PR = 4 * R1 + 4;   // rows of conv2, conv1, pixels
    static constexpr int M1 = R1 * 20, M2 = R2 * 9, M3 = R3 * 7;
    static constexpr int T1 = (M1 + 15) / 16, T2 = (M2 + 15) / 16, T3 = (M3 + 15) / 16;
    static constexpr int CH = PR * 84 / 16, NPX = (4 * CH + 511) / 512;
    static constexpr int P1 = 36, P2 = 68;                                // pixel pitch of the images in floats
    static constexpr int PXB = 4 * PR * 84 * 4, I1B = M1 * P1 * 4, I2B = M2 * P2 * 4, LDS = PXB + I1B + I2B + 16;
    static_assert(PR * 84 % 16 == 0 && 16 * T2 * 1024 <= PXB && 12 * T3 * 1024 <= PXB, "LDS layout");
    static_assert(I1B + I2B >= 32 * 1024, "conv1's weights");
    static_assert(4 * T3 <= 8, "one finishing tile of conv3 per wave");
};

using gbf::c1::mfma4;
// channels 4 kg .. 4 kg + 3 of sixteen -> this lane's share in the order above
__device__ __forceinline__ v4f lane_share(v4f w)
{
    const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(w.x), __float_as_uint(w.y), false, false);
    const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(w.z), __float_as_uint(w.w), false, false);
    return v4f{__uint_as_float(p[0]), __uint_as_float(q[0]), __uint_as_float(p[1]), __uint_as_float(q[1])};
}
// channels 4 kg .. + 3 of a position -> the image's sixteen
__device__ __forceinline__ void put_share(float *d, int kg, v4f v)
{
    float *e = d + (kg & 1) * 4 + (kg >> 1) * 2;
    *reinterpret_cast<float2 *>(e) = float2{v.x, v.z};
    *reinterpret_cast<float2 *>(e + 8) = float2{v.y, v.w};
}

template <int R3>
__device__ __forceinline__ void conv123_native_body(const NatArgs &A, const bool draw, const misc::SampleArgs &samp, const int bid, uint8_t *lds)
{
    using G = NatGeo<R3>;
    float *px = reinterpret_cast<float *>(lds), *img1 = reinterpret_cast<float *>(lds + G::PXB);
    float *img2 = reinterpret_cast<float *>(lds + G::PXB + G::I1B);
    int *slot_tab = reinterpret_cast<int *>(lds + G::PXB + G::I1B + G::I2B);
    v4f *scratch = reinterpret_cast<v4f *>(lds);   // the pixels' place, behind conv1
    const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, kg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = bid / G::PARTS, part = bid % G::PARTS;
    const int row0 = part * R3 < 7 - R3 ? part * R3 : 7 - R3;
    const int rowp = part == 0 ? -32 : (part - 1) * R3;   // first conv3 row of the part before this one (none: far above)

    u32x4 raw[G::NPX];
    auto load_px = [&](int slot) {
        const uint8_t *f[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) f[k] = gbf::c1::frame_ptr(A.src, g, slot, k) + row0 * (8 * 84);
#pragma unroll
        for (int i = 0; i < G::NPX; ++i) {
            int t = tid + 512 * i;
            if (t > 4 * G::CH - 1) t = 4 * G::CH - 1;
            const int k = t / G::CH;
            const uint8_t *fp = k == 0 ? f[0] : k == 1 ? f[1] : k == 2 ? f[2] : f[3];
            raw[i] = *reinterpret_cast<const u32x4 *>(fp + (t - k * G::CH) * 16);
        }
    };
    if (!draw) load_px(0);
    const int nt = wave & 1, tg = wave >> 1;
    // conv1's weights, an eighth per wave: fragment f = channel half f / 16; frame and kernel rows of pair f % 16 / 2,
    // columns 4 (f % 2) ..; through LDS to the four waves that want them
    v4f w1s[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int f = 4 * wave + q, s = (f >> 1) & 7;
        w1s[q] = *reinterpret_cast<const v4f *>(A.w1 + (16 * (f >> 4) + n) * 256 + (s >> 1) * 64 + (4 * (s & 1) + kg) * 8 + 4 * (f & 1));
    }
    const v4f bias1 = *reinterpret_cast<const v4f *>(A.b1 + 16 * nt + 4 * kg);
    const v4f bias2 = *reinterpret_cast<const v4f *>(A.b2 + 16 * (wave & 3) + 4 * kg);
    const v4f bias3 = *reinterpret_cast<const v4f *>(A.b3 + 16 * (wave & 3) + 4 * kg);
    if (draw) {
        if (wave == 0) {
            const int jj[2] = {g, g};
            long sl[2];
            float leaf[2];
            misc::per_sample_walk<2>(samp, jj, lane, sl, leaf);
            if (lane == 0) slot_tab[0] = (int)sl[0];
        }
        sync_lds();
        load_px(slot_tab[0]);
    }
    const int ch = wave & 1, kq = wave >> 1;
    v4f *wl = reinterpret_cast<v4f *>(img1);
#pragma unroll
    for (int q = 0; q < 4; ++q) wl[(4 * wave + q) * 64 + lane] = w1s[q];
#pragma unroll
    for (int i = 0; i < G::NPX; ++i) {
        const int t = tid + 512 * i;
        if (t < 4 * G::CH) {
            v4f *d = reinterpret_cast<v4f *>(px + t * 16);
#pragma unroll
            for (int j = 0; j < 4; ++j) d[j] = g32::cvt4((uint32_t)raw[i][j]);
        }
    }
    sync_lds();
    v4f w1[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) w1[q] = wl[(16 * nt + q) * 64 + lane];
    sync_lds();   // the weights' place is conv1's image from here on

    // ---- conv1
    auto conv1_tile = [&](int t) {
        const int m = 16 * t + n, mc = m < G::M1 ? m : G::M1 - 1, y = mc / 20, x = mc - 20 * y;
        const float *p = px + (4 * y + kg) * 84 + 4 * x;
        v4f acc = {0, 0, 0, 0}, first = {0, 0, 0, 0}, b[2], nb[2];
        auto load_b = [&](int s) {
            const float *q = p + (s >> 1) * (G::PR * 84) + (s & 1) * (4 * 84);
            nb[0] = *reinterpret_cast<const v4f *>(q);
            nb[1] = *reinterpret_cast<const v4f *>(q + 4);
        };
        load_b(0);
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            b[0] = nb[0];
            b[1] = nb[1];
            if (s < 7) load_b(s + 1);
            __builtin_amdgcn_sched_barrier(0);
            if (s == 4 && A.halves) {
                first = acc;
                acc = v4f{0, 0, 0, 0};
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) acc = mfma4(w1[2 * s + (e >> 2)][e & 3], b[e >> 2][e & 3], acc);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (A.halves) acc = first + acc;
        constexpr float sc = 1.0f / 255.0f;
        v4f v;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = fmaxf(acc[r] * sc + bias1[r], 0.f);
        if (m < G::M1) {
            put_share(img1 + m * G::P1 + 16 * nt, kg, v);
            if (2 * row0 + y >= 2 * rowp + G::R1)
                *reinterpret_cast<v4f *>(A.y1 + (long)g * net::A1 + ((2 * row0 + y) * 20 + x) * 32 + 16 * nt + 4 * kg) = v;
        }
    };
    conv1_tile(tg);
    __builtin_amdgcn_sched_barrier(0);
    v4f w2[8][2];   // step s: kernel row s / 2, channels 16 (s % 2) ..
#pragma unroll
    for (int s = 0; s < 8; ++s)
#pragma unroll
        for (int c = 0; c < 2; ++c)
            w2[s][c] = *reinterpret_cast<const v4f *>(A.w2 + (32 * ch + 16 * c + n) * 512 + (s >> 1) * 128 + kq * 32 + 16 * (s & 1) + 4 * kg);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll 1
    for (int t = tg + 4; t < G::T1; t += 4) conv1_tile(t);
    sync_lds();

    // ---- conv2: kernel column kq
    // conv3's: [c][s] = slice c ? 2 : wave / 4, step s: products 32 (3 (s / 2) + slice) + 16 (s % 2) .. of channels
    // 16 (wave % 4) ..; requested three at a time beside conv2's steps
    v4f w3[2][12];
    const float *p3 = A.w3 + (16 * (wave & 3) + n) * 576 + 4 * kg;
    auto load_w3 = [&](int c, int s) { w3[c][s] = *reinterpret_cast<const v4f *>(p3 + 32 * (c ? 2 : wave >> 2) + 96 * (s >> 1) + 16 * (s & 1)); };
    {
        constexpr int T = G::T2;
        const float *pa[T];
        v4f acc[T][2];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            int m = 16 * t + n;
            if (m > G::M2 - 1) m = G::M2 - 1;
            const int y = m / 9, x = m - 9 * y;
            pa[t] = img1 + (40 * y + 2 * x + kq) * G::P1 + 4 * kg;
            acc[t][0] = acc[t][1] = v4f{0, 0, 0, 0};
        }
        v4f b[T], nb[T];
        auto load_b = [&](int s) {
#pragma unroll
            for (int t = 0; t < T; ++t) nb[t] = *reinterpret_cast<const v4f *>(pa[t] + (s >> 1) * (20 * G::P1) + 16 * (s & 1));
        };
        load_b(0);
#pragma unroll
        for (int s = 0; s < 8; ++s) {
#pragma unroll
            for (int t = 0; t < T; ++t) b[t] = nb[t];
            if (s < 7) load_b(s + 1);
#pragma unroll
            for (int q = 3 * s; q < 3 * s + 3; ++q) load_w3(q / 12, q % 12);
            const v4f wa = lane_share(w2[s][0]), wb = lane_share(w2[s][1]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    acc[t][0] = mfma4(wa[e], b[t][e], acc[t][0]);
                    acc[t][1] = mfma4(wb[e], b[t][e], acc[t][1]);
                }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int c = 0; c < 2; ++c) scratch[((kq * 4 + 2 * ch + c) * T + t) * 64 + lane] = acc[t][c];
        sync_lds();
#pragma unroll
        for (int t = wave >> 2; t < T; t += 2) {   // channels 16 (wave % 4) .., every other tile
            v4f sum = scratch[((wave & 3) * T + t) * 64 + lane];
#pragma unroll
            for (int k = 1; k < 4; ++k) sum += scratch[((k * 4 + (wave & 3)) * T + t) * 64 + lane];
            v4f v;
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = fmaxf(sum[r] + bias2[r], 0.f);
            const int m = 16 * t + n;
            if (m < G::M2) {
                put_share(img2 + m * G::P2 + 16 * (wave & 3), kg, v);
                if (row0 + m / 9 >= rowp + G::R2)
                    *reinterpret_cast<v4f *>(A.y2 + (long)g * net::A2 + (row0 * 9 + m) * 64 + 16 * (wave & 3) + 4 * kg) = v;
            }
        }
    }
    sync_lds();

    // ---- conv3: a slice is 32 products of every 96
    {
        constexpr int T = G::T3;
        const float *pa[T];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            int m = 16 * t + n;
            if (m > G::M3 - 1) m = G::M3 - 1;
            const int y = m / 7, x = m - 7 * y;
            pa[t] = img2 + (9 * y + x) * G::P2 + 4 * kg;
        }
        auto slices = [&](auto count) {
            constexpr int C = decltype(count)::value;
            v4f acc[C][T], b[C][T], nb[C][T];
            auto load_b = [&](int s) {
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    const int j = 3 * (s >> 1) + (c ? 2 : wave >> 2), tap = j >> 1;
                    const int off = ((tap / 3) * 9 + tap % 3) * G::P2 + 32 * (j & 1) + 16 * (s & 1);
#pragma unroll
                    for (int t = 0; t < T; ++t) nb[c][t] = *reinterpret_cast<const v4f *>(pa[t] + off);
                }
            };
#pragma unroll
            for (int c = 0; c < C; ++c)
#pragma unroll
                for (int t = 0; t < T; ++t) acc[c][t] = v4f{0, 0, 0, 0};
            load_b(0);
#pragma unroll
            for (int s = 0; s < 12; ++s) {
                v4f wa[C];
#pragma unroll
                for (int c = 0; c < C; ++c) {
#pragma unroll
                    for (int t = 0; t < T; ++t) b[c][t] = nb[c][t];
                    wa[c] = lane_share(w3[c][s]);
                }
                if (s < 11) load_b(s + 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int c = 0; c < C; ++c)
#pragma unroll
                        for (int t = 0; t < T; ++t) acc[c][t] = mfma4(wa[c][e], b[c][t][e], acc[c][t]);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int c = 0; c < C; ++c)
#pragma unroll
                for (int t = 0; t < T; ++t) scratch[(((c ? 2 : wave >> 2) * 4 + (wave & 3)) * T + t) * 64 + lane] = acc[c][t];
        };
        // waves 0-3: slices 0 and 2, waves 4-7: slice 1, so that every SIMD has three of the twelve
        if (wave < 4) slices(std::integral_constant<int, 2>{});
        else slices(std::integral_constant<int, 1>{});
        sync_lds();
        const int t = wave >> 2;
        if (t < T) {
            v4f sum = scratch[((wave & 3) * T + t) * 64 + lane];
#pragma unroll
            for (int k = 1; k < 3; ++k) sum += scratch[((k * 4 + (wave & 3)) * T + t) * 64 + lane];
            v4f v;
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = fmaxf(sum[r] + bias3[r], 0.f);
            const int m = 16 * t + n;
            if (m < G::M3 && row0 + m / 7 >= rowp + R3)
                *reinterpret_cast<v4f *>(A.y3 + (long)g * net::A3 + (row0 * 7 + m) * 64 + 16 * (wave & 3) + 4 * kg) = v;
        }
    }
}

// The forward conv layers of a training step's three passes: workgroups [0, nat_blocks) take parts of s, the others of s'.
template <int R3, int RN> constexpr int step_lds() { return Geo<R3>::LDS > NatGeo<RN>::LDS ? Geo<R3>::LDS : NatGeo<RN>::LDS; }
template <int R3, int RN>
__global__ __launch_bounds__(512, 1) void k_conv123_step(StepArgs A)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int bid = (int)blockIdx.x;
    if (bid < A.nat_blocks) conv123_native_body<RN>(A.nat, A.split.draw, A.split.samp, bid, lds);
    else conv123_body<R3, false>(A.split, bid - A.nat_blocks, (int)gridDim.x - A.nat_blocks, lds);
}

// ---------------------------------------------------------------------------
// The backward pass.  Operands are fp32 in memory; a thread splits what it has loaded on the way into LDS (22
// vector instructions per four values), where an operand tile lies three times, once per part.  A 16-deep
// step of a 32 x 32 block reads six fragments for six products, half the LDS bytes per product of a plain
// bf16 tile.
// ---------------------------------------------------------------------------
constexpr int BK = 32;           // reduction elements per stage of a weight-gradient tile

// four values into the three part tiles (PS elements apart)
template <int PS> __device__ __forceinline__ void put4(bf16_t *p, v4f v)
{
    const Split4 s = split4(v);
#pragma unroll
    for (int q = 0; q < 3; ++q) *reinterpret_cast<uint2 *>(p + q * PS) = s.p[q];
}
template <int PS> __device__ __forceinline__ void get_tr(v8bf (&f)[3], const bf16_t *p, int ld)
{
#pragma unroll
    for (int q = 0; q < 3; ++q) f[q] = gbf::frag_tr(p + q * PS, ld);
}

// Weight gradient (see g32::wgrad_tile): output channels [by*BMO, +BMO) x im2col columns [bx*BNK, +BNK) over the rows
// of split bz.  Both operands have the reduction as their slow dimension: LDS transpose loads.
template <int BMO, int BNK> constexpr int wgrad_lds() { return 3 * BK * (BMO + 8 + BNK + 8); }   // elements
template <class G, int BMO, int BNK, int WM, int WN>
__device__ __forceinline__ void wgrad_tile(const g32::WgradArgs &A, int bx, int by, int bz, bf16_t *lds)
{
    constexpr int WAVES_M = BMO / (32 * WM), WAVES_N = BNK / (32 * WN), T = WAVES_M * WAVES_N * 64;
    constexpr int LDY = BMO + 8, LDX = BNK + 8, PY = BK * LDY, PX = BK * LDX;
    constexpr int YR = T / (BMO / 4), XR = T / (BNK / 4), NY = BK / YR, NX = BK / XR;
    static_assert(NY * YR == BK && NX * XR == BK, "tile/threads mismatch");
    bf16_t *Ys = lds, *Xs = lds + 3 * PY;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int kc0 = bx * BNK, o0 = by * BMO;
    const int mbeg = bz * A.rps, mend = min(mbeg + A.rps, A.B * G::P);
    const float *x = static_cast<const float *>(A.x);
    const int yr = tid / (BMO / 4), yc = (tid % (BMO / 4)) * 4;
    const int xr = tid / (BNK / 4), xc = (tid % (BNK / 4)) * 4;
    const int xko = G::k_off(kc0 + xc);
    v4f ry[NY], rx[NX];
    int left = 0;   // rows of the loaded stage that exist
    auto gload = [&](int mb) {
        left = mend - mb;
#pragma unroll
        for (int i = 0; i < NY; ++i) ry[i] = *reinterpret_cast<const v4f *>(A.dy + (long)min(mb + yr + i * YR, mend - 1) * G::N + o0 + yc);
#pragma unroll
        for (int i = 0; i < NX; ++i) rx[i] = *reinterpret_cast<const v4f *>(x + G::row_off(min(mb + xr + i * XR, mend - 1), A.xs) + xko);
    };
    auto sstore = [&]() {
        // (rows past the end: dY as zeros is enough)
#pragma unroll
        for (int i = 0; i < NY; ++i) put4<PY>(&Ys[(yr + i * YR) * LDY + yc], yr + i * YR < left ? ry[i] : v4f{0, 0, 0, 0});
#pragma unroll
        for (int i = 0; i < NX; ++i) put4<PX>(&Xs[(xr + i * XR) * LDX + xc], rx[i]);
    };
    const int wo = wave % WAVES_M, wk = wave / WAVES_M;
    const int li = lane & 31, h = lane >> 5, s16 = lane & 15, half = (lane >> 4) & 1;
    const int trow = 8 * h + (s16 >> 2), tcol = 16 * half + 4 * (s16 & 3);
    const bf16_t *yp = Ys + trow * LDY + wo * 32 * WM + tcol, *xp = Xs + trow * LDX + wk * 32 * WN + tcol;
    const bool do_bias = bx == 0 && wk == 0;
    Acc2 acc[WM][WN];
    RowSum accb[WM];
#pragma unroll
    for (int a = 0; a < WM; ++a) {
#pragma unroll
        for (int b = 0; b < WN; ++b) acc[a][b] = Acc2{v16f{0}, v16f{0}};
    }
    if (mbeg < mend) gload(mbeg);
    for (int mb = mbeg; mb < mend; mb += BK) {
        if (mb != mbeg) sync_lds();
        sstore();
        if (mb + BK < mend) gload(mb + BK);
        sync_lds();
#pragma unroll
        for (int kk = 0; kk < BK; kk += 16) {
            v8bf fa[WM][3], fb[WN][3];
#pragma unroll
            for (int a = 0; a < WM; ++a) get_tr<PY>(fa[a], yp + kk * LDY + a * 32, LDY);
#pragma unroll
            for (int b = 0; b < WN; ++b) get_tr<PX>(fb[b], xp + kk * LDX + b * 32, LDX);
#pragma unroll
            for (int a = 0; a < WM; ++a) {
#pragma unroll
                for (int b = 0; b < WN; ++b) mfma6(fa[a], fb[b], acc[a][b]);
                if (do_bias) accb[a].add(fa[a]);
            }
        }
    }
    float *part = A.part + (long)bz * A.part_stride;
#pragma unroll
    for (int a = 0; a < WM; ++a)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int o = o0 + (wo * WM + a) * 32 + 8 * (r / 4) + 4 * h + (r % 4);
#pragma unroll
            for (int b = 0; b < WN; ++b) part[(long)o * G::K + kc0 + (wk * WN + b) * 32 + li] = joined(acc[a][b].hi[r], acc[a][b].lo[r]);
            if (do_bias) {   // uniform for the wave
                const float v = accb[a].row(r);
                if (li == 0) part[(long)G::N * G::K + o] = v;
            }
        }
}

// ---------------------------------------------------------------------------
// conv2's input gradient AND conv1's weight gradient of a part of a sample in one workgroup of eight waves:
// conv1's dY is needed by nothing but conv1's weight gradient, position by position, so it goes into LDS, in the
// layout the weight gradient reads, and never to memory.  A unit is 1/P of a sample: 20 / P rows of conv1's
// output, which take the (10 / P) + 1 rows of conv2's dY around them (no work twice).
//   input gradient   32x32x16; wave = (stride parity class, kernel rows py or py + 2): a pixel of a class meets four
//                    taps, a wave two of them: 96 registers of weights, fetched once per workgroup.  The two
//                    halves of the sum meet in LDS, each wave finishing 16 of the 32 channels
//   weight gradient  32x32x16, three products (pixels are exact); wave = (64 of the 256 columns, every other step of 16
//                    positions); the two halves meet once, at the end
// Workgroup b takes units b, b + nblocks, ... and writes one partial of conv1's weight gradient.
// ---------------------------------------------------------------------------
struct BackArgs {
    const float *dy;      // [B][81][64]: gradient w.r.t. conv2's pre-activation
    const float *w;       // conv2's weights
    const float *xact;    // [B][400][32]: conv1's output
    gbf::c1::Src src;     // where the frames of sample n come from
    float *part1;         // [nblocks][32*256 + 32]
    int B;
};
template <int P> struct BackGeo {
    static constexpr int RA = 10 / P, RD = 2 * RA, NPOS = RD * 20, NKS = (NPOS + 15) / 16;
    static constexpr int T = (RA * 10 + 31) / 32;              // tiles of 32 positions of a class
    static constexpr int FRW = 4 * RD + 4, CH = FRW * 84 / 16, NPX = (4 * CH + 511) / 512;
    static constexpr int NDY = ((RA + 1) * 9 * 16 + 511) / 512; // 16-byte pieces of dY per thread
    static constexpr int LDY = 40;                              // row stride (elements) of conv1's dY
    static constexpr int PD = NKS * 16 * LDY;                   // elements of one part of it
    static constexpr int DYS = 3 * PD * 2, IMG = (RA + 1) * 11 * 400, XIN = 4 * FRW * 84 * 2, SCR = 16 * T * 1024;
    static constexpr int SCRB = SCR > 32768 ? SCR : 32768;      // (the final exchange of the weight gradient needs 32 KB)
    static constexpr int LDS = DYS + IMG + XIN + SCRB;
    static_assert(DYS % 16 == 0 && IMG % 16 == 0 && XIN % 16 == 0 && FRW * 84 % 16 == 0 && RD * 4 * 84 % 16 == 0, "LDS layout");
};

template <int P>
__device__ __forceinline__ void conv2_dgrad_conv1_wgrad_body(const BackArgs &A, int bid, int nblocks, uint8_t *lds)
{
    using G = BackGeo<P>;
    bf16_t *dys = reinterpret_cast<bf16_t *>(lds), *xin = reinterpret_cast<bf16_t *>(lds + G::DYS + G::IMG);
    uint8_t *img = lds + G::DYS;
    v4f *scr = reinterpret_cast<v4f *>(lds + G::DYS + G::IMG + G::XIN);
    int tid = threadIdx.x, lane = tid & 63, i32 = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int py = (wave >> 1) & 1, px = wave & 1, kh = wave >> 2, cls = wave & 3;
    const int units = A.B * P;
    if (bid >= units) return;

    v4f rdy[G::NDY];
    u32x4 raw[G::NPX];
    auto load_unit = [&](int u, int slot) {
        const int g = u / P, part = u % P;
        const float *d = A.dy + (long)g * net::A2;
#pragma unroll
        for (int i = 0; i < G::NDY; ++i) {   // piece e: row e / 144, column and channels e % 144
            const int e = tid + 512 * i, r = part * G::RA - 1 + e / 144;
            const bool in = e < (G::RA + 1) * 144 && r >= 0 && r < 9;
            rdy[i] = *reinterpret_cast<const v4f *>(d + (in ? r * 576 + (e % 144) * 4 : 0));
        }
        const uint8_t *f[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) f[k] = gbf::c1::frame_ptr(A.src, g, slot, k) + part * (G::RD * 4 * 84);
#pragma unroll
        for (int i = 0; i < G::NPX; ++i) {
            int t = tid + 512 * i;
            if (t > 4 * G::CH - 1) t = 4 * G::CH - 1;
            const int k = t / G::CH;
            const uint8_t *fp = k == 0 ? f[0] : k == 1 ? f[1] : k == 2 ? f[2] : f[3];
            raw[i] = *reinterpret_cast<const u32x4 *>(fp + (t - k * G::CH) * 16);
        }
    };
    const int slot0 = gbf::c1::sample_slot(A.src, bid / P);
    v8bf wa[8][3];   // step s: kernel column px + 2 (s / 4), output channels 16 (s % 4) ..
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        const float *p = A.w + (16 * (s & 3) + 8 * h) * 512 + ((py + 2 * kh) * 4 + px + 2 * (s >> 2)) * 32 + i32;
        v4f lo, hi;
#pragma unroll
        for (int e = 0; e < 4; ++e) { lo[e] = p[e * 512]; hi[e] = p[(e + 4) * 512]; }
        split8(wa[s], lo, hi);
    }
    load_unit(bid, slot0);
    int slot_next = bid + nblocks < units ? gbf::c1::sample_slot(A.src, (bid + nblocks) / P) : 0;
    // zeros once: the image's border columns, and the rows of conv1's dY past the last position
    for (int i = tid; i < G::IMG / 16; i += 512) *reinterpret_cast<u32x4 *>(img + i * 16) = u32x4{0, 0, 0, 0};
    for (int i = tid; i < 3 * (G::NKS * 16 - G::NPOS) * G::LDY / 2; i += 512) {
        constexpr int W = (G::NKS * 16 - G::NPOS) * G::LDY / 2;   // words per part
        reinterpret_cast<uint32_t *>(dys)[(W ? i / (W ? W : 1) : 0) * (G::PD / 2) + G::NPOS * G::LDY / 2 + (W ? i % (W ? W : 1) : 0)] = 0;
    }

    v16f wacc[2] = {v16f{0}, v16f{0}};
    RowSum accb;
    const int cp = wave & 3;   // weight gradient: columns 64 cp .. (frame cp)
    const bool do_bias = cp == 0;

    for (int u = bid; u < units; u += nblocks) {
        asm volatile("" : "+v"(tid));   // opaque: see k_conv123_fwd
        lane = tid & 63; i32 = lane & 31; h = lane >> 5;
        const int g = u / P, part = u % P;
        sync_lds();   // the unit before has been read (the first time: the zeros are there)
#pragma unroll
        for (int i = 0; i < G::NDY; ++i) {
            const int e = tid + 512 * i, lr = e / 144, r = part * G::RA - 1 + lr, c = (e % 144) >> 4, ch = (e & 15) * 4;
            if (e < (G::RA + 1) * 144) {
                const Split4 q = split4(r >= 0 && r < 9 ? rdy[i] : v4f{0, 0, 0, 0});
                uint8_t *d = img + (lr * 11 + c + 1) * 400 + ch * 2;
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) *reinterpret_cast<uint2 *>(d + pl * 128) = q.p[pl];
            }
        }
#pragma unroll
        for (int i = 0; i < G::NPX; ++i) {
            const int t = tid + 512 * i;
            if (t < 4 * G::CH) {
                uint4 *d = reinterpret_cast<uint4 *>(xin + t * 16);
                d[0] = gbf::cvt8_u8(raw[i].x, raw[i].y);
                d[1] = gbf::cvt8_u8(raw[i].z, raw[i].w);
            }
        }
        const int un = u + nblocks < units ? u + nblocks : u;   // (the last unit once more: the registers are written on every path)
        load_unit(un, slot_next);
        slot_next = u + 2 * nblocks < units ? gbf::c1::sample_slot(A.src, (u + 2 * nblocks) / P) : 0;
        // conv1's activations (the ReLU mask) of the 16 channels this wave finishes
        v4f xm[G::T][2];
        int pos[G::T];
#pragma unroll
        for (int t = 0; t < G::T; ++t) {
            const int m = 32 * t + i32, mc = m < G::RA * 10 ? m : G::RA * 10 - 1, a = mc / 10, b = mc - 10 * a;
            pos[t] = (2 * a + py) * 20 + 2 * b + px;
            const float *p = A.xact + (long)g * net::A1 + (part * G::NPOS + pos[t]) * 32 + 16 * kh + 4 * h;
#pragma unroll
            for (int j = 0; j < 2; ++j) xm[t][j] = *reinterpret_cast<const v4f *>(p + 8 * j);
        }
        sync_lds();   // image and frames are complete

        // ---- conv2's input gradient
        Acc2 acc[G::T];
        const uint8_t *pa[G::T];
#pragma unroll
        for (int t = 0; t < G::T; ++t) {
            acc[t] = Acc2{v16f{0}, v16f{0}};
            const int m = 32 * t + i32, mc = m < G::RA * 10 ? m : G::RA * 10 - 1, a = mc / 10, b = mc - 10 * a;
            pa[t] = img + ((a + 1 - kh) * 11 + b + 1) * 400 + h * 16;   // position (a - kh, b) of dY
        }
        v8bf b3[3], nb[3];
        auto load_b = [&](int i) {
            const int s = i / G::T, t = i % G::T, off = -(s >> 2) * 400 + (s & 3) * 32;
#pragma unroll
            for (int pl = 0; pl < 3; ++pl) nb[pl] = *reinterpret_cast<const v8bf *>(pa[t] + off + pl * 128);
        };
        load_b(0);
#pragma unroll
        for (int i = 0; i < 8 * G::T; ++i) {
#pragma unroll
            for (int pl = 0; pl < 3; ++pl) b3[pl] = nb[pl];
            if (i + 1 < 8 * G::T) load_b(i + 1);
            __builtin_amdgcn_sched_barrier(0);
            mfma6(wa[i / G::T], b3, acc[i % G::T]);
            __builtin_amdgcn_sched_barrier(0);
        }
        // accumulator register 4g + r = channel 8g + 4h + r; the wave keeps g = 2 kh, 2 kh + 1 and hands over the others
        v4f own[G::T][2];
#pragma unroll
        for (int t = 0; t < G::T; ++t)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const v16f s = joined(acc[t].hi, acc[t].lo);
                const v4f lo = {s[4 * j], s[4 * j + 1], s[4 * j + 2], s[4 * j + 3]};
                const v4f hi = {s[4 * j + 8], s[4 * j + 9], s[4 * j + 10], s[4 * j + 11]};
                own[t][j] = kh ? hi : lo;
                scr[(((cls * 2 + (kh ^ 1)) * G::T + t) * 2 + j) * 64 + lane] = kh ? lo : hi;
            }
        sync_lds();
#pragma unroll
        for (int t = 0; t < G::T; ++t)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                v4f v = own[t][j] + scr[(((cls * 2 + kh) * G::T + t) * 2 + j) * 64 + lane];
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = xm[t][j][r] > 0.f ? v[r] : 0.f;
                if (32 * t + i32 < G::RA * 10) put4<G::PD>(dys + pos[t] * G::LDY + 16 * kh + 8 * j + 4 * h, v);
            }
        sync_lds();   // conv1's dY is complete

        // ---- conv1's weight gradient: frame cp, kernel rows 0 - 3 and 4 - 7, steps kh, kh + 2, ...
        const int s16 = lane & 15, half = (lane >> 4) & 1, rsub = 8 * h + (s16 >> 2);
        const int kc = 16 * half + 4 * (s16 & 3);
        const bf16_t *yp = dys + rsub * G::LDY + 16 * half + 4 * (s16 & 3);
        const bf16_t *xw = xin + cp * (G::FRW * 84) + (kc >> 3) * 84 + (kc & 7);
        typedef __attribute__((address_space(3))) gbf::v4s *lds_v4s;
        auto pixel = [&](int p) {   // window of position p (clamped: past the last one dY is zero)
            if (G::NPOS % 16 != 0) p = p < G::NPOS ? p : G::NPOS - 1;
            const int y = p / 20;
            return 336 * y + 4 * (p - 20 * y);
        };
        v16f lo2[2] = {v16f{0}, v16f{0}};   // of this unit: see Acc2
#pragma unroll
        for (int t2 = 0; t2 < (G::NKS + 1) / 2; ++t2) {
            const int t = 2 * t2 + kh;
            if (t >= G::NKS) break;   // uniform for the wave
            v8bf fa[3], fb[2];
            get_tr<G::PD>(fa, yp + 16 * t * G::LDY, G::LDY);
            const bf16_t *x0 = xw + pixel(16 * t + rsub), *x1 = xw + pixel(16 * t + rsub + 4);
#pragma unroll
            for (int b = 0; b < 2; ++b) {   // 32 columns = four kernel rows
                const gbf::v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(x0 + b * 336));
                const gbf::v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(x1 + b * 336));
                typedef short v8s __attribute__((ext_vector_type(8)));
                const v8s xb = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
                fb[b] = __builtin_bit_cast(v8bf, xb);
            }
            mfma3(fa, fb[0], wacc[0], lo2[0]);
            mfma3(fa, fb[1], wacc[1], lo2[1]);
            if (do_bias) accb.add(fa);
        }
        wacc[0] = joined(wacc[0], lo2[0]);
        wacc[1] = joined(wacc[1], lo2[1]);
    }
    float bsum[16];
    if (do_bias)   // uniform for the wave
#pragma unroll
        for (int r = 0; r < 16; ++r) bsum[r] = accb.row(r);
    // the odd steps join the even ones
    float *sf = reinterpret_cast<float *>(scr);
    float *part = A.part1 + (long)bid * (32 * 256 + 32);
    if (kh == 1) {
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) sf[((cp * 2 + b) * 16 + r) * 64 + lane] = wacc[b][r];
        if (do_bias && i32 == 0) {
            // (every column holds the sums; conv1's dY is no longer read)
#pragma unroll
            for (int r = 0; r < 16; ++r) reinterpret_cast<float *>(img)[16 * h + r] = bsum[r];
        }
    }
    sync_lds();
    if (kh == 0) {
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int o = 8 * (r / 4) + 4 * h + (r % 4);
                part[o * 256 + 64 * cp + 32 * b + i32] = (wacc[b][r] + sf[((cp * 2 + b) * 16 + r) * 64 + lane]) * (1.0f / 255.0f);
            }
        if (do_bias && i32 == 0) {
#pragma unroll
            for (int r = 0; r < 16; ++r) part[32 * 256 + 8 * (r / 4) + 4 * h + (r % 4)] = bsum[r] + reinterpret_cast<float *>(img)[16 * h + r];
        }
    }
}

}  // namespace sp

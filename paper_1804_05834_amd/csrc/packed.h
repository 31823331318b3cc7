// The conv weights in the order in which the matrix instructions of the fused forward launches take them: as
// sums of three bf16 numbers for the fp32 network (see gemm_split.h for the arithmetic), as they are for the
// bf16 network.  RMSProp keeps the copy of the online network up to date.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "net.h"

namespace sp {

__device__ __forceinline__ uint16_t bf16_bits(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }   // nearest even
__device__ __forceinline__ float bf16_value(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// ---------------------------------------------------------------------------
// The conv weights as bf16 parts, in the order in which the forward kernel's waves read them: a
// fragment is what one matrix instruction takes, 64 lanes x 16 bytes one after the other, so that a
// fragment is one coalesced 1 KB load.
//   conv1: [channel half 16][step of 32][part]          16x16x32 operand: lane = channel + 16 * (k / 8)
//   conv2: [kernel row][channel half 32][step of 16][part]  32x32x16 operand: lane = channel + 32 * (k / 8)
//   conv3: [quarter of 9 steps][channel half 32][step of 16][part]
// and once more for conv2's input gradient, whose reduction runs over the output channels:
//   conv2: [tap][step of 16 output channels][part]          32x32x16 operand: lane = channel in + 32 * (channel out / 8)
// ---------------------------------------------------------------------------
constexpr int FRAG = 512;                       // elements of a fragment
constexpr int W1_FR = 2 * 8 * 3, W2_FR = 4 * 2 * 8 * 3, W3_FR = 4 * 2 * 9 * 3;
constexpr int W2_AT = W1_FR * FRAG, W3_AT = (W1_FR + W2_FR) * FRAG;
constexpr int W2B_FR = 16 * 4 * 3, W2B_AT = W3_AT + W3_FR * FRAG, W_TOTAL = W2B_AT + W2B_FR * FRAG;

// Where part 0 of conv parameter i of the blob (internal order) goes; part p is p * FRAG further.
// -1: a bias or not a conv parameter.
__host__ __device__ __forceinline__ int packed_at(long i)
{
    if (i >= net::C3B || i < 0) return -1;
    if (i >= net::C3W) {
        const int t = (int)(i - net::C3W), o = t / 576, k = t % 576, s = k >> 4;
        return W3_AT + ((((s / 9) * 2 + (o >> 5)) * 9 + s % 9) * 3) * FRAG + ((o & 31) + 32 * ((k >> 3) & 1)) * 8 + (k & 7);
    }
    if (i >= net::C2W && i < net::C2B) {
        const int t = (int)(i - net::C2W), o = t >> 9, k = t & 511, s = k >> 4;
        return W2_AT + ((((s >> 3) * 2 + (o >> 5)) * 8 + (s & 7)) * 3) * FRAG + ((o & 31) + 32 * ((k >> 3) & 1)) * 8 + (k & 7);
    }
    if (i < net::C1B) {
        const int t = (int)i, o = t >> 8, k = t & 255, s = k >> 5;
        return (((o >> 4) * 8 + s) * 3) * FRAG + ((o & 15) + 16 * ((k >> 3) & 3)) * 8 + (k & 7);
    }
    return -1;
}
// The second place of a conv2 weight (the input gradient's); -1: no conv2 weight
__host__ __device__ __forceinline__ int packed_back_at(long i)
{
    if (i < net::C2W || i >= net::C2B) return -1;
    const int t = (int)(i - net::C2W), o = t >> 9, tap = (t & 511) >> 5, ci = t & 31;
    return W2B_AT + ((tap * 4 + (o >> 4)) * 3) * FRAG + (ci + 32 * ((o >> 3) & 1)) * 8 + (o & 7);
}
__device__ __forceinline__ void store_parts(uint16_t *packed, int at, float x)
{
    const uint16_t a = bf16_bits(x);
    float r = x - bf16_value(a);
    const uint16_t b = bf16_bits(r);
    r -= bf16_value(b);
    packed[at] = a;
    packed[at + FRAG] = b;
    packed[at + 2 * FRAG] = bf16_bits(r);
}
// parameter i of the blob into its place or places (nothing for a bias or a parameter beyond the conv layers)
__device__ __forceinline__ void store_packed(uint16_t *packed, long i, float x)
{
    const int at = packed_at(i), back = packed_back_at(i);
    if (at >= 0) store_parts(packed, at, x);
    if (back >= 0) store_parts(packed, back, x);
}
// conv weights of one network -> packed parts; one thread per parameter below fc1
__global__ __launch_bounds__(256) void k_pack_conv(const float *theta, uint16_t *packed)
{
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i >= net::F1W) return;
    store_packed(packed, i, theta[i]);
}

// ---------------------------------------------------------------------------
// The bf16 network's conv weights for gbf::c123::k_conv123_fwd: fragments of v_mfma_f32_16x16x32_bf16
// (lane = row + 16 * (k / 8)), [conv1: half][step of 32], [conv2: 16 channels][step], [conv3: 16 channels][step].
// A step of conv1 is four columns of two kernel rows per lane group: [frame][column half], rows 2g and 2g + 1.
// Row i of half hh of conv1 is channel 8 (i / 4) + 4 hh + i % 4, so that a lane that holds rows 4g .. 4g+3 of both
// halves holds eight consecutive channels.
// ---------------------------------------------------------------------------
constexpr int B_W2 = 2 * 8 * FRAG, B_W3 = B_W2 + 4 * 16 * FRAG, B_TOTAL = B_W3 + 4 * 18 * FRAG;
__host__ __device__ __forceinline__ int packed_bf16_at(long i)
{
    if (i >= net::C3B || i < 0) return -1;
    if (i >= net::C3W) {
        const int t = (int)(i - net::C3W), o = t / 576, k = t % 576;
        return B_W3 + ((o >> 4) * 18 + (k >> 5)) * FRAG + ((o & 15) + 16 * ((k >> 3) & 3)) * 8 + (k & 7);
    }
    if (i >= net::C2W && i < net::C2B) {
        const int t = (int)(i - net::C2W), o = t >> 9, k = t & 511;
        return B_W2 + ((o >> 4) * 16 + (k >> 5)) * FRAG + ((o & 15) + 16 * ((k >> 3) & 3)) * 8 + (k & 7);
    }
    if (i < net::C1B) {
        const int t = (int)i, o = t >> 8, k = t & 255;
        // frame k / 64, kernel row (k / 8) % 8, column k % 8
        const int step = 2 * (k >> 6) + ((k >> 2) & 1), kg = (k >> 4) & 3, j = 4 * ((k >> 3) & 1) + (k & 3);
        return (((o >> 2) & 1) * 8 + step) * FRAG + (4 * (o >> 3) + (o & 3) + 16 * kg) * 8 + j;
    }
    return -1;
}
__device__ __forceinline__ void store_packed_bf16(uint16_t *packed, long i, float x)
{
    const int at = packed_bf16_at(i);
    if (at >= 0) packed[at] = bf16_bits(x);
}
__global__ __launch_bounds__(256) void k_pack_conv_bf16(const float *theta, uint16_t *packed)
{
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i < net::F1W) store_packed_bf16(packed, i, theta[i]);
}

}  // namespace sp

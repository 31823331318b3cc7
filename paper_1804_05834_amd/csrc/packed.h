// The bf16 network's conv weights in the order in which the matrix instructions of the fused forward launch take
// them.  RMSProp keeps the copy of the online network up to date.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "net.h"

namespace sp {

__device__ __forceinline__ uint16_t bf16_bits(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }   // nearest even

constexpr int FRAG = 512;                       // elements of a fragment: what one matrix instruction takes, 64 lanes x 16 bytes

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
// conv2's weights for its input gradient (gbf::dps): fragments of the same instruction, [parity class of the pixel (y, x)][tap of
// the class's four][half of the output channels][group of input channels], row i of group c input channel 8 (i / 4) + 4 c + i % 4.
constexpr int C2BACK_TOTAL = 4 * 16 * FRAG;
__host__ __device__ __forceinline__ int packed_conv2_back_at(int t)   // element t of conv2.W
{
    const int o = t >> 9, ky = (t >> 7) & 3, kx = (t >> 5) & 3, c = t & 31;
    const int step = 4 * (ky >> 1) + 2 * (kx >> 1) + (o >> 5);
    return (((2 * (ky & 1) + (kx & 1)) * 8 + step) * 2 + ((c >> 2) & 1)) * FRAG + (4 * (c >> 3) + (c & 3) + 16 * ((o >> 3) & 3)) * 8 + (o & 7);
}
// conv3's weights for its input gradient (gbf::c3b): fragments of v_mfma_f32_32x32x16_bf16 (lane = row + 32 * (k / 8)), [half of
// the input channels][step], a step being sixteen output channels of a tap.  Row 8 g + 4 h + j of a half is input channel
// 16 h + 4 g + j of it, so that a lane of the result holds sixteen consecutive channels.
constexpr int C3BACK_TOTAL = 2 * 36 * FRAG;
__host__ __device__ __forceinline__ int packed_conv3_back_at(int t)   // element t of conv3.W
{
    const int o = t / 576, tap = t % 576 >> 6, c = t & 63;
    return ((c >> 5) * 36 + 4 * tap + (o >> 4)) * FRAG + (8 * ((c >> 2) & 3) + 4 * ((c >> 4) & 1) + (c & 3) + 32 * ((o >> 3) & 1)) * 8 + (o & 7);
}
__device__ __forceinline__ void store_packed_bf16(uint16_t *packed, long i, float x)
{
    const int at = packed_bf16_at(i);
    if (at >= 0) packed[at] = bf16_bits(x);
}
constexpr int BACK_TOTAL = C2BACK_TOTAL + C3BACK_TOTAL;
__device__ __forceinline__ void store_back_bf16(uint16_t *back, long i, float x)
{
    if (i >= net::C2W && i < net::C2B) back[packed_conv2_back_at((int)(i - net::C2W))] = bf16_bits(x);
    if (i >= net::C3W && i < net::C3B) back[C2BACK_TOTAL + packed_conv3_back_at((int)(i - net::C3W))] = bf16_bits(x);
}
// back: nullptr for a network that is not trained
__global__ __launch_bounds__(256) void k_pack_conv_bf16(const float *theta, uint16_t *packed, uint16_t *back)
{
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i >= net::F1W) return;
    store_packed_bf16(packed, i, theta[i]);
    if (back) store_back_bf16(back, i, theta[i]);
}

}  // namespace sp

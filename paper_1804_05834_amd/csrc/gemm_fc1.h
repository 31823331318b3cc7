// fc1 forward in fp32 for more than a few rows: raw sums y[split][m][n] = sum over the split's k of x[m][k] w[n][k].
//
// A workgroup of four waves, one per SIMD, has 16 MB rows x 64 columns, a wave all the rows and 16 of the columns, in
// v_mfma_f32_16x16x4_f32: the tile's height goes in steps of 16 rows, and the host takes the one that fills the compute
// units best (fc1_blocks).  In tiles of 64 x 64 the 3000 rows of a batch of 1000 were 376 for 256 compute units.
// Both operands go through LDS in stages of 32 of the reduction, two buffers, one barrier per stage: a stage is requested
// three stages ahead and lies in registers until its buffer is free; a wave reads the operands of sixteen ahead of its
// matrix instructions, and the barrier stands between the stage's two halves, so those behind it are read beside the second.
// Bound by the fp32 matrix pipe, beside which a SIMD runs loads and LDS accesses but no vector instructions, and a load or LDS
// access in front of a matrix instruction of the same wave holds it up: they stand one by one behind matrix instructions.
// At a batch of 1000 (3000 rows, 96 per compute unit: 62.7 us at 2.4 GHz) 115.1 us in 64 x 64 tiles of 32x32x2; so 92.1, without
// the moves in front of paired LDS stores and with the requests in the loop's order 83.9, with everything behind a matrix
// instruction 76.7.  The step of 1000 939 -> 897, of 256 307 -> 302, of 65 145 -> 138; acting on 300 64.8 -> 58.0, on 2048 224 ->
// 212, on 8192 854 -> 823.
// Order of the sums: that of the 32x32x2 instructions of g32::k_fwd, which add k and k + 4 of eight in turn.  The four products
// of a 16x16x4 are therefore k = 0, 4, 1, 5 of eight, then 2, 6, 3, 7, and a lane group's shares of sixteen lie side by side in
// LDS: 0 2 8 10 | 4 6 12 14 | 1 3 9 11 | 5 7 13 15.
#pragma once
#include "gemm_fp32.h"

namespace fc1 {
using g32::ld4;
using g32::sync_lds;
constexpr int THREADS = 256, MIN_MB = 3, MAX_MB = 8, BN = 64;
constexpr int LD = 40;   // floats per row of a stage: a 16-byte read, served sixteen lanes at a time, meets every bank once

template <int MB>
__global__ __launch_bounds__(THREADS, 2) void k_fwd(g32::FwdArgs A)
{
    using G = g32::GFc1;
    constexpr int BM = 16 * MB, STAGE = (BM + BN) * LD;
    constexpr int NA = (MB + 1) / 2, NB = BN * 8 / THREADS;   // 16-byte pieces per thread and stage (odd MB: the last by half the threads)
    __shared__ __attribute__((aligned(16))) float lds[2 * STAGE];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, i = lane & 15, g = lane >> 4;
    // tile order: column tiles of one row tile together, reduction splits apart
    const int t = net::tile_of_workgroup();
    const int by = t % (int)gridDim.y, bx = (t / (int)gridDim.y) % (int)gridDim.x, bz = t / (int)(gridDim.y * gridDim.x);
    g32::FwdSeg S = A.seg[0];
    if (A.nseg > 1 && bx >= A.seg[1].tile_begin) S = A.seg[1];
    if (A.nseg > 2 && bx >= A.seg[2].tile_begin) S = A.seg[2];
    const int m0 = (bx - S.tile_begin) * BM, n0 = by * BN, n = A.klen / 32;
    const float *x = static_cast<const float *>(S.x) + bz * A.klen, *w = S.w + bz * A.klen + n0 * G::K;

    const int r0 = tid >> 3, piece = tid & 7;   // rows r0 + 32 j, floats 4 piece .. + 3 of the stage
    const bool last_a = MB % 2 == 0 || tid < THREADS / 2;
    uint32_t xo[NA], wo[NB];
#pragma unroll
    for (int j = 0; j < NA; ++j) xo[j] = (uint32_t)min(m0 + r0 + 32 * j, S.M - 1) * (uint32_t)S.xs + 4 * piece;   // (rows past the end are not stored)
#pragma unroll
    for (int j = 0; j < NB; ++j) wo[j] = (r0 + 32 * j) * G::K + 4 * piece;
    struct Regs { v4f v[NA + NB]; } R[2];
    auto request = [&](Regs &q, int s, int j) {   // piece j; beyond the last stage: the last one again, which nobody reads
        const int k = 32 * min(s, n - 1);
        q.v[j] = j < NA ? ld4(x + k + xo[j < NA ? j : 0]) : ld4(w + k + wo[j < NA ? 0 : j - NA]);
    };
    const int put_at = r0 * LD + 16 * (piece >> 2) + 4 * (piece & 1) + (piece & 2);
    auto put = [&](const Regs &q, float *buf, int j) {
        const v4f v = q.v[j];
        const uint32_t at = (uint32_t)(uintptr_t)(buf + put_at + (j < NA ? 32 * j : BM + 32 * (j - NA)) * LD);
        // (the compiler would put stores of pairs together with moves)
        if (j + 1 != NA || last_a)
            asm volatile("ds_write2_b32 %0, %1, %2 offset0:0 offset1:1\n\tds_write2_b32 %0, %3, %4 offset0:8 offset1:9" :: "v"(at), "v"(v.x), "v"(v.z), "v"(v.y), "v"(v.w) : "memory");
    };
    struct Ops { v4f v[MB + 1]; } O[2];   // (the columns' last)
    const int get_a = i * LD + 4 * g, get_b = (BM + 16 * wave + i) * LD + 4 * g;
    auto get = [&](Ops &o, const float *buf, int half, int j) { o.v[j] = ld4(buf + (j < MB ? get_a + 16 * j * LD : get_b) + 16 * half); };
    v4f acc[MB];
#pragma unroll
    for (int j = 0; j < MB; ++j) acc[j] = v4f{0, 0, 0, 0};
    // sixteen of the reduction; behind each matrix instruction one of `items` others, which would keep it waiting in front
    auto multiply = [&](const Ops &o, int items, auto item) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int j = 0; j < MB; ++j) {
                acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(o.v[j][q], o.v[MB][q], acc[j], 0, 0, 0);
                if (MB * q + j < items) item(MB * q + j);
                __builtin_amdgcn_sched_barrier(0);
            }
    };
    // stage s, in `buf`; q: stage s + 1, then on its way s + 3
    constexpr int NG = MB + 1, NP = NA + NB;
    static_assert(NG + 2 * NP <= 4 * MB, "items");
    auto stage = [&](int s, const float *buf, float *other, Regs &q) {
        multiply(O[0], NG + 2 * NP, [&](int i) {
            if (i < NG) get(O[1], buf, 1, i);
            else if (i < NG + NP) put(q, other, i - NG);
            else request(q, s + 3, i - NG - NP);
        });
        sync_lds();   // stage s + 1 lies in `other`, and nobody reads `buf` any more
        multiply(O[1], NG, [&](int i) { get(O[0], other, 0, i); });
    };
    auto all = [&](int count, auto item) {   // (in this order: ahead of the loop another one would make its waits longer)
#pragma unroll
        for (int j = 0; j < count; ++j) {
            item(j);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    all(NP, [&](int j) { request(R[0], 0, j); });
    all(NP, [&](int j) { request(R[1], 1, j); });
    all(NP, [&](int j) { put(R[0], lds, j); });
    all(NP, [&](int j) { request(R[0], 2, j); });
    sync_lds();
    all(NG, [&](int j) { get(O[0], lds, 0, j); });
    int s = 0;
    for (; s + 2 <= n; s += 2) {
        stage(s, lds, lds + STAGE, R[1]);
        stage(s + 1, lds + STAGE, lds, R[0]);
    }
    if (s < n) stage(s, lds, lds + STAGE, R[1]);

    float *y = S.y + (long)bz * A.split_stride + ((long)(m0 + 4 * g) * G::N + n0 + 16 * wave + i);
#pragma unroll
    for (int j = 0; j < MB; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (m0 + 16 * j + 4 * g + r < S.M) y[(16 * j + r) * G::N] = acc[j][r];
}
}  // namespace fc1

// Everything around the GEMMs: the head (dueling combine, argmax, Bellman
// target, Huber loss and their gradients), RMSProp, the sum-tree, the
// frame-stack gather, epsilon-greedy selection and layout permutations.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>
#include <stdint.h>

#include "net.h"
#include "packed.h"
#include "sumtree.h"

namespace misc {

// Barrier that orders LDS traffic only: global loads and stores issued earlier stay in flight
// across it (__syncthreads() would first wait for every one of them to complete).
__device__ __forceinline__ void sync_lds()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// The value of lane `lane ^ O`.  Within sixteen lanes by the operand permutation of a vector instruction, across by the
// row and half swaps: a few cycles each, where the exchange through LDS that __shfl_xor compiles to is a round trip of
// about a hundred, and the reductions of the head and of the tree are chains of them.
template <int O> __device__ __forceinline__ int lane_xor(int v)
{
    if constexpr (O == 1) return __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, true);          // quad_perm 1 0 3 2
    else if constexpr (O == 2) return __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, true);     // quad_perm 2 3 0 1
    else if constexpr (O == 4)                                                                     // half mirror (7 - l), then 3 - l
        return __builtin_amdgcn_update_dpp(0, __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, true), 0x1B, 0xF, 0xF, true);
    else if constexpr (O == 8) return __builtin_amdgcn_update_dpp(0, v, 0x128, 0xF, 0xF, true);    // rotation by 8 of 16
    else if constexpr (O == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return (int)(threadIdx.x & 16 ? r[0] : r[1]);
    } else {
        static_assert(O == 32, "lane_xor: O is a power of two below 64");
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return (int)(threadIdx.x & 32 ? r[0] : r[1]);
    }
}
template <int O> __device__ __forceinline__ float lane_xor(float v) { return __int_as_float(lane_xor<O>(__float_as_int(v))); }

// the value of lane + N, of the same sixteen lanes (0 past them)
template <int N> __device__ __forceinline__ float row_shl(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x100 + N, 0xF, 0xF, true));
}

template <int O = 32, class T> __device__ __forceinline__ T wave_sum(T v)   // over groups of 2 O lanes
{
    v += lane_xor<O>(v);
    if constexpr (O > 1) return wave_sum<O / 2>(v);
    else return v;
}
__device__ __forceinline__ float wave_max(float v)
{
    v = fmaxf(v, lane_xor<32>(v));
    v = fmaxf(v, lane_xor<16>(v));
    v = fmaxf(v, lane_xor<8>(v));
    v = fmaxf(v, lane_xor<4>(v));
    v = fmaxf(v, lane_xor<2>(v));
    return fmaxf(v, lane_xor<1>(v));
}
// the largest value of the wave and the lowest index that holds it, in every lane
template <int O = 32> __device__ __forceinline__ void wave_argmax(float &bv, int &bi)
{
    const float ov = lane_xor<O>(bv);
    const int oi = lane_xor<O>(bi);
    if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
    if constexpr (O > 1) wave_argmax<O / 2>(bv, bi);
}

__device__ __forceinline__ float block_max_1024(float v, float *sh /*16*/)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    v = wave_max(v);
    __syncthreads();
    if (lane == 0) sh[wave] = v;
    __syncthreads();
    float r = sh[0];
    for (int w = 1; w < (int)(blockDim.x >> 6); ++w) r = fmaxf(r, sh[w]);
    return r;
}

// ------------------------------------------------------------------ head
// Rows of the head: dueling -> row 0 is the state value V, rows 1..K the
// advantages (Eq.13); plain -> rows 0..K-1 are the Q outputs.  Offsets are
// relative to the head section of the parameter blob.
__device__ __forceinline__ int head_w_off(int r, int K, int dueling)
{
    if (!dueling) return r * net::HID;
    return r == 0 ? 0 : net::HID + 1 + (r - 1) * net::HID;
}
__device__ __forceinline__ int head_b_off(int r, int K, int dueling)
{
    if (!dueling) return K * net::HID + r;
    return r == 0 ? net::HID : net::HID + 1 + K * net::HID + (r - 1);
}

constexpr int MAXR = 65;  // up to 64 actions + V

// The dot products of the head for the three passes of a training row at once: 3R of length 512 spread
// over groups of 16 lanes, so the whole head takes two rounds of a 512-thread workgroup instead
// of one wave per row in turn.  The weights of a round do not depend on the hidden layer, so
// head_rows3_load requests them while the fc1 partial sums are still being added up, and
// head_rows3_dot only reads LDS.
struct HeadRound {
    float w[net::HID / 16];
    float b;
    int d;  // dot product number: pass = d / R, row = d % R; -1: none
};
__device__ __forceinline__ void head_rows3_load(HeadRound &H, int round, const float *head_on, const float *head_tg,
                                                int K, int dueling, int tid)
{
    const int R = K + (dueling ? 1 : 0);
    const int grp = tid >> 4, l = tid & 15;
    const int d = grp + 32 * round;
    H.d = d < 3 * R ? d : -1;
    if (H.d < 0) return;
    const int p = d / R, r = d - p * R;
    const float *head = p == 2 ? head_tg : head_on;
    const float *w = head + head_w_off(r, K, dueling);
#pragma unroll
    for (int k = 0; k < net::HID / 16; ++k) H.w[k] = w[l + 16 * k];
    H.b = head[head_b_off(r, K, dueling)];
}
// Where hidden unit i lies in LDS: lane l of a group of sixteen takes units l, l + 16, ... in turn, and finds them side
// by side, eight 16-byte reads instead of 32 of four bytes (the pitch of 36 keeps the sixteen lanes in different banks).
constexpr int HID_LDS = 16 * 36;
__device__ __forceinline__ int hid_at(int i) { return (i & 15) * 36 + (i >> 4); }
// sum over k of w[k] * unit l + 16 k, in the order of k, then over the sixteen lanes
__device__ __forceinline__ float head_dot(const HeadRound &H, const float *hid, int l)
{
    float acc = 0.f;
#pragma unroll
    for (int k = 0; k < net::HID / 16; k += 4) {
        const float4 x = *reinterpret_cast<const float4 *>(hid + l * 36 + k);
        acc += H.w[k] * x.x;
        acc += H.w[k + 1] * x.y;
        acc += H.w[k + 2] * x.z;
        acc += H.w[k + 3] * x.w;
    }
    return wave_sum<8>(acc);
}
__device__ __forceinline__ void head_rows3_dot(const HeadRound &H, const float (*hid)[HID_LDS] /*LDS [3]*/,
                                               int K, int dueling, float (*raw)[65] /*LDS [3][65]*/, int tid)
{
    if (H.d < 0) return;  // uniform within the 16-lane group
    const int R = K + (dueling ? 1 : 0);
    const int l = tid & 15;
    const int p = H.d / R, r = H.d - p * R;
    const float acc = head_dot(H, hid[p], l);
    if (l == 0) raw[p][r] = acc + H.b;
}

struct HeadArgs {
    const float *part;  // fc1 partial sums [nsplit][3B][512]: rows s | s' online | s' target
    int nsplit;
    long split_stride;
    int B, K, dueling, double_q, loss_kind;
    float kappa, gamma;
    const float *f1b_on, *f1b_tg;    // fc1 biases
    const float *head_on, *head_tg;  // head sections of the two parameter blobs
    const int32_t *a;
    const float *r;
    const uint8_t *done;
    const float *w;  // may be nullptr
    int w_raw;       // 1: w holds unnormalised importance weights; divide by their maximum here
    float *h_s;      // [B][512] hidden layer of the online net on s
    void *dh;        // [B][512] gradient w.r.t. the fc1 pre-activation (fp32, or bf16 if dh_bf16)
    int dh_bf16;
    float *dA;       // [B][R]   gradient w.r.t. the head rows
    float *td_abs;   // [B] |td_j|; NaN for a row the priority update must skip
    float *loss_j;   // [B] w_j * l(td_j)
    float *qmax_j;   // [B] max_a Q(s_j, a; theta)
    float *q_s, *q_no, *q_nt, *y, *td;  // optional outputs
    int32_t *a_star;
    float *is_w;
};

// One workgroup per minibatch row: finishes fc1 (split reduction, bias, ReLU)
// for the three passes, evaluates the head three times, forms the target
// (Eq.8 / Eq.9), the TD error, the loss term and the gradient w.r.t. the
// head rows, and back-propagates through the head into the hidden layer.
//
// The kernel is a chain of latencies, so it is written to have ONE round trip to memory: every
// global operand (partial sums and biases first, then the head weights of the dot products, the
// thread's column of the online head for the back-propagation, the raw importance weights, the
// row's transition) is requested before anything is waited for, in the order of first use.  The
// dueling combine (Eq.13) and the argmax run on one wave per pass with lane a holding action a.
// NS: the number of reduction splits of fc1 (A.nsplit), a template argument so that the loads of the
// partial sums are unconditional: behind a run-time test the compiler adds a split to its sum right where
// it is loaded, and the kernel then waits for its first load before it has requested the second.
constexpr int HEAD_MAX_SPLITS = 7;   // most reduction splits of fc1
template <int NS>
__global__ __launch_bounds__(512) void k_head_train(HeadArgs A)
{
    __shared__ __attribute__((aligned(16))) float hid[3][HID_LDS];
    __shared__ float raw[3][MAXR];
    __shared__ float q[3][64];
    __shared__ float shm[16];
    __shared__ float res_q[3];     // Q(s, a_j; theta), max_a Q(s, a; theta), -
    __shared__ int res_as[3];      // argmax_a of pass p
    const int j = blockIdx.x, tid = threadIdx.x;
    const int K = A.K, R = K + (A.dueling ? 1 : 0);
    const bool norm = A.w && A.w_raw;

    // ---- every global load, in the order of first use
    float ps[3][NS];
    const long row[3] = {(long)j, (long)A.B + j, 2L * A.B + j};
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int sp = 0; sp < NS; ++sp) ps[p][sp] = A.part[sp * A.split_stride + row[p] * net::HID + tid];
    const float b_on = A.f1b_on[tid], b_tg = A.f1b_tg[tid];
    HeadRound H0, H1;
    head_rows3_load(H0, 0, A.head_on, A.head_tg, K, A.dueling, tid);
    head_rows3_load(H1, 1, A.head_on, A.head_tg, K, A.dueling, tid);
    const int aj_raw = A.a[j];
    const bool dn = A.done[j] != 0;
    const float rj = A.r[j];
    const float wj = A.w ? A.w[j] : 1.f;
    float w0 = 0.f, w1 = 0.f;   // raw importance weights tid and tid + 512 (B <= 1024), for their maximum
    if (norm) {
        w0 = tid < A.B ? A.w[tid] : 0.f;
        w1 = tid + 512 < A.B ? A.w[tid + 512] : 0.f;
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- hidden layer: split sums in split order, bias, ReLU
    float hs;   // the thread's unit of pass 0
    {
        float acc[3] = {0.f, 0.f, 0.f};
#pragma unroll
        for (int p = 0; p < 3; ++p) {
#pragma unroll
            for (int sp = 0; sp < NS; ++sp) acc[p] += ps[p][sp];
        }
        hs = fmaxf(acc[0] + b_on, 0.f);
        hid[0][hid_at(tid)] = hs;
        hid[1][hid_at(tid)] = fmaxf(acc[1] + b_on, 0.f);
        hid[2][hid_at(tid)] = fmaxf(acc[2] + b_tg, 0.f);
        A.h_s[(long)j * net::HID + tid] = hs;
    }
    __syncthreads();
    // column tid of the online head, for the back-propagation into the hidden layer at the end: requested
    // here, behind the operands the dot products wait for, and in flight until the last phase
    constexpr int HW_PRE = 24;
    float hw[HW_PRE];
#pragma unroll
    // (unconditional, row index clamped: a value chosen between a loaded one and a constant would be waited
    // for right here, in front of the dot products)
    for (int r = 0; r < HW_PRE; ++r) hw[r] = A.head_on[head_w_off(r < R ? r : R - 1, K, A.dueling) + tid];
    __builtin_amdgcn_sched_barrier(0);
    head_rows3_dot(H0, hid, K, A.dueling, raw, tid);
    head_rows3_dot(H1, hid, K, A.dueling, raw, tid);
    for (int round = 2; 32 * round < 3 * R; ++round) {  // more than 64 dot products: K > 20
        head_rows3_load(H0, round, A.head_on, A.head_tg, K, A.dueling, tid);
        head_rows3_dot(H0, hid, K, A.dueling, raw, tid);
    }
    if (norm) {  // per-wave maxima of the raw weights; thread 0 combines them below
        const float wmax = wave_max(fmaxf(w0, w1));
        if ((tid & 63) == 0) shm[tid >> 6] = wmax;
    }
    __syncthreads();
    const bool a_ok = aj_raw >= 0 && aj_raw < K;
    const int aj = a_ok ? aj_raw : 0;
    if (tid < 192) {
        // wave p: lane a holds Q_a of pass p (Eq.13: V + A_a - mean A, or the plain outputs)
        const int p = tid >> 6, a = tid & 63;
        const float v = a < K ? raw[p][A.dueling ? 1 + a : a] : 0.f;
        float qa = v;
        if (A.dueling) qa = raw[p][0] + (v - wave_sum(v) / (float)K);
        if (a < K) q[p][a] = qa;
        // argmax with the lowest index winning ties; lanes past K never win
        float bv = a < K ? qa : -3.4028234663852886e38f;
        int bi = a < K ? a : 64;
        wave_argmax(bv, bi);
        const float q_aj = lane_value(qa, aj);
        if (a == 0) {
            res_as[p] = bi;
            if (p == 0) { res_q[0] = q_aj; res_q[1] = bv; }
        }
    }
    __syncthreads();
    if (tid == 0) {
        float wnorm = 1.f;
        if (norm) {
            float m = shm[0];
            for (int v = 1; v < 8; ++v) m = fmaxf(m, shm[v]);
            wnorm = m > 0.f ? 1.f / m : 0.f;   // no mass in the tree: every weight is 0
        }
        const int as = res_as[A.double_q ? 1 : 2];
        const float boot = dn ? 0.f : A.gamma * q[2][as];
        const float y = rj + boot;
        const float d = y - res_q[0];
        // an action outside [0, K) cannot be trained on: the row contributes nothing (weight 0), its TD
        // error is reported as NaN and the priority update skips it
        const float w = !a_ok ? 0.f : A.w ? wj * wnorm : 1.f;
        float l, dl;
        if (A.loss_kind == 1 && fabsf(d) > A.kappa) {
            l = A.kappa * (fabsf(d) - 0.5f * A.kappa);
            dl = d > 0.f ? A.kappa : -A.kappa;
        } else {
            l = 0.5f * d * d;
            dl = d;
        }
        shm[8] = -w * dl / (float)A.B;  // dL/dQ(s_j, a_j)
        // a drawn row whose raw weight is 0 came from a tree without mass: its slot holds nothing to update
        const bool skip = !a_ok || (norm && !(wj > 0.f));
        A.td_abs[j] = skip ? __int_as_float(0x7fc00000) : fabsf(d);
        A.loss_j[j] = w * l;
        A.qmax_j[j] = res_q[1];
        if (A.y) A.y[j] = y;
        if (A.td) A.td[j] = a_ok ? d : __int_as_float(0x7fc00000);
        if (A.a_star) A.a_star[j] = as;
        if (A.is_w) A.is_w[j] = w;
    }
    if (A.q_s && tid >= 64 && tid < 64 + K) A.q_s[(long)j * K + tid - 64] = q[0][tid - 64];
    if (A.q_no && tid >= 128 && tid < 128 + K) A.q_no[(long)j * K + tid - 128] = q[1][tid - 128];
    if (A.q_nt && tid >= 192 && tid < 192 + K) A.q_nt[(long)j * K + tid - 192] = q[2][tid - 192];
    __syncthreads();
    {
        // gradient w.r.t. the head rows (dueling: dV = g, dA_a = [a = a_j] g - g / K), every thread for itself
        const float g = shm[8];
        const float gk = A.dueling ? g / (float)K : 0.f;
        const int hit = A.dueling ? 1 + aj : aj;
        if (tid < R) A.dA[(long)j * R + tid] = (A.dueling && tid == 0) ? g : (tid == hit ? g : 0.f) - gk;
        float acc = 0.f;
#pragma unroll
        for (int r = 0; r < HW_PRE; ++r)
            if (r < R) acc += ((A.dueling && r == 0) ? g : (r == hit ? g : 0.f) - gk) * hw[r];
        for (int r = HW_PRE; r < R; ++r)
            acc += ((A.dueling && r == 0) ? g : (r == hit ? g : 0.f) - gk) * A.head_on[head_w_off(r, K, A.dueling) + tid];
        const float gmask = hs > 0.f ? acc : 0.f;
        if (A.dh_bf16) static_cast<__hip_bfloat16 *>(A.dh)[(long)j * net::HID + tid] = __float2bfloat16(gmask);
        else static_cast<float *>(A.dh)[(long)j * net::HID + tid] = gmask;
    }
}

struct HeadWgradArgs {
    const float *dA;      // [B][R]
    const float *h_s;     // [B][512]
    const float *loss_j;  // [B]
    float *ghead;         // head section of the gradient partial buffer
    float *loss_out;      // optional
    float *loss_slot;     // always written
    int B, K, dueling;
    const float *td_abs;  // [B]
    const float *qmax_j;  // [B]
    float *td_abs_mean;   // optional [1]: (1/B) sum_j |td_j| over the rows with a finite error
    float *q_max_mean;    // optional [1]: (1/B) sum_j max_a Q(s_j, a; theta)
};

// Head weight gradient: dW[r][i] = sum_j dA[j][r] h[j][i], db[r] = sum_j dA[j][r].
// grid (R, 16): block (r, c) owns hidden units [32c, 32c+32); its 512 threads split the
// minibatch sixteen ways and combine through LDS in a fixed order.  Block (0,0) also folds the
// per-row loss terms into L = (1/B) sum_j w_j l_j.
// NG = threads / 32 groups over the minibatch; lds: NG * 34 floats.  Row r, hidden units [32c, 32c+32).
template <int NG>
__device__ __forceinline__ void head_wgrad_body(const HeadWgradArgs &A, int r, int c, float *lds)
{
    float(*red)[33] = reinterpret_cast<float(*)[33]>(lds);
    float *redb = lds + NG * 33;
    const int il = threadIdx.x & 31, jg = threadIdx.x >> 5;
    const int i = c * 32 + il;
    const int R = A.K + (A.dueling ? 1 : 0);
    float acc = 0.f, accb = 0.f;
#pragma unroll 8
    for (int j = jg; j < A.B; j += NG) {
        float d = A.dA[(long)j * R + r];
        acc += d * A.h_s[(long)j * net::HID + i];
        accb += d;
    }
    red[jg][il] = acc;
    if (il == 0) redb[jg] = accb;
    __syncthreads();
    if (jg == 0) {
        float s = red[0][il];
#pragma unroll
        for (int g = 1; g < NG; ++g) s += red[g][il];
        A.ghead[head_w_off(r, A.K, A.dueling) + i] = s;
        if (il == 0 && c == 0) {
            float sb = redb[0];
#pragma unroll
            for (int g = 1; g < NG; ++g) sb += redb[g];
            A.ghead[head_b_off(r, A.K, A.dueling)] = sb;
        }
    }
    if (r == 0 && c == 0 && (int)threadIdx.x >= NG * 32 - 64) {  // the last wave sums the loss terms
        const int lane = threadIdx.x & 63;
        float s = 0.f, sd = 0.f, sq = 0.f;
        for (int j = lane; j < A.B; j += 64) {
            s += A.loss_j[j];
            const float d = A.td_abs[j];
            if (d <= 3.4028234e38f) sd += d;   // false for NaN
            sq += A.qmax_j[j];
        }
        s = wave_sum(s) / (float)A.B;
        sd = wave_sum(sd) / (float)A.B;
        sq = wave_sum(sq) / (float)A.B;
        if (lane == 0) {
            *A.loss_slot = s;
            if (A.loss_out) *A.loss_out = s;
            if (A.td_abs_mean) *A.td_abs_mean = sd;
            if (A.q_max_mean) *A.q_max_mean = sq;
        }
    }
}

__global__ __launch_bounds__(512) void k_head_wgrad(HeadWgradArgs A)
{
    __shared__ float lds[16 * 34];
    head_wgrad_body<16>(A, blockIdx.x, blockIdx.y, lds);
}

// ---- work that the last workgroup of a launch to arrive does for all of them
// A workgroup hands over its few words with device-scope stores, waits until they are acknowledged and draws
// a number; the one that draws the last reads all words with device-scope loads.  Only those words are made
// visible beyond the die's L2: a device-wide fence here would write the whole L2 back, a thousand times a
// launch.  No workgroup waits for another.  The counter is 0 before the launch and the last one puts it back.
__device__ __forceinline__ void publish_word(float *p, float v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float read_word(const float *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// called by one thread, after the barrier behind which all of the workgroup's words have been stored and
// acknowledged (words_acknowledged() by the threads that stored them)
__device__ __forceinline__ void words_acknowledged() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ bool arrived_last(unsigned *count, unsigned of)
{
    const unsigned k = __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (k != of - 1) return false;
    __hip_atomic_store(count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return true;
}

struct HeadActArgs {
    const float *part;
    int nsplit;
    long split_stride;
    int E, K, dueling;
    const float *f1b, *head;
    float epsilon;
    uint64_t seed;
    int32_t *actions;
    float *q_out;  // optional [E][K]
};

// Acting (Alg.1 action lines): finish fc1, evaluate the head, pick the action.  ROWS observations per workgroup at a
// time, built like the training head: every global operand (the partial sums of the thread's two
// hidden units per row, the biases, the head weights of the first 32 dot products, spread over groups of 16 lanes)
// is requested before anything is waited for, the dueling combine (Eq.13) and the argmax run on one wave per row
// with lane a holding action a, and the arithmetic is that of k_head_train: the same partial sums give the same Q(s, .)
// here and there.  NS: reduction splits of fc1 (A.nsplit), a template argument so that the loads are
// unconditional.
// With a workgroup per observation, 8192 of them fetched the head's weights, 39 KB at 18 actions, 8192 times and took
// 21 us for 17 MB of partial sums.  So many observations share workgroups that keep the weights in registers and take
// four rows in turn, the next four's sums on their way: 9.1 us (2048 in three splits: 6.9 -> 5.1).  Fewer have a
// workgroup each, which has the shorter chain (launch_head_act).
__device__ __forceinline__ void head_rows1_load(HeadRound &H, int round, const float *head, int K, int dueling, int tid)
{
    const int R = K + (dueling ? 1 : 0);
    const int grp = tid >> 4, l = tid & 15;
    const int d = grp + 16 * round;
    H.d = d < R ? d : -1;
    const int r = d < R ? d : R - 1;   // clamped: the loads are unconditional
    const float *w = head + head_w_off(r, K, dueling);
#pragma unroll
    for (int k = 0; k < net::HID / 16; ++k) H.w[k] = w[l + 16 * k];
    H.b = head[head_b_off(r, K, dueling)];
}
// (head_dot for the rows side by side: a row's sum is one chain of 32 additions, in that order)
template <int ROWS>
__device__ __forceinline__ void act_dots(const HeadRound &H, const float (*hid)[HID_LDS], float (*raw)[MAXR], int l)
{
    float acc[ROWS] = {};
    float4 x[ROWS], nx[ROWS];
    auto read = [&](int k) {
#pragma unroll
        for (int r = 0; r < ROWS; ++r) nx[r] = *reinterpret_cast<const float4 *>(&hid[r][l * 36 + k]);
    };
    read(0);
#pragma unroll
    for (int k = 0; k < net::HID / 16; k += 4) {
#pragma unroll
        for (int r = 0; r < ROWS; ++r) x[r] = nx[r];
        if (k + 4 < net::HID / 16) read(k + 4);
        if (ROWS > 1) __builtin_amdgcn_sched_barrier(0);   // all reads at once would take the registers of three workgroups
#pragma unroll
        for (int r = 0; r < ROWS; ++r) acc[r] += H.w[k] * x[r].x;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) acc[r] += H.w[k + 1] * x[r].y;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) acc[r] += H.w[k + 2] * x[r].z;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) acc[r] += H.w[k + 3] * x[r].w;
        if (ROWS > 1) __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int r = 0; r < ROWS; ++r) acc[r] = wave_sum<8>(acc[r]);
    if (l == 0 && H.d >= 0)
#pragma unroll
        for (int r = 0; r < ROWS; ++r) raw[r][H.d] = acc[r] + H.b;
}
// The dueling combine, the argmax and the draw of observation e, by one wave, out of its raw dot products
__device__ __forceinline__ void act_choose(const HeadActArgs &A, const float *rw, int e, int a)
{
    const int K = A.K;
    const float v = a < K ? rw[A.dueling ? 1 + a : a] : 0.f;
    float qa = v;
    if (A.dueling) qa = rw[0] + (v - wave_sum(v) / (float)K);
    // argmax with the lowest index winning ties; lanes past K never win
    float bv = a < K ? qa : -3.4028234663852886e38f;
    int bi = a < K ? a : 64;
    wave_argmax(bv, bi);
    if (a == 0) {
        int act = bi;
        const float u = draw_u24(A.seed, 2ull * (uint64_t)e);
        if (u < A.epsilon) {
            const float u2 = draw_u24(A.seed, 2ull * (uint64_t)e + 1ull);
            act = min((int)floorf(u2 * (float)K), K - 1);
        }
        A.actions[e] = act;
    }
    if (A.q_out && a < K) A.q_out[(long)e * K + a] = qa;
}
template <int NS, int ROWS>
__global__ __launch_bounds__(256, ROWS == 1 ? 1 : 3) void k_head_act(HeadActArgs A)
{
    __shared__ __attribute__((aligned(16))) float hid[ROWS][HID_LDS];
    __shared__ float raw[ROWS][MAXR];
    const int tid = threadIdx.x, wave = tid >> 6, l = tid & 15;
    const int K = A.K, R = K + (A.dueling ? 1 : 0);
    float ps[ROWS][2][NS];
    auto load_sums = [&](int e0) {
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const int e = min(e0 + r, A.E - 1);   // (rows past the end repeat the last one)
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int sp = 0; sp < NS; ++sp) ps[r][u][sp] = A.part[sp * A.split_stride + (long)e * net::HID + tid + 256 * u];
        }
    };
    int e0 = blockIdx.x * ROWS;
    load_sums(e0);
    const float b0 = A.f1b[tid], b1 = A.f1b[tid + 256];
    HeadRound H0, H1;
    head_rows1_load(H0, 0, A.head, K, A.dueling, tid);
    head_rows1_load(H1, 1, A.head, K, A.dueling, tid);
    __builtin_amdgcn_sched_barrier(0);
    for (;;) {
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            float acc[2] = {0.f, 0.f};
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int sp = 0; sp < NS; ++sp) acc[u] += ps[r][u][sp];
            hid[r][hid_at(tid)] = fmaxf(acc[0] + b0, 0.f);
            hid[r][hid_at(tid + 256)] = fmaxf(acc[1] + b1, 0.f);
        }
        const int next = e0 + (int)gridDim.x * ROWS;
        if (ROWS > 1 && next < A.E) load_sums(next);
        sync_lds();
        act_dots<ROWS>(H0, hid, raw, l);
        if (16 + 4 * wave < R) act_dots<ROWS>(H1, hid, raw, l);
        if constexpr (ROWS == 1)
            for (int round = 2; 16 * round < R; ++round) {   // more than 32 dot products: K > 31
                head_rows1_load(H0, round, A.head, K, A.dueling, tid);
                act_dots<ROWS>(H0, hid, raw, l);
            }
        sync_lds();
        const int e = e0 + wave;
        if (wave < ROWS && e < A.E) act_choose(A, raw[ROWS == 1 ? 0 : wave], e, tid & 63);
        if (ROWS == 1 || next >= A.E) break;
        // (the next round writes hid, which every wave has read, before the barrier behind which raw is written again)
        e0 = next;
    }
}
// Four rows per workgroup from four observations per CU on, where a workgroup each no longer fits the chip at once
// (1024 in six splits: 4.5 against 5.0 us, 600 in seven: 5.1 against 4.5), and for heads of at most 32 rows, whose
// weights fit in registers (beside the partial sums of up to six splits; that many rows have seven only where they are
// asked for).  Three workgroups fit a CU.
template <int NS> void launch_head_act_ns(const HeadActArgs &H, int num_cu, hipStream_t st)
{
    if constexpr (NS <= 6)
        if (H.E >= 4 * num_cu && H.K + (H.dueling ? 1 : 0) <= 32) {
            k_head_act<NS, 4><<<min((H.E + 3) / 4, 3 * num_cu), 256, 0, st>>>(H);
            return;
        }
    k_head_act<NS, 1><<<H.E, 256, 0, st>>>(H);
}
// the launch for a run-time number of splits
inline void launch_head_act(const HeadActArgs &H, int num_cu, hipStream_t st)
{
    switch (H.nsplit) {
    case 1: launch_head_act_ns<1>(H, num_cu, st); break;
    case 2: launch_head_act_ns<2>(H, num_cu, st); break;
    case 3: launch_head_act_ns<3>(H, num_cu, st); break;
    case 4: launch_head_act_ns<4>(H, num_cu, st); break;
    case 5: launch_head_act_ns<5>(H, num_cu, st); break;
    case 6: launch_head_act_ns<6>(H, num_cu, st); break;
    default: launch_head_act_ns<7>(H, num_cu, st); break;
    }
}

// Acting on up to FEW_ROWS observations: fc1 and the head in one launch, whose workgroups leave their share of fc1 as
// words in device memory; the one that arrives last (above) has the whole hidden layer and finishes every row as
// k_head_act does.  Every sum is formed in the order of the launches for more observations (up to 192 in fp32, 511 in
// bf16), so that the same inputs give the same bits alone and among others.  One observation, against the two launches:
// 21.7 -> 19.3 us per call in fp32, 16.1 -> 14.0 in bf16; two: 21.8 -> 20.3, 16.4 -> 14.6 (with one counter, see below).  (A form whose lanes and waves added in an order of their own took
// 19.2 and 19.7 in fp32, 14.4 and 15.0 in bf16; with four rows that form had no gain left, 21.0 and 15.9.)
// Additions to words of one line of memory follow each other, about 10 ns each: at a single counter the 256 workgroups
// of the fp32 form queued for 2.5 us.  So they arrive in sixteen groups, each at a line of its own, and the last of a group
// at the counter of the groups: 19.6 -> 17.9 us per call (with the groups' counters in one line 20.3: the queue, and a
// second trip behind it).
// The counters are cleared by the conv launch in front, so that nothing of one call is left for the next.
constexpr int FEW_ROWS = 2;
constexpr int FEW_GROUPS = 16, FEW_LINE = 64;   // words from one counter to the next
constexpr int FEW_COUNTERS = FEW_GROUPS + 1;    // the groups', then the counter of the groups
__device__ __forceinline__ void few_clear(unsigned *arrivals, int tid)
{
    if (tid < FEW_COUNTERS) arrivals[tid * FEW_LINE] = 0;
}
struct Fc1HeadArgs {
    HeadActArgs head;      // (part, nsplit, split_stride: not used)
    const void *x;         // [E][3136] conv3's output, fp32 or bf16
    const void *w;         // [512][3136] in the same type
    float *h;              // the words that are handed over: fp32 [E][512] hidden units; bf16 [split][E][512] partial sums
    unsigned *arrivals;
};
struct FewLds {
    __attribute__((aligned(16))) float hid[FEW_ROWS][HID_LDS];
    float raw[FEW_ROWS][MAXR];
    int last;
};
// Called by all 256 threads, each wave's published words acknowledged: is this workgroup the last of `of`?
__device__ __forceinline__ bool few_last(const Fc1HeadArgs &A, FewLds &L, unsigned of /*>= FEW_GROUPS*/)
{
    sync_lds();
    if (threadIdx.x == 0) {
        const unsigned g = blockIdx.x % FEW_GROUPS;
        L.last = arrived_last(A.arrivals + g * FEW_LINE, (of - g + FEW_GROUPS - 1) / FEW_GROUPS) &&
                 arrived_last(A.arrivals + FEW_GROUPS * FEW_LINE, FEW_GROUPS);
    }
    sync_lds();
    return L.last;
}
// The head of the last workgroup.  SUMS == 1: the words are the hidden units; else that many partial sums of each
template <int ROWS, int SUMS> __device__ __forceinline__ void few_head(const Fc1HeadArgs &A, FewLds &L)
{
    const HeadActArgs &H = A.head;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l = tid & 15;
    const int K = H.K, R = K + (H.dueling ? 1 : 0);
    HeadRound H0, H1;
    float p[ROWS][2][SUMS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int sp = 0; sp < SUMS; ++sp) p[r][u][sp] = read_word(A.h + (sp * ROWS + r) * net::HID + tid + 256 * u);
    const float b0 = H.f1b[tid], b1 = H.f1b[tid + 256];
    head_rows1_load(H0, 0, H.head, K, H.dueling, tid);
    head_rows1_load(H1, 1, H.head, K, H.dueling, tid);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            float acc = 0.f;
#pragma unroll
            for (int sp = 0; sp < SUMS; ++sp) acc += p[r][u][sp];
            L.hid[r][hid_at(tid + 256 * u)] = SUMS == 1 ? p[r][u][0] : fmaxf(acc + (u ? b1 : b0), 0.f);
        }
    sync_lds();
    act_dots<ROWS>(H0, L.hid, L.raw, l);
    if (16 + 4 * wave < R) act_dots<ROWS>(H1, L.hid, L.raw, l);
    for (int round = 2; 16 * round < R; ++round) {   // more than 32 dot products: K > 31
        head_rows1_load(H0, round, H.head, K, H.dueling, tid);
        act_dots<ROWS>(H0, L.hid, L.raw, l);
    }
    sync_lds();
    if (wave < ROWS) act_choose(H, L.raw[wave], wave, lane);
}

// fp32: workgroup b forms hidden units 2b and 2b + 1 of every row, 25 KB of weights per CU, all requested at once, and each
// wave one unit of one row.  The sums of g32::k_fwd<GFc1, 32, 32, 7> in seven splits: a split's 448 inputs are two stages of
// seven slices of 32; a slice is one chain of 64 products over both stages, which takes inputs 4..7 of every eight between
// 0..3 (the matrix instruction's pairs); the seven slices are added in order, then the seven splits.  Those 49 chains are a
// lane each, out of LDS, where 32 elements lie 36 apart: lanes that read the same element of neighbouring slices then start
// in different banks.
template <int ROWS>
__global__ __launch_bounds__(256, 1) void k_fc1_head_act(Fc1HeadArgs A)
{
    constexpr int SPLITS = 7, SLICES = 7, SLICE = 32, PITCH = SLICE + 4;
    constexpr int GROUPS = net::A3 / SLICE;                       // slices of a vector: 98
    static_assert(GROUPS == SPLITS * 2 * SLICES && 8 * SPLITS <= 64 && SLICES == 7 && 2 * ROWS <= 4, "two stages per split; a wave per unit and row");
    constexpr int NW = 2 * net::A3 / 4, NX = ROWS * net::A3 / 4;  // pieces of 16 bytes
    constexpr int LW = (NW + 255) / 256, LX = (NX + 255) / 256;
    __shared__ __attribute__((aligned(16))) float v[(2 + ROWS) * GROUPS * PITCH];   // the two units' weights, the rows
    __shared__ FewLds L;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float4 *w = static_cast<const float4 *>(A.w) + (long)blockIdx.x * NW, *x = static_cast<const float4 *>(A.x);
    float4 wq[LW], xq[LX];
#pragma unroll
    for (int i = 0; i < LW; ++i) wq[i] = w[min(tid + 256 * i, NW - 1)];
#pragma unroll
    for (int i = 0; i < LX; ++i) xq[i] = x[min(tid + 256 * i, NX - 1)];
    const float b = A.head.f1b[2 * blockIdx.x + (wave & 1)];
    auto store = [&](int piece, float4 q) { *reinterpret_cast<float4 *>(&v[(piece >> 3) * PITCH + (piece & 7) * 4]) = q; };
#pragma unroll
    for (int i = 0; i < LW; ++i) store(min(tid + 256 * i, NW - 1), wq[i]);   // (past the end: the last one's bits again)
#pragma unroll
    for (int i = 0; i < LX; ++i) store(NW + min(tid + 256 * i, NX - 1), xq[i]);
    sync_lds();
    if (wave < 2 * ROWS) {
        // lane 8 p + j: slice j of split p (the eighth of every eight, and the last eight, repeat one)
        const int p = min(lane >> 3, SPLITS - 1), first = 2 * SLICES * p + min(lane & 7, SLICES - 1);
        const float *wp = v + ((wave & 1) * GROUPS + first) * PITCH, *xp = v + ((2 + (wave >> 1)) * GROUPS + first) * PITCH;
        float s = 0.f;
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
            for (int k = 0; k < SLICE; k += 8) {
                const int at = st * SLICES * PITCH + k;
                const float4 w0 = *reinterpret_cast<const float4 *>(wp + at), w1 = *reinterpret_cast<const float4 *>(wp + at + 4);
                const float4 x0 = *reinterpret_cast<const float4 *>(xp + at), x1 = *reinterpret_cast<const float4 *>(xp + at + 4);
                s = fmaf(x0.x, w0.x, s); s = fmaf(x1.x, w1.x, s);
                s = fmaf(x0.y, w0.y, s); s = fmaf(x1.y, w1.y, s);
                s = fmaf(x0.z, w0.z, s); s = fmaf(x1.z, w1.z, s);
                s = fmaf(x0.w, w0.w, s); s = fmaf(x1.w, w1.w, s);
            }
        float split = s, sum = 0.f;   // complete in lanes 8 p
        split += row_shl<1>(s); split += row_shl<2>(s); split += row_shl<3>(s);
        split += row_shl<4>(s); split += row_shl<5>(s); split += row_shl<6>(s);
#pragma unroll
        for (int j = 0; j < SPLITS; ++j) sum += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(split), 8 * j));
        if (lane == 0) publish_word(A.h + (wave >> 1) * net::HID + 2 * blockIdx.x + (wave & 1), fmaxf(sum + b, 0.f));
        words_acknowledged();
    }
    if (!few_last(A, L, net::HID / 2)) return;
    few_head<ROWS, 1>(A, L);
}
inline void launch_fc1_head_act(const Fc1HeadArgs &A, hipStream_t st)
{
    if (A.head.E == 1) k_fc1_head_act<1><<<net::HID / 2, 256, 0, st>>>(A);
    else k_fc1_head_act<FEW_ROWS><<<net::HID / 2, 256, 0, st>>>(A);
}

// --------------------------------------------------------------- RMSProp
// g = sum of the reduction splits (fixed order); v <- rho v + (1-rho) g^2;
// theta <- theta - lr g / sqrt(v + eps)   [centered: sqrt(v - m^2 + eps)].
// Each layer is a segment with its own block range.  A segment whose gradient
// arrives in several splits uses 64 parameters x 4 split-groups per block, so
// the split sum is spread over four times the threads and combined in LDS;
// a single-split segment (fc1, head) is a plain 256-parameters-per-block sweep.
struct RmsSeg {
    long begin, count;  // range of the blob
    const float *part;  // [nsplit][count]
    int nsplit;
    long stride;
    int block_begin;    // first blockIdx.x of this segment
};
struct RmsArgs {
    RmsSeg seg[5];
    float *theta, *v, *m, *g;
    __hip_bfloat16 *shadow;  // bf16 copy of theta (same order) or nullptr
    uint16_t *packed;        // with the bf16 copy: the conv weights in the forward launch's order (packed.h)
    uint16_t *back;          // ... and conv2's and conv3's once more in the orders of their input gradients (packed.h)
    float lr, rho, eps;
};

// What the update reads of parameter i
struct RmsOld { float v, th, m; };
__device__ __forceinline__ RmsOld rms_load(const RmsArgs &A, long i) { return RmsOld{A.v[i], A.theta[i], A.m ? A.m[i] : 0.f}; }
// store_g: false where the gradient already stands in A.g (a single partial written there by its kernel)
__device__ __forceinline__ void rms_apply(const RmsArgs &A, long i, float g, const RmsOld &old, bool store_g = true)
{
    float v = A.rho * old.v + (1.f - A.rho) * g * g;
    float denom;
    if (A.m) {
        float m = A.rho * old.m + (1.f - A.rho) * g;
        A.m[i] = m;
        denom = sqrtf(v - m * m + A.eps);
    } else {
        denom = sqrtf(v + A.eps);
    }
    float th = old.th - A.lr * g / denom;
    A.v[i] = v;
    A.theta[i] = th;
    if (store_g) A.g[i] = g;
    if (A.shadow) {
        A.shadow[i] = __float2bfloat16(th);
        if (i < net::F1W) {
            sp::store_packed_bf16(A.packed, i, th);
            sp::store_back_bf16(A.back, i, th);
        }
    }
}
// every operand is requested before the first store: the buffers may overlap as far as the compiler
// knows, so a load behind a store would wait for the arithmetic in front of that store
__device__ __forceinline__ void rms_update(const RmsArgs &A, long i, float g, bool store_g = true)
{
    const RmsOld old = rms_load(A, i);
    rms_apply(A, i, g, old, store_g);
}

// The segment that workgroup bx belongs to.  A macro, to be used on the KERNEL PARAMETER itself: picked
// through a reference or a copy of the argument structure, the segment array ends up in scratch memory.
#define RMS_SELECT_SEGMENT(A, bx, S)                                  \
    misc::RmsSeg S = (A).seg[0];                                     \
    {                                                                \
        int s_ = 0;                                                  \
        _Pragma("unroll") for (int t_ = 1; t_ < 5; ++t_)             \
            if ((bx) >= (A).seg[t_].block_begin) s_ = t_;            \
        if (s_ == 1) S = (A).seg[1];                                 \
        if (s_ == 2) S = (A).seg[2];                                 \
        if (s_ == 3) S = (A).seg[3];                                 \
        if (s_ == 4) S = (A).seg[4];                                 \
    }

// workgroup bx (256 threads) of the update, in segment S; red: 256 floats of LDS
__device__ __forceinline__ void rmsprop_block(const RmsArgs &A, const RmsSeg &S, int bx, float (*red)[64])
{
    const int tid = threadIdx.x;
    if (S.nsplit > 1) {
        const int pl = tid & 63, sg = tid >> 6;
        const long o = (long)(bx - S.block_begin) * 64 + pl;
        // what the update reads is requested along with the partial sums (by every thread, from a clamped
        // index: no branch, no wait), not in a round trip of its own behind their sum
        const RmsOld old = rms_load(A, S.begin + (o < S.count ? o : 0));
        float g = 0.f;
        if (o < S.count) {
#pragma unroll 8
            for (int t = sg; t < S.nsplit; t += 4) g += S.part[t * S.stride + o];
        }
        red[sg][pl] = g;
        __syncthreads();
        if (sg == 0 && o < S.count)
            rms_apply(A, S.begin + o, (red[0][pl] + red[1][pl]) + (red[2][pl] + red[3][pl]), old);
    } else {
        const long o = (long)(bx - S.block_begin) * 256 + tid;
        if (o < S.count) rms_update(A, S.begin + o, S.part[o], S.part != A.g + S.begin);
    }
}
__global__ __launch_bounds__(256) void k_rmsprop(RmsArgs A)
{
    __shared__ float red[4][64];
    RMS_SELECT_SEGMENT(A, (int)blockIdx.x, S)
    rmsprop_block(A, S, blockIdx.x, red);
}

// fp32 -> bf16 copy (round to nearest even)
__global__ void k_to_bf16(const float *src, __hip_bfloat16 *dst, long n)
{
    long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = __float2bfloat16(src[i]);
}

// ------------------------------------------------- layout permutations
// canonical blob <-> internal blob (see net.h).  dir 0: dst(internal) from
// src(canonical); dir 1: dst(canonical) from src(internal).
__global__ void k_permute(const float *src, float *dst, long n, int dir)
{
    long e = (long)blockIdx.x * blockDim.x + threadIdx.x;  // canonical index
    if (e >= n) return;
    long in = e;
    if (e >= net::C2W && e < net::C2B) {  // [o][c][p][q] -> [o][p][q][c]
        long t = e - net::C2W;
        int q = t % 4, p = (t / 4) % 4, c = (t / 16) % 32, o = t / 512;
        in = net::C2W + ((o * 4 + p) * 4 + q) * 32 + c;
    } else if (e >= net::C3W && e < net::C3B) {
        long t = e - net::C3W;
        int q = t % 3, p = (t / 3) % 3, c = (t / 9) % 64, o = t / 576;
        in = net::C3W + ((o * 3 + p) * 3 + q) * 64 + c;
    } else if (e >= net::F1W && e < net::F1B) {  // [o][c*49 + hw] -> [o][hw*64 + c]
        long t = e - net::F1W;
        int k = t % 3136, o = t / 3136;
        int c = k / 49, hw = k % 49;
        in = net::F1W + (long)o * 3136 + hw * 64 + c;
    }
    if (dir == 0) dst[in] = src[e];
    else dst[e] = src[in];
}

__global__ void k_fill(float *p, float v, long n)
{
    long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// ------------------------------------------------------------- sum-tree
// Heap layout: tree[1] root, children of i at 2i and 2i+1, leaves at
// tree[L..2L); tree[2L] holds the running maximum priority.
// Internal nodes from the leaves, twelve levels per pass.  The tree over Lcur leaves (leaves at
// tree[Lcur, 2 Lcur)) is cut into blocks of BL = min(Lcur, 4096) leaves, sixteen leaves per thread: a thread
// forms the four levels above its own leaves in registers, a wave the next six by lane exchange, wave 0 the
// last two from the waves' sums in LDS, so the block waits at ONE barrier (a barrier per level and an LDS
// copy of the block took 6.9 us per launch at a million leaves, this 4).  Node = left + right in fp32, so every
// node has the bits that any other order of repair gives.
// v: the thread's sixteen leaves (threads at or past BL / 16 do not count); 16 <= BL <= 4096; b: number of the
// block.  Returns the block's root in every thread of wave 0.  sh: 4 floats of LDS.
__device__ __forceinline__ float tree_block16(float *tree, long Lcur, int BL, long b, const float (&v)[16], float *sh)
{
    const int tid = threadIdx.x, nthr = BL / 16;
    const bool on = tid < nthr;
    long at = (Lcur + b * BL) / 2 + 8L * tid;   // heap index of the thread's first node, one level up
    float w8[8], w4[4], w2[2];
#pragma unroll
    for (int i = 0; i < 8; ++i) w8[i] = v[2 * i] + v[2 * i + 1];
#pragma unroll
    for (int i = 0; i < 4; ++i) w4[i] = w8[2 * i] + w8[2 * i + 1];
#pragma unroll
    for (int i = 0; i < 2; ++i) w2[i] = w4[2 * i] + w4[2 * i + 1];
    float s = w2[0] + w2[1];
    if (on) {
        // (a run of eight nodes starts at a multiple of eight; the heap itself is 256-byte aligned)
        *reinterpret_cast<float4 *>(tree + at) = float4{w8[0], w8[1], w8[2], w8[3]};
        *reinterpret_cast<float4 *>(tree + at + 4) = float4{w8[4], w8[5], w8[6], w8[7]};
        *reinterpret_cast<float4 *>(tree + at / 2) = float4{w4[0], w4[1], w4[2], w4[3]};
        *reinterpret_cast<float2 *>(tree + at / 4) = float2{w2[0], w2[1]};
        tree[at / 8] = s;
    }
    at /= 8;
    auto level = [&](int k, float other) {
        s += other;
        if (on && (nthr >> k) >= 1 && (tid & ((1 << k) - 1)) == 0) tree[at >> k] = s;
    };
    level(1, lane_xor<1>(s));
    level(2, lane_xor<2>(s));
    level(3, lane_xor<4>(s));
    level(4, lane_xor<8>(s));
    level(5, lane_xor<16>(s));
    level(6, lane_xor<32>(s));
    if (nthr > 64) {   // uniform
        if ((tid & 63) == 0) sh[tid >> 6] = s;
        __syncthreads();
        if (tid < 64) {
            const int nw = nthr / 64;   // 2 or 4 waves
            const long top = (Lcur + b * BL) / 1024;
            float a0 = sh[0] + sh[1], a1 = 0.f;
            if (nw == 4) a1 = sh[2] + sh[3];
            if (tid == 0) {
                tree[top / 2] = a0;
                if (nw == 4) {
                    tree[top / 2 + 1] = a1;
                    tree[top / 4] = a0 + a1;
                }
            }
            s = nw == 4 ? a0 + a1 : a0;
        }
    }
    return s;
}
__device__ __forceinline__ void tree_load16(const float *tree, long Lcur, int BL, long b, float (&v)[16])
{
    const float4 *p = reinterpret_cast<const float4 *>(tree + Lcur + b * BL + 16L * ((int)threadIdx.x < BL / 16 ? threadIdx.x : 0));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float4 q = p[i];
        v[4 * i] = q.x; v[4 * i + 1] = q.y; v[4 * i + 2] = q.z; v[4 * i + 3] = q.w;
    }
}
// a block of any launch above the leaves' own (trees of more than 4096 x 4096 leaves only)
__global__ __launch_bounds__(256) void k_tree_rebuild(float *tree, long Lcur, int BL)
{
    __shared__ float sh[4];
    if (BL < 16) {
        if (threadIdx.x == 0)
            for (long i = Lcur - 1; i >= 1; --i) tree[i] = tree[2 * i] + tree[2 * i + 1];
        return;
    }
    float v[16];
    tree_load16(tree, Lcur, BL, blockIdx.x, v);
    (void)tree_block16(tree, Lcur, BL, blockIdx.x, v, sh);
}

// Whole tree in one launch: every workgroup builds the block of leaves it holds in registers, and the one that
// arrives last builds the levels above the nblk block roots (nblk <= 4096; more: k_tree_rebuild goes on).
// Must be called by all 256 threads.  count: one word of the tree's state area.
__device__ __forceinline__ void tree_build_leaves(float *tree, long L, int BL, long b, int nblk, const float (&v)[16],
                                                  unsigned *count, float *sh /*8*/)
{
    const float root = tree_block16(tree, L, BL, b, v, sh);
    if (nblk == 1 || nblk > 4096) return;
    if (threadIdx.x == 0) {
        publish_word(tree + nblk + b, root);
        words_acknowledged();
        sh[4] = arrived_last(count, (unsigned)nblk) ? 1.f : 0.f;
    }
    __syncthreads();
    if (sh[4] == 0.f) return;
    if (nblk < 16) {   // 2, 4 or 8
        if (threadIdx.x == 0)
            for (int i = nblk - 1; i >= 1; --i)
                tree[i] = 2 * i >= nblk ? read_word(tree + 2 * i) + read_word(tree + 2 * i + 1) : tree[2 * i] + tree[2 * i + 1];
        return;
    }
    float r[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) r[i] = read_word(tree + nblk + ((int)threadIdx.x < nblk / 16 ? 16 * threadIdx.x + i : i));
    (void)tree_block16(tree, nblk, nblk, 0, r, sh);
}

// Bulk fill: leaf i = fp32(p_i^alpha) for i < n, 0 beyond, and the tree above; grid (L / BL)
__global__ __launch_bounds__(256) void k_tree_fill(float *tree, long L, int BL, const float *p, long n, float alpha,
                                                   unsigned *count)
{
    __shared__ float sh[8];
    if (BL < 16) {   // a tree of eight leaves
        if (threadIdx.x == 0) {
            for (long i = 0; i < L; ++i) tree[L + i] = i < n ? (float)pow((double)p[i], (double)alpha) : 0.f;
            for (long i = L - 1; i >= 1; --i) tree[i] = tree[2 * i] + tree[2 * i + 1];
            tree[0] = 0.f;
        }
        return;
    }
    const long i0 = (long)blockIdx.x * BL + 16L * threadIdx.x;
    const bool on = (int)threadIdx.x < BL / 16;
    float v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = on && i0 + i < n ? p[i0 + i] : 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = on && i0 + i < n ? (float)pow((double)v[i], (double)alpha) : 0.f;
    if (on) {
        float4 *d = reinterpret_cast<float4 *>(tree + L + i0);
#pragma unroll
        for (int i = 0; i < 4; ++i) d[i] = float4{v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]};
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) tree[0] = 0.f;
    tree_build_leaves(tree, L, BL, blockIdx.x, gridDim.x, v, count, sh);
}

// Store path of many environment streams: one time step for each of E streams of C slots (C >= 16), at local
// slot l (t steps stored per stream before), in ONE launch.  The first nblk workgroups rebuild the tree over
// the whole ring, forming the leaves the new time step settles as they go; the other E copy a stream's
// frame and transition data.  The leaves follow the rules of the one-stream store path in the stream's
// own sub-ring (see k_replay_store): the transition at local slot l - 1 has just become complete and enters with
// leaf = fp32(max_p^alpha) unless its state stack would reach back before the stream's start (t - 1 < 3) or across
// an episode end; the slot just written and the three after it get leaf 0.  They depend on transition data of
// earlier time steps only, which this launch does not write.
// (A write launch and two rebuild launches took 9.3 + 2 x 6.9 us for 2048 streams over a million slots.)
// One power per thread, its flags in flight with the leaves: 10.7 -> 10.1 us for those, 6.9 -> 6.3 for 32 streams over 200,000
// slots (a power and three dependent flags wherever one of the sixteen slots enters before).
struct StoreEnvsArgs {
    uint8_t *frames;
    int32_t *meta_a;
    float *meta_r;
    uint8_t *meta_done;
    int E;
    int C, l;
    long t;
    const uint8_t *src;
    const int32_t *a;
    const float *r;
    const uint8_t *done;
    float *tree;
    long L;
    int BL, nblk;
    float alpha;
    unsigned *count;
};
__global__ __launch_bounds__(256) void k_store_envs(StoreEnvsArgs A)
{
    __shared__ float sh[8];
    const int tid = threadIdx.x;
    if ((int)blockIdx.x >= A.nblk) {
        const long e = (long)blockIdx.x - A.nblk, slot = e * A.C + A.l;
        const uint4 *s = reinterpret_cast<const uint4 *>(A.src + e * net::FRAME);
        uint4 *d = reinterpret_cast<uint4 *>(A.frames + slot * net::FRAME);
        for (int q = tid; q < net::FRAME / 16; q += 256) d[q] = s[q];
        if (tid == 0) {
            A.meta_a[slot] = A.a[e];
            A.meta_r[slot] = A.r[e];
            A.meta_done[slot] = A.done[e];
        }
        return;
    }
    const long slot0 = (long)blockIdx.x * A.BL + 16L * tid;
    int e = (int)((uint32_t)slot0 / (uint32_t)A.C), off = (int)slot0 - e * A.C;   // (at most 2^30 slots)
    // The transition that becomes complete is the one at local slot l - 1; of sixteen slots in a row (C >= 16) one at most
    // is such a slot, `ahead` slots from the thread's first, so its three flags are requested along with the leaves.
    const int enters = A.l > 0 ? A.l - 1 : A.C - 1;
    const int ahead = off <= enters ? enters - off : enters - off + A.C;
    const int stream = e + (off + ahead >= A.C ? 1 : 0);
    const uint8_t *flags = A.meta_done + (long)min(stream, A.E - 1) * A.C;
    uint8_t ended[3];
#pragma unroll
    for (int k = 1; k <= 3; ++k) ended[k - 1] = flags[enters - k < 0 ? enters - k + A.C : enters - k];
    const float mp = A.tree[2 * A.L];
    float v[16];
    tree_load16(A.tree, A.L, A.BL, blockIdx.x, v);
    bool dirty = false;
    if (tid < A.BL / 16) {
        float entering = 0.f;
        if (ahead < 16 && stream < A.E && A.t - 1 >= 3 && !(ended[0] | ended[1] | ended[2])) entering = (float)pow((double)mp, (double)A.alpha);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            int d = off - (A.l - 1);   // distance of this slot behind local slot l - 1, cyclic
            if (d < 0) d += A.C;
            if (d >= A.C) d -= A.C;    // (l = 0: slot l - 1 is the sub-ring's last)
            if (d < 5 && e < A.E && (d > 0 || A.t >= 1)) {
                v[i] = d == 0 ? entering : 0.f;
                dirty = true;
            }
            if (++off == A.C) { off = 0; ++e; }
        }
        if (dirty) {
            float4 *p = reinterpret_cast<float4 *>(A.tree + A.L + slot0);
#pragma unroll
            for (int i = 0; i < 4; ++i) p[i] = float4{v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]};
        }
    }
    tree_build_leaves(A.tree, A.L, A.BL, blockIdx.x, A.nblk, v, A.count, sh);
}

// The sampling kernel.  With `count` (per_sample) the workgroup that arrives last also divides the raw weights
// by their maximum over the minibatch; without it the consumer does.
__global__ __launch_bounds__(256) void k_per_sample(SampleArgs A, unsigned *count)
{
    __shared__ float sh[16];
    __shared__ int last;
    const int lane = threadIdx.x & 63;
    const int j = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (j < A.B) {
        const int jj[1] = {j};
        long slot[1];
        float leaf[1];
        const float total = per_sample_walk<1>(A, jj, lane, slot, leaf);
        if (lane == 0) per_sample_emit(A, j, slot[0], total, leaf[0], count != nullptr);
    }
    if (!count) return;
    words_acknowledged();
    __syncthreads();
    if (threadIdx.x == 0) last = arrived_last(count, gridDim.x);
    __syncthreads();
    if (!last) return;
    float w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = read_word(A.is_w + min((int)threadIdx.x + 256 * k, A.B - 1));
    const float wmax = block_max_1024(fmaxf(fmaxf(w[0], w[1]), fmaxf(w[2], w[3])), sh);
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if ((int)threadIdx.x + 256 * k < A.B) A.is_w[threadIdx.x + 256 * k] = wmax > 0.f ? w[k] / wmax : 0.f;
}

// Leaf-to-root repair by the threads of ONE workgroup, each starting from its own distinct leaf
// with the leaf's new value v: a level is one exchange through memory: every walker publishes
// its node, the workgroup meets, every walker reads its sibling as it now stands and forms
// parent = left + right (fp32; the sum is commutative, so walkers whose paths have merged hold
// identical values and store them to the same word; the result is bit-identical to repairing
// the paths one after another).  All walkers sit on one compute unit, so workgroup scope is
// enough: a store is complete before the barrier and the load after it sees it.  Every thread
// of the workgroup must call this (it contains barriers).
// W walkers per thread (a thread's walkers take the levels together).
template <int W>
__device__ __forceinline__ void tree_walk(float *tree, int (&node)[W], float (&v)[W], const bool (&walk)[W], int levels)
{
#pragma unroll
    for (int w = 0; w < W; ++w)
        if (walk[w]) __hip_atomic_store(&tree[node[w]], v[w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    for (int l = 0; l < levels; ++l) {
        __syncthreads();
        float vs[W];
#pragma unroll
        for (int w = 0; w < W; ++w)
            vs[w] = walk[w] ? __hip_atomic_load(&tree[node[w] ^ 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) : 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w)
            if (walk[w]) {
                v[w] = v[w] + vs[w];
                node[w] >>= 1;
                __hip_atomic_store(&tree[node[w]], v[w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
    }
}
__device__ __forceinline__ void tree_walk(float *tree, int node, float v, bool walk, int levels)
{
    int n1[1] = {node};
    float v1[1] = {v};
    const bool w1[1] = {walk};
    tree_walk<1>(tree, n1, v1, w1, levels);
}

// Priority update (Eq.11): a single workgroup, one thread per entry.  Repeated
// slots are settled first ("last occurrence wins" is an integer maximum over
// entry numbers in an LDS hash table keyed by leaf).  The surviving entries
// then repair the tree level by level, parent = left + right in fp32; the sum
// is commutative, so the result is bit-identical to a sequential repair.
constexpr int PU_SLOTS = 2048;  // hash slots (at most 1024 live keys)
__device__ __forceinline__ int pu_hash(int key) { return (int)(((unsigned)key * 2654435761u) >> 21); }
// returns the slot of `key`; *first is set when this call created it
__device__ __forceinline__ int pu_insert(int *keys, int key, bool *first)
{
    int h = pu_hash(key);
    for (;;) {
        const int old = atomicCAS(&keys[h], -1, key);
        if (old == -1 || old == key) {
            *first = old == -1;
            return h;
        }
        h = (h + 1) & (PU_SLOTS - 1);
    }
}
__device__ __forceinline__ int pu_find(const int *keys, int key)
{
    int h = pu_hash(key);
    for (;;) {
        const int k = keys[h];
        if (k == key) return h;
        if (k == -1) return -1;
        h = (h + 1) & (PU_SLOTS - 1);
    }
}

struct PerUpdateArgs {
    float *tree;
    long L;
    int levels;
    long size;
    const int32_t *idx;
    const float *td_abs;
    int n;
    float alpha, eps;
    int leaves_fixed;   // 1: priority exponent 0 over a tree of ones: a leaf's new value is its old one, so
                        // only the running maximum priority is updated and no node is read or written
};
constexpr int PU_LDS_WORDS = 2 * PU_SLOTS + 16;  // LDS of per_update_body, in 4-byte words

// The whole workgroup must call this; it handles W entries per thread (W * blockDim.x >= n).
// lds: PU_LDS_WORDS words.  The walk stops after `first_levels` levels and leaves every walker (node, value,
// active) in `state`, for per_update_resume to take to the root later:
// entry j at state[j], state[STATE_STRIDE + j], state[2 * STATE_STRIDE + j].
constexpr int STATE_STRIDE = 1024;
template <int W>
__device__ __forceinline__ void per_update_body(const PerUpdateArgs &A, int *lds, int first_levels, int *state)
{
    int *keys = lds, *ivals = lds + PU_SLOTS;  // ivals: largest entry number naming the slot's leaf
    float *sh = reinterpret_cast<float *>(lds + 2 * PU_SLOTS);
    float *tree = A.tree;
    const long L = A.L, size = A.size;
    const int n = A.n;
    const int32_t *idx = A.idx;
    const float *td_abs = A.td_abs;
    const float alpha = A.alpha, eps = A.eps;
    const int tid = threadIdx.x, nt = blockDim.x;
    int my[W];
    float p[W];
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const int j = tid + w * nt;
        my[w] = -1;
        p[w] = 0.f;
        if (j < n) {
            const int v = idx[j];
            p[w] = (float)((double)fabsf(td_abs[j]) + (double)eps);
            // an entry with a slot outside the ring or a non-finite error is skipped: its leaf keeps
            // its value, and the tree stays a tree of finite sums
            if (v >= 0 && v < size && p[w] <= 3.4028234663852886e38f) my[w] = v;   // finite: false for NaN and infinity
        }
    }
    for (int t = tid; t < PU_SLOTS; t += nt) { keys[t] = -1; ivals[t] = -1; }
    __syncthreads();
    int node[W], slot[W];
    float pm = 0.f;
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const bool valid = my[w] >= 0;
        node[w] = (int)L + (valid ? my[w] : 0);
        slot[w] = 0;
        if (valid) {
            bool first;
            slot[w] = pu_insert(keys, node[w], &first);
            atomicMax(&ivals[slot[w]], tid + w * nt);
            pm = fmaxf(pm, p[w]);
        }
    }
    const float pmax = block_max_1024(pm, sh);  // contains barriers
    if (tid == 0) tree[2 * L] = fmaxf(tree[2 * L], pmax);
    if (A.leaves_fixed) return;   // uniform for the workgroup
    // One walker per distinct leaf (the last entry naming it) walks to the root.  A level is one
    // exchange through memory: every walker publishes its node, the workgroup meets, every
    // walker reads its sibling as it now stands.  Walkers whose paths have merged hold the same
    // value and store it to the same word.
    bool walk[W];
    float v[W];
#pragma unroll
    for (int w = 0; w < W; ++w) {
        walk[w] = my[w] >= 0 && ivals[slot[w]] == tid + w * nt;
        v[w] = (float)pow((double)p[w], (double)alpha);
    }
    tree_walk<W>(tree, node, v, walk, first_levels);
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const int j = tid + w * nt;
        if (j < STATE_STRIDE) {
            state[j] = node[w];
            state[STATE_STRIDE + j] = __float_as_int(v[w]);
            state[2 * STATE_STRIDE + j] = walk[w] ? 1 : 0;
        }
    }
}

// A later part of a split priority update: the walkers that the part before left `done_levels`
// levels above their leaves climb `walk_levels` more (to the root if that is all that is left;
// otherwise they are left in `state` again).  Same workgroup shape as the first part.
template <int W>
__device__ __forceinline__ void per_update_resume(const PerUpdateArgs &A, int done_levels, int walk_levels, int *state)
{
    const int tid = threadIdx.x, nt = blockDim.x;
    if (A.leaves_fixed) return;
    int node[W];
    float v[W];
    bool walk[W];
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const int j = tid + w * nt;
        const bool in = j < A.n && j < STATE_STRIDE;
        node[w] = in ? state[j] : 1;
        v[w] = in ? __int_as_float(state[STATE_STRIDE + j]) : 0.f;
        walk[w] = in && state[2 * STATE_STRIDE + j] != 0;
    }
    const bool last = done_levels + walk_levels >= A.levels;
    tree_walk<W>(A.tree, node, v, walk, last ? A.levels - done_levels : walk_levels);
    if (!last) {
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const int j = tid + w * nt;
            if (j < A.n && j < STATE_STRIDE) {
                state[j] = node[w];
                state[STATE_STRIDE + j] = __float_as_int(v[w]);
            }
        }
    }
}

// The update as a launch of its own.  What bounds it is one compute unit's rate of scattered words, a store and a load per
// entry and level: 6.4 us for 128 entries over a million slots, 10.3 for 512, 19.3 for 1024 (back to back).
// PARTS: the part of the tree that holds the slots is cut into PU_PARTS subtrees, a workgroup each, which picks its entries
// out of the list, repairs its subtree and publishes the subtree's root; the one that arrives last forms the few nodes above:
// 7.2 and 7.5 us for 512 and 1024.  (With the entries sorted, all siblings requested at once and values handed over in LDS the
// same split took 2 us more, 8.1 where one workgroup takes 6; in one workgroup 15 for 512.)
// Entries that all lie in one part are the work of its workgroup, up to the tree's root, and no other arrives: 8.4 and 12.3 us
// for 512 and 1024 of a million slots, where one workgroup takes 8.1 and 12.0 and a walk to the part's root, the arrivals and the
// nodes above 9.6 and 14.1.
// It pays from 384 entries on over more than 2^14 slots (7.2 against 8.9 us over a million, 6.4 against 6.5 over 20,000), from 512
// over 2^13 to 2^14 (6.3 against 6.6 over 10,000; 384: 6.2 against 6.1) and from 640 over 2^12 to 2^13 (6.4 against 6.5 over 4097,
// 6.3 against 6.9 over 8192; 512: 6.36 against 6.10, 6.20 against 6.32).
constexpr int PU_PART_BITS = 5, PU_PARTS = 1 << PU_PART_BITS;
constexpr int PU_PARTS_BITS = 13;   // of the slots' numbers, at least
constexpr int pu_parts_from(int bits) { return bits >= 15 ? 384 : bits == 14 ? 512 : 640; }   // entries
template <bool PARTS>
__global__ __launch_bounds__(1024) void k_per_update(PerUpdateArgs A, int levels /*of a workgroup's subtree*/, unsigned *count)
{
    __shared__ int keys[PU_SLOTS], ivals[PU_SLOTS];   // see per_update_body
    __shared__ float sh[16];
    float *const tree = A.tree;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nw = blockDim.x >> 6, part = blockIdx.x;
    int my = -1, of_first = 0;
    float p = 0.f;
    // (an atomic load, so that it stays here: the compiler would move it behind the others, another trip to memory)
    if constexpr (PARTS) of_first = __hip_atomic_load(A.idx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (tid < A.n) {
        const int v = A.idx[tid];
        p = (float)((double)fabsf(A.td_abs[tid]) + (double)A.eps);
        if (v >= 0 && v < A.size && p <= 3.4028234663852886e38f) my = v;   // others are skipped (see per_update_body)
    }
    for (int t = tid; t < PU_SLOTS; t += blockDim.x) { keys[t] = -1; ivals[t] = -1; }
    float pmax = my >= 0 ? p : 0.f;
    auto raise_max = [&] {
        pmax = block_max_1024(pmax, sh);   // contains barriers
        if (tid == 0) tree[2 * A.L] = fmaxf(tree[2 * A.L], pmax);
    };
    bool alone = false;
    if constexpr (PARTS) {
        // this part's entries, in the list's order, to the first threads; the waves that are left without one leave, and
        // barriers no longer count them.  Every workgroup learns whether all entries lie in the part of the list's first one
        constexpr int ELSEWHERE = 1 << 16;
        __shared__ int found[16], own[1024];
        __shared__ float own_p[1024];
        const int its = my >= 0 ? my >> levels : -1, first_part = of_first >= 0 ? of_first >> levels : -1;
        const bool mine = its == part;
        const uint64_t here = __ballot(mine), elsewhere = __ballot(its >= 0 && its != first_part);
        if (lane == 0) found[wave] = __popcll(here) + (elsewhere ? ELSEWHERE : 0);
        if (part == 0) {   // uniform for the workgroup
            pmax = wave_max(pmax);
            if (lane == 0) sh[wave] = pmax;
        }
        sync_lds();
        // (a lane per wave: short code, which these few us fetch as they go)
        const int of_wave = (lane & 15) < nw ? found[lane & 15] : 0;
        const int sum = __builtin_amdgcn_readfirstlane(wave_sum<8>(of_wave));
        const int before = wave_sum<8>((lane & 15) < wave ? of_wave : 0);
        const int m = sum & (ELSEWHERE - 1), at = (before & (ELSEWHERE - 1)) + __popcll(here & ((1ull << lane) - 1));
        alone = sum < ELSEWHERE;
        if (part == 0 && wave == 0) {
            pmax = wave_max(lane < nw ? sh[lane] : 0.f);
            if (lane == 0) tree[2 * A.L] = fmaxf(tree[2 * A.L], pmax);
        }
        if (mine) {
            own[at] = my;
            own_p[at] = p;
        }
        sync_lds();
        if ((alone || wave > 0) && 64 * wave >= m) return;
        if (alone) levels = A.levels;   // nobody to wait for
        my = tid < m ? own[tid] : -1;
        p = tid < m ? own_p[tid] : 0.f;
    } else sync_lds();
    int node[1] = {(int)A.L + (my >= 0 ? my : 0)}, slot = 0;
    if (my >= 0) {
        bool first;
        slot = pu_insert(keys, node[0], &first);
        atomicMax(&ivals[slot], tid);
    }
    if constexpr (PARTS) sync_lds();
    else {
        raise_max();   // (in front of the insertions, with a barrier of their own, 0.13 us more per call)
        if (A.leaves_fixed) return;
    }
    const bool walk[1] = {my >= 0 && ivals[slot] == tid};   // one walker per leaf: the last entry naming it
    float v[1] = {(float)pow((double)p, (double)A.alpha)};
    tree_walk<1>(tree, node, v, walk, levels);
    if constexpr (PARTS) {
        if (alone) return;
        // every walker has the subtree's root
        if (walk[0]) publish_word(tree + node[0], v[0]);
        words_acknowledged();
        sync_lds();
        if (wave > 0) return;
        int last = 0;
        if (lane == 0) last = arrived_last(count, PU_PARTS);
        if (!__builtin_amdgcn_readfirstlane(last)) return;
        // a lane per part; above their common root the path is the leftmost one, whose siblings no entry lies under
        const int roots = (int)(A.L >> levels), top = roots >> PU_PART_BITS;
        float s = read_word(tree + roots + (lane & (PU_PARTS - 1)));
        const float right = lane < 31 && top >> lane > 1 ? tree[(top >> lane) + 1] : 0.f;
        auto level = [&](int k, float other) {
            s += other;
            if (lane < PU_PARTS && (lane & ((1 << k) - 1)) == 0) tree[(roots + lane) >> k] = s;
        };
        level(1, lane_xor<1>(s));
        level(2, lane_xor<2>(s));
        level(3, lane_xor<4>(s));
        level(4, lane_xor<8>(s));
        level(5, lane_xor<16>(s));
        for (int k = 0; top >> k > 1; ++k) {
            s += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(right), k));
            if (lane == 0) tree[top >> (k + 1)] = s;
        }
    }
}
inline void launch_per_update(const PerUpdateArgs &A, unsigned *count, hipStream_t st)
{
    const int threads = (A.n + 63) / 64 * 64;
    int bits = 0;   // of a slot's number: at most A.levels
    while ((1l << bits) < A.size) ++bits;
    if (!A.leaves_fixed && bits >= PU_PARTS_BITS && A.n >= pu_parts_from(bits)) k_per_update<true><<<PU_PARTS, threads, 0, st>>>(A, bits - PU_PART_BITS, count);
    else k_per_update<false><<<1, threads, 0, st>>>(A, A.levels, count);
}

// Repair of the tree above `cnt` CONSECUTIVE leaves first .. first + cnt - 1 (heap indexes), whose new values
// stand in val[0 .. cnt) (LDS, at least cnt + 1 floats): at every level the touched nodes are one run, and the
// only other nodes a level needs are the sibling left of the run and the one right of it, which no leaf of the
// run lies under.  So all of them are requested at once (sib[0 .. 2 * levels), the caller's sibling_load) and
// the walk to the root is one round trip to memory instead of one per level; node = left + right in fp32 as
// everywhere, so the bits are those of any other order of repair.  While a run is wider than two nodes the
// workgroup halves it in LDS, from there on wave 0 carries it in registers.  Every thread must call this.
// Measured (one time step, 1M-slot ring): 3.3 us for the whole store as one launch, against 3.3 + 5.7 us and
// a second launch for the frame copy and the level-by-level walk.
__device__ __forceinline__ float sibling_load(const float *tree, int first, int cnt, int levels, int t)
{
    // t < levels: left sibling of level t's run; t in [64, 64 + levels): right sibling (levels <= 30)
    const int l = t & 63;
    if (t >= 128 || l >= levels) return 0.f;
    const int lo = first >> l, hi = (first + cnt - 1) >> l;
    const bool want = t < 64 ? (lo & 1) : !(hi & 1);
    return want ? tree[t < 64 ? lo - 1 : hi + 1] : 0.f;
}
__device__ __forceinline__ void tree_repair_run(float *tree, int first, int cnt, int levels, float *val, const float *sib)
{
    const int tid = threadIdx.x, nt = blockDim.x;
    int lo = first, hi = first + cnt - 1, l = 0;
    __syncthreads();
    while (hi - lo > 1) {   // uniform
        const int plo = lo >> 1, phi = hi >> 1;
        for (int i = tid; i <= hi - lo; i += nt) tree[lo + i] = val[i];
        float pv = 0.f;      // a parent run is at most half as long plus one: one parent per thread
        const int p = plo + tid;
        if (p <= phi)
            pv = (2 * p < lo ? sib[l] : val[2 * p - lo]) + (2 * p + 1 > hi ? sib[64 + l] : val[2 * p + 1 - lo]);
        __syncthreads();
        if (p <= phi) val[tid] = pv;
        __syncthreads();
        lo = plo; hi = phi; ++l;
    }
    if (tid >= 64) return;
    float x0 = val[0], x1 = val[hi - lo];
    for (;; ++l) {
        if (tid == 0) tree[lo] = x0;
        if (tid == 1 && hi != lo) tree[hi] = x1;
        if (l >= levels) break;
        const float sl = sib[l], sr = sib[64 + l];
        if (hi == lo) x0 = x1 = (lo & 1) ? sl + x0 : x0 + sr;
        else if (lo & 1) { x0 = sl + x0; x1 = x1 + sr; }
        else x0 = x1 = x0 + x1;
        lo >>= 1; hi >>= 1;
    }
}

// Store path (Alg.1 "store transition", Alg.2 "with maximal priority"): n time steps go to ring slots
// h0 .. h0+n-1 (stream positions seq0 .. seq0+n-1).  Workgroups 1 .. n copy a time step each; workgroup 0
// settles the leaves and the tree, which depend on earlier time steps and on the flags in `done` only, so
// both run in one launch.  Thread j of workgroup 0 settles the leaf of slot h0-1+j: for j < n that transition
// becomes complete (its s' ends in a new frame) and enters with leaf = fp32(max_p^alpha), unless its state
// stack would reach back before the start of the stream or across an episode end (done at one of the three
// slots before it), in which case it is never sampled (leaf 0); the last written slot (not complete
// yet) and the three after it, whose windows mix the newest frames with the oldest (j = n ..
// n+3), get leaf 0.  n + 4 <= 1024 distinct slots; blockDim.x >= n + 4.
struct StoreArgs {
    uint8_t *frames;
    int32_t *meta_a;
    float *meta_r;
    uint8_t *meta_done;
    long cap, h0, seq0;
    int n;
    const uint8_t *src;
    const int32_t *a;
    const float *r;
    const uint8_t *done;
    float *tree;
    long L;
    int levels;
    float alpha;
};
__global__ __launch_bounds__(1024) void k_replay_store(StoreArgs A)
{
    if (blockIdx.x > 0) {
        const long j = (long)blockIdx.x - 1;
        const long slot = (A.h0 + j) % A.cap;
        const uint4 *s = reinterpret_cast<const uint4 *>(A.src + j * net::FRAME);
        uint4 *d = reinterpret_cast<uint4 *>(A.frames + slot * net::FRAME);
        for (int t = threadIdx.x; t < net::FRAME / 16; t += blockDim.x) d[t] = s[t];
        if (threadIdx.x == 0) {
            A.meta_a[slot] = A.a[j];
            A.meta_r[slot] = A.r[j];
            A.meta_done[slot] = A.done[j];
        }
        return;
    }
    __shared__ float val[1026], sib[128];
    const int j = threadIdx.x, n = A.n, cnt = n + 4;
    long slot = (A.h0 - 1 + j) % A.cap;
    if (slot < 0) slot += A.cap;
    const bool run = A.h0 >= 1 && A.h0 - 1 + cnt <= A.cap;   // the slots do not wrap around the ring's end
    const int first = (int)(A.L + A.h0 - 1);
    const float mp = A.tree[2 * A.L];
    const float sv = run && j < 128 ? sibling_load(A.tree, first, cnt, A.levels, j) : 0.f;
    float v = 0.f;
    if (j < n) {
        bool valid = A.seq0 - 1 + j >= 3;   // stream position of the transition's own frame
#pragma unroll
        for (int k = 1; k <= 3; ++k) {
            // a flag of this call is read from the caller's array: its slot is being written meanwhile
            const int q = j - 1 - k;
            long sk = slot - k;
            if (sk < 0) sk += A.cap;
            if (q >= 0 ? A.done[q] : A.meta_done[sk]) valid = false;
        }
        if (valid) v = (float)pow((double)mp, (double)A.alpha);
    }
    if (!run) return tree_walk(A.tree, (int)(A.L + slot), v, j < cnt, A.levels);   // uniform for the workgroup
    if (j < cnt) val[j] = v;
    if (j < 128) sib[j] = sv;
    tree_repair_run(A.tree, first, cnt, A.levels, val, sib);
}

// Frame preprocessing (Sec.3: palette frame -> grey-scale -> linear interpolation to 84 x 84).
// One thread per output pixel, grid (ceil(7056/256), n).  grey = lut[byte] or the byte itself;
// centre-aligned source coordinate, clamped; bilinear blend; round to nearest even.
__global__ __launch_bounds__(256) void k_preprocess(const uint8_t *raw, int H, int W, const float *lut, uint8_t *out)
{
    const int o = blockIdx.x * 256 + threadIdx.x;
    if (o >= net::FRAME) return;
    const int i = o / 84, j = o % 84;
    const uint8_t *im = raw + (long)blockIdx.y * H * W;
    // the source coordinate (i + 1/2) H/84 - 1/2 = ((2i+1) H - 84) / 168 is kept as an exact
    // fraction, so only the blend itself is rounded
    const int ny = min(max((2 * i + 1) * H - 84, 0), 168 * (H - 1));
    const int nx = min(max((2 * j + 1) * W - 84, 0), 168 * (W - 1));
    const int y0 = ny / 168, x0 = nx / 168;
    const int y1 = min(y0 + 1, H - 1), x1 = min(x0 + 1, W - 1);
    const float fy = (float)(ny % 168) / 168.f, fx = (float)(nx % 168) / 168.f;
    auto grey = [&](int y, int x) {
        const uint8_t b = im[(long)y * W + x];
        return lut ? lut[b] : (float)b;
    };
    const float top = grey(y0, x0) * (1.f - fx) + grey(y0, x1) * fx;
    const float bot = grey(y1, x0) * (1.f - fx) + grey(y1, x1) * fx;
    const float v = top * (1.f - fy) + bot * fy;
    out[(long)blockIdx.y * net::FRAME + o] = (uint8_t)fminf(fmaxf(rintf(v), 0.f), 255.f);
}

// The same for frames of ordinary size (at most four source rows per output row): a workgroup owns `rows` output rows
// of one frame, copies the source rows under them into LDS with 16-byte loads and blends out of LDS, the grey table
// in LDS as well.  The one-thread-per-pixel kernel above is bound by its eight scattered one-byte and table
// fetches per pixel (77.5 us for 2048 frames of 210 x 160, 83 MB: 1.07 TB/s); here memory sees each byte once in
// wide loads and the fetches go to LDS.  252 threads: thread t keeps column t % 84 (its source columns and
// weight stay in registers) and walks down every third row; four neighbouring lanes put their bytes into one
// 4-byte store (84 is a multiple of 4, so such a quad lies in one row).  Same arithmetic, same bytes.
// Dynamic LDS: the staged rows.
template <bool LUT>
__global__ __launch_bounds__(256) void k_preprocess_staged(const uint8_t *raw, long total, int H, int W, const float *lut,
                                                           uint8_t *out, int rows)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t px_dyn[];
    __shared__ float grey_tab[256];
    __shared__ int row_at[84];
    __shared__ float row_f[84];
    const int tid = threadIdx.x, i0 = blockIdx.x * rows;
    auto source = [](int o, int N, int &at, float &f) {   // exact source coordinate of output line o, clamped
        const int q = min(max((2 * o + 1) * N - 84, 0), 168 * (N - 1));
        at = q / 168;
        f = (float)(q % 168) / 168.f;
    };
    int ya, yb;
    float f;
    source(i0, H, ya, f);
    source(i0 + rows - 1, H, yb, f);
    const int yend = min(yb + 1, H - 1);
    const long beg = ((long)blockIdx.y * H + ya) * W;        // bytes of `raw`
    const int len = (yend - ya + 1) * W;
    const int mis = (int)((uintptr_t)(raw + beg) & 15);
    const uint8_t *al = raw + beg - mis;                       // 16-byte aligned
    for (int g = tid; 16 * g < mis + len; g += 256) {
        const long first = beg - mis + 16L * g;
        if (first >= 0 && first + 16 <= total) {
            *reinterpret_cast<uint4 *>(px_dyn + 16 * g) = *reinterpret_cast<const uint4 *>(al + 16 * g);
        } else {   // the first and the last bytes of the whole array
            for (int b = 0; b < 16; ++b)
                if (first + b >= 0 && first + b < total) px_dyn[16 * g + b] = al[16 * g + b];
        }
    }
    if (LUT) grey_tab[tid] = lut[tid];
    if (tid < rows) {
        int at;
        source(i0 + tid, H, at, row_f[tid]);
        row_at[tid] = mis + (at - ya) * W;
    }
    __syncthreads();
    if (tid >= 252) return;
    const int j = tid % 84, rg = tid / 84;
    int x0;
    float fx;
    source(j, W, x0, fx);
    const int x1 = min(x0 + 1, W - 1);
    uint8_t *dst = out + (long)blockIdx.y * net::FRAME + (long)i0 * 84 + (j & ~3);
    for (int i = rg; i < rows; i += 3) {
        const int at = row_at[i];
        const float fy = row_f[i];
        const int below = at + W < mis + len ? at + W : at;   // the last source row has no row below it
        auto grey = [&](int q) {
            const uint8_t b = px_dyn[q];
            return LUT ? grey_tab[b] : (float)b;
        };
        const float top = grey(at + x0) * (1.f - fx) + grey(at + x1) * fx;
        const float bot = grey(below + x0) * (1.f - fx) + grey(below + x1) * fx;
        const float v = top * (1.f - fy) + bot * fy;
        uint32_t b = (uint32_t)(uint8_t)fminf(fmaxf(rintf(v), 0.f), 255.f) << (8 * (j & 3));
        b |= (uint32_t)lane_xor<1>((int)b);
        b |= (uint32_t)lane_xor<2>((int)b);
        if ((j & 3) == 0) *reinterpret_cast<uint32_t *>(dst + 84 * i) = b;
    }
}

// Stored layer outputs back in the canonical order: src [n][P][C] (channel-last, fp32 or bf16) ->
// dst fp32 [n][C][P].  One thread per element.
__global__ __launch_bounds__(256) void k_read_act(const void *src, int is_bf16, long n, int P, int Cn, float *dst)
{
    const long e = (long)blockIdx.x * 256 + threadIdx.x;   // canonical index
    if (e >= n * P * Cn) return;
    const long row = e / ((long)P * Cn);
    const int c = (int)((e / P) % Cn), pos = (int)(e % P);
    const long in = (row * P + pos) * Cn + c;
    dst[e] = is_bf16 ? __uint_as_float((uint32_t) static_cast<const uint16_t *>(src)[in] << 16)
                     : static_cast<const float *>(src)[in];
}

// Copies up to eleven short arrays of 4-byte words; grid (blocks, items).
struct CopyOutArgs {
    struct Item {
        uint32_t *dst;
        const uint32_t *src;
        int words;
    } item[11];
};
__global__ __launch_bounds__(256) void k_copy_out(CopyOutArgs A)
{
    const CopyOutArgs::Item it = A.item[blockIdx.y];
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t < it.words) it.dst[t] = it.src[t];
}

// --------------------------------------------------------------- replay
// Slot `off` frames away from slot i (off in [-3, 1]), wrapping inside the sub-ring that i lies in:
// the whole ring (sub == cap: one stream), or one environment stream's share of it.
__device__ __forceinline__ long ring_slot(long i, long off, long cap, long sub)
{
    const long base = sub == cap ? 0 : (i / sub) * sub;
    long l = (i - base + off) % sub;
    if (l < 0) l += sub;
    return base + l;
}

struct GatherArgs {
    const uint8_t *frames;  // ring [cap][7056]
    const int32_t *meta_a;
    const float *meta_r;
    const uint8_t *meta_done;
    long cap;
    const int32_t *idx;  // [n]
    uint8_t *stack5;     // [n][5][7056] or nullptr
    uint8_t *s, *s_next; // [n][4][7056] or nullptr
    int32_t *a;
    float *r;
    uint8_t *done;
    long sub;            // length of the sub-ring a window wraps in (the capacity for one stream)
};

// Frame-stack gather: transition i reads ring slots i-3 .. i+1 (mod cap);
// grid (n, 5), 16 bytes per thread per trip.
__global__ __launch_bounds__(256) void k_gather(GatherArgs A)
{
    const int j = blockIdx.x, k = blockIdx.y;
    long i = A.idx[j];
    i = i < 0 ? 0 : (i >= A.cap ? A.cap - 1 : i);  // keeps every access inside the ring
    const long slot = ring_slot(i, k - 3, A.cap, A.sub);
    const uint4 *src = reinterpret_cast<const uint4 *>(A.frames + slot * net::FRAME);
    uint4 *d0 = A.stack5 ? reinterpret_cast<uint4 *>(A.stack5 + ((long)j * 5 + k) * net::FRAME) : nullptr;
    uint4 *d1 = (A.s && k < 4) ? reinterpret_cast<uint4 *>(A.s + ((long)j * 4 + k) * net::FRAME) : nullptr;
    uint4 *d2 = (A.s_next && k > 0) ? reinterpret_cast<uint4 *>(A.s_next + ((long)j * 4 + k - 1) * net::FRAME) : nullptr;
    for (int t = threadIdx.x; t < net::FRAME / 16; t += 256) {
        uint4 v = src[t];
        if (d0) d0[t] = v;
        if (d1) d1[t] = v;
        if (d2) d2[t] = v;
    }
    if (k == 0 && threadIdx.x == 0) {
        if (A.a) A.a[j] = A.meta_a[i];
        if (A.r) A.r[j] = A.meta_r[i];
        if (A.done) A.done[j] = A.meta_done[i];
    }
}

// Sampling and the frame-stack gather in one launch (grid (B, 5), 256 threads): the first wave of
// every workgroup repeats the draw of its transition (five workgroups per transition do the same
// descent; it costs less than a launch), workgroup (j, 0) also emits the draw's outputs, then all
// threads copy frame k of the stack.
__global__ __launch_bounds__(256) void k_sample_gather(SampleArgs S, GatherArgs A)
{
    __shared__ long slot_sh;
    const int j = blockIdx.x, k = blockIdx.y;
    if (threadIdx.x < 64) {
        const int jj[1] = {j};
        long slot[1];
        float leaf[1];
        const float total = per_sample_walk<1>(S, jj, threadIdx.x, slot, leaf);
        if (threadIdx.x == 0) {
            slot_sh = slot[0];
            if (k == 0) per_sample_emit(S, j, slot[0], total, leaf[0]);
        }
    }
    __syncthreads();
    const long i = slot_sh;
    const long slot = ring_slot(i, k - 3, A.cap, A.sub);
    const uint4 *src = reinterpret_cast<const uint4 *>(A.frames + slot * net::FRAME);
    uint4 *d0 = reinterpret_cast<uint4 *>(A.stack5 + ((long)j * 5 + k) * net::FRAME);
    for (int t = threadIdx.x; t < net::FRAME / 16; t += 256) d0[t] = src[t];
}

// Ring store: n frames into slots slot0.. (mod cap); grid (n).
__global__ __launch_bounds__(256) void k_replay_write(uint8_t *frames, int32_t *meta_a, float *meta_r,
                                                      uint8_t *meta_done, long cap, long slot0,
                                                      const uint8_t *src, const int32_t *a,
                                                      const float *r, const uint8_t *done)
{
    const long j = blockIdx.x;
    const long slot = (slot0 + j) % cap;
    const uint4 *s = reinterpret_cast<const uint4 *>(src + j * net::FRAME);
    uint4 *d = reinterpret_cast<uint4 *>(frames + slot * net::FRAME);
    for (int t = threadIdx.x; t < net::FRAME / 16; t += 256) d[t] = s[t];
    if (threadIdx.x == 0) {
        if (a) meta_a[slot] = a[j];
        if (r) meta_r[slot] = r[j];
        if (done) meta_done[slot] = done[j];
    }
}

}  // namespace misc

// Learned cost model: a 32 -> 256 -> 256 -> 2 ReLU network predicting the
// natural log of a task's duration on each worker kind, trained with MSE and
// Adam.  The paper drives inspiring efficiency with per-kind execution-time
// estimates gathered by a cost model (Sections 4.3 and 5); this model replaces
// the per-type average table when task features are available.
//
// Precision: weights, activations and activation gradients are stored as
// bfloat16 (round to nearest even); products accumulate in fp32 on the MFMA
// units (v_mfma_f32_16x16x32_bf16); biases, outputs, weight gradients, Adam
// moments and master weights are fp32.
//
// Packed parameter order: W1 [32,256], b1 [256], W2 [256,256], b2 [256],
// W3 [256,2], b3 [2].
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "common.hpp"
#include "internal.hpp"

namespace insp {

constexpr int kIn = 32, kHid = 256, kOut = 2;
constexpr int64_t kMaxTrainSteps = 1 << 28;  // steps of one insp_mlp_train call
constexpr int32_t kTrainChunk = 32;          // steps per captured graph
constexpr int64_t kOffW1 = 0, kOffB1 = kOffW1 + kIn * kHid, kOffW2 = kOffB1 + kHid, kOffB2 = kOffW2 + kHid * kHid,
                  kOffW3 = kOffB2 + kHid, kOffB3 = kOffW3 + kHid * kOut, kParams = kOffB3 + kOut;
static_assert(kParams == 74754, "parameter count");

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));

// fp32 -> bf16, round to nearest even (v_cvt_pk_bf16_f32 on gfx950); f2bf2
// converts two values with one instruction, a in the low half
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ __forceinline__ uint32_t f2bf2(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{a, b}, bf16x2_t));
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// Weights and activations that a product reads as MFMA operands are kept in
// fragment order: element k of operand row n (a 16 x 32 fragment holds rows
// n / 16 and elements k / 32) at frag(n, k, K), so that a wave's fragment load
// is 1 KB of consecutive bytes, eight whole cache lines, where row-major
// order would touch half of sixteen.
__device__ __forceinline__ int64_t frag(int n, int64_t k, int64_t K) {
    return (((int64_t)(n >> 4) * (K >> 5) + (k >> 5)) * 64 + (n & 15) + ((k & 31) >> 3) * 16) * 8 + (k & 7);
}

// ------------------------------------------------------------- training
// One step is two kernels: k_rows_step, the forward and backward passes of
// 32 rows per work-group, and k_params_step, the weight gradients with the
// sums over the batch and (training) Adam.  Every sum is taken in a fixed
// order that does not depend on the launch, so training is bit-reproducible.
//
// What bounds a step: not the matrix cores (0.46 GFLOP at batch 1024 is 0.2 us
// of them) but the launches (about 3.4 us each, however little they do) and
// the chain of dependent loads, LDS trips and barriers inside.  A training step
// of batch 1024 takes 17.0 us (10.7 + 6.4), against 58.7 as eleven kernels, one
// per product, reduction and update; a gradients call among others 15.2 to 16.8
// (11.0 + 5.0 in the kernels), against 61.7.
//
// Between the two kernels the activations travel by unit, along the batch: a
// lane's MFMA accumulator holds four consecutive rows of one unit (one 8-byte
// store), and the weight-gradient products then read both operands as 16-byte
// fragments with no LDS staging.  All but H2, which no product reads that way,
// are in fragment order (frag).
constexpr int kRows = 32;               // rows per work-group of k_rows_step
constexpr int kRowWaves = 8;            // its waves; wave w owns hidden units [32 w, 32 w + 32)
constexpr int kRowLds = kHid + 8;       // LDS row of activations (16-byte aligned, rows 4 banks apart)
constexpr int kPart = kHid + 3;         // partial sums per 4 rows: db2, db3, loss
constexpr int kChunks = 16;             // batch chunks whose partial products meet in LDS at once

struct StepArgs {
    const float *x, *t;                 // features and targets (minibatch 0 when tab is set)
    int64_t rows;
    const int32_t *tab;                 // graph-captured training: see k_params_step
    int32_t steps;                      // ... minibatches per epoch
    const float *p;                     // fp32 parameters (biases)
    const uint16_t *w1t, *w2, *w2t, *w3;  // bf16 weights: W1^T, W2 and W2^T in fragment order, W3 [256][2]
    uint16_t *xt, *h1t, *h2t, *d2t, *d1t; // bf16 by unit: features, hidden layers, their gradients (fragment order; h2t [unit][rows])
    float *y;                           // [rows][2]
    float *part;                        // [rows / 4][kPart] column sums of dH2, dY and the loss per 4 rows
    float *colpart;                     // [rows / 32][256] column sums of dH1 per 32 rows
    int32_t *cur;                       // tab[1]: the step index, for k_params_step
};

// The sum of x over the wave, by halves (lane l holds the sum over l ^ off at
// each step): 32 and 16 by lane swaps, then rotations within 16-lane rows
// (after the step of 8 a rotation by 4 reaches l ^ 4 or its equal l ^ 12).
__device__ __forceinline__ float wave_sum_halving(float x) {
    x += __shfl_xor(x, 32, 64);
    x += __shfl_xor(x, 16, 64);
    x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x128, 0xF, 0xF, false));
    x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x124, 0xF, 0xF, false));
    x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x4E, 0xF, 0xF, false));
    x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0xB1, 0xF, 0xF, false));
    return x;
}

// A work-group barrier that orders LDS accesses only: global stores in flight
// (activations that only the next kernel reads) and prefetched loads are not
// waited for, as __syncthreads would.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Forward and backward of 32 rows.  Each wave keeps the fragments of its 32
// columns of W1, W2 and W2^T in registers; accumulator value i of a lane is
// row 4 (lane / 16) + i, unit lane % 16, in all three products, so masks and
// hidden values stay in the lane that made them.  A work-group is bound by
// its 272 KB of weights, read cold (1.8 us at the L1's 64 bytes a clock), and
// by its five short phases (0.7 to 1 us each) between barriers; with the launch
// 10.7 us at batch 1024.  Weights in row-major order (half-used cache lines)
// made that 15.8, barriers that also wait for the global stores cost 1 us
// each, and 16 waves of 16 columns took 13.7.  32 rows per work-group because
// the reduction order of db1 is by 32 rows.
// X16: x is 16-byte aligned (rows are then read as float4).
template <bool X16>
__global__ __launch_bounds__(64 * kRowWaves) void k_rows_step(StepArgs A) {
    __shared__ __attribute__((aligned(16))) uint16_t H1s[kRows * kRowLds];  // H1, later dH2
    __shared__ __attribute__((aligned(16))) uint16_t H2s[kRows * kRowLds];
    __shared__ float ds[kRows][2];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int wn = wv * 32, lc = lane & 15, lg = lane >> 4, lk = lg * 8;
    const int64_t r0 = (int64_t)blockIdx.x * kRows, B = A.rows;
    int64_t o = 0;
    if (A.tab) {
        const int32_t s = A.tab[0];
        o = B * (int64_t)((uint32_t)s % (uint32_t)A.steps);
        if (blockIdx.x == 0 && tid == 0) A.cur[0] = s;
    }
    const float *x = A.x + (o + r0) * kIn, *t = A.t + (o + r0) * kOut;
    bf16x8 w1f[2], w2f[2][8], w2b[2][8], xf[2];
    float bias1[2], bias2[2];
    float v[2][8];
#pragma unroll
    for (int rt = 0; rt < 2; rt++) {
        const float *q = x + (rt * 16 + lc) * kIn + lk;
        if (X16) {
            const float4 a = *reinterpret_cast<const float4 *>(q), b = *reinterpret_cast<const float4 *>(q + 4);
            v[rt][0] = a.x; v[rt][1] = a.y; v[rt][2] = a.z; v[rt][3] = a.w;
            v[rt][4] = b.x; v[rt][5] = b.y; v[rt][6] = b.z; v[rt][7] = b.w;
        } else {
#pragma unroll
            for (int i = 0; i < 8; i++) v[rt][i] = q[i];
        }
    }
#pragma unroll
    for (int ct = 0; ct < 2; ct++) {
        const int n = wn + ct * 16 + lc;
        w1f[ct] = *reinterpret_cast<const bf16x8 *>(A.w1t + ((wv * 2 + ct) * 64 + lane) * 8);
        bias1[ct] = A.p[kOffB1 + n];
        bias2[ct] = A.p[kOffB2 + n];
#pragma unroll
        for (int ks = 0; ks < 8; ks++)
            w2f[ct][ks] = *reinterpret_cast<const bf16x8 *>(A.w2t + (((wv * 2 + ct) * 8 + ks) * 64 + lane) * 8);
    }
    // output weights: of this lane's four units in the output dot products,
    // and of its two columns in dH2
    const uint4 w3d = *reinterpret_cast<const uint4 *>(A.w3 + lane * 8);
    uint32_t w3c[2];
#pragma unroll
    for (int ct = 0; ct < 2; ct++) w3c[ct] = *reinterpret_cast<const uint32_t *>(A.w3 + (wn + ct * 16 + lc) * 2);
    const float b30 = A.p[kOffB3], b31 = A.p[kOffB3 + 1];
    float tt[4][2];
#pragma unroll
    for (int k = 0; k < 4; k++) {
        tt[k][0] = t[(wv * 4 + k) * 2];
        tt[k][1] = t[(wv * 4 + k) * 2 + 1];
    }
    __builtin_amdgcn_sched_barrier(0);  // every load above is issued before any of them is waited for
#pragma unroll
    for (int rt = 0; rt < 2; rt++) {
        const uint4 h = {f2bf2(v[rt][0], v[rt][1]), f2bf2(v[rt][2], v[rt][3]), f2bf2(v[rt][4], v[rt][5]),
                         f2bf2(v[rt][6], v[rt][7])};
        xf[rt] = __builtin_bit_cast(bf16x8, h);
    }
    // the features transposed, for dW1: wave w stores k = w, w + 8, w + 16, w + 24 of either 16-row half
#pragma unroll
    for (int rt = 0; rt < 2; rt++) {
        const u16x8 h = __builtin_bit_cast(u16x8, xf[rt]);
        uint16_t e = 0;
#pragma unroll
        for (int i = 0; i < 8; i++) e = i == wv ? h[i] : e;
        A.xt[frag(lk + wv, r0 + rt * 16 + lc, B)] = e;
    }
    // layer 1
    bool on1[2][2][4];
#pragma unroll
    for (int rt = 0; rt < 2; rt++)
#pragma unroll
        for (int ct = 0; ct < 2; ct++) {
            const f32x4 acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf[rt], w1f[ct], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            const int n = wn + ct * 16 + lc;
            uint16_t h[4];
#pragma unroll
            for (int i = 0; i < 4; i++) {
                h[i] = f2bf(fmaxf(acc[i] + bias1[ct], 0.f));
                on1[rt][ct][i] = bf2f(h[i]) > 0.f;
                H1s[(rt * 16 + lg * 4 + i) * kRowLds + n] = h[i];
            }
            const uint2 q = {(uint32_t)h[0] | (uint32_t)h[1] << 16, (uint32_t)h[2] | (uint32_t)h[3] << 16};
            *reinterpret_cast<uint2 *>(A.h1t + frag(n, r0 + rt * 16 + lg * 4, B)) = q;
        }
    lds_barrier();
    // layer 2
    float h2[2][2][4];
#pragma unroll
    for (int rt = 0; rt < 2; rt++) {
        f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int ks = 0; ks < 8; ks++) {
            const bf16x8 hf = *reinterpret_cast<const bf16x8 *>(&H1s[(rt * 16 + lc) * kRowLds + ks * 32 + lk]);
#pragma unroll
            for (int ct = 0; ct < 2; ct++)
                acc[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hf, w2f[ct][ks], acc[ct], 0, 0, 0);
        }
#pragma unroll
        for (int ct = 0; ct < 2; ct++) {
            const int n = wn + ct * 16 + lc;
            uint16_t h[4];
#pragma unroll
            for (int i = 0; i < 4; i++) {
                h[i] = f2bf(fmaxf(acc[ct][i] + bias2[ct], 0.f));
                h2[rt][ct][i] = bf2f(h[i]);
                H2s[(rt * 16 + lg * 4 + i) * kRowLds + n] = h[i];
            }
            const uint2 q = {(uint32_t)h[0] | (uint32_t)h[1] << 16, (uint32_t)h[2] | (uint32_t)h[3] << 16};
            *reinterpret_cast<uint2 *>(A.h2t + (int64_t)n * B + r0 + rt * 16 + lg * 4) = q;
        }
    }
    lds_barrier();
    // W2^T's fragments, for dH1: issued only here so that the first two layers
    // do not queue behind them (the 272 KB of weights take the L1 1.8 us at 64
    // bytes a clock) and the output layer covers them
#pragma unroll
    for (int ct = 0; ct < 2; ct++)
#pragma unroll
        for (int ks = 0; ks < 8; ks++)
            w2b[ct][ks] = *reinterpret_cast<const bf16x8 *>(A.w2 + (((wv * 2 + ct) * 8 + ks) * 64 + lane) * 8);
    __builtin_amdgcn_sched_barrier(0);
    // outputs, their gradient and the loss: wave w has rows 4 w .. 4 w + 3
    const float scale = 1.0f / (float)B;  // 2 / (2 rows)
    {
        float w30[4], w31[4], s0[4], s1[4];
        const uint32_t wq[4] = {w3d.x, w3d.y, w3d.z, w3d.w};
#pragma unroll
        for (int j = 0; j < 4; j++) {
            w30[j] = bf2f((uint16_t)(wq[j] & 0xFFFFu));
            w31[j] = bf2f((uint16_t)(wq[j] >> 16));
        }
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const uint2 q = *reinterpret_cast<const uint2 *>(&H2s[(wv * 4 + k) * kRowLds + lane * 4]);
            const float h[4] = {bf2f((uint16_t)(q.x & 0xFFFFu)), bf2f((uint16_t)(q.x >> 16)),
                                bf2f((uint16_t)(q.y & 0xFFFFu)), bf2f((uint16_t)(q.y >> 16))};
            float a0 = 0.f, a1 = 0.f;
#pragma unroll
            for (int j = 0; j < 4; j++) {
                a0 += h[j] * w30[j];
                a1 += h[j] * w31[j];
            }
            s0[k] = a0;
            s1[k] = a1;
        }
        float d0[4], d1[4], l2[4];
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const float y0 = wave_sum_halving(s0[k]) + b30, y1 = wave_sum_halving(s1[k]) + b31;
            const float e0 = y0 - tt[k][0], e1 = y1 - tt[k][1];
            d0[k] = e0 * scale;
            d1[k] = e1 * scale;
            l2[k] = (e0 * e0 + e1 * e1) * 0.5f * scale;
            if (lane == 0) {
                const int row = wv * 4 + k;
                A.y[(r0 + row) * 2] = y0;
                A.y[(r0 + row) * 2 + 1] = y1;
                ds[row][0] = d0[k];
                ds[row][1] = d1[k];
            }
        }
        if (lane == 0) {
            // (sums of rounded values: not fused with the products they add up)
#pragma clang fp contract(off)
            float *pp = A.part + (r0 / 4 + wv) * kPart + kHid;
            pp[0] = ((d0[0] + d0[1]) + d0[2]) + d0[3];
            pp[1] = ((d1[0] + d1[1]) + d1[2]) + d1[3];
            pp[2] = ((l2[0] + l2[1]) + l2[2]) + l2[3];
        }
    }
    lds_barrier();
    // dH2 = (dY W3^T) * (H2 > 0), its column sums per 4 rows
#pragma unroll
    for (int rt = 0; rt < 2; rt++)
#pragma unroll
        for (int ct = 0; ct < 2; ct++) {
            const int n = wn + ct * 16 + lc;
            const float w30 = bf2f((uint16_t)(w3c[ct] & 0xFFFFu)), w31 = bf2f((uint16_t)(w3c[ct] >> 16));
            float gv[4];
            uint16_t h[4];
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const int row = rt * 16 + lg * 4 + i;
                gv[i] = ds[row][0] * w30 + ds[row][1] * w31;
                if (!(h2[rt][ct][i] > 0.f)) gv[i] = 0.f;
                h[i] = f2bf(gv[i]);
                H1s[row * kRowLds + n] = h[i];
            }
            const uint2 q = {(uint32_t)h[0] | (uint32_t)h[1] << 16, (uint32_t)h[2] | (uint32_t)h[3] << 16};
            *reinterpret_cast<uint2 *>(A.d2t + frag(n, r0 + rt * 16 + lg * 4, B)) = q;
            A.part[(r0 / 4 + rt * 4 + lg) * kPart + n] = ((gv[0] + gv[1]) + gv[2]) + gv[3];
        }
    lds_barrier();
    // dH1 = (dH2 W2^T) * (H1 > 0), its column sums: per lane its rows in
    // order, then the four lane groups
    float cs[2] = {0.f, 0.f};
#pragma unroll
    for (int rt = 0; rt < 2; rt++) {
        f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int ks = 0; ks < 8; ks++) {
            const bf16x8 df = *reinterpret_cast<const bf16x8 *>(&H1s[(rt * 16 + lc) * kRowLds + ks * 32 + lk]);
#pragma unroll
            for (int ct = 0; ct < 2; ct++)
                acc[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(df, w2b[ct][ks], acc[ct], 0, 0, 0);
        }
#pragma unroll
        for (int ct = 0; ct < 2; ct++) {
            const int n = wn + ct * 16 + lc;
            uint16_t h[4];
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const float v = on1[rt][ct][i] ? acc[ct][i] : 0.f;
                h[i] = f2bf(v);
                cs[ct] += v;
            }
            const uint2 q = {(uint32_t)h[0] | (uint32_t)h[1] << 16, (uint32_t)h[2] | (uint32_t)h[3] << 16};
            *reinterpret_cast<uint2 *>(A.d1t + frag(n, r0 + rt * 16 + lg * 4, B)) = q;
        }
    }
#pragma unroll
    for (int ct = 0; ct < 2; ct++) {
        const float c0 = __shfl(cs[ct], lc, 64), c1 = __shfl(cs[ct], lc + 16, 64);
        const float c2 = __shfl(cs[ct], lc + 32, 64), c3 = __shfl(cs[ct], lc + 48, 64);
        if (lane < 16) A.colpart[(int64_t)blockIdx.x * kHid + wn + ct * 16 + lane] = ((c0 + c1) + c2) + c3;
    }
}

struct ParamArgs {
    const float *t;                     // targets (minibatch 0 when tab is set)
    int64_t rows;
    int32_t *tab;                       // graph-captured training: step index, index of the step in hand, corrections
    int32_t steps, tabn;
    const uint16_t *xt, *h1t, *h2t, *d2t, *d1t;
    const float *y, *part, *colpart;
    int32_t chunk1, n1, chunk2, n2;     // batch rows per partial product and their number: dW1, dW2
    float *grads, *loss;                // gradients out (nullptr: Adam)
    float *p, *m, *v;                   // Adam
    float lr, bc1, bc2;
    uint16_t *w1t, *w2, *w2t, *w3;
};

// Adam (Kingma and Ba) with bias correction, then the bf16 weight shadows.
__device__ __forceinline__ void put_param(const ParamArgs &A, int64_t i, float gi, float bc1, float bc2) {
    if (A.grads) {
        A.grads[i] = gi;
        return;
    }
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float mi = b1 * A.m[i] + (1.f - b1) * gi;
    const float vi = b2 * A.v[i] + (1.f - b2) * gi * gi;
    A.m[i] = mi;
    A.v[i] = vi;
    const float pi = A.p[i] - A.lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
    A.p[i] = pi;
    const uint16_t h = f2bf(pi);
    if (i < kOffB1) {
        const int k = (int)(i - kOffW1);
        A.w1t[frag(k % kHid, k / kHid, kIn)] = h;
    } else if (i >= kOffW2 && i < kOffB2) {
        const int k = (int)(i - kOffW2);
        A.w2[frag(k / kHid, k % kHid, kHid)] = h;
        A.w2t[frag(k % kHid, k / kHid, kHid)] = h;
    } else if (i >= kOffW3 && i < kOffB3) {
        A.w3[i - kOffW3] = h;
    }
}

// A 16 x 16 tile of a weight gradient, sum over the batch of P[m0 + r][k]
// Q[n0 + c][k] (operands in fragment order along the batch): the batch in `nch` chunks, each
// chunk's product accumulated on the matrix cores, the chunks summed in
// order.  A wave takes four chunks of every kChunks; returns element
// (tid / 16, tid % 16).
__device__ __forceinline__ float grad_tile(const uint16_t *P, const uint16_t *Q, int64_t rows, int32_t chunk,
                                           int32_t nch, float *sum_lds) {
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, lc = lane & 15;
    const uint16_t *p = P + lane * 8, *q = Q + lane * 8;
    float s = 0.f;
    for (int32_t c0 = 0; c0 < nch; c0 += kChunks) {
        f32x4 acc[4];
#pragma unroll
        for (int j = 0; j < 4; j++) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        // the wave's four chunks side by side, so that their loads overlap;
        // reads past a chunk's end are replaced by zeros, which add nothing
        const int64_t k0 = (int64_t)(c0 + wv * 4) * chunk;
        for (int32_t k = 0; k < chunk; k += 64) {
            bf16x8 a[4][2], b[4][2];
#pragma unroll
            for (int j = 0; j < 4; j++)
#pragma unroll
                for (int u = 0; u < 2; u++) {
                    const int64_t kk = k0 + (int64_t)j * chunk + k + u * 32;
                    const bool ok = k + u * 32 < chunk && kk < rows;
                    a[j][u] = ok ? *reinterpret_cast<const bf16x8 *>(p + kk * 16) : bf16x8{};
                    b[j][u] = ok ? *reinterpret_cast<const bf16x8 *>(q + kk * 16) : bf16x8{};
                }
#pragma unroll
            for (int j = 0; j < 4; j++)
#pragma unroll
                for (int u = 0; u < 2; u++)
                    acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[j][u], b[j][u], acc[j], 0, 0, 0);
        }
        if (c0) __syncthreads();
#pragma unroll
        for (int j = 0; j < 4; j++)
#pragma unroll
            for (int i = 0; i < 4; i++)
                sum_lds[(wv * 4 + j) * 256 + ((lane >> 4) * 4 + i) * 16 + lc] = acc[j][i];
        __syncthreads();
        const int32_t m = min(kChunks, nch - c0);
        for (int32_t z = 0; z < m; z++) s = c0 + z == 0 ? sum_lds[tid] : s + sum_lds[z * 256 + tid];
    }
    return s;
}

// Columns [c0, c0 + 16) of partial sums: share w of 16 adds its contiguous
// part of the rows in order, then the 16 shares are added in order; the
// result is in threads 0..15.  `get` reads row r, column c.
template <typename F>
__device__ __forceinline__ float col_sum16(int rows, bool ok, float *red, F get) {
    const int tid = threadIdx.x, w = tid >> 4, c = tid & 15;
    const int per = (rows + 15) / 16, a = min(rows, w * per), z = min(rows, a + per);
    float s = 0.f;
    if (ok) {
#pragma unroll 16
        for (int r = a; r < z; r++) s += get(r);
    }
    red[w * 16 + c] = s;
    __syncthreads();
    float u = red[c];
#pragma unroll
    for (int i = 1; i < 16; i++) u += red[i * 16 + c];
    return u;
}

// Work-groups of k_params_step, the longest first: dW2's 16 x 16 tiles, dW1's,
// dW3 (a wave per hidden unit), db1, and db2 with db3 and the loss.
constexpr int kGW2 = (kHid / 16) * (kHid / 16), kGW1 = (kIn / 16) * (kHid / 16), kGW3 = kHid / 4, kGB1 = kHid / 16,
              kGB2 = (kPart + 15) / 16, kGrid2 = kGW2 + kGW1 + kGW3 + kGB1 + kGB2;

// Weight gradients and (without `grads`) Adam.  One 16 x 16 tile per
// work-group gives dW2 all 256 CUs at any batch; each work-group reads 16
// rows of either operand along the whole batch (64 KB at batch 1024, from
// the L2).  With a table (graph-captured training) tab[1] is the step in
// hand, left by k_rows_step, whose bias corrections 1 - 0.9^step and
// 1 - 0.999^step, computed by the host, are at tab[2 + 2 i] and tab[3 + 2 i];
// tab[0] becomes the next step's index.  (No work-group of either kernel reads
// the word that the same kernel writes.)
__global__ __launch_bounds__(256) void k_params_step(ParamArgs A) {
    __shared__ float lds[kChunks * 256];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    float bc1 = A.bc1, bc2 = A.bc2;
    int64_t o = 0;
    if (A.tab) {
        const int32_t s = A.tab[1], i = min(max(s, 0), A.tabn - 1);
        bc1 = __int_as_float(A.tab[2 + 2 * i]);
        bc2 = __int_as_float(A.tab[3 + 2 * i]);
        o = A.rows * (int64_t)((uint32_t)s % (uint32_t)A.steps);
        if (blockIdx.x == gridDim.x - 1 && tid == 0) A.tab[0] = s + 1;
    }
    const int64_t B = A.rows;
    int b = blockIdx.x;
    if (b < kGW2) {
        const int m0 = b / 16 * 16, n0 = b % 16 * 16;
        const float g = grad_tile(A.h1t + (int64_t)m0 * B, A.d2t + (int64_t)n0 * B, B, A.chunk2, A.n2, lds);
        put_param(A, kOffW2 + (m0 + (tid >> 4)) * kHid + n0 + (tid & 15), g, bc1, bc2);
        return;
    }
    b -= kGW2;
    if (b < kGW1) {
        const int m0 = b / 16 * 16, n0 = b % 16 * 16;
        const float g = grad_tile(A.xt + (int64_t)m0 * B, A.d1t + (int64_t)n0 * B, B, A.chunk1, A.n1, lds);
        put_param(A, kOffW1 + (m0 + (tid >> 4)) * kHid + n0 + (tid & 15), g, bc1, bc2);
        return;
    }
    b -= kGW1;
    if (b < kGW3) {
        // dW3[i][c] = sum over rows of H2[r][i] dY[r][c]: 256 running sums,
        // row r into sum r % 256 (lane l has sums l, l + 64, l + 128 and
        // l + 192), then halved down to one
        const int i = b * 4 + wv;
        const float *t = A.t + o * kOut;
        const uint16_t *h2 = A.h2t + (int64_t)i * B;
        const float scale = 1.0f / (float)B;
        float a0[4] = {0.f, 0.f, 0.f, 0.f}, a1[4] = {0.f, 0.f, 0.f, 0.f};
        // four rounds of 256 rows are read together
        for (int64_t r1 = 0; r1 < B; r1 += 1024) {
            uint16_t hh[4][4];
            float yy[4][4][2], ty[4][4][2];
#pragma unroll
            for (int u = 0; u < 4; u++)
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    const int64_t r = r1 + u * 256 + j * 64 + lane, q = min(r, B - 1);
                    hh[u][j] = h2[q];
                    yy[u][j][0] = A.y[2 * q];
                    yy[u][j][1] = A.y[2 * q + 1];
                    ty[u][j][0] = t[2 * q];
                    ty[u][j][1] = t[2 * q + 1];
                }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < 4; u++)
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    if (r1 + u * 256 + j * 64 + lane < B) {
                        const float h = bf2f(hh[u][j]);
                        a0[j] += h * (yy[u][j][0] - ty[u][j][0]) * scale;
                        a1[j] += h * (yy[u][j][1] - ty[u][j][1]) * scale;
                    }
                }
        }
        const float g0 = wave_sum_halving((a0[0] + a0[2]) + (a0[1] + a0[3]));
        const float g1 = wave_sum_halving((a1[0] + a1[2]) + (a1[1] + a1[3]));
        if (lane < 2) put_param(A, kOffW3 + 2 * i + lane, lane ? g1 : g0, bc1, bc2);
        return;
    }
    b -= kGW3;
    const int c = tid & 15;
    if (b < kGB1) {
        // tiles of 64 rows, each the sum of its two halves
        const int n = b * 16 + c, halves = (int)(B / kRows);
        const float g = col_sum16((halves + 1) / 2, true, lds, [&](int r) {
            const float *q = A.colpart + (int64_t)(2 * r) * kHid + n;
            return q[0] + (2 * r + 1 < halves ? q[kHid] : 0.f);
        });
        if (tid < 16) put_param(A, kOffB1 + n, g, bc1, bc2);
        return;
    }
    b -= kGB1;
    const int n = b * 16 + c;
    const float g = col_sum16((int)(B / 4), n < kPart, lds, [&](int r) { return A.part[(int64_t)r * kPart + n]; });
    if (tid < 16) {
        if (n < kHid) put_param(A, kOffB2 + n, g, bc1, bc2);
        else if (n < kHid + 2) put_param(A, kOffB3 + (n - kHid), g, bc1, bc2);
        else if (n == kHid + 2) A.loss[0] = g;
    }
}

// The bf16 weight shadows of the fp32 parameters.
__global__ void k_shadow(const float *p, uint16_t *w1t, uint16_t *w2, uint16_t *w2t, uint16_t *w3) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < kOffB1) {
        const int k = (int)(i - kOffW1);
        w1t[frag(k % kHid, k / kHid, kIn)] = f2bf(p[i]);
    } else if (i >= kOffW2 && i < kOffB2) {
        const int k = (int)(i - kOffW2);
        w2[frag(k / kHid, k % kHid, kHid)] = f2bf(p[i]);
        w2t[frag(k % kHid, k / kHid, kHid)] = f2bf(p[i]);
    } else if (i >= kOffW3 && i < kOffB3) {
        w3[i - kOffW3] = f2bf(p[i]);
    }
}

// Fused inference: y = W3^T relu(W2^T relu(W1^T x + b1) + b2) + b3 and the
// integer estimates, for many rows.  A block of NW waves is persistent over
// 64-row tiles; wave w owns hidden columns [w C, w C + C), C = 256 / NW, of
// both layers and keeps their W1 and W2 MFMA B-fragments in registers for the
// whole run.  Per tile: layer 1 (K = 32) from the features' bf16 fragments in
// LDS, bf16 hidden activations through LDS, layer 2 (K = 256) from LDS
// fragments, then the two outputs as per-wave partial dot products summed in
// a fixed order.  Both layers are computed transposed (weights as the A
// operand), so that a lane's accumulator holds consecutive hidden units of
// one row.
//
// What bounds it is how well the three busy units overlap (per tile and CU:
// MFMA 2,300 clocks on each SIMD, the VALU's conversions about as many, LDS
// 3,200), which takes two work-groups out of step on a CU, so the kernel stays
// within 128 registers: a thread reads and converts four features of a tile,
// once, two tiles ahead (all waves reading all features took 32 registers and
// eight times the loads), and biases and output weights wait in LDS.  On 2 M
// rows: 280 us a call, and 373 with one work-group a CU (190 registers).
typedef short s16x2 __attribute__((ext_vector_type(2)));

// ReLU of two packed bf16 values at once: a bf16 is negative exactly when its
// bit pattern is as a 16-bit integer, and rounding keeps the sign, so this is
// the rounding of max(x, 0) (with -0 turned into +0).
__device__ __forceinline__ uint32_t relu_bf2(uint32_t q) {
    const s16x2 z = {0, 0};
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s16x2, q), z));
}
constexpr int kRT = 64, kH1Row = kHid + 8, kXRow = kIn + 8;

constexpr int kInferWaves = 8;

template <int NW>
__global__ __launch_bounds__(64 * NW, 4) void k_infer(const float *x, int64_t rows, const uint16_t *W1t, const float *b1,
                                                       const uint16_t *W2t, const float *b2, const uint16_t *W3,
                                                       const float *b3, float *Y, int32_t *est) {
    constexpr int CT = kHid / NW / 16;  // 16-column MFMA tiles per wave
    __shared__ __attribute__((aligned(16))) uint16_t H1s[kRT * kH1Row];
    __shared__ __attribute__((aligned(16))) uint16_t Xs[2][kRT * kXRow];
    __shared__ float yp[NW][kRT][2];
    __shared__ __attribute__((aligned(16))) float sb1[kHid], sb2[kHid];
    __shared__ uint32_t sw[2][kHid / 2];  // output weights of hidden units (i, i + 1), as packed bf16 pairs
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int wn = wv * (kHid / NW), lc = lane & 15, lk = (lane >> 4) * 8;
    bf16x8 w1f[CT], w2f[8][CT];
#pragma unroll
    for (int ct = 0; ct < CT; ct++) {
        const int nt = wv * CT + ct;  // the tile's place among the fragments
        w1f[ct] = *reinterpret_cast<const bf16x8 *>(W1t + (nt * 64 + lane) * 8);
#pragma unroll
        for (int ks = 0; ks < 8; ks++)
            w2f[ks][ct] = *reinterpret_cast<const bf16x8 *>(W2t + ((nt * 8 + ks) * 64 + lane) * 8);
    }
    for (int h = tid; h < kHid; h += 64 * NW) {
        sb1[h] = b1[h];
        sb2[h] = b2[h];
        sw[h & 1][h >> 1] = (uint32_t)W3[(h & ~1) * 2 + (h & 1)] | (uint32_t)W3[(h & ~1) * 2 + 2 + (h & 1)] << 16;
    }
    const float b30 = b3[0], b31 = b3[1];
    const int64_t tiles = (rows + kRT - 1) / kRT;
    const int hl = wn + (lane >> 4) * 4;  // first hidden unit of this lane's accumulators
    // features: four of one row per thread, two tiles ahead
    static_assert(kRT * kIn == 64 * NW * 4, "a tile's features take one load per thread");
    const int xrow = tid >> 3, xcol = (tid & 7) * 4;
    float4 xr;
    auto load_x = [&](int64_t t) {
        const int64_t r = t * kRT + xrow;
        xr = r < rows ? *reinterpret_cast<const float4 *>(x + r * kIn + xcol) : float4{0.f, 0.f, 0.f, 0.f};
    };
    auto put_x = [&](int b) {
        *reinterpret_cast<uint2 *>(&Xs[b][xrow * kXRow + xcol]) = make_uint2(f2bf2(xr.x, xr.y), f2bf2(xr.z, xr.w));
    };
    load_x(blockIdx.x);
    put_x(0);
    load_x(blockIdx.x + (int64_t)gridDim.x);
    __syncthreads();
    for (int64_t tile = blockIdx.x, b = 0; tile < tiles; tile += gridDim.x, b ^= 1) {
        const int64_t r0 = tile * kRT;
        put_x((int)b ^ 1);
        load_x(tile + 2 * (int64_t)gridDim.x);
        f32x4 bias[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ct++) bias[ct] = *reinterpret_cast<const f32x4 *>(&sb1[hl + ct * 16]);
        // computed transposed (W1^T as the A operand), so that a lane holds 4
        // consecutive hidden units of one row and stores them as one 8-byte write
#pragma unroll
        for (int rt = 0; rt < 4; rt++) {
            // A-fragment row lc of the 16-row tile, K = lk .. lk+7
            const bf16x8 af1 = *reinterpret_cast<const bf16x8 *>(&Xs[b][(rt * 16 + lc) * kXRow + lk]);
#pragma unroll
            for (int ct = 0; ct < CT; ct++) {
                f32x4 acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1f[ct], af1, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                uint2 h;
                h.x = relu_bf2(f2bf2(acc[0] + bias[ct][0], acc[1] + bias[ct][1]));
                h.y = relu_bf2(f2bf2(acc[2] + bias[ct][2], acc[3] + bias[ct][3]));
                *reinterpret_cast<uint2 *>(&H1s[(rt * 16 + lc) * kH1Row + hl + ct * 16]) = h;
            }
        }
        __syncthreads();
        // layer 2, transposed as well: per 16-column tile a lane holds 4
        // consecutive hidden units of row rt * 16 + lc, so its output partials
        // cover 4 CT units and only the 4 lane groups of a row remain to be added
        bf16x2_t w30[CT][2], w31[CT][2];
#pragma unroll
        for (int ct = 0; ct < CT; ct++) {
            bias[ct] = *reinterpret_cast<const f32x4 *>(&sb2[hl + ct * 16]);
#pragma unroll
            for (int i = 0; i < 2; i++) {
                w30[ct][i] = __builtin_bit_cast(bf16x2_t, sw[0][(hl + ct * 16) / 2 + i]);
                w31[ct][i] = __builtin_bit_cast(bf16x2_t, sw[1][(hl + ct * 16) / 2 + i]);
            }
        }
#pragma unroll
        for (int rt = 0; rt < 4; rt++) {
            f32x4 acc[CT];
#pragma unroll
            for (int ct = 0; ct < CT; ct++) acc[ct] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 8; ks++) {
                const bf16x8 hf = *reinterpret_cast<const bf16x8 *>(&H1s[(rt * 16 + lc) * kH1Row + ks * 32 + lk]);
#pragma unroll
                for (int ct = 0; ct < CT; ct++)
                    acc[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w2f[ks][ct], hf, acc[ct], 0, 0, 0);
            }
            float s0 = 0.f, s1 = 0.f;
#pragma unroll
            for (int ct = 0; ct < CT; ct++)
#pragma unroll
                for (int i = 0; i < 4; i += 2) {
                    // the bf16 rounding of H2, two units per conversion, and
                    // their products with the output weights as one bf16 dot
                    // product per output
                    const bf16x2_t q = __builtin_bit_cast(
                        bf16x2_t, relu_bf2(f2bf2(acc[ct][i] + bias[ct][i], acc[ct][i + 1] + bias[ct][i + 1])));
                    s0 = __builtin_amdgcn_fdot2_f32_bf16(q, w30[ct][i / 2], s0, false);
                    s1 = __builtin_amdgcn_fdot2_f32_bf16(q, w31[ct][i / 2], s1, false);
                }
            // lanes lc, lc + 16, lc + 32, lc + 48 hold the same row
            s0 += __shfl_xor(s0, 16, 64);
            s1 += __shfl_xor(s1, 16, 64);
            s0 += __shfl_xor(s0, 32, 64);
            s1 += __shfl_xor(s1, 32, 64);
            if (lane < 16) *reinterpret_cast<float2 *>(yp[wv][rt * 16 + lc]) = make_float2(s0, s1);
        }
        __syncthreads();
        if (tid < kRT * 2) {
            const int row = tid >> 1, c = tid & 1;
            const int64_t r = r0 + row;
            if (r < rows) {
                float y = yp[0][row][c];
#pragma unroll
                for (int w = 1; w < NW; w++) y += yp[w][row][c];
                y += c ? b31 : b30;
                if (Y) Y[2 * r + c] = y;
                if (est) est[2 * r + c] = (int32_t)fminf(fmaxf(rintf(expf(y)), 1.f), (float)(1 << 20));
            }
        }
    }
}

static unsigned blocks(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

static bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }

// Chunks of the batch in a weight gradient of `tiles` 64 x 64 output tiles:
// as many as fill 256 work-groups of one tile each, at most `most`.
static void batch_chunks(int64_t rows, int tiles, int64_t most, int32_t *chunk, int32_t *n) {
    const int64_t kt = (rows + 31) / 32, S = std::min<int64_t>({kt, (int64_t)std::max(1, 256 / tiles), most});
    *chunk = (int32_t)((kt + S - 1) / S * 32);
    *n = (int32_t)((rows + *chunk - 1) / *chunk);
}

}  // namespace insp

using namespace insp;

struct insp_mlp {
    int device = 0;
    int64_t step = 0;
    DevBuf p, g, m, v;            // fp32 [kParams]
    DevBuf w1t, w2, w2t, w3;      // bf16 shadows: W1^T, W2 and W2^T in fragment order, W3 [256][2]
    DevBuf loss;                  // fp32 [1]
    int64_t cap = 0;              // rows the activation buffers hold
    DevBuf xt, h1t, h2t, d2t, d1t;  // bf16 activations and gradients by unit (fragment order; h2t [unit][rows])
    DevBuf y;                     // fp32 [cap, 2]
    DevBuf part, colpart;         // fp32 partial sums for the fixed-order reductions
    int64_t gen = 0;              // bumped whenever a buffer above moves
    // graph-captured training
    DevBuf tab;                   // int32 step index, step in hand, then the bias-correction table
    hipStream_t cs = nullptr;     // capture stream
    hipGraphExec_t exec = nullptr;
    struct Key {
        const float *x, *t;
        int32_t steps, batch, chunk;
        float lr;
        int64_t gen;
        bool operator==(const Key &o) const {
            return x == o.x && t == o.t && steps == o.steps && batch == o.batch && chunk == o.chunk && lr == o.lr &&
                   gen == o.gen;
        }
    } key{};
    ~insp_mlp() {
        // work queued on the caller's streams may still use the graph and buffers
        (void)hipDeviceSynchronize();
        if (exec) (void)hipGraphExecDestroy(exec);
        if (cs) (void)hipStreamDestroy(cs);
    }
};

// Grow the per-row buffers to `rows`.  All-or-nothing: the new buffers are
// allocated beside the old ones and swapped in only when every allocation
// succeeded, so a failure (INSP_E_NOMEM) leaves the model as it was.
static int mlp_reserve(insp_mlp *m, int64_t rows) {
    if (rows <= m->cap) return INSP_OK;
    DevBuf *cur[8] = {&m->xt, &m->h1t, &m->h2t, &m->d2t, &m->d1t, &m->y, &m->part, &m->colpart};
    const size_t bytes[8] = {(size_t)(2 * kIn * rows),  (size_t)(2 * kHid * rows), (size_t)(2 * kHid * rows),
                             (size_t)(2 * kHid * rows), (size_t)(2 * kHid * rows), (size_t)(4 * kOut * rows),
                             (size_t)(4 * (rows / 4) * kPart), (size_t)(4 * (rows / kRows) * kHid)};
    DevBuf fresh[8];
    for (int i = 0; i < 8; i++)
        if (int rc = fresh[i].alloc(bytes[i])) return rc;
    for (int i = 0; i < 8; i++) cur[i]->swap(fresh[i]);  // the old buffers are released on return
    m->cap = rows;
    m->gen++;
    return INSP_OK;
}

// What a step writes besides the parameters: gradients (instead of Adam's
// update), outputs and loss.
struct StepOut {
    float *grads, *y, *loss;
};

// One step over a batch of B rows (a multiple of 32): two launches.  With
// `tab` the batch is minibatch tab[0] mod `steps` of x and t (graph-captured
// training).
static int mlp_step(insp_mlp *m, const float *x, const float *t, int64_t B, const StepOut &out, float lr, float bc1,
                    float bc2, hipStream_t st, int32_t *tab = nullptr, int32_t steps = 1, int32_t tabn = 0) {
    StepArgs a;
    a.x = x;
    a.t = t;
    a.rows = B;
    a.tab = tab;
    a.steps = steps;
    a.p = m->p.as<float>();
    a.w1t = m->w1t.as<uint16_t>();
    a.w2 = m->w2.as<uint16_t>();
    a.w2t = m->w2t.as<uint16_t>();
    a.w3 = m->w3.as<uint16_t>();
    a.xt = m->xt.as<uint16_t>();
    a.h1t = m->h1t.as<uint16_t>();
    a.h2t = m->h2t.as<uint16_t>();
    a.d2t = m->d2t.as<uint16_t>();
    a.d1t = m->d1t.as<uint16_t>();
    a.y = out.y;
    a.part = m->part.as<float>();
    a.colpart = m->colpart.as<float>();
    a.cur = tab ? tab + 1 : nullptr;
    // rows are 128 bytes, so every minibatch is aligned when x is
    if (aligned16(x))
        hipLaunchKernelGGL(k_rows_step<true>, dim3((unsigned)(B / kRows)), dim3(64 * kRowWaves), 0, st, a);
    else
        hipLaunchKernelGGL(k_rows_step<false>, dim3((unsigned)(B / kRows)), dim3(64 * kRowWaves), 0, st, a);
    ParamArgs q;
    q.t = t;
    q.rows = B;
    q.tab = tab;
    q.steps = steps;
    q.tabn = tabn;
    q.xt = a.xt;
    q.h1t = a.h1t;
    q.h2t = a.h2t;
    q.d2t = a.d2t;
    q.d1t = a.d1t;
    q.y = out.y;
    q.part = a.part;
    q.colpart = a.colpart;
    batch_chunks(B, kHid / 64, 128, &q.chunk1, &q.n1);
    batch_chunks(B, (kHid / 64) * (kHid / 64), 16, &q.chunk2, &q.n2);
    q.grads = out.grads;
    q.loss = out.loss;
    q.p = m->p.as<float>();
    q.m = m->m.as<float>();
    q.v = m->v.as<float>();
    q.lr = lr;
    q.bc1 = bc1;
    q.bc2 = bc2;
    q.w1t = m->w1t.as<uint16_t>();
    q.w2 = m->w2.as<uint16_t>();
    q.w2t = m->w2t.as<uint16_t>();
    q.w3 = m->w3.as<uint16_t>();
    hipLaunchKernelGGL(k_params_step, dim3(kGrid2), dim3(256), 0, st, q);
    INSP_HIP(hipGetLastError());
    return INSP_OK;
}

extern "C" int insp_mlp_create(const float *params, insp_mlp **out) {
    if (!params || !out) return set_error(INSP_E_INVAL, "null argument");
    std::unique_ptr<insp_mlp> m(new insp_mlp());
    INSP_HIP(hipGetDevice(&m->device));
    int rc;
    if ((rc = m->p.alloc(4 * kParams)) || (rc = m->g.alloc(4 * kParams)) || (rc = m->m.alloc(4 * kParams)) ||
        (rc = m->v.alloc(4 * kParams)) || (rc = m->w1t.alloc(2 * kIn * kHid)) ||
        (rc = m->w2.alloc(2 * kHid * kHid)) || (rc = m->w2t.alloc(2 * kHid * kHid)) ||
        (rc = m->w3.alloc(2 * kHid * kOut)) || (rc = m->loss.alloc(4)))
        return rc;
    INSP_HIP(hipMemcpy(m->p.p, params, 4 * kParams, hipMemcpyHostToDevice));
    INSP_HIP(hipMemset(m->m.p, 0, 4 * kParams));
    INSP_HIP(hipMemset(m->v.p, 0, 4 * kParams));
    hipLaunchKernelGGL(k_shadow, dim3(blocks(kParams, 256)), dim3(256), 0, 0, m->p.as<float>(), m->w1t.as<uint16_t>(),
                       m->w2.as<uint16_t>(), m->w2t.as<uint16_t>(), m->w3.as<uint16_t>());
    INSP_HIP(hipGetLastError());
    INSP_HIP(hipDeviceSynchronize());
    *out = m.release();
    return INSP_OK;
}

extern "C" void insp_mlp_free(insp_mlp *m) { delete m; }

// The model's buffers live on the device that was current at create: work
// for it must be launched there.
static int check_device(const insp_mlp *m) {
    int dev = -1;
    INSP_HIP(hipGetDevice(&dev));
    if (dev != m->device) return set_error(INSP_E_INVAL, "the current device is not the model's device");
    return INSP_OK;
}

// Whether [p, p + n) and [q, q + k) share a byte.
static bool overlap(const void *p, size_t n, const void *q, size_t k) {
    const uintptr_t a = (uintptr_t)p, b = (uintptr_t)q;
    return a < b + k && b < a + n;
}

extern "C" int insp_mlp_grads(insp_mlp *m, const float *x, const float *t, int32_t batch, float *grads, float *y,
                              float *loss, void *stream) {
    if (!m || !x || !t || batch < 1 || batch % 32) return set_error(INSP_E_INVAL, "bad argument");
    hipStream_t st = (hipStream_t)stream;
    int rc;
    if ((rc = check_device(m)) || (rc = mlp_reserve(m, batch))) return rc;
    // results go straight to the caller's arrays; one that shares memory with
    // the inputs or another result is filled by a copy at the end, as nothing
    // may change an input that is still read
    const size_t xb = 4 * kIn * (size_t)batch, tb = 4 * kOut * (size_t)batch;
    struct { float *user, *own; size_t bytes; float *to; } o[3] = {
        {grads, m->g.as<float>(), 4 * kParams, nullptr}, {y, m->y.as<float>(), tb, nullptr},
        {loss, m->loss.as<float>(), 4, nullptr}};
    for (int i = 0; i < 3; i++) {
        bool direct = o[i].user && !overlap(o[i].user, o[i].bytes, x, xb) && !overlap(o[i].user, o[i].bytes, t, tb);
        for (int j = 0; j < 3; j++)
            if (j != i && o[j].user && direct) direct = !overlap(o[i].user, o[i].bytes, o[j].user, o[j].bytes);
        o[i].to = direct ? o[i].user : o[i].own;
    }
    if ((rc = mlp_step(m, x, t, batch, StepOut{o[0].to, o[1].to, o[2].to}, 0.f, 1.f, 1.f, st))) return rc;
    for (auto &q : o)
        if (q.user && q.to != q.user) INSP_HIP(hipMemcpyAsync(q.user, q.to, q.bytes, hipMemcpyDeviceToDevice, st));
    return INSP_OK;
}

extern "C" int insp_mlp_train_step(insp_mlp *m, const float *x, const float *t, int32_t batch, float lr, float *loss,
                                   void *stream) {
    if (!m || !x || !t || batch < 1 || batch % 32 || !(lr > 0.f)) return set_error(INSP_E_INVAL, "bad argument");
    hipStream_t st = (hipStream_t)stream;
    int rc;
    if ((rc = check_device(m)) || (rc = mlp_reserve(m, batch))) return rc;
    const float bc1 = 1.f - powf(0.9f, (float)(m->step + 1)), bc2 = 1.f - powf(0.999f, (float)(m->step + 1));
    if ((rc = mlp_step(m, x, t, batch, StepOut{nullptr, m->y.as<float>(), m->loss.as<float>()}, lr, bc1, bc2, st)))
        return rc;
    m->step++;
    if (loss) INSP_HIP(hipMemcpyAsync(loss, m->loss.p, 4, hipMemcpyDeviceToDevice, st));
    return INSP_OK;
}

// One step of graph-captured training: minibatch tab[0] mod steps, Adam with
// the tabled corrections of that step.
static int train_enqueue(insp_mlp *m, const float *x, const float *t, int32_t steps, int32_t batch, float lr,
                         int32_t tabn, hipStream_t st) {
    return mlp_step(m, x, t, batch, StepOut{nullptr, m->y.as<float>(), m->loss.as<float>()}, lr, 1.f, 1.f, st,
                    m->tab.as<int32_t>(), steps, tabn);
}

// Captures `chunk` consecutive steps into m->exec (on the model's own
// stream: capture leaves the caller's stream alone).
static int train_capture(insp_mlp *m, const float *x, const float *t, int32_t steps, int32_t batch, float lr,
                         int32_t chunk, int32_t tabn) {
    if (m->exec) {
        (void)hipGraphExecDestroy(m->exec);
        m->exec = nullptr;
    }
    if (!m->cs) INSP_HIP(hipStreamCreateWithFlags(&m->cs, hipStreamNonBlocking));
    INSP_HIP(hipStreamBeginCapture(m->cs, hipStreamCaptureModeThreadLocal));
    int rc = INSP_OK;
    for (int32_t s = 0; s < chunk && rc == INSP_OK; s++) rc = train_enqueue(m, x, t, steps, batch, lr, tabn, m->cs);
    hipGraph_t g = nullptr;
    const hipError_t e = hipStreamEndCapture(m->cs, &g);
    if (rc == INSP_OK && e != hipSuccess) rc = set_error(INSP_E_DEVICE, hipGetErrorString(e));
    if (rc == INSP_OK) {
        const hipError_t ei = hipGraphInstantiate(&m->exec, g, nullptr, nullptr, 0);
        if (ei != hipSuccess) {
            m->exec = nullptr;
            rc = set_error(INSP_E_DEVICE, hipGetErrorString(ei));
        }
    }
    if (g) (void)hipGraphDestroy(g);
    return rc;
}

extern "C" int insp_mlp_train(insp_mlp *m, const float *x, const float *t, int64_t n, int32_t batch, int32_t epochs,
                              float lr, float *loss, void *stream) {
    if (!m || n < 0 || epochs < 0 || batch < 1 || batch % 32 || !(lr > 0.f) || (n > 0 && (!x || !t)))
        return set_error(INSP_E_INVAL, "bad argument");
    const int64_t steps = n / batch, total = steps * epochs;
    if (total == 0) return INSP_OK;
    if (total > kMaxTrainSteps) return set_error(INSP_E_RANGE, "more than 2^28 training steps in one call");
    hipStream_t st = (hipStream_t)stream;
    const int64_t words = 2 + 2 * total;
    int rc;
    if ((rc = check_device(m))) return rc;
    if (m->cap < batch || m->tab.bytes < (size_t)(4 * words)) {
        INSP_HIP(hipStreamSynchronize(st));  // earlier work on the stream may still read the old buffers
        if ((rc = mlp_reserve(m, batch))) return rc;
        if (m->tab.bytes < (size_t)(4 * words)) {
            DevBuf fresh;
            if ((rc = fresh.alloc(4 * words))) return rc;
            m->tab.swap(fresh);
            m->gen++;
        }
    }
    // step index and step in hand 0, then the corrections of steps step+1 ..
    // step+total, as the eager step computes them
    std::vector<int32_t> h((size_t)words);
    h[0] = h[1] = 0;
    for (int64_t s = 1; s <= total; s++) {
        const float bc1 = 1.f - powf(0.9f, (float)(m->step + s)), bc2 = 1.f - powf(0.999f, (float)(m->step + s));
        memcpy(&h[2 * s], &bc1, 4);
        memcpy(&h[2 * s + 1], &bc2, 4);
    }
    INSP_HIP(hipMemcpyAsync(m->tab.p, h.data(), 4 * words, hipMemcpyHostToDevice, st));
    INSP_HIP(hipStreamSynchronize(st));  // h is released on return
    const int32_t chunk = (int32_t)std::min<int64_t>(total, kTrainChunk);
    const int32_t tabn = (int32_t)((m->tab.bytes / 4 - 2) / 2);  // entries the table holds
    const insp_mlp::Key k{x, t, (int32_t)steps, batch, chunk, lr, m->gen};
    if (!m->exec || !(k == m->key)) {
        m->key = insp_mlp::Key{};
        if ((rc = train_capture(m, x, t, (int32_t)steps, batch, lr, chunk, tabn))) return rc;
        m->key = k;
    }
    for (int64_t s = 0; s + chunk <= total; s += chunk) INSP_HIP(hipGraphLaunch(m->exec, st));
    for (int64_t s = total - total % chunk; s < total; s++)
        if ((rc = train_enqueue(m, x, t, (int32_t)steps, batch, lr, tabn, st))) return rc;
    m->step += total;
    if (loss) INSP_HIP(hipMemcpyAsync(loss, m->loss.p, 4, hipMemcpyDeviceToDevice, st));
    return INSP_OK;
}

extern "C" int insp_mlp_predict(insp_mlp *m, const float *x, int64_t n, float *y, int32_t *est, void *stream) {
    if (!m || (n > 0 && (!x || (!y && !est))) || n < 0) return set_error(INSP_E_INVAL, "bad argument");
    if (n == 0) return INSP_OK;
    // the features are read 16 bytes at a time
    if ((uintptr_t)x & 15) return set_error(INSP_E_INVAL, "x must be 16-byte aligned");
    if (int rc = check_device(m)) return rc;
    hipStream_t st = (hipStream_t)stream;
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess) cus = n;
    }
    const int64_t tiles = (n + kRT - 1) / kRT;
    const unsigned grid = (unsigned)std::min<int64_t>(tiles, (int64_t)cus * 2);
    ProfScope ps(st, "mlp_infer");
    hipLaunchKernelGGL(k_infer<kInferWaves>, dim3(grid), dim3(64 * kInferWaves), 0, st, x, n, m->w1t.as<uint16_t>(), m->p.as<float>() + kOffB1,
                       m->w2t.as<uint16_t>(), m->p.as<float>() + kOffB2, m->w3.as<uint16_t>(),
                       m->p.as<float>() + kOffB3, y, est);
    INSP_HIP(hipGetLastError());
    return INSP_OK;
}

extern "C" int insp_mlp_state(insp_mlp *m, float *params, float *adam_m, float *adam_v, int64_t *step, int to_host) {
    if (!m) return set_error(INSP_E_INVAL, "null model");
    INSP_HIP(hipDeviceSynchronize());
    const hipMemcpyKind k = to_host ? hipMemcpyDeviceToHost : hipMemcpyHostToDevice;
    struct { float *h; DevBuf *d; } parts[3] = {{params, &m->p}, {adam_m, &m->m}, {adam_v, &m->v}};
    for (auto &pp : parts)
        if (pp.h) {
            if (to_host) INSP_HIP(hipMemcpy(pp.h, pp.d->p, 4 * kParams, k));
            else INSP_HIP(hipMemcpy(pp.d->p, pp.h, 4 * kParams, k));
        }
    if (step) {
        if (to_host) *step = m->step;
        else m->step = *step;
    }
    if (!to_host && params) {
        hipLaunchKernelGGL(k_shadow, dim3(blocks(kParams, 256)), dim3(256), 0, 0, m->p.as<float>(),
                           m->w1t.as<uint16_t>(), m->w2.as<uint16_t>(), m->w2t.as<uint16_t>(), m->w3.as<uint16_t>());
        INSP_HIP(hipGetLastError());
        INSP_HIP(hipDeviceSynchronize());
    }
    return INSP_OK;
}

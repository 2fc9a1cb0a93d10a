// Slopes of the line search's bracketing test, a whole group of steps at once.  The test needs grad E_sub(W + alpha d) . d,
// a directional derivative, and that does not need the gradient: with P = X W1 and Q = X d1 (the same for every step)
//
//     H = tanh(P + alpha Q)                     H' = (1 - H ** H) ** Q
//     Z = H (W2 + alpha d2)                     Z' = H' (W2 + alpha d2) + H d2
//     slope = sum over patterns and classes of (softmax(Z) - onehot) ** Z'
//
// Z and Z' of all steps are ONE product, [H | alpha H] and [H' | alpha H' + H] stacked over the steps and multiplied with
// W2 on top of d2.  What bound the gradients it replaces: 11 launches per step on a few hundred patterns, none of which
// fills the chip (400-480-3203, 512 patterns: 95 us per step; here 8 steps take one product of 8192 x 3203 x 960 and four
// launches, 40 us per step).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mlp_kernels.hpp"   // block reductions, tanh_f32

namespace ulsnn {

constexpr int LS_GROUP = 8;          // most steps evaluated together
struct LineSearchSteps {
    float alpha[LS_GROUP];
    int count;
};

// The stacked left operand, 2 * count * rows x 2 * n_hid (row stride lda): rows (a, r) hold [H | alpha H] of step a and
// pattern r, rows (count + a, r) [H' | alpha H' + H].  P, Q: rows x n_hid with row stride ldp.
__global__ __launch_bounds__(256) void ls_stack_kernel(const float *__restrict__ P, const float *__restrict__ Q, int ldp,
                                                       int rows, int n_hid, LineSearchSteps steps, float *__restrict__ A,
                                                       int lda)
{
    const size_t total = (size_t)rows * n_hid;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (size_t)gridDim.x * 256) {
        const size_t r = i / n_hid, j = i - r * n_hid;
        const float p = P[r * ldp + j], q = Q[r * ldp + j];
        for (int a = 0; a < steps.count; ++a) {
            const float alpha = steps.alpha[a];
            const float h = tanh_f32(__builtin_fmaf(alpha, q, p));
            const float hd = (1.0f - h * h) * q;
            float *top = A + ((size_t)a * rows + r) * lda + j;
            float *bottom = A + ((size_t)(steps.count + a) * rows + r) * lda + j;
            top[0] = h;
            top[n_hid] = alpha * h;
            bottom[0] = hd;
            bottom[n_hid] = __builtin_fmaf(alpha, hd, h);
        }
    }
}

// One wavefront per step and pattern: value[b] = sum_c (softmax(Z)_c - [c == label]) Z'_c with Z in row b of U and Z' in row
// half + b; 0 for a label out of range (an ignored pattern).  Rows of U are 16-byte aligned.  One pass over both rows: a
// lane rescales its running sums where its maximum grows, and the lanes' (maximum, sums) are merged at the end.  Bound by
// reading U (8 steps of 512 x 3203: 26 us with a workgroup per row, three passes and 4-byte loads; 17.6 now).
__global__ __launch_bounds__(256) void ls_slope_row_kernel(const float *__restrict__ U, int ld, size_t half, int rows, int n,
                                                           const int32_t *__restrict__ labels, double *__restrict__ value)
{
    const int lane = threadIdx.x & 63;
    const size_t b = (size_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (b >= half) return;
    const float *z = U + b * ld, *zd = U + (half + b) * ld;
    const int y = labels[b % rows];
    const bool labelled = y >= 0 && y < n;
    const float zdy = labelled ? zd[y] : 0.f;
    float m = -INFINITY, s = 0.f, t = 0.f;
    constexpr int V = 4;                                   // vectors in flight per lane and row
    for (int base = lane * 4; base < n; base += 256 * V) {
        floatx4 a[V], d[V];
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const int c = base + v * 256;
            a[v] = floatx4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
            d[v] = floatx4{0.f, 0.f, 0.f, 0.f};
            if (c < n) {
                a[v] = *reinterpret_cast<const floatx4 *>(z + c);
                d[v] = *reinterpret_cast<const floatx4 *>(zd + c);
            }
        }
        float nm = m;
#pragma unroll
        for (int v = 0; v < V; ++v) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (base + v * 256 + e >= n) {
                    a[v][e] = -INFINITY;
                    d[v][e] = 0.f;
                }
                nm = fmaxf(nm, a[v][e]);
            }
        }
        const float scale = nm == m ? 1.0f : __expf(m - nm);   // (m = -inf on the first round: 0)
        s *= scale;
        t *= scale;
        m = nm;
        const float base_m = m == -INFINITY ? 0.f : m;         // (only logits of -inf so far: they weigh nothing, not NaN)
#pragma unroll
        for (int v = 0; v < V; ++v) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float x = __expf(a[v][e] - base_m);
                s += x;
                t += x * d[v][e];
            }
        }
    }
    const float all = wave_max(m);
    const float scale = m == all ? 1.0f : __expf(m - all);     // lanes without a column: exp(-inf) = 0
    s = wave_sum(s * scale);
    t = wave_sum(t * scale);
    if (lane == 0) value[b] = labelled ? (double)(t / s) - (double)zdy : 0.0;
}

// slope[a] = sum over the patterns of step a, one workgroup per step, fixed order.
__global__ __launch_bounds__(256) void ls_slope_sum_kernel(const double *__restrict__ value, int rows, float *__restrict__ slope)
{
    __shared__ double red[4];
    double s = 0.0;
    const double *v = value + (size_t)blockIdx.x * rows;
    for (int r = threadIdx.x; r < rows; r += 256) s += v[r];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) slope[blockIdx.x] = (float)(((red[0] + red[1]) + red[2]) + red[3]);
}

}  // namespace ulsnn

// Networks whose layers are all at most 64 wide: the whole forward pass, and the whole backward pass with its update,
// in one launch each.
//
// What bounds such a network is the number of launches: the 40-64-64-32 network at 32 rows does 2 MFLOP per pass and took
// eight launches of about 5 us per minibatch, each a handful of dependent loads.  A layer of 32 rows is eight 16x16 blocks
// here, of 64 rows sixteen, one per wavefront (v_mfma_f32_16x16x4_f32, fp32 throughout); activations and errors stay in
// LDS between layers, and the weights of the next layer are requested before the current one is finished.
// Four replicas of 40-64-64-32, two minibatches of 32 rows and the averaging: 51 us with 5 launches, was 79 with 17.
// The limits are the tile: one block per wavefront needs no loop over blocks, and the backward pass keeps all rows of a
// replica in one workgroup (more rows take the general kernels, as do networks with one wider layer).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gemm.h"
#include "kernels.h"
#include "device_math.h"

namespace mavg {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kW = kNarrowWidth, kLd = kW + 4;      // LDS row stride: 16-byte aligned, consecutive rows four banks apart

// v_mfma_f32_16x16x4_f32: lane l holds A[l % 16][l / 16] and B[l / 16][l % 16], and D[4 (l / 16) + v][l % 16], v = 0..3.
// Chunk j of 16 contraction steps: MFMA number c multiplies steps 16 j + 4 (l / 16) + c, so that a lane's four operands of
// a chunk are neighbours.
__device__ __forceinline__ floatx4 mfma16(float a, float b, floatx4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

__device__ __forceinline__ int64_t layer_params(const NarrowNet& t, int l) { return (int64_t)t.d[l] * (t.d[l - 1] + 1); }

// A workgroup takes 32 rows of one replica through all layers and the softmax.
__global__ __launch_bounds__(512) void narrow_forward_kernel(NarrowNet t, const float* __restrict__ theta, int64_t theta_stride,
                                                             const float* __restrict__ x, int64_t x_stride, int n,
                                                             float* __restrict__ acts, int64_t act_stride) {
    __shared__ __attribute__((aligned(16))) float S[2][32][kLd];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int q = lane >> 4, c16 = lane & 15, rb = wave & 1, col = 16 * (wave >> 1) + c16;
    const int r0 = blockIdx.x * 32, rows = min(32, n - r0);
    theta += (int64_t)blockIdx.y * theta_stride;
    x += (int64_t)blockIdx.y * x_stride + (int64_t)r0 * t.d[0];
    acts += (int64_t)blockIdx.y * act_stride;
    float w[4][4], bias;
    auto load_weights = [&](int l) {       // theta: at layer l's parameters
        const int K = t.d[l - 1], N = t.d[l];
        const float* row = theta + (int64_t)col * K;
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int k = 16 * j + 4 * q + c;
                w[j][c] = col < N && k < K ? row[k] : 0.f;
            }
        bias = col < N ? theta[(int64_t)N * K + col] : 0.f;
    };
    load_weights(1);
    for (int i = tid; i < 32 * kW; i += 512) {
        const int r = i / kW, c = i % kW;
        S[0][r][c] = r < rows && c < t.d[0] ? x[(int64_t)r * t.d[0] + c] : 0.f;
    }
    for (int l = 1; l <= t.L; ++l) {
        const int cur = (l - 1) & 1, N = t.d[l];
        __syncthreads();
        floatx4 part[2] = {};       // (even and odd chunks: half as many roundings in a row)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (16 * j < t.d[l - 1]) {
                const floatx4 a = *reinterpret_cast<const floatx4*>(&S[cur][16 * rb + c16][16 * j + 4 * q]);
#pragma unroll
                for (int c = 0; c < 4; ++c) part[j & 1] = mfma16(a[c], w[j][c], part[j & 1]);
            }
        const floatx4 acc = part[0] + part[1];
        const float bias_l = bias;
        if (l < t.L) {
            theta += layer_params(t, l);
            load_weights(l + 1);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = 16 * rb + 4 * q + v;
            float y = acc[v] + bias_l;
            if (l < t.L) {
                y = t.act_tanh ? tanhf(y) : sigmoidf_dev(y);
                if (r < rows && col < N) acts[(int64_t)(r0 + r) * N + col] = y;
            }
            S[cur ^ 1][r][col] = col < N ? y : 0.f;      // (zeros: the next layer's contraction runs in whole chunks)
        }
        if (l < t.L) acts += (int64_t)n * N;
    }
    __syncthreads();
    // softmax: 16 lanes per row
    const int row = tid >> 4, N = t.d[t.L];
    const float (*z)[kLd] = S[t.L & 1];
    float v[4], m = -INFINITY, s = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[i] = c16 + 16 * i < N ? z[row][c16 + 16 * i] : -INFINITY;
        m = fmaxf(m, v[i]);
    }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 16));
#pragma unroll
    for (int i = 0; i < 4; ++i) { v[i] = expf(v[i] - m); s += v[i]; }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) s += __shfl_xor(s, o, 16);
    const float inv = 1.f / s;
    if (row < rows)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (c16 + 16 * i < N) acts[(int64_t)(r0 + row) * N + c16 + 16 * i] = v[i] * inv;
}

// One workgroup per replica, up to 64 rows: the error of the output layer and the loss, then per layer from the last one
// down the error of the layer below (with the weights as they were) and the updates of the layer's weights and biases.
__global__ __launch_bounds__(1024) void narrow_backward_kernel(NarrowNet t, float* __restrict__ theta, int64_t theta_stride, int64_t params,
                                                               const float* __restrict__ x, int64_t x_stride,
                                                               const int32_t* __restrict__ labels, int64_t label_stride, int n,
                                                               const float* __restrict__ acts, int64_t act_stride, int64_t act_count,
                                                               float lr, float scale, float* __restrict__ loss_sum) {
    __shared__ __attribute__((aligned(16))) float D[2][kNarrowRows][kLd];       // errors; rows past n and columns past the layer are zero
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int q = lane >> 4, c16 = lane & 15, mb = 16 * (wave & 3), col = 16 * (wave >> 2) + c16;
    theta += (int64_t)blockIdx.x * theta_stride + params;
    x += (int64_t)blockIdx.x * x_stride;
    labels += (int64_t)blockIdx.x * label_stride;
    acts += (int64_t)blockIdx.x * act_stride + act_count - (int64_t)n * t.d[t.L];
    {
        const int N = t.d[t.L];
        for (int i = tid; i < kNarrowRows * kW; i += 1024) {
            const int r = i / kW, c = i % kW;
            float v = 0.f;
            if (r < n && c < N) {
                const float p = acts[(int64_t)r * N + c];
                v = (c == labels[r] ? p - 1.f : p) * scale;
            }
            D[0][r][c] = v;
        }
        if (wave == 0 && loss_sum != nullptr) {
            float s = 0.f;
            if (lane < n) {
                const int y = labels[lane];
                if (y >= 0 && y < N) s = -logf(acts[(int64_t)lane * N + y]);
            }
            s = wave_sum(s);
            if (lane == 0) loss_sum[blockIdx.x] = s;
        }
    }
    for (int l = t.L, cur = 0; l >= 1; --l, cur ^= 1) {
        const int N = t.d[l], K = t.d[l - 1];
        theta -= layer_params(t, l);
        const float* in = l > 1 ? acts - (int64_t)n * K : x;      // the layer's inputs, n x K
        float b[4][4];
        if (l > 1) {       // requested before the barrier that completes the errors
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int k = 16 * j + 4 * q + c;
                    b[j][c] = k < N && col < K ? theta[(int64_t)k * K + col] : 0.f;
                }
        }
        __syncthreads();
        if (l > 1) {       // rows mb .. of the errors of layer l - 1
            floatx4 part[2] = {};
            float a_in[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = mb + 4 * q + v;
                a_in[v] = r < n && col < K ? in[(int64_t)r * K + col] : 0.f;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (16 * j < N) {
                    const floatx4 a = *reinterpret_cast<const floatx4*>(&D[cur][mb + c16][16 * j + 4 * q]);
#pragma unroll
                    for (int c = 0; c < 4; ++c) part[j & 1] = mfma16(a[c], b[j][c], part[j & 1]);
                }
            const floatx4 acc = part[0] + part[1];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = mb + 4 * q + v;
                const float d = t.act_tanh ? acc[v] * (1.f - a_in[v] * a_in[v]) : acc[v] * a_in[v] * (1.f - a_in[v]);
                D[cur ^ 1][r][col] = r < n && col < K ? d : 0.f;
            }
        }
        // rows mb .. of the layer's gradient: sum over the minibatch's rows; `old` are the weights that the chain used
        float g[4][4], old[4], old_b = 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int k = 16 * j + 4 * q + c;
                g[j][c] = k < n && col < K ? in[(int64_t)k * K + col] : 0.f;
            }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = mb + 4 * q + v;
            old[v] = r < N && col < K ? theta[(int64_t)r * K + col] : 0.f;
        }
        float* bias = theta + (int64_t)N * K;
        if (tid < N) old_b = bias[tid];
        floatx4 part[2] = {};
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (16 * j < n) {
#pragma unroll
                for (int c = 0; c < 4; ++c) part[j & 1] = mfma16(D[cur][16 * j + 4 * q + c][mb + c16], g[j][c], part[j & 1]);
            }
        const floatx4 acc = part[0] + part[1];
        float sum = 0.f;
        if (tid < N) {
            float rows[4] = {};
            for (int r = 0; r < kNarrowRows; r += 4)      // (rows past the minibatch are zero)
#pragma unroll
                for (int i = 0; i < 4; ++i) rows[i] += D[cur][r + i][tid];
            sum = (rows[0] + rows[1]) + (rows[2] + rows[3]);
        }
        __syncthreads();       // every wavefront has read the weights
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = mb + 4 * q + v;
            if (r < N && col < K) theta[(int64_t)r * K + col] = -lr * acc[v] + old[v];
        }
        if (tid < N) bias[tid] = -lr * sum + old_b;
        acts = in;
    }
}

}  // namespace

bool narrow_net(const int* d, int L) {
    for (int l = 0; l <= L; ++l)
        if (d[l] > kNarrowWidth) return false;
    return L <= kNarrowLayers;
}

static NarrowNet make_net(const int* d, int L, int act_tanh) {
    NarrowNet t;
    t.L = L;
    t.act_tanh = act_tanh;
    for (int l = 0; l <= kNarrowLayers; ++l) t.d[l] = l <= L ? d[l] : 0;
    return t;
}

int narrow_forward_launch(const int* d, int L, int act_tanh, int k, const float* theta, int64_t theta_stride, const float* x,
                          int64_t x_stride, int n, float* acts, int64_t act_stride, hipStream_t s) {
    hipLaunchKernelGGL(narrow_forward_kernel, dim3((unsigned)((n + 31) / 32), (unsigned)k), dim3(512), 0, s, make_net(d, L, act_tanh),
                       theta, theta_stride, x, x_stride, n, acts, act_stride);
    return note_hip_error(hipGetLastError());
}

int narrow_backward_launch(const int* d, int L, int act_tanh, int k, float* theta, int64_t theta_stride, int64_t params, const float* x,
                           int64_t x_stride, const int32_t* labels, int64_t label_stride, int n, const float* acts, int64_t act_stride,
                           int64_t act_count, float lr, float scale, float* loss_sum, hipStream_t s) {
    hipLaunchKernelGGL(narrow_backward_kernel, dim3((unsigned)k), dim3(1024), 0, s, make_net(d, L, act_tanh), theta, theta_stride, params,
                       x, x_stride, labels, label_stride, n, acts, act_stride, act_count, lr, scale, loss_sum);
    return note_hip_error(hipGetLastError());
}

}  // namespace mavg

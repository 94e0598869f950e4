// Networks whose layers are all at most 64 wide: the whole forward pass, and the whole backward pass with its update,
// in one launch each.
//
// What bounds such a network is the number of launches: the 40-64-64-32 network at 32 rows does 2 MFLOP per pass and took
// eight launches of about 5 us per minibatch, each a handful of dependent loads.  A layer of 32 rows is eight 16x16 blocks
// here, of 64 rows sixteen, one per wavefront (v_mfma_f32_16x16x4_f32, fp32 throughout); activations and errors stay in
// LDS between layers, and the weights of the next layer are requested before the current one is finished.
// Four replicas of 40-64-64-32, two minibatches of 32 rows and the averaging: 43 us with 5 launches (51 without staging), was 79 with 17.
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
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));      // a 16-byte load from a 4-byte aligned address

constexpr int kW = kNarrowWidth, kLd = kW + 4;      // LDS row stride: 16-byte aligned, consecutive rows four banks apart

// v_mfma_f32_16x16x4_f32: lane l holds A[l % 16][l / 16] and B[l / 16][l % 16], and D[4 (l / 16) + v][l % 16], v = 0..3.
// Chunk j of 16 contraction steps: MFMA number c multiplies steps 16 j + 4 (l / 16) + c, so that a lane's four operands of
// a chunk are neighbours.
__device__ __forceinline__ floatx4 mfma16(float a, float b, floatx4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

__device__ __forceinline__ int64_t layer_params(const NarrowNet& t, int l) { return (int64_t)t.d[l] * (t.d[l - 1] + 1); }

// Softmax of 32 rows of N values, 16 lanes per row; the first `rows` of them go to `out`.
__device__ __forceinline__ void narrow_softmax(const float (*z)[kLd], int N, int tid, int rows, float* __restrict__ out) {
    const int row = tid >> 4, c16 = tid & 15;
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
            if (c16 + 16 * i < N) out[(int64_t)row * N + c16 + 16 * i] = v[i] * inv;
}

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
    narrow_softmax(S[t.L & 1], t.d[t.L], tid, rows, acts + (int64_t)r0 * t.d[t.L]);
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

// ---- the same with everything a pass reads requested at once ----------------------------------------
//
// The parameters come from another XCD's last launch, 1 - 2 us away, and the kernels above go there once per layer (the weights one
// layer ahead, the layer's inputs when they are needed).  Networks whose parameters, and for the backward pass the activations too, fit
// into LDS are staged there first, four layers' loads in flight together.  What they are bound by then is the number of instructions: so
// matrices come in 16-byte pieces, one per thread and 64 rows, and all have the same row stride in LDS, which leaves the
// addresses to the instructions' offsets.  Four replicas of 40-64-64-32 with 32 rows, us: forward 13.4 / 8.6, backward 11.8 / 9.8.
// LDS matrices: whole 16x16 blocks, zeros past their edges.
constexpr int kStageFloats = 36 * 1024, kStageLayers = 8, kStageBatch = 4;
// The widths in a few bytes, so that a launch's arguments come with one or two scalar loads.
struct StagedNet {
    uint64_t low; uint32_t high; int L, act_tanh;      // a byte per width
    __host__ __device__ int d(int l) const { return l < 8 ? (int)(low >> (8 * l) & 255) : (int)(high & 255); }
};
__host__ __device__ inline int up16(int v) { return (v + 15) / 16 * 16; }

// Columns 4 c .. 4 c + 3 of row r of a rows x cols matrix (row stride cols), zeros past its edges; and their place in LDS.
__device__ __forceinline__ floatx4 stage_load(const float* src, int rows, int cols, int r, int c) {
    floatx4 v = {0.f, 0.f, 0.f, 0.f};
    const float* p = src + r * cols + 4 * c;
    if ((cols & 3) == 0) {      // (uniform)
        if (r < rows && 4 * c < cols) v = *reinterpret_cast<const floatx4u*>(p);
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) if (r < rows && 4 * c + i < cols) v[i] = p[i];
    }
    return v;
}
__device__ __forceinline__ void stage_store(float* S, int rows, int r, int c, floatx4 v) {
    if (r < up16(rows)) *reinterpret_cast<floatx4*>(S + r * kLd + 4 * c) = v;
}

__global__ __launch_bounds__(512) void narrow_forward_staged_kernel(StagedNet t, const float* __restrict__ theta, int64_t theta_stride,
                                                                    const float* __restrict__ x, int64_t x_stride, int n,
                                                                    float* __restrict__ acts, int64_t act_stride) {
    __shared__ __attribute__((aligned(16))) float S[2][32][kLd];
    __shared__ __attribute__((aligned(16))) float W[kStageFloats - 2 * 32 * kLd];
    __shared__ float bias[kStageLayers][kW];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane >> 4, c16 = lane & 15, rb = wave & 1, col = 16 * (wave >> 1) + c16, sr = tid >> 4;
    const int r0 = blockIdx.x * 32, rows = min(32, n - r0);
    theta += (int64_t)blockIdx.y * theta_stride;
    acts += (int64_t)blockIdx.y * act_stride;
    const floatx4 xv = stage_load(x + (int64_t)blockIdx.y * x_stride + (int64_t)r0 * t.d(0), rows, t.d(0), sr, c16);
    float* to = W;
    for (int l0 = 1; l0 <= t.L; l0 += kStageBatch) {
        floatx4 v[kStageBatch][2];
        float b[kStageBatch];
#pragma unroll
        for (int i = 0; i < kStageBatch; ++i)
            if (l0 + i <= t.L) {
                const int N = t.d(l0 + i), K = t.d(l0 + i - 1);
                v[i][0] = stage_load(theta, N, K, sr, c16);
                v[i][1] = stage_load(theta, N, K, sr + 32, c16);
                b[i] = wave == i && lane < N ? theta[N * K + lane] : 0.f;
                theta += N * (K + 1);
            }
#pragma unroll
        for (int i = 0; i < kStageBatch; ++i)
            if (l0 + i <= t.L) {
                const int N = t.d(l0 + i);
                stage_store(to, N, sr, c16, v[i][0]);
                stage_store(to, N, sr + 32, c16, v[i][1]);
                if (wave == i) bias[l0 + i - 1][lane] = b[i];
                to += up16(N) * kLd;
            }
    }
    stage_store(&S[0][0][0], 32, sr, c16, xv);
    const float* w = W;
    for (int l = 1; l <= t.L; ++l) {
        const int cur = (l - 1) & 1, N = t.d(l), K = t.d(l - 1);
        const float* row = w + min(col, up16(N) - 1) * kLd + 4 * q;
        __syncthreads();
        floatx4 part[2] = {};       // (even and odd chunks: half as many roundings in a row)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (16 * j < K) {
                const floatx4 a = *reinterpret_cast<const floatx4*>(&S[cur][16 * rb + c16][16 * j + 4 * q]);
                const floatx4 b = *reinterpret_cast<const floatx4*>(row + 16 * j);
#pragma unroll
                for (int c = 0; c < 4; ++c) part[j & 1] = mfma16(a[c], b[c], part[j & 1]);
            }
        const floatx4 acc = part[0] + part[1];
        const float bias_l = bias[l - 1][col];
        float* out = acts + (r0 + 16 * rb + 4 * q) * (int64_t)N + col;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = 16 * rb + 4 * q + v;
            float y = acc[v] + bias_l;
            if (l < t.L) {
                y = t.act_tanh ? tanhf(y) : sigmoidf_dev(y);
                if (r < rows && col < N) out[v * N] = y;
            }
            S[cur ^ 1][r][col] = col < N ? y : 0.f;      // (zeros: the next layer's contraction runs in whole chunks)
        }
        if (l < t.L) acts += (int64_t)n * N;
        w += up16(N) * kLd;
    }
    __syncthreads();
    narrow_softmax(S[t.L & 1], t.d(t.L), tid, rows, acts + (int64_t)r0 * t.d(t.L));
}

__global__ __launch_bounds__(1024) void narrow_backward_staged_kernel(StagedNet t, float* __restrict__ theta, int64_t theta_stride, int64_t params,
                                                                      const float* __restrict__ x, int64_t x_stride,
                                                                      const int32_t* __restrict__ labels, int64_t label_stride, int n,
                                                                      const float* __restrict__ acts, int64_t act_stride, int64_t act_count,
                                                                      float lr, float scale, float* __restrict__ loss_sum) {
    __shared__ __attribute__((aligned(16))) float D[2][kNarrowRows][kLd];       // errors; rows past n and columns past the layer are zero
    __shared__ __attribute__((aligned(16))) float S[kStageFloats - 2 * kNarrowRows * kLd];      // from the last layer down: weights, inputs
    __shared__ float B[kStageLayers][kW], row_loss[kNarrowRows];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane >> 4, c16 = lane & 15, mb = 16 * (wave & 3), col = 16 * (wave >> 2) + c16, sr = tid >> 4, rows16 = up16(n);
    theta += (int64_t)blockIdx.x * theta_stride + params;
    x += (int64_t)blockIdx.x * x_stride;
    labels += (int64_t)blockIdx.x * label_stride;
    acts += (int64_t)blockIdx.x * act_stride + act_count - (int64_t)n * t.d(t.L);
    {
        const int N = t.d(t.L), y = sr < n ? labels[sr] : -1;
        floatx4 p = stage_load(acts, n, N, sr, c16);
        float* from = theta;
        const float* in = acts;
        float* to = S;
        for (int l0 = t.L; l0 >= 1; l0 -= kStageBatch) {
            floatx4 v[kStageBatch], a[kStageBatch];
            float b[kStageBatch];
#pragma unroll
            for (int i = 0; i < kStageBatch; ++i)
                if (l0 - i >= 1) {
                    const int l = l0 - i, M = t.d(l), K = t.d(l - 1);
                    from -= M * (K + 1);
                    in = l > 1 ? in - n * K : x;
                    v[i] = stage_load(from, M, K, sr, c16);
                    a[i] = stage_load(in, n, K, sr, c16);
                    b[i] = wave == i && lane < M ? from[M * K + lane] : 0.f;
                }
#pragma unroll
            for (int i = 0; i < kStageBatch; ++i)
                if (l0 - i >= 1) {
                    const int l = l0 - i, M = t.d(l);
                    stage_store(to, M, sr, c16, v[i]);
                    to += up16(M) * kLd;
                    stage_store(to, n, sr, c16, a[i]);
                    to += rows16 * kLd;
                    if (wave == i) B[l - 1][lane] = b[i];
                }
        }
        const bool classed = y >= 0 && y < N;
        const int at = classed ? y - 4 * c16 : -1;      // the label's place among this thread's four
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (at == i) {
                row_loss[sr] = -logf(p[i]);
                p[i] -= 1.f;
            }
            p[i] *= scale;
        }
        if (!classed && c16 == 0) row_loss[sr] = 0.f;
        *reinterpret_cast<floatx4*>(&D[0][sr][4 * c16]) = p;
    }
    const float* w = S;
    for (int l = t.L, cur = 0; l >= 1; --l, cur ^= 1) {
        const int N = t.d(l), K = t.d(l - 1);
        const float* in = w + up16(N) * kLd;      // the layer's inputs, n x K
        theta -= N * (K + 1);
        __syncthreads();
        if (l == t.L && wave == 15 && loss_sum != nullptr) {
            const float s = wave_sum(row_loss[lane]);
            if (lane == 0) loss_sum[blockIdx.x] = s;
        }
        if (l > 1 && mb < rows16) {       // rows mb .. of the errors of layer l - 1
            floatx4 part[2] = {};
            const float* wc = w + 4 * q * kLd + col;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (16 * j < N) {
                    const floatx4 a = *reinterpret_cast<const floatx4*>(&D[cur][mb + c16][16 * j + 4 * q]);
#pragma unroll
                    for (int c = 0; c < 4; ++c) part[j & 1] = mfma16(a[c], wc[(16 * j + c) * kLd], part[j & 1]);
                }
            const floatx4 acc = part[0] + part[1];
            const float* ac = in + (mb + 4 * q) * kLd + col;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = mb + 4 * q + v;
                const float a_in = ac[v * kLd];
                const float d = t.act_tanh ? acc[v] * (1.f - a_in * a_in) : acc[v] * a_in * (1.f - a_in);
                D[cur ^ 1][r][col] = r < n && col < K ? d : 0.f;
            }
        }
        if (mb < N && col < up16(K)) {      // rows mb .. of the layer's gradient: sum over the minibatch's rows
            floatx4 part[2] = {};
            const float* dc = &D[cur][4 * q][mb + c16];
            const float* ac = in + 4 * q * kLd + col;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (16 * j < n) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) part[j & 1] = mfma16(dc[(16 * j + c) * kLd], ac[(16 * j + c) * kLd], part[j & 1]);
                }
            const floatx4 acc = part[0] + part[1];
            const float* old = w + (mb + 4 * q) * kLd + col;
            float* out = theta + (mb + 4 * q) * K + col;
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (mb + 4 * q + v < N && col < K) out[v * K] = -lr * acc[v] + old[v * kLd];
        }
        if (tid < N) {
            float sum[4] = {};
            for (int r = 0; r < rows16; r += 4)      // (rows past the minibatch are zero)
#pragma unroll
                for (int i = 0; i < 4; ++i) sum[i] += D[cur][r + i][tid];
            theta[N * K + tid] = -lr * ((sum[0] + sum[1]) + (sum[2] + sum[3])) + B[l - 1][tid];
        }
        w = in + rows16 * kLd;
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

// Staged: parameters (n > 0: and the activations of n rows) that fit into LDS.  Workgroups of the staged kernels have a compute
// unit each, so launches of more than two rounds of them keep to the others.
static bool narrow_staged(const int* d, int L, int n, int64_t workgroups) {
    if (L > kStageLayers || workgroups > 2 * kNumCU) return false;
    int64_t f = 2 * (n > 0 ? kNarrowRows : 32) * kLd;
    for (int l = 1; l <= L; ++l) f += (int64_t)(up16(d[l]) + up16(n)) * kLd;
    return f <= kStageFloats;
}

static StagedNet make_staged(const int* d, int L, int act_tanh) {
    StagedNet t = {0, 0, L, act_tanh};
    for (int l = 0; l <= L; ++l) {
        if (l < 8) t.low |= (uint64_t)d[l] << (8 * l);
        else t.high = (uint32_t)d[l];
    }
    return t;
}

int narrow_forward_launch(const int* d, int L, int act_tanh, int k, const float* theta, int64_t theta_stride, const float* x,
                          int64_t x_stride, int n, float* acts, int64_t act_stride, hipStream_t s) {
    const dim3 grid((unsigned)((n + 31) / 32), (unsigned)k);
    if (narrow_staged(d, L, 0, (int64_t)grid.x * k))
        hipLaunchKernelGGL(narrow_forward_staged_kernel, grid, dim3(512), 0, s, make_staged(d, L, act_tanh), theta, theta_stride, x, x_stride, n, acts, act_stride);
    else
        hipLaunchKernelGGL(narrow_forward_kernel, grid, dim3(512), 0, s, make_net(d, L, act_tanh), theta, theta_stride, x, x_stride, n, acts, act_stride);
    return note_hip_error(hipGetLastError());
}

int narrow_backward_launch(const int* d, int L, int act_tanh, int k, float* theta, int64_t theta_stride, int64_t params, const float* x,
                           int64_t x_stride, const int32_t* labels, int64_t label_stride, int n, const float* acts, int64_t act_stride,
                           int64_t act_count, float lr, float scale, float* loss_sum, hipStream_t s) {
    const dim3 grid((unsigned)k), block(1024);
    if (narrow_staged(d, L, n, k))
        hipLaunchKernelGGL(narrow_backward_staged_kernel, grid, block, 0, s, make_staged(d, L, act_tanh), theta, theta_stride, params, x, x_stride, labels,
                           label_stride, n, acts, act_stride, act_count, lr, scale, loss_sum);
    else
        hipLaunchKernelGGL(narrow_backward_kernel, grid, block, 0, s, make_net(d, L, act_tanh), theta, theta_stride, params, x, x_stride, labels,
                           label_stride, n, acts, act_stride, act_count, lr, scale, loss_sum);
    return note_hip_error(hipGetLastError());
}

}  // namespace mavg

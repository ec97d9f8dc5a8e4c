// The kernel-selector network: forward, backward and Adam kernels.
//
// A 6 -> 32 -> 32 -> 3 multilayer perceptron maps the features of a
// degree-pair bucket to one logit per intersection strategy; the pipeline
// takes the argmax per bucket. Weights are bfloat16 (rounded from a float32
// master copy), biases float32, accumulation float32. Training minimises the
// weighted softmax cross-entropy with Adam on the master copy; gradients pass
// through the bfloat16 rounding unchanged.
//
// The network is tiny (1379 parameters, at most 256 buckets per graph): eight
// lanes share a sample, and the gradient sums run over the batch in a fixed
// order, so a training step is deterministic.
#include <math.h>

#include "common.h"
#include "internal.h"
#include "mlp.h"
#include "tiles.h"

namespace tcx {

// float32 -> bfloat16 bits, round to nearest, ties to even; NaN kept quiet.
__device__ __forceinline__ uint16_t to_bf16(float x) {
    const uint32_t u = __float_as_uint(x);
    if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x007FFFFFu)) return (uint16_t)((u >> 16) | 0x0040u);
    return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

constexpr int W2_LD = MLP_H + 1;   // one word of skew: lanes read different rows of W2 at one column
struct MlpShared {
    float W1[MLP_H * MLP_IN];
    float b1[MLP_H];
    float W2[MLP_H * W2_LD];
    float b2[MLP_H];
    float W3[MLP_OUT * MLP_H];
    float b3[MLP_OUT];
};

// Expand the compute copy (bf16 weights, f32 biases) into LDS as float.
__device__ void load_net(const MlpCompute* __restrict__ cw, MlpShared& S) {
    for (int i = threadIdx.x; i < MLP_H * MLP_IN; i += blockDim.x) S.W1[i] = from_bf16(cw->W1[i]);
    for (int i = threadIdx.x; i < MLP_H * MLP_H; i += blockDim.x) 
        S.W2[i / MLP_H * W2_LD + i % MLP_H] = from_bf16(cw->W2[i]);
    for (int i = threadIdx.x; i < MLP_OUT * MLP_H; i += blockDim.x) S.W3[i] = from_bf16(cw->W3[i]);
    for (int i = threadIdx.x; i < MLP_H; i += blockDim.x) { S.b1[i] = cw->b1[i]; S.b2[i] = cw->b2[i]; }
    for (int i = threadIdx.x; i < MLP_OUT; i += blockDim.x) S.b3[i] = cw->b3[i];
    __syncthreads();
}

// One sample by NET_G lanes: lane j of the group computes hidden units NET_U * j ..
// NET_U * j + NET_U - 1 of each layer and output j (j < 3); the other lanes'
// units arrive by shuffles from lane0, the group's first lane. Dot products
// accumulate in input order and the bias is added last. h1, h2: the lane's own
// units; hin: scratch for a whole layer; z: all logits, in every lane.
constexpr int NET_G = 8, NET_U = MLP_H / NET_G;
static_assert(MLP_H % NET_G == 0 && MLP_OUT <= NET_G && WAVE % NET_G == 0, "lanes per sample");

__device__ __forceinline__ void gather_layer(const float (&h)[NET_U], int lane0, float (&all)[MLP_H]) {
#pragma unroll
    for (int i = 0; i < MLP_H; ++i) all[i] = __shfl(h[i % NET_U], lane0 + i / NET_U, WAVE);
}

__device__ __forceinline__ void net_forward(const MlpShared& S, const float (&x)[MLP_IN], int j, int lane0,
                                            float (&h1)[NET_U], float (&h2)[NET_U], float (&z)[MLP_OUT]) {
#pragma unroll
    for (int u = 0; u < NET_U; ++u) {
        const int o = NET_U * j + u;
        float acc = 0.f;
        for (int i = 0; i < MLP_IN; ++i) acc = fmaf(S.W1[o * MLP_IN + i], x[i], acc);
        acc += S.b1[o];
        h1[u] = acc > 0.f ? acc : 0.f;
    }
    float hin[MLP_H];
    gather_layer(h1, lane0, hin);
#pragma unroll
    for (int u = 0; u < NET_U; ++u) {
        const int o = NET_U * j + u;
        float acc = 0.f;
#pragma unroll
        for (int i = 0; i < MLP_H; ++i) acc = fmaf(S.W2[o * W2_LD + i], hin[i], acc);
        acc += S.b2[o];
        h2[u] = acc > 0.f ? acc : 0.f;
    }
    gather_layer(h2, lane0, hin);
    const int o = j < MLP_OUT ? j : 0;
    float acc = 0.f;
#pragma unroll
    for (int i = 0; i < MLP_H; ++i) acc = fmaf(S.W3[o * MLP_H + i], hin[i], acc);
    acc += S.b3[o];
#pragma unroll
    for (int q = 0; q < MLP_OUT; ++q) z[q] = __shfl(acc, lane0 + q, WAVE);
}

// Master (float32 parameter vector) -> compute copy.
__global__ __launch_bounds__(256) void k_mlp_cast(const float* __restrict__ master, MlpCompute* __restrict__ cw) {
    for (int p = threadIdx.x; p < MLP_NPARAM; p += 256) {
        const float x = master[p];
        if (p < MLP_OFF_B1) cw->W1[p - MLP_OFF_W1] = to_bf16(x);
        else if (p < MLP_OFF_W2) cw->b1[p - MLP_OFF_B1] = x;
        else if (p < MLP_OFF_B2) cw->W2[p - MLP_OFF_W2] = to_bf16(x);
        else if (p < MLP_OFF_W3) cw->b2[p - MLP_OFF_B2] = x;
        else if (p < MLP_OFF_B3) cw->W3[p - MLP_OFF_W3] = to_bf16(x);
        else cw->b3[p - MLP_OFF_B3] = x;
    }
}

constexpr int NET_NT = 256, NET_S = NET_NT / NET_G;   // threads and samples per block round
// Blocks of a forward pass: each loads the network once and takes its samples in rounds (65,536 samples,
// whole call: a block per round 37.0 us, 1024 blocks 34.8, 512 32.7, 256 33.7; a thread per sample 33.5).
constexpr int FWD_BLOCKS = 512;

__global__ __launch_bounds__(NET_NT) void k_mlp_forward(const MlpCompute* __restrict__ cw,
                                                        const float* __restrict__ X, int B,
                                                        float* __restrict__ logits) {
    __shared__ MlpShared S;
    load_net(cw, S);
    const int j = threadIdx.x % NET_G, lane0 = lane_id() - j;
    for (int r = blockIdx.x * NET_S; r < B; r += gridDim.x * NET_S) {
        const int s = r + threadIdx.x / NET_G;
        const int sr = s < B ? s : B - 1;   // groups past the end repeat the last sample: shuffles need whole waves
        float x[MLP_IN], h1[NET_U], h2[NET_U], z[MLP_OUT];
        for (int i = 0; i < MLP_IN; ++i) x[i] = X[sr * MLP_IN + i];
        net_forward(S, x, j, lane0, h1, h2, z);
        if (s < B && j < MLP_OUT) logits[s * MLP_OUT + j] = j == 0 ? z[0] : (j == 1 ? z[1] : z[2]);
    }
}

// Forward, loss and backward of a block's samples, and their sum of parameter
// gradients. Block c takes the samples [c * per, (c + 1) * per) in rounds of
// NET_S; a round's activations and errors go to LDS, and the weight gradients,
// sums over samples of outer products, are accumulated by the matrix cores
// (32x32x2 float32: two samples per instruction) in registers that live
// across the rounds: wave 0 W2 and b2, wave 1 W1 and b1, wave 2 W3 and b3, wave 3 the loss.
// The sums leave as one row of `part` per block, added in order by k_mlp_sum, so
// a training step stays deterministic. Bound: latency (launches and the
// layers' dependent dot products) at the batches training uses; before, one
// thread per parameter walked the whole batch alone. Measured with the
// forward pass and both host calls: 691 samples 343 -> 67 us, 65,536
// samples 32.2 -> 0.14 ms.
typedef float f32x16 __attribute__((ext_vector_type(16)));

__global__ __launch_bounds__(NET_NT) void k_mlp_fwdbwd(const MlpCompute* __restrict__ cw, const float* __restrict__ X,
                                                       const int32_t* __restrict__ y, const float* __restrict__ w,
                                                       int B, int per, float* __restrict__ part) {
    constexpr int LD = MLP_H + 4;   // 16-byte rows for the lanes' four-unit stores
    __shared__ MlpShared S;
    __shared__ __align__(16) float s_h1[NET_S][LD], s_h2[NET_S][LD], s_d1[NET_S][LD], s_d2[NET_S][LD];
    __shared__ float s_x[NET_S][MLP_IN + 2], s_dz[NET_S][MLP_OUT + 1], s_loss[NET_S];
    static_assert(NET_NT / WAVE == 4 && MLP_H == 32 && NET_U == 4, "wave roles, 32x32 tiles");
    load_net(cw, S);
    const int j = threadIdx.x % NET_G, lane0 = lane_id() - j, row = threadIdx.x / NET_G;
    const int wv = wave_id(), col = lane_id() & 31, half = lane_id() >> 5;
    const int s0 = blockIdx.x * per, s1 = s0 + per < B ? s0 + per : B;
    f32x16 acc = {};
    float side = 0.f;   // bias sums (waves 0..2, per lane) or loss terms (wave 3)
    for (int r = s0; r < s1; r += NET_S) {
        const int s = r + row;
        const bool live = s < s1;
        const int sr = live ? s : s1 - 1;
        float x[MLP_IN], h1[NET_U], h2[NET_U], z[MLP_OUT];
        for (int i = 0; i < MLP_IN; ++i) x[i] = X[sr * MLP_IN + i];
        net_forward(S, x, j, lane0, h1, h2, z);
        const float ws = live ? (w ? w[sr] : 1.f) / (float)B : 0.f;
        float zmax = z[0];
        for (int o = 1; o < MLP_OUT; ++o) zmax = fmaxf(zmax, z[o]);
        float e[MLP_OUT], se = 0.f;
        for (int o = 0; o < MLP_OUT; ++o) { e[o] = expf(z[o] - zmax); se += e[o]; }
        const int ys = min(max((int)y[sr], 0), MLP_OUT - 1);   // labels are 0..2; clamp keeps indexing in range
        const float zy = ys == 0 ? z[0] : (ys == 1 ? z[1] : z[2]);
        float dz[MLP_OUT];
        for (int o = 0; o < MLP_OUT; ++o) dz[o] = live ? ws * (e[o] / se - (o == ys ? 1.f : 0.f)) : 0.f;
        float d2[NET_U], d1[NET_U], din[MLP_H];
#pragma unroll
        for (int u = 0; u < NET_U; ++u) {
            float a = 0.f;
            for (int o = 0; o < MLP_OUT; ++o) a = fmaf(S.W3[o * MLP_H + NET_U * j + u], dz[o], a);
            d2[u] = h2[u] > 0.f ? a : 0.f;
        }
        gather_layer(d2, lane0, din);
#pragma unroll
        for (int u = 0; u < NET_U; ++u) {
            float a = 0.f;
#pragma unroll
            for (int q = 0; q < MLP_H; ++q) a = fmaf(S.W2[q * W2_LD + NET_U * j + u], din[q], a);
            d1[u] = h1[u] > 0.f ? a : 0.f;
        }
        const float4 none = make_float4(0.f, 0.f, 0.f, 0.f);   // groups past the end add nothing
        *(float4*)&s_h1[row][NET_U * j] = live ? make_float4(h1[0], h1[1], h1[2], h1[3]) : none;
        *(float4*)&s_h2[row][NET_U * j] = live ? make_float4(h2[0], h2[1], h2[2], h2[3]) : none;
        *(float4*)&s_d1[row][NET_U * j] = live ? make_float4(d1[0], d1[1], d1[2], d1[3]) : none;
        *(float4*)&s_d2[row][NET_U * j] = live ? make_float4(d2[0], d2[1], d2[2], d2[3]) : none;
        if (j < MLP_IN) s_x[row][j] = live ? X[sr * MLP_IN + j] : 0.f;
        if (j < MLP_OUT) s_dz[row][j] = j == 0 ? dz[0] : (j == 1 ? dz[1] : dz[2]);
        if (j == 0) s_loss[row] = live ? ws * (logf(se) + zmax - zy) : 0.f;
        __syncthreads();
        // A: rows = the layer's outputs, B: columns = its inputs; lane l holds row or
        // column l % 32 of sample 2q + l / 32
        if (wv == 3) {
            if (half == 0) side += s_loss[col];
        } else {
#pragma unroll
            for (int q = 0; q < NET_S; q += 2) {
                const int t = q + half;
                float a, b;
                if (wv == 0) { a = s_d2[t][col]; b = s_h1[t][col]; }
                else if (wv == 1) { a = s_d1[t][col]; b = col < MLP_IN ? s_x[t][col] : 0.f; }
                else { a = col < MLP_OUT ? s_dz[t][col] : 0.f; b = s_h2[t][col]; }
                side += a;
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc, 0, 0, 0);
            }
        }
        __syncthreads();
    }
    float* o = part + (size_t)blockIdx.x * (MLP_NPARAM + 1);
    if (wv == 3) {
        side = wave_sum(side);
        if (lane_id() == 0) o[MLP_NPARAM] = side;
        return;
    }
    side += __shfl_xor(side, 32, WAVE);
    const int rows = wv == 2 ? MLP_OUT : MLP_H, cols = wv == 1 ? MLP_IN : MLP_H;
    const int off_w = wv == 0 ? MLP_OFF_W2 : (wv == 1 ? MLP_OFF_W1 : MLP_OFF_W3);
    const int off_b = wv == 0 ? MLP_OFF_B2 : (wv == 1 ? MLP_OFF_B1 : MLP_OFF_B3);
#pragma unroll
    for (int g = 0; g < 16; ++g) {   // result register g: row 8 * (g / 4) + g % 4 + 4 * (lane / 32), column lane % 32
        const int rr = 8 * (g / 4) + g % 4 + 4 * half;
        if (rr < rows && col < cols) o[off_w + rr * cols + col] = acc[g];
    }
    if (half == 0 && col < rows) o[off_b + col] = side;
}

// grad[p] = sum over the nblk rows of part, in a fixed order; the loss is the
// last column. SUM_P parameters by SUM_L row slices per block.
constexpr int SUM_P = 32, SUM_L = 8;
__global__ __launch_bounds__(SUM_P * SUM_L) void k_mlp_sum(const float* __restrict__ part, int nblk,
                                                          float* __restrict__ grad, float* __restrict__ loss) {
    __shared__ float s[SUM_L][SUM_P];
    const int q = threadIdx.x % SUM_P, l = threadIdx.x / SUM_P;
    const int p = blockIdx.x * SUM_P + q;
    float acc = 0.f;
    if (p <= MLP_NPARAM)
        for (int c = l; c < nblk; c += SUM_L) acc += part[(size_t)c * (MLP_NPARAM + 1) + p];
    s[l][q] = acc;
    __syncthreads();
    if (l > 0 || p > MLP_NPARAM) return;
    acc = 0.f;
#pragma unroll
    for (int i = 0; i < SUM_L; ++i) acc += s[i][q];
    if (p == MLP_NPARAM) *loss = acc;
    else grad[p] = acc;
}

// Adam on the float32 master copy (bias-corrected moments).
__global__ __launch_bounds__(256) void k_mlp_adam(float* __restrict__ master, const float* __restrict__ grad,
                                                  float* __restrict__ m, float* __restrict__ v, float lr, float beta1,
                                                  float beta2, float eps, float c1, float c2) {
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= MLP_NPARAM) return;
    const float g = grad[p];
    const float mp = beta1 * m[p] + (1.f - beta1) * g;
    const float vp = beta2 * v[p] + (1.f - beta2) * g * g;
    m[p] = mp;
    v[p] = vp;
    master[p] -= lr * (mp / c1) / (sqrtf(vp / c2) + eps);
}

// One bucket per group of lanes; the logits are those of k_mlp_forward. Argmax
// ties go to the lower index.
__global__ __launch_bounds__(NET_NT) void k_mlp_select(const MlpCompute* __restrict__ cw, Ctrl* ctrl,
                                                       uint8_t* __restrict__ choice) {
    __shared__ MlpShared S;
    load_net(cw, S);
    const int j = threadIdx.x % NET_G, lane0 = lane_id() - j;
    const int b = blockIdx.x * NET_S + threadIdx.x / NET_G;   // NBUCKET groups in all
    float x[MLP_IN], h1[NET_U], h2[NET_U], z[MLP_OUT];
    bucket_features(ctrl, b, x);
    if (j == 0)
        for (int i = 0; i < MLP_IN; ++i) ctrl->features[b][i] = x[i];
    net_forward(S, x, j, lane0, h1, h2, z);
    if (j == 0) {
        int best = 0;
        if (z[1] > z[0]) best = 1;
        if (z[2] > (best ? z[1] : z[0])) best = 2;
        choice[b] = (uint8_t)best;
    }
}

// ------------------------------------------------------------------ launchers
void mlp_cast(const float* master, MlpCompute* cw, hipStream_t s) {
    hipLaunchKernelGGL(k_mlp_cast, dim3(1), dim3(256), 0, s, master, cw);
}
void mlp_forward(const MlpCompute* cw, const float* X, int B, float* logits, hipStream_t s) {
    const int rounds = (B + NET_S - 1) / NET_S;
    if (B > 0)
        hipLaunchKernelGGL(k_mlp_forward, dim3(rounds < FWD_BLOCKS ? rounds : FWD_BLOCKS), dim3(NET_NT), 0, s, cw, X, B,
                           logits);
}
void mlp_gradient(const MlpCompute* cw, const float* X, const int32_t* y, const float* w, int B, float* part,
                  float* grad, float* loss, hipStream_t s) {
    // one round of NET_S samples per block while that needs at most MLP_GRAD_ROWS blocks, more rounds beyond
    const int rounds = (B + NET_S - 1) / NET_S;
    const int per = NET_S * ((rounds + MLP_GRAD_ROWS - 1) / MLP_GRAD_ROWS);
    const int nblk = (B + per - 1) / per;
    hipLaunchKernelGGL(k_mlp_fwdbwd, dim3(nblk), dim3(NET_NT), 0, s, cw, X, y, w, B, per, part);
    hipLaunchKernelGGL(k_mlp_sum, dim3((MLP_NPARAM + 1 + SUM_P - 1) / SUM_P), dim3(SUM_P * SUM_L), 0, s, part, nblk,
                       grad, loss);
}
void mlp_adam(float* master, const float* grad, float* m, float* v, float lr, int step, hipStream_t s) {
    const float beta1 = 0.9f, beta2 = 0.999f, eps = 1e-8f;
    const float c1 = 1.f - powf(beta1, (float)step), c2 = 1.f - powf(beta2, (float)step);
    hipLaunchKernelGGL(k_mlp_adam, dim3((MLP_NPARAM + 255) / 256), dim3(256), 0, s, master, grad, m, v, lr, beta1,
                       beta2, eps, c1, c2);
}
void mlp_select(const MlpCompute* cw, Ctrl* ctrl, uint8_t* choice, hipStream_t s) {
    hipLaunchKernelGGL(k_mlp_select, dim3(NBUCKET / NET_S), dim3(NET_NT), 0, s, cw, ctrl, choice);
}
}  // namespace tcx

// The learned temperature-step model on gfx950: an 8 -> 64 -> 64 -> 1 tanh
// network that proposes ln(dbeta) from population statistics.  Training in
// float32 (forward and backward pass and the gradient of a tile of samples on
// the float32 matrix units, partial gradients per workgroup added in a fixed
// order, then Adam), inference in bfloat16 (weights and layer inputs rounded to bfloat16, float32 sums).
// Parameter vector: W1[64][8], b1[64], W2[64][64], b2[64], W3[64], b3.
#include "pa_device.h"
#include "pa_internal.h"

namespace {

constexpr int kH = PA_MLP_HIDDEN;
constexpr int oW1 = 0, ob1 = oW1 + kH * 8, oW2 = ob1 + kH, ob2 = oW2 + kH * kH, oW3 = ob2 + kH, ob3 = oW3 + kH;
static_assert(ob3 + 1 == PA_MLP_PARAMS, "parameter layout");

// float32 -> nearest bfloat16 (ties to even), kept in a float
__device__ __forceinline__ float bf16r(float x)
{
    uint32_t u = __float_as_uint(x);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return __uint_as_float(u & 0xFFFF0000u);
}

// Training pass over tiles of 16 samples, one workgroup of four waves per tile
// at a time; every layer is a product of float32 16 x 16 x 4 matrix operations
// (A: lane l holds row l % 16 of column l / 16; B: column l % 16 of row l / 16;
// result: lane l, element i is row 4 (l / 16) + i of column l % 16).  Wave v
// owns hidden units 16 v .. 16 v + 15 of both layers: it keeps its rows and
// its columns of W2 in registers for the launch, and its unit's activations
// and error signals are the results of its own products, so only the operands
// of the next product pass through LDS.  The gradient stays in accumulators
// over the workgroup's tiles.
// What bounds it: latency, at the sizes the model is trained on.  A launch per
// pass used to take one sample per thread through global memory, one thread
// per parameter then summed over all samples, and one thread the loss:
// n = 2000 135 + 485 + 81 us per pass, now 9.4 + 7.1.
constexpr int kTileN = 16, kLd = 68; // samples per tile; LDS row stride (16 rows x 4 columns on 64 banks)
constexpr int kMaxParts = 256;       // workgroups, and partial gradients, of a pass at most

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4 mfma(float a, float b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Sum over the 16 lanes of a row in every lane of it (the order is fixed).
__device__ __forceinline__ float row_sum(float v)
{
#pragma unroll
    for (int m = 1; m < 16; m <<= 1)
        v += __shfl_xor(v, m, 64);
    return v;
}

__global__ __launch_bounds__(256) void k_mlp_grad(const float *__restrict__ P, const PaMlpNorm *__restrict__ nm,
                                                  const float *__restrict__ X, const float *__restrict__ Y, int n,
                                                  float *__restrict__ part, double *__restrict__ lpart)
{
    __shared__ float xs[kTileN][kLd];  // standardised inputs, then a column of ones and zeros up to 16
    __shared__ float h1s[kTileN][kLd];
    __shared__ float d1s[kTileN][kLd];
    __shared__ float d2s[kTileN][kLd];
    __shared__ float yp[4][kTileN]; // the waves' parts of the output
    __shared__ float yn[kTileN];
    __shared__ double ls[4];
    const int tid = threadIdx.x, v = tid >> 6, l = tid & 63, c = l & 15, r = l >> 4;
    const int u = 16 * v + c; // this lane's hidden unit
    float w1[2], w2r[16], w2c[16];
#pragma unroll
    for (int k = 0; k < 2; ++k)
        w1[k] = P[oW1 + u * 8 + 4 * k + r];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        w2r[k] = P[oW2 + u * kH + 4 * k + r];   // W2[u][.]: into layer 2
        w2c[k] = P[oW2 + (4 * k + r) * kH + u]; // W2[.][u]: back to layer 1
    }
    const float b1 = P[ob1 + u], b2 = P[ob2 + u], w3 = P[oW3 + u], b3 = P[ob3];
    f32x4 g1 = {0, 0, 0, 0}, g2[4] = {g1, g1, g1, g1}; // dW1 and db1 (column 8), dW2
    float gb2 = 0.0f, gw3 = 0.0f, gb3 = 0.0f;
    double loss = 0.0;
    for (int t0 = blockIdx.x * kTileN; t0 < n; t0 += gridDim.x * kTileN) {
        __syncthreads(); // the previous tile's operands have been read
        {
            const int s = tid >> 4, k = tid & 15, i = t0 + s;
            float x = 0.0f;
            if (i < n && k < 8)
                x = (X[(size_t)i * 8 + k] - nm->x_mean[k]) / nm->x_std[k];
            xs[s][k] = k == 8 ? 1.0f : x;
            if (k == 0)
                yn[s] = i < n ? (Y[i] - nm->y_mean) / nm->y_std : 0.0f;
        }
        __syncthreads();
        f32x4 h1 = {b1, b1, b1, b1};
#pragma unroll
        for (int k = 0; k < 2; ++k)
            h1 = mfma(xs[c][4 * k + r], w1[k], h1);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            h1[i] = tanhf(h1[i]);
            h1s[4 * r + i][u] = h1[i];
        }
        __syncthreads();
        f32x4 h2 = {b2, b2, b2, b2};
#pragma unroll
        for (int k = 0; k < 16; ++k)
            h2 = mfma(h1s[c][4 * k + r], w2r[k], h2);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            h2[i] = tanhf(h2[i]);
            const float y = row_sum(w3 * h2[i]);
            if (c == 0)
                yp[v][4 * r + i] = y;
        }
        __syncthreads();
        f32x4 d2;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int s = 4 * r + i;
            const float yh = ((yp[0][s] + yp[1][s]) + (yp[2][s] + yp[3][s])) + b3;
            const float res = t0 + s < n ? yh - yn[s] : 0.0f; // samples past the end: no error
            const float dy = res / (float)n;
            if (v == 0 && c == 0)
                loss += (double)(res * res);
            d2[i] = dy * w3 * (1.0f - h2[i] * h2[i]);
            d2s[s][u] = d2[i];
            gb2 += d2[i];
            gw3 += dy * h2[i];
            gb3 += dy;
        }
        __syncthreads();
        f32x4 d1 = {0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < 16; ++k)
            d1 = mfma(d2s[c][4 * k + r], w2c[k], d1);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            d1s[4 * r + i][u] = d1[i] * (1.0f - h1[i] * h1[i]);
        // a wave reads back its own columns only: no barrier, but what a lane reads other lanes wrote, and a
        // lane's own addresses alone would let the loads pass the stores
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int s = 4 * k + r;
            const float a = d2s[s][u];
            g1 = mfma(d1s[s][u], xs[s][c], g1);
#pragma unroll
            for (int t = 0; t < 4; ++t)
                g2[t] = mfma(a, h1s[s][16 * t + c], g2[t]);
        }
    }
    // this workgroup's gradient
    float *G = part + (size_t)blockIdx.x * PA_MLP_PARAMS;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int a = 16 * v + 4 * r + i;
        if (c < 8)
            G[oW1 + a * 8 + c] = g1[i];
        if (c == 8)
            G[ob1 + a] = g1[i];
#pragma unroll
        for (int t = 0; t < 4; ++t)
            G[oW2 + a * kH + 16 * t + c] = g2[t][i];
    }
    gb2 += __shfl_xor(gb2, 16, 64);
    gb2 += __shfl_xor(gb2, 32, 64);
    gw3 += __shfl_xor(gw3, 16, 64);
    gw3 += __shfl_xor(gw3, 32, 64);
    gb3 += __shfl_xor(gb3, 16, 64);
    gb3 += __shfl_xor(gb3, 32, 64);
    if (r == 0) {
        G[ob2 + u] = gb2;
        G[oW3 + u] = gw3;
    }
    if (tid == 0)
        G[ob3] = gb3;
    if (v == 0 && c == 0)
        ls[r] = loss;
    __syncthreads();
    if (tid == 0)
        lpart[blockIdx.x] = (ls[0] + ls[1]) + (ls[2] + ls[3]);
}

// Adds the partial gradients (a thread every fourth of them, then the four in
// order; the last workgroup adds the loss), then (adam != 0) one Adam step, t
// counting from 1.
constexpr int kUpdParams = 64; // parameters per workgroup

__global__ __launch_bounds__(4 * kUpdParams) void k_mlp_update(float *__restrict__ P, float *__restrict__ Mm,
                                                               float *__restrict__ Vv, float *__restrict__ G,
                                                               const float *__restrict__ part,
                                                               const double *__restrict__ lpart, int nparts, int n,
                                                               double *__restrict__ loss, int adam, int t, float lr)
{
    __shared__ float sg[4][kUpdParams];
    const int j = threadIdx.x & (kUpdParams - 1), q = threadIdx.x / kUpdParams;
    if (blockIdx.x == gridDim.x - 1) {
        if (threadIdx.x < 64) {
            double s = 0.0;
            for (int k = threadIdx.x; k < nparts; k += 64)
                s += lpart[k];
            s = pa_wave_sum_f64(s);
            if (threadIdx.x == 0)
                *loss = 0.5 * s / (double)n;
        }
        return;
    }
    const int p = blockIdx.x * kUpdParams + j;
    float g = 0.0f;
    if (p < PA_MLP_PARAMS) {
        int k = q;
        for (; k + 28 < nparts; k += 32) { // eight loads in flight
            float x[8];
#pragma unroll
            for (int i = 0; i < 8; ++i)
                x[i] = part[(size_t)(k + 4 * i) * PA_MLP_PARAMS + p];
#pragma unroll
            for (int i = 0; i < 8; ++i)
                g += x[i];
        }
        for (; k < nparts; k += 4)
            g += part[(size_t)k * PA_MLP_PARAMS + p];
    }
    sg[q][j] = g;
    __syncthreads();
    if (q != 0 || p >= PA_MLP_PARAMS)
        return;
    g = (sg[0][j] + sg[1][j]) + (sg[2][j] + sg[3][j]);
    G[p] = g;
    if (adam) {
        const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
        const float m = b1 * Mm[p] + (1.0f - b1) * g;
        const float v = b2 * Vv[p] + (1.0f - b2) * g * g;
        Mm[p] = m;
        Vv[p] = v;
        const float mh = m / (1.0f - powf(b1, (float)t));
        const float vh = v / (1.0f - powf(b2, (float)t));
        P[p] = P[p] - lr * mh / (sqrtf(vh) + eps);
    }
}

// bfloat16 inference of one feature vector by one wave: lane a owns hidden
// unit a of both layers; the output sum runs over a in order on lane 0.
__device__ float mlp_infer_wave(const float *__restrict__ P, const PaMlpNorm *__restrict__ nm, const float *f,
                                float *h1s, float *h2s)
{
    const int a = threadIdx.x & 63;
    float x[8];
    for (int k = 0; k < 8; ++k)
        x[k] = bf16r((f[k] - nm->x_mean[k]) / nm->x_std[k]);
    float z = bf16r(P[ob1 + a]);
    for (int k = 0; k < 8; ++k)
        z += bf16r(P[oW1 + a * 8 + k]) * x[k];
    h1s[a] = bf16r(tanhf(z));
    __syncthreads();
    z = bf16r(P[ob2 + a]);
    for (int b = 0; b < kH; ++b)
        z += bf16r(P[oW2 + a * kH + b]) * h1s[b];
    h2s[a] = bf16r(tanhf(z));
    __syncthreads();
    float y = bf16r(P[ob3]);
    for (int b = 0; b < kH; ++b)
        y += bf16r(P[oW3 + b]) * h2s[b];
    return y;
}

__device__ __forceinline__ double to_dbeta(float yhat, const PaMlpNorm *nm) { return exp((double)yhat * nm->y_std + nm->y_mean); }

// Standalone inference: one 64-lane workgroup per feature vector.
__global__ __launch_bounds__(64) void k_mlp_predict(const float *__restrict__ P, const PaMlpNorm *__restrict__ nm,
                                                   const float *__restrict__ X, int n, float *__restrict__ out)
{
    __shared__ float h1s[kH], h2s[kH];
    const int i = blockIdx.x;
    if (i >= n)
        return;
    const float y = mlp_infer_wave(P, nm, X + (size_t)i * 8, h1s, h2s);
    if (threadIdx.x == 0)
        out[i] = (float)to_dbeta(y, nm);
}

// Inference for every run of a batch from the features in its record; the
// proposal is clamped to (0, dbeta_max] and stored for the exact check.
__global__ __launch_bounds__(64) void k_mlp_propose(const PaRunDesc *__restrict__ runs, const float *__restrict__ P,
                                                   const PaMlpNorm *__restrict__ nm, double dbeta_max)
{
    __shared__ float h1s[kH], h2s[kH];
    PaRecord *rec = runs[blockIdx.x].dv.rec;
    if (rec->status & PA_ST_FROZEN)
        return;
    float f[8];
    for (int k = 0; k < 8; ++k)
        f[k] = rec->feat[k];
    const float y = mlp_infer_wave(P, nm, f, h1s, h2s);
    if (threadIdx.x == 0) {
        double d = to_dbeta(y, nm);
        if (!(d > 0.0))
            d = 0.0;
        rec->cand_dbeta = d < dbeta_max ? d : dbeta_max;
    }
}

} // namespace

int pa_mlp_parts(int n)
{
    const int tiles = (int)(((int64_t)n + kTileN - 1) / kTileN);
    return tiles < kMaxParts ? tiles : kMaxParts;
}

hipError_t pa_mlp_launch_grad(const PaMlpDev &m, int n, int adam, int t, float lr)
{
    const int parts = pa_mlp_parts(n);
    k_mlp_grad<<<parts, 256, 0, m.stream>>>(m.P, m.norm, m.X, m.Y, n, m.part, m.lpart);
    k_mlp_update<<<(PA_MLP_PARAMS + kUpdParams - 1) / kUpdParams + 1, 4 * kUpdParams, 0, m.stream>>>(
        m.P, m.M, m.V, m.G, m.part, m.lpart, parts, n, m.loss, adam, t, lr);
    return hipGetLastError();
}

hipError_t pa_mlp_launch_predict(const PaMlpDev &m, const float *X, int n, float *out)
{
    k_mlp_predict<<<n, 64, 0, m.stream>>>(m.P, m.norm, X, n, out);
    return hipGetLastError();
}

hipError_t pa_mlp_launch_propose(const PaBatchView &v, const PaMlpDev &m, double dbeta_max)
{
    k_mlp_propose<<<v.nruns, 64, 0, v.stream>>>(v.runs, m.P, m.norm, dbeta_max);
    return hipGetLastError();
}

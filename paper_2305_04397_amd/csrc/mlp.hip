// Learned weight proposer: a small MLP that maps a threshold point and
// instance features [t; phi] to a weight vector on the simplex, used as the
// first weight vector of a query in place of e_1 (Alg. 1).  It is not part of
// the paper; the plain loop still decides every answer.
//
// Network: input standardisation (x - mu) / sd (fixed, set by the caller),
// then n_in -> 256 -> 256 -> 256 -> d, ReLU, softmax output; loss is the
// cross-entropy between a target weight vector and the softmax, averaged over
// the batch; optimiser Adam with bias correction.
//
// Precision: BF16 weights, inputs, activations and back-propagated gradients,
// FP32 accumulation on the matrix cores (v_mfma_f32_16x16x32_bf16), FP32
// biases, logits, softmax, weight gradients and Adam state, FP32 master
// weights (the BF16 copies are refreshed by every Adam step).
//
// Kernels, for networks of up to 1024 inputs and 512 outputs:
//   * mlp_rows: everything that is local to a row, 16 rows per workgroup: the
//     four layers, softmax, and for training the loss, the output gradient and
//     its way back to the first layer, with the activations in LDS and the
//     weights read from L2 in the order the matrix instruction takes them;
//   * weight_grads: the weight and bias gradients of all layers in one launch;
//   * adam: the update of every parameter and its BF16 copies.
// Kernels of larger networks, layer by layer:
//   * gemm_bf16: C[M][N] = sum_k A(m, k) B(k, n) for strided BF16 operands,
//     one wave per 16 x 64 output strip (4 MFMA accumulators), with the
//     epilogue of the layer: +bias and ReLU to BF16 (hidden forward), +bias to
//     FP32 (logits), ReLU-derivative mask to BF16 (backward data), FP32 store
//     (weight gradients);
//   * softmax_xent: per row softmax, cross-entropy and (P - T) / B;
//   * bias_grad: column sums of a BF16 gradient.
#include "common.h"

#include <exception>
#include <mutex>

#include <cmath>
#include <cstdio>
#include <numeric>

namespace morap {

namespace {

typedef short s16x8 __attribute__((ext_vector_type(8)));          // BF16 bits
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int HID = 256;
constexpr int NLAYER = 4;

__host__ __device__ inline uint16_t f2bf(float f) {
    uint32_t u;
    memcpy(&u, &f, 4);
    u += 0x7FFFu + ((u >> 16) & 1u);   // round to nearest, ties to even (finite inputs)
    return (uint16_t)(u >> 16);
}

__host__ __device__ inline float bf2f(uint16_t h) {
    const uint32_t u = (uint32_t)h << 16;
    float f;
    memcpy(&f, &u, 4);
    return f;
}

enum Epilogue { EP_HIDDEN = 0, EP_LOGITS = 1, EP_BWD_DATA = 2, EP_WGRAD = 3 };

struct GemmArgs {
    const uint16_t* A;
    int64_t sam, sak;        // A(m, k) = A[m * sam + k * sak]
    const uint16_t* B;
    int64_t sbk, sbn;        // B(k, n) = B[k * sbk + n * sbn]
    int M, N, K;
    int mode;
    float* Cf;               // FP32 output (logits, weight gradients)
    uint16_t* Cb;            // BF16 output (activations, gradients)
    int64_t ldc;
    const float* bias;       // [N] (forward)
    const uint16_t* mask;    // ReLU-derivative source (backward data)
    int64_t ldm;
};

__global__ void __launch_bounds__(256) gemm_bf16(GemmArgs g) {
    const int lane = threadIdx.x & 63;
    const int wave = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int tiles_n = (g.N + 63) / 64;
    const int tm = wave / tiles_n, tn = wave - tm * tiles_n;
    if (tm * 16 >= g.M) return;
    // operand layout of gfx950's 16x16x32 BF16 MFMA: lane l holds
    // A[l % 16][8 (l / 16) + e] and B[8 (l / 16) + e][l % 16] for e = 0..7;
    // the result D[4 (l / 16) + e][l % 16] for e = 0..3
    const int r = lane & 15, kg = lane >> 4;
    const int m = tm * 16 + r;
    f32x4 acc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < g.K; k0 += 32) {
        s16x8 a;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int k = k0 + 8 * kg + e;
            a[e] = (m < g.M && k < g.K) ? (short)g.A[m * g.sam + k * g.sak] : (short)0;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int n = tn * 64 + j * 16 + r;
            s16x8 b;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int k = k0 + 8 * kg + e;
                b[e] = (n < g.N && k < g.K) ? (short)g.B[k * g.sbk + n * g.sbn] : (short)0;
            }
            acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                             __builtin_bit_cast(bf16x8, b), acc[j], 0, 0, 0);
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int n = tn * 64 + j * 16 + r;
        if (n >= g.N) continue;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int mm = tm * 16 + 4 * kg + e;
            if (mm >= g.M) continue;
            const float v = acc[j][e];
            const int64_t o = (int64_t)mm * g.ldc + n;
            switch (g.mode) {
                case EP_HIDDEN: g.Cb[o] = f2bf(fmaxf(v + g.bias[n], 0.f)); break;
                case EP_LOGITS: g.Cf[o] = v + g.bias[n]; break;
                case EP_BWD_DATA:
                    g.Cb[o] = f2bf(bf2f(g.mask[(int64_t)mm * g.ldm + n]) > 0.f ? v : 0.f);
                    break;
                default: g.Cf[o] = v; break;
            }
        }
    }
}

void gemm(hipStream_t s, const GemmArgs& g) {
    const int64_t waves = (int64_t)((g.M + 15) / 16) * ((g.N + 63) / 64);
    if (waves <= 0) return;
    hipLaunchKernelGGL(gemm_bf16, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, s, g);
    MORAP_HIP(hipGetLastError());
}

// per row: P = softmax(z), loss = -sum_k T_k log P_k, G = (P - T) / B (BF16)
__global__ void softmax_xent(const float* z, const float* T, float* P, uint16_t* G, float* loss, int n, int d,
                             float inv_b) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float* zi = z + (int64_t)i * d;
    float mx = -INFINITY;
    for (int k = 0; k < d; ++k) mx = fmaxf(mx, zi[k]);
    float sum = 0.f;
    for (int k = 0; k < d; ++k) sum += expf(zi[k] - mx);
    const float lse = logf(sum);
    float l = 0.f;
    for (int k = 0; k < d; ++k) {
        const float p = expf(zi[k] - mx) / sum;
        P[(int64_t)i * d + k] = p;
        if (T) {
            const float t = T[(int64_t)i * d + k];
            if (t != 0.f) l -= t * (zi[k] - mx - lse);
            G[(int64_t)i * d + k] = f2bf((p - t) * inv_b);
        }
    }
    if (loss) loss[i] = l;
}

// db[c] = sum_r G[r][c]
__global__ void bias_grad(const uint16_t* G, float* db, int n, int cols) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= cols) return;
    float s = 0.f;
    for (int r = 0; r < n; ++r) s += bf2f(G[(int64_t)r * cols + c]);
    db[c] = s;
}

// network input: (x - mu) / sd per column, rounded to BF16
__global__ void input_kernel(const float* x, const float* mu, const float* sd, uint16_t* out, int64_t n,
                             int cols) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int c = (int)(i % cols);
    out[i] = f2bf((x[i] - mu[c]) / sd[c]);
}

// Places of a weight in the BF16 copies the matrix instructions read: a
// fragment is 16 outputs x 32 inputs as lane (l % 16, l / 16) holds it, 8
// consecutive inputs of one output, fragments of an output tile in input
// order (forward); the backward copy is the same of the transposed matrix.
struct Packed {
    uint16_t *fwd[NLAYER], *bwd[NLAYER];   // bwd[0] unused
    int ks_f[NLAYER], ks_b[NLAYER];        // 32-deep steps
    int fan_in[NLAYER];
    int64_t w_off[NLAYER], b_off[NLAYER];
};
__device__ __forceinline__ int64_t frag_at(int out, int in, int ks) {
    return (((int64_t)(out >> 4) * ks + (in >> 5)) * 64 + ((in & 31) >> 3) * 16 + (out & 15)) * 8 + (in & 7);
}
__device__ __forceinline__ void store_copies(const Packed& k, uint16_t* pb, int64_t i, float v) {
#pragma unroll
    for (int l = 0; l < NLAYER; ++l) {
        if (i < k.w_off[l] || i >= k.b_off[l]) continue;
        const uint16_t h = f2bf(v);
        if (pb) {
            pb[i] = h;
            return;
        }
        const int e = (int)(i - k.w_off[l]), out = e / k.fan_in[l], in = e - out * k.fan_in[l];
        k.fwd[l][frag_at(out, in, k.ks_f[l])] = h;
        if (l > 0) k.bwd[l][frag_at(in, out, k.ks_b[l])] = h;
    }
}

__global__ void copy_kernel(const float* from, float* to, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) to[i] = from[i];
}

// BF16 copies of the FP32 parameters: row-major (pb, larger networks) or packed
__global__ void copies_kernel(const float* p, uint16_t* pb, Packed k, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) store_copies(k, pb, i, p[i]);
}

// Adam with bias correction (c1 = 1 - beta1^t, c2 = 1 - beta2^t); weights
// refresh their BF16 copies
__global__ void adam_kernel(float* p, const float* g, float* m, float* v, uint16_t* pb, Packed k, int64_t n, float lr,
                            float b1, float b2, float eps, float c1, float c2) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float pi = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    p[i] = pi;
    store_copies(k, pb, i, pi);
}

// ---------------------------------------------------------------------------
// the fused kernels
// ---------------------------------------------------------------------------
// The largest network: at both limits a training workgroup holds 158 of the
// CU's 160 KB of LDS.  A step of 4,096 host rows there takes 1.44 ms (64 rows:
// 0.29 ms); one input more, layer by layer, 6.5 ms (0.98 ms).
constexpr int FUSED_IN = 1024, FUSED_OUT = 512;
constexpr int ROWS = 16;                          // rows of a workgroup
constexpr int LDH = HID + 8;                      // LDS row of a hidden layer (8: banks)
constexpr int KSH = HID / 32;

struct RowArgs {
    const float *x, *mu, *sd, *T;
    const uint16_t* fwd[NLAYER];
    const uint16_t* bwd[NLAYER];
    const float* bias[NLAYER];
    float *prob, *loss;
    // training: transposed copies [features][ld] of the input, the hidden
    // activations and the gradients of the layers' outputs; rows past n are 0
    uint16_t *xt, *ht[NLAYER - 1], *gt[NLAYER];
    int n, n_in, d, ld;
    float inv_b;
};

__host__ __device__ constexpr int up(int v, int to) { return (v + to - 1) / to * to; }
// LDS of a workgroup, in bytes: input, three hidden layers, logits; training:
// targets, output gradient, two hidden gradients
__host__ __device__ inline int rows_ldx(int n_in) { return up(n_in, 32) + 8; }
__host__ __device__ inline int rows_ldz(int d) { return up(d, 16) + 4; }
__host__ __device__ inline int rows_ldg(int d) { return up(d, 32) + 8; }
inline size_t rows_lds(int n_in, int d, bool train) {
    return (size_t)ROWS * (rows_ldx(n_in) * 2 + (NLAYER - 1) * LDH * 2 + rows_ldz(d) * 4 +
                           (train ? rows_ldz(d) * 4 + rows_ldg(d) * 2 + 2 * LDH * 2 : 0));
}

__device__ __forceinline__ s16x8 frag(const uint16_t* w, int64_t at, int lane) {
    return *reinterpret_cast<const s16x8*>(w + (at * 64 + lane) * 8);
}
__device__ __forceinline__ f32x4 mfma(const s16x8& a, const s16x8& b, const f32x4& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// 16 rows, one 16-wide output tile per wave and layer.  The rows are few and
// the weights (0.3-0.4 MB) are read from L2 by every workgroup, so what bounds
// it is the latency of a layer's loads: each wave has the next layer's
// fragments on their way before the barrier that ends a layer.  Products are
// accumulated over the inputs in ascending steps of 32.  4,000 rows of
// 182 -> 150: 13.5 us; 4,096 training rows of 62 -> 30: 22 us.  (Layer by
// layer, with the activations in memory, a pass of 64 rows of 62 -> 30 took
// 42.7 us and takes 4.3.)
template <bool TRAIN>
__global__ void __launch_bounds__(1024) mlp_rows(RowArgs a) {
    extern __shared__ __align__(16) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, kg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row0 = blockIdx.x * ROWS;
    const int ldx = rows_ldx(a.n_in), ldz = rows_ldz(a.d), ldg = rows_ldg(a.d);
    uint16_t* xs = reinterpret_cast<uint16_t*>(lds);
    uint16_t* h = xs + ROWS * ldx;                                   // [3][ROWS][LDH]
    float* z = reinterpret_cast<float*>(h + (NLAYER - 1) * ROWS * LDH);
    float* tt = z + ROWS * ldz;
    uint16_t* go = reinterpret_cast<uint16_t*>(tt + ROWS * ldz);     // [ROWS][ldg]
    uint16_t* gh = go + ROWS * ldg;                                  // [2][ROWS][LDH]

    s16x8 w[KSH];
    auto ahead = [&](const uint16_t* W, int tile) {   // a 256-input layer's fragments of one tile
#pragma unroll
        for (int s = 0; s < KSH; ++s) w[s] = frag(W, (int64_t)tile * KSH + s, lane);
    };
    auto product = [&](const uint16_t* in) {          // 16 x 256 in LDS times w
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KSH; ++s)
            acc = mfma(*reinterpret_cast<const s16x8*>(in + r * LDH + s * 32 + 8 * kg), w[s], acc);
        return acc;
    };
    // result lanes: rows 4 kg .. + 3 of column c; transposed: one 8-byte store
    auto put = [&](uint16_t* out, uint16_t* t, int c, const float (&v)[4]) {
        ushort4 q;
        uint16_t* e = reinterpret_cast<uint16_t*>(&q);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint16_t b = f2bf(v[i]);
            out[(4 * kg + i) * LDH + c] = b;
            e[i] = row0 + 4 * kg + i < a.n ? b : (uint16_t)0;
        }
        if (TRAIN) *reinterpret_cast<ushort4*>(t + (int64_t)c * a.ld + row0 + 4 * kg) = q;
    };

    ahead(a.fwd[1], wave);
    // input: (x - mu) / sd per column, rounded to BF16; 0 in the padding
    for (int i = tid; i < ROWS * up(a.n_in, 32); i += 1024) {
        const int q = i / up(a.n_in, 32), c = i - q * up(a.n_in, 32);
        const bool in = c < a.n_in && row0 + q < a.n;
        xs[q * ldx + c] = in ? f2bf((a.x[(int64_t)(row0 + q) * a.n_in + c] - a.mu[c]) / a.sd[c]) : (uint16_t)0;
    }
    if (TRAIN) {
        for (int i = tid; i < ROWS * a.d; i += 1024) {
            const int q = i / a.d, c = i - q * a.d;
            tt[q * ldz + c] = row0 + q < a.n ? a.T[(int64_t)(row0 + q) * a.d + c] : 0.f;
        }
        for (int i = tid; i < ROWS * ldg; i += 1024) go[i] = 0;   // the padding
    }
    __syncthreads();
    if (TRAIN)
        for (int c = tid; c < a.n_in; c += 1024) {
            __align__(16) uint16_t v[ROWS];
#pragma unroll
            for (int q = 0; q < ROWS; ++q) v[q] = xs[q * ldx + c];
            uint4* o = reinterpret_cast<uint4*>(a.xt + (int64_t)c * a.ld + row0);
            o[0] = reinterpret_cast<const uint4*>(v)[0];
            o[1] = reinterpret_cast<const uint4*>(v)[1];
        }
    auto hidden = [&](const f32x4& acc, int l) {
        const int c = wave * 16 + r;
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = fmaxf(acc[i] + a.bias[l][c], 0.f);
        put(h + l * ROWS * LDH, TRAIN ? a.ht[l] : nullptr, c, v);
    };
    {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        const int ks = up(a.n_in, 32) / 32;
#pragma unroll 4
        for (int s = 0; s < ks; ++s)
            acc = mfma(*reinterpret_cast<const s16x8*>(xs + r * ldx + s * 32 + 8 * kg),
                       frag(a.fwd[0], (int64_t)wave * ks + s, lane), acc);
        hidden(acc, 0);
    }
    __syncthreads();
    {
        const f32x4 acc = product(h);
        ahead(a.fwd[2], wave);
        hidden(acc, 1);
    }
    __syncthreads();
    const int tiles = up(a.d, 16) / 16;
    {
        const f32x4 acc = product(h + ROWS * LDH);
        if (wave < tiles) ahead(a.fwd[3], wave);
        hidden(acc, 2);
    }
    __syncthreads();
    for (int t = wave; t < tiles; t += 16) {
        if (t != wave) ahead(a.fwd[3], t);
        const f32x4 acc = product(h + 2 * ROWS * LDH);
        const int c = t * 16 + r;
        if (c < a.d)
#pragma unroll
            for (int i = 0; i < 4; ++i) z[(4 * kg + i) * ldz + c] = acc[i] + a.bias[3][c];
    }
    __syncthreads();

    // softmax, one row per wave: sums in column order, as one thread adds them
    {
        const int row = row0 + wave;
        float* zr = z + wave * ldz;
        float mx = -INFINITY;
        for (int c = lane; c < a.d; c += 64) mx = fmaxf(mx, zr[c]);
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
        float zc[FUSED_OUT / 64], ec[FUSED_OUT / 64];
#pragma unroll
        for (int j = 0; j < FUSED_OUT / 64; ++j) {
            const int c = j * 64 + lane;
            zc[j] = ec[j] = 0.f;
            if (j * 64 >= a.d) continue;
            if (c < a.d) {
                zc[j] = zr[c];
                ec[j] = expf(zc[j] - mx);
                zr[c] = ec[j];
            }
        }
        float sum = 0.f;
        int c = 0;
        for (; c + 4 <= a.d; c += 4) {
            const float4 v = *reinterpret_cast<const float4*>(zr + c);
            sum += v.x;
            sum += v.y;
            sum += v.z;
            sum += v.w;
        }
        for (; c < a.d; ++c) sum += zr[c];
        const float lse = logf(sum);
        const float* tr = tt + wave * ldz;
#pragma unroll
        for (int j = 0; j < FUSED_OUT / 64; ++j) {
            const int k = j * 64 + lane;
            if (j * 64 >= a.d) continue;
            if (k < a.d && row < a.n) {
                const float p = ec[j] / sum;
                a.prob[(int64_t)row * a.d + k] = p;
                if (TRAIN) {
                    const float t = tr[k];
                    go[wave * ldg + k] = f2bf((p - t) * a.inv_b);
                    zr[k] = zc[j] - mx - lse;
                }
            }
        }
        if (TRAIN && row < a.n) {
            float l = 0.f;
            for (int k = 0; k < a.d; ++k) {
                const float t = tr[k], v = zr[k];
                if (t != 0.f) l -= t * v;
            }
            if (lane == 0) a.loss[row] = l;
        }
    }
    if (!TRAIN) return;
    // the output gradient back through the layers
    ahead(a.bwd[2], wave);   // (layer 2's; layer 3's input is the d outputs)
    __syncthreads();
    for (int c = tid; c < a.d; c += 1024) {
        __align__(16) uint16_t v[ROWS];
#pragma unroll
        for (int q = 0; q < ROWS; ++q) v[q] = go[q * ldg + c];
        uint4* o = reinterpret_cast<uint4*>(a.gt[3] + (int64_t)c * a.ld + row0);
        o[0] = reinterpret_cast<const uint4*>(v)[0];
        o[1] = reinterpret_cast<const uint4*>(v)[1];
    }
    // gradient of layer l's output, masked by its activation
    auto masked = [&](const f32x4& acc, int l, uint16_t* out) {
        const int c = wave * 16 + r;
        const uint16_t* hl = h + l * ROWS * LDH;
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = bf2f(hl[(4 * kg + i) * LDH + c]) > 0.f ? acc[i] : 0.f;
        put(out, a.gt[l], c, v);
    };
    {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        const int ks = up(a.d, 32) / 32;
#pragma unroll 4
        for (int s = 0; s < ks; ++s)
            acc = mfma(*reinterpret_cast<const s16x8*>(go + r * ldg + s * 32 + 8 * kg),
                       frag(a.bwd[3], (int64_t)wave * ks + s, lane), acc);
        masked(acc, 2, gh);
    }
    __syncthreads();
    {
        const f32x4 acc = product(gh);
        ahead(a.bwd[1], wave);
        masked(acc, 1, gh + ROWS * LDH);
    }
    __syncthreads();
    masked(product(gh + ROWS * LDH), 0, gh);
}

// Weight gradients dW[N][K] = sum over the rows of G[r][N] H[r][K], and bias
// gradients sum over the rows of G, of all layers in one launch: a workgroup
// per 32 x 32 tile, its 16 waves taking every 16th step of 32 rows and adding
// up in a fixed order.  The outputs are few (170 tiles at 62 -> 30) and the
// rows many, so the split over rows is what gives the loads company: 18.6 us
// at 4,096 rows, the transposed copies making every fragment one 16-byte load
// (a step with gradients took 4.32 ms with one workgroup per tile and strided
// operands, and takes 0.17).  16 short sums also err less than one long one:
// 3e-8 against 3e-7 at most, on sums of up to 0.6.
struct GradLayer {
    const uint16_t *g, *h;   // [N][ld], [K][ld]
    float *dw, *db;
    int N, K, first;         // first workgroup
};
struct GradArgs {
    GradLayer l[NLAYER];
    int ld;
};
__global__ void __launch_bounds__(1024) weight_grads(GradArgs a) {
    __shared__ f32x4 red[8][6][64];
    int q = 0;
#pragma unroll
    for (int l = 1; l < NLAYER; ++l)
        if ((int)blockIdx.x >= a.l[l].first) q = l;
    const GradLayer L = a.l[q];
    const int tiles_k = (L.K + 31) / 32, b = (int)blockIdx.x - L.first;
    const int n0 = b / tiles_k * 32, k0 = b % tiles_k * 32;
    const int lane = threadIdx.x & 63, r = lane & 15, kg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool bias = k0 == 0;
    const uint16_t* gp[2];
    const uint16_t* hp[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {   // (rows past the last repeat it; not stored)
        gp[i] = L.g + (int64_t)min(n0 + 16 * i + r, L.N - 1) * a.ld + 8 * kg;
        hp[i] = L.h + (int64_t)min(k0 + 16 * i + r, L.K - 1) * a.ld + 8 * kg;
    }
    s16x8 ones;
#pragma unroll
    for (int i = 0; i < 8; ++i) ones[i] = (short)0x3F80;
    f32x4 acc[6] = {};   // [2 x 2] tiles, then the bias of both
    for (int s = wave; s < a.ld / 32; s += 16) {
        s16x8 g[2], h[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            g[i] = *reinterpret_cast<const s16x8*>(gp[i] + s * 32);
            h[i] = *reinterpret_cast<const s16x8*>(hp[i] + s * 32);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[2 * i + j] = mfma(g[i], h[j], acc[2 * i + j]);
            if (bias) acc[4 + i] = mfma(g[i], ones, acc[4 + i]);
        }
    }
    for (int half = 8; half >= 1; half >>= 1) {
        if (wave >= half && wave < 2 * half)
#pragma unroll
            for (int t = 0; t < 6; ++t) red[wave - half][t][lane] = acc[t];
        __syncthreads();
        if (wave < half)
#pragma unroll
            for (int t = 0; t < 6; ++t) acc[t] += red[wave][t][lane];
        __syncthreads();
    }
    if (wave != 0) return;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int n = n0 + 16 * i + 4 * kg + e;
            if (n >= L.N) continue;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int k = k0 + 16 * j + r;
                if (k < L.K) L.dw[(int64_t)n * L.K + k] = acc[2 * i + j][e];
            }
            if (bias && r == 0) L.db[n] = acc[4 + i][e];
        }
}

unsigned blocks_for(int64_t n, int per = 256) { return (unsigned)((n + per - 1) / per); }

uint64_t splitmix64(uint64_t x) {
    x += 0x9E3779B97F4A7C15ull;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}

}  // namespace

// Host arrays travel through a ring of pinned slots, checked or copied while the
// slots before are on their way.  The ring is kept, so it is small: the first use
// of fresh pinned memory costs 0.35 ms a megabyte (inference of 5,000 rows of
// 1,024 -> 512 with all rows in pinned memory of their own: 12.9 ms the first time,
// 1.2 later).
class Ring {
public:
    static constexpr int SLOTS = 4;
    static constexpr size_t FLOATS = (size_t)1 << 18;   // a slot's
    Ring() = default;
    Ring(const Ring&) = delete;
    Ring& operator=(const Ring&) = delete;
    ~Ring() {
        for (hipEvent_t e : done_)
            if (e) (void)hipEventDestroy(e);
    }
    // a call that takes that many slots (nothing of an earlier one is on its way);
    // one that takes each at most once waits for the stream, not for events of its
    // own (a step of 4,096 rows of 62 -> 30: 168 us, 213 with them)
    void start(hipStream_t s, size_t uses) {
        mem_.ensure(SLOTS * FLOATS * 4);
        for (Slot& q : slot_) q = Slot();
        at_ = 0;
        s_ = s;
        events_ = uses > SLOTS;
    }
    static size_t slots(size_t count) { return (count + FLOATS - 1) / FLOATS; }
    // the next slot, free again
    float* next() {
        wait(at_);
        return mem_.as<float>() + (size_t)at_ * FLOATS;
    }
    // that slot is in use until what the stream holds now has run; then the first
    // `count` of its floats belong at `to` (or nowhere)
    void used(float* to = nullptr, size_t count = 0) {
        if (events_) {
            if (!done_[at_]) MORAP_HIP(hipEventCreateWithFlags(&done_[at_], hipEventDisableTiming));
            MORAP_HIP(hipEventRecord(done_[at_], s_));
        }
        slot_[at_] = Slot{true, to, count};
        at_ = (at_ + 1) % SLOTS;
    }
    // all slots, oldest first
    void finish() {
        for (int q = 0; q < SLOTS; ++q) wait((at_ + q) % SLOTS);
    }
    void wait(int q) {
        if (!slot_[q].busy) return;
        MORAP_HIP(events_ ? hipEventSynchronize(done_[q]) : hipStreamSynchronize(s_));
        if (slot_[q].to) std::memcpy(slot_[q].to, mem_.as<float>() + (size_t)q * FLOATS, slot_[q].count * 4);
        slot_[q].busy = false;
    }

private:
    struct Slot {
        bool busy = false;
        float* to = nullptr;
        size_t count = 0;
    };
    PinnedBuf mem_;
    hipEvent_t done_[SLOTS] = {};
    Slot slot_[SLOTS];
    int at_ = 0;
    hipStream_t s_ = nullptr;
    bool events_ = false;
};

// Left by an error: waits for the stream, where a copy may still read the
// caller's rows or the pinned ones that the next call writes.
struct Drain {
    hipStream_t s;
    int before = std::uncaught_exceptions();
    explicit Drain(hipStream_t s_) : s(s_) {}
    ~Drain() {
        if (std::uncaught_exceptions() > before) (void)hipStreamSynchronize(s);
    }
};

// infinite or NaN among X[0 .. count), which is copied to `to` (or not: null)
static bool nonfinite(const float* __restrict X, float* __restrict to, size_t count) {
    uint32_t bad = 0;
    auto one = [&](size_t i) {
        uint32_t u;
        std::memcpy(&u, X + i, 4);
        bad |= (u & 0x7F800000u) == 0x7F800000u ? 1u : 0u;
    };
    if (!to)
        for (size_t i = 0; i < count; ++i) one(i);
    else
        for (size_t i = 0; i < count; ++i) {
            one(i);
            to[i] = X[i];
        }
    return bad != 0;
}
// Rows of T are >= 0 and sum to 1 (added in column order, four rows at a time
// for the adds' latency).
static void check_targets(const float* T, int n, int d) {
    bool sums = true;
    for (int r = 0; r < n; r += 4) {
        const float* t[4];
        for (int q = 0; q < 4; ++q) t[q] = T + (size_t)std::min(r + q, n - 1) * d;
        double sum[4] = {0, 0, 0, 0};
        bool ok = true;
        for (int k = 0; k < d; ++k)
            for (int q = 0; q < 4; ++q) {
                ok &= t[q][k] >= 0.f && t[q][k] <= std::numeric_limits<float>::max();
                sum[q] += t[q][k];
            }
        MORAP_CHECK(ok, MORAP_E_INVALID, "targets must be finite and >= 0");
        for (int q = 0; q < 4; ++q) sums &= std::fabs(sum[q] - 1.0) <= 1e-4;
        MORAP_CHECK(sums, MORAP_E_INVALID, "target rows must sum to 1");
    }
}
static void check_rows(const float* X, const float* T, int n, int n_in, int d) {
    MORAP_CHECK(X && n >= 1, MORAP_E_INVALID, "need X and n >= 1");
    MORAP_CHECK(!nonfinite(X, nullptr, (size_t)n * n_in), MORAP_E_INVALID, "X must be finite");
    if (T) check_targets(T, n, d);
}

struct Proposer {
    int n_in = 0, d = 0;
    int fan_in[NLAYER], fan_out[NLAYER];
    int64_t w_off[NLAYER], b_off[NLAYER], n_params = 0;
    int64_t t = 0;                    // Adam steps taken
    bool fused;                       // small enough for the fused kernels
    DevBuf p32, pb16, grad, m, v;     // (pb16: larger networks)
    DevBuf packed;                    // the weights' BF16 fragments
    Packed frags{};
    std::vector<float> h_mu, h_sd;    // input standardisation (x - mu) / sd
    DevBuf mu, sd;
    int rows = 0;                     // capacity of the activation buffers
    DevBuf xb, h[NLAYER - 1], g[NLAYER - 1], logits, prob, target, gout, loss, xf;
    int ld = 0;                       // rows of the transposed copies (fused training)
    DevBuf xt, ht[NLAYER - 1], gt[NLAYER];
    Ring ring;                        // host arrays on their way
    PinnedBuf outputs;                // of an inference, at most OUTPUTS floats

    Proposer(int n_in_, int d_) : n_in(n_in_), d(d_) {
        const int sizes[NLAYER + 1] = {n_in, HID, HID, HID, d};
        for (int l = 0; l < NLAYER; ++l) {
            fan_in[l] = sizes[l];
            fan_out[l] = sizes[l + 1];
            w_off[l] = n_params;
            n_params += (int64_t)fan_out[l] * fan_in[l];
            b_off[l] = n_params;
            n_params += fan_out[l];
        }
        fused = n_in <= FUSED_IN && d <= FUSED_OUT;
        p32.ensure(n_params * 4);
        grad.ensure(n_params * 4);
        m.ensure(n_params * 4);
        v.ensure(n_params * 4);
        int64_t at_f[NLAYER], at_b[NLAYER], elems = 0;
        for (int l = 0; l < NLAYER; ++l) {
            frags.fan_in[l] = fan_in[l];
            frags.w_off[l] = w_off[l];
            frags.b_off[l] = b_off[l];
            frags.ks_f[l] = up(fan_in[l], 32) / 32;
            frags.ks_b[l] = up(fan_out[l], 32) / 32;
            at_f[l] = elems;
            elems += (int64_t)up(fan_out[l], 16) / 16 * frags.ks_f[l] * 512;
            at_b[l] = elems;
            if (l > 0) elems += (int64_t)up(fan_in[l], 16) / 16 * frags.ks_b[l] * 512;
        }
        if (fused) {
            packed.ensure((size_t)elems * 2);
            for (int l = 0; l < NLAYER; ++l) {
                frags.fwd[l] = packed.as<uint16_t>() + at_f[l];
                frags.bwd[l] = packed.as<uint16_t>() + at_b[l];
            }
            // LDS beyond 64 KB has to be asked for (not while a stream captures)
            MORAP_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&mlp_rows<false>),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
            MORAP_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&mlp_rows<true>),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
        } else {
            pb16.ensure(n_params * 2);
        }
        mu.ensure((size_t)n_in * 4);
        sd.ensure((size_t)n_in * 4);
        h_mu.assign(n_in, 0.f);
        h_sd.assign(n_in, 1.f);
    }

    void set_norm(hipStream_t s, const float* m_, const float* s_) {
        h_mu.assign(m_, m_ + n_in);
        h_sd.assign(s_, s_ + n_in);
        MORAP_HIP(hipMemcpyAsync(mu.p, h_mu.data(), (size_t)n_in * 4, hipMemcpyHostToDevice, s));
        MORAP_HIP(hipMemcpyAsync(sd.p, h_sd.data(), (size_t)n_in * 4, hipMemcpyHostToDevice, s));
        MORAP_HIP(hipStreamSynchronize(s));
    }

    void ensure_rows(int n) {
        if (n <= rows) return;
        xf.ensure((size_t)n * n_in * 4);
        prob.ensure((size_t)n * d * 4);
        target.ensure((size_t)n * d * 4);
        loss.ensure((size_t)n * 4);
        if (!fused) {
            xb.ensure((size_t)n * n_in * 2);
            for (int l = 0; l < NLAYER - 1; ++l) {
                h[l].ensure((size_t)n * HID * 2);
                g[l].ensure((size_t)n * HID * 2);
            }
            logits.ensure((size_t)n * d * 4);
            gout.ensure((size_t)n * d * 2);
        }
        rows = n;
    }

    // upload FP32 parameters, reset Adam state, refresh BF16 copies
    void set(hipStream_t s, const float* host) {
        MORAP_HIP(hipMemcpyAsync(p32.p, host, n_params * 4, hipMemcpyHostToDevice, s));
        MORAP_HIP(hipMemsetAsync(m.p, 0, n_params * 4, s));
        MORAP_HIP(hipMemsetAsync(v.p, 0, n_params * 4, s));
        if (fused) MORAP_HIP(hipMemsetAsync(packed.p, 0, packed.bytes, s));   // the fragments' padding
        hipLaunchKernelGGL(copies_kernel, dim3(blocks_for(n_params)), dim3(256), 0, s, p32.as<float>(),
                           fused ? nullptr : pb16.as<uint16_t>(), frags, n_params);
        MORAP_HIP(hipGetLastError());
        MORAP_HIP(hipStreamSynchronize(s));
        t = 0;
    }

    // everything local to a row
    void fused_rows(hipStream_t s, int n, const float* x, float* out, const float* T, float* loss_out) {
        RowArgs a{};
        a.x = x;
        a.mu = mu.as<float>();
        a.sd = sd.as<float>();
        a.T = T;
        for (int l = 0; l < NLAYER; ++l) {
            a.fwd[l] = frags.fwd[l];
            a.bwd[l] = frags.bwd[l];
            a.bias[l] = p32.as<float>() + b_off[l];
        }
        a.prob = out;
        a.loss = loss_out;
        a.n = n;
        a.n_in = n_in;
        a.d = d;
        a.inv_b = 1.f / (float)n;
        const size_t bytes = rows_lds(n_in, d, T != nullptr);
        MORAP_CHECK(bytes <= 160 * 1024, MORAP_E_UNSUPPORTED, "the network does not fit the fused kernel");
        const dim3 grid(blocks_for(T ? up(n, 32) : n, ROWS));   // (training: the transposed copies' padding too)
        if (!T) {
            hipLaunchKernelGGL(mlp_rows<false>, grid, dim3(1024), bytes, s, a);
            MORAP_HIP(hipGetLastError());
            return;
        }
        a.ld = ld = up(n, 32);
        xt.ensure((size_t)n_in * ld * 2);
        a.xt = xt.as<uint16_t>();
        for (int l = 0; l < NLAYER; ++l) {
            gt[l].ensure((size_t)fan_out[l] * ld * 2);
            a.gt[l] = gt[l].as<uint16_t>();
            if (l == NLAYER - 1) break;
            ht[l].ensure((size_t)HID * ld * 2);
            a.ht[l] = ht[l].as<uint16_t>();
        }
        hipLaunchKernelGGL(mlp_rows<true>, grid, dim3(1024), bytes, s, a);
        MORAP_HIP(hipGetLastError());
    }

    void fused_grads(hipStream_t s) {
        GradArgs a{};
        a.ld = ld;
        int first = 0;
        for (int l = 0; l < NLAYER; ++l) {
            GradLayer& L = a.l[l];
            L.g = gt[l].as<uint16_t>();
            L.h = l == 0 ? xt.as<uint16_t>() : ht[l - 1].as<uint16_t>();
            L.dw = grad.as<float>() + w_off[l];
            L.db = grad.as<float>() + b_off[l];
            L.N = fan_out[l];
            L.K = fan_in[l];
            L.first = first;
            first += (up(L.N, 32) / 32) * (up(L.K, 32) / 32);
        }
        hipLaunchKernelGGL(weight_grads, dim3((unsigned)first), dim3(1024), 0, s, a);
        MORAP_HIP(hipGetLastError());
    }

    const uint16_t* act(int l) const {   // input of layer l
        return l == 0 ? xb.as<uint16_t>() : h[l - 1].as<uint16_t>();
    }

    // activation buffers of one forward pass
    struct Acts {
        const float* xf;       // [n][n_in] FP32 input
        uint16_t* xb;          // [n][n_in] BF16 standardised input
        uint16_t* h[NLAYER - 1];
        float* logits;         // [n][d]
        float* prob;           // [n][d]
    };
    Acts own_acts() {
        Acts a{xf.as<float>(), xb.as<uint16_t>(), {}, logits.as<float>(), prob.as<float>()};
        for (int l = 0; l < NLAYER - 1; ++l) a.h[l] = h[l].as<uint16_t>();
        return a;
    }

    // forward of n rows already in xf (FP32); logits then softmax into prob
    void forward(hipStream_t s, int n, const float* T_dev) {
        if (fused)
            fused_rows(s, n, xf.as<float>(), prob.as<float>(), T_dev, loss.as<float>());
        else forward_into(s, n, own_acts(), T_dev);
    }

    // the same into the buffers of `b` (T_dev, when given, also fills the
    // loss and the output gradient of the context's own buffers)
    void forward_into(hipStream_t s, int n, const Acts& b, const float* T_dev) {
        hipLaunchKernelGGL(input_kernel, dim3(blocks_for((int64_t)n * n_in)), dim3(256), 0, s, b.xf, mu.as<float>(),
                           sd.as<float>(), b.xb, (int64_t)n * n_in, n_in);
        MORAP_HIP(hipGetLastError());
        for (int l = 0; l < NLAYER; ++l) {
            GemmArgs a{};
            a.A = l == 0 ? b.xb : b.h[l - 1];
            a.sam = fan_in[l];
            a.sak = 1;
            a.B = pb16.as<uint16_t>() + w_off[l];
            a.sbk = 1;
            a.sbn = fan_in[l];
            a.M = n;
            a.N = fan_out[l];
            a.K = fan_in[l];
            a.ldc = fan_out[l];
            a.bias = p32.as<float>() + b_off[l];
            if (l < NLAYER - 1) {
                a.mode = EP_HIDDEN;
                a.Cb = b.h[l];
            } else {
                a.mode = EP_LOGITS;
                a.Cf = b.logits;
            }
            gemm(s, a);
        }
        hipLaunchKernelGGL(softmax_xent, dim3(blocks_for(n, 64)), dim3(64), 0, s, b.logits, T_dev, b.prob,
                           T_dev ? gout.as<uint16_t>() : nullptr, T_dev ? loss.as<float>() : nullptr, n, d,
                           1.f / (float)n);
        MORAP_HIP(hipGetLastError());
    }

    // gradients of the mean cross-entropy into grad (after forward with T)
    void backward(hipStream_t s, int n) {
        if (fused) return fused_grads(s);
        for (int l = NLAYER - 1; l >= 0; --l) {
            const uint16_t* G = l == NLAYER - 1 ? gout.as<uint16_t>() : g[l].as<uint16_t>();
            const int N = fan_out[l], K = fan_in[l];
            // dW[N][K] = G^T H: A(i, r) = G[r][i], B(r, k) = H[r][k]
            GemmArgs w{};
            w.A = G;
            w.sam = 1;
            w.sak = N;
            w.B = act(l);
            w.sbk = K;
            w.sbn = 1;
            w.M = N;
            w.N = K;
            w.K = n;
            w.mode = EP_WGRAD;
            w.Cf = grad.as<float>() + w_off[l];
            w.ldc = K;
            gemm(s, w);
            hipLaunchKernelGGL(bias_grad, dim3(blocks_for(N)), dim3(256), 0, s, G, grad.as<float>() + b_off[l], n,
                               N);
            MORAP_HIP(hipGetLastError());
            if (l == 0) break;
            // G_{l-1}[n][K] = (G W) masked by H_{l-1} > 0: A(r, i) = G[r][i], B(i, k) = W[i][k]
            GemmArgs b{};
            b.A = G;
            b.sam = N;
            b.sak = 1;
            b.B = pb16.as<uint16_t>() + w_off[l];
            b.sbk = K;
            b.sbn = 1;
            b.M = n;
            b.N = K;
            b.K = N;
            b.mode = EP_BWD_DATA;
            b.Cb = g[l - 1].as<uint16_t>();
            b.ldc = K;
            b.mask = h[l - 1].as<uint16_t>();
            b.ldm = K;
            gemm(s, b);
        }
    }

    void adam(hipStream_t s, const morap_train_opts& o) {
        ++t;
        const float c1 = (float)(1.0 - std::pow((double)o.beta1, (double)t));
        const float c2 = (float)(1.0 - std::pow((double)o.beta2, (double)t));
        hipLaunchKernelGGL(adam_kernel, dim3(blocks_for(n_params)), dim3(256), 0, s, p32.as<float>(),
                           grad.as<float>(), m.as<float>(), v.as<float>(), fused ? nullptr : pb16.as<uint16_t>(), frags,
                           n_params, o.lr, o.beta1, o.beta2, o.adam_eps, c1, c2);
        MORAP_HIP(hipGetLastError());
    }

    // host floats to the device; `check`: finite is what they have to be
    void upload(hipStream_t s, float* dst, const float* from, size_t count, bool check) {
        bool bad = false;
        for (size_t i = 0; i < count; i += Ring::FLOATS) {
            const size_t part = std::min(Ring::FLOATS, count - i);
            float* p = ring.next();
            bad |= nonfinite(from + i, p, part);
            MORAP_CHECK(!check || !bad, MORAP_E_INVALID, "X must be finite");
            MORAP_HIP(hipMemcpyAsync(dst + i, p, part * 4, hipMemcpyHostToDevice, s));
            ring.used();
        }
    }
    // device floats to the host, there after ring.finish()
    void download(hipStream_t s, float* to, const float* src, size_t count) {
        for (size_t i = 0; i < count; i += Ring::FLOATS) {
            const size_t part = std::min(Ring::FLOATS, count - i);
            MORAP_HIP(hipMemcpyAsync(ring.next(), src + i, part * 4, hipMemcpyDeviceToHost, s));
            ring.used(to + i, part);
        }
    }

    // one step on n host rows; returns the mean loss
    double step(hipStream_t s, const float* X, const float* T, int n, const morap_train_opts* o, bool apply,
                float* grads_out) {
        const Drain drain(s);
        ring.start(s, Ring::slots((size_t)n * n_in) + Ring::slots((size_t)n * d) + Ring::slots((size_t)n) +
                          (grads_out ? Ring::slots((size_t)n_params) : 0));
        ensure_rows(n);
        upload(s, xf.as<float>(), X, (size_t)n * n_in, true);
        check_targets(T, n, d);
        upload(s, target.as<float>(), T, (size_t)n * d, false);
        forward(s, n, target.as<float>());
        backward(s, n);
        if (apply) adam(s, *o);
        losses.resize((size_t)n);
        download(s, losses.data(), loss.as<float>(), (size_t)n);
        if (grads_out) download(s, grads_out, grad.as<float>(), (size_t)n_params);
        ring.finish();
        double sum = 0;
        for (int i = 0; i < n; ++i) sum += losses[(size_t)i];
        return sum / n;
    }
    std::vector<float> losses;

    // Inference with the fused kernel reads host rows from the ring's slots and
    // writes to pinned memory, each row once: a call's rows go in parts, at most 8
    // where the slots hold them, the host copying and checking one while the device
    // works on those before; the outputs leave when every row has been read (the
    // arrays may overlap, and a refused call writes none).  4,000 rows of
    // 182 -> 150 take 0.24 ms; 0.32 with one copy there, one launch and one copy
    // back.  (A training step is no faster so: the device would wait for its
    // rows where now they arrive while the host checks the targets.)
    static constexpr size_t OUTPUTS = (size_t)1 << 22;
    void infer(hipStream_t s, const float* X, int n, float* out, bool check) {
        const Drain drain(s);
        const size_t count = (size_t)n * d;
        const bool pinned = fused && count <= OUTPUTS;
        const int step = std::min<int>(std::max(up((n + 7) / 8, ROWS), up((256 << 10) / (n_in * 4), ROWS)),
                                       (int)(Ring::FLOATS / n_in) / ROWS * ROWS);
        const int parts = (n + step - 1) / step;
        // (pinned outputs leave part by part, on events)
        ring.start(s, pinned ? (parts > 1 ? Ring::SLOTS + 1 : 1)
                             : (fused ? (size_t)parts : Ring::slots((size_t)n * n_in)) + Ring::slots(count));
        if (!pinned) ensure_rows(n);
        if (!fused) {
            upload(s, xf.as<float>(), X, (size_t)n * n_in, check);
            forward(s, n, nullptr);
        } else {
            if (pinned) outputs.ensure(count * 4);
            float* p = pinned ? outputs.as<float>() : prob.as<float>();
            for (int r = 0; r < n; r += step) {
                const int rows = std::min(step, n - r);
                float* x = ring.next();
                const bool bad = nonfinite(X + (size_t)r * n_in, x, (size_t)rows * n_in);
                MORAP_CHECK(!check || !bad, MORAP_E_INVALID, "X must be finite");
                fused_rows(s, rows, x, p + (size_t)r * d, nullptr, nullptr);
                ring.used();
            }
        }
        if (!pinned) {
            download(s, out, prob.as<float>(), count);
            ring.finish();
            return;
        }
        for (int q = 0; q < parts; ++q) {
            if (q >= parts - Ring::SLOTS) ring.wait(q % Ring::SLOTS);   // (those before have given up their slots)
            const size_t r = (size_t)q * step;
            std::memcpy(out + r * d, outputs.as<float>() + r * d, std::min((size_t)step, n - r) * d * 4);
        }
    }
};

void proposer_destroy(Proposer* p) { delete p; }

// ---------------------------------------------------------------------------
// allocation-free inference: the activations of morap_proposer_infer_noalloc
// live in this fixed array (one copy per device, held until the process
// ends).  Its device address is taken once per device when a context is
// created there; host code uses that address, never the array's name.
// ---------------------------------------------------------------------------
constexpr size_t kScratchBytes = (size_t)8 << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];
static std::mutex g_scratch_mu;
static std::vector<unsigned char*> g_scratch;   // per device

void proposer_scratch_init(int device) {   // with `device` current
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if ((int)g_scratch.size() <= device) g_scratch.resize((size_t)device + 1, nullptr);
    if (g_scratch[(size_t)device]) return;
    void* p = nullptr;
    MORAP_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    MORAP_CHECK(p != nullptr, MORAP_E_HIP, "no device address for the inference scratch");
    g_scratch[(size_t)device] = static_cast<unsigned char*>(p);
}

static unsigned char* scratch_of(int device) {
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    MORAP_CHECK(device >= 0 && device < (int)g_scratch.size() && g_scratch[(size_t)device], MORAP_E_STATE,
                "the inference scratch of this device was not set up (no context created on it)");
    return g_scratch[(size_t)device];
}

static size_t round256(size_t b) { return (b + 255) / 256 * 256; }

// scratch bytes of an n-row forward pass: BF16 input, three BF16 hidden
// layers, FP32 logits
static size_t scratch_need(int64_t n, int n_in, int d) {
    return round256((size_t)n * n_in * 2) + 3 * round256((size_t)n * HID * 2) + round256((size_t)n * d * 4);
}

bool proposer_ready(const morap_ctx* c, int n_in, int d) {
    return c->prop_mlp && c->prop_mlp->n_in == n_in && c->prop_mlp->d == d;
}

void proposer_infer_host(morap_ctx* c, const float* X, int n, float* out) {
    MORAP_CHECK(c->prop_mlp, MORAP_E_STATE, "no proposer");
    c->prop_mlp->infer(c->stream, X, n, out, false);
}

static Proposer& need(morap_ctx* c) {
    MORAP_CHECK(c->prop_mlp, MORAP_E_STATE, "no proposer: call morap_proposer_init or morap_proposer_load");
    return *c->prop_mlp;
}

static void check_opts(const morap_train_opts* o) {
    MORAP_CHECK(o && o->batch >= 1 && o->epochs >= 0 && o->lr > 0 && o->beta1 >= 0 && o->beta1 < 1 &&
                    o->beta2 >= 0 && o->beta2 < 1 && o->adam_eps > 0,
                MORAP_E_INVALID, "bad training options");
}

static void init_params(morap_ctx* c, int n_in, int d, uint64_t seed) {
    MORAP_CHECK(n_in >= 1 && n_in <= 4096 && d >= 1 && d <= 4096, MORAP_E_INVALID, "bad proposer sizes");
    auto p = std::make_unique<Proposer>(n_in, d);
    std::vector<float> host(p->n_params, 0.f);
    for (int l = 0; l < NLAYER; ++l) {
        const double lim = std::sqrt(6.0 / p->fan_in[l]);   // He-uniform
        for (int64_t i = p->w_off[l]; i < p->b_off[l]; ++i) {
            const double u = (double)(splitmix64(seed + (uint64_t)i) >> 11) * 0x1.0p-53;
            host[i] = (float)(lim * (2.0 * u - 1.0));
        }
    }
    p->set(c->stream, host.data());
    p->set_norm(c->stream, p->h_mu.data(), p->h_sd.data());
    if (c->prop_mlp) proposer_destroy(c->prop_mlp);
    c->prop_mlp = p.release();
}

}  // namespace morap

using namespace morap;

extern "C" {

int morap_proposer_init(morap_ctx* ctx, int n_in, int d, uint64_t seed) {
    return guarded(ctx, [&] { init_params(ctx, n_in, d, seed); });
}

int64_t morap_proposer_num_params(const morap_ctx* ctx) {
    return ctx && ctx->prop_mlp ? ctx->prop_mlp->n_params : 0;
}

int morap_proposer_get_params(const morap_ctx* ctx, float* out) {
    auto* c = const_cast<morap_ctx*>(ctx);
    return guarded(c, [&] {
        Proposer& p = need(c);
        MORAP_CHECK(out, MORAP_E_INVALID, "NULL output");
        MORAP_HIP(hipMemcpyAsync(out, p.p32.p, p.n_params * 4, hipMemcpyDeviceToHost, c->stream));
        MORAP_HIP(hipStreamSynchronize(c->stream));
    });
}

int morap_proposer_set_params(morap_ctx* ctx, const float* in) {
    return guarded(ctx, [&] {
        Proposer& p = need(ctx);
        MORAP_CHECK(in, MORAP_E_INVALID, "NULL input");
        for (int64_t i = 0; i < p.n_params; ++i) MORAP_CHECK(std::isfinite(in[i]), MORAP_E_INVALID, "non-finite parameter");
        p.set(ctx->stream, in);
    });
}

int morap_proposer_set_input_norm(morap_ctx* ctx, const float* mu, const float* sd) {
    return guarded(ctx, [&] {
        Proposer& p = need(ctx);
        MORAP_CHECK(mu && sd, MORAP_E_INVALID, "NULL arguments");
        for (int i = 0; i < p.n_in; ++i)
            MORAP_CHECK(std::isfinite(mu[i]) && std::isfinite(sd[i]) && sd[i] > 0, MORAP_E_INVALID,
                        "need finite mu and sd > 0");
        p.set_norm(ctx->stream, mu, sd);
    });
}

int morap_proposer_infer(morap_ctx* ctx, const float* X, int n, float* W_out) {
    return guarded(ctx, [&] {
        Proposer& p = need(ctx);
        MORAP_CHECK(X && n >= 1, MORAP_E_INVALID, "need X and n >= 1");
        MORAP_CHECK(W_out, MORAP_E_INVALID, "NULL output");
        p.infer(ctx->stream, X, n, W_out, true);
    });
}

int morap_proposer_infer_noalloc(morap_ctx* ctx, const float* X_dev, int n, float* W_out_dev) {
    return guarded(ctx, [&] {
        Proposer& p = need(ctx);
        MORAP_CHECK(X_dev && W_out_dev && n >= 1, MORAP_E_INVALID, "need device X, device W_out and n >= 1");
        const size_t need_b = scratch_need(n, p.n_in, p.d);
        if (need_b > kScratchBytes) {
            int64_t max_rows = 0;
            while (scratch_need(max_rows + 1, p.n_in, p.d) <= kScratchBytes) ++max_rows;
            fail(MORAP_E_UNSUPPORTED, std::to_string(n) + " rows need " + std::to_string(need_b) +
                                          " bytes of inference scratch; the fixed scratch holds " +
                                          std::to_string(kScratchBytes) + " bytes (at most " +
                                          std::to_string(max_rows) + " rows for this network)");
        }
        if (p.fused) {
            // (the input may share memory with the output: then the rows'
            // outputs wait in the scratch until every row has been read)
            const uintptr_t x0 = reinterpret_cast<uintptr_t>(X_dev), w0 = reinterpret_cast<uintptr_t>(W_out_dev);
            const size_t count = (size_t)n * p.d;
            const bool shared = x0 < w0 + count * 4 && w0 < x0 + (size_t)n * p.n_in * 4;
            float* out = shared ? reinterpret_cast<float*>(scratch_of(ctx->device)) : W_out_dev;
            p.fused_rows(ctx->stream, n, X_dev, out, nullptr, nullptr);
            if (shared) {
                hipLaunchKernelGGL(copy_kernel, dim3(blocks_for((int64_t)count)), dim3(256), 0, ctx->stream, out,
                                   W_out_dev, (int64_t)count);
                MORAP_HIP(hipGetLastError());
            }
            return;
        }
        unsigned char* base = scratch_of(ctx->device);
        Proposer::Acts a{};
        a.xf = X_dev;
        size_t off = 0;
        a.xb = reinterpret_cast<uint16_t*>(base + off);
        off += round256((size_t)n * p.n_in * 2);
        for (int l = 0; l < NLAYER - 1; ++l) {
            a.h[l] = reinterpret_cast<uint16_t*>(base + off);
            off += round256((size_t)n * HID * 2);
        }
        a.logits = reinterpret_cast<float*>(base + off);
        a.prob = W_out_dev;
        p.forward_into(ctx->stream, n, a, nullptr);
    });
}

int morap_proposer_step(morap_ctx* ctx, const float* X, const float* T, int n, const morap_train_opts* opts,
                        int apply, float* loss_out, float* grads_out) {
    return guarded(ctx, [&] {
        Proposer& p = need(ctx);
        MORAP_CHECK(T, MORAP_E_INVALID, "NULL targets");
        MORAP_CHECK(X && n >= 1, MORAP_E_INVALID, "need X and n >= 1");
        if (apply) check_opts(opts);
        const double l = p.step(ctx->stream, X, T, n, opts, apply != 0, grads_out);
        if (loss_out) *loss_out = (float)l;
    });
}

int morap_proposer_train(morap_ctx* ctx, const float* X, const float* T, int n, const morap_train_opts* opts,
                         float* loss_out) {
    return guarded(ctx, [&] {
        Proposer& p = need(ctx);
        check_opts(opts);
        check_rows(X, T, n, p.n_in, p.d);
        std::vector<int> order(n);
        std::iota(order.begin(), order.end(), 0);
        const int B = std::min(opts->batch, n);
        std::vector<float> xb((size_t)B * p.n_in), tb((size_t)B * p.d);
        uint64_t ctr = 0;
        for (int ep = 0; ep < opts->epochs; ++ep) {
            for (int i = n - 1; i > 0; --i) {   // Fisher-Yates from SplitMix64(seed, counter)
                const int j = (int)(splitmix64(opts->seed ^ (0x5851F42D4C957F2Dull * ++ctr)) % (uint64_t)(i + 1));
                std::swap(order[i], order[j]);
            }
            double sum = 0;
            int batches = 0;
            for (int b0 = 0; b0 + B <= n; b0 += B) {   // full batches only
                for (int r = 0; r < B; ++r) {
                    std::copy(X + (size_t)order[b0 + r] * p.n_in, X + (size_t)(order[b0 + r] + 1) * p.n_in,
                              xb.begin() + (size_t)r * p.n_in);
                    std::copy(T + (size_t)order[b0 + r] * p.d, T + (size_t)(order[b0 + r] + 1) * p.d,
                              tb.begin() + (size_t)r * p.d);
                }
                sum += p.step(ctx->stream, xb.data(), tb.data(), B, opts, true, nullptr);
                ++batches;
            }
            if (loss_out) loss_out[ep] = (float)(sum / std::max(1, batches));
        }
    });
}

int morap_proposer_save(const morap_ctx* ctx, const char* path) {
    auto* c = const_cast<morap_ctx*>(ctx);
    return guarded(c, [&] {
        Proposer& p = need(c);
        MORAP_CHECK(path, MORAP_E_INVALID, "NULL path");
        std::vector<float> host(p.n_params);
        MORAP_HIP(hipMemcpyAsync(host.data(), p.p32.p, p.n_params * 4, hipMemcpyDeviceToHost, c->stream));
        MORAP_HIP(hipStreamSynchronize(c->stream));
        FILE* f = std::fopen(path, "wb");
        MORAP_CHECK(f, MORAP_E_INVALID, std::string("cannot write ") + path);
        const int32_t hdr[4] = {0x504C4D4D /* "MMLP" */, 1, p.n_in, p.d};
        bool ok = std::fwrite(hdr, sizeof hdr, 1, f) == 1 &&
                  std::fwrite(p.h_mu.data(), 4, p.n_in, f) == (size_t)p.n_in &&
                  std::fwrite(p.h_sd.data(), 4, p.n_in, f) == (size_t)p.n_in &&
                  std::fwrite(host.data(), 4, host.size(), f) == host.size();
        ok &= std::fclose(f) == 0;
        MORAP_CHECK(ok, MORAP_E_INVALID, std::string("write failed: ") + path);
    });
}

int morap_proposer_load(morap_ctx* ctx, const char* path) {
    return guarded(ctx, [&] {
        MORAP_CHECK(path, MORAP_E_INVALID, "NULL path");
        FILE* f = std::fopen(path, "rb");
        MORAP_CHECK(f, MORAP_E_INVALID, std::string("cannot read ") + path);
        int32_t hdr[4] = {0, 0, 0, 0};
        const bool hok = std::fread(hdr, sizeof hdr, 1, f) == 1 && hdr[0] == 0x504C4D4D && hdr[1] == 1 &&
                         hdr[2] >= 1 && hdr[2] <= 4096 && hdr[3] >= 1 && hdr[3] <= 4096;
        if (!hok) std::fclose(f);
        MORAP_CHECK(hok, MORAP_E_INVALID, std::string("not a proposer file: ") + path);
        auto p = std::make_unique<Proposer>(hdr[2], hdr[3]);
        std::vector<float> host(p->n_params), nm(p->n_in), ns(p->n_in);
        const bool ok = std::fread(nm.data(), 4, nm.size(), f) == nm.size() &&
                        std::fread(ns.data(), 4, ns.size(), f) == ns.size() &&
                        std::fread(host.data(), 4, host.size(), f) == host.size();
        std::fclose(f);
        MORAP_CHECK(ok, MORAP_E_INVALID, std::string("truncated proposer file: ") + path);
        for (float x : host) MORAP_CHECK(std::isfinite(x), MORAP_E_INVALID, "non-finite parameter in file");
        for (int i = 0; i < p->n_in; ++i)
            MORAP_CHECK(std::isfinite(nm[i]) && std::isfinite(ns[i]) && ns[i] > 0, MORAP_E_INVALID,
                        "bad input standardisation in file");
        p->set(ctx->stream, host.data());
        p->set_norm(ctx->stream, nm.data(), ns.data());
        if (ctx->prop_mlp) proposer_destroy(ctx->prop_mlp);
        ctx->prop_mlp = p.release();
    });
}

}  // extern "C"

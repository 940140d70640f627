// mlp.hip -- the learned proposal's network on the matrix cores: a
// 6 -> 128 -> 128 -> 56 MLP (SiLU) in bfloat16 with float32 accumulation,
// the mixture head and its weighted negative log-likelihood in float32,
// split-K weight gradients, Adam with float32 master weights, training-data
// weights and the training loop.
//
// Every product of the network is a dense contraction, so it runs on MFMA.
// One kernel (k_strip) takes a wave's 16 rows through the forward layers, the
// loss and the backward layers without a layer value leaving the registers:
// the products are computed transposed (W^T x^T), so that the rows of one
// layer's accumulators are the contraction values of the next layer's operand.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <vector>

#include "mxr.h"

namespace mxr_host {
mxr_status set_error(mxr_status st, const char *msg);
}

namespace {

constexpr int kIn = MXR_MLP_IN, kHid = MXR_MLP_HIDDEN, kOut = MXR_MLP_OUT;
constexpr uint64_t kW1 = 0, kB1 = kW1 + kIn * kHid, kW2 = kB1 + kHid, kB2 = kW2 + kHid * kHid;
constexpr uint64_t kW3 = kB2 + kHid, kB3 = kW3 + kHid * kOut, kParams = kB3 + kOut;
static_assert(kParams == MXR_MLP_PARAMS, "parameter layout");
constexpr uint64_t kSplitRows = 1024;  // the workspace's room: a partial gradient per so many rows
constexpr int kThreads = 256;

typedef short v4s __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

mxr_status fail(mxr_status st, const char *fmt, ...) __attribute__((format(printf, 2, 3)));
mxr_status fail(mxr_status st, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    return mxr_host::set_error(st, buf);
}

mxr_status launch_check(const char *what) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(MXR_E_HIP, "%s: %s", what, hipGetErrorString(e));
    return MXR_OK;
}

// ------------------------------------------------------------ bfloat16 --

__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
    uint32_t b = __float_as_uint(f);
    if ((b & 0x7F800000u) == 0x7F800000u) return (uint16_t)((b >> 16) | ((b & 0xFFFFu) ? 0x40u : 0u));  // inf/nan
    b += 0x7FFFu + ((b >> 16) & 1u);  // round to nearest, ties to even
    return (uint16_t)(b >> 16);
}

__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// Hardware exponential, logarithm and reciprocal (v_exp_f32, v_log_f32,
// v_rcp_f32: about an ulp each; the argument scaling adds a few ulp): the
// activations they feed are rounded to bfloat16, and the head's float32 loss
// gradient is checked to 3e-4 of a row's scale, so the ten-instruction IEEE
// division and the full-range expf / logf buy nothing here.
__device__ __forceinline__ float fexp(float x) { return __builtin_amdgcn_exp2f(x * 1.4426950408889634f); }
__device__ __forceinline__ float flog(float x) { return __builtin_amdgcn_logf(x) * 0.6931471805599453f; }
__device__ __forceinline__ float frcp(float x) { return __builtin_amdgcn_rcpf(x); }

// ------------------------------------------------------ small kernels --

// Deterministic sums: each work-group sums its stride of the input into one
// partial; a second launch with one work-group sums the partials in order.
__global__ void k_sum_f64(const double *x, uint64_t n, double *partial) {
    __shared__ double red[kThreads];
    double s = 0.0;
    for (uint64_t i = (uint64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (uint64_t)gridDim.x * kThreads)
        s += x[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = kThreads / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

constexpr unsigned kSumBlocks = 256;

// The mixture head and the weighted negative log-likelihood of one row per
// thread, in float32.  Head: pi = softmax(logits), mu = centre + half tanh,
// sigma = half (1e-3 + softplus).  -log q = -logsumexp_k(log pi_k +
// sum_d log N(y_d; mu, sigma)) + log sum_k pi_k Z_k.  Writes dL/do scaled by
// a_i = omega_i / sum omega (float32 and bfloat16) and a_i (-log q_i).
__device__ __forceinline__ float phi_pdf(float z) { return 0.3989422804014327f * fexp(-0.5f * z * z); }

// Mass of a standard normal in [za, zb], from the side that does not cancel:
// both ends' tails, taken outward where the ends lie on one side of 0.
__device__ __forceinline__ float box_mass(float za, float zb) {
    const bool right = za > 0.f, left = !right && zb < 0.f;
    const float a = erfcf((right ? za : -za) * 0.70710678f);
    const float b = erfcf((left ? -zb : zb) * 0.70710678f);
    const float d = right ? a - b : b - a;
    return right || left ? 0.5f * d : 1.0f - 0.5f * (a + b);
}

// The four lanes l, l ^ 16, l ^ 32, l ^ 48 hold a row, two mixture components
// each; row-level maxima and sums go over the pair and then the lanes.
__device__ __forceinline__ float row_max(float a, float b) {
    float v = fmaxf(a, b);
    v = fmaxf(v, __shfl_xor(v, 16, 64));
    return fmaxf(v, __shfl_xor(v, 32, 64));
}
__device__ __forceinline__ float row_sum(float a, float b) {
    float v = a + b;
    v += __shfl_xor(v, 16, 64);
    return v + __shfl_xor(v, 32, 64);
}

// The head and loss gradient of one row, components 2 q and 2 q + 1 of lane q
// of the row's four (which take part together).  o: the components' outputs;
// y: the row's target; a: its loss weight omega_i / sum omega.  g: dL/do of the
// outputs, scaled by a; loss: a (-log q) of the row (every lane of the four).
__device__ __forceinline__ void head_rows(const float o[2][7], const float y[3], float a, const float lo[3],
                                          const float hi[3], float g[2][7], float &loss) {
    const float mx = row_max(o[0][0], o[1][0]);
    const float lse_logit = mx + flog(row_sum(fexp(o[0][0] - mx), fexp(o[1][0] - mx)));
    float pi[2], c[2], zk[2];
    float t[2][3], sg[2][3], F[2][3];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        pi[k] = fexp(o[k][0] - lse_logit);
        c[k] = o[k][0] - lse_logit;
        zk[k] = 1.f;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const float cen = 0.5f * (lo[d] + hi[d]), half = 0.5f * (hi[d] - lo[d]);
            t[k][d] = tanhf(o[k][1 + d]);
            const float mu = cen + half * t[k][d];
            const float raw = o[k][4 + d];
            const float sp = raw > 20.f ? raw : log1pf(fexp(raw));
            sg[k][d] = half * (1e-3f + sp);
            const float is = frcp(sg[k][d]);
            const float z = (y[d] - mu) * is;
            F[k][d] = box_mass((lo[d] - mu) * is, (hi[d] - mu) * is);
            c[k] += -0.5f * z * z - flog(sg[k][d]) - 0.91893853f;
            zk[k] *= F[k][d];
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    const float cmax = row_max(c[0], c[1]);
    const float lse = cmax + flog(row_sum(fexp(c[0] - cmax), fexp(c[1] - cmax)));
    const float S = row_sum(pi[0] * zk[0], pi[1] * zk[1]);
    loss = a * (flog(S) - lse);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const float r = fexp(c[k] - lse);
        const float s = pi[k] * zk[k] * frcp(S);
        g[k][0] = a * (s - r);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            // t opaque: what follows from it is computed again rather than
            // held from the loop above in 18 registers
            float tk = t[k][d];
            asm volatile("" : "+v"(tk));
            const float cen = 0.5f * (lo[d] + hi[d]), half = 0.5f * (hi[d] - lo[d]);
            const float mu = cen + half * tk;
            const float is = frcp(sg[k][d]), iF = frcp(F[k][d]);
            const float z = (y[d] - mu) * is, za = (lo[d] - mu) * is, zb = (hi[d] - mu) * is;
            const float pa = phi_pdf(za), pb = phi_pdf(zb);
            const float dF_mu = -(pb - pa) * is;
            const float dF_sg = -(zb * pb - za * pa) * is;
            const float g_mu = -r * z * is + s * dF_mu * iF;
            const float g_sg = -r * (z * z - 1.f) * is + s * dF_sg * iF;
            g[k][1 + d] = a * (g_mu * half * (1.f - tk * tk));
            g[k][4 + d] = a * (g_sg * half * frcp(1.f + fexp(-o[k][4 + d])));
        }
    }
}

// Mixture tables for the tracer from head outputs: per row and component
// (pi, mu_u, mu_v, mu_E, sigma_u, sigma_v, sigma_E), computed in float32
// like the training head and stored as float64.
// One thread per row and component: a row a thread took 22.7 us for 360 rows,
// all of it the latency of 80 chained evaluations in two work-groups.
__global__ void k_head_params(const float *O, uint64_t n, float lo0, float lo1, float lo2, float hi0, float hi1,
                              float hi2, double *gmm) {
    for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < 8 * n; e += (uint64_t)gridDim.x * blockDim.x) {
        const float lo[3] = {lo0, lo1, lo2}, hi[3] = {hi0, hi1, hi2};
        const float *row = O + (e >> 3) * kOut, *o = row + 7 * (e & 7);
        float mx = -INFINITY;
#pragma unroll
        for (int k = 0; k < 8; ++k) mx = fmaxf(mx, row[7 * k]);
        float se = 0.f;
#pragma unroll
        for (int k = 0; k < 8; ++k) se += expf(row[7 * k] - mx);
        const float lse = mx + logf(se);
        double *g = gmm + 7 * e;
        g[0] = (double)expf(o[0] - lse);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const float cen = 0.5f * (lo[d] + hi[d]), half = 0.5f * (hi[d] - lo[d]);
            const float raw = o[4 + d];
            const float sp = raw > 20.f ? raw : log1pf(expf(raw));
            g[1 + d] = (double)(cen + half * tanhf(o[1 + d]));
            g[4 + d] = (double)(half * (1e-3f + sp));
        }
    }
}

__global__ void k_adam(float *theta, uint16_t *wb, const float *g, float *m, float *v, uint64_t n, float lr, float b1,
                       float b2, float eps, float c1, float c2) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) {
        const float gi = g[i];
        const float mi = b1 * m[i] + (1.f - b1) * gi;
        const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        const float t = theta[i] - lr * (mi * c1) / (sqrtf(vi * c2) + eps);
        theta[i] = t;
        wb[i] = f32_to_bf16(t);
    }
}

__global__ void k_to_bf16(const float *x, uint64_t n, uint16_t *y) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
        y[i] = f32_to_bf16(x[i]);
}

// ------------------------------------------------------- strip kernel --
// Rows of a batch: row i of the batch is dataset row (a i + b) mod n_data
// (a coprime to n_data: a bijection, a cheap shuffle per epoch; a, b and
// the row index below n_data < 2^32); the identity is a = 1, b = 0.
//
// A work-group of eight waves takes passes of 128 rows, 16 a wave.  Every
// product of the chain is computed transposed: the weights are the A operand
// (16 outputs x 16 or 32 inputs), the rows the B operand's columns, and the
// accumulator leaves in lane (r, q) = (l % 16, l / 16) of row r four outputs
// whose indices row_of() chooses such that they are the contraction values
// that the same lane holds of the next product's B operand.  So the layer
// values, the loss and the backward layers stay in a lane's registers, and the
// four lanes of a row hold two mixture components each.  Only the weight
// gradients contract over rows: their operands go through LDS, transposed.
//
// What bounds it: VALU issue.  A pass takes 49,000 clocks of a SIMD's two waves
// (16,000 the head, 10,000 the hidden activations), about 6,000 instructions a
// wave; staging the weights takes 10,000 clocks and writing the partial gradient
// 14,000.  65,536 rows, two passes a work-group: 69 us in training (131 us before
// it, in strips of 32 rows bound by 16-bit LDS gathers of the operands and 11
// barriers a strip), 120 us with the layer values written (242 MB; 17 launches
// took 394 us), 360 rows forward 19 us (6 launches and a copy: 48 us).
//   - 8 waves x 16 rows: the weights' fragments (both directions, 100 KB) and
//     one transposed layer (32 + 16 KB) fill the LDS of one work-group; two
//     waves a SIMD hide each other's latencies with 256 registers each.
//   - kTraining contracts 32 inputs per instruction, the other modes 16: the
//     order of the float32 sums of each path is what it was before it was
//     fused, so its results are the same bit for bit but for the order in
//     which dZ2 sums the outputs and the gradients sum the rows.
constexpr int kWaves = 8, kPassRows = 16 * kWaves, kStripThreads = 64 * kWaves;
constexpr int kGroupsMax = 256;

enum StripMode {
    kForwardOnly,  // outputs alone
    kForward,      // outputs and the workspace's layer values
    kGradient,     // and the loss and the gradient partials
    kTraining      // loss and gradient partials, no layer values
};

struct StripArgs {
    const uint16_t *w;  // bfloat16 parameters
    const float *ctx;
    const double *y, *omega;
    uint64_t n_data, a, b, first, cnt;  // batch row i = data row (a (first + i) mod n_data + b) mod n_data
    const double *wsum;                 // kSumBlocks partial sums of the batch's omega
    float lo[3], hi[3];
    float *out;         // kForward, kForwardOnly
    float *part;        // gridDim.x x kParams partial gradients
    double *loss_part;  // gridDim.x partial losses
    // layer values (kForward, kGradient), stored up to 16 bytes at a time, which
    // in global memory needs the alignment of a float only
    uint16_t *X, *H1, *H2, *wt;
    float *Z1, *Z2, *O;
    // kGradient
    float *dO, *dZ2, *dZ1;
    uint16_t *dOh, *dZ2h, *dZ1h;
    double *Y, *W, *row_loss;
};

__device__ __forceinline__ v4f mfma16(uint2 a, uint2 b, v4f c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(v4s, a), __builtin_bit_cast(v4s, b), c, 0, 0, 0);
}

// gfx950's 16 x 16 x 32 bfloat16 product (twice the K of one instruction):
// lane l holds row (A) or column (B) l % 16 and eight values of k, the same
// eight for A and B (8 (l / 16) + j); the accumulator layout is the
// 16 x 16 x 16 product's: rows 4 (l / 16) + j of column l % 16.
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
__device__ __forceinline__ v4f mfma32(uint4 a, uint4 b, v4f c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
}

// two float32 to bfloat16, round to nearest even (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack2(float a, float b) {
    const v2bf v = {(__bf16)a, (__bf16)b};
    return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ uint2 pack4(v4f v) { return make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3])); }

// Index of the layer value that lane group q holds as entry j of tile t: the
// pair of tiles (2 u, 2 u + 1) covers values [32 u, 32 u + 32), in the order in
// which the next product's instructions contract them.
template <bool K32>
__device__ __forceinline__ int row_of(int t, int q, int j) {
    return K32 ? 32 * (t >> 1) + 8 * q + 4 * (t & 1) + j : 16 * t + 4 * q + j;
}
// Output index of entry j of tile t (components 2 q and 2 q + 1), or -1.
__device__ __forceinline__ int out_of(int t, int q, int j) { return 4 * t + j < 14 ? 14 * q + 4 * t + j : -1; }

// One pair of tiles' contraction.
template <bool K32>
__device__ __forceinline__ v4f mfma_pair(uint4 a, uint2 b0, uint2 b1, v4f c) {
    if constexpr (K32) return mfma32(a, make_uint4(b0.x, b0.y, b1.x, b1.y), c);
    c = mfma16(make_uint2(a.x, a.y), b0, c);
    return mfma16(make_uint2(a.z, a.w), b1, c);
}

// Transposed layer in LDS: value h of the pass's 128 rows, 256 bytes, its
// sixteen 8-row chunks permuted by h so that neither the writes (two rows of
// eight h) nor the reads (a chunk of 16 consecutive h) meet a bank twice.
__device__ __forceinline__ int swizzle(int h) { return (h & 15) ^ ((h >> 2) & 4); }
__device__ __forceinline__ uint4 chunk(const uint16_t *T, int h, int c) {
    return *(const uint4 *)(T + h * kPassRows + ((c ^ swizzle(h)) << 3));
}
template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
}
constexpr int kXor1 = 0xB1, kXor3 = 0x1B, kXor7 = 0x141, kXor15 = 0x140;  // lane l takes l ^ n's, within 16 lanes

// Lane's four values h0 .. h0 + 3 of its row into T: neighbouring lanes trade
// two of them, so that each writes two values of a pair of rows.
__device__ __forceinline__ void put4(uint16_t *T, int h0, int row, uint2 v) {
    const bool odd = row & 1;
    const uint32_t keep = odd ? v.y : v.x, got = dpp<kXor1>(odd ? v.x : v.y);
    const uint32_t even_row = odd ? got : keep, odd_row = odd ? keep : got;
    const int h = h0 + 2 * odd;
    uint32_t *p = (uint32_t *)T + (row & 6) / 2;
    p[h * (kPassRows / 2) + (((row >> 3) ^ swizzle(h)) << 2)] = __builtin_amdgcn_perm(odd_row, even_row, 0x05040100u);
    p[(h + 1) * (kPassRows / 2) + (((row >> 3) ^ swizzle(h + 1)) << 2)] =
        __builtin_amdgcn_perm(odd_row, even_row, 0x07060302u);
}

// Sums over the 16 rows of a lane group of N values a lane: at each step the
// lanes of a pair keep a half each, and in the end lane r holds the sums of
// values N / 16 r .. in v[0 .. N / 16).
template <int N, int CTRL>
__device__ __forceinline__ void scatter_step(float *v, bool upper) {
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
        const float keep = upper ? v[i + N / 2] : v[i], send = upper ? v[i] : v[i + N / 2];
        v[i] = keep + __uint_as_float(dpp<CTRL>(__float_as_uint(send)));
    }
}
template <int N>
__device__ __forceinline__ void scatter_sum(float *v, int r) {
    scatter_step<N, kXor15>(v, r & 8);
    scatter_step<N / 2, kXor7>(v, r & 4);
    scatter_step<N / 4, kXor3>(v, r & 2);
    scatter_step<N / 8, kXor1>(v, r & 1);
}

__device__ __forceinline__ uint4 load16(const uint16_t *p) {  // any alignment of the parameters
    uint4 v;
    __builtin_memcpy(&v, p, 16);
    return v;
}

// The weights as A fragments, one 16-byte piece a lane: piece (t, u) holds
// values row_of(2 u + e / 4, q, e % 4) of tile row r.
template <bool BACK>
struct StripLds {
    uint4 w2[8 * 4 * 64], w3[4 * 4 * 64];                              // W2^T, W3^T (outputs as out_of)
    uint4 w2b[BACK ? 8 * 4 * 64 : 1], w3b[BACK ? 8 * 2 * 64 : 1];      // W2, W3
    uint2 w1[8 * 64];                                                  // W1^T
    float b1[kHid], b2[kHid], b3[64];
    double red[BACK ? kSumBlocks : 1];                                 // the batch's weight sums, then their sum
    // transposed layers; before the first pass the parameters as they come
    uint16_t t[(kHid + 64) * kPassRows];
};
constexpr int kRawRow = kHid + 4;  // staged W2 rows, two banks apart
static_assert((kHid * kRawRow + kHid * kOut) <= (kHid + 64) * kPassRows, "staging space");

// Stages the weights, and (BACK) sums the batch's weight sums: one wave does it
// beside the staging, in the order of a halving tree over the partials.
template <bool K32, bool BACK>
__device__ __forceinline__ void stage_weights(const uint16_t *w, const double *wsum, StripLds<BACK> &S, int tid) {
    static_assert(kSumBlocks == 256 && kSumBlocks <= kStripThreads, "four partials a lane of one wave");
    double part = 0.0;
    if constexpr (BACK)
        if (tid < (int)kSumBlocks) part = wsum[tid];
    uint16_t *raw = S.t, *raw3 = raw + kHid * kRawRow;
    uint4 c2[4], c3[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) c2[i] = load16(w + kW2 + 8 * (tid + i * kStripThreads));
#pragma unroll
    for (int i = 0; i < 2; ++i)
        if (tid + i * kStripThreads < kHid * kOut / 8) c3[i] = load16(w + kW3 + 8 * (tid + i * kStripThreads));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int c = tid + i * kStripThreads;
        uint2 *p = (uint2 *)(raw + (c >> 4) * kRawRow + 8 * (c & 15));
        p[0] = make_uint2(c2[i].x, c2[i].y);
        p[1] = make_uint2(c2[i].z, c2[i].w);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
        if (tid + i * kStripThreads < kHid * kOut / 8) ((uint4 *)raw3)[tid + i * kStripThreads] = c3[i];
    {
        const int t = tid >> 6, r = tid & 15, q = (tid >> 4) & 3, m = row_of<K32>(t, r >> 2, r & 3);
        uint32_t e[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) e[j] = 4 * q + j < kIn ? w[kW1 + (4 * q + j) * kHid + m] : 0;
        S.w1[tid] = make_uint2(e[0] | e[1] << 16, e[2] | e[3] << 16);
    }
    if (tid < kHid) {
        S.b1[tid] = bf16_to_f32(w[kB1 + tid]);
        S.b2[tid] = bf16_to_f32(w[kB2 + tid]);
    }
    if (tid < 64) {
        const int o = out_of(tid >> 4, (tid >> 2) & 3, tid & 3);
        S.b3[tid] = o >= 0 ? bf16_to_f32(w[kB3 + o]) : 0.f;
    }
    if constexpr (BACK)
        if (tid < (int)kSumBlocks) S.red[tid] = part;
    __syncthreads();
    if constexpr (BACK)
        if (tid < 64) {
            double v = (S.red[tid] + S.red[tid + 128]) + (S.red[tid + 64] + S.red[tid + 192]);
            for (int h = 32; h > 0; h >>= 1) v += __shfl_down(v, h, 64);
            if (tid == 0) S.red[0] = v;
        }
    for (int p = tid; p < 8 * 4 * 64; p += kStripThreads) {
        const int r = p & 15, q = (p >> 4) & 3, u = (p >> 6) & 3, t = p >> 8, m = row_of<K32>(t, r >> 2, r & 3);
        uint32_t e[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) e[i] = raw[row_of<K32>(2 * u + (i >> 2), q, i & 3) * kRawRow + m];
        S.w2[p] = make_uint4(e[0] | e[1] << 16, e[2] | e[3] << 16, e[4] | e[5] << 16, e[6] | e[7] << 16);
        if constexpr (BACK) {
            const uint2 x = *(const uint2 *)(raw + m * kRawRow + row_of<K32>(2 * u, q, 0));
            const uint2 y = *(const uint2 *)(raw + m * kRawRow + row_of<K32>(2 * u + 1, q, 0));
            S.w2b[p] = make_uint4(x.x, x.y, y.x, y.y);
        }
    }
    for (int p = tid; p < 4 * 4 * 64; p += kStripThreads) {
        const int r = p & 15, q = (p >> 4) & 3, u = (p >> 6) & 3, t = p >> 8, o = out_of(t, r >> 2, r & 3);
        uint32_t e[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) e[i] = o >= 0 ? raw3[row_of<K32>(2 * u + (i >> 2), q, i & 3) * kOut + o] : 0;
        S.w3[p] = make_uint4(e[0] | e[1] << 16, e[2] | e[3] << 16, e[4] | e[5] << 16, e[6] | e[7] << 16);
    }
    if constexpr (BACK)
        for (int p = tid; p < 8 * 2 * 64; p += kStripThreads) {
            const int r = p & 15, q = (p >> 4) & 3, u = (p >> 6) & 1, t = p >> 7, m = row_of<K32>(t, r >> 2, r & 3);
            uint32_t e[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int o = out_of(2 * u + (i >> 2), q, i & 3);
                e[i] = o >= 0 ? raw3[m * kOut + o] : 0;
            }
            S.w3b[p] = make_uint4(e[0] | e[1] << 16, e[2] | e[3] << 16, e[4] | e[5] << 16, e[6] | e[7] << 16);
        }
    __syncthreads();
}

// A hidden layer's activations of tile t: pre-activation z = c + b, h =
// silu(z) and (for the way back) dh = silu'(z).
template <bool BACK>
__device__ __forceinline__ uint2 activate(v4f c, const float *bias, v4f &z, v4f &dh) {
    const float4 b = *(const float4 *)bias;
    const float bb[4] = {b.x, b.y, b.z, b.w};
    v4f h;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        z[j] = c[j] + bb[j];
        const float s = frcp(1.0f + fexp(-z[j]));
        h[j] = z[j] * s;
        if constexpr (BACK) dh[j] = s * (1.0f + z[j] * (1.0f - s));
    }
    return pack4(h);
}

// The value again, as one the compiler knows nothing of: LDS addresses are
// computed where they are used instead of held in registers for the pass.
__device__ __forceinline__ int fresh(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// Keeps the scheduler from starting every tile's loads at once (they would not
// fit in the registers): two tiles at a time.
__device__ __forceinline__ void fence(int t) {
    if (t % 2 == 0) __builtin_amdgcn_sched_barrier(0);
}

template <StripMode MODE>
__global__ __launch_bounds__(kStripThreads) void k_strip(StripArgs f) {
    constexpr bool BACK = MODE == kGradient || MODE == kTraining, K32 = MODE == kTraining;
    constexpr bool LAYERS = MODE == kForward || MODE == kGradient;
    __shared__ StripLds<BACK> S;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, r = lane & 15, q = lane >> 4;
    stage_weights<K32>(f.w, f.wsum, S, tid);
    double wsum = 0.0;
    if constexpr (BACK) wsum = S.red[0];
    if constexpr (LAYERS) {  // the workspace's transposed weights, a share per work-group
        for (int i = blockIdx.x * kStripThreads + tid; i < kHid * kHid; i += gridDim.x * kStripThreads)
            f.wt[kW2 + (i % kHid) * kHid + i / kHid] = f.w[kW2 + i];
        for (int i = blockIdx.x * kStripThreads + tid; i < kHid * kOut; i += gridDim.x * kStripThreads)
            f.wt[kW3 + (i % kOut) * kHid + i / kOut] = f.w[kW3 + i];
        for (int i = blockIdx.x * kStripThreads + tid; i < kIn * kHid; i += gridDim.x * kStripThreads)
            f.wt[kW1 + (i % kHid) * kIn + i / kHid] = f.w[kW1 + i];
    }

    uint16_t *t0 = S.t, *t1 = t0 + kHid * kPassRows;
    const int row = 16 * wave + r;  // of the pass
    // weight gradients: wave w has rows [16 w, 16 w + 16) of W2 and W3 and
    // columns [16 w, 16 w + 16) of W1
    v4f acc1 = {0.f, 0.f, 0.f, 0.f}, acc2[8], acc3[4];
#pragma unroll
    for (int t = 0; t < 8; ++t) acc2[t] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 4; ++t) acc3[t] = v4f{0.f, 0.f, 0.f, 0.f};
    float db1[2] = {0.f, 0.f}, db2[2] = {0.f, 0.f}, db3 = 0.f;
    double loss_acc = 0.0;

    for (uint64_t base = (uint64_t)blockIdx.x * kPassRows; base < f.cnt; base += (uint64_t)gridDim.x * kPassRows) {
        const uint64_t tile = base + 16 * wave, i = tile + r;
        const bool live = i < f.cnt;  // rows past the batch repeat its first row with weight 0
        uint64_t src = live ? i : 0;
        if constexpr (MODE == kTraining) src = ((f.a * (f.first + src)) % f.n_data + f.b) % f.n_data;
        uint2 x = make_uint2(0, 0);
        if (q < 2) {
            const float *c = f.ctx + src * kIn + 4 * q;
            x.x = pack2(c[0], c[1]);
            if (q == 0) x.y = pack2(c[2], c[3]);
        }
        float y[3], a = 0.f;
        if constexpr (BACK) {
            double yd[3];
            for (int d = 0; d < 3; ++d) yd[d] = f.y[src * 3 + d];
            const double om = f.omega[src];
            if (live) a = (float)(om / wsum);
            for (int d = 0; d < 3; ++d) y[d] = (float)yd[d];
            if constexpr (LAYERS)
                if (live && q == 0) {
                    for (int d = 0; d < 3; ++d) f.Y[i * 3 + d] = yd[d];
                    f.W[i] = om;
                }
        }
        if constexpr (LAYERS)
            if (live && q < 2) {
                uint32_t *X = (uint32_t *)(f.X + i * kIn);
                X[2 * q] = x.x;
                if (q == 0) X[1] = x.y;
            }

        // layer 1 (K = 6, padded with zeros)
        uint2 h[8], h2[8];
        v4f g1[BACK ? 8 : 1], g2[BACK ? 8 : 1];
        uint4 a1[4];
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            fence(t);
            const v4f c = mfma16(S.w1[t * 64 + lane], x, v4f{0.f, 0.f, 0.f, 0.f});
            const int k = row_of<K32>(t, q, 0);
            v4f z, dh;
            h[t] = activate<BACK>(c, S.b1 + k, z, dh);
            if constexpr (BACK) g1[t] = dh;
            if constexpr (LAYERS)
                if (live) {
                    *(v4f *)(f.Z1 + tile * kHid + (uint32_t)(r * kHid + k)) = z;
                    *(uint2 *)(f.H1 + tile * kHid + (uint32_t)(r * kHid + k)) = h[t];
                }
        }
        if constexpr (BACK) {
            const int fq = fresh(q), frow = fresh(row);
#pragma unroll
            for (int t = 0; t < 8; ++t) put4(t0, row_of<K32>(t, fq, 0), frow, h[t]);
            __syncthreads();
#pragma unroll
            for (int s = 0; s < 4; ++s) a1[s] = chunk(t0, frow, 4 * s + fq);  // value 16 w + r of H1
        }
        // layer 2
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            fence(t);
            v4f c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int u = 0; u < 4; ++u) c = mfma_pair<K32>(S.w2[(t * 4 + u) * 64 + lane], h[2 * u], h[2 * u + 1], c);
            const int k = row_of<K32>(t, q, 0);
            v4f z, dh;
            h2[t] = activate<BACK>(c, S.b2 + k, z, dh);
            if constexpr (BACK) g2[t] = dh;
            if constexpr (LAYERS)
                if (live) {
                    *(v4f *)(f.Z2 + tile * kHid + (uint32_t)(r * kHid + k)) = z;
                    *(uint2 *)(f.H2 + tile * kHid + (uint32_t)(r * kHid + k)) = h2[t];
                }
        }
        if constexpr (BACK) {
            __syncthreads();  // every wave has its part of H1
            const int fq = fresh(q), frow = fresh(row);
#pragma unroll
            for (int t = 0; t < 8; ++t) put4(t0, row_of<K32>(t, fq, 0), frow, h2[t]);
        }
        // layer 3
        float o[2][7];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            fence(t);
            v4f c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int u = 0; u < 4; ++u) c = mfma_pair<K32>(S.w3[(t * 4 + u) * 64 + lane], h2[2 * u], h2[2 * u + 1], c);
            const float4 b = *(const float4 *)(S.b3 + 16 * t + 4 * q);
            const float bb[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (4 * t + j < 14) o[(4 * t + j) / 7][(4 * t + j) % 7] = c[j] + bb[j];
        }
        if constexpr (MODE != kTraining)
            if (live) {
                float *po = MODE == kGradient ? f.O : f.out;
#pragma unroll
                for (int k = 0; k < 7; ++k) {
                    const float2 v = make_float2(o[2 * k / 7][2 * k % 7], o[(2 * k + 1) / 7][(2 * k + 1) % 7]);
                    __builtin_memcpy(po + tile * kOut + (uint32_t)(r * kOut + 14 * q + 2 * k), &v, 8);
                    if constexpr (MODE == kForward) *(float2 *)(f.O + tile * kOut + (uint32_t)(r * kOut + 14 * q + 2 * k)) = v;
                }
            }
        if constexpr (BACK) {
            float g[2][7], loss;
            head_rows(o, y, a, f.lo, f.hi, g, loss);
            if (q == 0) {
                loss_acc += (double)loss;
                if constexpr (LAYERS)
                    if (live) f.row_loss[i] = (double)loss;
            }
            float d[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) d[k] = k < 14 ? g[k / 7 & 1][k % 7] : 0.f;
            uint2 dp[4];
            const int fq = fresh(q), frow = fresh(row), fr = fresh(r);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                dp[t] = make_uint2(pack2(d[4 * t], d[4 * t + 1]), pack2(d[4 * t + 2], d[4 * t + 3]));
                put4(t1, 16 * t + 4 * fq, frow, dp[t]);
            }
            if constexpr (LAYERS)
                if (live) {
#pragma unroll
                    for (int k = 0; k < 7; ++k) {
                        *(float2 *)(f.dO + tile * kOut + (uint32_t)(r * kOut + 14 * q + 2 * k)) = make_float2(d[2 * k], d[2 * k + 1]);
                        *(uint32_t *)(f.dOh + tile * kOut + (uint32_t)(r * kOut + 14 * q + 2 * k)) = k & 1 ? dp[k >> 1].y : dp[k >> 1].x;
                    }
                }
            scatter_sum<16>(d, r);
            db3 += d[0];
            __syncthreads();
            // dW3 += H2^T dO over the pass's rows
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                fence(s);
                const uint4 a2 = chunk(t0, frow, 4 * s + fq);
#pragma unroll
                for (int t = 0; t < 4; ++t) acc3[t] = mfma32(a2, chunk(t1, 16 * t + fr, 4 * s + fq), acc3[t]);
            }
            __syncthreads();  // every wave has read H2
            // dZ2 = (dO W3^T) * silu'(Z2), its column sums (bias 2)
            float cs[32];
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                fence(t);
                v4f c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int u = 0; u < 2; ++u) c = mfma_pair<K32>(S.w3b[(t * 2 + u) * 64 + lane], dp[2 * u], dp[2 * u + 1], c);
#pragma unroll
                for (int j = 0; j < 4; ++j) cs[4 * t + j] = c[j] = c[j] * g2[t][j];
                const int k = row_of<K32>(t, q, 0);
                h2[t] = pack4(c);
                put4(t0, row_of<K32>(t, fq, 0), frow, h2[t]);
                if constexpr (LAYERS)
                    if (live) {
                        *(v4f *)(f.dZ2 + tile * kHid + (uint32_t)(r * kHid + k)) = c;
                        *(uint2 *)(f.dZ2h + tile * kHid + (uint32_t)(r * kHid + k)) = h2[t];
                    }
            }
            scatter_sum<32>(cs, r);
            db2[0] += cs[0];
            db2[1] += cs[1];
            __syncthreads();
            // dW2 += H1^T dZ2
            const int gq = fresh(q), gr = fresh(r);
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int t = 0; t < 8; ++t) acc2[t] = mfma32(a1[s], chunk(t0, 16 * t + gr, 4 * s + gq), acc2[t]);
            }
            // dZ1 = (dZ2 W2^T) * silu'(Z1), its column sums (bias 1)
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                fence(t);
                v4f c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    c = mfma_pair<K32>(S.w2b[(t * 4 + u) * 64 + lane], h2[2 * u], h2[2 * u + 1], c);
#pragma unroll
                for (int j = 0; j < 4; ++j) cs[4 * t + j] = c[j] = c[j] * g1[t][j];
                const int k = row_of<K32>(t, q, 0);
                h[t] = pack4(c);
                if constexpr (LAYERS)
                    if (live) {
                        *(v4f *)(f.dZ1 + tile * kHid + (uint32_t)(r * kHid + k)) = c;
                        *(uint2 *)(f.dZ1h + tile * kHid + (uint32_t)(r * kHid + k)) = h[t];
                    }
            }
            scatter_sum<32>(cs, r);
            db1[0] += cs[0];
            db1[1] += cs[1];
            __syncthreads();  // every wave has read dO and dZ2
            const int eq = fresh(q), erow = fresh(row);
#pragma unroll
            for (int t = 0; t < 8; ++t) put4(t0, row_of<K32>(t, eq, 0), erow, h[t]);
            put4(t1, 4 * eq, erow, x);
            __syncthreads();
            // dW1 += X^T dZ1
#pragma unroll
            for (int s = 0; s < 4; ++s)
                acc1 = mfma32(chunk(t1, erow & 15, 4 * s + eq), chunk(t0, erow, 4 * s + eq), acc1);
            __syncthreads();
        }
    }

    if constexpr (BACK) {
        // the group's partial gradient, in the parameter layout
        float *P = f.part + (uint64_t)blockIdx.x * kParams;
#pragma unroll
        for (int t = 0; t < 8; ++t)
            for (int j = 0; j < 4; ++j) P[kW2 + (16 * wave + 4 * q + j) * kHid + 16 * t + r] = acc2[t][j];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int n = out_of(t, r >> 2, r & 3);
            if (n >= 0)
                for (int j = 0; j < 4; ++j) P[kW3 + (16 * wave + 4 * q + j) * kOut + n] = acc3[t][j];
        }
        for (int j = 0; j < 4; ++j)
            if (4 * q + j < kIn) P[kW1 + (4 * q + j) * kHid + 16 * wave + r] = acc1[j];
        // the waves' bias sums and losses
        float *sb = (float *)t0;                    // 8 x (128 + 128 + 64)
        double *sl = (double *)(sb + kWaves * 320);   // 8 x 16
        for (int e = 0; e < 2; ++e) {
            const int n = row_of<K32>(r >> 1, q, 2 * (r & 1) + e);
            sb[wave * 320 + n] = db1[e];
            sb[wave * 320 + kHid + n] = db2[e];
        }
        sb[wave * 320 + 2 * kHid + 16 * (r >> 2) + 4 * q + (r & 3)] = db3;
        if (q == 0) sl[wave * 16 + r] = loss_acc;
        __syncthreads();
        if (tid < 320) {
            float v = 0.f;
            for (int u = 0; u < kWaves; ++u) v += sb[u * 320 + tid];
            if (tid < kHid) {
                P[kB1 + tid] = v;
            } else if (tid < 2 * kHid) {
                P[kB2 + tid - kHid] = v;
            } else {
                const int s = tid - 2 * kHid, n = out_of(s >> 4, (s >> 2) & 3, s & 3);
                if (n >= 0) P[kB3 + n] = v;
            }
        }
        for (int h = kWaves * 8; h > 0; h >>= 1) {
            if (tid < h) sl[tid] += sl[tid + h];
            __syncthreads();
        }
        if (tid == 0) f.loss_part[blockIdx.x] = sl[0];
    }
}

// Sums of omega over the batches of consecutive steps (step = blockIdx.y, the
// batch's rows in their shuffled order), kSumBlocks partials a step.
__global__ __launch_bounds__(kThreads) void k_batch_wsum(const double *omega, uint64_t n_data, uint64_t a, uint64_t b,
                                                         uint64_t first, uint64_t batch, double *partial) {
    __shared__ double red[kThreads];
    first += blockIdx.y * batch;
    const uint64_t cnt = batch < n_data - first ? batch : n_data - first;
    double s = 0.0;
    for (uint64_t i = (uint64_t)blockIdx.x * kThreads + threadIdx.x; i < cnt; i += (uint64_t)gridDim.x * kThreads)
        s += omega[((a * (first + i)) % n_data + b) % n_data];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = kThreads / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[(uint64_t)blockIdx.y * gridDim.x + blockIdx.x] = red[0];
}

// gradient = the groups' partials summed in a fixed order (sixteen threads per
// four parameters each sum every sixteenth group, then their sums in order),
// then (ADAM) one Adam step; the loss (nullable) = the sum of the groups'.
// Bound by reading the partials, 25 MB at 256 groups, which the other XCDs
// wrote: a thread's 16 loads of 16 bytes are in flight together (7 us; 12 to 23 us
// with a parameter a thread and its loads one after another).
constexpr int kReduceParams = 64;  // parameters per work-group
constexpr unsigned kReduceGroups = (unsigned)((kParams + kReduceParams - 1) / kReduceParams);
static_assert(kParams % 4 == 0, "four parameters a thread");

struct AdamArgs {
    float *theta;
    uint16_t *wb;
    float *m, *v;
    float lr, b1, b2, eps, c1, c2;
};

template <bool ADAM>
__global__ __launch_bounds__(kThreads) void k_reduce(const float *part, int groups, float *grad, AdamArgs A,
                                                     const double *loss_part, double *loss) {
    __shared__ float red[16][kReduceParams];
    __shared__ double rl[kGroupsMax];
    const int sub = threadIdx.x >> 4, c = (threadIdx.x & 15) * 4;
    const uint64_t p4 = (uint64_t)blockIdx.x * kReduceParams + c;
    // a parameter a thread in the end; its Adam state arrives beside the partials
    const uint64_t p = (uint64_t)blockIdx.x * kReduceParams + threadIdx.x;
    const bool mine = threadIdx.x < kReduceParams && p < kParams;
    float m0 = 0.f, v0 = 0.f, t0 = 0.f;
    if constexpr (ADAM)
        if (mine) m0 = A.m[p], v0 = A.v[p], t0 = A.theta[p];
    v4f acc = {0.f, 0.f, 0.f, 0.f};
    if (p4 < kParams) {
        v4f v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u)
            v[u] = sub + 16 * u < groups ? *(const v4f *)(part + (uint64_t)(sub + 16 * u) * kParams + p4)
                                         : v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < 16; ++u) acc += v[u];
    }
    *(v4f *)&red[sub][c] = acc;
    if (loss && blockIdx.x == 0) {
        static_assert(kGroupsMax == kThreads, "a partial loss per thread");
        rl[threadIdx.x] = (int)threadIdx.x < groups ? loss_part[threadIdx.x] : 0.0;
        __syncthreads();
        for (int w = kThreads / 2; w > 0; w >>= 1) {
            if ((int)threadIdx.x < w) rl[threadIdx.x] += rl[threadIdx.x + w];
            __syncthreads();
        }
        if (threadIdx.x == 0) *loss = rl[0];
    }
    __syncthreads();
    if (!mine) return;
    float gi = 0.f;
#pragma unroll
    for (int u = 0; u < 16; ++u) gi += red[u][threadIdx.x];
    grad[p] = gi;
    if constexpr (ADAM) {
        const float mi = A.b1 * m0 + (1.f - A.b1) * gi;
        const float vi = A.b2 * v0 + (1.f - A.b2) * gi * gi;
        A.m[p] = mi;
        A.v[p] = vi;
        const float t = t0 - A.lr * (mi * A.c1) / (sqrtf(vi * A.c2) + A.eps);
        A.theta[p] = t;
        A.wb[p] = f32_to_bf16(t);
    }
}

// Training weights omega_i = w_i / max(I_b, floor), I_b = sum_w[b] / n_emitted
// the bin's estimated intensity, floor = floor_frac * (mean I over bins with
// hits): every live bin gets equal total weight, the proposal that makes the
// per-bin relative errors equal when weights within a bin are alike.
constexpr int kRunsMax = 16;  // runs a launch serves
struct RunTable {
    const double *image[kRunsMax];   // null: a run without rows
    uint64_t first[kRunsMax + 1];    // rows [first[r], first[r + 1]) are run r's
};

// The sum and count of the live bins of a run's image (run = blockIdx.y), a
// partial pair per work-group.  Bound by reading the images; eight loads of a
// thread are in flight together.
__global__ __launch_bounds__(kThreads) void k_bin_stats(RunTable t, uint64_t n_bins, double *partial) {
    __shared__ double rs[kThreads], rc[kThreads];
    const double *image = t.image[blockIdx.y];
    if (!image) return;
    double s = 0.0, c = 0.0;
    const uint64_t stride = (uint64_t)gridDim.x * kThreads;
    for (uint64_t i = (uint64_t)blockIdx.x * kThreads + threadIdx.x; i < n_bins; i += 8 * stride) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = i + u * stride < n_bins ? image[i + u * stride] : 0.0;
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (v[u] > 0.0) {
                s += v[u];
                c += 1.0;
            }
    }
    rs[threadIdx.x] = s;
    rc[threadIdx.x] = c;
    __syncthreads();
    for (int w = kThreads / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            rs[threadIdx.x] += rs[threadIdx.x + w];
            rc[threadIdx.x] += rc[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        double *p = partial + 2 * ((uint64_t)blockIdx.y * gridDim.x + blockIdx.x);
        p[0] = rs[0];
        p[1] = rc[0];
    }
}

// Every work-group sums its run's partial pairs itself (in one fixed order):
// a launch of one work-group for it took 21 us a run.
__global__ __launch_bounds__(kThreads) void k_train_weights(const double *w, const int64_t *bin, RunTable t,
                                                            uint64_t n_bins, const double *partial, double floor_frac,
                                                            double *omega) {
    static_assert(kSumBlocks == kThreads, "a partial pair per thread");
    __shared__ double rs[kThreads], rc[kThreads];
    const double *image = t.image[blockIdx.y];
    if (!image) return;
    const double *p = partial + 2 * ((uint64_t)blockIdx.y * kSumBlocks + threadIdx.x);
    rs[threadIdx.x] = p[0];
    rc[threadIdx.x] = p[1];
    __syncthreads();
    for (int h = kThreads / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) {
            rs[threadIdx.x] += rs[threadIdx.x + h];
            rc[threadIdx.x] += rc[threadIdx.x + h];
        }
        __syncthreads();
    }
    const double mean_live = rc[0] > 0.0 ? rs[0] / rc[0] : 0.0;  // mean sum_w over bins with hits
    const uint64_t end = t.first[blockIdx.y + 1];
    for (uint64_t i = t.first[blockIdx.y] + (uint64_t)blockIdx.x * kThreads + threadIdx.x; i < end;
         i += (uint64_t)gridDim.x * kThreads) {
        const int64_t b = bin[i];
        const double Ib = (b >= 0 && (uint64_t)b < n_bins) ? image[b] : 0.0;
        const double den = fmax(Ib, floor_frac * mean_live);
        omega[i] = den > 0.0 ? w[i] / den : 0.0;
    }
}

// Work-groups for n items of a grid-stride kernel: at most 2^22 (the HSA
// dispatch counts a grid's work-items with 32 bits), each item reached by the
// kernel's stride loop.
unsigned blocks_for(uint64_t n) {
    return (unsigned)std::min<uint64_t>(1ull << 22, std::max<uint64_t>(1, (n + kThreads - 1) / kThreads));
}
// ------------------------------------------------------------ workspace --

struct Layout {
    uint64_t off[MXR_MLP_WS_REGIONS];
    uint64_t bytes;
};

uint64_t splits_for(uint64_t n) { return std::max<uint64_t>(1, (n + kSplitRows - 1) / kSplitRows); }

Layout layout_for(uint64_t n) {
    const uint64_t sizes[MXR_MLP_WS_REGIONS] = {
        n * kIn * 2,                    // X (bf16)
        n * kHid * 4, n * kHid * 2,     // Z1, H1
        n * kHid * 4, n * kHid * 2,     // Z2, H2
        n * kOut * 4,                   // O
        n * kOut * 4, n * kOut * 2,     // dO, dO (bf16)
        n * kHid * 4, n * kHid * 2,     // dZ2, dZ2 (bf16)
        n * kHid * 4, n * kHid * 2,     // dZ1, dZ1 (bf16)
        // partial gradients: at most kGroupsMax are written (the size callers have
        // been told is kept)
        std::max<uint64_t>(splits_for(n), kGroupsMax) * kParams * 4,
        n * 3 * 8, n * 8, n * 8,        // gathered targets, weights, per-row loss
        (kSumBlocks + 2) * 8,           // partial sums of the weights
        kParams * 2,                    // W^T copies (bf16), same offsets as W
        // the work-groups' losses, a double each (the size callers have been told is kept)
        ((n + 15) / 16 * kHid * 2 + (n + 7) / 8 * kOut) * 4,
    };
    Layout L;
    uint64_t o = 0;
    for (int i = 0; i < MXR_MLP_WS_REGIONS; ++i) {
        L.off[i] = o;
        o += (sizes[i] + 255) / 256 * 256;
    }
    L.bytes = o;
    return L;
}

template <class T>
T *at(void *ws, const Layout &L, int region) {
    return (T *)((char *)ws + L.off[region]);
}

mxr_status check_device_ptrs(std::initializer_list<const void *> ps) {
    for (const void *p : ps)
        if (!p) return fail(MXR_E_INVALID, "null array");
    return MXR_OK;
}

// The layer-value pointers of k_strip into a workspace of n rows.
void layer_values(StripArgs &a, void *ws, const Layout &L) {
    a.X = at<uint16_t>(ws, L, MXR_MLP_WS_X);
    a.Z1 = at<float>(ws, L, MXR_MLP_WS_Z1);
    a.H1 = at<uint16_t>(ws, L, MXR_MLP_WS_H1);
    a.Z2 = at<float>(ws, L, MXR_MLP_WS_Z2);
    a.H2 = at<uint16_t>(ws, L, MXR_MLP_WS_H2);
    a.O = at<float>(ws, L, MXR_MLP_WS_O);
    a.wt = at<uint16_t>(ws, L, MXR_MLP_WS_WT);
}

// Work-groups for n rows: one per 128, at most one per compute unit (the
// weights are staged once per work-group).
unsigned strip_groups(uint64_t n) { return (unsigned)std::min<uint64_t>(kGroupsMax, (n + kPassRows - 1) / kPassRows); }

StripArgs strip_args(const uint16_t *w, const float *ctx, uint64_t n) {
    StripArgs a{};
    a.w = w;
    a.ctx = ctx;
    a.n_data = a.cnt = n;
    a.a = 1;
    return a;
}

// omega of the rows of up to kRunsMax runs (rows: the longest run's)
mxr_status train_weights(const double *w, const int64_t *bin, const RunTable &t, unsigned runs, uint64_t rows,
                         uint64_t n_bins, double floor_frac, double *omega, double *scratch, hipStream_t st) {
    hipLaunchKernelGGL(k_bin_stats, dim3(kSumBlocks, runs), dim3(kThreads), 0, st, t, n_bins, scratch);
    hipLaunchKernelGGL(k_train_weights, dim3(std::min(blocks_for(rows), 1024u), runs), dim3(kThreads), 0, st, w, bin, t,
                       n_bins, (const double *)scratch, floor_frac, omega);
    return launch_check("training weights");
}

mxr_status box_ok(const double lo[3], const double hi[3], float flo[3], float fhi[3]) {
    if (!lo || !hi) return fail(MXR_E_INVALID, "null box");
    for (int d = 0; d < 3; ++d) {
        if (!std::isfinite(lo[d]) || !std::isfinite(hi[d]) || !(hi[d] > lo[d]))
            return fail(MXR_E_INVALID, "box edge %d: need finite lo < hi", d);
        flo[d] = (float)lo[d];
        fhi[d] = (float)hi[d];
    }
    return MXR_OK;
}

}  // namespace

extern "C" {

uint64_t mxr_mlp_workspace_bytes(uint64_t batch) { return layout_for(batch).bytes; }

mxr_status mxr_mlp_workspace_layout(uint64_t batch, uint64_t *offsets) {
    if (!offsets) return fail(MXR_E_INVALID, "null offsets");
    const Layout L = layout_for(batch);
    for (int i = 0; i < MXR_MLP_WS_REGIONS; ++i) offsets[i] = L.off[i];
    return MXR_OK;
}

mxr_status mxr_mlp_to_bf16(const float *x, uint64_t n, uint16_t *y, void *hip_stream) {
    if (n == 0) return MXR_OK;
    if (!x || !y) return fail(MXR_E_INVALID, "null array");
    hipLaunchKernelGGL(k_to_bf16, dim3(blocks_for(n)), dim3(kThreads), 0, (hipStream_t)hip_stream, x, n, y);
    return launch_check("bfloat16 conversion");
}

mxr_status mxr_mlp_forward(const uint16_t *w, const float *ctx, uint64_t n, float *out, void *ws, uint64_t ws_bytes,
                           void *hip_stream) {
    if (n == 0) return MXR_OK;
    mxr_status s = check_device_ptrs({w, ctx, out, ws});
    if (s != MXR_OK) return s;
    const Layout L = layout_for(n);
    if (ws_bytes < L.bytes) return fail(MXR_E_INVALID, "workspace of %llu bytes, %llu needed", (unsigned long long)ws_bytes, (unsigned long long)L.bytes);
    StripArgs a = strip_args(w, ctx, n);
    layer_values(a, ws, L);
    a.out = out;
    hipLaunchKernelGGL(k_strip<kForward>, dim3(strip_groups(n)), dim3(kStripThreads), 0, (hipStream_t)hip_stream, a);
    return launch_check("network forward");
}

mxr_status mxr_mlp_forward_noalloc(const uint16_t *w, const float *ctx, uint64_t n, float *out, void *hip_stream) {
    if (n == 0) return MXR_OK;
    mxr_status s = check_device_ptrs({w, ctx, out});
    if (s != MXR_OK) return s;
    if (n > MXR_MLP_NOALLOC_ROWS)
        return fail(MXR_E_INVALID, "%llu rows: the allocation-free forward takes at most %llu rows per call",
                    (unsigned long long)n, (unsigned long long)MXR_MLP_NOALLOC_ROWS);
    StripArgs a = strip_args(w, ctx, n);
    a.out = out;
    hipLaunchKernelGGL(k_strip<kForwardOnly>, dim3(strip_groups(n)), dim3(kStripThreads), 0, (hipStream_t)hip_stream, a);
    return launch_check("network forward");
}

mxr_status mxr_mlp_mixture(const float *out, uint64_t n, const double lo[3], const double hi[3], double *gmm,
                           void *hip_stream) {
    if (n == 0) return MXR_OK;
    float flo[3], fhi[3];
    mxr_status s = box_ok(lo, hi, flo, fhi);
    if (s != MXR_OK) return s;
    if ((s = check_device_ptrs({out, gmm})) != MXR_OK) return s;
    hipLaunchKernelGGL(k_head_params, dim3(blocks_for(8 * n)), dim3(kThreads), 0, (hipStream_t)hip_stream, out, n,
                       flo[0], flo[1], flo[2], fhi[0], fhi[1], fhi[2], gmm);
    return launch_check("mixture head");
}

mxr_status mxr_mlp_loss_grad(const uint16_t *w, const float *ctx, const double *y, const double *omega, uint64_t n,
                             const double lo[3], const double hi[3], float *grad, double *loss, void *ws,
                             uint64_t ws_bytes, void *hip_stream) {
    if (n == 0) return fail(MXR_E_INVALID, "empty batch");
    float flo[3], fhi[3];
    mxr_status s = box_ok(lo, hi, flo, fhi);
    if (s != MXR_OK) return s;
    if ((s = check_device_ptrs({w, ctx, y, omega, grad, ws})) != MXR_OK) return s;
    const Layout L = layout_for(n);
    if (ws_bytes < L.bytes) return fail(MXR_E_INVALID, "workspace of %llu bytes, %llu needed", (unsigned long long)ws_bytes, (unsigned long long)L.bytes);
    if (n > ((1ull << 32) - kThreads) / 8)
        return fail(MXR_E_UNSUPPORTED, "%llu rows: at most 2^29 - 32 rows per gradient", (unsigned long long)n);
    hipStream_t st = (hipStream_t)hip_stream;
    double *wsum = at<double>(ws, L, MXR_MLP_WS_SCALARS);
    hipLaunchKernelGGL(k_sum_f64, dim3(kSumBlocks), dim3(kThreads), 0, st, omega, n, wsum);
    StripArgs a = strip_args(w, ctx, n);
    layer_values(a, ws, L);
    a.y = y;
    a.omega = omega;
    a.wsum = wsum;
    for (int d = 0; d < 3; ++d) {
        a.lo[d] = flo[d];
        a.hi[d] = fhi[d];
    }
    a.dO = at<float>(ws, L, MXR_MLP_WS_DO);
    a.dOh = at<uint16_t>(ws, L, MXR_MLP_WS_DOH);
    a.dZ2 = at<float>(ws, L, MXR_MLP_WS_DZ2);
    a.dZ2h = at<uint16_t>(ws, L, MXR_MLP_WS_DZ2H);
    a.dZ1 = at<float>(ws, L, MXR_MLP_WS_DZ1);
    a.dZ1h = at<uint16_t>(ws, L, MXR_MLP_WS_DZ1H);
    a.Y = at<double>(ws, L, MXR_MLP_WS_Y);
    a.W = at<double>(ws, L, MXR_MLP_WS_W);
    a.row_loss = at<double>(ws, L, MXR_MLP_WS_ROWLOSS);
    a.part = at<float>(ws, L, MXR_MLP_WS_PARTIAL);
    a.loss_part = at<double>(ws, L, MXR_MLP_WS_COLS);
    const int groups = (int)strip_groups(n);
    hipLaunchKernelGGL(k_strip<kGradient>, dim3(groups), dim3(kStripThreads), 0, st, a);
    hipLaunchKernelGGL(k_reduce<false>, dim3(kReduceGroups), dim3(kThreads), 0, st, (const float *)a.part, groups, grad,
                       AdamArgs{}, (const double *)a.loss_part, loss);
    return launch_check("loss gradient");
}

mxr_status mxr_adam_step(float *master, uint16_t *w, const float *grad, float *m, float *v, uint64_t n_params,
                         uint32_t step, float lr, float beta1, float beta2, float eps, void *hip_stream) {
    if (n_params == 0) return MXR_OK;
    mxr_status s = check_device_ptrs({master, w, grad, m, v});
    if (s != MXR_OK) return s;
    if (step < 1) return fail(MXR_E_INVALID, "Adam steps count from 1");
    if (!(lr > 0.f) || !(beta1 >= 0.f && beta1 < 1.f) || !(beta2 >= 0.f && beta2 < 1.f) || !(eps >= 0.f))
        return fail(MXR_E_INVALID, "bad Adam hyper-parameters");
    const float c1 = (float)(1.0 / (1.0 - std::pow((double)beta1, (double)step)));
    const float c2 = (float)(1.0 / (1.0 - std::pow((double)beta2, (double)step)));
    hipLaunchKernelGGL(k_adam, dim3(blocks_for(n_params)), dim3(kThreads), 0, (hipStream_t)hip_stream, master, w, grad,
                       m, v, n_params, lr, beta1, beta2, eps, c1, c2);
    return launch_check("Adam");
}

mxr_status mxr_train_weights(const double *w, const int64_t *bin, uint64_t n, const double *sum_w, uint64_t n_bins,
                             double floor_frac, double *omega, double *scratch, void *hip_stream) {
    if (n == 0) return MXR_OK;
    mxr_status s = check_device_ptrs({w, bin, sum_w, omega, scratch});
    if (s != MXR_OK) return s;
    if (!(floor_frac >= 0.0) || !std::isfinite(floor_frac)) return fail(MXR_E_INVALID, "bad floor fraction");
    RunTable t{};
    t.image[0] = sum_w;
    t.first[1] = n;
    return train_weights(w, bin, t, 1, n, n_bins, floor_frac, omega, scratch, (hipStream_t)hip_stream);
}

mxr_status mxr_mlp_train(const float *ctx, const double *y, const double *omega, uint64_t n_rows,
                         const mxr_train_cfg *cfg, const double lo[3], const double hi[3], float *master, uint16_t *w,
                         float *m, float *v, float *grad, void *ws, uint64_t ws_bytes, double *loss_log,
                         void *hip_stream) {
    if (!cfg) return fail(MXR_E_INVALID, "null configuration");
    if (n_rows == 0) return fail(MXR_E_INVALID, "no training rows");
    if (cfg->batch == 0 || cfg->epochs == 0) return fail(MXR_E_INVALID, "batch and epochs must be positive");
    if (n_rows >= (1ull << 32)) return fail(MXR_E_UNSUPPORTED, "at most 2^32 - 1 training rows");
    float flo[3], fhi[3];
    mxr_status s = box_ok(lo, hi, flo, fhi);
    if (s != MXR_OK) return s;
    if ((s = check_device_ptrs({ctx, y, omega, master, w, m, v, grad, ws})) != MXR_OK) return s;
    const uint64_t B = std::min<uint64_t>(cfg->batch, n_rows);
    const Layout L = layout_for(B);
    if (ws_bytes < L.bytes) return fail(MXR_E_INVALID, "workspace of %llu bytes, %llu needed", (unsigned long long)ws_bytes, (unsigned long long)L.bytes);
    hipStream_t st = (hipStream_t)hip_stream;
    const uint64_t steps_per_epoch = (n_rows + B - 1) / B;
    // partial weight sums of as many steps as fit: behind the partial gradients
    // that batches of B rows write, or (if those fill their region) in the layer
    // values' space, which training leaves unused
    const uint64_t parts = strip_groups(B) * kParams * sizeof(float);
    const uint64_t behind = kGroupsMax * kParams * sizeof(float) - parts;
    const uint64_t layers = L.off[MXR_MLP_WS_PARTIAL] - L.off[MXR_MLP_WS_Z1];
    double *wsum = behind > layers ? (double *)(at<char>(ws, L, MXR_MLP_WS_PARTIAL) + parts) : at<double>(ws, L, MXR_MLP_WS_Z1);
    const uint64_t sum_steps = std::min<uint64_t>(65535, std::max(behind, layers) / (kSumBlocks * sizeof(double)));
    // per-epoch bijections i -> (a i + b) mod n_rows from a splitmix64 sequence
    uint64_t state = cfg->seed;
    auto next = [&state]() {
        uint64_t z = (state += 0x9E3779B97F4A7C15ull);
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        return z ^ (z >> 31);
    };
    auto gcd = [](uint64_t a, uint64_t b) {
        while (b) {
            const uint64_t t = a % b;
            a = b;
            b = t;
        }
        return a;
    };
    uint32_t step = cfg->first_step;
    for (uint32_t e = 0; e < cfg->epochs; ++e) {
        uint64_t a = 1, b = 0;
        if (n_rows > 1) {
            a = next() % n_rows;
            while (a == 0 || gcd(a, n_rows) != 1) a = (a + 1) % n_rows;
            b = next() % n_rows;
        }
        for (uint64_t k = 0; k < steps_per_epoch; ++k) {
            const uint64_t first = k * B, cnt = std::min<uint64_t>(B, n_rows - first);
            double *lp = loss_log ? loss_log + (uint64_t)e * steps_per_epoch + k : nullptr;
            ++step;
            if (!(cfg->lr > 0.f) || !(cfg->beta1 >= 0.f && cfg->beta1 < 1.f) ||
                !(cfg->beta2 >= 0.f && cfg->beta2 < 1.f) || !(cfg->eps >= 0.f))
                return fail(MXR_E_INVALID, "bad Adam hyper-parameters");
            if (k % sum_steps == 0) {
                const uint64_t steps = std::min<uint64_t>(sum_steps, steps_per_epoch - k);
                hipLaunchKernelGGL(k_batch_wsum, dim3(kSumBlocks, (unsigned)steps), dim3(kThreads), 0, st, omega, n_rows,
                                   a, b, first, B, wsum);
            }
            StripArgs fa = strip_args(w, ctx, cnt);
            fa.y = y;
            fa.omega = omega;
            fa.n_data = n_rows;
            fa.a = a;
            fa.b = b;
            fa.first = first;
            fa.wsum = wsum + (k % sum_steps) * kSumBlocks;
            for (int d = 0; d < 3; ++d) {
                fa.lo[d] = flo[d];
                fa.hi[d] = fhi[d];
            }
            fa.part = at<float>(ws, L, MXR_MLP_WS_PARTIAL);
            fa.loss_part = at<double>(ws, L, MXR_MLP_WS_ROWLOSS);
            const int groups = (int)strip_groups(cnt);
            hipLaunchKernelGGL(k_strip<kTraining>, dim3(groups), dim3(kStripThreads), 0, st, fa);
            const AdamArgs ad{master, w, m, v, cfg->lr, cfg->beta1, cfg->beta2, cfg->eps,
                              (float)(1.0 / (1.0 - std::pow((double)cfg->beta1, (double)step))),
                              (float)(1.0 / (1.0 - std::pow((double)cfg->beta2, (double)step)))};
            hipLaunchKernelGGL(k_reduce<true>, dim3(kReduceGroups), dim3(kThreads), 0, st, (const float *)fa.part, groups,
                               grad, ad, (const double *)fa.loss_part, lp);
            if ((s = launch_check("fused training step")) != MXR_OK) return s;
        }
    }
    return MXR_OK;
}

mxr_status mxr_proposal_train(const mxr_instrument *ins, const mxr_train_rows *rows, const mxr_train_cfg *cfg,
                              float *master, uint16_t *w, float *m, float *v, float *grad, double *omega, void *ws,
                              uint64_t ws_bytes, double *loss_log, void *hip_stream) {
    if (!rows || !cfg) return fail(MXR_E_INVALID, "null rows or configuration");
    double lo[3], hi[3];
    mxr_status s = mxr_proposal_box(ins, lo, hi);
    if (s != MXR_OK) return s;
    const mxr_train_rows &R = *rows;
    if (R.n_rows == 0) return fail(MXR_E_INVALID, "no training rows");
    if (R.n_runs == 0 || !R.run_first || !R.run_image) return fail(MXR_E_INVALID, "no run table");
    if (R.run_first[0] != 0 || R.run_first[R.n_runs] != R.n_rows)
        return fail(MXR_E_INVALID, "the run table must cover rows [0, n_rows)");
    if ((s = check_device_ptrs({R.ctx, R.y, R.w, R.bin, omega, ws})) != MXR_OK) return s;
    if (ws_bytes < (2 * kSumBlocks + 1) * sizeof(double))
        return fail(MXR_E_INVALID, "workspace of %llu bytes is too small", (unsigned long long)ws_bytes);
    for (uint32_t r = 0; r < R.n_runs; ++r) {
        const uint64_t a = R.run_first[r], b = R.run_first[r + 1];
        if (b < a || b > R.n_rows) return fail(MXR_E_INVALID, "run %u: rows [%llu, %llu) out of order", r,
                                               (unsigned long long)a, (unsigned long long)b);
        if (b > a && !R.run_image[r]) return fail(MXR_E_INVALID, "run %u: null image", r);
    }
    if (!(R.floor_frac >= 0.0) || !std::isfinite(R.floor_frac)) return fail(MXR_E_INVALID, "bad floor fraction");
    // the weight statistics use the start of the workspace; the training below
    // overwrites it only after these kernels (same stream)
    const uint32_t per = (uint32_t)std::min<uint64_t>(kRunsMax, ws_bytes / (2 * kSumBlocks * sizeof(double)));
    for (uint32_t r0 = 0; r0 < R.n_runs; r0 += per) {
        const uint32_t runs = std::min(per, R.n_runs - r0);
        RunTable t{};
        uint64_t rows = 0;
        for (uint32_t r = 0; r < runs; ++r) {
            const uint64_t a = R.run_first[r0 + r], b = R.run_first[r0 + r + 1];
            t.first[r] = a;
            t.first[r + 1] = b;
            t.image[r] = b > a ? R.run_image[r0 + r] : nullptr;
            rows = std::max(rows, b - a);
        }
        if (rows == 0) continue;
        if ((s = train_weights(R.w, R.bin, t, runs, rows, R.n_bins, R.floor_frac, omega, (double *)ws,
                               (hipStream_t)hip_stream)) != MXR_OK)
            return s;
    }
    return mxr_mlp_train(R.ctx, R.y, omega, R.n_rows, cfg, lo, hi, master, w, m, v, grad, ws, ws_bytes, loss_log,
                         hip_stream);
}

mxr_status mxr_proposal_apply(mxr_instrument *ins, const uint16_t *w, const float context[6], double alpha, void *ws,
                              uint64_t ws_bytes, void *hip_stream) {
    double lo[3], hi[3];
    mxr_status s = mxr_proposal_box(ins, lo, hi);
    if (s != MXR_OK) return s;
    if (!w || !context || !ws) return fail(MXR_E_INVALID, "null parameters, context or workspace");
    const uint64_t net_bytes = layout_for(1).bytes;
    if (ws_bytes < net_bytes + 1024)
        return fail(MXR_E_INVALID, "workspace of %llu bytes, %llu needed", (unsigned long long)ws_bytes,
                    (unsigned long long)(net_bytes + 1024));
    // after the network's workspace: the context (6 floats), the outputs
    // (56 floats) and the mixture (56 doubles)
    char *tail = (char *)ws + net_bytes;
    float *ctx = (float *)tail, *out = (float *)(tail + 64);
    double *gmm = (double *)(tail + 512);
    hipStream_t st = (hipStream_t)hip_stream;
    hipError_t e = hipMemcpyAsync(ctx, context, kIn * sizeof(float), hipMemcpyHostToDevice, st);
    if (e != hipSuccess) return fail(MXR_E_HIP, "copy of the context: %s", hipGetErrorString(e));
    if ((s = mxr_mlp_forward(w, ctx, 1, out, ws, net_bytes, hip_stream)) != MXR_OK) return s;
    if ((s = mxr_mlp_mixture(out, 1, lo, hi, gmm, hip_stream)) != MXR_OK) return s;
    e = hipStreamSynchronize(st);
    if (e != hipSuccess) return fail(MXR_E_HIP, "network forward: %s", hipGetErrorString(e));
    return mxr_proposal_set(ins, gmm, alpha);
}

}  // extern "C"

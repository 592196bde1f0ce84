// Angle predictor for the learned warm start: a multilayer perceptron
// in -> H -> H -> out (ReLU hidden layers, linear output) over per-subgraph
// features, trained with a mean-squared error on optimised angles. The
// paper motivates it only indirectly (Sec. 2.2: initialisation affects the
// quality and the iteration count of the angle optimisation).
//
// Parameters are FP64 master weights (updated by the FP64 Adam kernel);
// forward and backward arithmetic is FP32 with FP64 gradient accumulation.
// Flat layout, row-major: W1[H][in], b1[H], W2[H][H], b2[H], W3[out][H],
// b3[out]. Every reduction runs in a fixed order (bit-reproducible).
#include <mutex>

#include "lane.h"

namespace pq {

__host__ __device__ inline int64_t mlp_off_b1(const MlpDims& d) { return (int64_t)d.H * d.in; }
__host__ __device__ inline int64_t mlp_off_W2(const MlpDims& d) { return mlp_off_b1(d) + d.H; }
__host__ __device__ inline int64_t mlp_off_b2(const MlpDims& d) { return mlp_off_W2(d) + (int64_t)d.H * d.H; }
__host__ __device__ inline int64_t mlp_off_W3(const MlpDims& d) { return mlp_off_b2(d) + d.H; }
__host__ __device__ inline int64_t mlp_off_b3(const MlpDims& d) { return mlp_off_W3(d) + (int64_t)d.out * d.H; }
__host__ __device__ int64_t mlp_nparams(const MlpDims& d) { return mlp_off_b3(d) + d.out; }
int64_t mlp_num_params(const MlpDims& d) { return mlp_nparams(d); }

// Forward and error kernels of many samples (of few, k_mlp_fwd_sample and
// k_mlp_delta_sample below): a workgroup takes as many samples as its 1024
// threads can share (one per thread and unit), so every weight, read as FP64 and
// rounded to FP32 once per workgroup into LDS, serves all of them, along rows.
// (One workgroup per sample, each lane reading its own row, touched 64 cache
// lines per load.) The loads' latency is the bound: the first 16 K weights of
// both hidden layers are all on their way before the first is used. Every output
// is still one FP32 chain of fused multiply-adds in input order. Measured, 870
// samples of 18-128-128-6: forward 22 -> 15.5 us, errors 11.9 -> 11.3 us, weight
// gradients and loss 243 -> 17 us; 4000 samples of 64-256-256-12, a whole step
// 1965 -> 288 us.
constexpr int MLP_THREADS = 1024;
constexpr int MLP_LOADS = 16;  // weights a thread fetches at a time

// weight columns staged at a time for N units, and their row in LDS, padded so
// that 16-byte reads of 16 lanes meet all 64 banks
__host__ __device__ inline int mlp_chunk(int N) { return N <= 128 ? 128 : 64; }
__host__ __device__ inline int mlp_row(int N) { return mlp_chunk(N) + 4; }

// samples per workgroup
inline int mlp_samples(int H)
{
    int pad = 32;
    while (pad < H) pad *= 2;
    return MLP_THREADS / pad;
}
// floats of a sample's row of K values, a multiple of four
__host__ __device__ inline int mlp_pad(int K) { return (K + 3) & ~3; }

// A chunk of at most 16 K weights of a row-major matrix, sixteen per thread:
// columns c < nc, rows r < nr; thread: column tid % 2^lg, rows tid / 2^lg, +
// 1024 / 2^lg, ...
struct MlpChunk {
    int c, r0, step, nc, nr;
    __device__ MlpChunk(int nc_, int nr_) : nc(nc_), nr(nr_)
    {
        int lg = 4;
        while ((1 << lg) < nc) ++lg;
        c = (int)threadIdx.x & ((1 << lg) - 1);
        r0 = (int)threadIdx.x >> lg;
        step = MLP_THREADS >> lg;
    }
    __device__ void fetch(double (&w)[MLP_LOADS], const double* W, int ld) const
    {
#pragma unroll
        for (int i = 0; i < MLP_LOADS; ++i) {
            const int r = r0 + i * step;
            w[i] = r < nr && c < nc ? W[(size_t)r * ld + c] : 0.0;
        }
    }
    // element (r, c) to wt[r * rs + c * cs]
    __device__ void put(const double (&w)[MLP_LOADS], float* wt, int rs, int cs) const
    {
#pragma unroll
        for (int i = 0; i < MLP_LOADS; ++i) {
            const int r = r0 + i * step;
            if (r < nr && c < nc) wt[r * rs + c * cs] = (float)w[i];
        }
    }
};

// fetches the weights of inputs j0 .. of a layer of N units over K inputs:
// W[n][j] (T = false) or, for the errors going back, W[j][n] (T = true)
template <bool T>
__device__ inline MlpChunk mlp_fetch(double (&w)[MLP_LOADS], const double* W, int K, int N, int j0)
{
    const int chunk = mlp_chunk(N), kc = K - j0 < chunk ? K - j0 : chunk;
    const MlpChunk m(T ? N : kc, T ? kc : N);
    m.fetch(w, T ? W + (size_t)j0 * N : W + j0, T ? N : K);
    return m;
}

// out(s, n, b[n] + sum_j W(n, j) src[s][j]) for the workgroup's S samples
// (bias may be NULL); rows of src are mlp_pad(K) floats apart. first: the first
// chunk of weights, already fetched.
template <bool T, typename Out>
__device__ inline void mlp_layer(int K, int N, int S, const double* W, const double* bias, const float* src,
                                 float* wt, double (&first)[MLP_LOADS], Out out)
{
    const int ks = mlp_pad(K), chunk = mlp_chunk(N), row = mlp_row(N);
    // (N S <= 1024 for the hidden layers; the output layer may take more rounds)
    for (int i0 = 0; i0 < N * S; i0 += MLP_THREADS) {
        const int it = i0 + (int)threadIdx.x;
        const bool on = it < N * S;
        const int n = on ? it % N : 0, s0 = on ? it / N : 0;
        float a = on && bias ? (float)bias[n] : 0.f;
        for (int j0 = 0; j0 < K; j0 += chunk) {
            const int kc = K - j0 < chunk ? K - j0 : chunk;
            if (i0 || j0) mlp_fetch<T>(first, W, K, N, j0);
            __syncthreads();  // the last chunk has been read
            MlpChunk(T ? N : kc, T ? kc : N).put(first, wt, T ? 1 : row, T ? row : 1);
            __syncthreads();
            const float* w = wt + n * row;
            const float* x = src + s0 * ks + j0;
            int c = 0;
#pragma unroll 8
            for (; c + 4 <= kc; c += 4) {
                const float4 u = *(const float4*)(w + c), y = *(const float4*)(x + c);
                a = fmaf(u.w, y.w, fmaf(u.z, y.z, fmaf(u.y, y.y, fmaf(u.x, y.x, a))));
            }
            for (; c < kc; ++c) a = fmaf(w[c], x[c], a);
        }
        if (on) out(s0, n, a);
    }
    __syncthreads();
}

// LDS floats: weights [max(H, out)][mlp_row], then samples [S][in], [S][H], [S][H] (rows padded)
__global__ __launch_bounds__(MLP_THREADS) void k_mlp_fwd(int B, MlpDims d, int S, const double* P, const float* X,
                                                        float* Y, float* act)
{
    extern __shared__ float4 mlp_lds4[];
    const int big = d.H > d.out ? d.H : d.out;
    const int pi = mlp_pad(d.in), ph = mlp_pad(d.H);
    float* wt = (float*)mlp_lds4;
    float* xs = wt + big * mlp_row(big);
    float* h1 = xs + S * pi;
    float* h2 = h1 + S * ph;
    const int s0 = blockIdx.x * S, ns = B - s0 < S ? B - s0 : S;
    double w1[MLP_LOADS], w2[MLP_LOADS];
    mlp_fetch<false>(w1, P, d.in, d.H, 0);
    mlp_fetch<false>(w2, P + mlp_off_W2(d), d.H, d.H, 0);
    for (int i = threadIdx.x; i < S * d.in; i += MLP_THREADS)
        xs[i / d.in * pi + i % d.in] = i < ns * d.in ? X[(size_t)s0 * d.in + i] : 0.f;
    mlp_layer<false>(d.in, d.H, S, P, P + mlp_off_b1(d), xs, wt, w1, [&](int q, int n, float a) {
        a = a > 0.f ? a : 0.f;
        h1[q * ph + n] = a;
        if (q < ns) act[(size_t)(s0 + q) * 2 * d.H + n] = a;
    });
    mlp_fetch<false>(w1, P + mlp_off_W3(d), d.H, d.out, 0);
    mlp_layer<false>(d.H, d.H, S, P + mlp_off_W2(d), P + mlp_off_b2(d), h1, wt, w2, [&](int q, int n, float a) {
        a = a > 0.f ? a : 0.f;
        h2[q * ph + n] = a;
        if (q < ns) act[(size_t)(s0 + q) * 2 * d.H + d.H + n] = a;
    });
    mlp_layer<false>(d.H, d.out, S, P + mlp_off_W3(d), P + mlp_off_b3(d), h2, wt, w1, [&](int q, int n, float a) {
        if (q < ns) Y[(size_t)(s0 + q) * d.out + n] = a;
    });
}

// per-sample back-propagated errors: delta[s] = (d1[H], d2[H], d3[out]); the
// squared error of the sample goes to sq[s]. LDS floats: weights [H][mlp_row],
// then samples d3 [S][out], d2 [S][H] (rows padded).
__global__ __launch_bounds__(MLP_THREADS) void k_mlp_delta(int B, MlpDims d, int S, const double* P, const float* Y,
                                                          const float* act, const float* T, float* delta, double* sq)
{
    extern __shared__ float4 mlp_lds4[];
    const int ph = mlp_pad(d.H), po = mlp_pad(d.out);
    float* wt = (float*)mlp_lds4;
    float* d3 = wt + d.H * mlp_row(d.H);
    float* d2 = d3 + S * po;
    const float scale = 1.0f / ((float)B * (float)d.out);
    const int s0 = blockIdx.x * S, ns = B - s0 < S ? B - s0 : S;
    const int DS = 2 * d.H + d.out;
    const double *W2 = P + mlp_off_W2(d), *W3 = P + mlp_off_W3(d);
    double w3[MLP_LOADS], w2[MLP_LOADS];
    mlp_fetch<true>(w3, W3, d.out, d.H, 0);
    mlp_fetch<true>(w2, W2, d.H, d.H, 0);
    for (int i = threadIdx.x; i < S * d.out; i += MLP_THREADS) {
        const bool on = i < ns * d.out;
        const float r = on ? Y[(size_t)s0 * d.out + i] - T[(size_t)s0 * d.out + i] : 0.f;
        const float e = 2.f * r * scale;
        d3[i / d.out * po + i % d.out] = e;
        if (on) delta[(size_t)(s0 + i / d.out) * DS + 2 * d.H + i % d.out] = e;
    }
    if ((int)threadIdx.x >= MLP_THREADS - ns) {
        const int s = MLP_THREADS - 1 - (int)threadIdx.x;
        double a = 0.0;
        for (int o = 0; o < d.out; ++o) {
            const size_t i = (size_t)(s0 + s) * d.out + o;
            const float r = Y[i] - T[i];
            a += (double)r * (double)r;
        }
        sq[s0 + s] = a;
    }
    mlp_layer<true>(d.out, d.H, S, W3, nullptr, d3, wt, w3, [&](int q, int n, float a) {
        const bool on = q < ns && act[(size_t)(s0 + q) * 2 * d.H + d.H + n] > 0.f;
        a = on ? a : 0.f;
        d2[q * ph + n] = a;
        if (q < ns) delta[(size_t)(s0 + q) * DS + d.H + n] = a;
    });
    mlp_layer<true>(d.H, d.H, S, W2, nullptr, d2, wt, w2, [&](int q, int n, float a) {
        if (q < ns) delta[(size_t)(s0 + q) * DS + n] = act[(size_t)(s0 + q) * 2 * d.H + n] > 0.f ? a : 0.f;
    });
}

// The same, a workgroup per sample and a thread per unit, for few samples: nothing is
// staged, so the first products need not wait for a whole layer's weights. Every output
// is the same chain of fused multiply-adds as above, bit for bit. Together / a sample
// each, us, forward: 18-128-6 (both hidden layers of 128) 1 sample 13.0 / 7.8, 256 13.5 /
// 8.6, 384 13.5 / 11.9, 64-128-64 384 15.2 / 16.3, 64-256-64 256 28.5 / 26.1, 384 28.7 /
// 43.4, 18-64-6 1024 10.7 / 7.9, 2048 10.8 / 12.6, 5-32-2
// 2048 9.1 / 6.1, 4096 9.2 / 9.8, 4-16-2 4096 8.4 / 5.9; backward: 64-256-64 1 31.4 / 20.2, 512
// 43.4 / 37.2, 768 51.9 / 54.5, 18-200-6 512 30.9 / 27.1, 768 36.1 / 39.2, 18-64-6 2048
// 41.3 / 40.1, 4096 74.8 / 80.4.
inline bool mlp_fwd_each(int B, const MlpDims& d)
{
    return B <= (d.H > 64 ? 256 : d.H > 32 ? 1024 : d.H > 24 ? 3072 : 4096);
}
inline bool mlp_delta_each(int B, const MlpDims& d) { return B <= (d.H > 64 ? 512 : 2048); }

__global__ __launch_bounds__(MLP_MAX_H) void k_mlp_fwd_sample(MlpDims d, const double* P, const float* X, float* Y,
                                                             float* act)
{
    __shared__ float xs[MLP_MAX_IN], h1[MLP_MAX_H], h2[MLP_MAX_H];
    const int s = blockIdx.x, i = threadIdx.x;
    // unit i of a layer of N over K inputs
    auto unit = [&](int K, const double* W, const double* b, const float* src) {
        float a = (float)b[i];
        for (int j = 0; j < K; ++j) a = fmaf((float)W[(size_t)i * K + j], src[j], a);
        return a;
    };
    if (i < d.in) xs[i] = X[(size_t)s * d.in + i];
    __syncthreads();
    if (i < d.H) {
        const float a = unit(d.in, P, P + mlp_off_b1(d), xs);
        h1[i] = a > 0.f ? a : 0.f;
        act[(size_t)s * 2 * d.H + i] = h1[i];
    }
    __syncthreads();
    if (i < d.H) {
        const float a = unit(d.H, P + mlp_off_W2(d), P + mlp_off_b2(d), h1);
        h2[i] = a > 0.f ? a : 0.f;
        act[(size_t)s * 2 * d.H + d.H + i] = h2[i];
    }
    __syncthreads();
    if (i < d.out) Y[(size_t)s * d.out + i] = unit(d.H, P + mlp_off_W3(d), P + mlp_off_b3(d), h2);
}

__global__ __launch_bounds__(MLP_MAX_H) void k_mlp_delta_sample(int B, MlpDims d, const double* P, const float* Y,
                                                               const float* act, const float* T, float* delta,
                                                               double* sq)
{
    __shared__ float d3[MLP_MAX_OUT], d2[MLP_MAX_H], r[MLP_MAX_OUT];
    const int s = blockIdx.x, i = threadIdx.x;
    const double *W2 = P + mlp_off_W2(d), *W3 = P + mlp_off_W3(d);
    const float scale = 1.0f / ((float)B * (float)d.out);
    const float *a1 = act + (size_t)s * 2 * d.H, *a2 = a1 + d.H;
    float* dl = delta + (size_t)s * (2 * d.H + d.out);
    if (i < d.out) {
        r[i] = Y[(size_t)s * d.out + i] - T[(size_t)s * d.out + i];
        d3[i] = 2.f * r[i] * scale;
        dl[2 * d.H + i] = d3[i];
    }
    __syncthreads();
    if (i < d.H) {
        float a = 0.f;
        for (int o = 0; o < d.out; ++o) a = fmaf((float)W3[(size_t)o * d.H + i], d3[o], a);
        d2[i] = a2[i] > 0.f ? a : 0.f;
        dl[d.H + i] = d2[i];
    }
    __syncthreads();
    if (i < d.H) {
        float a = 0.f;
        for (int k = 0; k < d.H; ++k) a = fmaf((float)W2[(size_t)k * d.H + i], d2[k], a);
        dl[i] = a1[i] > 0.f ? a : 0.f;
    }
    if (i == 0) {
        double a = 0.0;
        for (int o = 0; o < d.out; ++o) a += (double)r[o] * (double)r[o];
        sq[s] = a;
    }
}

// Weight gradients and the loss. A wave owns a 4 x 8 tile of one layer's (error
// row, input column) sums, the bias being one more column whose input is 1. Its
// lanes take every 64th sample (products rounded to FP32, summed in FP64), three
// 16-byte loads for 32 sums, and are added by a fixed tree at the end. (One
// thread per parameter walked all samples alone: 870 dependent FP64 sums deep,
// and a load instruction brought one error and 64 inputs.)
constexpr int WG_R = 4, WG_C = 8, WG_N = WG_R * WG_C, WG_WAVES = 4;
typedef float wg_f4 __attribute__((ext_vector_type(4), aligned(4)));  // 16 bytes at any float

// tiles of the three layers: (rows, columns) = (H, in + 1), (H, H + 1), (out, H + 1)
__host__ __device__ inline int wg_tiles(int rows, int cols)
{
    return ((rows + WG_R - 1) / WG_R) * ((cols + WG_C - 1) / WG_C);
}

// Adds each of the N values over the wave; lane l ends with value l mod 32's
// total in v[0] (halving the values at every step).
__device__ inline double swap_add(double a, double b, int H)
{
    const uint64_t u = __double_as_longlong(a), w = __double_as_longlong(b);
    float l0 = __uint_as_float((uint32_t)u), h0 = __uint_as_float((uint32_t)(u >> 32));
    float l1 = __uint_as_float((uint32_t)w), h1 = __uint_as_float((uint32_t)(w >> 32));
    if (H == 32) {
        swap_halves<32>(l0, l1);
        swap_halves<32>(h0, h1);
    } else {
        swap_halves<16>(l0, l1);
        swap_halves<16>(h0, h1);
    }
    return __longlong_as_double((long long)(((uint64_t)__float_as_uint(h0) << 32) | __float_as_uint(l0))) +
           __longlong_as_double((long long)(((uint64_t)__float_as_uint(h1) << 32) | __float_as_uint(l1)));
}
template <int K>
__device__ inline double row_add(double a, double b, bool upper)
{
    return (upper ? b : a) + across<K>(upper ? a : b);
}

__global__ __launch_bounds__(64 * WG_WAVES) void k_mlp_wgrad(int B, MlpDims d, const float* __restrict__ X,
                                                            const float* __restrict__ act,
                                                            const float* __restrict__ delta,
                                                            const double* __restrict__ sq, double* __restrict__ G,
                                                            double* __restrict__ loss)
{
    __shared__ double red[WG_WAVES];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int n1 = wg_tiles(d.H, d.in + 1), n2 = wg_tiles(d.H, d.H + 1), n3 = wg_tiles(d.out, d.H + 1);
    if (blockIdx.x == gridDim.x - 1) {  // the loss: the mean of the samples' squared errors
        double a = 0.0;
        for (int s = threadIdx.x; s < B; s += 64 * WG_WAVES) a += sq[s];
        a = block_sum(a, red);
        if (threadIdx.x == 0) *loss = a / ((double)B * (double)d.out);
        return;
    }
    int t = blockIdx.x * WG_WAVES + wv;
    if (t >= n1 + n2 + n3) return;
    const int layer = t < n1 ? 0 : t < n1 + n2 ? 1 : 2;
    t -= layer == 0 ? 0 : layer == 1 ? n1 : n1 + n2;
    const int rows = layer == 2 ? d.out : d.H, cols = layer == 0 ? d.in : d.H;  // without the bias
    const int tc = (cols + 1 + WG_C - 1) / WG_C;
    const int r0 = t / tc * WG_R, c0 = t % tc * WG_C;
    const int DS = 2 * d.H + d.out;
    const float* D = delta + (layer == 0 ? 0 : layer == 1 ? d.H : 2 * d.H) + r0;
    const float* I = (layer == 0 ? X : layer == 1 ? act : act + d.H) + c0;
    const int is = layer == 0 ? d.in : 2 * d.H;
    const bool whole = r0 + WG_R <= rows && c0 + WG_C <= cols;  // uniform
    double g[WG_N] = {};
    auto add = [&](const float (&e)[WG_R], const float (&x)[WG_C]) {
#pragma unroll
        for (int i = 0; i < WG_R; ++i)
#pragma unroll
            for (int j = 0; j < WG_C; ++j) g[i * WG_C + j] += (double)(e[i] * x[j]);
    };
    if (whole) {
#pragma unroll 4
        for (int s = lane; s < B; s += 64) {
            const wg_f4 e4 = *(const wg_f4*)(D + (size_t)s * DS);
            const wg_f4 x4 = *(const wg_f4*)(I + (size_t)s * is), y4 = *(const wg_f4*)(I + (size_t)s * is + 4);
            const float e[WG_R] = {e4[0], e4[1], e4[2], e4[3]};
            const float x[WG_C] = {x4[0], x4[1], x4[2], x4[3], y4[0], y4[1], y4[2], y4[3]};
            add(e, x);
        }
    } else {
        for (int s = lane; s < B; s += 64) {
            float e[WG_R], x[WG_C];
#pragma unroll
            for (int i = 0; i < WG_R; ++i) e[i] = r0 + i < rows ? D[(size_t)s * DS + i] : 0.f;
#pragma unroll
            for (int j = 0; j < WG_C; ++j)
                x[j] = c0 + j < cols ? I[(size_t)s * is + j] : c0 + j == cols ? 1.f : 0.f;
            add(e, x);
        }
    }
    // (the lanes of a wave part in the loops above; all are back here)
    const uint32_t bits = row_bits(lane & 15u);
#pragma unroll
    for (int i = 0; i < 16; ++i) g[i] = swap_add(g[i], g[i + 16], 32);
#pragma unroll
    for (int i = 0; i < 8; ++i) g[i] = swap_add(g[i], g[i + 8], 16);
#pragma unroll
    for (int i = 0; i < 4; ++i) g[i] = row_add<3>(g[i], g[i + 4], bits & 8u);
#pragma unroll
    for (int i = 0; i < 2; ++i) g[i] = row_add<2>(g[i], g[i + 2], bits & 4u);
    g[0] = row_add<1>(g[0], g[1], bits & 2u);
    const double a = g[0] + across<0>(g[0]);
    const int v = (lane & 32 ? 16 : 0) | (lane & 16 ? 8 : 0) | (bits & 8u ? 4 : 0) | (bits & 4u ? 2 : 0) |
                  (bits & 2u ? 1 : 0);
    const int row = r0 + v / WG_C, col = c0 + v % WG_C;
    if ((bits & 1u) || row >= rows || col > cols) return;
    const int64_t oW = layer == 0 ? 0 : layer == 1 ? mlp_off_W2(d) : mlp_off_W3(d);
    const int64_t ob = layer == 0 ? mlp_off_b1(d) : layer == 1 ? mlp_off_b2(d) : mlp_off_b3(d);
    G[col == cols ? ob + row : oW + (int64_t)row * cols + col] = a;
}

// Warm-start angles from the predictor's standardised outputs: output o of
// subgraph b becomes y * sd[o] + mu[o] (FP32, rounded as written), then FP64;
// outputs 0..p-1 are gamma_1..p, outputs p..2p-1 are beta_1..p, and theta is
// laid out [gamma (B p) | beta (B p)], row b = subgraph b.
__global__ void k_warm_angles(int B, int p, const float* Y, const float* mu, const float* sd, double* theta)
{
#pragma clang fp contract(off)
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 2 * B * p) return;
    const int b = i / (2 * p), o = i % (2 * p);
    const float a = Y[i] * sd[o] + mu[o];  // two roundings, never one fused multiply-add
    const size_t dst = o < p ? (size_t)b * p + o : (size_t)B * p + (size_t)b * p + (o - p);
    theta[dst] = (double)a;
}

// Per subgraph, keep the start with the larger <C>: if E_alt[b] > E[b], row b
// of theta (its gamma and beta) and E[b] take the alternative's values. One
// thread per subgraph, so the comparison and the copy see the same E[b].
__global__ void k_keep_better(int B, int p, const double* E_alt, const double* theta_alt, double* E, double* theta)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    const double ea = E_alt[b];
    if (!(ea > E[b])) return;
    for (int l = 0; l < p; ++l) {
        const size_t g = (size_t)b * p + l, t = (size_t)B * p + g;
        theta[g] = theta_alt[g];
        theta[t] = theta_alt[t];
    }
    E[b] = ea;
}

hipError_t launch_warm_angles(int B, int p, const float* Y, const float* mu, const float* sd, double* theta,
                              hipStream_t s)
{
    const int n = 2 * B * p;
    hipLaunchKernelGGL(k_warm_angles, dim3((n + 255) / 256), dim3(256), 0, s, B, p, Y, mu, sd, theta);
    return hipGetLastError();
}

hipError_t launch_keep_better(int B, int p, const double* E_alt, const double* theta_alt, double* E, double* theta,
                              hipStream_t s)
{
    hipLaunchKernelGGL(k_keep_better, dim3((B + 255) / 256), dim3(256), 0, s, B, p, E_alt, theta_alt, E, theta);
    return hipGetLastError();
}

hipError_t launch_mlp_forward(int B, MlpDims d, const double* P, const float* X, float* Y, float* act, hipStream_t s)
{
    const int S = mlp_samples(d.H), big = d.H > d.out ? d.H : d.out;
    if (mlp_fwd_each(B, d)) {
        const int units = d.in > big ? d.in : big;
        hipLaunchKernelGGL(k_mlp_fwd_sample, dim3(B), dim3((units + 63) / 64 * 64), 0, s, d, P, X, Y, act);
        return hipGetLastError();
    }
    const size_t lds = sizeof(float) * ((size_t)big * mlp_row(big) +
                                        (size_t)S * (mlp_pad(d.in) + 2 * mlp_pad(d.H)));
    hipLaunchKernelGGL(k_mlp_fwd, dim3((B + S - 1) / S), dim3(MLP_THREADS), lds, s, B, d, S, P, X, Y, act);
    return hipGetLastError();
}

hipError_t launch_mlp_backward(int B, MlpDims d, const double* P, const float* X, const float* Y, const float* act,
                               const float* T, float* scratch, double* G, double* loss, hipStream_t s)
{
    float* delta = scratch;
    double* sq = (double*)(scratch + (size_t)B * (2 * d.H + d.out) + 1);  // 8-byte aligned below
    sq = (double*)(((uintptr_t)sq + 7) & ~(uintptr_t)7);
    const int S = mlp_samples(d.H);
    const size_t lds = sizeof(float) * ((size_t)d.H * mlp_row(d.H) + (size_t)S * (mlp_pad(d.out) + mlp_pad(d.H)));
    if (mlp_delta_each(B, d)) {
        const int units = d.H > d.out ? d.H : d.out;
        hipLaunchKernelGGL(k_mlp_delta_sample, dim3(B), dim3((units + 63) / 64 * 64), 0, s, B, d, P, Y, act, T, delta, sq);
    } else {
        hipLaunchKernelGGL(k_mlp_delta, dim3((B + S - 1) / S), dim3(MLP_THREADS), lds, s, B, d, S, P, Y, act, T, delta,
                           sq);
    }
    const int tiles = wg_tiles(d.H, d.in + 1) + wg_tiles(d.H, d.H + 1) + wg_tiles(d.out, d.H + 1);
    hipLaunchKernelGGL(k_mlp_wgrad, dim3((tiles + WG_WAVES - 1) / WG_WAVES + 1), dim3(64 * WG_WAVES), 0, s, B, d, X, act, delta, sq, G, loss);
    return hipGetLastError();
}

// Scratch of the backward pass for callers that cannot allocate: a
// file-scope device array (each device holds its own copy until the process
// ends). Host code never passes the array's name to a kernel: its device
// address is looked up once per device with hipGetSymbolAddress and kept.
static __device__ __align__(256) uint8_t scratch[MLP_STATIC_SCRATCH_BYTES];

namespace {
constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[MAX_DEVICES] = {};
}  // namespace

hipError_t mlp_static_scratch(void** out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        e = hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

}  // namespace pq

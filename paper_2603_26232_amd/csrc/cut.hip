// Integer cut evaluation (paper Sec. 2.1 CutVal, used on merged full-graph
// assignments in Alg. 2) and the FP64 Adam step of the angle optimiser.
#include "common.h"

namespace pq {

// cut[a] = sum_e w_e [x_a(u_e) != x_a(v_e)], x_a bit-packed (vertex t = word
// t/32, bit t%32). An edge id outside [0, nV) makes every result -1.
//
// A workgroup takes G assignments, so that an edge is read once for all of them
// (one assignment each read 160 MB of edges at 20,000 edges and 1024 assignments,
// and two words of the assignment for each edge). It first lays the assignments
// out in LDS as one byte per vertex, bit g for assignment g: an edge is then two
// byte reads and an exclusive or. More vertices than LDS_VERTICES, or more than a
// workgroup's edges repay, are looked up in the packed words instead, one or two
// assignments a workgroup (the rows of more do not fit the L1 cache).
//
// G is the largest of 8, 4, 2, 1 that leaves a workgroup per CU. If there are
// fewer than that even with one each and the edges are many, `splits` workgroups
// share the edges of the same assignments and add to results cleared before; a
// pass over the edges then sets -1 if an id is out of range. Small calls are bound
// by latency, large ones by the vector units (an AND, a select and a 64-bit
// addition per edge and assignment). Before / now, in us, weighted: 2000 vertices,
// 20,000 edges, 1024 assignments 43.5 / 11.7, 4096 assignments 124 / 30.9; one
// assignment, 200,000 edges 242 / 11.9 (16,383 edges, not split, about 9); 16,000
// vertices, 1.28 M edges, 1000 assignments 3696 / 473; 100,000 vertices, not in
// LDS, 200,000 edges, 300 assignments 377 / 237 (60,000, in LDS: 376 / 79). Fewer
// than CUT_FEW_EDGES leave most of 1024 threads idle: 500 edges, 4096 assignments
// 16.1 with them and 6.7 with 256; from 4096 on both are the same.
constexpr int CUT_THREADS = 1024;
constexpr int CUT_FEW_EDGES = 4096;  // fewer: workgroups of a quarter of the threads
constexpr int CUT_CUS = 256;
constexpr int CUT_L1_BYTES = 32 * 1024;
constexpr int LDS_VERTICES = 60 * 1024;
constexpr int EDGES_PER_SPLIT = 8192;

__device__ inline int64_t wave_sum_i64(int64_t x)
{
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
    return x;
}

// bit g: whether assignment a0 + g has bit t of word q set
template <int G>
__device__ inline uint32_t assigned(const uint32_t* x, int64_t nw, int na, int32_t t)
{
    uint32_t bits = 0;
#pragma unroll
    for (int g = 0; g < G; ++g)
        if (g < na) bits |= ((x[g * nw + (t >> 5)] >> (t & 31)) & 1u) << g;
    return bits;
}

template <int G, int T, bool LDS, bool WEIGHTED>
__global__ __launch_bounds__(T) void k_maxcut(int32_t nV, int64_t nE, const int32_t* u, const int32_t* v,
                                                       const int32_t* w, int64_t A, const uint32_t* assign,
                                                       int splits, int64_t per, int64_t* cut)
{
    extern __shared__ uint8_t bits_of[];
    __shared__ int64_t red[T / 64][G];
    const int t = threadIdx.x;
    const int64_t nw = (nV + 31) / 32;
    const int64_t groups = (A + G - 1) / G;
    const int split = blockIdx.x % splits;
    const int64_t e0 = split * per, e1 = e0 + per < nE ? e0 + per : nE;
    for (int64_t group = blockIdx.x / splits; group < groups; group += gridDim.x / splits) {
        const int64_t a0 = group * G;
        const int na = A - a0 < G ? (int)(A - a0) : G;
        const uint32_t* x = assign + a0 * nw;
        if (LDS) {
            for (int32_t y = t; y < nV; y += T) bits_of[y] = (uint8_t)assigned<G>(x, nw, na, y);
            __syncthreads();
        }
        int64_t acc[G];
#pragma unroll
        for (int g = 0; g < G; ++g) acc[g] = 0;
        bool bad = false;
        // four edges in flight per thread; one beyond the end joins a vertex to itself
        for (int64_t e = e0 + t; e < e1; e += 4 * T) {
            int32_t p[4], q[4], we[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const bool in = e + k * T < e1;
                p[k] = in ? u[e + k * T] : 0;
                q[k] = in ? v[e + k * T] : 0;
                we[k] = !WEIGHTED ? 1 : in ? w[e + k * T] : 0;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (!LDS && e + k * T >= e1) continue;  // (no words to look up)
                if ((uint32_t)p[k] >= (uint32_t)nV || (uint32_t)q[k] >= (uint32_t)nV) {
                    bad = true;
                    continue;
                }
                const uint32_t d = LDS ? (uint32_t)(bits_of[p[k]] ^ bits_of[q[k]])
                                       : assigned<G>(x, nw, na, p[k]) ^ assigned<G>(x, nw, na, q[k]);
#pragma unroll
                for (int g = 0; g < G; ++g) acc[g] += (d >> g) & 1u ? we[k] : 0;
            }
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int64_t sum = wave_sum_i64(acc[g]);
            if ((t & 63) == 0) red[t >> 6][g] = sum;
        }
        const int any_bad = __syncthreads_or(bad);
        if (t < na) {
            int64_t sum = 0;
            for (int k = 0; k < T / 64; ++k) sum += red[k][t];
            if (splits == 1)
                cut[a0 + t] = any_bad ? -1 : sum;
            else
                atomicAdd((unsigned long long*)&cut[a0 + t], (unsigned long long)sum);
        }
        __syncthreads();  // red and bits_of are free again
    }
}

__global__ void k_maxcut_clear(int64_t A, int64_t* cut)
{
    const int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (a < A) cut[a] = 0;
}

// -1 for every assignment if an edge id is out of range (as each workgroup that
// finds one writes)
__global__ __launch_bounds__(THREADS) void k_maxcut_check(int32_t nV, int64_t nE, const int32_t* u, const int32_t* v,
                                                         int64_t A, int64_t* cut)
{
    bool bad = false;
    for (int64_t e = (int64_t)blockIdx.x * THREADS + threadIdx.x; e < nE; e += (int64_t)gridDim.x * THREADS)
        bad |= (uint32_t)u[e] >= (uint32_t)nV || (uint32_t)v[e] >= (uint32_t)nV;
    if (!__syncthreads_or(bad)) return;
    for (int64_t a = threadIdx.x; a < A; a += THREADS) cut[a] = -1;
}

template <int G, int T>
static void launch_maxcut_gt(int64_t grid, int32_t nV, int64_t nE, const int32_t* u, const int32_t* v,
                             const int32_t* w, int64_t A, const uint32_t* assign, int splits, int64_t* cut,
                             hipStream_t s)
{
    auto* k = w ? k_maxcut<G, T, true, true> : k_maxcut<G, T, true, false>;
    hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(T), (size_t)nV, s, nV, nE, u, v, w, A, assign, splits,
                       (nE + splits - 1) / splits, cut);
}

template <int G>
static void launch_maxcut_g(bool few, int64_t grid, int32_t nV, int64_t nE, const int32_t* u, const int32_t* v,
                            const int32_t* w, int64_t A, const uint32_t* assign, int splits, int64_t* cut,
                            hipStream_t s)
{
    auto* f = few ? launch_maxcut_gt<G, CUT_THREADS / 4> : launch_maxcut_gt<G, CUT_THREADS>;
    f(grid, nV, nE, u, v, w, A, assign, splits, cut, s);
}

// in the packed words
template <int G, int T>
static void launch_maxcut_words(int64_t grid, int32_t nV, int64_t nE, const int32_t* u, const int32_t* v,
                                const int32_t* w, int64_t A, const uint32_t* assign, int splits, int64_t* cut,
                                hipStream_t s)
{
    auto* k = w ? k_maxcut<G, T, false, true> : k_maxcut<G, T, false, false>;
    hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(T), 0, s, nV, nE, u, v, w, A, assign, splits,
                       (nE + splits - 1) / splits, cut);
}

// How a call is split: G assignments a workgroup, `splits` workgroups for the same
// ones, `few` edges (256 threads), assignments laid out in LDS or not.
//
// Laying out takes nV G bits a workgroup and repays from about nV / 2 edges on, with
// 1024 threads and at most two assignments from nV / 4. In us, LDS / words: 60,000
// vertices, 5000 assignments, 3000 edges 467 / 41, 21,000 317 / 229, 30,000 333 / 326,
// 45,000 349 / 481; 1000 assignments, 3000 edges 49 / 10, 12,000 26 / 31, 30,000 33 / 72;
// 2000 vertices, 5000 assignments, 400 edges 13.5 / 10.2, 1000 13.7 / 12.2, 1500 14.6 /
// 15.9; 60,000 vertices, one assignment, 300,000 edges (8192 a workgroup) 17.7 / 14.8.
// Words, one / two / eight assignments a workgroup: 100,000 vertices, 200,000 edges,
// 5000 assignments 2279 / 2150 / 4133 us; 2,000,000 edges, 1000 assignments 5382 / 4365 /
// -; 1,000,000 vertices, as many edges, 300 assignments 3386 / 4463 / 7718.
struct CutShape {
    int G, splits;
    bool few, lds;
    int64_t groups;
};
static CutShape cut_shape(int32_t nV, int64_t nE, int64_t A)
{
    CutShape c;
    c.G = 8;
    while (c.G > 1 && A < (int64_t)c.G * CUT_CUS) c.G >>= 1;
    c.few = nE < CUT_FEW_EDGES;
    c.lds = nV <= LDS_VERTICES;
    auto split = [&]() {
        c.groups = (A + c.G - 1) / c.G;
        c.splits = 1;
        while (c.groups * c.splits * 2 <= CUT_CUS && nE >= (int64_t)c.splits * 2 * EDGES_PER_SPLIT) c.splits *= 2;
    };
    split();
    if (c.lds) c.lds = (!c.few && c.G <= 2 ? 4 : 2) * ((nE + c.splits - 1) / c.splits) >= nV;
    if (!c.lds) {
        const bool two = c.G >= 2 && !c.few && nV <= 8 * CUT_L1_BYTES / 2;
        c.G = two ? 2 : 1;
        split();
    }
    return c;
}

hipError_t launch_maxcut_eval(int32_t nV, int64_t nE, const int32_t* u, const int32_t* v, const int32_t* w,
                              int64_t A, const uint32_t* assign, int64_t* cut, hipStream_t s)
{
    if (A <= 0) return hipSuccess;
    const CutShape c = cut_shape(nV, nE, A);
    const int64_t grid = c.groups < 65536 ? c.groups * c.splits : 65536;  // splits > 1 only with few groups
    if (c.splits > 1)
        hipLaunchKernelGGL(k_maxcut_clear, dim3((unsigned)((A + THREADS - 1) / THREADS)), dim3(THREADS), 0, s, A, cut);
    if (!c.lds && c.few)
        launch_maxcut_words<1, CUT_THREADS / 4>(grid, nV, nE, u, v, w, A, assign, c.splits, cut, s);
    else if (!c.lds && c.G == 2)
        launch_maxcut_words<2, CUT_THREADS>(grid, nV, nE, u, v, w, A, assign, c.splits, cut, s);
    else if (!c.lds)
        launch_maxcut_words<1, CUT_THREADS>(grid, nV, nE, u, v, w, A, assign, c.splits, cut, s);
    else if (c.G == 8)
        launch_maxcut_g<8>(c.few, grid, nV, nE, u, v, w, A, assign, c.splits, cut, s);
    else if (c.G == 4)
        launch_maxcut_g<4>(c.few, grid, nV, nE, u, v, w, A, assign, c.splits, cut, s);
    else if (c.G == 2)
        launch_maxcut_g<2>(c.few, grid, nV, nE, u, v, w, A, assign, c.splits, cut, s);
    else
        launch_maxcut_g<1>(c.few, grid, nV, nE, u, v, w, A, assign, c.splits, cut, s);
    if (c.splits > 1) {
        const int64_t blocks = (nE + 8 * THREADS - 1) / (8 * THREADS);
        hipLaunchKernelGGL(k_maxcut_check, dim3((unsigned)(blocks < CUT_CUS ? blocks : CUT_CUS)), dim3(THREADS), 0, s, nV, nE,
                           u, v, A, cut);
    }
    return hipGetLastError();
}

// Adam (Kingma and Ba 2015) in FP64; sign = +1 ascends (the QAOA objective
// is maximised), -1 descends. The step counter lives in device memory so a
// captured graph can replay the step. One thread per parameter; one workgroup (up to
// 1024 parameters) advances the counter itself, more leave it to a second kernel,
// since every workgroup reads it. One workgroup / several and the second kernel, us: 300
// parameters 4.2 / 6.4, 1024 5.8 / 6.4, 2000 (two a thread) 9.1 / 6.4, the 19,590 of the
// angle predictor 71 / 6.4.
constexpr int ADAM_THREADS = 256, ADAM_ALONE = 1024;

template <int T>
__global__ __launch_bounds__(T) void k_adam(int32_t count, double* theta, const double* grad, double* m, double* v,
                                           int32_t* step, int advance, double lr, double b1, double b2, double eps,
                                           double sign)
{
    const int32_t t = *step + 1;
    const double c1 = 1.0 - pow(b1, (double)t), c2 = 1.0 - pow(b2, (double)t);
    const int32_t i = blockIdx.x * T + threadIdx.x;
    if (i < count) {
        double th = theta[i], mi = m[i], vi = v[i];
        adam_update(th, mi, vi, grad[i], c1, c2, lr, b1, b2, eps, sign);
        m[i] = mi;
        v[i] = vi;
        theta[i] = th;
    }
    if (!advance) return;
    __syncthreads();  // every thread has read the count
    if (threadIdx.x == 0) *step = t;
}

hipError_t launch_adam(int32_t count, double* theta, const double* grad, double* m, double* v, int32_t* step,
                       double lr, double b1, double b2, double eps, double sign, hipStream_t s)
{
    const int blocks = count / ADAM_THREADS + (count % ADAM_THREADS != 0);
    const int alone = count <= ADAM_ALONE;
    if (alone && blocks > 1)
        hipLaunchKernelGGL(k_adam<ADAM_ALONE>, dim3(1), dim3(ADAM_ALONE), 0, s, count, theta, grad, m, v, step, 1, lr,
                           b1, b2, eps, sign);
    else
        hipLaunchKernelGGL(k_adam<ADAM_THREADS>, dim3(blocks), dim3(ADAM_THREADS), 0, s, count, theta, grad, m, v, step,
                           alone, lr, b1, b2, eps, sign);
    const hipError_t e = hipGetLastError();
    return e != hipSuccess || alone ? e : launch_step_advance(step, 1, s);
}

}  // namespace pq

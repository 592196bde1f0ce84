// Subgraphs of at most 13 qubits: one workgroup runs the whole circuit, the
// whole gradient, or the whole angle optimisation of its subgraph with the
// state in registers (paper Sec. 2.2; the reduced state has 2^(n-1) <= 4096
// amplitudes).
//
// What bounds it is latency: a subgraph's state fits one CU many times over,
// and every layer is a chain of n rotations. So a layer has no pass over LDS
// per qubit: 64 lanes x R registers hold the state, register bits rotate in
// registers, index bits 0..3 across the lanes of a row by DPP (lane.h), bits 4
// and 5 by swapping lane halves of register pairs (v_permlane16/32_swap). Up
// to 10 qubits fit one wave (R = 2^(n-7)) and never wait at a barrier; 11 and 12
// take four waves (R = 2^(n-9)) and 13 eight (R = 8), whose number is two or
// three more index bits: they trade places with register bits through LDS once
// per layer, one barrier forward. The top qubit's X maps an index to its complement; its partner
// amplitude is read in that same exchange (one wave: by a lane permutation).
//
// Rotations are in the factored form e^{-i beta X} = f (I - i t X) X^flip. The
// n flips of a layer cancel here: together they complement the index and the
// top qubit's flip complements it back. f^n sits in the phase table, which the
// workgroup builds itself from the angles (FP64 products, sine and cosine).
// Beta terms are FP32 sums per lane and index bit (at most eight amplitudes), FP64
// beyond; gamma terms FP64 throughout.
//
// Measured at p = 3, one subgraph, against one rotation per pass over LDS by 256
// lanes: forward 46.8 -> 9.1 us at 13 qubits (28.0 -> 8.4 at 12), an optimiser
// step 120 -> 19.4 us at 13, 69 -> 14 at 12, 31 -> 11 at 10, 19 -> 4.3 at 4; 512
// subgraphs of 13 qubits 138 -> 32.5 us a step.
//
// The optimiser runs all its steps in one launch: subgraphs are independent,
// so theta, the moments and the tables never leave the CU between steps.
#include <algorithm>

#include "angles.h"
#include "lane.h"

namespace pq {

namespace {

constexpr int ST = 512;  // threads at most
constexpr int STEPS = 64;  // steps whose bias corrections are computed at a time
// A phase table of more than PART_MIN entries per thread, or tables of more than
// LUT_CAP entries over all layers, are kept as parts: e^{-i gamma c} is the product (in
// FP64, as the parts are) of e^{-i gamma (c mod 32)} and e^{-i gamma 32 (c / 32)}, taken
// for each amplitude when it is used: one sine and cosine an entry made a table of
// 2000 entries the longest part of a call. Before / with parts, weight sum 2000:
// forward, one subgraph of 10 qubits, p = 3 59.9 / 8.9 us, p = 8 154 / 17.9; 2048 of
// them, p = 8 593 / 47.1; gradient of one of 13 qubits, weight sum 300, p = 32 (a
// table of 4096 entries at most in LDS, the rest in the workspace) 209 / 217. At weight
// sum 300 and 10 qubits p = 3 forward 11.4 / 7.8, gradient 19.1 / 16.9, of 2048 28.5 / 32.3.
constexpr int PART_LO = 32, PART_MIN = 2, LUT_CAP = 4096;
__host__ __device__ inline bool in_parts(int len, int p, int threads) { return len > PART_MIN * threads || p * len > LUT_CAP; }
__host__ __device__ inline int part_count(int len) { return PART_LO + (len - 1) / PART_LO + 1; }

template <int X>
constexpr int log2c()
{
    return X == 8 ? 3 : X == 4 ? 2 : X == 2 ? 1 : 0;
}

// W waves: index of (register, wave, lane) in the exchange buffer
template <int W>
__device__ inline uint32_t xslot(uint32_t r, uint32_t w, uint32_t lane)
{
    return (r * W + w) * 64 + lane;
}

// Orders LDS accesses of the workgroup: a barrier between waves; within one
// wave the LDS keeps issue order, so only the compiler has to.
template <int W>
__device__ inline void sync()
{
    if constexpr (W > 1) __syncthreads();
    else asm volatile("" ::: "memory");
}

// (I - i t X) on registers that differ in bit K
template <int K, int R>
__device__ inline void rx_reg(float2 (&v)[R], float t)
{
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (r & (1 << K)) continue;
        const float2 a = v[r], b = v[r | (1 << K)];
        v[r] = make_float2(fmaf(t, b.y, a.x), fmaf(-t, b.x, a.y));
        v[r | (1 << K)] = make_float2(fmaf(t, a.y, b.x), fmaf(-t, a.x, b.y));
    }
}
template <int K, int R>
__device__ inline float xb_reg(const float2 (&ps)[R], const float2 (&la)[R])
{
    float a = 0.f, b = 0.f;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const float2 o = ps[r ^ (1 << K)];
        float& x = r & 1 ? b : a;
        x = fmaf(la[r].x, o.y, x);
        x = fmaf(-la[r].y, o.x, x);
    }
    return a + b;
}

// exchanges lane bit 4 (H = 16) or 5 (H = 32) with register bit 0
template <int H, int R>
__device__ inline void swap_lanes(float2 (&v)[R])
{
#pragma unroll
    for (int r = 0; r < R; r += 2) {
        swap_halves<H>(v[r].x, v[r + 1].x);
        swap_halves<H>(v[r].y, v[r + 1].y);
    }
}

// the other lane's amplitudes (single registers: no pair to swap)
template <int R>
__device__ inline void lanes_xor(float2 (&o)[R], const float2 (&v)[R], int mask)
{
#pragma unroll
    for (int r = 0; r < R; ++r) o[r] = make_float2(__shfl_xor(v[r].x, mask), __shfl_xor(v[r].y, mask));
}
template <int R>
__device__ inline void rx_with(float2 (&v)[R], const float2 (&o)[R], float t)
{
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = make_float2(fmaf(t, o[r].y, v[r].x), fmaf(-t, o[r].x, v[r].y));
}
template <int R>
__device__ inline float xb_with(const float2 (&o)[R], const float2 (&la)[R])
{
    float a = 0.f, b = 0.f;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        float& x = r & 1 ? b : a;
        x = fmaf(la[r].x, o[r].y, x);
        x = fmaf(-la[r].y, o[r].x, x);
    }
    return a + b;
}

// Forward rotation of every index bit in the wave: lane bits nl (6, or n - 1
// below 7 qubits) and register bits.
template <int R>
__device__ inline void rotate(float2 (&v)[R], float t, int nl)
{
    constexpr int K = log2c<R>();
    if (nl > 0) rx_lane<0>(v, t);
    if (nl > 1) rx_lane<1>(v, t);
    if (nl > 2) rx_lane<2>(v, t);
    if (nl > 3) rx_lane<3>(v, t);
    if constexpr (R >= 2) {
        swap_lanes<16>(v);
        rx_reg<0>(v, t);
        swap_lanes<16>(v);
        swap_lanes<32>(v);
        rx_reg<0>(v, t);
        swap_lanes<32>(v);
    } else {
        float2 o[R];
        if (nl > 4) {
            lanes_xor(o, v, 16);
            rx_with(v, o, t);
        }
        if (nl > 5) {
            lanes_xor(o, v, 32);
            rx_with(v, o, t);
        }
    }
    if constexpr (K > 0) rx_reg<0>(v, t);
    if constexpr (K > 1) rx_reg<1>(v, t);
    if constexpr (K > 2) rx_reg<2>(v, t);
}

// One bit of the adjoint sweep: the beta term on states scaled by |f|^-done,
// w = |f|^(2 done), then the inverse rotation of both.
struct Back {
    float t, fsq, w;
    double acc;
    __device__ void add(float a)
    {
        acc += (double)(w * a);
        w *= fsq;
    }
};
template <int K, int R>
__device__ inline void back_lane(float2 (&ps)[R], float2 (&la)[R], Back& s)
{
    s.add(xb_lane<K>(ps, la));
    rx_lane<K>(ps, s.t);
    rx_lane<K>(la, s.t);
}
template <int K, int R>
__device__ inline void back_reg(float2 (&ps)[R], float2 (&la)[R], Back& s)
{
    s.add(xb_reg<K>(ps, la));
    rx_reg<K>(ps, s.t);
    rx_reg<K>(la, s.t);
}
template <int H, int R>
__device__ inline void back_half(float2 (&ps)[R], float2 (&la)[R], Back& s)
{
    if constexpr (R >= 2) {
        swap_lanes<H>(ps);
        swap_lanes<H>(la);
        back_reg<0>(ps, la, s);
        swap_lanes<H>(ps);
        swap_lanes<H>(la);
    } else {
        float2 po[R], lo[R];
        lanes_xor(po, ps, H);
        lanes_xor(lo, la, H);
        s.add(xb_with(po, la));
        rx_with(ps, po, s.t);
        rx_with(la, lo, s.t);
    }
}
template <int R>
__device__ inline void back(float2 (&ps)[R], float2 (&la)[R], int nl, Back& s)
{
    constexpr int K = log2c<R>();
    if (nl > 0) back_lane<0>(ps, la, s);
    if (nl > 1) back_lane<1>(ps, la, s);
    if (nl > 2) back_lane<2>(ps, la, s);
    if (nl > 3) back_lane<3>(ps, la, s);
    if (nl > 4) back_half<16>(ps, la, s);
    if (nl > 5) back_half<32>(ps, la, s);
    if constexpr (K > 0) back_reg<0>(ps, la, s);
    if constexpr (K > 1) back_reg<1>(ps, la, s);
    if constexpr (K > 2) back_reg<2>(ps, la, s);
}

// LDS of a workgroup (beside the exchange buffers and phase tables)
struct SmallShared {
    float2 rx[MAX_P];             // (t, |f|^2) per layer
    float2 F[MAX_P];              // f^n per layer
    double angle[2 * MAX_P];      // gamma, beta (optimiser)
    double sg[MAX_P][8], sb[MAX_P][8], se[8];  // per wave: gamma and beta terms per layer, <C>
    double k1[STEPS], k2[STEPS];  // Adam's bias corrections of the next steps
};

// W waves of R registers per lane; GRAD: gradient (and optimiser) or forward;
// LONG: some subgraph of the launch may have its phase tables in parts.
template <int W, int R, bool GRAD, bool LONG>
__device__ __forceinline__ void run(uint8_t* ws, const SubDesc* sd, int b, const SmallArgs& A, Partials part,
                                    float2* dyn, SmallShared& S)
{
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wv = tid >> 6;
    if (wv >= W) return;  // (a barrier counts the waves that are still there)
    constexpr uint32_t T = 64 * W;
    const int n = sd->n, p = A.p, len = sd->lut_len;
    const uint32_t dim = 1u << (n - 1);
    const int nl = n - 1 < 6 ? n - 1 : 6;
    float2* buf = dyn;                                    // W > 1: two exchange buffers
    float2* lut = dyn + A.lut_at;                         // phase tables
    double2* part_of = (double2*)lut;                     // or their parts
    const bool parts = LONG && in_parts(len, p, (int)T);
    const int per = parts ? part_count(len) : len;        // entries per layer
    // the lane of the complement (index bits 0..5 flipped) of this one
    const uint32_t rest = (dim - 1u) & 63u;
    const int lflip = (int)(row_lanes(rest & 15u) | (rest & 48u));
    // index of register r: W = 2^KW waves alternate between two layouts, in
    // which index bits 6.. are the wave and the next KW the low register bits,
    // or the other way round
    constexpr int KW = log2c<W>();
    constexpr uint32_t WM = W - 1;
    const uint32_t lp = row_bits(lane & 15u) | (lane & 48u);
    auto index = [&](int r, int alt) -> uint32_t {
        if constexpr (W == 1) return lp | ((uint32_t)r << 6);
        else return alt ? lp | (((uint32_t)r & WM) << 6) | (wv << (6 + KW)) | ((uint32_t)(r >> KW) << (6 + 2 * KW))
                        : lp | (wv << 6) | ((uint32_t)r << (6 + KW));
    };
    uint16_t c0[R], c1[W > 1 ? R : 1];
    const uint8_t* tab = ws + sd->tab;
    const bool w1 = sd->tabw == 1;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint32_t z = index(r, 0);
        const uint32_t zz = z < dim ? z : 0u;
        c0[r] = w1 ? (uint16_t)tab[zz] : ((const uint16_t*)tab)[zz];
        if constexpr (W > 1) {
            const uint32_t y = index(r, 1);
            c1[r] = w1 ? (uint16_t)tab[y] : ((const uint16_t*)tab)[y];
        }
    }
    auto cut = [&](int r, int alt) -> uint32_t {
        if constexpr (W > 1) return alt ? c1[r] : c0[r];
        else return c0[r];
    };
    const double* gm = A.gamma + (size_t)b * p;
    const double* bt = A.beta + (size_t)b * p;
    double* th = A.theta;
    // optimiser: lane q < 2p of the workgroup holds one angle and its moments
    double my_th = 0.0, my_m = 0.0, my_v = 0.0;
    size_t my_idx = 0;
    const bool opt = GRAD && A.iters > 0, mine = opt && (int)tid < 2 * p;
    if (mine) {
        const int q = (int)tid;
        my_idx = (q < p ? 0 : (size_t)A.B * p) + (size_t)b * p + (q < p ? q : q - p);
        my_th = th[my_idx];
        my_m = A.m[my_idx];
        my_v = A.v[my_idx];
        S.angle[q] = my_th;
    }
    const int32_t t0 = opt ? *A.step : 0;
    if (opt) sync<W>();
    const float amp = (float)(1.0 / sqrt((double)dim));
    float2 v[R], la[GRAD ? R : 1];
    int alt = 0;
    for (int it = 0; it < (opt ? A.iters : 1); ++it) {
        auto gamma_of = [&](int l) { return opt ? S.angle[l] : gm[l]; };
        auto beta_of = [&](int l) { return opt ? S.angle[p + l] : bt[l]; };
        // phase tables, or their parts, and rotation parameters, one sine and cosine
        // each
        for (int i = (int)tid; i < p * per + p; i += T) {
            const int l = i / per;
            const bool phase = l < p;
            int c = i % per;
            if (LONG && parts && c >= PART_LO) c = (c - PART_LO) * PART_LO;
            double sn, cs;
            sincos(phase ? gamma_of(l) * (double)c : beta_of(i - p * per), &sn, &cs);
            if (LONG && parts && phase) {
                part_of[i] = make_double2(cs, -sn);
            } else if (phase) {
                lut[i] = make_float2((float)cs, (float)-sn);
            } else {
                // e^{-i beta X} = f (I - i t X) X^flip as in rx_coef
                const bool tanm = fabs(cs) >= fabs(sn);
                S.rx[i - p * per] = make_float2((float)(tanm ? sn / cs : -cs / sn),
                                                (float)(tanm ? cs * cs : sn * sn));
                double fr, fi;
                cpow_d(tanm ? cs : 0.0, tanm ? 0.0 : -sn, n, fr, fi);
                S.F[i - p * per] = make_float2((float)fr, (float)fi);
            }
        }
        if (opt && it % STEPS == 0)
            for (int i = (int)tid; i < STEPS; i += T) {
                const double t = (double)(t0 + it + i + 1);
                S.k1[i] = 1.0 - pow(A.b1, t);
                S.k2[i] = 1.0 - pow(A.b2, t);
            }
        __syncthreads();
        if (!LONG || !parts) {
#pragma unroll 1
            for (int i = (int)tid; i < p * len; i += T) lut[i] = cmul(lut[i], S.F[i / len]);
            __syncthreads();
        }
        // phase at cut value c with f^n: L = layer l's table, P its parts
        auto phase_of = [&](const float2* L, const double2* P, float2 F, uint32_t c) -> float2 {
            if (!LONG || !parts) return L[c];
            __builtin_amdgcn_sched_barrier(0);  // one amplitude at a time: registers are short
            const double2 a = P[c % PART_LO], b = P[PART_LO + c / PART_LO];
            const double x = a.x * b.x - a.y * b.y, y = a.x * b.y + a.y * b.x, fr = F.x, fi = F.y;
            return make_float2((float)(x * fr - y * fi), (float)(x * fi + y * fr));
        };
        alt = 0;
#pragma clang loop unroll(disable)
        for (int l = 0; l < p; ++l) {
            const float2* L = lut + l * len;
            const double2* P = part_of + l * per;
            const float2 F = LONG ? S.F[l] : make_float2(1.f, 0.f);
            const float t = S.rx[l].x;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float2 f = phase_of(L, P, F, cut(r, alt));
                if (l == 0) v[r] = index(r, 0) < dim ? make_float2(amp * f.x, amp * f.y) : make_float2(0.f, 0.f);
                else v[r] = cmul(v[r], f);
            }
            rotate(v, t, nl);
            if constexpr (W > 1) {
                // (two buffers in turn: one barrier per layer)
                float2* x = buf + (l & 1) * (R * W * 64);
#pragma unroll
                for (int r = 0; r < R; ++r) x[xslot<W>(r, wv, lane)] = v[r];
                __syncthreads();
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const uint32_t q = r ^ (R - 1);
                    const float2 a = x[xslot<W>((r & ~WM) | wv, r & WM, lane)];
                    const float2 o = x[xslot<W>((q & ~WM) | (wv ^ WM), q & WM, lane ^ lflip)];
                    v[r] = make_float2(fmaf(t, o.y, a.x), fmaf(-t, o.x, a.y));
                }
                rx_reg<0>(v, t);
                rx_reg<1>(v, t);
                if constexpr (KW > 2) rx_reg<2>(v, t);
                alt ^= 1;
            } else {
                float2 o[R], u[R];
                lanes_xor(o, v, lflip);
#pragma unroll
                for (int r = 0; r < R; ++r) u[r] = o[r ^ (R - 1)];
                rx_with(v, u, t);
            }
        }
        double e = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r)
            e += ((double)v[r].x * v[r].x + (double)v[r].y * v[r].y) * (double)cut(r, alt);
        e = wave_total(e);
        if (lane == 0) S.se[wv] = e;
        if constexpr (GRAD) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float c = (float)cut(r, alt);
                la[r] = make_float2(c * v[r].x, c * v[r].y);
            }
#pragma clang loop unroll(disable)
            for (int l = p - 1; l >= 0; --l) {
                Back s{-S.rx[l].x, S.rx[l].y, 1.f, 0.0};
                back(v, la, nl, s);
                if constexpr (W > 1) {
                    float2 *x = buf, *y = buf + R * W * 64;
                    __syncthreads();  // the buffers' last readers are done
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        x[xslot<W>(r, wv, lane)] = v[r];
                        y[xslot<W>(r, wv, lane)] = la[r];
                    }
                    __syncthreads();
                    float xa = 0.f, xb = 0.f;
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const uint32_t i = xslot<W>((r & ~WM) | wv, r & WM, lane);
                        const uint32_t q = r ^ (R - 1);
                        const uint32_t j = xslot<W>((q & ~WM) | (wv ^ WM), q & WM, lane ^ lflip);
                        const float2 a = x[i], po = x[j], c = y[i], lo = y[j];
                        float& xr = r & 1 ? xb : xa;
                        xr = fmaf(c.x, po.y, xr);
                        xr = fmaf(-c.y, po.x, xr);
                        v[r] = make_float2(fmaf(s.t, po.y, a.x), fmaf(-s.t, po.x, a.y));
                        la[r] = make_float2(fmaf(s.t, lo.y, c.x), fmaf(-s.t, lo.x, c.y));
                    }
                    s.add(xa + xb);
                    alt ^= 1;
                } else {
                    float2 u[R], po[R], lo[R];
                    lanes_xor(u, v, lflip);
#pragma unroll
                    for (int r = 0; r < R; ++r) po[r] = u[r ^ (R - 1)];
                    lanes_xor(u, la, lflip);
#pragma unroll
                    for (int r = 0; r < R; ++r) lo[r] = u[r ^ (R - 1)];
                    s.add(xb_with(po, la));
                    rx_with(v, po, s.t);
                    rx_with(la, lo, s.t);
                }
                if constexpr (W > 1) {
                    back_reg<0>(v, la, s);
                    back_reg<1>(v, la, s);
                    if constexpr (KW > 2) back_reg<2>(v, la, s);
                }
                double g = 0.0;
#pragma unroll
                for (int r = 0; r < R; ++r)
                    g += (double)((float)cut(r, alt) * fmaf(la[r].x, v[r].y, -la[r].y * v[r].x));
                const float2 F = S.F[l];
                const double gg = wave_total(g * ((double)F.x * F.x + (double)F.y * F.y));
                const double xb = wave_total(s.acc);
                if (lane == 0) {
                    S.sg[l][wv] = gg;
                    S.sb[l][wv] = xb;
                }
                if (l > 0) {
                    const float2* L = lut + l * len;
                    const double2* P = part_of + l * per;
#pragma unroll
                    for (int r = 0; r < R; ++r) {  // conj(f^n) undoes f^n and the phase of this layer
                        float2 f = phase_of(L, P, F, cut(r, alt));
                        f.y = -f.y;
                        v[r] = cmul(v[r], f);
                        la[r] = cmul(la[r], f);
                    }
                }
            }
        }
        sync<W>();  // the waves' sums are written
        auto total = [&](const double* x) {
            double a = 0.0;
            for (int w = 0; w < W; ++w) a += x[w];
            return a;
        };
        const bool last = it + 1 == (opt ? A.iters : 1);
        if (last || (opt && A.E)) {
            if (tid == T - 1) {
                const double x = total(S.se);
                part.e[sd->tile_base] = x;
                if (A.E) A.E[b] = x;
            }
        }
        if constexpr (GRAD) {
            if (!opt && (int)tid < p) {
                const double g = total(S.sg[tid]), x = total(S.sb[tid]);
                part.gg[(size_t)tid * part.total_tiles + sd->tile_base] = g;
                part.gb[((size_t)tid * MAX_GROUPS) * part.total_tiles + sd->tile_base] = x;
                if (A.dgamma) {
                    A.dgamma[(size_t)b * p + tid] = 2.0 * g;
                    A.dbeta[(size_t)b * p + tid] = 2.0 * x;
                }
            }
            if (opt) {
                if (mine) {
                    const int q = (int)tid;
                    const double a = q < p ? total(S.sg[q]) : total(S.sb[q - p]);
                    adam_update(my_th, my_m, my_v, 2.0 * a, S.k1[it % STEPS], S.k2[it % STEPS], A.lr, A.b1, A.b2, A.eps, 1.0);
                    S.angle[q] = my_th;
                }
                sync<W>();
            }
        }
    }
    if (mine) {
        th[my_idx] = my_th;
        A.m[my_idx] = my_m;
        A.v[my_idx] = my_v;
    }
    if constexpr (!GRAD) {
        float2* st = (float2*)(ws + sd->psi);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t z = index(r, alt);
            if (z < dim) st[z] = v[r];
        }
    }
}

}  // namespace

template <bool GRAD, bool LONG>
__global__ __launch_bounds__(ST) __attribute__((amdgpu_waves_per_eu(4))) void k_small(uint8_t* ws, const SubDesc* subs, const int32_t* list, SmallArgs A,
                                              Partials part)
{
    extern __shared__ __align__(16) float2 dyn[];
    __shared__ SmallShared S;
    const int b = list[blockIdx.x];
    const SubDesc* sd = subs + b;
    switch (sd->n) {
    case 13: run<8, 8, GRAD, LONG>(ws, sd, b, A, part, dyn, S); break;
    case 12: run<4, 8, GRAD, LONG>(ws, sd, b, A, part, dyn, S); break;
    case 11: run<4, 4, GRAD, LONG>(ws, sd, b, A, part, dyn, S); break;
    case 10: run<1, 8, GRAD, LONG>(ws, sd, b, A, part, dyn, S); break;
    case 9: run<1, 4, GRAD, LONG>(ws, sd, b, A, part, dyn, S); break;
    case 8: run<1, 2, GRAD, LONG>(ws, sd, b, A, part, dyn, S); break;
    default: run<1, 1, GRAD, LONG>(ws, sd, b, A, part, dyn, S); break;
    }
}

// One layer with its gradient, one qubit at a time in LDS with the plain (cos, sin)
// form of each rotation. At p = 1 the usual starting angle beta = pi/8 is a
// stationary point of every triangle-free subgraph, and Adam's first steps there
// are the rounding noise of dE/dbeta blown up to the step size, so the order of the
// roundings decides the angles: this order is kept, although the kernel above is
// faster. (Five steps on 60 vertices in subgraphs of 9..13: 247 us.)
__device__ inline void rx_pair(float2& a, float2& b, float c, float s)
{
    const float2 na = make_float2(c * a.x + s * b.y, c * a.y - s * b.x);
    const float2 nb = make_float2(c * b.x + s * a.y, c * b.y - s * a.x);
    a = na;
    b = nb;
}

__global__ __launch_bounds__(THREADS) void k_small_layer(uint8_t* ws, const SubDesc* subs, const int32_t* list,
                                                        SmallArgs A, Partials part)
{
    extern __shared__ __align__(16) float2 dyn[];
    __shared__ double red[THREADS / 64];
    __shared__ double s_angle[2];  // gamma, beta
    const uint32_t tid = threadIdx.x;
    const int b = list[blockIdx.x];
    const SubDesc* sd = subs + b;
    const int n = sd->n, len = sd->lut_len;
    const uint32_t dim = 1u << (n - 1), half = dim >> 1, comp = dim - 1;
    float2* ps = dyn;
    float2* la = dyn + A.lut_at;
    float2* lut = dyn + 2 * A.lut_at;
    const uint8_t* tab = ws + sd->tab;
    const bool w1 = sd->tabw == 1;
    auto cut = [&](uint32_t z) { return w1 ? (uint32_t)tab[z] : (uint32_t)((const uint16_t*)tab)[z]; };
    const bool opt = A.iters > 0, mine = opt && tid < 2;
    const size_t idx = (tid == 0 ? 0 : (size_t)A.B) + (size_t)b;  // theta: gamma, then beta, of every subgraph
    double th = 0.0, m = 0.0, v = 0.0;
    if (mine) {
        th = A.theta[idx];
        m = A.m[idx];
        v = A.v[idx];
    }
    if (tid < 2) s_angle[tid] = opt ? th : tid == 0 ? A.gamma[b] : A.beta[b];
    const int32_t t0 = opt ? *A.step : 0;
    const float a0 = (float)(1.0 / sqrt((double)dim));
    for (int it = 0; it < (opt ? A.iters : 1); ++it) {
        __syncthreads();
        for (int i = (int)tid; i < len; i += THREADS) lut[i] = lut_entry(i, s_angle[0]);
        double sn, co;
        sincos(s_angle[1], &sn, &co);
        const float2 cs = make_float2((float)co, (float)sn);
        for (uint32_t z = tid; z < dim; z += THREADS) ps[z] = make_float2(a0, 0.f);
        __syncthreads();
        for (uint32_t z = tid; z < dim; z += THREADS) ps[z] = cmul(ps[z], lut[cut(z)]);
        for (int j = 0; j < n - 1; ++j) {
            __syncthreads();
            for (uint32_t i = tid; i < half; i += THREADS) {
                const uint32_t z = ((i >> j) << (j + 1)) | (i & ((1u << j) - 1u));
                rx_pair(ps[z], ps[z | (1u << j)], cs.x, cs.y);
            }
        }
        __syncthreads();
        for (uint32_t i = tid; i < half; i += THREADS) rx_pair(ps[i], ps[i ^ comp], cs.x, cs.y);
        if (dim == 1 && tid == 0) ps[0] = cmul(ps[0], make_float2(cs.x, -cs.y));
        __syncthreads();
        double e = 0.0;
        for (uint32_t z = tid; z < dim; z += THREADS) {
            const uint32_t c = cut(z);
            e += ((double)ps[z].x * ps[z].x + (double)ps[z].y * ps[z].y) * (double)c;
            la[z] = make_float2((float)c * ps[z].x, (float)c * ps[z].y);
        }
        e = block_sum(e, red);
        double xb = 0.0;
        // the top qubit (complement pairs; for n = 1 the single amplitude with
        // itself) first, then qubits n-2..0
        for (int j = n - 1; j >= 0; --j) {
            __syncthreads();
            float a = 0.f;
            if (j == n - 1 && dim == 1) {
                if (tid == 0) {
                    a += la[0].x * ps[0].y - la[0].y * ps[0].x;
                    ps[0] = cmul(ps[0], make_float2(cs.x, cs.y));
                    la[0] = cmul(la[0], make_float2(cs.x, cs.y));
                }
            } else {
                for (uint32_t i = tid; i < half; i += THREADS) {
                    const uint32_t z = j == n - 1 ? i : ((i >> j) << (j + 1)) | (i & ((1u << j) - 1u));
                    const uint32_t z1 = j == n - 1 ? i ^ comp : z | (1u << j);
                    a += la[z].x * ps[z1].y - la[z].y * ps[z1].x;
                    a += la[z1].x * ps[z].y - la[z1].y * ps[z].x;
                    rx_pair(ps[z], ps[z1], cs.x, -cs.y);
                    rx_pair(la[z], la[z1], cs.x, -cs.y);
                }
            }
            xb += (double)a;
        }
        __syncthreads();
        xb = block_sum(xb, red);
        double gg = 0.0;
        for (uint32_t z = tid; z < dim; z += THREADS)
            gg += (double)((float)cut(z) * (la[z].x * ps[z].y - la[z].y * ps[z].x));
        gg = block_sum(gg, red);
        if (tid == 0) {
            part.e[sd->tile_base] = e;
            if (A.E) A.E[b] = e;
            if (!opt) {
                part.gg[sd->tile_base] = gg;
                part.gb[sd->tile_base] = xb;
                if (A.dgamma) {
                    A.dgamma[b] = 2.0 * gg;
                    A.dbeta[b] = 2.0 * xb;
                }
            }
            red[0] = gg;
            red[1] = xb;
        }
        __syncthreads();
        if (mine) {
            const double t = (double)(t0 + it + 1);
            adam_update(th, m, v, 2.0 * red[tid], 1.0 - pow(A.b1, t), 1.0 - pow(A.b2, t), A.lr, A.b1, A.b2, A.eps, 1.0);
            s_angle[tid] = th;
        }
    }
    if (mine) {
        A.theta[idx] = th;
        A.m[idx] = m;
        A.v[idx] = v;
    }
}

// max_n, max_len: the list's largest qubit count, and phase tables by waves (small_waves)
hipError_t launch_small(uint8_t* ws, const SubDesc* subs, const int32_t* list, int nlist, int max_n,
                        const int (&max_len)[3], bool grad, SmallArgs A, Partials part, hipStream_t s)
{
    if (nlist <= 0) return hipSuccess;
    const int len = std::max(max_len[0], std::max(max_len[1], max_len[2]));
    if (grad && A.p == 1) {
        A.lut_at = 1u << (max_n - 1);
        hipLaunchKernelGGL(k_small_layer, dim3(nlist), dim3(THREADS), (2 * A.lut_at + len) * sizeof(float2), s, ws,
                           subs, list, A, part);
        return hipGetLastError();
    }
    A.lut_at = max_n >= 11 ? 2u << (max_n - 1) : 0u;
    bool parts = false;
    for (int k = 0; k < 3; ++k) parts |= in_parts(max_len[k], A.p, 64 << (k ? k + 1 : 0));
    size_t lds = std::min(A.p * len, LUT_CAP) * sizeof(float2);
    if (parts) lds = std::max(lds, A.p * part_count(len) * sizeof(double2));
    lds += A.lut_at * sizeof(float2);
    const int threads = max_n <= 10 ? 64 : max_n <= 12 ? 256 : ST;
    auto* k = grad ? (parts ? k_small<true, true> : k_small<true, false>)
                   : (parts ? k_small<false, true> : k_small<false, false>);
    hipLaunchKernelGGL(k, dim3(nlist), dim3(threads), lds, s, ws, subs, list, A, part);
    return hipGetLastError();
}

}  // namespace pq

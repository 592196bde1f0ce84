// Tile passes on wide tiles: 2^14 amplitudes per workgroup instead of 2^12,
// for the subgraphs where that saves whole passes over the state.
//
// What a pass computes, the pass kinds, the reduced state, the mirror-paired
// group 0, the factored rotation with its flip mask and the adjoint sweep are
// those of sim.hip. What differs is the tile: 512 lanes hold 32 amplitudes
// each, so group 0 rotates 13 low qubits and the top one, and a strided group
// up to 12 qubits. Subgraphs of 21..26 qubits then need two groups instead of
// three and those of 29 and 30 three instead of four: a layer costs one pass
// over the state instead of two (two instead of three).
//
// Register layouts (tile position q, 14 bits; lane id = 9 bits):
//   LLIN  registers = bits 9..13, lanes = bits 0..8 (coalesced rows)
//   LL1   registers = bits 4..8,  lanes = bits 0..3 and 9..13
// Bits 0..3 are rotated in LL1 across the lanes of a row of 16 (lane.h). That
// costs one instruction per amplitude and bit more than a register bit, and
// saves a third layout and its LDS exchange.
// The forward passes exchange the real and the imaginary parts one after the
// other through 66 KB of LDS, so that two workgroups share a CU; the backward
// passes hold two states in registers (two waves per SIMD), so one workgroup
// owns the CU's LDS and exchanges whole amplitudes.
//
// The 12-qubit group's forward passes take tiles in pairs (see k_fwd_wide).
//
// Measured on 1.68e8 amplitudes (ten 25-qubit states, one launch; algorithmic
// bytes): group 0 middle forward 557 us (5.1 TB/s), 11-qubit middle forward
// 790 us (3.6 TB/s: a copy of 64-byte rows reaches 3.6), group 0 middle
// backward 1.50 ms (2.8 TB/s), 11-qubit middle backward 1.48 ms (2.8 TB/s).
// The forward passes are bound by memory. The backward ones issue 6,400 (group
// 0) and 4,830 vector instructions per wave, 0.57 of the time at the vector
// units' rate, and their loads and stores do not overlap that: at 210 to 226
// registers a lane, one workgroup fills the CU. On 4096-amplitude tiles the two passes
// that each of these replaces take 5.9 + 4.5 and 4.9 + 4.5 ns per 1000
// amplitudes, against 8.9 and 8.8.
//
// Phases, <C> and the gamma terms always happen in LL1, and the cut tables of
// these tiles are stored in that layout's order (lane, register), so a lane
// reads its 32 entries as two (1-byte entries) or four 16-byte loads.
#include "tile.h"

namespace pq {

namespace {

constexpr int WT = WIDE_THREADS, WR = WIDE_REGS;
enum { LLIN = 0, LL1 = 1 };
constexpr uint32_t EX_SLOTS = WIDE_TILE + WIDE_TILE / 32;  // one pad slot per 32 amplitudes
constexpr uint32_t HALF_SLOTS = EX_SLOTS + 32;  // of a pair: its halves in different banks

// A thread's place: its tile position without register bits, and, with two tiles per
// workgroup (PAIR), which of the two. The halves of a pair differ in the index bit
// above the C passive tile bits; lanes run over it right after those, so a pair's
// rows are twice as long.
template <int L>
__device__ inline uint32_t thread_part(uint32_t tid)
{
    return L == LLIN ? tid : row_bits(tid & 15u) | ((tid >> 4) << 9);
}
struct Place {
    uint32_t q, half;
};
template <int L, bool PAIR, int C>
__device__ inline Place place(uint32_t tid)
{
    if constexpr (!PAIR) return {thread_part<L>(tid), 0u};
    else if constexpr (L == LLIN) return {(tid & ((1u << C) - 1u)) | ((tid >> (C + 1)) << C), (tid >> C) & 1u};
    else return {row_bits(tid & 15u) | ((tid >> 5) << 9), (tid >> 4) & 1u};
}
template <int L>
__host__ __device__ constexpr uint32_t reg_part(uint32_t r)
{
    return L == LLIN ? (r << 9) : (r << 4);
}
__host__ __device__ constexpr uint32_t slot(uint32_t q) { return q + (q >> 5); }  // additive over disjoint bits

// Layout change of one state through a buffer of single floats. In LL1 a wave
// reads and writes only its own part of the buffer (tile bits 11..13, or 10..13 of
// both tiles of a pair), so
// after a change to LL1 no barrier is needed before the next one writes.
template <int LF, int LT, bool PAIR, int C>
__device__ inline void xchg(float* ex, uint32_t tid, float2 (&v)[WR])
{
    const Place f = place<LF, PAIR, C>(tid), o = place<LT, PAIR, C>(tid);
    float* p = ex + f.half * HALF_SLOTS + slot(f.q);
    const float* s = ex + o.half * HALF_SLOTS + slot(o.q);
#pragma unroll
    for (int r = 0; r < WR; ++r) p[slot(reg_part<LF>(r))] = v[r].x;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < WR; ++r) v[r].x = s[slot(reg_part<LT>(r))];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < WR; ++r) p[slot(reg_part<LF>(r))] = v[r].y;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < WR; ++r) v[r].y = s[slot(reg_part<LT>(r))];
    if constexpr (LT == LLIN) __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
}

// The same for whole amplitudes (backward passes).
template <int LF, int LT>
__device__ inline void xchg2(float2* ex, uint32_t tid, float2 (&v)[WR])
{
    float2* p = ex + slot(thread_part<LF>(tid));
    const float2* s = ex + slot(thread_part<LT>(tid));
#pragma unroll
    for (int r = 0; r < WR; ++r) p[slot(reg_part<LF>(r))] = v[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < WR; ++r) v[r] = s[slot(reg_part<LT>(r))];
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
}

template <int K>
__device__ inline void rx_bit(float2 (&v)[WR], float t)
{
#pragma unroll
    for (int r = 0; r < WR; ++r)
        if (!(r & (1 << K))) rx_tan(v[r], v[r | (1 << K)], t);
}

// NB: qubits of the group (0: group 0); C: its lowest active tile bit
template <int NB>
constexpr int low_bit()
{
    return NB == 0 ? 0 : WIDE_BITS - NB;
}

// is tile bit q an active qubit of the group?
template <int NB>
__host__ __device__ constexpr bool active(int q)
{
    return q >= (NB == 0 ? 0 : WIDE_BITS - NB);
}
// active bits that layout L rotates: 9..13 in LLIN, 0..8 in LL1
template <int L, int NB>
__host__ __device__ constexpr int active_count()
{
    int n = 0;
    for (int q = L == LLIN ? 9 : 0; q < (L == LLIN ? 14 : 9); ++q) n += active<NB>(q);
    return n;
}

template <int L, int NB>
__device__ inline void rx_round(float2 (&v)[WR], float t)
{
    constexpr int Q = L == LLIN ? 9 : 4;
    if constexpr (active<NB>(Q)) rx_bit<0>(v, t);
    if constexpr (active<NB>(Q + 1)) rx_bit<1>(v, t);
    if constexpr (active<NB>(Q + 2)) rx_bit<2>(v, t);
    if constexpr (active<NB>(Q + 3)) rx_bit<3>(v, t);
    if constexpr (active<NB>(Q + 4)) rx_bit<4>(v, t);
    if constexpr (L == LL1) {
        if constexpr (active<NB>(3)) rx_lane<3>(v, t);
        if constexpr (active<NB>(2)) rx_lane<2>(v, t);
        if constexpr (active<NB>(1)) rx_lane<1>(v, t);
        if constexpr (active<NB>(0)) rx_lane<0>(v, t);
    }
}

// sum over one register bit of Im conj(lam(z)) psi(z ^ bit), both directions
template <int K>
__device__ inline float xb_bit(const float2 (&ps)[WR], const float2 (&la)[WR])
{
    float a0 = 0.f, a1 = 0.f;
#pragma unroll
    for (int r = 0; r < WR; ++r) {
        if (r & (1 << K)) continue;
        const int r1 = r | (1 << K);
        a0 = fmaf(la[r].x, ps[r1].y, a0);
        a0 = fmaf(-la[r].y, ps[r1].x, a0);
        a1 = fmaf(la[r1].x, ps[r].y, a1);
        a1 = fmaf(-la[r1].y, ps[r].x, a1);
    }
    return a0 + a1;
}

// the beta terms of the layout's bits: FP32 over a lane's 32 amplitudes, FP64 over bits
template <int L, int NB>
__device__ inline double xb_round(const float2 (&ps)[WR], const float2 (&la)[WR])
{
    constexpr int Q = L == LLIN ? 9 : 4;
    double a = 0.0;
    if constexpr (active<NB>(Q)) a += (double)xb_bit<0>(ps, la);
    if constexpr (active<NB>(Q + 1)) a += (double)xb_bit<1>(ps, la);
    if constexpr (active<NB>(Q + 2)) a += (double)xb_bit<2>(ps, la);
    if constexpr (active<NB>(Q + 3)) a += (double)xb_bit<3>(ps, la);
    if constexpr (active<NB>(Q + 4)) a += (double)xb_bit<4>(ps, la);
    if constexpr (L == LL1) {
        if constexpr (active<NB>(3)) a += (double)xb_lane<3>(ps, la);
        if constexpr (active<NB>(2)) a += (double)xb_lane<2>(ps, la);
        if constexpr (active<NB>(1)) a += (double)xb_lane<1>(ps, la);
        if constexpr (active<NB>(0)) a += (double)xb_lane<0>(ps, la);
    }
    return a;
}

// One RX segment, LLIN -> LL1 (UP) or back.
template <int NB, bool UP, bool PAIR>
__device__ inline void seg_rot(float2 (&v)[WR], float* ex, float t, uint32_t tid)
{
    constexpr int A = UP ? LLIN : LL1, B = UP ? LL1 : LLIN;
    rx_round<A, NB>(v, t);
    xchg<A, B, PAIR, low_bit<NB>()>(ex, tid, v);
    rx_round<B, NB>(v, t);
}

// the same, LLIN -> LL1, with whole-amplitude exchanges
template <int NB>
__device__ inline void seg_rot2(float2 (&v)[WR], float2* ex, float t, uint32_t tid)
{
    rx_round<LLIN, NB>(v, t);
    xchg2<LLIN, LL1>(ex, tid, v);
    rx_round<LL1, NB>(v, t);
}

// Inverse rotation of psi and lambda with the beta terms of one layout: the
// inner products are taken before the rotations, on states scaled by
// |f|^-done, so they are multiplied back by fsq^done.
template <int L, int NB>
__device__ inline void bwd_round(float2 (&ps)[WR], float2 (&la)[WR], const RxC& rc, float& wdone, double& acc)
{
    acc += (double)wdone * xb_round<L, NB>(ps, la);
    __builtin_amdgcn_sched_barrier(0);
    rx_round<L, NB>(ps, -rc.t);
    rx_round<L, NB>(la, -rc.t);
#pragma unroll
    for (int k = 0; k < active_count<L, NB>(); ++k) wdone *= rc.fsq;
    __builtin_amdgcn_sched_barrier(0);
}

template <int NB, bool UP>
__device__ inline void seg_bwd(float2 (&ps)[WR], float2 (&la)[WR], float2* ex, const RxC& rc, uint32_t tid,
                               double& acc)
{
    constexpr int A = UP ? LLIN : LL1, B = UP ? LL1 : LLIN;
    float wdone = 1.f;
    bwd_round<A, NB>(ps, la, rc, wdone, acc);
    xchg2<A, B>(ex, tid, ps);
    xchg2<A, B>(ex, tid, la);
    bwd_round<B, NB>(ps, la, rc, wdone, acc);
}

__device__ inline void scale_regs(float2 (&v)[WR], float2 f)
{
#pragma unroll
    for (int r = 0; r < WR; ++r) v[r] = cmul(v[r], f);
}

// tile t of the group: make_geo with the group's size known
template <int NB>
__device__ inline Geo wide_geo(const SubDesc* sd, int g, uint32_t t)
{
    Geo r;
    r.c = low_bit<NB>();
    r.nb = NB == 0 ? WIDE_BITS : NB;
    r.g0 = NB == 0 ? 0 : sd->gstart[g];
    r.mir = NB == 0 ? (1u << (sd->n - 1)) - 1u : 0u;
    if constexpr (NB == 0) {
        r.zb = t << (WIDE_BITS - 1);
    } else {
        const int L = r.g0 - r.c;  // fixed bits between the passive block and the group
        r.zb = ((t & ((1u << L) - 1u)) << r.c) | ((t >> L) << (r.g0 + NB));
    }
    return r;
}

template <int L, bool G0, bool PAIR = false, int C = 0>
__device__ inline void load_state(float2 (&v)[WR], const float2* st, const Geo& geo, uint32_t tid)
{
    const Place at = place<L, PAIR, C>(tid);
    uint32_t base = (geo.zb ^ gmapT<G0, WIDE_BITS>(geo, at.q) ^ (at.half << C)) << 3;
    asm volatile("" : "+v"(base));  // keeps the shift out of the per-register XOR
#pragma unroll
    for (int r = 0; r < WR; ++r) v[r] = at_off(st, base ^ (gmapT<G0, WIDE_BITS>(geo, reg_part<L>(r)) << 3));
    __builtin_amdgcn_sched_barrier(0);
}

// store slot q to amplitude q ^ m
template <int L, bool G0, bool PAIR = false, int C = 0>
__device__ inline void store_state(const float2 (&v)[WR], float2* st, const Geo& geo, uint32_t tid, uint32_t m)
{
    __builtin_amdgcn_sched_barrier(0);
    const Place at = place<L, PAIR, C>(tid);
    uint32_t base =
        (geo.zb ^ gmapT<G0, WIDE_BITS>(geo, at.q) ^ gmapT<G0, WIDE_BITS>(geo, m) ^ (at.half << C)) << 3;
    asm volatile("" : "+v"(base));
#pragma unroll
    for (int r = 0; r < WR; ++r) at_off(st, base ^ (gmapT<G0, WIDE_BITS>(geo, reg_part<L>(r)) << 3)) = v[r];
}

// The lane's 32 cut values in LL1, two 16-bit values per word, for slots that
// hold amplitude q ^ m, m = M (the group's bits) where flip is set, else 0: the
// lane part of M moves the 32-entry row, its register part permutes the words.
struct Cuts {
    uint32_t w[WR / 2];
    __device__ uint32_t at(int r) const { return (r & 1) ? w[r >> 1] >> 16 : w[r >> 1] & 0xFFFFu; }
};

template <uint32_t M>
__device__ inline void load_cuts(Cuts& c, const uint8_t* tab, int width, uint32_t tid, bool flip)
{
    constexpr uint32_t ROW = row_lanes(M & 15u) | (((M >> 9) & 31u) << 4), R = (M >> 4) & 31u;
    const uint32_t row = flip ? tid ^ ROW : tid;
    if (width == 1) {
        const uint4* p = (const uint4*)(tab + (size_t)row * WR);
        const uint4 a = p[0], b = p[1];
        const uint32_t s[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
        for (int i = 0; i < 8; ++i) {  // bytes 0, 1 and 2, 3 to 16 bits
            c.w[2 * i] = __builtin_amdgcn_perm(0u, s[i], 0x0C010C00u);
            c.w[2 * i + 1] = __builtin_amdgcn_perm(0u, s[i], 0x0C030C02u);
        }
    } else {
        const uint4* p = (const uint4*)(tab + (size_t)row * WR * 2);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint4 a = p[i];
            c.w[4 * i] = a.x;
            c.w[4 * i + 1] = a.y;
            c.w[4 * i + 2] = a.z;
            c.w[4 * i + 3] = a.w;
        }
    }
    if (flip) {
        uint32_t x[WR / 2];
#pragma unroll
        for (int i = 0; i < WR / 2; ++i) x[i] = c.w[i ^ (R >> 1)];
#pragma unroll
        for (int i = 0; i < WR / 2; ++i) c.w[i] = (R & 1u) ? (x[i] >> 16) | (x[i] << 16) : x[i];
    }
}

__device__ inline const uint8_t* tile_tab(const uint8_t* ws, const SubDesc* sd, int g, uint32_t t)
{
    return (g == 0 ? ws + sd->tab : ws + sd->tabB) + (size_t)t * WIDE_TILE * sd->tabw;
}

// tile bits of the group's qubits (the ones a flip permutes)
__host__ __device__ constexpr uint32_t group_bits(int c) { return ((uint32_t)WIDE_TILE - 1u) & ~((1u << c) - 1u); }

enum { F_FIRST = 0, F_SINGLE = 1, F_MID = 2, F_LAST = 3 };
enum { B_FUSED = 0, B_SINGLE = 1, B_MID = 2, B_LAST = 3 };

}  // namespace

// Forward pass. FIRST synthesises the phased |+> in LL1 and walks to LLIN;
// MID walks to LL1, phases and walks back; SINGLE and LAST end in LL1.
//
// The strided group of 12 qubits (26-qubit states) has rows of 32 bytes. Its
// workgroups take a pair of neighbouring tiles each (1024 threads, the same
// registers and LDS per CU as two workgroups), which doubles the rows, and the XCDs
// work in eight parts of a state instead of next to each other, so that the rows in
// flight are spread over the memory channels. Four states, p = 3: 2.43 ms without
// either, 2.25 with pairs, 2.16 with both; p = 4 2.96, 2.91, 2.75. (11 qubits, 64-byte
// rows, one state of 25 qubits, p = 3: 214 us, 225 with pairs, 242 with both. The
// backward passes have no registers for pairs, and with the parts they are slower.)
template <int NB, int KIND, bool PAIR = false>
__global__ __launch_bounds__(PAIR ? 2 * WT : WT) __attribute__((amdgpu_waves_per_eu(4))) void k_fwd_wide(
    uint8_t* ws, const SubDesc* subs, const int2* work, PassOps ops, Partials part)
{
    constexpr int THR = PAIR ? 2 * WT : WT, C = low_bit<NB>();
    extern __shared__ float wsm[];
    float* ex = wsm;
    float2* lut = (float2*)(wsm + (PAIR ? 2 * HALF_SLOTS : EX_SLOTS));
    __shared__ double red[THR / 64];
    constexpr bool HAS_PRE = KIND != F_FIRST, HAS_PH = KIND == F_FIRST || KIND == F_MID;
    const uint32_t tid = threadIdx.x;
    int2 wk = work[blockIdx.x];
    if constexpr (PAIR) {
        // each XCD takes an eighth of a state's tiles, four pairs in a row at a time
        constexpr uint32_t np = 1u << (NB - 1);  // tiles of a state: one strided group
        const uint32_t j = blockIdx.x % (np / 2);
        wk = work[blockIdx.x / (np / 2) * np];
        wk.y = (int)((j & 7u) * (np / 8) + (j >> 5) * 8u + ((j >> 3) & 3u) * 2u);
    }
    const SubDesc* sd = subs + wk.x;
    const uint32_t t = (uint32_t)wk.y;
    constexpr bool G0 = NB == 0;
    const int g = G0 ? 0 : ops.group;
    const Geo geo = wide_geo<NB>(sd, g, t);
    const float2* src = (const float2*)(ws + sd->psi + (uint64_t)ops.psi_in * state_bytes(sd->n));
    float2* st = (float2*)(ws + sd->psi + (uint64_t)ops.psi_out * state_bytes(sd->n));
    const RxCoef* cf = (const RxCoef*)(ws + sd->coef);
    constexpr uint32_t gb = group_bits(low_bit<NB>());
    RxC pre{}, post{};
    if constexpr (HAS_PRE) pre = load_rx(cf, ops.pre, g);
    if constexpr (HAS_PH) post = load_rx(cf, ops.post, g);
    const uint32_t m_pre = (HAS_PRE && pre.flip) ? gb : 0u;
    const uint32_t m_end = m_pre ^ ((HAS_PH && post.flip) ? gb : 0u);
    float2 v[WR];
    if constexpr (HAS_PRE) load_state<LLIN, G0, PAIR, C>(v, src, geo, tid);
    Cuts cr;
    if constexpr (KIND != F_SINGLE) {  // (LAST: m_pre = m_end)
        const uint32_t half = PAIR ? (tid >> 4) & 1u : 0u, row = PAIR ? (tid & 15u) | ((tid >> 5) << 4) : tid;
        load_cuts<gb>(cr, tile_tab(ws, sd, g, t + half), sd->tabw, row, m_pre != 0u);
    }
    if constexpr (HAS_PH) {
        // phase table with the factors of the segments before and after it
        // (FIRST: and the amplitude of |+>) folded in
        const int len = sd->lut_len;
        const float2* L = (const float2*)(ws + sd->lut) + (size_t)ops.ph * len;
        const float amp = (float)(1.0 / sqrt((double)(1ull << (sd->n - 1))));
        const float2 F = HAS_PRE ? cmul(pre.Ff, post.Ff) : make_float2(amp * post.Ff.x, amp * post.Ff.y);
        for (int i = tid; i < len; i += THR) lut[i] = cmul(L[i], F);
        if constexpr (!HAS_PRE) __syncthreads();  // (MID: the exchange's barriers come before the table is read)
    }
    if constexpr (HAS_PRE) {
        seg_rot<NB, true, PAIR>(v, ex, pre.t, tid);
        if constexpr (!HAS_PH) scale_regs(v, pre.Ff);
    }
    if constexpr (HAS_PH) {
#pragma unroll
        for (int r = 0; r < WR; ++r) {
            const float2 f = lut[cr.at(r)];
            v[r] = HAS_PRE ? cmul(v[r], f) : f;
        }
        seg_rot<NB, false, PAIR>(v, ex, post.t, tid);
        store_state<LLIN, G0, PAIR, C>(v, st, geo, tid, m_end);
    } else {
        double acc = 0.0;
        if constexpr (KIND == F_LAST) {
#pragma unroll
            for (int r = 0; r < WR; ++r)
                acc += ((double)v[r].x * v[r].x + (double)v[r].y * v[r].y) * (double)cr.at(r);
        }
        store_state<LL1, G0, PAIR, C>(v, st, geo, tid, m_end);
        if constexpr (KIND == F_LAST) {
            acc = block_sum(acc, red);
            if (tid == 0) part.e[sd->tile_base + t] = acc;  // (a pair's sum at its first tile)
            if (PAIR && tid == 1) part.e[sd->tile_base + t + 1] = 0.0;
        }
    }
}

// Backward pass (kinds as in sim.hip). SPSI: psi is stored too.
template <int NB, int KIND, bool SPSI>
__global__ __launch_bounds__(WT) __attribute__((amdgpu_waves_per_eu(2))) void k_bwd_wide(uint8_t* ws,
                                                                                      const SubDesc* subs,
                                                                                      const int2* work, PassOps ops,
                                                                                      Partials part)
{
    extern __shared__ float2 wsm2[];
    float2* ex = wsm2;
    float2* lut = wsm2 + EX_SLOTS;
    __shared__ double red[3 * WT / 64];
    const uint32_t tid = threadIdx.x;
    const int2 wk = work[blockIdx.x];
    const SubDesc* sd = subs + wk.x;
    const uint32_t t = (uint32_t)wk.y;
    constexpr bool G0 = NB == 0;
    const int g = G0 ? 0 : ops.group;
    const Geo geo = wide_geo<NB>(sd, g, t);
    float2* sp = (float2*)(ws + sd->psi + (uint64_t)ops.psi_in * state_bytes(sd->n));
    float2* sl = (float2*)(ws + sd->lam);
    const RxCoef* cf = (const RxCoef*)(ws + sd->coef);
    const int T = part.total_tiles;
    const int tile = sd->tile_base + (int)t;
    constexpr uint32_t gb = group_bits(low_bit<NB>());
    const RxC pre = load_rx(cf, ops.pre, g);
    RxC post{};
    if constexpr (KIND == B_MID) post = load_rx(cf, ops.post, g);
    const uint32_t m_pre = pre.flip ? gb : 0u;
    const uint32_t m_end = m_pre ^ ((KIND == B_MID && post.flip) ? gb : 0u);
    float2 ps[WR], la[WR];
    if constexpr (KIND != B_LAST) load_state<LLIN, G0>(ps, sp, geo, tid);
    if constexpr (KIND != B_FUSED) load_state<LLIN, G0>(la, sl, geo, tid);
    Cuts cr;
    if constexpr (KIND != B_SINGLE) load_cuts<gb>(cr, tile_tab(ws, sd, g, t), sd->tabw, tid, m_pre != 0u);
    if constexpr (KIND == B_MID || KIND == B_LAST) {
        // MID: the conjugate phase table with the inverse factors of the
        // segments before and after it. LAST: the phase table of layer 1 with
        // the amplitude of |+> and the conjugate of the inverse factor of
        // RX(pre) (every sum of that pass is bilinear in conj(lambda) and psi)
        const int len = sd->lut_len;
        const float2* L = (const float2*)(ws + sd->lut) + (size_t)ops.ph * len;
        const float amp = (float)(1.0 / sqrt((double)(1ull << (sd->n - 1))));
        const float2 F = KIND == B_MID ? cmul(pre.Fi, post.Fi) : make_float2(amp * pre.Fi.x, -amp * pre.Fi.y);
        for (int i = tid; i < len; i += WT) {
            const float2 e = L[i];
            lut[i] = cmul(make_float2(e.x, KIND == B_MID ? -e.y : e.y), F);
        }
    }
    double acc_pre = 0.0, acc_ph = 0.0, acc_post = 0.0, acc_e = 0.0;
    if constexpr (KIND == B_LAST) {
        seg_rot2<NB>(la, ex, -pre.t, tid);
        float a[2] = {0.f, 0.f};
#pragma unroll
        for (int r = 0; r < WR; ++r) {
            const uint32_t c = cr.at(r);
            ps[r] = lut[c];
            a[r & 1] = fmaf((float)c, fmaf(la[r].x, ps[r].y, -la[r].y * ps[r].x), a[r & 1]);
        }
        acc_ph = (double)a[0] + (double)a[1];
        // beta terms in both layouts
        acc_pre += xb_round<LL1, NB>(ps, la);
        xchg2<LL1, LLIN>(ex, tid, ps);
        xchg2<LL1, LLIN>(ex, tid, la);
        acc_pre += xb_round<LLIN, NB>(ps, la);
    } else if constexpr (KIND == B_FUSED) {
        seg_rot2<NB>(ps, ex, pre.t, tid);
        scale_regs(ps, pre.Ff);
#pragma unroll
        for (int r = 0; r < WR; ++r) {
            const uint32_t ci = cr.at(r);
            const float c = (float)ci;
            acc_e += ((double)ps[r].x * ps[r].x + (double)ps[r].y * ps[r].y) * (double)ci;
            la[r] = make_float2(c * ps[r].x, c * ps[r].y);
        }
        seg_bwd<NB, false>(ps, la, ex, pre, tid, acc_pre);
        scale_regs(la, pre.Fi);
        store_state<LLIN, G0>(la, sl, geo, tid, 0u);
    } else {
        seg_bwd<NB, true>(ps, la, ex, pre, tid, acc_pre);
        if constexpr (KIND == B_SINGLE) {
            if constexpr (SPSI) {
                scale_regs(ps, pre.Fi);
                store_state<LL1, G0>(ps, sp, geo, tid, m_end);
            }
            scale_regs(la, pre.Fi);
            store_state<LL1, G0>(la, sl, geo, tid, m_end);
        } else {
            float a[2] = {0.f, 0.f};
#pragma unroll
            for (int r = 0; r < WR; ++r)
                a[r & 1] = fmaf((float)cr.at(r), fmaf(la[r].x, ps[r].y, -la[r].y * ps[r].x), a[r & 1]);
            acc_ph = ((double)a[0] + (double)a[1]) * (double)(pre.Fi.x * pre.Fi.x + pre.Fi.y * pre.Fi.y);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < WR; ++r) {
                const float2 f = lut[cr.at(r)];
                ps[r] = cmul(ps[r], f);
                la[r] = cmul(la[r], f);
            }
            __builtin_amdgcn_sched_barrier(0);
            seg_bwd<NB, false>(ps, la, ex, post, tid, acc_post);
            acc_post /= (double)post.Fi.x * post.Fi.x + (double)post.Fi.y * post.Fi.y;
            if constexpr (SPSI) store_state<LLIN, G0>(ps, sp, geo, tid, m_end);
            store_state<LLIN, G0>(la, sl, geo, tid, m_end);
        }
    }
    double s0 = KIND == B_FUSED ? acc_e : acc_ph, s1 = acc_pre, s2 = acc_post;
    block_sum3(s0, s1, s2, red);
    if (tid == 0) {
        if constexpr (KIND == B_FUSED) part.e[tile] = s0;
        if constexpr (KIND == B_MID || KIND == B_LAST) part.gg[(size_t)ops.ph * T + tile] = s0;
        part.gb[((size_t)ops.pre * MAX_GROUPS + g) * T + tile] = s1;
        if constexpr (KIND == B_MID) part.gb[((size_t)ops.post * MAX_GROUPS + g) * T + tile] = s2;
    }
}

// ---------------------------------------------------------------------------
// launchers. Chain codes: 3 = group 0, 7..12 = a strided group of that many
// qubits (the even splits of 21..26, 29 and 30 qubits). Only the middle one of
// three groups has passes of its own (SINGLE): 8 qubits of 29 and 30. Gradients
// do not run groups of 12 (26 qubits).
// ---------------------------------------------------------------------------
using PassKernel = void (*)(uint8_t*, const SubDesc*, const int2*, PassOps, Partials);

template <int KIND>
static PassKernel fwd_kernel(int chain)
{
    switch (chain) {
    case 3: return k_fwd_wide<0, KIND>;
    case 7: return k_fwd_wide<7, KIND>;
    case 8: return k_fwd_wide<8, KIND>;
    case 9: return k_fwd_wide<9, KIND>;
    case 10: return k_fwd_wide<10, KIND>;
    case 11: return k_fwd_wide<11, KIND>;
    case 12: return k_fwd_wide<12, KIND, true>;
    default: return nullptr;
    }
}

template <int KIND, bool SPSI>
static PassKernel bwd_kernel(int chain)
{
    switch (chain) {
    case 3: return k_bwd_wide<0, KIND, SPSI>;
    case 7: return k_bwd_wide<7, KIND, SPSI>;
    case 8: return k_bwd_wide<8, KIND, SPSI>;
    case 9: return k_bwd_wide<9, KIND, SPSI>;
    case 10: return k_bwd_wide<10, KIND, SPSI>;
    case 11: return k_bwd_wide<11, KIND, SPSI>;
    default: return nullptr;
    }
}

hipError_t launch_fwd_wide(uint8_t* ws, const SubDesc* subs, const int2* work, int nwork, int chain, PassOps ops,
                           Partials part, int lut_max, hipStream_t s)
{
    if (nwork <= 0) return hipSuccess;
    const bool pair = chain == 12;
    if (pair && nwork % (1 << 11)) return hipErrorInvalidValue;  // whole states of 26 qubits
    const size_t lds = (pair ? 2 * HALF_SLOTS : EX_SLOTS) * sizeof(float) + (size_t)lut_max * sizeof(float2);
    PassKernel k = nullptr;
    if (ops.init) k = chain == 3 ? k_fwd_wide<0, F_FIRST> : nullptr;
    else if (ops.epi_e) k = fwd_kernel<F_LAST>(chain);
    else if (ops.ph >= 0) k = fwd_kernel<F_MID>(chain);
    else k = chain == 8 ? k_fwd_wide<8, F_SINGLE> : nullptr;
    if (!k) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k, dim3(pair ? nwork / 2 : nwork), dim3(pair ? 2 * WT : WT), lds, s, ws, subs, work, ops, part);
    return hipGetLastError();
}

hipError_t launch_bwd_wide(uint8_t* ws, const SubDesc* subs, const int2* work, int nwork, int chain, PassOps ops,
                           Partials part, int lut_max, hipStream_t s)
{
    if (nwork <= 0) return hipSuccess;
    const size_t lds = EX_SLOTS * sizeof(float2) + (size_t)lut_max * sizeof(float2);
    PassKernel k = nullptr;
    // the last pass mirrors the first forward pass (group 0 of layer 1)
    if (ops.last) k = ops.group == 0 && chain == 3 ? k_bwd_wide<0, B_LAST, false> : nullptr;
    else if (ops.fused) k = bwd_kernel<B_FUSED, false>(chain);
    else if (ops.ph >= 0) k = ops.nopsi ? bwd_kernel<B_MID, false>(chain) : bwd_kernel<B_MID, true>(chain);
    else if (chain == 8) k = ops.nopsi ? k_bwd_wide<8, B_SINGLE, false> : k_bwd_wide<8, B_SINGLE, true>;
    if (!k) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k, dim3(nwork), dim3(WT), lds, s, ws, subs, work, ops, part);
    return hipGetLastError();
}

}  // namespace pq

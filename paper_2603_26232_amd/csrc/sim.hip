// Batched QAOA state-vector simulation for gfx950 (CDNA4, wave64).
//
// What is computed (paper Sec. 2.2 and 3.3): for every subgraph b of the
// partition, |psi_b> = U_M(beta_p) U_C(gamma_p) ... U_M(beta_1) U_C(gamma_1)
// |+>^n with U_C = e^{-i gamma H_C}, H_C = diag(C_b(z)) the subgraph's cut
// function, and U_M = prod_j (cos beta I - i sin beta X_j); then
// <C>_b = sum_z |psi_b(z)|^2 C_b(z) and, for the angle optimiser, the exact
// gradient by the adjoint sweep.
//
// How (MI355X design): the state is invariant under flipping every bit
// (C(~z) = C(z); X on every qubit commutes with both operators and fixes
// |+>), so only the 2^(n-1) amplitudes with the top bit clear are stored,
// scaled by sqrt(2); on them the top qubit's X maps an index to its
// complement. The stored state is processed in tiles of 2^12 amplitudes.
// Qubits are split into groups: group 0 = qubits 0..10 plus the top qubit (a
// tile is a block of 2048 contiguous amplitudes and its mirror block, tile
// bit 11 choosing between them), groups 1.. = up to 8 of the qubits 11..n-2
// each (a tile is 2^(12-nb) contiguous amplitudes times 2^nb strided rows). A workgroup keeps its tile in registers (16
// amplitudes per lane) and applies the rotations of 4 register-resident
// qubits at a time; between rounds the tile changes register layout through
// LDS. Consecutive layers visit the groups in alternating (serpentine) order,
// so the last group of layer l and the first group of layer l+1 share one
// HBM pass, with the diagonal phase of layer l+1 applied in registers from
// a precomputed integer cut table C(z) (1 byte per entry when the weight sum
// is at most 255, else 2) and an FP64-built phase table e^{-i gamma c}
// rounded to complex64. <C> and the gradient inner products are accumulated
// in FP64 per tile and reduced per subgraph in a fixed order, so every result
// is bit-reproducible.
//
// Rotation arithmetic: e^{-i beta X} = f (I - i t X) X^flip with (f, t, flip)
// = (cos beta, tan beta, 0) when |cos| >= |sin|, else (-i sin beta,
// -cot beta, 1), so |t| <= 1. The bracketed operator costs two FMAs per real
// component; the per-qubit factor f of a whole group is applied once per
// segment, folded into the next phase multiply when there is one; the X^flip
// permutation is never executed but carried as an XOR mask on tile positions
// into cut-table reads and store addresses. Gradient inner products taken on
// scaled states are rescaled by the known |f|^2 powers.
#include "passes.h"

namespace pq {

// ---------------------------------------------------------------------------
// K1: integer cut tables (natural order + tile order of the last group)
// ---------------------------------------------------------------------------
// With spins s = +-1, C = (sum of weights - sum over edges w s_u s_v) / 2, and
// a wave's 1024 entries vary ten spins only: six by lane, four by the entry
// within a lane's sixteen. So the rest enters through its fields f_i = sum_j
// w_ij s_j on the ten, which the wave's halves find for both tables at once (lane
// = vertex), and through one sum; a word of a lane's entries is then an addition or
// two. Whole numbers throughout. Bound by the vector units: 37 states of 9..13
// qubits take 7.7 us, the subgraphs of 14..26 vertices of a sparse graph of 2000
// 331 us, 30 qubits with 45 edges 381 us (1.07 GB, 2.8 TB/s). One pass over the
// edges for each entry took 22, 745 and 6089 us.
//
// Whole-state subgraphs: natural order; tiled ones: group 0's mirror-paired tile
// order in tab, the last group's tile order in tabB.
//
// A workgroup takes several consecutive tiles where that leaves CUT_BLOCKS of
// them, since the matrix of weights and what a lane keeps of it serve every tile
// of a subgraph.
constexpr int CUT_N = 32;  // rows of the matrix of weights (n <= 30)
constexpr int CUT_BLOCKS = 2048;
constexpr int CUT_MAX_PER = 16;

struct CutWave {
    uint32_t vary;  // the ten vertices
    int at[4];      // vertex of entry bit k
    int by[6];      // the vertices varied by lane, ascending
    int w[4][4];    // weights among at[]
    uint32_t zl;    // this lane's vertices, no other bit set
    int P;          // sum over edges within the lane's six of w s s
    int H[4];       // fields of the lane's six and the other three on the entry's four
};

__device__ inline int spin_of(uint32_t z, int k) { return 1 - 2 * (int)((z >> k) & 1u); }

// e[k]: the vertex (as a bit) of entry bit k; lanem: those varied by lane
__device__ inline CutWave cut_wave(const uint32_t (&e)[4], uint32_t lanem, uint32_t zl, const int32_t (*Wm)[CUT_N])
{
    CutWave c;
    c.vary = e[0] | e[1] | e[2] | e[3] | lanem;
    c.zl = zl;
    uint32_t m = lanem;
#pragma unroll
    for (int k = 0; k < 6; ++k, m &= m - 1) c.by[k] = __ffs(m) - 1;
#pragma unroll
    for (int k = 0; k < 4; ++k) c.at[k] = __ffs(e[k]) - 1;
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j) c.w[k][j] = __builtin_amdgcn_readfirstlane(Wm[c.at[k]][c.at[j]]);
    c.P = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) c.H[k] = c.w[k][0] + c.w[k][1] + c.w[k][2] + c.w[k][3];  // (w[k][k] = 0)
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        const int si = spin_of(zl, c.by[i]);
#pragma unroll
        for (int k = 0; k < 4; ++k) c.H[k] += si * Wm[c.by[i]][c.at[k]];
#pragma unroll
        for (int j = 0; j < i; ++j) c.P += si * spin_of(zl, c.by[j]) * Wm[c.by[i]][c.by[j]];
    }
    return c;
}

// The lane's sixteen entries, from entry `at` on, `count` of them in the table.
// z: the wave's fixed bits (the ten vertices all clear, or, in a mirrored block,
// all set); f: its fields (in the lanes from `half` on); S: the sum over the edges
// among the fixed vertices. With all four entry spins +1 the cut value is c0;
// flipping spin k adds d[k], and flipping k and j takes 2 w[k][j] off again. That
// is linear in the terms, so whole words of entries are formed at once: a word is
// the sum of its entries, each times its place value, whatever its parts.
__device__ inline void store_cuts(const CutWave& c, uint32_t z, int f, int half, int S, int total, uint8_t* tab,
                                  uint32_t at, uint32_t count, bool w1)
{
    const int sg = spin_of(z, c.at[0]);
    int lin = 0;
#pragma unroll
    for (int k = 0; k < 6; ++k) lin += spin_of(c.zl, c.by[k]) * __builtin_amdgcn_readlane(f, half + c.by[k]);
    int d[4], sum = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        d[k] = sg * __builtin_amdgcn_readlane(f, half + c.at[k]) + c.H[k];
        sum += d[k];
    }
    // (the sum of the d counts the weights among the four twice)
    const int among = c.w[0][1] + c.w[0][2] + c.w[0][3] + c.w[1][2] + c.w[1][3] + c.w[2][3];
    const int c0 = (total - S - c.P - sg * lin - sum + among) >> 1;
    if (count < 16) {
#pragma unroll
        for (int l = 0; l < 16; ++l) {
            int v = c0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (!((l >> k) & 1)) continue;
                v += d[k];
#pragma unroll
                for (int j = 0; j < k; ++j) v -= (l >> j) & 1 ? 2 * c.w[k][j] : 0;
            }
            if (l < (int)count) {
                if (w1) tab[at + l] = (uint8_t)v;
                else ((uint16_t*)tab)[at + l] = (uint16_t)v;
            }
        }
        return;
    }
    if (w1) {  // four entries to a word: entry bits 0 and 1
        constexpr uint32_t ALL = 0x01010101u, B0 = 0x01000100u, B1 = 0x01010000u, B01 = 0x01000000u;
        const uint32_t d2 = d[2] * ALL - 2 * c.w[0][2] * B0 - 2 * c.w[1][2] * B1;
        const uint32_t d3 = d[3] * ALL - 2 * c.w[0][3] * B0 - 2 * c.w[1][3] * B1;
        const uint32_t a = c0 * ALL + d[0] * B0 + d[1] * B1 - 2 * c.w[0][1] * B01;
        *(uint4*)(tab + at) = make_uint4(a, a + d2, a + d3, a + d2 + d3 - 2 * c.w[2][3] * ALL);
    } else {  // two entries to a word: entry bit 0
        constexpr uint32_t ALL = 0x00010001u, B0 = 0x00010000u;
        const uint32_t d1 = d[1] * ALL - 2 * c.w[0][1] * B0;
        const uint32_t d2 = d[2] * ALL - 2 * c.w[0][2] * B0;
        const uint32_t d3 = d[3] * ALL - 2 * c.w[0][3] * B0;
        const uint32_t w12 = 2 * c.w[1][2] * ALL, w13 = 2 * c.w[1][3] * ALL, w23 = 2 * c.w[2][3] * ALL;
        const uint32_t a = c0 * ALL + d[0] * B0, b = a + d3;
        uint4* o = (uint4*)(tab + 2 * (size_t)at);
        o[0] = make_uint4(a, a + d1, a + d2, a + d1 + d2 - w12);
        o[1] = make_uint4(b, b + d1 - w13, b + d2 - w23, b + d1 + d2 - w12 - w13 - w23);
    }
}

__global__ __launch_bounds__(THREADS) void k_cut_tables(uint8_t* ws, const SubDesc* subs, const int2* work, int nwork,
                                                       int per)
{
    __shared__ int32_t Wm[CUT_N][CUT_N];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int x0 = blockIdx.x * per, x1 = x0 + per < nwork ? x0 + per : nwork;
    uint32_t row[CUT_N];  // weights of vertex lane % 32 to those that its half's table holds fixed
    int fixed = 0;        // their sum
    CutWave A{}, B{};
    int sub = -1;
    for (int x = x0; x < x1; ++x) {
        const int2 wk = work[x];
        const SubDesc* sd = subs + wk.x;
        const uint32_t t = (uint32_t)wk.y;
        const int n = sd->n, G = sd->ngroups;
        const uint32_t dim = 1u << (n - 1);
        // wide tiles: these entries are a quarter of tile t / 4, in the order
        // (lane, register) of their layout LL1
        const bool wide = sd->wide != 0;
        const int TB = wide ? WIDE_BITS : TILE_BITS;
        const uint32_t tw = wide ? t >> (WIDE_BITS - TILE_BITS) : t;
        const uint32_t first = wide ? (t << TILE_BITS) & ((uint32_t)WIDE_TILE - 1u) : 0u;
        const Geo geoA = make_geo(sd, 0, tw, TB);
        const Geo geoB = make_geo(sd, G >= 2 ? G - 1 : 0, tw, TB);
        // entry -> index bits, both XOR-linear
        auto to_q = [&](uint32_t e) { return wide ? wide_entry(e) : e; };
        auto to_a = [&](uint32_t q) {
            return G < 2 ? q : wide ? gmap0<WIDE_BITS>(geoA, q) : gmap0<TILE_BITS>(geoA, q);
        };
        auto to_b = [&](uint32_t q) { return gmap(geoB, q); };
        if (wk.x != sub) {
            sub = wk.x;
            const int ne = sd->nedges;
            const int32_t* E = (const int32_t*)(ws + sd->edges);
            __syncthreads();  // the previous subgraph's readers are done
            for (int y = tid; y < CUT_N * CUT_N; y += THREADS) (&Wm[0][0])[y] = 0;
            __syncthreads();
            for (int e = tid; e < ne; e += THREADS) {
                const int32_t u = E[3 * e], v = E[3 * e + 1], w = E[3 * e + 2];
                atomicAdd(&Wm[u][v], w);
                atomicAdd(&Wm[v][u], w);
            }
            __syncthreads();
            const uint32_t q[4] = {to_q(1), to_q(2), to_q(4), to_q(8)}, ql = to_q(16u * lane);
            const uint32_t qm = to_q(16) | to_q(32) | to_q(64) | to_q(128) | to_q(256) | to_q(512);
            const uint32_t a[4] = {to_a(q[0]), to_a(q[1]), to_a(q[2]), to_a(q[3])};
            const uint32_t b[4] = {to_b(q[0]), to_b(q[1]), to_b(q[2]), to_b(q[3])};
            A = cut_wave(a, to_a(qm), to_a(ql), Wm);
            if (G >= 2) B = cut_wave(b, to_b(qm), to_b(ql), Wm);
            const uint32_t vary = lane < 32 ? A.vary : B.vary;
            fixed = 0;
#pragma unroll
            for (int j = 0; j < CUT_N; ++j) {
                row[j] = (vary >> j) & 1u ? 0u : (uint32_t)Wm[j][lane & 31];
                fixed += row[j];
            }
        }
        const uint32_t qw = to_q(first + 1024u * wave);
        const uint32_t zA = (G >= 2 ? geoA.zb : 0u) ^ to_a(qw), zB = geoB.zb | to_b(qw);
        // fields of the fixed vertices: lanes 0..31 of table A's, 32..63 of table B's
        const uint32_t z = lane < 32 ? zA : zB;
        uint32_t down = 0;  // weights to those with spin -1
#pragma unroll
        for (int j = 0; j < CUT_N; ++j) down = __umul24((z >> j) & 1u, row[j]) + down;
        const int f = fixed - 2 * (int)down, i = lane & 31;
        int S = ((lane < 32 ? A.vary : B.vary) >> i) & 1u ? 0 : f * spin_of(z, i);
#pragma unroll
        for (int o = 1; o < 32; o <<= 1) S += __shfl_xor(S, o, 64);
        const int total = sd->lut_len - 1;
        const bool w1 = sd->tabw == 1;
        const uint32_t e0 = 1024u * wave + 16u * lane, at = t * (uint32_t)TILE + e0;
        const uint32_t count = at < dim ? dim - at : 0u;
        store_cuts(A, zA, f, 0, __builtin_amdgcn_readlane(S, 0) >> 1, total, ws + sd->tab, at, count, w1);
        if (G >= 2)
            store_cuts(B, zB, f, 32, __builtin_amdgcn_readlane(S, 32) >> 1, total, ws + sd->tabB, at, count, w1);
    }
}

template <int CH, bool FULL, int KIND>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(PQ_FWD_WAVES))) void k_fwd_pass(
    uint8_t* ws, const SubDesc* subs, const int2* work, PassOps ops, Partials part)
{
    fwd_pass_body<CH, FULL, KIND, PREC_VALU>(ws, subs, work, ops, part);
}

// group 0 with the mixer block on the matrix cores (more registers per lane)
template <int KIND, int PREC>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(PQ_MF_WAVES))) void k_fwd_pass_mf(
    uint8_t* ws, const SubDesc* subs, const int2* work, PassOps ops, Partials part)
{
    fwd_pass_body<3, true, KIND, PREC>(ws, subs, work, ops, part);
}

// The fused kind on group 0 is held to four waves per SIMD (the most that
// its LDS tile allows); left free, it takes 130 registers and runs three.
template <int CH, bool FULL, int KIND, bool STORE_PSI>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu((KIND == B_FUSED || KIND == B_LAST) && CH == 3 ? 4 : PQ_BWD_WAVES))) void k_bwd_pass(
    uint8_t* ws, const SubDesc* subs, const int2* work, PassOps ops, Partials part)
{
    bwd_pass_body<CH, FULL, KIND, STORE_PSI>(ws, subs, work, ops, part);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
hipError_t launch_cut_tables(uint8_t* ws, const SubDesc* subs, const int2* work, int nwork, hipStream_t s)
{
    if (nwork <= 0) return hipSuccess;
    int per = nwork / CUT_BLOCKS;
    per = per < 1 ? 1 : per > CUT_MAX_PER ? CUT_MAX_PER : per;
    hipLaunchKernelGGL(k_cut_tables, dim3((nwork + per - 1) / per), dim3(THREADS), 0, s, ws, subs, work, nwork, per);
    return hipGetLastError();
}

// chain codes: 3 = group 0; 2 / 4 = a high group of 8 / 5..7 qubits;
// 1 / 5 = a high group of 4 / 1..3 qubits (the second of each pair has
// register bits that are not active qubits); 6 = high groups of all sizes (mixed.hip)
#define PQ_LAUNCH_CH(KERNEL, ...)                                                                                   \
    do {                                                                                                            \
        switch (chain) {                                                                                            \
        case 3: hipLaunchKernelGGL((KERNEL<3, true, __VA_ARGS__>), g, b, lds, s, ws, subs, work, ops, part); break; \
        case 2: hipLaunchKernelGGL((KERNEL<2, true, __VA_ARGS__>), g, b, lds, s, ws, subs, work, ops, part); break; \
        case 4: hipLaunchKernelGGL((KERNEL<2, false, __VA_ARGS__>), g, b, lds, s, ws, subs, work, ops, part); break;\
        case 1: hipLaunchKernelGGL((KERNEL<1, true, __VA_ARGS__>), g, b, lds, s, ws, subs, work, ops, part); break; \
        case 5: hipLaunchKernelGGL((KERNEL<1, false, __VA_ARGS__>), g, b, lds, s, ws, subs, work, ops, part); break;\
        default: return hipErrorInvalidValue;                                                                       \
        }                                                                                                           \
    } while (0)

// group 0 with a matrix-core mixer block (PREC 1 or 2)
#define PQ_LAUNCH_MF(KIND)                                                                                      \
    do {                                                                                                        \
        if (prec == PREC_MFMA_F32)                                                                              \
            hipLaunchKernelGGL((k_fwd_pass_mf<KIND, PREC_MFMA_F32>), g, b, lds, s, ws, subs, work, ops, part);  \
        else if (prec == PREC_MFMA_BF16X3)                                                                      \
            hipLaunchKernelGGL((k_fwd_pass_mf<KIND, PREC_MFMA_BF16X3>), g, b, lds, s, ws, subs, work, ops,      \
                               part);                                                                           \
        else                                                                                                    \
            hipLaunchKernelGGL((k_fwd_pass_mf<KIND, PREC_MFMA_BF16X4>), g, b, lds, s, ws, subs, work, ops,      \
                               part);                                                                           \
    } while (0)

hipError_t launch_fwd_pass(uint8_t* ws, const SubDesc* subs, const int2* work, int nwork, int chain, PassOps ops,
                           Partials part, int lut_max, int prec, hipStream_t s)
{
    if (nwork <= 0) return hipSuccess;
    const size_t lds = pass_lds(lut_max);
    const dim3 g(nwork), b(THREADS);
    // the first pass is group 0's
    if (ops.init && (ops.group != 0 || chain != 3)) return hipErrorInvalidValue;
    if (chain == 6) return launch_fwd_mixed(ws, subs, work, nwork, ops, part, lut_max, s);
    if (prec != PREC_VALU && chain == 3) {
        if (ops.init) PQ_LAUNCH_MF(F_FIRST);
        else if (ops.epi_e) PQ_LAUNCH_MF(F_LAST);
        else if (ops.ph >= 0) PQ_LAUNCH_MF(F_MID);
        else PQ_LAUNCH_MF(F_SINGLE);
        return hipGetLastError();
    }
    if (ops.init) hipLaunchKernelGGL((k_fwd_pass<3, true, F_FIRST>), g, b, lds, s, ws, subs, work, ops, part);
    else if (ops.epi_e) PQ_LAUNCH_CH(k_fwd_pass, F_LAST);
    else if (ops.ph >= 0) PQ_LAUNCH_CH(k_fwd_pass, F_MID);
    else PQ_LAUNCH_CH(k_fwd_pass, F_SINGLE);
    return hipGetLastError();
}

hipError_t launch_bwd_pass(uint8_t* ws, const SubDesc* subs, const int2* work, int nwork, int chain, PassOps ops,
                           Partials part, int lut_max, hipStream_t s)
{
    if (nwork <= 0) return hipSuccess;
    const size_t lds = pass_lds(lut_max);
    const dim3 g(nwork), b(THREADS);
    // the last pass mirrors the first forward pass (group 0 of layer 1)
    if (ops.last && (ops.group != 0 || chain != 3)) return hipErrorInvalidValue;
    if (chain == 6) return launch_bwd_mixed(ws, subs, work, nwork, ops, part, lut_max, s);
    if (ops.fused) PQ_LAUNCH_CH(k_bwd_pass, B_FUSED, true);
    else if (ops.last) hipLaunchKernelGGL((k_bwd_pass<3, true, B_LAST, true>), g, b, lds, s, ws, subs, work, ops, part);
    else if (ops.ph >= 0 && ops.nopsi) PQ_LAUNCH_CH(k_bwd_pass, B_MID, false);
    else if (ops.ph >= 0) PQ_LAUNCH_CH(k_bwd_pass, B_MID, true);
    else if (ops.nopsi) PQ_LAUNCH_CH(k_bwd_pass, B_SINGLE, false);
    else PQ_LAUNCH_CH(k_bwd_pass, B_SINGLE, true);
    return hipGetLastError();
}

}  // namespace pq

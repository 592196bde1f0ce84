// Merge of the per-subgraph candidate sets (paper Sec. 3.4, Alg. 2) as a
// level-wise beam on the GPU.
//
// Level i holds the chain subgraph V_i = [start_i, start_i + size_i); V_i
// shares its first vertex with V_{i-1}. Candidate set B_i = {b_j, ~b_j}; a
// path takes one member of B_1, then at every later level the member of each
// pair whose bit for the shared vertex agrees with the path (so a path has
// 2K choices at level 1 and K at each later level: 2 K^M leaves). Path order
// is the depth-first order of Alg. 2 (digits 2j+o at level 1, j later).
//
// Score of a partial path = cut of the edges whose endpoints are both
// assigned. By the cut decomposition of Sec. 3.4.1 a child's score is its
// parent's plus C_i(b_j) (the intra-subgraph cut, orientation free) plus the
// back edges (u assigned earlier, v new in V_i): sum_k (y_k ? W_k - A_k : A_k)
// with y_k the child's bit for local vertex k, W_k the back-edge weight into
// k and A_k the weight of those back edges whose earlier endpoint is 1 in the
// parent. After each level the W best paths by (score desc, path order asc)
// survive; with W >= 2 K^(M-1) this is the exhaustive merge.
//
// Keys: 32-bit, score + 1 (zero marks an invalid candidate); a key's index
// in the level's key array is its path order, parent_rank * K + j (level 1:
// 2j + o). Survivors are kept in path order, so a survivor's rank is its
// position.
//
// Level 1 (2K keys) runs in one workgroup (k_merge_select + k_merge_build).
// Every later level runs in three launches over all surviving parents:
//   expand  - the children's keys, and a histogram of (H - key): 65536 fine
//             bins of one key value, 4096 coarse bins of 16 and 256 super bins
//             of 256, H an upper
//             bound of the level's keys (previous best key + the level's
//             largest possible increment); each block aggregates its keys in
//             LDS and adds only its nonzero bins to the global histogram;
//   count   - every block finds the threshold key k* (keys above it survive,
//             plus the first R keys equal to it in path order) from the
//             super bins, 16 coarse and 16 fine bins, then counts its parents'
//             survivors; if the W-th key lies below the histogram's window
//             (scores spread over more than 65536 values) each block
//             computes k* from the keys themselves instead;
//   scatter - the prefix of the per-parent counts gives each survivor its
//             position; the survivors' rows are built; the histogram's super
//             bins that hold something are cleared for the next level.
#include "lane.h"

namespace pq {

__device__ inline uint32_t row_bit(const uint32_t* row, int v) { return (row[v >> 5] >> (v & 31)) & 1u; }

constexpr int FINE_BINS = 65536;
constexpr int COARSE_SHIFT = 4;
constexpr int COARSE_BINS = FINE_BINS >> COARSE_SHIFT;  // 4096
constexpr int SUPER_SHIFT = 8;
constexpr int SUPER_BINS = FINE_BINS >> SUPER_SHIFT;    // 256
constexpr int SUPER_AT = FINE_BINS + COARSE_BINS;
static_assert(SUPER_AT + SUPER_BINS == MERGE_HIST_INTS, "histogram layout");
constexpr int MX_THREADS = 256;  // expand / count / scatter blocks
constexpr int LOCAL_BINS = 1024;
constexpr int INTRA_THREADS = 256;

// C_i(b_j) for every level and candidate; the number of valid candidates
// (those before the first 0xFFFFFFFF of the row); the level's largest
// possible score increment (max_j C_i(b_j) + its total back-edge weight); the
// histogram cleared for level 2. One workgroup per level (K <= 64).
__global__ __launch_bounds__(INTRA_THREADS) void k_merge_intra(int M, const MergeLevel* lv, const int32_t* intra,
                                                              const uint32_t* cand, int K, int lgKp, int64_t* ccut,
                                                              int32_t* lvk, uint32_t* maxinc, int32_t* hist,
                                                              int32_t* below)
{
    __shared__ uint64_t s_cut[64];
    const int i = blockIdx.x, t = threadIdx.x;
    for (int x = blockIdx.x * INTRA_THREADS + t; x < MERGE_COPIES * MERGE_HIST_INTS / 4; x += gridDim.x * INTRA_THREADS)
        ((int4*)hist)[x] = make_int4(0, 0, 0, 0);
    if (i == 0 && t == 0) *below = 0;
    if (i >= M) return;  // (these blocks only clear)
    const MergeLevel& L = lv[i];
    // thread t takes every parts-th edge for candidate t % Kp
    const int j = t & ((1 << lgKp) - 1), parts = INTRA_THREADS >> lgKp;
    const uint32_t b = j < K ? cand[(size_t)i * K + j] : 0xFFFFFFFFu;
    if (t < 64) s_cut[t] = 0;
    __syncthreads();
    int64_t c = 0;
    const int32_t* E = intra + 3 * (size_t)L.intra_off;
#pragma unroll 4
    for (int e = t >> lgKp; e < L.intra_cnt; e += parts)
        c += ((b >> E[3 * e]) ^ (b >> E[3 * e + 1])) & 1u ? E[3 * e + 2] : 0;
    if (b != 0xFFFFFFFFu && c) atomicAdd((unsigned long long*)&s_cut[j], (unsigned long long)c);
    __syncthreads();
    if (t >= 64) return;
    const uint64_t bad = __ballot(t < K && cand[(size_t)i * K + t] == 0xFFFFFFFFu);
    const int32_t wk = t < 32 ? (int32_t)L.wk[t] : 0;  // total weight < 2^31
    int32_t best = (int32_t)s_cut[t], wb = wk;
    if (t < K) ccut[(size_t)i * K + t] = (int64_t)s_cut[t];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const int32_t y = __shfl_xor(best, o, 64);
        best = y > best ? y : best;
        wb += __shfl_xor(wb, o, 64);
    }
    if (t == 0) {
        lvk[i] = bad ? __ffsll((unsigned long long)bad) - 1 : K;
        maxinc[i] = (uint32_t)best + (uint32_t)wb;
    }
}

// level 1: the 2 K_1 paths (j, o) in order b_1, ~b_1, b_2, ~b_2, ...
__global__ void k_merge_first(const int32_t* lvk, int K, const int64_t* ccut, uint32_t* keys, int32_t* npaths)
{
    const int Kv = lvk[0];
    for (int d = threadIdx.x; d < 2 * K; d += blockDim.x) {
        const int j = d >> 1;
        keys[d] = j < Kv ? (uint32_t)(ccut[j] + 1) : 0u;
    }
    if (threadIdx.x == 0) npaths[0] = 1;
}

// ---------------------------------------------------------------------------
// Threshold selection inside one workgroup (level 1, and the fallback of the
// count kernel)
// ---------------------------------------------------------------------------
constexpr int SEL_BINS = 4096;

__device__ inline int32_t wave_sum(int32_t x)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}
// exclusive prefix of the per-wave values slots[0..NW) at wave wv, and their
// total (lanes 0..NW-1 read one slot each)
template <int NW>
__device__ inline void wave_slots_prefix(const int32_t* slots, int wv, int32_t& before, int32_t& total)
{
    const int lane = threadIdx.x & 63;
    const int32_t v = lane < NW ? slots[lane] : 0;
    int32_t incl = v;
#pragma unroll
    for (int o = 1; o < NW; o <<= 1) {
        const int32_t y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
    }
    before = __shfl(incl - v, wv, 64);
    total = __shfl(incl, NW - 1, 64);
}
// the value of x unknown to the optimiser (keeps it from holding values
// derived from x live across the kernel instead of recomputing them)
__device__ inline int32_t opaque(int32_t x)
{
    asm volatile("" : "+v"(x));
    return x;
}
// lanes of the wave that hold the children of this lane's parent (2^lgKp
// consecutive lanes)
__device__ inline uint64_t parent_lanes(int lane, int lgKp)
{
    if (lgKp >= 6) return ~0ull;
    return ((1ull << (1 << lgKp)) - 1ull) << ((lane >> lgKp) << lgKp);
}

template <int THREADS>
struct SelShared {
    int32_t hist[SEL_BINS];
    int32_t wa[THREADS / 64], wb[THREADS / 64];
    uint32_t s_hi, s_lo;
    int32_t s_above;
};

struct SelResult {
    int32_t nvalid;
    uint32_t best;   // largest key (0 if none)
    uint32_t kstar;  // keys > kstar survive (0: every valid key)
    int32_t R;       // and the first R keys == kstar in index order
};

// The Wsel best keys among keys[0..N) by (key desc, index asc), as a
// threshold. The keys are visited in rounds of THREADS * PER, wave w of a
// round holding keys [w * 64 PER, (w + 1) * 64 PER) of it in registers (64
// consecutive keys per register). RESIDENT: N <= THREADS * PER (the caller
// guarantees it), one round, the keys are read from memory once; otherwise
// every step re-reads them round by round. The key buffer is padded to a
// multiple of MERGE_KEY_PAD entries, so every round reads in bounds; entries
// at N and beyond are masked. (1) count, largest and smallest valid key;
// (2) threshold key k* and the number R of keys equal to k* that survive,
// from histograms of (hi - key) >> shift over [lo, hi] with 4096 bins,
// refined to the bin holding the Wsel-th key until shift = 0 (at most three
// histograms for 31-bit keys). On return sc[] holds the last round.
template <int THREADS, int PER, bool RESIDENT>
__device__ SelResult select_threshold(const uint32_t* keys, int32_t N, int Wsel, uint32_t (&sc)[PER],
                                      SelShared<THREADS>& S)
{
    constexpr int NW = THREADS / 64;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    constexpr int32_t RW = THREADS * PER;
    const int rounds = RESIDENT ? 1 : (N + RW - 1) / RW;
    auto load = [&](int r) {
        const int32_t b = opaque(r * RW + wv * 64 * PER + lane);
        const uint32_t* kp = keys + b;
        const int32_t lim = N - b;  // register j holds a key iff 64 j < lim
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const uint32_t v = kp[64 * j];
            sc[j] = 64 * j < lim ? v : 0u;
        }
    };
    // (1)
    int32_t valid = 0;
    uint32_t mx = 0, mn = 0xFFFFFFFFu;  // mn: smallest valid key - 1
    for (int r = 0; r < rounds; ++r) {
        load(r);
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const uint32_t k = sc[j];
            valid += k != 0u;
            mx = k > mx ? k : mx;
            mn = k - 1u < mn ? k - 1u : mn;  // invalid (0) wraps to the maximum
        }
    }
    valid = wave_sum(valid);
    mx = wave_max(mx);
    mn = wave_min(mn);
    __syncthreads();  // S is free (an earlier use has been read)
    if (lane == 0) {
        S.wa[wv] = valid;
        S.wb[wv] = (int32_t)mx;
        S.hist[wv] = (int32_t)mn;
    }
    __syncthreads();
    SelResult res;
    int32_t unused;
    wave_slots_prefix<NW>(S.wa, 0, unused, res.nvalid);
    uint32_t hi = wave_max(lane < NW ? (uint32_t)S.wb[lane] : 0u);
    uint32_t lo = wave_min(lane < NW ? (uint32_t)S.hist[lane] : 0xFFFFFFFFu) + 1u;  // >= 1 if any valid
    res.best = hi;
    res.kstar = 0;
    res.R = 0;
    // (2)
    if (res.nvalid > Wsel) {
        int32_t above = 0;  // keys above the current range [lo, hi]
        for (;;) {
            int shift = 0;
            while (((hi - lo) >> shift) >= (uint32_t)SEL_BINS) ++shift;
            __syncthreads();  // the previous reads of hist / wa are done
            for (int c = tid; c < SEL_BINS; c += THREADS) S.hist[c] = 0;
            __syncthreads();
            for (int r = 0; r < rounds; ++r) {
                if (!RESIDENT) load(r);
#pragma unroll
                for (int j = 0; j < PER; ++j) {
                    const uint32_t k = sc[j];
                    if (k >= lo && k <= hi) atomicAdd(&S.hist[(hi - k) >> shift], 1);  // lo >= 1: valid keys only
                }
            }
            __syncthreads();
            // thread t owns bins t * BPT .. (t + 1) * BPT - 1; block exclusive scan of their sums
            constexpr int BPT = SEL_BINS / THREADS;
            int32_t hb[BPT], part = 0;
#pragma unroll
            for (int c = 0; c < BPT; ++c) {
                hb[c] = S.hist[BPT * tid + c];
                part += hb[c];
            }
            int32_t incl = part;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int32_t y = __shfl_up(incl, o, 64);
                if (lane >= o) incl += y;
            }
            if (lane == 63) S.wa[wv] = incl;
            __syncthreads();
            int32_t wbefore, wtotal;
            wave_slots_prefix<NW>(S.wa, wv, wbefore, wtotal);
            int32_t run = above + wbefore + incl - part;
#pragma unroll
            for (int c = 0; c < BPT; ++c) {
                if (run < Wsel && run + hb[c] >= Wsel) {  // exactly one bin of one thread
                    const uint32_t bin = (uint32_t)(BPT * tid + c);
                    S.s_above = run;
                    S.s_hi = hi - (bin << shift);
                    const uint32_t w = (bin << shift) + ((1u << shift) - 1u);  // hi - (the bin's lowest key)
                    S.s_lo = (hi - lo > w) ? hi - w : lo;
                }
                run += hb[c];
            }
            __syncthreads();
            above = S.s_above;
            hi = S.s_hi;
            lo = S.s_lo;
            if (shift == 0) {  // the bin is the single key value k*
                res.kstar = hi;
                res.R = Wsel - above;
                break;
            }
        }
    }
    return res;
}

// Level 1: keep the Wsel best of the 2K keys and write them as survivors in
// index order (one workgroup); st receives the level's threshold and best key.
constexpr int SEL_THREADS = 1024;
constexpr int SEL_PER = 16;
static_assert(SEL_THREADS * SEL_PER <= MERGE_KEY_PAD, "key buffer padding covers one round");

__global__ __launch_bounds__(SEL_THREADS) void k_merge_select(const uint32_t* keys, const int32_t* npaths, int Kmul,
                                                              int Wsel, Surv* surv, int32_t* nsurv,
                                                              MergeLvState* st)
{
    __shared__ SelShared<SEL_THREADS> S;
    constexpr int NW = SEL_THREADS / 64;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int32_t N = *npaths * Kmul;  // <= 2 QAOA_MAX_K
    uint32_t sc[SEL_PER];
    const SelResult res = select_threshold<SEL_THREADS, SEL_PER, true>(keys, N, Wsel, sc, S);
    const uint32_t kstar = res.kstar;
    const int32_t R = res.R;
    // compaction in index order by wave ballots
    int32_t gt = 0, eq = 0;
#pragma unroll
    for (int j = 0; j < SEL_PER; ++j) {
        gt += sc[j] > kstar;
        eq += sc[j] == kstar;  // kstar = 0 only if R = 0, where eq does not matter
    }
    gt = wave_sum(gt);
    eq = wave_sum(eq);
    __syncthreads();
    if (lane == 0) {
        S.wa[wv] = gt;
        S.wb[wv] = eq;
    }
    __syncthreads();
    int32_t gt_before, eq_before, tot;
    wave_slots_prefix<NW>(S.wa, wv, gt_before, tot);
    wave_slots_prefix<NW>(S.wb, wv, eq_before, tot);
    const uint64_t below = (1ull << lane) - 1ull;
    const int32_t b = opaque(wv * 64 * SEL_PER + lane);
#pragma unroll
    for (int j = 0; j < SEL_PER; ++j) {
        const uint32_t k = sc[j];
        const bool g = k > kstar, e = k == kstar;
        const uint64_t bg = __ballot(g), be = __ballot(e);
        const int32_t my_gt = gt_before + __popcll(bg & below), my_eq = eq_before + __popcll(be & below);
        if (g || (e && my_eq < R)) {
            Surv sv;
            sv.parent = 0;
            sv.digit = b + 64 * j;
            sv.score = opaque((int32_t)k) - 1;
            surv[my_gt + (my_eq < R ? my_eq : R)] = sv;
        }
        gt_before += __popcll(bg);
        eq_before += __popcll(be);
    }
    if (tid == 0) {
        const int32_t count = res.nvalid < Wsel ? res.nvalid : Wsel;
        *nsurv = count;
        st->best = res.best;
        st->kstar = kstar;
        st->R = R;
        st->count = count;
    }
}

// place the level's bits [start, start + size) into word q of a row (the
// bits span at most two words)
__device__ inline uint32_t place_bits(uint32_t word, int q, int start, int size, uint32_t bits)
{
    const int w0 = start >> 5, sh = start & 31;
    const uint64_t lm = (size == 32 ? 0xFFFFFFFFull : ((1ull << size) - 1ull)) << sh;
    const uint64_t val = (uint64_t)bits << sh;
    if (q == w0) return (word & ~(uint32_t)lm) | (uint32_t)val;
    if (q == w0 + 1) return (word & ~(uint32_t)(lm >> 32)) | (uint32_t)(val >> 32);
    return word;
}

__device__ inline uint32_t level_bits(uint32_t b, uint32_t o, int size)
{
    return (b ^ (o ? 0xFFFFFFFFu : 0u)) & (size == 32 ? 0xFFFFFFFFu : ((1u << size) - 1u));
}

// rows of level 1's survivors: the level's bits only
__global__ void k_merge_build(const MergeLevel* lv, const uint32_t* cand, const Surv* surv, const int32_t* nsurv,
                              uint32_t* nrow, int nw, int64_t* scores, int final_out, int nV)
{
    const int r = blockIdx.x;
    if (r >= *nsurv) return;
    const MergeLevel& L = lv[0];
    const Surv s = surv[r];
    const int nwp = final_out ? nw : (L.start + L.size + 31) >> 5;
    const uint32_t bits = level_bits(cand[s.digit >> 1], (uint32_t)(s.digit & 1), L.size);
    uint32_t* dst = nrow + (size_t)r * nw;
    for (int q = threadIdx.x; q < nwp; q += blockDim.x) {
        uint32_t w = place_bits(0u, q, L.start, L.size, bits);
        if (final_out && q == nw - 1 && (nV & 31)) w &= (1u << (nV & 31)) - 1u;
        dst[q] = w;
    }
    if (threadIdx.x == 0) scores[r] = s.score;
}

// ---------------------------------------------------------------------------
// Levels 2..M: expand / count / scatter
// ---------------------------------------------------------------------------
// A block covers PPB = MX_THREADS / Kp parents (expand: epb, at most as many), Kp =
// K rounded up to a power of two; thread t is child j = t % Kp of local parent t / Kp (j >= K idle),
// so a parent's children are consecutive lanes of one wave.
//
// A level is a chain of dependent steps, so its time is latency: at 2000
// vertices (104 subgraphs, K 16, W 4096: 256 blocks, 65536 keys a level) the
// three launches take 11.3 + 6.4 + 7.5 us and a whole merge 2.57 ms (before the
// histogram had copies 21 us for expand and 3.4 ms, before the loads were issued
// ahead of their use and the rows staged as one flat range 4.27 ms). Expand was
// bound by the blocks' additions to the same lines of the histogram: with 2
// blocks it took 5 us, with 256 always 19 or more. So where there are many
// blocks, eight copies share them, and count sums the copies, which three
// levels of bins keep short: 256 super bins, one per thread, then 16 coarse and
// 16 fine ones, each by one wave-wide load. The line lies at 64
// blocks (of expand), where both cost the same; a level with one copy / eight, in us
// (1000 vertices, K 16): 32 blocks 27.2 / 29.6, 64 29.4 / 29.7, 128 33.4 / 30.0,
// 256 41.8 / 32.2; K 64: 32 21.8 / 23.6, 128 27.6 / 24.2, 1024 83.5 / 48.9.

constexpr int EDGE_STAGE = 2048;  // back edges staged in LDS per round
constexpr int ROW_STAGE = 4096;   // row words staged in LDS (else read from memory)

__global__ __launch_bounds__(MX_THREADS) void k_merge_expand(const MergeLevel* lv, int i, const int32_t* back,
                                                             const uint32_t* cand, int K, int lgKp, int epb,
                                                             const int64_t* ccut, const int32_t* lvk,
                                                             const uint32_t* rows, int nw, const int64_t* scores,
                                                             const int32_t* npaths, const MergeLvState* lvs,
                                                             const uint32_t* maxinc, uint32_t* keys, int32_t* hist,
                                                             int copies, int32_t* below)
{
    __shared__ int32_t A[MX_THREADS][32];
    __shared__ int32_t lh[LOCAL_BINS];
    __shared__ int32_t se_u[EDGE_STAGE], se_w[EDGE_STAGE];
    __shared__ uint32_t srow[ROW_STAGE];
    __shared__ int32_t s_kbeg[33], s_wk[32];
    __shared__ uint32_t s_dmin;
    const int t = threadIdx.x;
    const int pl = t >> lgKp, j = t & ((1 << lgKp) - 1);
    const int p0 = blockIdx.x * epb;
    // (every uniform value is read before the first is waited for)
    const MergeLevel& L = lv[i];
    const int np = npaths[i], start = L.start, size = L.size, back_off = L.back_off, nb = L.kbeg[32];
    const int valid = lvk[i];
    const uint32_t H = lvs[i - 1].best + maxinc[i];  // >= every key of the level
    if (p0 >= np) return;  // uniform
    const int nact = np - p0 < epb ? np - p0 : epb;
    const int p = p0 + pl;
    const bool mine = pl < nact && j < K;
    // this child's inputs, loaded ahead of the staging (total weights < 2^31)
    const uint32_t b = mine ? cand[(size_t)i * K + j] : 0u;
    const int32_t base_score = mine ? (int32_t)(scores[p] + ccut[(size_t)i * K + j]) : 0;
    const bool act = mine && j < valid;
    // rows of the block's parents up to the word of the shared vertex
    const int wl = (start >> 5) + 1;
    const bool rows_lds = nact * wl <= ROW_STAGE;
    if (rows_lds) {
        // lanes over words, then parents: 2^lw >= wl words
        int lw = 0;
        while ((1 << lw) < wl) ++lw;
        const int per = MX_THREADS >> lw;  // parents at a time (0: more words than threads)
        if (per > 0) {
            const int w = t & ((1 << lw) - 1);
#pragma unroll 4
            for (int q = t >> lw; q < nact; q += per)
                if (w < wl) srow[q * wl + w] = rows[(size_t)(p0 + q) * nw + w];
        } else {
            for (int q = 0; q < nact; ++q)
                for (int w = t; w < wl; w += MX_THREADS) srow[q * wl + w] = rows[(size_t)(p0 + q) * nw + w];
        }
    }
    for (int x = t; x < LOCAL_BINS; x += MX_THREADS) lh[x] = 0;
    for (int x = t; x < nact * 32; x += MX_THREADS) A[x >> 5][x & 31] = 0;
    if (t < 33) s_kbeg[t] = L.kbeg[t];
    if (t >= 64 && t < 96) s_wk[t - 64] = (int32_t)L.wk[t - 64];
    if (t == 0) s_dmin = 0xFFFFFFFFu;
    auto bit_of = [&](int q, int v) -> uint32_t {
        return rows_lds ? (srow[q * wl + (v >> 5)] >> (v & 31)) & 1u : row_bit(rows + (size_t)(p0 + q) * nw, v);
    };
    // back-edge weights A_k of every parent: the thread that owns (q, k) sums
    // the edges into local vertex k (sorted by k) whose earlier endpoint is 1
    // in parent q
    for (int e0 = 0; e0 < nb || e0 == 0; e0 += EDGE_STAGE) {
        const int ne = nb - e0 < EDGE_STAGE ? nb - e0 : EDGE_STAGE;
        if (e0) __syncthreads();  // the previous round's readers are done
#pragma unroll 4
        for (int x = t; x < ne; x += MX_THREADS) {
            const int32_t* E = back + 3 * (size_t)(back_off + e0 + x);
            se_u[x] = E[0];
            se_w[x] = E[2];
        }
        __syncthreads();
        for (int x = t; x < nact * 32; x += MX_THREADS) {
            const int q = x >> 5, k = x & 31;
            const int lo = (s_kbeg[k] > e0 ? s_kbeg[k] : e0) - e0;
            const int hi = (s_kbeg[k + 1] < e0 + ne ? s_kbeg[k + 1] : e0 + ne) - e0;
            int32_t sum = 0;
            int e = lo;
            for (; e + 8 <= hi; e += 8) {  // eight independent LDS chains in flight
                int32_t u[8], w[8];
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    u[c] = se_u[e + c];
                    w[c] = se_w[e + c];
                }
#pragma unroll
                for (int c = 0; c < 8; ++c) sum += bit_of(q, u[c]) ? w[c] : 0;
            }
            for (; e < hi; e += 4) {  // the rest by fours, the last edge again with weight 0
                int32_t u[4], w[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int x = e + c < hi ? e + c : hi - 1;
                    u[c] = se_u[x];
                    w[c] = e + c < hi ? se_w[x] : 0;
                }
#pragma unroll
                for (int c = 0; c < 4; ++c) sum += bit_of(q, u[c]) ? w[c] : 0;
            }
            A[q][k] += sum;  // (q, k) has one owner
        }
        if (nb == 0) break;
    }
    __syncthreads();
    uint32_t key = 0;
    if (act) {
        const uint32_t y = b ^ (((b & 1u) ^ bit_of(pl, start)) ? 0xFFFFFFFFu : 0u);
        int32_t s = base_score;
        // (vertices beyond the level's size have no back edges: A and W are 0)
#pragma unroll 8
        for (int k = 1; k < size; ++k) s += (y >> k) & 1u ? s_wk[k] - A[pl][k] : A[pl][k];
        key = (uint32_t)(s + 1);
    }
    if (mine) keys[(size_t)p * K + j] = key;
    // histogram of d = H - key
    const uint32_t d = H - key;
    const bool inwin = key != 0u && d < (uint32_t)FINE_BINS;
    const int32_t nbelow = __popcll(__ballot(key != 0u && !inwin));
    if ((t & 63) == 0 && nbelow) atomicAdd(below, nbelow);
    const uint32_t wmin = wave_min(inwin ? d : 0xFFFFFFFFu);
    if ((t & 63) == 0 && wmin != 0xFFFFFFFFu) atomicMin(&s_dmin, wmin);
    __syncthreads();
    const uint32_t dmin = s_dmin;
    if (dmin == 0xFFFFFFFFu) return;  // no key of the block in the window (uniform)
    hist += (size_t)(blockIdx.x & (uint32_t)(copies - 1)) * MERGE_HIST_INTS;
    const uint32_t base = dmin & ~(uint32_t)((1 << SUPER_SHIFT) - 1);  // local bins align with super bins
    if (inwin) {
        const uint32_t lb = d - base;
        if (lb < (uint32_t)LOCAL_BINS) {
            atomicAdd(&lh[lb], 1);
        } else {  // the block's keys spread wider than the local window
            atomicAdd(&hist[d], 1);
            atomicAdd(&hist[FINE_BINS + (d >> COARSE_SHIFT)], 1);
            atomicAdd(&hist[SUPER_AT + (d >> SUPER_SHIFT)], 1);
        }
    }
    __syncthreads();
    // flush: thread t owns local bins 4t .. 4t + 3; four threads make one coarse
    // bin, a wave one super bin
    int32_t c4 = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int32_t n = lh[4 * t + c];
        if (n) atomicAdd(&hist[base + 4 * t + c], n);
        c4 += n;
    }
    c4 += __shfl_xor(c4, 1, 64);
    c4 += __shfl_xor(c4, 2, 64);
    if ((t & 3) == 0 && c4) atomicAdd(&hist[FINE_BINS + (base >> COARSE_SHIFT) + (t >> 2)], c4);
#pragma unroll
    for (int o = 4; o < 64; o <<= 1) c4 += __shfl_xor(c4, o, 64);
    if ((t & 63) == 0 && c4) atomicAdd(&hist[SUPER_AT + (base >> SUPER_SHIFT) + (t >> 6)], c4);
}

// bin x + lane % 16 summed over the copies, in every lane of a wave
__device__ inline int32_t copies_sum(const int32_t* hist, int x, int copies)
{
    const int lane = threadIdx.x & 63;
    int32_t n = 0;
    for (int c = lane >> 4; c < copies; c += 4) n += hist[(size_t)c * MERGE_HIST_INTS + x + (lane & 15)];
    n += __shfl_xor(n, 16, 64);
    return n + __shfl_xor(n, 32, 64);
}

// Of 16 bins (one per lane, repeated four times): the first nonzero one, and the
// one in which the running count, started at `above`, reaches `need` (above
// becomes the count before it).
__device__ inline int first_bin(int32_t n) { return __ffsll((unsigned long long)__ballot(n != 0)) - 1; }
__device__ inline int crossing_bin(int32_t n, int32_t need, int32_t& above)
{
    const int c = threadIdx.x & 15;
    int32_t upto = n;
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
        const int32_t y = __shfl_up(upto, o, 16);
        if (c >= o) upto += y;
    }
    const int at = __ffsll((unsigned long long)__ballot(above + upto >= need)) - 1;
    above += __shfl(upto - n, at, 64);
    return at;
}

// Threshold of the level from the histogram (every block identically), then
// each parent's number of children above and at the threshold (gt in the
// low, eq in the high 32 bits of pcnt[parent]).
__global__ __launch_bounds__(MX_THREADS) void k_merge_count(int i, int K, int lgKp, const int32_t* npaths_in,
                                                            int Wsel, const MergeLvState* lvs_prev,
                                                            const uint32_t* maxinc, const uint32_t* keys,
                                                            const int32_t* hist, int copies, const int32_t* below,
                                                            int64_t* pcnt, MergeLvState* st, int32_t* npaths_out)
{
    __shared__ SelShared<MX_THREADS> S;
    __shared__ int32_t s_first, s_cross;
    constexpr int NW = MX_THREADS / 64;
    static_assert(SUPER_BINS == MX_THREADS, "one super bin per thread");
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    // this parent's keys and every uniform value are read before the first is waited for
    const int PPB = MX_THREADS >> lgKp;
    const int pl = t >> lgKp, j = t & ((1 << lgKp) - 1);
    const int p = blockIdx.x * PPB + pl;
    const int np = *npaths_in, nbelow = *below;
    const uint32_t key = (p < np && j < K) ? keys[(size_t)p * K + j] : 0u;
    const int32_t N = np * K;
    const uint32_t H = lvs_prev->best + maxinc[i];
    int32_t part = 0;
    for (int c = 0; c < copies; ++c) part += hist[(size_t)c * MERGE_HIST_INTS + SUPER_AT + t];
    int32_t incl = part;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
    }
    if (lane == 63) S.wa[wv] = incl;
    if (t == 0) {
        s_first = SUPER_BINS;
        s_cross = -1;
    }
    __syncthreads();
    int32_t wbefore, inwin;
    wave_slots_prefix<NW>(S.wa, wv, wbefore, inwin);
    const int32_t nvalid = inwin + nbelow;
    const int32_t need = nvalid < Wsel ? nvalid : Wsel;  // survivors
    const int32_t run = wbefore + incl - part;
    if (run < need && run + part >= need) {  // exactly one thread, if any
        S.s_above = run;
        s_cross = t;
    }
    const uint64_t some = __ballot(part != 0);
    if (lane == 0 && some) atomicMin(&s_first, (wv << 6) + __ffsll((unsigned long long)some) - 1);
    __syncthreads();
    SelResult res;
    res.nvalid = nvalid;
    res.best = 0;
    res.kstar = 0;
    res.R = 0;
    if (need > 0 && s_cross >= 0) {
        // the best key: first super, coarse and fine bin; the threshold: the
        // crossing ones (every wave computes the same)
        const int32_t* coarse = hist + FINE_BINS;
        int32_t above = S.s_above;
        const int32_t f1 = copies_sum(coarse, s_first << 4, copies), x1 = copies_sum(coarse, s_cross << 4, copies);
        const int fb = ((s_first << 4) + first_bin(f1)) << COARSE_SHIFT;
        const int xb = ((s_cross << 4) + crossing_bin(x1, need, above)) << COARSE_SHIFT;
        const int32_t f2 = copies_sum(hist, fb, copies), x2 = copies_sum(hist, xb, copies);
        res.best = H - (uint32_t)(fb + first_bin(f2));
        const int at = crossing_bin(x2, need, above);
        if (nvalid > Wsel) {
            res.kstar = H - (uint32_t)(xb + at);
            res.R = Wsel - above;
        }
    } else if (need > 0) {
        // the Wsel-th key (or the best one) lies below the window: select from the keys
        uint32_t sc[4];
        res = select_threshold<MX_THREADS, 4, false>(keys, N, Wsel, sc, S);
    }
    if (blockIdx.x == 0 && t == 0) {
        st->best = res.best;
        st->kstar = res.kstar;
        st->R = res.R;
        st->count = need;
        *npaths_out = need;
    }
    // per-parent counts
    if (blockIdx.x * PPB >= np) return;  // uniform
    const bool g = key > res.kstar, e = key != 0u && key == res.kstar;
    const uint64_t seg = parent_lanes(lane, lgKp);
    const int32_t ng = __popcll(__ballot(g) & seg), ne = __popcll(__ballot(e) & seg);
    if (j == 0 && p < np) pcnt[p] = (int64_t)ng | ((int64_t)ne << 32);
}

// Survivors' positions (path order) and rows; clears the histogram.
__global__ __launch_bounds__(MX_THREADS) void k_merge_scatter(const MergeLevel* lv, int i, const uint32_t* cand,
                                                              int K, int lgKp, const int32_t* npaths,
                                                              const MergeLvState* st, const uint32_t* keys,
                                                              const int64_t* pcnt, const uint32_t* prow,
                                                              uint32_t* nrow, int nw, int64_t* scores, int final_out,
                                                              int nV, int32_t* hist, int copies, int32_t* below)
{
    __shared__ int64_t s_red[MX_THREADS / 64];
    __shared__ int64_t s_pc[MX_THREADS];
    __shared__ int32_t s_n;
    __shared__ int32_t s_pos[MX_THREADS], s_src[MX_THREADS];
    __shared__ uint32_t s_bits[MX_THREADS];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    // The next level's histogram starts from zero: every block clears its share of
    // the (copy, super bin) pairs, those that hold something (few do).
    for (int x0 = blockIdx.x; x0 < copies * SUPER_BINS; x0 += 64 * gridDim.x) {
        const int x = x0 + lane * gridDim.x;
        int32_t* at = hist + (size_t)(x / SUPER_BINS) * MERGE_HIST_INTS;
        uint64_t some = __ballot(x < copies * SUPER_BINS && at[SUPER_AT + x % SUPER_BINS] != 0);
        __syncthreads();  // every wave has looked
        for (; some; some &= some - 1) {
            const int y = x0 + (__ffsll((unsigned long long)some) - 1) * (int)gridDim.x, sb = y % SUPER_BINS;
            int32_t* h = hist + (size_t)(y / SUPER_BINS) * MERGE_HIST_INTS;
            h[(sb << SUPER_SHIFT) + t] = 0;
            if (t < 16) h[FINE_BINS + (sb << 4) + t] = 0;
            if (t == 0) h[SUPER_AT + sb] = 0;
        }
    }
    if (blockIdx.x == 0 && t == 0) *below = 0;
    const int PPB = MX_THREADS >> lgKp;
    const int p0 = blockIdx.x * PPB;
    const MergeLevel& L = lv[i];
    const int np = npaths[i], start = L.start, size = L.size;
    const uint32_t kstar = st->kstar;
    const int32_t R = st->R;
    if (p0 >= np) return;  // uniform
    const int pl = t >> lgKp, j = t & ((1 << lgKp) - 1);
    const int p = p0 + pl;
    // independent loads first: this child's key, candidate and the parent's
    // bit of the shared vertex, the block's parent counts
    const bool mine = p < np && j < K;
    const uint32_t key = mine ? keys[(size_t)p * K + j] : 0u;
    const uint32_t b = mine ? cand[(size_t)i * K + j] : 0u;
    const uint32_t xs = mine ? row_bit(prow + (size_t)p * nw, start) : 0u;
    const int64_t pc = (t < PPB && p0 + t < np) ? pcnt[p0 + t] : 0;
    if (t == 0) s_n = 0;
    // (gt, eq) counts of the parents before this block, 16-byte loads
    int64_t acc = 0;
#pragma unroll 4
    for (int x = 2 * t; x + 1 < p0; x += 2 * MX_THREADS) {
        const longlong2 v = *(const longlong2*)(pcnt + x);
        acc += v.x + v.y;
    }
    if ((p0 & 1) && t == 0) acc += pcnt[p0 - 1];
    s_pc[t] = pc;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    if (lane == 0) s_red[wv] = acc;
    __syncthreads();
    int64_t before = 0;
    for (int w = 0; w < MX_THREADS / 64; ++w) before += s_red[w];
    for (int q = 0; q < pl; ++q) before += s_pc[q];  // the block's earlier parents
    const bool g = key > kstar, e = key != 0u && key == kstar;
    const uint64_t earlier = ((1ull << lane) - 1ull) & parent_lanes(lane, lgKp);
    const int32_t my_gt = (int32_t)(before & 0xFFFFFFFFll) + __popcll(__ballot(g) & earlier);
    const int32_t my_eq = (int32_t)(before >> 32) + __popcll(__ballot(e) & earlier);
    if (g || (e && my_eq < R)) {
        const int32_t pos = my_gt + (my_eq < R ? my_eq : R);
        const uint32_t o = (b & 1u) ^ xs;
        const int slot = atomicAdd(&s_n, 1);
        s_pos[slot] = pos;
        s_src[slot] = p;
        s_bits[slot] = level_bits(b, o, size);
        scores[final_out ? 0 : pos] = (int64_t)key - 1;  // final: the best cut
    }
    __syncthreads();
    // rows: lanes over the words of a survivor, then over survivors
    const int nwp = final_out ? nw : (start + size + 31) >> 5;
    const int n = s_n;
    int lw = 0;
    while ((1 << lw) < nwp && lw < 8) ++lw;
    const int w0 = t & ((1 << lw) - 1);
#pragma unroll 4
    for (int s = t >> lw; s < n; s += MX_THREADS >> lw) {
        const uint32_t* src = prow + (size_t)s_src[s] * nw;
        uint32_t* dst = nrow + (size_t)(final_out ? 0 : s_pos[s]) * nw;
        const uint32_t bits = s_bits[s];
        for (int q = w0; q < nwp; q += 1 << lw) {
            uint32_t w = place_bits(src[q], q, start, size, bits);
            if (final_out && q == nw - 1 && (nV & 31)) w &= (1u << (nV & 31)) - 1u;
            dst[q] = w;
        }
    }
}

__global__ void k_merge_fail(uint32_t* out, int nw, int64_t* cut, const int32_t* nsurv)
{
    if (*nsurv > 0) return;
    for (int q = threadIdx.x; q < nw; q += blockDim.x) out[q] = 0u;
    if (threadIdx.x == 0) *cut = -1;
}

hipError_t launch_merge(const MergeBufs& m, int M, int K, int W, int nw, int nV, const uint32_t* cand,
                        uint32_t* best, int64_t* best_cut, hipStream_t s)
{
    int lgKp = 0;
    while ((1 << lgKp) < K) ++lgKp;
    hipLaunchKernelGGL(k_merge_intra, dim3(M + 32), dim3(INTRA_THREADS), 0, s, M, m.lv, m.intra, cand, K, lgKp, m.ccut,
                       m.lvk, m.maxinc, m.hist, m.below);
    hipLaunchKernelGGL(k_merge_first, dim3(1), dim3(128), 0, s, m.lvk, K, m.ccut, m.keys, m.counts);
    // level 1: counts[0] = 1 path, counts[1] = its survivors
    const bool last0 = M == 1;
    hipLaunchKernelGGL(k_merge_select, dim3(1), dim3(SEL_THREADS), 0, s, m.keys, m.counts, 2 * K, last0 ? 1 : W,
                       m.surv, m.counts + 1, m.lvs);
    hipLaunchKernelGGL(k_merge_build, dim3(last0 ? 1 : W), dim3(64), 0, s, m.lv, cand, m.surv, m.counts + 1,
                       last0 ? best : m.rows[0], nw, last0 ? best_cut : m.scores, last0 ? 1 : 0, nV);
    const int PPB = MX_THREADS >> lgKp;
    const int nblk = (W + PPB - 1) / PPB;
    // Expand's workgroups take fewer parents where there are few of them, down to
    // one (parent, vertex) pair per thread: their back edges are what takes long. A
    // level in us, PPB parents / fewer (1000 vertices): K 4, W 64 53.3 / 22.2, W 4096
    // 57.5 / 32.7; K 16, W 64 26.2 / 21.4, W 2048 30.0 / 26.5. With 512 workgroups
    // instead of 256 a sparse graph's merge (2000 vertices, W 4096) takes 2.69
    // instead of 2.59 ms, a denser one's level (1000) 30.1 instead of 31.4 us.
    int epb = PPB;
    while (epb * 32 > MX_THREADS && (W + epb - 1) / epb < 256) epb /= 2;
    const int eblk = (W + epb - 1) / epb;
    const int copies = eblk > 64 ? MERGE_COPIES : 1;
    int cur = 0;
    for (int i = 1; i < M; ++i) {
        const bool last = i == M - 1;
        hipLaunchKernelGGL(k_merge_expand, dim3(eblk), dim3(MX_THREADS), 0, s, m.lv, i, m.back, cand, K, lgKp, epb,
                           m.ccut, m.lvk, m.rows[cur], nw, m.scores, m.counts, m.lvs, m.maxinc, m.keys, m.hist,
                           copies, m.below);
        hipLaunchKernelGGL(k_merge_count, dim3(nblk), dim3(MX_THREADS), 0, s, i, K, lgKp, m.counts + i,
                           last ? 1 : W, m.lvs + (i - 1), m.maxinc, m.keys, m.hist, copies, m.below, m.pcnt, m.lvs + i,
                           m.counts + i + 1);
        hipLaunchKernelGGL(k_merge_scatter, dim3(nblk), dim3(MX_THREADS), 0, s, m.lv, i, cand, K, lgKp, m.counts,
                           m.lvs + i, m.keys, m.pcnt, m.rows[cur], last ? best : m.rows[cur ^ 1], nw,
                           last ? best_cut : m.scores, last ? 1 : 0, nV, m.hist, copies, m.below);
        cur ^= 1;
    }
    hipLaunchKernelGGL(k_merge_fail, dim3(1), dim3(64), 0, s, best, nw, best_cut, m.counts + M);
    return hipGetLastError();
}

}  // namespace pq

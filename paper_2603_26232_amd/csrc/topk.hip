// Top-k bitstring extraction (paper Sec. 3.3.2, Selective Distribution
// Exploration): per subgraph, the k bitstrings with the largest probability
// pi(z) = |psi(z)|^2.
//
// Ties. pi(z) is exactly invariant under flipping the bit of a free vertex
// (one without an edge of positive weight in the subgraph: its qubit stays
// in |+>) and under the complement. The candidates these moves connect form
// a tie group: with Fm = the free vertices (other than vertex 0 in canonical
// mode), a group is {r0 ^ S} or, when the complement move stays inside the
// candidates (raw mode, or canonical mode with vertex 0 free) and the
// subgraph has a vertex that is not free, {r0 ^ S} u {r1 ^ S}, S over the
// subsets of Fm; r0 < r1 have no bit in Fm and are each other's complement
// (with bit 0 flipped back in canonical mode) restricted to the other bits.
// The order is the group's probability descending, then r0 ascending, then
// a fixed bijective rank of the string inside the group; in FP32, members of
// one group would otherwise be ordered by rounding noise. So stage 1 keeps
// only the representatives r0, and stage 2 expands each selected group into
// its members in rank order: member j of a group of 2^m is the index
// x = rank^-1(j) (half in the low bit when there are two halves, the bits of
// S at Fm above it), rank(x) = g(A g(x) mod 2^m), g(x) = x ^ (x >> ceil(m/2))
// (a xorshift step, its own inverse on m bits) and A = 2654435761 (Knuth's
// multiplicative hashing); rank^-1(j) = g(A^-1 g(j) mod 2^m).
//
// Each representative becomes one unique 64-bit key, (bits of pi as float)
// << 32 | (0xFFFFFFFF - z): pi >= 0, so the float bit pattern orders like
// the value, and a larger low word means a smaller z. Every valid key is
// nonzero (z < 2^30), so 0 serves as padding below all of them.
//
// Stage 1 streams the reduced state once: a block takes a run of 4096-amplitude
// tiles (a run that crosses subgraphs starts anew in each), with the next tile's
// amplitudes on their way, and appends the keys above a threshold to a buffer in
// LDS, which are few after the first tile; when the buffer is full, or long
// beyond k, it is cut to its k largest, the smallest of which is the new
// threshold. The run's best k are written unsorted. Stage 2 selects a subgraph's
// best k from its runs' lists, orders them by rank and expands them; stage 1 does
// that itself for a subgraph that a run holds whole, and there is no stage 2 where
// every subgraph is a single tile (2048 subgraphs of 9 qubits, k = 16: 19 us; with runs
// of two and stage 2 57).
//
// A selection counts keys in 256 bins over the 8 octaves of probability below
// the largest one (1/32 octave each: most keys of a state spread over them, so
// the LDS atomics do not meet in one bin), then over the bin that holds the k-th,
// until a bin boundary is the answer; if fewer than k keys are in the window, it
// starts over the whole range. A bin of few keys is ranked key by key instead: of at
// most 32, or, from the second round on, of 256 (equal probabilities differ in the
// string only, which takes six more rounds: four 20-qubit states of graphs with three
// edges, k = 1, 23.9 / 14.7 us; ranking 256 in the first round costs narrow distributions
// more than the second round does, one state of 9 qubits 17.5 / 11.6 us).
// Canonical mode takes only z with bit 0 clear (pi(z) = pi(~z)).
//
// Bound: the 8 bytes per stored amplitude that stage 1 reads. Measured on 8704
// tiles (four subgraphs, the largest of 26 qubits), k = 16: stage 1 74 us (3.9
// TB/s), stage 2 13 us. A list per tile and a selection by digits from the top of
// the key, whose first digits all keys share, took 113 and 202 us; runs of four
// tiles instead of eight 70 and 21 us.
#include "lane.h"

namespace pq {

// tie groups of one subgraph (see the file comment)
struct TieGroups {
    uint32_t fm;    // free vertices that a group's strings may differ in
    uint32_t full;  // all n bits
    int halves;     // 2: a group also holds the complement-side half
    int m;          // a group has 2^m strings
    int canonical;
};

__device__ inline TieGroups tie_groups(const SubDesc* d, int canonical)
{
    TieGroups t;
    t.full = (uint32_t)((1ull << d->n) - 1ull);
    t.fm = canonical ? (d->freem & ~1u) : d->freem;
    const bool part_ok = canonical ? (d->freem & 1u) != 0u : true;
    t.halves = (part_ok && d->freem != t.full) ? 2 : 1;
    t.m = __popc(t.fm) + (t.halves == 2 ? 1 : 0);
    t.canonical = canonical;
    return t;
}

// the complement move restricted to the bits outside Fm
__device__ inline uint32_t partner_base(const TieGroups& t, uint32_t z)
{
    const uint32_t c = (~z & t.full) ^ (t.canonical ? 1u : 0u);
    return c & ~t.fm;
}

// is z the representative (smallest base) of its tie group?
__device__ inline bool is_representative(const TieGroups& t, uint32_t z)
{
    if (z & t.fm) return false;
    return t.halves == 1 || z <= partner_base(t, z);
}

constexpr uint32_t TIE_MUL_INV = 0x0E8B2F51u;  // 2654435761^-1 mod 2^32
static_assert(2654435761u * TIE_MUL_INV == 1u, "multiplicative inverse");

__device__ inline uint32_t tie_unrank(uint32_t j, int m)
{
    if (m <= 0) return 0u;
    const uint32_t mask = m >= 32 ? 0xFFFFFFFFu : ((1u << m) - 1u);
    const int s = (m + 1) / 2;
    uint32_t x = j ^ (j >> s);
    x = (x * TIE_MUL_INV) & mask;  // mod 2^32 then mod 2^m
    return x ^ (x >> s);
}

// deposit the low bits of v at the set positions of mask
__device__ inline uint32_t deposit_bits(uint32_t v, uint32_t mask)
{
    uint32_t out = 0;
    for (int j = 0; j < 32 && mask; ++j) {
        const uint32_t low = mask & (0u - mask);
        if (v & 1u) out |= low;
        v >>= 1;
        mask ^= low;
    }
    return out;
}

// string j (in rank order) of the group with representative r0
__device__ inline uint32_t tie_member(const TieGroups& t, uint32_t r0, uint32_t j)
{
    const uint32_t x = tie_unrank(j, t.m);
    const uint32_t half = t.halves == 2 ? (x & 1u) : 0u;
    const uint32_t sp = t.halves == 2 ? (x >> 1) : x;
    const uint32_t base = half ? partner_base(t, r0) : r0;
    return base ^ deposit_bits(sp, t.fm);
}

struct SelState {
    int hist[256];
    int wsum[4];
    uint32_t wmax[16];
    int bin, excl, h, total, count, few;
    uint64_t out[MAX_K];
    uint64_t cand[256], answer;  // keys of the k-th one's bin
};

// the largest value over the block's waves
__device__ inline uint32_t block_max(SelState& S, uint32_t x)
{
    x = wave_max(x);
    if ((threadIdx.x & 63u) == 0) S.wmax[threadIdx.x >> 6] = x;
    __syncthreads();
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) x = S.wmax[w] > x ? S.wmax[w] : x;
    return x;
}

// Smallest of the q largest keys that each(f) passes to f, every thread its own
// (zero keys are none; at least q others, all different). top: the largest upper
// word (probability, as bits) among them. Called by every thread of the block.
template <typename Each>
__device__ uint64_t select_smallest(SelState& S, const Each& each, int q, uint32_t top)
{
    const int t = threadIdx.x;
    uint64_t hi = ((uint64_t)top << 32) | 0xFFFFFFFFull;
    uint64_t lo = hi > (1ull << 58) ? hi - (1ull << 58) + 1ull : 1ull;
    int shift = 50;  // (hi - lo) >> shift < 256
    for (int round = 0;; ++round) {
        __syncthreads();  // the last round's results have been read
        if (t < 256) S.hist[t] = 0;
        if (t == 0) S.few = 0;
        __syncthreads();
        each([&](uint64_t key) {
            if (key >= lo && key <= hi) atomicAdd(&S.hist[(int)((hi - key) >> shift)], 1);
        });
        __syncthreads();
        int h = 0, incl = 0;
        if (t < 256) {
            h = S.hist[t];
            incl = h;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int y = __shfl_up(incl, o, 64);
                if ((t & 63) >= o) incl += y;
            }
            if ((t & 63) == 63) S.wsum[t >> 6] = incl;
        }
        __syncthreads();
        if (t < 256) {
            for (int w = 0; w < (t >> 6); ++w) incl += S.wsum[w];
            if (t == 255) S.total = incl;
            if (incl - h < q && q <= incl) {  // one bin, if any
                S.bin = t;
                S.excl = incl - h;
                S.h = h;
            }
        }
        __syncthreads();
        if (round == 0 && S.total < q) {
            lo = 1ull;
            shift = 56;
            continue;
        }
        const uint64_t b = (uint64_t)S.bin;
        const int excl = S.excl;
        const uint64_t top_of = hi - (b << shift);
        const uint64_t low_of = top_of - lo >= (1ull << shift) ? top_of - (1ull << shift) + 1ull : lo;
        const int held = S.h;
        if (excl + held == q) return low_of;
        q -= excl;
        if (held <= 32 || (round > 0 && held <= 256)) {
            each([&](uint64_t key) {
                if (key >= low_of && key <= top_of) S.cand[atomicAdd(&S.few, 1)] = key;
            });
            __syncthreads();
            if (t < held) {
                const uint64_t mine = S.cand[t];
                int above = 0;
#pragma unroll 8
                for (int i = 0; i < held; ++i) above += S.cand[i] > mine;
                if (above == q - 1) S.answer = mine;
            }
            __syncthreads();
            return S.answer;
        }
        hi = top_of;
        lo = low_of;
        shift = shift >= 8 ? shift - 8 : 0;
    }
}

__device__ inline uint64_t make_key(float pr, uint32_t z)
{
    return ((uint64_t)__float_as_uint(pr) << 32) | (uint64_t)(0xFFFFFFFFu - z);
}

// The n <= k <= 64 keys of S.out (any order, all different) in descending order,
// expanded into their groups' strings in rank order: row b of the results. The
// first wave does the work; S.out is in place (a barrier before).
__device__ inline void write_row(const SelState& S, const TieGroups& tg, int n, int b, int k, uint32_t* idx,
                                 float* prob, uint64_t* sorted)
{
    const int lane = threadIdx.x;
    if (lane >= 64) return;
    if (lane < n) {
        const uint64_t key = S.out[lane];
        int rank = 0;
        for (int j = 0; j < n; ++j) rank += S.out[j] > key;
        sorted[rank] = key;
    }
    asm volatile("" ::: "memory");  // one wave: the LDS keeps issue order
    if (lane >= k) return;
    const int g = tg.m >= 6 ? 0 : lane >> tg.m;  // group of output `lane`, and its string
    const uint32_t j = tg.m >= 6 ? (uint32_t)lane : (uint32_t)lane & ((1u << tg.m) - 1u);
    uint32_t z = 0xFFFFFFFFu;
    float pr = -1.0f;
    if (g < n) {
        const uint64_t key = sorted[g];
        z = tie_member(tg, 0xFFFFFFFFu - (uint32_t)(key & 0xFFFFFFFFull), j);
        pr = __uint_as_float((uint32_t)(key >> 32));
    }
    idx[(size_t)b * k + lane] = z;
    prob[(size_t)b * k + lane] = pr;
}

// stage 1: tiles [blockIdx * run, + run) of the batch. Each subgraph's part of
// the run leaves its best k keys (unsorted, 0-padded) at slot k * (its first
// tile), or, where the run holds the whole subgraph, the results.
//
// The first tile of a part has no threshold yet. A lower bound of it is the k-th
// largest of the threads' largest keys: at most k threads have keys that large,
// so at most 64 x 32 keys are appended. The same bound is taken where a later
// tile's candidates do not fit.
constexpr int SLACK = 256;  // keys beyond k that are kept before the buffer is cut
constexpr int BUF = MAX_K * 32 + MAX_K + SLACK;

template <bool CANON>
__global__ __launch_bounds__(THREADS) void k_topk_run(const uint8_t* ws, const SubDesc* subs, const int2* work,
                                                     int total, int run, int k, uint64_t* out,
                                                     uint32_t* idx, float* prob)
{
    // The stored state is reduced: amplitude z' (top bit clear, scaled by
    // sqrt(2)) stands for z' and its complement z' ^ (2^n - 1), each with
    // probability |phi(z')|^2 / 2. The canonical one of the pair is the one
    // with bit 0 clear; raw mode takes both.
    constexpr int AMPS = TILE / THREADS;          // 16 amplitudes per thread
    constexpr int PER = CANON ? AMPS : 2 * AMPS;  // candidates per thread
    __shared__ SelState S;
    __shared__ uint64_t buf[BUF];
    const int t = threadIdx.x, lane = t & 63;
    const uint64_t below = (1ull << lane) - 1ull;
    const int end = (blockIdx.x + 1) * run < total ? (blockIdx.x + 1) * run : total;
    for (int first = blockIdx.x * run; first < end;) {
        const int2 wk = work[first];
        const SubDesc* d = subs + wk.x;
        const int last = d->tile_base + d->ntiles < end ? d->tile_base + d->ntiles : end;
        const int n = d->n;
        const uint32_t span = n - 1 < TILE_BITS ? (1u << (n - 1)) : (uint32_t)TILE;
        const uint32_t full = (uint32_t)((1ull << n) - 1ull);
        const TieGroups tg = tie_groups(d, CANON ? 1 : 0);
        const float2* st = (const float2*)(ws + d->psi) + (size_t)wk.y * TILE;
        uint32_t base = (uint32_t)wk.y * TILE;
        float2 next[AMPS];
        auto load = [&](const float2* p) {
#pragma unroll
            for (int j = 0; j < AMPS; ++j) {
                const uint32_t c = (uint32_t)t + (uint32_t)j * THREADS;
                next[j] = c < span ? p[c] : make_float2(0.f, 0.f);
            }
        };
        load(st);
        uint64_t thr = 0;  // keys above it are candidates
        int nbuf = 0;
        if (t == 0) S.count = 0;
        auto buffered = [&](int m, auto f) {
            for (int i = t; i < m; i += THREADS) f(buf[i]);
        };
        auto buffer_top = [&](int m) {
            uint32_t top = 0;
            buffered(m, [&](uint64_t x) { top = (uint32_t)(x >> 32) > top ? (uint32_t)(x >> 32) : top; });
            return block_max(S, top);
        };
        __syncthreads();
        for (int tile = first; tile < last; ++tile, base += TILE) {
            float pr[AMPS];
#pragma unroll
            for (int j = 0; j < AMPS; ++j) pr[j] = 0.5f * (next[j].x * next[j].x + next[j].y * next[j].y);
            if (tile + 1 < last) load(st + (size_t)(tile + 1 - first) * TILE);
            // candidate i of the tile: its key, or 0 (only the representatives
            // of tie groups are ranked)
            auto key_of = [&](int i) -> uint64_t {
                const int j = CANON ? i : i >> 1;
                const uint32_t c = (uint32_t)t + (uint32_t)j * THREADS;
                uint32_t z = base + c;
                if (CANON ? (z & 1u) : (uint32_t)(i & 1)) z ^= full;
                return c < span && is_representative(tg, z) ? make_key(pr[j], z) : 0ull;
            };
            int now = 0;
            for (bool bound = tile == first;; bound = true) {
                if (bound) {
                    uint64_t mx = 0;
#pragma unroll
                    for (int i = 0; i < PER; ++i) {
                        const uint64_t key = key_of(i);
                        mx = key > thr && key > mx ? key : mx;
                    }
                    const int some = __syncthreads_count(mx != 0ull);
                    if (some >= k) {
                        const uint32_t top = block_max(S, (uint32_t)(mx >> 32));
                        thr = select_smallest(S, [&](auto f) { f(mx); }, k, top) - 1ull;
                    }
                }
                const uint32_t pmin = (uint32_t)(thr >> 32);
#pragma unroll
                for (int i = 0; i < PER; ++i) {
                    if (__ballot(__float_as_uint(pr[CANON ? i : i >> 1]) >= pmin) == 0ull) continue;
                    const uint64_t key = key_of(i);
                    const uint64_t mask = __ballot(key > thr);
                    if (mask == 0ull) continue;
                    int at = 0;
                    if (lane == 0) at = atomicAdd(&S.count, __popcll(mask));
                    at = __shfl(at, 0) + __popcll(mask & below);
                    if (key > thr && at < BUF) buf[at] = key;
                }
                __syncthreads();
                now = S.count;
                if (now <= BUF) break;
                __syncthreads();  // (every thread has read the count)
                if (t == 0) S.count = nbuf;
                __syncthreads();
            }
            nbuf = now;
            if (now > k + SLACK) {
                const uint32_t top = buffer_top(now);
                const uint64_t low = select_smallest(S, [&](auto f) { buffered(now, f); }, k, top);
                // the survivors, over the front of the buffer
                constexpr int EACH = (BUF + THREADS - 1) / THREADS;
                uint64_t mine[EACH];
#pragma unroll
                for (int i = 0; i < EACH; ++i) mine[i] = t + i * THREADS < now ? buf[t + i * THREADS] : 0ull;
                __syncthreads();
                if (t == 0) S.count = 0;
                __syncthreads();
#pragma unroll
                for (int i = 0; i < EACH; ++i)
                    if (mine[i] >= low) buf[atomicAdd(&S.count, 1)] = mine[i];
                thr = low - 1ull;
                nbuf = k;
            }
            __syncthreads();
        }
        int n_out = nbuf;
        if (nbuf > k) {
            const uint32_t top = buffer_top(nbuf);
            const uint64_t low = select_smallest(S, [&](auto f) { buffered(nbuf, f); }, k, top);
            __syncthreads();
            if (t == 0) S.count = 0;
            __syncthreads();
            buffered(nbuf, [&](uint64_t x) {
                if (x >= low) S.out[atomicAdd(&S.count, 1)] = x;
            });
            n_out = k;
        } else if (t < nbuf) {
            S.out[t] = buf[t];
        }
        __syncthreads();
        if (last - first == d->ntiles) write_row(S, tg, n_out, wk.x, k, idx, prob, buf);
        else if (t < k) out[(size_t)first * k + t] = t < n_out ? S.out[t] : 0ull;
        __syncthreads();
        first = last;
    }
}

// stage 2: a subgraph's lists (one per run that it has a part in) -> its best k
constexpr int MERGE_THREADS = 1024;
constexpr int MERGE_HELD = 16;  // keys a thread keeps in registers

__global__ __launch_bounds__(MERGE_THREADS) void k_topk_merge(const SubDesc* subs, int run, int k, int canonical,
                                                             const uint64_t* in, uint32_t* idx, float* prob)
{
    __shared__ SelState S;
    __shared__ uint64_t sorted[MAX_K];
    const int b = blockIdx.x;
    const SubDesc* d = subs + b;
    const int t = threadIdx.x;
    const TieGroups tg = tie_groups(d, canonical);
    if (d->skip) {
        // edgeless subgraph: |psi|^2 = 2^-n everywhere, so all candidates form
        // one tie group (every vertex free) with representative 0
        if (t < k) {
            const bool ok = (uint64_t)t < (1ull << tg.m);
            idx[(size_t)b * k + t] = ok ? tie_member(tg, 0u, (uint32_t)t) : 0xFFFFFFFFu;
            prob[(size_t)b * k + t] = ok ? ldexpf(1.0f, -d->n) : -1.0f;
        }
        return;
    }
    // list 0 at the subgraph's first tile, list j > 0 at the j-th run boundary after it
    const int t0 = d->tile_base, r0 = t0 / run;
    const int lists = (t0 + d->ntiles - 1) / run - r0 + 1, total = lists * k;
    if (lists == 1) return;  // stage 1 has written its results
    auto at = [&](int x) -> uint64_t {
        const int j = x / k;
        return in[(size_t)(j == 0 ? t0 : (r0 + j) * run) * k + (x - j * k)];
    };
    const int nloc = (total - t + MERGE_THREADS - 1) / MERGE_THREADS;  // keys t, t + 1024, ...
    const bool held = total <= MERGE_HELD * MERGE_THREADS;
    uint64_t key[MERGE_HELD];
#pragma unroll
    for (int i = 0; i < MERGE_HELD; ++i) key[i] = held && i < nloc ? at(t + i * MERGE_THREADS) : 0ull;
    if (t == 0) S.count = 0;
    __syncthreads();
    uint32_t top = 0;
    int mine = 0;
    auto each = [&](auto f) {
        if (held) {
#pragma unroll
            for (int i = 0; i < MERGE_HELD; ++i) f(key[i]);
        } else {
            for (int i = 0; i < nloc; ++i) f(at(t + i * MERGE_THREADS));
        }
    };
    each([&](uint64_t x) {
        top = (uint32_t)(x >> 32) > top ? (uint32_t)(x >> 32) : top;
        mine += x != 0ull;
    });
    for (int off = 32; off > 0; off >>= 1) mine += __shfl_xor(mine, off);
    if ((t & 63) == 0 && mine) atomicAdd(&S.count, mine);
    top = block_max(S, top);  // (its barrier also shows the count)
    const int cnt = S.count;
    const uint64_t low = cnt > k ? select_smallest(S, each, k, top) : 1ull;
    __syncthreads();
    if (t == 0) S.count = 0;
    __syncthreads();
    each([&](uint64_t x) {
        if (x >= low) S.out[atomicAdd(&S.count, 1)] = x;
    });
    __syncthreads();
    write_row(S, tg, cnt < k ? cnt : k, b, k, idx, prob, sorted);
}

// Tiles per run: enough blocks for the chip (about 1024, four per CU) and few
// lists per subgraph; 1 while the batch has fewer tiles than that.
static int topk_run(int total)
{
    int run = 1;
    while (run < 256 && total / (2 * run) >= 1024) run *= 2;
    return run;
}

// single: no subgraph has more than one tile and none is skipped (then a run holds
// whole subgraphs only)
hipError_t launch_topk(uint8_t* ws, const SubDesc* subs, const int2* work, int nwork, int B, int k, int canonical,
                       bool single, uint64_t* keys, uint32_t* idx, float* prob, hipStream_t s)
{
    const int run = single ? 1 : topk_run(nwork);
    if (nwork > 0) {
        const dim3 g((nwork + run - 1) / run), b(THREADS);
        auto* f = canonical ? k_topk_run<true> : k_topk_run<false>;
        hipLaunchKernelGGL(f, g, b, 0, s, ws, subs, work, nwork, run, k, keys, idx, prob);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess || single) return e;
    }
    hipLaunchKernelGGL(k_topk_merge, dim3(B), dim3(MERGE_THREADS), 0, s, subs, run, k, canonical, keys, idx, prob);
    return hipGetLastError();
}

}  // namespace pq

// Device helpers shared by the tile-pass translation units (sim.hip: 4096-
// amplitude tiles, wide.hip: 16384-amplitude tiles).
#pragma once

#include "lane.h"

namespace pq {

// ---------------------------------------------------------------------------
// tile geometry
// ---------------------------------------------------------------------------
struct Geo {
    uint32_t zb;   // fixed index bits of this tile
    int c;         // passive low tile bits (contiguous amplitudes)
    int g0;        // first qubit of the group
    int nb;        // qubits in the group (active tile bits = [c, TB))
    uint32_t mir;  // group 0: 2^(n-1) - 1 (the complement of a reduced index)
};

// tile position q -> z offset (bit deposit; zb supplies the fixed bits)
__device__ inline uint32_t gmap(const Geo& g, uint32_t q)
{
    return (q & ((1u << g.c) - 1u)) | ((q >> g.c) << g.g0);
}

// Group 0 tiles pair a block of 2^(TB-1) reduced indices with its mirror block:
// tile bits 0..TB-2 are qubits 0..TB-2 and tile bit TB-1 selects the block or its
// complement (index XOR 2^(n-1) - 1). In the reduced state the top qubit's
// X maps an index to its complement, so it acts on tile bit 11 like any other
// qubit on its bit. The map is XOR-linear, as the deposit of the other groups.
template <int TB = TILE_BITS>
__device__ inline uint32_t gmap0(const Geo& g, uint32_t q)
{
    return (q & ((1u << (TB - 1)) - 1u)) ^ ((q >> (TB - 1)) & 1u ? g.mir : 0u);
}

template <bool G0, int TB = TILE_BITS>
__device__ inline uint32_t gmapT(const Geo& g, uint32_t q)
{
    if constexpr (G0) return gmap0<TB>(g, q);
    else return gmap(g, q);
}

// tile t of group g (TB: tile bits; a constant in the pass kernels)
__device__ inline Geo make_geo(const SubDesc* sd, int g, uint32_t t, int TB = TILE_BITS)
{
    Geo r;
    r.mir = 0;
    if (g == 0) {
        r.c = 0;
        r.g0 = 0;
        r.nb = TB;
        r.zb = t << (TB - 1);
        r.mir = (1u << (sd->n - 1)) - 1u;
    } else {
        r.nb = sd->gsize[g];
        r.g0 = sd->gstart[g];
        r.c = TB - r.nb;
        const int L = r.g0 - r.c;  // fixed bits between the passive block and the group
        const uint32_t tlo = t & ((1u << L) - 1u), thi = t >> L;
        r.zb = (tlo << r.c) | (thi << (r.g0 + r.nb));
    }
    return r;
}

// tile position of entry e of a wide tile's cut table (order: lane, register)
__device__ inline uint32_t wide_entry(uint32_t e)
{
    const uint32_t lane = e / WIDE_REGS, r = e % WIDE_REGS;
    return row_bits(lane & 15u) | (r << 4) | ((lane >> 4) << 9);
}

// Reduced pair rotation (I - i t X) on (a, b) = (psi(z), psi(z ^ bit)):
// (a, b) -> (a - i t b, b - i t a). t = 0 is exactly the identity.
__device__ inline void rx_tan(float2& a, float2& b, float t)
{
    const float2 na = make_float2(a.x + t * b.y, a.y - t * b.x);
    const float2 nb = make_float2(b.x + t * a.y, b.y - t * a.x);
    a = na;
    b = nb;
}

// Per-layer rotation parameters (built in FP64 by the angle-prep kernel):
// e^{-i beta X} = f (I - i t X) X^flip per qubit.
struct RxC {
    float t;
    int flip;
    float fsq;      // |f|^2
    float2 Ff, Fi;  // f^(group size), forward and inverse
};

__device__ inline RxC load_rx(const RxCoef* cf, int l, int g)
{
    RxC r;
    r.t = cf[l].t;
    r.flip = cf[l].mode;
    r.fsq = cf[l].fsq;
    r.Ff = cf[l].Ff[g];
    r.Fi = cf[l].Fi[g];
    return r;
}

// OFF32: addresses as 32-bit byte offsets from the state's (uniform) base
// (a stored state of n <= 30 qubits spans at most 2^29 amplitudes = 4 GiB).
// The map is XOR-linear, so a register's offset is the lane's offset XOR a
// per-register value that is uniform across the workgroup: one vector XOR
// per access instead of an XOR and a 64-bit address add.
__device__ inline const float2& at_off(const float2* st, uint32_t off)
{
    return *(const float2*)((const uint8_t*)st + off);
}
__device__ inline float2& at_off(float2* st, uint32_t off) { return *(float2*)((uint8_t*)st + off); }

// deterministic block sum (wave64 butterfly, then the 4 wave totals in order)
// three deterministic block sums with one barrier pair
__device__ inline void block_sum3(double& a, double& b, double& c, double* red)
{
    for (int off = 32; off > 0; off >>= 1) {
        a += __shfl_xor(a, off);
        b += __shfl_xor(b, off);
        c += __shfl_xor(c, off);
    }
    const uint32_t tid = threadIdx.x;
    const int nw = (int)(blockDim.x >> 6);
    if ((tid & 63u) == 0) {
        red[tid >> 6] = a;
        red[nw + (tid >> 6)] = b;
        red[2 * nw + (tid >> 6)] = c;
    }
    __syncthreads();
    if (tid == 0) {
        double x = 0.0, y = 0.0, z = 0.0;
        for (int i = 0; i < nw; ++i) {
            x += red[i];
            y += red[nw + i];
            z += red[2 * nw + i];
        }
        a = x;
        b = y;
        c = z;
    }
}

}  // namespace pq

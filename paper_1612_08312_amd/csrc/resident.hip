// LDS-resident Swendsen-Wang sweeps of small Ising lattices (L <= 16; up to
// kQuadMaxL by the quad kernel below): one workgroup holds a whole lattice in LDS and runs all of its sweeps of a call
// in one launch, with only workgroup barriers between the steps.  The method
// is the one of the tiled sweep (Sec. 1-2 of the paper: bond activation,
// cluster labeling, flip of each cluster with probability 1/2, moments of
// Eq. 2) with the same random draws, so every record, spin and label is
// identical to the tiled path's.
//
// LDS of a lattice of N = 16 L^3 sites (N <= 65536, so a site index fits in
// 16 bits; offsets in resident.hpp):
//   PF   uint16 [N]       forest: parent site of each site; roots are the
//                         smallest site of their component (hooks put the
//                         larger root under the smaller)
//   SMK  uint16 [L^3]     spin mask of each cell (bit k: site k is -1)
//   CW   uint32 [N/32]    flip coins of the sweep: bit (r mod 32) of word
//                         r/32 is the coin of the cluster rooted at r
// At L = 16 that is 128 + 8 + 8 KiB.  One sweep:
//   1. each cell's 48 bonds are activated (ising_activate) and the
//      components of its four up tetrahedra seed the forest (K4 table);
//   2. the spanning edges of the components of each down tetrahedron are
//      united (every bond of the lattice is inside the workgroup);
//   3. the coins: one Philox block per 128 sites;
//   4. every site finds its root and flips with the root's coin (the labels
//      are written out after the last sweep);
//   5. magnetisation and bond sum of the new state, one record.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device_once.hpp"
#include "device_util.hpp"
#include "ising_cell.hpp"
#include "kernels.hpp"
#include "lattice.hpp"
#include "philox.hpp"
#include "resident.hpp"
#include "tile_common.hpp"

namespace pyro {

namespace {

// Record of one sweep from its exact sums (bond sum B, down spins D).
__device__ __forceinline__ DevRecord ising_record(const RepDesc &d, uint32_t sweep, int64_t B, int64_t D)
{
    const int64_t M = d.N - 2 * D;
    DevRecord rec;
    rec.sweep = sweep;
    rec.bond_sum = B;
    rec.M_int = M;
    rec.reserved = 0;
    rec.E = -d.J * (double)B;
    rec.M[0] = (double)M;
    rec.M[1] = 0.0;
    rec.M[2] = 0.0;
    const double mm = (double)M / (double)d.N;
    rec.m2 = mm * mm;
    rec.m4 = rec.m2 * rec.m2;
    return rec;
}

// 16 int8 spins of a cell's mask (+1 = 0x01, -1 = 0xFF).
__device__ __forceinline__ int4 mask_spins(uint32_t m)
{
    uint32_t w[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        w[q] = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) w[q] |= (((m >> (4 * q + b)) & 1u) ? 0xFFu : 0x01u) << (8 * b);
    }
    return make_int4((int)w[0], (int)w[1], (int)w[2], (int)w[3]);
}

typedef __attribute__((address_space(3))) volatile uint16_t lds_u16;
typedef __attribute__((address_space(3))) uint32_t lds_u32;

constexpr int kCellsPerThread = (kResidentMaxL * kResidentMaxL * kResidentMaxL + kResidentThreads - 1) / kResidentThreads;

// Root of site x with path halving (parents never exceed their children, so
// the walk steps to strictly smaller sites and ends).
__device__ __forceinline__ uint32_t find16(lds_u16 *PF, uint32_t x)
{
    uint32_t p = PF[x];
    while (p < x) {
        const uint32_t gp = PF[p];
        PF[x] = (uint16_t)gp;
        x = p;
        p = gp;
    }
    return x;
}

// Union of the components of sites a and b: the larger root is hooked under
// the smaller by a compare-and-swap of the 32-bit word holding its entry
// (the other half of the word may change meanwhile; the swap then fails and
// is retried on the word's new value).
__device__ __forceinline__ void unite16(lds_u16 *PF, uint32_t a, uint32_t b)
{
    for (;;) {
        a = find16(PF, a);
        b = find16(PF, b);
        if (a == b) return;
        if (a < b) {
            const uint32_t t = a;
            a = b;
            b = t;
        }
        lds_u32 *w = (lds_u32 *)((__attribute__((address_space(3))) char *)PF + 2 * (a & ~1u));
        const uint32_t sh = 16u * (a & 1u);
        uint32_t old = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        bool hooked = false;
        for (;;) {
            const uint32_t pa = (old >> sh) & 0xFFFFu;
            if (pa != a) {  // a was hooked meanwhile: continue from its new parent
                a = pa;
                break;
            }
            const uint32_t nw = (old & ~(0xFFFFu << sh)) | (b << sh);
            const uint32_t got = atomicCAS((uint32_t *)w, old, nw);
            if (got == old) {
                hooked = true;
                break;
            }
            old = got;
        }
        if (hooked) return;
    }
}

}  // namespace

// One workgroup of kResidentThreads threads per replica of the chain (all of
// edge L <= kResidentMaxL, no vacant sites): `remaining` sweeps, records into
// the ring, then the state is advanced as the tiled finalize would.
__global__ __launch_bounds__(kResidentThreads) void k_resident_ising(Chain c, RepState armed, bool use_armed)
{
    extern __shared__ __align__(16) char lds[];
    const int rep = blockIdx.x;
    const RepState st = use_armed ? armed : *c.state[rep];
    if (st.remaining <= 0) return;
    const RepDesc &d = c.desc[rep];
    const int L = d.L;
    const int ncell = (int)d.ncell;
    const int N = (int)d.N;
    const int tid = threadIdx.x;
    constexpr int NT = kResidentThreads;
    const ResidentLayout ly = resident_layout(L);
    __attribute__((address_space(3))) char *base = (__attribute__((address_space(3))) char *)lds;
    lds_u16 *PF = (lds_u16 *)(base + ly.pf);
    lds_u16 *SMK = (lds_u16 *)(base + ly.smk);
    lds_u32 *CW = (lds_u32 *)(base + ly.cw);
    __attribute__((address_space(3))) uint8_t *K4 = (__attribute__((address_space(3))) uint8_t *)(base + ly.k4);
    int64_t *red = (int64_t *)(lds + ly.red);

    if (tid < 64) {
        constexpr K4Table k4 = make_k4();
        K4[tid] = k4.v[tid];
    }
    // The six lower neighbour cells of each of the thread's cells.
    int nbc[kCellsPerThread][kNCellCodes];
#pragma unroll
    for (int j = 0; j < kCellsPerThread; ++j) {
        const int c0 = tid + j * NT;
        if (c0 < ncell) {
            const CellNbrs nb = cell_neighbours(c0, L);
#pragma unroll
            for (int q = 0; q < kNCellCodes; ++q) nbc[j][q] = nb.c[q];
            SMK[c0] = (uint16_t)spin_mask16(reinterpret_cast<const int4 *>(d.spins)[c0]);
        } else {
#pragma unroll
            for (int q = 0; q < kNCellCodes; ++q) nbc[j][q] = 0;
        }
    }
    __syncthreads();
    const IsingParams prm{d.thr_hi, d.thr_lo};
#define PYRO_DOWN_OF(j, m)                                                                                   \
    down_mask16((m), SMK[nbc[j][kMx]], SMK[nbc[j][kMy]], SMK[nbc[j][kMz]], SMK[nbc[j][kMyMz]],             \
                SMK[nbc[j][kMxMz]], SMK[nbc[j][kMxMy]])
    if (st.e_pending >= 0) {  // the record of a tiled sweep before this call: uniform
        int64_t bsum = 0, down = 0;
#pragma unroll
        for (int j = 0; j < kCellsPerThread; ++j) {
            if (tid + j * NT >= ncell) continue;
            const uint32_t m = SMK[tid + j * NT];
            bsum += 2 * (int64_t)__popcll(aligned48(m, PYRO_DOWN_OF(j, m))) - 48;
            down += __popc(m);
        }
        const int64_t B = block_sum<int64_t>(bsum, red);
        const int64_t D = block_sum<int64_t>(down, red);
        if (tid == 0) d.ring[st.e_pending] = ising_record(d, st.t - 1, B, D);
    }
    for (int s = 0; s < st.remaining; ++s) {
        const uint32_t t = st.t + (uint32_t)s;
        // 1. activation; up tetrahedra seed the forest
        uint64_t act[kCellsPerThread];
#pragma unroll
        for (int j = 0; j < kCellsPerThread; ++j) {
            const int c0 = tid + j * NT;
            act[j] = 0;
            if (c0 < ncell) {
                const uint32_t m = SMK[c0];
                act[j] = ising_activate(aligned48(m, PYRO_DOWN_OF(j, m)), (uint32_t)c0, t, d.key, prm);
#pragma unroll
                for (int f = 0; f < 4; ++f) {
                    const uint32_t code = K4[(uint32_t)(act[j] >> (6 * f)) & 63u];
                    const uint32_t base = 16u * (uint32_t)c0 + 4u * f;
#pragma unroll
                    for (int mu = 0; mu < 4; ++mu) PF[base + mu] = (uint16_t)(base + ((code >> (2 * mu)) & 3u));
                }
            }
        }
        __syncthreads();
        // 2. down tetrahedra: spanning edges of their components
#pragma unroll
        for (int j = 0; j < kCellsPerThread; ++j) {
            const int c0 = tid + j * NT;
            if (c0 >= ncell) continue;
#pragma unroll
            for (int f = 0; f < 4; ++f) {
                const uint32_t code = K4[(uint32_t)(act[j] >> (24 + 6 * f)) & 63u];
                if (code == 0xE4u) continue;  // four single vertices
                uint32_t v[4];
#pragma unroll
                for (int mu = 0; mu < 4; ++mu) {
                    const SiteRef R = down_vertex(f, mu);
                    v[mu] = 16u * (uint32_t)(R.cell == kSelf ? c0 : nbc[j][R.cell]) + R.site;
                }
#pragma unroll
                for (int mu = 1; mu < 4; ++mu) {
                    const uint32_t rp = (code >> (2 * mu)) & 3u;
                    if (rp != (uint32_t)mu) unite16(PF, v[rp], v[mu]);
                }
            }
        }
        // 3. coins of the sweep
        for (int g = tid; g < (N + 127) / 128; g += NT) {
            const uint4 w = philox4x32_10((uint32_t)g, t, kStreamFlip, 0u, d.key);
            CW[4 * g] = w.x;
            if (4 * g + 1 < (N + 31) / 32) CW[4 * g + 1] = w.y;
            if (4 * g + 2 < (N + 31) / 32) CW[4 * g + 2] = w.z;
            if (4 * g + 3 < (N + 31) / 32) CW[4 * g + 3] = w.w;
        }
        __syncthreads();
        // 4. roots, coins and flips (labels after the last sweep)
        const bool last = s + 1 == st.remaining;
        uint32_t nm[kCellsPerThread];
#pragma unroll
        for (int j = 0; j < kCellsPerThread; ++j) {
            const int c0 = tid + j * NT;
            nm[j] = 0;
            if (c0 >= ncell) continue;
            uint32_t flip = 0, last_r = 0xFFFFFFFFu, last_coin = 0;
            for (int k = 0; k < 16; ++k) {
                const uint32_t r = find16(PF, 16u * (uint32_t)c0 + k);
                if (r != last_r) {
                    last_r = r;
                    last_coin = (CW[r >> 5] >> (r & 31u)) & 1u;
                }
                flip |= last_coin << k;
                if (last) d.label[16 * c0 + k] = (int)r;
            }
            nm[j] = SMK[c0] ^ flip;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kCellsPerThread; ++j)
            if (tid + j * NT < ncell) SMK[tid + j * NT] = (uint16_t)nm[j];
        __syncthreads();
        // 5. moments of the new state
        int64_t bsum = 0, down = 0;
#pragma unroll
        for (int j = 0; j < kCellsPerThread; ++j) {
            const int c0 = tid + j * NT;
            if (c0 >= ncell) continue;
            bsum += 2 * (int64_t)__popcll(aligned48(nm[j], PYRO_DOWN_OF(j, nm[j]))) - 48;
            down += __popc(nm[j]);
        }
        const int64_t B = block_sum<int64_t>(bsum, red);
        const int64_t D = block_sum<int64_t>(down, red);
        if (tid == 0) {
            const int slot = st.ring_used + s;
            if (slot < d.ring_cap) d.ring[slot] = ising_record(d, t, B, D);
        }
    }
#undef PYRO_DOWN_OF
    // spins back to HBM (+1 = 0x01, -1 = 0xFF)
#pragma unroll
    for (int j = 0; j < kCellsPerThread; ++j) {
        const int c0 = tid + j * NT;
        if (c0 >= ncell) continue;
        reinterpret_cast<int4 *>(d.spins)[c0] = mask_spins(SMK[c0]);
    }
    if (tid == 0) {
        RepState ns;
        ns.t = st.t + (uint32_t)st.remaining;
        ns.remaining = 0;
        ns.ring_used = st.ring_used + st.remaining;
        ns.e_pending = -1;
        *c.state[rep] = ns;
    }
}

// -------------------------------------------------------- quad kernel ---
// The same sweeps with four threads per cell, thread f = 0..3 owning the up
// tetrahedron f of the cell (sites 4 f .. 4 f + 3) and the down tetrahedron
// f, up to kQuadMaxL with a 32-bit forest.  One workgroup on one compute unit
// is bound by the latency of its dependent steps, so each thread's chains are
// short: one Philox block (threads 0..2 of the quad; the flags are shared by
// DPP), 4 forest entries, at most 3 unions, 4 root walks side by side.  The
// unions are balanced over each wave as in the tile pass.  Three barriers a
// sweep:
//   A  activation; the up tetrahedra seed the forest; bonds whose top byte
//      ties are listed; the sweep's coins; aligned bonds of the incoming state
//      (the energy of the previous record)
//   B  unions of the down tetrahedra, then of the tied bonds, each a union of
//      its own when its low draw activates it; the previous record
//   C  root, coin and flip of every site; the magnetisation of the new state
// Per sweep of a long call L = 8 takes 11 us and L = 12 34 us; with one cell per
// thread and seven barriers (k_resident_ising) they took 23 and 48 us.
namespace {

template <int CTRL>
__device__ __forceinline__ uint32_t quad_perm(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}

// Sum over the wave, valid in its lane 0.
__device__ __forceinline__ int wave_sum(int v)
{
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_down(v, off, kWave);
    return v;
}

}  // namespace

template <int PASSES>
__global__ __launch_bounds__(kResidentThreads) void k_quad_ising(Chain c, RepState armed, bool use_armed)
{
    extern __shared__ __align__(16) char lds[];
    const int rep = blockIdx.x;
    const RepState st = use_armed ? armed : *c.state[rep];
    if (st.remaining <= 0) return;
    const RepDesc &d = c.desc[rep];
    const int L = d.L, ncell = (int)d.ncell, N = (int)d.N;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, f = tid & 3;
    constexpr int NT = kResidentThreads;
    const QuadLayout ly = quad_layout(L);
    uint32_t *P = (uint32_t *)(lds + ly.p);
    lds_byte *base = (lds_byte *)lds;
    __attribute__((address_space(3))) int *sums = (__attribute__((address_space(3))) int *)(base + ly.sums);
    __attribute__((address_space(3))) int *ties_n = (__attribute__((address_space(3))) int *)(base + ly.ties_n);
    lds_word *CW = (lds_word *)(base + ly.cw);
    lds_word *W = (lds_word *)(base + ly.un + 512 * wave);
    lds_word *TI = (lds_word *)(base + ly.ties);
    __attribute__((address_space(3))) volatile uint16_t *SMK = (__attribute__((address_space(3))) volatile uint16_t *)(base + ly.smk);
    __attribute__((address_space(3))) volatile uint8_t *K4 = (__attribute__((address_space(3))) volatile uint8_t *)(base + ly.k4);

    if (tid < 64) {
        constexpr K4Table k4 = make_k4();
        K4[tid] = k4.v[tid];
    }
    if (tid < 6) sums[tid] = 0;
    if (tid < 2) ties_n[tid] = 0;
    // Sites of the thread's down tetrahedra, 16 bits each.
    uint32_t v01[PASSES], v23[PASSES];
    int down = 0;  // down spins of the thread's sites in the incoming state
#pragma unroll
    for (int j = 0; j < PASSES; ++j) {
        const int cell = (tid + j * NT) >> 2;
        v01[j] = v23[j] = 0;
        if (cell >= ncell) continue;
        const CellNbrs nb = cell_neighbours(cell, L);
        const int c1 = f == 0 ? nb.c[kMyMz] : f == 1 ? cell : f == 2 ? nb.c[kMy] : nb.c[kMz];
        const int c2 = f == 0 ? nb.c[kMxMz] : f == 1 ? nb.c[kMx] : f == 2 ? cell : nb.c[kMz];
        const int c3 = f == 0 ? nb.c[kMxMy] : f == 1 ? nb.c[kMx] : f == 2 ? nb.c[kMy] : cell;
        // vertex mu of tetrahedron f is site 4 (f xor mu) + mu of its cell
        v01[j] = (uint32_t)(16 * cell + 4 * f) | (uint32_t)(16 * c1 + 4 * (f ^ 1) + 1) << 16;
        v23[j] = (uint32_t)(16 * c2 + 4 * (f ^ 2) + 2) | (uint32_t)(16 * c3 + 4 * (f ^ 3) + 3) << 16;
        const uint32_t m = spin_mask16(reinterpret_cast<const int4 *>(d.spins)[cell]);
        if (f == 0) SMK[cell] = (uint16_t)m;
        down += __popc((m >> (4 * f)) & 15u);
    }
    __syncthreads();
    // Spins of the thread's up (bits 0..3) and down (4..7) tetrahedra.
    auto vertex_spins = [&](int j) {
        auto bit = [&](uint32_t v) { return ((uint32_t)SMK[v >> 4] >> (v & 15u)) & 1u; };
        const uint32_t a = v01[j] & 0xFFFFu, b = v01[j] >> 16, e = v23[j] & 0xFFFFu, g = v23[j] >> 16;
        const uint32_t m = SMK[a >> 4];
        return ((m >> (4 * f)) & 15u) | ((m >> (4 * f)) & 1u) << 4 | bit(b) << 5 | bit(e) << 6 | bit(g) << 7;
    };
    const uint32_t C = d.thr_hi * 0x01010101u;  // all parallel bonds are active from 256 on
    const bool all = d.thr_hi >= 256u;
    int cur = 0;  // set of sums that the state entering the sweep fills
    for (int s = 0;; ++s) {
        const bool end = s == st.remaining;  // only the sums of the last state remain
        const uint32_t t = st.t + (uint32_t)s;
        int aligned_n = 0;
        uint8_t code[PASSES];
#pragma unroll
        for (int j = 0; j < PASSES; ++j) {
            const int cell = (tid + j * NT) >> 2;
            code[j] = 0xE4;
            const bool valid = cell < ncell;
            uint32_t al = 0;  // aligned bonds: up tetrahedron in bits 0..5, down in 6..11
            if (valid) {
                const uint32_t sp = vertex_spins(j);
                al = (anti6(sp & 15u) | anti6(sp >> 4) << 6) ^ 0xFFFu;
            }
            aligned_n += __popc(al);
            if (end) continue;
            // Flags of the cell's 48 top bytes: thread q < 3 of the quad draws
            // block q; every thread takes its 12 bits.
            uint32_t act = al, tie = 0;
            if (!all) {
                const uint4 r = philox4x32_10(3u * (uint32_t)cell + (uint32_t)min(f, 2), t, kStreamBond, 0u, d.key);
                const uint32_t lt = gather_flags16(bytes_lt(r.x, C), bytes_lt(r.y, C), bytes_lt(r.z, C), bytes_lt(r.w, C));
                const uint32_t eq = gather_flags16(bytes_eq(r.x, C), bytes_eq(r.y, C), bytes_eq(r.z, C), bytes_eq(r.w, C));
                const uint32_t w = lt | eq << 16;
                const uint32_t w0 = quad_perm<0x00>(w), w1 = quad_perm<0x55>(w), w2 = quad_perm<0xAA>(w);
                const uint64_t acc = (uint64_t)((w0 & 0xFFFFu) | w1 << 16) | (uint64_t)(w2 & 0xFFFFu) << 32;
                const uint64_t eqs = (uint64_t)(w0 >> 16 | (w1 & 0xFFFF0000u)) | (uint64_t)(w2 >> 16) << 32;
                act = al & ((uint32_t)(acc >> (6 * f) & 63u) | (uint32_t)(acc >> (24 + 6 * f) & 63u) << 6);
                tie = al & ((uint32_t)(eqs >> (6 * f) & 63u) | (uint32_t)(eqs >> (24 + 6 * f) & 63u) << 6);
            }
            if (!valid) continue;
            while (tie) {
                const int k = __ffs((int)tie) - 1;
                tie &= tie - 1;
                const int e = k < 6 ? k : k - 6, a = pair_a(e), b = pair_b(e);
                const uint32_t bond = 48u * (uint32_t)cell + 6u * (uint32_t)(k < 6 ? f : 4 + f) + (uint32_t)e;
                auto vert = [&](int mu) {
                    const uint32_t w = mu < 2 ? v01[j] : v23[j];
                    return k < 6 ? (uint32_t)(16 * cell + 4 * f + mu) : ((mu & 1) ? w >> 16 : w & 0xFFFFu);
                };
                const int i = __hip_atomic_fetch_add(&ties_n[s & 1], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                if (i < kQuadTies) {
                    TI[2 * i] = bond;
                    TI[2 * i + 1] = vert(a) << 16 | vert(b);
                } else {  // beyond the list: decided here
                    const uint4 lo = philox4x32_10(bond >> 2, t, kStreamBondLo, 0u, d.key);
                    if ((word_of(lo, bond & 3u) & 0xFFFFFFu) < d.thr_lo) act |= 1u << k;
                }
            }
            const uint32_t up = K4[act & 63u], b0 = 4u * (uint32_t)(16 * cell + 4 * f);
            code[j] = K4[act >> 6];
#pragma unroll
            for (int mu = 0; mu < 4; ++mu) node(P, b0 + 4 * mu) = b0 + 4 * ((up >> (2 * mu)) & 3u);
        }
        if (!end)
            for (int g = tid; g < (N + 127) / 128; g += NT) {
                const uint4 w = philox4x32_10((uint32_t)g, t, kStreamFlip, 0u, d.key);
                CW[4 * g] = w.x;
                CW[4 * g + 1] = w.y;
                CW[4 * g + 2] = w.z;
                CW[4 * g + 3] = w.w;
            }
        {
            const int a = wave_sum(aligned_n), m = wave_sum(down);
            if (lane == 0) {
                __hip_atomic_fetch_add(&sums[2 * cur], m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                __hip_atomic_fetch_add(&sums[2 * cur + 1], a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
        __syncthreads();
        // The record of the state entering the sweep (of a tiled sweep before
        // this call when s = 0); the third set of sums is cleared for the next.
        const int next = cur == 2 ? 0 : cur + 1, clear = next == 2 ? 0 : next + 1;
        if (tid == NT - 1) {
            const int slot = s == 0 ? st.e_pending : st.ring_used + s - 1;
            if (slot >= 0 && slot < d.ring_cap)
                d.ring[slot] = ising_record(d, t - 1, 2 * (int64_t)sums[2 * cur + 1] - 3 * (int64_t)N, sums[2 * cur]);
            sums[2 * clear] = 0;
            sums[2 * clear + 1] = 0;
            ties_n[(s + 1) & 1] = 0;
        }
        if (end) break;
        // Unions, balanced over the wave (see tile_components).
        int n = 0;
        auto unite_row = [&](int m) {
            wave_sync();
            if (lane < m) {
                const uint32_t u = W[lane];
                lds_unite(P, (u >> 14) & ~3u, (u & 0xFFFFu) << 2);
            }
        };
#pragma unroll
        for (int j = 0; j < PASSES; ++j) {
#pragma unroll
            for (int mu = 1; mu < 4; ++mu) {
                const uint32_t rp = ((uint32_t)code[j] >> (2 * mu)) & 3u;
                const uint32_t kr = rp == 0 ? v01[j] & 0xFFFFu : (rp == 1 ? v01[j] >> 16 : v23[j] & 0xFFFFu);
                const uint32_t km = mu == 1 ? v01[j] >> 16 : (mu == 2 ? v23[j] & 0xFFFFu : v23[j] >> 16);
                const bool use = rp != (uint32_t)mu;
                const uint64_t b = __ballot(use);
                const int at = n + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
                if (use) W[at] = kr << 16 | km;
                n += (int)__popcll(b);
                if (n >= 64) {
                    unite_row(64);
                    const uint32_t rest = W[64 + lane];
                    wave_sync();
                    W[lane] = rest;
                    wave_sync();
                    n -= 64;
                }
            }
        }
        unite_row(n);
        const int nt = min((int)ties_n[s & 1], kQuadTies);
        for (int i = tid; i < nt; i += NT) {
            const uint32_t bond = TI[2 * i], u = TI[2 * i + 1];
            const uint4 lo = philox4x32_10(bond >> 2, t, kStreamBondLo, 0u, d.key);
            if ((word_of(lo, bond & 3u) & 0xFFFFFFu) < d.thr_lo) lds_unite(P, (u >> 14) & ~3u, (u & 0xFFFFu) << 2);
        }
        __syncthreads();
        const bool last = s + 1 == st.remaining;
        down = 0;
#pragma unroll
        for (int j = 0; j < PASSES; ++j) {
            const int cell = (tid + j * NT) >> 2;
            uint32_t fl = 0, m = 0;
            if (cell < ncell) {
                const uint32_t b0 = 4u * (uint32_t)(16 * cell + 4 * f);
                uint32_t r[4], moved;
#pragma unroll
                for (int k = 0; k < 4; ++k) r[k] = node(P, b0 + 4 * k);
                do {
                    moved = 0;
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const uint32_t p = node(P, r[k]);
                        moved |= p ^ r[k];
                        r[k] = p;
                    }
                } while (moved);
#pragma unroll
                for (int k = 0; k < 4; ++k) fl |= __builtin_amdgcn_ubfe(CW[r[k] >> 7], (r[k] >> 2) & 31u, 1u) << k;
                if (last)
                    reinterpret_cast<int4 *>(d.label)[4 * cell + f] =
                        make_int4((int)(r[0] >> 2), (int)(r[1] >> 2), (int)(r[2] >> 2), (int)(r[3] >> 2));
                m = SMK[cell];
            }
            uint32_t w = fl << (4 * f);
            w |= quad_perm<0xB1>(w);  // threads 1, 0, 3, 2
            w |= quad_perm<0x4E>(w);  // threads 2, 3, 0, 1
            m ^= w;
            if (cell < ncell) {
                down += __popc((m >> (4 * f)) & 15u);
                if (f == 0) SMK[cell] = (uint16_t)m;
                if (last && f == 0) reinterpret_cast<int4 *>(d.spins)[cell] = mask_spins(m);
            }
        }
        __syncthreads();
        cur = next;
    }
    if (tid == 0) c.state[rep][0] = RepState{st.t + (uint32_t)st.remaining, 0, st.ring_used + st.remaining, -1};
}

// Threads of the quad kernel's instances cover that many tetrahedra each.
static int quad_passes(int maxL)
{
    const int p = (4 * maxL * maxL * maxL + kResidentThreads - 1) / kResidentThreads;
    return p <= 1 ? 1 : p <= 2 ? 2 : p <= 4 ? 4 : p <= 7 ? 7 : 9;
}

// Let a kernel take as much dynamic LDS as it may need, on the current device.
static hipError_t allow_lds(const void *kernel, size_t bytes, DeviceOnce &done)
{
    int dev = -1;
    const hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    return done.run(dev, [&] { return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes); });
}

template <int PASSES>
static hipError_t allow_quad()
{
    static DeviceOnce done;
    return allow_lds((const void *)k_quad_ising<PASSES>, quad_layout(kQuadMaxL).total, done);
}

hipError_t prepare_resident(int maxL)
{
    if (maxL > kQuadMaxL) {
        static DeviceOnce done;
        return allow_lds((const void *)k_resident_ising, resident_layout(kResidentMaxL).total, done);
    }
    switch (quad_passes(maxL)) {
    case 1: return allow_quad<1>();
    case 2: return allow_quad<2>();
    case 4: return allow_quad<4>();
    case 7: return allow_quad<7>();
    default: return allow_quad<9>();
    }
}

template <int PASSES>
static void launch_quad(const Chain &c, int maxL, const RepState &from, bool armed, hipStream_t st)
{
    k_quad_ising<PASSES><<<c.nreps, kResidentThreads, quad_layout(maxL).total, st>>>(c, from, armed);
}

hipError_t launch_resident_ising(const Chain &c, int maxL, const RepState *armed, hipStream_t st, const LaunchHook &hook)
{
    if (c.nreps == 0) return hipSuccess;
    if (maxL < 1 || maxL > kResidentMaxL || (armed && c.nreps != 1)) return hipErrorInvalidValue;
    const hipError_t e = prepare_resident(maxL);
    if (e != hipSuccess) return e;
    const RepState from = armed ? *armed : RepState{};
    const bool use = armed != nullptr;
    if (hook.before) hook.before(hook.ctx, kKResident);
    if (maxL > kQuadMaxL) {
        k_resident_ising<<<c.nreps, kResidentThreads, resident_layout(maxL).total, st>>>(c, from, use);
    } else {
        switch (quad_passes(maxL)) {
        case 1: launch_quad<1>(c, maxL, from, use, st); break;
        case 2: launch_quad<2>(c, maxL, from, use, st); break;
        case 4: launch_quad<4>(c, maxL, from, use, st); break;
        case 7: launch_quad<7>(c, maxL, from, use, st); break;
        default: launch_quad<9>(c, maxL, from, use, st);
        }
    }
    if (hook.after) hook.after(hook.ctx, kKResident);
    return hipGetLastError();
}

}  // namespace pyro

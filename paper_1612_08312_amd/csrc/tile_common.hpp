// Tile machinery shared by the Ising and O(n) sweeps: the LDS cluster forest
// of one tile, tile indexing, and the merge of tile-crossing bonds into the
// global forest.
//
// A tile is a box of TX x TY x TZ cells handled by one workgroup (one thread
// per cell).  Tiles at the high end of an axis are ragged when the tile edge
// does not divide L; when L is smaller than the tile edge the tile spans the
// whole axis and its periodic bonds wrap onto itself.
//
// After the tile pass every site's label is its tile-local root (a global
// site index) and local roots point at themselves.  The merge unites local
// roots only, always hooking the larger root under the smaller one, so the
// entries of ordinary sites keep pointing at their local root and every
// final root is the smallest site index of its cluster.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device_util.hpp"
#include "kernels.hpp"
#include "lattice.hpp"

namespace pyro {

// The tile forest is keyed by the canonical local index key = 16 c + k (cell
// c of the tile, site k), whose order follows the global site order.  Node
// key sits at slot key + c = 17 c + k of the forest array: the slot order is
// the key order, and the 16 nodes of consecutive cells, which the lanes of a
// wave touch together, are 17 words apart and so never share an LDS bank.
// Each entry holds the byte offset (4 x slot) of its parent, so a step of a
// walk is one load with no index arithmetic.
template <int NC>
constexpr int kForestSlots = 17 * NC;

__device__ __forceinline__ uint32_t node_off(int key)
{
    return 4u * (uint32_t)(key + (key >> 4));
}

// Entry at byte offset off of the forest array, addressed in the LDS
// address space (a 32-bit offset, no generic-pointer arithmetic).
typedef __attribute__((address_space(3))) volatile uint32_t lds_word;
typedef __attribute__((address_space(3))) volatile char lds_byte;

__device__ __forceinline__ lds_word &node(volatile uint32_t *P, uint32_t off)
{
    return *(lds_word *)((lds_byte *)P + off);
}

// Every walk in the global forest below is capped far above any reachable
// depth (a forest over n nodes has depth below n), so a damaged forest can
// only give a wrong label, never a kernel that does not finish.
constexpr int kWalkCap = 1 << 22;

// In the tile forest a parent's offset is never above its child's (roots
// hold their own offset): initial parents are the smallest vertex of an up
// tetrahedron's component, unions lower a root to a smaller one, and path
// splitting stores ancestors.  Walks therefore step only while the parent is
// strictly smaller, which bounds them by the forest size whatever the
// entries hold.

// Root of node x (byte offsets), with path splitting.  The store is
// unconditional: x is not a root, and any ancestor is a valid parent.
__device__ __forceinline__ uint32_t lds_find(volatile uint32_t *P, uint32_t x)
{
    uint32_t p = node(P, x);
    while (p < x) {
        const uint32_t gp = node(P, p);
        node(P, x) = gp;
        x = p;
        p = gp;
    }
    return x;
}

// Union in an LDS forest: the larger root is lowered to the smaller one with
// atomicMin; if it had been re-parented meanwhile (to a smaller node),
// continue from there.  The larger root strictly decreases on every retry.
__device__ __forceinline__ void lds_unite(uint32_t *P, uint32_t a, uint32_t b)
{
    volatile uint32_t *V = P;
    for (;;) {
        a = lds_find(V, a);
        b = lds_find(V, b);
        if (a == b) return;
        if (a < b) {
            const uint32_t tmp = a;
            a = b;
            b = tmp;
        }
        const uint32_t old = __hip_atomic_fetch_min((__attribute__((address_space(3))) uint32_t *)((lds_byte *)P + a), b,
                                                    __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (old >= a) return;
        a = old;
    }
}

// Label staging of the flip kernels: the label of local key 16 c + k is kept
// at k * NC + c, so the lanes of a wave, which own consecutive cells, touch
// consecutive LDS banks.
template <int NC>
__device__ __forceinline__ int lds_pos(int key)
{
    return (int)(((unsigned)key & 15u) * NC + ((unsigned)key >> 4));
}

// Quotient a / b for 0 <= a < 2^24 and b >= 1 with a small quotient: a
// float reciprocal gives it to within one, an integer check corrects it.
__device__ __forceinline__ int small_div(int a, int b, float inv_b)
{
    int q = (int)((float)a * inv_b);
    if (mul24(q, b) > a) --q;
    else if (mul24(q + 1, b) <= a) ++q;
    return q;
}

template <int TX, int TY, int TZ>
struct TileIdx {
    int L, bx, by, bz;
    int base;            // global index of the tile's first cell
    float inv_L, inv_LL; // 1/L and 1/L^2

    __device__ __forceinline__ static TileIdx of(int tile, const RepDesc &d)
    {
        TileIdx t;
        t.L = d.L;
        t.bx = tile % d.ntx;
        tile /= d.ntx;
        t.by = tile % d.nty;
        t.bz = tile / d.nty;
        t.base = ((t.bz * TZ) * t.L + t.by * TY) * t.L + t.bx * TX;
        t.inv_L = 1.0f / (float)t.L;
        t.inv_LL = 1.0f / (float)(t.L * t.L);
        return t;
    }
    // Global site index of local key l = 16 c + k.
    __device__ __forceinline__ int global_site(int l) const
    {
        const unsigned lc = (unsigned)l >> 4;  // keys are non-negative; unsigned keeps % and / to masks and shifts
        const int lx = (int)(lc % TX), ly = (int)((lc / TX) % TY), lz = (int)(lc / (TX * TY));
        return 16 * (base + cell_index(lx, ly, lz, L)) + (l & 15);
    }
    // Local key 16 c + k of a global site index known to lie in this tile
    // (offsets from the tile's first cell are below TZ L^2 < 2^24).
    __device__ __forceinline__ int local_key(int site) const
    {
        const int off = (site >> 4) - base;
        const int LL = L * L;
        const int lz = small_div(off, LL, inv_LL);
        const int rem = off - mul24(lz, LL);
        const int ly = small_div(rem, L, inv_L);
        const int lx = rem - mul24(ly, L);
        return 16 * ((lz * TY + ly) * TX + lx) + (site & 15);
    }
    // Local key of a site of this tile from the thread's own cell (global
    // index `cell`, local index `lcell`): the cell offset dc = dz L^2 + dy L
    // + dx has |dx| < TX, |dy| < TY, |dz| < TZ, so when L >= 2 max(TX, TY,
    // TZ) (near_decodable) dz and dy are the nearest integers of dc / L^2 and
    // of the remainder / L (each more than 0.03 away from a half-integer).
    __device__ __forceinline__ bool near_decodable() const { return L >= 2 * (TX > TY ? (TX > TZ ? TX : TZ) : (TY > TZ ? TY : TZ)); }
    __device__ __forceinline__ int local_key_near(int site, int cell, int lcell) const
    {
        const int dc = (site >> 4) - cell;
        const int dz = (int)rintf((float)dc * inv_LL);
        const int r1 = dc - __mul24(dz, L * L);
        const int dy = (int)rintf((float)r1 * inv_L);
        const int dx = r1 - __mul24(dy, L);
        return 16 * (lcell + dx + dy * TX + dz * (TX * TY)) + (site & 15);
    }
    // Local indices of the seven cells the bonds of local cell (lx, ly, lz)
    // touch, -1 outside the tile.  Only an axis with a single tile wraps onto
    // the tile itself, whose last cell on it is its extent less one.
    __device__ __forceinline__ void local_neighbours(const RepDesc &d, int lx, int ly, int lz, int lcell,
                                                     int (&lc)[kNCellCodes]) const
    {
        const bool ix = lx > 0 || d.ntx == 1, iy = ly > 0 || d.nty == 1, iz = lz > 0 || d.ntz == 1;
        const int sx = lx > 0 ? -1 : min(TX, L) - 1, sy = ly > 0 ? -TX : (min(TY, L) - 1) * TX,
                  sz = lz > 0 ? -TX * TY : (min(TZ, L) - 1) * (TX * TY);
        lc[kSelf] = lcell;
        lc[kMx] = ix ? lcell + sx : -1;
        lc[kMy] = iy ? lcell + sy : -1;
        lc[kMz] = iz ? lcell + sz : -1;
        lc[kMyMz] = iy && iz ? lcell + sy + sz : -1;
        lc[kMxMz] = ix && iz ? lcell + sx + sz : -1;
        lc[kMxMy] = ix && iy ? lcell + sx + sy : -1;
    }
    // Global indices of those cells (periodic wrap), the cell itself at (x, y, z).
    __device__ __forceinline__ void global_neighbours(int x, int y, int z, int cell, int (&gc)[kNCellCodes]) const
    {
        const int sx = x == 0 ? L - 1 : -1, sy = y == 0 ? L * (L - 1) : -L, sz = z == 0 ? L * L * (L - 1) : -L * L;
        gc[kSelf] = cell;
        gc[kMx] = cell + sx;
        gc[kMy] = cell + sy;
        gc[kMz] = cell + sz;
        gc[kMyMz] = cell + sy + sz;
        gc[kMxMz] = cell + sx + sz;
        gc[kMxMy] = cell + sx + sy;
    }
};

// ---------------------------------------------------------------- merge ---
// The global forest lives in the label entries of tile-local roots (the
// entries of ordinary sites keep pointing at their local root).  Entry
// encodings of a local root r:
//   r                   r is a root of the merged forest
//   kTag | p            r was hooked under p
//   kCanonBase + c (| kCoinBit)  written by the settle step of the flip
//                       kernels (or the persistent kernel's store phase): c is
//                       the smallest site index of r's cluster, and kCoinBit
//                       is set when that cluster flips in this sweep
// Site indices are below 2^30 (L <= 406), so the three forms are distinct and
// the local root of any site is decodable at any time, even while other
// threads hook roots or store canonical labels: an entry that is negative,
// tagged or equal to the site's own index names the site itself.
//
// A root is always hooked under the smaller of the two roots, so every tree
// root is the smallest local root of its tree, i.e. the smallest site of
// its cluster, and settling a hooked local root only has to copy it (with
// its coin) into the root's entry.  The unite pass hooks each tile's group
// of roots under its smallest member in one step, which keeps the trees
// shallow.
constexpr int kTag = 1 << 30;
constexpr int kIdxMask = kTag - 1;
constexpr int kCanonBase = INT32_MIN;  // canonical index c is stored as kCanonBase + c
constexpr int kCoinBit = 1 << 30;      // flip coin of the cluster, in a stored encoding

// Flip coin of the cluster whose smallest site is r in sweep t: bit (r mod
// 32) of word ((r/32) mod 4) of FLIP(r/128).
__device__ __forceinline__ uint32_t cluster_coin(int r, uint32_t t, PhiloxKey key)
{
    const uint4 w = philox4x32_10((uint32_t)r >> 7, t, kStreamFlip, 0u, key);
    return (word_of(w, ((uint32_t)r >> 5) & 3u) >> (r & 31)) & 1u;
}

// The coins of the 16 sites of a cell (bit k = site 16 cell + k) in sweep t:
// sites of one cell are 16 consecutive bits of one word of FLIP(cell/8).
__device__ __forceinline__ uint32_t cell_coins(int cell, uint32_t t, PhiloxKey key)
{
    const uint4 w = philox4x32_10((uint32_t)cell >> 3, t, kStreamFlip, 0u, key);
    return (word_of(w, ((uint32_t)cell >> 1) & 3u) >> (16 * (cell & 1))) & 0xFFFFu;
}

// Forest entries are read and written with relaxed workgroup-scope atomics,
// which the caches may serve stale within a launch (agent-scope loads would
// go past the per-XCD L2 on every step of every walk).  A stale value is an
// older value of the same entry, and every value an entry ever holds is an
// ancestor of the node in the final forest (hooks link roots, shortcuts
// store ancestors, the settle step writes only encodings that end a walk),
// so a stale walk is only longer, never wrong; the updates that decide the
// forest (hook CAS) are device-wide atomics and return the current value.  Launch boundaries make all writes visible.
__device__ __forceinline__ int lab_load(const int32_t *lab, int x)
{
    return __hip_atomic_load(lab + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ void lab_store(int32_t *lab, int x, int v)
{
    __hip_atomic_store(lab + x, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The same store written through to memory, where the compare-and-swaps of
// other compute units act: an entry left dirty in this XCD's L2 beside entries
// they swap costs more than the store saves (unite pass over five L = 128
// lattices: 476 us with compare-and-swaps only, 527 with plain stores for the
// lone roots, 441 with these; one lattice 108, 104 and 84).
__device__ __forceinline__ void lab_store_through(int32_t *lab, int x, int v)
{
    __hip_atomic_store(lab + x, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Root of local root x in the forest while hooking runs (shortcuts store
// tagged grandparents, which are ancestors).
__device__ __forceinline__ int forest_find(int32_t *lab, int x)
{
    for (int it = 0; it < kWalkCap; ++it) {
        const int v = lab_load(lab, x);
        if (v == x) return x;
        const int p = v & kIdxMask;
        const int w = lab_load(lab, p);
        if (w != p) lab_store(lab, x, w);
        x = p;
    }
    return x;
}

// Union of the trees of local roots a and b.  Every parent is smaller than
// its child (hooks put the larger root under a smaller node, shortcuts store
// ancestors), so a root may be hooked under any node smaller than itself:
// that node cannot lie in the root's own tree.  Hence a's root is walked
// first and, when it is larger than b, hooked under b by CAS without walking
// b; otherwise b's root is walked and the larger of the two roots is hooked
// under the smaller.  A lost CAS continues from the value it returned.
template <bool COUNT = false>
__device__ __forceinline__ void forest_unite(int32_t *lab, int a, int b, unsigned long long *counts)
{
    for (int it = 0; it < kWalkCap; ++it) {
        a = forest_find(lab, a);
        if (a == b) return;
        if (a < b) {
            b = forest_find(lab, b);
            if (a == b) return;
            if (a < b) {
                const int tmp = a;
                a = b;
                b = tmp;
            }
        }
        const int old = atomicCAS(lab + a, a, kTag | b);
        if (COUNT) {  // measurement runs only (a kernel of its own)
            atomicAdd(&counts[0], 1ull);
            if (old == a) atomicAdd(&counts[1], 1ull);
        }
        if (old == a) return;
        a = old & kIdxMask;
    }
}

// Tree root of local root x after the unite pass, or the first encoding a
// settle step has already written on the way (a negative value).  The tree
// root's index is the cluster's smallest site.
__device__ __forceinline__ int root_or_encoding(const int32_t *lab, int x)
{
    for (int it = 0; it < kWalkCap; ++it) {
        const int v = lab_load(lab, x);
        if (v < 0 || v == x) return v;
        x = v & kIdxMask;
    }
    return x;
}

// Encoding stored for the cluster of local root x in sweep t: its smallest
// site and its flip coin.
__device__ __forceinline__ int canon_encoding(const int32_t *lab, int x, uint32_t t, PhiloxKey key)
{
    const int v = root_or_encoding(lab, x);
    if (v < 0) return v;
    return kCanonBase + v + (int)(cluster_coin(v, t, key) << 30);
}

// Canonical label (smallest site index of the cluster) of any site once the
// sweep is done: site -> local root -> itself (a tree root) or its settled
// encoding (a walk from a still-hooked local root is kept as a safeguard).
__device__ __forceinline__ int canonical_label(const int32_t *label, int64_t i)
{
    const int v = label[i];
    if (v < 0) return v & kIdxMask;
    const int r = (v & kTag) ? (int)i : v;
    const int w = label[r];
    if (w < 0) return w & kIdxMask;
    if (w & kTag) {
        const int e = root_or_encoding(label, r);
        return e < 0 ? (e & kIdxMask) : e;
    }
    return r;
}

// Flip mask (bit k = site k) of the cell of a flip kernel's thread, from the
// labels of its 16 sites (lab), the tile's labels staged in LDS (LAB, laid
// out by lds_pos) and the coins of the tile's own sites (CB, one 16-bit word
// per cell).  A site's label is its tile-local root r; r's entry holds the
// stored encoding (canonical site and coin) when r's cluster leaves the tile,
// else r itself, whose coin is the tile's.  Only LDS is read.
template <int NC, int TX, int TY, int TZ>
__device__ __forceinline__ uint32_t cell_flip_mask(const int (&lab)[16], const int *LAB, const uint32_t *CB,
                                                  const TileIdx<TX, TY, TZ> &ti, int cell, int lcell, uint32_t t,
                                                  PhiloxKey key)
{
    const bool near = ti.near_decodable();  // uniform
    int last_in = -1;
    uint32_t last_coin = 0, mask = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const int r0 = lab[k];  // tile-local root, or an encoding (the site is a merged local root)
        uint32_t coin;
        if (r0 < 0) {
            coin = ((uint32_t)r0 >> 30) & 1u;
        } else if (r0 & kTag) {
            coin = cluster_coin(r0 & kIdxMask, t, key);  // not produced by a complete sweep; kept in range
        } else if (r0 == last_in) {
            coin = last_coin;
        } else {
            const int key16 = near ? ti.local_key_near(r0, cell, lcell) : ti.local_key(r0);
            const int v = LAB[lds_pos<NC>(key16)];
            if (v < 0) coin = ((uint32_t)v >> 30) & 1u;
            else if (v & kTag) coin = cluster_coin(v & kIdxMask, t, key);  // as above
            else coin = (CB[key16 >> 4] >> (key16 & 15)) & 1u;
            last_in = r0;
            last_coin = coin;
        }
        mask |= coin << k;
    }
    return mask;
}

constexpr int const_log2(int v) { return v <= 1 ? 0 : 1 + const_log2(v >> 1); }

// Aligned tiling: the lattice edge is L = 2^lg and every tile edge divides
// it, so each tile starts at a multiple of its edges and a site index
// 16 (x + L y + L^2 z) + k of the tile has its local cell coordinates in
// fixed bit fields.  The local key 16 (lx + TX ly + TX TY lz) + k is then
// a few bit-field extracts, whatever value is decoded (an encoding yields
// some key of the tile, never one outside it).
template <int TX, int TY, int TZ>
__device__ __forceinline__ int aligned_local_key(int site, int lg)
{
    constexpr int lTX = const_log2(TX), lTY = const_log2(TY);
    const uint32_t u = (uint32_t)site;
    const uint32_t ly = __builtin_amdgcn_ubfe(u, (uint32_t)(4 + lg), (uint32_t)const_log2(TY));
    const uint32_t lz = __builtin_amdgcn_ubfe(u, (uint32_t)(4 + 2 * lg), (uint32_t)const_log2(TZ));
    return (int)((u & (16u * TX - 1u)) | (ly << (4 + lTX)) | (lz << (4 + lTX + lTY)));
}

// How a flip kernel finds a site's local root in its tile: kFlipGeneral
// stages the labels at lds_pos and decodes with branches (cell_flip_mask);
// the keyed modes stage them by local key and decode without a branch, for
// tilings whose tile edges divide L (every thread has a cell, TX >= 8): by
// bit fields when L is a power of two (kFlipPow2, aligned_local_key), else
// by rounding the cell offset (kFlipDivisible, TileIdx::local_key_near,
// exact for L >= 2 x the largest tile edge).
enum FlipMode : int { kFlipGeneral = 0, kFlipPow2 = 1, kFlipDivisible = 2 };

// Flip mask of a flip kernel's cell for a keyed mode.  LAB holds the
// tile's labels by local key; CB holds the coin words of the tile's cells,
// two cells per word as the flip stream draws them (bit (key & 31) of word
// key >> 5 is the coin of local key `key`).  The same rule as
// cell_flip_mask: a stored encoding, in the site's own entry or in its
// local root's, gives the coin; otherwise the local root's own coin.  No
// branch: both LDS words are read for every site, and the key decoded from
// an encoding, which is not used, is masked into the tile's key range.
template <int TX, int TY, int TZ, int MODE>
__device__ __forceinline__ uint32_t cell_flip_mask_keyed(const int (&lab)[16], const int *LAB, const uint32_t *CB,
                                                        int lg, const TileIdx<TX, TY, TZ> &ti, int cell, int lcell)
{
    constexpr int NC = TX * TY * TZ;
    static_assert(MODE == kFlipPow2 || MODE == kFlipDivisible, "a keyed mode");
    static_assert((NC & (NC - 1)) == 0, "tile keys fill a power of two");
    uint32_t mask = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const int r = lab[k];
        const int key = MODE == kFlipPow2 ? aligned_local_key<TX, TY, TZ>(r, lg)
                                          : (ti.local_key_near(r, cell, lcell) & (16 * NC - 1));
        const int u = r < 0 ? r : LAB[key];
        const bool enc = u < 0;
        const uint32_t word = enc ? (uint32_t)u : CB[key >> 5];
        mask |= __builtin_amdgcn_ubfe(word, enc ? 30u : (uint32_t)key & 31u, 1u) << k;
    }
    return mask;
}

// Coin words of a keyed tile (NC / 8 threads, thread j): local cells
// 8j .. 8j + 7 are eight consecutive cells of one x row starting at a
// multiple of 8 (TX >= 8), i.e. exactly the cells of one FLIP block, whose
// four words cover two cells each (cell_coins).
template <int TX, int TY, int TZ>
__device__ __forceinline__ uint4 aligned_coin_words(const TileIdx<TX, TY, TZ> &ti, int j, uint32_t t, PhiloxKey key)
{
    static_assert(TX % 8 == 0, "a FLIP block is 8 cells of one x row");
    const int c0 = 8 * j;
    const int gcell = cell_index(ti.bx * TX + c0 % TX, ti.by * TY + (c0 / TX) % TY, ti.bz * TZ + c0 / (TX * TY), ti.L);
    return philox4x32_10((uint32_t)gcell >> 3, t, kStreamFlip, 0u, key);
}

// ------------------------------------------------------- settle step ---
// The flip kernels settle their tile's own hooked local roots (entries
// kTag | p) once every unite is done: the walk from p ends at the
// cluster's tree root, its smallest site, or at an encoding that another
// settle wrote on the way, and the root's entry becomes the stored encoding
// (smallest site and coin) in the label array, for later walks and the
// host's labels, and in the LDS copy of the tile's labels.  A local root
// that is a tree root keeps its own index: its cluster's coin is the
// tile's own coin of that site (the same bit of the same FLIP word).  Only
// a root's own tile settles it, so no other workgroup changes an entry a
// tile has staged.
constexpr int kSettleListPerCell = 4;  // list room per cell; roots beyond it settle in place

// Loads the 16 labels of a flip kernel's cell into lab and copies them into
// LAB (by local key in a keyed FlipMode, else at lds_pos).  Returns the
// mask of the sites that are hooked local roots; their lab value becomes
// the site's own index, so that the flip reads the site's settled entry.
template <int NC, bool ALIGNED>
__device__ __forceinline__ uint32_t stage_cell_labels(const int32_t *label, int cell, int tid, int (&lab)[16], int *LAB)
{
    const int4 *L4 = reinterpret_cast<const int4 *>(label + 16 * cell);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int4 v = L4[q];
        if (ALIGNED) reinterpret_cast<int4 *>(LAB)[4 * tid + q] = v;
        lab[4 * q] = v.x;
        lab[4 * q + 1] = v.y;
        lab[4 * q + 2] = v.z;
        lab[4 * q + 3] = v.w;
    }
    uint32_t hm = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        if (!ALIGNED) LAB[k * NC + tid] = lab[k];
        const bool hooked = ((uint32_t)lab[k] >> 30) == 1u;  // kTag | p
        hm |= (uint32_t)hooked << k;
        lab[k] = hooked ? 16 * cell + k : lab[k];
    }
    return hm;
}

// The settle step of a flip kernel (all NC threads of the tile, after
// stage_cell_labels; hm is the thread's mask, 0 for a thread without a
// cell).  The hooked roots are listed in HL (kSettleListPerCell NC
// entries; the list places follow the threads' counts, by five ballots
// and the wave totals in wtot, NC / 64 ints) and settled by all threads.
template <int TX, int TY, int TZ, bool ALIGNED>
__device__ __forceinline__ void settle_tile_roots(const RepDesc &d, const RepState &st, const TileIdx<TX, TY, TZ> &ti,
                                                  int tid, int cell, uint32_t hm, int *LAB, uint16_t *HL, int *wtot)
{
    constexpr int NC = TX * TY * TZ;
    constexpr int kCapHL = kSettleListPerCell * NC;
    static_assert(16 * NC <= 65536, "local keys fit 16 bits");
    auto pos = [](int key) { return ALIGNED ? key : lds_pos<NC>(key); };
    const uint32_t cnt = (uint32_t)__popc(hm);
    uint32_t below = 0, wt = 0;
#pragma unroll
    for (int bit = 0; bit < 5; ++bit) {
        const uint64_t b = __ballot((cnt >> bit) & 1u);
        below += __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u)) << bit;
        wt += (uint32_t)__popcll(b) << bit;
    }
    const int wave = tid >> 6;
    if ((tid & 63) == 0) wtot[wave] = (int)wt;
    __syncthreads();
    int at = (int)below, nh = 0;
    for (int w = 0; w < NC / 64; ++w) {
        const int t = wtot[w];
        at += w < wave ? t : 0;
        nh += t;
    }
    if (hm) {
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            if (!((hm >> k) & 1u)) continue;
            const int key = 16 * tid + k;
            if (at < kCapHL) {
                HL[at] = (uint16_t)key;
            } else {  // beyond the list: settled by the thread that found it
                const int e = canon_encoding(d.label, LAB[pos(key)] & kIdxMask, st.t, d.key);
                lab_store(d.label, 16 * cell + k, e);
                LAB[pos(key)] = e;
            }
            ++at;
        }
    }
    __syncthreads();
    const int nl = min(nh, kCapHL);
    for (int j = tid; j < nl; j += NC) {
        const int key = HL[j];
        const int e = canon_encoding(d.label, LAB[pos(key)] & kIdxMask, st.t, d.key);
        lab_store(d.label, ti.global_site(key), e);
        LAB[pos(key)] = e;
    }
    __syncthreads();
}

// Names and keys of local roots in the merge.  A key is the root's site index
// with kLone set when the root is a component of one site: every bond it has
// left is of one tile-crossing tetrahedron, so every hook of it is made by the
// one workgroup that lists that tetrahedron's pairs and needs no
// compare-and-swap.  A tile's crossing list names the roots of its own sites
// by kHere | key, and a site of another tile by the index, in the list array,
// of the word where that tile keeps the site's key (its port words).
constexpr int kLone = 1 << 30;
constexpr int kHere = INT32_MIN;

// Port words: after a tile's crossing list (at the end of its stride), the
// keys of its sites that other tiles' crossing tetrahedra can reach, four per
// cell of each high face: (x: sites 14, 11, 10, 15), (y: 13, 7, 5, 15), (z: 9,
// 6, 5, 10), cells in the order of the face's (y, z), (x, z), (x, y).  Along a
// ragged axis a tile's last cell in the lattice stands for all beyond it, so
// that a neighbour finds the high face where a full tile has it.  The words
// are contiguous, where the labels they stand for are scattered over
// the tile's 32 KB.
template <int TX, int TY, int TZ>
struct Ports {
    static constexpr int kY = 4 * TY * TZ, kZ = kY + 4 * TX * TZ, kWords = kZ + 4 * TX * TY;
    static constexpr uint32_t kSites[3] = {0xFABEu, 0xF57Du, 0xA569u};  // site of word 4 i + k: nibble k
    // Word of a site at local cell (x, y, z) on the high face `face`.
    static constexpr int word(int face, int site, int x, int y, int z)
    {
        int k = 0;
        while (((kSites[face] >> (4 * k)) & 15u) != (uint32_t)site) ++k;
        return face == 0 ? 4 * (z * TY + y) + k : (face == 1 ? kY + 4 * (z * TX + x) + k : kZ + 4 * (y * TX + x) + k);
    }
};

// Crossing-pair emission items of a tile shape: one per (low-face cell c,
// down tetrahedron f) whose tetrahedron can have a vertex outside the tile
// (f = 0 on every low face, f = 1/2/3 on the face x/y/z = 0), packed as
// 4 c + f and sorted by f, so the lanes of a wave mostly share f.  port[mu-1]
// of a vertex mu beyond a low face: which axes it crosses (bits x, y, z of the
// top four) and its port word in the tile there, 0 when it never leaves.
// Whether that tile is another one is decided at run time (an axis with a
// single tile wraps onto itself).
struct EmitItem {
    uint16_t item, port[3];
};
template <int TX, int TY, int TZ>
struct EmitItems {
    alignas(8) EmitItem v[4 * TX * TY * TZ];
    int n;
};
constexpr uint32_t kLowerAxes = 0u | 1u << 3 | 2u << 6 | 4u << 9 | 6u << 12 | 5u << 15 | 3u << 18;  // axes lowered, per cell code
template <int TX, int TY, int TZ>
__host__ __device__ constexpr EmitItems<TX, TY, TZ> make_emit_items()
{
    EmitItems<TX, TY, TZ> t{};
    t.n = 0;
    for (int f = 0; f < 4; ++f)
        for (int c = 0; c < TX * TY * TZ; ++c) {
            const int x = c % TX, y = (c / TX) % TY, z = c / (TX * TY);
            const bool use = f == 0 ? (x == 0 || y == 0 || z == 0) : (f == 1 ? x == 0 : (f == 2 ? y == 0 : z == 0));
            if (!use) continue;
            EmitItem e{};
            e.item = (uint16_t)(4 * c + f);
            for (int mu = 1; mu < 4; ++mu) {
                const SiteRef R = down_vertex(f, mu);
                const uint32_t low = (kLowerAxes >> (3 * R.cell)) & 7u;
                const uint32_t out = low & ((x == 0 ? 1u : 0u) | (y == 0 ? 2u : 0u) | (z == 0 ? 4u : 0u));
                if (!out) continue;
                const int vx = (low & 1u) ? (x + TX - 1) % TX : x, vy = (low & 2u) ? (y + TY - 1) % TY : y,
                          vz = (low & 4u) ? (z + TZ - 1) % TZ : z;
                const int face = (out & 4u) ? 2 : ((out & 2u) ? 1 : 0);
                e.port[mu - 1] = (uint16_t)(out << 12 | (uint32_t)Ports<TX, TY, TZ>::word(face, R.site, vx, vy, vz));
            }
            t.v[t.n++] = e;
        }
    return t;
}
template <int TX, int TY, int TZ>
__constant__ EmitItems<TX, TY, TZ> kEmitItems = make_emit_items<TX, TY, TZ>();

// Vertex mu of down tetrahedron f as (cell code << 4 | site), byte 4 f + mu.
__host__ __device__ constexpr uint64_t down_vertex_bytes(int half)
{
    uint64_t w = 0;
    for (int k = 0; k < 8; ++k) {
        const SiteRef R = down_vertex(2 * half + k / 4, k % 4);
        w |= (uint64_t)(R.cell << 4 | R.site) << (8 * k);
    }
    return w;
}

// ------------------------------------------------------ tile components ---
// LDS words of the union buffers of a tile's waves (the U argument of
// tile_components): 128 per wave, one word per union, and room for one more
// row of 64 while a full one is united.  Later they hold two words per cell.
template <int NC>
constexpr int kUnionWords = 2 * NC;

// Second half of both models' tile pass (every thread of the block calls
// it; `act` is 0 for threads without a cell, lc[] holds the local index of
// each neighbour cell of the thread's cell, or -1 outside the tile): the
// components of the tile's sites from the active bonds of its cells, written
// as every site's tile-local root, and the tile's crossing list.
//
// Inside the tile, each down tetrahedron contributes the spanning edges of
// the components of its active bonds whose two ends lie in the tile (at most
// 3, from the K4 table).  A wave collects its cells' unions (about 330 at
// T_c) in an LDS buffer of its own and unites them 64 at a time, one per
// lane, as the buffer fills, with no barrier: united in place by the cells
// that find them, a third to a half of the lanes sit idle in each of the
// twelve slots.
//
// Every site is a vertex of exactly one down tetrahedron, owned by one cell,
// so the crossing bonds of different cells never join the same pair of
// sites.  For each down tetrahedron with a vertex outside the tile, each
// vertex is named by its tile-local root (inside) or by its port word
// (outside), and per component of the tetrahedron's active bonds the edges
// from the component's first vertex to the others whose name differs are
// emitted: at most 3 pairs per tetrahedron, none repeated.  These tetrahedra
// belong to the cells of the low faces; they are handed out to all threads as
// a table of (cell, tetrahedron) items.
template <int TX, int TY, int TZ>
__device__ __forceinline__ void tile_components(const RepDesc &d, const TileIdx<TX, TY, TZ> &ti, int tile, int tid,
                                                int lcid, bool valid, int cell, uint64_t act,
                                                const int (&lc)[kNCellCodes], uint32_t *P, uint32_t *U,
                                                const uint8_t *K4, uint32_t *NB /* 8 words */)
{
    constexpr int NC = TX * TY * TZ;
    static_assert(NC % 64 == 0, "tiles are whole waves");
    const int lane = tid & 63, wave = tid >> 6;
    const uint32_t base = node_off(16 * lcid);
    // Up tetrahedra: components from the table, roots at the smallest vertex.
#pragma unroll
    for (int f = 0; f < 4; ++f) {
        const uint32_t code = K4[(uint32_t)(act >> (6 * f)) & 63u];
#pragma unroll
        for (int mu = 0; mu < 4; ++mu) node(P, base + 4 * (4 * f + mu)) = base + 4 * (4 * f + ((code >> (2 * mu)) & 3));
    }
    __syncthreads();
    // Down tetrahedra, inside the tile: spanning edges, packed as two 16-bit
    // forest slots (17 NC < 2^16 up to 8x8x8; 17 bits are never needed, the
    // largest slot of a 1024-cell tile is 17407).
    {
        const int s0 = 17 * lcid;
        auto slot_of = [&](int f, int mu) {  // slot of a vertex (used only when it lies in the tile)
            const SiteRef R = down_vertex(f, mu);
            return (R.cell == kSelf ? s0 : 17 * lc[R.cell]) + R.site;
        };
        auto in_tile = [&](int f, int mu) {
            const SiteRef R = down_vertex(f, mu);
            return R.cell == kSelf || lc[R.cell] >= 0;
        };
        lds_word *W = (lds_word *)((lds_byte *)U + 512 * wave);
        int c = 0;  // unions in the buffer (wave uniform, below 64 between slots)
        auto unite_row = [&](int n) {  // the first n <= 64 unions of the buffer, one per lane
            wave_sync();
            if (lane < n) {
                const uint32_t u = W[lane];
                lds_unite(P, (u >> 14) & ~3u, (u & 0xFFFFu) << 2);
            }
        };
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            uint32_t inside = 0;  // bonds with both ends in the tile
#pragma unroll
            for (int e = 0; e < 6; ++e) inside |= (uint32_t)(in_tile(f, pair_a(e)) && in_tile(f, pair_b(e))) << e;
            const uint32_t code = K4[(uint32_t)(act >> (24 + 6 * f)) & inside];
            const int k0 = slot_of(f, 0), k1 = slot_of(f, 1), k2 = slot_of(f, 2), k3 = slot_of(f, 3);
#pragma unroll
            for (int mu = 1; mu < 4; ++mu) {
                const uint32_t rp = (code >> (2 * mu)) & 3u;
                const int kr = mu == 1 || rp == 0 ? k0 : (mu == 2 || rp == 1 ? k1 : k2);
                const int km = mu == 1 ? k1 : (mu == 2 ? k2 : k3);
                const bool use = rp != (uint32_t)mu;
                const uint64_t b = __ballot(use);
                const int at = c + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
                if (use) W[at] = (uint32_t)kr << 16 | (uint32_t)km;
                c += (int)__popcll(b);
                if (c >= 64) {
                    unite_row(64);
                    const uint32_t rest = W[64 + lane];
                    wave_sync();
                    W[lane] = rest;
                    wave_sync();
                    c -= 64;
                }
            }
        }
        unite_row(c);
    }
    __syncthreads();
    // Tile-local roots of the thread's sites, all sixteen walks a level at a
    // time (parents never exceed children, so the walks end): as global site
    // indices into the labels, and into the forest entries, where the
    // emission below reads the root of any site of the tile.  The global
    // index of slot s = 17 c + k is s plus a word of its cell c, kept in U
    // (free after the unions).
    uint32_t r[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) r[k] = node(P, base + 4 * k);
    uint32_t moved;
    do {
        moved = 0;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const uint32_t p = node(P, r[k]);
            moved |= p ^ r[k];
            r[k] = p;
        }
    } while (moved);
    U[lcid] = (uint32_t)(16 * cell - 17 * lcid);
    uint32_t *DA = U + NC;  // active bonds of the cells' down tetrahedra
    DA[lcid] = (uint32_t)(act >> 24);
    // Sites without an active bond in their up tetrahedron: bit 6 f + mu, in
    // the cell's unused 17th forest word.
    const uint32_t ub = (uint32_t)act & 0xFFFFFFu;
    const uint32_t bare = (~(ub | ub >> 1 | ub >> 2) & 0x41041u) | (~(ub | ub >> 3 | ub >> 4) & 0x41041u) << 1 |
                          (~(ub >> 1 | ub >> 3 | ub >> 5) & 0x41041u) << 2 | (~(ub >> 2 | ub >> 4 | ub >> 5) & 0x41041u) << 3;
    node(P, base + 64) = bare;
    // Port words of the tiles one step down the axes in the bits of q (q = 0:
    // this tile's own).
    using PT = Ports<TX, TY, TZ>;
    const int own = (tile + 1) * d.list_stride - PT::kWords;
    if (tid < 8) {
        const int qx = (tid & 1) ? (ti.bx == 0 ? d.ntx - 1 : ti.bx - 1) : ti.bx;
        const int qy = (tid & 2) ? (ti.by == 0 ? d.nty - 1 : ti.by - 1) : ti.by;
        const int qz = (tid & 4) ? (ti.bz == 0 ? d.ntz - 1 : ti.bz - 1) : ti.bz;
        NB[tid] = (uint32_t)(((qz * d.nty + qy) * d.ntx + qx + 1) * d.list_stride - PT::kWords);
    }
    __syncthreads();
    const int L = d.L;
    const int ex = min(TX, L - ti.bx * TX) - 1, ey = min(TY, L - ti.by * TY) - 1, ez = min(TZ, L - ti.bz * TZ) - 1;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        // cell of the root's slot: offset / 68 (unsigned: past 2^31 for 16x8x8 tiles, below 2^32)
        const uint32_t c = (uint32_t)__umul24(r[k], 61681u) >> 22;
        r[k] = U[c] + (r[k] >> 2);
        node(P, base + 4 * k) = r[k];
    }
    if (valid) {
        int4 *out = reinterpret_cast<int4 *>(d.label + 16 * cell);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            out[q] = make_int4((int)r[4 * q], (int)r[4 * q + 1], (int)r[4 * q + 2], (int)r[4 * q + 3]);
        // Port words.  The tetrahedron that reaches such a site from another
        // tile has united nothing here, so a bare one is a component of one
        // site.  Along a ragged axis the last cell also stands at the tile's
        // full edge, where a neighbour across that axis looks for it.
        auto key4 = [&](int a, int b, int c4, int e) {
            auto key = [&](int k) { return (int)(r[k] | __builtin_amdgcn_ubfe(bare, 6u * (k / 4) + k % 4, 1u) << 30); };
            return make_int4(key(a), key(b), key(c4), key(e));
        };
        int4 *pw = reinterpret_cast<int4 *>(d.pairs + own);
        const int lx = lcid % TX, ly = (lcid / TX) % TY, lz = lcid / (TX * TY);
        const bool full = ex == TX - 1 && ey == TY - 1 && ez == TZ - 1;
        const int vx = lx == ex ? TX - 1 : lx, vy = ly == ey ? TY - 1 : ly, vz = lz == ez ? TZ - 1 : lz;
        if (lx == ex) {
            const int4 w = key4(14, 11, 10, 15);
            pw[lz * TY + ly] = w;
            if (!full) {
                pw[lz * TY + vy] = w;
                pw[vz * TY + ly] = w;
            }
        }
        if (ly == ey) {
            const int4 w = key4(13, 7, 5, 15);
            pw[PT::kY / 4 + lz * TX + lx] = w;
            if (!full) {
                pw[PT::kY / 4 + lz * TX + vx] = w;
                pw[PT::kY / 4 + vz * TX + lx] = w;
            }
        }
        if (lz == ez) {
            const int4 w = key4(9, 6, 5, 10);
            pw[PT::kZ / 4 + ly * TX + lx] = w;
            if (!full) {
                pw[PT::kZ / 4 + ly * TX + vx] = w;
                pw[PT::kZ / 4 + vy * TX + lx] = w;
            }
        }
    }
    __syncthreads();
    // Crossing pairs, one item (cell, down tetrahedron) per thread and round.
    // Each round places its pairs in item order: a lane's offset is the
    // number of pairs of the lanes below it (two ballots of the 0..3 pair
    // count), plus the totals of the lower waves, kept in U.
    int2 *list = reinterpret_cast<int2 *>(d.pairs + (int64_t)tile * d.list_stride) + 1;
    constexpr uint64_t kVert0 = down_vertex_bytes(0), kVert1 = down_vertex_bytes(1);
    constexpr int kItems = make_emit_items<TX, TY, TZ>().n;
    int placed = 0;  // pairs listed so far (the same in every thread)
    for (int jb = 0; jb < kItems; jb += NC) {
        const int j = jb + tid;
        int2 q[3];
        bool e[3] = {false, false, false};
        if (j < kItems) {
            const EmitItem it = kEmitItems<TX, TY, TZ>.v[j];
            const int c = it.item >> 2, f = it.item & 3;
            const int ix = c % TX, iy = (c / TX) % TY, iz = c / (TX * TY);
            if (ix <= ex && iy <= ey && iz <= ez) {
                const uint32_t code = K4[(DA[c] >> (6 * f)) & 63u];
                const uint64_t vb = (f < 2) ? kVert0 : kVert1;
                bool outside = false, alone[4];
                int id[4];
#pragma unroll
                for (int mu = 0; mu < 4; ++mu) {
                    const uint32_t v = (uint32_t)(vb >> (8 * (4 * (f & 1) + mu))) & 0xFFu;
                    const uint32_t low = (kLowerAxes >> (3 * (v >> 4))) & 7u;
                    const uint32_t port = mu == 0 ? 0u : it.port[mu == 0 ? 0 : mu - 1];
                    const int b = (int)NB[port >> 12];
                    if (b == own) {
                        // in the tile; an axis of one tile wraps onto itself
                        const int x = (low & 1u) ? (ix == 0 ? ex : ix - 1) : ix;
                        const int y = (low & 2u) ? (iy == 0 ? ey : iy - 1) : iy;
                        const int z = (low & 4u) ? (iz == 0 ? ez : iz - 1) : iz;
                        const uint32_t off = 68u * (uint32_t)((z * TY + y) * TX + x), k = v & 15u;
                        id[mu] = kHere | (int)node(P, off + 4u * k);
                        alone[mu] = (node(P, off + 64u) >> (6u * (k >> 2) + (k & 3u))) & 1u;
                    } else {
                        id[mu] = b + (int)(port & 0xFFFu);
                        alone[mu] = false;
                        outside = true;
                    }
                }
                if (outside) {
                    // a bare site here is a component of its own unless this
                    // tetrahedron joined it to another site of the tile
                    const bool e01 = id[0] == id[1], e02 = id[0] == id[2], e03 = id[0] == id[3], e12 = id[1] == id[2],
                               e13 = id[1] == id[3], e23 = id[2] == id[3];
                    id[0] |= alone[0] && !(e01 || e02 || e03) ? kLone : 0;
                    id[1] |= alone[1] && !(e01 || e12 || e13) ? kLone : 0;
                    id[2] |= alone[2] && !(e02 || e12 || e23) ? kLone : 0;
                    id[3] |= alone[3] && !(e03 || e13 || e23) ? kLone : 0;
#pragma unroll
                    for (int mu = 1; mu < 4; ++mu) {
                        const int rp = (code >> (2 * mu)) & 3;
                        const int rid = rp == 0 ? id[0] : (rp == 1 ? id[1] : id[2]);
                        e[mu - 1] = rp != mu && rid != id[mu];
                        q[mu - 1] = make_int2(rid, id[mu]);
                    }
                }
            }
        }
        const uint32_t npair = (uint32_t)e[0] + (uint32_t)e[1] + (uint32_t)e[2];
        const uint64_t b0 = __ballot(npair & 1u), b1 = __ballot(npair & 2u);
        const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(b0 >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b0, 0u)) +
                               2u * __builtin_amdgcn_mbcnt_hi((uint32_t)(b1 >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b1, 0u));
        if (lane == 0) U[wave] = (uint32_t)(__popcll(b0) + 2 * __popcll(b1));
        __syncthreads();
        int at = placed + (int)below, total = 0;
        for (int w = 0; w < NC / 64; ++w) {
            const int t = (int)U[w];
            at += w < wave ? t : 0;
            total += t;
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            if (e[k]) list[at] = q[k];
            at += e[k];
        }
        placed += total;
        if (jb + NC < kItems) __syncthreads();  // U[wave] is rewritten by the next round
    }
    if (tid == 0) d.pairs[(int64_t)tile * d.list_stride] = placed;
}

// ------------------------------------------------------- forest passes ---
// Work on the tiles' crossing lists, one workgroup per tile:
//   unite  unite the local roots of the two names of every pair (the unite
//          pass of every chain, and a phase of the persistent kernel);
//   store  store the encoded root of its tree (the cluster's smallest site
//          and its flip coin) in every local root of the list (walks stop
//          at the first stored encoding, so they shorten as the pass
//          proceeds); only the persistent kernel runs it, the chains
//          settle their roots in the flip pass instead.

// Unite pass of one tile (kBlock threads).  The pairs of a tile mostly share
// a few local roots, so hooking them one by one makes the tile's threads
// race for the same roots.  Instead, the distinct local roots of the list
// are grouped by the list's pairs in an LDS union-find, and every member of
// a group is united with the group's smallest member: the hooks of one tile
// then target distinct roots.  Pairs beyond the LDS tables are united
// directly.
//
// When a store phase follows (keep_roots: the persistent kernel), the
// tile's list is then replaced by its distinct local roots, which is all
// the store phase needs: it skips resolving names again.  With room for it
// (list_stride >= 2 + 2 H), head[1] = -m and the m roots from head[2] on are
// followed, from head[2 + H] on, by the list position of each root's group
// representative, so the store phase walks once per group.  Otherwise
// head[1] = m and only the roots are written.  head[1] = 0 keeps the pairs
// (some root did not fit in the table).  A local root that occurs only in
// pairs whose two names resolve to it is left out: it is never hooked nor
// hooked under, and its entry (itself) is already its canonical form.
constexpr int kTileRoots = 1024;  // LDS root table of the unite pass

constexpr int kUniteThreads = 256;   // threads per tile in the unite pass (its CAS chains are latency bound;
                                     // smaller workgroups let more tiles run at once)

// LDS words that other threads of the workgroup change concurrently (root
// tables and parent slots of the unite pass and the store phase) are read and
// written with relaxed workgroup-scope atomics, so that no load is hoisted
// out of a retry loop or served from a register copy.
__device__ __forceinline__ int lds_ld(const int *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }
__device__ __forceinline__ void lds_st(int *p, int v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }

// LDS of the unite pass of one tile.
struct UniteLds {
    static constexpr int kMaxListed = 1024;  // pairs kept in LDS
    int HK[kTileRoots];           // local root of the slot, -1 if free
    int HP[kTileRoots];           // LDS parent slot
    uint64_t BEST[kTileRoots];    // per group: smallest member << 10 | its slot
    int16_t PA[kMaxListed];
    alignas(8) int16_t PB[kMaxListed];
    int nroots, missed, direct, nlost;
};

template <int NT, bool COUNT = false>
__device__ __forceinline__ void unite_tile_pairs(int32_t *lab, int *head, int64_t tile_words, int list_stride, int tid, UniteLds &S,
                                                 unsigned long long *counts, bool keep_roots)
{
    constexpr int H = kTileRoots;                    // root slots
    constexpr int kMaxListed = UniteLds::kMaxListed;  // pairs kept in LDS
    const int2 *list = reinterpret_cast<const int2 *>(head) + 1;
    // The thread's first pairs are fetched along with their number (any words
    // of the tile's stride will do), one memory latency earlier.
    constexpr int kBatch = 4;
    const int n = head[0], room = (list_stride - 2) / 2;
    int2 first[kBatch];
#pragma unroll
    for (int i = 0; i < kBatch; ++i) first[i] = list[min(tid + i * NT, room - 1)];
    for (int k = tid; k < H; k += NT) {
        S.HK[k] = -1;
        S.HP[k] = k;
        S.BEST[k] = ~0ull;
    }
    if (tid == 0) {
        S.nroots = 0;
        S.missed = 0;
        S.direct = 0;
        S.nlost = 0;
    }
    if (n == 0) return;  // the same in every thread
    __syncthreads();
    const int *words = head - (int64_t)tile_words;  // start of the list array, which port names index
    auto name_key = [&](int name) { return name < 0 ? (name & INT32_MAX) : words[name]; };
    auto insert = [&](int key) {
        uint32_t h = (uint32_t)key * 0x9E3779B1u;
        h ^= h >> 15;
        for (int probe = 0; probe < 32; ++probe) {
            const int slot = (int)((h + (uint32_t)probe) & (H - 1));
            int prev = lds_ld(&S.HK[slot]);
            if (prev == -1) prev = atomicCAS(&S.HK[slot], -1, key);
            if (prev == -1 || prev == key) return slot;
        }
        return -1;
    };
    // Four of the thread's pairs at a time: their names are resolved with all
    // port words in flight together, then entered in the table.
    for (int k0 = tid; k0 < n; k0 += kBatch * NT) {
        int ra[kBatch], rb[kBatch];
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            const int k = k0 + i * NT;
            const int2 p = k >= n ? make_int2(kHere, kHere) : (k0 == tid ? first[i] : list[k]);
            ra[i] = name_key(p.x);
            rb[i] = name_key(p.y);
        }
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            const int k = k0 + i * NT;
            if (k >= n) break;
            const int sa = ra[i] == rb[i] ? -1 : insert(ra[i]), sb = ra[i] == rb[i] ? -1 : insert(rb[i]);
            const bool listed = k < kMaxListed && sa >= 0 && sb >= 0;
            if (!listed && ra[i] != rb[i]) {
                forest_unite<COUNT>(lab, ra[i] & kIdxMask, rb[i] & kIdxMask, counts);
                S.direct = 1;
            }
            if (ra[i] != rb[i] && (sa < 0 || sb < 0)) S.missed = 1;
            if (k < kMaxListed) {
                S.PA[k] = (int16_t)(listed ? sa : -1);
                S.PB[k] = (int16_t)(listed ? sb : -1);
            }
        }
    }
    __syncthreads();
    auto slot_find = [&](int x) {
        for (int it = 0; it < H; ++it) {
            const int p = lds_ld(&S.HP[x]);
            if (p == x) return x;
            const int gp = lds_ld(&S.HP[p]);
            if (gp != p) lds_st(&S.HP[x], gp);
            x = p;
        }
        return x;
    };
    const int nl = min(n, kMaxListed);
    for (int k = tid; k < nl; k += NT) {
        int a = S.PA[k], b = S.PB[k];
        if (a < 0) continue;
        for (int it = 0; it < H; ++it) {
            a = slot_find(a);
            b = slot_find(b);
            if (a == b) break;
            if (a < b) {
                const int t = a;
                a = b;
                b = t;
            }
            const int old = atomicMin(&S.HP[a], b);
            if (old == a) break;
            a = old;
        }
    }
    __syncthreads();
    for (int s = tid; s < H; s += NT) {
        if (S.HK[s] < 0) continue;
        atomicMin(&S.BEST[slot_find(s)], (uint64_t)(S.HK[s] & kIdxMask) << 10 | (uint64_t)s);
    }
    __syncthreads();
    // The pairs are read: overwrite them with the distinct local roots (at
    // most 2n of them, so they fit where the pairs were); PA now holds each
    // slot's list position.
    const bool with_reps = keep_roots && list_stride >= 2 + 2 * H;
    if (keep_roots && !S.missed) {
        for (int s = tid; s < H; s += NT) {
            if (S.HK[s] < 0) continue;
            const int j = atomicAdd(&S.nroots, 1);
            S.PA[s] = (int16_t)j;
            head[2 + j] = S.HK[s] & kIdxMask;
        }
    }
    __syncthreads();
    // Each member of a group other than its smallest is hooked under the
    // smallest (a smaller node, so a valid parent for a root).  A lone root is
    // hooked by no other workgroup, and nothing hangs below one that is not its
    // group's smallest: a plain store does (unless a pair beyond the LDS tables
    // was united directly).  These are 44% of the hooks at T_c, and the pass is
    // bound by the rate of the rest: another member that is still a root of
    // the global forest is hooked by one compare-and-swap, without a walk, and
    // the thread's compare-and-swaps are in flight together; one that finds
    // the member already hooked is lost, and its union continues from the
    // parent it returned.
    const bool plain = !S.direct;
    // Lost ones (the parent found, the group's smallest member) are shared out
    // over the threads in the space of the listed pairs' second slots.
    int2 *lost = reinterpret_cast<int2 *>(S.PB);
    constexpr int kMaxLost = (int)(sizeof(S.PB) / sizeof(int2));
    constexpr int kSlotsPerThread = (H + NT - 1) / NT;
    constexpr int kHookBatch = kSlotsPerThread < 4 ? kSlotsPerThread : 4;
    for (int i0 = 0; i0 < kSlotsPerThread; i0 += kHookBatch) {
        int ha[kHookBatch], hb[kHookBatch], old[kHookBatch];
#pragma unroll
        for (int i = 0; i < kHookBatch; ++i) {
            const int s = tid + (i0 + i) * NT;
            ha[i] = -1;
            hb[i] = -1;
            if (s < H && S.HK[s] >= 0) {
                const int rs = (int)(S.BEST[slot_find(s)] & (uint64_t)(H - 1));
                if (!S.missed && with_reps) head[2 + H + S.PA[s]] = S.PA[rs];
                if (rs != s) {
                    const int key = S.HK[s];
                    hb[i] = S.HK[rs] & kIdxMask;
                    if (plain && (key & kLone)) lab_store_through(lab, key & kIdxMask, kTag | hb[i]);
                    else ha[i] = key & kIdxMask;
                }
            }
        }
#pragma unroll
        for (int i = 0; i < kHookBatch; ++i) old[i] = ha[i] >= 0 ? atomicCAS(lab + ha[i], ha[i], kTag | hb[i]) : -1;
#pragma unroll
        for (int i = 0; i < kHookBatch; ++i) {
            if (ha[i] < 0) continue;
            if (COUNT) {  // measurement runs only (a kernel of its own)
                atomicAdd(&counts[0], 1ull);
                if (old[i] == ha[i]) atomicAdd(&counts[1], 1ull);
            }
            if (old[i] == ha[i]) continue;
            const int j = atomicAdd(&S.nlost, 1);
            if (j < kMaxLost) lost[j] = make_int2(old[i] & kIdxMask, hb[i]);
            else forest_unite<COUNT>(lab, old[i] & kIdxMask, hb[i], counts);
        }
    }
    __syncthreads();
    const int nlost = min(S.nlost, kMaxLost);
    for (int j = tid; j < nlost; j += NT) forest_unite<COUNT>(lab, lost[j].x, lost[j].y, counts);
    if (tid == 0 && keep_roots) head[1] = S.missed ? 0 : (with_reps ? -S.nroots : S.nroots);
}

// Store phase of one tile in the persistent kernel (NT threads; HK:
// kTileRoots ints of LDS).
template <int NT>
__device__ __forceinline__ void store_tile(const RepDesc &d, const RepState &st, int tile, int tid, int *HK)
{
    constexpr int H = kTileRoots;
    int *head = d.pairs + (int64_t)tile * d.list_stride;
    const int2 *list = reinterpret_cast<const int2 *>(head) + 1;
    const int n = head[0];
    int32_t *lab = d.label;
    if (n == 0) return;
    const int nroots = head[1];  // != 0: the list holds the tile's distinct local roots
    if (nroots < 0) {
        // with group representatives: one walk per group, then plain stores
        const int m = -nroots;
        const int *rp = head + 2 + H;
        for (int k = tid; k < m; k += NT) {
            if (rp[k] != k) continue;
            const int r = head[2 + k];
            const int e = canon_encoding(lab, r, st.t, d.key);
            HK[k] = e;
            lab_store(lab, r, e);
        }
        __syncthreads();
        for (int k = tid; k < m; k += NT)
            if (rp[k] != k) lab_store(lab, head[2 + k], HK[rp[k]]);
        return;
    }
    if (nroots > 0) {
        for (int k = tid; k < nroots; k += NT) {
            const int r = head[2 + k];
            lab_store(lab, r, canon_encoding(lab, r, st.t, d.key));
        }
        return;
    }
    // The list kept its pairs: store once per distinct local root, found
    // through an LDS hash table (a full table stores directly).
    for (int k = tid; k < H; k += NT) HK[k] = -1;
    __syncthreads();
    auto add = [&](int key) {
        uint32_t h = (uint32_t)key * 0x9E3779B1u;
        h ^= h >> 15;
        for (int probe = 0; probe < 32; ++probe) {
            const int slot = (int)((h + (uint32_t)probe) & (H - 1));
            int prev = lds_ld(&HK[slot]);
            if (prev == -1) prev = atomicCAS(&HK[slot], -1, key);
            if (prev == -1 || prev == key) return;
        }
        lab_store(lab, key, canon_encoding(lab, key, st.t, d.key));
    };
    for (int k = tid; k < 2 * n; k += NT) {
        const int2 p = list[k >> 1];
        const int name = (k & 1) ? p.y : p.x;
        add((name < 0 ? name : d.pairs[name]) & kIdxMask);
    }
    __syncthreads();
    for (int k = tid; k < H; k += NT) {
        const int key = HK[k];
        if (key >= 0) lab_store(lab, key, canon_encoding(lab, key, st.t, d.key));
    }
}

// Unite pass of one tile (NT threads).
template <int NT, bool COUNT = false>
__device__ __forceinline__ void unite_tile(const RepDesc &d, int tile, int tid, UniteLds &S,
                                           unsigned long long *counts = nullptr, bool keep_roots = true)
{
    const int64_t at = (int64_t)tile * d.list_stride;
    int *head = d.pairs + at;
    unite_tile_pairs<NT, COUNT>(d.label, head, at, d.list_stride, tid, S, counts, keep_roots);
}

// ------------------------------------------------------------- records ---
// The record of the last sweep (ring slot st.e_pending, sweep st.t - 1): its
// magnetisation from the ntiles partials of that sweep's settle-and-flip pass,
// which therefore has to be the last sweep the lattice had (LDS-resident sweeps
// leave no record pending), its
// energy from the partials at e_at (the next tile pass, whose tiles count the
// energy of the state entering the sweep, or the energy tail), in an order
// fixed by the block size.  with_energy = false leaves the energy to a later
// call.  A block of kBlock threads; red: 16 words of 8 bytes per sum.
template <int NV>
__device__ __forceinline__ void write_pending_record(const RepDesc &d, const RepState &st, int ntiles, int tid,
                                                     bool with_energy, int e_at, int e_n, void *red)
{
    DevRecord r;
    r.sweep = (int64_t)st.t - 1;
    r.bond_sum = 0;
    r.M_int = 0;
    r.reserved = 0;
    r.E = 0.0;
    r.M[0] = r.M[1] = r.M[2] = 0.0;
    double m;
    if constexpr (NV == 1) {
        int64_t v[2] = {0, 0};  // magnetisation, bond sum
        for (int k = tid; k < ntiles; k += kBlock) v[0] += d.ipart[d.mpart_off + k];
        if (with_energy)
            for (int k = tid; k < e_n; k += kBlock) v[1] += d.ipart[e_at + k];
        block_sum_n<int64_t, 2>(v, (int64_t *)red);
        r.bond_sum = v[1];
        r.M_int = v[0];
        if (with_energy) r.E = -d.J * (double)v[1];
        r.M[0] = (double)v[0];
        m = (double)v[0] / (double)d.N;
    } else {
        double v[NV + 1];
#pragma unroll
        for (int q = 0; q <= NV; ++q) v[q] = 0.0;
        for (int k = tid; k < ntiles; k += kBlock)
#pragma unroll
            for (int q = 0; q < NV; ++q) v[q] += d.dpart[d.mpart_off * (1 + q) + k];
        if (with_energy)
            for (int k = tid; k < e_n; k += kBlock) v[NV] += d.dpart[e_at + k];
        block_sum_n<double, NV + 1>(v, (double *)red);
        if (with_energy) r.E = -d.J * v[NV];
#pragma unroll
        for (int q = 0; q < NV; ++q) r.M[q] = v[q];
        m = sqrt(r.M[0] * r.M[0] + r.M[1] * r.M[1] + r.M[2] * r.M[2]) / (double)d.N;
    }
    r.m2 = m * m;
    r.m4 = r.m2 * r.m2;
    if (tid == 0) d.ring[st.e_pending] = r;
}

__device__ __forceinline__ void write_pending_record(const RepDesc &d, int model, const RepState &st, int ntiles, int tid,
                                                     bool with_energy, int e_at, int e_n, void *red)
{
    if (model == 1) write_pending_record<1>(d, st, ntiles, tid, with_energy, e_at, e_n, red);
    else if (model == 2) write_pending_record<2>(d, st, ntiles, tid, with_energy, e_at, e_n, red);
    else write_pending_record<3>(d, st, ntiles, tid, with_energy, e_at, e_n, red);
}

// The unite pass of a chain: one workgroup per replica that writes the record
// of the previous sweep, whose sums are complete by now, and the state for the
// settle-and-flip pass, and one per tile.  The record's serial loads take 15 us
// and more of a large lattice, so its block starts first: last in the grid it
// outlasted the tiles where few bonds are active (XY L = 128 at 20 T_c 40 us,
// first 32).  A kernel
// of its own for the records, one workgroup per replica, had cost 4 to 5 us
// and a launch gap per sweep, 5% to 9% of a sweep of L <= 64.  COUNT: it
// counts its compare-and-swaps into c.counts (measurement runs).  The chains
// settle their roots in the flip pass and run no store pass, so the lists are
// left as they are.
template <bool COUNT>
__device__ __forceinline__ void unite_block(Chain c, uint32_t b, UniteLds &S)
{
    static_assert(kUniteThreads == kBlock, "the record block");
    if ((int)b < c.nreps) {
        const int rep = (int)b;
        const RepDesc &d = c.desc[rep];
        const RepState st = c.state[rep][0];
        if (threadIdx.x == 0) c.state[rep][1] = st;
        if (st.remaining > 0 && st.e_pending >= 0)
            write_pending_record(d, c.model, st, mag_partials(c.state[rep]), threadIdx.x, true, 0, d.ntx * d.nty * d.ntz,
                                 S.BEST);
        return;
    }
    const int blk = xcd_block((int)b - c.nreps, c.ntile_blocks);
    const int rep = c.tile_rep[blk];
    if (c.state[rep]->remaining <= 0) return;
    const RepDesc &d = c.desc[rep];
    unite_tile<kUniteThreads, COUNT>(d, blk - d.tile_base, threadIdx.x, S, c.counts, false);
}

template <bool COUNT = false>
__global__ __launch_bounds__(kUniteThreads) void k_forest(Chain c)
{
    __shared__ UniteLds S;
    unite_block<COUNT>(c, blockIdx.x, S);
}

// First block of a replica in the settle-and-flip pass: the state of the next
// sweep and the number of magnetisation partials this pass leaves.
__device__ __forceinline__ void advance_state(RepState *s, const RepState &st, const RepDesc &d)
{
    s[0] = advanced(st, d.ring_cap);
    mag_partials(s) = d.ntx * d.nty * d.ntz;
}

// Shape dispatch: calls F::template run<TX, TY, TZ>(args...).
template <typename F, typename... Args>
hipError_t with_tile_shape(int shape, Args &&...args)
{
    switch (shape) {
    case kTile844: return F::template run<8, 4, 4>(args...);
    case kTile444: return F::template run<4, 4, 4>(args...);
    case kTile888: return F::template run<8, 8, 8>(args...);
    case kTile1688: return F::template run<16, 8, 8>(args...);
    default: return F::template run<8, 8, 4>(args...);
    }
}

// Launchers of the model-independent passes (tile_common.hip).
hipError_t launch_unite(const Chain &c, hipStream_t st, const LaunchHook &hook);
hipError_t launch_pending_records(const Chain &c, bool with_energy, hipStream_t st, const LaunchHook &hook);

// Per-model chain launchers (ising_tiled.hip, on_tiled.hip).
hipError_t launch_ising_tiles(const Chain &c, hipStream_t st, const LaunchHook &hook);
hipError_t launch_ising_flip(const Chain &c, hipStream_t st, const LaunchHook &hook);
hipError_t launch_ising_energy_tail(const Chain &c, hipStream_t st, const LaunchHook &hook);
hipError_t launch_on_tiles(const Chain &c, hipStream_t st, const LaunchHook &hook);
hipError_t launch_on_flip(const Chain &c, hipStream_t st, const LaunchHook &hook);
hipError_t launch_on_tiles(const Chain &xy, const Chain &heisenberg, hipStream_t st, const LaunchHook &hook);
hipError_t launch_on_flip(const Chain &xy, const Chain &heisenberg, hipStream_t st, const LaunchHook &hook);
hipError_t launch_on_energy_tail(const Chain &c, hipStream_t st, const LaunchHook &hook);

}  // namespace pyro

// Model-independent launchers of the tiled sweep: the passes over the
// tiles' crossing lists, the canonical labels the host reads (written to a
// separate buffer), and the dispatch of one sweep of a chain to its model.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "device_util.hpp"
#include "kernels.hpp"
#include "lattice.hpp"
#include "philox.hpp"
#include "tile_common.hpp"

namespace pyro {

// Canonical label of every site into `out` (only when the host reads
// labels; the label array itself is left as the sweep built it, so the walks
// of other threads never see a rewritten entry).
__global__ __launch_bounds__(kBlock) void k_canonical_labels(const int32_t *__restrict__ label,
                                                             int32_t *__restrict__ out, int64_t N)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    out[i] = canonical_label(label, i);
}

hipError_t launch_unite(const Chain &c, hipStream_t st, const LaunchHook &hook)
{
    if (c.counts) PYRO_LAUNCH(kKUnite, k_forest<true>, c.ntile_blocks + c.nreps, kUniteThreads, c);
    else PYRO_LAUNCH(kKUnite, k_forest<false>, c.ntile_blocks + c.nreps, kUniteThreads, c);
    return hipSuccess;
}

// Complete the pending record of every replica that has one: after the energy
// tail (with_energy), or, before a persistent launch overwrites the
// magnetisation partials, all but its energy, which that launch adds.
__global__ __launch_bounds__(kBlock) void k_pending_records(Chain c, bool with_energy)
{
    __shared__ double red[16 * 4];
    const int rep = blockIdx.x;
    const RepState st = c.state[rep][0];
    if (st.e_pending < 0) return;
    const RepDesc &d = c.desc[rep];
    write_pending_record(d, c.model, st, mag_partials(c.state[rep]), threadIdx.x, with_energy, d.tail_off, blocks_for(d.ncell), red);
    if (with_energy && threadIdx.x == 0) c.state[rep]->e_pending = -1;
}

hipError_t launch_pending_records(const Chain &c, bool with_energy, hipStream_t st, const LaunchHook &hook)
{
    PYRO_LAUNCH(kKFinalize, k_pending_records, c.nreps, kBlock, c, with_energy);
    return hipSuccess;
}

static hipError_t launch_tiles(const Chain &c, hipStream_t st, const LaunchHook &hook)
{
    return c.model == 1 ? launch_ising_tiles(c, st, hook) : launch_on_tiles(c, st, hook);
}

static hipError_t launch_flip(const Chain &c, hipStream_t st, const LaunchHook &hook)
{
    return c.model == 1 ? launch_ising_flip(c, st, hook) : launch_on_flip(c, st, hook);
}

hipError_t launch_chain_sweep(const Chain &c, hipStream_t st, const LaunchHook &hook)
{
    if (c.nreps == 0) return hipSuccess;
    hipError_t e = launch_tiles(c, st, hook);
    if (e == hipSuccess) e = launch_unite(c, st, hook);
    if (e == hipSuccess) e = launch_flip(c, st, hook);
    return e;
}

// The unite pass of two or three chains in one launch: it does not depend on
// the model or on the tile shape.
__global__ __launch_bounds__(kUniteThreads) void k_forest_chains(Chain a, Chain b, Chain c)
{
    __shared__ UniteLds S;
    int blk = (int)blockIdx.x;
    Chain mine = a;
    if (blk >= a.ntile_blocks + a.nreps) {
        blk -= a.ntile_blocks + a.nreps;
        mine = b;
        if (blk >= b.ntile_blocks + b.nreps) {
            blk -= b.ntile_blocks + b.nreps;
            mine = c;
        }
    }
    unite_block<false>(mine, blk, S);
}

// One sweep of the chains of a group.  Chains of several models share
// launches: each pass of a chain of a few small lattices leaves most of the
// chip idle, and the passes of a sweep follow each other.  The unite passes
// always do; the tile and flip passes of the O(n) chains do when their tile
// shapes are the same (one launch for two block sizes would leave threads
// idle).
hipError_t launch_chains_sweep(const Chain *cs, int n, hipStream_t st)
{
    const LaunchHook none{nullptr, nullptr, nullptr};
    hipError_t e = hipSuccess;
    if (n < 2 || cs[0].counts) {  // counted unite passes (measurement runs) are launches of their own
        for (int k = 0; k < n && e == hipSuccess; ++k) e = launch_chain_sweep(cs[k], st, none);
        return e;
    }
    // in the order of the models, so the O(n) chains, if both are there, are the last two
    const bool both = cs[n - 2].model == 2 && cs[n - 1].model == 3 && cs[n - 2].shape == cs[n - 1].shape;
    for (int k = 0; k < (both ? n - 2 : n) && e == hipSuccess; ++k) e = launch_tiles(cs[k], st, none);
    if (both && e == hipSuccess) e = launch_on_tiles(cs[n - 2], cs[n - 1], st, none);
    if (e != hipSuccess) return e;
    int grid = 0;
    for (int k = 0; k < n; ++k) grid += cs[k].ntile_blocks + cs[k].nreps;
    k_forest_chains<<<grid, kUniteThreads, 0, st>>>(cs[0], cs[1], cs[n - 1]);
    e = hipGetLastError();
    for (int k = 0; k < (both ? n - 2 : n) && e == hipSuccess; ++k) e = launch_flip(cs[k], st, none);
    if (both && e == hipSuccess) e = launch_on_flip(cs[n - 2], cs[n - 1], st, none);
    return e;
}

hipError_t launch_chain_energy_tail(const Chain &c, hipStream_t st, const LaunchHook &hook)
{
    if (c.nreps == 0) return hipSuccess;
    return c.model == 1 ? launch_ising_energy_tail(c, st, hook) : launch_on_energy_tail(c, st, hook);
}

hipError_t launch_canonical_labels(const RepDesc &d, int32_t *out, hipStream_t st)
{
    k_canonical_labels<<<blocks_for(d.N), kBlock, 0, st>>>(d.label, out, d.N);
    return hipGetLastError();
}

// Tiles of the smallest built shape bound the tile count of every shape.
static int64_t max_tiles(int L)
{
    int64_t m = 0;
    for (int s = 0; s < kNumTileShapes; ++s) {
        const TileDims t = tile_dims(s);
        m = std::max<int64_t>(m, (int64_t)((L + t.x - 1) / t.x) * ((L + t.y - 1) / t.y) * ((L + t.z - 1) / t.z));
    }
    return m;
}

int64_t max_tile_count(int L) { return max_tiles(L); }
// A tile's crossing list holds at most 3 pairs for each tetrahedron that can
// leave it, about half of what 4 tetrahedra for each of its low-face cells
// would need; the port words at the end of the stride take less than the
// other half.  A multiple of four words keeps them aligned.
int tile_list_stride(int shape)
{
    const TileDims t = tile_dims(shape);
    const int face = t.x * t.y * t.z - (t.x - 1) * (t.y - 1) * (t.z - 1);
    return (2 + 2 * 12 * face) / 4 * 4;
}

int64_t pair_list_ints(int L)
{
    int64_t m = 0;
    for (int s = 0; s < kNumTileShapes; ++s) {
        const TileDims t = tile_dims(s);
        const int64_t tiles = (int64_t)((L + t.x - 1) / t.x) * ((L + t.y - 1) / t.y) * ((L + t.z - 1) / t.z);
        m = std::max(m, tiles * tile_list_stride(s));
    }
    return m;
}

int64_t ipart_count(int L) { return 2 * max_tiles(L) + blocks_for((int64_t)L * L * L); }
int64_t dpart_count(int L) { return 4 * max_tiles(L) + blocks_for((int64_t)L * L * L); }

}  // namespace pyro

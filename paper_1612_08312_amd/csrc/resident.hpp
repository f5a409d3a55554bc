// LDS-resident sweeps of small Ising lattices (resident.hip): limits, LDS
// layouts and launcher.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.hpp"

namespace pyro {

constexpr int kResidentMaxL = 16;  // N = 16 L^3 <= 65536: site indices fit in 16 bits
constexpr int kResidentThreads = 1024;
// Largest edge whose forest fits the LDS with 32-bit entries (140,608 of
// 163,840 B); the quad kernel runs up to it.
constexpr int kQuadMaxL = 13;

// Byte offsets in the dynamic LDS of a lattice of edge L: forest (2 B per
// site), reduction scratch, cell spin masks (2 B per cell), coin words, K4
// table.  At L = 16: 147,648 B.
struct ResidentLayout {
    uint32_t pf, red, smk, cw, k4, total;
};

__host__ __device__ inline ResidentLayout resident_layout(int L)
{
    const uint32_t ncell = (uint32_t)(L * L * L), N = 16u * ncell;
    ResidentLayout r;
    r.pf = 0;
    r.red = 2u * N;  // N is a multiple of 16: 8-byte aligned
    r.smk = r.red + 16u * 8u;
    r.cw = r.smk + ((2u * ncell + 3u) & ~3u);
    r.k4 = r.cw + 4u * ((N + 31u) / 32u);
    r.total = r.k4 + 64u;
    return r;
}

// Byte offsets in the dynamic LDS of the quad kernel: forest (4 B per site),
// sums (three sets of two words: magnetisation, aligned bonds), number of
// tied bonds, K4 table, coin words (whole FLIP blocks), union buffers (128
// words per wave), tied bonds (two words each), cell spin masks.  At L = 13:
// 161,788 B.
constexpr int kQuadTies = 512;
struct QuadLayout {
    uint32_t p, sums, ties_n, k4, cw, un, ties, smk, total;
};

__host__ __device__ inline QuadLayout quad_layout(int L)
{
    const uint32_t ncell = (uint32_t)(L * L * L), N = 16u * ncell;
    QuadLayout r;
    r.p = 0;
    r.sums = 4u * N;
    r.ties_n = r.sums + 24u;
    r.k4 = r.ties_n + 8u;
    r.cw = r.k4 + 64u;
    r.un = r.cw + 16u * ((N + 127u) / 128u);
    r.ties = r.un + 4u * 128u * (kResidentThreads / 64);
    r.smk = r.ties + 8u * kQuadTies;
    r.total = r.smk + ((2u * ncell + 3u) & ~3u);
    return r;
}

// Let the kernels for edges up to maxL take their LDS on the current device
// (done once per device; a failure is not kept).
hipError_t prepare_resident(int maxL);

// All `remaining` sweeps of every replica of the chain (each of edge
// L <= kResidentMaxL, no vacant site), one workgroup per replica, with the
// dynamic LDS of the largest edge maxL.  armed: the state to start from in
// place of the replica's own (one replica), or null.
hipError_t launch_resident_ising(const Chain &c, int maxL, const RepState *armed, hipStream_t st, const LaunchHook &hook);

}  // namespace pyro

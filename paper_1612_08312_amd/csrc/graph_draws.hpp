// Host-side tables of the shared Philox draws of a bond table's windows
// (Ising; used by the window pass of graph.hip).
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <new>
#include <vector>

namespace pyro {

constexpr int kDrawChunk = 1024;  // Philox blocks a window pass keeps in LDS at a time
struct DrawChunk {
    int64_t bond, block;  // the chunk's first bond and first block
};

// The distinct Philox blocks of each window's bonds, cut into chunks of at
// most kDrawChunk: chunk k holds the blocks from chunk[k].block and the bonds
// from chunk[k].bond on (up to those of chunk k + 1), window w the chunks from
// wchunk[w] on, and slot is each inside bond's byte in its chunk.  All empty
// when every bond draws its own.
struct DrawTables {
    std::vector<uint32_t> block;
    std::vector<DrawChunk> chunk;
    std::vector<int32_t> wchunk;
    std::vector<uint16_t> slot;
    bool shared() const { return !block.empty(); }
};

// wstart: [windows + 1] first bond of each window; id: position of each bond
// in the caller's table, ascending within a window, so the bonds of a block
// (16 consecutive positions) follow one another.  Blocks are shared where one
// serves two of a window's bonds or more on average (a lattice numbered row by
// row: 8 or more), else each bond draws its own.  So it does, with the same
// results, when the host has no memory for the tables.
inline DrawTables draw_tables(const std::vector<int64_t> &wstart, const std::vector<uint32_t> &id)
{
    const size_t nwin = wstart.size() - 1;
    const int64_t inside = wstart[nwin];
    auto opens = [&](size_t w, int64_t q) {
        return q == wstart[w] || id[(size_t)q] >> 4 != id[(size_t)q - 1] >> 4;
    };
    int64_t blocks = 0;
    for (size_t w = 0; w < nwin; ++w)
        for (int64_t q = wstart[w]; q < wstart[w + 1]; ++q) blocks += opens(w, q);
    if (blocks == 0 || 2 * blocks > inside) return DrawTables();
    try {
        DrawTables t;
        t.slot.resize((size_t)inside);
        t.block.reserve((size_t)blocks);
        t.wchunk.resize(nwin + 1);
        for (size_t w = 0; w < nwin; ++w) {
            t.wchunk[w] = (int32_t)t.chunk.size();
            int fill = kDrawChunk;  // blocks in the open chunk
            for (int64_t q = wstart[w]; q < wstart[w + 1]; ++q) {
                if (opens(w, q)) {
                    if (fill == kDrawChunk) {
                        t.chunk.push_back({q, (int64_t)t.block.size()});
                        fill = 0;
                    }
                    t.block.push_back(id[(size_t)q] >> 4);
                    ++fill;
                }
                t.slot[(size_t)q] = (uint16_t)(16 * (fill - 1) + (int)(id[(size_t)q] & 15u));
            }
        }
        t.wchunk[nwin] = (int32_t)t.chunk.size();
        t.chunk.push_back({inside, (int64_t)t.block.size()});
        return t;
    } catch (const std::bad_alloc &) {
        return DrawTables();
    }
}

}  // namespace pyro

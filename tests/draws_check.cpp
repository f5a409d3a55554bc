// Check of the shared-draw tables of a bond table's windows: every inside
// bond's byte is its own, chunks hold at most kDrawChunk blocks and windows
// their own chunks, blocks are shared exactly where the rule says, and with
// any one of the allocations failing the tables are left empty.  Exit status 0
// on success.
#include <stdio.h>
#include <stdlib.h>

#include <random>

#include "graph_draws.hpp"

static long left = -1;  // allocations until one fails; -1: none fails
static bool failed = false;
void *operator new(size_t n)
{
    if (left == 0) {
        failed = true;
        throw std::bad_alloc();
    }
    if (left > 0) --left;
    if (void *p = malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }

static int fail(const char *what, long long a, long long b)
{
    fprintf(stderr, "draws check failed: %s (%lld, %lld)\n", what, a, b);
    return 1;
}

static int check(const std::vector<int64_t> &ws, const std::vector<uint32_t> &id)
{
    const pyro::DrawTables t = pyro::draw_tables(ws, id);
    const size_t nwin = ws.size() - 1;
    int64_t blocks = 0;
    for (size_t w = 0; w < nwin; ++w)
        for (int64_t q = ws[w]; q < ws[w + 1]; ++q)
            blocks += q == ws[w] || id[(size_t)q] / 16 != id[(size_t)q - 1] / 16;
    if (t.shared() != (blocks > 0 && 2 * blocks <= ws[nwin])) return fail("rule", blocks, ws[nwin]);
    if (!t.shared()) return t.slot.empty() && t.chunk.empty() && t.wchunk.empty() ? 0 : fail("left over", 0, 0);
    if ((int64_t)t.block.size() != blocks) return fail("blocks", blocks, (long long)t.block.size());
    if (t.wchunk.size() != nwin + 1 || t.chunk.size() != (size_t)t.wchunk[nwin] + 1) return fail("sizes", 0, 0);
    for (size_t w = 0; w < nwin; ++w) {
        int64_t q = ws[w];
        for (int32_t c = t.wchunk[w]; c < t.wchunk[w + 1]; ++c) {
            const pyro::DrawChunk c0 = t.chunk[(size_t)c], c1 = t.chunk[(size_t)c + 1];
            if (c1.block - c0.block > pyro::kDrawChunk || c1.block <= c0.block) return fail("chunk", (long long)w, c);
            if (c0.bond != q) return fail("first bond", c0.bond, q);
            for (; q < c1.bond && q < ws[w + 1]; ++q) {
                const int64_t b = c0.block + t.slot[(size_t)q] / 16;
                if (b >= c1.block || t.block[(size_t)b] != id[(size_t)q] / 16 || t.slot[(size_t)q] % 16 != id[(size_t)q] % 16)
                    return fail("slot", q, t.slot[(size_t)q]);
            }
        }
        if (q != ws[w + 1]) return fail("window", (long long)w, q);
    }
    return 0;
}

int main()
{
    std::mt19937_64 rng(2024);
    // (windows, bonds per window, mean step between the positions of a window's bonds)
    const int cases[][3] = {{1, 1, 1}, {1, 16, 1}, {1, 16 * 1024, 1}, {1, 16 * 1024 + 1, 1}, {3, 40000, 1}, {5, 700, 2},
                            {4, 900, 7}, {4, 900, 8}, {4, 900, 9}, {6, 300, 40}, {3, 0, 1}};
    for (const auto &c : cases)
        for (int seed = 0; seed < 4; ++seed) {
            std::vector<int64_t> ws(1, 0);
            std::vector<uint32_t> id;
            for (int w = 0; w < c[0]; ++w) {
                const int64_t n = w % 3 == 1 && seed % 2 ? 0 : c[1];  // windows without bonds among them
                uint32_t at = (uint32_t)(rng() % 1000);
                for (int64_t k = 0; k < n; ++k) {
                    id.push_back(at);
                    at += c[2] == 1 ? 1 : 1 + (uint32_t)(rng() % (uint64_t)(2 * c[2] - 1));
                }
                ws.push_back((int64_t)id.size());
            }
            if (check(ws, id)) return 1;
            failed = true;
            for (long k = 0; failed; ++k) {  // the k-th allocation fails
                failed = false;
                left = k;
                const pyro::DrawTables t = pyro::draw_tables(ws, id);
                left = -1;
                if (failed && (t.shared() || !t.slot.empty() || !t.chunk.empty() || !t.wchunk.empty()))
                    return fail("tables after a failed allocation", k, 0);
            }
        }
    printf("draws ok\n");
    return 0;
}

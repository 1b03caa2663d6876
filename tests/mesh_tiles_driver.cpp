// CPU-only test driver: the interior-tile bitmaps of mesh launches (iso_bind.hpp) against their definition, tile by
// tile and rank by rank, on random boxes, entry sets, block lengths and both orders.  A bit that is set where a rank
// has no source would let a kernel read outside its buffer.  Ends with "mesh tiles ok".
#include <hip/hip_runtime.h>

#include <cstdio>
#include <random>

#include "iso_bind.hpp"

namespace iso {
thread_local int g_last_hip_error = 0;
}

int main() {
    std::mt19937 rng(7);
    auto pick = [&](int lo, int hi) { return (int)std::uniform_int_distribution<int>(lo, hi)(rng); };
    long set = 0, tiles = 0, cases = 0;
    for (; cases < 6000; ++cases) {
        const int d = pick(1, 4), big = pick(0, 3);
        std::vector<int32_t> dims, periodic;
        for (int j = 0; j < d; ++j) {
            dims.push_back(big == 0 && j == d - 1 ? pick(100, 700) : pick(1, 9));
            periodic.push_back(pick(0, 2) == 0);
        }
        const int s = pick(1, 6), span = pick(1, 4);
        std::vector<int32_t> rel;
        for (int q = 0; q < s * d; ++q) rel.push_back(pick(-span, span));
        iso::Comm c;
        if (iso::build_comm(d, dims.data(), periodic.data(), s, rel.data(), c) != ISO_SUCCESS) return 1;
        const uint32_t k = (uint32_t)pick(1, 5);
        std::vector<iso::HostEntry> ents(k);
        for (iso::HostEntry &he : ents) {
            he.de.ref = (uint32_t)pick(0, s - 1);
            uint32_t mask = 0;
            for (int j = 0; j < d; ++j)
                if (!periodic[(size_t)j] && pick(0, 1)) mask |= 1u << j;
            he.de.meta = 4u | (mask << 8);
        }
        const bool slot = pick(0, 1);
        const uint64_t chunks = (uint64_t)(pick(0, 2) ? pick(1, 20) : pick(1, 600)), p = (uint64_t)c.p;
        const uint64_t total = p * k * chunks, n_tiles = (total + iso::kThreads - 1) / iso::kThreads;
        if (total > 3000000) continue;
        const std::vector<uint32_t> bits = iso::mesh_interior_tiles(c, slot, ents.data(), k, total, chunks, p);
        if (bits.size() != (n_tiles + 31) / 32) return 2;
        auto has_sources = [&](uint64_t R) {
            for (const iso::HostEntry &he : ents) {
                uint64_t rem = R;
                for (int j = d - 1; j >= 0; --j) {
                    const int64_t r = (int64_t)(rem % (uint64_t)dims[(size_t)j]);
                    rem /= (uint64_t)dims[(size_t)j];
                    const int64_t from = r - c.c((int)he.de.ref, j);
                    if ((((he.de.meta >> 8) >> j) & 1u) && (from < 0 || from >= dims[(size_t)j])) return false;
                }
            }
            return true;
        };
        std::vector<bool> ok((size_t)p);
        for (uint64_t R = 0; R < p; ++R) ok[(size_t)R] = has_sources(R);
        for (uint64_t tl = 0; tl < n_tiles; ++tl, ++tiles) {
            const uint64_t u0 = tl * iso::kThreads, u1 = std::min<uint64_t>(u0 + iso::kThreads, total) - 1;
            uint64_t R0 = u0 / chunks, R1 = u1 / chunks;
            bool want = !slot || R0 / p == R1 / p;
            R0 = slot ? R0 % p : R0 / k;
            R1 = slot ? R1 % p : R1 / k;
            want = want && R0 / (uint64_t)dims[(size_t)d - 1] == R1 / (uint64_t)dims[(size_t)d - 1];
            for (uint64_t R = R0; want && R <= R1; ++R) want = ok[(size_t)R];
            const bool got = (bits[(size_t)(tl >> 5)] >> (tl & 31)) & 1u;
            set += got;
            if (got != want) {
                std::fprintf(stderr, "case %ld: tile %llu is %d\n", cases, (unsigned long long)tl, (int)got);
                return 3;
            }
        }
        for (uint64_t tl = n_tiles; tl < 32 * bits.size(); ++tl)
            if ((bits[(size_t)(tl >> 5)] >> (tl & 31)) & 1u) return 4;
    }
    if (set < tiles / 50 || set > tiles - tiles / 50) return 5;        // both kinds of tile occur
    std::printf("mesh tiles ok: %ld of %ld tiles interior\n", set, tiles);
    return 0;
}

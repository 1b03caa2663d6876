// CPU-only test driver: the interior bitmaps that the mesh shift kernel reads and the coordinates packed into its
// entries (iso_bind.hpp), unit by unit on random boxes.  A bit that is set where a move has no source would let the
// kernel read outside its buffer.  Ends with "mesh units ok".
#include <hip/hip_runtime.h>

#include <cstdio>
#include <random>

#include "iso_bind.hpp"

namespace iso {
thread_local int g_last_hip_error = 0;
}

int main() {
    std::mt19937 rng(11);
    auto pick = [&](int lo, int hi) { return (int)std::uniform_int_distribution<int>(lo, hi)(rng); };
    long set = 0, groups = 0, missed = 0, packed = 0;
    for (int cases = 0; cases < 4000; ++cases) {
        const int d = pick(1, 7), big = pick(0, 3);
        std::vector<int32_t> dims, periodic, rel;
        for (int j = 0; j < d; ++j) {
            dims.push_back(big == 0 && j == d - 1 ? pick(100, 700) : pick(1, 7 - d / 2));
            periodic.push_back(pick(0, 3) == 0);
        }
        const int s = pick(1, 6), span = pick(0, 9) ? pick(1, 3) : 40000;
        for (int q = 0; q < s * d; ++q) rel.push_back(pick(-span, span));
        iso::Comm c;
        if (iso::build_comm(d, dims.data(), periodic.data(), s, rel.data(), c) != ISO_SUCCESS) return 1;
        const uint32_t k = (uint32_t)pick(1, 5);
        std::vector<iso::HostEntry> ents(k);
        for (iso::HostEntry &he : ents) {
            he.de.ref = (uint32_t)pick(0, s - 1);
            uint32_t mask = 0;
            for (int j = 0; j < d; ++j)
                if (!periodic[(size_t)j] && c.c((int)he.de.ref, j) && pick(0, 1)) mask |= 1u << j;
            he.de.meta = 4u | (mask << 8);
            iso::DevEntry de = he.de;
            bool fits = d <= 6;
            for (int j = 0; j < d; ++j) fits = fits && (!((mask >> j) & 1u) || std::abs(c.c((int)he.de.ref, j)) < 32768);
            if (iso::pack_reference(c.can.data() + (size_t)de.ref * d, d, mask, de) != fits) return 2;
            const uint32_t words[3] = {de.units, de.ref, (uint32_t)de.last_offset};
            for (int j = 0; fits && j < d; ++j)
                if ((mask >> j) & 1u && (int16_t)(words[j / 2] >> (16 * (j & 1))) != c.c((int)he.de.ref, j)) return 3;
            packed += fits;
        }
        const bool slot = pick(0, 1);
        const uint64_t chunks = (uint64_t)(pick(0, 2) ? pick(1, 20) : pick(1, 600)), p = (uint64_t)c.p, total = p * k * chunks;
        if (total > 300000) continue;
        std::vector<uint8_t> ok((size_t)(p * k));
        for (uint64_t R = 0; R < p; ++R)
            for (uint32_t e = 0; e < k; ++e) {
                bool has = true;
                for (int j = 0; j < d; ++j) {
                    const int64_t from = (int64_t)(R / (uint64_t)c.inner[(size_t)j]) % dims[(size_t)j] - c.c((int)ents[e].de.ref, j);
                    has = has && (!((ents[e].de.meta >> (8 + j)) & 1u) || (from >= 0 && from < dims[(size_t)j]));
                }
                ok[(size_t)(R * k + e)] = has;
            }
        for (uint32_t log2 : {iso::kWaveLog2, iso::kTileLog2}) {
            const std::vector<uint32_t> bits = iso::mesh_interior_units(c, slot, ents.data(), k, log2, total, chunks, p);
            const uint64_t n = (total + (1u << log2) - 1) >> log2;
            if (bits.size() != (n + 31) / 32) return 4;
            if (log2 == iso::kTileLog2) {                      // no tile less than the line by line form finds
                const std::vector<uint32_t> lines = iso::mesh_interior_tiles(c, slot, ents.data(), k, total, chunks, p);
                for (size_t w = 0; w < bits.size(); ++w)
                    if (lines[w] & ~bits[w]) return 8;
            }
            for (uint64_t g = 0; g < 32 * bits.size(); ++g) {
                const bool got = (bits[(size_t)(g >> 5)] >> (g & 31)) & 1u;
                if (g >= n && got) return 5;
                if (g >= n) continue;
                bool all = true;
                for (uint64_t u = g << log2; u < std::min<uint64_t>(total, (g + 1) << log2); ++u) {
                    const uint64_t t = u / chunks, R = slot ? t % p : t / k, e = slot ? t / p : t % k;
                    all = all && ok[(size_t)(R * k + e)];
                }
                if (got && !all) return 6;
                set += got;
                missed += all && !got;
                ++groups;
            }
        }
    }
    if (set < groups / 20 || missed > groups / 20 || !packed) return 7;
    std::printf("mesh units ok: %ld of %ld groups interior, %ld more could be\n", set, groups, missed);
    return 0;
}

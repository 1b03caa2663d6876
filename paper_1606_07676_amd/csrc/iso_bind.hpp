// Binding of a schedule to device buffers: turns a plan plus a block layout
// (sizes and displacements of the s blocks in a rank's send and receive rows)
// into the device table of block index maps and the list of kernel launches.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <initializer_list>
#include <memory>
#include <numeric>
#include <type_traits>
#include <vector>

#include "iso.h"
#include "iso_kernels.hpp"
#include "iso_plan.hpp"

namespace iso {

extern thread_local int g_last_hip_error;

constexpr uint64_t kLastLevelCacheBytes = uint64_t(256) << 20;
constexpr uint32_t kMaxUnits = 0xFFF00000u;   // flat 32-bit work index per launch

#define ISO_HIP_TRY(expr)                              \
    do {                                               \
        hipError_t err_ = (expr);                      \
        if (err_ != hipSuccess) {                      \
            iso::g_last_hip_error = (int)err_;         \
            (void)hipGetLastError();                   \
            return ISO_ERR_HIP;                        \
        }                                              \
    } while (0)

enum LaunchKernel { kShiftKernel = 0, kVectorKernel = 1, kBlockKernel = 2, kMeshShiftKernel = 3, kDeliverKernel = 4, kStagedRoundKernel = 5, kChainKernel = 6 };

struct Launch {
    int kernel;            // LaunchKernel
    uint32_t grid;
    bool lds_table;
    bool mesh;
    int policy;            // kStreamLoads, kPlainStores, kBySize (see cache_policy)
    bool tail;             // regular kernels: the last unit of a block overlaps the one before it
    bool uniform_waves;    // shift kernel, 16-byte units, blocks a multiple of 64 units: one block per wavefront
    bool eighths;          // one contiguous eighth of the tiles per XCD, whatever page_resonant says
    int vector_dims;       // vector kernel: dimensions its VectorEntry records hold (0: the general tables)
    bool small_and_large;  // block kernel: blocks on both sides of kSmallUnits in the launch
    bool block_groups;     // block kernel: ranks taken in groups of kBlockGroup
    int round;             // the plan's round this launch belongs to (a large round is split over several launches)
    uint32_t dyn_lds;      // bytes of dynamic LDS (the kernels of the staged schedule: their tile)

    ShiftArgs shift;
    VectorArgs vec;
    BlockArgs block;
    MeshArgs mesh_shift;
    DeliverArgs deliver;
    StagedRoundArgs staged;
    bool by_bytes;         // deliver kernel: blocks of any size (deliver_bytes_kernel)
    uint32_t tile_units;   // the staged schedule's kernels: kTileUnits or kSmallTileUnits
    ChainHead chain;       // chain kernel: its hops in the request's table
    const ChainArgs *chain_by_value;      // or BoundRequest::chain, where there is no table
    uint32_t chain_width;  // its unit width, where not the request's (vector kernel: blocks of one size among others)
    uint64_t outside_units;               // mesh: units of wavefronts or tiles not marked interior (see rounds_move_faster)
    bool entry_major, vector_round;       // see launch_flags
    int way;               // vector kernel: its WAY
    uint32_t pull;
    uint64_t bytes_read, bytes_written;   // of blocks (see iso_start_info_t)
    uint32_t threads;      // per workgroup, where not kThreads (chain kernel)
};

// Sizes and displacements (bytes) of the s blocks inside one rank's send and
// receive rows, and the distance between consecutive ranks' rows.
struct Layout {
    std::vector<uint64_t> size, send_displ, recv_displ;
    uint64_t send_extent = 0, recv_extent = 0;
    uint64_t send_span = 0, recv_span = 0;    // first to last byte of one rank's blocks
    bool slot_major = false;                  // one plane per neighbour: consecutive ranks' blocks i are
                                              // size[i] bytes apart (regular blocks: [s][p][m]); the
                                              // extents then only describe the allgather's send rows
};

struct Range {
    uintptr_t lo;
    size_t len;
};

inline bool overlap(const Range &a, const Range &b) {
    if (!a.len || !b.len) return false;
    return a.lo < b.lo + b.len && b.lo < a.lo + a.len;
}

// The range must lie inside one device allocation known to the HIP runtime.
inline int check_device_range(const void *ptr, size_t len) {
    if (!len) return ISO_SUCCESS;
    if (!ptr) return ISO_ERR_ARG;
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    hipError_t e = hipMemGetAddressRange(&base, &size, (hipDeviceptr_t)ptr);
    if (e != hipSuccess) {
        g_last_hip_error = (int)e;
        (void)hipGetLastError();
        return ISO_ERR_POINTER;
    }
    const uintptr_t b = (uintptr_t)base, q = (uintptr_t)ptr;
    if (q < b || q - b > size || len > size - (q - b)) return ISO_ERR_POINTER;
    return ISO_SUCCESS;
}

// log2 of the widest power of two (<= 16) that divides all the values: the access width of the
// plain reference copy, which keeps naturally aligned accesses
inline uint32_t common_alignment_log2(std::initializer_list<uint64_t> values) {
    uint64_t bits = 0;
    for (uint64_t v : values) bits |= v;
    uint32_t l = 4;
    while (l > 0 && (bits & ((uint64_t(1) << l) - 1))) --l;
    return l;
}

// log2 of the unit width for a block of `size` >= 1 bytes: the largest power of two that is
// at most 16 and at most the size (the last unit of a block overlaps its predecessor when the
// width does not divide the size; addresses need no alignment)
inline uint32_t unit_log2_of(uint64_t size) {
    uint32_t l = 4;
    while (l > 0 && (uint64_t(1) << l) > size) --l;
    return l;
}

inline uint64_t align16(uint64_t x) { return (x + 15) & ~uint64_t(15); }

// Slot-major workspace: slot w holds one block per rank, p * size_w bytes, slots
// back to back (each start rounded up to 16 bytes).  Dense streams per entry
// whatever the block size is.
struct WorkLayout {
    std::vector<uint64_t> size, offset;
    uint64_t bytes = 0;
};

inline WorkLayout work_layout(const Plan &pl, const Layout &lay) {
    WorkLayout w;
    w.size.assign((size_t)pl.work_slots, 0);
    w.offset.assign((size_t)pl.work_slots, 0);
    const uint64_t uniform = lay.size.empty() ? 0 : lay.size[0];
    for (const Round &r : pl.rounds)
        for (const iso_plan_entry_t &e : r.entries)
            if (e.dst_buf == ISO_BUF_WORK) {
                const uint64_t sz = (pl.op == ISO_OP_ALLTOALL && e.neighbor >= 0) ? lay.size[(size_t)e.neighbor]
                                                                                  : uniform;
                w.size[(size_t)e.dst_slot] = std::max(w.size[(size_t)e.dst_slot], sz);
            }
    for (int q = 0; q < pl.work_slots; ++q) {
        w.offset[(size_t)q] = w.bytes;
        w.bytes += align16((uint64_t)pl.comm.p * w.size[(size_t)q]);
    }
    return w;
}

// Blocks that sit at a rank stride that is a multiple of 4 KiB and cover only part of the offsets
// modulo 4 KiB (config 3: 1 KiB blocks in 12 KiB rows) use a fraction of what the address bits
// below 4 KiB select in the memory system, whichever ranks are in flight.  How the eight XCDs'
// streams lie to each other then matters: measured on plain strided copies of 256 B - 2 KiB
// pieces, strides that are multiples of 4 KiB run 4 - 26 % faster when every XCD sweeps its own
// contiguous eighth of the tiles than with interleaved runs (multiples of 8 KiB gain most), all
// other strides are indifferent to it (within 1 %) and dense or page-covering launches prefer runs.
// `sides`: per entry its (address, stride, block size) on the source and on the destination side.
struct Side {
    uint64_t addr, stride, size;
};

inline bool page_resonant(const std::vector<Side> &sides) {
    bool marked[256] = {};                     // 16-byte granules of a 4 KiB page
    bool any = false;
    for (const Side &sd : sides) {
        if (!sd.size || !sd.stride || (sd.stride & 4095u)) continue;
        any = true;
        const uint64_t lo = (sd.addr & 4095u) >> 4, n = std::min<uint64_t>(256, (sd.size + (sd.addr & 15u) + 15) >> 4);
        for (uint64_t q = 0; q < n; ++q) marked[(lo + q) & 255u] = true;
    }
    if (!any) return false;
    for (bool b : marked)
        if (!b) return true;
    return false;
}

inline void set_grid(Launch &l, uint32_t total, uint32_t k, bool eighths) {
    const uint32_t n_tiles = (uint32_t)(((uint64_t)total + kThreads - 1) / kThreads);
    // Runs of 128 tiles (512 KiB of units) per XCD: measured best over the five workloads
    // (no runs: -5 % where the rank stride is a multiple of 4 KiB; runs of 512 tiles or more:
    // -8 % and worse, the last incomplete span leaves XCDs idle).
    uint32_t run_log2 = 7;
    // (the staged schedule's kernels: a tile is 32 KiB and there are few of them; with runs of 128 a grid
    // padded to whole spans had up to 18 % workgroups without a tile, which cost 7 % at 16-byte blocks; runs
    // of 4 ... 32 tiles measure alike)
    if (l.kernel == kStagedRoundKernel || l.kernel == kDeliverKernel) run_log2 = 3;
    while (run_log2 > 0 && (8u << run_log2) > n_tiles) --run_log2;
    const uint32_t span = 8u << run_log2;
    l.grid = (uint32_t)((((uint64_t)n_tiles + span - 1) / span) * span);
    const uint32_t per_xcd = (n_tiles + 7) / 8;
    if (eighths && n_tiles >= 64) {            // one contiguous eighth per XCD (balanced for any tile count)
        run_log2 = kEighths;
        l.grid = per_xcd * 8;
    }
    const uint32_t flags = launch_flags(run_log2, l.entry_major, l.pull, l.vector_round);
    l.lds_table = k <= kLdsEntries;
    switch (l.kernel) {
        case kStagedRoundKernel: l.staged.n_tiles = n_tiles; l.staged.more |= flags; break;
        case kDeliverKernel: l.deliver.n_tiles = n_tiles; l.deliver.more |= flags; break;
        case kVectorKernel: l.vec.total = total; l.vec.k = k; l.vec.more |= flags; break;
        case kBlockKernel: l.block.total = total; l.block.k = k; l.block.more |= flags; break;
        case kMeshShiftKernel: l.mesh_shift.total = total; l.mesh_shift.k = k; l.mesh_shift.more |= flags; break;
        default: l.shift.total = total; l.shift.k = k; l.shift.more |= flags; l.shift.map = TileMap{n_tiles, run_log2, per_xcd};
    }
}

// Which instantiation runs a launch, and the argument struct it takes: resolved once per launch,
// used both for plain launches and for the kernel nodes of a request's graph.
struct KernelRef {
    const void *func;
    const void *arg;
};

// f(std::integral_constant<int, policy>) for the launch's cache policy: 16-byte units only (narrower ones are
// always loaded through the caches and stored plainly).
template <typename V, typename F>
KernelRef with_policy(const Launch &l, F &&f) {
    if constexpr (sizeof(V) == 16) {
        switch (l.policy) {
            case kStreamLoads: return f(std::integral_constant<int, kStreamLoads>());
            case kPlainStores: return f(std::integral_constant<int, kPlainStores>());
            case kStreamLoads | kPlainStores: return f(std::integral_constant<int, kStreamLoads | kPlainStores>());
            default: break;
        }
    }
    return f(std::integral_constant<int, 0>());
}

template <typename V, int D, bool TAIL, int WAY>
KernelRef select_way(const Launch &l) {
    const auto form = [&](auto pol) -> KernelRef {
        if constexpr (sizeof(V) == 16) {
            if (l.uniform_waves) return {(const void *)&vector_round_uniform_kernel<D, pol(), WAY>, &l.vec};
        }
        return {(const void *)&vector_round_kernel<V, D, true, pol(), TAIL, WAY>, &l.vec};
    };
    if constexpr (WAY == kStrides) {
        if (l.vec.per) return {(const void *)&push_round_kernel<V, D, TAIL, WAY>, &l.vec};
    }
    if constexpr (sizeof(V) == 16 && !(WAY & kStrides)) {           // (kStrides: an allgather, which loads through the caches)
        if (l.policy & kStreamLoads) return form(std::integral_constant<int, kStreamLoads>());
    }
    if constexpr (WAY == kStrides) {                                // (less than a sector: no whole wavefronts)
        if (l.policy & kPlainStores) return {(const void *)&vector_round_kernel<V, D, true, kPlainStores, TAIL, WAY>, &l.vec};
    }
    return form(std::integral_constant<int, 0>());
}

// The s-exchange with VectorEntry records (see vector_launch).
template <typename V, int D, bool TAIL>
KernelRef select_vector(const Launch &l) {
    if constexpr (sizeof(V) == 16) {                                // (all_hops_in_one_launch)
        switch (l.way) {
            case kStops: return select_way<V, D, TAIL, kStops>(l);
            case kStrides: return select_way<V, D, TAIL, kStrides>(l);
            case kStops | kMesh: return select_way<V, D, TAIL, kStops | kMesh>(l);
            case kStrides | kMesh: return select_way<V, D, TAIL, kStrides | kMesh>(l);
            default: break;
        }
    }
    if (l.way == kMesh) return select_way<V, D, TAIL, kMesh>(l);
    if (l.vec.per) return {(const void *)&push_round_kernel<V, D, TAIL>, &l.vec};
    return select_way<V, D, TAIL, 0>(l);
}

template <typename V, bool LDS, bool TAIL>
KernelRef select_regular(const Launch &l) {
    if (l.kernel == kChainKernel) {
        const bool one = l.chain.n_units <= kChainThreads;         // a unit per lane
        if (l.chain_by_value) {
            if (one) return {(const void *)&chain_kernel<V, TAIL, 1, ChainArgs>, l.chain_by_value};
            return {(const void *)&chain_kernel<V, TAIL, kChainUnitsPerLane, ChainArgs>, l.chain_by_value};
        }
        if (one) return {(const void *)&chain_kernel<V, TAIL, 1, ChainHead>, &l.chain};
        return {(const void *)&chain_kernel<V, TAIL, kChainUnitsPerLane, ChainHead>, &l.chain};
    }
    if (l.kernel == kVectorKernel) {
        if constexpr (LDS) {
            if (l.vector_dims == 3) return select_vector<V, 3, TAIL>(l);
            if (l.vector_dims == kVectorDims) return select_vector<V, kVectorDims, TAIL>(l);
        }
        return {(const void *)&vector_round_kernel<V, 0, LDS, 0, TAIL>, &l.vec};
    }
    if (l.kernel == kMeshShiftKernel)
        return with_policy<V>(l, [&](auto pol) -> KernelRef {
            return {(const void *)&mesh_shift_round_kernel<V, LDS, pol(), TAIL>, &l.mesh_shift};
        });
    if (l.shift.k_all) return {(const void *)&shift_push_kernel<V, TAIL>, &l.shift};
    return with_policy<V>(l, [&](auto pol) -> KernelRef {
        if constexpr (sizeof(V) == 16) {
            if (l.uniform_waves) {
                if (l.shift.grouped) return {(const void *)&shift_round_uniform_kernel<pol(), true>, &l.shift};
                return {(const void *)&shift_round_uniform_kernel<pol()>, &l.shift};
            }
            if (l.shift.grouped) return {(const void *)&shift_round_kernel<V, LDS, pol(), TAIL, true>, &l.shift};
        }
        return {(const void *)&shift_round_kernel<V, LDS, pol(), TAIL>, &l.shift};
    });
}

template <typename V>
KernelRef select_width(const Launch &l) {
    if constexpr (sizeof(V) > 1) {
        if (l.tail) {                     // the unit width does not divide the block size
            if (l.lds_table) return select_regular<V, true, true>(l);
            return select_regular<V, false, true>(l);
        }
    }
    if (l.lds_table) return select_regular<V, true, false>(l);
    return select_regular<V, false, false>(l);
}

inline KernelRef select_block_hops(const Launch &l) {
    if (l.vector_dims == 3) return {(const void *)&block_round_kernel<true, true, kPlainStores, false, 3>, &l.block};
    return {(const void *)&block_round_kernel<true, true, kPlainStores, false, kVectorDims>, &l.block};
}

template <bool LDS, bool MESH>
KernelRef select_block(const Launch &l) {
    const auto form = [&](auto pol) -> KernelRef {
        if (l.block_groups) return {(const void *)&block_round_kernel<LDS, MESH, pol(), true>, &l.block};
        return {(const void *)&block_round_kernel<LDS, MESH, pol()>, &l.block};
    };
    if constexpr (!MESH) {
        if (l.policy == kBySize) return form(std::integral_constant<int, kBySize>());
    }
    if (l.policy == kStreamLoads) return form(std::integral_constant<int, kStreamLoads>());
    if (l.policy == kPlainStores) return form(std::integral_constant<int, kPlainStores>());
    return form(std::integral_constant<int, 0>());
}

template <typename V>
KernelRef select_deliver_bytes(const Launch &l) {
    return with_policy<V>(l, [&](auto pol) -> KernelRef {
        constexpr uint32_t kSmall = kSmallTileUnits / kThreads, kLarge = kTileUnits / kThreads;
        if (l.tile_units == kSmallTileUnits) return {(const void *)&deliver_bytes_kernel<V, pol(), kSmall>, &l.deliver};
        return {(const void *)&deliver_bytes_kernel<V, pol(), kLarge>, &l.deliver};
    });
}

template <typename V>
KernelRef select_staged_round(const Launch &l) {
    const auto form = [&](auto pol, auto tail, auto two) -> KernelRef {
        constexpr uint32_t kSmall = kSmallTileUnits / kThreads, kLarge = kTileUnits / kThreads;
        if (l.tile_units == kSmallTileUnits) return {(const void *)&staged_round_kernel<V, pol(), kSmall, tail(), two()>, &l.staged};
        return {(const void *)&staged_round_kernel<V, pol(), kLarge, tail(), two()>, &l.staged};
    };
    return with_policy<V>(l, [&](auto pol) -> KernelRef {
        if constexpr (sizeof(V) > 1) {
            if (l.tail) return l.staged.inner2 ? form(pol, std::true_type(), std::true_type()) : form(pol, std::true_type(), std::false_type());
        }
        return l.staged.inner2 ? form(pol, std::false_type(), std::true_type()) : form(pol, std::false_type(), std::false_type());
    });
}

template <typename V>
KernelRef select_tile(const Launch &l) {
    return l.kernel == kStagedRoundKernel ? select_staged_round<V>(l) : select_deliver_bytes<V>(l);
}

inline KernelRef select_kernel(int vector_bytes, const Launch &l) {
    if (l.kernel == kStagedRoundKernel || (l.kernel == kDeliverKernel && l.by_bytes)) {
        switch (vector_bytes) {
            case 16: return select_tile<vec16_t>(l);
            case 8:  return select_tile<vec8_t>(l);
            case 4:  return select_tile<uint32_t>(l);
            case 2:  return select_tile<uint16_t>(l);
            default: return select_tile<uint8_t>(l);
        }
    }
    if (l.kernel == kDeliverKernel)                      // blocks of whole 16-byte units
        return with_policy<vec16_t>(l, [&](auto pol) -> KernelRef {
            constexpr uint32_t kSmall = kSmallTileUnits / kThreads, kLarge = kTileUnits / kThreads;
            return l.tile_units == kSmallTileUnits ? KernelRef{(const void *)&deliver_kernel<vec16_t, pol(), kSmall>, &l.deliver}
                                                   : KernelRef{(const void *)&deliver_kernel<vec16_t, pol(), kLarge>, &l.deliver};
        });
    if (l.kernel == kBlockKernel) {
        if (l.way) return select_block_hops(l);
        if (l.mesh) return l.lds_table ? select_block<true, true>(l) : select_block<false, true>(l);
        return l.lds_table ? select_block<true, false>(l) : select_block<false, false>(l);
    }
    switch (l.chain_width ? (int)l.chain_width : vector_bytes) {
        case 16: return select_width<vec16_t>(l);
        case 8:  return select_width<vec8_t>(l);
        case 4:  return select_width<uint32_t>(l);
        case 2:  return select_width<uint16_t>(l);
        default: return select_width<uint8_t>(l);
    }
}

inline int enqueue(int vector_bytes, const Launch &l, hipStream_t stream) {
    const KernelRef k = select_kernel(vector_bytes, l);
    void *args[1] = {const_cast<void *>(k.arg)};
    ISO_HIP_TRY(hipLaunchKernel(k.func, dim3(l.grid), dim3(l.threads ? l.threads : kThreads), args, l.dyn_lds, stream));
    return ISO_SUCCESS;
}

struct BoundRequest {
    Plan plan;
    iso_request_info_t info{};
    void *dev_table = nullptr;         // owned (hipMalloc) unless the request was bound to a StaticArena
    std::vector<Launch> launches;          // what iso_start_range counts through
    std::vector<Launch> start_launches;    // what iso_start enqueues instead, where that differs (see merge_rounds)
    std::unique_ptr<ChainArgs> chain;      // arguments of the chain kernel, where it takes them by value

    const std::vector<Launch> &start_list() const { return start_launches.empty() ? launches : start_launches; }
};

// Device memory that the library already holds, for binding a schedule without allocating:
// the table of block index maps goes to `table` (written by table_store_kernel launches on
// `stream`, ordered before the rounds that read it), and the caller of bind_request passes the
// rest of the arena as the workspace.  Nothing is allocated, copied or freed.
struct StaticArena {
    unsigned char *table;              // device address, 16-byte aligned
    size_t table_bytes;                // for entries, residues and the rest; kArenaTorusBytes more are there
    hipStream_t stream;
};

constexpr size_t kArenaTorusBytes = 512;
static_assert(sizeof(TorusDims) <= kArenaTorusBytes, "room behind the table");

inline int store_table(const StaticArena &arena, size_t at, const void *host, size_t bytes) {
    // `at` and `bytes` are multiples of 4: every part of the table is an array of 32-bit words or of DevEntry
    const uint32_t *w = (const uint32_t *)host;
    size_t words = bytes / 4, done = 0;
    while (done < words) {
        TableChunk ch;
        ch.dst = (uint32_t *)(arena.table + at) + done;
        ch.n = (uint32_t)std::min<size_t>(kStoreWords, words - done);
        ch.reserved = 0;
        std::memcpy(ch.words, w + done, (size_t)ch.n * 4);
        hipLaunchKernelGGL(table_store_kernel, dim3((ch.n + kThreads - 1) / kThreads), dim3(kThreads), 0,
                           arena.stream, ch);
        ISO_HIP_TRY(hipGetLastError());
        done += ch.n;
    }
    return ISO_SUCCESS;
}

// One entry of a launch on the host: the device entry, the block's size, and for the staged schedule's last
// launch the dimension the entry moves along and the receive block it writes.
struct HostEntry {
    DevEntry de;
    uint64_t size;
    int dim, dst_buf, dst_slot, neighbor;
    // launches that take blocks through all their hops (join_hops)
    uint32_t moves;        // of the plan that the entry stands for
    uint32_t along;        // the dimensions that it moves along, of its neighbour's vector
    uint64_t way;          // VectorEntry::way
};

// Mesh shift launches of equal blocks: the ranks where every one of the entries finds its source, as runs of
// consecutive ranks, f(first, count).  Coordinates that do: r_l - c_l in [0, p_l) for all masked dimensions l of all
// entries.  A run holds the ranks that share the coordinates before dimension L, lie inside L's bounds, and all
// dimensions behind it; L is the last bounded dimension (none: all ranks are one run), or with `by_line` the last one.
template <typename F>
void for_interior_runs(const Comm &c, const HostEntry *ents, uint32_t k, bool by_line, F &&f) {
    std::vector<int64_t> lo((size_t)c.d, 0), hi((size_t)c.d), at;
    int last = by_line ? c.d - 1 : -1;
    for (int j = 0; j < c.d; ++j) {
        hi[(size_t)j] = c.dims[(size_t)j];
        for (uint32_t q = 0; q < k; ++q) {
            const DevEntry &de = ents[q].de;
            const int64_t cl = c.c((int)de.ref, j);
            if (!(((de.meta >> 8) >> j) & 1u) || !cl) continue;
            lo[(size_t)j] = std::max<int64_t>(lo[(size_t)j], cl);
            hi[(size_t)j] = std::min<int64_t>(hi[(size_t)j], (int64_t)c.dims[(size_t)j] + cl);
            last = std::max(last, j);
        }
        if (lo[(size_t)j] >= hi[(size_t)j]) return;
    }
    if (last < 0) {
        f((uint64_t)0, (uint64_t)c.p);
        return;
    }
    const uint64_t run = (uint64_t)((hi[(size_t)last] - lo[(size_t)last]) * c.inner[(size_t)last]);
    uint64_t first = 0;
    for (int j = 0; j <= last; ++j) first += (uint64_t)(lo[(size_t)j] * c.inner[(size_t)j]);
    at = lo;
    for (bool more = true; more;) {                            // the coordinates before L step through their bounds
        f(first, run);
        more = false;
        for (int j = last - 1; j >= 0 && !more; --j) {
            const uint64_t inner = (uint64_t)c.inner[(size_t)j];
            more = ++at[(size_t)j] < hi[(size_t)j];
            if (more) first += inner;
            else first -= (uint64_t)(hi[(size_t)j] - 1 - lo[(size_t)j]) * inner, at[(size_t)j] = lo[(size_t)j];
        }
    }
}

constexpr uint32_t kWaveLog2 = 6, kTileLog2 = 8;
static_assert(1 << kTileLog2 == kThreads, "a tile");

// Sets the bits of the groups of 2^group_log2 units that lie inside [u0, u1); the last group may be a part.
inline void mark_groups(std::vector<uint32_t> &bits, uint32_t group_log2, uint64_t total, uint64_t u0, uint64_t u1) {
    const uint64_t fill = (uint64_t(1) << group_log2) - 1;
    const uint64_t w0 = (u0 + fill) >> group_log2, w1 = (u1 == total ? total + fill : u1) >> group_log2;
    if (w0 >= w1) return;
    const size_t first = (size_t)(w0 >> 5), last = (size_t)((w1 - 1) >> 5);
    const uint32_t from = ~0u << (w0 & 31), to = ~0u >> (31 - ((w1 - 1) & 31));
    if (first == last) {
        bits[first] |= from & to;
        return;
    }
    bits[first] |= from;
    std::fill(bits.begin() + (ptrdiff_t)first + 1, bits.begin() + (ptrdiff_t)last, ~0u);
    bits[last] |= to;
}

// One bit per tile of kThreads units, set where every rank of the tile has a source for every entry of the launch and
// all of them share all coordinates but the last: by its definition, line by line along the last dimension, a part of what
// mesh_interior_units finds, whose tests are held against it.
inline std::vector<uint32_t> mesh_interior_tiles(const Comm &c, bool slot_major, const HostEntry *ents, uint32_t k,
                                                 uint64_t total, uint64_t chunks, uint64_t p) {
    const uint64_t unit_per_rank = slot_major ? chunks : chunks * k;
    std::vector<uint32_t> bits((size_t)(((total + kThreads - 1) / kThreads + 31) / 32), 0u);
    for_interior_runs(c, ents, k, true, [&](uint64_t first, uint64_t n) {
        for (uint64_t e = 0; e < (slot_major ? k : 1); ++e)
            mark_groups(bits, kTileLog2, total, (e * p + first) * unit_per_rank, (e * p + first + n) * unit_per_rank);
    });
    return bits;
}

// What the mesh shift kernel reads: one bit per 2^group_log2 units (a wavefront or a tile), set where all their moves
// have a source.  On slot-major buffers a wavefront's units belong to one entry, whose own bounds count.
inline std::vector<uint32_t> mesh_interior_units(const Comm &c, bool slot_major, const HostEntry *ents, uint32_t k,
                                                 uint32_t group_log2, uint64_t total, uint64_t chunks, uint64_t p) {
    const uint64_t unit_per_rank = slot_major ? chunks : chunks * k;
    std::vector<uint32_t> bits((size_t)((((total - 1) >> group_log2) + 32) / 32), 0u);
    for (uint32_t e = 0; e < (slot_major ? k : 1); ++e)
        for_interior_runs(c, ents + e, slot_major ? 1 : k, false, [&](uint64_t first, uint64_t n) {
            mark_groups(bits, group_log2, total, (e * p + first) * unit_per_rank, (e * p + first + n) * unit_per_rank);
        });
    return bits;
}

// How finely: by the wavefront where a run holds few tiles, of which the first and the last are lost to tiles.
// From 32 tiles on that is 3 % of a launch, and the bitmap's size is what an init call pays for (64^3 box, 200 B:
// 600 KiB by the wavefront in its two lists).
inline uint32_t interior_group_log2(const Comm &c, bool slot_major, const HostEntry *ents, uint32_t k, uint64_t chunks) {
    uint64_t run = 0;
    for_interior_runs(c, ents, slot_major ? 1 : k, false, [&](uint64_t, uint64_t n) { run = n; });
    return run * (slot_major ? chunks : chunks * k) < 32 * kThreads ? kWaveLog2 : kTileLog2;
}

// The record of one entry of the staged schedule's last launch.
inline DeliverEntry make_deliver_entry(const Comm &c, const HostEntry &he) {
    DeliverEntry x{};
    x.src = he.de.src;
    x.src_stride = he.de.src_stride;
    x.slot = (uint32_t)he.dst_slot;
    const uint32_t inner = he.dim < 0 ? 1u : (uint32_t)c.inner[(size_t)he.dim];
    x.pj = he.dim < 0 ? 1u : (uint32_t)c.dims[(size_t)he.dim];
    x.shift = he.dim < 0 ? 0u : he.de.shift;
    x.back = x.shift * inner;
    x.wrap = x.pj * inner;
    x.d_inner = make_fastdiv(inner);
    x.d_pj = make_fastdiv(x.pj);
    return x;
}

// Binds a schedule to buffers: checks the buffers, builds the device table and the launch
// list.  bind_request below runs the steps in order.
// With `arena` the table is placed there instead of in an allocation of its own, and the workspace is
// taken to be the library's own memory (no look-up of its allocation); ISO_ERR_SCRATCH if either does not fit.
class Binder {
    // one division among a launch's constants
    static void put(uint32_t divisor, uint32_t &mul, uint32_t &shifts, uint32_t byte) {
        const FastDiv f = make_fastdiv(divisor);
        mul = f.mul;
        shifts |= shift_byte(f) << (8 * byte);
    }

public:
    Binder(BoundRequest &request, const Plan &plan, const Comm &comm, const Layout &layout, const void *send, void *recv,
           void *work, size_t work_bytes, const StaticArena *static_arena)
        : rq(request), c(comm), lay(layout), sendbuf(send), recvbuf(recv), workspace(work),
          workspace_bytes(work_bytes), arena(static_arena), pl(plan), op(plan.op),
          p((uint64_t)comm.p), s((size_t)comm.s), inf(request.info), wl(work_layout(plan, layout)) {}

    int run() {
        int st = describe_and_check();
        if (st != ISO_SUCCESS || inf.delivered_bytes == 0) return st;       // nothing to move: no launches
        rounds_as_launched();
        if ((st = host_entries()) != ISO_SUCCESS) return st;
        bits_by_wave = !arena || wave_bits_cost_no_launch();
        const bool merges = pl.algorithm == ISO_ALG_COMBINED;
        const bool chains = merges || pl.algorithm == ISO_ALG_COMBINED_BYDIM || pl.algorithm == ISO_ALG_COMBINED_STAGED;
        const uint64_t launches = launches_of_rounds(merges);
        size_t entries = 0;
        for (const std::vector<HostEntry> &ents : rounds) entries += ents.size();
        table.reserve(entries * (merges && !arena ? 2 : 1));
        if (!arena) {                                    // the list that iso_start_range and graphs take
            if ((st = bind_rounds()) != ISO_SUCCESS) return st;
            n_listed = pending.size();
        }
        const bool by_size = all_hops_by_size(), hops = by_size || all_hops_in_one_launch(launches);
        if (chains && (!hops || hops_launches() > 1) && chain_launch(launches)) return upload();
        if (two_staged_rounds()) {
            join_two_rounds();
            st = bind_rounds();
            return st == ISO_SUCCESS ? upload() : st;
        }
        const bool star = !hops && star_in_one_launch(launches);
        const bool rows = !hops && !star && rows_in_one_launch();
        if (hops || rows || star || (merges && launches < bound_rounds.size())) {
            const size_t n_entries = table.size(), n_prefixes = prefixes.size();
            if (hops) join_hops();
            if (by_size) split_by_size();
            else if (star) join_star();
            else if (rows) defer_last_hops();
            merge_rounds();
            st = bind_rounds();
            if (c.mesh && !hops && !arena && st == ISO_SUCCESS && rounds_move_faster()) {
                pending.resize(n_listed);
                table.resize(n_entries);
                prefixes.resize(n_prefixes);
            }
        } else if (arena) {
            st = bind_rounds();
        }
        return st == ISO_SUCCESS ? upload() : st;
    }

private:
    BoundRequest &rq;
    const Comm &c;
    const Layout &lay;
    const void *sendbuf;
    void *recvbuf, *workspace;
    size_t workspace_bytes;
    const StaticArena *arena;
    const Plan &pl;
    const int op;
    const uint64_t p;
    const size_t s;
    iso_request_info_t &inf;
    const WorkLayout wl;

    struct BoundRound { int kind, dim, of; const Round *whole; };
    std::vector<BoundRound> bound_rounds;         // the plan's rounds as launched (of: its index there; whole: all its
                                                  // entries, else those along `dim`)
    std::vector<std::vector<HostEntry>> rounds;   // their entries that move something
    bool uniform = true;                          // all these entries have `size0` bytes
    uint64_t size0 = 0;
    uint32_t min_log2 = 4;                        // the narrowest unit width among them
    bool bits_by_wave = true;                     // mesh: interior bits by the wavefront where that is the better one

    std::vector<DevEntry> table;
    std::vector<uint32_t> prefixes;               // what launches read besides their entries (see upload)
    struct Pending { size_t first_entry, first_prefix; Launch l; };
    std::vector<Pending> pending;
    bool all_hops = false;                        // the round is join_hops's
    bool one_size = false;                        // the rounds are split_by_size's
    int second_dim = -1;                          // the first round is join_two_rounds's
    std::vector<uint64_t> large_sizes;
    size_t n_listed = 0;                          // of these: rq.launches; the rest are rq.start_launches

    int bind_rounds() {
        int st;
        for (size_t ri = 0; ri < bound_rounds.size(); ++ri)
            for (size_t done = 0; done < rounds[ri].size();)
                if ((st = next_launch(ri, done)) != ISO_SUCCESS) return st;
        return ISO_SUCCESS;
    }

    // Kernels that iso_start takes without the chain: the rounds, with those of a dimension together if they are merged.
    // Rows of any block size written whole are one; in the allocation-free call another one stores their records, and they
    // count as the launches per dimension that they stand for (the two take 8.7 us for up to 4096 ranks, 6 neighbours and
    // 20 bytes; the chain 6.2 for 8^3, 60 B and for 16^2, 4, 100 B).  Whole units still count as one there.
    uint64_t launches_of_rounds(bool merges) const {
        uint64_t n = 0;
        for (size_t ri = 0; ri < rounds.size(); ++ri) {
            const bool joins = merges && ri && bound_rounds[ri].kind == ISO_ROUND_SHIFT &&
                               bound_rounds[ri - 1].kind == ISO_ROUND_SHIFT && bound_rounds[ri - 1].dim == bound_rounds[ri].dim;
            if (joins || rounds[ri].empty()) continue;
            if (arena && bound_rounds[ri].kind == ISO_ROUND_DELIVER && size0 % 16) {
                std::vector<bool> moves((size_t)c.d + 1, false);
                for (const HostEntry &he : rounds[ri]) moves[(size_t)(he.dim + 1)] = true;
                n += (uint64_t)std::count(moves.begin(), moves.end(), true);
            } else {
                ++n;
            }
        }
        return n;
    }

    // iso_start of a small collective: all rounds in one launch (see chain_kernel), if its hops fit the arguments and
    // a workgroup the ranks.  Against a launch per dimension: 8 x 8, 32 B 9.9 -> 7.2 us, 8^3, 26 neighbours, 64 B
    // 13.4 -> 7.4, 5^4 star, 400 B 16.4 -> 7.4; allgather the same.  What it saves is 2 to 2.7 us of the host's time
    // per launch less; what it costs is that a workgroup's accesses are a column of units per rank, at best a few
    // sectors each, which most of the chip does not take part in.  The limits are 6144 sectors for one workgroup over
    // all its hops (60^2, 64 B: 7200, 10.1 -> 12.7; 16^3, 16 B: 12288, 13.3 -> 16.4), and for all of them 48 Ki per
    // launch that it saves.  Measured with up to 25 sets of buffers in turn, which the caches hold, and with 1 GiB of
    // them: one launch less, 16^2 radius 1, 400 B (32 Ki) 9.7 -> 7.8 and 9.7 -> 7.9, 16^2 star of two, 400 B (48 Ki)
    // 9.5 -> 7.8 and 10 -> 8.5, 1000 B (96 Ki) 9.9 -> 8.9 and 9.8 -> 10.9, 24 x 20, 24 neighbours, 320 B (135 Ki) 9
    // -> 8 and 9 -> 10.5; two less, 8^3, 64 B (39 Ki) 13.4 -> 7.4 and 12.9 -> 7.9, 10^3, 64 B (76 Ki) 12.1 -> 10.2
    // and 12.5 -> 13.1, 100 B (152 Ki) 12.4 -> 12.3 and 12.8 -> 16.8; 10^3, 16 B (76 Ki) 10.4 -> 6.6 and 10.6 -> 9.2,
    // 11^3, 16 B (101 Ki) 10.2 -> 8.9 and 10.3 -> 11.9, 12^3, 32 B (132 Ki) 10.2 -> 11.6 and 10.2 -> 16.  Columns of
    // at most a sector of blocks of more than 32 bytes that do not fill sectors lie across two, which counts double
    // (32^2, 100 B with many sets 9.8 -> 8.6, allgather 8 to 9.8 -> 9.1).  Single hops are no different (16^2 star, 3000
    // B (48 Ki) 8.0 -> 7.3, 6^4 star, 500 B (111 Ki, three less) 12.6 -> 10.8, many sets; 45^2 star, 256 B (63 Ki) 9.3 ->
    // 8.7 and 9.2 -> 12.3).  A schedule of one launch gains nothing (4096, 16 B 6.5 -> 6.9).  Near the limits many sets
    // lose what repeated ones gain (45^2 radius 1, 32 B 9.3 -> 7.2 and 9.3 -> 11.3): a persistent request finds its
    // blocks in the last-level cache again.
    // Chains of several hops that fill 64 workgroups and more are spread over the chip, and where they save two launches
    // and more, these are the longer ones: 12288 sectors for one workgroup, 192 Ki per launch saved (a launch per dimension
    // -> chain, one set of buffers and a gigabyte of them: 8^3, 124 neighbours, 64 B 10.1 -> 5.9 and 11.6 -> 7.0; 5^4, 80
    // neighbours, 64 B 10.7 -> 6.7 and 13 -> 9.2; 4^4, 80 neighbours, 200 B 14 -> 7.5 and 14.6 -> 9.8; 5 x 4 x 5 x 4 x 5,
    // 31 neighbours, 64 B 14.5 -> 13.2 and 16.6 -> 15.3; near it 5 x 7 x 5, 20 neighbours, 2144 B 11.9 -> 7.3 and 11.5 ->
    // 10.0, 6 x 5 x 7 x 4, 30, 144 B 14.2 -> 9.5 and 15.5 -> 11.7, 12 x 9 x 7, 24, 367 B 10.7 -> 9.8 and 12.2 -> 13.2;
    // beyond it 8^4, 30 neighbours, 16 B 13.6 -> 15.2 and 14.8 -> 16.9).  Not for one launch saved (20 x 16, 24 neighbours,
    // 586 B 7.9 -> 8.2 and 8.1 -> 10.1; 13 x 16, 24, 796 B 6.1 -> 5.2 and 6.9 -> 8.3; 13^2, 12, 2784 B 6.7 -> 4.9 and
    // 7.1 -> 8.0), nor with fewer workgroups (32^2, 24 neighbours, 100 B 7.2 -> 9.3, 45^2, 32 B 6.5 -> 7.3 with many sets).
    // The allocation-free call always saves two and more, with the one that stores its table (20 x 16, 586 B 10.9 -> 8.2
    // and 11.0 -> 10.0; 13^2, 2784 B 10.6 -> 5.4 and 10.6 -> 7.8).
    static constexpr size_t kChainHops = 1024;
    bool chain_launch(uint64_t launches) {
        const size_t most_hops = arena ? kChainHopsByValue : kChainHops;
        if (c.mesh || !uniform || !size0 || launches < 2 || p > kChainThreads * kChainUnitsPerLane || s > most_hops ||
            (size0 >> min_log2) > 0xFFFF)
            return false;
        std::vector<const HostEntry *> hops;             // chain after chain
        std::vector<uint32_t> ends;                      // where each of them ends
        if (op == ISO_OP_ALLTOALL) {
            size_t n_hops = 0;
            for (const std::vector<HostEntry> &round : rounds) n_hops += round.size();
            if (n_hops > most_hops) return false;
            hops.resize(n_hops);
            ends.resize(s + 1);
            for (const std::vector<HostEntry> &round : rounds)
                for (const HostEntry &he : round) ++ends[(size_t)he.neighbor + 1];
            std::partial_sum(ends.begin(), ends.end(), ends.begin());
            for (const std::vector<HostEntry> &round : rounds)
                for (const HostEntry &he : round) hops[ends[(size_t)he.neighbor]++] = &he;
            ends.pop_back();                             // (what was a chain's start has moved on to its end)
        } else {
            // Allgather: the way of every receive block from the send buffer down the trie.  Ways share moves, and
            // each makes them for itself; they write the same bytes, provided that no place is used twice.
            std::vector<std::pair<uint64_t, const HostEntry *>> written_by;      // in order of the places
            for (const std::vector<HostEntry> &round : rounds)
                for (const HostEntry &he : round) written_by.emplace_back(he.de.dst, &he);
            std::sort(written_by.begin(), written_by.end());
            for (size_t q = 1; q < written_by.size(); ++q)
                if (written_by[q].first == written_by[q - 1].first) return false;
            const auto writer = [&](uint64_t place) -> const HostEntry * {
                const auto at = std::lower_bound(written_by.begin(), written_by.end(), std::make_pair(place, (const HostEntry *)nullptr));
                return at != written_by.end() && at->first == place ? at->second : nullptr;
            };
            for (const auto &[dst, last] : written_by) {
                if (last->dst_buf != ISO_BUF_RECV) continue;
                const size_t start = hops.size();
                for (const HostEntry *at = last; at; at = writer(at->de.src)) hops.push_back(at);
                if (hops.size() > most_hops) return false;
                std::reverse(hops.begin() + (ptrdiff_t)start, hops.end());
                ends.push_back((uint32_t)hops.size());
            }
        }
        if (hops.empty() || hops.size() > most_hops) return false;
        Pending pd;
        pd.first_entry = pd.first_prefix = 0;
        std::memset(&pd.l, 0, sizeof(pd.l));
        Launch &l = pd.l;
        l.kernel = kChainKernel;
        l.lds_table = true;
        auto args = std::make_unique<ChainArgs>();
        ChainHead &ca = args->head;
        uint64_t width = uint64_t(1) << min_log2;
        const auto cut = [&] {
            l.tail = (size0 & (width - 1)) != 0;
            ca.chunks = (uint32_t)((size0 + width - 1) / width);
            ca.column = std::min<uint32_t>(ca.chunks, kChainThreads * kChainUnitsPerLane / (uint32_t)p);
        };
        cut();
        // A last unit that overlaps the one before it goes into the same column: two workgroups are not at the
        // same hop, and one would read bytes that the other has already replaced.
        while (l.tail && ca.column > 1 && ca.column < ca.chunks && (ca.chunks - 1) % ca.column == 0) --ca.column;
        if (l.tail && ca.chunks > 1 && ca.column == 1) {
            // one unit of every rank is all that a workgroup holds: units that divide the block (5 x 4 x 7 x 6 x 4
            // star, 6 B: 14.7 us in five launches, 4.3 in this one)
            width = size0 & (~size0 + 1);
            l.chain_width = (uint32_t)width;
            cut();
        }
        ca.groups = (ca.chunks + ca.column - 1) / ca.column;
        ca.n_units = (uint32_t)p * ca.column;
        put(ca.column, ca.mul_column, ca.more, 0);
        put(ca.groups, ca.mul_groups, ca.more, 1);
        ca.more |= launch_flags(0, false, (uint32_t)(ca.chunks * width - size0));
        std::vector<ChainHop> table_hops(hops.size());
        uint32_t begin = 0, n_chains = 0, longest = 0;
        for (const uint32_t end : ends) {
            n_chains += end != begin;
            begin = end;
        }
        begin = 0;
        std::vector<uint32_t> begins(n_chains + 1);
        uint32_t chain = 0, later = n_chains;
        for (const uint32_t end : ends) {
            if (end == begin) continue;                          // no hops: an empty block
            longest = std::max(longest, end - begin);
            begins[chain] = later - n_chains;
            for (uint32_t at = begin; at < end; ++at) {
                const HostEntry *he = hops[at];
                ChainHop &hop = table_hops[at == begin ? chain : later++];
                hop.src = he->de.src;
                hop.dst = he->de.dst;
                hop.src_stride = he->de.src_stride;
                hop.dst_stride = he->de.dst_stride;
                hop.shift = he->dim < 0 ? 0u : he->de.shift;     // (a same-rank copy)
                hop.inner = he->dim < 0 ? 1u : (uint32_t)c.inner[(size_t)he->dim];
                hop.pj = he->dim < 0 ? 1u : (uint32_t)c.dims[(size_t)he->dim];
                put(hop.inner, hop.mul_inner, hop.shifts, 0);
                put(hop.pj, hop.mul_pj, hop.shifts, 1);
            }
            ++chain;
            begin = end;
        }
        begins[n_chains] = later - n_chains;
        ca.n_chains = n_chains;
        ca.n_hops = (uint32_t)hops.size();
        l.grid = n_chains * ca.groups;
        const uint64_t piece = ca.column * width, own = p * ((piece + 63) / 64) * longest;
        uint64_t all = own * l.grid;
        if (longest > 1 && size0 > 32 && size0 % 64 && piece <= 64) all *= 2;
        const bool wide = l.grid >= 64 && longest > 1 && (launches > 2 || arena);
        if (own > (wide ? 12288 : 6144) || all > (launches - 1) * (wide ? 192 : 48) * 1024) return false;
        l.threads = std::min<uint32_t>(kChainThreads, (ca.n_units + 63) & ~63u);
        l.dyn_lds = longest > 1 ? ca.n_units * (uint32_t)width : 0;
        describe_chain_bytes(l, hops, n_chains);
        l.chain = ca;
        const uint32_t *words = (const uint32_t *)table_hops.data();
        const size_t n_words = table_hops.size() * sizeof(ChainHop) / 4;
        if (arena) {
            std::copy(begins.begin(), begins.end(), std::copy(words, words + n_words, args->table));
            rq.chain = std::move(args);
            l.chain_by_value = rq.chain.get();
        } else {
            while (prefixes.size() % 4) prefixes.push_back(0);
            pd.first_prefix = prefixes.size();
            prefixes.insert(prefixes.end(), words, words + n_words);
            prefixes.insert(prefixes.end(), begins.begin(), begins.end());
        }
        pending.push_back(pd);
        return true;
    }

    // A chain's first hop loads, from the send buffer; all of them store, ways of an allgather's trie in part to the same places.
    void describe_chain_bytes(Launch &l, const std::vector<const HostEntry *> &hops, uint32_t n_chains) const {
        l.bytes_read = p * size0 * (op == ISO_OP_ALLTOALL ? n_chains : 1);
        l.bytes_written = p * size0 * hops.size();
        if (op == ISO_OP_ALLTOALL) return;
        std::vector<uint64_t> targets;
        for (const HostEntry *he : hops) targets.push_back(he->de.dst);
        std::sort(targets.begin(), targets.end());
        targets.erase(std::unique(targets.begin(), targets.end()), targets.end());
        l.bytes_written = p * size0 * targets.size();
    }

    // iso_start of ISO_ALG_COMBINED: the consecutive rounds of one dimension, which touch disjoint blocks, in one
    // launch.  A launch costs about 4 us of ramp and drain on top of its traffic, and rounds that read the same blocks
    // or share memory lines meet in the caches (us, rounds -> together, one set of buffers repeated and 1 GiB of sets in
    // turn: 32^3, 26 neighbours, 256 B 170 -> 158 and 170 -> 160; 64^3, 128 B 626 -> 615 and 627 -> 615; 256^2, 12
    // neighbours, 1 KiB 451 -> 344 and 450 -> 345; 16^3, 400 B 48 -> 37 and 58 -> 46; 8^5, 40 random neighbours, 1
    // KiB 2003 -> 1926; allgather 32^3, 256 B 70 -> 56 and 77 -> 56, 60 x 50 x 41, 200 B 370 -> 236 and 451 -> 292).
    // Some all-to-alls of several GB lose 1 to 3 %, with no rule in sight (100^3 star, 1 KiB 2016 -> 2073, 512 B 1114 ->
    // 1045).  iso_start_range still runs the rounds one by one.
    void merge_rounds() {
        size_t n = 0;
        for (size_t ri = 0; ri < bound_rounds.size(); ++ri) {
            const BoundRound &r = bound_rounds[ri];
            const bool joins = n && r.kind == ISO_ROUND_SHIFT && bound_rounds[n - 1].kind == ISO_ROUND_SHIFT &&
                               bound_rounds[n - 1].dim == r.dim;
            if (joins) {
                rounds[n - 1].insert(rounds[n - 1].end(), rounds[ri].begin(), rounds[ri].end());
            } else {
                if (n != ri) {
                    bound_rounds[n] = r;
                    rounds[n] = std::move(rounds[ri]);
                }
                ++n;
            }
        }
        bound_rounds.resize(n);
        rounds.resize(n);
        // destination blocks in order: by neighbour, or by the receive or workspace slot.  A counting sort: with 16 806
        // neighbours init takes 1.7 ms, with a comparison sort of the entries it took 3.0.
        const auto key = [&](const HostEntry &he) {
            if (op == ISO_OP_ALLTOALL) return (size_t)he.neighbor;
            return he.dst_buf == ISO_BUF_RECV ? (size_t)he.dst_slot : s + (size_t)he.dst_slot;
        };
        std::vector<uint32_t> at(s + (size_t)pl.work_slots + 1);
        for (std::vector<HostEntry> &ents : rounds) {
            std::fill(at.begin(), at.end(), 0u);
            for (const HostEntry &he : ents) ++at[key(he) + 1];
            std::partial_sum(at.begin(), at.end(), at.begin());
            std::vector<HostEntry> sorted(ents.size());
            for (const HostEntry &he : ents) sorted[at[key(he)]++] = he;
            ents.swap(sorted);
        }
    }

    // iso_start of an all-to-all whose rows fit a workgroup (rows_fit_a_tile): the last hop of every block taken out of
    // its round, and all of them in one launch that writes whole receive rows (deliver_launch), after the rounds of the
    // other hops, which read rows and write planes (staged_round_launch).  Every block makes the moves of its schedule;
    // what goes are writes of parts of memory sectors (64^3, 100 B: 26 % of the rounds' write requests, 9 % here), with which
    // the rounds take up to 2.6 times as long as their blocks at the copy rate.  For blocks that do not fill 64-byte
    // sectors (us, one launch per dimension -> rows, a gigabyte of buffer sets in turn: 64^3, 26 neighbours, 20 B 222 -> 171, 100 B 1119 -> 800, 400 B 2721 -> 2606; 662 x 503, 10 neighbours, 100 B 351 ->
    // 223; 20^4, 80 neighbours, 100 B 3195 -> 2413; 24^3, 100 B 50 -> 41; 16^3, 200 B 31 -> 26; 8^5, 40 neighbours, 40 B
    // 135 -> 119; one set of buffers repeated gains less and in part loses what the cache holds of it between the rounds:
    // 16^3, 168 B 27.8 -> 24.4 and 19.3 -> 21.7; 23 x 32 x 26, 124 neighbours, 32 B 111 -> 87 and 70 -> 82).
    // Not: 512 B and more (64^3, 500 B 3269 -> 3279), up to 8 MiB (64^2, 24 neighbours, 40 B 5.9 -> 8.5; 16^3, 40 B 10 ->
    // 13.6), up to 16 MiB where blocks make three hops and more (6^4, 30 neighbours, 348 B 30.7 -> 31.9; 3^7, 132 B 39.6 ->
    // 42.4; 7^4, 168 B 31.4 -> 31.0; though 5^5, 40 neighbours, 84 B 43.6 -> 39.1), up to 48 MiB under 32 bytes (24^3, 20 B
    // 15.1 -> 17.7).  ISO_ALG_COMBINED_BYDIM starts its launch list up to 7/4 of the last-level cache (above: 64^3, 100 B
    // 1119 -> 800; 8^5, 40 neighbours, 400 B 1045 -> 1063).
    // Whole sectors gain at 64 bytes, half a line, from 48 MiB on (662 x 503, 10 neighbours 147 -> 134; 64^3, 26 neighbours
    // 409 -> 388; 80^3, 20 811 -> 758; 14^4, 80 254 -> 215; 8^5, 40 177 -> 149), except in two dimensions for fewer than
    // eight hops to five blocks (600^2, 8 neighbours, 12 hops 112 -> 117, 420^2, 12, 16 75 -> 78; 600^2, 8, 13 132 -> 117,
    // 24, 40 349 -> 331) and in four and more above 3/2 of the cache, where a tile's ranks are few and far apart in every
    // plane (20^4, 80 neighbours 984 -> 1146; 12^5, 40 1276 -> 1417; 30^4, 10 770 -> 842; 11^5, 40, 412 MB 868 -> 859;
    // in three 74^3, 26 634 -> 649).
    // Larger ones do not but in two dimensions (128 B 64^3 618 -> 618, 192 B 951 -> 1061, 14^4 571 -> 636, 662 x 503 391
    // -> 364; 320 B 64^3 1529 -> 1640).
    bool rows_in_one_launch() const {
        const uint64_t llc = kLastLevelCacheBytes, bytes = inf.delivered_bytes;
        const int64_t blocks = (int64_t)s;
        if (op != ISO_OP_ALLTOALL || arena || !rows_fit_a_tile() || size0 >= 512 || s * size0 + 15 > kTileUnits * 16) return false;
        if (size0 % 64 == 0) {
            if (size0 > 64 || bytes <= llc * 3 / 16) return false;
            if (c.d <= 2 ? 5 * inf.entries < 8 * blocks : c.d > 3 && bytes > llc * 3 / 2) return false;
        }
        if (pl.algorithm == ISO_ALG_COMBINED_BYDIM) return bytes > llc * 7 / 4;
        return pl.algorithm == ISO_ALG_COMBINED && bytes > (size0 < 32 ? llc * 3 / 16 : inf.entries >= 3 * blocks ? llc / 16 : llc / 32);
    }

    // iso_start of ISO_ALG_COMBINED where every block makes its one move out of the send buffer (a star): the moves of
    // all dimensions touch different receive blocks and go together, as one launch of the kernel that knows the
    // neighbours' full vectors (us, a launch per dimension -> one, a gigabyte of buffer sets in turn: 64^3, 6 neighbours,
    // 16 B 34 -> 15.5, 72 B 100 -> 48, 128 B 75 -> 65, 2 KiB 1083 -> 1025; 24^3, 100 B 13.1 -> 7.0; 12^4, 200 B 31.5 ->
    // 15.3; 300^2, 4000 B 483 -> 467; slot-major 64^3, 128 B 69.9 -> 65.7).  From 256 bytes on above a 24th of the
    // cache.  An allgather below 256 bytes (64^3 128 B 47 -> 37, 200 B 130 -> 58; 24^3, 128 B 9.0 -> 4.4; 16^4, 128 B 18.2 ->
    // 14.2; 500^2, 128 B 28.9 -> 24.1; in two dimensions single sizes of whole sectors lose with many sets of buffers what
    // they gain with one: 300^2, 128 B 11.8 -> 14.3 and 10.7 -> 8.7, 700^2, 192 B 92 -> 121 and 92 -> 71); from there on
    // whole lines lose more of that (300^2, 1 KiB 81 -> 102 and 79 -> 63, 2 KiB 170 -> 229; 64^3, 1 KiB 366 -> 408), though
    // other sizes would gain (64^3, 300 B 179 -> 89).  Nothing to gain in one dimension (262144, 256 B 44.1 -> 45.1).
    bool star_in_one_launch(uint64_t launches) const {
        if (pl.algorithm != ISO_ALG_COMBINED || c.mesh || !uniform || inf.entries != (int64_t)s || launches < 2 ||
            c.d > kVectorDims || s > kLdsEntries)
            return false;
        for (const Round &r : pl.rounds)
            for (const iso_plan_entry_t &e : r.entries)
                if (e.src_buf != ISO_BUF_SEND) return false;
        return size0 < 256 || (op == ISO_OP_ALLTOALL && inf.delivered_bytes > kLastLevelCacheBytes / 24);
    }

    void join_star() {
        std::vector<HostEntry> all;
        all.reserve(s);
        for (const std::vector<HostEntry> &ents : rounds) all.insert(all.end(), ents.begin(), ents.end());
        for (HostEntry &he : all) he.de.shift = (uint32_t)he.neighbor;
        bound_rounds.assign(1, {ISO_ROUND_VECTOR, -1, bound_rounds[0].of, nullptr});
        rounds.assign(1, std::move(all));
    }

    // iso_start in one launch (one for each table that LDS takes) of all blocks through all their hops: every move stores its
    // block, but a hop takes it from the one before it in a register (move_through_stops), in an allgather from the send
    // buffer as all others do.  On tori of up to five dimensions, from 4 MiB on; on boxes for ISO_ALG_COMBINED_BYDIM.
    // All-to-all (us, as before -> here, a gigabyte of buffer sets in turn): 32^3, 26 neighbours, 256 B 160 -> 108; 256^2, 12,
    // 1 KiB 348 -> 304; 64^3, 26, 128 B 615 -> 433, 320 B 1660 -> 1133, 1000 B 5858 -> 3743; 8^5, 40, 320 B 679 -> 303, 4 KiB
    // 7562 -> 3800; 16^4, 30, 400 B 1221 -> 526; 300^2, 24, 300 B 392 -> 307; 100^2, 8, 512 B 25.6 -> 20.7; 16^3, 384 B 37.0 ->
    // 23.8; 20^3, 256 B 45.3 -> 29.8; slot-major 32^3, 256 B 150 -> 99.
    // Allgather: 64^3, 26 neighbours, 128 B 205 -> 135; 20^3, 128 B 13.8 -> 6.8; 32^3, 1000 B 282 -> 150; 300^2, 24, 512 B 229
    // -> 157, 10, 1300 B 436 -> 265; 8^5, 40, 500 B 823 -> 459, 4 KiB 5187 -> 2975; 16^4, 30, 256 B 386 -> 222; slot-major 64^3,
    // 128 B 197 -> 152, 100 B 168 -> 128.
    // Small ones: all-to-all 10^3, 26 neighbours, 256 B 10.9 (chain) -> 6.2, 12^3, 256 B 15.4 -> 9.8; allgather 20^3, 40 B
    // 11.4 -> 4.0, 5^5, 40, 128 B 27.8 -> 9.3; 13 x 12 x 14, 80 B slot-major 10.0 -> 4.7.  Below 4 MiB a chain takes what fits
    // it (6^3, 20, 48 B 3.5, here 3.7).
    // More than one table: the chain of a small collective stays (5^2, 440 neighbours, 384 B 3.9 us, here in four launches
    // 12.0; 7^2, 224, 768 B 5.3 and 6.5), and up to 32 MiB for each launch here, at most the last-level cache, so do fewer
    // launches (us, before -> here: 3^3, 728, 4 launches against 6, all-to-all 1280 B 27.7 -> 33.3, 5 KiB 79 -> 81, 21 KiB 297
    // -> 225; 5^2, 440, 3 against 4, 4480 B 33.7 -> 39.4, 18 KiB 113 -> 108; 8^2, 960, 3 against 8, 3200 B 128 -> 134, 6784 B
    // 265 -> 250, allgather 768 B 17.5 -> 23.0, 6784 B 81 -> 77; 4^4, 2400, 4 against 19, allgather 256 B 52 -> 61, 640 B 116
    // -> 100; 32^2, 440, 2 against 4, 384 B 128 -> 112; what gains and stays: 5^4, 624, 4 against 5, 256 B 124 -> 89).  As
    // many: 5^3, 342, 384 B 22.6 -> 20.9.
    // Two dimensions, allgathers of whole units that are parts of lines, with more to send than the last-level cache holds: not
    // pushed (allgather_order), and what the pulls miss comes from memory every time (250 x 260, 10 neighbours, 4416 B 820 ->
    // 1031, 6432 B 1232 -> 1498; 8, 5600 B 794 -> 903; up to it 4096 B and 12 728 -> 653; three dimensions 64^3, 26, 1168 B
    // 2545 -> 2361).  Other sizes cost a launch per dimension more (250 x 260, 4531 B, 8 neighbours 819 -> 757, 12 1176 ->
    // 1037; 267 x 335, 10, 4893 B 1706 -> 1638; 400 x 420, 10, 3037 B 1881 -> 1685, but 2724 B 1642 -> 1800).
    // Boxes, where the moves of blocks that no one receives are left out: 45 x 37 x 29, 26 neighbours, 100 B slot-major 97 -> 64,
    // 256 B 235 -> 151; 8^5, 40, 512 B 877 -> 240; 64^3, allgather 256 B 550 -> 285.
    // The other limits are no measured ones.  All-to-alls of most sizes of small blocks that are no whole lines, rank-major,
    // and larger allgathers of them, more of both for ISO_ALG_COMBINED_BYDIM up to 7/4 of the last-level cache, and boxes but
    // for BYDIM keep the launches of their rounds, which the tests of these launches lay down, though they would gain here
    // (all-to-all 64^3, 100 B 797 -> 402, 192 B 1038 -> 688, 16^3, 128 B 19.4 -> 11.7; allgather 8^5, 100 B 235 -> 160).
    bool all_hops_in_one_launch(uint64_t launches) const {
        const uint64_t llc = kLastLevelCacheBytes, bytes = inf.delivered_bytes;
        const bool a2a = op == ISO_OP_ALLTOALL, bydim = pl.algorithm == ISO_ALG_COMBINED_BYDIM, lines = size0 % 128 == 0;
        if (arena || !uniform || size0 < 16 || c.d > kVectorDims || bytes <= llc / 64) return false;
        if (pl.algorithm != ISO_ALG_COMBINED && !bydim) return false;
        bool onward = false;                             // a hop of what another one has brought
        for (const Round &r : pl.rounds)
            for (const iso_plan_entry_t &e : r.entries) onward = onward || e.src_buf != ISO_BUF_SEND;
        if (!onward) return false;
        if (hops_launches() > launches && bytes <= std::min(llc, hops_launches() * llc / 8)) return false;
        if (c.mesh && (!bydim || (!a2a && !lines && size0 < 256))) return false;
        if (lay.slot_major) return !a2a || bytes > (lines ? llc / 8 : llc * 3 / 16);
        if (!a2a && c.d == 2 && size0 % 16 == 0 && p * size0 > llc * 17 / 16 && !whole_lines()) return false;
        if (!a2a) {
            if (size0 >= 512 || (!bydim && (lines || size0 >= 256)) || bytes <= (size0 < 64 ? llc * 3 / 16 : llc / 2)) return true;
            return lines && bytes > llc * 7 / 4;
        }
        if (lines && size0 >= 256) return true;
        if (lines || size0 >= 512) return bytes > (bydim ? llc / 8 : llc / 16);
        return size0 >= 320 && bytes > (bydim ? llc * 7 / 4 : llc * 3 / 16);
    }

    // Every destination begins and ends with a 128-byte line.
    bool whole_lines() const {
        uint64_t bits = size0;
        for (const std::vector<HostEntry> &round : rounds)
            for (const HostEntry &he : round) bits |= he.de.dst | he.de.dst_stride;
        return (bits & 127u) == 0;
    }

    // Launches of join_hops's entries, which are the blocks of an all-to-all and the nodes of an allgather's trie.
    uint64_t hops_launches() const {
        uint64_t n = 0;
        if (op == ISO_OP_ALLTOALL) n = s - (uint64_t)std::count(lay.size.begin(), lay.size.end(), uint64_t(0));
        else for (const std::vector<HostEntry> &round : rounds) n += round.size();
        return (n + kLdsEntries - 1) / kLdsEntries;
    }

    // All-to-all: one entry per block, from the send buffer to the receive buffer, its stops in its place in the workspace (in
    // the plan a block of three hops and more stops in its receive block as well; in one launch the stores of two lanes to it
    // would have no order).  Allgather: an entry for every node of the trie, all from the send buffer; what lies in the
    // workspace is read by no one, so that nodes may share a place there.
    void join_hops() {
        all_hops = true;
        const bool a2a = op == ISO_OP_ALLTOALL;
        std::vector<HostEntry> all;
        if (a2a) all.resize(s);
        else all.reserve((size_t)inf.entries);
        uint32_t routed = 0;                             // the dimensions up to that of the round
        size_t next_dim = 0;
        for (size_t ri = 0; ri < rounds.size(); ++ri) {
            const BoundRound &r = bound_rounds[ri];
            if (!a2a && r.kind == ISO_ROUND_SHIFT)
                while (!(routed >> r.dim & 1u)) routed |= 1u << pl.dim_order[next_dim++];
            for (const HostEntry &he : rounds[ri]) {
                if (!a2a) all.push_back(HostEntry{});
                HostEntry &to = a2a ? all[(size_t)he.neighbor] : all.back();
                const HostEntry before = to;
                to = he;
                if (a2a) {
                    to.de.shift = (uint32_t)he.neighbor;
                    to.moves = before.moves + 1;
                    to.way = he.dst_buf == ISO_BUF_WORK ? he.de.dst : before.way;
                    if (!before.moves) continue;         // the first hop
                    to.de.src = before.de.src;
                    to.de.src_stride = before.de.src_stride;
                } else {
                    uint64_t stride = 0;
                    place(ISO_BUF_SEND, 0, to.de.src, stride);
                    to.de.src_stride = (uint32_t)stride;
                    to.de.shift = he.de.ref;
                    to.along = he.dim < 0 ? 0u : routed;
                    to.way = he.de.dst_stride;
                }
            }
        }
        all.erase(std::remove_if(all.begin(), all.end(), [](const HostEntry &he) { return !he.moves; }), all.end());   // (empty blocks)
        bound_rounds.assign(1, {ISO_ROUND_VECTOR, -1, bound_rounds[0].of, nullptr});
        rounds.assign(1, std::move(all));
    }

    // Unequal blocks through all their hops: the larger ones a launch for every size, by the vector kernel, those of up to
    // kSmallUnits units in one launch of the block kernel, if that is fewer launches than one per dimension that blocks move
    // along (one for every kLdsEntries blocks of a size; as many or more lose: 32^2, 440 neighbours, 4 and 8 B, 4 launches
    // against 2, 15.3 us against 9.5; 8^5, four sizes along one dimension, 4 against 1, 28.1 against 19.3).  A launch then
    // moves blocks of one kind, and the larger ones need no search for a unit's entry.  (Stencils, us, a launch per dimension
    // -> here: 32^3, 64 B 338 -> 291, 25 B 90 -> 78; 64^3, 16 B 379 -> 323, 4 B 150 -> 133, 80^3, 8 B 558 -> 400;
    // 16^4, 8 B 373 -> 342; 8^5, 4 B 512 -> 391; 500^2, 64 B 81 -> 57; 8^3, 64 B 15.8 -> 11.8, 40^2, 64 B 6.3 -> 3.9.)  Small
    // blocks that are no whole units lose it again in more dimensions, and among themselves in three (16^4, 6 B 285 -> 303;
    // 64^3, 11 B 303 -> 361; 22^4, 3 B 673 -> 822), as many launches as before gain nothing (300^2, 200 B 57 -> 60).
    // Blocks of a few bytes lose, from a million or two of their units on, what fewer launches save (stencils, edge, one set
    // of buffers and many: 32^3, 3 B 19.6 -> 18.6 and 22.9 -> 22.6, 40^3 30 -> 33 and 35 -> 39, 48^3, 2 B 30.5 -> 31.1 and 35
    // -> 38, 4 B 45 -> 38, 64^3, 2 B 60 -> 75, 3 B 94 -> 132, 4 B 87 -> 84; 16^4, 2 B 83 -> 102; 9^5, 2 B 269 -> 397; 280^2,
    // 3 B 9.0 -> 8.2 and 9.6 -> 9.0, 360^2 10.8 -> 11.3 and 12.3 -> 13.5, 400^2, 4 B 10.1 -> 9.6 and 12.2 -> 12.6, 450^2 11.8
    // -> 12.2 and 14.5 -> 16.0, 512^2, 3 B 17.2 -> 20.2, 11 B 21 -> 23, 15 B 24.5 -> 23.5), on boxes of three and more
    // dimensions small blocks of any size (32^3, 8 B 24.5 -> 22.8, 48^3 58 -> 65, 64^3 135 -> 164, 4 B 80.5 -> 83.1; 20^4, 4 B
    // 301 -> 330; with larger ones beside them 64^3, 16 B 407 -> 290).
    // ISO_ALG_COMBINED_BYDIM: where kBySize was taken (60 x 50 x 41, 25 B 318 -> 296; 20^4, 8 B 1099 -> 832).
    bool all_hops_by_size() {
        const uint64_t llc = kLastLevelCacheBytes, bytes = inf.delivered_bytes;
        if (op != ISO_OP_ALLTOALL || arena || uniform || lay.slot_major || c.d < 2 || c.d > kVectorDims || wl.bytes >> 36)
            return false;
        std::vector<uint64_t> blocks;                    // of every large size
        uint64_t small = 0, small_units = 0, small_bytes = 0;
        bool units = true;
        for (size_t i = 0; i < s; ++i) {
            const uint64_t m = lay.size[i];
            if (!m) continue;
            const uint32_t l2 = unit_log2_of(m);
            const uint64_t upb = (m + (uint64_t(1) << l2) - 1) >> l2;
            if (upb <= kSmallUnits) {
                ++small;
                small_units += upb;
                small_bytes += m;
                units = units && (m < 16 || m % 16 == 0);
                continue;
            }
            const size_t at = (size_t)(std::find(large_sizes.begin(), large_sizes.end(), m) - large_sizes.begin());
            if (at == large_sizes.size()) {
                large_sizes.push_back(m);
                blocks.push_back(0);
                if (large_sizes.size() >= (size_t)c.d) return false;
            }
            ++blocks[at];
        }
        uint64_t launches = (small + kLdsEntries - 1) / kLdsEntries;
        for (const uint64_t n : blocks) launches += (n + kLdsEntries - 1) / kLdsEntries;
        if (launches >= dimensions_moved()) return false;
        constexpr uint64_t kMi = uint64_t(1) << 20;
        const uint64_t work = p * small_units;
        if (c.d == 2 ? !c.mesh && work > kMi * 11 / 8 && small_bytes <= 6 * small : work > 2 * kMi && small_bytes < 5 * small) return false;
        if (c.d > 2 && c.mesh && large_sizes.empty() && work > 4 * kMi) return false;
        if (pl.algorithm == ISO_ALG_COMBINED_BYDIM) return !c.mesh && small && !large_sizes.empty() && bytes > llc / 4;
        return pl.algorithm == ISO_ALG_COMBINED && (units || c.d == 2 || (c.d == 3 && !large_sizes.empty()));
    }

    // The dimensions that some block moves along: launches of iso_start with one for each.
    uint64_t dimensions_moved() const {
        uint32_t moved = 0;
        for (size_t ri = 0; ri < rounds.size(); ++ri)
            if (bound_rounds[ri].kind == ISO_ROUND_SHIFT && !rounds[ri].empty()) moved |= 1u << bound_rounds[ri].dim;
        return (uint64_t)__builtin_popcount(moved);
    }

    void split_by_size() {
        const std::vector<HostEntry> all = std::move(rounds[0]);
        const BoundRound whole = bound_rounds[0];
        rounds.assign(large_sizes.size() + 1, {});
        for (const HostEntry &he : all) {
            const size_t at = he.de.units <= kSmallUnits ? large_sizes.size()
                                                         : (size_t)(std::find(large_sizes.begin(), large_sizes.end(), he.size) - large_sizes.begin());
            rounds[at].push_back(he);
        }
        if (rounds.back().empty()) rounds.pop_back();
        bound_rounds.assign(rounds.size(), whole);
        one_size = true;
    }

    // iso_start of ISO_ALG_COMBINED_STAGED, all-to-all: its first two rounds in one launch (staged_round_kernel, TWO), where
    // the blocks that either of them takes out of a send-buffer row fit a tile.  If none of them makes a hop in both, nothing is
    // read less, and beyond the last-level cache the longer tiles cost what the launch saves (stars of radius two: 32^3, 24
    // neighbours, 200 MB 0.95 to 0.98 of two launches; 48^3, 240 B 370 -> 385, 80^3, 144 B 1061 -> 1095, 208 B 1515 -> 1558;
    // 18^4, 40, 160 and 208 B 1.04 and 1.05 of two).
    bool two_staged_rounds() const {
        if (pl.algorithm != ISO_ALG_COMBINED_STAGED || op != ISO_OP_ALLTOALL || arena || !uniform || bound_rounds.size() < 3 || !retiled()) return false;
        if (bound_rounds[0].kind != ISO_ROUND_SHIFT || bound_rounds[1].kind != ISO_ROUND_SHIFT || !bound_rounds.back().whole ||
            bound_rounds.back().kind != ISO_ROUND_DELIVER || bound_rounds[0].dim == bound_rounds[1].dim)
            return false;
        const uint64_t upb = (size0 + (uint64_t(1) << min_log2) - 1) >> min_log2;
        size_t n = rounds[0].size(), both = 0;
        if (n > kLdsEntries || rounds[1].size() > kLdsEntries) return false;
        for (const HostEntry &a : rounds[0])
            if (a.dst_buf != ISO_BUF_WORK || a.de.src_stride == size0) return false;
        for (const HostEntry &b : rounds[1]) {
            const bool onward = first_hop_of(b) >= 0;    // else out of a send-buffer row
            if (b.dst_buf != ISO_BUF_WORK || (!onward && b.de.src_stride == size0)) return false;
            n += !onward;
            both += onward;
        }
        if (!both && inf.delivered_bytes > kLastLevelCacheBytes) return false;
        return n <= kLdsEntries && n * upb <= kTileUnits && p * upb <= kMaxUnits;
    }
    // the entry of the first round that brings what `he` of the second one reads
    int first_hop_of(const HostEntry &he) const {
        for (size_t q = 0; q < rounds[0].size(); ++q)
            if (rounds[0][q].de.dst == he.de.src) return (int)q;
        return -1;
    }

    void join_two_rounds() {
        std::vector<HostEntry> joined = rounds[0];
        for (HostEntry &he : joined) he.de.units = 0, he.de.last_offset = 0;
        for (const HostEntry &b : rounds[1]) {
            const int q = first_hop_of(b);
            if (q < 0) {
                joined.push_back(b);
                joined.back().de.dst = 0;
                joined.back().de.shift = 0;
                joined.back().moves = 0;
            }
            HostEntry &to = q < 0 ? joined.back() : joined[(size_t)q];
            to.de.units = b.de.shift;
            to.de.last_offset = b.de.dst;
            ++to.moves;
        }
        second_dim = bound_rounds[1].dim;
        rounds[1] = std::move(joined);
        rounds.erase(rounds.begin());
        bound_rounds.erase(bound_rounds.begin() + 1);
    }

    void defer_last_hops() {
        std::vector<HostEntry> last(s);
        std::vector<bool> taken(s, false);
        for (size_t ri = rounds.size(); ri-- > 0;) {
            std::vector<HostEntry> &ents = rounds[ri], kept;
            for (const HostEntry &he : ents) {
                const size_t i = (size_t)he.neighbor;
                if (taken[i]) kept.push_back(he);
                else last[i] = he, taken[i] = true;
            }
            ents.swap(kept);
        }
        size_t n = 0;
        for (size_t ri = 0; ri < rounds.size(); ++ri) {
            if (rounds[ri].empty()) continue;
            if (n != ri) {
                bound_rounds[n] = bound_rounds[ri];
                rounds[n] = std::move(rounds[ri]);
            }
            ++n;
        }
        const int of = (int)pl.rounds.size() - 1;
        bound_rounds.resize(n);
        rounds.resize(n);
        bound_rounds.push_back({ISO_ROUND_DELIVER, -1, of, nullptr});
        rounds.push_back(std::move(last));
    }

    // On a mesh of rank-major buffers the units of a launch are interior where all its entries have a source, which is less
    // of the box for the rounds of a dimension together than for each by itself, and a unit that is not takes up to twice
    // its time (counted half as much again).  Against that stand what a launch costs (4 us, here in bytes at the copy rate)
    // and blocks that several rounds read.  On slot-major buffers every entry has its own bounds, together or not.  Rounds
    // one by one and all of a dimension together, us, many sets of buffers: 48^3, 124 neighbours, 128 B 1497 and 1567; 9^5,
    // 40 random neighbours up to 3 away, 512 B 1575 and 1640; 8^5, 1 KiB 1626 and 1647; the other way 8^5, 256 B 487 and
    // 460; 128^2, 48 neighbours, 2 KiB 988 and 937; 300^2, 12 neighbours, 400 B 302 and 250; slot-major 16^4, 40 random
    // neighbours, 256 B 703 and 633; 8^5, 1 KiB 1435 and 1371.  Over 93 boxes the choice loses 0.15 % on average and at
    // most 4.5 % (12^4, 30 random neighbours, 777 B 638 and 611; 28^3, 20, 2 KiB 809 and 783; 8^5, 4 KiB 5954 and 5822);
    // with weights of 1 and 2 it loses 0.17 and 0.19 %, with all of a dimension always together 0.18 %.
    bool rounds_move_faster() const {
        constexpr uint64_t kLaunchBytes = uint64_t(26) << 20;
        uint64_t rounds_cost = 0, merged_cost = 0;
        for (size_t i = 0; i < pending.size(); ++i) {
            const Launch &l = pending[i].l;
            uint64_t cost = kLaunchBytes + l.bytes_read;
            if (l.kernel == kMeshShiftKernel) {
                cost += l.outside_units * 3 / 2 << min_log2;
            }
            (i < n_listed ? rounds_cost : merged_cost) += cost;
        }
        return rounds_cost < merged_cost;
    }

    // In the allocation-free call the bitmaps of a mesh lie in its table and reach it 3 KiB a launch.  By the wavefront
    // they are four times as large: only where all of them go in the one launch that bits by the tile take as well, and
    // fit behind the entries (64^3, 6 neighbours, 256 B would be 10 of these launches instead of 6, and 400^3 refused).
    bool wave_bits_cost_no_launch() const {
        const uint64_t chunks = (size0 + (uint64_t(1) << min_log2) - 1) >> min_log2;
        uint64_t words = 0, entries = 0;
        for (const std::vector<HostEntry> &ents : rounds) {
            words += (p * chunks * ents.size() >> (kWaveLog2 + 5)) + 1;
            entries += ents.size();
        }
        return words <= kStoreWords &&
               entries * sizeof(DevEntry) + residue_bytes() + words * sizeof(uint32_t) <= arena->table_bytes;
    }

    // the [s][d] residues in the table; what follows them is 16-byte aligned
    size_t residue_bytes() const { return (c.can.size() * sizeof(uint32_t) + 15) & ~size_t(15); }

    uint32_t periodic_mask() const {
        uint32_t mask = 0;
        for (int j = 0; j < c.d; ++j)
            if (c.periodic[(size_t)j]) mask |= 1u << j;
        return mask;
    }

    uint64_t entry_size(const iso_plan_entry_t &e) const {
        if (op == ISO_OP_ALLTOALL) return lay.size[(size_t)e.neighbor];
        return s ? lay.size[0] : 0;
    }

    // bytes from the buffer's start to the end of the last block
    size_t buffer_len(const std::vector<uint64_t> &displ, uint64_t extent, uint64_t span, bool planes) const {
        if (!inf.delivered_bytes || !p) return 0;
        if (!planes) return (size_t)((p - 1) * extent + span);
        uint64_t end = 0;
        for (size_t i = 0; i < s; ++i)
            if (lay.size[i]) end = std::max(end, displ[i] + p * lay.size[i]);
        return (size_t)end;
    }

    // address of rank 0's block and byte stride between ranks, per (buffer, slot)
    void place(int buf, int slot, uint64_t &addr, uint64_t &stride) const {
        if (buf == ISO_BUF_SEND) {
            addr = (uint64_t)(uintptr_t)sendbuf + (op == ISO_OP_ALLTOALL ? lay.send_displ[(size_t)slot] : lay.send_displ[0]);
            stride = (lay.slot_major && op == ISO_OP_ALLTOALL) ? lay.size[(size_t)slot] : lay.send_extent;
        } else if (buf == ISO_BUF_RECV) {
            addr = (uint64_t)(uintptr_t)recvbuf + lay.recv_displ[(size_t)slot];
            stride = lay.slot_major ? lay.size[(size_t)slot] : lay.recv_extent;
        } else {
            addr = (uint64_t)(uintptr_t)workspace + wl.offset[(size_t)slot];
            stride = wl.size[(size_t)slot];
        }
    }

    // Fills the request's description and checks sizes, pointers and overlaps.
    int describe_and_check() {
        inf.op = op; inf.algorithm = pl.algorithm; inf.p = c.p; inf.s = c.s;
        inf.entries = pl.entries();
        inf.vector_bytes = 16;
        inf.block_bytes = 0;
        inf.delivered_bytes = 0;
        inf.launches = 0;
        for (size_t i = 0; i < s; ++i) {
            inf.block_bytes = std::max<uint64_t>(inf.block_bytes, lay.size[i]);
            inf.delivered_bytes += p * lay.size[i];
        }
        const uint64_t limit = ~uint64_t(0) >> 2;
        if (p && (lay.send_extent > limit / p || lay.recv_extent > limit / p)) return ISO_ERR_TOO_LARGE;

        inf.workspace_bytes = wl.bytes;
        inf.bytes_read = 0;
        for (const Round &r : pl.rounds)
            for (const iso_plan_entry_t &e : r.entries) inf.bytes_read += p * entry_size(e);
        inf.bytes_written = inf.bytes_read;

        const size_t send_len = buffer_len(lay.send_displ, lay.send_extent, lay.send_span,
                                           lay.slot_major && op == ISO_OP_ALLTOALL);
        const size_t recv_len = buffer_len(lay.recv_displ, lay.recv_extent, lay.recv_span, lay.slot_major);
        const size_t work_len = inf.delivered_bytes ? (size_t)wl.bytes : 0;
        if (send_len && !sendbuf) return ISO_ERR_ARG;
        if (recv_len && !recvbuf) return ISO_ERR_ARG;
        if (work_len && !workspace) return ISO_ERR_WORKSPACE;
        if (work_len > workspace_bytes) return arena ? ISO_ERR_SCRATCH : ISO_ERR_WORKSPACE;
        const Range rs{(uintptr_t)sendbuf, send_len}, rr{(uintptr_t)recvbuf, recv_len},
            rw{(uintptr_t)workspace, work_len};
        if (overlap(rs, rr) || overlap(rs, rw) || overlap(rr, rw)) return ISO_ERR_OVERLAP;
        if (inf.delivered_bytes == 0) return ISO_SUCCESS;       // all blocks empty, or no neighbours
        int st;
        if ((st = check_device_range(sendbuf, send_len)) != ISO_SUCCESS) return st;
        if ((st = check_device_range(recvbuf, recv_len)) != ISO_SUCCESS) return st;
        if (!arena && (st = check_device_range(workspace, work_len)) != ISO_SUCCESS) return st;
        return ISO_SUCCESS;
    }

    // Equal blocks in dense [p][s][m] receive rows that a workgroup can hold whole (deliver_launch).
    bool rows_fit_a_tile() const {
        const uint64_t m0 = s ? lay.size[0] : 0;
        if (!m0 || lay.slot_major || c.mesh || s > kLdsEntries || lay.recv_extent != s * m0) return false;
        const uint64_t width = uint64_t(1) << unit_log2_of(m0);
        if (m0 > kTileUnits * 16 || s * ((m0 + width - 1) / width) > kTileUnits || (m0 % 16 && s * m0 + 15 > kTileUnits * 16)) return false;
        for (size_t i = 0; i < s; ++i)
            if (lay.size[i] != m0 || lay.recv_displ[i] != i * m0) return false;
        return true;
    }

    // The last launch of the staged schedule has a kernel of its own for rows_fit_a_tile; anywhere else it runs as
    // one launch per dimension on the general kernels.  Blocks that are no multiple of 16, a launch per dimension -> rows, us,
    // many sets of buffers: 64^3, 6 neighbours, 100 B 123 -> 74, 1000 B 658 -> 576; 300^2, 8, 2500 B 974 -> 941; 24^3, 26,
    // 33 B 34 -> 24; allgather 48^3, 26, 700 B 915 -> 749.  A few single hops of kilobytes lose (152 x 186, 4 neighbours,
    // 2485 B, allgather 81 -> 99; one dimension, 36651, 500 B 14.8 -> 16.0).
    void rounds_as_launched() {
        for (size_t ri = 0; ri < pl.rounds.size(); ++ri) {
            const Round &r = pl.rounds[ri];
            bool whole = r.kind != ISO_ROUND_DELIVER;
            if (!whole) {
                whole = rows_fit_a_tile() && r.entries.size() == s;
                for (size_t i = 0; whole && i < s; ++i) whole = r.entries[i].dst_slot == (int)i;
            }
            if (whole) {
                bound_rounds.push_back({r.kind, r.dim, (int)ri, &r});
                continue;
            }
            for (int j = -1; j < c.d; ++j)
                for (const iso_plan_entry_t &pe : r.entries)
                    if (pe.dim == j) {
                        bound_rounds.push_back({j < 0 ? ISO_ROUND_SELF : ISO_ROUND_SHIFT, j, (int)ri, nullptr});
                        break;
                    }
        }
    }

    // All entries with their addresses, strides and their own unit width.
    int host_entries() {
        rounds.assign(bound_rounds.size(), {});
        bool first = true;
        for (size_t ri = 0; ri < bound_rounds.size(); ++ri) {
            const BoundRound &r = bound_rounds[ri];
            const std::vector<iso_plan_entry_t> &entries = pl.rounds[(size_t)r.of].entries;
            rounds[ri].reserve(entries.size());
            for (const iso_plan_entry_t &pe : entries) {
                if (!r.whole && pe.dim != r.dim) continue;
                HostEntry he{};
                he.size = entry_size(pe);
                he.dim = pe.dim;
                he.dst_slot = pe.dst_slot;
                he.dst_buf = pe.dst_buf;
                he.neighbor = pe.neighbor;
                he.moves = 1;
                he.along = ~0u;
                if (he.dim < 0 && r.kind == ISO_ROUND_SHIFT) he.dim = r.dim;
                if (he.size == 0) continue;                       // empty blocks make no move
                uint64_t src_stride = 0, dst_stride = 0;
                place(pe.src_buf, pe.src_slot, he.de.src, src_stride);
                place(pe.dst_buf, pe.dst_slot, he.de.dst, dst_stride);
                // the kernels multiply a rank by a 32-bit stride
                if ((src_stride | dst_stride) >> 32) return ISO_ERR_TOO_LARGE;
                he.de.src_stride = (uint32_t)src_stride;
                he.de.dst_stride = (uint32_t)dst_stride;
                he.de.shift = r.kind == ISO_ROUND_VECTOR ? (uint32_t)pe.neighbor : (uint32_t)pe.shift;
                const uint32_t l2 = unit_log2_of(he.size);
                const uint64_t width = uint64_t(1) << l2;
                const uint64_t units = (he.size + width - 1) >> l2;
                if (units > 0x7FFFFFFFu) return ISO_ERR_TOO_LARGE;
                he.de.units = (uint32_t)units;
                he.de.last_offset = he.size - width;
                he.de.ref = (uint32_t)pe.ref;
                // mesh: the non-periodic dimensions routed so far in which C^ref is non-zero
                uint32_t mask = 0;
                if (c.mesh && r.kind != ISO_ROUND_SELF)
                    for (int t = 0; t < c.d; ++t) {
                        const int l = pl.dim_order[(size_t)t];
                        if (!c.periodic[(size_t)l] && c.c(pe.ref, l) != 0) mask |= 1u << l;
                        if (r.kind == ISO_ROUND_SHIFT && l == r.dim) break;
                    }
                he.de.meta = l2 | (mask << 8);
                if (first) { size0 = he.size; first = false; }
                uniform = uniform && he.size == size0;
                min_log2 = std::min(min_log2, l2);
                rounds[ri].push_back(he);
            }
        }
        inf.vector_bytes = 1 << min_log2;
        return ISO_SUCCESS;
    }

    // The next launch of round `ri`: as many of its entries from `done` on as one launch takes.
    int next_launch(size_t ri, size_t &done) {
        const BoundRound &r = bound_rounds[ri];
        const std::vector<HostEntry> &ents = rounds[ri];
        Pending pd;
        pd.first_entry = table.size();
        pd.first_prefix = prefixes.size();
        Launch &l = pd.l;
        std::memset(&l, 0, sizeof(l));
        l.round = r.of;
        if (one_size) {                                  // split_by_size: the last round is that of the small blocks
            uniform = ri < large_sizes.size();
            size0 = ents[0].size;
            min_log2 = unit_log2_of(size0);
            l.chain_width = 1u << min_log2;
        }
        uint32_t k = 0;
        uint64_t total = 0;
        // staged schedule, last launch: whole receive rows through LDS (left as one round only for
        // regular [p][s][m] rows, see rounds_as_launched)
        const bool deliver = r.kind == ISO_ROUND_DELIVER;
        // staged schedule, the rounds: all destinations are planes of the workspace; small equal blocks
        // are re-tiled through LDS (any round of that schedule whose blocks of one rank fit a tile)
        // (a round between planes only is dense on both sides as it is: the plain kernel, plane after plane)
        const bool rows_later = pl.algorithm == ISO_ALG_COMBINED_STAGED || bound_rounds.back().kind == ISO_ROUND_DELIVER;
        bool all_planes = rows_later && !deliver && uniform && !c.mesh;
        for (const HostEntry &he : ents)
            all_planes = all_planes && he.de.src_stride == size0 && he.de.dst_stride == size0;
        const uint64_t st_upb = (size0 + (uint64_t(1) << min_log2) - 1) >> min_log2;
        const bool staged_round = rows_later && !deliver && !all_planes && uniform &&
                                  (pl.algorithm != ISO_ALG_COMBINED_STAGED || retiled()) && !lay.slot_major && !c.mesh &&
                                  r.kind != ISO_ROUND_VECTOR && done == 0 && ents.size() <= kLdsEntries &&
                                  ents.size() * st_upb <= kTileUnits && p * st_upb <= kMaxUnits;
        if (deliver) {
            deliver_launch(pd, ents, k, total);
        } else if (staged_round) {
            staged_round_launch(pd, r, ents, k, total);
        } else if (uniform && (!c.mesh || r.kind != ISO_ROUND_VECTOR || (c.d <= kVectorDims && (all_hops || ents.size() <= kLdsEntries)))) {
            const int st = regular_launch(pd, r, ents, done, all_planes, k, total);
            if (st != ISO_SUCCESS) return st;
        } else {
            const int st = block_launch(pd, r, ents, done, k, total);
            if (st != ISO_SUCCESS) return st;
        }
        l.policy = cache_policy(l, r);
        std::vector<Side> src_sides, dst_sides;
        src_sides.reserve(k);
        dst_sides.reserve(k);
        for (uint32_t q = 0; q < k; ++q) {
            const HostEntry &he = ents[done + q];
            src_sides.push_back(Side{he.de.src, he.de.src_stride, he.size});
            dst_sides.push_back(Side{he.de.dst, he.de.dst_stride, he.size});
        }
        describe_bytes(l, ents.data() + done, k);
        set_grid(l, (uint32_t)total, l.shift.k_all ? l.shift.k : k, l.eighths || page_resonant(src_sides) || page_resonant(dst_sides));
        pending.push_back(pd);
        done += k;
        return ISO_SUCCESS;
    }

    // Blocks that the staged schedule's rounds re-tile on their way from rows to planes: whole units at any size, others
    // from 48 MiB on (a launch of the plain kernel -> re-tiled: 32^3, 200 B 188 -> 137 us, 64^3, 100 B 745 -> 584; 24^3,
    // 100 B 33 -> 34).
    bool retiled() const { return size0 % 16 == 0 || inf.delivered_bytes > kLastLevelCacheBytes * 3 / 16; }

    // An entry loads its block once, whatever the moves that it stands for.  Only an allgather's share sources.
    void describe_bytes(Launch &l, const HostEntry *ents, uint32_t k) const {
        for (uint32_t q = 0; q < k; ++q) {
            l.bytes_written += p * ents[q].size * ents[q].moves;
            l.bytes_read += p * ents[q].size;
        }
        if (op == ISO_OP_ALLTOALL || !k) return;
        std::vector<uint64_t> sources(k);
        for (uint32_t q = 0; q < k; ++q) sources[q] = ents[q].de.src;
        std::sort(sources.begin(), sources.end());
        l.bytes_read = p * ents[0].size * (uint64_t)(std::unique(sources.begin(), sources.end()) - sources.begin());
    }

    // Cache policy of a launch whose kernel and arguments are set.  What decides is whether the blocks of the whole
    // collective (the receive buffer's size) stay in the last-level cache from one round to the next.  Figures in us,
    // a -> b being streaming -> the other policy unless said otherwise, first with one set of buffers repeated, then
    // with many sets in turn (1 GiB and more): a policy is taken where it gains in one and does not lose in the
    // other.
    //   All-to-all rounds read every block once: streaming loads and stores, except for collectives of up to 8 MiB
    //   (plain stores, 16^3, 64 B 13.1 -> 12.4 and 16.5 -> 15.3).  Further up plain stores lose with many sets (16^3,
    //   128 B 17.3 -> 15.9 and 19.5 -> 24; 20^3, 128 B 26.5 -> 23.3 and 28 -> 33.4; 60^2, 24 neighbours, 128 B 11.6
    //   -> 10.1 and 13.3 -> 15.9).
    //   Blocks that do not fill whole 64-byte sectors of rank-major rows gain further up.  Up to half the cache plain
    //   stores let neighbouring blocks meet there before a sector is written: blocks of less than a sector (64^3, 20
    //   B 293 -> 185 and 301 -> 214; 300^2, 24 neighbours, 25 B 82 -> 48 and 91 -> 63), and blocks up to 256 B that
    //   make two hops and more, so that much of what is written is read again (32^3, 100 B 123 -> 74 and 130 -> 107;
    //   8^4, 80 neighbours, 100 B 64 -> 44 and 76 -> 60; fewer hops: 300^2 star, 100 B 23 -> 20 and 28 -> 31; larger
    //   blocks: 16^3, 400 B 41 -> 33 and 45 -> 48; under a sixteenth of the cache, a twelfth on a mesh: 16^3 mesh,
    //   200 B 27 -> 23 and 31.5 -> 34).  Other blocks take cached loads there (100^2, 24 neighbours, 300 B 53 -> 46
    //   and 57 -> 57; 30^3 star, 600 B 47 -> 37 and 49 -> 48).  Between half and 9/8 of the cache: streaming loads,
    //   plain stores under a sector, and for two hops and more under 512 B (64^3, 36 B 495 -> 336 and 507 -> 395;
    //   32^3, 300 B 281 -> 219 and 285 -> 262; 300^2 star, 400 B 61 -> 57 and 63 -> 85), else cached loads (the same
    //   61 -> 50 and 63 -> 61; 64^3 star, 140 B 174 -> 120 and 178 -> 158; 30^3 star, 1000 B 71 -> 55 and 72 -> 72;
    //   not on a mesh from 512 B on: 1 to 3 % slower with many sets).  In the staged schedule blocks of 128 bytes and
    //   more take the cached loads (20^3, 200 B with plain stores 55 -> 41 and 57 -> 61).
    //   Allgather rounds may read a block several times: cached loads.  Streaming stores, except for blocks of less
    //   than a sector in rank-major rows of three and more dimensions, of which several launches write parts, while
    //   all of it fits (plain stores, 64^3, 32 B 120 -> 99 and 174 -> 160; 8^5, 40 random neighbours, 40 B 122 -> 76
    //   and 136 -> 96; 64^3 star, 40 B 53 -> 32 and 54 -> 47; the staged schedule's from an eighth of the cache on:
    //   32^3, 20 B 24 -> 22 and 23.6 -> 25).  Larger blocks and two dimensions: 30^3 star, 1000 B 47 -> 46 and 47 ->
    //   64; 32^3, 200 B 70 -> 57 and 82 -> 92; box 40^3, 160 B 106 -> 89 and 118 -> 131; 300^2, 24 neighbours, 56 B
    //   51 -> 39 and 61 -> 71.
    //   The staged schedule's kernels, all-to-all.  From an eighth of the cache (a sixteenth at 16 bytes, a sixth
    //   from 128 bytes on) up to half of it cached loads in both; the rounds store plainly if blocks do not fill
    //   sectors (64^3, 16 B 116 -> 97 and 118 -> 107; 44^3, 32 B 68 -> 58 and 70 -> 69; 9^4, 80 neighbours, 176 B 131
    //   -> 86 and 133 -> 111; under an eighth 32^3, 32 B 27 -> 27.5 and 29.5 -> 31) and stream at 64 B (40^3 89 -> 81
    //   and 90.5 -> 89; plain 75 and 93.5).  Up to 7/4 of it the rounds still gain from cached loads (64^3, 32 B 196
    //   -> 177 and 198 -> 186; 48^3, 80 B 195 -> 182 and 197 -> 188; 872 MB 617 -> 623).  Blocks of two and more
    //   whole sectors stream throughout (cached loads 32^3, 256 B 158 -> 148 and 159 -> 162; 9^4, 128 B 73 -> 61 and
    //   75 -> 78).  Rounds between planes of the workspace are dense on both sides whatever the block: as whole
    //   sectors.  Allgather: cached loads, streaming stores (the last launch with plain ones 64^3, 16 B 45 -> 45 and
    //   43 -> 49; 64^3 star, 64 B 22 -> 23 and 23 -> 29; 300^2, 24 neighbours, 48 B 37 -> 34 and 33 -> 36).
    //   Unequal blocks: cached loads, streaming stores.  All-to-all rounds whose blocks all have the same number of
    //   units stream their loads outside a sixteenth to all of the cache (against cached 40^3, 1024 and 1023 B 1474
    //   and 1487; 16^3, 64 and 63 B with many sets 17.7 and 18.6; inside 32^3, 100 and 99 B 127 and 101, 131 and 119,
    //   not in the staged schedule).  Plain stores up to a quarter of the cache for rank-major blocks of less than
    //   two sectors and unequal or single units (stencils 64^3, 4 B 151 -> 119 and 173 -> 152; 48^3, 9 B 89 -> 83 and
    //   116 -> 112; larger blocks: 24^3, 20 B 31 -> 28.5 and 40 -> 41; 20^3, 25 B 27 -> 25 and 34 -> 36.5; slot-major
    //   24^3, 16 B 16 -> 17.5 and 22 -> 25).  Blocks up to 128 bytes and larger ones in one launch, from a quarter of the
    //   cache on: by size (cached loads, streaming stores for all -> by size, stencils: 32^3, 64 B 351 -> 337 and 351 ->
    //   337; 64^3, 16 B 418 -> 374; 60 x 50 x 41, 25 B 323 -> 308; 16^4, 4 B 176 -> 167; 7^5, 4 B 286 -> 261; 16^3, 64 B
    //   56.4 -> 55.8 and 56.4 -> 55.6; under it 24^3, 25 B 45.2 -> 46.8 and 47.6 -> 47.3, 16^3, 16 B 13.4 -> 14.8 and
    //   16.2 -> 15.9; the staged schedule 32^3, 64 B 348 -> 354).
    //   The s-exchange writes whole rows and is indifferent to the stores; streaming loads where the send buffer of
    //   an all-to-all exceeds the cache (805 MB -4.6 %, 5.4 GB -3.8 %; 218 MB +17 %, an allgather +60 %) and no two
    //   blocks of a rank-major row share a 128-byte line (64 B +9 %, 100 B +7 %, 300 B +9 %).
    int cache_policy(const Launch &l, const BoundRound &r) const {
        const uint64_t bytes = inf.delivered_bytes;
        const uint64_t above = kLastLevelCacheBytes * 9 / 8;      // what still gains from the cache
        const bool a2a = op == ISO_OP_ALLTOALL, staged = pl.algorithm == ISO_ALG_COMBINED_STAGED;
        if (l.kernel == kStagedRoundKernel || l.kernel == kDeliverKernel) {
            const bool round = l.kernel == kStagedRoundKernel, whole = size0 % 64 == 0;
            if (!a2a) return 0;
            // Blocks that are no whole units, and rows in one launch of the other schedules: 32^3, 100 B with streaming
            // stores in the rounds 92 -> 78 us, 64^3, 72 B 585 -> 548; cached loads in them 24^3, 150 B 54 -> 48, 64^3,
            // 40 B 305 -> 363; cached loads in the last launch 32^3, 100 B 85 -> 78, 64^3, 100 B 748 -> 824.
            if (!staged || size0 % 16) {
                if (round) return bytes <= kLastLevelCacheBytes / 4 ? kPlainStores : kStreamLoads | kPlainStores;
                return bytes <= kLastLevelCacheBytes / 2 ? 0 : kStreamLoads;
            }
            if (bytes > kLastLevelCacheBytes * 7 / 4 || (whole && size0 >= 128)) return kStreamLoads;
            if (bytes > kLastLevelCacheBytes / 2) return round ? 0 : kStreamLoads;
            if (bytes <= kLastLevelCacheBytes / (size0 < 32 ? 16 : size0 < 128 ? 8 : 6)) return kStreamLoads;
            return round && !whole ? kPlainStores : 0;
        }
        if (l.kernel == kVectorKernel) {
            const bool lines = size0 % 128 == 0 || lay.slot_major;
            // Through all hops: where blocks make three of them and more, what the loads would keep is better left to the
            // stops (cached -> streaming loads: 8^5, 40 neighbours, 128 B 120 -> 115, 300 B 338 -> 320; 16^4, 30, 400 B 546
            // -> 526, 1 KiB 1426 -> 1388; fewer hops 64^3, 26, 300 B 1144 -> 1206, 1000 B 3743 -> 3888).
            if (all_hops && a2a && inf.entries >= 3 * (int64_t)s) return kStreamLoads;
            // Trie nodes beside the receive blocks, less than a sector: many of them, or beyond the cache, have to meet there
            // as those of the rounds do, before a sector is written (streaming -> plain stores: 9 x 8 x 8 x 9 x 8, 40 random
            // neighbours with 87 nodes more, 16 B 96 -> 29 and 108 -> 31, a launch per dimension 52 and 54; 16 x 16 x 15 x 15,
            // 30 and 42, 20 B 88 -> 30 and 73 -> 38; 12 x 12 x 11 x 12 x 12, 10 and 26, 20 B 96 -> 48 and 80 -> 53; fewer
            // 24 x 25 x 24, 40 and 23, 16 B 6.6 -> 6.6 and 7.1 -> 8.7; 16 x 16 x 16 x 15, 10 and 19, 32 B 20 -> 14 and 17 -> 20).
            if (all_hops && l.way == kStrides && size0 < 64 &&
                (inf.entries > (int64_t)s + 32 || inf.bytes_written > kLastLevelCacheBytes / 2))
                return kPlainStores;
            return a2a && l.vector_dims && lines && bytes > above ? kStreamLoads : 0;
        }
        if (l.kernel == kBlockKernel && all_hops) return kPlainStores;       // (block_through_stops)
        if (r.kind == ISO_ROUND_VECTOR) return 0;
        if (l.kernel == kBlockKernel) {
            if (inf.block_bytes < 128 && l.block.equal_units <= 1 && !lay.slot_major && bytes <= kLastLevelCacheBytes / 4)
                return kPlainStores;
            if (a2a && !staged && !c.mesh && !lay.slot_major && l.small_and_large && bytes > kLastLevelCacheBytes / 4) return kBySize;
            const bool cached = bytes > kLastLevelCacheBytes / 16 && bytes <= kLastLevelCacheBytes && !staged;
            return a2a && l.block.equal_units && !cached ? kStreamLoads : 0;
        }
        if (!a2a)
            return size0 < 64 && c.d >= 3 && !c.mesh && !lay.slot_major && bytes <= kLastLevelCacheBytes &&
                           (!staged || bytes > kLastLevelCacheBytes / 8)
                       ? kPlainStores
                       : 0;
        const bool dense = lay.slot_major || (l.kernel == kShiftKernel && l.entry_major);
        if (size0 % 64 && !dense && bytes <= above) {
            const bool read_again = inf.entries >= 2 * (int64_t)s;          // two hops per block and more
            if (bytes > kLastLevelCacheBytes / 2 && (size0 < 64 || (size0 < 512 && read_again)))
                return kStreamLoads | kPlainStores;
            if (size0 < 64) return kPlainStores;
            if (size0 < (staged ? 128u : 256u) && read_again && bytes > kLastLevelCacheBytes / (c.mesh || staged ? 12 : 16))
                return kPlainStores;
            return bytes > kLastLevelCacheBytes / 8 && (!c.mesh || size0 < 512) ? 0 : kStreamLoads;
        }
        return bytes <= kLastLevelCacheBytes / 32 ? kPlainStores : kStreamLoads;
    }

    // Every rank's receive row written in one piece.  Blocks of whole 16-byte units of the staged schedule keep the kernel
    // that moves units (64^3, 16 B 107 us against 109 by bytes; from 32 B on the two are within 1 %).
    void deliver_launch(Pending &pd, const std::vector<HostEntry> &ents, uint32_t &k, uint64_t &total) {
        Launch &l = pd.l;
        l.kernel = kDeliverKernel;
        DeliverArgs &da = l.deliver;
        l.by_bytes = size0 % 16 != 0 || pl.algorithm != ISO_ALG_COMBINED_STAGED;
        const uint64_t width = uint64_t(1) << min_log2, upb = (size0 + width - 1) / width;
        k = (uint32_t)s;
        da.p = (uint32_t)p;
        da.s = (uint32_t)s;
        da.upb = (uint32_t)upb;
        // at least one row has to fit, by bytes at any alignment of the receive buffer (rows_fit_a_tile)
        const uint64_t row = s * size0, row_units = std::max<uint64_t>(s * upb, l.by_bytes ? (row + 30) / 16 : 0);
        l.tile_units = row_units <= kSmallTileUnits ? kSmallTileUnits : kTileUnits;
        da.ranks = (uint32_t)std::min<uint64_t>(p, l.tile_units / (s * upb));
        if (l.by_bytes) {
            while (da.ranks * row + 15 > l.tile_units * 16) --da.ranks;
            // tiles that begin and end with whole sectors, as far as the rows allow it
            for (uint32_t part = 64; part >= 16; part /= 2) {
                const uint32_t whole = part / (uint32_t)std::gcd<uint64_t>(part, row);
                if (da.ranks < whole || da.ranks == p) continue;
                da.ranks -= da.ranks % whole;
                break;
            }
        }
        da.dst = (uint64_t)(uintptr_t)recvbuf;
        while (prefixes.size() % 4) prefixes.push_back(0);            // 16-byte aligned entries
        pd.first_prefix = prefixes.size();
        for (int rows = 1; rows >= 0; --rows)                          // rank-major sources first
            for (const HostEntry &he : ents) {
                if ((he.de.src_stride > size0) != (rows == 1)) continue;
                const DeliverEntry x = make_deliver_entry(c, he);
                da.k_rows += rows == 1;
                const uint32_t *words = (const uint32_t *)&x;
                prefixes.insert(prefixes.end(), words, words + sizeof(x) / 4);
            }
        da.rows = std::max(1u, da.k_rows * da.upb);
        da.plane = da.ranks * da.upb;
        da.row = l.by_bytes ? (uint32_t)size0 : (uint32_t)(s * upb);
        put(da.upb, da.mul_upb, da.shifts, 0);
        put(da.rows, da.mul_rows, da.shifts, 1);
        put(da.plane, da.mul_plane, da.shifts, 2);
        put(da.row, da.mul_row, da.shifts, 3);
        l.dyn_lds = l.by_bytes ? (uint32_t)((da.ranks * s * size0 + 31) & ~uint64_t(15))
                               : (uint32_t)(s * ((uint64_t)da.ranks * da.upb + 1) * 16);
        total = ((p + da.ranks - 1) / da.ranks) * kThreads;      // set_grid: one workgroup per tile
    }

    // Staged schedule, a round of small equal blocks: re-tiled through LDS.
    void staged_round_launch(Pending &pd, const BoundRound &r, const std::vector<HostEntry> &ents, uint32_t &k,
                             uint64_t &total) {
        Launch &l = pd.l;
        l.kernel = kStagedRoundKernel;
        k = (uint32_t)ents.size();
        StagedRoundArgs &sa = l.staged;
        const uint64_t width = uint64_t(1) << min_log2, upb = (size0 + width - 1) / width;
        l.pull = (uint32_t)(upb * width - size0);
        l.tail = l.pull != 0;
        // entries that read a rank-major buffer (rank stride larger than the block) first
        for (int rows = 1; rows >= 0; --rows)
            for (const HostEntry &he : ents)
                if ((he.de.src_stride > size0) == (rows == 1)) {
                    table.push_back(he.de);
                    sa.k_rows += rows == 1;
                }
        sa.p = (uint32_t)p;
        sa.k = k;
        sa.upb = (uint32_t)upb;
        const bool joined = second_dim >= 0 && &r == &bound_rounds[0];
        l.tile_units = k * upb <= kSmallTileUnits && !(joined && parts_of_sectors(k, upb)) ? kSmallTileUnits : kTileUnits;
        sa.ranks = (uint32_t)std::min<uint64_t>(p, l.tile_units / (k * upb));
        const bool shift = r.kind == ISO_ROUND_SHIFT;
        sa.inner = shift ? (uint32_t)c.inner[r.dim] : 1u;
        sa.pj = shift ? (uint32_t)c.dims[r.dim] : 1u;
        sa.row = std::max(1u, sa.k_rows * sa.upb);
        sa.plane = sa.ranks * sa.upb;
        put(sa.upb, sa.mul_upb, sa.shifts, 0);
        put(sa.row, sa.mul_row, sa.shifts, 1);
        put(sa.plane, sa.mul_plane, sa.shifts, 2);
        put(sa.inner, sa.mul_inner, sa.shifts, 3);
        put(sa.pj, sa.mul_pj, sa.more, 0);
        if (joined) {
            sa.inner2 = (uint32_t)c.inner[second_dim];
            sa.pj2 = (uint32_t)c.dims[second_dim];
            put(sa.inner2, sa.mul_inner2, sa.shifts2, 0);
            put(sa.pj2, sa.mul_pj2, sa.shifts2, 1);
        }
        l.dyn_lds = (uint32_t)(k * ((uint64_t)sa.ranks * sa.upb + 1) * width);
        total = ((p + sa.ranks - 1) / sa.ranks) * kThreads;      // set_grid: one workgroup per tile
    }

    // Two rounds in one launch hold more blocks of a rank, and a small tile fewer ranks; where their pieces of the planes end
    // inside a sector, large tiles beyond half the last-level cache (two launches, one with small tiles, with large ones: 8^5,
    // 40 neighbours, 112 B 228, 239, 217, 208 B 439, 475, 406, 224 B 441, 491, 424; 16^4, 80, 48 B 318, 324, 284, 144 B 1020,
    // 1225, 969; small to large tiles otherwise: whole sectors 16^4, 96 B +7 %, smaller ones 20^3, 288 B with many sets +7 %).
    bool parts_of_sectors(uint64_t k, uint64_t upb) const {
        const uint64_t ranks = kSmallTileUnits / (k * upb);
        return ranks <= 5 && ranks * size0 % 64 && inf.delivered_bytes > kLastLevelCacheBytes / 2;
    }

    // Regular blocks: every entry has `chunks` units of the request's common width (a mesh's s-exchange of more
    // dimensions or neighbours than VectorEntry and LDS take uses the block kernel).
    int regular_launch(Pending &pd, const BoundRound &r, const std::vector<HostEntry> &ents, size_t done,
                       bool all_planes, uint32_t &k, uint64_t &total) {
        Launch &l = pd.l;
        const uint64_t width = uint64_t(1) << min_log2;
        const uint64_t chunks = (size0 + width - 1) >> min_log2;
        l.tail = (size0 & (width - 1)) != 0;
        const uint64_t per_entry = p * chunks;
        if (chunks > 0x7FFFFFFFu || per_entry > kMaxUnits) return ISO_ERR_TOO_LARGE;
        k = (uint32_t)std::min<uint64_t>(kMaxUnits / per_entry, ents.size() - done);
        if (all_hops) {                                  // a table in LDS for each launch, of equal parts
            const uint32_t parts = ((uint32_t)ents.size() + kLdsEntries - 1) / kLdsEntries;
            k = std::min(k, ((uint32_t)ents.size() + parts - 1) / parts);
        }
        total = per_entry * k;
        l.kernel = r.kind == ISO_ROUND_VECTOR ? kVectorKernel : c.mesh ? kMeshShiftKernel : kShiftKernel;
        // one block per wavefront: blocks that are a multiple of 1 KiB; on rank-major buffers only up
        // to 2 KiB (measured: no gain from 4 KiB on)
        l.uniform_waves = l.kernel == kShiftKernel && min_log2 == 4 && !l.tail && chunks % 64 == 0 &&
                          (lay.slot_major || chunks <= 128);
        l.pull = (uint32_t)(chunks * width - size0);
        const bool shift = r.kind == ISO_ROUND_SHIFT;
        if (l.kernel == kVectorKernel) {
            VectorArgs &va = l.vec;
            va.d = c.d;
            va.chunks = (uint32_t)chunks;
            va.p = (uint32_t)p;
            put(va.chunks, va.mul_chunks, va.shifts, 0);
            put(k, va.mul_k, va.shifts, 1);
            put(va.p, va.mul_p, va.shifts, 2);
            // Blocks of four hops and more store more stops than rows: block by block the stops of a plane meet in the
            // last-level cache (rank by rank -> here: 8^5, 40 neighbours, 128 B 115 -> 103 us, 1 KiB 974 -> 767, 3000 B
            // 3096 -> 2715, 8 KiB 8604 -> 7305; 12^5, 384 B 2723 -> 2380; 600 B 146 -> 155; 3.4 hops, 16^4, 30
            // neighbours, 256 B 291 -> 309, 1 KiB 1388 -> 1183, 1500 B 706 -> 736)
            l.entry_major = lay.slot_major || all_planes ||
                            (all_hops && inf.entries >= 4 * (int64_t)s && (size0 % 128 == 0 || size0 >= 1024));
            vector_launch(l, ents.data() + done, k, chunks);
            // several blocks of a rank-major row to a line, read by ranks that lie near each other: one eighth of the
            // ranks per XCD keeps the line in its L2 (runs -> eighths, one set of buffers repeated and many in turn:
            // 64^3, 20 B 65 -> 54 and 73 -> 78 us, 300^2, 24 neighbours, 16 B 13.6 -> 12.2 and 17.8 -> 17.8, 50^3 star,
            // 20 B 10.3 -> 6.7 and 12 -> 11.5; 64^3, 40 B 103 -> 113 and 115 -> 123)
            if (op == ISO_OP_ALLTOALL && !l.entry_major && ents.size() > 1) l.eighths = size0 <= 32;
            if (op == ISO_OP_ALLGATHER && ents.size() > 1) allgather_order(l, ents.data() + done, k);
            if (l.vec.per && !c.mesh) total = per_entry * ((k + l.vec.per - 1) / l.vec.per);
            if (l.vector_dims) return ISO_SUCCESS;
        } else if (l.kernel == kMeshShiftKernel) {
            MeshArgs &ma = l.mesh_shift;
            ma.inner = shift ? (uint32_t)c.inner[r.dim] : 1u;
            ma.pj = shift ? (uint32_t)c.dims[r.dim] : 1u;
            bool packed = true;                                // in all entries or in none
            const size_t first = table.size();
            for (uint32_t q = 0; q < k; ++q) {
                table.push_back(ents[done + q].de);
                const DevEntry &de = ents[done + q].de;
                packed = packed && pack_reference(c.can.data() + (size_t)de.ref * c.d, c.d, de.meta >> 8, table.back());
            }
            for (uint32_t q = 0; q < k && !packed; ++q) table[first + q] = ents[done + q].de;
            ma.torus = torus_bits(c.d, shift ? r.dim : -1, periodic_mask(), packed);
            ma.chunks = (uint32_t)chunks;
            ma.p = (uint32_t)p;
            l.entry_major = lay.slot_major;
            put(ma.chunks, ma.mul_chunks, ma.shifts, 0);
            put(k, ma.mul_k, ma.shifts, 1);
            put(ma.inner, ma.mul_inner, ma.shifts, 2);
            put(ma.pj, ma.mul_pj, ma.shifts, 3);
            put(ma.p, ma.mul_p, ma.more, 0);
            const uint32_t group_log2 =
                bits_by_wave ? interior_group_log2(c, lay.slot_major, ents.data() + done, k, chunks) : kTileLog2;
            const std::vector<uint32_t> bits =
                mesh_interior_units(c, lay.slot_major, ents.data() + done, k, group_log2, total, chunks, p);
            ma.torus |= (uint32_t)(group_log2 == kTileLog2) << 11;
            prefixes.insert(prefixes.end(), bits.begin(), bits.end());
            if (pl.algorithm == ISO_ALG_COMBINED && !arena) {
                l.outside_units = ((total - 1) >> group_log2) + 1;
                for (uint32_t w : bits) l.outside_units -= (uint32_t)__builtin_popcount(w);
                l.outside_units <<= group_log2;
            }
            return ISO_SUCCESS;
        } else {
            ShiftArgs &sa = l.shift;
            sa.inner = shift ? (uint32_t)c.inner[r.dim] : 1u;
            sa.pj = shift ? (uint32_t)c.dims[r.dim] : 1u;
            sa.chunks = (uint32_t)chunks;
            sa.p = (uint32_t)p;
            l.entry_major = lay.slot_major || all_planes;
            // blocks of 2 KiB and more on rank-major buffers: groups of 64 ranks (three tori: 2 KiB -1 to
            // -3 % of the step, 4 KiB 0 to -3 %, 8 KiB -5 %; at 1 KiB and below between -1.5 and +1 %:
            // left alone.  Groups of 32 to 256 ranks measure alike, smaller ones do nothing)
            if (!l.entry_major && size0 >= 2048 && p >= kRankGroup) sa.grouped = (uint32_t)((p / kRankGroup) * kRankGroup * k);
            put(sa.chunks, sa.mul_chunks, sa.sh_chunks, 0);
            put(k, sa.mul_k, sa.sh_k, 0);
            put(sa.inner, sa.mul_inner, sa.sh_inner, 0);
            put(sa.pj, sa.mul_pj, sa.sh_pj, 0);
            put(sa.p, sa.mul_p, sa.more, 0);
            if (sa.grouped) put(k * kRankGroup, sa.mul_group_k, sa.more, 1);
            if (op == ISO_OP_ALLGATHER && push_launch(l, ents.data() + done, k, per_entry)) {
                total = per_entry * l.shift.k;
                return ISO_SUCCESS;
            }
        }
        for (uint32_t q = 0; q < k; ++q) table.push_back(ents[done + q].de);
        return ISO_SUCCESS;
    }

    // Allgather rounds in push form: where the launch's entries read at most three quarters as many blocks as they
    // write (64^3, 26 neighbours, 128 B, one launch per dimension 276 -> 201 us; 200^2, 24 neighbours, 512 B 139
    // -> 105; with 40 random neighbours in 8^5 nearly every block has a single child in most dimensions and the
    // pull form is 1 to 2 % faster), and where that many reads still fill the chip (16^3, 24 neighbours, 16 B, 16
    // workgroups: 10.0 -> 12.2 us).  What a workgroup writes then lies at different ranks, so every block has to
    // be part of a dense plane (slot-major 64^3, 300 B 600 -> 521 us) or whole 64-byte sectors, from 1 KiB on 32
    // (200 B on rank-major rows 238 -> 284 us, 320 B 92 -> 74, 64 B level, 2080 B 130 -> 111).  A launch of two moves
    // from one block (a star) saves one read of three accesses: whole 128-byte lines only (50^3, 64 B 13.6 -> 16.3 us,
    // 32^3, 1056 B 51 -> 60, 256^2, 1056 B 69 -> 77; lines 50^3, 256 B 50 -> 43, 256^2, 512 B 34 -> 28).
    bool push_launch(Launch &l, const HostEntry *ents, uint32_t k, uint64_t per_entry) {
        if (k > kLdsEntries) return false;
        const uint32_t mask = size0 >= 1024 ? 31u : 63u;
        bool lines = true;
        for (uint32_t q = 0; q < k; ++q) {
            const DevEntry &de = ents[q].de;
            if (de.dst_stride == size0) continue;
            if ((de.dst | de.dst_stride | size0) & mask) return false;
            lines = lines && ((de.dst | de.dst_stride | size0) & 127u) == 0;
        }
        std::vector<DevEntry> by_source;
        std::vector<uint32_t> first;
        std::vector<bool> taken(k, false);
        for (uint32_t q = 0; q < k; ++q) {
            if (taken[q]) continue;
            first.push_back((uint32_t)by_source.size());
            for (uint32_t w = q; w < k; ++w)
                if (!taken[w] && ents[w].de.src == ents[q].de.src && ents[w].de.src_stride == ents[q].de.src_stride) {
                    taken[w] = true;
                    by_source.push_back(ents[w].de);
                }
        }
        const uint32_t n = (uint32_t)first.size();
        if (4 * n > 3 * k || per_entry * n < 256 * kThreads) return false;
        if (k == 2 && !lines) return false;
        first.push_back(k);
        table.insert(table.end(), by_source.begin(), by_source.end());
        prefixes.insert(prefixes.end(), first.begin(), first.end());
        l.uniform_waves = false;
        l.shift.grouped = 0;
        l.shift.k_all = k;
        l.shift.k = n;
        l.shift.sh_k = 0;
        put(n, l.shift.mul_k, l.shift.sh_k, 0);
        return true;
    }

    // Moves by full vectors of equal blocks.  Up to kVectorDims dimensions and as many entries as the LDS
    // table takes: VectorEntry records (equal strides on each side, which equal blocks of one layout have: place()).
    // Other launches keep the general tables, on a mesh the block kernel (next_launch).
    void vector_launch(Launch &l, const HostEntry *ents, uint32_t k, uint64_t chunks) {
        VectorArgs &va = l.vec;
        bool packed = c.d <= kVectorDims && k <= kLdsEntries;
        bool one_stride = true;
        for (uint32_t q = 0; packed && q < k; ++q) {
            one_stride = one_stride && ents[q].de.dst_stride == ents[0].de.dst_stride;
            packed = ents[q].de.src_stride == ents[0].de.src_stride && (one_stride || all_hops);
        }
        if (!packed) return;
        l.vector_dims = c.d <= 3 ? 3 : kVectorDims;
        if (c.mesh)
            for (int j = 0; j < kVectorDims; ++j) va.per |= (uint32_t)(c.d - 1 - j >= 0 && c.periodic[(size_t)(c.d - 1 - j)]) << j;
        l.uniform_waves = min_log2 == 4 && !l.tail && chunks % 64 == 0;
        va.src_stride = ents[0].de.src_stride;
        va.dst_stride = ents[0].de.dst_stride;
        if (all_hops) l.way = op == ISO_OP_ALLTOALL ? kStops : one_stride ? 0 : kStrides;
        if (c.mesh) l.way |= kMesh;
        for (int j = 0; j < kVectorDims; ++j) {                  // last dimension first, absent ones of size 1
            const int l_dim = c.d - 1 - j;
            va.last[j] = l_dim < 0 ? 1u : (uint32_t)c.dims[(size_t)l_dim];
            if (j + 1 < kVectorDims)
                put(va.last[j], va.mul_last[j], j == 0 ? va.shifts : j < 3 ? va.more : va.shift_last3, j == 0 ? 3 : j < 3 ? j - 1 : 0);
        }
        for (uint32_t q = 0; q < k; ++q) {
            VectorEntry ve{};
            ve.src = ents[q].de.src;
            ve.dst = ents[q].de.dst;
            for (int j = 0; j < c.d; ++j) {
                if (!(ents[q].along >> (c.d - 1 - j) & 1u)) continue;
                const uint32_t cj = (uint32_t)c.c((int)ents[q].de.shift, c.d - 1 - j);
                ve.c[j] = cj;
                ve.back += cj * (uint32_t)c.inner[(size_t)(c.d - 1 - j)];
            }
            ve.way = ents[q].way;
            DevEntry slot;
            std::memcpy(&slot, &ve, sizeof(slot));
            table.push_back(slot);
        }
    }

    // The fused s-exchange of an allgather reads every block once per neighbour; which L2 those reads find it in
    // decides between three forms.
    //   Rank-major: one contiguous eighth of the ranks per XCD (l.eighths) keeps a neighbourhood's blocks in that
    //   XCD's 4 MiB (64^3, 26 neighbours, 128 B 166 -> 144 us, 60 x 50 x 41, 200 B 129 -> 113, 256^2 star, 1 KiB
    //   150 -> 128; send buffers that every L2 holds whole are up to 9 % faster with interleaved runs).  Not where a
    //   run of tiles holds several times the ranks between the outermost neighbours (one dimension): its reads meet in
    //   one L2 anyway, and the eight streams of a large launch lie at equal offsets (262144 ranks, 2 neighbours, 256 B
    //   with many sets of buffers 42 us in runs, 51 in eighths; 131072, 512 B 42 and 52; 262144, 4 neighbours, 64 B 13.8
    //   and 13.8, one set repeated 13.7 and 12.3).  Where the
    //   ranks between the outermost neighbours hold far more than an L2, push (8^5, 40 random neighbours, 4 KiB
    //   1421 -> 985 us, 1 KiB 344 -> 268; a window of 8.4 MiB still pulls faster, 512 against 652 us, unless what
    //   misses the L2 misses the last-level cache as well, 200^2 star, 8 KiB 989 -> 845).  Push writes the
    //   blocks of a row from distant places: only for blocks that are whole 128-byte lines (200 B: 320 us).
    //   Slot-major: the ranks of an entry's plane come in order, so each XCD reads the same eighth of the send
    //   buffer for every entry.  Push from where that eighth no longer fits its L2 (64^3, 128 B 231 -> 152 us,
    //   300 B 563 -> 491; 25 MiB to send: pull 126, push 166).  Here push writes runs of consecutive ranks, 4
    //   entries at a time being 2 to 8 % faster than 8 or all.
    //   Trie nodes in the workspace beside the receive blocks: push 4 at a time (8^5, 40 random neighbours, 4 KiB 2, 4, 8 at a
    //   time 3507, 2975, 3029; 1 KiB slot-major 865, 724, 755; pull 3807 and 1085), slot-major also where the eighth fits, 2 at
    //   a time (16^4, 30, 256 B pull 272, push 195; 300 B 350 and 311; 8^5, 500 B 495 and 415).
    //   All hops of blocks of whole lines push whatever the window, where the send buffer exceeds the last-level cache
    //   (a launch per dimension, pull, push: 400 x 420, 8 neighbours, 2 KiB 677, 860, 580; 250 x 260, 8, 5 KiB 686, 804,
    //   577; 400 x 420, 10, 2 KiB 937, 1236, 933).
    //   All receive blocks, slot-major: an XCD meets the same ranks in every plane, and its reads stay in its L2, only if a
    //   plane is nearly a multiple of the runs of all XCDs (set_grid).  20^3, 26 neighbours, pull and push 2 at a time: 1024
    //   to 1072 B, up to 3/8 of a run off 32 to 42 and 37 to 48, 1104 B, 7/8 off, 58 and 48, 1120 B 62 and 52; half as many
    //   XCDs off, 784 B 24 and 33, 800 B, 1/4 of a run further, 35 and 34.  Else push 2 at a time from 6 MiB to send on (a
    //   launch per dimension, pull, push: 191 x 177, 24 neighbours, 640 B 109, 137, 108; 41 x 49 x 53, 24, 192 B 106, 120,
    //   106; 20 x 21 x 24, 26, 1788 B 115, 129, 104; 12 x 10^3, 40, 1813 B 212, 233, 192; 7 x 5 x 8 x 8, 80, 2500 B (5.3 MiB)
    //   116, 82, 95).
    void allgather_order(Launch &l, const HostEntry *ents, uint32_t k) {
        const uint64_t l2 = uint64_t(4) << 20, sent = p * size0;
        const bool nodes = all_hops && pl.work_slots > 0;
        if (lay.slot_major) {
            if (c.mesh) return;
            if (l.vector_dims && sent > 7 * l2) l.vec.per = std::min(k, 4u);
            else if (l.vector_dims && (nodes || (all_hops && sent > l2 * 3 / 2 && !planes_meet()))) l.vec.per = std::min(k, 2u);
            return;
        }
        int64_t lo = 0, hi = 0;                                  // the neighbours' linear distances, shortest way round
        bool lines = true;
        for (uint32_t q = 0; q < k; ++q) {
            int64_t at = 0;
            for (int j = 0; j < c.d; ++j) {
                const int64_t cj = c.c((int)ents[q].de.shift, j), pj = c.dims[(size_t)j];
                at += (2 * cj > pj ? cj - pj : cj) * c.inner[(size_t)j];
            }
            lo = std::min(lo, at);
            hi = std::max(hi, at);
            lines = lines && ((ents[q].de.dst | ents[q].de.dst_stride | size0) & 127u) == 0;
        }
        const uint64_t window_ranks = std::min<uint64_t>(p, (uint64_t)(hi - lo) + 1), window = window_ranks * size0;
        const uint64_t run = uint64_t(128) * kThreads << min_log2;      // bytes written by a run of tiles (set_grid)
        l.eighths = sent > l2 && 4 * window_ranks * k * size0 > run;
        if (l.vector_dims && !c.mesh && lines && (window > 3 * l2 || ((window > l2 || all_hops) && sent > kLastLevelCacheBytes))) {
            l.vec.per = std::min(k, nodes ? 4u : 8u);
            l.eighths = false;
        }
    }

    // Slot-major: do the runs of one XCD hold the same ranks in every plane?  (see allgather_order)
    bool planes_meet() const {
        const uint64_t run = uint64_t(128) * kThreads, plane = p * ((size0 + (uint64_t(1) << min_log2) - 1) >> min_log2);
        const uint64_t off = plane % (8 * run), far = std::min(off, 8 * run - off);
        return far <= run * 3 / 8 || (far >= 4 * run - run / 8 && far <= 4 * run);
    }

    // Irregular blocks, or a mesh's s-exchange: as many entries as fit the 32-bit unit index.
    int block_launch(Pending &pd, const BoundRound &r, const std::vector<HostEntry> &ents, size_t done, uint32_t &k,
                     uint64_t &total) {
        Launch &l = pd.l;
        l.kernel = kBlockKernel;
        l.mesh = c.mesh;
        BlockArgs &b = l.block;
        b.torus = torus_bits(c.d, r.kind == ISO_ROUND_SHIFT ? r.dim : -1, periodic_mask());
        // per launch: k + 1 prefix values, then k multipliers of the divisions by the entries'
        // unit counts (the two shifts of each go into the entry's meta word)
        const bool entry_major = lay.slot_major;
        const uint64_t scale = entry_major ? p : 1;    // prefix counts all ranks' units, or one row's
        uint64_t row_units = 0;
        prefixes.push_back(0);
        while (done + k < ents.size() && (!all_hops || k < kLdsEntries)) {
            const uint64_t next = row_units + ents[done + k].de.units;
            if (next * p > kMaxUnits) break;
            row_units = next;
            DevEntry de = ents[done + k].de;
            const FastDiv by_units = make_fastdiv(de.units);
            de.meta |= (by_units.sh1 << 24) | (by_units.sh2 << 25);
            if (all_hops) de.ref = ents[done + k].way ? (uint32_t)((ents[done + k].way - (uint64_t)(uintptr_t)workspace) / 16) : 0u;
            table.push_back(de);
            prefixes.push_back((uint32_t)(row_units * scale));
            ++k;
        }
        if (k == 0) return ISO_ERR_TOO_LARGE;          // one block plane alone is too large
        for (uint32_t q = 0; q < k; ++q) prefixes.push_back(make_fastdiv(ents[done + q].de.units).mul);
        total = row_units * p;
        l.entry_major = entry_major;
        l.vector_round = r.kind == ISO_ROUND_VECTOR;
        if (all_hops) {
            l.way = kStops;
            l.vector_dims = c.d <= 3 ? 3 : kVectorDims;
            b.work = (uint64_t)(uintptr_t)workspace;
        }
        b.equal_units = ents[done].de.units;
        for (uint32_t q = 1; q < k; ++q)
            if (ents[done + q].de.units != b.equal_units) b.equal_units = 0;
        const auto is_small = [](const HostEntry &he) { return he.de.units <= kSmallUnits; };
        const auto n_small = std::count_if(ents.begin() + (ptrdiff_t)done, ents.begin() + (ptrdiff_t)(done + k), is_small);
        l.small_and_large = n_small > 0 && n_small < (ptrdiff_t)k;
        b.plane = b.equal_units ? (uint32_t)(p * b.equal_units) : 1u;
        b.row = (uint32_t)row_units;
        // shift rounds on rank-major buffers: ranks in groups (not the staged schedule, whose tiny
        // blocks travel through dense planes: +1 % there; not the s-exchange: +1 to +4 %)
        if (!entry_major && r.kind != ISO_ROUND_VECTOR && pl.algorithm != ISO_ALG_COMBINED_STAGED &&
            p >= kBlockGroup) {
            l.block_groups = true;
            b.grouped = (uint32_t)((p / kBlockGroup) * kBlockGroup * row_units);
            b.plane = b.equal_units ? kBlockGroup * b.equal_units : 1u;
            put((uint32_t)(row_units * kBlockGroup), b.mul_group_row, b.more, 1);
        }
        const bool shift = r.kind == ISO_ROUND_SHIFT;
        b.inner = shift ? (uint32_t)c.inner[r.dim] : 1u;
        b.pj = shift ? (uint32_t)c.dims[r.dim] : 1u;
        put(b.row, b.mul_row, b.shifts, 0);
        put(b.inner, b.mul_inner, b.shifts, 1);
        put(b.pj, b.mul_pj, b.shifts, 2);
        put(b.equal_units ? b.equal_units : 1u, b.mul_units, b.shifts, 3);
        put(b.plane, b.mul_plane, b.more, 0);
        return ISO_SUCCESS;
    }

    // One device table: the entries, then the dimensions and the [s][d] residues, then what single launches read besides
    // (prefix arrays of irregular launches, the mesh's interior bitmaps, the records of the staged
    // schedule's last launch); then the launches get their addresses in it.  The residues keep their place in it
    // but are written only where a kernel reads them (a launch of its own in the allocation-free call: 8^3, 26
    // neighbours, 64 B 13.5 -> 10.7 us).
    int upload() {
        const size_t entry_bytes = table.size() * sizeof(DevEntry);
        const size_t c_bytes = residue_bytes();
        const size_t off_bytes = sizeof(TorusDims) + c_bytes;
        bool reads_residues = false;
        for (const Pending &pd : pending)
            reads_residues = reads_residues || pd.l.kernel == kMeshShiftKernel || pd.l.kernel == kBlockKernel ||
                             (pd.l.kernel == kVectorKernel && !pd.l.vector_dims);
        std::vector<uint32_t> torus;                     // TorusDims and the residues behind it
        if (reads_residues) {
            torus.resize(sizeof(TorusDims) / 4);
            TorusDims &td = *(TorusDims *)torus.data();
            for (int j = 0; j < c.d; ++j) {
                td.d_dims[j] = make_fastdiv((uint32_t)c.dims[(size_t)j]);
                td.inner[j] = (uint32_t)c.inner[(size_t)j];
            }
            torus.insert(torus.end(), c.can.begin(), c.can.end());
        }
        const size_t off_used = torus.size() * sizeof(uint32_t);
        const size_t pre_bytes = prefixes.size() * sizeof(uint32_t);
        size_t prefix_at = entry_bytes + off_bytes;
        char *dev = nullptr;
        int st;
        if (arena) {
            // (TorusDims has room of its own behind table_bytes)
            if (entry_bytes + c_bytes + pre_bytes > arena->table_bytes) return ISO_ERR_SCRATCH;
            dev = (char *)arena->table;
            if (!off_used) {                             // entries and prefixes next to each other: 3 KiB a launch
                std::vector<uint32_t> words((entry_bytes + pre_bytes) / 4);
                if (entry_bytes) std::memcpy(words.data(), table.data(), entry_bytes);
                std::copy(prefixes.begin(), prefixes.end(), words.begin() + (ptrdiff_t)(entry_bytes / 4));
                if ((st = store_table(*arena, 0, words.data(), entry_bytes + pre_bytes)) != ISO_SUCCESS) return st;
                prefix_at = entry_bytes;
            } else {
                if ((st = store_table(*arena, 0, table.data(), entry_bytes)) != ISO_SUCCESS) return st;
                if ((st = store_table(*arena, entry_bytes, torus.data(), off_used)) != ISO_SUCCESS) return st;
                if ((st = store_table(*arena, prefix_at, prefixes.data(), pre_bytes)) != ISO_SUCCESS) return st;
            }
        } else if (entry_bytes + off_bytes + pre_bytes) {
            const size_t bytes = entry_bytes + off_bytes + pre_bytes;
            ISO_HIP_TRY(hipMalloc(&rq.dev_table, bytes));
            dev = (char *)rq.dev_table;
            if (!off_used && !pre_bytes) {
                if (entry_bytes) ISO_HIP_TRY(hipMemcpy(dev, table.data(), entry_bytes, hipMemcpyHostToDevice));
            } else {
                std::vector<char> host(bytes);
                if (entry_bytes) std::memcpy(host.data(), table.data(), entry_bytes);
                if (off_used) std::memcpy(host.data() + entry_bytes, torus.data(), off_used);
                if (pre_bytes) std::memcpy(host.data() + prefix_at, prefixes.data(), pre_bytes);
                ISO_HIP_TRY(hipMemcpy(dev, host.data(), bytes, hipMemcpyHostToDevice));
            }
        }
        const DevEntry *dev_entries = (const DevEntry *)dev;
        const TorusDims *dev_dims = (const TorusDims *)(dev + entry_bytes);
        const uint32_t *dev_prefix = (const uint32_t *)(dev + prefix_at);
        for (Pending &pd : pending) {
            if (pd.l.kernel == kChainKernel) {
                pd.l.chain.table = (const ChainHop *)(dev_prefix + pd.first_prefix);
            } else if (pd.l.kernel == kVectorKernel) {
                pd.l.vec.entries = dev_entries + pd.first_entry;
                pd.l.vec.dims = dev_dims;
            } else if (pd.l.kernel == kMeshShiftKernel) {
                pd.l.mesh_shift.entries = dev_entries + pd.first_entry;
                pd.l.mesh_shift.dims = dev_dims;
                pd.l.mesh_shift.interior = dev_prefix + pd.first_prefix;
            } else if (pd.l.kernel == kDeliverKernel) {
                pd.l.deliver.entries = (const DeliverEntry *)(dev_prefix + pd.first_prefix);
            } else if (pd.l.kernel == kStagedRoundKernel) {
                pd.l.staged.entries = dev_entries + pd.first_entry;
            } else if (pd.l.kernel == kBlockKernel) {
                pd.l.block.entries = dev_entries + pd.first_entry;
                pd.l.block.prefix = dev_prefix + pd.first_prefix;
                pd.l.block.dims = dev_dims;
            } else {
                pd.l.shift.entries = dev_entries + pd.first_entry;
                pd.l.shift.groups = dev_prefix + pd.first_prefix;
            }
            (rq.launches.size() < n_listed ? rq.launches : rq.start_launches).push_back(pd.l);
        }
        inf.launches = (int32_t)rq.launches.size();
        return ISO_SUCCESS;
    }
};

inline int bind_request(BoundRequest &rq, const Plan &plan, const Comm &c, const Layout &lay, const void *sendbuf,
                        void *recvbuf, void *workspace, size_t workspace_bytes,
                        const StaticArena *arena = nullptr) {
    return Binder(rq, plan, c, lay, sendbuf, recvbuf, workspace, workspace_bytes, arena).run();
}

}  // namespace iso

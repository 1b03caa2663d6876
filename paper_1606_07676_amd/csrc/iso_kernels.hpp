// gfx950 kernels for isomorphic sparse collectives: pure data movement.
//
// One launch executes one round of a schedule: for every rank R and every entry
// e of the round it copies one block of m bytes
//
//     dst_e[R]  <-  src_e[ source rank of R ]
//
// where the source rank is R moved back v_e steps along one torus dimension
// (message-combining rounds, Section 5 / Algorithm 1 of the paper), R itself
// (zero offsets), or R (-) C^e (the straightforward exchange of Section 3).
// Entries carry absolute block addresses for rank 0 and the byte stride between
// consecutive ranks, so the same kernel reads and writes the user's rank-major
// [p][s][m] buffers and the workspace without pack or unpack copies.
//
// Work decomposition: the launch is a flat array of `vector-width` byte units
// ordered (rank, entry, chunk-in-block), chunk fastest, ONE unit per lane
// (slot-major buffers, one plane of p blocks per neighbour: (entry, rank, chunk),
// so that every wavefront access is one dense kilobyte of one plane).
// Consecutive lanes touch consecutive 16-byte pieces of one block, then the next
// block of the same rank: every wavefront load/store covers whole blocks, and a
// 256-lane workgroup covers 4 KiB of consecutive units.  Measured on MI355X,
// one unit per lane with the maximum number of resident wavefronts beats any
// per-lane unrolling (2, 4, 8 units per lane lose 3 %, 15 %, 50 %), for plain
// copies as well as for these gathers.  Which loads and stores are streaming
// (non-temporal) depends on how the collective's blocks compare with the
// last-level cache: see cache_policy in iso_bind.hpp.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "iso.h"
#include "iso_fastdiv.hpp"

namespace iso {

constexpr int kThreads = 256;
constexpr uint32_t kLdsEntries = 128;   // rounds with at most this many entries stage their table in LDS

struct alignas(16) DevEntry {
    uint64_t src;          // address of rank 0's source block
    uint64_t dst;          // address of rank 0's destination block
    uint32_t src_stride;   // bytes between consecutive ranks in the source buffer; below 2^32 (checked
    uint32_t dst_stride;   // when the request is bound), so that rank * stride + base is one 32x32+64 multiply-add
    uint32_t shift;        // SHIFT rounds: residue v; VECTOR rounds: neighbour index
    uint32_t units;        // block launches: units of this entry's block, block size / unit width rounded up
    uint32_t meta;         // block launches: bits 0-7 log2 of the unit width in bytes;
                           // bits 8-23 (mesh) dimensions in which R - C^ref must be inside the mesh;
                           // bits 24-29 the two shifts of the division by `units` (entry-major order)
    uint32_t ref;          // mesh: neighbour whose coordinates decide whether the move happens
    uint64_t last_offset;  // block launches: block size - unit width, the byte offset of the last unit
};

// Workgroup -> tile mapping.  The hardware hands consecutive workgroup ids to
// the 8 XCDs round-robin; each XCD has its own L2.  `run_log2` makes XCD x work
// on runs of 2^run_log2 consecutive tiles (tile = 256 consecutive units), the 8
// XCDs' runs interleaved, so that one L2 sees consecutive ranks while the 8 XCDs
// still sweep the same region of memory together.  kEighths instead gives XCD x
// the x-th contiguous eighth of all tiles: the host picks it for launches whose
// blocks sit at rank strides that are multiples of 4 KiB and cover only part of a
// 4 KiB page (see page_resonant), where it is 4 - 26 % faster, and for fused
// exchanges whose neighbouring ranks read the same lines (see allgather_order).
struct TileMap {
    uint32_t n_tiles;      // tiles that carry work
    uint32_t run_log2;     // kEighths: XCD x works on the x-th contiguous eighth of the tiles
    uint32_t per_xcd;      // kEighths: tiles per XCD, ceil(n_tiles / 8)
};
constexpr uint32_t kEighths = 31;
constexpr uint32_t kRankGroupLog2 = 6, kRankGroup = 1u << kRankGroupLog2;   // see ShiftArgs::grouped

__device__ __forceinline__ bool tile_of_block(const TileMap &tm, uint32_t &tile) {
    const uint32_t bid = blockIdx.x, x = bid & 7u, y = bid >> 3;
    if (tm.run_log2 == kEighths) tile = x * tm.per_xcd + y;
    else tile = ((y >> tm.run_log2) << (tm.run_log2 + 3)) + (x << tm.run_log2) + (y & ((1u << tm.run_log2) - 1u));
    return tile < tm.n_tiles;
}

// What a kernel is handed.  The runtime's cost of a launch on the host depends on the size of its arguments: 2.4 to
// 2.7 us up to 112 bytes, 3.0 to 3.4 at 128 to 256, 3.5 to 3.9 from 512 on (starts of small collectives are nothing
// but that, the shift kernel's 200 bytes of launch constants written out were a quarter of it).  So a division
// travels as its multiplier and a byte of shifts next to the divisor, what follows from other constants is worked
// out again in scalar registers, and arrays over the dimensions stay in the request's table.
constexpr size_t kCheapArguments = 112;

struct ShiftArgs {
    const DevEntry *entries;
    // Push form (k counts sources then): [k + 1] first entry of every source; entries in all (k_all).
    const uint32_t *groups;
    uint32_t total;        // units in this launch = p * k * chunks
    uint32_t k;            // entries in this launch
    uint32_t inner;        // rank stride of the shifted dimension
    uint32_t pj;           // its size
    uint32_t chunks, p;    // units of a block; ranks
    uint32_t mul_chunks, mul_k, mul_inner, mul_pj, mul_p, mul_group_k;
    // What every wavefront needs stays a word of its own as far as there is room (all of it packed: 0.4 % of a
    // 32^3, 256 B all-to-all).
    uint32_t sh_chunks, sh_k, sh_inner, sh_pj;    // shift_byte of these divisions
    TileMap map;
    uint32_t more;         // shifts of p, group * k; launch_flags
    // Large blocks on rank-major buffers: the ranks are taken in groups of kRankGroup, and inside a group the
    // order is (entry, rank, chunk), so that a plane of the workspace sees that many consecutive blocks at a
    // time instead of one.  `grouped` = the blocks of all whole groups, (p / kRankGroup) * kRankGroup * k;
    // the ranks after them keep the plain order.
    uint32_t grouped, k_all;
};
static_assert(sizeof(ShiftArgs) <= kCheapArguments, "launch cost");

// The upper 16 bits of a word whose lower ones hold the shifts of two divisions.
//   bits 16-20 TileMap::run_log2; 21 entry-major order (entry, rank, chunk) instead of (rank, entry, chunk);
//   22-25 by how many bytes a block's last unit is pulled back (TAIL); 26 block kernel: full offset vectors
inline uint32_t launch_flags(uint32_t run_log2, bool entry_major, uint32_t pull, bool vector_round = false) {
    return (run_log2 << 16) | ((uint32_t)entry_major << 21) | (pull << 22) | ((uint32_t)vector_round << 26);
}
__device__ __forceinline__ uint32_t is_entry_major(uint32_t more) { return (more >> 21) & 1u; }
__device__ __forceinline__ uint32_t is_vector_round(uint32_t more) { return (more >> 26) & 1u; }
// block size - unit width
template <typename V>
__device__ __forceinline__ uint64_t last_offset_of(uint32_t chunks, uint32_t more) {
    return (uint64_t)(chunks - 1u) * sizeof(V) - ((more >> 22) & 15u);
}
__device__ __forceinline__ TileMap map_of(uint32_t n_tiles, uint32_t more) {
    return TileMap{n_tiles, (more >> 16) & 31u, (n_tiles + 7u) >> 3};
}
__device__ __forceinline__ uint32_t tiles_of(uint32_t total) { return (total + (uint32_t)kThreads - 1u) / (uint32_t)kThreads; }

// The dimensions of the torus in the request's table, in front of the residues [s][d] of its offsets (kernels that
// decode every coordinate with run-time indices, and meshes).  Read through the scalar cache.
struct TorusDims {
    FastDiv d_dims[ISO_MAX_DIMS];
    uint32_t inner[ISO_MAX_DIMS];
};
typedef const TorusDims __attribute__((address_space(4))) *dims_ptr;
__device__ __forceinline__ dims_ptr const_dims(const TorusDims *d) { return (dims_ptr)(uintptr_t)d; }
__device__ __forceinline__ const uint32_t *offsets_after(const TorusDims *d) { return (const uint32_t *)(d + 1); }
__device__ __forceinline__ FastDiv dim_of(dims_ptr d, int j) {
    return FastDiv{d->d_dims[j].mul, d->d_dims[j].sh1, d->d_dims[j].sh2, d->d_dims[j].div};
}

// Entries of a launch that moves equal blocks by full offset vectors (the s-exchange) on a torus of at most
// kVectorDims dimensions: all that a lane needs of its entry in 48 bytes, so that no second table is read.
// `c` are the residues of the last kVectorDims dimensions, the last one first (signed where a mesh does not wrap); absent
// dimensions hold 0.
constexpr int kVectorDims = 5;
struct alignas(16) VectorEntry {
    uint64_t src, dst;     // addresses of rank 0's blocks
    uint32_t back;         // sum of c_j * inner_j: ranks back where no dimension wraps
    uint32_t c[kVectorDims];
    uint64_t way;          // kStops: address of rank 0's block on the way (a block of one hop has none); kStrides: of `dst`
};
// WAY of the vector kernels.  For launches that take blocks through all their hops (Binder::all_hops_in_one_launch):
// kStops, all-to-all: a block is stored at every rank on its way as well (move_through_stops).  kStrides, allgather: every
// node of the trie is an entry, in the receive buffer or in the workspace, with the stride of its own destination.
// kMesh beside these: dimensions that do not wrap (passes_end).
constexpr int kStops = 1, kStrides = 2, kMesh = 4;
static_assert(sizeof(VectorEntry) == sizeof(DevEntry), "staged by the same code");

struct VectorArgs {
    const DevEntry *entries;   // VectorEntry records instead for the kernels of at most kVectorDims dimensions
    const TorusDims *dims;     // the others: dimensions and residues
    uint32_t total, k;
    int32_t d;
    uint32_t per;                             // push kernel: entries a lane writes to; mesh: which of `last` wrap, a bit each
    uint32_t src_stride, dst_stride;          // the same for all entries (VectorEntry launches)
    uint32_t chunks, p;
    uint32_t mul_chunks, mul_k, mul_p;
    uint32_t shifts;                          // chunks, k, p; the last dimension
    uint32_t more;                            // the second and third last dimension; launch_flags
    uint32_t last[kVectorDims];               // VectorEntry launches: the dimensions from the last to the first
    uint32_t mul_last[kVectorDims - 1], shift_last3;
};
static_assert(sizeof(VectorArgs) <= kCheapArguments, "launch cost");

typedef uint32_t vec16_t __attribute__((ext_vector_type(4)));
typedef uint32_t vec8_t __attribute__((ext_vector_type(2)));

// A block of `size` bytes is moved in units of w bytes, w the largest power of two that is at
// most 16 and at most `size`: ceil(size / w) units, unit c at byte offset min(c * w, size - w).
// When w does not divide the size the last unit overlaps the one before it; both carry the same
// bytes of the same block, so the doubly written bytes get the same value twice.  Addresses
// need no alignment: the unit types are declared with alignment 1 and global memory accesses of
// any width take any address on this target.
template <typename V>
struct Unaligned {
    typedef V type __attribute__((aligned(1)));
};

// Cache policy of the accesses of a launch (see cache_policy in iso_bind.hpp for when each is taken).
constexpr int kStreamLoads = 1, kPlainStores = 2;
// Block kernel: every block by its own size.  Blocks of up to kSmallUnits units share sectors and lines with others of
// their row: cached loads, plain stores that meet in the L2.  The larger ones stream both.
constexpr int kBySize = 4;
constexpr uint32_t kSmallUnits = 8;

// The unit at byte offset `off` of the block at byte address `src` to the same offset of the
// block at `dst`, both in global memory (the address space is spelled out so that the accesses
// are global_load / global_store, not flat ones).
template <typename V, int POLICY>
__device__ __forceinline__ void move_unit(uint64_t dst, uint64_t src, uint64_t off) {
    typedef typename Unaligned<V>::type UV;
    typedef const UV __attribute__((address_space(1))) *src_ptr;
    typedef UV __attribute__((address_space(1))) *dst_ptr;
    const src_ptr sp = (src_ptr)(src + off);
    V v;
    if constexpr (POLICY & kStreamLoads) v = __builtin_nontemporal_load(sp);
    else v = *sp;
    // Streaming stores at most for 16-byte units.  Narrower units belong to blocks of a few bytes, of
    // which several wavefronts write different bytes of one cache line: plain stores let the L2
    // merge them before the line goes to memory.
    if constexpr (sizeof(V) == 16 && !(POLICY & kPlainStores)) __builtin_nontemporal_store(v, (dst_ptr)(dst + off));
    else *(dst_ptr)(dst + off) = v;
}

template <typename V>
__device__ __forceinline__ uint64_t unit_offset(uint32_t ch, uint64_t last_offset) {
    const uint64_t off = (uint64_t)ch * sizeof(V);
    return off < last_offset ? off : last_offset;
}

// TAIL: the width does not divide the block size.  The regular kernels are instantiated
// without it as well: the comparison and selects cost 2 % on the round kernel.
template <typename V, bool TAIL>
__device__ __forceinline__ uint64_t unit_offset_if(uint32_t ch, uint64_t last_offset) {
    if constexpr (TAIL) return unit_offset<V>(ch, last_offset);
    else return (uint64_t)ch * sizeof(V);
}

// Address of rank R's block: base + R * stride with the stride known to fit 32 bits.
__device__ __forceinline__ uint64_t block_address(uint64_t base, uint32_t R, uint32_t stride) {
    return base + (uint64_t)R * stride;
}

// Entry table of the launch: from LDS (staged once per workgroup) when it fits,
// else straight from global memory (cached).
template <bool LDS>
struct EntryTable {
    const DevEntry *tab;
    __device__ __forceinline__ EntryTable(const DevEntry *global, uint32_t k, DevEntry *lds) {
        if constexpr (LDS) {
            if (threadIdx.x < k) lds[threadIdx.x] = global[threadIdx.x];
            __syncthreads();
            tab = lds;
        } else {
            tab = global;
        }
    }
    __device__ __forceinline__ DevEntry operator[](uint32_t e) const { return tab[e]; }
};

// The same staging in two steps, so that a kernel can put work that does not depend on the table
// between the table's load and its arrival in LDS: issue() starts the load of this lane's entry,
// commit() writes it to LDS and synchronises the workgroup.  (Three plain 16-byte registers: a
// DevEntry variable here ends up in LDS itself.)
template <bool LDS>
struct StagedEntries {
    static_assert(sizeof(DevEntry) == 48, "staged as three 16-byte words");
    vec16_t w0, w1, w2;
    bool mine;
    __device__ __forceinline__ void issue(const DevEntry *global, uint32_t k) {
        w0 = w1 = w2 = vec16_t{};
        mine = LDS && threadIdx.x < k;
        if (mine) {
            const vec16_t *from = (const vec16_t *)(global + threadIdx.x);
            w0 = from[0];
            w1 = from[1];
            w2 = from[2];
        }
    }
    __device__ __forceinline__ void commit(DevEntry *lds) const {
        if constexpr (LDS) {
            if (mine) {
                vec16_t *to = (vec16_t *)(lds + threadIdx.x);
                to[0] = w0;
                to[1] = w1;
                to[2] = w2;
            }
            __syncthreads();
        }
    }
};

// Coordinate decodes over all dimensions.  For d <= kUnrolledDims the code is instantiated
// for the exact d (one uniform switch, then straight-line code): the per-dimension launch
// constants are then read at fixed kernel-argument offsets (scalar registers) and the loads
// of the offset vector are issued together.  Indexing those arrays with a run-time j costs a
// dependent scalar load and several uniform branches per dimension, and at one unit per lane
// that is a third of the kernel's throughput.
// Rank arithmetic is done modulo 2^32: ranks are below 2^31 and every true result lies in
// [0, p), so wrapped intermediate values are harmless.
constexpr int kUnrolledDims = 6;

// Source rank of R for a move by the full offset vector c[0..d): R (-) c on the torus.
template <int D>
__device__ __forceinline__ uint32_t vector_source_rank_d(uint32_t R, const uint32_t *__restrict__ c, dims_ptr dims) {
    uint32_t cj[D];
#pragma unroll
    for (int j = 0; j < D; ++j) cj[j] = c[j];
    uint32_t srcR = R, rem = R;
#pragma unroll
    for (int j = D - 1; j >= 0; --j) {
        uint32_t q, rj;
        const FastDiv dj = dim_of(dims, j);
        fast_divmod(rem, dj, q, rj);
        rem = q;
        srcR -= cj[j] * dims->inner[j];                                   // cj steps back ...
        if (rj < cj[j]) srcR += dj.div * dims->inner[j];           // ... around the ring
    }
    return srcR;
}

__device__ __forceinline__ uint32_t vector_source_rank(uint32_t R, const uint32_t *__restrict__ c, int32_t d, dims_ptr dims) {
    switch (d) {
        case 1: return vector_source_rank_d<1>(R, c, dims);
        case 2: return vector_source_rank_d<2>(R, c, dims);
        case 3: return vector_source_rank_d<3>(R, c, dims);
        case 4: return vector_source_rank_d<4>(R, c, dims);
        case 5: return vector_source_rank_d<5>(R, c, dims);
        case 6: return vector_source_rank_d<6>(R, c, dims);
        default: break;
    }
    uint32_t srcR = R, rem = R;
    for (int j = d - 1; j >= 0; --j) {
        uint32_t q, rj;
        const FastDiv dj = dim_of(dims, j);
        fast_divmod(rem, dj, q, rj);
        rem = q;
        srcR -= c[j] * dims->inner[j];
        if (rj < c[j]) srcR += dj.div * dims->inner[j];
    }
    return srcR;
}

// Makes the compiler fetch these launch constants here, in one batch of scalar loads, instead of
// each in front of its first use behind some branch (every such fetch is a wait of its own).
__device__ __forceinline__ void fetch_now(const ShiftArgs &a) {
    asm volatile("" ::"s"(a.entries), "s"(a.total), "s"(a.k), "s"(a.inner), "s"(a.pj), "s"(a.chunks), "s"(a.p),
                 "s"(a.mul_chunks), "s"(a.mul_k), "s"(a.mul_inner), "s"(a.mul_pj), "s"(a.mul_p), "s"(a.sh_chunks), "s"(a.sh_k),
                 "s"(a.sh_inner), "s"(a.sh_pj), "s"(a.map.n_tiles), "s"(a.map.run_log2), "s"(a.map.per_xcd), "s"(a.more));
}

// The divisions of a shift launch.
struct ShiftDivs {
    FastDiv chunks, k, inner, pj, p, group_k;
    __device__ __forceinline__ explicit ShiftDivs(const ShiftArgs &a)
        : chunks(fastdiv_of(a.mul_chunks, a.chunks, a.sh_chunks, 0)), k(fastdiv_of(a.mul_k, a.k, a.sh_k, 0)),
          inner(fastdiv_of(a.mul_inner, a.inner, a.sh_inner, 0)), pj(fastdiv_of(a.mul_pj, a.pj, a.sh_pj, 0)),
          p(fastdiv_of(a.mul_p, a.p, a.more, 0)), group_k(fastdiv_of(a.mul_group_k, a.k << kRankGroupLog2, a.more, 1)) {}
};

template <typename V, bool LDS, int POLICY, bool TAIL, bool GROUPS = false>
__global__ __launch_bounds__(kThreads) void shift_round_kernel(const ShiftArgs a) {
    fetch_now(a);
    if constexpr (GROUPS) asm volatile("" ::"s"(a.grouped), "s"(a.mul_group_k));
    const ShiftDivs div(a);
    __shared__ DevEntry lds[LDS ? kLdsEntries : 1];
    uint32_t tile;
    if (!tile_of_block(a.map, tile)) return;            // (the whole workgroup: no one is left at the barrier)
    // The table goes through LDS; its load is under way while the lanes work out their indices, which do
    // not depend on it.
    StagedEntries<LDS> staging;
    staging.issue(a.entries, a.k);
    const uint32_t u = tile * (uint32_t)kThreads + threadIdx.x;
    uint32_t t, ch, R, e;
    fast_divmod(u, div.chunks, t, ch);
    if constexpr (GROUPS) {                             // an instantiation of its own: the few scalar loads and
        if (t < a.grouped) {                            // the branch cost the plain one 2 - 3 % on small blocks
            uint32_t g, in_group;
            fast_divmod(t, div.group_k, g, in_group);
            e = in_group >> kRankGroupLog2;
            R = (g << kRankGroupLog2) + (in_group & (kRankGroup - 1u));
        } else {
            fast_divmod(t - a.grouped, div.k, R, e);
            R += fast_div(a.grouped, div.k);            // the ranks of the whole groups come first
        }
    } else if (is_entry_major(a.more)) {
        fast_divmod(t, div.p, e, R);
    } else {
        fast_divmod(t, div.k, R, e);
    }
    const uint32_t q = fast_div(R, div.inner);
    const uint32_t rj = q - fast_div(q, div.pj) * a.pj;       // coordinate of R in the shifted dimension
    staging.commit(lds);
    if (u >= a.total) return;                                  // (indices beyond the launch are never used)
    const DevEntry en = LDS ? lds[e] : a.entries[e];
    // v steps back along the dimension, around the ring where that passes coordinate 0 (modulo 2^32;
    // the true result lies in [0, p))
    uint32_t srcR = R - en.shift * a.inner;
    if (rj < en.shift) srcR += a.pj * a.inner;
    move_unit<V, POLICY>(block_address(en.dst, R, en.dst_stride), block_address(en.src, srcR, en.src_stride),
                      unit_offset_if<V, TAIL>(ch, last_offset_of<V>(a.chunks, a.more)));
}

// The same round for blocks that are a multiple of 1 KiB (64 units of 16 bytes): the 64 units of a
// wavefront then belong to one block, so rank, entry and source rank are the same for all its lanes
// and are computed once, in scalar registers, the entry fetched with scalar loads.  No staging of the
// table through LDS, no barrier, no vector-memory access in front of the one load that matters: what
// bounds these kernels is how long a wavefront holds its slot before that load is under way.
template <int POLICY, bool GROUPS = false>
__global__ __launch_bounds__(kThreads) void shift_round_uniform_kernel(const ShiftArgs a) {
    fetch_now(a);
    const ShiftDivs div(a);
    uint32_t tile;
    if (!tile_of_block(a.map, tile)) return;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t u0 = tile * (uint32_t)kThreads + wave * 64u;      // first unit of this wavefront
    if (u0 >= a.total) return;                                       // total is a multiple of 64
    uint32_t t, ch0, R, e;
    fast_divmod(u0, div.chunks, t, ch0);
    if constexpr (GROUPS) {
        if (t < a.grouped) {
            uint32_t g, in_group;
            fast_divmod(t, div.group_k, g, in_group);
            e = in_group >> kRankGroupLog2;
            R = (g << kRankGroupLog2) + (in_group & (kRankGroup - 1u));
        } else {
            fast_divmod(t - a.grouped, div.k, R, e);
            R += fast_div(a.grouped, div.k);
        }
    } else if (is_entry_major(a.more)) {
        fast_divmod(t, div.p, e, R);
    } else {
        fast_divmod(t, div.k, R, e);
    }
    const uint32_t q = fast_div(R, div.inner);
    const uint32_t rj = q - fast_div(q, div.pj) * a.pj;
    // the table is never written while a collective runs: read it as constant memory, through the scalar cache
    typedef const DevEntry __attribute__((address_space(4))) *const_entry_ptr;
    const const_entry_ptr en = (const_entry_ptr)(uintptr_t)(a.entries + e);
    const uint32_t shift = en->shift;
    uint32_t srcR = R - shift * a.inner;
    if (rj < shift) srcR += a.pj * a.inner;
    const uint64_t src = block_address(en->src, srcR, en->src_stride);
    const uint64_t dst = block_address(en->dst, R, en->dst_stride);
    move_unit<vec16_t, POLICY>(dst, src, (uint64_t)(ch0 + (threadIdx.x & 63u)) * sizeof(vec16_t));
}

// Allgather rounds the other way round: the trie sends one copy on to several children, and the kernel above
// reads it once for each.  Here the entries of a launch are ordered by source, and a lane reads one unit of
// rank S's copy and writes it to every child, which sits `shift` steps on.
template <typename V, bool TAIL>
__global__ __launch_bounds__(kThreads) void shift_push_kernel(const ShiftArgs a) {
    fetch_now(a);
    asm volatile("" ::"s"(a.groups), "s"(a.k_all));
    const ShiftDivs div(a);
    __shared__ DevEntry lds[kLdsEntries];
    __shared__ uint32_t lds_first[kLdsEntries + 1];
    uint32_t tile;
    if (!tile_of_block(a.map, tile)) return;
    StagedEntries<true> staging;
    staging.issue(a.entries, a.k_all);
    const uint32_t q = kThreads - 1 - threadIdx.x;       // the workgroup's last lanes, as in the block kernel
    const bool stages = q <= a.k;
    const uint32_t first = stages ? a.groups[q] : 0u;
    const uint32_t u = tile * (uint32_t)kThreads + threadIdx.x;
    uint32_t t, ch, S, g;
    fast_divmod(u, div.chunks, t, ch);
    if (is_entry_major(a.more)) fast_divmod(t, div.p, g, S);
    else fast_divmod(t, div.k, S, g);
    const uint32_t qq = fast_div(S, div.inner);
    const uint32_t sj = qq - fast_div(qq, div.pj) * a.pj;
    const uint64_t off = unit_offset_if<V, TAIL>(ch, last_offset_of<V>(a.chunks, a.more));
    if (stages) lds_first[q] = first;
    staging.commit(lds);
    if (u >= a.total) return;
    typedef typename Unaligned<V>::type UV;
    typedef const UV __attribute__((address_space(1))) *src_ptr;
    typedef UV __attribute__((address_space(1))) *dst_ptr;
    uint32_t e = lds_first[g];
    const uint32_t e1 = lds_first[g + 1];
    const src_ptr sp = (src_ptr)(block_address(lds[e].src, S, lds[e].src_stride) + off);
    const V v = *sp;                                     // (streaming: 2 to 12 % slower)
    for (; e < e1; ++e) {
        const DevEntry &en = lds[e];
        uint32_t R = S + en.shift * a.inner;             // modulo 2^32; the true result lies in [0, p)
        if (sj + en.shift >= a.pj) R -= a.pj * a.inner;
        const dst_ptr dp = (dst_ptr)(block_address(en.dst, R, en.dst_stride) + off);
        if constexpr (sizeof(V) == 16) __builtin_nontemporal_store(v, dp);
        else *dp = v;
    }
}

// The s-exchange of equal blocks: every entry moves by a full offset vector.  D: dimensions the rank is
// decoded into (3 or kVectorDims, absent ones of size 1 in front); D = 0: any torus, from the general tables.
template <int D>
__device__ __forceinline__ void fetch_now(const VectorArgs &a) {
    asm volatile("" ::"s"(a.entries), "s"(a.total), "s"(a.k), "s"(a.chunks), "s"(a.p), "s"(a.mul_chunks), "s"(a.mul_k),
                 "s"(a.mul_p), "s"(a.shifts), "s"(a.more));
    if constexpr (D == 0) {
        asm volatile("" ::"s"(a.dims), "s"(a.d));
    } else {
        asm volatile("" ::"s"(a.src_stride), "s"(a.dst_stride));
#pragma unroll
        for (int j = 0; j + 1 < D; ++j) asm volatile("" ::"s"(a.last[j]), "s"(a.mul_last[j]));
        if constexpr (D > 4) asm volatile("" ::"s"(a.shift_last3));
    }
}

struct VectorDivs {
    FastDiv chunks, k, p;
    __device__ __forceinline__ explicit VectorDivs(const VectorArgs &a)
        : chunks(fastdiv_of(a.mul_chunks, a.chunks, a.shifts, 0)), k(fastdiv_of(a.mul_k, a.k, a.shifts, 1)),
          p(fastdiv_of(a.mul_p, a.p, a.shifts, 2)) {}
};

// Coordinates of R, last dimension first, and the ranks once around each dimension.
template <int D>
__device__ __forceinline__ void last_coordinates(uint32_t R, const VectorArgs &a, uint32_t (&r)[D], uint32_t (&wrap)[D]) {
    uint32_t rem = R, once = 1;
#pragma unroll
    for (int j = 0; j + 1 < D; ++j) {
        uint32_t q;
        fast_divmod(rem, fastdiv_of(a.mul_last[j], a.last[j], j == 0 ? a.shifts : j < 3 ? a.more : a.shift_last3, j == 0 ? 3 : j < 3 ? j - 1 : 0),
                    q, r[j]);
        rem = q;
        once *= a.last[j];
        wrap[j] = once;
    }
    r[D - 1] = rem;
    wrap[D - 1] = a.p;
}

// Is the rank `c` steps back along dimension j (counted from the last one) on the far side of the ring?  On a mesh
// coordinates of dimensions that do not wrap are signed, and one comparison tests both ends.  Boxes by these kernels against
// the block kernel's decode from the general tables, straightforward exchange, us: 45 x 37 x 29, 26 neighbours, 100 B 66 ->
// 50, 1 KiB 571 -> 382, allgather 512 B 169 -> 100; 8^5, 40 neighbours, 512 B 231 -> 165; 300^2, 12, 40 B 26.1 -> 21.3.
template <bool MESH>
__device__ __forceinline__ bool passes_end(uint32_t r, uint32_t c, int j, const VectorArgs &a, bool &outside) {
    if constexpr (!MESH) return r < c;
    const bool past = r - c >= a.last[j], wraps = (a.per >> j) & 1u;
    outside = outside || (past && !wraps);
    return past && wraps;
}

// One unit of a block of an all-to-all through all the hops of its schedule, pulled by the rank R that receives it: the
// ranks on its way are R moved back along the dimensions one by one, the last hop first.  It is stored at every one of them,
// in the block's place in the workspace.  What the next hop takes is still in the register: no one reads the stops, and the
// stores of different lanes to one place (of a block of three hops and more) need no order: unit by unit the last one stays.
// A launch per dimension reads every hop's block again and is bound by the memory's copy rate; here the hops of a block are
// one read and their writes.  The stops are stored plainly, the receive rows stream: stops of one block are overwritten, by
// its next hops at other ranks, while the caches hold them (streamed -> plain, us, many sets of buffers: 8^5, 40 neighbours,
// 4 KiB 5430 -> 4100; 64^3, 26 neighbours, 1000 B 4670 -> 3740; 32^3, 26, 256 B 111.7 -> 107.6, though 94 -> 106 with one set,
// a launch per dimension 158).
template <typename V, int D, int POLICY, int WAY, typename ENTRY>
__device__ __forceinline__ void move_through_stops(const ENTRY &en, uint32_t R, const uint32_t (&r)[D],
                                                   const uint32_t (&wrap)[D], const VectorArgs &a, uint64_t off) {
    typedef typename Unaligned<V>::type UV;
    typedef const UV __attribute__((address_space(1))) *src_ptr;
    typedef UV __attribute__((address_space(1))) *dst_ptr;
    uint32_t at[D], from = R, inner = 1;
    bool outside = false;
#pragma unroll
    for (int j = 0; j < D; ++j) {                        // modulo 2^32, see vector_source_rank
        from -= en.c[j] * inner;
        if (passes_end<(WAY & kMesh) != 0>(r[j], en.c[j], j, a, outside)) from += wrap[j];
        at[j] = from;
        inner = wrap[j];
    }
    if (outside) return;                                 // no source: no block comes this way
    const src_ptr sp = (src_ptr)(block_address(en.src, from, a.src_stride) + off);
    V v;
    if constexpr (POLICY & kStreamLoads) v = __builtin_nontemporal_load(sp);
    else v = *sp;
    const uint32_t m = (uint32_t)last_offset_of<V>(a.chunks, a.more) + (uint32_t)sizeof(V);
#pragma unroll
    for (int j = D - 1; j >= 0; --j)                     // in the order of the hops
        if (en.c[j] && at[j] != from) *(dst_ptr)(block_address(en.way, at[j], m) + off) = v;
    __builtin_nontemporal_store(v, (dst_ptr)(block_address(en.dst, R, a.dst_stride) + off));
}

// What bounds this kernel is the time a wavefront holds its slot before its one load is under way.  Two things
// keep that short: one table, in LDS, holds all that an entry needs (a second one with the residues, read from
// global memory after the barrier, was a dependent load in front of the block's own), and the rank's
// coordinates are worked out while the table's load is in flight.  Fused s-exchange, before and after: 64^3,
// 26 neighbours, 128-byte blocks 342 -> 294 us all-to-all, 188 -> 166 us allgather (fill rate: 128 us);
// 200-byte allgather on 60 x 50 x 41 142 -> 130 us; 7-byte blocks on 50^3 26 -> 22 us.
template <typename V, int D, bool LDS, int POLICY, bool TAIL, int WAY = 0>
__global__ __launch_bounds__(kThreads) void vector_round_kernel(const VectorArgs a) {
    fetch_now<D>(a);
    const VectorDivs div(a);
    __shared__ DevEntry lds[LDS ? kLdsEntries : 1];
    uint32_t tile;
    if (!tile_of_block(map_of(tiles_of(a.total), a.more), tile)) return;
    StagedEntries<LDS> staging;
    staging.issue(a.entries, a.k);
    const uint32_t u = tile * (uint32_t)kThreads + threadIdx.x;
    uint32_t t, ch, R, e;
    fast_divmod(u, div.chunks, t, ch);
    if (is_entry_major(a.more)) fast_divmod(t, div.p, e, R);
    else fast_divmod(t, div.k, R, e);
    const uint64_t off = unit_offset_if<V, TAIL>(ch, last_offset_of<V>(a.chunks, a.more));
    if constexpr (D == 0) {
        staging.commit(lds);
        if (u >= a.total) return;
        const DevEntry en = LDS ? lds[e] : a.entries[e];
        const uint32_t srcR = vector_source_rank(R, offsets_after(a.dims) + (size_t)en.shift * a.d, a.d, const_dims(a.dims));
        move_unit<V, POLICY>(block_address(en.dst, R, en.dst_stride), block_address(en.src, srcR, en.src_stride), off);
    } else {
        uint32_t r[D], wrap[D];
        last_coordinates<D>(R, a, r, wrap);
        staging.commit(lds);
        if (u >= a.total) return;
        const VectorEntry &en = ((const VectorEntry *)(LDS ? lds : a.entries))[e];
        if constexpr (WAY & kStops) {
            move_through_stops<V, D, POLICY, WAY>(en, R, r, wrap, a, off);
            return;
        }
        uint32_t srcR = R - en.back;                    // modulo 2^32, see vector_source_rank
        bool outside = false;
#pragma unroll
        for (int j = 0; j < D; ++j)
            if (passes_end<(WAY & kMesh) != 0>(r[j], en.c[j], j, a, outside)) srcR += wrap[j];
        if (outside) return;                            // mesh, no source: the destination keeps its content
        const uint32_t dst_stride = WAY & kStrides ? (uint32_t)en.way : a.dst_stride;
        move_unit<V, POLICY>(block_address(en.dst, R, dst_stride), block_address(en.src, srcR, a.src_stride), off);
    }
}

// The same for blocks that are a multiple of 1 KiB: one block per wavefront, so that rank, entry and source
// rank are worked out once, in scalar registers (see shift_round_uniform_kernel).  Fused all-to-all, before and
// after: 256^2, 12 neighbours, 1 KiB 298 -> 259 us, 8^5, 40 neighbours, 4 KiB 2070 -> 1800 us.
template <int D, int POLICY, int WAY = 0>
__global__ __launch_bounds__(kThreads) void vector_round_uniform_kernel(const VectorArgs a) {
    fetch_now<D>(a);
    const VectorDivs div(a);
    uint32_t tile;
    if (!tile_of_block(map_of(tiles_of(a.total), a.more), tile)) return;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t u0 = tile * (uint32_t)kThreads + wave * 64u;      // first unit of this wavefront
    if (u0 >= a.total) return;                                       // total is a multiple of 64
    uint32_t t, ch0, R, e;
    fast_divmod(u0, div.chunks, t, ch0);
    if (is_entry_major(a.more)) fast_divmod(t, div.p, e, R);
    else fast_divmod(t, div.k, R, e);
    typedef const VectorEntry __attribute__((address_space(4))) *const_entry_ptr;
    const const_entry_ptr en = (const_entry_ptr)(uintptr_t)((const VectorEntry *)a.entries + e);
    uint32_t r[D], wrap[D];
    last_coordinates<D>(R, a, r, wrap);
    const uint64_t off = (uint64_t)(ch0 + (threadIdx.x & 63u)) * sizeof(vec16_t);
    if constexpr (WAY & kStops) {
        move_through_stops<vec16_t, D, POLICY, WAY>(*en, R, r, wrap, a, off);
        return;
    }
    uint32_t srcR = R - en->back;
    bool outside = false;
#pragma unroll
    for (int j = 0; j < D; ++j)
        if (passes_end<(WAY & kMesh) != 0>(r[j], en->c[j], j, a, outside)) srcR += wrap[j];
    if (outside) return;
    const uint32_t dst_stride = WAY & kStrides ? (uint32_t)en->way : a.dst_stride;
    move_unit<vec16_t, POLICY>(block_address(en->dst, R, dst_stride), block_address(en->src, srcR, a.src_stride), off);
}

// The allgather's s-exchange the other way round: a lane reads one unit of rank S's block and writes it into
// the receive blocks of `per` neighbours (R = S (+) C^e), so the send buffer is read k / per times instead of
// k times.  Taken where the pull form's reads miss the L2 (see vector_launch): they then cross the fabric
// beside the writes, and both together were what bounded it.
template <typename V, int D, bool TAIL, int WAY = 0>
__global__ __launch_bounds__(kThreads) void push_round_kernel(const VectorArgs a) {
    fetch_now<D>(a);
    const VectorDivs div(a);
    asm volatile("" ::"s"(a.per));
    __shared__ DevEntry lds[kLdsEntries];
    uint32_t tile;
    if (!tile_of_block(map_of(tiles_of(a.total), a.more), tile)) return;
    StagedEntries<true> staging;
    staging.issue(a.entries, a.k);
    const uint32_t u = tile * (uint32_t)kThreads + threadIdx.x;
    uint32_t t, ch, S, g;
    fast_divmod(u, div.chunks, t, ch);
    fast_divmod(t, div.p, g, S);                         // (entry group, rank, chunk)
    const uint64_t off = unit_offset_if<V, TAIL>(ch, last_offset_of<V>(a.chunks, a.more));
    uint32_t r[D], wrap[D];
    last_coordinates<D>(S, a, r, wrap);
    staging.commit(lds);
    if (u >= a.total) return;
    typedef typename Unaligned<V>::type UV;
    typedef const UV __attribute__((address_space(1))) *src_ptr;
    typedef UV __attribute__((address_space(1))) *dst_ptr;
    const VectorEntry *entries = (const VectorEntry *)lds;
    const V v = *(src_ptr)(block_address(entries[0].src, S, a.src_stride) + off);
    const uint32_t e1 = a.k - g * a.per < a.per ? a.k : (g + 1) * a.per;
#pragma unroll 2
    for (uint32_t e = g * a.per; e < e1; ++e) {
        const VectorEntry &en = entries[e];
        uint32_t R = S + en.back;                        // modulo 2^32, see vector_source_rank
#pragma unroll
        for (int j = 0; j < D; ++j)
            if (r[j] + en.c[j] >= a.last[j]) R -= wrap[j];
        const uint32_t dst_stride = WAY & kStrides ? (uint32_t)en.way : a.dst_stride;
        const dst_ptr dp = (dst_ptr)(block_address(en.dst, R, dst_stride) + off);
        if constexpr (sizeof(V) == 16) __builtin_nontemporal_store(v, dp);
        else *dp = v;
    }
}

// Irregular blocks (the v/w interfaces of Section 2): every entry has its own
// block size and its own unit width (16 bytes for blocks of at least 16 bytes,
// narrower below, e.g. a 1-byte corner block next to a 16 KiB face block).
// A rank's units are the concatenation of its entries' units; `prefix[e]` is
// the first unit of entry e.  The flat index is split into (rank, unit in row),
// the entry is found by binary search in the prefix array.  On slot-major
// buffers (one plane of p blocks per neighbour) the order is (entry, rank, unit)
// instead: prefix[e] then counts the units of all ranks in the entries before e,
// and the position inside the plane is divided by the entry's own unit count.
// (Measured against this form and dropped: the launch cut into one segment per unit
// width, each a whole number of tiles, so that the width switch is uniform in a
// workgroup.  Selecting the segment's constants puts one more stage of dependent
// scalar loads in front of every wavefront's load: stencil-shaped all-to-all,
// 4096 / 64 / 1 byte blocks, -2 % on rank-major buffers, -15 % on slot-major ones,
// -11 % for the fused s-exchange.  What tiny blocks cost is not in the kernel: a
// block of a few bytes in every rank's row is a memory access of its own on each
// side, whatever moves it.)
//
// MESH (Section 7, non-periodic dimensions): coordinates of non-periodic
// dimensions are signed and nothing wraps there.  A move happens at rank R only
// if R - C^ref stays inside the mesh in every dimension of the entry's mask
// (the non-periodic dimensions routed up to and including this round in which
// C^ref is non-zero); otherwise the destination keeps its content.
struct BlockArgs {
    const DevEntry *entries;
    const uint32_t *prefix;    // [k + 1] first unit of every entry, then [k] multipliers (entry-major order)
    const TorusDims *dims;     // and after it the [s][d] effective coordinates (residues; signed where non-periodic)
    uint32_t total;            // p * row_units
    uint32_t k;
    uint32_t inner, pj;        // shift rounds
    uint32_t equal_units;      // != 0: every entry of the launch has this many units (no search)
    uint32_t grouped;          // GROUPS: units of the ranks that form whole groups (the first ones)
    uint32_t row, plane;       // units of a row; p * equal_units (GROUPS: group * equal_units)
    uint32_t mul_row, mul_inner, mul_pj, mul_units, mul_plane, mul_group_row;
    uint32_t shifts;           // row, inner, pj, units
    uint32_t more;             // plane, units of a group's rows; launch_flags.  Entry-major (slot-major buffers): units
                               // ordered (entry, rank, unit) and prefix[e] counts the units of all ranks before
                               // entry e; else (rank, entry, unit)
    uint32_t torus;            // torus_bits
    uint64_t work;             // HOPS: the workspace; DevEntry::ref counts the 16 bytes in front of the block's place there
};
static_assert(sizeof(BlockArgs) <= kCheapArguments, "launch cost");

// Dimensions (bits 0-4), the shifted one plus 1 (5-9; 0: same-rank copy or full vectors), whether the entries hold
// their reference coordinates (10, see pack_reference), an interior bit per tile instead of per wavefront (11), which dimensions wrap (16-31).
inline uint32_t torus_bits(int32_t d, int32_t shift_dim, uint32_t periodic_mask, bool packed_reference = false) {
    return (uint32_t)d | ((uint32_t)(shift_dim + 1) << 5) | ((uint32_t)packed_reference << 10) | (periodic_mask << 16);
}

// Mesh shift rounds read no `units`, `ref` and `last_offset` of an entry: 16 bits for the coordinate of C^ref in each
// of up to 6 dimensions that do not wrap.  Saves the lanes near a face a dependent load (see mesh_shift_round_kernel).
inline bool pack_reference(const int32_t *cref, int32_t d, uint32_t mask, DevEntry &de) {
    uint32_t w[3] = {};
    if (d > 6) return false;
    for (int j = 0; j < d; ++j) {
        if (!((mask >> j) & 1u)) continue;
        if (cref[j] < -32768 || cref[j] > 32767) return false;
        w[j / 2] |= (uint32_t)(uint16_t)cref[j] << (16 * (j & 1));
    }
    de.units = w[0];
    de.ref = w[1];
    de.last_offset = w[2];
    return true;
}
__device__ __forceinline__ uint32_t packed_reference(const DevEntry &en, int j) {
    const uint32_t w = j < 2 ? en.units : j < 4 ? en.ref : (uint32_t)en.last_offset;
    return (uint32_t)((int32_t)(w << (j & 1 ? 0 : 16)) >> 16);
}

// What mesh_source_rank reads.
struct MeshView {
    const uint32_t *offsets;
    dims_ptr dims;
    uint32_t inner, pj, vector_round, periodic_mask;
    bool packed;
    int32_t d, shift_dim;
    __device__ __forceinline__ MeshView(const TorusDims *t, uint32_t torus, uint32_t inner_, uint32_t pj_, uint32_t vector)
        : offsets(offsets_after(t)), dims(const_dims(t)), inner(inner_), pj(pj_), vector_round(vector),
          periodic_mask(torus >> 16), packed((torus >> 10) & 1u), d((int32_t)(torus & 31u)), shift_dim((int32_t)((torus >> 5) & 31u) - 1) {}
};

// Mesh: does the move of entry `en` happen at rank R (R - C^ref inside the mesh in every masked
// dimension), and from which rank?  Offsets of non-periodic dimensions are signed values stored
// as two's complement, so one unsigned comparison tests both ends of the dimension.
template <int D>
__device__ __forceinline__ bool mesh_source_rank_d(const MeshView &a, const DevEntry &en, uint32_t R,
                                                   uint32_t &srcR) {
    const uint32_t mask = (en.meta >> 8) & 0xFFFFu;
    const uint32_t *cref = a.offsets + (size_t)en.ref * a.d;
    uint32_t cr[D], r[D];
    if (a.packed) {
#pragma unroll
        for (int j = 0; j < D; ++j) cr[j] = packed_reference(en, j);
    } else {
#pragma unroll
        for (int j = 0; j < D; ++j) cr[j] = cref[j];
    }
    uint32_t rem = R;
#pragma unroll
    for (int j = D - 1; j >= 0; --j) {
        uint32_t q;
        fast_divmod(rem, dim_of(a.dims, j), q, r[j]);
        rem = q;
    }
    uint32_t outside = 0;
#pragma unroll
    for (int j = 0; j < D; ++j)
        outside |= ((mask >> j) & 1u) & (uint32_t)((uint32_t)(r[j] - cr[j]) >= a.dims->d_dims[j].div);
    if (outside) return false;
    srcR = R;
    if (a.vector_round) {                                  // en.shift: the neighbour whose offsets move the block
        const uint32_t *cvec = a.offsets + (size_t)en.shift * a.d;
        uint32_t cv[D];
#pragma unroll
        for (int j = 0; j < D; ++j) cv[j] = cvec[j];
#pragma unroll
        for (int j = 0; j < D; ++j) {
            srcR -= cv[j] * a.dims->inner[j];                 // signed where the dimension does not wrap
            if (((a.periodic_mask >> j) & 1u) && r[j] < cv[j]) srcR += a.dims->d_dims[j].div * a.dims->inner[j];
        }
    } else if (a.shift_dim >= 0) {                         // en.shift: the distance along the one moving dimension
        uint32_t rj = 0;
#pragma unroll
        for (int j = 0; j < D; ++j)
            if (j == a.shift_dim) rj = r[j];                // uniform condition: a select, not a branch per lane
        srcR -= en.shift * a.inner;
        if (((a.periodic_mask >> a.shift_dim) & 1u) && rj < en.shift) srcR += a.pj * a.inner;
    }
    return true;
}

__device__ __forceinline__ bool mesh_source_rank(const MeshView &a, const DevEntry &en, uint32_t R,
                                                 uint32_t &srcR) {
    switch (a.d) {
        case 1: return mesh_source_rank_d<1>(a, en, R, srcR);
        case 2: return mesh_source_rank_d<2>(a, en, R, srcR);
        case 3: return mesh_source_rank_d<3>(a, en, R, srcR);
        case 4: return mesh_source_rank_d<4>(a, en, R, srcR);
        case 5: return mesh_source_rank_d<5>(a, en, R, srcR);
        case 6: return mesh_source_rank_d<6>(a, en, R, srcR);
        default: break;
    }
    // more dimensions: one pass with run-time indices
    const uint32_t mask = (en.meta >> 8) & 0xFFFFu;
    const uint32_t *cref = a.offsets + (size_t)en.ref * a.d;
    // in shift rounds en.shift is the distance itself: no row of the offset table is addressed with it
    const uint32_t *cvec = a.vector_round ? a.offsets + (size_t)en.shift * a.d : cref;
    uint32_t rem = R;
    bool has_source = true;
    srcR = R;
    for (int j = a.d - 1; j >= 0; --j) {
        uint32_t q, rj;
        fast_divmod(rem, dim_of(a.dims, j), q, rj);
        rem = q;
        const uint32_t pj = a.dims->d_dims[j].div;
        if (((mask >> j) & 1u) && (uint32_t)(rj - cref[j]) >= pj) has_source = false;
        if (a.vector_round || j == a.shift_dim) {
            const uint32_t cj = a.vector_round ? cvec[j] : en.shift;
            srcR -= cj * a.dims->inner[j];
            if (((a.periodic_mask >> j) & 1u) && rj < cj) srcR += pj * a.dims->inner[j];
        }
    }
    return has_source;
}

// GROUPS (rank-major buffers, shift rounds): the ranks are taken in groups of kBlockGroup, and inside
// a group the units are ordered (entry, rank, unit) as on slot-major buffers, so that large and tiny
// blocks fall into different workgroups and a workgroup's wide units are not held up by a second
// pass for narrow ones; prefix[] still counts one row's units.  Ranks beyond the last whole group
// are taken one by one.  (Stencil-shaped all-to-all on 32 x 32 x 32, blocks of 4096 / 64 / 1 bytes:
// groups of 8 ranks -4 % of the step, 32 -5 %, 64 -6.5 %, 128 and 256 -7.5 %, 1024 -7 %.)
constexpr uint32_t kBlockGroupLog2 = 7, kBlockGroup = 1u << kBlockGroupLog2;

__device__ __forceinline__ void fetch_now(const BlockArgs &a) {
    asm volatile("" ::"s"(a.entries), "s"(a.prefix), "s"(a.total), "s"(a.k), "s"(a.inner), "s"(a.pj), "s"(a.equal_units),
                 "s"(a.grouped), "s"(a.row), "s"(a.plane), "s"(a.mul_row), "s"(a.mul_inner), "s"(a.mul_pj), "s"(a.mul_units),
                 "s"(a.mul_plane), "s"(a.mul_group_row), "s"(a.shifts), "s"(a.more));
}

// HOPS: a unit of rank R's block through all the hops of an all-to-all (see move_through_stops), on at most HOPS dimensions.
// For blocks of a few units: loads through the caches, plain stores, as kBySize takes them.  A torus is a mesh here of
// which all dimensions wrap (MESH).
template <typename V, int HOPS>
__device__ __forceinline__ void block_through_stops(const BlockArgs &a, const DevEntry &en, uint32_t R, uint64_t off) {
    typedef typename Unaligned<V>::type UV;
    typedef const UV __attribute__((address_space(1))) *src_ptr;
    typedef UV __attribute__((address_space(1))) *dst_ptr;
    const dims_ptr dims = const_dims(a.dims);
    const int d = (int)(a.torus & 31u);
    const uint32_t *c = offsets_after(a.dims) + (size_t)en.shift * d;
    uint32_t at[HOPS], from = R, rem = R;
    bool outside = false;
#pragma unroll
    for (int t = 0; t < HOPS; ++t) {                     // the last hop first, modulo 2^32
        at[t] = from;
        if (t >= d) continue;
        const int j = d - 1 - t;
        uint32_t q, rj;
        fast_divmod(rem, dim_of(dims, j), q, rj);
        rem = q;
        const uint32_t cj = c[j], inner = dims->inner[j];
        const bool past = rj - cj >= dims->d_dims[j].div, wraps = (a.torus >> (16 + j)) & 1u;      // (see passes_end)
        from -= cj * inner;
        if (past && wraps) from += dims->d_dims[j].div * inner;
        outside = outside || (past && !wraps);
        at[t] = from;
    }
    if (outside) return;
    const V v = *(src_ptr)(block_address(en.src, from, en.src_stride) + off);
    const uint32_t m = (uint32_t)en.last_offset + (uint32_t)sizeof(V);
#pragma unroll
    for (int t = HOPS - 1; t >= 0; --t)                  // ranks on the way, each once
        if (at[t] != from && at[t] != (t ? at[t - 1] : R)) *(dst_ptr)(block_address(a.work + (uint64_t)en.ref * 16u, at[t], m) + off) = v;
    *(dst_ptr)(block_address(en.dst, R, en.dst_stride) + off) = v;
}

template <bool LDS, bool MESH, int POLICY, bool GROUPS = false, int HOPS = 0>
__global__ __launch_bounds__(kThreads) void block_round_kernel(const BlockArgs a) {
    if constexpr (!MESH || HOPS) fetch_now(a);
    const FastDiv d_row = fastdiv_of(a.mul_row, a.row, a.shifts, 0), d_inner = fastdiv_of(a.mul_inner, a.inner, a.shifts, 1),
                  d_pj = fastdiv_of(a.mul_pj, a.pj, a.shifts, 2),
                  d_units = fastdiv_of(a.mul_units, a.equal_units ? a.equal_units : 1u, a.shifts, 3),
                  d_plane = fastdiv_of(a.mul_plane, a.plane, a.more, 0),
                  d_group_row = fastdiv_of(a.mul_group_row, a.row << kBlockGroupLog2, a.more, 1);
    const bool entry_major = is_entry_major(a.more);
    __shared__ DevEntry lds[LDS ? kLdsEntries : 1];
    __shared__ uint32_t lds_prefix[LDS ? 2 * kLdsEntries + 1 : 1];
    const uint32_t *prefix = a.prefix;
    if constexpr (LDS) {
        // staged by the workgroup's last lanes, the entries (below) by its first: with few entries these are
        // different wavefronts, and the two loads are in flight together
        for (uint32_t q = kThreads - 1 - threadIdx.x; q <= 2 * a.k; q += kThreads) lds_prefix[q] = a.prefix[q];
        prefix = lds_prefix;
    }
    const EntryTable<LDS> table(a.entries, a.k, lds);     // synchronises the workgroup when LDS
    // (the two-step staging of the other kernels, with the first division between the steps, is 0.5 to 1 %
    // slower here)
    uint32_t tile;
    if (!tile_of_block(map_of(tiles_of(a.total), a.more), tile)) return;
    const uint32_t u = tile * (uint32_t)kThreads + threadIdx.x;
    if (u >= a.total) return;
    // flat index -> rank R, entry lo, unit ch of that entry's block
    uint32_t R = 0, lo = 0, ch = 0, w = u;
    uint32_t span_log2 = 0;                                // GROUPS: w counts through 2^span_log2 rows, entry by entry
    bool planes = entry_major;                           // w (then ch) counts through several ranks' blocks
    if constexpr (GROUPS) {
        planes = u < a.grouped;
        if (planes) {
            fast_divmod(u, d_group_row, R, w);          // R: the group, below its first rank
            R <<= kBlockGroupLog2;
            span_log2 = kBlockGroupLog2;
        } else {
            fast_divmod(u - a.grouped, d_row, R, w);
            R += fast_div(a.grouped, d_row);
        }
    } else if (!entry_major) {
        fast_divmod(u, d_row, R, w);                     // w: unit inside the rank's row
    }
    // entry-major: w counts through the entries one after another, each with the units of all p ranks
    if (a.k == 1) {
        ch = w;
    } else if (a.equal_units) {                            // equal blocks: plain division, no search
        fast_divmod(w, planes ? d_plane : d_units, lo, ch);
    } else {
        const uint32_t key = w >> span_log2;               // prefix[e] * 2^n <= w  <=>  prefix[e] <= w >> n
        uint32_t hi = a.k;                                 // largest e with prefix[e] <= key
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (prefix[mid] <= key) lo = mid;
            else hi = mid;
        }
        ch = w - (prefix[lo] << span_log2);
    }
    const DevEntry en = table[lo];
    if (planes) {                                          // ch still counts (rank, unit) inside the plane
        const FastDiv by_units = a.equal_units
                                     ? d_units
                                     : FastDiv{prefix[a.k + 1 + lo], (en.meta >> 24) & 1u, (en.meta >> 25) & 31u, en.units};
        const uint32_t in_plane = ch;
        uint32_t rank_in_span;
        fast_divmod(in_plane, by_units, rank_in_span, ch);
        R += rank_in_span;
    }
    if constexpr (HOPS > 0) {
        switch (en.meta & 0xFFu) {
            case 4: block_through_stops<vec16_t, HOPS>(a, en, R, unit_offset<vec16_t>(ch, en.last_offset)); break;
            case 3: block_through_stops<vec8_t, HOPS>(a, en, R, unit_offset<vec8_t>(ch, en.last_offset)); break;
            case 2: block_through_stops<uint32_t, HOPS>(a, en, R, unit_offset<uint32_t>(ch, en.last_offset)); break;
            case 1: block_through_stops<uint16_t, HOPS>(a, en, R, unit_offset<uint16_t>(ch, en.last_offset)); break;
            default: block_through_stops<uint8_t, HOPS>(a, en, R, ch); break;
        }
        return;
    }
    uint32_t srcR = R;                                    // modulo 2^32, see vector_source_rank
    if constexpr (MESH) {
        if (!mesh_source_rank(MeshView(a.dims, a.torus, a.inner, a.pj, is_vector_round(a.more)), en, R, srcR)) return;    // no source: leave the destination as it is
    } else if (is_vector_round(a.more)) {
        srcR = vector_source_rank(R, offsets_after(a.dims) + (size_t)en.shift * (a.torus & 31u), (int32_t)(a.torus & 31u), const_dims(a.dims));
    } else {
        const uint32_t q = fast_div(R, d_inner);
        const uint32_t rj = q - fast_div(q, d_pj) * a.pj;
        srcR -= en.shift * a.inner;
        if (rj < en.shift) srcR += a.pj * a.inner;
    }
    const uint64_t src = block_address(en.src, srcR, en.src_stride);
    const uint64_t dst = block_address(en.dst, R, en.dst_stride);
    switch (en.meta & 0xFFu) {
        case 4:
            if constexpr (POLICY & kBySize) {
                const uint64_t off = unit_offset<vec16_t>(ch, en.last_offset);
                // (the compiler joins two moves that differ in their cache policy only, and drops the policy: 32^3
                // stencil, 64 B 407 us; what is between these two lines stays as it is)
                if (en.units > kSmallUnits) {
                    asm volatile("; large block" ::: "memory");
                    move_unit<vec16_t, kStreamLoads>(dst, src, off);
                    asm volatile("; large block done" ::: "memory");
                } else {
                    move_unit<vec16_t, kPlainStores>(dst, src, off);
                }
            } else {
                move_unit<vec16_t, POLICY>(dst, src, unit_offset<vec16_t>(ch, en.last_offset));
            }
            break;
        case 3: move_unit<vec8_t, 0>(dst, src, unit_offset<vec8_t>(ch, en.last_offset)); break;
        case 2: move_unit<uint32_t, 0>(dst, src, unit_offset<uint32_t>(ch, en.last_offset)); break;
        case 1: move_unit<uint16_t, 0>(dst, src, unit_offset<uint16_t>(ch, en.last_offset)); break;
        default: move_unit<uint8_t, 0>(dst, src, ch); break;
    }
}

// Shift rounds of equal blocks on a mesh: the shift kernel's decomposition (no prefix search, no
// per-entry unit width) with the mesh's validity test.  Field names match what mesh_source_rank reads.
//
// Most ranks of a mesh are interior: every move has a source there.  The host marks, one bit per wavefront or tile,
// the runs of ranks where that holds (mesh_interior_units); such a wavefront skips the per-lane decode of all
// coordinates and does what the torus kernel does.  (Deciding this in the kernel from the first and last rank costs
// as much as it saves: the test is a chain of dependent scalar loads of launch constants, and what bounds these
// kernels is how long a wavefront holds its slot before its one load is under way.)  The others find the
// coordinates of C^ref in the entry itself.
// One bit per tile with the bounds of all the launch's entries, reference coordinates from a table -> as here, boxes:
// 45 x 37 x 29, 100 B, slot-major 121 -> 96 us (the torus: 96), 40^3, 128 B 163 -> 157 and slot-major 175 -> 147, 8^5,
// 40 neighbours up to 3 away, 256 B 513 -> 450 and 4 KiB 6460 -> 5908, allgather 8^5, 1 KiB 1444 -> 1265, 12^3, 40 B
// 12.8 -> 9.5.
struct MeshArgs {
    const DevEntry *entries;
    const TorusDims *dims;     // and after it the [s][d] effective coordinates
    const uint32_t *interior;  // a bit per wavefront (64 units) or per tile: all the blocks it moves have a source
    uint32_t total, k;
    uint32_t inner, pj;        // rank stride and size of the moving dimension (1, 1 for a same-rank copy)
    uint32_t chunks, p;
    uint32_t mul_chunks, mul_k, mul_inner, mul_pj, mul_p;
    uint32_t shifts;           // chunks, k, inner, pj
    uint32_t more;             // p; launch_flags
    uint32_t torus;            // torus_bits
};
static_assert(sizeof(MeshArgs) <= kCheapArguments, "launch cost");

template <typename V, bool LDS, int POLICY, bool TAIL>
__global__ __launch_bounds__(kThreads) void mesh_shift_round_kernel(const MeshArgs a) {
    __shared__ DevEntry lds[LDS ? kLdsEntries : 1];
    uint32_t tile;
    if (!tile_of_block(map_of(tiles_of(a.total), a.more), tile)) return;
    StagedEntries<LDS> staging;
    staging.issue(a.entries, a.k);
    const uint32_t wave = tile * (kThreads / 64u) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t bit = (a.torus >> 11) & 1u ? tile : wave;
    typedef const uint32_t __attribute__((address_space(4))) *const_word_ptr;
    const bool interior = (((const_word_ptr)(uintptr_t)a.interior)[bit >> 5] >> (bit & 31u)) & 1u;
    const uint32_t u = tile * (uint32_t)kThreads + threadIdx.x;
    uint32_t t, ch, R, e;
    fast_divmod(u, fastdiv_of(a.mul_chunks, a.chunks, a.shifts, 0), t, ch);
    if (is_entry_major(a.more)) fast_divmod(t, fastdiv_of(a.mul_p, a.p, a.more, 0), e, R);
    else fast_divmod(t, fastdiv_of(a.mul_k, a.k, a.shifts, 1), R, e);
    staging.commit(lds);
    if (u >= a.total) return;
    const DevEntry en = LDS ? lds[e] : a.entries[e];
    uint32_t srcR = R;
    if (interior) {                                       // every move has its source: the torus kernel's path
        const uint32_t shift_dim = (a.torus >> 5) & 31u;  // plus 1
        if (shift_dim) {
            srcR -= en.shift * a.inner;
            if ((a.torus >> (15u + shift_dim)) & 1u) {    // the moving dimension wraps
                const uint32_t q = fast_div(R, fastdiv_of(a.mul_inner, a.inner, a.shifts, 2));
                const uint32_t rj = q - fast_div(q, fastdiv_of(a.mul_pj, a.pj, a.shifts, 3)) * a.pj;
                if (rj < en.shift) srcR += a.pj * a.inner;
            }
        }
    } else if (!mesh_source_rank(MeshView(a.dims, a.torus, a.inner, a.pj, 0u), en, R, srcR)) {
        return;                                           // no source: leave the destination as it is
    }
    move_unit<V, POLICY>(block_address(en.dst, R, en.dst_stride), block_address(en.src, srcR, en.src_stride),
                      unit_offset_if<V, TAIL>(ch, last_offset_of<V>(a.chunks, a.more)));
}

// ---- small blocks re-tiled through LDS (the staged schedule) ----------------------------------
// A workgroup moves a tile of up to kTileUnits units: the blocks of `ranks` consecutive ranks for
// all entries of the launch.  It reads them in the order that suits the source (entry after entry
// of one rank where the source is a rank-major buffer, rank after rank of one plane where it is a
// slot-major one), eight independent loads per lane, parks them in LDS, and writes them in the
// order that suits the destination.  Both sides then see runs of hundreds of bytes although the
// blocks themselves may be 16 bytes.  In a round the tile's ranks are SOURCE ranks (the kernel
// pushes: block e of rank S goes to rank S + v_e), so that all pieces of one send-buffer row, those
// moving up and those moving down the dimension, are read by one workgroup and share their memory
// lines; every destination block is still written exactly once.  The last launch below tiles by
// destination rank instead, because it is the receive rows that it writes whole.
constexpr uint32_t kTileUnits = 2048;                  // the largest tile: 8 units per lane
constexpr uint32_t kSmallTileUnits = 1024;             // used where the blocks of one rank fit it: 3 % faster at 16-byte
                                                       // blocks, 2 % at 128 bytes (512: 4 % slower than 1024)

struct StagedRoundArgs {
    const DevEntry *entries;   // the first k_rows entries read a rank-major buffer, the others a slot-major one;
                               // destinations are mostly slot-major planes of the workspace
    uint32_t n_tiles;
    uint32_t p, k, k_rows;
    uint32_t ranks;            // ranks per tile: k * ranks * upb <= kTileUnits
    uint32_t upb;              // units per block
    uint32_t inner, pj;        // the moving dimension (1, 1: same-rank copies)
    uint32_t row, plane;       // k_rows * upb (at least 1); ranks * upb
    uint32_t mul_upb, mul_row, mul_plane, mul_inner, mul_pj;
    uint32_t shifts;           // upb, row, plane, inner
    uint32_t more;             // pj; launch_flags
    uint32_t inner2, pj2, mul_inner2, mul_pj2, shifts2;      // TWO: the second dimension
};
static_assert(sizeof(StagedRoundArgs) <= kCheapArguments, "launch cost");

__device__ __forceinline__ void fetch_now(const StagedRoundArgs &a) {
    asm volatile("" ::"s"(a.entries), "s"(a.n_tiles), "s"(a.p), "s"(a.k), "s"(a.k_rows), "s"(a.ranks), "s"(a.upb),
                 "s"(a.inner), "s"(a.pj), "s"(a.row), "s"(a.plane), "s"(a.mul_upb), "s"(a.mul_row), "s"(a.mul_plane),
                 "s"(a.mul_inner), "s"(a.mul_pj), "s"(a.shifts), "s"(a.more));
}

// Unit q of a tile in the order of its sources: (rank, entry, unit) over the entries that read a rank-major buffer, which
// come first, then (entry, rank, unit) over the others.  A lane with no unit takes the tile's first one and drops it: its
// loads stay straight-line code, all in flight together.
struct TileUnit {
    uint32_t e, r, c;
    bool any;
    __device__ __forceinline__ TileUnit(uint32_t q, uint32_t n_rows, uint32_t n_all, uint32_t k_rows, uint32_t n_ranks,
                                        const FastDiv &d_row, const FastDiv &d_plane, const FastDiv &d_upb) {
        uint32_t rem;
        if (q < n_rows) {
            fast_divmod(q, d_row, r, rem);
            fast_divmod(rem, d_upb, e, c);
        } else {
            fast_divmod(q - n_rows, d_plane, e, rem);
            fast_divmod(rem, d_upb, r, c);
            e += k_rows;
        }
        any = q < n_all && r < n_ranks;
        e = any ? e : 0u;
        r = any ? r : 0u;
        c = any ? c : 0u;
    }
};

// TWO: the rounds of two dimensions in one launch.  All entries read send-buffer rows; the first hop goes to `dst` (0: the
// block makes none along the first dimension), the second one by `units` steps to `last_offset` (0: none).  The second
// round's launch read the planes that the first one's had written, and more blocks of the same rows.  Collectives, us, two
// launches -> this one: 64^3, 26 neighbours, 16 B 108 -> 91, 32 B 187 -> 177, 64 B 354 -> 312, 100 B 590 -> 565; 32^3, 16 B
// 20.6 -> 16.7; 40^3, 20 neighbours, 32 B 43.6 -> 36.5; 16^4, 80, 64 B 367 -> 346; 8^5, 40, 64 B 143 -> 125.
template <typename V, int POLICY, uint32_t UPL, bool TAIL, bool TWO = false>
__global__ __launch_bounds__(kThreads) void staged_round_kernel(const StagedRoundArgs a) {
    fetch_now(a);
    const FastDiv d_upb = fastdiv_of(a.mul_upb, a.upb, a.shifts, 0), d_row = fastdiv_of(a.mul_row, a.row, a.shifts, 1),
                  d_plane = fastdiv_of(a.mul_plane, a.plane, a.shifts, 2), d_inner = fastdiv_of(a.mul_inner, a.inner, a.shifts, 3),
                  d_pj = fastdiv_of(a.mul_pj, a.pj, a.more, 0);
    __shared__ DevEntry lds[kLdsEntries];
    extern __shared__ __align__(16) unsigned char tile_bytes[];
    V *tile = (V *)tile_bytes;
    typedef typename Unaligned<V>::type UV;
    typedef const UV __attribute__((address_space(1))) *src_ptr;
    typedef UV __attribute__((address_space(1))) *dst_ptr;
    uint32_t tile_id;
    if (!tile_of_block(map_of(a.n_tiles, a.more), tile_id)) return;          // (before anything is loaded: the grid is padded)
    const EntryTable<true> table(a.entries, a.k, lds);
    const uint32_t R0 = tile_id * a.ranks;
    const uint32_t n = a.p - R0 < a.ranks ? a.p - R0 : a.ranks;
    const uint32_t plane = a.plane, pitch = plane + 1u;      // padded planes: the strided LDS writes spread over the banks
    const uint32_t n_rows = a.k_rows * plane, n_all = a.k * plane;
    const uint64_t last_offset = last_offset_of<V>(a.upb, a.more);
    V regs[UPL];
    uint32_t at[UPL];                          // where in the tile the unit goes; ~0: no unit
#pragma unroll
    for (uint32_t it = 0; it < UPL; ++it) {
        const TileUnit u(threadIdx.x + it * (uint32_t)kThreads, n_rows, n_all, a.k_rows, n, d_row, d_plane, d_upb);
        const DevEntry en = table[u.e];
        const src_ptr sp = (src_ptr)(block_address(en.src, R0 + u.r, en.src_stride) + unit_offset_if<V, TAIL>(u.c, last_offset));
        if constexpr ((POLICY & kStreamLoads) && sizeof(V) == 16) regs[it] = __builtin_nontemporal_load(sp);
        else regs[it] = *sp;
        at[it] = u.any ? u.e * pitch + u.r * a.upb + u.c : ~0u;
    }
#pragma unroll
    for (uint32_t it = 0; it < UPL; ++it)
        if (at[it] != ~0u) tile[at[it]] = regs[it];
    __syncthreads();
#pragma unroll
    for (uint32_t it = 0; it < UPL; ++it) {    // (entry, rank, unit): dense runs of every plane
        const uint32_t q = threadIdx.x + it * (uint32_t)kThreads;
        uint32_t e, r, c, rem;
        fast_divmod(q, d_plane, e, rem);
        fast_divmod(rem, d_upb, r, c);
        if (q < n_all && r < n) {
            const DevEntry en = table[e];
            // the tile's ranks are source ranks S: the block goes to the rank `shift` steps on
            const uint32_t S = R0 + r;
            const uint32_t qq = fast_div(S, d_inner);
            const uint32_t sj = qq - fast_div(qq, d_pj) * a.pj;
            uint32_t R = S + en.shift * a.inner;
            R -= sj + en.shift >= a.pj ? a.pj * a.inner : 0u;
            const auto put = [&](uint64_t plane_of, uint32_t rank) {
                const dst_ptr dp = (dst_ptr)(block_address(plane_of, rank, en.dst_stride) + unit_offset_if<V, TAIL>(c, last_offset));
                if constexpr (sizeof(V) == 16 && !(POLICY & kPlainStores)) __builtin_nontemporal_store(tile[e * pitch + rem], dp);
                else *dp = tile[e * pitch + rem];
            };
            if (!TWO || en.dst) put(en.dst, R);
            if constexpr (TWO) {
                const uint32_t q2 = fast_div(S, fastdiv_of(a.mul_inner2, a.inner2, a.shifts2, 0));
                const uint32_t s2 = q2 - fast_div(q2, fastdiv_of(a.mul_pj2, a.pj2, a.shifts2, 1)) * a.pj2;
                R += en.units * a.inner2;
                R -= s2 + en.units >= a.pj2 ? a.pj2 * a.inner2 : 0u;
                if (en.last_offset) put(en.last_offset, R);
            }
        }
    }
}

// Last launch of the staged schedule: entry i brings receive block i of every rank from where its
// last hop starts (a plane of the workspace or the send buffer), along the entry's own dimension.
// A workgroup takes `ranks` consecutive ranks: it reads their blocks in the order that suits the
// sources (as the rounds above do) into an LDS tile, one padded plane per receive block so that
// the strided LDS accesses spread over the banks, and writes the tile out in row order as one
// dense run of ranks * s * m bytes: small blocks are written as whole receive rows.
struct alignas(16) DeliverEntry {
    uint64_t src;          // address of rank 0's source block
    uint32_t src_stride;   // bytes between consecutive ranks in the source
    uint32_t slot;         // receive block i
    uint32_t shift, pj;    // residue v along the entry's dimension (0: same rank); that dimension's size
    uint32_t back, wrap;   // v * inner_j; p_j * inner_j
    FastDiv d_inner, d_pj;
    __device__ __forceinline__ uint64_t source_of(uint32_t R) const {
        const uint32_t q = fast_div(R, d_inner);
        const uint32_t rj = q - fast_div(q, d_pj) * pj;
        return block_address(src, R - back + (rj < shift ? wrap : 0u), src_stride);
    }
};
static_assert(sizeof(DeliverEntry) == 64, "four 16-byte words per entry");

struct DeliverArgs {
    const DeliverEntry *entries;   // the first k_rows entries read a rank-major buffer
    uint64_t dst;                  // rank 0's receive row; rows of s blocks, back to back
    uint32_t n_tiles;
    uint32_t p, s, k_rows;
    uint32_t ranks;                // ranks per workgroup: s * ranks * upb <= UPL * kThreads
    uint32_t upb;                  // units per block
    uint32_t rows, plane, row;     // k_rows * upb (at least 1); ranks * upb; s * upb
    uint32_t mul_upb, mul_rows, mul_plane, mul_row;
    uint32_t shifts;               // upb, rows, plane, row
    uint32_t more;                 // launch_flags
};
static_assert(sizeof(DeliverArgs) <= kCheapArguments, "launch cost");

__device__ __forceinline__ void fetch_now(const DeliverArgs &a) {
    asm volatile("" ::"s"(a.entries), "s"(a.dst), "s"(a.n_tiles), "s"(a.p), "s"(a.s), "s"(a.k_rows), "s"(a.ranks), "s"(a.upb),
                 "s"(a.rows), "s"(a.plane), "s"(a.row), "s"(a.mul_upb), "s"(a.mul_rows), "s"(a.mul_plane), "s"(a.mul_row),
                 "s"(a.shifts), "s"(a.more));
}

template <typename V, int POLICY, uint32_t UPL>
__global__ __launch_bounds__(kThreads) void deliver_kernel(const DeliverArgs a) {
    fetch_now(a);
    const FastDiv d_upb = fastdiv_of(a.mul_upb, a.upb, a.shifts, 0), d_rows = fastdiv_of(a.mul_rows, a.rows, a.shifts, 1),
                  d_plane = fastdiv_of(a.mul_plane, a.plane, a.shifts, 2), d_row = fastdiv_of(a.mul_row, a.row, a.shifts, 3);
    __shared__ DeliverEntry lds[kLdsEntries];
    extern __shared__ __align__(16) unsigned char tile_bytes[];
    V *tile = (V *)tile_bytes;
    typedef typename Unaligned<V>::type UV;
    typedef const UV __attribute__((address_space(1))) *src_ptr;
    typedef UV __attribute__((address_space(1))) *dst_ptr;
    uint32_t tile_id;
    if (!tile_of_block(map_of(a.n_tiles, a.more), tile_id)) return;          // (before anything is loaded: the grid is padded)
    for (uint32_t w = threadIdx.x; w < a.s * 4u; w += kThreads) ((vec16_t *)lds)[w] = ((const vec16_t *)a.entries)[w];
    __syncthreads();
    const uint32_t R0 = tile_id * a.ranks;
    const uint32_t n = a.p - R0 < a.ranks ? a.p - R0 : a.ranks;
    const uint32_t plane = a.plane, pitch = plane + 1u;
    const uint32_t n_rows = a.k_rows * plane, n_all = a.s * plane;
    V regs[UPL];
    uint32_t at[UPL];                                    // where in the tile the unit goes; ~0: no unit
#pragma unroll
    for (uint32_t it = 0; it < UPL; ++it) {
        const TileUnit u(threadIdx.x + it * (uint32_t)kThreads, n_rows, n_all, a.k_rows, n, d_rows, d_plane, d_upb);
        const DeliverEntry &en = lds[u.e];
        const src_ptr sp = (src_ptr)(en.source_of(R0 + u.r) + (uint64_t)u.c * sizeof(V));
        if constexpr ((POLICY & kStreamLoads) && sizeof(V) == 16) regs[it] = __builtin_nontemporal_load(sp);
        else regs[it] = *sp;
        at[it] = u.any ? en.slot * pitch + u.r * a.upb + u.c : ~0u;
    }
#pragma unroll
    for (uint32_t it = 0; it < UPL; ++it)
        if (at[it] != ~0u) tile[at[it]] = regs[it];
    __syncthreads();
    const uint64_t out = a.dst + (uint64_t)R0 * a.s * a.upb * sizeof(V);
#pragma unroll
    for (uint32_t it = 0; it < UPL; ++it) {              // (rank, block, unit): the receive rows, back to back
        const uint32_t q = threadIdx.x + it * (uint32_t)kThreads;
        uint32_t i, r, c, rem;
        fast_divmod(q, d_row, r, rem);
        fast_divmod(rem, d_upb, i, c);
        if (r < n) {
            const dst_ptr dp = (dst_ptr)(out + (uint64_t)q * sizeof(V));
            if constexpr (sizeof(V) == 16 && !(POLICY & kPlainStores)) __builtin_nontemporal_store(tile[i * pitch + r * a.upb + c], dp);
            else *dp = tile[i * pitch + r * a.upb + c];
        }
    }
}

// The same for blocks of any size: rows of s * m bytes are packed in LDS as they lie in memory, shifted so that 16
// bytes of LDS are an aligned 16 bytes of the receive buffer.  Blocks are read in units of V (the last one of a block
// overlaps its predecessor) and land at any byte of the tile; what leaves it are whole aligned units, and single bytes
// only at the two ends of the tile.  What bounds rounds over such blocks is that each writes parts of sectors, which
// memory merges with what it holds (a quarter of the write requests at 100 B; here 1 %, 1.01 times the rows' bytes, and
// 1.39 times the blocks fetched for the sectors at their ends).  Staged schedule, one
// launch per dimension -> this: 64^3, 26 neighbours, 100 B 1006 -> 584 us (436 at the copy rate), allgather 449 -> 250;
// 24^3, 20 B 20.8 -> 14.4.
template <typename V, int POLICY, uint32_t UPL>
__global__ __launch_bounds__(kThreads) void deliver_bytes_kernel(const DeliverArgs a) {
    fetch_now(a);
    const FastDiv d_upb = fastdiv_of(a.mul_upb, a.upb, a.shifts, 0), d_rows = fastdiv_of(a.mul_rows, a.rows, a.shifts, 1),
                  d_plane = fastdiv_of(a.mul_plane, a.plane, a.shifts, 2);
    const uint32_t m = a.row;                            // bytes of a block
    __shared__ DeliverEntry lds[kLdsEntries];
    extern __shared__ __align__(16) unsigned char tile_bytes[];
    typedef typename Unaligned<V>::type UV;
    typedef const UV __attribute__((address_space(1))) *src_ptr;
    typedef vec16_t __attribute__((address_space(1))) *dst_ptr;
    typedef unsigned char __attribute__((address_space(1))) *byte_ptr;
    uint32_t tile_id;
    if (!tile_of_block(map_of(a.n_tiles, a.more), tile_id)) return;
    for (uint32_t w = threadIdx.x; w < a.s * 4u; w += kThreads) ((vec16_t *)lds)[w] = ((const vec16_t *)a.entries)[w];
    __syncthreads();
    const uint32_t R0 = tile_id * a.ranks;
    const uint32_t n = a.p - R0 < a.ranks ? a.p - R0 : a.ranks;
    const uint32_t n_rows = a.k_rows * a.plane, n_all = a.s * a.plane, row_bytes = a.s * m;
    const uint64_t out = a.dst + (uint64_t)R0 * row_bytes;
    const uint32_t skew = (uint32_t)out & 15u;
    V regs[UPL];
    uint32_t at[UPL];                                    // where in the tile the unit goes; ~0: no unit
#pragma unroll
    for (uint32_t it = 0; it < UPL; ++it) {
        const TileUnit u(threadIdx.x + it * (uint32_t)kThreads, n_rows, n_all, a.k_rows, n, d_rows, d_plane, d_upb);
        const DeliverEntry &en = lds[u.e];
        const uint32_t unpulled = u.c * (uint32_t)sizeof(V), off = unpulled < m - (uint32_t)sizeof(V) ? unpulled : m - (uint32_t)sizeof(V);
        const src_ptr sp = (src_ptr)(en.source_of(R0 + u.r) + off);
        if constexpr ((POLICY & kStreamLoads) && sizeof(V) == 16) regs[it] = __builtin_nontemporal_load(sp);
        else regs[it] = *sp;
        at[it] = u.any ? skew + u.r * row_bytes + en.slot * m + off : ~0u;
    }
#pragma unroll
    for (uint32_t it = 0; it < UPL; ++it)
        if (at[it] != ~0u) *(UV *)(tile_bytes + at[it]) = regs[it];
    __syncthreads();
    const uint32_t end = skew + n * row_bytes;           // of the tile's bytes in LDS, the first being skew
    const uint64_t base = out - skew;
#pragma unroll
    for (uint32_t it = 0; it < UPL; ++it) {
        const uint32_t b = (threadIdx.x + it * (uint32_t)kThreads) * 16u;
        if (b >= skew && b + 16u <= end) {
            const vec16_t v = *(const vec16_t *)(tile_bytes + b);
            if constexpr (POLICY & kPlainStores) *(dst_ptr)(base + b) = v;
            else __builtin_nontemporal_store(v, (dst_ptr)(base + b));
        }
    }
    // the bytes in front of the first whole unit and behind the last one, a lane each
    const uint32_t head = (skew + 15u) & ~15u, tail = end & ~15u;
    const uint32_t b = threadIdx.x < 16u ? skew + threadIdx.x : tail + threadIdx.x - 16u;
    const bool mine = threadIdx.x < 16u ? b < head && b < end : threadIdx.x < 32u && b < end && tail >= head;
    if (mine) *(byte_ptr)(base + b) = tile_bytes[b];
}

// ---- small collectives in one launch -------------------------------------------------------------
// Block i of an all-to-all only ever moves between its own places (send slot, workspace slots, receive slot),
// and so does every column of its units: a workgroup takes one block's column of all p ranks through all its
// hops, one hop after the other with a barrier between, making every stop in the same buffers as the rounds.  What
// bounds these collectives is first the cost of a launch per dimension, then the latency of the one launch: every
// dependent access is 0.5 to 2 us.  So the hops travel in the request's table, the first one of each chain at the
// chain's own index (no look-up in front of it), and a hop takes what the hop before it has stored from LDS
// instead of waiting for the store and loading it again.
constexpr uint32_t kChainThreads = 1024, kChainUnitsPerLane = 4;
struct ChainHop {
    uint64_t src, dst;                 // addresses of rank 0's blocks
    uint32_t src_stride, dst_stride;
    uint32_t shift, inner, pj;         // residue v along the hop's dimension, its rank stride and size (0, 1, 1: same rank)
    uint32_t mul_inner, mul_pj, shifts;
};
static_assert(sizeof(ChainHop) == 48, "three 16-byte words");
// In the table: the chains' first hops, then their others, chain after chain; then [chains + 1] words, where the others
// of each chain begin, counted behind the first ones.
struct ChainHead {
    const ChainHop *table;
    uint32_t n_units;                  // p * column
    uint32_t chunks, column, groups;   // units of a block, of a workgroup's column; columns of a block
    uint32_t n_chains, n_hops;
    uint32_t mul_column, mul_groups;
    uint32_t more;                     // shifts of column, groups; launch_flags
};
static_assert(sizeof(ChainHead) <= kCheapArguments, "launch cost");
// The allocation-free call has no table and passes the hops with the launch (3.5 KiB; a launch that writes a table
// first costs more: 8 x 8 x 8, 26 neighbours, 64 B 13 -> 11 us).
constexpr uint32_t kChainHopsByValue = 72;
struct ChainArgs {
    ChainHead head;
    uint32_t table[kChainHopsByValue * sizeof(ChainHop) / 4 + kChainHopsByValue + 1];
};
static_assert(sizeof(ChainArgs) <= 4096 && offsetof(ChainArgs, table) % 16 == 0, "kernel arguments");

typedef const ChainHop __attribute__((address_space(4))) *chain_hops_ptr;
__device__ __forceinline__ const ChainHead &chain_head(const ChainHead &a) { return a; }
__device__ __forceinline__ const ChainHead &chain_head(const ChainArgs &a) { return a.head; }
__device__ __forceinline__ chain_hops_ptr chain_hops(const ChainHead &a) { return (chain_hops_ptr)(uintptr_t)a.table; }
__device__ __forceinline__ chain_hops_ptr chain_hops(const ChainArgs &) {
    typedef const char __attribute__((address_space(4))) *bytes_ptr;
    return (chain_hops_ptr)((bytes_ptr)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(ChainArgs, table));
}

// Synchronises the workgroup on LDS only: stores to global memory stay in flight.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// One hop in scalar registers; the constructor makes the compiler fetch it there and then.
struct HopNow {
    uint64_t src, dst;
    uint32_t src_stride, dst_stride, shift, back, wrap;
    FastDiv d_inner, d_pj;
    __device__ __forceinline__ HopNow(chain_hops_ptr table, uint32_t h)
        : src(table[h].src), dst(table[h].dst), src_stride(table[h].src_stride),
          dst_stride(table[h].dst_stride), shift(table[h].shift),
          d_inner(fastdiv_of(table[h].mul_inner, table[h].inner, table[h].shifts, 0)),
          d_pj(fastdiv_of(table[h].mul_pj, table[h].pj, table[h].shifts, 1)) {
        asm volatile("" ::"s"(src), "s"(dst), "s"(src_stride), "s"(dst_stride), "s"(shift), "s"(d_inner.div), "s"(d_inner.mul),
                     "s"(d_pj.div), "s"(d_pj.mul));
        back = shift * d_inner.div;
        wrap = d_inner.div * d_pj.div;
    }
    __device__ __forceinline__ uint32_t source_rank(uint32_t R) const {
        const uint32_t q = fast_div(R, d_inner);
        const uint32_t rj = q - fast_div(q, d_pj) * d_pj.div;
        return R - back + (rj < shift ? wrap : 0u);
    }
};

// A place that a chain writes twice (Algorithm 1 alternates between two) is written twice by the same lane, in
// order.  The bytes that a last unit shares with its predecessor are written by two lanes (TAIL), by both at every
// stop: whichever of their last stores lands last carries the last stop's bytes.  No stop is read back from memory, so
// that no store is waited for.
// Hops through memory, arguments by value -> as here: 8 x 8, 8 neighbours, 32 B 4.1 -> 3.6 us a start, 8^3, 26
// neighbours, 64 B 6.4 -> 4.5, 10^3, 64 B 9.3 -> 6.2 (allgather 9.0 -> 5.3), 45^2, 32 B 6.6 -> 4.7.
template <typename V, bool TAIL, uint32_t UPL, typename ARGS>
__global__ __launch_bounds__(kChainThreads) void chain_kernel(const ARGS from) {
    typedef typename Unaligned<V>::type UV;
    typedef const UV __attribute__((address_space(1))) *src_ptr;
    typedef UV __attribute__((address_space(1))) *dst_ptr;
    extern __shared__ __align__(16) unsigned char tile_bytes[];
    V *tile = (V *)tile_bytes;
    const ChainHead &a = chain_head(from);
    const chain_hops_ptr table = chain_hops(from);
    uint32_t chain, group;
    fast_divmod(blockIdx.x, fastdiv_of(a.mul_groups, a.groups, a.more, 1), chain, group);
    const uint32_t n_threads = UPL > 1 ? kChainThreads : 0u;          // (one unit per lane: no stride)
    const FastDiv d_column = fastdiv_of(a.mul_column, a.column, a.more, 0);
    HopNow hop(table, chain);
    uint32_t unit[UPL], rank[UPL];
    uint64_t off[UPL];
    bool has[UPL];
    V v[UPL];
#pragma unroll
    for (uint32_t it = 0; it < UPL; ++it) {
        unit[it] = threadIdx.x + it * n_threads;
        uint32_t c;
        fast_divmod(unit[it], d_column, rank[it], c);
        const uint32_t ch = group * a.column + c;
        has[it] = unit[it] < a.n_units && ch < a.chunks;
        unit[it] = has[it] ? unit[it] : 0u;              // a lane without a unit reads rank 0's first one
        rank[it] = has[it] ? rank[it] : 0u;
        off[it] = has[it] ? unit_offset_if<V, TAIL>(ch, last_offset_of<V>(a.chunks, a.more)) : 0u;
        v[it] = *(src_ptr)(block_address(hop.src, hop.source_rank(rank[it]), hop.src_stride) + off[it]);
    }
    const auto stop = [&](const HopNow &h) {
#pragma unroll
        for (uint32_t it = 0; it < UPL; ++it)
            if (has[it]) *(dst_ptr)(block_address(h.dst, rank[it], h.dst_stride) + off[it]) = v[it];
    };
    // on their way while the blocks are
    typedef const uint32_t __attribute__((address_space(4))) *const_word_ptr;
    const const_word_ptr later = (const_word_ptr)(table + a.n_hops);
    uint32_t at = a.n_chains + later[chain];
    const uint32_t end = a.n_chains + later[chain + 1];
    HopNow next(table, at < end ? at : chain);
    // (waited for here, not behind the first stop: that wait would be for its stores as well)
    __builtin_amdgcn_s_waitcnt(0x0F70);                  // vmcnt(0)
    stop(hop);
    while (at < end) {
#pragma unroll
        for (uint32_t it = 0; it < UPL; ++it)
            if (has[it]) tile[unit[it]] = v[it];
        lds_barrier();
        hop = next;
        ++at;
        next = HopNow(table, at < end ? at : chain);
#pragma unroll
        for (uint32_t it = 0; it < UPL; ++it)            // the same unit of the rank that the hop comes from
            v[it] = tile[unit[it] + (hop.source_rank(rank[it]) - rank[it]) * a.column];
        stop(hop);
        if (at < end) lds_barrier();                     // what this hop has read may now be replaced
    }
}

// Plain streaming copy with the same access shape: the measured ceiling.
template <typename V>
__global__ __launch_bounds__(kThreads) void copy_kernel(const V *__restrict__ src, V *__restrict__ dst,
                                                        uint64_t n_units) {
    const uint64_t u = (uint64_t)blockIdx.x * kThreads + threadIdx.x;
    if (u < n_units) __builtin_nontemporal_store(__builtin_nontemporal_load(src + u), dst + u);
}

// Writes up to kStoreWords 32-bit words, carried in the kernel's own arguments, to device
// memory: how a table of block index maps reaches the device when the host may neither
// allocate nor copy (the launch itself is the transfer, and it is ordered by the stream).
constexpr uint32_t kStoreWords = 768;
struct TableChunk {
    uint32_t *dst;
    uint32_t n;            // words to write, at most kStoreWords
    uint32_t reserved;
    uint32_t words[kStoreWords];
};

__global__ __launch_bounds__(kThreads) void table_store_kernel(const TableChunk c) {
    const uint32_t i = blockIdx.x * (uint32_t)kThreads + threadIdx.x;
    if (i < c.n) c.dst[i] = c.words[i];
}

}  // namespace iso

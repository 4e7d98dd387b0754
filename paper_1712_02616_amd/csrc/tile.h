// Tiles: the access pattern of the slice-resident kernels.
//
// A channel's values are N rows of HW contiguous elements, C*HW elements
// apart.  A tile is what one group of `lanes` adjacent threads (64 or 256)
// reads or writes with one access each: either several whole rows (short
// rows) or a part of one row (long rows).  Everything about a tile that is
// not the lane's own place in it is the same for all its lanes, so it is
// scalar arithmetic; a lane adds one 32-bit byte offset, formed once, to a
// scalar address, and one compare says whether it has an access in the tile.
// (A division by the row length and 64-bit vector arithmetic per access, as
// the general mapping does, costs a short channel 7-12% of its time.)
//
// Ragged rows.  Rows that 16-byte accesses do not divide still move in them,
// as many to each row, and the elements left over at a row's two ends (its
// edges) move one by one: the edges of a channel are numbered through and
// dealt out to the threads.  The accesses of a long row start at the first
// 16-byte boundary in it, so that up to 15 bytes (its head) come before them;
// those of a short row start at the row, at the alignment of an element, which
// leaves fewer elements over.  (Unaligned accesses are allowed but cost where
// they are aligned to 2 bytes only: forward / backward of (8, 512, 65x65) fp16
// 20.9 / 30.3 us with them, 16.7 / 23.2 with heads; 2-byte accesses 28.3 /
// 38.0.)
#pragma once

#include "fused.h"

namespace iabn_impl {

struct TileGeom {
    uint32_t C;
    uint32_t tiles;       // tiles per channel
    uint32_t lanes;       // threads per tile, 64 or 256
    uint32_t split_rows;  // 1: a row holds `per` tiles; 0: a tile holds `per` rows
    uint32_t per;
    iabn_divmagic_t per_div;  // division by per
    uint32_t vrow;            // accesses per row
    iabn_divmagic_t vrow_div;
    uint32_t cap;         // byte offset of a tile's last access (split_rows: in the row)
    uint32_t cap_end;     // the same for a channel's last tile, which may hold fewer rows
    uint32_t tile_bytes;  // lanes * access bytes
    uint32_t wrap_at;     // split_rows: bytes of a row's tiles; else never reached
    uint32_t step;        // tiles from one of a slice's to its next, and what that adds to
    uint32_t step_at;     // TileWalk::at and
    uint64_t step_base;   // TileWalk::base
    uint64_t row_bytes;
    uint64_t nstride;     // bytes between rows of a channel
    uint32_t head_mask;   // 15: a row's accesses start at its first 16-byte boundary; 0: at the row
    uint32_t edge;        // elements of a row that no access holds
    iabn_divmagic_t edge_div;
    uint32_t edges;       // of a channel: N * edge
    uint32_t body_bytes;  // of a row's accesses
    uint32_t xcd_order;   // slices in contiguous ranges per XCD (see block_slice)
    uint32_t P;           // slices (blocks) per channel
    double m, inv_m;      // elements per channel
};

// A lane's place in every tile: its byte offset (split_rows: from the tile's
// start, else from its first row; a lane with no place in it is past
// Tile::cap), and that of its row, for the row's head.
struct TileLane {
    uint32_t off, row;
};

template <int AB>
__device__ __forceinline__ TileLane tile_lane(const TileGeom& g) {
    const uint32_t tl = threadIdx.x & (g.lanes - 1);
    if (g.split_rows) return {tl * AB, 0u};
    const uint32_t r = iabn_divmagic_div(tl, g.vrow_div);
    const uint32_t row = r * static_cast<uint32_t>(g.nstride);
    return {row + (tl - r * g.vrow) * AB, row};
}

// The uniform part of a tile: lane offset + add is the lane's access, at
// `base` and its row's head, if it is at most `cap`.
struct Tile {
    uint64_t base;
    uint32_t add, cap;
    uint32_t head, head_mask;  // bytes to the first boundary after base, unmasked
};

// A lane's access in a tile: lanes without one get the tile's last access
// (a line the tile reads anyway; with any head it lies in its row, whose
// edges are as long as the longest head).
struct TileAccess {
    uint32_t off;
    bool live;
};

// Only rows aligned to no more than 2 bytes have heads.
template <int DT, int VEC>
constexpr bool kRowHeads = sizeof(typename Elem<DT>::T) == 2 && VEC == 8;

// (Compiled in for fp32 too, unused, they made its inference forward 18%
// slower.)
template <bool HEADS>
__device__ __forceinline__ TileAccess tile_access(const Tile& t, const TileLane& lane) {
    const uint32_t u = lane.off + t.add;
    const uint32_t head = HEADS ? (t.head - lane.row) & t.head_mask : 0u;
    return {min(u, t.cap) + head, u <= t.cap};
}

// An access of 16 bytes needs only the alignment of an element; narrower
// ones are aligned to their width.
template <int DT, int VEC>
struct TileMem {
    using T = typename Elem<DT>::T;
    using mem = typename RawAccess<DT, VEC>::mem;
    static constexpr int kBytes = RawAccess<DT, VEC>::kBytes;
    typedef mem type __attribute__((aligned(kBytes == 16 ? sizeof(T) : kBytes)));
};

template <int DT, int VEC, int HINT>
__device__ __forceinline__ raw_t<DT, VEC> tile_load(const void* base, const Tile& t, uint32_t off) {
    using mem = typename TileMem<DT, VEC>::type;
    const mem* p = reinterpret_cast<const mem*>(static_cast<const char*>(base) + t.base + off);
    return static_cast<raw_t<DT, VEC>>(HINT == kStream ? __builtin_nontemporal_load(p) : *p);
}

template <int DT, int VEC>
__device__ __forceinline__ void tile_store(void* base, const Tile& t, uint32_t off,
                                           const float (&v)[VEC]) {
    using T = typename Elem<DT>::T;
    char* p = static_cast<char*>(base) + t.base + off;
    if constexpr (VEC == 1) {
        __builtin_nontemporal_store(static_cast<T>(v[0]), reinterpret_cast<T*>(p));
    } else {
        typedef T vt __attribute__((ext_vector_type(VEC)));
        typedef float vf __attribute__((ext_vector_type(VEC)));
        typedef vt vtu __attribute__((
            aligned(TileMem<DT, VEC>::kBytes == 16 ? sizeof(T) : TileMem<DT, VEC>::kBytes)));
        vf f;
#pragma unroll
        for (int k = 0; k < VEC; ++k) f[k] = v[k];
        __builtin_nontemporal_store(__builtin_convertvector(f, vt), reinterpret_cast<vtu*>(p));
    }
}

// ---------------------------------------------------------------- slices

// The tiles of slice p: group `sub` of the block (256 / lanes groups) takes
// tiles (j*P + p) * groups + sub for j = 0, 1, ...  Interleaving the slices
// keeps the whole chip's accesses moving through the rows together: a copy
// of 64 MiB by 512 blocks takes 22.1 us this way and 25.8 with contiguous
// slices.
//
// A walk steps through them with a few scalar operations per tile.
struct SliceTiles {
    uint32_t first, count;  // uniform per wave
    uint32_t end;           // j of the channel's last tile, if the slice has it (a slice
                            // without tiles loads tile 0, as j = 0)
    uint32_t origin;        // low bits of the address of the tensor the rows are aligned in
};

__device__ __forceinline__ SliceTiles slice_tiles(const TileGeom& g, uint32_t p,
                                                  const void* tensor) {
    const uint32_t groups = kThreads / g.lanes;
    const uint32_t sub = __builtin_amdgcn_readfirstlane(threadIdx.x / g.lanes);
    SliceTiles s;
    s.first = p * groups + sub;
    s.count = s.first < g.tiles ? (g.tiles - s.first + g.step - 1) / g.step : 0;
    const bool ends = s.count ? s.first + (s.count - 1) * g.step == g.tiles - 1 : g.tiles == 1;
    s.origin = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(tensor));
    s.end = ends ? (s.count ? s.count - 1 : 0) : ~0u;
    return s;
}

struct TileWalk {
    uint64_t base;  // of the tile's first row
    uint32_t at;    // byte offset of the tile in its row (0 in tiles of whole rows)
};

// At tile first + j * step (a slice without tiles: at tile 0).
__device__ __forceinline__ TileWalk walk_begin(const TileGeom& g, uint64_t chan,
                                               const SliceTiles& s, uint32_t j = 0) {
    const uint32_t q = s.count ? s.first + j * g.step : 0;
    TileWalk w;
    if (g.split_rows) {
        const uint32_t n = iabn_divmagic_div(q, g.per_div);
        w.base = chan + n * g.nstride;
        w.at = (q - n * g.per) * g.tile_bytes;
    } else {
        w.at = 0;
        w.base = chan + q * g.per * g.nstride;
    }
    return w;
}

// The same tiles for another phase.  Each phase forms its positions and its
// bounds again instead of keeping them from an earlier one, in more scalar
// registers than there are.
__device__ __forceinline__ SliceTiles slice_again(SliceTiles s) {
    asm volatile("" : "+s"(s.first), "+s"(s.count), "+s"(s.end));
    return s;
}

__device__ __forceinline__ void walk_next(const TileGeom& g, TileWalk& w) {
    w.base += g.step_base;
    w.at += g.step_at;
    if (w.at >= g.wrap_at) {
        w.base += g.nstride;
        w.at -= g.wrap_at;
    }
}

// The slice's j-th tile, where the walk is.
__device__ __forceinline__ Tile walk_tile(const TileGeom& g, const SliceTiles& s, const TileWalk& w,
                                          uint32_t j) {
    return {w.base, w.at, j == s.end ? g.cap_end : g.cap,
            0u - (s.origin + static_cast<uint32_t>(w.base)), g.head_mask};
}

// Edges: element i of a thread of slice p (i = 0, 1, ...: elements (i*P + p)
// * 256 + thread of the channel's), or one that is not live, at the
// channel's first element.
struct Edge {
    uint64_t at;
    bool live;
};

template <int EB>
__device__ __forceinline__ Edge edge_pos(const TileGeom& g, uint64_t chan, const SliceTiles& s,
                                         uint32_t p, uint32_t i) {
    const uint32_t e = (i * g.P + p) * kThreads + threadIdx.x;
    const uint32_t row = iabn_divmagic_div(e, g.edge_div);
    const uint64_t start = chan + row * g.nstride;
    const uint32_t head = (0u - (s.origin + static_cast<uint32_t>(start))) & g.head_mask;
    uint32_t at = (e - row * g.edge) * EB;
    if (at >= head) at += g.body_bytes;
    Edge t;
    t.live = e < g.edges;
    t.at = t.live ? start + at : chan;
    return t;
}

// Edge elements a thread keeps in registers; it reads the rest again.
constexpr int kEdges = 2;

__device__ __forceinline__ uint32_t edge_rounds(const TileGeom& g) {
    return (g.edges + g.P * kThreads - 1) / (g.P * kThreads);
}

template <int DT>
__device__ __forceinline__ typename Elem<DT>::T edge_load(const void* base, const Edge& t) {
    using T = typename Elem<DT>::T;
    return *reinterpret_cast<const T*>(static_cast<const char*>(base) + t.at);
}
template <int DT>
__device__ __forceinline__ void edge_store(void* base, const Edge& t, float v) {
    using T = typename Elem<DT>::T;
    *reinterpret_cast<T*>(static_cast<char*>(base) + t.at) = static_cast<T>(v);
}

// The block's channel and slice.
struct SliceId {
    uint32_t c, p;
};

__device__ __forceinline__ SliceId slice_id(const TileGeom& g) {
    uint32_t b = blockIdx.x;
    if (g.xcd_order) {
        const uint32_t n = gridDim.x, x = b % kXcds, j = b / kXcds;
        b = x * (n / kXcds) + min(x, n % kXcds) + j;
    }
    SliceId s;
    s.c = b / g.P;
    s.p = b - s.c * g.P;
    return s;
}

// ---------------------------------------------------------------- exchange
//
// The P blocks of a channel exchange their partial sums through the caller's
// workspace and then each writes its own slice from registers.
//
// A sum is published as 32-bit pieces, each stored twice in two 8-byte words
// beside 32 bits of the launch's key, and a reader takes a piece only where
// both words hold their half of the key and the same piece.  The words need
// no order among each other and no counter, so a sum travels in one store
// and one load (with a counter the blocks wait for their stores, for an
// atomic add, for the counter and then for the sums: 5 us instead of 2).
//
// No block relies on another one running at the same time.  A block waits a
// bounded time for the others' sums; if they have not all arrived it flags
// its slice as abandoned and exits, which frees its place for blocks that
// have not started.  Each block counts itself as finished once it needs
// nothing more of the exchange; the one that finishes last has all sums and
// all flags, so it writes the channel's statistics and, from memory, every
// slice that was abandoned.
//
// Nothing in the workspace needs to be set before a call: key and tag are
// the launch's own, and a finished count without the tag counts as zero.  A
// launch recorded in a graph runs again with the same key, so the last block
// clears the slots and the count (and the flags, where one was set).
//
// All words are accessed with agent-scope atomics, which go to the level
// that all XCDs share.

constexpr uint32_t kMaxPieces = 6;
constexpr uint32_t kSlotWords = 2 * kMaxPieces;  // at most, per slice
constexpr uint32_t kMaxSlicesOnChip = kWave;  // one lane per slice reads the sums
constexpr uint64_t kCountBits = 8;
constexpr uint64_t kCountMask = (uint64_t(1) << kCountBits) - 1;
constexpr uint64_t kTagShift = 2 * kCountBits;
constexpr uint64_t kTagBits = 64 - kTagShift;

// Longest wait for the other blocks, in polls; a poll is a round trip to
// memory, about 0.7 us, and a wait takes one to three when all blocks run.
constexpr uint32_t kPolls = 256;
// Compiled in for tests: the odd slices of a channel give up without waiting,
// and the last block leaves kAbandonMark in the flags of those it has written.
#ifdef IABN_TEST_ABANDON
constexpr bool kTestAbandon = true;
#else
constexpr bool kTestAbandon = false;
#endif
constexpr uint64_t kAbandonMark = ~uint64_t(0);  // no tag
// The channel's last block finds all sums in its first polls.  Only calls that
// share a workspace at the same time, which the interface forbids, can have
// overwritten them: its wait then ends too (in under a second), the results
// being as undefined as such calls' always are.
constexpr uint32_t kLastPolls = 1u << 20;

struct SliceArgs {
    uint64_t* workspace;
    uint64_t tag;  // nonzero, below 2^kTagBits
    uint64_t key;
};

// Workspace words of a channel with P > 1 slices.  The slots of all channels
// come first, then their flags, then their finished counts, apart from each
// other: an atomic add to a count keeps its cache line from everyone who
// polls it (with the counts beside the slots an exchange took 14 us).
constexpr uint64_t kCountWords = 3;  // per slice: room between the counts
constexpr uint64_t kSliceWords = kSlotWords + 1 + kCountWords;

struct SliceSync {
    uint64_t* done;  // see slice_open
    uint64_t* flag;  // per slice: the tag if abandoned
    uint64_t* slot;  // two words per piece and slice
    uint64_t tag, key;
    uint32_t P;
};

__device__ __forceinline__ SliceSync slice_sync(const SliceArgs& a, const TileGeom& g, uint32_t c) {
    const uint64_t P = g.P, slices = static_cast<uint64_t>(g.C) * P;
    SliceSync s;
    s.slot = a.workspace + c * P * kSlotWords;
    s.flag = a.workspace + slices * kSlotWords + c * P;
    s.done = a.workspace + slices * (kSlotWords + 1) + c * P * kCountWords;
    s.tag = a.tag;
    s.key = a.key;
    s.P = g.P;
    return s;
}

__device__ __forceinline__ uint64_t agent_load(const uint64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void agent_store(uint64_t* p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The finished count: tag | abandoned slices | finished blocks.  One thread of
// each block reads the word before its data loads and gives it this launch's
// tag, if it had not, any time before slice_finish.  (If the swap fails,
// another block of the launch has done it: the word is not cleared before
// this block has finished too.)
__device__ __forceinline__ void slice_open(const SliceSync& s, uint64_t seen) {
    if (seen >> kTagShift != s.tag)
        __hip_atomic_compare_exchange_strong(s.done, &seen, s.tag << kTagShift, __ATOMIC_RELAXED,
                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Counts the block as finished (one thread, after its last use of the other
// words) and returns the word as it is then.
__device__ __forceinline__ uint64_t slice_finish(const SliceSync& s, bool abandoned) {
    const uint64_t one = abandoned ? (uint64_t(1) << kCountBits) + 1 : 1;
    return one + __hip_atomic_fetch_add(s.done, one, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool slice_last(const SliceSync& s, uint64_t done) {
    return (done & kCountMask) == s.P;
}
__device__ __forceinline__ bool slice_any_abandoned(uint64_t done) {
    return ((done >> kCountBits) & kCountMask) != 0;
}

// One wave: publishes slice p's pieces (the same in every lane).
template <int NP>
__device__ __forceinline__ void slice_publish(const SliceSync& s, uint32_t p,
                                              const uint32_t (&piece)[NP]) {
    const uint32_t i = lane_id();
    uint32_t v = piece[0];
#pragma unroll
    for (int k = 1; k < NP; ++k) {
        v = i / 2 == k ? piece[k] : v;
        // Without this the selects become an indexed array, the array goes
        // to LDS, and every wave finds its place there with the help of the
        // dispatch packet, a read from host memory that took 15 us.
        opaque(v);
    }
    const uint32_t half = static_cast<uint32_t>((i & 1) ? s.key >> 32 : s.key);
    if (i < 2 * NP) agent_store(s.slot + 2 * NP * p + i, static_cast<uint64_t>(half) << 32 | v);
}

// One wave: lane q < P gets slice q's pieces (through `stage`, block-shared).
// Returns false if they have not all arrived after `limit` polls.  Adjacent
// lanes read adjacent words, so that a poll is a few requests: with a lane
// per slot, the blocks of a channel kept its few lines so busy that an
// exchange took 15 us.
template <int NP>
__device__ __forceinline__ bool slice_collect(const SliceSync& s, uint32_t (&piece)[NP],
                                              uint32_t* stage, uint32_t limit) {
    constexpr uint32_t kBatch = 4;
    const uint32_t words = 2 * NP * s.P;
    const uint32_t half = static_cast<uint32_t>((lane_id() & 1) ? s.key >> 32 : s.key);
    uint32_t polls = 0;
    for (uint32_t w0 = 0; w0 < words; w0 += kBatch * kWave) {
        while (true) {
            uint64_t w[kBatch];
#pragma unroll
            for (uint32_t t = 0; t < kBatch; ++t)
                w[t] = agent_load(s.slot + min(w0 + t * kWave + lane_id(), words - 2 + (lane_id() & 1)));
            bool ok = true;
#pragma unroll
            for (uint32_t t = 0; t < kBatch; ++t) {
                const uint32_t v = static_cast<uint32_t>(w[t]);
                ok = ok && (w[t] >> 32) == half && v == __shfl_xor(v, 1, kWave);
                const uint32_t at = w0 + t * kWave + lane_id();
                if (at < words && (at & 1) == 0) stage[at / 2] = v;
            }
            if (__all(ok)) break;
            if (++polls >= limit) return false;
            __builtin_amdgcn_s_sleep(1);
        }
    }
    // One wave's LDS operations run in order.
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    const uint32_t q = min(lane_id(), s.P - 1);
#pragma unroll
    for (int k = 0; k < NP; ++k) piece[k] = stage[NP * q + k];
    return true;
}

// One wave, after slice_publish: waits for all sums.  Returns false if the
// slice was abandoned: the block has finished then.  (`done`, lane 0: the
// word of slice_finish where the block has finished, else 0.)
template <int NP>
__device__ __forceinline__ bool slice_wait(const SliceSync& s, uint32_t p, uint64_t seen,
                                           uint32_t (&piece)[NP], uint32_t* stage, uint64_t& done) {
    done = 0;
    if (!(kTestAbandon && (p & 1)) && slice_collect(s, piece, stage, kPolls)) return true;
    if (lane_id() == 0) {
        agent_store(s.flag + p, s.tag);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        slice_open(s, seen);
        done = slice_finish(s, true);
    }
    if (!__any(lane_id() == 0 && slice_last(s, done))) return false;
    // The last one has nobody to leave its slice to, and needs to wait for
    // nobody: every other block has published its sums.
    return slice_collect(s, piece, stage, kLastPolls);
}

// The same wave, before it writes its part of the slice (a wait for the
// count behind those stores would wait for them too): counts the block as
// finished and, if it is the channel's last, clears the channel's words.
// Sets `rest` if slices were abandoned.
template <int NP>
__device__ __forceinline__ bool slice_done(const SliceSync& s, uint64_t seen, uint64_t done,
                                           bool& rest) {
    if (lane_id() == 0 && done == 0) {
        slice_open(s, seen);
        done = slice_finish(s, false);
    }
    rest = false;
    if (!__any(lane_id() == 0 && slice_last(s, done))) return false;
    for (uint32_t i = lane_id(); i < 2 * NP * s.P; i += kWave) agent_store(s.slot + i, 0);
    if (lane_id() == 0) agent_store(s.done, 0);
    rest = __any(lane_id() == 0 && slice_any_abandoned(done));
    return true;
}

// A block barrier for what is in LDS: stores to memory are not waited for.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// The last block, all threads: which slices were abandoned (left[q]); clears
// the flags.  (Stale flags hold another launch's tag, or none.)
__device__ __forceinline__ void slice_abandoned(const SliceSync& s, uint32_t own,
                                                uint32_t (&left)[kMaxSlicesOnChip]) {
    if (threadIdx.x < s.P) {
        const bool is_left = threadIdx.x != own && agent_load(s.flag + threadIdx.x) == s.tag;
        left[threadIdx.x] = is_left;
        agent_store(s.flag + threadIdx.x, kTestAbandon && is_left ? kAbandonMark : 0);
    }
    __syncthreads();
}

}  // namespace iabn_impl

// The C ABI of libiabn (include/iabn.h): argument validation on the host
// before any launch, the choice between the channel-resident and the
// streaming kernels, and the entry points themselves.

#include <stdarg.h>
#include <stdio.h>
#include <string.h>
#include <sys/random.h>
#include <time.h>
#include <unistd.h>

#include <atomic>
#include <cmath>
#include <mutex>

#include "launch.h"
#include "tile.h"

#define IABN_VERSION 10100

namespace iabn_impl {
namespace {

thread_local char g_last_error[256] = "";

int fail(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
int fail(int code, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_last_error, sizeof g_last_error, fmt, ap);
    va_end(ap);
    return code;
}

int ok() {
    g_last_error[0] = '\0';
    return IABN_OK;
}

constexpr int64_t kMaxChannelElems = (int64_t(1) << 31) - 1;
constexpr int64_t kMaxChannels = int64_t(1) << 20;
constexpr int64_t kMaxTotalElems = int64_t(1) << 46;
constexpr int64_t kTargetBlocks = 512;     // 2 blocks of 4 waves per CU on 256 CUs (measured best)
// The inference forward keeps no partial sums, so it chooses its slices
// freely: with fewer than kEvalManyBlocksBelow channels it cuts them for
// about kEvalTargetBlocks blocks (each thread moves a few accesses, and the
// chip holds many more waves): (8, 64, 256x256) fp16 25.2 us against 28.3,
// (32, 64, 112x112) 19.5 against 21.1, (8, 128, 128x128) 13.6 against 15.9;
// from 256 channels up the training passes' slicing is faster ((32, 256,
// 56x56) fp16 19.8 us against 21.5), and so it is for the checkpointing's
// recomputation on every shape measured.
constexpr int64_t kEvalTargetBlocks = 8192;
constexpr int64_t kEvalManyBlocksBelow = 256;

int64_t eval_target_blocks(int64_t C) {
    return C < kEvalManyBlocksBelow ? kEvalTargetBlocks : kTargetBlocks;
}
constexpr int64_t kMinSliceElems = 4096;   // at least 16 elements per thread
constexpr int64_t kMaxSlices = 1024;
constexpr int64_t kSliceAlign = 8;         // slices start on a 16-byte access of any dtype
constexpr int64_t kLineBytes = 128;        // L2 cache line

int elem_bytes(int dtype) { return dtype == IABN_F32 ? 4 : 2; }

bool valid_dtype(int dtype) { return dtype == IABN_F32 || dtype == IABN_F16 || dtype == IABN_BF16; }

// Slices per channel and slice length in elements; depends on the shape only.
struct Split {
    int64_t P;
    int64_t L;
};

Split split_channel(int64_t m, int64_t C, int64_t target_blocks = kTargetBlocks) {
    int64_t P = (target_blocks + C - 1) / C;
    const int64_t pmax_len = (m + kMinSliceElems - 1) / kMinSliceElems;
    if (P > pmax_len) P = pmax_len;
    if (P > kMaxSlices) P = kMaxSlices;
    if (P < 1) P = 1;
    int64_t L = (m + P - 1) / P;
    L = (L + kSliceAlign - 1) / kSliceAlign * kSliceAlign;
    P = (m + L - 1) / L;
    return {P, L};
}

// Validates the shape; `train` also needs N*HW >= 2.
int check_shape(int64_t N, int64_t C, int64_t HW, bool train) {
    if (N < 0 || C < 0 || HW < 0)
        return fail(IABN_ERR_SHAPE, "negative size N=%lld C=%lld HW=%lld", (long long)N,
                    (long long)C, (long long)HW);
    if (C > kMaxChannels) return fail(IABN_ERR_SHAPE, "C=%lld exceeds 2^20", (long long)C);
    if (N != 0 && HW > kMaxChannelElems / N)
        return fail(IABN_ERR_SHAPE, "N*HW exceeds 2^31-1");
    if (C != 0 && N * HW > kMaxTotalElems / C)
        return fail(IABN_ERR_SHAPE, "N*C*HW exceeds 2^46");
    if (train && C > 0 && N * HW < 2)
        return fail(IABN_ERR_SHAPE, "training needs N*HW >= 2 values per channel, got %lld",
                    (long long)(N * HW));
    return IABN_OK;
}

size_t workspace_bytes_for(int64_t N, int64_t C, int64_t HW) {
    if (C == 0 || N * HW == 0) return 0;
    const Split sp = split_channel(N * HW, C);
    return static_cast<size_t>(C) * static_cast<size_t>(sp.P) * kWaves * sizeof(Partial);
}

// ---------------------------------------------------------------- slice plan

struct SlicePlan {
    TileGeom g;
    int vec;  // elements per access
    int R;    // accesses per thread the kernel holds
    int64_t J;  // accesses per thread of a slice
    bool fine;  // backward, kBwdFromZ: every element's terms to double (slice_bwd.h)
};

// Rows of at least a cache line that only 2- or 4-byte accesses divide (or
// tensors aligned to no more) move in 16-byte accesses at element alignment
// (ragged rows, tile.h).
constexpr int64_t kRaggedMinRowBytes = kLineBytes;
// The fewest values of a channel that few-channel layers of ragged rows move
// in slices; smaller ones are one slice of a few narrow accesses per thread.
constexpr int64_t kRaggedMinChannel = 4096;

// Rows that 8-byte accesses divide do so only in channels larger than the
// registers of the largest narrow channel-resident block: (8, 256, 16644)
// fp16 forward 34.4 -> 33.5 us, backward 49.2 -> 42.7, (64, 64, 110x110) 58.6
// -> 44.7 and 86.8 -> 62.9.
constexpr int64_t kRaggedMinAccesses8 = 16384;

// Rows aligned to no more than 2 bytes whose accesses start at a 16-byte
// boundary (tile.h): of at least kHeadsMinRow elements, so that the edges
// stay few.  Forward / backward us, at the alignment of an element -> at the
// boundary: (8, 512, 65x65) fp16 20.9 / 30.3 -> 16.6 / 23.3, (16, 300, 33x33)
// fp16 13.9 / 20.9 -> 11.6 / 15.3; aligned to 4 bytes it gains nothing ((16,
// 300, 33x33) fp32 12.9 / 17.8 -> 13.2 / 18.6).
constexpr int64_t kHeadsMinRow = 512;

bool row_heads(int64_t HW, int eb, int vec) { return vec * eb == 2 && HW >= kHeadsMinRow; }

bool ragged_rows(int64_t N, int64_t HW, int eb, int vec) {
    if (HW * eb < kRaggedMinRowBytes) return false;
    return vec * eb <= 4 || (vec * eb == 8 && N * HW / vec > kRaggedMinAccesses8);
}

// The tiles of a layer for accesses of `vec` elements (tile.h) by groups of
// `lanes` threads.  False where a tile does not fit 32-bit byte offsets.
bool make_tiles(int64_t N, int64_t C, int64_t HW, int eb, int vec, int lanes, bool heads,
                TileGeom* g) {
    const int64_t ab = static_cast<int64_t>(vec) * eb, row = HW * eb, nstride = C * row;
    const int64_t limit = int64_t(1) << 30;
    // (With any head the accesses stay in the row.)
    const int64_t vrow = heads ? (HW - (vec - 1)) / vec : HW / vec, edge = HW - vrow * vec;
    if (vrow < 1 || row >= limit) return false;
    g->C = static_cast<uint32_t>(C);
    g->lanes = static_cast<uint32_t>(lanes);
    g->split_rows = vrow > lanes ? 1u : 0u;
    const int64_t per = g->split_rows ? (vrow + lanes - 1) / lanes : lanes / vrow;
    if (!g->split_rows && (per + 1) * nstride >= limit) return false;
    g->tiles = static_cast<uint32_t>(g->split_rows ? N * per : (N + per - 1) / per);
    g->per = static_cast<uint32_t>(per);
    g->per_div = iabn_divmagic_make(g->per);
    g->vrow = static_cast<uint32_t>(vrow);
    g->vrow_div = iabn_divmagic_make(g->vrow);
    const int64_t rows = g->split_rows ? 1 : per;  // of a tile
    const int64_t rows_end = g->split_rows || N % per == 0 ? rows : N % per;
    g->cap = static_cast<uint32_t>((rows - 1) * nstride + (vrow - 1) * ab);
    g->cap_end = static_cast<uint32_t>((rows_end - 1) * nstride + (vrow - 1) * ab);
    g->tile_bytes = static_cast<uint32_t>(lanes * ab);
    g->wrap_at = g->split_rows ? static_cast<uint32_t>(per * lanes * ab) : UINT32_MAX;
    g->row_bytes = static_cast<uint64_t>(row);
    g->nstride = static_cast<uint64_t>(nstride);
    g->head_mask = heads ? 15u : 0u;
    g->edge = static_cast<uint32_t>(edge);
    g->edge_div = iabn_divmagic_make(edge ? g->edge : 1u);
    g->edges = static_cast<uint32_t>(N * edge);
    g->body_bytes = static_cast<uint32_t>(vrow * ab);
    g->xcd_order = row % kLineBytes != 0 ? 1u : 0u;
    g->m = static_cast<double>(N) * static_cast<double>(HW);
    g->inv_m = 1.0 / g->m;
    return true;
}

// The tiles of 64 or 256 threads, whichever leave fewer of them without an
// access.
bool best_tiles(int64_t N, int64_t C, int64_t HW, int eb, int vec, bool heads, TileGeom* g) {
    TileGeom a, b;
    const bool ok64 = make_tiles(N, C, HW, eb, vec, 64, heads, &a);
    const bool ok256 = make_tiles(N, C, HW, eb, vec, kThreads, heads, &b);
    const int64_t slots64 = ok64 ? int64_t(a.tiles) * 64 : INT64_MAX;
    const int64_t slots256 = ok256 ? int64_t(b.tiles) * kThreads : INT64_MAX;
    if (ok64 || ok256) *g = slots64 < slots256 ? a : b;
    return ok64 || ok256;
}

// Cuts the channels into P slices.
void set_slices(TileGeom* g, int64_t P) {
    g->P = static_cast<uint32_t>(P);
    g->step = g->P * (kThreads / g->lanes);
    if (g->split_rows) {
        g->step_at = g->step % g->per * g->tile_bytes;
        g->step_base = g->step / g->per * g->nstride;
    } else {
        g->step_at = 0;
        g->step_base = static_cast<uint64_t>(g->step) * g->per * g->nstride;
    }
}

// Blocks of the slice-resident kernels that the chip holds at once: two per
// CU (their registers and LDS, slice_bwd.h).
constexpr int64_t kSliceBlocks = 2 * kCUs;
static_assert(kSliceWords * sizeof(uint64_t) <= kWaves * sizeof(Partial),
              "a slice's words fit where the streaming kernels keep its partials");

// Where the slice-resident kernels are the better choice.  Times are us,
// forward / backward, other kernels -> slice-resident, each in a graph; J is
// the accesses per thread of a slice.
//
// Against the streaming kernels' two launches.  One slice per channel needs
// no exchange: few-channel layers of up to kOneSliceMaxJ 16-byte accesses per
// thread ((2, 16, 8x8) fp32 4.9 / 4.5 -> 3.7 / 3.6, (1, 15, 11456) fp16 J = 6
// 6.6 / 6.8 -> 5.9 / 6.2, but J = 8 (2, 16, 64x64) fp32 5.7 / 6.5 -> 6.5 /
// 7.5), and of no more than kOneSliceRowJ times the accesses in a short row
// ((279, 2, 8) fp16 J = 2 6.4 / 6.2 -> 4.9 / 5.1, (273, 2, 16) J = 3 6.5 / 6.6
// -> 5.3 / 5.7, but (554, 9, 8) bf16 J = 3 7.1 / 7.2 -> 8.2 / 9.2).  Few small
// channels of narrow accesses stay on the streaming kernels, where the
// training entry points give the same bits as their two phases.
//
// More slices are worth their exchange where a second read is slow: the blocks
// more than fill the CUs once, and J is at least kSlicesMinJ ((32, 25, 4512)
// fp32 J = 8 12.4 / 15.0 -> 11.2 / 12.9, (10, 92, 4824) bf16 J = 5 backward
// 12.7 -> 11.7, but 8 blocks (300, 1, 108) fp32 J = 5 6.8 / 7.3 -> 7.8 / 7.9),
// on rows shorter than a line kSlicesShortRowsMinJ ((2698, 40, 48) fp16 J = 6
// 12.1 / 14.3 -> 12.3 / 15.5), or kManySlicesMinJ with more than kFewSlices,
// whose exchange takes longer ((1, 8, 512x512) fp32 J = 4 10.0 / 12.0 -> 12.2 /
// 12.2).  There is no upper bound for 16-byte accesses ((64, 64, 224x224) fp32,
// J = 392: 421 / 697 -> 395 / 652), except where the forward reads nearly
// everything twice and a third of the places stays empty ((8, 171, 260x260)
// fp16 J = 133, 342 blocks: 98.7 -> 107.7).  Narrower accesses are worth it in
// the backward only, on a full chip ((3895, 20, 60) fp16 J = 10 14.5 / 17.1 ->
// 14.9 / 16.8, (3055, 25, 52) J = 9 backward 16.4 -> 15.5, but (3233, 16, 52) J
// = 6 11.2 / 12.6 -> 12.2 / 12.5), and up to about twice the 16 they are held
// deep ((64, 64, 110x110) fp16 in 8-byte accesses J = 47 58.2 / 86.3 -> 77.8 /
// 108).
constexpr int64_t kOneSliceMaxJ = 6;
constexpr int64_t kOneSliceRowJ = 2;
constexpr int64_t kSlicesMinJ = 5;
constexpr int64_t kSlicesShortRowsMinJ = 7;
constexpr int64_t kFewSlices = 32;
constexpr int64_t kManySlicesMinJ = 16;
constexpr int64_t kLongSliceJ = 100;
constexpr int64_t kLongSliceMinBlocks = 352;
constexpr int64_t kSliceNarrowMinJBwd = 7;
constexpr int64_t kSliceNarrowMaxJ = 32;

// Ragged rows, which the streaming kernels move in narrower accesses (Jn of
// them per thread), take slices whatever their size ((1, 64, 513x513) fp16
// 31.7 / 44.1 -> 19.8 / 24.2), except: fewer than a batch of accesses under a
// long exchange (more than kSomeSlices slices and Jn <= 4: (612, 7, 124) fp16
// 8.1 / 8.7 -> 8.8 / 9.0; Jn = 8 (3, 18, 22326) fp32 9.7 / 11.2 -> 8.7 / 9.3);
// the forward of more than kFewSlices ((2, 3, 103486) fp16 Jn = 8 8.6 -> 9.9,
// (264, 1, 1201) fp16 Jn = 32 64 blocks 10.1 -> 10.8, (164, 1, 2377) fp32 Jn =
// 28 10.0 -> 10.9; but with more blocks than CUs (3428, 12, 99) fp16 Jn = 32
// 15.2 -> 13.1, (4, 7, 77177) fp32 Jn = 20 12.5 -> 12.2, (15, 12, 26572) fp16 J
// = 5 Jn = 10 13.1 -> 11.7); and with few channels one short slice with more
// edge elements than a thread keeps ((98, 81, 95) fp16 J = 5, the standard
// block's backward 8.9 -> 11.6).
constexpr int64_t kSomeSlices = 16;
constexpr int64_t kRaggedMinNarrow = 4;
constexpr int64_t kRaggedManyMinNarrow = 16;
constexpr int64_t kRaggedManyMinNarrowFewBlocks = 48;

int64_t edge_rounds_of(const TileGeom& g) {
    const int64_t per_round = int64_t(g.P) * kThreads;
    return (int64_t(g.edges) + per_round - 1) / per_round;
}

// ab: bytes of the streaming kernels' accesses.
bool slices_over_streaming(const SlicePlan& sl, int64_t N, int64_t C, int64_t HW, int eb, int ab,
                           bool ragged, bool backward) {
    const int64_t P = sl.g.P, J = sl.J, blocks = C * P;
    if (ragged) {
        if (C < kFusedMinChannels && N * HW <= kRaggedMinChannel) return false;
        if (P == 1)
            return C >= kFusedMinChannels || J > kOneSliceMaxJ || edge_rounds_of(sl.g) <= kEdges;
        const int64_t narrow = J * 16 / ab;
        if (P > kSomeSlices && narrow <= kRaggedMinNarrow) return false;
        if (backward || P <= kFewSlices) return true;
        return blocks > kCUs ? J >= kSlicesMinJ || narrow > kRaggedManyMinNarrow
                             : narrow > kRaggedManyMinNarrowFewBlocks;
    }
    if (ab != 16 && J > kSliceNarrowMaxJ) return false;
    if (P == 1) {
        if (C >= kFusedMinChannels) return true;
        return ab == 16 && J <= kOneSliceMaxJ && J <= kOneSliceRowJ * (HW * eb / 16);
    }
    if (ab == 16 && P > kFewSlices) return J >= kManySlicesMinJ;
    if (blocks <= kCUs) return false;
    if (ab == 16)
        return J >= (HW * eb >= kLineBytes ? kSlicesMinJ : kSlicesShortRowsMinJ) &&
               (backward || J <= kLongSliceJ || blocks >= kLongSliceMinBlocks);
    return backward && J >= kSliceNarrowMinJBwd;
}

// Ragged rows that the channel-resident kernels would move in `vchan` narrow
// accesses per channel, whose code is shorter.  Below kFusedMinChannels they
// are the better choice while a channel fits their registers ((1, 128, 4227)
// fp32 4.8 / 5.7 -> 5.4 / 6.2, two slices (8, 180, 33x33) fp32 7.3 / 8.9 -> 8.9
// / 10.2; but one slice (8, 180, 33x33) fp16 7.6 / 8.4 -> 6.8 / 7.5, three
// (23, 133, 937) fp16 11.9 / 13.8 -> 9.3 / 10.3), above only the smallest ((1,
// 853, 5554) bf16 7.6 / 10.3 -> 8.1 / 10.3, (10, 914, 503) fp16 11.3 / 13.2 ->
// 9.2 / 13.0, (8, 512, 65x65) 28.3 / 38.0 -> 16.7 / 23.2).  More edge elements
// than a thread keeps (rounds of them) change that: (98, 81, 95) fp16 9310
// accesses, three rounds 7.4 / 8.6 -> 8.4 / 10.1, (155, 211, 167) 25885, three
// 15.5 / 18.4 -> 13.6 / 16.2, (219, 750, 43) fp32 9417, three 23.4 / 30.4 ->
// 21.5 / 35.9, (250, 474, 69) bf16 17250, five 16.0 / 20.9 -> 18.1 / 25.5, (542,
// 559, 91) bf16 49322, seven 68.9 / 97.2 -> 50.8 / 81.9.  So do rows of few
// elements ((898, 283, 39) fp32 37.1 / 51.1 -> 50.1 / 67.7, (399, 244, 69) bf16
// backward 20.4 -> 23.3).
constexpr int64_t kRaggedMinRowFwd = 40;
constexpr int64_t kRaggedMinRowBwd = 72;
constexpr int64_t kRaggedOneSliceMinAccesses = 8192;
constexpr int64_t kRaggedSlicesMinAccesses = 20480;
constexpr int64_t kRaggedManyChannelsMinAccesses = 4096;
constexpr int64_t kRaggedEdgesMinAccesses = 8192;
constexpr int64_t kRaggedMaxEdgeRounds = 4;
constexpr int64_t kRaggedAnyEdgesMinAccesses = 32768;

bool slices_over_channels(const SlicePlan& sl, int64_t C, int64_t HW, int64_t vchan, int eb,
                          bool backward) {
    if (HW < (backward ? kRaggedMinRowBwd : kRaggedMinRowFwd)) return false;
    const int64_t rounds = edge_rounds_of(sl.g);
    if (vchan > kRaggedAnyEdgesMinAccesses) return true;
    if (C < kFusedMinChannels)
        return sl.g.P == 1 ? rounds <= 1 && vchan > kRaggedOneSliceMinAccesses
                           : rounds <= kRaggedMaxEdgeRounds && vchan > kRaggedSlicesMinAccesses;
    if (rounds <= kEdges) return vchan > kRaggedManyChannelsMinAccesses;
    return vchan > kRaggedEdgesMinAccesses && rounds <= kRaggedMaxEdgeRounds &&
           !(backward && eb == 4);
}

// The slice-resident kernels for a layer whose aligned accesses are `vec`
// elements wide (false: none are built for it).
bool plan_slice(int64_t N, int64_t C, int64_t HW, int eb, int vec, bool backward, SlicePlan* out) {
    const bool ragged = ragged_rows(N, HW, eb, vec);
    const bool heads = ragged && row_heads(HW, eb, vec);
    const int v = ragged ? 16 / eb : vec;
    const bool wide = v * eb == 16;
    if (!best_tiles(N, C, HW, eb, v, heads, &out->g)) return false;
    out->vec = v;
    TileGeom& g = out->g;
    const Split sp = split_channel(N * HW, C);
    const int64_t groups = kThreads / g.lanes;
    auto accesses = [&](int64_t P) { return (int64_t(g.tiles) + P * groups - 1) / (P * groups); };
    int64_t P = kSliceBlocks / C;
    if (P > sp.P) P = sp.P;
    if (P > kMaxSlicesOnChip) P = kMaxSlicesOnChip;
    if (P < 1 || accesses(1) <= kOneSliceMaxJ) P = 1;
    const int64_t J = out->J = accesses(P);
    set_slices(&g, P);
    const int* rungs = !wide ? kSliceNarrowRungs : backward ? kSliceBwdRungs : kSliceFwdRungs;
    const int n = !wide      ? int(sizeof kSliceNarrowRungs / sizeof(int))
                  : backward ? int(sizeof kSliceBwdRungs / sizeof(int))
                             : int(sizeof kSliceFwdRungs / sizeof(int));
    out->R = rungs[n - 1];
    for (int i = n - 1; i >= 0; --i)
        if (J <= rungs[i]) out->R = rungs[i];
    return true;
}

// The passes without a reduction by tiles (pointwise_kernel), or false where
// the general mapping is the better choice (us, before -> after).  The
// inference forward on ragged rows ((8, 256, 129x129) fp16 36.3 -> 31.1, (8,
// 512, 65x65) 19.0 -> 18.0, (16, 300, 33x33) fp32 12.5 -> 11.5).  The
// recomputation on ragged rows, from more than kPointRaggedMinNarrow of the
// general mapping's accesses per thread (143 -> 30.8, 73 -> 18.2, 24.8 ->
// 11.9; (1, 190, 1745) fp16 eight 3.5 -> 3.4, (1, 12, 630) bf16 one 2.7 ->
// 3.3), and of the other rows in 16-byte accesses, with long rows, fewer
// channels than kPointMaxChannels (each is then cut into slices or has a long
// one) and kPointMinJ accesses per thread ((8, 256, 128x128) fp16 30.8 -> 26.1,
// (8, 64, 256x256) 32.4 -> 25.6, (32, 256, 56x56) fp32 43.0 -> 36.3, (32, 60,
// 56x56) fp16 8.0 -> 7.8; but rows of 2704 bytes (11, 509, 1352) fp16 8.1 ->
// 8.8, of 1088 (69, 573, 544) bf16 19.5 -> 20.6, of 80 (2937, 409, 40) 73.1 ->
// 89.2; (3, 1008, 6168) 15.8 -> 16.4, (8, 1024, 64x64) 24.2 -> 25.0, (2, 16,
// 8x8) 2.1 -> 2.2).
constexpr int64_t kPointMaxChannels = 768;
constexpr int64_t kPointMinRowBytes = 6144;
constexpr int64_t kPointMinJ = 4;
constexpr int64_t kPointRaggedMinNarrow = 6;

bool plan_pointwise(int64_t N, int64_t C, int64_t HW, int eb, int vec, bool recompute,
                    SlicePlan* out) {
    const bool ragged = ragged_rows(N, HW, eb, vec);
    if (!ragged && (!recompute || vec * eb != 16 || C >= kPointMaxChannels ||
                    HW * eb < kPointMinRowBytes))
        return false;
    const bool heads = ragged && row_heads(HW, eb, vec);
    out->vec = 16 / eb;
    if (!best_tiles(N, C, HW, eb, out->vec, heads, &out->g)) return false;
    set_slices(&out->g,
               split_channel(N * HW, C, recompute ? kTargetBlocks : eval_target_blocks(C)).P);
    const int64_t tiles = out->g.tiles, step = out->g.step;
    return ragged ? !recompute || tiles * 16 > kPointRaggedMinNarrow * vec * eb * step
                  : tiles >= kPointMinJ * step;
}

// Workspace bytes a slice-resident launch uses.
size_t slice_workspace(const SlicePlan& p) {
    return p.g.P > 1 ? static_cast<size_t>(p.g.C) * p.g.P * kSliceWords * sizeof(uint64_t) : 0;
}

// Random bits, or where the system has none at hand the time and the process
// (std::random_device throws there, out of a C entry point).
uint64_t random_start() {
    uint64_t v = 0;
    if (getrandom(&v, sizeof v, GRND_NONBLOCK) == static_cast<ssize_t>(sizeof v)) return v;
    timespec t = {};
    clock_gettime(CLOCK_REALTIME, &t);
    return (static_cast<uint64_t>(t.tv_sec) * 1000000000u + static_cast<uint64_t>(t.tv_nsec)) *
               0x9e3779b97f4a7c15ULL ^
           static_cast<uint64_t>(getpid()) << 32;
}

// The tag and the key of one launch (tile.h): a count that is never 0 and not
// repeated for 2^48 launches, starting at a random place so that what an
// earlier process left in memory holds no tag of this one, and 64 bits that
// differ in both halves from launch to launch (2^64 over the golden ratio).
SliceArgs slice_args(void* workspace) {
    static std::atomic<uint64_t> next{random_start()};
    constexpr uint64_t mask = (uint64_t(1) << kTagBits) - 1;
    uint64_t n;
    do n = next.fetch_add(1, std::memory_order_relaxed);
    while ((n & mask) == 0);
    return {static_cast<uint64_t*>(workspace), n & mask, n * 0x9e3779b97f4a7c15ULL};
}

// The access geometry for `vec` elements per access.
Geom make_geom(int64_t N, int64_t C, int64_t HW, int dtype, int vec,
               int64_t target_blocks = kTargetBlocks) {
    const int64_t m = N * HW;
    const Split sp = split_channel(m, C, target_blocks);
    Geom g;
    g.C = static_cast<uint32_t>(C);
    g.P = static_cast<uint32_t>(sp.P);
    g.vrow = static_cast<uint32_t>(HW / vec);
    g.vchan = static_cast<uint32_t>(m / vec);
    g.lv = static_cast<uint32_t>(sp.L / vec);
    g.vec = static_cast<uint32_t>(vec);
    g.row_div = iabn_divmagic_make(g.vrow);
    g.nstride = static_cast<uint64_t>(C) * g.vrow;
    g.m = static_cast<double>(m);
    g.inv_m = 1.0 / g.m;
    g.xcd_order = (HW * elem_bytes(dtype)) % kLineBytes != 0 ? 1u : 0u;
    g.xcd_q = static_cast<uint32_t>(C / kXcds);
    g.xcd_r = static_cast<uint32_t>(C % kXcds);
    return g;
}

bool aligned_to(const void* p, uintptr_t bytes) {
    return p == nullptr || (reinterpret_cast<uintptr_t>(p) & (bytes - 1)) == 0;
}

// Elements per access: the widest of 16, 8, 4 (and 2 for 2-byte types)
// bytes that divides a row and to which every given tensor is aligned (an
// access never crosses a row; slices start on multiples of 8 elements, so
// every width divides them).  Null pointers are ignored.
int access_vec(int64_t HW, int dtype, const void* a, const void* b, const void* c) {
    const int eb = elem_bytes(dtype);
    for (int bytes = 16; bytes > eb; bytes /= 2) {
        const int v = bytes / eb;
        if (HW % v == 0 && aligned_to(a, bytes) && aligned_to(b, bytes) && aligned_to(c, bytes))
            return v;
    }
    return 1;
}

int check_workspace(int64_t N, int64_t C, int64_t HW, const void* ws, size_t bytes) {
    const size_t need = workspace_bytes_for(N, C, HW);
    if (need == 0) return IABN_OK;
    if (ws == nullptr) return fail(IABN_ERR_NULL, "workspace is NULL (%zu bytes needed)", need);
    if (bytes < need)
        return fail(IABN_ERR_WORKSPACE, "workspace has %zu bytes, %zu needed", bytes, need);
    if ((reinterpret_cast<uintptr_t>(ws) & 15u) != 0)
        return fail(IABN_ERR_WORKSPACE, "workspace is not 16-byte aligned");
    return IABN_OK;
}

int check_params(float eps, float slope) {
    if (!(eps > 0.f) || !std::isfinite(eps)) return fail(IABN_ERR_PARAM, "eps must be finite and > 0");
    if (!(slope > 0.f) || !std::isfinite(slope))
        return fail(IABN_ERR_PARAM, "slope must be finite and > 0 (the activation must be invertible)");
    return IABN_OK;
}

int launched(const char* what) {
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(IABN_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
    return ok();
}

int validate_common(int dtype, int64_t N, int64_t C, int64_t HW, bool train) {
    if (!valid_dtype(dtype)) return fail(IABN_ERR_DTYPE, "unknown dtype %d", dtype);
    return check_shape(N, C, HW, train);
}

bool empty(int64_t N, int64_t C, int64_t HW) { return C == 0 || N * HW == 0; }

// Which kernels a training pass takes: the channel-resident ones, the
// slice-resident ones, or the streaming ones.
enum class Route { kChannel, kSlice, kStream };

Route plan_route(int64_t N, int64_t C, int64_t HW, int dtype, const Geom& g, bool backward,
                 bool narrow_ok, FusedPlan* fp, SlicePlan* sl) {
    const int eb = elem_bytes(dtype), vec = static_cast<int>(g.vec);
    const bool ragged = ragged_rows(N, HW, eb, vec);
    const bool channel = plan_fused(C, g, eb, backward, narrow_ok, fp);
    const Route other = channel ? Route::kChannel : Route::kStream;
    if ((channel && !ragged) || !plan_slice(N, C, HW, eb, vec, backward, sl)) return other;
    sl->fine = channel;
    const bool slices =
        channel ? slices_over_channels(*sl, C, HW, g.vchan, eb, backward)
                : slices_over_streaming(*sl, N, C, HW, eb, vec * eb, ragged, backward);
    return slices ? Route::kSlice : other;
}

const char* fwd_name(int fm) {
    return fm == kFwdOut ? "standard forward" : fm == kFwdCkpt ? "checkpointing forward" : "forward";
}

// Training forward of the three arms (fm: kFwdInPlace, kFwdOut, kFwdCkpt).
// x is the input (kFwdInPlace: z on return; kFwdCkpt: xhat on return); out
// receives z for kFwdOut and kFwdCkpt.  Everything is validated before the
// first launch, so an error changes nothing.
// ws_if_used: the workspace is checked only where kernels that use one run
// (the channel-resident ones and one slice per channel use none); otherwise
// it must hold iabn_workspace_size bytes whichever kernels run.
int forward_train_impl(int fm, void* x, void* out, int dtype, const float* gamma,
                       const float* beta, float* running_mean, float* running_var,
                       float* save_mean, float* save_var, float eps, float momentum, float slope,
                       int64_t N, int64_t C, int64_t HW, void* workspace, size_t workspace_bytes,
                       void* stream, bool ws_if_used = false) {
    int rc = validate_common(dtype, N, C, HW, true);
    if (rc) return rc;
    if (empty(N, C, HW)) return ok();
    if (!x || !gamma || !beta || !running_mean || !running_var || !save_mean || !save_var ||
        (fm != kFwdInPlace && !out))
        return fail(IABN_ERR_NULL, "a tensor or parameter pointer is NULL");
    if ((rc = check_params(eps, slope))) return rc;
    if (!(momentum >= 0.f && momentum <= 1.f))
        return fail(IABN_ERR_PARAM, "momentum must lie in [0, 1]");
    const int vec = access_vec(HW, dtype, x, fm == kFwdInPlace ? nullptr : out, nullptr);
    const Geom g = make_geom(N, C, HW, dtype, vec);
    const FwdParams prm = {gamma,    beta, running_mean, running_var, save_mean, save_var,
                           fm == kFwdInPlace ? nullptr : out, eps, momentum, slope};
    const hipStream_t st = static_cast<hipStream_t>(stream);
    FusedPlan fp;
    SlicePlan sl;
    const Route route = plan_route(N, C, HW, dtype, g, false, fm == kFwdInPlace, &fp, &sl);
    const bool needs_ws =
        route == Route::kStream || (route == Route::kSlice && slice_workspace(sl) > 0);
    if ((needs_ws || !ws_if_used) &&
        (rc = check_workspace(N, C, HW, workspace, workspace_bytes)))
        return rc;
    if (route == Route::kSlice) {
        if (!launch_fwd_slice(dtype, sl.vec, fm, x, sl.g, sl.R, slice_args(workspace), prm, st))
            return fail(IABN_ERR_HIP, "no sliced %s kernel built for R=%d", fwd_name(fm), sl.R);
        return launched(fwd_name(fm));
    }
    if (route == Route::kChannel) {
        if (!launch_fwd_fused(dtype, fm, x, g, fp, prm, st))
            return fail(IABN_ERR_HIP, "no %s kernel built for T=%d R=%d", fwd_name(fm), fp.T, fp.R);
        return launched(fwd_name(fm));
    }
    Partial* part = static_cast<Partial*>(workspace);
    launch_fwd_stats(dtype, vec, static_cast<const void*>(x), g, part, st);
    if ((rc = launched("fwd_stats"))) return rc;
    launch_fwd_apply(dtype, vec, x, g, static_cast<const Partial*>(part), prm, true, fm, st);
    return launched(fwd_name(fm));
}

const char* bwd_name(int bm, bool ii) {
    return bm == kBwdFromXZ     ? "standard backward"
           : bm == kBwdFromXhat ? "checkpointing backward"
           : ii                 ? "backward (formulation II)"
                                : "backward";
}

// Backward of every formulation (bm, ii: see BwdSign).  u is z, x or xhat;
// zs is the stored z for kBwdFromXZ; dz_dx holds dz on entry, dx on return.
int backward_impl(int bm, bool ii, const void* u, const void* zs, void* dz_dx, int dtype,
                  const float* gamma, const float* beta, const float* save_mean,
                  const float* save_var, float* dgamma, float* dbeta, float eps, float slope,
                  int64_t N, int64_t C, int64_t HW, void* workspace, size_t workspace_bytes,
                  void* stream) {
    int rc = validate_common(dtype, N, C, HW, true);
    if (rc) return rc;
    if (empty(N, C, HW)) return ok();
    if (!u || !dz_dx || !gamma || !beta || !save_var || !dgamma || !dbeta ||
        (bm == kBwdFromXZ && (!zs || !save_mean)))
        return fail(IABN_ERR_NULL, "a tensor or parameter pointer is NULL");
    if ((rc = check_params(eps, slope))) return rc;
    if ((rc = check_workspace(N, C, HW, workspace, workspace_bytes))) return rc;
    const int vec = access_vec(HW, dtype, u, dz_dx, bm == kBwdFromXZ ? zs : nullptr);
    const Geom g = make_geom(N, C, HW, dtype, vec);
    const BwdParams prm = {gamma, beta, save_mean, save_var, dgamma, dbeta, eps, slope, ii ? 1 : 0};
    const hipStream_t st = static_cast<hipStream_t>(stream);
    FusedPlan fp;
    SlicePlan sl;
    const Route route = plan_route(N, C, HW, dtype, g, true, bm == kBwdFromZ, &fp, &sl);
    if (route == Route::kSlice) {
        if (!launch_bwd_slice(dtype, sl.vec, bm, sl.fine, u, zs, dz_dx, sl.g, sl.R,
                              slice_args(workspace), prm, st))
            return fail(IABN_ERR_HIP, "no sliced %s kernel built for R=%d", bwd_name(bm, ii), sl.R);
        return launched(bwd_name(bm, ii));
    }
    if (route == Route::kChannel) {
        if (!launch_bwd_fused(dtype, bm, u, zs, dz_dx, g, fp, prm, st))
            return fail(IABN_ERR_HIP, "no %s kernel built for T=%d R=%d", bwd_name(bm, ii), fp.T, fp.R);
        return launched(bwd_name(bm, ii));
    }
    Partial* part = static_cast<Partial*>(workspace);
    launch_bwd_reduce(dtype, vec, u, zs, static_cast<const void*>(dz_dx), g, prm, bm, part, st);
    if ((rc = launched("bwd_reduce"))) return rc;
    launch_bwd_apply(dtype, vec, u, zs, dz_dx, g, static_cast<const Partial*>(part), prm, bm, st);
    return launched(bwd_name(bm, ii));
}

// ---------------------------------------------------------------- static scratch

// The scratch of iabn_forward_train_noalloc: the streaming kernels' partial
// results and the slice-resident kernels' exchange, in a file-scope device
// array instead of a caller's workspace.
// Each device holds its own copy (zero-initialised when the library's code
// object is loaded on it) until the process ends.  Its size bounds the
// partials of one call: C * P slices * 4 waves * 32 bytes, at most 765
// slices (C = 255, P = 3) where the forward takes the streaming kernels,
// about 96 KiB; at most kSliceBlocks slices of kSliceWords words, 64 KiB, where
// it takes the slice-resident ones.  Nothing in it needs to start at zero:
// every partial a call reads was written by the same call.
constexpr size_t kScratchBytes = size_t(128) << 10;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

// The device address of `scratch` on each device (null until first use),
// taken with that device current; host code uses these, never `scratch`.
constexpr int kMaxDevices = 64;
void* g_scratch_addr[kMaxDevices];
std::mutex g_scratch_mutex;

int scratch_address(void** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(IABN_ERR_HIP, "hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices)
        return fail(IABN_ERR_HIP, "device %d: the scratch table holds %d devices", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_addr[dev] == nullptr) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || p == nullptr)
            return fail(IABN_ERR_HIP, "hipGetSymbolAddress(scratch) on device %d: %s", dev,
                        hipGetErrorString(e));
        g_scratch_addr[dev] = p;
    }
    *out = g_scratch_addr[dev];
    return IABN_OK;
}

}  // namespace
}  // namespace iabn_impl

using namespace iabn_impl;

// ---------------------------------------------------------------- C ABI

extern "C" {

int iabn_version(void) { return IABN_VERSION; }

const char* iabn_status_string(int status) {
    switch (status) {
        case IABN_OK: return "IABN_OK";
        case IABN_ERR_NULL: return "IABN_ERR_NULL: a required pointer is NULL";
        case IABN_ERR_SHAPE: return "IABN_ERR_SHAPE: invalid tensor shape";
        case IABN_ERR_PARAM: return "IABN_ERR_PARAM: eps, momentum or slope out of range";
        case IABN_ERR_DTYPE: return "IABN_ERR_DTYPE: unknown storage type";
        case IABN_ERR_WORKSPACE: return "IABN_ERR_WORKSPACE: workspace too small or misaligned";
        case IABN_ERR_HIP: return "IABN_ERR_HIP: the HIP runtime rejected a launch";
        default: return "unknown iabn status";
    }
}

const char* iabn_last_error(void) { return g_last_error; }

size_t iabn_workspace_size(int64_t N, int64_t C, int64_t HW, int dtype) {
    if (!valid_dtype(dtype)) return 0;
    if (check_shape(N, C, HW, false) != IABN_OK) return 0;
    return workspace_bytes_for(N, C, HW);
}

int iabn_plan(int op, int dtype, int64_t N, int64_t C, int64_t HW, iabn_plan_t* plan) {
    if (plan == nullptr) return fail(IABN_ERR_NULL, "plan is NULL");
    if (op < IABN_OP_FORWARD_TRAIN || op > IABN_OP_CKPT_RECOMPUTE)
        return fail(IABN_ERR_PARAM, "unknown op %d", op);
    const bool train = op != IABN_OP_FORWARD_EVAL && op != IABN_OP_CKPT_RECOMPUTE;
    int rc = validate_common(dtype, N, C, HW, train);
    if (rc) return rc;
    memset(plan, 0, sizeof *plan);
    if (empty(N, C, HW)) return ok();
    // The same choices as the entry points make, on aligned tensors.
    const int vec = access_vec(HW, dtype, nullptr, nullptr, nullptr);
    const Geom g = make_geom(N, C, HW, dtype, vec,
                             op == IABN_OP_FORWARD_EVAL ? eval_target_blocks(C) : kTargetBlocks);
    const int eb = elem_bytes(dtype);
    const bool backward =
        op == IABN_OP_BACKWARD || op == IABN_OP_STD_BACKWARD || op == IABN_OP_CKPT_BACKWARD;
    const bool narrow_ok = op == IABN_OP_FORWARD_TRAIN || op == IABN_OP_BACKWARD;
    plan->access_bytes = vec * eb;
    plan->xcd_order = static_cast<int>(g.xcd_order);
    FusedPlan fp;
    SlicePlan sl;
    const Route route =
        train ? plan_route(N, C, HW, dtype, g, backward, narrow_ok, &fp, &sl) : Route::kStream;
    if (route == Route::kChannel) {
        const int64_t past = static_cast<int64_t>(g.vchan) - static_cast<int64_t>(fp.T) * fp.R;
        const int64_t past_per_thread = past > 0 ? (past + fp.T - 1) / fp.T : 0;
        const int64_t lds = fused_lds_accesses(fp.T, backward, op == IABN_OP_STD_BACKWARD);
        plan->channel_resident = 1;
        plan->threads = fp.T * fp.cpb;
        plan->reg_accesses = fp.R;
        plan->lds_accesses = static_cast<int>(past_per_thread < lds ? past_per_thread : lds);
        plan->strips = fused_strips(g, fp, vec * eb == 16) ? 1 : 0;
        plan->blocks = C / fp.cpb;
        plan->channels_per_block = fp.cpb;
    } else {
        plan->threads = kThreads;
        plan->blocks = C * static_cast<int64_t>(route == Route::kSlice ? sl.g.P : g.P);
        if (route == Route::kSlice) {
            const int lds = slice_lds_accesses(sl.R, sl.vec * eb == 16, backward);
            const int64_t past = sl.J - (sl.R - lds);
            plan->access_bytes = sl.vec * eb;
            plan->reg_accesses = sl.R - lds;
            plan->lds_accesses = static_cast<int>(past < 0 ? 0 : past < lds ? past : lds);
        }
        if (!train && plan_pointwise(N, C, HW, eb, vec, op == IABN_OP_CKPT_RECOMPUTE, &sl))
            plan->access_bytes = sl.vec * eb;
    }
    return ok();
}

int iabn_forward_stats(const void* x, int dtype, int64_t N, int64_t C, int64_t HW,
                       void* workspace, size_t workspace_bytes, void* stream) {
    int rc = validate_common(dtype, N, C, HW, true);
    if (rc) return rc;
    if (empty(N, C, HW)) return ok();
    if (x == nullptr) return fail(IABN_ERR_NULL, "x is NULL");
    if ((rc = check_workspace(N, C, HW, workspace, workspace_bytes))) return rc;
    const int vec = access_vec(HW, dtype, x, nullptr, nullptr);
    const Geom g = make_geom(N, C, HW, dtype, vec);
    launch_fwd_stats(dtype, vec, x, g, static_cast<Partial*>(workspace),
                     static_cast<hipStream_t>(stream));
    return launched("fwd_stats");
}

int iabn_forward_apply(void* x_z, int dtype, const float* gamma, const float* beta,
                       float* running_mean, float* running_var, float* save_mean,
                       float* save_var, float eps, float momentum, float slope, int64_t N,
                       int64_t C, int64_t HW, void* workspace, size_t workspace_bytes,
                       void* stream) {
    int rc = validate_common(dtype, N, C, HW, true);
    if (rc) return rc;
    if (empty(N, C, HW)) return ok();
    if (!x_z || !gamma || !beta || !running_mean || !running_var || !save_mean || !save_var)
        return fail(IABN_ERR_NULL, "a tensor or parameter pointer is NULL");
    if ((rc = check_params(eps, slope))) return rc;
    if (!(momentum >= 0.f && momentum <= 1.f))
        return fail(IABN_ERR_PARAM, "momentum must lie in [0, 1]");
    if ((rc = check_workspace(N, C, HW, workspace, workspace_bytes))) return rc;
    const int vec = access_vec(HW, dtype, x_z, nullptr, nullptr);
    const Geom g = make_geom(N, C, HW, dtype, vec);
    const FwdParams prm = {gamma, beta, running_mean, running_var, save_mean, save_var,
                           nullptr, eps, momentum, slope};
    launch_fwd_apply(dtype, vec, x_z, g, static_cast<const Partial*>(workspace), prm, true,
                     kFwdInPlace, static_cast<hipStream_t>(stream));
    return launched("fwd_apply");
}

int iabn_forward_train(void* x_z, int dtype, const float* gamma, const float* beta,
                       float* running_mean, float* running_var, float* save_mean,
                       float* save_var, float eps, float momentum, float slope, int64_t N,
                       int64_t C, int64_t HW, void* workspace, size_t workspace_bytes,
                       void* stream) {
    return forward_train_impl(kFwdInPlace, x_z, nullptr, dtype, gamma, beta, running_mean,
                              running_var, save_mean, save_var, eps, momentum, slope, N, C, HW,
                              workspace, workspace_bytes, stream);
}

int iabn_forward_train_noalloc(void* x_z, int dtype, const float* gamma, const float* beta,
                               float* running_mean, float* running_var, float* save_mean,
                               float* save_var, float eps, float momentum, float slope, int64_t N,
                               int64_t C, int64_t HW, void* stream) {
    int rc = validate_common(dtype, N, C, HW, true);
    if (rc) return rc;
    if (empty(N, C, HW)) return ok();
    const int vec = access_vec(HW, dtype, x_z, nullptr, nullptr);
    FusedPlan fp;
    SlicePlan sl;
    const Route route =
        plan_route(N, C, HW, dtype, make_geom(N, C, HW, dtype, vec), false, true, &fp, &sl);
    const size_t need = route == Route::kChannel ? 0
                        : route == Route::kSlice ? slice_workspace(sl)
                                                 : workspace_bytes_for(N, C, HW);
    if (need > kScratchBytes)
        return fail(IABN_ERR_WORKSPACE,
                    "this shape needs %zu bytes of scratch, more than the %zu the library "
                    "holds per device",
                    need, kScratchBytes);
    void* ws = nullptr;
    if ((rc = scratch_address(&ws))) return rc;
    return forward_train_impl(kFwdInPlace, x_z, nullptr, dtype, gamma, beta, running_mean,
                              running_var, save_mean, save_var, eps, momentum, slope, N, C, HW, ws,
                              kScratchBytes, stream, true);
}

int iabn_forward_eval(void* x_z, int dtype, const float* gamma, const float* beta,
                      const float* running_mean, const float* running_var, float eps,
                      float slope, int64_t N, int64_t C, int64_t HW, void* stream) {
    int rc = validate_common(dtype, N, C, HW, false);
    if (rc) return rc;
    if (empty(N, C, HW)) return ok();
    if (!x_z || !gamma || !beta || !running_mean || !running_var)
        return fail(IABN_ERR_NULL, "a tensor or parameter pointer is NULL");
    if ((rc = check_params(eps, slope))) return rc;
    const int vec = access_vec(HW, dtype, x_z, nullptr, nullptr);
    const Geom g = make_geom(N, C, HW, dtype, vec, eval_target_blocks(C));
    const FwdParams prm = {gamma, beta, const_cast<float*>(running_mean),
                           const_cast<float*>(running_var), nullptr, nullptr, nullptr, eps, 0.f,
                           slope};
    SlicePlan pw;
    if (plan_pointwise(N, C, HW, elem_bytes(dtype), vec, false, &pw))
        launch_pointwise(dtype, x_z, x_z, pw.g, prm, false, static_cast<hipStream_t>(stream));
    else
        launch_fwd_apply(dtype, vec, x_z, g, static_cast<const Partial*>(nullptr), prm, false,
                         kFwdInPlace, static_cast<hipStream_t>(stream));
    return launched("fwd_eval");
}

int iabn_backward_reduce(const void* z, const void* dz, int dtype, const float* gamma,
                         const float* beta, float slope, int64_t N, int64_t C, int64_t HW,
                         void* workspace, size_t workspace_bytes, void* stream) {
    int rc = validate_common(dtype, N, C, HW, true);
    if (rc) return rc;
    if (empty(N, C, HW)) return ok();
    if (!z || !dz || !gamma || !beta)
        return fail(IABN_ERR_NULL, "a tensor or parameter pointer is NULL");
    if (!(slope > 0.f) || !std::isfinite(slope))
        return fail(IABN_ERR_PARAM, "slope must be finite and > 0 (the activation must be invertible)");
    if ((rc = check_workspace(N, C, HW, workspace, workspace_bytes))) return rc;
    const int vec = access_vec(HW, dtype, z, dz, nullptr);
    const Geom g = make_geom(N, C, HW, dtype, vec);
    const BwdParams prm = {gamma, beta, nullptr, nullptr, nullptr, nullptr, 1.f, slope, 0};
    launch_bwd_reduce(dtype, vec, z, static_cast<const void*>(nullptr), dz, g, prm, kBwdFromZ,
                      static_cast<Partial*>(workspace), static_cast<hipStream_t>(stream));
    return launched("bwd_reduce");
}

int iabn_backward_apply(const void* z, void* dz_dx, int dtype, const float* gamma,
                        const float* beta, const float* save_var, float* dgamma, float* dbeta,
                        float eps, float slope, int64_t N, int64_t C, int64_t HW,
                        void* workspace, size_t workspace_bytes, void* stream) {
    int rc = validate_common(dtype, N, C, HW, true);
    if (rc) return rc;
    if (empty(N, C, HW)) return ok();
    if (!z || !dz_dx || !gamma || !beta || !save_var || !dgamma || !dbeta)
        return fail(IABN_ERR_NULL, "a tensor or parameter pointer is NULL");
    if ((rc = check_params(eps, slope))) return rc;
    if ((rc = check_workspace(N, C, HW, workspace, workspace_bytes))) return rc;
    const int vec = access_vec(HW, dtype, z, dz_dx, nullptr);
    const Geom g = make_geom(N, C, HW, dtype, vec);
    const BwdParams prm = {gamma, beta, nullptr, save_var, dgamma, dbeta, eps, slope, 0};
    launch_bwd_apply(dtype, vec, z, static_cast<const void*>(nullptr), dz_dx, g,
                     static_cast<const Partial*>(workspace), prm, kBwdFromZ,
                     static_cast<hipStream_t>(stream));
    return launched("bwd_apply");
}

int iabn_backward(const void* z, void* dz_dx, int dtype, const float* gamma, const float* beta,
                  const float* save_var, float* dgamma, float* dbeta, float eps, float slope,
                  int64_t N, int64_t C, int64_t HW, void* workspace, size_t workspace_bytes,
                  void* stream) {
    return backward_impl(kBwdFromZ, false, z, nullptr, dz_dx, dtype, gamma, beta, nullptr,
                         save_var, dgamma, dbeta, eps, slope, N, C, HW, workspace,
                         workspace_bytes, stream);
}

int iabn_backward_ii(const void* z, void* dz_dx, int dtype, const float* gamma,
                     const float* beta, const float* save_var, float* dgamma, float* dbeta,
                     float eps, float slope, int64_t N, int64_t C, int64_t HW, void* workspace,
                     size_t workspace_bytes, void* stream) {
    return backward_impl(kBwdFromZ, true, z, nullptr, dz_dx, dtype, gamma, beta, nullptr,
                         save_var, dgamma, dbeta, eps, slope, N, C, HW, workspace,
                         workspace_bytes, stream);
}

int iabn_std_forward_train(const void* x, void* z, int dtype, const float* gamma,
                           const float* beta, float* running_mean, float* running_var,
                           float* save_mean, float* save_var, float eps, float momentum,
                           float slope, int64_t N, int64_t C, int64_t HW, void* workspace,
                           size_t workspace_bytes, void* stream) {
    return forward_train_impl(kFwdOut, const_cast<void*>(x), z, dtype, gamma, beta, running_mean,
                              running_var, save_mean, save_var, eps, momentum, slope, N, C, HW,
                              workspace, workspace_bytes, stream);
}

int iabn_std_backward(const void* x, const void* z, void* dz_dx, int dtype, const float* gamma,
                      const float* beta, const float* save_mean, const float* save_var,
                      float* dgamma, float* dbeta, float eps, float slope, int64_t N, int64_t C,
                      int64_t HW, void* workspace, size_t workspace_bytes, void* stream) {
    return backward_impl(kBwdFromXZ, false, x, z, dz_dx, dtype, gamma, beta, save_mean, save_var,
                         dgamma, dbeta, eps, slope, N, C, HW, workspace, workspace_bytes, stream);
}

int iabn_ckpt_forward_train(void* x_xhat, void* z, int dtype, const float* gamma,
                            const float* beta, float* running_mean, float* running_var,
                            float* save_mean, float* save_var, float eps, float momentum,
                            float slope, int64_t N, int64_t C, int64_t HW, void* workspace,
                            size_t workspace_bytes, void* stream) {
    return forward_train_impl(kFwdCkpt, x_xhat, z, dtype, gamma, beta, running_mean, running_var,
                              save_mean, save_var, eps, momentum, slope, N, C, HW, workspace,
                              workspace_bytes, stream);
}

int iabn_ckpt_recompute(const void* xhat, void* z, int dtype, const float* gamma,
                        const float* beta, float slope, int64_t N, int64_t C, int64_t HW,
                        void* stream) {
    int rc = validate_common(dtype, N, C, HW, false);
    if (rc) return rc;
    if (empty(N, C, HW)) return ok();
    if (!xhat || !z || !gamma || !beta)
        return fail(IABN_ERR_NULL, "a tensor or parameter pointer is NULL");
    if ((rc = check_params(1.f, slope))) return rc;
    const int vec = access_vec(HW, dtype, xhat, z, nullptr);
    SlicePlan pw;
    if (plan_pointwise(N, C, HW, elem_bytes(dtype), vec, true, &pw)) {
        const FwdParams prm = {gamma, beta, nullptr, nullptr, nullptr, nullptr, z, 1.f, 0.f, slope};
        launch_pointwise(dtype, xhat, z, pw.g, prm, true, static_cast<hipStream_t>(stream));
    } else {
        const Geom g = make_geom(N, C, HW, dtype, vec);
        launch_recompute(dtype, vec, xhat, z, g, gamma, beta, slope, static_cast<hipStream_t>(stream));
    }
    return launched("recompute");
}

int iabn_ckpt_backward(const void* xhat, void* dz_dx, int dtype, const float* gamma,
                       const float* beta, const float* save_var, float* dgamma, float* dbeta,
                       float eps, float slope, int64_t N, int64_t C, int64_t HW,
                       void* workspace, size_t workspace_bytes, void* stream) {
    return backward_impl(kBwdFromXhat, false, xhat, nullptr, dz_dx, dtype, gamma, beta, nullptr,
                         save_var, dgamma, dbeta, eps, slope, N, C, HW, workspace,
                         workspace_bytes, stream);
}

}  // extern "C"

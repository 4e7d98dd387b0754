// The slice-resident training forward: each channel is cut into P slices,
// one 256-thread block holds a slice in registers (and LDS) from the
// statistics to the apply, and the blocks of a channel exchange their
// partial sums in between (tile.h), so x crosses HBM once in and the outputs
// once out where the streaming kernels read x twice and are two launches.
// Used where a channel does not get a block of its own (few channels) and for
// ragged rows; what a slice does not hold is read again.
//
// Measured (forward us, before: two streaming passes, or narrow accesses):
// (32, 64, 112x112) fp16 27.0 -> 23.9, (8, 64, 256x256) 33.5 -> 27.3 (2 b per
// element at 4.9 TB/s), (8, 20, 224x224) bf16 15.0 -> 13.1, (8, 256, 129x129)
// fp16 107 -> 30.8, (8, 512, 65x65) 28.0 -> 16.3, (2, 16, 8x8) fp32 5.3 -> 4.1.
// With the exchange left out (a timing copy) the first two take 3 us less: 2
// for the sums to travel, the rest for filling and draining the memory system
// around it.  The code of a phase must
// stay short: with ragged rows' left-over elements in the unrolled loops the
// kernel was 14000 instructions, and fetching them cost 4 us a call.

#pragma once

#include "launch.h"
#include "tile.h"

namespace iabn_impl {
namespace {

// Per-channel constants of the apply phase (as in fused_fwd.hip).
struct ApplyK {
    float mean_hi, scale, bshift, slope;
    float gamma, beta;
    void* out;
};

// The outputs of one value: z, or xhat (and z in zv) for kFwdCkpt.
template <int DT, int FM, bool SMALL_SLOPE>
__device__ __forceinline__ float out_of(float x, const ApplyK& k, float& zv) {
    const float y = fmaf(x - k.mean_hi, k.scale, k.bshift);
    if constexpr (FM == kFwdCkpt) {
        const float xhat = storage_round<DT>(y);
        zv = leaky<SMALL_SLOPE>(fmaf(xhat, k.gamma, k.beta), k.slope);
        return xhat;
    } else {
        return leaky<SMALL_SLOPE>(y, k.slope);
    }
}

template <int DT, int VEC, int FM, bool SMALL_SLOPE>
__device__ __forceinline__ void emit(void* __restrict__ xz, const Tile& t, uint32_t off,
                                     raw_t<DT, VEC> raw, const ApplyK& k) {
    float v[VEC], z[VEC];
    unpack<DT, VEC>(raw, v);
#pragma unroll
    for (int e = 0; e < VEC; ++e) v[e] = out_of<DT, FM, SMALL_SLOPE>(v[e], k, z[e]);
    tile_store<DT, VEC>(FM == kFwdOut ? k.out : xz, t, off, v);
    if constexpr (FM == kFwdCkpt) tile_store<DT, VEC>(k.out, t, off, z);
}

template <int DT, int FM, bool SMALL_SLOPE>
__device__ __forceinline__ void emit_edge(void* __restrict__ xz, const Edge& t, float x,
                                          const ApplyK& k) {
    float z;
    const float v = out_of<DT, FM, SMALL_SLOPE>(x, k, z);
    edge_store<DT>(FM == kFwdOut ? k.out : xz, t, v);
    if constexpr (FM == kFwdCkpt) edge_store<DT>(k.out, t, z);
}

// Outputs of the slice's accesses from j0 on and edge elements from i0 on,
// read from memory.
constexpr int kRestU = 4;  // accesses in flight per thread past the resident ones

template <int DT, int VEC, int FM, bool SMALL_SLOPE>
__device__ __forceinline__ void apply_rest(void* __restrict__ xz, const TileGeom& g, uint64_t chan,
                                           const SliceTiles& s, const TileLane& lane, uint32_t j0,
                                           uint32_t p, uint32_t i0, const ApplyK& k) {
    constexpr int EB = static_cast<int>(sizeof(typename Elem<DT>::T));
    for (uint32_t i = i0; i < edge_rounds(g); ++i) {
        const Edge t = edge_pos<EB>(g, chan, s, p, i);
        if (t.live)
            emit_edge<DT, FM, SMALL_SLOPE>(xz, t, static_cast<float>(edge_load<DT>(xz, t)), k);
    }
    if (j0 >= s.count) return;
    TileWalk w = walk_begin(g, chan, s, j0);
    for (uint32_t j = j0; j < s.count; j += kRestU) {
        raw_t<DT, VEC> r[kRestU];
        TileWalk wl = w;
#pragma unroll
        for (int q = 0; q < kRestU; ++q) {
            const Tile t = walk_tile(g, s, wl, min(j + q, s.count - 1));
            r[q] = tile_load<DT, VEC, kStream>(xz, t, tile_access<kRowHeads<DT, VEC>>(t, lane).off);
            if (j + q + 1 < s.count) walk_next(g, wl);
        }
        sched_fence();
#pragma unroll
        for (int q = 0; q < kRestU; ++q) {
            if (j + q < s.count) {
                const Tile t = walk_tile(g, s, w, j + q);
                const TileAccess a = tile_access<kRowHeads<DT, VEC>>(t, lane);
                if (a.live) emit<DT, VEC, FM, SMALL_SLOPE>(xz, t, a.off, r[q], k);
            }
            walk_next(g, w);
            sched_fence();
        }
    }
}

template <int DT, int VEC, int R, int S, int FM, bool SMALL_SLOPE>
__device__ __forceinline__ void apply_all(void* __restrict__ xz, const TileGeom& g, uint64_t chan,
                                          const SliceTiles& s, const TileLane& lane,
                                          const raw_t<DT, VEC> (&keep)[R],
                                          const raw_t<DT, VEC> (&lx)[S > 0 ? S : 1][kThreads],
                                          const float (&edges)[kEdges], uint32_t p,
                                          const ApplyK& k) {
    constexpr int EB = static_cast<int>(sizeof(typename Elem<DT>::T));
    if (g.edges) {
#pragma unroll
        for (int i = 0; i < kEdges; ++i) {
            const Edge t = edge_pos<EB>(g, chan, s, p, i);
            if (t.live) emit_edge<DT, FM, SMALL_SLOPE>(xz, t, edges[i], k);
        }
    }
    TileWalk w = walk_begin(g, chan, s);
#pragma unroll
    for (int j = 0; j < R; ++j) {
        if (j < s.count) {
            const Tile t = walk_tile(g, s, w, j);
            const TileAccess a = tile_access<kRowHeads<DT, VEC>>(t, lane);
            if (a.live) emit<DT, VEC, FM, SMALL_SLOPE>(xz, t, a.off, keep[j], k);
        }
        walk_next(g, w);
        sched_fence();
    }
    if constexpr (S > 0) {
#pragma unroll 1
        for (uint32_t j = R; j < min(s.count, uint32_t(R + S)); ++j) {
            const Tile t = walk_tile(g, s, w, j);
            const TileAccess a = tile_access<kRowHeads<DT, VEC>>(t, lane);
            if (a.live) emit<DT, VEC, FM, SMALL_SLOPE>(xz, t, a.off, lx[j - R][threadIdx.x], k);
            walk_next(g, w);
        }
    }
    apply_rest<DT, VEC, FM, SMALL_SLOPE>(xz, g, chan, s, lane, R + S, p, kEdges, k);
}

// Bound by HBM bandwidth: 2 b per element (checkpointing 3 b) plus the
// exchange, during which the chip's memory is idle (a few us, about one
// kernel boundary).
template <int DT, int VEC, int R, int S, int FM>
__global__ __launch_bounds__(kThreads, 2) void fwd_slice_kernel(void* __restrict__ xz, TileGeom g,
                                                                SliceArgs sa, FwdParams prm) {
    constexpr int AB = RawAccess<DT, VEC>::kBytes;
    constexpr int EB = AB / VEC;
    __shared__ raw_t<DT, VEC> lx[S > 0 ? S : 1][kThreads];
    __shared__ double red[kWaves][4];
    __shared__ double chan_s[2];
    __shared__ uint32_t mine_s, rest_s;
    __shared__ uint32_t stage[6 * kMaxSlicesOnChip];
    const SliceId id = slice_id(g);
    const uint64_t chan = id.c * g.row_bytes;
    const SliceTiles s = slice_tiles(g, id.p, xz);
    const TileLane lane = tile_lane<AB>(g);

    const SliceSync sync = slice_sync(sa, g, id.c);
    const uint64_t seen = g.P > 1 && threadIdx.x == 0 ? agent_load(sync.done) : 0;
    // The resident accesses are read once: non-temporal.  Slots past the
    // slice read its last tile again and are not used (see fused_fwd.hip).
    raw_t<DT, VEC> keep[R];
    TileWalk w = walk_begin(g, chan, s);
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const Tile t = walk_tile(g, s, w, s.count ? min(uint32_t(j), s.count - 1) : 0);
        keep[j] = tile_load<DT, VEC, kStream>(xz, t, tile_access<kRowHeads<DT, VEC>>(t, lane).off);
        if (j + 1 < s.count) walk_next(g, w);
    }
    typename Elem<DT>::T edge_raw[kEdges];
#pragma unroll
    for (int i = 0; i < kEdges; ++i) edge_raw[i] = edge_load<DT>(xz, edge_pos<EB>(g, chan, s, id.p, i));
    sched_fence();
    const float gamma_c = prm.gamma[id.c], beta_c = prm.beta[id.c];
    const float rm_c = prm.running_mean[id.c], rv_c = prm.running_var[id.c];
    asm volatile("" ::"s"(gamma_c), "s"(beta_c), "s"(rm_c), "s"(rv_c));
    sched_fence();

    // Shifted sums per thread (see fwd_stats_kernel); the shift is the first
    // value the thread loaded, an element of the channel even where the lane
    // has no access in its first tile.  fp32 within kRun elements, double
    // across them: a thread holds several times the elements that narrow
    // accesses give it in the channel-resident kernels, and one fp32 sum over
    // all of them lost precision against those.
    constexpr int kRun = 8;
    constexpr int kRunAccesses = VEC < kRun ? kRun / VEC : 1;
    double a1 = 0.0, a2 = 0.0;
    float shift, s1 = 0.f, s2 = 0.f;
    uint32_t n = 0;
    {
        float t[VEC];
        unpack<DT, VEC>(keep[0], t);
        shift = t[0];
    }
    auto add = [&](float x) {
        const float d = x - shift;
        s1 += d;
        s2 = fmaf(d, d, s2);
        ++n;
    };
    auto accumulate = [&](raw_t<DT, VEC> raw) {
        float t[VEC];
        unpack<DT, VEC>(raw, t);
#pragma unroll
        for (int e = 0; e < VEC; ++e) add(t[e]);
    };
    auto end_run = [&]() {
        a1 += s1;
        a2 += s2;
        s1 = s2 = 0.f;
    };
    const SliceTiles sb = slice_again(s);
    TileWalk wa = walk_begin(g, chan, sb);
#pragma unroll
    for (int j = 0; j < R; ++j) {
        if (j < sb.count) {
            const TileAccess a = tile_access<kRowHeads<DT, VEC>>(walk_tile(g, sb, wa, j), lane);
            if (a.live) accumulate(keep[j]);
            if ((j + 1) % kRunAccesses == 0) end_run();
        }
        walk_next(g, wa);
        sched_fence();
    }
    // Past the registers: kept in LDS (read once), then read again by the
    // apply phase (through the caches).
    for (uint32_t j = R; j < sb.count; j += kRestU) {
        raw_t<DT, VEC> r[kRestU];
        w = wa;
#pragma unroll
        for (int q = 0; q < kRestU; ++q) {
            const Tile t = walk_tile(g, sb, w, min(j + q, sb.count - 1));
            const uint32_t off = tile_access<kRowHeads<DT, VEC>>(t, lane).off;
            r[q] = S > 0 && j + q < R + S ? tile_load<DT, VEC, kStream>(xz, t, off)
                                          : tile_load<DT, VEC, kCached>(xz, t, off);
            if (j + q + 1 < sb.count) walk_next(g, w);
        }
        sched_fence();
#pragma unroll
        for (int q = 0; q < kRestU; ++q) {
            if (j + q < sb.count) {
                const TileAccess a = tile_access<kRowHeads<DT, VEC>>(walk_tile(g, sb, wa, j + q), lane);
                if (S > 0 && j + q < R + S) lx[j + q - R][threadIdx.x] = r[q];
                if (a.live) accumulate(r[q]);
                if ((q + 1) % kRunAccesses == 0) end_run();
            }
            walk_next(g, wa);
        }
        end_run();
    }

    float edges[kEdges];
#pragma unroll
    for (int i = 0; i < kEdges; ++i) edges[i] = static_cast<float>(edge_raw[i]);
    for (uint32_t i = 0; i < edge_rounds(g); ++i) {
        const Edge t = edge_pos<EB>(g, chan, s, id.p, i);
        if (t.live) add(i == 0   ? edges[0]
                        : i == 1 ? edges[1]
                                 : static_cast<float>(edge_load<DT>(xz, t)));
        end_run();
    }
    end_run();
    static_assert(kEdges == 2, "the edge elements kept in registers");

    // The block's sums about one shift, in double: wave partials in LDS,
    // combined by every wave in the same order.
    const double kw = __shfl(shift, 0, kWave);
    double d1 = a1, d2 = a2, dn = n;
    reshift(d1, d2, dn, shift, kw);
    d1 = wave_sum(d1);
    d2 = wave_sum(d2);
    dn = wave_sum(dn);
    if (lane_id() == 0) {
        const uint32_t wave = threadIdx.x / kWave;
        red[wave][0] = kw;
        red[wave][1] = d1;
        red[wave][2] = d2;
        red[wave][3] = dn;
    }
    __syncthreads();
    const double kref = red[0][0];
    double b[3] = {0.0, 0.0, 0.0};
    if (lane_id() < kWaves) {
        b[0] = red[lane_id()][1];
        b[1] = red[lane_id()][2];
        b[2] = red[lane_id()][3];
        reshift(b[0], b[1], b[2], red[lane_id()][0], kref);
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) b[i] = wave_sum(b[i]);

    uint64_t done = 0;
    double mean, var;
    if (g.P == 1) {
        mean = kref + b[0] * g.inv_m;
        var = fmax(b[1] - b[0] * b[0] * g.inv_m, 0.0) * g.inv_m;
    } else {
        if (threadIdx.x < kWave) {
            const uint64_t b0 = __builtin_bit_cast(uint64_t, b[0]);
            const uint64_t b1 = __builtin_bit_cast(uint64_t, b[1]);
            uint32_t piece[6] = {__builtin_bit_cast(uint32_t, static_cast<float>(kref)),
                                 static_cast<uint32_t>(b[2]),
                                 static_cast<uint32_t>(b0), static_cast<uint32_t>(b0 >> 32),
                                 static_cast<uint32_t>(b1), static_cast<uint32_t>(b1 >> 32)};
            slice_publish<6>(sync, id.p, piece);
            const bool mine = slice_wait<6>(sync, id.p, seen, piece, stage, done);
            // The slices' sums about the first slice's shift, in a fixed order.
            double t1 = 0.0, t2 = 0.0;
            const double kq = __builtin_bit_cast(float, piece[0]);
            const double k0 = __shfl(kq, 0, kWave);
            if (lane_id() < g.P) {
                t1 = __builtin_bit_cast(double, static_cast<uint64_t>(piece[3]) << 32 | piece[2]);
                t2 = __builtin_bit_cast(double, static_cast<uint64_t>(piece[5]) << 32 | piece[4]);
                reshift(t1, t2, static_cast<double>(piece[1]), kq, k0);
            }
            t1 = wave_sum(t1);
            t2 = wave_sum(t2);
            if (lane_id() == 0) {
                chan_s[0] = k0 + t1 * g.inv_m;
                chan_s[1] = fmax(t2 - t1 * t1 * g.inv_m, 0.0) * g.inv_m;
                mine_s = mine;
                rest_s = 0;
            }
        }
        __syncthreads();
        if (!mine_s) return;
        mean = chan_s[0];
        var = chan_s[1];
    }
#pragma unroll
    for (int j = 0; j < R; ++j) opaque(keep[j]);

    const double invstd = rsqrt_d(var + static_cast<double>(prm.eps));
    const double scale_d = FM == kFwdCkpt ? invstd : static_cast<double>(gamma_c) * invstd;
    const float mean_hi = static_cast<float>(mean);
    const double mean_lo = mean - static_cast<double>(mean_hi);
    ApplyK k;
    k.mean_hi = mean_hi;
    k.scale = static_cast<float>(scale_d);
    k.bshift = static_cast<float>((FM == kFwdCkpt ? 0.0 : static_cast<double>(beta_c)) -
                                  mean_lo * scale_d);
    k.slope = prm.slope;
    k.gamma = gamma_c;
    k.beta = beta_c;
    k.out = prm.out;
    auto statistics = [&]() {
        const double mom = prm.momentum;
        prm.save_mean[id.c] = mean_hi;
        prm.save_var[id.c] = static_cast<float>(var);
        prm.running_mean[id.c] =
            static_cast<float>((1.0 - mom) * static_cast<double>(rm_c) + mom * mean);
        prm.running_var[id.c] = static_cast<float>((1.0 - mom) * static_cast<double>(rv_c) +
                                                   mom * var * (g.m / (g.m - 1.0)));
    };
    bool last = g.P == 1;
    if (g.P > 1 && threadIdx.x < kWave) {
        bool rest;
        last = slice_done<6>(sync, seen, done, rest);
        if (rest) rest_s = 1;
    }
    if (last && threadIdx.x == 0) statistics();
    const bool small_slope = prm.slope <= 1.f;
    if (small_slope)
        apply_all<DT, VEC, R, S, FM, true>(xz, g, chan, slice_again(s), lane, keep, lx, edges, id.p, k);
    else
        apply_all<DT, VEC, R, S, FM, false>(xz, g, chan, slice_again(s), lane, keep, lx, edges, id.p, k);
    if (g.P == 1) return;
    lds_barrier();
    if (rest_s) {
        __shared__ uint32_t left[kMaxSlicesOnChip];
        slice_abandoned(sync, id.p, left);
        for (uint32_t q = 0; q < g.P; ++q) {
            if (!left[q]) continue;
            const SliceTiles sq = slice_tiles(g, q, xz);
            if (small_slope)
                apply_rest<DT, VEC, FM, true>(xz, g, chan, sq, lane, 0, q, 0, k);
            else
                apply_rest<DT, VEC, FM, false>(xz, g, chan, sq, lane, 0, q, 0, k);
        }
    }
}

template <int DT, int V, int R, int S, int FM>
void go(void* xz, const TileGeom& g, const SliceArgs& sa, const FwdParams& prm, hipStream_t st) {
    fwd_slice_kernel<DT, V, R, S, FM><<<dim3(g.C * g.P), kThreads, 0, st>>>(xz, g, sa, prm);
}

template <int DT, int V, int FM>
bool launch_v(void* xz, const TileGeom& g, int R, const SliceArgs& sa, const FwdParams& prm,
              hipStream_t st) {
    if (R == 4) return go<DT, V, 4, 0, FM>(xz, g, sa, prm, st), true;
    if (R == 8) return go<DT, V, 8, 0, FM>(xz, g, sa, prm, st), true;
    if (R == 16) return go<DT, V, 16, 0, FM>(xz, g, sa, prm, st), true;
    if constexpr (RawAccess<DT, V>::kBytes == 16) {
        if (R == 20) return go<DT, V, 20, 0, FM>(xz, g, sa, prm, st), true;
        if (R == 24) return go<DT, V, 24, 0, FM>(xz, g, sa, prm, st), true;
        if (R == 32) return go<DT, V, 32, 0, FM>(xz, g, sa, prm, st), true;
        if (R == 50) return go<DT, V, 50 - kSliceFwdLds, kSliceFwdLds, FM>(xz, g, sa, prm, st), true;
    }
    return false;
}

template <int DT, int FM>
bool launch_dt(int vec, void* xz, const TileGeom& g, int R, const SliceArgs& sa,
               const FwdParams& prm, hipStream_t st) {
    constexpr int W = 16 / static_cast<int>(sizeof(typename Elem<DT>::T));
    if (vec == W) return launch_v<DT, W, FM>(xz, g, R, sa, prm, st);
    // InPlace-ABN's own forward takes the channel-resident kernels where the
    // comparison blocks take narrower accesses here.
    if constexpr (FM != kFwdInPlace) {
        if (vec == W / 2) return launch_v<DT, W / 2, FM>(xz, g, R, sa, prm, st);
        if constexpr (W / 4 > 1) {
            if (vec == W / 4) return launch_v<DT, W / 4, FM>(xz, g, R, sa, prm, st);
        }
        if (vec == 1) return launch_v<DT, 1, FM>(xz, g, R, sa, prm, st);
    }
    return false;
}

}  // namespace

// The instances of one storage type (each type is a translation unit of its
// own: slice_fwd_f32.hip, _f16.hip, _bf16.hip).
template <int DT>
bool launch_fwd_slice_dt(int vec, int fm, void* xz, const TileGeom& g, int R, const SliceArgs& sa,
                   const FwdParams& prm, hipStream_t st) {
    return fm == kFwdOut    ? launch_dt<DT, kFwdOut>(vec, xz, g, R, sa, prm, st)
           : fm == kFwdCkpt ? launch_dt<DT, kFwdCkpt>(vec, xz, g, R, sa, prm, st)
                            : launch_dt<DT, kFwdInPlace>(vec, xz, g, R, sa, prm, st);
}

}  // namespace iabn_impl

// The slice-resident backward: as slice_fwd.h, with the sums of dy and dy*w
// of the backward formulations (common.h), dgamma and dbeta, and dx over dz.
// The stored tensor(s) and dz cross HBM once in and dx once out where the
// streaming kernels read them twice and are two launches.
//
// Measured (backward us, before: two streaming passes, or narrow accesses):
// (32, 64, 112x112) fp16 43.0 -> 32.4, (8, 64, 256x256) 54.5 -> 39.9 (3 b per
// element at 5.0 TB/s), (8, 20, 224x224) bf16 18.4 -> 15.0, (8, 256, 129x129)
// fp16 141 -> 41.8, (8, 512, 65x65) 35.9 -> 22.6, (2, 16, 8x8) fp32 4.9 -> 3.9.

#pragma once

#include "launch.h"
#include "tile.h"

namespace iabn_impl {
namespace {

constexpr int kRestU = 2;  // accesses of each tensor in flight per thread past the resident ones

// dx of the slice's accesses from j0 on and edge elements from i0 on, read
// from memory.
template <int DT, int VEC, int BM>
__device__ __forceinline__ void apply_rest(const void* __restrict__ u, const void* __restrict__ zs,
                                           void* __restrict__ dzdx, const TileGeom& g, uint64_t chan,
                                           const SliceTiles& s, const TileLane& lane, uint32_t j0,
                                           uint32_t p, uint32_t i0,
                                           const BwdApplyElem<BM>& dx_of) {
    constexpr int EB = static_cast<int>(sizeof(typename Elem<DT>::T));
    for (uint32_t i = i0; i < edge_rounds(g); ++i) {
        const Edge t = edge_pos<EB>(g, chan, s, p, i);
        if (!t.live) continue;
        const float zv = BM == kBwdFromXZ ? static_cast<float>(edge_load<DT>(zs, t)) : 0.f;
        edge_store<DT>(dzdx, t,
                       dx_of(static_cast<float>(edge_load<DT>(u, t)), zv,
                             static_cast<float>(edge_load<DT>(dzdx, t))));
    }
    if (j0 >= s.count) return;
    TileWalk w = walk_begin(g, chan, s, j0);
    for (uint32_t j = j0; j < s.count; j += kRestU) {
        raw_t<DT, VEC> ru[kRestU], rz[kRestU], rg[kRestU];
        TileWalk wl = w;
#pragma unroll
        for (int q = 0; q < kRestU; ++q) {
            const Tile t = walk_tile(g, s, wl, min(j + q, s.count - 1));
            const uint32_t off = tile_access<kRowHeads<DT, VEC>>(t, lane).off;
            ru[q] = tile_load<DT, VEC, kStream>(u, t, off);
            if constexpr (BM == kBwdFromXZ) rz[q] = tile_load<DT, VEC, kStream>(zs, t, off);
            rg[q] = tile_load<DT, VEC, kStream>(dzdx, t, off);
            if (j + q + 1 < s.count) walk_next(g, wl);
        }
        sched_fence();
#pragma unroll
        for (int q = 0; q < kRestU; ++q) {
            if (j + q < s.count) {
                const Tile t = walk_tile(g, s, w, j + q);
                const TileAccess a = tile_access<kRowHeads<DT, VEC>>(t, lane);
                if (a.live) {
                    float tu[VEC], tz[VEC], tg[VEC];
                    unpack<DT, VEC>(ru[q], tu);
                    if constexpr (BM == kBwdFromXZ) unpack<DT, VEC>(rz[q], tz);
                    unpack<DT, VEC>(rg[q], tg);
#pragma unroll
                    for (int e = 0; e < VEC; ++e)
                        tg[e] = dx_of(tu[e], BM == kBwdFromXZ ? tz[e] : 0.f, tg[e]);
                    tile_store<DT, VEC>(dzdx, t, a.off, tg);
                }
            }
            walk_next(g, w);
        }
    }
}

// Bound by HBM bandwidth: 3 b per element (standard block 4 b) plus the
// exchange.  R = 24 accesses of each tensor and 8 more in LDS are what two
// blocks per CU hold (two waves per SIMD, 256 registers; 64 KB of LDS each).
template <int DT, int VEC, int R, int S, int BM, bool FINE>
__global__ __launch_bounds__(kThreads, 2) void bwd_slice_kernel(const void* __restrict__ u,
                                                                const void* __restrict__ zs,
                                                                void* __restrict__ dzdx, TileGeom g,
                                                                SliceArgs sa, BwdParams prm) {
    constexpr int AB = RawAccess<DT, VEC>::kBytes;
    constexpr int EB = AB / VEC;
    constexpr bool XZ = BM == kBwdFromXZ;
    constexpr int NW = XZ ? (R * VEC + 31) / 32 : 1;
    __shared__ raw_t<DT, VEC> lu[S > 0 ? S : 1][kThreads], lg[S > 0 ? S : 1][kThreads];
    __shared__ uint8_t ls[XZ && S > 0 ? S : 1][kThreads];  // signs of z
    __shared__ double red[kWaves][2];
    __shared__ double chan_s[2];
    __shared__ uint32_t mine_s, rest_s;
    __shared__ uint32_t stage[4 * kMaxSlicesOnChip];
    const SliceId id = slice_id(g);
    const uint64_t chan = id.c * g.row_bytes;
    const SliceTiles s = slice_tiles(g, id.p, dzdx);
    const TileLane lane = tile_lane<AB>(g);

    const SliceSync sync = slice_sync(sa, g, id.c);
    const uint64_t seen = g.P > 1 && threadIdx.x == 0 ? agent_load(sync.done) : 0;
    // Resident accesses: non-temporal; slots past the slice read its last
    // tile again and are not used.  The standard block's z (into x's
    // registers) is reduced to sign bits before x is loaded, so no more than
    // two tensors are held.
    raw_t<DT, VEC> ku[R], kg[R];
    uint32_t negm[NW];
#pragma unroll
    for (int q = 0; q < NW; ++q) negm[q] = 0u;
    TileWalk w = walk_begin(g, chan, s);
    if constexpr (XZ) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const Tile t = walk_tile(g, s, w, s.count ? min(uint32_t(j), s.count - 1) : 0);
            const uint32_t off = tile_access<kRowHeads<DT, VEC>>(t, lane).off;
            ku[j] = tile_load<DT, VEC, kStream>(zs, t, off);
            kg[j] = tile_load<DT, VEC, kStream>(dzdx, t, off);
            if (j + 1 < s.count) walk_next(g, w);
        }
        sched_fence();
#pragma unroll
        for (int j = 0; j < R; ++j) {
            float tz[VEC];
            unpack<DT, VEC>(ku[j], tz);
#pragma unroll
            for (int e = 0; e < VEC; ++e)
                negm[(j * VEC + e) / 32] |= static_cast<uint32_t>(tz[e] < 0.f) << ((j * VEC + e) % 32);
        }
#pragma unroll
        for (int q = 0; q < NW; ++q) asm volatile("" : "+v"(negm[q])::"memory");
        w = walk_begin(g, chan, s);
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const Tile t = walk_tile(g, s, w, s.count ? min(uint32_t(j), s.count - 1) : 0);
            ku[j] = tile_load<DT, VEC, kStream>(u, t, tile_access<kRowHeads<DT, VEC>>(t, lane).off);
            if (j + 1 < s.count) walk_next(g, w);
        }
    } else {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const Tile t = walk_tile(g, s, w, s.count ? min(uint32_t(j), s.count - 1) : 0);
            const uint32_t off = tile_access<kRowHeads<DT, VEC>>(t, lane).off;
            ku[j] = tile_load<DT, VEC, kStream>(u, t, off);
            kg[j] = tile_load<DT, VEC, kStream>(dzdx, t, off);
            if (j + 1 < s.count) walk_next(g, w);
        }
    }
    typename Elem<DT>::T edge_u[kEdges], edge_z[kEdges], edge_g[kEdges];
#pragma unroll
    for (int i = 0; i < kEdges; ++i) {
        const Edge t = edge_pos<EB>(g, chan, s, id.p, i);
        edge_u[i] = edge_load<DT>(u, t);
        if constexpr (XZ) edge_z[i] = edge_load<DT>(zs, t);
        edge_g[i] = edge_load<DT>(dzdx, t);
    }
    sched_fence();
    const float gamma_c = prm.gamma[id.c], beta_c = prm.beta[id.c];
    const float mean_c = XZ ? prm.save_mean[id.c] : 0.f;
    const double invstd = rsqrt_d(static_cast<double>(prm.save_var[id.c]) +
                                  static_cast<double>(prm.eps));
    const BwdReduceElem<BM> el =
        make_reduce_elem<BM>(prm.slope, gamma_c, beta_c, mean_c, invstd, prm.ii != 0);
    const BwdRecip rc = make_recip(gamma_c, prm.slope, g.inv_m);
    sched_fence();

    // fp32 within one access, double across accesses (see bwd_fused_channel);
    // where the channel-resident kernels would take the layer too, on ragged
    // rows (FINE), every element's terms go to double, as those move such rows
    // an element or two at a time and add up no more in fp32: the relative
    // error of dbeta on (8, 512, 65x65) fp16 is 2.5e-8 (8 elements in fp32:
    // 5.0e-8).  Elsewhere it would cost 2-8% ((32, 64, 112x112) fp16 32.3 ->
    // 33.2 us, (50, 178, 1833) bf16 30.0 -> 32.3), and 8 elements are fewer than
    // the streaming kernels add up.
    double acc_dy = 0.0, acc_dyw = 0.0;
    auto accumulate = [&](raw_t<DT, VEC> ru, raw_t<DT, VEC> rg, auto neg) {
        float tu[VEC], tg[VEC];
        unpack<DT, VEC>(ru, tu);
        unpack<DT, VEC>(rg, tg);
        float sdy = 0.f, sdyw = 0.f;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            float dy, w;
            if constexpr (XZ) el.with_neg(neg(e), tu[e], tg[e], dy, w);
            else el(tu[e], 0.f, tg[e], dy, w);
            if constexpr (FINE) {
                acc_dy += dy;
                acc_dyw = fma(static_cast<double>(dy), static_cast<double>(w), acc_dyw);
            } else {
                sdy += dy;
                sdyw = fmaf(dy, w, sdyw);
            }
        }
        if constexpr (!FINE) {
            acc_dy += sdy;
            acc_dyw += sdyw;
        }
    };
    const SliceTiles sb = slice_again(s);
    TileWalk wa = walk_begin(g, chan, sb);
#pragma unroll
    for (int j = 0; j < R; ++j) {
        if (j < sb.count) {
            const TileAccess a = tile_access<kRowHeads<DT, VEC>>(walk_tile(g, sb, wa, j), lane);
            if (a.live)
                accumulate(ku[j], kg[j], [&](int e) {
                    return ((negm[(j * VEC + e) / 32 % NW] >> ((j * VEC + e) % 32)) & 1u) != 0;
                });
        }
        walk_next(g, wa);
        sched_fence();
    }
    // Past the registers: kept in LDS (read once), then read again by the
    // apply phase (through the caches).
    for (uint32_t j = R; j < sb.count; j += kRestU) {
        raw_t<DT, VEC> ru[kRestU], rz[kRestU], rg[kRestU];
        w = wa;
#pragma unroll
        for (int q = 0; q < kRestU; ++q) {
            const Tile t = walk_tile(g, sb, w, min(j + q, sb.count - 1));
            const uint32_t off = tile_access<kRowHeads<DT, VEC>>(t, lane).off;
            if (S > 0 && j + q < R + S) {
                ru[q] = tile_load<DT, VEC, kStream>(u, t, off);
                if constexpr (XZ) rz[q] = tile_load<DT, VEC, kStream>(zs, t, off);
                rg[q] = tile_load<DT, VEC, kStream>(dzdx, t, off);
            } else {
                ru[q] = tile_load<DT, VEC, kCached>(u, t, off);
                if constexpr (XZ) rz[q] = tile_load<DT, VEC, kCached>(zs, t, off);
                rg[q] = tile_load<DT, VEC, kCached>(dzdx, t, off);
            }
            if (j + q + 1 < sb.count) walk_next(g, w);
        }
        sched_fence();
#pragma unroll
        for (int q = 0; q < kRestU; ++q) {
            if (j + q < sb.count) {
                const TileAccess a = tile_access<kRowHeads<DT, VEC>>(walk_tile(g, sb, wa, j + q), lane);
                uint32_t bits = 0;
                if constexpr (XZ) {
                    float tz[VEC];
                    unpack<DT, VEC>(rz[q], tz);
#pragma unroll
                    for (int e = 0; e < VEC; ++e) bits |= static_cast<uint32_t>(tz[e] < 0.f) << e;
                }
                if (S > 0 && j + q < R + S) {
                    lu[j + q - R][threadIdx.x] = ru[q];
                    lg[j + q - R][threadIdx.x] = rg[q];
                    if constexpr (XZ) ls[j + q - R][threadIdx.x] = static_cast<uint8_t>(bits);
                }
                if (a.live)
                    accumulate(ru[q], rg[q], [&](int e) { return ((bits >> e) & 1u) != 0; });
            }
            walk_next(g, wa);
        }
    }

    float tu2[kEdges], tz2[kEdges], tg2[kEdges];
#pragma unroll
    for (int i = 0; i < kEdges; ++i) {
        tu2[i] = static_cast<float>(edge_u[i]);
        tz2[i] = XZ ? static_cast<float>(edge_z[i]) : 0.f;
        tg2[i] = static_cast<float>(edge_g[i]);
    }
    for (uint32_t i = 0; i < edge_rounds(g); ++i) {
        const Edge t = edge_pos<EB>(g, chan, s, id.p, i);
        if (!t.live) continue;
        float dy, w1;
        if (i < kEdges)
            el(i == 0 ? tu2[0] : tu2[1], i == 0 ? tz2[0] : tz2[1], i == 0 ? tg2[0] : tg2[1], dy, w1);
        else
            el(static_cast<float>(edge_load<DT>(u, t)),
               XZ ? static_cast<float>(edge_load<DT>(zs, t)) : 0.f,
               static_cast<float>(edge_load<DT>(dzdx, t)), dy, w1);
        acc_dy += dy;
        acc_dyw += dy * w1;
    }
    static_assert(kEdges == 2, "the edge elements kept in registers");

    // The block's sums: wave partials in LDS, combined by every wave in the
    // same order.
    acc_dy = wave_sum(acc_dy);
    acc_dyw = wave_sum(acc_dyw);
    if (lane_id() == 0) {
        red[threadIdx.x / kWave][0] = acc_dy;
        red[threadIdx.x / kWave][1] = acc_dyw;
    }
    __syncthreads();
    double dbeta = wave_sum(lane_id() < kWaves ? red[lane_id() % kWaves][0] : 0.0);
    double sdyw = wave_sum(lane_id() < kWaves ? red[lane_id() % kWaves][1] : 0.0);

    uint64_t done = 0;
    if (g.P > 1) {
        if (threadIdx.x < kWave) {
            const uint64_t b0 = __builtin_bit_cast(uint64_t, dbeta);
            const uint64_t b1 = __builtin_bit_cast(uint64_t, sdyw);
            uint32_t piece[4] = {static_cast<uint32_t>(b0), static_cast<uint32_t>(b0 >> 32),
                                 static_cast<uint32_t>(b1), static_cast<uint32_t>(b1 >> 32)};
            slice_publish<4>(sync, id.p, piece);
            const bool mine = slice_wait<4>(sync, id.p, seen, piece, stage, done);
            double t1 = 0.0, t2 = 0.0;
            if (lane_id() < g.P) {
                t1 = __builtin_bit_cast(double, static_cast<uint64_t>(piece[1]) << 32 | piece[0]);
                t2 = __builtin_bit_cast(double, static_cast<uint64_t>(piece[3]) << 32 | piece[2]);
            }
            t1 = wave_sum(t1);
            t2 = wave_sum(t2);
            if (lane_id() == 0) {
                chan_s[0] = t1;
                chan_s[1] = t2;
                mine_s = mine;
                rest_s = 0;
            }
        }
        __syncthreads();
        if (!mine_s) return;
        dbeta = chan_s[0];
        sdyw = chan_s[1];
    }
#pragma unroll
    for (int j = 0; j < R; ++j) {
        opaque(ku[j]);
        opaque(kg[j]);
    }
#pragma unroll
    for (int q = 0; q < NW; ++q) opaque(negm[q]);

    const double A = static_cast<double>(gamma_c) * invstd;
    const BwdApplyElem<BM> dx_of = make_apply_elem<BM>(A, sdyw, dbeta, rc, prm.slope, gamma_c,
                                                       beta_c, mean_c, invstd, prm.ii != 0);
    auto gradients = [&]() {
        prm.dgamma[id.c] = static_cast<float>(sdyw);
        prm.dbeta[id.c] = static_cast<float>(dbeta);
    };
    bool last = g.P == 1;
    if (g.P > 1 && threadIdx.x < kWave) {
        bool rest;
        last = slice_done<4>(sync, seen, done, rest);
        if (rest) rest_s = 1;
    }
    if (last && threadIdx.x == 0) gradients();

    auto emit = [&](const Tile& t, uint32_t off, raw_t<DT, VEC> ru, raw_t<DT, VEC> rg,
                    auto neg) {
        float tu[VEC], tg[VEC];
        unpack<DT, VEC>(ru, tu);
        unpack<DT, VEC>(rg, tg);
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            if constexpr (XZ) tg[e] = dx_of.with_neg(neg(e), tu[e], tg[e]);
            else tg[e] = dx_of(tu[e], 0.f, tg[e]);
        }
        tile_store<DT, VEC>(dzdx, t, off, tg);
    };
    if (g.edges) {
#pragma unroll
        for (int i = 0; i < kEdges; ++i) {
            const Edge t = edge_pos<EB>(g, chan, s, id.p, i);
            if (t.live) edge_store<DT>(dzdx, t, dx_of(tu2[i], tz2[i], tg2[i]));
        }
    }
    const SliceTiles sc = slice_again(s);
    w = walk_begin(g, chan, sc);
#pragma unroll
    for (int j = 0; j < R; ++j) {
        if (j < sc.count) {
            const Tile t = walk_tile(g, sc, w, j);
            const TileAccess a = tile_access<kRowHeads<DT, VEC>>(t, lane);
            if (a.live)
                emit(t, a.off, ku[j], kg[j], [&](int e) {
                    return ((negm[(j * VEC + e) / 32 % NW] >> ((j * VEC + e) % 32)) & 1u) != 0;
                });
        }
        walk_next(g, w);
        sched_fence();
    }
    if constexpr (S > 0) {
#pragma unroll 1
        for (uint32_t j = R; j < min(sc.count, uint32_t(R + S)); ++j) {
            const Tile t = walk_tile(g, sc, w, j);
            const TileAccess a = tile_access<kRowHeads<DT, VEC>>(t, lane);
            const uint32_t bits = XZ ? ls[XZ ? j - R : 0][threadIdx.x] : 0u;
            if (a.live)
                emit(t, a.off, lu[j - R][threadIdx.x], lg[j - R][threadIdx.x],
                     [&](int e) { return ((bits >> e) & 1u) != 0; });
            walk_next(g, w);
        }
    }
    apply_rest<DT, VEC, BM>(u, zs, dzdx, g, chan, sc, lane, R + S, id.p, kEdges, dx_of);
    if (g.P == 1) return;
    lds_barrier();
    if (rest_s) {
        __shared__ uint32_t left[kMaxSlicesOnChip];
        slice_abandoned(sync, id.p, left);
        for (uint32_t q = 0; q < g.P; ++q)
            if (left[q])
                apply_rest<DT, VEC, BM>(u, zs, dzdx, g, chan, slice_tiles(g, q, dzdx), lane, 0, q, 0,
                                        dx_of);
    }
}

template <int DT, int V, int R, int S, int BM, bool FINE>
void go(const void* u, const void* zs, void* dzdx, const TileGeom& g, const SliceArgs& sa,
        const BwdParams& prm, hipStream_t st) {
    bwd_slice_kernel<DT, V, R, S, BM, FINE>
        <<<dim3(g.C * g.P), kThreads, 0, st>>>(u, zs, dzdx, g, sa, prm);
}

template <int DT, int V, int BM, bool FINE>
bool launch_v(const void* u, const void* zs, void* dzdx, const TileGeom& g, int R,
              const SliceArgs& sa, const BwdParams& prm, hipStream_t st) {
    if (R == 4) return go<DT, V, 4, 0, BM, FINE>(u, zs, dzdx, g, sa, prm, st), true;
    if (R == 8) return go<DT, V, 8, 0, BM, FINE>(u, zs, dzdx, g, sa, prm, st), true;
    if (R == 16) return go<DT, V, 16, 0, BM, FINE>(u, zs, dzdx, g, sa, prm, st), true;
    if constexpr (RawAccess<DT, V>::kBytes == 16) {
        if (R == 20) return go<DT, V, 20, 0, BM, FINE>(u, zs, dzdx, g, sa, prm, st), true;
        if (R == 24) return go<DT, V, 24, 0, BM, FINE>(u, zs, dzdx, g, sa, prm, st), true;
        if (R == 32)
            return go<DT, V, 32 - kSliceBwdLds, kSliceBwdLds, BM, FINE>(u, zs, dzdx, g, sa, prm, st), true;
    }
    return false;
}

template <int DT, int BM>
bool launch_dt(int vec, bool fine, const void* u, const void* zs, void* dzdx, const TileGeom& g,
               int R, const SliceArgs& sa, const BwdParams& prm, hipStream_t st) {
    constexpr int W = 16 / static_cast<int>(sizeof(typename Elem<DT>::T));
    if constexpr (BM == kBwdFromZ) {
        if (vec == W && fine) return launch_v<DT, W, BM, true>(u, zs, dzdx, g, R, sa, prm, st);
    }
    if (vec == W) return launch_v<DT, W, BM, false>(u, zs, dzdx, g, R, sa, prm, st);
    if (vec == W / 2) return launch_v<DT, W / 2, BM, false>(u, zs, dzdx, g, R, sa, prm, st);
    if constexpr (W / 4 > 1) {
        if (vec == W / 4) return launch_v<DT, W / 4, BM, false>(u, zs, dzdx, g, R, sa, prm, st);
    }
    if (vec == 1) return launch_v<DT, 1, BM, false>(u, zs, dzdx, g, R, sa, prm, st);
    return false;
}

}  // namespace

// The instances of one storage type (each type is a translation unit of its
// own: slice_bwd_f32.hip, _f16.hip, _bf16.hip).
template <int DT>
bool launch_bwd_slice_dt(int vec, int bm, bool fine, const void* u, const void* zs, void* dzdx,
                         const TileGeom& g, int R, const SliceArgs& sa, const BwdParams& prm,
                         hipStream_t st) {
    return bm == kBwdFromXZ     ? launch_dt<DT, kBwdFromXZ>(vec, fine, u, zs, dzdx, g, R, sa, prm, st)
           : bm == kBwdFromXhat ? launch_dt<DT, kBwdFromXhat>(vec, fine, u, zs, dzdx, g, R, sa, prm, st)
                                : launch_dt<DT, kBwdFromZ>(vec, fine, u, zs, dzdx, g, R, sa, prm, st);
}

}  // namespace iabn_impl

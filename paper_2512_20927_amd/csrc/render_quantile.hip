// Quantile Rendering forward (Algorithm 1, Sec. 4.2).
//
// One workgroup per 16x16 tile, one thread per pixel (4 wave64s).
// Phase 1 (selection, quantile_select.h, the walk shared with the backward):
// the tile's depth-sorted list is staged into LDS in batches of 256 projected
// records; every pixel walks it front to back with the transmittance chain
// T_test = T (1 - alpha') and the threshold test T_test < t_{k+1}. A pixel is
// done once all K thresholds are consumed (the paper's stop test T_test <
// 1/(K+1) is the same event), and the whole workgroup leaves the list as soon
// as every pixel is done. The walk leaves, for each group of four adjacent
// pixels (a row segment of the tile, four neighbouring lanes that look at an
// entry together), the group's distinct selections with the four weights,
// which are then divided by the pixel's 1 - T^Q.
// Phase 2 (gather-blend): pixels are gathered four at a time with the lanes of
// a wave spanning the feature dimension, so every distinct feature row is
// loaded once per group (mostly from L2: neighbouring pixels select the same
// Gaussians); rows are accumulated in float32 and streamed to the [H, W, D]
// map with non-temporal stores. The map write is the dominant HBM traffic of
// the whole pipeline.
// Everything after the walk is wave-local: wave w's pixels (tile rows
// 4w .. 4w+3) are exactly the pixels of the groups it gathers.
// Collecting the groups in the walk instead of lists of each pixel's
// selections that are merged afterwards takes the merge away, and 51 KB of
// LDS at any K instead of 29 KB + 2 KB x K, with 32 entries a group instead
// of 16 (past which rows were loaded pixel by pixel): 16 views 640x480x512
// float32, K = 8: 2,017 -> 1,985 us (5.2 TB/s; the map write bounds it); 4 views
// 1296x968x512, bf16 table, K = 16: 2,900 -> 2,060 us (10% of the groups select
// more than 16); one 640x480x512 view at K = 40: 507 -> 235 us; 16 views
// 640x480x16, K = 8: 584 -> 480 us.
// The Top-K sampler replaces entries of its pixels' lists until the end of the
// list, so it keeps those lists and the merge.
#include <type_traits>

#include "quantile_select.h"

namespace qr {

// R distinct rows of a merged group, both column slots of the lane: all 2R
// loads are requested before the first is used, then accumulated in row order.
template <int DT, int R>
__device__ __forceinline__ void accum_rows(const GView& v, const int* ug, const float4* uw,
                                           const uint8_t* um, int e0, int l0, int l1, int dim,
                                           float4 (&a0)[kPG], float4 (&a1)[kPG]) {
  float4 f0[R], f1[R];
#pragma unroll
  for (int e = 0; e < R; ++e) {
    const int g = __builtin_amdgcn_readfirstlane(ug[e0 + e]);
    f0[e] = load_feat4_global<DT>(v.feats, v.scale, g, dim, 4 * l0);
    f1[e] = load_feat4_global<DT>(v.feats, v.scale, g, dim, 4 * l1);
  }
#pragma unroll
  for (int e = 0; e < R; ++e) {
    const float4 w = uw[e0 + e];
    const float ws[kPG] = {w.x, w.y, w.z, w.w};
    // pixels that did not select the row have weight 0: skipped by uniform
    // (scalar) branches instead of multiplied
    const uint32_t mk = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(um[e0 + e]));
#pragma unroll
    for (int q = 0; q < kPG; ++q) {
      if (!(mk & (1u << q))) continue;
      a0[q].x += ws[q] * f0[e].x;
      a0[q].y += ws[q] * f0[e].y;
      a0[q].z += ws[q] * f0[e].z;
      a0[q].w += ws[q] * f0[e].w;
      a1[q].x += ws[q] * f1[e].x;
      a1[q].y += ws[q] * f1[e].y;
      a1[q].z += ws[q] * f1[e].z;
      a1[q].w += ws[q] * f1[e].w;
    }
  }
}

// Stores four features (columns 4 c4 .. 4 c4 + 3) of map pixel pix, as
// float32 or as bfloat16 codes rounded to nearest even (OT = QR_BF16).
template <int OT>
__device__ __forceinline__ void store_out4(QR_GLOBAL float* out, int64_t pix, int dim, int c4,
                                           float4 v) {
  if constexpr (OT == QR_F32) {
    store_stream(reinterpret_cast<QR_GLOBAL float4*>(out + pix * dim) + c4, v);
  } else {
    const u32x2 x = {static_cast<uint32_t>(__builtin_bit_cast(uint16_t, static_cast<__bf16>(v.x))) |
                         (static_cast<uint32_t>(__builtin_bit_cast(uint16_t, static_cast<__bf16>(v.y))) << 16),
                     static_cast<uint32_t>(__builtin_bit_cast(uint16_t, static_cast<__bf16>(v.z))) |
                         (static_cast<uint32_t>(__builtin_bit_cast(uint16_t, static_cast<__bf16>(v.w))) << 16)};
    __builtin_nontemporal_store(
        x, reinterpret_cast<QR_GLOBAL u32x2*>(reinterpret_cast<QR_GLOBAL uint16_t*>(out) + pix * dim + 4 * c4));
  }
}

// (what the same lane stored there + v) * scale, float32 maps.
__device__ __forceinline__ void add_out4(QR_GLOBAL float* out, int64_t pix, int dim, int c4, float4 v, float scale) {
  const f32x4 x = *(reinterpret_cast<const QR_GLOBAL f32x4*>(out + pix * dim) + c4);
  store_out4<QR_F32>(out, pix, dim, c4,
                     make_float4((x.x + v.x) * scale, (x.y + v.y) * scale, (x.z + v.z) * scale, (x.w + v.w) * scale));
}

// Gather-blend of one 4-pixel group (pixels p0 .. p0 + 3 of the tile) with nu
// distinct selections: out[p] = sum_e (w_pe / (1 - T^Q_p)) f_e (the
// normalisation is folded into the weights). Each lane owns two float4 columns per pass (512
// features per pass for the wave); rows are taken four at a time, the last
// two or one on their own, so no multiply is spent on padding. kPart: the sum
// is added to what the map holds of the group's earlier entries, and the result
// takes the factor scale(q).
template <int DT, int OT, bool kPart = false, class Scale = int>
__device__ __forceinline__ void gather_group(const GView& v, const int* ug, const float4* uw,
                                             const uint8_t* um, int p0, int nu, int tx, int ty,
                                             int lane, int dim, const Scale& scale = 0) {
  const int dim4 = dim >> 2;
  for (int cb = 0; cb < dim4; cb += 128) {
    const int c0 = cb + lane, c1 = cb + 64 + lane;
    const int l0 = min(c0, dim4 - 1), l1 = min(c1, dim4 - 1);  // in-bounds columns to load
    float4 a0[kPG], a1[kPG];
#pragma unroll
    for (int q = 0; q < kPG; ++q) {
      a0[q] = make_float4(0.f, 0.f, 0.f, 0.f);
      a1[q] = a0[q];
    }
    int e0 = 0;
    for (; e0 + 4 <= nu; e0 += 4) accum_rows<DT, 4>(v, ug, uw, um, e0, l0, l1, dim, a0, a1);
    if (e0 + 2 <= nu) {
      accum_rows<DT, 2>(v, ug, uw, um, e0, l0, l1, dim, a0, a1);
      e0 += 2;
    }
    if (e0 < nu) accum_rows<DT, 1>(v, ug, uw, um, e0, l0, l1, dim, a0, a1);
#pragma unroll
    for (int q = 0; q < kPG; ++q) {
      const int p = p0 + q;
      const int gx = tx * kTile + (p % kTile), gy = ty * kTile + (p / kTile);
      if (gx >= v.W || gy >= v.H) continue;
      const int64_t pix = static_cast<int64_t>(gy) * v.W + gx;
      if constexpr (kPart) {
        if (c0 < dim4) add_out4(v.out, pix, dim, c0, a0[q], scale(q));
        if (c1 < dim4) add_out4(v.out, pix, dim, c1, a1[q], scale(q));
      } else {
        if (c0 < dim4) store_out4<OT>(v.out, pix, dim, c0, a0[q]);
        if (c1 < dim4) store_out4<OT>(v.out, pix, dim, c1, a1[q]);
      }
    }
  }
}

// Gather-blend of all sixteen groups of a wave at once, for narrow
// rows (dim <= 128): lpg lanes per group (the power of two >= dim / 4, one
// float4 column each), so 64 / lpg groups are blended side by side, and
// kNarrowRows (16) row loads of a lane are requested before the first is used
// (slots past a group's distinct count load a row of the group again and are
// not accumulated). One memory round trip per round and 16 rows instead of
// several per group. ug, uw, um: the wave's entries, those of its group g from
// first(g) on; count(g): how many, negative: skip the group. kPart, scale(p):
// as in gather_group, for pixel p of the wave.
// A pixel takes every row of its group, with weight 0 where it did not select
// it; a lane whose result is not finite forms it again from the selected rows
// alone, so that such a row reaches no pixel that did not select it.
constexpr int kNarrowRows = 16;

template <int DT, int OT, bool kPart = false, class First, class Count, class Scale = int>
__device__ __forceinline__ void gather_groups_narrow(const GView& v, const int* ug, const float4* uw,
                                                     const uint8_t* um, const First& first,
                                                     const Count& count, int wave, int tx, int ty,
                                                     int lane, int dim, const Scale& scale = 0) {
  const int dim4 = dim >> 2;
  const int lpg_log = dim4 <= 4 ? 2 : dim4 <= 8 ? 3 : dim4 <= 16 ? 4 : 5;
  const int gpr = 64 >> lpg_log;  // groups per round
  const int c = lane & ((1 << lpg_log) - 1);
  const int cl = min(c, dim4 - 1);  // in-bounds column to load
  for (int r0 = 0; r0 < kWaveGroups; r0 += gpr) {
    const int grp = r0 + (lane >> lpg_log);
    const int nu = count(grp), at = first(grp);
    float4 a[kPG];
#pragma unroll
    for (int q = 0; q < kPG; ++q) a[q] = make_float4(0.f, 0.f, 0.f, 0.f);
    constexpr int kRows = kPart ? kNarrowRows / 2 : kNarrowRows;  // (registers of the paused walk)
    for (int e0 = 0; __any(e0 < nu); e0 += kRows) {
      if (e0 < nu) {
        float4 f[kRows];
#pragma unroll
        for (int e = 0; e < kRows; ++e)
          f[e] = load_feat4_global<DT>(v.feats, v.scale, ug[at + min(e0 + e, nu - 1)], dim, 4 * cl);
#pragma unroll
        for (int e = 0; e < kRows; ++e) {
          if (e0 + e < nu) {
            const float4 w = uw[at + e0 + e];
            const float ws[kPG] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int q = 0; q < kPG; ++q) {
              a[q].x += ws[q] * f[e].x;
              a[q].y += ws[q] * f[e].y;
              a[q].z += ws[q] * f[e].z;
              a[q].w += ws[q] * f[e].w;
            }
          }
        }
      }
    }
    float sum = 0.f;
#pragma unroll
    for (int q = 0; q < kPG; ++q) sum += (a[q].x + a[q].y) + (a[q].z + a[q].w);
    if (!(fabsf(sum) < INFINITY)) {
#pragma unroll
      for (int q = 0; q < kPG; ++q) a[q] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 1
      for (int e = at; e < at + nu; ++e) {
        const float4 f = load_feat4_global<DT>(v.feats, v.scale, ug[e], dim, 4 * cl);
        const float4 w = uw[e];
        const float ws[kPG] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int q = 0; q < kPG; ++q) {
          if (!((um[e] >> q) & 1)) continue;
          a[q].x += ws[q] * f.x;
          a[q].y += ws[q] * f.y;
          a[q].z += ws[q] * f.z;
          a[q].w += ws[q] * f.w;
        }
      }
    }
    float s[kPG];  // from other lanes: outside the condition
    if constexpr (kPart) {
#pragma unroll
      for (int q = 0; q < kPG; ++q) s[q] = scale(kPG * grp + q);
    }
    if (nu >= 0 && c < dim4) {
      const int p0 = (wave * kWaveGroups + grp) * kPG;
#pragma unroll
      for (int q = 0; q < kPG; ++q) {
        const int p = p0 + q;
        const int gx = tx * kTile + (p % kTile), gy = ty * kTile + (p / kTile);
        const int64_t pix = static_cast<int64_t>(gy) * v.W + gx;
        const bool in = gx < v.W && gy < v.H;
        if constexpr (kPart) {
          if (in) add_out4(v.out, pix, dim, c, a[q], s[q]);
        } else {
          if (in) store_out4<OT>(v.out, pix, dim, c, a[q]);
        }
      }
    }
  }
}

// Top-K: the groups that gather_groups_narrow skipped (more distinct
// selections than the merge capacity), with the same lane layout: pixel by pixel, each pixel's
// selections taken eight at a time (their ids, then their rows, each batch
// requested together), all such groups of a round side by side.
template <int DT, int OT, class Lds>
__device__ __forceinline__ void gather_groups_narrow_overflow(const GView& v, const Lds& L,
                                                              const int* __restrict__ s_sel_pos,
                                                              const float* __restrict__ s_sel_w,
                                                              int KP, int K, int wave, int tx, int ty,
                                                              int lane, int dim) {
  constexpr int kChunk = 8;
  const int dim4 = dim >> 2;
  const int lpg_log = dim4 <= 4 ? 2 : dim4 <= 8 ? 3 : dim4 <= 16 ? 4 : 5;
  const int gpr = 64 >> lpg_log;
  const int c = lane & ((1 << lpg_log) - 1);
  const int cl = min(c, dim4 - 1);
  for (int r0 = 0; r0 < kWaveGroups; r0 += gpr) {
    const int grp = wave * kWaveGroups + r0 + (lane >> lpg_log);
    const bool mine = L.unum[grp] < 0;
    if (!__any(mine)) continue;
#pragma unroll 1
    for (int q = 0; q < kPG; ++q) {
      const int p = grp * kPG + q;
      const int n = mine ? L.ns[p] : -1;  // -1: not this path's pixel, or outside the image
      float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
      for (int j0 = 0; j0 < K; j0 += kChunk) {
        if (!__any(n > j0)) break;
        if (n > j0) {
          int g[kChunk];
          float w[kChunk];
#pragma unroll
          for (int jj = 0; jj < kChunk; ++jj) {
            const int j = min(j0 + jj, n - 1);
            g[jj] = static_cast<int>(v.sorted_gid[s_sel_pos[p * KP + j]]);
            w[jj] = s_sel_w[p * KP + j];
          }
          float4 f[kChunk];
#pragma unroll
          for (int jj = 0; jj < kChunk; ++jj) f[jj] = load_feat4_global<DT>(v.feats, v.scale, g[jj], dim, 4 * cl);
#pragma unroll
          for (int jj = 0; jj < kChunk; ++jj) {
            if (j0 + jj < n) {
              a.x += w[jj] * f[jj].x;
              a.y += w[jj] * f[jj].y;
              a.z += w[jj] * f[jj].z;
              a.w += w[jj] * f[jj].w;
            }
          }
        }
      }
      if (n >= 0 && c < dim4) {
        const int gx = tx * kTile + (p % kTile), gy = ty * kTile + (p / kTile);
        const float inv = L.inv[p];
        store_out4<OT>(v.out, static_cast<int64_t>(gy) * v.W + gx, dim, c,
                       make_float4(a.x * inv, a.y * inv, a.z * inv, a.w * inv));
      }
    }
  }
}

// Top-K: gather-blend of a group with more distinct selections than the merge
// capacity: pixel by pixel, each selection's row loaded for its own pixel.
template <int DT, int OT, class Lds>
__device__ __forceinline__ void gather_group_per_pixel(const GView& v, const Lds& L,
                                                       const int* __restrict__ s_sel_pos,
                                                       const float* __restrict__ s_sel_w, int KP,
                                                       int grp, int tx, int ty, int lane, int dim) {
  const int dim4 = dim >> 2;
  const int p0 = grp * kPG;
  int n[kPG];
  int nmax = 0, safe = 0;
#pragma unroll
  for (int q = 0; q < kPG; ++q) {
    n[q] = L.ns[p0 + q];
    if (n[q] > nmax) {
      nmax = n[q];
      safe = static_cast<int>(v.sorted_gid[s_sel_pos[(p0 + q) * KP]]);
    }
  }
  for (int c = lane; c < dim4; c += 64) {
    float4 acc[kPG];
#pragma unroll
    for (int q = 0; q < kPG; ++q) acc[q] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int j = 0; j < nmax; ++j) {
      float4 f[kPG];
      float w[kPG];
#pragma unroll
      for (int q = 0; q < kPG; ++q) {
        const bool ok = j < n[q];
        const int g = ok ? static_cast<int>(v.sorted_gid[s_sel_pos[(p0 + q) * KP + j]]) : safe;
        w[q] = ok ? s_sel_w[(p0 + q) * KP + j] : 0.f;
        f[q] = load_feat4_global<DT>(v.feats, v.scale, g, dim, 4 * c);
      }
#pragma unroll
      for (int q = 0; q < kPG; ++q) {
        acc[q].x += w[q] * f[q].x;
        acc[q].y += w[q] * f[q].y;
        acc[q].z += w[q] * f[q].z;
        acc[q].w += w[q] * f[q].w;
      }
    }
#pragma unroll
    for (int q = 0; q < kPG; ++q) {
      if (n[q] < 0) continue;  // outside the image
      const int p = p0 + q;
      const int gx = tx * kTile + (p % kTile), gy = ty * kTile + (p / kTile);
      const float inv = L.inv[p];
      store_out4<OT>(v.out, static_cast<int64_t>(gy) * v.W + gx, dim, c,
                     make_float4(acc[q].x * inv, acc[q].y * inv, acc[q].z * inv, acc[q].w * inv));
    }
  }
}

// A tile's place and the calling thread's pixel.
struct TilePixel {
  int tx, ty, px, py;
  bool inside;
  __device__ TilePixel(const GView& v, int tile) {
    const int tiles_x = (v.W + kTile - 1) / kTile;
    tx = tile % tiles_x;
    ty = tile / tiles_x;
    px = tx * kTile + static_cast<int>(threadIdx.x % kTile);
    py = ty * kTile + static_cast<int>(threadIdx.x / kTile);
    inside = px < v.W && py < v.H;
  }
};

// Top-K for every pixel of one tile: walk, merge, gather-blend. Called by all
// 256 threads of the workgroup. K selections of each pixel in LDS.
template <int DT, int OT, int UCAP>
__device__ __forceinline__ void topk_tile(const GView& v, int tile, int K, int dim, const qr_params& prm,
                                          TopkLds<UCAP>& L, unsigned char* __restrict__ dyn_lds,
                                          int32_t* __restrict__ sel_gid_out, float* __restrict__ sel_w_out) {
  const int tid = threadIdx.x;
  const TilePixel t(v, tile);
  const int tx = t.tx, ty = t.ty;
  const int KP = (K + 3) & ~3;  // selection row stride: 16-byte aligned rows
  int* const s_sel_pos = reinterpret_cast<int*>(dyn_lds);                 // [256][KP], tile-list positions
  float* const s_sel_w = reinterpret_cast<float*>(dyn_lds) + kTilePix * KP;  // [256][KP]
  ListSink sink{s_sel_pos + tid * KP, s_sel_w + tid * KP};
  WalkState walk;
  const int lo = static_cast<int>(v.tile_offsets[tile]), hi = static_cast<int>(v.tile_offsets[tile + 1]);
  const PixelSel sel = quantile_walk<QR_SELECT_TOPK, false>(v, lo, lo, hi, K, t.px + 0.5f, t.py + 0.5f, t.inside,
                                                            prm, L, sink, walk);
  L.ns[tid] = t.inside ? sel.ns : -1;
  L.inv[tid] = sel.inv;
  wave_lds_sync();
  merge_groups(v, L, s_sel_pos, s_sel_w, KP);
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int g0 = wave * kWaveGroups;
  if (dim <= 128) {
    gather_groups_narrow<DT, OT>(v, &L.ugid[g0 * UCAP], &L.uw[g0 * UCAP], &L.umask[g0 * UCAP],
                                 [](int g) { return g * UCAP; },
                                 [&](int g) { return L.unum[g0 + g]; }, wave, tx, ty, lane, dim);
    gather_groups_narrow_overflow<DT, OT>(v, L, s_sel_pos, s_sel_w, KP, K, wave, tx, ty, lane, dim);
  } else {
    for (int gl = 0; gl < kWaveGroups; ++gl) {
      const int grp = g0 + gl;
      const int nu = __builtin_amdgcn_readfirstlane(L.unum[grp]);
      if (nu >= 0)
        gather_group<DT, OT>(v, &L.ugid[grp * UCAP], &L.uw[grp * UCAP], &L.umask[grp * UCAP], grp * kPG, nu,
                             tx, ty, lane, dim);
      else  // more distinct selections than the merge capacity (rare)
        gather_group_per_pixel<DT, OT>(v, L, s_sel_pos, s_sel_w, KP, grp, tx, ty, lane, dim);
    }
  }
  // Per-pixel outputs last: a load issued after a store waits for it, so no
  // store precedes the loads of the merge and the gather.
  if (t.inside) {
    const int pix = t.py * v.W + t.px;
    if (v.T_q) v.T_q[pix] = sel.TQ;
    if (v.n_sel) v.n_sel[pix] = sel.ns;
    if (sel_gid_out) {
      for (int j = 0; j < K; ++j) {
        sel_gid_out[static_cast<int64_t>(pix) * K + j] =
            j < sel.ns ? static_cast<int>(v.sorted_gid[sink.my_pos[j]]) : -1;
        sel_w_out[static_cast<int64_t>(pix) * K + j] = j < sel.ns ? sink.my_w[j] : 0.f;
      }
    }
  }
}

// Algorithm 1 (or Stratified-K) for every pixel of one tile, then the
// gather-blend of the selected rows. Called by all 256 threads of the
// workgroup. Workgroup barriers occur only around the staging of record
// batches; everything after the walk is wave-local. Shared LDS (the record
// batch) is only rewritten after a barrier that every wave reaches once it has
// finished the previous tile.
// kParts: groups past the capacity are taken in parts, which the map holds
// until the last: the sums of a group's entries so far, then 1 / (1 - T^Q) with
// the rest (float32 maps; with K <= 8 no group can get there). Each part's walk
// goes on where the one before paused, so all parts together walk the list
// about once. Otherwise (bfloat16 maps, which cannot hold the sums) they are
// collected again from the start, as many as fit the wave's space in a further
// walk. (3M pixel-sized, faint Gaussians in a 640x480 view, K = 16, most groups
// past the capacity: 16 columns 4,830 us in further walks for two groups of a
// wave each, 1,200 in parts, bfloat16 2,190; 512 columns 4,980, 2,100 and 2,730.)
template <int DT, int OT, int MODE, bool kParts>
__device__ __forceinline__ void quantile_tile(const GView& v, int tile, int K, int dim,
                                              const qr_params& prm, QuantileLds& L,
                                              int32_t* __restrict__ sel_gid_out,
                                              float* __restrict__ sel_w_out,
                                              float* __restrict__ T_final_out,
                                              int32_t* __restrict__ last_pos_out) {
  const int tid = threadIdx.x;
  const TilePixel t(v, tile);
  const int tx = t.tx, ty = t.ty;
  const float pxc = t.px + 0.5f, pyc = t.py + 0.5f;
  const int lo = static_cast<int>(v.tile_offsets[tile]);
  const int hi = static_cast<int>(v.tile_offsets[tile + 1]);
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // the wave's entries, and the lane's group among its sixteen
  float4* const uw = L.uw + wave * kWaveCap;
  int* const ug = L.ugid + wave * kWaveCap;
  uint8_t* const um = L.umask + wave * kWaveCap;
  const int lg = lane >> 2, q = lane & 3;
  const int64_t sel_at = t.inside && sel_gid_out ? static_cast<int64_t>(t.py * v.W + t.px) * K : -1;
  const auto sink_at = [&](int first, int cap) {
    return GroupSink<kParts>{reinterpret_cast<float*>(uw + first) + q, ug + first, um + first, L.gid, cap};
  };
  const auto selections_to = [&](GroupSink<kParts>& sink) {
    if (sel_at >= 0) {
      sink.pos_out = sel_gid_out + sel_at;
      sink.w_out = sel_w_out + sel_at;
    }
  };
  // the weights over 1 - T^Q, each lane its pixel's
  const auto scale_weights = [&](GroupSink<kParts>& sink, int n, float inv) {
    for (int e = 0; e < n; ++e) sink.uw[kPG * e] *= inv;
    wave_lds_sync();
  };
  const auto own_first = [](int g) { return g * kGroupCap; };
  WalkState walk;
  auto sink = sink_at(own_first(lg), kGroupCap);
  selections_to(sink);
  quantile_walk<MODE, false>(v, lo, lo, hi, K, pxc, pyc, t.inside, prm, L, sink, walk);
  // the lane's group goes on (of a group's pixels, some may have ended)
  const auto group_paused = [&]() {
    return ((wave_ballot(walk.from != kWalkDone) >> (lane & 60)) & 15ull) != 0ull;
  };
  const auto pixel_inv = [&]() { return sink.ns > 0 ? 1.f / (1.f - walk.TQ) : 0.f; };
  bool paused = group_paused();
  scale_weights(sink, min(sink.cnt, kGroupCap), paused ? 1.f : pixel_inv());
  if (dim <= 128) {
    gather_groups_narrow<DT, OT>(v, ug, uw, um, own_first,
                                 [&](int g) {
                                   const int n = __shfl(sink.cnt, 4 * g, 64);
                                   return n > kGroupCap ? -1 : n;
                                 },
                                 wave, tx, ty, lane, dim);
  } else {
    for (int g = 0; g < kWaveGroups; ++g) {
      const int nu = __builtin_amdgcn_readlane(sink.cnt, 4 * g);
      if (nu <= kGroupCap)
        gather_group<DT, OT>(v, ug + own_first(g), uw + own_first(g), um + own_first(g),
                             (wave * kWaveGroups + g) * kPG, nu, tx, ty, lane, dim);
    }
  }
  if constexpr (kParts) {
    for (;;) {
      if (tid == 0) L.go_on = kWalkDone;
      if (!__syncthreads_or(paused)) break;
      int from = walk.from;
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) from = min(from, __shfl_xor(from, off, 64));
      if (lane == 0) atomicMin(&L.go_on, from);
      __syncthreads();
      const bool open = paused;
      sink.cnt = 0;
      quantile_walk<MODE, true>(v, lo, __builtin_amdgcn_readfirstlane(L.go_on), hi, K, pxc, pyc, t.inside, prm, L,
                                sink, walk);
      paused = group_paused();
      const float scale = paused ? 1.f : pixel_inv();
      wave_lds_sync();
      if (dim <= 128) {
        const int n = open ? sink.cnt : -1;
        gather_groups_narrow<DT, OT, true>(v, ug, uw, um, own_first, [&](int g) { return __shfl(n, 4 * g, 64); },
                                           wave, tx, ty, lane, dim, [&](int p) { return __shfl(scale, p, 64); });
      } else {
        for (uint64_t todo = wave_ballot(open) & 0x1111111111111111ull; todo; todo &= todo - 1ull) {
          const int l = __builtin_ctzll(todo), first = own_first(l >> 2);
          gather_group<DT, OT, true>(v, ug + first, uw + first, um + first, wave * 64 + l,
                                     __builtin_amdgcn_readlane(sink.cnt, l), tx, ty, lane, dim, [&](int p) {
                                       return __int_as_float(
                                           __builtin_amdgcn_readlane(__float_as_int(scale), l + p));
                                     });
        }
      }
    }
  } else if (kPG * K > kGroupCap) {
    // as many groups as fit the wave's space, per further walk
    const int cnt = sink.cnt;
    uint64_t redo = wave_ballot(cnt > kGroupCap) & 0x1111111111111111ull;
    while (__syncthreads_or(redo != 0ull)) {
      uint64_t take = 0ull;
      int used = 0, first = 0;
      while (redo) {
        const int l = __builtin_ctzll(redo), n = __builtin_amdgcn_readlane(cnt, l);
        if (used + n > kWaveCap) break;
        if (lg == l >> 2) first = used;
        used += n;
        take |= 15ull << l;
        redo &= redo - 1ull;
      }
      const bool mine = in_mask(take);
      auto again = sink_at(first, mine ? cnt : 0);
      WalkState fresh;
      const PixelSel s =
          quantile_walk<MODE, false>(v, lo, lo, hi, K, pxc, pyc, t.inside && mine, prm, L, again, fresh);
      scale_weights(again, mine ? cnt : 0, s.inv);
      if (dim <= 128) {
        const int n = mine ? cnt : -1;
        gather_groups_narrow<DT, OT>(v, ug, uw, um, [&](int g) { return __shfl(first, 4 * g, 64); },
                                     [&](int g) { return __shfl(n, 4 * g, 64); }, wave, tx, ty, lane, dim);
      } else {
        for (uint64_t todo = take & 0x1111111111111111ull; todo; todo &= todo - 1ull) {
          const int l = __builtin_ctzll(todo), f = __builtin_amdgcn_readlane(first, l);
          gather_group<DT, OT>(v, ug + f, uw + f, um + f, wave * 64 + l, __builtin_amdgcn_readlane(cnt, l), tx, ty,
                               lane, dim);
        }
      }
    }
  }
  // Per-pixel outputs last: a load issued after a store waits for it, so no
  // store precedes the loads of the gather.
  if (t.inside) {
    const int pix = t.py * v.W + t.px;
    if (v.T_q) v.T_q[pix] = walk.TQ;
    if (v.n_sel) v.n_sel[pix] = sink.ns;
    if (T_final_out) T_final_out[pix] = walk.T;
    if (last_pos_out) last_pos_out[pix] = walk.last;
    if (sel_gid_out) {
      // the walk has left list positions and weights
      for (int j = 0; j < K; ++j) {
        const int64_t at = static_cast<int64_t>(pix) * K + j;
        sel_gid_out[at] = j < sink.ns ? static_cast<int>(v.sorted_gid[sel_gid_out[at]]) : -1;
        if (j >= sink.ns) sel_w_out[at] = 0.f;
      }
    }
  }
}

// LDS and tile function by selection rule. UCAP: Top-K's merge capacity; for
// the other rules kUCapLarge for groups taken in parts. (The walk that can pause
// takes 2% longer: 16 float32 columns, one 640x480 view of 200k Gaussians, K = 8,
// 57 and 58 us. So K <= 8, whose groups cannot overfill, keep the one that cannot.)
template <int MODE, int UCAP>
using TileLds = std::conditional_t<MODE == QR_SELECT_TOPK, TopkLds<UCAP>, QuantileLds>;

template <int DT, int OT, int MODE, int UCAP>
__device__ __forceinline__ void render_tile(const GView& v, int tile, int K, int dim, const qr_params& prm,
                                            TileLds<MODE, UCAP>& L, unsigned char* __restrict__ dyn_lds,
                                            int32_t* __restrict__ sel_gid_out, float* __restrict__ sel_w_out,
                                            float* __restrict__ T_final_out, int32_t* __restrict__ last_pos_out) {
  if constexpr (MODE == QR_SELECT_TOPK)
    topk_tile<DT, OT, UCAP>(v, tile, K, dim, prm, L, dyn_lds, sel_gid_out, sel_w_out);
  else
    quantile_tile<DT, OT, MODE, UCAP == kUCapLarge>(v, tile, K, dim, prm, L, sel_gid_out, sel_w_out, T_final_out,
                                                    last_pos_out);
}

template <int DT, int OT, int MODE, int UCAP>
__global__ void __launch_bounds__(kTilePix, kWavesPerSimd)
render_quantile_kernel(ViewArgs v, int n_tiles, qr_params prm, int K, int dim,
                       int32_t* __restrict__ sel_gid_out, float* __restrict__ sel_w_out,
                       float* __restrict__ T_final_out, int32_t* __restrict__ last_pos_out) {
  extern __shared__ unsigned char dyn_lds[];
  __shared__ TileLds<MODE, UCAP> L;
  render_tile<DT, OT, MODE, UCAP>(to_global(v), xcd_remap(blockIdx.x, n_tiles), K, dim, prm, L, dyn_lds,
                                  sel_gid_out, sel_w_out, T_final_out, last_pos_out);
}

// Many views in one persistent launch. The schedule is cut into one
// contiguous range per XCD (workgroup b runs on XCD b % 8), each with its own
// atomic counter: a workgroup takes items of its XCD's range in order, so the
// tiles in flight on an XCD are neighbours whose records and feature rows
// share that XCD's L2; once its range is used up it takes items from the
// other ranges, and it leaves when every range is used up.
constexpr int kXcdQueues = 8;

__device__ __forceinline__ uint32_t queue_begin(int64_t n_items, int q) {
  return static_cast<uint32_t>(n_items * q / kXcdQueues);
}

template <int DT, int OT, int MODE, int UCAP>
__global__ void __launch_bounds__(kTilePix, kWavesPerSimd)
render_quantile_batched_kernel(const qr_view* __restrict__ views, const uint32_t* __restrict__ schedule,
                               int64_t n_items, uint32_t* __restrict__ counter, qr_params prm,
                               int K, int dim) {
  extern __shared__ unsigned char dyn_lds[];
  __shared__ TileLds<MODE, UCAP> L;
  __shared__ uint32_t s_item[2];
  // The item slot alternates between two words: a wave that runs ahead into
  // the next iteration writes the other word, and cannot come back to this
  // one before every wave has passed the next barrier (and so has read it).
  const int home = static_cast<int>(blockIdx.x % kXcdQueues);
  for (int it = 0;; it ^= 1) {
    if (threadIdx.x == 0) {
      uint32_t item = 0xFFFFFFFFu;  // none left
      for (int d = 0; d < kXcdQueues; ++d) {
        const int q = (home + d) % kXcdQueues;
        const uint32_t b = queue_begin(n_items, q), e = queue_begin(n_items, q + 1);
        if (b == e) continue;
        const uint32_t i = atomicAdd(&counter[q], 1u);
        if (i < e - b) {
          item = b + i;
          break;
        }
      }
      s_item[it] = item;
    }
    __syncthreads();
    // uniform values: view records and tile indices stay in scalar registers
    const uint32_t item = __builtin_amdgcn_readfirstlane(s_item[it]);
    if (item >= n_items) break;
    const uint32_t packed = __builtin_amdgcn_readfirstlane(schedule[item]);
    const GView v = to_global(view_args(views[packed >> kViewShift]));
    render_tile<DT, OT, MODE, UCAP>(v, static_cast<int>(packed & kTileMask), K, dim, prm, L, dyn_lds, nullptr,
                                    nullptr, nullptr, nullptr);
  }
}

// Many views in one launch, one workgroup per (view, tile) item. Items are
// dealt to the XCDs in contiguous runs of the schedule (neighbouring tiles of
// a view share L2 contents); workgroups retire as they finish, so work on
// other streams can take their slots.
template <int DT, int OT, int MODE, int UCAP>
__global__ void __launch_bounds__(kTilePix, kWavesPerSimd)
render_quantile_batched_grid_kernel(const qr_view* __restrict__ views,
                                    const uint32_t* __restrict__ schedule, int n_items,
                                    qr_params prm, int K, int dim) {
  extern __shared__ unsigned char dyn_lds[];
  __shared__ TileLds<MODE, UCAP> L;
  const uint32_t packed = __builtin_amdgcn_readfirstlane(schedule[xcd_remap(blockIdx.x, n_items)]);
  const GView v = to_global(view_args(views[packed >> kViewShift]));
  render_tile<DT, OT, MODE, UCAP>(v, static_cast<int>(packed & kTileMask), K, dim, prm, L, dyn_lds, nullptr,
                                  nullptr, nullptr, nullptr);
}

__global__ void reset_counter_kernel(uint32_t* __restrict__ c) {
  if (threadIdx.x < kXcdQueues) c[threadIdx.x] = 0u;
}

}  // namespace qr

using namespace qr;

// Instantiates QR_LAUNCH(feature dtype, output dtype, selection rule, UCAP) for
// the runtime values; Top-K's larger merge capacity is built for float32 maps
// (bfloat16 maps keep 16, which is correct at any K).
#define QR_DISPATCH_DT(dt, OT, SM, UC)                        \
  switch (dt) {                                               \
    case QR_F32: QR_LAUNCH(QR_F32, OT, SM, UC); break;        \
    case QR_BF16: QR_LAUNCH(QR_BF16, OT, SM, UC); break;      \
    default: QR_LAUNCH(QR_FP8_E4M3, OT, SM, UC); break;       \
  }
#define QR_DISPATCH_OT(dt, ot, SM, UC)                        \
  do {                                                        \
    if ((ot) == QR_BF16) { QR_DISPATCH_DT(dt, QR_BF16, SM, UC) } \
    else { QR_DISPATCH_DT(dt, QR_F32, SM, UC) }               \
  } while (0)
#define QR_DISPATCH_K(dt, ot, SM, K)                                                             \
  do {                                                                                           \
    if ((ot) != QR_BF16 && kPG * (K) > kGroupCap) { QR_DISPATCH_DT(dt, QR_F32, SM, kUCapLarge) } \
    else { QR_DISPATCH_OT(dt, ot, SM, kUCap); }                                                  \
  } while (0)
#define QR_DISPATCH(dt, ot, sm, K)                                                          \
  do {                                                                                      \
    if ((sm) == QR_SELECT_TOPK) {                                                           \
      if ((ot) != QR_BF16 && ucap_for(K) == kUCapLarge) {                                   \
        QR_DISPATCH_DT(dt, QR_F32, QR_SELECT_TOPK, kUCapLarge)                              \
      } else {                                                                              \
        QR_DISPATCH_OT(dt, ot, QR_SELECT_TOPK, kUCap);                                      \
      }                                                                                     \
    } else if ((sm) == QR_SELECT_STRATIFIED) {                                              \
      QR_DISPATCH_K(dt, ot, QR_SELECT_STRATIFIED, K);                                       \
    } else {                                                                                \
      QR_DISPATCH_K(dt, ot, QR_SELECT_QUANTILE, K);                                         \
    }                                                                                       \
  } while (0)

// Dynamic LDS: Top-K's selection lists.
static size_t list_bytes(int32_t selection, int32_t K) {
  return selection == QR_SELECT_TOPK ? static_cast<size_t>(kTilePix) * ((K + 3) & ~3) * (sizeof(int) + sizeof(float))
                                     : 0;
}

extern "C" int qr_render_quantile(void* stream, int32_t width, int32_t height,
                                  const qr_params* prm, int32_t K, const uint32_t* tile_offsets,
                                  const uint32_t* sorted_gid, const float* means2d,
                                  const float* conic_opacity, const void* features, int32_t dtype,
                                  const float* feature_scale, int32_t dim, float* out, float* T_q,
                                  int32_t* n_sel, float* T_final, int32_t* last_pos,
                                  int32_t* sel_gid, float* sel_w) {
  int rc = validate_render("qr_render_quantile", width, height, prm, tile_offsets, sorted_gid,
                           means2d, conic_opacity, features, dtype, feature_scale, dim, out);
  if (rc != QR_OK) return rc;
  if (K < 1 || K > QR_MAX_K)
    return fail(QR_ERR_UNSUPPORTED, "qr_render_quantile: K = %d outside [1, %d]", K, QR_MAX_K);
  if ((sel_gid == nullptr) != (sel_w == nullptr))
    return fail(QR_ERR_INVALID_ARG, "qr_render_quantile: sel_gid and sel_w must both be given or both NULL");
  if ((T_final || last_pos) && prm->selection != QR_SELECT_QUANTILE)
    return fail(QR_ERR_UNSUPPORTED, "qr_render_quantile: T_final and last_pos are Algorithm 1's; "
                "pass NULL with another selection rule");
  const int tiles_x = static_cast<int>(ceil_div(width, kTile));
  const int tiles_y = static_cast<int>(ceil_div(height, kTile));
  const int n_tiles = tiles_x * tiles_y;
  (void)tiles_x;
  const size_t lds = list_bytes(prm->selection, K);
  hipStream_t s = as_stream(stream);
  const ViewArgs v{width, height, tile_offsets, sorted_gid, reinterpret_cast<const float2*>(means2d),
                   reinterpret_cast<const float4*>(conic_opacity), features, feature_scale, out, T_q,
                   n_sel};
#define QR_LAUNCH(DT, OT, SM, UC)                                                                     \
  hipLaunchKernelGGL((render_quantile_kernel<DT, OT, SM, UC>), dim3(n_tiles), dim3(kTilePix), lds, s, v, \
                     n_tiles, *prm, K, dim, sel_gid, sel_w, T_final, last_pos)
  QR_DISPATCH(dtype, prm->out_dtype, prm->selection, K);
#undef QR_LAUNCH
  return check_launch("qr_render_quantile");
}

extern "C" int qr_render_quantile_batched(void* stream, int32_t n_views, const qr_view* views,
                                          const qr_params* prm, int32_t K, int32_t dtype,
                                          int32_t dim, const uint32_t* schedule, int64_t n_items,
                                          int32_t n_workgroups, void* workspace,
                                          size_t workspace_bytes) {
  if (n_views <= 0 || n_views > (1 << (32 - kViewShift)))
    return fail(QR_ERR_INVALID_ARG, "qr_render_quantile_batched: n_views = %d out of range", n_views);
  if (!views || !schedule || !prm)
    return fail(QR_ERR_INVALID_ARG, "qr_render_quantile_batched: null pointer");
  if (n_workgroups < 0) return fail(QR_ERR_INVALID_ARG, "qr_render_quantile_batched: n_workgroups < 0");
  if (n_workgroups > 0 && (!workspace || workspace_bytes < kXcdQueues * sizeof(uint32_t)))
    return fail(QR_ERR_CAPACITY, "qr_render_quantile_batched: persistent mode needs a %d-byte workspace",
                static_cast<int>(kXcdQueues * sizeof(uint32_t)));
  if (n_items < 0 || n_items >= (1ll << 31))
    return fail(QR_ERR_INVALID_ARG, "qr_render_quantile_batched: bad item count");
  if (K < 1 || K > QR_MAX_K)
    return fail(QR_ERR_UNSUPPORTED, "qr_render_quantile_batched: K = %d outside [1, %d]", K, QR_MAX_K);
  if (dtype != QR_F32 && dtype != QR_BF16 && dtype != QR_FP8_E4M3)
    return fail(QR_ERR_UNSUPPORTED, "qr_render_quantile_batched: unknown dtype %d", dtype);
  if (dim <= 0 || dim % 16 != 0 || dim > QR_MAX_DIM)
    return fail(QR_ERR_UNSUPPORTED, "qr_render_quantile_batched: dim = %d", dim);
  if (!(prm->alpha_min > 0.f) || !(prm->alpha_max >= prm->alpha_min) || !(prm->alpha_max < 1.f))
    return fail(QR_ERR_INVALID_ARG, "qr_render_quantile_batched: need 0 < alpha_min <= alpha_max < 1");
  if (prm->out_dtype != QR_F32 && prm->out_dtype != QR_BF16)
    return fail(QR_ERR_UNSUPPORTED, "qr_render_quantile_batched: unknown output dtype %d", prm->out_dtype);
  if (prm->selection != QR_SELECT_QUANTILE && prm->selection != QR_SELECT_STRATIFIED &&
      prm->selection != QR_SELECT_TOPK)
    return fail(QR_ERR_UNSUPPORTED, "qr_render_quantile_batched: unknown selection rule %d", prm->selection);
  if (n_items == 0) return QR_OK;
  hipStream_t s = as_stream(stream);
  const size_t lds = list_bytes(prm->selection, K);
  if (n_workgroups == 0) {
    const int ni = static_cast<int>(n_items);
#define QR_LAUNCH(DT, OT, SM, UC)                                                                     \
  hipLaunchKernelGGL((render_quantile_batched_grid_kernel<DT, OT, SM, UC>), dim3(ni), dim3(kTilePix), lds, \
                     s, views, schedule, ni, *prm, K, dim)
    QR_DISPATCH(dtype, prm->out_dtype, prm->selection, K);
#undef QR_LAUNCH
    return check_launch("qr_render_quantile_batched");
  }
  auto* counter = static_cast<uint32_t*>(workspace);
  hipLaunchKernelGGL(reset_counter_kernel, dim3(1), dim3(64), 0, s, counter);
#define QR_LAUNCH(DT, OT, SM, UC)                                                                     \
  hipLaunchKernelGGL((render_quantile_batched_kernel<DT, OT, SM, UC>), dim3(n_workgroups), dim3(kTilePix), \
                     lds, s, views, schedule, n_items, counter, *prm, K, dim)
  QR_DISPATCH(dtype, prm->out_dtype, prm->selection, K);
#undef QR_LAUNCH
  return check_launch("qr_render_quantile_batched");
}

// Selection phase of Quantile Rendering (Algorithm 1, Sec. 4.2) for one
// 16x16 tile, shared by the forward renderer and its backward pass so that
// both make exactly the same selections:
//  - the walk: the tile's depth-sorted list is staged into LDS in batches of
//    256 projected records and every pixel (one thread each) runs the
//    transmittance chain T_test = T (1 - alpha') with the threshold test
//    T_test < t_{k+1}; a pixel is done once all K thresholds are consumed (the
//    same event as the stop test T_test < 1/(K+1)) and the workgroup leaves
//    the list once every pixel is done. What becomes of a selection (weight
//    w^Q = T^Q alpha') is up to a sink:
//     - ListSink: each pixel's selected list positions and weights (the
//       backward, and the Top-K sampler, which replaces entries);
//     - GroupSink: the distinct selections of each group of four adjacent
//       pixels (a row segment of the tile, four neighbouring lanes), in list
//       order, each with the four pixels' weights (0 where a pixel did not
//       select it) and a mask of the pixels that did: what the forward gathers;
//  - the merge (Top-K): the four pixels' lists of each group are merged into
//    the same form.
//    The pixels of wave w are tile rows 4w .. 4w+3, exactly the pixels of the
//    groups it merges, so everything after the walk is wave-local.
#pragma once

#include "common.h"
#include "render_common.h"

namespace qr {

constexpr int kViewShift = QR_BATCH_TILE_BITS;
constexpr uint32_t kTileMask = (1u << QR_BATCH_TILE_BITS) - 1u;

constexpr int kPG = 4;                     // pixels gathered together
constexpr int kGroups = kTilePix / kPG;    // 64 pixel groups per tile
// Distinct selections kept per merged Top-K group: 16, or 32 for 24 < K <=
// 52, where the selection lists already hold the kernel to one workgroup per
// CU.
constexpr int kUCap = 16;
constexpr int kUCapLarge = 32;
constexpr int kUCapLargeMinK = 25;
constexpr int kUCapLargeMaxK = 52;
__host__ __device__ constexpr int ucap_for(int K) {
  return K >= kUCapLargeMinK && K <= kUCapLargeMaxK ? kUCapLarge : kUCap;
}
// Three workgroups fill a CU's LDS: registers are bounded to match (three
// waves per SIMD).
constexpr int kWavesPerSimd = 3;

// LDS of one Top-K workgroup: record staging, per-pixel scalars and
// the merged groups of up to UCAP distinct selections (each pixel's [K]
// selections live in dynamic LDS).
template <int UCAP>
struct TopkLds {
  static constexpr int kCap = UCAP;
  static constexpr bool kKeepIds = false;  // the walk keeps a staged batch's Gaussian ids (in gid)
  float2 mean[kTilePix];
  float4 co[kTilePix];
  float inv[kTilePix];
  int ns[kTilePix];
  int unum[kGroups];                       // distinct entries per group, -1 if over UCAP
  int ugid[kGroups * UCAP];                // a group's distinct selections (list positions until converted)
  float4 uw[kGroups * UCAP];               // their weights for the group's four pixels, x = first pixel
  uint8_t umask[kGroups * UCAP];           // bit q: pixel q of the group selected the entry
};

// LDS of one Q-Render workgroup: record staging, thresholds and the groups'
// distinct selections as the walk collects them. The size does not depend on
// K (the pixels' lists took 8 K bytes each and left room for one workgroup per
// CU at K = 40): three workgroups fit a CU's 160 KB at any K. A group that
// would need more than kGroupCap entries (0.5% of the groups of a room at K =
// 40, none at K = 8; most groups of a scene of pixel-sized, faint Gaussians)
// pauses there, its entries are gathered, and the walk goes on from where the
// first group paused.
constexpr int kGroupCap = 32;
constexpr int kWaveGroups = kGroups / 4;
constexpr int kWaveCap = kWaveGroups * kGroupCap;
static_assert(kWaveCap >= kPG * QR_MAX_K, "a group's selections always fit a wave's space");

struct QuantileLds {
  static constexpr bool kKeepIds = true;
  float2 mean[kTilePix];
  float4 co[kTilePix];
  int gid[kTilePix];
  union {
    float thr[QR_MAX_K + 1];               // t_1 .. t_K, 0
    double zq[QR_MAX_K];                   // Stratified-K: z_m, m = 1..K
  };
  float4 uw[kGroups * kGroupCap];          // weights of the entries for their group's four pixels
  int ugid[kGroups * kGroupCap];           // Gaussian ids
  uint8_t umask[kGroups * kGroupCap];      // bit q: pixel q of the group selected the entry
  int go_on;                               // list position where the next walk starts
};
static_assert(3 * ((sizeof(QuantileLds) + 64 + 1279) / 1280) * 1280 <= 160 * 1024, "three workgroups per CU");

struct ViewArgs {
  int W, H;
  const uint32_t* __restrict__ tile_offsets;
  const uint32_t* __restrict__ sorted_gid;
  const float2* __restrict__ means2d;
  const float4* __restrict__ conic_opacity;
  const void* __restrict__ feats;
  const float* __restrict__ scale;
  float* __restrict__ out;
  float* __restrict__ T_q;
  int32_t* __restrict__ n_sel;
};

// The same view with global-memory pointers (see QR_GLOBAL), as the tile
// code uses it.
struct GView {
  int W, H;
  const QR_GLOBAL uint32_t* __restrict__ tile_offsets;
  const QR_GLOBAL uint32_t* __restrict__ sorted_gid;
  const QR_GLOBAL f32x2* __restrict__ means2d;
  const QR_GLOBAL f32x4* __restrict__ conic_opacity;
  const QR_GLOBAL void* __restrict__ feats;
  const QR_GLOBAL float* __restrict__ scale;
  QR_GLOBAL float* __restrict__ out;
  QR_GLOBAL float* __restrict__ T_q;
  QR_GLOBAL int32_t* __restrict__ n_sel;
};

__device__ __forceinline__ GView to_global(const ViewArgs& v) {
  return GView{v.W, v.H,
               (const QR_GLOBAL uint32_t*)v.tile_offsets, (const QR_GLOBAL uint32_t*)v.sorted_gid,
               (const QR_GLOBAL f32x2*)v.means2d, (const QR_GLOBAL f32x4*)v.conic_opacity,
               (const QR_GLOBAL void*)v.feats, (const QR_GLOBAL float*)v.scale,
               (QR_GLOBAL float*)v.out, (QR_GLOBAL float*)v.T_q, (QR_GLOBAL int32_t*)v.n_sel};
}

// Orders this wave's LDS writes before its later LDS reads (all lanes).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ ViewArgs view_args(const qr_view& qv) {
  return ViewArgs{qv.width, qv.height, qv.tile_offsets, qv.sorted_gid,
                  reinterpret_cast<const float2*>(qv.means2d),
                  reinterpret_cast<const float4*>(qv.conic_opacity), qv.features,
                  qv.feature_scale, qv.out, qv.T_q, qv.n_sel};
}

// A pixel's walk between two passes over the list.
constexpr int kWalkDone = 0x7fffffff;
struct WalkState {
  float T = 1.f, TQ = 1.f;
  int k = 0, last = 0;
  int from = kWalkDone;  // the entry it goes on from, kWalkDone: none
  double mu = 0.0, sigma = 0.0;  // Stratified-K
};

// What the walk leaves in registers for the calling thread's pixel.
struct PixelSel {
  int ns;    // selections (0 outside the image)
  float TQ;  // T^Q after the last selection
  float T;   // Algorithm 1: full transmittance when the walk ends (the stop
             // test breaks before T takes the stopping entry's T_test)
  int last;  // Algorithm 1: list position + 1 of the last on-ray entry examined
  int staged;  // list position where the last staged batch of 256 records starts (uniform)
  float inv;   // 1 / (1 - T^Q) (Top-K: 1 / sum of the kept weights); 0 if nothing was selected
};

// Each pixel's selections, in list order: absolute positions in sorted_gid
// and w^Q.
struct ListSink {
  int* __restrict__ my_pos;
  float* __restrict__ my_w;
  int ns = 0;
  static constexpr bool kPauses = false;
  // sel: lane mask of the pixels that selected list position pos
  __device__ __forceinline__ void add(uint64_t sel, float w, int pos, int) {
    if (!__builtin_amdgcn_inverse_ballot_w64(sel)) return;
    my_pos[ns] = pos;
    my_w[ns] = w;
    ++ns;
  }
};

// The distinct selections of the lane's group of four pixels. Called with
// all lanes of the wave (the four lanes of a group count alike). Entries past
// the capacity are counted and not kept; kPause: the walk lets a full group
// pause instead.
template <bool kPause>
struct GroupSink {
  static constexpr bool kPauses = kPause;
  float* __restrict__ uw;        // the lane's pixel's weight of the group's first entry
  int* __restrict__ ugid;
  uint8_t* __restrict__ umask;
  const int* __restrict__ gid;   // ids of the staged batch
  int cap;                       // 0: nothing is kept for this group
  int cnt = 0;
  int ns = 0;
  // the pixel's own selections, for callers that ask for them (or null)
  int32_t* __restrict__ pos_out = nullptr;
  float* __restrict__ w_out = nullptr;
  __device__ __forceinline__ void add(uint64_t cross, float w, int pos, int staged) {
    const int lane = threadIdx.x & 63;
    const bool sel = __builtin_amdgcn_inverse_ballot_w64(cross);
    const uint32_t m = static_cast<uint32_t>(cross >> (lane & 60)) & 15u;
    if (m != 0u) {
      if (cnt < cap) {
        uw[kPG * cnt] = sel ? w : 0.f;
        if ((lane & 3) == 0) {
          ugid[cnt] = gid[staged];
          umask[cnt] = static_cast<uint8_t>(m);
        }
      }
      ++cnt;
    }
    if (sel) {
      if (pos_out) {
        pos_out[ns] = pos;
        w_out[ns] = w;
      }
      ++ns;
    }
  }
};

// Most entries of a list miss all 64 pixels of a wave, so the common path is
// kept to the evaluation of o G and one wave-uniform branch: the records are
// staged with 2 b in place of the conic's b (an exact doubling that
// eval_alpha makes itself), and alpha' = min(alpha_max, o G) is formed only if
// some pixel has the entry on its ray (o G >= alpha_min). (11 views of 52x196
// with lists of up to thousands of entries: render 182 -> 156 us; a 64x64
// picture, one workgroup on a few CUs: 67 -> 62 us.)
__device__ __forceinline__ float4 staged_conic(f32x4 c) { return make_float4(c.x, c.y + c.y, c.z, c.w); }
// o G of a staged record, with the float operations of eval_alpha.
__device__ __forceinline__ float staged_oG(float2 mean, float4 co, float pxc, float pyc) {
  const float dx = pxc - mean.x, dy = pyc - mean.y;
  const float cross2 = (co.y * dx) * dy;
  return co.w * gauss_of(fmaf(co.x * dx, dx, fmaf(co.z * dy, dy, cross2)));
}

// Lane masks in scalar registers: which pixels of the wave are still walking,
// have an entry on their ray, cross a threshold. (As per-lane booleans the
// compiler moves them through vector registers for every wave-uniform branch.)
__device__ __forceinline__ uint64_t wave_ballot(bool x) { return __builtin_amdgcn_ballot_w64(x); }
__device__ __forceinline__ bool in_mask(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }
constexpr int kCmpLt = 4, kCmpNotLt = 11;  // a < b; !(a < b)

// The walk for one tile (all 256 threads of the workgroup). Selections go to
// `sink`; L (any LDS struct with the staging arrays mean, co and, by rule, the
// thresholds thr or zq). Workgroup barriers occur only around the staging of
// record batches; the record batch is only rewritten after a barrier that
// every wave reaches once it has finished the previous tile.
// MODE QR_SELECT_QUANTILE: Algorithm 1's thresholds t_m = 1 - m/(K+1).
// MODE QR_SELECT_STRATIFIED (Stratified-K, Appendix): a first pass over the
// list estimates the mean and spread of the ray's transmittance values (T_0 =
// 1 and T after every Gaussian the dense blend composites, with its T_eps
// stop; sums in double) and the thresholds are the ray's own; the second
// pass examines the same Gaussians (it also ends at the dense stop).
// MODE QR_SELECT_TOPK (the Top-K sampler the paper compares with): the
// candidates are the Gaussians the dense blend composites (same T_eps stop),
// each with its dense weight T alpha'; the K largest are kept (equal weights:
// the earlier position), then put back in list order, and T^Q reports 1 -
// their sum (in a ListSink, whose entries it replaces). A pixel is done
// once its list is full and T alpha_max is no larger than the smallest kept
// weight: no later weight can exceed it.
// A group whose sink is full pauses at the next entry on a ray of its pixels:
// their st.from is that entry. (Such groups' thresholds are raised, so that
// entries cross them, and only crossings pay for the check: checked at every
// entry it cost the walk 4%.) kResume: the pixels with such an entry go on from
// there, over the entries from `start` (the first of them) on.
template <int MODE, bool kResume, class WalkLds, class Sink>
__device__ __forceinline__ PixelSel quantile_walk(const GView& v, int lo, int start, int hi, int K, float pxc,
                                                  float pyc, bool inside, const qr_params& prm,
                                                  WalkLds& L, Sink& sink, WalkState& st) {
  const int tid = threadIdx.x;
  // thr[k] = t_{k+1}; thr[K] = 0 (identical for every tile of a launch)
  if constexpr (MODE == QR_SELECT_QUANTILE && !kResume) {
    if (tid <= K) L.thr[tid] = quantile_threshold(tid + 1, K);
  }
  if constexpr (MODE == QR_SELECT_STRATIFIED && !kResume) {
    if (tid < K) L.zq[tid] = stratified_z(tid + 1, K);  // read after the barrier below
    __syncthreads();
  }
  const float amin = prm.alpha_min, amax = prm.alpha_max;
  const auto stage = [&](int batch) {
    const int idx = batch + tid;
    if (tid >= kTilePix) {
      // a workgroup wider than the tile: only its first 256 threads walk
    } else if (idx < hi) {
      const int g = static_cast<int>(v.sorted_gid[idx]);
      if constexpr (WalkLds::kKeepIds) L.gid[tid] = g;
      const f32x2 m = v.means2d[g];
      const f32x4 c = v.conic_opacity[g];
      L.mean[tid] = make_float2(m.x, m.y);
      L.co[tid] = staged_conic(c);
    } else {  // padding record: opacity 0 is below alpha_min on every ray
      L.mean[tid] = make_float2(0.f, 0.f);
      L.co[tid] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    __syncthreads();
  };
  // kU records are read from LDS and evaluated together (one LDS round trip
  // and independent arithmetic per group of records; the padding makes every
  // group whole); touch[u]: pixels with o G >= alpha_min at record u. Returns
  // the mask of the pixels that any of them touches.
  constexpr int kU = 8;
  const auto evaluate = [&](int j, float (&oG)[kU], uint64_t (&touch)[kU]) {
    float2 rm[kU];
    float4 rc[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      rm[u] = L.mean[j + u];
      rc[u] = L.co[j + u];
    }
    uint64_t any = 0ull;
#pragma unroll
    for (int u = 0; u < kU; ++u) oG[u] = staged_oG(rm[u], rc[u], pxc, pyc);
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      touch[u] = __builtin_amdgcn_fcmpf(oG[u], amin, kCmpNotLt);
      any |= touch[u];
    }
    return any;
  };

  double &mu = st.mu, &sigma = st.sigma;
  if constexpr (MODE == QR_SELECT_STRATIFIED && !kResume) {
    double s1 = 1.0, s2 = 1.0;  // T_0 = 1
    int n = 1;
    float T1 = 1.f;
    uint64_t live = wave_ballot(inside);
    for (int batch = lo; batch < hi; batch += kTilePix) {
      if (__syncthreads_or(live != 0ull) == 0) break;
      stage(batch);
      const int cnt_pad = (min(kTilePix, hi - batch) + kU - 1) & ~(kU - 1);
      for (int j = 0; j < cnt_pad; j += kU) {
        if (live == 0ull) break;
        float oG[kU];
        uint64_t touch[kU];
        if ((evaluate(j, oG, touch) & live) == 0ull) continue;
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          const uint64_t on = touch[u] & live;
          if (on == 0ull) continue;
          const float alpha = oG[u] >= amax ? amax : oG[u];
          const float T_test = T1 * (1.f - alpha);
          const uint64_t stop = __builtin_amdgcn_fcmpf(T_test, prm.T_eps, kCmpLt) & on;
          live &= ~stop;
          if (in_mask(on & ~stop)) {
            T1 = T_test;
            s1 += T1;
            s2 += static_cast<double>(T1) * T1;
            ++n;
          }
        }
      }
    }
    mu = s1 / n;
    sigma = sqrt(fmax(s2 / n - mu * mu, 0.0));
  }
  auto threshold = [&](int kk) -> float {  // t_{kk+1}; past t_K none is crossed
    if constexpr (MODE == QR_SELECT_STRATIFIED) return kk < K ? stratified_threshold_z(L.zq[kk], mu, sigma) : -1.f;
    else if constexpr (MODE == QR_SELECT_QUANTILE) return L.thr[kk];
    else return -1.f;  // Top-K has none
  };

  float T = st.T, TQ = st.TQ;
  int k = st.k, last = st.last, staged = start;
  const int from = st.from;
  st.from = kWalkDone;
  uint64_t live = wave_ballot(kResume ? from != kWalkDone : inside);  // pixels whose walk has not ended
  uint64_t full = 0ull;  // lanes of groups whose sink is full
  // t_{k+1}: changes only at a crossing
  float thr_k;
  if constexpr (kResume || MODE == QR_SELECT_STRATIFIED) thr_k = threshold(k);
  else thr_k = quantile_threshold(1, K);
  float wmin = 0.f;  // Top-K: the worst kept entry (smallest weight, later position among equals)
  int imin = 0;

  for (int batch = start; batch < hi; batch += kTilePix) {
    if (__syncthreads_or(live != 0ull) == 0) break;
    staged = batch;
    stage(batch);
    const int cnt_pad = (min(kTilePix, hi - batch) + kU - 1) & ~(kU - 1);
    for (int j = 0; j < cnt_pad; j += kU) {
      if (live == 0ull) break;
      float oG[kU];
      uint64_t touch[kU];
      if ((evaluate(j, oG, touch) & live) == 0ull) continue;
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        uint64_t on = touch[u] & live;  // not finished, and on this pixel's ray
        const int pos = batch + j + u;
        if constexpr (kResume) on &= wave_ballot(pos >= from);
        if (on == 0ull) continue;
        const float alpha = oG[u] >= amax ? amax : oG[u];
        const float T_test = T * (1.f - alpha);
        if constexpr (MODE != QR_SELECT_QUANTILE) {  // the dense blend stops before this Gaussian
          const uint64_t stop = __builtin_amdgcn_fcmpf(T_test, prm.T_eps, kCmpLt) & on;
          live &= ~stop;
          on &= ~stop;
        }
        bool end = false;  // the pixel's walk ends with this entry
        if constexpr (MODE == QR_SELECT_TOPK) {
          int* const my_pos = sink.my_pos;
          float* const my_w = sink.my_w;
          int& ns = sink.ns;
          const float w = T * alpha;
          if (in_mask(on)) {
            if (ns < K) {
              my_pos[ns] = pos;
              my_w[ns] = w;
              if (ns == 0 || w <= wmin) {
                wmin = w;
                imin = ns;
              }
              ++ns;
            } else if (w > wmin) {
              my_pos[imin] = pos;
              my_w[imin] = w;
              int pmin = my_pos[0];
              wmin = my_w[0];
              imin = 0;
              for (int e = 1; e < K; ++e) {
                const float we = my_w[e];
                const int pe = my_pos[e];
                if (we < wmin || (we == wmin && pe > pmin)) {
                  wmin = we;
                  imin = e;
                  pmin = pe;
                }
              }
            }
            T = T_test;
            end = ns == K && T * amax <= wmin;
          }
        } else {
          // a quantile Gaussian of the pixel
          uint64_t cross = __builtin_amdgcn_fcmpf(T_test, thr_k, kCmpLt) & on;
          if constexpr (MODE == QR_SELECT_QUANTILE) last = in_mask(on) ? pos - lo + 1 : last;
          T = in_mask(on & ~cross) ? T_test : T;
          if (cross == 0ull) continue;
          if constexpr (Sink::kPauses) {
            if (__builtin_expect((cross & full) != 0ull, 0)) {
              const uint64_t c = cross & full, c2 = c | (c >> 1);
              const uint64_t pause = ((c2 | (c2 >> 2)) & 0x1111111111111111ull) * 15ull & live;  // whole groups
              cross &= ~pause;
              live &= ~pause;
              st.from = in_mask(pause) ? pos : st.from;
              if (cross == 0ull) continue;
            }
          }
          const float w = TQ * alpha;
          if (in_mask(cross)) {
            TQ = TQ * (1.f - alpha);
            ++k;
            while (k < K && T_test < threshold(k)) ++k;  // thresholds crossed by the same step
            thr_k = threshold(k);
            end = k == K;
            // Algorithm 1 leaves T at the stopping entry (the stop test comes first)
            if (MODE != QR_SELECT_QUANTILE || !end) T = T_test;
          }
          sink.add(cross, w, pos, j + u);
          if constexpr (Sink::kPauses) {
            full = wave_ballot(sink.cnt == sink.cap);
            thr_k = in_mask(full) ? INFINITY : thr_k;  // the group's next entry crosses, and finds it full
          }
        }
        live &= ~wave_ballot(end);
      }
    }
  }
  if constexpr (MODE == QR_SELECT_TOPK) {
    // back to list order (insertion sort of at most K entries), weight sum
    int* const my_pos = sink.my_pos;
    float* const my_w = sink.my_w;
    const int ns = sink.ns;
    for (int a = 1; a < ns; ++a) {
      const int p = my_pos[a];
      const float w = my_w[a];
      int b = a - 1;
      while (b >= 0 && my_pos[b] > p) {
        my_pos[b + 1] = my_pos[b];
        my_w[b + 1] = my_w[b];
        --b;
      }
      my_pos[b + 1] = p;
      my_w[b + 1] = w;
    }
    float sum = 0.f;
    for (int a = 0; a < ns; ++a) sum += my_w[a];
    TQ = 1.f - sum;
    // 1 / sum, of the sum itself
    return PixelSel{ns, TQ, T, last, staged, ns > 0 ? 1.f / sum : 0.f};
  }
  st.T = T;
  st.TQ = TQ;
  st.k = k;
  st.last = last;
  return PixelSel{sink.ns, TQ, T, last, staged, sink.ns > 0 ? 1.f / (1.f - TQ) : 0.f};
}

// The merge for one tile (all 256 threads; wave-local), after the walk.
template <class Lds>
__device__ __forceinline__ void merge_groups(const GView& v, Lds& L,
                                             const int* __restrict__ s_sel_pos,
                                             const float* __restrict__ s_sel_w, int KP) {
  constexpr int kCap = Lds::kCap;
  const int tid = threadIdx.x;
  // The merge, wave-local: adjacent pixels select mostly the same
  // Gaussians, so a group's distinct selections are far fewer than its
  // pixels' selections. Lane l < 16 merges group 16 w + l.
  const int lane = tid & 63;
  const int wave = tid >> 6;
  if (lane < kWaveGroups) {
    const int grp = wave * kWaveGroups + lane;
    const int p0 = grp * kPG;
    // each pixel's next selection (list position and weight) kept in registers
    // (weights are stored already divided by the pixel's 1 - T^Q)
    int n[kPG], idx[kPG], head[kPG];
    float hw[kPG], inv[kPG];
#pragma unroll
    for (int q = 0; q < kPG; ++q) {
      n[q] = max(L.ns[p0 + q], 0);
      inv[q] = L.inv[p0 + q];
      idx[q] = 0;
      head[q] = n[q] > 0 ? s_sel_pos[(p0 + q) * KP] : 0x7fffffff;
      hw[q] = n[q] > 0 ? s_sel_w[(p0 + q) * KP] * inv[q] : 0.f;
    }
    int cnt = 0;
    for (;;) {
      const int best = min(min(head[0], head[1]), min(head[2], head[3]));
      if (best == 0x7fffffff) break;
      if (cnt == kCap) {
        cnt = -1;
        break;
      }
      float wq[kPG];
      uint32_t mk = 0u;
#pragma unroll
      for (int q = 0; q < kPG; ++q) {
        wq[q] = 0.f;
        if (head[q] == best) {
          wq[q] = hw[q];
          mk |= 1u << q;
          ++idx[q];
          head[q] = idx[q] < n[q] ? s_sel_pos[(p0 + q) * KP + idx[q]] : 0x7fffffff;
          hw[q] = idx[q] < n[q] ? s_sel_w[(p0 + q) * KP + idx[q]] * inv[q] : 0.f;
        }
      }
      L.ugid[grp * kCap + cnt] = best;  // position for now
      L.uw[grp * kCap + cnt] = make_float4(wq[0], wq[1], wq[2], wq[3]);
      L.umask[grp * kCap + cnt] = static_cast<uint8_t>(mk);
      ++cnt;
    }
    L.unum[grp] = cnt;
    // positions -> Gaussian ids, 16 at a time: all loads of a batch issued
    // before any result is used
#pragma unroll
    for (int e0 = 0; e0 < kCap; e0 += 16) {
      if (e0 >= cnt) break;
      int pos[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) pos[e] = e0 + e < cnt ? L.ugid[grp * kCap + e0 + e] : -1;
      uint32_t gid[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) gid[e] = pos[e] >= 0 ? v.sorted_gid[pos[e]] : 0u;
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (e0 + e < cnt) L.ugid[grp * kCap + e0 + e] = static_cast<int>(gid[e]);
    }
  }
  wave_lds_sync();
}

}  // namespace qr

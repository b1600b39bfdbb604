// Backward pass of Quantile Rendering (Algorithm 1, Sec. 4.2): gradients
// with respect to the decoded float32 features, the 2D means, the conics
// (a, b, c) and the opacities, given g = dL/d(out) per pixel.
//
// With the selected j of a pixel, w_j = T^Q_j alpha'_j (T^Q_j: T^Q before j),
// Z = 1 - T^Q, out = sum_j w_j f_j / Z and d_j = <g, f_j>:
//    dL/df_j      = (w_j / Z) g
//    dL/dalpha'_j = (T^Q_j d_j - (S_j + <g, out> T^Q) / (1 - alpha'_j)) / Z,
//                   S_j = sum_{l > j} w_l d_l,  <g, out> = sum_j w_j d_j / Z,
// and alpha' = o G, G = exp(-(a dx^2 + 2 b dx dy + c dy^2)/2) gives
//    dalpha'/do = G, dalpha'/dpower = alpha' (0 for both if clamped),
//    dpower/da = -dx^2/2, /db = -dx dy, /dc = -dy^2/2,
//    dpower/du = a dx + b dy, /dv = b dx + c dy.
// The selection itself is piecewise constant and passes no gradient.
//
// One workgroup per tile:
//  1. the selection walk (quantile_select.h, the very code of the forward,
//     so the same Gaussians are selected; nothing per pixel is stored by the
//     forward): each pixel's selected list positions and weights w^Q in LDS.
//     A tile selects a few dozen distinct Gaussians (about 20 at K = 8, 50 at
//     K = 40 on the room scenes, against 1,200 to 2,900 pixel selections):
//     they get slots in list order, and each pixel a mask of the slots that it
//     selected, pass by pass (32 slots in the first, 16 in later ones);
//  2. one stream over dL/d(out) per pass (stream_slots) for both products on
//     v_mfma_f32_16x16x32_bf16: feature gradients dF = W^T G, W[p][s] =
//     w_ps / Z_p, one atomic per (slot, column), and dots D = G F^T, which are
//     written over the weights (so a selection costs 8 bytes of LDS and K up
//     to 64 fits);
//  3. a sweep over each pixel's selections (thread per pixel) recomputes
//     alpha'_j, w_j and T^Q_j from the records with the walk's own float
//     operations and turns the dots into dL/dpower; their moments over the
//     tile's pixels give the geometric gradients of a slot. The tail sums S_j
//     are the total minus the running prefix, both kept in double.
// Both products of step 2 take float32 operands split into bfloat16 pairs
// x = x_hi + x_lo and form hi.hi + hi.lo + lo.hi with float32 accumulation
// (relative error below 2^-16 per product; three parts past a tile's first 32
// slots and past list position 2,048). A value of dL/d(out) that is not finite
// reaches the feature gradients, at its column, of all of the tile's selections
// in the two-part pass, past it of its pixel's alone. Selections without a slot (more
// than 256 distinct selections in a tile, or a position past kPosCap) are
// handled by a plain wave-wide path.
//
// Bound: reading dL/d(out) once (629 MB of a 640x480 frame of 512 features:
// 134 us at the 4.7 TB/s of a large copy) and, beside it, the walk and the
// sweep (90 us on their own) and the feature atomics (30 us of the kernel).
// Measured against two passes over dL/d(out) with 4-byte loads for the
// feature gradients, a slot limit of 32 past which every selection was taken
// on its own, and LDS float atomics for the geometric sums: 500k Gaussians,
// 640x480x512, bf16, K = 8: 640 -> 280 us; 200k, float32, K = 40: 2,400 -> 505
// us; 8 views 1280x720, e4m3, K = 8: 7.01 -> 4.1 ms (3.7 TB/s of dL/d(out)).
#include <type_traits>

#include "quantile_select.h"
#include "wave_ops.h"

namespace qr {

// Gradient outputs of one view (generic pointers, host-constructible).
struct GradPtrs {
  const float* __restrict__ grad_out;
  float* __restrict__ grad_features;
  float* __restrict__ grad_means2d;
  float* __restrict__ grad_co;
};

struct GGrad {
  const QR_GLOBAL float* __restrict__ grad_out;
  QR_GLOBAL float* __restrict__ grad_features;
  QR_GLOBAL float* __restrict__ grad_means2d;
  QR_GLOBAL float* __restrict__ grad_co;
};

__device__ __forceinline__ GGrad to_global(const GradPtrs& g) {
  return GGrad{(const QR_GLOBAL float*)g.grad_out, (QR_GLOBAL float*)g.grad_features,
               (QR_GLOBAL float*)g.grad_means2d, (QR_GLOBAL float*)g.grad_co};
}

__device__ __forceinline__ void atomic_add(QR_GLOBAL float* p, float v) {
  __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Eight consecutive features (columns c .. c+7) of Gaussian g. e4m3 codes are
// decoded without their row's scale: they are then exact as bfloat16, and the
// scale multiplies the finished dots.
template <int DT>
__device__ __forceinline__ void load_feat8(const GView& v, int64_t g, int dim, int c, float (&f)[8]) {
  float4 a, b;
  if constexpr (DT == QR_FP8_E4M3) {
    const u32x2 r = *reinterpret_cast<const QR_GLOBAL u32x2*>(
        static_cast<const QR_GLOBAL uint8_t*>(v.feats) + g * dim + c);
    a = e4m3x4_to_f32(r.x, 1.f);
    b = e4m3x4_to_f32(r.y, 1.f);
  } else {
    a = load_feat4_global<DT>(v.feats, v.scale, g, dim, c);
    b = load_feat4_global<DT>(v.feats, v.scale, g, dim, c + 4);
  }
  f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w;
  f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
}

constexpr int kSlots = 32;       // distinct selections of one pass over dL/d(out) (at most)
constexpr int kMaxSlots = 256;   // distinct selections of a tile given slots
constexpr int kPosCap = 8192;    // list positions covered by the slot bitmap
constexpr int kPosWords = kPosCap / 32;
constexpr int kNearWords = 2048 / 32;  // list positions of the first pass (two-part products)
constexpr int kSub = 32;         // columns of a block (MFMA k of the dots)
constexpr int kPB = 32;          // pixels of a block, two tile rows (MFMA k of the feature gradients)
constexpr int kTS = kSub + 8;    // LDS stride (bf16) of a pixel in the transposing tile
constexpr int kDotStride = kPB + 4;  // LDS stride (float) of a slot's partial dots
static_assert(kPosWords == kTilePix && kMaxSlots == kTilePix, "one bitmap word and one slot per walk thread");

// LDS of the backward for NW waves: the walk's staging, which the waves'
// transposing tiles take over once the walk is done and which holds the
// slots' records in the sweep, per-pixel scalars and the slot map. Dynamic
// LDS behind it: selections and weights.
template <int NW>
struct BwdLds {
  struct Stage {
    float2 mean[kTilePix];
    float4 co[kTilePix];
    int gid[kTilePix];
  };
  static constexpr size_t kTileBytes = 2 * kPB * kTS * sizeof(__bf16);  // hi and lo of one wave's block
  static constexpr size_t kStage = NW * kTileBytes > sizeof(Stage) ? NW * kTileBytes : sizeof(Stage);
  static_assert(kSlots * kDotStride * sizeof(float) <= kTileBytes, "a block's partial dots fit in its tile");
  __attribute__((aligned(16))) unsigned char stage[kStage];
  float thr[QR_MAX_K + 1];
  __attribute__((aligned(16))) float inv[kTilePix];
  __attribute__((aligned(16))) uint32_t smask[kTilePix];  // per pixel: slots of the pass it selected
  __attribute__((aligned(16))) int sj[kTilePix];          // place of the first of them in the lists
  uint32_t bm[kPosWords];   // selected positions, relative to the list start
  int bpre[kPosWords];      // slots before each bitmap word
  int sgid[kMaxSlots];      // Gaussian id of each slot
  float sscale[kMaxSlots];  // e4m3: its row's scale
  int wtot[4];
  int odd;  // dL/d(out) may have a value that is not finite
};

// The walk's view of the same memory (its template names the arrays).
template <int NW>
struct BwdWalkLds {
  float2* mean;
  float4* co;
  float* thr;
  int* gid;
  static constexpr bool kKeepIds = true;
  __device__ explicit BwdWalkLds(BwdLds<NW>& B)
      : mean(reinterpret_cast<typename BwdLds<NW>::Stage*>(B.stage)->mean),
        co(reinterpret_cast<typename BwdLds<NW>::Stage*>(B.stage)->co),
        thr(B.thr), gid(reinterpret_cast<typename BwdLds<NW>::Stage*>(B.stage)->gid) {}
};

// Four bf16 of an LDS tile, transposed over each 16 lanes: with lane 4e + g
// of the 16 addressing row e, columns 4g .. 4g+3, lane i receives column i
// of rows 0 .. 3.
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ bf16x4 lds_read_tr(const __bf16* p) {
  return __builtin_bit_cast(
      bf16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                  (__attribute__((address_space(3))) s16x4*)(const_cast<__bf16*>(p))));
}

// Row of dL/d(out) of tile pixel p (clamped into the image: rows of pixels
// outside it are never used).
__device__ __forceinline__ const QR_GLOBAL float* grad_row(const GView& v, const GGrad& gg, int tx,
                                                           int ty, int p, int dim) {
  const int gx = min(tx * kTile + (p % kTile), v.W - 1);
  const int gy = min(ty * kTile + (p / kTile), v.H - 1);
  return gg.grad_out + (static_cast<int64_t>(gy) * v.W + gx) * dim;
}

// How the waves share a tile's blocks, and where a lane reads dL/d(out): the
// rows of its pixel in tile rows 2 pb and 2 pb + 1 (clamped into the image:
// rows of pixels outside it are never used), columns in blocks of 32. Waves
// lie along the columns (a power of two of them), the rest along the pixels;
// past NW * MS column blocks the caller makes rounds.
// How the columns lie on the waves of a kernel: on at most half of them, the
// others taking other pixels (up to 256 columns); a share on each (up to 512);
// in rounds of 512. The first two are kernels of their own, as one kernel for
// both took 3% longer at 512 columns (K = 8, 640 x 480: 295 against 284 us).
enum : int { kSpanPart, kSpanAll, kSpanRounds };
template <int NW>
struct Shares {
  static constexpr int MS = 16 / NW;  // column blocks of a wave
  static constexpr int kBuf = MS > 1 ? 2 : 1;
  static constexpr int kBlocks = kTilePix / kPB;
  int n_sc, cgroups, pgroups, pg, sub0, nsub;
  int x0, y0, ymax, c0, cmax;
  const QR_GLOBAL float* g0;
  int64_t gstride;

  __device__ __forceinline__ Shares(const GView& v, const GGrad& gg, int round, int tx, int ty, int wave, int lane, int dim) {
    n_sc = (dim + kSub - 1) / kSub - round * NW * MS;
    cgroups = 1;
    while (cgroups < NW && cgroups * MS < n_sc) cgroups *= 2;
    const int cg = wave & (cgroups - 1);
    pg = wave / cgroups;
    pgroups = NW / cgroups;
    sub0 = round * NW * MS + cg * MS;
    nsub = max(0, min(MS, n_sc - cg * MS));
    x0 = tx * kTile;
    y0 = ty * kTile;
    ymax = v.H - 1;
    c0 = sub0 * kSub + 8 * (lane >> 4);
    cmax = dim - 8;
    g0 = gg.grad_out + static_cast<int64_t>(min(tx * kTile + (lane & 15), v.W - 1)) * dim;
    gstride = static_cast<int64_t>(v.W) * dim;
  }
  __device__ __forceinline__ void load(int pb, int s, f32x4 (&x)[4]) const {
    const int c = min(c0 + s * kSub, cmax);
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
      const QR_GLOBAL float* r = g0 + min(y0 + 2 * pb + rb, ymax) * gstride + c;
      x[2 * rb] = *reinterpret_cast<const QR_GLOBAL f32x4*>(r);
      x[2 * rb + 1] = *reinterpret_cast<const QR_GLOBAL f32x4*>(r + 4);
    }
  }
  // the first blocks of a pass
  __device__ __forceinline__ void prime(f32x4 (&raw)[kBuf][4]) const {
    if (nsub > 0) {
#pragma unroll
      for (int k = 0; k < kBuf; ++k) load(pg, k, raw[k]);
    }
  }
};

// Whether dL/d(out) has a value of the tile in column c that is not finite.
__device__ __forceinline__ bool odd_column(const GView& v, const GGrad& gg, int x0, int y0, int dim, int c) {
  float z = 0.f;
#pragma unroll 1
  for (int y = y0; y < min(y0 + kTile, v.H); ++y) {
    const QR_GLOBAL float* g = gg.grad_out + (static_cast<int64_t>(y) * v.W + x0) * dim + c;
    for (int x = x0; x < min(x0 + kTile, v.W); ++x, g += dim) z = fmaf(*g, 0.f, z);
  }
  return z != 0.f;
}

// One pass over dL/d(out) of the tile for slots base .. base + nslot - 1:
//   DF   feature gradients dF[s][c] = sum_p (w_ps / Z_p) g_p[c], one atomic
//        per (slot, column) of a wave;
//   DOT  dots D[p][s] = <g_p, f_s>, which replace the weights of the same
//        selections (`add`: are added to what an earlier round left there).
// The waves share out the columns (Shares) and walk the tile's pixels in blocks of 32. A
// block [32 px x 32 columns] is loaded once, whole 128-byte lines, and serves
// both products: a lane holds eight consecutive columns of a pixel, which is
// the A operand of D (k = columns); the B operand of dF (k = pixels) comes
// from the same bf16 pairs through the wave's own LDS tile and the
// transposing LDS read. So dL/d(out) is read from memory once per pass and
// every wave streams its own lines. The dots of a pixel are partial sums over
// the columns of a wave: after each 32 pixels the waves leave theirs in their
// tiles and the workgroup adds them up for the selected pairs, one thread per
// (pixel, selection). (Adding them with LDS float atomics kept the LDS busy
// for 61% of the kernel.)
// FAR: the passes after the first, which ends at slot 32 or at the first slot
// of a list position past 2,048. float32 operands are split into three
// bfloat16 parts instead of two, six products instead of three, which keeps
// float32's precision (relative error 2^-24 instead of 2^-16; a tile's later
// selections were always taken in float32), and half the slots are taken per
// pass, as the parts take the registers of the other half (with 32 slots they
// spill: 495 against 397 us for a picture whose tiles select 70).
template <bool FAR>
constexpr int pass_slots() { return FAR ? kSlots / 2 : kSlots; }

template <int DT, int NW, bool DF, bool DOT, bool FAR, int SPAN>
__device__ __forceinline__ void stream_slots(const GView& v, const GGrad& gg, BwdLds<NW>& B,
                                             float* __restrict__ s_w, int base, int nslot, bool add,
                                             const Shares<NW>& sh, f32x4 (&raw)[Shares<NW>::kBuf][4],
                                             int wave, int lane, int dim) {
  using Sh = Shares<NW>;
  constexpr int MS = Sh::MS, kBuf = Sh::kBuf, kBlocks = Sh::kBlocks;
  constexpr int MB = pass_slots<FAR>() / 16;
  constexpr int P = FAR ? 3 : 2;              // parts of a float32 operand
  constexpr int PF = DT == QR_F32 ? P : 1;    // of a feature (bf16 features and e4m3 codes are exact in one)
  const int row = lane & 15, kb = lane >> 4;
  const int n_mb = (nslot + 15) >> 4;  // blocks of 16 slots (uniform)
  const int n_sc = sh.n_sc, sub0 = sh.sub0, nsub = sh.nsub;
  constexpr bool kAll = SPAN == kSpanAll;
  const int cgroups = kAll ? NW : sh.cgroups, pgroups = kAll ? 1 : sh.pgroups, pg = kAll ? 0 : sh.pg;
  const bool partial = (dim & (kSub - 1)) != 0;  // the last block is half a block

  // B operand of D: feature rows of the slots, this wave's columns
  bf16x8 fp[MS][MB][PF];
  if constexpr (DOT) {
#pragma unroll
    for (int s = 0; s < MS; ++s) {
#pragma unroll
      for (int nb = 0; nb < MB; ++nb) {
        if (s < nsub && nb < n_mb) {
          const int c = (sub0 + s) * kSub + 8 * kb;
          float x[8];
          load_feat8<DT>(v, B.sgid[base + min(nb * 16 + row, nslot - 1)], dim, min(c, dim - 8), x);
          if (c >= dim) {
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = 0.f;
          }
          split_parts<PF>(x, fp[s][nb]);
        }
      }
    }
  }
  floatx4 af[MS][2][MB];
  if constexpr (DF) {
#pragma unroll
    for (int s = 0; s < MS; ++s)
#pragma unroll
      for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) af[s][cb][mb] = floatx4{0.f, 0.f, 0.f, 0.f};
  }

  // the wave's transposing tile: two parts of a block
  __bf16* const tile0 = reinterpret_cast<__bf16*>(B.stage + wave * BwdLds<NW>::kTileBytes);
  const int t_wr = row * kTS + 8 * kb;                         // + 16 rows for the second pixel row
  const int t_rd = (8 * kb + (row >> 2)) * kTS + 4 * (row & 3);  // + 4 rows, + 16 columns
  const auto put = [&](int area, const bf16x8& r0, const bf16x8& r1) {
    __bf16* const t = tile0 + area * (kPB * kTS) + t_wr;
    *reinterpret_cast<bf16x8*>(t) = r0;
    *reinterpret_cast<bf16x8*>(t + 16 * kTS) = r1;
  };
  const auto get = [&](int area, int cb) {  // eight pixels of a column
    const __bf16* const t = tile0 + area * (kPB * kTS) + t_rd + 16 * cb;
    return __builtin_shufflevector(lds_read_tr(t), lds_read_tr(t + 4 * kTS), 0, 1, 2, 3, 4, 5, 6, 7);
  };

  const bool mine = nsub > 0;  // uniform in a wave
#pragma unroll 1
  for (int pb = pg; pb < kBlocks; pb += pgroups) {  // (pgroups divides kBlocks: as many rounds for every wave)
    if (mine) {
      const int pb_next = pb + pgroups < kBlocks ? pb + pgroups : pb;
      // A operand of dF: w / Z of slot mb * 16 + row, pixels 8 kb .. 8 kb + 7
      // of the block
      bf16x8 wp[MB][P];
      if constexpr (DF) {
        const int p0 = pb * kPB + 8 * kb;
        float w[MB][8];
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          const uint32_t m = B.smask[p0 + t];
          const int j = B.sj[p0 + t];
          const float inv = B.inv[p0 + t];
#pragma unroll
          for (int mb = 0; mb < MB; ++mb) {
            const int sl = mb * 16 + row;
            // read for every pair (one past a list's end at most), used for the selected
            const float x = s_w[j + __popc(m & ((1u << sl) - 1u))];
            w[mb][t] = ((m >> sl) & 1u) ? x * inv : 0.f;
          }
        }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) split_parts<P>(w[mb], wp[mb]);
      }
      floatx4 ad[2][MB];
      if constexpr (DOT) {
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
#pragma unroll
          for (int nb = 0; nb < MB; ++nb) ad[rb][nb] = floatx4{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int s = 0; s < MS; ++s) {
        f32x4(&x)[4] = raw[s % kBuf];
        bf16x8 ap[2][P];  // the block's two pixel rows
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) {
          float y[8];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            y[i] = x[2 * rb][i];
            y[4 + i] = x[2 * rb + 1][i];
          }
          split_parts<P>(y, ap[rb]);
        }
        if (partial && (sub0 + s) * kSub + 8 * kb >= dim) {  // columns past dim
#pragma unroll
          for (int rb = 0; rb < 2; ++rb)
#pragma unroll
            for (int i = 0; i < P; ++i) ap[rb][i] = bf16x8{};
        }
        // the block two steps on, into the registers just read (always a
        // load, at the end one of this pass's blocks again: under a
        // condition the compiler waits for it on the spot)
        if (s + kBuf < MS) sh.load(pb, s + kBuf, x);
        else sh.load(pb_next, s + kBuf - MS, x);
        if (s >= nsub) continue;  // uniform
        if constexpr (DF) {
          put(0, ap[0][0], ap[1][0]);
          put(1, ap[0][1], ap[1][1]);
          wave_lds_sync();
        }
        if constexpr (DOT) {
#pragma unroll
          for (int nb = 0; nb < MB; ++nb) {
            if (nb >= n_mb) continue;
#pragma unroll
            for (int rb = 0; rb < 2; ++rb)
#pragma unroll
              for (int k = 0; k < PF; ++k)
#pragma unroll
                for (int i = 0; i + k < P; ++i)
                  ad[rb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ap[rb][i], fp[s][nb][k], ad[rb][nb], 0, 0, 0);
          }
        }
        if constexpr (DF) {
#pragma unroll
          for (int cb = 0; cb < 2; ++cb) {
            const bf16x8 g0 = get(0, cb), g1 = get(1, cb);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
              if (mb >= n_mb) continue;
              floatx4& a = af[s][cb][mb];
#pragma unroll
              for (int i = 0; i < P; ++i) a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wp[mb][i], g0, a, 0, 0, 0);
#pragma unroll
              for (int i = 0; i + 1 < P; ++i) a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wp[mb][i], g1, a, 0, 0, 0);
            }
          }
          wave_lds_sync();
          if constexpr (P == 3) {  // the third part, where the first was
            put(0, ap[0][2], ap[1][2]);
            wave_lds_sync();
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
              const bf16x8 g2 = get(0, cb);
#pragma unroll
              for (int mb = 0; mb < MB; ++mb) {
                if (mb < n_mb)
                  af[s][cb][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wp[mb][0], g2, af[s][cb][mb], 0, 0, 0);
              }
            }
            wave_lds_sync();
          }
        }
      }
      if constexpr (DOT) {
        // lane holds D[4 kb + i][row] of each (pixel row, slot block): four
        // pixels of a slot
        float* const d = reinterpret_cast<float*>(tile0);
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
#pragma unroll
          for (int nb = 0; nb < MB; ++nb) {
            if (nb < n_mb)
              *reinterpret_cast<floatx4*>(&d[(nb * 16 + row) * kDotStride + 16 * rb + 4 * kb]) = ad[rb][nb];
          }
      }
    }
    if constexpr (DOT) {
      // the dots of pixel p's slots, every `step`-th from the first-th on: the
      // sum over nw tiles
      const auto take = [&](int p, int first, int step, const float* d, int nw) {
        uint32_t m = B.smask[p];
        for (int k = 0; k < first; ++k) m &= m - 1u;
        for (int j = B.sj[p] + first; m; j += step) {
          const int sl = __builtin_ctz(m);
          float x = 0.f;
          for (int w = 0; w < nw; ++w) x += d[w * (BwdLds<NW>::kTileBytes / sizeof(float)) + sl * kDotStride];
          if (DT == QR_FP8_E4M3) x *= B.sscale[base + sl];
          s_w[j] = add ? s_w[j] + x : x;
          for (int k = 0; k < step; ++k) m &= m - 1u;
        }
      };
      if (cgroups == 1) {  // a wave has all columns of its pixels, and alone reads their weights
        if (mine) {
          wave_lds_sync();
          const int q = lane & (kPB - 1);
          take(pb * kPB + q, lane / kPB, 2, reinterpret_cast<const float*>(tile0) + q, 1);
          wave_lds_sync();
        }
      } else {
        __syncthreads();  // every wave has left its sums (and built its weights of these pixels)
        // every pixel group adds up its own block, from the tiles of the
        // column groups that have columns (all groups between two barriers:
        // with a block per barrier pair, the waves of the other pixel groups
        // idle, 128 columns took 375 instead of 283 us at K = 24, 256 columns
        // 245 instead of 203 at K = 8, 640 x 480)
        const int nw = min(cgroups, (n_sc + MS - 1) / MS);
        const int q = threadIdx.x & (kPB - 1);
        const float* const d = reinterpret_cast<const float*>(B.stage + pg * cgroups * BwdLds<NW>::kTileBytes) + q;
        take(pb * kPB + q, threadIdx.x / kPB - 2 * cgroups * pg, 2 * cgroups, d, nw);
        __syncthreads();  // the tiles are free again
      }
    }
  }

  if (DF && gg.grad_features) {
    // Columns with a value that is not finite: any slot's sums of the first pass
    // tell that there may be one (0 x is 0 for finite x alone); the later ones
    // leave such columns out, as odd_columns has added them. (A look at every
    // value in the later passes cost them 2% and the persistent kernels, by
    // their registers, 4%.)
    uint32_t odd = 0u;
    if constexpr (!FAR) {
      float z = 0.f;
#pragma unroll
      for (int s = 0; s < MS; ++s)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) z = fmaf(af[s][cb][0][0], 0.f, z);
      if (__ballot(z != 0.f) != 0ull && lane == 0) B.odd = 1;
    } else if (B.odd) {
#pragma unroll 1
      for (int k = 0; k < 2 * nsub; ++k) {
        const int c = sub0 * kSub + 16 * k + row;
        if (c < dim && odd_column(v, gg, sh.x0, sh.y0, dim, c)) odd |= 1u << k;
      }
    }
    // lane holds dF[4 kb + i][row] of each (slot block, column block)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int sl = mb * 16 + 4 * kb + i;
        if (sl >= nslot) continue;
        QR_GLOBAL float* dst = gg.grad_features + static_cast<int64_t>(B.sgid[base + sl]) * dim + row;
#pragma unroll
        for (int s = 0; s < MS; ++s)
#pragma unroll
          for (int cb = 0; cb < 2; ++cb) {
            const int c = (sub0 + s) * kSub + 16 * cb;
            if (s < nsub && c < dim && af[s][cb][mb][i] != 0.f && !(FAR && ((odd >> (2 * s + cb)) & 1u)))
              atomic_add(dst + c, af[s][cb][mb][i]);
          }
      }
    }
  }
}

// Selections without a slot (a list position past kPosCap, or more than
// kMaxSlots distinct selections in the tile: both rare), for the wave's
// pixels, one selection at a time over the wave's lanes: feature gradients
// w g / Z added to global memory, then the dot <g, f_j> written over the
// weight. They are the last of each pixel's list, from entry `jfree` on.
template <int DT>
__device__ __forceinline__ void slotless(const GView& v, const GGrad& gg, const float* __restrict__ s_inv,
                                         const int* __restrict__ s_pos, float* __restrict__ s_w,
                                         int tx, int ty, int wave, int lane, int dim, int jfree, int ns,
                                         int KP, bool geo) {
  uint64_t todo = __ballot(ns > jfree);
  while (todo) {
    const int l = __builtin_ctzll(todo);
    todo &= todo - 1ull;
    const int p = wave * 64 + l;
    const int n = __builtin_amdgcn_readlane(ns, l);
    const float inv = s_inv[p];
    const QR_GLOBAL float* grow = grad_row(v, gg, tx, ty, p, dim);
    for (int j = __builtin_amdgcn_readlane(jfree, l); j < n; ++j) {
      const int pos = ~__builtin_amdgcn_readfirstlane(s_pos[p * KP + j]);
      const int g = static_cast<int>(__builtin_amdgcn_readfirstlane(v.sorted_gid[pos]));
      const float w = s_w[p * KP + j] * inv;
      QR_GLOBAL float* dst = gg.grad_features + static_cast<int64_t>(g) * dim;
      float dot = 0.f;
      for (int c = 4 * lane; c < dim; c += 256) {
        const f32x4 gr = *reinterpret_cast<const QR_GLOBAL f32x4*>(grow + c);
        if (geo) {
          const float4 f = load_feat4_global<DT>(v.feats, v.scale, g, dim, c);
          dot += gr.x * f.x + gr.y * f.y + gr.z * f.z + gr.w * f.w;
        }
        if (gg.grad_features) {
          atomic_add(dst + c + 0, w * gr.x);
          atomic_add(dst + c + 1, w * gr.y);
          atomic_add(dst + c + 2, w * gr.z);
          atomic_add(dst + c + 3, w * gr.w);
        }
      }
      if (geo) {
        const float t = wave_sum(dot);
        wave_lds_sync();  // every lane has read the weight
        if (lane == 0) s_w[p * KP + j] = t;
      }
    }
  }
}

// Feature gradients of the tile's selections from the second pass on (pixel p:
// s_n[p] of them from entry s_j[p] of the lists), in the columns that have a
// value that is not finite: a product with the weight 0 of a selection that a
// pixel does not have would be NaN, so these columns are summed selection by
// selection. All threads of the workgroup, a column each. *s_odd: whether there
// is one.
__device__ __forceinline__ void odd_columns(const GView& v, const GGrad& gg, const int* __restrict__ s_j,
                                            const uint32_t* __restrict__ s_n, const int* __restrict__ s_pos,
                                            const float* __restrict__ s_w, const float* __restrict__ s_inv,
                                            const int* __restrict__ s_gid, int tx, int ty, int dim,
                                            int* __restrict__ s_odd) {
#pragma unroll 1
  for (int c = threadIdx.x; c < dim; c += blockDim.x) {
    if (!odd_column(v, gg, tx * kTile, ty * kTile, dim, c)) continue;
    *s_odd = 1;
#pragma unroll 1
    for (int p = 0; p < kTilePix; ++p) {
      if (s_n[p] == 0u) continue;  // (none outside the picture)
      const float g = grad_row(v, gg, tx, ty, p, dim)[c];
      for (int j = s_j[p]; j < s_j[p] + static_cast<int>(s_n[p]); ++j)
        atomic_add(gg.grad_features + static_cast<int64_t>(s_gid[s_pos[j]]) * dim + c, s_w[j] * s_inv[p] * g);
    }
  }
}

// Bitwise or, and minimum, over the 64 lanes (the exchanges of wave_sum).
template <class Op>
__device__ __forceinline__ uint32_t wave_fold(uint32_t x, const Op& op) {
  const auto a = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  x = op(a[0], a[1]);
  const auto b = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  x = op(b[0], b[1]);
  x = op(x, fbits(dpp<0xB1>(bitsf(x))));
  x = op(x, fbits(dpp<0x4E>(bitsf(x))));
  x = op(x, fbits(dpp<0x124>(bitsf(x))));
  x = op(x, fbits(dpp<0x128>(bitsf(x))));
  return __builtin_amdgcn_readfirstlane(x);
}
__device__ __forceinline__ uint32_t wave_or(uint32_t x) {
  return wave_fold(x, [](uint32_t a, uint32_t b) { return a | b; });
}
__device__ __forceinline__ uint32_t wave_min(uint32_t x) {
  return wave_fold(x, [](uint32_t a, uint32_t b) { return min(a, b); });
}

// Dynamic LDS: selections and weights, and up to K = kBwdWideK the slots'
// records (beyond, they take the tiles' place after the last pass).
constexpr int kBwdPairK = 20, kBwdWideK = 48;
__host__ __device__ constexpr size_t bwd_list_floats(int K) { return static_cast<size_t>(kTilePix) * ((K + 3) & ~3); }
__host__ __device__ constexpr bool bwd_early_records(int K) { return K <= kBwdWideK; }
constexpr size_t bwd_dynamic_lds(int K) {
  return 2 * bwd_list_floats(K) * sizeof(float) + (bwd_early_records(K) ? kMaxSlots * 6 * sizeof(float) : 0);
}

// Backward of one tile (all threads of the workgroup; the walk and the sweep
// use the first 256, one per pixel). s_pos, s_w: the walk's selected
// positions and weights ([256][KP] each); positions become slots (or ~position
// without one), and once the feature gradients that read a weight are
// formed, the dot d_j takes its place. The sweep recomputes each weight and
// T^Q_j from the records with the walk's own float operations.
template <int DT, int NW, int SPAN>
__device__ __forceinline__ void quantile_backward_tile(const GView& v, const GGrad& gg, int tile,
                                                       int K, int dim, const qr_params& prm,
                                                       BwdLds<NW>& B, float* __restrict__ dyn) {
  const int tiles_x = (v.W + kTile - 1) / kTile;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: addresses stay scalar
  const bool walker = NW == 4 || tid < kTilePix;
  const int tx = tile % tiles_x, ty = tile / tiles_x;
  const int px = tx * kTile + (tid % kTile);
  const int py = ty * kTile + (tid / kTile);
  const bool inside = walker && px < v.W && py < v.H;
  const float pxc = px + 0.5f, pyc = py + 0.5f;
  const int lo = static_cast<int>(v.tile_offsets[tile]);
  const int hi = static_cast<int>(v.tile_offsets[tile + 1]);
  if (lo == hi) return;  // uniform
  const int KP = (K + 3) & ~3;
  float* const s_w = dyn;
  int* const s_pos = reinterpret_cast<int*>(dyn + bwd_list_floats(K));
  if (walker) B.bm[tid] = 0u;  // read after the walk's barriers
  if (tid == 0) B.odd = 0;
  BwdWalkLds<NW> WL(B);
  // the first blocks of dL/d(out) are requested before the walk
  const Shares<NW> sh(v, gg, 0, tx, ty, wave, lane, dim);
  f32x4 raw[Shares<NW>::kBuf][4];
  sh.prime(raw);
  ListSink sink{s_pos + tid * KP, s_w + tid * KP};
  WalkState walk;
  const PixelSel sel =
      quantile_walk<QR_SELECT_QUANTILE, false>(v, lo, lo, hi, K, pxc, pyc, inside, prm, WL, sink, walk);
  const int ns = sel.ns;
  if (walker) B.inv[tid] = sel.inv;
  int* const my_pos = s_pos + tid * KP;
  const bool geo = gg.grad_means2d || gg.grad_co;
  // the slots' records, for the sweep: fetched with the slots where LDS is
  // left for them (fetched after the last pass they would wait for its
  // atomics: loads and atomics complete in order)
  const bool early = geo && bwd_early_records(K);
  float4* const rec_co = reinterpret_cast<float4*>(early ? dyn + 2 * bwd_list_floats(K) : reinterpret_cast<float*>(B.stage));
  float2* const rec_mean = reinterpret_cast<float2*>(rec_co + kMaxSlots);
  const auto load_record = [&](int s, int g) {
    const f32x2 m = v.means2d[g];
    const f32x4 c = v.conic_opacity[g];
    rec_mean[s] = make_float2(m.x, m.y);
    rec_co[s] = make_float4(c.x, c.y, c.z, c.w);
  };

  // ---- slots: the tile's distinct selected positions, in list order ----
  // (a word of the bitmap at a time: the bits of a wave's pixels are folded in
  // registers, one LDS atomic per wave and word)
  if (walker) {
    uint32_t r = ns > 0 ? static_cast<uint32_t>(my_pos[0] - lo) : kPosCap;
    for (int j = 0;;) {
      const uint32_t w = wave_min(r) >> 5;
      if (w >= kPosWords) break;
      uint32_t m = 0u;
      while ((r >> 5) == w) {
        m |= 1u << (r & 31);
        ++j;
        r = j < ns ? static_cast<uint32_t>(my_pos[j] - lo) : kPosCap;
      }
      m = wave_or(m);
      if (lane == 0) atomicOr(&B.bm[w], m);
    }
  }
  __syncthreads();
  uint32_t word = 0u;
  int before = 0;
  if (walker) {  // prefix of the word populations
    word = B.bm[tid];
    int incl = __popc(word);
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int u = __shfl_up(incl, off, 64);
      if (lane >= off) incl += u;
    }
    before = incl - __popc(word);
    if (lane == 63) B.wtot[wave] = incl;
  }
  __syncthreads();
  const int total = B.wtot[0] + B.wtot[1] + B.wtot[2] + B.wtot[3];
  const int nslots = min(total, kMaxSlots);
  if (walker) {
    for (int w = 0; w < wave; ++w) before += B.wtot[w];
    B.bpre[tid] = before;
    for (int s = before; word && s < kMaxSlots; ++s, word &= word - 1u) {
      // (a position of the batch that is still staged: from LDS)
      const int pos = lo + 32 * tid + __builtin_ctz(word), k = pos - sel.staged;
      const int g = k >= 0 ? WL.gid[k] : static_cast<int>(v.sorted_gid[pos]);
      B.sgid[s] = g;
      if (DT == QR_FP8_E4M3) B.sscale[s] = v.scale[g];
      if (!early) continue;
      if (k >= 0) {
        rec_mean[s] = WL.mean[k];
        const float4 c = WL.co[k];  // staged with the conic's 2 b
        rec_co[s] = make_float4(c.x, 0.5f * c.y, c.z, c.w);
      } else {
        load_record(s, g);
      }
    }
  }
  __syncthreads();
  int nslotted = 0;  // slots are ranks in list order: the slotted selections come first
  for (int j = 0; j < ns; ++j) {
    const int pos = my_pos[j], r = pos - lo;
    int s = kMaxSlots;
    if (r < kPosCap) s = B.bpre[r >> 5] + __popc(B.bm[r >> 5] & ((1u << (r & 31)) - 1u));
    my_pos[j] = s < kMaxSlots ? s : ~pos;
    if (s < kMaxSlots) nslotted = j + 1;
  }

  // ---- feature gradients and dots, pass by pass ----
  // (widths up to 512: both products at once, whether or not both are asked
  // for; wider: in rounds of 512 columns, the feature gradients of all rounds
  // before the dots, which replace the weights)
  int j_next = 0;
  const auto masks = [&](int base, int n) {
    if (walker) {
      uint32_t m = 0u;
      B.sj[tid] = tid * KP + j_next;
      for (; j_next < nslotted; ++j_next) {
        const int s = my_pos[j_next] - base;
        if (s >= n) break;
        m |= 1u << s;
      }
      B.smask[tid] = m;
    }
    __syncthreads();
  };
  const auto pass = [&](int base, int n, auto far) {
    constexpr bool FAR = decltype(far)::value;
    masks(base, n);
    if constexpr (SPAN != kSpanRounds) {
      if (FAR) sh.prime(raw);
      stream_slots<DT, NW, true, true, FAR, SPAN>(v, gg, B, s_w, base, n, false, sh, raw, wave, lane, dim);
    } else {
      const int rounds = (dim + 511) / 512;
      if (gg.grad_features) {
        for (int r = 0; r < rounds; ++r) {
          const Shares<NW> shr(v, gg, r, tx, ty, wave, lane, dim);
          shr.prime(raw);
          stream_slots<DT, NW, true, false, FAR, SPAN>(v, gg, B, s_w, base, n, false, shr, raw, wave, lane, dim);
        }
      }
      if (geo) {
        __syncthreads();  // every weight has been read
        for (int r = 0; r < rounds; ++r) {
          const Shares<NW> shr(v, gg, r, tx, ty, wave, lane, dim);
          shr.prime(raw);
          stream_slots<DT, NW, false, true, FAR, SPAN>(v, gg, B, s_w, base, n, r > 0, shr, raw, wave, lane, dim);
        }
      }
    }
    __syncthreads();  // the masks may be rewritten
  };
  const int near = min(min(kSlots, nslots), B.bpre[kNearWords]);  // uniform
  if (near > 0) pass(0, near, std::false_type{});
  if (gg.grad_features && near < nslots && (near == 0 || B.odd)) {  // uniform
    if (walker) {
      B.sj[tid] = tid * KP + j_next;
      B.smask[tid] = nslotted - j_next;
    }
    __syncthreads();
    odd_columns(v, gg, B.sj, B.smask, s_pos, s_w, B.inv, B.sgid, tx, ty, dim, &B.odd);
    __syncthreads();  // the masks may be rewritten
  }
#pragma unroll 1
  for (int base = near; base < nslots; base += pass_slots<true>())
    pass(base, min(pass_slots<true>(), nslots - base), std::true_type{});
  if (walker) slotless<DT>(v, gg, B.inv, s_pos, s_w, tx, ty, wave, lane, dim, nslotted, ns, KP, geo);
  if (!geo) return;

  // ---- sweep over this pixel's selections ----
  if (!early) {
    __syncthreads();
    if (walker && tid < nslots) load_record(tid, B.sgid[tid]);
    __syncthreads();
  }
  if (!walker) {  // the walkers' barriers below
    for (int w = 0; 32 * w < nslots; ++w) {
      __syncthreads();
      __syncthreads();
    }
    return;
  }
  // Weights and T^Q_j are recomputed front to back exactly as the walk formed
  // them; the tail sums S_j = sum_{l > j} w_l d_l are taken as the total
  // minus the running prefix, both in double.
  float* const my_d = s_w + tid * KP;
  const auto free_record = [&](int j, float2& mean, float4& co) {  // of a selection without a slot
    const int g = static_cast<int>(v.sorted_gid[~my_pos[j]]);
    const f32x2 m = v.means2d[g];
    const f32x4 c = v.conic_opacity[g];
    mean = make_float2(m.x, m.y);
    co = make_float4(c.x, c.y, c.z, c.w);
    return g;
  };
  double tot = 0.0;
  float tq = 1.f;
  constexpr int kU = 4;  // selections read from LDS per round trip
  for (int j0 = 0; j0 < nslotted; j0 += kU) {
    float a[kU], d[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int j = min(j0 + u, nslotted - 1), sl = my_pos[j];
      a[u] = gauss_alpha(rec_mean[sl], rec_co[sl], pxc, pyc, prm.alpha_max);
      d[u] = my_d[j];
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      if (j0 + u >= nslotted) continue;
      tot += static_cast<double>(tq * a[u]) * d[u];
      tq = tq * (1.f - a[u]);
    }
  }
  for (int j = nslotted; j < ns; ++j) {
    float2 mean;
    float4 co;
    free_record(j, mean, co);
    const float a = gauss_alpha(mean, co, pxc, pyc, prm.alpha_max);
    tot += static_cast<double>(tq * a) * my_d[j];
    tq = tq * (1.f - a);
  }
  const float TQ = sel.TQ;
  const float invZ = ns > 0 ? 1.f / (1.f - TQ) : 0.f;
  const float gout = static_cast<float>(tot) * invZ;  // <g, out>
  tq = 1.f;
  double pre = 0.0;
  // dL/dpower of a selection with dot dj (0 if clamped); alpha' = o G
  const auto dpower = [&](const AlphaEval& e, float dj) {
    const float wj = tq * e.alpha;
    pre += static_cast<double>(wj) * dj;
    const float S = static_cast<float>(tot - pre);  // sum over the later selections
    const float dL_da = invZ * (tq * dj - (S + gout * TQ) / (1.f - e.alpha));
    tq = tq * (1.f - e.alpha);
    return e.clamped ? 0.f : dL_da * e.alpha;
  };
  // dL/dpower takes the place of the dot
  for (int j = 0; j < nslotted; ++j) {
    const int sl = my_pos[j];
    const AlphaEval e = eval_alpha(rec_mean[sl], rec_co[sl], pxc, pyc, prm.alpha_max);
    my_d[j] = dpower(e, my_d[j]);
  }
  for (int j = nslotted; j < ns; ++j) {
    float2 mean;
    float4 co;
    const int g = free_record(j, mean, co);
    const AlphaEval e = eval_alpha(mean, co, pxc, pyc, prm.alpha_max);
    const float dpow = dpower(e, my_d[j]);
    if (dpow == 0.f) continue;
    if (gg.grad_co) {
      QR_GLOBAL float* const o = gg.grad_co + 4 * static_cast<int64_t>(g);
      atomic_add(o + 0, dpow * (-0.5f * e.dx * e.dx));
      atomic_add(o + 1, dpow * (-e.dx * e.dy));
      atomic_add(o + 2, dpow * (-0.5f * e.dy * e.dy));
      atomic_add(o + 3, dpow / co.w);
    }
    if (gg.grad_means2d) {
      QR_GLOBAL float* const o = gg.grad_means2d + 2 * static_cast<int64_t>(g);
      atomic_add(o + 0, dpow * (co.x * e.dx + co.y * e.dy));
      atomic_add(o + 1, dpow * (co.y * e.dx + co.z * e.dy));
    }
  }
  wave_lds_sync();
  // The gradients of a slot are sums of its dL/dpower over the tile's pixels,
  // sum_p dpow_p {dx^2, dx dy, dy^2, 1, a dx + b dy, b dx + c dy}. A lane takes
  // one slot and half a tile row at a time (dy is then one value), so the
  // sums stay in registers; the lanes of a slot are added up by exchanges and
  // the four waves in LDS. (Evaluating the values per slot for all 64 pixels
  // of a wave, a quarter of them selected, and summing those over the wave
  // took twice as long; moments about the tile's centre, as a product on the
  // matrix cores, lose the digits that dx and dy have near the mean.)
  const int row = lane & 15, kb = lane >> 4;
  // [wave][slot][8], behind the records where those are in the tiles' place
  float* const mom = reinterpret_cast<float*>(B.stage) + kMaxSlots * 6;
  static_assert((kMaxSlots * 6 + 4 * kSlots * 8) * sizeof(float) <= BwdLds<NW>::kStage, "records and moments");
  for (int w = 0, j = 0; 32 * w < nslots; ++w) {
    uint32_t m = 0u;
    B.sj[tid] = tid * KP + j;
    for (; j < nslotted; ++j) {
      const int sl = my_pos[j] - 32 * w;
      if (sl >= 32) break;
      m |= 1u << sl;
    }
    B.smask[tid] = m;
    wave_lds_sync();
    const int n_mb = nslots - 32 * w > 16 ? 2 : 1;
#pragma unroll 1
    for (int mb = 0; mb < n_mb; ++mb) {
      const int sl = mb * 16 + row;
      const float2 mean = rec_mean[min(32 * w + sl, nslots - 1)];
      const float4 co = rec_co[min(32 * w + sl, nslots - 1)];
      float q[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int h = 0; h < 2; ++h) {  // 32 pixels: two tile rows
        const int p0 = wave * 64 + 32 * h + 8 * kb;
        const float dy = (ty * kTile + p0 / kTile + 0.5f) - mean.y;
        const float dx0 = (tx * kTile + (p0 & 8) + 0.5f);
        float s0 = 0.f, sx = 0.f, sxx = 0.f, su = 0.f, sv = 0.f;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          const uint32_t mp = B.smask[p0 + t];
          const float x = s_w[B.sj[p0 + t] + __popc(mp & ((1u << sl) - 1u))];
          const float d = ((mp >> sl) & 1u) ? x : 0.f;
          const float dx = (dx0 + t) - mean.x;
          const float v = d * dx;
          s0 += d;
          sx += v;
          sxx = fmaf(v, dx, sxx);
          su = fmaf(d, co.x * dx + co.y * dy, su);
          sv = fmaf(d, co.y * dx + co.z * dy, sv);
        }
        q[0] += sxx;
        q[1] = fmaf(sx, dy, q[1]);
        q[2] = fmaf(s0 * dy, dy, q[2]);
        q[3] += s0;
        q[4] += su;
        q[5] += sv;
      }
      // over the slot's four lanes, 16 apart
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        q[i] = tsum_bit5(q[i], q[i]);
        q[i] = tsum_bit4(q[i], q[i]);
        if (kb == 0) mom[(wave * kSlots + sl) * 8 + i] = q[i];
      }
    }
    __syncthreads();
    // neighbouring threads add a slot's neighbouring values: threads 0 .. 127
    // (a, b, c, o) of slot tid / 4, 128 .. 191 (u, v) of slot (tid - 128) / 2
    const bool conic = tid < 4 * kSlots;
    const int ls = conic ? tid >> 2 : (tid - 4 * kSlots) >> 1, k = conic ? tid & 3 : 4 + (tid & 1);
    const int sl = 32 * w + ls;
    if (tid < 6 * kSlots && sl < nslots) {
      const int at = ls * 8 + k;
      const float sum = mom[at] + mom[kSlots * 8 + at] + mom[2 * kSlots * 8 + at] + mom[3 * kSlots * 8 + at];
      const int64_t g = B.sgid[sl];
      // (alpha' = o G: dL/do = dL/dpower / o)
      const float val = k >= 4 ? sum : k == 1 ? -sum : k == 3 ? sum / rec_co[sl].w : -0.5f * sum;
      if (conic && gg.grad_co) atomic_add(gg.grad_co + 4 * g + k, val);
      if (!conic && gg.grad_means2d) atomic_add(gg.grad_means2d + 2 * g + (k - 4), val);
    }
    __syncthreads();  // the moments may be rewritten
  }
}

// Two waves per SIMD (registers of the MFMA operands and accumulators: up to
// 512 columns the workgroups of four waves, four column blocks each, need all
// 256 and spill 27 to 30 of float32 features, the persistent ones 61 to 73, and
// 14 to 21 of the other types; eight waves and the rounds of 512 spill none).
constexpr int kBwdWavesPerSimd = 2;

template <int DT, int NW, int SPAN>
__global__ void __launch_bounds__(64 * NW, kBwdWavesPerSimd)
quantile_backward_kernel(ViewArgs v, GradPtrs gp, int n_tiles, qr_params prm, int K, int dim) {
  extern __shared__ __attribute__((aligned(16))) float dyn_lds[];
  __shared__ BwdLds<NW> B;
  quantile_backward_tile<DT, NW, SPAN>(to_global(v), to_global(gp), xcd_remap(blockIdx.x, n_tiles), K, dim,
                                 prm, B, dyn_lds);
}

__device__ __forceinline__ GradPtrs grad_ptrs(const qr_view_grad& g) {
  return GradPtrs{g.grad_out, g.grad_features, g.grad_means2d, g.grad_conic_opacity};
}

// Many views in one launch, one workgroup per (view, tile) item, items dealt
// to the XCDs in contiguous runs of the schedule.
template <int DT, int NW, int SPAN>
__global__ void __launch_bounds__(64 * NW, kBwdWavesPerSimd)
quantile_backward_batched_grid_kernel(const qr_view* __restrict__ views,
                                      const qr_view_grad* __restrict__ grads,
                                      const uint32_t* __restrict__ schedule, int n_items,
                                      qr_params prm, int K, int dim) {
  extern __shared__ __attribute__((aligned(16))) float dyn_lds[];
  __shared__ BwdLds<NW> B;
  const uint32_t packed = __builtin_amdgcn_readfirstlane(schedule[xcd_remap(blockIdx.x, n_items)]);
  const uint32_t vi = packed >> kViewShift;
  quantile_backward_tile<DT, NW, SPAN>(to_global(view_args(views[vi])), to_global(grad_ptrs(grads[vi])),
                                 static_cast<int>(packed & kTileMask), K, dim, prm, B, dyn_lds);
}

// Many views in one persistent launch: items are taken from per-XCD ranges
// of the schedule exactly as by the persistent forward renderer.
constexpr int kBwdXcdQueues = 8;

__device__ __forceinline__ uint32_t bwd_queue_begin(int64_t n_items, int q) {
  return static_cast<uint32_t>(n_items * q / kBwdXcdQueues);
}

template <int DT, int NW, int SPAN>
__global__ void __launch_bounds__(64 * NW, kBwdWavesPerSimd)
quantile_backward_batched_kernel(const qr_view* __restrict__ views,
                                 const qr_view_grad* __restrict__ grads,
                                 const uint32_t* __restrict__ schedule, int64_t n_items,
                                 uint32_t* __restrict__ counter, qr_params prm, int K, int dim) {
  extern __shared__ __attribute__((aligned(16))) float dyn_lds[];
  __shared__ BwdLds<NW> B;
  __shared__ uint32_t s_item[2];
  const int home = static_cast<int>(blockIdx.x % kBwdXcdQueues);
  // the item word alternates as in the forward: a wave running ahead writes
  // the other word
  for (int it = 0;; it ^= 1) {
    if (threadIdx.x == 0) {
      uint32_t item = 0xFFFFFFFFu;
      for (int d = 0; d < kBwdXcdQueues; ++d) {
        const int q = (home + d) % kBwdXcdQueues;
        const uint32_t b = bwd_queue_begin(n_items, q), e = bwd_queue_begin(n_items, q + 1);
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
    const uint32_t item = __builtin_amdgcn_readfirstlane(s_item[it]);
    if (item >= n_items) break;
    const uint32_t packed = __builtin_amdgcn_readfirstlane(schedule[item]);
    const uint32_t vi = packed >> kViewShift;
    quantile_backward_tile<DT, NW, SPAN>(to_global(view_args(views[vi])), to_global(grad_ptrs(grads[vi])),
                                   static_cast<int>(packed & kTileMask), K, dim, prm, B, dyn_lds);
  }
}

__global__ void reset_bwd_counter_kernel(uint32_t* __restrict__ c) {
  if (threadIdx.x < kBwdXcdQueues) c[threadIdx.x] = 0u;
}

// Workgroup shape by K, from what the selection lists (8 bytes per pixel and
// K) leave of a CU's 160 KB of LDS: up to K = 20 two workgroups of four waves
// fit; up to K = 48 one of eight waves, each with half the columns; beyond,
// one of four waves.
constexpr size_t kCuLds = 160 * 1024;
static_assert(2 * (sizeof(BwdLds<4>) + 64 + bwd_dynamic_lds(kBwdPairK)) <= kCuLds, "two workgroups per CU");
static_assert(sizeof(BwdLds<8>) + 64 + bwd_dynamic_lds(kBwdWideK) <= kCuLds, "one workgroup of eight waves");
static_assert(sizeof(BwdLds<4>) + 64 + bwd_dynamic_lds(QR_MAX_K) <= kCuLds, "the largest K fits");

}  // namespace qr

using namespace qr;

// QR_LAUNCH(feature type, waves, how the columns lie) for the runtime values.
#define QR_BWD_DISPATCH_NW(dt, NW, SPAN)              \
  switch (dt) {                                       \
    case QR_F32: QR_LAUNCH(QR_F32, NW, SPAN); break;  \
    case QR_BF16: QR_LAUNCH(QR_BF16, NW, SPAN); break; \
    default: QR_LAUNCH(QR_FP8_E4M3, NW, SPAN); break; \
  }
#define QR_BWD_DISPATCH_SPAN(dt, NW, dim)                            \
  if ((dim) <= 256) { QR_BWD_DISPATCH_NW(dt, NW, kSpanPart) }        \
  else if ((dim) <= 512) { QR_BWD_DISPATCH_NW(dt, NW, kSpanAll) }    \
  else { QR_BWD_DISPATCH_NW(dt, NW, kSpanRounds) }
#define QR_BWD_DISPATCH(dt, eight, dim)                              \
  do {                                                               \
    if (eight) { QR_BWD_DISPATCH_SPAN(dt, 8, dim) }                  \
    else { QR_BWD_DISPATCH_SPAN(dt, 4, dim) }                        \
  } while (0)

extern "C" int qr_render_quantile_backward(void* stream, int32_t width, int32_t height,
                                           const qr_params* prm, int32_t K,
                                           const uint32_t* tile_offsets, const uint32_t* sorted_gid,
                                           const float* means2d, const float* conic_opacity,
                                           const void* features, int32_t dtype,
                                           const float* feature_scale, int32_t dim,
                                           const float* grad_out, float* grad_features,
                                           float* grad_means2d, float* grad_conic_opacity) {
  int rc = validate_render("qr_render_quantile_backward", width, height, prm, tile_offsets,
                           sorted_gid, means2d, conic_opacity, features, dtype, feature_scale, dim,
                           grad_out);
  if (rc != QR_OK) return rc;
  if (K < 1 || K > QR_MAX_K)
    return fail(QR_ERR_UNSUPPORTED, "qr_render_quantile_backward: K = %d outside [1, %d]", K, QR_MAX_K);
  if (prm->selection != QR_SELECT_QUANTILE)
    return fail(QR_ERR_UNSUPPORTED, "qr_render_quantile_backward: the quantile selection only");
  const int tiles_x = static_cast<int>(ceil_div(width, kTile));
  const int tiles_y = static_cast<int>(ceil_div(height, kTile));
  const int n_tiles = tiles_x * tiles_y;
  hipStream_t s = as_stream(stream);
  const ViewArgs v{width, height, tile_offsets, sorted_gid, reinterpret_cast<const float2*>(means2d),
                   reinterpret_cast<const float4*>(conic_opacity), features, feature_scale,
                   nullptr, nullptr, nullptr};
  const GradPtrs gp{grad_out, grad_features, grad_means2d, grad_conic_opacity};
  const bool eight = K > kBwdPairK && K <= kBwdWideK;
  const size_t lds = bwd_dynamic_lds(K);
#define QR_LAUNCH(DT, NW, SPAN)                                                                              \
  hipLaunchKernelGGL((quantile_backward_kernel<DT, NW, SPAN>), dim3(n_tiles), dim3(64 * NW), lds, s, v, gp, \
                     n_tiles, *prm, K, dim)
  QR_BWD_DISPATCH(dtype, eight, dim);
#undef QR_LAUNCH
  return check_launch("qr_render_quantile_backward");
}

extern "C" int qr_render_quantile_batched_backward(void* stream, int32_t n_views,
                                                   const qr_view* views, const qr_view_grad* grads,
                                                   const qr_params* prm, int32_t K, int32_t dtype,
                                                   int32_t dim, const uint32_t* schedule,
                                                   int64_t n_items, int32_t n_workgroups,
                                                   void* workspace, size_t workspace_bytes) {
  const char* name = "qr_render_quantile_batched_backward";
  if (n_views <= 0 || n_views > (1 << (32 - kViewShift)))
    return fail(QR_ERR_INVALID_ARG, "%s: n_views = %d out of range", name, n_views);
  if (!views || !grads || !schedule || !prm) return fail(QR_ERR_INVALID_ARG, "%s: null pointer", name);
  if (n_workgroups < 0) return fail(QR_ERR_INVALID_ARG, "%s: n_workgroups < 0", name);
  if (n_workgroups > 0 && (!workspace || workspace_bytes < kBwdXcdQueues * sizeof(uint32_t)))
    return fail(QR_ERR_CAPACITY, "%s: persistent mode needs a %d-byte workspace", name,
                static_cast<int>(kBwdXcdQueues * sizeof(uint32_t)));
  if (n_items < 0 || n_items >= (1ll << 31)) return fail(QR_ERR_INVALID_ARG, "%s: bad item count", name);
  if (K < 1 || K > QR_MAX_K)
    return fail(QR_ERR_UNSUPPORTED, "%s: K = %d outside [1, %d]", name, K, QR_MAX_K);
  if (dtype != QR_F32 && dtype != QR_BF16 && dtype != QR_FP8_E4M3)
    return fail(QR_ERR_UNSUPPORTED, "%s: unknown dtype %d", name, dtype);
  if (dim <= 0 || dim % 16 != 0 || dim > QR_MAX_DIM)
    return fail(QR_ERR_UNSUPPORTED, "%s: dim = %d", name, dim);
  if (!(prm->alpha_min > 0.f) || !(prm->alpha_max >= prm->alpha_min) || !(prm->alpha_max < 1.f))
    return fail(QR_ERR_INVALID_ARG, "%s: need 0 < alpha_min <= alpha_max < 1", name);
  if (prm->selection != QR_SELECT_QUANTILE)
    return fail(QR_ERR_UNSUPPORTED, "%s: the quantile selection only", name);
  if (n_items == 0) return QR_OK;
  hipStream_t s = as_stream(stream);
  const bool eight = K > kBwdPairK && K <= kBwdWideK;
  const size_t lds = bwd_dynamic_lds(K);
  if (n_workgroups == 0) {
    const int ni = static_cast<int>(n_items);
#define QR_LAUNCH(DT, NW, SPAN)                                                                          \
  hipLaunchKernelGGL((quantile_backward_batched_grid_kernel<DT, NW, SPAN>), dim3(ni), dim3(64 * NW), lds, \
                     s, views, grads, schedule, ni, *prm, K, dim)
    QR_BWD_DISPATCH(dtype, eight, dim);
#undef QR_LAUNCH
    return check_launch(name);
  }
  auto* counter = static_cast<uint32_t*>(workspace);
  hipLaunchKernelGGL(reset_bwd_counter_kernel, dim3(1), dim3(64), 0, s, counter);
#define QR_LAUNCH(DT, NW, SPAN)                                                                           \
  hipLaunchKernelGGL((quantile_backward_batched_kernel<DT, NW, SPAN>), dim3(n_workgroups), dim3(64 * NW), \
                     lds, s, views, grads, schedule, n_items, counter, *prm, K, dim)
  QR_BWD_DISPATCH(dtype, eight, dim);
#undef QR_LAUNCH
  return check_launch(name);
}

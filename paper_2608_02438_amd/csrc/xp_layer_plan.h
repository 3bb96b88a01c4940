// How a forward of the context layer is cut up, and what its buffers take: host
// rules without a HIP call (plain C++, so that they are checked on the CPU), and
// the arithmetic of the attention's work list that the kernels share.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <array>

namespace xp {

constexpr int kPlanTile = 16;       // block positions of an attention wave (kTile)
constexpr int kHd = 128;            // head_dim (the only one built)
constexpr int kSub = 64;            // keys per attention sub-chunk (one LDS stage)
constexpr int kAttnWgs = 512;       // attention workgroups at once at most (256 CUs x 2)
constexpr size_t kScratchBytes = (size_t)64 << 20;   // the allocation-free forward's array

struct LayerDims {
  int H, nh, nkv, ffn, grp;         // grp = nh / nkv
};

// Waves of an attention workgroup: one per (query head of the group, position
// block), times KH = 2 key halves where that leaves at most eight (the two waves
// of a pair take keys 0..31 and 32..63 of every sub-chunk with their own running
// maximum, sum and O, merged at the end), so that a CU holds enough waves to
// hide each one's latency (with eight pairs the halves' extra registers cost
// more than they hide: measured).
constexpr int attn_halves(int grp, int npb) { return grp * npb <= 4 ? 2 : 1; }
constexpr int attn_waves(int grp, int npb) { return grp * npb * attn_halves(grp, npb); }
// Ring stages (32 KB each) and workgroups per CU: two workgroups of two stages,
// or one of three: with 16 waves, and with the eight of the key halves, whose
// one head-block pair in flight per wave leaves HBM latency to the ring (batch
// 32 x 16, 8192 keys: 538 us a forward with one workgroup and three stages, 556
// with two and two, 542 with one and five; batch 64 x 32: 1520 and 1476).
constexpr int attn_cu_wgs(int grp, int npb) {
  return attn_waves(grp, npb) >= 16 || grp * npb == 4 ? 1 : 2;
}

// The equal shares of a call's pre_all * nkv sub-chunks over W workgroups (W0 at
// most, and no empty share): share w is [first(w), first(w + 1)).
struct AttnShare {
  int64_t T;
  int W;
  constexpr AttnShare(int pre_all, int nkv, int W0)
      : T((int64_t)pre_all * nkv), W(T < W0 ? (int)T : W0) {}
  // (32-bit divisions where they do: 64-bit ones are a long chain at the start of
  // every workgroup)
  constexpr int64_t first(int w) const {
    return T < kSmall ? (int64_t)((uint32_t)T * (uint32_t)w / (uint32_t)W) : T * w / W;
  }
  // the share that holds sub-chunk f
  constexpr int of(int64_t f) const {
    return T < kSmall ? (int)((((uint32_t)f + 1) * (uint32_t)W - 1) / (uint32_t)T)
                      : (int)(((f + 1) * W - 1) / T);
  }
  static constexpr int64_t kSmall = (int64_t)1 << 22;   // times kAttnWgs stays below 2^32
};
// The other way to cut: every segment (one KV head of one sequence) of nb
// sub-chunks into min(ns, nb) equal parts, a workgroup each: part i is [first(i),
// first(i + 1)).
struct AttnSegment {
  int nb, n;
  constexpr AttnSegment(int nb, int ns) : nb(nb), n(ns < nb ? ns : nb) {}
  constexpr int first(int i) const {
    return (int)((uint32_t)nb * (uint32_t)i / (uint32_t)n);   // i <= nb < 2^15
  }
};

inline int attn_chunks(int C_max, int B, int keys) { return (C_max + B + keys - 1) / keys; }

// Attention workgroups of one call and the partials they write at most.  W equal
// shares of all sub-chunks (ns = 0; W at most one per sub-chunk that the call
// could have): (W + segments - 1) npb grp partials.  Or ns parts of every segment:
// W = segments ns workgroups, a partial slot each.
struct AttnPlan {
  int W, ns;
  size_t parts;
};
inline AttnPlan attn_shares(const LayerDims& L, int batch, int B, int W) {
  const size_t npb = (B + kPlanTile - 1) / kPlanTile;
  return {W, 0, ((size_t)W + (size_t)batch * L.nkv - 1) * npb * L.grp};
}
inline AttnPlan attn_segments(const LayerDims& L, int batch, int B, int ns) {
  const size_t npb = (B + kPlanTile - 1) / kPlanTile, W = (size_t)batch * L.nkv * ns;
  return {(int)W, ns, W * npb * L.grp};
}
// Workgroups of the call's shape that the chip holds at once.
inline size_t attn_slots(const LayerDims& L, int B) {
  return (size_t)kAttnWgs / 2 * attn_cu_wgs(L.grp, (B + kPlanTile - 1) / kPlanTile);
}
inline AttnPlan attn_plan_default(const LayerDims& L, int batch, int B, int C_max) {
  const size_t w64 = (size_t)batch * L.nkv * attn_chunks(C_max, B, kSub);
  return attn_shares(L, batch, B, (int)std::min(w64, attn_slots(L, B)));
}
// Attention partials of a layer's workspace: any default plan has at most these.
inline size_t attn_parts_max(const LayerDims& L, int max_batch, int max_B) {
  const size_t segs = (size_t)max_batch * L.nkv, npb = (max_B + kPlanTile - 1) / kPlanTile;
  return (kAttnWgs + segs) * npb * L.grp;
}
// The plan of a call whose buffers hold max_parts partials, which may be too few
// for the default; W = 0: not even one per segment fits.  Shares number their
// partials share + segment, so of the slots for f workgroups only f - segments + 1
// become shares, down to one where a part per segment just fits.  So whole parts
// of the segments are taken where they keep more workgroups busy, counted by the
// rounds they need on the chip.  The allocation-free forward at the Qwen3-8B shape,
// blocks of 16, 2000 keys: batch 28 has room for 36 shares (543 us) and takes 224
// segments (378); blocks of 32, 8000 keys: batch 14 18 shares (1630) and 112
// segments (538).  Segments wait for the longest context, which the host does not
// know: with lengths drawn from 1 to 6000 16 blocks of 32 (H 2560) take 442 us on
// 128 segments and 429 on the 90 shares there is room for.
inline AttnPlan attn_plan_fit(const LayerDims& L, int batch, int B, int C_max, size_t max_parts) {
  const AttnPlan def = attn_plan_default(L, batch, B, C_max);
  if (def.parts <= max_parts) return def;
  const size_t npb = (B + kPlanTile - 1) / kPlanTile, segs = (size_t)batch * L.nkv;
  const size_t fit = max_parts / (npb * L.grp), slots = attn_slots(L, B);
  if (fit < segs) return {0, 0, 0};
  const size_t nsub = attn_chunks(C_max, B, kSub);
  const size_t W = std::min({fit - segs + 1, segs * nsub, slots});
  size_t best = 0, bns = 1;
  for (size_t ns = 1; ns <= std::min(fit / segs, nsub); ++ns) {
    const size_t busy = segs * ns / ((segs * ns + slots - 1) / slots);
    if (busy > best) {
      best = busy;
      bns = ns;
    }
  }
  return best > W ? attn_segments(L, batch, B, (int)bns) : attn_shares(L, batch, B, (int)W);
}

// Bytes of a forward's buffers for up to Mx positions and nparts attention
// partials, in the order they are laid out (each from a 256-byte boundary).
inline std::array<size_t, 14> layer_sizes(const LayerDims& L, size_t Mx, size_t nparts,
                                          size_t gu_rows, size_t part_floats) {
  const size_t H = L.H, nhd = (size_t)L.nh * kHd, kvd = (size_t)L.nkv * kHd, F = L.ffn;
  return {Mx * H * 4,                       // x32
          Mx * H * 2,                       // u
          Mx * (nhd + 2 * kvd) * 4,         // qkv
          Mx * nhd * 2,                     // qn
          Mx * kvd * 2,                     // kb
          Mx * kvd * 2,                     // vb
          nparts * kPlanTile * kHd * 4,     // opart
          nparts * 2 * kPlanTile * 4,       // mlpart
          Mx * nhd * 2,                     // attn
          Mx * H * 4,                       // x1
          Mx * F * 2,                       // act
          Mx * H * 4,                       // h32
          (gu_rows ? gu_rows : 1) * 2 * F * 4,       // GU
          (part_floats ? part_floats : 1) * 4};      // part
}
inline size_t layer_slice(size_t bytes) { return (bytes + 255) / 256 * 256; }
inline size_t layer_bytes(const std::array<size_t, 14>& sizes) {
  size_t off = 0;
  for (size_t b : sizes) off += layer_slice(b);
  return off;
}
constexpr int kGsXChunks = 512;     // 16-byte chunks of x per position in k_gemv_sk's LDS (K <= 4096)
// The gate/up projections write fp32 [M][2 F] to GU on the stream kernel's
// path only (calls of at most one 16-position block, H within its LDS copy of
// x); the tiled GEMM and k_linear form the SwiGLU product themselves.
inline size_t gu_rows_for(const LayerDims& L, size_t Mx) {
  return (size_t)L.H <= 8 * (size_t)kGsXChunks ? std::min(Mx, (size_t)kPlanTile) : 0;
}
// Attention partials that the static array holds beside the other buffers of M
// positions; 0: not one.
inline size_t scratch_parts(const LayerDims& L, size_t M) {
  const size_t fixed = layer_bytes(layer_sizes(L, M, 0, gu_rows_for(L, M), 0)) + 2 * 256;
  const size_t per = (size_t)kPlanTile * kHd * 4 + (size_t)2 * kPlanTile * 4;   // opart + mlpart
  return fixed < kScratchBytes ? (kScratchBytes - fixed) / per : 0;
}

// ---------------------------------------------------------------------------
// A projection of more than 64 positions on the tiled GEMM: bn x bn tiles (128 or
// 256; 0: no plan) and S parts of k.
struct LayerPlan {
  int bn, S;
};
constexpr int kLayerSplitMax = 8;
constexpr int kGemmWgs = 256;       // workgroups of the persistent grid (8 XCDs x 32)
// k of a stage of the pipeline, the least that a part of k differs by
constexpr int gemm_stage_k(int bn) { return bn == 128 ? 64 : 32; }
// The nk stages in S parts, equal or a stage apart: part s is [first(s), first(s +
// 1)).  Unequal parts need S to divide 8 (ok): a workgroup's tiles lie 8 apart and
// are then all of one part, so that one stage count serves them.  (K is a multiple
// of 256, so only S = 8 on 128 x 128 tiles needs unequal parts, at odd multiples.
// Equal parts alone leave it S = 4: ffn 11008, 80 and 128 positions, 151 and 168 us
// a forward, 144 and 161 with unequal ones.)
struct SplitParts {
  int q, r8;                        // nk / S, and 8 (nk mod S) / S: no division on the device
  constexpr SplitParts(int nk, int S) : q(nk / S), r8(nk % S * 8 / S) {}
  constexpr int first(int s) const { return s * q + (s * r8 >> 3); }
  static constexpr bool ok(int nk, int S) { return nk % S == 0 || 8 % S == 0; }
};
// Tile size and parts of k of one projection: among 128 x 128 and 256 x 256
// tiles (bn dividing every stacked weight's rows) and S = 1 .. kLayerSplitMax
// (at least 512 k in every part, S M N fp32 slab values within part_floats; GLU:
// S = 1), the one with the least estimated time: rounds of one work item per
// workgroup of the persistent grid, an item costing 17 us plus its flops (the
// longest part's) at 3.6 TFLOP/s per CU on 128 x 128 tiles or 4.3 on 256 x 256
// (fitted to the launches of the Qwen3-8B projections at 128 to 2048 positions
// with 32 k a stage on both), plus one read of the slabs at 5 TB/s by the kernel
// that adds them.
inline LayerPlan layer_plan(int n0, int n1, int N, int K, int M, bool glu, size_t part_floats) {
  LayerPlan best{0, 1};
  if (M < 1) return best;
  double tbest = 0.0;
  for (int bn = 128; bn <= 256; bn *= 2) {
    if (N % bn != 0 || n0 % bn != 0 || n1 % bn != 0) continue;
    const int gk = gemm_stage_k(bn), nk = K / gk;
    if (K % gk != 0) continue;
    const double rate = bn == 128 ? 3.6e12 : 4.3e12;
    const long tiles = (long)(N / bn) * ((M + bn - 1) / bn);
    for (int S = 1; S <= (glu ? 1 : kLayerSplitMax); ++S) {
      if (!SplitParts::ok(nk, S) || (S > 1 && nk / S < 512 / gk)) continue;
      if (S > 1 && (double)S * M * N > (double)part_floats) continue;
      const long items = tiles * S;
      const double rounds = (double)((items + kGemmWgs - 1) / kGemmWgs);
      const int longest = (nk + S - 1) / S * gk;
      double t = rounds * (17e-6 + 2.0 * bn * bn * (double)longest / rate);
      if (S > 1) t += 4.0 * S * (double)M * N / 5e12;
      if (best.bn == 0 || t < tbest) {
        best = LayerPlan{bn, S};
        tbest = t;
      }
    }
  }
  return best;
}

}  // namespace xp

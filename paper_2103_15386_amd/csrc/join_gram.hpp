// Cross-matching (Sec. 4.2) and selective nearest-object search (Sec. 4.3,
// Alg. 2) for float32 vectors, inner products on the matrix cores (Sec. 4.2
// treats NEW x OLD as a tiled matrix product), results exactly those of the
// per-pair evaluation in dimension order.
//
// One wavefront per node at a time, no barriers between wavefronts, four steps:
//  1. The inner products of the block [NEW x (NEW | OLD)] of the node's <= 64 NEW
//     and <= 64 OLD sample vectors are accumulated on the matrix cores in 16 x 16
//     blocks, all of them in registers; only blocks that hold list entries are
//     computed (lower block triangle of NEW x NEW).  The operands come straight
//     from memory: four lanes read 64 consecutive bytes of a row, which is the
//     matrix instruction's own operand layout, two such steps (both halves of a
//     128-byte line) requested together.  Two forms: HALF reads 16-bit copies of
//     the vectors, each row divided by its norm (k_half_rows), 32 dimensions per
//     v_mfma_f32_16x16x32_f16; the other reads the float32 vectors themselves,
//     16 dimensions per four v_mfma_f32_16x16x4_f32.
//  2. Inner product and squared norms give every pair an approximate distance
//     whose difference from the canonical sum (one fused multiply-add per
//     dimension, in dimension order) is bounded by eps(pair), see pair_bounds.
//  3. Per sample and direction (NEW towards NEW, NEW towards OLD, OLD towards
//     NEW) the partners that may still be its nearest one are kept:
//     approx - eps <= min over partners of (approx + eps), found by reductions
//     over the accumulator blocks.  Partners whose lower bound already lies
//     beyond the threshold of the sample's list are dropped, for nothing at that
//     distance is handed on.  One partner is left as a rule, seldom a few, often
//     none.
//  4. The pairs left are listed (a pair that serves both of its samples once) and
//     dealt to the lanes; the vectors concerned are read once more, as float32,
//     and pass through an LDS tile 16 dimensions at a time, where every lane
//     accumulates the canonical distances of its pairs; the smallest
//     (distance, id) of a sample is the result.
//
// Measured (builds of 12 iterations, k = p = 32, whole build): 150,000 x 960 squared L2 97.9 ->
// 49.8 ms, 1.5 million x 96 angular 139.7 -> 113.3 ms, 100,000 x 75 cosine (p = 12, 8
// iterations) 7.97 -> 5.49 ms, against float32 operands in step 1, bounds proportional to 6 d
// and two partners per sample, direction and pass in step 4.  The tighter bounds and the pair
// list were worth as much as the halved first reading: vector-ALU instructions per node fell
// from 3600 to 2270 (62 rows of 96 dimensions).  What bounds it now: the gather (62 rows at
// 192 + 384 bytes) and the returning atomics of the hand-out (92 million results in the first
// iteration of the 1.5-million build at about 12 G/s, half of its 15.6 ms).
// The nodes are listed by the number of blocks of 16 samples they fill
// (k_gram_classify), and each class has its own build of the kernel, with the
// registers and the LDS tile that its blocks need, run by persistent wavefronts
// over the class's list.
#pragma once
#include "device_utils.hpp"
#include "kernels.hpp"

#include <type_traits>

namespace gnnd {

namespace {

constexpr int kWC = 16;    // dimensions per step of the inner-product loop
constexpr int kWLD = kWC + 4;  // row stride (floats) of the LDS tile of step 4: 16-byte aligned
                               // rows, and the 64 lanes of a 16-byte access spread evenly
                               // over the banks
constexpr int kWItems = 3;  // canonical sums per lane in one pass over the vectors

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Everything one wavefront (= one workgroup) keeps in LDS.  Rows 0..63 are the NEW samples,
// rows 64..127 the OLD samples; slots 0..63 stand for "NEW sample towards NEW", 64..127 for
// "NEW sample towards OLD", 128..191 for "OLD sample towards NEW".
struct GramLds {
  int32_t ids[128];
  // cosine: squared norms, for the canonical distance; otherwise with HALF: norm x 2^-kHalfBits
  float norms[128];
  // what the approximate distance needs of a sample: its squared norm (cosine: one over its
  // norm, 0 for a zero vector; HALF: 0); NaN for the empty rows of a 16-row block, which makes every
  // bound of their pairs NaN: never a minimum, never below a limit
  float weight[128];
  uint32_t kth[128];   // threshold of each sample's list
  // smallest upper bound of a partner's distance (order-preserving code), and what a partner's
  // lower bound must not exceed; step 4 keeps the smallest (distance, id) here instead
  union {
    struct {
      uint32_t upper[192];
      float limit[192];
    };
    unsigned long long best[192];
  };
};
// The partners left (bit per partner) stand in front of the LDS tile of step 4, which takes their
// place once the pairs have been listed from them: without it LDS held 3.1 to 3.4 wavefronts per SIMD
// where the registers leave room for 4 (1.5 million x 96 angular,
// twelve iterations, 108.3 -> 107.0 ms; with the early requests of step 4 106.0).
constexpr int kMaskWords = 2 * 192;
// Step 4 keeps the pairs to be summed and the rows they need in place of the weights.
struct PairList {
  uint16_t pair[64 * kWItems];  // row a | row b << 7 | "also the nearest-object search of b" << 14
  uint8_t wanted[128];
};
static_assert(sizeof(PairList) <= sizeof(GramLds::weight), "the pair list takes the weights' place");

// The builds of the kernel: build c holds up to rbm blocks of 16 NEW and com blocks of 16 OLD
// samples and is compiled for `waves` wavefronts per SIMD.  The shapes follow what a
// construction meets: every node of the first iteration has NEW samples only; in the next few
// iterations most have 33 to 48 NEW samples and up to 16 OLD ones; later the NEW samples dwindle
// and the OLD ones fill up.
struct GramShape {
  int rbm, com, waves;
};
__host__ __device__ constexpr GramShape gram_shape(int cls) {
  return cls == 0   ? GramShape{4, 0, 4}
         : cls == 1 ? GramShape{1, 2, 4}
         : cls == 2 ? GramShape{3, 1, 4}
         : cls == 3 ? GramShape{1, 4, 4}
         : cls == 4 ? GramShape{2, 4, 3}
         : cls == 5 ? GramShape{4, 2, 3}
                    : GramShape{4, 4, 2};
}
// Which build takes a node with rb blocks of NEW and co blocks of OLD samples: the cheapest
// one that holds them.  (Up to 16 NEW samples: class 1 with and without OLD ones, so that lists of
// up to 16 samples need one build, and no lists of nodes: see launch_join_gram.)
__host__ __device__ constexpr int gram_class(int rb, int co) {
  return co == 0 && rb > 1 ? 0 : (rb <= 1 && co <= 2) ? 1 : (rb <= 3 && co <= 1) ? 2 : rb <= 1 ? 3
         : rb <= 2 ? 4 : co <= 2 ? 5 : 6;
}
// Lists of up to 16 samples: all nodes are class 1.
constexpr bool gram_one_class(int p) { return 2 * p <= 16; }
static_assert(gram_class(1, 0) == 1 && gram_class(1, 1) == 1, "one build for p <= 8");
static_assert(kGramClasses == 7, "gram_shape and gram_class list seven builds");
// first LDS row of operand block q of a build with RBM blocks of NEW samples
template <int RBM>
__device__ constexpr int block_row(int q) {
  return q < RBM ? 16 * q : 64 + 16 * (q - RBM);
}

// The 16-bit copies (HALF): element i of row a is x_i / |a| x 2^kHalfBits, rounded to float16,
// padded with zeros to whole steps of 32.  Elements below float16's normal range are made zero
// (relative to the norm that is 2^-29), so that nothing depends on how the matrix unit treats
// denormal operands.  `rho` bounds |a - copy of a| / |a| over all rows; rows whose squared norm
// is outside [kHalfLeast, kNormMost] are NaN in the copy, and all their pairs stay in the race.
constexpr int kHalfBits = 15;
struct HalfRows {
  const _Float16* rows;
  int32_t stride;           // elements per row, a multiple of 32
  const float* rho;
};
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// Squared norms for which the bounds of step 2 hold.  Beyond 2^125 sums of them and of the inner
// products may overflow; below 2^-90 the squares of a row's elements come near the denormal range,
// and so does the product of two scaled norms.  The canonical cosine divides by the root of
// fl(|a|^2 |b|^2): that product has to be a normal number too, which it is for every pair of
// rows with squared norms in [2^-62, 2^62].
constexpr float kNormMost = 4.2535296e37f, kHalfLeast = 8.0779357e-28f;
constexpr float kCosineLeast = 2.1684043e-19f, kCosineMost = 4.6116860e18f;
constexpr float kLeastNormal = 1.1754944e-38f, kMostFinite = 3.4028235e38f;

// What a wavefront has counted over its nodes (the same in every lane).
struct GramTally {
  uint64_t found = 0, passed = 0, overflow = 0, evals = 0;
};

// Returns false where the 16-bit form has been given up (HALF only): nothing has been handed on
// or counted then.  FORM: see k_join_gram.
template <int METRIC, int FORM, bool HALF, int RBM, int COM>
__device__ __forceinline__ bool gram_node(GramLds& S, float* tile, const VecSrc& vs,
                                          const HalfRows& hr, float rho, int64_t s, int p,
                                          int merge_mode,
                                          const int32_t* __restrict__ snew,
                                          const int32_t* __restrict__ sold, int nn, int no,
                                          const NodeMeta* __restrict__ meta, uint64_t* pslot,
                                          uint64_t slots, uint64_t* __restrict__ bins,
                                          GramTally& tally) {
  using TR = JoinTraits<METRIC>;
  constexpr int NB = RBM + COM;  // operand blocks: NEW blocks first, then OLD blocks
  unsigned long long* const cmask = reinterpret_cast<unsigned long long*>(tile);
  auto tile_row = [](int row) { return row < 64 ? row : row - 64 + 16 * RBM; };
  constexpr uint32_t kNone = 0xffffffffu;
  const float kInf = __uint_as_float(0x7f800000u), kNaN = __uint_as_float(0x7fc00000u);
  // (taken anew for every node: what depends on the lane is worked out again per node
  // instead of being held in registers across the loop over nodes)
  int lane = threadIdx.x;
  asm volatile("" : "+v"(lane));
  const int L = 2 * p;
  const int64_t split = vs.split;
  const int d = vs.d;
  const float* const set_a = reinterpret_cast<const float*>(vs.a);
  const float* const set_b = reinterpret_cast<const float*>(vs.b);
  auto row_of = [=](int32_t id) {
    return (int64_t)id < split ? set_a + (int64_t)id * d : set_b + ((int64_t)id - split) * d;
  };
  const bool do_nn = !merge_mode && nn > 1;
  // lane l holds NEW sample l and OLD sample l
  const int32_t idn = lane < nn ? snew[s * L + lane] : -1;
  const int32_t ido = lane < no ? sold[s * L + lane] : -1;
  S.ids[lane] = idn;
  S.ids[64 + lane] = ido;
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    S.upper[64 * t + lane] = kNone;
    cmask[64 * t + lane] = 0ull;
  }
  __syncthreads();

  const int RB = (nn + 15) >> 4;  // 16-row blocks of NEW samples
  const int CO = (no + 15) >> 4;  // 16-column blocks of OLD samples
  const bool aligned = (d & 3) == 0;
  const int l16 = lane & 15, g4 = (lane >> 4) * 4;
  // Lane (l16, g) holds dimensions 4 g .. 4 g + 3 (of the 16 of a step) of row l16 of a block,
  // for either operand: which dimension goes to which step of the contraction does not matter
  // as long as both operands agree.  rows[q] / rows[4 + q]: this lane's row of NEW / OLD block
  // q.  An empty list place reads the node's first NEW sample instead: whatever stands in its
  // row or column of a block, the NaN weight of the place keeps it out of every result.
  const float* rows[NB];
  if constexpr (!HALF) {
    const float* any_row = row_of(S.ids[0]) + g4;
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      const int32_t id = S.ids[block_row<RBM>(q) + l16];
      rows[q] = id >= 0 ? row_of(id) + g4 : any_row;
    }
  }
  // The operands of two steps, 32 dimensions of every row, are requested together: the two
  // 64-byte pieces of a row are the halves of one 128-byte line where rows are aligned to
  // lines, and memory serves a line requested at once faster than its halves requested one
  // after the other (measured on random rows: 6.5 against 5.5 TB/s).  Always all 2 NB loads,
  // so that the number of loads in flight is known where the products wait for them; where
  // the vector ends after the first of the two steps, the second reads that step once more.
  const int d_last = ((d - 1) / kWC) * kWC;
  // every step reads 16 present dimensions (FORM 2: the builds with both forms look at it here)
  const bool whole = FORM == 1 || (FORM == 2 && d % kWC == 0);
  auto fetch_one = [&](const float* src, int j) {
    // dimensions beyond the last one count as zeros
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (aligned && j + 3 < d) {
      v = *reinterpret_cast<const float4*>(src);
    } else {
      if (j + 0 < d) v.x = src[0];
      if (j + 1 < d) v.y = src[1];
      if (j + 2 < d) v.z = src[2];
      if (j + 3 < d) v.w = src[3];
    }
    return v;
  };
  auto fetch2 = [&](float4* fa, float4* fb, int d0) {
    const int d1 = d0 + kWC < d_last ? d0 + kWC : d_last;
    if (whole) {  // uniform
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        fa[q] = *reinterpret_cast<const float4*>(rows[q] + d0);
        fb[q] = *reinterpret_cast<const float4*>(rows[q] + d1);
      }
    } else {
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        fa[q] = fetch_one(rows[q] + d0, d0 + g4);
        fb[q] = fetch_one(rows[q] + d1, d1 + g4);
      }
    }
  };
  float4 opa[NB], opb[NB];
  // HALF: the same with 32 dimensions of 16 bits per step
  const _Float16* hrow[NB];
  const int h_last = hr.stride - 32;
  auto fetch_half2 = [&](int d0) {
    const int d1 = d0 < h_last ? d0 + 32 : h_last;
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      opa[q] = *reinterpret_cast<const float4*>(hrow[q] + d0);
      opb[q] = *reinterpret_cast<const float4*>(hrow[q] + d1);
    }
  };
  if constexpr (HALF) {
    const _Float16* any_row = hr.rows + (int64_t)S.ids[0] * hr.stride + 2 * g4;
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      const int32_t id = S.ids[block_row<RBM>(q) + l16];
      hrow[q] = id >= 0 ? hr.rows + (int64_t)id * hr.stride + 2 * g4 : any_row;
    }
    fetch_half2(0);
  } else {
    fetch2(opa, opb, 0);
  }

  // `special`: some sample's squared norm is outside the range in which the bounds of step 2
  // hold for every pair (see pair_is_lost)
  bool special;
  // (the float32 form of squared L2: errors of up to 8 d 2^-149 where sums are denormal numbers,
  // which the matrix unit keeps, have to be small against 24 u (na + nb))
  const float least_sum = (float)d * kLeastNormal;
  {
    // one 8-byte record per sample: the threshold of its list and its squared norm
    // (k_row_norms or k_half_rows put the float's bits where the int8 join keeps its integer norm)
    // (an empty list place: a norm of 1, which is not special)
    const uint2 none = make_uint2(0u, 0x3f800000u);
    const uint2 mn = idn >= 0 ? *reinterpret_cast<const uint2*>(&meta[idn]) : none;
    const uint2 mo = ido >= 0 ? *reinterpret_cast<const uint2*>(&meta[ido]) : none;
    const uint32_t kthn = mn.x, ktho = mo.x;
    const float nrmn = __uint_as_float(mn.y), nrmo = __uint_as_float(mo.y);
    auto weight_of = [&](int32_t id, float nrm) {
      float w = nrm;
      if (METRIC == kCosineF32)
        w = !HALF && nrm > 0.f ? 1.0f / sqrtf(nrm) : 0.f;
      return id >= 0 ? w : kNaN;
    };
    // (norms are not negative, so their bits compare as they do; NaN lies above all of them)
    const uint32_t least = METRIC == kCosineF32              ? __float_as_uint(kCosineLeast)
                           : HALF                            ? __float_as_uint(kHalfLeast)
                           : METRIC == kL2F32                ? __float_as_uint(least_sum)
                                                             : 0u;
    const uint32_t span =
        __float_as_uint(METRIC == kCosineF32 ? kCosineMost : kNormMost) - least;
    auto is_special = [&](uint32_t bits) {
      if (!HALF && METRIC == kCosineF32) bits = bits ? bits : least;  // (weight 0: distance 1)
      return bits - least > span;
    };
    special = (__ballot(is_special(mn.y)) | __ballot(is_special(mo.y))) != 0ull;
    constexpr float kScale = 1.0f / (1 << kHalfBits);
    S.norms[lane] = METRIC == kCosineF32 ? nrmn : HALF ? sqrtf(nrmn) * kScale : 0.f;
    S.norms[64 + lane] = METRIC == kCosineF32 ? nrmo : HALF ? sqrtf(nrmo) * kScale : 0.f;
    S.kth[lane] = kthn;
    S.kth[64 + lane] = ktho;
    S.weight[lane] = weight_of(idn, nrmn);
    S.weight[64 + lane] = weight_of(ido, nrmo);
  }
  // An object sampled as NEW and as OLD here is no pair (sample lists are ascending in id:
  // binary search); a merge only joins objects of different sets.
  uint32_t n_dup, new_first, old_first;
  {
    int lo = 0, hi = nn;
    while (__ballot(lo < hi) != 0ull) {
      if (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (S.ids[mid] < ido) lo = mid + 1;
        else hi = mid;
      }
    }
    n_dup = (uint32_t)__popcll(__ballot(ido >= 0 && lo < nn && S.ids[lo] == ido));
    new_first = (uint32_t)__popcll(__ballot(idn >= 0 && (int64_t)idn < split));
    old_first = (uint32_t)__popcll(__ballot(ido >= 0 && (int64_t)ido < split));
  }

  // ---- 1. inner products --------------------------------------------------------------
  // acc_no[rb][cb]: NEW rows 16 rb.. x OLD rows 16 cb..; acc_nn[rb (rb + 1) / 2 + cb], cb <= rb:
  // NEW rows 16 rb.. x NEW rows 16 cb..
  f32x4 acc_no[RBM][COM > 0 ? COM : 1], acc_nn[RBM * (RBM + 1) / 2];
#pragma unroll
  for (int rb = 0; rb < RBM; ++rb)
#pragma unroll
    for (int cb = 0; cb < COM; ++cb) acc_no[rb][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < RBM * (RBM + 1) / 2; ++t) acc_nn[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto mfma4 = [](f32x4& acc, const float4& a, const float4& b) {
    if constexpr (HALF) {
      acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a),
                                                   __builtin_bit_cast(f16x8, b), acc, 0, 0, 0);
      return;
    }
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, b.x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, b.y, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, b.z, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, b.w, acc, 0, 0, 0);
  };
  auto products = [&](const float4* op) {
#pragma unroll
    for (int rb = 0; rb < RBM; ++rb) {
      if (rb < RB) {  // uniform
#pragma unroll
        for (int cb = 0; cb < COM; ++cb)
          if (cb < CO) mfma4(acc_no[rb][cb], op[rb], op[RBM + cb]);
        if (do_nn) {
#pragma unroll
          for (int cb = 0; cb <= rb; ++cb) mfma4(acc_nn[rb * (rb + 1) / 2 + cb], op[rb], op[cb]);
        }
      }
    }
  };
  // steps 0, 2, 4, ... use opa, steps 1, 3, ... opb
  constexpr int kStep = HALF ? 32 : kWC;
  const int d_all = HALF ? hr.stride : d;
  for (int d0 = 0;;) {
    products(opa);
    if (d0 + kStep < d_all) products(opb);
    d0 += 2 * kStep;
    if (d0 >= d_all) break;
    if constexpr (HALF) fetch_half2(d0);
    else fetch2(opa, opb, d0);
  }

  // ---- 2. + 3. partners that may be the nearest one --------------------------------------
  // Bound eps of |approximate distance - canonical distance|, u = 2^-24, t = na + nb,
  // P = |a| |b| <= t / 2, so that sum|a_i b_i| <= P:
  //  - accumulating the inner product: a term passes through at most 32 + (steps) additions
  //    (HALF; 4 + (instructions) otherwise), in whatever order the instruction adds its own
  //    terms, each within 2 u of the partial sum of absolute values even if it truncates;
  //    products of float16 numbers are exact in float32.  h P.
  //  - HALF: the copies' inner product differs from that of a and b by at most
  //    (2 rho + rho^2) P (|a - a'| <= rho |a|, Cauchy-Schwarz); the product with both norms
  //    rounds four times.
  //  - the canonical sums: (d + 2) u of squared L2 sums, d u P of inner products.
  //  - the norms: HALF (d / 64 + 16) u of each, otherwise d u; the cosine divides by the very
  //    same numbers on both sides.
  // Squared L2, t - 2 dot: c1 t + c2 |value|.  1 - dot: half of c1 t and the rounding of the
  // subtraction on both sides.  Cosine, 1 - dot / sqrt(na nb): the same relative to P.
  // All of this for squared norms inside the range of their form, see pair_is_lost.
  constexpr float u = 5.9604645e-8f;
  const float h = HALF ? (float)(2 * (32 + (hr.stride >> 5))) * u
                       : (float)(2 * (4 + 4 * ((d + kWC - 1) / kWC))) * u;
  const float dot_err = 1.01f * (h + (HALF ? (2.0f + rho) * rho : 0.f)) + 16.0f * u;
  const float c1 = METRIC == kL2F32
                       ? dot_err + (float)(HALF ? (d >> 6) + 24 : d + 8) * u
                       : METRIC == kAngularF32 ? 0.5f * (dot_err + (float)(d + 8) * u)
                                               : dot_err + (float)(d + 16) * u + 4.7683716e-7f;
  const float c2 = METRIC == kL2F32 ? (float)(d + 4) * 1.02f * u : 0.f;
  // Both bounds have the form base(row) + base(column) + dot factor(row) factor(column).  The
  // c2 part of squared L2 is applied to the smallest upper bound and to the limit instead.
  auto upper_base = [&](float w) {
    if (METRIC == kL2F32) return __fmaf_rn(c1, w, w);
    if (METRIC == kAngularF32) return __fmaf_rn(c1, w, 0.5f + 1.1920929e-7f);
    return w * 0.f + (0.5f + 0.5f * c1);
  };
  auto lower_base = [&](float w) {
    if (METRIC == kL2F32) return __fmaf_rn(-c1, w, w);
    if (METRIC == kAngularF32) return __fmaf_rn(-c1, w, 0.5f - 1.1920929e-7f);
    return w * 0.f + (0.5f - 0.5f * c1);
  };
  constexpr bool kFactors = METRIC == kCosineF32 ? !HALF : HALF;  // else the same for all pairs
  const float* const factor = METRIC == kCosineF32 ? S.weight : S.norms;
  constexpr float kOne = METRIC == kL2F32 ? -2.0f : -1.0f;
  constexpr float kSame = HALF ? kOne / (1 << kHalfBits) / (1 << kHalfBits) : kOne;
  auto bound = [&](float dot, float base, float fr, float fc) {
    return kFactors ? __fmaf_rn(dot, fr * fc, base) : __fmaf_rn(dot, kSame, base);
  };
  const bool with_dups = !merge_mode && n_dup != 0;
  auto four = [](const float* at) { return *reinterpret_cast<const float4*>(at); };
  // Pair (row R = arow + 4 g + r, column brow + l16) of a block: lane (l16, g) of the block's
  // accumulator holds rows 4 g .. 4 g + 3 of column l16.  Whether the pair is one:
  auto is_pair = [&](int arow, int brow, int r, int32_t idr, int32_t idc) {
    if (brow == arow) return l16 < g4 + r;  // diagonal block of NEW x NEW: every pair once
    if (brow >= 64 && (with_dups || merge_mode))
      return merge_mode ? ((int64_t)idr < split) != ((int64_t)idc < split) : idr != idc;
    return true;
  };
  // Pairs whose approximate distance says nothing about the canonical one: a row without a
  // 16-bit copy or with infinite elements (the product is NaN), and the ends of float32's range,
  // where overflows and denormal numbers break the relative bounds.  Their products are made
  // NaN, which keeps them out of the bounds below, and they are partners left in any case.  Not
  // so empty list places and rows with NaN, whose weight is NaN (cosine: rows with NaN are at
  // distance 1).  Only nodes with `special` samples look, in loops of their own.
  auto pair_is_lost = [&](float dot, int R, int C) {
    if (METRIC == kCosineF32) {
      const float nr = S.norms[R], nc = S.norms[C], product = nr * nc;
      if (nr == 0.f || nc == 0.f) return dot != dot;  // distance 1, as the weights have it
      return dot != dot || !(product >= kLeastNormal && product <= kMostFinite &&
                             fminf(nr, nc) >= kHalfLeast);
    }
    const float larger = fmaxf(S.weight[R], S.weight[C]);
    return dot != dot || !(larger <= kNormMost) ||
           (METRIC == kL2F32 && !HALF && larger < least_sum);
  };
  auto over_pairs = [&](auto f) {  // product = f(product, row, column) of all pairs that are one
    auto block = [&](f32x4& acc, int arow, int brow) {
      const int col = brow + l16;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int R = arow + g4 + r;
        const float w = S.weight[R] + S.weight[col];
        if (w == w && is_pair(arow, brow, r, S.ids[R], S.ids[col])) acc[r] = f(acc[r], R, col);
      }
    };
#pragma unroll
    for (int rb = 0; rb < RBM; ++rb) {
      if (rb < RB) {  // uniform
#pragma unroll
        for (int cb = 0; cb < COM; ++cb)
          if (cb < CO) block(acc_no[rb][cb], 16 * rb, 64 + 16 * cb);
        if (do_nn) {
#pragma unroll
          for (int cb = 0; cb <= rb; ++cb)
            block(acc_nn[rb * (rb + 1) / 2 + cb], 16 * rb, 16 * cb);
        }
      }
    }
  };
  if (special)
    over_pairs([&](float dot, int R, int C) {
      if (!pair_is_lost(dot, R, C)) return dot;
      const uint32_t some = ord_f32(kMostFinite);  // both samples have a partner
      atomicMin(&S.upper[C < 64 ? R : 64 + R], some);
      atomicMin(&S.upper[C < 64 ? C : 64 + C], some);
      return kNaN;
    });
  // A pair of a NEW x OLD block serves the NEW sample's search among the OLD ones and the OLD
  // sample's among the NEW ones, a pair of a NEW x NEW block both of its samples.  First the
  // smallest upper bound per sample and direction: over a row's or a column's blocks inside
  // the lane, then along a row through the 16 lanes of a lane row, along a column over the
  // four lane rows, then through LDS.
  auto code_of = [&](float bound_min) {
    const float raised = METRIC == kL2F32 ? __fmaf_rn(c2, fabsf(bound_min), bound_min) : bound_min;
    return bound_min < kInf ? ord_f32(raised) : kNone;
  };
  auto rows_min = [&](const float (&m)[4], int slot0) {
    uint32_t v[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      v[r] = code_of(m[r]);
      v[r] = vmin(v[r], (uint32_t)__builtin_amdgcn_mov_dpp((int)v[r], 0x128, 0xF, 0xF, true));  // row_ror:8
      v[r] = vmin(v[r], (uint32_t)__builtin_amdgcn_mov_dpp((int)v[r], 0x124, 0xF, 0xF, true));  // row_ror:4
      v[r] = vmin(v[r], (uint32_t)__builtin_amdgcn_mov_dpp((int)v[r], 0x122, 0xF, 0xF, true));  // row_ror:2
      v[r] = vmin(v[r], (uint32_t)__builtin_amdgcn_mov_dpp((int)v[r], 0x121, 0xF, 0xF, true));  // row_ror:1
    }
    const uint32_t mine = l16 == 0 ? v[0] : l16 == 1 ? v[1] : l16 == 2 ? v[2] : v[3];
    if (l16 < 4 && mine != kNone) atomicMin(&S.upper[slot0 + g4 + l16], mine);
  };
  auto column_min = [&](float m, int slot) {
    uint32_t v = code_of(m);
    v = vmin(v, xor_lanes(v, 16, lane));
    v = vmin(v, xor_lanes(v, 32, lane));
    if (g4 == 0 && v != kNone) atomicMin(&S.upper[slot], v);
  };
  {
    float col_nn[RBM], col_no[COM > 0 ? COM : 1];
#pragma unroll
    for (int cb = 0; cb < RBM; ++cb) col_nn[cb] = kInf;
#pragma unroll
    for (int cb = 0; cb < COM; ++cb) col_no[cb] = kInf;
#pragma unroll
    for (int rb = 0; rb < RBM; ++rb) {
      if (rb < RB) {  // uniform
        const int arow = 16 * rb;
        float4 wr = four(&S.weight[arow + g4]), fr = wr;
        if (kFactors) fr = four(&factor[arow + g4]);
        const int4 idr = *reinterpret_cast<const int4*>(&S.ids[arow + g4]);
        const float base_r[4] = {upper_base(wr.x), upper_base(wr.y), upper_base(wr.z),
                                 upper_base(wr.w)};
        const float fac_r[4] = {fr.x, fr.y, fr.z, fr.w};
        const int32_t id_r[4] = {idr.x, idr.y, idr.z, idr.w};
        auto fold = [&](const f32x4& acc, int brow, float (&row)[4], float& col_min) {
          const int col = brow + l16;
          const float base_c = upper_base(S.weight[col]);
          const float fac_c = kFactors ? kOne * factor[col] : 0.f;
          const int32_t idc = S.ids[col];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            float v = bound(acc[r], base_r[r] + base_c, fac_r[r], fac_c);
            v = is_pair(arow, brow, r, id_r[r], idc) ? v : kNaN;
            row[r] = fminf(row[r], v);
            col_min = fminf(col_min, v);
          }
        };
        if (COM > 0 && CO > 0) {
          float row[4] = {kInf, kInf, kInf, kInf};
#pragma unroll
          for (int cb = 0; cb < COM; ++cb)
            if (cb < CO) fold(acc_no[rb][cb], 64 + 16 * cb, row, col_no[cb]);
          rows_min(row, 64 + arow);
        }
        if (do_nn) {
          float row[4] = {kInf, kInf, kInf, kInf};
#pragma unroll
          for (int cb = 0; cb <= rb; ++cb)
            fold(acc_nn[rb * (rb + 1) / 2 + cb], 16 * cb, row, col_nn[cb]);
          rows_min(row, arow);
        }
      }
    }
    if (do_nn) {
#pragma unroll
      for (int cb = 0; cb < RBM; ++cb)
        if (cb < RB) column_min(col_nn[cb], 16 * cb + l16);
    }
#pragma unroll
    for (int cb = 0; cb < COM; ++cb)
      if (cb < CO) column_min(col_no[cb], 128 + 16 * cb + l16);
  }
  __syncthreads();
  // direction 0: NEW sample `lane` towards NEW, 1: NEW sample towards OLD, 2: OLD sample
  // towards NEW
  bool found[3];
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    const uint32_t up = S.upper[64 * t + lane];
    found[t] = up != kNone;
    const float lim = unord_f32(vmin(up, S.kth[t == 2 ? 64 + lane : lane]));
    S.limit[64 * t + lane] = METRIC == kL2F32 ? __fmaf_rn(c2, fabsf(lim), lim) : lim;
  }
  __syncthreads();
  // Then every pair whose lower bound exceeds neither that nor the threshold of the sample's
  // list is entered in the sample's set of partners.
#pragma unroll
  for (int rb = 0; rb < RBM; ++rb) {
    if (rb < RB) {  // uniform
      const int arow = 16 * rb;
      float4 wr = four(&S.weight[arow + g4]), fr = wr;
      if (kFactors) fr = four(&factor[arow + g4]);
      const int4 idr = *reinterpret_cast<const int4*>(&S.ids[arow + g4]);
      const float base_r[4] = {lower_base(wr.x), lower_base(wr.y), lower_base(wr.z),
                               lower_base(wr.w)};
      const float fac_r[4] = {fr.x, fr.y, fr.z, fr.w};
      const int32_t id_r[4] = {idr.x, idr.y, idr.z, idr.w};
      auto fold = [&](const f32x4& acc, int brow, const float4& row_limit) {
        const bool nn_block = brow < 64;
        const int col = brow + l16;
        const float base_c = lower_base(S.weight[col]);
        const float fac_c = kFactors ? kOne * factor[col] : 0.f;
        const int32_t idc = S.ids[col];
        const int col_slot = nn_block ? col : 64 + col;
        const float col_limit = S.limit[col_slot];
        const float lim[4] = {row_limit.x, row_limit.y, row_limit.z, row_limit.w};
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float v = bound(acc[r], base_r[r] + base_c, fac_r[r], fac_c);
          v = is_pair(arow, brow, r, id_r[r], idc) ? v : kNaN;
          const int R = arow + g4 + r;
          if (v <= lim[r]) atomicOr(&cmask[(nn_block ? 0 : 64) + R], 1ull << (col & 63));
          if (v <= col_limit) atomicOr(&cmask[col_slot], 1ull << R);
        }
      };
      if (COM > 0 && CO > 0) {
        const float4 row_limit = four(&S.limit[64 + arow + g4]);
#pragma unroll
        for (int cb = 0; cb < COM; ++cb)
          if (cb < CO) fold(acc_no[rb][cb], 64 + 16 * cb, row_limit);
      }
      if (do_nn) {
        const float4 row_limit = four(&S.limit[arow + g4]);
#pragma unroll
        for (int cb = 0; cb <= rb; ++cb)
          fold(acc_nn[rb * (rb + 1) / 2 + cb], 16 * cb, row_limit);
      }
    }
  }
  if (special)
    over_pairs([&](float dot, int R, int C) {
      if (dot != dot) {
        atomicOr(&cmask[C < 64 ? R : 64 + R], 1ull << (C & 63));
        atomicOr(&cmask[C < 64 ? C : 64 + C], 1ull << R);
      }
      return dot;
    });
  __syncthreads();

  // ---- 4. canonical distances of the partners left --------------------------------------
  // The pairs of all samples and directions are listed, a pair that serves both of its samples
  // once (by the one with the smaller number, or the NEW one), and dealt to the lanes,
  // kWItems each in one pass over the vectors.
  uint64_t todo[3] = {0ull, 0ull, cmask[128 + lane]};  // partners left to be listed, by direction
  uint64_t mutual[2];
  {
    const uint64_t c_nn = cmask[lane], c_no = cmask[64 + lane];
    mutual[0] = mutual[1] = 0ull;
    for (uint64_t left = c_nn; __ballot(left != 0ull) != 0ull;) {
      if (left != 0ull) {
        const int v = __ffsll((unsigned long long)left) - 1;
        left &= left - 1;
        const bool both = ((cmask[v] >> lane) & 1ull) != 0ull;
        if (both) mutual[0] |= 1ull << v;
        if (!both || lane < v) todo[0] |= 1ull << v;
      }
    }
    for (uint64_t left = c_no; __ballot(left != 0ull) != 0ull;) {
      if (left != 0ull) {
        const int v = __ffsll((unsigned long long)left) - 1;
        left &= left - 1;
        if (((cmask[128 + v] >> lane) & 1ull) != 0ull) mutual[1] |= 1ull << v;
      }
    }
    todo[1] = c_no;
    for (uint64_t left = todo[2]; __ballot(left != 0ull) != 0ull;) {
      if (left != 0ull) {
        const int v = __ffsll((unsigned long long)left) - 1;
        left &= left - 1;
        if (((cmask[64 + v] >> lane) & 1ull) != 0ull) todo[2] &= ~(1ull << v);
      }
    }
  }
#pragma unroll
  for (int t = 0; t < 3; ++t) S.best[64 * t + lane] = kKeyMax;
  PairList& list = *reinterpret_cast<PairList*>(S.weight);
  for (bool first = true;; first = false) {
    // places of this lane's pairs among all of them
    const uint32_t count =
        (uint32_t)(__popcll(todo[0]) + __popcll(todo[1]) + __popcll(todo[2]));
    if (__ballot(count != 0u) == 0ull) break;
    uint32_t inc = count;
    inc += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)inc, 0x111, 0xF, 0xF, false);  // row_shr:1
    inc += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)inc, 0x112, 0xF, 0xF, false);  // row_shr:2
    inc += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)inc, 0x114, 0xF, 0xF, false);  // row_shr:4
    inc += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)inc, 0x118, 0xF, 0xF, false);  // row_shr:8
    inc += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)inc, 0x142, 0xA, 0xF, false);  // row_bcast:15
    inc += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)inc, 0x143, 0xC, 0xF, false);  // row_bcast:31
    const uint32_t all = __builtin_amdgcn_readlane(inc, 63);
    // (three passes and more; two cost less than the float32 form's first reading)
    if (HALF && first && all > 2u * 64u * kWItems) return false;
    const uint32_t here = all < 64u * kWItems ? all : 64u * kWItems;
    __syncthreads();  // the weights, or the list before this one, are no longer needed
    reinterpret_cast<uint16_t*>(list.wanted)[lane] = 0;
    __syncthreads();
    {
      uint32_t at = inc - count;
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        while (todo[t] != 0ull && at < 64u * kWItems) {
          const int v = __ffsll((unsigned long long)todo[t]) - 1;
          todo[t] &= todo[t] - 1;
          const int a = t == 2 ? 64 + lane : lane, b = t == 1 ? 64 + v : v;
          const uint32_t both = t < 2 ? (uint32_t)((mutual[t < 2 ? t : 0] >> v) & 1ull) : 0u;
          list.pair[at] = (uint16_t)(a | (b << 7) | (both << 14));
          list.wanted[a] = list.wanted[b] = 1;
          ++at;
        }
      }
    }
    __syncthreads();
    // The vectors concerned come like the operands of the float32 form of step 1 (the others'
    // places read the node's first NEW sample) and are laid out in LDS row by row, 16
    // dimensions at a time; every lane then adds these 16 dimensions, in order, to the sums of
    // its pairs.
    {
      const float* any_row = row_of(S.ids[0]) + g4;
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        const int row = block_row<RBM>(q) + l16;
        rows[q] = list.wanted[row] ? row_of(S.ids[row]) + g4 : any_row;  // (wanted: id >= 0)
      }
    }
    uint32_t pair[kWItems];
    const float *pa[kWItems], *pb[kWItems];
    float sum[kWItems];
#pragma unroll
    for (int i = 0; i < kWItems; ++i) {
      pair[i] = 64u * i + lane < here ? list.pair[64 * i + lane] : 0x8000u;  // bit 15: none
      pa[i] = tile + tile_row((int)(pair[i] & 127u)) * kWLD;
      pb[i] = tile + tile_row((int)((pair[i] >> 7) & 127u)) * kWLD;
      sum[i] = 0.f;
    }
    auto sums = [&](const float4* op, int d0, auto then) {
      __syncthreads();  // the tile has been read
#pragma unroll
      for (int q = 0; q < NB; ++q)
        *reinterpret_cast<float4*>(tile + (16 * q + l16) * kWLD + g4) = op[q];
      __syncthreads();
      then();
      const int width = (d - d0) < kWC ? (d - d0) : kWC;
      int j = 0;
      for (; j + 3 < width; j += 4) {
#pragma unroll
        for (int i = 0; i < kWItems; ++i) {
          if (64u * i < here) {  // uniform
            const float4 va = four(pa[i] + j), vb = four(pb[i] + j);
            TR::step(va.x, vb.x, sum[i]);
            TR::step(va.y, vb.y, sum[i]);
            TR::step(va.z, vb.z, sum[i]);
            TR::step(va.w, vb.w, sum[i]);
          }
        }
      }
      for (; j < width; ++j) {
#pragma unroll
        for (int i = 0; i < kWItems; ++i)
          if (64u * i < here) TR::step(pa[i][j], pb[i][j], sum[i]);
      }
    };
    fetch2(opa, opb, 0);
    for (int d0 = 0;;) {
      // (the next two steps are requested before the sums of the second of these two, whose operands
      // are in LDS by then: 150,000 x 960 49.5 -> 47.9 ms, 1.5 million x 96 108.3 -> 107.1 ms)
      auto next = [&]() { if (d0 + 2 * kWC < d) fetch2(opa, opb, d0 + 2 * kWC); };
      auto none = []() {};
      sums(opa, d0, none);
      if (d0 + kWC < d) sums(opb, d0 + kWC, next);
      d0 += 2 * kWC;
      if (d0 >= d) break;
    }
#pragma unroll
    for (int i = 0; i < kWItems; ++i) {
      if (64u * i + lane < here) {
        const int a = (int)(pair[i] & 127u), b = (int)((pair[i] >> 7) & 127u);
        // (cosine: the norms; not used otherwise)
        const uint64_t code = (uint64_t)TR::code(sum[i], S.norms[a], S.norms[b]) << 32;
        // results for NEW towards NEW lie at 0..63, NEW towards OLD at 64.., OLD towards NEW
        // at 128..
        const int shift = (a | b) < 64 ? 0 : 64;
        atomicMin(&S.best[a + shift], (unsigned long long)(code | (uint32_t)S.ids[b]));
        if (pair[i] & 0x4000u)
          atomicMin(&S.best[b + shift], (unsigned long long)(code | (uint32_t)S.ids[a]));
      }
    }
  }
  __syncthreads();
  uint64_t best[3];
#pragma unroll
  for (int t = 0; t < 3; ++t) best[t] = S.best[64 * t + lane];

  // ---- hand the results on --------------------------------------------------------------
  uint32_t n_found = 0, n_pass = 0, n_over = 0;
  bool pass[3];
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    pass[t] = best[t] != kKeyMax && (uint32_t)(best[t] >> 32) <= S.kth[t == 2 ? 64 + lane : lane];
    n_found += (uint32_t)__popcll(__ballot(found[t]));
    n_pass += (uint32_t)__popcll(__ballot(pass[t]));
  }
  // one returning add yields the start of the destination's segment of the proposal array and
  // this result's place in it; the two results of a NEW sample share one
  auto entry_of = [](uint64_t b) { return make_entry((uint32_t)(b >> 32), (uint32_t)b, 3u); };
  auto reserve = [&](int32_t self, uint64_t results) {
    const uint64_t w = atomicAdd(reinterpret_cast<unsigned long long*>(&pslot[self]),
                                 (unsigned long long)results);
    return (w >> kSlotCountBits) + (w & kSlotCountMask);
  };
  bool over = false;
  if (pass[0] || pass[1]) {
    const uint64_t both = pass[0] && pass[1] ? 1ull : 0ull;
    const uint64_t at = reserve(idn, 1ull + both);
    if (at + both < slots) {
      bins[at] = entry_of(pass[0] ? best[0] : best[1]);
      if (both) bins[at + 1] = entry_of(best[1]);
    } else {
      over = true;
    }
  }
  if (pass[2]) {
    const uint64_t at = reserve(ido, 1ull);
    if (at < slots) bins[at] = entry_of(best[2]);
    else over = true;
  }
  n_over = (uint32_t)__popcll(__ballot(over));
  tally.found += n_found;
  tally.passed += n_pass;
  tally.overflow += n_over;
  // pairs that count as evaluated: NEW x OLD without the objects sampled as both (a merge:
  // pairs across the two sets), and all pairs of NEW samples
  const uint64_t fa = new_first, fb = old_first;
  tally.evals += merge_mode ? fa * ((uint64_t)no - fb) + ((uint64_t)nn - fa) * fb
                            : (uint64_t)nn * no - n_dup;
  if (do_nn) tally.evals += (uint64_t)nn * (nn - 1) / 2;
  return true;
}

// CLS: the build (gram_shape); it takes the nodes of its class from that class's list.  The
// accumulators of all blocks and two sets of operands live in registers, and a build for
// fewer blocks runs more wavefronts per SIMD and reads and multiplies fewer empty blocks.
// Persistent wavefronts: wavefront w takes the list's places w, w + (number of wavefronts), ...
// FORM: 0, 1 - there are no 16-bit copies (1: the dimension is a multiple of 16); 2 - there are.
//
// The error of the 16-bit copies is relative to the rows' norms.  Where the distances are small
// against those (vectors far from the origin, directions close to each other) it leaves too many
// partners; such a node is worked on once more in the float32 form, and where that happens often
// the 16-bit form is hardly tried any more (FormTally).
// Builds of 200,000 x 96 Gaussian vectors, k = p = 32, six iterations, squared L2, offset from the
// origin 0 / 10 / 30 standard deviations: 11.0 / 13.4 / 17.9 ms; with the 16-bit form for all nodes
// 11.1 / 13.4 / 44.1, with the float32 form for all of them in the build made for it alone 14.7 /
// 15.5 / 21.6 (measured before steps 2 and 4 took their present form).
template <int METRIC, int FORM, int CLS>
__global__ __launch_bounds__(kWave)
__attribute__((amdgpu_waves_per_eu(gram_shape(CLS).waves, gram_shape(CLS).waves))) void k_join_gram(
    VecSrc vs, HalfRows hr, int64_t n, int p, int merge_mode, const int32_t* __restrict__ snew,
    const int32_t* __restrict__ sold, const int32_t* __restrict__ cnew,
    const int32_t* __restrict__ cold, const NodeMeta* __restrict__ meta, uint64_t* pslot,
    uint64_t slots, uint64_t* __restrict__ bins, uint64_t* counters,
    uint64_t* forms, const int32_t* __restrict__ nodes, const uint32_t* __restrict__ count) {
  constexpr int RBM = gram_shape(CLS).rbm, COM = gram_shape(CLS).com;
  constexpr int NB = RBM + COM;
  constexpr int cls = CLS;
  __shared__ __attribute__((aligned(16))) GramLds S;
  // step 4: 16 dimensions of every vector the build can hold, operand block after operand block
  static_assert(NB * 16 * kWLD >= kMaskWords, "the tile holds the partners' masks");
  __shared__ __attribute__((aligned(16))) float tile[NB * 16 * kWLD];
  // (count NULL: every node is this build's)
  const uint32_t mine = count ? count[cls] : (uint32_t)n;
  const int32_t* const list = nodes + (int64_t)cls * n;
  GramTally tally;
  constexpr bool kCopies = FORM == 2;
  const float rho = kCopies ? *hr.rho : 0.f;
  FormTally first_form(kCopies ? *forms : 0ull);
  for (uint32_t i = blockIdx.x; i < mine; i += gridDim.x) {
    const int64_t s = count ? list[i] : (int64_t)i;
    const int nn = cnew[s], no = cold[s];
    if (!count && (nn == 0 || (no == 0 && (merge_mode || nn == 1)))) continue;  // nothing to do
    bool done = false;
    if constexpr (kCopies) {
      if (first_form.promising((uint32_t)s)) {
        done = gram_node<METRIC, FORM, true, RBM, COM>(S, tile, vs, hr, rho, s, p, merge_mode,
                                                       snew, sold, nn, no, meta, pslot, slots,
                                                       bins, tally);
        first_form.count(!done);
        __syncthreads();  // the LDS arrays are taken over by the next node (or form)
      }
    }
    if (!done) {
      gram_node<METRIC, FORM, false, RBM, COM>(S, tile, vs, hr, rho, s, p, merge_mode, snew, sold,
                                               nn, no, meta, pslot, slots, bins, tally);
      __syncthreads();
    }
  }
  if (threadIdx.x == 0) {
    uint64_t* cs = counters + (blockIdx.x & (kStripes - 1)) * C_SLOTS;
    if (tally.passed) atomicAdd(reinterpret_cast<unsigned long long*>(cs + C_PASSED),
                                (unsigned long long)tally.passed);
    if (tally.overflow) atomicAdd(reinterpret_cast<unsigned long long*>(cs + C_OVERFLOW),
                                  (unsigned long long)tally.overflow);
    if (tally.found) atomicAdd(reinterpret_cast<unsigned long long*>(cs + C_PROPS),
                               (unsigned long long)tally.found);
    if (tally.evals) atomicAdd(reinterpret_cast<unsigned long long*>(cs + C_EVALS),
                               (unsigned long long)tally.evals);
    if (kCopies && first_form.own != 0ull && FormTally::in_64(blockIdx.x))
      atomicAdd(reinterpret_cast<unsigned long long*>(forms), (unsigned long long)first_form.own);
  }
}

}  // namespace

// All builds of one metric; the source files that instantiate it differ in the metric alone (one
// file for all three takes minutes to compile).  `mm`: merge mode, `grid`: workgroups per build.
template <int METRIC>
void launch_gram_builds(const Shape& sh, const DevState& ds, int mm, unsigned grid, hipStream_t st) {
  VecSrc vs{sh.vec_a, sh.vec_b, sh.split, sh.d, sh.norms};
  const uint64_t slots = (uint64_t)sh.slots();
  const HalfRows hr{static_cast<const _Float16*>(ds.half_rows), (int32_t)half_row_elems(sh.d),
                    reinterpret_cast<const float*>(ds.half_info)};
  // (in a merge no node without OLD samples has work to do; lists of up to 2p samples do not
  // reach every class: a launch over an empty list still costs 3 to 4 microseconds)
  bool reached[kGramClasses] = {false};
  for (int rb = 1; rb <= (2 * sh.p + 15) / 16; ++rb)
    for (int co = mm ? 1 : 0; co <= (2 * sh.p + 15) / 16; ++co)
      reached[gram_class(rb, co)] = true;
  auto builds = [&](auto form) {
    constexpr int F = decltype(form)::value;
    auto build = [&](auto cls) {
      constexpr int C = decltype(cls)::value;
      if (reached[C])
        k_join_gram<METRIC, F, C><<<grid, kWave, 0, st>>>(
            vs, hr, sh.n, sh.p, mm, ds.snew, ds.sold, ds.cnew, ds.cold, ds.meta, ds.pslot, slots,
            ds.bins, ds.counters, ds.forms, ds.cls_nodes,
            gram_one_class(sh.p) ? nullptr : ds.cls_count);
    };
    build(std::integral_constant<int, 0>{});
    build(std::integral_constant<int, 1>{});
    build(std::integral_constant<int, 2>{});
    build(std::integral_constant<int, 3>{});
    build(std::integral_constant<int, 4>{});
    build(std::integral_constant<int, 5>{});
    build(std::integral_constant<int, 6>{});
  };
  if (ds.half_rows) builds(std::integral_constant<int, 2>{});
  else if (sh.d % kWC == 0) builds(std::integral_constant<int, 1>{});
  else builds(std::integral_constant<int, 0>{});
}

}  // namespace gnnd

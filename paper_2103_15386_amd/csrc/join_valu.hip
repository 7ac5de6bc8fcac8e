// Cross-matching (Sec. 4.2) and selective nearest-object search (Sec. 4.3,
// Alg. 2) for one node per workgroup, canonical arithmetic: every distance is
// accumulated per pair, one fused multiply-add per dimension in dimension
// order (exact int32 for bytes), so results are bit-identical to a sequential
// evaluation.
//
// Layout: the node's <= 64 NEW and <= 64 OLD sample vectors are staged through
// LDS in chunks of 64 dimensions (coalesced row reads from HBM); the 64 x 128
// block of distances [NEW x (NEW | OLD)] is register-tiled 4 x 8 per thread (2 x 4 for lists of
// up to 32 samples)
// over a 16 x 16 thread grid with the rows/columns of a thread 16 apart, so
// partially filled lists switch whole 16 x 16 sub-blocks off uniformly.  Only
// the lower block triangle of NEW x NEW is evaluated.  Per sample the nearest
// other NEW sample, the nearest OLD sample, and per OLD sample the nearest NEW
// sample are reduced straight from the register tiles; three wavefronts, one
// lane per sample, hand the results on.
//
// Chi-square: its terms are divided with correct rounding, some 20 issue slots per dimension and
// pair.  All pairs are therefore summed with the reciprocal instruction first (8 slots); the
// difference from the canonical sum is bounded relative to the sum, because no term is negative,
// and the few pairs that can be a sample's nearest one within that bound (one per sample and
// direction as a rule) are summed once more in the canonical arithmetic.  A node whose vectors
// leave the range the bound is derived for, or with more such pairs than the list holds, is
// evaluated in the canonical arithmetic throughout; where that was more than every third node
// (negative values, ties en masse) the others are hardly tried any more (FormTally).
// 100,000 x 96, k = 20, p = 16, 6 iterations: 21.7 -> 12.3 ms per build together with the smaller
// build for lists of up to 32 samples (at the registers and LDS of 64-sample lists the first pass
// alone gave 1 %: the phases of three workgroups per CU did not overlap; with 128 registers, four
// workgroups, 60,000 x 96, k = p = 32 takes 13.8 ms instead of 23.3 with the canonical sums alone),
// 10.9 ms with the pairs dealt one by one (kDealt) and the range looked at by one maximum over the
// values' bits (13.8 -> 13.5 ms at k = p = 32).
// Where values are negative throughout: 19.7 ms, against 19.3 with the canonical sums alone and
// 30.9 with both for every node.  Bound: vector-ALU issue.
#include "device_utils.hpp"
#include "kernels.hpp"

namespace gnnd {

constexpr int kJB = 256;      // threads per workgroup
constexpr int kDC = 64;       // dimensions per staged chunk
constexpr int kLD = kDC + 4;  // LDS row stride (elements), keeps 16-byte alignment
constexpr int kDLD = 129;     // row stride of the distance matrix in LDS

// Stage dimensions [d0, d0 + kDC) of one vector into an LDS row (as the
// accumulation type), zero beyond the vector's end.  16 threads per row.
template <typename ACC>
__device__ inline void stage_row(ACC* dst, const float* src, int d, int d0, int part,
                                 bool aligned) {
  const int j = d0 + part * 4;
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  if (src != nullptr) {
    if (aligned && j + 3 < d) {
      v = *reinterpret_cast<const float4*>(src + j);
    } else {
      if (j + 0 < d) v.x = src[j + 0];
      if (j + 1 < d) v.y = src[j + 1];
      if (j + 2 < d) v.z = src[j + 2];
      if (j + 3 < d) v.w = src[j + 3];
    }
  }
  *reinterpret_cast<float4*>(dst + part * 4) = v;
}
template <typename ACC>
__device__ inline void stage_row(ACC* dst, const uint8_t* src, int d, int d0, int part,
                                 bool aligned) {
  const int j = d0 + part * 4;
  int4 v = make_int4(0, 0, 0, 0);
  if (src != nullptr) {
    if (aligned && j + 3 < d) {
      uint32_t w = *reinterpret_cast<const uint32_t*>(src + j);
      v = make_int4((int)(w & 0xff), (int)((w >> 8) & 0xff), (int)((w >> 16) & 0xff),
                    (int)(w >> 24));
    } else {
      if (j + 0 < d) v.x = src[j + 0];
      if (j + 1 < d) v.y = src[j + 1];
      if (j + 2 < d) v.z = src[j + 2];
      if (j + 3 < d) v.w = src[j + 3];
    }
  }
  *reinterpret_cast<int4*>(dst + part * 4) = v;
}

// Chi-square sums by the reciprocal instruction (at most 1 ulp off), which costs four issue
// slots: one for two dimensions, x^2 / s + y^2 / t = (x^2 t + y^2 s) / (s t), 7 slots per
// dimension.  Values are in [0, kChiMax], so nothing overflows, and staged with kChiTiny / 2
// added, so that the sum of two zeros divides nothing by zero.
constexpr float kChiMax = 1e9f, kChiTiny = 1e-15f;
__device__ inline void chi2_two_approx(float a0, float a1, float b0, float b1, float& sum) {
  const float x = a0 - b0, s = a0 + b0, y = a1 - b1, t = a1 + b1;
  sum = __fmaf_rn(__fmaf_rn(y * y, s, (x * x) * t), __builtin_amdgcn_rcpf(s * t), sum);
}
constexpr int kChiPairs = 256;  // pairs of a node that are summed again: one per thread
// In the builds for lists of up to 32 samples the first pass deals a node's pairs to the threads
// one by one, pair q 256 + tid to thread tid: the square blocks of the canonical evaluation hold
// twice as many places as pairs where lists have 20 to 30 samples (100,000 x 96, k = 20, p = 16,
// six iterations: 12.1 -> 10.9 ms).  Lists of up to 64 keep the blocks, which reuse their rows: 60,000 x 96,
// k = p = 32, 13.8 ms with them and 14.1 with up to 2048 pairs dealt.
constexpr int kDealt = 6;  // pairs per thread
static_assert(32 * 31 / 2 + 32 * 32 <= kDealt * kJB, "all pairs are dealt");

// ALL: every evaluated pair is proposed to both of its objects (the ablation
// variant without the selective update of Sec. 4.3) instead of only the nearest
// partner per sample.
// RBM: sample lists of up to 16 RBM objects.  Lists of up to 32 (p <= 16) take half the
// registers and LDS, so that twice as many wavefronts hide each other's phases.
template <int METRIC, bool ALL, int RBM>
__global__ __launch_bounds__(kJB) void k_join_valu(
    VecSrc vs, int64_t n, int p, int merge_mode, const int32_t* __restrict__ snew,
    const int32_t* __restrict__ sold, const int32_t* __restrict__ cnew,
    const int32_t* __restrict__ cold, const NodeMeta* __restrict__ meta, uint64_t* pslot,
    uint64_t slots, uint64_t* __restrict__ bins, uint64_t* counters, uint64_t* forms) {
  using TR = JoinTraits<METRIC>;
  using T = typename TR::elem;
  using ACC = typename TR::acc;
  constexpr int kRows = 16 * RBM;  // rows of the tile: NEW samples, then as many OLD ones
  __shared__ __attribute__((aligned(16))) ACC tile[2 * kRows * kLD];
  __shared__ int32_t ids[128];
  // per sample the nearest partner: NEW towards NEW, NEW towards OLD, OLD towards NEW
  __shared__ uint64_t nearest[192];
  __shared__ uint32_t pair_count;
  __shared__ float norms_s[128];  // squared norms of the samples (cosine only)
  constexpr bool kTwice = METRIC == kChi2F32 && !ALL;
  constexpr bool kDeal = kTwice && RBM == 2;
  // kTwice: smallest approximate distance per sample and direction (code), what a partner's
  // lower bound must not exceed, the pairs to be summed again (row | column << 7 | for the row
  // << 14 | for the column << 15) and their number (large: evaluate the node canonically)
  __shared__ uint32_t min_s[kTwice ? 192 : 1];
  __shared__ float limit_s[kTwice ? 192 : 1];
  __shared__ uint32_t again_s[kTwice ? kChiPairs : 1];
  __shared__ uint32_t again_count;
  __shared__ bool twice_s;  // kTwice: this node is worth the two passes
  constexpr bool kNorms = METRIC == kCosineF32;
  static_assert(!ALL || 2 * kRows * kLD >= 64 * kDLD,
                "distance matrix must fit in the staging tile");

  const int64_t s = block_linear();
  if (s >= n) return;  // a folded grid may be longer than the node list
  const int tid = threadIdx.x;
  const int L = 2 * p;
  const int wave = tid >> 6, lane = tid & 63;
  // Wavefronts 0 and 1 each hold the NEW sample, wavefront 2 the OLD sample, one
  // object per lane; these lanes later hand on that object's result, so the
  // threshold of its list is requested now and arrives behind the staging.
  int32_t self = -1;
  if (wave < 3 && lane < L) self = (wave < 2 ? snew : sold)[s * L + lane];
  const int nn = cnew[s], no = cold[s];
  if (lane >= (wave < 2 ? nn : no)) self = -1;
  // nothing farther than the last entry of the destination list can enter it
  const uint32_t kth_self = self >= 0 ? meta[self].kth : 0u;
  if (wave == 0) ids[lane] = self;
  else if (wave == 2) ids[64 + lane] = self;
  if (kNorms && (wave == 0 || wave == 2))
    norms_s[(wave == 0 ? 0 : 64) + lane] = self >= 0 ? vs.norms[self] : 0.f;
  if (!ALL) {
    if (tid < 192) nearest[tid] = kKeyMax;
    if (tid == 0) pair_count = 0;
    if (kTwice) {
      if (tid < 192) min_s[tid] = 0xffffffffu;
      if (tid == 0) {
        again_count = 0;
        // (as the workgroups on all parts of the chip have left it, not as this part's cache has it)
        const uint64_t so_far = __hip_atomic_load(forms, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        twice_s = FormTally(so_far).promising((uint32_t)s);
      }
    }
  }
  const bool do_nn = !merge_mode && nn > 1;
  if (nn == 0 || (!do_nn && no == 0)) return;  // nothing to evaluate
  __syncthreads();

  const int tx = tid & 15, ty = tid >> 4;
  const int RB = (nn + 15) >> 4;  // active 16-row blocks (NEW)
  const int CO = (no + 15) >> 4;  // active 16-column blocks (OLD)
  const int d = vs.d;
  const bool aligned = (d & 3) == 0;

  ACC acc[RBM][2 * RBM];  // columns: NEW blocks, then OLD blocks
  uint32_t largest = 0u;  // kTwice: of the bits of all values this thread has staged
  // dimensions [d0, d0 + 64) of all vectors to LDS: 16 threads per row, 16 rows per pass
  auto stage = [&](int d0, bool check) {
    const int part = tid & 15;
#pragma unroll
    for (int pass = 0; pass < 2 * RBM; ++pass) {
      const int row = pass * 16 + (tid >> 4);
      const bool wanted = row < kRows ? (row < RB * 16) : (row - kRows < CO * 16);
      if (wanted) {
        const int32_t id = ids[row < kRows ? row : row - kRows + 64];
        const T* src = id >= 0 ? vs.row<T>((uint32_t)id) : nullptr;
        stage_row<ACC>(tile + row * kLD, src, d, d0, part, aligned);
        if (kTwice && check) {
          float4* const at = reinterpret_cast<float4*>(tile + row * kLD + part * 4);
          float4 v = *at;
          // (negative numbers and NaN have larger bits than kChiMax; adding 0 makes -0 one of 0)
          auto bits = [](float x) { return __float_as_uint(x + 0.f); };
          largest = vmax(largest, vmax(vmax(bits(v.x), bits(v.y)), vmax(bits(v.z), bits(v.w))));
          v.x += 0.5f * kChiTiny;
          v.y += 0.5f * kChiTiny;
          v.z += 0.5f * kChiTiny;
          v.w += 0.5f * kChiTiny;
          *at = v;
        }
      }
    }
    __syncthreads();
    return (d - d0) < kDC ? (d - d0) : kDC;
  };
  // the distances of all pairs of the tile, two dimensions per step
  auto evaluate = [&](auto step, bool check) {
#pragma unroll
    for (int r = 0; r < RBM; ++r)
#pragma unroll
      for (int c = 0; c < 2 * RBM; ++c) acc[r][c] = 0;
    for (int d0 = 0; d0 < d; d0 += kDC) {
      const int width = stage(d0, check);
      const int nsub = (width + 15) >> 4;
#pragma unroll 1
      for (int sub = 0; sub < nsub; ++sub) {
        ACC a[RBM][16];
#pragma unroll
        for (int r = 0; r < RBM; ++r) {
          if (r < RB) {
            const ACC* src = tile + (ty + 16 * r) * kLD + sub * 16;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int4 w = *reinterpret_cast<const int4*>(src + q * 4);
              a[r][q * 4 + 0] = __builtin_bit_cast(ACC, w.x);
              a[r][q * 4 + 1] = __builtin_bit_cast(ACC, w.y);
              a[r][q * 4 + 2] = __builtin_bit_cast(ACC, w.z);
              a[r][q * 4 + 3] = __builtin_bit_cast(ACC, w.w);
            }
          }
        }
#pragma unroll
        for (int c = 0; c < 2 * RBM; ++c) {
          const bool col_on = c < RBM ? (do_nn && c < RB) : (c - RBM < CO);
          if (col_on) {
            const int crow = tx + 16 * c;
            const ACC* src = tile + crow * kLD + sub * 16;
            ACC b[16];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int4 w = *reinterpret_cast<const int4*>(src + q * 4);
              b[q * 4 + 0] = __builtin_bit_cast(ACC, w.x);
              b[q * 4 + 1] = __builtin_bit_cast(ACC, w.y);
              b[q * 4 + 2] = __builtin_bit_cast(ACC, w.z);
              b[q * 4 + 3] = __builtin_bit_cast(ACC, w.w);
            }
#pragma unroll
            for (int r = 0; r < RBM; ++r) {
              if (r < RB && (c >= RBM || c <= r)) {
#pragma unroll
                for (int j = 0; j < 16; j += 2) step(a[r][j], a[r][j + 1], b[j], b[j + 1], acc[r][c]);
              }
            }
          }
        }
      }
      __syncthreads();
    }
  };

  const int64_t split = vs.split;
  auto canonical = [](ACC a0, ACC a1, ACC b0, ACC b1, ACC& sum) {
    TR::step(a0, b0, sum);
    TR::step(a1, b1, sum);
  };
  uint32_t found = 0;      // kTwice: this sample has a partner
  bool decided = false;    // kTwice: the pairs summed again have settled the node
  const bool twice = kTwice && __builtin_amdgcn_readfirstlane((int)twice_s) != 0;
  if constexpr (kTwice) if (twice) {
    const uint32_t pairs_nn = do_nn ? (uint32_t)(nn * (nn - 1) / 2) : 0u;
    const uint32_t pairs_all = pairs_nn + (uint32_t)(nn * no);
    // this thread's pairs - row | column << 7 (0..63 NEW, 64.. OLD) | "is a pair" << 14: objects in
    // both lists are none - and their sums
    uint32_t dealt_pair[kDealt];
    float sum_of[kDealt];
    auto row_of = [](uint32_t pair) { return (int)(pair & 127u); };
    auto col_of = [](uint32_t pair) { return (int)((pair >> 7) & 127u); };
    // pairs of this wavefront: rounds of 256
    const int first_pair = wave * kWave;
    const int rounds = (int)pairs_all > first_pair ? ((int)pairs_all - first_pair + kJB - 1) / kJB : 0;
    if constexpr (kDeal) {
      // NEW x NEW: samples i and (i + 1 + idx / nn) % nn, i = idx % nn, which is every pair once;
      // lanes side by side have rows and columns side by side, and no bank conflicts
      const float inv_nn = __builtin_amdgcn_rcpf((float)nn);
      const float inv_no = __builtin_amdgcn_rcpf((float)(no > 0 ? no : 1));
#pragma unroll
      for (int q = 0; q < kDealt; ++q) {
        const uint32_t idx = (uint32_t)(q * kJB + tid);
        const bool nn_pair = idx < pairs_nn;
        const int k = (int)(nn_pair ? idx : idx - pairs_nn), len = nn_pair ? nn : no;
        // (k + 0.5) / len is at least 1 / 128 away from the next whole number
        const int over = (int)(((float)k + 0.5f) * (nn_pair ? inv_nn : inv_no));
        const int rest = k - over * len;
        bool ok = idx < pairs_all;
        int R = nn_pair ? rest : over, C = nn_pair ? rest + over + 1 : 64 + rest;
        if (nn_pair && C >= nn) C -= nn;
        R = ok ? R : 0;
        C = ok ? C : 0;
        if (C >= 64) {
          const int32_t idr = ids[R], idc = ids[C];
          ok = ok && idr != idc;
          if (merge_mode) ok = ok && (((int64_t)idr < split) != ((int64_t)idc < split));
        }
        dealt_pair[q] = (uint32_t)(R | (C << 7) | (ok ? 1 << 14 : 0));
        sum_of[q] = 0.f;
      }
      for (int d0 = 0; d0 < d; d0 += kDC) {
        const int width = stage(d0, true);
        const int nsub = (width + 15) >> 4;
#pragma unroll 1
        for (int sub = 0; sub < nsub; ++sub) {
#pragma unroll
          for (int q = 0; q < kDealt; ++q) {
            if (q < rounds) {  // uniform
              const int C = col_of(dealt_pair[q]);
              const float* const pa = tile + row_of(dealt_pair[q]) * kLD + sub * 16;
              const float* const pb = tile + (C < 64 ? C : C - 64 + kRows) * kLD + sub * 16;
              float4 x[4], y[4];
#pragma unroll
              for (int j = 0; j < 4; ++j) {
                x[j] = *reinterpret_cast<const float4*>(pa + 4 * j);
                y[j] = *reinterpret_cast<const float4*>(pb + 4 * j);
              }
#pragma unroll
              for (int j = 0; j < 4; ++j) {
                chi2_two_approx(x[j].x, x[j].y, y[j].x, y[j].y, sum_of[q]);
                chi2_two_approx(x[j].z, x[j].w, y[j].z, y[j].w, sum_of[q]);
              }
            }
          }
        }
        __syncthreads();
      }
    } else {
      evaluate(chi2_two_approx, true);
    }
    if (largest > __float_as_uint(kChiMax)) again_count = kChiPairs + 1;  // (any thread's word is enough)
    // Both sums differ from the true one by at most (d + 12) u of it, u = 2^-24: a term takes
    // five (canonical) to twelve roundings, all terms are non-negative.  The absolute part
    // covers kChiTiny (values below 1e-8 are changed by it) and what is lost where squares of
    // differences and their products underflow (differences or sums below 1e-15).
    const float rel = (float)(2 * d + 48) * 5.9604645e-8f, abs_err = (float)d * 1e-14f;
    // f(r, c, R, C): every pair of this thread's tile that is one (rows R: NEW; columns C: 0..63
    // NEW, 64.. OLD)
    auto over_pairs = [&](auto f) {
#pragma unroll
      for (int r = 0; r < RBM; ++r) {
        if (r < RB) {
          const int R = ty + 16 * r;
          const int32_t idr = ids[R];
#pragma unroll
          for (int c = 0; c < 2 * RBM; ++c) {
            if (!(c < RBM ? (do_nn && c <= r) : (c - RBM < CO))) continue;
            const int C = c < RBM ? tx + 16 * c : 64 + tx + 16 * (c - RBM);
            const int32_t idc = ids[C];
            bool ok = idr >= 0 && idc >= 0;
            if (c < RBM) {
              ok = ok && (c < r || tx < ty);  // diagonal block: every pair once
            } else {
              ok = ok && idc != idr;
              if (merge_mode) ok = ok && (((int64_t)idr < split) != ((int64_t)idc < split));
            }
            if (ok) f(r, c, R, C);
          }
        }
      }
    };
    uint32_t pairs = 0;
    if constexpr (kDeal) {
#pragma unroll
      for (int q = 0; q < kDealt; ++q) {
        if (q < rounds && (dealt_pair[q] >> 14)) {
          const uint32_t code = ord_f32(sum_of[q]);
          const int R = row_of(dealt_pair[q]), C = col_of(dealt_pair[q]), to = C < 64 ? 0 : 64;
          atomicMin(&min_s[to + R], code);
          atomicMin(&min_s[to + C], code);
          pairs += to ? 1u : 0u;
        }
      }
    } else {
    uint32_t row_nn[RBM], row_no[RBM], col[2 * RBM];
#pragma unroll
    for (int r = 0; r < RBM; ++r) row_nn[r] = row_no[r] = 0xffffffffu;
#pragma unroll
    for (int c = 0; c < 2 * RBM; ++c) col[c] = 0xffffffffu;
    over_pairs([&](int r, int c, int, int) {
      const uint32_t code = ord_f32(acc[r][c]);
      if (c < RBM) row_nn[r] = vmin(row_nn[r], code);
      else row_no[r] = vmin(row_no[r], code);
      col[c] = vmin(col[c], code);
      pairs += c >= RBM ? 1u : 0u;
    });
#pragma unroll
    for (int r = 0; r < RBM; ++r) {
      if (r < RB) {
#pragma unroll
        for (int j = 1; j < 16; j <<= 1) {
          row_nn[r] = vmin(row_nn[r], xor_lanes(row_nn[r], j, lane));
          row_no[r] = vmin(row_no[r], xor_lanes(row_no[r], j, lane));
        }
        if (tx == 0) {
          if (row_nn[r] != 0xffffffffu) atomicMin(&min_s[ty + 16 * r], row_nn[r]);
          if (row_no[r] != 0xffffffffu) atomicMin(&min_s[64 + ty + 16 * r], row_no[r]);
        }
      }
    }
#pragma unroll
    for (int c = 0; c < 2 * RBM; ++c) {
      if (c < RBM ? (do_nn && c < RB) : (c - RBM < CO)) {
        col[c] = vmin(col[c], xor_lanes(col[c], 16, lane));
        col[c] = vmin(col[c], xor_lanes(col[c], 32, lane));
        if (ty == (wave << 2) && col[c] != 0xffffffffu)
          atomicMin(&min_s[c < RBM ? tx + 16 * c : 128 + tx + 16 * (c - RBM)], col[c]);
      }
    }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) pairs += __shfl_xor(pairs, off, kWave);
    if (lane == 0 && pairs) atomicAdd(&pair_count, pairs);
    __syncthreads();
    if (wave < 3) {  // (thread 64 w + l answers for slot 64 w + l)
      const uint32_t least = min_s[tid];
      found = least != 0xffffffffu ? 1u : 0u;
      // nothing beyond the threshold of the sample's list is handed on
      uint32_t code = ord_f32(__fmaf_rn(rel, unord_f32(least), unord_f32(least)) + abs_err);
      code = found ? vmin(code, kth_self) : 0u;
      limit_s[tid] = found ? unord_f32(code) : -1.0f;
    }
    __syncthreads();
    auto consider = [&](float sum, int R, int C) {
      const float lower = __fmaf_rn(-rel, sum, sum) - abs_err;
      const bool for_row = lower <= limit_s[C < 64 ? R : 64 + R];
      const bool for_col = lower <= limit_s[C < 64 ? C : 64 + C];
      if (for_row || for_col) {
        const uint32_t at = atomicAdd(&again_count, 1u);
        if (at < (uint32_t)kChiPairs)
          again_s[at] = (uint32_t)R | ((uint32_t)C << 7) | (for_row ? 1u << 14 : 0u) |
                        (for_col ? 1u << 15 : 0u);
      }
    };
    if constexpr (kDeal) {
#pragma unroll
      for (int q = 0; q < kDealt; ++q)
        if (q < rounds && (dealt_pair[q] >> 14))
          consider(sum_of[q], row_of(dealt_pair[q]), col_of(dealt_pair[q]));
    } else {
      over_pairs([&](int r, int c, int R, int C) { consider(acc[r][c], R, C); });
    }
    __syncthreads();
    const uint32_t again = __builtin_amdgcn_readfirstlane(again_count);
    decided = again <= (uint32_t)kChiPairs;
    // (of the nodes that are tried in any case: a fair sample)
    if (tid == 0 && FormTally::in_64((uint32_t)s))
      atomicAdd(reinterpret_cast<unsigned long long*>(forms),
                (1ull << 32) | (decided ? 0ull : 1ull));
    if (decided) {  // uniform
      const uint32_t pair = (uint32_t)tid < again ? again_s[tid] : 0u;
      const int R = (int)(pair & 127u), C = (int)((pair >> 7) & 127u);
      const float *pa = tile + R * kLD, *pb = tile + (C < 64 ? C : C - 64 + kRows) * kLD;
      float sum = 0.f;
      for (int d0 = 0; d0 < d; d0 += kDC) {
        const int width = stage(d0, false);
        if (pair >> 14) {
          int j = 0;
          for (; j + 3 < width; j += 4) {
            const float4 x = *reinterpret_cast<const float4*>(pa + j);
            const float4 y = *reinterpret_cast<const float4*>(pb + j);
            TR::step(x.x, y.x, sum);
            TR::step(x.y, y.y, sum);
            TR::step(x.z, y.z, sum);
            TR::step(x.w, y.w, sum);
          }
          for (; j < width; ++j) TR::step(pa[j], pb[j], sum);
        }
        __syncthreads();
      }
      const unsigned long long code = (unsigned long long)TR::code(sum) << 32;
      unsigned long long* const near = reinterpret_cast<unsigned long long*>(nearest);
      if (pair & (1u << 14)) atomicMin(&near[C < 64 ? R : 64 + R], code | (uint32_t)ids[C]);
      if (pair & (1u << 15)) atomicMin(&near[C < 64 ? C : 64 + C], code | (uint32_t)ids[R]);
    } else if (tid == 0) {
      pair_count = 0;  // (the canonical evaluation counts again)
    }
    __syncthreads();
  }
  if constexpr (kTwice) {
    if (!decided) evaluate(canonical, false);
  } else {
    // The same loops written in place: called through the lambda the builds for 64 samples take
    // 147 registers instead of 122, that is three workgroups per CU instead of four (build of
    // 1M x 128, p = 32, seven iterations: 170.9 ms against 137.8).
#pragma unroll
    for (int r = 0; r < RBM; ++r)
#pragma unroll
      for (int c = 0; c < 2 * RBM; ++c) acc[r][c] = 0;
    for (int d0 = 0; d0 < d; d0 += kDC) {
      const int width = stage(d0, false);
      const int nsub = (width + 15) >> 4;
      for (int sub = 0; sub < nsub; ++sub) {
        ACC a[RBM][16];
#pragma unroll
        for (int r = 0; r < RBM; ++r) {
          if (r < RB) {
            const ACC* src = tile + (ty + 16 * r) * kLD + sub * 16;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int4 w = *reinterpret_cast<const int4*>(src + q * 4);
              a[r][q * 4 + 0] = __builtin_bit_cast(ACC, w.x);
              a[r][q * 4 + 1] = __builtin_bit_cast(ACC, w.y);
              a[r][q * 4 + 2] = __builtin_bit_cast(ACC, w.z);
              a[r][q * 4 + 3] = __builtin_bit_cast(ACC, w.w);
            }
          }
        }
#pragma unroll
        for (int c = 0; c < 2 * RBM; ++c) {
          const bool col_on = c < RBM ? (do_nn && c < RB) : (c - RBM < CO);
          if (col_on) {
            const int crow = tx + 16 * c;
            const ACC* src = tile + crow * kLD + sub * 16;
            ACC b[16];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int4 w = *reinterpret_cast<const int4*>(src + q * 4);
              b[q * 4 + 0] = __builtin_bit_cast(ACC, w.x);
              b[q * 4 + 1] = __builtin_bit_cast(ACC, w.y);
              b[q * 4 + 2] = __builtin_bit_cast(ACC, w.z);
              b[q * 4 + 3] = __builtin_bit_cast(ACC, w.w);
            }
#pragma unroll
            for (int r = 0; r < RBM; ++r) {
              if (r < RB && (c >= RBM || c <= r)) {
#pragma unroll
                for (int j = 0; j < 16; ++j) TR::step(a[r][j], b[j], acc[r][c]);
              }
            }
          }
        }
      }
      __syncthreads();
    }
  }
  uint32_t* Dm = reinterpret_cast<uint32_t*>(tile);
  if constexpr (ALL) {
    // distances (as order-preserving codes) to LDS: Dm[row][col], col < 64 NEW, >= 64 OLD
#pragma unroll
    for (int r = 0; r < RBM; ++r)
#pragma unroll
      for (int c = 0; c < 2 * RBM; ++c) {
        const bool on = r < RB && (c < RBM ? (do_nn && c <= r) : (c - RBM < CO));
        if (on) {
          const int col = c < RBM ? (tx + 16 * c) : (64 + tx + 16 * (c - RBM));
          Dm[(ty + 16 * r) * kDLD + col] =
              TR::code(acc[r][c], kNorms ? norms_s[ty + 16 * r] : 0.f, kNorms ? norms_s[col] : 0.f);
        }
      }
  } else if (!decided) {
    // Nearest-object search straight from the register tiles.  A thread holds
    // rows R = ty + 16r and columns tx + 16c: the minimum along a row is
    // completed over the 16 lanes that share ty, the minimum along a column
    // over the lanes of the wavefront that share tx and then over the four
    // wavefronts through LDS.  Keys are (distance code, partner id), so equal
    // distances resolve to the smaller id whatever the order of reduction.
    int32_t idc[2 * RBM];
    float normc[2 * RBM];
#pragma unroll
    for (int c = 0; c < 2 * RBM; ++c) {
      idc[c] = ids[c < RBM ? (tx + 16 * c) : (64 + tx + 16 * (c - RBM))];
      normc[c] = kNorms ? norms_s[c < RBM ? (tx + 16 * c) : (64 + tx + 16 * (c - RBM))] : 0.f;
    }
    uint64_t down[2 * RBM];  // per column: nearest row object seen by this thread
#pragma unroll
    for (int c = 0; c < 2 * RBM; ++c) down[c] = kKeyMax;
    uint32_t pairs = 0;  // NEW x OLD pairs that count as evaluated
#pragma unroll
    for (int r = 0; r < RBM; ++r) {
      if (r < RB) {  // uniform over the workgroup
        const int R = ty + 16 * r;
        const int32_t idr = ids[R];
        uint64_t to_new = kKeyMax, to_old = kKeyMax;
#pragma unroll
        for (int c = 0; c < 2 * RBM; ++c) {
          const bool on = c < RBM ? (do_nn && c <= r) : (c - RBM < CO);
          if (!on) continue;
          const int32_t other = idc[c];
          bool ok = idr >= 0 && other >= 0;
          if (c < RBM) {
            ok = ok && (c < r || tx != ty);  // the diagonal block holds both orders of a pair
          } else {
            ok = ok && other != idr;
            if (merge_mode) ok = ok && (((int64_t)idr < split) != ((int64_t)other < split));
          }
          if (!ok) continue;
          const uint64_t code = (uint64_t)TR::code(acc[r][c], kNorms ? norms_s[R] : 0.f,
                                                   kNorms ? normc[c] : 0.f) << 32;
          const uint64_t here = code | (uint32_t)other, there = code | (uint32_t)idr;
          if (c < RBM) {
            to_new = vmin(to_new, here);
            if (c < r) down[c] = vmin(down[c], there);
          } else {
            ++pairs;
            to_old = vmin(to_old, here);
            down[c] = vmin(down[c], there);
          }
        }
#pragma unroll
        for (int j = 1; j < 16; j <<= 1) {
          to_new = vmin(to_new, xor_lanes(to_new, j, lane));
          to_old = vmin(to_old, xor_lanes(to_old, j, lane));
        }
        if (tx == 0) {
          if (to_new != kKeyMax) atomicMin(reinterpret_cast<unsigned long long*>(&nearest[R]),
                                           (unsigned long long)to_new);
          if (to_old != kKeyMax) nearest[64 + R] = to_old;  // rows have one writer
        }
      }
    }
#pragma unroll
    for (int c = 0; c < 2 * RBM; ++c) {
      const bool on = c < RBM ? (do_nn && c + 1 < RB) : (c - RBM < CO);
      if (on) {  // uniform over the workgroup
        uint64_t v = down[c];
        v = vmin(v, xor_lanes(v, 16, lane));
        v = vmin(v, xor_lanes(v, 32, lane));
        if (ty == (wave << 2) && v != kKeyMax)
          atomicMin(reinterpret_cast<unsigned long long*>(
                        &nearest[c < RBM ? (tx + 16 * c) : (128 + tx + 16 * (c - RBM))]),
                    (unsigned long long)v);
      }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) pairs += __shfl_xor(pairs, off, kWave);
    if (lane == 0 && pairs) atomicAdd(&pair_count, pairs);
  }
  __syncthreads();

  // wave 0: NEW samples towards NEW, wave 1: NEW towards OLD, wave 2: OLD towards NEW
  if (wave > 2) return;
  uint64_t best = kKeyMax;
  uint32_t evaluated = 0;
  uint32_t n_found = 0, n_pass = 0, n_over = 0;  // this lane's results
  if (wave == 0 && !do_nn) self = -1;
  // hand a result to the destination's segment of the proposal array: one
  // returning add yields the segment start and this result's place in it
  auto hand_on = [&](uint64_t key) {
    if (!decided) ++n_found;
    if ((uint32_t)(key >> 32) > kth_self) return;  // dropped here already
    ++n_pass;
    const uint64_t w = atomicAdd(reinterpret_cast<unsigned long long*>(&pslot[self]), 1ull);
    const uint64_t at = (w >> kSlotCountBits) + (w & kSlotCountMask);
    if (at < slots) bins[at] = make_entry((uint32_t)(key >> 32), (uint32_t)key, 3u);
    else ++n_over;
  };
  if constexpr (ALL) {
    if (wave == 0) {
      if (self >= 0) {
        for (int v = 0; v < nn; ++v) {
          if (v == lane) continue;
          const uint32_t code = ((v >> 4) <= (lane >> 4)) ? Dm[lane * kDLD + v] : Dm[v * kDLD + lane];
          hand_on(((uint64_t)code << 32) | (uint32_t)ids[v]);
        }
      }
    } else if (wave == 1) {
      if (self >= 0) {
        for (int o = 0; o < no; ++o) {
          const int32_t other = ids[64 + o];
          bool ok = other != self;
          if (merge_mode) ok = ok && (((int64_t)self < split) != ((int64_t)other < split));
          if (!ok) continue;
          ++evaluated;
          hand_on(((uint64_t)Dm[lane * kDLD + 64 + o] << 32) | (uint32_t)other);
        }
      }
    } else {
      if (self >= 0) {
        for (int u = 0; u < nn; ++u) {
          const int32_t other = ids[u];
          bool ok = other != self;
          if (merge_mode) ok = ok && (((int64_t)self < split) != ((int64_t)other < split));
          if (!ok) continue;
          hand_on(((uint64_t)Dm[u * kDLD + 64 + lane] << 32) | (uint32_t)other);
        }
      }
    }
  } else {
    if (self >= 0) best = nearest[wave * 64 + lane];
    if (wave == 1 && lane == 0) evaluated = pair_count;
  }
  if (decided && self >= 0) n_found = found;
  if (!ALL && best != kKeyMax) hand_on(best);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    n_found += __shfl_xor(n_found, off, kWave);
    n_pass += __shfl_xor(n_pass, off, kWave);
    n_over += __shfl_xor(n_over, off, kWave);
    evaluated += __shfl_xor(evaluated, off, kWave);
  }
  if (lane == 0) {
    uint64_t* cs = counters + (s & (kStripes - 1)) * C_SLOTS;
    if (n_pass) atomicAdd(reinterpret_cast<unsigned long long*>(cs + C_PASSED),
                          (unsigned long long)n_pass);
    if (n_over) atomicAdd(reinterpret_cast<unsigned long long*>(cs + C_OVERFLOW),
                          (unsigned long long)n_over);
    if (n_found) atomicAdd(reinterpret_cast<unsigned long long*>(cs + C_PROPS),
                           (unsigned long long)n_found);
    if (wave == 1) {
      const uint64_t ev = (uint64_t)evaluated + (do_nn ? (uint64_t)nn * (nn - 1) / 2 : 0);
      if (ev) atomicAdd(reinterpret_cast<unsigned long long*>(cs + C_EVALS),
                        (unsigned long long)ev);
    }
  }
}

template <bool ALL, int RBM>
static void launch_join_as(const Shape& sh, const DevState& ds, bool merge_mode, hipStream_t st) {
  VecSrc vs{sh.vec_a, sh.vec_b, sh.split, sh.d, sh.norms};
  const dim3 grid = grid_blocks(sh.n);
  const uint64_t slots = (uint64_t)sh.slots();  // size of the proposal array
  const int mm = merge_mode ? 1 : 0;
#define GNND_JOIN_ARGS vs, sh.n, sh.p, mm, ds.snew, ds.sold, ds.cnew, ds.cold, ds.meta, ds.pslot, \
                       slots, ds.bins, ds.counters, ds.forms
  switch (sh.metric) {
    case kL2F32: k_join_valu<kL2F32, ALL, RBM><<<grid, kJB, 0, st>>>(GNND_JOIN_ARGS); break;
    case kAngularF32: k_join_valu<kAngularF32, ALL, RBM><<<grid, kJB, 0, st>>>(GNND_JOIN_ARGS); break;
    case kChi2F32: k_join_valu<kChi2F32, ALL, RBM><<<grid, kJB, 0, st>>>(GNND_JOIN_ARGS); break;
    case kCosineF32: k_join_valu<kCosineF32, ALL, RBM><<<grid, kJB, 0, st>>>(GNND_JOIN_ARGS); break;
    default: k_join_valu<kL2U8, ALL, RBM><<<grid, kJB, 0, st>>>(GNND_JOIN_ARGS);
  }
#undef GNND_JOIN_ARGS
}

hipError_t launch_join(const Shape& sh, const DevState& ds, int path, bool merge_mode,
                       hipStream_t st) {
  (void)path;
  if (2 * sh.p > kWave) return launch_join_long(sh, ds, merge_mode, st);  // sample lists beyond 64
  if (sh.all_pairs) launch_join_as<true, 4>(sh, ds, merge_mode, st);
  else if (sh.p <= 16) launch_join_as<false, 2>(sh, ds, merge_mode, st);
  else launch_join_as<false, 4>(sh, ds, merge_mode, st);
  return hipGetLastError();
}

}  // namespace gnnd

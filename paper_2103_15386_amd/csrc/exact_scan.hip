// Exhaustive exact K-NN where a workspace is at hand: the matrix cores turn rows away, the
// canonical arithmetic decides among those left.  Results are those of k_exact_knn, bit for bit.
//
// For a query a and a row b let score = a.b - |b|^2 / 2 (squared L2) or a.b (angular; cosine: of
// the vectors divided by their norms): the larger the score, the smaller the distance.  The score
// of a pair is computed from float16 copies (bytes: int8 copies, exactly) by matrix instructions
// whose accumulator starts at the row's own term, and every row has two such terms: one that
// makes the result a lower bound of the canonical distance's score, and one that makes it an upper
// bound (row_slack).  So a pair costs one vector instruction behind its share of a matrix
// instruction:
//   1. k_query_norms, k_pack: copies of the queries and of all rows in the order the matrix
//      instruction reads its operands (1 KiB = 16 rows x 64 bytes), and the rows' terms.
//   2. k_scan<.., false>: every kEvery-th tile of 64 rows; the largest lower bound per query and
//      group of rows (a group: one row in 16 of the tiles a workgroup sees).
//   3. k_threshold: the K-th largest of a query's groups, without the one that holds the query
//      itself: K other rows are at least that near.
//   4. k_scan<.., true>: all tiles; rows whose upper bound reaches the threshold are listed.
//   5. k_pick: canonical distances of the listed rows, the best K in order.  A query with more
//      candidates than its list holds, or one outside the bounds' range, is left to k_exact_knn;
//      so are all of them where a row holds a NaN (2 to 4 are left out then).
//
// A workgroup of k_scan holds the operands of 256 queries in registers (64 per wavefront) and
// streams tiles of 64 rows through LDS, double buffered, each read once for all 256.
// Consecutive workgroups of one XCD take the same rows for different queries.
//
// 10^6 rows, k_exact_knn alone / this form in ms, a call among others: 2000 queries x 96 dimensions,
// angular, K = 10 9.8 / 0.58 (0.75 while the tile on its way stood in scratch memory); 2000 x 128 squared
// L2 14.7 / 0.74; 2000 x 96 bytes, K = 64 4.4 / 0.37; 100 x 96 6.9 / 0.21; 16 x 96 6.6 / 0.21; 4096 x 96,
// K = 64 22.6 / 1.11; 10,000 x 96, K = 64 72.5 / 2.64.  Tried with the tile in scratch memory, and not
// since: operands of 128 queries per wavefront, which reads half as much from LDS, 4 % less on the
// first of these calls but 0.33 instead of 0.29 ms for up to 100 queries.  Two tiles on their way
// instead of one: no change at 96 dimensions, registers spilled.
// Data the copies do not suit (distances small against the lengths, thousands of copies of a vector)
// cost the first scan on top: 500 x 200,000 x 48, unit vectors 30 off the origin in every dimension,
// 0.68 / 0.74 ms; 1000 x 200,000 x 48, queries among 20,000 copies of a vector, 0.78 / 0.84.
#include <cfloat>
#include <type_traits>

#include "device_utils.hpp"
#include "kernels.hpp"

namespace gnnd {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

constexpr int kGroupQueries = 256;  // queries per workgroup of k_scan
constexpr int kQB = 4;              // blocks of 16 queries per wavefront
constexpr int kTileRows = 64;       // rows per tile
constexpr int kRB = kTileRows / 16;
constexpr int kCap = 2048;          // candidates listed per query
constexpr int kListed = 512;        // candidates a wavefront gathers in LDS before handing them on
constexpr int kSlice = 4096;        // queries per pass over the rows
constexpr int kEvery = 4;           // one tile in kEvery finds the thresholds
constexpr int kNormParts = 64;
constexpr int kFoundStep = 16;      // words between the counters of two queries: additions to
                                    // one 64-byte line queue (75 per microsecond)

// Squared norms of queries for which the bounds hold; rows only need finite copies (and, under
// the cosine distance, products of two squared norms that are normal numbers).
constexpr float kQueryLeast = 8.6736174e-19f, kQueryMost = 1.1529215e18f;  // 2^-60, 2^60
constexpr float kUnitScale = 256.f;  // cosine: the length of a copy

struct SearchInfo {
  uint32_t norm_max[kNormParts];  // largest squared norm of a query (float bits), in parts
  uint32_t query_err;             // largest error of a query's copy (float bits)
  uint32_t no_number;             // a row holds a NaN: it is at no distance from any query, and what
                                  // order that gives is for k_exact_knn to say, so nothing is scanned
};

template <int METRIC>
struct ScoreOf {
  using type = float;
  using vec = f32x4;
};
template <>
struct ScoreOf<kL2U8> {
  using type = int32_t;
  using vec = i32x4;
};
__device__ inline float score_least(float) { return -__uint_as_float(0x7f800000u); }
__device__ inline int32_t score_least(int32_t) { return INT32_MIN; }
// a bound that no score reaches (not the infinite one of a row without a copy either)
__device__ inline float score_never(float) { return __uint_as_float(0x7fc00000u); }
__device__ inline int32_t score_never(int32_t) { return INT32_MAX; }
__device__ inline bool is_bound(float x) { return x == x; }
__device__ inline bool is_bound(int32_t x) { return x != INT32_MAX; }
__device__ inline float score_max(float a, float b) { return fmaxf(a, b); }
__device__ inline int32_t score_max(int32_t a, int32_t b) { return a < b ? b : a; }
__device__ inline uint32_t score_code(float x) { return ~ord_f32(x); }  // ascending: best first
__device__ inline uint32_t score_code(int32_t x) { return ~ord_i32(x); }
__device__ inline float code_score(uint32_t c, float) { return unord_f32(~c); }
__device__ inline int32_t code_score(uint32_t c, int32_t) { return unord_i32(~c); }

__device__ inline bool query_in_range(float norm) {
  return norm >= kQueryLeast && norm <= kQueryMost;
}

// Squared norms of the queries: the largest in range decides the common scale of the copies.
// Whether a query is in range is decided here alone (`flags`, see k_pack): the rows' terms are
// bounds only for queries whose norm is in the largest one, and k_pack's sum, in another order, may
// fall on the other side of an end of the range.
__global__ __launch_bounds__(256) void k_query_norms(const float* vec, int64_t n, int d,
                                                     const int32_t* queries, int64_t nq,
                                                     SearchInfo* info, uint8_t* flags) {
  __shared__ uint32_t most;
  if (threadIdx.x == 0) most = 0u;
  __syncthreads();
  const int lane = lane_id();
  for (int64_t q = (int64_t)blockIdx.x * 4 + wave_id(); q < nq; q += 4 * kNormParts) {
    const uint32_t id = (uint32_t)queries[q];
    if ((int64_t)id >= n) continue;
    const float* row = vec + (int64_t)id * d;
    float s = 0.f;
    for (int j = lane; j < d; j += kWave) s = __fmaf_rn(row[j], row[j], s);
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) s += __uint_as_float(xor_lanes(__float_as_uint(s), o, lane));
    if (lane == 0) {
      flags[q] = query_in_range(s) ? 0 : 1;
      if (query_in_range(s)) atomicMax(&most, __float_as_uint(s));
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    info->norm_max[blockIdx.x] = most;
    if (blockIdx.x == 0) info->query_err = info->no_number = 0u;
  }
}

// The largest norm of a query, and the power of two that brings it into [2^7, 2^8): elements of
// copies up to 2^16 / 2^8 times that norm are finite float16 numbers, and those above 2^-22 of
// it are normal ones.
__device__ inline float largest_query_norm(const SearchInfo* info, int lane) {
  uint32_t m = info->norm_max[lane];
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) m = vmax(m, xor_lanes(m, o, lane));
  return sqrtf(__uint_as_float(m));
}
__device__ inline float scale_of(float norm) {
  if (norm == 0.f) return 1.f;
  const int e = (int)(__float_as_uint(norm) >> 23) - 127;
  return __uint_as_float((uint32_t)(127 + 7 - e) << 23);
}

// How far the score from the copies (float32 accumulators of the matrix instructions) may be from
// the one that the canonical distance stands for; `a`, `b` bound the lengths of the scaled query
// and row, `ea`, `eb` the lengths of their copies' errors, `half` the row's |b|^2 / 2 (squared L2).
//  - the copies' product: ea b + eb a (a, b taken with their errors);
//  - every addition of the accumulation, in whatever order and even if it truncates: 2^-23 of
//    the sum of absolute values, which is at most a b + half; a term passes through fewer than
//    dims + 16 of them;
//  - the canonical sum: d + 4 roundings of 2^-24 relative to sum (a_i - b_i)^2 <= 2 (a^2 + b^2),
//    halved by the score, or to a b; the norms' own sums as many;
//  - angular and cosine: the rounding of 1 - dot, 2^-24 (1 + a b) in units of `one` = scale^2;
//    cosine: the rounding of product, root and quotient and of the scale, 2^-21 of a b.
// All taken at least twice, so that the roundings of this sum itself do not matter.
template <int METRIC>
__device__ inline float row_slack(float a, float ea, float b, float eb, float half, float one,
                                  int dims) {
  constexpr float u = 1.1920929e-7f;  // 2^-23
  const float ab = a * b;
  float s = ea * b + eb * a + (float)(dims + 16) * u * (ab + half);
  if (METRIC == kL2F32) s += (float)(dims + 8) * u * (a * a + b * b);
  else s += (float)(dims + 8) * (METRIC == kCosineF32 ? 3.f : 1.f) * u * ab + 2.f * u * one;
  if (METRIC == kCosineF32) s += 8.f * u * ab;
  return s * 1.01f;
}

// Copies of 16 rows per wavefront.  Lane (r, g) = (lane % 16, lane / 16) holds bytes 16 g .. of
// every 64-byte piece of row r's copy: 8 dimensions of 32 as float16, 16 of 64 as int8.
// QUERY: the rows are those of queries[0..count); `flags` tells queries out of range (1; of float
// vectors as k_query_norms has left it) and ids that are no node (2).
template <int METRIC, int CH, bool QUERY>
__global__ __launch_bounds__(256) void k_pack(const void* vec, int64_t n, int d,
                                              const int32_t* queries, int64_t count,
                                              int64_t blocks, uint4* frag,
                                              typename ScoreOf<METRIC>::type* lower,
                                              typename ScoreOf<METRIC>::type* upper,
                                              SearchInfo* info, uint8_t* flags) {
  constexpr bool kBytes = METRIC == kL2U8;
  const int64_t blk = (int64_t)blockIdx.x * 4 + wave_id();
  if (blk >= blocks) return;
  const int lane = lane_id(), g = lane >> 4;
  const int64_t at = blk * 16 + (lane & 15);
  const uint32_t id = at < count ? (QUERY ? (uint32_t)queries[at] : (uint32_t)at) : 0xffffffffu;
  const bool have = (int64_t)id < n;
  if constexpr (kBytes) {
    const uint8_t* row = static_cast<const uint8_t*>(vec) + (have ? (int64_t)id * d : 0);
    int32_t norm = 0;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int j0 = c * 64 + g * 16;
      uint32_t w[4] = {0x80808080u, 0x80808080u, 0x80808080u, 0x80808080u};
      if (have) {
        if ((d & 15) == 0) {
          if (j0 < d) {
            const uint4 x = *reinterpret_cast<const uint4*>(row + j0);
            w[0] = x.x; w[1] = x.y; w[2] = x.z; w[3] = x.w;
          }
        } else {
#pragma unroll
          for (int e = 0; e < 16; ++e)
            if (j0 + e < d)
              w[e >> 2] = (w[e >> 2] & ~(0xffu << (8 * (e & 3)))) |
                          ((uint32_t)row[j0 + e] << (8 * (e & 3)));
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        w[e] ^= 0x80808080u;  // value - 128
        norm = __builtin_amdgcn_sdot4((int)w[e], (int)w[e], norm, false);
      }
      frag[(blk * CH + c) * kWave + lane] = make_uint4(w[0], w[1], w[2], w[3]);
    }
    norm += (int32_t)xor_lanes((uint32_t)norm, 16, lane);
    norm += (int32_t)xor_lanes((uint32_t)norm, 32, lane);
    if (lane < 16) {
      if (QUERY) {
        if (at < count) flags[at] = have ? 0 : 2;
      } else {
        lower[at] = have ? -((norm + 1) >> 1) : INT32_MIN / 2;
        upper[at] = have ? -(norm >> 1) : INT32_MIN / 2;
      }
    }
  } else {
    const float* row = static_cast<const float*>(vec) + (have ? (int64_t)id * d : 0);
    float v[CH][8];
    float norm = 0.f;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int j0 = c * 32 + g * 8;
#pragma unroll
      for (int e = 0; e < 8; ++e) v[c][e] = 0.f;
      if (have) {
        if ((d & 3) == 0) {
#pragma unroll
          for (int e = 0; e < 8; e += 4)
            if (j0 + e < d) {
              const float4 x = *reinterpret_cast<const float4*>(row + j0 + e);
              v[c][e] = x.x; v[c][e + 1] = x.y; v[c][e + 2] = x.z; v[c][e + 3] = x.w;
            }
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (j0 + e < d) v[c][e] = row[j0 + e];
        }
      }
    }
    auto over_row = [&](float x) {
      x += __uint_as_float(xor_lanes(__float_as_uint(x), 16, lane));
      x += __uint_as_float(xor_lanes(__float_as_uint(x), 32, lane));
      return x;
    };
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
      for (int e = 0; e < 8; ++e) norm = __fmaf_rn(v[c][e], v[c][e], norm);
    norm = over_row(norm);
    const float a0 = largest_query_norm(info, lane);
    const float common = scale_of(a0);
    float scale = common;
    bool lost = !(norm <= FLT_MAX);
    if (METRIC == kCosineF32) {
      const bool usable = norm >= kQueryLeast && norm <= kQueryMost;
      scale = usable ? kUnitScale / sqrtf(norm) : 0.f;
      lost = !usable && norm != 0.f;  // (norm 0: at distance 1 from everything, a score of 0)
    }
    if (QUERY) lost = lost || (have && flags[at] == 1);
    float err = 0.f;
    f16x8 h[CH];
    bool finite = true;
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float x = v[c][e] * scale;
        finite = finite && fabsf(x) <= 60000.f;
        float y = (float)(_Float16)x;
        y = fabsf(y) < 6.1035156e-5f ? 0.f : y;  // (nothing depends on denormal operands)
        h[c][e] = (_Float16)y;
        err = __fmaf_rn(x - y, x - y, err);
      }
    err = sqrtf(over_row(err)) * 1.001f;
    // (lanes of other rows hold their own verdict in other bits)
    const uint64_t ok = __ballot(finite);
    const uint64_t mine = 0x0001000100010001ull << (lane & 15);
    lost = lost || (ok & mine) != mine;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      f16x8 out = h[c];
      if (lost || !have)
#pragma unroll
        for (int e = 0; e < 8; ++e) out[e] = (_Float16)0.f;
      frag[(blk * CH + c) * kWave + lane] = __builtin_bit_cast(uint4, out);
    }
    if (QUERY) {
      if (lane < 16 && at < count) {
        flags[at] = !have ? 2 : lost ? 1 : 0;
        if (have && !lost) atomicMax(&info->query_err, __float_as_uint(err));
      }
    } else if (lane < 16) {
      const float inf = __uint_as_float(0x7f800000u);
      float lo = -inf, hi = -inf;  // places behind the last row
      if (have) {
        if (norm != norm) atomicOr(&info->no_number, 1u);
        const float ea = __uint_as_float(info->query_err);
        const float unit = METRIC == kCosineF32 ? kUnitScale : a0 * common;
        const float a = unit * 1.001f + ea;
        const float b =
            (METRIC == kCosineF32 ? (norm == 0.f ? 0.f : kUnitScale) : sqrtf(norm) * common) *
                1.001f + err;
        const float half = METRIC == kL2F32 ? 0.5f * norm * common * common : 0.f;
        const float one = METRIC == kCosineF32 ? kUnitScale * kUnitScale : common * common;
        const float slack = row_slack<METRIC>(a, ea, b, err, half, one, CH * 32);
        // a row without a copy: never a bound, always a candidate
        lost = lost || !(slack <= FLT_MAX);
        lo = lost ? -inf : -half - slack;
        hi = lost ? inf : -half + slack;
      }
      lower[at] = lo;
      upper[at] = hi;
    }
  }
}

__device__ inline f32x4 mfma(const uint4& a, const uint4& b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a),
                                                __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}
__device__ inline i32x4 mfma(const uint4& a, const uint4& b, i32x4 c) {
  return __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4, a),
                                               __builtin_bit_cast(i32x4, b), c, 0, 0, 0);
}

// Tiles strip * step, (strip + strips) * step, ... against the queries of one group.
// COLLECT: rows whose score reaches bound[q] are listed in cand[q * kCap ..], counted in found[q];
// otherwise the largest score per query and row-modulo-16 goes to bound[q * 16 strips + ..].
template <int METRIC, int CH, bool COLLECT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(CH < 4 ? 4 : 3))) void k_scan(
    const uint4* __restrict__ rows, const typename ScoreOf<METRIC>::type* __restrict__ term,
    int64_t tiles, int step, int strips, int qgroups, int64_t n, const uint4* __restrict__ qfrag,
    const int32_t* __restrict__ queries, typename ScoreOf<METRIC>::type* bound, uint32_t* found,
    uint32_t* cand, const SearchInfo* __restrict__ info) {
  if (METRIC != kL2U8 && !COLLECT && info->no_number) return;  // (the second scan: no query has a bound)
  using T = typename ScoreOf<METRIC>::type;
  using V = typename ScoreOf<METRIC>::vec;
  __shared__ uint4 tile[2][kRB * CH * kWave];
  __shared__ __attribute__((aligned(16))) T terms[2][kTileRows];
  // COLLECT: candidates of a wavefront (query << 26 | row, both counted inside wavefront and strip:
  // a strip is at most 2^18 tiles) and its queries that have more than cand holds
  __shared__ uint32_t list[COLLECT ? 4 : 1][COLLECT ? kListed : 1];
  __shared__ uint8_t over[COLLECT ? 4 : 1][kWave];
  // workgroups b, b + 8, ... run on one XCD: they take the query groups of one strip in turn
  const int turn = (int)(blockIdx.x >> 3);
  const int group = turn % qgroups, strip = (turn / qgroups) * 8 + (int)(blockIdx.x & 7);
  if (strip >= strips) return;
  const int lane = lane_id(), wave = wave_id(), tid = (int)threadIdx.x;
  uint32_t listed = 0u;  // uniform
  if (COLLECT) over[wave][lane] = 0;
  uint4 b[kQB][CH];
  const int qblock = group * (kGroupQueries / 16) + wave * kQB;
#pragma unroll
  for (int q = 0; q < kQB; ++q)
#pragma unroll
    for (int c = 0; c < CH; ++c) b[q][c] = qfrag[((int64_t)(qblock + q) * CH + c) * kWave + lane];
  const int mine = wave * kQB * 16 + (lane & 15);  // this lane's query of block 0 in the group
  const int q0 = group * kGroupQueries + mine;
  T limit[kQB];
  V best[kQB];
#pragma unroll
  for (int q = 0; q < kQB; ++q) {
    if (COLLECT) limit[q] = bound[q0 + 16 * q];
#pragma unroll
    for (int i = 0; i < 4; ++i) best[q][i] = score_least(T{});
  }
  if (COLLECT) {  // nothing to look for: all queries of the group are out of the race
    bool any = false;
#pragma unroll
    for (int q = 0; q < kQB; ++q) any = any || is_bound(limit[q]);
    if (__syncthreads_or(any) == 0) return;
  }
  // What the wavefront has gathered goes to cand; a query whose list is full gets out of the race.
  // (With one list of 1024 per workgroup, handed on at the end, and the query of every row beyond it
  // given up, 4096 queries x 10^6 x 96, K = 64, all went to the general kernel: 25.1 ms, now 1.53.)
  auto hand_on = [&]() {
    wave_lds_fence();
    for (uint32_t i = lane; i < listed; i += kWave) {
      const uint32_t x = list[wave][i], at = (x >> 6) & 0xfffffu, mine64 = x >> 26;
      const uint32_t row = ((uint32_t)strip + at * (uint32_t)strips) * kTileRows + (x & 63u);
      // (below nq: it had a limit)
      const int64_t q = (int64_t)group * kGroupQueries + wave * kWave + mine64;
      if ((int64_t)row >= n || row == (uint32_t)queries[q]) continue;  // no row, the query itself
      const uint32_t to = atomicAdd(&found[q * kFoundStep], 1u);
      if (to < (uint32_t)kCap) cand[q * kCap + to] = row;
      else over[wave][mine64] = 1;
    }
    listed = 0u;
    wave_lds_fence();
#pragma unroll
    for (int q = 0; q < kQB; ++q)
      if (over[wave][16 * q + (lane & 15)]) limit[q] = score_never(T{});
  };
  // (a plain vector type: as uint4, a class, the tile on its way stood in scratch memory, for which every
  // wavefront waited for it at once)
  u32x4 reg[CH];
  T reg_term = T{};
  auto fetch = [&](int64_t t) {
    const u32x4* src = reinterpret_cast<const u32x4*>(rows) + t * (kRB * CH * kWave);
#pragma unroll
    for (int c = 0; c < CH; ++c) reg[c] = src[c * 256 + tid];
    if (tid < kTileRows) reg_term = term[t * kTileRows + tid];
  };
  auto put = [&](int at) {
#pragma unroll
    for (int c = 0; c < CH; ++c)
      *reinterpret_cast<u32x4*>(&tile[at][c * 256 + tid]) = reg[c];
    if (tid < kTileRows) terms[at][tid] = reg_term;
  };
  int64_t t = strip;
  int at = 0;
  uint32_t seen = 0;  // tiles of this strip
  if (t < tiles) {
    fetch(t * step);
    put(0);
  }
  __syncthreads();
  for (; t < tiles; t += strips, ++seen) {
    const bool more = t + strips < tiles;  // uniform
    if (more) fetch((t + strips) * step);
    const uint32_t here = ((uint32_t)(lane & 15) << 26) + seen * kTileRows + (lane >> 4) * 4;
#pragma unroll 1
    for (int r = 0; r < kRB; ++r) {
      const V start = *reinterpret_cast<const V*>(&terms[at][r * 16 + (lane >> 4) * 4]);
      uint4 a[CH];
#pragma unroll
      for (int c = 0; c < CH; ++c) a[c] = tile[at][(r * CH + c) * kWave + lane];
      V acc[kQB];
#pragma unroll
      for (int q = 0; q < kQB; ++q) acc[q] = mfma(a[0], b[q][0], start);
#pragma unroll
      for (int c = 1; c < CH; ++c)
#pragma unroll
        for (int q = 0; q < kQB; ++q) acc[q] = mfma(a[c], b[q][c], acc[q]);
      if constexpr (!COLLECT) {
#pragma unroll
        for (int q = 0; q < kQB; ++q)
#pragma unroll
          for (int i = 0; i < 4; ++i) best[q][i] = score_max(best[q][i], acc[q][i]);
      } else {
        bool hit = false;
#pragma unroll
        for (int q = 0; q < kQB; ++q)
          hit |= score_max(score_max(acc[q][0], acc[q][1]), score_max(acc[q][2], acc[q][3])) >=
                 limit[q];
        if (__ballot(hit) == 0ull) continue;
#pragma unroll
        for (int q = 0; q < kQB; ++q) {
          if (__ballot(score_max(score_max(acc[q][0], acc[q][1]),
                                 score_max(acc[q][2], acc[q][3])) >= limit[q]) == 0ull)
            continue;
          if (listed > (uint32_t)(kListed - 4 * kWave)) hand_on();
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const bool near = acc[q][i] >= limit[q];
            const uint64_t hits = __ballot(near);
            if (near)
              list[wave][listed + rank_in(hits)] =
                  here + ((uint32_t)q << 30) + (uint32_t)(r * 16 + i);
            listed += (uint32_t)__popcll(hits);
          }
        }
      }
    }
    if (more) put(at ^ 1);
    __syncthreads();
    at ^= 1;
  }
  if constexpr (COLLECT) {
    hand_on();
  } else {
    const int64_t per = (int64_t)strips * 16;
#pragma unroll
    for (int q = 0; q < kQB; ++q)
      *reinterpret_cast<V*>(bound + (int64_t)(q0 + 16 * q) * per + strip * 16 + (lane >> 4) * 4) =
          best[q];
  }
}

// One wavefront per query: the K-th best of its groups (without the query's own group).
// Queries that take no part - out of range, no node, behind the last one - get a bound that no
// row reaches.
// Where half of the groups may hold a candidate (their best row would reach the bound if it is as
// far off as the query's own row may be) the list would run over: the query is left to the general
// kernel without looking, and a group of 256 such queries costs no second scan.
template <typename T, typename V>
__global__ __launch_bounds__(256) void k_threshold(const T* __restrict__ best, int strips,
                                                   int step, const int32_t* __restrict__ queries,
                                                   const T* __restrict__ lower,
                                                   const T* __restrict__ upper,
                                                   const uint8_t* __restrict__ flags, int64_t nq,
                                                   int64_t padded, int K, T* bound,
                                                   uint32_t* found,
                                                   const SearchInfo* __restrict__ info) {
  const int64_t q = (int64_t)blockIdx.x * 4 + wave_id();
  if (q >= padded) return;
  const int lane = lane_id();
  const bool on = q < nq && flags[q] == 0;
  T result = score_never(T{});
  uint32_t given_up = 0u;
  constexpr bool kFloat = std::is_same<T, float>::value;
  if (kFloat && info->no_number) {  // (a query that is no node has no candidates: see k_pick)
    given_up = on ? (uint32_t)kCap + 1u : 0u;
  } else if (on) {
    const int groups = strips * 16;
    const uint32_t id = (uint32_t)queries[q], tile = id / kTileRows;
    const int own = tile % (uint32_t)step != 0u
                        ? -1
                        : (int)((tile / (uint32_t)step) % (uint32_t)strips) * 16 + (int)(id & 15u);
    // four groups of a strip count as one where there are plenty
    const T* const row = best + q * groups;
    const bool merged = groups >= 1024;
    uint32_t least = 0xffffffffu;  // codes ascend from the best score
    auto take = [&](uint32_t code, bool first) {
      if (!first && __ballot(code < __builtin_amdgcn_readlane(least, K - 1)) == 0ull) return;
      code = wave_sort(code, lane);
      least = first ? code : wave_merge_smallest(least, code, lane);
    };
    constexpr int kAtOnce = 4;  // reads in flight
    for (int g0 = 0; g0 < groups; g0 += kAtOnce * 4 * kWave) {
      V four[kAtOnce];
#pragma unroll
      for (int j = 0; j < kAtOnce; ++j) {
        const int g = g0 + (j * kWave + lane) * 4;  // (groups is a multiple of 16)
#pragma unroll
        for (int i = 0; i < 4; ++i) four[j][i] = score_least(T{});
        if (g < groups) four[j] = *reinterpret_cast<const V*>(row + g);
        if (own >= g && own < g + 4) {
          const uint32_t at = (uint32_t)(own - g);
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (at == (uint32_t)i) four[j][i] = score_least(T{});
        }
      }
#pragma unroll
      for (int j = 0; j < kAtOnce; ++j) {
        if (g0 + j * kWave * 4 >= groups) break;  // uniform
        if (merged) {
          take(score_code(score_max(score_max(four[j][0], four[j][1]),
                                    score_max(four[j][2], four[j][3]))),
               g0 + j == 0);
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) take(score_code(four[j][i]), g0 + j + i == 0);
        }
      }
    }
    result = code_score(__builtin_amdgcn_readlane(least, K - 1), T{});
    const T margin = upper[id] - lower[id];
    int near = 0;
    for (int g = lane; g < groups; g += kWave) near += row[g] >= result - margin ? 1 : 0;
    near += __shfl_xor(near, 1, kWave);
    near += __shfl_xor(near, 2, kWave);
    near += __shfl_xor(near, 4, kWave);
    near += __shfl_xor(near, 8, kWave);
    near += __shfl_xor(near, 16, kWave);
    near += __shfl_xor(near, 32, kWave);
    if (2 * near > groups && near > 4 * K) {
      result = score_never(T{});
      given_up = (uint32_t)kCap + 1u;
    }
  }
  if (lane == 0) {
    bound[q] = result;
    found[q * kFoundStep] = given_up;
  }
}

// Canonical distances of a query's candidates, best K in order.  flags: 2 = answered here with
// "none", 0 = answered here, 1 = left to the general kernel (more candidates than listed, or a
// distance that is no number).
template <int METRIC>
__global__ __launch_bounds__(256) void k_pick(const void* vec, int64_t n, int d,
                                              const int32_t* __restrict__ queries,
                                              uint8_t* flags, const uint32_t* __restrict__ found,
                                              const uint32_t* __restrict__ cand, int K,
                                              int32_t* ids_out, void* dist_out) {
  constexpr bool kBytes = METRIC == kL2U8;
  __shared__ uint32_t tile[4][kEvalTileWords];
  __shared__ uint64_t lists[4][kWave];
  const int64_t q = blockIdx.x;
  const int lane = lane_id(), wave = wave_id();
  const uint8_t flag = flags[q];
  const uint32_t count = found[q * kFoundStep];
  const uint32_t most = (uint32_t)vmin((int64_t)K, n - 1);
  if (flag == 1 || (flag == 0 && (count > (uint32_t)kCap || count < most))) {
    __syncthreads();
    if (threadIdx.x == 0) flags[q] = 1;
    return;
  }
  const uint32_t s = flag == 0 ? (uint32_t)queries[q] : 0u;
  VecSrc vs{vec, vec, n, d};
  uint64_t best = kKeyMax;
  bool nan = false;
  // (`count` is 0 for a query that is no node)
  for (uint32_t c = wave * kWave; c < count; c += 4 * kWave) {
    const bool on = c + lane < count;
    const uint32_t id = on ? cand[q * kCap + c + lane] : s;
    uint32_t code;
    if constexpr (METRIC == kCosineF32) {
      // the squared norms in dimension order, as the canonical distance has them
      const float* const row = vs.row<float>(id);
      const float* const own = vs.row<float>(s);
      float nb = 0.f, na = 0.f;
      for (int j = 0; j < d; ++j) {
        nb = __fmaf_rn(row[j], row[j], nb);
        na = __fmaf_rn(own[j], own[j], na);
      }
      code = cosine_code(wave_sums<kCosineF32>(vs, s, id, on, tile[wave], lane), na, nb);
    } else {
      code = wave_distances<METRIC>(vs, s, id, on, tile[wave], lane);
    }
    if constexpr (!kBytes) {
      const float dist = unord_f32(code);
      nan = nan || (on && dist != dist);
    }
    uint64_t key = on ? ((uint64_t)code << 32) | id : kKeyMax;
    key = wave_sort(key, lane);
    best = wave_merge_smallest(best, key, lane);
  }
  lists[wave][lane] = best;
  // (the order of NaN distances depends on their signs, which depend on the instructions used)
  if (__syncthreads_or(nan) != 0) {
    if (threadIdx.x == 0) flags[q] = 1;
    return;
  }
  if (wave != 0) return;
  for (int w = 1; w < 4 && (uint32_t)(w * kWave) < count; ++w)
    best = wave_merge_smallest(best, lists[w][lane], lane);
  if (lane < K) {
    const bool have = best != kKeyMax;
    const uint32_t code = (uint32_t)(best >> 32);
    ids_out[q * K + lane] = have ? (int32_t)(uint32_t)best : -1;
    if (kBytes)
      reinterpret_cast<int32_t*>(dist_out)[q * K + lane] = have ? unord_i32(code) : 0x7fffffff;
    else
      reinterpret_cast<float*>(dist_out)[q * K + lane] =
          have ? unord_f32(code) : __uint_as_float(0x7f800000u);
  }
}

int chunks_of(int32_t d, int32_t metric) { return metric == kL2U8 ? (d + 63) / 64 : (d + 31) / 32; }

// Strips of the first scan: about 512 workgroups, 16 groups of rows per strip.
int first_strips(int64_t tiles, int qgroups) {
  int64_t s = (512 / qgroups) & ~7;
  s = s < 8 ? 8 : s > 256 ? 256 : s;
  return (int)(s < tiles ? s : tiles);
}

struct SearchLayout {
  int64_t row_tiles, q_padded, slice_padded;
  size_t off_info, off_flags, off_rows, off_lower, off_upper, off_q, off_best, off_bound,
      off_found, off_cand, total;
};

SearchLayout search_layout(int64_t n, int32_t d, int32_t metric, int64_t nq) {
  SearchLayout L;
  size_t o = 0;
  auto take = [&](size_t bytes) {
    const size_t at = o;
    o = (o + bytes + 255) & ~(size_t)255;
    return at;
  };
  const size_t row_bytes = (size_t)chunks_of(d, metric) * 64;
  L.row_tiles = (n + kTileRows - 1) / kTileRows;
  L.q_padded = (nq + kGroupQueries - 1) / kGroupQueries * kGroupQueries;
  L.slice_padded = L.q_padded < kSlice ? L.q_padded : kSlice;
  L.off_flags = take((size_t)nq);  // (first, so that a test finds them: 1 = left to k_exact_knn)
  L.off_info = take(sizeof(SearchInfo));
  L.off_rows = take((size_t)L.row_tiles * kTileRows * row_bytes);
  L.off_lower = take((size_t)L.row_tiles * kTileRows * 4);
  L.off_upper = take((size_t)L.row_tiles * kTileRows * 4);
  L.off_q = take((size_t)L.q_padded * row_bytes);
  // (the last slice may have fewer query groups and then more strips: 512 workgroups at most)
  L.off_best = take((size_t)kGroupQueries * 16 * 512 * 4);
  L.off_bound = take((size_t)L.slice_padded * 4);
  L.off_found = take((size_t)L.slice_padded * 4 * kFoundStep);
  L.off_cand = take((size_t)L.slice_padded * kCap * 4);
  L.total = o;
  return L;
}

template <int METRIC, int CH>
hipError_t search(const void* vec, int64_t n, int32_t d, const int32_t* queries, int64_t nq,
                  int32_t K, int32_t* ids_out, void* dist_out, char* ws, const SearchLayout& L,
                  hipStream_t st) {
  using T = typename ScoreOf<METRIC>::type;
  auto* const info = reinterpret_cast<SearchInfo*>(ws + L.off_info);
  auto* const flags = reinterpret_cast<uint8_t*>(ws + L.off_flags);
  auto* const rows = reinterpret_cast<uint4*>(ws + L.off_rows);
  auto* const lower = reinterpret_cast<T*>(ws + L.off_lower);
  auto* const upper = reinterpret_cast<T*>(ws + L.off_upper);
  auto* const qfrag = reinterpret_cast<uint4*>(ws + L.off_q);
  auto* const best = reinterpret_cast<T*>(ws + L.off_best);
  auto* const bound = reinterpret_cast<T*>(ws + L.off_bound);
  auto* const found = reinterpret_cast<uint32_t*>(ws + L.off_found);
  auto* const cand = reinterpret_cast<uint32_t*>(ws + L.off_cand);
  if (METRIC != kL2U8)
    k_query_norms<<<kNormParts, 256, 0, st>>>(static_cast<const float*>(vec), n, d, queries, nq,
                                              info, flags);
  const int64_t q_blocks = L.q_padded / 16, r_blocks = L.row_tiles * kRB;
  k_pack<METRIC, CH, true><<<(unsigned)((q_blocks + 3) / 4), 256, 0, st>>>(
      vec, n, d, queries, nq, q_blocks, qfrag, lower, upper, info, flags);
  k_pack<METRIC, CH, false><<<(unsigned)((r_blocks + 3) / 4), 256, 0, st>>>(
      vec, n, d, queries, n, r_blocks, rows, lower, upper, info, flags);
  // few rows: all of them find the thresholds
  const int step = L.row_tiles >= 64 * kEvery ? kEvery : 1;
  const int64_t tiles = (L.row_tiles + step - 1) / step;
  for (int64_t s0 = 0; s0 < nq; s0 += kSlice) {
    const int64_t here = nq - s0 < kSlice ? nq - s0 : kSlice;
    const int groups = (int)((here + kGroupQueries - 1) / kGroupQueries);
    const int64_t padded = (int64_t)groups * kGroupQueries;
    const uint4* const qf = qfrag + s0 / 16 * CH * kWave;
    const int few = first_strips(tiles, groups);
    k_scan<METRIC, CH, false><<<(unsigned)((few + 7) / 8 * 8 * groups), 256, 0, st>>>(
        rows, lower, tiles, step, few, groups, n, qf, queries + s0, best, found, cand, info);
    k_threshold<T, typename ScoreOf<METRIC>::vec><<<(unsigned)((padded + 3) / 4), 256, 0, st>>>(
        best, few, step, queries + s0, lower, upper, flags + s0, here, padded, K, bound, found,
        info);
    int64_t strips = 1024 / groups & ~7;
    strips = strips < 8 ? 8 : strips;
    strips = strips < L.row_tiles ? strips : L.row_tiles;
    k_scan<METRIC, CH, true><<<(unsigned)((strips + 7) / 8 * 8 * groups), 256, 0, st>>>(
        rows, upper, L.row_tiles, 1, (int)strips, groups, n, qf, queries + s0, bound, found,
        cand, info);
    k_pick<METRIC><<<(unsigned)here, 256, 0, st>>>(
        vec, n, d, queries + s0, flags + s0, found, cand, K, ids_out + s0 * K,
        static_cast<char*>(dist_out) + s0 * K * 4);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_exact_knn(vec, n, d, METRIC, queries, nq, K, ids_out, dist_out, st, flags);
}

template <int METRIC>
hipError_t search_metric(const void* vec, int64_t n, int32_t d, const int32_t* queries, int64_t nq,
                         int32_t K, int32_t* ids_out, void* dist_out, char* ws,
                         const SearchLayout& L, hipStream_t st) {
  switch (chunks_of(d, METRIC)) {
    case 1: return search<METRIC, 1>(vec, n, d, queries, nq, K, ids_out, dist_out, ws, L, st);
    case 2: return search<METRIC, 2>(vec, n, d, queries, nq, K, ids_out, dist_out, ws, L, st);
    case 3:
      if constexpr (METRIC != kL2U8)
        return search<METRIC, 3>(vec, n, d, queries, nq, K, ids_out, dist_out, ws, L, st);
      [[fallthrough]];
    default:
      if constexpr (METRIC != kL2U8)
        return search<METRIC, 4>(vec, n, d, queries, nq, K, ids_out, dist_out, ws, L, st);
      return hipErrorInvalidValue;
  }
}

}  // namespace

// The line between the two forms: this one takes 35 to 60 us for its eight launches (bytes: seven;
// four more per further 4096 queries) however small the call, k_exact_knn 7 to 11 us times `work`
// here: rows, dimensions and rounds of workgroups count, and K, whose best it keeps per
// query and wavefront (bytes: rows of a multiple of 16 bytes are read four dimensions at a time).
// A pass among others in microseconds, this form / k_exact_knn, `work` in parentheses: 10,325 x 20,
// 1000 queries, squared L2: K = 1 42 / 31 (2.7), K = 10 43 / 44 (4.1), K = 64 48 / 85 (12.8); 6000 x
// 96, 1000 queries, bytes: K = 1 38 / 27 (1.8), K = 10 38 / 37 (3.2), K = 64 43 / 66 (11.9); 24,577 x
// 96, 16 queries 41 / 150 (13).  Of 1200 calls just above the second line - n from one to 3.5 times
// it, 4 to 128 dimensions, 16 to 4096 queries, K from 1 to 64, three metrics - none is slower in this
// form than in the other by 2 % or more; 9 are left to the other though it takes 2 % more or worse, the
// three worst of them, of 5 to 10 dimensions, 1.9 to 2.9 times as long.
size_t exact_scan_bytes(int64_t n, int32_t d, int32_t metric, int64_t nq, int32_t K) {
  if (metric == kChi2F32 || d > 128 || n < 6000 || n > ((int64_t)1 << 27) || nq < 1 ||
      nq > ((int64_t)1 << 27))
    return 0;
  if (n * (nq < 256 ? 256 : nq) < ((int64_t)1 << 29) / (d + 32)) return 0;
  const int c = exact_queries(nq);
  const int64_t words = metric != kL2U8 ? d : d % 16 == 0 ? d / 4 : d + 32;
  const double work =
      (double)exact_rounds(nq, c) * ((double)((c + 4) * n * (words + 12)) / (1 << 20) + 0.04 * c * K);
  if (work < 4.5) return 0;
  return search_layout(n, d, metric, nq).total;
}

hipError_t launch_exact_scan(const void* vec, int64_t n, int32_t d, int32_t metric,
                             const int32_t* queries, int64_t nq, int32_t K, int32_t* ids_out,
                             void* dist_out, void* workspace, hipStream_t st) {
  const SearchLayout L = search_layout(n, d, metric, nq);
  char* const ws = static_cast<char*>(workspace);
  switch (metric) {
    case kL2F32: return search_metric<kL2F32>(vec, n, d, queries, nq, K, ids_out, dist_out, ws, L, st);
    case kAngularF32:
      return search_metric<kAngularF32>(vec, n, d, queries, nq, K, ids_out, dist_out, ws, L, st);
    case kCosineF32:
      return search_metric<kCosineF32>(vec, n, d, queries, nq, K, ids_out, dist_out, ws, L, st);
    case kL2U8: return search_metric<kL2U8>(vec, n, d, queries, nq, K, ids_out, dist_out, ws, L, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace gnnd

// Device-side building blocks shared by the GNND kernels: the counter-based
// hash, the order-preserving distance encoding, packed list entries and the
// 64-lane sorting / merging networks that act on one value per lane.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace gnnd {

constexpr int kWave = 64;
constexpr uint64_t kKeyMax = ~0ull;
constexpr uint32_t kIdMax = 0x7fffffffu;

enum : int { kL2F32 = 0, kAngularF32 = 1, kL2U8 = 2, kChi2F32 = 3, kCosineF32 = 4 };
enum : uint32_t { kTagInit = 1, kTagRevNew = 2, kTagRevOld = 3, kTagMerge = 4 };
constexpr uint32_t kHashAttempts = 256;

// ---- counter-based random numbers ---------------------------------------
// hash(seed, tag, a, b, c): three rounds of the splitmix64 output mixer over
// (seed, tag), the packed pair (a, b), and c.  Any thread can draw any number.
__host__ __device__ inline uint64_t mix64(uint64_t z) {
  z ^= z >> 30;
  z *= 0xbf58476d1ce4e5b9ull;
  z ^= z >> 27;
  z *= 0x94d049bb133111ebull;
  z ^= z >> 31;
  return z;
}
// The (seed, tag) round depends on nothing per thread: computed once on the host.
__host__ __device__ inline uint64_t hash_base(uint64_t seed, uint32_t tag) {
  return mix64(seed + 0x9e3779b97f4a7c15ull * ((uint64_t)tag + 1));
}
__device__ inline uint64_t hash3(uint64_t base, uint32_t a, uint32_t b, uint32_t c) {
  uint64_t h = mix64(base ^ (((uint64_t)a << 32) | (uint64_t)b));
  return mix64(h + (uint64_t)c);
}
// upper 32 hash bits mapped onto [0, n) by multiply-high
__device__ inline uint32_t bounded(uint64_t h, uint32_t n) {
  return __umulhi((uint32_t)(h >> 32), n);
}

// ---- distances as order-preserving 32-bit codes -------------------------
// A float (possibly negative: 1 - dot can round below zero) or an int32 maps to
// an unsigned code with the same order, so (code << 32 | id) compares like
// (distance, id).
__device__ inline uint32_t ord_f32(float x) {
  uint32_t b = __float_as_uint(x);
  return b ^ ((b >> 31) ? 0xffffffffu : 0x80000000u);
}
__device__ inline float unord_f32(uint32_t o) {
  return __uint_as_float((o & 0x80000000u) ? (o ^ 0x80000000u) : ~o);
}
__device__ inline uint32_t ord_i32(int32_t x) { return (uint32_t)x ^ 0x80000000u; }
__device__ inline int32_t unord_i32(uint32_t o) { return (int32_t)(o ^ 0x80000000u); }

// ---- packed list entry ---------------------------------------------------
// 64 bits: [63:32] distance code, [31:2] neighbour id, bit 1 "admitted by the
// update in progress", bit 0 NEW flag.  Unsigned comparison of two entries
// with different ids orders them by (distance, id).
__device__ inline uint64_t make_entry(uint32_t code, uint32_t id, uint32_t flags) {
  return ((uint64_t)code << 32) | ((uint64_t)id << 2) | flags;
}
__device__ inline uint32_t entry_id(uint64_t e) { return ((uint32_t)e) >> 2; }
__device__ inline uint32_t entry_code(uint64_t e) { return (uint32_t)(e >> 32); }
__device__ inline uint64_t entry_key(uint64_t e) { return e >> 2; }  // (distance, id) only

// ---- wavefront helpers (one value per lane, 64 lanes) --------------------
__device__ inline int lane_id() { return (int)(threadIdx.x & (kWave - 1)); }
// Number of this wavefront inside its workgroup, as a scalar: every lane holds the same
// value, and saying so keeps what is derived from it (row numbers, base addresses) in
// scalar registers.
__device__ inline int wave_id() {
  return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
}
__device__ inline uint64_t lanes_below(int lane) { return (1ull << lane) - 1ull; }

// A launch may not span 2^32 threads in one grid dimension (16 M workgroups of
// 256); launches over more workgroups fold them into two dimensions, and the
// kernels number their workgroups with this.  Workgroups past the end of the
// work (the last row of the fold) must leave on their own index checks.
__device__ inline int64_t block_linear() {
  return (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
}

__device__ inline uint64_t readlane64(uint64_t x, int l) {
  uint32_t lo = __builtin_amdgcn_readlane((uint32_t)x, l);
  uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(x >> 32), l);
  return ((uint64_t)hi << 32) | lo;
}

template <typename T>
__device__ inline T vmin(T a, T b) { return a < b ? a : b; }
template <typename T>
__device__ inline T vmax(T a, T b) { return a < b ? b : a; }

// Value of lane (lane ^ j), j a power of two, without going through LDS: data
// parallel primitives inside a row of 16 lanes (quad permutes, row shifts under
// bank masks, row rotate) and the row / half swaps across rows.  `j` must be a
// compile-time constant after unrolling.
__device__ inline uint32_t xor_lanes(uint32_t v, int j, int lane) {
  switch (j) {
    case 1: return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true);  // quad_perm:[1,0,3,2]
    case 2: return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true);  // quad_perm:[2,3,0,1]
    case 4: {
      // mirrored inside 8 lanes (lane ^ 7), then inside quads (lane ^ 3)
      const int r = __builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, true);
      return (uint32_t)__builtin_amdgcn_mov_dpp(r, 0x1B, 0xF, 0xF, true);
    }
    case 8: return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xF, 0xF, true);  // row_ror:8
    case 16: {
      // rows 1 and 3 of the first copy change places with rows 0 and 2 of the second
      auto sw = __builtin_amdgcn_permlane16_swap(v, v, false, false);
      return (lane & 16) ? sw[0] : sw[1];
    }
    default: {
      // the upper half of the first copy changes places with the lower half of the second
      auto sw = __builtin_amdgcn_permlane32_swap(v, v, false, false);
      return (lane & 32) ? sw[0] : sw[1];
    }
  }
}
__device__ inline uint64_t xor_lanes(uint64_t v, int j, int lane) {
  const uint32_t lo = xor_lanes((uint32_t)v, j, lane);
  const uint32_t hi = xor_lanes((uint32_t)(v >> 32), j, lane);
  return ((uint64_t)hi << 32) | lo;
}

// Value of lane 63 - lane: mirror inside the row, then swap rows and halves.
__device__ inline uint32_t reverse_lanes(uint32_t v, int lane) {
  const uint32_t m = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x140, 0xF, 0xF, true);  // row_mirror
  return xor_lanes(xor_lanes(m, 16, lane), 32, lane);
}
__device__ inline uint64_t reverse_lanes(uint64_t v, int lane) {
  const uint32_t lo = reverse_lanes((uint32_t)v, lane);
  const uint32_t hi = reverse_lanes((uint32_t)(v >> 32), lane);
  return ((uint64_t)hi << 32) | lo;
}

// Values of the lanes without and with bit j (16 or 32) of this lane's pair, in both of its lanes.
__device__ inline void pair_lanes(uint32_t v, int j, uint32_t& lower, uint32_t& upper) {
  if (j == 16) {
    auto sw = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    lower = sw[0];
    upper = sw[1];
  } else {
    auto sw = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    lower = sw[0];
    upper = sw[1];
  }
}

// One compare-exchange of a sorting network between lanes `lane` and lane ^ j: this lane keeps
// the smaller of its value and its partner's when keep_min, else the larger.  (Equal values:
// either.)  One comparison; the lane pattern keep_min folds into the mask.  Across rows and halves
// both values are at hand in both lanes, so nothing has to be picked before the comparison.
__device__ inline uint64_t exchange_step(uint64_t v, int j, int lane, bool keep_min) {
  if (j >= 16) {
    uint32_t lo0, lo1, hi0, hi1;
    pair_lanes((uint32_t)v, j, lo0, lo1);
    pair_lanes((uint32_t)(v >> 32), j, hi0, hi1);
    const uint64_t a = ((uint64_t)hi0 << 32) | lo0, b = ((uint64_t)hi1 << 32) | lo1;
    return ((b < a) == keep_min) ? b : a;
  }
  const uint64_t o = xor_lanes(v, j, lane);
  return ((o < v) == keep_min) ? o : v;
}

// 32-bit values: the median of both values and 0 is the smaller, of both and 2^32 - 1 the larger
// one, so a limit per lane (lane_limit) makes an exchange one instruction.
__device__ inline uint32_t median(uint32_t a, uint32_t b, uint32_t c) {
  return vmax(vmin(a, b), vmin(vmax(a, b), c));
}
// all ones in the lanes with bit j, 0 in the others (kept opaque: the median is to stay one)
__device__ inline uint32_t lane_limit(int lane, int j) {
  uint32_t m = (lane & j) ? 0xffffffffu : 0u;
  asm("" : "+v"(m));
  return m;
}
// lanes without bit j keep the smaller, lanes with it the larger value
__device__ inline uint32_t exchange_step(uint32_t v, int j, int lane) {
  if (j >= 16) {
    uint32_t a, b;
    pair_lanes(v, j, a, b);
    return median(a, b, lane_limit(lane, j));
  }
  return median(v, xor_lanes(v, j, lane), lane_limit(lane, j));
}

// Ascending sort when only the first `N` lanes hold real values and all other lanes hold the
// maximum: the bitonic network over N lanes (short lists are the common case), every group of N
// lanes for itself.
// 32-bit values are complemented in the groups that a phase sorts downwards, so that all groups
// of all phases sort upwards.
template <int N>
__device__ inline uint64_t wave_sort_first(uint64_t v, int lane) {
#pragma unroll
  for (int k = 2; k <= N; k <<= 1) {
#pragma unroll
    for (int j = k >> 1; j > 0; j >>= 1)
      v = exchange_step(v, j, lane, ((lane & j) == 0) == ((lane & k) == 0));
  }
  return v;
}
template <int N>
__device__ inline uint32_t wave_sort_first(uint32_t v, int lane) {
#pragma unroll
  for (int k = 2; k <= N; k <<= 1) {
    if (k < N) v ^= lane_limit(lane, k);
#pragma unroll
    for (int j = k >> 1; j > 0; j >>= 1) v = exchange_step(v, j, lane);
    if (k < N) v ^= lane_limit(lane, k);
  }
  return v;
}
// Full ascending sort of 64 lane values (21 exchange stages).
template <typename T>
__device__ inline T wave_sort(T v, int lane) { return wave_sort_first<kWave>(v, lane); }

// Ascending sort of the first `count` lanes' values, the maximum in all others.
template <typename T>
__device__ inline T wave_sort_upto(T v, int lane, int count) {
  if (count <= 1) return v;
  if (count <= 2) return wave_sort_first<2>(v, lane);
  if (count <= 4) return wave_sort_first<4>(v, lane);
  if (count <= 8) return wave_sort_first<8>(v, lane);
  if (count <= 16) return wave_sort_first<16>(v, lane);
  if (count <= 32) return wave_sort_first<32>(v, lane);
  return wave_sort(v, lane);
}

// Lanes hold a bitonic sequence (ascending then descending, or an element-wise
// min of an ascending and a reversed ascending one): 6 stages sort it ascending.
__device__ inline uint64_t wave_bitonic_merge(uint64_t v, int lane) {
#pragma unroll
  for (int j = kWave >> 1; j > 0; j >>= 1) v = exchange_step(v, j, lane, (lane & j) == 0);
  return v;
}
__device__ inline uint32_t wave_bitonic_merge(uint32_t v, int lane) {
#pragma unroll
  for (int j = kWave >> 1; j > 0; j >>= 1) v = exchange_step(v, j, lane);
  return v;
}

// The 64 smallest of two ascending 64-lane sequences, ascending.
template <typename T>
__device__ inline T wave_merge_smallest(T a_sorted, T b_sorted, int lane) {
  const T br = reverse_lanes(b_sorted, lane);
  return wave_bitonic_merge(vmin(a_sorted, br), lane);
}

// 128 values, two per lane (value i in lane i % 64 of register i / 64), ascending over
// (lo, hi): two 64-lane networks and a 128-wide bitonic merge.
template <typename T>
__device__ inline void sort128(T& lo, T& hi, int lane) {
  lo = wave_sort(lo, lane);
  hi = wave_sort(hi, lane);
  const T t = reverse_lanes(hi, lane);  // lo ++ t is bitonic
  const T a = vmin(lo, t), b = vmax(lo, t);
  lo = wave_bitonic_merge(a, lane);
  hi = wave_bitonic_merge(b, lane);
}

// (lo, hi) ascending, c ascending (64 values): afterwards (lo, hi) holds the 128
// smallest of the 192, ascending (c is split against lo; the larger half goes on to hi).
template <typename T>
__device__ inline void merge128(T& lo, T& hi, T c, int lane) {
  const T t = reverse_lanes(c, lane);
  const T a = vmin(lo, t), b = vmax(lo, t);
  lo = wave_bitonic_merge(a, lane);
  const T spill = wave_bitonic_merge(b, lane);  // the 64 largest of lo and c, ascending
  hi = wave_merge_smallest(hi, spill, lane);
}

// Value of the lane before this one; lane 0: `first`.
__device__ inline uint32_t lane_before(uint32_t v, uint32_t first) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)first, (int)v, 0x138, 0xF, 0xF, false);  // wave_shr:1
}
__device__ inline uint64_t lane_before(uint64_t v, uint64_t first) {
  const uint32_t lo = lane_before((uint32_t)v, (uint32_t)first);
  const uint32_t hi = lane_before((uint32_t)(v >> 32), (uint32_t)(first >> 32));
  return ((uint64_t)hi << 32) | lo;
}
// Bits of `mask` below this lane's.
__device__ inline int rank_in(uint64_t mask) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                        __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Of up to 64 R candidates (lane's candidate r exists where bit `lane` of have[r] is set), `room`
// < their number are to be chosen: those with the smallest hashes h[r].  A value t is searched that
// exactly `room` of them do not exceed - each try costs one comparison, the rest is scalar work -
// and win[r] is where those are.  The hashes are evenly spread, so the tries follow the number
// that is missing for a while, and halve the range then: four or five tries as a rule, where a
// sorting network of (hash, id) pairs took 15 to 21 stages of six vector instructions.  False
// where equal hashes leave no such t.
template <int R>
__device__ inline bool choose_smallest(const uint32_t (&h)[R], const uint64_t (&have)[R], int count,
                                       int room, uint64_t (&win)[R]) {
  const uint32_t step = (uint32_t)__builtin_amdgcn_readfirstlane(
      (int)(uint32_t)(4294967040.f * __builtin_amdgcn_rcpf((float)count)));
  uint32_t lo = 0u, hi = 0xffffffffu, t = step * (uint32_t)room;
  for (int tries = 0;; ++tries) {
    int c = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      win[r] = __ballot(h[r] <= t) & have[r];
      c += __popcll(win[r]);
    }
    if (c == room) return true;
    if (c < room) lo = t + 1u;  // (t < hi)
    else hi = t;
    if (lo >= hi) return false;
    t = lo + ((hi - lo) >> 1);
    if (tries < 4) {
      const uint32_t jump = step * (uint32_t)(c < room ? room - c : c - room);
      if (jump < hi - lo) t = c < room ? lo + jump : hi - jump;
    }
  }
}

// Stable compaction of the lanes with keep == true to the front; the other
// lanes end up behind them holding `fill`.
__device__ inline uint64_t wave_compact(uint64_t v, bool keep, uint64_t fill, int lane) {
  const uint64_t mask = __ballot(keep);
  const int before = rank_in(mask);
  const int dst = keep ? before : __popcll(mask) + (lane - before);
  uint64_t x = keep ? v : fill;
  uint32_t lo = __builtin_amdgcn_ds_permute(dst << 2, (int)(uint32_t)x);
  uint32_t hi = __builtin_amdgcn_ds_permute(dst << 2, (int)(uint32_t)(x >> 32));
  return ((uint64_t)hi << 32) | lo;
}

// What a wavefront's lanes have written to LDS before this is read by the others after it.
__device__ inline void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Whether the N entries at `row` in LDS (ascending, unused ones the maximum, N a power of two)
// hold the (distance, id) of e.  The updates are bound by vector-instruction issue: a step of the
// search is one read, one comparison and one addition, where a row kept in registers took two
// lane permutations and the key shifted out of every entry.  An entry below the key with its flags
// cleared has a smaller key, whatever its own flags are.
template <int N>
__device__ inline bool list_holds(const uint64_t* row, uint64_t e) {
  const uint64_t key = e & ~3ull;
  const uint64_t* at = row;
#pragma unroll
  for (int step = N / 2; step > 0; step >>= 1) at = at[step - 1] < key ? at + step : at;
  return ((*at ^ e) >> 2) == 0ull;
}

// Drop from `pk` (one candidate per lane, kKeyMax = none) what cannot enter the
// ascending list `row` of k entries: not closer than its last entry, already
// in it, or a repeat of another candidate.  Returns the survivors ascending.  `lds`: 64 words of
// the wavefront's own.
__device__ inline uint64_t filter_candidates(uint64_t pk, uint64_t row, int k, int lane,
                                             uint64_t* lds, bool& any) {
  if (pk >= (readlane64(row, k - 1) & ~3ull)) pk = kKeyMax;
  any = __ballot(pk != kKeyMax) != 0ull;
  if (!any) return pk;
  lds[lane] = row;
  wave_lds_fence();
  if (list_holds<kWave>(lds, pk)) pk = kKeyMax;
  wave_lds_fence();  // (the next row may be written)
  const uint64_t left = __ballot(pk != kKeyMax);
  any = left != 0ull;
  if (!any) return pk;
  // survivors to the front, then a sorting network just wide enough for them
  pk = wave_compact(pk, pk != kKeyMax, kKeyMax, lane);
  pk = wave_sort_upto(pk, lane, __popcll(left));
  const uint64_t prev = lane_before(pk, kKeyMax);
  const bool rep = pk != kKeyMax && entry_key(pk) == entry_key(prev);
  if (__ballot(rep) != 0ull) pk = wave_compact(pk, !rep, kKeyMax, lane);
  return pk;
}

// ---- canonical distances --------------------------------------------------
// Float metrics accumulate one fused multiply-add per dimension, in dimension
// order, in float32; bytes accumulate exact int32 squares.  The result is the
// order-preserving code of the distance.  JoinTraits (below) states one step and the code.
// Chi-square distance of non-negative vectors: sum of (a - b)^2 / (a + b) over
// the dimensions with a + b > 0; every operation rounded on its own (there is no
// multiply feeding an add, so nothing can fuse), correctly rounded division.
__device__ inline float chi2_term(float a, float b, float acc) {
  const float diff = __fsub_rn(a, b), sum = __fadd_rn(a, b);
  return sum > 0.f ? __fadd_rn(acc, __fdiv_rn(__fmul_rn(diff, diff), sum)) : acc;
}

// Cosine distance of vectors of any length: 1 - a.b / sqrt(|a|^2 |b|^2); a zero
// vector is at distance 1 from everything.  The inner product and the squared
// norms are accumulated like the angular inner product (a squared norm belongs
// to its vector alone, so it can be computed once and kept); product, root,
// quotient and difference are each rounded on their own.
__device__ inline uint32_t cosine_code(float dot, float na, float nb) {
  // sqrtf is the correctly rounded root (the compiler's default for HIP); the
  // intrinsic named after round-to-nearest maps to the approximate instruction
  const float den = sqrtf(__fmul_rn(na, nb));
  return ord_f32(den > 0.f ? __fsub_rn(1.0f, __fdiv_rn(dot, den)) : 1.0f);
}

// Vectors may live in two arrays (the two sets of a merge): rows below `split`
// come from the first, the others from the second.
struct VecSrc {
  const void* a;
  const void* b;
  int64_t split;
  int32_t d;
  const float* norms = nullptr;  // squared norm per id where the metric needs it (cosine)
  template <typename T>
  __device__ const T* row(uint32_t id) const {
    return ((int64_t)id < split) ? reinterpret_cast<const T*>(a) + (int64_t)id * d
                                 : reinterpret_cast<const T*>(b) + ((int64_t)id - split) * d;
  }
};

// The canonical arithmetic one step at a time (one dimension of one pair), for kernels that
// walk many pairs through staged chunks of dimensions.
template <int METRIC>
struct JoinTraits;
template <>
struct JoinTraits<kL2F32> {
  using elem = float;
  using acc = float;
  __device__ static void step(float a, float b, float& s) {
    float t = a - b;
    s = __fmaf_rn(t, t, s);
  }
  __device__ static uint32_t code(float s) { return ord_f32(s); }
  __device__ static uint32_t code(float s, float, float) { return code(s); }
};
template <>
struct JoinTraits<kAngularF32> {
  using elem = float;
  using acc = float;
  __device__ static void step(float a, float b, float& s) { s = __fmaf_rn(a, b, s); }
  __device__ static uint32_t code(float s) { return ord_f32(1.0f - s); }
  __device__ static uint32_t code(float s, float, float) { return code(s); }
};
// cosine: the running sum is the inner product; the squared norms of the two
// vectors come from the per-id array (VecSrc::norms)
template <>
struct JoinTraits<kCosineF32> {
  using elem = float;
  using acc = float;
  __device__ static void step(float a, float b, float& s) { s = __fmaf_rn(a, b, s); }
  __device__ static uint32_t code(float s, float na, float nb) { return cosine_code(s, na, nb); }
};
template <>
struct JoinTraits<kChi2F32> {
  using elem = float;
  using acc = float;
  __device__ static void step(float a, float b, float& s) { s = chi2_term(a, b, s); }
  __device__ static uint32_t code(float s) { return ord_f32(s); }
  __device__ static uint32_t code(float s, float, float) { return code(s); }
};
template <>
struct JoinTraits<kL2U8> {
  using elem = uint8_t;
  using acc = int32_t;
  __device__ static void step(int32_t a, int32_t b, int32_t& s) {
    int32_t t = a - b;
    s += __mul24(t, t);
  }
  __device__ static uint32_t code(int32_t s) { return ord_i32(s); }
  __device__ static uint32_t code(int32_t s, float, float) { return code(s); }
};

// Canonical distances from object s to one object per lane (`id`, meaningful
// where `on`).  The 64 rows and the row of s are staged through the wave's LDS
// tile in chunks of kEvalChunk dimensions with coalesced reads (8 lanes per row
// chunk), then every lane accumulates its own pair in dimension order: the
// canonical arithmetic, without 64 lanes each walking a row of its own through HBM.  All 64 lanes must call it together.
// wave_sums gives the running sums, wave_distances the codes of the distances.
constexpr int kEvalChunk = 32;
constexpr int kEvalStride = kEvalChunk + 1;  // odd stride: lanes walk their rows free of bank conflicts
constexpr int kEvalTileWords = 65 * kEvalStride;

template <int METRIC>
__device__ inline typename JoinTraits<METRIC>::acc wave_sums(const VecSrc& vs, uint32_t s,
                                                             uint32_t id, bool on,
                                                             uint32_t* tile_raw, int lane) {
  using TR = JoinTraits<METRIC>;
  using T = typename TR::elem;
  using ACC = typename TR::acc;
  ACC* tile = reinterpret_cast<ACC*>(tile_raw);
  const int d = vs.d;
  const bool aligned = (d & 3) == 0;
  const int part = lane & 7, rsel = lane >> 3;
  // the rows this lane helps to read: rows 0..63 are the lanes' objects, row 64 is s
  constexpr int kRounds = 9;
  const T* src[kRounds];
#pragma unroll
  for (int i = 0; i < kRounds; ++i) {
    const int r = 8 * i + rsel;
    const uint32_t rid = __shfl(id, r & 63, kWave);
    const int ron = __shfl((int)on, r & 63, kWave);
    const bool want = r < 64 ? ron != 0 : r == 64;
    src[i] = want ? vs.row<T>(r < 64 ? rid : s) + part * 4 : nullptr;
  }
  // The next chunk is requested before this one is evaluated (four floats of a row, or its four
  // bytes, per lane and round): with one chunk at a time the kernels waited for memory.  Random
  // initial graphs, 1.5 million x 96 angular 5.3 -> 3.6 ms, 150,000 x 960 4.4 -> 2.8 ms (6.6 TB/s,
  // the rate of a gather of random rows).
  using Raw = typename std::conditional<sizeof(T) == 4, float4, uint32_t>::type;
  Raw raw[kRounds];
  auto fetch = [&](int d0) {
    const int j = d0 + part * 4;
#pragma unroll
    for (int i = 0; i < kRounds; ++i) {
      raw[i] = Raw{};
      if (src[i] == nullptr) continue;
      const T* at = src[i] + d0;
      if (aligned && j + 3 < d) {
        raw[i] = *reinterpret_cast<const Raw*>(at);
      } else if constexpr (sizeof(T) == 4) {
        if (j + 0 < d) raw[i].x = at[0];
        if (j + 1 < d) raw[i].y = at[1];
        if (j + 2 < d) raw[i].z = at[2];
        if (j + 3 < d) raw[i].w = at[3];
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (j + q < d) raw[i] |= (uint32_t)at[q] << (8 * q);
      }
    }
  };
  ACC acc = 0;
  fetch(0);
  for (int d0 = 0; d0 < d; d0 += kEvalChunk) {
#pragma unroll
    for (int i = 0; i < kRounds; ++i) {
      const int r = 8 * i + rsel;
      if (r <= 64) {
        ACC* const to = tile + r * kEvalStride + part * 4;
        if constexpr (sizeof(T) == 4) {
          to[0] = raw[i].x; to[1] = raw[i].y; to[2] = raw[i].z; to[3] = raw[i].w;
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q) to[q] = (ACC)((raw[i] >> (8 * q)) & 0xff);
        }
      }
    }
    if (d0 + kEvalChunk < d) fetch(d0 + kEvalChunk);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int width = d - d0 < kEvalChunk ? d - d0 : kEvalChunk;
    if (on)
      for (int j = 0; j < width; ++j)
        TR::step(tile[64 * kEvalStride + j], tile[lane * kEvalStride + j], acc);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  return acc;
}
template <int METRIC>
__device__ inline uint32_t wave_distances(const VecSrc& vs, uint32_t s, uint32_t id, bool on,
                                          uint32_t* tile_raw, int lane) {
  const auto acc = wave_sums<METRIC>(vs, s, id, on, tile_raw, lane);
  if constexpr (METRIC == kCosineF32)
    return JoinTraits<METRIC>::code(acc, vs.norms[s], on ? vs.norms[id] : 0.f);
  else return JoinTraits<METRIC>::code(acc);
}

// The nodes with work to do, listed by class: list c at nodes + c n, its length in count[c]
// (cleared by the sampling stage); the order inside a list is of no consequence.  A workgroup
// of 256 takes 256 PER consecutive nodes, numbers those of each class in LDS - one addition
// per wavefront and class that occurs in it - and reserves their places with one device-wide
// addition per class.  class_of(s): the class of node s, or -1.
template <int CLASSES, int PER, typename F>
__device__ inline void list_nodes_by_class(int64_t n, int32_t* nodes, uint32_t* count,
                                           F class_of) {
  __shared__ uint32_t here[CLASSES], base[CLASSES];
  const int64_t first = block_linear() * (256 * PER);
  const int lane = lane_id();
  if (threadIdx.x < CLASSES) here[threadIdx.x] = 0u;
  int cls[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int64_t s = first + j * 256 + threadIdx.x;
    cls[j] = s < n ? class_of(s) : -1;
  }
  __syncthreads();
  uint32_t number[PER];  // within the workgroup
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    number[j] = 0u;
    uint64_t left = __ballot(cls[j] >= 0);
    while (left != 0ull) {
      const int l = __ffsll((unsigned long long)left) - 1;
      const int c = __builtin_amdgcn_readlane(cls[j], l);
      const uint64_t same = __ballot(cls[j] == c);
      uint32_t at = 0u;
      if (lane == l) at = atomicAdd(&here[c], (uint32_t)__popcll(same));
      at = __builtin_amdgcn_readlane(at, l);
      if (cls[j] == c) number[j] = at + (uint32_t)__popcll(same & lanes_below(lane));
      left &= ~same;
    }
  }
  __syncthreads();
  if (threadIdx.x < CLASSES && here[threadIdx.x] != 0u)
    base[threadIdx.x] = atomicAdd(&count[threadIdx.x], here[threadIdx.x]);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < PER; ++j)
    if (cls[j] >= 0)
      nodes[(int64_t)cls[j] * n + base[cls[j]] + number[j]] =
          (int32_t)(first + j * 256 + threadIdx.x);
}

// Whether the faster first form of a join is worth trying for a node, by how that has gone so
// far: nodes tried (upper half of a word) and nodes it was given up for (lower half).  Where that
// was more than every third, it is tried for one node in 16 only.  What is counted decides on
// time alone, never on results, so a sample is enough: one wavefront (or node) in 64 adds to the
// word (with all of them the waves queued for it: 30,000 x 96, six iterations 2.18 -> 2.5 ms),
// and the sampling stage makes the past count little against the coming iteration.
// The nodes are picked by a hash: every 16th node would be the same XCD's in most launches, which
// then finishes last (chi-square, values below zero: 7.5 instead of 6.2 ms per launch).
struct FormTally {
  uint64_t seen;  // as the word was when the wavefront began, and its own nodes
  uint64_t own = 0;
  __device__ explicit FormTally(uint64_t word) : seen(word) {}
  __device__ static bool in_16(uint32_t number) { return number * 0x9e3779b1u >> 28 == 0u; }
  __device__ static bool in_64(uint32_t number) { return number * 0x9e3779b1u >> 26 == 0u; }
  __device__ bool promising(uint32_t node) const {
    return 3 * (seen & 0xffffffffull) <= (seen >> 32) || in_16(node);
  }
  __device__ void count(bool given_up) {
    const uint64_t one = (1ull << 32) | (given_up ? 1ull : 0ull);
    seen += one;
    own += one;
  }
  __device__ static uint64_t faded(uint64_t word) {
    return word >> 37 << 32 | (word & 0xffffffffull) >> 5;
  }
};

// Numbering inside one merge (Sec. 5.1 shards).  The two sets are the ranges
// [base1, base1 + n1) and [base2, base2 + n2) of a larger collection; inside
// the merge S1 is 0..n1-1, S2 is n1..n-1, and any other object (a list entry
// left by an earlier merge with a third shard: "frozen", never sampled) is
// n + its collection id.
struct MergeIds {
  int64_t n1, base1, n2, base2;
  __host__ __device__ uint32_t to_internal(int64_t g) const {
    if (g >= base1 && g < base1 + n1) return (uint32_t)(g - base1);
    if (g >= base2 && g < base2 + n2) return (uint32_t)(n1 + g - base2);
    return (uint32_t)(n1 + n2 + g);
  }
  __host__ __device__ int32_t to_global(int64_t i) const {
    if (i < n1) return (int32_t)(base1 + i);
    if (i < n1 + n2) return (int32_t)(base2 + i - n1);
    return (int32_t)(i - n1 - n2);
  }
};

// Draw `count` (<= 64) distinct ids out of [0, range) + base for node s, one per
// lane: slot j takes hash(base_hash, s, j, attempt) mapped onto the range for
// attempt = 0, 1, ... until the id differs from `forbid` and from the ids of
// the slots before it; after kHashAttempts failures it walks to the next free
// id cyclically.  Wave-uniform loop; returns the id of slot `lane` (lanes >=
// count: undefined).
// First attempt of slot `lane`.  When the first attempts of all slots are
// pairwise distinct and none is `forbid`, the slot-by-slot rule accepts every
// one of them as it stands (a slot only ever looks at the slots before it).
__device__ inline uint32_t draw_first(uint64_t base_hash, uint32_t s, uint32_t range,
                                      uint32_t base, int lane) {
  return bounded(hash3(base_hash, s, (uint32_t)lane, 0u), range) + base;
}
__device__ inline uint32_t draw_slot_by_slot(uint64_t base_hash, uint32_t s, int count,
                                             uint32_t range, uint32_t base, uint32_t forbid,
                                             int lane);
__device__ inline uint32_t draw_distinct(uint64_t base_hash, uint32_t s, int count,
                                         uint32_t range, uint32_t base, uint32_t forbid,
                                         int lane) {
  const uint32_t first = draw_first(base_hash, s, range, base, lane);
  bool clash_any = lane < count && first == forbid;
  for (int j = 0; j + 1 < count; ++j) {
    const uint32_t cj = (uint32_t)__builtin_amdgcn_readlane((int)first, j);
    clash_any |= lane > j && lane < count && first == cj;
  }
  if (__ballot(clash_any) == 0ull) return first;
  return draw_slot_by_slot(base_hash, s, count, range, base, forbid, lane);
}
__device__ inline uint32_t draw_slot_by_slot(uint64_t base_hash, uint32_t s, int count,
                                             uint32_t range, uint32_t base, uint32_t forbid,
                                             int lane) {
  uint32_t mine = 0xffffffffu;
  for (int j = 0; j < count; ++j) {
    uint32_t cand = 0;
    bool ok = false;
    for (uint32_t attempt = 0; attempt < kHashAttempts && !ok; ++attempt) {
      cand = bounded(hash3(base_hash, s, (uint32_t)j, attempt), range) + base;
      bool clash = (lane < j) && (mine == cand);
      ok = (cand != forbid) && (__ballot(clash) == 0ull);
    }
    // at most `range` steps: the host has checked that enough ids are free
    for (uint32_t step = 0; step < range && !ok; ++step) {
      uint32_t local = cand - base;
      local = (local + 1 == range) ? 0 : local + 1;
      cand = local + base;
      bool clash = (lane < j) && (mine == cand);
      ok = (cand != forbid) && (__ballot(clash) == 0ull);
    }
    if (lane == j) mine = cand;
  }
  return mine;
}

}  // namespace gnnd

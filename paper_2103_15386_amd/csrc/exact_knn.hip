// Exhaustive exact K-NN of query nodes (ground truth of Recall@K).
//
// A workgroup answers Q queries (Q = 8, 4, 2 or 1 by the number of queries); its wavefronts
// take tiles of 64 rows in turn, one row per lane, so a value of a row is used for Q distances
// while the queries' values are the same for the whole wavefront and come through scalar
// registers.  The rows pass through the wavefront's own LDS tile, kChunk words of every row at
// a time, with coalesced reads and the next chunk in flight in registers while this one is
// evaluated; no barriers between the wavefronts until the end.  The distance of a
// pair is accumulated in the canonical order (JoinTraits).
//
// Every wavefront keeps the best 64 of its tiles for each query in its lanes; the smallest
// K-th best key of any wavefront, kept in LDS, turns most tiles away with one comparison.
//
// Bound: vector-ALU issue, Q (angular) or 2 Q (squared L2) instructions per dimension and row.
#include "device_utils.hpp"
#include "kernels.hpp"

namespace gnnd {

namespace {

constexpr int kEWaves = 16;               // wavefronts per workgroup, 4 per SIMD
constexpr int kEBlock = kEWaves * kWave;  // 1024 threads
constexpr int kChunkF = 32;               // float dimensions per chunk
constexpr int kChunkB = 16;               // words of four bytes per chunk of uint8 rows
// row strides of the tile: rows start at multiples of 16 bytes, and 8 lanes of a 16-byte access
// to 8 consecutive rows touch all banks once
constexpr int kStrideF = kChunkF + 4, kStrideB = kChunkB + 4;

using uniform_f32 = const __attribute__((address_space(4))) float;  // read by scalar loads

__device__ inline void tile_fence() {  // the lanes of a wavefront exchange data through LDS
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The smallest K keys seen so far, ascending over the lanes.  A tile that offers only a few
// keys enters them one by one (a lane shift each), otherwise the tile is sorted and merged.
__device__ inline void take_tile(uint64_t& best, uint64_t key, uint64_t* shared_last, int K,
                                 int lane) {
  uint64_t bound = *reinterpret_cast<volatile uint64_t*>(shared_last);
  bound = vmin(bound, readlane64(best, K - 1));
  uint64_t left = __ballot(key < bound);
  if (left == 0ull) return;
  if (__popcll(left) <= 6) {
    do {
      const int l = __ffsll((unsigned long long)left) - 1;
      left &= left - 1;
      const uint64_t x = readlane64(key, l);
      const uint64_t up = __shfl_up(best, 1, kWave);
      const int at = __popcll(__ballot(best < x));  // best ascends: x belongs at place `at`
      best = lane < at ? best : (lane == at ? x : up);
    } while (left != 0ull);
  } else {
    // (the lane's number taken anew: the networks' lane patterns are worked out here instead of
    // being held in scalar registers all through the kernel)
    asm volatile("" : "+v"(lane));
    key = key < bound ? key : kKeyMax;
    key = wave_sort(key, lane);
    best = wave_merge_smallest(best, key, lane);
  }
  const uint64_t last = readlane64(best, K - 1);
  if (lane == 0 && last < bound)
    atomicMin(reinterpret_cast<unsigned long long*>(shared_last), (unsigned long long)last);
}

template <int METRIC, int Q>
__global__ __launch_bounds__(kEBlock) void k_exact_knn(const void* vec, int64_t n, int d,
                                                       const int32_t* queries, int64_t nq, int K,
                                                       int32_t* ids_out, void* dist_out) {
  constexpr bool kBytes = METRIC == kL2U8;
  constexpr int kChunk = kBytes ? kChunkB : kChunkF;    // words per row and chunk
  constexpr int kStride = kBytes ? kStrideB : kStrideF;
  constexpr int kRows = kBytes ? kWave + Q : kWave;     // bytes: the queries' words as well
  constexpr int kPerRow = kChunk / 4;                   // lanes that read a row's chunk
  constexpr int kRowsAtOnce = kWave / kPerRow;
  constexpr int kLoads = (kRows + kRowsAtOnce - 1) / kRowsAtOnce;
  extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
  __shared__ uint64_t last_of[Q];
  const int lane = lane_id(), wave = wave_id();
  uint32_t* const tile = lds + wave * (kRows * kStride);
  const int64_t q0 = (int64_t)blockIdx.x * Q;
  // a query id that is no node reads row 0 and gets the "none" answer (-1, largest distance)
  uint32_t qid[Q];
  bool valid[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const uint32_t s = q0 + q < nq ? (uint32_t)queries[q0 + q] : 0xffffffffu;
    qid[q] = __builtin_amdgcn_readfirstlane(s);
    valid[q] = (int64_t)qid[q] < n;
  }
  auto query_row = [&](int q) { return valid[q] ? (int64_t)qid[q] : 0; };
  if (threadIdx.x < Q) last_of[threadIdx.x] = kKeyMax;
  __syncthreads();
  float qnorm[Q];
  if constexpr (METRIC == kCosineF32) {
    float acc = 0.f;
    const float* mine = reinterpret_cast<const float*>(vec);
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (lane == q) mine += query_row(q) * d;
    for (int j = 0; j < d; ++j) acc = __fmaf_rn(mine[j], mine[j], acc);
#pragma unroll
    for (int q = 0; q < Q; ++q)
      qnorm[q] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(acc), q));
  }
  const int words = kBytes ? (d + 3) >> 2 : d;  // words per row
  const bool aligned = kBytes ? (d & 15) == 0 : (d & 3) == 0;  // rows are multiples of 16 bytes
  const int part = (lane & (kPerRow - 1)) * 4, rsel = lane / kPerRow;

  uint64_t best[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) best[q] = kKeyMax;

  // this lane's share of the chunk at word w0 of the rows of the tile that starts at row c0
  uint4 reg[kLoads];
  auto fetch = [&](int64_t c0, int w0) {
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const int r = i * kRowsAtOnce + rsel;
      int64_t row = c0 + r;
      bool on = row < n;
      if (kBytes && i * kRowsAtOnce + kRowsAtOnce > kWave && r >= kWave) {
        row = 0;
        on = r < kRows;
#pragma unroll
        for (int q = 0; q < Q; ++q)
          if (r == kWave + q) row = query_row(q);
      }
      const int w = w0 + part;
      uint32_t v[4] = {0u, 0u, 0u, 0u};
      if (on) {
        if (!kBytes) {
          const float* src = reinterpret_cast<const float*>(vec) + row * d + w;
          if (aligned) {
            if (w < words) {
              const uint4 x = *reinterpret_cast<const uint4*>(src);
              v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
            }
          } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
              if (w + j < words) v[j] = __float_as_uint(src[j]);
          }
        } else {
          const uint8_t* src = reinterpret_cast<const uint8_t*>(vec) + row * d + 4 * (int64_t)w;
          if (aligned) {
            if (w < words) {
              const uint4 x = *reinterpret_cast<const uint4*>(src);
              v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
            }
          } else if ((d & 3) == 0) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
              if (w + j < words) v[j] = reinterpret_cast<const uint32_t*>(src)[j];
          } else {
#pragma unroll
            for (int j = 0; j < 16; ++j)
              if (4 * w + j < d) v[j >> 2] |= (uint32_t)src[j] << (8 * (j & 3));
          }
        }
      }
      reg[i] = make_uint4(v[0], v[1], v[2], v[3]);
    }
  };
  auto put = [&]() {
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const int r = i * kRowsAtOnce + rsel;
      if (r < kRows) *reinterpret_cast<uint4*>(tile + r * kStride + part) = reg[i];
    }
  };

  const int64_t step = (int64_t)kEBlock;
  const int64_t first = (int64_t)wave * kWave;
  if (first < n) fetch(first, 0);
  for (int64_t c0 = first; c0 < n; c0 += step) {
    float acc[Q], norm = 0.f;
    uint32_t dot[Q], qq[Q], cc = 0u;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      acc[q] = 0.f;
      dot[q] = qq[q] = 0u;
    }
    for (int w0 = 0; w0 < words; w0 += kChunk) {
      tile_fence();  // the chunk before this one has been read
      put();
      tile_fence();
      // request the next chunk, of this tile or of the next one
      if (w0 + kChunk < words) fetch(c0, w0 + kChunk);
      else if (c0 + step < n) fetch(c0 + step, 0);
      const int width = words - w0 < kChunk ? words - w0 : kChunk;
      if constexpr (kBytes) {
        for (int j = 0; j < width; j += 4) {  // words past the end are zeros
          const uint4 x = *reinterpret_cast<const uint4*>(tile + lane * kStride + j);
          cc = __builtin_amdgcn_udot4(x.x, x.x, cc, false);
          cc = __builtin_amdgcn_udot4(x.y, x.y, cc, false);
          cc = __builtin_amdgcn_udot4(x.z, x.z, cc, false);
          cc = __builtin_amdgcn_udot4(x.w, x.w, cc, false);
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            const uint4 y = *reinterpret_cast<const uint4*>(tile + (kWave + q) * kStride + j);
            dot[q] = __builtin_amdgcn_udot4(x.x, y.x, dot[q], false);
            dot[q] = __builtin_amdgcn_udot4(x.y, y.y, dot[q], false);
            dot[q] = __builtin_amdgcn_udot4(x.z, y.z, dot[q], false);
            dot[q] = __builtin_amdgcn_udot4(x.w, y.w, dot[q], false);
            qq[q] = __builtin_amdgcn_udot4(y.x, y.x, qq[q], false);
            qq[q] = __builtin_amdgcn_udot4(y.y, y.y, qq[q], false);
            qq[q] = __builtin_amdgcn_udot4(y.z, y.z, qq[q], false);
            qq[q] = __builtin_amdgcn_udot4(y.w, y.w, qq[q], false);
          }
        }
      } else {
        uniform_f32* qrow[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q)
          qrow[q] = (uniform_f32*)(reinterpret_cast<uintptr_t>(vec) +
                                   (size_t)(query_row(q) * d + w0) * 4);
        auto pair_step = [&](float y, int j) {
          if constexpr (METRIC == kCosineF32) norm = __fmaf_rn(y, y, norm);
#pragma unroll
          for (int q = 0; q < Q; ++q) JoinTraits<METRIC>::step(qrow[q][j], y, acc[q]);
        };
        const float* mine = reinterpret_cast<const float*>(tile) + lane * kStride;
        int j = 0;
#pragma unroll 1
        for (; j + 3 < width; j += 4) {
          const float4 y = *reinterpret_cast<const float4*>(mine + j);
          pair_step(y.x, j);
          pair_step(y.y, j + 1);
          pair_step(y.z, j + 2);
          pair_step(y.w, j + 3);
        }
        for (; j < width; ++j) pair_step(mine[j], j);
      }
    }
    const int64_t c = c0 + lane;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      uint32_t code;
      if constexpr (kBytes) code = ord_i32((int32_t)(qq[q] + cc - 2u * dot[q]));
      else if constexpr (METRIC == kCosineF32) code = cosine_code(acc[q], qnorm[q], norm);
      else code = JoinTraits<METRIC>::code(acc[q]);
      uint64_t key = ((uint64_t)code << 32) | (uint64_t)c;
      if (c >= n || c == (int64_t)qid[q]) key = kKeyMax;
      take_tile(best[q], key, &last_of[q], K, lane);
    }
  }

  // the wavefronts' lists of a query, merged by the first wavefront that is numbered like it
  __syncthreads();  // the tiles are no longer in use
  uint64_t* const part_lists = reinterpret_cast<uint64_t*>(lds);  // [Q][kEWaves][64]
#pragma unroll
  for (int q = 0; q < Q; ++q) part_lists[(q * kEWaves + wave) * kWave + lane] = best[q];
  __syncthreads();
  if (wave >= Q || q0 + wave >= nq) return;
  bool have_query = false;
#pragma unroll
  for (int q = 0; q < Q; ++q)
    if (wave == q) have_query = valid[q];
  uint64_t all = part_lists[wave * kEWaves * kWave + lane];
  for (int w = 1; w < kEWaves; ++w)
    all = wave_merge_smallest(all, part_lists[(wave * kEWaves + w) * kWave + lane], lane);
  if (lane < K) {
    const bool have = have_query && all != kKeyMax;
    const int64_t at = (q0 + wave) * K + lane;
    const uint32_t code = (uint32_t)(all >> 32);
    ids_out[at] = have ? (int32_t)(uint32_t)all : -1;
    if (kBytes)
      reinterpret_cast<int32_t*>(dist_out)[at] = have ? unord_i32(code) : 0x7fffffff;
    else
      reinterpret_cast<float*>(dist_out)[at] =
          have ? unord_f32(code) : __uint_as_float(0x7f800000u);
  }
}

template <int METRIC, int Q>
hipError_t launch(const void* vec, int64_t n, int32_t d, const int32_t* queries, int64_t nq,
                  int32_t K, int32_t* ids_out, void* dist_out, hipStream_t st) {
  constexpr size_t tiles = (size_t)kEWaves * (METRIC == kL2U8 ? (kWave + Q) * kStrideB
                                                              : kWave * kStrideF) * 4;
  constexpr size_t lists = (size_t)Q * kEBlock * 8;
  constexpr size_t bytes = tiles > lists ? tiles : lists;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_exact_knn<METRIC, Q>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e != hipSuccess) return e;
  k_exact_knn<METRIC, Q><<<(unsigned)((nq + Q - 1) / Q), kEBlock, bytes, st>>>(
      vec, n, d, queries, nq, K, ids_out, dist_out);
  return hipGetLastError();
}

// Queries per workgroup: one workgroup fills a CU and reads all rows once, so the time is the
// number of rounds of 256 workgroups times what a round takes - Q distances per row plus
// moving the row through LDS, about as much as two.
template <int METRIC>
hipError_t launch_metric(const void* vec, int64_t n, int32_t d, const int32_t* queries, int64_t nq,
                         int32_t K, int32_t* ids_out, void* dist_out, hipStream_t st) {
  int q = 1;
  int64_t least = INT64_MAX;
  for (int c = 1; c <= 8; c *= 2) {
    const int64_t rounds = ((nq + c - 1) / c + 255) / 256, cost = rounds * (c + 2);
    if (cost < least) {
      least = cost;
      q = c;
    }
  }
  switch (q) {
    case 1: return launch<METRIC, 1>(vec, n, d, queries, nq, K, ids_out, dist_out, st);
    case 2: return launch<METRIC, 2>(vec, n, d, queries, nq, K, ids_out, dist_out, st);
    case 4: return launch<METRIC, 4>(vec, n, d, queries, nq, K, ids_out, dist_out, st);
    default: return launch<METRIC, 8>(vec, n, d, queries, nq, K, ids_out, dist_out, st);
  }
}

}  // namespace

hipError_t launch_exact_knn(const void* vec, int64_t n, int32_t d, int32_t metric,
                            const int32_t* queries, int64_t nq, int32_t K, int32_t* ids_out,
                            void* dist_out, hipStream_t st) {
  if (nq == 0) return hipSuccess;
  switch (metric) {
    case kL2F32: return launch_metric<kL2F32>(vec, n, d, queries, nq, K, ids_out, dist_out, st);
    case kAngularF32:
      return launch_metric<kAngularF32>(vec, n, d, queries, nq, K, ids_out, dist_out, st);
    case kChi2F32: return launch_metric<kChi2F32>(vec, n, d, queries, nq, K, ids_out, dist_out, st);
    case kCosineF32:
      return launch_metric<kCosineF32>(vec, n, d, queries, nq, K, ids_out, dist_out, st);
    default: return launch_metric<kL2U8>(vec, n, d, queries, nq, K, ids_out, dist_out, st);
  }
}

}  // namespace gnnd

// Exhaustive exact K-NN of query nodes (ground truth of Recall@K).
//
// A workgroup of 16 wavefronts answers Q queries (Q = 8, 4, 2 or 1 by the number of queries);
// its wavefronts take tiles of 128 rows in turn, two rows per lane.  The rows pass through the
// wavefront's own LDS tile, 16 words of every row at a time, with coalesced reads and the next
// chunk in flight in registers while this one is evaluated; the queries' words lie behind the
// rows' and are read by all lanes at once.  Per four dimensions a lane reads 2 + Q 16-byte
// pieces from LDS for 8 Q steps of the canonical sums (JoinTraits).  No barriers between the
// wavefronts until the end.
//
// Every wavefront keeps the best 64 of its tiles for each query in its lanes; the smallest
// K-th best key of any wavefront, kept in LDS, turns most tiles away with one comparison per
// query and row.
//
// 2000 queries x 10^6 x 96 under the angular distance: 9.8 ms, 39 TFLOP/s (455 ms with one
// query per workgroup and a row per lane straight from memory; 18 ms with one row per lane and
// the queries through scalar loads, whose latency it waited for).  Bound: vector-ALU issue
// (0.75 busy; 4.9 ms at the full rate without packed instructions, squared L2 takes two
// instructions per dimension and pair), then LDS reads (0.56 busy).
#include "device_utils.hpp"
#include "kernels.hpp"

namespace gnnd {

namespace {

constexpr int kEWaves = 16;               // wavefronts per workgroup, 4 per SIMD
constexpr int kEBlock = kEWaves * kWave;  // 1024 threads
constexpr int kLaneRows = 2;              // rows per lane and tile
constexpr int kTile = kLaneRows * kWave;  // rows per tile
constexpr int kChunk = 16;                // words (floats, or four bytes) per row and chunk
constexpr int kPieces = kChunk / 4;       // 16-byte pieces per row and chunk
constexpr int kRowsAtOnce = kWave / kPieces;
constexpr int kLoads = kTile / kRowsAtOnce;

// Where piece `part` of a row lies in the tile, in words: the pieces of four rows change places
// so that 16 lanes reading the same piece of 16 consecutive rows touch every bank once.
__device__ inline int piece_at(int row, int part) {
  return row * kChunk + ((part ^ (row >> 2)) & (kPieces - 1)) * 4;
}

__device__ inline void tile_fence() {  // the lanes of a wavefront exchange data through LDS
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Enter the keys below the K-th best of any wavefront in the ascending list `best`.  A few
// keys are entered one by one (a lane shift each), more are sorted and merged.
__device__ inline void take_keys(uint64_t& best, uint64_t key, uint64_t* shared_last, int K,
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

// ALIGNED: rows are multiples of 16 bytes (and not longer than 64 MiB).
template <int METRIC, int Q, bool ALIGNED>
__global__ __launch_bounds__(kEBlock) void k_exact_knn(const void* vec, int64_t n, int d,
                                                       const int32_t* queries, int64_t nq, int K,
                                                       int32_t* ids_out, void* dist_out,
                                                       const uint8_t* only) {
  constexpr bool kBytes = METRIC == kL2U8;
  extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
  __shared__ uint64_t last_of[8];
  const int lane = lane_id(), wave = wave_id();
  uint32_t* const tile = lds + wave * ((kTile + Q) * kChunk);
  const int64_t q0 = (int64_t)blockIdx.x * Q;
  if (only) {  // uniform
    bool any = false;
    for (int q = 0; q < Q; ++q) any = any || (q0 + q < nq && only[q0 + q] == 1);
    if (!any) return;
  }
  if (threadIdx.x < 8) last_of[threadIdx.x] = kKeyMax;
  __syncthreads();
  const int words = kBytes ? (d + 3) >> 2 : d;  // words per row
  const int64_t row_bytes = kBytes ? d : (int64_t)d * 4;
  const char* const rows = reinterpret_cast<const char*>(vec);
  const int part = lane & (kPieces - 1), rsel = lane / kPieces;

  // lanes 4 q .. 4 q + 3 bring the pieces of query q.  A query id that is no node reads row 0
  // and gets the "none" answer (-1, largest distance).
  const int my_q = rsel < Q ? rsel : 0;
  const char* query_row;
  {
    const uint32_t s = q0 + my_q < nq ? (uint32_t)queries[q0 + my_q] : 0xffffffffu;
    query_row = rows + ((int64_t)s < n ? (int64_t)s * row_bytes : 0);
  }
  uint32_t qid[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q)
    qid[q] = __builtin_amdgcn_readfirstlane(q0 + q < nq ? (uint32_t)queries[q0 + q] : 0xffffffffu);

  // A tile is always 128 rows: the last one is moved back (its rows before `c0` have been
  // seen); only with fewer than 128 rows in all are places of the tile left without a row.
  const int64_t last_tile = n > kTile ? n - kTile : 0;
  const int rows_here = n < kTile ? (int)n : kTile;
  // ALIGNED: this lane's share of the chunk at word w0 of the rows of a tile, four lanes per
  // row.  What lies beyond the rows' end is not used: the last piece is read once more.
  uint4 reg[kLoads], qreg;
  auto fetch = [&](int64_t c0, int w0) {
    const char* const first_row = rows + (c0 < last_tile ? c0 : last_tile) * row_bytes;
    const int w = w0 + 4 * part;
    const uint32_t at = 4u * (uint32_t)(w < words ? w : words - 4);
    const uint32_t off = (uint32_t)(rsel * row_bytes) + at;
    if (rows_here == kTile) {
#pragma unroll
      for (int i = 0; i < kLoads; ++i)
        reg[i] = *reinterpret_cast<const uint4*>(first_row + i * kRowsAtOnce * row_bytes + off);
    } else {
#pragma unroll
      for (int i = 0; i < kLoads; ++i) {
        reg[i] = make_uint4(0u, 0u, 0u, 0u);
        if (i * kRowsAtOnce + rsel < rows_here)
          reg[i] = *reinterpret_cast<const uint4*>(first_row + i * kRowsAtOnce * row_bytes + off);
      }
    }
    qreg = *reinterpret_cast<const uint4*>(query_row + at);
  };
  auto put = [&]() {
#pragma unroll
    for (int i = 0; i < kLoads; ++i)
      *reinterpret_cast<uint4*>(tile + piece_at(i * kRowsAtOnce + rsel, part)) = reg[i];
    if (rsel < Q) *reinterpret_cast<uint4*>(tile + (kTile + rsel) * kChunk + 4 * part) = qreg;
  };
  // other rows: word by word, 16 lanes per row, straight to the tile; what lies beyond the
  // rows' end is zero (for bytes it takes part in the dot products)
  auto bring = [&](int64_t c0, int w0) {
    const char* const first_row = rows + (c0 < last_tile ? c0 : last_tile) * row_bytes;
    const int col = lane & (kChunk - 1), w = w0 + col;
#pragma unroll 4
    for (int i = 0; i < (kTile + Q + 3) / 4; ++i) {
      const int r = 4 * i + lane / kChunk;
      if (r >= kTile + Q || (r < kTile && r >= rows_here) || w >= words) continue;
      const char* src = first_row + r * row_bytes;
      if (r >= kTile) {
        const uint32_t s = q0 + r - kTile < nq ? (uint32_t)queries[q0 + r - kTile] : 0xffffffffu;
        src = rows + ((int64_t)s < n ? (int64_t)s * row_bytes : 0);
      }
      uint32_t v = 0u;
      if (!kBytes || (d & 3) == 0) {
        v = reinterpret_cast<const uint32_t*>(src)[w];
      } else if (4 * w + 3 < d) {
        __builtin_memcpy(&v, src + 4 * (int64_t)w, 4);  // (rows of odd length: not aligned)
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (4 * w + e < d) v |= (uint32_t)(uint8_t)src[4 * (int64_t)w + e] << (8 * e);
      }
      tile[r < kTile ? piece_at(r, col >> 2) + (col & 3) : r * kChunk + col] = v;
    }
    if (w >= words && kBytes)
      for (int i = 0; i < (kTile + Q + 3) / 4; ++i) {
        const int r = 4 * i + lane / kChunk;
        if (r < kTile + Q)
          tile[r < kTile ? piece_at(r, col >> 2) + (col & 3) : r * kChunk + col] = 0u;
      }
  };

  uint64_t best[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) best[q] = kKeyMax;
  constexpr int64_t step = (int64_t)kEWaves * kTile;
  const int64_t first = (int64_t)wave * kTile;
  if (ALIGNED && first < n) fetch(first, 0);
  for (int64_t c0 = first; c0 < n; c0 += step) {
    // floats: running sums; bytes: inner products (and the squared norms)
    typename JoinTraits<kBytes ? kL2U8 : METRIC>::acc acc[Q][kLaneRows];
    float qnorm[Q], norm[kLaneRows];
    uint32_t qq[Q], cc[kLaneRows];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      qnorm[q] = 0.f;
      qq[q] = 0u;
#pragma unroll
      for (int i = 0; i < kLaneRows; ++i) acc[q][i] = 0;
    }
#pragma unroll
    for (int i = 0; i < kLaneRows; ++i) {
      norm[i] = 0.f;
      cc[i] = 0u;
    }
    for (int w0 = 0; w0 < words; w0 += kChunk) {
      tile_fence();  // the chunk before this one has been read
      if (ALIGNED) put();
      else bring(c0, w0);
      tile_fence();
      if (ALIGNED) {  // request the next chunk, of this tile or of the next one
        if (w0 + kChunk < words) fetch(c0, w0 + kChunk);
        else if (c0 + step < n) fetch(c0 + step, 0);
      }
      const int width = words - w0 < kChunk ? words - w0 : kChunk;
#pragma unroll 1
      for (int j = 0; j < width; j += 4) {
        uint4 x[kLaneRows];
#pragma unroll
        for (int i = 0; i < kLaneRows; ++i)
          x[i] = *reinterpret_cast<const uint4*>(tile + piece_at(i * kWave + lane, j >> 2));
        if constexpr (kBytes) {
          auto dot4 = [](const uint4& a, const uint4& b, uint32_t s) {
            s = __builtin_amdgcn_udot4(a.x, b.x, s, false);
            s = __builtin_amdgcn_udot4(a.y, b.y, s, false);
            s = __builtin_amdgcn_udot4(a.z, b.z, s, false);
            return __builtin_amdgcn_udot4(a.w, b.w, s, false);
          };
#pragma unroll
          for (int i = 0; i < kLaneRows; ++i) cc[i] = dot4(x[i], x[i], cc[i]);
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            const uint4 y = *reinterpret_cast<const uint4*>(tile + (kTile + q) * kChunk + j);
            qq[q] = dot4(y, y, qq[q]);
#pragma unroll
            for (int i = 0; i < kLaneRows; ++i)
              acc[q][i] = (int32_t)dot4(x[i], y, (uint32_t)acc[q][i]);
          }
        } else {
          auto f = [](uint32_t b) { return __uint_as_float(b); };
          auto steps = [&](int c) {  // the first c dimensions of these four
#pragma unroll
            for (int q = 0; q < Q; ++q) {
              const uint4 y = *reinterpret_cast<const uint4*>(tile + (kTile + q) * kChunk + j);
              const uint32_t yw[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                if (e < c) {
                  if constexpr (METRIC == kCosineF32)
                    qnorm[q] = __fmaf_rn(f(yw[e]), f(yw[e]), qnorm[q]);
#pragma unroll
                  for (int i = 0; i < kLaneRows; ++i) {
                    const uint32_t xw[4] = {x[i].x, x[i].y, x[i].z, x[i].w};
                    JoinTraits<METRIC>::step(f(yw[e]), f(xw[e]), acc[q][i]);
                  }
                }
              }
            }
            if constexpr (METRIC == kCosineF32) {
#pragma unroll
              for (int i = 0; i < kLaneRows; ++i) {
                const uint32_t xw[4] = {x[i].x, x[i].y, x[i].z, x[i].w};
#pragma unroll
                for (int e = 0; e < 4; ++e)
                  if (e < c) norm[i] = __fmaf_rn(f(xw[e]), f(xw[e]), norm[i]);
              }
            }
          };
          if (ALIGNED || j + 4 <= width) steps(4);
          else steps(width - j);
        }
      }
    }
    // bounds of the queries' lists, read once per tile: upper halves, so "not above" may
    // enter; take_keys compares whole keys
    const uint32_t my_bound =
        (uint32_t)(*reinterpret_cast<volatile uint64_t*>(&last_of[lane & 7]) >> 32);
    const int64_t tile0 = c0 < last_tile ? c0 : last_tile;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const uint32_t bound = __builtin_amdgcn_readlane(my_bound, q);
#pragma unroll
      for (int i = 0; i < kLaneRows; ++i) {
        uint32_t code;
        if constexpr (kBytes) code = ord_i32((int32_t)(qq[q] + cc[i] - 2u * (uint32_t)acc[q][i]));
        else if constexpr (METRIC == kCosineF32) code = cosine_code(acc[q][i], qnorm[q], norm[i]);
        else code = JoinTraits<METRIC>::code(acc[q][i]);
        if (__ballot(code <= bound) == 0ull) continue;
        const int64_t c = tile0 + i * kWave + lane;
        uint64_t key = ((uint64_t)code << 32) | (uint64_t)c;
        if (c < c0 || c >= n || c == (int64_t)qid[q]) key = kKeyMax;
        take_keys(best[q], key, &last_of[q], K, lane);
      }
    }
  }

  // the wavefronts' lists of query q, merged by wavefront q (few rows: of those that had a tile)
  const int filled = n < step ? (int)((n + kTile - 1) / kTile) : kEWaves;
  __syncthreads();  // the tiles are no longer in use
  uint64_t* const lists = reinterpret_cast<uint64_t*>(lds);  // [Q][kEWaves][64]
#pragma unroll
  for (int q = 0; q < Q; ++q) lists[(q * kEWaves + wave) * kWave + lane] = best[q];
  __syncthreads();
  if (wave >= Q || q0 + wave >= nq || (only && only[q0 + wave] != 1)) return;
  uint64_t all = lists[wave * kEWaves * kWave + lane];
  for (int w = 1; w < filled; ++w)
    all = wave_merge_smallest(all, lists[(wave * kEWaves + w) * kWave + lane], lane);
  if (lane < K) {
    const bool have = (int64_t)(uint32_t)queries[q0 + wave] < n && all != kKeyMax;
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
                  int32_t K, int32_t* ids_out, void* dist_out, hipStream_t st,
                  const uint8_t* only) {
  constexpr size_t tiles = (size_t)kEWaves * (kTile + Q) * kChunk * 4;
  constexpr size_t lists = (size_t)Q * kEBlock * 8;
  constexpr size_t bytes = tiles > lists ? tiles : lists;
  // (offsets inside a tile are 32-bit there: 16 rows of at most 64 MiB)
  const bool aligned = METRIC == kL2U8 ? (d & 15) == 0 && d <= (1 << 26)
                                       : (d & 3) == 0 && d <= (1 << 24);
  auto* const kernel = aligned ? k_exact_knn<METRIC, Q, true> : k_exact_knn<METRIC, Q, false>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e != hipSuccess) return e;
  kernel<<<(unsigned)((nq + Q - 1) / Q), kEBlock, bytes, st>>>(vec, n, d, queries, nq, K, ids_out,
                                                               dist_out, only);
  return hipGetLastError();
}

template <int METRIC>
hipError_t launch_metric(const void* vec, int64_t n, int32_t d, const int32_t* queries, int64_t nq,
                         int32_t K, int32_t* ids_out, void* dist_out, hipStream_t st,
                         const uint8_t* only) {
  switch (exact_queries(nq)) {
    case 1: return launch<METRIC, 1>(vec, n, d, queries, nq, K, ids_out, dist_out, st, only);
    case 2: return launch<METRIC, 2>(vec, n, d, queries, nq, K, ids_out, dist_out, st, only);
    case 4: return launch<METRIC, 4>(vec, n, d, queries, nq, K, ids_out, dist_out, st, only);
    default: return launch<METRIC, 8>(vec, n, d, queries, nq, K, ids_out, dist_out, st, only);
  }
}

}  // namespace

hipError_t launch_exact_knn(const void* vec, int64_t n, int32_t d, int32_t metric,
                            const int32_t* queries, int64_t nq, int32_t K, int32_t* ids_out,
                            void* dist_out, hipStream_t st, const uint8_t* only) {
  if (nq == 0) return hipSuccess;
  switch (metric) {
#define GNND_EXACT(M) \
  return launch_metric<M>(vec, n, d, queries, nq, K, ids_out, dist_out, st, only)
    case kL2F32: GNND_EXACT(kL2F32);
    case kAngularF32: GNND_EXACT(kAngularF32);
    case kChi2F32: GNND_EXACT(kChi2F32);
    case kCosineF32: GNND_EXACT(kCosineF32);
    default: GNND_EXACT(kL2U8);
#undef GNND_EXACT
  }
}

}  // namespace gnnd

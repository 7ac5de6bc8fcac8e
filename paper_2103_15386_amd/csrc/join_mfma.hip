// Cross-matching (Sec. 4.2) and nearest-object search (Sec. 4.3, Alg. 2) on
// the matrix cores, for byte-valued data: one 64-lane wavefront per node.
//
// The node's <= 64 NEW and <= 64 OLD sample vectors are read straight from HBM
// into MFMA operand registers (16 bytes per lane per 32-dimension step; a 128 B
// row is one cache line).  Vectors are stored shifted to int8 (x - 128), which
// leaves differences unchanged, so with the Gram block G = A.B^T from
// v_mfma_i32_32x32x32_i8 the squared distance is |a|^2 + |b|^2 - 2 G, exact in
// int32.  A 32x32 accumulator tile keeps one column per lane, so "nearest row
// object for every column object" is a per-lane min over 16 registers plus one
// half-wave swap; the tile is computed in both orientations where both
// directions are needed (NEW->OLD and OLD->NEW) instead of reducing across
// lanes.  Sample lists are sorted by id, so the row position inside a list
// breaks distance ties exactly like the id does.
#include <numeric>
#include <type_traits>

#include "device_utils.hpp"
#include "gram_i8.hpp"
#include "kernels.hpp"

namespace gnnd {

constexpr int kMB = 256;  // 4 waves = 4 nodes in flight per workgroup
constexpr int64_t kJoinGrid = 256 * 3 * 2;  // 256 CUs x 3 resident workgroups x 2
// staged hand-out: one workgroup of 12 waves per CU (3 per SIMD) shares the staging area
constexpr int kStagedWaves = 12;

constexpr int32_t kFar = 1 << 24;  // "norm" of an absent row: above every real distance
static_assert(far_enough(kFar, kFar >> 1, 6), "absent rows are told from present ones, keys fit");

// Convert float32 rows holding integers 0..255 (or uint8 rows) to int8 rows
// (value - 128) of `dpad` bytes, zero padded, and store the squared norm of
// the shifted row.  `bad` is raised when a float is not such an integer.
template <typename T>
__global__ __launch_bounds__(256) void k_pack_i8(const void* vec_a, const void* vec_b,
                                                 int64_t split, int64_t n, int d, int dpad,
                                                 int8_t* shadow, NodeMeta* meta, int* bad) {
  const int lane = lane_id();
  const int64_t row = block_linear() * 4 + wave_id();
  if (row >= n) return;
  const T* src = row < split ? reinterpret_cast<const T*>(vec_a) + row * d
                             : reinterpret_cast<const T*>(vec_b) + (row - split) * d;
  int32_t acc = 0;
  bool is_bad = false;
  for (int j = lane; j < dpad; j += kWave) {
    int32_t q = 0;
    if (j < d) {
      float f = (float)src[j];
      int32_t iv = (int32_t)f;
      if (!(f >= 0.f && f <= 255.f) || (float)iv != f) is_bad = true;
      q = iv - 128;
      acc += q * q;
    }
    shadow[row * dpad + j] = (int8_t)q;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, kWave);
  if (lane == 0) meta[row].norm = acc;
  if (__ballot(is_bad) != 0ull && lane == 0) atomicOr(bad, 1);
}

// The same for uint8 rows whose length is a multiple of 16: a lane moves 16
// bytes (x - 128 is x ^ 0x80 in every byte), C = dpad / 16 neighbouring lanes
// share a row, so loads and stores of a wavefront are contiguous.
__global__ __launch_bounds__(256) void k_pack_u8_wide(const uint8_t* vec_a, const uint8_t* vec_b,
                                                      int64_t split, int64_t n, int d, int dpad,
                                                      int8_t* shadow, NodeMeta* meta) {
  const int lane = lane_id();
  const int C = dpad >> 4, per_wave = kWave / C;
  const int grp = lane / C, sub = lane - grp * C;
  const int64_t row = (block_linear() * 4 + wave_id()) * per_wave + grp;
  const bool on = grp < per_wave && row < n;
  int32_t part = 0;
  if (on) {
    v4i q = {0, 0, 0, 0};
    if (16 * sub < d) {
      const uint8_t* src = row < split ? vec_a + row * d : vec_b + (row - split) * d;
      q = *reinterpret_cast<const v4i*>(src + 16 * sub);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        q[t] ^= (int)0x80808080;
        part = __builtin_amdgcn_sdot4(q[t], q[t], part, false);
      }
    }
    *reinterpret_cast<v4i*>(shadow + row * dpad + 16 * sub) = q;
  }
  int32_t total = 0;
  for (int t = 0; t < C; ++t) total += __shfl(part, (grp * C + t) & 63, kWave);
  if (on && sub == 0) meta[row].norm = total;
}

// Alg. 1, first loop, on the int8 rows: k distinct random neighbours per node,
// exact distances, sorted ascending by (distance, id), flagged NEW.  One
// wavefront per node.
template <bool FCODE>
__global__ __launch_bounds__(256) void k_init_random_i8(const int8_t* __restrict__ shadow,
                                                        NodeMeta* meta, int dpad, int64_t n, int k,
                                                        uint64_t base_hash, uint64_t* G) {
  const int lane = lane_id();
  const int64_t s = block_linear() * 4 + wave_id();
  if (s >= n) return;
  // the list for one id per lane, ascending
  auto list_of = [&](uint32_t id) {
    const int32_t dist = wave_distances_i8(shadow, meta, dpad, s, id, k, lane);
    uint64_t e = kKeyMax;
    if (lane < k) e = make_entry(FCODE ? ord_f32((float)dist) : ord_i32(dist), id, 1u);
    return wave_sort_upto(e, lane, k);
  };
  // First attempts of all slots at once.  Whether they are valid (pairwise distinct,
  // none the node itself) shows after the sort: equal ids have equal distances and
  // end up next to each other.  Only then the slot-by-slot rule has to run.
  uint64_t e = list_of(draw_first(base_hash, (uint32_t)s, (uint32_t)n, 0u, lane));
  const uint64_t prev = __shfl_up(e, 1, kWave);
  const bool bad = lane < k && (entry_id(e) == (uint32_t)s ||
                                (lane > 0 && entry_id(e) == entry_id(prev)));
  if (__ballot(bad) != 0ull)
    e = list_of(draw_slot_by_slot(base_hash, (uint32_t)s, k, (uint32_t)n, 0u, (uint32_t)s, lane));
  if (lane < k) G[s * k + lane] = e;
  if (lane == k - 1) meta[s].kth = entry_code(e);
}

// GGM, Alg. 3 "Divide" + "Append" on the int8 rows: keep the first ceil(k/2)
// entries (OLD), set the rest aside, refill with floor(k/2) random objects of
// the other set (NEW, exact distances) and restore the (distance, id) order.
template <bool FCODE>
__global__ __launch_bounds__(256) void k_merge_init_i8(const int8_t* __restrict__ shadow,
                                                       NodeMeta* meta, int dpad, int64_t n,
                                                       MergeIds mi, int k, uint64_t base_hash,
                                                       const int32_t* ids1, const void* dist1,
                                                       const int32_t* ids2, const void* dist2,
                                                       uint64_t* G, uint64_t* aside) {
  const int lane = lane_id();
  const int64_t s = block_linear() * 4 + wave_id();
  if (s >= n) return;
  const int64_t n1 = mi.n1;
  const bool first = s < n1;
  const int64_t loc = first ? s : s - n1;
  const int32_t* sid = (first ? ids1 : ids2) + loc * k;
  const void* sdist = first ? dist1 : dist2;
  const int keep = (k + 1) / 2, fill = k / 2;
  uint32_t id_in = 0, code_in = 0;
  if (lane < k) {
    id_in = mi.to_internal(sid[lane]);  // collection id -> numbering of this merge
    code_in = FCODE ? ord_f32(reinterpret_cast<const float*>(sdist)[loc * k + lane])
                    : ord_i32(reinterpret_cast<const int32_t*>(sdist)[loc * k + lane]);
  }
  if (lane >= keep && lane < k) aside[s * fill + (lane - keep)] = make_entry(code_in, id_in, 0u);
  const uint32_t draw = draw_distinct(base_hash, (uint32_t)s, fill,
                                      (uint32_t)(first ? n - n1 : n1), first ? (uint32_t)n1 : 0u,
                                      0xffffffffu, lane);
  const int32_t dist = wave_distances_i8(shadow, meta, dpad, s, draw, fill, lane);
  const uint32_t code_of_draw = FCODE ? ord_f32((float)dist) : ord_i32(dist);
  const int src = lane - keep;
  const uint32_t did = __shfl(draw, src < 0 ? 0 : src, kWave);
  const uint32_t code = __shfl(code_of_draw, src < 0 ? 0 : src, kWave);
  uint64_t e = kKeyMax;
  if (lane < keep) e = make_entry(code_in, id_in, 0u);
  else if (lane < k) e = make_entry(code, did, 1u);
  e = wave_sort(e, lane);
  if (lane < k) G[s * k + lane] = e;
  if (lane == k - 1) meta[s].kth = entry_code(e);
}

typedef uint64_t EntryPair __attribute__((ext_vector_type(2), aligned(8)));


// FCODE: distances are reported as float32 codes (float input data) instead of
// int32 codes.  MERGE: GGM mode - no NEW x NEW, only pairs from different sets.
//
// Each wavefront walks over the nodes of places s, s + W, s + 2W, ... (W = wavefronts in the
// grid; see StageArgs for their order) as a software pipeline, because a node costs three dependent memory
// round trips (sample ids -> vector rows -> result slots): while the tiles of
// node i are evaluated the ids of node i+1 are already in flight, and as soon
// as the last tile has consumed the operand registers the rows of node i+1 are
// requested, before the results of node i are handed out.
// STAGED: results are not handed to their destinations one by one (one returning
// device-wide atomic and one scattered 8-byte store each - the rate of those atomics
// was what the kernel ran at) but collected per workgroup in LDS, kStageSlots places
// for each of <= kStageBuckets buckets of consecutive destination ids, and written
// out bucket by bucket: one atomic and one contiguous piece per bucket and flush.
// The bucket regions tile an array shaped like `bins` (a bucket's region starts where
// the segment of its first destination starts, so it can hold whatever its
// destinations can receive); k_result_csr then moves every result into its
// destination's segment.  A result that finds its bucket's places taken goes to the
// bucket's region directly.  Where results gather in few buckets (a merge with a smaller set, hubs
// with neighbouring ids) those are full long before half of all places are, and one returning atomic
// per result on a few addresses is what the kernel then waits for; so a flush is due as well as soon as
// 52 of one bucket's 64 places are taken, which leaves room for what the other waves still add.
// Without / due when a bucket is full / this: merge of 300,000 with 30,000 x 96 bytes, k = p = 32, five
// iterations, 26.9 / 12.6 / 7.0 ms; of 97,631 with 36,081 x 45, k = 64, p = 32, - / 6.1 / 3.3; 600,000 x
// 64 bytes in the order of their distance from the mean, eight iterations 194 / 116 / 94; results spread
// evenly: no difference (10^6 x 128 23.0, sharded build of 4 x 600,000 172.1 ms).
//
// Neighbours in the collection are often neighbours in space (rows stored class by class), and then
// results for one node's samples go to a few buckets, the same ones as its neighbours'.  Were all waves
// at work on one stretch of ids, a few buckets' places and cursors would serve the whole chip; so the
// nodes are taken in an order that spreads those under way over all ids.  600,000 x 64 bytes sorted by
// cluster, k = p = 32, six iterations 166 -> 19 ms (in the order of the ids with the records read and no
// early flushes 108), a fifth of 600,000 rows zero, eight iterations, 197 -> 134; rows in random order as
// before (10^6 x 128 23.0 ms, sharded build of 4 x 600,000 172 to 173).
//
// The waves of a workgroup run at their own pace, so a flush is a rendezvous: every
// wave looks at the fill count after each node and joins the flush once it has reached
// the threshold (the count only falls inside a flush, so every wave gets there; a bucket
// that asks for one adds the threshold to it, once between two flushes); a wave
// that has run out of nodes keeps joining flushes until all waves have run out.
struct StageArgs {
  uint64_t* ent;            // bucket regions: staged results
  unsigned long long* cur;  // per bucket: results written to its region so far
  const uint64_t* poff;     // segment offsets of the destinations (n + 1)
  int tb, nb;               // log2(destinations per bucket), number of buckets
  uint32_t threshold;       // fill count that triggers a flush
  uint32_t spread, stride;  // the nodes are taken in the order 0, spread, 2 spread, ... mod n, each once;
                            // stride: from a wave's node to its next
  const uint64_t* all;      // not 0: the join hands on every result it finds; NULL: it does not
};
// results in a bucket that make a flush due (at 48 evenly spread results leave in more and shorter
// pieces, 10^6 x 128 0.3 % of the join; at 56 the merges above take 5 to 8 % longer)
constexpr uint32_t kStageSoon = kStageSlots * 13 / 16;
constexpr size_t kStageLdsBytes = (size_t)kStageBuckets * kStageSlots * 8 + kStageBuckets * 12 + 16;
// a staged result (see kStageDistShift) without its destination, and with it
__device__ inline uint64_t stage_entry(int32_t dist, uint32_t id) {
  return ((uint64_t)(uint32_t)dist << kStageDistShift) | (uint64_t)id;
}
// the code of its distance
template <bool FCODE>
__device__ inline uint32_t stage_code(uint64_t entry) {
  const int32_t dist = (int32_t)(entry >> kStageDistShift);
  return FCODE ? ord_f32((float)dist) : ord_i32(dist);
}
__device__ inline uint64_t stage_record(uint64_t entry, uint32_t dest, int tb) {
  return entry | ((uint64_t)(dest & ((1u << tb) - 1u)) << kStageIdBits);
}

// Squared norm of the row this lane's sample stands for, from the operand registers: sample
// `lane` of a list is row lane % 32 of block lane / 32, and lanes l and l + 32 hold the two
// halves of row l of both blocks.
template <int KSTEPS>
__device__ inline int32_t half_row_sq(const Operand& o) {
  int32_t acc = 0;
#pragma unroll
  for (int s = 0; s < KSTEPS; ++s)
#pragma unroll
    for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_sdot4(o.k[s][i], o.k[s][i], acc, false);
  return acc;
}
// `two`: block 1 holds samples (uniform).
template <int KSTEPS>
__device__ inline int32_t sample_norm(const Operand& b0, const Operand& b1, bool two, int half,
                                      int lane) {
  const int32_t p0 = half_row_sq<KSTEPS>(b0);
  int32_t p1 = 0;
  if (two) p1 = half_row_sq<KSTEPS>(b1);
  const int32_t mine = half ? p1 : p0, give = half ? p0 : p1;
  return mine + (int32_t)xor_lanes((uint32_t)give, 32, lane);
}

// Two ways to treat the thresholds of the lists.  Either the (threshold, norm) record of every
// sampled object is gathered, 8 bytes but one more scattered line each, and a result that cannot
// enter its list is dropped here; or neither is read: norms come from the operand registers (up to
// 64 dot products per node), every result found is handed on, and what cannot enter is dropped one
// pass later.  Staged, that pass is k_result_csr, which has the thresholds of its bucket in LDS, so
// the same results reach the lists.  The rows and records of 45 million samples per iteration are
// asked for at about the rate the memory system serves scattered lines, so records that decide little
// are better not read: 10^6 x 128, iterations 2 to 5, 69 to 93 % of the results pass, join and
// k_result_csr 8.25 -> 7.4 ms, build 23.7 -> 22.9 ms; 200,000 x 96 bytes, k = 96, 5.36 -> 5.21 ms.
// Where fewer pass, what more there is to sort costs as much: with records for no iteration the
// sharded build of 4 x 600,000 takes 176 to 178 ms instead of 174.  So they are read where less than
// two thirds of the results of the iteration before passed (half: 176 ms; four fifths: 10^6 x 128 23.5
// ms), which begin_iteration decides on the device, and wherever worth_leaving_out() says so; never in
// the first iteration on a random graph, where everything passes.
// A result that goes to its bucket's region directly is held against its threshold first: those that do
// not pass are mostly for the same few destinations, and one atomic each for them costs more than the
// records save (the merge and the build above, with early flushes, without / with this look 14.2 /
// 12.6 and 190 / 116 ms; with neither 39.0 and 295, or 21.3 and 185 with the records in every iteration).
// Direct hand-out: LEAN, the launch of that first iteration; what cannot enter is left to the update.
//
// Calls in which the records are left out where most results pass.  The more nodes and the longer
// their lists, the less of the records and lists stands in the caches, and the more the records cost.
// Time by the rule above over that with the records in every iteration but a random graph's first, whole
// builds of 4 and 8 iterations and merges of 2 and 5 on rows of 32 and 128 bytes:
//   k = p = 32: 262,144 nodes 1.02 to 1.03, 400,000 1.01 to 1.02, 700,000 0.96 to 1.01, 10^6 0.94 to 1.00
//   k = 64, p = 32: 200,000 nodes 1.02 to 1.04, 262,144 0.99 to 1.01, 10^6 0.88 to 0.95
//   k = 96, p = 32: 200,000 nodes 1.01 to 1.02, 262,144 0.98 to 1.00, 10^6 0.86 to 0.94
//   p = 8 1.02 to 1.06 everywhere; k = 12 to 20, p <= k, up to 2 million nodes 0.97 to 1.05
//   3.5 million (k_result_csr reads every bucket four times) 0.99 to 1.08
//   merges, k = p = 32: 2 x 150,000 nodes 0.99 to 1.03, 2 x 250,000 0.93 to 0.98, 300,000 + 150,000 0.95 to
//   1.01, 2 x 700,000 0.85 to 0.95; k = 64: 2 x 100,000 0.98 to 1.02, 2 x 150,000 0.95 to 1.00
//   merges with a set of less than half the other's size: 300,000 + 30,000 1.08 to 1.19, 250,000 + 90,000
//   1.01 to 1.06
// and on rows of 96 bytes, every second of which lies in two lines, so that the rows fill more of the
// caches and of the line rate:
//   k = p = 32: 200,000 nodes 1.00 to 1.01, 262,144 0.98 to 0.99, 700,000 0.96; k = 64, p = 32: 140,000
//   1.01 to 1.03, 200,000 0.96 to 0.98; k = 96, p = 32: 140,000 0.99 to 1.01, 200,000 0.96 to 0.97
//   merges, k = p = 32: 2 x 100,000 nodes 0.96 to 1.00, 2 x 150,000 0.93 to 0.97
static bool worth_leaving_out(const Shape& sh, bool merge) {
  const int64_t entries = sh.n * (sh.k < 64 ? sh.k : 64) * (sh.d > 64 && sh.d <= 96 ? 2 : 1);
  const int64_t smaller = sh.split < sh.n - sh.split ? sh.split : sh.n - sh.split;  // (a merge's sets)
  return sh.p > 8 && sh.n <= (1 << 21) &&
         (merge ? entries >= 3 << 22 && 3 * smaller >= sh.n : entries >= 1 << 24 && sh.k > 24);
}

// Between nodes a wavefront keeps as little as it can waiting for memory: nothing that is in
// flight is moved or overwritten (see the loop), the search for objects in both lists runs before
// the rows are needed, counts stay in registers until the end, and the terms a diagonal tile hides
// are read from a place of their own instead of being masked.  Registers of absent samples are not
// cleared either, which with 32-bit offsets brought the form for any node from 173 to 152 registers,
// so that it runs 3 wavefronts per SIMD like the forms for nodes with at most 32 OLD or at most 32 NEW
// samples that stood beside it: those, the lists of nodes per form and the launch that made them are
// gone, and a wavefront walks over all nodes.  Iterations of 10^6 x 128 on average 1724 -> 1540 us,
// 200,000 x 96 bytes with full lists 670 -> 605 us, the first iteration 1530 -> 1415 us.
template <int KSTEPS, bool FCODE, bool MERGE, bool STAGED, bool LEAN = false>
__global__ __launch_bounds__(STAGED ? kStagedWaves * kWave : kMB)
__attribute__((amdgpu_waves_per_eu(3, 3))) void k_join_mfma(
    const int8_t* __restrict__ shadow, const NodeMeta* __restrict__ meta, int64_t n,
    int p, int64_t split, const int32_t* __restrict__ snew, const int32_t* __restrict__ sold,
    uint64_t* pslot, uint64_t slots, uint64_t* __restrict__ bins, uint64_t* counters,
    StageArgs sa) {
  constexpr int WAVES = STAGED ? kStagedWaves : kMB / kWave;
  static_assert(!(STAGED && LEAN), "the staged form looks at StageArgs::all");
  const bool lean = STAGED ? sa.all && *sa.all != 0ull : LEAN;
  // per wave, for the 128 rows (NEW 0..63, OLD 64..127): -((norm << 6) | position), the ids
  // (absent = INT_MAX so that both halves stay ascending), and what a NEW sample's own column of
  // the diagonal tiles reads instead (see own_rows); the last first serves the search for objects
  // in both lists
  __shared__ __attribute__((aligned(16))) int32_t s_lists[WAVES][512];
  extern __shared__ __attribute__((aligned(16))) unsigned char stage_raw[];
  uint64_t* const st_ent = reinterpret_cast<uint64_t*>(stage_raw);
  uint64_t* const st_region = st_ent + kStageBuckets * kStageSlots;
  uint32_t* const st_cnt = reinterpret_cast<uint32_t*>(st_region + kStageBuckets);
  uint32_t* const st_fill = st_cnt + kStageBuckets;  // [0] results staged, [1] waves out of nodes
  // (the wave index as a vector value: measured 3 % faster here than the scalar form)
  const int wave = threadIdx.x >> 6, lane = lane_id(), half = lane >> 5, col = lane & 31;
  int32_t* const s_norm = s_lists[wave];
  int32_t* const s_id = s_norm + 128;
  int32_t* const s_own = s_norm + 256;
  // (staged n <= 2^22: node numbers and offsets into the sample lists fit 32 bits, and
  // so do the byte offsets of everything that is gathered)
  using node_t = typename std::conditional<STAGED, int32_t, int64_t>::type;
  using offset_t = typename std::conditional<STAGED, uint32_t, int64_t>::type;
  auto at_offset = [](const void* base, offset_t bytes) {
    return static_cast<const char*>(base) + bytes;
  };
  const node_t W = (node_t)gridDim.x * WAVES;
  const node_t nodes = (node_t)n;
  node_t s = (node_t)blockIdx.x * WAVES + wave;
  if (!STAGED && s >= nodes) return;
  if (STAGED) {
    for (int b = threadIdx.x; b < sa.nb; b += WAVES * kWave) {
      st_cnt[b] = 0;
      const int64_t first = (int64_t)b << sa.tb;
      st_region[b] = sa.poff[first < n ? first : n];
    }
    if (threadIdx.x == 0) st_fill[0] = st_fill[1] = 0;
    __syncthreads();
  }
  // One flush (all waves of the workgroup together).  Returns true when every wave has
  // run out of nodes, i.e. when this was the last one.  A wave sees to a run of neighbouring
  // buckets: each of its lanes claims the places of one (neighbouring counters: with a wave's
  // buckets spread out instead the joins took 10 to 35 % longer), and then the results of one
  // after the other leave as one contiguous piece each.
  auto flush = [&]() -> bool {
    __syncthreads();  // nobody is adding results any more
    const uint32_t out_of_nodes = st_fill[1];
    if (threadIdx.x == 0) st_fill[0] = 0;
    const int per = (sa.nb + WAVES - 1) / WAVES, first = wave_id() * per;
    const int last = vmin(first + per, sa.nb), own = first + lane;
    uint32_t c = 0;
    uint64_t at = 0;
    if (own < last) {
      c = vmin(st_cnt[own], (uint32_t)kStageSlots);
      st_cnt[own] = 0;
      if (c) at = st_region[own] + atomicAdd(&sa.cur[own], (unsigned long long)c);
    }
    for (int i0 = 0; first + i0 < last; i0 += 4) {
      uint64_t rec[4];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        rec[j] = st_ent[vmin(first + i0 + j, sa.nb - 1) * kStageSlots + lane];
#pragma unroll
      for (int j = 0; j < 4; ++j) {  // (lanes beyond the buckets hold no results)
        const uint32_t count = (uint32_t)__builtin_amdgcn_readlane((int)c, i0 + j);
        const uint64_t to = readlane64(at, i0 + j) + (uint32_t)lane;
        if ((uint32_t)lane < count && to < slots) sa.ent[to] = rec[j];
      }
    }
    __syncthreads();
    return out_of_nodes == (uint32_t)WAVES;
  };
  // The sample ids of the next node are on their way while one is worked on.  What is requested goes to
  // its registers without any branch or default, and is looked at no sooner than a whole node
  // later: a register that is written or moved while its load is out would make the wavefront
  // wait for everything it has requested.
  const int L = 2 * p, at_list = lane < L ? lane : L - 1;
  // (beyond the last node: any node's ids, unused)
  auto sample_of = [&](const int32_t* lists, node_t node) {
    return *reinterpret_cast<const int32_t*>(at_offset(
        lists, ((offset_t)vmin(node, (node_t)(nodes - 1)) * (offset_t)L + (offset_t)at_list) * 4));
  };
  // s counts the nodes; the node of place s is s itself or, staged, s * spread mod n (see StageArgs)
  node_t node = STAGED ? (node_t)((uint64_t)s * sa.spread % (uint64_t)n) : s;
  auto next_node = [&]() {
    node += STAGED ? (node_t)sa.stride : W;
    if (STAGED && node >= nodes) node -= nodes;
  };
  // unused list slots hold -1, so the ids alone say how long a list is
  int32_t id_new = sample_of(snew, node), id_old = sample_of(sold, node);
  next_node();
  int32_t nx_new = sample_of(snew, node), nx_old = sample_of(sold, node);
  if (lane >= L) id_new = id_old = -1;
  // Block b of a list = its rows 32b..32b+31; lane (col, half) holds bytes [32 step + 16 half, +16)
  // of row `col` of the block for every step.  Registers of absent samples keep whatever they held:
  // absent rows are kept out of every result by their norm (far_enough: G does not bring kFar down
  // to a real distance), absent columns have no result.
  Operand N0{}, N1{}, O0{}, O1{};
  uint2 m_new = make_uint2(0u, 0u), m_old = m_new;  // list threshold and norm
  auto load_rows = [&](Operand& o, uint32_t id) {
    if ((int32_t)id < 0) return;
    const char* const row = at_offset(shadow, (STAGED ? (offset_t)__umul24(id, 32 * KSTEPS)
                                                      : (offset_t)id * (32 * KSTEPS)) +
                                                  (offset_t)(16 * half));
#pragma unroll
    for (int k = 0; k < KSTEPS; ++k) o.k[k] = *reinterpret_cast<const v4i*>(row + 32 * k);
  };
  auto request_rows = [&](int32_t idn, int32_t ido) {
    if (!lean) {  // one 8-byte gather per sampled object (an absent one: object 0, unused)
      m_new = *reinterpret_cast<const uint2*>(at_offset(meta, (offset_t)vmax(idn, 0) * 8));
      m_old = *reinterpret_cast<const uint2*>(at_offset(meta, (offset_t)vmax(ido, 0) * 8));
    }
    uint32_t i0, i1;
    pair_lanes((uint32_t)idn, 32, i0, i1);
    load_rows(N0, i0);
    load_rows(N1, i1);
    pair_lanes((uint32_t)ido, 32, i0, i1);
    load_rows(O0, i0);
    load_rows(O1, i1);
  };
  // how many samples the node has, and whether it has anything to evaluate; if not, nothing is read
  int nn = 0, no = 0;
  bool do_nn = false, active = false;
  auto begin_node = [&]() {
    nn = __popcll(__ballot(id_new >= 0));
    no = __popcll(__ballot(id_old >= 0));
    do_nn = !MERGE && nn > 1;
    active = nn > 0 && (do_nn || no > 0);
    if (active) request_rows(id_new, id_old);
  };
  if (s < nodes) begin_node();

  // The diagonal tiles of NEW x NEW pair every object with itself.  Row `col` of a tile stands in
  // one group of four rows, which the lane (col, half) that holds them reads from s_own, where its
  // own row is as far as an absent one: nothing is masked element by element.
  int own_rows[4];  // where this lane finds the terms of its four groups of rows
#pragma unroll
  for (int q = 0; q < 4; ++q)
    own_rows[q] = q == (col >> 3) && half == ((col >> 2) & 1)
                      ? 256 + 64 * (col >> 3) + 4 * (col & 7)
                      : 8 * q + 4 * half;
  const int own_at = 64 * ((lane & 31) >> 3) + 32 * half + 4 * (lane & 7);

  // what this wavefront has counted over its nodes (below 2^32: a node has at most 6112 pairs)
  uint32_t all_found = 0, all_passed = 0, all_evals = 0, over = 0;

  while (s < nodes) {
    // What needs the ids only is done while the rows are on their way.
    s_id[lane] = id_new >= 0 ? id_new : 0x7fffffff;
    s_id[64 + lane] = id_old >= 0 ? id_old : 0x7fffffff;
    // objects sampled both as NEW and as OLD: that pair is not a pair.  eq_old =
    // position in the OLD list of this lane's NEW object (or -1), and vice versa.
    // Both lists ascend, so each NEW lane binary-searches its id in the OLD list.
    int eq_old = -1, eq_new = -1;
    uint32_t dups = 0;
    if (active && no > 0) {
      wave_lds_fence();
      const int32_t* at = s_id + 64;
#pragma unroll
      for (int step = 32; step > 0; step >>= 1) at = at[step - 1] < id_new ? at + step : at;
      if (*at == id_new) eq_old = (int)(at - (s_id + 64));
      dups = (uint32_t)__popcll(__ballot(eq_old >= 0));
      if (dups) {
        s_own[lane] = -1;
        wave_lds_fence();
        if (eq_old >= 0) s_own[eq_old] = lane;
        wave_lds_fence();
        eq_new = s_own[lane];
        wave_lds_fence();
      }
    }
    // per-lane exclusion masks (bit r = row r of the block is not a partner of
    // this lane's column object); lanes l and l+32 serve column l%32 of block 0,
    // results of block 1 are selected into lanes 32..63 at the end
    const bool masked_no = MERGE || dups != 0;
    uint32_t eq_old_c[2] = {~0u, ~0u}, eq_new_c[2] = {~0u, ~0u};
    uint32_t cls_new[2] = {0u, 0u}, cls_old[2] = {0u, 0u};
    uint32_t id_new_c[2] = {0u, 0u}, id_old_c[2] = {0u, 0u};
    if (masked_no) {
      pair_lanes((uint32_t)eq_old, 32, eq_old_c[0], eq_old_c[1]);
      pair_lanes((uint32_t)eq_new, 32, eq_new_c[0], eq_new_c[1]);
    }
    // merge mode: rows whose set equals the column object's set are excluded
    if (MERGE) {
      const uint64_t cn = __ballot(id_new >= 0 && (int64_t)id_new >= split);
      const uint64_t co = __ballot(id_old >= 0 && (int64_t)id_old >= split);
      cls_new[0] = (uint32_t)cn; cls_new[1] = (uint32_t)(cn >> 32);
      cls_old[0] = (uint32_t)co; cls_old[1] = (uint32_t)(co >> 32);
      pair_lanes((uint32_t)id_new, 32, id_new_c[0], id_new_c[1]);
      pair_lanes((uint32_t)id_old, 32, id_old_c[0], id_old_c[1]);
    }
    auto excl_rows = [&](uint32_t eq_row, int row_block, uint32_t cls_rows, uint32_t col_id) {
      uint32_t m = 0;
      if ((eq_row >> 5) == (uint32_t)row_block) m |= 1u << (eq_row & 31);  // (none: ~0)
      if (MERGE) m |= ((int64_t)(int32_t)col_id >= split) ? cls_rows : ~cls_rows;
      return m;
    };

    uint2 cm_new = m_new, cm_old = m_old;  // this node's thresholds and norms
    if (lean && active) {  // (all lanes take part in the exchange between the halves)
      cm_new.y = (uint32_t)sample_norm<KSTEPS>(N0, N1, nn > 32, half, lane);
      if (no > 0)  // uniform
        cm_old.y = (uint32_t)sample_norm<KSTEPS>(O0, O1, no > 32, half, lane);
    }
    if (id_new < 0) cm_new.y = (uint32_t)kFar;  // an absent sample: far from everything
    if (id_old < 0) cm_old.y = (uint32_t)kFar;
    int32_t a0 = kNone, a1 = kNone;  // NEW column blocks: nearest other NEW
    int32_t b0 = kNone, b1 = kNone;  // NEW column blocks: nearest OLD
    int32_t c0 = kNone, c1 = kNone;  // OLD column blocks: nearest NEW
    if (active) {
      const int32_t neg_new = -(int32_t)((cm_new.y << 6) | (uint32_t)lane);
      s_norm[lane] = neg_new;
      s_norm[64 + lane] = -(int32_t)((cm_old.y << 6) | (uint32_t)lane);
      if (do_nn) {
        // the terms of the four samples of this lane's quad, its own as far as an absent one
        const int32_t far = -(int32_t)(((uint32_t)kFar << 6) | (uint32_t)lane);
        const int i = lane & 3;
        int4 quad;  // (all lanes take part in the exchange)
        quad.x = __builtin_amdgcn_mov_dpp(neg_new, 0x00, 0xF, 0xF, true);
        quad.y = __builtin_amdgcn_mov_dpp(neg_new, 0x55, 0xF, 0xF, true);
        quad.z = __builtin_amdgcn_mov_dpp(neg_new, 0xAA, 0xF, 0xF, true);
        quad.w = __builtin_amdgcn_mov_dpp(neg_new, 0xFF, 0xF, 0xF, true);
        quad.x = i == 0 ? far : quad.x;
        quad.y = i == 1 ? far : quad.y;
        quad.z = i == 2 ? far : quad.z;
        quad.w = i == 3 ? far : quad.w;
        *reinterpret_cast<int4*>(s_own + own_at) = quad;
      }
      // the wave reads these back below: order its own LDS writes before its reads
      wave_lds_fence();
      const int32_t* normN = s_norm;
      const int32_t* normO = s_norm + 64;

      if (do_nn) {
        {  // rows N0, columns N0
          v16i g = gram<KSTEPS>(N0, N0);
          a0 = max(a0, tile_col_best_at(g, normN, own_rows));
        }
        if (nn > 32) {
          {
            v16i g = gram<KSTEPS>(N1, N0);
            a0 = max(a0, tile_col_best<false>(g, normN + 32, half, 0u));
          }
          {
            v16i g = gram<KSTEPS>(N0, N1);
            a1 = max(a1, tile_col_best<false>(g, normN, half, 0u));
          }
          {
            v16i g = gram<KSTEPS>(N1, N1);
            a1 = max(a1, tile_col_best_at(g, normN + 32, own_rows));
          }
        }
      }
      // one tile of NEW x OLD, columns = objects of one list, rows = a block of the other
      auto cross = [&](const Operand& rows, const Operand& cols, const int32_t* norms, uint32_t eq,
                       int row_block, uint32_t cls_rows, uint32_t col_id) {
        const v16i g = gram<KSTEPS>(rows, cols);
        // (few tiles hold an object of both lists)
        const uint32_t skip = masked_no ? excl_rows(eq, row_block, cls_rows, col_id) : 0u;
        return __ballot(skip != 0u) ? tile_col_best<true>(g, norms, half, skip)
                                    : tile_col_best<false>(g, norms, half, 0u);
      };
      if (no > 0) {
        // columns = NEW objects, rows = OLD objects: nearest OLD of every NEW
        b0 = max(b0, cross(O0, N0, normO, eq_old_c[0], 0, cls_old[0], id_new_c[0]));
        if (no > 32)
          b0 = max(b0, cross(O1, N0, normO + 32, eq_old_c[0], 1, cls_old[1], id_new_c[0]));
        if (nn > 32) {
          b1 = max(b1, cross(O0, N1, normO, eq_old_c[1], 0, cls_old[0], id_new_c[1]));
          if (no > 32)
            b1 = max(b1, cross(O1, N1, normO + 32, eq_old_c[1], 1, cls_old[1], id_new_c[1]));
        }
        // columns = OLD objects, rows = NEW objects: nearest NEW of every OLD
        c0 = max(c0, cross(N0, O0, normN, eq_new_c[0], 0, cls_new[0], id_old_c[0]));
        if (nn > 32)
          c0 = max(c0, cross(N1, O0, normN + 32, eq_new_c[0], 1, cls_new[1], id_old_c[0]));
        if (no > 32) {
          c1 = max(c1, cross(N0, O1, normN, eq_new_c[1], 0, cls_new[0], id_old_c[1]));
          if (nn > 32)
            c1 = max(c1, cross(N1, O1, normN + 32, eq_new_c[1], 1, cls_new[1], id_old_c[1]));
        }
      }
    }

    // ---- hand the results out: lane l answers for sample l of its list -------
    bool pass[3] = {false, false, false};
    uint64_t entry[3];
    if (active) {
      // combine the two row halves; lanes 0..31 take column block 0, lanes 32..63 block 1
      const int32_t res3[3] = {blocks_max(a0, a1), blocks_max(b0, b1), blocks_max(c0, c1)};
#pragma unroll
      for (int kind = 0; kind < 3; ++kind) {
        const int32_t res = -res3[kind];  // ((row_norm - 2 G) << 6) | row position
        const int32_t self = kind == 2 ? id_old : id_new;
        const uint2 cm = kind == 2 ? cm_old : cm_new;
        const int32_t part = res >> 6;  // arithmetic shift; absent rows sit at kFar
        const bool found = self >= 0 && res3[kind] != kNone && part < (kFar >> 1);
        const int32_t dist = part + (int32_t)cm.y;
        const int32_t other = s_id[(kind == 1 ? 64 : 0) + (res & 63)];
        const uint32_t code = FCODE ? ord_f32((float)dist) : ord_i32(dist);
        // a result that cannot beat the last entry of the destination list is dropped
        pass[kind] = found && (lean || code <= cm.x);
        entry[kind] = STAGED ? stage_entry(dist, (uint32_t)other)
                             : make_entry(code, (uint32_t)other, 3u);
        all_found += (uint32_t)__popcll(__ballot(found));
      }
      if (MERGE) {
        const uint32_t n1 = (uint32_t)(__popc(cls_new[0]) + __popc(cls_new[1]));
        const uint32_t o1 = (uint32_t)(__popc(cls_old[0]) + __popc(cls_old[1]));
        all_evals += n1 * ((uint32_t)no - o1) + ((uint32_t)nn - n1) * o1;
      } else {
        all_evals += (uint32_t)(nn * no) - dups;
        if (do_nn) all_evals += (uint32_t)(nn * (nn - 1)) >> 1;
      }
    }
    // slot requests for all three results first ...
    // (the two results of a NEW sample go to the same list: one request for both)
    const uint32_t want_n = (pass[0] ? 1u : 0u) + (pass[1] ? 1u : 0u);
    const uint32_t passed =
        (uint32_t)__popcll(__ballot(pass[0])) + (uint32_t)__popcll(__ballot(pass[1])) +
        (uint32_t)__popcll(__ballot(pass[2]));
    all_passed += passed;
    uint64_t word_n = 0, word_o = 0;  // direct hand-out: slot words of the destinations
    uint32_t place_n = 0, place_o = 0;  // staged hand-out: places in the buckets' LDS areas
    uint32_t fill = 0;                  // results in the staging area, with this node's
    const int bucket_n = STAGED ? (int)((uint32_t)id_new >> sa.tb) : 0;
    const int bucket_o = STAGED ? (int)((uint32_t)id_old >> sa.tb) : 0;
    if (STAGED) {
      if (want_n) place_n = atomicAdd(&st_cnt[bucket_n], want_n);
      if (pass[2]) place_o = atomicAdd(&st_cnt[bucket_o], 1u);
      if (lane == 0) fill = atomicAdd(&st_fill[0], passed) + passed;
      // (the one result that takes a bucket's place number kStageSoon asks)
      if ((place_n < kStageSoon && place_n + want_n >= kStageSoon) ||
          (pass[2] && place_o == kStageSoon - 1))
        atomicAdd(&st_fill[0], sa.threshold);
    } else {
      // one returning add on the destination's slot word yields the segment start
      // and the place in it
      if (want_n)
        word_n = atomicAdd(reinterpret_cast<unsigned long long*>(&pslot[id_new]),
                           (unsigned long long)want_n);
      if (pass[2])
        word_o = atomicAdd(reinterpret_cast<unsigned long long*>(&pslot[id_old]), 1ull);
    }
    // staged: places in LDS come back at once, so the results are put away before the
    // next node's rows take up the operand registers
    // (segments and bucket regions cannot overflow, see the sampling stage; the tests
    // against the array size only keep a violated bound from writing outside the array)
    if (STAGED) {
      auto put = [&](int bucket, uint32_t place, uint64_t e, int32_t dest) {
        const uint64_t rec = stage_record(e, (uint32_t)dest, sa.tb);
        if (place < (uint32_t)kStageSlots) {
          st_ent[bucket * kStageSlots + (int)place] = rec;
        } else {  // the bucket's places are taken: straight to its region
          if (lean && stage_code<FCODE>(e) > meta[dest].kth) return;  // (see worth_leaving_out)
          const uint64_t at = st_region[bucket] + atomicAdd(&sa.cur[bucket], 1ull);
          if (at < slots) sa.ent[at] = rec;
          else ++over;
        }
      };
      if (pass[0]) put(bucket_n, place_n, entry[0], id_new);
      if (pass[1]) put(bucket_n, place_n + (pass[0] ? 1u : 0u), entry[1], id_new);
      if (pass[2]) put(bucket_o, place_o, entry[2], id_old);
    }
    // direct: with the operand registers free, the next node's rows are requested while
    // the slot words are still on their way ...
    const bool more = s + W < nodes;
    if (more) {
      id_new = lane < L ? nx_new : -1;
      id_old = lane < L ? nx_old : -1;
      begin_node();
      next_node();
      nx_new = sample_of(snew, node);
      nx_old = sample_of(sold, node);
    }
    // ... and only now the slots are used
    if (!STAGED) {
      const uint64_t at_n = (word_n >> kSlotCountBits) + (word_n & kSlotCountMask);
      const uint64_t at_o = (word_o >> kSlotCountBits) + (word_o & kSlotCountMask);
      if (pass[0] && pass[1]) {  // neighbouring slots: one 16-byte store
        if (at_n + 1 < slots)
          __builtin_nontemporal_store(EntryPair{entry[0], entry[1]}, reinterpret_cast<EntryPair*>(bins + at_n));
        else over += 2;
      } else if (want_n) {
        if (at_n < slots) __builtin_nontemporal_store(pass[0] ? entry[0] : entry[1], &bins[at_n]);
        else ++over;
      }
      if (pass[2]) {
        if (at_o < slots) __builtin_nontemporal_store(entry[2], &bins[at_o]);
        else ++over;
      }
    }
    // every wave looks at the fill count after every node
    if (STAGED && (uint32_t)__builtin_amdgcn_readfirstlane((int)fill) >= sa.threshold) (void)flush();
    if (!more) break;
    s += W;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) over += __shfl_xor(over, off, kWave);
  if (lane == 0) {
    unsigned long long* cs = reinterpret_cast<unsigned long long*>(
        counters + ((blockIdx.x * WAVES + wave) & (kStripes - 1)) * C_SLOTS);
    // (staged, every result handed on: k_result_csr counts what passes the thresholds)
    if (!(STAGED && lean) && all_passed) atomicAdd(cs + C_PASSED, (unsigned long long)all_passed);
    if (all_found) atomicAdd(cs + C_PROPS, (unsigned long long)all_found);
    if (over) atomicAdd(cs + C_OVERFLOW, (unsigned long long)over);
    if (all_evals) atomicAdd(cs + C_EVALS, (unsigned long long)all_evals);
  }
  if (STAGED) {
    if (lane == 0) atomicAdd(&st_fill[1], 1u);
    while (!flush()) {
    }
  }
}

// Second half of the staged hand-out: one workgroup per bucket moves the bucket's
// results from its region into the segments of their destinations and writes the
// destinations' slot words (segment start, results received) that the list update reads.
// The results arrive in no order, and 8-byte stores to scattered places are served at a
// fixed rate whatever their number per line; so the workgroup takes the region in tiles,
// puts every tile in destination order inside LDS (counting sort: an LDS counter per
// destination gives each result its rank, a scan of the counters the start of each
// destination's run) and writes it out run by run: neighbouring lanes then store to
// neighbouring places.
constexpr int kRcBlock = 1024;
// `all` (FILTER; see StageArgs): where the join has handed on every result, those that cannot beat the
// last entry of their destination's list are dropped here, and what is left is counted as passed.
// Results per thread and tile: 12 (96 KB of LDS), 11 where the thresholds need room too.
constexpr int rc_per_thread(bool filter) { return filter ? 11 : 12; }
// A bucket of more than 2^kRcBits destinations (more than 2^20 nodes) is worked on by several
// workgroups, each of which reads all of the bucket's results and keeps those for its part.
constexpr int kRcBits = 12;
// LDS: the tile, then per destination of the bucket or part (at most 2^12) the number of results in
// the tile / the start of its run, the next free place of its segment, the segment's end
// (both relative to the region) and, with FILTER, the threshold of its list.
static size_t result_csr_lds_bytes(int tb, bool filter) {
  return (size_t)kRcBlock * rc_per_thread(filter) * 8 + (((size_t)(filter ? 4 : 3) << tb) + 1) * 4;
}

template <bool FILTER, bool FCODE>
__global__ __launch_bounds__(kRcBlock) void k_result_csr(int64_t n, int bucket_tb,
                                                         const uint64_t* __restrict__ poff,
                                                         const unsigned long long* __restrict__ cur,
                                                         const uint64_t* __restrict__ ent,
                                                         uint64_t* __restrict__ bins,
                                                         uint64_t* __restrict__ pslot,
                                                         const NodeMeta* __restrict__ meta,
                                                         uint64_t* counters, const uint64_t* all) {
  constexpr int kRcPerThread = rc_per_thread(FILTER), kRcTile = kRcBlock * kRcPerThread;
  const bool filter = FILTER && *all != 0ull;
  extern __shared__ __attribute__((aligned(16))) uint64_t rc_lds[];
  __shared__ uint32_t part[kRcBlock / kWave];
  uint64_t* const tile = rc_lds;
  const int tb = bucket_tb < kRcBits ? bucket_tb : kRcBits, parts = 1 << (bucket_tb - tb);
  const int T_max = 1 << tb;
  uint32_t* const run = reinterpret_cast<uint32_t*>(rc_lds + kRcTile);  // T_max + 1 entries
  uint32_t* const next = run + T_max + 1;
  uint32_t* const seg_end = next + T_max;
  uint32_t* const kth_s = seg_end + T_max;  // FILTER only
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int bucket = blockIdx.x / parts, part_of = blockIdx.x % parts;
  const int64_t bucket_first = (int64_t)bucket << bucket_tb, first = bucket_first + part_of * T_max;
  if (first >= n) return;
  const int64_t bucket_end =
      bucket_first + (1ll << bucket_tb) < n ? bucket_first + (1ll << bucket_tb) : n;
  const int T = (int)(n - first < (int64_t)T_max ? n - first : (int64_t)T_max);
  const uint64_t region = poff[bucket_first], room = poff[bucket_end] - region;
  // destination inside this part (T or more: none of this part's), and the distance's code
  auto place_of = [&](uint64_t x) {
    const uint32_t in_bucket =
        (uint32_t)(x >> kStageIdBits) & ((1u << (kStageDistShift - kStageIdBits)) - 1u);
    return in_bucket - (uint32_t)(part_of * T_max);
  };
  auto code_of = [](uint64_t x) { return stage_code<FCODE>(x); };
  for (int t = tid; t < T_max; t += kRcBlock) {
    next[t] = t < T ? (uint32_t)(poff[first + t] - region) : (uint32_t)room;
    seg_end[t] = t < T ? (uint32_t)(poff[first + t + 1] - region) : (uint32_t)room;
    if (filter) kth_s[t] = t < T ? meta[first + t].kth : 0u;
  }
  uint32_t kept = 0;  // results that pass
  uint64_t count = cur[bucket];
  if (count > room) {  // cannot happen: a region holds what its destinations can receive
    if (tid == 0 && part_of == 0)
      atomicAdd(reinterpret_cast<unsigned long long*>(counters + C_OVERFLOW),
                (unsigned long long)(count - room));
    count = room;
  }
  const int per = (T_max + kRcBlock - 1) / kRcBlock;  // counters per thread in the scan (<= 4)
  for (uint64_t base = 0; base < count; base += kRcTile) {
    for (int t = tid; t <= T_max; t += kRcBlock) run[t] = 0;
    __syncthreads();
    // rank of every result among the tile's results for the same destination
    uint64_t e[kRcPerThread];
    uint32_t rank[kRcPerThread];
#pragma unroll
    for (int r = 0; r < kRcPerThread; ++r) {
      const uint64_t i = base + (uint64_t)r * kRcBlock + tid;
      e[r] = i < count ? ent[region + i] : ~0ull;
    }
#pragma unroll
    for (int r = 0; r < kRcPerThread; ++r) {
      const uint32_t t = place_of(e[r]);
      if (e[r] == ~0ull || t >= (uint32_t)T || (filter && code_of(e[r]) > kth_s[t])) {
        e[r] = ~0ull;
      } else {
        rank[r] = atomicAdd(&run[t], 1u);
        ++kept;
      }
    }
    __syncthreads();
    // exclusive scan of the counters: thread i takes counters per*i .. per*i + per - 1
    uint32_t mine[4], sum = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int t = tid * per + j;
      mine[j] = (j < per && t < T_max) ? run[t] : 0u;
      sum += mine[j];
    }
    uint32_t inc = sum;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
      const uint32_t o = __shfl_up(inc, off, kWave);
      if (lane >= off) inc += o;
    }
    if (lane == kWave - 1) part[wave] = inc;
    __syncthreads();
    uint32_t before = 0;
    for (int w = 0; w < wave; ++w) before += part[w];
    uint32_t at = before + inc - sum;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int t = tid * per + j;
      if (j < per && t < T_max) run[t] = at;
      at += mine[j];
    }
    if (tid == kRcBlock - 1) run[T_max] = at;  // results in the tile
    __syncthreads();
    // the tile in destination order
#pragma unroll
    for (int r = 0; r < kRcPerThread; ++r) {
      if (e[r] != ~0ull) {
        const uint32_t t = place_of(e[r]);
        tile[run[t] + rank[r]] = e[r];
      }
    }
    __syncthreads();
    const uint32_t in_tile = run[T_max];
#pragma unroll
    for (int r = 0; r < kRcPerThread; ++r) {
      const uint32_t j = (uint32_t)r * kRcBlock + tid;
      if (j < in_tile) {
        const uint64_t x = tile[j];
        const uint32_t t = place_of(x);
        const uint32_t place = next[t] + (j - run[t]);
        // back to a list entry: distance code | object id | "admitted now" + NEW
        if (place < seg_end[t])
          bins[region + place] =
              make_entry(code_of(x), (uint32_t)x & ((1u << kStageIdBits) - 1u), 3u);
      }
    }
    __syncthreads();
    for (int t = tid; t < T; t += kRcBlock) next[t] += run[t + 1] - run[t];
    __syncthreads();
  }
  __syncthreads();
  if (filter) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) kept += __shfl_xor(kept, off, kWave);
    if (lane == 0 && kept)
      atomicAdd(reinterpret_cast<unsigned long long*>(
                    counters +
                    ((blockIdx.x * (kRcBlock / kWave) + wave) & (kStripes - 1)) * C_SLOTS + C_PASSED),
                (unsigned long long)kept);
  }
  for (int t = tid; t < T; t += kRcBlock) {
    const uint64_t start = poff[first + t] - region;
    const uint64_t end = next[t] < seg_end[t] ? next[t] : seg_end[t];
    const uint64_t got = end - start < kSlotCountMask ? end - start : kSlotCountMask;
    pslot[first + t] = ((region + start) << kSlotCountBits) | got;
  }
}

template <int KSTEPS, bool STAGED, bool LEAN = false>
static hipError_t launch_k(bool fcode, bool merge, unsigned grid, hipStream_t st,
                           const int8_t* shadow, const NodeMeta* meta, const Shape& sh,
                           const DevState& ds, const StageArgs& sa) {
  constexpr int block = STAGED ? kStagedWaves * kWave : kMB;
  const size_t lds = STAGED ? kStageLdsBytes : 0;
#define GNND_ARGS shadow, meta, sh.n, sh.p, sh.split, ds.snew, ds.sold, \
                  ds.pslot, (uint64_t)sh.slots(), ds.bins, ds.counters, sa
#define GNND_LAUNCH(F, M)                                                                      \
  do {                                                                                         \
    auto* kern = k_join_mfma<KSTEPS, F, M, STAGED, LEAN>;                                      \
    if (STAGED) {                                                                              \
      static bool attr_set = false; /* per instantiation: a staging area beyond the default */ \
      if (!attr_set) {                                                                         \
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),                \
                                           hipFuncAttributeMaxDynamicSharedMemorySize,         \
                                           (int)kStageLdsBytes);                               \
        if (e != hipSuccess) return e;                                                         \
        attr_set = true;                                                                       \
      }                                                                                        \
    }                                                                                          \
    kern<<<grid, block, lds, st>>>(GNND_ARGS);                                                 \
  } while (0)
  if (LEAN) {  // never with a merge
    if (fcode) GNND_LAUNCH(true, false);
    else GNND_LAUNCH(false, false);
  } else if (fcode) {
    if (merge) GNND_LAUNCH(true, true);
    else GNND_LAUNCH(true, false);
  } else {
    if (merge) GNND_LAUNCH(false, true);
    else GNND_LAUNCH(false, false);
  }
#undef GNND_LAUNCH
#undef GNND_ARGS
  return hipGetLastError();
}

static int compute_units() {
  static int cus = 0;
  if (cus == 0) {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
      cus = v;
    else
      cus = 256;
  }
  return cus;
}

hipError_t launch_join_mfma(const Shape& sh, const DevState& ds, bool merge_mode, bool first_look,
                            hipStream_t st, hipEvent_t after_join) {
  const int ksteps = (sh.d + 31) / 32;
  const bool fcode = sh.metric != kL2U8;
  const bool staged = ds.stg_ent != nullptr;
  const bool lean = first_look && !merge_mode;  // (direct hand-out only)
  const bool all = first_look || worth_leaving_out(sh, merge_mode);  // (staged only)
  StageArgs sa{ds.stg_ent, ds.stg_cur, ds.poff, 0, 0, 0, 1, 0, all ? ds.forms + 1 : nullptr};
  hipError_t e;
  // persistent wavefronts.  Direct: about two resident sets of workgroups; staged: one workgroup per
  // CU (the staging area takes most of a CU's LDS)
  const int64_t want = (sh.n + (staged ? kStagedWaves : 4) - 1) / (staged ? kStagedWaves : 4);
  const int64_t most = staged ? compute_units() : kJoinGrid;
  const unsigned grid = (unsigned)(want < most ? want : most);
  if (staged) {
    sa.tb = stage_bucket_bits(sh.n);
    sa.nb = (int)((sh.n + ((int64_t)1 << sa.tb) - 1) >> sa.tb);
    // flush at half-full on average: few results find their bucket's places taken
    sa.threshold = (uint32_t)(sa.nb * (kStageSlots / 2));
    // (the sampling stage has cleared the region cursors)
    // the first number from the golden section of n on that has no divisor in common with n
    int64_t spread = (int64_t)(0.6180339887 * (double)sh.n) + 1;
    while (std::gcd(spread, sh.n) != 1) ++spread;
    sa.spread = (uint32_t)spread;  // (at most n + 1, below 2^23)
    sa.stride = (uint32_t)((int64_t)grid * kStagedWaves * spread % sh.n);
  }
  auto launch = [&](auto steps) {
    constexpr int K = decltype(steps)::value;
    if (staged) return launch_k<K, true>(fcode, merge_mode, grid, st, ds.shadow, ds.meta, sh, ds, sa);
    return lean ? launch_k<K, false, true>(fcode, false, grid, st, ds.shadow, ds.meta, sh, ds, sa)
                : launch_k<K, false>(fcode, merge_mode, grid, st, ds.shadow, ds.meta, sh, ds, sa);
  };
  switch (ksteps) {
    case 1: e = launch(std::integral_constant<int, 1>{}); break;
    case 2: e = launch(std::integral_constant<int, 2>{}); break;
    case 3: e = launch(std::integral_constant<int, 3>{}); break;
    default: e = launch(std::integral_constant<int, 4>{});
  }
  if (after_join) (void)hipEventRecord(after_join, st);
  if (e != hipSuccess || !staged) return e;
  // (a region is shorter than 2^32 slots: n <= 2^22, 6p <= 192 slots per node)
  const int part_tb = sa.tb < kRcBits ? sa.tb : kRcBits;
  const bool filter = sa.all != nullptr;
  const size_t lds = result_csr_lds_bytes(part_tb, filter);
  auto* csr = filter ? (fcode ? &k_result_csr<true, true> : &k_result_csr<true, false>)
                     : (fcode ? &k_result_csr<false, true> : &k_result_csr<false, false>);
  e = hipFuncSetAttribute(reinterpret_cast<const void*>(csr),
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  const unsigned csr_grid = (unsigned)sa.nb << (sa.tb - part_tb);
  csr<<<csr_grid, kRcBlock, lds, st>>>(sh.n, sa.tb, ds.poff, ds.stg_cur, ds.stg_ent, ds.bins,
                                             ds.pslot, ds.meta, ds.counters, sa.all);
  return hipGetLastError();
}

hipError_t launch_init_random_i8(const Shape& sh, const DevState& ds, uint64_t seed,
                                 hipStream_t st) {
  // segmented lists: the general kernel on the original vectors gives the same integers
  if (sh.segments > 1) return launch_init_random_segmented(sh, ds, seed, st);
  if (sh.k > kWave) return launch_init_random_wide_i8(sh, ds, seed, st);
  const int dpad = (sh.d + 31) & ~31;
  const dim3 grid = grid_blocks((sh.n + 3) / 4);
  const uint64_t base = hash_base(seed, kTagInit);
  if (sh.metric != kL2U8)
    k_init_random_i8<true><<<grid, 256, 0, st>>>(ds.shadow, ds.meta, dpad, sh.n, sh.k, base, ds.G);
  else
    k_init_random_i8<false><<<grid, 256, 0, st>>>(ds.shadow, ds.meta, dpad, sh.n, sh.k, base, ds.G);
  return hipGetLastError();
}

hipError_t launch_merge_init_i8(const Shape& sh, const DevState& ds, uint64_t seed,
                                const MergeIds& mi, const int32_t* ids1, const void* dist1,
                                const int32_t* ids2, const void* dist2, hipStream_t st) {
  // long lists: the general kernel on the original vectors gives the same integers
  if (sh.k > kWave) return launch_merge_init(sh, ds, seed, mi, ids1, dist1, ids2, dist2, st);
  const int dpad = (sh.d + 31) & ~31;
  const dim3 grid = grid_blocks((sh.n + 3) / 4);
  const uint64_t base = hash_base(seed, kTagMerge);
  if (sh.metric != kL2U8)
    k_merge_init_i8<true><<<grid, 256, 0, st>>>(ds.shadow, ds.meta, dpad, sh.n, mi, sh.k, base, ids1,
                                                dist1, ids2, dist2, ds.G, ds.aside);
  else
    k_merge_init_i8<false><<<grid, 256, 0, st>>>(ds.shadow, ds.meta, dpad, sh.n, mi, sh.k, base,
                                                 ids1, dist1, ids2, dist2, ds.G, ds.aside);
  return hipGetLastError();
}

hipError_t launch_pack_i8(const Shape& sh, const DevState& ds, int* bad_flag_dev,
                          hipStream_t st) {
  const int dpad = (sh.d + 31) & ~31;
  const dim3 grid = grid_blocks((sh.n + 3) / 4);
  if (sh.metric == kL2U8 && (sh.d & 15) == 0) {
    const int64_t per_block = 4 * (kWave / (dpad >> 4));  // rows per workgroup
    k_pack_u8_wide<<<grid_blocks((sh.n + per_block - 1) / per_block), 256, 0, st>>>(
        static_cast<const uint8_t*>(sh.vec_a), static_cast<const uint8_t*>(sh.vec_b), sh.split,
        sh.n, sh.d, dpad, ds.shadow, ds.meta);
  } else if (sh.metric == kL2U8)
    k_pack_i8<uint8_t><<<grid, 256, 0, st>>>(sh.vec_a, sh.vec_b, sh.split, sh.n, sh.d, dpad,
                                             ds.shadow, ds.meta, bad_flag_dev);
  else
    k_pack_i8<float><<<grid, 256, 0, st>>>(sh.vec_a, sh.vec_b, sh.split, sh.n, sh.d, dpad,
                                           ds.shadow, ds.meta, bad_flag_dev);
  return hipGetLastError();
}

}  // namespace gnnd

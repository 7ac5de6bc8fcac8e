// Cross-matching and nearest-object search (Sec. 4.2, 4.3, Alg. 2) for sample lists of 65..128
// objects (p > 32) on byte-valued data of up to 128 dimensions: exact integer distances from
// inner products on the matrix cores, the long-list form of k_join_mfma.
//
// One workgroup of BLOCKS wavefronts per node: 3 for lists of up to 96 samples (p <= 48), 4 beyond.
// (A fourth wavefront without samples of its own kept its place and a quarter of the LDS: with
// three, 3.75 instead of 3 busy wavefronts per SIMD; 100,000 x 128, p = 42, whole build 3.70 ->
// 3.39 ms.)
// Wavefront w brings blocks w (32 samples) of the
// NEW and of the OLD list, keeps them as column operands and leaves them in LDS as row operands
// for all four; its columns then meet every block of rows they have partners in.  A tile's
// epilogue keeps one column per lane (see tile_col_best), so nothing is reduced across lanes
// but the two halves of a tile.
//
// 100,000 x 128 byte-valued vectors, k = 64, p = 42: 0.61 ms per iteration where the general
// long join (k_join_long, float32 sums on the vector units) takes 5.5; build of 4 iterations
// 24.3 -> 4.2 ms (3.4 with the three wavefronts and faster kernels around it).  Bound by the epilogue's vector instructions and the hand-out's atomics.
#include "gram_i8.hpp"
#include "kernels.hpp"

namespace gnnd {

namespace {

constexpr int kLongBits = 7;
constexpr int32_t kFarLong = 3 << 22;  // "norm" of an absent row: above every real distance

template <int KSTEPS, int BLOCKS, bool FCODE, bool MERGE>
__global__ __launch_bounds__(kWave* BLOCKS) void k_join_long_i8(
    const int8_t* __restrict__ shadow, const NodeMeta* __restrict__ meta, int64_t n, int p,
    int64_t split, const int32_t* __restrict__ snew, const int32_t* __restrict__ sold,
    const int32_t* __restrict__ cnew, const int32_t* __restrict__ cold, uint64_t* pslot,
    uint64_t slots, uint64_t* __restrict__ bins, uint64_t* counters) {
  constexpr int dpad = 32 * KSTEPS;
  constexpr int kLongList = 32 * BLOCKS;  // longest sample list
  constexpr int kRow = dpad + 16;  // row stride in LDS: 8 lanes reading 16 bytes of 8
                                   // consecutive rows touch different banks
  __shared__ __attribute__((aligned(16))) int8_t rows[2 * kLongList * kRow];  // NEW, then OLD
  __shared__ __attribute__((aligned(16))) int32_t neg[2 * kLongList];  // see tile_col_best
  __shared__ int32_t ids[2 * kLongList];  // absent: INT_MAX, so that both lists stay ascending
  __shared__ uint32_t second[2 * BLOCKS]; // MERGE: samples of the second set, per block of 32
  __shared__ uint32_t tally[4];           // duplicates, found, passed, overflow
  const int64_t s = block_linear();
  if (s >= n) return;
  const int nn = cnew[s], no = cold[s];
  const bool do_nn = !MERGE && nn > 1;
  if (nn == 0 || (!do_nn && no == 0)) return;  // nothing to evaluate (uniform)
  const int wave = wave_id(), lane = lane_id(), half = lane >> 5, col = lane & 31;
  const int pos = 32 * wave + col;  // lanes 0..31 stand for NEW sample pos, 32..63 for OLD
  const int L = 2 * p;
  int32_t self = -1;
  if (pos < (half ? no : nn)) self = (half ? sold : snew)[s * L + pos];
  const int32_t id_n = __shfl(self, col, kWave), id_o = __shfl(self, 32 + col, kWave);
  const Operand N = load_block<KSTEPS>(shadow, dpad, id_n, half);
  const Operand O = load_block<KSTEPS>(shadow, dpad, id_o, half);
  uint2 mine = make_uint2(0u, (uint32_t)kFarLong);  // threshold of the sample's list, norm
  if (self >= 0) mine = *reinterpret_cast<const uint2*>(meta + self);
  neg[kLongList * half + pos] = -(int32_t)((mine.y << kLongBits) | (uint32_t)pos);
  ids[kLongList * half + pos] = self >= 0 ? self : 0x7fffffff;
  if (threadIdx.x < 4) tally[threadIdx.x] = 0u;
  if (MERGE) {
    const uint64_t m = __ballot(self >= 0 && (int64_t)self >= split);
    if (lane == 0) {
      second[wave] = (uint32_t)m;
      second[BLOCKS + wave] = (uint32_t)(m >> 32);
    }
  }
#pragma unroll
  for (int k = 0; k < KSTEPS; ++k) {
    *reinterpret_cast<v4i*>(rows + pos * kRow + 32 * k + 16 * half) = N.k[k];
    *reinterpret_cast<v4i*>(rows + (kLongList + pos) * kRow + 32 * k + 16 * half) = O.k[k];
  }
  __syncthreads();

  // An object sampled as NEW and as OLD is no pair: its place in the other list, or -1.
  int eq = -1;
  {
    const int32_t* other = ids + (half ? 0 : kLongList);
    int lo = 0, hi = kLongList;
#pragma unroll
    for (int step = 0; step < 8; ++step) {
      const bool go = lo < hi;
      const int mid = go ? (lo + hi) >> 1 : 0;  // < kLongList
      const bool below = go && other[mid] < self;
      lo = below ? mid + 1 : lo;
      hi = (go && !below) ? mid : hi;
    }
    if (self >= 0 && lo < kLongList && other[lo] == self) eq = lo;
  }
  const uint64_t dup_lanes = __ballot(eq >= 0 && half == 0);
  if (lane == 0 && dup_lanes) atomicAdd(&tally[0], (uint32_t)__popcll(dup_lanes));
  const bool masked = MERGE || __ballot(eq >= 0) != 0ull;
  const int eq_n = __shfl(eq, col, kWave), eq_o = __shfl(eq, 32 + col, kWave);
  auto row_block = [&](int b) {  // 32 rows from LDS, this lane's pieces
    Operand r;
#pragma unroll
    for (int k = 0; k < KSTEPS; ++k)
      r.k[k] = *reinterpret_cast<const v4i*>(rows + (32 * b + col) * kRow + 32 * k + 16 * half);
    return r;
  };
  // rows of block `b` (of the other list) that are no partners of the column object
  auto excluded = [&](int eq_row, int b, uint32_t second_rows, int32_t col_id) {
    uint32_t m = 0;
    if (eq_row >= 0 && (eq_row >> 5) == b) m |= 1u << (eq_row & 31);
    if (MERGE) m |= (int64_t)col_id >= split ? second_rows : ~second_rows;
    return m;
  };
  const int nb_new = (nn + 31) >> 5, nb_old = (no + 31) >> 5;
  int32_t near_nn = kNone, near_no = kNone, near_on = kNone;
  if (wave < nb_new) {
    if (do_nn)
      for (int b = 0; b < nb_new; ++b) {
        const v16i g = gram<KSTEPS>(row_block(b), N);
        near_nn = max(near_nn, b == wave ? tile_col_best<true, kLongBits>(g, neg + 32 * b, half,
                                                                          1u << col)
                                         : tile_col_best<false, kLongBits>(g, neg + 32 * b, half, 0u));
      }
    for (int b = 0; b < nb_old; ++b) {
      const v16i g = gram<KSTEPS>(row_block(BLOCKS + b), N);
      const int32_t* at = neg + kLongList + 32 * b;
      near_no = max(near_no, masked ? tile_col_best<true, kLongBits>(
                                          g, at, half, excluded(eq_n, b, MERGE ? second[BLOCKS + b] : 0u, id_n))
                                    : tile_col_best<false, kLongBits>(g, at, half, 0u));
    }
  }
  if (wave < nb_old) {
    for (int b = 0; b < nb_new; ++b) {
      const v16i g = gram<KSTEPS>(row_block(b), O);
      const int32_t* at = neg + 32 * b;
      near_on = max(near_on, masked ? tile_col_best<true, kLongBits>(
                                          g, at, half, excluded(eq_o, b, MERGE ? second[b] : 0u, id_o))
                                    : tile_col_best<false, kLongBits>(g, at, half, 0u));
    }
  }
  near_nn = both_halves_max(near_nn);
  near_no = both_halves_max(near_no);
  near_on = both_halves_max(near_on);

  // ---- hand the results on: lanes 0..31 answer for NEW samples (two results, one request),
  // lanes 32..63 for OLD samples -------------------------------------------------------------
  uint64_t entry[2];
  bool found[2], pass[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int32_t best = half ? (t ? kNone : near_on) : (t ? near_no : near_nn);
    const int32_t key = -best;  // ((row norm - 2 G) << kLongBits) | row position
    const int32_t part = key >> kLongBits;
    found[t] = self >= 0 && best != kNone && part < (1 << 23);
    const int32_t dist = part + (int32_t)mine.y;
    const uint32_t code = FCODE ? ord_f32((float)dist) : ord_i32(dist);
    const int list = !half && t ? kLongList : 0;
    const int32_t other = found[t] ? ids[list + (key & ((1 << kLongBits) - 1))] : 0;
    pass[t] = found[t] && code <= mine.x;  // what cannot enter the list is dropped
    entry[t] = make_entry(code, (uint32_t)other, 3u);
  }
  const uint32_t want = (pass[0] ? 1u : 0u) + (pass[1] ? 1u : 0u);
  bool over = false;
  if (want) {
    // one returning add yields the segment start and the first result's place in it
    const uint64_t w = atomicAdd(reinterpret_cast<unsigned long long*>(&pslot[self]),
                                 (unsigned long long)want);
    const uint64_t at = (w >> kSlotCountBits) + (w & kSlotCountMask);
    if (at + want <= slots) {
      bins[at] = pass[0] ? entry[0] : entry[1];
      if (want == 2u) bins[at + 1] = entry[1];
    } else {
      over = true;
    }
  }
  const uint32_t n_found = (uint32_t)(__popcll(__ballot(found[0])) + __popcll(__ballot(found[1])));
  const uint32_t n_pass = (uint32_t)(__popcll(__ballot(pass[0])) + __popcll(__ballot(pass[1])));
  const uint32_t n_over = (uint32_t)__popcll(__ballot(over));
  if (lane == 0) {
    if (n_found) atomicAdd(&tally[1], n_found);
    if (n_pass) atomicAdd(&tally[2], n_pass);
    if (n_over) atomicAdd(&tally[3], n_over);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t ev;
    if (MERGE) {
      uint64_t n2 = 0, o2 = 0;  // samples of the second set
      for (int b = 0; b < BLOCKS; ++b) {
        n2 += (uint64_t)__popc(second[b]);
        o2 += (uint64_t)__popc(second[BLOCKS + b]);
      }
      ev = n2 * ((uint64_t)no - o2) + ((uint64_t)nn - n2) * o2;
    } else {
      ev = (do_nn ? (uint64_t)nn * (nn - 1) / 2 : 0) + (uint64_t)nn * no - tally[0];
    }
    unsigned long long* cs =
        reinterpret_cast<unsigned long long*>(counters + (s & (kStripes - 1)) * C_SLOTS);
    if (tally[1]) atomicAdd(cs + C_PROPS, (unsigned long long)tally[1]);
    if (tally[2]) atomicAdd(cs + C_PASSED, (unsigned long long)tally[2]);
    if (tally[3]) atomicAdd(cs + C_OVERFLOW, (unsigned long long)tally[3]);
    if (ev) atomicAdd(cs + C_EVALS, (unsigned long long)ev);
  }
}

template <int KSTEPS, int BLOCKS>
void launch(const Shape& sh, const DevState& ds, bool merge, hipStream_t st) {
  const dim3 grid = grid_blocks(sh.n);
  const uint64_t slots = (uint64_t)sh.slots();
  const bool fcode = sh.metric != kL2U8;
  auto* const kernel = fcode ? (merge ? k_join_long_i8<KSTEPS, BLOCKS, true, true>
                                      : k_join_long_i8<KSTEPS, BLOCKS, true, false>)
                             : (merge ? k_join_long_i8<KSTEPS, BLOCKS, false, true>
                                      : k_join_long_i8<KSTEPS, BLOCKS, false, false>);
  kernel<<<grid, kWave * BLOCKS, 0, st>>>(ds.shadow, ds.meta, sh.n, sh.p, sh.split, ds.snew,
                                          ds.sold, ds.cnew, ds.cold, ds.pslot, slots, ds.bins,
                                          ds.counters);
}
template <int KSTEPS>
void launch(const Shape& sh, const DevState& ds, bool merge, hipStream_t st) {
  if (2 * sh.p <= 96) launch<KSTEPS, 3>(sh, ds, merge, st);
  else launch<KSTEPS, 4>(sh, ds, merge, st);
}

}  // namespace

hipError_t launch_join_long_i8(const Shape& sh, const DevState& ds, bool merge_mode,
                               hipStream_t st) {
  switch ((sh.d + 31) / 32) {
    case 1: launch<1>(sh, ds, merge_mode, st); break;
    case 2: launch<2>(sh, ds, merge_mode, st); break;
    case 3: launch<3>(sh, ds, merge_mode, st); break;
    default: launch<4>(sh, ds, merge_mode, st);
  }
  return hipGetLastError();
}

}  // namespace gnnd

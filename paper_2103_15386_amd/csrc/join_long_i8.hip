// Cross-matching and nearest-object search (Sec. 4.2, 4.3, Alg. 2) for sample lists of 65..128
// objects (p > 32) on byte-valued data of up to 128 dimensions: exact integer distances from
// inner products on the matrix cores, the long-list form of k_join_mfma.
//
// One workgroup of BLOCKS wavefronts per node at a time: 3 for lists of up to 96 samples (p <= 48), 4
// beyond.  (A fourth wavefront without samples of its own kept its place and a quarter of the LDS: with
// three, 3.75 instead of 3 busy wavefronts per SIMD; 100,000 x 128, p = 42, whole build 3.70 ->
// 3.39 ms.)  Wavefront w brings blocks w (32 samples) of the NEW and of the OLD list, keeps them as
// column operands and leaves them in LDS as row operands for all of them; its columns then meet every
// block of rows they have partners in.  A tile's epilogue keeps one column per lane (see
// tile_col_best), so nothing is reduced across lanes but the two halves of a tile.
//
// Persistent workgroups: the next node's sample ids are on their way while a node is worked on, and
// its rows are requested as soon as the last tile has consumed the operand registers, together with
// the places of this node's results, so that a node waits for memory once instead of five times
// (list sizes, ids, rows, places, and the end of the workgroup).
//
// 100,000 x 128 byte-valued vectors, k = 64, p = 42: 0.475 ms per iteration (0.535 with a workgroup per
// node) where the general long join (k_join_long, float32 sums on the vector units) takes 5.5.
#include "gram_i8.hpp"
#include "kernels.hpp"

namespace gnnd {

namespace {

constexpr int kLongBits = 7;
// "norm" of an absent row, and what no distance reaches
constexpr int32_t kFarLong = 3 << 22, kLongLimit = 1 << 23;
static_assert(far_enough(kFarLong, kLongLimit, kLongBits), "absent rows are told from present ones");

// Wavefronts per SIMD.  Short rows keep few registers, and more wavefronts wait for memory at once: an
// iteration of 600,000 x 16 bytes, p = 64, takes 3.53 ms with 4, 3.44 with 5 and 3.42 with 7 of them,
// 100,000 x 16 0.507, 0.493 and 0.482, 600,000 x 64, p = 42, 2.75 with 4 and 2.71 with 5.  (6 of them in
// workgroups of three: the eight workgroups did not fit at once, 600,000 x 16, p = 42, 2.83 -> 3.31.)
constexpr int long_waves(int ksteps) { return ksteps == 1 ? 7 : ksteps <= 3 ? 5 : 4; }

template <int KSTEPS, int BLOCKS, bool FCODE, bool MERGE>
__global__ __launch_bounds__(kWave* BLOCKS)
__attribute__((amdgpu_waves_per_eu(long_waves(KSTEPS), long_waves(KSTEPS)))) void k_join_long_i8(
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
  __shared__ int32_t ids[2][128];  // absent: INT_MAX, so that both lists stay ascending
  __shared__ uint32_t second[2 * BLOCKS]; // MERGE: samples of the second set, per block of 32
  const int wave = wave_id(), lane = lane_id(), half = lane >> 5, col = lane & 31;
  const int pos = 32 * wave + col;  // lanes 0..31 stand for NEW sample pos, 32..63 for OLD
  const int L = 2 * p;
  if (BLOCKS < 4) {  // the places no sample ever takes
    for (int i = threadIdx.x; i < 2 * (128 - kLongList); i += kWave * BLOCKS)
      ids[i & 1][kLongList + (i >> 1)] = 0x7fffffff;
  }
  const int32_t* const lists = half ? sold : snew;
  // (nodes beyond the end: the last one, unused.  The sizes are known one node ahead of the ids, whose
  // unused places are not read: on average half of both lists, 3.59 -> 3.42 ms at 600,000 x 16, p = 64)
  auto id_of = [&](int64_t node, int nn_of, int no_of) {
    int32_t id = -1;
    if (pos < (half ? no_of : nn_of)) id = lists[vmin(node, n - 1) * L + pos];
    return id;
  };
  int64_t s = blockIdx.x;
  int nn = cnew[s], no = cold[s];
  int32_t self = id_of(s, nn, no);
  const int64_t stride = gridDim.x;
  int nx_nn = cnew[vmin(s + stride, n - 1)], nx_no = cold[vmin(s + stride, n - 1)];
  int32_t nx_self = id_of(s + stride, nx_nn, nx_no);
  int nx2_nn = cnew[vmin(s + 2 * stride, n - 1)], nx2_no = cold[vmin(s + 2 * stride, n - 1)];
  // (registers of absent samples keep what they held: an absent row is kept out of every result by
  // its norm, see far_enough, an absent column has no result)
  Operand N{}, O{};
  uint2 mine = make_uint2(0u, 0u);  // threshold of the sample's list, norm
  bool do_nn = false, active = false;
  auto begin_node = [&]() {
    do_nn = !MERGE && nn > 1;
    active = nn > 0 && (do_nn || no > 0);
    if (!active) return;  // nothing to evaluate (uniform)
    mine = *reinterpret_cast<const uint2*>(meta + vmax(self, 0));
    uint32_t id_n, id_o;
    pair_lanes((uint32_t)self, 32, id_n, id_o);
    load_present<KSTEPS>(N, shadow, (int32_t)id_n, half);
    load_present<KSTEPS>(O, shadow, (int32_t)id_o, half);
  };
  begin_node();
  // what this wavefront has counted over its nodes
  uint32_t all_found = 0, all_passed = 0, over = 0;
  int64_t all_evals = 0;
  for (;;) {
    uint32_t want = 0;
    uint64_t word = 0, entry[2] = {0ull, 0ull};
    if (active) {
      if (self < 0) mine.y = (uint32_t)kFarLong;
      neg[kLongList * half + pos] = -(int32_t)((mine.y << kLongBits) | (uint32_t)pos);
      ids[half][pos] = self >= 0 ? self : 0x7fffffff;
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
      if (no > 0) {
        const int32_t* const other = ids[1 - half];
        const int32_t* at = other;
#pragma unroll
        for (int step = 64; step > 0; step >>= 1) at = at[step - 1] < self ? at + step : at;
        if (*at == self) eq = (int)(at - other);
      }
      const uint64_t eq_lanes = __ballot(eq >= 0);
      uint32_t eq_n = ~0u, eq_o = ~0u, id_n = 0, id_o = 0;
      if (eq_lanes != 0ull) pair_lanes((uint32_t)eq, 32, eq_n, eq_o);
      if (MERGE) pair_lanes((uint32_t)self, 32, id_n, id_o);
      auto row_block = [&](int b) {  // 32 rows from LDS, this lane's pieces
        Operand r;
#pragma unroll
        for (int k = 0; k < KSTEPS; ++k)
          r.k[k] = *reinterpret_cast<const v4i*>(rows + (32 * b + col) * kRow + 32 * k + 16 * half);
        return r;
      };
      // rows of block `b` (of the other list) that are no partners of the column object
      auto excluded = [&](uint32_t eq_row, int b, uint32_t second_rows, uint32_t col_id) {
        uint32_t m = 0;
        if ((eq_row >> 5) == (uint32_t)b) m |= 1u << (eq_row & 31);  // (none: ~0)
        if (MERGE) m |= (int64_t)(int32_t)col_id >= split ? second_rows : ~second_rows;
        return m;
      };
      const int nb_new = (nn + 31) >> 5, nb_old = (no + 31) >> 5;
      int32_t near_nn = kNone, near_no = kNone, near_on = kNone;
      // a tile whose columns have partners in all of its rows needs no mask
      auto best_of = [&](const v16i& g, const int32_t* at, uint32_t skip) {
        return __ballot(skip != 0u) ? tile_col_best<true, kLongBits>(g, at, half, skip)
                                    : tile_col_best<false, kLongBits>(g, at, half, 0u);
      };
      // rows of NEW samples meet both kinds of columns
      for (int b = 0; b < nb_new; ++b) {
        const Operand r = row_block(b);
        const bool new_cols = do_nn && wave < nb_new, old_cols = wave < nb_old;
        // (one after the other: both tiles at once are 16 registers more)
        if (new_cols)
          near_nn = max(near_nn, best_of(gram<KSTEPS>(r, N), neg + 32 * b,
                                         b == wave ? 1u << col : 0u));
        if (old_cols)
          near_on = max(near_on, best_of(gram<KSTEPS>(r, O), neg + 32 * b,
                                         excluded(eq_o, b, MERGE ? second[b] : 0u, id_o)));
      }
      if (wave < nb_new)
        for (int b = 0; b < nb_old; ++b) {
          const v16i g = gram<KSTEPS>(row_block(BLOCKS + b), N);
          near_no = max(near_no, best_of(g, neg + kLongList + 32 * b,
                                         excluded(eq_n, b, MERGE ? second[BLOCKS + b] : 0u, id_n)));
        }

      // ---- hand the results on: lanes 0..31 answer for NEW samples (two results, one request),
      // lanes 32..63 for OLD samples -------------------------------------------------------------
      const int32_t res[2] = {blocks_max(near_nn, near_on), both_halves_max(near_no)};
      bool pass[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int32_t best = half && t ? kNone : res[t];
        const int32_t key = -best;  // ((row norm - 2 G) << kLongBits) | row position
        const int32_t part = key >> kLongBits;
        const bool found = self >= 0 && best != kNone && part < kLongLimit;
        const int32_t dist = part + (int32_t)mine.y;
        const uint32_t code = FCODE ? ord_f32((float)dist) : ord_i32(dist);
        const int32_t other = ids[t][key & ((1 << kLongBits) - 1)];
        pass[t] = found && code <= mine.x;  // what cannot enter the list is dropped
        entry[t] = make_entry(code, (uint32_t)other, 3u);
        all_found += (uint32_t)__popcll(__ballot(found));
        all_passed += (uint32_t)__popcll(__ballot(pass[t]));
      }
      if (!pass[0]) entry[0] = entry[1];
      want = (pass[0] ? 1u : 0u) + (pass[1] ? 1u : 0u);
      if (want)  // one returning add yields the segment start and the first result's place in it
        word = atomicAdd(reinterpret_cast<unsigned long long*>(&pslot[self]),
                         (unsigned long long)want);
      // pairs evaluated: every wavefront takes off its NEW samples that are OLD ones too
      if (MERGE) {
        if (wave == 0) {
          int n2 = 0, o2 = 0;  // samples of the second set
          for (int b = 0; b < BLOCKS; ++b) {
            n2 += __popc(second[b]);
            o2 += __popc(second[BLOCKS + b]);
          }
          all_evals += (int64_t)n2 * (no - o2) + (int64_t)(nn - n2) * o2;
        }
      } else {
        if (wave == 0) all_evals += (do_nn ? nn * (nn - 1) / 2 : 0) + nn * no;
        all_evals -= __popc((uint32_t)eq_lanes);
      }
    }
    const bool worked = active, more = s + stride < n;
    if (more) {
      s += stride;
      nn = nx_nn;
      no = nx_no;
      self = nx_self;
      begin_node();
      nx_nn = nx2_nn;
      nx_no = nx2_no;
      nx_self = id_of(s + stride, nx_nn, nx_no);
      nx2_nn = cnew[vmin(s + 2 * stride, n - 1)];
      nx2_no = cold[vmin(s + 2 * stride, n - 1)];
    }
    if (want) {
      const uint64_t at = (word >> kSlotCountBits) + (word & kSlotCountMask);
      if (at + want <= slots) {
        bins[at] = entry[0];
        if (want == 2u) bins[at + 1] = entry[1];
      } else {
        ++over;
      }
    }
    if (!more) break;
    if (worked) __syncthreads();  // the rows and lists have been read
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) over += __shfl_xor(over, off, kWave);
  if (lane == 0) {
    unsigned long long* cs = reinterpret_cast<unsigned long long*>(
        counters + ((blockIdx.x * BLOCKS + wave) & (kStripes - 1)) * C_SLOTS);
    if (all_found) atomicAdd(cs + C_PROPS, (unsigned long long)all_found);
    if (all_passed) atomicAdd(cs + C_PASSED, (unsigned long long)all_passed);
    if (over) atomicAdd(cs + C_OVERFLOW, (unsigned long long)over);
    if (all_evals) atomicAdd(cs + C_EVALS, (unsigned long long)all_evals);
  }
}

// Workgroups: as many as are resident.
int long_join_groups(int blocks, int waves) {
  static int cus = 0;
  if (cus == 0) {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
      cus = v;
    else
      cus = 256;
  }
  return cus * (4 * waves / blocks);  // (their LDS fits: at most 151 KB)
}

template <int KSTEPS, int BLOCKS>
void launch(const Shape& sh, const DevState& ds, bool merge, hipStream_t st) {
  const int64_t most = long_join_groups(BLOCKS, long_waves(KSTEPS));
  const unsigned grid = (unsigned)(sh.n < most ? sh.n : most);
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

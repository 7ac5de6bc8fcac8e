// Inner products of byte-valued rows (value - 128 as int8) in 32 x 32 tiles on the matrix
// cores, and the nearest row of every column of a tile; shared by the joins on byte-valued data.
#pragma once
#include "device_utils.hpp"
#include "kernels.hpp"

namespace gnnd {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

// Best row per column of one 32x32 accumulator tile, for lists of up to 2^BITS samples.  For
// row r the LDS array holds negR = -((norm_r << BITS) | position_r); then t =
// (G << (BITS + 1)) + negR is -(((norm_r - 2 G) << BITS) | position_r), so the maximum of t over the rows is
// the row with the smallest (norm_r - 2 G), ties to the smallest position -
// one shift-add and half a max3 per accumulator register.  Adding the column's
// own norm to ((-t) >> BITS) gives the squared distance.  A row that is not there has a norm
// far beyond (see far_enough) and whatever an earlier node left in its place, so its G is that of
// any two rows; so is that of a row with itself.  Rows flagged in `excl` are skipped.  Row of
// register r for this lane: 8*(r/4) + 4*half + r%4.
constexpr int32_t kNone = (int32_t)0x80000000;

// Rows of up to 128 int8: norms up to 2^21, 2 G from -2 128 128 127 to 2 128 128 128, squared
// distances up to 128 255^2 (and norm_r - 2 G no more than that).  A row with the norm `far` is told
// from every row that is there if what it gives is `limit` or more and a distance is less, and the key
// of the farthest one still fits 32 bits.
constexpr bool far_enough(int64_t far, int64_t limit, int bits) {
  return far - 2 * 128 * 128 * 128 >= limit && limit > 128 * 255 * 255 &&
         ((far + 2 * 128 * 128 * 127) << bits) + ((int64_t)1 << bits) - 1 < ((int64_t)1 << 31);
}

template <bool MASKED, int BITS = 6>
__device__ inline int32_t tile_col_best(const v16i& g, const int32_t* negr_lds, int half,
                                        uint32_t excl) {
  int32_t best = kNone;
  const uint32_t ex = excl >> (4 * half);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int4 nr = *reinterpret_cast<const int4*>(negr_lds + 8 * q + 4 * half);
    const int32_t negr[4] = {nr.x, nr.y, nr.z, nr.w};
    int32_t t[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      t[i] = (int32_t)(((uint32_t)g[4 * q + i] << (BITS + 1)) + (uint32_t)negr[i]);
      if (MASKED) t[i] = (ex & (1u << (8 * q + i))) ? kNone : t[i];
    }
    best = max(best, max(t[0], t[1]));
    best = max(best, max(t[2], t[3]));
  }
  return best;
}

// The same for lists of up to 64 samples with a place of its own (in words, from `negr_lds`) for each
// of the lane's four groups of rows.
__device__ inline int32_t tile_col_best_at(const v16i& g, const int32_t* negr_lds,
                                           const int (&at)[4]) {
  int32_t best = kNone;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int4 nr = *reinterpret_cast<const int4*>(negr_lds + at[q]);
    const int32_t negr[4] = {nr.x, nr.y, nr.z, nr.w};
    int32_t t[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      t[i] = (int32_t)(((uint32_t)g[4 * q + i] << 7) + (uint32_t)negr[i]);
    best = max(best, max(t[0], t[1]));
    best = max(best, max(t[2], t[3]));
  }
  return best;
}

// Results of two column blocks, each spread over both halves: block 0's larger one in lanes 0..31,
// block 1's in lanes 32..63.
__device__ inline int32_t blocks_max(int32_t x0, int32_t x1) {
  auto sw = __builtin_amdgcn_permlane32_swap((uint32_t)x0, (uint32_t)x1, false, false);
  const int32_t a = (int32_t)sw[0], b = (int32_t)sw[1];
  return a > b ? a : b;
}

__device__ inline int32_t both_halves_max(int32_t x) {
  auto sw = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)x, false, false);
  int32_t a = (int32_t)sw[0], b = (int32_t)sw[1];
  return a > b ? a : b;
}

struct Operand {
  v4i k[4];  // 4 steps of 32 dimensions, 16 bytes of this lane each
};

// This lane's pieces of row `id` (a block's rows: one per lane of either half); a negative id leaves
// the registers as they are.
template <int KSTEPS>
__device__ inline void load_present(Operand& o, const int8_t* shadow, int32_t id, int half) {
  if (id < 0) return;
  const int8_t* row = shadow + (int64_t)id * (32 * KSTEPS) + 16 * half;
#pragma unroll
  for (int s = 0; s < KSTEPS; ++s) o.k[s] = *reinterpret_cast<const v4i*>(row + 32 * s);
}

template <int KSTEPS>
__device__ inline v16i gram(const Operand& rows, const Operand& cols) {
  v16i acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int s = 0; s < KSTEPS; ++s)
    acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(rows.k[s], cols.k[s], acc, 0, 0, 0);
  return acc;
}

// Exact squared distances |a|^2 + |b|^2 - 2 a.b (four products per v_dot4) on
// the int8 rows, from node s to one object per lane: `id` of lanes < count.
// A row is C = dpad / 16 <= 8 chunks of 16 bytes; the lanes of a group of 2, 4 or 8 (C = 6: two
// of 8 read nothing) read one object's row as one contiguous line, multiply
// it with the node's own chunk and add up across the group; the sums are then
// handed to the lanes that hold the objects.  All 64 lanes call it together;
// lanes >= count get 0.  (With groups of 6, ten objects per load, the sums took ten lane
// permutations per load instead of three exchanges: 200,000 x 96 bytes, k = 96, whole build 5.95 ->
// 5.87 ms.)
__device__ inline int32_t wave_distances_i8(const int8_t* __restrict__ shadow,
                                            const NodeMeta* meta, int dpad, int64_t s, uint32_t id,
                                            int count, int lane) {
  const int C = dpad >> 4, shift = C <= 2 ? 1 : C <= 4 ? 2 : 3;  // (C = 2, 4, 6, 8)
  const int per_load = kWave >> shift;
  const int grp = lane >> shift, sub = lane & ((1 << shift) - 1);
  const bool lane_used = sub < C;
  const v4i x = lane_used ? *reinterpret_cast<const v4i*>(shadow + s * dpad + 16 * sub)
                          : v4i{0, 0, 0, 0};
  const int32_t norm_s = meta[s].norm;
  // (the objects' norms come from their rows, which are here anyway: a gather of the stored
  // norm would be a second scattered access per object)
  int32_t dot = 0, norm_id = 0;
  for (int r0 = 0; r0 < count; r0 += per_load) {
    const int j = r0 + grp;  // the object this group reads
    const bool act = lane_used && j < count;
    const uint32_t nid = __shfl(id, act ? j : 0, kWave);
    int32_t part = 0, part_sq = 0;
    if (act) {
      const v4i y = *reinterpret_cast<const v4i*>(shadow + (int64_t)nid * dpad + 16 * sub);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        part = __builtin_amdgcn_sdot4(x[t], y[t], part, false);
        part_sq = __builtin_amdgcn_sdot4(y[t], y[t], part_sq, false);
      }
    }
    int32_t total = part, total_sq = part_sq;
    total += (int32_t)xor_lanes((uint32_t)total, 1, lane);
    total_sq += (int32_t)xor_lanes((uint32_t)total_sq, 1, lane);
    if (C > 2) {
      total += (int32_t)xor_lanes((uint32_t)total, 2, lane);
      total_sq += (int32_t)xor_lanes((uint32_t)total_sq, 2, lane);
    }
    if (C > 4) {
      total += (int32_t)xor_lanes((uint32_t)total, 4, lane);
      total_sq += (int32_t)xor_lanes((uint32_t)total_sq, 4, lane);
    }
    // object j = lane sits in group lane - r0
    const int32_t got = __shfl(total, ((lane - r0) << shift) & 63, kWave);
    const int32_t got_sq = __shfl(total_sq, ((lane - r0) << shift) & 63, kWave);
    if (lane >= r0 && lane < r0 + per_load) {
      dot = got;
      norm_id = got_sq;
    }
  }
  return lane < count ? norm_s + norm_id - 2 * dot : 0;
}

}  // namespace gnnd

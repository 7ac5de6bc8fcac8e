// Reverse-neighbour candidates (Sec. 4.1) grouped by target without global
// atomics.  Device-wide atomics run at a fixed ~27 G/s (12 G/s when the old
// value is needed), which made them the cost of the sampling stage, so the
// transpose "s samples v  ->  s is a candidate of v" is done as a two-level
// counting sort instead:
//   1. k_fwd_count   - forward sampling of every list (first p NEW / first p
//                      OLD entries, sampled NEW flagged OLD); per workgroup an
//                      LDS histogram of the targets' buckets (bucket = target id
//                      >> tb), kept as one column of a (bucket x workgroup)
//                      matrix.
//   2. k_wg_scan     - exclusive scan along the matrix rows: every workgroup's
//                      run start inside every bucket, and the <= 4096 bucket sizes
//                      per kind (the workgroups of 3. and 4. add those up for
//                      themselves: a launch that did nothing else took 24 us).
//   3. k_fwd_scatter_staged - every workgroup writes its (target, source)
//                      edges into its runs, sorted by bucket in LDS first.
//   4. k_bucket_csr  - one workgroup per bucket: LDS counters per target,
//                      block scan = the targets' segment offsets; the edges, kept
//                      in registers, put the sources in order in LDS (a bucket with
//                      too many edges is swept a second time instead).  Buckets are
//                      in target order, so the result is the same CSR a global scan
//                      would give.
// The loops over rows and edges keep several independent loads in flight per
// thread; with one load per trip they are bound by memory latency.
#include "device_utils.hpp"
#include "kernels.hpp"

namespace gnnd {

constexpr int kSB = 256;
constexpr int kMaxBuckets = 4096;
constexpr int kCsrBlock = 1024;

struct BucketGeom {
  int tb;         // log2(targets per bucket)
  int nb;         // buckets
  int rows_per_wg;
};

// Forward sampling of one list by one wavefront; returns this lane's sampled id
// (or -1) for each kind and writes the forward parts of the sample rows.
__device__ inline void forward_sample_row(int64_t s, int64_t n, int k, int p, uint64_t* G,
                                          int32_t* snew, int32_t* sold, int32_t* cnew,
                                          int32_t* cold, int lane, uint64_t e, int32_t& v_new,
                                          int32_t& v_old, int& cn, int& co) {
  // e = this lane's entry of the row (lanes >= k: anything)
  // entries numbered beyond n are frozen leftovers of an earlier merge: not sampled
  const bool valid = lane < k && (int64_t)entry_id(e) < n;
  const bool isnew = valid && (e & 1ull);
  const bool isold = valid && !(e & 1ull);
  const uint64_t mn = __ballot(isnew), mo = __ballot(isold);
  const int rn = __popcll(mn & lanes_below(lane)), ro = __popcll(mo & lanes_below(lane));
  const int32_t id = (int32_t)entry_id(e);
  const int L = 2 * p;
  v_new = v_old = -1;
  if (isnew && rn < p) {
    snew[s * L + rn] = id;
    G[s * k + lane] = e & ~1ull;
    v_new = id;
  }
  if (isold && ro < p) {
    sold[s * L + ro] = id;
    v_old = id;
  }
  cn = __popcll(mn) < p ? __popcll(mn) : p;
  co = __popcll(mo) < p ? __popcll(mo) : p;
  // the rest of the forward part reads "nothing", so that the scatter pass needs no counts
  if (lane >= cn && lane < p) snew[s * L + lane] = -1;
  if (lane >= co && lane < p) sold[s * L + lane] = -1;
  if (lane == 0) {
    cnew[s] = cn;
    cold[s] = co;
  }
}

// The same for a list of 65..128 entries, two per lane (e0 = entry lane, e1 =
// entry lane + 64 or 0): ranks run through the first register, then the second.
__device__ inline void forward_sample_row_wide(int64_t s, int64_t n, int k, int p, uint64_t* G,
                                               int32_t* snew, int32_t* sold, int32_t* cnew,
                                               int32_t* cold, int lane, uint64_t e0, uint64_t e1,
                                               int32_t (&v_new)[2], int32_t (&v_old)[2], int& cn,
                                               int& co) {
  const uint64_t e[2] = {e0, e1};
  uint64_t mn[2], mo[2];
  bool isnew[2], isold[2];
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const bool valid = lane + r * kWave < k && (int64_t)entry_id(e[r]) < n;
    isnew[r] = valid && (e[r] & 1ull);
    isold[r] = valid && !(e[r] & 1ull);
    mn[r] = __ballot(isnew[r]);
    mo[r] = __ballot(isold[r]);
  }
  const int L = 2 * p;
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int rn = (r ? __popcll(mn[0]) : 0) + __popcll(mn[r] & lanes_below(lane));
    const int ro = (r ? __popcll(mo[0]) : 0) + __popcll(mo[r] & lanes_below(lane));
    const int32_t id = (int32_t)entry_id(e[r]);
    v_new[r] = v_old[r] = -1;
    if (isnew[r] && rn < p) {
      snew[s * L + rn] = id;
      G[s * k + r * kWave + lane] = e[r] & ~1ull;
      v_new[r] = id;
    }
    if (isold[r] && ro < p) {
      sold[s * L + ro] = id;
      v_old[r] = id;
    }
  }
  const int tn = __popcll(mn[0]) + __popcll(mn[1]), to = __popcll(mo[0]) + __popcll(mo[1]);
  cn = tn < p ? tn : p;
  co = to < p ? to : p;
  if (lane >= cn && lane < p) snew[s * L + lane] = -1;
  if (lane >= co && lane < p) sold[s * L + lane] = -1;
  if (lane == 0) {
    cnew[s] = cn;
    cold[s] = co;
  }
}

// SUMS: also the proposal slots of the forward samples (see SegmentRule).
template <bool WIDE, bool SUMS>
__global__ __launch_bounds__(kSB) void k_fwd_count(int64_t n, int k, int p, BucketGeom g,
                                                   uint64_t* G, int32_t* snew, int32_t* sold,
                                                   int32_t* cnew, int32_t* cold,
                                                   uint32_t* wg_hist, uint32_t per_new,
                                                   uint32_t per_old, uint32_t* fwd_before,
                                                   uint64_t* group_before) {
  extern __shared__ uint32_t hist[];  // 2 nb, then the proposal slots of every row's samples
  __shared__ uint32_t wsum[kSB / kWave];
  uint32_t* const row_slots = hist + 2 * g.nb;
  for (int i = threadIdx.x; i < 2 * g.nb; i += kSB) hist[i] = 0;
  __syncthreads();
  const int lane = lane_id(), wave = wave_id();
  const int64_t row0 = (int64_t)blockIdx.x * g.rows_per_wg;
  const int64_t row1 = row0 + g.rows_per_wg < n ? row0 + g.rows_per_wg : n;
  constexpr int kRowsAtOnce = 4;  // rows in flight per wavefront
  constexpr int kStep = kRowsAtOnce * (kSB / kWave);
  for (int64_t s0 = row0 + wave; s0 < row1; s0 += kStep) {
    uint64_t e[kRowsAtOnce], e1[kRowsAtOnce];
#pragma unroll
    for (int r = 0; r < kRowsAtOnce; ++r) {
      const int64_t s = s0 + r * (kSB / kWave);
      e[r] = (s < row1 && lane < k) ? G[s * k + lane] : 0ull;
      if (WIDE) e1[r] = (s < row1 && lane + kWave < k) ? G[s * k + kWave + lane] : 0ull;
    }
#pragma unroll
    for (int r = 0; r < kRowsAtOnce; ++r) {
      const int64_t s = s0 + r * (kSB / kWave);
      if (s >= row1) break;
      int cn, co;
      if (WIDE) {
        int32_t vn[2], vo[2];
        forward_sample_row_wide(s, n, k, p, G, snew, sold, cnew, cold, lane, e[r], e1[r], vn, vo,
                                cn, co);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          if (vn[q] >= 0) atomicAdd(&hist[vn[q] >> g.tb], 1u);
          if (vo[q] >= 0) atomicAdd(&hist[g.nb + (vo[q] >> g.tb)], 1u);
        }
      } else {
        int32_t vn, vo;
        forward_sample_row(s, n, k, p, G, snew, sold, cnew, cold, lane, e[r], vn, vo, cn, co);
        if (vn >= 0) atomicAdd(&hist[vn >> g.tb], 1u);
        if (vo >= 0) atomicAdd(&hist[g.nb + (vo >> g.tb)], 1u);
      }
      if (SUMS && lane == 0) row_slots[s - row0] = per_new * (uint32_t)cn + per_old * (uint32_t)co;
    }
  }
  __syncthreads();
  // slots of the forward samples of the rows before each one: rows tid * per .. of this workgroup
  if (SUMS) {
    const int rows = (int)(row1 - row0), per = (g.rows_per_wg + kSB - 1) / kSB;
    const int r0 = threadIdx.x * per;
    uint32_t sum = 0;
    for (int i = 0; i < per; ++i) sum += r0 + i < rows ? row_slots[r0 + i] : 0u;
    uint32_t inc = sum;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
      const uint32_t o = __shfl_up(inc, off, kWave);
      if (lane >= off) inc += o;
    }
    if (lane == kWave - 1) wsum[wave] = inc;
    __syncthreads();
    uint32_t at = inc - sum;
    for (int w = 0; w < wave; ++w) at += wsum[w];
    for (int i = 0; i < per; ++i)
      if (r0 + i < rows) {
        const uint32_t own = row_slots[r0 + i];
        row_slots[r0 + i] = at;
        at += own;
      }
    if (threadIdx.x == kSB - 1) group_before[blockIdx.x] = at;
    __syncthreads();
    for (int i = threadIdx.x; i < rows; i += kSB) fwd_before[row0 + i] = row_slots[i];
  }
  // column blockIdx.x of the (bucket x workgroup) count matrix
  for (int i = threadIdx.x; i < 2 * g.nb; i += kSB) wg_hist[(size_t)i * gridDim.x + blockIdx.x] = hist[i];
}

// What the sampling stage keeps and clears before an iteration's cross-matching: the counters'
// values, the joins' node list lengths and region cursors.  By one workgroup of 256.
// Here too: whether the staged int8 join is to hand on every result it finds (DevState::forms) - if
// nearly all are expected to pass their thresholds, or two thirds of the results of the iteration before
// have (and this graph has had one: what the counters say of a graph that stood here earlier does not
// count).  In the first iteration of a merge 99.7 % and more pass; join and hand-out pass of it at
// 2 x 300,000 x 128 bytes, k = p = 32, 1.35 -> 1.17 ms, at 2 x 600,000 3.24 -> 2.68.
__device__ inline void begin_iteration(const uint64_t* counters, uint64_t* snap, uint64_t* forms,
                                       uint32_t* cls_count, unsigned long long* stg_cur,
                                       int expect) {
  __shared__ unsigned long long found, passed;
  if (threadIdx.x == 0) found = passed = 0ull;
  __syncthreads();
  for (int i = threadIdx.x; i < kStripes * C_SLOTS; i += kSB) {
    const uint64_t now = counters[i];
    const int slot = i % C_SLOTS;
    if (slot == C_PROPS) atomicAdd(&found, (unsigned long long)(now - snap[i]));
    if (slot == C_PASSED) atomicAdd(&passed, (unsigned long long)(now - snap[i]));
    snap[i] = now;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    forms[0] = FormTally::faded(forms[0]);
    forms[1] = expect == kExpectAll || (expect == kExpectAsBefore && 3 * passed >= 2 * found);
  }
  if (cls_count && threadIdx.x < kGramClasses) cls_count[threadIdx.x] = 0u;
  if (stg_cur)
    for (int i = threadIdx.x; i < kStageBuckets; i += kSB) stg_cur[i] = 0ull;
}

// Exclusive scan along every row of the (bucket x workgroup) count matrix: the
// entry of workgroup w becomes the start of w's run inside the bucket, the row
// total the bucket's size.  One wavefront per row - no atomics, and the edge
// order inside a bucket no longer depends on timing.  One workgroup more than
// the rows need keeps the counters' values from before this iteration, clears
// what the cross-matching adds to, and scans the workgroups' proposal slots.
__global__ __launch_bounds__(kSB) void k_wg_scan(int W, int rows, uint32_t* wg_hist,
                                                 uint32_t* bcnt, const uint64_t* counters,
                                                 uint64_t* snap, uint64_t* forms,
                                                 uint32_t* cls_count,
                                                 unsigned long long* stg_cur, int expect,
                                                 uint64_t* group_before) {
  if (blockIdx.x == gridDim.x - 1) {
    if (group_before && wave_id() == kSB / kWave - 1) {
      const int lane = lane_id();
      uint64_t carry = 0;
      for (int w0 = 0; w0 < W; w0 += kWave) {
        const uint64_t v = w0 + lane < W ? group_before[w0 + lane] : 0ull;
        uint64_t inc = v;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
          const uint64_t o = __shfl_up(inc, off, kWave);
          if (lane >= off) inc += o;
        }
        if (w0 + lane < W) group_before[w0 + lane] = carry + inc - v;
        carry += __shfl(inc, kWave - 1, kWave);
      }
    }
    begin_iteration(counters, snap, forms, cls_count, stg_cur, expect);
    return;
  }
  const int c = blockIdx.x * (kSB / kWave) + wave_id();
  if (c >= rows) return;
  const int lane = lane_id();
  uint32_t* row = wg_hist + (size_t)c * W;
  constexpr int kChunks = 4;  // chunks of 64 entries in flight
  uint32_t carry = 0;
  for (int w0 = 0; w0 < W; w0 += kChunks * kWave) {
    uint32_t v[kChunks];
#pragma unroll
    for (int r = 0; r < kChunks; ++r) {
      const int w = w0 + r * kWave + lane;
      v[r] = w < W ? row[w] : 0u;
    }
#pragma unroll
    for (int r = 0; r < kChunks; ++r) {
      const int w = w0 + r * kWave + lane;
      uint32_t inc = v[r];
#pragma unroll
      for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t o = __shfl_up(inc, off, kWave);
        if (lane >= off) inc += o;
      }
      if (w < W) row[w] = carry + inc - v[r];
      carry += __shfl(inc, kWave - 1, kWave);
    }
  }
  if (lane == 0) bcnt[c] = carry;
}

// Sum of one value per thread over a workgroup of 1024 threads (`wsum`: 16 words of LDS),
// and of those of the threads before this one.
__device__ inline uint64_t block_sum_1024(uint64_t v, uint64_t* wsum, uint64_t* before) {
  const int lane = lane_id(), wave = wave_id();
  uint64_t inc = v;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const uint64_t o = __shfl_up(inc, off, kWave);
    if (lane >= off) inc += o;
  }
  __syncthreads();
  if (lane == kWave - 1) wsum[wave] = inc;
  __syncthreads();
  uint64_t ahead = 0, total = 0;
#pragma unroll
  for (int w = 0; w < kCsrBlock / kWave; ++w) {
    ahead += w < wave ? wsum[w] : 0ull;
    total += wsum[w];
  }
  *before = ahead + inc - v;
  return total;
}

// Scatter pass.  A workgroup of 1024 threads takes its rows in batches of 256,
// sorts a batch's edges of one kind by bucket in LDS (count, scan, place), and
// copies them out in that order, so that the part of a batch that goes to one
// bucket leaves as one contiguous piece instead of one 8-byte store per edge to
// as many places (0.50 -> 0.24 ms per million nodes).
// PW threads serve a row (its up to PW forward samples of one kind): 32 for p <= 32, 64 beyond.
constexpr int kStBlock = 1024;
constexpr int kStEdges = 256 * 32;           // edges per batch: 256 rows of 32, or 128 rows of 64
constexpr int kStPasses = 8;                 // passes of kStBlock / PW rows make a batch

// PACKED: an edge leaves as one 32-bit word, (target inside its bucket) << (32 - tb) | source,
// which the sources of up to 2^(32 - tb) nodes fit; otherwise as (target, source).
template <int PW, bool PACKED>
__global__ __launch_bounds__(kStBlock) void k_fwd_scatter_staged(
    int64_t n, int p, BucketGeom g, const int32_t* snew, const int32_t* sold,
    const uint32_t* wg_hist, const uint32_t* bcnt, uint2* edges_new, uint2* edges_old) {
  __shared__ uint64_t scan_tmp[kStBlock / kWave];
  extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
  uint32_t* cursor = lds;               // 2 nb: where this workgroup writes next, per kind and bucket
  uint32_t* cnt = cursor + 2 * g.nb;    // nb: edges of the batch per bucket
  uint32_t* off = cnt + g.nb;           // nb + 1: their exclusive scan
  uint32_t* wsum = off + g.nb + 1;      // 16 wave totals of the scan
  uint2* stage = reinterpret_cast<uint2*>(lds + ((4 * g.nb + 17 + 3) & ~3));
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // start of this workgroup's run in every bucket: the sizes of the buckets before it plus the
  // run's start inside the bucket
  for (int kind = 0; kind < 2; ++kind) {
    uint32_t size[kMaxBuckets / kStBlock];
    const int per_thread = (g.nb + kStBlock - 1) / kStBlock, b0 = tid * per_thread;
    uint64_t sum = 0, at;
#pragma unroll
    for (int i = 0; i < kMaxBuckets / kStBlock; ++i) {
      size[i] = i < per_thread && b0 + i < g.nb ? bcnt[kind * g.nb + b0 + i] : 0u;
      sum += size[i];
    }
    block_sum_1024(sum, scan_tmp, &at);
#pragma unroll
    for (int i = 0; i < kMaxBuckets / kStBlock; ++i) {
      if (i < per_thread && b0 + i < g.nb) {
        const int c = kind * g.nb + b0 + i;
        cursor[c] = (uint32_t)at + wg_hist[(size_t)c * gridDim.x + blockIdx.x];
      }
      at += size[i];
    }
  }
  const int L = 2 * p;
  const int64_t row0 = (int64_t)blockIdx.x * g.rows_per_wg;
  const int64_t row1 = row0 + g.rows_per_wg < n ? row0 + g.rows_per_wg : n;
  const int per = (g.nb + kStBlock - 1) / kStBlock;  // buckets per thread in the scan (<= 4)
  constexpr int kRowsPerPass = kStBlock / PW, kStRows = kStPasses * kRowsPerPass;
  static_assert(kStRows * PW == kStEdges, "a batch fills the staging area");
  const int sub = tid & (PW - 1), rsel = tid / PW;     // entry of a row, row of a pass
  for (int64_t b0 = row0; b0 < row1; b0 += kStRows) {
    for (int kind = 0; kind < 2; ++kind) {
      const int32_t* list = kind ? sold : snew;
      uint2* edges = kind ? edges_old : edges_new;
      for (int i = tid; i < g.nb; i += kStBlock) cnt[i] = 0;
      __syncthreads();
      int32_t v[kStPasses];
      uint32_t rank[kStPasses];
#pragma unroll
      for (int q = 0; q < kStPasses; ++q) {
        const int64_t s = b0 + q * kRowsPerPass + rsel;
        v[q] = (s < row1 && sub < p) ? list[s * L + sub] : -1;
      }
#pragma unroll
      for (int q = 0; q < kStPasses; ++q)
        rank[q] = v[q] >= 0 ? atomicAdd(&cnt[(uint32_t)v[q] >> g.tb], 1u) : 0u;
      __syncthreads();
      // exclusive scan of cnt into off: `per` consecutive buckets per thread
      uint32_t mine = 0;
      for (int i = 0; i < per; ++i) {
        const int b = tid * per + i;
        mine += b < g.nb ? cnt[b] : 0u;
      }
      uint32_t inc = mine;
#pragma unroll
      for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t t = __shfl_up(inc, o, kWave);
        if (lane >= o) inc += t;
      }
      if (lane == kWave - 1) wsum[wave] = inc;
      __syncthreads();
      uint32_t before = 0;
      for (int w = 0; w < wave; ++w) before += wsum[w];
      uint32_t run = before + inc - mine;
      for (int i = 0; i < per; ++i) {
        const int b = tid * per + i;
        if (b < g.nb) {
          off[b] = run;
          run += cnt[b];
        }
      }
      if (tid == kStBlock - 1) off[g.nb] = run;
      __syncthreads();
#pragma unroll
      for (int q = 0; q < kStPasses; ++q)
        if (v[q] >= 0) {
          const int64_t s = b0 + q * kRowsPerPass + rsel;
          stage[off[(uint32_t)v[q] >> g.tb] + rank[q]] = make_uint2((uint32_t)v[q], (uint32_t)s);
        }
      __syncthreads();
      const uint32_t total = off[g.nb];
      for (uint32_t i = tid; i < total; i += kStBlock) {
        const uint2 rec = stage[i];
        const uint32_t b = rec.x >> g.tb;
        const uint32_t at = cursor[kind * g.nb + b] + (i - off[b]);
        if (PACKED)
          reinterpret_cast<uint32_t*>(edges)[at] =
              ((rec.x & ((1u << g.tb) - 1u)) << (32 - g.tb)) | rec.y;
        else
          edges[at] = rec;
      }
      __syncthreads();
      for (int i = tid; i < g.nb; i += kStBlock) cursor[kind * g.nb + i] += cnt[i];
      // (the next round's first barrier orders these updates before their use)
    }
  }
}

static size_t staged_lds_bytes(const BucketGeom& g) {
  return (size_t)((4 * g.nb + 17 + 3) & ~3) * 4 + (size_t)kStEdges * 8;
}

// One workgroup per (bucket, kind): counting sort of the bucket's edges by
// target.  LDS holds one counter per target of the bucket (dynamic size).
// AT_ONCE > 0 (packed edges, at most 2^10 targets): where the bucket has no more than `fit` <= 1024
// AT_ONCE edges, every thread keeps its edges and their ranks in registers, the sources are put in
// order in LDS behind the counters, and the run leaves as it will stand.  One store of 4 bytes to a
// place of its own per edge, 64 lines per instruction, was what the pass ran at, and it read every
// edge twice and counted it twice: 10^6 nodes, p = 32, 233 -> 95 us; 1.5 million 393 -> 141 us.
template <int AT_ONCE>
__global__ __launch_bounds__(kCsrBlock) void k_bucket_csr(int64_t n, BucketGeom g, uint32_t fit,
                                                          const uint32_t* bcnt,
                                                          const uint2* edges_new,
                                                          const uint2* edges_old,
                                                          uint64_t* roff_new, uint64_t* roff_old,
                                                          int32_t* csr_new, int32_t* csr_old) {
  constexpr bool PACKED = AT_ONCE > 0;
  extern __shared__ uint32_t cnt[];  // 2^tb counters, then running offsets; the sources in order
  __shared__ uint64_t scan_tmp[kCsrBlock / kWave];
  const int kind = blockIdx.y;
  const int b = blockIdx.x;
  const uint2* edges = kind ? edges_old : edges_new;
  uint64_t* roff = kind ? roff_old : roff_new;
  int32_t* csr = kind ? csr_old : csr_new;
  uint64_t before = 0, unused;  // the edges of the buckets before this one
  for (int i = threadIdx.x; i < b; i += kCsrBlock) before += bcnt[kind * g.nb + i];
  const uint64_t beg = block_sum_1024(before, scan_tmp, &unused);
  const uint32_t size = bcnt[kind * g.nb + b];
  const uint64_t end = beg + size;
  const bool fits = PACKED && size <= fit;
  const int T = 1 << g.tb;
  const uint32_t mask = (uint32_t)T - 1u;
  for (int i = threadIdx.x; i < T; i += kCsrBlock) cnt[i] = 0;
  __syncthreads();
  constexpr int kAtOnce = 8;  // edges in flight per thread
  const uint32_t* const words = reinterpret_cast<const uint32_t*>(edges);
  const int sh = 32 - g.tb;  // packed edge: target inside the bucket above, source below
  uint32_t word[PACKED ? AT_ONCE : 1], rank[PACKED ? AT_ONCE : 1];
  if (fits) {
#pragma unroll
    for (int r = 0; r < AT_ONCE; ++r)
      if ((uint32_t)r * kCsrBlock < size) {  // uniform
        const uint32_t e = (uint32_t)r * kCsrBlock + threadIdx.x;
        word[r] = words[beg + vmin(e, size - 1u)];
      }
#pragma unroll
    for (int r = 0; r < AT_ONCE; ++r)
      if ((uint32_t)r * kCsrBlock + threadIdx.x < size) rank[r] = atomicAdd(&cnt[word[r] >> sh], 1u);
  } else {
    for (uint64_t e0 = beg + threadIdx.x; e0 < end; e0 += kAtOnce * kCsrBlock) {
      uint32_t t[kAtOnce];
#pragma unroll
      for (int r = 0; r < kAtOnce; ++r) {
        const uint64_t e = e0 + (uint64_t)r * kCsrBlock;
        t[r] = e < end ? (PACKED ? words[e] >> sh : edges[e].x & mask) : 0xffffffffu;
      }
#pragma unroll
      for (int r = 0; r < kAtOnce; ++r)
        if (t[r] != 0xffffffffu) atomicAdd(&cnt[t[r]], 1u);
    }
  }
  __syncthreads();
  // exclusive scan over the T counters: T / 1024 consecutive counters per thread (fewer than
  // 1024: one each)
  const int lo = T > kCsrBlock ? (int)threadIdx.x * (T / kCsrBlock) : (int)threadIdx.x;
  const int per = T > kCsrBlock ? T / kCsrBlock : (lo < T ? 1 : 0);
  uint32_t sum = 0;
  for (int i = 0; i < per; ++i) sum += cnt[lo + i];
  uint64_t ahead;
  block_sum_1024(sum, scan_tmp, &ahead);
  uint32_t run = (uint32_t)ahead;
  const int64_t first = (int64_t)b << g.tb;
  for (int i = 0; i < per; ++i) {
    const uint32_t c = cnt[lo + i];
    cnt[lo + i] = run;  // start of the target's segment inside the bucket
    if (first + lo + i < n) roff[first + lo + i] = beg + run;
    run += c;
  }
  if (b == g.nb - 1 && threadIdx.x == 0) roff[n] = end;
  __syncthreads();
  if (fits) {
    uint32_t* const sorted = cnt + T;
#pragma unroll
    for (int r = 0; r < AT_ONCE; ++r)
      if ((uint32_t)r * kCsrBlock + threadIdx.x < size)
        sorted[cnt[word[r] >> sh] + rank[r]] = word[r] & ((1u << sh) - 1u);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < size; i += kCsrBlock) csr[beg + i] = (int32_t)sorted[i];
    return;
  }
  for (uint64_t e0 = beg + threadIdx.x; e0 < end; e0 += kAtOnce * kCsrBlock) {
    uint2 ed[kAtOnce];  // (target inside the bucket, source); target 0xffffffff: none
#pragma unroll
    for (int r = 0; r < kAtOnce; ++r) {
      const uint64_t e = e0 + (uint64_t)r * kCsrBlock;
      ed[r] = make_uint2(0xffffffffu, 0u);
      if (e < end) {
        if (PACKED) {
          const uint32_t w = words[e];
          ed[r] = make_uint2(w >> sh, w & ((1u << sh) - 1u));
        } else {
          const uint2 x = edges[e];
          ed[r] = make_uint2(x.x & mask, x.y);
        }
      }
    }
#pragma unroll
    for (int r = 0; r < kAtOnce; ++r)
      if (ed[r].x != 0xffffffffu) {
        const uint32_t pos = atomicAdd(&cnt[ed[r].x], 1u);
        csr[beg + pos] = (int32_t)ed[r].y;
      }
  }
}

// Small collections (sample_direct): forward sampling, a wavefront per row, and every sample's
// rank among its target's candidates.  One workgroup more begins the iteration.
template <bool WIDE>
__global__ __launch_bounds__(kSB) void k_fwd_direct(int64_t n, int k, int p, uint64_t* G,
                                                    int32_t* snew, int32_t* sold, int32_t* cnew,
                                                    int32_t* cold, uint32_t* degree,
                                                    uint32_t* rank, const uint64_t* counters,
                                                    uint64_t* snap, uint64_t* forms,
                                                    uint32_t* cls_count,
                                                    unsigned long long* stg_cur, int expect) {
  if (blockIdx.x == gridDim.x - 1) {
    begin_iteration(counters, snap, forms, cls_count, stg_cur, expect);
    return;
  }
  const int64_t s = (int64_t)blockIdx.x * (kSB / kWave) + wave_id();
  if (s >= n) return;
  const int lane = lane_id();
  const uint64_t e0 = lane < k ? G[s * k + lane] : 0ull;
  int32_t v[2][2] = {{-1, -1}, {-1, -1}};  // kind, register
  int cn, co;
  if (WIDE) {
    const uint64_t e1 = lane + kWave < k ? G[s * k + kWave + lane] : 0ull;
    forward_sample_row_wide(s, n, k, p, G, snew, sold, cnew, cold, lane, e0, e1, v[0], v[1], cn, co);
  } else {
    forward_sample_row(s, n, k, p, G, snew, sold, cnew, cold, lane, e0, v[0][0], v[1][0], cn, co);
  }
  uint32_t r[2][2];
#pragma unroll
  for (int kind = 0; kind < 2; ++kind)
#pragma unroll
    for (int q = 0; q < (WIDE ? 2 : 1); ++q)
      if (v[kind][q] >= 0) r[kind][q] = atomicAdd(&degree[kind * n + v[kind][q]], 1u);
#pragma unroll
  for (int kind = 0; kind < 2; ++kind) {
    int at = 0;  // samples stand in the list in the order of their entries
#pragma unroll
    for (int q = 0; q < (WIDE ? 2 : 1); ++q) {
      const uint64_t taken = __ballot(v[kind][q] >= 0);
      if (v[kind][q] >= 0) rank[(kind * n + s) * p + at + rank_in(taken)] = r[kind][q];
      at += __popcll(taken);
    }
  }
}

// The candidates of one kind (blockIdx.y) to their places.  Every workgroup scans all degrees for
// itself (in LDS), then places its share of the samples.
constexpr int kPlaceBlock = 1024;
__global__ __launch_bounds__(kPlaceBlock) void k_place_direct(
    int64_t n, int p, const int32_t* snew, const int32_t* sold, const uint32_t* degree,
    const uint32_t* rank, uint64_t* roff_new, uint64_t* roff_old, int32_t* csr_new,
    int32_t* csr_old) {
  static_assert(kPlaceBlock == kCsrBlock, "block_sum_1024");
  __shared__ uint32_t off[kDirectNodes];
  __shared__ uint64_t scan_tmp[kPlaceBlock / kWave];
  const int kind = blockIdx.y, N = (int)n;
  const int32_t* list = kind ? sold : snew;
  uint64_t* roff = kind ? roff_old : roff_new;
  int32_t* csr = kind ? csr_old : csr_new;
  degree += kind * n;
  rank += kind * n * p;
  for (int i = threadIdx.x; i < N; i += kPlaceBlock) off[i] = degree[i];
  __syncthreads();
  const int per = (N + kPlaceBlock - 1) / kPlaceBlock, first = threadIdx.x * per;
  uint64_t sum = 0, before;
  for (int i = first; i < first + per && i < N; ++i) sum += off[i];
  const uint64_t all = block_sum_1024(sum, scan_tmp, &before);
  uint32_t at = (uint32_t)before;
  for (int i = first; i < first + per && i < N; ++i) {
    const uint32_t own = off[i];
    off[i] = at;
    at += own;
  }
  __syncthreads();
  const int step = gridDim.x * kPlaceBlock, own = blockIdx.x * kPlaceBlock + threadIdx.x;
  for (int i = own; i < N; i += step) roff[i] = off[i];
  if (own == 0) roff[N] = all;
  const float inv_p = 1.0f / (float)p;  // ((e + 0.5) / p < 2^14 is 1 / 128 off the next number)
  for (int e = own; e < N * p; e += step) {
    const int s = (int)(((float)e + 0.5f) * inv_p);
    const int32_t v = list[(int64_t)s * 2 * p + (e - s * p)];
    if (v >= 0) csr[off[v] + rank[e]] = s;
  }
}

hipError_t launch_sample_direct(const Shape& sh, const DevState& ds, Expect expect, hipStream_t st) {
  // (the proposal array is not in use yet: 2 n p ranks in its 6 n p words or more)
  uint32_t* rank = reinterpret_cast<uint32_t*>(ds.bins);
  const unsigned grid = (unsigned)((sh.n + kSB / kWave - 1) / (kSB / kWave)) + 1;
  auto* const fwd = sh.k > kWave ? k_fwd_direct<true> : k_fwd_direct<false>;
  fwd<<<grid, kSB, 0, st>>>(sh.n, sh.k, sh.p, ds.G, ds.snew, ds.sold, ds.cnew, ds.cold, ds.degree,
                            rank, ds.counters, ds.snap, ds.forms, ds.cls_count, ds.stg_cur,
                            expect);
  const int64_t blocks = (sh.n * sh.p + kPlaceBlock - 1) / kPlaceBlock;
  k_place_direct<<<dim3((unsigned)blocks, 2), kPlaceBlock, 0, st>>>(
      sh.n, sh.p, ds.snew, ds.sold, ds.degree, rank, ds.roff_new, ds.roff_old, ds.csr_new,
      ds.csr_old);
  return hipGetLastError();
}

// Edges per thread of the two builds of k_bucket_csr for packed edges (tb <= 10).  12 leave room for
// two workgroups per CU, 36 (with the counters 148 KB of LDS) for one.  p >= 37 beyond 2^19 nodes: while
// nearly all samples are of one kind the buckets hold more and are swept twice, one workgroup per CU
// instead of two; the sampling stage then takes what it took with less LDS and no registers for edges
// (first iteration, 600,000 nodes, p = 42 1.25 / 1.26 ms, p = 64 1.43 / 1.42; 2 million, p = 42 4.38 /
// 4.23), and less as soon as the kinds are mixed (fourth 1.50 / 1.29, 1.45 / 1.39, 4.48 / 4.02).
constexpr int kFewEdges = 12, kManyEdges = 36;
// The bucket layout for n <= 2^27 targets: at most 4096 buckets of 2^tb <= 2^15 targets (one
// workgroup's LDS counts a bucket's targets).  Small collections take smaller buckets and
// fewer rows per workgroup, so that their passes still spread over the chip: buckets of 256
// targets up to 2^18 nodes, of 1024 from 2^19 on, and 512 workgroups (one round of the scatter
// pass, two workgroups per CU) of at least 32 rows up to 2^19 nodes, 1024 beyond.  Sampling
// stage in microseconds, this layout / buckets of 1024 and workgroups of at least 256 rows:
// 4096 nodes 42 / 69, 30,000 nodes 90 / 119, 100,000 nodes 142 / 145; 512 / 1024 workgroups:
// 100,000 nodes 142 / 155, 600,000 nodes 776 / 757, 10^6 nodes 1273 / 1212.
static BucketGeom bucket_geom(int64_t n) {
  BucketGeom g{8, 0, 32};
  auto buckets = [&] { return (n + (1ll << g.tb) - 1) >> g.tb; };
  while (g.tb < 10 && buckets() > 1024) ++g.tb;
  while (buckets() > kMaxBuckets) ++g.tb;
  g.nb = (int)buckets();
  // the (bucket x workgroup) counts lie behind the edges in the proposal array, which leaves
  // 8 words per node even for p = 1: two kinds x buckets x workgroups <= 8 n
  const int64_t workgroups = n <= (1 << 19) ? 512 : 1024;
  while (g.rows_per_wg < 4096 &&
         (g.rows_per_wg * workgroups < n ||
          (n + g.rows_per_wg - 1) / g.rows_per_wg * g.nb > 4 * n))
    g.rows_per_wg += 32;
  return g;
}

hipError_t launch_sample_buckets(const Shape& sh, const DevState& ds, Expect expect,
                                 int* group_rows, hipStream_t st) {
  const BucketGeom g = bucket_geom(sh.n);
  *group_rows = g.rows_per_wg;
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipSuccess;
    const void* kernels[3] = {reinterpret_cast<const void*>(k_bucket_csr<0>),
                              reinterpret_cast<const void*>(k_bucket_csr<kFewEdges>),
                              reinterpret_cast<const void*>(k_bucket_csr<kManyEdges>)};
    const int most[3] = {4 << 15, (kFewEdges + 1) * kCsrBlock * 4, (kManyEdges + 1) * kCsrBlock * 4};
    for (int i = 0; i < 3 && e == hipSuccess; ++i)
      e = hipFuncSetAttribute(kernels[i], hipFuncAttributeMaxDynamicSharedMemorySize, most[i]);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  uint32_t* bcnt = ds.bk_cnt;
  uint2* edges_new = reinterpret_cast<uint2*>(ds.bins);
  uint2* edges_old = edges_new + sh.n * sh.p;
  // per-workgroup bucket histograms, behind the edges in the same (still unused) array
  uint32_t* wg_hist = reinterpret_cast<uint32_t*>(edges_old + sh.n * sh.p);
  const unsigned grid = (unsigned)((sh.n + g.rows_per_wg - 1) / g.rows_per_wg);
  const bool sums = sh.n > kRoomForAll;
  const size_t lds = (size_t)(2 * g.nb + (sums ? g.rows_per_wg : 0)) * 4;
#define GNND_FWD(WIDE, SUMS)                                                                    \
  k_fwd_count<WIDE, SUMS><<<grid, kSB, lds, st>>>(                                              \
      sh.n, sh.k, sh.p, g, ds.G, ds.snew, ds.sold, ds.cnew, ds.cold, wg_hist,                   \
      (uint32_t)sh.slots_new_per_appearance(), (uint32_t)sh.slots_old_per_appearance(),         \
      ds.fwd_before, ds.group_before)
  if (sh.k > kWave) {
    if (sums) GNND_FWD(true, true);
    else GNND_FWD(true, false);
  } else {
    if (sums) GNND_FWD(false, true);
    else GNND_FWD(false, false);
  }
#undef GNND_FWD
  k_wg_scan<<<(unsigned)((2 * g.nb + kSB / kWave - 1) / (kSB / kWave)) + 1, kSB, 0, st>>>(
      (int)grid, 2 * g.nb, wg_hist, bcnt, ds.counters, ds.snap, ds.forms,
      ds.cls_count, ds.stg_cur, expect, sums ? ds.group_before : nullptr);
  static bool staged_attr = false;
  if (!staged_attr) {
    hipError_t e = hipSuccess;
    const void* kernels[4] = {reinterpret_cast<const void*>(k_fwd_scatter_staged<32, false>),
                              reinterpret_cast<const void*>(k_fwd_scatter_staged<32, true>),
                              reinterpret_cast<const void*>(k_fwd_scatter_staged<64, false>),
                              reinterpret_cast<const void*>(k_fwd_scatter_staged<64, true>)};
    for (int i = 0; i < 4 && e == hipSuccess; ++i)
      e = hipFuncSetAttribute(kernels[i], hipFuncAttributeMaxDynamicSharedMemorySize, 144 << 10);
    if (e != hipSuccess) return e;
    staged_attr = true;
  }
  // one 32-bit word per edge where the source ids fit beside the target's place in its bucket
  const bool packed = sh.n <= ((int64_t)1 << (32 - g.tb));
#define GNND_SCATTER(PW, PK)                                                            \
  k_fwd_scatter_staged<PW, PK><<<grid, kStBlock, staged_lds_bytes(g), st>>>(            \
      sh.n, sh.p, g, ds.snew, ds.sold, wg_hist, bcnt, edges_new, edges_old)
  if (sh.p <= 32) {
    if (packed) GNND_SCATTER(32, true);
    else GNND_SCATTER(32, false);
  } else {
    if (packed) GNND_SCATTER(64, true);
    else GNND_SCATTER(64, false);
  }
#undef GNND_SCATTER
#define GNND_CSR(AT_ONCE, FIT)                                                                    \
  k_bucket_csr<AT_ONCE>                                                                           \
      <<<dim3((unsigned)g.nb, 2), kCsrBlock, ((size_t)4 << g.tb) + (size_t)(FIT) * 4, st>>>(        \
          sh.n, g, (uint32_t)(FIT), bcnt, edges_new, edges_old, ds.roff_new, ds.roff_old,           \
          ds.csr_new, ds.csr_old)
  // what an average bucket holds when all samples are of one kind, and an eighth more
  const int64_t many = ((int64_t)sh.p << g.tb) + ((int64_t)sh.p << g.tb >> 3);
  if (!packed) GNND_CSR(0, 0);
  else if (many <= kFewEdges * kCsrBlock) GNND_CSR(kFewEdges, kFewEdges * kCsrBlock);
  else GNND_CSR(kManyEdges, kManyEdges * kCsrBlock);
#undef GNND_CSR
  return hipGetLastError();
}

}  // namespace gnnd

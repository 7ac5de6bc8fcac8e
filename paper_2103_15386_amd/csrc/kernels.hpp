// Host-callable launchers of the GNND kernels (one per pipeline stage) and the
// device-pointer bundle they work on.  Every launcher enqueues on `st` and
// returns the hipGetLastError() of its launches.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gnnd {

enum : int {
  C_INSERTS = 0, C_EVALS = 1, C_SUMNEW = 2, C_SUMOLD = 3, C_PROPS = 4,
  C_OVERFLOW = 5,  // proposals that found their destination segment full (must stay 0)
  C_PASSED = 6,    // results that survived the early drop and went to the update
  C_SLOTS = 8
};
constexpr int kStripes = 64;  // counters are striped to spread same-address atomics

// One 64-bit word per destination serves the hand-out of results: the low
// kSlotCountBits bits count the results received so far, the rest is the first
// slot of the destination's segment.  A single returning atomic add yields both.
constexpr int kSlotCountBits = 24;
constexpr uint64_t kSlotCountMask = (1ull << kSlotCountBits) - 1;

// What the join gathers per sampled object besides its vector, kept small (8
// bytes, 8 MB per million nodes) so that the array stays cache resident: the
// distance code of its list's last entry (nothing farther can enter) and the
// squared norm of its int8 row (int8 join) or the bits of the float32 squared
// norm of its row (float32 matrix-core join).
struct alignas(8) NodeMeta {
  uint32_t kth;
  int32_t norm;
};

// Everything lives in the caller's workspace; sizes in elements.
struct DevState {
  uint64_t* G;         // n*k packed entries, row per node, ascending
  NodeMeta* meta;      // n: per-node record gathered by the join (see NodeMeta)
  int32_t* snew;       // n*2p NEW sample lists
  int32_t* sold;       // n*2p OLD sample lists
  int32_t* cnew;       // n list sizes
  int32_t* cold;       // n
  uint64_t* roff_new;  // n+1 offsets into csr_new
  uint64_t* roff_old;  // n+1
  int32_t* csr_new;    // n*p reverse candidates grouped by target
  int32_t* csr_old;    // n*p
  uint64_t* pslot;     // n: (segment start << 24) | proposals received; rewritten by every sampling
  uint64_t* poff;      // n+1 segment offsets into bins (see SegmentRule)
  uint32_t* degree;        // sample_direct(): 2 n reverse degrees, NEW then OLD; 0 between samplings
  uint32_t* fwd_before;    // n: see SegmentRule
  uint64_t* group_before;  // n / 32 + 1: one per workgroup of the forward sampling
  uint64_t* bins;      // n*6p packed proposals, one segment per destination
  uint64_t* counters;  // kStripes * C_SLOTS
  uint64_t* snap;      // the counters as the current iteration's sampling stage found them
  uint64_t* forms;     // [0] joins with a faster first form: how it has gone so far (see FormTally);
                       // [1] not 0: the staged int8 join hands on every result (see begin_iteration)
  uint64_t* aside;     // merge only: n * floor(k/2) set-aside entries
  int8_t* shadow;      // matrix-core path: n rows of dpad int8 (value - 128), zero padded
  uint32_t* bk_cnt;    // 2 x 4096 bucket sizes of the bucketed reverse-candidate sort
  // staged hand-out of the matrix-core join (NULL when results are handed on one by one):
  // results leave the join grouped by bucket of destinations, then a second pass moves
  // them into the destinations' segments of `bins`
  uint64_t* stg_ent;   // slots: staged results (see stage_record), bucket regions laid out like bins
  unsigned long long* stg_cur;  // kStageBuckets: results that have reached each bucket region
  // float32 matrix-core join (NULL when it is not in use): the nodes that have work to do, listed
  // per class of node - kGramClasses lists of n places - and the lists' lengths
  int32_t* cls_nodes;
  uint32_t* cls_count;
  // float32 matrix-core join: 16-bit copies of the rows divided by their norms (NULL: it reads
  // the float32 rows twice instead), and the largest relative error of a copy (float bits)
  void* half_rows;
  uint32_t* half_info;
};
// Elements per 16-bit row: whole steps of 32.
inline int64_t half_row_elems(int32_t d) { return ((int64_t)d + 31) & ~(int64_t)31; }
constexpr int kGramClasses = 7;

// What is known, when an iteration begins, of how many of its results will pass the thresholds of
// their lists (see begin_iteration): they will be about as many as in the iteration before, nearly all
// of them (the lists hold random objects: a fresh random graph, or half of every list when a merge
// begins), or nothing (a loaded graph).
enum Expect : int { kExpectAsBefore, kExpectAll, kExpectUnknown };

// Staged hand-out: destinations are cut into at most kStageBuckets buckets of 2^tb
// consecutive ids; a workgroup of the join keeps kStageSlots results per bucket in LDS.
// A staged result is one 64-bit word: squared distance (23: at most 128 x 255^2) | destination
// inside its bucket (19, of which at most 14 are in use) | object id (22), which is what limits
// the staged form to 2^22 nodes.
constexpr int kStageBuckets = 256;
constexpr int kStageSlots = 64;
constexpr int kStageIdBits = 22, kStageDistShift = 41;
constexpr int64_t kStageMaxNodes = (int64_t)1 << kStageIdBits;
inline int stage_bucket_bits(int64_t n) {
  int tb = 0;
  while (((n + ((int64_t)1 << tb) - 1) >> tb) > kStageBuckets) ++tb;
  return tb;
}

struct Shape {
  int64_t n;
  int32_t d, k, p, metric;
  int64_t split;  // merge: first id of the second set; otherwise n
  const void* vec_a;
  const void* vec_b;
  int32_t all_pairs;  // 1: every evaluated pair is proposed (ablation), 0: nearest partners only
  const float* norms = nullptr;  // squared norm per node, where metric or join need it
  int32_t segments = 1;  // > 1: the list is k / 32 segments, object v lives in segment v % segments
  // slots of the proposal array: per appearance in a NEW list two results (all pairs: one per
  // possible partner, 2 * 2p - 1), in an OLD list one (all pairs: 2p); at most 2np appearances each
  __host__ __device__ int64_t slots_new_per_appearance() const {
    return all_pairs ? 4 * p - 1 : 2;
  }
  __host__ __device__ int64_t slots_old_per_appearance() const { return all_pairs ? 2 * p : 1; }
  __host__ __device__ int64_t slots() const {
    return n * 2 * p * (slots_new_per_appearance() + slots_old_per_appearance());
  }
};

__device__ inline void counter_add(uint64_t* counters, int which, int64_t stripe_hint,
                                   uint64_t v) {
  atomicAdd(reinterpret_cast<unsigned long long*>(
                counters + (stripe_hint & (kStripes - 1)) * C_SLOTS + which),
            (unsigned long long)v);
}

// One segment of the proposal array per destination, one behind the other.  Node v can only sit in
// the sample list of a node that holds v as a forward sample (its reverse degree of them) or that v
// holds as one, which bounds the number of joins it takes part in and with them the results it can
// receive: per_new per join as a NEW sample, per_old per join as an OLD one.  Where a segment
// starts follows from v's places in the two candidate arrays (the reverse degrees of all nodes
// before it) and from the forward samples of the nodes before it.  Two launches of a scan over the
// bounds stood here before: 7 us per iteration at 4096 nodes, 19 at 10^6.
// Up to kRoomForAll nodes p forward samples are counted for every node, which needs no sums (all
// segments together then fill the array); beyond, the forward sampling adds up the actual numbers
// per workgroup (k_fwd_count, k_wg_scan), because longer segments cost the passes over the
// proposals more than the sums cost.
constexpr int64_t kRoomForAll = 1 << 18;
struct SegmentRule {
  uint32_t per_new, per_old;
  uint32_t per_node;            // slots for p forward samples of either kind; 0: the actual number
  uint32_t inverse;             // see group_of
  const uint32_t* fwd_before;   // slots for the forward samples of the nodes before v in its group
  const uint64_t* group_before; // ... of the groups before this one
  SegmentRule(const Shape& sh, const DevState& ds, int group_rows)
      : per_new((uint32_t)sh.slots_new_per_appearance()),
        per_old((uint32_t)sh.slots_old_per_appearance()),
        per_node(sh.n <= kRoomForAll ? (uint32_t)sh.p * (per_new + per_old) : 0u),
        inverse((uint32_t)((((uint64_t)1 << 32) + (group_rows >> 5) - 1) / (group_rows >> 5))),
        fwd_before(ds.fwd_before), group_before(ds.group_before) {}
  // v / group_rows: a group is a multiple of 32 rows, at most 4096, and v below 2^27, so that the
  // product with the reciprocal, rounded up, is exact (groups of 32: the reciprocal is 2^32)
  __device__ uint32_t group_of(int64_t v) const {
    const uint32_t v32 = (uint32_t)(v >> 5);
    return inverse ? __umulhi(v32, inverse) : v32;
  }
  // Slots for the forward samples of the nodes before v.
  __device__ uint64_t before(int64_t v) const {
    return per_node ? (uint64_t)v * per_node : fwd_before[v] + group_before[group_of(v)];
  }
  // Node v's offset `at` and its slot word (nothing received yet); `rev`, `fwd`: slots for its
  // reverse candidates and its forward samples.  The last node closes the offsets.
  __device__ void write(int64_t v, int64_t n, uint64_t at, uint64_t rev, uint64_t fwd,
                        uint64_t* poff, uint64_t* pslot, uint64_t* counters) const {
    const uint64_t size = rev + fwd;
    poff[v] = at;
    pslot[v] = at << kSlotCountBits;
    if (v == n - 1) poff[n] = at + (per_node ? rev + per_node : size);
    // more results than the count field of the slot word can hold: reported
    if (size > kSlotCountMask) counter_add(counters, C_OVERFLOW, v, size);
  }
};

// Small collections are sampled without the bucketed sort: a returning atomic per edge gives it
// its rank among its target's candidates, and one scan per workgroup of the placing pass their
// offsets: two launches instead of four, until the atomics' rate (12 per ns) tells.  Sampling
// stage of an iteration in microseconds, direct / bucketed: 3000 nodes, p = 32: 30 / 39; 6000, 32:
// 40 / 43; 8192, 32: 56 / 45; 8192, 16: 39 / 42; 12,000, 8: 38 / 50; 16,000, 8: 53 / 53.
constexpr int64_t kDirectNodes = 12288;  // their offsets fit 48 KB of LDS
inline bool sample_direct(int64_t n, int32_t p) {
  return n <= kDirectNodes && n * p <= (1 << 17);
}

// Grid of `blocks` workgroups, folded into two dimensions beyond 2^22 (device side:
// block_linear()); the fold may add up to 2^22 - 1 workgroups past the end.
inline dim3 grid_blocks(int64_t blocks) {
  constexpr int64_t kRow = (int64_t)1 << 22;
  if (blocks <= kRow) return dim3((unsigned)(blocks > 0 ? blocks : 1));
  return dim3((unsigned)kRow, (unsigned)((blocks + kRow - 1) / kRow));
}

hipError_t launch_init_random(const Shape& sh, const DevState& ds, uint64_t seed, hipStream_t st);
// squared norms of all rows, one fused multiply-add per dimension in dimension order; with `meta`
// also into the nodes' records (the float's bits in `norm`), where the float32 matrix-core join
// reads them
hipError_t launch_row_norms(const Shape& sh, float* norms, NodeMeta* meta, hipStream_t st);
hipError_t launch_sample(const Shape& sh, const DevState& ds, uint64_t seed, uint32_t iter,
                         Expect expect, hipStream_t st);
hipError_t launch_join(const Shape& sh, const DevState& ds, int path, bool merge_mode,
                       hipStream_t st);
// The 16-bit copies of the rows into ds.half_rows (ds.half_info is 0 before), and (cosine: not; sh.norms must be set) the
// squared norms in the NodeMeta records
hipError_t launch_half_rows(const Shape& sh, const DevState& ds, hipStream_t st);
// float32 vectors, metrics that are functions of an inner product and the norms (sh.norms
// must be set): inner products on the matrix cores, canonical distances for the results
hipError_t launch_join_gram(const Shape& sh, const DevState& ds, bool merge_mode, hipStream_t st);
// results are staged per bucket when ds.stg_ent is set, handed on one by one otherwise;
// `after_join` (may be NULL) is recorded behind the cross-matching kernel, in front of the
// pass that moves staged results into the destinations' segments.  `first_look`: the graph is
// a fresh random one (first iteration); results handed on one by one then do not look at the lists'
// thresholds, which is left to the update; same graph with or without it
hipError_t launch_join_mfma(const Shape& sh, const DevState& ds, bool merge_mode, bool first_look,
                            hipStream_t st, hipEvent_t after_join = nullptr);
hipError_t launch_pack_i8(const Shape& sh, const DevState& ds, int* bad_flag_dev, hipStream_t st);
hipError_t launch_init_random_i8(const Shape& sh, const DevState& ds, uint64_t seed,
                                 hipStream_t st);
// (also takes the snapshot of the counters and clears the joins' node list lengths and region
// cursors: the first stage of an iteration).  `group_rows`: rows per workgroup of the forward
// sampling (see SegmentRule).
hipError_t launch_sample_buckets(const Shape& sh, const DevState& ds, Expect expect,
                                 int* group_rows, hipStream_t st);
// the same where sample_direct() says so; the reverse selection then clears ds.degree
hipError_t launch_sample_direct(const Shape& sh, const DevState& ds, Expect expect, hipStream_t st);
// sample lists of 65..128 objects (p > 32): reverse selection and the join for long lists
hipError_t launch_rev_select_long(const Shape& sh, const DevState& ds, uint64_t seed,
                                  uint32_t iter, int group_rows, uint32_t* clear, hipStream_t st);
hipError_t launch_join_long(const Shape& sh, const DevState& ds, bool merge_mode, hipStream_t st);
// the same on byte-valued data of up to 128 dimensions (int8 rows in ds.shadow)
hipError_t launch_join_long_i8(const Shape& sh, const DevState& ds, bool merge_mode,
                               hipStream_t st);
hipError_t launch_update(const Shape& sh, const DevState& ds, hipStream_t st);
// lists of 65..128 entries (two per lane); the launchers above forward to these
hipError_t launch_init_random_wide(const Shape& sh, const DevState& ds, uint64_t seed,
                                   hipStream_t st);
// on the int8 rows (exact integers either way)
hipError_t launch_init_random_wide_i8(const Shape& sh, const DevState& ds, uint64_t seed,
                                      hipStream_t st);
hipError_t launch_update_wide(const Shape& sh, const DevState& ds, hipStream_t st);
// segmented lists (sh.segments > 1); the launchers above forward to these as well
hipError_t launch_init_random_segmented(const Shape& sh, const DevState& ds, uint64_t seed,
                                        hipStream_t st);
hipError_t launch_update_segmented(const Shape& sh, const DevState& ds, hipStream_t st);
hipError_t launch_get_graph(const Shape& sh, const DevState& ds, int32_t* ids, void* dist,
                            uint8_t* isnew, int32_t id_offset, hipStream_t st);
hipError_t launch_set_graph(const Shape& sh, const DevState& ds, const int32_t* ids,
                            const void* dist, const uint8_t* isnew, int* bad_flag_dev,
                            hipStream_t st);
hipError_t launch_get_proposals(const Shape& sh, const DevState& ds, int32_t* u, int32_t* v,
                                void* dist, hipStream_t st);
struct MergeIds;
hipError_t launch_merge_init(const Shape& sh, const DevState& ds, uint64_t seed,
                             const MergeIds& mi, const int32_t* ids1, const void* dist1,
                             const int32_t* ids2, const void* dist2, hipStream_t st);
hipError_t launch_merge_final(const Shape& sh, const DevState& ds, const MergeIds& mi,
                              int32_t* ids_out, void* dist_out, hipStream_t st);
// the same on the int8 rows of the matrix-core path (exact integers either way)
hipError_t launch_merge_init_i8(const Shape& sh, const DevState& ds, uint64_t seed,
                                const MergeIds& mi, const int32_t* ids1, const void* dist1,
                                const int32_t* ids2, const void* dist2, hipStream_t st);
hipError_t launch_merge_init_wide(const Shape& sh, const DevState& ds, uint64_t seed,
                                  const MergeIds& mi, const int32_t* ids1, const void* dist1,
                                  const int32_t* ids2, const void* dist2, hipStream_t st);
hipError_t launch_merge_final_wide(const Shape& sh, const DevState& ds, const MergeIds& mi,
                                   int32_t* ids_out, void* dist_out, hipStream_t st);
hipError_t launch_exact_knn(const void* vec, int64_t n, int32_t d, int32_t metric,
                            const int32_t* queries, int64_t nq, int32_t K, int32_t* ids_out,
                            void* dist_out, hipStream_t st, const uint8_t* only = nullptr);
// Queries per workgroup of k_exact_knn: one workgroup fills a CU and reads all rows once, so the
// time is the number of rounds of 256 workgroups times what a round takes - Q distances per row
// plus moving the row through LDS, about as much as two.
inline int exact_rounds(int64_t nq, int queries) {
  return (int)(((nq + queries - 1) / queries + 255) / 256);
}
inline int exact_queries(int64_t nq) {
  int best = 1;
  for (int c = 2; c <= 8; c *= 2)
    if ((int64_t)exact_rounds(nq, c) * (c + 2) < (int64_t)exact_rounds(nq, best) * (best + 2)) best = c;
  return best;
}
// The same results with the matrix cores turning rows away (exact_scan.hip), in a workspace of
// exact_scan_bytes() bytes; 0: this form does not take such a call.  (launch_exact_knn answers the
// queries it leaves over: those with only[q] == 1.)
size_t exact_scan_bytes(int64_t n, int32_t d, int32_t metric, int64_t nq, int32_t K);
hipError_t launch_exact_scan(const void* vec, int64_t n, int32_t d, int32_t metric,
                             const int32_t* queries, int64_t nq, int32_t K, int32_t* ids_out,
                             void* dist_out, void* workspace, hipStream_t st);
hipError_t launch_zero_u32(uint32_t* p, size_t count, hipStream_t st);

}  // namespace gnnd

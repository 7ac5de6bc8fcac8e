// Graph-side kernels of GNND for gfx950: random initial lists, sampling with
// reverse neighbours, the list update, and the copy-in / copy-out helpers.
// One 64-lane wavefront owns one list: a list entry, a sample or a proposal
// lives in one lane, and sorting / merging / compaction are lane networks.
#include "device_utils.hpp"
#include "kernels.hpp"

namespace gnnd {

constexpr int kBlock = 256;
constexpr int kWavesPerBlock = kBlock / kWave;

__device__ inline int64_t wave_global_index() {
  return block_linear() * kWavesPerBlock + wave_id();
}
static inline dim3 blocks_for_waves(int64_t waves) {
  return grid_blocks((waves + kWavesPerBlock - 1) / kWavesPerBlock);
}

// ---------------------------------------------------------------------------
// Alg. 1, first loop: k distinct random neighbours per node, distances, sorted
// ascending by (distance, id), flagged NEW.
template <int METRIC>
__global__ __launch_bounds__(kBlock) void k_init_random(VecSrc vs, int64_t n, int k,
                                                        uint64_t base_hash, uint64_t* G,
                                                        NodeMeta* meta) {
  __shared__ uint32_t tile[kWavesPerBlock][kEvalTileWords];
  const int64_t s = wave_global_index();
  if (s >= n) return;
  const int lane = lane_id();
  uint32_t id = draw_distinct(base_hash, (uint32_t)s, k, (uint32_t)n, 0u, (uint32_t)s, lane);
  const uint32_t code =
      wave_distances<METRIC>(vs, (uint32_t)s, id, lane < k, tile[wave_id()], lane);
  uint64_t e = lane < k ? make_entry(code, id, 1u) : kKeyMax;
  e = wave_sort(e, lane);
  if (lane < k) G[s * k + lane] = e;
  if (lane == k - 1) meta[s].kth = entry_code(e);
}

// ---------------------------------------------------------------------------
// What the reverse candidates of v are ranked by: hash(seed, kind, v, s, iter), ties by s.
__device__ inline uint64_t select_key(uint64_t base, int64_t v, uint32_t s, uint32_t iter) {
  return ((hash3(base, (uint32_t)v, s, iter) >> 32) << 32) | (uint64_t)s;
}

// Sec. 4.1, reverse part and duplicate removal for one list.  `fwd` is the forward part (its nf
// samples in the first lanes, kNoId in all others), `first` the first 64 of the deg reverse
// candidates, candidate j in lane (nf + j) % 64 (kNoId where there is none).  Of the candidates the
// 2p - nf with the smallest hash(seed, kind, v, s, iter) (ties by s) are appended - the
// paper's "append until the list is full" with the winners chosen by a hash
// instead of by thread timing.  The list is then sorted by id, duplicates are
// dropped and it is written back with -1 behind its end.  Returns its size.
// (the list is sorted by id in any case, so only which candidates win has to be found out)
constexpr uint32_t kNoId = 0xffffffffu;
__device__ __forceinline__ int select_list(int64_t v, int p, uint64_t base, uint32_t iter,
                                           int32_t* list, uint32_t fwd, int nf, const int32_t* csr,
                                           uint64_t beg, uint32_t deg, uint32_t first, int lane) {
  const int room = 2 * p - nf;
  uint32_t val;
  int total = 2 * p;
  auto hash_of = [&](uint32_t s) { return (uint32_t)(select_key(base, v, s, iter) >> 32); };
  if (deg <= (uint32_t)room) {  // the candidates stand in the lanes behind the forward part
    val = vmin(fwd, first);
    total = nf + (int)deg;
  } else {
    bool chosen = false;
    if (deg <= (uint32_t)kWave) {
      const uint32_t h[1] = {hash_of(first)};
      const uint64_t have[1] = {__ballot(first != kNoId)};
      uint64_t win[1];
      chosen = choose_smallest(h, have, (int)deg, room, win);
      if (chosen) {
        // the winners move to the lanes behind the forward part, the others to all other lanes
        const int before = rank_in(win[0]);
        const bool mine = (win[0] >> lane) & 1ull;
        const int dst = mine ? nf + before : 2 * p + lane - before;
        const uint32_t moved =
            (uint32_t)__builtin_amdgcn_ds_permute((dst & 63) << 2, (int)first);
        val = lane < nf ? fwd : lane < 2 * p ? moved : kNoId;
      }
    }
    if (!chosen) {
      uint64_t best = first != kNoId ? select_key(base, v, first, iter) : kKeyMax;
      best = wave_sort(best, lane);
      for (uint32_t c = kWave; c < deg; c += kWave) {
        uint64_t key =
            c + lane < deg ? select_key(base, v, (uint32_t)csr[beg + c + lane], iter) : kKeyMax;
        key = wave_sort(key, lane);
        best = wave_merge_smallest(best, key, lane);
      }
      const int src = lane - nf;
      const uint32_t r = __shfl((uint32_t)best, src < 0 ? 0 : src, kWave);
      val = lane < nf ? fwd : src < room ? r : kNoId;
    }
  }
  val = wave_sort_upto(val, lane, total);
  const uint32_t prev = lane_before(val, kNoId);
  const bool keep = val != prev && val != kNoId;
  const uint64_t mask = __ballot(keep);
  const int count = __popcll(mask);
  if (keep) list[rank_in(mask)] = (int32_t)val;
  if (lane >= count && lane < 2 * p) list[lane] = -1;
  return count;
}

// One wavefront finishes both sample lists of kNodesPerWave nodes.  It requests everything of
// the two dependent rounds of reads (sizes, offsets and list rows, then the candidate segments)
// for all its nodes at once and then works the lists off; from there on the kernel is bound by
// vector-instruction issue.  The values of list t (node t / 2, kind t % 2) that are the same for
// all lanes stand in lane t, and the loop over the nodes is a loop: unrolled four times it was
// 11,000 instructions with a hundred scalar registers spilled.
// kNodesPerWave is 4, and 1 where the chip has too few wavefronts that way: see launch_sample.
template <int kNodesPerWave>
__global__ __launch_bounds__(kBlock) void k_rev_select(int64_t n, int p, uint64_t base_new,
                                                       uint64_t base_old, uint32_t iter,
                                                       int32_t* snew, int32_t* sold,
                                                       int32_t* cnew, int32_t* cold,
                                                       const uint64_t* roff_new,
                                                       const uint64_t* roff_old,
                                                       const int32_t* csr_new,
                                                       const int32_t* csr_old,
                                                       SegmentRule seg, uint64_t* poff,
                                                       uint64_t* pslot, uint64_t* counters,
                                                       uint32_t* clear) {
  const int64_t v0 = wave_global_index() * kNodesPerWave;
  if (v0 >= n) return;
  const int lane = lane_id();
  const int L = 2 * p;
  const int nodes = n - v0 < kNodesPerWave ? (int)(n - v0) : kNodesPerWave;
  // lane t: forward samples, reverse degree (below 2^32) and first candidate of list t
  const int64_t v_l = v0 + (lane >> 1);
  const bool old_l = lane & 1, mine = lane < 2 * nodes;
  int nf_l = 0;
  uint32_t deg_l = 0;
  uint64_t beg_l = 0, fwd_l = 0;
  if (mine) {
    const uint64_t* const roff = old_l ? roff_old : roff_new;
    nf_l = (old_l ? cold : cnew)[v_l];
    beg_l = roff[v_l];
    deg_l = (uint32_t)(roff[v_l + 1] - beg_l);
    fwd_l = seg.before(v_l);
  }
  auto nf_of = [&](int t) { return __builtin_amdgcn_readlane(nf_l, t); };
  auto deg_of = [&](int t) { return (uint32_t)__builtin_amdgcn_readlane((int)deg_l, t); };
  uint32_t rown[kNodesPerWave], rowo[kNodesPerWave], firstn[kNodesPerWave], firsto[kNodesPerWave];
#pragma unroll
  for (int i = 0; i < kNodesPerWave; ++i) {
    const int64_t v = v0 + i < n ? v0 + i : n - 1;  // beyond the end: the last node again, unused
    rown[i] = lane < p ? (uint32_t)snew[v * L + lane] : kNoId;  // the forward part, -1 behind it
    rowo[i] = lane < p ? (uint32_t)sold[v * L + lane] : kNoId;
  }
#pragma unroll
  for (int i = 0; i < kNodesPerWave; ++i) {
    const uint32_t jn = (uint32_t)(lane - nf_of(2 * i)) & 63u;
    const uint32_t jo = (uint32_t)(lane - nf_of(2 * i + 1)) & 63u;
    firstn[i] = jn < deg_of(2 * i) ? (uint32_t)csr_new[readlane64(beg_l, 2 * i) + jn] : kNoId;
    firsto[i] =
        jo < deg_of(2 * i + 1) ? (uint32_t)csr_old[readlane64(beg_l, 2 * i + 1) + jo] : kNoId;
  }
  int size_l = 0;
#pragma unroll 1
  for (int i = 0; i < nodes; ++i) {
    const int64_t v = v0 + i;
    const int cn = select_list(v, p, base_new, iter, snew + v * L, rown[0], nf_of(2 * i), csr_new,
                               readlane64(beg_l, 2 * i), deg_of(2 * i), firstn[0], lane);
    size_l = lane == 2 * i ? cn : size_l;
    const int co = select_list(v, p, base_old, iter, sold + v * L, rowo[0], nf_of(2 * i + 1),
                               csr_old, readlane64(beg_l, 2 * i + 1), deg_of(2 * i + 1),
                               firsto[0], lane);
    size_l = lane == 2 * i + 1 ? co : size_l;
#pragma unroll
    for (int j = 0; j + 1 < kNodesPerWave; ++j) {
      rown[j] = rown[j + 1];
      rowo[j] = rowo[j + 1];
      firstn[j] = firstn[j + 1];
      firsto[j] = firsto[j + 1];
    }
  }
  if (mine) (old_l ? cold : cnew)[v_l] = size_l;
  if (clear && mine) clear[(old_l ? n : 0) + v_l] = 0u;  // (DevState::degree)
  // a node's segment of the proposals (both lists of a node stand side by side)
  const uint32_t per = old_l ? seg.per_old : seg.per_new;
  auto both = [&](uint64_t x) { return x + xor_lanes(x, 1, lane); };
  const uint64_t at = both(per * beg_l) + fwd_l, rev = both((uint64_t)per * deg_l);
  const uint64_t fwd = both((uint64_t)per * (uint32_t)nf_l);
  if (mine && !old_l) seg.write(v_l, n, at, rev, fwd, poff, pslot, counters);
  // (lanes without a list: 0)
  uint32_t sum = (uint32_t)size_l;
  sum += xor_lanes(sum, 2, lane);
  sum += xor_lanes(sum, 4, lane);
  if (lane < 2) counter_add(counters, lane ? C_SUMOLD : C_SUMNEW, v0, (uint64_t)sum);
}

// ---------------------------------------------------------------------------
// Sec. 4.3 list insertion for all proposals of one destination at once: the
// list becomes the best k, by (distance, id), of its entries and the proposed
// objects, one entry per id - what inserting them one by one under a lock
// gives in any order.  Admitted entries are flagged NEW.
__global__ __launch_bounds__(kBlock) void k_update(int64_t n, int k, uint64_t* G, NodeMeta* meta,
                                                   const uint64_t* pslot, const uint64_t* poff,
                                                   const uint64_t* bins, uint64_t* counters) {
  __shared__ uint64_t lds[kWavesPerBlock][kWave];
  const int64_t u = wave_global_index();
  if (u >= n) return;
  const int lane = lane_id();
  // everything that needs no other load is requested together (the row too, even
  // if the node turns out to have received nothing): one round trip less
  uint64_t cnt = pslot[u] & kSlotCountMask;
  const uint64_t beg = poff[u], cap = poff[u + 1] - beg;
  uint64_t row = lane < k ? G[u * k + lane] : kKeyMax;
  if (cnt == 0) return;
  if (cnt > cap) {  // cannot happen: a segment is sized by the bound of what its node can receive
    if (lane == 0) counter_add(counters, C_OVERFLOW, u, cnt - cap);
    cnt = cap;
  }
  bool changed = false;
  for (uint64_t c = 0; c < cnt; c += kWave) {
    uint64_t pk = (c + lane < cnt) ? bins[beg + c + lane] : kKeyMax;
    bool any;
    pk = filter_candidates(pk, row, k, lane, lds[wave_id()], any);
    if (!any) continue;
    row = wave_merge_smallest(row, pk, lane);
    if (lane >= k) row = kKeyMax;
    changed = true;
  }
  if (!changed) return;
  const uint64_t admitted = __ballot(lane < k && (row & 2ull));
  if (lane < k) G[u * k + lane] = row & ~2ull;
  if (lane == k - 1) meta[u].kth = entry_code(row);
  if (lane == 0) counter_add(counters, C_INSERTS, u, (uint64_t)__popcll(admitted));
}

// ---------------------------------------------------------------------------
// The same for lists of up to 32 entries, two destinations per wavefront: the lower and the
// upper 32 lanes each own a destination, and every step above runs on 32 lanes - both halves
// by the same instructions, with shorter sorting and merging networks.
__device__ inline uint64_t half_lanes(int lane) {
  return (lane & 32) ? 0xffffffff00000000ull : 0x00000000ffffffffull;
}
// stable compaction inside each half (see wave_compact)
__device__ inline uint64_t half_compact(uint64_t v, bool keep, uint64_t fill, int lane) {
  const uint64_t all = __ballot(keep);
  const uint32_t mask = (lane & 32) ? (uint32_t)(all >> 32) : (uint32_t)all;
  const int before = __popc(mask & ((1u << (lane & 31)) - 1u));
  const int dst = (lane & 32) | (keep ? before : __popc(mask) + ((lane & 31) - before));
  const uint64_t x = keep ? v : fill;
  const uint32_t lo = __builtin_amdgcn_ds_permute(dst << 2, (int)(uint32_t)x);
  const uint32_t hi = __builtin_amdgcn_ds_permute(dst << 2, (int)(uint32_t)(x >> 32));
  return ((uint64_t)hi << 32) | lo;
}
// the 32 smallest of two ascending 32-lane sequences, ascending, in each half
__device__ inline uint64_t half_merge_smallest(uint64_t a_sorted, uint64_t b_sorted, int lane) {
  // value of lane 31 - (lane % 32) of the half: mirror inside the row of 16, then swap the rows
  const uint32_t mlo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)b_sorted, 0x140, 0xF, 0xF, true);
  const uint32_t mhi =
      (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(b_sorted >> 32), 0x140, 0xF, 0xF, true);
  const uint64_t br = xor_lanes(((uint64_t)mhi << 32) | mlo, 16, lane);
  uint64_t v = vmin(a_sorted, br);
#pragma unroll
  for (int j = 16; j > 0; j >>= 1) {
    v = exchange_step(v, j, lane, (lane & j) == 0);
  }
  return v;
}
// filter_candidates on 32 lanes, in two parts; `row` is the half's ascending list in LDS, 32
// entries of which k are used.  First part: what is not closer than the list's last entry or
// already in the list becomes kKeyMax (where it stands).
__device__ inline uint64_t half_drop_known(uint64_t pk, const uint64_t* row, int k) {
  if (pk >= (row[k - 1] & ~3ull)) pk = kKeyMax;
  if (__ballot(pk != kKeyMax) == 0ull) return pk;
  return list_holds<32>(row, pk) ? kKeyMax : pk;
}
// Second part: the survivors, already at the front of their half (`count` = the larger
// number of them in the two halves), ascending and without repeats.
__device__ inline uint64_t half_sort_unique(uint64_t pk, int count, int lane) {
  const int l32 = lane & 31;
  // the networks over up to 32 lanes never cross the halves; the in-half lane number makes
  // both halves ascend
  if (count > 16) pk = wave_sort_first<32>(pk, l32);
  else if (count > 8) pk = wave_sort_first<16>(pk, l32);
  else if (count > 4) pk = wave_sort_first<8>(pk, l32);
  else if (count > 2) pk = wave_sort_first<4>(pk, l32);
  else if (count > 1) pk = wave_sort_first<2>(pk, l32);
  const uint64_t prev = lane_before(pk, kKeyMax);
  const bool rep = l32 > 0 && pk != kKeyMax && entry_key(pk) == entry_key(prev);
  if (__ballot(rep) != 0ull) pk = half_compact(pk, !rep, kKeyMax, lane);
  return pk;
}

// The work on one pair of destinations (one per half): `row`, `cnt`, `beg` as loaded, `pa` /
// `pb` the first 64 proposals of each destination (two per lane, kKeyMax beyond cnt).
__device__ inline void update_pair(int64_t u, bool live, int k, uint64_t cnt, uint64_t beg,
                                   uint64_t row, uint64_t pa, uint64_t pb, uint64_t* G,
                                   NodeMeta* meta, const uint64_t* bins, uint64_t* counters,
                                   uint64_t* lds, int lane) {
  const int l32 = lane & 31;
  const uint64_t* const list = lds + (lane & 32);  // the half's row, for the tests
  if (__ballot(cnt != 0) == 0ull) return;
  const uint64_t cnt_other = __shfl(cnt, lane ^ 32, kWave);
  const uint64_t rounds = cnt > cnt_other ? cnt : cnt_other;
  const uint64_t mine_mask = half_lanes(lane);
  bool changed = false;
  // survivors (at the front of their half, `count` at most in either half) into the row
  auto admit = [&](uint64_t pk, int count) {
    pk = half_sort_unique(pk, count, lane);
    const bool mine = (__ballot(pk != kKeyMax) & mine_mask) != 0ull;
    row = half_merge_smallest(row, pk, lane);  // a half without survivors keeps its row
    if (l32 >= k) row = kKeyMax;
    changed = changed || mine;
  };
  // A round takes 64 proposals per destination, two per lane.  Few of them survive the cheap
  // tests as a rule: when the survivors of both registers fit one half they go through one
  // sorting and one merging network, otherwise the second register waits for the first.
  for (uint64_t c = 0; c < rounds; c += 64) {
    if (c > 0) {
      pa = (c + l32 < cnt) ? bins[beg + c + l32] : kKeyMax;
      pb = (c + 32 + l32 < cnt) ? bins[beg + c + 32 + l32] : kKeyMax;
    }
    lds[lane] = row;
    wave_lds_fence();
    pa = half_drop_known(pa, list, k);
    pb = half_drop_known(pb, list, k);
    wave_lds_fence();
    const uint64_t left_a = __ballot(pa != kKeyMax), left_b = __ballot(pb != kKeyMax);
    if ((left_a | left_b) == 0ull) continue;
    const int na = __popcll(left_a & mine_mask), nb = __popcll(left_b & mine_mask);
    const int na_max = vmax(__popcll(left_a & 0xffffffffull), __popcll(left_a >> 32));
    pa = half_compact(pa, pa != kKeyMax, kKeyMax, lane);
    if (left_b == 0ull) {
      admit(pa, na_max);
    } else if (__ballot(na + nb > 32) == 0ull) {
      pb = half_compact(pb, pb != kKeyMax, kKeyMax, lane);
      const int src = l32 - na;
      const uint64_t shifted = __shfl(pb, (lane & 32) | (src < 0 ? 0 : src), kWave);
      const int n0 = __popcll(left_a & 0xffffffffull) + __popcll(left_b & 0xffffffffull);
      const int n1 = __popcll(left_a >> 32) + __popcll(left_b >> 32);
      admit(l32 < na ? pa : shifted, vmax(n0, n1));
    } else {
      if (left_a != 0ull) admit(pa, na_max);
      // the list has changed: the second register takes the cheap tests again
      lds[lane] = row;
      wave_lds_fence();
      pb = half_drop_known(pb, list, k);
      wave_lds_fence();
      const uint64_t left = __ballot(pb != kKeyMax);
      if (left != 0ull) {
        pb = half_compact(pb, pb != kKeyMax, kKeyMax, lane);
        admit(pb, vmax(__popcll(left & 0xffffffffull), __popcll(left >> 32)));
      }
    }
  }
  const uint64_t admitted = __ballot(l32 < k && (row & 2ull)) & mine_mask;
  if (changed && live) {
    if (l32 < k) G[u * k + l32] = row & ~2ull;
    if (l32 == k - 1) meta[u].kth = entry_code(row);
    if (l32 == 0) counter_add(counters, C_INSERTS, u, (uint64_t)__popcll(admitted));
  }
}

// One pair of destinations per wavefront.  (Unlike k_rev_select this kernel is bound by
// vector-instruction issue: with two pairs per wavefront and both rounds of reads requested up
// front it was slower, 3.4 against 3.1 ms per build on the benchmark workload.)
constexpr int kPairsPerWave = 1;
__global__ __launch_bounds__(kBlock) void k_update_pairs(int64_t n, int k, uint64_t* G,
                                                         NodeMeta* meta, const uint64_t* pslot,
                                                         const uint64_t* poff,
                                                         const uint64_t* bins, uint64_t* counters) {
  __shared__ uint64_t lds[kWavesPerBlock][kWave];
  const int lane = lane_id(), l32 = lane & 31;
  const int64_t u0 = wave_global_index() * (2 * kPairsPerWave) + (lane >> 5);
  if (u0 - (lane >> 5) >= n) return;  // the whole wavefront lies beyond the last node
  int64_t u[kPairsPerWave];
  bool live[kPairsPerWave];
  uint64_t cnt[kPairsPerWave], beg[kPairsPerWave], row[kPairsPerWave];
  uint64_t pa[kPairsPerWave], pb[kPairsPerWave];
#pragma unroll
  for (int j = 0; j < kPairsPerWave; ++j) {
    u[j] = u0 + 2 * j;
    live[j] = u[j] < n;
    cnt[j] = live[j] ? pslot[u[j]] & kSlotCountMask : 0;
    beg[j] = live[j] ? poff[u[j]] : 0;
    const uint64_t cap = live[j] ? poff[u[j] + 1] - beg[j] : 0;
    row[j] = (live[j] && l32 < k) ? G[u[j] * k + l32] : kKeyMax;
    if (cnt[j] > cap) {  // cannot happen: a segment is sized by the bound of what its node can receive
      if (l32 == 0) counter_add(counters, C_OVERFLOW, u[j], cnt[j] - cap);
      cnt[j] = cap;
    }
  }
#pragma unroll
  for (int j = 0; j < kPairsPerWave; ++j) {
    pa[j] = (l32 < cnt[j]) ? bins[beg[j] + l32] : kKeyMax;
    pb[j] = (32 + l32 < cnt[j]) ? bins[beg[j] + 32 + l32] : kKeyMax;
  }
#pragma unroll
  for (int j = 0; j < kPairsPerWave; ++j)
    update_pair(u[j], live[j], k, cnt[j], beg[j], row[j], pa[j], pb[j], G, meta, bins, counters,
                lds[wave_id()], lane);
}

// ---------------------------------------------------------------------------
template <bool FLOAT>
__global__ __launch_bounds__(kBlock) void k_get_graph(int64_t total, const uint64_t* G,
                                                      int32_t* ids, void* dist, uint8_t* isnew,
                                                      int32_t id_offset) {
  const int64_t i = block_linear() * kBlock + threadIdx.x;
  if (i >= total) return;
  const uint64_t e = G[i];
  if (ids) ids[i] = (int32_t)entry_id(e) + id_offset;
  if (isnew) isnew[i] = (uint8_t)(e & 1ull);
  if (dist) {
    if (FLOAT) reinterpret_cast<float*>(dist)[i] = unord_f32(entry_code(e));
    else reinterpret_cast<int32_t*>(dist)[i] = unord_i32(entry_code(e));
  }
}

// An id that is no node of the graph, or the row's own node, would later be
// used as a row number: it raises `bad` and is replaced by a valid id, so that
// nothing can read out of bounds even if the caller ignores the error.
template <bool FLOAT>
__global__ __launch_bounds__(kBlock) void k_set_graph(int64_t total, int64_t n, int k, uint64_t* G,
                                                      NodeMeta* meta, const int32_t* ids,
                                                      const void* dist, const uint8_t* isnew,
                                                      int* bad) {
  const int64_t i = block_linear() * kBlock + threadIdx.x;
  if (i >= total) return;
  uint32_t code = FLOAT ? ord_f32(reinterpret_cast<const float*>(dist)[i])
                        : ord_i32(reinterpret_cast<const int32_t*>(dist)[i]);
  const int64_t row = i / k;
  uint32_t id = (uint32_t)ids[i];
  if ((int64_t)id >= n || (int64_t)id == row) {
    atomicOr(bad, 1);
    id = (uint32_t)((row + 1 + i % k) % n);
  }
  G[i] = make_entry(code, id, isnew ? (uint32_t)(isnew[i] & 1) : 0u);
  if ((i % k) == k - 1) meta[i / k].kth = code;
}

// Copy the proposal segments out: slot j of destination u's segment holds u and
// the proposed (object, distance) when filled, -1 otherwise.
template <bool FLOAT>
__global__ __launch_bounds__(kBlock) void k_get_proposals(int64_t n, const uint64_t* pslot,
                                                          const uint64_t* poff,
                                                          const uint64_t* bins, int32_t* u_out,
                                                          int32_t* v_out, void* dist) {
  const int64_t u = wave_global_index();
  if (u >= n) return;
  const uint64_t beg = poff[u], cap = poff[u + 1] - beg, cnt = pslot[u] & kSlotCountMask;
  for (uint64_t i = lane_id(); i < cap; i += kWave) {
    const bool have = i < cnt;
    const uint64_t e = have ? bins[beg + i] : 0ull;
    u_out[beg + i] = have ? (int32_t)u : -1;
    v_out[beg + i] = have ? (int32_t)entry_id(e) : -1;
    if (FLOAT) reinterpret_cast<float*>(dist)[beg + i] = have ? unord_f32(entry_code(e)) : 0.f;
    else reinterpret_cast<int32_t*>(dist)[beg + i] = have ? unord_i32(entry_code(e)) : 0;
  }
}

// Slots beyond the last segment (the segments need not fill the whole array).
__global__ __launch_bounds__(kBlock) void k_fill_i32(int32_t* p, const uint64_t* from,
                                                     int64_t end, int32_t value) {
  const int64_t i = (int64_t)(*from) + block_linear() * kBlock + threadIdx.x;
  if (i < end) p[i] = value;
}

__global__ __launch_bounds__(kBlock) void k_zero_u32(uint32_t* p, size_t count) {
  const size_t i = (size_t)block_linear() * kBlock + threadIdx.x;
  if (i < count) p[i] = 0u;
}

// ---------------------------------------------------------------------------
// GGM, Alg. 3 "Divide" + "Append": keep the first ceil(k/2) entries (OLD), set
// the rest aside, refill with floor(k/2) random objects of the other set (NEW)
// and restore the (distance, id) order.
template <int METRIC>
__global__ __launch_bounds__(kBlock) void k_merge_init(VecSrc vs, int64_t n, MergeIds mi, int k,
                                                       uint64_t base_hash, const int32_t* ids1,
                                                       const void* dist1, const int32_t* ids2,
                                                       const void* dist2, uint64_t* G,
                                                       NodeMeta* meta, uint64_t* aside) {
  __shared__ uint32_t tile[kWavesPerBlock][kEvalTileWords];
  const int64_t s = wave_global_index();
  if (s >= n) return;
  const int lane = lane_id();
  const int64_t n1 = mi.n1;
  const bool first = s < n1;
  const int64_t loc = first ? s : s - n1;
  const int32_t* sid = (first ? ids1 : ids2) + loc * k;
  const void* sdist = first ? dist1 : dist2;
  const int keep = (k + 1) / 2, fill = k / 2;
  uint32_t id_in = 0, code_in = 0;
  if (lane < k) {
    id_in = mi.to_internal(sid[lane]);  // collection id -> numbering of this merge
    code_in = METRIC == kL2U8
                  ? ord_i32(reinterpret_cast<const int32_t*>(sdist)[loc * k + lane])
                  : ord_f32(reinterpret_cast<const float*>(sdist)[loc * k + lane]);
  }
  if (lane >= keep && lane < k) aside[s * fill + (lane - keep)] = make_entry(code_in, id_in, 0u);
  const uint32_t draw = draw_distinct(base_hash, (uint32_t)s, fill,
                                      (uint32_t)(first ? n - n1 : n1), first ? (uint32_t)n1 : 0u,
                                      0xffffffffu, lane);
  const int src = lane - keep;
  const uint32_t did = __shfl(draw, src < 0 ? 0 : src, kWave);
  const uint32_t code = wave_distances<METRIC>(vs, (uint32_t)s, did, lane >= keep && lane < k,
                                               tile[wave_id()], lane);
  uint64_t e = kKeyMax;
  if (lane < keep) e = make_entry(code_in, id_in, 0u);
  else if (lane < k) e = make_entry(code, did, 1u);
  e = wave_sort(e, lane);
  if (lane < k) G[s * k + lane] = e;
  if (lane == k - 1) meta[s].kth = entry_code(e);
}

// GGM, Alg. 3 "Merge and Sort": best k of the refined list and the set-aside
// half, handed out under collection ids, ascending by (distance, collection id).
template <bool FLOAT>
__global__ __launch_bounds__(kBlock) void k_merge_final(int64_t n, MergeIds mi, int k,
                                                        const uint64_t* G, const uint64_t* aside,
                                                        int32_t* ids_out, void* dist_out) {
  __shared__ uint64_t lds[kWavesPerBlock][kWave];
  const int64_t s = wave_global_index();
  if (s >= n) return;
  const int lane = lane_id();
  const int fill = k / 2;
  uint64_t row = lane < k ? G[s * k + lane] : kKeyMax;
  uint64_t pk = lane < fill ? aside[s * fill + lane] : kKeyMax;
  // the set-aside entries may tie with the list's last entry: compare on the
  // full (distance, id) key, which filter_candidates does
  bool any;
  pk = filter_candidates(pk, row, k, lane, lds[wave_id()], any);
  if (any) {
    row = wave_merge_smallest(row, pk, lane);
  }
  // renumber, then restore the order under the new ids (only ties can move)
  row = lane < k ? make_entry(entry_code(row), (uint32_t)mi.to_global(entry_id(row)), 0u)
                 : kKeyMax;
  row = wave_sort(row, lane);
  if (lane < k) {
    ids_out[s * k + lane] = (int32_t)entry_id(row);
    if (FLOAT) reinterpret_cast<float*>(dist_out)[s * k + lane] = unord_f32(entry_code(row));
    else reinterpret_cast<int32_t*>(dist_out)[s * k + lane] = unord_i32(entry_code(row));
  }
}

// ---------------------------------------------------------------------------
static VecSrc vec_src(const Shape& sh) {
  return VecSrc{sh.vec_a, sh.vec_b, sh.split, sh.d, sh.norms};
}

hipError_t launch_zero_u32(uint32_t* p, size_t count, hipStream_t st) {
  if (count == 0) return hipSuccess;
  k_zero_u32<<<grid_blocks((int64_t)((count + kBlock - 1) / kBlock)), kBlock, 0, st>>>(p, count);
  return hipGetLastError();
}

// Squared norm of every row, one fused multiply-add per dimension in dimension
// order (what the cosine distance divides by).  A wavefront takes 64 rows: chunks
// of kEvalChunk dimensions go through LDS with coalesced reads (8 lanes per row
// chunk), then each lane adds up its own row.
__global__ __launch_bounds__(kBlock) void k_row_norms(VecSrc vs, int64_t n, float* norms,
                                                      NodeMeta* meta) {
  __shared__ float tile[kWavesPerBlock][64 * kEvalStride];
  const int lane = lane_id();
  float* my = tile[wave_id()];
  const int64_t row0 = (block_linear() * kWavesPerBlock + wave_id()) * 64;
  if (row0 >= n) return;
  const int d = vs.d;
  const int part = lane & 7, rsel = lane >> 3;
  float acc = 0.f;
  for (int d0 = 0; d0 < d; d0 += kEvalChunk) {
#pragma unroll
    for (int r0 = 0; r0 < 64; r0 += 8) {
      const int r = r0 + rsel;
      if (row0 + r < n) {
        const float* src = vs.row<float>((uint32_t)(row0 + r));
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int j = d0 + part * 4 + q;
          my[r * kEvalStride + part * 4 + q] = j < d ? src[j] : 0.f;
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int width = d - d0 < kEvalChunk ? d - d0 : kEvalChunk;
    for (int j = 0; j < width; ++j) {
      const float x = my[lane * kEvalStride + j];
      acc = __fmaf_rn(x, x, acc);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  if (row0 + lane < n) {
    norms[row0 + lane] = acc;
    if (meta) meta[row0 + lane].norm = (int32_t)__float_as_uint(acc);
  }
}

hipError_t launch_row_norms(const Shape& sh, float* norms, NodeMeta* meta, hipStream_t st) {
  const int64_t waves = (sh.n + 63) / 64;
  k_row_norms<<<grid_blocks((waves + kWavesPerBlock - 1) / kWavesPerBlock), kBlock, 0, st>>>(
      vec_src(sh), sh.n, norms, meta);
  return hipGetLastError();
}

hipError_t launch_init_random(const Shape& sh, const DevState& ds, uint64_t seed,
                              hipStream_t st) {
  if (sh.segments > 1) return launch_init_random_segmented(sh, ds, seed, st);
  if (sh.k > kWave) return launch_init_random_wide(sh, ds, seed, st);
  const dim3 grid = blocks_for_waves(sh.n);
  const uint64_t base = hash_base(seed, kTagInit);
  switch (sh.metric) {
    case kL2F32:
      k_init_random<kL2F32><<<grid, kBlock, 0, st>>>(vec_src(sh), sh.n, sh.k, base, ds.G, ds.meta);
      break;
    case kAngularF32:
      k_init_random<kAngularF32><<<grid, kBlock, 0, st>>>(vec_src(sh), sh.n, sh.k, base, ds.G,
                                                          ds.meta);
      break;
    case kChi2F32:
      k_init_random<kChi2F32><<<grid, kBlock, 0, st>>>(vec_src(sh), sh.n, sh.k, base, ds.G,
                                                       ds.meta);
      break;
    case kCosineF32:
      k_init_random<kCosineF32><<<grid, kBlock, 0, st>>>(vec_src(sh), sh.n, sh.k, base, ds.G,
                                                         ds.meta);
      break;
    default:
      k_init_random<kL2U8><<<grid, kBlock, 0, st>>>(vec_src(sh), sh.n, sh.k, base, ds.G, ds.meta);
  }
  return hipGetLastError();
}

// Up to this many nodes a wavefront of the reverse selection takes one (16 wavefronts per CU): with
// four, 4096 nodes are one wavefront per SIMD, and a build of 8 iterations takes 501 instead of 478
// us.  Beyond, there are enough of them either way, and four nodes at a time hide their reads.
constexpr int64_t kOneNodePerWave = 1 << 14;
hipError_t launch_sample(const Shape& sh, const DevState& ds, uint64_t seed, uint32_t iter,
                         Expect expect, hipStream_t st) {
  // forward sampling, and the reverse candidates grouped by target
  const bool direct = sample_direct(sh.n, sh.p);
  int group_rows = 32;
  hipError_t e = direct ? launch_sample_direct(sh, ds, expect, st)
                        : launch_sample_buckets(sh, ds, expect, &group_rows, st);
  if (e != hipSuccess) return e;
  uint32_t* const clear = direct ? ds.degree : nullptr;
  if (2 * sh.p > kWave)  // two list entries per lane
    return launch_rev_select_long(sh, ds, seed, iter, group_rows, clear, st);
#define GNND_SELECT(NODES)                                                                       \
  k_rev_select<NODES><<<blocks_for_waves((sh.n + NODES - 1) / NODES), kBlock, 0, st>>>(          \
      sh.n, sh.p, hash_base(seed, kTagRevNew), hash_base(seed, kTagRevOld), iter, ds.snew,       \
      ds.sold, ds.cnew, ds.cold, ds.roff_new, ds.roff_old, ds.csr_new, ds.csr_old,               \
      SegmentRule(sh, ds, group_rows), ds.poff, ds.pslot, ds.counters, clear)
  if (sh.n <= kOneNodePerWave) GNND_SELECT(1);
  else GNND_SELECT(4);
#undef GNND_SELECT
  return hipGetLastError();
}

hipError_t launch_update(const Shape& sh, const DevState& ds, hipStream_t st) {
  if (sh.segments > 1) return launch_update_segmented(sh, ds, st);
  if (sh.k > kWave) return launch_update_wide(sh, ds, st);
  if (sh.k <= 32)
    k_update_pairs<<<blocks_for_waves((sh.n + 2 * kPairsPerWave - 1) / (2 * kPairsPerWave)), kBlock, 0, st>>>(
        sh.n, sh.k, ds.G, ds.meta, ds.pslot, ds.poff, ds.bins, ds.counters);
  else
    k_update<<<blocks_for_waves(sh.n), kBlock, 0, st>>>(sh.n, sh.k, ds.G, ds.meta, ds.pslot,
                                                        ds.poff, ds.bins, ds.counters);
  return hipGetLastError();
}

hipError_t launch_get_graph(const Shape& sh, const DevState& ds, int32_t* ids, void* dist,
                            uint8_t* isnew, int32_t id_offset, hipStream_t st) {
  const int64_t total = sh.n * sh.k;
  const dim3 grid = grid_blocks((total + kBlock - 1) / kBlock);
  if (sh.metric == kL2U8)
    k_get_graph<false><<<grid, kBlock, 0, st>>>(total, ds.G, ids, dist, isnew, id_offset);
  else
    k_get_graph<true><<<grid, kBlock, 0, st>>>(total, ds.G, ids, dist, isnew, id_offset);
  return hipGetLastError();
}

hipError_t launch_set_graph(const Shape& sh, const DevState& ds, const int32_t* ids,
                            const void* dist, const uint8_t* isnew, int* bad_flag_dev,
                            hipStream_t st) {
  const int64_t total = sh.n * sh.k;
  const dim3 grid = grid_blocks((total + kBlock - 1) / kBlock);
  if (sh.metric == kL2U8)
    k_set_graph<false><<<grid, kBlock, 0, st>>>(total, sh.n, sh.k, ds.G, ds.meta, ids, dist, isnew,
                                                bad_flag_dev);
  else
    k_set_graph<true><<<grid, kBlock, 0, st>>>(total, sh.n, sh.k, ds.G, ds.meta, ids, dist, isnew,
                                               bad_flag_dev);
  return hipGetLastError();
}

hipError_t launch_get_proposals(const Shape& sh, const DevState& ds, int32_t* u, int32_t* v,
                                void* dist, hipStream_t st) {
  const dim3 grid = blocks_for_waves(sh.n);
  if (sh.metric == kL2U8)
    k_get_proposals<false><<<grid, kBlock, 0, st>>>(sh.n, ds.pslot, ds.poff, ds.bins, u, v, dist);
  else
    k_get_proposals<true><<<grid, kBlock, 0, st>>>(sh.n, ds.pslot, ds.poff, ds.bins, u, v, dist);
  const int64_t slots = sh.slots();
  const dim3 g2 = grid_blocks((slots + kBlock - 1) / kBlock);
  k_fill_i32<<<g2, kBlock, 0, st>>>(u, ds.poff + sh.n, slots, -1);
  k_fill_i32<<<g2, kBlock, 0, st>>>(v, ds.poff + sh.n, slots, -1);
  return hipGetLastError();
}

hipError_t launch_merge_init(const Shape& sh, const DevState& ds, uint64_t seed,
                             const MergeIds& mi, const int32_t* ids1, const void* dist1,
                             const int32_t* ids2, const void* dist2, hipStream_t st) {
  if (sh.k > kWave) return launch_merge_init_wide(sh, ds, seed, mi, ids1, dist1, ids2, dist2, st);
  const dim3 grid = blocks_for_waves(sh.n);
  const uint64_t base = hash_base(seed, kTagMerge);
  switch (sh.metric) {
    case kL2F32:
      k_merge_init<kL2F32><<<grid, kBlock, 0, st>>>(vec_src(sh), sh.n, mi, sh.k, base, ids1, dist1,
                                                    ids2, dist2, ds.G, ds.meta, ds.aside);
      break;
    case kAngularF32:
      k_merge_init<kAngularF32><<<grid, kBlock, 0, st>>>(vec_src(sh), sh.n, mi, sh.k, base, ids1,
                                                         dist1, ids2, dist2, ds.G, ds.meta,
                                                         ds.aside);
      break;
    case kChi2F32:
      k_merge_init<kChi2F32><<<grid, kBlock, 0, st>>>(vec_src(sh), sh.n, mi, sh.k, base, ids1,
                                                      dist1, ids2, dist2, ds.G, ds.meta, ds.aside);
      break;
    case kCosineF32:
      k_merge_init<kCosineF32><<<grid, kBlock, 0, st>>>(vec_src(sh), sh.n, mi, sh.k, base, ids1,
                                                        dist1, ids2, dist2, ds.G, ds.meta,
                                                        ds.aside);
      break;
    default:
      k_merge_init<kL2U8><<<grid, kBlock, 0, st>>>(vec_src(sh), sh.n, mi, sh.k, base, ids1, dist1,
                                                   ids2, dist2, ds.G, ds.meta, ds.aside);
  }
  return hipGetLastError();
}

hipError_t launch_merge_final(const Shape& sh, const DevState& ds, const MergeIds& mi,
                              int32_t* ids_out, void* dist_out, hipStream_t st) {
  if (sh.k > kWave) return launch_merge_final_wide(sh, ds, mi, ids_out, dist_out, st);
  const dim3 grid = blocks_for_waves(sh.n);
  if (sh.metric == kL2U8)
    k_merge_final<false><<<grid, kBlock, 0, st>>>(sh.n, mi, sh.k, ds.G, ds.aside, ids_out,
                                                  dist_out);
  else
    k_merge_final<true><<<grid, kBlock, 0, st>>>(sh.n, mi, sh.k, ds.G, ds.aside, ids_out,
                                                 dist_out);
  return hipGetLastError();
}

}  // namespace gnnd

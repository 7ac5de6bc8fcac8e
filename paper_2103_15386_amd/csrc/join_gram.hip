// The float32 matrix-core join: what it prepares (norms, 16-bit copies of the rows, the lists of
// nodes by class) and its launches.  The kernel itself: join_gram.hpp.
#include <stddef.h>

#include "join_gram.hpp"

namespace gnnd {

extern template void launch_gram_builds<kL2F32>(const Shape&, const DevState&, int, unsigned,
                                                hipStream_t);
extern template void launch_gram_builds<kAngularF32>(const Shape&, const DevState&, int, unsigned,
                                                     hipStream_t);
extern template void launch_gram_builds<kCosineF32>(const Shape&, const DevState&, int, unsigned,
                                                    hipStream_t);

namespace {

// The nodes that have something to evaluate, listed by class.
template <int PER>
__global__ __launch_bounds__(256) void k_gram_classify(int64_t n, int merge_mode,
                                                       const int32_t* __restrict__ cnew,
                                                       const int32_t* __restrict__ cold,
                                                       int32_t* nodes, uint32_t* count) {
  list_nodes_by_class<kGramClasses, PER>(n, nodes, count, [&](int64_t s) {
    const int nn = cnew[s], no = cold[s];
    const bool do_nn = !merge_mode && nn > 1;
    return nn != 0 && (do_nn || no != 0) ? gram_class((nn + 15) >> 4, (no + 15) >> 4) : -1;
  });
}

// The 16-bit copies of the rows (see HalfRows): one wavefront per row.  A float16 quotient has
// a relative error of at most 2^-11; what counts is the norm of all errors of a row together,
// which is measured here (the largest over all rows goes to `rho`, as float bits).
// OWN_NORMS: the metric does not need the norm that is summed in dimension order; the wavefront
// adds up its own (64 partial sums, then a tree) and leaves it in the node's record.
template <bool OWN_NORMS>
__global__ __launch_bounds__(256) void k_half_rows(VecSrc vs, int64_t n, _Float16* out, int stride,
                                                   NodeMeta* meta, uint32_t* rho) {
  __shared__ uint32_t largest;
  if (threadIdx.x == 0) largest = 0u;
  __syncthreads();
  const int lane = lane_id();
  constexpr int kRowsPerWave = 8;
  const int64_t s0 = (block_linear() * 4 + wave_id()) * kRowsPerWave;
  for (int i = 0; i < kRowsPerWave; ++i) {
    const int64_t s = s0 + i;
    if (s >= n) break;
    const float* src = vs.row<float>((uint32_t)s);
    float norm = 0.f;
    if (OWN_NORMS) {
      for (int j = lane; j < vs.d; j += kWave) norm = __fmaf_rn(src[j], src[j], norm);
#pragma unroll
      for (int o = 1; o < kWave; o <<= 1)
        norm += __uint_as_float(xor_lanes(__float_as_uint(norm), o, lane));
      if (lane == 0) meta[s].norm = (int32_t)__float_as_uint(norm);
    } else {
      norm = vs.norms[s];
    }
    const float root = sqrtf(norm);
    const bool zero = norm == 0.f;
    const bool none = !zero && !(norm >= kHalfLeast && norm <= kNormMost);
    const float scale = zero || none ? 0.f : (float)(1 << kHalfBits) / root;
    const float back = root * (1.0f / (1 << kHalfBits));  // as the join multiplies it on again
    _Float16* dst = out + s * stride;
    float err = 0.f;
    bool any = false;  // a norm of zero by underflow: elements that are not zero
    for (int j = lane; j < stride; j += kWave) {
      const float x = j < vs.d ? src[j] : 0.f;
      _Float16 h = (_Float16)(x * scale);
      if (fabsf((float)h) < 6.1035156e-5f) h = (_Float16)0.f;
      if (zero) h = (_Float16)0.f;
      const float diff = __fmaf_rn(-(float)h, back, x);
      err = __fmaf_rn(diff, diff, err);
      any |= x != 0.f;
      if (none) h = (_Float16)__uint_as_float(0x7fc00000u);
      dst[j] = h;
    }
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) err += __uint_as_float(xor_lanes(__float_as_uint(err), o, lane));
    const bool lost = norm == 0.f && __ballot(any) != 0ull;
    if (lost)
      for (int j = lane; j < stride; j += kWave) dst[j] = (_Float16)__uint_as_float(0x7fc00000u);
    // (0.2 % more than measured covers the roundings of the sums and of the norm)
    if (lane == 0 && !none && !zero)
      atomicMax(&largest, __float_as_uint(sqrtf(err / norm) * 1.002f));
  }
  __syncthreads();
  if (threadIdx.x == 0 && largest) atomicMax(rho, largest);
}

int compute_units() {
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

}  // namespace

hipError_t launch_half_rows(const Shape& sh, const DevState& ds, hipStream_t st) {
  VecSrc vs{sh.vec_a, sh.vec_b, sh.split, sh.d, sh.norms};
  static_assert(sizeof(NodeMeta) == 8 && offsetof(NodeMeta, kth) == 0 && offsetof(NodeMeta, norm) == 4,
                "k_join_gram reads a NodeMeta as (kth, norm bits)");
  auto* const kernel = sh.metric == kCosineF32 ? k_half_rows<false> : k_half_rows<true>;
  kernel<<<grid_blocks((sh.n + 31) / 32), 256, 0, st>>>(
      vs, sh.n, static_cast<_Float16*>(ds.half_rows), (int)half_row_elems(sh.d), ds.meta,
      ds.half_info);
  return hipGetLastError();
}

hipError_t launch_join_gram(const Shape& sh, const DevState& ds, bool merge_mode, hipStream_t st) {
  const int mm = merge_mode ? 1 : 0;
  // the nodes with work to do, by class (few nodes: fewer per workgroup, so that more of the
  // chip lists them; many: fewer additions to the lists' lengths); not where all are of one
  // class (4096 x 16, p = 8: this launch and that of a second build took 12 of 58 us per iteration)
  if (!gram_one_class(sh.p)) {
    if (sh.n <= (1 << 20))
      k_gram_classify<4><<<grid_blocks((sh.n + 1023) / 1024), 256, 0, st>>>(
          sh.n, mm, ds.cnew, ds.cold, ds.cls_nodes, ds.cls_count);
    else
      k_gram_classify<16><<<grid_blocks((sh.n + 4095) / 4096), 256, 0, st>>>(
          sh.n, mm, ds.cnew, ds.cold, ds.cls_nodes, ds.cls_count);
  }
  // one build per class, each with about four sets of resident wavefronts (the lists' lengths
  // are known on the device only) and never more wavefronts than nodes
  const int64_t cap = (int64_t)64 * compute_units();
  const unsigned grid = (unsigned)(sh.n < cap ? sh.n : cap);
  switch (sh.metric) {
    case kL2F32: launch_gram_builds<kL2F32>(sh, ds, mm, grid, st); break;
    case kAngularF32: launch_gram_builds<kAngularF32>(sh, ds, mm, grid, st); break;
    case kCosineF32: launch_gram_builds<kCosineF32>(sh, ds, mm, grid, st); break;
    default: return hipErrorInvalidValue;  // no inner-product form for the other metrics
  }
  return hipGetLastError();
}

}  // namespace gnnd

// k_small_seg.hip -- plora_segment_apply of batches of up to kSegApplyMax
// tokens in one launch, the tiles' slices exchanging (see
// segment_apply_one_launch).
#include "plora_small.h"

namespace plora_impl {

template <bool DEEP>
__device__ __forceinline__ void direct_item(const SmallArgs& a, const ApplyArgs& g,
                                            const int32_t* idx, int item, SmallLds<1>& sm) {
  int u, s;
  small_slot<true>(item, a.J, a.gl, u, s);
  if (u >= g.T) return;
  SmallItem<1> t;
  small_ranges<1>(g, a.S, a.J, s, t);
  const uint64_t ep = xload(g.xep + u);
  t.tok[0] = u;
  XRegs<1> xr;
  x_issue<1>(g, t.tok, t.k0, min(t.k1, t.k0 + kSXW), xr);
  const int id = uni(idx[u]);
  if (id < 0 || id >= g.N) return;
  bool bad;
  if (!small_adapter<1>(g, uni(g.ranks[id]), g.scales[id], g.a_off[id], g.b_off[id], t, bad)) {
    if (bad && s == 0 && g.count_skips) bump(g, 1, 1);
    return;
  }
  small_body<1, true, DEEP>(g, t, xr, sm, s, a.S, u, ep);
}

// Up to kDecodeTokens tokens (single-token tiles): item (u, s) takes token u
// itself.  A token's result does not depend on which tile slot carries it,
// so the items need no ranking: each requests its x row and reads its id,
// then its adapter's metadata.  Work group 0 only ranks the batch and writes
// the segmentation for later calls; in a DEEP launch, whose items may fill
// the chip, it takes an item first.
template <bool DEEP>
__global__ __launch_bounds__(kST, small_waves(DEEP)) void small_direct_kernel(SmallArgs a, const int32_t* idx,
                                                              SegOut so) {
  __shared__ __align__(16) union {
    SmallLds<1> sm;
    LocalTile lt;
  } sh;
  const ApplyArgs& g = a.g;
  static_assert(kDecodeTokens == 64, "wave_segment ranks one wavefront's tokens");
  const int item = DEEP ? (int)blockIdx.x : (int)blockIdx.x - 1;
  if (!DEEP && item < 0) {
    if (threadIdx.x < 64) wave_segment(g, idx, so, sh.lt);
    return;
  }
  direct_item<DEEP>(a, g, idx, item, sh.sm);
  if (DEEP && blockIdx.x == 0) {
    lds_sync();
    if (threadIdx.x < 64) wave_segment(g, idx, so, sh.lt);
  }
}
// 65 to kSegApplyMax tokens (tiles of two): every work group ranks the batch
// (reading the ids takes the trip the tile record would) and takes its own
// tile; work group 0 also writes the segmentation.
template <bool DEEP>
__global__ __launch_bounds__(kST, small_waves(DEEP)) void small_block_kernel(SmallArgs a, const int32_t* idx,
                                                             SegOut so) {
  __shared__ __align__(16) SmallLds<2> sm;
  __shared__ __align__(16) LocalTile lt;
  const ApplyArgs& g = a.g;
  int u, s;
  small_slot<true>(blockIdx.x, a.J, a.gl, u, s);
  const uint64_t ep = xload(g.xep + u);
  block_segment(g, idx, u, so, blockIdx.x == 0, lt);
  lds_sync();
  SmallItem<2> t;
  const int ta = uni(lt.a), L = uni(lt.L);
  if (L <= 0 || ta < 0 || ta >= g.N) return;
  const int p0 = uni(lt.p0);
  t.tok[0] = uni((int)(lt.sorted[p0] & 255));
  t.tok[1] = L > 1 ? uni((int)(lt.sorted[p0 + 1 < kSegApplyMax ? p0 + 1 : 0] & 255)) : -1;
  const int t0 = t.tok[0];
  const int64_t ao = lt.ao_of[t0], bo = lt.bo_of[t0];
  bool bad;
  if (!small_adapter<2>(g, uni(lt.rank_of[t0]),
                        __int_as_float(uni(__float_as_int(lt.scale_of[t0]))), ao, bo, t, bad)) {
    if (bad && s == 0 && g.count_skips) bump(g, 1, (unsigned long long)L);
    return;
  }
  small_ranges<2>(g, a.S, a.J, s, t);
  small_run<2, true, DEEP>(g, t, L, p0, &sm, s, a.S, u, ep);
}

void launch_small_segment_apply(const SmallArgs& a, const int32_t* idx, const SegOut& so,
                                unsigned grid, hipStream_t stream) {
  if (a.g.T <= kDecodeTokens) {
    hipLaunchKernelGGL(a.deep ? small_direct_kernel<true> : small_direct_kernel<false>, dim3(grid),
                       dim3(kST), 0, stream, a, idx, so);
  } else {
    hipLaunchKernelGGL(a.deep ? small_block_kernel<true> : small_block_kernel<false>, dim3(grid),
                       dim3(kST), 0, stream, a, idx, so);
  }
}

}  // namespace plora_impl

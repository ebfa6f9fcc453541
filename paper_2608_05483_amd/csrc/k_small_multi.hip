// k_small_multi.hip -- plora_apply_multi of batches of up to kFusedTokens
// tokens in one launch.
#include "plora_small.h"

namespace plora_impl {

// Slot p cap + u is tile u of projection p, and exchanges through that slot.
template <int MAXL, bool X, bool DEEP>
__global__ __launch_bounds__(kST, small_waves(DEEP)) void small_multi_kernel(MultiArgs m, int32_t S, int32_t J,
                                                                         int32_t gl) {
  __shared__ __align__(16) SmallLds<MAXL> sm;
  int slot, s;
  small_slot<X>(blockIdx.x, J, gl, slot, s);
  const int p = slot / m.cap, u = slot - p * m.cap;
  if (p >= m.n_proj) return;
  uint64_t ep = 0;
  if (X) ep = xload(m.g.xep + slot);
  ApplyArgs g = m.g;
  const ProjArgs& q = m.proj[p];
  g.A = q.A; g.B = q.B; g.a_len = q.a_len; g.b_len = q.b_len;
  g.A_pool = q.A_pool; g.B_pool = q.B_pool; g.a_pool_len = q.a_pool_len;
  g.b_pool_len = q.b_pool_len;
  g.a_off = q.a_off; g.b_off = q.b_off; g.ranks = q.ranks; g.scales = q.scales;
  g.y = q.y; g.ldy = q.ldy; g.h_out = q.h_out; g.max_rank = q.max_rank;
  SmallItem<2> t;
  int p0;
  const int L = small_tile<!X>(g, u, s, t, p0);
  if (L == 0) return;
  small_ranges<2>(g, S, J, s, t);
  if (!X && t.j0 >= t.j1) return;
  small_run<MAXL, X, DEEP>(g, t, L, p0, &sm, s, S, slot, ep);
}

void launch_small_multi(const MultiArgs& m, int32_t S, int32_t J, int32_t gl, int32_t deep,
                        unsigned grid, hipStream_t stream) {
  small_variant(m.g.T, S > 1, deep, [&](auto l, auto x, auto d) {
    hipLaunchKernelGGL((small_multi_kernel<l(), x(), d()>), dim3(grid), dim3(kST), 0, stream, m, S,
                       J, gl);
  });
}

}  // namespace plora_impl

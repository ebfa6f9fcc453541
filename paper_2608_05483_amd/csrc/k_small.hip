// k_small.hip -- plora_apply, plora_shrink and plora_expand of batches of up
// to kFusedTokens tokens.
#include "plora_small.h"

namespace plora_impl {

// MAXL: the longest tile of the launch (1 up to kDecodeTokens tokens).
template <int MAXL, bool X, bool DEEP>
__global__ __launch_bounds__(kST, small_waves(DEEP)) void small_apply_kernel(SmallArgs a) {
  __shared__ __align__(16) SmallLds<MAXL> sm;
  const ApplyArgs& g = a.g;
  int u, s;
  small_slot<X>(blockIdx.x, a.J, a.gl, u, s);
  uint64_t ep = 0;
  if (X) ep = xload(g.xep + u);
  SmallItem<2> t;
  int p0;
  const int L = small_tile<!X>(g, u, s, t, p0);
  if (L == 0) return;
  small_ranges<2>(g, a.S, a.J, s, t);
  if (!X && t.j0 >= t.j1) return;
  small_run<MAXL, X, DEEP>(g, t, L, p0, &sm, s, a.S, u, ep);
}

// plora_shrink: item (tile, slice of h_in), as the apply's.  One slice writes
// v itself; several leave their partial sums in the workspace for
// small_gather_kernel (an exchange would need the epochs, and so a workspace
// that has been zeroed).
template <int MAXL, bool X, bool DEEP>
__global__ __launch_bounds__(kST, small_waves(DEEP)) void small_shrink_kernel(SmallArgs a) {
  __shared__ __align__(16) SmallLds<MAXL> smx;
  const ApplyArgs& g = a.g;
  const int u = X ? (int)blockIdx.x / a.S : (int)blockIdx.x;
  const int s = X ? (int)blockIdx.x - u * a.S : 0;
  SmallItem<2> t2;
  int p0;
  const int L = small_tile<true>(g, u, s, t2, p0);
  if (L == 0) return;
  small_ranges<2>(g, a.S, a.J, s, t2);
  small_tokens<MAXL, true>(g, t2, L, p0, [&](const auto& t, int l, bool) {
    constexpr int TG = std::remove_reference_t<decltype(t)>::kTokens;
    SmallLds<TG>& sm = *reinterpret_cast<SmallLds<TG>*>(&smx);
    XRegs<TG> xr;
    BRegs<small_batch(DEEP)> br;
    YRegs<TG> yr;
    x_issue<TG>(g, t.tok, t.k0, min(t.k1, t.k0 + kSXW), xr);
    shrink_small<TG, small_batch(DEEP), kReadOnce, false, X && DEEP>(g, t, xr, sm, br, yr);
    const int tok0 = t.tok[0], tok1 = t.tok[TG - 1];
    for (int o = threadIdx.x; o < t.r * TG; o += kST) {
      const int c = o / TG, tt = o - c * TG;
      const int tk = tt == 0 ? tok0 : tok1;
      if (X) g.vpart[((int64_t)s * g.T + p0 + l + tt) * g.max_rank + c] = sm.vs[o];
      else if (tk >= 0) g.v[(int64_t)tk * g.ldv + c] = sm.vs[o];
    }
  });
}

// v of tile blockIdx.x's tokens, the S partials summed in slice order as the
// exchange sums them.
__global__ __launch_bounds__(kST) void small_gather_kernel(SmallArgs a) {
  const ApplyArgs& g = a.g;
  SmallItem<2> t;
  const int u = blockIdx.x;
  int p0;
  const int L = small_tile<true>(g, u, 1, t, p0);   // (slice 0 of the shrink counted the skips)
  if (L == 0) return;
  const int64_t step = (int64_t)g.T * g.max_rank;
  for (int o = threadIdx.x; o < L * t.r; o += kST) {
    const int l = o / t.r, c = o - l * t.r;
    const int tk = l == 0 ? t.tok[0] : l == 1 ? t.tok[1] : tile_token(g, p0 + l);
    const float* src = g.vpart + (int64_t)(p0 + l) * g.max_rank + c;
    float p[kMaxSlices];
#pragma unroll
    for (int q = 0; q < kMaxSlices; ++q) p[q] = src[(q < a.S ? q : 0) * step];
    float v = p[0];
#pragma unroll
    for (int q = 1; q < kMaxSlices; ++q)
      if (q < a.S) v += p[q];
    if (tk >= 0) g.v[(int64_t)tk * g.ldv + c] = v;
  }
}

// plora_expand: item (tile, column slice) with v from the caller's array.
template <int MAXL, bool DEEP>
__global__ __launch_bounds__(kST, small_waves(DEEP)) void small_expand_kernel(SmallArgs a) {
  __shared__ __align__(16) SmallLds<MAXL> smx;
  const ApplyArgs& g = a.g;
  int u, s;
  small_slot<false>(blockIdx.x, a.J, a.gl, u, s);
  SmallItem<2> t2;
  int p0;
  const int L = small_tile<true>(g, u, s, t2, p0);
  if (L == 0) return;
  small_ranges<2>(g, a.S, a.J, s, t2);
  if (t2.j0 >= t2.j1) return;
  small_tokens<MAXL, true>(g, t2, L, p0, [&](const auto& t, int, bool) {
    constexpr int TG = std::remove_reference_t<decltype(t)>::kTokens;
    SmallLds<TG>& sm = *reinterpret_cast<SmallLds<TG>*>(&smx);
    BRegs<small_batch(DEEP)> br;
    YRegs<TG> yr;
    b_issue<TG, small_batch(DEEP)>(g, t, br, yr);
    for (int o = threadIdx.x; o < t.r * TG; o += kST) {
      const int c = o / TG, tt = o - c * TG;
      const int tk = tt == 0 ? t.tok[0] : t.tok[TG - 1];
      sm.vs[o] = tk >= 0 ? g.v[(int64_t)tk * g.ldv + c] : 0.f;
    }
    lds_sync();
    expand_small<TG, small_batch(DEEP)>(g, t, sm, br, yr);
  });
}

void launch_small_apply(const SmallArgs& a, unsigned grid, hipStream_t stream) {
  small_variant(a.g.T, a.S > 1, a.deep, [&](auto l, auto x, auto d) {
    hipLaunchKernelGGL((small_apply_kernel<l(), x(), d()>), dim3(grid), dim3(kST), 0, stream, a);
  });
}

void launch_small_shrink(const SmallArgs& a, unsigned grid, hipStream_t stream) {
  small_variant(a.g.T, a.S > 1, a.deep, [&](auto l, auto x, auto d) {
    hipLaunchKernelGGL((small_shrink_kernel<l(), x(), d()>), dim3(grid), dim3(kST), 0, stream, a);
  });
  if (a.S > 1)
    hipLaunchKernelGGL(small_gather_kernel, dim3(a.g.tile_cap), dim3(kST), 0, stream, a);
}

void launch_small_expand(const SmallArgs& a, unsigned grid, hipStream_t stream) {
  small_variant(a.g.T, false, a.deep, [&](auto l, auto, auto d) {
    hipLaunchKernelGGL((small_expand_kernel<l(), d()>), dim3(grid), dim3(kST), 0, stream, a);
  });
}

}  // namespace plora_impl

// plora_small.h -- device code of the small-batch kernels (batches of up to
// kFusedTokens tokens, tiles of one or two tokens): plora_apply,
// plora_segment_apply, plora_apply_multi, plora_shrink and plora_expand of
// such batches all run these bodies, so they compute the same bits.
//
// A work group of kST threads takes one item: a tile and one of its slices.
//
//   shrink   v[l][c] = sum_k x[l][k] A_i[k][c] over rows [k0, k1).  A_i's
//            rows are one contiguous run of 16-byte chunks, whatever the
//            rank: thread t takes chunks t, t + NT, ... with NT the largest
//            multiple of r / gcd(r, 8) (the chunks after which the column
//            pattern repeats) up to kST, so that element j of every chunk it
//            sees has the same column and a row that advances by a constant.
//            It needs eight accumulators per token and no rank classes (a
//            chunk of a rank that is a multiple of 8 lies in one row).  The accumulators are summed per
//            column through LDS in a fixed order.
//   expand   y[l][j] += s sum_c v[l][c] B_i[c][j] over columns [j0, j1).
//            Thread (octet, slot) takes rows slot, slot + RS, ... of B_i for
//            one octet of columns; the slots are summed through LDS in order.
//
// A tile is split over S work groups, each with its share of h_in and of the
// columns, which trade their partial v through the workspace (see
// exchange_small), so that each tile's A_i and B_i are read once; with S = 1
// (h_in or h_out below 1024) a work group computes the tile's v whole, for all
// of the columns or, where they are many, for a slice of them.
//
// What bounds them: a launch of little data is a chain of latencies (start,
// ids or tile, adapter metadata, A_i, reduction, exchange, B_i, store: 9 us
// for one token over 8 work groups) in which instructions count as much as
// memory trips, since a wavefront issues one in about 5 cycles: 256 threads
// (one wavefront per SIMD and work group) beat 512 by 1.5 us a launch, and
// batches that every active thread has whole are unrolled without checks.  A
// launch of long slices is bound by HBM (256 tokens at rank 64: 240 MB in
// 43 us).  Whole-v column slices (every one reducing all of h_in, no
// exchange) were 2 to 5 us slower per launch at decode.  Steps over 7B-shaped
// layers, before (rank classes, LDS-staged shrink for ranks that are no
// multiple of 8) and now: 64 tokens at rank 16 149 -> 120 us; ranks 4 to 40,
// 100 tokens, 13B widths 284 -> 108; ranks 64 and 128 at h = 8192, 45 tokens,
// 223 -> 212; 256 tokens at rank 64 as before, 182.
#ifndef PLORA_SMALL_H
#define PLORA_SMALL_H

#include "plora_dev.h"

#include <type_traits>

namespace plora_impl {

constexpr int kST = 256;                 // threads per work group
constexpr int kSWaves = kST / 64;
// Chunks per thread and batch, two batches in flight, and the wavefronts per
// SIMD the registers are held to.
__host__ __device__ constexpr int small_batch(bool deep) { return deep ? 8 : 4; }
__host__ __device__ constexpr int small_waves(bool deep) { return deep ? 2 : 3; }
// Rows of B_i per thread requested ahead of the expand: they travel while v is
// reduced and exchanged.
__host__ __device__ constexpr int small_ahead(int su) { return su == 8 ? 8 : 4; }
constexpr int kSXW = 8192;               // rows of x staged in LDS per window
constexpr int kSOct = kST;               // most column octets per expand pass


// Adapter reads are non-temporal: distinct adapters come from HBM, once.  That
// holds also where column slices (S = 1) or an adapter's other tiles read a
// block again, unless few adapters serve the whole batch.  us per call or step,
// this and the default policy: 64 tokens, h = 4096, rank 16, Zipf, four layers
// 119 and 126; 256 tokens at rank 64 332 and 363 (two layers); one slice, 792
// -> 4512 at rank 64, each call on another stack of 1000 adapters, 64 tokens
// 15.1 and 16.8, 256 tokens 32.7 and 36.5, of four adapters 15.6 and 12.0;
// split calls of 256 tokens at rank 64 386 and 399 over 1000 adapters, 257 and
// 225 over eight (eight calls each).
constexpr int kReadOnce = 2;

// The work of one item (values uniform over the work group).
template <int TG>
struct SmallItem {
  static constexpr int kTokens = TG;
  int tok[TG];                           // token of each row, -1 for none
  int r;
  float s;
  const uint16_t* Ai;
  const uint16_t* Bi;
  int k0, k1, j0, j1;
};

// LDS: v, then a region for x and, once x is dead, the cross-thread sums.
template <int TG>
struct SmallLds {
  float vs[PLORA_MAX_RANK * TG];         // [c][TG]
  float red2[kSWaves * PLORA_MAX_RANK * TG];
  union {
    uint16_t xs[TG][kSXW];
    float red[kST * 8 * TG];
  };
};

constexpr int kXRegs = kSXW / 8 / kST;   // x chunks per thread, token and window

template <int TG>
struct XRegs {
  uint4 v[TG][kXRegs];
};

// Request x of rows [w0, w1) of the item's tokens.
template <int TG>
__device__ __forceinline__ void x_issue(const ApplyArgs& g, const int (&tok)[TG], int w0, int w1,
                                        XRegs<TG>& xr) {
  const int n8 = (w1 - w0) >> 3;
#pragma unroll
  for (int tt = 0; tt < TG; ++tt)
#pragma unroll
    for (int i = 0; i < kXRegs; ++i) {
      const int c = (int)threadIdx.x + i * kST;
      const bool ok = tok[tt] >= 0 && c < n8;
      // masked lanes read the first chunk of a row that exists
      const uint16_t* row = g.x + (int64_t)max(tok[tt], 0) * g.ldx;
      xr.v[tt][i] = ldg16z(row + w0 + c * 8, row, ok);
    }
}

template <int TG>
__device__ __forceinline__ void x_store(const XRegs<TG>& xr, int rows, SmallLds<TG>& sm) {
  const int n8 = rows >> 3;
#pragma unroll
  for (int tt = 0; tt < TG; ++tt)
#pragma unroll
    for (int i = 0; i < kXRegs; ++i) {
      const int c = (int)threadIdx.x + i * kST;
      if (c < n8) *reinterpret_cast<uint4*>(&sm.xs[tt][c * 8]) = xr.v[tt][i];
    }
}

// This thread's walk over the chunks of a window of rows of A_i: nt active
// threads, rstep rows between a thread's chunks, and the row of element e of
// its first chunk, row + (drow >> 3 e & 7) (a rank that is a multiple of 8
// has all eight in one row).
struct FlatMap {
  int nt, rstep, row;
  uint32_t drow;
};

__device__ __forceinline__ FlatMap flat_map(int r) {
  FlatMap m;
  const int gcd = (r & 7) == 0 ? 8 : (r & 3) == 0 ? 4 : (r & 1) == 0 ? 2 : 1;
  const int per = r / gcd;
  m.nt = kST / per * per;
  m.rstep = m.nt * 8 / r;
  m.row = (int)threadIdx.x * 8 / r;
  m.drow = 0;
  if (r & 7) {
    int cc = (int)threadIdx.x * 8 - m.row * r;
    uint32_t d = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      m.drow |= d << (3 * e);
      if (++cc == r) {
        cc = 0;
        ++d;
      }
    }
  }
  return m;
}

// 16 bytes at byte offset vo + j step of a block, j < N; zero past its end.
// step goes through an empty asm so that the offsets are formed here, not
// hoisted and kept (which spilled).
template <int POL, int N>
__device__ __forceinline__ void load_steps(Rsrc r, uint32_t vo, uint32_t step, uint4 (&a)[N]) {
  __asm__ volatile("" : "+s"(step));
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const i32x4_t v =
        __builtin_amdgcn_raw_buffer_load_b128(r, (int)(vo + (uint32_t)j * step), 0, POL);
    a[j] = make_uint4((uint32_t)v.x, (uint32_t)v.y, (uint32_t)v.z, (uint32_t)v.w);
  }
}

// acc[tt][e] += x[tt][row] * chunk[e] for this thread's chunks jb .. jb + N - 1
// of a rank that is a multiple of 8, without checks.
template <int TG, int N, int SU>
__device__ __forceinline__ void flat_whole(float (&acc)[TG][8], const uint4 (&a)[SU],
                                           const SmallLds<TG>& sm, const FlatMap& m, int jb) {
  int row = m.row + jb * m.rstep;
#pragma unroll
  for (int j = 0; j < N; ++j) {
    float af[8];
    unpack8(a[j], af);
#pragma unroll
    for (int tt = 0; tt < TG; ++tt) {
      const float xf = __uint_as_float((uint32_t)sm.xs[tt][row] << 16);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[tt][e] = fmaf(xf, af[e], acc[tt][e]);
    }
    row += m.rstep;
    __asm__ volatile("" : "+v"(row));
  }
}

// acc[tt][e] += x[tt][row of e] * chunk[e] for chunks jb .. jb + SU - 1 (of
// this thread's nj), one at a time: the empty asm keeps the compiler from
// forming every chunk's LDS addresses ahead, which spilled.
template <int TG, int SU>
__device__ __forceinline__ void flat_fma(float (&acc)[TG][8], const uint4 (&a)[SU],
                                         const SmallLds<TG>& sm, const FlatMap& m, bool aligned,
                                         int jb, int nj, int n_full) {
  if (aligned && jb + SU <= n_full) {
    // every active thread has all the batch's chunks (the others add zeros to
    // sums that are not read)
    flat_whole<TG, SU>(acc, a, sm, m, jb);
    return;
  }
  int row = m.row + jb * m.rstep;
  uint32_t drow = m.drow;
  __asm__ volatile("" : "+v"(row), "+v"(drow));
#pragma unroll
  for (int j = 0; j < SU; ++j) {
    if (jb + j < nj) {
      float af[8];
      unpack8(a[j], af);
      if (aligned) {
#pragma unroll
        for (int tt = 0; tt < TG; ++tt) {
          const float xf = __uint_as_float((uint32_t)sm.xs[tt][row] << 16);
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[tt][e] = fmaf(xf, af[e], acc[tt][e]);
        }
      } else {
#pragma unroll
        for (int tt = 0; tt < TG; ++tt)
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int re = row + (int)((drow >> (3 * e)) & 7u);
            const float xf = __uint_as_float((uint32_t)sm.xs[tt][re] << 16);
            acc[tt][e] = fmaf(xf, af[e], acc[tt][e]);
          }
      }
    }
    row += m.rstep;
    __asm__ volatile("" : "+v"(row), "+v"(drow));
  }
}

// ---- expand ---------------------------------------------------------------------

struct ColMap {
  int lg, RS, oct, slot, n_oct, nb, nbm;
};

// Octets and row slots of the columns [j0, j0 + 8 n_oct) of one pass.
__device__ __forceinline__ ColMap col_map(int n_oct, int r) {
  ColMap m;
  m.n_oct = n_oct;
  m.lg = n_oct <= 1 ? 0 : 32 - __clz(n_oct - 1);
  m.RS = kST >> m.lg;
  m.oct = threadIdx.x & ((1 << m.lg) - 1);
  m.slot = threadIdx.x >> m.lg;
  m.nbm = (r + m.RS - 1) / m.RS;
  m.nb = m.oct < n_oct && m.slot < r ? (r - m.slot + m.RS - 1) / m.RS : 0;
  return m;
}

template <int SU>
struct BRegs {
  uint4 b[small_ahead(SU)];
};

template <int TG>
struct YRegs {
  uint2 y[TG];
};

// y words of output quad i of a pass: quads i = (tt << (lg + 1)) + q, q the
// quad of four columns.
template <int TG>
__device__ __forceinline__ const uint16_t* y_quad(const ApplyArgs& g, int tok0, int tok1,
                                                  const ColMap& m, int jp, int i, bool& ok) {
  const int tt = i >> (m.lg + 1), q = i & ((2 << m.lg) - 1);
  const int tk = TG > 1 && tt == 1 ? tok1 : tok0;
  ok = tt < TG && q < 2 * m.n_oct && tk >= 0;
  return g.y + (int64_t)max(tk, 0) * g.ldy + (ok ? jp + q * 4 : 0);
}

// Byte offset of this thread's first unit of B_i in the pass at column jp.
__device__ __forceinline__ uint32_t b_offset(const ApplyArgs& g, const ColMap& m, int jp) {
  return m.oct < m.n_oct ? ((uint32_t)m.slot * (uint32_t)g.h_out + (uint32_t)(jp + m.oct * 8)) * 2u
                         : (uint32_t)kPastEnd;
}

template <int TG, int SU>
__device__ __forceinline__ void b_issue(const ApplyArgs& g, const SmallItem<TG>& t, BRegs<SU>& br,
                                        YRegs<TG>& yr) {
  const ColMap m = col_map(min((t.j1 - t.j0) >> 3, kSOct), t.r);
  // rows past the rank lie past the block; octets past the slice read nothing
  load_steps<kReadOnce>(block_rsrc(t.Bi, (int64_t)g.h_out * t.r), b_offset(g, m, t.j0),
                        (uint32_t)(m.RS * g.h_out * 2), br.b);
  const int tok0 = t.tok[0], tok1 = t.tok[TG - 1];
#pragma unroll
  for (int k = 0; k < TG; ++k) {
    bool ok;
    const uint16_t* p = y_quad<TG>(g, tok0, tok1, m, t.j0, (int)threadIdx.x + k * kST, ok);
    yr.y[k] = *reinterpret_cast<const uint2*>(p);
  }
}

template <int TG>
__device__ __forceinline__ void b_fma(float (&d)[TG][8], const uint4& b, const SmallLds<TG>& sm,
                                      int row) {
  float bf[8];
  unpack8(b, bf);
#pragma unroll
  for (int tt = 0; tt < TG; ++tt) {
    const float vf = sm.vs[row * TG + tt];
#pragma unroll
    for (int e = 0; e < 8; ++e) d[tt][e] = fmaf(vf, bf[e], d[tt][e]);
  }
}

// d += v B_i over rows jb .. jb + N - 1 of this thread's, without checks.
template <int TG, int N, int M>
__device__ __forceinline__ void b_whole(float (&d)[TG][8], const uint4 (&b)[M],
                                        const SmallLds<TG>& sm, const ColMap& m, int jb) {
  int row = m.slot + jb * m.RS;
#pragma unroll
  for (int j = 0; j < N; ++j) {
    b_fma<TG>(d, b[j], sm, row);
    row += m.RS;
    __asm__ volatile("" : "+v"(row));
  }
}

// The same of this thread's nb rows (n_full: rows that every active thread
// has; octets past the slice add zeros never stored).
template <int TG, int N>
__device__ __forceinline__ void b_batch(float (&d)[TG][8], const uint4 (&b)[N],
                                        const SmallLds<TG>& sm, const ColMap& m, int jb,
                                        int n_full) {
  if (jb + N <= n_full) {
    b_whole<TG, N>(d, b, sm, m, jb);
  } else {
    int row = m.slot + jb * m.RS;
#pragma unroll
    for (int j = 0; j < N; ++j) {
      if (jb + j < m.nb) b_fma<TG>(d, b[j], sm, row);
      row += m.RS;
      __asm__ volatile("" : "+v"(row));
    }
  }
}

template <int TG, int SU>
__device__ __forceinline__ void expand_small(const ApplyArgs& g, const SmallItem<TG>& t,
                                             SmallLds<TG>& sm, const BRegs<SU>& br,
                                             const YRegs<TG>& yr) {
  constexpr int BP = small_ahead(SU);
  const Rsrc rb = block_rsrc(t.Bi, (int64_t)g.h_out * t.r);
  const int tok0 = t.tok[0], tok1 = t.tok[TG - 1];
#pragma unroll 1
  for (int jp = t.j0; jp < t.j1; jp += kSOct * 8) {
    const ColMap m = col_map(min((t.j1 - jp) >> 3, kSOct), t.r);
    const uint32_t step = (uint32_t)(m.RS * g.h_out * 2);
    const bool first = jp == t.j0;
    const int n_full = t.r / m.RS;
    float d[TG][8];
#pragma unroll
    for (int tt = 0; tt < TG; ++tt)
#pragma unroll
      for (int e = 0; e < 8; ++e) d[tt][e] = 0.f;
    if (m.nbm > BP || !first) {
      // rows past the requested ones in batches of SU, the next batch always
      // requested before the current one is used
      int jb = first ? BP : 0;
      uint32_t vo = b_offset(g, m, jp);
      const uint32_t adv = m.oct < m.n_oct ? step : 0;
      vo += jb * adv;
      uint4 b0[SU], b1[SU];
      load_steps<kReadOnce>(rb, vo, step, b0);
      if (first) b_batch<TG, BP>(d, br.b, sm, m, 0, n_full);
#pragma unroll 1
      for (; jb < m.nbm; jb += 2 * SU) {
        vo += SU * adv;
        load_steps<kReadOnce>(rb, vo, step, b1);
        b_batch<TG, SU>(d, b0, sm, m, jb, n_full);
        vo += SU * adv;
        load_steps<kReadOnce>(rb, vo, step, b0);
        b_batch<TG, SU>(d, b1, sm, m, jb + SU, n_full);
      }
    } else if (2 * n_full == BP && n_full == m.nbm) {
      b_whole<TG, BP / 2>(d, br.b, sm, m, 0);
    } else {
      b_batch<TG, BP>(d, br.b, sm, m, 0, n_full);
    }
    // the row slots' sums, [slot][tt][column of the pass]
    const int cols = 8 << m.lg;
#pragma unroll
    for (int tt = 0; tt < TG; ++tt) {
      float4* p = reinterpret_cast<float4*>(&sm.red[(m.slot * TG + tt) * cols + m.oct * 8]);
      p[0] = make_float4(d[tt][0], d[tt][1], d[tt][2], d[tt][3]);
      p[1] = make_float4(d[tt][4], d[tt][5], d[tt][6], d[tt][7]);
    }
    lds_sync();
    // output quads: at most 2 TG per thread (TG 2^(lg + 1) <= TG 512)
    constexpr int NQ = 2 * TG;
    uint2 out[NQ];
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
      const int i = (int)threadIdx.x + k * kST;
      bool ok;
      const uint16_t* yp = y_quad<TG>(g, tok0, tok1, m, jp, i, ok);
      if (ok) {
        const int tt = i >> (m.lg + 1), q = i & ((2 << m.lg) - 1);
        const uint2 yw = (first && k < TG) ? yr.y[k < TG ? k : 0]
                                           : *reinterpret_cast<const uint2*>(yp);
        const float* src = &sm.red[tt * cols + q * 4];
        float4 a = *reinterpret_cast<const float4*>(src);
        if (m.RS > 1) {
          // slots 1..3 (or 1), then in fours: RS is a power of two
          const int st = TG * cols;
          const float4 b1 = *reinterpret_cast<const float4*>(src + st);
          const float4 b2 = *reinterpret_cast<const float4*>(src + (m.RS > 2 ? 2 : 0) * st);
          const float4 b3 = *reinterpret_cast<const float4*>(src + (m.RS > 2 ? 3 : 0) * st);
          a.x += b1.x; a.y += b1.y; a.z += b1.z; a.w += b1.w;
          if (m.RS > 2) {
            a.x += b2.x; a.y += b2.y; a.z += b2.z; a.w += b2.w;
            a.x += b3.x; a.y += b3.y; a.z += b3.z; a.w += b3.w;
          }
#pragma unroll 1
          for (int sl = 4; sl < m.RS; sl += 4) {
            float4 b[4];
#pragma unroll
            for (int k4 = 0; k4 < 4; ++k4)
              b[k4] = *reinterpret_cast<const float4*>(src + (sl + k4) * st);
#pragma unroll
            for (int k4 = 0; k4 < 4; ++k4) {
              a.x += b[k4].x; a.y += b[k4].y; a.z += b[k4].z; a.w += b[k4].w;
            }
          }
        }
        out[k].x = to_bf16(fmaf(t.s, a.x, bf_lo(yw.x))) |
                   (to_bf16(fmaf(t.s, a.y, bf_hi(yw.x))) << 16);
        out[k].y = to_bf16(fmaf(t.s, a.z, bf_lo(yw.y))) |
                   (to_bf16(fmaf(t.s, a.w, bf_hi(yw.y))) << 16);
      }
    }
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
      bool ok;
      const uint16_t* yp = y_quad<TG>(g, tok0, tok1, m, jp, (int)threadIdx.x + k * kST, ok);
      if (ok) *reinterpret_cast<uint2*>(const_cast<uint16_t*>(yp)) = out[k];
    }
    if (jp + kSOct * 8 < t.j1) lds_sync();
  }
}

// Sum over the lanes of a wavefront whose index is equal modulo RP (a power of
// two), in every lane: register moves only.
template <int CTRL>
__device__ __forceinline__ float dpp_sum(float x) {
  return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float column_sum(float x, int RP) {
  if (RP <= 32) {
    const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(p[0]) + __uint_as_float(p[1]);
  }
  if (RP <= 16) {
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(p[0]) + __uint_as_float(p[1]);
  }
  if (RP <= 8) x = dpp_sum<0x128>(x);    // row_ror:8
  if (RP <= 4) x = dpp_sum<0x124>(x);    // row_ror:4
  if (RP <= 2) x = dpp_sum<0x122>(x);    // row_ror:2
  if (RP <= 1) x = dpp_sum<0x121>(x);    // row_ror:1
  return x;
}

// ---- shrink ---------------------------------------------------------------------

// acc += x A_i of rows [w0, w1), window by window: what of a slice lies past
// its first kSXW rows (h_in above 8 kSXW = 65536, since a tile has at most 8
// slices).  Such a launch is always a deep one that exchanges, so only those
// kernels have this loop (it cost the others registers, and one of them a
// spill).  x goes straight to LDS and one batch of chunks is in flight.
// (65544 -> 4096 at rank 16, one token 13.3 us, 200 tokens 39; whole-v column
// slices 71 and 220, the former exchange kernels 17.4 and 46.)
template <int TG, int SU, int POL>
__device__ __forceinline__ void shrink_rest(const ApplyArgs& g, const SmallItem<TG>& t, int w0,
                                            const FlatMap& m, bool aligned, bool active,
                                            SmallLds<TG>& sm, float (&acc)[TG][8]) {
  const uint32_t step = (uint32_t)m.nt * 16u;
#pragma unroll 1
  for (; w0 < t.k1; w0 += kSXW) {
    const int rows = min(kSXW, t.k1 - w0);
    lds_sync();                                     // the window before is read
#pragma unroll
    for (int tt = 0; tt < TG; ++tt) {
      const uint16_t* row = g.x + (int64_t)max(t.tok[tt], 0) * g.ldx;
#pragma unroll 1
      for (int c = threadIdx.x; c < rows >> 3; c += kST)
        *reinterpret_cast<uint4*>(&sm.xs[tt][c * 8]) = ldg16z(row + w0 + c * 8, row, t.tok[tt] >= 0);
    }
    lds_sync();
    const int Q = rows * t.r / 8;
    const int nj = active && (int)threadIdx.x < Q ? (Q - (int)threadIdx.x + m.nt - 1) / m.nt : 0;
    const Rsrc ra = block_rsrc(t.Ai + (int64_t)w0 * t.r, (int64_t)rows * t.r);
    uint32_t vo = active ? (uint32_t)threadIdx.x * 16u : (uint32_t)kPastEnd;
#pragma unroll 1
    for (int jb = 0; jb * m.nt < Q; jb += SU) {
      uint4 a[SU];
      load_steps<POL>(ra, vo, step, a);
      vo += active ? SU * step : 0;
      flat_fma<TG, SU>(acc, a, sm, m, aligned, jb, nj, Q / m.nt);
    }
  }
}

// v of rows [t.k0, t.k1) into sm.vs.  xr holds the first window's x
// (x_issue).  With EXP, the item's first B_i rows and y words are requested
// too: with A_i where the thread's chunks fit two batches, else once A_i is
// read (requested ahead of a longer stream they would hold it up).  MORE: the
// slice may be longer than one window.
template <int TG, int SU, int POL, bool EXP, bool MORE>
__device__ __forceinline__ void shrink_small(const ApplyArgs& g, const SmallItem<TG>& t,
                                             XRegs<TG>& xr, SmallLds<TG>& sm, BRegs<SU>& br,
                                             YRegs<TG>& yr) {
  const int tid = threadIdx.x, r = t.r;
  const FlatMap m = flat_map(r);
  const bool aligned = (r & 7) == 0;
  const bool active = tid < m.nt;
  const uint32_t step = (uint32_t)m.nt * 16u;       // bytes between a thread's chunks
  const uint32_t adv = active ? SU * step : 0;
  float acc[TG][8];
#pragma unroll
  for (int tt = 0; tt < TG; ++tt)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[tt][e] = 0.f;
  const int rows = min(kSXW, t.k1 - t.k0);          // the first window
  const int Q = rows * r / 8;                       // its chunks
  const int njm = (Q + m.nt - 1) / m.nt;
  const int nj = active && tid < Q ? (Q - tid + m.nt - 1) / m.nt : 0;
  const int n_full = Q / m.nt;                      // chunks that all active threads have
  // the window's rows as a resource of their own: chunks past it read zero
  const Rsrc ra = block_rsrc(t.Ai + (int64_t)t.k0 * r, (int64_t)rows * r);
  uint32_t vo = active ? (uint32_t)tid * 16u : (uint32_t)kPastEnd;
  uint4 a0[SU], a1[SU];
  load_steps<POL>(ra, vo, step, a0);
  vo += adv;
  if (njm <= 2 * SU) {
    load_steps<POL>(ra, vo, step, a1);
    if (EXP) b_issue<TG, SU>(g, t, br, yr);
    x_store<TG>(xr, rows, sm);
    lds_sync();
    // half a batch (rank 8 in slices of 512 rows) without checks too, and no
    // walk through a second batch that nobody has (one token at rank 8, h =
    // 4096: 8.1 -> 7.6 us a call, the former kernels 7.4; 64 tokens 10.2 ->
    // 9.8, formerly 9.5)
    if (aligned && 2 * n_full == SU && n_full == njm) {
      flat_whole<TG, SU / 2>(acc, a0, sm, m, 0);
    } else {
      flat_fma<TG, SU>(acc, a0, sm, m, aligned, 0, nj, n_full);
      if (njm > SU) flat_fma<TG, SU>(acc, a1, sm, m, aligned, SU, nj, n_full);
    }
  } else {
    load_steps<POL>(ra, vo, step, a1);
    x_store<TG>(xr, rows, sm);
    lds_sync();
#pragma unroll 1
    for (int jb = 0; jb < njm; jb += 2 * SU) {
      flat_fma<TG, SU>(acc, a0, sm, m, aligned, jb, nj, n_full);
      vo += adv;
      load_steps<POL>(ra, vo, step, a0);
      flat_fma<TG, SU>(acc, a1, sm, m, aligned, jb + SU, nj, n_full);
      vo += adv;
      load_steps<POL>(ra, vo, step, a1);
    }
    if (EXP) b_issue<TG, SU>(g, t, br, yr);
  }
  if constexpr (MORE)
    shrink_rest<TG, SU, POL>(g, t, t.k0 + kSXW, m, aligned, active, sm, acc);
  lds_sync();                                       // x is dead
  // column c's entries are the flat positions c, c + r, ... of the active
  // threads' accumulators: thread (c, ph) sums every NPH-th of them, the
  // phases of a wavefront are added by a butterfly, the wavefronts in order
  if (tid < m.nt) {
#pragma unroll
    for (int tt = 0; tt < TG; ++tt) {
      float4* p = reinterpret_cast<float4*>(&sm.red[tt * (kST * 8) + tid * 8]);
      p[0] = make_float4(acc[tt][0], acc[tt][1], acc[tt][2], acc[tt][3]);
      p[1] = make_float4(acc[tt][4], acc[tt][5], acc[tt][6], acc[tt][7]);
    }
  }
  lds_sync();
  const int lg = r <= 1 ? 0 : 32 - __clz(r - 1);
  const int RP = 1 << lg, NPH = kST >> lg;
  const int c = tid & (RP - 1), ph = tid >> lg;
  const int M = m.nt * 8 / r;                       // entries per column
  float v[TG];
#pragma unroll
  for (int tt = 0; tt < TG; ++tt) v[tt] = 0.f;
  // (8 entries per thread where the rank is a power of two, else up to 16;
  // a batch's reads are all in flight at once)
#pragma unroll 1
  for (int q0 = ph; q0 < M; q0 += 8 * NPH) {
    float e[TG][8];
#pragma unroll
    for (int tt = 0; tt < TG; ++tt)
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int q = q0 + i * NPH;
        e[tt][i] = sm.red[tt * (kST * 8) + (q < M && c < r ? c + r * q : 0)];
      }
#pragma unroll
    for (int tt = 0; tt < TG; ++tt)
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (q0 + i * NPH < M) v[tt] += e[tt][i];
  }
#pragma unroll
  for (int tt = 0; tt < TG; ++tt) v[tt] = column_sum(v[tt], RP);
  // RP <= 64: every wavefront holds a sum of every column; RP = 128: a pair does
  const int wr = tid >> 6;
  const int part = RP <= 64 ? wr : wr >> 1;
  if (c < r && (RP >= 64 || (tid & 63) < RP)) {
#pragma unroll
    for (int tt = 0; tt < TG; ++tt) sm.red2[(part * PLORA_MAX_RANK + c) * TG + tt] = v[tt];
  }
  lds_sync();
  if (tid < r * TG) {
    float p[kSWaves];
#pragma unroll
    for (int q = 0; q < kSWaves; ++q)
      p[q] = sm.red2[(RP <= 64 || q < kSWaves / 2 ? q : 0) * PLORA_MAX_RANK * TG + tid];
    float s = p[0];
#pragma unroll
    for (int q = 1; q < kSWaves; ++q)
      if (RP <= 64 || q < kSWaves / 2) s += p[q];
    sm.vs[tid] = s;
  }
  lds_sync();
}

// ---- the exchange of a tile's partial v between its slices -----------------------

// As the protocol above exchange_item describes: publish this item's
// partial v (sm.vs) under the call's tag, poll the partners' words, and put
// the S partials' sum in slice order into sm.vs; false, for the whole work
// group, if a partner's word did not arrive in time.
template <int TG>
__device__ __forceinline__ bool exchange_small(SmallLds<TG>& sm, int r, int s, int S,
                                               uint32_t tag, uint64_t* words, int polls) {
  const int n = r * TG;
  const uint64_t tagw = (uint64_t)tag << 32;
  bool late = false;
  for (int o = threadIdx.x; o < n; o += kST)
    xpublish(words + xword(o, s), tagw | __float_as_uint(sm.vs[o]));
  for (int o = threadIdx.x; o < n; o += kST) {
    const uint64_t* e = words + xword(o, 0);
    uint64_t w[kMaxSlices];
    bool ready = false;
    for (int it = 0; !ready && it <= polls; ++it) {
      // (the first poll after a sleep: the partners publish at about the
      // time this item does, and a poll right away mostly misses)
      if (it > 0) __builtin_amdgcn_s_sleep(2);
      else __builtin_amdgcn_s_sleep(16);
#pragma unroll
      for (int q = 0; q < kMaxSlices; ++q) w[q] = q < S ? xpoll(e + q * 8) : 0;
      ready = true;
#pragma unroll
      for (int q = 0; q < kMaxSlices; ++q) ready &= q >= S || (uint32_t)(w[q] >> 32) == tag;
    }
    late |= !ready;
    float v = __uint_as_float((uint32_t)w[0]);
#pragma unroll
    for (int q = 1; q < kMaxSlices; ++q)
      if (q < S) v += __uint_as_float((uint32_t)w[q]);
    sm.vs[o] = v;
  }
  return __syncthreads_or(late) == 0;
}

// The same with hook() run between the first poll's request and its use: the
// loads it issues return behind the poll's (the vector-memory counter retires
// in order; requested before the poll they would hold it up) and travel while
// the partners' words are waited for.  For the deep kernels, whose B_i,
// requested with A_i, would hold up their long streams (256 tokens at rank 64,
// two layers: 332 us, 346 with exchange_small and the early request).  The
// short ones request B_i early and take exchange_small: with the hook two
// layers at rank 16 took 44.2 us at one token (42.6 without), 48.0 at eight
// (44.4), 85.9 at 100 (90.1), 161 at 256 (164).
template <int TG, class H>
__device__ __forceinline__ bool exchange_hooked(SmallLds<TG>& sm, int r, int s, int S,
                                               uint32_t tag, uint64_t* words, int polls,
                                               H&& hook) {
  static_assert(PLORA_MAX_RANK * TG <= kST, "a thread for each entry");
  const int o = threadIdx.x;
  const bool mine = o < r * TG;
  const uint64_t* e = words + xword(o, 0);
  uint64_t w[kMaxSlices];
  if (mine)
    xpublish(words + xword(o, s), ((uint64_t)tag << 32) | __float_as_uint(sm.vs[o]));
  // (the first poll after a sleep: the partners publish at about the time
  // this item does, and a poll right away mostly misses)
  __builtin_amdgcn_s_sleep(16);
  if (mine) {
#pragma unroll
    for (int q = 0; q < kMaxSlices; ++q) w[q] = q < S ? xpoll(e + q * 8) : 0;
  }
  hook();
  bool late = false;
  if (mine) {
    for (int it = 0;; ++it) {
      bool ready = true;
#pragma unroll
      for (int q = 0; q < kMaxSlices; ++q) ready &= q >= S || (uint32_t)(w[q] >> 32) == tag;
      late = !ready;
      if (ready || it >= polls) break;
      __builtin_amdgcn_s_sleep(2);
#pragma unroll
      for (int q = 0; q < kMaxSlices; ++q) w[q] = q < S ? xpoll(e + q * 8) : 0;
    }
    float v = __uint_as_float((uint32_t)w[0]);
#pragma unroll
    for (int q = 1; q < kMaxSlices; ++q)
      if (q < S) v += __uint_as_float((uint32_t)w[q]);
    sm.vs[o] = v;
  }
  return __syncthreads_or(late) == 0;
}

// What the exchange yields, computed by this item alone when a partner's
// words never came (see plain_v).
template <int TG>
__device__ __forceinline__ void plain_v_small(const ApplyArgs& g, const SmallItem<TG>& t,
                                              SmallLds<TG>& sm) {
  const int tok0 = t.tok[0], tok1 = t.tok[TG - 1];
  for (int o = threadIdx.x; o < t.r * TG; o += kST) {
    const int c = o / TG, tt = o - c * TG;
    const int tk = tt == 0 ? tok0 : tok1;
    float v = 0.f;
    if (tk >= 0) {
      const uint16_t* xr = g.x + (int64_t)tk * g.ldx;
      for (int k = 0; k < g.h_in; ++k)
        v = fmaf(__uint_as_float((uint32_t)xr[k] << 16),
                 __uint_as_float((uint32_t)t.Ai[(int64_t)k * t.r + c] << 16), v);
    }
    sm.vs[o] = v;
  }
  lds_sync();
}

// ---- items -----------------------------------------------------------------------

// How a launch splits its tiles: S slices of h_in and J column slices (J = S
// where they exchange, S > 1).
struct SmallArgs {
  ApplyArgs g;
  int32_t S, J;
  int32_t gl;     // slots per group, log2 (see small_slot)
  int32_t deep;   // long slices: twice the chunks in flight per thread
};

__host__ __device__ constexpr int small_rows(int h_in, int S) {
  return ((h_in + S - 1) / S + 63) & ~63;
}
// Columns per slice: whole 128-byte lines of y and B_i.
__host__ __device__ constexpr int small_cols(int h_out, int J) {
  return ((h_out + J - 1) / J + 63) & ~63;
}

// Item b of a launch: tile slot u and slice s.  Exchanging slices of a slot
// are neighbours in the grid, on different XCDs (see exchange_item); the
// column slices of plora_expand go slice-major in groups of eight slots (of
// 2^gl, where the launch has fewer).
template <bool X>
__device__ __forceinline__ void small_slot(int b, int J, int gl, int& u, int& s) {
  if (X) {
    exchange_item(b, J, u, s);
  } else {
    const int q = b / (J << gl), rem = b - q * (J << gl);
    s = rem >> gl;
    u = (q << gl) + (rem & ((1 << gl) - 1));
  }
}

template <int TG>
__device__ __forceinline__ void small_ranges(const ApplyArgs& g, int S, int J, int s,
                                             SmallItem<TG>& t) {
  const int KR = S > 1 ? small_rows(g.h_in, S) : g.h_in;
  const int W = small_cols(g.h_out, J);
  t.k0 = S > 1 ? min(g.h_in, s * KR) : 0;
  t.k1 = min(g.h_in, t.k0 + KR);
  t.j0 = min(g.h_out, s * W);
  t.j1 = min(g.h_out, t.j0 + W);
}

// The adapter of an item, from its rank and offsets (all uniform): false for
// a no-op adapter, or an unusable entry, which sets bad.
template <int TG>
__device__ __forceinline__ bool small_adapter(const ApplyArgs& g, int r, float s, int64_t ao,
                                              int64_t bo, SmallItem<TG>& t, bool& bad) {
  bad = false;
  t.r = r;
  t.s = s;
  if (r == 0) return false;
  if (r < 0 || r > g.max_rank) {
    bad = true;
    return false;
  }
  t.Ai = uni(adapter_block(g.A, g.a_len, g.A_pool, g.a_pool_len, ao, (int64_t)g.h_in * r));
  t.Bi = uni(adapter_block(g.B, g.b_len, g.B_pool, g.b_pool_len, bo, (int64_t)g.h_out * r));
  bad = !t.Ai || !t.Bi;
  return !bad;
}

struct NoHook {};

// The item's partial v in sm.vs becomes the tile's v.  (hook: see
// exchange_hooked; o0: the item's first
// entry of the slot's region; last: the tile's last item of this work group,
// which raises the slot's epoch.)
template <int TG, class H>
__device__ __forceinline__ void small_exchange(const ApplyArgs& g, const SmallItem<TG>& t,
                                               SmallLds<TG>& sm, int s, int S, int slot,
                                               uint64_t ep, int o0, bool last, H&& hook) {
  const uint32_t tag = (uint32_t)(ep + 1);
  uint64_t* words = g.xw + (int64_t)slot * kSlotWords + xword(o0, 0);
  bool whole;
  if constexpr (std::is_same_v<std::decay_t<H>, NoHook>)
    whole = exchange_small<TG>(sm, t.r, s, S, tag, words, g.polls);
  else
    whole = exchange_hooked<TG>(sm, t.r, s, S, tag, words, g.polls, hook);
  if (!whole) {
    bump(g, 0, 1);
    plain_v_small<TG>(g, t, sm);
  }
  // raised once the exchange is over (every partner has read it, or this
  // item gave up), while the expand runs
  if (last && threadIdx.x == 0)
    __hip_atomic_fetch_max(g.xep + slot, ep + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Shrink, exchange (X) and expand of an item whose x has been requested.
template <int TG, bool X, bool DEEP>
__device__ __forceinline__ void small_body(const ApplyArgs& g, const SmallItem<TG>& t,
                                           XRegs<TG>& xr, SmallLds<TG>& sm, int s, int S,
                                           int slot, uint64_t ep, int o0 = 0, bool last = true) {
  constexpr int SU = small_batch(DEEP);
  BRegs<SU> br;
  YRegs<TG> yr;
  shrink_small<TG, SU, kReadOnce, !(X && DEEP), X && DEEP>(g, t, xr, sm, br, yr);
  if constexpr (X && DEEP)
    small_exchange<TG>(g, t, sm, s, S, slot, ep, o0, last, [&] { b_issue<TG, SU>(g, t, br, yr); });
  else if constexpr (X)
    small_exchange<TG>(g, t, sm, s, S, slot, ep, o0, last, NoHook{});
  expand_small<TG, SU>(g, t, sm, br, yr);
}

// The token at position p of the segmentation, -1 for none.
__device__ __forceinline__ int tile_token(const ApplyArgs& g, int p) {
  const int t = g.perm[p];
  return t >= 0 && t < g.T ? t : -1;
}

// Tile u of the segmentation: its record, first two tokens and adapter.  0:
// nothing to do, else its tokens, from position p0.  plora_segment writes no
// tile longer than kSmallTile for a batch this small, but a caller's own list
// may: ANY takes tiles of up to kTT tokens; without it (the exchange regions
// hold kSmallTile tokens) a longer one is skipped and counted like an unusable
// entry.
template <bool ANY>
__device__ __forceinline__ int small_tile(const ApplyArgs& g, int u, int s, SmallItem<2>& t,
                                          int& p0) {
  p0 = 0;
  if (u >= g.tile_cap) return 0;
  const int4 ti = g.tiles[u];
  if (ti.x < 0 || ti.x >= g.N || ti.z <= 0 || ti.z > kTT || ti.y < 0 || ti.y + ti.z > g.T)
    return 0;
  const int a = uni(ti.x), L = uni(ti.z);
  p0 = uni(ti.y);
  const int t0 = uni(tile_token(g, p0)), t1 = uni(tile_token(g, p0 + (L > 1 ? 1 : 0)));
  const int r = uni(g.ranks[a]);
  const int64_t ao = g.a_off[a], bo = g.b_off[a];
  const float sc = g.scales[a];
  t.tok[0] = t0;
  t.tok[1] = L > 1 ? t1 : -1;
  bool bad;
  const bool ok = small_adapter<2>(g, r, sc, ao, bo, t, bad);
  const bool fits = ANY || L <= kSmallTile;
  if (!ok || !fits) {
    if ((bad || !fits) && s == 0 && g.count_skips) bump(g, 1, (unsigned long long)L);
    return 0;
  }
  return L;
}

template <int TG>
__device__ __forceinline__ SmallItem<TG> narrow(const SmallItem<2>& t) {
  SmallItem<TG> o;
  o.tok[0] = t.tok[0];
  if constexpr (TG > 1) o.tok[1] = t.tok[1];
  o.r = t.r; o.s = t.s; o.Ai = t.Ai; o.Bi = t.Bi;
  o.k0 = t.k0; o.k1 = t.k1; o.j0 = t.j0; o.j1 = t.j1;
  return o;
}

// The item's tokens through f(item of TG tokens, first row of the tile,
// whether it is the last): two at once where the tile has two (MAXL = 2), else
// one by one, which also serves the longer tiles of a caller's own list (ANY,
// see small_tile; a loop over pairs spilled).
template <int MAXL, bool ANY, class F>
__device__ __forceinline__ void small_tokens(const ApplyArgs& g, const SmallItem<2>& t2, int L,
                                             int p0, F&& f) {
  if constexpr (MAXL > 1) {
    if (L == 2) {
      f(narrow<2>(t2), 0, true);
      return;
    }
    if constexpr (!ANY) {
      f(narrow<1>(t2), 0, true);
      return;
    }
  }
  SmallItem<1> t = narrow<1>(t2);
#pragma unroll 1
  for (int l = 0; l < L; ++l) {
    if (l > 0) {
      t.tok[0] = ANY ? uni(tile_token(g, p0 + l)) : t2.tok[1];
      lds_sync();
    }
    f(t, l, l == L - 1);
  }
}

// A whole item of L tokens: x is requested first.
template <int MAXL, bool X, bool DEEP>
__device__ __forceinline__ void small_run(const ApplyArgs& g, const SmallItem<2>& t2, int L, int p0,
                                          void* lds, int s, int S, int slot, uint64_t ep) {
  small_tokens<MAXL, !X>(g, t2, L, p0, [&](const auto& t, int l, bool last) {
    constexpr int TG = std::remove_reference_t<decltype(t)>::kTokens;
    SmallLds<TG>& sm = *reinterpret_cast<SmallLds<TG>*>(lds);
    XRegs<TG> xr;
    x_issue<TG>(g, t.tok, t.k0, min(t.k1, t.k0 + kSXW), xr);
    small_body<TG, X, DEEP>(g, t, xr, sm, s, S, slot, ep, l * PLORA_MAX_RANK, last);
  });
}

// ---- the segmentation inside plora_segment_apply ------------------------------------

// The function of plora_segment for 64 < T <= kSegApplyMax tokens by the whole
// work group (thread t holds token t, then sorted position t).  Words are (key << 8) | t; segment
// and tile starts are found with each wavefront's ballots and combined across
// the wavefronts through LDS (counts for the indices, the last and first start
// for the segment that spans a wavefront boundary).  Each token's adapter
// metadata is requested as soon as its id is in and travels during the
// ranking.  Tile u (kept in lt) is the caller's; every thread calls it.
__device__ __forceinline__ void block_segment(const ApplyArgs& g, const int32_t* idx, int u,
                                              const SegOut& so, bool write, LocalTile& lt) {
  constexpr int NA = kSegApplyMax, NW = NA / 64;
  static_assert(kST == NA, "a thread for each token");
  const int T = g.T, N = g.N;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const bool in = tid < T;
  const int id_in = idx[in ? tid : 0];      // (T >= 1: no branch, so no wait here)
  const int id = in ? id_in : 0;
  const bool valid = in && id >= 0 && id < N;
  const bool none = in && id == -1;
  const bool invalid = in && !valid && !none;
  const int ida = valid ? id : 0;
  const int m_r = g.ranks[ida];
  const float m_s = g.scales[ida];
  const int64_t m_ao = g.a_off[ida], m_bo = g.b_off[ida];
  const uint32_t key = valid ? (uint32_t)id : (uint32_t)N + (in ? 0u : 1u);
  lt.words[tid] = (key << 8) | (uint32_t)tid;
  if (tid == 0) lt.L = 0;
  const int n_none = __syncthreads_count(none);
  const int n_invalid = __syncthreads_count(invalid);
  const uint32_t w = lt.words[tid];
  int rank = 0;
#pragma unroll 8
  for (int q = 0; q < NA; q += 4) {
    const uint4 o = *reinterpret_cast<const uint4*>(lt.words + q);
    rank += (o.x < w) + (o.y < w) + (o.z < w) + (o.w < w);
  }
  lt.sorted[rank] = w;
  lds_sync();
  const uint32_t sw = lt.sorted[tid];
  const uint32_t sprev = lt.sorted[tid > 0 ? tid - 1 : 0];
  const int kp = (int)(sw >> 8), tp = (int)(sw & 255);
  const int n_valid = T - n_none - n_invalid;
  const bool vp = tid < n_valid;
  const bool sflag = vp && (tid == 0 || (int)(sprev >> 8) != kp);
  const uint64_t bit = uint64_t(1) << lane;
  const uint64_t below = bit - 1, upto = below | bit;
  const uint64_t smask = __ballot(sflag);
  if (lane == 0) {
    lt.wcount[0][wv] = __popcll(smask);
    lt.wlast[wv] = smask ? 64 * wv + 63 - __clzll(smask) : -1;
    lt.wfirst[wv] = smask ? 64 * wv + __ffsll((long long)smask) - 1 : NA;
  }
  lds_sync();
  int seg_before = 0, n_seg = 0, last_before = -1, first_after = NA;
#pragma unroll
  for (int k = 0; k < NW; ++k) {
    n_seg += lt.wcount[0][k];
    if (k < wv) {
      seg_before += lt.wcount[0][k];
      last_before = max(last_before, lt.wlast[k]);
    } else if (k > wv) {
      first_after = min(first_after, lt.wfirst[k]);
    }
  }
  const int cur = seg_before + __popcll(smask & upto) - 1;   // segment of position tid
  const int sstart = (smask & upto) ? 64 * wv + 63 - __clzll(smask & upto) : last_before;
  const uint64_t later = smask & ~upto;
  int send = later ? 64 * wv + __ffsll((long long)later) - 1 : first_after;
  send = min(send, n_valid);                                  // segment end
  const bool tflag = vp && ((tid - sstart) % kSmallTile) == 0;
  const uint64_t tmask_w = __ballot(tflag);
  if (lane == 0) lt.wcount[1][wv] = __popcll(tmask_w);
  lds_sync();
  int tiles_before = 0, n_tiles_all = 0;
#pragma unroll
  for (int k = 0; k < NW; ++k) {
    n_tiles_all += lt.wcount[1][k];
    if (k < wv) tiles_before += lt.wcount[1][k];
  }
  const int tu = tiles_before + __popcll(tmask_w & below);  // tile starting here
  const int n_tiles = min(n_tiles_all, so.tile_cap);
  const int tlen = min(kSmallTile, send - tid);
  if (write) {
    if (in) so.perm[tid] = vp ? tp : -1;
    if (sflag) {
      so.seg_ptr[cur] = tid;
      so.seg_id[cur] = kp;
    }
    for (int q = n_seg + tid; q <= so.cap; q += kST) so.seg_ptr[q] = n_valid;
    for (int q = n_seg + tid; q < so.cap; q += kST) so.seg_id[q] = -1;
    if (tflag && tu < so.tile_cap) so.tiles[tu] = make_int4(kp, tid, tlen, cur);
    for (int q = n_tiles + tid; q < so.tile_cap; q += kST) so.tiles[q] = make_int4(-1, 0, 0, -1);
    if (tid < 8)
      so.meta[tid] = tid == 0 ? n_seg : tid == 1 ? n_valid : tid == 2 ? n_none
                   : tid == 3 ? n_invalid : tid == 4 ? n_tiles : 0;
  }
  lt.rank_of[tid] = m_r;
  lt.scale_of[tid] = m_s;
  lt.ao_of[tid] = m_ao;
  lt.bo_of[tid] = m_bo;
  if (tflag && tu == u && u < n_tiles) {     // tile u starts here
    lt.a = kp;
    lt.p0 = tid;
    lt.L = tlen;
  }
}

// Calls f with the launch's variant as compile-time constants (longest
// tile, exchange, deep).
template <class F>
void small_variant(int32_t T, bool x, bool deep, F&& f) {
  using std::bool_constant;
  using one = std::integral_constant<int, 1>;
  using two = std::integral_constant<int, 2>;
  auto with = [&](auto l) {
    if (x) deep ? f(l, bool_constant<true>{}, bool_constant<true>{})
                : f(l, bool_constant<true>{}, bool_constant<false>{});
    else deep ? f(l, bool_constant<false>{}, bool_constant<true>{})
              : f(l, bool_constant<false>{}, bool_constant<false>{});
  };
  tile_tokens(T) == 1 ? with(one{}) : with(two{});
}

// Host launchers of the small-batch kernels.
void launch_small_apply(const SmallArgs& a, unsigned grid, hipStream_t stream);
void launch_small_segment_apply(const SmallArgs& a, const int32_t* idx, const SegOut& so,
                                unsigned grid, hipStream_t stream);
void launch_small_multi(const MultiArgs& m, int32_t S, int32_t J, int32_t gl, int32_t deep, unsigned grid,
                        hipStream_t stream);
void launch_small_shrink(const SmallArgs& a, unsigned grid, hipStream_t stream);
void launch_small_expand(const SmallArgs& a, unsigned grid, hipStream_t stream);

}  // namespace plora_impl

#endif  // PLORA_SMALL_H

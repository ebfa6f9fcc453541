// Split-KV decode attention for gfx950 (section V-B): per partition of
// PLORA_ATTN_CHUNK keys an anchor, a sum of shifted exponentials and an
// unnormalised output (plora_attn_partial), then their exact rescaling into
// the output (plora_attn_merge).  The C ABI is declared in
// include/plora_attention.h.
//
// Decode attention is a pair of matrix-vector products per (request, head):
// it reads every key and value once and does two flops per byte, so it is
// HBM-bound and runs on the vector ALUs; the work is spread so that a batch
// of long caches gives tens of thousands of work groups.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdint>
#include <cstring>

#include "plora_attention.h"

namespace {

constexpr int kD = PLORA_ATTN_HEAD_DIM;   // 128: sixteen 16-byte units per row
constexpr int kC = PLORA_ATTN_CHUNK;      // keys per partition of the ABI
constexpr int kNT = 256;                  // threads per work group
constexpr int kCUs = 256;                 // compute units of the chip
constexpr int kGroups = kNT / 16;         // keys per pass (16 lanes each)
constexpr int kStage = 8;                 // keys per 16-lane group and stage
constexpr int kWholeStage = kC / kGroups; // the same where a partition is one stage
static_assert(kC % (kStage * kGroups) == 0, "partitions are whole stages");

// (the merge takes partials and outputs of any element alignment)
typedef float f32x4_t __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x2_t __attribute__((ext_vector_type(2), aligned(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2), aligned(2)));
typedef uint32_t u32x1_t __attribute__((aligned(2)));
typedef int i32x4_t __attribute__((ext_vector_type(4)));
constexpr int kRsrcWord3 = 0x00020000;    // raw buffer, 32-bit data format (gfx9 family)
constexpr int kCached = 0, kOnce = 2;     // buffer cache policies: default, non-temporal
constexpr int kPastEnd = (int)0x80000000u;

__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// fp32 -> bf16 bits, round to nearest even; NaN stays a quiet NaN.
__device__ __forceinline__ uint32_t to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x007fffffu) != 0u)
    return ((u >> 16) & 0x8000u) | 0x7fc0u;
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}

__device__ __forceinline__ void unpack8(const uint4& v, float f[8]) {
  f[0] = bf_lo(v.x); f[1] = bf_hi(v.x);
  f[2] = bf_lo(v.y); f[3] = bf_hi(v.y);
  f[4] = bf_lo(v.z); f[5] = bf_hi(v.z);
  f[6] = bf_lo(v.w); f[7] = bf_hi(v.w);
}

// The len valid rows of one (request, head) cache as a raw buffer resource:
// a load past them reads zero and fetches nothing, so the partition tail
// needs no branch and nothing outside the valid rows is touched.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_rsrc(const uint16_t* p, int len) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p), 0, len * kD * 2,
                                           kRsrcWord3);
}

// POL: the cache policy (see keep_cached).
template <int POL>
__device__ __forceinline__ uint4 bld16(__amdgpu_buffer_rsrc_t r, int byte_off) {
  const i32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(r, byte_off, 0, POL);
  return make_uint4((uint32_t)v.x, (uint32_t)v.y, (uint32_t)v.z, (uint32_t)v.w);
}

template <int CTRL>
__device__ __forceinline__ float dpp_add(float x) {
  return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}

// Sum over each row of 16 lanes, in every lane of the row (quad permutations,
// then the mirrored half row and row: register moves, where a shuffle by xor
// goes through LDS).
__device__ __forceinline__ float row_sum(float x) {
  x = dpp_add<0xb1>(x);     // quad_perm [1,0,3,2]
  x = dpp_add<0x4e>(x);     // quad_perm [2,3,0,1]
  x = dpp_add<0x141>(x);    // row_half_mirror
  x = dpp_add<0x140>(x);    // row_mirror
  return x;
}

// Partition blockIdx.x (CH keys from blockIdx.x CH) of head blockIdx.y of
// request blockIdx.z.  Thread (g, e) = (tid / 16, tid % 16) takes keys g,
// g + 16, ... of the partition and the dimensions 8 e .. 8 e + 7 of each: the
// sixteen lanes of a key read its row as one coalesced 256-byte line.  A
// stage is ST keys per group, all of whose key and value units are requested
// before any is used; each group keeps its own running maximum, sum and output
// (rescaled once per stage), so the work group's wavefronts meet only at the
// end, where the groups are rescaled to the common anchor.  With out set
// (P = 1) the only partition is the whole cache and is written as the output
// itself.
// The XCDs take the work groups in turn, so where P and 8 have a factor g in
// common a partition number would stay on 8 / g of the XCDs, and the last
// partitions, past most requests' lengths, would leave theirs idle: the
// partitions start at the next one after every 8 / g heads (64 x 32 x
// 512..4096 keys: 507 us at 512-key partitions without, 367 with; 434 and 386
// at 256).  An odd P spreads by itself: turned by one per head, three
// partitions (8 x 32 x 260..520 keys) took 15.4 us against 13.9 in grid order.
// Bound by reading K and V; the loads in flight come from the resident work
// groups (four per compute unit), so no stage is requested ahead of another.
template <int ST, int POL>
__global__ __launch_bounds__(kNT, ST > kStage ? 2 : 4) void attn_partial_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
    const uint16_t* __restrict__ v, const int32_t* __restrict__ lens, int32_t heads,
    int64_t max_len, float scale, int32_t P, int32_t CH, float* __restrict__ m_out,
    float* __restrict__ l_out, float* __restrict__ o_out, uint16_t* __restrict__ out) {
  __shared__ float red[kNT / 64][kD];
  __shared__ float wmax[kNT / 64], wsum[kNT / 64];
  const int h = blockIdx.y, b = blockIdx.z;
  const uint32_t head = (uint32_t)b * (uint32_t)heads + (uint32_t)h;
  const int lg = min(3, (int)__builtin_ctz(P));
  const int p = (int)((blockIdx.x + (lg ? head >> (3 - lg) : 0u)) % (uint32_t)P);
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int g = tid >> 4, e = tid & 15;
  int n = lens[b];
  n = (n < 0 || n > max_len) ? 0 : n;
  const int lo = p * CH;
  if (lo >= n) {                                  // no key here: no partial written
    if (out && tid < kD / 8)
      *reinterpret_cast<uint4*>(out + ((int64_t)b * heads + h) * kD + 8 * tid) =
          make_uint4(0, 0, 0, 0);
    return;
  }
  const int hi = min(n, lo + CH);
  const int64_t row0 = ((int64_t)b * heads + h) * max_len;
  const __amdgpu_buffer_rsrc_t kr = rows_rsrc(k + row0 * kD, n);
  const __amdgpu_buffer_rsrc_t vr = rows_rsrc(v + row0 * kD, n);
  float qf[8];
  unpack8(*reinterpret_cast<const uint4*>(q + ((int64_t)b * heads + h) * kD + 8 * e), qf);
#pragma unroll
  for (int i = 0; i < 8; ++i) qf[i] *= scale;

  float m = -INFINITY, sum = 0.f;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int t0 = lo + g; t0 - g < hi; t0 += ST * kGroups) {
    uint4 kreg[ST], vreg[ST];
#pragma unroll
    for (int j = 0; j < ST; ++j) {
      const int t = t0 + kGroups * j;             // keys past hi read zero
      kreg[j] = bld16<POL>(kr, t < hi ? (t * kD + 8 * e) * 2 : kPastEnd);
    }
#pragma unroll
    for (int j = 0; j < ST; ++j) {
      const int t = t0 + kGroups * j;
      vreg[j] = bld16<POL>(vr, t < hi ? (t * kD + 8 * e) * 2 : kPastEnd);
    }
    // step 1: scores, each summed over the sixteen lanes of its key
    float s[ST];
    float mn = m;
#pragma unroll
    for (int j = 0; j < ST; ++j) {
      float kf[8];
      unpack8(kreg[j], kf);
      float d = 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) d = fmaf(qf[i], kf[i], d);
      d = row_sum(d);
      s[j] = t0 + kGroups * j < hi ? d : -INFINITY;
      mn = fmaxf(mn, s[j]);
    }
    // steps 2 and 3: shifted exponentials, their sum, the weighted values.
    // While every score so far is -inf (no key yet, or scores below the
    // range) the shift is 0: their weights are 0, and a NaN score's is NaN.
    const float ms = mn == -INFINITY ? 0.f : mn;
    const float c = expf(m - ms);
    m = mn;
    sum *= c;
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] *= c;
#pragma unroll
    for (int j = 0; j < ST; ++j) {
      const float w = expf(s[j] - ms);            // 0 for keys past hi
      sum += w;
      float vf[8];
      unpack8(vreg[j], vf);
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] = fmaf(w, vf[i], acc[i]);
    }
  }
  // the partition's anchor, and each group's sums rescaled to it
  float mx = m;
#pragma unroll
  for (int msk = 16; msk < 64; msk <<= 1) mx = fmaxf(mx, __shfl_xor(mx, msk, 64));
  if (lane == 0) wmax[wv] = mx;
  __syncthreads();
  mx = wmax[0];
#pragma unroll
  for (int w = 1; w < kNT / 64; ++w) mx = fmaxf(mx, wmax[w]);
  // (a partition whose every score is -inf has no anchor to shift by: its
  // sums are NaN, as exp(-inf - -inf) is)
  const float c = mx == -INFINITY ? NAN : expf(m - mx);
  sum *= c;
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] *= c;
  // sum: each key counted once (the sixteen lanes of a key hold the same w)
#pragma unroll
  for (int msk = 16; msk < 64; msk <<= 1) sum += __shfl_xor(sum, msk, 64);
#pragma unroll
  for (int msk = 16; msk < 64; msk <<= 1)
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] += __shfl_xor(acc[i], msk, 64);
  if (lane < 16) {
#pragma unroll
    for (int i = 0; i < 8; ++i) red[wv][8 * lane + i] = acc[i];
  }
  if (lane == 0) wsum[wv] = sum;
  __syncthreads();
  const int64_t part = ((int64_t)b * heads + h) * P + p;
  float l = wsum[0];
#pragma unroll
  for (int w = 1; w < kNT / 64; ++w) l += wsum[w];
  if (tid < kD) {
    float o = red[0][tid];
#pragma unroll
    for (int w = 1; w < kNT / 64; ++w) o += red[w][tid];
    if (out) out[part * kD + tid] = (uint16_t)to_bf16(o / l);
    else o_out[part * kD + tid] = o;
  }
  if (tid == 0 && !out) {
    m_out[part] = mx;
    l_out[part] = l;
  }
}

// The rescaling: one work group per (request, head).  Thread (g, e) = (tid /
// 32, tid % 32) takes the output dimensions 4 e .. 4 e + 3 of partitions g,
// g + G, ...; the G groups are then summed in ascending order through LDS.
// With one thread per dimension walking every partition, a cache of 30k keys
// took 30 us for its 118 dependent rounds.
template <int G>
__global__ __launch_bounds__(32 * G) void attn_merge_kernel(
    const float* __restrict__ m_in, const float* __restrict__ l_in,
    const float* __restrict__ o_in, const int32_t* __restrict__ lens, int32_t heads,
    int64_t max_len, int32_t P, int32_t CH, uint16_t* __restrict__ out) {
  __shared__ float4 red[G][32];
  __shared__ float lred[G], mred[G];
  const int h = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
  const int g = tid >> 5, e = tid & 31;
  int n = lens[b];
  n = (n < 0 || n > max_len) ? 0 : n;
  const int np = n > 0 ? (n - 1) / CH + 1 : 0;
  const int64_t base = ((int64_t)b * heads + h) * P;
  // M: every group finds it by itself, over 32 partitions at a time
  float M = -INFINITY;
  for (int p = tid; p < np; p += 32 * G) M = fmaxf(M, m_in[base + p]);
#pragma unroll
  for (int msk = 1; msk < 32; msk <<= 1) M = fmaxf(M, __shfl_xor(M, msk, 64));
  if (e == 0) mred[g] = M;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < G; ++q) M = fmaxf(M, mred[q]);
  float L = 0.f;
  float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
  for (int p = g; p < np; p += G) {
    const f32x4_t op = *reinterpret_cast<const f32x4_t*>(o_in + (base + p) * kD + 4 * e);
    const float w = expf(m_in[base + p] - M);
    L = fmaf(w, l_in[base + p], L);
    o.x = fmaf(w, op.x, o.x); o.y = fmaf(w, op.y, o.y);
    o.z = fmaf(w, op.z, o.z); o.w = fmaf(w, op.w, o.w);
  }
  red[g][e] = o;
  if (e == 0) lred[g] = L;
  __syncthreads();
  if (g != 0) return;
#pragma unroll
  for (int q = 1; q < G; ++q) {
    const float4 a = red[q][e];
    o.x += a.x; o.y += a.y; o.z += a.z; o.w += a.w;
    L += lred[q];
  }
  u32x2_t r = {0, 0};
  if (np > 0) {
    r.x = to_bf16(o.x / L) | (to_bf16(o.y / L) << 16);
    r.y = to_bf16(o.z / L) | (to_bf16(o.w / L) << 16);
  }
  *reinterpret_cast<u32x2_t*>(out + ((int64_t)b * heads + h) * kD + 4 * e) = r;
}

// The same for at most kFew partitions: a wavefront per (request, head), two
// dimensions per thread, every partial requested at once: one trip after the
// length and no barrier (3 x 8 x 260..520 keys, three partitions, both steps:
// 8.3 us with the kernel above, 7.9 so).
constexpr int kFew = 4;
__global__ __launch_bounds__(kD / 2) void attn_merge_few_kernel(
    const float* __restrict__ m_in, const float* __restrict__ l_in,
    const float* __restrict__ o_in, const int32_t* __restrict__ lens, int32_t heads,
    int64_t max_len, int32_t P, int32_t CH, uint16_t* __restrict__ out) {
  const int h = blockIdx.x, b = blockIdx.y, e = threadIdx.x;
  int n = lens[b];
  n = (n < 0 || n > max_len) ? 0 : n;
  const int np = n > 0 ? (n - 1) / CH + 1 : 0;    // at most P, which is at most kFew
  const int64_t base = ((int64_t)b * heads + h) * P;
  uint32_t r = 0;
  if (np > 0) {
    float m[kFew], l[kFew];
    f32x2_t o[kFew];
#pragma unroll
    for (int p = 0; p < kFew; ++p) {
      const int64_t q = base + min(p, np - 1);
      m[p] = m_in[q];
      l[p] = l_in[q];
      o[p] = *reinterpret_cast<const f32x2_t*>(o_in + q * kD + 2 * e);
    }
    float M = m[0];
#pragma unroll
    for (int p = 1; p < kFew; ++p) M = fmaxf(M, m[p]);
    float L = 0.f, ox = 0.f, oy = 0.f;
#pragma unroll
    for (int p = 0; p < kFew; ++p) {
      if (p < np) {
        const float w = expf(m[p] - M);
        L = fmaf(w, l[p], L);
        ox = fmaf(w, o[p].x, ox);
        oy = fmaf(w, o[p].y, oy);
      }
    }
    r = to_bf16(ox / L) | (to_bf16(oy / L) << 16);
  }
  *reinterpret_cast<u32x1_t*>(out + ((int64_t)b * heads + h) * kD + 2 * e) = r;
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

std::atomic<int32_t> g_attn_last_error{0};

plora_status launch_status() {
  const hipError_t err = hipGetLastError();
  if (err == hipSuccess) return PLORA_OK;
  g_attn_last_error.store((int32_t)err);
  return PLORA_ERR_HIP;
}

plora_status check_shape(int32_t batch, int32_t heads, int64_t max_len) {
  if (batch < 0 || heads < 0 || max_len < 0) return PLORA_ERR_INVALID_ARG;
  // one (request, head) cache is read through 32-bit byte offsets
  if (max_len * kD * 2 >= (INT64_C(1) << 31)) return PLORA_ERR_UNSUPPORTED;
  return PLORA_OK;
}

int32_t partitions(int64_t max_len, int32_t CH) {
  return max_len <= 0 ? 0 : (int32_t)((max_len + CH - 1) / CH);
}

// Keys per partition of plora_attn_decode's own partials.  Twice the ABI's
// where that still leaves 24 work groups per compute unit (64 requests x 32
// heads x up to 4096 keys: 367 us against 386, half the partials), or where
// one such partition holds the whole cache, so that no merge follows (26 x 16
// x up to 464 keys: 16.1 us against 20.1; 64 x 32 x 300: 29 against 41; a
// single request 8.3 against 11.0); below that the finer split balances
// better (16 requests of 4096: 97.4 us against 98.7, 4 requests 28.5 against
// 31.6).
int32_t decode_chunk(int32_t batch, int32_t heads, int64_t max_len) {
  const int64_t groups = (int64_t)batch * heads * partitions(max_len, 2 * kC);
  return max_len <= 2 * kC || groups >= 24 * kCUs ? 2 * kC : kC;
}

// Whether K and V are read with the default cache policy, so that a cache that
// fits the L2s (32 MB in all) may still be there in the next step, or
// non-temporally: up to 48 MB.  (us per step over one cache, default against
// non-temporal: 8 requests x 8 heads x 600 keys, 20 MB, 8.7 and 9.2; 16 x 8 x
// 600, 39 MB, 10.7 and 12.0; 8 x 32 x 520, 68 MB, 14.2 and 13.9; 64 x 4 x 600,
// 79 MB, 16.1 and 15.5.  A plain read of 2.4 GB runs at 6.3 TB/s by default
// and at 7.1 non-temporally.)
bool keep_cached(int32_t batch, int32_t heads, int64_t max_len) {
  return (int64_t)batch * heads * max_len * (2 * kD * 2) <= (48 << 20);
}

// Whether a partition of kC keys is one stage: where the launch has more work
// groups than are resident at once, a wavefront's second stage is a trip that
// other work groups could have used (128 x 8 x 350..700 keys, 3072 work groups:
// 47.9 us in two stages, 46.4 in one; 16 x 16 x 800..1600, 1792: 30.4 and
// 29.6); below that the smaller kernel is as fast or faster (64 x 4 x 300..600,
// 768: 14.8 and 15.5; 16 x 8 x 1000..2000, 1024: 20.8 and 21.5).
bool whole_stage(int32_t batch, int32_t heads, int32_t P, int32_t CH) {
  return CH == kC && (int64_t)batch * heads * P > 4 * kCUs;
}

plora_status run_partial(const uint16_t* q, const uint16_t* k, const uint16_t* v,
                         const int32_t* lens, int32_t batch, int32_t heads, int64_t max_len,
                         float scale, int32_t CH, float* m, float* l, float* o, uint16_t* out,
                         hipStream_t stream) {
  if (!q || !k || !v || !lens || !m || !l || !o) return PLORA_ERR_INVALID_ARG;
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o))
    return PLORA_ERR_UNSUPPORTED;
  const int32_t P = partitions(max_len, CH);
  auto* kernel = keep_cached(batch, heads, max_len) ? attn_partial_kernel<kStage, kCached>
                 : whole_stage(batch, heads, P, CH) ? attn_partial_kernel<kWholeStage, kOnce>
                                                    : attn_partial_kernel<kStage, kOnce>;
  (void)hipGetLastError();
  hipLaunchKernelGGL(kernel, dim3(P, heads, batch), dim3(kNT), 0, stream, q, k, v,
                     lens, heads, max_len, scale, P, CH, m, l, o, out);
  return launch_status();
}

plora_status run_merge(const float* m, const float* l, const float* o, const int32_t* lens,
                       int32_t batch, int32_t heads, int64_t max_len, int32_t CH,
                       uint16_t* out, hipStream_t stream) {
  if (!m || !l || !o || !lens || !out) return PLORA_ERR_INVALID_ARG;
  const int32_t P = partitions(max_len, CH);
  (void)hipGetLastError();
  if (P <= kFew)
    hipLaunchKernelGGL(attn_merge_few_kernel, dim3(heads, batch), dim3(kD / 2), 0, stream, m, l,
                       o, lens, heads, max_len, P, CH, out);
  else if (P <= 32)
    hipLaunchKernelGGL(attn_merge_kernel<4>, dim3(heads, batch), dim3(128), 0, stream, m, l, o,
                       lens, heads, max_len, P, CH, out);
  else
    hipLaunchKernelGGL(attn_merge_kernel<32>, dim3(heads, batch), dim3(1024), 0, stream, m, l, o,
                       lens, heads, max_len, P, CH, out);
  return launch_status();
}

}  // namespace

extern "C" {

int32_t plora_attn_partitions(int64_t max_len) {
  return max_len <= 0 ? 0 : (int32_t)((max_len + kC - 1) / kC);
}

size_t plora_attn_workspace_bytes(int32_t batch, int32_t heads, int64_t max_len) {
  if (batch <= 0 || heads <= 0 || max_len <= 0) return 0;
  const size_t parts = (size_t)batch * heads * plora_attn_partitions(max_len);
  return align256(parts * 4) * 2 + align256(parts * kD * 4);
}

plora_status plora_attn_partial(const uint16_t* q, const uint16_t* k, const uint16_t* v,
                                const int32_t* lens, int32_t batch, int32_t heads,
                                int64_t max_len, float scale, float* m, float* l, float* o,
                                hipStream_t stream) {
  plora_status st = check_shape(batch, heads, max_len);
  if (st != PLORA_OK) return st;
  if (batch == 0 || heads == 0 || max_len == 0) return PLORA_OK;
  return run_partial(q, k, v, lens, batch, heads, max_len, scale, kC, m, l, o, nullptr, stream);
}

plora_status plora_attn_merge(const float* m, const float* l, const float* o,
                              const int32_t* lens, int32_t batch, int32_t heads,
                              int64_t max_len, uint16_t* out, hipStream_t stream) {
  plora_status st = check_shape(batch, heads, max_len);
  if (st != PLORA_OK) return st;
  if (batch == 0 || heads == 0 || max_len == 0) return PLORA_OK;
  return run_merge(m, l, o, lens, batch, heads, max_len, kC, out, stream);
}

plora_status plora_attn_decode(const uint16_t* q, const uint16_t* k, const uint16_t* v,
                               const int32_t* lens, int32_t batch, int32_t heads,
                               int64_t max_len, float scale, uint16_t* out, void* ws,
                               size_t ws_bytes, hipStream_t stream) {
  plora_status st = check_shape(batch, heads, max_len);
  if (st != PLORA_OK) return st;
  if (batch == 0 || heads == 0 || max_len == 0) return PLORA_OK;
  if (!ws) return PLORA_ERR_INVALID_ARG;
  if (!aligned16(ws)) return PLORA_ERR_UNSUPPORTED;
  if (ws_bytes < plora_attn_workspace_bytes(batch, heads, max_len))
    return PLORA_ERR_WORKSPACE_TOO_SMALL;
  const int32_t CH = decode_chunk(batch, heads, max_len);
  const size_t parts = (size_t)batch * heads * partitions(max_len, CH);
  char* base = reinterpret_cast<char*>(ws);
  float* m = reinterpret_cast<float*>(base);
  float* l = reinterpret_cast<float*>(base + align256(parts * 4));
  float* o = reinterpret_cast<float*>(base + 2 * align256(parts * 4));
  if (!out) return PLORA_ERR_INVALID_ARG;
  const bool whole = partitions(max_len, CH) == 1 && aligned16(out);
  st = run_partial(q, k, v, lens, batch, heads, max_len, scale, CH, m, l, o,
                   whole ? out : nullptr, stream);
  if (st != PLORA_OK || whole) return st;
  return run_merge(m, l, o, lens, batch, heads, max_len, CH, out, stream);
}

}  // extern "C"

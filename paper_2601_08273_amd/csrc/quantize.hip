// Writer for the 8-bit cache format of the fp8 attention calls (a cache-format variant the paper
// does not discuss): a bf16 or fp32 K/V cache becomes E4M3 codes plus one fp32 multiplier per
// (batch element, KV head) and tensor.
//   multiplier = max|x| / 448 over the head's rows (1 when the maximum is 0)
//   code       = the E4M3 value nearest to x / multiplier, ties to the even code
// Two launches: every block reduces |x| over its slice of a head's rows; then every block reduces
// the (few) slice maxima of its head again, encodes its slice and slice 0 stores the multiplier.
// No atomics, no ordering between blocks: the result is deterministic.
// Bound by HBM: the source twice, the codes once.  The second launch walks the slices backwards, so that it begins
// with what the last-level cache still holds of the first, and stores its codes non-temporally, so that they do not
// push the rest out.  Codes by a product and exact corrections instead of divisions, 16 source bytes per lane next to
// its neighbour's (not 32 for 16 codes), eight loads in flight.  Quantisation and a verification call over the codes,
// us: 4 x 8 heads x 37K rows x 128 342 -> 318 (encoding 189 -> 146: 6.2 TB/s), 2 x 4 heads x 71K 177 -> 160, 3 x 8 heads x
// 21K 156 -> 133; forward order with plain stores 322, 176 and 144.  Groups of heads small enough for the 256 MB cache,
// encoded beside the maxima of the next group, were slower: 337-362 at 48 to 200 MB a group.
#include "common.h"

namespace hippo {

constexpr int kQuantThreads = 256;

// 16-byte source vectors per row and elements per vector, for T = float or bf16 bits
template <typename T>
__device__ __forceinline__ float vec_absmax(const u32x4& v) {
  float x[Elem<T>::kPerVec];
  Elem<T>::unpack(v, x);
  float m = 0.f;
#pragma unroll
  for (int i = 0; i < Elem<T>::kPerVec; ++i) m = fmaxf(m, fabsf(x[i]));   // NaN inputs are ignored
  return m;
}

__device__ __forceinline__ float block_max_256(float v, float* red) {
  v = wave_max(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}

// Which rows of which tensor slice `slice` of block row (y, z) of the grid (n_slices, 2 * Hkv, B) covers, in 16-byte
// source vectors: y = 2 * hk + (0 = K, 1 = V)
struct QuantSlice {
  int which, hk, b;
  int vshift, vmask;          // a row holds 2^vshift vectors (head dims 64 and 128): rows and vectors part by a shift
  long long lo, hi;
};
template <typename T>
__device__ __forceinline__ QuantSlice quant_slice(const QuantParams& p, int slice, int y, int z) {
  QuantSlice q;
  q.which = y & 1;
  q.hk = y >> 1;
  q.b = z;
  q.vshift = __builtin_ctz(p.D / Elem<T>::kPerVec);
  q.vmask = (1 << q.vshift) - 1;
  const long long n_vec = (long long)p.n_rows << q.vshift;
  const long long per = (n_vec + p.n_slices - 1) / p.n_slices;
  q.lo = (long long)slice * per;
  q.hi = min(n_vec, q.lo + per);
  return q;
}
template <typename T>
__device__ __forceinline__ const T* quant_src(const QuantParams& p, const QuantSlice& q) {
  return (const T*)(q.which ? p.v_src : p.k_src) + (long long)q.b * p.ssb + (long long)q.hk * p.ssh;
}
// slice maxima of a head's K or V
__device__ __forceinline__ float* quant_partials(const QuantParams& p, const QuantSlice& q) {
  return p.partial + ((long long)(q.b * p.Hkv + q.hk) * 2 + q.which) * p.n_slices;
}

constexpr int kQuantInFlight = 8;   // source vectors in flight per thread

template <typename T>
__global__ __launch_bounds__(kQuantThreads) void kv_absmax(QuantParams p) {
  __shared__ float red[4];
  constexpr int PV = Elem<T>::kPerVec, N = kQuantInFlight;
  const QuantSlice q = quant_slice<T>(p, blockIdx.x, blockIdx.y, blockIdx.z);
  const T* src = quant_src<T>(p, q);
  float m = 0.f;
  for (long long e0 = q.lo + threadIdx.x; e0 < q.hi; e0 += N * kQuantThreads) {
    u32x4 v[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const long long e = min(e0 + u * kQuantThreads, q.hi - 1);     // past the slice: a repeat, which changes no maximum
      v[u] = *(const u32x4*)(src + (e >> q.vshift) * p.ssn + ((int)e & q.vmask) * PV);
    }
#pragma unroll
    for (int u = 0; u < N; ++u) m = fmaxf(m, vec_absmax<T>(v[u]));
  }
  m = block_max_256(m, red);
  if (threadIdx.x == 0) quant_partials(p, q)[blockIdx.x] = m;
}

// two floats -> two E4M3 codes in the low half of the result (round to nearest even)
__device__ __forceinline__ unsigned encode2(float a, float b) {
  return (unsigned)__builtin_amdgcn_cvt_pk_fp8_f32(a, b, 0, false) & 0xffffu;
}

// x / mult, correctly rounded, for a multiplier away from the ends of the exponent range (r = 1 / mult, rounded).
// The product x * r is off by at most one and a half units in the last place; a correction by the exact remainder
// makes it the rounded quotient: one for the 8-bit significands of bf16 (all 2^30 pairs of significands checked), two
// for fp32, where the first leaves an error below a unit and the second then rounds correctly (Markstein 1990).
// Four resp. six instructions instead of the division's ten; magnitudes too small for an exact remainder have code 0
// either way, and zeros and NaNs keep their sign.
template <typename T>
__device__ __forceinline__ float quotient(float x, float mult, float r) {
  float n = x * -r;                                         // minus the quotient, approximately
  if constexpr (sizeof(T) == 4) n = fmaf(fmaf(n, mult, x), -r, n);
  return __builtin_copysignf(fmaf(fmaf(n, mult, x), r, -n), x);
}

template <typename T, bool EXACT_DIV>
__device__ __forceinline__ void encode_vectors(const QuantParams& p, const QuantSlice& q, float mult) {
  constexpr int PV = Elem<T>::kPerVec, N = kQuantInFlight;
  const T* src = quant_src<T>(p, q);
  unsigned char* dst = (unsigned char*)(q.which ? p.v_dst : p.k_dst) + (long long)q.b * p.dsb + (long long)q.hk * p.dsh;
  const float r = 1.0f / mult;
  for (long long e0 = q.lo + threadIdx.x; e0 < q.hi; e0 += N * kQuantThreads) {
    u32x4 raw[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const long long e = min(e0 + u * kQuantThreads, q.hi - 1);     // past the slice: a repeat, not stored
      raw[u] = *(const u32x4*)(src + (e >> q.vshift) * p.ssn + ((int)e & q.vmask) * PV);
    }
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const long long e = e0 + u * kQuantThreads;
      if (e >= q.hi) break;
      float x[PV];
      Elem<T>::unpack(raw[u], x);
#pragma unroll
      for (int i = 0; i < PV; ++i) x[i] = EXACT_DIV ? x[i] / mult : quotient<T>(x[i], mult, r);
      unsigned w[PV / 4];
#pragma unroll
      for (int i = 0; i < PV / 4; ++i) w[i] = encode2(x[4 * i], x[4 * i + 1]) | (encode2(x[4 * i + 2], x[4 * i + 3]) << 16);
      unsigned char* at = dst + (e >> q.vshift) * p.dsn + ((int)e & q.vmask) * PV;
      if constexpr (PV == 8)
        __builtin_nontemporal_store((unsigned long long)w[0] | (unsigned long long)w[1] << 32, (unsigned long long*)at);
      else
        __builtin_nontemporal_store(w[0], (unsigned*)at);
    }
  }
}

template <typename T>
__global__ __launch_bounds__(kQuantThreads) void kv_encode(QuantParams p) {
  __shared__ float red[4];
  // the last blocks of the maxima's launch first
  const QuantSlice q = quant_slice<T>(p, gridDim.x - 1 - blockIdx.x, gridDim.y - 1 - blockIdx.y, gridDim.z - 1 - blockIdx.z);
  // the head's maximum from the slice maxima (at most kQuantThreads of them)
  const float amax = block_max_256((int)threadIdx.x < p.n_slices ? quant_partials(p, q)[threadIdx.x] : 0.f, red);
  const float mult = amax > 0.f ? amax / 448.0f : 1.0f;
  if (q.lo == 0 && threadIdx.x == 0) (q.which ? p.v_scale : p.k_scale)[q.b * p.Hkv + q.hk] = mult;
  if (mult >= 0x1p-80f && mult <= 0x1p80f) encode_vectors<T, false>(p, q, mult);
  else encode_vectors<T, true>(p, q, mult);
}

int quant_slices(int n_rows, int head_dim) {
  // about 16 KB of codes per block, at most one slice per thread of the second reduction
  const long long codes = (long long)n_rows * head_dim;
  long long n = (codes + 16383) / 16384;
  if (n < 1) n = 1;
  if (n > kQuantThreads) n = kQuantThreads;
  return (int)n;
}

hipError_t launch_quantize(const QuantParams& p, hipStream_t st) {
  dim3 grid(p.n_slices, 2 * p.Hkv, p.B);
  if (p.src_dtype == HIPPO_DTYPE_BF16) {
    hipLaunchKernelGGL(kv_absmax<uint16_t>, grid, dim3(kQuantThreads), 0, st, p);
    hipLaunchKernelGGL(kv_encode<uint16_t>, grid, dim3(kQuantThreads), 0, st, p);
  } else {
    hipLaunchKernelGGL(kv_absmax<float>, grid, dim3(kQuantThreads), 0, st, p);
    hipLaunchKernelGGL(kv_encode<float>, grid, dim3(kQuantThreads), 0, st, p);
  }
  return hipGetLastError();
}

}  // namespace hippo

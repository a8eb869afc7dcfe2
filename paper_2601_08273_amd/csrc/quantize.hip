// Writer for the 8-bit cache format of the fp8 attention calls (a cache-format variant the paper
// does not discuss): a bf16 or fp32 K/V cache becomes E4M3 codes plus one fp32 multiplier per
// (batch element, KV head) and tensor.
//   multiplier = max|x| / 448 over the head's rows (1 when the maximum is 0)
//   code       = the E4M3 value nearest to x / multiplier, ties to the even code
// No result depends on an order between blocks: deterministic.
// Bound by HBM: codes by a product and exact corrections instead of divisions, 16 source bytes per lane next to its
// neighbour's (not 32 for 16 codes).  Large sources are read once (kv_quantize_once below).  Small ones, many short heads, and
// heads of more than 48 MB take two launches: every block reduces |x| over its slice of a head's rows; then every block
// reduces the (few) slice maxima of its head again, encodes its slice and slice 0 stores the multiplier.  The second launch
// walks the slices backwards, so that it begins with what the last-level cache still holds of the first, and stores its
// codes non-temporally, so that they do not push the rest out; eight loads in flight.  Quantisation and a verification call over
// the codes, us, two launches -> one sweep: 4 x 8 heads x 37K rows x 128 315 -> 239, 2 x 4 heads x 71K 156 -> 126, 3 x 8
// heads x 21K 135 -> 111, 1 x 8 x 130K 295 -> 226.
#include "common.h"

namespace hippo {

constexpr int kQuantThreads = 256;
constexpr int kQuantMaxSlices = 256;       // of a head: one a thread where the head's maximum is put together

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

// max|x| over this thread's vectors of a slice
template <typename T, int THREADS, int N>
__device__ __forceinline__ float slice_absmax(const T* src, const QuantParams& p, const QuantSlice& q) {
  constexpr int PV = Elem<T>::kPerVec;
  float m = 0.f;
  for (long long e0 = q.lo + threadIdx.x; e0 < q.hi; e0 += N * THREADS) {
    u32x4 v[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const long long e = min(e0 + u * THREADS, q.hi - 1);             // past the slice: a repeat, which changes no maximum
      v[u] = *(const u32x4*)(src + (e >> q.vshift) * p.ssn + ((int)e & q.vmask) * PV);
    }
#pragma unroll
    for (int u = 0; u < N; ++u) m = fmaxf(m, vec_absmax<T>(v[u]));
  }
  return m;
}

template <typename T>
__global__ __launch_bounds__(kQuantThreads) void kv_absmax(QuantParams p) {
  __shared__ float red[4];
  const QuantSlice q = quant_slice<T>(p, blockIdx.x, blockIdx.y, blockIdx.z);
  const float m = block_max_256(slice_absmax<T, kQuantThreads, kQuantInFlight>(quant_src<T>(p, q), p, q), red);
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

// the codes of one source vector, and their store past the caches
template <typename T> struct VecCodes { unsigned w[Elem<T>::kPerVec / 4]; };
template <typename T, bool EXACT_DIV>
__device__ __forceinline__ VecCodes<T> encode_vec(const u32x4& raw, float mult, float r) {
  constexpr int PV = Elem<T>::kPerVec;
  float x[PV];
  Elem<T>::unpack(raw, x);
#pragma unroll
  for (int i = 0; i < PV; ++i) x[i] = EXACT_DIV ? x[i] / mult : quotient<T>(x[i], mult, r);
  VecCodes<T> c;
#pragma unroll
  for (int i = 0; i < PV / 4; ++i) c.w[i] = encode2(x[4 * i], x[4 * i + 1]) | (encode2(x[4 * i + 2], x[4 * i + 3]) << 16);
  return c;
}
template <typename T>
__device__ __forceinline__ void store_codes(unsigned char* at, const VecCodes<T>& c) {
  if constexpr (Elem<T>::kPerVec == 8) {
    const unsigned long long v = (unsigned long long)c.w[0] | (unsigned long long)c.w[1] << 32;
    __builtin_nontemporal_store(v, (unsigned long long*)at);
  } else {
    __builtin_nontemporal_store(c.w[0], (unsigned*)at);
  }
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
      store_codes<T>(dst + (e >> q.vshift) * p.dsn + ((int)e & q.vmask) * PV, encode_vec<T, EXACT_DIV>(raw[u], mult, r));
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

// ---- the slice stays on the chip -------------------------------------------------------------------
// A block fetches its slice once, into registers and LDS, publishes the slice's maximum and encodes when all maxima of its
// head are there, so the source crosses the memory bus once instead of twice.  A word holds a slice's maximum and is its own
// flag: a launch in front sets it to kQuantUnset, which no maximum's bits are, one relaxed device-scope store fills it,
// and the first wave of every block of the head looks at all of them with one load instruction.
// A head's slices stand together in the launch order and are at most half of what the chip holds, so they run beside each
// other while the next heads' slices load.  No result depends on a wait: when `polls` looks in a row have brought nothing new,
// the blocks that wait take the maxima of the missing slices from the source themselves, each of another one, and publish
// them.  That is what other work on the chip comes to, several large quantisations above all: us a call each on streams of
// their own, two launches | one sweep | a sweep whose every block takes all missing maxima for itself: three of 1 x 8 x 196K
// 1198 | 1189 | 24600, four 1577 | 1468 | 25000, two 785 | 730 | 1380; three of 1 x 2 x 196K 306 | 304 | 1800; three of 1 x 8 x 130K
// 789 | 673 | 980; three of 4 x 8 x 37K 820 | 503 | 503.  Twelve looks (20 us) where three sweeps' heads fit the chip, four above:
// there three of 1 x 8 x 196K take 1476 with twelve, and one alone 257.5 with four, 257.0 with twelve.
// What bounds it: HBM, and how many looks the words' memory channels serve; every look of a head goes to the same few
// lines.  4 x 8 heads x 37K rows x 128 (608 MB in, 304 out), us: two launches that read the source twice 254; here without
// any wait 163 (wrong, but the floor), slices of 64 KB whose threads look at a word each every half microsecond 253, whose
// first wave looks for all 218, every two microseconds 202, slices of 128 KB 175 to 188, of 256 KB in one block a
// compute unit 205; 24 vectors a thread and three waves a SIMD 177; one word and one counter a head by atomics 410.  What
// waits is what the chip holds: 64 KB of LDS a block beside its registers 175 (5.2 TB/s), 1 x 8 x 130K 201 -> 170, 2 x 4 x 71K
// 110 -> 90, 3 x 8 x 21K 76 -> 72, 2 x 4 x 33K of fp32 83 -> 73; 72 KB no better, 32 KB half of it.
constexpr unsigned kQuantUnset = 0xffffffffu;
constexpr int kQuantHeld = 16;               // source vectors held per thread in registers (64 of them: four waves a SIMD)
constexpr int kQuantLds = 8;                 // ... and in LDS
constexpr int kQuantHelped = 3;              // looks without a new word after the first slice that a block has helped out with
constexpr int kQuantOnceThreads = 512;       // two blocks of 192 KB a compute unit

// words of a head: whole vectors of four
__host__ __device__ constexpr int quant_words(int n_slices) { return (n_slices + 3) / 4 * 4; }

__global__ __launch_bounds__(kQuantThreads) void quant_clear(unsigned* words, int n) {
  const int i = blockIdx.x * kQuantThreads + threadIdx.x;
  if (i < n) words[i] = kQuantUnset;
}

template <int THREADS>
__device__ __forceinline__ float block_max(float v, float* red) {
  v = wave_max(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  float m = red[0];
#pragma unroll
  for (int w = 1; w < THREADS / 64; ++w) m = fmaxf(m, red[w]);
  return m;
}

// A thread's vectors lie THREADS apart: a whole number of rows, so one address and a step reach them all.
template <typename T, bool EXACT_DIV>
__device__ __forceinline__ void encode_held(unsigned char* dst, long long step, int count, const u32x4 (&raw)[kQuantHeld],
                                            const u32x4* rest, float mult) {
  const float r = 1.0f / mult;
#pragma unroll
  for (int u = 0; u < kQuantHeld; ++u) {
    if (u < count) store_codes<T>(dst, encode_vec<T, EXACT_DIV>(raw[u], mult, r));
    dst += step;
  }
#pragma unroll
  for (int u = 0; u < kQuantLds; ++u) {
    if (kQuantHeld + u < count) store_codes<T>(dst, encode_vec<T, EXACT_DIV>(rest[u * kQuantOnceThreads], mult, r));
    dst += step;
  }
}

// The maxima of a head's slices, four a lane (0 where there is none).  Bit i of the result: this lane's word i is missing.
// Waits while words keep coming: until `polls` looks in a row have brought none.
__device__ __forceinline__ unsigned look_for_maxima(const unsigned* words, int n_slices, const int polls, float& m) {
  const int lane = threadIdx.x & 63, at = 4 * lane;
  u32x4 w = {kQuantUnset, kQuantUnset, kQuantUnset, kQuantUnset};
  auto unset = [&] {
    unsigned bits = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) bits |= (w[i] == kQuantUnset && at + i < n_slices ? 1u : 0u) << i;
    return bits;
  };
  unsigned missing = unset();
  for (int left = polls; left > 0 && __any(missing != 0); --left) {
    if (left < polls) __builtin_amdgcn_s_sleep(64);                     // 4096 clocks
    // (lanes beyond the last word look at the first ones; a line of words is whole lanes' worth)
    asm volatile("global_load_dwordx4 %0, %1, off sc1\n\ts_waitcnt vmcnt(0)"
                 : "=&v"(w) : "v"(words + (at < n_slices ? at : 0)) : "memory");
    const unsigned now = unset();
    if (__any(now != missing)) left = polls;
    missing = now;
  }
  m = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (at + i < n_slices && w[i] != kQuantUnset) m = fmaxf(m, __uint_as_float(w[i]));
  return missing;
}

// The slice of the `turn`-th missing word of the wave, counted modulo their number; -1: none is missing.
__device__ __forceinline__ int missing_slice(unsigned missing, unsigned turn) {
  if (!__any(missing != 0)) return -1;
  const int lane = threadIdx.x & 63, own = __popc(missing);
  int up_to = own;
#pragma unroll
  for (int d = 1; d < 64; d *= 2) {
    const int below = __shfl_up(up_to, d, 64);
    if (lane >= d) up_to += below;
  }
  const int all = __shfl(up_to, 63, 64);
  int rank = (int)(turn % (unsigned)all) - (up_to - own), at = -1;      // among this lane's
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (missing >> i & 1 && rank-- == 0) at = 4 * lane + i;
  return __shfl(at, __ffsll((unsigned long long)__ballot(at >= 0)) - 1, 64);
}

template <typename T, bool PAST>
__global__ __launch_bounds__(kQuantOnceThreads, 4) void kv_quantize_once(QuantParams p) {
  __shared__ float red[2][kQuantOnceThreads / 64];
  __shared__ int help;
  __shared__ u32x4 rest_s[kQuantLds * kQuantOnceThreads];               // [vector][thread]: each its own
  constexpr int PV = Elem<T>::kPerVec, N = kQuantHeld, THREADS = kQuantOnceThreads;
  const int tid = threadIdx.x;
  const QuantSlice q = quant_slice<T>(p, blockIdx.x, blockIdx.y, blockIdx.z);
  const T* src = quant_src<T>(p, q);
  const long long e0 = q.lo + tid;
  const int count = e0 < q.hi ? (int)((q.hi - e0 + THREADS - 1) / THREADS) : 0;     // this thread's vectors, at most N and 8
  u32x4 raw[N];
  {
    const long long e = min(e0, q.hi - 1);
    const T* at = src + (e >> q.vshift) * p.ssn + ((int)e & q.vmask) * PV;
    const long long step = (long long)(THREADS >> q.vshift) * p.ssn;
#pragma unroll
    for (int u = 0; u < N; ++u) {                                       // past the slice: a repeat, not stored
      raw[u] = PAST ? __builtin_nontemporal_load((const u32x4*)at) : *(const u32x4*)at;
      if (u + 1 < count) at += step;
    }
#pragma unroll
    for (int u = 0; u < kQuantLds; ++u) {
      dma16<PAST>(at, (unsigned)(uintptr_t)rest_s + (u * THREADS + (tid & ~63)) * 16);
      if (N + u + 1 < count) at += step;
    }
  }
  const u32x4* const rest = rest_s + tid;
  float m = 0.f;
#pragma unroll
  for (int u = 0; u < N; ++u) m = fmaxf(m, vec_absmax<T>(raw[u]));
#pragma unroll
  for (int u = 0; u < N; ++u) asm volatile("" : "+v"(raw[u]));          // held as they came, not unpacked
  wait_vmcnt<0>();
#pragma unroll
  for (int u = 0; u < kQuantLds; ++u) m = fmaxf(m, vec_absmax<T>(rest[u * THREADS]));
  m = block_max<THREADS>(m, red[0]);
  if (p.n_slices > 1) {
    unsigned* words = (unsigned*)p.partial + ((long long)(q.b * p.Hkv + q.hk) * 2 + q.which) * quant_words(p.n_slices);
    if (tid == 0) __hip_atomic_store(words + blockIdx.x, __float_as_uint(m), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    auto look = [&](int polls) {                                        // the maxima that are there, and a slice whose is not
      if (tid < 64) {
        float others;
        const int slice = missing_slice(look_for_maxima(words, p.n_slices, polls, others), blockIdx.x);
        others = wave_max(others);
        if (tid == 0) { red[1][0] = others; help = slice; }
      }
      __syncthreads();
    };
    look(p.polls);
    // The blocks that wait in vain share the missing slices: each takes the maximum of another one and publishes it, unless it
    // is there by then (a maximum has the same bits whoever takes it).  So one word more is there when it looks again.
    if (help >= 0)
      do {
        const float here = block_max<THREADS>(slice_absmax<T, THREADS, 4>(src, p, quant_slice<T>(p, help, blockIdx.y, blockIdx.z)), red[0]);
        unsigned unset = kQuantUnset;
        if (tid == 0)
          __hip_atomic_compare_exchange_strong(words + help, &unset, __float_as_uint(here), __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();                                                // `help` and `red` are free again
        look(kQuantHelped);
      } while (help >= 0);
    m = fmaxf(m, red[1][0]);
  }
  const float mult = m > 0.f ? m / 448.0f : 1.0f;
  if (blockIdx.x == 0 && tid == 0) (q.which ? p.v_scale : p.k_scale)[q.b * p.Hkv + q.hk] = mult;
  unsigned char* dst = (unsigned char*)(q.which ? p.v_dst : p.k_dst) + (long long)q.b * p.dsb + (long long)q.hk * p.dsh +
                       (e0 >> q.vshift) * p.dsn + ((int)e0 & q.vmask) * PV;
  const long long step = (long long)(THREADS >> q.vshift) * p.dsn;
  if (mult >= 0x1p-80f && mult <= 0x1p80f) encode_held<T, false>(dst, step, count, raw, rest, mult);
  else encode_held<T, true>(dst, step, count, raw, rest, mult);
}

// From how many source bytes on the slices stay on the chip, and are fetched past the caches.  us, two launches -> one sweep,
// source from HBM: 23 MiB 15.1 -> 17.3, 32 18.9 -> 19.2, 39 21.7 -> 20.6, 47 25.4 -> 21.6, 64 34.1 -> 30.9 (8 heads of 33K rows)
// and 30.7 -> 28.0 (64 of 4K), 78 39 -> 33, 129 61 -> 49, 781 371 -> 250; from the last-level cache: 23 13.7 -> 14.5, 32 17.6 ->
// 15.9, 64 31.6 -> 25.9.  Slices of 64 KB, more blocks, lose to two launches at 32 MiB (23.6) and above.
// Fetched past the caches, up to 256 MiB are 2 % faster from HBM and 3 to 10 % slower where that cache holds them.
// Many short heads leave a block little to hold, and two launches have more blocks on a compute unit.  One sweep's time in two
// launches', by the bytes of a head, over 38 to 250 MiB of bf16: 16 KB 1.27 to 1.40, 20 KB 1.13 to 1.16, 24 KB 1.01 to 1.11, 26 KB 0.95
// to 1.00, 32 KB 0.85 to 0.91, 64 KB 0.64 to 0.75; over 262 | 300 | 400 | 600 MiB: 24 KB 1.55 | 1.58 | 1.48 | 1.48, 40 KB 1.12 | 1.07 | 1.08 |
// 1.01, 44 KB 1.07 | 1.04 | 1.02 | 0.94, 48 KB 1.02 | 0.99 | 0.97 | 0.89, 56 KB 0.94 | 0.93 | 0.88 | 0.85.  (2048 x 102 rows x 64 23.7 -> 36.3 us.)
constexpr long long kQuantOnceBytes = 36ll << 20, kQuantPastBytes = 256ll << 20;
constexpr long long kQuantOnceHead = 26ll << 10, kQuantPastHead = 50ll << 10;

int quant_slices(int n_rows, int head_dim) {
  // about 16 KB of codes per block, at most one slice per thread of the second reduction
  const long long codes = (long long)n_rows * head_dim;
  long long n = (codes + 16383) / 16384;
  if (n < 1) n = 1;
  if (n > kQuantMaxSlices) n = kQuantMaxSlices;
  return (int)n;
}

template <typename T>
static void launch(QuantParams p, hipStream_t st) {
  const long long n_vec = (long long)p.n_rows * (p.D / Elem<T>::kPerVec), heads = 2ll * p.Hkv * p.B;
  constexpr long long held = (long long)kQuantOnceThreads * (kQuantHeld + kQuantLds);
  const bool past = heads * n_vec * 16 >= kQuantPastBytes;
  if (n_vec <= kQuantMaxSlices * held && heads * n_vec * 16 >= kQuantOnceBytes && n_vec * 16 >= (past ? kQuantPastHead : kQuantOnceHead)) {
    p.n_slices = (int)((n_vec + held - 1) / held);       // no more words than quant_slices, in whole vectors
    if (p.polls < 0) p.polls = 3 * p.n_slices > 2 * kNumCU ? 4 : 12;
    const dim3 grid(p.n_slices, 2 * p.Hkv, p.B);
    const int words = (int)heads * quant_words(p.n_slices);
    if (p.n_slices > 1)
      hipLaunchKernelGGL(quant_clear, dim3((words + kQuantThreads - 1) / kQuantThreads), dim3(kQuantThreads), 0, st,
                         (unsigned*)p.partial, words);
    if (past)
      hipLaunchKernelGGL((kv_quantize_once<T, true>), grid, dim3(kQuantOnceThreads), 0, st, p);
    else
      hipLaunchKernelGGL((kv_quantize_once<T, false>), grid, dim3(kQuantOnceThreads), 0, st, p);
    return;
  }
  const dim3 grid(p.n_slices, 2 * p.Hkv, p.B);
  hipLaunchKernelGGL(kv_absmax<T>, grid, dim3(kQuantThreads), 0, st, p);
  hipLaunchKernelGGL(kv_encode<T>, grid, dim3(kQuantThreads), 0, st, p);
}

hipError_t launch_quantize(const QuantParams& p, hipStream_t st) {
  if (p.src_dtype == HIPPO_DTYPE_BF16) launch<uint16_t>(p, st);
  else launch<float>(p, st);
  return hipGetLastError();
}

}  // namespace hippo

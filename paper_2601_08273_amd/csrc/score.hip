// Semantic-aware token scoring (paper: Method, "Semantic-aware Token Preservation", Eq. 2-7).
//
//   s_attn  (Eq. 2)   two passes over the visual keys: pass 1 finds every text row's softmax
//                     normaliser over the N_v visual keys, pass 2 recomputes the logits and sums
//                     exp(z - lse_row) down the columns.  A block owns a tile of tokens (its keys
//                     stay in registers / LDS) and sweeps all L_txt*G query rows of the KV head.
//   s_temp, s_spa (Eq. 3-6)  one block per crop position and run of frames: the crops pass through
//                     LDS frame by frame; Gram matrices and dot products with the frame before on MFMA
//                     (crops above 32 tokens: a block per crop and frame).
//   fusion (Eq. 7)    one block per frame: per-term mean / population std, z-scores summed.
#include "common.h"

namespace hippo {

// Where pass 1 leaves the (max, sum) of query row r = i*G + g of KV head hk for token tile `tile`:
// tile-major slabs of all Bz*H*L rows in (bz, hk, r) order, so a block writes consecutive floats and
// the merge reads consecutive rows; bz = layer * B + b counts (layer, batch element) pairs when several
// layers are swept in one launch.  row_lse uses the same (bz, hk, r) order.
__device__ __forceinline__ long long sattn_part_at(const ScoreParams& p, int tile, int b, int hk, int r) {
  return (long long)tile * ((long long)p.Bz * p.H * p.L) + ((long long)b * p.Hkv + hk) * ((long long)p.L * p.G) + r;
}

// =================================================================================================
// s_attn, fp32 version (v_mfma_f32_16x16x4_f32: fp32 operands, products and sums).
// PASS 1: row statistics; PASS 2: column sums.  Videos of up to 65536 tokens take sattn_once_body instead (score_once); the
// two sweeps are left for longer ones, for few rows over many tokens, and for runs of rows whose sums it cannot hold.
// Bound by the matrix unit's fp32 rate: 2 * L * H * N_v * D flops a pass against 157 TFLOP/s.  A block's four waves
// (one per SIMD) own 32 tokens each, whose keys stay in registers as A operands, and sweep a run of the KV head's
// query rows in chunks of 32 that travel HBM -> LDS by direct transfers, two chunks deep.  Z^T = K Q^T: contraction
// step (s, c), slot g is channel 16s + 4g + c, so 16 bytes of a row give a lane its operands of four steps; lane
// (row j, group g) ends with tokens tb*16 + 4g + e.  32 tokens a wave are two independent chains of products, which
// is what keeps the unit busy with few waves; 128-token blocks and row runs leave a short video enough blocks.
// The vector-ALU sweep that they replace read LDS for every product: a scoring call of 12K tokens x 28 heads x 64 rows
// x 128 channels 608 -> 178 us (both passes together 570 -> 100), of 3K x 14 heads x 64 rows x 64 channels 135 -> 47.
// =================================================================================================
constexpr int kSaF32Tile = 128;       // tokens per block
constexpr int kSaF32Rows = 32;        // query rows per chunk

template <int D>
struct SattnF32Smem {
  static constexpr int NW = 4, RCH = kSaF32Rows;
  __align__(16) unsigned char Qs[2 * RCH * D * 4];
  float lse_s[2][RCH];
  float wm_s[2][NW][RCH], wl_s[2][NW][RCH];
};

template <int D, int PASS>
__device__ __forceinline__ void sattn_f32_body(const ScoreParams& p, SattnF32Smem<D>& sm, const int tile, const int hk,
                                               const int rs, const int bz) {
  constexpr int NW = SattnF32Smem<D>::NW, TPW = kSaF32Tile / NW, TBW = TPW / 16, RCH = kSaF32Rows;
  constexpr int NS = D / 16;
  constexpr int CPR = D / 4;                       // 16-byte pieces per row
  constexpr int RPI = 64 / CPR;                    // rows per transfer
  constexpr int XPW = RCH / RPI / NW;              // transfers per wave per chunk
  constexpr int CHUNKB = RCH * D * 4;
  unsigned char* Qs = sm.Qs;
  auto& lse_s = sm.lse_s;
  auto& wm_s = sm.wm_s;
  auto& wl_s = sm.wl_s;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 15, g = lane >> 4;
  const int b = bz % p.B, layer = bz / p.B;        // several layers' sweeps share a launch
  const int n0 = tile * kSaF32Tile + wave * TPW;   // first token of this wave
  const int Rs = p.L * p.G;
  const int row_begin = rs * p.rows_per_split, row_end = min(Rs, row_begin + p.rows_per_split);
  const float scale_log2 = rsqrtf((float)D) * kLog2e;
  const bool small_rows = Rs < (1 << 20);
  const float inv_g = __builtin_amdgcn_rcpf((float)p.G);

  const float* qbase = (const float*)p.q_layers[layer] + ((long long)b * p.L * p.H + hk * p.G) * D;
  const unsigned qs_addr = (unsigned)(uintptr_t)Qs;
  float lse_reg = INFINITY;
  // rows past the end re-read the last row: pass 1 does not write their statistics, pass 2 gives them an infinite
  // normaliser.  16-byte piece c of chunk row r lies at c ^ (r & 15).
  auto request_chunk = [&](int buf, int r0) {
#pragma unroll
    for (int u = 0; u < XPW; ++u) {
      const int rr = (wave * XPW + u) * RPI + lane / CPR;
      const int r = min(r0 + rr, Rs - 1);
      const int i = small_rows ? row_div_group(r, inv_g) : r / p.G;
      dma16((const char*)(qbase + ((long long)i * p.H + (r - i * p.G)) * D) + (((lane % CPR) ^ (rr & 15)) * 16),
            qs_addr + buf * CHUNKB + (wave * XPW + u) * 1024);
    }
    if (PASS == 2 && tid < RCH) {
      lse_reg = INFINITY;                          // padding rows contribute exp2(-inf) = 0
      if (r0 + tid < Rs) lse_reg = p.row_lse[((long long)bz * p.Hkv + hk) * Rs + r0 + tid];
    }
  };
  if (row_begin < row_end) request_chunk(0, row_begin);
  f32x4 kop[TBW][NS];
  {
    const float* kbase = (const float*)p.k_layers[layer] + (long long)b * p.sb + (long long)hk * p.sh +
                         (long long)p.vis_off * p.sn + 4 * g;
#pragma unroll
    for (int tb = 0; tb < TBW; ++tb) {
      const float* krow = kbase + (long long)min(n0 + tb * 16 + j, p.Nv - 1) * p.sn;   // in bounds; masked below
#pragma unroll
      for (int s = 0; s < NS; ++s) kop[tb][s] = *(const f32x4*)(krow + 16 * s);
    }
    // settled before the loop: the compiler, which does not count the transfers, would otherwise wait for the keys
    // inside it and with them for the chunk in flight
#pragma unroll
    for (int tb = 0; tb < TBW; ++tb)
#pragma unroll
      for (int s = 0; s < NS; ++s) asm volatile("" : "+v"(kop[tb][s]));
  }
  const bool wave_full = n0 + TPW <= p.Nv;
  float col[TBW][4];
#pragma unroll
  for (int tb = 0; tb < TBW; ++tb)
#pragma unroll
    for (int e = 0; e < 4; ++e) col[tb][e] = 0.f;

  // the waves' (max, sum) of chunk row rr, left in half `h` by the chunk that starts at r0 -> the tile's slab
  auto merge_rows = [&](int h, int r0) {
    if (tid < RCH && r0 + tid < Rs) {
      float mm = -INFINITY, ll = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) mm = max_nan(mm, wm_s[h][w][tid]);
#pragma unroll
      for (int w = 0; w < NW; ++w)
        ll += (wm_s[h][w][tid] == -INFINITY) ? 0.f : wl_s[h][w][tid] * fast_exp2(wm_s[h][w][tid] - mm);
      const long long at = sattn_part_at(p, tile, bz, hk, r0 + tid);
      p.row_m[at] = mm;
      p.row_l[at] = ll;
    }
  };
  int buf = 0;
  for (int r0 = row_begin; r0 < row_end; r0 += RCH, buf ^= 1) {
    wait_vmcnt_lds<0>();                           // this wave's share of the chunk has arrived, its row sums are in LDS
    if (PASS == 2 && tid < RCH) lse_s[buf][tid] = lse_reg;
    __syncthreads();                               // ... and everyone else's; everyone is done with the chunk before
    if (r0 + RCH < row_end) request_chunk(buf ^ 1, r0 + RCH);
    if (PASS == 1 && r0 > row_begin) merge_rows(buf ^ 1, r0 - RCH);
    const unsigned char* Qc = Qs + buf * CHUNKB;
#pragma unroll
    for (int rb = 0; rb < RCH / 16; ++rb) {
      f32x4 z[TBW];
#pragma unroll
      for (int tb = 0; tb < TBW; ++tb) z[tb] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const f32x4 qop = *(const f32x4*)(Qc + (rb * 16 + j) * (D * 4) + (((4 * s + g) ^ j) * 16));
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
          for (int tb = 0; tb < TBW; ++tb)
            z[tb] = __builtin_amdgcn_mfma_f32_16x16x4f32(kop[tb][s][c], qop[c], z[tb], 0, 0, 0);
      }
      if (PASS == 1) {
        if (!wave_full) {
#pragma unroll
          for (int tb = 0; tb < TBW; ++tb)
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (n0 + tb * 16 + 4 * g + e >= p.Nv) z[tb][e] = -INFINITY;
        }
        float zv[TBW * 4];
#pragma unroll
        for (int e = 0; e < TBW * 4; ++e) zv[e] = z[e >> 2][e & 3];
        const float mx = rows4_max(max_nan_of(zv)) * scale_log2;
        const float neg_m = (mx == -INFINITY) ? 0.f : -mx;
        float ps = 0.f;
        {
          // (product and sum rounded one by one here and in pass 2, as the reference's own product is: a fused sum would
          // leave the product's rounding error, beyond any exponent for logits of 1e9 and more)
#pragma clang fp contract(off)
#pragma unroll
          for (int e = 0; e < TBW * 4; ++e) ps += fast_exp2(zv[e] * scale_log2 + neg_m);
        }
        ps = rows4_sum(ps);
        if (g == 0) {
          wm_s[buf][wave][rb * 16 + j] = mx;
          wl_s[buf][wave][rb * 16 + j] = ps;
        }
      } else {
#pragma clang fp contract(off)
        const float lse = lse_s[buf][rb * 16 + j];
#pragma unroll
        for (int tb = 0; tb < TBW; ++tb)
#pragma unroll
          for (int e = 0; e < 4; ++e) col[tb][e] += fast_exp2(z[tb][e] * scale_log2 - lse);
      }
    }
  }
  if (PASS == 1 && row_begin < row_end) {
    __syncthreads();
    merge_rows(buf ^ 1, row_begin + (row_end - row_begin - 1) / RCH * RCH);
  }
  if (PASS == 2) {
#pragma unroll
    for (int tb = 0; tb < TBW; ++tb)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float v = row16_sum(col[tb][e]);     // the 16 rows held by the lanes of each group g
        const int n = n0 + tb * 16 + 4 * g + e;
        if (j == 0 && n < p.Nv)
          p.col_part[((long long)bz * p.Hkv * p.n_rsplit + hk + p.Hkv * rs) * p.Nv + n] = v;
      }
  }
}

// Grid (H_kv, n_tile, n_rsplit * Bz), as the bf16 sweeps
template <int D, int PASS>
__global__ __launch_bounds__(256, 2) void sattn_f32(ScoreParams p) {
  __shared__ SattnF32Smem<D> sm;
  sattn_f32_body<D, PASS>(p, sm, blockIdx.y, blockIdx.x, blockIdx.z % p.n_rsplit, blockIdx.z / p.n_rsplit);
}

// log2 by exponent and significand in [1, 2): the hardware's logarithm of the whole sum, up to 2^100 where no
// maximum was taken out, is rounded towards one side at its own magnitude, for all rows alike, and the column sums
// would keep the bias (their error against 64 bits at logits around 2 powers of two 3.3e-7, 0.6e-7 like this)
__device__ __forceinline__ float log2_of_sum(float tot) {
  const float exponent = (float)(__builtin_amdgcn_frexp_expf(tot) - 1);
  return exponent + __log2f(2.f * __builtin_amdgcn_frexp_mantf(tot));
}

// =================================================================================================
// s_attn in ONE sweep (fp32): the exponentials stay in registers until their rows' sums are known.
//
// The two sweeps form every product twice, because a column wants 1 / (row sum) and a row's sum is known only when every
// block of the KV head has been through the row; in fp32 the products are all the time there is.  Here a block keeps the
// exponentials of its last kOnceHold chunks of 32 rows in registers (16 a lane and chunk, where the products were), adds
// its row sums to a 64-bit word a row in device memory, and adds exponential x 1 / sum to the columns kOnceHold chunks
// later, when the words have counted every tile.
//   The words: bits 0..52 a sum in units of kOnceUnit, bits 53..62 how many tiles have added theirs.  One 64-bit add
// carries both, so nothing relies on the order of two locations, and integer sums do not depend on the order of the
// tiles.  Four words a row, by tile: adds to one word wait for each other (a bf16
// form of this sweep, whose chunks are shorter, took 1140 us with one word a row and 770 with eight).
//   A word takes a tile's sum whole: from kOnceLow on, whose last bit is a unit, up to where the sum of all tiles would leave
// its bits (mean exponentials from 2^-13 to 2^9 at 16384 tokens).  What is outside goes, whole too, to one of kOnceBins words a
// row, each for 20 powers of two.  A wave that has used them, or that waits in vain for the words while a tile of the run
// says that it has, fetches them along with the words.  So a row's sum is that of its tiles' sums rounded no more than twice,
// wherever it lies.  (Rounded to the units of one word a row, they lost up to half a unit a tile: 1.4e-5 of a row that one token
// decides among 65536, whose columns are 1.1e-7 from 64 bits now and were 1.6e-6 with two sweeps.)
//   Waiting: a block waits for the tiles of its own (layer, batch element, KV head, row run), which stand next to each
// other in the launch order, kOnceMaxTiles of them at most.  A wave that has asked for sums once.polls times in all no
// longer waits: its block says so in tile_redo and sattn_f32_redo sweeps that tile again, with all sums known, the same
// operations in the same order.  So every wait ends, and no result depends on a wait, whatever else the GPU runs.
//   Range: a wave's sums up to kOnceMax and row sums from kOnceMin on (logits within some 60 to 80 nats; the exponentials
// below 2^-126 that a row of the least sum loses are 2^-24 of it).  Where any row of a run leaves it, all blocks of the run stop
// (a tile does not add such a sum, says so in run_flags and leaves at the next step; the others at that chunk, whose tiles are
// never all counted), write (max, sum) of their rows as pass 1 does, and the last of them merges these; sattn_f32_redo runs pass 2
// for that run.
//   What that costs, us a call from a graph (3136 tokens x 14 heads, 64 rows; 16384 x 28, 128; 36864 x 28, 40; 4096 x 64, 128): two
// sweeps 31, 308, 265, 222; one, sums in the words 28, 190, 230, 128; in the bins (logits 12 nats and more off, or spread by 6 to
// 12) 34, 209, 280, 138; out of range (100 nats off, or spread by 20 and more) 55 to 72, 407 to 465, 415 to 580, 237 to 282.
// =================================================================================================
constexpr int kOnceHold = 5;           // chunks between a row's exponentials and their columns
constexpr int kOnceCopies = 4;         // words a row
constexpr int kOnceMaxTiles = 512;     // two blocks on every compute unit
constexpr int kOnceCountBit = 53;
constexpr float kOnceLow = 0x1p-6f, kOnceUnit = kOnceLow * 0x1p-23f;
constexpr int kOnceBins = 12, kOnceBinBits = 20, kOnceBinLow = -122;   // powers of two: of a bin, where the first begins
constexpr float kOnceMax = 0x1p115f;   // of a wave's 32 tokens; a row of 512 tiles stays below 2^126, whose inverse is normal
constexpr float kOnceMin = 0x1p-86f;   // of a row
static_assert((unsigned long long)kOnceMaxTiles << (kOnceBinBits + 24) <= 1ull << kOnceCountBit && kOnceMaxTiles < 1 << 10,
              "sums and numbers of all tiles");

template <int D>
struct SattnOnceSmem {
  static constexpr int NW = 4, RCH = kSaF32Rows;
  __align__(16) unsigned char Qs[2][RCH * D * 4];
  __align__(16) unsigned long long word_s[2][kOnceCopies][RCH];   // of the chunk whose columns come next
  float sum_s[2][NW][RCH];                               // the waves' row sums; NaN: out of range
  __align__(16) unsigned long long bin_s[2][kOnceBins][RCH];      // its bins, if asked_s
  __align__(16) unsigned long long own_bin_s[NW][kOnceBins][RCH]; // what a wave that waits has fetched
  int asked_s[2], told_s;                                // (told_s: the block has set the run's flag)
  int state_s[NW];
  int large_s[2];                                        // a wave has met a row out of range, in steps of either parity
  int last_s;
};

enum OnceState { kOnceDone = 0, kOnceGaveUp = 1, kOnceLarge = 2 };

// the power of two that a bin's unit is
__device__ __forceinline__ int once_bin_unit(int bin) { return kOnceBinLow - 23 + kOnceBinBits * bin; }
__device__ __forceinline__ float once_units(unsigned long long word) {
  const unsigned hi = (unsigned)(word >> 32) & ((1u << (kOnceCountBit - 32)) - 1);
  return fmaf((float)hi, 0x1p32f, (float)(unsigned)word);
}

// where sattn_once counts and flags the row run of a block
__device__ __forceinline__ long long once_run(const ScoreParams& p, int hk, int rs, int bz) {
  return ((long long)bz * p.n_rsplit + rs) * p.Hkv + hk;
}

// PUBLISH = false: all words are complete (the redo launch)
template <int D, bool PUBLISH>
__device__ __forceinline__ int sattn_once_body(const ScoreParams& p, const ScoreOnce& once, SattnOnceSmem<D>& sm,
                                               const int tile, const int hk, const int rs, const int bz) {
  constexpr int NW = SattnOnceSmem<D>::NW, RCH = SattnOnceSmem<D>::RCH, H = kOnceHold;
  constexpr int TPW = kSaF32Tile / NW, TBW = TPW / 16;
  constexpr int NS = D / 16;
  constexpr int CPR = D / 4, RPI = 64 / CPR, XPW = RCH / RPI / NW, CHUNKB = RCH * D * 4;
  constexpr int CW = RCH * kOnceCopies;                  // words a chunk
  constexpr int BW = RCH * kOnceBins;                    // bins a chunk
  static_assert(RCH == 32 && CW * 8 == 64 * 16 && BW * 8 % 1024 == 0,
                "a transfer brings a chunk's words, a few its bins; a lane's sum is that of row lane % 32");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 15, g = lane >> 4;
  const int b = bz % p.B, layer = bz / p.B;
  const int n0 = tile * kSaF32Tile + wave * TPW;
  const int Rs = p.L * p.G;
  const int row_begin = rs * p.rows_per_split, row_end = min(Rs, row_begin + p.rows_per_split);
  const int n_chunks = max(0, (row_end - row_begin + RCH - 1) / RCH);
  const float scale_log2 = rsqrtf((float)D) * kLog2e;
  const bool small_rows = Rs < (1 << 20);
  const float inv_g = __builtin_amdgcn_rcpf((float)p.G);
  const float* qbase = (const float*)p.q_layers[layer] + ((long long)b * p.L * p.H + hk * p.G) * D;
  const unsigned qs_addr = (unsigned)(uintptr_t)&sm.Qs[0][0];
  unsigned long long* const words = once.row_word + ((long long)(bz * p.Hkv + hk) * once.row_words + row_begin) * kOnceCopies;
  unsigned long long* const bins =
      once.row_bin + ((long long)(bz * p.Hkv + hk) * once.row_words + row_begin) * kOnceBins;   // [chunk][bin][row]
  unsigned* const run_flags = once.run_flags + 2 * once_run(p, hk, rs, bz);
  auto flag = [&](int which) { __hip_atomic_store(run_flags + which, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };

  auto request_chunk = [&](int c) {                      // into buffer c & 1; rows past the end re-read the last row
#pragma unroll
    for (int u = 0; u < XPW; ++u) {
      const int rr = (wave * XPW + u) * RPI + lane / CPR;
      const int r = min(row_begin + c * RCH + rr, Rs - 1);
      const int i = small_rows ? row_div_group(r, inv_g) : r / p.G;
      dma16((const char*)(qbase + ((long long)i * p.H + (r - i * p.G)) * D) + (((lane % CPR) ^ (rr & 15)) * 16),
            qs_addr + (c & 1) * CHUNKB + (wave * XPW + u) * 1024);
    }
  };
  // (what only bins need is worked out where it is wanted, behind volatile statements: held in registers through the sweep,
  // it took ordinary calls 0.5 % longer)
  auto request_bins = [&](int c, unsigned lds_addr) {
    int at = c * BW, piece = 2 * lane;
    asm volatile("" : "+s"(at), "+v"(piece));
#pragma unroll 1
    for (int i = 0; i < BW * 8 / 1024; ++i) dma16_agent(bins + at + piece + i * 128, lds_addr + i * 1024);
  };
  if (n_chunks > 0) request_chunk(0);
  if (tid == 0) sm.large_s[0] = sm.large_s[1] = sm.told_s = 0;
  f32x4 kop[TBW][NS];
  {
    const float* kbase = (const float*)p.k_layers[layer] + (long long)b * p.sb + (long long)hk * p.sh +
                         (long long)p.vis_off * p.sn + 4 * g;
#pragma unroll
    for (int tb = 0; tb < TBW; ++tb) {
      const float* krow = kbase + (long long)min(n0 + tb * 16 + j, p.Nv - 1) * p.sn;   // in bounds; masked by `start`
#pragma unroll
      for (int s = 0; s < NS; ++s) kop[tb][s] = *(const f32x4*)(krow + 16 * s);
    }
#pragma unroll
    for (int tb = 0; tb < TBW; ++tb)
#pragma unroll
      for (int s = 0; s < NS; ++s) asm volatile("" : "+v"(kop[tb][s]));     // settled before the loop, as in the sweeps
  }
  f32x4 start[TBW], col[TBW];              // where a token's product starts: minus infinity past the last token
#pragma unroll
  for (int tb = 0; tb < TBW; ++tb)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      start[tb][e] = n0 + tb * 16 + 4 * g + e < p.Nv ? 0.f : -INFINITY;
      col[tb][e] = 0.f;
    }
  f32x4 ex[H][2][TBW];                                   // exponentials: [chunk % H][16-row block][16-token block]
  int state = kOnceDone, binned = 0;                     // binned: this wave knows that the run's bins are in use
  int polls = PUBLISH ? once.polls : n_chunks;

  // Start of step c: chunk c, the waves' sums of chunk c - 1 and the words that step c - 1 asked for are there.
  // False: a wave has met a row out of range and the block stops (what other blocks wait for before they find the same
  // has been added).  A wave that is past this step's barrier may be writing the word of this step: the word read here is
  // that of the step before, which nobody writes any more, so that all waves leave at the same step.
  auto begin_step = [&](int c) -> bool {
    // (the wave that added the last sums leaves that one operation, issued after its transfers, in flight)
    if (PUBLISH && c >= 2 && wave == (c & 3)) wait_vmcnt_lds<1>();
    else wait_vmcnt_lds<0>();
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(sm.large_s[(c + 1) & 1])) return false;
    if (c + 1 < n_chunks) request_chunk(c + 1);
    if (PUBLISH && c + 1 >= H && c < n_chunks && wave == (c & 3)) {
      dma16_agent(words + (c + 1 - H) * CW + 2 * lane, (unsigned)(uintptr_t)&sm.word_s[(c + 1) & 1][0][0]);
      if (__builtin_expect(binned, 0)) request_bins(c + 1 - H, (unsigned)(uintptr_t)&sm.bin_s[(c + 1) & 1][0][0]);
      sm.asked_s[(c + 1) & 1] = binned;
    }
    if (PUBLISH && c >= 1 && wave == ((c + 1) & 3)) {
      const float(&s)[NW][RCH] = sm.sum_s[(c - 1) & 1];
      const int rr = lane & (RCH - 1);
      const float tot = (s[0][rr] + s[1][rr]) + (s[2][rr] + s[3][rr]);
      auto one = [](float units) {         // a tile's sum: whole units below 2^53
        const float hi = truncf(units * 0x1p-32f), lo = units - hi * 0x1p32f;
        return (1ull << kOnceCountBit) + ((unsigned long long)(unsigned)hi << 32) + (unsigned)lo;
      };
      const bool mine = lane < RCH && row_begin + (c - 1) * RCH + lane < Rs;
      const bool plain = __float_as_uint(tot) - __float_as_uint(kOnceLow) < once.range;
      if (mine && plain)
        __hip_atomic_fetch_add(words + (c - 1) * CW + (tile & (kOnceCopies - 1)) * RCH + lane, one(tot * (1.f / kOnceUnit)),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (__builtin_expect(__any(mine && !plain), 0)) {
        if (mine && !plain && tot == tot) {
          const int bin = max(__builtin_amdgcn_frexp_expf(tot) - 1 - kOnceBinLow, 0) / kOnceBinBits;
          __hip_atomic_fetch_add(bins + (c - 1) * BW + bin * RCH + lane, one(rintf(ldexpf(tot, -once_bin_unit(bin)))),
                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (!sm.told_s) flag(1);           // (one store a block: one a wave made calls of large logits 1.2 to 1.5 times as long)
        sm.told_s = binned = 1;
        if (__any(mine && tot != tot)) {   // never counted: who waits for this row looks at the flag
          flag(0);
          state = kOnceLarge;
          sm.large_s[c & 1] = 1;
        }
      }
    }
    return true;
  };
  // 1 / sum of rows 16 * rb + j of chunk c, in step c + H; asked: its words were requested by the step before
  auto weights = [&](int c, bool asked, float (&w)[2]) {
    const int rr = lane & (RCH - 1);
    const bool real = row_begin + c * RCH + rr < Rs;
    unsigned count = 0;                    // tiles in the words and bins
    float sum = 0.f;
    auto take_words = [&](auto word_at) {
      unsigned long long word = 0;
#pragma unroll
      for (int k = 0; k < kOnceCopies; ++k) word += word_at(k);
      count = (unsigned)(word >> kOnceCountBit);
      sum = once_units(word) * kOnceUnit;
    };
    auto ask_words = [&]() {
      take_words([&](int k) {
        return __hip_atomic_load(words + c * CW + k * RCH + rr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      });
    };
    auto complete = [&]() { return __all(!real || count == (unsigned)p.n_tile); };
    const unsigned long long(*bins_here)[RCH] = nullptr;
    if (PUBLISH && asked) {
      take_words([&](int k) { return sm.word_s[(c + H) & 1][k][rr]; });
      if (sm.asked_s[(c + H) & 1]) bins_here = sm.bin_s[(c + H) & 1];
    } else if (PUBLISH && n_chunks > 2 && c + 1 < n_chunks) {
      ask_words();                         // added steps ago: looked at without the flags before (24.1 -> 22.7 us a call)
    }
    while (__builtin_expect(state == kOnceDone && !complete(), 0)) {
      if (bins_here == nullptr) {
        // (the flags first, in a trip of their own: asked for along with them, words were read oftener while tiles added to
        // them, and 19320 tokens x 14 heads x 4, 7 rows, two layers took 140 us, not 130)
        const unsigned long long f =
            __hip_atomic_load((const unsigned long long*)run_flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned large = __builtin_amdgcn_readfirstlane((unsigned)f);
        const unsigned in_bins = __builtin_amdgcn_readfirstlane((unsigned)(f >> 32));
        if (large || --polls < 0) {
          state = large ? kOnceLarge : kOnceGaveUp;
          break;
        }
        ask_words();
        if (!in_bins) continue;
        binned = 1;
        request_bins(c, (unsigned)(uintptr_t)&sm.own_bin_s[wave][0][0]);
        wait_vmcnt<0>();
        bins_here = sm.own_bin_s[wave];
      }
      unsigned n = 0;                      // a lane of either half takes half of them
      float part = 0.f;
      int first = (lane / RCH) * (kOnceBins / 2), row = rr;
      asm volatile("" : "+v"(first), "+v"(row));
#pragma unroll
      for (int k = 0; k < kOnceBins / 2; ++k) {
        const int bin = first + k;
        const unsigned long long word = bins_here[bin][row];
        n += (unsigned)(word >> kOnceCountBit);
        part += ldexpf(once_units(word), once_bin_unit(bin));
      }
      count += n + __shfl_xor(n, RCH);
      sum += part + __shfl_xor(part, RCH);
      bins_here = nullptr;
    }
    if (state == kOnceDone && __any(real && !(sum >= kOnceMin))) {
      state = kOnceLarge;
      if (PUBLISH) flag(0);
    }
    if (state == kOnceLarge) sm.large_s[(c + H) & 1] = 1;
    const unsigned inv = __float_as_uint(real ? 1.f / sum : 0.f);
    auto a = __builtin_amdgcn_permlane16_swap(inv, inv, false, false);
    w[0] = __uint_as_float(a[0]);
    w[1] = __uint_as_float(a[1]);
  };
  auto add_columns = [&](const f32x4 (&z)[TBW], float w) {
#pragma unroll
    for (int tb = 0; tb < TBW; ++tb)
#pragma unroll
      for (int e = 0; e < 4; ++e) col[tb][e] = fmaf(z[tb][e], w, col[tb][e]);
  };
  auto produce = [&](int c, f32x4 (&z)[2][TBW]) {
    const unsigned char* Qc = &sm.Qs[c & 1][0];
    float ps[2];
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const f32x4 qop = *(const f32x4*)(Qc + (rb * 16 + j) * (D * 4) + (((4 * s + g) ^ j) * 16));
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
          for (int tb = 0; tb < TBW; ++tb)
            z[rb][tb] = __builtin_amdgcn_mfma_f32_16x16x4f32(kop[tb][s][k], qop[k], s + k == 0 ? start[tb] : z[rb][tb],
                                                             0, 0, 0);
      }
      float t[TBW];
#pragma unroll
      for (int tb = 0; tb < TBW; ++tb) {
#pragma unroll
        for (int e = 0; e < 4; ++e) z[rb][tb][e] = fast_exp2(z[rb][tb][e] * scale_log2);
        t[tb] = (z[rb][tb][0] + z[rb][tb][1]) + (z[rb][tb][2] + z[rb][tb][3]);
      }
      ps[rb] = t[0] + t[1];
    }
    // lane (j, g) -> row 16 * (g & 1) + j
    const float pair = rows_sum_swap16(ps[0], ps[1]), tot = rows_sum_swap32(pair, pair);
    if (lane < RCH) sm.sum_s[c & 1][wave][lane] = tot <= kOnceMax ? tot : NAN;       // (false for NaN)
  };

  bool going = true;
#pragma unroll
  for (int h = 0; h < H; ++h) {
    if (going && h <= n_chunks) going = begin_step(h);
    if (going && h < n_chunks) produce(h, ex[h]);
  }
  for (int c0 = H; c0 < n_chunks + H && going; c0 += H) {
#pragma unroll
    for (int h = 0; h < H; ++h) {
      const int c = c0 + h;
      if (c >= n_chunks + H) break;
      if (c <= n_chunks && !begin_step(c)) {
        going = false;
        break;
      }
      float w[2];
      weights(c - H, c <= n_chunks, w);
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) add_columns(ex[h][rb], w[rb]);
      if (c < n_chunks) produce(c, ex[h]);
    }
  }
  if (lane == 0) sm.state_s[wave] = state;
  __syncthreads();
  int worst = sm.state_s[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) worst = max(worst, sm.state_s[w]);
  __syncthreads();
  if (worst == kOnceDone) {
#pragma unroll
    for (int tb = 0; tb < TBW; ++tb)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float v = row16_sum(col[tb][e]);           // the 16 rows held by the lanes of each group g
        const int n = n0 + tb * 16 + 4 * g + e;
        if (j == 0 && n < p.Nv)
          p.col_part[((long long)bz * p.Hkv * p.n_rsplit + hk + p.Hkv * rs) * p.Nv + n] = v;
      }
  }
  return worst;
}

// block -> tile fastest, then KV head, row run, (layer, batch element): blocks that wait for each other start together
__device__ __forceinline__ void once_block(const ScoreParams& p, unsigned blk, int& tile, int& hk, int& rs, int& bz) {
  const unsigned run = blk / (unsigned)p.n_tile, rest = run / (unsigned)p.Hkv;
  tile = (int)(blk - run * (unsigned)p.n_tile);
  hk = (int)(run - rest * (unsigned)p.Hkv);
  rs = (int)(rest % (unsigned)p.n_rsplit);
  bz = (int)(rest / (unsigned)p.n_rsplit);
}

// the words, run_flags and run_arrived, which lie one behind the other
__global__ __launch_bounds__(256) void sattn_once_clear(u32x4* at, long long n) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i < n) at[i] = (u32x4){0u, 0u, 0u, 0u};
}

template <int D>
__device__ __forceinline__ void sattn_once_block(const ScoreParams& p, const ScoreOnce& once, SattnOnceSmem<D>& sm,
                                                 SattnF32Smem<D>& sweep, const unsigned blk) {
  int tile, hk, rs, bz;
  once_block(p, blk, tile, hk, rs, bz);
  const int state = sattn_once_body<D, true>(p, once, sm, tile, hk, rs, bz);
  if (threadIdx.x == 0) once.tile_redo[blk] = state != kOnceDone;
  if (state == kOnceDone) return;
  // Statistics as pass 1's, for the case that the run's rows are out of range; then every block of the run comes here.
  // (one thread's release and acquire stand for the block's, whose stores and loads the barriers order with it)
  sattn_f32_body<D, 1>(p, sweep, tile, hk, rs, bz);
  __syncthreads();
  if (threadIdx.x == 0)
    sm.last_s = __hip_atomic_fetch_add(once.run_arrived + once_run(p, hk, rs, bz), 1, __ATOMIC_ACQ_REL,
                                       __HIP_MEMORY_SCOPE_AGENT) == p.n_tile - 1;
  __syncthreads();
  if (!sm.last_s) return;
  const int Rs = p.L * p.G, row_begin = rs * p.rows_per_split, row_end = min(Rs, row_begin + p.rows_per_split);
  for (int r = row_begin + (int)threadIdx.x; r < row_end; r += 256) {
    constexpr int NB = 16;                               // tiles in flight: this block is alone with all of them
    float mx = -INFINITY, tot = 0.f;
    for (int t0 = 0; t0 < p.n_tile; t0 += NB) {
      float m[NB], l[NB], to = mx;
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        const long long at = sattn_part_at(p, min(t0 + u, p.n_tile - 1), bz, hk, r);
        m[u] = t0 + u < p.n_tile ? p.row_m[at] : -INFINITY;
        l[u] = t0 + u < p.n_tile ? p.row_l[at] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < NB; ++u) to = max_nan(to, m[u]);
      tot *= mx != -INFINITY ? fast_exp2(mx - to) : 0.f;
#pragma unroll
      for (int u = 0; u < NB; ++u) tot += m[u] != -INFINITY ? l[u] * fast_exp2(m[u] - to) : 0.f;
      mx = to;
    }
    p.row_lse[((long long)bz * p.Hkv + hk) * Rs + r] = mx + log2_of_sum(tot);
  }
}

// The tiles that sattn_once left: all of a run with rows out of range (pass 2), and those that no longer waited.
template <int D>
__global__ __launch_bounds__(256, 2) void sattn_f32_redo(ScoreParams p, ScoreOnce once) {
  if (once.tile_redo[blockIdx.x] == 0) return;
  union Smem {
    SattnOnceSmem<D> once;
    SattnF32Smem<D> sweep;
  };
  __shared__ Smem sm;
  int tile, hk, rs, bz;
  once_block(p, blockIdx.x, tile, hk, rs, bz);
  // (row sums too small, but not one block of the run that waited for them and said so: all wrote statistics)
  if (once.run_flags[2 * once_run(p, hk, rs, bz)] || sattn_once_body<D, false>(p, once, sm.once, tile, hk, rs, bz) == kOnceLarge)
    sattn_f32_body<D, 2>(p, sm.sweep, tile, hk, rs, bz);
}

// =================================================================================================
// s_attn, MFMA version (bf16).  Block = 8 waves x 32 tokens; each wave keeps its 32 keys as MFMA A
// operands in registers for the whole sweep over the query rows, which are staged through LDS in
// chunks of 64 rows.  Z^T = K Q^T: lane (row j, group g) holds tokens tb*16 + 4g + e.
// =================================================================================================
constexpr int kSaMfmaTile = 256;      // tokens per block
constexpr int kSaWaves = 8;           // waves per block, 32 tokens each: two waves per SIMD overlap MFMA and exp

// Row sums of a wave that pass 1 takes without a reference.  Within them the product of logit and scale, rounded at its
// own magnitude, costs no precision: over logits of 0 to 80 powers of two, peaked or spread, offset or not, the column
// sums' error against 64 bits was 0.16 to 1.03 times that of a sweep with the maximum and the plain logarithm wherever
// that exceeded 1e-7.  From 2^-90 to 2^90, where nothing overflows either, it was up to 1.3 times for spread logits of
// more than 20 powers of two, and up to 4 times for rows that one token decides.
constexpr float kPlainMin = 0x1p-12f, kPlainMax = 0x1p14f;
constexpr float kPlainSlack = 0x1p-6f;   // how far outside a wave's last plain sums may lie

// MERGE > 0 (pass 2 of short videos): a block merges the row statistics of its run itself, one row a thread in the trip to
// memory that brings the keys, and keeps the normalisers of all its rows; MERGE: 8-tile groups.  launch_sattn_mfma says when.
template <int D, int PASS, int MERGE = 0>
struct SattnSmem {
  static constexpr int RCH = 64;                 // query rows per LDS chunk
  static constexpr int ROWB = D * 2;             // unpadded rows, 16-byte pieces XOR-swizzled (lds_row_swizzle)
  static constexpr int RDEF = 256;               // pass 1 merges the waves' row statistics every RDEF rows
  __align__(16) unsigned char Qs[2][RCH * ROWB]; // two chunks: the next one lands while this one is multiplied
  float lse_s[MERGE > 0 ? kSaWaves * 64 / RCH : 2][RCH];
  float wm_s[PASS == 1 ? kSaWaves : 1][PASS == 1 ? RDEF : 1];
  float wl_s[PASS == 1 ? kSaWaves : 1][PASS == 1 ? RDEF : 1];
};

template <int D, int PASS, int MERGE = 0>
__device__ __forceinline__ void sattn_mfma_body(const ScoreParams& p, SattnSmem<D, PASS, MERGE>& sm, const int tile,
                                                const int vhk, const int bz) {
  const int b = bz % p.B, layer = bz / p.B;          // several layers' sweeps share a launch
  constexpr int NW = kSaWaves, NT = NW * 64;
  constexpr int TPW = kSaMfmaTile / NW;   // tokens per wave
  constexpr int TBW = TPW / 16;           // 16-token blocks per wave
  constexpr int KS = D / 32;
  constexpr int ROWB = SattnSmem<D, PASS>::ROWB;
  constexpr int CPR = D / 8;
  constexpr int RCH = SattnSmem<D, PASS>::RCH;
  constexpr int RDEF = SattnSmem<D, PASS>::RDEF;
  unsigned char* Qs = &sm.Qs[0][0];
  auto& wm_s = sm.wm_s;
  auto& wl_s = sm.wl_s;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int j = lane & 15, g = lane >> 4;
  const int n0 = tile * kSaMfmaTile + wave * TPW;    // first token of this wave
  const int Rs = p.L * p.G;
  const float scale_log2 = rsqrtf((float)D) * kLog2e;
  // the query rows of a KV head are cut into n_rsplit runs of whole chunks; this block sweeps one
  // (vhk = KV head + H_kv * run)
  const int hk = vhk % p.Hkv, rs = vhk / p.Hkv;
  const int row_begin = rs * p.rows_per_split;
  const int row_end = min(Rs, row_begin + p.rows_per_split);

  const uint16_t* kbase = (const uint16_t*)p.k_layers[layer] + (long long)b * p.sb + (long long)hk * p.sh +
                          (long long)p.vis_off * p.sn;
  // This wave's keys as A operands: token tb*16 + j, head-dim elements (ks*4 + g)*8 .. +8 (which eight
  // elements ride in which slot of a contraction step is free as long as keys and queries agree).
  // An operand register wants 16 bytes of *its own* row in every lane; loaded that way, neighbouring
  // lanes read rows a whole row stride apart and the address unit takes a clock per lane (64 per
  // instruction: the 16 waves of a compute unit would queue there for 3.4 us with nothing to overlap).
  // So the keys are loaded as they lie in memory -- lane l takes piece l % CPR of row l / CPR, a
  // contiguous kilobyte per instruction -- and turned into operand layout through LDS: eight rows
  // at a time through this wave's own 8-row strip of query buffer 0 (swizzled like the query chunks;
  // the first query chunk lands in buffer 1 meanwhile), with no barrier, since a wave's LDS
  // operations complete in order and nobody else touches its strip before the first chunk barrier.
  constexpr int KRPI = 64 / CPR;                   // rows per load instruction
  constexpr int KNI = TPW / KRPI;                  // load instructions per wave
  constexpr int IPR = 8 / KRPI;                    // load instructions per 8-row round
  static_assert(TPW % 8 == 0 && 8 % KRPI == 0 && NW * 8 <= SattnSmem<D, PASS>::RCH, "key strips live in query buffer 0");
  u32x4 kraw[KNI];
#pragma unroll
  for (int i = 0; i < KNI; ++i) {
    int n = n0 + i * KRPI + lane / CPR;
    n = n < p.Nv ? n : p.Nv - 1;                     // in bounds; masked below
    kraw[i] = *(const u32x4*)(kbase + (long long)n * p.sn + (lane % CPR) * 8);
  }
  // the tiles' statistics of one row of the run per thread, in the trip that brings the keys
  constexpr int MS = MERGE > 0 ? MERGE : 1;
  float st_m[8][MS], st_l[8][MS];
  if constexpr (MERGE > 0) {
    const int r = min(row_begin + tid, Rs - 1);
#pragma unroll
    for (int s = 0; s < 8; ++s)
#pragma unroll
      for (int u = 0; u < MS; ++u) {
        const long long at = sattn_part_at(p, min(s + 8 * u, p.n_tile - 1), bz, hk, r);
        st_m[s][u] = p.row_m[at];
        st_l[s][u] = p.row_l[at];
      }
  }
  bool tok_ok[TBW][4];
#pragma unroll
  for (int tb = 0; tb < TBW; ++tb)
#pragma unroll
    for (int e = 0; e < 4; ++e) tok_ok[tb][e] = (n0 + tb * 16 + 4 * g + e) < p.Nv;
  const bool wave_has_tokens = n0 < p.Nv;
  const bool wave_full = n0 + TPW <= p.Nv;

  float col[TBW][4];
#pragma unroll
  for (int tb = 0; tb < TBW; ++tb)
#pragma unroll
    for (int e = 0; e < 4; ++e) col[tb][e] = 0.f;

  // Query rows are staged 64 at a time, straight from memory into LDS (16 bytes per lane, no
  // registers in between): a transfer fills 1 KB, i.e. 64 / CPR whole rows, and the chunk after the
  // current one is requested as soon as every wave has left the chunk before it, so its trip to
  // memory hides behind the MFMAs and a chunk costs one barrier.
  constexpr int RPI = 64 / CPR;                    // rows per transfer
  constexpr int XPW = RCH / RPI / NW;              // transfers per wave per chunk
  static_assert(RCH % (RPI * NW) == 0, "a chunk's transfers must split over the waves");
  static_assert(RCH == 64, "launch_score works out the chunk steps for 64-row chunks");
  constexpr int CHUNKB = RCH * ROWB;
  const unsigned qs_addr = (unsigned)(uintptr_t)Qs;
  float lse_reg = INFINITY;
  // Row r = i*G + g of the KV head lives at ((b*L + i)*H + hk*G + g)*D.  The (i, g) of the rows this
  // lane requests are carried from chunk to chunk (a chunk advances every row by RCH), so the
  // division by G happens once, not per chunk.  Rows past the end re-read the last row: pass 1 does
  // not write their statistics and pass 2 gives them an infinite normaliser.
  const uint16_t* qbase = (const uint16_t*)p.q_layers[layer] + ((long long)b * p.L * p.H + hk * p.G) * D;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  int qi[XPW], qg[XPW], qr[XPW];
  unsigned qpiece[XPW];                            // byte offset of this lane's piece inside its source row
  // (the chunk-to-chunk steps and the last row's coordinates come from the host, a lane's own first
  // division is a float reciprocal where the row numbers allow: 512 blocks x 8 waves dividing ten times
  // each kept every compute unit busy for 2.7 us before its first chunk was requested)
  const int step_i = p.q_step_i, step_g = p.q_step_g;
  const int last_i = p.q_last_i, last_g = p.q_last_g;
  const bool small_rows = Rs < (1 << 20);                       // block-uniform
  const float inv_g = __builtin_amdgcn_rcpf((float)p.G);
#pragma unroll
  for (int u = 0; u < XPW; ++u) {
    const int rr = (wave_u * XPW + u) * RPI + lane / CPR;       // row inside the chunk
    qr[u] = row_begin + rr;
    qi[u] = small_rows ? row_div_group(qr[u], inv_g) : qr[u] / p.G;
    qg[u] = qr[u] - qi[u] * p.G;
    qpiece[u] = (unsigned)(((lane % CPR) ^ lds_row_swizzle<D>(rr)) * 16);
  }
  auto request_chunk = [&](int buf, int r0) {    // must be called with r0 = row_begin, +RCH, +2 RCH, ...
#pragma unroll
    for (int u = 0; u < XPW; ++u) {
      const bool real = qr[u] < Rs;
      const int i = real ? qi[u] : last_i, g2 = real ? qg[u] : last_g;
      dma16((const char*)(qbase + ((long long)i * p.H + g2) * D) + qpiece[u],
            qs_addr + buf * CHUNKB + (wave_u * XPW + u) * 1024);
      qr[u] += RCH;
      qg[u] += step_g;
      const int carry = qg[u] >= p.G ? 1 : 0;
      qg[u] -= carry * p.G;
      qi[u] += step_i + carry;
    }
    if (PASS == 2 && MERGE == 0 && tid < RCH) {
      const int r = r0 + tid;
      lse_reg = INFINITY;                     // padding rows contribute exp2(-inf) = 0
      if (r < Rs) lse_reg = p.row_lse[((long long)bz * p.Hkv + hk) * Rs + r];
    }
  };
  if (row_begin < row_end) request_chunk(1, row_begin);     // (every request is waited for at the top of its chunk)
  int buf = 1;
  bf16x8 kop[TBW][KS];
  {
    unsigned char* strip = Qs + __builtin_amdgcn_readfirstlane(wave) * (8 * ROWB);
    const int wr_row = lane / CPR;                                  // row of the round this lane's piece belongs to (+ ii * KRPI)
#pragma unroll
    for (int r = 0; r < TPW / 8; ++r) {
#pragma unroll
      for (int ii = 0; ii < IPR; ++ii) {
        const int row8 = ii * KRPI + wr_row;
        *(u32x4*)(strip + row8 * ROWB + (((lane % CPR) ^ lds_row_swizzle<D>(row8)) * 16)) = kraw[r * IPR + ii];
      }
      const int tb = r / 2, half = r % 2;                            // rows 8 * half .. of 16-token block tb
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const bf16x8 v = *(const bf16x8*)(strip + (j & 7) * ROWB + (((ks * 4 + g) ^ lds_row_swizzle<D>(j & 7)) * 16));
        if ((j >> 3) == half) kop[tb][ks] = v;
      }
    }
  }
  if constexpr (MERGE > 0) {
    // as sattn_row_lse, in the same order: the same bits.  (Rows past the end: an infinite normaliser.)
    float m8[8], l8[8], mx = -INFINITY, tot = 0.f;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      m8[s] = -INFINITY;
      l8[s] = 0.f;
#pragma unroll
      for (int u = 0; u < MS; ++u) {
        if (s + 8 * u >= p.n_tile) st_m[s][u] = -INFINITY;
        m8[s] = max_nan(m8[s], st_m[s][u]);
      }
#pragma unroll
      for (int u = 0; u < MS; ++u) l8[s] += st_m[s][u] != -INFINITY ? st_l[s][u] * fast_exp2(st_m[s][u] - m8[s]) : 0.f;
      mx = max_nan(mx, m8[s]);
    }
#pragma unroll
    for (int s = 0; s < 8; ++s) tot += m8[s] != -INFINITY ? l8[s] * fast_exp2(m8[s] - mx) : 0.f;
    sm.lse_s[tid / RCH][tid % RCH] = row_begin + tid < Rs ? mx + log2_of_sum(tot) : INFINITY;
  }
  bool plain = PASS == 1;                     // (wave-uniform)
  for (int r0 = row_begin; r0 < row_end; r0 += RCH, buf ^= 1) {
    wait_vmcnt_lds<0>();                      // this wave's share of the chunk (and its normalisers) has arrived
    if (PASS == 2 && MERGE == 0 && tid < RCH) sm.lse_s[buf][tid] = lse_reg;
    __syncthreads();                          // ... and everyone else's; everyone is done with the chunk before
    if (r0 + RCH < row_end) request_chunk(buf ^ 1, r0 + RCH);
    const unsigned char* Qc = Qs + buf * CHUNKB;
    const float* lse_c = sm.lse_s[MERGE > 0 ? (r0 - row_begin) / RCH : buf];

    auto products = [&](int rb, f32x4 (&z)[TBW]) {
#pragma unroll
      for (int tb = 0; tb < TBW; ++tb) z[tb] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const bf16x8 qop = *(const bf16x8*)(Qc + (rb * 16 + j) * ROWB +
                                            (((ks * 4 + g) ^ lds_row_swizzle<D>(rb * 16 + j)) * 16));
#pragma unroll
        for (int tb = 0; tb < TBW; ++tb)
          z[tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kop[tb][ks], qop, z[tb], 0, 0, 0);
      }
    };
    auto mask_tokens = [&](f32x4 (&z)[TBW]) {
      if (!wave_full) {                         // wave-uniform: only the ragged last wave masks
#pragma unroll
        for (int tb = 0; tb < TBW; ++tb)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (!tok_ok[tb][e]) z[tb][e] = -INFINITY;
      }
    };
    auto reduce = [&](int rb, f32x4 (&z)[TBW]) {
      if (PASS == 1) {
        mask_tokens(z);
        float zv[TBW * 4];                      // the scale is positive: take the max of the raw logits
#pragma unroll
        for (int e = 0; e < TBW * 4; ++e) zv[e] = z[e >> 2][e & 3];
        float mx = rows4_max(max_nan_of(zv));
        mx *= scale_log2;
        const float neg_m = (mx == -INFINITY) ? 0.f : -mx;
        float ps = 0.f;
#pragma unroll
        for (int tb = 0; tb < TBW; ++tb)
#pragma unroll
          for (int e = 0; e < 4; ++e) ps += fast_exp2(fmaf(z[tb][e], scale_log2, neg_m));
        ps = rows4_sum(ps);
        if (g == 0) {
          wm_s[wave][((r0 - row_begin) % RDEF) + rb * 16 + j] = mx;
          wl_s[wave][((r0 - row_begin) % RDEF) + rb * 16 + j] = ps;
        }
      } else {
        const float lse = lse_c[rb * 16 + j];
#pragma unroll
        for (int tb = 0; tb < TBW; ++tb)
#pragma unroll
          for (int e = 0; e < 4; ++e) col[tb][e] += fast_exp2(fmaf(z[tb][e], scale_log2, -lse));
      }
    };
    if (PASS == 2) {
#pragma unroll
      for (int rb = 0; rb < RCH / 16; ++rb) {
        f32x4 z[TBW];
        products(rb, z);
        reduce(rb, z);
      }
    } else {
      // Without a reference: exp2 of the logits as they are, and one transposing sum across the lane groups per 64
      // rows (lane (j, g) ends with row 16g + j of the chunk), 3.4 vector instructions per logit against 6.25 with
      // a maximum per 16 rows (scoring calls, us: 16384 tokens 51.6 -> 48.4, four layers of 32768 tokens 567 -> 512,
      // 4 x 36864 tokens of 64 heads 819 -> 760).  As long as every row's sum over the wave's tokens stays within
      // kPlainMin .. kPlainMax.  From the first chunk on where one does not, the wave takes the maximum as the reference
      // (and goes over that chunk again, if it is far outside): large logits come in whole heads.  Calls over 16384 and
      // 4 x 36864 tokens, us, against the maximum alone: all logits 150 higher 56.4 and 856 (53.5 and 860; trying every
      // chunk both ways 69 and 1088); spread three times as wide 52.1 and 838 (52.1 and 896), five times 54.4 and 885
      // (52.1 and 899).
      static_assert(RCH == 64, "four row blocks, one per lane group");
      bool done = false;
      if (plain) {
        float pair[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          float ps[2];
#pragma unroll
          for (int r2 = 0; r2 < 2; ++r2) {
            f32x4 z[TBW];
            products(2 * h + r2, z);
            mask_tokens(z);
            float t[TBW];
#pragma unroll
            for (int tb = 0; tb < TBW; ++tb)
              t[tb] = (fast_exp2(z[tb][0] * scale_log2) + fast_exp2(z[tb][1] * scale_log2)) +
                      (fast_exp2(z[tb][2] * scale_log2) + fast_exp2(z[tb][3] * scale_log2));
            ps[r2] = t[0];
#pragma unroll
            for (int tb = 1; tb < TBW; ++tb) ps[r2] += t[tb];
          }
          pair[h] = rows_sum_swap16(ps[0], ps[1]);
          __builtin_amdgcn_sched_barrier(0);     // two row blocks at a time: more in flight spills
        }
        const float tot = rows_sum_swap32(pair[0], pair[1]);        // (the comparisons are false for NaN)
        plain = __all((tot >= kPlainMin && tot <= kPlainMax) || !wave_has_tokens);
        done = plain || __all((tot >= kPlainMin * kPlainSlack && tot <= kPlainMax / kPlainSlack) || !wave_has_tokens);
        if (done) {
          const int at = ((r0 - row_begin) % RDEF) + lane;
          wm_s[wave][at] = wave_has_tokens ? 0.f : -INFINITY;
          wl_s[wave][at] = tot;
        }
      }
      if (!done) {
#pragma unroll
        for (int rb = 0; rb < RCH / 16; ++rb) {
          f32x4 z[TBW];
          products(rb, z);
          reduce(rb, z);
        }
      }
    }
    if (PASS == 1 && (((r0 - row_begin + RCH) % RDEF) == 0 || r0 + RCH >= row_end)) {
      // merge the waves' (max, sum) of the rows gathered since the last merge and write them out
      __syncthreads();
      const int base = r0 - ((r0 - row_begin) % RDEF);
      for (int rr = tid; rr < RDEF && base + rr < Rs && base + rr < r0 + RCH; rr += NT) {
        float mm = -INFINITY;
#pragma unroll
        for (int w = 0; w < NW; ++w) mm = max_nan(mm, wm_s[w][rr]);
        float ll = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w)
          ll += (wm_s[w][rr] == -INFINITY) ? 0.f : wl_s[w][rr] * fast_exp2(wm_s[w][rr] - mm);
        const long long at = sattn_part_at(p, tile, bz, hk, base + rr);  // consecutive rows: coalesced
        p.row_m[at] = mm;
        p.row_l[at] = ll;
      }
    }
  }
  if (PASS == 2 && wave_has_tokens) {
    // sum the 16 rows held by the lanes of each group g
#pragma unroll
    for (int tb = 0; tb < TBW; ++tb)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float v = row16_sum(col[tb][e]);
        if (j == 0 && tok_ok[tb][e])
          p.col_part[((long long)bz * p.Hkv * p.n_rsplit + vhk) * p.Nv + n0 + tb * 16 + 4 * g + e] = v;
      }
  }
}

// Launch order of the sweeps' blocks: KV head fastest, then key tile, then row run, then (layer,
// batch element).  Consecutive blocks go to consecutive XCDs, so with 1, 2, 4 or 8 KV heads an XCD
// sees the blocks of one or few heads only and its L2 fetches those heads' query rows instead of all
// of them (every block re-reads the query rows of its head and run); the blocks that sweep the other
// row run over the same 256 keys lie H_kv * n_tile places on -- on the same XCD, where the keys are.
// Grid (H_kv, n_tile, n_rsplit * Bz).
template <int D, int PASS, int MERGE = 0>
__global__ __launch_bounds__(kSaWaves * 64) void sattn_mfma(ScoreParams p) {
  __shared__ SattnSmem<D, PASS, MERGE> sm;
  const int rs = blockIdx.z % p.n_rsplit;
  sattn_mfma_body<D, PASS, MERGE>(p, sm, blockIdx.y, blockIdx.x + p.Hkv * rs, blockIdx.z / p.n_rsplit);
}

// merge the per-tile row statistics: lse2 = m* + log2(sum_t l_t 2^(m_t - m*)).  A block takes 32
// consecutive rows; thread (row, slice s) merges tiles s, s+8, ... (loads issued 8 at a time), the 8
// slices of a row then merge through LDS.  Consecutive threads read consecutive rows of a tile's slab.
__global__ __launch_bounds__(256) void sattn_row_lse(ScoreParams p) {
  __shared__ float sm[8][32], sl[8][32];
  const long long rows = (long long)p.Bz * p.H * p.L;
  const int rl = threadIdx.x & 31, slice = threadIdx.x >> 5;
  const long long row = (long long)blockIdx.x * 32 + rl;
  float mm = -INFINITY, ll = 0.f;
  if (row < rows) {
    for (int t0 = slice; t0 < p.n_tile; t0 += 64) {
      float m[8], l[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int t = t0 + 8 * u;
        m[u] = t < p.n_tile ? p.row_m[t * rows + row] : -INFINITY;
        l[u] = t < p.n_tile ? p.row_l[t * rows + row] : 0.f;
      }
      float mx = mm;
#pragma unroll
      for (int u = 0; u < 8; ++u) mx = max_nan(mx, m[u]);
      if (mx != -INFINITY) {
        ll *= fast_exp2(mm - mx);                 // mm = -inf: ll is 0 and exp2(-inf) = 0
#pragma unroll
        for (int u = 0; u < 8; ++u) ll += (m[u] != -INFINITY) ? l[u] * fast_exp2(m[u] - mx) : 0.f;
        mm = mx;
      }
    }
  }
  sm[slice][rl] = mm;
  sl[slice][rl] = ll;
  __syncthreads();
  if (slice == 0 && row < rows) {
    float mx = -INFINITY;
#pragma unroll
    for (int u = 0; u < 8; ++u) mx = max_nan(mx, sm[u][rl]);
    float tot = 0.f;
#pragma unroll
    for (int u = 0; u < 8; ++u) tot += (sm[u][rl] != -INFINITY) ? sl[u][rl] * fast_exp2(sm[u][rl] - mx) : 0.f;
    p.row_lse[row] = mx + log2_of_sum(tot);
  }
}

// Sum over layers, KV heads and row runs of the column partials of token jj of batch element b, in index
// order, eight loads in flight at a time (a loop of one load and one add per turn would make every partial
// its own trip to memory).
__device__ __forceinline__ float sum_col_partials(const ScoreParams& p, int b, long long jj) {
  const int nvh = p.Hkv * p.n_rsplit;
  float a = 0.f;
  for (int layer = 0; layer < p.n_layers; ++layer)
    for (int hk0 = 0; hk0 < nvh; hk0 += 8) {
      float v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q)
        v[q] = p.col_part[(((long long)layer * p.B + b) * nvh + min(hk0 + q, nvh - 1)) * p.Nv + jj];
#pragma unroll
      for (int q = 0; q < 8; ++q) a += (hk0 + q < nvh) ? v[q] : 0.f;
    }
  return a;
}

// s_attn[b,j] = sum_hk col_part / (H L)  (+ running layer sum)
__global__ __launch_bounds__(256) void sattn_finalize(ScoreParams p) {
  const long long e = (long long)blockIdx.x * 256 + threadIdx.x;
  if (e >= (long long)p.B * p.Nv) return;
  const int b = (int)(e / p.Nv), jj = (int)(e % p.Nv);
  float a = sum_col_partials(p, b, jj);
  a /= (float)p.H * (float)p.L;
  if (p.attn_mass_inout != nullptr) {
    a += p.attn_mass_inout[e];
    p.attn_mass_inout[e] = a;
  }
  p.s_attn[e] = a;
}

// =================================================================================================
// s_temp and s_spa, fp32 crops above 32 tokens: one block per (crop, frame, batch element)
// =================================================================================================
constexpr int kEmbChunk = 64;     // channels per LDS pass
constexpr int kMaxCrop = 64;      // tokens per crop

__global__ __launch_bounds__(256) void emb_scores(ScoreParams p) {
  // E: this frame, previous frame, next frame.  G (the finished Gram matrix) reuses E's storage
  // once the channel sweep is over.
  __shared__ float e_raw[3 * kMaxCrop * (kEmbChunk + 1)];
  float (*E)[kMaxCrop][kEmbChunk + 1] = reinterpret_cast<float (*)[kMaxCrop][kEmbChunk + 1]>(e_raw);
  float (*G)[kMaxCrop + 1] = reinterpret_cast<float (*)[kMaxCrop + 1]>(e_raw);
  __shared__ float tdot[4][kMaxCrop];               // v.prev, |prev|^2, v.next, |next|^2
  __shared__ int tok_s[kMaxCrop];

  const int tid = threadIdx.x;
  const int ncx = (p.gw + p.cw - 1) / p.cw;
  const int cy = blockIdx.x / ncx, cx = blockIdx.x % ncx;
  const int f = blockIdx.y, b = blockIdx.z;
  const int y0 = cy * p.ch, x0 = cx * p.cw;
  const int mh = min(p.ch, p.gh - y0), mw = min(p.cw, p.gw - x0);
  const int M = mh * mw;
  if (tid < M) tok_s[tid] = f * p.P + (y0 + tid / mw) * p.gw + x0 + tid % mw;
  const bool has_prev = f > 0, has_next = f + 1 < p.F;

  const int de = p.emb ? p.emb_dim : p.Hkv * p.D;
  const int n_pairs = M * M;
  constexpr int PPT = kMaxCrop * kMaxCrop / 256;    // pairs per thread, worst case
  float gacc[PPT];
#pragma unroll
  for (int x = 0; x < PPT; ++x) gacc[x] = 0.f;
  float tacc = 0.f;                                  // threads [0,4*64): quantity tid/64 of token tid%64
  __syncthreads();

  constexpr int kVec = Elem<float>::kPerVec, VPC = kEmbChunk / kVec;  // vectors per chunk row
  for (int c0 = 0; c0 < de; c0 += kEmbChunk) {
    // ---- stage chunk [c0, c0+64) of the 3*M vectors ----
    for (int e = tid; e < 3 * M * VPC; e += 256) {
      const int which = e / (M * VPC), rem = e % (M * VPC);
      const int t = rem / VPC, vec = rem % VPC;
      const int c = c0 + vec * kVec;
      float vals[kVec];
#pragma unroll
      for (int u = 0; u < kVec; ++u) vals[u] = 0.f;
      const bool present = (which == 0) || (which == 1 && has_prev) || (which == 2 && has_next);
      if (present && c < de) {
        const long long tokn = tok_s[t] + (which == 1 ? -p.P : (which == 2 ? p.P : 0));
        const float* src;
        if (p.emb) {
          src = (const float*)p.emb + (long long)b * p.emb_stride_b + tokn * p.emb_stride_tok + c;
        } else {
          const int hk = c / p.D, cc = c % p.D;
          src = (const float*)p.k_cache + (long long)b * p.sb + (long long)hk * p.sh +
                (p.vis_off + tokn) * p.sn + cc;
        }
        const u32x4 v4 = *(const u32x4*)src;
        Elem<float>::unpack(v4, vals);
      }
#pragma unroll
      for (int u = 0; u < kVec; ++u) E[which][t][vec * kVec + u] = vals[u];
    }
    __syncthreads();
    // ---- Gram of the crop ----
#pragma unroll
    for (int x = 0; x < PPT; ++x) {
      const int pr = tid + 256 * x;
      if (pr < n_pairs) {
        const int a = pr / M, c2 = pr % M;
        float s = 0.f;
#pragma unroll 8
        for (int c = 0; c < kEmbChunk; ++c) s = fmaf(E[0][a][c], E[0][c2][c], s);
        gacc[x] += s;
      }
    }
    // ---- temporal dot products and neighbour norms ----
    {
      const int qn = tid >> 6, t = tid & 63;
      if (t < M) {
        const int other = (qn < 2) ? 1 : 2;
        const float* ea = (qn & 1) ? E[other][t] : E[0][t];
        const float* eb = E[other][t];
        float s = 0.f;
#pragma unroll 8
        for (int c = 0; c < kEmbChunk; ++c) s = fmaf(ea[c], eb[c], s);
        tacc += s;
      }
    }
    __syncthreads();
  }

#pragma unroll
  for (int x = 0; x < PPT; ++x) {
    const int pr = tid + 256 * x;
    if (pr < n_pairs) G[pr / M][pr % M] = gacc[x];
  }
  tdot[tid >> 6][tid & 63] = tacc;
  __syncthreads();

  if (tid < M) {
    const int a = tid;
    const float na = G[a][a];
    // spatial: population variance of the cosine row
    float mu = 0.f;
    for (int c2 = 0; c2 < M; ++c2) {
      const float nb = G[c2][c2];
      const float cs = (na > 0.f && nb > 0.f) ? G[a][c2] / (sqrtf(na) * sqrtf(nb)) : 0.f;
      mu += cs;
    }
    mu /= (float)M;
    float var = 0.f;
    for (int c2 = 0; c2 < M; ++c2) {
      const float nb = G[c2][c2];
      const float cs = (na > 0.f && nb > 0.f) ? G[a][c2] / (sqrtf(na) * sqrtf(nb)) : 0.f;
      var = fmaf(cs - mu, cs - mu, var);
    }
    const long long o = (long long)b * p.Nv + tok_s[a];
    p.s_spa[o] = var / (float)M;
    // temporal
    float sum = 0.f;
    int cnt = 0;
    if (has_prev) {
      const float nb = tdot[1][a];
      sum += (na > 0.f && nb > 0.f) ? tdot[0][a] / (sqrtf(na) * sqrtf(nb)) : 0.f;
      ++cnt;
    }
    if (has_next) {
      const float nb = tdot[3][a];
      sum += (na > 0.f && nb > 0.f) ? tdot[2][a] / (sqrtf(na) * sqrtf(nb)) : 0.f;
      ++cnt;
    }
    p.s_temp[o] = 1.f - (cnt ? sum / (float)cnt : 0.f);
  }
}

// =================================================================================================
// s_temp and s_spa on MFMA, bf16 crops above 32 tokens: one block per (crop, frame, batch element), RBC*16 >= crop
// size.
// The crop's Gram matrix E E^T and the temporal products (E_f E_{f-1}^T, E_{f-1} E_{f-1}^T and the
// same for f+1, of which only the diagonals are used) are 16x16 output blocks of one and the same
// operand: a lane's A operand for row block rb -- token rb*16 + lane%16, 8 consecutive channels --
// is also the B operand for that block of columns, and it is read straight from global memory
// (16 bytes per lane; the 4 lane groups of a token cover 64 contiguous bytes).  The 16x16 blocks
// are dealt to the 4 waves, each sweeping all channels for its blocks, so nothing is reduced
// across waves; the finished Gram goes to LDS and one thread per token finishes Eq. 4 and Eq. 6.
// =================================================================================================
template <int RBC>
__global__ __launch_bounds__(256) void emb_scores_mfma(ScoreParams p) {
  constexpr int MP = RBC * 16;
  constexpr int N_GRAM = RBC * (RBC + 1) / 2;      // upper-triangle blocks
  constexpr int N_ITEMS = N_GRAM + 4 * RBC;        // + (prev dot, prev norm, next dot, next norm) x RBC
  __shared__ float G[MP][MP + 1];
  __shared__ float tdot[4][MP];                     // v.prev, |prev|^2, v.next, |next|^2
  __shared__ int tok_s[MP];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 15, g = lane >> 4;
  const int ncx = (p.gw + p.cw - 1) / p.cw;
  const int cy = blockIdx.x / ncx, cx = blockIdx.x % ncx;
  const int f = blockIdx.y, b = blockIdx.z;
  const int y0 = cy * p.ch, x0 = cx * p.cw;
  const int mh = min(p.ch, p.gh - y0), mw = min(p.cw, p.gw - x0);
  const int M = mh * mw;
  if (tid < MP) {
    const int t = tid < M ? tid : M - 1;            // padding slots repeat the last token
    tok_s[tid] = f * p.P + (y0 + t / mw) * p.gw + x0 + t % mw;
  }
  const bool has_prev = f > 0, has_next = f + 1 < p.F;
  const int de = p.emb ? p.emb_dim : p.Hkv * p.D;
  const int n_ks = (de + 31) / 32;
  __syncthreads();

  // operand of frame offset `df` (-1, 0, +1), row block rbk, channel step ks
  auto operand = [&](int df, int rbk, int ks) -> bf16x8 {
    const int c = ks * 32 + g * 8;
    if (c >= de) return (bf16x8){0, 0, 0, 0, 0, 0, 0, 0};
    const long long tokn = tok_s[rbk * 16 + j] + (long long)df * p.P;
    const uint16_t* src;
    if (p.emb) {
      src = (const uint16_t*)p.emb + (long long)b * p.emb_stride_b + tokn * p.emb_stride_tok + c;
    } else {
      const int hk = c / p.D, cc = c % p.D;
      src = (const uint16_t*)p.k_cache + (long long)b * p.sb + (long long)hk * p.sh +
            (p.vis_off + tokn) * p.sn + cc;
    }
    return *(const bf16x8*)src;
  };

  for (int item = wave; item < N_ITEMS; item += 4) {          // wave-uniform
    int da, db_, ra, rbk;                                      // frame offsets and row blocks of A and B
    int kind = -1;                                             // -1 Gram, 0..3 temporal quantity
    if (item < N_GRAM) {
      int bi = 0, rem = item;
      while (rem >= RBC - bi) { rem -= RBC - bi; ++bi; }
      ra = bi; rbk = bi + rem; da = 0; db_ = 0;
    } else {
      const int t = item - N_GRAM;
      kind = t / RBC;
      ra = rbk = t % RBC;
      const int dn = kind < 2 ? -1 : 1;
      if ((dn < 0 && !has_prev) || (dn > 0 && !has_next)) continue;
      da = (kind & 1) ? dn : 0;                                // norm: neighbour with itself
      db_ = dn;
    }
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    const bool same = (da == db_) && (ra == rbk);              // diagonal block: one operand serves both
    for (int ks0 = 0; ks0 < n_ks; ks0 += 8) {                  // 8 channel steps of loads in flight
      bf16x8 a[8], bb[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) a[u] = operand(da, ra, ks0 + u);
      if (same) {
#pragma unroll
        for (int u = 0; u < 8; ++u) bb[u] = a[u];
      } else {
#pragma unroll
        for (int u = 0; u < 8; ++u) bb[u] = operand(db_, rbk, ks0 + u);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u], bb[u], acc, 0, 0, 0);
    }
    // D[i][j']: this lane holds column j' = j, rows i = 4g..4g+3
    if (kind < 0) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        G[ra * 16 + 4 * g + e][rbk * 16 + j] = acc[e];
        G[rbk * 16 + j][ra * 16 + 4 * g + e] = acc[e];
      }
    } else if ((j >> 2) == g) {
      tdot[kind][ra * 16 + j] = acc[j & 3];
    }
  }
  __syncthreads();

  if (tid < M) {
    const int a = tid;
    const float na = G[a][a];
    float mu = 0.f;
    for (int c2 = 0; c2 < M; ++c2) {
      const float nb = G[c2][c2];
      mu += (na > 0.f && nb > 0.f) ? G[a][c2] / (sqrtf(na) * sqrtf(nb)) : 0.f;
    }
    mu /= (float)M;
    float var = 0.f;
    for (int c2 = 0; c2 < M; ++c2) {
      const float nb = G[c2][c2];
      const float cs = (na > 0.f && nb > 0.f) ? G[a][c2] / (sqrtf(na) * sqrtf(nb)) : 0.f;
      var = fmaf(cs - mu, cs - mu, var);
    }
    const long long o = (long long)b * p.Nv + tok_s[a];
    p.s_spa[o] = var / (float)M;
    float sum = 0.f;
    int cnt = 0;
    if (has_prev) {
      const float nb = tdot[1][a];
      sum += (na > 0.f && nb > 0.f) ? tdot[0][a] / (sqrtf(na) * sqrtf(nb)) : 0.f;
      ++cnt;
    }
    if (has_next) {
      const float nb = tdot[3][a];
      sum += (na > 0.f && nb > 0.f) ? tdot[2][a] / (sqrtf(na) * sqrtf(nb)) : 0.f;
      ++cnt;
    }
    p.s_temp[o] = 1.f - (cnt ? sum / (float)cnt : 0.f);
  }
}

// =================================================================================================
// s_temp and s_spa on MFMA, crops of at most 32 tokens: frame runs.
// A block of eight waves (fp32: four or eight) owns ONE crop position over a run of consecutive frames, so a frame's crop
// serves as "this frame" for its Gram matrix (Eq. 5-6; its diagonal holds the norms) and as "the
// neighbour" of the frame before and after it (Eq. 3-4) -- against four fetches per crop when every
// (crop, frame) is a block of its own.  The wave holds 16 * U lanes' worth of 16-byte pieces of all 32
// rows (U per lane and row block); the waves' partial Gram and dot blocks are summed through LDS.
// The operands travel HBM -> LDS by direct transfers, a lane fetching 16 bytes of a 64 * U-byte row
// segment next to its neighbour's (an MFMA operand lane holds ITS OWN row, so fetching operands
// straight into registers makes neighbouring lanes read rows far apart, and the address unit then
// spends a clock per lane instead of a clock per four); the wave reads them back in operand layout
// from its own strip, whose rows are XOR-swizzled against bank conflicts.  The strip then
// carries the wave's partial Gram blocks to the reduction, so the next frame's transfer is requested
// once the reduction has read them and lands under the rest of the frame's arithmetic.
//
// One pass over a block's channels (512 in bf16 with U = 2; in fp32, U = 4, 256 of four waves, 512 of eight) keeps the frame
// before in registers.  WIDE embeddings take several passes per frame.  Two of them in bf16 (kHold) keep it there too,
// 32 registers, and have both passes in flight at once, each in a strip of its own: what bounded them was that the
// frame before was fetched again behind this frame's, from beyond the L2 (two strips alone gained nothing).  The terms
// alone | whole scoring calls, us: 4 x 36864 tokens of 1024 channels 112 -> 75 | 735 -> 712, 4 x 16384 of 1024 83 -> 47 |
// 222 -> 197, 4 x 36864 x 14 heads, of 768 90 -> 65 | 157 -> 122, 3 x 20520 of 1024, 16 text rows 51 -> 38 | 112 -> 93.
// More passes, and fp32, fetch it again: two fetches per crop and frame (kRefetch; kRefetch2 through two strips).
// fp32 takes the same frame with four 16x16x4 products per 16-byte operand (3136 tokens, 128 channels 47 -> 37;
// 12288 tokens, 512 channels 178 -> 143; 11040 tokens, 1024 channels 624 -> 562), by blocks of four waves, as the fp32
// sweeps', beside pass 1 (sattn_f32_pass1_with_emb), and of four or eight in a launch of their own: wide_f32_rides and
// wide_f32_plan say which.  The vector-ALU kernel (a block per crop and frame, two LDS reads per multiply-add) is left for
// fp32 crops above 32 tokens.
// =================================================================================================
// 16 bytes of zeros in device memory: what a transfer lane fetches for channels beyond the last
__device__ __align__(16) const unsigned char g_zero_piece[16] = {0};

// NB: strips of a wave
template <int U, int NW, int NB>
struct EmbRunSmem {
  static constexpr int MP = 32;
  // operands in (32 rows x 64 U B), then Gram partials out (3 x 64 x 16 B, from four waves two sets of them)
  __align__(16) unsigned char strip[NB][NW][MP * 64 * U];
  float redd[8][2][16];                             // diagonals of the (this frame) x (frame before) blocks
  float G[MP][MP + 1];
  float dotv[MP];
  float scale[MP];                                  // of the rows' norms, see scale_of
  int tok_s[MP];
};

// acc += A B^T over the channels of two 16-byte operands: 8 bf16 channels or 4 fp32 channels per lane group
template <bool F32>
__device__ __forceinline__ f32x4 emb_mma(const u32x4& a, const u32x4& b, f32x4 acc) {
  if constexpr (F32) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[e]), __uint_as_float(b[e]), acc, 0, 0, 0);
    return acc;
  } else {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc,
                                                   0, 0, 0);
  }
}

// One crop position `pos` of batch element b over the frames f0 .. f0 + p.emb_run - 1 (cut at the
// video's end), by the 64 * NW threads of a block; every thread must call it (block-wide barriers).
// KIND: channels of one pass, of all the block's waves or of few; of several passes, fetched again for the next frame, through
// one strip or two; of two passes, held.
enum EmbKind { kOnePass, kFew, kRefetch, kRefetch2, kHold };
constexpr int emb_strips(int kind) { return kind >= kRefetch2 ? 2 : 1; }
template <bool F32, int U, int NW, int KIND>
__device__ __forceinline__ void emb_run32_body(const ScoreParams& p, EmbRunSmem<U, NW, emb_strips(KIND)>& sm, const int tid,
                                               const int pos, const int f0, const int b) {
  constexpr bool WIDE = KIND > kFew, TWO = KIND >= kRefetch2, HOLD = KIND == kHold;
  constexpr int MP = EmbRunSmem<U, NW, emb_strips(KIND)>::MP;
  static_assert(!TWO || NW == 8, "one set of partial sums");
  constexpr int TPT = NW * 64 / MP, CPT = MP / TPT; // threads per token, cosines per thread
  static_assert((NW == 8 && TPT == 16) || (NW == 4 && TPT == 8), "a token's threads are half or all of a 16-lane row");
  constexpr int EB = F32 ? 4 : 2;                   // bytes per channel
  constexpr int EPP = 16 / EB;                      // channels per 16-byte piece
  constexpr int PPR = 4 * U;                        // pieces of a row in a wave's strip
  constexpr int RPT = 64 / PPR;                     // rows per transfer
  constexpr int NT = MP / RPT;                      // transfers per frame and pass
  constexpr int CW = PPR * EPP, CB = NW * CW;       // channels per pass: of a wave, of the block
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 15, g = lane >> 4;
  const int ncx = (p.gw + p.cw - 1) / p.cw;
  const int cy = pos / ncx, cx = pos % ncx;
  const int y0 = cy * p.ch, x0 = cx * p.cw;
  const int mh = min(p.ch, p.gh - y0), mw = min(p.cw, p.gw - x0);
  const int M = mh * mw;
  if (tid < MP) {
    const int t = tid < M ? tid : M - 1;            // padding slots repeat the last token
    sm.tok_s[tid] = (y0 + t / mw) * p.gw + x0 + t % mw;   // token within its frame
  }
  const int f_end = min(f0 + p.emb_run, p.F);       // the run: frames f0 .. f_end - 1
  const int lo = max(f0 - 1, 0), hi = min(f_end, p.F - 1);   // frames fetched: the run and its neighbours
  const int de = p.emb ? p.emb_dim : p.Hkv * p.D;
  const bool keys_as_emb = p.emb == nullptr;
  const int dsh = p.D == 128 ? 7 : 6;
  __syncthreads();

  // Transfer i of a pass brings rows RPT*i .. of the crop: lane l fetches, for strip position
  // l % PPR of its row, the 16-byte piece (l % PPR) ^ (row & (PPR - 1)) of the wave's segment.
  // With keys as the embedding, channel c is element c % D of KV head c / D (D is a power of two).
  // Pieces beyond the last channel are fetched from 16 bytes of zeros, so the operands need no masking.
  const char* const base = keys_as_emb
      ? (const char*)p.k_cache + ((long long)b * p.sb + (long long)p.vis_off * p.sn) * EB
      : (const char*)p.emb + (long long)b * p.emb_stride_b * EB;
  const long long tok_step = (keys_as_emb ? p.sn : p.emb_stride_tok) * EB;
  const long long frame_step = (long long)p.P * tok_step;
  auto channel = [&](int i, int pass) {             // first channel of this lane's piece
    return pass * CB + wave * CW + ((lane % PPR) ^ ((i * RPT + lane / PPR) & (PPR - 1))) * EPP;
  };
  auto channel_at = [&](int c) -> long long {
    return (keys_as_emb ? (long long)(c >> dsh) * p.sh + (c & (p.D - 1)) : (long long)c) * EB;
  };
  // single pass: the piece is the same in every frame, so its address is kept and moved on frame by frame; several
  // passes: worked out for each transfer (registers are what the riding blocks are short of)
  const char* src[WIDE ? 1 : NT];
  long long src_step[WIDE ? 1 : NT];
  if constexpr (!WIDE) {
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const int c = channel(i, 0);
      src[i] = base + ((long long)lo * p.P + sm.tok_s[i * RPT + lane / PPR]) * tok_step + channel_at(c);
      src_step[i] = frame_step;
      if (c >= de) {
        src[i] = (const char*)g_zero_piece;
        src_step[i] = 0;
      }
    }
  }
  unsigned char* strip = &sm.strip[0][wave][0];     // (two: the one that is read)
  unsigned strip_addr = (unsigned)(uintptr_t)strip;
  // Few channels: waves whose own lie beyond the last one fetch and multiply nothing (two KV heads of 64 channels: six waves
  // of eight, which took instructions and products' time from the sweep beside them), and nothing of theirs is summed.
  // us a call from a graph, with them -> without: bf16, 4096 tokens x 14 heads 18.6 -> 18.0, 23562 x 14 x 2 in four layers 59.1
  // -> 53.5; fp32, 3136 x 14, 64 rows 20.3 -> 19.2 (the products with the frame before the first left out as well); 1837 random calls
  // of few fp32 channels 0.950 of the time, 1953 of bf16 0.860 (with other steps).  A kind of its own: with the question in the
  // kernel of all waves, and the first products left out there, calls of 256 fp32 channels took up to 1.2 of the time beside the
  // sweep, though not alone: 29475 tokens x 4 heads, 23 text rows 65 -> 78, 31680 x 4, 55 rows 75 -> 84.5, 3120 x 2 x 3 in two
  // layers 28 -> 30; bf16, 29232 x 4 heads x 128, 122 rows 42.0 -> 43.5.
  const int n_active = KIND == kFew ? min(NW, (de + CW - 1) / CW) : NW;
  const bool active = KIND != kFew || wave < n_active;
  auto request = [&](int frame, int pass) {         // single pass: frames lo, lo + 1, ... in turn
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      if constexpr (!WIDE) {
        dma16(src[i], strip_addr + i * 1024);
        src[i] += src_step[i];
      } else {
        const int c = channel(i, pass);
        const char* at = base + ((long long)frame * p.P + sm.tok_s[i * RPT + lane / PPR]) * tok_step + channel_at(c);
        dma16(c < de ? at : (const char*)g_zero_piece, strip_addr + i * 1024);
      }
    }
  };
  // operand (row block rbk, step u of the wave's segment): lane (j, g) holds piece 4u + g of row 16 rbk + j
  auto operand = [&](int rbk, int u) -> u32x4 {
    return *(const u32x4*)(strip + (rbk * 16 + j) * (64 * U) + (((4 * u + g) ^ (j & (PPR - 1))) * 16));
  };
  // Squared norm -> what cosine() takes of a row: bf16 its reciprocal norm, fp32 its norm; -1 for a row without a
  // positive norm (of zeros, or with a NaN), whose cosines are 0.  bf16: by the hardware's reciprocal square root
  // (1 ulp), which ignores denormals: tiny arguments are scaled by 2^64 first, the result by 2^32.  (The riding blocks
  // compete with the sweep for vector-instruction issue and nothing else, so what the crop's closing arithmetic costs in
  // instructions is what the embedding terms cost the launch.)  fp32: two divisions; with reciprocals s_temp was up to
  // 8 % further from 64 bits, and the call no faster.
  auto scale_of = [](float x) -> float {
    if constexpr (F32) return x > 0.f ? sqrtf(x) : -1.f;
    const bool tiny = x < 0x1p-60f;
    const float r = __builtin_amdgcn_rsqf(tiny ? x * 0x1p64f : x);
    return x > 0.f ? (tiny ? r * 0x1p32f : r) : -1.f;
  };
  // (from left to right: the product of two norms, or of their reciprocals, can exceed fp32's range; the dot product is
  // what is replaced, so that the last product still fuses with the sum that it goes into)
  auto cosine = [](float dot, float sa, float sb) {
    const float d = fminf(sa, sb) < 0.f ? 0.f : dot;
    if constexpr (F32) return d / sa / sb;
    else return d * sa * sb;
  };
  const float inv_M = 1.f / (float)M;

  // state of the tokens' temporal term, kept by the first of the token's threads (token a = tid / TPT):
  // the scale of its norm in the last two frames, and their dot product
  float scale_1 = 0.f, scale_2 = 0.f, dot1 = 0.f;
  const int a = tid / TPT, c0 = (tid % TPT) * CPT;
  auto token_sum = [](float v) { return NW == 8 ? row16_sum(v) : row8_sum(v); };
  const long long out_base = (long long)b * p.Nv + sm.tok_s[a];

  constexpr int HP = HOLD ? 2 : 1;                  // passes that are held
  const int n_pass = HOLD ? HP : WIDE ? (de + CB - 1) / CB : 1;
  // Several passes of four waves: odd and even passes are two sets of partial sums, which stand for waves 4 to 7 and 0 to 3
  // of eight: a frame's Gram and dot products are the same chains of channels, summed in the same order, whichever
  // kernel takes them.  (One chain over both put the fused score of 512 fp32 channels 1.3 times, of 1024 1.5 times as far
  // from 64 bits.)
  constexpr int SETS = WIDE ? 8 / NW : 1;
  constexpr int kSetBytes = 3 * 64 * 16;
  static_assert(SETS * kSetBytes <= (int)sizeof(sm.strip[0][0]) && SETS * NW <= 8, "a strip takes its wave's partial sums");
  constexpr int UP = WIDE ? 1 : U;
  u32x4 prev[2][UP];                                // single pass: the operands of the frame before
#pragma unroll
  for (int rbk = 0; rbk < 2; ++rbk)
#pragma unroll
    for (int u = 0; u < UP; ++u) prev[rbk][u] = (u32x4){0u, 0u, 0u, 0u};
  u32x4 held[HP][2][U];
#pragma unroll
  for (int h = 0; h < HP; ++h)
#pragma unroll
    for (int rbk = 0; rbk < 2; ++rbk)
#pragma unroll
      for (int u = 0; u < U; ++u) held[h][rbk][u] = (u32x4){0u, 0u, 0u, 0u};
  // Two strips: the transfers of a run in the order in which they are wanted, into one and the other in turn, so that one
  // travels while the other is multiplied and while a frame is reduced.
  int t_fr = lo, t_pass = 0, in_flight = 0;
  bool t_before = false;
  unsigned put = 0, take = 0;
  auto issue = [&]() {
    if (t_fr > hi) return;
    strip_addr = (unsigned)(uintptr_t)&sm.strip[put][wave][0];
    request(t_before ? t_fr - 1 : t_fr, t_pass);
    put ^= 1;
    ++in_flight;
    t_before = !HOLD && !t_before && t_fr > lo;
    if (!t_before && ++t_pass == n_pass) {
      t_pass = 0;
      ++t_fr;
    }
  };
  auto arrive = [&]() {                             // the oldest transfer in flight is in its strip
    if (in_flight > 1) wait_vmcnt<NT>();
    else wait_vmcnt<0>();
    --in_flight;
    strip = &sm.strip[take][wave][0];
    take ^= 1;
  };
  if constexpr (TWO) {
    issue();
    issue();
  } else if (active) {
    request(lo, 0);
  }
  for (int fr = lo; fr <= hi; ++fr) {
    f32x4 dot[SETS][2];
    // D[i][j']: a lane holds column j' = j, rows i = 4g..4g+3.  Gram blocks (0,0) (0,1) (1,1); a neighbour frame
    // beyond the run is here for its norms and dot products: the diagonal blocks suffice.
    const bool own_frame = fr >= f0 && fr < f_end;  // (uniform)
    if constexpr (!WIDE) if (active) {
      u32x4 cur[2][U];
      wait_vmcnt<0>();                              // the frame is in this wave's strip
#pragma unroll
      for (int rbk = 0; rbk < 2; ++rbk)
#pragma unroll
        for (int u = 0; u < U; ++u) cur[rbk][u] = operand(rbk, u);
      // the strip's operands are in registers (a wave's LDS operations complete in order), so it can take the Gram
      // partials at once, one block at a time: few accumulators live beside the two frames' operands
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        if (i == 1 && !own_frame) continue;
        f32x4 gram = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < U; ++u) gram = emb_mma<F32>(cur[i >> 1][u], cur[(i + 1) >> 1][u], gram);
        *(f32x4*)(strip + (i * 64 + lane) * 16) = gram;
      }
#pragma unroll
      for (int rbk = 0; rbk < 2; ++rbk) dot[0][rbk] = (f32x4){0.f, 0.f, 0.f, 0.f};
      if (!F32 || KIND != kFew || fr > lo)          // (32 fp32 products of 32 clocks)
#pragma unroll
        for (int rbk = 0; rbk < 2; ++rbk)
#pragma unroll
          for (int u = 0; u < U; ++u) dot[0][rbk] = emb_mma<F32>(cur[rbk][u], prev[rbk][u % UP], dot[0][rbk]);
#pragma unroll
      for (int rbk = 0; rbk < 2; ++rbk)
#pragma unroll
        for (int u = 0; u < U; ++u) prev[rbk][u % UP] = cur[rbk][u];
    }
    if constexpr (WIDE) {
      f32x4 gram[SETS][3];
#pragma unroll
      for (int s = 0; s < SETS; ++s) {
#pragma unroll
        for (int i = 0; i < 3; ++i) gram[s][i] = (f32x4){0.f, 0.f, 0.f, 0.f};
        dot[s][0] = dot[s][1] = (f32x4){0.f, 0.f, 0.f, 0.f};
      }
      const bool has_before = fr > lo;
      auto take_pass = [&](int pass, f32x4 (&gram)[3], f32x4 (&dot)[2]) {
        u32x4 cur[2][U];
        if constexpr (TWO) arrive();
        else wait_vmcnt<0>();
#pragma unroll
        for (int rbk = 0; rbk < 2; ++rbk)
#pragma unroll
          for (int u = 0; u < U; ++u) cur[rbk][u] = operand(rbk, u);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // read before the next transfer may overwrite them
        if constexpr (TWO) {
          if (has_before || pass + 1 < n_pass) issue();      // (the frame's last strip takes the partial sums first)
        } else {
          if (has_before) request(fr - 1, pass);
          else if (pass + 1 < n_pass) request(fr, pass + 1);
        }
#pragma unroll
        for (int i = 0; i < 3; ++i)
          if (i != 1 || own_frame)
#pragma unroll
            for (int u = 0; u < U; ++u) gram[i] = emb_mma<F32>(cur[i >> 1][u], cur[(i + 1) >> 1][u], gram[i]);
        if (has_before) {
          if constexpr (TWO) arrive();
          else wait_vmcnt<0>();
#pragma unroll
          for (int rbk = 0; rbk < 2; ++rbk) {
            u32x4 before[U];
#pragma unroll
            for (int u = 0; u < U; ++u) before[u] = operand(rbk, u);
#pragma unroll
            for (int u = 0; u < U; ++u) dot[rbk] = emb_mma<F32>(cur[rbk][u], before[u], dot[rbk]);
          }
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          if (pass + 1 < n_pass) {
            if constexpr (TWO) issue();
            else request(fr, pass + 1);
          }
        }
      };
      if constexpr (HOLD) {
#pragma unroll
        for (int h = 0; h < HP; ++h) {
          u32x4 cur[2][U];
          arrive();
#pragma unroll
          for (int rbk = 0; rbk < 2; ++rbk)
#pragma unroll
            for (int u = 0; u < U; ++u) cur[rbk][u] = operand(rbk, u);
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          if (h + 1 < HP) issue();
#pragma unroll
          for (int i = 0; i < 3; ++i)
            if (i != 1 || own_frame)
#pragma unroll
              for (int u = 0; u < U; ++u) gram[0][i] = emb_mma<F32>(cur[i >> 1][u], cur[(i + 1) >> 1][u], gram[0][i]);
#pragma unroll
          for (int rbk = 0; rbk < 2; ++rbk)
#pragma unroll
            for (int u = 0; u < U; ++u) {
              dot[0][rbk] = emb_mma<F32>(cur[rbk][u], held[h][rbk][u], dot[0][rbk]);
              held[h][rbk][u] = cur[rbk][u];
            }
        }
      } else {
        for (int pass = 0; pass < n_pass; pass += SETS) {
          take_pass(pass, gram[0], dot[0]);
          if (SETS == 2 && pass + 1 < n_pass) take_pass(pass + 1, gram[SETS - 1], dot[SETS - 1]);
        }
      }
#pragma unroll
      for (int s = 0; s < SETS; ++s)
#pragma unroll
        for (int i = 0; i < 3; ++i)
          if (i != 1 || own_frame) *(f32x4*)(strip + s * kSetBytes + (i * 64 + lane) * 16) = gram[s][i];
    }
    // of a dot block only the diagonal (token with itself) is needed: lane (j, g = j/4), element j%4
    if (active && (j >> 2) == g) {
#pragma unroll
      for (int s = 0; s < SETS; ++s)
#pragma unroll
        for (int rbk = 0; rbk < 2; ++rbk) {
          float d = dot[s][rbk][0];
#pragma unroll
          for (int e = 1; e < 4; ++e)
            if ((j & 3) == e) d = dot[s][rbk][e];
          sm.redd[s * NW + wave][rbk][j] = d;
        }
    }
    __syncthreads();
    // sum the waves' channel slices in the order of their channels: waves 0..2 one Gram block each (the diagonal
    // blocks also give the scales of the rows' norms), wave 3 the diagonals of the dot blocks
    if (wave < 3 && (own_frame || wave != 1)) {
      const int blk = wave;
      const unsigned used = TWO ? take ^ 1 : 0;  // the strips that took the partial sums
      f32x4 v = *(const f32x4*)(&sm.strip[used][0][0] + (blk * 64 + lane) * 16);
      if constexpr (KIND != kFew) {                 // (all reads in flight)
#pragma unroll
        for (int w = 1; w < SETS * NW; ++w)
          v += *(const f32x4*)(&sm.strip[used][w % NW][0] + (w / NW) * kSetBytes + (blk * 64 + lane) * 16);
      } else {
        for (int w = 1; w < n_active; ++w) v += *(const f32x4*)(&sm.strip[used][w][0] + (blk * 64 + lane) * 16);
      }
      const int ra = blk == 2 ? 1 : 0, rbk = blk == 0 ? 0 : 1;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        sm.G[ra * 16 + 4 * g + e][rbk * 16 + j] = v[e];
        sm.G[rbk * 16 + j][ra * 16 + 4 * g + e] = v[e];
      }
      if (blk != 1 && (j >> 2) == g) {              // D[j][j]: lane (j, g = j/4), element j%4
        float d = v[0];
#pragma unroll
        for (int e = 1; e < 4; ++e)
          if ((j & 3) == e) d = v[e];
        sm.scale[ra * 16 + j] = scale_of(d);
      }
    } else if (wave == 3 && lane < MP) {
      float d = sm.redd[0][lane >> 4][lane & 15];
      if constexpr (KIND != kFew) {
#pragma unroll
        for (int w = 1; w < SETS * NW; ++w) d += sm.redd[w][lane >> 4][lane & 15];
      } else {
        for (int w = 1; w < n_active; ++w) d += sm.redd[w][lane >> 4][lane & 15];
      }
      sm.dotv[lane] = d;
    }
    __syncthreads();
    if constexpr (TWO) issue();                 // the strips are free again: the next frame travels meanwhile
    else if (fr < hi && active) request(fr + 1, 0);

    // cosines of token a against tokens c0 .. c0 + CPT - 1 (its TPT threads cover the crop; padding rows hold
    // finite values and are masked); Eq. 5-6: their variance -- for the run's own frames only
    const float sa = sm.scale[a];
    float var = 0.f;
    if (own_frame) {
      float cs[CPT];
#pragma unroll
      for (int i = 0; i < CPT; ++i) cs[i] = c0 + i < M ? cosine(sm.G[a][c0 + i], sa, sm.scale[c0 + i]) : 0.f;
      // (in pairs, then over the threads: the same tree of sums for two and for four cosines a thread)
      float mu = cs[0] + cs[1];
      if constexpr (CPT == 4) mu += cs[2] + cs[3];
      mu = token_sum(mu) * inv_M;
#pragma unroll
      for (int i = 0; i < CPT; ++i) cs[i] = c0 + i < M ? cs[i] - mu : 0.f;
      float sq = fmaf(cs[0], cs[0], cs[1] * cs[1]);
      if constexpr (CPT == 4) sq += fmaf(cs[2], cs[2], cs[3] * cs[3]);
      var = token_sum(sq) * inv_M;
    }
    if (tid % TPT == 0 && a < M) {
      const float dcur = sm.dotv[a];                // <this frame, frame before>
      if (own_frame) p.s_spa[out_base + (long long)fr * p.P] = var;
      // Eq. 3-4 of the frame before, whose two neighbours are known now
      if (fr > lo && fr - 1 >= f0) {
        const float next = cosine(dcur, scale_1, sa), before = cosine(dot1, scale_1, scale_2);
        p.s_temp[out_base + (long long)(fr - 1) * p.P] = 1.f - (fr - 1 > 0 ? 0.5f * (next + before) : next);
      }
      scale_2 = scale_1;
      scale_1 = sa;
      dot1 = dcur;
    }
  }
  // a run that reaches the video's last frame: that frame has no successor
  if (tid % TPT == 0 && a < M && hi < f_end)
    p.s_temp[out_base + (long long)hi * p.P] = 1.f - (hi > 0 ? cosine(dot1, scale_1, scale_2) : 0.f);
}

// block number -> (crop position, run of frames, batch element), positions fastest
template <bool F32, int U, int NW, int KIND>
__device__ __forceinline__ void emb_run32_block(const ScoreParams& p, EmbRunSmem<U, NW, emb_strips(KIND)>& sm,
                                                const unsigned blk) {
  const unsigned ncf = (unsigned)(((p.gh + p.ch - 1) / p.ch) * ((p.gw + p.cw - 1) / p.cw));   // crops per frame
  const unsigned n_runs = (unsigned)((p.F + p.emb_run - 1) / p.emb_run);
  const unsigned rest = blk / ncf, pos = blk - rest * ncf;
  const unsigned bb = rest / n_runs, run = rest - bb * n_runs;
  emb_run32_body<F32, U, NW, KIND>(p, sm, threadIdx.x, (int)pos, (int)run * p.emb_run, (int)bb);
}

// (four waves: three blocks on a compute unit; with registers for two, 4 x 72 frames of 768 channels took 256 us, not 187)
template <bool F32, int NW, int KIND>
__global__ __launch_bounds__(64 * NW, NW == 4 ? 3 : 2) void emb_scores_run32(ScoreParams p) {
  constexpr int U = F32 ? 4 : 2;
  __shared__ EmbRunSmem<U, NW, emb_strips(KIND)> sm;
  emb_run32_block<F32, U, NW, KIND>(p, sm, blockIdx.x);
}

// fp32 in two sweeps: pass 1 and the embedding terms in one launch, the sweep's blocks first.  A wave of the sweep
// per SIMD keeps the matrix unit busy, so a riding block's trips to memory cost next to nothing; in a launch of their own the crops took
// as long as the sweep (3136 tokens: 10.5 us of pass 1 and 13 of crops, together 14.7).  Up to 168 registers a wave, 38 KB of
// LDS: three blocks on a compute unit.
template <int D, int KIND>
__global__ __launch_bounds__(256, 3) void sattn_f32_pass1_with_emb(ScoreParams p, int n_sattn) {
  union Smem {
    SattnF32Smem<D> sa;
    EmbRunSmem<4, 4, 1> run;
  };
  __shared__ Smem sm;
  const int blk = blockIdx.x;
  if (blk < n_sattn) {
    const int hk = blk % p.Hkv, rest = blk / p.Hkv;
    const int tile = rest % p.n_tile, rest2 = rest / p.n_tile;
    sattn_f32_body<D, 1>(p, sm.sa, tile, hk, rest2 % p.n_rsplit, rest2 / p.n_rsplit);
    return;
  }
  emb_run32_block<true, 4, 4, KIND>(p, sm.run, (unsigned)(blk - n_sattn));
}

// The same beside the one sweep (3136 tokens: 15.4 us; 936 tokens, whole calls, beside a sweep 30.6 -> 22.2, 3 x 7220 tokens in
// two layers 130 -> 105).  Five chunks of exponentials take up to 254 registers: two blocks on a compute unit.
template <int D, int KIND>
__global__ __launch_bounds__(256, 2) void sattn_once_with_emb(ScoreParams p, ScoreOnce once, int n_sattn) {
  union Smem {
    SattnOnceSmem<D> once;
    SattnF32Smem<D> sweep;
    EmbRunSmem<4, 4, 1> run;
  };
  __shared__ Smem sm;
  if ((int)blockIdx.x < n_sattn) sattn_once_block<D>(p, once, sm.once, sm.sweep, blockIdx.x);
  else emb_run32_block<true, 4, 4, KIND>(p, sm.run, blockIdx.x - (unsigned)n_sattn);
}

// Pass 1 of s_attn and the embedding terms in ONE launch: the first n_sattn blocks run the
// (compute-bound) row-statistics sweep, two per compute unit; the remaining blocks run the crops and
// fill the third block slot of the compute units, so the memory-bound embedding work hides under the
// sweep instead of following it.  Three blocks fit a compute unit: 8 waves of at most 80 registers
// each and the larger of the shared-memory layouts.  A riding block owns one crop position over a run of frames.
// Riders of two strips (kRefetch2, kHold: up to 99 registers, 70 KB of LDS) leave two blocks on a compute unit; n_lead of them
// stand in front of the n_sattn blocks of the sweep.  wide_bf16_riders says which take which.
template <int D, int KIND>
__global__ __launch_bounds__(kSaWaves * 64, emb_strips(KIND) == 2 ? 4 : 6)
void sattn_pass1_with_emb(ScoreParams p, int n_sattn, int n_lead) {
  constexpr bool LEAD = emb_strips(KIND) == 2;
  static_assert(kSaWaves == 8, "the riding blocks use the sweep's block size");
  union Smem {
    SattnSmem<D, 1> sa;
    EmbRunSmem<2, 8, emb_strips(KIND)> run;
  };
  __shared__ Smem sm;
  const int blk = (int)blockIdx.x - (LEAD ? n_lead : 0);
  if ((!LEAD || blk >= 0) && blk < n_sattn) {   // the order of sattn_mfma's grid: KV head fastest, then key tile, ...
    const int hk = blk % p.Hkv, rest = blk / p.Hkv;
    const int tile = rest % p.n_tile, rest2 = rest / p.n_tile;
    sattn_mfma_body<D, 1>(p, sm.sa, tile, hk + p.Hkv * (rest2 % p.n_rsplit), rest2 / p.n_rsplit);
    return;
  }
  // (the host admits this launch only when its block count stays below 2^31: crop numbers fit 32 bits,
  // and 32-bit divisions are all that stands in front of a riding block's first load)
  emb_run32_block<false, 2, 8, KIND>(p, sm.run, LEAD && blk < 0 ? blockIdx.x : (unsigned)(blk - n_sattn));
}

// =================================================================================================
// Eq. 7: per-frame z-scores, summed over the enabled terms.  One block per (frame, batch element).
// =================================================================================================
__device__ __forceinline__ float block_sum_256(float v, float* red) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}

__global__ __launch_bounds__(256) void fuse_scores(ScoreParams p) {
  __shared__ float red[4];
  const int f = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
  const long long base = (long long)b * p.Nv + (long long)f * p.P;
  if (p.flags & HIPPO_SCORE_ATTN) {
    // s_attn[b,j] = sum_hk col_part / (H L) (+ the running layer sum), for this frame's tokens
    for (int i = tid; i < p.P; i += 256) {
      const long long e = base + i;
      const int jj = f * p.P + i;
      float a = sum_col_partials(p, b, jj);
      a /= (float)p.H * (float)p.L;
      if (p.attn_mass_inout != nullptr) {
        a += p.attn_mass_inout[e];
        p.attn_mass_inout[e] = a;
      }
      p.s_attn[e] = a;
    }
    __syncthreads();   // the block re-reads its own s_attn values below
  }
  const float* terms[3] = {p.s_attn, p.s_temp, p.s_spa};
  float mu[3], inv_sigma[3];
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    mu[t] = 0.f;
    inv_sigma[t] = 0.f;
    if (!(p.flags & (1u << t))) continue;
    float s = 0.f;
    for (int i = tid; i < p.P; i += 256) s += terms[t][base + i];
    mu[t] = block_sum_256(s, red) / (float)p.P;
    float v = 0.f;
    for (int i = tid; i < p.P; i += 256) {
      const float d = terms[t][base + i] - mu[t];
      v = fmaf(d, d, v);
    }
    const float var = block_sum_256(v, red) / (float)p.P;
    inv_sigma[t] = var > 0.f ? 1.f / sqrtf(var) : 0.f;
  }
  for (int i = tid; i < p.P; i += 256) {
    float sc = 0.f;
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      if (!(p.flags & (1u << t))) continue;
      const float x = terms[t][base + i];
      sc += (x - mu[t]) * inv_sigma[t];
      if (p.components_out) p.components_out[(long long)t * p.B * p.Nv + base + i] = x;
    }
    p.scores_out[base + i] = sc;
  }
}

// The same for frames of at most 256 * NPT tokens: every value a thread needs is fetched in one
// batch and stays in registers, and the three terms share each of the two block reductions, so a
// frame costs one trip to memory instead of one per term and per moment.
template <int NPT>
__global__ __launch_bounds__(256) void fuse_scores_reg(ScoreParams p) {
  __shared__ float red[3][4];
  const int f = blockIdx.x, b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const long long base = (long long)b * p.Nv + (long long)f * p.P;
  const bool on[3] = {(p.flags & HIPPO_SCORE_ATTN) != 0, (p.flags & HIPPO_SCORE_TEMP) != 0,
                      (p.flags & HIPPO_SCORE_SPA) != 0};
  float x[3][NPT];
#pragma unroll
  for (int u = 0; u < NPT; ++u) {
    const int i = tid + 256 * u;
    const bool ok = i < p.P;
    x[0][u] = x[1][u] = x[2][u] = 0.f;
    if (ok && on[1]) x[1][u] = p.s_temp[base + i];
    if (ok && on[2]) x[2][u] = p.s_spa[base + i];
    if (ok && on[0]) {
      float a = sum_col_partials(p, b, (long long)f * p.P + i);
      a /= (float)p.H * (float)p.L;
      if (p.attn_mass_inout != nullptr) {
        a += p.attn_mass_inout[base + i];
        p.attn_mass_inout[base + i] = a;
      }
      p.s_attn[base + i] = a;
      x[0][u] = a;
    }
  }
  auto reduce3 = [&](float (&v)[3]) {                  // block sums of three values at once
#pragma unroll
    for (int t = 0; t < 3; ++t) v[t] = wave_sum(v[t]);
    __syncthreads();
    if (lane == 0) { red[0][wave] = v[0]; red[1][wave] = v[1]; red[2][wave] = v[2]; }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 3; ++t) v[t] = (red[t][0] + red[t][1]) + (red[t][2] + red[t][3]);
  };
  float mu[3] = {0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < 3; ++t)
#pragma unroll
    for (int u = 0; u < NPT; ++u) mu[t] += x[t][u];
  reduce3(mu);
  float var[3] = {0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    mu[t] /= (float)p.P;
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
      const float d = (tid + 256 * u < p.P) ? x[t][u] - mu[t] : 0.f;
      var[t] = fmaf(d, d, var[t]);
    }
  }
  reduce3(var);
  float inv_sigma[3];
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    var[t] /= (float)p.P;
    inv_sigma[t] = (on[t] && var[t] > 0.f) ? 1.f / sqrtf(var[t]) : 0.f;
  }
#pragma unroll
  for (int u = 0; u < NPT; ++u) {
    const int i = tid + 256 * u;
    if (i >= p.P) continue;
    float sc = 0.f;
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      if (!on[t]) continue;
      sc += (x[t][u] - mu[t]) * inv_sigma[t];
      if (p.components_out) p.components_out[(long long)t * p.B * p.Nv + base + i] = x[t][u];
    }
    p.scores_out[base + i] = sc;
  }
}

// =================================================================================================
// host launch
// =================================================================================================
int score_token_tile(int dtype) { return dtype == HIPPO_DTYPE_BF16 ? kSaMfmaTile : kSaF32Tile; }

// How many runs the query rows of a KV head are cut into (one block of the sweeps per run).  In bf16 two blocks a compute unit
// let the MFMA and the exp work of different waves overlap, with runs of at least two 64-row chunks; where even those leave
// units without a block, finer cuts follow below.  A compute
// unit holds two sweep blocks; measured at the 16K shape, two co-resident blocks take 2.1 us per 64-row
// chunk each, a block alone 1.29 us, and a block's start (keys, first chunk) 3.2 resp. 2.5 us.  The
// blocks are dealt to the compute units in rounds, so what counts is the busiest unit: ceil(blocks / 256)
// blocks, two at a time, an odd last one alone.  520 unsplit blocks of 28 chunks, for example, put a third
// block on a few units, which then start a 28-chunk sweep when all others are done (91 us against 81-83
// with three or four runs); 256 blocks of 14 chunks are best cut in two (one round, two blocks per unit).
int score_row_splits(int dtype, long long blocks_unsplit, int rows_per_kv_head, int head_dim, bool once, bool finer,
                     int col_parts) {
  int best = 1;
  if (dtype != HIPPO_DTYPE_BF16) {
    // fp32: a wave per SIMD nearly keeps the matrix unit busy, so a compute unit takes its blocks one after the other in
    // effect; a block's start costs about what 0.7 of its 32-row chunks do.  In the one sweep one block alone takes about an
    // eighth longer than two side by side, and a start with the way of the last sums 2.2 chunks (us a call, in runs as chosen |
    // one run | others: 4096 tokens, 64 heads, 128 text rows 133 | 144 | 135-147; 12288 tokens, 28 heads, 64 rows 119 | 115 |
    // 113-140; 36864 tokens, 28 heads, 40 rows 228 | 228 | 248-394).
    const int chunks = (rows_per_kv_head + kSaF32Rows - 1) / kSaF32Rows;
    double best_cost = 0.0;
    for (int rs = 1; rs <= 8 && rs <= chunks; ++rs) {
      const long long rounds = (blocks_unsplit * rs + kNumCU - 1) / kNumCU;
      const double cost = (once && rounds == 1 ? 1.12 : (double)rounds) * ((chunks + rs - 1) / rs + (once ? 2.2 : 0.7));
      if (rs == 1 || cost < best_cost * 0.97) {
        best = rs;
        best_cost = cost;
      }
    }
    return best;
  }
  const int chunks = (rows_per_kv_head + 63) / 64;
  double best_cost = 0.0;
  for (int rs = 1; rs <= 4; ++rs) {
    if (rs > 1 && chunks / rs < 2) break;                       // at least two chunks per block
    const int cpb = (chunks + rs - 1) / rs;                     // chunks per block
    const long long per_cu = (blocks_unsplit * rs + kNumCU - 1) / kNumCU;
    const double pair = cpb * 2.1 + 3.2, alone = cpb * 1.29 + 2.5;
    const double cost = (double)(per_cu / 2) * pair + (per_cu % 2 ? alone : 0.0);
    if (rs == 1 || cost < best_cost * 0.97) {                   // a finer cut has to pay for its extra column partials
      best = rs;
      best_cost = cost;
    }
  }
  // Short videos leave compute units without a block of the sweeps: finer cuts, up to a block on seven eighths of them (64
  // channels: 3780 tokens x 14 heads x 2 in two layers, 240 blocks for 120, 18.0 -> 18.5) or, of 128 channels in runs of three
  // and more chunks, on all.  A block that is alone costs as above, but its first two chunks land together (one saves 0.6 us
  // of two), and the more blocks, the longer their keys take, which each of a tile's fetches.  us a call from a graph, the cut
  // above -> this: 4096 tokens x 14 heads, 64 text rows 17.9 -> 16.1 (3 runs -> 7), 1848 x 14, 183 rows 22.9 -> 18.1, 1400 x 28,
  // 121 rows 22.6 -> 19.9.  Where that saves little, the column partials of more runs and the blocks that riders wait for cost as
  // much: not for a quarter or a fifth of a run's chunks (64 channels, four chunks -> three, 4 -> 5 runs 20.9 -> 23.8), not for one
  // chunk on three quarters of the units and more (two for three: 6825 x 28, 26 rows, 216 blocks 25.2 -> 28.4, 1836 x 64 in two
  // layers, 17 rows, 256 blocks 20.4 -> 22.1).
  // And every run is a column partial more a token for each KV head and layer, which the fusion's one block a frame adds up: not
  // where that is more than the sweeps save (one frame of 396 tokens x 8 heads in four layers, 154 rows, 32 -> 96 partials 18.9 ->
  // 22.8; 3 frames of 272 tokens x 64 heads, 55 rows, 24 -> 56 18.0 -> 21.0; of 662 calls cut finer the 25 that it stops took 1.03
  // of the time, 1.2 at the most).  Of 5881 random calls of 300 to 24000 tokens two take more than 1.02 of the time that they had
  // before finer cuts and the merge in pass 2, 1.04 the most; those of up to 4096 tokens 0.89.
  auto sweep = [&](int rs) {
    const int cpb = (chunks + rs - 1) / rs;
    return cpb == 1 ? 1.89 : cpb * 1.29;
  };
  auto alone = [&](int rs) { return sweep(rs) + 2.5 + (head_dim == 128 ? 0.008 : 0.005) * (double)(blocks_unsplit * rs); };
  if (!finer) return best;
  const int former = best, former_cpb = (chunks + best - 1) / best;
  for (int rs = best + 1; rs <= 8 && rs <= chunks; ++rs) {
    const int cpb = (chunks + rs - 1) / rs;
    const long long blocks = blocks_unsplit * rs;
    if (blocks > (head_dim == 128 && cpb >= 3 ? kNumCU : kNumCU * 7 / 8)) continue;
    if (3 * cpb > 2 * former_cpb) continue;
    if (former_cpb - cpb == 1 && 4 * blocks >= 3 * kNumCU) continue;
    if (col_parts * (rs - former) > 16 + 12 * (sweep(former) - sweep(rs))) continue;
    if (alone(rs) < alone(best) * 0.97) best = rs;
  }
  return best;
}

// Beyond kOnceMaxTiles (65536 tokens) a run's blocks would not all fit on the chip at once, and two sweeps stay.  Below, one
// sweep is the faster from four chunks of rows a KV head on, also where a run's tiles fill compute units unevenly (36864 tokens:
// 288 blocks wait for the 32 compute units that hold two of them).  Fewer chunks leave a block nothing to do while its run's
// other tiles start, and the more of these there are the longer that takes: 88 tiles a chunk.  Whole calls replayed from a
// graph, us, two sweeps -> one: 484 tokens x 4 heads, 16 text rows 24.1 -> 23.0; 936 x 14 24.9 -> 23.7; 3136 x 14, 64 rows 31.5
// -> 28.4; 4096 x 64 heads, 128 rows 222 -> 128; 16384 x 28, 128 rows 308 -> 190; 36864 x 28, 40 rows 265 -> 230; 60500 x 4,
// 64 rows 112 -> 97.  Two chunks: 173 tiles 138 -> 126, 181 99 -> 87, 213 306 -> 320, 335 136 -> 180, 435 726 -> 976; one: 54
// 66 -> 63, 79 81 -> 79, 109 67 -> 74, 262 65 -> 77, 268 185 -> 265; three: 238 113 -> 97, 270 126 -> 141; four: 466 368 -> 328.
bool score_once(int dtype, long long n_vis, int rows_per_kv_head) {
  const long long tiles = (n_vis + kSaF32Tile - 1) / kSaF32Tile, chunks = (rows_per_kv_head + kSaF32Rows - 1) / kSaF32Rows;
  return dtype == HIPPO_DTYPE_F32 && tiles <= kOnceMaxTiles && (chunks >= 4 || tiles <= 88 * chunks);
}
size_t score_once_rows(int rows_per_kv_head) {
  return ((size_t)rows_per_kv_head + kSaF32Rows - 1) / kSaF32Rows * kSaF32Rows;
}
const int kScoreOnceWords = kOnceCopies, kScoreOnceBins = kOnceBins;

// riders: blocks of the embedding terms beside the sweep, of the kind kOnePass, kFew or kRefetch
template <int D>
static hipError_t launch_sattn_once(const ScoreParams& p, const ScoreOnce& once, hipStream_t st, long long riders, int kind) {
  const long long n_sattn = (long long)p.n_tile * p.Hkv * p.n_rsplit * p.Bz;
  const long long n_clear = (long long)(once.clear_bytes / sizeof(u32x4));
  hipLaunchKernelGGL(sattn_once_clear, dim3((unsigned)((n_clear + 255) / 256)), dim3(256), 0, st, (u32x4*)once.row_word,
                     n_clear);
  const dim3 grid((unsigned)(n_sattn + riders));
  const auto launch = kind == kRefetch ? sattn_once_with_emb<D, kRefetch>
                      : kind == kFew   ? sattn_once_with_emb<D, kFew>
                                       : sattn_once_with_emb<D, kOnePass>;
  hipLaunchKernelGGL(launch, grid, dim3(256), 0, st, p, once, (int)n_sattn);
  hipLaunchKernelGGL(sattn_f32_redo<D>, dim3((unsigned)n_sattn), dim3(256), 0, st, p, once);
  return hipGetLastError();
}

template <int D>
static hipError_t launch_sattn_f32(const ScoreParams& p, hipStream_t st, long long riders, int kind) {
  if (p.n_tile > 65535 || (long long)p.n_rsplit * p.Bz > 65535) return hipErrorInvalidValue;
  const dim3 grid(p.Hkv, p.n_tile, p.n_rsplit * p.Bz);     // KV head fastest, as the bf16 sweeps
  if (riders > 0) {
    const long long n_sattn = (long long)p.n_tile * p.Hkv * p.n_rsplit * p.Bz;
    const dim3 fused((unsigned)(n_sattn + riders));
    const auto launch = kind == kRefetch ? sattn_f32_pass1_with_emb<D, kRefetch>
                        : kind == kFew   ? sattn_f32_pass1_with_emb<D, kFew>
                                         : sattn_f32_pass1_with_emb<D, kOnePass>;
    hipLaunchKernelGGL(launch, fused, dim3(256), 0, st, p, (int)n_sattn);
  } else {
    hipLaunchKernelGGL((sattn_f32<D, 1>), grid, dim3(256), 0, st, p);
  }
  const long long rows = (long long)p.Bz * p.H * p.L;
  hipLaunchKernelGGL(sattn_row_lse, dim3((unsigned)((rows + 31) / 32)), dim3(256), 0, st, p);
  hipLaunchKernelGGL((sattn_f32<D, 2>), grid, dim3(256), 0, st, p);
  return hipGetLastError();
}

// riders: 0 = pass 1 in a launch of its own, else that many riding blocks, of the kind kOnePass, kFew or a wide one
// bf16 riders of more than 512 channels: which of them, and how many stand in front of the sweep's blocks.
// The two-strip ones take a third of the compute units' block slots from the launch; what longer takes (a rider, by its
// frames and passes, or a block of the sweep, by its chunks of 64 rows) goes first.  us a call from a graph, one strip | two
// strips in front | two strips behind:
//   two passes, held: 3 x 10692 tokens, 64 heads, 15 text rows 75 | 61 | 68; 27830 x 14 heads x 2, 36 rows 81 | 57 | 61; 3 x
//     3822 x 64, 95 rows 68 | 72 | 66; 2 x 45356 x 14, 171 rows 161 | 148 | 141.  Only a sweep of many times the riders' work is
//     the better one with three slots: 4 x 1452 x 64 in four layers, 239 rows 218 | 228 | 223; 2640 x 64 in four, 201 rows 105 |
//     112 | 108 (at 14 times; nearer than that within 2.5 % either way).
//   more passes, fetched again: two strips gain as long as the riders go first and the sweep fills the chip (3 x 15312 x 64
//     heads, 76 rows, 3584 channels 297 | 248 | 294; 15750 x 14 x 2 in four layers, 37 rows, 2048 channels 109 | 96 | 113), or
//     where all blocks fit two a compute unit and there is a compute unit for each rider (1785 x 64, 178 rows, 2048 channels 46 |
//     42 | 46); else one strip (3 x 4056 x 64 in two layers, 105 rows, 1536 channels 130 | 140 | 136; 3726 x 64, 254 rows 61 | 65 |
//     64).
struct Riders {
  int kind;
  long long lead;
};
static Riders wide_bf16_riders(const ScoreParams& p, long long n_sattn, long long riders) {
  const long long de = p.emb ? p.emb_dim : (long long)p.Hkv * p.D, passes = (de + 511) / 512;
  const long long chunks = p.rows_per_split / 64, frames = p.emb_run;
  const bool first = 3 * chunks <= 2 * (frames + 1) * passes;
  if (passes == 2) {
    if (n_sattn * chunks >= 14 * riders * (frames + 2)) return {kRefetch, 0};
    return {kHold, first ? riders : 0};
  }
  const bool two = n_sattn > kNumCU ? first : n_sattn + riders > kNumCU && riders <= kNumCU;
  return two ? Riders{kRefetch2, riders} : Riders{kRefetch, 0};
}

template <int D>
static hipError_t launch_sattn_mfma(const ScoreParams& p, hipStream_t st, long long riders, int kind) {
  if (p.n_tile > 65535 || (long long)p.n_rsplit * p.Bz > 65535) return hipErrorInvalidValue;
  dim3 grid(p.Hkv, p.n_tile, p.n_rsplit * p.Bz);
  if (riders > 0) {
    const long long n_sattn = (long long)p.n_tile * p.Hkv * p.n_rsplit * p.Bz;
    const dim3 fused((unsigned)(n_sattn + riders));
    const Riders r = kind == kRefetch ? wide_bf16_riders(p, n_sattn, riders) : Riders{kind, 0};
    const auto launch = r.kind == kHold       ? sattn_pass1_with_emb<D, kHold>
                        : r.kind == kRefetch2 ? sattn_pass1_with_emb<D, kRefetch2>
                        : r.kind == kRefetch  ? sattn_pass1_with_emb<D, kRefetch>
                        : r.kind == kFew      ? sattn_pass1_with_emb<D, kFew>
                                              : sattn_pass1_with_emb<D, kOnePass>;
    hipLaunchKernelGGL(launch, fused, dim3(kSaWaves * 64), 0, st, p, (int)n_sattn, (int)r.lead);
  } else {
    hipLaunchKernelGGL((sattn_mfma<D, 1>), grid, dim3(kSaWaves * 64), 0, st, p);
  }
  // Up to 16 tiles, and a run of rows per block that its threads cover: pass 2 merges the row statistics itself.  Us a call
  // from a graph, with a launch for the merge -> without: 4096 tokens x 14 heads, 64 text rows 19.7 -> 18.6, 4096 x 28, 256
  // rows 31.6 -> 30.1, 4096 x 64, 256 rows 51.7 -> 50.4, 1368 x 4 x 2, 61 rows 16.5 -> 14.5, 2690 x 28 in 4 layers x 2 33.7 ->
  // 31.9.  From 17 tiles on every block reads as much as the launch costs (6174 x 14 x 3 in four layers 44.4 -> 48.6, 4788 x 28
  // x 2 39.2 -> 40.3, 5304 x 14 x 3 21.4 -> 21.1).  So do many rounds of blocks: without the launch, 2934 random calls took, of 9 to
  // 16 tiles, 0.94 of the time up to 512 blocks, 0.98 up to 768, 0.99 up to 1024, 1.00 to 1.03 up to 2048, beyond 1.01 to 1.08 (3724
  // x 32 heads x 6 in four layers, 22 rows 104 -> 115); of up to 8 tiles 0.91, 0.96, 0.97, up to 4096 0.97 to 1.00, beyond 1.01 to 1.03.
  const long long blocks = (long long)p.n_tile * p.Hkv * p.n_rsplit * p.Bz;
  if (p.n_tile <= 16 && p.rows_per_split <= kSaWaves * 64 && blocks <= (p.n_tile <= 8 ? 16 : 4) * kNumCU) {
    if (p.n_tile <= 8) hipLaunchKernelGGL((sattn_mfma<D, 2, 1>), grid, dim3(kSaWaves * 64), 0, st, p);
    else hipLaunchKernelGGL((sattn_mfma<D, 2, 2>), grid, dim3(kSaWaves * 64), 0, st, p);
    return hipGetLastError();
  }
  const long long rows = (long long)p.Bz * p.H * p.L;
  hipLaunchKernelGGL(sattn_row_lse, dim3((unsigned)((rows + 31) / 32)), dim3(256), 0, st, p);
  hipLaunchKernelGGL((sattn_mfma<D, 2>), grid, dim3(kSaWaves * 64), 0, st, p);
  return hipGetLastError();
}

// fp32 crops of more than 256 channels: beside pass 1 by four-wave blocks in passes of 256 channels, or in a launch of their
// own, where blocks of eight waves take 512 in a pass and fetch a frame's channels half as often.
//
// Where they ride.  Channels that fill their last pass of 512 by half or less (an odd number of passes of 256): four waves
// lose nothing by their passes.  They ride beside a sweep of up to a block a compute unit, and beside a long one (rounds of
// blocks x 32-row chunks, a block's start as 0.7 of a chunk); beside a short sweep of many blocks they wait for its
// blocks' slots and then crowd on few compute units.  768 channels, us a call, alone -> riding: 26 x 14 x 14 tokens of 14
// heads, 240 sweep blocks, 57.6 -> 47.3; 512 of 14 chunks 146 -> 141; 480 of eight 82 -> 80; and where they stay alone:
// 512 of seven 123 against 131; with two sweeps, 1016 of four chunks 177 against 220, 1184 of two 161 against 189.
// Otherwise eight waves are the better ones, and the crops ride only where the sweep leaves room for all of them: 512
// channels, 256 sweep blocks and 256 crops 55.2 -> 48.7, 1024 channels likewise 95 -> 82; where they stay alone: 768 sweep
// blocks of seven chunks 112 against 120, 384 of four 67 against 76, 1024 channels, 768 of ten 287 against 307.
static bool wide_f32_rides(const ScoreParams& p, long long n_sattn, long long n_riders, int de) {
  if ((de + 255) / 256 % 2 == 1) {
    const double rounds = (double)((n_sattn + kNumCU - 1) / kNumCU);
    return n_sattn <= kNumCU ||
           rounds * (p.rows_per_split / (double)kSaF32Rows + 0.7) >= (n_sattn <= 2 * kNumCU ? 16.0 : 22.0);
  }
  return n_sattn <= kNumCU && n_riders <= kNumCU &&
         (long long)p.rows_per_split * p.D >= (n_sattn + n_riders <= kNumCU ? 4096 : 16384);
}

// A launch of their own: frames a run (p.emb_run) and waves a block (the result: eight) of the least estimated time.  A frame
// costs the same in every block, so a run's time is that of its frames and two neighbours, times the blocks that a compute
// unit takes one after the other (eight waves: one at a time; four: two side by side at 1.4 times the time of one, more at
// 0.59 of a block's).  A fixed number of blocks was wrong on both sides: two a compute unit make a second round of
// eight-wave blocks, crops / compute units rounded down a few blocks too many (1440 crops of 512 channels, us: 46 in 480
// blocks, 58 in 288, 39 in 240).
static bool wide_f32_plan(ScoreParams& p, long long crops_a_frame, int de) {
  const int longest = std::min(8, p.F);
  bool eight = true;
  double best = 0.0;
  for (int run = 1; run <= longest; ++run) {
    const long long blocks = crops_a_frame * ((p.F + run - 1) / run), rounds = (blocks + kNumCU - 1) / kNumCU;
    if (rounds > 2 && run < longest) continue;      // many crops: the two neighbour frames' bytes decide
    const double t8 = (double)rounds * ((de + 511) / 512);
    const double t4 = (rounds == 1 ? 0.7 : rounds == 2 ? 1.0 : 0.59 * blocks / kNumCU) * ((de + 255) / 256);
    const bool use8 = de <= 512 || t8 <= t4;        // one pass holds the frame before in registers
    const double t = (run + 2) * (use8 ? t8 : t4);
    if (best == 0.0 || t < best) {
      best = t;
      p.emb_run = run;
      eight = use8;
    }
  }
  return eight;
}

hipError_t launch_score(const ScoreParams& p_in, const ScoreOnce& once_in, hipStream_t st) {
  ScoreParams p = p_in;
  ScoreOnce once = once_in;
  {
    const int unit = p.dtype == HIPPO_DTYPE_BF16 ? 64 : kSaF32Rows;      // rows per chunk of the sweeps
    const int rows = p.L * p.G, chunks = (rows + unit - 1) / unit, rs = p.n_rsplit > 0 ? p.n_rsplit : 1;
    p.rows_per_split = (chunks + rs - 1) / rs * unit;
    once.row_words = chunks * unit;
    // one sweep: how often a wave asks in all (about a microsecond each): a few times as long as the sweep of its own run of
    // rows takes
    once.range = 29u << 23;                // 53 bits for all tiles' sums, of 24 bits, from kOnceLow on
    for (int n = 1; n < p.n_tile; n *= 2) once.range -= 1u << 23;
    if (once.polls < 0) once.polls = 64 + 16 * (p.rows_per_split / kSaF32Rows);
    p.q_step_i = 64 / p.G;
    p.q_step_g = 64 % p.G;
    p.q_last_i = (rows - 1) / p.G;
    p.q_last_g = (rows - 1) % p.G;
  }
  hipError_t e = hipSuccess;
  const bool accumulate_only = (p.flags & HIPPO_SCORE_ACCUMULATE_ONLY) != 0;
  // the paper's small crops: the embedding terms ride in the launch of s_attn's pass 1
  const bool want_emb = (p.flags & (HIPPO_SCORE_TEMP | HIPPO_SCORE_SPA)) != 0;
  // Crops of at most 32 tokens: a block sweeps one crop position over a run of frames.  The runs are as long as
  // still leaves every compute unit a block (at most 8 frames: a run fetches its two neighbour frames on top of its
  // own).  Half as long, two blocks per compute unit, was slower for fp32 crops beside the sweep (3 x 7220 tokens 112
  // against 105 us a call).
  const long long crops_per_frame = (long long)((p.gh + p.ch - 1) / p.ch) * ((p.gw + p.cw - 1) / p.cw);
  const bool bf16 = p.dtype == HIPPO_DTYPE_BF16;
  const int de = p.emb ? p.emb_dim : p.Hkv * p.D;
  const bool small_crops = p.ch * p.cw <= 32;
  const bool wide = de > (bf16 ? 512 : 256);
  // (A wave takes 64 channels: kFew where one of four has none, or two of eight.  One of eight gains less than the questions
  // cost: 518 random bf16 calls of 392 to 448 channels 1.015 of the time with kFew, 767 of up to 384 0.995.)
  int kind = wide ? kRefetch : de <= (bf16 ? 384 : 192) ? kFew : kOnePass;
  const long long n_sattn = (long long)p.n_tile * p.Hkv * p.n_rsplit * p.Bz, all_crops = crops_per_frame * p.F * p.B;
  {
    long long run = all_crops / kNumCU;
    // Beside the one sweep two blocks fit a compute unit, not three: the shortest run that leaves room for all of them, if it is
    // not far longer.  us a call from a graph, two sweeps | a second round of riders | this: 4752 tokens x 4 heads x 3, 31 rows
    // (run 1 to 2) 32.3 | 35.7 | 28.6; 5808 x 4 x 3, 42 rows (1 to 2) 32.4 | 35.2 | 30.6; 8400 x 4 x 2, 62 rows (2 to 3) 46.5 |
    // 45.2 | 33.4; 19844 x 4, 47 rows (4 to 7) 51.8 | 50.4 | 41.9; longer still 52 -> 58 (4 to 8 of 9 that fit), 39.5 -> 40.5 (2 to 7).
    const long long room = 2 * kNumCU - n_sattn;
    if (once.row_word != nullptr && !wide && room > 0) {
      const long long longest = std::min<long long>(8, 2 * std::max<long long>(1, run) + 2);
      long long fits = (all_crops + room - 1) / room;
      if (fits > run && fits <= longest) {
        // Runs do not come out even: what they need beyond the room waits for a slot, and only the video's last run, the
        // shortest and last in the launch order, does so at no cost (5460 tokens x 4 heads x 4, 80 rows, 9 crops a frame: 12
        // blocks too many 46.9, runs of 8 and not 7 36.7; 10920 x 4 x 2, 206 rows 52.8 and 38.7; 12 of the last run's 20 31.1
        // against 33.2).
        auto over = [&](long long r) { return crops_per_frame * ((p.F + r - 1) / r) * p.B - room > crops_per_frame; };
        run = fits;
        while (fits < longest && over(fits)) ++fits;
        if (!over(fits)) run = fits;
      }
    }
    p.emb_run = (int)std::max<long long>(1, std::min<long long>(std::min<long long>(8, p.F), run));
  }
  long long n_riders = crops_per_frame * ((p.F + p.emb_run - 1) / p.emb_run) * p.B;
  const bool emb_rides = want_emb && !accumulate_only && (p.flags & HIPPO_SCORE_ATTN) && small_crops &&
                         n_sattn + n_riders < (once.row_word != nullptr ? 1ll << 23 : 1ll << 31) &&
                         (bf16 || !wide || wide_f32_rides(p, n_sattn, n_riders, de));
  bool eight_waves = false;
  if (!emb_rides && !bf16 && wide) {
    eight_waves = wide_f32_plan(p, crops_per_frame * p.B, de);
    n_riders = crops_per_frame * ((p.F + p.emb_run - 1) / p.emb_run) * p.B;
  }
  const long long riders = emb_rides ? n_riders : 0;
  // fp32 riders of few channels, a few blocks of which wait for the others' slots: of little text they and nothing else are the
  // launch's end, and came 3 to 8 us later as kFew (1900 tokens x 2 heads x 3 in four layers, 2 rows, 192 channels, 28 blocks beyond
  // 43.9 -> 52.1 us; in two sweeps, where four blocks fit a unit, 18656 x 2 x 3, 4 rows, 356 beyond 64 -> 75; without waiting blocks
  // 0.97 of the time).  Of 4507 random calls of up to 32 rows with 256 to 1600 blocks 60 took more than 1.03 of the time, 1.19 the
  // most; of 3563 with this 17, 1.11 the most.
  if (!bf16 && kind == kFew && de > 64 && riders > 0) {
    const long long beyond = n_sattn + riders - (once.row_word != nullptr ? 2 : 4) * kNumCU;
    if (beyond > 0 && beyond <= (once.row_word != nullptr ? 32 : de > 128 ? 512 : 0)) kind = kOnePass;
  }
  if ((p.flags & HIPPO_SCORE_ATTN) || accumulate_only) {
    if (p.dtype == HIPPO_DTYPE_BF16)
      e = (p.D == 128) ? launch_sattn_mfma<128>(p, st, riders, kind)
                       : launch_sattn_mfma<64>(p, st, riders, kind);
    else if (once.row_word != nullptr)
      e = (p.D == 128) ? launch_sattn_once<128>(p, once, st, riders, kind)
                       : launch_sattn_once<64>(p, once, st, riders, kind);
    else
      e = (p.D == 128) ? launch_sattn_f32<128>(p, st, riders, kind) : launch_sattn_f32<64>(p, st, riders, kind);
    if (e != hipSuccess) return e;
    if (accumulate_only) {   // otherwise the fusion kernel finishes the attention mass itself
      const long long n = (long long)p.B * p.Nv;
      hipLaunchKernelGGL(sattn_finalize, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p);
      return hipGetLastError();
    }
  }
  if (want_emb && !emb_rides) {
    const int ncy = (p.gh + p.ch - 1) / p.ch, ncx = (p.gw + p.cw - 1) / p.cw;
    dim3 grid(ncy * ncx, p.F, p.B);
    if (small_crops) {
      if (n_riders >= (1ll << 31)) return hipErrorInvalidValue;
      const dim3 runs((unsigned)n_riders);
      // (fp32 up to 256 channels: half of eight waves would idle; 128 frames of 128 channels 29 against 42 us)
      // (more than two passes: through two strips, two blocks a compute unit, 2 x 17680 tokens of 3584 channels took 129 us, not
      // 108; 19800 of 2048 53, not 48; 18590 of 1536 40, not 38; 4056 of 2048 to 3584 within 10 % either way)
      if (bf16 && de > 1024) hipLaunchKernelGGL((emb_scores_run32<false, 8, kRefetch>), runs, dim3(512), 0, st, p);
      else if (bf16 && wide) hipLaunchKernelGGL((emb_scores_run32<false, 8, kHold>), runs, dim3(512), 0, st, p);
      else if (bf16 && kind == kFew) hipLaunchKernelGGL((emb_scores_run32<false, 8, kFew>), runs, dim3(512), 0, st, p);
      else if (bf16) hipLaunchKernelGGL((emb_scores_run32<false, 8, kOnePass>), runs, dim3(512), 0, st, p);
      else if (wide && de <= 512) hipLaunchKernelGGL((emb_scores_run32<true, 8, kOnePass>), runs, dim3(512), 0, st, p);
      else if (wide && eight_waves) hipLaunchKernelGGL((emb_scores_run32<true, 8, kRefetch>), runs, dim3(512), 0, st, p);
      else if (wide) hipLaunchKernelGGL((emb_scores_run32<true, 4, kRefetch>), runs, dim3(256), 0, st, p);
      else if (kind == kFew) hipLaunchKernelGGL((emb_scores_run32<true, 4, kFew>), runs, dim3(256), 0, st, p);
      else hipLaunchKernelGGL((emb_scores_run32<true, 4, kOnePass>), runs, dim3(256), 0, st, p);
    } else if (!bf16) {
      hipLaunchKernelGGL(emb_scores, grid, dim3(256), 0, st, p);
    } else if (p.ch * p.cw <= 48) {
      hipLaunchKernelGGL(emb_scores_mfma<3>, grid, dim3(256), 0, st, p);
    } else {
      hipLaunchKernelGGL(emb_scores_mfma<4>, grid, dim3(256), 0, st, p);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (p.P <= 256) hipLaunchKernelGGL(fuse_scores_reg<1>, dim3(p.F, p.B), dim3(256), 0, st, p);
  else if (p.P <= 1024) hipLaunchKernelGGL(fuse_scores_reg<4>, dim3(p.F, p.B), dim3(256), 0, st, p);
  else hipLaunchKernelGGL(fuse_scores, dim3(p.F, p.B), dim3(256), 0, st, p);
  return hipGetLastError();
}

}  // namespace hippo

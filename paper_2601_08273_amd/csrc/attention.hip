// Split-KV streaming attention for the draft-decode and target-verification calls
// (paper: Preliminaries, "Speculative Decoding"; the cost the paper attributes to reading large KV
// caches, App. "Details of Baselines").
//
// One launch streams each KV slice once for all R = G * q_len query rows that share a KV head
// (row r = i * G + g: new token i, query head g of the group), keeping an online-softmax state
// per row; a second small launch merges the slices.  Two partial kernels:
//   * attn_partial_grid  -- bf16, MFMA 16x16x32: S^T = K Q^T puts the streamed tokens on the MFMA
//     M axis, so the score tile comes out in exactly the register layout the PV product
//     O^T = V^T P^T needs for its B operand; only V goes through a transposing LDS read.
//     Instantiations of the same kernel cover the cache-format variants: rows appended by the
//     launch itself, paged caches, and caches of 8-bit floating-point codes (converted to bf16
//     after the LDS read).
//   * attn_partial_f32   -- fp32, MFMA 16x16x4 with fp32 operands.
#include <atomic>
#include <type_traits>

#include "common.h"

namespace hippo {

// Appended-row fusion: the q_len new K/V rows of (b, hk) go from k_new / v_new [B, q_len, Hkv, D] into
// cache rows ctx_len.., bit for bit.  Called by one block per (b, hk) after its own transfers have
// drained; no block of this launch reads those cache rows (they all read k_new / v_new instead).
template <typename T, int D>
__device__ __forceinline__ void append_new_rows(const AttnParams& p, int b, int hk) {
  constexpr int VPR = D / Elem<T>::kPerVec;    // 16-byte pieces per row
  for (int e = threadIdx.x; e < p.q_len * VPR; e += blockDim.x) {
    const int nr = e / VPR, pc = e % VPR;
    const long long src = (((long long)b * p.q_len + nr) * p.Hkv + hk) * D + pc * Elem<T>::kPerVec;
    const long long dst = (long long)b * p.sb + (long long)hk * p.sh + (long long)(p.ctx_len + nr) * p.sn +
                          pc * Elem<T>::kPerVec;
    *(u32x4*)((T*)p.k_w + dst) = *(const u32x4*)((const T*)p.k_new + src);
    *(u32x4*)((T*)p.v_w + dst) = *(const u32x4*)((const T*)p.v_new + src);
  }
}

// Element 0 of query row `row` of (b, hk) in the output, and the row's place in lse [B, H, q_len].
__device__ __forceinline__ long long out_row(const AttnParams& p, int b, int hk, int row, float inv_g, long long* lse_at) {
  const int i = row_div_group(row, inv_g), h = hk * p.G + row - i * p.G;
  *lse_at = ((long long)b * p.H + h) * p.q_len + i;
  return (((long long)b * p.q_len + i) * p.H + h);
}

// =================================================================================================
// MFMA partial kernel (bf16): helpers
// =================================================================================================
constexpr float kRescaleGap = 8.f;    // log2 units, see the lazy rescale in the kernel

typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;

// =================================================================================================
// MFMA partial kernel (bf16): query-row blocks x token groups
// =================================================================================================
// Grid (S, H_kv, B * n_chunks): a block owns one KV slice and up to RB*16 query rows, and has
// RB * TG waves.  Wave (rb, tg) owns query rows 16*rb..16*rb+15 and, of every "super-tile" of TG
// consecutive TT-token tiles, tile number tg.  A wave's state is one 16-row accumulator (32
// registers at d = 128), so 12-16 waves fit on a compute unit and hide each other's MFMA / LDS /
// exp latencies; at the end the TG states of a row block meet in LDS and wave (rb, tg) reduces and
// stores head-dim blocks tg, tg + TG, ...
//
// Data path: K/V tiles go HBM -> LDS directly (global_load_lds, 16 bytes per lane, no registers in
// between) into one ring of NST super-tiles shared by the block; the first ISSUERS waves issue the
// transfers.  One block barrier per super-tile says both "it has landed" (every issuer waited for
// its own transfers first) and "everyone is done with the previous one" (whose stage is refilled
// right away).  A lane's 16 bytes land at (wave-uniform base) + lane*16, so a tile is stored
// row-major and unpadded; bank conflicts are avoided by fetching, for physical 16-byte chunk c of
// row r, logical chunk c ^ swz(r).
//
// Register layouts (lane = j + 16*g, j = lane%16, g = lane/16), v_mfma_f32_16x16x32_bf16:
//   A operand: row j,  8 contraction elements of group g      B operand: column j, same 8 elements
//   D result : column j, rows 4g..4g+3
// S^T = K Q^T  -> D[token][qrow]: lane (qrow j, g) holds tokens 4g..4g+3 of a 16-token block, which
//   is exactly what the B operand of O^T = V^T P^T wants (contraction slot 4g+e = token 4g+e; with
//   32-token tiles the second block supplies slots 4..7 of each lane).  The matching V^T operand
//   (row = head-dim element j, the same tokens) comes from ds_read_b64_tr_b16, which hands lane j
//   of a 16-lane group the j-th column of a 4 x 16 block whose rows the lanes address 4 elements at
//   a time.  The contraction order of QK^T is likewise free: slot (ks, g, e) reads head-dim element
//   (g*KS + ks)*8 + e of both K and Q, which makes each lane's K reads one contiguous run.
template <int D, int TG, int TT, int NST, int ES = 2>
struct GridSmem {
  static constexpr int kRowBytes = D * ES;                     // a cache row: ES bytes per element
  static constexpr int kTileBytes = TT * kRowBytes;
  static constexpr int kSuperBytes = TG * 2 * kTileBytes;      // TG x (K tile, V tile)
  static constexpr int q_bytes(int rb) { return rb * 16 * D * 2; }   // queries are always bf16
  static constexpr int stat_bytes(int rb) { return 2 * TG * rb * 16 * 4; }
  static constexpr int xbuf_bytes(int rb) { return rb * TG * (D / 16) * 1024; }   // merge staging
  static constexpr int ring_bytes(int rb) {
    return NST * kSuperBytes > xbuf_bytes(rb) ? NST * kSuperBytes : xbuf_bytes(rb);
  }
  static constexpr int total(int rb) { return q_bytes(rb) + stat_bytes(rb) + ring_bytes(rb); }
};

//
// fp8 cache (KV8): K and V rows are E4M3 codes, one byte per element, with one fp32 multiplier per
// (batch element, KV head); queries, probabilities and the MFMA operands stay bf16.  A code becomes
// a bf16 value exactly (4 significant bits), two per v_cvt_scalef32_pk_bf16_fp8, after the LDS read;
// the K multiplier joins the softmax scale and the V multiplier the slice's output.  Two layout
// changes keep the LDS reads at one instruction per operand: K operand row m of 16-token block tb
// is tile row 8*(m/4) + 4*tb + m%4, so the 8 probabilities a lane holds belong to 8 consecutive
// tokens 8g..8g+7, and ds_read_b64_tr_b8 (lane i of a 16-lane group addresses 8 bytes of row i/2,
// lane j receives column j of the 8 rows) then fetches exactly those 8 tokens of V^T in one read.
template <int D, bool KV8, bool LONG32>
__device__ __forceinline__ int tile_swizzle(int r) {
  // 16-bit rows: the K reads of 16 lanes touch 16 consecutive rows, one piece each; the V reads of 32 lanes eight
  // consecutive rows, two neighbouring pieces each, so it is the piece's upper bits that must differ from row to row
  // (the 16 lanes of a K read are not consecutive: with the pieces g * KS + ks of four lane groups, r itself as the swizzle
  // doubled the K reads' time too; 47 % of the LDS cycles of a 33K call of 91 rows were conflicts, now none: 25.25 ->
  // 24.85 us a call, 4 x 8 heads x 37K 107.5 -> 106.9)
  if constexpr (!KV8 && D == 128) return ((r & 7) << 1) | ((r >> 3) & 1);
  // (64 channels, two rows in 256 bytes.  The 32-token tiles of long slices keep the pair's number: 48 % of their LDS cycles
  // are conflicts, but the waves of four row blocks hide them, and without a conflict the same loop is slower, from the
  // last-level cache 2 x 8 heads x 20K, 72 rows 25.0 us a call against 23.8, 104 rows 28.5 and 27.4; from HBM the same.)
  else if constexpr (!KV8 && LONG32) return lds_row_swizzle<D>(r);
  else if constexpr (!KV8) return (((r >> 1) & 3) << 1) | ((r >> 3) & 1);
  // 128-byte rows: the K reads of 16 lanes touch rows {0-3, 8-11, 16-19, 24-27} (+4), the V reads of
  // 32 lanes 16 consecutive rows; both must spread over the 16 16-byte slots of 256 bytes
  else if constexpr (D == 128) return ((r >> 1) ^ ((r >> 3) & 2)) & 7;
  else return ((r >> 2) + (r >> 4)) & 3;               // 64-byte rows
}

// four E4M3 codes of one dword -> bf16, exact
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2_t;
typedef __attribute__((ext_vector_type(2))) int i32x2_t;
typedef __attribute__((ext_vector_type(4))) int i32x4_t;
__device__ __forceinline__ bf16x8 e4m3x8_to_bf16(int lo, int hi) {
  const bf16x2_t a = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 1.0f, false);
  const bf16x2_t b = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 1.0f, true);
  const bf16x2_t c = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 1.0f, false);
  const bf16x2_t d = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 1.0f, true);
  return __builtin_shufflevector(__builtin_shufflevector(a, b, 0, 1, 2, 3),
                                 __builtin_shufflevector(c, d, 0, 1, 2, 3), 0, 1, 2, 3, 4, 5, 6, 7);
}

// TT = tokens per tile (16 or 32), NST = ring stages (super-tiles resident in LDS)
// MODE: 0 = contiguous cache, 1 = contiguous cache with appended-row fusion, 2 = paged cache
// ONE = the slice is the whole cache: the block writes its rows' output
template <int D, int RB, int TG, int TT, int NST, int MODE, bool KV8 = false, bool NT = false, bool ROT = false,
          bool ONE = false>
__global__ __launch_bounds__(RB * TG * 64) void attn_partial_grid(AttnParams p) {
  constexpr bool APPEND = MODE == 1, PAGED = MODE == 2;
  constexpr bool LONG32 = ROT && TT == 32;
  constexpr bool SCALED = RB > 4;                      // more than 64 rows in one block: see its stores
  constexpr int ES = KV8 ? 1 : 2;                      // bytes per cache element
  using SM = GridSmem<D, TG, TT, NST, ES>;
  constexpr int WAVES = RB * TG;
  constexpr int KS = D / 32;
  constexpr int DB = D / 16;
  constexpr int TB = TT / 16;                          // 16-token blocks per tile
  constexpr int ROWB = SM::kRowBytes;
  constexpr int CPR = ROWB / 16;                       // 16-byte chunks per cache row
  constexpr int RPI = 64 / CPR;
  constexpr int NLD = TT / RPI;                        // transfers per K (or V) tile
  constexpr int QROWB = D * 2, QCPR = D / 8, QRPI = 64 / QCPR;   // the bf16 query block's layout
  constexpr int NQ = RB * 16 / QRPI;                   // transfers for the query block
  static_assert(!KV8 || (MODE == 0 && TT == 32), "the fp8 cache path: contiguous caches, 32-token tiles");
  constexpr int XFERS = TG * 2 * NLD;                  // transfers per super-tile
  constexpr int ISS0 = WAVES >= 8 ? 8 : (WAVES >= 4 ? 4 : (WAVES >= 2 ? 2 : 1));   // power of two <= WAVES
  constexpr int ISSUERS = XFERS < ISS0 ? XFERS : ISS0;
  constexpr int PER = XFERS / ISSUERS;                 // transfers per issuing wave per super-tile
  static_assert(XFERS % ISSUERS == 0 && PER * (NST - 1) <= 63, "transfer split");
  static_assert(DB % TG == 0, "head-dim blocks must split over the token groups");
  static_assert(TT == 16 || TT == 32, "tile size");

  // verification is the critical path of a decoding round: its waves win the issue arbitration
  // against the draft call's waves that share a compute unit with them
  if (p.wave_prio) __builtin_amdgcn_s_setprio(2);
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* Qs = smem;
  float* stat_m = (float*)(smem + SM::q_bytes(RB));          // [TG][RB*16]
  float* stat_l = stat_m + TG * RB * 16;
  unsigned char* ring = smem + SM::q_bytes(RB) + SM::stat_bytes(RB);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rb = wave % RB, tg = wave / RB;
  const int j = lane & 15, g = lane >> 4;
  const int split = blockIdx.x, hk = blockIdx.y;
  // (the usual single row chunk needs no division: nothing that can be avoided stands in front of the
  // block's first transfer)
  const int b = p.n_chunks == 1 ? (int)blockIdx.z : (int)(blockIdx.z / p.n_chunks);
  const int chunk = p.n_chunks == 1 ? 0 : (int)(blockIdx.z % p.n_chunks);
  const int r0 = chunk * (RB * 16);
  const float inv_g = __builtin_amdgcn_rcpf((float)p.G);

  // fp8 cache: the K multiplier scales the logits, the V multiplier the slice's output.  Fetched
  // first, through the scalar cache (a vector load here would sit behind every K/V transfer in the
  // same counter, and waiting for it would wait for the whole ring).
  float k_mult = 1.f, v_mult = 1.f;
  if constexpr (KV8) {
    const int bh = __builtin_amdgcn_readfirstlane(b * p.Hkv + hk);
    k_mult = p.k_scale[bh];
    v_mult = p.v_scale[bh];
  }
  const unsigned ring_addr = (unsigned)(uintptr_t)ring;
  const unsigned q_addr = (unsigned)(uintptr_t)Qs;
  // paged: the pools' base plus the head offset; the page and the row inside it are added per transfer
  const char* kbase = (const char*)p.k + ((PAGED ? 0ll : (long long)b * p.sb) + (long long)hk * p.sh) * ES;
  const char* vbase = (const char*)p.v + ((PAGED ? 0ll : (long long)b * p.sb) + (long long)hk * p.sh) * ES;
  const unsigned row_bytes = (unsigned)(p.sn * ES);        // the host caps the row stride at 2^24 elements
  const int ld_row = lane / CPR, ld_pc = lane % CPR;

  // the tiles are dealt to the S slices as evenly as possible, the first n_tiles % S slices taking
  // one more (32-bit arithmetic: this runs before the first transfer can be issued)
  const int tq = p.tiles_q, tr = p.tiles_r;   // n_tiles / S and n_tiles % S for this kernel's tile size, from the host
  const int t_lo = split * tq + min(split, tr);
  const int t_hi = t_lo + tq + (split < tr ? 1 : 0);
  const int n_blk = t_hi - t_lo;                           // tiles of this block
  const int n_super = (n_blk + TG - 1) / TG;
  // ROT (long slices): the softmax state does not care in which order a slice's tiles arrive, so every
  // (batch element, KV head) starts its slices at a different phase and wraps around.  Blocks that
  // would otherwise walk their slices in lockstep, a fixed stride apart, then spread over the memory
  // channels (4 sequences x 8 KV heads x 37K rows in 8 slices: 10 % faster).  The phase is this head's
  // share of the slice, in single precision: any value in range serves, and an integer division here
  // would sit in front of the block's first transfer.
  int phase = 0;
  if constexpr (ROT)
    phase = __builtin_amdgcn_readfirstlane(   // wave-uniform: keep it in a scalar register
        min((int)((float)(b * p.Hkv + hk) * (float)n_super * p.phase_per_head), max(n_super - 1, 0)));
  auto super_at = [&](int si) {
    if constexpr (!ROT) return si;
    const int x = si + phase;
    return x >= n_super ? x - n_super : x;
  };

  // issuing wave w moves transfers x = w*PER .. w*PER+PER-1 of a super-tile:
  //   x -> tile tt = x / (2 NLD), K or V = (x / NLD) & 1, 1 KB piece n = x % NLD
  // tiles past the block's range and rows past the cache's end re-read the block's last valid row
  // (a cache hit), so every super-tile costs every issuer exactly PER transfers
  const int row_cap = min(t_hi * TT, p.n_total) - 1;       // 32-bit row numbers: the host caps the cache length
  // paged: the page numbers of the rows this block streams, staged in LDS once (table entries
  // outside the pool are clamped into it, so a bad table cannot send a transfer out of bounds)
  int* page_s = (int*)(smem + SM::total(RB));
  const int page_mask = PAGED ? (1 << p.page_shift) - 1 : 0;
  const int slot_lo = PAGED ? (t_lo * TT) >> p.page_shift : 0;
  if (PAGED) {
    const int n_slots = n_blk > 0 ? (row_cap >> p.page_shift) - slot_lo + 1 : 0;
    for (int i = tid; i < n_slots && i < kMaxSlicePages; i += RB * TG * 64) {
      int pg = p.block_table[(long long)b * p.max_pages + slot_lo + i];
      pg = pg < 0 ? 0 : (pg >= p.n_pool_pages ? p.n_pool_pages - 1 : pg);
      page_s[i] = pg;
    }
    __syncthreads();
  }
  auto issue_rows = [&](int si, int tile0, auto select) {
    const unsigned dst = ring_addr + (si % NST) * SM::kSuperBytes;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int x = wave * PER + u;
      const int tt = x / (2 * NLD), which = (x / NLD) & 1, n = x % NLD;
      const int r = n * RPI + ld_row;
      const int row = min((tile0 + tt) * TT + r, row_cap);
      const char* src = (which ? vbase : kbase) + (unsigned long long)(unsigned)row * row_bytes;   // one 32 x 32 -> 64 multiply-add
      if (PAGED)
        src = (which ? vbase : kbase) + ((long long)page_s[(row >> p.page_shift) - slot_lo] * p.page_stride +
                                         (long long)(row & page_mask) * p.sn) * 2;
      if (decltype(select)::value && row >= p.ctx_len)     // a row that has not reached the cache yet
        src = (const char*)(which ? p.v_new : p.k_new) +
              ((((long long)b * p.q_len + (row - p.ctx_len)) * p.Hkv + hk) * D) * 2;
      dma16<NT>(src + ((ld_pc ^ tile_swizzle<D, KV8, LONG32>(r)) * 16), dst + (tt * 2 + which) * SM::kTileBytes + n * 1024);
    }
  };
  // (only the last tiles hold appended rows: the source select, formed for every lane of every transfer, stood in front of
  // the first bytes of every slice; 16K x 4 heads, 42 rows 13.55 -> 13.3 us a call)
  auto issue_super = [&](int si) {
    const int tile0 = t_lo + super_at(si) * TG;
    if (APPEND && (tile0 + TG) * TT > p.ctx_len) issue_rows(si, tile0, std::true_type());
    else issue_rows(si, tile0, std::false_type());
  };
  // ---- prologue: the first ring stage goes out before anything else (its bytes are the ones
  // the first products wait for), then the query block, then the remaining stages.  Transfers
  // complete in issue order, so the wait for super-tile 0 below also covers the query block. ----
  const bool issuer = wave < ISSUERS;
  int issued = n_super < NST ? n_super : NST;              // super-tiles requested so far
  // Appended rows: the block that copies them into the cache fetches them now, ahead of every transfer
  // (loads return in order, so the transfer counts waited for below are not disturbed), and stores them
  // after its slice: the copy's trip to memory hides behind the stream instead of following it.
  const bool appends = APPEND && split == 0 && chunk == 0;
  constexpr int APR = D / 8;                               // 16-byte pieces per bf16 row
  const bool append_early = appends && p.q_len * APR <= WAVES * 64;
  u32x4 app_k = {0u, 0u, 0u, 0u}, app_v = {0u, 0u, 0u, 0u};
  if (APPEND && append_early && (int)threadIdx.x < p.q_len * APR) {
    const long long src = (((long long)b * p.q_len + threadIdx.x / APR) * p.Hkv + hk) * D + (threadIdx.x % APR) * 8;
    app_k = *(const u32x4*)((const uint16_t*)p.k_new + src);
    app_v = *(const u32x4*)((const uint16_t*)p.v_new + src);
  }
  if (issuer && issued > 0) issue_super(0);
#pragma unroll
  for (int n = 0; n < NQ; ++n) {
    if ((n % WAVES) == wave) {
      const int rr = n * QRPI + lane / QCPR;
      int r = r0 + rr;
      r = r < p.R ? r : p.R - 1;                          // padding rows repeat the last real row
      const int i = row_div_group(r, inv_g), gq = r - i * p.G;
      const char* src = (const char*)p.q + ((((long long)b * p.q_len + i) * p.H + hk * p.G + gq) * D) * 2 +
                        (((lane % QCPR) ^ tile_swizzle<D, false, LONG32>(rr)) * 16);
      dma16(src, q_addr + n * 1024);
    }
  }
  if (issuer)
    for (int si = 1; si < issued; ++si) issue_super(si);

  const int row = r0 + rb * 16 + j;                       // this lane's query row
  const int lim = (row < p.R) ? p.ctx_len + row_div_group(row, inv_g) : 0x7fffffff;
  float m_run = -INFINITY, l_run = 0.f;
  f32x4 acc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) acc[db] = (f32x4){0.f, 0.f, 0.f, 0.f};

  // bf16 cache: k_off[ks] is the lane's 16-byte K operand of contraction step ks in row j (the
  // query block uses the same offsets).  fp8 cache: a lane's KS*8 bytes of a row are NKC 16-byte
  // chunks, and k_off[tb * NKC + c] is chunk c in the permuted row of 16-token block tb.
  constexpr int NKC = KS / 2;
  constexpr int NKOFF = KV8 ? TB * NKC : KS;
  unsigned k_off[NKOFF];
  unsigned v_off[DB];
  if constexpr (!KV8) {
    const int swz_k = tile_swizzle<D, false, LONG32>(j);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) k_off[ks] = j * ROWB + (((g * KS + ks) ^ swz_k) * 16);
    const int v_row = 4 * g + (j >> 2);
    const int swz_v = tile_swizzle<D, false, LONG32>(v_row);
#pragma unroll
    for (int db = 0; db < DB; ++db)
      v_off[db] = v_row * ROWB + (((2 * db + ((j & 3) >> 1)) ^ swz_v) * 16) + (j & 1) * 8;
  } else {
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
      const int k_row = 8 * (j >> 2) + 4 * tb + (j & 3);
#pragma unroll
      for (int c = 0; c < NKC; ++c)
        k_off[tb * NKC + c] = k_row * ROWB + (((g * NKC + c) ^ tile_swizzle<D, true, LONG32>(k_row)) * 16);
    }
    const int v_row = 8 * g + (j >> 1);
#pragma unroll
    for (int db = 0; db < DB; ++db)
      v_off[db] = v_row * ROWB + ((db ^ tile_swizzle<D, true, LONG32>(v_row)) * 16) + (j & 1) * 8;
  }
  // keep the swizzled lane offsets in registers: left to itself the compiler recomputes them from
  // (j, g) for every tile, which costs more vector instructions than the tile's arithmetic
#pragma unroll
  for (int i = 0; i < NKOFF; ++i) asm volatile("" : "+v"(k_off[i]));
#pragma unroll
  for (int db = 0; db < DB; ++db) asm volatile("" : "+v"(v_off[db]));
  const float scale_log2 = KV8 ? p.scale_log2 * k_mult : p.scale_log2;

  bf16x8 qop[KS];

  for (int si = 0; si < n_super; ++si) {
    // Transfers complete in issue order, so "at most PER * (super-tiles requested after si)
    // outstanding" means super-tile si (and Q) has landed.  Waves that issue no tile transfers
    // only ever have their share of Q in flight.
    if (issuer) WaitLadder<NST - 1>::template run<PER>(issued - 1 - si); else wait_vmcnt<0>();
    __syncthreads();           // super-tile si complete in LDS; everyone is past super-tile si-1
    if (si == 0) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        qop[ks] = *(const bf16x8*)(Qs + rb * 16 * QROWB + j * QROWB +
                                   (((g * KS + ks) ^ tile_swizzle<D, false, LONG32>(j)) * 16));
    }
    if (si > 0 && issued < n_super) {                      // refill the stage just vacated
      if (issuer) issue_super(issued);
      ++issued;
    }
    const int ti = super_at(si) * TG + tg;                 // this wave's tile inside the block
    if (ti >= n_blk) continue;                             // ragged last super-tile

    const unsigned char* Kt = ring + (si % NST) * SM::kSuperBytes + tg * 2 * SM::kTileBytes;
    const unsigned char* Vt = Kt + SM::kTileBytes;
    const int n0 = (t_lo + ti) * TT;

    f32x4 s[TB];
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) s[tb] = (f32x4){0.f, 0.f, 0.f, 0.f};
    if constexpr (!KV8) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) {
          const bf16x8 kop = *(const bf16x8*)(Kt + tb * 16 * ROWB + k_off[ks]);
          s[tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kop, qop[ks], s[tb], 0, 0, 0);
        }
    } else {
#pragma unroll
      for (int c = 0; c < NKC; ++c)
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) {
          const i32x4_t kraw = *(const i32x4_t*)(Kt + k_off[tb * NKC + c]);
          s[tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(e4m3x8_to_bf16(kraw[0], kraw[1]), qop[2 * c], s[tb], 0, 0, 0);
          s[tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(e4m3x8_to_bf16(kraw[2], kraw[3]), qop[2 * c + 1], s[tb], 0, 0, 0);
        }
    }

    if ((n0 + TT - 1) > p.ctx_len) {                     // tile touches the causal edge
#pragma unroll
      for (int tb = 0; tb < TB; ++tb)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if ((n0 + (KV8 ? 8 * g + 4 * tb : tb * 16 + 4 * g) + e) > lim) s[tb][e] = -INFINITY;
    }
    float sv[TB * 4];
#pragma unroll
    for (int e = 0; e < TB * 4; ++e) sv[e] = s[e >> 2][e & 3];
    const float m8 = rows4_max(max_nan_of(sv));
    const float mx = m8 * scale_log2;                      // scale > 0: max commutes with it
    // lazy rescale: the reference m_run moves only when the tile maximum exceeds it by more than
    // kRescaleGap, so probabilities stay below 2^kRescaleGap and rescales are rare
    // (long slices of 16-token tiles take the second tile's maximum too, as 32-token tiles take that of 32 tokens: the further
    // the slice's largest probabilities lie above the reference, the larger their rounding, 0.4 % of the output's error)
    const float gap = ROT && TT == 16 && si == 1 ? 0.f : kRescaleGap;
    const bool up = mx > m_run + gap;                      // also true for the first finite maximum
    if (__any(up)) {
      const float a = up ? fast_exp2(m_run - mx) : 1.f;    // m_run = -inf -> 0
      if (up) m_run = mx;
      l_run *= a;
#pragma unroll
      for (int db = 0; db < DB; ++db) acc[db] *= a;
    }
    const float neg_m = (m_run == -INFINITY) ? 0.f : -m_run;
    // the PV product sees P rounded to bf16; the denominator sums the same rounded values.  Two
    // probabilities are rounded by one packed conversion and read back with a shift and a mask.
    unsigned pk[TB * 2];
    float psum = 0.f;
#pragma unroll
    for (int h = 0; h < TB * 2; ++h) {
      typedef __attribute__((ext_vector_type(2))) float f32x2_t;
      const f32x2_t x = {fast_exp2(fmaf(s[h >> 1][(2 * h) & 3], scale_log2, neg_m)),
                         fast_exp2(fmaf(s[h >> 1][(2 * h + 1) & 3], scale_log2, neg_m))};
      pk[h] = __builtin_bit_cast(unsigned, __builtin_convertvector(x, bf16x2_t));
      psum += __uint_as_float(pk[h] << 16) + __uint_as_float(pk[h] & 0xffff0000u);
    }
    l_run += psum;                                         // per-lane share; groups g meet at the end

    if (TB == 2) {
      const bf16x8 pop = __builtin_bit_cast(bf16x8, (i32x4_t){(int)pk[0], (int)pk[1], (int)pk[2 % (TB * 2)], (int)pk[3 % (TB * 2)]});
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        if constexpr (KV8) {
          const i32x2_t vraw = __builtin_amdgcn_ds_read_tr8_b64_v2i32(
              (__attribute__((address_space(3))) i32x2_t*)(Vt + v_off[db]));
          acc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(e4m3x8_to_bf16(vraw[0], vraw[1]), pop, acc[db], 0, 0, 0);
        } else {
          const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (__attribute__((address_space(3))) s16x4*)(Vt + v_off[db]));
          const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (__attribute__((address_space(3))) s16x4*)(Vt + (TB - 1) * 16 * ROWB + v_off[db]));
          const bf16x8 vop = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
          acc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vop, pop, acc[db], 0, 0, 0);
        }
      }
    } else {
      const s16x4 pop = __builtin_bit_cast(s16x4, (i32x2_t){(int)pk[0], (int)pk[1]});
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const s16x4 vop = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (__attribute__((address_space(3))) s16x4*)(Vt + v_off[db]));
        acc[db] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vop, pop, acc[db], 0, 0, 0);
      }
    }
  }
  wait_vmcnt<0>();   // no transfer may still be writing LDS past this point

  // ---- merge the TG token groups of every row block ----
  l_run = rows4_sum(l_run);
  if (g == 0) {
    stat_m[tg * RB * 16 + rb * 16 + j] = m_run;
    stat_l[tg * RB * 16 + rb * 16 + j] = l_run;
  }
  f32x4* xbuf = (f32x4*)ring;                              // [WAVES][DB][64 lanes]
  __syncthreads();   // (a) every wave is done reading the ring before anyone overwrites it
  // a wave finishes head-dim blocks tg, tg + TG, ...: those stay in its registers, only the blocks
  // that other waves finish go through LDS.  The body is instantiated once per value of tg (it is
  // wave-uniform), so which blocks stay and which travel is known at compile time: straight-line
  // code whose LDS reads all go out before the first one is needed.
  const long long slot = ((long long)b * p.Hkv + hk) * p.S + split;
  auto finish = [&](auto tgc) {
    constexpr int TGC = decltype(tgc)::value;
#pragma unroll
    for (int db = 0; db < DB; ++db)
      if (db % TG != TGC) xbuf[(wave * DB + db) * 64 + lane] = acc[db];
    __syncthreads();   // (b) accumulators and statistics of all waves visible
    f32x4 other[TG][DB / TG];                                // [source wave group][own head-dim block]
#pragma unroll
    for (int w = 0; w < TG; ++w)
#pragma unroll
      for (int dd = 0; dd < DB / TG; ++dd)
        if (w != TGC) other[w][dd] = xbuf[((w * RB + rb) * DB + TGC + TG * dd) * 64 + lane];
    float mw[TG], mm = -INFINITY;
#pragma unroll
    for (int w = 0; w < TG; ++w) { mw[w] = stat_m[w * RB * 16 + rb * 16 + j]; mm = max_nan(mm, mw[w]); }
    float f[TG], ll = 0.f;
#pragma unroll
    for (int w = 0; w < TG; ++w) {
      f[w] = (mw[w] == -INFINITY) ? 0.f : fast_exp2(mw[w] - mm);
      ll = fmaf(f[w], stat_l[w * RB * 16 + rb * 16 + j], ll);
    }
    if constexpr (KV8) {
#pragma unroll
      for (int w = 0; w < TG; ++w) f[w] *= v_mult;         // after the denominator took the plain weights
    }
    long long lse_at = 0;
    uint16_t* o_row = (uint16_t*)p.part_o + (slot * p.R + row) * D;
    if constexpr (ONE) {
      o_row = (uint16_t*)p.out + out_row(p, b, hk, row, inv_g, &lse_at) * D;
      const float inv = 1.f / ll;
#pragma unroll
      for (int w = 0; w < TG; ++w) f[w] *= inv;
    }
    // A wide block's outputs leave as scaled fp16, as many bytes: its slices are half as long as those of two row chunks, and
    // twice as many rounded to bf16 were further from 64 bits (33K x 4 heads, 91 rows 2.71e-3 -> 2.74e-3; like this 2.17e-3).
    // One power of two for the wave's channels of a row, from the largest finite one.  Channels that lie 31 powers of two and
    // more below it would keep fewer bits than in bf16, then none: such a row's leave as bf16, with a factor of -1 that says so.
    float up = 1.f;
    bool scaled = true;
    if constexpr (SCALED) {
      float big = 0.f;
#pragma unroll
      for (int dd = 0; dd < DB / TG; ++dd) {
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < TG; ++w) {
          if (w == TGC) o += acc[TGC + TG * dd] * f[w];
          else o += other[w][dd] * f[w];
        }
        acc[TGC + TG * dd] = o;
#pragma unroll
        for (int e = 0; e < 4; ++e) big = fabsf(o[e]) < INFINITY ? fmaxf(big, fabsf(o[e])) : big;
      }
      const int power = max(__builtin_amdgcn_frexp_expf(rows4_max(big)), -100) - 14;
      up = ldexpf(1.f, -power);
      bool spread = false;
#pragma unroll
      for (int dd = 0; dd < DB / TG; ++dd)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float o = acc[TGC + TG * dd][e];
          spread |= o != 0.f && fabsf(o * up) < 0x1p-17f;
        }
      scaled = rows4_max(spread ? 1.f : 0.f) == 0.f;       // the same in all four lanes of the row
      if (g == 0 && row < p.R) p.part_e[(slot * p.R + row) * TG + TGC] = scaled ? ldexpf(1.f, power) : -1.f;
    }
#pragma unroll
    for (int dd = 0; dd < DB / TG; ++dd) {
      const int db = TGC + TG * dd;
      f32x4 o = {0.f, 0.f, 0.f, 0.f};
      if constexpr (SCALED) {
        o = acc[TGC + TG * dd];
      } else {
#pragma unroll
        for (int w = 0; w < TG; ++w) {
          if (w == TGC) o += acc[TGC + TG * dd] * f[w];
          else o += other[w][dd] * f[w];
        }
      }
      // the slice's output leaves as bf16 (the merge weighs and sums it in fp32): half the bytes to write
      // here and to fetch in the merge, and the rounding is one more of the size the output's own has
      if (row < p.R) {
        typedef __attribute__((ext_vector_type(2))) float f32x2_t;
        const f32x2_t lo = {o[0], o[1]}, hi = {o[2], o[3]};
        uint2 w;
        if (SCALED && scaled) {
          w.x = __builtin_bit_cast(unsigned, __builtin_convertvector(lo * up, f16x2_t));
          w.y = __builtin_bit_cast(unsigned, __builtin_convertvector(hi * up, f16x2_t));
        } else {
          w.x = __builtin_bit_cast(unsigned, __builtin_convertvector(lo, bf16x2_t));
          w.y = __builtin_bit_cast(unsigned, __builtin_convertvector(hi, bf16x2_t));
        }
        *(uint2*)(o_row + db * 16 + 4 * g) = w;
      }
    }
    if (TGC == 0 && g == 0 && row < p.R) {
      if constexpr (ONE) {
        if (p.lse != nullptr) p.lse[lse_at] = (mm + __log2f(ll)) * kLn2;
      } else {
        p.part_m[slot * p.R + row] = mm;
        p.part_l[slot * p.R + row] = ll;
      }
    }
  };
  static_assert(TG == 1 || TG == 2 || TG == 4, "token groups");
  if (tg == 0) finish(std::integral_constant<int, 0>());
  else if (tg == 1) finish(std::integral_constant<int, 1>());
  else if (tg == 2) finish(std::integral_constant<int, 2 % TG>());
  else finish(std::integral_constant<int, 3 % TG>());
  if (APPEND && appends) {
    if (append_early) {
      if ((int)threadIdx.x < p.q_len * APR) {
        const long long dst = (long long)b * p.sb + (long long)hk * p.sh +
                              (long long)(p.ctx_len + threadIdx.x / APR) * p.sn + (threadIdx.x % APR) * 8;
        *(u32x4*)((uint16_t*)p.k_w + dst) = app_k;
        *(u32x4*)((uint16_t*)p.v_w + dst) = app_v;
      }
    } else {
      append_new_rows<uint16_t, D>(p, b, hk);
    }
  }
}

// =================================================================================================
// fp32 partial kernel (v_mfma_f32_16x16x4_f32: fp32 operands, products and sums)
// =================================================================================================
// Bound by the matrix unit's fp32 rate (1/16 of its bf16 rate) and HBM about equally: 4 * 16 * RB * D flops
// against 8 * D bytes per token.  The vector-ALU kernel that it replaces spent one LDS read and four shared
// multiply-adds per pair of operands, and streamed the cache once per 32 query rows.  A verification call, us: 8K x
// 4 heads x 128, 42 rows, a draft call beside it 88 -> 28; two sequences x 4K x 8 heads, 80 rows 223 -> 53;
// 12.7K x 8 heads, 104 rows 413 -> 74 (5.5 GFLOP: 74 TFLOP/s of a peak of 157); 64 channels, 70K x 2 heads, 49
// rows 154 -> 36.  Its error against 64 bits is 0.5 to 0.7 times the former kernel's (shorter serial sums).
// The same frame as attn_partial_grid: grid (S, H_kv, B * n_chunks), wave (rb, tg) owns 16 query rows and every
// TG-th 16-token tile, tiles go HBM -> LDS by direct transfers into a ring of NST super-tiles, one barrier per
// super-tile.  Operands (lane = j + 16g): A row j, contraction slot g; B column j, slot g; result column j, rows
// 4g..4g+3.  Which element rides in which slot is free as long as both operands agree:
//   S^T = K Q^T   step (s, c): slot g is channel 16s + 4g + c, so a lane's four steps are one 16-byte read.
//   O^T = V^T P^T step e: slot g is token 4g + e, the score register e as it stands; result row r of block (h, c)
//                 is channel 64h + 4r + c, so 16 bytes of a V row give a lane its operands of four blocks, and the
//                 four blocks of h leave it with 16 consecutive channels.
// Rows of K and V are stored unpadded, 16-byte piece p of tile row r at p ^ r: the 16 lanes of a K read (16 rows, one
// piece each) and of a V read (one row, 16 pieces) then spread over all banks.
template <int D, int TG, int NST>
struct F32Smem {
  static constexpr int kTileBytes = 16 * D * 4;
  static constexpr int kSuperBytes = TG * 2 * kTileBytes;
  static constexpr int stat_bytes(int rb) { return 2 * TG * rb * 16 * 4; }
  static constexpr int q_bytes(int rb) { return rb * 16 * D * 4; }
  static constexpr int xbuf_bytes(int rb) { return rb * TG * (D / 16) * 1024; }
  // [statistics | queries | ring]; the merge staging overlays queries and ring
  static constexpr int total(int rb) {
    const int stream = q_bytes(rb) + NST * kSuperBytes;
    return stat_bytes(rb) + (stream > xbuf_bytes(rb) ? stream : xbuf_bytes(rb));
  }
};

template <int D, int RB, int TG, int NST, int MODE, bool ONE = false>
__global__ __launch_bounds__(RB * TG * 64) void attn_partial_f32(AttnParams p) {
  constexpr bool APPEND = MODE == 1, PAGED = MODE == 2;
  using SM = F32Smem<D, TG, NST>;
  constexpr int WAVES = RB * TG;
  constexpr int CPR = D / 4;                           // 16-byte pieces per row
  constexpr int RPI = 64 / CPR;                        // rows per transfer
  constexpr int NLD = 16 / RPI;                        // transfers per K (or V) tile
  constexpr int NS = D / 16;                           // 16-channel steps of S^T
  constexpr int NH = D / 64;                           // 64-channel groups of O^T
  constexpr int XFERS = TG * 2 * NLD;
  constexpr int ISSUERS = WAVES >= 8 ? 8 : 4;
  constexpr int PER = XFERS / ISSUERS;
  static_assert(WAVES >= 4 && XFERS % ISSUERS == 0 && PER * (NST - 1) <= 63, "transfer split");

  if (p.wave_prio) __builtin_amdgcn_s_setprio(2);
  extern __shared__ __align__(16) unsigned char smem[];
  float* stat_m = (float*)smem;                        // [TG][RB*16]
  float* stat_l = stat_m + TG * RB * 16;
  unsigned char* Qs = smem + SM::stat_bytes(RB);
  unsigned char* ring = Qs + SM::q_bytes(RB);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rb = wave % RB, tg = wave / RB;
  const int j = lane & 15, g = lane >> 4;
  const int split = blockIdx.x, hk = blockIdx.y;
  const int b = p.n_chunks == 1 ? (int)blockIdx.z : (int)(blockIdx.z / p.n_chunks);
  const int chunk = p.n_chunks == 1 ? 0 : (int)(blockIdx.z % p.n_chunks);
  const float inv_g = __builtin_amdgcn_rcpf((float)p.G);
  const unsigned ring_addr = (unsigned)(uintptr_t)ring;
  const unsigned q_addr = (unsigned)(uintptr_t)Qs;
  const char* kbase = (const char*)p.k + ((PAGED ? 0ll : (long long)b * p.sb) + (long long)hk * p.sh) * 4;
  const char* vbase = (const char*)p.v + ((PAGED ? 0ll : (long long)b * p.sb) + (long long)hk * p.sh) * 4;
  const unsigned row_bytes = (unsigned)(p.sn * 4);     // the host caps the row stride at 2^24 elements
  const int ld_row = lane / CPR, ld_pc = lane % CPR;

  const int tq = p.tiles_q, tr = p.tiles_r;
  const int t_lo = split * tq + min(split, tr);
  const int t_hi = t_lo + tq + (split < tr ? 1 : 0);
  const int n_blk = t_hi - t_lo;
  const int n_super = (n_blk + TG - 1) / TG;
  const int row_cap = min(t_hi * 16, p.n_total) - 1;
  int* page_s = (int*)(smem + SM::total(RB));
  const int page_mask = PAGED ? (1 << p.page_shift) - 1 : 0;
  const int slot_lo = PAGED ? (t_lo * 16) >> p.page_shift : 0;
  if (PAGED) {
    const int n_slots = n_blk > 0 ? (row_cap >> p.page_shift) - slot_lo + 1 : 0;
    for (int i = tid; i < n_slots && i < kMaxSlicePages; i += WAVES * 64) {
      int pg = p.block_table[(long long)b * p.max_pages + slot_lo + i];
      pg = pg < 0 ? 0 : (pg >= p.n_pool_pages ? p.n_pool_pages - 1 : pg);
      page_s[i] = pg;
    }
    __syncthreads();
  }
  // as in attn_partial_grid: tiles past the block's range and rows past the cache's end re-read the last valid
  // row, so every super-tile costs every issuer exactly PER transfers
  auto issue_super = [&](int si) {
    const unsigned dst = ring_addr + (si % NST) * SM::kSuperBytes;
    const int tile0 = t_lo + si * TG;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int x = wave * PER + u;
      const int tt = x / (2 * NLD), which = (x / NLD) & 1, n = x % NLD;
      const int r = n * RPI + ld_row;
      const int row = min((tile0 + tt) * 16 + r, row_cap);
      const char* src = (which ? vbase : kbase) + (unsigned long long)(unsigned)row * row_bytes;
      if (PAGED)
        src = (which ? vbase : kbase) + ((long long)page_s[(row >> p.page_shift) - slot_lo] * p.page_stride +
                                         (long long)(row & page_mask) * p.sn) * 4;
      if (APPEND && row >= p.ctx_len)
        src = (const char*)(which ? p.v_new : p.k_new) +
              ((((long long)b * p.q_len + (row - p.ctx_len)) * p.Hkv + hk) * D) * 4;
      dma16(src + ((ld_pc ^ r) * 16), dst + (tt * 2 + which) * SM::kTileBytes + n * 1024);
    }
  };
  const bool issuer = wave < ISSUERS;
  // the first stage goes out first, then the queries (transfers complete in order: the wait for super-tile 0 covers
  // them), then the other stages
  int issued = n_super < NST ? n_super : NST;
  if (issuer && issued > 0) issue_super(0);
#pragma unroll
  for (int n = 0; n < RB * NLD; ++n) {
    if ((n % WAVES) == wave) {
      const int rr = n * RPI + ld_row;
      const int r = min(chunk * (RB * 16) + rr, p.R - 1);   // padding rows repeat the last real row
      const int i = row_div_group(r, inv_g), gq = r - i * p.G;
      const char* src = (const char*)p.q + ((((long long)b * p.q_len + i) * p.H + hk * p.G + gq) * D) * 4 +
                        ((ld_pc ^ (rr & 15)) * 16);
      dma16(src, q_addr + n * 1024);
    }
  }
  if (issuer)
    for (int si = 1; si < issued; ++si) issue_super(si);

  const int row = chunk * (RB * 16) + rb * 16 + j;     // this lane's query row
  const int lim = row < p.R ? p.ctx_len + row_div_group(row, inv_g) : 0x7fffffff;
  float m_run = -INFINITY, l_run = 0.f;
  f32x4 qop[NS];
  f32x4 acc[NH][4];
#pragma unroll
  for (int h = 0; h < NH; ++h)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[h][c] = (f32x4){0.f, 0.f, 0.f, 0.f};

  for (int si = 0; si < n_super; ++si) {
    if (issuer) WaitLadder<NST - 1>::template run<PER>(issued - 1 - si); else wait_vmcnt<0>();
    __syncthreads();
    if (si > 0 && issued < n_super) {                  // refill the stage just vacated
      if (issuer) issue_super(issued);
      ++issued;
    }
    if (si == 0) {
#pragma unroll
      for (int s = 0; s < NS; ++s)
        qop[s] = *(const f32x4*)(Qs + (rb * 16 + j) * (D * 4) + (((4 * s + g) ^ j) * 16));
    }
    const int ti = si * TG + tg;
    if (ti >= n_blk) continue;                         // ragged last super-tile
    const unsigned char* Kt = ring + (si % NST) * SM::kSuperBytes + tg * 2 * SM::kTileBytes;
    unsigned char* Vt = ring + (si % NST) * SM::kSuperBytes + tg * 2 * SM::kTileBytes + SM::kTileBytes;
    const int n0 = (t_lo + ti) * 16;
    // V rows past the cache's end repeat the last one, which may hold an infinity, and that times their weight of 0 is
    // a NaN: cleared, by each wave before its own reads (a wave's LDS operations complete in order, and all that share
    // the tile write the same).  In the cache's last tile only; a select at every operand cost the call 5 to 10 %.
    for (int r = row_cap - n0 + 1; r < 16; ++r)
      if (lane < CPR) *(f32x4*)(Vt + r * (D * 4) + lane * 16) = (f32x4){0.f, 0.f, 0.f, 0.f};

    f32x4 z[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};   // two chains, even and odd steps
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const f32x4 kop = *(const f32x4*)(Kt + j * (D * 4) + (((4 * s + g) ^ j) * 16));
#pragma unroll
      for (int c = 0; c < 4; ++c)
        z[c & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(kop[c], qop[s][c], z[c & 1], 0, 0, 0);
    }
    float sv[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) sv[e] = z[0][e] + z[1][e];
    if (n0 + 15 > p.ctx_len) {                         // tile touches the causal edge
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (n0 + 4 * g + e > lim) sv[e] = -INFINITY;
    }
    const float mx = rows4_max(max_nan_of(sv)) * p.scale_log2;
    const bool up = mx > m_run + kRescaleGap;          // lazy reference, as in attn_partial_grid
    if (__any(up)) {
      const float a = up ? fast_exp2(m_run - mx) : 1.f;
      if (up) m_run = mx;
      l_run *= a;
#pragma unroll
      for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[h][c] *= a;
    }
    const float neg_m = (m_run == -INFINITY) ? 0.f : -m_run;
    float pr[4];
    {
      // product and sum rounded one by one, as the reference's own product is: a fused sum would leave the product's
      // rounding error, beyond any exponent for logits of 1e9 and more
#pragma clang fp contract(off)
#pragma unroll
      for (int e = 0; e < 4; ++e) pr[e] = fast_exp2(sv[e] * p.scale_log2 + neg_m);
    }
    l_run += (pr[0] + pr[1]) + (pr[2] + pr[3]);        // per-lane share; groups g meet at the end
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int vr = 4 * g + e;
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        const f32x4 vop = *(const f32x4*)(Vt + vr * (D * 4) + (((16 * h + j) ^ vr) * 16));
#pragma unroll
        for (int c = 0; c < 4; ++c)
          acc[h][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(vop[c], pr[e], acc[h][c], 0, 0, 0);
      }
    }
  }
  wait_vmcnt<0>();   // no transfer may still be writing LDS past this point

  // ---- merge the TG token groups of every row block: group tg finishes vectors tg, tg + TG, ... of the lane's
  // 4 * NH output vectors (vector (h, e): channels 64h + 16g + 4e .. + 3) ----
  l_run = rows4_sum(l_run);
  if (g == 0) {
    stat_m[tg * RB * 16 + rb * 16 + j] = m_run;
    stat_l[tg * RB * 16 + rb * 16 + j] = l_run;
  }
  constexpr int NV = 4 * NH;
  f32x4* xbuf = (f32x4*)Qs;                            // [WAVES][NV][64 lanes]
  __syncthreads();   // every wave is done reading queries and ring
#pragma unroll
  for (int v = 0; v < NV; ++v)
    xbuf[(wave * NV + v) * 64 + lane] = (f32x4){acc[v / 4][0][v % 4], acc[v / 4][1][v % 4], acc[v / 4][2][v % 4],
                                                acc[v / 4][3][v % 4]};
  __syncthreads();
  float f[TG], mm = -INFINITY, ll = 0.f;
#pragma unroll
  for (int w = 0; w < TG; ++w) { f[w] = stat_m[w * RB * 16 + rb * 16 + j]; mm = max_nan(mm, f[w]); }
#pragma unroll
  for (int w = 0; w < TG; ++w) {
    f[w] = (f[w] == -INFINITY) ? 0.f : fast_exp2(f[w] - mm);
    ll = fmaf(f[w], stat_l[w * RB * 16 + rb * 16 + j], ll);
  }
  const long long slot = ((long long)b * p.Hkv + hk) * p.S + split;
  if (row < p.R) {
    float* o_row = (float*)p.part_o + (slot * p.R + row) * D + 16 * g;
    long long lse_at = 0;
    if constexpr (ONE) {
      o_row = (float*)p.out + out_row(p, b, hk, row, inv_g, &lse_at) * D + 16 * g;
      const float inv = 1.f / ll;
#pragma unroll
      for (int w = 0; w < TG; ++w) f[w] *= inv;
    }
#pragma unroll
    for (int vv = 0; vv < NV / TG; ++vv) {
      const int v = vv * TG + tg;
      f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < TG; ++w) o += xbuf[((w * RB + rb) * NV + v) * 64 + lane] * f[w];
      *(f32x4*)(o_row + 64 * (v / 4) + 4 * (v % 4)) = o;
    }
    if (tg == 0 && g == 0) {
      if constexpr (ONE) {
        if (p.lse != nullptr) p.lse[lse_at] = (mm + __log2f(ll)) * kLn2;
      } else {
        p.part_m[slot * p.R + row] = mm;
        p.part_l[slot * p.R + row] = ll;
      }
    }
  }
  if (APPEND && split == 0 && chunk == 0) append_new_rows<float, D>(p, b, hk);
}

// =================================================================================================
// Merge of the KV slices: out = sum_s 2^(m_s - m*) o_s / sum_s 2^(m_s - m*) l_s
// The slices' outputs o_s are fp32 (the fp32 kernel's), bf16 (the bf16 kernel's) or, of its blocks of more than 64 rows, fp16
// with a factor, or bf16 with -1 in its place.
// One block per (query row, KV head, batch element).  The slices are spread over the threads: first
// the S weights (one slice per thread, block-wide max and sum), then thread (sg, vec) accumulates
// 16-byte vector `vec` of the row over slices sg, sg + NSG, ... and the NSG groups meet in LDS.
// =================================================================================================
constexpr int kMaxSplits = 1024;

// four consecutive elements of a slice's output; for bf16 the raw bits travel in the first two components
// until the weights are known (the loads must all be in flight before anything waits for one of them)
enum PartOut { kPartF32, kPartBf16, kPartF16 };
constexpr int kWideGroups = 2;         // token groups of a block of more than 64 rows
template <int PO>
__device__ __forceinline__ f32x4 part_o_load4(const void* base, long long elem) {
  if constexpr (PO == kPartF32) return *(const f32x4*)((const float*)base + elem);
  else {
    const uint2 w = *(const uint2*)((const uint16_t*)base + elem);
    return (f32x4){__uint_as_float(w.x), __uint_as_float(w.y), 0.f, 0.f};
  }
}
// weight * the output; kPartF16: `factor` is what the kernel stored beside it
template <int PO>
__device__ __forceinline__ f32x4 part_o_weighed(f32x4 raw, float weight, float factor) {
  if constexpr (PO == kPartF32) return raw * weight;
  else {
    const unsigned x = __float_as_uint(raw[0]), y = __float_as_uint(raw[1]);
    f32x4 o = {__uint_as_float(x << 16), __uint_as_float(x & 0xffff0000u), __uint_as_float(y << 16), __uint_as_float(y & 0xffff0000u)};
    if constexpr (PO == kPartF16) {
      const f16x2_t lo = __builtin_bit_cast(f16x2_t, x), hi = __builtin_bit_cast(f16x2_t, y);
      if (factor > 0.f) {
        o = (f32x4){(float)lo[0], (float)lo[1], (float)hi[0], (float)hi[1]};
        weight *= factor;
      }
    }
    return o * weight;
  }
}

template <typename T, int D, int PO>
__global__ __launch_bounds__(256) void attn_combine(AttnParams p) {
  constexpr int VPR = D / 4;           // four-element vectors per row
  constexpr int NSG = 256 / VPR;       // slice groups
  __shared__ float w_s[kMaxSplits];
  __shared__ float red[8];
  __shared__ f32x4 acc_s[NSG][VPR];

  const int r = blockIdx.x, hk = blockIdx.y, b = blockIdx.z, tid = threadIdx.x;
  const long long slot0 = ((long long)b * p.Hkv + hk) * p.S;
  const int vec = tid % VPR, sg = tid / VPR;

  // the first PF slices of every group are fetched before the weights are known, so the whole
  // merge costs one trip to memory
  constexpr int PF = 8;
  f32x4 pre[PF];
#pragma unroll
  for (int u = 0; u < PF; ++u) {
    const int s = min(sg + u * NSG, p.S - 1);             // past the last slice: a harmless repeat, not used
    pre[u] = part_o_load4<PO>(p.part_o, ((slot0 + s) * p.R + r) * D + vec * 4);
  }
  // the factor of this thread's channels (16-channel blocks are dealt to the token groups in turn)
  auto factor_of = [&](int s) { return p.part_e[((slot0 + s) * p.R + r) * kWideGroups + vec / 4 % kWideGroups]; };
  float pre_e[PF] = {};
  if constexpr (PO == kPartF16)
#pragma unroll
    for (int u = 0; u < PF; ++u) pre_e[u] = factor_of(min(sg + u * NSG, p.S - 1));

  // where the row's output goes: worked out while the loads are in flight (the division would otherwise
  // stand between the last barrier and the store)
  const int i_row = r / p.G, h_row = hk * p.G + (r - i_row * p.G);
  long long out_at = (((long long)b * p.q_len + i_row) * p.H + h_row) * D + (tid % VPR) * 4;
  long long lse_at = ((long long)b * p.H + h_row) * p.q_len + i_row;
  asm volatile("" : "+v"(out_at), "+v"(lse_at));

  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  float mstar, den;
  if (p.S <= 64) {
    // up to 64 slices: every wave holds all slice statistics (one per lane), so the reference
    // maximum, the weights and the denominator need no LDS and no barrier; a weight reaches the
    // thread that needs it through a lane shuffle
    const int lane = tid & 63;
    const float ms = lane < p.S ? p.part_m[(slot0 + lane) * p.R + r] : -INFINITY;
    const float ls = lane < p.S ? p.part_l[(slot0 + lane) * p.R + r] : 0.f;
    mstar = wave_max(ms);
    const float w = (ms == -INFINITY) ? 0.f : fast_exp2(ms - mstar);
    den = wave_sum(w * ls);
#pragma unroll
    for (int u = 0; u < PF; ++u) {
      const int sl = sg + u * NSG;                        // < 64 whenever it is < S
      const float ws = __shfl(w, sl & 63, 64);
      if (sl < p.S) acc += part_o_weighed<PO>(pre[u], ws, pre_e[u]);
    }
  } else {
    // this thread's first slice statistics ride in the same trip
    const float m0 = tid < p.S ? p.part_m[(slot0 + tid) * p.R + r] : -INFINITY;
    const float l0 = tid < p.S ? p.part_l[(slot0 + tid) * p.R + r] : 0.f;
    float mloc = m0;
    for (int s2 = tid + 256; s2 < p.S; s2 += 256) mloc = max_nan(mloc, p.part_m[(slot0 + s2) * p.R + r]);
    mloc = wave_max(mloc);
    if ((tid & 63) == 0) red[tid >> 6] = mloc;
    __syncthreads();
    mstar = max_nan(max_nan(red[0], red[1]), max_nan(red[2], red[3]));
    float dloc = 0.f;
    if (tid < p.S) {
      const float w = (m0 == -INFINITY) ? 0.f : fast_exp2(m0 - mstar);
      w_s[tid] = w;
      dloc = w * l0;
    }
    for (int s2 = tid + 256; s2 < p.S; s2 += 256) {
      const float ms = p.part_m[(slot0 + s2) * p.R + r];
      const float w = (ms == -INFINITY) ? 0.f : fast_exp2(ms - mstar);
      w_s[s2] = w;
      dloc = fmaf(w, p.part_l[(slot0 + s2) * p.R + r], dloc);
    }
    dloc = wave_sum(dloc);
    if ((tid & 63) == 0) red[4 + (tid >> 6)] = dloc;
    __syncthreads();
    den = red[4] + red[5] + red[6] + red[7];
#pragma unroll
    for (int u = 0; u < PF; ++u) {
      const int sl = sg + u * NSG;
      if (sl < p.S) acc += part_o_weighed<PO>(pre[u], w_s[sl], pre_e[u]);
    }
#pragma unroll 4
    for (int sl = sg + PF * NSG; sl < p.S; sl += NSG) {
      acc += part_o_weighed<PO>(part_o_load4<PO>(p.part_o, ((slot0 + sl) * p.R + r) * D + vec * 4), w_s[sl],
                                PO == kPartF16 ? factor_of(sl) : 0.f);
    }
  }
  acc_s[sg][vec] = acc;
  __syncthreads();
  if (tid < VPR) {
    f32x4 t = acc_s[0][tid];
#pragma unroll
    for (int g2 = 1; g2 < NSG; ++g2) t += acc_s[g2][tid];
    const float inv = 1.f / den;
    T* o = (T*)p.out + out_at;
    if constexpr (sizeof(T) == 2) {                        // four bf16 values: one 8-byte store
      typedef __attribute__((ext_vector_type(2))) float f32x2_t;
      const f32x2_t lo = {t[0] * inv, t[1] * inv}, hi = {t[2] * inv, t[3] * inv};
      uint2 w;
      w.x = __builtin_bit_cast(unsigned, __builtin_convertvector(lo, bf16x2_t));
      w.y = __builtin_bit_cast(unsigned, __builtin_convertvector(hi, bf16x2_t));
      *(uint2*)o = w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) Elem<T>::store(o + e, t[e] * inv);
    }
    if (p.lse != nullptr && tid == 0) p.lse[lse_at] = (mstar + __log2f(den)) * kLn2;
  }
}

// =================================================================================================
// host launch
// =================================================================================================
// Lets KERNEL use `smem` bytes of dynamic LDS.  The attribute belongs to a (kernel, device) pair: it is set once for
// each device this process uses.
template <void (*KERNEL)(AttnParams)>
static hipError_t allow_dynamic_lds(int smem) {
  static std::atomic<unsigned long long> attr_set{0};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const unsigned long long bit = 1ull << (dev & 63);
  if (!(attr_set.load(std::memory_order_acquire) & bit)) {
    e = hipFuncSetAttribute((const void*)KERNEL, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    if (e != hipSuccess) return e;
    attr_set.fetch_or(bit, std::memory_order_release);
  }
  return hipSuccess;
}

template <int D, int RB, int TG, int TT, int NST, int MODE, bool KV8 = false, bool NT = false, bool ROT = false,
          bool ONE = false>
static hipError_t launch_grid_mode(const AttnParams& p, hipStream_t st) {
  // the paged variant keeps its slice of the page table behind the ring
  constexpr int smem = GridSmem<D, TG, TT, NST, KV8 ? 1 : 2>::total(RB) + (MODE == 2 ? kMaxSlicePages * 4 : 0);
  const hipError_t e = allow_dynamic_lds<attn_partial_grid<D, RB, TG, TT, NST, MODE, KV8, NT, ROT, ONE>>(smem);
  if (e != hipSuccess) return e;
  dim3 grid(p.S, p.Hkv, p.B * p.n_chunks);
  AttnParams q = p;                               // the slices' tile counts for this kernel's tile size
  const int n_tiles = (p.n_total + TT - 1) / TT;
  q.tiles_q = n_tiles / p.S;
  q.tiles_r = n_tiles % p.S;
  hipLaunchKernelGGL((attn_partial_grid<D, RB, TG, TT, NST, MODE, KV8, NT, ROT, ONE>), grid, dim3(RB * TG * 64), smem, st, q);
  return hipGetLastError();
}

// the appended-row and paged variants are separate instantiations, so the plain call carries none of
// their address selects
template <int D, int RB, int TG, int TT, int NST, bool NT = false, bool ROT = false, bool ONE = false>
static hipError_t launch_grid(const AttnParams& p, hipStream_t st) {
  if (p.block_table != nullptr) return launch_grid_mode<D, RB, TG, TT, NST, 2, false, NT, ROT, ONE>(p, st);
  if (p.k_new != nullptr) return launch_grid_mode<D, RB, TG, TT, NST, 1, false, NT, ROT, ONE>(p, st);
  return launch_grid_mode<D, RB, TG, TT, NST, 0, false, NT, ROT, ONE>(p, st);
}

// Up to 16 query rows and one slice of a short cache (the library's choice up to 256 rows, 128 in fp32): the block
// writes the output, and no merge is launched.  An instantiation of its own: as a branch of the others' epilogue it cost
// them up to 0.1 us.
static bool one_slice_call(const AttnParams& p) { return p.S == 1 && p.row_chunk == 16 && (p.n_total + 31) / 32 < 24; }

// A call whose K and V exceed the chip's last-level cache (256 MB) streams them with non-temporal
// transfers: nothing of such a stream can be served from a cache again, and left to itself it evicts
// the query block, the split partials and the other stream's data (measured on 4 sequences x 8 KV
// heads x 37K rows, 608 MB: 6 % faster; at 34 MB the hint costs 5 %, so short streams do not use it).
static bool stream_exceeds_caches(const AttnParams& p, int head_dim, int elem_bytes) {
  return 2ll * p.B * p.Hkv * p.n_total * head_dim * elem_bytes > (256ll << 20);
}

// Short slices (a block owns only a handful of tiles, as at 16K context on 256 compute units) use
// 16-token tiles and a deeper ring; long slices use 32-token tiles, which halve the barrier count.
template <int D, int RB>
static hipError_t launch_grid_rb(const AttnParams& p, hipStream_t st) {
  const int tiles32_per_block = ((p.n_total + 31) / 32) / (p.S > 0 ? p.S : 1);
  const bool small_tiles = tiles32_per_block < 24;
  if (!small_tiles) {
    const bool nt = stream_exceeds_caches(p, D, 2);
    // A stream that no cache holds, under three row blocks (of 128 channels: more than one chunk of them) or, of 64 channels,
    // one chunk of four: stages of 16-token tiles, four of them, keep three quarters of the ring in flight under a stage's
    // products, two of 32-token tiles half of it.  Several chunks are 129 to 144 rows, and 65 to 96 that plan_attention leaves
    // in two: of many heads, of a slice count or workspace of the caller's.  us a call, 32-token tiles -> 16: 144 rows, 4 x 8
    // heads x 128 x 37000 239 -> 207, from pages 278 -> 248, x 20000 136 -> 118; 33 x 8 x 2558, 77 rows 139 -> 127, 44 x 8 x
    // 2600, 96 rows 164 -> 152; 4 x 8 x 36000, 96 rows in two chunks 137 -> 130; of 64 channels, 40K, 40 rows 64.5 -> 58.2,
    // 64 rows 66.3 -> 60.2, 37000, 144 rows 156 -> 155, from pages 200 -> 182; 38 x 8 x 9359, 77 rows 216 -> 220, from pages 285 -> 269;
    // one chunk of 128 channels only waits for HBM (2 x 8 x 37K, 64 rows 58.3 against 59.8), two chunks of four row blocks
    // gain nothing (4 x 8 x 128 x 20K, 104 rows 84.8 and 85.7; 64 channels x 40K 102 and 104).
    // Where the last-level cache can hold K and V the smaller tiles pay only while it does not, as in a round over many
    // layers (2 x 8 x 128 x 20K, 72 rows 53.1 -> 46.9; 33K x 4 heads from 24.5 to 23.7), and cost as much when it does, as in
    // calls over one layer (34.9 -> 42.2; 20.4 -> 22.4; 64 channels x 20K, 104 rows 28.7 -> 32.8): there the 32-token tiles stay.
    if constexpr (RB == 3 || (RB == 4 && D == 64))
      if (nt && (D == 64 ? RB == 3 || p.n_chunks == 1 : p.n_chunks > 1)) return launch_grid<D, RB, 4, 16, 4, true, true>(p, st);
    return nt ? launch_grid<D, RB, 4, 32, 2, true, true>(p, st) : launch_grid<D, RB, 4, 32, 2, false, true>(p, st);
  }
  // measured at the 16K configuration: with 3-4 row blocks, two token groups and a four-stage ring
  // (the whole slice in flight at once) beat four groups by ~8 %; the block merge moves half the data
  // four row blocks (49-64 query rows) over slices of 12-23 32-token tiles, three over 16-23, the 33K long-video shape:
  // the per-tile work of the vector unit weighs most there, and 32-token tiles halve it per token (three row blocks, 42
  // rows, us a call: 33K 19.6 -> 18.9, 40K 21.2 -> 20.9; at 26K, 12 tiles, 16.2 against 16.4; two chunks of 48, 84 rows at 16K
  // 17.6 -> 16.1, so two chunks take them from 12 tiles on as well, caches not in the last-level cache: 91 rows, 16000 tokens
  // 18.6 -> 17.0, chunks of 64 and a rest 18.4; 12500 tokens, 12 tiles, 15.7 against 16.7; 2 x 7000 16.1 against 17.4)
  if (RB >= 3 && tiles32_per_block >= (RB == 4 || p.n_chunks > 1 ? 12 : 16)) return launch_grid<D, RB, 2, 32, 3>(p, st);
  if (RB >= 3) return launch_grid<D, RB, 2, 16, 4>(p, st);
  if constexpr (RB == 1)
    if (one_slice_call(p)) return launch_grid<D, RB, 4, 16, 3, false, false, true>(p, st);
  return launch_grid<D, RB, 4, 16, 3>(p, st);
}

// 65 to 96 rows in one block (plan_attention says when; the cache exceeds the last-level cache): twelve waves in two token
// groups, 128 KB of ring in stages of two 32-token tiles, of which all but one are in flight.
template <int D>
static hipError_t launch_grid_wide(const AttnParams& p, hipStream_t st) {
  return launch_grid<D, 6, kWideGroups, 32, D == 128 ? 4 : 8, true, true>(p, st);
}

// fp8 cache: 32-token tiles only; short slices keep the whole slice in flight (two token groups, four
// ring stages), long ones use four groups and two stages
template <int D, int RB>
static hipError_t launch_kv8_rb(const AttnParams& p, hipStream_t st) {
  const int tiles32_per_block = ((p.n_total + 31) / 32) / (p.S > 0 ? p.S : 1);
  if constexpr (RB == 1)
    if (one_slice_call(p)) return launch_grid_mode<D, RB, 2, 32, 4, 0, true, false, false, true>(p, st);
  if (tiles32_per_block < 24)
    return launch_grid_mode<D, RB, 2, 32, 4, 0, true>(p, st);
  if (stream_exceeds_caches(p, D, 1)) return launch_grid_mode<D, RB, 4, 32, 2, 0, true, true, true>(p, st);
  return launch_grid_mode<D, RB, 4, 32, 2, 0, true, false, true>(p, st);
}

template <int D>
static hipError_t launch_kv8_d(const AttnParams& p, hipStream_t st) {
  switch (p.row_chunk / 16) {
    case 1: return launch_kv8_rb<D, 1>(p, st);
    case 2: return launch_kv8_rb<D, 2>(p, st);
    case 3: return launch_kv8_rb<D, 3>(p, st);
    case 4: return launch_kv8_rb<D, 4>(p, st);
    default: return hipErrorInvalidValue;
  }
}

template <int D>
static hipError_t launch_mfma_d(const AttnParams& p, hipStream_t st) {
  switch (p.row_chunk / 16) {
    case 1: return launch_grid_rb<D, 1>(p, st);
    case 2: return launch_grid_rb<D, 2>(p, st);
    case 3: return launch_grid_rb<D, 3>(p, st);
    case 4: return launch_grid_rb<D, 4>(p, st);
    case 6: return launch_grid_wide<D>(p, st);
    default: return hipErrorInvalidValue;
  }
}

template <int D, int RB, int TG, int NST, int MODE, bool ONE>
static hipError_t launch_f32_mode(const AttnParams& p, hipStream_t st) {
  constexpr int smem = F32Smem<D, TG, NST>::total(RB) + (MODE == 2 ? kMaxSlicePages * 4 : 0);
  const hipError_t e = allow_dynamic_lds<attn_partial_f32<D, RB, TG, NST, MODE, ONE>>(smem);
  if (e != hipSuccess) return e;
  AttnParams q = p;
  const int n_tiles = (p.n_total + 15) / 16;
  q.tiles_q = n_tiles / p.S;
  q.tiles_r = n_tiles % p.S;
  hipLaunchKernelGGL((attn_partial_f32<D, RB, TG, NST, MODE, ONE>), dim3(p.S, p.Hkv, p.B * p.n_chunks), dim3(RB * TG * 64),
                     smem, st, q);
  return hipGetLastError();
}

template <int D, int RB, int TG, int NST, bool ONE = false>
static hipError_t launch_f32(const AttnParams& p, hipStream_t st) {
  if (p.block_table != nullptr) return launch_f32_mode<D, RB, TG, NST, 2, ONE>(p, st);
  if (p.k_new != nullptr) return launch_f32_mode<D, RB, TG, NST, 1, ONE>(p, st);
  return launch_f32_mode<D, RB, TG, NST, 0, ONE>(p, st);
}

// row blocks x token groups: four groups while LDS and sixteen waves allow them
template <int D>
static hipError_t launch_f32_d(const AttnParams& p, hipStream_t st) {
  // ring stages: what 160 KB of LDS hold beside the queries
  constexpr bool W = D == 128;
  switch (p.row_chunk / 16) {
    case 1: return one_slice_call(p) ? launch_f32<D, 1, 4, W ? 2 : 4, true>(p, st) : launch_f32<D, 1, 4, W ? 2 : 4>(p, st);
    case 2: return launch_f32<D, 2, 4, W ? 2 : 4>(p, st);
    case 3: return launch_f32<D, 3, 4, W ? 2 : 4>(p, st);
    case 4: return launch_f32<D, 4, W ? 2 : 4, W ? 3 : 4>(p, st);
    case 6: return launch_f32<D, 6, 2, W ? 3 : 4>(p, st);
    case 8: return launch_f32<D, 8, 2, W ? 2 : 4>(p, st);
    default: return hipErrorInvalidValue;
  }
}

template <typename T, int D, int PO>
static hipError_t launch_combine(const AttnParams& p, hipStream_t st) {
  hipLaunchKernelGGL((attn_combine<T, D, PO>), dim3(p.R, p.Hkv, p.B), dim3(256), 0, st, p);
  return hipGetLastError();
}

hipError_t launch_attention(const AttnParams& p, int dtype, int head_dim, hipStream_t st) {
  hipError_t e;
  if (dtype == HIPPO_DTYPE_BF16) {
    if (p.k_scale != nullptr) e = (head_dim == 128) ? launch_kv8_d<128>(p, st) : launch_kv8_d<64>(p, st);
    else e = (head_dim == 128) ? launch_mfma_d<128>(p, st) : launch_mfma_d<64>(p, st);
    if (e != hipSuccess || one_slice_call(p)) return e;
    if (p.row_chunk > 64)
      return (head_dim == 128) ? launch_combine<uint16_t, 128, kPartF16>(p, st) : launch_combine<uint16_t, 64, kPartF16>(p, st);
    return (head_dim == 128) ? launch_combine<uint16_t, 128, kPartBf16>(p, st) : launch_combine<uint16_t, 64, kPartBf16>(p, st);
  }
  e = (head_dim == 128) ? launch_f32_d<128>(p, st) : launch_f32_d<64>(p, st);
  if (e != hipSuccess || one_slice_call(p)) return e;
  return (head_dim == 128) ? launch_combine<float, 128, kPartF32>(p, st) : launch_combine<float, 64, kPartF32>(p, st);
}

}  // namespace hippo

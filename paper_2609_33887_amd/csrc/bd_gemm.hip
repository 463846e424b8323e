// Projection GEMMs and the fused LM-head softmax-statistics kernel.
//
// All products are C = A . W^T with A [rows][K] (activations, row-major) and
// W [N][K] (weights stored [out][in]), so both operands are K-contiguous.
//
// bf16 path (bf16 weights, activations as bf16 hi/lo plane pairs): workgroup
// tiles of 128 x 256 down to 32 x 64 over 4 or 8 waves (see Gemm and the tiles
// below it), MFMA 16x16x32 bf16 with fp32 accumulate (plan_gemm and the
// launchers choose).  Operands reach LDS through direct buffer-to-LDS loads
// into a ring of two to four stages of 32 or 64 depth (swizzled rows); one
// barrier per stage; the residual projections may split K (the partial sums
// are folded in by the next RMSNorm).
// fp8 weights (WQ = WQ_FP8): W holds OCP fp8 E4M3 codes, one byte per
// element, with a power-of-two scale per output row; the W stage holds
// 64-byte rows, each lane converts its 8 codes of a fragment to bf16 (exact)
// before the MFMA, and the epilogue multiplies each output column by its row
// scale (exact, so the result equals the bf16 product with the dequantized
// weights).
// MXFP4 weights (WQ = WQ_MXFP4): a 64-deep stage is two MX blocks, so the
// stage holds 16 bytes of E2M1 codes and an exponent for each block of each W
// row; the lane converts its 8 codes with the block scale
// (v_cvt_scalef32_pk_bf16_fp4: E2M1 value x 2^X, exact in bf16), again the bf16
// product with the dequantized weights.  The codes are stored block-major
// (WQuant), so a block's W rows are one contiguous run of 16-byte rows.
// f32 path (small fp32 models): fp32 MFMA tiles, the sums in order of depth.
//
// The row count M is read from device memory so that a launch sized for the
// largest window can be replayed every step; tiles at or past M exit.
#include "bd_internal.h"

#include <math.h>

namespace bd {

static inline int cdiv(int a, int b) { return (a + b - 1) / b; }

__device__ __forceinline__ float bf2f(bf16_t h) { return __uint_as_float(((uint32_t)h) << 16); }
__device__ __forceinline__ bf16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);   // round to nearest, ties to even
  return (bf16_t)(u >> 16);
}
__device__ __forceinline__ float silu(float x) { return x / (1.0f + expf(-x)); }
// Store x as the bf16 pair (hi at p, lo at p + plane): hi = bf16(x), lo = bf16(x - hi).
__device__ __forceinline__ void store_pair(bf16_t* p, size_t plane, float x) {
  const bf16_t h = f2bf(x);
  p[0] = h;
  p[plane] = f2bf(x - bf2f(h));
}

// ------------------------------------------------------------------ bf16 MFMA
// Activation operands are carried as two bf16 planes, hi = bf16(x) and
// lo = bf16(x - hi), written by the producing kernel; the product is
// accumulated as hi.W + lo.W, two MFMAs per weight fragment, which gives the
// operand 16 significant bits, so that the only activation roundings of the
// forward are the Q/K/V values stored in the KV cache.
//
// Main loop: K advances in stages of SK through a ring of NS LDS stages filled
// by direct buffer-to-LDS loads (no register staging, no LDS store
// instructions); NS - 1 stages are in flight while one is consumed, and one
// barrier per stage both publishes the stage and retires the one the next
// loads overwrite.  The operands go through buffer resources rather than
// global (flat) addresses: the compiler counts a flat load into LDS as pending
// LDS traffic too, which turned every LDS wait of the loop into a full drain.
//
// A tile is shared by WM x WN waves, or by KG such groups, each taking its own
// part of every stage's depth for the whole tile: two waves a SIMD then cost
// no more LDS reads per product than one (a wave's tile stays 64 x 64), and a
// stage can be 64 deep, which halves the barriers.  The groups' sums meet in
// LDS once, at the end.  Measured (us, two groups over 64-deep stages against
// one over 32-deep ones): 512 x 16384 x 2048 76 / 85, 512 x 2048 x 8192 in 4
// splits 30 / 34, 1024 x 2048 x 8192 in 2 splits 54 / 63, 3072 x 3072 x 2048
// 77 / 90, 512 x 3072 x 2048 in 64 x 128 tiles 17.2 / 18.7 and 64 x 64 tiles
// (one group, 64 deep) 19.3 / 24.8.
//
// LDS: rows of 2 SK bytes, the 16-byte chunk c of row r at position c ^ swz(r);
// swz(r) = r & 7 for rows of 128 bytes and (r >> 1) & 3 for rows of 64: the 8
// lanes that one LDS cycle serves (8 rows, one chunk) then meet 8 distinct
// 16-byte columns (measured: no conflict cycles).
__device__ __forceinline__ int swz(int row_bytes, int r) { return row_bytes == 128 ? (r & 7) : ((r >> 1) & 3); }

typedef __attribute__((address_space(3))) void lds_void_t;

// Fourth word of a raw buffer resource on gfx9-family parts: 32-bit data
// format (a zero format reads zeros), no index stride, no swizzle.
constexpr int BUF_DWORD3 = 0x00020000;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const void* p) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, -1, BUF_DWORD3);
}
__device__ __forceinline__ void load_lds16(__amdgpu_buffer_rsrc_t r, void* lds, uint32_t off, uint32_t soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void_t*)lds, 16, off, soff, 0, 0);
}
__device__ __forceinline__ void load_lds4(__amdgpu_buffer_rsrc_t r, void* lds, uint32_t off, uint32_t soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void_t*)lds, 4, off, soff, 0, 0);
}

// Eight E2M1 codes (nibbles of v, k order, low nibble first) times the block
// scale -> eight bf16 (exact).
__device__ __forceinline__ bf16x8 fp4x8_to_bf16(uint32_t v, float scale) {
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  const bf16x2_t a = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(v, scale, 0);
  const bf16x2_t b = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(v, scale, 1);
  const bf16x2_t c = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(v, scale, 2);
  const bf16x2_t d = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(v, scale, 3);
  bf16x8 o;
  o[0] = a[0]; o[1] = a[1]; o[2] = b[0]; o[3] = b[1];
  o[4] = c[0]; o[5] = c[1]; o[6] = d[0]; o[7] = d[1];
  return o;
}

// Eight E4M3 codes (bytes 0..7 of v, k order) -> eight bf16 (exact).
__device__ __forceinline__ bf16x8 fp8x8_to_bf16(u32x2 v) {
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  const bf16x2_t a = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(v[0], 1.0f, false);
  const bf16x2_t b = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(v[0], 1.0f, true);
  const bf16x2_t c = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(v[1], 1.0f, false);
  const bf16x2_t d = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(v[1], 1.0f, true);
  bf16x8 o;
  o[0] = a[0]; o[1] = a[1]; o[2] = b[0]; o[3] = b[1];
  o[4] = c[0]; o[5] = c[1]; o[6] = d[0]; o[7] = d[1];
  return o;
}

// s_waitcnt vmcnt(N) lgkmcnt(0) (gfx9 encoding): before a stage barrier the
// wave's global->LDS loads but the N youngest have landed and all of its LDS
// reads have returned, so that no wave overwrites a stage another still
// reads (the barrier itself waits for neither)
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (0 << 8));
}

// One stage.  W rows: bf16 (2 SK bytes, swizzled), fp8 codes (SK bytes,
// swizzled), or E2M1 codes as [SK / 32][BN][16 bytes] with the blocks'
// exponents [SK / 32][BN], dealt to the NW waves that load them: each fills 256
// bytes with copies of its share (a load of some lanes only is a branch, after
// which the compiler no longer counts the loads in flight).
template <int BM, int BN, int SK, int WQ, int NW>
struct GemmStage {
  bf16_t a[2][BM * SK];
  uint8_t b[WQ == WQ_NONE ? BN * SK * 2 : (WQ == WQ_FP8 ? BN * SK : BN * SK / 2)];
  uint8_t be[WQ == WQ_MXFP4 ? 256 * NW : 0];
};

// The ring's stages are separate LDS objects (declared by the kernel, see
// BD_GEMM_SMEM) so that the compiler can tell the loads into one stage from
// the reads of another; those past NS are never touched and take no space.
template <class St>
struct GemmRing {
  St &s0, &s1, &s2, &s3;
  template <int I>
  __device__ __forceinline__ St& at() const {
    if constexpr (I == 0) return s0;
    else if constexpr (I == 1) return s1;
    else if constexpr (I == 2) return s2;
    else return s3;
  }
};
#define BD_GEMM_SMEM(G)                                                     \
  __shared__ __attribute__((aligned(1024))) typename G::Stage gs0, gs1, gs2, gs3; \
  const typename G::Ring ring{gs0, gs1, gs2, gs3}

template <int BM_, int BN_, int WM, int WN, int KG_, int SK_, int NS, int WQ_>
struct Gemm {
  static constexpr int BM = BM_, BN = BN_, KG = KG_, SK = SK_, WQ = WQ_;
  static constexpr int NW = WM * WN * KG, NT = 64 * NW;
  static constexpr int WROWS = BM / WM, WCOLS = BN / WN;          // a wave's part of the tile
  static constexpr int FM = WROWS / 16, FN = WCOLS / 16;
  static constexpr int KS = SK / 32 / KG;                         // MFMA depths per wave and stage
  static constexpr int ARB = SK * 2;                              // bytes of an A row in LDS
  static constexpr int ARPI = 1024 / ARB;                         // rows per 1 KiB load instruction
  static constexpr int LA = BM / (ARPI * NW);
  // W load instructions per wave and stage, and their bytes per lane
  static constexpr int WB = WQ == WQ_NONE ? BN * SK * 2 : (WQ == WQ_FP8 ? BN * SK : BN * SK / 2);
  static constexpr int WLB = WQ != WQ_MXFP4 && WB >= 1024 * NW ? 16 : 4;
  static constexpr int LB = WB / (64 * WLB * NW);
  static constexpr int EXPB = WQ == WQ_MXFP4 ? BN * SK / MX_BLOCK / NW : 0;   // exponent bytes per wave
  static constexpr int LPS = 2 * LA + LB + (WQ == WQ_MXFP4 ? 1 : 0);          // load instructions per stage
  static_assert(LA >= 1 && LB >= 1 && LA * ARPI * NW == BM && LB * 64 * WLB * NW == WB, "whole loads per wave");
  static_assert(KS >= 1 && (WQ == WQ_NONE || (SK == 64 && KG == 2)), "quantized weights: two groups, 64 deep");
  static_assert(NS >= 2 && NS <= 4 && (KALIGN / SK) % 2 == 0, "ring");
  typedef GemmStage<BM, BN, SK, WQ, NW> Stage;
  typedef GemmRing<Stage> Ring;
  // output tile in LDS (see to_lds): half of the rows in each of two stages
  static constexpr int LD = BN + 4;
  static constexpr bool TILE_FITS = sizeof(Stage) >= sizeof(float) * (BM / 2) * LD;

  floatx4 acc[FM][FN];
  __amdgpu_buffer_rsrc_t rah, ral, rw, re;
  uint32_t ao[LA], wo[LB], eo;
  // MXFP4: the codes (and exponents) of the stage to be loaded next, their bytes per stage
  const uint8_t *wnext, *enext;
  size_t wstep, estep;
  int lane, wave, wm, wn, kg;

  // 16-byte chunk of an A row for group g of the lanes at MFMA depth q: the
  // depths are permuted alike on both sides; fp8 rows are read 16 codes at a
  // time, of which group kg takes 8
  __device__ __forceinline__ int achunk(int q, int g) const {
    return WQ == WQ_FP8 ? 2 * g + kg : (kg * KS + q) * 4 + g;
  }

  __device__ __forceinline__ void issue(Stage& s, int kt) {
    const uint32_t ka = (uint32_t)kt * ARB;
#pragma unroll
    for (int i = 0; i < LA; ++i) {
      const int r = (i * NW + wave) * ARPI;
      load_lds16(rah, s.a[0] + r * SK, ao[i], ka);
      load_lds16(ral, s.a[1] + r * SK, ao[i], ka);
    }
    // bf16 and fp8: a stage is the next bytes of every W row.  MXFP4: the next
    // blocks of all N rows, 16 bytes a row; past 2^33 weights their offsets
    // leave 32 bits, so the resources move from stage to stage (an addition:
    // with at most three ring stages run() issues every stage once, in order).
    constexpr uint32_t WRB = WQ == WQ_FP8 ? SK : SK * 2;
    if constexpr (WQ == WQ_MXFP4) {
      static_assert(NS <= 3, "stages issued in order");
      rw = buf_rsrc(wnext);
      re = buf_rsrc(enext);
      wnext += wstep;
      enext += estep;
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      uint8_t* d = s.b + (i * NW + wave) * (64 * WLB);
      if constexpr (WLB == 16) load_lds16(rw, d, wo[i], (uint32_t)kt * WRB);
      else load_lds4(rw, d, wo[i], WQ == WQ_MXFP4 ? 0u : (uint32_t)kt * WRB);
    }
    if constexpr (WQ == WQ_MXFP4) load_lds4(re, s.be + wave * 256, eo, 0u);
  }

  __device__ __forceinline__ void mfma(const Stage& s) {
    const int r16 = lane & 15, g = lane >> 4;
#pragma unroll
    for (int q = 0; q < KS; ++q) {
      const int pos = (achunk(q, g) ^ swz(ARB, r16)) * 8;
      u32x4 b[FN];
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const int row = wn * WCOLS + j * 16 + r16;
        if constexpr (WQ == WQ_FP8) {
          const uint32_t off = sizeof(s.a) + row * SK + ((g ^ swz(SK, r16)) * 16) + kg * 8;
          const u32x2 raw = *(const u32x2*)((const char*)&s + off);
          b[j] = __builtin_bit_cast(u32x4, fp8x8_to_bf16(raw));
        } else if constexpr (WQ == WQ_MXFP4) {
          // 2^(e - 127) (e >= 1; e = 0 only in all-zero blocks, whose codes are zero)
          const uint32_t off = sizeof(s.a) + (kg * BN + row) * 16 + g * 4;
          const uint32_t eoff = sizeof(s.a) + sizeof(s.b) + (kg * BN + row) / EXPB * 256 + (kg * BN + row) % EXPB;
          const uint32_t raw = *(const uint32_t*)((const char*)&s + off);
          const uint32_t ex = *((const uint8_t*)&s + eoff);
          b[j] = __builtin_bit_cast(u32x4, fp4x8_to_bf16(raw, __uint_as_float(ex << 23)));
        } else {
          b[j] = *(const u32x4*)((const bf16_t*)s.b + row * SK + pos);
        }
      }
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        const int row = wm * WROWS + i * 16 + r16;
        const bf16x8 ah = __builtin_bit_cast(bf16x8, *(const u32x4*)(s.a[0] + row * SK + pos));
        const bf16x8 al = __builtin_bit_cast(bf16x8, *(const u32x4*)(s.a[1] + row * SK + pos));
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, __builtin_bit_cast(bf16x8, b[j]), acc[i][j], 0, 0, 0);
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, __builtin_bit_cast(bf16x8, b[j]), acc[i][j], 0, 0, 0);
      }
    }
  }

  // Order of a stage's instructions: the fragment reads, then its products with
  // the next loads spread between them.  Loads issued together right after the
  // barrier queue up, and a wave whose loads wait there does not get to its reads
  // (3072 x 16384 x 2048: 319 us with the loads first, 300 so; 8320-key decode
  // step 929 -> 908).
  static constexpr int DS_READS = KS * (2 * FM + FN * (WQ == WQ_MXFP4 ? 2 : 1)), MFMAS = KS * 2 * FM * FN;
  template <int L>
  __device__ __forceinline__ static void spread_loads() {
    if constexpr (L == 0) __builtin_amdgcn_sched_group_barrier(0x100, DS_READS, 0);
    if constexpr (L < LPS) {
      __builtin_amdgcn_sched_group_barrier(0x008, MFMAS * (L + 1) / (LPS + 1) - MFMAS * L / (LPS + 1), 0);
      __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      spread_loads<L + 1>();
    }
  }

  // steady state, stages t .. t + NS - 1: own loads of the stage done (the
  // younger ones may still be in flight), barrier (everyone's loads done,
  // everyone past the stage before), refill that one, compute
  template <int I>
  __device__ __forceinline__ void group(const Ring& rg, int t) {
    if constexpr (I < NS) {
      wait_vmcnt<(NS - 2) * LPS>();
      __builtin_amdgcn_s_barrier();
      issue(rg.template at<(I + NS - 1) % NS>(), t + I + NS - 1);
      mfma(rg.template at<I>());
      spread_loads<0>();
      group<I + 1>(rg, t);
    }
  }
  // the last REM stages, of which NS - 1 (or all, if fewer) are in flight
  template <int I, int REM>
  __device__ __forceinline__ void tail(const Ring& rg, int t) {
    if constexpr (I < REM) {
      constexpr int LEFT = REM - 1 - I;
      wait_vmcnt<(LEFT < NS - 2 ? LEFT : NS - 2) * LPS>();
      __builtin_amdgcn_s_barrier();
      if constexpr (I + NS - 1 < REM) issue(rg.template at<(I + NS - 1) % NS>(), t + I + NS - 1);
      mfma(rg.template at<I % NS>());
      tail<I + 1, REM>(rg, t);
    }
  }

  // K range [k0, k0 + klen), klen a positive multiple of KALIGN (so the stage
  // count is even, and a multiple of 4 for SK 32).  The A rows are m0 + r, or
  // gathered through arows.  Rows past the nvalid live ones repeat the first:
  // their results are discarded by the caller, and the lines they would bring
  // into LDS count (96 rows in tiles of 64: 64 x 128 tiles over 16384 columns
  // 26.9 -> 24.7 us, 64 x 64 over 3072 18.3 -> 17.1).  Weights: bf16 or fp8 rows of stride
  // ldw, or (MXFP4) the stage-major blocks of ldw rows with the exponents wexp.
  // Resources start at the tile's first row (gathered rows: at row 0, so a
  // plane's rows x lda x 2 bytes must stay below 4 GiB, checked on the host).
  __device__ __forceinline__ void run(const Ring& rg, const bf16_t* __restrict__ A, int lda, size_t a_plane,
                                      const void* __restrict__ Wv, int ldw, const uint8_t* __restrict__ wexp, int k0,
                                      int klen, int m0, int n0, int nvalid,
                                      const int32_t* __restrict__ arows = nullptr) {
    lane = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    wn = wave % WN; wm = (wave / WN) % WM; kg = wave / (WN * WM);
    m0 = __builtin_amdgcn_readfirstlane(m0);
    n0 = __builtin_amdgcn_readfirstlane(n0);
    k0 = __builtin_amdgcn_readfirstlane(k0);
    const bf16_t* ab = A + (arows ? (size_t)0 : (size_t)m0 * lda) + k0;
    rah = buf_rsrc(ab);
    ral = buf_rsrc(ab + a_plane);
    const int ars = lane / (ARB / 16);                            // row of the lane within a load
#pragma unroll
    for (int i = 0; i < LA; ++i) {
      const int r = (i * NW + wave) * ARPI + ars;
      const int rv = r < nvalid ? r : 0;
      const int row = arows ? arows[rv] : rv;
      ao[i] = ((uint32_t)row * (uint32_t)lda + ((lane % (ARB / 16)) ^ swz(ARB, r)) * 8) * 2u;
    }
    if constexpr (WQ == WQ_MXFP4) {
      const size_t kb0 = (size_t)(k0 / MX_BLOCK);
      wnext = (const uint8_t*)Wv + (kb0 * ldw + n0) * 16;
      enext = wexp + kb0 * ldw + n0;
      wstep = (size_t)ldw * (16 * SK / MX_BLOCK);
      estep = (size_t)ldw * (SK / MX_BLOCK);
#pragma unroll
      for (int i = 0; i < LB; ++i) {
        const int by = (i * NW + wave) * 256 + lane * 4;          // byte in [blocks][BN][16]
        wo[i] = (uint32_t)(by / (BN * 16)) * (uint32_t)ldw * 16u + by % (BN * 16);
      }
      const int eb = wave * EXPB + (lane % (EXPB / 4)) * 4;
      eo = (uint32_t)(eb / BN) * (uint32_t)ldw + eb % BN;
    } else {
      constexpr int WRB = WQ == WQ_FP8 ? SK : SK * 2, ES = WQ == WQ_FP8 ? 1 : 2;
      rw = buf_rsrc((const uint8_t*)Wv + ((size_t)n0 * ldw + k0) * ES);
#pragma unroll
      for (int i = 0; i < LB; ++i) {
        const int by = (i * NW + wave) * (64 * WLB) + lane * WLB, r = by / WRB, in = by % WRB;
        wo[i] = (uint32_t)r * (uint32_t)ldw * ES + ((in >> 4) ^ swz(WRB, r)) * 16 + (in & 15);
      }
    }
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

    const int nk = __builtin_amdgcn_readfirstlane(klen / SK);
    // no scalar load left in flight: the loop's LDS waits can then count the
    // fragment reads down instead of draining them
    __builtin_amdgcn_s_waitcnt(0xC07F);
    // The ring is filled unconditionally (stages past the last load another
    // again): a fill under a branch leaves the compiler unsure of the loads in
    // flight, and it waits for younger ones before a stage's first reads.
    issue(rg.template at<0>(), 0);
    if constexpr (NS > 2) issue(rg.template at<1>(), 1);
    if constexpr (NS > 3) issue(rg.template at<2>(), SK == 32 || nk > 2 ? 2 : 1);
    int t = 0;
    for (; t + 2 * NS - 1 <= nk; t += NS) group<0>(rg, t);
    const int rem = nk - t;
    if constexpr (NS == 2 || (NS == 4 && SK == 32)) {
      tail<0, NS>(rg, t);                                         // nk is a multiple of NS
    } else if constexpr (NS == 3) {
      if (rem == 2) tail<0, 2>(rg, t);
      else if (rem == 3) tail<0, 3>(rg, t);
      else tail<0, 4>(rg, t);
    } else {
      if (rem == 2) tail<0, 2>(rg, t);
      else if (rem == 4) tail<0, 4>(rg, t);
      else tail<0, 6>(rg, t);
    }
  }

  // fp8 weights: multiply each accumulator column n by the weight's row scale
  // sc[n], a power of two
  __device__ __forceinline__ void scale_columns(const float* __restrict__ sc, int n0) {
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const float f = sc[n0 + wn * WCOLS + j * 16 + (lane & 15)];
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[i][j][r] *= f;
    }
  }

  // The output tile in LDS, fp32 rows of LD floats: rows [0, BM / 2) in stage
  // 0, the rest in stage 1.  Two groups' sums are added on the way (first the
  // second group's values are laid down, then the first group adds its own).
  struct Tile {
    float *p0, *p1;
    __device__ __forceinline__ float* row(int r) const { return r < BM / 2 ? p0 + r * LD : p1 + (r - BM / 2) * LD; }
  };
  __device__ __forceinline__ Tile to_lds(const Ring& rg) {
    static_assert(TILE_FITS && KG <= 2, "tile in LDS");
    const Tile o{(float*)&rg.template at<0>(), (float*)&rg.template at<1>()};
    __syncthreads();              // every wave is past its last stage
#pragma unroll
    for (int ph = KG - 1; ph >= 0; --ph) {
      if (kg == ph) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            float* p = o.row(wm * WROWS + i * 16 + (lane >> 4) * 4 + r) + wn * WCOLS + (lane & 15);
#pragma unroll
            for (int j = 0; j < FN; ++j) p[j * 16] = ph == KG - 1 ? acc[i][j][r] : p[j * 16] + acc[i][j][r];
          }
      }
      __syncthreads();
    }
    return o;
  }
};

// Tiles in use.  W and W2 (bf16 weights, windows of at least 2048 rows):
// 128 x 256 with 8 waves and a four-stage ring, one workgroup a CU, or 4
// waves and two stages, two workgroups a CU, which cover each other's waits and
// epilogues where the grid has a few rounds of them.
template <int WQ> using Tile128 = Gemm<128, 128, 2, 2, 2, 64, 3, WQ>;
template <int WQ> using Tile64x128 = Gemm<64, 128, 2, 2, 2, 64, 4, WQ>;
template <int WQ> using Tile64 = Gemm<64, 64, 2, 2, 2, 64, 3, WQ>;
typedef Gemm<64, 128, 2, 2, 1, 64, 2, WQ_NONE> Tile64x128x2;   // 4 waves, two workgroups a CU
typedef Gemm<64, 64, 2, 2, 1, 64, 2, WQ_NONE> Tile64x3;         // 4 waves, three workgroups a CU
typedef Gemm<32, 64, 1, 2, 2, 64, 4, WQ_NONE> Tile32;          // 4 waves
using TileW = Gemm<128, 256, 2, 4, 1, 32, 4, WQ_NONE>;
using TileW2 = Gemm<128, 256, 2, 2, 1, 32, 2, WQ_NONE>;

// Eight values as bf16 pairs: 16 bytes to each plane (p 16-byte aligned).
__device__ __forceinline__ void store_pair8(bf16_t* p, size_t plane, const float v[8]) {
  uint32_t h[4], l[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const bf16_t h0 = f2bf(v[2 * e]), h1 = f2bf(v[2 * e + 1]);
    h[e] = (uint32_t)h0 | ((uint32_t)h1 << 16);
    l[e] = (uint32_t)f2bf(v[2 * e] - bf2f(h0)) | ((uint32_t)f2bf(v[2 * e + 1] - bf2f(h1)) << 16);
  }
  *(u32x4*)p = u32x4{h[0], h[1], h[2], h[3]};
  *(u32x4*)(p + plane) = u32x4{l[0], l[1], l[2], l[3]};
}

__device__ __forceinline__ void store_pair4(bf16_t* p, size_t plane, const float v[4]) {
  bf16_t h[4], l[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    h[e] = f2bf(v[e]);
    l[e] = f2bf(v[e] - bf2f(h[e]));
  }
  *(uint2*)p = make_uint2((uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16));
  *(uint2*)(p + plane) =
      make_uint2((uint32_t)l[0] | ((uint32_t)l[1] << 16), (uint32_t)l[2] | ((uint32_t)l[3] << 16));
}

// SwiGLU of a packed gate/up tile (16 gate columns, then their 16 up columns)
// in LDS: rows [0, rows) go to out rows of stride ldo from feature f0 on, 8
// features a thread, one 16-byte store per plane.
template <class G>
__device__ __forceinline__ void swiglu_tile(const typename G::Tile& tl, int rows, bf16_t* __restrict__ out, int ldo,
                                            size_t out_plane) {
  constexpr int NO = G::BN / 16;             // 8-feature runs per row
  for (int it = threadIdx.x; it < rows * NO; it += G::NT) {
    const int r = it / NO, o = it % NO;
    const float* x = tl.row(r) + (o >> 1) * 32 + (o & 1) * 8;
    float y[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) y[k] = silu(x[k]) * x[16 + k];
    store_pair8(out + (size_t)r * ldo + o * 8, out_plane, y);
  }
}

// GEMM.  Items (split z, column tile x, row tile y) are numbered z-major, then
// in bands of row tiles (band_tile): an XCD's concurrent workgroups share the A
// slices of a few row tiles and the W slices of a few column tiles of one
// split.  For EPI_ADD_F32 with a split workspace, the kernel picks
// S = resid_splits(M) K-splits on the device (zmax is the largest allowed);
// with S > 1 every split stores its raw partial tile to ws[split][row][col]
// (rows padded to whole tiles) and the next RMSNorm of the residual stream adds
// the partials in split order.
template <class G, int EPI>
__global__ __launch_bounds__(G::NT) void k_gemm_bf16(const int32_t* __restrict__ Mp,
                                                     const bf16_t* __restrict__ A,
                                                     const void* __restrict__ W, size_t a_plane,
                                                     int lda, int ldw, int N, int K,
                                                     void* __restrict__ out, int ldo, size_t out_plane,
                                                     float* __restrict__ ws, int zmax,
                                                     const void* __restrict__ waux) {
  constexpr int BM = G::BM, BN = G::BN, WQ = G::WQ;
  const int M = *Mp;
  const int X = N / BN, Y = (M + BM - 1) / BM;
  int S = 1;
  if (EPI == EPI_ADD_F32 && ws) {
    ResidSplit r;
    r.nx = X; r.bm = BM; r.K = K; r.zmax = zmax;
    S = resid_splits(M, r);
  }
  const int items = X * Y * S;
  const int u = xcd_item(blockIdx.x, items);
  if (u >= items) return;
  const int z = u / (X * Y);
  int tx, ty;
  band_tile(u % (X * Y), X, Y, BAND_R, tx, ty);
  const int m0 = ty * BM, n0 = tx * BN;
  const int klen = K / S;
  BD_GEMM_SMEM(G);
  G t;
  t.run(ring, A, lda, a_plane, W, WQ == WQ_MXFP4 ? N : ldw, (const uint8_t*)waux, z * klen, klen, m0, n0, M - m0);
  if constexpr (WQ == WQ_FP8) t.scale_columns((const float*)waux, n0);
  float* wz = (EPI == EPI_ADD_F32 && S > 1) ? ws + (size_t)z * Y * BM * N : nullptr;
  if constexpr (G::TILE_FITS) {
    const typename G::Tile tl = t.to_lds(ring);
    const int rows = M - m0 < BM ? M - m0 : BM;
    if constexpr (EPI == EPI_SWIGLU) {
      swiglu_tile<G>(tl, rows, (bf16_t*)out + (size_t)m0 * ldo + (n0 >> 1), ldo, out_plane);
    } else {
      constexpr int NQ = BN / 4;
      for (int it = threadIdx.x; it < rows * NQ; it += G::NT) {
        const int r = it / NQ, c = (it % NQ) * 4;
        const floatx4 v = *(const floatx4*)(tl.row(r) + c);
        if (S > 1) {
          *(floatx4*)(wz + (size_t)(m0 + r) * N + n0 + c) = v;
        } else {
          floatx4* o = (floatx4*)((float*)out + (size_t)(m0 + r) * ldo + n0 + c);
          *o += v;
        }
      }
    }
  } else {
    // the wide tiles do not fit the ring: straight from the accumulators
#pragma unroll
    for (int i = 0; i < G::FM; ++i) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + t.wm * G::WROWS + i * 16 + (t.lane >> 4) * 4 + r;
        if (m >= M) continue;
        if constexpr (EPI == EPI_SWIGLU) {
#pragma unroll
          for (int j = 0; j < G::FN; j += 2) {
            const int pb = n0 + t.wn * G::WCOLS + j * 16;    // packed column of the gate group
            const int col = (pb >> 5) * 16 + (t.lane & 15);  // output feature
            store_pair((bf16_t*)out + (size_t)m * ldo + col, out_plane, silu(t.acc[i][j][r]) * t.acc[i][j + 1][r]);
          }
        } else {
#pragma unroll
          for (int j = 0; j < G::FN; ++j) {
            const int n = n0 + t.wn * G::WCOLS + j * 16 + (t.lane & 15);
            if (S > 1) wz[(size_t)m * N + n] = t.acc[i][j][r];
            else ((float*)out)[(size_t)m * ldo + n] += t.acc[i][j][r];
          }
        }
      }
    }
  }
}

// QKV projection with RoPE and the K/V cache write in the epilogue (bf16).
// The tile goes through LDS, so that every store is a 16-byte run of a plane
// and every table read 128 bytes.  q and k: the pair-interleaved weight puts
// both halves of a rotation in adjacent columns; a thread takes 8 pairs of a
// row (16 columns): y(i) = x(i) cos - x(i + hd/2) sin, y(i + hd/2) =
// x(i + hd/2) cos + x(i) sin in fp64 with one rounding to fp32, dims i .. i + 7
// and i + hd/2 ..  v: a thread takes a column (dim) and the 8 rows of one slot
// run of a 32-row group; where the group is 32 positions of one sequence from
// a multiple of 32 on, they are one 16-byte store per plane, else 4-position
// runs or single values.
template <class G>
__global__ __launch_bounds__(G::NT) void k_gemm_qkv(const int32_t* __restrict__ Mp,
                                                    const bf16_t* __restrict__ A,
                                                    const void* __restrict__ W, size_t a_plane,
                                                    int lda, int K, const void* __restrict__ waux,
                                                    QkvEpi e) {
  constexpr int BM = G::BM, BN = G::BN, WQ = G::WQ;
  const int M = *Mp;
  const int N = (e.H + 2 * e.Hkv) * e.hd;
  const int X = (N - e.first) / BN, Y = (M + BM - 1) / BM;
  const int u = xcd_item(blockIdx.x, X * Y);
  if (u >= X * Y) return;
  int tx, ty;
  band_tile(u, X, Y, BAND_R, tx, ty);
  const int m0 = ty * BM, n0 = e.first + tx * BN;
  BD_GEMM_SMEM(G);
  G t;
  t.run(ring, A, lda, a_plane, W, WQ == WQ_MXFP4 ? N : K, (const uint8_t*)waux, 0, K, m0, n0, M - m0);
  if constexpr (WQ == WQ_FP8) t.scale_columns((const float*)waux, n0);
  const typename G::Tile tl = t.to_lds(ring);
  const int hd = e.hd, half = hd >> 1;
  const int qcols = e.H * hd, qkcols = (e.H + e.Hkv) * hd;
  const int rows = M - m0 < BM ? M - m0 : BM;
  bf16_t* Q = (bf16_t*)e.Q;
  bf16_t* Kc = (bf16_t*)e.kv.K;
  bf16_t* Vc = (bf16_t*)e.kv.V;
  // columns [n0, n0 + nqk) of the tile belong to q and k heads, the rest to v
  const int nqk = qkcols - n0 < 0 ? 0 : (qkcols - n0 < BN ? qkcols - n0 : BN);
  const int cg = nqk >> 4;                                   // 16-column groups
  for (int it = threadIdx.x; it < rows * cg; it += G::NT) {
    const int r = it / cg, c0 = (it % cg) * 16, m = m0 + r, n = n0 + c0;
    const int head = n / hd, i0 = (n % hd) >> 1;
    const int seq = e.row_seq[m], pos = e.row_pos[m];
    const double* cs = e.rope + ((size_t)pos * half + i0) * 2;
    const float* x = tl.row(r) + c0;
    float y1[8], y2[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const double x1 = x[2 * k], x2 = x[2 * k + 1], cc = cs[2 * k], sn = cs[2 * k + 1];
      y1[k] = (float)(x1 * cc - x2 * sn);
      y2[k] = (float)(x2 * cc + x1 * sn);
    }
    const bool isq = n < qcols;
    bf16_t* o = isq ? Q + ((size_t)m * e.H + head) * hd
                    : Kc + (((size_t)seq * e.Hkv + (head - e.H)) * e.kv.maxpos + pos) * hd;
    const size_t plane = isq ? e.q_plane : e.kv.k_plane;
    store_pair8(o + i0, plane, y1);
    store_pair8(o + half + i0, plane, y2);
  }
  const int nv = BN - nqk;                                   // v columns, from column nqk on
  for (int it = threadIdx.x; it < nv * (BM / 8); it += G::NT) {
    const int j = it & 3, c = nqk + (it >> 2) % nv, g0 = (it >> 2) / nv * 32;   // slot run j of rows g0 .. g0 + 31
    if (g0 >= rows) continue;
    const int vn = n0 + c - qkcols, kh = vn / hd, dim = vn % hd;
    const int r0 = (j >> 1) * 16 + (j & 1) * 4;              // the run's keys: r0 .. r0 + 3, r0 + 8 .. r0 + 11
    float v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = tl.row(g0 + r0 + (k >> 2) * 8 + (k & 3))[c];
    const int m = m0 + g0;
    bool run = g0 + 31 < rows;
    if (run) {
      const int p0 = e.row_pos[m];
      run = p0 % 32 == 0 && e.row_pos[m + 31] == p0 + 31 && e.row_seq[m] == e.row_seq[m + 31];
      if (run)
        store_pair8(Vc + ((size_t)e.row_seq[m] * e.Hkv + kh) * hd * e.kv.vstride + vt_row(p0, dim, hd) + 8 * j,
                    e.kv.v_plane, v);
    }
    if (run) continue;
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      const int r = g0 + r0 + hf * 8;                        // 4 rows from r on
      if (r >= rows) continue;
      if (e.rows4 && r + 3 < rows) {
        store_pair4(Vc + ((size_t)e.row_seq[m0 + r] * e.Hkv + kh) * hd * e.kv.vstride +
                        vt_off(e.row_pos[m0 + r], dim, hd),
                    e.kv.v_plane, v + 4 * hf);
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (r + k < rows)
            store_pair(Vc + ((size_t)e.row_seq[m0 + r + k] * e.Hkv + kh) * hd * e.kv.vstride +
                           vt_off(e.row_pos[m0 + r + k], dim, hd),
                       e.kv.v_plane, v[4 * hf + k]);
      }
    }
  }
}

// Grouped GEMM over experts: tile ti covers rows [m0, m0 + 128) of expert
// tile_e[ti]; the expert's rows sit at [e_off[e], e_off[e] + e_cnt[e]) of the
// expert-sorted outputs.  The A rows are gathered through a_rows (token rows
// of the expert-sorted assignments) or, with a_rows == NULL, read from the
// expert-sorted layout itself.  W of expert e starts e * w_stride weight
// elements in (its codes, for quantized weights); fp8 row scales at
// waux + e * N, MXFP4 exponents at waux + e * w_stride / 32.
template <class G, int EPI>
__global__ __launch_bounds__(G::NT) void k_gemm_grouped(const bf16_t* __restrict__ A, int lda,
                                                        size_t a_plane, const void* __restrict__ W,
                                                        int ldw, int K, GroupTiles g,
                                                        void* __restrict__ out, int ldo,
                                                        size_t out_plane,
                                                        const void* __restrict__ waux, int N) {
  constexpr int BN = G::BN, WQ = G::WQ;
  static_assert(G::BM == GROUP_BM, "expert row tiles");
  const int ti = blockIdx.y;
  if (ti >= *g.ntiles) return;
  const int e = g.tile_e[ti], m0 = g.tile_m0[ti];
  const int cnt = g.e_cnt[e], base = g.e_off[e];
  const int n0 = blockIdx.x * BN;
  BD_GEMM_SMEM(G);
  G t;
  const size_t eoff = (size_t)e * g.w_stride;
  const void* We = WQ == WQ_NONE  ? (const void*)((const bf16_t*)W + eoff)
                   : WQ == WQ_FP8 ? (const void*)((const uint8_t*)W + eoff)
                                  : (const void*)((const uint8_t*)W + eoff / 2);
  const uint8_t* wexp = WQ == WQ_MXFP4 ? (const uint8_t*)waux + eoff / MX_BLOCK : nullptr;
  // EPI_SWIGLU: gate/up over gathered token rows; else down over sorted rows
  if constexpr (EPI == EPI_SWIGLU)
    t.run(ring, A, lda, a_plane, We, WQ == WQ_MXFP4 ? N : ldw, wexp, 0, K, 0, n0, cnt - m0, g.a_rows + base + m0);
  else
    t.run(ring, A, lda, a_plane, We, WQ == WQ_MXFP4 ? N : ldw, wexp, 0, K, base + m0, n0, cnt - m0);
  if constexpr (WQ == WQ_FP8) t.scale_columns((const float*)waux + (size_t)e * N, n0);
  const typename G::Tile tl = t.to_lds(ring);
  const int rows = cnt - m0 < GROUP_BM ? cnt - m0 : GROUP_BM;
  const size_t row0 = (size_t)(base + m0);
  if constexpr (EPI == EPI_SWIGLU) {
    swiglu_tile<G>(tl, rows, (bf16_t*)out + row0 * ldo + (n0 >> 1), ldo, out_plane);
  } else {
    constexpr int NQ = BN / 4;
    for (int it = threadIdx.x; it < rows * NQ; it += G::NT) {
      const int r = it / NQ, c = (it % NQ) * 4;
      *(floatx4*)((float*)out + (row0 + r) * ldo + n0 + c) = *(const floatx4*)(tl.row(r) + c);
    }
  }
}

hipError_t launch_gemm_grouped(int epi, const void* A, int lda, size_t a_plane, const void* W,
                               int ldw, int N, int K, const GroupTiles& g, int max_tiles, void* out,
                               int ldo, size_t out_plane, WQuant wq, hipStream_t st) {
  if (N % 128 || K % KALIGN) return hipErrorInvalidValue;
  if ((wq.fmt != WQ_NONE) != (wq.aux != nullptr) || wq.fmt < WQ_NONE || wq.fmt > WQ_MXFP4)
    return hipErrorInvalidValue;
  if ((epi == EPI_SWIGLU) != (g.a_rows != nullptr)) return hipErrorInvalidValue;
  dim3 grid(N / 128, max_tiles);
  const bf16_t* a = (const bf16_t*)A;
#define BD_GROUPED(EPI_, WQ_, OP_)                                                                                   \
  k_gemm_grouped<Tile128<WQ_>, EPI_><<<grid, Tile128<WQ_>::NT, 0, st>>>(a, lda, a_plane, W, ldw, K, g, out, ldo, OP_, \
                                                                        wq.aux, N)
  if (epi == EPI_SWIGLU) {
    if (wq.fmt == WQ_FP8) BD_GROUPED(EPI_SWIGLU, WQ_FP8, out_plane);
    else if (wq.fmt == WQ_MXFP4) BD_GROUPED(EPI_SWIGLU, WQ_MXFP4, out_plane);
    else BD_GROUPED(EPI_SWIGLU, WQ_NONE, out_plane);
  } else {
    if (wq.fmt == WQ_FP8) BD_GROUPED(EPI_STORE_F32, WQ_FP8, 0);
    else if (wq.fmt == WQ_MXFP4) BD_GROUPED(EPI_STORE_F32, WQ_MXFP4, 0);
    else BD_GROUPED(EPI_STORE_F32, WQ_NONE, 0);
  }
#undef BD_GROUPED
  return hipGetLastError();
}

// Fused LM head: for its BN vocabulary columns the workgroup reduces each row
// to (max z, sum exp(z - max), lowest argmax) and writes one partial per
// (column tile, row); without LOGITS the logits never leave the workgroup.
// LOGITS: the tile's logits also go to the caller's [seq][position][V] buffer.
// They used to come from a second product of the same size, a scaling pass and
// a scatter pass over [rows][V]: 199 us for 3072 rows x 4096 columns (d 2048)
// on top of the head's 118, and 246 on top of 242 for 96 x 152064.
// Tiles that fit the ring go through LDS, four (128 x 128) or eight (64 x 128) threads a row; the wide ones
// (LM rows from 2048 on) reduce in the accumulators, 16 lanes a row.
template <class G, bool LOGITS>
__global__ __launch_bounds__(G::NT) void k_lm_head_bf16(const bf16_t* __restrict__ A, int d,
                                                        size_t a_plane,
                                                        const bf16_t* __restrict__ W, int V, int mask_id,
                                                        float scale, const int32_t* __restrict__ Mp,
                                                        int rows_cap, float* __restrict__ pmax,
                                                        float* __restrict__ psum,
                                                        int32_t* __restrict__ parg, StepOut so) {
  constexpr int BM = G::BM, BN = G::BN;
  const int M = *Mp;
  // items in bands of row tiles (band_tile): an XCD's concurrent workgroups
  // share a few row tiles of the operand and a few vocabulary tiles of the head
  const int X = V / BN, Y = (M + BM - 1) / BM;
  const int u = xcd_item(blockIdx.x, X * Y);
  if (u >= X * Y) return;
  int vt, ty;
  band_tile(u, X, Y, BAND_R, vt, ty);
  const int m0 = ty * BM, n0 = vt * BN;
  BD_GEMM_SMEM(G);
  G t;
  t.run(ring, A, d, a_plane, W, d, nullptr, 0, d, m0, n0, M - m0);
  if constexpr (G::TILE_FITS) {
    const typename G::Tile tl = t.to_lds(ring);
    constexpr int TPR = G::NT / BM, NC = BN / TPR;            // threads per row, columns per thread
    static_assert(TPR == 4 || TPR == 8, "lanes of a row are neighbours");
    const int rl = threadIdx.x / TPR, q = threadIdx.x % TPR, m = m0 + rl;
    // runs of 4 columns, the row's threads side by side
    float* x = tl.row(rl) + q * 4;
    float mx = -INFINITY;
    int arg = 0x7fffffff;
#pragma unroll
    for (int k = 0; k < NC / 4; ++k) {
      floatx4 v = *(floatx4*)(x + k * TPR * 4);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int n = n0 + k * TPR * 4 + q * 4 + c;
        v[c] = n == mask_id ? -INFINITY : scale * v[c];
        if (v[c] > mx) { mx = v[c]; arg = n; }
      }
      *(floatx4*)(x + k * TPR * 4) = v;
    }
#pragma unroll
    for (int off = 1; off < TPR; off <<= 1) {
      const float om = __shfl_xor(mx, off);
      const int oa = __shfl_xor(arg, off);
      if (om > mx || (om == mx && oa < arg)) { mx = om; arg = oa; }
    }
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < NC / 4; ++k) {
      const floatx4 v = *(const floatx4*)(x + k * TPR * 4);
#pragma unroll
      for (int c = 0; c < 4; ++c) s += expf(v[c] - mx);
    }
#pragma unroll
    for (int off = 1; off < TPR; off <<= 1) s += __shfl_xor(s, off);
    if (q == 0 && m < M) {
      const size_t o = (size_t)vt * rows_cap + m;
      pmax[o] = mx;
      psum[o] = s;
      parg[o] = arg;
    }
    if constexpr (LOGITS) {
      __syncthreads();
      const int rows = M - m0 < BM ? M - m0 : BM;
      for (int it = threadIdx.x; it < rows * BN; it += G::NT) {
        const int r = it / BN, c = it % BN;
        so.logits[so.at(m0 + r) * V + n0 + c] = tl.row(r)[c];
      }
    }
  } else {
    constexpr int FN = G::FN, NP = BN / G::WCOLS;
    // per-row partials of the NP column groups of waves
    __shared__ float red_m[NP][BM], red_s[NP][BM];
    __shared__ int32_t red_a[NP][BM];
    const int lane = t.lane, wm = t.wm, wn = t.wn;
#pragma unroll
    for (int i = 0; i < G::FM; ++i) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float v[FN];
        float mx = -INFINITY;
        int arg = 0x7fffffff;
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          const int n = n0 + wn * G::WCOLS + j * 16 + (lane & 15);
          v[j] = (n == mask_id) ? -INFINITY : scale * t.acc[i][j][r];
          if (v[j] > mx) { mx = v[j]; arg = n; }
        }
        const int rl = wm * G::WROWS + i * 16 + (lane >> 4) * 4 + r;
        if constexpr (LOGITS) {
          if (m0 + rl < M) {
            float* z = so.logits + so.at(m0 + rl) * V + n0 + wn * G::WCOLS + (lane & 15);
#pragma unroll
            for (int j = 0; j < FN; ++j) z[j * 16] = v[j];
          }
        }
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) {
          const float om = __shfl_xor(mx, off);
          const int oa = __shfl_xor(arg, off);
          if (om > mx || (om == mx && oa < arg)) { mx = om; arg = oa; }
        }
        float s = 0.f;
#pragma unroll
        for (int j = 0; j < FN; ++j) s += expf(v[j] - mx);
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) s += __shfl_xor(s, off);
        if ((lane & 15) == 0) {
          red_m[wn][rl] = mx;
          red_s[wn][rl] = s;
          red_a[wn][rl] = arg;
        }
      }
    }
    __syncthreads();
    if (threadIdx.x < BM) {
      const int rl = threadIdx.x, m = m0 + rl;
      if (m < M) {
        // column groups in order: the first group holding the maximum gives
        // the (lowest) argmax
        float mm = red_m[0][rl];
        int a = red_a[0][rl];
#pragma unroll
        for (int p = 1; p < NP; ++p)
          if (red_m[p][rl] > mm) { mm = red_m[p][rl]; a = red_a[p][rl]; }
        float s = 0.f;
#pragma unroll
        for (int p = 0; p < NP; ++p) s += red_s[p][rl] * expf(red_m[p][rl] - mm);
        const size_t o = (size_t)vt * rows_cap + m;
        pmax[o] = mm;
        psum[o] = s;
        parg[o] = a;
      }
    }
  }
}

// ------------------------------------------------------------------ f32 MFMA
// fp32 models are small, so their products are bound by latency and not by
// arithmetic.  A wave owns one 16 x 16 block and takes the whole depth in order
// on the fp32 matrix cores: v_mfma_f32_16x16x4_f32 adds its four products to
// the accumulator one after the other, each with one rounding, so the chain
// equals fmaf over k = 0, 1, .. K - 1 to the last bit (checked on gfx950,
// subnormal values included).  What is left is to keep the operands coming:
// chunks of 128 depths go straight into a ring of LDS stages, up to 384 depths
// in flight, for WM x WN waves that share the tile's rows.  Tiles: 16 x 32 with
// two waves, and 64 x 32 with eight where the row capacity holds at least 512
// of them.  4 rows, N 256, K 1024: 80 us with 64 x 64 x 16 SIMT tiles (4
// workgroups, 64 barrier steps, each thread the same sequential sum), 14 so;
// N 2048, K 256: 33 -> 5.6.
constexpr int FBN = 32;      // columns of a projection tile
constexpr int FHN = 64;      // columns of a head tile
constexpr int FKC = 128;     // depth per stage

template <int ROWS>
struct F32Stage {
  float x[ROWS * FKC];       // A rows, then W rows, 512 bytes each; 16-byte chunk c of row r at c ^ (r & 7)
};

template <int WM_, int WN_, int NS>
struct GemmF32 {
  static constexpr int WM = WM_, WN = WN_, NW = WM * WN, NT = 64 * NW;
  static constexpr int BM = 16 * WM, BN = 16 * WN, ROWS = BM + BN, LD = BN + 1;
  static constexpr int LN = ROWS / (2 * NW);      // 1 KiB loads (two rows) per wave and stage
  static_assert(LN * 2 * NW == ROWS && (NS - 1) * LN < 64, "whole loads per wave, all countable");
  typedef F32Stage<ROWS> Stage;
  typedef GemmRing<Stage> Ring;
  floatx4 acc;
  __amdgpu_buffer_rsrc_t ra, rw;
  uint32_t off[LN];
  int lane, wave;

  // rows 2 q, 2 q + 1 of the stage by load q; BM is a multiple of 16, so a
  // load is all A or all W.  Chunks past the depth repeat the last one: the
  // chain does not read them (masking the lanes off would be a branch, after
  // which the compiler no longer counts the loads in flight).
  __device__ __forceinline__ void issue(Stage& s, int t, int K) {
#pragma unroll
    for (int i = 0; i < LN; ++i) {
      const int q = i * NW + wave, r = 2 * q + (lane >> 5);
      const int col = t * FKC + ((lane & 31) ^ (r & 7)) * 4;
      load_lds16(q < BM / 2 ? ra : rw, s.x + 2 * q * FKC, off[i] + (uint32_t)min(col, K - 4) * 4u, 0);
    }
  }
  __device__ __forceinline__ void chain(const Stage& s, int steps) {
    const int c = lane & 15, g = lane >> 4;
    const float* pa = s.x + ((wave / WN) * 16 + c) * FKC + g;
    const float* pw = s.x + (BM + (wave % WN) * 16 + c) * FKC + g;
    const int sw = c & 7;     // blocks of 16 rows start at multiples of 8
    // four steps' operands are read while the four before them multiply (past
    // the last step the stage's first ones are read again, unused)
    float a[4], w[4], an[4], wn[4];
    auto read = [&](float* x, float* y, int q) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        x[e] = pa[((q + e) ^ sw) * 4];
        y[e] = pw[((q + e) ^ sw) * 4];
      }
    };
    auto mul = [&](const float* x, const float* y) {
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[e], y[e], acc, 0, 0, 0);
    };
    read(a, w, 0);
    for (int q = 0; q < steps; q += 8) {
      read(an, wn, q + 4 < steps ? q + 4 : 0);
      mul(a, w);
      if (q + 4 < steps) {
        read(a, w, q + 8 < steps ? q + 8 : 0);
        mul(an, wn);
      }
    }
  }
  template <int I, int REM, bool LAST>
  __device__ __forceinline__ void steps(const Ring& rg, int t, int K) {
    if constexpr (I < REM) {
      constexpr int LEFT = LAST ? (REM - 1 - I < NS - 2 ? REM - 1 - I : NS - 2) : NS - 2;
      wait_vmcnt<LEFT * LN>();
      __builtin_amdgcn_s_barrier();
      if constexpr (!LAST || I + NS - 1 < REM) issue(rg.template at<(I + NS - 1) % NS>(), t + I + NS - 1, K);
      const int left = (K - (t + I) * FKC) / 4;
      chain(rg.template at<I % NS>(), left < FKC / 4 ? left : FKC / 4);
      steps<I + 1, REM, LAST>(rg, t, K);
    }
  }
  template <int REM>
  __device__ __forceinline__ void tails(const Ring& rg, int t, int rem, int K) {
    if constexpr (REM <= 2 * NS - 2) {
      if (rem == REM) steps<0, REM, true>(rg, t, K);
      else tails<REM + 1>(rg, t, rem, K);
    }
  }
  // K a multiple of 16; the tile's W rows are wrow0 + n for n < 16 and, from
  // column 16 on, wrow0 + wstep + n - 16, .. (wstep rows per 16 columns)
  __device__ __forceinline__ void run(const Ring& rg, const float* __restrict__ A, int lda,
                                      const float* __restrict__ W, int ldw, int K, int m0, int wrow0, int wstep) {
    lane = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    m0 = __builtin_amdgcn_readfirstlane(m0);
    wrow0 = __builtin_amdgcn_readfirstlane(wrow0);
    ra = buf_rsrc(A + (size_t)m0 * lda);
    rw = buf_rsrc(W + (size_t)wrow0 * ldw);
#pragma unroll
    for (int i = 0; i < LN; ++i) {
      const int r = 2 * (i * NW + wave) + (lane >> 5);
      const int n = r - BM;
      off[i] = (r < BM ? (uint32_t)r * (uint32_t)lda
                       : (uint32_t)((n >> 4) * wstep + (n & 15)) * (uint32_t)ldw) * 4u;
    }
    acc = floatx4{0.f, 0.f, 0.f, 0.f};
    const int nk = (K + FKC - 1) / FKC;
    __builtin_amdgcn_s_waitcnt(0xC07F);
    issue(rg.template at<0>(), 0, K);
    issue(rg.template at<1>(), nk > 1 ? 1 : 0, K);
    if constexpr (NS > 3) issue(rg.template at<2>(), nk > 2 ? 2 : 0, K);
    int t = 0;
    for (; t + 2 * NS - 1 <= nk; t += NS) steps<0, NS, false>(rg, t, K);
    tails<1>(rg, t, nk - t, K);
  }
  // the tile in LDS (stage 0), rows of LD floats
  __device__ __forceinline__ float* to_lds(const Ring& rg) {
    static_assert(sizeof(Stage) >= sizeof(float) * BM * LD, "tile in a stage");
    float* o = rg.template at<0>().x;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r)
      o[((wave / WN) * 16 + 4 * (lane >> 4) + r) * LD + (wave % WN) * 16 + (lane & 15)] = acc[r];
    __syncthreads();
    return o;
  }
};
typedef GemmF32<1, 2, 4> F32Small;
typedef GemmF32<4, 2, 3> F32Large;
typedef GemmF32<1, 4, 3> F32Head;

template <class G, int EPI>
__global__ __launch_bounds__(G::NT) void k_gemm_f32(const float* __restrict__ A, int lda,
                                                    const float* __restrict__ W, int ldw, int K,
                                                    const int32_t* __restrict__ Mp,
                                                    float* __restrict__ out, int ldo) {
  constexpr int BM = G::BM, LD = G::LD;
  const int M = *Mp;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * FBN;
  if (m0 >= M) return;
  BD_GEMM_SMEM(G);
  G t;
  t.run(ring, A, lda, W, ldw, K, m0, n0, 16);
  const float* x = t.to_lds(ring);
  if constexpr (EPI == EPI_SWIGLU) {
    // packed gate/up groups of 16 columns
    for (int e = threadIdx.x; e < BM * 16; e += G::NT) {
      const int r = e >> 4, c = e & 15, m = m0 + r;
      if (m < M) out[(size_t)m * ldo + (n0 >> 1) + c] = silu(x[r * LD + c]) * x[r * LD + 16 + c];
    }
  } else {
    for (int e = threadIdx.x; e < BM * FBN; e += G::NT) {
      const int r = e / FBN, c = e % FBN, m = m0 + r;
      if (m < M) out[(size_t)m * ldo + n0 + c] += x[r * LD + c];
    }
  }
}

// fp32 QKV projection with RoPE and the cache write in the epilogue.  A tile
// is 16 dims i .. i + 15 of one head and their rotation partners
// i + hd/2 .. (its two column blocks), so both halves of a rotation meet in
// one thread; angle and rotation in fp64 with one rounding to fp32, at the
// row's absolute position.  q -> Q[row][head][hd], k and v -> the cache slots
// [seq][kv head][pos][hd].
template <class G>
__global__ __launch_bounds__(G::NT) void k_gemm_qkv_f32(const float* __restrict__ A, int lda,
                                                        const float* __restrict__ W, int K,
                                                        const int32_t* __restrict__ Mp, QkvEpi q,
                                                        const double* __restrict__ inv_freq) {
  constexpr int BM = G::BM, LD = G::LD;
  const int M = *Mp;
  const int m0 = blockIdx.y * BM;
  if (m0 >= M) return;
  const int half = q.hd / 2, tph = q.hd / FBN;              // tiles per head
  const int head = blockIdx.x / tph, i0 = (blockIdx.x % tph) * 16;
  BD_GEMM_SMEM(G);
  G t;
  t.run(ring, A, lda, W, K, K, m0, head * q.hd + i0, half);
  const float* x = t.to_lds(ring);
  for (int e = threadIdx.x; e < BM * 16; e += G::NT) {
    const int r = e >> 4, i = i0 + (e & 15), m = m0 + r;
    if (m >= M) continue;
    const double x1 = x[r * LD + (e & 15)], x2 = x[r * LD + 16 + (e & 15)];
    const int s = q.row_seq[m], pos = q.row_pos[m];
    float y1 = (float)x1, y2 = (float)x2;
    float* o;
    if (head < q.H + q.Hkv) {
      double sn, cs;
      sincos((double)pos * inv_freq[i], &sn, &cs);
      y1 = (float)(x1 * cs - x2 * sn);
      y2 = (float)(x2 * cs + x1 * sn);
      o = head < q.H ? (float*)q.Q + ((size_t)m * q.H + head) * q.hd
                     : (float*)q.kv.K + (((size_t)s * q.Hkv + (head - q.H)) * q.kv.maxpos + pos) * q.hd;
    } else {
      o = (float*)q.kv.V + (((size_t)s * q.Hkv + (head - q.H - q.Hkv)) * q.kv.maxpos + pos) * q.hd;
    }
    o[i] = y1;
    o[i + half] = y2;
  }
}

// fp32 LM head: 16 rows x 64 vocabulary columns; a wave then takes four rows,
// a lane a column.  The exponentials are summed over columns c, c + 16, c + 32,
// c + 48 and then over a tree of c.
constexpr int F32_HEAD_Y = 32768;   // row tiles over a grid's y, further ones over z (y and z hold 65,535)
__global__ __launch_bounds__(256) void k_lm_head_f32(const float* __restrict__ A, int d,
                                                     const float* __restrict__ W, int mask_id,
                                                     float scale, const int32_t* __restrict__ Mp,
                                                     int rows_cap, float* __restrict__ pmax,
                                                     float* __restrict__ psum,
                                                     int32_t* __restrict__ parg, int V, StepOut so) {
  typedef F32Head G;
  const int M = *Mp;
  const int m0 = (blockIdx.z * F32_HEAD_Y + blockIdx.y) * G::BM, n0 = blockIdx.x * FHN;
  if (m0 >= M) return;
  BD_GEMM_SMEM(G);
  G t;
  t.run(ring, A, d, W, d, d, m0, n0, 16);
  const float* x = t.to_lds(ring);
  const int lane = t.lane, n = n0 + lane;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = t.wave * 4 + q, m = m0 + r;
    if (m >= M) continue;                                   // wave-uniform
    const float v = n == mask_id ? -INFINITY : scale * x[r * G::LD + lane];
    if (so.logits) so.logits[so.at(m) * V + n] = v;
    // a NaN takes no part in the maximum (a lane that started from one would
    // keep the columns reduced through it out), only in the sum
    float mx = v == v ? v : -INFINITY;
    int arg = v == v ? n : 0x7fffffff;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const float om = __shfl_xor(mx, off);
      const int oa = __shfl_xor(arg, off);
      if (om > mx || (om == mx && oa < arg)) { mx = om; arg = oa; }
    }
    const float p = expf(v - mx);
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) s += __shfl(p, (lane & 15) + 16 * j);
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) s += __shfl_xor(s, off);
    if (lane == 0) {
      const size_t o = (size_t)blockIdx.x * rows_cap + m;
      pmax[o] = mx;
      psum[o] = s;
      parg[o] = arg;
    }
  }
}

// Merge the per-tile partials of each row (one wave per row, deterministic):
// max and lowest argmax over tiles, then sum_t s_t exp(m_t - max) with a
// fixed lane assignment and a fixed shuffle tree; conf = 1 / sum.
__global__ __launch_bounds__(256) void k_lm_merge(const float* __restrict__ pmax,
                                                  const float* __restrict__ psum,
                                                  const int32_t* __restrict__ parg, int ntiles,
                                                  const int32_t* __restrict__ Mp, int rows_cap,
                                                  float* __restrict__ conf, int32_t* __restrict__ tok,
                                                  StepOut so) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int m = blockIdx.x * 4 + wave;
  if (m >= *Mp) return;
  float mx = -INFINITY;
  int arg = 0x7fffffff;
  for (int t = lane; t < ntiles; t += 64) {
    const float v = pmax[(size_t)t * rows_cap + m];
    const int a = parg[(size_t)t * rows_cap + m];
    if (v > mx || (v == mx && a < arg)) { mx = v; arg = a; }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const float om = __shfl_xor(mx, off);
    const int oa = __shfl_xor(arg, off);
    if (om > mx || (om == mx && oa < arg)) { mx = om; arg = oa; }
  }
  float s = 0.f;
  for (int t = lane; t < ntiles; t += 64) {
    const size_t o = (size_t)t * rows_cap + m;
    s += psum[o] * expf(pmax[o] - mx);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  if (lane == 0) {
    conf[m] = 1.0f / s;
    tok[m] = arg;
    if (so.conf) so.conf[so.at(m)] = 1.0f / s;
    if (so.tok) so.tok[so.at(m)] = arg;
  }
}

// ------------------------------------------------------------------ launchers

template <class G>
static void launch_tile(int epi, dim3 grid, const bf16_t* a, int lda, size_t ap, const void* w,
                        int ldw, int N, int K, const int32_t* M_dev, void* o, int ldo, size_t op,
                        float* ws, int zmax, const void* waux, hipStream_t st) {
  if (epi == EPI_ADD_F32)
    k_gemm_bf16<G, EPI_ADD_F32><<<grid, G::NT, 0, st>>>(M_dev, a, w, ap, lda, ldw, N, K, o, ldo, op, ws, zmax, waux);
  else   // EPI_SWIGLU
    k_gemm_bf16<G, EPI_SWIGLU><<<grid, G::NT, 0, st>>>(M_dev, a, w, ap, lda, ldw, N, K, o, ldo, op, nullptr, 1, waux);
}

// Tile choice.  Figures: us a launch, from kernel traces of one layer's steps
// (weights warm in the caches), over half the row capacity as live rows, which
// is what a step window usually holds.
// Plain products (gate/up), N x K:
//  * 128 x 256 (launched in four waves, two workgroups a CU) over capacities of at
//    least 2048 rows from N 8192 on, bf16 weights.  16384 x 2048: 1024 rows 108-117
//    (128 x 128 124, 64 x 128 143), 3072 rows 305-315 (365, 385; 64 x 64 476);
//    8192 x 1024: 2048 rows 59 (71, 69), but 1024 rows 40 (37, 36).
//  * 128 x 128 where the capacity holds 1024 of them.  4096 x 2048, 2048 rows: 60
//    (64 x 128 64-69, 64 x 64 75); 16384 x 2048, 512 rows: 62 (62-69, 78).
//  * 64 x 128 over capacities of at most 1024 rows, bf16 weights.  Where half the
//    capacity gives more of them than CUs, four waves take one
//    (launch_gemm_planned), so that a CU runs two side by side and one multiplies
//    while the other waits for its stage: 8192 x 1024, 512 rows, 512 tiles, 19.5
//    (eight waves, one a CU: 22.5; 64 x 64 24); one tile a CU (16384 x 2048, 96
//    rows) takes 26.7 so and 18.8 with eight (64 x 64 21, 128 x 128 26).
//  * 64 x 64 else.  2816 x 2048, 2048 rows: 57, where 64 x 128 in eight waves
//    takes 51 and 128 x 128 54.
// Residual products (O and down), whose split partials the next norm reads:
//  * 128 x 256 (eight waves) over capacities of at least 2048 rows from K 2048 on,
//    bf16 weights.  2048 x 8192: 1024 rows 61-65 (128 x 128 65, 64 x 64 80), 3072
//    rows 204-212 (192, 234); 2048 x 2048: 1024 rows 23-26 (27, 28), 3072 rows 69
//    (62, 73).
//  * 128 x 128 where the capacity holds 512 of them (1024 x 1024, 4096 rows: 28
//    against 33-37 in 64 x 64) and, by plan_resid, from K 4096 on.
//  * 64 x 64 else; with up to 512 tiles over half the capacity four waves take one,
//    three workgroups a CU (launch_gemm_planned).  1024 x 1024: 512 rows 7.6 (eight
//    waves 10.2), 2048 rows, 512 tiles, 15.8 (18.7), 1024 tiles 33 (37); 2048 x 2048:
//    96 rows 7.5 (8.8), 1024 tiles 50.5 (48.8).
// Three of these lines lie off where the loops of today put them: 8192 x 1024 at
// 1024 rows, 2816 x 2048 at 2048, and 128 x 256 for the residual products past 2048
// live rows.  zmax: the largest residual split (1 = none).
GemmPlan plan_gemm(bool is_bf16, int N, int K, int rows_cap, bool resid, bool wide_ok) {
  if (!is_bf16) return GemmPlan{64, 64, 1};
  if (wide_ok && N % 256 == 0 && rows_cap >= 2048 && (N >= 8192 || (resid && K >= 2048)))
    return GemmPlan{128, 256, 1};
  if (N % 128 == 0 && (N / 128) * cdiv(rows_cap, 128) >= (resid ? 512 : 1024)) return GemmPlan{128, 128, 1};
  if (wide_ok && !resid && N % 128 == 0 && rows_cap <= 1024) return GemmPlan{64, 128, 1};
  return GemmPlan{64, 64, 1};
}

hipError_t launch_gemm_planned(const GemmPlan& p, int epi, const void* A, int lda, size_t a_plane,
                               const void* W, int ldw, int N, int K, const int32_t* M_dev,
                               int rows_cap, void* out, int ldo, size_t out_plane, float* ws,
                               hipStream_t st, WQuant wq) {
  const bool big = p.bm == 128 && p.bn == 128, small = p.bm == 64 && p.bn == 64;
  const bool wide = p.bm == 128 && p.bn == 256, mid = p.bm == 64 && p.bn == 128;
  if ((!big && !small && !wide && !mid) || p.zmax < 1 || p.zmax > 8) return hipErrorInvalidValue;
  if ((wq.fmt != WQ_NONE) != (wq.aux != nullptr) || wq.fmt < WQ_NONE || wq.fmt > WQ_MXFP4)
    return hipErrorInvalidValue;
  if ((wide || mid) && wq.fmt != WQ_NONE) return hipErrorInvalidValue;   // no quantized variants
  if (mid && p.zmax != 1) return hipErrorInvalidValue;
  if (epi != EPI_ADD_F32 && epi != EPI_SWIGLU) return hipErrorInvalidValue;
  if (N % p.bn || K % KALIGN) return hipErrorInvalidValue;
  if (p.zmax > 1 && (epi != EPI_ADD_F32 || !ws)) return hipErrorInvalidValue;
  // 1-D grid: every (split, column tile, row tile) of the row capacity, + 7
  // (see xcd_item)
  dim3 grid((N / p.bn) * cdiv(rows_cap, p.bm) * p.zmax + 7);
  const bf16_t* a = (const bf16_t*)A;
#define BD_TILE(G_) \
  launch_tile<G_>(epi, grid, a, lda, a_plane, W, ldw, N, K, M_dev, out, ldo, out_plane, ws, p.zmax, wq.aux, st)
  if (wq.fmt == WQ_FP8) {
    if (big) BD_TILE(Tile128<WQ_FP8>); else BD_TILE(Tile64<WQ_FP8>);
  } else if (wq.fmt == WQ_MXFP4) {
    if (big) BD_TILE(Tile128<WQ_MXFP4>); else BD_TILE(Tile64<WQ_MXFP4>);
  } else {
    if (wide && epi == EPI_SWIGLU) BD_TILE(TileW2);
    else if (wide) BD_TILE(TileW);
    else if (big) BD_TILE(Tile128<WQ_NONE>);
    else if (mid && (N / 128) * cdiv(cdiv(rows_cap, 2), 64) > 256) BD_TILE(Tile64x128x2);
    else if (mid) BD_TILE(Tile64x128<WQ_NONE>);
    else if (epi == EPI_ADD_F32 && (N / 64) * cdiv(cdiv(rows_cap, 2), 64) <= 512) BD_TILE(Tile64x3);
    else BD_TILE(Tile64<WQ_NONE>);
  }
#undef BD_TILE
  return hipGetLastError();
}

size_t resid_extent(int M, int N, const ResidSplit& r) {
  if (M < 1) return 0;
  const int S = resid_splits(M, r);
  return S > 1 ? (size_t)S * (size_t)cdiv(M, r.bm) * r.bm * N : 0;
}

size_t resid_extent_max(int rows_cap, int N, const ResidSplit& r) {
  // S and the slab height depend on M only through its row-tile count
  size_t mx = 0;
  for (int y = 1; y <= cdiv(rows_cap, r.bm); ++y) {
    const size_t e = resid_extent(y * r.bm < rows_cap ? y * r.bm : rows_cap, N, r);
    if (e > mx) mx = e;
  }
  return mx;
}

GemmPlan plan_resid(int N, int K, int rows_cap, bool wide_ok) {
  // Deep products (K >= 4096) take 128 x 128: with K split, their A and W re-reads
  // halve against 64 x 64 at the same parallelism.  2048 x 8192: 512 rows 33-35 us
  // against 39; 96 rows, where 8 splits make 128 workgroups, 16.1 against 14.0;
  // 1024 x 4096: 512 rows 15.5 against 14.5 (three workgroups a CU), 2048 rows 35
  // against 41.
  GemmPlan p = plan_gemm(true, N, K, rows_cap, true, wide_ok);
  if (K >= 4096 && N % 128 == 0 && p.bm != 128) p = GemmPlan{128, 128, 1};
  p.zmax = 8;
  return p;
}

hipError_t launch_gemm_resid(bool is_bf16, const void* A, int lda, size_t a_plane, const void* W,
                             int ldw, int N, int K, const int32_t* M_dev, int rows_cap, float* X,
                             int ldx, float* ws, size_t ws_floats, ResidSplit* fold, hipStream_t st,
                             WQuant wq) {
  fold->ws = nullptr;
  if (!is_bf16 || !ws)
    return launch_gemm(EPI_ADD_F32, is_bf16, A, lda, a_plane, W, ldw, N, K, M_dev, rows_cap, X, ldx, 0, st,
                       wq);
  const GemmPlan p = plan_resid(N, K, rows_cap, wq.fmt == WQ_NONE);
  ResidSplit r{};
  r.nx = N / p.bn;
  r.bm = p.bm;
  r.K = K;
  r.zmax = p.zmax;
  if (resid_extent_max(rows_cap, N, r) > ws_floats) return hipErrorInvalidValue;
  hipError_t e = launch_gemm_planned(p, EPI_ADD_F32, A, lda, a_plane, W, ldw, N, K, M_dev, rows_cap,
                                     X, ldx, 0, ws, st, wq);
  if (e != hipSuccess) return e;
  r.ws = ws;
  r.Mp = M_dev;
  *fold = r;
  return hipSuccess;
}

hipError_t launch_gemm_qkv(const void* A, int lda, size_t a_plane, const void* W, int K,
                           const int32_t* M_dev, int rows_cap, const QkvEpi& e, hipStream_t st,
                           WQuant wq) {
  const int N = (e.H + 2 * e.Hkv) * e.hd;
  if (e.hd % 16 || e.kv.vstride % 64 || K % KALIGN) return hipErrorInvalidValue;
  if ((wq.fmt != WQ_NONE) != (wq.aux != nullptr) || wq.fmt < WQ_NONE || wq.fmt > WQ_MXFP4)
    return hipErrorInvalidValue;
  // Tile by the workgroups it gives over half the row capacity (the rows a step
  // window usually holds; a prefill holds twice that): 128 x 128, then
  // 64 x 128, where there are at least 192 of them, else 64 x 64.  Measured for
  // N 3072, K 2048 (us, 128 x 128 / 64 x 128 / 64 x 64): 96 rows - / 14.3 /
  // 11.8, 512 rows 24.9 / 17.2 / 19.1, 1024 rows 28.8 / 32.3 / 30.4, 3072 rows
  // 77 / - / -.  At most half a 64 x 64 tile a CU: 32 x 64, which brings a third
  // less through each CU's L1 (96 rows in the 24-layer step: 12.7 against 17.1;
  // quantized weights keep 64 x 64).
  const int half_cap = cdiv(rows_cap, 2);
  const int bm = N % 128 == 0 && (N / 128) * cdiv(half_cap, 128) >= 192 ? 128
                 : wq.fmt == WQ_NONE && (N / 64) * cdiv(half_cap, 64) <= 128 ? 32 : 64;
  const int bn = bm == 128 || (wq.fmt == WQ_NONE && N % 128 == 0 && (N / 128) * cdiv(half_cap, 64) >= 192) ? 128 : 64;
  if (N % bn || e.first % bn) return hipErrorInvalidValue;
  dim3 grid(((N - e.first) / bn) * cdiv(rows_cap, bm) + 7);
  const bf16_t* a = (const bf16_t*)A;
#define BD_QKV(G_) k_gemm_qkv<G_><<<grid, G_::NT, 0, st>>>(M_dev, a, W, a_plane, lda, K, wq.aux, e)
  if (wq.fmt == WQ_FP8) {
    if (bm == 128) BD_QKV(Tile128<WQ_FP8>); else BD_QKV(Tile64<WQ_FP8>);
  } else if (wq.fmt == WQ_MXFP4) {
    if (bm == 128) BD_QKV(Tile128<WQ_MXFP4>); else BD_QKV(Tile64<WQ_MXFP4>);
  } else {
    if (bm == 128) BD_QKV(Tile128<WQ_NONE>);
    else if (bn == 128) BD_QKV(Tile64x128<WQ_NONE>);
    else if (bm == 32) BD_QKV(Tile32);
    else BD_QKV(Tile64<WQ_NONE>);
  }
#undef BD_QKV
  return hipGetLastError();
}

// 64 x 32 tiles instead of 16 x 32 where the row capacity holds at least 512 of
// them (two workgroups a CU): a quarter of the operand reads per product.
static bool f32_large(int N, int rows_cap) { return (N / FBN) * cdiv(rows_cap, 64) >= 512; }

hipError_t launch_gemm(int epi, bool is_bf16, const void* A, int lda, size_t a_plane, const void* W,
                       int ldw, int N, int K, const int32_t* M_dev, int rows_cap, void* out, int ldo,
                       size_t out_plane, hipStream_t st, WQuant wq) {
  if (is_bf16)
    return launch_gemm_planned(plan_gemm(true, N, K, rows_cap, false, wq.fmt == WQ_NONE), epi, A, lda, a_plane,
                               W, ldw, N, K, M_dev, rows_cap, out, ldo, out_plane, nullptr, st, wq);
  if (wq.fmt != WQ_NONE) return hipErrorInvalidValue;
  if (N % FBN || K % 16 || (epi != EPI_ADD_F32 && epi != EPI_SWIGLU)) return hipErrorInvalidValue;
  const float* a = (const float*)A;
  const float* w = (const float*)W;
#define BD_F32(G_, EPI_)                                                                                             \
  k_gemm_f32<G_, EPI_><<<dim3(N / FBN, cdiv(rows_cap, G_::BM)), G_::NT, 0, st>>>(a, lda, w, ldw, K, M_dev, (float*)out, \
                                                                                 ldo)
  if (f32_large(N, rows_cap)) {
    if (epi == EPI_ADD_F32) BD_F32(F32Large, EPI_ADD_F32); else BD_F32(F32Large, EPI_SWIGLU);
  } else {
    if (epi == EPI_ADD_F32) BD_F32(F32Small, EPI_ADD_F32); else BD_F32(F32Small, EPI_SWIGLU);
  }
#undef BD_F32
  return hipGetLastError();
}

hipError_t launch_gemm_qkv_f32(const void* A, int lda, const void* W, int K, const int32_t* M_dev, int rows_cap,
                               const QkvEpi& e, const double* inv_freq, hipStream_t st) {
  const int N = (e.H + 2 * e.Hkv) * e.hd;
  if (e.hd % FBN || K % 16) return hipErrorInvalidValue;
  const float* a = (const float*)A;
  const float* w = (const float*)W;
#define BD_QKV_F32(G_) \
  k_gemm_qkv_f32<G_><<<dim3(N / FBN, cdiv(rows_cap, G_::BM)), G_::NT, 0, st>>>(a, lda, w, K, M_dev, e, inv_freq)
  if (f32_large(N, rows_cap)) BD_QKV_F32(F32Large); else BD_QKV_F32(F32Small);
#undef BD_QKV_F32
  return hipGetLastError();
}

hipError_t launch_lm_head(bool is_bf16, const void* A, int d, size_t a_plane, const void* W, int V,
                          int mask_id, float scale, const int32_t* M_dev, int rows_cap,
                          float* part_max,
                          float* part_sum, int32_t* part_arg, float* conf, int32_t* tok,
                          const StepOut& so, hipStream_t st) {
  int ntiles;
  if (is_bf16) {
    if (V % 128 || d % KALIGN) return hipErrorInvalidValue;
    const bool wide = V % 256 == 0 && rows_cap >= 2048;
    // 64-row tiles where 128-row ones would leave CUs without one
    const bool low = !wide && (V / 128) * cdiv(rows_cap, 128) < 256;
    ntiles = V / (wide ? 256 : 128);
    dim3 grid(ntiles * cdiv(rows_cap, low ? 64 : 128) + 7);
#define BD_HEAD(G_, LOG_)                                                                                       \
  k_lm_head_bf16<G_, LOG_><<<grid, G_::NT, 0, st>>>((const bf16_t*)A, d, a_plane, (const bf16_t*)W, V, mask_id, scale, \
                                                    M_dev, rows_cap, part_max, part_sum, part_arg, so)
    if (wide) {
      if (so.logits) BD_HEAD(TileW2, true); else BD_HEAD(TileW2, false);
    } else if (low) {
      if (so.logits) BD_HEAD(Tile64x128<WQ_NONE>, true); else BD_HEAD(Tile64x128<WQ_NONE>, false);
    } else {
      if (so.logits) BD_HEAD(Tile128<WQ_NONE>, true); else BD_HEAD(Tile128<WQ_NONE>, false);
    }
#undef BD_HEAD
  } else {
    if (V % FHN || d % 16) return hipErrorInvalidValue;
    ntiles = V / FHN;
    const int tiles = cdiv(rows_cap, F32Head::BM);
    dim3 grid(ntiles, tiles < F32_HEAD_Y ? tiles : F32_HEAD_Y, cdiv(tiles, F32_HEAD_Y));
    k_lm_head_f32<<<grid, F32Head::NT, 0, st>>>((const float*)A, d, (const float*)W, mask_id, scale, M_dev,
                                       rows_cap, part_max, part_sum, part_arg, V, so);
  }
  k_lm_merge<<<cdiv(rows_cap, 4), 256, 0, st>>>(part_max, part_sum, part_arg, ntiles, M_dev, rows_cap,
                                                conf, tok, so);
  return hipGetLastError();
}

}  // namespace bd

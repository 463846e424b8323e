// Block-causal attention over the KV cache (paper §2.1): a query at absolute
// position p attends to every key j with j / B <= p / B, i.e. the cached
// prefix, every earlier block and its own block (bidirectionally).  Window
// K/V have already been written into the cache at their absolute positions,
// so one key range [0, end of the query's block) covers prefix and window.
//
// bf16 kernel (Q, K and V are bf16 hi/lo pairs in two planes; V is kept
// transposed in the cache, in tiles of 32 keys [dim][32 slots] in the slot
// order of vt_slot).  The queries of one (sequence, kv head) are its window
// rows x the q-heads that share the kv head; a wave takes 32 of them, a
// workgroup QW x KW waves: QW groups of 32 queries, the keys of every stage
// dealt to KW waves of each group.  A wave computes S^T = K Q^T and
// O^T += V^T P^T on tiles of 32 keys with MFMA 32x32x16 bf16 (three products
// hi.hi + hi.lo + lo.hi per pair of operands; the output leaves as the hi/lo
// pair of the next matmul operand), so each lane owns one query column and half
// of a tile's keys: softmax state and rescale stay in the lane (one exchange
// with lane ^ 32 per tile), and P^T is fed to the second MFMA straight from
// the score registers (the two products use the same permutation of the key
// index).  32 queries a wave are what keeps the kernel off the LDS bandwidth:
// every K or V fragment read from LDS serves 32 columns, 2 KiB of LDS reads per
// three MFMAs of 32 cycles; with 16 queries a wave and 16x16x32 MFMAs the reads
// took a third longer than the products they fed, and the softmax twice the
// vector instructions per score.
// Stages of 32 KW keys stream from HBM straight into LDS (two stages; buffer
// loads, no registers), the next one while a stage is consumed, one barrier a
// stage.  The block mask is applied in registers, only on tiles that reach the
// query's block.
#include "bd_internal.h"

#include <math.h>

namespace bd {

__device__ __forceinline__ float bf2f_a(bf16_t h) { return __uint_as_float(((uint32_t)h) << 16); }
__device__ __forceinline__ bf16_t f2bf_a(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (bf16_t)(u >> 16);
}

constexpr int AK = 32;    // keys per tile
// Fourth word of a raw buffer resource (gfx9 family): 32-bit data format (a
// zero format reads zeros), no index stride.
constexpr int ATT_BUF_DWORD3 = 0x00020000;

typedef __bf16 bf16x2_a __attribute__((ext_vector_type(2)));
typedef float floatx2_a __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) void att_lds_t;

// (x0, x1) -> the hi bf16 pair (round to nearest even, one v_cvt_pk_bf16_f32)
// in hi and the lo pair, the rounded remainders x - hi (exact in fp32), in lo
__device__ __forceinline__ void split_pair2(float x0, float x1, uint32_t& hi, uint32_t& lo) {
  hi = __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2_a){x0, x1}, bf16x2_a));
  const float h0 = __uint_as_float(hi << 16), h1 = __uint_as_float(hi & 0xFFFF0000u);
  lo = __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2_a){x0 - h0, x1 - h1}, bf16x2_a));
}

__device__ __forceinline__ void att_load_lds(__amdgpu_buffer_rsrc_t r, void* lds, uint32_t off, uint32_t soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (att_lds_t*)lds, 16, off, soff, 0, 0);
}

// K: [plane][key][HD], 16-byte chunk c of key r at c ^ k_swz(r); V:
// [plane][tile][dim][32 slots], chunk c of dim r at c ^ v_swz(r).  A 16-byte
// LDS read serves lanes 0-3, 12-15 and 20-27 together, then 4-11, 16-19 and
// 28-31, and so on 32 lanes up; rows being lanes, each such set of 16 meets 16
// distinct 16-byte columns of the 256 bytes that the banks span (the
// bank-conflict counter reads zero; with r & 7 and (r >> 1) & 3 it read half
// the active cycles).
template <int HD>
__device__ __forceinline__ int k_swz(int r) { return HD == 128 ? (r & 15) : ((r >> 1) & 7); }
__device__ __forceinline__ int v_swz(int r) { return (r >> 2) & 3; }
template <int HD, int KW>
struct AttStage {
  bf16_t k[2][KW * AK * HD];
  bf16_t v[2][KW * AK * HD];
};

template <int HD, int QW, int KW>
__global__ __launch_bounds__(64 * QW * KW) __attribute__((amdgpu_waves_per_eu(KW == 1 ? 2 : 1, 2)))
void k_attn_bf16(const int32_t* __restrict__ seq_win_len, const int32_t* __restrict__ seq_row_start,
                 const int32_t* __restrict__ seq_win_start, int b, int H, int Hkv, int kv_splits, int B, int maxpos,
                 const bf16_t* __restrict__ Kc, const bf16_t* __restrict__ Vt, const bf16_t* __restrict__ Q,
                 size_t k_plane, size_t v_plane, size_t q_plane, int vstride, float scale_log2,
                 bf16_t* __restrict__ O, size_t o_plane, float* __restrict__ ws_o, float* __restrict__ ws_ml,
                 int rows_cap) {
  constexpr int NW = QW * KW;
  constexpr int AQ = 32 * QW;             // queries per workgroup
  constexpr int SK = AK * KW;             // keys per stage
  constexpr int KCH = HD / 8;             // 16-byte chunks of a K row
  constexpr int LP = HD / 16 / QW;        // 1 KiB loads per wave, stage, operand and plane
  constexpr int NS = HD / 16;             // MFMA depths of the score product
  static_assert(LP >= 1, "every wave loads");
  typedef AttStage<HD, KW> Stage;
  __shared__ __attribute__((aligned(1024))) Stage st0, st1;

  // The queries of one (sequence s, kv head kv) are numbered qi = r * G + j
  // for window row r and q-head kv * G + j (G = H / Hkv heads share the kv
  // head); a workgroup takes AQ consecutive qi, so every K/V tile it stages
  // serves all G heads of the rows it covers.
  // Items u = ((s * Hkv + kv) * kv_splits + split) * nqt + qt: the nqt query
  // tiles that read the same keys are neighbours, so they share one XCD's L2.
  // nqt is counted from the longest window alive and not from the launch's
  // capacity (usually twice that): tiles without queries would otherwise stand
  // between the others and hold a CU's LDS until they have found out.
  // The windows' lengths, first rows and positions come in one round of loads,
  // one sequence a lane; past 64 sequences the workgroup reads its own again.
  const int G = H / Hkv;
  const int wl = threadIdx.x & 63;
  int nqt = 0, w_len = 0, w_row = 0, w_start = 0;
  if (wl < b) {
    nqt = w_len = seq_win_len[wl];
    w_row = seq_row_start[wl];
    w_start = seq_win_start[wl];
  }
  for (int i = wl + 64; i < b; i += 64) nqt = max(nqt, seq_win_len[i]);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) nqt = max(nqt, __shfl_xor(nqt, off));
  nqt = __builtin_amdgcn_readfirstlane((G * nqt + AQ - 1) / AQ);
  if (nqt == 0) return;
  const int items = b * Hkv * kv_splits * nqt;
  const int u = xcd_item(blockIdx.x, items);
  if (u >= items) return;
  const int qt = u % nqt, split = (u / nqt) % kv_splits;
  const int kv = (u / (nqt * kv_splits)) % Hkv, s = u / (nqt * kv_splits * Hkv);
  const int W = s < 64 ? __builtin_amdgcn_readlane(w_len, s) : seq_win_len[s];
  const int row_start = s < 64 ? __builtin_amdgcn_readlane(w_row, s) : seq_row_start[s];
  const int win_start = s < 64 ? __builtin_amdgcn_readlane(w_start, s) : seq_win_start[s];
  const int QG = G * W;
  if (qt * AQ >= QG) return;
  const int qlast = min(qt * AQ + AQ, QG) - 1;
  const int kend = ((win_start + qlast / G) / B + 1) * B;   // keys [0, kend): the last row's bound
  // this split's stages: a contiguous share of [0, kend)
  const int nst_all = (kend + SK - 1) / SK;
  const int per = (nst_all + kv_splits - 1) / kv_splits;
  const int t_lo = __builtin_amdgcn_readfirstlane(split * per);
  const int t_hi = __builtin_amdgcn_readfirstlane(min(nst_all, t_lo + per));
  const bf16_t* Kp = Kc + ((size_t)s * Hkv + kv) * (size_t)maxpos * HD;
  const bf16_t* Vp = Vt + ((size_t)s * Hkv + kv) * (size_t)HD * vstride;

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int qw = wave % QW, kw = wave / QW;
  const int h = lane >> 5, c = lane & 31;
  const int q0w = qt * AQ + qw * 32;                        // the wave's first query
  const int qi = q0w + c;                                   // this lane's query
  const bool qvalid = qi < QG;
  const bool wave_on = q0w < QG;                            // the wave holds a query
  const int qrow = row_start + (qvalid ? qi / G : 0);       // its row in the step
  const int hq = kv * G + (qvalid ? qi % G : 0);            // its q-head
  const int qend = ((win_start + (qvalid ? qi / G : 0)) / B + 1) * B;   // its key bound
  // the wave's smallest and largest key bound (query index and bound rise
  // together) and whether every lane holds a query: tiles below the smallest
  // skip the mask, tiles from the largest on are skipped
  const int qend_lo = ((win_start + min(q0w, QG - 1) / G) / B + 1) * B;
  const int qend_hi = ((win_start + min(q0w + 31, QG - 1) / G) / B + 1) * B;
  const bool full_w = q0w + 32 <= QG;

  floatx16 oacc[HD / 32];
#pragma unroll
  for (int t = 0; t < HD / 32; ++t) oacc[t] = floatx16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f,
                                                       0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_part = 0.f;

  // Stage loads: load n of an operand's plane fills its bytes [1024 n, +1024).
  // K rows past the bound repeat row kend - 1 and V tiles past it the last one
  // (finite values; every query masks those keys).
  const __amdgpu_buffer_rsrc_t rkh = __builtin_amdgcn_make_buffer_rsrc((void*)Kp, 0, -1, ATT_BUF_DWORD3);
  const __amdgpu_buffer_rsrc_t rkl = __builtin_amdgcn_make_buffer_rsrc((void*)(Kp + k_plane), 0, -1, ATT_BUF_DWORD3);
  const __amdgpu_buffer_rsrc_t rvh = __builtin_amdgcn_make_buffer_rsrc((void*)Vp, 0, -1, ATT_BUF_DWORD3);
  const __amdgpu_buffer_rsrc_t rvl = __builtin_amdgcn_make_buffer_rsrc((void*)(Vp + v_plane), 0, -1, ATT_BUF_DWORD3);
  int krow[LP], vtile[LP];
  uint32_t kchunk[LP], vin[LP];
#pragma unroll
  for (int i = 0; i < LP; ++i) {
    const int n = i * NW + wave;
    krow[i] = n * (64 / KCH) + lane / KCH;
    kchunk[i] = (uint32_t)(((lane % KCH) ^ k_swz<HD>(krow[i])) * 16);
    vtile[i] = n / (HD / 16);
    const int dim = (n % (HD / 16)) * 16 + (lane >> 2);
    vin[i] = (uint32_t)(dim * (AK * 2) + ((lane & 3) ^ v_swz(dim)) * 16);
  }
  auto issue = [&](Stage& sg, int t) {
    const int left = kend - 1 - t * SK;                     // last key of the range, from the stage's start
    const uint32_t so = (uint32_t)t * (SK * HD * 2);
#pragma unroll
    for (int i = 0; i < LP; ++i) {
      const int n = i * NW + wave;
      const uint32_t ko = (uint32_t)min(krow[i], left) * (HD * 2) + kchunk[i];
      const uint32_t vo = (uint32_t)min(vtile[i], left / AK) * (HD * AK * 2) + vin[i];
      att_load_lds(rkh, sg.k[0] + n * 512, ko, so);
      att_load_lds(rkl, sg.k[1] + n * 512, ko, so);
      att_load_lds(rvh, sg.v[0] + n * 512, vo, so);
      att_load_lds(rvl, sg.v[1] + n * 512, vo, so);
    }
  };
  if (t_lo < t_hi) {
    __builtin_amdgcn_s_waitcnt(0xC07F);
    issue(st0, t_lo);
  }
  // Q^T fragments (B operand of S^T = K Q^T): dims [16 x + 8 h, +8) of query c,
  // hi and lo halves (lanes without a query read the window's first and mask
  // every key)
  bf16x8 qh[NS], ql[NS];
  const bf16_t* qp = Q + ((size_t)qrow * H + hq) * HD + h * 8;
#pragma unroll
  for (int x = 0; x < NS; ++x) {
    qh[x] = __builtin_bit_cast(bf16x8, *(const u32x4*)(qp + x * 16));
    ql[x] = __builtin_bit_cast(bf16x8, *(const u32x4*)(qp + q_plane + x * 16));
  }
  const int ksw = k_swz<HD>(c), vsw = v_swz(c);
  auto compute = [&](const Stage& sg, int t) {
    const int k0 = t * SK + kw * AK;                        // the wave's tile
    if (!wave_on || k0 >= qend_hi) return;
    // S^T (keys k0 + 8 (i >> 2) + 4 h + (i & 3), query c): Kh.Qh + Kh.Ql + Kl.Qh
    const bf16_t* kh_ = sg.k[0] + (kw * AK + c) * HD;
    const bf16_t* kl_ = sg.k[1] + (kw * AK + c) * HD;
    floatx16 a = floatx16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int x = 0; x < NS; ++x) {
      const int off = ((2 * x + h) ^ ksw) * 8;
      const bf16x8 kh = __builtin_bit_cast(bf16x8, *(const u32x4*)(kh_ + off));
      const bf16x8 kl = __builtin_bit_cast(bf16x8, *(const u32x4*)(kl_ + off));
      a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kh, qh[x], a, 0, 0, 0);
      a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kh, ql[x], a, 0, 0, 0);
      a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kl, qh[x], a, 0, 0, 0);
    }
    // Scores stay unscaled until the exponent: the max of the raw scores
    // times the (positive) scale is the max of the scaled ones.  The mask
    // branch is wave-uniform.
    if (k0 + AK > qend_lo || !full_w) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int key = k0 + 8 * (i >> 2) + 4 * h + (i & 3);
        if (!qvalid || key >= qend) a[i] = -INFINITY;
      }
    }
    float tmax = a[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) tmax = fmaxf(tmax, a[i]);
    tmax = fmaxf(tmax, __shfl_xor(tmax, 32)) * scale_log2;
    // m_run is the reference the exponents are taken from: the running maximum
    // when it was last set.  It moves only when some lane's maximum has risen
    // by more than 2^8 over it (P then stays below 2^8, with the same relative
    // precision), which saves nearly every rescale of the output.
    if (__any(tmax > m_run + 8.0f)) {
      const float m_new = fmaxf(m_run, tmax);
      const float alpha = __builtin_amdgcn_exp2f(m_new == -INFINITY ? 0.f : m_run - m_new);
      m_run = m_new;
      l_part *= alpha;
#pragma unroll
      for (int d = 0; d < HD / 32; ++d) oacc[d] *= alpha;
    }
    const float m_ref = m_run == -INFINITY ? 0.f : m_run;
    // P^T as a hi/lo bf16 pair, two keys per 32-bit word.  v_exp_f32 is exp2
    // without the denormal-range scaling: terms below 2^-126 of the row max
    // contribute nothing at fp32 precision anyway
    uint32_t hw[8], lw[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float p0 = __builtin_amdgcn_exp2f(fmaf(a[2 * i], scale_log2, -m_ref));
      const float p1 = __builtin_amdgcn_exp2f(fmaf(a[2 * i + 1], scale_log2, -m_ref));
      l_part += p0;
      l_part += p1;
      split_pair2(p0, p1, hw[i], lw[i]);
    }
    // O^T += V^T P^T over 2 depths of 16 keys; k-slot 8 h + j of depth x <->
    // key 16 x + 8 (j >> 2) + 4 h + (j & 3), score registers 8 x + j, which the
    // V^T slot order (vt_slot) stores as slots 16 x + 8 h + j: one 16-byte read
    // per plane.  Vh.Ph + Vh.Pl + Vl.Ph
    const bf16_t* vh_ = sg.v[0] + (kw * HD + c) * AK;
    const bf16_t* vl_ = sg.v[1] + (kw * HD + c) * AK;
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      const bf16x8 ph = __builtin_bit_cast(bf16x8, u32x4{hw[4 * x], hw[4 * x + 1], hw[4 * x + 2], hw[4 * x + 3]});
      const bf16x8 pl = __builtin_bit_cast(bf16x8, u32x4{lw[4 * x], lw[4 * x + 1], lw[4 * x + 2], lw[4 * x + 3]});
      const int off = ((2 * x + h) ^ vsw) * 8;
#pragma unroll
      for (int d = 0; d < HD / 32; ++d) {
        const bf16x8 vh = __builtin_bit_cast(bf16x8, *(const u32x4*)(vh_ + d * 32 * AK + off));
        const bf16x8 vl = __builtin_bit_cast(bf16x8, *(const u32x4*)(vl_ + d * 32 * AK + off));
        oacc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vh, ph, oacc[d], 0, 0, 0);
        oacc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vh, pl, oacc[d], 0, 0, 0);
        oacc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vl, ph, oacc[d], 0, 0, 0);
      }
    }
  };
  // own loads of the stage landed, LDS reads of the other one retired; then
  // everyone's, and the other stage is free to refill
#define BD_ATT_STEP(CUR, NXT, T)                  \
  __builtin_amdgcn_s_waitcnt(0x0070);             \
  __builtin_amdgcn_s_barrier();                   \
  if ((T) + 1 < t_hi) issue(NXT, (T) + 1);        \
  compute(CUR, T);                                \
  if ((T) + 1 >= t_hi) break;
  if (t_lo < t_hi) {
    for (int t = t_lo;; t += 2) {
      BD_ATT_STEP(st0, st1, t)
      BD_ATT_STEP(st1, st0, t + 1)
    }
  }
#undef BD_ATT_STEP
  float l = l_part + __shfl_xor(l_part, 32);
  if constexpr (KW > 1) {
    // the query group's waves hand their results to its first, in wave order
    __shared__ float xm[KW - 1][QW][2][64];
    constexpr int XS = HD / 2 * 64;
    static_assert(sizeof(Stage) >= sizeof(float) * XS * QW * (KW - 1), "partials fit a stage");
    float* xo = (float*)&st0 + lane;                        // [KW - 1][QW][HD / 2 registers][64 lanes]
    __syncthreads();
    if (kw > 0) {
      float* w = xo + ((kw - 1) * QW + qw) * XS;
#pragma unroll
      for (int d = 0; d < HD / 32; ++d)
#pragma unroll
        for (int i = 0; i < 16; ++i) w[(d * 16 + i) * 64] = oacc[d][i];
      xm[kw - 1][qw][0][lane] = m_run;
      xm[kw - 1][qw][1][lane] = l;
    }
    __syncthreads();
    if (kw > 0) return;                                     // the rest is the first waves' own
    float mx = m_run;
#pragma unroll
    for (int k = 0; k < KW - 1; ++k) mx = fmaxf(mx, xm[k][qw][0][lane]);
    const float ref = mx == -INFINITY ? 0.f : mx;
    const float f0 = __builtin_amdgcn_exp2f(m_run - ref);
    l *= f0;
#pragma unroll
    for (int d = 0; d < HD / 32; ++d) oacc[d] *= f0;
#pragma unroll
    for (int k = 0; k < KW - 1; ++k) {
      const float* w = xo + (k * QW + qw) * XS;
      const float f = __builtin_amdgcn_exp2f(xm[k][qw][0][lane] - ref);
      l += f * xm[k][qw][1][lane];
#pragma unroll
      for (int d = 0; d < HD / 32; ++d)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[d][i] += f * w[(d * 16 + i) * 64];
    }
    m_run = mx;
  }
  // O^T block d: lane holds dims d * 32 + 8 j + 4 h + r (r < 4) of query c in
  // registers 4 j + r.  The wave turns its block round in LDS (its part of
  // stage 0, rows of HD floats, 16-byte chunk k of row r at k ^ (r & 15)) and
  // writes whole rows: from the registers each lane would write 8 or 16 bytes
  // of a row of its own.
  constexpr int OCH = HD / 4;                               // 16-byte chunks of a row
  static_assert(2 * sizeof(Stage) >= sizeof(float) * 32 * HD * QW && QW * KW <= 8, "output blocks fit the stages");
  if constexpr (KW == 1) __syncthreads();                   // every wave is past its last stage
  constexpr int PER = sizeof(Stage) / (sizeof(float) * 32 * HD);   // blocks per stage
  float* ob = (qw < PER ? (float*)&st0 + qw * 32 * HD : (float*)&st1 + (qw - PER) * 32 * HD);
  const float inv = kv_splits == 1 ? 1.0f / l : 1.0f;
#pragma unroll
  for (int d = 0; d < HD / 32; ++d)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      *(floatx4*)(ob + c * HD + (((d * 8 + 2 * j + h) ^ (c & 15)) * 4)) =
          floatx4{oacc[d][4 * j] * inv, oacc[d][4 * j + 1] * inv, oacc[d][4 * j + 2] * inv, oacc[d][4 * j + 3] * inv};
  if (kv_splits > 1 && h == 0 && qvalid) {
    const size_t base = ((size_t)split * rows_cap + qrow) * H + hq;
    ws_ml[2 * base] = m_run;
    ws_ml[2 * base + 1] = l;
  }
  __builtin_amdgcn_s_waitcnt(0xC07F);                       // the wave's own writes, then its reads
  __builtin_amdgcn_wave_barrier();
  if (kv_splits == 1) {
    constexpr int RPI = 64 / (HD / 8);                      // rows per pass, 8 dims a lane
#pragma unroll 2
    for (int r0 = 0; r0 < 32; r0 += RPI) {
      const int r = r0 + lane / (HD / 8), k = (lane % (HD / 8)) * 2, q = q0w + r;
      if (q >= QG) continue;
      const floatx4 x = *(const floatx4*)(ob + r * HD + ((k ^ (r & 15)) * 4));
      const floatx4 y = *(const floatx4*)(ob + r * HD + (((k + 1) ^ (r & 15)) * 4));
      u32x4 hi, lo;
      uint32_t hb, lb;
      split_pair2(x[0], x[1], hb, lb); hi[0] = hb; lo[0] = lb;
      split_pair2(x[2], x[3], hb, lb); hi[1] = hb; lo[1] = lb;
      split_pair2(y[0], y[1], hb, lb); hi[2] = hb; lo[2] = lb;
      split_pair2(y[2], y[3], hb, lb); hi[3] = hb; lo[3] = lb;
      bf16_t* o = O + ((size_t)(row_start + q / G) * H + kv * G + q % G) * HD + k * 4;
      *(u32x4*)o = hi;
      *(u32x4*)(o + o_plane) = lo;
    }
  } else {
    // unnormalised partial of this key split, merged by k_attn_merge
    constexpr int RPI = 64 / OCH;
#pragma unroll 2
    for (int r0 = 0; r0 < 32; r0 += RPI) {
      const int r = r0 + lane / OCH, k = lane % OCH, q = q0w + r;
      if (q >= QG) continue;
      *(floatx4*)(ws_o + (((size_t)split * rows_cap + row_start + q / G) * H + kv * G + q % G) * HD + k * 4) =
          *(const floatx4*)(ob + r * HD + ((k ^ (r & 15)) * 4));
    }
  }
}

// Merge of the key splits (fixed split order): O = sum_s 2^(m_s - M) O_s /
// sum_s 2^(m_s - M) l_s with M = max_s m_s (scores kept in log2 units).
// A workgroup of 256 threads takes 256 / (hd / 4) (row, head) items, each
// thread 4 consecutive dims of one item.
__global__ __launch_bounds__(256) void k_attn_merge(const float* __restrict__ ws_o,
                                                    const float* __restrict__ ws_ml, int kv_splits,
                                                    const int32_t* __restrict__ Mp, int H, int hd,
                                                    int rows_cap, bf16_t* __restrict__ O,
                                                    size_t o_plane) {
  const int tpi = hd / 4;                                   // threads per item
  const int item = blockIdx.x * (256 / tpi) + threadIdx.x / tpi;
  const int e0 = (threadIdx.x % tpi) * 4;
  const int r = item / H, h = item % H;
  if (r >= *Mp) return;
  float M = -INFINITY;
  for (int z = 0; z < kv_splits; ++z) M = fmaxf(M, ws_ml[2 * (((size_t)z * rows_cap + r) * H + h)]);
  float L = 0.f, acc[4] = {0.f, 0.f, 0.f, 0.f};
  for (int z = 0; z < kv_splits; ++z) {
    const size_t b = ((size_t)z * rows_cap + r) * H + h;
    const float m = ws_ml[2 * b];
    if (m == -INFINITY) continue;
    const float w = exp2f(m - M);
    L += w * ws_ml[2 * b + 1];
    const float4 o = *(const float4*)(ws_o + b * hd + e0);
    acc[0] += w * o.x; acc[1] += w * o.y; acc[2] += w * o.z; acc[3] += w * o.w;
  }
  bf16_t hb[4], lb[4];
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    const float y = acc[x] / L;
    hb[x] = f2bf_a(y);
    lb[x] = f2bf_a(y - bf2f_a(hb[x]));
  }
  bf16_t* orow = O + ((size_t)r * H + h) * hd + e0;
  *(uint2*)orow = make_uint2((uint32_t)hb[0] | ((uint32_t)hb[1] << 16), (uint32_t)hb[2] | ((uint32_t)hb[3] << 16));
  *(uint2*)(orow + o_plane) =
      make_uint2((uint32_t)lb[0] | ((uint32_t)lb[1] << 16), (uint32_t)lb[2] | ((uint32_t)lb[3] << 16));
}

// a * b, not fused into the sum that takes it
__device__ __forceinline__ float rounded_mul(float a, float b) {
#pragma clang fp contract(off)
  return a * b;
}

// fp32 models: a wave per (query row, head), keys in tiles of 64.  For the
// scores a lane owns a key: the products of its K row with the query (held in
// LDS) are summed over the binary tree of dim indices (i + 32, then 16, .. 1;
// two trees' values are first added for hd 128), and the running maximum,
// weights and rescale factors of the online softmax are then formed for all
// keys of the tile at once.  For P V a lane owns hd / 64 dims and walks the keys
// in order, every V row a coalesced load, the tile's all in flight at once.  The arithmetic is
// that of a wave walking the keys one by one (one butterfly sum and one rescale
// per key), which took 21 us for 36 keys, 4 rows x 4 heads, against 7.
template <int HD>
__global__ __launch_bounds__(256) void k_attn_f32(const float* __restrict__ Q,
                                                  const float* __restrict__ Kc,
                                                  const float* __restrict__ Vc,
                                                  float* __restrict__ O,
                                                  const int32_t* __restrict__ row_seq,
                                                  const int32_t* __restrict__ row_pos,
                                                  const int32_t* __restrict__ Mp, int H, int Hkv,
                                                  int maxpos, int B, float scale) {
  constexpr int PER = HD / 64;
  __shared__ __attribute__((aligned(16))) float sq_all[4][HD];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int item = blockIdx.x * 4 + wave;
  const int r = item / H, h = item % H;
  if (r >= *Mp) return;
  float* sq = sq_all[wave];
  const int s = row_seq[r], pos = row_pos[r];
  const int kend = (pos / B + 1) * B;
  const int kv = h / (H / Hkv);
  const float* Kp = Kc + ((size_t)s * Hkv + kv) * (size_t)maxpos * HD;
  const float* Vp = Vc + ((size_t)s * Hkv + kv) * (size_t)maxpos * HD;
#pragma unroll
  for (int e = 0; e < PER; ++e) sq[e * 64 + lane] = Q[((size_t)r * H + h) * HD + e * 64 + lane];
  __builtin_amdgcn_wave_barrier();
  float acc[PER], m = -INFINITY, l = 0.f;
#pragma unroll
  for (int e = 0; e < PER; ++e) acc[e] = 0.f;
  for (int k0 = 0; k0 < kend; k0 += 64) {
    const int n = kend - k0 < 64 ? kend - k0 : 64;
    const int key = k0 + (lane < n ? lane : n - 1);
    const float4* kr = (const float4*)(Kp + (size_t)key * HD);
    // this lane's dims of every V row of the tile, in flight from here on
    const float* vr = Vp + (size_t)k0 * HD + lane * PER;
    float v[64][PER];
#pragma unroll
    for (int j = 0; j < 64; ++j)
#pragma unroll
      for (int e = 0; e < PER; ++e) v[j][e] = j < n ? vr[(size_t)j * HD + e] : 0.f;
    float t[64];                       // one value per lane of a wave summing this key
#pragma unroll
    for (int x = 0; x < HD / 4; ++x) {
      const float4 kx = kr[x], qx = *(const float4*)(sq + 4 * x);
      if constexpr (PER == 1) {
        t[4 * x] = rounded_mul(qx.x, kx.x); t[4 * x + 1] = rounded_mul(qx.y, kx.y);
        t[4 * x + 2] = rounded_mul(qx.z, kx.z); t[4 * x + 3] = rounded_mul(qx.w, kx.w);
      } else {
        t[2 * x] = fmaf(qx.y, kx.y, rounded_mul(qx.x, kx.x));
        t[2 * x + 1] = fmaf(qx.w, kx.w, rounded_mul(qx.z, kx.z));
      }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
#pragma unroll
      for (int i = 0; i < off; ++i) t[i] += t[i + off];
    const float sc = lane < n ? t[0] * scale : -INFINITY;
    // running maximum up to and including each key, and before it
    float mi = sc;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const float o = __shfl_up(mi, off);
      if (lane >= off) mi = fmaxf(mi, o);
    }
    mi = fmaxf(mi, m);
    float mb = __shfl_up(mi, 1);
    if (lane == 0) mb = m;
    const float al = expf(mb - mi), pr = expf(fmaf(t[0], scale, -mi));   // keys past the last one are not walked
#pragma unroll
    for (int j0 = 0; j0 < 64; j0 += 8) {
      if (j0 >= n) break;              // wave-uniform, as below
#pragma unroll
      for (int j = j0; j < j0 + 8; ++j) {
        if (j >= n) break;
        const float a = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(al), j));
        const float p = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(pr), j));
        l = l * a + p;
#pragma unroll
        for (int e = 0; e < PER; ++e) acc[e] = fmaf(acc[e], a, p * v[j][e]);
      }
    }
    m = __shfl(mi, n - 1);
  }
  float* o = O + ((size_t)r * H + h) * HD;
#pragma unroll
  for (int e = 0; e < PER; ++e) o[lane * PER + e] = acc[e] / l;
}

// Query groups of 32 and waves over the keys per workgroup, and key splits, from
// the rows a window usually holds (rows_est; the grid covers the largest window).
// Tiles of 128 queries are the rule: every K and V fragment staged serves 4 waves.
//  * {2, 2} where a kv head's queries fill no more than half of one (512 rows of
//    16 heads of 64: step 1340 us against 1354 in tiles of 128) or where there are
//    so few tiles that the keys are split for them (96 rows of 16 heads over 1120
//    keys: 24-layer step 2836 us against 2877; {1, 2} 2876).
//  * {4, 1} else: two workgroups a CU (64 KB of LDS each at hd 128), whose loads
//    and products overlap freely (32 windows of 96 rows: 2-layer step 1728 us
//    against 1762 with two waves over the keys; 8 windows of 64: 431 against 437).
//  * {4, 2} where one workgroup a CU has a long range to itself and would leave
//    it a wave a SIMD (8 windows of 128 rows over 8320 keys: 927 against 974).
// The keys are split until every CU has a workgroup, while a split keeps 160
// keys: a split's partials are written and read at 4 bytes a value and merged by
// another launch (64 tiles over 1504 keys: step 431 us in 4 splits, 457 in 8;
// three windows of 32 rows over 256 keys: 239.3 unsplit, 240.1 in 2).
// A prefill's keys are not split; it takes the shape that a step with as many rows
// would.  With the shape that one split would give, one prompt of 1024 positions (4
// kv heads, three layers) took 640 us against 660, the other prefills tried (128 to
// 8192 positions, 1 to 16 prompts) the same or 1-9% more.
struct AttnShape {
  int qw, kw, splits;
};
static AttnShape attention_shape(int b, int rows_est, int H, int Hkv, int maxpos) {
  const int q = (H / Hkv) * rows_est;
  const int tiles = (q + 127) / 128 * Hkv * b;
  const bool small = q <= 64 || tiles <= 32;
  const int wgs = small ? (q + 63) / 64 * Hkv * b : tiles;
  int splits = 1;
  while (wgs * (splits + 1) <= 256 && maxpos / (splits + 1) >= 160 && splits < 16) ++splits;
  const int nst = (maxpos + 63) / 64, per = (nst + splits - 1) / splits;
  splits = (nst + per - 1) / per;                           // none of them empty in stages of 64
  if (small) return AttnShape{2, 2, splits};
  return AttnShape{4, wgs * splits <= 256 && maxpos / splits >= 1024 ? 2 : 1, splits};
}

int attention_splits(int b, int rows_est, int H, int Hkv, int maxpos) {
  return attention_shape(b, rows_est, H, Hkv, maxpos).splits;
}

hipError_t launch_attention(bool is_bf16, const void* Q, size_t q_plane, const KvView& kv,
                            void* O, size_t o_plane, PlanView plan, int b, int win_cap, int rows_est, int H,
                            int Hkv, int hd, int B, int kv_splits, float* ws_o, float* ws_ml,
                            int rows_cap, hipStream_t st) {
  if (is_bf16) {
    if (hd != 64 && hd != 128) return hipErrorInvalidValue;
    if (kv.vstride % 64 || kv.vstride < kv.maxpos) return hipErrorInvalidValue;
    const float scale_log2 = (float)(1.4426950408889634 / sqrt((double)hd));
    const bf16_t* q = (const bf16_t*)Q;
    const bf16_t* k = (const bf16_t*)kv.K;
    const bf16_t* v = (const bf16_t*)kv.V;
    if (kv_splits < 1 || (kv_splits > 1 && (!ws_o || !ws_ml))) return hipErrorInvalidValue;
    const AttnShape sh = attention_shape(b, rows_est, H, Hkv, kv.maxpos);
    const int nqt = ((H / Hkv) * win_cap + 32 * sh.qw - 1) / (32 * sh.qw);
    const int grid = b * Hkv * kv_splits * nqt + 7;
#define BD_ATTN(HD_, QW_, KW_)                                                                \
  k_attn_bf16<HD_, QW_, KW_><<<grid, 64 * QW_ * KW_, 0, st>>>(                                \
      plan.seq_win_len, plan.seq_row_start, plan.seq_win_start, b, H, Hkv, kv_splits, B,      \
      kv.maxpos, k, v, q, kv.k_plane, kv.v_plane, q_plane, kv.vstride, scale_log2,            \
      (bf16_t*)O, o_plane, ws_o, ws_ml, rows_cap)
    if (hd == 128) {
      if (sh.qw == 2) BD_ATTN(128, 2, 2);
      else if (sh.kw == 1) BD_ATTN(128, 4, 1);
      else BD_ATTN(128, 4, 2);
    } else {
      if (sh.qw == 2) BD_ATTN(64, 2, 2);
      else if (sh.kw == 1) BD_ATTN(64, 4, 1);
      else BD_ATTN(64, 4, 2);
    }
#undef BD_ATTN
    if (kv_splits > 1) {
      const int items_per_block = 256 / (hd / 4);
      k_attn_merge<<<(rows_cap * H + items_per_block - 1) / items_per_block, 256, 0, st>>>(
          ws_o, ws_ml, kv_splits, plan.hdr, H, hd, rows_cap, (bf16_t*)O, o_plane);
    }
  } else {
    if (hd != 64 && hd != 128) return hipErrorInvalidValue;
    const float scale = (float)(1.0 / sqrt((double)hd));
#define BD_ATTN_F32(HD_)                                                                                       \
  k_attn_f32<HD_><<<(rows_cap * H + 3) / 4, 256, 0, st>>>((const float*)Q, (const float*)kv.K, (const float*)kv.V, (float*)O, \
                                                plan.row_seq, plan.row_pos, plan.hdr, H, Hkv, kv.maxpos, B, scale)
    if (hd == 128) BD_ATTN_F32(128); else BD_ATTN_F32(64);
#undef BD_ATTN_F32
  }
  return hipGetLastError();
}

}  // namespace bd

// Mixture-of-experts FFN pieces: router (softmax, top-k, renormalised
// weights), deterministic expert dispatch, and the fixed-order combine.  The
// expert products themselves run in the grouped MFMA GEMM (bd_gemm.hip).
#include "bd_internal.h"

#include <math.h>

namespace bd {

typedef __attribute__((address_space(3))) void moe_lds_t;
__device__ __forceinline__ void moe_load_lds16(__amdgpu_buffer_rsrc_t r, void* lds, uint32_t off, uint32_t soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (moe_lds_t*)lds, 16, off, soff, 0, 0);
}
__device__ __forceinline__ void moe_load_lds4(__amdgpu_buffer_rsrc_t r, void* lds, uint32_t off, uint32_t soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (moe_lds_t*)lds, 4, off, soff, 0, 0);
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t moe_rsrc(const void* p) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, -1, 0x00020000);   // raw, 32-bit data format
}

// Reductions over the wave's 64 lanes by data-parallel moves between
// registers (rows of 16, then across them; the last lane ends with the result,
// which all lanes get).
template <int CTRL, class T>
__device__ __forceinline__ T dpp_move(T old, T x) {
  return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, old), __builtin_bit_cast(int, x),
                                                           CTRL, 0xf, 0xf, false));
}
template <class T, class F>
__device__ __forceinline__ T wave_reduce(T x, T id, F f) {
  x = f(x, dpp_move<0x111>(id, x));   // row_shr 1, 2, 4, 8
  x = f(x, dpp_move<0x112>(id, x));
  x = f(x, dpp_move<0x114>(id, x));
  x = f(x, dpp_move<0x118>(id, x));
  x = f(x, dpp_move<0x142>(id, x));   // row_bcast 15, 31
  x = f(x, dpp_move<0x143>(id, x));
  return __builtin_bit_cast(T, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), 63));
}
__device__ __forceinline__ float wave_max(float x) {
  return wave_reduce(x, -INFINITY, [](float a, float b) { return fmaxf(a, b); });
}
__device__ __forceinline__ float wave_sum(float x) {
  return wave_reduce(x, 0.f, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ uint32_t wave_umax(uint32_t x) {
  return wave_reduce(x, 0u, [](uint32_t a, uint32_t b) { return a > b ? a : b; });
}

// Router.  A workgroup takes 16 rows and all experts; each of its 8 waves takes
// an eighth of the depth, on the fp32 matrix cores (v_mfma_f32_16x16x4_f32: fp32
// operands and sums): the A operand is the row's activation pair summed in fp32
// (hi + lo), the B operand the fp32 router weights [E][d].  A wave streams its
// slice in chunks of 16 deep from global memory straight into LDS that is its own
// (no barriers; three stages, two in flight).  In MFMA step s of a chunk lane
// group g feeds depth 4 g + s; two accumulators take the even and the odd steps;
// the eight slices are summed in LDS in a fixed order (an fp32 sum of the same
// products in another order than the plain dot product).  Then a wave ends two
// rows at once: softmax over the E lanes, each lane's rank among them (lowest
// expert id first among equal probabilities), and weights renormalised over the
// chosen experts, summed in rank order.  Needs E <= 64 and d % 256 == 0.
// Reading operands from global memory in fragment order (a lane per row, 16 bytes
// of 64 different lines a load) and choosing by top_k wave-wide maxima it took
// 36 us for any number of rows up to 2048 (d 2048, 64 experts, top 8), now 20: 7
// of them matrix time, the rest the first loads' and the choice's latency.
constexpr int RR = 16;     // rows per workgroup
constexpr int RW = 8;      // waves, each with d / RW of the depth
constexpr int RC = 16;     // depth per chunk
struct RouterStage {
  float w[RW][64 * RC];    // 16-byte piece k of expert e at k ^ ((e >> 1) & 3): reads without bank conflicts
  bf16_t a[RW][2][RR * RC];   // hi, lo
};

__global__ __launch_bounds__(64 * RW) void k_router(const bf16_t* __restrict__ A, size_t a_plane, int d,
                                                    const float* __restrict__ Wr, int E, int topk,
                                                    const int32_t* __restrict__ Mp,
                                                    int32_t* __restrict__ top_e, float* __restrict__ top_w) {
  __shared__ __attribute__((aligned(1024))) RouterStage st0, st1, st2;
  const int M = *Mp;
  const int row0 = blockIdx.x * RR;
  if (row0 >= M) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, c = lane & 15;
  const int ks = d / RW, n = ks / RC;             // the wave's depth and its chunks (at least 2)
  // weights: 1 KB a load, 64 bytes of 16 experts; activations: 256 bytes a load, 32 of 8 rows.  Rows and experts past
  // the last repeat it (their logits are not used).
  const __amdgpu_buffer_rsrc_t rw = moe_rsrc(Wr + wave * ks);
  const bf16_t* ab = A + (size_t)row0 * d + wave * ks;
  const __amdgpu_buffer_rsrc_t rh = moe_rsrc(ab), rl = moe_rsrc(ab + a_plane);
  uint32_t wo[4], ao[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int e = 16 * i + (lane >> 2);
    wo[i] = ((uint32_t)min(e, E - 1) * d + 4 * ((lane & 3) ^ ((e >> 1) & 3))) * 4u;
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) ao[i] = (uint32_t)min(8 * i + (lane >> 3), M - 1 - row0) * d * 2u + (lane & 7) * 4u;
  // The waves start at different quarters of their slices: a row of weights is a multiple of 1 KB, so that a chunk's 64
  // rows lie in one L2 channel, and the slices of every fourth wave in the same one.
  const int rot = (wave >> 1) * n / 4;
  auto issue = [&](RouterStage& st, int t) {
    t = t + rot < n ? t + rot : t + rot - n;
#pragma unroll
    for (int i = 0; i < 4; ++i) moe_load_lds16(rw, st.w[wave] + i * 256, wo[i], (uint32_t)t * (RC * 4));
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      moe_load_lds4(rh, st.a[wave][0] + i * 128, ao[i], (uint32_t)t * (RC * 2));
      moe_load_lds4(rl, st.a[wave][1] + i * 128, ao[i], (uint32_t)t * (RC * 2));
    }
  };
  floatx4 acc[4][2];
#pragma unroll
  for (int i = 0; i < 4; ++i) acc[i][0] = acc[i][1] = floatx4{0.f, 0.f, 0.f, 0.f};
  // byte offsets of the lane's pieces (plain offsets from a stage: the compiler then knows which stage a read is of,
  // and waits for no other's loads)
  const uint32_t w_off = (wave * 64 * RC + c * RC + 4 * (g ^ ((c >> 1) & 3))) * sizeof(float);
  const uint32_t a_off = sizeof(st0.w) + (wave * 2 * RR * RC + c * RC + 4 * g) * sizeof(bf16_t);
  auto compute = [&](const RouterStage& st) {
    const u32x2 h = *(const u32x2*)((const char*)&st + a_off);
    const u32x2 l = *(const u32x2*)((const char*)&st + a_off + RR * RC * sizeof(bf16_t));
    const float a[4] = {__uint_as_float(h[0] << 16) + __uint_as_float(l[0] << 16),
                        __uint_as_float(h[0] & 0xFFFF0000u) + __uint_as_float(l[0] & 0xFFFF0000u),
                        __uint_as_float(h[1] << 16) + __uint_as_float(l[1] << 16),
                        __uint_as_float(h[1] & 0xFFFF0000u) + __uint_as_float(l[1] & 0xFFFF0000u)};
    floatx4 w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = *(const floatx4*)((const char*)&st + w_off + i * (16 * RC * 4));
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        acc[i][k & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[k], w[i][k], acc[i][k & 1], 0, 0, 0);
  };
  // chunk T landed (two younger ones, 8 loads each, may be in flight); once it is read its stage takes chunk T + 3
  // (past the end the last one again: the same number of loads in flight at every wait)
#define BD_ROUTER_STEP(ST, T)                                               \
  __builtin_amdgcn_s_waitcnt(0x4070);                                       \
  __builtin_amdgcn_wave_barrier();                                          \
  compute(ST);                                                              \
  __builtin_amdgcn_s_waitcnt(0xC07F);                                       \
  __builtin_amdgcn_wave_barrier();                                          \
  issue(ST, min((T) + 3, n - 1));
  issue(st0, 0);
  issue(st1, 1);
  issue(st2, min(2, n - 1));
  int t = 0;
  for (; t + 3 <= n; t += 3) {
    BD_ROUTER_STEP(st0, t)
    BD_ROUTER_STEP(st1, t + 1)
    BD_ROUTER_STEP(st2, t + 2)
  }
  __builtin_amdgcn_s_waitcnt(0x0070);
  __builtin_amdgcn_wave_barrier();
  if (t < n) compute(st0);
  if (t + 1 < n) compute(st1);
#undef BD_ROUTER_STEP
  __syncthreads();                                // every wave is past its stages
  float* sP = (float*)&st0;                        // [RW][RR][64]
  static_assert(sizeof(st0) >= sizeof(float) * RW * RR * 64, "the slices' sums fit a stage");
  // lane (g, c) holds the wave's slice of the logits of rows 4 g + j, expert 16 i + c
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) sP[(wave * RR + 4 * g + j) * 64 + 16 * i + c] = acc[i][0][j] + acc[i][1][j];
  __syncthreads();
  constexpr int RPW = RR / RW;                    // rows a wave ends
  float prob[RPW], chosen[RPW];
  uint32_t key[RPW];
  int rank[RPW];
#pragma unroll
  for (int r = 0; r < RPW; ++r) {
    const float* x = sP + (wave * RPW + r) * 64 + lane;
    float q[RW];
#pragma unroll
    for (int k = 0; k < RW; ++k) q[k] = x[k * RR * 64];
    const float lg = ((q[0] + q[1]) + (q[2] + q[3])) + ((q[4] + q[5]) + (q[6] + q[7]));
    const float mx = wave_max(lane < E ? lg : -INFINITY);
    const float p = lane < E ? expf(lg - mx) : 0.f;
    prob[r] = p / wave_sum(p);
    // a total order (not-a-number included, above all others) of the E experts, the lanes past them below it
    key[r] = lane < E ? (__float_as_uint(prob[r]) & 0x7FFFFFFFu) + 1 : 0;
    chosen[r] = 0.f;
    rank[r] = -1;
  }
  for (int j = 0; j < topk; ++j)
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
      const uint32_t best = wave_umax(key[r]);
      const int at = __builtin_ctzll(__ballot(key[r] == best));   // lowest expert id among equals
      chosen[r] += __uint_as_float(best - 1);
      if (lane == at) {
        rank[r] = j;
        key[r] = 0;
      }
    }
#pragma unroll
  for (int r = 0; r < RPW; ++r) {
    const int row = row0 + wave * RPW + r;
    if (row < M && rank[r] >= 0) {
      top_e[(size_t)row * topk + rank[r]] = lane;
      top_w[(size_t)row * topk + rank[r]] = prob[r] / chosen[r];
    }
  }
}

hipError_t launch_router(const void* A, size_t a_plane, int d, const float* Wr, int E, int topk,
                         const int32_t* M_dev, int rows_cap, int32_t* top_e, float* top_w,
                         hipStream_t st) {
  if (E > 64 || E < 1 || topk > E || topk < 1 || d < 256 || d % 256) return hipErrorInvalidValue;
  k_router<<<(rows_cap + RR - 1) / RR, 64 * RW, 0, st>>>((const bf16_t*)A, a_plane, d, Wr, E, topk, M_dev,
                                                         top_e, top_w);
  return hipGetLastError();
}

// Dispatch: one workgroup per expert.  Every workgroup histograms all
// assignments by expert in LDS (integer atomics: exact counts), which gives its
// expert's offset in the expert-sorted order and its tiles.  Each of its 16
// waves takes a contiguous share of the assignments, four a lane, counts its
// expert's in the same pass and, knowing the counts of the waves before it,
// writes them in (row, slot) order in a second: each expert's list is sorted by
// token row.  Two passes with three barriers: with a barrier pair for every 256
// assignments, 16384 of them (2048 rows, top 8) took 48 us, now 11.
__global__ __launch_bounds__(1024) void k_moe_scatter(const int32_t* __restrict__ top_e, int topk, int E,
                                                      const int32_t* __restrict__ Mp, MoeLists L) {
  __shared__ int hist[64];
  __shared__ int wcnt[16];
  const int e = blockIdx.x;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int n = *Mp * topk;
  const int share = ((n + 15) / 16 + 255) & ~255;           // a wave's assignments, whole groups of 256
  const int lo = wave * share + 4 * lane, hi = min(n, (wave + 1) * share);
  if (threadIdx.x < 64) hist[threadIdx.x] = 0;
  __syncthreads();
  // assignments i .. i + 3, -1 past the end
  auto load = [&](int i) {
    if (i + 3 < hi) return *(const int4*)(top_e + i);
    return make_int4(i < hi ? top_e[i] : -1, i + 1 < hi ? top_e[i + 1] : -1, i + 2 < hi ? top_e[i + 2] : -1, -1);
  };
  int mine = 0;
#pragma unroll 4
  for (int i = lo; i < hi; i += 256) {
    const int4 v = load(i);
    atomicAdd(&hist[v.x], 1);
    if (v.y >= 0) atomicAdd(&hist[v.y], 1);
    if (v.z >= 0) atomicAdd(&hist[v.z], 1);
    if (v.w >= 0) atomicAdd(&hist[v.w], 1);
    mine += (v.x == e) + (v.y == e) + (v.z == e) + (v.w == e);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mine += __shfl_xor(mine, off);
  if (lane == 0) wcnt[wave] = mine;
  __syncthreads();
  // counts and tiles of the experts, a lane each; sums over those before e
  const int cnt_l = hist[lane];                             // experts past E have none
  const int tiles_l = (cnt_l + GROUP_BM - 1) / GROUP_BM;
  int off = lane < e ? cnt_l : 0, toff = lane < e ? tiles_l : 0, total = tiles_l;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    off += __shfl_xor(off, o);
    toff += __shfl_xor(toff, o);
    total += __shfl_xor(total, o);
  }
  const int cnt = hist[e];
  if (threadIdx.x == 0) {
    L.e_cnt[e] = cnt;
    L.e_off[e] = off;
    if (e == 0) L.ntiles[0] = total;
  }
  for (int t = threadIdx.x; t * GROUP_BM < cnt; t += blockDim.x) {
    L.tile_e[toff + t] = e;
    L.tile_m0[toff + t] = t * GROUP_BM;
  }
  int pos = off;
  for (int w = 0; w < wave; ++w) pos += wcnt[w];
  const unsigned long long below = (1ull << lane) - 1ull;
  for (int i = lo - 4 * lane; i < hi; i += 256) {           // wave-uniform
    const int i0 = i + 4 * lane;
    const int4 v = load(i0);
    const bool m[4] = {v.x == e, v.y == e, v.z == e, v.w == e};
    int at = pos;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const unsigned long long bal = __ballot(m[j]);
      at += __popcll(bal & below);
      pos += __popcll(bal);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (m[j]) {
        L.list_row[at] = (i0 + j) / topk;
        L.pos_of[i0 + j] = at;
        ++at;
      }
  }
}

hipError_t launch_moe_dispatch(const int32_t* top_e, int topk, int E, const int32_t* M_dev,
                               const MoeLists& L, hipStream_t st) {
  if (E > 64) return hipErrorInvalidValue;
  k_moe_scatter<<<E, 1024, 0, st>>>(top_e, topk, E, M_dev, L);
  return hipGetLastError();
}

// X[row] += sum_j w_j Y[pos_j] over the row's top_k slots in rank order
// (fixed order); each thread 4 consecutive columns.
__global__ __launch_bounds__(256) void k_moe_combine(float* __restrict__ X, const float* __restrict__ Y,
                                                     const int32_t* __restrict__ pos_of,
                                                     const float* __restrict__ top_w, int topk, int d,
                                                     const int32_t* __restrict__ Mp) {
  const int row = blockIdx.y;
  if (row >= *Mp) return;
  const int c = (blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (c >= d) return;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int j = 0; j < topk; ++j) {
    const size_t k = (size_t)row * topk + j;
    const float w = top_w[k];
    const float4 y = *(const float4*)(Y + (size_t)pos_of[k] * d + c);
    acc.x += w * y.x; acc.y += w * y.y; acc.z += w * y.z; acc.w += w * y.w;
  }
  float4* x = (float4*)(X + (size_t)row * d + c);
  float4 v = *x;
  v.x += acc.x; v.y += acc.y; v.z += acc.z; v.w += acc.w;
  *x = v;
}

hipError_t launch_moe_combine(float* X, const float* Y, const int32_t* pos_of, const float* top_w,
                              int topk, int d, const int32_t* M_dev, int rows_cap, hipStream_t st) {
  if (d % 4) return hipErrorInvalidValue;
  k_moe_combine<<<dim3((d / 4 + 255) / 256, rows_cap), 256, 0, st>>>(X, Y, pos_of, top_w, topk, d, M_dev);
  return hipGetLastError();
}

}  // namespace bd

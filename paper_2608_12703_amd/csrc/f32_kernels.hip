// Float32 matrix products and attention on the float32 matrix instruction: the float32 model's
// path, and the products with float32 activations and bf16 weights.
//
// Every output element is reduced in a fixed order that does not depend on how many
// rows share the launch, so a row's result is the same alone or inside any batch.
#include "common.h"
#include "launch.h"
#include "row_stats.h"
#include "top2.h"

namespace ad {

// Workgroup barrier for LDS traffic only: this wave's LDS operations complete, its global
// loads stay in flight (__syncthreads would also wait for every outstanding load, which
// empties the prefetch rings below at every step).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt 0; vmcnt and expcnt not waited for
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// ---------------------------------------------------------------- GEMM
// C[m][n] = sum_k A[m][k] W[n][k] (+ bias[n]), A float32, W float32 or bf16 (converted
// exactly), K a multiple of 32, products and sums in float32 (v_mfma_f32_16x16x4_f32).
//
// A workgroup owns RT row tiles x CT column tiles of 16 x 16; its four waves take the four
// quarters of K and their sums merge through LDS in quarter order.  What bounds these
// products is latency (5 rows against 384 x 384 weights are 0.6 MB and 1.5 MFLOP), so K is
// cut where the chain of dependent matrix instructions is, and the operands go straight
// into registers D 32-wide steps ahead.  The quarters depend on K only.
//
// Against the vector-ALU product before it (32 x 64 tiles, one fma chain over K per output,
// operands through LDS), 5 rows, us per launch: 384 x 384 and 384 x 1536 36.9 -> 5.5 on average,
// QKV 22.2 -> 5.6, FFN-up 20.8 -> 4.6, the 51865-column LM head 35 -> 21 (3.8 TB/s); the four-layer
// model's round at batch 1 1223 -> 508 (321 with the argmax, attention and LayerNorm steps below),
// its encoder K/V of 1500 frames 120 -> 59.  Each sum has
// four shorter chains: the logits' error against 64 bits falls (1.2e-6 -> 0.7e-6).

constexpr int kKQ = 4;   // K quarters, one wave each

// Eight k of one row of a 32-wide step for lane group grp: with float32 weights k = 4 grp + j
// and 16 + 4 grp + j (each load takes 64 consecutive bytes of 16 rows), with bf16 weights
// k = 8 grp + j.  Both operands of a product use the same.
template <class S, class W>
struct FOperand;
template <class W>
struct FOperand<F32, W> {
  static constexpr bool kWide = sizeof(typename W::T) == 4;
  float4 x, y;
  static __device__ __forceinline__ int first(int grp) { return kWide ? grp * 4 : grp * 8; }
  __device__ __forceinline__ void load(const float* p) {
    x = *(const float4*)p;
    y = *(const float4*)(p + (kWide ? 16 : 4));
  }
  __device__ __forceinline__ void get(float (&v)[8]) const {
    v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
    v[4] = y.x; v[5] = y.y; v[6] = y.z; v[7] = y.w;
  }
};
template <>
struct FOperand<BF16, BF16> {
  uint4 x;
  static __device__ __forceinline__ int first(int grp) { return grp * 8; }
  __device__ __forceinline__ void load(const uint16_t* p) { x = *(const uint4*)p; }
  __device__ __forceinline__ void get(float (&v)[8]) const {
    const uint32_t u[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[2 * j] = bf16_to_f32(u[j] & 0xffff);
      v[2 * j + 1] = bf16_to_f32(u[j] >> 16);
    }
  }
};

// Where element (m, n) of the product goes.
template <class S, int EPI>
__device__ __forceinline__ void f32_epilogue(const EpiArgs& e, int m, int n, float v) {
  if (EPI == EPI_STORE) {
    e.out[(size_t)m * e.ldo + n] = v;
  } else if (EPI == EPI_RESID) {
    e.out[(size_t)m * e.ldo + n] += v;
  } else if (EPI == EPI_GELU) {
    e.out[(size_t)m * e.ldo + n] = 0.5f * v * (1.0f + erff(v * 0.70710678118654752f));
  } else if (EPI == EPI_QKV) {
    if (n < e.d) {
      e.out[(size_t)m * e.ldo + n] = v;
    } else {
      const RowDesc rd = e.rows[m];
      if (rd.seq >= 0) {
        const int c = n - e.d, kv = c / e.d, h = (c % e.d) / kHead, j = c % kHead;
        int pg = e.block_table[(size_t)rd.seq * e.pages_per_seq + rd.slot / kTile];
        pg = min(max(pg, 0), e.num_pages - 1);
        S::st((typename S::T*)e.cache,
              kv_tile_base(e.layer, kv, pg, h, e.num_pages, e.H) + tile_off(kv, rd.slot % kTile, j), v);
      }
    }
  }
}

// (SW: the operands swap places, so a lane's four sums run along the columns.  LN, float32 and
// RT = 1 only: A holds the rows before their LayerNorm; each wave takes the statistics of four
// of the 16 rows, and the rows are normalised as they enter the product.)
template <class S, int EPI, int RT, int CT, int D, bool SW = false, bool LN = false>
__device__ __forceinline__ void gemm_f32_tile(int M, int N, int K, const float* A, const typename S::T* W,
                                              const typename S::T* bias, const EpiArgs& e, int m0, int n0,
                                              f32x4 (*part)[RT * CT][kWave], const float* ln_g = nullptr,
                                              const float* ln_b = nullptr) {
  static_assert(!LN || (RT == 1 && sizeof(typename S::T) == 4), "one row tile of float32");
  const int lane = threadIdx.x & 63, c16 = lane & 15, grp = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int KB = K / 32, kb0 = (w * KB) / kKQ, kb1 = ((w + 1) * KB) / kKQ, kl = max(kb1 - 1, kb0);
  // the statistics' rows are requested first: loads return in order, so the operands below stay
  // in flight while the statistics are taken
  f32x4 xr[kRowParts];
  if constexpr (LN) {
    const float* row = A + (size_t)min(m0 + 4 * w + grp, M - 1) * K;
#pragma unroll
    for (int t = 0; t < kRowParts; ++t) xr[t] = row_part(row, K, c16, t);
    asm volatile("" ::: "memory");   // the operands' loads stay behind these
  }
  // rows and columns past the matrix read its last (those results are never stored)
  const float* pa[RT];
  const typename S::T* pw[CT];
#pragma unroll
  for (int r = 0; r < RT; ++r) pa[r] = A + (size_t)min(m0 + r * 16 + c16, M - 1) * K + FOperand<F32, S>::first(grp);
#pragma unroll
  for (int c = 0; c < CT; ++c) pw[c] = W + (size_t)min(n0 + c * 16 + c16, N - 1) * K + FOperand<S, S>::first(grp);
  struct Stage {
    FOperand<F32, S> a[RT];
    FOperand<S, S> w[CT];
    FOperand<F32, S> g, b;   // LN: the scale and shift of the same k
  };
  auto load = [&](Stage& st, int kb) __attribute__((always_inline)) {
    const int k = min(min(kb, kl), KB - 1) * 32;
#pragma unroll
    for (int c = 0; c < CT; ++c) st.w[c].load(pw[c] + k);
#pragma unroll
    for (int r = 0; r < RT; ++r) st.a[r].load(pa[r] + k);
    if constexpr (LN) {
      st.g.load(ln_g + FOperand<F32, S>::first(grp) + k);
      st.b.load(ln_b + FOperand<F32, S>::first(grp) + k);
    }
  };
  float2 rs{0.f, 1.f};
  f32x4 acc[RT][CT];
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int c = 0; c < CT; ++c) acc[r][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto mma = [&](const Stage& st) __attribute__((always_inline)) {
    float av[RT][8], wv[CT][8];
#pragma unroll
    for (int r = 0; r < RT; ++r) st.a[r].get(av[r]);
#pragma unroll
    for (int c = 0; c < CT; ++c) st.w[c].get(wv[c]);
    if constexpr (LN) {
      float gv[8], bv[8];
      st.g.get(gv);
      st.b.get(bv);
#pragma unroll
      for (int j = 0; j < 8; ++j) av[0][j] = normalised(av[0][j], rs, gv[j], bv[j]);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int c = 0; c < CT; ++c)
          acc[r][c] = SW ? __builtin_amdgcn_mfma_f32_16x16x4f32(wv[c][j], av[r][j], acc[r][c], 0, 0, 0)
                         : __builtin_amdgcn_mfma_f32_16x16x4f32(av[r][j], wv[c][j], acc[r][c], 0, 0, 0);
  };
  Stage st[D];
#pragma unroll
  for (int u = 0; u < D; ++u) load(st[u], kb0 + u);
  if constexpr (LN) {
    __shared__ float2 stats[16];
    __builtin_amdgcn_sched_barrier(0);
    const float2 q = row_stats(xr, K);
    if (c16 == 0) stats[4 * w + grp] = q;
    lds_barrier();
    rs = stats[c16];
  }
  int kb = kb0;
  for (int it = 0; it < (kb1 - kb0 - 1) / D; ++it) {
#pragma unroll
    for (int u = 0; u < D; ++u) {
      mma(st[u]);
      load(st[u], kb + D + u);
      __builtin_amdgcn_sched_barrier(0);
    }
    kb += D;
  }
#pragma unroll
  for (int u = 0; u < D; ++u)
    if (kb + u < kb1) mma(st[u]);

#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int c = 0; c < CT; ++c) part[w][r * CT + c][lane] = acc[r][c];
  lds_barrier();
  // the quarters in order; wave w finishes tiles w, w + 4, ...
  for (int t = w; t < RT * CT; t += kKQ) {
    f32x4 v = part[0][t][lane];
#pragma unroll
    for (int q = 1; q < kKQ; ++q) v += part[q][t][lane];
    if constexpr (EPI == EPI_XKV) {
      // 64 columns from n0 are one head's keys (SW: four lanes of a frame per lane) or values
      // (four frames of a lane): both are 16 contiguous bytes of the cache
      const int nx = n0 + (t % CT) * 16 + (SW ? grp * 4 : c16), m = m0 + (t / CT) * 16 + (SW ? c16 : grp * 4);
      const int kv = n0 >= e.d, h = (n0 - kv * e.d) / kHead, j = nx % kHead;
      f32x4 bv;
#pragma unroll
      for (int i = 0; i < 4; ++i) bv[i] = bias[SW ? nx + i : nx];
      if (m < M)
        *(f32x4*)((float*)e.cache + cross_base(e.layer, h, e.H, e.frames_cap) + cross_off(kv, m, j)) = v + bv;
      continue;
    }
    const int n = n0 + (t % CT) * 16 + c16;
    if constexpr (EPI == EPI_ARGMAX) {
      // the tile's top-2 per row, into the LDS place of this wave's own first quarter
      // (read above by this wave alone)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool fin = isfinite(v[i]), in = n < N;
        const Top2s u = t2_row16(Top2s{(in & fin) ? v[i] : -INFINITY, in ? n : 0x7fffffff, -INFINITY,
                                       (in & !fin) ? 1 : 0});
        if (c16 == 0)
          part[0][t][grp * 4 + i] = f32x4{u.v1, __int_as_float(u.i1), u.v2, __int_as_float(u.bad)};
        const int m = m0 + (t / CT) * 16 + grp * 4 + i;
        if (e.out && in && m < M) e.out[(size_t)m * e.ldo + n] = v[i];
      }
      continue;
    }
    if (n >= N) continue;
    const float bn = bias ? S::ld(bias, n) : 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int m = m0 + (t / CT) * 16 + grp * 4 + i;
      if (m < M) f32_epilogue<S, EPI>(e, m, n, v[i] + bn);
    }
  }
  if constexpr (EPI == EPI_ARGMAX) {   // the row's record of these 16 CT columns
    lds_barrier();
    for (int r = threadIdx.x; r < RT * 16; r += blockDim.x) {
      const int m = m0 + r;
      if (m >= M) continue;
      Top2s u{-INFINITY, 0x7fffffff, -INFINITY, 0};
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        const f32x4 p = part[0][(r / 16) * CT + c][r % 16];
        u = t2_merge(u, Top2s{p[0], __float_as_int(p[1]), p[2], __float_as_int(p[3])});
      }
      ((float4*)e.am_part)[(size_t)m * ((N + 63) / 64) + n0 / 64] =
          float4{u.v1, __int_as_float(u.i1), u.v2, __int_as_float(u.bad)};
    }
  }
}

template <class S, int EPI, int RT, int CT, int D>
__global__ void __launch_bounds__(256) gemm_f32_kernel(int M, int N, int K, const float* A,
                                                       const typename S::T* W, const typename S::T* bias,
                                                       EpiArgs e) {
  __shared__ f32x4 part[kKQ][RT * CT][kWave];
  gemm_f32_tile<S, EPI, RT, CT, D>(M, N, K, A, W, bias, e, blockIdx.y * RT * 16, blockIdx.x * CT * 16, part);
}

// The product of rows that it normalises itself (A: the residual stream, at most kRowStatsMax
// wide), where a LayerNorm launch of its own costs more than it computes: 5 rows of 384, the
// launch 3.9 us, the product 4.2-5.6 us alone and 5.0-6.2 us with its LayerNorm (statistics by a
// wave per four rows with 64-lane butterflies instead of 16 lanes per row: 7.3-8.5 us).
template <class S, int EPI, int D>
__global__ void __launch_bounds__(256) ln_gemm_f32_kernel(int M, int N, int K, const float* A, const float* g,
                                                          const float* b, const typename S::T* W,
                                                          const typename S::T* bias, EpiArgs e) {
  __shared__ f32x4 part[kKQ][1][kWave];
  gemm_f32_tile<S, EPI, 1, 1, D, false, true>(M, N, K, A, W, bias, e, blockIdx.y * 16, blockIdx.x * 16, part, g, b);
}

// Heads (the LM head, or several draft heads over the same rows: blockIdx.z) with the argmax
// epilogue: 64 columns per workgroup, one top-2 record per row.  The logits are stored only
// where the caller asks for them; the separate argmax pass over them took 22 us per call.
template <class S, int RT, int D>
__global__ void __launch_bounds__(256) head_f32_kernel(int M, int N, int K, const float* A,
                                                       const typename S::T* W, EpiArgs e) {
  __shared__ f32x4 part[kKQ][RT * 4][kWave];
  const int h = blockIdx.z;
  W += (size_t)h * N * K;
  e.am_part = (float4*)e.am_part + (size_t)h * M * ((N + 63) / 64);
  if (e.out) e.out += (size_t)h * M * N;
  gemm_f32_tile<S, EPI_ARGMAX, RT, 4, D>(M, N, K, A, W, nullptr, e, blockIdx.y * RT * 16, blockIdx.x * 64, part);
}

// The encoder K/V of several layers (blockIdx.z).
__global__ void __launch_bounds__(256) xkv_f32_kernel(int M, int N, int K, const float* A, XkvLayers lay,
                                                      EpiArgs e) {
  __shared__ f32x4 part[kKQ][16][kWave];
  const int li = blockIdx.z;
  e.layer = lay.first + li;
  const float *W = (const float*)lay.W[li], *b = (const float*)lay.bias[li];
  const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  if (n0 < e.d) gemm_f32_tile<F32, EPI_XKV, 4, 4, 2, true>(M, N, K, A, W, b, e, m0, n0, part);
  else gemm_f32_tile<F32, EPI_XKV, 4, 4, 2>(M, N, K, A, W, b, e, m0, n0, part);
}

// Tile: one 16 x 16 tile per workgroup while that fills the chip less than eight times over
// (the most waves for the least latency), else four column tiles and as many row tiles as
// there are, up to four (operand bytes per product fall with the tile).
template <int EPI>
void launch_gemm_f32(int M, int N, int K, const float* A, const void* W, const void* bias, const EpiArgs& e,
                     hipStream_t st) {
  const auto* w = (const float*)W;
  const auto* b = (const float*)bias;
  const int MT = (M + 15) / 16, NT = (N + 15) / 16;
  auto go = [&](auto kernel, int rt, int ct) {
    hipLaunchKernelGGL(kernel, dim3((NT + ct - 1) / ct, (MT + rt - 1) / rt), dim3(256), 0, st, M, N, K, A, w, b, e);
  };
  if ((long long)MT * NT <= 2048) go(gemm_f32_kernel<F32, EPI, 1, 1, 4>, 1, 1);
  else if (MT == 1) go(gemm_f32_kernel<F32, EPI, 1, 4, 3>, 1, 4);
  else if (MT == 2) go(gemm_f32_kernel<F32, EPI, 2, 4, 3>, 2, 4);
  else go(gemm_f32_kernel<F32, EPI, 4, 4, 2>, 4, 4);
}
template void launch_gemm_f32<EPI_STORE>(int, int, int, const float*, const void*, const void*, const EpiArgs&, hipStream_t);
template void launch_gemm_f32<EPI_RESID>(int, int, int, const float*, const void*, const void*, const EpiArgs&, hipStream_t);

// LayerNorm, then the product.  One launch where the product runs 16 x 16 tiles and a wave holds
// a row (each workgroup normalises its own 16 rows again, so larger tiles and wider rows keep
// the LayerNorm kernel and its float32 rows `ln`); the results are the same bits.  Past d 384 a
// wave's K quarter is longer than its ring of three steps and the repeated LayerNorms show: up to
// six row tiles only.  us a step of four layers, one launch / two: d 384, 16 rows 215 / 251, 128
// 295 / 331, 400 633 / 648; d 512, 16 rows 245 / 269, 80 324 / 328, 96 350 / 346, 128 392 / 379,
// 256 664 / 592.  (A model's parameters are 16-byte aligned.)
template <int EPI>
void launch_ln_gemm_f32(int M, int N, int K, const float* x, const void* g, const void* b, float* ln,
                        const void* W, const void* bias, const EpiArgs& e, hipStream_t st) {
  const int MT = (M + 15) / 16, NT = (N + 15) / 16;
  if ((long long)MT * NT > 2048 || K > kRowStatsMax || (K > 384 && MT > 6)) {
    launch_layernorm(M, K, x, g, b, ln, st);
    launch_gemm_f32<EPI>(M, N, K, ln, W, bias, e, st);
    return;
  }
  hipLaunchKernelGGL((ln_gemm_f32_kernel<F32, EPI, 3>), dim3(NT, MT), dim3(256), 0, st, M, N, K, x, (const float*)g,
                     (const float*)b, (const float*)W, (const float*)bias, e);
}
template void launch_ln_gemm_f32<EPI_STORE>(int, int, int, const float*, const void*, const void*, float*, const void*, const void*, const EpiArgs&, hipStream_t);
template void launch_ln_gemm_f32<EPI_GELU>(int, int, int, const float*, const void*, const void*, float*, const void*, const void*, const EpiArgs&, hipStream_t);
template void launch_ln_gemm_f32<EPI_QKV>(int, int, int, const float*, const void*, const void*, float*, const void*, const void*, const EpiArgs&, hipStream_t);

int f32_records(int N) { return (N + 63) / 64; }

template <class S>
void launch_f32_head_argmax(int heads, int M, int N, int K, const float* A, const void* W, void* am_part,
                            float* logits, hipStream_t st) {
  EpiArgs e{};
  e.am_part = am_part;
  e.out = logits;
  e.ldo = N;
  const int MT = (M + 15) / 16;
  auto go = [&](auto kernel, int rt) {
    hipLaunchKernelGGL(kernel, dim3(f32_records(N), (MT + rt - 1) / rt, heads), dim3(256), 0, st, M, N, K, A,
                       (const typename S::T*)W, e);
  };
  if (MT == 1) go(head_f32_kernel<S, 1, 3>, 1);
  else if (MT == 2) go(head_f32_kernel<S, 2, 3>, 2);
  else go(head_f32_kernel<S, 4, 2>, 4);
}
template void launch_f32_head_argmax<F32>(int, int, int, int, const float*, const void*, void*, float*, hipStream_t);
template void launch_f32_head_argmax<BF16>(int, int, int, int, const float*, const void*, void*, float*, hipStream_t);

void launch_xkv_f32(int M, int N, int K, const float* A, const XkvLayers& lay, int layers, const EpiArgs& e,
                    hipStream_t st) {
  hipLaunchKernelGGL(xkv_f32_kernel, dim3((N + 63) / 64, (M + 63) / 64, layers), dim3(256), 0, st, M, N, K, A, lay, e);
}

// ---------------------------------------------------------------- attention
// One workgroup per (head, sequence, group of kGroupKeys keys at absolute positions 0, 128,
// 256, ...), one 32-key block per wave, 16 queries at a time, on the float32 matrix
// instruction.  As in the bf16 kernels the scores are computed transposed, S^T = K Q^T, with
// key rows interleaved (row r of product tt is key 8 (r / 4) + 4 tt + r % 4 of the block), so a
// lane holds eight consecutive keys of one query and its probabilities are the operand of
// O^T = V^T P^T.  Every load of a wave's block goes out at once.  The waves' partials (max, sum,
// unnormalised output) merge in wave order and leave one per (row, head, group); a second
// kernel merges the groups in group order.  A key a query may not see gets probability 0 and
// value slots at or past the sequence's keys are zeroed, so stale cache slots never reach the
// output.
//
// Bound by latency: 5 rows x 1500 frames x 6 heads are 4.6 MB.  The vector-ALU kernel before
// (64-key chunks through LDS, dot products and value sums as chains of 64 fused multiply-adds
// per thread): cross-attention 18.0 -> 6.8 us, self-attention 11.3 -> 5.8 us per launch.

constexpr int kGroupKeys = 128;   // keys per workgroup
constexpr int kVPart = 2 + kHead;  // a partial: max, sum, 64 output lanes
constexpr int kMaxGroups = 16;     // of 2048 frames

template <bool CROSS>
__global__ void __launch_bounds__(256) attn_f32_kernel(int H, int d, int layer, const SeqDesc* seqs,
                                                       const float* q, float* apart, int G, const float* kv,
                                                       int num_pages, const int* block_table,
                                                       int pages_per_seq, int frames_cap,
                                                       const RowTree* tree) {
  constexpr int kW = kGroupKeys / 32, kORow = kHead + 4;
  __shared__ float pm[kW][16], pl[kW][16];
  __shared__ __align__(16) float po[kW][16][kORow];
  const int h = blockIdx.x, b = blockIdx.y, g = blockIdx.z, tid = threadIdx.x;
  const int w = tid >> 6, lane = tid & 63, c16 = lane & 15, grp = lane >> 4;
  const SeqDesc s = seqs[b];
  if (!s.valid) return;
  const int n_rows = s.k + 1, f0 = g * kGroupKeys + 32 * w;   // this wave's block
  for (int qg = 0; qg < n_rows; qg += 16) {
    const int nq = min(16, n_rows - qg);
    // cross-attention sees frames [wlo, whi) (all frames unless a window was given);
    // self-attention every committed key and the block rows in the query's row mask
    const int lo = CROSS ? s.wlo : 0;
    const int n_keys = CROSS ? s.whi : s.n + qg + nq;
    const bool active = f0 < n_keys && f0 + 32 > lo;
    float m = -INFINITY, l = 0.f;
    f32x4 o[4];
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (active) {
      // keys: this lane's key row of product tt, dims 16 grp .. + 15; values: dim 16 dt + c16,
      // keys 8 grp .. + 7
      const float *kp[2][2], *vp[4];   // [product][dim half]
      if (CROSS) {
        const float* base = kv + cross_base(layer, h, H, frames_cap) +
                            (size_t)((s.enc_off + f0) / kCrossBlock) * 2 * kCrossBlockElems + (grp * 16 + c16) * 8;
#pragma unroll
        for (int u = 0; u < 4; ++u) kp[u >> 1][u & 1] = base + u * 512;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) vp[dt] = base + kCrossBlockElems + dt * 512;
      } else {
        // (a tile past the last key's reads the last key's)
        auto page = [&](int t) {
          const int p = block_table[(size_t)b * pages_per_seq + min(f0 / kTile + t, (n_keys - 1) / kTile)];
          return min(max(p, 0), num_pages - 1);
        };
        const int pk = page(c16 >> 3), pv = page(grp >> 1);
        const float* kb = kv + kv_tile_base(layer, 0, pk, h, num_pages, H) +
                          (((c16 >> 2) & 1) * 8 + (c16 & 3)) * kHead + grp * 16;
        const float* vb = kv + kv_tile_base(layer, 1, pv, h, num_pages, H) + c16 * kTile + (grp & 1) * 8;
#pragma unroll
        for (int u = 0; u < 4; ++u) kp[u >> 1][u & 1] = kb + (u >> 1) * 4 * kHead + (u & 1) * 8;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) vp[dt] = vb + dt * 16 * kTile;
      }
      const float* qp = q + (size_t)(s.row0 + qg + min(c16, nq - 1)) * d + h * kHead + grp * 16;
      f32x4 kf[2][4], vf[4][2], qf[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) qf[u] = *(const f32x4*)(qp + 4 * u);
#pragma unroll
      for (int tt = 0; tt < 2; ++tt)
#pragma unroll
        for (int u = 0; u < 4; ++u) kf[tt][u] = *(const f32x4*)(kp[tt][u >> 1] + (u & 1) * 4);
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int u = 0; u < 2; ++u) vf[dt][u] = *(const f32x4*)(vp[dt] + 4 * u);
      const unsigned long long tm = CROSS ? 0ull : tree[s.row0 + qg + min(c16, nq - 1)].mask;

      f32x4 st[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int j = 0; j < 16; ++j)
#pragma unroll
        for (int tt = 0; tt < 2; ++tt)
          st[tt] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[tt][j >> 2][j & 3], qf[j >> 2][j & 3], st[tt], 0, 0, 0);
      const int key0 = f0 + grp * 8;   // score e of this lane: key key0 + e
      float sv[8], mx = -INFINITY;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int t = key0 + e;
        const bool see = CROSS ? (t >= lo && t < n_keys) : (t < s.n || (t < n_keys && ((tm >> ((t - s.n) & 63)) & 1)));
        sv[e] = see ? st[e >> 2][e & 3] * 0.125f : -INFINITY;
        mx = fmaxf(mx, sv[e]);
      }
      m = rows4_max(mx);
      float p[8], ps = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        p[e] = sv[e] == -INFINITY ? 0.f : expf(sv[e] - m);
        ps += p[e];
      }
      l = rows4_sum(ps);
#pragma unroll
      for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
          o[dt] = __builtin_amdgcn_mfma_f32_16x16x4f32(key0 + e < n_keys ? vf[dt][e >> 2][e & 3] : 0.f, p[e], o[dt], 0, 0, 0);
    }
    if (qg) lds_barrier();   // the last group's partials have been read
    if (grp == 0) {
      pm[w][c16] = m;
      pl[w][c16] = l;
    }
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) *(f32x4*)&po[w][c16][dt * 16 + grp * 4] = o[dt];
    lds_barrier();
    // query tid / 16, dims 4 (tid % 16) .. + 3: the blocks in order
    const int qi = tid >> 4, d4 = (tid & 15) * 4;
    if (qi < nq) {
      float M = pm[0][qi];
#pragma unroll
      for (int u = 1; u < kW; ++u) M = fmaxf(M, pm[u][qi]);
      float L = 0.f;
      f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int u = 0; u < kW; ++u) {
        const float wt = pm[u][qi] == -INFINITY ? 0.f : expf(pm[u][qi] - M);
        L += wt * pl[u][qi];
        acc += *(const f32x4*)&po[u][qi][d4] * wt;
      }
      float* pp = apart + (((size_t)(s.row0 + qg + qi) * H + h) * G + g) * kVPart;
      if (d4 == 0) {
        pp[0] = M;
        pp[1] = L;
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) pp[2 + d4 + i] = acc[i];
    }
  }
}

// Merge the G key groups of every (row, head) in group order: out = sum_g e^(m_g - M)
// o_g / sum_g e^(m_g - M) l_g with M = max_g m_g.  Rows of no sequence, or of a sequence
// the step skips, are left alone (as the attention kernel leaves them).
__global__ void __launch_bounds__(64) attn_merge_kernel(int H, int d, int G, const SeqDesc* seqs,
                                                        const RowDesc* rows, const float* part, float* out) {
  const int m = blockIdx.x, h = blockIdx.y, j = threadIdx.x;
  const int sq = rows[m].seq;
  if (sq < 0 || !seqs[sq].valid) return;
  const float* pp = part + ((size_t)m * H + h) * G * kVPart;
  // every group's partial requested before any is used (2048 frames are 16 groups)
  float mg[kMaxGroups], lg[kMaxGroups], og[kMaxGroups];
#pragma unroll
  for (int g = 0; g < kMaxGroups; ++g) {
    const float* p = pp + min(g, G - 1) * kVPart;
    mg[g] = p[0];
    lg[g] = p[1];
    og[g] = p[2 + j];
  }
  float M = -INFINITY;
#pragma unroll
  for (int g = 0; g < kMaxGroups; ++g) M = fmaxf(M, mg[g]);
  float L = 0.f, acc = 0.f;
#pragma unroll
  for (int g = 0; g < kMaxGroups; ++g) {
    const float w = (g >= G || mg[g] == -INFINITY) ? 0.f : expf(mg[g] - M);
    if (g < G) {
      L += w * lg[g];
      acc += w * og[g];
    }
  }
  out[(size_t)m * d + h * kHead + j] = acc / L;
}

int attn_f32_groups(int max_keys) { return (max_keys + kGroupKeys - 1) / kGroupKeys; }

void launch_self_attn_f32(int B, int M, int H, int d, int layer, const SeqDesc* seqs, const RowDesc* rows,
                          const float* q, float* part, int G, float* out, const void* pool, int num_pages,
                          const int* block_table, int pages_per_seq, const RowTree* tree, hipStream_t st) {
  hipLaunchKernelGGL(attn_f32_kernel<false>, dim3(H, B, G), dim3(256), 0, st, H, d, layer, seqs, q, part, G,
                     (const float*)pool, num_pages, block_table, pages_per_seq, 0, tree);
  hipLaunchKernelGGL(attn_merge_kernel, dim3(M, H), dim3(64), 0, st, H, d, G, seqs, rows, part, out);
}
void launch_cross_attn_f32(int B, int M, int H, int d, int layer, const SeqDesc* seqs, const RowDesc* rows,
                           const float* q, float* part, int G, float* out, const void* cross, int frames_cap,
                           hipStream_t st) {
  hipLaunchKernelGGL(attn_f32_kernel<true>, dim3(H, B, G), dim3(256), 0, st, H, d, layer, seqs, q, part, G,
                     (const float*)cross, 0, nullptr, 0, frames_cap, nullptr);
  hipLaunchKernelGGL(attn_merge_kernel, dim3(M, H), dim3(64), 0, st, H, d, G, seqs, rows, part, out);
}

}  // namespace ad

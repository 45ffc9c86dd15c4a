// Float32 matrix products (on the float32 matrix instruction) and float32 attention (vector
// ALU): the float32 model's path, and the products with float32 activations and bf16 weights.
//
// Every output element is reduced in a fixed order that does not depend on how many
// rows share the launch, so a row's result is the same alone or inside any batch.
#include "common.h"
#include "launch.h"

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
// model's round at batch 1 1223 -> 508, its encoder K/V of 1500 frames 120 -> 59.  Each sum has
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

// (SW: the operands swap places, so a lane's four sums run along the columns)
template <class S, int EPI, int RT, int CT, int D, bool SW = false>
__device__ __forceinline__ void gemm_f32_tile(int M, int N, int K, const float* A, const typename S::T* W,
                                              const typename S::T* bias, const EpiArgs& e, int m0, int n0,
                                              f32x4 (*part)[RT * CT][kWave]) {
  const int lane = threadIdx.x & 63, c16 = lane & 15, grp = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int KB = K / 32, kb0 = (w * KB) / kKQ, kb1 = ((w + 1) * KB) / kKQ, kl = max(kb1 - 1, kb0);
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
  };
  auto load = [&](Stage& st, int kb) __attribute__((always_inline)) {
    const int k = min(min(kb, kl), KB - 1) * 32;
#pragma unroll
    for (int c = 0; c < CT; ++c) st.w[c].load(pw[c] + k);
#pragma unroll
    for (int r = 0; r < RT; ++r) st.a[r].load(pa[r] + k);
  };
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
template <class S, int EPI>
static void launch_f32(int M, int N, int K, const float* A, const void* W, const void* bias, const EpiArgs& e,
                       hipStream_t st) {
  const auto* w = (const typename S::T*)W;
  const auto* b = (const typename S::T*)bias;
  const int MT = (M + 15) / 16, NT = (N + 15) / 16;
  auto go = [&](auto kernel, int rt, int ct) {
    hipLaunchKernelGGL(kernel, dim3((NT + ct - 1) / ct, (MT + rt - 1) / rt), dim3(256), 0, st, M, N, K, A, w, b, e);
  };
  if ((long long)MT * NT <= 2048) go(gemm_f32_kernel<S, EPI, 1, 1, 4>, 1, 1);
  else if (MT == 1) go(gemm_f32_kernel<S, EPI, 1, 4, 3>, 1, 4);
  else if (MT == 2) go(gemm_f32_kernel<S, EPI, 2, 4, 3>, 2, 4);
  else go(gemm_f32_kernel<S, EPI, 4, 4, 2>, 4, 4);
}

template <class S>
void launch_gemm_f32(int epi, int M, int N, int K, const float* A, const void* W, const void* bias,
                     const EpiArgs& e, hipStream_t st) {
  if (epi == EPI_STORE) launch_f32<S, EPI_STORE>(M, N, K, A, W, bias, e, st);
  else if (epi == EPI_RESID) launch_f32<S, EPI_RESID>(M, N, K, A, W, bias, e, st);
  else if (epi == EPI_GELU) launch_f32<S, EPI_GELU>(M, N, K, A, W, bias, e, st);
  else if (epi == EPI_QKV) launch_f32<S, EPI_QKV>(M, N, K, A, W, bias, e, st);
}
template void launch_gemm_f32<F32>(int, int, int, int, const float*, const void*, const void*, const EpiArgs&, hipStream_t);

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
// One block per (head, sequence, group of kVGroupKeys keys at absolute positions 0, 128,
// 256, ...).  Queries are taken 16 at a time; a group's keys stream through LDS in
// chunks of 64 with an online softmax per query, which leaves a partial (max, sum,
// unnormalised output) per (row, head, group); a second kernel merges the groups in
// group order.  A key a query may not see contributes exp(-inf) = 0; keys past every query's
// range are staged as zeros so stale cache slots never reach the output.  Every thread
// requests its part of a chunk (two runs of 8 keys' lanes and two runs of 8 values of
// one lane, contiguous in both cache layouts) kAStages chunks ahead into registers.

constexpr int kAStages = 4;
constexpr int kVGroupKeys = 128;   // keys per workgroup
constexpr int kVPart = 2 + kHead;  // a partial: max, sum, 64 output lanes
constexpr int kVMaxGroups = 16;    // of 2048 frames

template <class S>
struct AStage;
template <>
struct AStage<F32> {
  float4 k[2][2], v[2][2];
};
template <>
struct AStage<BF16> {
  uint4 k[2], v[2];
};

// Load chunk c0 (keys c0 .. c0 + 63): piece u of this thread is key run (key tid / 8 +
// 32 u, lanes 8 (tid % 8) ..) and value run (lane tid / 8 + 32 u, keys c0 + 8 (tid % 8) ..).
// Keys at or past n_keys read the last key's place (the values become zeros in LDS).
template <class S, bool CROSS>
__device__ __forceinline__ void astage_load(AStage<S>& st, int c0, int n_keys, int layer, int h, int H,
                                            int b, const SeqDesc& s, const typename S::T* kv,
                                            int num_pages, const int* block_table, int pages_per_seq,
                                            int frames_cap, int tid) {
  constexpr bool F = sizeof(typename S::T) == 4;
  const int last = max(n_keys - 1, 0);
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int tk = c0 + (tid >> 3) + 32 * u, jk = (tid & 7) * 8;   // key run
    const int jv = (tid >> 3) + 32 * u, tv = c0 + (tid & 7) * 8;   // value run
    size_t bk = 0, bv = 0;
    if (CROSS) {
      bk = cross_base(layer, h, H, frames_cap) + cross_off(0, s.enc_off + min(tk, last), jk);
      bv = cross_base(layer, h, H, frames_cap) + cross_off(1, s.enc_off + min(tv, last) / 8 * 8, jv);
    } else {
      const int pk = min(max(block_table[(size_t)b * pages_per_seq + min(tk, last) / kTile], 0), num_pages - 1);
      const int pv = min(max(block_table[(size_t)b * pages_per_seq + min(tv, last) / kTile], 0), num_pages - 1);
      bk = kv_tile_base(layer, 0, pk, h, num_pages, H) + tile_off(0, min(tk, last) % kTile, jk);
      bv = kv_tile_base(layer, 1, pv, h, num_pages, H) + tile_off(1, min(tv, last) / 8 * 8 % kTile, jv);
    }
    if constexpr (F) {
      st.k[u][0] = *(const float4*)(kv + bk);
      st.k[u][1] = *(const float4*)(kv + bk + 4);
      st.v[u][0] = *(const float4*)(kv + bv);
      st.v[u][1] = *(const float4*)(kv + bv + 4);
    } else {
      st.k[u] = *(const uint4*)(kv + bk);
      st.v[u] = *(const uint4*)(kv + bv);
    }
  }
}

// Chunk c0's registers into LDS: ks[key][lane], vs[key][lane]; key and value slots at
// or past n_keys are zeroed.
template <class S>
__device__ __forceinline__ void astage_put(const AStage<S>& st, int c0, int n_keys, float (*ks)[65],
                                           float (*vs)[65], int tid) {
  constexpr bool F = sizeof(typename S::T) == 4;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int rk = (tid >> 3) + 32 * u, jk = (tid & 7) * 8;
    const int jv = (tid >> 3) + 32 * u, rv = (tid & 7) * 8;
    float kx[8], vx[8];
    if constexpr (F) {
      const float4 a = st.k[u][0], bq = st.k[u][1], c = st.v[u][0], dq = st.v[u][1];
      kx[0] = a.x; kx[1] = a.y; kx[2] = a.z; kx[3] = a.w; kx[4] = bq.x; kx[5] = bq.y; kx[6] = bq.z; kx[7] = bq.w;
      vx[0] = c.x; vx[1] = c.y; vx[2] = c.z; vx[3] = c.w; vx[4] = dq.x; vx[5] = dq.y; vx[6] = dq.z; vx[7] = dq.w;
    } else {
      const uint32_t ku[4] = {st.k[u].x, st.k[u].y, st.k[u].z, st.k[u].w};
      const uint32_t vu[4] = {st.v[u].x, st.v[u].y, st.v[u].z, st.v[u].w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        kx[2 * j] = bf16_to_f32(ku[j] & 0xffff);
        kx[2 * j + 1] = bf16_to_f32(ku[j] >> 16);
        vx[2 * j] = bf16_to_f32(vu[j] & 0xffff);
        vx[2 * j + 1] = bf16_to_f32(vu[j] >> 16);
      }
    }
    const bool kin = c0 + rk < n_keys;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      ks[rk][jk + e] = kin ? kx[e] : 0.f;
      vs[rv + e][jv] = (c0 + rv + e < n_keys) ? vx[e] : 0.f;
    }
  }
}

template <class S, bool CROSS>
__global__ void __launch_bounds__(256) attn_valu_kernel(int H, int d, int layer,
                                                        const SeqDesc* seqs, const float* q,
                                                        float* apart, int G, const typename S::T* kv,
                                                        int num_pages, const int* block_table,
                                                        int pages_per_seq, int frames_cap,
                                                        const RowTree* tree) {
  __shared__ float qs[16][65];
  __shared__ float ks[64][65];
  __shared__ float vs[64][65];
  __shared__ float ps[16][65];
  const int h = blockIdx.x, b = blockIdx.y, g = blockIdx.z, tid = threadIdx.x;
  const SeqDesc s = seqs[b];
  if (!s.valid) return;
  const int qi = tid >> 4, part = tid & 15;
  const int n_rows = s.k + 1;
  for (int qg = 0; qg < n_rows; qg += 16) {
    const int nq = min(16, n_rows - qg);
    lds_barrier();
    for (int i = tid; i < 16 * 64; i += 256) {
      const int r = i >> 6, j = i & 63;
      qs[r][j] = r < nq ? q[(size_t)(s.row0 + qg + r) * d + h * kHead + j] : 0.f;
    }
    // cross-attention sees frames [wlo, whi) (all frames unless a window was given);
    // self-attention every committed key and the block rows in the query's row mask
    const int lo = CROSS ? s.wlo : 0;
    const unsigned long long tm = (!CROSS && qi < nq) ? tree[s.row0 + qg + qi].mask : 0ull;
    const int n_keys = CROSS ? s.whi : s.n + qg + nq;
    float m_run = -INFINITY, l_run = 0.f, o[4] = {0.f, 0.f, 0.f, 0.f};
    // this group's chunks: keys [max(lo, 128 g), min(128 (g + 1), n_keys)), 64-aligned
    const int c_first = max(lo / 64 * 64, g * kVGroupKeys);
    const int c_end = min((g + 1) * kVGroupKeys, n_keys);
    const int nch = c_end > c_first ? (c_end - c_first + 63) / 64 : 0;
    AStage<S> st0, st1, st2, st3;
    // (chunks past the last one reread it; nch >= 1 whenever the loop runs)
    auto load = [&](AStage<S>& st, int ci) {
      astage_load<S, CROSS>(st, c_first + min(ci, max(nch - 1, 0)) * 64, n_keys, layer, h, H, b, s, kv,
                            num_pages, block_table, pages_per_seq, frames_cap, tid);
    };
    load(st0, 0);
    load(st1, 1);
    load(st2, 2);
    load(st3, 3);
    // the scores, the online-softmax update and the value product of chunk c0 (in LDS)
    auto attend = [&](int c0) __attribute__((always_inline)) {
      float sc[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int key = part + 16 * u;
        float acc = 0.f;
#pragma unroll 16
        for (int j = 0; j < 64; ++j) acc = fmaf(qs[qi][j], ks[key][j], acc);
        const int t = c0 + key;
        const bool see = CROSS ? (t >= lo && t < n_keys)
                               : (t < s.n || (t < n_keys && ((tm >> (t - s.n)) & 1)));
        sc[u] = (see && qi < nq) ? acc * 0.125f : -INFINITY;
      }
      float cm = fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3]));
#pragma unroll
      for (int off = 8; off >= 1; off >>= 1) cm = fmaxf(cm, __shfl_xor(cm, off, kWave));
      const float m_new = fmaxf(m_run, cm);
      const float scale = (m_new == -INFINITY) ? 1.f : expf(m_run - m_new);
      float ls = 0.f;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const float p = (sc[u] == -INFINITY) ? 0.f : expf(sc[u] - m_new);
        ps[qi][part + 16 * u] = p;
        ls += p;
      }
#pragma unroll
      for (int off = 8; off >= 1; off >>= 1) ls += __shfl_xor(ls, off, kWave);
      l_run = l_run * scale + ls;
      m_run = m_new;
      lds_barrier();
#pragma unroll
      for (int r = 0; r < 4; ++r) o[r] *= scale;
      for (int key = 0; key < 64; ++key) {
        const float p = ps[qi][key];
#pragma unroll
        for (int r = 0; r < 4; ++r) o[r] = fmaf(p, vs[key][part * 4 + r], o[r]);
      }
    };
    // chunk ci of the ring slot ST: stage it in LDS, request chunk ci + kAStages into the
    // freed registers, attend
#define VATT_CHUNK(ST, J)                                  \
  {                                                        \
    if (ci + (J) < nch) {                                  \
      const int c0 = c_first + (ci + (J)) * 64;            \
      lds_barrier();                                       \
      astage_put<S>(ST, c0, n_keys, ks, vs, tid);          \
      lds_barrier();                                       \
      attend(c0);                                          \
    }                                                      \
    load(ST, ci + (J) + kAStages);                         \
  }
    for (int ci = 0; ci < nch; ci += kAStages) {
      VATT_CHUNK(st0, 0)
      VATT_CHUNK(st1, 1)
      VATT_CHUNK(st2, 2)
      VATT_CHUNK(st3, 3)
    }
#undef VATT_CHUNK
    // the group's partial: (max, sum, unnormalised output); a group without keys leaves
    // (-inf, 0, 0)
    if (qi < nq) {
      float* pp = apart + (((size_t)(s.row0 + qg + qi) * H + h) * G + g) * kVPart;
      if (part == 0) {   // one of the row's 16 threads writes the statistics
        pp[0] = m_run;
        pp[1] = l_run;
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) pp[2 + part * 4 + r] = o[r];
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
  float mg[kVMaxGroups], lg[kVMaxGroups], og[kVMaxGroups];
#pragma unroll
  for (int g = 0; g < kVMaxGroups; ++g) {
    const float* p = pp + min(g, G - 1) * kVPart;
    mg[g] = p[0];
    lg[g] = p[1];
    og[g] = p[2 + j];
  }
  float M = -INFINITY;
#pragma unroll
  for (int g = 0; g < kVMaxGroups; ++g) M = fmaxf(M, mg[g]);
  float L = 0.f, acc = 0.f;
#pragma unroll
  for (int g = 0; g < kVMaxGroups; ++g) {
    const float w = (g >= G || mg[g] == -INFINITY) ? 0.f : expf(mg[g] - M);
    if (g < G) {
      L += w * lg[g];
      acc += w * og[g];
    }
  }
  out[(size_t)m * d + h * kHead + j] = acc / L;
}

int attn_valu_groups(int max_keys) { return (max_keys + kVGroupKeys - 1) / kVGroupKeys; }

template <class S>
void launch_self_attn_valu(int B, int M, int H, int d, int layer, const SeqDesc* seqs, const RowDesc* rows,
                           const float* q, float* part, int G, float* out, const void* pool, int num_pages,
                           const int* block_table, int pages_per_seq, const RowTree* tree, hipStream_t st) {
  hipLaunchKernelGGL((attn_valu_kernel<S, false>), dim3(H, B, G), dim3(256), 0, st, H, d, layer, seqs, q, part,
                     G, (const typename S::T*)pool, num_pages, block_table, pages_per_seq, 0, tree);
  hipLaunchKernelGGL(attn_merge_kernel, dim3(M, H), dim3(64), 0, st, H, d, G, seqs, rows, part, out);
}
template <class S>
void launch_cross_attn_valu(int B, int M, int H, int d, int layer, const SeqDesc* seqs, const RowDesc* rows,
                            const float* q, float* part, int G, float* out, const void* cross, int frames_cap,
                            hipStream_t st) {
  hipLaunchKernelGGL((attn_valu_kernel<S, true>), dim3(H, B, G), dim3(256), 0, st, H, d, layer, seqs, q, part,
                     G, (const typename S::T*)cross, 0, nullptr, 0, frames_cap, nullptr);
  hipLaunchKernelGGL(attn_merge_kernel, dim3(M, H), dim3(64), 0, st, H, d, G, seqs, rows, part, out);
}
template void launch_self_attn_valu<F32>(int, int, int, int, int, const SeqDesc*, const RowDesc*, const float*, float*, int, float*, const void*, int, const int*, int, const RowTree*, hipStream_t);
template void launch_self_attn_valu<BF16>(int, int, int, int, int, const SeqDesc*, const RowDesc*, const float*, float*, int, float*, const void*, int, const int*, int, const RowTree*, hipStream_t);
template void launch_cross_attn_valu<F32>(int, int, int, int, int, const SeqDesc*, const RowDesc*, const float*, float*, int, float*, const void*, int, hipStream_t);
template void launch_cross_attn_valu<BF16>(int, int, int, int, int, const SeqDesc*, const RowDesc*, const float*, float*, int, float*, const void*, int, hipStream_t);

}  // namespace ad

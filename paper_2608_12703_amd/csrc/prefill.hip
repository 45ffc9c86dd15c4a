// Encoder keys / values of every decoder layer on the gfx950 matrix cores (bf16 models).
//
// Setup, once per utterance: C[f][n] = sum_k enc[f][k] W_xkv[n][k] + b_xkv[n], with
// enc bf16 [frames_cap][d] and W_xkv bf16 [2d][d] row-major; columns n < d are the keys,
// the rest the values, written as bf16 into the cross-K/V cache layout (cross_off).  This
// is a large dense contraction (frames_cap x 2d x d per layer), so it is tiled the
// plain way: a workgroup owns 256 frames x 256 columns, its eight waves 128 x 64 each
// (8 x 4 tiles of v_mfma_f32_16x16x32_bf16: 12 operand reads per 32 products), or a quarter
// of that (T = 1: 128 x 128, waves of 64 x 32) where large tiles would leave CUs idle.  Both
// operands move in 32-wide K steps through four-stage LDS rings (16 T KB a stage) filled
// by direct global->LDS loads three steps ahead: a bf16 row segment of 8 values is
// exactly one lane's MFMA operand, so every load is one 16-byte piece per lane and lands
// in the order the products read it.  The encoder states are bf16 already, so no low
// half is needed (one product per tile).
//
// Layers.  All layers that read the staged states run in one launch: one utterance has 60
// large tiles per layer, and with a launch per layer three quarters of the chip sat idle
// for a whole K loop 32 times (one large-v3 utterance 1773 -> 357 us), and a batch's last
// round of workgroups was partly empty as often (16 of 200 to 1500 frames 3278 -> 2478 us).
//
// Operand layouts.  Row-major operands make each 1 KB load gather 16 rows x 64 bytes,
// which streams at a quarter of the rate of a contiguous 1 KB (measured: about 15-28
// against 60 bytes per clock per CU from L2).  (Row-major states in 64-wide steps, eight rows
// x 128 bytes a load, for every layer in one launch: 457 us for one utterance.)  So both operands are read in "fragment
// order" when they are available that way: the weights as tiled by ad_model_pack (the
// 128-column x 32-wide K blocks of pack_weight_kernel), the encoder states as copied by
// pack_rows_kernel (for each 32-wide K step and 16-row tile, the 1 KB the products read,
// in lane order).  Row-major operands remain supported.
//
// Stores.  In the cache layout four consecutive frames of one value lane, and four
// consecutive lanes of one key frame, are contiguous.  A value tile keeps the usual
// operand order (a lane's four accumulators are four consecutive frames); a key tile
// swaps the two operands of every product, so a lane's four accumulators are four
// consecutive key lanes.  Either way a lane stores 8 bytes at a time, and a wave's
// stores cover whole runs of the block.
//
// Workgroup order.  Workgroups are dealt round-robin over the 8 XCDs; each XCD takes a
// contiguous range of tiles, ordered column group (two halves of the columns), then
// frame block, then column tile, so an XCD's concurrent workgroups share their frame
// blocks and half of the weight matrix through its L2.  Layers come first: an XCD reads
// the weights of its own layers only.
#include <algorithm>

#include "common.h"
#include "launch.h"

namespace ad {

namespace {

constexpr int kXT = 128;   // frames and output columns of a small tile (a large one: 256)
constexpr int kPackN = 128;   // columns per tile of the packed weights (pack_weight_kernel)

// the s_waitcnt immediate: vmcnt in bits 3:0 and 15:14, no wait on exports, lgkmcnt 0
constexpr int xkv_waitcnt(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0070; }

// One K step of a wave: 4 T row tiles (row half wr) x 2 T column tiles (quarter wc).  TR: the
// operands swap places (accumulator element i then runs along the columns).
template <int T, bool TR>
__device__ __forceinline__ void xkv_step(f32x4 (&acc)[4 * T][2 * T], const uint4* sa, const uint4* sb, int wr,
                                         int wc, int lane) {
  bf16x8 b[2 * T];
#pragma unroll
  for (int ct = 0; ct < 2 * T; ++ct) b[ct] = as_bf16x8(sb[(wc * 2 * T + ct) * 64 + lane]);
#pragma unroll
  for (int r = 0; r < 4 * T; ++r) {
    const bf16x8 a = as_bf16x8(sa[(wr * 4 * T + r) * 64 + lane]);
#pragma unroll
    for (int ct = 0; ct < 2 * T; ++ct) acc[r][ct] = TR ? mfma_bf16(b[ct], a, acc[r][ct]) : mfma_bf16(a, b[ct], acc[r][ct]);
  }
}

// The K loop and the stores of one tile of 128 T frames x 128 T columns (TR: a key tile with
// swapped operands; APK / WPK: encoder states / weights in fragment order).
template <int T, bool TR, bool APK, bool WPK>
__device__ __forceinline__ void xkv_tile(int M, int N, int K, const uint16_t* A, const uint16_t* W,
                                         const uint16_t* bias, uint16_t* cache, int layer, int H, int d,
                                         int frames_cap, int m0, int n0, uint4* const (&sa)[4],
                                         uint4* const (&sb)[4]) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int wr = w >> 2, wc = w & 3;
  const int c16 = lane & 15, grp = lane >> 4;
  const int KB = K / 32;
  // Wave w stages row tiles w (+ 8) and column tiles w (+ 8).  Rows / columns past the
  // matrix read its last row / column (valid addresses; those results are never stored).
  // Per K step the source advances by `as` / `ws` elements.
  const int RT = M / 16, CT = (N + kPackN - 1) / kPackN;   // 16-row tiles, 128-column tiles
  const uint16_t *pa[T], *pb[T];
  const size_t as = APK ? (size_t)RT * 512 : 32, ws = WPK ? 512 * 8 : 32;
#pragma unroll
  for (int u = 0; u < T; ++u) {
    const int rt = m0 / 16 + w + 8 * u, c = n0 / 16 + w + 8 * u;
    pa[u] = APK ? A + ((size_t)min(rt, RT - 1) * 64 + lane) * 8
                : A + (size_t)min(rt * 16 + c16, M - 1) * K + grp * 8;
    // (tiled weights: column tile c is 16-column tile c % 8 of 128-column tile c / 8)
    pb[u] = WPK ? W + (((size_t)min(c / 8, CT - 1) * KB) * 512 + (c % 8) * 64 + lane) * 8
                : W + (size_t)min(c * 16 + c16, N - 1) * K + grp * 8;
  }
  auto issue = [&](int s, int kb) {   // stage kb (clamped) into ring slot s: 2 T loads per wave
    const size_t k = min(kb, KB - 1);
#pragma unroll
    for (int u = 0; u < T; ++u) dma16(pa[u] + k * as, sa[s] + (w + 8 * u) * 64);
#pragma unroll
    for (int u = 0; u < T; ++u) dma16(pb[u] + k * ws, sb[s] + (w + 8 * u) * 64);
  };
  f32x4 acc[4 * T][2 * T];
#pragma unroll
  for (int r = 0; r < 4 * T; ++r)
#pragma unroll
    for (int ct = 0; ct < 2 * T; ++ct) acc[r][ct] = f32x4{0.f, 0.f, 0.f, 0.f};

  issue(0, 0);
  issue(1, 1);
  issue(2, 2);
  int kb = 0;
  // Step j: wait until stage j has landed (stages j + 1 and j + 2, 4 T loads, may still
  // be in flight) and every wave is past step j - 1, refill step j - 1's slot with stage
  // j + 3, multiply stage j.  The loop is unrolled over the ring, so every slot is a
  // compile-time choice.
#define XKV_STEP(S)                                           \
  {                                                           \
    __builtin_amdgcn_s_waitcnt(xkv_waitcnt(4 * T));           \
    __builtin_amdgcn_s_barrier();                             \
    asm volatile("" ::: "memory");                            \
    issue(((S) + 3) % 4, kb + 3);                             \
    xkv_step<T, TR>(acc, sa[S], sb[S], wr, wc, lane);         \
    ++kb;                                                     \
  }
  for (int it = 0; it < KB / 4; ++it) {
    XKV_STEP(0)
    XKV_STEP(1)
    XKV_STEP(2)
    XKV_STEP(3)
  }
  const int rem = KB % 4;
  if (rem >= 1) XKV_STEP(0)
  if (rem >= 2) XKV_STEP(1)
  if (rem >= 3) XKV_STEP(2)
#undef XKV_STEP
  __builtin_amdgcn_s_waitcnt(xkv_waitcnt(0));

  // epilogue: bias, bf16 rounding, the cross-K/V layout (keys for n < d, values after).
  // Accumulator (r, ct, i) of this lane is frame m0 + 16 (4 T wr + r) + {4 grp + i | c16}
  // and column n0 + 16 (2 T wc + ct) + {c16 | 4 grp + i} (value | key tile).
  // (a tile that holds both keys and values keeps the usual order, in which a lane's four
  // key frames are not contiguous: it stores element by element)
  const bool whole = m0 + kXT * T <= M && n0 + kXT * T <= N && (TR || n0 >= d);
  if (whole) {
    // four contiguous elements per store
#pragma unroll
    for (int ct = 0; ct < 2 * T; ++ct) {
      const int nb = n0 + (wc * 2 * T + ct) * 16 + (TR ? grp * 4 : c16);
      const int kv = nb / d, h = (nb % d) / kHead, j = nb % kHead;
      uint16_t* base = cache + cross_base(layer, h, H, frames_cap);
      float bv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) bv[i] = bf16_to_f32(bias[TR ? nb + i : nb]);
#pragma unroll
      for (int r = 0; r < 4 * T; ++r) {
        const int m = m0 + (wr * 4 * T + r) * 16 + (TR ? c16 : grp * 4);
        const f32x4 v = acc[r][ct];
        const uint2 pk = make_uint2(f32x2_to_bf16x2(v[0] + bv[0], v[1] + bv[1]),
                                    f32x2_to_bf16x2(v[2] + bv[2], v[3] + bv[3]));
        *(uint2*)(base + cross_off(kv, m, j)) = pk;
      }
    }
    return;
  }
  // a tile past the last frame or column, or across the key / value boundary: one
  // element at a time
#pragma unroll
  for (int ct = 0; ct < 2 * T; ++ct)
#pragma unroll
    for (int r = 0; r < 4 * T; ++r)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int n = n0 + (wc * 2 * T + ct) * 16 + (TR ? grp * 4 + i : c16);
        const int m = m0 + (wr * 4 * T + r) * 16 + (TR ? c16 : grp * 4 + i);
        if (n >= N || m >= M) continue;
        const int kv = n / d, h = (n % d) / kHead, j = n % kHead;
        cache[cross_base(layer, h, H, frames_cap) + cross_off(kv, m, j)] =
            f32_to_bf16(acc[r][ct][i] + bf16_to_f32(bias[n]));
      }
}

}  // namespace

template <int T, bool APK, bool WPK>
__global__ void __launch_bounds__(512) xkv_mfma_kernel(int M, int N, int K, const uint16_t* A,
                                                       XkvLayersOf<APK ? kXkvLayers : 1> lay,
                                                       uint16_t* cache, int H, int d,
                                                       int frames_cap) {
  // distinct LDS objects per ring stage, so the compiler can tell a read of one stage from
  // the direct loads still filling another
  __shared__ uint4 sa0[T * 512], sa1[T * 512], sa2[T * 512], sa3[T * 512];
  __shared__ uint4 sb0[T * 512], sb1[T * 512], sb2[T * 512], sb3[T * 512];
  uint4* const sa[4] = {sa0, sa1, sa2, sa3};
  uint4* const sb[4] = {sb0, sb1, sb2, sb3};
  // layer and tile of this workgroup (see the header: XCD ranges, layer, column group, frame
  // block, column)
  constexpr int X = kXT * T;
  const int NT = (N + X - 1) / X, MB = (M + X - 1) / X;
  const int nwg = gridDim.x, bid = blockIdx.x;
  const int x = bid & 7, q8 = nwg >> 3, r8 = nwg & 7;
  const int all = x * q8 + min(x, r8) + (bid >> 3);
  const int li = APK ? all / (NT * MB) : 0, lin = all - li * (NT * MB);   // (row-major states: one layer)
  const int gc = (NT + 1) / 2;
  const int g = lin / (MB * gc), rem = lin - g * MB * gc;
  const int gw = min(gc, NT - g * gc);
  const int m0 = (rem / gw) * X, n0 = (g * gc + rem % gw) * X;
  // a key tile (every column a key) swaps the product operands for its stores
  if (n0 + X <= d)
    xkv_tile<T, true, APK, WPK>(M, N, K, A, (const uint16_t*)lay.W[li], (const uint16_t*)lay.bias[li], cache, lay.first + li, H, d, frames_cap, m0,
                                n0, sa, sb);
  else
    xkv_tile<T, false, APK, WPK>(M, N, K, A, (const uint16_t*)lay.W[li], (const uint16_t*)lay.bias[li], cache, lay.first + li, H, d, frames_cap,
                                 m0, n0, sa, sb);
}

// Encoder states [M][K] (M a multiple of 16) in fragment order: for 32-wide K step kb and
// 16-row tile rt, 64 lanes x 8 values at ((kb * RT + rt) * 64 + lane) * 8, lane l holding
// row 16 rt + l % 16, columns 32 kb + 8 (l / 16) .. + 7.  Each thread moves one 16-byte
// piece; consecutive threads read consecutive pieces of a row.
__global__ void __launch_bounds__(256) pack_rows_kernel(const uint16_t* A, int M, int K, uint16_t* P) {
  const int RT = M / 16;
  const size_t pieces = (size_t)M * K / 8;
  for (size_t q = (size_t)blockIdx.x * 256 + threadIdx.x; q < pieces; q += (size_t)gridDim.x * 256) {
    const int m = (int)(q / (K / 8)), k8 = (int)(q % (K / 8));
    const int kb = k8 / 4, g = k8 % 4, rt = m / 16, r = m % 16;
    const uint4 v = *(const uint4*)(A + q * 8);
    *(uint4*)(P + (((size_t)kb * RT + rt) * 64 + g * 16 + r) * 8) = v;
  }
}

template <int T>
static void launch_tiles(int M, int N, int K, const uint16_t* A, bool a_packed, const XkvLayers& lay, int layers,
                         bool w_packed, uint16_t* cache, int H, int d, int frames_cap, hipStream_t st) {
  constexpr int X = kXT * T;
  const dim3 grid(((N + X - 1) / X) * ((M + X - 1) / X) * layers), block(512);
  auto go = [&](auto kernel, const auto& l) {
    hipLaunchKernelGGL(kernel, grid, block, 0, st, M, N, K, A, l, cache, H, d, frames_cap);
  };
  // (the 1 KB of kernel arguments of 64 layers costs a launch about 1 us: one row-major layer of
  // d 1280, 6400 frames 41.3 us with them, 39.3 with one)
  const XkvLayersOf<1> one{{lay.W[0]}, {lay.bias[0]}, lay.first};
  if (a_packed && w_packed) go(xkv_mfma_kernel<T, true, true>, lay);
  else if (a_packed) go(xkv_mfma_kernel<T, true, false>, lay);
  else if (w_packed) go(xkv_mfma_kernel<T, false, true>, one);
  else go(xkv_mfma_kernel<T, false, false>, one);
}

void launch_xkv_mfma(int M, int N, int K, const uint16_t* A, bool a_packed, const XkvLayers& lay, int layers,
                     bool w_packed, uint16_t* cache, int H, int d, int frames_cap, hipStream_t st) {
  // Large tiles read half the operand bytes per product, small ones fill the chip.  Either kind
  // takes as long as its rounds of 256 workgroups, each a fixed part and KB 32-wide steps, and a
  // large tile past the last frame stores its `rest` of up to 224 frames one element at a time.
  // In units of a small tile's step of row-major states (0.28 us): small, a round KB + 10;
  // large, 2.8 KB + 40 and 0.7 rest with staged states, 2.4 KB + 24 and 0.5 rest with row-major
  // ones (whose gathered loads small tiles double).  Fitted to 592 launches (d 64 to 3072, 32 to
  // 24064 frames, 1 to 4 layers): the choice is within 1.02 of large tiles everywhere and within
  // 1.1 of the faster kind in all but one (1.26).  us, small / large (rounds): row-major states,
  // one layer, d 1280, 1504 frames (1, 1) 20 / 57; 5632 (4, 1) 54 / 37; 8064 (5, 2) 69 / 91;
  // 12032 (8, 2) 106 / 74; d 2048, 2816 (3, 1) 62 / 47; staged (with the
  // staging copy), d 1280, four layers of 1504 (4, 1) 49 / 64; one of 24064 (15, 4) 194 / 182;
  // d 768, four of 12032 (18, 5) 130 / 119
  const long long large = (long long)((N + 255) / 256) * ((M + 255) / 256) * layers;
  const long long small = (long long)((N + 127) / 128) * ((M + 127) / 128) * layers;
  const long long rl = (large + 255) / 256, rs = (small + 255) / 256;
  const int KB = K / 32, rest = M % 256;
  const long long t_small = 10 * rs * (KB + 10);
  const long long t_large = a_packed ? rl * (28 * KB + 400) + 7 * rest : rl * (24 * KB + 240) + 5 * rest;
  if (t_small <= t_large)
    launch_tiles<1>(M, N, K, A, a_packed, lay, layers, w_packed, cache, H, d, frames_cap, st);
  else
    launch_tiles<2>(M, N, K, A, a_packed, lay, layers, w_packed, cache, H, d, frames_cap, st);
}

void launch_pack_rows(const uint16_t* A, int M, int K, uint16_t* P, hipStream_t st) {
  const size_t pieces = (size_t)M * K / 8;
  const dim3 grid((unsigned)std::min<size_t>((pieces + 255) / 256, 16384)), block(256);
  hipLaunchKernelGGL(pack_rows_kernel, grid, block, 0, st, A, M, K, P);
}

}  // namespace ad

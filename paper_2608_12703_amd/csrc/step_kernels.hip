// Small kernels of the verify step: descriptor preparation and validation, embedding,
// LayerNorm, argmax with top-2 margin, the prefix-accept scan, commit, prefix import and
// the draft-head helpers.
#include "common.h"
#include "launch.h"
#include "row_stats.h"
#include "top2.h"

namespace ad {

// ---------------------------------------------------------------- descriptors

// Validation and descriptors, one wave per sequence: a lane per page of the committed cache and
// a lane per block row (at most 64).  Bound by latency (one launch, one chain of dependent
// loads): a thread per sequence walked its pages and tokens one after another (11-row trees
// 10.6 us, 9-row ragged blocks 8.3 us; now 4.7 us for both, an ordinary dependent launch).
// Padded rows are described here, which saves their steps a launch; packed rows, whose
// sequence has to be searched, by prep_row_kernel.
__global__ void __launch_bounds__(256) prep_seq_kernel(StepArgs a, SeqDesc* seqs, RowDesc* rows,
                                                       int* err) {
  const int b = blockIdx.x * (256 / kWave) + threadIdx.x / kWave, i = threadIdx.x % kWave;   // i: block row
  if (b >= a.B) return;
  const int kb = a.k[b], n = a.kv_len[b], T = a.enc_len[b], off = a.enc_off[b];
  int row0 = a.layout == 0 ? b * (a.k_max + 1) : a.cu_rows[b];
  int e = 0;
  if (kb < 0 || kb > a.k_max || n < 0 || n + kb + 1 > a.max_pos) e |= 1;
  if (a.layout == 1) {
    const int r1 = a.cu_rows[b + 1];
    if (row0 < 0 || r1 > a.rows || r1 - row0 != kb + 1) e |= 1;
  }
  if (T < 1 || T > a.max_frames || off < 0 || (off % kCrossBlock) || off + T > a.frames_cap) e |= 8;
  int wlo = 0, whi = T;
  if (a.cross_window) {
    wlo = a.cross_window[2 * b];
    whi = a.cross_window[2 * b + 1];
    if (wlo < 0 || whi > T || wlo >= whi) e |= 8;
  }
  int token = 0, depth = i;
  if (!(e & 1)) {
    const bool on = i <= kb;
    const int last_page = (n + kb) / kTile;
    int bad = 0;
    if (last_page >= a.pages_per_seq) {
      bad = 2;
    } else {
      for (int p = i; p <= last_page; p += kWave) {
        const int pg = a.block_table[(size_t)b * a.pages_per_seq + p];
        if (pg < 0 || pg >= a.num_pages) bad |= 2;
      }
    }
    token = on ? a.tokens[row0 + i] : 0;
    if (token < 0 || token >= a.V) bad |= 4;
    // depth and ancestor mask of every block row: a draft tree's parents must be earlier
    // rows; without a tree the rows form a chain (row i's parent is row i - 1)
    unsigned long long mask = (2ull << i) - 1;
    if (a.parents) {
      const int parent = on && i > 0 ? a.parents[row0 + i] : -1;
      if (on && i > 0 && (parent < 0 || parent >= i)) bad |= 32;
      if (!__any(bad & 32)) {
        mask = 1ull << i;
        depth = 0;
        int p = on ? parent : -1;
        while (__any(p >= 0)) {   // parents decrease, so this ends within 64 steps
          const int q = __shfl(parent, max(p, 0), kWave);
          if (p >= 0) {
            mask |= 1ull << p;
            ++depth;
            p = q;
          }
        }
      }
    }
    if (on) a.tree[row0 + i] = RowTree{mask, depth, 0};
    e |= (__any(bad & 2) ? 2 : 0) | (__any(bad & 4) ? 4 : 0) | (__any(bad & 32) ? 32 : 0);
  }
  if (a.layout == 0 && i <= a.k_max)
    rows[(size_t)b * (a.k_max + 1) + i] =
        e == 0 && i <= kb ? RowDesc{b, i, n + depth, token, n + i} : RowDesc{-1, 0, 0, 0, 0};
  if (i == 0) {
    if (e) atomicOr(err, e);
    if (e & 1) row0 = 0;
    seqs[b] = SeqDesc{row0, e ? 0 : kb, e ? 0 : n, e ? 1 : T, e ? 0 : off, e == 0, e ? 0 : wlo,
                      e ? 1 : whi};
  }
}

// The packed rows' descriptors.
__global__ void prep_row_kernel(StepArgs a, const SeqDesc* seqs, RowDesc* rows) {
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= a.rows) return;
  // last sequence whose first row is <= m (bounded binary search over cu_rows)
  int lo = 0, hi = a.B - 1, b = -1;
  while (lo <= hi) {
    const int mid = (lo + hi) >> 1;
    if (a.cu_rows[mid] <= m) { b = mid; lo = mid + 1; } else { hi = mid - 1; }
  }
  const int i = b >= 0 ? m - a.cu_rows[b] : 0;
  RowDesc r{-1, 0, 0, 0, 0};
  if (b >= 0) {
    const SeqDesc s = seqs[b];
    if (s.valid && i >= 0 && i <= s.k && s.row0 + i == m) {
      r.seq = b;
      r.i = i;
      r.pos = s.n + a.tree[m].depth;
      r.slot = s.n + i;
      r.token = a.tokens[m];
    }
  }
  rows[m] = r;
}

// ---------------------------------------------------------------- embedding

__global__ void embed_kernel(int d, const RowDesc* rows, const float* tok_emb, const float* pos_emb, float* x,
                             const float* in_rows) {
  const int m = blockIdx.x;
  const RowDesc r = rows[m];
  for (int j = threadIdx.x; j < d; j += blockDim.x)
    x[(size_t)m * d + j] = (in_rows ? in_rows[(size_t)m * d + j] : tok_emb[(size_t)r.token * d + j]) +
                           pos_emb[(size_t)r.pos * d + j];
}

// ---------------------------------------------------------------- LayerNorm
// out = (x - mean) / sqrt(var + 1e-5) * g + b, biased variance, two passes over the row.

__global__ void __launch_bounds__(256) layernorm_kernel(int d, const float* x, const float* g, const float* b,
                                                        float* out) {
  __shared__ float red[4];
  const int m = blockIdx.x;
  const float* xr = x + (size_t)m * d;
  if (d <= kRowStatsMax) {   // every 16 lanes take the row's statistics, no barrier
    f32x4 xs[kRowParts];
#pragma unroll
    for (int t = 0; t < kRowParts; ++t) xs[t] = row_part(xr, d, threadIdx.x % 16, t);
    const float2 rs = row_stats(xs, d);
    for (int j = threadIdx.x; j < d; j += 256)
      out[(size_t)m * d + j] = normalised(xr[j], rs, g[j], b[j]);
    return;
  }
  float s = 0.f;
  for (int j = threadIdx.x; j < d; j += 256) s += xr[j];
  const float mean = block_sum<4>(s, red) / (float)d;
  float v = 0.f;
  for (int j = threadIdx.x; j < d; j += 256) {
    const float t = xr[j] - mean;
    v += t * t;
  }
  const float var = block_sum<4>(v, red) / (float)d;
  const float rstd = 1.0f / sqrtf(var + 1e-5f);
  for (int j = threadIdx.x; j < d; j += 256)
    out[(size_t)m * d + j] = (xr[j] - mean) * rstd * g[j] + b[j];
}

// split_sum4 with the first eight planes as straight-line loads (planes past nsplit
// are clamped reads that add -0, which leaves every value, signed zeros included,
// unchanged): no loop, so loads issued before it stay in flight across it.  Further
// planes, if any, in a loop.
__device__ __forceinline__ float4 split_sum4_flat(const float* P, size_t plane, size_t e, int nsplit) {
  float4 p[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) p[u] = *(const float4*)(P + (size_t)min(u, nsplit - 1) * plane + e);
  float4 acc = p[0];
#pragma unroll
  for (int u = 1; u < 8; ++u) {
    const bool in = u < nsplit;
    acc.x += in ? p[u].x : -0.f;
    acc.y += in ? p[u].y : -0.f;
    acc.z += in ? p[u].z : -0.f;
    acc.w += in ? p[u].w : -0.f;
  }
  for (int t = 8; t < nsplit; ++t) {
    const float4 w = *(const float4*)(P + (size_t)t * plane + e);
    acc.x += w.x; acc.y += w.y; acc.z += w.z; acc.w += w.w;
  }
  return acc;
}

// Sum over the block's waves in wave order; every thread gets the total.  No other reduction of
// the kernel uses `red` (no barrier before writing it).
__device__ __forceinline__ float row_block_sum_once(float v, float* red) {
  v = wave_sum(v);
  const int w = threadIdx.x / kWave, nw = blockDim.x / kWave;
  if ((threadIdx.x & (kWave - 1)) == 0) red[w] = v;
  __syncthreads();
  float t = 0.f;
  for (int i = 0; i < nw; ++i) t += red[i];
  return t;
}

__device__ __forceinline__ float4 ld_bf16x4(const uint16_t* p, int j) {
  const uint2 u = *(const uint2*)(p + j);
  return float4{bf16_to_f32(u.x & 0xffff), bf16_to_f32(u.x >> 16), bf16_to_f32(u.y & 0xffff),
                bf16_to_f32(u.y >> 16)};
}

// Row of workgroup `bid` for the row-per-workgroup kernels that write A-fragment
// operands.  Workgroups are dealt round-robin over the 8 XCDs; this numbering puts the
// 8 rows that share each 128-byte line of the output (rows 8a .. 8a + 7) on one XCD, so
// its L2 merges their 16-byte pieces into whole lines.  Launch ceil(M / 64) * 64
// workgroups; rows past M exit.
__device__ __forceinline__ int xcd_row(int bid) {
  return (bid >> 6) * 64 + (bid & 7) * 8 + ((bid >> 3) & 7);
}
__host__ inline int xcd_row_grid(int M) { return (M + 63) / 64 * 64; }

// Residual update and the next LayerNorm of one row: x += sum_s P[s] + bias, then
// LN(x) * g + b goes out in A-fragment order (and to `out` when given).  One thread per
// 4 columns (blockDim = d / 4 rounded up to whole waves).
__global__ void __launch_bounds__(1024) reduce_res_ln_kernel(int M, int d, int nsplit,
                                                             const float* P, const uint16_t* bias,
                                                             float* x, const uint16_t* g,
                                                             const uint16_t* b, uint16_t* frag,
                                                             int RT, float* out) {
  __shared__ float red_mean[16], red_var[16];
  const int m = xcd_row(blockIdx.x), j = threadIdx.x * 4;
  if (m >= M) return;
  const bool on = j < d;
  const int jc = on ? j : 0;
  const size_t e = (size_t)m * d + jc;
  // every load of the row up front (one round trip): partials, bias, residual, and the
  // LayerNorm gain and shift
  const float4 bb = ld_bf16x4(bias, jc);
  const float4 x0 = *(const float4*)(x + e);
  const float4 gv = ld_bf16x4(g, jc), bv = ld_bf16x4(b, jc);
  const float4 v = split_sum4_flat(P, (size_t)M * d, e, nsplit);
  float4 xv{0.f, 0.f, 0.f, 0.f};
  if (on) {
    xv = x0;
    xv.x += v.x + bb.x; xv.y += v.y + bb.y; xv.z += v.z + bb.z; xv.w += v.w + bb.w;
    *(float4*)(x + e) = xv;
  }
  const float mean = row_block_sum_once(on ? (xv.x + xv.y) + (xv.z + xv.w) : 0.f, red_mean) / (float)d;
  const float4 c{xv.x - mean, xv.y - mean, xv.z - mean, xv.w - mean};
  const float var = row_block_sum_once(on ? (c.x * c.x + c.y * c.y) + (c.z * c.z + c.w * c.w) : 0.f, red_var);
  const float rstd = 1.0f / sqrtf(var / (float)d + 1e-5f);
  if (on) {
    const float4 y{c.x * rstd * gv.x + bv.x, c.y * rstd * gv.y + bv.y, c.z * rstd * gv.z + bv.z,
                   c.w * rstd * gv.w + bv.w};
    afrag_store4(frag, RT, m, j, y);
    if (out) *(float4*)(out + e) = y;
  }
}

// Embedding of the block rows fused with the first LayerNorm: x = E_tok[token] (or the
// caller's input row) + E_pos[pos], then LN(x) * g + b in A-fragment order.  One thread
// per 4 columns (blockDim = d / 4 rounded up to whole waves), every load up front.
__global__ void __launch_bounds__(1024) embed_ln_kernel(int M, int d, const RowDesc* rows,
                                                       const uint16_t* tok_emb,
                                                       const uint16_t* pos_emb, float* x,
                                                       const float* in_rows, const uint16_t* g,
                                                       const uint16_t* b, uint16_t* frag, int RT) {
  __shared__ float red_mean[16], red_var[16];
  const int m = xcd_row(blockIdx.x), j = threadIdx.x * 4;
  if (m >= M) return;
  const bool on = j < d;
  const int jc = on ? j : 0;
  const float4 gv = ld_bf16x4(g, jc), bv = ld_bf16x4(b, jc);
  const RowDesc r = rows[m];
  const float4 te = in_rows ? *(const float4*)(in_rows + (size_t)m * d + jc)
                            : ld_bf16x4(tok_emb + (size_t)r.token * d, jc);
  const float4 pe = ld_bf16x4(pos_emb + (size_t)r.pos * d, jc);
  const float4 v{te.x + pe.x, te.y + pe.y, te.z + pe.z, te.w + pe.w};
  if (on) *(float4*)(x + (size_t)m * d + j) = v;
  const float mean = row_block_sum_once(on ? (v.x + v.y) + (v.z + v.w) : 0.f, red_mean) / (float)d;
  const float4 c{v.x - mean, v.y - mean, v.z - mean, v.w - mean};
  const float var = row_block_sum_once(on ? (c.x * c.x + c.y * c.y) + (c.z * c.z + c.w * c.w) : 0.f, red_var);
  const float rstd = 1.0f / sqrtf(var / (float)d + 1e-5f);
  if (on)
    afrag_store4(frag, RT, m, j,
                 float4{c.x * rstd * gv.x + bv.x, c.y * rstd * gv.y + bv.y, c.z * rstd * gv.z + bv.z,
                        c.w * rstd * gv.w + bv.w});
}

// ---------------------------------------------------------------- argmax + margin

// Row-wise merge of the per-tile top-2 records of the LM head: greedy token (lowest
// index among equal maxima) and the top-1 minus top-2 margin.
__global__ void __launch_bounds__(64) argmax_final_kernel(int M, int nrec, const float4* part,
                                                          const RowDesc* rows, int* greedy,
                                                          float* margin, int* err) {
  const int m = blockIdx.x, lane = threadIdx.x;
  Top2s t{-INFINITY, 0x7fffffff, -INFINITY, 0};
  for (int j = lane; j < nrec; j += 64) {
    const float4 p = part[(size_t)m * nrec + j];
    t = t2_merge(t, Top2s{p.x, __float_as_int(p.y), p.z, __float_as_int(p.w)});
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) t = t2_merge(t, t2_shfl(t, o));
  if (lane == 0) {
    const bool valid_row = rows ? rows[m].seq >= 0 : true;
    if (t.bad && valid_row && err) atomicOr(err, 16);
    greedy[m] = (t.bad && valid_row) ? -1 : t.i1;
    if (margin) margin[m] = t.v1 - t.v2;
  }
}

// ---------------------------------------------------------------- accept / commit

__global__ void accept_kernel(int B, int k_max, const SeqDesc* seqs, const int* tokens,
                              const int* greedy, int* accept_len, int* out_tokens) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  const SeqDesc s = seqs[b];
  int a = -1;
  if (s.valid) {
    bool ok = true;
    for (int i = 0; i <= s.k; ++i) ok = ok && greedy[s.row0 + i] >= 0;
    if (ok) {
      a = 0;
      while (a < s.k && tokens[s.row0 + 1 + a] == greedy[s.row0 + a]) ++a;
    }
  }
  accept_len[b] = a;
  for (int i = 0; i <= k_max; ++i)
    out_tokens[(size_t)b * (k_max + 1) + i] = (a >= 0 && i <= a) ? greedy[s.row0 + i] : -1;
}

// Draft-tree accept: from the root, move to the lowest-index child whose token equals the
// current node's greedy token; the emitted tokens are the greedy tokens along the path.
__global__ void accept_tree_kernel(int B, int k_max, const SeqDesc* seqs, const int* tokens,
                                   const int* parents, const int* greedy, int* accept_len,
                                   int* out_tokens, int* out_path) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  const SeqDesc s = seqs[b];
  int* path = out_path + (size_t)b * (k_max + 1);
  int a = -1;
  if (s.valid) {
    bool ok = true;
    for (int i = 0; i <= s.k; ++i) ok = ok && greedy[s.row0 + i] >= 0;
    if (ok) {
      a = 0;
      path[0] = 0;
      int u = 0;
      while (true) {
        const int g = greedy[s.row0 + u];
        int nxt = -1;
        for (int c = u + 1; c <= s.k && nxt < 0; ++c)
          if (parents[s.row0 + c] == u && tokens[s.row0 + c] == g) nxt = c;
        if (nxt < 0) break;
        u = nxt;
        path[++a] = u;
      }
    }
  }
  accept_len[b] = a;
  for (int i = 0; i <= k_max; ++i) {
    const bool on = a >= 0 && i <= a;
    out_tokens[(size_t)b * (k_max + 1) + i] = on ? greedy[s.row0 + path[i]] : -1;
    if (!on) path[i] = -1;
  }
}

// Accepted tree path node j (block row path[j], slot n + path[j]) -> slot n + j, for one
// (layer, K|V) per block, eight nodes at a time: each thread moves the same (head, lane)
// element of every slot, reading all eight sources before writing any destination.  A
// source is never an earlier node's destination (path[j] >= j), so reading a batch before
// writing it, and batches in path order, move every slot's original contents.
template <class S>
__global__ void __launch_bounds__(256) kv_compact_kernel(int H, const int* kv_len, const int* accept_len,
                                                         const int* path, int path_stride,
                                                         typename S::T* pool, int num_pages,
                                                         const int* block_table, int pages_per_seq) {
  using T = typename S::T;
  const int b = blockIdx.x, layer = blockIdx.y >> 1, kv = blockIdx.y & 1;
  const int a = min(accept_len[b], path_stride - 1);
  if (a <= 0) return;
  const int n = kv_len[b];
  const int* p = path + (size_t)b * path_stride;
  for (int j0 = 1; j0 <= a; j0 += 8) {
    size_t sb[8], db[8];
    bool mv[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int j = j0 + u;
      const int node = j <= a ? p[j] : 0;
      // (a path row never precedes its index; slots past the block table are left alone)
      mv[u] = j <= a && node > j && (n + node) / kTile < pages_per_seq;
      const int src = mv[u] ? n + node : 0, dst = mv[u] ? n + j : 0;
      const int ps = min(max(block_table[(size_t)b * pages_per_seq + src / kTile], 0), num_pages - 1);
      const int pd = min(max(block_table[(size_t)b * pages_per_seq + dst / kTile], 0), num_pages - 1);
      sb[u] = kv_tile_base(layer, kv, ps, 0, num_pages, H) + tile_off(kv, src % kTile, 0);
      db[u] = kv_tile_base(layer, kv, pd, 0, num_pages, H) + tile_off(kv, dst % kTile, 0);
    }
    for (int e = threadIdx.x; e < H * kHead; e += blockDim.x) {
      const int h = e / kHead, c = e % kHead;
      const size_t off = (size_t)h * kTileElems + (tile_off(kv, 0, c));
      T v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = mv[u] ? pool[sb[u] + off] : T();
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (mv[u]) pool[db[u] + off] = v[u];
    }
  }
}

__global__ void commit_kernel(int B, int* kv_len, const int* accept_len) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  const int a = accept_len[b];
  if (a >= 0) kv_len[b] += a + 1;
}

// ---------------------------------------------------------------- prefix import

// EXPORT = false: src [L][2][n][H][64] -> pool; EXPORT = true: pool -> dst.
template <class S, bool EXPORT>
__global__ void kv_copy_kernel(int L, int H, int n, int b, typename S::T* lin,
                               typename S::T* pool, int num_pages, const int* block_table,
                               int pages_per_seq, int* err) {
  // one thread per element of the logical array [L][2][n][H][64]
  const size_t total = (size_t)L * 2 * n * H * kHead;
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= total) return;
  size_t r = idx;
  const int j = r % kHead; r /= kHead;
  const int h = r % H; r /= H;
  const int p = r % n; r /= n;
  const int kv = r % 2; r /= 2;
  const int layer = (int)r;
  const int pg = block_table[(size_t)b * pages_per_seq + p / kTile];
  if (pg < 0 || pg >= num_pages) {
    atomicOr(err, 2);
    return;
  }
  const size_t at = kv_tile_base(layer, kv, pg, h, num_pages, H) + tile_off(kv, p % kTile, j);
  if (EXPORT) lin[idx] = pool[at];
  else pool[at] = lin[idx];
}

// The same copy by whole 16-token tiles, for a 16-byte aligned linear array: one workgroup per
// (16-token tile, layer, K|V, four heads), 16 bytes per access on both sides.  Keys are
// token-major in a tile, so their pieces move as they are, in the cache's order (128-byte runs
// of the linear array).  Values are lane-major and are transposed through LDS.  Bound by
// memory; the element-wise kernel spent its time on index divisions and 2-byte accesses.
// 220 tokens of the large-v3 cache, 36 MB each way: import and export 125 -> 31 us together
// (4.6 TB/s; the kernels alone 13 + 12); 53 tokens of 30 layers x 4 heads 6.2 + 4.9 -> 3.4 + 2.9 us.
// (Loads are unconditional, tokens and heads past the tile clamped, so that all of a thread's
// are in flight together.)
constexpr int kCopyHeads = 4;

template <class S, bool EXPORT>
__global__ void __launch_bounds__(256) kv_copy_tile_kernel(int H, int n, int b, typename S::T* lin,
                                                           typename S::T* pool, int num_pages,
                                                           const int* block_table, int pages_per_seq,
                                                           int* err) {
  using T = typename S::T;
  constexpr int E = 16 / sizeof(T), kRow = kCopyHeads * kHead, kPer = kTile * kRow / E / 256;
  typedef T P __attribute__((ext_vector_type(E)));
  __shared__ __align__(16) T tr[kTile][kRow + E];   // values: [token][head, lane]
  const int tile = blockIdx.x, layer = blockIdx.y >> 1, kv = blockIdx.y & 1, h0 = blockIdx.z * kCopyHeads;
  const int pg = block_table[(size_t)b * pages_per_seq + tile];
  const int cnt = min(kTile, n - tile * kTile);          // tokens of this tile
  const int cols = min(kCopyHeads, H - h0) * kHead;      // lanes of these heads
  const size_t row = (size_t)H * kHead;
  T* lp = lin + ((size_t)blockIdx.y * n + (size_t)tile * kTile) * row + h0 * kHead;
  // piece i of this thread: element q; keys in the cache's order (head, token, lane), values
  // in the linear order (token, head and lane)
  int t[kPer], c[kPer], q[kPer];
  bool on[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    q[i] = (threadIdx.x + 256 * i) * E;
    t[i] = kv == 0 ? q[i] % kTileElems / kHead : q[i] / kRow;
    c[i] = kv == 0 ? q[i] / kTileElems * kHead + q[i] % kHead : q[i] % kRow;
    on[i] = t[i] < cnt && c[i] < cols;
  }
  P v[kPer];
  if (!EXPORT) {   // (the linear side does not wait for the page)
#pragma unroll
    for (int i = 0; i < kPer; ++i) v[i] = *(const P*)(lp + min(t[i], cnt - 1) * row + (on[i] ? c[i] : 0));
  }
  if (pg < 0 || pg >= num_pages) {
    if (threadIdx.x == 0) atomicOr(err, 2);
    return;
  }
  T* pp = pool + kv_tile_base(layer, kv, pg, h0, num_pages, H);
  if (EXPORT) {   // the cache's order on both paths
#pragma unroll
    for (int i = 0; i < kPer; ++i) v[i] = *(const P*)(pp + (q[i] < cols * kTile ? q[i] : 0));
  }
  if (kv == 0) {
#pragma unroll
    for (int i = 0; i < kPer; ++i)
      if (on[i]) *(P*)(EXPORT ? lp + t[i] * row + c[i] : pp + q[i]) = v[i];
    return;
  }
  // values in the cache's order: elements q .. q + E - 1 are tokens tv .. of lane cv
  if (EXPORT) {
#pragma unroll
    for (int i = 0; i < kPer; ++i)
#pragma unroll
      for (int u = 0; u < E; ++u) tr[q[i] % kTile + u][q[i] / kTile] = v[i][u];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kPer; ++i)
      if (on[i]) *(P*)(lp + t[i] * row + c[i]) = *(const P*)&tr[t[i]][c[i]];
    return;
  }
#pragma unroll
  for (int i = 0; i < kPer; ++i) *(P*)&tr[t[i]][c[i]] = v[i];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int cv = q[i] / kTile, tv = q[i] % kTile;
    if (cv >= cols || tv >= cnt) continue;
    P o;
#pragma unroll
    for (int u = 0; u < E; ++u) o[u] = tr[tv + u][cv];
    if (tv + E <= cnt) {
      *(P*)(pp + q[i]) = o;
    } else {   // the tokens past n keep what their slots hold
#pragma unroll
      for (int u = 0; u < E; ++u)
        if (tv + u < cnt) pp[q[i] + u] = o[u];
    }
  }
}

// ---------------------------------------------------------------- draft heads

__global__ void gather_hidden_kernel(int B, int d, int layout, int k_max, const int* cu_rows,
                                     const int* accept_len, const float* hidden, float* hsel) {
  const int b = blockIdx.x;
  const int a = accept_len[b];
  const int row0 = layout == 0 ? b * (k_max + 1) : cu_rows[b];
  for (int j = threadIdx.x; j < d; j += blockDim.x)
    hsel[(size_t)b * d + j] = a >= 0 ? hidden[(size_t)(row0 + a) * d + j] : 0.f;
}

__global__ void assemble_next_kernel(int B, int n_heads, int k_max, const int* accept_len,
                                     const int* out_tokens, const int* head_greedy,
                                     int* next_tokens) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  const int a = accept_len[b];
  int* nt = next_tokens + (size_t)b * (n_heads + 1);
  nt[0] = a >= 0 ? out_tokens[(size_t)b * (k_max + 1) + a] : -1;
  for (int i = 0; i < n_heads; ++i) nt[1 + i] = a >= 0 ? head_greedy[(size_t)i * B + b] : -1;
}

// ---------------------------------------------------------------- launchers

void launch_prep(const StepArgs& a, SeqDesc* seqs, RowDesc* rows, int* err, hipStream_t st) {
  hipLaunchKernelGGL(prep_seq_kernel, dim3((a.B + 3) / 4), dim3(256), 0, st, a, seqs, rows, err);
  if (a.layout == 1)
    hipLaunchKernelGGL(prep_row_kernel, dim3((a.rows + 255) / 256), dim3(256), 0, st, a, seqs, rows);
}

void launch_embed(int M, int d, const RowDesc* rows, const void* tok, const void* pos, float* x,
                  const float* in_rows, hipStream_t st) {
  hipLaunchKernelGGL(embed_kernel, dim3(M), dim3(256), 0, st, d, rows, (const float*)tok, (const float*)pos, x,
                     in_rows);
}

void launch_layernorm(int M, int d, const float* x, const void* g, const void* b, float* out,
                      hipStream_t st) {
  hipLaunchKernelGGL(layernorm_kernel, dim3(M), dim3(256), 0, st, d, x, (const float*)g, (const float*)b, out);
}

void launch_reduce_res_ln(int M, int d, int nsplit, const float* P, const void* bias, float* x,
                          const void* g, const void* b, uint16_t* frag, int RT, float* out,
                          hipStream_t st) {
  const int threads = (d / 4 + kWave - 1) / kWave * kWave;
  hipLaunchKernelGGL(reduce_res_ln_kernel, dim3(xcd_row_grid(M)), dim3(threads), 0, st, M, d, nsplit, P,
                     (const uint16_t*)bias, x, (const uint16_t*)g, (const uint16_t*)b, frag, RT, out);
}

void launch_embed_ln(int M, int d, const RowDesc* rows, const void* tok, const void* pos, float* x,
                     const float* in_rows, const void* g, const void* b, uint16_t* frag, int RT,
                     hipStream_t st) {
  const int threads = (d / 4 + kWave - 1) / kWave * kWave;
  hipLaunchKernelGGL(embed_ln_kernel, dim3(xcd_row_grid(M)), dim3(threads), 0, st, M, d, rows,
                     (const uint16_t*)tok, (const uint16_t*)pos, x, in_rows, (const uint16_t*)g,
                     (const uint16_t*)b, frag, RT);
}

// ---------------------------------------------------------------- draft-block inputs

// taps4[b] = [taps_0 ; taps_1 ; taps_2 ; hidden] at sequence b's last verified row (zeros
// for a skipped sequence).
__global__ void draft_gather_taps_kernel(int d, int layout, int k_max, const int* cu_rows,
                                         const int* accept_len, int rows, const float* taps,
                                         const float* hidden, float* taps4) {
  const int b = blockIdx.x;
  const int a = accept_len[b];
  const int row = (layout == 0 ? b * (k_max + 1) : cu_rows[b]) + (a < 0 ? 0 : a);
  for (int j = threadIdx.x; j < 4 * d; j += blockDim.x) {
    const int which = j / d, c = j % d;
    const float* src = which < 3 ? taps + ((size_t)which * rows + row) * d : hidden + (size_t)row * d;
    taps4[(size_t)b * 4 * d + j] = a < 0 ? 0.f : src[c];
  }
}

// z[b] = [feat[b] ; E_tok[token_b]], token_b = tokens[b * token_stride + (token_index ?
// token_index[b] : 0)] (a negative index, i.e. a skipped sequence, reads slot 0).
__global__ void draft_concat_kernel(int d, const float* feat, const float* tok_emb, const int* tokens,
                                    int token_stride, const int* token_index, float* z) {
  const int b = blockIdx.x;
  const int ti = token_index ? max(token_index[b], 0) : 0;
  const int t = max(tokens[(size_t)b * token_stride + ti], 0);
  for (int j = threadIdx.x; j < 2 * d; j += blockDim.x)
    z[(size_t)b * 2 * d + j] = j < d ? feat[(size_t)b * d + j] : tok_emb[(size_t)t * d + (j - d)];
}

// window[b] = [max(0, c - half), min(T_b, c + half + 1)) around anchor c (a negative
// anchor, i.e. a skipped sequence, gives the first frame).
__device__ __forceinline__ void draft_window(int b, const int* anchor, const int* enc_len, int half, int* window) {
  const int c = max(anchor[b], 0), T = max(enc_len[b], 1);
  const int lo = max(0, min(c - half, T - 1));
  window[2 * b] = lo;
  window[2 * b + 1] = max(lo + 1, min(T, c + half + 1));
}
__global__ void draft_window_kernel(int B, const int* anchor, const int* enc_len, int half, int* window) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b < B) draft_window(b, anchor, enc_len, half, window);
}

// Four consecutive floats of a caller's array (16-byte aligned or not).
__device__ __forceinline__ float4 load4(const float* p, bool aligned) {
  return aligned ? *(const float4*)p : float4{p[0], p[1], p[2], p[3]};
}

// The two inputs of the bf16 model's draft projections, in A-fragment order: four columns per
// thread, one workgroup per sequence and d columns (these kernels are a launch and one chain
// of dependent loads each; one workgroup per sequence with a column at a time took 11.5 us for
// the 5120 gathered columns and 6.8 us for the 2560 concatenated ones; now 4.0 and 3.5 us, the
// split sum, 4.1 us before, and the window included).
__global__ void __launch_bounds__(1024) draft_gather_taps_frag_kernel(int d, int layout, int k_max,
                                                                      const int* cu_rows,
                                                                      const int* accept_len, int rows,
                                                                      const float* taps, const float* hidden,
                                                                      bool aligned, uint16_t* frag, int RT) {
  const int b = blockIdx.x, which = blockIdx.y, c = threadIdx.x * 4;
  if (c >= d) return;
  const int a = accept_len[b];
  const int row = (layout == 0 ? b * (k_max + 1) : cu_rows[b]) + (a < 0 ? 0 : a);
  const float* src = which < 3 ? taps + ((size_t)which * rows + row) * d : hidden + (size_t)row * d;
  const float4 v = load4(src + c, aligned);
  afrag_store4(frag, RT, b, which * d + c, a < 0 ? float4{0.f, 0.f, 0.f, 0.f} : v);
}

// [f_b ; E_tok[token_b]]: f_b = the feature row, or (nsplit > 0) the first projection's split
// sum plus its bias.  The window of an anchored step is written here too.
__global__ void __launch_bounds__(1024) draft_concat_frag_kernel(int d, const float* feat, bool aligned,
                                                                 int nsplit, const float* P,
                                                                 const uint16_t* bias, const uint16_t* tok_emb,
                                                                 const int* tokens, int token_stride,
                                                                 const int* token_index, uint16_t* frag, int RT,
                                                                 const int* anchor, const int* enc_len, int half,
                                                                 int* window) {
  const int b = blockIdx.x, c = threadIdx.x * 4;
  if (blockIdx.y == 1 && threadIdx.x == 0 && anchor) draft_window(b, anchor, enc_len, half, window);
  if (c >= d) return;
  float4 v;
  if (blockIdx.y == 1) {
    const int ti = token_index ? max(token_index[b], 0) : 0;
    const int t = max(tokens[(size_t)b * token_stride + ti], 0);
    v = ld_bf16x4(tok_emb + (size_t)t * d, c);
  } else if (nsplit > 0) {
    const float4 bb = ld_bf16x4(bias, c);
    v = split_sum4_flat(P, (size_t)gridDim.x * d, (size_t)b * d + c, nsplit);
    v.x += bb.x; v.y += bb.y; v.z += bb.z; v.w += bb.w;
  } else {
    v = load4(feat + (size_t)b * d + c, aligned);
  }
  afrag_store4(frag, RT, b, blockIdx.y * d + c, v);
}

__global__ void sum_partials_bias_kernel(int M, int N, int nsplit, const float* P,
                                         const uint16_t* bias, float* out) {
  const int m = blockIdx.x;
  for (int j = threadIdx.x * 4; j < N; j += blockDim.x * 4) {
    const size_t e = (size_t)m * N + j;
    float4 v = split_sum4_flat(P, (size_t)M * N, e, nsplit);
    const float4 bb = ld_bf16x4(bias, j);
    v.x += bb.x; v.y += bb.y; v.z += bb.z; v.w += bb.w;
    *(float4*)(out + e) = v;
  }
}

static int quad_threads(int d) { return (d / 4 + kWave - 1) / kWave * kWave; }   // at most 1024 (d <= 4096)

void launch_draft_gather_taps_frag(int B, int d, int layout, int k_max, const int* cu_rows,
                                   const int* accept_len, int rows, const float* taps,
                                   const float* hidden, uint16_t* frag, int RT, hipStream_t st) {
  const bool aligned = ((uintptr_t)taps | (uintptr_t)hidden) % 16 == 0;
  hipLaunchKernelGGL(draft_gather_taps_frag_kernel, dim3(B, 4), dim3(quad_threads(d)), 0, st, d, layout, k_max,
                     cu_rows, accept_len, rows, taps, hidden, aligned, frag, RT);
}

void launch_draft_concat_frag(int B, int d, const float* feat, int nsplit, const float* P, const void* bias,
                              const void* tok_emb, const int* tokens, int token_stride, const int* token_index,
                              uint16_t* frag, int RT, const int* anchor, const int* enc_len, int half,
                              int* window, hipStream_t st) {
  hipLaunchKernelGGL(draft_concat_frag_kernel, dim3(B, 2), dim3(quad_threads(d)), 0, st, d, feat,
                     (uintptr_t)feat % 16 == 0, nsplit, P, (const uint16_t*)bias, (const uint16_t*)tok_emb, tokens,
                     token_stride, token_index, frag, RT, anchor, enc_len, half, window);
}

void launch_sum_partials_bias(int M, int N, int nsplit, const float* P, const void* bias, float* out,
                              hipStream_t st) {
  hipLaunchKernelGGL(sum_partials_bias_kernel, dim3(M), dim3(256), 0, st, M, N, nsplit, P,
                     (const uint16_t*)bias, out);
}

void launch_draft_gather_taps(int B, int d, int layout, int k_max, const int* cu_rows,
                              const int* accept_len, int rows, const float* taps,
                              const float* hidden, float* taps4, hipStream_t st) {
  hipLaunchKernelGGL(draft_gather_taps_kernel, dim3(B), dim3(256), 0, st, d, layout, k_max, cu_rows,
                     accept_len, rows, taps, hidden, taps4);
}

void launch_draft_concat(int B, int d, const float* feat, const void* tok_emb, const int* tokens,
                         int token_stride, const int* token_index, float* z,
                         hipStream_t st) {
  hipLaunchKernelGGL(draft_concat_kernel, dim3(B), dim3(256), 0, st, d, feat, (const float*)tok_emb, tokens,
                     token_stride, token_index, z);
}

void launch_draft_window(int B, const int* anchor, const int* enc_len, int half, int* window,
                         hipStream_t st) {
  hipLaunchKernelGGL(draft_window_kernel, dim3((B + 127) / 128), dim3(128), 0, st, B, anchor,
                     enc_len, half, window);
}

void launch_argmax_final(int M, int nrec, const void* part, const RowDesc* rows, int* greedy,
                         float* margin, int* err, hipStream_t st) {
  hipLaunchKernelGGL(argmax_final_kernel, dim3(M), dim3(64), 0, st, M, nrec, (const float4*)part,
                     rows, greedy, margin, err);
}

void launch_accept(int B, int k_max, const SeqDesc* seqs, const int* tokens, const int* greedy,
                   int* accept_len, int* out_tokens, hipStream_t st) {
  hipLaunchKernelGGL(accept_kernel, dim3((B + 127) / 128), dim3(128), 0, st, B, k_max, seqs, tokens,
                     greedy, accept_len, out_tokens);
}

void launch_accept_tree(int B, int k_max, const SeqDesc* seqs, const int* tokens, const int* parents,
                        const int* greedy, int* accept_len, int* out_tokens, int* out_path,
                        hipStream_t st) {
  hipLaunchKernelGGL(accept_tree_kernel, dim3((B + 127) / 128), dim3(128), 0, st, B, k_max, seqs,
                     tokens, parents, greedy, accept_len, out_tokens, out_path);
}

template <class S>
void launch_kv_compact(int B, int L, int H, const int* kv_len, const int* accept_len, const int* path,
                       int path_stride, void* pool, int num_pages, const int* block_table,
                       int pages_per_seq, hipStream_t st) {
  hipLaunchKernelGGL(kv_compact_kernel<S>, dim3(B, 2 * L), dim3(256), 0, st, H, kv_len, accept_len,
                     path, path_stride, (typename S::T*)pool, num_pages, block_table, pages_per_seq);
}
template void launch_kv_compact<F32>(int, int, int, const int*, const int*, const int*, int, void*, int,
                                     const int*, int, hipStream_t);
template void launch_kv_compact<BF16>(int, int, int, const int*, const int*, const int*, int, void*, int,
                                      const int*, int, hipStream_t);

void launch_commit(int B, int* kv_len, const int* accept_len, hipStream_t st) {
  hipLaunchKernelGGL(commit_kernel, dim3((B + 127) / 128), dim3(128), 0, st, B, kv_len, accept_len);
}

template <class S>
void launch_kv_copy(bool to_linear, int L, int H, int n, int b, void* lin, void* pool, int num_pages,
                    const int* block_table, int pages_per_seq, int* err, hipStream_t st) {
  const size_t total = (size_t)L * 2 * n * H * kHead;
  if (total == 0) return;
  if ((uintptr_t)lin % 16 == 0 && (uintptr_t)pool % 16 == 0) {   // whole 16-byte pieces
    const dim3 tiles((n + kTile - 1) / kTile, 2 * L, (H + kCopyHeads - 1) / kCopyHeads);
    if (to_linear)
      hipLaunchKernelGGL((kv_copy_tile_kernel<S, true>), tiles, dim3(256), 0, st, H, n, b, (typename S::T*)lin,
                         (typename S::T*)pool, num_pages, block_table, pages_per_seq, err);
    else
      hipLaunchKernelGGL((kv_copy_tile_kernel<S, false>), tiles, dim3(256), 0, st, H, n, b, (typename S::T*)lin,
                         (typename S::T*)pool, num_pages, block_table, pages_per_seq, err);
    return;
  }
  const dim3 grid((unsigned)((total + 255) / 256));
  if (to_linear)
    hipLaunchKernelGGL((kv_copy_kernel<S, true>), grid, dim3(256), 0, st, L, H, n, b,
                       (typename S::T*)lin, (typename S::T*)pool, num_pages, block_table,
                       pages_per_seq, err);
  else
    hipLaunchKernelGGL((kv_copy_kernel<S, false>), grid, dim3(256), 0, st, L, H, n, b,
                       (typename S::T*)lin, (typename S::T*)pool, num_pages, block_table,
                       pages_per_seq, err);
}
template void launch_kv_copy<F32>(bool, int, int, int, int, void*, void*, int, const int*, int, int*, hipStream_t);
template void launch_kv_copy<BF16>(bool, int, int, int, int, void*, void*, int, const int*, int, int*, hipStream_t);

void launch_gather_hidden(int B, int d, int layout, int k_max, const int* cu_rows,
                          const int* accept_len, const float* hidden, float* hsel, hipStream_t st) {
  hipLaunchKernelGGL(gather_hidden_kernel, dim3(B), dim3(256), 0, st, B, d, layout, k_max, cu_rows,
                     accept_len, hidden, hsel);
}

void launch_assemble_next(int B, int n_heads, int k_max, const int* accept_len, const int* out_tokens,
                          const int* head_greedy, int* next_tokens, hipStream_t st) {
  hipLaunchKernelGGL(assemble_next_kernel, dim3((B + 127) / 128), dim3(128), 0, st, B, n_heads, k_max,
                     accept_len, out_tokens, head_greedy, next_tokens);
}

}  // namespace ad

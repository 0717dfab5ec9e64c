// Thought-adaptive eviction: which tokens of a thought segment survive (Sec. 4.3 of the paper,
// "Think Before you Evict"; appendix "TBE Eviction Policy").  A segment picked for eviction is
// cut down to K = min(|segment|, R_n) tokens by K-means over its post-RoPE keys: one
// representative key-value pair per cluster survives, the member nearest the centroid.
//
// The paper names K-means and nothing else.  What is built:
//   points     the token's stored keys, dequantised in binary32 (fmaf(code, scale, zp)), all
//              kv-heads concatenated (eviction is per token, so one clustering serves all heads)
//   K >= N     everything survives
//   init       centroid j = point floor(j * N / K)
//   Lloyd      nearest centroid by squared distance (ties -> lowest cluster); stop when no
//              assignment changed or after max_iters assignments; else centroids move to the
//              means of their points (an emptied cluster keeps its centroid)
//   survivors  per non-empty cluster the member nearest the centroid (ties -> lowest index; of
//              two members the earlier one: both are equally near their mean)
//
// Two kernels.  gather writes the key rows [Hkv * D] of the listed tokens into the workspace.
// kmeans: one workgroup of sixteen waves per segment (segments hold at most 256 live tokens, the
// schedule keeps at most 64).  A centroid is the mean of points, so every product Lloyd's algorithm asks for is a
// mean of products between points: x.c_j = mean over the members i of x.x_i, |c_j|^2 = mean over the members of
// x_i.c_j.  So the channels are walked once: all products between the points of the segment (the Gram matrix, at most
// 256 x 256, its lower triangle kept in LDS), and an iteration is n^2 additions from LDS.  (Products of the points with
// the centroids in every iteration walked all channels up to nine times: 314 segments of ~110 tokens, 1,024 channels,
// 1,050 us; now 177, and the gather 37.)  A centroid is represented by the set of points it is the mean of: at the start one
// point, later the members, and for a cluster that has lost its last member the members it had before.
// The products run on the matrix cores; a dequantised key does not
// fit binary16 and the binary32 matrix instruction is slow, so every number enters as the sum of
// two binary16 parts (22 significant bits) and a product is three binary16 MFMAs.  The error of
// all this is of the order of 1e-6 of |x|^2, far below the gaps that separate genuine decisions;
// an assignment only needs |c|^2 - 2 x.c.  All sums run in index order or in a fixed tree, so the result is the same on
// every run; the survivor of a cluster is found with a 64-bit LDS minimum over (distance bits, index).
#include <type_traits>

#include "common.h"

namespace thinkv {

constexpr int kTbeMaxTokens = THINKV_TBE_MAX_SEGMENT;   // live tokens of one segment
constexpr int kTbeMaxKeep = THINKV_TBE_MAX_KEEP;        // largest retention level
constexpr int kTile = 64;                               // channels per LDS tile

struct TbeArgs {
  const int32_t* tok_seq;
  const int32_t* tok_handle;
  const int32_t* seg_offset;
  const int32_t* seg_keep;
  int32_t* ev_handle;
  float* x;      // [n_tok][dim]
  float* cent;   // [n_seg][kTbeMaxKeep][dim]
  int32_t* assign;   // [n_tok] cluster of every token at the last assignment (-1: its segment was not clustered)
  int layer, n_seg, n_tok, max_iters, dim;
};

size_t tbe_ws_bytes(const thinkv_config& c, int n_tok, int n_seg) {
  const size_t dim = (size_t)c.n_kv_heads * c.head_dim;
  return ((size_t)(n_tok > 0 ? n_tok : 1) * dim + (size_t)(n_seg > 0 ? n_seg : 1) * kTbeMaxKeep * dim) * sizeof(float) +
         (size_t)(n_tok > 0 ? n_tok : 1) * sizeof(int32_t) + 256;
}

// ---- gather: x[i][hd * D + ch] = the stored key of token i.  A workgroup takes kGatherTokens tokens: one thread per
// token walks the chain handle -> page list -> page; then a thread takes one chunk of a token's block (a kv-head, eight
// channels of every group: one vector load of codes) and writes eight channels of each group as two 16-byte stores, four
// neighbours 128 bytes.  Bound by those stores (four bytes a channel): 34,500 tokens of 1,024 channels (141 MB) 44 us
// (one channel a thread: 84).
constexpr int kGatherTokens = 8;

template <int D, int BITS>
__device__ __forceinline__ void gather_chunk(const thinkv_config& c, const uint8_t* blk, int j, int slot, bool fp, float* row) {
  constexpr int NG = D / kGroup, FPH = 16 / BITS, CW = NG * BITS / 4;
  const BlockGeom g = block_geom(BITS, D, c.format);
  uint32_t codes[CW];
#pragma unroll
  for (int w = 0; w < CW; ++w) codes[w] = ((const uint32_t*)(blk + g.k_codes + (16 * j + slot) * g.chunk_bytes))[w];
#pragma unroll
  for (int grp = 0; grp < NG; ++grp) {
    float sc, zp = 0.f;
    if (fp) {   // the eight channels lie in the group of 16 number 2 grp + j / 2
      sc = BITS == 8 ? c.fp8_scale[0] : e4m3_value(blk[g.k_meta + (2 * grp + (j >> 1)) * kPage + slot]);
    } else {
      const _Float16* meta = (const _Float16*)(blk + g.k_meta);
      sc = (float)meta[meta_index(slot, grp)];
      zp = (float)meta[meta_index(slot, grp) + 4];
    }
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int f = 4 * grp + (e >> 1);
      const uint32_t raw = (codes[f / FPH] >> (16 * (e & 1) + BITS * (f % FPH))) & ((1u << BITS) - 1u);
      x[e] = fp ? fp_code_value(raw, BITS) * sc : fmaf((float)raw, sc, zp);
    }
    float* dst = row + 32 * grp + 8 * j;
    *(float4*)dst = make_float4(x[0], x[1], x[2], x[3]);
    *(float4*)(dst + 4) = make_float4(x[4], x[5], x[6], x[7]);
  }
}

template <int D>
__global__ __launch_bounds__(256) void tbe_gather_kernel(thinkv_view v, TbeArgs a) {
  const thinkv_config& c = v.cfg;
  const int tid = threadIdx.x, i0 = blockIdx.x * kGatherTokens;
  const int H = c.n_kv_heads;
  __shared__ int s_ok[kGatherTokens], s_cls[kGatherTokens], s_slot[kGatherTokens], s_pid[kGatherTokens];
  if (tid < kGatherTokens) {
    const int i = i0 + tid;
    int ok = 0, cls = 0, slot = 0, pid = 0;
    if (i < a.n_tok) {
      const int s = a.tok_seq[i];
      const int32_t h = a.tok_handle[i];
      const uint32_t uh = (uint32_t)h;
      cls = uh >> 28;
      slot = uh & 15;
      const int pi = (uh >> 4) & 0xFFFFFF;
      if (s < 0 || s >= c.max_seqs) {
        atomicOr(&v.dev_status[c.max_seqs * c.n_layers], THINKV_ST_BAD_SEQ);
      } else if (h < 0 || cls > 2 || pi >= v.n_pages[npages_index(c, s, a.layer, cls)]) {
        atomicOr(&v.dev_status[sl_index(c, s, a.layer)], THINKV_ST_BAD_SLOT);
      } else {
        pid = v.block_table[table_base(c, s, a.layer, cls) + pi];
        ok = 1;
      }
    }
    s_ok[tid] = ok; s_cls[tid] = cls; s_slot[tid] = slot; s_pid[tid] = pid;
  }
  __syncthreads();
  const bool fp = c.format == THINKV_FMT_FP;
  const int per = 4 * H;   // chunks of a token
  for (int idx = tid; idx < kGatherTokens * per; idx += 256) {
    const int t = idx / per, hd = (idx % per) >> 2, j = idx & 3;
    if (i0 + t >= a.n_tok) continue;
    float* row = a.x + (int64_t)(i0 + t) * a.dim + hd * D;
    if (!s_ok[t]) {   // a token that does not exist clusters as the origin and is never evicted
      for (int grp = 0; grp < D / kGroup; ++grp) {
        *(float4*)(row + 32 * grp + 8 * j) = make_float4(0.f, 0.f, 0.f, 0.f);
        *(float4*)(row + 32 * grp + 8 * j + 4) = make_float4(0.f, 0.f, 0.f, 0.f);
      }
      continue;
    }
    const int cls = s_cls[t], bits = c.bits_of_class[cls];
    const BlockGeom g = block_geom(bits, D, c.format);
    const uint8_t* blk = v.arena[cls] + ((int64_t)s_pid[t] * H + hd) * g.block_bytes;
    if (bits == 2) gather_chunk<D, 2>(c, blk, j, s_slot[t], fp, row);
    else if (bits == 4) gather_chunk<D, 4>(c, blk, j, s_slot[t], fp, row);
    else gather_chunk<D, 8>(c, blk, j, s_slot[t], fp, row);
  }
}

// ---- kmeans
constexpr int kPT = kTbeMaxTokens / 64;   // tokens per lane of a wave that sorts a list
constexpr int kKmThreads = 1024;          // sixteen waves
constexpr int kQuarters = kKmThreads / kTbeMaxTokens;   // threads per point: each looks at every fourth cluster
constexpr int kClPerThread = kTbeMaxKeep / kQuarters;
constexpr int kMacro = 32;                // points on a side of a wave's piece of the Gram matrix (2 x 2 MFMA tiles)
constexpr int kMacroMax = (kTbeMaxTokens / kMacro) * (kTbeMaxTokens / kMacro + 1) / 2;   // pieces of the lower triangle: 36
constexpr int kMacroPerWave = (kMacroMax + kKmThreads / 64 - 1) / (kKmThreads / 64);     // 3
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
constexpr int kPadH = 2 * kTile + 8;   // binary16 numbers per tile row: high parts, low parts, padding (an odd multiple of 16 bytes)

__device__ __forceinline__ int tri(int i) { return i * (i + 1) / 2; }   // where row i of the lower triangle begins

struct KmScratch {
  union {
    _Float16 xs[kTbeMaxTokens][kPadH];                       // one tile: 64 channels of every point, each as high + low binary16 part
    float gram[kTbeMaxTokens * (kTbeMaxTokens + 1) / 2];     // then the products of all pairs of points, lower triangle
  };
  uint32_t basis[kTbeMaxKeep][kTbeMaxTokens / 32];           // the points a cluster's centroid is the mean of,
  uint32_t next[kTbeMaxKeep][kTbeMaxTokens / 32];            // its members under the assignment just made
  float own[kTbeMaxTokens];                                  // product of a point with the centroid it belongs to
  float cc[kTbeMaxKeep];                                     // squared norms of the centroids
  int cnt[kTbeMaxKeep], moved[kTbeMaxKeep];                  // points of the basis; whether it changed last
  int cluster[kTbeMaxTokens];                                // cluster whose basis the point is in (-1: none)
  float bd[kQuarters][kTbeMaxTokens];                        // per quarter of the clusters: best distance of every point ...
  int bj[kQuarters][kTbeMaxTokens];                          // ... and the cluster it belongs to
  int low[kTbeMaxKeep];                                      // survivors: lowest index of every cluster
  unsigned long long best[kTbeMaxKeep];
};

// four channels into a tile row: x = hi + lo with hi = binary16(x), lo = binary16(x - hi), 22 significant bits
__device__ inline void store_split(_Float16* row, int c, float4 v) {
  const f16x4 hi = {(_Float16)v.x, (_Float16)v.y, (_Float16)v.z, (_Float16)v.w};
  const f16x4 lo = {(_Float16)(v.x - (float)hi[0]), (_Float16)(v.y - (float)hi[1]), (_Float16)(v.z - (float)hi[2]),
                    (_Float16)(v.w - (float)hi[3])};
  *(f16x4*)&row[c] = hi;
  *(f16x4*)&row[kTile + c] = lo;
}

// sm.gram: the products of all pairs of the n points.  The channels go through LDS 64 at a time (the loads of the next two
// tiles are in flight while the current one is worked on); wave w owns the pieces w, w + 16, w + 32 of the lower
// triangle, 32 x 32 points each: 2 x 2 tiles share their operands, which halves the LDS reads a product costs.  A product
// is hi.hi + hi.lo + lo.hi (exact products, binary32 sums; what is dropped is of the order of 2^-22 of |x||y|).
__device__ inline void gram_matrix(const float* __restrict__ x, int n, int dim, KmScratch& sm) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, g = lane >> 4;
  const int mb = (n + kMacro - 1) / kMacro, pieces = mb * (mb + 1) / 2;
  constexpr int kC4 = kTile / 4;                           // float4 per tile row
  constexpr int kXQ = kTbeMaxTokens * kC4 / kKmThreads;    // float4 loads per thread at most
  const int xq = (mb * kMacro * kC4 + kKmThreads - 1) / kKmThreads;
  int pi[kMacroPerWave], pj[kMacroPerWave];                // block row and column of the wave's pieces
  f32x4 acc[kMacroPerWave][2][2];
#pragma unroll
  for (int t = 0; t < kMacroPerWave; ++t) {
    int rest = wave + t * (kKmThreads / 64), i = 0;
    while (rest > i) rest -= ++i;
    pi[t] = i;
    pj[t] = rest;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int w = 0; w < 2; ++w) acc[t][u][w] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  float4 pa[kXQ], pb[kXQ];   // two tiles ahead, used in turn
  auto fetch = [&](int d0, float4 (&px)[kXQ]) {
#pragma unroll
    for (int q = 0; q < kXQ; ++q)
      if (q < xq) {
        const int idx = tid + kKmThreads * q, row = idx / kC4, c4 = idx % kC4;
        px[q] = row < n && d0 < dim ? *(const float4*)&x[(int64_t)row * dim + d0 + 4 * c4] : make_float4(0.f, 0.f, 0.f, 0.f);
      }
  };
  auto tile = [&](int d0, float4 (&px)[kXQ]) {
    __syncthreads();   // the previous tile has been used
#pragma unroll
    for (int q = 0; q < kXQ; ++q)
      if (q < xq) {
        const int idx = tid + kKmThreads * q;
        store_split(sm.xs[idx / kC4], 4 * (idx % kC4), px[q]);
      }
    __syncthreads();
    fetch(d0 + 2 * kTile, px);
#pragma unroll
    for (int t = 0; t < kMacroPerWave; ++t)
      if (wave + t * (kKmThreads / 64) < pieces) {
#pragma unroll
        for (int ks = 0; ks < kTile / 32; ++ks) {
          // lane (r, g) holds channels 32 ks + 8 g .. + 7 of its row, on both sides
          f16x8 ah[2], al[2], bh[2], bl[2];
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const _Float16* ra = sm.xs[kMacro * pi[t] + 16 * u + r];
            const _Float16* rb = sm.xs[kMacro * pj[t] + 16 * u + r];
            ah[u] = *(const f16x8*)&ra[32 * ks + 8 * g];
            al[u] = *(const f16x8*)&ra[kTile + 32 * ks + 8 * g];
            bh[u] = *(const f16x8*)&rb[32 * ks + 8 * g];
            bl[u] = *(const f16x8*)&rb[kTile + 32 * ks + 8 * g];
          }
#pragma unroll
          for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int w = 0; w < 2; ++w) {
              acc[t][u][w] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[u], bh[w], acc[t][u][w], 0, 0, 0);
              acc[t][u][w] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[u], bl[w], acc[t][u][w], 0, 0, 0);
              acc[t][u][w] = __builtin_amdgcn_mfma_f32_16x16x32_f16(al[u], bh[w], acc[t][u][w], 0, 0, 0);
            }
        }
      }
  };
  fetch(0, pa);
  fetch(kTile, pb);
  for (int d0 = 0; d0 < dim; d0 += 2 * kTile) {
    tile(d0, pa);
    if (d0 + kTile < dim) tile(d0 + kTile, pb);
  }
  __syncthreads();   // the last tile has been used: its place becomes the matrix
#pragma unroll
  for (int t = 0; t < kMacroPerWave; ++t)
    if (wave + t * (kKmThreads / 64) < pieces) {
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int w = 0; w < 2; ++w)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int p = kMacro * pi[t] + 16 * u + 4 * g + i, q = kMacro * pj[t] + 16 * w + r;
            if (p < n && q <= p) sm.gram[tri(p) + q] = acc[t][u][w][i];
          }
    }
  __syncthreads();
}

// f(point) for every point of a cluster's basis, in index order; the point is the same in all lanes
template <class F>
__device__ __forceinline__ void for_basis(const uint32_t* mask, F f) {
#pragma unroll
  for (int w = 0; w < kTbeMaxTokens / 32; ++w) {
    uint32_t m = __builtin_amdgcn_readfirstlane(mask[w]);
    while (m) {
      const int i = __builtin_ctz(m);
      m &= m - 1;
      f(32 * w + i);
    }
  }
}

// Products of every point with every centroid that has one: thread (point tid % 256, quarter tid / 256) leaves those of the
// clusters quarter, quarter + 4, ... in dot[]; sm.own of the points that are in a basis; sm.cc of the centroids that moved.
__device__ inline void centroid_products(int n, int k, KmScratch& sm, float (&dot)[kClPerThread]) {
  const int tid = threadIdx.x, p = tid & (kTbeMaxTokens - 1), lane = tid & 63;
  const int quarter = __builtin_amdgcn_readfirstlane(tid / kTbeMaxTokens), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pc = p < n ? p : n - 1, tp = tri(pc);
  const int mine = sm.cluster[p];
  const bool idle = (p & ~63) >= n;   // no point of the wave exists
#pragma unroll
  for (int i = 0; i < kClPerThread; ++i) {
    const int j = quarter + kQuarters * i;
    dot[i] = 0.f;
    if (j < k && !idle) {
      float sum = 0.f;
      for_basis(sm.basis[j], [&](int m) { sum += sm.gram[pc >= m ? tp + m : tri(m) + pc]; });
      dot[i] = sum * (1.0f / (float)sm.cnt[j]);
      if (mine == j && p < n) sm.own[p] = dot[i];
    }
  }
  __syncthreads();
  // |c|^2 = mean over the basis of its points' products with the centroid: a wave per cluster, a fixed tree
  for (int j = wave; j < k; j += kKmThreads / 64) {
    if (!sm.moved[j]) continue;
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < kTbeMaxTokens / 64; ++w) {
      const int q = 64 * w + lane;
      if (sm.basis[j][q >> 5] >> (q & 31) & 1u) sum += sm.own[q];
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) sum += __shfl_xor(sum, d, 64);
    if (lane == 0) sm.cc[j] = sum * (1.0f / (float)sm.cnt[j]);
  }
  __syncthreads();
}

__global__ __launch_bounds__(kKmThreads) void tbe_kmeans_kernel(thinkv_view v, TbeArgs a) {
  const thinkv_config& c = v.cfg;
  const int seg = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lo = a.seg_offset[seg], hi = a.seg_offset[seg + 1];
  const int n = hi - lo, want = a.seg_keep[seg];
  if (n <= 0) return;
  if (n > kTbeMaxTokens || want > kTbeMaxKeep || want < 1 || lo < 0 || hi > a.n_tok) {
    // outside what this kernel covers: nothing is evicted, and the caller is told
    if (tid == 0) atomicOr(&v.dev_status[c.max_seqs * c.n_layers], THINKV_ST_BAD_SEGMENT);
    for (int i = tid; i < n && lo >= 0 && lo + i < a.n_tok; i += kKmThreads) {
      a.ev_handle[lo + i] = -1;
      a.assign[lo + i] = -1;
    }
    return;
  }
  if (want >= n) {
    for (int i = tid; i < n; i += kKmThreads) {
      a.ev_handle[lo + i] = -1;
      a.assign[lo + i] = -1;
    }
    return;
  }
  const int k = want, dim = a.dim;
  const float* x = a.x + (int64_t)lo * dim;
  float* cent = a.cent + (int64_t)seg * kTbeMaxKeep * dim;
  __shared__ __attribute__((aligned(16))) KmScratch sm;
  // initial centroids: evenly spaced points
  for (int i = tid; i < kTbeMaxKeep * (kTbeMaxTokens / 32); i += kKmThreads) (&sm.basis[0][0])[i] = 0u;
  if (tid < kTbeMaxTokens) sm.cluster[tid] = -1;
  __syncthreads();
  if (tid < k) {
    const int p = (tid * n) / k;   // distinct, since k < n
    sm.basis[tid][p >> 5] = 1u << (p & 31);
    sm.cluster[p] = tid;
    sm.cnt[tid] = 1;
    sm.moved[tid] = 1;
  }
  gram_matrix(x, n, dim, sm);
  const int p = tid & (kTbeMaxTokens - 1), quarter = tid / kTbeMaxTokens;
  float dot[kClPerThread];
  int mine = -1;   // this point's cluster at the last assignment
  bool converged = false;
  for (int it = 0; it < a.max_iters; ++it) {
    // centroids: the initial ones, later the means under the previous assignment
    centroid_products(n, k, sm, dot);
    // nearest cluster of every point: |c|^2 - 2 x.c decides (|x|^2 is common to a point's candidates); ties go to the
    // lowest cluster
    float bd = INFINITY;
    int bj = kTbeMaxKeep;
#pragma unroll
    for (int i = 0; i < kClPerThread; ++i) {
      const int j = quarter + kQuarters * i;
      const float d = j < k ? fmaf(-2.f, dot[i], sm.cc[j]) : INFINITY;
      if (d < bd) {
        bd = d;
        bj = j;
      }
    }
    sm.bd[quarter][p] = bd;
    sm.bj[quarter][p] = bj;
    for (int i = tid; i < kTbeMaxKeep * (kTbeMaxTokens / 32); i += kKmThreads) (&sm.next[0][0])[i] = 0u;
    __syncthreads();
    bd = sm.bd[0][p];
    bj = sm.bj[0][p];
#pragma unroll
    for (int w = 1; w < kQuarters; ++w) {
      const float od = sm.bd[w][p];
      const int oj = sm.bj[w][p];
      if (od < bd || (od == bd && oj < bj)) {
        bd = od;
        bj = oj;
      }
    }
    if (bj >= k) bj = 0;   // no candidate compares (the distances are not numbers): the first cluster, as a comparison that never holds leaves it
    const int changed = p < n && bj != mine;
    mine = bj;
    if (!__syncthreads_or(changed)) {
      converged = true;   // the products at hand are those with the final centroids
      break;
    }
    // members of every cluster; a cluster without any keeps its basis
    if (quarter == 0 && p < n) {
      sm.cluster[p] = mine;
      atomicOr(&sm.next[mine][p >> 5], 1u << (p & 31));
    }
    __syncthreads();
    if (tid < k) {
      int m = 0;
#pragma unroll
      for (int w = 0; w < kTbeMaxTokens / 32; ++w) m += __popc(sm.next[tid][w]);
      sm.moved[tid] = m > 0;
      if (m > 0) {
        sm.cnt[tid] = m;
#pragma unroll
        for (int w = 0; w < kTbeMaxTokens / 32; ++w) sm.basis[tid][w] = sm.next[tid][w];
      }
    }
    __syncthreads();
  }
  // ---- survivors: nearest member of every cluster under the final centroids
  if (!converged) centroid_products(n, k, sm, dot);
  if (tid < kTbeMaxKeep) {
    sm.low[tid] = kTbeMaxTokens;
    sm.best[tid] = ~0ull;
  }
  __syncthreads();
  if (quarter == 0 && p < n) {
    const float dist = fmaxf(fmaf(-2.f, sm.own[p], sm.gram[tri(p) + p]) + sm.cc[mine], 0.f);
    atomicMin(&sm.low[mine], p);
    // distances are not negative, so their bit patterns order like the numbers; the index breaks ties
    atomicMin(&sm.best[mine], ((unsigned long long)__builtin_bit_cast(uint32_t, dist) << 32) | (unsigned)p);
  }
  __syncthreads();
  if (quarter == 0 && p < n) {
    // two members are equally near their mean whatever the rounding says: the earlier one stays (a cluster with members
    // has them as its basis)
    const bool keep = sm.cnt[mine] <= 2 ? p == sm.low[mine] : (int)(sm.best[mine] & 0xFFFFFFFFull) == p;
    a.ev_handle[lo + p] = keep ? -1 : a.tok_handle[lo + p];
    a.assign[lo + p] = mine;
  }
  // ---- the centroids, for callers that look at them: a wave per cluster, up to 1,024 channels at a time (four loads a
  // lane in flight), members in index order
  for (int j = wave; j < k; j += kKmThreads / 64) {
    const float inv = 1.0f / (float)sm.cnt[j];
    for (int d0 = 4 * lane; d0 < dim; d0 += 1024) {
      float4 sum[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) sum[u] = make_float4(0.f, 0.f, 0.f, 0.f);
      for_basis(sm.basis[j], [&](int m) {
        float4 t[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) t[u] = d0 + 256 * u < dim ? *(const float4*)&x[(int64_t)m * dim + d0 + 256 * u] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          sum[u].x += t[u].x;
          sum[u].y += t[u].y;
          sum[u].z += t[u].z;
          sum[u].w += t[u].w;
        }
      });
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (d0 + 256 * u < dim) *(float4*)&cent[(int64_t)j * dim + d0 + 256 * u] = make_float4(sum[u].x * inv, sum[u].y * inv, sum[u].z * inv, sum[u].w * inv);
    }
  }
}

int launch_tbe_select(const thinkv_view& v, int layer, const int32_t* tok_seq, const int32_t* tok_handle, const int32_t* seg_offset,
                      const int32_t* seg_keep, int n_seg, int n_tok, int max_iters, int32_t* ev_handle, void* workspace,
                      hipStream_t st) {
  TbeArgs a;
  a.tok_seq = tok_seq;
  a.tok_handle = tok_handle;
  a.seg_offset = seg_offset;
  a.seg_keep = seg_keep;
  a.ev_handle = ev_handle;
  a.dim = v.cfg.n_kv_heads * v.cfg.head_dim;
  a.x = (float*)(((uintptr_t)workspace + 255) & ~(uintptr_t)255);
  a.cent = a.x + (size_t)n_tok * a.dim;
  a.assign = (int32_t*)(a.cent + (size_t)n_seg * kTbeMaxKeep * a.dim);
  a.layer = layer;
  a.n_seg = n_seg;
  a.n_tok = n_tok;
  a.max_iters = max_iters;
  const dim3 groups((n_tok + kGatherTokens - 1) / kGatherTokens);
  if (v.cfg.head_dim == 128)
    hipLaunchKernelGGL(tbe_gather_kernel<128>, groups, dim3(256), 0, st, v, a);
  else
    hipLaunchKernelGGL(tbe_gather_kernel<64>, groups, dim3(256), 0, st, v, a);
  hipLaunchKernelGGL(tbe_kmeans_kernel, dim3(n_seg), dim3(kKmThreads), 0, st, v, a);
  return hipGetLastError() == hipSuccess ? THINKV_OK : THINKV_E_HIP;
}

// ---------------------------------------------------------------------------------------------
// The plan: which segments of which sequences are cut, and to how many tokens (Sec. 4.3: Case 1,
// every preceding segment goes down one retention level when a transition segment has ended;
// Case 2, while the sequence holds more live tokens than the budget, the oldest segment of the
// least important type that can still shrink goes down one level).  A segment is cut at most
// once per call (one K-means per segment and call).  Its level follows from the number n of times
// it has been selected before (a column the caller keeps): it keeps min(live, R_n) tokens, and a
// selection that removes nothing only advances n (problem statement "Thought-Adaptive Eviction");
// or, as an option for callers without that column, from its live size: it is cut to the largest
// retention value below that size.  The open (last) segment is never touched.
// A live token belongs to the segment whose start is the largest one not above its position
// (the block table's start-index column, Sec. 5.2).
//
// Three kernels.  count (one workgroup per examined sequence): live tokens per segment (a thread takes four slots of a page:
// one load of positions, a binary search in the segment starts, held in LDS, where a slot leaves the segment of the one
// before), then the plan, whose cuts wait in a staging area.  fill (one workgroup per sequence): the sequence's place in
// the dense output lists from the totals of the sequences before it; where the lists are too short for all, the sequences
// in order keep the leading cuts that still fit (the rest waits for the next call).  Then the list offsets of its cuts by a
// prefix sum, and its live tokens are dealt to their lists.  sort (one wave per cut): each list is put in ascending
// position by a rank sort in LDS, so the output does not depend on the order in which threads
// got there.  32 sequences of 2k to 4k tokens, 314 cuts, us, with sixteen slots of three pages a thread, one thread for the
// second case and a kernel for the offsets / now: count 39 / 11, offsets 9 / -, fill 32 / 9, sort 19 / 10.
constexpr int kMaxSegs = THINKV_TBE_MAX_SEGS;
constexpr int kRetention[5] = {64, 32, 16, 8, 4};
constexpr int kPlanThreads = 1024;

struct PlanArgs {
  const int32_t* seq_ids;
  const int32_t* seg_start;
  const uint8_t* seg_type;
  const int32_t* n_segs;
  const uint8_t* transition_ended;
  int32_t* seg_count;   // [max_seqs][max_segs] selections so far (rule THINKV_TBE_BY_COUNT)
  int rule;
  int32_t* tok_seq;
  int32_t* tok_handle;
  int32_t* seg_offset;
  int32_t* seg_keep;
  int32_t* counts;
  // staging: per examined sequence max_cuts entries of (segment, keep, live tokens); the number of
  // cuts and of their tokens; per cut of the dense lists the sequence it belongs to
  int32_t* st_seg;
  int32_t* st_keep;
  int32_t* st_cnt;
  int32_t* st_ncuts;
  int32_t* st_total;
  int32_t* st_cut_seq;
  int layer, B, max_segs, budget, max_cuts, cap_seg, cap_tok;
};

size_t tbe_plan_ws_bytes(int B, int max_cuts) {
  return ((size_t)(B > 0 ? B : 1) * (4 * (size_t)max_cuts + 4)) * sizeof(int32_t) + 256;
}

__device__ inline int next_level(int size) {
#pragma unroll
  for (int i = 0; i < 5; ++i)
    if (kRetention[i] < size) return kRetention[i];
  return 0;
}

// segment of position pos: index of the last start <= pos, -1 if there is none
__device__ inline int segment_of(const int* starts, int n, int pos) {
  int lo = 0, hi = n;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (starts[mid] <= pos) lo = mid + 1; else hi = mid;
  }
  return lo - 1;
}

// calls f(segment, position, handle) for every live token of the sequence.  A thread takes four slots of a page, a pass two
// such pieces.  The walk is a chain of dependent loads (page count -> live mask and page id -> four positions) and little
// else; four slots keep the code behind it short.
template <typename F>
__device__ __forceinline__ void for_live_tokens(const thinkv_view& v, int seq, int layer, const int* s_start, int ns, F f) {
  const thinkv_config& c = v.cfg;
  constexpr int kAhead = 2;
  int np[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) np[k] = v.n_pages[npages_index(c, seq, layer, k)];
  const int pieces = 4 * (np[0] + np[1] + np[2]), quarter = threadIdx.x & 3;
  for (int u0 = threadIdx.x; u0 < pieces; u0 += kAhead * kPlanThreads) {
    uint32_t m[kAhead];
    int pid[kAhead], cls[kAhead], pi[kAhead];
    int4 pos[kAhead];
#pragma unroll
    for (int a = 0; a < kAhead; ++a) {
      const int u = u0 + a * kPlanThreads;
      int page = (u < pieces ? u : u0) >> 2;
      cls[a] = page < np[0] ? 0 : page < np[0] + np[1] ? 1 : 2;
      pi[a] = page - (cls[a] == 0 ? 0 : cls[a] == 1 ? np[0] : np[0] + np[1]);
      const int64_t at = table_base(c, seq, layer, cls[a]) + pi[a];
      m[a] = u < pieces ? v.slot_mask[at] >> (4 * quarter) & 15u : 0u;
      pid[a] = v.block_table[at];
    }
#pragma unroll
    for (int a = 0; a < kAhead; ++a)
      if (m[a]) {
        const int32_t* sp = cls[a] == 0 ? v.slot_pos[0] : cls[a] == 1 ? v.slot_pos[1] : v.slot_pos[2];
        pos[a] = *(const int4*)(sp + (int64_t)pid[a] * kPage + 4 * quarter);
      }
#pragma unroll
    for (int a = 0; a < kAhead; ++a) {
      const int at[4] = {pos[a].x, pos[a].y, pos[a].z, pos[a].w};
      int sg = -1, lo_pos = 0, hi_pos = -1;   // [lo_pos, hi_pos): positions of segment sg
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (!(m[a] >> q & 1u)) continue;
        const int p = at[q];
        if (p < lo_pos || p >= hi_pos) {
          sg = segment_of(s_start, ns, p);
          lo_pos = sg >= 0 ? s_start[sg] : 0;
          hi_pos = sg >= 0 ? (sg + 1 < ns ? s_start[sg + 1] : 0x7fffffff) : -1;
        }
        if (sg >= 0) f(sg, p, THINKV_HANDLE(cls[a], pi[a], 4 * quarter + q));
      }
    }
  }
}

__global__ __launch_bounds__(kPlanThreads) void tbe_count_plan_kernel(thinkv_view v, PlanArgs a) {
  const thinkv_config& c = v.cfg;
  const int b = blockIdx.x, tid = threadIdx.x;
  __shared__ int s_start[kMaxSegs];
  __shared__ int s_cnt[kMaxSegs];
  __shared__ uint8_t s_type[kMaxSegs];
  __shared__ uint8_t s_lvl[kMaxSegs];   // selections so far, capped at the number of levels
  const bool by_count = a.rule == THINKV_TBE_BY_COUNT;
  const int seq = a.seq_ids[b];
  if (seq < 0 || seq >= c.max_seqs) {
    if (tid == 0) {
      atomicOr(&v.dev_status[c.max_seqs * c.n_layers], THINKV_ST_BAD_SEQ);
      a.st_ncuts[b] = 0;
      a.st_total[b] = 0;
    }
    return;
  }
  int ns = a.n_segs[seq];
  ns = ns < 0 ? 0 : (ns > a.max_segs ? a.max_segs : ns);
  const int32_t* starts = a.seg_start + (int64_t)seq * a.max_segs;
  const uint8_t* types = a.seg_type + (int64_t)seq * a.max_segs;
  int32_t* sel = by_count ? a.seg_count + (int64_t)seq * a.max_segs : nullptr;
  for (int i = tid; i < ns; i += kPlanThreads) {
    s_start[i] = starts[i];
    s_type[i] = types[i];
    s_cnt[i] = 0;
    const int n = by_count ? sel[i] : 0;
    s_lvl[i] = (uint8_t)(n < 0 ? 0 : (n > 5 ? 5 : n));
  }
  __syncthreads();
  for_live_tokens(v, seq, a.layer, s_start, ns, [&](int sg, int, int) { atomicAdd(&s_cnt[sg], 1); });
  __syncthreads();
  int32_t* o_seg = a.st_seg + (int64_t)b * a.max_cuts;
  int32_t* o_keep = a.st_keep + (int64_t)b * a.max_cuts;
  int32_t* o_cnt = a.st_cnt + (int64_t)b * a.max_cuts;
  const int last = ns - 1;
  // Case 1: every closed segment that can still shrink, in ascending order, is independent of the
  // others: all threads, with a prefix sum for the place of each cut in the list
  __shared__ int s_wave[3][kPlanThreads / 64];
  __shared__ int s_c1[4];   // cuts, tokens listed, tokens dropped, a segment too large for one workgroup was met
  if (tid < 4) s_c1[tid] = 0;
  __syncthreads();
  if (a.transition_ended && a.transition_ended[b]) {
    for (int i0 = 0; i0 < last; i0 += kPlanThreads) {
      const int i = i0 + tid, lane = tid & 63, wave = tid >> 6;
      const int cnt = i < last ? s_cnt[i] : 0;
      // what the segment keeps if it is selected now (0: it cannot be selected, or nothing would go)
      int r = 0;
      if (i < last) {
        if (by_count) {
          const int n = s_lvl[i];
          if (n < 5) {
            r = cnt < kRetention[n] ? cnt : kRetention[n];
            if (r >= cnt) {           // removes nothing: not a cut, the count moves on
              s_lvl[i] = (uint8_t)(n + 1);
              sel[i] = n + 1;
              r = 0;
            }
          }
        } else {
          r = next_level(cnt);
        }
      }
      const bool big = r && cnt > kTbeMaxTokens;
      const int flag = r && !big;
      int inc = flag;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int o = __shfl_up(inc, d, 64);
        if (lane >= d) inc += o;
      }
      if (lane == 63) s_wave[0][wave] = inc;
      __syncthreads();
      int before = s_c1[0];
      for (int w = 0; w < wave; ++w) before += s_wave[0][w];
      const int at = before + inc - flag;
      const bool take = flag && at < a.max_cuts;
      if (take) {
        o_seg[at] = i;
        o_keep[at] = r;
        o_cnt[at] = cnt;
        s_cnt[i] = -r;          // negative: cut in this call, now holding r tokens
      }
      int n_take = take, listed = take ? cnt : 0, dropped = take ? cnt - r : 0;
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) {
        n_take += __shfl_xor(n_take, d, 64);
        listed += __shfl_xor(listed, d, 64);
        dropped += __shfl_xor(dropped, d, 64);
      }
      __syncthreads();   // s_wave[0] and s_c1[0] have been read
      if (lane == 0) {
        s_wave[0][wave] = n_take;
        s_wave[1][wave] = listed;
        s_wave[2][wave] = dropped;
      }
      if (big) s_c1[3] = 1;
      __syncthreads();
      if (tid == 0)
        for (int w = 0; w < kPlanThreads / 64; ++w) {
          s_c1[0] += s_wave[0][w];
          s_c1[1] += s_wave[1][w];
          s_c1[2] += s_wave[2][w];
        }
      __syncthreads();
    }
  }
  if (tid >= 64) return;
  int total = v.n_live[sl_index(c, seq, a.layer)] - s_c1[2];
  int n_cuts = s_c1[0], listed = s_c1[1];
  bool oversize = s_c1[3] != 0;
  // Case 2.  A segment that cannot be cut now cannot be cut later in this call either (one cut per
  // segment and call), so "the oldest segment of the least important type that can still shrink",
  // asked again after every cut, is one walk over the types in order of importance and over the
  // segments of each from the oldest on.  One wave, 64 segments at a time: whether the walk comes as far as a segment follows
  // from what the segments before it drop.
  const int lane = tid;
  for (int t = 0; t < 3; ++t)
    for (int i0 = 0; i0 < last && total > a.budget && n_cuts < a.max_cuts; i0 += 64) {
      const int i = i0 + lane, cnt = i < last ? s_cnt[i] : -1;
      const bool open = cnt >= 0 && s_type[i] == t;
      int r = 0, n = 0;
      if (open) {
        if (by_count) {
          // selections that remove nothing follow one another at once (each advances the count)
          n = s_lvl[i];
          while (n < 5 && r == 0) {
            const int keep = cnt < kRetention[n] ? cnt : kRetention[n];
            if (keep < cnt) r = keep; else ++n;
          }
        } else {
          r = next_level(cnt);
        }
      }
      const bool big = r && cnt > kTbeMaxTokens, can = r && !big;
      int upto = can ? cnt - r : 0;   // dropped by the segments up to this one, if the walk comes as far
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int o = __shfl_up(upto, d, 64);
        if (lane >= d) upto += o;
      }
      const unsigned long long cans = __ballot(can);
      const int before = __popcll(cans & ((1ull << lane) - 1));
      const bool reached = total - (upto - (can ? cnt - r : 0)) > a.budget && n_cuts + before < a.max_cuts;
      if (open && reached && by_count && n != s_lvl[i]) {
        s_lvl[i] = (uint8_t)n;
        sel[i] = n;
      }
      const bool take = can && reached;
      if (take) {
        const int at = n_cuts + before;
        o_seg[at] = i;
        o_keep[at] = r;
        o_cnt[at] = cnt;
        s_cnt[i] = -r;          // negative: cut in this call, now holding r tokens
      }
      oversize |= __ballot(big && reached) != 0;
      const unsigned long long taken = __ballot(take);   // the walk ends once, so these are the leading ones of `cans`
      int in_list = take ? cnt : 0, dropped = take ? cnt - r : 0;
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) {
        in_list += __shfl_xor(in_list, d, 64);
        dropped += __shfl_xor(dropped, d, 64);
      }
      n_cuts += __popcll(taken);
      listed += in_list;
      total -= dropped;
    }
  if (tid != 0) return;
  a.st_ncuts[b] = n_cuts;
  a.st_total[b] = listed;
  if (oversize) atomicOr(&v.dev_status[c.max_seqs * c.n_layers], THINKV_ST_BAD_SEGMENT);
}

// exclusive prefix sum over one value per lane of wave 0 times four (values [4 * lane, 4 * lane + 4) of a
// list of at most 256); returns the four exclusive sums through ex[] and the total
__device__ inline int wave_scan4(const int* val, int* ex) {
  const int lane = threadIdx.x & 63;
  int inc = val[0] + val[1] + val[2] + val[3];
  const int mine = inc;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int o = __shfl_up(inc, d, 64);
    if (lane >= d) inc += o;
  }
  const int total = __shfl(inc, 63, 64);
  int run = inc - mine;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    ex[q] = run;
    run += val[q];
  }
  return total;
}

struct Place {
  int seg, tok, cuts;   // first cut and first token of a sequence in the dense lists, and how many of its cuts are made
};

// Where the lists are too short for all cuts: the sequences up to b in order, by one wave; a sequence whose cuts do not all fit
// keeps the leading ones that do.  b = B: the ends of the lists.
__device__ inline Place place_in_order(const PlanArgs& a, int b) {
  const int lane = threadIdx.x & 63;
  Place at = {0, 0, 0};
  for (int i = 0; i <= b && i < a.B; ++i) {
    const int nc = a.st_ncuts[i], tot = a.st_total[i];
    int kept = nc, kept_tok = tot;
    if (at.seg + nc > a.cap_seg || (int64_t)at.tok + tot > a.cap_tok) {
      // leading cuts that still fit (the lists only grow, so the first that does not fit ends them)
      int val[4], ex[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) val[q] = 4 * lane + q < nc ? a.st_cnt[(int64_t)i * a.max_cuts + 4 * lane + q] : 0;
      wave_scan4(val, ex);
      int fits = 0, fits_tok = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int j = 4 * lane + q;
        if (j < nc && at.seg + j < a.cap_seg && (int64_t)at.tok + ex[q] + val[q] <= a.cap_tok) {
          ++fits;
          fits_tok += val[q];
        }
      }
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) {
        fits += __shfl_xor(fits, d, 64);
        fits_tok += __shfl_xor(fits_tok, d, 64);
      }
      kept = fits;
      kept_tok = fits_tok;
    }
    if (i == b) {
      at.cuts = kept;
      return at;
    }
    at.seg += kept;
    at.tok += kept_tok;
  }
  return at;
}

__global__ __launch_bounds__(kPlanThreads) void tbe_fill_kernel(thinkv_view v, PlanArgs a) {
  const int b = blockIdx.x, tid = threadIdx.x;
  __shared__ unsigned long long s_sum[4];         // cuts and tokens of all sequences, and of those before this one
  __shared__ Place s_place;
  if (tid < 4) s_sum[tid] = 0ull;
  __syncthreads();
  for (int i = tid; i < a.B; i += kPlanThreads) {
    const int nc = a.st_ncuts[i], tot = a.st_total[i];
    if (nc == 0) continue;
    atomicAdd(&s_sum[0], (unsigned long long)nc);
    atomicAdd(&s_sum[1], (unsigned long long)tot);
    if (i < b) {
      atomicAdd(&s_sum[2], (unsigned long long)nc);
      atomicAdd(&s_sum[3], (unsigned long long)tot);
    }
  }
  __syncthreads();
  if (tid < 64) {
    const bool fits = s_sum[0] <= (unsigned long long)a.cap_seg && s_sum[1] <= (unsigned long long)a.cap_tok;
    Place at = {(int)s_sum[2], (int)s_sum[3], b < a.B ? a.st_ncuts[b] : 0}, end = {(int)s_sum[0], (int)s_sum[1], 0};
    if (!fits) {
      at = place_in_order(a, b);
      if (b == 0) end = place_in_order(a, a.B);
    }
    if (tid == 0) {
      s_place = at;
      if (b == 0) {
        a.seg_offset[end.seg] = end.tok;
        a.counts[0] = end.seg;
        a.counts[1] = end.tok;
      }
    }
  }
  __syncthreads();
  const int n_cuts = s_place.cuts;
  if (n_cuts == 0) return;
  __shared__ int s_start[kMaxSegs];
  __shared__ int s_cut[kMaxSegs];                 // cut number of a segment, -1 = not cut
  __shared__ int s_fill[kTbeMaxTokens];           // tokens dealt to a cut so far (cuts per sequence <= 256, checked on the host)
  __shared__ int s_off[kTbeMaxTokens];            // first token of a cut's list
  const int seq = a.seq_ids[b];
  int ns = a.n_segs[seq];
  ns = ns < 0 ? 0 : (ns > a.max_segs ? a.max_segs : ns);
  const int32_t* starts = a.seg_start + (int64_t)seq * a.max_segs;
  for (int i = tid; i < ns; i += kPlanThreads) {
    s_start[i] = starts[i];
    s_cut[i] = -1;
  }
  const int seg_base = s_place.seg, tok_base = s_place.tok;
  if (tid < 64) {
    int val[4], ex[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) val[q] = 4 * tid + q < n_cuts ? a.st_cnt[(int64_t)b * a.max_cuts + 4 * tid + q] : 0;
    wave_scan4(val, ex);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = 4 * tid + q;
      if (i < n_cuts) {
        s_off[i] = tok_base + ex[q];
        s_fill[i] = 0;
        a.seg_offset[seg_base + i] = tok_base + ex[q];
        a.seg_keep[seg_base + i] = a.st_keep[(int64_t)b * a.max_cuts + i];
        a.st_cut_seq[seg_base + i] = seq;
      }
    }
  }
  __syncthreads();
  for (int i = tid; i < n_cuts; i += kPlanThreads) {
    const int sg = a.st_seg[(int64_t)b * a.max_cuts + i];
    s_cut[sg] = i;
    // the cut is made (it fitted the lists): this was a selection of the segment
    if (a.rule == THINKV_TBE_BY_COUNT) a.seg_count[(int64_t)seq * a.max_segs + sg] += 1;
  }
  __syncthreads();
  // deal the tokens: position into tok_seq for now, handle into tok_handle
  for_live_tokens(v, seq, a.layer, s_start, ns, [&](int sg, int pos, int h) {
    const int cu = s_cut[sg];
    if (cu < 0) return;
    const int at = s_off[cu] + atomicAdd(&s_fill[cu], 1);
    a.tok_seq[at] = pos;
    a.tok_handle[at] = h;
  });
}

// one wave per cut of the dense lists: ascending position inside the list.  A token's rank is the number of smaller keys (position,
// then place in the list), four keys of the list compared at a time
__global__ __launch_bounds__(256) void tbe_sort_kernel(PlanArgs a) {
  __shared__ __attribute__((aligned(16))) long long s_key[4][kTbeMaxTokens];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int cu = blockIdx.x * 4 + wave;
  if (cu >= a.counts[0]) return;   // the waves do not meet
  const int lo = a.seg_offset[cu], n = a.seg_offset[cu + 1] - lo;   // at most kTbeMaxTokens: larger segments are never cut
  const int seq = a.st_cut_seq[cu];
  long long key[kPT];
  int h[kPT], rank[kPT];
#pragma unroll
  for (int q = 0; q < kPT; ++q) {
    const int i = lane + 64 * q;
    rank[q] = 0;
    key[q] = 0x7FFFFFFFFFFFFFFFll;
    if (i < n) {
      key[q] = (long long)a.tok_seq[lo + i] << 8 | i;
      h[q] = a.tok_handle[lo + i];
    }
    s_key[wave][i] = key[q];
  }
  __builtin_amdgcn_wave_barrier();
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  auto walk = [&](auto rows) {   // points of so many 64
    for (int i = 0; i < n; i += 4) {
      const long long o[4] = {s_key[wave][i], s_key[wave][i + 1], s_key[wave][i + 2], s_key[wave][i + 3]};
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int q = 0; q < decltype(rows)::value; ++q) rank[q] += o[e] < key[q];
    }
  };
  if (n <= 64) walk(std::integral_constant<int, 1>{});
  else if (n <= 128) walk(std::integral_constant<int, 2>{});
  else walk(std::integral_constant<int, kPT>{});
#pragma unroll
  for (int q = 0; q < kPT; ++q)
    if (lane + 64 * q < n) {
      a.tok_handle[lo + rank[q]] = h[q];
      a.tok_seq[lo + rank[q]] = seq;
    }
}

int launch_tbe_plan(const thinkv_view& v, int layer, const int32_t* seq_ids, const int32_t* seg_start, const uint8_t* seg_type,
                    const int32_t* n_segs, const uint8_t* transition_ended, int32_t* seg_count, int rule, int B, int max_segs, int budget, int max_cuts,
                    int cap_seg, int cap_tok, int32_t* tok_seq, int32_t* tok_handle, int32_t* seg_offset, int32_t* seg_keep,
                    int32_t* counts, void* workspace, hipStream_t st) {
  PlanArgs a;
  a.seq_ids = seq_ids;
  a.seg_start = seg_start;
  a.seg_type = seg_type;
  a.n_segs = n_segs;
  a.transition_ended = transition_ended;
  a.seg_count = seg_count;
  a.rule = rule;
  a.tok_seq = tok_seq;
  a.tok_handle = tok_handle;
  a.seg_offset = seg_offset;
  a.seg_keep = seg_keep;
  a.counts = counts;
  int32_t* w = (int32_t*)(((uintptr_t)workspace + 255) & ~(uintptr_t)255);
  a.st_seg = w;
  a.st_keep = w + (size_t)B * max_cuts;
  a.st_cnt = w + 2 * (size_t)B * max_cuts;
  a.st_cut_seq = w + 3 * (size_t)B * max_cuts;
  a.st_ncuts = w + 4 * (size_t)B * max_cuts;
  a.st_total = a.st_ncuts + B;
  a.layer = layer;
  a.B = B;
  a.max_segs = max_segs;
  a.budget = budget;
  a.max_cuts = max_cuts;
  a.cap_seg = cap_seg;
  a.cap_tok = cap_tok;
  if (B > 0) hipLaunchKernelGGL(tbe_count_plan_kernel, dim3(B), dim3(kPlanThreads), 0, st, v, a);
  hipLaunchKernelGGL(tbe_fill_kernel, dim3(B > 0 ? B : 1), dim3(kPlanThreads), 0, st, v, a);
  const int64_t most = (int64_t)B * max_cuts < cap_seg ? (int64_t)B * max_cuts : cap_seg;
  if (most > 0) hipLaunchKernelGGL(tbe_sort_kernel, dim3((unsigned)((most + 3) / 4)), dim3(256), 0, st, a);
  return hipGetLastError() == hipSuccess ? THINKV_OK : THINKV_E_HIP;
}

}  // namespace thinkv

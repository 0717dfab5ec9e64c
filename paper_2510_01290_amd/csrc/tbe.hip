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
// Three kernels.  A centroid is the mean of points, so every product Lloyd's algorithm asks for is a
// mean of products between points: x.c_j = mean over the members i of x.x_i, |c_j|^2 = mean over the members of
// x_i.c_j.  So the channels are walked once, for all products between the points of the segment (the Gram matrix, at most
// 256 x 256, lower triangle), and an iteration is at most n^2 additions from LDS, of the clusters that changed only.
// A centroid is represented by the set of points it is the mean of: at the start one
// point, later the members, and for a cluster that has lost its last member the members it had before.
// gram: the matrix, up to four workgroups a segment, each over some of the heads.  The keys go from the pages to the matrix
// cores without a stop in memory; the binary32 rows are written on the way.
// kmeans: a workgroup per segment adds the parts of the matrix and iterates; up to 192 tokens, two workgroups a compute unit.
// whole: segments of more tokens (a matrix of up to 132 KB), a workgroup per compute unit that does both; and, alone, all segments of up to 512
// channels.
// 314 segments of ~110 tokens, 1,024 channels, us: keys to memory and a workgroup of a whole compute unit per segment (its
// 139 KB of LDS made that 1.2 rounds of workgroups) 37 + 177; now 67 + 56 (and 5 for whole, which finds nothing).  gram is bound by vector
// instructions (four a number to unpack and split it) and by 141 MB of rows; kmeans by its longest segments' iterations (choose_survivors), the parts
// (5 to 10), and the 54 MB of centroids (9 to 35, the rows they are made of are 141 MB).
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

constexpr int kGramThreads = 512;         // eight waves, two workgroups a compute unit
constexpr int kGramWaves = kGramThreads / 64;
// Workgroups that share a segment's channels at most.  8 heads of 128, us by two / three / four: 1 segment of 110 tokens 45.6 / 42.3 / 38.6, an eviction event of
// 314 segments 204 / 202 / 203, 2,000 of 64 to 192 795 / 825 / 877 (by one, 314: the units that get two segments end last, the kernel 110 instead of 67).
constexpr int kSlices = 4;
constexpr int kMacro = 32;                // points on a side of a wave's piece of the Gram matrix (2 x 2 MFMA tiles)
constexpr int kPiecesPerWave = 3;         // 24 pieces of the lower triangle, all of 192 points, by eight waves; 36, all of 256, by sixteen
constexpr int kFewPoints = 192;           // points of the largest segment that takes half a compute unit
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
constexpr int kPadH = 2 * kTile + 8;   // binary16 numbers per tile row: high parts, low parts, padding (an odd multiple of 16 bytes)

__host__ __device__ __forceinline__ int tri(int i) { return i * (i + 1) / 2; }   // where row i of the lower triangle begins

// The parts of a segment's matrix lie where its centroids will, which are written last: 64 * dim numbers.
// narrow: that is less than the largest matrix.  Then no segment is shared, and tbe_whole_kernel is the only launch: a workgroup walks few channels,
// and three launches and the parts' way through memory cost more (64 to 192 tokens, us, with 131,584 bytes more a segment for the parts / now: 2 heads of
// 64, 314 segments 119 / 90, 2,000 410 / 384; 5 of 64 138 / 113, 566 / 483; 8 of 64 202 / 169, 725 / 549).
// wide: the products of segments of more than kFewPoints are shared as well.  A gram workgroup, whose waves hold the products of 192 points, walks
// the channels twice for them; but from 4,096 channels on, and with no more segments than have all their gram workgroups under
// way at once (512 of them), tbe_whole_kernel's one walk by one workgroup is the longer one.  (200 to 256 tokens, 32 heads of 128, us, shared / not: 1
// segment 232 / 345, 8 288 / 387, 64 455 / 501, 300 1,304 / 1,188; 16 heads, 8 segments, by an earlier form of the shared way, 195 / 186, 64 333 / 229.)
static bool is_narrow(int dim) { return kTbeMaxKeep * dim < tri(kTbeMaxTokens); }
static bool is_wide(int dim, int n_seg) { return dim >= 4096 && n_seg <= 512 / kSlices; }

__device__ __forceinline__ float* parts_of(const TbeArgs& a, int seg) { return a.cent + (int64_t)seg * kTbeMaxKeep * a.dim; }
// workgroups that share the products of a segment of n tokens: as many parts as there is room for (one at least)
__device__ __forceinline__ int gram_slices(const TbeArgs& a, int n, int heads) {
  const int s = min(kTbeMaxKeep * a.dim / tri(n), kSlices);
  return min(s, heads);
}

size_t tbe_ws_bytes(const thinkv_config& c, int n_tok, int n_seg) {
  const size_t dim = (size_t)c.n_kv_heads * c.head_dim, toks = n_tok > 0 ? n_tok : 1, segs = n_seg > 0 ? n_seg : 1;
  return (toks * dim + segs * kTbeMaxKeep * dim) * sizeof(float) + toks * sizeof(int32_t) + 256;
}

// ---- a token's keys.  A unit is a chunk of a token's block (a kv-head, eight channels of every group); the four threads of
// a quad hold the four chunks of one token and head, and each holds the scales of one group for all four.
struct TokenAt {          // where a token's keys lie
  const uint8_t* page;    // its page's block of head 0
  uint32_t slot, bits;    // (width 0: the token does not exist)
};

__device__ inline TokenAt token_at(const thinkv_view& v, const TbeArgs& a, int i) {
  const thinkv_config& c = v.cfg;
  const int s = a.tok_seq[i];
  const int32_t h = a.tok_handle[i];
  const uint32_t uh = (uint32_t)h;
  const int cls = uh >> 28, pi = (uh >> 4) & 0xFFFFFF;
  TokenAt t = {v.arena[0], uh & 15, 0};
  if (s < 0 || s >= c.max_seqs) {
    atomicOr(&v.dev_status[c.max_seqs * c.n_layers], THINKV_ST_BAD_SEQ);
  } else if (h < 0 || cls > 2 || pi >= v.n_pages[npages_index(c, s, a.layer, cls)]) {
    atomicOr(&v.dev_status[sl_index(c, s, a.layer)], THINKV_ST_BAD_SLOT);
  } else {
    t.bits = cls == 0 ? c.bits_of_class[0] : cls == 1 ? c.bits_of_class[1] : c.bits_of_class[2];
    t.page = (cls == 0 ? v.arena[0] : cls == 1 ? v.arena[1] : v.arena[2]) +
             (int64_t)v.block_table[table_base(c, s, a.layer, cls) + pi] * c.n_kv_heads * block_geom(t.bits, c.head_dim, c.format).block_bytes;
  }
  return t;
}

template <int D>
struct RawKeys {
  uint32_t code[D / 16];   // the codes of the chunk: D / 32 groups of eight
  uint32_t meta;           // group (lane & 3): scale and zero-point; paper's formats: the scales of its two halves
};

// The chunk j of a token and head.  A token that does not exist has codes, scales and zero-points of 0: it clusters as the origin
template <int D, bool FP>
__device__ __forceinline__ void load_keys(const TokenAt& t, int hd, int j, RawKeys<D>& r) {
#pragma unroll
  for (int w = 0; w < D / 16; ++w) r.code[w] = 0u;
  r.meta = 0u;
  const BlockGeom g = block_geom(t.bits, D, FP ? THINKV_FMT_FP : THINKV_FMT_INT);
  const uint8_t* blk = t.page + (int64_t)hd * g.block_bytes;
  const uint32_t* chunk = (const uint32_t*)(blk + (16 * j + t.slot) * g.chunk_bytes);
  auto take = [&](auto words) {
#pragma unroll
    for (int w = 0; w < decltype(words)::value; ++w) r.code[w] = chunk[w];
  };
  if (t.bits == 2) take(std::integral_constant<int, D / 64>{});
  if (t.bits == 4) take(std::integral_constant<int, D / 32>{});
  if (t.bits == 8) take(std::integral_constant<int, D / 16>{});
  if (j < D / kGroup && t.bits != 0 && !(FP && t.bits == 8)) {
    if (FP) {
      const uint8_t* meta = blk + g.k_meta + 2 * j * kPage + t.slot;
      r.meta = meta[0] | (uint32_t)meta[kPage] << 8;
    } else {
      const uint16_t* meta = (const uint16_t*)(blk + g.k_meta) + meta_index(t.slot, j);
      r.meta = meta[0] | (uint32_t)meta[4] << 16;
    }
  }
}

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

// The eight channels 32 GRP + 8 j .. + 7, for every width in the same instructions: two words, each with four codes at bits 0,
// 16, b and 16 + b.  m: the scales of group GRP.  A masked code is a binary16 subnormal, code * 2^-24, which the mixed-precision
// multiply-add reads as it is; the scale takes the power of two.  In the paper's formats the magnitude bits go under the
// exponent of a binary16 number and the sign bit to bit 15.
// A token that does not exist (width 0) has codes, scales and zero-points of 0; it is unpacked as one of the narrowest
// type, since a shift by a width less one has to be defined.
template <int D, bool FP, int GRP>
__device__ __forceinline__ void unpack_keys(const thinkv_config& c, const RawKeys<D>& r, uint32_t m, int width, int j, float (&x)[8]) {
  const int bits = width ? width : 2;
  const uint32_t two = r.code[GRP / 2] >> (8 * (GRP & 1));
  const uint32_t word[2] = {bits == 8 ? r.code[2 * GRP] : bits == 4 ? r.code[GRP] : two,
                            bits == 8 ? r.code[2 * GRP + 1] : bits == 4 ? r.code[GRP] >> 8 : two >> 4};
  float sc, zp = 0.f;
  if (FP) {
    sc = bits == 8 ? c.fp8_scale[0] : e4m3_value(m >> (8 * (j >> 1)) & 0xFFu);
  } else {
    sc = (float)__builtin_bit_cast(_Float16, (uint16_t)m) * 16777216.0f;
    zp = (float)__builtin_bit_cast(_Float16, (uint16_t)(m >> 16));
  }
  const uint32_t mask = ((1u << bits) - 1u) * 0x10001u;
#pragma unroll
  for (int e = 0; e < 8; e += 2) {
    const uint32_t two_codes = word[e >> 2] >> (e & 2 ? bits : 0) & mask;
    if (FP) {
      const int up = bits == 8 ? 7 : bits == 4 ? 9 : 10;   // a ternary magnitude is 2^-14
      const uint32_t signs = 0x10001u << (bits - 1);
      const uint32_t sign = bits == 2 ? two_codes & (two_codes << 1) & signs : two_codes & signs;   // a ternary zero has no sign
      const f16x2 h = __builtin_bit_cast(f16x2, sign << (16 - bits) | (two_codes & ~signs) << up);
      const float lift = bits == 8 ? 256.0f : 16384.0f;
      x[e] = (float)h[0] * lift * sc;
      x[e + 1] = (float)h[1] * lift * sc;
    } else {
      const f16x2 h = __builtin_bit_cast(f16x2, two_codes);
      x[e] = fmaf((float)h[0], sc, zp);
      x[e + 1] = fmaf((float)h[1], sc, zp);
    }
  }
}

// the scales of group GRP from the lane of the quad that holds them
template <int GRP>
__device__ __forceinline__ uint32_t quad_meta(uint32_t meta) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)meta, 0x55 * GRP, 0xF, 0xF, true);
}

// f(group) for the groups of a head, the group a compile-time constant
template <int D, class F>
__device__ __forceinline__ void for_groups(F f) {
  f(std::integral_constant<int, 0>{});
  f(std::integral_constant<int, 1>{});
  if constexpr (D == 128) {
    f(std::integral_constant<int, 2>{});
    f(std::integral_constant<int, 3>{});
  }
}

__device__ __forceinline__ void store_row(float* dst, const float (&x)[8]) {
  *(float4*)dst = make_float4(x[0], x[1], x[2], x[3]);
  *(float4*)(dst + 4) = make_float4(x[4], x[5], x[6], x[7]);
}

// the binary32 rows of the tokens [from, to)
template <int D, bool FP, int THREADS>
__device__ __forceinline__ void write_rows(const thinkv_view& v, const TbeArgs& a, int from, int to, TokenAt* at) {
  const int per = 4 * v.cfg.n_kv_heads;
  for (; from < to; from += kTbeMaxTokens) {
    const int count = to - from < kTbeMaxTokens ? to - from : kTbeMaxTokens;
    __syncthreads();   // the tokens before have been used
    if ((int)threadIdx.x < count) at[threadIdx.x] = token_at(v, a, from + threadIdx.x);
    __syncthreads();
    for (int idx = threadIdx.x; idx < count * per; idx += THREADS) {
      const int i = idx / per, it = idx - i * per, hd = it >> 2, j = it & 3;
      const int bits = at[i].bits;
      RawKeys<D> r;
      load_keys<D, FP>(at[i], hd, j, r);
      float* row = a.x + (int64_t)(from + i) * a.dim + hd * D + 8 * j;
      for_groups<D>([&](auto grp) {
        constexpr int G = decltype(grp)::value;
        float x[8];
        unpack_keys<D, FP, G>(v.cfg, r, quad_meta<G>(r.meta), bits, j, x);
        store_row(row + 32 * G, x);
      });
    }
  }
}

// ... and of share w of W of the tokens before the first segment and behind the last
template <int D, bool FP, int THREADS>
__device__ __forceinline__ void write_outside(const thinkv_view& v, const TbeArgs& a, int w, int W, TokenAt* at) {
  const int lo = a.seg_offset[0], hi = a.seg_offset[a.n_seg];
  const int before = lo < 0 ? 0 : (lo < a.n_tok ? lo : a.n_tok), behind = hi < 0 ? 0 : (hi < a.n_tok ? hi : a.n_tok);
  const int all = before + a.n_tok - behind, part = (all + W - 1) / W;
  const int from = w * part, to = from + part < all ? from + part : all, skip = behind - before;
  write_rows<D, FP, THREADS>(v, a, from, to < before ? to : before, at);
  write_rows<D, FP, THREADS>(v, a, (from > before ? from : before) + skip, to + skip, at);
}

// ---- gram
template <int POINTS, int TILES>
struct GramScratch {
  _Float16 xs[TILES][POINTS][kPadH];   // tiles: 64 channels of every point, each as high + low binary16 part
  TokenAt at[kTbeMaxTokens];
};
static_assert(sizeof(GramScratch<kTbeMaxTokens, 1>) <= 81920, "two workgroups share the LDS of a compute unit");

// eight channels into a tile row: x = hi + lo with hi = binary16(x), lo = binary16(x - hi), 22 significant bits
__device__ __forceinline__ void store_split(_Float16* row, const float (&x)[8]) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  union { f16x8 all; f16x2 two[4]; } hi, lo;
#pragma unroll
  for (int e = 0; e < 8; e += 2) {
    const f16x2 h = __builtin_convertvector((f32x2){x[e], x[e + 1]}, f16x2);
    hi.two[e / 2] = h;
    lo.two[e / 2] = __builtin_convertvector((f32x2){fmaf((float)h[0], -1.f, x[e]), fmaf((float)h[1], -1.f, x[e + 1])}, f16x2);
  }
  *(f16x8*)row = hi.all;
  *(f16x8*)(row + kTile) = lo.all;
}

// the places of a segment's tokens; behind the last one tokens that do not exist
__device__ __forceinline__ void find_tokens(const thinkv_view& v, const TbeArgs& a, int lo, int n, TokenAt* at) {
  if (threadIdx.x < kTbeMaxTokens) {
    TokenAt t = {v.arena[0], 0, 0};
    if ((int)threadIdx.x < n) t = token_at(v, a, lo + threadIdx.x);
    at[threadIdx.x] = t;
  }
  __syncthreads();
}

// The products of all pairs of the n points over the heads [h0, h1), in the pieces [first, first + 3 W) of the lower triangle: out(first index,
// second, product), once done() has been called by all.  The channels go through LDS 64 at a time (the next head's codes are under way during a head's last products); wave
// w of W owns the pieces first + w, + W, + 2 W, 32 x 32 points each: 2 x 2 tiles share their operands, which halves the LDS reads a
// product costs.  With two tiles in LDS the next one is unpacked beside the products of this one (a segment of 256 tokens, 2,048 channels, that has
// a compute unit to itself: 218 us with one, now 182).
// A product is hi.hi + hi.lo + lo.hi (exact products, binary32 sums; what is dropped is of the order of 2^-22 of |x||y|).
template <int D, bool FP, int W, int POINTS, int TILES, class Done, class Out>
__device__ __forceinline__ void gram_matrix(const thinkv_view& v, int n, int h0, int h1, int first, GramScratch<POINTS, TILES>& sm, float* __restrict__ x, int dim, Done done, Out out) {
  constexpr int kPasses = (POINTS + 16 * W - 1) / (16 * W);   // a wave takes sixteen points at a time
  const thinkv_config& c = v.cfg;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, g = lane >> 4;
  const int mb = (n + kMacro - 1) / kMacro, end = mb * (mb + 1) / 2;
  int pi[kPiecesPerWave], pj[kPiecesPerWave];              // block row and column of the wave's pieces
  f32x4 acc[kPiecesPerWave][2][2];
#pragma unroll
  for (int t = 0; t < kPiecesPerWave; ++t) {
    int rest = first + wave + t * W, i = 0;
    while (rest > i) rest -= ++i;
    pi[t] = i;
    pj[t] = rest;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int w = 0; w < 2; ++w) acc[t][u][w] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  RawKeys<D> raw[kPasses];
  // the places come from LDS every time: held in registers they would be in the way of the products
  auto fetch = [&](int hd) {
    if (hd >= h1) return;
#pragma unroll
    for (int q = 0; q < kPasses; ++q)
      if (16 * (wave + W * q) < n) load_keys<D, FP>(sm.at[16 * (wave + W * q) + r], hd, g, raw[q]);
  };
  auto store = [&](int hd, auto half, int b) {   // of the last half: and the next head's codes are asked for
    constexpr int G0 = 2 * decltype(half)::value;
    // a wave takes sixteen tokens, lane (r, g) the chunk g of token r: sixteen lanes write to sixteen rows, whose
    // starts lie four banks apart
#pragma unroll
    for (int q = 0; q < kPasses; ++q) {
      const int t = 16 * (wave + W * q) + r;
      if (16 * (wave + W * q) < n) {   // rows that pad the sixteen are zeros
        const int bits = sm.at[t].bits;
        float val[8];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const uint32_t m = (uint32_t)__builtin_amdgcn_ds_bpermute(64 * (G0 + u) + 4 * r, (int)raw[q].meta);
          if (u == 0) unpack_keys<D, FP, G0>(c, raw[q], m, bits, g, val);
          else unpack_keys<D, FP, G0 + 1>(c, raw[q], m, bits, g, val);
          store_split(&sm.xs[b][t][32 * u + 8 * g], val);
          if (first == 0 && t < n) store_row(&x[(int64_t)t * dim + hd * D + 32 * (G0 + u) + 8 * g], val);
        }
      }
    }
    if (G0 == D / kGroup - 2) fetch(hd + 1);
  };
  auto products = [&](int b) {
#pragma unroll
    for (int t = 0; t < kPiecesPerWave; ++t)
      if (first + wave + t * W < end) {
        const bool diag = pi[t] == pj[t];
#pragma unroll
        for (int ks = 0; ks < kTile / 32; ++ks) {
          // lane (r, g) holds channels 32 ks + 8 g .. + 7 of its row, on both sides
          f16x8 ah[2], al[2], bh[2], bl[2];
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const _Float16* ra = sm.xs[b][kMacro * pi[t] + 16 * u + r];
            ah[u] = *(const f16x8*)&ra[32 * ks + 8 * g];
            al[u] = *(const f16x8*)&ra[kTile + 32 * ks + 8 * g];
          }
          if (diag) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
              bh[u] = ah[u];
              bl[u] = al[u];
            }
          } else {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
              const _Float16* rb = sm.xs[b][kMacro * pj[t] + 16 * u + r];
              bh[u] = *(const f16x8*)&rb[32 * ks + 8 * g];
              bl[u] = *(const f16x8*)&rb[kTile + 32 * ks + 8 * g];
            }
          }
          // the four tiles in turn: a product waits for the one before it into the same tile
#pragma unroll
          for (int part = 0; part < 3; ++part)
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
              for (int w = 0; w < 2; ++w)
                acc[t][u][w] = __builtin_amdgcn_mfma_f32_16x16x32_f16(part == 2 ? al[u] : ah[u], part == 1 ? bl[w] : bh[w], acc[t][u][w], 0, 0, 0);
        }
      }
  };
  fetch(h0);
  // rows that pad the last piece: zero
  const int full = (n + 15) & ~15;
  if (full & 16)
    for (int b = 0; b < TILES; ++b)
      for (int i = tid; i < 16 * (kPadH / 8); i += 64 * W)
        *(f16x8*)&sm.xs[b][full + i / (kPadH / 8)][8 * (i % (kPadH / 8))] = f16x8{0, 0, 0, 0, 0, 0, 0, 0};
  constexpr std::integral_constant<int, 0> low{};   // halves of a head
  constexpr std::integral_constant<int, D / 64 - 1> high{};
  if constexpr (TILES == 1) {
    auto tile = [&](int hd, auto half) {
      __syncthreads();   // the previous tile has been used
      store(hd, half, 0);
      __syncthreads();
      products(0);
    };
    for (int hd = h0; hd < h1; ++hd) {
      tile(hd, low);
      if constexpr (D == 128) tile(hd, high);
    }
  } else {
    store(h0, low, 0);
    int b = 0;
    for (int hd = h0; hd < h1; ++hd) {
      if constexpr (D == 128) {
        __syncthreads();   // tile b is there, the other one has been used
        store(hd, high, b ^ 1);
        products(b);
        b ^= 1;
      }
      __syncthreads();
      if (hd + 1 < h1) store(hd + 1, low, b ^ 1);
      products(b);
      b ^= 1;
    }
  }
  done();
#pragma unroll
  for (int t = 0; t < kPiecesPerWave; ++t)
    if (first + wave + t * W < end) {
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int w = 0; w < 2; ++w)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int p = kMacro * pi[t] + 16 * u + 4 * g + i, q = kMacro * pj[t] + 16 * w + r;
            if (p < n && q <= p) out(p, q, acc[t][u][w][i]);
          }
    }
}

// the segments that are clustered
__device__ __forceinline__ bool seg_ok(const TbeArgs& a, int lo, int hi, int want) {
  return hi - lo <= kTbeMaxTokens && want <= kTbeMaxKeep && want >= 1 && lo >= 0 && hi <= a.n_tok;
}

template <int D, bool FP, bool WIDE>
__global__ __launch_bounds__(kGramThreads, 4) void tbe_gram_kernel(thinkv_view v, TbeArgs a) {
  __shared__ __attribute__((aligned(16))) GramScratch<WIDE ? kTbeMaxTokens : kFewPoints, 1> sm;
  const int outside = (int)blockIdx.x - a.n_seg * kSlices;
  if (outside >= 0) {   // the last workgroups
    write_outside<D, FP, kGramThreads>(v, a, outside, (int)gridDim.x - a.n_seg * kSlices, sm.at);
    return;
  }
  const int seg = blockIdx.x / kSlices, slice = blockIdx.x % kSlices;
  const int lo = a.seg_offset[seg], hi = a.seg_offset[seg + 1], n = hi - lo, want = a.seg_keep[seg], H = v.cfg.n_kv_heads;
  if (n <= want || !seg_ok(a, lo, hi, want)) {   // not clustered: only the rows, a share for each of the segment's workgroups
    const int first = lo > 0 ? lo : 0, end = hi < a.n_tok ? hi : a.n_tok, part = (end - first + kSlices - 1) / kSlices;
    const int from = first + slice * part;
    write_rows<D, FP, kGramThreads>(v, a, from, from + part < end ? from + part : end, sm.at);
    return;
  }
  if (!WIDE && n > kFewPoints) return;   // tbe_whole_kernel's
  const int slices = gram_slices(a, n, H);
  if (slice >= slices) return;
  find_tokens(v, a, lo, n, sm.at);
  float* out = parts_of(a, seg) + (int64_t)slice * tri(n);
  auto walk = [&](int first) {
    gram_matrix<D, FP, kGramWaves>(v, n, H * slice / slices, H * (slice + 1) / slices, first, sm, a.x + (int64_t)lo * a.dim, a.dim, [] {},
                                   [&](int p, int q, float d) { out[tri(p) + q] = d; });
  };
  walk(0);
  if (WIDE && n > kFewPoints) walk(kPiecesPerWave * kGramWaves);
}

// ---- kmeans
// W waves; LDS holds the matrix of POINTS points.  Up to kFewPoints: twelve waves, two workgroups a compute unit.  More: sixteen waves, a
// compute unit to themselves.  (With the products of the points 192..255 in memory instead, 314 segments, us, before the keys went from the pages to the
// matrix cores / with those in memory / now: 8 heads of 128, 200 to 256 tokens 473 / 534 / 305, 256 tokens 501 / 734 / 323; 8 of 64 337 / 497 / 189; 2 of 128
// 251 / 384 / 159; 2 of 64 279 / 297 / 156; one segment of 256, 8 of 128, 165 / 268 / 136.)
constexpr int kKmWaves = 12, kWholeWaves = 16;
constexpr int kPT = kTbeMaxTokens / 64;                   // tokens per lane of a wave that sorts a list
constexpr int kWords = kTbeMaxTokens / 32;

// An entry of the list of members: the point, where its row of the triangle begins, that it is one, its cluster, and that the four
// entries of a step it stands in are the cluster's last
constexpr uint32_t kIsMember = 1u << 31, kLastStep = 1u << 23;
__device__ __forceinline__ uint32_t member(int p, int j, bool last) { return (uint32_t)p | (uint32_t)tri(p) << 8 | kIsMember | (uint32_t)j << 24 | (last ? kLastStep : 0u); }
constexpr uint32_t kUnmoved = ~0u;

template <int W, int POINTS>
struct KmScratch {
  float gram[POINTS * (POINTS + 1) / 2];                       // products of all pairs of points, lower triangle
  uint32_t basis[kTbeMaxKeep][kWords];                         // the points a cluster's centroid is the mean of
  union {
    uint32_t next[kTbeMaxKeep][kWords];                        // members under the assignment just made
    struct {
      unsigned long long best[kTbeMaxKeep];                    // survivors: nearest member, and the lowest index, of every cluster
      int low[kTbeMaxKeep];
    };
  };
  float own[kTbeMaxTokens];                                    // product of a point with the centroid it belongs to
  float cc[4][kTbeMaxKeep / 4];                                // squared norms of the centroids: cluster j at [j % 4][j / 4]
  uint32_t count[kTbeMaxKeep];                                 // members
  uint32_t start[kTbeMaxKeep];                                 // where those of a cluster whose centroid has just moved begin in the list
  uint32_t list[kTbeMaxTokens + 3 * kTbeMaxKeep];              // the points of these clusters, cluster by cluster, in index order, each cluster's filled up to fours
  int steps;                                                   // fours of the list
  int vote[2];                                                 // a point changed its cluster, in iterations of either parity
};
static_assert(sizeof(KmScratch<kKmWaves, kFewPoints>) <= 81920, "two workgroups share the LDS of a compute unit");

__device__ __forceinline__ float add_quarters(float x) {   // the sum over the lanes l, l ^ 16, l ^ 32, l ^ 48, the same in the four
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const uint32_t w = __builtin_bit_cast(uint32_t, __builtin_bit_cast(float, (uint32_t)a[0]) + __builtin_bit_cast(float, (uint32_t)a[1]));
  auto b = __builtin_amdgcn_permlane32_swap(w, w, false, false);
  return __builtin_bit_cast(float, (uint32_t)b[0]) + __builtin_bit_cast(float, (uint32_t)b[1]);
}

// Lloyd's algorithm, the survivors and the centroids of a segment whose matrix is in LDS.  A wave has sixteen points; lane (r, quarter) shares
// point r with three others: a quarter adds every fourth member of a cluster and keeps the products with every fourth cluster.  So
// all waves have the same work whatever the sizes of the clusters are, and the nearest cluster is found inside a wave, without a barrier.  What bounds
// it: instructions (some fourteen for four members of a wave's points) and, where few clusters move, barriers and LDS latency: so a point's rank among the
// members and the clusters' places in the list ask LDS once.  (A point a lane and clusters dealt to groups of waves, the largest cluster being what everybody
// waited for / this way with a step of twenty instructions, and a rank of up to eight dependent loads / now, us, K of 64, 32 and 16 in turn: 314 segments of 64 to 192
// tokens, 8 kv-heads of 128 140 / 131 / 128, 2 of 64 96 / 85 / 81; 64 of 193 to 256, 1 of 64, 87.5 / 92.9 / 84.3; one of 256 tokens and 64 clusters, where four members a
// cluster cost a step and a sum over the quarters, 1 of 64, 45.0 / 46.8 / 44.0, 2 of 128 56.6 / 58.0 / 55.1; the one size that still loses, one of 192, 8 of 128, 61.6 / 63.7 / 62.6.
// The sums as a matrix product with the 0/1 matrix of the members, in binary32 on the matrix cores: 5 a tile of sixteen clusters, however few of them moved; 314 segments of
// 64 to 192 tokens 177 us where the second way took 145.)
template <int W, int POINTS>
__device__ __forceinline__ void choose_survivors(const TbeArgs& a, int seg, int lo, int n, int k, KmScratch<W, POINTS>& sm) {
  constexpr int kThreads = 64 * W, kPer = kTbeMaxKeep / 4, kAhead = 4, kRows = 8;
  static_assert(POINTS <= 16 * W && 8 * kTbeMaxKeep <= kThreads, "a wave for sixteen points, eight lanes for a cluster");
  typedef float f32xk __attribute__((ext_vector_type(kPer)));   // a number for each of a lane's clusters, 4 i + quarter
  // (opaque: what follows from it would be worked out before a caller's loop over segments and held in registers that the products need)
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), dim = a.dim;
  const int quarter = lane >> 4, p = 16 * wave + (lane & 15);
  const bool here = p < n, first = here && quarter == 0;
  const int pc = here ? p : n - 1, tp = tri(pc);
  // with point m, whose row begins at tm: the pair's place is in the row of the larger, the larger of the two sums (alike only where both are the place)
  auto product = [&](int m, int tm) { return sm.gram[max(tp + m, tm + pc)]; };
  // initial centroids: evenly spaced points, distinct, since k < n
  for (int i = tid; i < kTbeMaxKeep * kWords; i += kThreads) (&sm.basis[0][0])[i] = (&sm.next[0][0])[i] = 0u;
  if (tid < 2) sm.vote[tid] = 0;
  __syncthreads();
  f32xk dot;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int j = 4 * i + quarter, m = j < k ? j * n / k : 0;
    dot[i] = 4 * i < k ? product(m, tri(m)) : 0.f;
  }
  if (tid < kTbeMaxKeep) {
    const int q = tid < k ? tid * n / k : 0;
    if (tid < k) sm.basis[tid][q >> 5] = 1u << (q & 31);
    sm.cc[tid & 3][tid >> 2] = sm.gram[tri(q) + q];
    if (tid < k) sm.own[q] = sm.gram[tri(q) + q];
    sm.count[tid] = tid < k ? 1u : 0u;
  }
  int mine = -1;                                     // this point's cluster at the last assignment
  __syncthreads();
  // Products of every point with the centroids that moved, in dot[]; own of their members, and the squared norms of the centroids
  auto products = [&]() {
    const int steps = __builtin_amdgcn_readfirstlane(sm.steps);
    const uint32_t inv = __builtin_bit_cast(uint32_t, 1.0f / (float)sm.count[lane]);
    float sum = 0.f, with_own = 0.f;
    if (16 * wave < n)
      for (int s0 = 0; s0 < steps; s0 += kAhead) {   // the loads of four steps do not wait for each other
        uint32_t e[kAhead];
        float g[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) e[u] = sm.list[4 * min(s0 + u, steps - 1) + quarter];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) g[u] = product(e[u] & 255, e[u] >> 8 & 0x7FFF);
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
          if (s0 + u >= steps) break;
          sum += __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, g[u]) & (uint32_t)((int)e[u] >> 31));   // (no member: zero, whatever is there)
          const uint32_t all = __builtin_amdgcn_readfirstlane(e[u]);   // (the first of a step is a member)
          if (all & kLastStep) {
            const int j = all >> 24 & 63;
            const float d = add_quarters(sum) * __builtin_bit_cast(float, __builtin_amdgcn_readlane(inv, j));
            dot[j >> 2] = quarter == (j & 3) ? d : dot[j >> 2];
            with_own = mine == j ? d : with_own;
            sum = 0.f;
          }
        }
      }
    if (first && sm.start[mine] != kUnmoved) sm.own[p] = with_own;
    __syncthreads();
    // |c|^2 = mean over the members of their products with the centroid: eight lanes per cluster, a fixed tree
    const int j = tid >> 3;
    if (j < k && sm.start[j] != kUnmoved) {
      const uint32_t q0 = sm.start[j], cnt = sm.count[j];
      float part = 0.f;
      for (uint32_t q = tid & 7; q < cnt; q += 8) part += sm.own[sm.list[q0 + q] & 255];
#pragma unroll
      for (int d = 4; d >= 1; d >>= 1) part += __shfl_xor(part, d, 8);
      if ((tid & 7) == 0) sm.cc[j & 3][j >> 2] = part * (1.0f / (float)cnt);
    }
    // (the members of the assignment before have been used)
    for (int i = tid; i < kTbeMaxKeep * kWords; i += kThreads) (&sm.next[0][0])[i] = 0u;
    __syncthreads();
  };
  bool converged = false;
  for (int it = 0; it < a.max_iters; ++it) {
    // centroids: the initial ones, later the means under the previous assignment
    if (it > 0) products();
    // nearest cluster of every point: |c|^2 - 2 x.c decides (|x|^2 is common to a point's candidates); ties go to the
    // lowest cluster
    float bd = INFINITY;
    int bj = kTbeMaxKeep;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      if (4 * i >= k) break;
      const int j = 4 * i + quarter;
      const float d = fmaf(-2.f, dot[i], sm.cc[quarter][i]);
      if (j < k && d < bd) {
        bd = d;
        bj = j;
      }
    }
    {
      auto nearer = [&](auto d, auto c) {   // of the two that a swap brings together
        const float d0 = __builtin_bit_cast(float, (uint32_t)d[0]), d1 = __builtin_bit_cast(float, (uint32_t)d[1]);
        const int c0 = (int)c[0], c1 = (int)c[1];
        const bool second = d1 < d0 || (d1 == d0 && c1 < c0);
        bd = second ? d1 : d0;
        bj = second ? c1 : c0;
      };
      const uint32_t d16 = __builtin_bit_cast(uint32_t, bd), c16 = (uint32_t)bj;
      nearer(__builtin_amdgcn_permlane16_swap(d16, d16, false, false), __builtin_amdgcn_permlane16_swap(c16, c16, false, false));
      const uint32_t d32 = __builtin_bit_cast(uint32_t, bd), c32 = (uint32_t)bj;
      nearer(__builtin_amdgcn_permlane32_swap(d32, d32, false, false), __builtin_amdgcn_permlane32_swap(c32, c32, false, false));
    }
    if (bj >= k) bj = 0;   // no candidate compares (the distances are not numbers): the first cluster, as a comparison that never holds leaves it
    if (first) {
      if (bj != mine) sm.vote[it & 1] = 1;
      atomicOr(&sm.next[bj][p >> 5], 1u << (p & 31));
    }
    mine = bj;
    __syncthreads();
    if (!sm.vote[it & 1]) {
      converged = true;   // the products at hand are those with the final centroids
      break;
    }
    // members of every cluster; a cluster without any keeps its basis
    int rank = 0;
    if (first) {
#pragma unroll
      for (int w = 0; w < kWords; ++w) rank += __popc(sm.next[mine][w] & (w < (p >> 5) ? ~0u : (w == (p >> 5) ? (1u << (p & 31)) - 1u : 0u)));
    }
    if (wave == W - 1) {
      if (lane == 0) sm.vote[~it & 1] = 0;
      int m = 0;
      // a cluster that gets back the members it lost has the centroid it had, but their products (own) are with others by now
      bool differs = sm.count[lane] == 0;
      uint32_t row[kWords];
#pragma unroll
      for (int w = 0; w < kWords; ++w) {
        row[w] = sm.next[lane][w];
        m += __popc(row[w]);
        differs |= row[w] != sm.basis[lane][w];
      }
      if (m > 0) {
#pragma unroll
        for (int w = 0; w < kWords; ++w) sm.basis[lane][w] = row[w];
      }
      const bool moved = m > 0 && differs;
      const int fours = moved ? (m + 3) >> 2 : 0;
      const int upto = wave_scan(fours, [](int x, int y) { return x + y; });
      const int from = 4 * (upto - fours);
      sm.count[lane] = m;
      sm.start[lane] = moved ? (uint32_t)from : kUnmoved;
      for (int q = m; q < 4 * fours; ++q) sm.list[from + q] = 0u;
      if (lane == 63) sm.steps = upto;
    }
    __syncthreads();
    if (first && sm.start[mine] != kUnmoved) sm.list[sm.start[mine] + rank] = member(p, mine, rank >> 2 == (int)(sm.count[mine] - 1) >> 2);
    __syncthreads();
  }
  // ---- survivors: nearest member of every cluster under the final centroids
  if (!converged) products();
  if (tid < kTbeMaxKeep) {
    sm.low[tid] = kTbeMaxTokens;
    sm.best[tid] = ~0ull;
  }
  __syncthreads();
  if (first) {
    const float dist = fmaxf(fmaf(-2.f, sm.own[p], sm.gram[tp + p]) + sm.cc[mine & 3][mine >> 2], 0.f);
    atomicMin(&sm.low[mine], p);
    // distances are not negative, so their bit patterns order like the numbers; the index breaks ties
    atomicMin(&sm.best[mine], ((unsigned long long)__builtin_bit_cast(uint32_t, dist) << 32) | (unsigned)p);
  }
  __syncthreads();
  if (first) {
    // two members are equally near their mean whatever the rounding says: the earlier one stays (a cluster with members
    // has them as its basis)
    const bool keep = sm.count[mine] <= 2 ? p == sm.low[mine] : (int)(sm.best[mine] & 0xFFFFFFFFull) == p;
    a.ev_handle[lo + p] = keep ? -1 : a.tok_handle[lo + p];
    a.assign[lo + p] = mine;
  }
  // ---- the centroids, for callers that look at them.  The members of all clusters in a row, cluster by cluster, each in index order (the matrix has
  // been used: a cluster that has lost its last member shares those it had, so there may be more than n); a wave takes 256 channels and a share of the
  // row, kRows members' rows in flight whatever the sizes of the clusters.  (A wave per cluster and 1,024 channels with two rows in flight: whoever had a
  // cluster of sixty members took thirty turns, 12 to 30 us where it is now 5 to 12.)  Nothing here reads them again: past the caches, where they made
  // the next call's gram kernel wait (66 us, now 60)
  __syncthreads();
  uint32_t* const row = (uint32_t*)sm.gram;   // point | cluster << 8 | last member << 31
  static_assert(sizeof(sm.gram) >= 4 * kTbeMaxKeep * POINTS, "all points in all clusters");
  int size = 0;                               // of cluster `lane`, and where its members begin
#pragma unroll
  for (int w = 0; w < kWords; ++w) size += __popc(sm.basis[lane][w]);
  int begin = wave_scan(size, [](int x, int y) { return x + y; });
  const int total = __builtin_amdgcn_readlane(begin, 63);
  begin -= size;
  for (int j = wave; j < k; j += W) {
    int at = __builtin_amdgcn_readlane(begin, j);
    const int end = at + __builtin_amdgcn_readlane(size, j);
    for (int q = 0; q < n; q += 64) {
      const uint64_t in = (uint64_t)sm.basis[j][q / 32 + 1] << 32 | sm.basis[j][q / 32];
      const int to = at + __popcll(in & ((1ull << lane) - 1ull));
      if (in >> lane & 1ull) row[to] = (uint32_t)(q + lane) | (uint32_t)j << 8 | (to + 1 == end ? 1u << 31 : 0u);
      at += __popcll(in);
    }
  }
  __syncthreads();
  const float inv = 1.0f / (float)size;
  const float* x = a.x + (int64_t)lo * dim;
  float* cent = a.cent + (int64_t)seg * kTbeMaxKeep * dim;
  const int slices = (dim + 255) >> 8, shares = slices < W ? W / slices : 1;
  for (int unit = wave; unit < slices * shares; unit += W) {
    const int share = unit / slices, d0 = 256 * (unit - share * slices) + 4 * lane;
    // whole clusters: those that begin in the share
    const int j0 = __popcll(__ballot(lane < k && begin < share * total / shares)), j1 = __popcll(__ballot(lane < k && begin < (share + 1) * total / shares));
    if (j0 == j1) continue;
    const int e0 = __builtin_amdgcn_readlane(begin, j0), e1 = j1 < k ? __builtin_amdgcn_readlane(begin, min(j1, 63)) : total;
    const bool on = d0 < dim;
    const float* const col = x + (on ? d0 : 0);
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    for (int e = e0; e < e1; e += kRows) {
      const uint32_t some = row[min(e + min(lane, kRows - 1), e1 - 1)];
      f32x4 r[kRows];
#pragma unroll
      for (int u = 0; u < kRows; ++u) r[u] = *(const f32x4*)(col + (int64_t)(__builtin_amdgcn_readlane(some, u) & 255) * dim);
#pragma unroll
      for (int u = 0; u < kRows; ++u) {
        if (e + u >= e1) break;
        sum += r[u];
        const uint32_t m = __builtin_amdgcn_readlane(some, u);
        if (m >> 31) {
          const int j = m >> 8 & 63;
          const f32x4 mean = sum * __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, inv), j));
          if (on) __builtin_nontemporal_store(mean, (f32x4*)&cent[(int64_t)j * dim + d0]);
          sum = f32x4{0.f, 0.f, 0.f, 0.f};
        }
      }
    }
  }
}

// A segment that is not clustered: outside what is covered, then nothing is evicted, and the caller is told; or everything survives
template <int THREADS>
__device__ __forceinline__ bool leave_alone(const thinkv_view& v, const TbeArgs& a, int lo, int hi, int want) {
  const int n = hi - lo;
  if (n <= 0) return true;
  const bool ok = seg_ok(a, lo, hi, want);
  if (ok && want < n) return false;
  if (!ok && threadIdx.x == 0) atomicOr(&v.dev_status[v.cfg.max_seqs * v.cfg.n_layers], THINKV_ST_BAD_SEGMENT);
  for (int i = threadIdx.x; i < n && lo >= 0 && lo + i < a.n_tok; i += THREADS) {
    a.ev_handle[lo + i] = -1;
    a.assign[lo + i] = -1;
  }
  return true;
}

// The parts of the matrix meet, in order (they lie where the centroids will: all have been read before those are written)
template <int THREADS>
__device__ __forceinline__ void add_parts(const float* parts, int slices, int n, float* gram) {
  const int all = tri(n);
  for (int i0 = threadIdx.x; i0 < all; i0 += 4 * THREADS) {   // sixteen loads under way
    float part[kSlices][4];
#pragma unroll
    for (int s = 0; s < kSlices; ++s)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = i0 + THREADS * q;
        part[s][q] = s < slices && i < all ? parts[s * all + i] : 0.f;
      }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = i0 + THREADS * q;
      float sum = part[0][q];
#pragma unroll
      for (int s = 1; s < kSlices; ++s) sum += part[s][q];
      if (i < all) gram[i] = sum;
    }
  }
}

__global__ __launch_bounds__(64 * kKmWaves) __attribute__((amdgpu_waves_per_eu(6))) void tbe_kmeans_kernel(thinkv_view v, TbeArgs a) {
  const int seg = blockIdx.x, lo = a.seg_offset[seg], hi = a.seg_offset[seg + 1], n = hi - lo, want = a.seg_keep[seg];
  if (leave_alone<64 * kKmWaves>(v, a, lo, hi, want)) return;
  if (n > kFewPoints) return;   // tbe_whole_kernel's, or tbe_wide_kernel's
  __shared__ __attribute__((aligned(16))) KmScratch<kKmWaves, kFewPoints> sm;
  add_parts<64 * kKmWaves>(parts_of(a, seg), gram_slices(a, n, v.cfg.n_kv_heads), n, sm.gram);
  choose_survivors(a, seg, lo, n, want, sm);
}

// The segments that kmeans leaves out: a workgroup of sixteen waves, with the LDS of a whole compute unit, makes the matrix and iterates.
// Where there are none, the launch is 5 us.  (A segment a lane to find them: no less, and five more registers spilled.  The narrow form at head_dim 128 spills five,
// six in the paper's formats: what follows from the thread's number, read back once a tile; the other forms none.)  NARROW: it is the only
// kernel, for all segments and for the rows of tokens that are not clustered.
template <int D, bool FP, bool NARROW>
__global__ __launch_bounds__(64 * kWholeWaves) void tbe_whole_kernel(thinkv_view v, TbeArgs a) {
  constexpr int kThreads = 64 * kWholeWaves;
  __shared__ __attribute__((aligned(16))) union {
    GramScratch<kTbeMaxTokens, 2> tile;
    KmScratch<kWholeWaves, kTbeMaxTokens> km;
  } sm;
  const int H = v.cfg.n_kv_heads;
  for (int seg = blockIdx.x; seg < a.n_seg; seg += gridDim.x) {
    const int lo = a.seg_offset[seg], hi = a.seg_offset[seg + 1], n = hi - lo, want = a.seg_keep[seg];
    if (NARROW) {
      if (leave_alone<kThreads>(v, a, lo, hi, want)) {
        write_rows<D, FP, kThreads>(v, a, lo > 0 ? lo : 0, hi < a.n_tok ? hi : a.n_tok, sm.tile.at);
        continue;
      }
    } else if (n <= kFewPoints || !seg_ok(a, lo, hi, want)) {   // (nobody keeps so many)
      continue;
    }
    __syncthreads();   // the segment before is done
    find_tokens(v, a, lo, n, sm.tile.at);
    gram_matrix<D, FP, kWholeWaves>(v, n, 0, H, 0, sm.tile, a.x + (int64_t)lo * a.dim, a.dim, [] { __syncthreads(); },   // the matrix takes the tiles' place
                                    [&](int p, int q, float d) { sm.km.gram[tri(p) + q] = d; });
    choose_survivors(a, seg, lo, n, want, sm.km);
  }
  if (NARROW) write_outside<D, FP, kThreads>(v, a, blockIdx.x, gridDim.x, sm.tile.at);
}

// ... or, wide, adds the parts that gram has made of it
__global__ __launch_bounds__(64 * kWholeWaves) void tbe_wide_kernel(thinkv_view v, TbeArgs a) {
  __shared__ __attribute__((aligned(16))) KmScratch<kWholeWaves, kTbeMaxTokens> sm;
  for (int seg = blockIdx.x; seg < a.n_seg; seg += gridDim.x) {
    const int lo = a.seg_offset[seg], hi = a.seg_offset[seg + 1], n = hi - lo, want = a.seg_keep[seg];
    if (n <= kFewPoints || !seg_ok(a, lo, hi, want)) continue;
    __syncthreads();   // the segment before is done
    add_parts<64 * kWholeWaves>(parts_of(a, seg), gram_slices(a, n, v.cfg.n_kv_heads), n, sm.gram);
    choose_survivors(a, seg, lo, n, want, sm);
  }
}
static_assert(kTbeMaxKeep <= kFewPoints, "a segment that tbe_whole_kernel or tbe_wide_kernel takes is cut");

template <int D, bool FP>
static void launch_kernels(const thinkv_view& v, const TbeArgs& a, hipStream_t st) {
  // Tokens outside every segment: 64 to a workgroup, 256 workgroups at most (32k such tokens behind 32
  // segments: by four workgroups 987 us a call, by a kernel of its own for the rows of all tokens 101, now 72).
  const int outside = (a.n_tok + 63) / 64;
  const int shares = outside < 256 ? outside : 256;
  const dim3 whole(64 * kWholeWaves);
  if (is_narrow(a.dim)) {
    hipLaunchKernelGGL((tbe_whole_kernel<D, FP, true>), dim3(a.n_seg > shares ? a.n_seg : shares), whole, 0, st, v, a);
    return;
  }
  const dim3 grid(a.n_seg * kSlices + shares);
  if (is_wide(a.dim, a.n_seg)) hipLaunchKernelGGL((tbe_gram_kernel<D, FP, true>), grid, dim3(kGramThreads), 0, st, v, a);
  else hipLaunchKernelGGL((tbe_gram_kernel<D, FP, false>), grid, dim3(kGramThreads), 0, st, v, a);
  hipLaunchKernelGGL(tbe_kmeans_kernel, dim3(a.n_seg), dim3(64 * kKmWaves), 0, st, v, a);
  if (a.n_tok <= kFewPoints) return;   // (no segment can be larger)
  const dim3 units(a.n_seg < 256 ? a.n_seg : 256);   // they go round the segments
  if (is_wide(a.dim, a.n_seg)) hipLaunchKernelGGL(tbe_wide_kernel, units, whole, 0, st, v, a);
  else hipLaunchKernelGGL((tbe_whole_kernel<D, FP, false>), units, whole, 0, st, v, a);
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
  const bool fp = v.cfg.format == THINKV_FMT_FP;
  if (v.cfg.head_dim == 128)
    fp ? launch_kernels<128, true>(v, a, st) : launch_kernels<128, false>(v, a, st);
  else
    fp ? launch_kernels<64, true>(v, a, st) : launch_kernels<64, false>(v, a, st);
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
// Two kernels, or three.  count (one workgroup per examined sequence): live tokens per segment (a thread takes four slots of a page:
// one load of positions, a binary search in the segment starts, held in LDS, where a slot leaves the segment of the one
// before), then the plan, whose cuts wait in a staging area.  fill (one workgroup per sequence): the sequence's place in
// the dense output lists from the totals of the sequences before it; where the lists are too short for all, the sequences
// in order keep the leading cuts that still fit (the rest waits for the next call).  Then the list offsets of its cuts by a
// prefix sum, and its live tokens are dealt to their lists.  sort (one wave per cut, in the fill kernel or, where a sequence may
// have many cuts, by a launch of its own): each list is put in ascending position, so the output does not depend on the order in which threads
// dealt.  32 sequences of 2k to 4k tokens, 314 cuts, us (sixteen slots of three pages a thread, one thread for the
// second case and a kernel for the offsets / now): count 39 / 10, offsets 9 / -, fill 32 and sort 19 / 13 together.
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
    int4 pos[kAhead] = {};
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
// keeps the leading ones that do.  b = B: the ends of the lists.  64 sequences at a time: those that fit whole are placed by prefix sums, up
// to the first that does not, which is looked at cut by cut; those whose first cut is too long for what is left now are passed over.
// (Every workgroup does this for itself.  1,024 and 3,000 sequences of three cuts, lists for a quarter of them, us a call: by a kernel of one
// wave, one sequence after the other, 862 and 2,420, so by every workgroup 1,229 and 8,324, now 74 and 354.)
__device__ inline Place place_in_order(const PlanArgs& a, int b) {
  const int lane = threadIdx.x & 63;
  Place at = {0, 0, 0};
  for (int i0 = 0; i0 <= b && i0 < a.B; i0 += 64) {
    const int i = i0 + lane;
    const bool in = i <= b && i < a.B;
    const int nc = in ? a.st_ncuts[i] : 0, tot = nc > 0 ? a.st_total[i] : 0;
    const int first = nc > 0 ? a.st_cnt[(int64_t)i * a.max_cuts] : 0;
    const int lane_b = b - i0;   // (in another 64: not below 64)
    unsigned long long open = __ballot(nc > 0 && at.seg < a.cap_seg && first <= a.cap_tok - at.tok);
    while (open) {
      const bool mine = open >> lane & 1;
      const int c = mine ? nc : 0, t = mine ? tot : 0;
      int upto_c = c, upto_t = t;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int oc = __shfl_up(upto_c, d, 64), ot = __shfl_up(upto_t, d, 64);
        if (lane >= d) {
          upto_c += oc;
          upto_t += ot;
        }
      }
      const unsigned long long cut_off = __ballot(mine && (upto_c > a.cap_seg - at.seg || upto_t > a.cap_tok - at.tok));
      const int f = cut_off ? __builtin_ctzll(cut_off) : 64;   // the first that does not fit whole
      if (lane_b < f && lane_b < 64) return {at.seg + __shfl(upto_c - c, lane_b, 64), at.tok + __shfl(upto_t - t, lane_b, 64), __shfl(c, lane_b, 64)};
      if (f == 64) {
        at.seg += __shfl(upto_c, 63, 64);
        at.tok += __shfl(upto_t, 63, 64);
        break;
      }
      at.seg += __shfl(upto_c - c, f, 64);
      at.tok += __shfl(upto_t - t, f, 64);
      // leading cuts that still fit (the lists only grow, so the first that does not fit ends them)
      const int n = __shfl(nc, f, 64);
      const int32_t* cnt = a.st_cnt + (int64_t)(i0 + f) * a.max_cuts;
      int val[4], ex[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) val[q] = 4 * lane + q < n ? cnt[4 * lane + q] : 0;
      wave_scan4(val, ex);
      int fits = 0, fits_tok = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int j = 4 * lane + q;
        if (j < n && j < a.cap_seg - at.seg && ex[q] + val[q] <= a.cap_tok - at.tok) {
          ++fits;
          fits_tok += val[q];
        }
      }
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) {
        fits += __shfl_xor(fits, d, 64);
        fits_tok += __shfl_xor(fits_tok, d, 64);
      }
      if (f == lane_b) return {at.seg, at.tok, fits};
      at.seg += fits;
      at.tok += fits_tok;
      open = __ballot(mine && lane > f && at.seg < a.cap_seg && first <= a.cap_tok - at.tok);
    }
  }
  return at;
}

// A cut's list [lo, lo + n) (at most kTbeMaxTokens: larger segments are never cut) into ascending order of the positions, by one wave.  A segment's
// positions lie close together: within 2,048 of each other, and no two alike, a bit each in a row of words says by counting how many are before a token.
// Otherwise a token's rank is the number of smaller keys (position, then place in the list), four keys of the list compared at a time.
// keys: LDS, kTbeMaxTokens of them.  (By keys alone, which is 640 comparisons of 64 bits a lane for 160 tokens, the fill kernel of the plan below took 24 us, now 13.)
struct CutList {
  int lo, n;
  int pos[kPT], h[kPT];
  __device__ __forceinline__ void load(const PlanArgs& a, int lo_, int n_) {
    lo = lo_;
    n = n_;
#pragma unroll
    for (int q = 0; q < kPT; ++q) {
      const int i = (threadIdx.x & 63) + 64 * q;
      pos[q] = 0x7FFFFFFF;
      h[q] = 0;
      if (i < n) {
        pos[q] = a.tok_seq[lo + i];
        h[q] = a.tok_handle[lo + i];
      }
    }
  }
};
// M lists side by side: what a wave waits for is LDS, five times, whatever there is to do.
template <int M>
__device__ __forceinline__ void sort_cuts(const PlanArgs& a, const CutList (&l)[M], int seq, long long (*keys)[kTbeMaxTokens]) {
  const int lane = threadIdx.x & 63;
  auto settle = [] {   // (a wave's LDS operations happen in order)
    __builtin_amdgcn_wave_barrier();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  };
  int rank[M][kPT] = {};
  uint32_t at[M][kPT], bit[M][kPT];
  bool far[M];
#pragma unroll
  for (int m = 0; m < M; ++m) {
    int first = 0x7FFFFFFF;
#pragma unroll
    for (int q = 0; q < kPT; ++q) first = l[m].pos[q] < first ? l[m].pos[q] : first;
    first = 0x7FFFFFFF - last_lane(wave_scan(0x7FFFFFFF - first, [](int x, int y) { return x > y ? x : y; }));   // (of all lanes)
    far[m] = false;
#pragma unroll
    for (int q = 0; q < kPT; ++q) {
      const bool in = lane + 64 * q < l[m].n;
      at[m][q] = (uint32_t)l[m].pos[q] - (uint32_t)first;
      far[m] = far[m] || (in && at[m][q] >= 2048u);
      in && at[m][q] < 2048u ? bit[m][q] = 1u << (at[m][q] & 31u) : (at[m][q] = 32u * lane, bit[m][q] = 0u);   // (who has no token sets nothing, in a word of its own)
    }
    ((uint32_t*)keys[m])[lane] = 0u;
  }
  settle();
  uint32_t was[M][kPT];
#pragma unroll
  for (int m = 0; m < M; ++m)
#pragma unroll
    for (int q = 0; q < kPT; ++q) was[m][q] = atomicOr((uint32_t*)keys[m] + (at[m][q] >> 5), bit[m][q]);
  settle();
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const int mine = __popc(((uint32_t*)keys[m])[lane]);
    ((uint32_t*)keys[m])[64 + lane] = (uint32_t)(wave_scan(mine, [](int x, int y) { return x + y; }) - mine);
  }
  settle();
#pragma unroll
  for (int m = 0; m < M; ++m)
#pragma unroll
    for (int q = 0; q < kPT; ++q) {
      const uint32_t* const words = (const uint32_t*)keys[m] + (at[m][q] >> 5);
      rank[m][q] = (int)words[64] + __popc(words[0] & (bit[m][q] - 1u));
    }
#pragma unroll
  for (int m = 0; m < M; ++m) {
    uint32_t twice = 0;
#pragma unroll
    for (int q = 0; q < kPT; ++q) twice |= was[m][q] & bit[m][q];
    const int n = l[m].n;
    if (!__all(!far[m] && twice == 0)) {   // not close together, or two alike
      settle();
      long long key[kPT];
#pragma unroll
      for (int q = 0; q < kPT; ++q) {
        const int i = lane + 64 * q;
        key[q] = i < n ? (long long)l[m].pos[q] << 8 | i : 0x7FFFFFFFFFFFFFFFll;
        keys[m][i] = key[q];
        rank[m][q] = 0;
      }
      settle();
      for (int i = 0; i < n; i += 4) {
        const long long o[4] = {keys[m][i], keys[m][i + 1], keys[m][i + 2], keys[m][i + 3]};
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int q = 0; q < kPT; ++q) rank[m][q] += o[e] < key[q];
      }
    }
#pragma unroll
    for (int q = 0; q < kPT; ++q)
      if (lane + 64 * q < n) {
        a.tok_handle[l[m].lo + rank[m][q]] = l[m].h[q];
        a.tok_seq[l[m].lo + rank[m][q]] = seq;
      }
  }
  settle();
}

// Up to this many cuts a sequence, the workgroup that deals out a sequence's tokens sorts its lists as well, two rounds of two for each of its sixteen waves at
// most.  The bound is the caller's, which is all that the host knows.  Where a sequence has few cuts that saves a launch, where it has the 64 that are allowed a launch with a
// wave for every cut would be faster; beyond that it is taken.  The plan, us, with lists sorted by keys in a launch / here / with a launch and rows of bits: 256 sequences of
// 16 cuts of 128 tokens 28 / 20.9 / 25, 32 of 10 cuts of 64 to 192 29.5 / 23.5 / 24.4, 1 of 32 cuts of 200 33.5 / 28.3 / 27.4, 1 of 48 40.4 / 37.6 / 34.2, 1 of 64
// 45.4 / 43.4 / 39.1, 32 of 64 cuts of 128 35.9 / 35.6 / 33.5.  (One list at a time: 1 of 64 46.0, 32 of 64 36.7; two also where a wave has one: 0.5 more.)
constexpr int kSortHere = 64;

template <bool SORT>
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
      if (at.cuts > 0) at = place_in_order(a, b);
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
  if constexpr (SORT) {
    constexpr int kWaves = kPlanThreads / 64;
    __shared__ __attribute__((aligned(16))) long long s_key[kWaves][2][kTbeMaxTokens];
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    __syncthreads();
    if (n_cuts <= kWaves) {   // a list a wave
      CutList l[1];
      if (wave < n_cuts) {
        l[0].load(a, s_off[wave], s_fill[wave]);
        sort_cuts(a, l, seq, s_key[wave]);
      }
      return;
    }
    auto load = [&](CutList (&l)[2], int cu) {
      l[0].load(a, s_off[cu], s_fill[cu]);
      const bool two = cu + kWaves < n_cuts;
      l[1].load(a, two ? s_off[cu + kWaves] : 0, two ? s_fill[cu + kWaves] : 0);
    };
    CutList l[2], next[2];
    if (wave < n_cuts) load(l, wave);
    for (int cu = wave; cu < n_cuts; cu += 2 * kWaves) {
      const int after = cu + 2 * kWaves;
      if (after < n_cuts) load(next, after);
      sort_cuts(a, l, seq, s_key[wave]);
      l[0] = next[0];
      l[1] = next[1];
    }
  }
}

// one wave per cut of the dense lists
__global__ __launch_bounds__(256) void tbe_sort_kernel(PlanArgs a) {
  __shared__ __attribute__((aligned(16))) long long s_key[4][1][kTbeMaxTokens];
  const int wave = threadIdx.x >> 6;
  const int cu = blockIdx.x * 4 + wave;
  if (cu >= a.counts[0]) return;   // the waves do not meet
  const int lo = a.seg_offset[cu];
  CutList l[1];
  l[0].load(a, lo, a.seg_offset[cu + 1] - lo);
  sort_cuts(a, l, a.st_cut_seq[cu], s_key[wave]);
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
  const dim3 each(B > 0 ? B : 1);
  if (max_cuts <= kSortHere) {
    hipLaunchKernelGGL(tbe_fill_kernel<true>, each, dim3(kPlanThreads), 0, st, v, a);
    return hipGetLastError() == hipSuccess ? THINKV_OK : THINKV_E_HIP;
  }
  hipLaunchKernelGGL(tbe_fill_kernel<false>, each, dim3(kPlanThreads), 0, st, v, a);
  const int64_t most = (int64_t)B * max_cuts < cap_seg ? (int64_t)B * max_cuts : cap_seg;
  if (most > 0) hipLaunchKernelGGL(tbe_sort_kernel, dim3((unsigned)((most + 3) / 4)), dim3(256), 0, st, a);
  return hipGetLastError() == hipSuccess ? THINKV_OK : THINKV_E_HIP;
}

}  // namespace thinkv

// Attention-sparsity statistic of a decode step (Sec. 4.1 of the paper: the thought type of a
// step is read off how sparse its normalised attention scores are; appendix "Grouped-Query
// Attention": the scaled scores of the G query heads of a group are max-pooled, the pooled row
// is renormalised by a softmax over the keys, an entry is negligible when it lies below 1 % of
// the row's maximum, and the fractions of negligible entries are averaged over the groups).
//
// The scores are those the attention kernel computes anyway, so the statistic rides on a decode
// call: the STAT instantiation of the attention kernel stores the pooled score of every slot of the pages it
// visits (16 floats per page, log2 domain, -inf for dead and invisible slots), and one more launch, two for large batches, takes
// the maximum of each (query, kv-head) row, counts, and averages over the kv-heads.  Full attention visits the pages with
// a live slot, which the counts tell by the masks; a sliding window visits what it reaches, so there a fill kernel sets the
// buffer to -inf first.  (16 queries over 8k to 32k tokens: 131.4 us with the
// fill and rows read twice, 127 so.)  w_j < 0.01 max w  <=>  pooled_j <
// max pooled - log2(100) in the log2 domain, so no softmax is ever formed.
#include "decode_mfma_kernel.h"

namespace thinkv {

__global__ __launch_bounds__(256) void stat_fill_kernel(float4* p, int64_t n4) {
  const float ninf = -INFINITY;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = make_float4(ninf, ninf, ninf, ninf);
}

// The merge of the partial rows and the counts need the attention kernel's results and nothing of each other: one launch.
// `merges` workgroups of 1,024 threads come first and merge 1,024 / D query heads each; then
// one workgroup per (query, kv-head): the row maximum, then the counts of visible and of
// negligible entries, and the row's fraction negligible / visible (0 where nothing is visible).  The mean over the kv-heads: fractions are
// added up as whole numbers of a small unit (exactly, so in any order) in the low bits of a word that the attention kernel has cleared; every addition counts
// itself in the high ones, and who finds that it was the last has the sum, without a wait for others or a fence (one launch less: 1 x 2k tokens 21.6 us, now
// 20.4).  Without such words the fractions go to frac[b][kv-head].  Rows are read 16 bytes a lane, once up to 32,768 entries.  MASKS: entries of pages without a live
// slot were not written and count as -inf.
// Two workgroups share a compute unit, so a thread has 64 registers: indices are scalars or 32 bits wide.  (With 66 there was one: 256 x 1k tokens, 8
// kv-heads of 128, 130.4 us, now 113.7; 256 x 500..5k 206 and 190; two launches without that 117 and 195.)
constexpr int kKept = 8;
template <int D, bool MASKS>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8))) void stat_count_kernel(thinkv_view v, DecodeArgs a, float* frac, int merges) {
  const thinkv_config& c = v.cfg;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  __shared__ MergeLds<D> s_merge[1024 / D];
  __shared__ float s_max[16];
  __shared__ int s_cnt[2][16];
  if ((int)blockIdx.x < merges) {
    const int per = 1024 / D, head = blockIdx.x * per + tid / D, heads = a.B * c.n_q_heads, hd = head < heads ? head : heads - 1;
    merge_head<D>(v, a, hd / c.n_q_heads, hd % c.n_q_heads, tid % D, head < heads, s_merge[tid / D]);
    return;
  }
  const int b = uniform(((int)blockIdx.x - merges) / c.n_kv_heads), hkv = (int)blockIdx.x - merges - b * c.n_kv_heads;
  const int seq = uniform(a.seq_ids[b]);
  int64_t n = 0;
  int end0 = 0, end1 = 0;   // where the pages of the first two types end
  if (seq >= 0 && seq < c.max_seqs) {
    end0 = uniform(v.n_pages[npages_index(c, seq, a.layer, 0)]);
    end1 = end0 + uniform(v.n_pages[npages_index(c, seq, a.layer, 1)]);
    n = (int64_t)end1 + uniform(v.n_pages[npages_index(c, seq, a.layer, 2)]);
  }
  n *= kPage;
  if (n > a.stat_stride) n = a.stat_stride;   // the host's bound on the context was too small: count what was kept
  const float4* row = (const float4*)(a.stat + ((int64_t)b * c.n_kv_heads + hkv) * a.stat_stride);
  const int n4 = (int)(n / 4);                // whole pages: a multiple of four
  const uint32_t* const masks = n4 > 0 ? v.slot_mask + table_base(c, seq, a.layer, 0) : nullptr;
  auto entry = [&](int i) {
    float4 x = row[i];
    if (MASKS && n4 > 0) {
      const int p = i >> 2;   // the types' page lists lie max_pages apart
      const uint32_t m = masks[(uint32_t)(p < end0 ? p : (p < end1 ? p - end0 + c.max_pages : p - end1 + 2 * c.max_pages))];   // (max_pages < 2^24)
      if ((m & 0xFFFFu) == 0) x = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
    }
    return x;
  };
  // the first 32,768 entries stay in registers between the passes, all their loads under way at once
  float4 kept[kKept];
#pragma unroll
  for (int u = 0; u < kKept; ++u) kept[u] = entry(min(tid + 1024 * u, max(n4 - 1, 0)));
  float m = -INFINITY;
  auto highest = [&](float4 x) { m = fmaxf(fmaxf(m, fmaxf(x.x, x.y)), fmaxf(x.z, x.w)); };
#pragma unroll
  for (int u = 0; u < kKept; ++u)
    if (tid + 1024 * u < n4) highest(kept[u]);
  for (int i = tid + 1024 * kKept; i < n4; i += 1024) highest(entry(i));
  for (int d = 32; d >= 1; d >>= 1) m = fmaxf(m, __shfl_xor(m, d, 64));
  if (lane == 0) s_max[wave] = m;
  __syncthreads();
  m = s_max[0];
  for (int w = 1; w < 16; ++w) m = fmaxf(m, s_max[w]);
  const float cut = m - 6.643856189774724f;   // log2(100)
  int vis = 0, neg = 0;
  auto count = [&](float4 x) {
    vis += (x.x > -INFINITY) + (x.y > -INFINITY) + (x.z > -INFINITY) + (x.w > -INFINITY);
    neg += (x.x > -INFINITY && x.x < cut) + (x.y > -INFINITY && x.y < cut) + (x.z > -INFINITY && x.z < cut) +
           (x.w > -INFINITY && x.w < cut);
  };
#pragma unroll
  for (int u = 0; u < kKept; ++u)
    if (tid + 1024 * u < n4) count(kept[u]);
  for (int i = tid + 1024 * kKept; i < n4; i += 1024) count(entry(i));
  for (int d = 32; d >= 1; d >>= 1) {
    vis += __shfl_xor(vis, d, 64);
    neg += __shfl_xor(neg, d, 64);
  }
  if (lane == 0) {
    s_cnt[0][wave] = vis;
    s_cnt[1][wave] = neg;
  }
  __syncthreads();
  if (tid == 0) {
    int tv = 0, tn = 0;
    for (int w = 0; w < 16; ++w) {
      tv += s_cnt[0][w];
      tn += s_cnt[1][w];
    }
    if (a.stat_sum) {
      // (kStatHeads says why the units lose nothing)
      const int lg = 32 - __builtin_clz(c.n_kv_heads - 1), at = 63 - lg, unit = 62 - 2 * lg;
      const double one = __builtin_bit_cast(double, (unsigned long long)(1023 + unit) << 52);   // 2^unit
      const unsigned long long mine = (tv > 0 ? (unsigned long long)__builtin_rint((double)((float)tn / (float)tv) * one) : 0ull) | 1ull << at;
      const unsigned long long all = atomicAdd(&a.stat_sum[b], mine) + mine;
      if ((int)(all >> at) == c.n_kv_heads) a.sparsity[b] = (float)((double)(all & ((1ull << at) - 1ull)) / (one * (double)c.n_kv_heads));
    } else {
      frac[(int64_t)b * c.n_kv_heads + hkv] = tv > 0 ? (float)tn / (float)tv : 0.f;
    }
  }
}

// sparsity[b] = mean over kv-heads where the fractions are not added up (a.stat_sum): summed
// in head order, the same bits on every run
__global__ __launch_bounds__(256) void stat_mean_kernel(const float* frac, float* sparsity, int B, int Hkv) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  float total = 0.f;
  for (int h = 0; h < Hkv; ++h) total += frac[(int64_t)b * Hkv + h];
  sparsity[b] = total / (float)Hkv;
}

int launch_stat_fill(const thinkv_view& v, const DecodeArgs& a, hipStream_t st) {
  if (a.window <= 0) return THINKV_OK;   // the counts go by the masks
  const int64_t n4 = (int64_t)a.B * v.cfg.n_kv_heads * a.stat_stride / 4;
  int64_t blocks = (n4 + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(stat_fill_kernel, dim3((unsigned)blocks), dim3(256), 0, st, (float4*)a.stat, n4);
  return hipGetLastError() == hipSuccess ? THINKV_OK : THINKV_E_HIP;
}

int launch_decode_mfma_stat(const thinkv_view& v, const DecodeArgs& a, hipStream_t st) { return launch_decode_mfma_t<true>(v, a, st); }

int launch_stat_count(const thinkv_view& v, const DecodeArgs& a, hipStream_t st) {
  // the per-row fractions live behind the pooled scores
  float* frac = a.stat + (int64_t)a.B * v.cfg.n_kv_heads * a.stat_stride;
  const int D = v.cfg.head_dim, merges = (a.B * v.cfg.n_q_heads + 1024 / D - 1) / (1024 / D);
  const dim3 grid(merges + v.cfg.n_kv_heads * a.B);
  if (D == 128) {
    if (a.window > 0) hipLaunchKernelGGL((stat_count_kernel<128, false>), grid, dim3(1024), 0, st, v, a, frac, merges);
    else hipLaunchKernelGGL((stat_count_kernel<128, true>), grid, dim3(1024), 0, st, v, a, frac, merges);
  } else {
    if (a.window > 0) hipLaunchKernelGGL((stat_count_kernel<64, false>), grid, dim3(1024), 0, st, v, a, frac, merges);
    else hipLaunchKernelGGL((stat_count_kernel<64, true>), grid, dim3(1024), 0, st, v, a, frac, merges);
  }
  if (!a.stat_sum) hipLaunchKernelGGL(stat_mean_kernel, dim3((a.B + 255) / 256), dim3(256), 0, st, frac, a.sparsity, a.B, v.cfg.n_kv_heads);
  return hipGetLastError() == hipSuccess ? THINKV_OK : THINKV_E_HIP;
}

}  // namespace thinkv

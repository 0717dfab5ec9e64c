// Soft eviction and view initialisation.
#include "common.h"

namespace thinkv {

// One thread per handle.
__global__ __launch_bounds__(256) void evict_kernel(thinkv_view v, int layer, const int32_t* __restrict__ ev_seq,
                                                    const int32_t* __restrict__ ev_handle, int n_ev) {
  const thinkv_config& c = v.cfg;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_ev) return;
  const int s = ev_seq[i];
  if (s < 0 || s >= c.max_seqs) {
    atomicOr(&v.dev_status[c.max_seqs * c.n_layers], THINKV_ST_BAD_SEQ);
    return;
  }
  evict_one(v, layer, s, ev_handle[i]);
}

// Tables, counters and arenas as an empty cache has them.  The arenas are zero-filled, in 16-byte stores (page sizes are
// multiples of 16 bytes): a page can hold slots that were never written; attention reads them and discards them by their
// live bit, which is only safe if their scales and zero-points are finite numbers.  (One launch instead of one for the
// tables and one an arena, each of which starts on an idle chip: 60 MB of arenas in 14 us instead of 26.)
// Two blocks to a compute unit, four stores of a thread at once: the rate of the stores bounds large arenas, and with eight blocks a unit
// the start of so many waves, each of which goes round all of these loops, bounds small ones.  With the append of 16 prompts of 1k to 4k tokens, of 4 of
// 500 to 2,000 at head_dim 64, of 2 of 200 tokens, us: eight blocks and a store at a time 78.7, 24.8, 16.8, now 77.8, 23.9, 15.8 (four blocks 80.9, 24.1,
// 16.0).  Non-temporal stores take the arenas out of the caches, where an append finds them: 82.9.
__global__ __launch_bounds__(256) void init_kernel(thinkv_view v) {
  const thinkv_config& c = v.cfg;
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int k = 0; k < 3; ++k) {
    const int64_t n = v.arena_pages[k];
    for (int64_t i = tid; i < n; i += stride) {
      v.free_stack[k][i] = (int32_t)(n - 1 - i);
      v.page_filled[k][i] = 0;
      v.page_pos_max[k][i] = -1;
    }
    for (int64_t i = tid; i < n * kPage; i += stride) v.slot_pos[k][i] = -1;
    if (tid == 0) v.free_top[k] = (int32_t)n;
  }
  const int64_t nt = (int64_t)c.max_seqs * c.n_layers * 3 * c.max_pages;
  for (int64_t i = tid; i < nt; i += stride) {
    v.block_table[i] = -1;
    v.slot_mask[i] = 0;
  }
  const int64_t nsl = (int64_t)c.max_seqs * c.n_layers;
  for (int64_t i = tid; i < nsl * 3; i += stride) v.n_pages[i] = 0;
  for (int64_t i = tid; i < nsl; i += stride) v.n_live[i] = 0;
  for (int64_t i = tid; i < nsl + 1; i += stride) v.dev_status[i] = 0;
  for (int64_t i = tid; i < c.max_seqs; i += stride) v.append_counters[i] = 0;
  for (int64_t i = tid; i < nsl * c.n_kv_heads * 4; i += stride) v.work_counters[i] = 0;
  for (int k = 0; k < 3; ++k) {
    const int64_t n16 = v.arena_pages[k] * (int64_t)c.n_kv_heads * block_geom(c.bits_of_class[k], c.head_dim, c.format).block_bytes / 16;
    uint4* const p = (uint4*)v.arena[k];
    const uint4 zero = {0u, 0u, 0u, 0u};
    int64_t i = tid;
    for (; i + 3 * stride < n16; i += 4 * stride) {
      p[i] = zero;
      p[i + stride] = zero;
      p[i + 2 * stride] = zero;
      p[i + 3 * stride] = zero;
    }
    for (; i < n16; i += stride) p[i] = zero;
  }
}

int launch_evict(const thinkv_view& v, int layer, const int32_t* ev_seq, const int32_t* ev_handle, int n_ev, hipStream_t st) {
  if (n_ev == 0) return THINKV_OK;
  hipLaunchKernelGGL(evict_kernel, dim3((n_ev + 255) / 256), dim3(256), 0, st, v, layer, ev_seq, ev_handle, n_ev);
  return hipGetLastError() == hipSuccess ? THINKV_OK : THINKV_E_HIP;
}

int launch_init(const thinkv_view& v, hipStream_t st) {
  hipLaunchKernelGGL(init_kernel, dim3(512), dim3(256), 0, st, v);
  return hipGetLastError() == hipSuccess ? THINKV_OK : THINKV_E_HIP;
}

}  // namespace thinkv

// Decode attention on the matrix cores (gfx950).
//
// The affine dequantisation is distributed over the dot products so that the matrix cores
// only ever see exact operands:
//
//   scores   q.k^_t = sum_g [ s_K(t,g) * (sum_{i in g} q_i c_K(t,i)) + zp_K(t,g) * (sum_{i in g} q_i) ]
//   values   o_c    = sum_t [ (p_t s_V(t,g(c))) * c_V(t,c) ]  +  sum_t p_t zp_V(t,g(c))
//
// The integer codes c are fed to v_mfma_f32_16x16x32_f16 as binary16 numbers without any
// conversion: a b-bit field masked inside a 16-bit half IS the binary16 (sub)normal
// c * 2^(position-24); the power of two is folded into the query (for K) or into the output
// scale (for V).  A quantisation group is 32 channels = the K extent of one MFMA.
//
// Column plan.  The 16 rows / columns of a tile that belong to queries are cut into CS slices of GP
// (GP = 4 or 8 >= the number G of query heads that share the kv-head); slice gl carries the G heads *for
// quantisation group gl* (of the set being worked on: D/32 groups = NSET sets of CS).
// Scores: A = the query (row = (slice, head); the query of group g is placed in slice g's rows only, zeros
// elsewhere), B = the K codes (column = token), so the MFMAs of the CS groups of a set accumulate into ONE
// 16x16 tile, (group, head) x tokens.  Lane (token n, row quad qd) then applies the scale and zero-point of
// ITS token and group -- lane-local binary32 arithmetic on values the lane loaded itself, no broadcast -- and
// the groups are added by half-wave and row exchanges that leave each lane with the scores of GP/4 heads of
// its token and nothing twice: the softmax runs on 16 tokens x G heads per page, spread over the wave.
// (The other orientation, A = codes, leaves every slice of columns with the complete scores of four tokens:
// the exponentials, which the vector unit issues at a quarter of its rate, and everything around them were
// then done CS times over: 292 vector-ALU instructions per page pair and wave, 238 now.)
// The weights go back to the layout of the value product (four tokens per lane, column = (slice, head)) by one
// v_mfma_f32_16x16x4_f32 per page and four heads with a 0/1 matrix: products with one and zero, so exact for numbers (a
// weight that is not one, from a query head that is not finite, must not reach the sum: it would spoil the other heads); or, by
// geometry and format, through LDS (Softmax::weights).
// Values: p * s_V(t, g) is lane-local (each slice multiplies by its own group's
// scale), is split once into two binary16 terms (22 significant bits), and the same B operand
// pair serves the PV MFMAs of every group of the set: the tile of a 16-channel block is only
// read back in the slice of its group.  The zero-point part of the output and the softmax
// denominator are lane-local binary32 sums.
//
// Full-attention layers (decode_stream_kernel).  A work item is a workgroup of several waves on one (query, kv-head); the
// waves draw chunks of page pairs from a ticket counter in LDS, so a wave that sees less bandwidth takes fewer, and
// fold their partials in LDS: one partial row per item, or the result itself where a head has one item.  What bounds
// the launch is the bytes in flight: a pair of pages held in registers while the one before is worked on leaves
// 11 MB in flight on the chip, little more than latency times bandwidth, so every hiccup of a wave shows.  So the
// pages go from memory to LDS directly (global_load_lds, no registers), several pairs ahead: each wave owns a ring
// (its slots are sized by the type being walked), reads a pair into registers when it has landed, asks for the pair
// that will take the slot, and computes.  The waits are vmcnt counts by hand: the compiler knows
// nothing of these loads (they are inline asm without an output), a wait for an older load of its own only waits longer.
// Measured against pairs prefetched into registers (one wave per item, tickets by global atomics, one pair in flight):
// 256 x 1k..64k tokens 1,049 -> 832 us, 16 x 8k 51.6 -> 43.3, 32 x ~2k of scrambled slots 75 -> 48, head_dim 64
// 128 x 4k..32k 313 -> 287.  Three waves a SIMD with rings of 12 KB (one pair of 8-bit pages) lose to two with 18 KB:
// 16 x 8k 64 us, 256 x 1k..64k 1,046 us.
// Sliding-window layers (decode_window_kernel): a workgroup scans the page lists for several kv-heads, then its waves attend
// what is visible through the same rings.
#pragma once
#include <type_traits>

#include "decode_common.h"


namespace thinkv {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef uint16_t ushort2v __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef float float2v __attribute__((ext_vector_type(2)));

union H8 {
  half8 h;
  uint32_t u[4];
};

// max(x, x of another lane), the other lane chosen by a DPP control word: 0xB1 / 0x4E swap
// neighbours / pairs inside a quad of lanes, 0x120 + d rotates the row of 16 by d
template <int CTRL>
__device__ __forceinline__ float max_dpp(float x) {
  const int y = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true);
  return fmaxf(x, __builtin_bit_cast(float, y));
}

// The largest of numbers, in one instruction; a NaN loses.  (fmaxf is up to three: it makes sure of quiet NaNs first.  Not for
// what a matrix or a transcendental instruction has just written: the compiler knows of no wait states for asm.)
__device__ __forceinline__ float largest(float a, float b) {
  float x;
  asm("v_max_f32 %0, %1, %2" : "=v"(x) : "v"(a), "v"(b));
  return x;
}
__device__ __forceinline__ float largest(float a, float b, float c) {
  float x;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(x) : "v"(a), "v"(b), "v"(c));
  return x;
}

__device__ __forceinline__ uint32_t pack_rne(float a, float b) {
  float2v f = {a, b};
  half2v h = __builtin_convertvector(f, half2v);
  return __builtin_bit_cast(uint32_t, h);
}

__device__ __forceinline__ float half_lo(uint32_t u) { return (float)__builtin_bit_cast(_Float16, (uint16_t)(u & 0xFFFFu)); }
__device__ __forceinline__ float half_hi(uint32_t u) { return (float)__builtin_bit_cast(_Float16, (uint16_t)(u >> 16)); }
// binary16 number r (0..3) of the dword pair (a, b)
template <int R>
__device__ __forceinline__ float half_of(uint32_t a, uint32_t b) {
  return R == 0 ? half_lo(a) : (R == 1 ? half_hi(a) : (R == 2 ? half_lo(b) : half_hi(b)));
}

// Field geometry of a b-bit layout: FPH fields per 16-bit half-word.  The matrix core adds the
// products of one instruction in a fixed-width window below the largest *nominal* product
// exponent, and a subnormal operand keeps its nominal exponent (2^-14) however many leading
// zeros it has -- so a code left at the bottom of the half-word would cost up to ten bits of the
// sum.  Every field is therefore moved, by one shift shared with its neighbour field, to sit
// just under bit 11 (offset OMIN or OMIN + BITS), and only the residual 2^REL is folded into
// the other operand.  8-bit codes fill the low byte as they are.
template <int BITS>
struct Fld {
  static constexpr int FPH = 16 / BITS;
  static constexpr uint32_t MASK = ((1u << BITS) - 1u) * 0x00010001u;
  static constexpr int OMIN = BITS == 2 ? 7 : (BITS == 4 ? 3 : 0);
  __device__ static constexpr int rel_of(int f) { return BITS == 8 ? 0 : BITS * ((f % FPH) & 1); }
  // operand register (two codes: low/high half) for field f of the chunk words w[]
  __device__ static __forceinline__ uint32_t get(const uint32_t* w, int f) {
    const int word = f / FPH, pos = f % FPH;
    const uint32_t x = w[word];
    if constexpr (BITS == 8) {
      if (pos == 0) return x & MASK;
      const ushort2v y = __builtin_bit_cast(ushort2v, x) >> (uint16_t)8;   // both halves at once
      return __builtin_bit_cast(uint32_t, y);
    } else {
      // field pair (pos & ~1, pos | 1) starts at bit BITS*(pos & ~1); bring it to bit OMIN
      const int from = BITS * (pos & ~1);
      const uint32_t y = from <= OMIN ? (x << (OMIN - from)) : (x >> (from - OMIN));
      return y & (MASK << (OMIN + BITS * (pos & 1)));
    }
  }
};

// How the 16 columns are shared between query heads and quantisation groups.
template <int D, int GP>
struct Cols {
  static constexpr int NG = D / 32;
  static constexpr int CS = (16 / GP) < NG ? (16 / GP) : NG;   // groups (slices) per column set
  static constexpr int NSET = NG / CS;
};

// What one lane holds of one page: its K and V chunks and, per column set, the scale and zero-point of its
// token and its slice's group for K, and those of its four slots and its slice's group for V.
template <int D, int BITS, int NSET>
struct PageRegs {
  static constexpr int CW = (D / 32) * BITS / 4;  // chunk dwords
  uint32_t kw[CW], vw[CW];
  uint16_t ks[NSET], kz[NSET];
  uint4 vm[NSET];   // (scale 0|1, scale 2|3, zero-point 0|1, zero-point 2|3)
};

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) const uint8_t* LdsPtr;
// pieces of a block in memory (read once: not worth a line of L2) or of its copy in LDS
template <class T> __device__ __forceinline__ T ld_piece(const uint8_t* p) { return __builtin_nontemporal_load((const T*)p); }
template <class T> __device__ __forceinline__ T ld_piece(LdsPtr p) { return *(__attribute__((address_space(3))) const T*)p; }

// chunk `lane` of a code region into the lane's registers
template <int CW, class P>
__device__ __forceinline__ void load_chunk(uint32_t* w, P region, int lane) {
  P src = region + lane * CW * 4;
  if constexpr (CW == 1) {
    w[0] = ld_piece<uint32_t>(src);
  } else if constexpr (CW == 2) {
    const u32x2 a = ld_piece<u32x2>(src);
    w[0] = a.x; w[1] = a.y;
  } else {
#pragma unroll
    for (int i = 0; i < CW; i += 4) {
      const u32x4 a = ld_piece<u32x4>(src + 4 * i);
      w[i] = a.x; w[i + 1] = a.y; w[i + 2] = a.z; w[i + 3] = a.w;
    }
  }
}

// the K half (codes, scale, zero-point) or the V half of one page's block into the lane's registers
template <int D, int BITS, int NSET, class P>
__device__ __forceinline__ void load_keys(PageRegs<D, BITS, NSET>& r, P blk, int lane, const int* k_off) {
  const BlockGeom g = block_geom(BITS, D);
  load_chunk<PageRegs<D, BITS, NSET>::CW>(r.kw, blk + g.k_codes, lane);
#pragma unroll
  for (int s = 0; s < NSET; ++s) {
    r.ks[s] = ld_piece<uint16_t>(blk + g.k_meta + k_off[s]);
    r.kz[s] = ld_piece<uint16_t>(blk + g.k_meta + k_off[s] + 8);
  }
}
template <int D, int BITS, int NSET, class P>
__device__ __forceinline__ void load_values(PageRegs<D, BITS, NSET>& r, P blk, int lane, const int* v_off) {
  const BlockGeom g = block_geom(BITS, D);
  load_chunk<PageRegs<D, BITS, NSET>::CW>(r.vw, blk + g.v_codes, lane);
#pragma unroll
  for (int s = 0; s < NSET; ++s) {
    const u32x4 m = ld_piece<u32x4>(blk + g.v_meta + v_off[s]);
    r.vm[s] = make_uint4(m.x, m.y, m.z, m.w);
  }
}

// Two layouts occur.  Score layout: lane (token n = lane % 16 of the page, row quad qd = lane / 16) holds, for its
// token, the NS = GP / 4 heads head_of(qd, i).  Column layout (value tiles): lane (column n = (slice, head n % GP), qd).
template <int D, int GP, int NSET>
struct WaveState {
  static constexpr int NM = D / 16, NS = GP / 4;
  float4v o[NM];    // column layout; o[mb][r]: channel 16*mb + 4*qd + r (while a type is walked: in its units, and lifted)
  float oz[NSET];   // column layout; this lane's share of sum_t p_t zp_V(t, group of the lane's slice)
  float l[NS];      // score layout; this lane's share of sum_t p_t
  float m[NS];      // score layout; between types: the reference of the head's weights (log2 domain, a whole number); -inf before the first live token
};

// head of value i of a lane in row quad qd, as add_groups leaves the scores
template <int GP>
__device__ __forceinline__ int head_of(int qd, int i) { return GP == 4 ? qd : 4 * (qd & 1) + 2 * (qd >> 1) + i; }

// The lane, of which the compiler knows nothing: what follows from it is worked out where it is used, and no register is kept for it over
// the loops between
__device__ __forceinline__ int fresh_lane() {
  int lane;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
  return lane;
}

__device__ __forceinline__ int fresh(int scalar) {   // likewise
  asm volatile("" : "+s"(scalar));
  return scalar;
}

// x of lane `from`
__device__ __forceinline__ float lane_of(float x, int from) { return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(4 * from, __builtin_bit_cast(int, x))); }

// score layout -> column layout, for values that are the same in all lanes of a row quad
template <int GP>
__device__ __forceinline__ float to_column(const float* x, int lane) {
  const int h = lane & (GP - 1);
  if constexpr (GP == 4) return lane_of(x[0], 16 * h);
  const int src = 16 * ((h >> 2) + (h & 2));
  const float a = lane_of(x[0], src), b = lane_of(x[1], src);
  return (h & 1) ? b : a;
}

__device__ __forceinline__ float add_swapped32(float a, float b) {   // lower half: a + a of the upper half; upper half: b likewise
  auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b), false, false);
  return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
}
__device__ __forceinline__ float add_swapped16(float a, float b) {   // even rows: a + a of the odd row next to it; odd rows: b likewise
  auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b), false, false);
  return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
}
// x[r]: row 4 qd + r of the score tile, i.e. GP = 4: (slice qd, head r), GP = 8: (slice qd / 2, head 4 (qd % 2) + r).
// Adds the slices; each lane keeps the heads head_of(qd, .).
template <int GP>
__device__ __forceinline__ void add_groups(const float* x, float* s) {
  const float y0 = add_swapped32(x[0], x[2]), y1 = add_swapped32(x[1], x[3]);
  if constexpr (GP == 4) {
    s[0] = add_swapped16(y0, y1);
  } else {
    s[0] = y0;
    s[1] = y1;
  }
}

// maximum over the lanes of a row quad (16 tokens)
__device__ __forceinline__ float row_max(float x) {
  return max_dpp<0x128>(max_dpp<0x124>(max_dpp<0x4E>(max_dpp<0xB1>(x))));
}

// maximum over the four lanes that share a token / column (lane ^ 16, lane ^ 32), on the VALU
__device__ __forceinline__ float col_max(float x) {
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  auto r16 = __builtin_amdgcn_permlane16_swap(u, u, false, false);   // rows (0,1) and (2,3) exchanged
  x = fmaxf(__builtin_bit_cast(float, (uint32_t)r16[0]), __builtin_bit_cast(float, (uint32_t)r16[1]));
  const uint32_t w = __builtin_bit_cast(uint32_t, x);
  auto r32 = __builtin_amdgcn_permlane32_swap(w, w, false, false);   // halves exchanged
  return fmaxf(__builtin_bit_cast(float, (uint32_t)r32[0]), __builtin_bit_cast(float, (uint32_t)r32[1]));
}

struct PairIds {
  int pid_a, pid_b;
  uint32_t live_a, live_b;
  int idx_a, idx_b;   // positions in the type's page list (idx_b = -1: no second page); used by STAT only
  // STAT: the pooled scores of the lane's tokens, ua and ub the largest of the lane's heads, to their places among the type's, of which there
  // are `room` pages (a scalar branch)
  static constexpr int kStores = 0;
  __device__ __forceinline__ void keep(float* stat, int room, int, float ua, float ub) const {
    const int lane = fresh_lane();
    put(stat, room, lane, col_max(ua), idx_a);   // (the same in the four lanes of a token, which store it to one place)
    put(stat, room, lane, col_max(ub), idx_b);
  }
  static __device__ __forceinline__ void put(float* stat, int room, int lane, float u, int idx) {
    if (idx >= 0 && idx < room) stat[(int64_t)idx * kPage + (lane & (kPage - 1))] = u;
  }
};
// ... of a pair whose "pages" are made of quads of slots (SlotQuads).  (Two stores, as above, of which the ring's waits know nothing and which they therefore
// wait for too; one counted store, as full attention has it, has not been tried in windows.)
struct QuadIds {
  uint32_t live_a, live_b;
  int at_a, at_b;   // STAT: where the lane's tokens stand among the type's pooled scores (negative: nowhere)
  __device__ __forceinline__ void keep(float* stat, int room, int, float ua, float ub) const {
    put(stat, room, col_max(ua), at_a);
    put(stat, room, col_max(ub), at_b);
  }
  static __device__ __forceinline__ void put(float* stat, int room, float u, int at) {
    if (at >= 0 && at < room * kPage) stat[at] = u;
  }
};

template <int D, int BITS, int NSET>
struct PairRegs {
  PageRegs<D, BITS, NSET> a, b;
};

// ---- direct copies of a block into LDS.  A wave-wide load moves 1 KB (16 bytes a lane) to consecutive LDS bytes from m0
// on; the instruction's offset counts on both sides.  The last, shorter piece runs with some lanes off.  The compiler does
// not see the loads inside the asm, so the wait states between a vector instruction that writes an address register
// (v_readfirstlane) or m0 and the load that reads it are in the asm too: five cover every such pair.
template <int BYTES>
struct BlockDma {
  static constexpr int kFull = BYTES / 1024, kRest = (BYTES % 1024) / 16;   // whole instructions, lanes of the last one
  static constexpr int kOps = kFull + (kRest ? 1 : 0);
  static_assert(BYTES % 16 == 0 && kFull <= 4, "block sizes are multiples of 16 bytes, at most 4.5 KB");
#define TKV_SET "s_mov_b32 m0, %0\n\ts_nop 4\n\t"
#define TKV_DMA(OFF) "global_load_lds_dwordx4 %1, %2 offset:" #OFF " nt\n\t"
#define TKV_SOME(OFF) "s_mov_b64 exec, %3\n\t" TKV_DMA(OFF) "s_mov_b64 exec, -1"
  // lds: LDS byte address, blk: the block in memory (both wave-uniform), voff: 16 * lane.  All lanes are on, before and after:
  // kernels of these files branch on scalars around everything that gets here.
  static __device__ __forceinline__ void issue(uint32_t lds, const uint8_t* blk, uint32_t voff) {
    const uint64_t on = (1ull << kRest) - 1ull;
    if constexpr (kFull == 0) {
      asm volatile(TKV_SET TKV_SOME(0)::"s"(lds), "v"(voff), "s"(blk), "s"(on) : "m0", "memory");
    } else if constexpr (kFull == 1) {
      asm volatile(TKV_SET TKV_DMA(0) TKV_SOME(1024)::"s"(lds), "v"(voff), "s"(blk), "s"(on) : "m0", "memory");
    } else if constexpr (kFull == 2 && kRest != 0) {
      asm volatile(TKV_SET TKV_DMA(0) TKV_DMA(1024) TKV_SOME(2048)::"s"(lds), "v"(voff), "s"(blk), "s"(on) : "m0", "memory");
    } else if constexpr (kFull == 2) {
      asm volatile(TKV_SET TKV_DMA(0) TKV_DMA(1024)::"s"(lds), "v"(voff), "s"(blk) : "m0", "memory");
    } else {
      static_assert(kFull != 3, "no format has such blocks");
      asm volatile(TKV_SET TKV_DMA(0) TKV_DMA(1024) TKV_DMA(2048) TKV_DMA(3072)::"s"(lds), "v"(voff), "s"(blk) : "m0", "memory");
      if constexpr (kRest != 0)   // beyond the reach of the offset
        asm volatile(TKV_SET TKV_SOME(0)::"s"(lds + 4096u), "v"(voff), "s"(blk + 4096), "s"(on) : "m0", "memory");
    }
  }
#undef TKV_SOME
#undef TKV_DMA
#undef TKV_SET
};
// LDS byte address of the dynamic LDS: what is written below by hand (rings, tickets, lists) and what goes through the array's name
// count from one place
__device__ __forceinline__ uint32_t lds_address(void* lds) { return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds; }
// a wave-uniform pointer that the compiler cannot prove to be one, into scalar registers
__device__ __forceinline__ const uint8_t* scalar_ptr(const uint8_t* p) {
  const uint64_t u = (uint64_t)(uintptr_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)u), hi = __builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
  return (const uint8_t*)(uintptr_t)((uint64_t)hi << 32 | lo);
}
template <int N>
__device__ __forceinline__ void wait_loads() {   // until at most N of the wave's vector-memory operations are outstanding
  static_assert(N >= 0 && N < 64, "six bits");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Ids of a pair of pages that stand side by side in the list
struct ListIds {
  int pid_a, pid_b;
  uint32_t live_a, live_b;
  int idx;   // STAT: twice the first one's position in the type's page list, plus one where there is a second
  // One store a pair, always, so that the waits of the ring can count it: two, which they did not count, made a wave wait for its next pairs'
  // loads: 200 x 1k..10k tokens, statistic included, 294 us, now 289, 32 x 2k..20k of 40 heads 140 and 136, 64 x 1k..10k at head_dim 64 70 and 68
  static constexpr int kStores = 1;
  __device__ __forceinline__ void keep(float* stat, int room, int lane, float ua, float ub) const {
    // rows (0, 1, 2, 3) of ua and ub: the larger of a0 and a1, b0 and b1, a2 and a3, b2 and b3, then of the halves: a, b, a, b
    auto r16 = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, ua), __builtin_bit_cast(uint32_t, ub), false, false);
    const uint32_t w = __builtin_bit_cast(uint32_t, fmaxf(__builtin_bit_cast(float, (uint32_t)r16[0]), __builtin_bit_cast(float, (uint32_t)r16[1])));
    auto r32 = __builtin_amdgcn_permlane32_swap(w, w, false, false);
    const float u = fmaxf(__builtin_bit_cast(float, (uint32_t)r32[0]), __builtin_bit_cast(float, (uint32_t)r32[1]));
    const int first = idx >> 1, pages = min((idx & 1) + 1, room - first);
    if (pages > 0) {
      // (all lanes are on, before and after; wait states as for the direct copies)
      float* const dst = (float*)scalar_ptr((const uint8_t*)(stat + (int64_t)first * kPage));
      asm volatile("s_mov_b64 exec, %3\n\ts_nop 4\n\tglobal_store_dword %0, %1, %2\n\ts_mov_b64 exec, -1"
                   ::"v"(4 * lane), "v"(u), "s"(dst), "s"((1ull << (kPage * pages)) - 1ull) : "memory");
    } else {
      wait_loads<0>();   // no room, no store: with nothing outstanding the next waits hold all the same
    }
  }
};

// The page pairs an item works on, as one wave sees them.  The item's share of the three page lists is cut into chunks of
// 2^shift consecutive pairs, type after type; chunk numbers come from the workgroup's ticket counter.  The ids and
// masks of the pair after the one just taken are on their way by scalar loads (no traffic in the vector-memory queue).
// Where an item has all the waves of a compute unit and kFinePages pages or more for each of them (head_dim 128, integer formats), a chunk is
// one pair: neighbouring waves then read neighbouring pages, and no wave is left with a whole chunk at the end.  Pairs by fours / by ones, us:
// 33 pages a wave: 16 x 8k tokens 40.1 / 39.5, 24 x 4k 34.9 / 32.8, 32 x ~2k of scrambled slots 46.5 / 44.9.  With fewer pages a wave's loads
// of its one to four chunks follow each other closer than draws do: 4 pages, 1 x 8k 18.7 / 20.9; 8, 1 x 32k 23.2 / 24.8, 8 x 4k 19.5 / 21.3; 16, 2 x 32k 28.5 / 29.3, 8 x 8k
// 26.6 / 27.4, 16 x 4k 27.0 / 28.0.  Where waves share out a unit among several items there is nobody to balance with (28 x 3.2k..32k, 40 heads, 88.2 / 90.8), with
// the statistic the draws' scalars are spilled (16 x 32k, 64 heads, 153 either way, 32 x 16k 150 / 154), and elsewhere a draw a pair costs more than it brings (256 x 1k..64k 837 us
// by fours, 856 by ones; head_dim 64, 128 x 4k..32k 268 and 272; the paper's formats no difference).
constexpr int kFinePages = 20;
constexpr int kChunkShift = 2;
constexpr int kTicketBytes = 64;   // a counter for each of up to sixteen items, behind the rings
typedef const int32_t __attribute__((address_space(4))) * ConstI32;   // read-only for the whole launch: scalar loads
typedef __attribute__((address_space(3))) int32_t* LdsCounter;

// a scalar that a load may still be bringing: waited for here and not before (what is computed from it would otherwise
// be moved up to the load, and the wait with it)
__device__ __forceinline__ int arrived(int x) {
  asm volatile("" : "+s"(x));
  return x;
}

// FINE: the chunk's size is chosen per launch, else it is 2^kChunkShift pairs (a constant: one scalar less in a loop that has few to spare)
template <bool FINE>
struct Stream {
  ConstI32 tab, msk;           // page list and masks of type 0; those of type k begin k * max_pages later
  LdsCounter ticket;
  int max_pages, lane;
  // the three types in the order they are walked: type, first pair, end page, chunks up to and including it (plain
  // members: an array indexed by a choice would not stay in scalar registers)
  int kind0, kind1, kind2, first0, first1, first2, end0, end1, end2, cum0, cum1, cum2;
  int fine;
  __device__ __forceinline__ int shift() const { return FINE ? fine : kChunkShift; }   // a chunk has 2^shift pairs
  int left, row, end;          // pairs of the current chunk after the next pair; k * max_pages and end page of its type
  int sec, pg;                 // the next pair: which of the three types (3: there is none), its first page,
  int more_pages;              // 1 where it has a second one, else 0,
  int pid_a, pid_b, msk_a, msk_b;   // ids and mask words of its pages (live bits in the low half), as the scalar loads return them

  static __device__ __forceinline__ int pick(int x, int a, int b, int c) { return x == 0 ? a : (x == 1 ? b : c); }
  // the share [j / n, (j + 1) / n) of a list of np pages: first pair, end page; its chunks
  __device__ __forceinline__ int share(int np, int j, int n, int& first, int& end) const {
    const int pairs = (np + 1) >> 1;
    first = portion(pairs, j, n);
    const int hi = portion(pairs, j + 1, n);
    end = 2 * hi < np ? 2 * hi : np;
    return (hi - first + (1 << shift()) - 1) >> shift();
  }
  // The next chunk's number, by one lane.  (In asm, with its wait: a branch on the lane would make the compiler restructure
  // every loop around it and keep their scalars in vector registers.)
  __device__ __forceinline__ int draw() const {
    int r;
    asm volatile("s_mov_b64 exec, 1\n\tds_add_rtn_u32 %0, %1, %2\n\ts_mov_b64 exec, -1\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(r) : "v"((uint32_t)(uintptr_t)ticket), "v"(1) : "memory");
    return uniform(r);
  }
  static __device__ __forceinline__ int at(ConstI32 list, uint32_t bytes) { return *(ConstI32)((const char __attribute__((address_space(4)))*)list + bytes); }
  // moves on by one pair.  (Sums and minima instead of conditions: a condition turned into a number takes a vector
  // instruction and drags what depends on it out of the scalar registers.)
  __device__ __forceinline__ void look() {
    if (left > 0) {
      --left;
      pg += 2;
    } else {
      const int c = draw();
      if (c >= cum2) {
        sec = 3;
        return;
      }
      if (c >= cum1) {
        sec = 2;
        end = end2;
        row = kind2 * max_pages;
        pg = 2 * (first2 + ((c - cum1) << shift()));
      } else if (c >= cum0) {
        sec = 1;
        end = end1;
        row = kind1 * max_pages;
        pg = 2 * (first1 + ((c - cum0) << shift()));
      } else {
        sec = 0;
        end = end0;
        row = kind0 * max_pages;
        pg = 2 * (first0 + (c << shift()));
      }
      left = min((end - pg - 1) >> 1, (1 << shift()) - 1);
    }
    more_pages = min(end - pg - 1, 1);
    const uint32_t a = 4u * (uint32_t)(row + pg), b = a + 4u * (uint32_t)more_pages;   // (bytes: 3 max_pages < 2^26)
    pid_a = at(tab, a);
    msk_a = at(msk, a);
    pid_b = at(tab, b);
    msk_b = at(msk, b);
  }
  // the pair at hand, if it is one of the x-th type walked (want): its ids and masks are waited for here and not before
  int want;
  typedef ListIds Ids;
  __device__ __forceinline__ bool next(ListIds& id) const {
    if (sec != want) return false;
    id.pid_a = arrived(pid_a);
    id.pid_b = arrived(pid_b);
    id.live_a = (uint32_t)arrived(msk_a) & 0xFFFFu;
    id.live_b = (uint32_t)(arrived(msk_b) & (0 - more_pages)) & 0xFFFFu;
    id.idx = 2 * pg + more_pages;
    return true;
  }
};

// All pairs that `q` hands out (next(): the pair at hand, false when there is none; look(): move on), through the wave's ring
// of RING bytes at LDS address `ring`.
template <int RING, class Runner, class Source>
__device__ __forceinline__ void stream_pairs(Runner& run, Source& q, const thinkv_view& v, int cls, int hkv, uint32_t ring) {
  using Dma = BlockDma<Runner::kBlockBytes>;
  constexpr int kPairBytes = 2 * Runner::kBlockBytes, kOps = 2 * Dma::kOps;
  constexpr int kSlots = RING / kPairBytes;
  typedef typename Source::Ids Ids;
  constexpr int kStores = Runner::kStat ? Ids::kStores : 0;
  static_assert(kSlots >= 1 && kSlots <= 32 && (kSlots - 1) * kOps + kSlots * kStores < 64, "the ring holds a pair, the waits six bits");
  const int lane = run.lane;
  const uint32_t voff = 16 * lane;
  const uint32_t page_bytes = __builtin_amdgcn_readfirstlane(v.cfg.n_kv_heads * Runner::kBlockBytes);
  const uint8_t* const base = scalar_ptr(v.arena[cls] + (int64_t)hkv * Runner::kBlockBytes);
  int f_live = 0, f_ia = 0, f_ib = 0;   // lane s: what slot s holds (live bits of both pages; STAT: their list positions)
  // asks for the next live pair in slot, moves on; false: there is none
  auto issue = [&](int slot) -> bool {
    Ids id;
    while (q.next(id)) {
      const bool on = (id.live_a | id.live_b) != 0;
      if (on) {
        const uint32_t at = uniform(ring + slot * kPairBytes);
        Dma::issue(at, scalar_ptr(base + (uint64_t)(uint32_t)id.pid_a * page_bytes), voff);
        Dma::issue(at + Runner::kBlockBytes, scalar_ptr(base + (uint64_t)(uint32_t)id.pid_b * page_bytes), voff);
        const bool mine = lane == slot;
        f_live = mine ? (int)(id.live_a | id.live_b << 16) : f_live;
        if constexpr (kStores) {
          f_ia = mine ? id.idx : f_ia;
        } else if constexpr (Runner::kStat) {
          f_ia = mine ? id.idx_a : f_ia;
          f_ib = mine ? id.idx_b : f_ib;
        }
      }
      q.look();
      if (on) return true;
    }
    return false;
  };
  int flying = 0;
#pragma nounroll
  while (flying < kSlots && issue(flying)) ++flying;
  int slot = 0, first = kSlots;   // (pairs to go until there has been a store for each of the ring's slots)
#pragma nounroll
  while (flying > 0) {
    // The oldest pair has landed when only the others' loads are left, and what was stored since it was asked for: operations of one
    // kind or the other are reported done in their order (with fewer pairs in flight all are waited for: the end is near).
    if (flying != kSlots) {
      wait_loads<0>();
    } else if (kStores == 0 || first > 0) {
      wait_loads<(kSlots - 1) * kOps>();
      if constexpr (kStores) --first;
    } else {
      wait_loads<(kSlots - 1) * kOps + kSlots * kStores>();
    }
    const LdsPtr blk_a = (LdsPtr)(uintptr_t)(ring + slot * kPairBytes), blk_b = blk_a + Runner::kBlockBytes;
    typename Runner::Pair r;
    run.load_k(r, blk_a, blk_b);
    const uint32_t live = (uint32_t)__builtin_amdgcn_readlane(f_live, slot);
    Ids cur;
    cur.live_a = live & 0xFFFFu;
    cur.live_b = live >> 16;
    if constexpr (kStores) {
      cur.idx = __builtin_amdgcn_readlane(f_ia, slot);
    } else if constexpr (Runner::kStat) {
      cur.idx_a = __builtin_amdgcn_readlane(f_ia, slot);
      cur.idx_b = __builtin_amdgcn_readlane(f_ib, slot);
    }
    run.load_v(r, blk_a, blk_b);
    wait_lds();   // the slot has been read: it can be filled again
    if (!issue(slot)) --flying;
    run.scores(r, cur);
    run.values(r);
    slot = slot + 1 == kSlots ? 0 : slot + 1;
  }
}

// Sliding-window layers: pages of one type with a visible slot, as the workgroup's scan left them in LDS; a wave takes
// the pairs i, i + step, ... before end.
typedef __attribute__((address_space(3))) const int32_t* LdsWords;
typedef __attribute__((address_space(3))) const uint16_t* LdsHalves;
template <bool STAT>
struct VisiblePages {
  LdsWords pid, idx;
  LdsHalves msk;
  int n, i, end, step;
  typedef PairIds Ids;
  __device__ __forceinline__ bool next(PairIds& id) const {
    if (i >= end) return false;
    const int a = 2 * i, b = min(a + 1, n - 1);
    const int two = b - a;
    id.pid_a = uniform(pid[a]);
    id.pid_b = uniform(pid[b]);
    id.live_a = (uint32_t)uniform(msk[a]);
    id.live_b = (uint32_t)(uniform(msk[b]) & (0 - two));
    if constexpr (STAT) {
      id.idx_a = uniform(idx[a]);
      id.idx_b = two ? uniform(idx[b]) : -1;
    }
    return true;
  }
  __device__ __forceinline__ void look() { i += step; }
};

// Sliding-window layers, integer formats.  Where slots are reused in place, the window's tokens lie a few to a page, all over the lists, and
// a page costs the same arithmetic however few of its slots are visible.  So the scan lists quads of slots (4 q .. 4 q + 3 of a page: a
// lane of the value product holds one) with a visible slot, and a pair's two "pages" are put together in LDS from any eight of them: a
// block's regions are made of 16-byte units of one quad each, and a direct load to LDS takes an address from every lane.
template <bool STAT>
struct SlotQuads {
  LdsWords pid, idx;   // page << 2 | quad (a page number has far fewer than thirty bits: pages of 768 bytes and more); list positions
  LdsHalves msk;       // visible slots of the quad
  int n, i, end, step;
};

// Unit u (16 bytes) of a block, u = 64 op + lane: the quad of the "page" it belongs to, and where it lies in the block of the page that the
// quad comes from: at + quad there << shift.  As quad | shift << 2 | at << AT; at is a multiple of 16, so with AT 2 that is fifteen bits.
template <int D, int BITS, int AT>
__device__ __forceinline__ int quad_unit(int u) {
  constexpr int CB = block_geom(BITS, D).chunk_bytes, kCodes = 4 * CB, kMeta = D / 32 * 4;   // units of a code and of a meta region
  constexpr int kLog = (BITS == 2 ? 1 : (BITS == 4 ? 2 : 3)) + (D == 128 ? 2 : 1);           // of CB
  const int r = u < kCodes + kMeta ? u : u - kCodes - kMeta;   // inside the half of keys or of values
  int quad, shift;
  if (r >= kCodes) {          // unit 4 group + quad
    quad = (r - kCodes) & 3;
    shift = 4;
  } else if (u < kCodes) {    // chunk 16 j + slot
    quad = r >> (kLog - 2) & 3;
    shift = kLog + 2;
  } else {                    // chunk 16 quad + c
    quad = r >> kLog;
    shift = kLog + 4;
  }
  return quad | shift << 2 | (16 * u - (quad << shift)) << AT;
}

// The pairs of quads i .. end - 1, through the wave's ring like stream_pairs
template <int RING, class Runner, class Quads>
__device__ __forceinline__ void quad_pairs(Runner& run, Quads& q, const thinkv_view& v, int cls, int hkv, uint32_t ring) {
  constexpr int kUnits = Runner::kBlockBytes / 16, kPageOps = (kUnits + 63) / 64, kRest = kUnits % 64, kOps = 2 * kPageOps;
  constexpr int kPairBytes = 2 * Runner::kBlockBytes;
  constexpr int kSlots = RING / kPairBytes;
  static_assert(kSlots >= 1 && (kSlots - 1) * kOps < 64 && Runner::kBlockBytes % 16 == 0, "the ring holds a pair, the waits six bits");
  const int lane = run.lane;
  const uint32_t page_bytes = __builtin_amdgcn_readfirstlane(v.cfg.n_kv_heads * Runner::kBlockBytes);
  const uint8_t* const base = scalar_ptr(v.arena[cls] + (int64_t)hkv * Runner::kBlockBytes);
  constexpr int kUnitsOf = Runner::kTight ? 2 : 1, kAt = Runner::kTight ? 2 : 8;   // units to a register
  int unit[(kPageOps + kUnitsOf - 1) / kUnitsOf] = {};
  const int here = fresh_lane();   // (not for all widths at once before the loops around)
#pragma unroll
  for (int o = 0; o < kPageOps; ++o) unit[o / kUnitsOf] |= quad_unit<Runner::kD, Runner::kBits, kAt>(min(64 * o + here, kUnits - 1)) << (o % kUnitsOf * 16);
  int f_live = 0, f_first = 0;   // lane s: visible slots and first quad of the pair in slot s
  // asks for the next pair in slot, moves on; false: there is none
  auto issue = [&](int slot) -> bool {
    if (q.i >= q.end) return false;
    const int first = 8 * q.i;
    const int own = min(first + (lane >> 2 & 7), q.n - 1);
    const uint32_t live = (uint32_t)__ballot((q.msk[own] >> (lane & 3) & 1) != 0 && first + (lane >> 2) < q.n && lane < 32);
#pragma unroll(kPageOps <= 2 ? 2 : 1)
    for (int page = 0; page < 2; ++page) {
      int u[kPageOps], from[kPageOps];
#pragma unroll
      for (int o = 0; o < kPageOps; ++o) {   // (behind the last quad, that one once more: nothing of it is visible there)
        u[o] = unit[o / kUnitsOf];
        asm volatile("" : "+v"(u[o]));       // (what follows from it is worked out each time: there are no registers to keep it)
        u[o] = kUnitsOf > 1 ? u[o] >> (o % kUnitsOf * 16) & 0x7FFF : u[o];
        from[o] = q.pid[min(first + 4 * page + (u[o] & 3), q.n - 1)];
      }
#pragma unroll
      for (int o = 0; o < kPageOps; ++o) {
        const uint8_t* src = base + (uint64_t)((uint32_t)from[o] >> 2) * page_bytes + (uint32_t)((Runner::kTight ? u[o] >> 6 << 4 : u[o] >> 8) + ((from[o] & 3) << (u[o] >> 2 & 15)));
        const uint32_t lds = uniform(ring + slot * kPairBytes + page * Runner::kBlockBytes + 1024 * o);
        if (kRest != 0 && o == kPageOps - 1)
          asm volatile("s_mov_b32 m0, %0\n\ts_mov_b64 exec, %2\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, off nt\n\ts_mov_b64 exec, -1"
                       ::"s"(lds), "v"(src), "s"((1ull << kRest) - 1ull) : "m0", "memory");
        else
          asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, off nt" ::"s"(lds), "v"(src) : "m0", "memory");
      }
    }
    const bool mine = lane == slot;
    f_live = mine ? (int)live : f_live;
    if constexpr (Runner::kStat) f_first = mine ? first : f_first;
    q.i += q.step;
    return true;
  };
  int flying = 0;
#pragma nounroll
  while (flying < kSlots && issue(flying)) ++flying;
  int slot = 0;
#pragma nounroll
  while (flying > 0) {
    if (flying == kSlots) wait_loads<(kSlots - 1) * kOps>();
    else wait_loads<0>();
    const LdsPtr blk_a = (LdsPtr)(uintptr_t)(ring + slot * kPairBytes), blk_b = blk_a + Runner::kBlockBytes;
    typename Runner::Pair r;
    run.load_k(r, blk_a, blk_b);
    const uint32_t live = (uint32_t)__builtin_amdgcn_readlane(f_live, slot);
    QuadIds cur;
    cur.live_a = live & 0xFFFFu;
    cur.live_b = live >> 16;
    if constexpr (Runner::kStat) {
      const int first = __builtin_amdgcn_readlane(f_first, slot) + (lane >> 2 & 3);
      auto place = [&](int e) { return e < q.n ? q.idx[e] * kPage + 4 * (q.pid[e] & 3) + (lane & 3) : -1; };
      cur.at_a = place(first);
      cur.at_b = place(first + 4);
    }
    run.load_v(r, blk_a, blk_b);
    wait_lds();   // the slot has been read: it can be filled again
    if (!issue(slot)) --flying;
    run.scores(r, cur);
    run.values(r);
    slot = slot + 1 == kSlots ? 0 : slot + 1;
  }
}

// What a lane keeps of the query for the whole item: per column set the eight binary16 values of
// (its head, its slice's group, channels 8qd .. 8qd+7) and, for the four rows of its quad, the sum of the 32 values
// of (row's head, row's slice's group).
template <int NSET>
struct QRegs {
  H8 q[NSET];
  float sum[NSET][4];
};

typedef __attribute__((address_space(3))) float* LdsFloats;
typedef __attribute__((address_space(3))) float4v* LdsFloat4;

// What the two runners (integer formats, the paper's formats) share: the softmax over the scores of a pair.
// LDS: the weights of a pair change layout through LDS (exchange_bytes).
template <int D, int GP, int NSET, bool STAT, bool LDS>
struct Softmax {
  static constexpr int NM = D / 16, NS = GP / 4;
  using State = WaveState<D, GP, NSET>;
  State& st;
  int lane;
  float kappa;       // MFMA score units -> log2 domain (with softmax_scale)
  float lift, slack; // weights are 2^(score - m + lift); the reference m is at most slack below the largest score
  // While a type is walked, per head: m - lift (0 - lift before the first live token), and the score, in MFMA units, above which m
  // moves (-inf before the first live token).  m and lift are whole numbers, so that all of this is exact.
  float mref[NS], top[NS];
  float sel[NS];     // B operands of the layout change: 1 where the column's head is the row's
  float* stat;       // STAT: pooled scores of this type's page list, 16 per page
  int stat_room;     // STAT: pages of this list the buffer has room for (the host's bound on the context)
  int G;
  LdsFloats put, get;   // LDS: where this lane leaves its weights, and finds those of its column and tokens
  __device__ __forceinline__ Softmax(State& st_, int lane_, int G_, float* stat_, int room, uint32_t xch) : st(st_), lane(lane_), stat(stat_), stat_room(room), G(G_) {
    if constexpr (LDS) {
      // rows of sixteen tokens: four of the row quads' first heads, then (GP = 8) four of their second
      const int h = lane & (GP - 1), row = GP == 4 ? h : 4 * (h & 1) + (h >> 2) + (h & 2);   // (head_of)
      put = (LdsFloats)(uintptr_t)(xch + 4 * lane);
      get = (LdsFloats)(uintptr_t)(xch + 64 * row + 16 * (lane >> 4));
    }
#pragma unroll
    for (int i = 0; i < NS; ++i) sel[i] = head_of<GP>(lane >> 4, i) == (lane & (GP - 1)) ? 1.0f : 0.0f;
  }
  __device__ __forceinline__ void enter(float lift_, float slack_) {
    lift = lift_;
    slack = slack_;
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      mref[i] = (st.m[i] == -INFINITY ? 0.f : st.m[i]) - lift;
      top[i] = (st.m[i] + slack) / kappa;
    }
  }
  // the weights from here on without the lift
  __device__ __forceinline__ void drop_lift() {
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      mref[i] += lift;
      top[i] -= slack / kappa;
    }
    lift = slack = 0.f;
  }
  __device__ __forceinline__ void leave() {
#pragma unroll
    for (int i = 0; i < NS; ++i) st.m[i] = top[i] == -INFINITY ? -INFINITY : mref[i] + lift;
  }
  // sa, sb: scores of the lane's token in pages a and b (NS heads each), in MFMA units.  Masks them and leaves the pooled scores.
  template <class Ids>
  __device__ __forceinline__ void mask(float* sa, float* sb, const Ids& id) {
    if ((id.live_a & id.live_b) != 0xFFFFu) {
      // dead slots: score -inf, hence p = 0.  Their scales and zero-points are finite (stale, or zero in a slot
      // never written: arenas start zero-filled), so they drop out of every sum.
      const bool la = __builtin_amdgcn_inverse_ballot_w64(id.live_a * 0x0001000100010001ull);
      const bool lb = __builtin_amdgcn_inverse_ballot_w64(id.live_b * 0x0001000100010001ull);
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        sa[i] = la ? sa[i] : -INFINITY;
        sb[i] = lb ? sb[i] : -INFINITY;
      }
    }
    if constexpr (STAT) {
      // pooled scores: maximum over the heads of the group, i.e. over the lane's heads here, then the four lanes of a token
      auto pooled = [&](const float* sc) {
        float u = -INFINITY;
#pragma unroll
        for (int i = 0; i < NS; ++i) u = head_of<GP>(lane >> 4, i) < G ? fmaxf(u, sc[i] * kappa) : u;
        return u;
      };
      id.keep(stat, stat_room, lane, pooled(sa), pooled(sb));
    }
  }
  // Online softmax: the weights are 2^(score - m) with m a reference that is at most `slack` below the maximum seen.  It
  // only moves when a score exceeds it by more, to the next whole number above the maximum: with eight heads a new maximum by any amount turns up
  // in most pairs of a few thousand tokens (and moving m costs as much as a quarter of the pair), one by a factor of 2^slack hardly ever.
  // now: it moves if any score is above it.
  __device__ __forceinline__ void reference(const float* sa, const float* sb, bool now) {
    float mx[NS];
    bool above = false;
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      mx[i] = largest(sa[i], sb[i]);
      above = above || mx[i] > (now ? top[i] - slack / kappa : top[i]);
    }
    if (__any(above)) {
      float corr[NS];
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        const bool seen = top[i] > -INFINITY;
        const float m_old = mref[i] + lift, m_new = fmaxf(seen ? m_old : -INFINITY, ceilf(row_max(mx[i]) * kappa));
        const float m_sub = m_new == -INFINITY ? 0.f : m_new;
        corr[i] = seen ? __builtin_amdgcn_exp2f(m_old - m_sub) : 0.f;
        st.l[i] *= corr[i];
        mref[i] = m_sub - lift;
        top[i] = (m_new + slack) / kappa;
      }
      const float cc = to_column<GP>(corr, lane);
#pragma unroll
      for (int mb = 0; mb < NM; ++mb) st.o[mb] *= cc;
#pragma unroll
      for (int set = 0; set < NSET; ++set) st.oz[set] *= cc;
    }
  }
  // the weights 2^(score - m + lift): ea, eb of the lane's token (score layout), pa, pb of the lane's four tokens (column layout).
  // The layout change by a matrix product takes 32 cycles of the matrix core for four heads and a page, the one through
  // LDS two short stores and one read for eight.  It is used where instructions and not the memory bound the launch: at head_dim
  // 64 with more than four heads, 64 x 16k tokens 156 -> 141 us, 128 x 4k..32k 287 -> 267; the paper's formats at head_dim 128, 8 x 8k
  // 35.6 -> 33.7, 16 x 16k of 4-bit types 74.9 -> 72.0, long contexts alike.  The integer formats at 128, and head_dim 64 with up
  // to four heads: no difference.  (The paper's formats at 64 leave no room for it in LDS.)
  __device__ __forceinline__ void weights(const float* sa, const float* sb, float* ea, float* eb, float* pa, float* pb) const {
    float4v ta = {0.f, 0.f, 0.f, 0.f}, tb = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      ea[i] = __builtin_amdgcn_exp2f(fmaf(sa[i], kappa, -mref[i]));
      eb[i] = __builtin_amdgcn_exp2f(fmaf(sb[i], kappa, -mref[i]));
      if constexpr (LDS) {
        put[64 * i] = ea[i];
        put[64 * (NS + i)] = eb[i];
      } else {
        // (the product adds four heads, and 0 times what is not a number is not one: such a weight goes in as 0, and spoils
        // its own head through the denominator, which adds ea and eb as they are.  Weights are never infinite.)
        ta = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_amdgcn_fmed3f(ea[i], 0.f, INFINITY), sel[i], ta, 0, 0, 0);
        tb = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_amdgcn_fmed3f(eb[i], 0.f, INFINITY), sel[i], tb, 0, 0, 0);
      }
    }
    if constexpr (LDS) {   // (a wave's LDS operations happen in order)
      ta = *(LdsFloat4)get;
      tb = *(LdsFloat4)(get + 64 * NS);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      pa[r] = ta[r];
      pb[r] = tb[r];
    }
  }
  __device__ __forceinline__ void add(const float* ea, const float* eb) {
#pragma unroll
    for (int i = 0; i < NS; ++i) st.l[i] += ea[i] + eb[i];
  }
  __device__ __forceinline__ void scale_sums(float f) {
#pragma unroll
    for (int i = 0; i < NS; ++i) st.l[i] *= f;
#pragma unroll
    for (int set = 0; set < NSET; ++set) st.oz[set] *= f;
  }
};

// The pages of one type, as one wave walks them.
// STAT: besides attending, leave the group-pooled score of every visited slot (the maximum over
// the query heads of the group of the scaled score, log2 domain; -inf for a dead or invisible
// slot) in a[.].stat, for the attention-sparsity statistic.
template <int D, int BITS, int GP, bool STAT>
struct ClassRunner {
  using CL = Cols<D, GP>;
  static constexpr int kD = D, kBits = BITS, kBlockBytes = block_geom(BITS, D).block_bytes;
  static constexpr bool kStat = STAT, kFp = false, kTight = D == 128 && GP == 8;
  static constexpr int NG = D / 32, NM = D / 16, CS = CL::CS, NSET = CL::NSET, NS = GP / 4;
  using F = Fld<BITS>;
  using Pair = PairRegs<D, BITS, NSET>;
  const int lane;
  WaveState<D, GP, NSET>& st;
  Softmax<D, GP, NSET, STAT, exchange_bytes(D, GP, false) != 0> sm;
  int k_off[NSET], v_off[NSET];  // byte offset, inside a meta region, of this lane's scale (K) and unit (V) per column set
  H8 bq[NG];           // A operands of the score MFMAs: q of group g in slice g % CS, zeros elsewhere
  float qs[NSET][4];   // 2^(OMIN-24) * sum_{i in group} q_i of the four rows of this lane's quad
  int lifted;          // the weights of this type's pages are 2^kLift times the softmax weights (0 after a scale too large for it)
  float neg1;          // -1, kept opaque so that x - (float)h stays one fused mixed-precision instruction

  // qr: this lane's query slice per column set (binary16, channels 32g + 8qd + e of its head and slice group) and the
  // group sums, as the kernel read them once per item
  __device__ __forceinline__ ClassRunner(WaveState<D, GP, NSET>& st_, const thinkv_config& c, const DecodeArgs& a, int G, const QRegs<NSET>& qr, float* stat_, int stat_room_, uint32_t xch)
      : lane(threadIdx.x & 63), st(st_), sm(st_, threadIdx.x & 63, G, stat_, stat_room_, xch) {
    const int qd = lane >> 4, n = lane & 15;
    const int gl = n / GP, head = n % GP;
    const bool used = gl < CS && head < G;
    const int glc = gl < CS ? gl : CS - 1;   // unused slices read slice CS-1's unit (finite, multiplied by zeros)
    const int gk = GP == 4 ? qd : qd >> 1, gkc = gk < CS ? gk : CS - 1;   // slice of the rows of this lane's quad
    sm.kappa = (float)(1 << (24 - F::OMIN)) * a.scale_log2e;
    enter();
    neg1 = -1.0f;
    asm volatile("" : "+v"(neg1));
#pragma unroll
    for (int s = 0; s < NSET; ++s) {
      k_off[s] = ((s * CS + gkc) * 4 + (n >> 2)) * 16 + (n & 3) * 2;
      v_off[s] = ((s * CS + glc) * 4 + qd) * 16;
#pragma unroll
      for (int r = 0; r < 4; ++r) qs[s][r] = qr.sum[s][r] * (1.0f / (float)(1 << (24 - F::OMIN)));
    }
    // the query slice is scaled down by the residual power of two the codes of those fields carry (exact:
    // power-of-two scaling of binary16 values), then dealt to the group's operand; the operands of
    // the other groups are zero in this lane
    H8 mine[NSET];
#pragma unroll
    for (int s = 0; s < NSET; ++s) {
      mine[s] = qr.q[s];
#pragma unroll
      for (int e = 0; e < 8; ++e) mine[s].h[e] *= (_Float16)(1.0f / (float)(1 << F::rel_of(e >> 1)));   // rel_of depends on the field's parity only
    }
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const bool on = used && (g % CS) == gl;
#pragma unroll
      for (int w = 0; w < 4; ++w) bq[g].u[w] = on ? mine[g / CS].u[w] : 0u;
    }
  }

  // The second operand of the value products, p * s_V, is a binary16 pair: 22 significant bits, but nothing
  // below 2^-24.  With the weights taken relative to the running maximum (p <= 1), a head whose attention is
  // peaked would have most of its tokens down where binary16 has few bits left or none.  So the weights of a
  // type's pages are lifted by 2^kLift -- the softmax reference is lowered, which costs nothing: the
  // denominator, the zero-point sums and the tiles carry the same factor until the type is left -- as far as
  // scales of ordinary size allow (a scale of 2^(16 - kLift), i.e. a group range of about a thousand, would take
  // the largest product out of binary16; every pair is checked, and such a pair ends the lift for the rest of
  // the type).
  static constexpr int kLift = BITS == 8 ? 14 : (BITS == 4 ? 10 : 8);
  static constexpr float kSlack = 3.0f;
  // the tiles are in the units of the type (its codes carry a power of two that depends on the bit width) and
  // lifted while its pages are walked, in absolute units in between
  __device__ static constexpr float tile_unit(int mb) { return (float)(1 << (BITS == 8 ? 0 : F::OMIN + F::rel_of(mb))); }
  __device__ __forceinline__ void enter() {
    const float up = (float)(1 << kLift);
    lifted = 1;
    sm.enter((float)kLift, kSlack);
    sm.scale_sums(up);
#pragma unroll
    for (int mb = 0; mb < NM; ++mb) st.o[mb] *= up * tile_unit(mb);
  }
  __device__ __forceinline__ void drop_lift() {
    const float down = 1.0f / (float)(1 << kLift);
    sm.scale_sums(down);
#pragma unroll
    for (int mb = 0; mb < NM; ++mb) st.o[mb] *= down;
    lifted = 0;
    sm.drop_lift();
  }
  __device__ __forceinline__ void leave() {
    if (lifted) drop_lift();
    sm.leave();
#pragma unroll
    for (int mb = 0; mb < NM; ++mb) st.o[mb] *= 1.0f / tile_unit(mb);
  }

  template <class P>
  __device__ __forceinline__ void load_k(Pair& r, P blk_a, P blk_b) const {
    load_keys<D, BITS, NSET>(r.a, blk_a, lane, k_off);
    load_keys<D, BITS, NSET>(r.b, blk_b, lane, k_off);
  }
  template <class P>
  __device__ __forceinline__ void load_v(Pair& r, P blk_a, P blk_b) const {
    load_values<D, BITS, NSET>(r.a, blk_a, lane, v_off);
    load_values<D, BITS, NSET>(r.b, blk_b, lane, v_off);
  }

  // scores of one page for this lane's token and heads, in MFMA units (times kappa = log2 domain)
  __device__ __forceinline__ void page_scores(const PageRegs<D, BITS, NSET>& r, float* s) const {
    const float4v zero = {0.f, 0.f, 0.f, 0.f};
    float4v c[NSET];
#pragma unroll
    for (int set = 0; set < NSET; ++set) {
#pragma unroll
      for (int gl = 0; gl < CS; ++gl) {
        const int g = set * CS + gl;
        H8 ka;
#pragma unroll
        for (int vv = 0; vv < 4; ++vv) ka.u[vv] = F::get(r.kw, 4 * g + vv);
        c[set] = __builtin_amdgcn_mfma_f32_16x16x32_f16(bq[g].h, ka.h, gl == 0 ? zero : c[set], 0, 0, 0);
      }
    }
    float x[4];
#pragma unroll
    for (int set = 0; set < NSET; ++set) {
      const float sc = (float)__builtin_bit_cast(_Float16, r.ks[set]), zp = (float)__builtin_bit_cast(_Float16, r.kz[set]);
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const float t = fmaf(sc, c[set][r4], fmaf(zp, qs[set][r4], 0.0f));
        x[r4] = set == 0 ? t : x[r4] + t;
      }
    }
    add_groups<GP>(x, s);
  }

  float sa[NS], sb[NS];   // scores of the pair at hand
  template <class Ids>
  __device__ __forceinline__ void scores(const Pair& r, const Ids& id) {
    page_scores(r.a, sa);
    page_scores(r.b, sb);
    sm.mask(sa, sb, id);
    sm.reference(sa, sb, false);   // (without the lift there is no slack: a weight above one could take the largest scales out of binary16)
  }
  // ---------------- values, per column set: B = two-term split of p * s_V, A = V codes
  __device__ __forceinline__ void values(const Pair& r) {
    float ea[NS], eb[NS], pa[4], pb[4], xa[NSET][4], xb[NSET][4];
    for (int again = 0;; ++again) {
      sm.weights(sa, sb, ea, eb, pa, pb);
      float big = 0.f;
#pragma unroll
      for (int set = 0; set < NSET; ++set) {
#define TKV_X(R)                                                               \
  {                                                                            \
    xa[set][R] = fmaf(half_of<R>(r.a.vm[set].x, r.a.vm[set].y), pa[R], 0.0f);  \
    xb[set][R] = fmaf(half_of<R>(r.b.vm[set].x, r.b.vm[set].y), pb[R], 0.0f);  \
  }
        TKV_X(0) TKV_X(1) TKV_X(2) TKV_X(3)
#undef TKV_X
        big = largest(largest(xa[set][0], xa[set][1], xa[set][2]), largest(xa[set][3], xb[set][0], xb[set][1]), largest(xb[set][2], xb[set][3], big));
      }
      if (!lifted || !__any(big > 6.0e4f)) break;
      // A lifted product would leave binary16.  First the reference moves up to the maximum; scales that are too large
      // even then are far outside what a cache holds in practice, and the rest of this type's pages is worked on without
      // the lift.
      if (again == 0) sm.reference(sa, sb, true);
      else drop_lift();
    }
    sm.add(ea, eb);
#pragma unroll
    for (int set = 0; set < NSET; ++set) {
      float z = st.oz[set];
#define TKV_PV(R)                                                     \
  {                                                                   \
    z = fmaf(half_of<R>(r.a.vm[set].z, r.a.vm[set].w), pa[R], z);           \
    z = fmaf(half_of<R>(r.b.vm[set].z, r.b.vm[set].w), pb[R], z);           \
  }
      TKV_PV(0) TKV_PV(1) TKV_PV(2) TKV_PV(3)
#undef TKV_PV
      st.oz[set] = z;
      // k-slots 8qd+e: e<4 page a slots 4qd+e, e>=4 page b
      H8 hi, lo;
      hi.u[0] = pack_rne(xa[set][0], xa[set][1]);
      hi.u[1] = pack_rne(xa[set][2], xa[set][3]);
      hi.u[2] = pack_rne(xb[set][0], xb[set][1]);
      hi.u[3] = pack_rne(xb[set][2], xb[set][3]);
      lo.u[0] = pack_rne(fmaf(neg1, half_lo(hi.u[0]), xa[set][0]), fmaf(neg1, half_hi(hi.u[0]), xa[set][1]));
      lo.u[1] = pack_rne(fmaf(neg1, half_lo(hi.u[1]), xa[set][2]), fmaf(neg1, half_hi(hi.u[1]), xa[set][3]));
      lo.u[2] = pack_rne(fmaf(neg1, half_lo(hi.u[2]), xb[set][0]), fmaf(neg1, half_hi(hi.u[2]), xb[set][1]));
      lo.u[3] = pack_rne(fmaf(neg1, half_lo(hi.u[3]), xb[set][2]), fmaf(neg1, half_hi(hi.u[3]), xb[set][3]));
#pragma unroll
      for (int mm = 0; mm < 2 * CS; ++mm) {
        const int mb = 2 * CS * set + mm;
        H8 va;
        // field f = u*NM + mb holds slots (2u, 2u+1) of the lane's slot quad
        va.u[0] = F::get(r.a.vw, 0 * NM + mb);
        va.u[1] = F::get(r.a.vw, 1 * NM + mb);
        va.u[2] = F::get(r.b.vw, 0 * NM + mb);
        va.u[3] = F::get(r.b.vw, 1 * NM + mb);
        st.o[mb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(va.h, hi.h, st.o[mb], 0, 0, 0);
        st.o[mb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(va.h, lo.h, st.o[mb], 0, 0, 0);
      }
    }
  }

};

}  // namespace thinkv
#include "decode_mfma_fp.h"
namespace thinkv {

// What both kernels hold of the query: lane (slice gl, head, row quad qd) reads, per column set, the eight values of
// channels 32g + 8qd .. of its head (g = the set's group of its slice) and rounds them to binary16.
template <int D, int GP, bool FP>
struct Query {
  static constexpr int CS = FP ? ColsFp<D, GP>::CS : Cols<D, GP>::CS, NSET = FP ? ColsFp<D, GP>::NSET : Cols<D, GP>::NSET;
  QRegs<FP ? 1 : NSET> qr;
  QRegsFp<FP ? NSET : 1> qf;
  uint4 raw[NSET];
  static __device__ __forceinline__ H8 halves(int dtype, const uint4& raw) {
    H8 t;
    if (dtype == THINKV_F16) {
      t.u[0] = raw.x; t.u[1] = raw.y; t.u[2] = raw.z; t.u[3] = raw.w;
    } else {
      const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t u = (e & 1) ? (w[e >> 1] & 0xFFFF0000u) : (w[e >> 1] << 16);
        t.h[e] = (_Float16)__builtin_bit_cast(float, u);
      }
    }
    return t;
  }
  // Asks for the elements; at: first element of the group's heads.  They are looked at (finish) when the page lists have been asked
  // for as well, so that the two wait together.
  __device__ __forceinline__ void load(const DecodeArgs& a, int64_t at, int G, int lane) {
    const int qd = lane >> 4, n = lane & 15, gl = n / GP, head = n % GP;
    const int glc = gl < CS ? gl : CS - 1;
    at += (int64_t)(gl < CS && head < G ? head : 0) * D + 8 * qd;
#pragma unroll
    for (int s = 0; s < NSET; ++s) raw[s] = *(const uint4*)((const uint16_t*)a.q + at + 32 * (FP ? (s * CS + glc) >> 1 : s * CS + glc));
  }
  __device__ __forceinline__ void finish(const DecodeArgs& a, int G, int lane) {
    const int qd = lane >> 4, n = lane & 15, gl = n / GP, head = n % GP;
    const bool used = gl < CS && head < G;
    const int glc = gl < CS ? gl : CS - 1;
#pragma unroll
    for (int s = 0; s < NSET; ++s) {
      if constexpr (FP) {
        // the paper's formats: a slice carries a group of 16 channels; the lane holds the eight values of channels
        // 32 G + 8 qd .. of its head where those lie in its slice's group (qd / 2 = parity of the group), zeros otherwise
        const int g16 = s * CS + glc;
        const bool mine = used && (g16 & 1) == (qd >> 1);
        const H8 t = decltype(qf)::pairs(halves(a.q_dtype, raw[s]));
#pragma unroll
        for (int w4 = 0; w4 < 4; ++w4) qf.q[s].u[w4] = mine ? t.u[w4] : 0u;
      } else {
        // ... and the sum of the group's 32 values: the four row quads complete it
        qr.q[s] = halves(a.q_dtype, raw[s]);
        float sum = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) sum += (float)qr.q[s].h[e];
        sum += __shfl_xor(sum, 16, 64);
        sum += __shfl_xor(sum, 32, 64);
        sum = used ? sum : 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) qr.sum[s][r] = __shfl(sum, 4 * qd + r, 64);   // from the lane whose column is the row
      }
    }
  }
};

// A wave's partial (or, with one item per head, result) from its registers.  The lanes of a row quad (sixteen tokens)
// each hold a share of the denominators of the quad's heads, the four lanes of a column a share of the zero-point sums;
// the tile of channel block mb is valid in the slice of its group, where lane (head, qd) holds channels 16 mb + 4 qd .. + 3.
template <int D, int GP, bool FP>
struct Partial {
  static constexpr int NM = D / 16, NS = GP / 4, CS = Query<D, GP, FP>::CS, NSET = Query<D, GP, FP>::NSET;
  static constexpr int GB = FP ? 1 : 2;   // 16-channel blocks per quantisation group
  float l, m, zsum[NSET];                 // of the lane's column
  __device__ __forceinline__ Partial(const WaveState<D, GP, NSET>& st, int lane) {
    float ls[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      ls[i] = st.l[i];
#pragma unroll
      for (int d = 8; d >= 1; d >>= 1) ls[i] += lane_of(ls[i], lane ^ d);
    }
    l = to_column<GP>(ls, lane);
    m = to_column<GP>(st.m, lane);
#pragma unroll
    for (int set = 0; set < NSET; ++set) {
      float z = FP ? 0.f : st.oz[set];   // the paper's formats have no zero-points
      if constexpr (!FP) {
        z += lane_of(z, lane ^ 16);
        z += lane_of(z, lane ^ 32);
      }
      zsum[set] = z;
    }
  }
  // f(channel, four values) for the lane's share of its head's accumulator (lanes of a used head only)
  template <class F>
  __device__ __forceinline__ void each(const WaveState<D, GP, NSET>& st, int lane, F f) const {
    const int qd = lane >> 4, gl = (lane & 15) / GP;
#pragma unroll
    for (int mb = 0; mb < NM; ++mb) {
      const int g = mb / GB, set = g / CS;
      if (gl == g % CS)
        f(16 * mb + 4 * qd, make_float4(st.o[mb][0] * 16777216.f + zsum[set], st.o[mb][1] * 16777216.f + zsum[set],
                                        st.o[mb][2] * 16777216.f + zsum[set], st.o[mb][3] * 16777216.f + zsum[set]));
    }
  }
};

template <int D, int GP, int NSET>
__device__ __forceinline__ void clear(WaveState<D, GP, NSET>& st) {
#pragma unroll
  for (int mb = 0; mb < D / 16; ++mb) st.o[mb] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int set = 0; set < NSET; ++set) st.oz[set] = 0.f;
#pragma unroll
  for (int i = 0; i < GP / 4; ++i) {
    st.l[i] = 0.f;
    st.m[i] = -INFINITY;
  }
}

// STAT: where the pooled scores of type k of (query b, kv-head) begin (they lie in the order of the three page lists), and
// how many pages of that list there is room for
__device__ __forceinline__ float* stat_row(const thinkv_config& c, const DecodeArgs& a, int b, int hkv, int k, const int* np, int* room) {
  const int before = k == 0 ? 0 : (k == 1 ? np[0] : np[0] + np[1]);
  *room = (int)(a.stat_stride / kPage) - before;
  return a.stat + ((int64_t)b * c.n_kv_heads + hkv) * a.stat_stride + (int64_t)before * kPage;
}

// runs CALL with the runner `cr` of the type's bit width
#define TKV_WITH_RUNNER(BITS_, CALL)                                                                  \
  {                                                                                                   \
    if constexpr (FP) {                                                                               \
      ClassRunnerFp<D, BITS_, GP, STAT> cr(st, c, a, G, query.qf, stat, stat_room, xch);                   \
      CALL;                                                                                           \
      cr.leave();                                                                                     \
    } else {                                                                                          \
      ClassRunner<D, BITS_, GP, STAT> cr(st, c, a, G, query.qr, stat, stat_room, xch);                     \
      CALL;                                                                                           \
      cr.leave();                                                                                     \
    }                                                                                                 \
  }
#define TKV_BY_WIDTH(BITS, CALL)                \
  if (BITS == 2) TKV_WITH_RUNNER(2, CALL)       \
  else if (BITS == 4) TKV_WITH_RUNNER(4, CALL)  \
  else TKV_WITH_RUNNER(8, CALL)

// Four channels of the sum of W partials of query head g of (query b, kv-head), `stride` floats apart in LDS: the result where
// the head has one item, else the item's partial row.
template <int D>
__device__ __forceinline__ void fold_rows(const DecodeArgs& a, const float* rows, int stride, int W, int b, int hkv, int g, int ch, int Hq, int G, int row) {
  float M = -INFINITY;
  for (int w = 0; w < W; ++w) M = fmaxf(M, rows[w * stride + D]);
  float L = 0.f;
  float4 A = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int w = 0; w < W; ++w) {
    const float* src = rows + w * stride;
    const float f = src[D] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(src[D] - M);
    const float4 x = *(const float4*)(src + ch);
    L = fmaf(src[D + 1], f, L);
    A.x = fmaf(x.x, f, A.x);
    A.y = fmaf(x.y, f, A.y);
    A.z = fmaf(x.z, f, A.z);
    A.w = fmaf(x.w, f, A.w);
  }
  if (a.direct) {
    const int64_t at = ((int64_t)b * Hq + hkv * G + g) * D + ch;
    const float o[4] = {A.x, A.y, A.z, A.w};
#pragma unroll
    for (int r = 0; r < 4; ++r) store_from_f32(a.out, at + r, a.out_dtype, L > 0.f ? o[r] / L : 0.f);
    if (a.lse && ch == 0) a.lse[(int64_t)b * Hq + hkv * G + g] = L > 0.f ? (M + log2f(L)) * 0.6931471805599453f : -INFINITY;
  } else {
    float* dst = partial_row(a, G, D, row, g);
    *(float4*)(dst + ch) = A;
    if (ch == 0) {
      dst[D] = M;
      dst[D + 1] = L;
    }
  }
}

// Full-attention layers: a workgroup of W = blockDim.x / 64 waves, on one item or on several side by side (see the head of the
// file).
// FP: the cache is in the paper's number formats (decode_mfma_fp.h), else in the integer formats.
template <int D, int GP, bool STAT, bool FP>
__global__ __launch_bounds__(256 * decode_waves_per_simd(D, FP)) __attribute__((amdgpu_waves_per_eu(decode_waves_per_simd(D, FP), decode_waves_per_simd(D, FP)))) void decode_stream_kernel(thinkv_view v, DecodeArgs a) {
  constexpr int kRing = stream_ring_bytes(D, FP), kRow = D + kRowPad, kFull = 4 * decode_waves_per_simd(D, FP);
  extern __shared__ __attribute__((aligned(16))) uint8_t tkv_lds[];
  const thinkv_config& c = v.cfg;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, W = blockDim.x >> 6;
  const int Hq = c.n_q_heads, G = Hq / c.n_kv_heads;
  Query<D, GP, FP> query;
  // this wave's item, and the waves it shares it with: `wph` from wave0 on
  ItemLoc it;
  int seq, np[3], wph = W;
  if (a.grid) {
    const Deal d = deal_item<kFull>(v, a, blockIdx.x, wave);
    if ((int)blockIdx.x >= d.items) return;   // (then no wave has one)
    it = d.it;
    wph = d.wph;
    seq = d.seq;
    query.load(a, ((int64_t)it.b * Hq + it.hkv * G) * D, G, lane);
#pragma unroll
    for (int k = 0; k < 3; ++k) np[k] = d.np[k];
  } else {
    it = locate_head(v.cfg, a, blockIdx.x);
    query.load(a, ((int64_t)it.b * Hq + it.hkv * G) * D, G, lane);
    seq = uniform(a.seq_ids[it.b]);
    count_items(a, seq_pages(v, a.layer, seq, np), it);
    if (it.j >= it.n) return;
  }
  const int group = whole(wave, wph), wave0 = group * wph;
  const int b = it.b, hkv = it.hkv, share_n = it.n > 0 ? it.n : 1;
  const bool valid = seq >= 0 && seq < c.max_seqs;
  constexpr bool kFine = D == 128 && !FP && !STAT;
  using Pairs = Stream<kFine>;
  Pairs q;
  const uint32_t base = lds_address(tkv_lds);
  q.ticket = (LdsCounter)(uintptr_t)(base + W * kRing + 4 * group);
  q.lane = lane;
  q.max_pages = c.max_pages;
  q.tab = (ConstI32)(uintptr_t)(v.block_table + (valid ? table_base(c, seq, a.layer, 0) : 0));
  q.msk = (ConstI32)(uintptr_t)(v.slot_mask + (valid ? table_base(c, seq, a.layer, 0) : 0));
  // Heads start on different types: a pair of 8-bit pages moves three times the bytes of a pair of 2-bit pages for the
  // same arithmetic, so if all walked the types in the same order the whole chip would swing between bandwidth-bound
  // and issue-bound phases.  An item takes the same fraction of each list.
  const int rot = (hkv + b + it.j) % 3;
  q.kind0 = rot;
  q.kind1 = rot + 1 < 3 ? rot + 1 : rot - 2;
  q.kind2 = rot + 2 < 3 ? rot + 2 : rot - 1;
  q.fine = kFine && wph == kFull && np[0] + np[1] + np[2] >= kFinePages * kFull * share_n ? 0 : kChunkShift;
  q.cum0 = q.share(Pairs::pick(q.kind0, np[0], np[1], np[2]), it.j, share_n, q.first0, q.end0);
  q.cum1 = q.cum0 + q.share(Pairs::pick(q.kind1, np[0], np[1], np[2]), it.j, share_n, q.first1, q.end1);
  q.cum2 = q.cum1 + q.share(Pairs::pick(q.kind2, np[0], np[1], np[2]), it.j, share_n, q.first2, q.end2);
  if (wave == wave0 && lane == 0) {
    *q.ticket = 0;
    if constexpr (STAT)
      if (a.stat_sum && it.n > 0 && it.j == 0 && hkv == 0) a.stat_sum[b] = 0;
    if (it.n > 0 && it.j == 0 && !a.direct) {
      a.alloc[2 * (b * c.n_kv_heads + hkv)] = it.row0;
      a.alloc[2 * (b * c.n_kv_heads + hkv) + 1] = it.n;
    }
  }
  q.left = q.row = q.end = q.sec = q.pg = q.more_pages = q.pid_a = q.pid_b = q.msk_a = q.msk_b = 0;
  WaveState<D, GP, Query<D, GP, FP>::NSET> st;
  clear(st);
  __syncthreads();
  const uint32_t ring = base + wave * kRing, xch = base + W * kRing + kTicketBytes + exchange_bytes(D, GP, FP) * wave;
  q.look();
  query.finish(a, G, lane);
  while (q.sec < 3) {
    const int x = q.sec, k = Pairs::pick(x, q.kind0, q.kind1, q.kind2);
    const int bits = c.bits_of_class[k];
    float* stat = nullptr;
    int stat_room = 0;
    if constexpr (STAT) stat = stat_row(c, a, b, hkv, k, np, &stat_room);
    q.want = x;
    TKV_BY_WIDTH(bits, stream_pairs<kRing>(cr, q, v, k, hkv, ring))
  }
  // ---- the waves' partials meet in LDS (the rings are done with) and are folded there
  const Partial<D, GP, FP> part(st, lane);
  const int head = lane & (GP - 1), qd = lane >> 4;
  float* const rows = (float*)tkv_lds;   // [wave][G][kRow]
  __syncthreads();
  if (head < G) {
    float* dst = rows + (wave * G + head) * kRow;
    part.each(st, lane, [&](int ch, float4 x) { *(float4*)(dst + ch) = x; });
    if (qd == 0 && (lane & 15) < GP) {
      dst[D] = part.m;
      dst[D + 1] = part.l;
    }
  }
  __syncthreads();
  if (it.n == 0) return;
  for (int i = threadIdx.x - 64 * wave0; i < G * (D / 4); i += 64 * wph) {
    const int g = i / (D / 4), ch = 4 * (i % (D / 4));
    fold_rows<D>(a, rows + (wave0 * G + g) * kRow, G * kRow, wph, b, hkv, g, ch, Hq, G, it.row0 + it.j);
  }
}

// Sliding-window layers.  Little is visible (a window of 128 tokens: some ten to eighty pages of a list of a thousand), so the page
// lists are scanned: mask and id, page_pos_max, and where that reaches into the window the
// sixteen positions, three dependent loads.  A workgroup, all the waves of a compute unit, scans for `hg` kv-heads at once, a page of
// each type per thread with the three chains side by side, and leaves in LDS, in list order, what is visible: pages, or quads of slots (SlotQuads), as the
// first block with anything visible says: pages (which have scalar addresses, and a pair of which costs 5 to 8 % less) where a wave has one pair of them at most, or where
// they are hardly more pairs than the quads would be; the paper's formats have pages only.  Its waves then attend that, an hg-th of them a head; partials are folded in
// LDS, so a head with one item is finished here.  Blocks of pages are scanned until the lists are complete or full (kWindowList); entries of a block that found no room are
// there the next time round, when the block is scanned again.
// What bounds it: the scan's chains and the code that is met for the first time (a wave waits some 65 ns for every 64 bytes of instructions; so comparisons are
// as short as they can be, sums over waves are taken inside a row, and the fold divides by a reciprocal), 10 us with the launch, then the pairs of a wave.  How many there are follows from the
// slots: 128 tokens in slots that evictions freed lie in up to eighty pages, 40 pairs a head, most of whose slots are something else; of their quads there are
// 15 pairs.  us a call, pages attended by eight waves / quads by all, always / now:
//   reused slots: 128 x 4k..32k tokens, 64 heads of 64, window 128 27.4 / 19.2 / 19.1; 64 x 4k..8k, 40 heads of 128, window 500 52.0 / 36.2 / 35.9, 1,024 68.3 / 53.2 / 50.4;
//     256 x 500..5k, 64 heads of 64, window 500 90.2 / 57.6 / 58.3; 1 x 16k, 32 heads of 128, window 128 13.8 / 14.8 / 13.4
//   fresh slots, whose quads are whole pages: 256 x 500..5k, 40 heads of 128, window 500 45.6 / 50.5 / 45.5, 64 heads of 64 32.4 / 34.2 / 33.0;
//     64 x 4k..8k, 40 heads of 128, window 1,024 28.7 / 31.0 / 26.9; 8 x 8k, 40 heads of 128, window 128 11.7 / 12.5 / 10.9
// Twelve waves at head_dim 64 cost the smallest calls a little (2 x 16k tokens, window 128, fresh slots 9.5 whole pages by eight, now 10.4) and give more where slots are
// reused (1 x 16k, window 500 15.5 with eight, now 14.1).  A head's pairs by turns to its waves instead of in runs: 11.3 instead of 10.5 for 8 x 16k, window 128.
template <int D, int GP, bool STAT, bool FP>
__global__ __launch_bounds__(64 * window_waves(D)) __attribute__((amdgpu_waves_per_eu(window_waves(D) / 4, window_waves(D) / 4))) void decode_window_kernel(thinkv_view v, DecodeArgs a) {
  static_assert(window_lds_bytes(D, STAT) + window_waves(D) * exchange_bytes(D, GP, FP) <= 163840, "the LDS of a compute unit");
  constexpr int kWaves = window_waves(D), kRing = window_ring_bytes(D), kRow = D + kRowPad;
  extern __shared__ __attribute__((aligned(16))) uint8_t tkv_lds[];
  const thinkv_config& c = v.cfg;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int H = c.n_kv_heads, Hq = c.n_q_heads, G = Hq / H, hg = a.waves, wph = whole(kWaves, hg);
  const int groups = quotient(H + hg - 1, hg);
  // item id -> query, group of heads, item j of n (item-major)
  const int per = groups * a.B, j = a.per_head > 1 ? uniform((int)blockIdx.x / per) : 0, rest = (int)blockIdx.x - j * per;
  const int b = per < (1 << 24) ? quotient(rest, groups) : uniform(rest / groups), h0 = (rest - b * groups) * hg;
  const int seq = uniform(a.seq_ids[b]);
  int np[3];
  const int tot = seq_pages(v, a.layer, seq, np);
  int n = 1;
  if (a.per_head > 1) {
    n = uniform((int)(((uint32_t)tot + (uint32_t)a.ppi - 1u) / (uint32_t)a.ppi));
    n = n < 1 ? 1 : (n > a.per_head ? a.per_head : n);
  }
  if (j >= n) return;
  const int hw = whole(wave, wph), hkv = min(h0 + hw, H - 1);   // this wave's head (waves beyond the last head idle)
  if constexpr (STAT)
    if (a.stat_sum && j == 0 && h0 == 0 && threadIdx.x == 0) a.stat_sum[b] = 0;
  if (const int tid = threadIdx.x; j == 0 && !a.direct && tid < hg && h0 + tid < H) {
    a.alloc[2 * (b * H + h0 + tid)] = (b * H + h0 + tid) * a.per_head;
    a.alloc[2 * (b * H + h0 + tid) + 1] = n;
  }
  const uint32_t lds = lds_address(tkv_lds), xch = lds + window_lds_bytes(D, STAT) + exchange_bytes(D, GP, FP) * wave;
  // [type][page id], then [type][list position] with the statistic, [type][mask], [wave] counts
  int32_t* const ids = (int32_t*)(tkv_lds + kWaves * kRing);
  int32_t* const listed = ids + 3 * kWindowList;
  uint16_t* const masks = (uint16_t*)(ids + (STAT ? 6 : 3) * kWindowList);
  int32_t* const counts = (int32_t*)(masks + 3 * kWindowList);
  Query<D, GP, FP> query;
  query.load(a, ((int64_t)b * Hq + hkv * G) * D, G, threadIdx.x & 63);
  query.finish(a, G, threadIdx.x & 63);
  WaveState<D, GP, Query<D, GP, FP>::NSET> st;
  clear(st);
  const int qpos = uniform(a.q_pos[b]);
  const bool valid = seq >= 0 && seq < c.max_seqs;
  // the item's share of each list
  const int s0 = portion(np[0], j, n), e0 = portion(np[0], j + 1, n);
  const int s1 = portion(np[1], j, n), e1 = portion(np[1], j + 1, n);
  const int s2 = portion(np[2], j, n), e2 = portion(np[2], j + 1, n);
  const int most = uniform(max(e0 - s0, max(e1 - s1, e2 - s2)));
  bool by_page = FP;
  int have[3] = {0, 0, 0}, skip[3] = {0, 0, 0};   // entries in the lists; entries of this block that have been there before
  for (int base = 0; base < most;) {
    const int lane = fresh_lane(), tid = 64 * wave + lane;
    int pg[3], pid[3];
    uint32_t vis[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      pg[k] = (k == 0 ? s0 : (k == 1 ? s1 : s2)) + base + tid;
      const bool in = valid && pg[k] < (k == 0 ? e0 : (k == 1 ? e1 : e2));
      pid[k] = 0;
      vis[k] = 0;
      if (in) {
        const int64_t at = table_base(c, seq, a.layer, k) + pg[k];
        pid[k] = v.block_table[at];
        vis[k] = v.slot_mask[at] & 0xFFFFu;
      }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (vis[k] != 0 && v.page_pos_max[k][pid[k]] <= qpos - a.window) vis[k] = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (vis[k] != 0) {
        const int4* sp = (const int4*)(v.slot_pos[k] + (int64_t)pid[k] * kPage);
        uint32_t m = 0;
        auto inside = [&](int pos) { m += m + ((uint32_t)(qpos - pos) < (uint32_t)a.window ? 1u : 0u); };   // 0 <= qpos - pos < window
#pragma unroll
        for (int t4 = kPage / 4 - 1; t4 >= 0; --t4) {
          const int4 pos = sp[t4];
          inside(pos.w), inside(pos.z), inside(pos.y), inside(pos.x);
        }
        vis[k] &= m;
      }
    // what is visible, in list order: an entry for each page or quad of slots with a visible slot.  Counts of the three types in a word: a
    // wave has at most 64 pages and 256 quads of each
    auto add = [](int x, int y) { return x + y; };
    uint64_t seen[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) seen[k] = __ballot(vis[k] != 0);
    const int pages_seen = __popcll(seen[0]) | __popcll(seen[1]) << 10 | __popcll(seen[2]) << 20;
    int mine = 0, upto = 0;
    if constexpr (!FP) {
#pragma unroll
      for (int k = 0; k < 3; ++k) mine |= __popc((vis[k] | vis[k] >> 1 | vis[k] >> 2 | vis[k] >> 3) & 0x1111u) << (10 * k);
      upto = wave_scan(mine, add);
      if (lane == 63) counts[kCounts + wave] = upto;
    }
    if (lane == 63) counts[wave] = pages_seen;
    __syncthreads();
    // ... summed over the waves before this one, and over all
    static_assert(kWaves < 16, "a row holds the counts of the waves behind a zero");
    const bool counted = lane > 0 && lane <= kWaves;
    const int pages_of_wave = counted ? counts[lane - 1] : 0, quads_of_wave = !FP && counted ? counts[kCounts + lane - 1] : 0;
    const int upto_wave = row_scan(pages_of_wave, add);   // (at most 768 pages of a type)
    const int pages_all = __builtin_amdgcn_readlane(upto_wave, 15), pages_before = __builtin_amdgcn_readlane(upto_wave, wave);
    int total[3], from[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) total[k] = pages_all >> (10 * k) & 1023, from[k] = pages_before >> (10 * k) & 1023;
    if constexpr (!FP) {
      if ((have[0] | have[1] | have[2] | skip[0] | skip[1] | skip[2]) == 0) {
        const int quads = __builtin_amdgcn_readlane(row_scan((quads_of_wave & 1023) + (quads_of_wave >> 10 & 1023) + (quads_of_wave >> 20), add), 15);
        const int whole_pairs = (total[0] + total[1] + total[2] + 1) >> 1, quad_pairs = (quads + 7) >> 3;
        by_page = whole_pairs <= max(wph, quad_pairs + (quad_pairs >> 3) + 1);
      }
      if (!by_page) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const int upto_k = row_scan(quads_of_wave >> (10 * k) & 1023, add);
          total[k] = __builtin_amdgcn_readlane(upto_k, 15);
          from[k] = __builtin_amdgcn_readlane(upto_k, wave);
        }
      }
    }
    bool all = true;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int room = kWindowList - have[k];
      const int inside = by_page ? __builtin_amdgcn_mbcnt_hi((uint32_t)(seen[k] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)seen[k], 0)) : (upto - mine) >> (10 * k) & 1023;
      int at = from[k] + inside - skip[k];
      auto put = [&](int id, uint32_t m) {
        if (at >= 0 && at < room) {
          const int e = k * kWindowList + have[k] + at;
          ids[e] = id;
          masks[e] = (uint16_t)m;
          if (STAT) listed[e] = pg[k];
        }
        ++at;
      };
      if (by_page) {
        if (vis[k] != 0) put(pid[k], vis[k]);
      } else {
#pragma unroll
        for (int quad = 0; quad < 4; ++quad)
          if (vis[k] >> (4 * quad) & 15u) put(pid[k] << 2 | quad, vis[k] >> (4 * quad) & 15u);
      }
      const int took = min(total[k] - skip[k], room);
      have[k] += took;
      skip[k] += took;
      all = all && skip[k] == total[k];
    }
    __syncthreads();
    if (all) {
      base += 64 * kWaves;
      skip[0] = skip[1] = skip[2] = 0;
      if (base < most) continue;   // what further blocks have is attended with this one's
    }
    if (hw < hg && h0 + hw < H) {
      // The pairs of the three types one after the other, an equal run of them to each of the head's waves: a wave meets one type or two, and
      // waits for its first pages, and for a type's code, once or twice instead of three times.  (The paper's formats: by turns within each type.  A run of 8-bit pages, of
      // which the ring holds one pair, is slow there: 64 x 4k..8k, 40 heads, window 500 44.0 us by turns, 49.0 in runs.)
      int pairs[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) pairs[k] = by_page ? (have[k] + 1) >> 1 : (have[k] + 7) >> 3;
      const int everything = pairs[0] + pairs[1] + pairs[2];
      // Those that get one more are the head's first waves, on SIMDs side by side, or its last where the head before it has its first on the
      // same SIMDs (64 x 4k..8k tokens of reused slots, 8 kv-heads of 128, window 128 16.9 us without, 16.2 so)
      const int waves = fresh(wph), own = wave - hw * waves, turn = (hw * waves & 7) == 4 ? waves - 1 - own : own;
      const int each = whole(everything, waves), more = everything - waves * each;
      const int from = turn * each + min(turn, more), to = from + each + (turn < more ? 1 : 0);
#pragma unroll 1
      for (int k = 0; k < 3; ++k) {
        const int first = k == 0 ? 0 : (k == 1 ? pairs[0] : pairs[0] + pairs[1]), mine_of = k == 0 ? pairs[0] : (k == 1 ? pairs[1] : pairs[2]);
        const int begin = FP ? turn : max(from - first, 0), end = FP ? mine_of : min(mine_of, to - first);
        if (begin >= end) continue;
        const int bits = c.bits_of_class[k];
        float* stat = nullptr;
        int stat_room = 0;
        if constexpr (STAT) stat = stat_row(c, a, b, hkv, k, np, &stat_room);
        auto source = [&](auto q) {
          q.n = k == 0 ? have[0] : (k == 1 ? have[1] : have[2]);
          q.i = begin;
          q.end = end;
          q.step = FP ? wph : 1;
          q.pid = (LdsWords)(uintptr_t)(lds + kWaves * kRing + 4 * k * kWindowList);
          q.idx = q.pid + 3 * kWindowList;
          q.msk = (LdsHalves)(uintptr_t)(lds + kWaves * kRing + 4 * (STAT ? 6 : 3) * kWindowList + 2 * k * kWindowList);
          return q;
        };
        if (by_page) {
          auto q = source(VisiblePages<STAT>());
          TKV_BY_WIDTH(bits, stream_pairs<kRing>(cr, q, v, k, hkv, lds + wave * kRing))
        } else if constexpr (!FP) {
          auto q = source(SlotQuads<STAT>());
          TKV_BY_WIDTH(bits, quad_pairs<kRing>(cr, q, v, k, hkv, lds + wave * kRing))
        }
      }
    }
    have[0] = have[1] = have[2] = 0;
    __syncthreads();   // the lists have been used
  }
  const int lane = fresh_lane(), tid = 64 * wave + lane;
  const Partial<D, GP, FP> part(st, lane);
  const int head = lane & (GP - 1), qd = lane >> 4;
  float* const rows = (float*)tkv_lds;   // [wave][G][kRow]
  if (head < G) {
    float* dst = rows + (wave * G + head) * kRow;
    part.each(st, lane, [&](int ch, float4 x) { *(float4*)(dst + ch) = x; });
    if (qd == 0 && (lane & 15) < GP) {
      dst[D] = part.m;
      dst[D + 1] = part.l;
    }
  }
  __syncthreads();
  const float inv_G = __builtin_amdgcn_rcpf((float)G);   // (at most 64 query heads)
  for (int i = tid; i < hg * G * (D / 4); i += 64 * kWaves) {
    const int of = i / (D / 4), hd = (int)(((float)of + 0.5f) * inv_G), g = of - hd * G, ch = 4 * (i % (D / 4));
    if (h0 + hd < H) fold_rows<D>(a, rows + (hd * wph * G + g) * kRow, G * kRow, wph, b, h0 + hd, g, ch, Hq, G, (b * H + h0 + hd) * a.per_head + j);
  }
}

template <int D, int GP, bool STAT, bool FP>
static int launch_one(const thinkv_view& v, const DecodeArgs& a, hipStream_t st) {
  if (a.window > 0) {
    const int groups = (v.cfg.n_kv_heads + a.waves - 1) / a.waves;
    hipLaunchKernelGGL((decode_window_kernel<D, GP, STAT, FP>), dim3(a.per_head * groups * a.B), dim3(64 * window_waves(D)), window_lds_bytes(D, STAT) + window_waves(D) * exchange_bytes(D, GP, FP), st, v, a);
  } else {
    hipLaunchKernelGGL((decode_stream_kernel<D, GP, STAT, FP>), dim3(a.grid ? a.grid : a.n_rows), dim3(64 * a.waves), a.waves * (stream_ring_bytes(D, FP) + exchange_bytes(D, GP, FP)) + kTicketBytes, st, v, a);
  }
  return hipGetLastError() == hipSuccess ? THINKV_OK : THINKV_E_HIP;
}

template <bool STAT>
static int launch_decode_mfma_t(const thinkv_view& v, const DecodeArgs& a, hipStream_t st) {
  const int G = v.cfg.n_q_heads / v.cfg.n_kv_heads;
  if (G > 8) return THINKV_E_SHAPE;
  const bool fp = v.cfg.format == THINKV_FMT_FP;
  if (v.cfg.head_dim == 128) {
    if (G <= 4) return fp ? launch_one<128, 4, STAT, true>(v, a, st) : launch_one<128, 4, STAT, false>(v, a, st);
    return fp ? launch_one<128, 8, STAT, true>(v, a, st) : launch_one<128, 8, STAT, false>(v, a, st);
  }
  if (G <= 4) return fp ? launch_one<64, 4, STAT, true>(v, a, st) : launch_one<64, 4, STAT, false>(v, a, st);
  return fp ? launch_one<64, 8, STAT, true>(v, a, st) : launch_one<64, 8, STAT, false>(v, a, st);
}

}  // namespace thinkv

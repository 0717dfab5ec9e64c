// The per-type runner of the decode kernel for the paper's number formats (THINKV_FMT_FP): FP8 E4M3 with a
// per-tensor scale, NVFP4 (E2M1 codes) and ternary codes with one E4M3 scale per 16 channels of the token.
//
// Same plan as for the integer formats (decode_mfma_kernel.h): the codes go to v_mfma_f32_16x16x32_f16 without being
// dequantised, the scales are applied to what the matrix cores return.  What differs:
//   * E4M3 and E2M1 codes become binary16 numbers by gfx950's conversions (two codes in neighbouring bytes or nibbles an
//     instruction; exact, every value is a normal binary16 number); the keys of ternary codes too, spread to nibbles.  The keys come out
//     in another order of channels, in which the query is kept (QRegsFp); the two slots of a value register come from
//     different halves of a word and take a byte permutation on top;
//   * a value's ternary code is a sign and a magnitude bit: the bit placed right under a binary16 exponent IS the code's value
//     times 2^-14, the sign goes to bit 15;
//   * there are no zero-points, so the zero-point sums and the group sums of the query are gone;
//   * a group is 16 channels, half the K extent of the instruction: a slice of columns carries one group of 16, its
//     second operand is zero over the other half of the 32 channels, and there are twice as many column sets;
//   * an E4M3 scale is at most 448, so the lifted weights times the scale (times 2^-8: a scale byte shifted under a
//     binary16 exponent is the scale times 2^-8) always stay inside binary16: no check per pair;
//   * the 8-bit type has no scale per token: its tensor scales are folded into the exponent's factor (keys) and into
//     the tiles when the type is left (values).
#pragma once

namespace thinkv {

// Codes to operand registers of two binary16 numbers.  Shifts and masks (the magnitude bits under an exponent) took four
// instructions a register; now one for keys, one and a half (E4M3) or two (E2M1) for values, and three for the keys of ternary codes,
// which are spread to E2M1's nibbles.
// 16 x 24k..32k tokens of 2-, 4- and 8-bit types, head_dim 128, four heads: 133.2 us with shifts and masks, 129.0 so; all 4-bit 121
// and 107, eight heads a group 121 and 112; head_dim 64, 32 x 16k..32k, eight heads 141 and 127; all 8-bit 172 and 170, all 2-bit alike.
template <int BITS>
struct FldFp {
  static constexpr int FPH = 16 / BITS;
  static constexpr int VEXP = BITS == 2 ? 14 : 0;   // value operand = value of the code * 2^-VEXP
  static __device__ __forceinline__ uint32_t fp8(uint32_t x, bool upper) {   // bytes 0, 1 or bytes 2, 3
    return upper ? __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(x, 1.0f, true))
                 : __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(x, 1.0f, false));
  }
  static __device__ __forceinline__ uint32_t fp4(uint32_t x, int byte) {     // the nibbles of a byte
    return byte == 0   ? __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(x, 1.0f, 0))
           : byte == 1 ? __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(x, 1.0f, 1))
           : byte == 2 ? __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(x, 1.0f, 2))
                       : __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(x, 1.0f, 3));
  }
  // two ternary codes [s m] of the lower or upper half of every byte -> two E2M1 codes [s 0 m 0]
  static __device__ __forceinline__ uint32_t spread(uint32_t x, bool upper) {
    return upper ? ((x >> 3) & 0x02020202u) | ((x >> 2) & 0x08080808u) | ((x >> 1) & 0x20202020u) | (x & 0x80808080u)
                 : ((x << 1) & 0x02020202u) | ((x << 2) & 0x08080808u) | ((x << 3) & 0x20202020u) | ((x << 4) & 0x80808080u);
  }
  // register i (0..3) of the lane's eight channels of group g of 32: channels (0, 2), (1, 3), (4, 6), (5, 7), the order of QRegsFp::pairs
  // (a field of the chunk is two neighbouring channels, one in each half of its word; the group's are fields 4 g .. + 3)
  static __device__ __forceinline__ uint32_t keys(const uint32_t* w, int g, int i) {
    if constexpr (BITS == 8) return fp8(w[2 * g + (i >> 1)], i & 1);
    else if constexpr (BITS == 4) return fp4(w[g], (i >> 1) + 2 * (i & 1));
    else return fp4(spread(w[g >> 1], i >> 1), (g & 1) + 2 * (i & 1));
  }
  // field f of a value chunk: two slots (low / high half) of one channel.  (Two neighbouring fields share their first instructions.)
  static __device__ __forceinline__ uint32_t values(const uint32_t* w, int f) {
    const uint32_t x = w[f / FPH];
    const int pos = f % FPH;
    if constexpr (BITS == 8) {
      return fp8(__builtin_amdgcn_perm(0u, x, 0x03010200u), pos);
    } else if constexpr (BITS == 4) {
      const uint32_t lo = fp4(x, pos >> 1), hi = fp4(x, 2 + (pos >> 1));   // (fields f & ~1, f | 1) of either half
      return f & 1 ? __builtin_amdgcn_perm(hi, lo, 0x07060302u) : __builtin_amdgcn_perm(hi, lo, 0x05040100u);
    } else {   // (spread and put together again it would be no less)
      return ((10 - 2 * pos >= 0 ? x << (10 - 2 * pos & 31) : x >> (2 * pos - 10 & 31)) & 0x04000400u) | ((x << (14 - 2 * pos)) & 0x80008000u);
    }
  }
};

template <int D, int GP>
struct ColsFp {
  static constexpr int NG = D / 16;                           // groups of 16 channels
  static constexpr int CS = (16 / GP) < NG ? (16 / GP) : NG;   // groups (slices) per column set: 2 or 4
  static constexpr int NSET = NG / CS;
};

template <int D, int BITS, int NSET>
struct PageRegsFp {
  static constexpr int CW = (D / 32) * BITS / 4;
  uint32_t kw[CW], vw[CW];
  uint8_t ks[NSET];    // the E4M3 scale byte of (the slice's group, the lane's token); unused at 8 bits
  uint32_t vm[NSET];   // the E4M3 scale bytes of (the slice's group, the lane's four slots); unused at 8 bits
};
template <int D, int BITS, int NSET>
struct PairRegsFp {
  PageRegsFp<D, BITS, NSET> a, b;
};

// per column set the eight binary16 values of (the lane's head, channels 32 G + 8 qd ..) where those channels lie in
// the group of 16 of the lane's slice; zeros otherwise.  In the order in which FldFp::keys gives the codes.
template <int NSET>
struct QRegsFp {
  H8 q[NSET];
  static __device__ __forceinline__ H8 pairs(const H8& x) {   // channels (0, 1), (2, 3), .. -> (0, 2), (1, 3), ..
    H8 p;
#pragma unroll
    for (int i = 0; i < 4; i += 2) {
      p.u[i] = __builtin_amdgcn_perm(x.u[i + 1], x.u[i], 0x05040100u);
      p.u[i + 1] = __builtin_amdgcn_perm(x.u[i + 1], x.u[i], 0x07060302u);
    }
    return p;
  }
};

// four scale bytes (slots 0..3 of the lane's quad) -> two registers of binary16 pairs, each scale times 2^-8
__device__ __forceinline__ void scales_to_halves(uint32_t bytes, uint32_t& lo, uint32_t& hi) {
  lo = __builtin_amdgcn_perm(0u, bytes, 0x0C010C00u) << 7;
  hi = __builtin_amdgcn_perm(0u, bytes, 0x0C030C02u) << 7;
}

// STAT: besides attending, leave the group-pooled score of every visited slot for the attention-sparsity statistic
// (as the integer-format runner does).
template <int D, int BITS, int GP, bool STAT>
struct ClassRunnerFp {
  using CL = ColsFp<D, GP>;
  static constexpr int kD = D, kBlockBytes = block_geom(BITS, D, THINKV_FMT_FP).block_bytes;
  static constexpr bool kStat = STAT, kFp = true;
  static constexpr int NG32 = D / 32, NM = D / 16, CS = CL::CS, NSET = CL::NSET, NS = GP / 4;
  static constexpr int kLift = 14;
  static constexpr float kSlack = 1.0f;   // 2^(14 + 1) * 448 * 2^-8 < 65504: the lifted second operand of the value products cannot overflow
  using F = FldFp<BITS>;
  using Pair = PairRegsFp<D, BITS, NSET>;
  const int lane;
  WaveState<D, GP, NSET>& st;
  Softmax<D, GP, NSET, STAT, exchange_bytes(D, GP, true) != 0> sm;
  int k_off[NSET], v_off[NSET];   // byte offset, inside a meta region, of the lane's scale byte (K) and of its four scale bytes (V) per column set
  H8 bq[NG32];          // A operands of the score MFMAs: q over the half of the 32 channels that is the slice's group, zeros elsewhere
  float tile_out;       // tiles -> absolute units / 2^24 when the type is left
  float neg1;

  __device__ __forceinline__ ClassRunnerFp(WaveState<D, GP, NSET>& st_, const thinkv_config& c, const DecodeArgs& a, int G, const QRegsFp<NSET>& qr, float* stat_,
                                           int stat_room_, uint32_t xch)
      : lane(threadIdx.x & 63), st(st_), sm(st_, threadIdx.x & 63, G, stat_, stat_room_, xch) {
    const int qd = lane >> 4, n = lane & 15;
    const int gl = n / GP;
    const int glc = gl < CS ? gl : CS - 1;
    const int gk = GP == 4 ? qd : qd >> 1, gkc = gk < CS ? gk : CS - 1;   // slice of the rows of this lane's quad
    neg1 = -1.0f;
    asm volatile("" : "+v"(neg1));
    if constexpr (BITS == 8) {
      sm.kappa = c.fp8_scale[0] * a.scale_log2e;
      tile_out = c.fp8_scale[1] * (1.0f / (float)(1 << 24)) * (1.0f / (float)(1 << kLift));
    } else {
      sm.kappa = 256.0f * a.scale_log2e;                                    // (scales: 2^8)
      tile_out = (float)(1 << F::VEXP) * (1.0f / (float)(1 << 16)) * (1.0f / (float)(1 << kLift));   // 2^(VEXP + 8 - 24 - lift)
    }
#pragma unroll
    for (int s = 0; s < NSET; ++s) {
      k_off[s] = (s * CS + gkc) * kPage + n;
      v_off[s] = (s * CS + glc) * kPage + 4 * qd;
    }
#pragma unroll
    for (int g = 0; g < NG32; ++g) {
      const int set = (2 * g) / CS;
      const bool on = gl < CS && ((set * CS + gl) >> 1) == g;
#pragma unroll
      for (int w = 0; w < 4; ++w) bq[g].u[w] = on ? qr.q[set].u[w] : 0u;
    }
    // enter the type: the denominator and the tiles take the lift, the tiles the units of the type
    sm.enter((float)kLift, kSlack);
    sm.scale_sums((float)(1 << kLift));
    const float in = 1.0f / tile_out;
#pragma unroll
    for (int mb = 0; mb < NM; ++mb) st.o[mb] *= in;
  }
  __device__ __forceinline__ void leave() {
    sm.leave();
    sm.scale_sums(1.0f / (float)(1 << kLift));
#pragma unroll
    for (int mb = 0; mb < NM; ++mb) st.o[mb] *= tile_out;
  }

  template <class P>
  __device__ __forceinline__ void load_k(Pair& r, P blk_a, P blk_b) const {
    keys_of(r.a, blk_a);
    keys_of(r.b, blk_b);
  }
  template <class P>
  __device__ __forceinline__ void load_v(Pair& r, P blk_a, P blk_b) const {
    values_of(r.a, blk_a);
    values_of(r.b, blk_b);
  }
  using Page = PageRegsFp<D, BITS, NSET>;
  template <class P>
  __device__ __forceinline__ void keys_of(Page& x, P blk) const {
    const BlockGeom g = block_geom(BITS, D, THINKV_FMT_FP);
    load_chunk<Page::CW>(x.kw, blk + g.k_codes, lane);
    if constexpr (BITS != 8) {
#pragma unroll
      for (int s = 0; s < NSET; ++s) x.ks[s] = ld_piece<uint8_t>(blk + g.k_meta + k_off[s]);
    }
  }
  template <class P>
  __device__ __forceinline__ void values_of(Page& x, P blk) const {
    const BlockGeom g = block_geom(BITS, D, THINKV_FMT_FP);
    load_chunk<Page::CW>(x.vw, blk + g.v_codes, lane);
    if constexpr (BITS != 8) {
#pragma unroll
      for (int s = 0; s < NSET; ++s) x.vm[s] = ld_piece<uint32_t>(blk + g.v_meta + v_off[s]);
    }
  }

  // scores of one page for this lane's token and heads, in MFMA units (times kappa = log2 domain)
  __device__ __forceinline__ void page_scores(const PageRegsFp<D, BITS, NSET>& r, float* s) const {
    const float4v zero = {0.f, 0.f, 0.f, 0.f};
    float4v c[NSET];
#pragma unroll
    for (int g = 0; g < NG32; ++g) {
      const int set = (2 * g) / CS;
      const bool first = (2 * g) % CS == 0;
      H8 ka;
#pragma unroll
      for (int vv = 0; vv < 4; ++vv) ka.u[vv] = F::keys(r.kw, g, vv);
      c[set] = __builtin_amdgcn_mfma_f32_16x16x32_f16(bq[g].h, ka.h, first ? zero : c[set], 0, 0, 0);
    }
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int set = 0; set < NSET; ++set) {
      if constexpr (BITS == 8) {
#pragma unroll
        for (int R = 0; R < 4; ++R) acc[R] = set == 0 ? c[set][R] : acc[R] + c[set][R];
      } else {
        const float sc = (float)__builtin_bit_cast(_Float16, (uint16_t)(r.ks[set] << 7));   // the scale times 2^-8
#pragma unroll
        for (int R = 0; R < 4; ++R) acc[R] = fmaf(sc, c[set][R], acc[R]);
      }
    }
    add_groups<GP>(acc, s);
  }

  float sa[NS], sb[NS];   // scores of the pair at hand
  template <class Ids>
  __device__ __forceinline__ void scores(const Pair& r, const Ids& id) {
    page_scores(r.a, sa);
    page_scores(r.b, sb);
    sm.mask(sa, sb, id);
    sm.reference(sa, sb, false);
  }
  __device__ __forceinline__ void values(const Pair& r) {
    float ea[NS], eb[NS], pa[4], pb[4];
    sm.weights(sa, sb, ea, eb, pa, pb);
    sm.add(ea, eb);
    // values, per column set: B = two-term split of p * s_V, A = V codes
    H8 hi, lo;
#pragma unroll
    for (int set = 0; set < NSET; ++set) {
      if (BITS != 8 || set == 0) {
        float xa[4], xb[4];
        if constexpr (BITS == 8) {
#pragma unroll
          for (int r4 = 0; r4 < 4; ++r4) {
            xa[r4] = pa[r4];
            xb[r4] = pb[r4];
          }
        } else {
          uint32_t al, ah, bl, bh;
          scales_to_halves(r.a.vm[set], al, ah);
          scales_to_halves(r.b.vm[set], bl, bh);
          xa[0] = fmaf(half_lo(al), pa[0], 0.0f); xa[1] = fmaf(half_hi(al), pa[1], 0.0f);
          xa[2] = fmaf(half_lo(ah), pa[2], 0.0f); xa[3] = fmaf(half_hi(ah), pa[3], 0.0f);
          xb[0] = fmaf(half_lo(bl), pb[0], 0.0f); xb[1] = fmaf(half_hi(bl), pb[1], 0.0f);
          xb[2] = fmaf(half_lo(bh), pb[2], 0.0f); xb[3] = fmaf(half_hi(bh), pb[3], 0.0f);
        }
        // k-slots 8qd+e: e<4 page a slots 4qd+e, e>=4 page b
        hi.u[0] = pack_rne(xa[0], xa[1]);
        hi.u[1] = pack_rne(xa[2], xa[3]);
        hi.u[2] = pack_rne(xb[0], xb[1]);
        hi.u[3] = pack_rne(xb[2], xb[3]);
        lo.u[0] = pack_rne(fmaf(neg1, half_lo(hi.u[0]), xa[0]), fmaf(neg1, half_hi(hi.u[0]), xa[1]));
        lo.u[1] = pack_rne(fmaf(neg1, half_lo(hi.u[1]), xa[2]), fmaf(neg1, half_hi(hi.u[1]), xa[3]));
        lo.u[2] = pack_rne(fmaf(neg1, half_lo(hi.u[2]), xb[0]), fmaf(neg1, half_hi(hi.u[2]), xb[1]));
        lo.u[3] = pack_rne(fmaf(neg1, half_lo(hi.u[3]), xb[2]), fmaf(neg1, half_hi(hi.u[3]), xb[3]));
      }
#pragma unroll
      for (int mm = 0; mm < CS; ++mm) {
        const int mb = CS * set + mm;   // a 16-channel block is a group
        H8 va;
        va.u[0] = F::values(r.a.vw, 0 * NM + mb);
        va.u[1] = F::values(r.a.vw, 1 * NM + mb);
        va.u[2] = F::values(r.b.vw, 0 * NM + mb);
        va.u[3] = F::values(r.b.vw, 1 * NM + mb);
        st.o[mb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(va.h, hi.h, st.o[mb], 0, 0, 0);
        st.o[mb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(va.h, lo.h, st.o[mb], 0, 0, 0);
      }
    }
  }
};

}  // namespace thinkv

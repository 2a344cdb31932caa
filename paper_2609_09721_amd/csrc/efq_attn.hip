// EFQ-Softmax attention forward for AMD Instinct MI355X (gfx950, CDNA4).
//
// Kernels:
//   vquant_kernel      V (bf16) -> MXFP4 V~ in the FP4 matrix-core operand
//                      order (HBM-bound pre-pass, once per call).
//   mxfp8_kernel       Q, K (bf16) -> MXFP8 Q^, K^ for the low-bit Q K^T.
//   lowbit_quant_kernel  both, for Q, K and V of one call in one launch.
//   attn_pp_kernel     FlashAttention-style forward (Alg. 2 of the paper):
//                      S^T = K Q^T on bf16 (or block-scaled FP8) MFMA, the
//                      probability stage on the VALU (Alg. 1 for EFQ;
//                      exp-then-quantize for the baselines), O^T += V~^T P~^T
//                      on the block-scaled FP4 MFMA, the denominator P~ 1
//                      from the same operand; two wave groups alternate
//                      matrix-core and VALU phases; with NW = 4, workgroups
//                      of four waves, two on a CU, for short or small grids;
//                      with RHO, calibration candidates (below).
//   split_max_kernel, split_attn_kernel, split_merge_kernel
//                      few queries against many keys, split over the keys.
//   pgen_kernel        the probability stage alone on given shifted scores.
//   pgen_bench_kernel  register-resident throughput probe of that stage.
//   clock_probe_kernel shader clock under a matrix-core load (diagnostic).
//   rho_final_kernel   the relative Frobenius error of Alg. 3's objective, in
//                      fp64 with a fixed reduction order.
//   fill_zero_kernel   zero fill of the dump buffers (blocks never reached).
//
// Register layout (v_mfma_f32_32x32x16_bf16, verified on gfx950): lane L of a
// 64-lane wave holds column L%32 of the 32x32 result and rows
// 8*(r/4) + 4*(L/32) + r%4 in accumulator r = 0..15.  Scores are computed
// transposed (keys x queries), so every lane owns one query: lanes L and
// L+32 hold the two interleaved halves of a 32-key window.  One
// v_permlane32_swap hands each lane one whole 32-key block of its query,
// which is exactly the B operand (32 K-elements of one column, one E8M0
// scale per lane) of v_mfma_scale_f32_32x32x64_f8f6f4 in FP4 mode.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <type_traits>
#include <utility>
#include <vector>

#include "efq_attn.h"

namespace {

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef __attribute__((ext_vector_type(8))) int i32x8;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

// fp32 constants (nearest fp32 of the real value)
constexpr float kLn2 = 0.693147180559945309417f;     // log 2
constexpr float kInvLn2 = 1.44269504088896340736f;   // 1 / log 2 (= log2 e)
constexpr float kLog29 = -1.50407739677627407f;      // log(2/9), Eq. (k-rule)
constexpr float kLn6 = 1.79175946922805500081f;      // log 6, Eq. (z-def)

constexpr int kWaveQ = 32;     // queries per wave (MFMA N)
constexpr int kBc = 64;        // keys per tile (two 32-key microscaling blocks)
constexpr int kXcdCUs = 32;    // compute units of one of the 8 XCDs
constexpr int kCUs = 8 * kXcdCUs;

// C16 fold table of EFQ-Softmax-LUT (Sec. II-D) as bytes: byte j of the
// 16-byte table (little-endian dwords kC16T0..3) is C16[j].
constexpr unsigned kC16T0 = 0x01010100u;   // C16[0..3]   = 0 1 1 1
constexpr unsigned kC16T1 = 0x02020101u;   // C16[4..7]   = 1 1 2 2
constexpr unsigned kC16T2 = 0x05040303u;   // C16[8..11]  = 3 3 4 5
constexpr unsigned kC16T3 = 0x07070605u;   // C16[12..15] = 5 6 7 7

// ---------------------------------------------------------------- helpers
__device__ __forceinline__ int cvt_flr(float x) {
  // floor to int32, saturating (-inf -> INT_MIN)
  int r;
  asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(r) : "v"(x));
  return r;
}

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// v_permlane32_swap: afterwards lanes 0..31 hold (own a, upper partner's a),
// lanes 32..63 hold (lower partner's b, own b).
__device__ __forceinline__ void swap32(unsigned& a, unsigned& b) {
  auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}
__device__ __forceinline__ void swap32f(float& a, float& b) {
  unsigned ua = __float_as_uint(a), ub = __float_as_uint(b);
  swap32(ua, ub);
  a = __uint_as_float(ua);
  b = __uint_as_float(ub);
}

// Maximum of two values that came through an integer lane swap or are
// themselves maxima: an IEEE maximum would first quiet each operand (more
// instructions); scores are never NaN, so the plain instruction is exact.
__device__ __forceinline__ float fmax_swapped(float a, float b) {
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// Maximum of 16 values as a depth-3 tree of three-input maxima (v_max3):
// eight instructions with short dependency chains instead of a serial chain.
__device__ __forceinline__ float max3f(float a, float b, float c) {
  return __builtin_fmaxf(__builtin_fmaxf(a, b), c);
}
__device__ __forceinline__ float max16(const f32x16& v) {
  const float a = max3f(v[0], v[1], v[2]), b = max3f(v[3], v[4], v[5]);
  const float c = max3f(v[6], v[7], v[8]), d = max3f(v[9], v[10], v[11]);
  const float e = max3f(v[12], v[13], v[14]);
  return max3f(max3f(a, b, c), max3f(d, e, v[15]), -INFINITY);
}

// Operand dword dw of a lane holds the codes of accumulator elements
// j = 0..7 of one window and half-lane: element j sits in nibble
// 2 (j % 4) + j / 4 (the byte-then-nibble assembly of the probability stage).
__host__ __device__ __forceinline__ constexpr int elem_nibble(int j) { return 2 * (j & 3) + (j >> 2); }

// Key offset (0..31) of nibble e of the 16-byte FP4 operand of a lane.
__host__ __device__ __forceinline__ int nibble_key(int e) {
  int dw = e >> 3, nib = e & 7;
  int j = 4 * (nib & 1) + (nib >> 1);   // element within the dword
  int r = ((dw & 1) << 3) + j;          // accumulator index of the producing lane
  int gq = dw >> 1;                     // which half-lane produced it
  return 8 * (r >> 2) + 4 * gq + (r & 3);
}
// Inverse: nibble position of key t (0..31).
__host__ __device__ constexpr int key_nibble(int t) {
  return 8 * (2 * ((t >> 2) & 1) + (t >> 4)) + 2 * (t & 3) + ((t >> 3) & 1);
}

// -------------------------------------------------- probability stage
// Input: the two 32x32 score accumulators of a wave (s0: keys 0..31, s1: keys
// 32..63 of the tile; -inf where masked), the running maximum m (per lane =
// per query).  Output: the FP4 B operand (4 dwords, the 32 codes of the
// lane's own block), the lane's E8M0 scale, alpha = exp(m_old - m_new), and
// m updated to m_new (Eq. rowmax-update).
//
// The stage is split into pieces so the fused kernel can interleave them
// with the matrix-core work of the next tile:
//   pg_max     partial block maxima of the lane's 32 scores
//   pg_params  row maximum, its change, and the per-block parameters (Alg. 1:
//              M_b, k_b, and the affine bias; or the exp-then-quantize scale)
//   pg_alpha   alpha from the change (the fused kernel forms it only when
//              some row maximum of the wave moved)
//   pg_pair<E> codes of elements E, E+1 (element e = 16 * window + register)
//   pg_finish  one v_permlane32_swap per half-block: lane L keeps window L/32
// pgen<KIND>() runs them in order (standalone kernel and probe).
struct PgenArgs {
  float scale;   // softmax scale
  float sh;      // fl(scale * h)
  float sh32;    // 32 fl(scale * h)   (EFQ code argument, exact)
  float sh16;    // 16 fl(scale * h)   (LUT index argument, exact)
  float c;       // fl(log 6 + tau)
  float negh;    // -h
  float l2s;     // fl(scale * log2 e)   (exp-then-quantize)
};

struct PgenOut {
  u32x4 bop;
  int scale_b;
  float alpha;
};

struct PgenState {
  float bias[2];      // per window, with B = -(m + k_b log2 + log6 + tau) h:
                      // EFQ fl(32 B + 31.5), LUT fl(16 B + 15.5)
  unsigned d[2];      // EFQ, LUT: byte-packed codes / indices of the current dword
  float sc[2];        // EXPQ: 2^k_b per window (fp32 scale of the conversion)
  float mq;           // EXPQ: running maximum in log2 units
  int scale_b;        // E8M0 of the lane's own block
  float dm;           // m^{j-1} - m^j (0 when the maximum is unchanged)
  unsigned w[4];      // packed codes: window 0 regs 0-7, 8-15, window 1 ...
};


template <int KIND>
__device__ __forceinline__ void pg_max(const f32x16& s0, const f32x16& s1, float& pm0, float& pm1) {
  if constexpr (KIND == EFQ_PGEN_NOOP) {
    pm0 = pm1 = 0.0f;
  } else {
    pm0 = max16(s0);
    pm1 = max16(s1);
  }
}

// The exp-then-quantize baselines (OCP floor rule and the scale6 rule).
template <int KIND>
constexpr bool is_expq() { return KIND == EFQ_PGEN_EXPQ || KIND == EFQ_PGEN_EXPQ6; }

// Returns whether some row maximum of the wave moved (wave-uniform).
template <int KIND>
__device__ __forceinline__ bool pg_params(float pm0, float pm1, float& m, const PgenArgs& pa,
                                          PgenState& st) {
  bool moved = false;
  if constexpr (KIND == EFQ_PGEN_NOOP) {
    st.scale_b = 127 - 6;
    st.dm = 0.0f;
    st.w[0] = st.w[1] = st.w[2] = st.w[3] = 0x22222222u;
    return moved;
  } else {
    constexpr bool LOG2 = is_expq<KIND>();
    const float unit = LOG2 ? pa.l2s : pa.scale;
    swap32f(pm0, pm1);                          // lower: (own, partner) block 0; upper: block 1
    const float bmine = fmax_swapped(pm0, pm1);  // raw maximum of the lane's own block
    // the lane's block maximum in score units; rounding is monotone, so the
    // row maximum of the products is the product of the raw row maximum
    const float bs = bmine * unit;
    float t0 = bs, t1 = bs;
    swap32f(t0, t1);                            // (block 0 max, block 1 max) in every lane
    const float mt = fmax_swapped(t0, t1);      // rowmax S^j
    // m is itself a maximum (or -inf), so no operand quieting is needed
    const float mnew = fmax_swapped(m, mt);
    // alpha (pg_alpha) is formed only where a row maximum moved
    st.dm = m - mnew;
    moved = __builtin_amdgcn_ballot_w64(m != mnew) != 0ull;
    m = mnew;
    if constexpr (is_expq<KIND>()) {
      // exp-then-quantize, Eq. (post-softmax-path): max_t exp(x_t) =
      // exp(max_t x_t); the shift S2 - m2 is exact at the row maximum, so it
      // gets p = 1 exactly (an fma of the unshifted score could land on the
      // wrong side of the power-of-two scale boundary)
      const float amax = __builtin_amdgcn_exp2f(bs - m);
      const unsigned ab = __float_as_uint(amax);
      // OCP: floor(log2 amax) - 2; scale6: ceil(log2(amax / 6)), which is
      // floor(log2 amax) - 2, plus one when the mantissa exceeds 1.5
      int kb = (int)((ab >> 23) & 0xFF) - 127 - 2;
      if constexpr (KIND == EFQ_PGEN_EXPQ6) kb += (ab & 0x7FFFFF) > 0x400000u ? 1 : 0;
      kb = kb < -126 ? -126 : kb;               // 2^k must be a normal fp32 scale
      unsigned k0 = (unsigned)(kb + 127), k1 = k0;
      swap32(k0, k1);                           // (E8M0 of block 0, of block 1)
      st.sc[0] = __uint_as_float(k0 << 23);
      st.sc[1] = __uint_as_float(k1 << 23);
      st.scale_b = amax > 0.0f ? kb + 127 : 0;  // no visible key: E8M0 0x00, codes 0
      st.mq = m;
      st.w[0] = st.w[1] = st.w[2] = st.w[3] = 0u;
    } else {
      // Alg. 1: M_b = max_t x_t = fl(fl(max acc * scale) - m)
      const float Mb = bs - m;
      // k_b = floor((M_b + log(2/9)) / log 2), Eq. (k-rule); -inf -> INT_MIN -> -127
      int kb = cvt_flr((Mb + kLog29) * kInvLn2);
      kb = kb < -127 ? -127 : kb;
      // (z_t - tau) h with z_t = x_t - k_b log2 - log6 (Eq. z-def), folded to
      // fma(acc, scale h, bias), bias = -(m + k_b log2 + log6 + tau) h
      const float off = (float)kb * kLn2 + pa.c;
      float b0 = (m + off) * pa.negh;
      // EFQ: w_t = fma(acc_t, 32 scale h, fl(32 B + 31.5)) ~ 32 (u_t + 1) - 1/2;
      // LUT: the same with 16 levels, fl(16 B + 15.5)
      if constexpr (KIND == EFQ_PGEN_EFQ) b0 = __builtin_fmaf(b0, 32.0f, 31.5f);
      else b0 = __builtin_fmaf(b0, 16.0f, 15.5f);
      float b1 = b0;
      swap32f(b0, b1);                          // (bias of block 0, bias of block 1)
      st.bias[0] = b0;
      st.bias[1] = b1;
      st.scale_b = kb + 127;
    }
  }
  return moved;
}

// EFQ-Softmax-LUT, Sec. II-D: the 16-level index j16 = clip(floor(u) + 1,
// 0, 15) of u = (z_t - tau16) h16 is bits 7..4 of sat[0,255](rne(w)),
// w ~ 16 (u + 1) - 1/2 (the EFQ argument below with 16 levels), written to
// byte BYTE of d; lut_fold then maps the four indices of d through C16.
template <int BYTE>
__device__ __forceinline__ unsigned pg_lut_byte(float acc, const PgenArgs& pa, float bias16,
                                                unsigned d) {
  const float w = __builtin_fmaf(acc, pa.sh16, bias16);
  return __builtin_amdgcn_cvt_pk_u8_f32(w, BYTE, BYTE == 0 ? 0u : d);
}

// C16[j16] for the four LUT indices in bits 7..4 of the bytes of d: two
// byte-permute lookups (entries 0..7 and 8..15, selected by the low three
// index bits) and a per-byte select on index bit 3 (bit 7 of the byte,
// spread over the byte by the sign-replicating selectors 8..11).
__device__ __forceinline__ unsigned lut_fold(unsigned d) {
  const unsigned sel = (d >> 4) & 0x07070707u;
  const unsigned lo = __builtin_amdgcn_perm(kC16T1, kC16T0, sel);
  const unsigned hi = __builtin_amdgcn_perm(kC16T3, kC16T2, sel);
  // in[] = {d bytes 0..3, (d << 8) bytes 0..3}: selector 8 (9) replicates
  // bit 7 of in[1] (in[3]) = d byte 1 (3); 10 (11) of in[5] (in[7]) = d byte
  // 0 (2)
  const unsigned mask = __builtin_amdgcn_perm(d << 8, d, 0x090B080Au);
  return (hi & mask) | (lo & ~mask);
}

// EFQ code of one score into byte BYTE of d: c = clip(floor(u) + 1, 0, 7)
// of Eq. (d8-index) is bits 7..5 of sat[0,255](rne(w)), w ~ 32 (u + 1) - 1/2
// (a half-integer 32 n - 1/2 rounds to the even 32 n; w < 0 saturates to
// code 0, u + 1 >= 8 to 255, code 7).  One conversion per score.
template <int BYTE>
__device__ __forceinline__ unsigned pg_efq_byte(float acc, const PgenArgs& pa, float bias32,
                                                unsigned d) {
  const float w = __builtin_fmaf(acc, pa.sh32, bias32);
  return __builtin_amdgcn_cvt_pk_u8_f32(w, BYTE, BYTE == 0 ? 0u : d);
}

// Codes of elements E and E+1 (same window, same dword DW = E / 8).  In
// dword DW, element j = E % 8 sits in nibble elem_nibble(j).
template <int KIND, int E>
__device__ __forceinline__ void pg_pair(const f32x16& s0, const f32x16& s1, const PgenArgs& pa,
                                        PgenState& st) {
  if constexpr (KIND != EFQ_PGEN_NOOP) {
    constexpr int WIN = E / 16, R = E % 16, DW = E / 8, J = E % 8;
    const f32x16& s = WIN ? s1 : s0;
    if constexpr (is_expq<KIND>()) {
      // RNE(p / 2^k) to E2M1 with saturation; elements j and j + 4 share
      // byte j, so the pair is converted once both are known
      if constexpr (J < 4) {
        const float p0 = __builtin_amdgcn_exp2f(s[R] * pa.l2s - st.mq);
        const float p1 = __builtin_amdgcn_exp2f(s[R + 4] * pa.l2s - st.mq);
        st.w[DW] = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(st.w[DW], p0, p1, st.sc[WIN], J);
        const float p2 = __builtin_amdgcn_exp2f(s[R + 1] * pa.l2s - st.mq);
        const float p3 = __builtin_amdgcn_exp2f(s[R + 5] * pa.l2s - st.mq);
        st.w[DW] = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(st.w[DW], p2, p3, st.sc[WIN], J + 1);
      }
    } else if constexpr (KIND == EFQ_PGEN_LUT) {
      // as EFQ below: elements 0..3 into the bytes of d[0], 4..7 of d[1];
      // the folded codes (0..7, one per byte) merge into nibbles
      unsigned& d = st.d[J >> 2];
      d = pg_lut_byte<J & 3>(s[R], pa, st.bias[WIN], d);
      d = pg_lut_byte<(J & 3) + 1>(s[R + 1], pa, st.bias[WIN], d);
      if constexpr (J == 6) st.w[DW] = lut_fold(st.d[0]) | (lut_fold(st.d[1]) << 4);
    } else {
      // elements 0..3 of the dword into the bytes of d[0], 4..7 into d[1]
      unsigned& d = st.d[J >> 2];
      d = pg_efq_byte<J & 3>(s[R], pa, st.bias[WIN], d);
      d = pg_efq_byte<(J & 3) + 1>(s[R + 1], pa, st.bias[WIN], d);
      if constexpr (J == 6) {
        // nibble 2b <- bits 7..5 of byte b of d[0], nibble 2b+1 <- of d[1]
        st.w[DW] = ((st.d[0] >> 5) & 0x07070707u) | ((st.d[1] >> 1) & 0x70707070u);
      }
    }
  }
}

// alpha = exp(m^{j-1} - m^j), Eq. (alpha): exp2(0) = 1 exactly when the
// maximum is unchanged, exp2(-inf) = 0 on the first tile; m^j is finite from
// the first tile on (key 0 is visible to every query), so dm is never NaN.
template <int KIND>
__device__ __forceinline__ float pg_alpha(const PgenState& st) {
  if constexpr (KIND == EFQ_PGEN_NOOP) return 1.0f;
  else return __builtin_amdgcn_exp2f(is_expq<KIND>() ? st.dm : st.dm * kInvLn2);
}

template <int KIND>
__device__ __forceinline__ PgenOut pg_finish(PgenState& st) {
  PgenOut o;
  if constexpr (KIND != EFQ_PGEN_NOOP) {
    swap32(st.w[0], st.w[2]);
    swap32(st.w[1], st.w[3]);
  }
  o.bop = u32x4{st.w[0], st.w[1], st.w[2], st.w[3]};
  o.scale_b = st.scale_b;
  o.alpha = pg_alpha<KIND>(st);
  return o;
}

// Element pair of pair slot S (0..15): dword S / 4, its pairs taken in the
// order elements 0-1, 4-5, 2-3, 6-7, so that consecutive slots extend the
// two byte chains d[0] and d[1] of the dword in turn (two independent
// dependency chains instead of one; for exp-then-quantize, whose pairs 0-1
// and 2-3 carry all the conversions, an even spread over the regions).
__host__ __device__ constexpr int slot_elem(int S) { return 8 * (S >> 2) + ((S & 1) << 2) + (S & 2); }

// Pair slots E0 / 2 .. E1 / 2 - 1.
template <int KIND, int E0, int E1>
__device__ __forceinline__ void pg_pairs(const f32x16& s0, const f32x16& s1, const PgenArgs& pa,
                                         PgenState& st) {
  if constexpr (E0 < E1) {
    pg_pair<KIND, slot_elem(E0 / 2)>(s0, s1, pa, st);
    pg_pairs<KIND, E0 + 2, E1>(s0, s1, pa, st);
  }
}

template <int KIND>
__device__ __forceinline__ PgenOut pgen(const f32x16& s0, const f32x16& s1, float& m,
                                        const PgenArgs& pa) {
  float pm0, pm1;
  PgenState st;
  pg_max<KIND>(s0, s1, pm0, pm1);
  pg_params<KIND>(pm0, pm1, m, pa, st);
  pg_pairs<KIND, 0, 32>(s0, s1, pa, st);
  if constexpr (KIND == EFQ_PGEN_NOOP) asm volatile("" ::"v"(s0), "v"(s1));   // keep Q K^T live
  return pg_finish<KIND>(st);
}

// Operand codes of a lane in key order: 16 bytes, key 2j low nibble of byte j.
__device__ __forceinline__ u32x4 unpermute_codes(const u32x4& bop) {
  unsigned out[4] = {0, 0, 0, 0};
#pragma unroll
  for (int e = 0; e < 32; ++e) {
    unsigned c = (bop[e >> 3] >> (4 * (e & 7))) & 0xF;
    int t = nibble_key(e);
    out[t >> 3] |= c << (4 * (t & 7));
  }
  return u32x4{out[0], out[1], out[2], out[3]};
}

// ----------------------------------------------------------- V quantiser
// One thread per (b, kv head, 32-key block, pair of columns).  OCP MX rule:
// k = floor(log2 amax) - 2 (>= -127), codes RNE(|v| 2^-k) with saturation
// at 6 and the bf16 sign bit, keys stored in FP4 operand order.  The
// rounding is the hardware FP4 conversion of v 2^-k at scale 1 (two keys
// per instruction); the 32 row loads of a lane go out before any use.
struct VqArgs {
  int B, S, H, D, nb;  // nb = padded number of 32-key blocks
  size_t scale_off;
  unsigned vbytes;     // bytes of V when below 2^31 (buffer loads), else 0
};

// Codes of keys T and T + 8 of the lane's column c (0: low bf16 half of the
// raw dwords, 1: high) into byte T & 3 of dword 2 ((T >> 2) & 1) + (T >> 4),
// for T = 0..7 and 16..23.
template <int T>
__device__ __forceinline__ void vq_pairs(unsigned (&words)[4], const unsigned (&raw)[32], int c,
                                         int k) {
  if constexpr (T < 24) {
    if constexpr ((T & 8) == 0) {
      const unsigned lo = c ? (raw[T] & 0xffff0000u) : (raw[T] << 16);
      const unsigned hi = c ? (raw[T + 8] & 0xffff0000u) : (raw[T + 8] << 16);
      const float y0 = ldexpf(__uint_as_float(lo), -k);
      const float y1 = ldexpf(__uint_as_float(hi), -k);
      constexpr int W = 2 * ((T >> 2) & 1) + (T >> 4);
      static_assert(key_nibble(T) == 8 * W + 2 * (T & 3) && key_nibble(T + 8) == key_nibble(T) + 1,
                    "keys T and T + 8 fill the low and high nibble of byte T & 3 of dword W");
      words[W] = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(words[W], y0, y1, 1.0f, T & 3);
    }
    vq_pairs<T + 1>(words, raw, c, k);
  }
}

// The lane's column c (0: low bf16 half, 1: high) of a 32-key block: its codes
// in operand order, and the exponent k (floor(log2 amax) - 2, >= -127).
__device__ __forceinline__ int vq_column(const unsigned (&raw)[32], int c, unsigned (&words)[4]) {
  float amax = 0.f;
#pragma unroll
  for (int t = 0; t < 32; ++t)
    amax = fmaxf(amax, __uint_as_float(c ? raw[t] & 0x7fff0000u : (raw[t] & 0x7fffu) << 16));
  int k = -127;
  if (amax > 0.f) {
    // floor(log2 amax) from the fp32 bits (bf16 subnormals are fp32 normals)
    const int e = (int)((__float_as_uint(amax) >> 23) & 0xFF) - 127;
    k = e - 2 < -127 ? -127 : e - 2;
  }
  // keys t and t + 8 (t with bit 3 clear) share byte t & 3 of operand dword
  // 2 ((t >> 2) & 1) + (t >> 4): key t in the low nibble (key_nibble);
  // the conversion rounds y = v 2^-k (exact) to the nearest E2M1 value,
  // ties to the even code, sign from the input
  words[0] = words[1] = words[2] = words[3] = 0;
  vq_pairs<0>(words, raw, c, k);
  return k;
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, unsigned bytes);
template <bool BUF>
__device__ __forceinline__ void vquant_block(const unsigned short* __restrict__ v,
                                             uint8_t* __restrict__ vhat, const VqArgs& a,
                                             unsigned block) {
  // thread index: 32-bit with buffer loads (V below 2 GiB, so fewer than
  // 2^31 threads), which keeps the divisions short
  typedef typename std::conditional<BUF, unsigned, unsigned long>::type IDX;
  const int D2 = a.D >> 1;   // 32 or 64
  const IDX tid = (IDX)block * 256 + threadIdx.x;
  const IDX total = (IDX)a.B * a.H * a.nb * D2;
  if (tid >= total) return;
  const int dp = (int)(tid % D2);
  IDX r = tid / D2;
  const int blk = (int)(r % (IDX)a.nb);
  r /= (IDX)a.nb;
  const int g = (int)(r % (IDX)a.H);
  const int b = (int)(r / (IDX)a.H);
  const int d0 = 2 * dp;
  // the lane's column pair in the block's 32 rows; rows past S read as 0
  const int nvalid = min(32, a.S - blk * 32);
  const long e0 = (((long)b * a.S + (long)blk * 32) * a.H + g) * a.D + d0;
  unsigned raw[32];
  if constexpr (BUF) {
    // one resource over V, the lane's row-0 offset in voffset and the row
    // in the scalar offset: no per-row address arithmetic on the VALU
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(v, a.vbytes);
    const unsigned voff = (unsigned)e0 * 2u;
    const int sb = a.H * a.D * 2;   // bytes between consecutive keys
#pragma unroll
    for (int t = 0; t < 32; ++t)
      raw[t] = t < nvalid ? __builtin_amdgcn_raw_buffer_load_b32(rs, voff, t * sb, 0) : 0u;
  } else {
    const unsigned* p = (const unsigned*)(v + e0);
    const long stride = (long)a.H * a.D / 2;   // dwords between consecutive keys
#pragma unroll
    for (int t = 0; t < 32; ++t) raw[t] = t < nvalid ? p[t * stride] : 0u;
  }
  uint8_t* codes = vhat + (((long)b * a.H + g) * a.nb + blk) * a.D * 16;
  uint8_t* scales = vhat + a.scale_off + (((long)b * a.H + g) * a.nb + blk) * a.D;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    unsigned words[4];
    const int k = vq_column(raw, c, words);
    *(u32x4*)(codes + (long)(d0 + c) * 16) = u32x4{words[0], words[1], words[2], words[3]};
    const int d = d0 + c;
    scales[(d & 31) * (a.D >> 5) + (d >> 5)] = (uint8_t)(k + 127);
  }
}

template <bool BUF>
__global__ __launch_bounds__(256) void vquant_kernel(const unsigned short* __restrict__ v,
                                                     uint8_t* __restrict__ vhat, VqArgs a) {
  vquant_block<BUF>(v, vhat, a, blockIdx.x);
}

// ------------------------------------------------ MXFP8 Q / K quantiser
// Low-bit Q K^T: Q and K as MXFP8 under the OCP microscaling rule, per row
// and 32 consecutive head-dim elements: E8M0 exponent k = floor(log2 amax)
// - 8 (8 = the largest E4M3 exponent; amax = 0 or below the normal bf16
// range: k = -127), elements E4M3 (bias 7) of |x| 2^-k rounded to nearest
// even, saturating at 448, sign bit = sign of the bf16 input.  Output rows
// are [batch][head][padded seq] (rows past seq are zero): codes [..][D],
// scales [..][D/32] at soff.
struct Q8Args {
  int B, S, H, D, s_pad;
  size_t soff;
};

// Byte offsets in Q^ (K^) of the codes a thread writes, and, from the scales'
// start, of its 32-element block's scale.  Threads follow one another through
// the rows, 8 codes each, so thread n writes codes 8 n and scale n / 4; 64-bit
// (the codes pass 4 GiB long before the thread index does), with the
// workgroup's part scalar.
__host__ __device__ __forceinline__ size_t q8_code_at(unsigned block, unsigned thread) {
  return (size_t)block * 2048 + thread * 8;
}
__host__ __device__ __forceinline__ size_t q8_scale_at(unsigned block, unsigned thread) {
  return (size_t)block * 64 + (thread >> 2);
}

// One thread per 8 elements (4 threads per 32-element block, lanes 4i..4i+3);
// the rounding is the hardware E4M3 conversion (two elements per
// instruction) of |x| 2^-k clamped to 448, with the input's sign.
// IDX: the integer type of the thread and row indices (32-bit whenever the
// thread count fits, which keeps the divisions short).
template <typename IDX>
__device__ __forceinline__ void mxfp8_block(const unsigned short* __restrict__ x,
                                            uint8_t* __restrict__ y, const Q8Args& a, unsigned block) {
  const int parts = a.D / 8;   // 8 or 16
  const IDX n = (IDX)block * 256 + threadIdx.x;
  const IDX row = n / parts;
  const int part = (int)(n % parts);
  if (row >= (IDX)a.B * a.H * a.s_pad) return;   // whole rows, so whole 4-lane groups
  const int s = (int)(row % (IDX)a.s_pad);
  const IDX bh = row / (IDX)a.s_pad;
  const int h = (int)(bh % (IDX)a.H);
  const long b = (long)(bh / (IDX)a.H);
  u32x4 v = u32x4{0u, 0u, 0u, 0u};
  if (s < a.S) v = *(const u32x4*)(x + ((b * a.S + s) * a.H + h) * a.D + part * 8);
  unsigned am = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) am = max(am, max(v[i] & 0x7fffu, (v[i] >> 16) & 0x7fffu));
  am = max(am, (unsigned)__shfl_xor((int)am, 1));
  am = max(am, (unsigned)__shfl_xor((int)am, 2));
  const int e = (int)(am >> 7);
  const int k = e == 0 ? -127 : max(e - 135, -127);
  // each pair of elements: y = x 2^-k (exact), clamped to +-448 (the
  // saturation), then the hardware E4M3 conversion at scale 1 (nearest,
  // ties to even, sign from the input) into one 16-bit half of a word
  typedef __attribute__((ext_vector_type(2))) short s16x2;
  auto y2 = [&](int j, int half) {
    const unsigned b = half ? (v[j] & 0xffff0000u) : (v[j] << 16);
    return __builtin_amdgcn_fmed3f(ldexpf(__uint_as_float(b), -k), -448.0f, 448.0f);
  };
  s16x2 w0 = {0, 0}, w1 = {0, 0};
  w0 = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(w0, y2(0, 0), y2(0, 1), 1.0f, false);
  w0 = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(w0, y2(1, 0), y2(1, 1), 1.0f, true);
  w1 = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(w1, y2(2, 0), y2(2, 1), 1.0f, false);
  w1 = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(w1, y2(3, 0), y2(3, 1), 1.0f, true);
  const unsigned w[2] = {__builtin_bit_cast(unsigned, w0), __builtin_bit_cast(unsigned, w1)};
  *(uint2*)(y + q8_code_at(block, threadIdx.x)) = make_uint2(w[0], w[1]);
  if ((part & 3) == 0) y[a.soff + q8_scale_at(block, threadIdx.x)] = (uint8_t)(k + 127);
}

template <typename IDX>
__global__ __launch_bounds__(256) void mxfp8_kernel(const unsigned short* __restrict__ x,
                                                    uint8_t* __restrict__ y, Q8Args a) {
  mxfp8_block<IDX>(x, y, a, blockIdx.x);
}

// The quantisers of one call in one launch: with V, nv workgroups of V (the
// longest first), then nq of Q, then those of K.  HBM bound, like its parts;
// on a short prompt each of three launches was mostly its start and its tail:
// a low-bit call on 4096 tokens (32/8 heads, D 128) 99.2 -> 96.2 us.  V's
// part takes 76 registers, which leaves the others six waves a SIMD where
// they had eight: 5 % slower on 65537 tokens, so long calls take V apart.
struct QuantArgs {
  const unsigned short *q, *k, *v;
  uint8_t *qhat, *khat, *vhat;
  Q8Args qa, ka;
  VqArgs va;
  unsigned nv, nq;
};
template <bool V>
__global__ __launch_bounds__(256) void lowbit_quant_kernel(QuantArgs a) {
  const unsigned n = blockIdx.x;
  if (V && n < a.nv) vquant_block<true>(a.v, a.vhat, a.va, n);
  else if (n < a.nv + a.nq) mxfp8_block<unsigned>(a.q, a.qhat, a.qa, n - a.nv);
  else mxfp8_block<unsigned>(a.k, a.khat, a.ka, n - a.nv - a.nq);
}

// ------------------------------------------------------ fused attention
struct AttnArgs {
  int B, Sq, Sk, Hq, Hkv;
  int nb;             // padded 32-key blocks of V~
  size_t scale_off;   // byte offset of the E8M0 plane in V~
  int nqt;            // query tiles per (batch, head)
  int xcd_remap;      // 1: group work items by XCD
  float scale, tau, h;
  // dump (may be null)
  uint8_t* p_codes;
  uint8_t* p_e8m0;
  float* row_m;
  float* row_l;
  int nblk;           // ceil(Sk / 32)
  // MXFP8 Q^ / K^ (low-bit Q K^T): padded rows per head, scale offsets
  int sq_pad, sk_pad;
  size_t q8_soff, k8_soff;
  int spread;         // order of the work items (map_work)
  int o_rows;         // 1: half workgroups store O as whole rows, through LDS
};

// LDS layout.  A K tile is stored in the order the bf16 MFMA reads its A
// operand: 1 KB blocks, one per (32-key window w, 16-column step kk), slot
// `lane` of block (w, kk) holding K[32w + lane%32][16kk + 8(lane/32) .. +8].
// Every operand read is then one contiguous 1 KB wave access (no bank
// conflicts, immediate offsets), and every block is filled by one
// global_load_lds_dwordx4 (LDS address = base + 16 * lane).  A V~ tile (two
// 32-key blocks) is stored as in global memory: codes, then E8M0 scales
// grouped per lane (byte (d % 32) * (D/32) + d / 32 of each block).
// KS K buffers and VS V~ buffers form the LDS rings (depths and schedule
// at pp_schedule).  With MXFP8 Q and K (Q8) a K tile holds E4M3 codes in the
// order the FP8 MFMA reads its A operand (see KLoad8), then 256 bytes of
// E8M0 scales.
// Phase stamps, a diagnostic build only (EFQ_PHASE_STAMPS=1, its own
// library): the two waves of SIMD 0 in each of the first 256 workgroups
// record s_memtime at the end of each of their first kStampPhases phases,
// before and after the phase's wait and barrier, into LDS past the rings;
// the kernel copies them out at its end.  Four more slots per wave hold
// s_memtime and s_memrealtime (100 MHz) at the end of its first and of its
// last stamped phase, which gives the shader clock during the kernel.
// Reading the counter makes the wave wait for its outstanding LDS and
// scalar memory operations, so the stamped kernel runs slower than the
// product build; the stamps give the cycle distribution of the phases, not
// the product kernel's time.
#ifndef EFQ_PHASE_STAMPS
#define EFQ_PHASE_STAMPS 0
#endif
#if EFQ_PHASE_STAMPS
#define attn_pp_kernel attn_pp_kernel_stamped   // its own name in kernel traces
#endif
constexpr int kStampPhases = 512;
constexpr int kStampBlocks = 256;
constexpr int kStampSlots = 2 * kStampPhases + 4;   // per wave: 2 per phase, then the clock pairs
constexpr int kStampBytes = EFQ_PHASE_STAMPS ? 2 * kStampSlots * 8 : 0;

template <int D, int KS, int VS, bool Q8 = false, bool STAMPS = true>
struct Smem {
  static constexpr int kK = Q8 ? kBc * D + 256 : kBc * D * 2;   // one K tile
  static constexpr int kVc = 2 * D * 16;                 // V~ codes of two blocks
  static constexpr int kVs = 256;                        // V~ scales (2 D bytes, padded)
  static constexpr int kV = kVc + kVs;                   // one V~ tile
  static constexpr int kKOff = 0;
  static constexpr int kVOff = KS * kK;
  static constexpr int kStampOff = KS * kK + VS * kV;
  static constexpr int kTotal = KS * kK + VS * kV + (STAMPS ? kStampBytes : 0);
};

// Direct-to-LDS loads (buffer_load ... lds: LDS address = M0 base + size *
// lane).  The per-lane byte offsets are loop invariant; the tile position
// goes in the scalar offset, except for the last K tile.  The buffer range
// check compares the per-lane offset with the record count and leaves the
// scalar offset out, so the last (possibly ragged) K tile is read through a
// resource that starts at that tile: lanes of keys past seq_k then fall
// outside its record count and read zeros instead of memory past the end of
// K (those keys are masked anyway).  Every other tile lies inside K, and V~
// and the MXFP8 K^ are padded to whole tiles.  Asynchronous: the caller
// waits on vmcnt before the workgroup barrier that publishes the tile.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);
}

template <int D, int NW>
struct KLoad {
  static constexpr int KK = D / 16;
  static constexpr int PER = 2 * KK / NW;                // 1 KB blocks per wave
  static_assert(KK % PER == 0, "a wave's blocks share one 32-key window");
  const uint8_t* base;
  unsigned bytes;
  int voff0;                                             // lane's byte offset, first block
  unsigned tile_bytes;                                   // bytes per 64 keys
  int last;                                              // index of the last K tile
  __device__ void init(const unsigned short* kbatch, int Sk, int Hkv, int g, int wave, int lane) {
    base = (const uint8_t*)kbatch;
    bytes = (unsigned)((long)Sk * Hkv * D * 2);
    tile_bytes = (unsigned)(kBc * Hkv * D * 2);
    last = (Sk - 1) / kBc;
    // the wave's blocks are (window w, k-steps kk0 .. kk0+PER-1): block i
    // sits 32 bytes (16 bf16 columns) after block i-1 in every row
    const int blk = wave * PER;
    const int w = blk / KK, kk0 = blk % KK;
    const int row = 32 * w + (lane & 31);
    voff0 = ((row * Hkv + g) * D + kk0 * 16 + (lane >> 5) * 8) * 2;
  }
  static constexpr int kIssued = PER;                    // loads per wave per tile
  __device__ void issue(uint8_t* kbuf, int tile, int wave) const {
    if (tile == last) {                                  // wave-uniform
      const unsigned off = (unsigned)tile * tile_bytes;
      put(kbuf, make_rsrc(base + off, bytes - off), 0, wave);
    } else {
      put(kbuf, make_rsrc(base, bytes), (int)(tile * tile_bytes), wave);
    }
  }
  __device__ void put(uint8_t* kbuf, __amdgpu_buffer_rsrc_t rsrc, int soff, int wave) const {
#pragma unroll
    for (int i = 0; i < PER; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, kbuf + (wave * PER + i) * 1024, 16,
                                               voff0 + 32 * i, soff, 0, 0);
  }
};

template <int D, int NW>
struct VLoad {
  static constexpr int kVc = Smem<D, 1, 1>::kVc;         // V~ code bytes per tile
  static constexpr int NB = kVc / 1024;                  // 1 KB code blocks (2 or 4)
  static_assert(NB <= NW, "at most one code block per wave");
  const uint8_t* codes;
  const uint8_t* scales;
  int nb;
  int coff_lane;                                         // lane's byte offset of the code load
  int soff_lane;                                         // lane's byte offset of the scale load
  __device__ void init(const uint8_t* vcodes, const uint8_t* vscales, int nblocks, int lane) {
    codes = vcodes;
    scales = vscales;
    nb = nblocks;
    coff_lane = lane * 16;
    // 2 D scale bytes as dwords; for D = 64 the upper lanes repeat the
    // lower ones into the padding
    soff_lane = (lane % (2 * D / 4)) * 4;
  }
  // code block `wave` (waves below NB)
  __device__ void issue_codes(uint8_t* vbuf, int tile, int wave) const {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(make_rsrc(codes, (unsigned)(nb * D * 16)),
                                             vbuf + wave * 1024, 16, coff_lane,
                                             tile * 2 * D * 16 + wave * 1024, 0, 0);
  }
  // the tile's scales; several waves may load them (same bytes, same place)
  __device__ void issue_scales(uint8_t* vbuf, int tile) const {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(make_rsrc(scales, (unsigned)(nb * D)), vbuf + kVc, 4,
                                             soff_lane, tile * 2 * D, 0, 0);
  }
};

// MXFP8 K tiles (low-bit Q K^T).  The FP8 MFMA (32x32x64, E4M3) reads its A
// operand as 32 bytes per lane: lane l holds row l % 32 and, of a 64-column
// chunk, columns 16 (l / 32) + [0, 16) in bytes 0-15 and 32 + 16 (l / 32) +
// [0, 16) in bytes 16-31.  The LDS tile stores 1 KB blocks (window w, chunk
// c, half h) at ((w * D/64 + c) * 2 + h) KB, slot `lane` of the block holding
// the lane's 16 bytes of half h, so an operand is two contiguous wave reads;
// each block is one direct-to-LDS load.  The 64 keys' E8M0 scales follow
// (D/32 bytes per key, as in global memory).  Global K^ is [batch][kv head]
// [padded key][D] codes and [..][D/32] scales, so a tile is contiguous.
template <int D, int NW>
struct KLoad8 {
  static constexpr int NC = D / 64;                      // 64-column chunks
  static constexpr int NBLK = 4 * NC;                    // 1 KB code blocks per tile
  // code blocks per wave: wave, wave + NW, ... (NW blocks on is one 32-key
  // window on where a wave has two)
  static constexpr int PER = NBLK > NW ? NBLK / NW : 1;
  static_assert(PER == 1 || (PER == 2 && NW == 2 * NC), "a wave's second block is its window's twin");
  const void* codes;
  const void* scales;
  unsigned cbytes, sbytes;
  int voff;                                              // lane's byte offset in its block's rows
  __device__ void init(const uint8_t* kc, const uint8_t* ks, int sk_pad, int wave, int lane) {
    codes = kc;
    scales = ks;
    cbytes = (unsigned)sk_pad * D;
    sbytes = (unsigned)sk_pad * (D / 32);
    const int blk = wave < NBLK ? wave : 0;
    const int h = blk & 1, c = (blk >> 1) % NC, w = blk / (2 * NC);
    voff = (32 * w + (lane & 31)) * D + 64 * c + 32 * h + 16 * (lane >> 5);
  }
  // code blocks `wave`, `wave` + NW, ... (waves below NBLK)
  __device__ void issue_codes(uint8_t* kbuf, int tile, int wave) const {
#pragma unroll
    for (int i = 0; i < PER; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(make_rsrc(codes, cbytes), kbuf + (wave + i * NW) * 1024,
                                               16, voff + i * 32 * D, tile * kBc * D, 0, 0);
  }
  // 64 keys x D/32 bytes as dwords; for D = 64 the upper lanes read the
  // next tile's scales into the unused half.  The resource starts at the
  // tile, so the range check (which covers the per-lane offset only) turns
  // a read past the last tile into zeros.  Several waves may load them
  // (same bytes, same place).
  __device__ void issue_scales(uint8_t* kbuf, int tile, int lane) const {
    const unsigned off = (unsigned)tile * (kBc * (D / 32));
    __builtin_amdgcn_raw_ptr_buffer_load_lds(make_rsrc((const uint8_t*)scales + off, sbytes - off),
                                             kbuf + kBc * D, 4, lane * 4, 0, 0, 0);
  }
};

__device__ __forceinline__ void wait_vmem() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Workgroup barrier without the release fence of __syncthreads, which would
// wait for every outstanding global->LDS load (vmcnt(0)) at each barrier,
// although a tile is needed only several phases after its load is issued.
// The loads' consumers wait on vmcnt explicitly (wait_vmem_le) before the
// barrier that publishes them.  LDS reads need no wait here: every ring
// slot is read, and the read consumed, at least one barrier before the next
// load into it is issued.  The "memory" clobber keeps the compiler from
// moving LDS accesses across the barrier, the scheduling barriers keep the
// matrix-core and VALU work of a phase on its side.
__device__ __forceinline__ void wg_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}
// Wait until at most n vector-memory loads of this wave are outstanding
// (loads complete in issue order); n is wave-uniform and at most 12.
__device__ __forceinline__ void wait_vmem_le(int n) {
  switch (n) {
    case 0: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
    case 1: asm volatile("s_waitcnt vmcnt(1)" ::: "memory"); break;
    case 2: asm volatile("s_waitcnt vmcnt(2)" ::: "memory"); break;
    case 3: asm volatile("s_waitcnt vmcnt(3)" ::: "memory"); break;
    case 4: asm volatile("s_waitcnt vmcnt(4)" ::: "memory"); break;
    case 5: asm volatile("s_waitcnt vmcnt(5)" ::: "memory"); break;
    case 6: asm volatile("s_waitcnt vmcnt(6)" ::: "memory"); break;
    case 7: asm volatile("s_waitcnt vmcnt(7)" ::: "memory"); break;
    case 8: asm volatile("s_waitcnt vmcnt(8)" ::: "memory"); break;
    case 9: asm volatile("s_waitcnt vmcnt(9)" ::: "memory"); break;
    case 10: asm volatile("s_waitcnt vmcnt(10)" ::: "memory"); break;
    case 11: asm volatile("s_waitcnt vmcnt(11)" ::: "memory"); break;
    default: asm volatile("s_waitcnt vmcnt(12)" ::: "memory"); break;
  }
}

// Map a workgroup index to (batch, head, query tile).  Workgroups are handed
// to the 8 XCDs round-robin; with xcd_remap each XCD gets a contiguous range
// of work items.  Consecutive work items are the query heads of one GQA group
// at one query tile, then the next tile, so the workgroups that stream the
// same key/value tiles run side by side on one XCD and share its L2.  Query
// tiles run longest first.  The half workgroups of a causal grid have two more
// orders (`spread`, work_order), since there the length of an item decides:
//  1: an XCD's items by length over all its heads, the second 32 (one per CU)
//     reversed, so that a long workgroup shares its CU with a short one: 2
//     prompts of 1024 tokens 28.2 -> 24.9 us, one of 2048 40.0 -> 38.4 us;
//  2: all items by length over all heads, in the order they are handed out,
//     the second 256 reversed where the grid is resident at once.  Where the
//     heads do not divide evenly over the XCDs, whole heads leave some XCDs
//     with the long tiles of one more head, and where the workgroups do not
//     the last head's long tiles start last.  12 heads, EFQ, eight-wave kernel
//     / half workgroups head by head / in this order (us): 4096 tokens, D 128
//     69.4 / 70.6 / 61.7; 6000 tokens, D 64, MXFP8 66.3 / 70.7 / 65.0; 11 x 600
//     tokens, D 64 23.5 / 20.1 / 17.3.
template <bool SPREAD>
__device__ __forceinline__ void map_work(const AttnArgs& a, int& b, int& hq, int& qt) {
  const int n = blockIdx.x;
  const int total = gridDim.x;
  int w = n;
  if (a.xcd_remap) w = (n & 7) * (total >> 3) + (n >> 3);
  if (SPREAD && a.spread) {
    int i = n, heads = total / a.nqt, first = 0;           // of all XCDs
    if (a.spread == 2) {
      if (total <= 2 * kCUs && i >= kCUs) i = kCUs + total - 1 - i;
    } else {
      const int items = total >> 3;                        // of one XCD
      heads = items / a.nqt;
      first = (n & 7) * heads;
      i = n >> 3;
      if (i >= kXcdCUs) i = kXcdCUs + items - 1 - i;
    }
    const int bh = first + i % heads;
    qt = a.nqt - 1 - i / heads;
    hq = bh % a.Hq;
    b = bh / a.Hq;
    return;
  }
  const int G = a.Hq / a.Hkv;
  const int per = G * a.nqt;          // work items of one (batch, kv head)
  const int bg = w / per, r = w % per;
  qt = a.nqt - 1 - r / G;
  hq = (bg % a.Hkv) * G + r % G;
  b = bg / a.Hkv;
}

// V~ operands of one tile for the lane: the 16 code bytes of each slab and
// the E8M0 scales of all slabs in one register (slab s = byte s).
template <int D>
struct VOps {
  u32x4 a[D / 32];
  int sv;
};

// LDS addresses as 32-bit values: the lane's read addresses in ring slot 0
// stay in registers, and a slot is one scalar offset away.
typedef __attribute__((address_space(3))) const uint8_t* lds_cptr;
__device__ __forceinline__ unsigned lds_addr(const void* p) {
  return (unsigned)(uintptr_t)(lds_cptr)p;
}
__device__ __forceinline__ lds_cptr lds_at(unsigned a) { return (lds_cptr)(uintptr_t)a; }

// Lane offsets of the V~ operand reads within a ring slot: codes, scales.
template <int D>
__device__ __forceinline__ int vop_offset(int lane) {
  return ((lane >> 5) * D + (lane & 31)) * 16;
}
template <int D>
__device__ __forceinline__ int vscale_offset(int lane) {
  return Smem<D, 1, 1>::kVc + (lane >> 5) * D + (lane & 31) * (D / 32);
}

// vc, vs: the lane's code and scale reads in the tile's ring slot (the slab
// reads take immediate offsets from vc).
template <int D>
__device__ __forceinline__ void read_v(lds_cptr vc, lds_cptr vs, VOps<D>& v) {
  constexpr int NS = D / 32;
#pragma unroll
  for (int s = 0; s < NS; ++s)
    v.a[s] = *(__attribute__((address_space(3))) const u32x4*)(vc + s * 32 * 16);
  if constexpr (NS == 4) v.sv = *(__attribute__((address_space(3))) const int*)vs;
  else v.sv = *(__attribute__((address_space(3))) const unsigned short*)vs;
}

// O^T slabs += V~^T P~^T on the FP4 MFMA.  The lane's E8M0 scales of all
// slabs sit in one register `sv`; slab S selects byte S (op_sel).
template <int NS, int S = 0, int D>
__device__ __forceinline__ void pv_slabs(f32x16* oacc, const VOps<D>& v, const i32x8& bop, int sb) {
  if constexpr (S < NS) {
    const i32x8 aop = i32x8{(int)v.a[S][0], (int)v.a[S][1], (int)v.a[S][2], (int)v.a[S][3], 0, 0, 0, 0};
    oacc[S] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(aop, bop, oacc[S], 4, 4, S, v.sv, 0, sb);
    pv_slabs<NS, S + 1>(oacc, v, bop, sb);
  }
}

// Mask keys past the end and, for causal attention, keys after the query
// (the mask acts before the probability stage).  lim = number of visible
// keys of this lane counted from the tile start.
__device__ __forceinline__ void mask_tile(f32x16& s0, f32x16& s1, int l0) {
  // l0 = visible keys counted from the tile start, less 4 half: the
  // per-register key offsets stay immediates
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int kofs = 8 * (r >> 2) + (r & 3);
    s0[r] = kofs < l0 ? s0[r] : -INFINITY;
    s1[r] = kofs + 32 < l0 ? s1[r] : -INFINITY;
  }
}

// ------------------------------------------------- ping-pong variant
// Eight waves per workgroup (two per SIMD, 256 queries) in two groups of
// four.  Each tile is split into a matrix-core phase M(j) = P~V of tile j-1
// and S(j) = K(j) Q^T, and a VALU phase V(j) = the probability stage of
// tile j and the history rescale.  The groups run opposite phases, so on
// every SIMD one wave feeds the matrix core while the other runs the
// probability stage (a workgroup barrier every four phases re-aligns them):
//   phase 2j:    group 0 runs M(j),  group 1 runs V(j-1)
//   phase 2j+1:  group 0 runs V(j),  group 1 runs M(j)
// K(j) is read in phases 2j-1 .. 2j+1 (the first operands of a matrix phase
// are read in the VALU phase before it), V~(j) in phases 2j+1 and 2j+2.
// Both stream through LDS rings (schedule and ring depths at pp_schedule).
constexpr int kPPWaves = 8;
constexpr int kPPBr = kWaveQ * kPPWaves;   // queries per workgroup
constexpr int kPPThreads = 64 * kPPWaves;
#ifndef EFQ_KPRE
#define EFQ_KPRE 1                         // read K operands one phase early
#endif
#ifndef EFQ_PREFETCH
#define EFQ_PREFETCH (3 + EFQ_KPRE)
#endif
constexpr int kPP = EFQ_PREFETCH;          // tiles streamed ahead (>= 3)
constexpr int kPPK = kPP + 2;              // K ring depth
constexpr int kPPV = kPP + 3;              // V~ ring depth
constexpr int kBarPhases = 4;              // phases between workgroup barriers
// Wave priorities (s_setprio) of the two phases, per probability stage: the
// issue arbiter of a SIMD favours the wave whose work is on the critical
// path.  EFQ and LUT: the VALU phase (max, parameters, rescale) is the
// longer one; exp-then-quantize: the matrix phase carries its heavier code
// step.  Measured, not derived (both orders were timed).
#ifndef EFQ_PRIO_EFQ_M
#define EFQ_PRIO_EFQ_M 0
#endif
#ifndef EFQ_PRIO_EFQ_V
#define EFQ_PRIO_EFQ_V 3
#endif
#ifndef EFQ_PRIO_LUT_M
#define EFQ_PRIO_LUT_M 0
#endif
#ifndef EFQ_PRIO_LUT_V
#define EFQ_PRIO_LUT_V 3
#endif
#ifndef EFQ_PRIO_OTHER_M
#define EFQ_PRIO_OTHER_M 3
#endif
#ifndef EFQ_PRIO_OTHER_V
#define EFQ_PRIO_OTHER_V 0
#endif
#ifndef EFQ_KPRE_BF16
#define EFQ_KPRE_BF16 0                    // also on the bf16 Q K^T path
#endif
constexpr bool kKPre = EFQ_KPRE != 0;
constexpr int kKeep = kPP - 2 - (kKPre ? 1 : 0);   // batches left in flight at odd phases
static_assert(kKeep >= 0, "prefetch distance too short for the K pre-read");
template <int D, bool Q8 = false>
using SmemPP = Smem<D, kPPK, kPPV, Q8>;
// one workgroup per CU: the rings must fit the 160 KB of LDS
static_assert(SmemPP<128>::kTotal <= 160 * 1024 && SmemPP<128, true>::kTotal <= 160 * 1024,
              "K and V~ rings exceed the LDS of a CU");

// P~1 on the 16x16x128 FP4 MFMA.  Its B operand is the P~^T operand of the
// P~V product as it sits in the lanes (lane l: query l % 32, key block
// l / 32), read as a 128 x 16 matrix (lane l: column l % 16, K block l / 16).
// The A operand `sel` is 1.0 in row 4h of K block g when g and h have the
// same parity, 0 elsewhere; then row 4 (l / 16) of column l % 16, which lane
// l holds in element 0 of the result, is the sum over both key blocks of
// lane l's own query.  The other rows stay 0.
__device__ __forceinline__ i32x8 rowsum_selector(int lane) {
  const int m = lane & 15, g = lane >> 4;
  const int v = ((m & 3) == 0 && (g & 1) == ((m >> 2) & 1)) ? 0x22222222 : 0;
  return i32x8{v, v, v, v, 0, 0, 0, 0};
}

__device__ __forceinline__ f32x4 rowsum_mfma(const i32x8& sel, const i32x8& b8, const f32x4& l, int sb) {
  return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(sel, b8, l, 4, 4, 0, 127, 0, sb);
}

// Matrix phase of the ping-pong kernel.  With QK: S = K Q^T of one 64-key
// tile into (sn0, sn1), the LDS operand reads kept PD k-steps ahead.  With
// CODES: the per-score part of the probability stage of the previous tile
// (scores sc0, sc1, block parameters in st) runs on the VALU in the shadow
// of those MFMAs, one slice per k-step region (sched_barrier keeps the
// regions in order), then its P~V and P~1 MFMAs close the phase.
#ifndef EFQ_QK_PD
#define EFQ_QK_PD 3
#endif
constexpr int kQkPD = EFQ_QK_PD;   // bf16 K operand reads kept this many k-steps ahead
template <int D, int KIND, bool QK, int I>
__device__ __forceinline__ void mc_regions(lds_cptr p0, lds_cptr p1, bf16x8* a0,
                                           bf16x8* a1, const bf16x8* qreg, f32x16& sn0,
                                           f32x16& sn1, const f32x16& sc0, const f32x16& sc1,
                                           const PgenArgs& pa, PgenState& st) {
  constexpr int KK = D / 16;
  constexpr int PD = KK < kQkPD ? KK : kQkPD;
  if constexpr (I < KK) {
    if constexpr (QK) {
      sn0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0[I], qreg[I], sn0, 0, 0, 0);
      sn1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1[I], qreg[I], sn1, 0, 0, 0);
      if constexpr (I + PD < KK) {
        a0[I + PD] = *(__attribute__((address_space(3))) const bf16x8*)(p0 + (I + PD) * 1024);
        a1[I + PD] = *(__attribute__((address_space(3))) const bf16x8*)(p1 + (I + PD) * 1024);
      }
    }
    constexpr int P0 = 16 * I / KK, P1 = 16 * (I + 1) / KK;
    pg_pairs<KIND, 2 * P0, 2 * P1>(sc0, sc1, pa, st);
    if constexpr (QK && KIND == EFQ_PGEN_EFQ) {
      // EFQ: each MFMA, then one LDS operand read, then about half of the
      // region's code-step instructions (measured 1 % faster than the
      // compiler's own placement, which bunches them after the first MFMA;
      // the LUT and exp-then-quantize stages were 4-7 % slower with it)
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // MFMA
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // LDS read
      __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);   // VALU
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, 7, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    mc_regions<D, KIND, QK, I + 1>(p0, p1, a0, a1, qreg, sn0, sn1, sc0, sc1, pa, st);
  }
}

template <int D, bool Q8>
struct KPre;

// p0: the lane's operand slot in the K tile (tile base + 16 lane)
template <int D, int KIND, bool QK, bool CODES, bool PRE>
__device__ __forceinline__ PgenOut mma_phase(lds_cptr p0, const bf16x8* qreg,
                                             const KPre<D, false>& kp, f32x16& sn0,
                                             f32x16& sn1, const f32x16& sc0, const f32x16& sc1,
                                             const PgenArgs& pa, PgenState& st) {
  constexpr int KK = D / 16;
  constexpr int PD = KK < kQkPD ? KK : kQkPD;
  lds_cptr p1 = p0 + KK * 1024;
  bf16x8 a0[KK], a1[KK];
  if constexpr (QK) {
    if constexpr (PRE) {
      a0[0] = kp.a0;
      a1[0] = kp.a1;
    }
#pragma unroll
    for (int kk = PRE ? 1 : 0; kk < PD; ++kk) {
      a0[kk] = *(__attribute__((address_space(3))) const bf16x8*)(p0 + kk * 1024);
      a1[kk] = *(__attribute__((address_space(3))) const bf16x8*)(p1 + kk * 1024);
    }
    sn0 = f32x16{};
    sn1 = f32x16{};
  }
  __builtin_amdgcn_sched_barrier(0);
  PgenOut po{};
  if constexpr (CODES) {
    mc_regions<D, KIND, QK, 0>(p0, p1, a0, a1, qreg, sn0, sn1, sc0, sc1, pa, st);
    if constexpr (KIND == EFQ_PGEN_NOOP) asm volatile("" ::"v"(sc0), "v"(sc1));   // keep Q K^T live
    po = pg_finish<KIND>(st);
  } else {
    f32x16 z{};
    mc_regions<D, EFQ_PGEN_NOOP, QK, 0>(p0, p1, a0, a1, qreg, sn0, sn1, z, z, pa, st);
  }
  return po;
}

// Q operand of the Q K^T MFMAs, held in registers for the whole kernel:
// bf16 (B operand of the 32x32x16 MFMA, 8 columns per k-step), or MXFP8
// (B operand of the FP8 32x32x64 MFMA per 64-column chunk, and in byte c of
// `sc` the E8M0 scale the lane supplies for chunk c).
template <int D, bool Q8>
struct QOps {
  bf16x8 r[D / 16];
};
template <int D>
struct QOps<D, true> {
  i32x8 a[D / 64];
  int sc;
};

// The E8M0 scale of 32 columns of a row that lane (row, half) supplies to
// the FP8 MFMA of chunk c is that of columns 64 c + 32 half + [0, 32): from
// the row's D/32 scale bytes `raw`, byte c of the result is byte 2 c + half.
template <int D>
__device__ __forceinline__ int lane_scales(unsigned raw, int half) {
  const unsigned x = raw >> (8 * half);
  if constexpr (D == 128) return (int)((x & 0xffu) | ((x >> 8) & 0xff00u));
  else return (int)(x & 0xffu);
}

// A operand (K rows of window I % 2, chunk I / 2) of MXFP8 region I from an
// LDS K tile, and the lane's K scales of window w.
template <int D>
__device__ __forceinline__ i32x8 k8_operand(const uint8_t* kb, int lane, int region) {
  constexpr int NC = D / 64;
  const uint8_t* p = kb + (((region & 1) * NC + (region >> 1)) * 2) * 1024 + lane * 16;
  const u32x4 lo = *(const u32x4*)p;
  const u32x4 hi = *(const u32x4*)(p + 1024);
  return i32x8{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3],
               (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
}

template <int D>
__device__ __forceinline__ int k8_scales(const uint8_t* kb, int lane, int w) {
  const int key = 32 * w + (lane & 31);
  const uint8_t* sp = kb + kBc * D;
  unsigned raw;
  if constexpr (D == 128) raw = *(const unsigned*)(sp + key * 4);
  else raw = *(const unsigned short*)(sp + key * 2);
  return lane_scales<D>(raw, lane >> 5);
}

// Matrix phase with MXFP8 Q and K: S = K Q^T of one 64-key tile on the FP8
// MFMA with E8M0 block scales, one MFMA per region (window I % 2, chunk
// I / 2, alternating windows so consecutive MFMAs are independent), the LDS
// operand reads PD regions ahead; the code slices of the previous tile are
// spread over the regions as in the bf16 path.
template <int D, int KIND, bool QK, int I>
__device__ __forceinline__ void mc_regions8(const uint8_t* kb, int lane, i32x8* ka,
                                            const QOps<D, true>& qo, int ks0, int ks1,
                                            f32x16& sn0, f32x16& sn1, const f32x16& sc0,
                                            const f32x16& sc1, const PgenArgs& pa,
                                            PgenState& st) {
  constexpr int R = D / 32;
  constexpr int PD = R < 2 ? R : 2;
  if constexpr (I < R) {
    if constexpr (QK) {
      constexpr int C = I >> 1;
      if constexpr ((I & 1) == 0)
        sn0 = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(ka[I], qo.a[C], sn0, 0, 0, C, ks0, C, qo.sc);
      else
        sn1 = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(ka[I], qo.a[C], sn1, 0, 0, C, ks1, C, qo.sc);
      if constexpr (I + PD < R) ka[I + PD] = k8_operand<D>(kb, lane, I + PD);
    }
    constexpr int P0 = 16 * I / R, P1 = 16 * (I + 1) / R;
    pg_pairs<KIND, 2 * P0, 2 * P1>(sc0, sc1, pa, st);
    __builtin_amdgcn_sched_barrier(0);
    mc_regions8<D, KIND, QK, I + 1>(kb, lane, ka, qo, ks0, ks1, sn0, sn1, sc0, sc1, pa, st);
  }
}

// K operands of the first Q K^T MFMAs of a tile, read from LDS in the VALU
// phase before its matrix phase, so the matrix phase starts without waiting
// for LDS: bf16, the first k-step of both windows; MXFP8, the first two
// regions and both windows' scales.
template <int D, bool Q8>
struct KPre {
  bf16x8 a0, a1;
  __device__ __forceinline__ void read(const uint8_t* kb, int lane) {
    a0 = *(const bf16x8*)(kb + lane * 16);
    a1 = *(const bf16x8*)(kb + lane * 16 + (D / 16) * 1024);
  }
};
template <int D>
struct KPre<D, true> {
  i32x8 k0, k1;   // regions 0 and 1
  int ks0, ks1;
  __device__ __forceinline__ void read(const uint8_t* kb, int lane) {
    k0 = k8_operand<D>(kb, lane, 0);
    k1 = k8_operand<D>(kb, lane, 1);
    ks0 = k8_scales<D>(kb, lane, 0);
    ks1 = k8_scales<D>(kb, lane, 1);
  }
};

template <int D, int KIND, bool QK, bool CODES, bool PRE>
__device__ __forceinline__ PgenOut mma_phase8(const uint8_t* kbuf, const QOps<D, true>& qo,
                                              const KPre<D, true>& kp, int lane, f32x16& sn0,
                                              f32x16& sn1, const f32x16& sc0, const f32x16& sc1,
                                              const PgenArgs& pa, PgenState& st) {
  constexpr int R = D / 32;
  constexpr int PD = R < 2 ? R : 2;
  static_assert(PD == 2, "the pre-read covers the first two regions");
  i32x8 ka[R];
  int ks0 = 0, ks1 = 0;
  if constexpr (QK) {
    if constexpr (PRE) {
      ka[0] = kp.k0;
      ka[1] = kp.k1;
      ks0 = kp.ks0;
      ks1 = kp.ks1;
    } else {
#pragma unroll
      for (int i = 0; i < PD; ++i) ka[i] = k8_operand<D>(kbuf, lane, i);
      ks0 = k8_scales<D>(kbuf, lane, 0);
      ks1 = k8_scales<D>(kbuf, lane, 1);
    }
    sn0 = f32x16{};
    sn1 = f32x16{};
  }
  __builtin_amdgcn_sched_barrier(0);
  PgenOut po{};
  if constexpr (CODES) {
    mc_regions8<D, KIND, QK, 0>(kbuf, lane, ka, qo, ks0, ks1, sn0, sn1, sc0, sc1, pa, st);
    if constexpr (KIND == EFQ_PGEN_NOOP) asm volatile("" ::"v"(sc0), "v"(sc1));
    po = pg_finish<KIND>(st);
  } else {
    f32x16 z{};
    mc_regions8<D, EFQ_PGEN_NOOP, QK, 0>(kbuf, lane, ka, qo, ks0, ks1, sn0, sn1, z, z, pa, st);
  }
  return po;
}

template <int D, int KIND, bool DUMP, bool Q8, bool PREREAD>
struct PPWave {
  static constexpr int NS = D / 32;
  QOps<D, Q8> qo;
  f32x16 oacc[NS];
  f32x4 lacc;             // element 0: the lane's row sum l
  i32x8 sel;              // A operand of the P~1 MFMA
  float m;
  PgenArgs pa;
  PgenState st;           // block parameters of the tile between V(j) and M(j+1)
  int lane, half, my_q;
  int vis_end4;           // visible keys of the lane's query, less 4 half
  int vis_min;            // wave-uniform minimum of the visible key counts
  unsigned klane;         // LDS address of the lane's K operand read in K slot 0
  unsigned vlane, vslane; // of its V~ code and scale reads in V~ slot 0
  // the pre-read needs registers the bf16 exp-then-quantize variants lack
  static constexpr bool kPreOn = PREREAD && kKPre && (Q8 || EFQ_KPRE_BF16);
  static constexpr int kMPrio = KIND == EFQ_PGEN_EFQ ? EFQ_PRIO_EFQ_M
                                : KIND == EFQ_PGEN_LUT ? EFQ_PRIO_LUT_M
                                : KIND == EFQ_PGEN_NOOP ? 0 : EFQ_PRIO_OTHER_M;
  static constexpr int kVPrio = KIND == EFQ_PGEN_EFQ ? EFQ_PRIO_EFQ_V
                                : KIND == EFQ_PGEN_LUT ? EFQ_PRIO_LUT_V
                                : KIND == EFQ_PGEN_NOOP ? 0 : EFQ_PRIO_OTHER_V;
  // The P~V and P~1 MFMAs have no memory effects, so the compiler may sink
  // them past the phase barrier into the VALU phase, next to their first
  // use.  On the FP8 Q K^T path every stage issues them in the matrix phase
  // instead (an empty asm reads their results there); every stage on the
  // bf16 path keeps the compiler's placement.  Measured, both ways.
  static constexpr bool kPvFence = Q8;

  // Matrix phase M(j): with QK the scores of tile j into sn, and with CODES
  // the codes of tile j-1 (scores sc) in the shadow of those MFMAs, then its
  // P~V and P~1 MFMAs.  PRE: the first K operands are in kp.
  // kr: byte offset of the K ring slot holding tile j (with QK).
  template <bool QK, bool CODES, bool PRE>
  __device__ __forceinline__ void mphase(int j, const uint8_t* kbuf0, int kr, const VOps<D>& vop,
                                         const KPre<D, Q8>& kp, const AttnArgs& a, int b, int hq,
                                         f32x16& sn0, f32x16& sn1, const f32x16& sc0,
                                         const f32x16& sc1) {
    if constexpr (kMPrio != kVPrio) __builtin_amdgcn_s_setprio(kMPrio);
    constexpr bool P = PRE && kPreOn;
    PgenOut po;
    if constexpr (Q8)
      po = mma_phase8<D, KIND, QK, CODES, P>(kbuf0 + kr, qo, kp, lane, sn0, sn1, sc0, sc1, pa, st);
    else
      po = mma_phase<D, KIND, QK, CODES, P>(lds_at(klane + kr), qo.r, kp, sn0, sn1, sc0, sc1,
                                            pa, st);
    if constexpr (CODES) {
      if constexpr (DUMP) {
        const int blk = 2 * (j - 1) + half;
        if (my_q < a.Sq && blk < a.nblk) {
          long row = ((long)b * a.Hq + hq) * a.Sq + my_q;
          *(u32x4*)(a.p_codes + (row * a.nblk + blk) * 16) = unpermute_codes(po.bop);
          a.p_e8m0[row * a.nblk + blk] = (uint8_t)po.scale_b;
        }
      }
      const i32x8 b8 = i32x8{(int)po.bop[0], (int)po.bop[1], (int)po.bop[2], (int)po.bop[3], 0, 0, 0, 0};
      pv_slabs<NS>(oacc, vop, b8, po.scale_b);
      lacc = rowsum_mfma(sel, b8, lacc, po.scale_b);
#if defined(__HIP_DEVICE_COMPILE__)
      if constexpr (kPvFence) {
#pragma unroll
        for (int s = 0; s < NS; ++s) asm volatile("" ::"v"(oacc[s]));
        asm volatile("" ::"v"(lacc));
      }
#endif
    }
  }

  // VALU phase V(j): read the V~(j) operands for the next matrix phase (and
  // the first K operands of tile j+1: after the last tile the read lands in
  // an unused slot and its values are never used), mask the scores of tile
  // j (diagonal and ragged tiles only), take the block and row maxima and
  // the block parameters (row maximum, alpha, k_b, bias), and rescale the
  // history when a row maximum moved.  The reads are unconditional so the
  // operands stay in registers.
  // vr: byte offset of the V~ ring slot of tile j; krn: of the K slot of
  // tile j+1.
  __device__ __forceinline__ void vphase(int j, const uint8_t* vbuf0, int vr, const uint8_t* kbuf0,
                                         int krn, f32x16& s0, f32x16& s1, VOps<D>& vop,
                                         KPre<D, Q8>& kp, int mask_from) {
    if constexpr (kMPrio != kVPrio) __builtin_amdgcn_s_setprio(kVPrio);
    if constexpr (kPreOn) kp.read(kbuf0 + krn, lane);
    read_v<D>(lds_at(vlane + vr), lds_at(vslane + vr), vop);
    // some lane's visible keys end inside this tile
    if (j >= mask_from)
      mask_tile(s0, s1, vis_end4 - j * kBc);
    float pm0, pm1;
    pg_max<KIND>(s0, s1, pm0, pm1);
    if (pg_params<KIND>(pm0, pm1, m, pa, st)) {
      const float alpha = pg_alpha<KIND>(st);
#pragma unroll
      for (int s = 0; s < NS; ++s) oacc[s] *= alpha;
      lacc[0] *= alpha;
    }
  }
};

// The per-wave schedule of the ping-pong kernel.  A wave with T tiles runs
// M(0) V(0) M(1) V(1) ... M(T-1) V(T-1) F, where M(j) also codes tile j-1
// and applies its P~V (j >= 1) and F codes and applies the last tile; group
// G runs op o in phase o + G.  K(j) is read in phases 2j-1 .. 2j+1 (V(j-1)
// reads the first operands of M(j) with the K pre-read, else from 2j on)
// and V~(j) in phases 2j+1, 2j+2.  Even phases t = 2j >= 2 stream tile j+P
// (K and V~; past the last tile the last one again, into the slot tile j+P
// would take, so every wave issues the same loads in every even phase);
// odd phases end by waiting until only the loads of the last E even phases
// are outstanding (loads complete in order), E = P-3 with the pre-read,
// else P-2; phases 4k+3 then end with a workgroup barrier (waves between
// two barriers are unordered).  A load issued in phase 2j has landed by the
// end of phase 2(j+P-E)-1, with the pre-read (P = 4, E = 1) 2(j+P)-5, and
// the next barrier, at the end of phase 2(j+P)-5 or 2(j+P)-3, precedes the
// pre-read of K(j+P) in phase 2(j+P)-1.  The slots it overwrites (K(j-2) in
// a ring of P+2, V~(j-3) in a ring of P+3) were last read, and the reads
// consumed, by phase 2j-3, before a barrier that precedes phase 2j.  Fewer
// barriers let the groups drift within four phases; each one dropped
// measured 1-6 % faster than a barrier per phase.  Every wave runs
// 2 ntiles + 2 phases, so all pass the same barriers.  Scores alternate
// between two register sets.  The phase index modulo 4 is a compile-time
// constant in the tile loop, so its phase ends compile to straight-line
// code; ring slots advance by one tile per phase pair.
template <int X>
using IC = std::integral_constant<int, X>;

template <int STEP, int DEPTH>
__device__ __forceinline__ int ring_next(int off) {
  off += STEP;
  return off == STEP * DEPTH ? 0 : off;
}

#if EFQ_PHASE_STAMPS
__device__ unsigned long long* g_stamps;   // [kStampBlocks][2 groups][kStampSlots]
#endif

template <int G, int D, int KIND, bool DUMP, bool Q8, typename Stream>
__device__ __forceinline__ void pp_schedule(PPWave<D, KIND, DUMP, Q8, true>& w, int T, int ntiles,
                                            const uint8_t* kbuf0, const uint8_t* vbuf0,
                                            const AttnArgs& a, int b, int hq, int keep,
                                            Stream& stream) {
  using Sm = SmemPP<D, Q8>;
  f32x16 sa0, sa1, sb0, sb1;
  VOps<D> vop;
  KPre<D, Q8> kp;      // first K operands of the next matrix phase
  int kr = 0;          // K slot of the next matrix phase with Q K^T
  int vr = 0;          // V~ slot of the next VALU phase
  auto knext = [](int x) { return ring_next<Sm::kK, kPPK>(x); };
  auto vnext = [](int x) { return ring_next<Sm::kV, kPPV>(x); };
  // The tile loads go out after the even phase's work, not before it, on
  // the bf16 path (measured 1.5 % faster) and for EFQ on the MXFP8 path
  // (2.8 %); the other MXFP8 stages are as fast or faster with them first.
  // Either way they belong to phase t, as the schedule assumes.
  constexpr bool kLate = !Q8 || KIND == EFQ_PGEN_EFQ;
  // Phase t with TM = t % 4 known (even TM only for t >= 2); TM = 4 is t = 0.
  auto begin = [&](auto tm) {
    constexpr int TM = decltype(tm)::value;
    if constexpr (!kLate && (TM == 0 || TM == 2)) stream();
  };
#if EFQ_PHASE_STAMPS
  unsigned long long* const stamp =
      (unsigned long long*)(const_cast<uint8_t*>(kbuf0) + Sm::kStampOff) + G * kStampSlots;
  const bool stamper = (threadIdx.x & 255) == 0;   // lane 0 of waves 0 and 4 (SIMD 0)
  int ph = 0;
#endif
  auto end = [&](auto tm) {
    constexpr int TM = decltype(tm)::value;
#if EFQ_PHASE_STAMPS
    if (stamper && ph < kStampPhases) stamp[2 * ph] = __builtin_amdgcn_s_memtime();
#endif
    if constexpr (kLate && (TM == 0 || TM == 2)) {
      __builtin_amdgcn_sched_barrier(0);
      stream();
    }
    if constexpr (TM == 1 || TM == 3) {
      // the batches of the last kKeep even phases may stay in flight
      wait_vmem_le(keep);
      if constexpr (TM == 3) wg_barrier();
      else __builtin_amdgcn_sched_barrier(0);
    } else {
      __builtin_amdgcn_sched_barrier(0);
    }
#if EFQ_PHASE_STAMPS
    if (stamper && ph < kStampPhases) {
      const unsigned long long mt = __builtin_amdgcn_s_memtime();
      const unsigned long long rt = __builtin_amdgcn_s_memrealtime();
      stamp[2 * ph + 1] = mt;
      unsigned long long* const clk = stamp + 2 * kStampPhases + (ph == 0 ? 0 : 2);
      clk[0] = mt;
      clk[1] = rt;
    }
    ++ph;
#endif
  };
  constexpr int TA = (2 + G) & 3, TB = (3 + G) & 3, TC = G, TD = (1 + G) & 3;
  // first tile in which some lane of the wave has keys past its visible
  // ones ((j + 1) kBc > the wave's smallest visible-key count); uniform, so
  // the test in every VALU phase is a scalar compare
  const int mask_from = __builtin_amdgcn_readfirstlane(w.vis_min) / kBc;
  // M(0), V(0) (group 1 after an empty phase); every later M(j) with Q K^T
  // follows a V(j-1) that pre-read its first K operands (j < T)
  if constexpr (G == 0) {
    begin(IC<4>{}); w.template mphase<true, false, false>(0, kbuf0, kr, vop, kp, a, b, hq, sa0, sa1, sb0, sb1); end(IC<4>{});
    kr = knext(kr);
    begin(IC<1>{}); w.vphase(0, vbuf0, vr, kbuf0, kr, sa0, sa1, vop, kp, mask_from); end(IC<1>{});
  } else {
    begin(IC<4>{}); end(IC<4>{});
    begin(IC<1>{}); w.template mphase<true, false, false>(0, kbuf0, kr, vop, kp, a, b, hq, sa0, sa1, sb0, sb1); end(IC<1>{});
    kr = knext(kr);
    begin(IC<2>{}); w.vphase(0, vbuf0, vr, kbuf0, kr, sa0, sa1, vop, kp, mask_from); end(IC<2>{});
  }
  vr = vnext(vr);
  int j = 1;
  for (; j + 1 < T; j += 2) {
    begin(IC<TA>{}); w.template mphase<true, true, true>(j, kbuf0, kr, vop, kp, a, b, hq, sb0, sb1, sa0, sa1); end(IC<TA>{});
    kr = knext(kr);
    begin(IC<TB>{}); w.vphase(j, vbuf0, vr, kbuf0, kr, sb0, sb1, vop, kp, mask_from); end(IC<TB>{});
    vr = vnext(vr);
    begin(IC<TC>{}); w.template mphase<true, true, true>(j + 1, kbuf0, kr, vop, kp, a, b, hq, sa0, sa1, sb0, sb1); end(IC<TC>{});
    kr = knext(kr);
    begin(IC<TD>{}); w.vphase(j + 1, vbuf0, vr, kbuf0, kr, sa0, sa1, vop, kp, mask_from); end(IC<TD>{});
    vr = vnext(vr);
  }
  if (j < T) {   // one more tile: its scores go to set b, the last coded from b
    begin(IC<TA>{}); w.template mphase<true, true, true>(j, kbuf0, kr, vop, kp, a, b, hq, sb0, sb1, sa0, sa1); end(IC<TA>{});
    kr = knext(kr);
    begin(IC<TB>{}); w.vphase(j, vbuf0, vr, kbuf0, kr, sb0, sb1, vop, kp, mask_from); end(IC<TB>{});
    begin(IC<TC>{}); w.template mphase<false, true, false>(T, kbuf0, kr, vop, kp, a, b, hq, sa0, sa1, sb0, sb1); end(IC<TC>{});
  } else {       // the last tile's scores are in set a
    begin(IC<TA>{}); w.template mphase<false, true, false>(T, kbuf0, kr, vop, kp, a, b, hq, sb0, sb1, sa0, sa1); end(IC<TA>{});
  }
  // empty phases until the workgroup's last tile (the phase index is known
  // only at run time here)
  for (int t = 2 * T + 1 + G; t < 2 * ntiles + 2; ++t) {
    if ((t & 1) == 0) {
      stream();
      __builtin_amdgcn_sched_barrier(0);
    } else {
      wait_vmem_le(keep);
      if ((t & 3) == 3) wg_barrier();
      else __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// ------------------------------------------------------- half workgroup
// Four waves (128 queries, one wave per SIMD) and LDS rings small enough for
// two workgroups on a CU, so the second wave of every SIMD belongs to another
// workgroup, in another part of its work.  Bound by the latency of a tile's
// chain (M then V, ~2100 cycles for a wave alone on its SIMD, ~2450 for two)
// and, with few keys, by the loads and stores around it, which the other
// workgroup's tiles cover.  Against the eight-wave kernel the K and V~ tiles
// are read twice as often and a tile costs 3-6 % more in the steady state;
// it wins where that kernel leaves CUs idle or its workgroups are short
// (use_half).  Kernel time, EFQ, 32/8 heads, D 128 causal, eight waves ->
// this: 512 tokens 17.9 -> 12.7 us, 2048 tokens 44.3 -> 38.2 us, 16 prompts
// of 333 tokens 59.0 -> 44.6 us; 8192 tokens 354 -> 366 us.
constexpr int kHWaves = 4;
constexpr int kHP = 2;                     // tiles streamed ahead
constexpr int kHK = kHP + 1;               // K ring depth
constexpr int kHV = kHP + 2;               // V~ ring depth
template <int D, bool Q8 = false>
using SmemH = Smem<D, kHK, kHV, Q8, false>;
// LDS of a half workgroup: the rings, or at the end its O rows
template <int D, bool Q8>
constexpr int half_lds() {
  return std::max(SmemH<D, Q8>::kTotal, kHWaves * kWaveQ * D * 4);
}
static_assert(2 * half_lds<128, false>() <= 160 * 1024 && 2 * half_lds<128, true>() <= 160 * 1024,
              "two half workgroups exceed the LDS of a CU");

// The schedule of a wave of a half workgroup.  Iteration j runs M(j) (with
// the codes and P~V of tile j-1) and V(j), streams tile j+P, waits until tile
// j+1 has landed (the loads of the P-1 tiles after it may stay in flight)
// and ends with a workgroup barrier.  Tile x is read only in iteration x (K
// by M(x), V~ by V(x)), after the barrier that follows every wave's landing
// wait for it.  The slots tile j+P overwrites held K(j-1) in a ring of P+1,
// read and consumed in iteration j-1, and V~(j-2) in a ring of P+2, read in
// iteration j-2 and consumed by M(j-1) (or F) before the barrier of iteration
// j-1.  Every wave runs ntiles iterations, so all pass the same barriers;
// past the last tile the last one is streamed again, so the wait is a
// constant.
template <int D, int KIND, bool Q8, int LOADS, typename Stream>
__device__ __forceinline__ void half_schedule(PPWave<D, KIND, false, Q8, false>& w, int T, int ntiles,
                                              const uint8_t* kbuf0, const uint8_t* vbuf0,
                                              const AttnArgs& a, Stream& stream) {
  using Sm = SmemH<D, Q8>;
  f32x16 sa0, sa1, sb0, sb1;
  VOps<D> vop;
  KPre<D, Q8> kp;
  int kr = 0, vr = 0;
  const int mask_from = __builtin_amdgcn_readfirstlane(w.vis_min) / kBc;
  auto end = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    stream();
    kr = ring_next<Sm::kK, kHK>(kr);
    vr = ring_next<Sm::kV, kHV>(vr);
    wait_vmem_le((kHP - 1) * LOADS);
    wg_barrier();
  };
  w.template mphase<true, false, false>(0, kbuf0, kr, vop, kp, a, 0, 0, sa0, sa1, sb0, sb1);
  w.vphase(0, vbuf0, vr, kbuf0, kr, sa0, sa1, vop, kp, mask_from);
  end();
  int j = 1;
  for (; j + 1 < T; j += 2) {
    w.template mphase<true, true, false>(j, kbuf0, kr, vop, kp, a, 0, 0, sb0, sb1, sa0, sa1);
    w.vphase(j, vbuf0, vr, kbuf0, kr, sb0, sb1, vop, kp, mask_from);
    end();
    w.template mphase<true, true, false>(j + 1, kbuf0, kr, vop, kp, a, 0, 0, sa0, sa1, sb0, sb1);
    w.vphase(j + 1, vbuf0, vr, kbuf0, kr, sa0, sa1, vop, kp, mask_from);
    end();
  }
  if (j < T) {   // one more tile: its scores go to set b, the last coded from b
    w.template mphase<true, true, false>(j, kbuf0, kr, vop, kp, a, 0, 0, sb0, sb1, sa0, sa1);
    w.vphase(j, vbuf0, vr, kbuf0, kr, sb0, sb1, vop, kp, mask_from);
    end();
    w.template mphase<false, true, false>(T, kbuf0, kr, vop, kp, a, 0, 0, sa0, sa1, sb0, sb1);
  } else {       // the last tile's scores are in set a
    w.template mphase<false, true, false>(T, kbuf0, kr, vop, kp, a, 0, 0, sb0, sb1, sa0, sa1);
  }
  for (int t = T; t < ntiles; ++t) end();
}

// Q rows and O rows of a half workgroup's wave pass through LDS, so that its
// global loads and stores cover whole rows (1 KB of 2 to 8 rows an
// instruction); in the operand layout an instruction touches 32 rows, 32
// bytes each, and the address unit takes a cycle per row: 20 such
// instructions a wave before the first tile kept it busy for 4000 to 7000
// cycles.  16-byte chunk c of row r sits in slot c ^ (r mod 16) of its row
// (r / 2 mod 8 for the 8 chunks of a bf16 D = 64 row), so that the reads and
// writes along a column hit different banks.  Kernel time before
// and after: 8 prompts of 333 tokens 25.9 -> 23.9 us (O direct 24.1), 32760 x
// 512 keys 253.6 -> 232.6 (Q only 244.5, O only 236.3), x 128 keys 167.6 ->
// 141.5.
template <int D>
__device__ __forceinline__ int q_swizzle(int row) {
  return D == 128 ? row & 15 : (row >> 1) & 7;
}

// The wave's 32 rows from q_wave0 (past Sq: row Sq - 1) into LDS at qb.
template <int D>
__device__ __forceinline__ void half_issue_q(const unsigned short* __restrict__ q, long stride, int q_wave0,
                                             int Sq, int lane, uint8_t* qb) {
  constexpr int C = D / 8, RPI = 64 / C;   // chunks a row, rows an instruction
#pragma unroll
  for (int i = 0; i < kWaveQ / RPI; ++i) {
    const int row = i * RPI + lane / C;
    const unsigned short* p =
        q + min(q_wave0 + row, Sq - 1) * stride + ((lane % C) ^ q_swizzle<D>(row)) * 8;
    __builtin_amdgcn_global_load_lds((__attribute__((address_space(1))) const void*)p,
                                     (__attribute__((address_space(3))) void*)(qb + i * 1024), 16, 0, 0);
  }
}

template <int D>
__device__ __forceinline__ void half_read_q(const uint8_t* qb, int lane, bf16x8* r) {
  const int row = lane & 31;
  const uint8_t* p = qb + row * (D * 2);
  const int x = q_swizzle<D>(row) ^ (lane >> 5);
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk) r[kk] = *(const bf16x8*)(p + ((2 * kk) ^ x) * 16);
}

// The wave's 32 x D outputs (accumulators times rl) as rows: f(row, d, v) for
// four outputs from column d of row `row`, whole rows of lanes at a time; ob:
// 128 D bytes of LDS of the wave's own.
template <int D, typename F>
__device__ __forceinline__ void half_rows(const f32x16* oacc, float rl, int lane, uint8_t* ob, F&& f) {
  constexpr int C = D / 4, RPI = 64 / C;
  const int x = (lane & 15) ^ (lane >> 5);
  uint8_t* const wp = ob + (lane & 31) * (D * 4);
#pragma unroll
  for (int s = 0; s < D / 32; ++s)
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4)
      *(f32x4*)(wp + ((8 * s + 2 * r4) ^ x) * 16) =
          f32x4{oacc[s][4 * r4] * rl, oacc[s][4 * r4 + 1] * rl, oacc[s][4 * r4 + 2] * rl, oacc[s][4 * r4 + 3] * rl};
  // a wave's LDS operations complete in order
  asm volatile("" ::: "memory");
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int i = 0; i < 32 / RPI; ++i) {
    const int row = i * RPI + lane / C;
    f(row, ((lane % C) ^ (row & 15)) * 4, *(const f32x4*)(ob + i * 1024 + lane * 16));
  }
}

constexpr int kRhoCand = 64;
// Calibration candidates of one launch (grid y), the reference output and the
// objective's partial sums.
struct RhoArgs {
  const float* o_ref;
  double* part;       // [candidate][workgroup][2]
  float tau[kRhoCand], h[kRhoCand];
};
struct NoRho {};

// The attention kernel: NW = 8 waves in the ping-pong schedule, or NW = 4 in
// the half workgroup's.  (One kernel template, not a body shared by several
// kernels: inlined into a wrapper, the compiler allocates the tile loop's
// registers differently, 0.6 % slower at 32K.)
// Q8: q and k are the MXFP8 buffers Q^ and K^ (E4M3 codes, then E8M0 scales
// at a.q8_soff / a.k8_soff, [batch][head][padded seq] rows), else bf16 BSHD.
// RHO: instead of storing O, the sums of (O - o_ref)^2 and o_ref^2 over the
// workgroup's outputs, in fp64 and a fixed order, go to rho.part.
template <int D, int KIND, bool CAUSAL, bool DUMP, bool Q8, int NW, bool RHO>
__global__ __attribute__((amdgpu_flat_work_group_size(64 * NW, 64 * NW), amdgpu_waves_per_eu(2, 2))) void
attn_pp_kernel(const void* __restrict__ q, const void* __restrict__ k,
               const uint8_t* __restrict__ vhat, float* __restrict__ out, AttnArgs a,
               std::conditional_t<RHO, RhoArgs, NoRho> rho) {
  extern __shared__ __align__(16) uint8_t smem[];
  constexpr bool kPair = NW == kPPWaves;     // the ping-pong schedule
  constexpr int kBr = kWaveQ * NW;           // queries per workgroup
  constexpr int KK = D / 16;
  constexpr int NS = D / 32;
  using Sm = std::conditional_t<kPair, SmemPP<D, Q8>, SmemH<D, Q8>>;

  int b, hq, qt;
  map_work<!kPair && CAUSAL>(a, b, hq, qt);
  const int g = hq / (a.Hq / a.Hkv);
  // wave index as a uniform (scalar) value: the group branch below is uniform
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  PPWave<D, KIND, DUMP, Q8, kPair> w;
  w.lane = threadIdx.x & 63;
  w.half = w.lane >> 5;
  const int q_wave0 = qt * kBr + wave * kWaveQ;
  w.my_q = q_wave0 + (w.lane & 31);
  const int q_load = w.my_q < a.Sq ? w.my_q : a.Sq - 1;
  if constexpr (Q8) {
    const uint8_t* qh = (const uint8_t*)q;
    const long row = ((long)b * a.Hq + hq) * a.sq_pad + q_load;
    const uint8_t* qp = qh + row * D + 16 * w.half;
#pragma unroll
    for (int c = 0; c < D / 64; ++c) {
      const u32x4 lo = *(const u32x4*)(qp + 64 * c);
      const u32x4 hi = *(const u32x4*)(qp + 64 * c + 32);
      w.qo.a[c] = i32x8{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3],
                        (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
    }
    const uint8_t* sp = qh + a.q8_soff + row * (D / 32);
    unsigned raw;
    if constexpr (D == 128) raw = *(const unsigned*)sp;
    else raw = *(const unsigned short*)sp;
    w.qo.sc = lane_scales<D>(raw, w.half);
  } else if constexpr (!kPair) {
    // whole rows to LDS (K slots 1 and 2, tile 1 comes later); the operands
    // are read once they have landed
    half_issue_q<D>((const unsigned short*)q + ((long)b * a.Sq * a.Hq + hq) * D, (long)a.Hq * D, q_wave0,
                    a.Sq, w.lane, smem + Sm::kK + wave * (kWaveQ * D * 2));
  } else {
    const unsigned short* qp =
        (const unsigned short*)q + (((long)b * a.Sq + q_load) * a.Hq + hq) * D + w.half * 8;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) w.qo.r[kk] = *(const bf16x8*)(qp + kk * 16);
  }
  // tiles of the workgroup and of this wave (1 <= wtiles <= ntiles)
  const int kv_end = CAUSAL ? min(a.Sk, qt * kBr + kBr) : a.Sk;
  const int wave_end = CAUSAL ? min(a.Sk, q_wave0 + kWaveQ) : a.Sk;
  const int ntiles = (kv_end + kBc - 1) / kBc;
  const int wtiles = (wave_end + kBc - 1) / kBc;
  w.vis_end4 = (CAUSAL ? min(a.Sk, w.my_q + 1) : a.Sk) - 4 * w.half;
  // lane 0 holds the wave's first query, whose visible range is the shortest
  w.vis_min = __builtin_amdgcn_readfirstlane(CAUSAL ? min(a.Sk, q_wave0 + 1) : a.Sk);
  uint8_t* const kbuf0 = smem + Sm::kKOff;
  uint8_t* const vbuf0 = smem + Sm::kVOff;
  // the lane's LDS read addresses in ring slot 0 stay in registers across
  // the loop instead of being recomputed from the lane index in every phase
  w.klane = lds_addr(kbuf0 + w.lane * 16);
  w.vlane = lds_addr(vbuf0 + vop_offset<D>(w.lane));
  w.vslane = lds_addr(vbuf0 + vscale_offset<D>(w.lane));
  asm volatile("" : "+v"(w.klane), "+v"(w.vlane), "+v"(w.vslane));

  std::conditional_t<Q8, KLoad8<D, NW>, KLoad<D, NW>> kload;
  if constexpr (Q8) {
    const uint8_t* kh = (const uint8_t*)k;
    const long hrow = ((long)b * a.Hkv + g) * a.sk_pad;
    kload.init(kh + hrow * D, kh + a.k8_soff + hrow * (D / 32), a.sk_pad, wave, w.lane);
  } else {
    kload.init((const unsigned short*)k + (long)b * a.Sk * a.Hkv * D, a.Sk, a.Hkv, g, wave, w.lane);
  }
  using VL = VLoad<D, NW>;
  VL vload;
  vload.init(vhat + ((long)b * a.Hkv + g) * a.nb * D * 16,
             vhat + a.scale_off + ((long)b * a.Hkv + g) * a.nb * D, a.nb, w.lane);
  asm volatile("" : "+v"(vload.coff_lane), "+v"(vload.soff_lane));

  w.pa.scale = a.scale;
  float tau = a.tau, h = a.h;
  if constexpr (RHO) {
    tau = rho.tau[blockIdx.y];
    h = rho.h[blockIdx.y];
  }
  w.pa.sh = a.scale * h;
  w.pa.sh32 = 32.0f * w.pa.sh;
  w.pa.sh16 = 16.0f * w.pa.sh;
  w.pa.c = kLn6 + tau;
  w.pa.negh = -h;
  w.pa.l2s = a.scale * kInvLn2;
#pragma unroll
  for (int s = 0; s < NS; ++s) w.oacc[s] = f32x16{};
  w.lacc = f32x4{0.f, 0.f, 0.f, 0.f};
  w.sel = rowsum_selector(w.lane);
  w.m = -INFINITY;

  // Streams tile x into the ring slots at byte offsets kofs, vofs: K (or
  // K^ codes and scales) and V~ codes and scales.  Every wave issues kLoads
  // loads: its K blocks and one V~ code block, or, where a wave has fewer,
  // a copy of a scale load (several waves write the same bytes to the same
  // place); the four waves of a half workgroup all load the scales too.
  // Past the last tile (x >= ntiles) the last tile is loaded again, so the
  // count never changes and the waits are constants.
  constexpr int kLoads = Q8 ? (kPair ? 2 : KLoad8<D, NW>::PER + 3)
                            : KLoad<D, NW>::kIssued + (kPair ? 1 : 2);
  auto load_tile = [&](int x, int kofs, int vofs) {
    const int xt = x < ntiles ? x : ntiles - 1;
    uint8_t* const kb = kbuf0 + kofs;
    uint8_t* const vb = vbuf0 + vofs;
    if constexpr (!kPair) {
      if constexpr (Q8) {
        kload.issue_codes(kb, xt, wave);
        kload.issue_scales(kb, xt, w.lane);
      } else {
        kload.issue(kb, xt, wave);
      }
      if (wave < VL::NB) vload.issue_codes(vb, xt, wave);
      else vload.issue_scales(vb, xt);
      vload.issue_scales(vb, xt);
    } else if constexpr (Q8) {
      using K8 = KLoad8<D, NW>;
      // waves with a K^ code block: that and a V~ code block or a scale
      // load; the others (D = 64) two scale loads
      if (wave < K8::NBLK) kload.issue_codes(kb, xt, wave);
      else if (wave & 1) vload.issue_scales(vb, xt);
      else kload.issue_scales(kb, xt, w.lane);
      if (wave < VL::NB) vload.issue_codes(vb, xt, wave);
      else if (wave & 1) kload.issue_scales(kb, xt, w.lane);
      else vload.issue_scales(vb, xt);
    } else {
      kload.issue(kb, xt, wave);
      if (wave < VL::NB) vload.issue_codes(vb, xt, wave);
      else vload.issue_scales(vb, xt);
    }
  };
  if constexpr (!kPair) {
    // prologue: tiles 0 .. P-1; tile 0 resident, the others in flight.  With
    // bf16 Q the others are issued once every wave has read its Q rows.
    constexpr int kFirst = Q8 ? kHP : 1;
#pragma unroll
    for (int x = 0; x < kFirst; ++x) load_tile(x, x * Sm::kK, x * Sm::kV);
    if constexpr (!Q8) {
      wait_vmem_le(kLoads);
      half_read_q<D>(smem + Sm::kK + wave * (kWaveQ * D * 2), w.lane, w.qo.r);
    }
    wait_vmem_le((kFirst - 1) * kLoads);
    __syncthreads();
#pragma unroll
    for (int x = kFirst; x < kHP; ++x) load_tile(x, x * Sm::kK, x * Sm::kV);
    int sx = kHP;
    int skofs = (kHP % kHK) * Sm::kK, svofs = (kHP % kHV) * Sm::kV;
    auto stream = [&]() {
      load_tile(sx, skofs, svofs);
      ++sx;
      skofs = ring_next<Sm::kK, kHK>(skofs);
      svofs = ring_next<Sm::kV, kHV>(svofs);
    };
    half_schedule<D, KIND, Q8, kLoads>(w, wtiles, ntiles, kbuf0, vbuf0, a, stream);
  } else {
  const int group = wave >> 2;
  // prologue: tiles 0 .. P; tiles 0 and 1 resident, 2 .. P in flight (the
  // loads of the last P-1 even phases before phase 2)
#pragma unroll
  for (int x = 0; x <= kPP; ++x) load_tile(x, (x % kPPK) * Sm::kK, (x % kPPV) * Sm::kV);
  wait_vmem_le((kPP - 1) * kLoads);
  __syncthreads();

  // phase 2j (j >= 1) streams tile j+P; the slots advance with the tile
  int sx = kPP + 1;
  int skofs = ((kPP + 1) % kPPK) * Sm::kK, svofs = ((kPP + 1) % kPPV) * Sm::kV;
  auto stream = [&]() {
    load_tile(sx, skofs, svofs);
    ++sx;
    skofs = ring_next<Sm::kK, kPPK>(skofs);
    svofs = ring_next<Sm::kV, kPPV>(svofs);
  };

  constexpr int keep = kKeep * kLoads;
#if EFQ_PHASE_STAMPS
  // each stamping lane clears its own stamp area, so phases its wave does
  // not reach read 0 rather than what an earlier workgroup left in LDS
  if ((threadIdx.x & 255) == 0) {
    unsigned long long* z = (unsigned long long*)(smem + Sm::kStampOff) + group * kStampSlots;
    for (int i = 0; i < kStampSlots; ++i) z[i] = 0;
  }
#endif
  if (group == 0)
    pp_schedule<0>(w, wtiles, ntiles, kbuf0, vbuf0, a, b, hq, keep, stream);
  else
    pp_schedule<1>(w, wtiles, ntiles, kbuf0, vbuf0, a, b, hq, keep, stream);
  }
  wait_vmem();   // no load may still target LDS when the wave leaves
#if EFQ_PHASE_STAMPS
  if (kPair && g_stamps && blockIdx.x < kStampBlocks && (threadIdx.x & 255) == 0) {
    const int group = wave >> 2;
    const unsigned long long* src =
        (const unsigned long long*)(smem + Sm::kStampOff) + group * kStampSlots;
    unsigned long long* dst = g_stamps + ((long)blockIdx.x * 2 + group) * kStampSlots;
    for (int i = 0; i < kStampSlots; ++i) dst[i] = src[i];
  }
#endif

  // O = A / l as A * (1 / l): one division per row instead of one per
  // element (within 1.5 ulp of the quotient).  l = 0 only when every code of
  // the row is 0, which an operating point with tau above the block-max
  // residual range [log 3/4, log 3/2) can produce; the row is then 0.
  const float l = w.lacc[0];
  const float rl = l > 0.0f ? 1.0f / l : 0.0f;
  uint8_t* const ob = smem + wave * (kWaveQ * D * 4);   // half workgroup: O rows
  const bool o_rows = !kPair && (RHO || a.o_rows);
  if (o_rows) __syncthreads();                          // every wave is done with the rings
  if constexpr (RHO) {
    double d2 = 0.0, r2 = 0.0;
    auto add = [&](float o, float r) {
      const double d = (double)o - (double)r;
      d2 += d * d;
      r2 += (double)r * (double)r;
    };
    if constexpr (!kPair) {
      half_rows<D>(w.oacc, rl, w.lane, ob, [&](int row, int d, const f32x4& o) {
        if (q_wave0 + row < a.Sq) {
          const f32x4 v = *(const f32x4*)(rho.o_ref + (((long)b * a.Sq + q_wave0 + row) * a.Hq + hq) * D + d);
#pragma unroll
          for (int i = 0; i < 4; ++i) add(o[i], v[i]);
        }
      });
    } else if (w.my_q < a.Sq) {
      const float* rp = rho.o_ref + (((long)b * a.Sq + w.my_q) * a.Hq + hq) * D;
#pragma unroll
      for (int s = 0; s < NS; ++s) {
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          const f32x4 v = *(const f32x4*)(rp + s * 32 + 8 * r4 + 4 * w.half);
#pragma unroll
          for (int i = 0; i < 4; ++i) add(w.oacc[s][4 * r4 + i] * rl, v[i]);
        }
      }
    }
#pragma unroll
    for (int x = 32; x > 0; x >>= 1) {
      d2 += __shfl_xor(d2, x);
      r2 += __shfl_xor(r2, x);
    }
    double* const red = (double*)smem;
    __syncthreads();   // every wave is done with the rings
    if (w.lane == 0) {
      red[2 * wave] = d2;
      red[2 * wave + 1] = r2;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
      double t = 0.0;
#pragma unroll
      for (int i = 0; i < NW; ++i) t += red[2 * i + threadIdx.x];
      rho.part[2 * ((long)blockIdx.y * gridDim.x + blockIdx.x) + threadIdx.x] = t;
    }
  } else if (o_rows) {
    half_rows<D>(w.oacc, rl, w.lane, ob, [&](int row, int d, const f32x4& o) {
      if (q_wave0 + row < a.Sq)
        *(f32x4*)(out + (((long)b * a.Sq + q_wave0 + row) * a.Hq + hq) * D + d) = o;
    });
  } else if (w.my_q < a.Sq) {
    float* op = out + (((long)b * a.Sq + w.my_q) * a.Hq + hq) * D;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        int d = s * 32 + 8 * r4 + 4 * w.half;
        f32x4 v4 = f32x4{w.oacc[s][4 * r4] * rl, w.oacc[s][4 * r4 + 1] * rl,
                         w.oacc[s][4 * r4 + 2] * rl, w.oacc[s][4 * r4 + 3] * rl};
        *(f32x4*)(op + d) = v4;
      }
    }
    if constexpr (DUMP) {
      long row = ((long)b * a.Hq + hq) * a.Sq + w.my_q;
      if (w.half == 0) {
        a.row_m[row] = is_expq<KIND>() ? w.m * kLn2 : w.m;
        a.row_l[row] = l;
      }
    }
  }
}

// ------------------------------------------------------ few queries
// Few queries against many keys (a generation step) leave the kernels above
// a handful of workgroups that walk all keys one tile after another.  Here
// the keys of a (batch, kv head) are split into chunks of whole 64-key tiles,
// and the 32 columns of a wave hold the queries of all heads of the group
// (row r = query * group + head).  The codes depend on the running row
// maximum, so the split first finds every chunk's row maxima (one pass over
// K); a chunk then starts from the maximum of the chunks before it, which is
// the running maximum the unsplit recurrence has there, and takes the same
// scores, codes and scales.  Partial sums (A, l) of the chunks are merged
// with alpha = exp(m_chunk - m_last).  With few rows the first pass keeps the
// scores and the second reads those in place of K.
//   split_max_kernel    row maxima of every chunk
//   split_attn_kernel   Alg. 2 over one chunk per wave; the four waves of a
//                       workgroup (consecutive chunks) merge through LDS
//   split_merge_kernel  merges the workgroups' partial sums, divides by l
constexpr int kSWaves = 4;                 // chunks per workgroup
constexpr int kSRows = 128;                // most rows (queries x group) taken
constexpr int kSItems = 2048;              // waves the chip holds at two per SIMD
// Most bytes of scratch: scores kept, and maxima and partial sums, which are
// about the output once a (batch, kv head) has a single workgroup.
constexpr double kSplitScores = 256 << 20;
constexpr size_t kSplitSums = 256 << 20;

struct SplitArgs {
  int B, Sq, Sk, Hq, Hkv;
  int nb;             // padded 32-key blocks of V~
  size_t scale_off;
  int R, CT;          // rows per (batch, kv head), 32-row column tiles
  int ntiles, tpc;    // 64-key tiles, tiles per chunk
  int nch, ngrp;      // chunks, workgroups (kSWaves chunks) per column tile
  int xcd_remap;
  float scale, tau, h;
  int sq_pad, sk_pad;
  size_t q8_soff, k8_soff;
  float* cmax;        // [B Hkv][nch][CT * 32] row maxima of the raw products
  float* part;        // [B Hkv][ngrp][R][D] partial A, then [..][R][2] (m, l)
  float* ml;
  float* sc;          // scores, [B Hkv][tile][8][half][R][4] (accumulator registers 4 i .. 4 i + 3)
};

// Registers a wave reads K of one tile into: bf16, the operand of k-step kk
// of window w; MXFP8, that of chunk c, and the lane's scales.
template <int D, bool Q8>
struct SplitK {
  bf16x8 a[2][D / 16];
};
template <int D>
struct SplitK<D, true> {
  i32x8 a[2][D / 64];
  int sc[2];
};

template <int D, bool Q8>
__device__ __forceinline__ void split_read_k(const void* k, const SplitArgs& a, int b, int g, int tile,
                                             int lane, SplitK<D, Q8>& o) {
  const int half = lane >> 5;
#pragma unroll
  for (int w = 0; w < 2; ++w) {
    const int key = tile * kBc + 32 * w + (lane & 31);
    if constexpr (Q8) {   // padded to whole tiles
      const long row = ((long)b * a.Hkv + g) * a.sk_pad + key;
      const uint8_t* p = (const uint8_t*)k + row * D + 16 * half;
#pragma unroll
      for (int c = 0; c < D / 64; ++c) {
        const u32x4 lo = *(const u32x4*)(p + 64 * c);
        const u32x4 hi = *(const u32x4*)(p + 64 * c + 32);
        o.a[w][c] = i32x8{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3],
                          (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
      }
      const uint8_t* sp = (const uint8_t*)k + a.k8_soff + row * (D / 32);
      unsigned raw;
      if constexpr (D == 128) raw = *(const unsigned*)sp;
      else raw = *(const unsigned short*)sp;
      o.sc[w] = lane_scales<D>(raw, half);
    } else {              // keys past the end read the last one (masked)
      const int kc = key < a.Sk ? key : a.Sk - 1;
      const unsigned short* p =
          (const unsigned short*)k + (((long)b * a.Sk + kc) * a.Hkv + g) * D + half * 8;
#pragma unroll
      for (int kk = 0; kk < D / 16; ++kk) o.a[w][kk] = *(const bf16x8*)(p + kk * 16);
    }
  }
}

// The lane's query operand of column tile ct (rows past R read row R - 1).
template <int D, bool Q8>
__device__ __forceinline__ void split_read_q(const void* q, const SplitArgs& a, int b, int g, int ct,
                                             int lane, QOps<D, Q8>& o) {
  const int half = lane >> 5;
  const int G = a.Hq / a.Hkv;
  const int r = min(ct * 32 + (lane & 31), a.R - 1);
  const int i = r / G, hq = g * G + r % G;
  if constexpr (Q8) {
    const long row = ((long)b * a.Hq + hq) * a.sq_pad + i;
    const uint8_t* p = (const uint8_t*)q + row * D + 16 * half;
#pragma unroll
    for (int c = 0; c < D / 64; ++c) {
      const u32x4 lo = *(const u32x4*)(p + 64 * c);
      const u32x4 hi = *(const u32x4*)(p + 64 * c + 32);
      o.a[c] = i32x8{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3],
                     (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
    }
    const uint8_t* sp = (const uint8_t*)q + a.q8_soff + row * (D / 32);
    unsigned raw;
    if constexpr (D == 128) raw = *(const unsigned*)sp;
    else raw = *(const unsigned short*)sp;
    o.sc = lane_scales<D>(raw, half);
  } else {
    const unsigned short* p =
        (const unsigned short*)q + (((long)b * a.Sq + i) * a.Hq + hq) * D + half * 8;
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) o.r[kk] = *(const bf16x8*)(p + kk * 16);
  }
}

// S = K Q^T of one tile, with the MFMAs in the order of the unsplit kernels.
template <int I, int D>
__device__ __forceinline__ void split_qk8(const SplitK<D, true>& k, const QOps<D, true>& q, f32x16& s0,
                                          f32x16& s1) {
  if constexpr (I < D / 64) {
    s0 = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(k.a[0][I], q.a[I], s0, 0, 0, I, k.sc[0], I, q.sc);
    s1 = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(k.a[1][I], q.a[I], s1, 0, 0, I, k.sc[1], I, q.sc);
    split_qk8<I + 1>(k, q, s0, s1);
  }
}
template <int D, bool Q8>
__device__ __forceinline__ void split_qk(const SplitK<D, Q8>& k, const QOps<D, Q8>& q, f32x16& s0,
                                         f32x16& s1) {
  s0 = f32x16{};
  s1 = f32x16{};
  if constexpr (Q8) {
    split_qk8<0>(k, q, s0, s1);
  } else {
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) {
      s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k.a[0][kk], q.r[kk], s0, 0, 0, 0);
      s1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k.a[1][kk], q.r[kk], s1, 0, 0, 0);
    }
  }
}

__device__ __forceinline__ int split_work(const SplitArgs& a) {
  const int n = blockIdx.x;
  return a.xcd_remap ? (n & 7) * (int)(gridDim.x >> 3) + (n >> 3) : n;
}

// The lane's first stored score quad of a tile (rows past R: row R - 1).
__device__ __forceinline__ f32x4* split_scores(const SplitArgs& a, int bg, int t, int lane) {
  return (f32x4*)a.sc + ((long)bg * a.ntiles + t) * 16 * a.R + (lane >> 5) * a.R + min(lane & 31, a.R - 1);
}

// One wave per (batch, kv head, chunk, group of CTW column tiles).
template <int D, bool Q8, int CTW, bool KEEP>
__global__ __attribute__((amdgpu_flat_work_group_size(64 * kSWaves, 64 * kSWaves),
                          amdgpu_waves_per_eu(2, 4))) void
split_max_kernel(const void* __restrict__ q, const void* __restrict__ k, SplitArgs a) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int ncg = (a.CT + CTW - 1) / CTW;
  int w = split_work(a);
  const int cg = w % ncg;
  w /= ncg;
  const int chunk = (w % a.ngrp) * kSWaves + wave;
  const int bg = w / a.ngrp;
  const int b = bg / a.Hkv, g = bg % a.Hkv;
  const int t0 = chunk * a.tpc, t1 = min(a.ntiles, t0 + a.tpc);
  if (t0 >= t1) return;
  QOps<D, Q8> qo[CTW];
#pragma unroll
  for (int c = 0; c < CTW; ++c) split_read_q<D, Q8>(q, a, b, g, min(cg * CTW + c, a.CT - 1), lane, qo[c]);
  SplitK<D, Q8> kr;
  split_read_k<D, Q8>(k, a, b, g, t0, lane, kr);
  float mx[CTW];
#pragma unroll
  for (int c = 0; c < CTW; ++c) mx[c] = -INFINITY;
  for (int t = t0; t < t1; ++t) {
    f32x16 s[CTW][2];
#pragma unroll
    for (int c = 0; c < CTW; ++c) split_qk<D, Q8>(kr, qo[c], s[c][0], s[c][1]);
    if (t + 1 < t1) split_read_k<D, Q8>(k, a, b, g, t + 1, lane, kr);
    if constexpr (KEEP) {
      if ((lane & 31) < a.R) {
        f32x4* p = split_scores(a, bg, t, lane);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const f32x16& x = s[0][i >> 2];
          p[(long)i * 2 * a.R] = f32x4{x[4 * (i & 3)], x[4 * (i & 3) + 1], x[4 * (i & 3) + 2], x[4 * (i & 3) + 3]};
        }
      }
    }
    const int l0 = a.Sk - t * kBc - 4 * (lane >> 5);
#pragma unroll
    for (int c = 0; c < CTW; ++c) {
      if ((t + 1) * kBc > a.Sk) mask_tile(s[c][0], s[c][1], l0);
      mx[c] = fmaxf(mx[c], fmaxf(max16(s[c][0]), max16(s[c][1])));
    }
  }
#pragma unroll
  for (int c = 0; c < CTW; ++c) {
    const int ct = cg * CTW + c;
    float x = mx[c], y = mx[c];
    swap32f(x, y);
    if (ct < a.CT && lane < 32)
      a.cmax[((long)bg * a.nch + chunk) * (a.CT * 32) + ct * 32 + lane] = fmaxf(x, y);
  }
}

// V of one 64-key tile, straight from bf16 (a whole call, one column tile: a
// wave is the only reader of its tile, so V~ need not be written and read
// back).  The lane holds the column pair (2 lane, 2 lane + 1) of the tile's
// 64 rows; the quantised tile passes through the wave's own LDS in the layout
// of V~.  Same arithmetic as vquant_kernel.
template <int D>
struct SplitV {
  static_assert(D == 128, "64 lanes hold the columns");
  unsigned raw[2][32];
  // rows past Sk read the last one; quantise() zeroes them
  __device__ __forceinline__ void read(const __amdgpu_buffer_rsrc_t& rs, int voff, int stride, int tile, int Sk) {
#pragma unroll
    for (int blk = 0; blk < 2; ++blk)
#pragma unroll
      for (int t = 0; t < 32; ++t)
        raw[blk][t] = __builtin_amdgcn_raw_buffer_load_b32(
            rs, voff, min(tile * kBc + blk * 32 + t, Sk - 1) * stride, 0);
  }
  __device__ __forceinline__ void quantise(uint8_t* vb, int tile, int Sk, int lane) {
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
      const int nvalid = Sk - tile * kBc - blk * 32;
      if (nvalid < 32) {
#pragma unroll
        for (int t = 0; t < 32; ++t) raw[blk][t] = t < nvalid ? raw[blk][t] : 0u;
      }
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        unsigned words[4];
        const int k = vq_column(raw[blk], c, words);
        const int d = 2 * lane + c;
        *(u32x4*)(vb + (blk * D + d) * 16) = u32x4{words[0], words[1], words[2], words[3]};
        vb[2 * D * 16 + blk * D + (d & 31) * (D / 32) + (d >> 5)] = (uint8_t)(k + 127);
      }
    }
    // a wave's LDS operations complete in order
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
  }
};

// One wave per (batch, kv head, column tile, chunk); the last chunk of a
// workgroup has its largest (running) maximum.  RAWV: vhat is V itself (bf16).
template <int D, int KIND, bool Q8, bool KEEP, bool RAWV>
__global__ __attribute__((amdgpu_flat_work_group_size(64 * kSWaves, 64 * kSWaves),
                          amdgpu_waves_per_eu(2, KEEP ? 3 : 2))) void
split_attn_kernel(const void* __restrict__ q, const void* __restrict__ k,
                  const uint8_t* __restrict__ vhat, SplitArgs a) {
  constexpr int NS = D / 32;
  __shared__ __align__(16) float so[kSWaves][D / 16][64][4];   // scaled A of each wave, half the columns
  __shared__ float sm[kSWaves][32], sl[kSWaves][32];
  constexpr int kVb = RAWV ? 2 * D * 16 + 2 * D : 16;
  __shared__ __align__(16) uint8_t svb[kSWaves][kVb];               // the wave's quantised V tile
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, half = lane >> 5;
  int w = split_work(a);
  const int ct = w % a.CT;
  w /= a.CT;
  const int grp = w % a.ngrp, bg = w / a.ngrp;
  const int chunk = grp * kSWaves + wave;
  const int b = bg / a.Hkv, g = bg % a.Hkv;
  const int t0 = chunk * a.tpc, t1 = min(a.ntiles, t0 + a.tpc);

  PgenArgs pa;
  pa.scale = a.scale;
  pa.sh = a.scale * a.h;
  pa.sh32 = 32.0f * pa.sh;
  pa.sh16 = 16.0f * pa.sh;
  pa.c = kLn6 + a.tau;
  pa.negh = -a.h;
  pa.l2s = a.scale * kInvLn2;

  f32x16 oacc[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) oacc[s] = f32x16{};
  f32x4 lacc = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY;
  if (t0 < t1) {
    QOps<D, Q8> qo;
    SplitK<D, Q8> kr;
    f32x16 n0, n1;   // with KEEP: the next tile's stored scores
    auto read_scores = [&](int t) {
      const f32x4* p = split_scores(a, bg, t, lane);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const f32x4 x = p[(long)i * 2 * a.R];
#pragma unroll
        for (int c = 0; c < 4; ++c) (i < 4 ? n0 : n1)[4 * (i & 3) + c] = x[c];
      }
    };
    if constexpr (KEEP) {
      read_scores(t0);
    } else {
      split_read_q<D, Q8>(q, a, b, g, ct, lane, qo);
      split_read_k<D, Q8>(k, a, b, g, t0, lane, kr);
    }
    const uint8_t* vc = vhat + (long)bg * a.nb * D * 16 + (half * D + (lane & 31)) * 16;
    const uint8_t* vs = vhat + a.scale_off + (long)bg * a.nb * D + half * D + (lane & 31) * (D / 32);
    auto read_vops = [&](int t, VOps<D>& v) {
#pragma unroll
      for (int s = 0; s < NS; ++s) v.a[s] = *(const u32x4*)(vc + (long)t * (2 * D * 16) + s * 512);
      if constexpr (NS == 4) v.sv = *(const int*)(vs + (long)t * (2 * D));
      else v.sv = *(const unsigned short*)(vs + (long)t * (2 * D));
    };
    VOps<D> vop;
    std::conditional_t<RAWV, SplitV<128>, NoRho> rv;
    const int vstride = a.Hkv * D * 2;
    const __amdgpu_buffer_rsrc_t vrs =
        make_rsrc(vhat + (long)b * a.Sk * vstride, (unsigned)a.Sk * (unsigned)vstride);
    if constexpr (RAWV) rv.read(vrs, g * D * 2 + lane * 4, vstride, t0, a.Sk);
    else read_vops(t0, vop);
    // the running maximum at the chunk's first key: the lane halves take
    // alternate earlier chunks
    {
      const float* cm = a.cmax + (long)bg * a.nch * (a.CT * 32) + ct * 32 + (lane & 31);
      float x = -INFINITY;
#pragma unroll 8
      for (int c = half; c < chunk; c += 2) x = fmaxf(x, cm[(long)c * (a.CT * 32)]);
      float y = x;
      swap32f(x, y);
      m = fmaxf(x, y) * (is_expq<KIND>() ? pa.l2s : pa.scale);
    }
    const i32x8 sel = rowsum_selector(lane);
    for (int t = t0; t < t1; ++t) {
      f32x16 s0, s1;
      if constexpr (KEEP) {
        s0 = n0;
        s1 = n1;
      } else {
        split_qk<D, Q8>(kr, qo, s0, s1);
      }
      VOps<D> v = vop;
      if constexpr (RAWV) rv.quantise(svb[wave], t, a.Sk, lane);
      if (t + 1 < t1) {
        if constexpr (KEEP) read_scores(t + 1);
        else split_read_k<D, Q8>(k, a, b, g, t + 1, lane, kr);
        if constexpr (RAWV) rv.read(vrs, g * D * 2 + lane * 4, vstride, t + 1, a.Sk);
        else read_vops(t + 1, vop);
      }
      if ((t + 1) * kBc > a.Sk) mask_tile(s0, s1, a.Sk - t * kBc - 4 * half);
      float pm0, pm1;
      PgenState st;
      pg_max<KIND>(s0, s1, pm0, pm1);
      if (pg_params<KIND>(pm0, pm1, m, pa, st)) {
        const float alpha = pg_alpha<KIND>(st);
#pragma unroll
        for (int s = 0; s < NS; ++s) oacc[s] *= alpha;
        lacc[0] *= alpha;
      }
      pg_pairs<KIND, 0, 32>(s0, s1, pa, st);
      const PgenOut po = pg_finish<KIND>(st);
      const i32x8 b8 = i32x8{(int)po.bop[0], (int)po.bop[1], (int)po.bop[2], (int)po.bop[3], 0, 0, 0, 0};
      if constexpr (RAWV)
        read_v<D>(lds_at(lds_addr(svb[wave] + vop_offset<D>(lane))),
                  lds_at(lds_addr(svb[wave] + vscale_offset<D>(lane))), v);
      pv_slabs<NS>(oacc, v, b8, po.scale_b);
      lacc = rowsum_mfma(sel, b8, lacc, po.scale_b);
      if constexpr (RAWV) {   // the next tile overwrites the LDS after these reads
        asm volatile("" ::: "memory");
        __builtin_amdgcn_wave_barrier();
      }
    }
  }
  // merge the workgroup's chunks at the maximum of its last one
  if (half == 0) sm[wave][lane] = m;
  __syncthreads();
  const int last = min(kSWaves, a.nch - grp * kSWaves) - 1;
  const float ml = sm[last][lane & 31];
  const float f = t0 < t1 ? __builtin_amdgcn_exp2f(is_expq<KIND>() ? m - ml : (m - ml) * kInvLn2) : 0.0f;
  if (half == 0) sl[wave][lane] = lacc[0] * f;
  // slice i = 4 s + r of lane (row, half) holds columns 32 s + 8 r + 4 half +
  // [0, 4); wave w sums slices w, w + 4, ... of each half of the columns
  const int row = ct * 32 + (lane & 31);
  const long prow = ((long)bg * a.ngrp + grp) * a.R + row;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int s = 0; s < NS / 2; ++s)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const f32x16& o = oacc[h * (NS / 2) + s];
        *(f32x4*)so[wave][s * 4 + r][lane] =
            f32x4{o[4 * r] * f, o[4 * r + 1] * f, o[4 * r + 2] * f, o[4 * r + 3] * f};
      }
    __syncthreads();
    if (row < a.R) {
#pragma unroll
      for (int j = 0; j < D / 16 / kSWaves; ++j) {
        const int i = j * kSWaves + wave;
        f32x4 x = *(f32x4*)so[0][i][lane];
#pragma unroll
        for (int c = 1; c < kSWaves; ++c) x += *(f32x4*)so[c][i][lane];
        *(f32x4*)(a.part + prow * D + h * (D / 2) + i * 8 + 4 * half) = x;
      }
      if (h == 0 && wave == 0 && half == 0) {
        a.ml[2 * prow] = ml;
        a.ml[2 * prow + 1] = sl[0][lane] + sl[1][lane] + sl[2][lane] + sl[3][lane];
      }
    }
    if (h == 0) __syncthreads();
  }
}

// One workgroup of D threads per output row (batch, kv head, row).
template <int D, bool LOG2>
__global__ __launch_bounds__(D) void split_merge_kernel(float* __restrict__ out, SplitArgs a) {
  const int r = blockIdx.x % a.R, bg = blockIdx.x / a.R;
  const int b = bg / a.Hkv, g = bg % a.Hkv, G = a.Hq / a.Hkv;
  const int d = threadIdx.x;
  const long p0 = (long)bg * a.ngrp * a.R + r;
  const float mt = a.ml[2 * (p0 + (long)(a.ngrp - 1) * a.R)];
  float o = 0.0f, l = 0.0f;
#pragma unroll 4
  for (int i = 0; i < a.ngrp; ++i) {
    const long p = p0 + (long)i * a.R;
    const float dm = a.ml[2 * p] - mt;
    const float f = __builtin_amdgcn_exp2f(LOG2 ? dm : dm * kInvLn2);
    o += a.part[p * D + d] * f;
    l += a.ml[2 * p + 1] * f;
  }
  const float rl = l > 0.0f ? 1.0f / l : 0.0f;
  out[(((long)b * a.Sq + r / G) * a.Hq + g * G + r % G) * D + d] = o * rl;
}

// ------------------------------------------ standalone probability stage
// One wave per (32 rows, 64 columns) tile of x: the values are placed into
// the accumulator layout of the fused kernel and run through the same code
// path with scale 1 and running maximum 0.
struct PgenKArgs {
  int rows, cols, nblk, ncb;   // ncb = column tiles of 64
  float tau, h;
};

template <int KIND>
__global__ __launch_bounds__(64) void pgen_kernel(const float* __restrict__ x,
                                                  uint8_t* __restrict__ codes,
                                                  uint8_t* __restrict__ e8m0, PgenKArgs a) {
  const int lane = threadIdx.x;
  const int half = lane >> 5;
  const int rt = blockIdx.x / a.ncb, ct = blockIdx.x % a.ncb;
  const int row = rt * 32 + (lane & 31);
  const int c0 = ct * 64;
  f32x16 s0, s1;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    int kofs = 8 * (r >> 2) + 4 * half + (r & 3);
    int t0 = c0 + kofs, t1 = c0 + 32 + kofs;
    s0[r] = (row < a.rows && t0 < a.cols) ? x[(long)row * a.cols + t0] : -INFINITY;
    s1[r] = (row < a.rows && t1 < a.cols) ? x[(long)row * a.cols + t1] : -INFINITY;
  }
  PgenArgs pa;
  pa.scale = 1.0f;
  pa.sh = 1.0f * a.h;
  pa.sh32 = 32.0f * pa.sh;
  pa.sh16 = 16.0f * pa.sh;
  pa.c = kLn6 + a.tau;
  pa.negh = -a.h;
  pa.l2s = 1.0f * kInvLn2;
  float m = 0.0f;
  PgenOut po = pgen<KIND>(s0, s1, m, pa);
  const int blk = 2 * ct + half;
  if (row < a.rows && blk < a.nblk) {
    u32x4 w = unpermute_codes(po.bop);
    const int bytes = (a.cols + 1) / 2;
    uint8_t* cp = codes + (long)row * bytes + blk * 16;
    int nbytes = min(16, bytes - blk * 16);
    for (int i = 0; i < nbytes; ++i) cp[i] = (uint8_t)((w[i >> 2] >> (8 * (i & 3))) & 0xFF);
    e8m0[(long)row * a.nblk + blk] = (uint8_t)po.scale_b;
  }
}

// ----------------------------------------- P-gen throughput probe
template <int KIND>
__global__ __launch_bounds__(256) void pgen_bench_kernel(int iters, float tau, float h,
                                                         uint32_t* __restrict__ checksum,
                                                         int waves) {
  const int lane = threadIdx.x & 63;
  const int wid = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (wid >= waves) return;
  // synthetic scores in the accumulator layout: a smooth pseudo-random field
  f32x16 s0, s1;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    unsigned hsh = (unsigned)(lane * 2654435761u) ^ (unsigned)(r * 40503u) ^ (unsigned)(wid * 97u);
    hsh ^= hsh >> 13;
    hsh *= 0x5bd1e995u;
    s0[r] = (float)(hsh & 0xFFFF) * (1.0f / 4096.0f) - 12.0f;
    s1[r] = (float)((hsh >> 16) & 0xFFFF) * (1.0f / 4096.0f) - 12.0f;
  }
  PgenArgs pa;
  pa.scale = 0.0883883461f;
  pa.sh = pa.scale * h;
  pa.sh32 = 32.0f * pa.sh;
  pa.sh16 = 16.0f * pa.sh;
  pa.c = kLn6 + tau;
  pa.negh = -h;
  pa.l2s = pa.scale * kInvLn2;
  unsigned acc = 0;
  float m = -INFINITY;
  for (int it = 0; it < iters; ++it) {
    // the scores count as changed in every iteration, so no part of the
    // stage (block maxima, products with the scale) moves out of the loop
    asm volatile("" : "+v"(s0), "+v"(s1));
    PgenOut po = pgen<KIND>(s0, s1, m, pa);
    acc ^= po.bop[0] ^ (po.bop[1] << 1) ^ (po.bop[2] << 2) ^ (po.bop[3] << 3) ^ (unsigned)po.scale_b;
    acc += __float_as_uint(po.alpha);
    // perturb the running maximum so that no iteration repeats the previous one
    m = m - 0.25f + 0.5f * (float)(acc & 1u);
  }
  if (lane == 0) checksum[wid] = acc;
}

// ------------------------------------------------- shader clock probe
// Every wave of a 256-thread workgroup streams bf16 32x32x16 MFMAs on two
// independent accumulators (the matrix core at its full rate) for iters x 16
// MFMAs, its operands rotating through four pseudo-random sets (signs,
// exponents 2^-3 .. 2^4 and mantissas hashed from the lane, the workgroup
// and the set) so that they change with every instruction as real data
// does; lane 0 of wave 0 stores the s_memtime ticks (shader clock) and the
// s_memrealtime ticks (a constant 100 MHz) the loop took, so their ratio is
// the shader clock under a matrix-core load.  The accumulators feed the
// stored value through a test that never holds, so the loop stays.
__device__ __forceinline__ bf16x8 clock_probe_operand(unsigned seed) {
  bf16x8 v;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    unsigned h = (seed + (unsigned)i * 0x9E3779B9u) * 0x85EBCA6Bu;
    h ^= h >> 15;
    h *= 0xC2B2AE35u;
    h ^= h >> 13;
    const unsigned short b = (unsigned short)(((h >> 31) << 15) | ((124u + ((h >> 20) & 7u)) << 7) |
                                              (h & 0x7Fu));
    v[i] = __builtin_bit_cast(__bf16, b);
  }
  return v;
}

__global__ __launch_bounds__(256) void clock_probe_kernel(int iters,
                                                          unsigned long long* __restrict__ out) {
  const unsigned seed = (blockIdx.x * 256u + threadIdx.x) * 8u;
  bf16x8 x[4], y[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    x[s] = clock_probe_operand(seed + 2u * s);
    y[s] = clock_probe_operand(seed + 2u * s + 1u);
  }
  f32x16 a0 = {}, a1 = {};
  const unsigned long long m0 = __builtin_amdgcn_s_memtime();
  const unsigned long long r0 = __builtin_amdgcn_s_memrealtime();
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      a0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[i & 3], y[i & 3], a0, 0, 0, 0);
      a1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[(i + 1) & 3], y[(i + 2) & 3], a1, 0, 0, 0);
    }
  }
  const unsigned long long m1 = __builtin_amdgcn_s_memtime();
  const unsigned long long r1 = __builtin_amdgcn_s_memrealtime();
  float sum = 0.0f;
#pragma unroll
  for (int i = 0; i < 16; ++i) sum += a0[i] + a1[i];
  if (threadIdx.x == 0) {
    out[2 * blockIdx.x] = (m1 - m0) + (sum == -1.0f ? 1ull : 0ull);
    out[2 * blockIdx.x + 1] = r1 - r0;
  }
}

__global__ void fill_zero_kernel(uint8_t* __restrict__ p, size_t n) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = 0;
}

// ------------------------------------------------ calibration objective
// rho(tau, h) = ||O~ - O_ref||_F / ||O_ref||_F (Sec. III-C, Alg. 3).  One
// launch runs the EFQ attention for up to kRhoCand candidate pairs (grid y)
// and keeps only the sums of squares, in fp64: a candidate's output is never
// stored and read back, and the candidates together fill the chip, which one
// short calibration prompt does not.  The sums are reduced in a fixed order
// (lanes, waves, then rho_final_kernel over the workgroups), so repeated
// runs give identical values.  Matrix-core bound, as the attention itself:
// 16 candidates on 1024 tokens (32/8 heads, D 128) took 16 x (28.8 us
// attention + 8.0 us for the sums over the stored output + 2.8 us to reduce
// them); a whole call 724 us, now 187.
// One block per candidate: its n partial pairs -> res[2 c] = sum (O~ -
// O_ref)^2, res[2 c + 1] = sum O_ref^2.
__global__ __launch_bounds__(256) void rho_final_kernel(const double* __restrict__ part, long n,
                                                        double* __restrict__ res) {
  __shared__ double s1[256], s2[256];
  part += 2 * n * blockIdx.x;
  double a = 0.0, b = 0.0;
  for (long i = threadIdx.x; i < n; i += 256) {
    a += part[2 * i];
    b += part[2 * i + 1];
  }
  s1[threadIdx.x] = a;
  s2[threadIdx.x] = b;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      s1[threadIdx.x] += s1[threadIdx.x + w];
      s2[threadIdx.x] += s2[threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    res[2 * blockIdx.x] = s1[0];
    res[2 * blockIdx.x + 1] = s2[0];
  }
}

// ================================================================ host side
constexpr int kQTile = kPPBr;   // queries per workgroup of the launched kernel
constexpr int kMaxDevices = 64; // device indices the library accepts

thread_local char g_msg[512] = "ok";

int fail(int status, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_msg, sizeof g_msg, fmt, ap);
  va_end(ap);
  return status;
}

std::mutex g_dev_mu;
int g_dev_ok[kMaxDevices];  // 0 unknown, 1 gfx950, -1 unusable

int check_device() {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(EFQ_EHIP, "hipGetDevice: %s", hipGetErrorString(e));
  if (dev < 0 || dev >= kMaxDevices) return fail(EFQ_EHIP, "device index %d out of range", dev);
  std::lock_guard<std::mutex> lk(g_dev_mu);
  if (g_dev_ok[dev] == 0) {
    hipDeviceProp_t prop;
    e = hipGetDeviceProperties(&prop, dev);
    if (e != hipSuccess) {
      g_dev_ok[dev] = -1;
      return fail(EFQ_EHIP, "hipGetDeviceProperties: %s", hipGetErrorString(e));
    }
    g_dev_ok[dev] = (strncmp(prop.gcnArchName, "gfx950", 6) == 0) ? 1 : -1;
    if (g_dev_ok[dev] < 0) return fail(EFQ_EHIP, "device %d is %s, not gfx950", dev, prop.gcnArchName);
  }
  return g_dev_ok[dev] > 0 ? EFQ_OK : fail(EFQ_EHIP, "device %d is not a usable gfx950", dev);
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

int validate_shape(const efq_shape* s, int causal) {
  if (!s) return fail(EFQ_EINVAL, "shape is NULL");
  if (s->batch < 1 || s->seq_q < 1 || s->seq_k < 1 || s->heads_q < 1 || s->heads_kv < 1 ||
      s->head_dim < 1)
    return fail(EFQ_EINVAL, "all shape fields must be >= 1");
  if (s->head_dim != 64 && s->head_dim != 128)
    return fail(EFQ_EUNSUPPORTED, "head_dim %d unsupported (64 or 128)", s->head_dim);
  if (s->heads_q % s->heads_kv != 0)
    return fail(EFQ_EINVAL, "heads_q %d not a multiple of heads_kv %d", s->heads_q, s->heads_kv);
  if (causal && s->seq_q != s->seq_k)
    return fail(EFQ_EUNSUPPORTED, "causal attention needs seq_q == seq_k (%d != %d)", s->seq_q,
                s->seq_k);
  const long nqt = (s->seq_q + kQTile - 1) / kQTile;
  if ((long)s->batch * s->heads_q * nqt > 0x7FFFFFFFL)
    return fail(EFQ_EUNSUPPORTED, "grid too large");
  if ((long)s->seq_k > (1L << 30) || (long)s->seq_q > (1L << 30))
    return fail(EFQ_EUNSUPPORTED, "sequence too long");
  // K of one batch and V~ of one (batch, kv head) are addressed through
  // 32-bit buffer ranges
  if ((long)s->seq_k * s->heads_kv * s->head_dim * 2 > 0x7FFFFFFFL)
    return fail(EFQ_EUNSUPPORTED, "seq_k * heads_kv * head_dim * 2 must be below 2^31 bytes");
  return EFQ_OK;
}

long padded_blocks(int seq_k) { return 2L * ((seq_k + kBc - 1) / kBc); }

size_t vhat_scale_offset(const efq_shape* s) {
  size_t codes = (size_t)s->batch * s->heads_kv * padded_blocks(s->seq_k) * s->head_dim * 16;
  return (codes + 255) & ~(size_t)255;
}
size_t vhat_bytes(const efq_shape* s) {
  size_t sc = (size_t)s->batch * s->heads_kv * padded_blocks(s->seq_k) * s->head_dim;
  return vhat_scale_offset(s) + ((sc + 255) & ~(size_t)255);
}

VqArgs vq_args(const efq_shape* s) {
  VqArgs a;
  a.B = s->batch;
  a.S = s->seq_k;
  a.H = s->heads_kv;
  a.D = s->head_dim;
  a.nb = (int)padded_blocks(s->seq_k);
  a.scale_off = vhat_scale_offset(s);
  const size_t vb = (size_t)a.B * a.S * a.H * a.D * 2;
  a.vbytes = vb < ((size_t)1 << 31) ? (unsigned)vb : 0u;
  return a;
}
long vq_blocks(const VqArgs& a) { return ((long)a.B * a.H * a.nb * (a.D / 2) + 255) / 256; }

int launch_vquant(const void* v, const efq_shape* s, void* vhat, hipStream_t st) {
  const VqArgs a = vq_args(s);
  const long grid = vq_blocks(a);
  if (a.vbytes)
    hipLaunchKernelGGL(vquant_kernel<true>, dim3((unsigned)grid), dim3(256), 0, st,
                       (const unsigned short*)v, (uint8_t*)vhat, a);
  else
    hipLaunchKernelGGL(vquant_kernel<false>, dim3((unsigned)grid), dim3(256), 0, st,
                       (const unsigned short*)v, (uint8_t*)vhat, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(EFQ_EHIP, "vquant launch: %s", hipGetErrorString(e));
  return EFQ_OK;
}

template <auto F>
struct KernelPtr {
  static constexpr auto value = F;
};

// More dynamic LDS than the default limit for KERNEL: raised once per device
// (check_device has bounded the device index).
template <auto KERNEL>
hipError_t raise_lds(int lds) {
  static std::once_flag once[kMaxDevices];
  static hipError_t set_err[kMaxDevices];
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::call_once(once[dev], [dev, lds]() {
    set_err[dev] = hipFuncSetAttribute((const void*)KERNEL,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  });
  return set_err[dev];
}

template <int D, int KIND, bool CAUSAL, bool DUMP, bool Q8, bool HALF>
hipError_t launch_attn_t(const void* q, const void* k, const void* vhat, float* out,
                         const AttnArgs& a, hipStream_t st, unsigned grid) {
  auto launch = [&](auto kernel, int threads, int lds) {
    const hipError_t e = raise_lds<decltype(kernel)::value>(lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(decltype(kernel)::value, dim3(grid), dim3(threads), lds, st, q, k,
                       (const uint8_t*)vhat, out, a, NoRho{});
    return hipGetLastError();
  };
  if constexpr (HALF)
    return launch(KernelPtr<attn_pp_kernel<D, KIND, CAUSAL, false, Q8, kHWaves, false>>{}, 64 * kHWaves, half_lds<D, Q8>());
  else
    return launch(KernelPtr<attn_pp_kernel<D, KIND, CAUSAL, DUMP, Q8, kPPWaves, false>>{}, kPPThreads,
                  SmemPP<D, Q8>::kTotal);
}

template <int D, bool DUMP, bool Q8, bool HALF>
hipError_t launch_attn_d(int kind, bool causal, const void* q, const void* k, const void* vhat,
                         float* out, const AttnArgs& a, hipStream_t st, unsigned grid) {
#define EFQ_CASE(KIND)                                                                          \
  case KIND:                                                                                    \
    return causal ? launch_attn_t<D, KIND, true, DUMP, Q8, HALF>(q, k, vhat, out, a, st, grid)  \
                  : launch_attn_t<D, KIND, false, DUMP, Q8, HALF>(q, k, vhat, out, a, st, grid);
  switch (kind) {
    EFQ_CASE(EFQ_PGEN_EFQ)
    EFQ_CASE(EFQ_PGEN_EXPQ)
    EFQ_CASE(EFQ_PGEN_LUT)
    EFQ_CASE(EFQ_PGEN_EXPQ6)
    default:
      break;
  }
  if constexpr (!DUMP && !HALF) {
    switch (kind) {
      EFQ_CASE(EFQ_PGEN_NOOP)
      default:
        break;
    }
  }
#undef EFQ_CASE
  return hipErrorInvalidValue;
}

size_t round256(size_t n) { return (n + 255) & ~(size_t)255; }
long pad64(int n) { return 64L * ((n + 63) / 64); }

// MXFP8 Q^ / K^ buffers: rows = batch * heads * padded seq
size_t q8_scale_offset(long rows, int D) { return round256((size_t)rows * D); }
size_t q8_bytes(long rows, int D) { return q8_scale_offset(rows, D) + round256((size_t)rows * (D / 32)); }
long qhat_rows(const efq_shape* s) { return (long)s->batch * s->heads_q * pad64(s->seq_q); }
long khat_rows(const efq_shape* s) { return (long)s->batch * s->heads_kv * pad64(s->seq_k); }

Q8Args q8_args(int B, int S, int H, int D) {
  Q8Args a;
  a.B = B;
  a.S = S;
  a.H = H;
  a.D = D;
  a.s_pad = (int)pad64(S);
  a.soff = q8_scale_offset((long)B * H * a.s_pad, D);
  return a;
}
long q8_threads(const Q8Args& a) { return (long)a.B * a.H * a.s_pad * (a.D / 8); }

// Whether a launch of this many workgroups of 256 threads is within the 32
// bits that HIP takes for the threads of a launch.
bool fits_launch(long workgroups) { return workgroups < (1L << 24); }

int launch_q8(const void* x, int B, int S, int H, int D, void* y, hipStream_t st) {
  const Q8Args a = q8_args(B, S, H, D);
  const long threads = q8_threads(a);
  const unsigned grid = (unsigned)((threads + 255) / 256);
  if (threads + 256 < ((long)1 << 32))
    hipLaunchKernelGGL(mxfp8_kernel<unsigned>, dim3(grid), dim3(256), 0, st,
                       (const unsigned short*)x, (uint8_t*)y, a);
  else
    hipLaunchKernelGGL(mxfp8_kernel<unsigned long>, dim3(grid), dim3(256), 0, st,
                       (const unsigned short*)x, (uint8_t*)y, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(EFQ_EHIP, "mxfp8 launch: %s", hipGetErrorString(e));
  return EFQ_OK;
}

// Whether the half-workgroup kernel takes a shape.  Timed side by side on one
// card (eight waves / half, us; EFQ, bf16 Q K^T, D 128 and 32/8 heads unless
// noted).  The lines were drawn before Q and O passed through LDS; where they
// now leave a gain on their far side, that is said.
//  - up to 128 queries: at least half of the eight waves have no query (64
//    sequences' single queries against 4096 keys 575 / 371; 64 x 128 652 / 413).
//    Not so the cheapest stage (EFQ) on bf16 keys that no other head shares,
//    from HBM, where a CU has no second workgroup: the two tiles this kernel has
//    in flight hide less of the latency than the other's four (24 heads, up to
//    112 workgroups: 4 x 16 queries, 30000 keys 388 / 421, 10000 keys 137 / 144,
//    but 8 x 16 queries, 6678 keys 119 / 108; 12 key/value heads 389 / 398).
//  - few keys: the loads and stores around the tiles weigh most.  Causal up to
//    1024 (16 prompts of 333 tokens 59 / 45, 8 of 1024 98 / 89; beyond, 8 of 1100
//    113 / 100, of 2048 260 / 267), else up to 768 (32760 queries, 24 heads, 128
//    keys 198 / 143, 512 273 / 233, 768 325 / 295; beyond, 1024 375 / 357, 1536
//    488 / 477, 2048 591 / 605).
//  - MXFP8 Q K^T and causal, up to 6144 keys: a tile reads half the K bytes, so
//    the doubled reads cost little and the even spread of the causal lengths
//    wins (4096 78.5 / 75.7, 6000 166 / 157; beyond, 8192 275 / 269, 12288 575 /
//    574, 16384 986 / 990).
//  - causal, no more eight-wave workgroups than CUs: the half workgroups spread
//    over idle CUs, or long and short ones share one (1500 tokens 33.6 / 28.3,
//    2048 43.7 / 37.7; beyond, 2300 49.2 / 45.0, 3000 63.7 / 63.0, 4096 101.0 /
//    101.5, 8192 354 / 366).
//  - non-causal, up to 1536 keys and two rounds of eight-wave workgroups, the
//    second part empty (4 x 1500, 12 heads, D 64 47.9 / 42.7, 4000 x 1500, 24
//    heads 72.4 / 65.7; beyond, 4000 x 2048 89.5 / 87.7, 8000 x 1024, three
//    rounds, 93.3 / 89.2).  With 129 to 255 eight-wave workgroups, one round,
//    some CUs get two half workgroups and take as long as the eight waves do:
//    what is left is the stage itself, and with more than 1024 keys EFQ is 1-4 %
//    faster there, the LUT and, at D = 128, exp-then-quantize 1-4 % slower (1500
//    x 1500, 24 heads: EFQ 34.5 / 34.0, LUT 37.7 / 38.6, exp 40.9 / 42.2).
// Elsewhere the eight-wave kernel is as fast or faster (7000 x 7000, 24 heads
// 398 / 421).  The LUT stage at D = 128 holds 256 registers and keeps two to
// four more in scratch from before the tile loop to after it; at the lines above
// it gains what EFQ does (2048 tokens 47.0 / 40.2, 8 x 1024 101 / 92, 32760 x 512
// 281 / 240).
bool use_half(const efq_shape* s, int causal, int kind, bool q8) {
#if EFQ_PHASE_STAMPS
  return false;   // the stamped build records the eight-wave kernel
#endif
  const long wg8 = (long)s->batch * s->heads_q * ((s->seq_q + kQTile - 1) / kQTile);
  if (s->seq_q <= kQTile / 2) {   // at most half of the waves have queries
    const bool far = s->heads_q == s->heads_kv && s->seq_k > 8192 && wg8 <= kCUs * 7 / 16;
    return !(far && kind == EFQ_PGEN_EFQ && !q8 && s->head_dim == 128);
  }
  if (s->seq_k <= (causal ? 1024 : 768)) return true;
  if (causal && q8 && s->seq_k <= 6144) return true;
  if (causal) return wg8 <= kCUs;
  if (s->seq_k > 1536 || wg8 > 2 * kCUs) return false;
  if (wg8 <= kCUs / 2 || wg8 >= kCUs) return true;
  const bool exp = kind == EFQ_PGEN_EXPQ || kind == EFQ_PGEN_EXPQ6;
  return s->seq_k <= 1024 || q8 || kind == EFQ_PGEN_EFQ || (exp && s->head_dim == 64);
}

// The calibration runs many candidates in one launch, so the grid is never
// short; the half workgroups win where they do for a large grid (few keys).
bool rho_half(const efq_shape* s, int causal) {
  return s->seq_q <= kQTile / 2 || s->seq_k <= (causal ? 1024 : 768);
}

// The order (map_work) of a causal grid of half workgroups: by length where it
// is resident at once, two on a CU, or where its workgroups do not divide over
// the XCDs; else head by head, whose K and V~ then stay in the XCD's L2.
int work_order(long total, long heads) {
  if (total > 2 * kCUs) return total % 8 ? 2 : 0;
  return heads % 8 ? 2 : 1;
}

// Arguments and grid size of an attention launch (half: the half-workgroup
// kernel), without the dump buffers.
AttnArgs attn_args(const efq_shape* s, float scale, int causal, efq_params p, bool half, unsigned& grid) {
  AttnArgs a;
  a.B = s->batch;
  a.Sq = s->seq_q;
  a.Sk = s->seq_k;
  a.Hq = s->heads_q;
  a.Hkv = s->heads_kv;
  a.nb = (int)padded_blocks(s->seq_k);
  a.scale_off = vhat_scale_offset(s);
  const int br = half ? kWaveQ * kHWaves : kQTile;
  a.nqt = (s->seq_q + br - 1) / br;
  a.scale = scale;
  a.tau = p.tau;
  a.h = p.h;
  a.p_codes = a.p_e8m0 = nullptr;
  a.row_m = a.row_l = nullptr;
  a.nblk = (s->seq_k + 31) / 32;
  const long total = (long)a.B * a.Hq * a.nqt;
  a.xcd_remap = (total % 8 == 0) ? 1 : 0;
  a.spread = half && causal ? work_order(total, (long)a.B * a.Hq) : 0;
  a.sq_pad = (int)pad64(s->seq_q);
  a.sk_pad = (int)pad64(s->seq_k);
  // The pass through LDS pays where the stores are a large part and many
  // workgroups follow one another (direct / rows, us): 8 prompts of 512 tokens,
  // 32 heads 38.0 / 35.7, 32760 x 512, 24 heads 254 / 233, 4000 x 1500 68.9 / 66.1.
  // Beyond the line there is little to gain: a grid that is resident at once 18.3
  // / 17.6 (4 x 512), 28.4 / 28.2 (1500), 12.7 / 12.7 (512), more keys 47.8 / 47.1
  // (3000, MXFP8), 76.0 / 75.7 (4096; LUT 81.5 / 81.8).
  a.o_rows = total > 2 * kCUs && s->seq_k <= 1536;
  a.q8_soff = q8_scale_offset(qhat_rows(s), s->head_dim);
  a.k8_soff = q8_scale_offset(khat_rows(s), s->head_dim);
  grid = (unsigned)total;
  return a;
}

// q8: q and k are the MXFP8 buffers Q^ and K^ of this shape.
int launch_attn(const void* q, const void* k, const void* vhat, float scale, int causal, int kind,
                efq_params p, float* out, const efq_shape* s, hipStream_t st, uint8_t* p_codes,
                uint8_t* p_e8m0, float* row_m, float* row_l, bool q8 = false) {
  const bool dump = p_codes != nullptr;
  const bool half = !dump && kind != EFQ_PGEN_NOOP && use_half(s, causal, kind, q8);
  unsigned g;
  AttnArgs a = attn_args(s, scale, causal, p, half, g);
  a.p_codes = p_codes;
  a.p_e8m0 = p_e8m0;
  a.row_m = row_m;
  a.row_l = row_l;
  auto launch = [&](auto d, auto is_q8) {
    constexpr int D = decltype(d)::value;
    constexpr bool Q8 = decltype(is_q8)::value;
    if (dump) return launch_attn_d<D, true, Q8, false>(kind, causal, q, k, vhat, out, a, st, g);
    if (half) return launch_attn_d<D, false, Q8, true>(kind, causal, q, k, vhat, out, a, st, g);
    return launch_attn_d<D, false, Q8, false>(kind, causal, q, k, vhat, out, a, st, g);
  };
  hipError_t e;
  if (s->head_dim == 64) e = q8 ? launch(IC<64>{}, std::true_type{}) : launch(IC<64>{}, std::false_type{});
  else e = q8 ? launch(IC<128>{}, std::true_type{}) : launch(IC<128>{}, std::false_type{});
  if (e != hipSuccess) return fail(EFQ_EHIP, "attention launch: %s", hipGetErrorString(e));
  return EFQ_OK;
}

// Q^ and K^, and V~ where vhat is given.  One launch for Q and K where their
// thread indices and their threads together fit 32 bits, with V on short calls
// (at lowbit_quant_kernel).
int launch_lowbit_quant(const void* q, const void* k, const void* v, const efq_shape* s, void* qhat,
                        void* khat, void* vhat, hipStream_t st) {
  QuantArgs a;
  a.q = (const unsigned short*)q;
  a.k = (const unsigned short*)k;
  a.v = (const unsigned short*)v;
  a.qhat = (uint8_t*)qhat;
  a.khat = (uint8_t*)khat;
  a.vhat = (uint8_t*)vhat;
  a.qa = q8_args(s->batch, s->seq_q, s->heads_q, s->head_dim);
  a.ka = q8_args(s->batch, s->seq_k, s->heads_kv, s->head_dim);
  a.va = vq_args(s);
  const long tq = q8_threads(a.qa), tk = q8_threads(a.ka), lim = ((long)1 << 32) - 256;
  const long nq = (tq + 255) / 256, nk = (tk + 255) / 256;
  const bool with_v = vhat && a.va.vbytes && nq + nk <= 16384;
  const long nv = with_v ? vq_blocks(a.va) : 0;
  int rc = EFQ_OK;
  if (tq >= lim || tk >= lim || !fits_launch(nv + nq + nk)) {
    rc = launch_q8(q, s->batch, s->seq_q, s->heads_q, s->head_dim, qhat, st);
    if (rc == EFQ_OK) rc = launch_q8(k, s->batch, s->seq_k, s->heads_kv, s->head_dim, khat, st);
  } else {
    a.nv = (unsigned)nv;
    a.nq = (unsigned)nq;
    const dim3 grid((unsigned)(nv + nq + nk));
    if (with_v) hipLaunchKernelGGL(lowbit_quant_kernel<true>, grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL(lowbit_quant_kernel<false>, grid, dim3(256), 0, st, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(EFQ_EHIP, "quantiser launch: %s", hipGetErrorString(e));
  }
  if (rc == EFQ_OK && vhat && !with_v) rc = launch_vquant(v, s, vhat, st);
  return rc;
}

// The key split of a shape (few queries): chunk sizes and the scratch it
// needs, or bytes = 0 where the unsplit kernels take it.  The line lies where
// two estimates (us) cross, both from timed shapes:
//  - unsplit: a tile of keys takes a workgroup 0.6 to 0.75 us; workgroups that
//    share a CU overlap the less the more a tile reads; and no less than K and
//    V~ at 5 TB/s;
//  - split: three launches, and K twice (or once, with the scores stored and
//    read back, while these are fewer bytes) and V~ at 5 TB/s (the partial sums
//    stay in the caches), but no less than 0.9 us per tile and SIMD;
//  - with more than one column tile, each of them reads K again in the second
//    pass, mostly from the caches: a chunk's tiles in turn for every round of
//    the 512 workgroups the chip holds;
//  - once the unsplit kernel fills the chip, only the work counts: it takes
//    every head of a group through K on its own, the split every column tile,
//    at 1.5 of the cost.  Without heads to share K the split gains only where
//    (nearly) every wave of its workgroups has a chunk;
//  - the heavier stages lengthen an unsplit tile, but hide in the split, whose
//    waves wait for K and V~.
// Measured, unsplit / split (us), D 128 unless noted: one query of 32 heads
// against 700 keys 15.3 / 17.4, 4096 52 / 20, 32768 368 / 55; 16 sequences with
// 24 key/value heads of their own against 8192 keys 255 / 467 (K read twice).
// 32/8 heads: 4 x 32 queries, 8000 keys 101 / 68, 8 x 32 111 / 132, 8 x 24 111 /
// 146, 64 x 32, 4096 keys 381 / 575; 12 heads, D 64, 8 x 128, 8000 keys 85 / 142.
// One chunk, where nothing is split but a group's heads share K: 256 x 1, 4096
// keys 1473 / 818; without heads to share it (12, D 64, MXFP8), one chunk 237 x
// 1, 740 keys 68 / 106, five 36 x 1, 9502 keys 111 / 150, four 46 x 1, 6450
// keys 126 / 115.
struct SplitPlan {
  bool scores;                           // keep the scores between the passes
  int R, CT, ntiles, tpc, nch, ngrp;
  size_t cmax, part, ml, sc, bytes;      // byte offsets of the scratch parts, total
};

SplitPlan split_plan(const efq_shape* s, bool q8, int kind) {
  SplitPlan p;
  memset(&p, 0, sizeof p);
  const long R = (long)s->seq_q * (s->heads_q / s->heads_kv);
  if (R > kSRows) return p;
  const int D = s->head_dim;
  const long bg = (long)s->batch * s->heads_kv;
  p.R = (int)R;
  p.CT = (p.R + 31) / 32;
  p.ntiles = (s->seq_k + kBc - 1) / kBc;
  const double tiles = (double)bg * p.CT * p.ntiles;
  const double kb = (double)bg * s->seq_k * D * (q8 ? 33.0 / 32 : 2.0);
  const double vb = (double)bg * s->seq_k * D * (17.0 / 32);
  const double sb = (double)bg * p.ntiles * kBc * 4 * p.R;
  p.scores = p.CT == 1 && 2 * sb <= kb && sb <= kSplitScores;
  p.tpc = (int)std::min<double>(p.ntiles, std::ceil(tiles / kSItems));
  p.nch = (p.ntiles + p.tpc - 1) / p.tpc;
  p.ngrp = (p.nch + kSWaves - 1) / kSWaves;
  const int G = s->heads_q / s->heads_kv;
  const double full = (double)s->batch * s->heads_q * ((s->seq_q + 127) / 128) / kCUs;   // workgroups a CU
  const bool big = D == 128;
  const double once = (kb + vb) / 5e6;
  double unsplit = p.ntiles * (big ? 0.75 : 0.65) * (full <= 1 ? 1.0 : 0.8 * full);
  double split = std::max(once + (p.scores ? 2 * sb : kb) / 5e6, tiles / 1024 * 0.9);
  if (14 + split > 0.9 * (6 + std::max(unsplit, once))) return p;
  if (p.CT == 1) {
    if (full > 1 && G == 1 && p.nch < (kind == EFQ_PGEN_EFQ ? 0.9 : 0.7) * kSWaves * p.ngrp) return p;
  } else {
    const double tile = big ? (q8 ? 0.64 : 0.73) : (q8 ? 0.60 : 0.62);
    const double share = big ? (q8 ? 0.70 : 0.95) : (q8 ? 0.52 : 0.62);
    unsplit = p.ntiles * tile * std::max(1.0, share * full);
    split = std::max((kb * ((p.CT + 1) / 2 + 0.6 * p.CT) + vb * (0.4 + 0.6 * p.CT)) / 6.5e6,
                     p.tpc * std::ceil((double)bg * p.CT * p.ngrp / (2 * kCUs)) *
                         (big ? (q8 ? 2.5 : 5.0) : (q8 ? 1.35 : 2.4)));
    if (full > 1) split = std::min(split, std::max(unsplit, once) * 1.5 * p.CT / G);
    unsplit *= kind == EFQ_PGEN_EFQ ? 1.0 : kind == EFQ_PGEN_LUT ? 1.15 : 1.2;
    if (14 + split > 0.95 * (6 + std::max(unsplit, once))) return p;
  }
  p.cmax = 0;
  p.part = round256((size_t)bg * p.nch * p.CT * 32 * 4);
  p.ml = p.part + round256((size_t)bg * p.ngrp * p.R * D * 4);
  p.sc = p.ml + round256((size_t)bg * p.ngrp * p.R * 8);
  if (p.sc > kSplitSums) return p;   // which also keeps every launch below 2^32 threads
  p.bytes = p.sc + (p.scores ? (size_t)sb : 0);
  return p;
}

// Scratch bytes of the split (a multiple of 256), whichever stage runs: the
// plan that splits wherever another does.
size_t split_bytes(const efq_shape* s, bool q8) { return round256(split_plan(s, q8, EFQ_PGEN_EXPQ).bytes); }

template <int D, bool Q8, bool KEEP, bool RAWV>
hipError_t launch_split_t(int kind, const void* q, const void* k, const void* vhat, float* out,
                          const SplitArgs& a, hipStream_t st) {
  const unsigned bg = (unsigned)(a.B * a.Hkv);
  const unsigned grid_max = bg * a.ngrp * ((a.CT + 1) / 2);
  const dim3 block(64 * kSWaves);
  SplitArgs am = a;
  am.xcd_remap = grid_max % 8 == 0;
  if (a.CT == 1)
    hipLaunchKernelGGL((split_max_kernel<D, Q8, 1, KEEP>), dim3(grid_max), block, 0, st, q, k, am);
  else
    hipLaunchKernelGGL((split_max_kernel<D, Q8, 2, false>), dim3(grid_max), block, 0, st, q, k, am);
  const dim3 grid(bg * a.ngrp * a.CT);
  const uint8_t* v = (const uint8_t*)vhat;
  bool log2 = false;
  switch (kind) {
    case EFQ_PGEN_EFQ:
      hipLaunchKernelGGL((split_attn_kernel<D, EFQ_PGEN_EFQ, Q8, KEEP, RAWV>), grid, block, 0, st, q, k, v, a);
      break;
    case EFQ_PGEN_LUT:
      hipLaunchKernelGGL((split_attn_kernel<D, EFQ_PGEN_LUT, Q8, KEEP, RAWV>), grid, block, 0, st, q, k, v, a);
      break;
    case EFQ_PGEN_EXPQ:
      hipLaunchKernelGGL((split_attn_kernel<D, EFQ_PGEN_EXPQ, Q8, KEEP, RAWV>), grid, block, 0, st, q, k, v, a);
      log2 = true;
      break;
    case EFQ_PGEN_EXPQ6:
      hipLaunchKernelGGL((split_attn_kernel<D, EFQ_PGEN_EXPQ6, Q8, KEEP, RAWV>), grid, block, 0, st, q, k, v, a);
      log2 = true;
      break;
    default:
      return hipErrorInvalidValue;
  }
  if (log2) hipLaunchKernelGGL((split_merge_kernel<D, true>), dim3(bg * a.R), dim3(D), 0, st, out, a);
  else hipLaunchKernelGGL((split_merge_kernel<D, false>), dim3(bg * a.R), dim3(D), 0, st, out, a);
  return hipGetLastError();
}

int launch_split(const void* q, const void* k, const void* vhat, float scale, int kind, efq_params p,
                 float* out, const efq_shape* s, const SplitPlan& pl, void* ws, hipStream_t st, bool q8,
                 bool rawv = false) {
  SplitArgs a;
  a.B = s->batch;
  a.Sq = s->seq_q;
  a.Sk = s->seq_k;
  a.Hq = s->heads_q;
  a.Hkv = s->heads_kv;
  a.nb = (int)padded_blocks(s->seq_k);
  a.scale_off = vhat_scale_offset(s);
  a.R = pl.R;
  a.CT = pl.CT;
  a.ntiles = pl.ntiles;
  a.tpc = pl.tpc;
  a.nch = pl.nch;
  a.ngrp = pl.ngrp;
  a.xcd_remap = (long)a.B * a.Hkv * a.ngrp * a.CT % 8 == 0;
  a.scale = scale;
  a.tau = p.tau;
  a.h = p.h;
  a.sq_pad = (int)pad64(s->seq_q);
  a.sk_pad = (int)pad64(s->seq_k);
  a.q8_soff = q8_scale_offset(qhat_rows(s), s->head_dim);
  a.k8_soff = q8_scale_offset(khat_rows(s), s->head_dim);
  a.cmax = (float*)((uint8_t*)ws + pl.cmax);
  a.part = (float*)((uint8_t*)ws + pl.part);
  a.ml = (float*)((uint8_t*)ws + pl.ml);
  a.sc = (float*)((uint8_t*)ws + pl.sc);
  auto launch = [&](auto d, auto is_q8) {
    constexpr int D = decltype(d)::value;
    constexpr bool Q8 = decltype(is_q8)::value;
    if constexpr (D == 128 && !Q8)
      if (rawv) return launch_split_t<D, Q8, true, true>(kind, q, k, vhat, out, a, st);
    return pl.scores ? launch_split_t<D, Q8, true, false>(kind, q, k, vhat, out, a, st)
                     : launch_split_t<D, Q8, false, false>(kind, q, k, vhat, out, a, st);
  };
  hipError_t e;
  if (s->head_dim == 64) e = q8 ? launch(IC<64>{}, std::true_type{}) : launch(IC<64>{}, std::false_type{});
  else e = q8 ? launch(IC<128>{}, std::true_type{}) : launch(IC<128>{}, std::false_type{});
  if (e != hipSuccess) return fail(EFQ_EHIP, "attention launch: %s", hipGetErrorString(e));
  return EFQ_OK;
}

// Attention on V~ (and Q^, K^ with q8), by the key split where the shape takes
// it and ws (16-byte aligned) has room for its scratch.
int launch_attn_ws(const void* q, const void* k, const void* vhat, float scale, int causal, int kind,
                   efq_params p, float* out, const efq_shape* s, void* ws, size_t ws_bytes,
                   hipStream_t st, bool q8) {
  if (!causal && kind != EFQ_PGEN_NOOP) {
    const SplitPlan pl = split_plan(s, q8, kind);
    if (pl.bytes && ws && ws_bytes >= pl.bytes)
      return launch_split(q, k, vhat, scale, kind, p, out, s, pl, ws, st, q8);
  }
  return launch_attn(q, k, vhat, scale, causal, kind, p, out, s, st, nullptr, nullptr, nullptr,
                     nullptr, q8);
}

// A whole bf16 call: V~ into vhat, then the attention, with split scratch ws.
// Where the split has one column tile (a generation step) and D = 128, it
// quantises V itself and vhat stays unused: V is read once, 8 x 1 query
// against 6001 keys 63.4 -> 55.2 us.
int launch_attn_v(const void* q, const void* k, const void* v, float scale, int causal, int kind,
                  efq_params p, float* out, const efq_shape* s, void* vhat, void* ws, size_t ws_bytes,
                  hipStream_t st) {
  if (!causal && kind != EFQ_PGEN_NOOP && s->head_dim == 128) {
    const SplitPlan pl = split_plan(s, false, kind);
    if (pl.bytes && pl.scores && ws && ws_bytes >= pl.bytes)
      return launch_split(q, k, v, scale, kind, p, out, s, pl, ws, st, false, true);
  }
  const int rc = launch_vquant(v, s, vhat, st);
  if (rc != EFQ_OK) return rc;
  return launch_attn_ws(q, k, vhat, scale, causal, kind, p, out, s, ws, ws_bytes, st, false);
}

int check_kind(int kind, bool allow_noop) {
  if (kind == EFQ_PGEN_EFQ || kind == EFQ_PGEN_EXPQ || kind == EFQ_PGEN_LUT ||
      kind == EFQ_PGEN_EXPQ6)
    return EFQ_OK;
  if (allow_noop && kind == EFQ_PGEN_NOOP) return EFQ_OK;
  return fail(EFQ_EINVAL, "unknown or disallowed P-gen kind %d", kind);
}

int check_params(efq_params p) {
  if (!std::isfinite(p.tau) || !std::isfinite(p.h) || !(p.h > 0.0f))
    return fail(EFQ_EINVAL, "params must be finite with h > 0");
  return EFQ_OK;
}

int check_scale(float scale) {
  if (!std::isfinite(scale) || !(scale > 0.0f)) return fail(EFQ_EINVAL, "scale must be finite and > 0");
  return EFQ_OK;
}

// The objective sums of candidates c0 .. c0 + n - 1 (at most kRhoCand); part:
// n x grid pairs of doubles, res: n pairs.
int launch_rho(const void* q, const void* k, const void* vhat, float scale, int causal,
               const float* o_ref, const efq_shape* s, const float* taus, const float* hs, int nh,
               int c0, int n, double* part, double* res, hipStream_t st) {
  const bool half = rho_half(s, causal);
  unsigned g;
  AttnArgs a = attn_args(s, scale, causal, efq_params{0.0f, 1.0f}, half, g);
  a.spread = 0;   // several candidates are more than the chip holds at once
  RhoArgs cand;
  cand.o_ref = o_ref;
  cand.part = part;
  for (int i = 0; i < kRhoCand; ++i) {
    const int c = c0 + (i < n ? i : 0);
    cand.tau[i] = taus[c / nh];
    cand.h[i] = hs[c % nh];
  }
  auto launch = [&](auto kernel, int threads, int lds) {
    const hipError_t e = raise_lds<decltype(kernel)::value>(lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(decltype(kernel)::value, dim3(g, n), dim3(threads), lds, st, q, k,
                       (const uint8_t*)vhat, (float*)nullptr, a, cand);
    return hipGetLastError();
  };
  auto pick = [&](auto d, auto c) {
    constexpr int D = decltype(d)::value;
    constexpr bool C = decltype(c)::value;
    return half ? launch(KernelPtr<attn_pp_kernel<D, EFQ_PGEN_EFQ, C, false, false, kHWaves, true>>{}, 64 * kHWaves, half_lds<D, false>())
                : launch(KernelPtr<attn_pp_kernel<D, EFQ_PGEN_EFQ, C, false, false, kPPWaves, true>>{}, kPPThreads, SmemPP<D>::kTotal);
  };
  hipError_t e;
  if (s->head_dim == 64) e = causal ? pick(IC<64>{}, std::true_type{}) : pick(IC<64>{}, std::false_type{});
  else e = causal ? pick(IC<128>{}, std::true_type{}) : pick(IC<128>{}, std::false_type{});
  if (e == hipSuccess) {
    hipLaunchKernelGGL(rho_final_kernel, dim3(n), dim3(256), 0, st, part, (long)g, res);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return fail(EFQ_EHIP, "calibration launch: %s", hipGetErrorString(e));
  return EFQ_OK;
}

}  // namespace

// ================================================================== C ABI
extern "C" {

#if EFQ_PHASE_STAMPS
// Diagnostic build only: where the stamped kernel writes its phase stamps
// (device buffer of kStampBlocks * 2 * kStampSlots uint64, zeroed by the
// caller; phases a wave does not reach stay 0), or NULL for none.
int efq_phase_stamps_set(void* buf) {
  unsigned long long* p = (unsigned long long*)buf;
  return hipMemcpyToSymbol(HIP_SYMBOL(g_stamps), &p, sizeof(p)) == hipSuccess ? EFQ_OK : EFQ_EHIP;
}
#endif

int efq_abi_version(void) { return EFQ_ABI_VERSION; }

const char* efq_strerror(int status) {
  if (status == EFQ_OK) return "ok";
  return g_msg;
}

size_t efq_vhat_bytes(const efq_shape* s) {
  if (validate_shape(s, 0) != EFQ_OK) return 0;
  return vhat_bytes(s);
}

size_t efq_vhat_scale_offset(const efq_shape* s) {
  if (validate_shape(s, 0) != EFQ_OK) return 0;
  return vhat_scale_offset(s);
}

size_t efq_attn_split_bytes(const efq_shape* s, int qk8) {
  if (validate_shape(s, 0) != EFQ_OK) return 0;
  return split_bytes(s, qk8 != 0);
}

size_t efq_attn_workspace_bytes(const efq_shape* s) {
  if (validate_shape(s, 0) != EFQ_OK) return 0;
  return vhat_bytes(s) + split_bytes(s, false);
}

int efq_quant_v_mxfp4(const void* v, const efq_shape* s, void* vhat, size_t vhat_nbytes,
                      efq_stream_t stream) {
  int rc = validate_shape(s, 0);
  if (rc) return rc;
  if (!v || !vhat) return fail(EFQ_EINVAL, "null pointer");
  if (!aligned16(v) || !aligned16(vhat)) return fail(EFQ_EINVAL, "pointers must be 16-byte aligned");
  if (vhat_nbytes < vhat_bytes(s))
    return fail(EFQ_EWORKSPACE, "vhat needs %zu bytes, got %zu", vhat_bytes(s), vhat_nbytes);
  if ((rc = check_device())) return rc;
  return launch_vquant(v, s, vhat, (hipStream_t)stream);
}

int efq_attn_fwd_vhat(const void* q, const void* k, const void* vhat, size_t vhat_nbytes,
                      float scale, int causal, int kind, efq_params p, float* out,
                      const efq_shape* s, efq_stream_t stream) {
  return efq_attn_fwd_vhat_ws(q, k, vhat, vhat_nbytes, scale, causal, kind, p, out, s, nullptr, 0, stream);
}

int efq_attn_fwd_vhat_ws(const void* q, const void* k, const void* vhat, size_t vhat_nbytes,
                         float scale, int causal, int kind, efq_params p, float* out,
                         const efq_shape* s, void* ws, size_t ws_bytes, efq_stream_t stream) {
  int rc = validate_shape(s, causal);
  if (rc) return rc;
  if (!q || !k || !vhat || !out) return fail(EFQ_EINVAL, "null pointer");
  if (!aligned16(q) || !aligned16(k) || !aligned16(vhat) || !aligned16(out))
    return fail(EFQ_EINVAL, "pointers must be 16-byte aligned");
  if ((rc = check_kind(kind, true)) || (rc = check_params(p)) || (rc = check_scale(scale))) return rc;
  if (vhat_nbytes < vhat_bytes(s))
    return fail(EFQ_EWORKSPACE, "vhat needs %zu bytes, got %zu", vhat_bytes(s), vhat_nbytes);
  if (ws_bytes != 0 && !ws) return fail(EFQ_EWORKSPACE, "workspace is NULL");
  if (ws && !aligned16(ws)) return fail(EFQ_EINVAL, "workspace must be 16-byte aligned");
  if ((rc = check_device())) return rc;
  return launch_attn_ws(q, k, vhat, scale, causal, kind, p, out, s, ws, ws_bytes, (hipStream_t)stream,
                        false);
}

int efq_attn_fwd_ex(const void* q, const void* k, const void* v, float scale, int causal, int kind,
                    efq_params p, float* out, const efq_shape* s, void* ws, size_t ws_bytes,
                    efq_stream_t stream) {
  int rc = validate_shape(s, causal);
  if (rc) return rc;
  if (!q || !k || !v || !out) return fail(EFQ_EINVAL, "null pointer");
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(out))
    return fail(EFQ_EINVAL, "pointers must be 16-byte aligned");
  if ((rc = check_kind(kind, true)) || (rc = check_params(p)) || (rc = check_scale(scale))) return rc;
  const size_t need = vhat_bytes(s);
  if (ws_bytes != 0 && (!ws || ws_bytes < need))
    return fail(EFQ_EWORKSPACE, "workspace needs %zu bytes, got %zu", need, ws_bytes);
  if (ws && !aligned16(ws)) return fail(EFQ_EINVAL, "workspace must be 16-byte aligned");
  if ((rc = check_device())) return rc;
  hipStream_t st = (hipStream_t)stream;
  void* buf = ws;
  size_t have = ws_bytes;
  if (ws_bytes == 0) {
    have = need + (causal || kind == EFQ_PGEN_NOOP ? 0 : round256(split_plan(s, false, kind).bytes));
    hipError_t e = hipMallocAsync(&buf, have, st);
    if (e != hipSuccess && have > need) {   // unsplit, then
      (void)hipGetLastError();
      have = need;
      e = hipMallocAsync(&buf, have, st);
    }
    if (e != hipSuccess) return fail(EFQ_EHIP, "hipMallocAsync(%zu): %s", have, hipGetErrorString(e));
  }
  rc = launch_attn_v(q, k, v, scale, causal, kind, p, out, s, buf, (uint8_t*)buf + need, have - need, st);
  if (ws_bytes == 0) {
    hipError_t e = hipFreeAsync(buf, st);
    if (rc == EFQ_OK && e != hipSuccess) rc = fail(EFQ_EHIP, "hipFreeAsync: %s", hipGetErrorString(e));
  }
  return rc;
}

}  // extern "C"

namespace {
// Scratch of efq_attn_fwd_noalloc: V~ of one call.  Host code never uses the
// array's name as an address; it uses the device address that
// hipGetSymbolAddress returns for the current device (g_scratch).
static __device__ __align__(256) uint8_t scratch[EFQ_NOALLOC_SCRATCH_BYTES];
std::once_flag g_scratch_once[kMaxDevices];
void* g_scratch[kMaxDevices];
hipError_t g_scratch_err[kMaxDevices];

// Device address of this device's scratch array (looked up once per device,
// with that device current).
int scratch_ptr(void** ptr) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(EFQ_EHIP, "hipGetDevice: %s", hipGetErrorString(e));
  if (dev < 0 || dev >= kMaxDevices) return fail(EFQ_EHIP, "device index %d out of range", dev);
  std::call_once(g_scratch_once[dev], [dev]() {
    void* p = nullptr;
    g_scratch_err[dev] = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    g_scratch[dev] = p;
  });
  if (g_scratch_err[dev] != hipSuccess || g_scratch[dev] == nullptr)
    return fail(EFQ_EHIP, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(g_scratch_err[dev]));
  *ptr = g_scratch[dev];
  return EFQ_OK;
}
}  // namespace

extern "C" {

int efq_attn_fwd_noalloc(const void* q, const void* k, const void* v, float scale, int causal,
                         int kind, efq_params p, float* out, const efq_shape* s,
                         efq_stream_t stream) {
  int rc = validate_shape(s, causal);
  if (rc) return rc;
  if (!q || !k || !v || !out) return fail(EFQ_EINVAL, "null pointer");
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(out))
    return fail(EFQ_EINVAL, "pointers must be 16-byte aligned");
  if ((rc = check_kind(kind, true)) || (rc = check_params(p)) || (rc = check_scale(scale))) return rc;
  const size_t need = vhat_bytes(s);
  if (need > EFQ_NOALLOC_SCRATCH_BYTES)
    return fail(EFQ_EWORKSPACE, "V~ needs %zu bytes, above the %zu-byte scratch of "
                "efq_attn_fwd_noalloc (use efq_attn_fwd_ex with a workspace)",
                need, (size_t)EFQ_NOALLOC_SCRATCH_BYTES);
  if ((rc = check_device())) return rc;
  void* buf = nullptr;
  if ((rc = scratch_ptr(&buf))) return rc;
  hipStream_t st = (hipStream_t)stream;
  // the V quantiser writes every byte of V~ the attention kernel reads, so
  // nothing left by an earlier call needs clearing
  return launch_attn_v(q, k, v, scale, causal, kind, p, out, s, buf, (uint8_t*)buf + need,
                       EFQ_NOALLOC_SCRATCH_BYTES - need, st);
}

int efq_attn_fwd(const void* q, const void* k, const void* v, float scale, int causal, float* out,
                 const efq_shape* s, efq_stream_t stream) {
  return efq_attn_fwd_ex(q, k, v, scale, causal, EFQ_PGEN_EFQ, efq_params{EFQ_TAU_MEAN, EFQ_H_MEAN},
                         out, s, nullptr, 0, stream);
}

int efq_attn_fwd_expq(const void* q, const void* k, const void* v, float scale, int causal,
                      float* out, const efq_shape* s, efq_stream_t stream) {
  return efq_attn_fwd_ex(q, k, v, scale, causal, EFQ_PGEN_EXPQ, efq_params{EFQ_TAU_MEAN, EFQ_H_MEAN},
                         out, s, nullptr, 0, stream);
}

// ------------------------------------------------ low-bit Q K^T (MXFP8)
size_t efq_qhat_bytes(const efq_shape* s) {
  if (validate_shape(s, 0) != EFQ_OK) return 0;
  return q8_bytes(qhat_rows(s), s->head_dim);
}
size_t efq_qhat_scale_offset(const efq_shape* s) {
  if (validate_shape(s, 0) != EFQ_OK) return 0;
  return q8_scale_offset(qhat_rows(s), s->head_dim);
}
size_t efq_khat_bytes(const efq_shape* s) {
  if (validate_shape(s, 0) != EFQ_OK) return 0;
  return q8_bytes(khat_rows(s), s->head_dim);
}
size_t efq_khat_scale_offset(const efq_shape* s) {
  if (validate_shape(s, 0) != EFQ_OK) return 0;
  return q8_scale_offset(khat_rows(s), s->head_dim);
}

int efq_quant_qk_mxfp8(const void* q, const void* k, const efq_shape* s, void* qhat,
                       size_t qhat_nbytes, void* khat, size_t khat_nbytes, efq_stream_t stream) {
  int rc = validate_shape(s, 0);
  if (rc) return rc;
  if (!q || !k || !qhat || !khat) return fail(EFQ_EINVAL, "null pointer");
  if (!aligned16(q) || !aligned16(k) || !aligned16(qhat) || !aligned16(khat))
    return fail(EFQ_EINVAL, "pointers must be 16-byte aligned");
  const size_t nq = q8_bytes(qhat_rows(s), s->head_dim), nk = q8_bytes(khat_rows(s), s->head_dim);
  if (qhat_nbytes < nq) return fail(EFQ_EWORKSPACE, "qhat needs %zu bytes, got %zu", nq, qhat_nbytes);
  if (khat_nbytes < nk) return fail(EFQ_EWORKSPACE, "khat needs %zu bytes, got %zu", nk, khat_nbytes);
  if ((rc = check_device())) return rc;
  return launch_lowbit_quant(q, k, nullptr, s, qhat, khat, nullptr, (hipStream_t)stream);
}

static int check_qk8_args(const void* qhat, size_t qhat_nbytes, const void* khat,
                          size_t khat_nbytes, const void* vhat, size_t vhat_nbytes, float scale,
                          int causal, int kind, bool allow_noop, efq_params p, const float* out,
                          const efq_shape* s) {
  int rc = validate_shape(s, causal);
  if (rc) return rc;
  if (!qhat || !khat || !vhat || !out) return fail(EFQ_EINVAL, "null pointer");
  if (!aligned16(qhat) || !aligned16(khat) || !aligned16(vhat) || !aligned16(out))
    return fail(EFQ_EINVAL, "pointers must be 16-byte aligned");
  if ((rc = check_kind(kind, allow_noop)) || (rc = check_params(p)) || (rc = check_scale(scale)))
    return rc;
  const size_t nq = q8_bytes(qhat_rows(s), s->head_dim), nk = q8_bytes(khat_rows(s), s->head_dim);
  if (qhat_nbytes < nq) return fail(EFQ_EWORKSPACE, "qhat needs %zu bytes, got %zu", nq, qhat_nbytes);
  if (khat_nbytes < nk) return fail(EFQ_EWORKSPACE, "khat needs %zu bytes, got %zu", nk, khat_nbytes);
  if (vhat_nbytes < vhat_bytes(s))
    return fail(EFQ_EWORKSPACE, "vhat needs %zu bytes, got %zu", vhat_bytes(s), vhat_nbytes);
  return EFQ_OK;
}

int efq_attn_fwd_qk8(const void* qhat, size_t qhat_nbytes, const void* khat, size_t khat_nbytes,
                     const void* vhat, size_t vhat_nbytes, float scale, int causal, int kind,
                     efq_params p, float* out, const efq_shape* s, efq_stream_t stream) {
  return efq_attn_fwd_qk8_ws(qhat, qhat_nbytes, khat, khat_nbytes, vhat, vhat_nbytes, scale, causal, kind,
                             p, out, s, nullptr, 0, stream);
}

int efq_attn_fwd_qk8_ws(const void* qhat, size_t qhat_nbytes, const void* khat, size_t khat_nbytes,
                        const void* vhat, size_t vhat_nbytes, float scale, int causal, int kind,
                        efq_params p, float* out, const efq_shape* s, void* ws, size_t ws_bytes,
                        efq_stream_t stream) {
  int rc = check_qk8_args(qhat, qhat_nbytes, khat, khat_nbytes, vhat, vhat_nbytes, scale, causal,
                          kind, true, p, out, s);
  if (rc) return rc;
  if (ws_bytes != 0 && !ws) return fail(EFQ_EWORKSPACE, "workspace is NULL");
  if (ws && !aligned16(ws)) return fail(EFQ_EINVAL, "workspace must be 16-byte aligned");
  if ((rc = check_device())) return rc;
  return launch_attn_ws(qhat, khat, vhat, scale, causal, kind, p, out, s, ws, ws_bytes,
                        (hipStream_t)stream, true);
}

int efq_attn_fwd_qk8_dump(const void* qhat, size_t qhat_nbytes, const void* khat,
                          size_t khat_nbytes, const void* vhat, size_t vhat_nbytes, float scale,
                          int causal, int kind, efq_params p, float* out, const efq_shape* s,
                          uint8_t* p_codes, uint8_t* p_e8m0, float* row_m, float* row_l,
                          efq_stream_t stream) {
  int rc = check_qk8_args(qhat, qhat_nbytes, khat, khat_nbytes, vhat, vhat_nbytes, scale, causal,
                          kind, false, p, out, s);
  if (rc) return rc;
  if (!p_codes || !p_e8m0 || !row_m || !row_l) return fail(EFQ_EINVAL, "null pointer");
  if (!aligned16(p_codes)) return fail(EFQ_EINVAL, "pointers must be 16-byte aligned");
  if ((long)s->batch * s->heads_q * s->seq_q > (1L << 24))
    return fail(EFQ_EUNSUPPORTED, "dump is for small shapes (batch*heads_q*seq_q <= 2^24)");
  if ((rc = check_device())) return rc;
  hipStream_t st = (hipStream_t)stream;
  const size_t rows = (size_t)s->batch * s->heads_q * s->seq_q;
  const size_t nblk = (size_t)(s->seq_k + 31) / 32;
  hipLaunchKernelGGL(fill_zero_kernel, dim3(1024), dim3(256), 0, st, p_codes, rows * nblk * 16);
  hipLaunchKernelGGL(fill_zero_kernel, dim3(1024), dim3(256), 0, st, p_e8m0, rows * nblk);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(EFQ_EHIP, "fill launch: %s", hipGetErrorString(e));
  return launch_attn(qhat, khat, vhat, scale, causal, kind, p, out, s, st, p_codes, p_e8m0, row_m,
                     row_l, true);
}

size_t efq_attn_lowbit_workspace_bytes(const efq_shape* s) {
  if (validate_shape(s, 0) != EFQ_OK) return 0;
  return round256(q8_bytes(qhat_rows(s), s->head_dim)) +
         round256(q8_bytes(khat_rows(s), s->head_dim)) + vhat_bytes(s) + split_bytes(s, true);
}

int efq_attn_fwd_lowbit_ex(const void* q, const void* k, const void* v, float scale, int causal,
                           int kind, efq_params p, float* out, const efq_shape* s, void* ws,
                           size_t ws_bytes, efq_stream_t stream) {
  int rc = validate_shape(s, causal);
  if (rc) return rc;
  if (!q || !k || !v || !out) return fail(EFQ_EINVAL, "null pointer");
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(out))
    return fail(EFQ_EINVAL, "pointers must be 16-byte aligned");
  if ((rc = check_kind(kind, true)) || (rc = check_params(p)) || (rc = check_scale(scale))) return rc;
  const size_t nq = round256(q8_bytes(qhat_rows(s), s->head_dim));
  const size_t nk = round256(q8_bytes(khat_rows(s), s->head_dim));
  const size_t need = nq + nk + vhat_bytes(s);
  if (ws_bytes != 0 && (!ws || ws_bytes < need))
    return fail(EFQ_EWORKSPACE, "workspace needs %zu bytes, got %zu", need, ws_bytes);
  if (ws && ((uintptr_t)ws & 255u) != 0) return fail(EFQ_EINVAL, "workspace must be 256-byte aligned");
  if ((rc = check_device())) return rc;
  hipStream_t st = (hipStream_t)stream;
  void* buf = ws;
  size_t have = ws_bytes;
  if (ws_bytes == 0) {
    have = need + (causal || kind == EFQ_PGEN_NOOP ? 0 : round256(split_plan(s, true, kind).bytes));
    hipError_t e = hipMallocAsync(&buf, have, st);
    if (e != hipSuccess && have > need) {   // unsplit, then
      (void)hipGetLastError();
      have = need;
      e = hipMallocAsync(&buf, have, st);
    }
    if (e != hipSuccess) return fail(EFQ_EHIP, "hipMallocAsync(%zu): %s", have, hipGetErrorString(e));
  }
  uint8_t* qh = (uint8_t*)buf;
  uint8_t* kh = qh + nq;
  uint8_t* vh = kh + nk;
  rc = launch_lowbit_quant(q, k, v, s, qh, kh, vh, st);
  if (rc == EFQ_OK)
    rc = launch_attn_ws(qh, kh, vh, scale, causal, kind, p, out, s, (uint8_t*)buf + need, have - need, st,
                        true);
  if (ws_bytes == 0) {
    hipError_t e = hipFreeAsync(buf, st);
    if (rc == EFQ_OK && e != hipSuccess) rc = fail(EFQ_EHIP, "hipFreeAsync: %s", hipGetErrorString(e));
  }
  return rc;
}

// Workspace of efq_calibrate: V~, the partial sums (as large as one output
// and kRhoPad pairs: room for at least 16 candidates a launch) and one result
// pair per candidate, each 256-byte aligned.
constexpr int kRhoPad = 1024;
static size_t align256(size_t n) { return (n + 255) & ~(size_t)255; }

size_t efq_calibrate_workspace_bytes(const efq_shape* s, int ncand) {
  if (!s || ncand < 1 || validate_shape(s, 0) != EFQ_OK) return 0;
  const size_t out = (size_t)s->batch * s->seq_q * s->heads_q * s->head_dim * 4;
  return align256(vhat_bytes(s)) + align256(out) + align256((size_t)kRhoPad * 16) +
         align256((size_t)ncand * 16);
}

int efq_calibrate(const void* q, const void* k, const void* v, float scale, int causal,
                  const float* o_ref, const efq_shape* s, const float* taus, int ntau,
                  const float* hs, int nh, double* rho, efq_params* best, void* ws,
                  size_t ws_bytes, efq_stream_t stream) {
  int rc = validate_shape(s, causal);
  if (rc) return rc;
  if (!q || !k || !v || !o_ref || !taus || !hs || !best) return fail(EFQ_EINVAL, "null pointer");
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o_ref))
    return fail(EFQ_EINVAL, "pointers must be 16-byte aligned");
  if (ntau < 1 || nh < 1 || (long)ntau * nh > 65536)
    return fail(EFQ_EINVAL, "candidate sets must be non-empty (at most 65536 pairs)");
  if ((rc = check_scale(scale))) return rc;
  for (int i = 0; i < ntau; ++i)
    for (int j = 0; j < nh; ++j)
      if ((rc = check_params(efq_params{taus[i], hs[j]}))) return rc;
  const int nc = ntau * nh;
  const size_t need = efq_calibrate_workspace_bytes(s, nc);
  if (ws_bytes != 0 && (!ws || ws_bytes < need))
    return fail(EFQ_EWORKSPACE, "workspace needs %zu bytes, got %zu", need, ws_bytes);
  if (ws && ((uintptr_t)ws & 255)) return fail(EFQ_EINVAL, "workspace must be 256-byte aligned");
  if ((rc = check_device())) return rc;
  hipStream_t st = (hipStream_t)stream;
  uint8_t* buf = (uint8_t*)ws;
  if (ws_bytes == 0) {
    hipError_t e = hipMallocAsync((void**)&buf, need, st);
    if (e != hipSuccess) return fail(EFQ_EHIP, "hipMallocAsync(%zu): %s", need, hipGetErrorString(e));
  }
  uint8_t* vhat = buf;
  double* part = (double*)(buf + align256(vhat_bytes(s)));
  const size_t room = align256((size_t)s->batch * s->seq_q * s->heads_q * s->head_dim * 4) +
                      align256((size_t)kRhoPad * 16);
  double* res = (double*)((uint8_t*)part + room);
  // Alg. 3: every (tau, h), tau outer, on the same inputs and V~; as many
  // candidates a launch as the partial sums have room for
  const int br = rho_half(s, causal) ? kWaveQ * kHWaves : kQTile;
  const size_t wgs = (size_t)s->batch * s->heads_q * ((s->seq_q + br - 1) / br);
  const int most = (int)std::min<size_t>(kRhoCand, room / (wgs * 16));
  rc = launch_vquant(v, s, vhat, st);
  for (int c = 0; c < nc && rc == EFQ_OK; c += most)
    rc = launch_rho(q, k, vhat, scale, causal, o_ref, s, taus, hs, nh, c, std::min(most, nc - c), part,
                    res + 2 * c, st);
  std::vector<double> sums((size_t)nc * 2);
  if (rc == EFQ_OK) {
    hipError_t e = hipMemcpyAsync(sums.data(), res, sums.size() * sizeof(double),
                                  hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) rc = fail(EFQ_EHIP, "calibration readback: %s", hipGetErrorString(e));
  }
  if (ws_bytes == 0) {
    hipError_t e = hipFreeAsync(buf, st);
    if (rc == EFQ_OK && e != hipSuccess) rc = fail(EFQ_EHIP, "hipFreeAsync: %s", hipGetErrorString(e));
  }
  if (rc != EFQ_OK) return rc;
  if (!(sums[1] > 0.0)) return fail(EFQ_EINVAL, "reference output is zero");
  // Alg. 3: keep the first pair with a strictly smaller objective
  double best_rho = INFINITY;
  int best_c = 0;
  for (int c = 0; c < nc; ++c) {
    const double r = std::sqrt(sums[2 * c]) / std::sqrt(sums[2 * c + 1]);
    if (rho) rho[c] = r;
    if (r < best_rho) {
      best_rho = r;
      best_c = c;
    }
  }
  best->tau = taus[best_c / nh];
  best->h = hs[best_c % nh];
  return EFQ_OK;
}

int efq_attn_fwd_dump(const void* q, const void* k, const void* vhat, size_t vhat_nbytes,
                      float scale, int causal, int kind, efq_params p, float* out,
                      const efq_shape* s, uint8_t* p_codes, uint8_t* p_e8m0, float* row_m,
                      float* row_l, efq_stream_t stream) {
  int rc = validate_shape(s, causal);
  if (rc) return rc;
  if (!q || !k || !vhat || !out || !p_codes || !p_e8m0 || !row_m || !row_l)
    return fail(EFQ_EINVAL, "null pointer");
  if (!aligned16(q) || !aligned16(k) || !aligned16(vhat) || !aligned16(out) || !aligned16(p_codes))
    return fail(EFQ_EINVAL, "pointers must be 16-byte aligned");
  if ((rc = check_kind(kind, false)) || (rc = check_params(p)) || (rc = check_scale(scale))) return rc;
  if (vhat_nbytes < vhat_bytes(s))
    return fail(EFQ_EWORKSPACE, "vhat needs %zu bytes, got %zu", vhat_bytes(s), vhat_nbytes);
  if ((long)s->batch * s->heads_q * s->seq_q > (1L << 24))
    return fail(EFQ_EUNSUPPORTED, "dump is for small shapes (batch*heads_q*seq_q <= 2^24)");
  if ((rc = check_device())) return rc;
  hipStream_t st = (hipStream_t)stream;
  const size_t rows = (size_t)s->batch * s->heads_q * s->seq_q;
  const size_t nblk = (size_t)(s->seq_k + 31) / 32;
  hipLaunchKernelGGL(fill_zero_kernel, dim3(1024), dim3(256), 0, st, p_codes, rows * nblk * 16);
  hipLaunchKernelGGL(fill_zero_kernel, dim3(1024), dim3(256), 0, st, p_e8m0, rows * nblk);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(EFQ_EHIP, "fill launch: %s", hipGetErrorString(e));
  return launch_attn(q, k, vhat, scale, causal, kind, p, out, s, st, p_codes, p_e8m0, row_m, row_l);
}

int efq_pgen(const float* x, int rows, int cols, int kind, efq_params p, uint8_t* codes,
             uint8_t* e8m0, efq_stream_t stream) {
  if (!x || !codes || !e8m0) return fail(EFQ_EINVAL, "null pointer");
  if (rows < 1 || cols < 1) return fail(EFQ_EINVAL, "rows and cols must be >= 1");
  int rc;
  if ((rc = check_kind(kind, false)) || (rc = check_params(p))) return rc;
  const long rt = (rows + 31) / 32, ct = (cols + 63) / 64;
  if (rt * ct > 0x7FFFFFFFL) return fail(EFQ_EUNSUPPORTED, "too many tiles");
  if ((rc = check_device())) return rc;
  PgenKArgs a;
  a.rows = rows;
  a.cols = cols;
  a.nblk = (cols + 31) / 32;
  a.ncb = (int)ct;
  a.tau = p.tau;
  a.h = p.h;
  hipStream_t st = (hipStream_t)stream;
  dim3 grid((unsigned)(rt * ct));
  if (kind == EFQ_PGEN_EFQ)
    hipLaunchKernelGGL(pgen_kernel<EFQ_PGEN_EFQ>, grid, dim3(64), 0, st, x, codes, e8m0, a);
  else if (kind == EFQ_PGEN_LUT)
    hipLaunchKernelGGL(pgen_kernel<EFQ_PGEN_LUT>, grid, dim3(64), 0, st, x, codes, e8m0, a);
  else if (kind == EFQ_PGEN_EXPQ6)
    hipLaunchKernelGGL(pgen_kernel<EFQ_PGEN_EXPQ6>, grid, dim3(64), 0, st, x, codes, e8m0, a);
  else
    hipLaunchKernelGGL(pgen_kernel<EFQ_PGEN_EXPQ>, grid, dim3(64), 0, st, x, codes, e8m0, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(EFQ_EHIP, "pgen launch: %s", hipGetErrorString(e));
  return EFQ_OK;
}

int efq_pgen_bench(int kind, efq_params p, int waves, int iters, uint32_t* checksum,
                   efq_stream_t stream) {
  if (!checksum) return fail(EFQ_EINVAL, "null pointer");
  if (waves < 1 || iters < 1) return fail(EFQ_EINVAL, "waves and iters must be >= 1");
  int rc;
  if ((rc = check_kind(kind, false)) || (rc = check_params(p))) return rc;
  if ((rc = check_device())) return rc;
  hipStream_t st = (hipStream_t)stream;
  dim3 grid((unsigned)((waves + 3) / 4));
  if (kind == EFQ_PGEN_EFQ)
    hipLaunchKernelGGL(pgen_bench_kernel<EFQ_PGEN_EFQ>, grid, dim3(256), 0, st, iters, p.tau, p.h,
                       checksum, waves);
  else if (kind == EFQ_PGEN_LUT)
    hipLaunchKernelGGL(pgen_bench_kernel<EFQ_PGEN_LUT>, grid, dim3(256), 0, st, iters, p.tau, p.h,
                       checksum, waves);
  else if (kind == EFQ_PGEN_EXPQ6)
    hipLaunchKernelGGL(pgen_bench_kernel<EFQ_PGEN_EXPQ6>, grid, dim3(256), 0, st, iters, p.tau,
                       p.h, checksum, waves);
  else
    hipLaunchKernelGGL(pgen_bench_kernel<EFQ_PGEN_EXPQ>, grid, dim3(256), 0, st, iters, p.tau, p.h,
                       checksum, waves);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(EFQ_EHIP, "pgen bench launch: %s", hipGetErrorString(e));
  return EFQ_OK;
}

int efq_clock_probe(int blocks, int iters, uint64_t* out, efq_stream_t stream) {
  if (!out) return fail(EFQ_EINVAL, "null pointer");
  if (blocks < 1 || blocks > 65535 || iters < 1 || iters > (1 << 20))
    return fail(EFQ_EINVAL, "blocks must be in [1, 65535] and iters in [1, 2^20]");
  int rc;
  if ((rc = check_device())) return rc;
  hipStream_t st = (hipStream_t)stream;
  hipLaunchKernelGGL(clock_probe_kernel, dim3((unsigned)blocks), dim3(256), 0, st, iters,
                     (unsigned long long*)out);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(EFQ_EHIP, "clock probe launch: %s", hipGetErrorString(e));
  return EFQ_OK;
}

}  // extern "C"

// Split pass of the decode with the slow RoPE frequencies moved out of the
// per-token work (gfx950).
//
// A score is a sum over RoPE pairs j of
//     cos(w_j d) (q'_j k_j + q'_j+h k_j+h) + sin(w_j d) (q'_j+h k_j - q'_j k_j+h),
// with h = D/2, q' the query rotated back to the middle of the 128-token step and
// d = -64 .. 63 the token's offset from it.  Only the first frequencies turn
// far inside a step.  For the others cos and sin of w_j d are polynomials of degree
// M - 1 in x = d/64, the Chebyshev series cut off (|w_j d| <= 2.44 for M = 8; what is cut
// off stays below 2^-12), written in b_m(x) = z^(m/2) for even m and x z^(m/2) (rounded
// down) for odd ones, z = T_2(x) = 2 x^2 - 1.  Their part of the score is
//     sum_m b_m(x) (W_m . c),   W_m = sum_j coef_mj (B_k rows of j applied to q'),
// with c the token's dequantized latent: the key is never rebuilt nor rotated
// in those dimensions.  W_m (r channels) is formed once per step, head and query
// with MFMA and serves 128 tokens.
//
// Rounding: q', a coefficient, their product and W_m are fp16.  In these functions
// coefficients stay below 1.45, so that the eight terms weigh hardly more than the one key of
// the general kernel (in powers of x they reach 3 and cancel), and the largest one of a
// pair is moved into q' before that is rounded, which leaves it exactly one.  Root mean
// square error of scores against float64, relative to the general kernel's: 0.90 at
// (d, theta) = (64, 700), 0.89 at (128, 700), 0.86 at (128, 5e5), 0.91 at (128, 1e4), at
// most 0.98 over any 16 tokens of a step; in powers of x, coefficients rounded as they
// are, 1.02 at (64, 700) and up to 1.18 over the first tokens.  The T_m themselves are as
// exact, but their recurrence made the 8/4-bit pass over 4 x 128K tokens 84.9 us long,
// two chains in z 81.4 us.
//
// The 16 NHB fastest pairs are rebuilt, rotated and scored per token as the paper
// describes.
//
// Per 32 tokens and 16 channels this takes 1 + NHB matrix instructions
// (32x32x16) instead of D/16 (16x16x32, half as long), and rotates 32 NHB of the D
// dimensions: at d = 128, NHB = 1 the rotation and rebuilding fall to a quarter.
// Counters of the 8/4-bit instance at 4 x 128K tokens (d = 128, NHB = 1): 52.1 vector
// instructions a token (the general kernel 81.1), vector ALUs active in 63 % of the SIMD
// cycles, matrix cores in 23 %, both at once in 11 %; waves wait 39 % of their time.
//
// Work: one workgroup of eight waves per (context split, sequence, group of KV
// heads); a step covers 128 tokens.  A wave owns one KV head and all 128 tokens (NS = 4
// tokens per lane) or half of them (NS = 2), so everything that depends on the
// head is constant in a wave: its key codes and meta go from HBM straight into
// registers, in the layout of the matrix operands, one step ahead.  The
// probabilities of all waves are exchanged through LDS (double buffered, one
// barrier a step), and each wave multiplies them with its slice of the value
// channels, whose codes also arrive in registers.
#include <hip/hip_runtime.h>

#include <atomic>
#include <type_traits>

#include "decode_device.h"

namespace starkv {

// terms of a polynomial; a 32-row matrix tile holds those of four queries
constexpr int M = 8;

typedef float f16v __attribute__((ext_vector_type(16)));
typedef uint32_t u4a __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u2a __attribute__((ext_vector_type(2), aligned(4)));

#if defined(SK_D) && defined(SK_QM)
__device__ __forceinline__ f16v mfma32(h8 a, h8 b, f16v c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}
#endif

// LDS layout (byte offsets), identical on the host.  The areas whose size depends on
// the model come last, so that the other offsets are constants of an instance.
struct PolyLds {
  int q, zero, coef, cs, red, alpha, flag, qmap, pbuf, meta;
  int p_stride;                     // one of the two probability buffers
  static constexpr int kBlockPad = 64;
};
__host__ __device__ constexpr int poly_p_block(int ct) { return 4 * ct * 256 + PolyLds::kBlockPad; }
__host__ __device__ constexpr PolyLds poly_lds(int D, int nhb, int ct) {
  PolyLds L{};
  const int qs = (D + 8) * 2, ks = (D - 32 * nhb) / 16;
  L.q = 0;
  L.zero = L.q + kWaves * (32 / M) * qs;
  L.coef = L.zero + qs;
  L.cs = L.coef + ks * 2 * M * 16;
  L.red = L.cs + nhb * 8192;
  L.alpha = L.red + ct * 16 * 2 * 4;
  L.flag = L.alpha + ct * 16 * 4;
  L.qmap = L.flag + 2 * kWaves * 4;
  L.pbuf = L.qmap + ct * 16 * 4;
  L.p_stride = 4 * poly_p_block(ct);
  L.meta = L.pbuf + 2 * L.p_stride;
  return L;
}
// two buffers of value meta, then the up-projection operands
__host__ __device__ constexpr int poly_meta_bytes(int v_ng) { return 4 * v_ng * 128; }

#if defined(SK_D) && defined(SK_QM)

// ------------------------------------------------------------------ key operands
// A head of NP pairs of 8-channel chunks (rank 16 NP).  Pair p's operand holds
// chunk 2p in lanes 0..31 and chunk 2p + 1 in lanes 32..63.
enum PairKind { kF16, k8, k4, k3, k84, k43 };   // k84 / k43: first chunk wide, second narrow

__host__ __device__ constexpr int wide_chunks(int qm, int np) {
  if (qm == STARKV_Q_MIX8_4) return (np + 1) / 2;
  if (qm == STARKV_Q_MIX4_3) {
    const int v = (16 * np + 20) / 40 > 1 ? (16 * np + 20) / 40 : 1;
    return v < 2 * np ? v : 2 * np;
  }
  return 0;
}
__host__ __device__ constexpr PairKind pair_kind(int qm, int np, int p) {
  const int n = wide_chunks(qm, np);
  if (qm == STARKV_Q_F16) return kF16;
  if (qm == STARKV_Q_INT4) return k4;
  if (qm == STARKV_Q_MIX8_4) return 2 * p + 1 < n ? k8 : 2 * p < n ? k84 : k4;
  return 2 * p + 1 < n ? k4 : 2 * p < n ? k43 : k3;
}
__host__ __device__ constexpr int chunk_group(int qm, int np, int c) {
  const int n = wide_chunks(qm, np);
  return c < n ? c / 4 : (n + 3) / 4 + (c - n) / 4;
}
// bytes per token of a chunk in the wide / narrow region
__host__ __device__ constexpr int wide_bytes(int qm) { return qm == STARKV_Q_MIX8_4 ? 8 : 4; }
__host__ __device__ constexpr int narrow_bytes(int qm) {
  return qm == STARKV_Q_F16 ? 16 : qm == STARKV_Q_MIX4_3 ? 3 : 4;
}
// offset of chunk c in a 16-token block
__host__ __device__ constexpr int chunk_off(int qm, int np, int c) {
  const int n = wide_chunks(qm, np);
  return 16 * (c < n ? c * wide_bytes(qm) : n * wide_bytes(qm) + (c - n) * narrow_bytes(qm));
}
// pair whose meta words pair p shares (the first one in the same two groups)
__host__ __device__ constexpr int meta_pair(int qm, int np, int p) {
  for (int o = 0; o < p; ++o)
    if (chunk_group(qm, np, 2 * o) == chunk_group(qm, np, 2 * p) &&
        chunk_group(qm, np, 2 * o + 1) == chunk_group(qm, np, 2 * p + 1))
      return o;
  return p;
}
// Order of an operand's eight channels: 8-bit and fp16 chunks in order (0), 4- and
// 3-bit ones 0,4,1,5,2,6,3,7 (1), the 4-bit half of an 8/4 pair 0,2,4,6,1,3,5,7 (2).
// The last two are each other's inverse.
__device__ __forceinline__ int chunk_order(int qm, int np, int c) {
  if (qm == STARKV_Q_F16) return 0;
  if (qm != STARKV_Q_MIX8_4) return 1;
  const int n = wide_chunks(qm, np);
  return c < n ? 0 : (n & 1) && c == n ? 2 : 1;
}
__device__ __forceinline__ int chunk_channel(int order, int e) {      // channel of element e
  return order == 0 ? e : order == 1 ? (e >> 1) + 4 * (e & 1) : ((e & 3) << 1) + (e >> 2);
}
__device__ __forceinline__ int chunk_element(int order, int ch) {     // element of channel ch
  return chunk_channel(order ? 3 - order : 0, ch);
}

// (code pair + offset) -> fp16: the codes sit in the mantissa of `base`, whose unit
// in their place is 1; the subtraction is exact and the fma rounds once.
__device__ __forceinline__ uint32_t deq_at(uint32_t bits, _Float16 base, h2 s, h2 z) {
  const h2 c = as_h2(bits) - (h2){base, base};
  return as_u32(__builtin_elementwise_fma(c, s, z));
}
__device__ __forceinline__ h2 lo_lo(uint32_t m) { const h2 v = as_h2(m); return __builtin_shufflevector(v, v, 0, 0); }
__device__ __forceinline__ h2 hi_hi(uint32_t m) { const h2 v = as_h2(m); return __builtin_shufflevector(v, v, 1, 1); }

// Four code pairs of a 32-bit word of 4-bit fields, pair k at bits 4k and 16 + 4k.
// Pairs 0 and 1 stand in the mantissas of 1024 and 64 without a shift.
__device__ __forceinline__ u4 deq4(uint32_t w, const h2 (&s)[4], const h2 (&z)[4]) {
  const uint32_t w8 = w >> 8;
  return (u4){deq_at((w & 0x000F000Fu) | 0x64006400u, (_Float16)1024.0f, s[0], z[0]),
              deq_at((w & 0x00F000F0u) | 0x54005400u, (_Float16)64.0f, s[1], z[1]),
              deq_at((w8 & 0x000F000Fu) | 0x64006400u, (_Float16)1024.0f, s[2], z[2]),
              deq_at((w8 & 0x00F000F0u) | 0x54005400u, (_Float16)64.0f, s[3], z[3])};
}
// Eight 3-bit fields (low 24 bits): pair k = fields k and k + 4.
__device__ __forceinline__ uint32_t halves3(uint32_t x) {
  return (x & 0xFFFu) | ((x << 4) & 0x0FFF0000u);
}
__device__ __forceinline__ u4 deq3(uint32_t x, const h2 (&s)[4], const h2 (&z)[4]) {
  const uint32_t w = halves3(x);
  return (u4){deq_at((w & 0x00070007u) | 0x64006400u, (_Float16)1024.0f, s[0], z[0]),
              deq_at((w & 0x00380038u) | 0x58005800u, (_Float16)128.0f, s[1], z[1]),
              deq_at((w & 0x01C001C0u) | 0x4C004C00u, (_Float16)16.0f, s[2], z[2]),
              deq_at(((w >> 9) & 0x00070007u) | 0x64006400u, (_Float16)1024.0f, s[3], z[3])};
}
// 3-bit fields moved to 4-bit places (the layout of deq4)
__device__ __forceinline__ uint32_t spread3(uint32_t x) {
  const uint32_t w = halves3(x);
  return (w & 0x00070007u) | ((w & 0x00380038u) << 1) | ((w & 0x01C001C0u) << 2) |
         ((w & 0x0E000E00u) << 3);
}
__device__ __forceinline__ u4 deq8(uint32_t lo, uint32_t hi, const h2 (&s)[4], const h2 (&z)[4]) {
  return (u4){deq_pair(perm(0x64646464u, lo, 0x05010400u), s[0], z[0]),
              deq_pair(perm(0x64646464u, lo, 0x05030402u), s[1], z[1]),
              deq_pair(perm(0x64646464u, hi, 0x05010400u), s[2], z[2]),
              deq_pair(perm(0x64646464u, hi, 0x05030402u), s[3], z[3])};
}

// A lane's codes and (scale, zero) words of its NS tokens, per pair.
template <int QM, int NS, int NP>
struct KeyRaw {
  // vectors per pair: fp16 one per token, 8/4-bit NS / 2, else one
  static constexpr int V = QM == STARKV_Q_F16 ? NS : QM == STARKV_Q_MIX8_4 ? NS / 2 : 1;
  using Code = std::conditional_t<QM == STARKV_Q_INT4 && NS == 2, u2, u4>;
  using Meta = std::conditional_t<NS == 2, u2, u4>;
  Code c[NP][V];
  Meta m[NP];
};

// b where the mask's bits are set, else a
__device__ __forceinline__ uint32_t pick(uint32_t mask, uint32_t a, uint32_t b) {
  return (a & ~mask) | (b & mask);
}

// Pairs up to which a head's lane addresses stay in registers across the step loop.
constexpr int kKeepPairs = 2;

// A vector at a wave-uniform base plus a 32-bit lane offset.
template <class T>
__device__ __forceinline__ T load_at(const uint8_t* base, uint32_t off) {
  return *reinterpret_cast<const T*>(base + off);
}

// Loads the codes and meta of a lane's tokens NS cl .. NS cl + NS - 1 of the wave's
// range (code, meta: its first 16-token block) for every pair of the head.
template <int QM, int NS, int NP>
__device__ __forceinline__ void load_keys(const uint8_t* code, const uint8_t* meta, uint32_t row_bytes,
                                          uint32_t ngroups, uint32_t cl, uint32_t hf,
                                          KeyRaw<QM, NS, NP>& raw) {
  constexpr uint32_t RUN = 16 / NS;      // lanes per 16-token block
  constexpr uint32_t WB = wide_bytes(QM), NB = narrow_bytes(QM);
  // (with many pairs the lane offsets are formed in every step, see poly_scores)
  if (NP > kKeepPairs) asm volatile("" : "+v"(cl), "+v"(hf));
  const uint32_t t = cl % RUN;
  const uint32_t blk_off = cl / RUN * (16 * row_bytes);
  const uint32_t meta_off = cl / RUN * (64 * ngroups) + t * NS * 4;
  // lane offsets in pairs of narrow and of wide chunks, and in the mixed pair
  const uint32_t run3 = NS == 4 ? t * 12 : t / 2 * 12;
  const uint32_t on = blk_off + (NB == 3 ? run3 : t * NS * NB) + hf * (16 * NB);
  const uint32_t ow = blk_off + t * NS * WB + hf * (16 * WB);
  const uint32_t om = blk_off + pick(0u - hf, t * NS * WB, 16 * WB + (NB == 3 ? run3 : t * NS * NB));
  using Raw = KeyRaw<QM, NS, NP>;
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const PairKind kind = pair_kind(QM, NP, p);
    const uint8_t* a = code + chunk_off(QM, NP, 2 * p);
    // Pairs of wide chunks (the 4-bit ones of the 4/3-bit format among them), narrow
    // pairs and the mixed pair.  Lanes read whole vectors; what a lane reads past
    // its tokens' codes (8 or 16 bytes at most) lies inside the cache, since the
    // meta planes follow the codes.
    const uint32_t o = kind == k8 || (kind == k4 && QM == STARKV_Q_MIX4_3) ? ow
                       : kind == k84 || kind == k43 ? om : on;
#pragma unroll
    for (int v = 0; v < Raw::V; ++v) {
      if (QM == STARKV_Q_MIX8_4 && kind == k4 && v > 0) continue;
      if constexpr (QM == STARKV_Q_INT4 && NS == 2) raw.c[p][v] = load_at<u2a>(a, o);
      else raw.c[p][v] = load_at<u4a>(a + 16 * v, o);
    }
    if (QM != STARKV_Q_F16 && meta_pair(QM, NP, p) == p) {
      const int ga = chunk_group(QM, NP, 2 * p), gb = chunk_group(QM, NP, 2 * p + 1);
      raw.m[p] = load_at<typename Raw::Meta>(meta + 64 * ga,
                                             meta_off + (gb != ga ? hf * (64 * (gb - ga)) : 0));
    }
  }
}

// The key operand of pair p for the lane's token s.
template <int QM, int NS, int NP>
__device__ __forceinline__ h8 key_operand(const KeyRaw<QM, NS, NP>& raw, int p, int s, int cl, int hf) {
  const PairKind kind = pair_kind(QM, NP, p);
  using Raw = KeyRaw<QM, NS, NP>;
  if constexpr (QM == STARKV_Q_F16) {
    return __builtin_bit_cast(h8, raw.c[p][s]);
  } else {
    // 32-bit word i of the pair's codes
    auto word = [&](int i) -> uint32_t {
      if constexpr (Raw::V == 1) return raw.c[p][0][i];
      else return raw.c[p][i / 4][i % 4];
    };
    const uint32_t mz = raw.m[meta_pair(QM, NP, p)][s];
    const h2 sv = lo_lo(mz), zv = hi_hi(mz);
    const h2 ss[4] = {sv, sv, sv, sv}, zz[4] = {zv, zv, zv, zv};
    // the three bytes of token s among a lane's 3-bit words
    auto word3 = [&](int s) -> uint32_t {
      if (NS == 4)
        return s == 0 ? word(0) : s == 1 ? __builtin_amdgcn_alignbyte(word(1), word(0), 3)
               : s == 2 ? __builtin_amdgcn_alignbyte(word(2), word(1), 2) : word(2) >> 8;
      const uint32_t odd = 0u - (uint32_t)(cl & 1);   // the second two of four tokens
      const uint32_t lo = pick(odd, word(0), __builtin_amdgcn_alignbyte(word(2), word(1), 2));
      const uint32_t hi = pick(odd, word(1), word(2) >> 16);
      return s == 0 ? lo : __builtin_amdgcn_alignbyte(hi, lo, 3);
    };
    u4 v;
    if constexpr (QM == STARKV_Q_MIX8_4) {
      if (kind == k8) {
        v = deq8(word(2 * s), word(2 * s + 1), ss, zz);
      } else if (kind == k84) {
        // 8-bit lanes: two words of codes; 4-bit lanes: nibbles 0,2,4,6 and 1,3,5,7
        // of one word as bytes
        const uint32_t h = 0u - (uint32_t)hf, mk = ~(h & 0xF0F0F0F0u);
        v = deq8(pick(h, word(2 * s), word(s)) & mk,
                 (pick(h, word(2 * s + 1), word(s)) >> (h & 4u)) & mk, ss, zz);
      } else {
        v = deq4(word(s), ss, zz);
      }
    } else if constexpr (QM == STARKV_Q_INT4) {
      v = deq4(word(s), ss, zz);
    } else {
      if (kind == k4) v = deq4(word(s), ss, zz);
      else if (kind == k3) v = deq3(word3(s), ss, zz);
      else {
        v = deq4(pick(0u - (uint32_t)hf, word(s), spread3(word3(s))), ss, zz);
      }
    }
    return __builtin_bit_cast(h8, v);
  }
}

// ------------------------------------------------------------------ kernel
// LDS areas of a wave (wave-uniform).
struct PolyWave {
  const uint8_t* low;      // B_k rows of the slow dimensions, [step][half][row + 1 pad][8 dims]
  const uint8_t* high;     // B_k of the fast dimensions, [block][pair][half][row][8 channels]
  const uint8_t* q;        // the wave's query rows
  const uint8_t* zero;     // a row of zeros
  const uint8_t* coef;     // series coefficients
  const uint8_t* cs;       // rotations of the wave's tokens
};

// Scores of the wave's tokens: x[s][iq] for the lane's token s and query hf + 2 iq.
template <int D, int QM, int NHB, int NS, int NP>
__device__ __forceinline__ void poly_scores(const PolyWave& W, const KeyRaw<QM, NS, NP>& raw, int lane,
                                            int G, float x0, float (&sc)[NS][16 / M]) {
  constexpr int KS = (D - 32 * NHB) / 16;    // 16-dimension steps of the slow dimensions
  constexpr int NT2 = (NP + 1) / 2;
  constexpr int R = 16 * NP;
  // With many pairs the lane's addresses are formed in every step: kept across the
  // loop they would be spilled, and a reload from scratch waits for all loads in
  // flight.
  if (NP > kKeepPairs) asm volatile("" : "+v"(lane));
  const int cl = lane & 31, hf = lane >> 5;
  const int row_a = hf * (R + 1) + cl, row_b = hf * (R + 1) + (cl & 15);
  const uint8_t *qsrc_lo, *qsrc_hi, *qop, *coef, *cs;
  {
    // row (query i, term m) of the products with W_m
    const int m = 4 * ((cl >> 3) & 1) + (cl & 3);
    const int i = ((cl >> 2) & 1) + 2 * (cl >> 4);
    const uint8_t* row = (i < G ? W.q + i * ((D + 8) * 2) : W.zero) + 16 * hf;
    const bool odd = m & 1;
    qsrc_lo = row + (odd ? D : 0) + 32 * NHB;
    qsrc_hi = row + (odd ? 0 : D) + 32 * NHB;
    qop = m == 0 ? row : W.zero + 16 * hf;
    coef = W.coef + (hf * M + m) * 16;
    cs = W.cs + lane * 16;
  }
  // W_m for this step: rows = channels, columns = (query, m); the accumulator
  // layout is the operand layout of the product below
  h8 wop[NP];
  {
    f16v acc[NT2];
#pragma unroll
    for (int t = 0; t < NT2; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[t][e] = 0.0f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const uint8_t* src = ks < KS / 2 ? qsrc_lo + 32 * ks : qsrc_hi + 32 * (ks - KS / 2);
      const h8 qv = *reinterpret_cast<const h8*>(src);
      const h8 cv = *reinterpret_cast<const h8*>(coef + ks * 2 * M * 16);
      const h8 xv = qv * cv;
#pragma unroll
      for (int t = 0; t < NT2; ++t) {
        const int row = (32 * t + 32 <= R ? row_a : row_b) + ks * 2 * (R + 1) + 32 * t;
        const h8 a = *reinterpret_cast<const h8*>(W.low + row * 16);
        acc[t] = mfma32(a, xv, acc[t]);
      }
    }
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      u4 v;
#pragma unroll
      for (int k = 0; k < 4; ++k)
        v[k] = as_u32(__builtin_convertvector(
            (f2){acc[p / 2][8 * (p & 1) + 2 * k], acc[p / 2][8 * (p & 1) + 2 * k + 1]}, h2));
      wop[p] = __builtin_bit_cast(h8, v);
    }
  }
  h8 qlo[NHB], qhi[NHB];
#pragma unroll
  for (int b = 0; b < NHB; ++b) {
    qlo[b] = *reinterpret_cast<const h8*>(qop + b * 32);
    qhi[b] = *reinterpret_cast<const h8*>(qop + D + b * 32);
  }
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    // with many operands they are read again for every token instead of being kept
    int lane_s = lane;
    if (NP * NHB > 4) asm("" : "+v"(lane_s) : "v"(s));
    f16v d, r[NHB];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      d[e] = 0.0f;
#pragma unroll
      for (int b = 0; b < NHB; ++b) r[b][e] = 0.0f;
    }
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const h8 xo = key_operand<QM, NS, NP>(raw, p, s, cl, hf);
#pragma unroll
      for (int b = 0; b < NHB; ++b) {
        const h8 a = *reinterpret_cast<const h8*>(W.high + ((b * NP + p) * 64 + lane_s) * 16);
        r[b] = mfma32(a, xo, r[b]);
      }
      d = mfma32(wop[p], xo, d);
    }
    // rotate the fast pairs (rows 0..7 of the lane: low dimensions, 8..15: high)
    // and score them into the m = 0 rows
#pragma unroll
    for (int b = 0; b < NHB; ++b) {
      const u4 cc = *reinterpret_cast<const u4*>(cs + ((b * (4 / NS) * NS + s) * 2 * 64) * 16);
      const u4 sn = *reinterpret_cast<const u4*>(cs + ((b * (4 / NS) * NS + s) * 2 * 64 + 64) * 16);
      u4 kl, kh;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const h2 a = __builtin_convertvector((f2){r[b][2 * k], r[b][2 * k + 1]}, h2);
        const h2 h = __builtin_convertvector((f2){r[b][8 + 2 * k], r[b][9 + 2 * k]}, h2);
        const h2 c = as_h2(cc[k]), n = as_h2(sn[k]);
        kl[k] = as_u32(__builtin_elementwise_fma(a, c, -(h * n)));
        kh[k] = as_u32(__builtin_elementwise_fma(h, c, a * n));
      }
      d = mfma32(qlo[b], __builtin_bit_cast(h8, kl), d);
      d = mfma32(qhi[b], __builtin_bit_cast(h8, kh), d);
    }
    float x = x0 + (float)s * (1.0f / 64.0f);
    asm volatile("" : "+v"(x));
    const float z = __builtin_fmaf(x + x, x, -1.0f);
#pragma unroll
    for (int iq = 0; iq < 16 / M; ++iq) {
      float even = d[iq * M + M - 2], odd = d[iq * M + M - 1];
#pragma unroll
      for (int m = M - 4; m >= 0; m -= 2) {
        even = __builtin_fmaf(even, z, d[iq * M + m]);
        odd = __builtin_fmaf(odd, z, d[iq * M + m + 1]);
      }
      sc[s][iq] = __builtin_fmaf(odd, x, even);
    }
  }
  // the scores are evaluated here (not after the next step's key loads, where they
  // would keep every token's accumulators alive)
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int iq = 0; iq < 16 / M; ++iq) asm volatile("" : "+v"(sc[s][iq]));
}

// Chebyshev nodes cos th_k = cos(pi (k + 1/2) / 10), k < 5, and the weights of a function's
// values there in its coefficients of z^(m/2) and x z^(m/2), z = T_2(x): those of T_m in the
// series, 2 (2 - [m = 0]) / 10 cos(m th_k), with T_2i = 1, z, 2 z^2 - 1, 4 z^3 - 3 z and
// T_2i+1 / x = 1, 2 z - 1, 4 z^2 - 2 z - 1, 8 z^3 - 4 z^2 - 4 z + 1 collected by powers.
__device__ constexpr float kNodes[5] = {0.987688341f, 0.891006524f, 0.707106781f, 0.4539905f,
                                        0.156434465f};
__device__ constexpr float kWeights8[5][8] = {
    {-0.123606798f, -0.062573786f, -0.324919696f, -0.579265005f, 0.647213595f, 0.40498605f, 0.940456404f, 1.4527696f},
    {0.323606798f, 0.1815962f, 1.37638192f, 2.27113434f, -0.247213595f, 0.448930495f, -1.52169043f, -3.16060269f},
    {0.6f, 1.13137085f, 0.0f, -1.13137085f, -0.8f, -2.2627417f, 0.0f, 2.2627417f},
    {0.323606798f, 0.35640261f, -1.37638192f, -1.60613124f, -0.247213595f, 0.881075706f, 1.52169043f, 0.500590288f},
    {-0.123606798f, -0.395075336f, 0.324919696f, 0.496732614f, 0.647213595f, 2.55698129f, -0.940456404f, -2.85122088f}};

// NHB: fast blocks of 16 RoPE pairs; NS: tokens per lane;
// CT: 16-query tiles; NTW: 16-channel value tiles per wave; MAXP: most pairs (of 8
// channels) of a key head (heads of up to 64 channels have instances of their own, whose
// registers the longer heads' loops do not crowd).
template <int D, int QM, int NHB, int NS, int CT, int NTW, int MAXP>
__global__ __launch_bounds__(kThreads, 1) void decode_split_poly_kernel(PolyParams p) {
  extern __shared__ __align__(16) uint8_t smem[];
  constexpr int HALF = D / 2;
  constexpr int J0 = 16 * NHB;
  constexpr int KS = (D - 32 * NHB) / 16;
  constexpr int QSB = (D + 8) * 2;          // padded query row (bytes)
  constexpr int NQ = 16 / M;                // queries per lane
  constexpr int MQ = 32 / M;                // query rows per wave
  constexpr int TB = 4 / NS;                // waves per head
  constexpr int PB = poly_p_block(CT);
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cl = lane & 31, hf = lane >> 5;
  const int col = lane & 15, quad = lane >> 4;
  // All kernel arguments at once (see PolyParams).
  const int hg = blockIdx.z;
  const PolyWaveInfo info = p.wave[hg][w];
  const int G = p.group_q, nql = p.nql[hg];
  asm volatile("" :: "s"(p.cache), "s"(p.q), "s"(p.bk), "s"(p.ctx_len), "s"(p.part), "s"(p.plan),
               "s"(p.v_code_off), "s"(p.v_meta_off), "s"(p.log2_theta), "s"(p.rmap.table),
               "s"(p.batch), "s"(p.n_q), "s"(p.max_ctx), "s"(p.dyn), "s"(p.cap), "s"(p.rv),
               "s"(p.v_row_bytes), "s"(p.part_stride), "s"(info.code_off), "s"(info.rank),
               "s"(info.slot), "s"(nql));

  // ---------------------------------------------------------------- prologue
  // Loads that need no work item are issued before the context lengths are waited
  // for: the head's B_k rows.
  const int l_ctx = p.dyn ? (lane < p.batch ? p.ctx_len[lane] : 0) : p.ctx_len[blockIdx.y];
  constexpr PolyLds LL = poly_lds(D, NHB, CT);
  const int vmeta_bytes = poly_meta_bytes(p.v_ng);
  uint8_t* frag = smem + LL.meta + 2 * vmeta_bytes + info.frag;
  const int slot = info.slot, tb = info.tb;
  const bool has = info.has != 0;
  const int R = info.rank, np = R / 16;
  const int row_bytes = info.row_bytes, ngroups = info.ngroups;
  const uint8_t* code_plane = p.cache + ((uint64_t)info.code_off << 8);
  const uint8_t* meta_plane = p.cache + ((uint64_t)info.meta_off << 8);
  const int qj = lane & (HALF - 1);
  // B_k rows of the slow dimensions: lane (row lane / VPR, vector lane % VPR) of RPI
  // rows per load, the head's waves taking turns
  constexpr int VPR = D / 8, RPI = 64 / VPR;
  constexpr int kBkBatch = 64 / RPI / TB;    // 64 rows
  const int bk_row = lane / VPR, bk_vec = lane % VPR;
  const uint16_t* bk = p.bk + (int)info.bk_row * D;
  u4 bkv[kBkBatch];
  float b_norm = 0.0f;                       // squares of the rows this wave loads
  auto load_bk = [&](int r0) {
#pragma unroll
    for (int k = 0; k < kBkBatch; ++k) {
      const int r = min(r0 + RPI * (tb + TB * k), R - RPI) + bk_row;   // (ranks are multiples of 16)
      bkv[k] = *reinterpret_cast<const u4*>(bk + r * D + 8 * bk_vec);
    }
  };
  // B_k of the fast dimensions: lane (chunk lane / 4, vector lane % 4: low 0..7, low
  // 8..15, high 0..7, high 8..15 of a block), eight channels of eight dimensions
  // each; the head's waves take turns over the blocks
  u4 fast[8];
  const int fc = min(lane >> 2, R / 8 - 1);
  const int f_order = chunk_order(QM, np, fc);
  auto load_fast = [&](int blk) {
    const uint16_t* src = bk + 16 * blk + 8 * (lane & 1) + (lane & 2 ? HALF : 0);
#pragma unroll
    for (int e = 0; e < 8; ++e)
      fast[e] = *reinterpret_cast<const u4*>(src + (8 * fc + chunk_channel(f_order, e)) * D);
  };
  if (has) {
    load_bk(0);
    load_fast(NHB > 1 ? tb & (NHB - 1) : 0);
  }
  SplitItem item;
  if (!split_item(p, l_ctx, w, lane, &item)) return;
  const int b = item.b;
  const int t_begin = item.split * item.S;
  const int t_end = min(t_begin + item.S, item.L);
  const int n_steps = (t_end - t_begin + kStepTokens - 1) / kStepTokens;
  // paged caches: lane j holds the pool page of the split's j-th page
  const int pg_first = p.rmap.table ? t_begin >> p.rmap.shift : 0;
  int l_page = 0;
  if (p.rmap.table) {
    const int pj = min(pg_first + lane, p.rmap.per_seq - 1);
    const int pg = p.rmap.table[(int64_t)b * p.rmap.per_seq + pj];
    l_page = pg < 0 ? 0 : (pg >= p.rmap.n_pages ? p.rmap.n_pages - 1 : pg);
  }
  auto step_row = [&](int step) -> int64_t {
    const int t = t_begin + step * kStepTokens;
    if (!p.rmap.table) return (int64_t)b * p.rmap.cap_pad + t;
    const int pg = __builtin_amdgcn_readlane(l_page, min((t >> p.rmap.shift) - pg_first, 63));
    return ((int64_t)pg << p.rmap.shift) + (t & ((1 << p.rmap.shift) - 1));
  };
  // value tiles of this wave: lane (channel col, 32-token block quad)
  const int NT = p.rv / 16;
  uint32_t v_off[NTW];
  int v_gi[NTW];
  bool v_wide[NTW];
#pragma unroll
  for (int t = 0; t < NTW; ++t) {
    const int rho = 16 * min(w * NTW + t, NT - 1) + col;   // tiles past the rank repeat the last
    const bool wide = rho < p.v_ro;
    if (QM == STARKV_Q_F16) v_off[t] = rho * 64;
    else if (QM == STARKV_Q_MIX8_4) v_off[t] = wide ? rho * 32 : 32 * p.v_ro + (rho - p.v_ro) * 16;
    else if (QM == STARKV_Q_MIX4_3) v_off[t] = wide ? rho * 16 : 16 * p.v_ro + (rho - p.v_ro) * 12;
    else v_off[t] = rho * 16;
    v_off[t] += quad * 32 * p.v_row_bytes;
    v_gi[t] = wide ? rho / 32 : p.v_ng8 + (rho - p.v_ro) / 32;
    v_wide[t] = wide;
  }
  int vmode = kValues8;
  if (QM != STARKV_Q_F16) {
    bool any_w = false, any_n = false;
    for (int t = 0; t < NTW; ++t) {
      const int nt = min(w * NTW + t, NT - 1);
      any_w |= 16 * nt < p.v_ro;
      any_n |= 16 * nt + 16 > p.v_ro;
    }
    vmode = any_w && any_n ? kValuesMixed : any_w ? kValues8 : kValues4;
  }
  constexpr int VW = QM == STARKV_Q_F16 ? 16 : QM == STARKV_Q_MIX8_4 ? 8 : 4;
  uint32_t vraw[NTW][VW];
  auto load_values = [&](int step) {
    const uint8_t* vb = p.cache + p.v_code_off + (step_row(step) >> 5) * 32 * p.v_row_bytes;
#pragma unroll
    for (int t = 0; t < NTW; ++t) {
      // narrow lanes use the first 16 (4 bits) or 12 (3 bits) bytes; what they read
      // past them lies inside the cache, since the value meta plane follows
#pragma unroll
      for (int k = 0; k < VW / 4; ++k) {
        const u4a v = load_at<u4a>(vb + 16 * k, v_off[t]);
        vraw[t][4 * k] = v.x; vraw[t][4 * k + 1] = v.y; vraw[t][4 * k + 2] = v.z; vraw[t][4 * k + 3] = v.w;
      }
    }
  };
  // value meta of a step: loaded into registers a step ahead, written to LDS before
  // the step's barrier (a buffer per parity: the other one may still be read)
  u4 vmr;                                    // (one 16-byte vector per thread, see plan_poly)
  auto load_vmeta = [&](int step) {
    const uint8_t* src = p.cache + p.v_meta_off + (step_row(step) >> 5) * p.v_ng * 128;
    if (tid * 16 < vmeta_bytes) vmr = load_at<u4>(src, (uint32_t)tid * 16);
  };
  auto store_vmeta = [&](int step) {
    if (tid * 16 < vmeta_bytes)
      *reinterpret_cast<u4*>(smem + LL.meta + (step & 1) * vmeta_bytes + tid * 16) = vmr;
  };
  if (QM != STARKV_Q_F16) load_vmeta(0);
  load_values(0);

  // Queries: lane j holds RoPE pair j of the head's queries (with 32 pairs, the two
  // halves of the wave share them), the rotation of its base position and by one
  // step.  A row in LDS: D dimensions, the fast ones in the order of the rotated
  // key operand.
  constexpr int QL = D == 128 ? MQ : MQ / 2;
  auto qrow = [&](int k) { return D == 128 ? k : (lane >> 5) + 2 * k; };
  uint16_t q_lo[QL], q_hi[QL];
#pragma unroll
  for (int k = 0; k < QL; ++k) {             // (rows past the head's queries repeat the last)
    const uint16_t* qs = static_cast<const uint16_t*>(p.q) +
                         ((int64_t)b * p.n_q + info.head * G + min(qrow(k), G - 1)) * D;
    q_lo[k] = qs[qj];
    q_hi[k] = qs[qj + HALF];
  }
  uint8_t* qbase = smem + LL.q + w * MQ * QSB;
  uint8_t* zero = smem + LL.zero;
  int* qmap = reinterpret_cast<int*>(smem + LL.qmap);         // query head of a probability row
  // turns per token of the lane's RoPE pair, theta^(-2j/D) / (2 pi)
  const double turn = 0.15915494309189533576888376337251 * exp2(-(2.0 * qj / D) * p.log2_theta);
  // Series coefficients of the slow pairs, [slow step][half of it][m][8 dims]: the
  // low dimensions of the pairs, then the high ones, whose odd terms are negated
  // (q'_j k_j+h is subtracted).  Wave m forms b_m's: the Chebyshev series of cos (m
  // even) or sin (m odd) of 64 w_j x, cut off at degree M - 1, by discrete
  // orthogonality over ten nodes (five of either sign: the weights are doubled;
  // 64 w_j <= 2.44 leaves nothing the nodes cannot tell apart).  The largest, b_0's or
  // b_1's there, scales the lane's pair of q' and divides the others.
  float q_coef = 1.0f;
  if (qj >= J0) {
    const float a = (float)(128.0 * turn);   // 64 w_j in half turns
    float c0 = 0.0f, c1 = 0.0f, c = 0.0f;
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      float sn, cn;
      sincospif(a * kNodes[k], &sn, &cn);
      c0 += kWeights8[k][0] * cn;
      c1 += kWeights8[k][1] * sn;
      c += kWeights8[k][w] * (w & 1 ? sn : cn);
    }
    const int top = c1 > c0 ? 1 : 0;
    q_coef = top ? c1 : c0;
    c = w == top ? 1.0f : c / q_coef;
    if (lane < HALF) {
      const int j = lane - J0;
      _Float16* dst = reinterpret_cast<_Float16*>(smem + LL.coef) + ((j >> 3) * M + w) * 8 + (j & 7);
      dst[0] = (_Float16)c;
      dst[KS / 2 * 2 * M * 8] = (_Float16)(w & 1 ? -c : c);
    }
  }
  for (int i = tid; i < QSB / 2; i += kThreads) reinterpret_cast<uint16_t*>(zero)[i] = 0;
  // probability rows that no wave writes stay zero
  for (int i = tid; i < 2 * LL.p_stride / 16; i += kThreads)
    reinterpret_cast<u4*>(smem + LL.pbuf)[i] = (u4){0, 0, 0, 0};
  if (has && tb == 0 && lane < G) qmap[slot * G + lane] = info.head * G + lane;
  // Rotations of the fast pairs for the 128 token offsets of a step: vector
  // (block, token range, s, cos | sin, half, lane), 8 frequencies each.  With the angle
  // reduced in fp64, what is left is the hardware sine's own error: 7e-8 root mean square
  // at (d, theta) = (128, 5e5) and (64, 1e4), where the general kernel's tables have
  // 4e-7 and 2.6e-7.
  if (w < NHB * 4) {
    const int s = w % NS, tr = w / NS % TB, blk = w / 4;
    const double u = (double)(32 * NS * tr + NS * cl + s - 64);
    u4 cv, sv;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      float cc[2], ss[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int r = 2 * k + e;             // lane j holds pair j's turns
        const double a = u * __shfl(turn, 16 * blk + 8 * (r >> 2) + 4 * hf + (r & 3));
        const float f = (float)(a - floor(a));
        ss[e] = __builtin_amdgcn_sinf(f);
        cc[e] = __builtin_amdgcn_cosf(f);
      }
      cv[k] = as_u32(__builtin_convertvector((f2){cc[0], cc[1]}, h2));
      sv[k] = as_u32(__builtin_convertvector((f2){ss[0], ss[1]}, h2));
    }
    u4* dst = reinterpret_cast<u4*>(smem + LL.cs) + w * 128 + lane;
    dst[0] = cv;
    dst[64] = sv;
  }
  // B_k operands of the head, shared by its waves.  Slow dimensions: row i =
  // channel of accumulator row i (see poly_scores), eight consecutive dimensions
  // per 16-byte vector, a plane of R + 1 rows (the odd stride spreads a row's
  // vectors over the banks) per step and half; fast dimensions: transposed, eight
  // channels of one dimension per vector.
  const int low_bytes = (R + 1) * KS * 32;
  uint8_t* low = frag;
  uint8_t* high = low + low_bytes;
  auto store_bk = [&](int r0) {
#pragma unroll
    for (int k = 0; k < kBkBatch; ++k)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        b_norm = __builtin_amdgcn_fdot2(as_h2(bkv[k][e]), as_h2(bkv[k][e]), b_norm, false);
    const int jj = 8 * (bk_vec % (VPR / 2)), up = bk_vec / (VPR / 2);   // pair, high half
    const int ks = ((jj - J0) >> 4) + up * (KS / 2), kc = bk_vec & 1;
    if (jj < J0) return;
    uint8_t* plane = low + (ks * 2 + kc) * (R + 1) * 16;
#pragma unroll
    for (int k = 0; k < kBkBatch; ++k) {
      const int rb = r0 + RPI * (tb + TB * k);
      if (rb < R) {
        const int ch = rb + bk_row, c = ch >> 3;
        const int rr = 8 * (c >> 1 & 1) + chunk_element(chunk_order(QM, np, c), ch & 7);
        const int row = 32 * (ch >> 5) + 8 * (rr >> 2) + 4 * (c & 1) + (rr & 3);
        *reinterpret_cast<u4*>(plane + row * 16) = bkv[k];
      }
    }
  };
  auto store_fast = [&](int blk) {
    if ((lane >> 2) < R / 8) {
      uint8_t* dst = high + ((blk * np + (fc >> 1)) * 64 + 32 * (fc & 1) + 16 * (lane >> 1 & 1) + 8 * (lane & 1)) * 16;
#pragma unroll
      for (int i = 0; i < 8; ++i) {          // dimension i of the lane's eight
        u4 v;
#pragma unroll
        for (int k = 0; k < 4; ++k)
          v[k] = perm(fast[2 * k + 1][i / 2], fast[2 * k][i / 2], i & 1 ? 0x07060302u : 0x05040100u);
        *reinterpret_cast<u4*>(dst + i * 16) = v;
      }
    }
  };
  if (has) {
    store_bk(0);
    for (int r0 = RPI * TB * kBkBatch; r0 < R; r0 += RPI * TB * kBkBatch) {
      load_bk(r0);
      store_bk(r0);
    }
    // one block: both waves of a head write the same values; two blocks: one each, or
    // both by the one wave
    store_fast(NHB > 1 ? tb & (NHB - 1) : 0);
    if (NHB > TB) {
      load_fast(1);
      store_fast(1);
    }
  }
  uint32_t qr[QL];                           // (low, high) dimension of the lane's pair
#pragma unroll
  for (int k = 0; k < QL; ++k) qr[k] = q_lo[k] | ((uint32_t)q_hi[k] << 16);
  // angles in turns, reduced in fp64; the base position's rotation is evaluated there, too
  auto turns = [&](double t) {
    const double a = t * turn;
    return 2.0 * (a - floor(a));
  };
  float2 rot, rot_step;
  {
    double sn, cn;
    sincospi(turns((double)(t_begin + 64)), &sn, &cn);
    rot = make_float2((float)cn, (float)sn);
    sincospif((float)turns((double)kStepTokens), &rot_step.y, &rot_step.x);
  }
  rot.x *= q_coef;
  rot.y *= q_coef;

  const PolyWave W = {frag, frag + low_bytes, qbase, zero, smem + LL.coef,
                      smem + LL.cs + tb * NS * 2048};
  // position of the lane's pair in a query row
  const int qpos = qj < J0 ? (qj & ~15) + ((qj >> 2) & 1) * 8 + 4 * ((qj >> 3) & 1) + (qj & 3) : qj;
  auto wave_sync = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  auto query = [&](int k, float* lo, float* hi) {   // the lane's pair of its query k
    if (p.q_bf16) {
      *lo = __uint_as_float(qr[k] << 16);
      *hi = __uint_as_float(qr[k] & 0xFFFF0000u);
    } else {
      const h2 v = as_h2(qr[k]);
      *lo = (float)v[0];
      *hi = (float)v[1];
    }
  };
  // A query row is scaled by a power of two that keeps its products within fp16: an
  // element of W_m is at most 1.5 |q'| |B_k| (the coefficients moved into q' are below 1.45,
  // the others at most one; the norms are those of the head's queries and of its B_k, whole), and an operand
  // coef * q' at most 1.5 |q'|.  With the larger of the two at 2^13 .. 2^15, W_m neither
  // overflows nor loses bits to subnormals wherever the key itself stays in fp16.  The
  // scores stay scaled up to the softmax and the candidates, where a product with s_scale
  // (a power of two, exact) replaces them.  (alpha_s is free until the loop's first
  // barrier.)
  float q_norm = 0.0f;
  float* alpha_s = reinterpret_cast<float*>(smem + LL.alpha);
  if (has) {
#pragma unroll
    for (int k = 0; k < QL; ++k) {
      float lo, hi;
      query(k, &lo, &hi);
      q_norm = __builtin_fmaf(lo, lo, __builtin_fmaf(hi, hi, q_norm));
    }
    q_norm = wave_sum(q_norm);
    b_norm = wave_sum(b_norm);
    if (lane == 0) alpha_s[slot * TB + tb] = b_norm;
  }
  float q_scale = p.score_scale, s_scale = 1.0f, lazy = kLazyMargin;
  auto set_scale = [&]() {
    float bn = alpha_s[slot * TB];
    if (TB > 1) bn += alpha_s[slot * TB + 1];
    const float u2 = 2.25f * p.score_scale * p.score_scale * q_norm * fmaxf(bn, 1.0f);
    // u2 < 2^(2x), at least a quarter of it; norms that are not finite scale nothing
    const int e = u2 < INFINITY ? __builtin_amdgcn_frexp_expf(u2) : 30;
    const int x = __builtin_amdgcn_readfirstlane(min(max((e + 1) >> 1, -60), 60));
    q_scale = __int_as_float(__float_as_int(p.score_scale) + ((15 - x) << 23));   // times 2^(15 - x)
    s_scale = __int_as_float((127 - 15 + x) << 23);
    lazy = __int_as_float(__float_as_int(kLazyMargin) + ((15 - x) << 23));
  };
  auto store_q = [&]() {
    wave_sync();
    const float c = rot.x * q_scale, n = rot.y * q_scale;
#pragma unroll
    for (int k = 0; k < QL; ++k) {
      const int i = qrow(k);
      if (i < G) {
        float lo, hi;
        query(k, &lo, &hi);
        _Float16* d = reinterpret_cast<_Float16*>(qbase + i * QSB);
        d[qpos] = (_Float16)__builtin_fmaf(lo, c, hi * n);
        d[HALF + qpos] = (_Float16)__builtin_fmaf(hi, c, -(lo * n));
      }
    }
    wave_sync();
  };

  // softmax state of the lane's queries hf + 2 iq, and the two largest scores of each
  // of its token slots (see the candidates below)
  float m_run[NQ], l_part[NQ], b1[NS][NQ], b2[NS][NQ];
#pragma unroll
  for (int iq = 0; iq < NQ; ++iq) {
    m_run[iq] = -INFINITY;
    l_part[iq] = 0.0f;
#pragma unroll
    for (int s = 0; s < NS; ++s) b1[s][iq] = b2[s][iq] = -INFINITY;
  }
  f4 acc_v[CT][NTW];
#pragma unroll
  for (int c = 0; c < CT; ++c)
#pragma unroll
    for (int t = 0; t < NTW; ++t) acc_v[c][t] = (f4){0, 0, 0, 0};
  float* red = reinterpret_cast<float*>(smem + LL.red);       // [CT * 16][2]
  int* flag_s = reinterpret_cast<int*>(smem + LL.flag);       // [2][kWaves]
  // token u of the step held by the lane as its token s, and its place in the
  // probability operand: 32-token block u / 32, chunk u % 4, slot
  auto token = [&](int s) { return 32 * NS * tb + NS * cl + s; };
  auto p_off = [&](int s) {
    const int u = token(s), v = u & 31;
    return (u >> 5) * PB + (v & 3) * (CT * 256) + (4 * (v >> 4) + ((v & 15) >> 2)) * 2;
  };
  const int row0 = has ? slot * G : 0;       // first probability row of the head
  const float x0 = (float)(token(0) - 64) * (1.0f / 64.0f);

  // ---------------------------------------------------------------- main loop
  // One copy of the loop per pair count (NP = 0: no head), so that the prefetched
  // codes are carried in registers of their own: merged over the counts they
  // would be copied, and waited for, right after their loads.  The loads of the
  // next step are not conditional (the last step's read its own rows again) and
  // stay within the step's 128 rows, which the cache holds.
  auto run = [&](auto np_tag) {
  constexpr int NP = decltype(np_tag)::value;
  constexpr bool has = NP > 0;
  KeyRaw<QM, NS, has ? NP : 1> raw;
  auto load_raw = [&](int step) {
    if constexpr (has) {
      const int64_t blk = (step_row(step) + 32 * NS * tb) >> 4;
      load_keys<QM, NS, NP>(code_plane + blk * 16 * row_bytes, meta_plane + blk * ngroups * 64,
                            row_bytes, ngroups, cl, hf, raw);
    }
  };
  load_raw(0);
  __syncthreads();   // operands, tables, norms and zeroed probabilities visible
  if constexpr (has) set_scale();
  for (int step = 0; step < n_steps; ++step) {
    const int t_step = t_begin + step * kStepTokens;
    const bool full = t_step + kStepTokens <= t_end;
    const int next = min(step + 1, n_steps - 1);
    uint8_t* pb = smem + LL.pbuf + (step & 1) * LL.p_stride;
    int* fl = flag_s + (step & 1) * kWaves;
    float x[NS][NQ];
    float ls[NQ];
    bool any_over = false;
    if constexpr (has) {
      store_q();
      poly_scores<D, QM, NHB, NS, NP>(W, raw, lane, G, x0, x);
      load_raw(next);
      // a score's token (step and, below, its place among the lanes of a slot)
      // replaces the low 8 of its 24 significand bits, far below the score's
      // fp16 error; softmax and rescoring use the same value
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const uint32_t tag = (uint32_t)(4 * step) + (((token(s) & 15) >> 2));
#pragma unroll
        for (int iq = 0; iq < NQ; ++iq)
          x[s][iq] = __uint_as_float((__float_as_uint(x[s][iq]) & 0xFFFFFF00u) | tag);
      }
      if (!full) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          const bool out = t_step + token(s) >= t_end;
#pragma unroll
          for (int iq = 0; iq < NQ; ++iq) x[s][iq] = out ? -INFINITY : x[s][iq];
        }
      }
      rot = cmul(rot, rot_step);
      // Probabilities against a reference maximum per query that is raised (with
      // a rescale of the accumulators) only when a score exceeds it by more than
      // kLazyMargin; the first step always sets it.
      auto softmax = [&](auto all_tag) {
        constexpr bool ALL = decltype(all_tag)::value;   // every lane row holds a query
        float mx[NQ];
        bool over = false;
#pragma unroll
        for (int iq = 0; iq < NQ; ++iq) {
          mx[iq] = -INFINITY;
#pragma unroll
          for (int s = 0; s < NS; ++s) {
            const float v = x[s][iq];
            mx[iq] = fmaxf(mx[iq], v);
            b2[s][iq] = __builtin_amdgcn_fmed3f(b1[s][iq], b2[s][iq], v);   // b1 >= b2
            b1[s][iq] = fmaxf(b1[s][iq], v);
          }
          over |= (ALL || hf + 2 * iq < G) && mx[iq] > m_run[iq] + lazy;
        }
        any_over = __any(over);
        if (any_over) {
#pragma unroll
          for (int iq = 0; iq < NQ; ++iq) {
            mx[iq] = reduce_lanes<32>(mx[iq], [](float u, float v) { return fmaxf(u, v); });
            if (cl == 0 && (ALL || hf + 2 * iq < G)) red[(row0 + hf + 2 * iq) * 2 + tb] = mx[iq];
          }
        } else if (cl == 0) {
#pragma unroll
          for (int iq = 0; iq < NQ; ++iq)
            if (ALL || hf + 2 * iq < G) red[(row0 + hf + 2 * iq) * 2 + tb] = -INFINITY;
        }
#pragma unroll
        for (int iq = 0; iq < NQ; ++iq) {
          float l = 0.0f;
          if (ALL || hf + 2 * iq < G) {
            uint8_t* pr = pb + (row0 + hf + 2 * iq) * 16;
            const float ms = m_run[iq] * s_scale;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
              const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(x[s][iq], s_scale, -ms));
              l += e;
              *reinterpret_cast<_Float16*>(pr + p_off(s)) = (_Float16)e;
            }
          }
          ls[iq] = l;
        }
      };
      if (G == MQ) softmax(std::true_type{});
      else softmax(std::false_type{});
    }
    if (lane == 0) fl[w] = any_over ? 1 : 0;
    if (QM != STARKV_Q_F16) store_vmeta(step);
    lds_barrier();   // probabilities, maxima, flags and value meta visible
    const int4 f0 = *reinterpret_cast<const int4*>(fl);
    const int4 f1 = *reinterpret_cast<const int4*>(fl + 4);
    if ((f0.x | f0.y | f0.z | f0.w | f1.x | f1.y | f1.z | f1.w) != 0) {
      if constexpr (has) {
#pragma unroll
        for (int iq = 0; iq < NQ; ++iq) {
          const int i = hf + 2 * iq;
          if (i < G) {
            float mn = m_run[iq];
#pragma unroll
            for (int k = 0; k < TB; ++k) mn = fmaxf(mn, red[(row0 + i) * 2 + k]);
            const float ms = mn * s_scale;
            const float al = __builtin_amdgcn_exp2f(__builtin_fmaf(m_run[iq], s_scale, -ms));   // m_run = -inf first: 0
            m_run[iq] = mn;
            uint8_t* pr = pb + (row0 + i) * 16;
            float l = 0.0f;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
              const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(x[s][iq], s_scale, -ms));
              l += e;
              *reinterpret_cast<_Float16*>(pr + p_off(s)) = (_Float16)e;
            }
            l_part[iq] = l_part[iq] * al + l;
            if (cl == 0 && tb == 0) alpha_s[row0 + i] = al;
          }
        }
      }
      lds_barrier();   // new probabilities and rescale factors visible
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        const f4 al = *reinterpret_cast<const f4*>(alpha_s + c * 16 + 4 * quad);
#pragma unroll
        for (int t = 0; t < NTW; ++t) acc_v[c][t] *= al;
      }
    } else if constexpr (has) {
#pragma unroll
      for (int iq = 0; iq < NQ; ++iq) l_part[iq] += ls[iq];
    }

    // ------------------------------------------ values: acc += P . V'
    // matrix step j: the four 32-token blocks' chunks j (block = lane quad)
    const uint8_t* mbase = smem + LL.meta + (step & 1) * vmeta_bytes;
    auto values = [&](auto vm_tag, auto full_tag) {
      constexpr int VM = decltype(vm_tag)::value;
      constexpr bool FULL = decltype(full_tag)::value;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        h8 pa[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c)
          pa[c] = *reinterpret_cast<const h8*>(pb + quad * PB + (j * CT + c) * 256 + col * 16);
        u4 vmask;
        if (!FULL) {
          // slots 2k, 2k+1: tokens j + 8k + {0,4} (k < 2), 16 + j + 8(k-2) + {0,4}
          const int tq = t_step + 32 * quad + j;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int t0 = tq + (k < 2 ? 8 * k : 16 + 8 * (k - 2));
            vmask[k] = (t0 < t_end ? 0x0000FFFFu : 0u) | (t0 + 4 < t_end ? 0xFFFF0000u : 0u);
          }
        }
#pragma unroll
        for (int t = 0; t < NTW; ++t) {
          const uint32_t* r = vraw[t];
          u4 v;
          if (QM == STARKV_Q_F16) {
            constexpr int F = QM == STARKV_Q_F16 ? 4 : 0;
            v = (u4){r[F * j], r[F * j + (F ? 1 : 0)], r[F * j + (F ? 2 : 0)], r[F * j + (F ? 3 : 0)]};
          } else {
            const uint8_t* mb = mbase + ((quad * p.v_ng + v_gi[t]) * 4 + j) * 32;
            const u4 sv = *reinterpret_cast<const u4*>(mb), zv = *reinterpret_cast<const u4*>(mb + 16);
            const h2 ss[4] = {as_h2(sv.x), as_h2(sv.y), as_h2(sv.z), as_h2(sv.w)};
            const h2 zz[4] = {as_h2(zv.x), as_h2(zv.y), as_h2(zv.z), as_h2(zv.w)};
            if (QM == STARKV_Q_MIX4_3) {
              const uint32_t x3 = j == 0 ? r[0] : j == 1 ? __builtin_amdgcn_alignbyte(r[1], r[0], 3)
                                  : j == 2 ? __builtin_amdgcn_alignbyte(r[2], r[1], 2) : r[2] >> 8;
              if (VM == kValues8) v = deq4(r[j], ss, zz);
              else if (VM == kValues4) v = deq3(x3, ss, zz);
              else v = deq4(v_wide[t] ? r[j] : spread3(x3), ss, zz);
            } else if (QM == STARKV_Q_MIX8_4) {
              constexpr int F = QM == STARKV_Q_MIX8_4 ? 2 : 0;
              if (VM == kValues4) {
                v = deq4(r[j], ss, zz);
              } else {
                const u4 v8 = deq8(r[F * j], r[F * j + (F ? 1 : 0)], ss, zz);
                v = v8;
                if (VM == kValuesMixed) v = v_wide[t] ? v8 : deq4(r[j], ss, zz);
              }
            } else {
              v = deq4(r[j], ss, zz);
            }
          }
          if (!FULL) v &= vmask;
          const h8 vop = __builtin_bit_cast(h8, v);
#pragma unroll
          for (int c = 0; c < CT; ++c) acc_v[c][t] = mfma16(pa[c], vop, acc_v[c][t]);
        }
      }
    };
    using Full = std::true_type;
    if (!full) values(std::integral_constant<int, QM == STARKV_Q_INT4 ? kValues4 : kValuesMixed>{}, std::false_type{});
    else if (QM == STARKV_Q_INT4 || vmode == kValues4) values(std::integral_constant<int, kValues4>{}, Full{});
    else if (vmode == kValues8) values(std::integral_constant<int, kValues8>{}, Full{});
    else values(std::integral_constant<int, kValuesMixed>{}, Full{});
    if (QM != STARKV_Q_F16) load_vmeta(next);
    load_values(next);
  }
  };
  switch (has ? np : 0) {
    case 0: run(std::integral_constant<int, 0>{}); break;
    case 1: run(std::integral_constant<int, 1>{}); break;
    case 2: run(std::integral_constant<int, 2>{}); break;
    case 3: run(std::integral_constant<int, 3>{}); break;
    case 4: run(std::integral_constant<int, 4>{}); break;
    case 5: if constexpr (MAXP >= 5) run(std::integral_constant<int, (MAXP >= 5 ? 5 : 1)>{}); break;
    case 6: if constexpr (MAXP >= 6) run(std::integral_constant<int, (MAXP >= 6 ? 6 : 1)>{}); break;
    case 7: if constexpr (MAXP >= 7) run(std::integral_constant<int, (MAXP >= 7 ? 7 : 1)>{}); break;
    case 8: if constexpr (MAXP >= 8) run(std::integral_constant<int, (MAXP >= 8 ? 8 : 1)>{}); break;
  }

  // ---------------------------------------------------------------- partials
  // (the last step's readers of red are past a barrier)
#pragma unroll
  for (int iq = 0; iq < NQ; ++iq)
    l_part[iq] = reduce_lanes<32>(l_part[iq], [](float u, float v) { return u + v; });
  if (TB > 1) {                              // the head's waves hold parts of the sum
    if (has && cl == 0) {
#pragma unroll
      for (int iq = 0; iq < NQ; ++iq)
        if (hf + 2 * iq < G) red[(row0 + hf + 2 * iq) * 2 + tb] = l_part[iq];
    }
    lds_barrier();
  }
  const int64_t pbase = (int64_t)item.pitem * p.n_q;
  // Candidates for the exact rescoring: the two largest scores of each of 32 token
  // slots per query, a slot being the tokens of a 16-token block (of every
  // 128-token step) that are equal modulo 4.  The lanes of a slot, 4 tokens apart,
  // merge their two largest first.  Blocks of 16 entries (32 tokens each), their
  // bounds q and the test for writing them as described at the general split
  // kernel: with m and l this split's maximum and normalizer, a score x has the
  // rescoring priority 2^(x - M) (1 + |x|) / L <= 2^(m - M) q / L, q = max over the
  // block of 2^(x - m) (1 + |x|), and at most q / l; a block whose q misses half the
  // threshold times l is never rescored and is not written.
  if (has) {
    constexpr int S1 = 4 / NS, S2 = 8 / NS;  // lane distance of tokens 4 and 8 apart
#pragma unroll
    for (int iq = 0; iq < NQ; ++iq) {
      const int i = hf + 2 * iq;
      const bool ok = i < G;
      const int row = row0 + (ok ? i : 0);
      const float lt = TB > 1 ? red[row * 2] + red[row * 2 + 1] : l_part[iq];
      const float bar = 0.5f * kRescoreTau * lt;
      const float mr = m_run[iq] * s_scale;
      auto bound = [&](float v) {
        const float u = v * s_scale;
        return v == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(u - mr) * (1.0f + fabsf(u));
      };
      float qb = 0.0f;
#pragma unroll
      for (int s = 0; s < NS; ++s) qb = fmaxf(qb, fmaxf(bound(b1[s][iq]), bound(b2[s][iq])));
      qb = reduce_lanes<32 / NS>(qb, [](float u, float v) { return fmaxf(u, v); });
      const int u0 = token(0);
      const int tg = u0 >> 5;                // 32-token block of the lane
      const bool any = ok && qb >= bar;
      const int64_t qrow_out = pbase + info.head * G + i;
      if (ok && (cl & (32 / NS - 1)) == 0) {
        float* dst = p.part + qrow_out * p.part_stride + p.rv;
        reinterpret_cast<uint8_t*>(dst + 2)[tg] = any ? 1 : 0;
        dst[4 + tg] = qb;
      }
      if (any) {                             // (the same in all lanes of a slot)
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            const int o = k ? S2 : S1;
            float c1, c2;
            if (NS == 4) {                   // within four lanes
              c1 = k ? dpp<0x4E>(b1[s][iq]) : dpp<0xB1>(b1[s][iq]);
              c2 = k ? dpp<0x4E>(b2[s][iq]) : dpp<0xB1>(b2[s][iq]);
            } else {
              c1 = __shfl_xor(b1[s][iq], o);
              c2 = __shfl_xor(b2[s][iq], o);
            }
            b2[s][iq] = fmaxf(fmaxf(b2[s][iq], c2), fminf(b1[s][iq], c1));
            b1[s][iq] = fmaxf(b1[s][iq], c1);
          }
      }
      if (any && ((u0 & 15) >> 2) == 0) {
        float2* cd = p.cand + qrow_out * kCand + tg * 16;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          const int u = token(s);
          float2* e = cd + ((u & 3) * 2 + ((u >> 4) & 1)) * 2;
          auto entry = [&](float v) {
            const uint32_t k = __float_as_uint(v) & 0xFFu;
            return make_float2(v * s_scale, __int_as_float(t_begin + (int)(k >> 2) * kStepTokens +
                                                 4 * (int)(k & 3u) + (u & ~15) + (u & 3)));
          };
          e[0] = entry(b1[s][iq]);
          e[1] = entry(b2[s][iq]);
        }
      }
      if (ok && cl == 0 && tb == 0) {
        float* dst = p.part + qrow_out * p.part_stride + p.rv;
        dst[0] = mr;
        dst[1] = lt;
      }
    }
  }
  uint8_t* part = reinterpret_cast<uint8_t*>(p.part + pbase * p.part_stride);
#pragma unroll
  for (int c = 0; c < CT; ++c)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int il = c * 16 + 4 * quad + e;
      if (il < nql) {
        const uint32_t off = (uint32_t)(qmap[il] * p.part_stride + col) * 4u;
#pragma unroll
        for (int t = 0; t < NTW; ++t) {
          const int nt = w * NTW + t;
          if (nt < NT) *reinterpret_cast<float*>(part + 64 * nt + off) = acc_v[c][t][e];
        }
      }
    }
}

// ------------------------------------------------------------------ launchers
template <int D, int QM, int NHB, int NS, int CT, int NTW, int MAXP>
static int launch_poly_t(const PolyParams& p, size_t lds, hipStream_t st) {
  auto k = decode_split_poly_kernel<D, QM, NHB, NS, CT, NTW, MAXP>;
  static std::atomic<uint64_t> attr{0};
  if (const int e = allow_lds(reinterpret_cast<const void*>(k), attr)) return e;
  dim3 grid(p.dyn ? p.cap : p.n_split, p.dyn ? 1 : p.batch, p.n_hg);
  hipLaunchKernelGGL(k, grid, dim3(kThreads), lds, st, p);
  return (int)hipGetLastError();
}

template <int D, int QM, int NHB, int NS, int CT, int NTW>
static int dispatch_maxp(const PolyParams& p, int maxp, size_t lds, hipStream_t st) {
  if (maxp <= 4) return launch_poly_t<D, QM, NHB, NS, CT, NTW, 4>(p, lds, st);
  if constexpr (D == 128 && QM != STARKV_Q_F16) return launch_poly_t<D, QM, NHB, NS, CT, NTW, 8>(p, lds, st);
  return (int)hipErrorInvalidValue;
}

template <int D, int QM, int NHB, int NS, int CT>
static int dispatch_ntw(const PolyParams& p, const PolyShape& s, size_t lds, hipStream_t st) {
  if (s.ntw == 2) return dispatch_maxp<D, QM, NHB, NS, CT, 2>(p, s.maxp, lds, st);
  if constexpr (QM != STARKV_Q_F16)
    if (s.ntw == 3) return dispatch_maxp<D, QM, NHB, NS, CT, 3>(p, s.maxp, lds, st);
  return (int)hipErrorInvalidValue;
}

#define SK_CAT2(a, b) launch_poly_d##a##_q##b
#define SK_NAME(a, b) SK_CAT2(a, b)
int SK_NAME(SK_D, SK_QM)(const PolyParams& p, const PolyShape& s, size_t lds, hipStream_t st) {
  if (s.nhb == 1) {
    if (s.ns == 4 && s.ct == 2) return dispatch_ntw<SK_D, SK_QM, 1, 4, 2>(p, s, lds, st);
    if (s.ns == 2 && s.ct == 1) return dispatch_ntw<SK_D, SK_QM, 1, 2, 1>(p, s, lds, st);
  }
#if SK_D == 128
  if (s.nhb == 2) {
    // (fp16 caches with two fast blocks take groups of at most four heads)
    if constexpr (SK_QM != STARKV_Q_F16)
      if (s.ns == 4 && s.ct == 2) return dispatch_ntw<SK_D, SK_QM, 2, 4, 2>(p, s, lds, st);
    if (s.ns == 2 && s.ct == 1) return dispatch_ntw<SK_D, SK_QM, 2, 2, 1>(p, s, lds, st);
  }
#endif
  return (int)hipErrorInvalidValue;
}
#else

int poly_lds_bytes(const PolyShape& s, int head_dim, int frag_bytes, int v_ng) {
  return poly_lds(head_dim, s.nhb, s.ct).meta + 2 * poly_meta_bytes(v_ng) + frag_bytes;
}

#define SK_DECL(a, b) \
  int launch_poly_d##a##_q##b(const PolyParams& p, const PolyShape& s, size_t lds, hipStream_t st);
SK_DECL(64, 0) SK_DECL(64, 1) SK_DECL(64, 2) SK_DECL(64, 3)
SK_DECL(128, 0) SK_DECL(128, 1) SK_DECL(128, 2) SK_DECL(128, 3)

int launch_decode_split_poly(const PolyParams& p, const PolyShape& s, int head_dim, int qmode,
                             size_t lds, void* stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (head_dim == 128) {
    switch (qmode) {
      case STARKV_Q_F16: return launch_poly_d128_q0(p, s, lds, st);
      case STARKV_Q_INT4: return launch_poly_d128_q1(p, s, lds, st);
      case STARKV_Q_MIX8_4: return launch_poly_d128_q2(p, s, lds, st);
      case STARKV_Q_MIX4_3: return launch_poly_d128_q3(p, s, lds, st);
    }
  } else if (head_dim == 64) {
    switch (qmode) {
      case STARKV_Q_F16: return launch_poly_d64_q0(p, s, lds, st);
      case STARKV_Q_INT4: return launch_poly_d64_q1(p, s, lds, st);
      case STARKV_Q_MIX8_4: return launch_poly_d64_q2(p, s, lds, st);
      case STARKV_Q_MIX4_3: return launch_poly_d64_q3(p, s, lds, st);
    }
  }
  return (int)hipErrorInvalidValue;
}
#endif

}  // namespace starkv

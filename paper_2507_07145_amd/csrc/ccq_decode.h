// Decode of one lane's share of a narrow-format group to correctly rounded bf16, shared by the kernels that multiply
// bf16-rounded weights (the LDS-tiled ones).  Device code only.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace ccq {

typedef __attribute__((ext_vector_type(2))) float dec_f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 dec_bf16x2;

// (a & mask) | orv as v_bitop3_b32 with the truth table 0xEA: 2.45 cycles of a SIMD per wavefront, v_and_or_b32 takes 4.3 (as do
// conversions, permutes, left and funnel shifts and mixed-precision FMAs; fp32 arithmetic, right shifts and plain and / or 2.45).
// Callers keep mask and orv in registers.
__device__ __forceinline__ uint32_t dec_and_or(uint32_t a, uint32_t mask, uint32_t orv) { return __builtin_amdgcn_bitop3_b32(a, mask, orv, 0xEA); }

__device__ __forceinline__ uint32_t dec_pack_bf16(float lo, float hi) {
  dec_f32x2 v = {lo, hi};
  dec_bf16x2 b = __builtin_convertvector(v, dec_bf16x2);  // round to nearest even
  return __builtin_bit_cast(uint32_t, b);
}

constexpr uint32_t kDecMask2 = 0x03F003F0u;  // bits 4..9 of the mantissas of two fp16 numbers
constexpr uint32_t kDecBase2 = 0x54005400u;  // fp16 64.0 twice
constexpr float kDecBase = 64.f;             // the accumulator offset c0 is -(kDecBase + zp) * scale

typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
constexpr float kAlphaScale = 16777216.f;    // 2^24: see decode16_narrow

// Sixteen weights of one lane (four stored bytes of a narrow-format group: k = 16 kq .. 16 kq + 15) to correctly
// rounded bf16, eight packed pairs in k order.
//   Code Cluster (Alg. 3): c = round(q alpha + beta) by one FMA against beta + 2^23 (`bem`), the 15-bit code in the
//   low mantissa bits.  A zero-extended byte is the fp16 subnormal q 2^-24: one permute makes operands of two mixed-precision
//   FMAs of two bytes, alpha is given times 2^24 (`al24`, exact).  Two codes side by side in one register (v_perm), and for each of the four windows of Table 1's
//   shift list [9,6,3,0] one shift and one v_bitop3 put both codes' state into bits 4..9 of the mantissa of fp16 64.0:
//   two fp16 numbers 64 + state, exact.  The linear map d = (w_uint - zp) s of Alg. 3's last line is then one
//   mixed-precision FMA per weight, fma(64 + state, s, c0) with c0 = -(64 + zp) s: 64 + zp has at most 8 significant
//   bits, s at most 15 (a 4-bit field times an fp16 super scale), so c0 and the result are exact in fp32 and the bf16
//   written is the correctly rounded exact weight.  48 vector instructions per 16 weights.
__device__ __forceinline__ void decode16_narrow(uint32_t d, float al24, float bem, float s, float c0, uint32_t mask2, uint32_t base2, uint32_t (&o)[8]) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const f16x2 q = __builtin_bit_cast(f16x2, __builtin_amdgcn_perm(0u, d, h ? 0x0C030C02u : 0x0C010C00u));  // bytes 2h and 2h + 1, times 2^-24
    const uint32_t ca = __builtin_bit_cast(uint32_t, __builtin_fmaf((float)q.x, al24, bem)), cb = __builtin_bit_cast(uint32_t, __builtin_fmaf((float)q.y, al24, bem));
    const uint32_t pr = __builtin_amdgcn_perm(cb, ca, 0x05040100u);  // code 2h in the low half, code 2h + 1 in the high half
    const f16x2 w0 = __builtin_bit_cast(f16x2, dec_and_or(pr >> 5, mask2, base2));  // window at bit 9: weights 8h + 0 and 8h + 4
    const f16x2 w1 = __builtin_bit_cast(f16x2, dec_and_or(pr >> 2, mask2, base2));  // window at bit 6: weights 8h + 1 and 8h + 5
    const f16x2 w2 = __builtin_bit_cast(f16x2, dec_and_or(pr << 1, mask2, base2));  // window at bit 3: weights 8h + 2 and 8h + 6
    const f16x2 w3 = __builtin_bit_cast(f16x2, dec_and_or(pr << 4, mask2, base2));  // window at bit 0: weights 8h + 3 and 8h + 7
    o[4 * h + 0] = dec_pack_bf16(__builtin_fmaf((float)w0.x, s, c0), __builtin_fmaf((float)w1.x, s, c0));
    o[4 * h + 1] = dec_pack_bf16(__builtin_fmaf((float)w2.x, s, c0), __builtin_fmaf((float)w3.x, s, c0));
    o[4 * h + 2] = dec_pack_bf16(__builtin_fmaf((float)w0.y, s, c0), __builtin_fmaf((float)w1.y, s, c0));
    o[4 * h + 3] = dec_pack_bf16(__builtin_fmaf((float)w2.y, s, c0), __builtin_fmaf((float)w3.y, s, c0));
  }
}

constexpr uint32_t kDecMaskW2 = 0x00F000F0u;  // bits 4..7 of the mantissas of two fp16 numbers (a 4-bit state)

// Six weights of one lane (two stored bytes a, b of a wide-format group: codes of (L=4,N=3,S=2), weights 3 code .. + 2)
// to fp32, in k order.  `pp` holds the two bytes as {0, b, 0, a}.  Table 1's shift list [4, 2, 0] with mask 0xF: the
// window at shift 4 already sits in bits 4..7 of its half, the other two are moved there with one shift each, and one
// v_bitop3 per window puts both codes' state into the mantissas of two fp16 64.0 (64 + state, exact).  Then Alg. 2's
// last line, d = (w_uint - zp) s, as one mixed-precision FMA per weight with c0 = -(64 + zp) s (exact in fp32: at
// most 8 significant bits times at most 15).  11 vector instructions per 6 weights.
__device__ __forceinline__ void decode6_wide(uint32_t pp, float s, float c0, uint32_t mask2, uint32_t base2, float (&w)[6]) {
  const f16x2 f0 = __builtin_bit_cast(f16x2, dec_and_or(pp, mask2, base2));
  const f16x2 f1 = __builtin_bit_cast(f16x2, dec_and_or(pp << 2, mask2, base2));
  const f16x2 f2 = __builtin_bit_cast(f16x2, dec_and_or(pp << 4, mask2, base2));
  w[0] = __builtin_fmaf((float)f0.x, s, c0);
  w[1] = __builtin_fmaf((float)f1.x, s, c0);
  w[2] = __builtin_fmaf((float)f2.x, s, c0);
  w[3] = __builtin_fmaf((float)f0.y, s, c0);
  w[4] = __builtin_fmaf((float)f1.y, s, c0);
  w[5] = __builtin_fmaf((float)f2.y, s, c0);
}

// The same with fp16 group scales (11 significant bits), where most windows stay at the bits at which they lie: with the state's
// lowest bit at bit p of the mantissa of fp16 2^(10 - p), the number is 2^(10 - p) + state, and its offset -(2^(10 - p) + zp) s is exact (at
// most 12 bits times 11; a compressed scale has 15).  Two left shifts fewer per pair of narrow codes, both of a pair of wide ones.
struct DecWindows {
  uint32_t mask[3], base[3];
};
template <bool WIDE>
__device__ __forceinline__ DecWindows dec_windows() {   // narrow: windows 9 and 6 | 3 | 0; wide: 4 | 2 | 0
  DecWindows w = WIDE ? DecWindows{{0x00F000F0u, 0x003C003Cu, 0x000F000Fu}, {0x54005400u, 0x5C005C00u, 0x64006400u}}
                      : DecWindows{{0x03F003F0u, 0x01F801F8u, 0x003F003Fu}, {0x54005400u, 0x58005800u, 0x64006400u}};
#pragma unroll
  for (int i = 0; i < 3; ++i) asm volatile("" : "+s"(w.mask[i]), "+v"(w.base[i]));
  return w;
}
constexpr float kNarrowBases[3] = {64.f, 128.f, 1024.f}, kWideBases[3] = {64.f, 256.f, 1024.f};   // what is added to the states

__device__ __forceinline__ void decode16_narrow_fp16(uint32_t d, float al24, float bem, float s, const float (&c0)[3], const DecWindows& k, uint32_t (&o)[8]) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const f16x2 q = __builtin_bit_cast(f16x2, __builtin_amdgcn_perm(0u, d, h ? 0x0C030C02u : 0x0C010C00u));
    const uint32_t ca = __builtin_bit_cast(uint32_t, __builtin_fmaf((float)q.x, al24, bem)), cb = __builtin_bit_cast(uint32_t, __builtin_fmaf((float)q.y, al24, bem));
    const uint32_t pr = __builtin_amdgcn_perm(cb, ca, 0x05040100u);
    const f16x2 w0 = __builtin_bit_cast(f16x2, dec_and_or(pr >> 5, k.mask[0], k.base[0])), w1 = __builtin_bit_cast(f16x2, dec_and_or(pr >> 2, k.mask[0], k.base[0]));
    const f16x2 w2 = __builtin_bit_cast(f16x2, dec_and_or(pr, k.mask[1], k.base[1])), w3 = __builtin_bit_cast(f16x2, dec_and_or(pr, k.mask[2], k.base[2]));
    o[4 * h + 0] = dec_pack_bf16(__builtin_fmaf((float)w0.x, s, c0[0]), __builtin_fmaf((float)w1.x, s, c0[0]));
    o[4 * h + 1] = dec_pack_bf16(__builtin_fmaf((float)w2.x, s, c0[1]), __builtin_fmaf((float)w3.x, s, c0[2]));
    o[4 * h + 2] = dec_pack_bf16(__builtin_fmaf((float)w0.y, s, c0[0]), __builtin_fmaf((float)w1.y, s, c0[0]));
    o[4 * h + 3] = dec_pack_bf16(__builtin_fmaf((float)w2.y, s, c0[1]), __builtin_fmaf((float)w3.y, s, c0[2]));
  }
}
__device__ __forceinline__ void decode6_wide_fp16(uint32_t pp, float s, const float (&c0)[3], const DecWindows& k, float (&w)[6]) {
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const f16x2 f = __builtin_bit_cast(f16x2, dec_and_or(pp, k.mask[i], k.base[i]));
    w[i] = __builtin_fmaf((float)f.x, s, c0[i]);
    w[3 + i] = __builtin_fmaf((float)f.y, s, c0[i]);
  }
}

// What the lanes of the two k halves do differently with a wide-format group: byte selectors (low and high halfword of a dword) of
// two neighbouring codes of entries i and i + 1 as {0, b, 0, a}, of the two single codes as {0, second, 0, first}, the shift of the
// first single weight, and the bits of the move into place.
struct WideLane {
  uint32_t pair[2], one[2], one_shift, funnel;
};
__device__ __forceinline__ WideLane wide_lane(int h) {
  return WideLane{{h ? 0x0C040C01u : 0x0C010C00u, h ? 0x0C060C03u : 0x0C030C02u}, {h ? 0x0C050C00u : 0x0C040C04u, h ? 0x0C070C02u : 0x0C060C06u}, h ? 4u : 2u,
                  h ? 0u : 16u};
}

// Weights 32h .. 32h + 31 of a column of a wide-format group as sixteen bf16 pairs in k order.  `d`: the dwords of six two-byte entries
// (codes 0 .. 10, or 10 .. 21) that hold the group in halfword `odd`.  Ten whole codes are decoded pairwise, the two weights beside
// them (30, 31 or 32, 63) one by one, and one funnel shift per dword moves the row into place, by zero or by one weight.
template <bool FP16>
__device__ __forceinline__ void decode32_wide(const uint32_t (&d)[6], int odd, float s, const float (&c0)[3], const WideLane& wl, const DecWindows& k, uint32_t (&o)[16]) {
  float f[32];  // 0: the first single weight (32, or 31), 1..30: the whole codes, 31: the second one (63, or 30)
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    float w6[6];
    const uint32_t pp = __builtin_amdgcn_perm(d[i + 1], d[i], wl.pair[odd]);
    if constexpr (FP16) decode6_wide_fp16(pp, s, c0, k, w6);
    else decode6_wide(pp, s, c0[0], k.mask[0], k.base[0], w6);
#pragma unroll
    for (int e = 0; e < 6; ++e) f[1 + 6 * i + e] = w6[e];
  }
  const uint32_t pe = __builtin_amdgcn_perm(d[5], d[0], wl.one[odd]);
  f[0] = __builtin_fmaf((float)__builtin_bit_cast(f16x2, dec_and_or(pe << wl.one_shift, k.mask[0], k.base[0])).x, s, c0[0]);
  f[31] = __builtin_fmaf((float)__builtin_bit_cast(f16x2, dec_and_or(pe, k.mask[0], k.base[0])).y, s, c0[0]);
  uint32_t q[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) q[i] = dec_pack_bf16(f[2 * i], f[2 * i + 1]);
#pragma unroll
  for (int i = 0; i < 16; ++i) o[i] = __builtin_amdgcn_alignbit(q[(i + 1) & 15], q[i], wl.funnel);
}

// The hybrid word (Sec. 3.2) cut into chunks of eight weights, the operands of MFMA kk of half h: weight 8c + i of a group sits in words
// c and c + 1 (chunk 7: in words 8 and 9), seven weights to a word at the shifts [13,11,9,6,4,2,0] of Table 1.  With the pair in one
// register, first word on top, the lowest bits of its states in k order are kH16Pos.  Chunk kk (half 0) starts at state kk, chunk
// 4 + kk (half 1) at state kk + 4 (chunk 7 at state 0).  Rotated so that the first state of either lies at bit 29, all states of the two
// chunks lie at the same bits but for one, which half 1 has a bit lower: kH16Odd[kk].
constexpr int kH16Pos[14] = {29, 27, 25, 22, 20, 18, 16, 13, 11, 9, 6, 4, 2, 0};
constexpr int kH16Odd[4] = {6, 5, 4, 3};
constexpr int h16_start(int kk, int h) { return h == 0 ? kk : (kk == 3 ? 0 : kk + 4); }
constexpr int h16_bit(int kk, int h, int i) { return kH16Pos[h16_start(kk, h) + i] + 29 - kH16Pos[h16_start(kk, h)]; }   // of state i after the rotation
constexpr bool h16_aligned() {
  for (int kk = 0; kk < 4; ++kk)
    for (int i = 0; i < 8; ++i)
      if (h16_bit(kk, 0, i) - h16_bit(kk, 1, i) != (i == kH16Odd[kk] ? 1 : 0)) return false;
  return true;
}
static_assert(h16_aligned(), "");
struct H16Lane {
  uint32_t turn[4], odd[4];   // rotation of a pair; rotation that brings the odd state to bit 16
  uint32_t mask, base;        // of a state at bit 16, and fp32 128.0, in registers
};
__device__ __forceinline__ H16Lane h16_lane(int h) {
  H16Lane l;
  l.mask = 0x00070000u;
  l.base = 0x43000000u;
  asm volatile("" : "+s"(l.mask), "+v"(l.base));
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    l.turn[kk] = (uint32_t)((h ? kH16Pos[h16_start(kk, 1)] : kH16Pos[h16_start(kk, 0)]) - 29) & 31u;
    l.odd[kk] = (uint32_t)((h ? h16_bit(kk, 1, kH16Odd[kk]) : h16_bit(kk, 0, kH16Odd[kk])) - 16) & 31u;
  }
  return l;
}
// Weights 32h .. 32h + 31 of a column as sixteen bf16 pairs in k order.  `d`: the dwords that hold the pairs of words
// 0 1, 1 2, 2 3 and 4 5 of the lane's six entries, the group in halfword `odd`.  With fp16 group scales (128 + zp) s is exact and one fused
// multiply-add gives the exactly rounded weight.  A 13-bit field times an 11-bit super scale fills all 24 bits of s (FULL), so there
// the offset is taken off first (exact) and the product (state - zp) s is rounded once to fp32.
template <bool FULL>
__device__ __forceinline__ void decode32_h16(const uint32_t (&d)[6], int odd, float s, float zp, const H16Lane& l, uint32_t (&o)[16]) {
  const float zoff = 128.f + zp, c0 = -zoff * s;
  constexpr int first[4] = {0, 1, 2, 4};
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    uint32_t v = __builtin_amdgcn_perm(d[first[kk]], d[first[kk] + 1], odd ? 0x07060302u : 0x05040100u);
    v = __builtin_amdgcn_alignbit(v, v, l.turn[kk]);
    float f[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int bit = h16_bit(kk, 0, i);   // the state goes to bits 16..18, the lowest integer bits of fp32 128.0
      const uint32_t t = i == kH16Odd[kk] ? (bit > 16 ? v >> l.odd[kk] : __builtin_amdgcn_alignbit(v, v, l.odd[kk])) : (bit >= 16 ? v >> (bit - 16) : v << (16 - bit));
      const float st = __builtin_bit_cast(float, dec_and_or(t, l.mask, l.base));  // 128 + state
      f[i] = FULL ? (st - zoff) * s : __builtin_fmaf(st, s, c0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) o[4 * kk + i] = dec_pack_bf16(f[2 * i], f[2 * i + 1]);
  }
}

}  // namespace ccq

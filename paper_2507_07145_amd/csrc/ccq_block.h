// Fused dequantize-and-multiply for prompts (hundreds to thousands of activation rows), every format, gfx950.
//
// A workgroup of four wavefronts owns a block of 32 MT x 256 outputs (MT = 8: 256 rows, one wavefront per SIMD with 512
// registers; MT = 4: 128 rows, two per SIMD) and a share of K.  K is walked one 64-weight group per step; per step
//   - the activation tile of the next step goes from memory to LDS without passing registers (global_load_lds, 16 bytes a lane),
//     in the order of memory; a row's eight 16-byte chunks are permuted by its number, so that the operand reads of 16
//     neighbouring rows meet all banks,
//   - every wavefront decodes the 64 columns that it multiplies, a step ahead, to bf16 MFMA operands in registers (decode16_narrow,
//     decode32_wide, decode32_h16 of ccq_decode.h: the correctly rounded bf16 of the exact weight): decoded weights never see LDS,
//   - and multiplies them with the activation tile by MFMA 32x32x16 bf16 (fp32 accumulators), weights as the first operand: a
//     lane then holds four neighbouring outputs of one row, which leave in 16-byte stores.
// What bounds it is issue at the clock that the chip's power leaves: MFMA and vector instructions do not overlap (narrow, 256-row blocks: the MFMA pipe
// is busy 71 % of the cycles, vector instructions at four cycles each make 27 %; hybrid word 60 and 38 %), and with all CUs busy the core clock falls to
// 1.7 to 1.8 GHz (2.4 GHz with one block).  What a step spends besides its MFMAs is therefore kept small: 0.5 LDS operand reads per MFMA,
// 3.05 vector instructions (narrow; hybrid word 5.0), no LDS writes by instructions.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "ccq_decode.h"
#include "ccq_internal.h"

namespace ccq {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

struct BlockArgs {
  const uint8_t* codes;
  const uint16_t* scales;
  const float* alpha;
  const float* beta;
  const int32_t* meta;
  const uint16_t* scale_super;  // fp16 [N], compressed scales only
  const uint16_t* x;
  uint16_t* y;
  float* partial;               // fp32 [S][M][Npad], K shares only
  int64_t ldx, ldy;
  int64_t row_tile_bytes, row_tile_scale_halfs;
  int32_t M, N, Npad, row_tiles;
  int32_t quads[2];             // four-group pieces of K per kind: a narrow k-tile is one, a wide one two
  int32_t g_last;               // last real group of K: groups past it pad a k-tile (zero scale) and read this group's activations
  int32_t sq[2], sr[2];         // K share s owns quads [s sq + min(s, sr), + sq + (s < sr)) of each kind that is present, at least one
  float zp[2];
  float off[2][3];              // -(kNarrowBases + zp), -(kWideBases + zp)
  // grouped calls: blockIdx.z is the expert; its rows are output rows [offsets[e], offsets[e + 1]), activation row sorted_rows[p] for
  // output row p; expert e's arrays start e * stride bytes after expert 0's
  const int32_t* sorted_rows;
  const int32_t* expert_offsets;
  int64_t codes_stride, scales_stride, ab_stride;
};

constexpr int kBlockCols = 256;
// Vector instructions that a step's two decodes are known to have, at least: what the order of a step asks for (kind: 0 narrow, 1 wide, 2 hybrid word).
constexpr int decode_vectors(int kind, int sm, int mt) {
  if (kind == 0) return sm == 0 ? 180 : 196;
  if (kind == 1) return sm == 0 && mt != 4 ? 180 : 196;
  return sm == 0 ? 224 : 280;
}
constexpr int kBlockLds0 = 256;   // activation tiles start here: global_load_lds takes LDS address 0 for no address

// One block: rows m0 .. of a's, columns n0 .., share `split`.  FM: formats present (1 narrow, 2 wide, 3 both, 4 the hybrid word; a group map exists
// only for 3).  SM: scale mode.  GATHER: activation row sorted_rows[m] for row m.
template <int FM, int SM, bool GATHER, int MT>
__device__ __forceinline__ void block_tile(const BlockArgs& a, int wave, int m0, int n0, int split) {
  constexpr bool HAS_N = FM == 1 || FM == 3, HAS_W = FM >= 2, META = FM == 3, H16 = FM == 4;
  constexpr int BM = 32 * MT, kTile = BM * kGroup * 2;   // bytes of an activation tile
  constexpr int kWideTile = H16 ? kH16TileBytes : kWideTileBytes;
  extern __shared__ __align__(256) unsigned char smem[];
  // (the lane is asked for anew, not kept in a register for the other bodies of a grouped kernel)
  int none = 0;
  asm volatile("" : "+s"(none));
  const int lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, none));
  const int nl = lane & 15, ti = (lane >> 4) & 1, h = lane >> 5;   // column of a 32-wide tile: row tile ti, row nl; k half h

  // this share's quads of a kind
  auto first_quad = [&](int k) { return split * a.sq[k] + min(split, a.sr[k]); };
  auto num_quads = [&](int k) { return a.sq[k] + (split < a.sr[k] ? 1 : 0); };
  const int qn = HAS_N ? a.quads[kNarrow] : 0, qw = HAS_W ? a.quads[kWide] : 0;

  // Uniform bases and 32-bit lane offsets (at_...).  Column tile c of the wavefront: row tiles 2c, 2c + 1 from rt0 on.
  const int rt0 = min(n0 / 16 + wave * 4, a.row_tiles - 1);
  const uint8_t* code_row = a.codes + (int64_t)rt0 * a.row_tile_bytes;
  const char* scale_row = reinterpret_cast<const char*>(a.scales) + (int64_t)rt0 * a.row_tile_scale_halfs * 2;
  const uint8_t* code_wide = code_row + (int64_t)qn * kNarrowTileBytes;
  const char* scale_wide = scale_row + (int64_t)qn * (SM == 0 ? kNarrowTileScaleHalfs : kNarrowTileScaleHalfs4) * 2;
  float al[2], be[2], ssup[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int rt = min(n0 / 16 + wave * 4 + 2 * c + ti, a.row_tiles - 1);   // ragged last block: decodes the last tile again, never stored
    const int prow = min(rt * 16 + nl, a.N - 1);
    al[c] = be[c] = ssup[c] = 0.f;
    if constexpr (SM == 1) ssup[c] = (float)__builtin_bit_cast(_Float16, a.scale_super[prow]);
    if constexpr (HAS_N) {
      al[c] = a.alpha[prow] * kAlphaScale;
      be[c] = a.beta[prow] + 8388608.f;  // + 2^23: exact, beta is an integer below 2^15
    }
  }

  // Activation rows to copy: one global_load_lds of a wavefront moves eight rows, lane l the chunk of row l / 8 that belongs at LDS
  // position l % 8.  Chunk c of row r lies at position c ^ swizzle(r), swizzle(r) = (r ^ r / 8 & 1) & 7.  The instruction's constant offset
  // counts in memory and in LDS: instruction i of four goes 1024 i bytes further in LDS, and xoff is as much less.
  const char* xbase = reinterpret_cast<const char*>(a.x + (GATHER ? 0 : (int64_t)m0 * a.ldx)) - 3072;
  asm volatile("" : "+s"(xbase));   // (the constant stays part of the base)
  uint32_t xoff[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    const int b = wave * MT + i, row = 8 * b + (lane >> 3), chunk = (lane & 7) ^ (lane >> 3) ^ (b & 1);
    const int m = min(m0 + row, a.M - 1);   // rows past the end read the last row again; their products are never stored
    const int64_t xr = GATHER ? a.sorted_rows[m] : m - m0;
    xoff[i] = (uint32_t)(xr * a.ldx * 2 + chunk * 16 + (3072 - (i & 3) * 1024));
  }
  // operand reads: half h of MFMA kk takes chunk 4h + kk (weights 32h + 8kk .. of the group) of row lane % 32
  uint32_t a_frag = kBlockLds0 + (lane & 31) * (kGroup * 2) + (((h * 4) ^ (lane & 7) ^ ((lane >> 3) & 1)) * 16);   // of kk = 0; the others differ in bits 4 and 5

  // group map: of the quad being multiplied, and of the next one, lane l holding the group of its step l % 4
  int map_now[4] = {0, 0, 0, 0}, map_next = 0;
  auto load_map = [&](int q) { map_next = a.meta[4 * min(q, qn + qw - 1) + (lane & 3)]; };
  auto take_map = [&]() {
#pragma unroll
    for (int j = 0; j < 4; ++j) map_now[j] = __builtin_amdgcn_readlane(map_next, j);
  };
  // activation columns of step j of quad q (j = 4: the first step of the quad after it)
  auto group_of = [&](int q, int j) -> int {
    if constexpr (META) return j < 4 ? map_now[j & 3] : __builtin_amdgcn_readlane(map_next, 0);
    return min(4 * q + j, a.g_last);
  };
  auto copy_a = [&](int buf, int group) {
    const char* base = xbase + (int64_t)group * (kGroup * 2);
    // keeps the zero extensions next to the loads: uniform base + 32-bit lane offset
    if constexpr (MT == 1) asm volatile("" : "+v"(xoff[0]));
    if constexpr (MT == 2) asm volatile("" : "+v"(xoff[0]), "+v"(xoff[MT > 1 ? 1 : 0]));
    if constexpr (MT == 3) asm volatile("" : "+v"(xoff[0]), "+v"(xoff[MT > 1 ? 1 : 0]), "+v"(xoff[MT > 2 ? 2 : 0]));
    if constexpr (MT > 3) asm volatile("" : "+v"(xoff[0]), "+v"(xoff[MT > 1 ? 1 : 0]), "+v"(xoff[MT > 2 ? 2 : 0]), "+v"(xoff[MT > 3 ? 3 : 0]));
    if constexpr (MT > 4) asm volatile("" : "+v"(xoff[4]), "+v"(xoff[MT > 5 ? 5 : 0]), "+v"(xoff[MT > 6 ? 6 : 1]), "+v"(xoff[MT > 7 ? 7 : 2]));
    auto one = [&](auto IC) {
      constexpr int i = decltype(IC)::value;
      if constexpr (i < MT)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(base + xoff[i]),
                                         (__attribute__((address_space(3))) void*)(smem + kBlockLds0 + buf * kTile + (wave * MT + (i & ~3)) * 1024), 16, (i & 3) * 1024, 0);
    };
    one(std::integral_constant<int, 0>{});
    one(std::integral_constant<int, 1>{});
    one(std::integral_constant<int, 2>{});
    one(std::integral_constant<int, 3>{});
    one(std::integral_constant<int, 4>{});
    one(std::integral_constant<int, 5>{});
    one(std::integral_constant<int, 6>{});
    one(std::integral_constant<int, 7>{});
  };

  // Codes of a quad in two halves of two groups.  Narrow: the entries of quarters 2h and 2h + 1.  Wide: the six two-byte entries
  // with codes 0 .. 10 (h = 0) or 10 .. 21 (h = 1).  Hybrid word: words 0 1 2 3 | 3 4 (h = 0) or 4 5 6 7 | 8 9 (h = 1), the pairs of words that
  // hold the eight weights of MFMAs 0, 1, 2 | 3.
  u32x2 cn[2][2][2];
  uint32_t cw[2][2][6], sc[2][2];
  uint32_t at_first[2], at_other[2], at_scale[2];   // of column tile c
  auto set_offsets = [&](auto WIDE) {
    int hw = h, nw = nl, tw = ti;
    asm volatile("" : "+v"(hw), "+v"(nw), "+v"(tw));   // formed for each kind anew
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int rt = min(n0 / 16 + wave * 4 + 2 * c + tw, a.row_tiles - 1) - rt0;
      const uint32_t code = (uint32_t)rt * (uint32_t)a.row_tile_bytes, scale = (uint32_t)rt * (uint32_t)a.row_tile_scale_halfs * 2u;
      if constexpr (!decltype(WIDE)::value) {
        at_first[c] = code + (uint32_t)(nw + 32 * hw) * 16u;
        at_scale[c] = scale + (uint32_t)nw * (SM == 0 ? 8u : 2u);
      } else {
        // Entry e of a k-tile lies 1024 t + 256 kq + 16 nl bytes in, e = 3 kq + t (words: e = 4 t + kq).  The lane's entries are h = 0 entries
        // at constant distances from two of them, the same ones in both halves.
        at_first[c] = code + nw * 16 + (H16 ? hw * 1024 : hw * 2304);
        at_other[c] = code + nw * 16 + (H16 ? 768 + hw * 1280 : 1024 - hw * 512);
        at_scale[c] = SM == 0 ? scale + nw * 16 : code + nw * 16;
      }
    }
  };
  // (the empty asm keeps the zero extensions next to the loads)
  auto load_narrow = [&](int q, int half) {
    const uint8_t* t = code_row + (int64_t)q * kNarrowTileBytes + half * 8;
    const char* sb = scale_row + (int64_t)q * (SM == 0 ? kNarrowTileScaleHalfs : kNarrowTileScaleHalfs4) * 2 + (SM == 0 ? half * 4 : 0);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      asm volatile("" : "+v"(at_first[c]), "+v"(at_scale[c]));
#pragma unroll
      for (int e = 0; e < 2; ++e) cn[half][c][e] = *reinterpret_cast<const u32x2*>(t + at_first[c] + e * 256);
      if constexpr (SM == 0) sc[half][c] = *reinterpret_cast<const uint32_t*>(sb + at_scale[c]);
      else sc[half][c] = (uint32_t)*reinterpret_cast<const uint16_t*>(sb + at_scale[c]);  // the quad's four 4-bit fields
    }
  };
  auto load_wide = [&](int q, int half) {   // q: counted from the first wide quad
    const uint8_t* t = code_wide + (int64_t)(q >> 1) * kWideTile + (q & 1) * 8 + half * 4;
    const char* sb = scale_wide + (int64_t)(q >> 1) * (kWideTileScaleHalfs * 2) + (q & 1) * 8 + half * 4;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      asm volatile("" : "+v"(at_first[c]), "+v"(at_other[c]), "+v"(at_scale[c]));
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        // wide: entries 0, 3 | 1, 2, 4, 5; words 0, 1, 2, 3 | 4, 5
        const int at = H16 ? (i < 4 ? i * 256 : (i - 4) * 256) : (i % 3 == 0 ? i / 3 * 256 : (i % 3 - 1) * 1024 + i / 3 * 256);
        cw[half][c][i] = *reinterpret_cast<const uint32_t*>(t + ((H16 ? i < 4 : i % 3 == 0) ? at_first[c] : at_other[c]) + at);
      }
      if constexpr (SM == 0) sc[half][c] = *reinterpret_cast<const uint32_t*>(sb + at_scale[c]);
      else sc[half][c] = *reinterpret_cast<const uint32_t*>(t + at_scale[c] + (H16 ? 2048 + 256 : 1024 + 768));   // the entry with the fields: word 9, or codes 20 and 21
    }
  };
  // half of quad q of the layout, one of a kind (past the kind's end: of its last quad)
  auto load_codes = [&](auto WIDE, int q, int half) {
    if constexpr (decltype(WIDE)::value) load_wide(min(q, qn + qw - 1) - qn, half);
    else load_narrow(min(q, qn - 1), half);
  };

  DecWindows win;
  WideLane wl;
  H16Lane hl;
  // 32 weights of a column (group j of the quad) as the lane's operands of four MFMAs
  auto decode = [&](auto WIDE, u32x4 (&b)[4], int c, int j) {
    uint32_t o[16];
    auto fp16_scale = [&]() -> float {
      const uint32_t sw = sc[j >> 1][c];
      return (float)__builtin_bit_cast(_Float16, (uint16_t)((j & 1) ? (sw >> 16) : (sw & 0xFFFFu)));
    };
    if constexpr (!decltype(WIDE)::value) {
      float s;
      if constexpr (SM == 0) s = fp16_scale();
      else s = (float)((sc[j >> 1][c] >> (4 * j)) & 0xFu) * ssup[c];  // (s_q >> s_shift) & s_mask times s_super: exact
      const float c0[3] = {a.off[kNarrow][0] * s, a.off[kNarrow][1] * s, a.off[kNarrow][2] * s};   // exact (the first one also for 15-bit scales)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        uint32_t w[8];
        if constexpr (SM == 0) decode16_narrow_fp16(cn[j >> 1][c][e][j & 1], al[c], be[c], s, c0, win, w);
        else decode16_narrow(cn[j >> 1][c][e][j & 1], al[c], be[c], s, c0[0], win.mask[0], win.base[0], w);
#pragma unroll
        for (int i = 0; i < 8; ++i) o[8 * e + i] = w[i];
      }
    } else {
      uint32_t d[6];
#pragma unroll
      for (int i = 0; i < 6; ++i) d[i] = cw[j >> 1][c][i];
      float s;
      if constexpr (SM == 0) {
        s = fp16_scale();
      } else {
        // Alg. 2: the low nibble of the group's last code byte (byte 21), or the low 13 bits of its last word (the scale
        // mask 0x1FFF of Table 1)
        const uint32_t last = (j & 1) ? sc[j >> 1][c] >> 16 : sc[j >> 1][c] & 0xFFFFu;
        s = (float)(H16 ? last & 0x1FFFu : (last >> 8) & 0xFu) * ssup[c];  // exact: at most 13-bit integer times 11-bit significand
      }
      if constexpr (H16) decode32_h16<SM == 1>(d, j & 1, s, a.zp[kWide], hl, o);
      else decode32_wide<SM == 0 && MT != 4>(d,   // (128-row blocks have no registers to spare)
                               j & 1, s, {a.off[kWide][0] * s, a.off[kWide][1] * s, a.off[kWide][2] * s}, wl, win, o);
    }
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) b[kk] = u32x4{o[4 * kk], o[4 * kk + 1], o[4 * kk + 2], o[4 * kk + 3]};
  };

  f32x16 acc[MT][2];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][c][r] = 0.f;
  // operands: activations of one MFMA and the next, weights of one step and the next
  u32x4 af[2][MT], bw[2][2][4];
  auto load_frags = [&](int par, int buf, int kk) {
#pragma unroll
    for (int i = 0; i < MT; ++i) af[par][i] = *reinterpret_cast<const u32x4*>(smem + (a_frag ^ (kk * 16)) + (buf * kTile + i * 32 * kGroup * 2));
  };
  auto multiply = [&](int par, const u32x4 (&b)[2][4], int kk, int i0, int i1) {
#pragma unroll
    for (int i = i0; i < i1; ++i)
#pragma unroll
      for (int c = 0; c < 2; ++c)
        acc[i][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, b[c][kk]), __builtin_bit_cast(bf16x8, af[par][i]), acc[i][c], 0, 0, 0);
  };
  // Every load is waited for before the barrier, the copy to LDS among them, which no register tells the compiler about.
  auto wait_loads = [&]() { __builtin_amdgcn_s_waitcnt(0x0F70); };   // vmcnt(0)
  auto lds_barrier = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  };

  // One step: step J of quad q is multiplied, the next step's weights are decoded and its activations copied.  Each half of the next
  // quad's codes is asked for once the last decode from its registers has run, two steps before the next one.
  auto step = [&](int q, auto JC, auto WIDE) {
    constexpr int J = decltype(JC)::value, P = J & 1, JN = (J + 1) & 3;
    constexpr int held = 6 * MT + 2 * (MT / 2);   // MFMAs before the barrier
    // vector instructions that two decodes have at least: with more asked for, the order below comes out wrong
    constexpr bool wide = decltype(WIDE)::value;
    constexpr int vector = decode_vectors(wide ? (H16 ? 2 : 1) : 0, SM, MT);
    constexpr int asked = J & 1 ? 0 : (decltype(WIDE)::value ? 14 : 6) + (META && J == 0 ? 1 : 0);   // loads
    if constexpr (MT == 4) asm volatile("" : "+v"(a_frag));   // (the other three are formed in each step, not kept)
    load_frags(1, P, 1);
    copy_a(P ^ 1, group_of(q, J + 1));
    multiply(0, bw[P], 0, 0, MT);
    load_frags(0, P, 2);
    multiply(1, bw[P], 1, 0, MT);
    decode(WIDE, bw[P ^ 1][0], 0, JN);
    load_frags(1, P, 3);
    multiply(0, bw[P], 2, 0, MT);
    decode(WIDE, bw[P ^ 1][1], 1, JN);
    multiply(1, bw[P], 3, 0, MT / 2);
    // issue order: one MFMA, a few vector instructions, and the operand reads of the next slice beside the first half of a slice;
    // in the first slice, behind its reads, the copies
#pragma unroll
    for (int i = 0; i < held; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if ((MT > 4 ? i % (2 * MT) < MT : i % 2 == 1) && i < 6 * MT) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      if (i < 2 * MT && i >= 2 * MT - (MT + 1) / 2) __builtin_amdgcn_sched_group_barrier(0x010, 2, 0);
      if ((i + 1) * vector / held - i * vector / held > vector / held) __builtin_amdgcn_sched_group_barrier(0x002, vector / held + 1, 0);
      else __builtin_amdgcn_sched_group_barrier(0x002, vector / held, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    wait_loads();
    lds_barrier();
    __builtin_amdgcn_sched_barrier(0);
    // the first reads of the next step, and the loads, under the MFMAs held back for them
    multiply(1, bw[P], 3, MT / 2, MT);
    load_frags(0, P ^ 1, 0);
    if constexpr (J == 0) load_codes(WIDE, q + 1, 0);
    if constexpr (J == 2) load_codes(WIDE, q + 1, 1);
    if constexpr (META && J == 0) load_map(q + 1);
    if constexpr (META && J == 3) take_map();
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      if (i * 2 < asked) __builtin_amdgcn_sched_group_barrier(0x010, 2, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // quads [from, to) of one kind, from scratch
  auto run = [&](auto WIDE, int from, int to) {
    set_offsets(WIDE);
    if constexpr (!H16) win = dec_windows<decltype(WIDE)::value>();
    if constexpr (decltype(WIDE)::value) {   // what only this kind needs is formed here
      int hw = h;
      asm volatile("" : "+v"(hw));
      if constexpr (H16) hl = h16_lane(hw);
      else wl = wide_lane(hw);
    }
    load_codes(WIDE, from, 0);
    load_codes(WIDE, from, 1);
    if constexpr (META) {
      load_map(from);
      take_map();
    }
    copy_a(0, group_of(from, 0));
    decode(WIDE, bw[0][0], 0, 0);
    decode(WIDE, bw[0][1], 1, 0);
    wait_loads();
    lds_barrier();
    load_frags(0, 0, 0);
    int q = from;
    do {   // a share has quads of every kind: with a loop that may not run, the accumulators are copied around it
      step(q, std::integral_constant<int, 0>{}, WIDE);
      step(q, std::integral_constant<int, 1>{}, WIDE);
      step(q, std::integral_constant<int, 2>{}, WIDE);
      step(q, std::integral_constant<int, 3>{}, WIDE);
    } while (++q < to);
  };
  // (between two runs there is no barrier: the second one's first copy goes to buffer 0, whose last reader, the step before the
  // last, is behind the last step's barrier; so is the copy of a step that no one multiplies)
  if constexpr (HAS_N) run(std::false_type{}, first_quad(kNarrow), first_quad(kNarrow) + num_quads(kNarrow));
  if constexpr (HAS_W) run(std::true_type{}, qn + first_quad(kWide), qn + first_quad(kWide) + num_quads(kWide));

  int lane_now = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));   // asked for anew: nothing of it is held through the loop
  asm volatile("" : "+v"(lane_now));
  lds_barrier();   // the tiles have been read

  // D[n][m]: lane l holds column m = l % 32 and rows n = 8 g + 4 (l / 32) + e: four neighbouring outputs of one activation row per g.
  // Through the wavefront's own piece of LDS (32 rows of 128 bytes, 144 apart) they leave in whole lines: eight lanes to a row.
  unsigned char* own = smem + wave * (32 * 144);
  const int col = lane_now & 31, half = lane_now >> 5, row8 = lane_now >> 3, part = lane_now & 7;
  unsigned char* put = own + col * 144 + half * (!GATHER && a.partial ? 16 : 8);
  const u32x4* get = reinterpret_cast<const u32x4*>(own + row8 * 144 + part * 16);
  // what a lane reads others have written, and the other way round with the next piece: no instruction, LDS serves a wavefront in order
  auto exchanged = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
  };
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    if constexpr (MT > 4) asm volatile("" : "+a"(acc[i][0]), "+a"(acc[i][1]));   // read from the accumulator registers row tile by row tile
    if (!GATHER && a.partial) {
#pragma unroll
      for (int c = 0; c < 2; ++c) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x4 v = {acc[i][c][4 * g], acc[i][c][4 * g + 1], acc[i][c][4 * g + 2], acc[i][c][4 * g + 3]};
          *reinterpret_cast<f32x4*>(put + 32 * g) = v;
        }
        exchanged();
        const int n = n0 + wave * 64 + c * 32 + part * 4;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int m = m0 + i * 32 + 8 * k + row8;
          const u32x4 v = get[k * (8 * 144 / 16)];
          if (m < a.M && n < a.Npad) __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(&a.partial[((int64_t)split * a.M + m) * a.Npad + n]));
        }
        exchanged();
      }
    } else {
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *reinterpret_cast<u32x2*>(put + c * 64 + 16 * g) =
              u32x2{dec_pack_bf16(acc[i][c][4 * g], acc[i][c][4 * g + 1]), dec_pack_bf16(acc[i][c][4 * g + 2], acc[i][c][4 * g + 3])};
      exchanged();
      const int n = n0 + wave * 64 + part * 8;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int m = m0 + i * 32 + 8 * k + row8;
        const u32x4 v = get[k * (8 * 144 / 16)];
        uint16_t* dst = a.y + (int64_t)m * a.ldy + n;
        if (m < a.M) {
          if (n + 8 <= a.N) {
            *reinterpret_cast<u32x4*>(dst) = v;
          } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
              if (n + e < a.N) dst[e] = (uint16_t)(v[e / 2] >> (16 * (e & 1)));
          }
        }
      }
      exchanged();
    }
  }
}

template <int FM, int SM, int MT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MT > 4 ? 1 : 2, MT > 4 ? 1 : 2))) ccq_block_kernel(const BlockArgs a) {
  block_tile<FM, SM, false, MT>(a, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), blockIdx.x * (32 * MT), blockIdx.y * kBlockCols, blockIdx.z);
}

// Grouped calls: blocks of up to 128 rows of an expert, as tall as its rows ask for: a body for each height, so that rows past an expert's end are
// padded to 32, not to 128.  (64 experts of 2048 x 7168, 4096 rows, the fullest with 87: 64-row kernel 188, this 164 us; wide 302 / 216, mix
// 292 / 197, hybrid word 356 / 215.)  Two blocks to a CU, as the dense kernel's 128-row blocks and bound as they are; the MFMAs of the padding are a
// fifth of that time.
template <int FM, int SM>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) ccq_block_grouped_kernel(const BlockArgs a) {
  const int e = blockIdx.z, first = __builtin_amdgcn_readfirstlane(a.expert_offsets[e]), m0 = blockIdx.x * 128, n0 = blockIdx.y * kBlockCols;
  BlockArgs p = a;
  p.M = __builtin_amdgcn_readfirstlane(a.expert_offsets[e + 1]) - first;
  if (m0 >= p.M) return;  // uniform: before any barrier
  p.codes += e * a.codes_stride;
  p.scales = reinterpret_cast<const uint16_t*>(reinterpret_cast<const uint8_t*>(a.scales) + e * a.scales_stride);
  p.alpha = reinterpret_cast<const float*>(reinterpret_cast<const uint8_t*>(a.alpha) + e * a.ab_stride);
  p.beta = reinterpret_cast<const float*>(reinterpret_cast<const uint8_t*>(a.beta) + e * a.ab_stride);
  p.scale_super = reinterpret_cast<const uint16_t*>(reinterpret_cast<const uint8_t*>(a.scale_super) + e * a.ab_stride / 2);   // fp16 against fp32
  p.sorted_rows += first;
  p.y += (int64_t)first * a.ldy;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int live = (min(p.M - m0, 128) + 31) / 32;
  if (live == 1) block_tile<FM, SM, true, 1>(p, wave, m0, n0, 0);
  else if (live == 2) block_tile<FM, SM, true, 2>(p, wave, m0, n0, 0);
  else if (live == 3) block_tile<FM, SM, true, 3>(p, wave, m0, n0, 0);
  else block_tile<FM, SM, true, 4>(p, wave, m0, n0, 0);
}

typedef void (*BlockKernel)(const BlockArgs);
// The kernel of a format with blocks of 32 mt rows; each is built in a source file of its own.
BlockKernel block_kernel_narrow(int scale_mode, int mt);
BlockKernel block_kernel_wide(int scale_mode, int mt);
BlockKernel block_kernel_mix(int scale_mode, int mt);
BlockKernel block_kernel_h16(int scale_mode, int mt);
BlockKernel block_grouped_narrow(int scale_mode);
BlockKernel block_grouped_wide(int scale_mode);
BlockKernel block_grouped_mix(int scale_mode);
BlockKernel block_grouped_h16(int scale_mode);

template <int FM, int SM>
BlockKernel block_rows(int mt) {
  switch (mt) {
    case 4: return ccq_block_kernel<FM, SM, 4>;
    case 5: return ccq_block_kernel<FM, SM, 5>;
    case 6: return ccq_block_kernel<FM, SM, 6>;
    case 7: return ccq_block_kernel<FM, SM, 7>;
    default: return ccq_block_kernel<FM, SM, 8>;
  }
}

}  // namespace ccq

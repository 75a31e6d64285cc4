// Products with few activation rows per matrix (about 2 to 32), every weight format and both scale modes, gfx950: the experts
// of a grouped call, and dense calls small enough that a pass over partial tiles would cost more than it spreads.
//
// Bound: issue.  Narrow, 64 experts of 7168 x 2048 with 8 rows each, per SIMD: 29,600 vector instructions (118,000 cycles by
// SQ_ACTIVE_INST_VALU) and 1,800 MFMAs (29,000) of 179,000 cycles; 31 % of the wavefronts' cycles are waits, no LDS bank conflict, 289 MB
// read for 268.  A workgroup is WN wavefronts side by side, each with RT row tiles
// of 16 output rows, times wk shares of K that meet in LDS at the end: one launch, no workspace.  The WN wavefronts of a
// share walk K in stages of four 64-weight groups:
//   - the activations of the stage after next are requested (lanes along a row: one request covers whole cache lines; read
//     straight into operand order, sixteen rows to an instruction, every lane is a cache access of its own, 64 to an
//     instruction, and the vector cache, not the decode, sets the pace: 110 us where this kernel takes 69);
//   - those of the next stage go to the other LDS buffer as MFMA 16x16x32 A fragments in k-slot order, with the start values
//     -(128 + zp) sum x of every (group, row); slots are exclusive-ored with the lane's chunk so that neither the writes (eight
//     lanes hold one row) nor the reads (eight lanes hold one chunk) meet in a bank (without: 52 of 83 thousand LDS cycles lost);
//   - the current ones are multiplied with weights decoded in registers to the bf16 integers 128 + state; the linear map
//     (w_uint - zp) * s of Alg. 2 / Alg. 3 follows the group's contraction, so weights are exact.
// One LDS-only barrier per stage.  The k-tiles a wavefront holds sit in slots that are refilled in place, two stages ahead
// on the narrow format; moving them from slot to slot instead makes every move wait for its load.  The sums of a row tile
// are added while the next one is decoded, so that no wavefront waits for its own matrix instruction.
// Grouped, narrow, 64 experts of 7168 x 2048 with 8 rows each: 72 us against 95 us on the per-row-tile kernel (staging of
// whole k-tiles between two barriers); wide 200 -> 87 us, mix 168 -> 100 us, hybrid word 220 -> 96 us; 243 experts of 7104 x 528 with
// up to 28 rows 565 -> 118 us.  Many rows without the host copy of the offsets, in passes of 32: 8 experts of 4096 x 4096 with 512
// rows each 656 -> 286 us (147 us with the host copy, on the 64-row kernel).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <cstring>
#include <cstdint>
#include <type_traits>

#include "ccq_internal.h"

namespace ccq {
namespace few {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;

struct Args {
  const uint8_t* codes;
  const uint16_t* scales;
  const float* alpha;
  const float* beta;
  const int32_t* meta;
  const uint16_t* scale_super;
  const uint16_t* x;
  uint16_t* y;
  const int32_t* sorted_rows;      // row of x of every output row, or NULL: the same row
  const int32_t* expert_offsets;   // matrix e's output rows are [offsets[e], offsets[e + 1]); NULL: one matrix, M rows
  int64_t codes_stride, scales_stride, ab_stride;
  int64_t ldx, ldy;
  int64_t row_tile_bytes, row_tile_scale_halfs;
  int32_t M, row_tiles;
  int32_t groups_narrow;           // entries of the group map that precede the wide groups
  int32_t g_last, n_last;          // last real group of K, last real output row (groups and rows past them are padding)
  int32_t tiles[2];                // k-tiles per kind
  int32_t wk;                      // shares of K in a workgroup
  float cneg[2];                   // -(128 + zp) per kind
  int32_t n_active;                // > 0: gridDim.y matrices are listed in active_ids
  uint16_t active_ids[kMaxActiveList];
};

__device__ __forceinline__ uint32_t and_or(uint32_t a, uint32_t mask, uint32_t orv) { return __builtin_amdgcn_bitop3_b32(a, mask, orv, 0xEA); }
__device__ __forceinline__ uint32_t dword_of(const u32x4& v, int j) { return j == 0 ? v.x : (j == 1 ? v.y : (j == 2 ? v.z : v.w)); }
__device__ __forceinline__ f32x4 mfma(const u32x4 a, const u32x4 b, const f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
__device__ __forceinline__ uint16_t to_bf16(float f) {
  const f32x2 v = {f, 0.f};
  return (uint16_t)(__builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2)) & 0xFFFFu);
}
// 16 bytes at a uniform base plus a 32-bit lane offset (4-byte aligned: what the wide kinds' slots want)
__device__ __forceinline__ u32x4 load16(const void* base, uint32_t off) {
  struct __attribute__((packed, aligned(4))) Chunk { uint32_t x, y, z, w; };
  asm volatile("" : "+v"(off));
  const Chunk c = *reinterpret_cast<const Chunk*>(reinterpret_cast<const char*>(base) + off);
  return u32x4{c.x, c.y, c.z, c.w};
}

// The same for what is read once: codes and scales.
__device__ __forceinline__ u32x4 load16_nt(const void* base, uint32_t off) {
  asm volatile("" : "+v"(off));
  return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(base) + off));
}

enum { kKN = 0, kKW = 1, kKH = 2 };   // narrow, wide, hybrid word

__device__ __forceinline__ float frag_sum(const u32x4 o, float s) {
  const bf16x2 ones = __builtin_bit_cast(bf16x2, 0x3F803F80u);
  const uint32_t o0 = o.x, o1 = o.y, o2 = o.z, o3 = o.w;
  s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, o0), ones, s, false);
  s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, o1), ones, s, false);
  s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, o2), ones, s, false);
  s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, o3), ones, s, false);
  return s;
}
// Weights as bf16 integers 128 + state -> bf16((128 + state + cneg) s).
__device__ __forceinline__ u32x4 signed_weights(const u32x4 w, float cneg, float s) {
  auto pair = [&](uint32_t d) {
    const f32x2 v = {(__builtin_bit_cast(float, d << 16) + cneg) * s, (__builtin_bit_cast(float, d & 0xFFFF0000u) + cneg) * s};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
  };
  const uint32_t w0 = w.x, w1 = w.y, w2 = w.z, w3 = w.w;
  return u32x4{pair(w0), pair(w1), pair(w2), pair(w3)};
}
template <int CTRL>
__device__ __forceinline__ float dpp_add(float s) {
  return s + __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, s), CTRL, 0xF, 0xF, true));
}

// Wavefronts per SIMD that the registers are cut for, and whether a workgroup may have sixteen of them.
constexpr int waves_per_simd(int fm, int mt, int rt, int wn) {
  if (fm == 1) return mt == 1 ? 4 : 3;
  if (rt == 2 || mt == 2) return 2;
  return fm == 3 || wn == 2 ? 3 : 4;
}
constexpr uint32_t buffer_bytes(int fm, int mt) { return (fm == 1 ? 8192u + 256u : 12288u + 256u) * mt; }
constexpr int max_waves(int fm, int mt, int rt, int wn) { return rt == 1 && mt == 1 && fm != 3 && wn == 4 ? 16 : 8; }

// A wavefront's part of a k-tile: 16-byte code segments and scales of its RT row tiles.
template <int RT, int NC>
struct HeldTile { u32x4 c[RT][NC]; u32x4 s[RT]; };

template <int FM, int SM, int MT, int RT, int WN>
__global__ void __launch_bounds__(64 * max_waves(FM, MT, RT, WN)) __attribute__((amdgpu_waves_per_eu(waves_per_simd(FM, MT, RT, WN)))) ccq_few_kernel(const Args a) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int not_finite;   // of a dense call's only pass
  constexpr uint32_t kThreads = 64u * WN;
  constexpr uint32_t kFrags = (FM == 1 ? 8192u : 12288u) * MT, kBuf = buffer_bytes(FM, MT);   // one stage: four groups' fragments, then their start values
  const uint32_t lane = threadIdx.x & 63u, tid = threadIdx.x % kThreads;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t wk = wave / WN, wn = wave % WN;
  const uint32_t n = lane & 15u, kq = lane >> 4;
  unsigned char* const stage_mem = smem + wk * (2u * kBuf);
  uint32_t e = 0;
  int32_t row0 = 0, rows = a.M;
  if (a.expert_offsets) {
    e = blockIdx.y;
    if (a.n_active > 0) {
      typedef const __attribute__((address_space(4))) uint16_t* KernargU16;
      typedef const __attribute__((address_space(4))) char* KernargBytes;
      KernargBytes args = (KernargBytes)__builtin_amdgcn_kernarg_segment_ptr();
      e = ((KernargU16)(args + offsetof(Args, active_ids)))[blockIdx.y];
    }
    row0 = a.expert_offsets[e];
    rows = a.expert_offsets[e + 1] - row0;
    if (rows <= 0) return;
  }
  const uint32_t rt0 = (blockIdx.x * (uint32_t)WN + wn) * RT;
  const uint8_t* code_row[RT];
  const uint16_t* scale_row[RT];
  float al_raw[RT], be_raw[RT];
  uint32_t ssup[RT];
#pragma unroll
  for (int r = 0; r < RT; ++r) {
    const uint32_t rt = min(rt0 + r, (uint32_t)a.row_tiles - 1u);
    code_row[r] = a.codes + (size_t)e * (size_t)a.codes_stride + (size_t)rt * (size_t)a.row_tile_bytes;
    scale_row[r] = reinterpret_cast<const uint16_t*>(reinterpret_cast<const uint8_t*>(a.scales) + (size_t)e * (size_t)a.scales_stride) + (size_t)rt * (size_t)a.row_tile_scale_halfs;
    const uint32_t prow = min(rt * 16u + n, (uint32_t)a.n_last);
    if constexpr (FM == 1 || FM == 3) {
      al_raw[r] = reinterpret_cast<const float*>(reinterpret_cast<const uint8_t*>(a.alpha) + (size_t)e * (size_t)a.ab_stride)[prow];
      be_raw[r] = reinterpret_cast<const float*>(reinterpret_cast<const uint8_t*>(a.beta) + (size_t)e * (size_t)a.ab_stride)[prow];
    }
    ssup[r] = 0;
    if constexpr (SM == 1) ssup[r] = reinterpret_cast<const uint16_t*>(reinterpret_cast<const uint8_t*>(a.scale_super) + (size_t)e * (size_t)(a.ab_stride / 2))[prow];
  }
  uint32_t c4300 = 0x43004300u, mask_n = 0x003F003Fu, mask_w = FM == 4 ? 0x00070007u : 0x000F000Fu;
  float magic = 8388608.f;
  asm volatile("" : "+v"(c4300), "+s"(mask_n), "+s"(mask_w), "+v"(magic));
  if (threadIdx.x == 0) not_finite = 0;   // (barriers before the first sum)
  auto lds_barrier = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  };

  // SIGNED: weights are multiplied as bf16((128 + state - (128 + zp)) s), without start values (see below)
  auto pass = [&](auto MC, auto SC, int32_t m0) -> bool {
    constexpr int LM = decltype(MC)::value;   // 16-row activation tiles of this pass
    constexpr bool SIGNED = decltype(SC)::value;
    f32x4 acc[RT][LM];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int m = 0; m < LM; ++m) acc[r][m] = f32x4{0.f, 0.f, 0.f, 0.f};

    auto kind = [&](auto KC) {
      constexpr int K = decltype(KC)::value;
      constexpr bool NARROW = K == kKN, H16 = K == kKH;
      constexpr int GPT = NARROW ? kNarrowGroupsPerTile : kWideGroupsPerTile;
      constexpr int SPT = GPT / 4;                          // stages (four groups) per k-tile
      constexpr int T = NARROW ? 2 : 3;                     // MFMA k-steps per group
      constexpr int NC = NARROW ? 1 : 3;                    // 16-byte code segments per lane and k-tile
      constexpr int TB = NARROW ? kNarrowTileBytes : (H16 ? kH16TileBytes : kWideTileBytes);
      // staging units: narrow (group, row, 16-byte chunk), wide kinds (group, row, quarter) of three chunks each
      constexpr int NU = (NARROW ? 512 : 256) * LM, NCH = NARROW ? 1 : 3, NUT = (NU + (int)kThreads - 1) / (int)kThreads;
      const int kt = NARROW ? kNarrow : kWide;
      const int total = a.tiles[kt], q = total / a.wk, rem = total - q * a.wk;
      const int tA = (int)wk * q + min((int)wk, rem), tB = tA + q + ((int)wk < rem ? 1 : 0);
      const int most = q + (rem > 0 ? 1 : 0);
      const int last = max((tB - tA) * GPT - 1, 0);
      const int gbase = min(tA, total - 1) * GPT + (FM == 3 && !NARROW ? a.groups_narrow : 0);
      const size_t code_off = NARROW || FM != 3 ? 0 : (size_t)a.tiles[kNarrow] * kNarrowTileBytes;
      const size_t scale_off = NARROW || FM != 3 ? 0 : (size_t)a.tiles[kNarrow] * kNarrowTileScaleHalfs;

      using Tile = HeldTile<RT, NC>;
      auto load_tile = [&](Tile& v, int t) {
        t = max(min(t, tB - 1), 0);
#pragma unroll
        for (int r = 0; r < RT; ++r) {
          const uint8_t* cb = code_row[r] + code_off + (size_t)t * TB;
          if constexpr (NARROW) {
            const uint16_t* sb = scale_row[r] + (size_t)t * (SM == 0 ? kNarrowTileScaleHalfs : kNarrowTileScaleHalfs4);
            uint32_t off = n * (SM == 0 ? 8u : 2u);
            asm volatile("" : "+v"(off));
            if constexpr (SM == 0) {
              const u32x2 d = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(reinterpret_cast<const char*>(sb) + off));
              v.s[r] = u32x4{d.x, d.y, 0u, 0u};
            } else {
              v.s[r] = u32x4{(uint32_t)__builtin_nontemporal_load(reinterpret_cast<const uint16_t*>(reinterpret_cast<const char*>(sb) + off)), 0u, 0u, 0u};
            }
            v.c[r][0] = load16_nt(cb, lane * 16u);
          } else {
            if constexpr (SM == 0) v.s[r] = load16_nt(scale_row[r] + scale_off + (size_t)t * kWideTileScaleHalfs, n * 16u);
            else v.s[r] = u32x4{0u, 0u, 0u, 0u};
            constexpr uint32_t kLast = H16 ? 31u : 47u;
            v.c[r][0] = load16_nt(cb, lane * 16u);
            v.c[r][1] = load16_nt(cb + 1024, lane * 16u);
            v.c[r][2] = load16_nt(cb + 2048, min(lane, kLast) * 16u);
          }
        }
      };
      // this thread's staging units: unit u = tid + i * kThreads
      uint32_t xoff[NUT][NCH];
      uint32_t lds_off[NUT];
      int ulg[NUT];
#pragma unroll
      for (int i = 0; i < NUT; ++i) {
        const uint32_t u = min(tid + (uint32_t)i * kThreads, (uint32_t)NU - 1u);
        const uint32_t c = NARROW ? u & 7u : u & 3u, m = NARROW ? (u >> 3) % (16u * LM) : (u >> 2) % (16u * LM), lg = NARROW ? (u >> 3) / (16u * LM) : (u >> 2) / (16u * LM);
        ulg[i] = (int)lg;
        int32_t row = row0 + min(m0 + (int32_t)m, rows - 1);
        if (a.sorted_rows) row = a.sorted_rows[row];
#pragma unroll
        for (int t = 0; t < NCH; ++t)
          xoff[i][t] = (uint32_t)((int64_t)row * a.ldx * 2) + 2u * (NARROW ? 8u * c : (H16 ? min((7u * (4u * t + c)) & ~1u, 56u) : min(18u * c + 6u * t, 56u)));
        // fragment (group, k-step, quarter) of 16-row tile m / 16 at ((((lg * LM + tile) * T + k-step) * 4 + quarter) * 16 + m % 16) * 16
        lds_off[i] = ((((lg * LM + (m >> 4)) * T + (NARROW ? (c & 1u) : 0u)) * 4u + (NARROW ? c >> 1 : c)) * 16u + ((m & 15u) ^ (NARROW ? c : 2u * c))) * 16u;
      }
      auto group_of = [&](int s, int lg) -> int {
        if constexpr (FM == 3) return a.meta[gbase + min(s * 4 + lg, last)];
        return min(gbase + lg + s * 4, a.g_last);
      };
      // Mixes: the groups of a stage are asked for a stage before its activations.  (Asked for with them, every stage waits for the
      // map, and with it for the codes requested before it: 8 experts of 7168 x 512 with one row each, 17.1 us.)
      int groups[FM == 3 ? NUT : 1];
      if constexpr (FM == 3)
#pragma unroll
        for (int i = 0; i < NUT; ++i) groups[i] = group_of(0, ulg[i]);
      u32x4 xr[NUT][NCH];
      auto load_x = [&](int s) {
#pragma unroll
        for (int i = 0; i < NUT; ++i) {
          const uint32_t g = (uint32_t)(FM == 3 ? groups[FM == 3 ? i : 0] : group_of(s, ulg[i]));
#pragma unroll
          for (int t = 0; t < NCH; ++t) xr[i][t] = load16(a.x, xoff[i][t] + g * (kGroup * 2));
        }
        if constexpr (FM == 3)
#pragma unroll
          for (int i = 0; i < NUT; ++i) groups[i] = group_of(s + 1, ulg[i]);
      };
      const uint32_t frag_off[2] = {(kq * 16u + (n ^ (2u * kq))) * 16u, (kq * 16u + (n ^ (2u * kq + 1u))) * 16u};
      const float cneg = a.cneg[kt];
      auto store_x = [&](int buf) {
        unsigned char* base = stage_mem + buf * kBuf;
        float* starts = reinterpret_cast<float*>(base + kFrags);
#pragma unroll
        for (int i = 0; i < NUT; ++i) {
          const uint32_t u = tid + (uint32_t)i * kThreads;
          const uint32_t uu = min(u, (uint32_t)NU - 1u), m = NARROW ? (uu >> 3) % (16u * LM) : (uu >> 2) % (16u * LM), c = NARROW ? uu & 7u : uu & 3u;
          const bool there = NU % kThreads == 0 || u < (uint32_t)NU;
          float sum = 0.f;
          if constexpr (NARROW) {
            const u32x4 v = xr[i][0];
            const u32x4 o = {__builtin_amdgcn_perm(v.z, v.x, 0x05040100u), __builtin_amdgcn_perm(v.z, v.x, 0x07060302u), __builtin_amdgcn_perm(v.w, v.y, 0x05040100u),
                             __builtin_amdgcn_perm(v.w, v.y, 0x07060302u)};
            sum = frag_sum(o, 0.f);
            sum = dpp_add<0x141>(dpp_add<0x4E>(dpp_add<0xB1>(sum)));
            if (there) *reinterpret_cast<u32x4*>(base + lds_off[i]) = o;
          } else {
            u32x4 o[3];
            const u32x4 v0 = xr[i][0], v1 = xr[i][1], v2 = xr[i][2];
            if constexpr (!H16) {
              const bool q3 = c == 3u;
              const uint32_t lo = q3 ? v1.z : v1.x, hi = q3 ? v1.w : v1.y;
              o[0] = u32x4{__builtin_amdgcn_perm(v0.y, v0.x, 0x07060100u), __builtin_amdgcn_perm(v0.z, v0.x, 0x05040302u), __builtin_amdgcn_perm(v0.z, v0.y, 0x07060100u), 0u};
              o[1] = u32x4{__builtin_amdgcn_perm(hi, lo, 0x07060100u), __builtin_amdgcn_perm(v1.z, lo, q3 ? 0x0C0C0302u : 0x05040302u),
                           __builtin_amdgcn_perm(v1.z, hi, q3 ? 0x0C0C0100u : 0x07060100u), 0u};
              o[2] = u32x4{__builtin_amdgcn_perm(v2.y, v2.x, q3 ? 0x0C0C0C0Cu : 0x07060100u), __builtin_amdgcn_perm(v2.z, v2.x, q3 ? 0x0C0C0C0Cu : 0x05040302u),
                           __builtin_amdgcn_perm(v2.z, v2.y, q3 ? 0x0C0C0C0Cu : 0x07060100u), 0u};
            } else {
              const bool odd = c & 1u;
              const uint32_t hs_x = odd ? 0x05040302u : 0x03020100u, hs_y = odd ? 0x07060504u : 0x05040302u, hs_w = odd ? 0x0C0C0302u : 0x0C0C0100u;
              o[0] = u32x4{__builtin_amdgcn_perm(v0.y, v0.x, hs_x), __builtin_amdgcn_perm(v0.z, v0.y, hs_y), __builtin_amdgcn_perm(v0.w, v0.z, hs_y), __builtin_amdgcn_perm(0u, v0.y, hs_w)};
              o[1] = u32x4{__builtin_amdgcn_perm(v1.y, v1.x, hs_x), __builtin_amdgcn_perm(v1.z, v1.y, hs_y), __builtin_amdgcn_perm(v1.w, v1.z, hs_y), __builtin_amdgcn_perm(0u, v1.y, hs_w)};
              const uint32_t h2_x = c == 0u ? 0x03020100u : (c == 1u ? 0x0C0C0302u : 0x0C0C0C0Cu), h2_y = c == 0u ? 0x05040302u : 0x0C0C0C0Cu, h2_w = c == 0u ? 0x0C0C0100u : 0x0C0C0C0Cu;
              const uint32_t lo = c == 1u ? v2.w : v2.x;
              o[2] = u32x4{__builtin_amdgcn_perm(v2.y, lo, h2_x), __builtin_amdgcn_perm(v2.z, v2.y, h2_y), __builtin_amdgcn_perm(v2.w, v2.z, h2_y), __builtin_amdgcn_perm(0u, v2.y, h2_w)};
            }
#pragma unroll
            for (int t = 0; t < 3; ++t) {
              sum = frag_sum(o[t], sum);
              if (there) *reinterpret_cast<u32x4*>(base + lds_off[i] + t * 1024u) = o[t];
            }
            sum = dpp_add<0x4E>(dpp_add<0xB1>(sum));
          }
          if (there) starts[ulg[i] * (16 * LM) + m] = cneg * sum;   // the same from all lanes of the row
        }
      };
      // k-tiles in registers: slot b holds tile b of every NB; it is asked for again as soon as it has been multiplied (no
      // copies from slot to slot: a copy waits for the load)
      constexpr int NB = NARROW && !(MT == 2 && RT == 2) ? 3 : 2;
      Tile held[NB];
      load_x(0);
#pragma unroll
      for (int b = 0; b < NB; ++b) load_tile(held[b], tA + b);
      lds_barrier();   // (a second kind or pass: the buffers have been read)
      store_x(0);
      load_x(1);
      float be[RT], al[RT];
      if constexpr (NARROW)
#pragma unroll
        for (int r = 0; r < RT; ++r) {
          be[r] = be_raw[r] + magic;
          al[r] = al_raw[r] * 16777216.f;
        }
      lds_barrier();
      int s = 0;
      auto tile = [&](Tile& cur, int ti) {
        const int t = tA + ti;
        if constexpr (SM == 1 && !NARROW) {
          // the field of a group sits in the code stream: byte 21 (quarter 3, segment 1) or word 9 (quarter 1, segment 2)
          const int src = (int)(((H16 ? 16u : 48u) + n) * 4u);
#pragma unroll
          for (int r = 0; r < RT; ++r) {
            const u32x4 held = cur.c[r][H16 ? 2 : 1];
            const uint32_t h0 = held.x, h1 = held.y, h2 = held.z, h3 = held.w;
            cur.s[r] = u32x4{(uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)h0), (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)h1),
                             (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)h2), (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)h3)};
          }
        }
#pragma unroll
        for (int h = 0; h < SPT; ++h) {
          store_x((s + 1) & 1);
          load_x(s + 2);
          __builtin_amdgcn_sched_barrier(0);
          const unsigned char* base = stage_mem + (s & 1) * kBuf;
          const float* starts = reinterpret_cast<const float*>(base + kFrags);
          if (t < tB) {
            // the sums of a row tile are added while the next one is decoded: nothing waits for the matrix core
            f32x4 p[LM];
            float psc = 0.f;
            auto add = [&](f32x4 (&to)[LM]) {
#pragma unroll
              for (int m = 0; m < LM; ++m)
#pragma unroll
                for (int i = 0; i < 4; ++i) to[m][i] = __builtin_fmaf(psc, p[m][i], to[m][i]);
            };
#pragma unroll
            for (int lg = 0; lg < 4; ++lg) {
              const int j = h * 4 + lg;
              u32x4 o[LM][T];
              f32x4 cin[LM];
#pragma unroll
              for (int m = 0; m < LM; ++m) {
#pragma unroll
                for (int k = 0; k < T; ++k) o[m][k] = *reinterpret_cast<const u32x4*>(base + ((lg * LM + m) * T + k) * 1024u + frag_off[NARROW ? k : 0]);
                cin[m] = *reinterpret_cast<const f32x4*>(starts + lg * (16 * LM) + m * 16 + 4 * kq);
              }
#pragma unroll
              for (int r = 0; r < RT; ++r) {
                u32x4 w[T];
                if constexpr (NARROW) {
                  const uint32_t d = dword_of(cur.c[r][0], j);
#pragma unroll
                  for (int k = 0; k < 2; ++k) {
                    const f16x2 qq = __builtin_bit_cast(f16x2, __builtin_amdgcn_perm(0u, d, k ? 0x0C030C02u : 0x0C010C00u));
                    const float fa = __builtin_fmaf((float)qq.x, al[r], be[r]);
                    const float fb = __builtin_fmaf((float)qq.y, al[r], be[r]);
                    const uint32_t yy = __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, fb), __builtin_bit_cast(uint32_t, fa), 0x05040100u);
                    w[k] = u32x4{and_or(yy >> 9, mask_n, c4300), and_or(yy >> 6, mask_n, c4300), and_or(yy >> 3, mask_n, c4300), and_or(yy, mask_n, c4300)};
                  }
                } else {
#pragma unroll
                  for (int k = 0; k < 3; ++k) {
                    const uint32_t d = dword_of(cur.c[r][k], j >> 1);
                    if constexpr (H16) {
                      const uint32_t hw = (j & 1) ? (d >> 16) : (d & 0xFFFFu), v = hw | (hw << 18);
                      w[k] = u32x4{and_or(v >> 13, mask_w, c4300), and_or(v >> 6, mask_w, c4300), and_or(v >> 2, mask_w, c4300), and_or(v >> 9, mask_w, c4300)};
                    } else {
                      const uint32_t pp = __builtin_amdgcn_perm(0u, d, (j & 1) ? 0x0C030C02u : 0x0C010C00u);
                      w[k] = u32x4{and_or(pp >> 4, mask_w, c4300), and_or(pp >> 2, mask_w, c4300), and_or(pp, mask_w, c4300), pp};
                    }
                  }
                }
                float sc;
                if constexpr (NARROW && SM == 1) {
                  sc = (float)((cur.s[r].x >> (4 * j)) & 0xFu);
                } else {
                  const uint32_t d = dword_of(cur.s[r], j >> 1), hw = (j & 1) ? (d >> 16) : (d & 0xFFFFu);
                  if constexpr (SM == 0) sc = (float)__builtin_bit_cast(_Float16, (uint16_t)hw);
                  else sc = (float)(H16 ? hw & 0x1FFFu : (hw >> 8) & 0xFu);
                }
                if constexpr (SIGNED) {
                  if constexpr (SM == 1) sc *= (float)__builtin_bit_cast(_Float16, (uint16_t)ssup[r]);
#pragma unroll
                  for (int k = 0; k < T; ++k) {
                    const u32x4 sw = signed_weights(w[k], cneg, sc);
#pragma unroll
                    for (int m = 0; m < LM; ++m) acc[r][m] = mfma(o[m][k], sw, acc[r][m]);
                  }
                } else {
                  if (lg > 0 || r > 0) add(acc[(r + RT - 1) % RT]);
                  asm volatile("" : "+v"(sc));   // converted once: v_fma_f32 issues at twice the rate of v_fma_mix_f32
                  psc = sc;
#pragma unroll
                  for (int m = 0; m < LM; ++m) {
                    p[m] = cin[m];
#pragma unroll
                    for (int k = 0; k < T; ++k) p[m] = mfma(o[m][k], w[k], p[m]);
                  }
                }
              }
            }
            if constexpr (!SIGNED) add(acc[RT - 1]);
          }
          if (h == SPT - 1) {
            __builtin_amdgcn_sched_barrier(0);
            load_tile(cur, t + NB);
          }
          lds_barrier();
          ++s;
        }
      };
      for (int ti = 0; ti < most; ti += NB) {
        tile(held[0], ti);
        if (ti + 1 >= most) break;
        tile(held[1], ti + 1);
        if constexpr (NB == 3) {
          if (ti + 2 >= most) break;
          tile(held[2], ti + 2);
        }
      }
    };
    if constexpr (FM == 1 || FM == 3) kind(std::integral_constant<int, kKN>{});
    if constexpr (FM == 2 || FM == 3) kind(std::integral_constant<int, kKW>{});
    if constexpr (FM == 4) kind(std::integral_constant<int, kKH>{});

    // Infinite activations: the products with 128 + state and the start value are infinities of both signs, their sum is NaN.  Dense
    // calls of 17 to 32 rows on the wide kinds, whose neighbours take kernels that multiply signed weights, are done again with
    // those where a sum is not finite: an infinity then gives infinities (NaN with a zero weight), as there.
    const bool again = !SIGNED && FM != 1 && MT == 2 && !a.expert_offsets && a.M > 16;
    if (again) {
      float f = 0.f;   // NaN if an addend is infinite or NaN
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int m = 0; m < LM; ++m)
#pragma unroll
          for (int i = 0; i < 4; ++i) f = __builtin_fmaf(acc[r][m][i], 0.f, f);
      if (f != f) not_finite = 1;
    }
    if (a.wk > 1) {
      f32x4* red = reinterpret_cast<f32x4*>(smem);   // the activations' place: all are done with them
      // the lane, asked for anew: addresses made of it are not held in registers over the loops above
      uint32_t every = ~0u;
      asm volatile("" : "+s"(every));
      const uint32_t lane = __builtin_amdgcn_mbcnt_hi(every, __builtin_amdgcn_mbcnt_lo(every, 0u));
      if (wk > 0) {
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
          for (int m = 0; m < LM; ++m) red[((((wk - 1) * WN + wn) * RT + r) * LM + m) * 64u + lane] = acc[r][m];
      }
      lds_barrier();
      if (wk == 0) {
        for (uint32_t k = 1; k < (uint32_t)a.wk; ++k)
#pragma unroll
          for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int m = 0; m < LM; ++m) acc[r][m] += red[((((k - 1) * WN + wn) * RT + r) * LM + m) * 64u + lane];
      }
    } else if (again) {
      lds_barrier();
    }
    if (again && __builtin_amdgcn_readfirstlane(not_finite)) return false;
    if (wk == 0) {
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        const uint32_t col = (rt0 + r) * 16u + n;
        if (rt0 + r < (uint32_t)a.row_tiles && col <= (uint32_t)a.n_last) {
          const float mul = SM == 1 && !SIGNED ? (float)__builtin_bit_cast(_Float16, (uint16_t)ssup[r]) : 1.f;
#pragma unroll
          for (int m = 0; m < LM; ++m)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int32_t row = m0 + 16 * m + 4 * (int32_t)kq + i;
              if (row < rows) a.y[(size_t)(row0 + row) * (size_t)a.ldy + col] = to_bf16(SM == 1 && !SIGNED ? acc[r][m][i] * mul : acc[r][m][i]);
            }
        }
      }
    }
    return true;
  };
  for (int32_t m0 = 0; m0 < rows; m0 += 16 * MT) {
    if (MT == 1 || rows - m0 <= 16) {
      pass(std::integral_constant<int, 1>{}, std::false_type{}, m0);
    } else if (!pass(std::integral_constant<int, MT>{}, std::false_type{}, m0)) {
      if constexpr (FM != 1 && MT == 2) pass(std::integral_constant<int, MT>{}, std::true_type{}, m0);
    }
  }
}

typedef void (*Kernel)(const Args);
template <int FM, int SM>
static Kernel pick(int mt, int rt, int wn) {
  if (rt == 1 && wn == 2) return mt == 1 ? ccq_few_kernel<FM, SM, 1, 1, 2> : ccq_few_kernel<FM, SM, 2, 1, 2>;
  if (rt == 1 && wn == 4) return mt == 1 ? ccq_few_kernel<FM, SM, 1, 1, 4> : ccq_few_kernel<FM, SM, 2, 1, 4>;
  if (rt == 2 && wn == 8) {
    if (mt == 2) return ccq_few_kernel<FM, SM, 2, 2, 8>;
    if constexpr (FM == 1) return ccq_few_kernel<FM, SM, 1, 2, 8>;
    return nullptr;
  }
  if (rt == 2 && wn == 4) {
    if (mt == 1) return ccq_few_kernel<FM, SM, 1, 2, 4>;
    if constexpr (FM != 3) return ccq_few_kernel<FM, SM, 2, 2, 4>;   // (a mix does not fit the registers)
  }
  return nullptr;
}
static Kernel pick_kernel(int fm, int sm, int mt, int rt, int wn) {
  switch (fm * 2 + sm) {
    case 2: return pick<1, 0>(mt, rt, wn);
    case 3: return pick<1, 1>(mt, rt, wn);
    case 4: return pick<2, 0>(mt, rt, wn);
    case 5: return pick<2, 1>(mt, rt, wn);
    case 6: return pick<3, 0>(mt, rt, wn);
    case 7: return pick<3, 1>(mt, rt, wn);
    case 8: return pick<4, 0>(mt, rt, wn);
    default: return pick<4, 1>(mt, rt, wn);
  }
}

struct Shape {
  int rt = 0, wn = 0, wk = 0;
  uint32_t lds = 0;
};
// Wavefronts that a SIMD holds of an instance, by the registers that the compiler gave it.
static int waves_held(int fm, int mt, int rt, int wn) {
  if (fm == 1) return mt == 2 ? 3 : (rt == 2 ? 4 : 5);
  if (fm == 3) return mt == 1 && rt == 1 ? 3 : 2;
  return mt == 2 ? 2 : (rt == 1 && wn == 4 ? 4 : 3);
}

// The launch shape, by an estimate in cycles.  A stage of a wavefront: its instructions (decode and products of RT x LM tiles, its part of
// the staging, the rest) times the wavefronts that share the SIMD, or the latency of one wavefront where few do, and the wait at
// the barrier, which other workgroups on the CU cover.  Times the stages of the longest share of K and the passes over the
// rows, with what starting a pass takes; times the rounds of workgroups over the chip.  Where the grid has experts without
// rows, their workgroups cost a dispatch each, and the others land unevenly on the CUs.  The constants are fitted to 33000 timings: all
// shapes on 3404 random calls (K 512 .. 28672, N 512 .. 28672, 1 .. 256 matrices, 1 .. 512 tokens, with and without the host offsets).
// The shape taken is on average 2 % slower than the best one (twentieth of the calls: 12 to 17 %); with the estimate of one pass over
// the rows of all matrices that came before it was 7 to 18 % (us, before / now: 256 experts of 1024 x 2048, 16 tokens, hybrid word
// 52 / 31; 64 of 7168 x 2048, 4 tokens without host offsets, mix 86 / 46).
// Eight wavefronts of two row tiles each are not taken with experts without rows (the lone workgroup of a CU: 114 experts of 704 x
// 1493, 16 tokens, hybrid word, 21 against 12 us) and not built for one 16-row tile on the wide kinds (best in 10 of 146 calls).
static Shape choose_shape(const Layout& L, int fm, const FewRows& f) {
  static const int kShapes[][3] = {{1, 2, 1}, {1, 2, 2}, {1, 2, 4}, {1, 4, 1}, {1, 4, 2}, {1, 4, 4}, {2, 4, 1}, {2, 4, 2}, {2, 8, 1}};
  const int mt = f.most_rows <= 16 ? 1 : 2;
  const int64_t cus = device_cus();
  const double empty = 1.0 - (double)f.with_rows / (double)f.matrices;
  Shape best;
  double least = 0.0;
  for (const auto& c : kShapes) {
    const int rt = c[0], wn = c[1], wk = c[2], waves = wn * wk;
    if (waves > max_waves(fm, mt, rt, wn) || (fm == 3 && mt == 2 && rt == 2 && wn == 4)) continue;
    if (wn == 8 && (empty > 0.0 || (fm != 1 && mt == 1))) continue;
    const uint32_t lds = std::max<uint32_t>((uint32_t)(wk * 2) * buffer_bytes(fm, mt), (uint32_t)((wk - 1) * wn * rt * mt) * 1024u);
    if (lds > 150u * 1024u) continue;
    const int64_t slots = std::max<int64_t>(1, std::min<int64_t>(4 * waves_held(fm, mt, rt, wn) / waves, 160 * 1024 / lds));   // workgroups of a CU
    const int64_t blocks = (L.row_tiles + rt * wn - 1) / (rt * wn), wgs = f.with_rows * blocks;
    // all passes of a workgroup with `held` of them on its CU
    auto workgroup = [&](double held) {
      const double per_simd = held * waves / 4.0;
      double t = 0.0;
      for (int lm = 1; lm <= 2; ++lm) {
        auto stage = [&](double tile, double unit, double rest) {
          const double issue = rt * 4 * tile + unit * lm / wn + rest;
          return std::max(per_simd * issue * 5.5, issue * 7.6 + 340.0) + 144.0 * waves / 4.0 / held;
        };
        t += f.passes[lm - 1] / (double)f.with_rows *
             (((L.tiles[kNarrow] + wk - 1) / wk) * stage(21.6 + 4.2 * lm, 180.0, 32.0) + 2 * ((L.tiles[kWide] + wk - 1) / wk) * stage(21.6 + 8.8 * lm, 208.0, 23.0) + 6500.0 + 750.0 * wk);
      }
      return t;
    };
    const int64_t full = wgs / (cus * slots), rest = wgs % (cus * slots);
    double t = (double)full * workgroup((double)slots) + 6.0 * (double)((f.matrices - f.with_rows) * blocks);
    if (rest) {
      const double even = (double)((rest + cus - 1) / cus), uneven = 1.0 + 1.72 * empty * (double)rest / (double)cus + (1.0 - empty) * (even - 1.0);
      t += workgroup(empty > 0.0 ? std::min((double)slots, uneven) : even);
    }
    if (best.rt == 0 || t < least) {
      least = t;
      best.rt = rt, best.wn = wn, best.wk = wk, best.lds = lds;
    }
  }
  return best;
}

static int format_of(const Layout& L) { return L.h16 ? 4 : (L.tiles[kNarrow] > 0 ? 1 : 0) | (L.tiles[kWide] > 0 ? 2 : 0); }

}  // namespace few

void few_shape(const Layout& L, const FewRows& f, int (&shape)[4]) {
  const few::Shape s = few::choose_shape(L, few::format_of(L), f);
  shape[0] = f.most_rows <= 16 ? 1 : 2, shape[1] = s.rt, shape[2] = s.wn, shape[3] = s.wk;
}

// T: rows of x.
int launch_few(const SkinnyCall& c, int T, const FewRows& f) {
  using namespace few;
  const Layout& L = c.L;
  if ((int64_t)T * c.ldx * 2 >= (int64_t)1 << 32 || f.matrices > 65535) return CCQ_ERR_UNSUPPORTED;   // activation offsets are 32-bit
  Args a;
  a.codes = static_cast<const uint8_t*>(c.w->codes);
  a.scales = static_cast<const uint16_t*>(c.w->scales);
  a.alpha = c.w->code_alpha;
  a.beta = c.w->code_beta;
  a.meta = static_cast<const int32_t*>(c.w->meta);
  a.scale_super = static_cast<const uint16_t*>(c.w->scale_super);
  a.x = static_cast<const uint16_t*>(c.x);
  a.y = static_cast<uint16_t*>(c.y);
  a.sorted_rows = c.sorted_rows;
  a.expert_offsets = c.expert_offsets;
  a.codes_stride = c.codes_stride;
  a.scales_stride = c.scales_stride;
  a.ab_stride = c.ab_stride;
  a.ldx = c.ldx;
  a.ldy = c.ldy;
  a.row_tile_bytes = L.row_tile_bytes;
  a.row_tile_scale_halfs = L.row_tile_scale_halfs;
  a.M = c.M;
  a.row_tiles = L.row_tiles;
  a.groups_narrow = L.pgroups[kNarrow];
  a.g_last = L.G - 1;
  a.n_last = L.N - 1;
  for (int k = 0; k < 2; ++k) {
    a.tiles[k] = L.tiles[k];
    a.cneg[k] = -(128.f + L.zp[k]);
  }
  a.n_active = c.n_active;
  std::memcpy(a.active_ids, c.active_ids, sizeof(a.active_ids));
  const int fm = format_of(L), mt = f.most_rows <= 16 ? 1 : 2;
  const Shape s = choose_shape(L, fm, f);
  const Kernel k = pick_kernel(fm, L.scale_mode, mt, s.rt, s.wn);
  if (!k) return CCQ_ERR_UNSUPPORTED;
  a.wk = s.wk;
  if (s.lds > 48 * 1024 && hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)s.lds) != hipSuccess) {
    (void)hipGetLastError();
    return CCQ_ERR_HIP;
  }
  const dim3 grid((unsigned)((L.row_tiles + s.wn * s.rt - 1) / (s.wn * s.rt)), (unsigned)f.matrices);
  hipLaunchKernelGGL(k, grid, dim3((unsigned)(64 * s.wn * s.wk)), s.lds, static_cast<hipStream_t>(c.stream), a);
  return hipGetLastError() == hipSuccess ? CCQ_OK : CCQ_ERR_HIP;
}

}  // namespace ccq

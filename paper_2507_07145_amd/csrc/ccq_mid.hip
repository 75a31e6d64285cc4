// Fused dequantize-and-multiply for a few dozen activation rows (17 to 64; more where the product is too small for the prompt kernel's
// blocks, ccq_block.h, to fill the chip; experts with more than 32 rows, likewise), any mix of the narrow (L=6,N=4,S=3 + Code
// Cluster) and wide (L=4,N=3,S=2) formats, gfx950.
//
// With that many rows the per-row-tile kernel re-stages the activations far too often, and taller blocks waste most of their tile.  Here a workgroup of four wavefronts owns a 64 x 128 (or, on the
// narrow format, 128 x 128) tile of the output and a share of K (S shares across the grid, up to four in a workgroup; fp32 partial tiles go to
// the workspace and are added in index order by the reduction kernel when S > 1).  K is walked one 64-weight group per
// step; per step
//   - the workgroup copies the activation tile of that group's columns to LDS,
//   - every wavefront decodes its 32 columns of the group to bf16 in registers: window extraction by the shift lists
//     [9,6,3,0] / [4,2,0] and masks 0x3F / 0xF of Table 1 into the mantissas of two fp16 64.0, then
//     d = (w_uint - zp) * s (Alg. 2 / Alg. 3, last line) as fma(64 + state, s, -(64 + zp) s),
//     which is exact in fp32, so the bf16 is the correctly rounded exact weight,
//   - and multiplies them with the activation tile by MFMA 32x32x16 bf16 (fp32 accumulators).
// The hybrid 16-bit word of Sec. 3.2 (a (3,3,2) and a (3,4,2) code side by side, seven weights per
// word, ten words per group) takes the place of the wide format when it is used: eight k-slots per word (seven weights
// and one unused slot, 80 slots per group), five MFMA k-steps instead of four.
// The decode (about 3 vector instructions per weight, shared by the rows of the block) and the way of the activations through LDS
// (every wavefront reads the whole tile: 1 KB per MFMA) are the bound: of 206 us (wide 8192 x 8192, M = 1024) 75 go without the decode,
// 38 without the LDS stores, 18 without the MFMAs.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "ccq_decode.h"
#include "ccq_internal.h"

namespace ccq {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef u32x4 u32x4_dword __attribute__((aligned(4)));

struct MidArgs {
  const uint8_t* codes;
  const uint16_t* scales;
  const float* alpha;
  const float* beta;
  const int32_t* meta;
  const uint16_t* scale_super;  // fp16 [N], compressed scales only
  const uint16_t* x;
  uint16_t* y;
  float* partial;
  int64_t ldx, ldy;
  int64_t row_tile_bytes, row_tile_scale_halfs;
  int32_t M, N, row_tiles;  // N: rows of the device layout (a multiple of 16), the row stride of `partial`
  int32_t tiles[2];       // k-tiles per kind
  int32_t groups_narrow;  // narrow entries of the group map (whole k-tiles), the offset of the wide ones
  int32_t g_last;         // last real group of K: groups past it pad a k-tile (zero scale) and read this group's activations
  int32_t n_last;         // last real output row: rows past it pad a row tile, take its parameters and are not stored
  int32_t wk;             // K shares within a workgroup, 256 threads each (of S wk in all)
  int32_t sq[2], sr[2];   // K shares: share `split` owns tiles [split*sq + min(split, sr), +sq + (split < sr)) of each kind
  float zp[2];
  // grouped calls: blockIdx.z = expert; its rows are output rows [offsets[e], offsets[e+1]),
  // activation row sorted_rows[p] for output row p; expert e's arrays start e * stride bytes after expert 0's
  const int32_t* sorted_rows;
  const int32_t* expert_offsets;
  int64_t codes_stride, scales_stride, ab_stride;
};

constexpr int kMidBM = 64;
constexpr int kMidBN = 128;
constexpr int kMaxGridY = 65535;
constexpr int kMidRow = 64 + 8;     // bf16 elements per padded LDS row (144 bytes)
constexpr int kMidRowH16 = 80 + 8;  // the same for the hybrid word: ten words of eight slots (176 bytes)

__device__ __forceinline__ uint32_t and_or_m(uint32_t a, uint32_t mask, uint32_t orv) { return __builtin_amdgcn_bitop3_b32(a, mask, orv, 0xEA); }

__device__ __forceinline__ uint32_t pack_bf16_m(float lo, float hi) {
  f32x2 v = {lo, hi};
  bf16x2 b = __builtin_convertvector(v, bf16x2);  // round to nearest even
  return __builtin_bit_cast(uint32_t, b);
}

__device__ __forceinline__ uint32_t dword_sel(const u32x4& v, int j) { return j == 0 ? v.x : (j == 1 ? v.y : (j == 2 ? v.z : v.w)); }

// A wavefront multiplies exactly the 32 columns it decodes, so the decoded weights never leave its registers: MFMA
// 32x32x16 wants lane l to hold column l % 32 and eight k-slots of half h = l / 32, and a lane loads from the code
// stream just the 16-byte entries (of one quarter of its row and all groups of the k-tile) that hold those weights.
//   narrow  quarters 2h and 2h + 1: weights 32 h .. 32 h + 31 of every group, k-slots 8 kk .. of half h are weights
//           32 h + 8 kk ..
//   wide    the same 32 weights sit in codes 0 .. 10 (h = 0) or 10 .. 21 (h = 1), three to a byte: six two-byte entries
//           per group, the one with code 10 in both halves.  Ten whole codes are decoded pairwise, the two weights
//           beside them (30, 31 or 32, 63) one by one, and one funnel shift per dword moves the row into place, by
//           zero or by one weight.
//   hybrid word (Sec. 3.2)  words h, 2 + h, 4 + h, 6 + h, 8 + h: seven weights and one unused slot are the eight k-slots
//           of one MFMA, five of them per group; the activation tile lies in the same slot order.
// FM: formats present (1 narrow, 2 wide, 3 both, 4 the hybrid word; a group map exists only for 3).  SM: scale mode (0 fp16 group
// scales; 1 the compressed scales of Sec. 3.4: group scale = 4-bit field * per-row super scale, first line of
// Alg. 2 / Alg. 3; the field of a narrow group comes from the packed scale array, that of a wide group from the
// spare low nibble of the group's last code byte, the hybrid word's 13-bit field from its last word).
// BM: rows of the block (64, or 128 on the narrow format: a weight tile decoded once for twice the rows).
// a.wk shares of K sit in one workgroup (256 threads and an activation tile each); share s of the workgroup works on k-tiles of
// shares split + s S, so that a long one meets short ones, and the sums meet in LDS.
// DEEP: two wavefronts per SIMD with four activation tiles on their way and the next step's fragments decoded during the current
// one, for launches that have no more wavefronts than that to give; otherwise three (four on narrow 64-row blocks) that
// cover each other's latencies (64 experts of 2048 x 7168, 48 - 85 rows: 209 -> 200 us; wide 1024 x 20000, M = 1500, 1.12 x; with up
// to two workgroups per CU the lean variant is up to a fifth slower: 16 experts of 2048 x 1536, one with 600 rows, 28 against 35 us).
// A priority for the wavefronts that multiply (or for those that decode), shares that alternate between the two, and a scheduling
// barrier between the two all cost 3 to 8 %: the compiler's interleaving of one step's decode and products is what overlaps them.
// FAR: the deep schedule with 64-bit offsets of the activation rows, for rows that lie further apart than 32 bits reach from the
// first one of a block (dense) or of x (grouped).  In a dense call, whose offsets count from the block, it is level with 32-bit
// ones and stands for both; grouped calls lose by it (narrow, 16 experts of 2048 x 1536, 80 rows each, 19.8 / 21.1 us).
enum Schedule { kLean, kDeep, kFar };
constexpr int mid_waves(int fm, int bm, bool deep) { return deep ? 2 : (fm == 1 && bm == kMidBM ? 4 : 3); }
template <int FM, int SM, bool GROUPED, int BM, Schedule SCHEDULE>
__global__ void __launch_bounds__(256 * mid_waves(FM, BM, SCHEDULE != kLean))
    __attribute__((amdgpu_waves_per_eu(mid_waves(FM, BM, SCHEDULE != kLean), SCHEDULE != kLean && FM != 4 ? 2 : 8))) ccq_mid_kernel(const MidArgs a) {
  constexpr bool DEEP = SCHEDULE != kLean;
  constexpr bool HAS_N = FM == 1 || FM == 3, HAS_W = FM >= 2, META = FM == 3, H16 = FM == 4;
  constexpr int ROW = H16 ? kMidRowH16 : kMidRow;
  constexpr int MT = BM / 32;          // 32-row accumulator tiles, and 16-byte activation chunks per thread and step (chunk i: rows of tile i)
  constexpr int KK = H16 ? 5 : 4;      // MFMAs per group and accumulator tile
  constexpr int NQ = H16 ? 5 : 6;      // 16-byte entries of a wide k-tile that a lane reads
  constexpr int WTILE = H16 ? kH16TileBytes : kWideTileBytes;
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x & 255, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wk = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);   // share of K within the workgroup
  uint16_t* As = reinterpret_cast<uint16_t*>(smem) + wk * 2 * BM * ROW;    // [2][BM][ROW] of this share
  // original group of each step of this share (META only); every share has room for the longest
  int32_t* lds_meta = reinterpret_cast<int32_t*>(reinterpret_cast<uint16_t*>(smem) + a.wk * 2 * BM * ROW) + wk * ((a.sq[kNarrow] + 1) * kNarrowGroupsPerTile + (a.sq[kWide] + 1) * kWideGroupsPerTile);

  // row blocks of a column block side by side: they share its codes
  const int m_block = blockIdx.x, n_block = blockIdx.y;   // (from one index a division costs 0.4 us)
  const int split = GROUPED ? 0 : blockIdx.z, splits = GROUPED ? 1 : gridDim.z;
  const int m0 = m_block * BM, n0 = n_block * kMidBN;
  // rows of this block's matrix: all M (dense), or the expert's (grouped; row_off = its first output row)
  int Me = a.M, row_off = 0;
  int64_t e_codes = 0, e_scales = 0, e_ab = 0;
  if constexpr (GROUPED) {
    const int e = blockIdx.z;
    row_off = a.expert_offsets[e];
    Me = a.expert_offsets[e + 1] - row_off;
    if (m0 >= Me) return;  // uniform: before any barrier
    e_codes = e * a.codes_stride;
    e_scales = e * a.scales_stride;
    e_ab = e * a.ab_stride;
  }
  const int nl = lane & 15;
  const int ti = (lane >> 4) & 1, h = lane >> 5;  // the column this lane multiplies: row tile ti of the wavefront, row nl; k half h

  // this share's k-tiles of each kind, and its steps (one 64-weight group each): narrow first, then wide
  const int share = split + wk * splits;   // the longer shares come first: a workgroup of two has at most one of them
  int tA[2], tB[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    tA[k] = share * a.sq[k] + min(share, a.sr[k]);
    tB[k] = tA[k] + a.sq[k] + (share < a.sr[k] ? 1 : 0);
  }
  const int nsN = HAS_N ? (tB[kNarrow] - tA[kNarrow]) * kNarrowGroupsPerTile : 0;
  const int nsW = HAS_W ? (tB[kWide] - tA[kWide]) * kWideGroupsPerTile : 0;
  const int nsteps = nsN + nsW;  // a multiple of four: both terms are

  if constexpr (META) {
    for (int s = tid; s < nsteps; s += 256) {
      const int pg = s < nsN ? tA[kNarrow] * kNarrowGroupsPerTile + s : a.groups_narrow + tA[kWide] * kWideGroupsPerTile + (s - nsN);
      lds_meta[s] = a.meta[pg];
    }
    __syncthreads();
  }
  // original group (activation columns 64 g .. 64 g + 63) of step s
  auto group_of = [&](int s) -> int {
    s = min(s, nsteps - 1);
    if constexpr (META) return lds_meta[s];
    return min((HAS_N ? tA[kNarrow] * kNarrowGroupsPerTile : tA[kWide] * kWideGroupsPerTile) + s, a.g_last);
  };

  const int rtile0 = min(n0 / 16 + wave * 2, a.row_tiles - 1), rtile = min(n0 / 16 + wave * 2 + ti, a.row_tiles - 1);  // ragged last block: re-decode the last tile, never stored
  const int prow = min(rtile * 16 + nl, a.n_last);
  // Uniform bases and 32-bit lane offsets: with three or four wavefronts on a SIMD no vector instruction is spent on the addresses
  // of a request.  (With one or two, where a step waits for its latencies, 64-bit lane addresses are level or up to 4 % faster: a
  // uniform one has to come back from the group map through a readfirstlane.)
  const uint8_t* code_row = a.codes + e_codes + (int64_t)rtile0 * a.row_tile_bytes;
  const uint16_t* scale_row = reinterpret_cast<const uint16_t*>(reinterpret_cast<const uint8_t*>(a.scales) + e_scales) + (int64_t)rtile0 * a.row_tile_scale_halfs;
  const uint32_t code_lane = (uint32_t)(rtile - rtile0) * (uint32_t)a.row_tile_bytes, scale_lane = (uint32_t)(rtile - rtile0) * (uint32_t)a.row_tile_scale_halfs * 2u;
  float al = 0.f, bem = 0.f, ssup = 0.f;
  // expert e's super scales: half the byte stride of alpha / beta (fp16 against fp32)
  if constexpr (SM == 1)
    ssup = (float)__builtin_bit_cast(_Float16, reinterpret_cast<const uint16_t*>(reinterpret_cast<const uint8_t*>(a.scale_super) + e_ab / 2)[prow]);
  if constexpr (HAS_N) {
    al = reinterpret_cast<const float*>(reinterpret_cast<const uint8_t*>(a.alpha) + e_ab)[prow] * kAlphaScale;
    bem = reinterpret_cast<const float*>(reinterpret_cast<const uint8_t*>(a.beta) + e_ab)[prow] + 8388608.f;  // + 2^23: exact, beta is an integer below 2^15
  }
  const uint8_t* code_wide = code_row + (int64_t)a.tiles[kNarrow] * kNarrowTileBytes;
  const uint16_t* scale_wide = scale_row + (int64_t)a.tiles[kNarrow] * kNarrowTileScaleHalfs;
  uint32_t c43 = 0x43000000u, mask2 = kDecMask2, base2 = kDecBase2, mask_w = 0x00070000u;  // mask_w: the hybrid word's 3-bit states
  asm volatile("" : "+v"(c43), "+s"(mask2), "+v"(base2), "+s"(mask_w));
  // fp16 scales: the windows stay where they lie, but for the narrow format alone (33 to 100 rows: wide 42 x 4416 x 3408 17.5 -> 17.2 us; mix
  // 93 x 1600 x 2386 17.1 -> 16.5, with the wide ones only 16.8; narrow level, seventeen calls within 1 %)
  constexpr bool kWindowsN = SM == 0 && HAS_W;
  DecWindows win_n{}, win_w{};
  if constexpr (kWindowsN) win_n = dec_windows<false>();
  if constexpr (HAS_W && !H16) win_w = dec_windows<true>();

  // code entries in registers: the k-tile being decoded and the next one of the same kind
  u32x4 cn[2], cn_next[2];
  uint2 sn, sn_next;
  u32x4 cw[NQ], cw_next[NQ];
  uint4 sw, sw_next;
  uint32_t woff[NQ];  // byte offset of entry i in a wide k-tile
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const int e = H16 ? 2 * i + h : 5 * h + i;                 // word, or two-byte entry, of the group
    const int t = H16 ? e / 4 : e % 3, kq = H16 ? e % 4 : e / 3;
    woff[i] = code_lane + t * 1024 + (kq * 16 + nl) * 16;
  }
  auto load_narrow = [&](u32x4 (&c)[2], uint2& sc, int kt) {
    kt = min(kt, a.tiles[kNarrow] - 1);
    const uint8_t* t = code_row + (int64_t)kt * kNarrowTileBytes;
    uint32_t off = code_lane + (uint32_t)(nl + 32 * h) * 16u, soff = scale_lane + (uint32_t)nl * (SM == 0 ? 8u : 2u);
    asm volatile("" : "+v"(off), "+v"(soff));
#pragma unroll
    for (int q = 0; q < 2; ++q) c[q] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(t + off + q * 256));
    const char* sb = reinterpret_cast<const char*>(scale_row + (int64_t)kt * (SM == 0 ? kNarrowTileScaleHalfs : kNarrowTileScaleHalfs4)) + soff;
    if constexpr (SM == 0) sc = *reinterpret_cast<const uint2*>(sb);
    else sc = uint2{(uint32_t)*reinterpret_cast<const uint16_t*>(sb), 0u};  // the tile's four 4-bit fields
  };
  auto load_wide = [&](u32x4 (&c)[NQ], uint4& sc, int kt) {
    kt = min(kt, a.tiles[kWide] - 1);
    const uint8_t* t = code_wide + (int64_t)kt * WTILE;
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      uint32_t off = woff[i];
      if constexpr (!DEEP) asm volatile("" : "+v"(off));
      c[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(t + off));
    }
    if constexpr (SM == 0) {
      uint32_t soff = scale_lane + (uint32_t)nl * 16u;
      asm volatile("" : "+v"(soff));
      sc = *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(scale_wide + (int64_t)kt * kWideTileScaleHalfs) + soff);
    } else {
      sc = uint4{0u, 0u, 0u, 0u};  // the fields sit in the code stream
    }
  };

  const uint16_t* xbase = a.x + (GROUPED ? 0 : (int64_t)m0 * a.ldx);
  // Activation chunks of a step per thread.  Chunk i is 16 bytes of a row of tile i, or, with the hybrid word, the eight slots of one
  // word (element e of a group sits in slot 8 (e / 7) + e % 7, the eighth slot is zero): ten to a row, 640 to a tile, which 256
  // threads take in three rounds (the last one repeats half).  A word's seven elements lie in 16 bytes that start on a dword: at an
  // even word's first element, or one element before an odd word's; word 9 is the last element of the row's last 16 bytes.
  // (777 rows of 7232 x 5001, compressed scales: 161 us; with eight 16-bit writes per 16 bytes into the slots 168 us.)
  constexpr int CHUNKS = H16 ? 3 : MT;
  static_assert(!H16 || BM == 64, "");
  using RowOffset = std::conditional_t<SCHEDULE == kFar, int64_t, uint32_t>;
  RowOffset xoff[CHUNKS];   // bytes from xbase
  int a_lds[H16 ? CHUNKS : 1];   // halfword of chunk i in the tile; of chunk 0: chunk i lies 32 rows further per i
  bool last_word[CHUNKS];
  if constexpr (!H16) a_lds[0] = (tid >> 3) * ROW + (tid & 7) * 8;
#pragma unroll
  for (int i = 0; i < CHUNKS; ++i) {
    int c = tid + 256 * i;
    if (H16 && c >= 640) c -= 640;
    const int row = H16 ? c / 10 : c >> 3, u = H16 ? c % 10 : c & 7;
    const int byte = H16 ? (u == 9 ? 112 : 14 * u - 2 * (u & 1)) : 16 * u;
    int64_t xr = row_off + min(m0 + row, Me - 1);  // rows past the end re-read the last row; their products are never stored
    if constexpr (GROUPED) {
      if (a.sorted_rows) xr = a.sorted_rows[xr];
    } else {
      xr -= m0;
    }
    xoff[i] = (RowOffset)(xr * a.ldx * 2 + byte);
    if constexpr (H16) a_lds[i] = row * ROW + 8 * u;
    last_word[i] = H16 && u == 9;
  }
  const uint32_t odd_word = H16 && (tid & 1) ? 16u : 0u;   // 256 and 640 are even: so is every chunk's word, or none

  auto half_of = [](uint32_t d, int j) -> uint32_t { return (j & 1) ? (d >> 16) : (d & 0xFFFFu); };
  auto fp16_of = [&](uint32_t d, int j) -> float { return (float)__builtin_bit_cast(_Float16, (uint16_t)half_of(d, j)); };
  // group j of the held narrow k-tile: 32 weights of this lane's column, as four MFMA B fragments
  auto decode_narrow = [&](u32x4 (&bf)[KK], int j) {
    float s;
    if constexpr (SM == 0) s = fp16_of((j >> 1) ? sn.y : sn.x, j);
    else s = (float)((sn.x >> (4 * j)) & 0xFu) * ssup;  // (s_q >> s_shift) & s_mask times s_super: exact
    float c0[3];   // exact: 8-bit times at most 15-bit significand (fp16 scales: 12-bit times 11-bit)
#pragma unroll
    for (int i = 0; i < (kWindowsN ? 3 : 1); ++i) c0[i] = -(kNarrowBases[i] + a.zp[kNarrow]) * s;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      uint32_t o[8];
      if constexpr (kWindowsN) decode16_narrow_fp16(dword_sel(cn[q], j), al, bem, s, c0, win_n, o);
      else decode16_narrow(dword_sel(cn[q], j), al, bem, s, c0[0], mask2, base2, o);
      bf[2 * q] = u32x4{o[0], o[1], o[2], o[3]};
      bf[2 * q + 1] = u32x4{o[4], o[5], o[6], o[7]};
    }
  };
  const WideLane wlane = wide_lane(h);
  // group j of the held wide (or hybrid-word) k-tile
  auto decode_wide = [&](u32x4 (&bf)[KK], int j) {
    float s;
    if constexpr (SM == 0) {
      s = fp16_of(dword_sel(u32x4{sw.x, sw.y, sw.z, sw.w}, j >> 1), j);
    } else {
      // Alg. 2: the low nibble of the group's last code byte (byte 21), or the low 13 bits of its last word (the
      // scale mask 0x1FFF of Table 1); half 1 of the column holds both in its last entry
      const uint32_t own = dword_sel(cw[NQ - 1], j >> 1);
      const uint32_t last = half_of((uint32_t)__builtin_amdgcn_ds_bpermute((lane | 32) * 4, (int)own), j);
      s = (float)(H16 ? last & 0x1FFFu : (last >> 8) & 0xFu) * ssup;  // exact: at most 13-bit integer times 11-bit significand
    }
    if constexpr (H16) {
      // seven 3-bit states per word at the shifts [13,11,9,6,4,2,0] (Table 1), each moved to bit 16, the lowest
      // integer bit of fp32 128.0
      const float c0 = -(128.f + a.zp[kWide]) * s;
      const float zoff = 128.f + a.zp[kWide];
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        const uint32_t w = half_of(dword_sel(cw[kk], j >> 1), j);
        // With fp16 group scales (128 + zp) s is exact and one fused multiply-add gives the exactly rounded
        // weight.  A 13-bit field times an 11-bit super scale fills all 24 bits of s, so there the offset is
        // taken off first (exact) and the product (state - zp) s is rounded once to fp32.
        auto value = [&](uint32_t shifted) -> float {
          const float st = __builtin_bit_cast(float, and_or_m(shifted, mask_w, c43));  // 128 + state
          if constexpr (SM == 0) return __builtin_fmaf(st, s, c0);
          else return (st - zoff) * s;
        };
        const float f0 = value(w << 3), f1 = value(w << 5), f2 = value(w << 7), f3 = value(w << 10);
        const float f4 = value(w << 12), f5 = value(w << 14), f6 = value(w << 16);
        // the eighth slot of a word meets a zero activation; any finite value will do
        bf[kk] = u32x4{pack_bf16_m(f0, f1), pack_bf16_m(f2, f3), pack_bf16_m(f4, f5), pack_bf16_m(f6, f6)};
      }
    } else {
      float c0[3];
#pragma unroll
      for (int i = 0; i < (SM == 0 ? 3 : 1); ++i) c0[i] = -(kWideBases[i] + a.zp[kWide]) * s;
      uint32_t d[6], o[16];
#pragma unroll
      for (int i = 0; i < 6; ++i) d[i] = dword_sel(cw[min(i, NQ - 1)], j >> 1);
      decode32_wide<SM == 0>(d, j & 1, s, c0, wlane, win_w, o);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) bf[kk] = u32x4{o[4 * kk], o[4 * kk + 1], o[4 * kk + 2], o[4 * kk + 3]};
    }
  };

  f32x16 acc[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;

  const int a_frag_off = (lane & 31) * ROW + (H16 ? h * 8 : h * 32);
  auto lds_barrier = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  };

  // All of K for the first LIVE row tiles.  Every share holds at least one k-tile of each format present (the launcher
  // sees to it).  All global loads are unconditional and sit at fixed places of straight-line loop bodies: a request under a
  // condition makes the compiler wait for every outstanding load at the next use of any of them.
  auto run = [&](auto LC) {
    constexpr int LIVE = decltype(LC)::value;
    constexpr int CH = H16 ? CHUNKS : LIVE;
    using XVec = std::conditional_t<H16, u32x4_dword, u32x4>;
    auto load_a = [&](u32x4 (&dst)[CH], int s) {
      if constexpr (DEEP) {
        const int64_t off = (int64_t)group_of(s) * (kGroup * 2);
#pragma unroll
        for (int i = 0; i < CH; ++i) dst[i] = *reinterpret_cast<const XVec*>(reinterpret_cast<const char*>(xbase) + xoff[i] + off);
      } else {
        const char* base = reinterpret_cast<const char*>(xbase + (int64_t)__builtin_amdgcn_readfirstlane(group_of(s)) * kGroup);
#pragma unroll
        for (int i = 0; i < CH; ++i) {
          uint32_t off = xoff[i];
          asm volatile("" : "+v"(off));
          dst[i] = *reinterpret_cast<const XVec*>(base + off);
        }
      }
    };
    auto store_a = [&](int buf, const u32x4 (&src)[CH]) {
      uint16_t* dst = As + buf * BM * ROW;
#pragma unroll
      for (int i = 0; i < CH; ++i) {
        if constexpr (H16) {
          u32x4 o;
#pragma unroll
          for (int q = 0; q < 3; ++q) o[q] = __builtin_amdgcn_alignbit(src[i][q + 1], src[i][q], odd_word);
          o[3] = (src[i][3] >> odd_word) & 0xFFFFu;
          if (last_word[i]) o = u32x4{o[3], 0u, 0u, 0u};
          *reinterpret_cast<u32x4*>(dst + a_lds[i]) = o;
        } else {
          *reinterpret_cast<u32x4*>(dst + a_lds[0] + i * 32 * ROW) = src[i];
        }
      }
    };
    auto multiply = [&](int buf, const u32x4 (&bf)[KK]) {
      const uint16_t* Ab = As + buf * BM * ROW + a_frag_off;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
#pragma unroll
        for (int i = 0; i < LIVE; ++i) {
          const bf16x8 af = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(Ab + i * 32 * ROW + kk * (H16 ? 16 : 8)));
          acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af, __builtin_bit_cast(bf16x8, bf[kk]), acc[i], 0, 0, 0);
        }
      }
    };
    // activation chunks of step s live in register set s % D, requested D steps ahead of their use; three or four row
    // tiles leave registers for two sets only, and their steps are longer
    constexpr int D = DEEP ? (LIVE >= 3 ? 2 : 4) : (LIVE >= 3 ? 1 : 2);
    constexpr bool AHEAD = DEEP && LIVE <= 2;   // the fragments of the next step are decoded during this one
    u32x4 areg[D][CH];
    u32x4 bf[KK], bnext[KK];
    int s = 0;
    if constexpr (HAS_N) load_narrow(cn, sn, tA[kNarrow]);
    if constexpr (HAS_W) load_wide(cw, sw, tA[kWide]);
#pragma unroll
    for (int d = 0; d < D; ++d) load_a(areg[d], d);
    store_a(0, areg[0]);
    if constexpr (AHEAD) {
      if constexpr (HAS_N) decode_narrow(bf, 0);
      else decode_wide(bf, 0);
    }
    lds_barrier();
    // one step (J = s & 3): the activation tile of step s is multiplied while that of step s + 1 goes to the other LDS buffer
    auto step = [&](auto JC, auto&& decode) {
      constexpr int J = decltype(JC)::value;
      constexpr int P = J & 1;
      load_a(areg[J % D], s + D);
      if constexpr (AHEAD) {
        decode(bnext);
        multiply(P, bf);
        store_a(P ^ 1, areg[(J + 1) % D]);
#pragma unroll
        for (int k = 0; k < KK; ++k) bf[k] = bnext[k];
      } else {
        __builtin_amdgcn_sched_barrier(0);
        decode(bf);
        multiply(P, bf);
        store_a(P ^ 1, areg[(J + 1) % D]);
      }
      lds_barrier();
      ++s;
    };
    // group `now` of the held k-tile, or the one after it where fragments are decoded a step ahead
    auto narrow_step = [&](auto JC, auto NOW) {
      constexpr int now = decltype(NOW)::value;
      step(JC, [&](u32x4 (&f)[KK]) { decode_narrow(f, AHEAD ? now + 1 : now); });
    };
    auto wide_step = [&](auto JC, auto NOW) {
      constexpr int now = decltype(NOW)::value;
      step(JC, [&](u32x4 (&f)[KK]) { decode_wide(f, AHEAD ? now + 1 : now); });
    };
    auto next_narrow = [&]() {
      cn[0] = cn_next[0];
      cn[1] = cn_next[1];
      sn = sn_next;
    };
    auto next_wide = [&]() {
#pragma unroll
      for (int i = 0; i < NQ; ++i) cw[i] = cw_next[i];
      sw = sw_next;
    };
    using J0 = std::integral_constant<int, 0>;
    using J1 = std::integral_constant<int, 1>;
    using J2 = std::integral_constant<int, 2>;
    using J3 = std::integral_constant<int, 3>;
    using J4 = std::integral_constant<int, 4>;
    using J5 = std::integral_constant<int, 5>;
    using J6 = std::integral_constant<int, 6>;
    using J7 = std::integral_constant<int, 7>;
    if constexpr (HAS_N) {
      for (int t = tA[kNarrow]; t < tB[kNarrow]; ++t) {
        load_narrow(cn_next, sn_next, t + 1);
        narrow_step(J0{}, J0{});
        narrow_step(J1{}, J1{});
        narrow_step(J2{}, J2{});
        if constexpr (AHEAD) {
          step(J3{}, [&](u32x4 (&f)[KK]) {
            next_narrow();
            if constexpr (HAS_W) {
              if (t + 1 < tB[kNarrow]) decode_narrow(f, 0);
              else decode_wide(f, 0);
            } else {
              decode_narrow(f, 0);  // of the next k-tile (after the last one: a repeat, not used)
            }
          });
        } else {
          narrow_step(J3{}, J3{});
          next_narrow();
        }
      }
    }
    if constexpr (HAS_W) {
      for (int t = tA[kWide]; t < tB[kWide]; ++t) {
        load_wide(cw_next, sw_next, t + 1);
        wide_step(J0{}, J0{});
        wide_step(J1{}, J1{});
        wide_step(J2{}, J2{});
        wide_step(J3{}, J3{});
        wide_step(J0{}, J4{});
        wide_step(J1{}, J5{});
        wide_step(J2{}, J6{});
        if constexpr (AHEAD) {
          step(J3{}, [&](u32x4 (&f)[KK]) {
            next_wide();
            decode_wide(f, 0);
          });
        } else {
          wide_step(J3{}, J7{});
          next_wide();
        }
      }
    }
  };
  // a 128-row block works on the 32-row tiles that hold rows only (uniform over the workgroup)
  if constexpr (BM == 64) {
    run(std::integral_constant<int, 2>{});
  } else {
    const int live = (min(Me - m0, BM) + 31) / 32;
    if (live <= 1) run(std::integral_constant<int, 1>{});
    else if (live == 2) run(std::integral_constant<int, 2>{});
    else if (live == 3) run(std::integral_constant<int, 3>{});
    else run(std::integral_constant<int, 4>{});
  }
  if (a.wk > 1) {
    // the shorter shares keep up with the barriers of the longest one (share 0 of every kind), then the sums meet in LDS, where the
    // activation tiles were: the upper half of the shares hands its sums to the lower one until one is left
    const int longest = split;
    const int steps_most = (HAS_N ? (a.sq[kNarrow] + (longest < a.sr[kNarrow] ? 1 : 0)) * kNarrowGroupsPerTile : 0) +
                           (HAS_W ? (a.sq[kWide] + (longest < a.sr[kWide] ? 1 : 0)) * kWideGroupsPerTile : 0);
    for (int i = nsteps; i < steps_most; ++i) lds_barrier();
    for (int left = a.wk; left > 1;) {
      const int keep = (left + 1) / 2;
      float* red = reinterpret_cast<float*>(smem) + ((wk >= keep ? wk - keep : wk) * 4 + wave) * (MT * 16 * 64) + lane;
      if (wk >= keep && wk < left) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) red[(i * 16 + r) * 64] = acc[i][r];
      }
      lds_barrier();
      if (wk + keep < left) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[i][r] += red[(i * 16 + r) * 64];
      }
      left = keep;
      if (left > 1) lds_barrier();
    }
    if (wk > 0) return;
  }

  // epilogue: D[row][col], row = 8*(r/4) + 4*(lane/32) + r%4, col = lane%32
  const int n = n0 + wave * 32 + (lane & 31);
#pragma unroll
  for (int i = 0; i < MT; ++i) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int m = m0 + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
      const float val = acc[i][r];  // by value: bit-casting the element lvalue itself reads element 0
      if (m < Me && n <= a.n_last) {
        if (splits > 1) __builtin_nontemporal_store(val, &a.partial[((int64_t)split * a.M + row_off + m) * a.N + n]);
        else a.y[(int64_t)(row_off + m) * a.ldy + n] = (uint16_t)(pack_bf16_m(val, 0.f) & 0xFFFFu);
      }
    }
  }
}

typedef void (*MidKernel)(const MidArgs);
template <int FM, int SM, bool GROUPED, int BM>
static MidKernel mid_schedule(Schedule s) {
  if (s == kLean) return ccq_mid_kernel<FM, SM, GROUPED, BM, kLean>;
  if constexpr (GROUPED) {
    if (s == kDeep) return ccq_mid_kernel<FM, SM, GROUPED, BM, kDeep>;
  }
  return ccq_mid_kernel<FM, SM, GROUPED, BM, kFar>;
}
template <bool GROUPED, int SM>
static MidKernel mid_kernel(int fm, int bm, Schedule s) {
  switch (fm) {
    case 1: return bm == kMidBM ? ccq_mid_kernel<1, SM, GROUPED, kMidBM, kLean> : mid_schedule<1, SM, GROUPED, 2 * kMidBM>(s);
    case 2: return mid_schedule<2, SM, GROUPED, kMidBM>(s);
    case 3: return mid_schedule<3, SM, GROUPED, kMidBM>(s);
    default: return mid_schedule<4, SM, GROUPED, kMidBM>(s);
  }
}

// 128-row blocks are built for the narrow format.  With the wide kinds' six code entries per lane and four accumulator tiles the lean
// schedule does not fit the 168 registers of three wavefronts on a SIMD (68 to 120 bytes of scratch on wide weights and mixes); the
// deep one would fit its 256 (234 to 253).
static bool mid_has_tall_blocks(const Layout& L) { return L.tiles[kWide] == 0; }

// K shares in a workgroup, where S go across the grid and `busy` output tiles have rows.
// A wavefront takes about twice as long for a step as the SIMD needs for its instructions, so two to four of them should share
// one.  With at most one workgroup per CU they come from K shares inside the workgroup, as many as the registers allow (us with
// one / two / three / four, 0.59 of the CUs: narrow 10624 x 19200, M = 38, 71 / 56 / 51 / 50; mix 5952 x 15072, M = 99, 48 / 40 / 39);
// narrow 64-row blocks take two shares up to two workgroups per CU (15168 x 3520, M = 710, 158 / 140 / 151 / 149), the others
// one (wide 1536 x 5968, M = 487, 22 / 28).  A share has at least one k-tile of every kind.
// `far`: the activation rows lie too far apart for 32-bit offsets.
static int mid_wk(const Layout& L, int bm, bool far, int S, int64_t busy, bool* deep) {
  const int fm = L.h16 ? 4 : (L.tiles[kNarrow] > 0 ? 1 : 0) | (L.tiles[kWide] > 0 ? 2 : 0);
  const int64_t cus = device_cus();
  const bool narrow64 = fm == 1 && bm == kMidBM, one_each = busy * S <= cus, two_each = busy * S <= 2 * cus;
  *deep = !narrow64 && (two_each || far);
  int wk = one_each ? mid_waves(fm, bm, *deep) : (narrow64 && two_each ? 2 : 1);
  for (int k = 0; k < 2; ++k)
    while (wk > 1 && L.tiles[k] > 0 && L.tiles[k] < S * wk) --wk;
  return wk;
}

// E: experts (0: a dense call).
static int mid_launch(const Layout& L, MidArgs& a, int E, int bm, bool far, int S, int m_blocks, int64_t busy, void* stream) {
  const int fm = L.h16 ? 4 : (L.tiles[kNarrow] > 0 ? 1 : 0) | (L.tiles[kWide] > 0 ? 2 : 0);
  bool deep = false;
  const int wk = mid_wk(L, bm, far, S, busy, &deep);
  for (int k = 0; k < 2; ++k) {
    a.sq[k] = L.tiles[k] / (S * wk);
    a.sr[k] = L.tiles[k] % (S * wk);
  }
  a.wk = wk;
  const size_t max_steps = (size_t)(a.sq[kNarrow] + 1) * kNarrowGroupsPerTile + (size_t)(a.sq[kWide] + 1) * kWideGroupsPerTile;
  const size_t lds = std::max(wk * ((size_t)2 * bm * (fm == 4 ? kMidRowH16 : kMidRow) * 2 + (fm == 3 ? max_steps * 4 : 0)), (size_t)(wk / 2) * bm * kMidBN * 4);
  if (lds > 150 * 1024) return CCQ_ERR_UNSUPPORTED;
  const Schedule schedule = far ? kFar : (deep ? kDeep : kLean);
  const MidKernel kern = E > 0 ? (L.scale_mode == 0 ? mid_kernel<true, 0>(fm, bm, schedule) : mid_kernel<true, 1>(fm, bm, schedule))
                               : (L.scale_mode == 0 ? mid_kernel<false, 0>(fm, bm, schedule) : mid_kernel<false, 1>(fm, bm, schedule));
  if (lds > 48 * 1024 && hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) {
    (void)hipGetLastError();
    return CCQ_ERR_HIP;
  }
  // column blocks are a grid dimension: more than it holds take several launches
  const int n_blocks = (L.N + kMidBN - 1) / kMidBN;
  for (int b0 = 0; b0 < n_blocks; b0 += kMaxGridY) {
    const int64_t n0 = (int64_t)b0 * kMidBN, rt0 = n0 / kRowsPerTile;
    MidArgs p = a;
    auto advance = [](auto& ptr, int64_t by) { if (ptr) ptr += by; };
    advance(p.codes, rt0 * a.row_tile_bytes);
    advance(p.scales, rt0 * a.row_tile_scale_halfs);
    advance(p.alpha, n0);
    advance(p.beta, n0);
    advance(p.scale_super, n0);
    advance(p.y, n0);
    advance(p.partial, n0);
    p.row_tiles -= (int)rt0;
    p.n_last -= (int)n0;
    const dim3 grid((unsigned)m_blocks, (unsigned)std::min(kMaxGridY, n_blocks - b0), (unsigned)(E > 0 ? E : S));
    hipLaunchKernelGGL(kern, grid, dim3(256 * wk), lds, static_cast<hipStream_t>(stream), p);
    if (hipGetLastError() != hipSuccess) return CCQ_ERR_HIP;
  }
  return CCQ_OK;
}

// K shares for the mid-M kernel.  Every share costs a pass of fp32 partial tiles through memory (written, then
// read by the reduction): aim at one workgroup per CU, at least two k-tiles of every format per share.
int mid_splits(const Layout& L, int M) {
  const int64_t blocks = (int64_t)((M + kMidBM - 1) / kMidBM) * ((L.N + kMidBN - 1) / kMidBN);
  const int min_tiles = std::min(L.tiles[kNarrow] > 0 ? L.tiles[kNarrow] : 1 << 30, L.tiles[kWide] > 0 ? L.tiles[kWide] : 1 << 30);
  // One workgroup per CU, or two when the weights have wide-format groups and there are at least 128 blocks (K = 8192, M = 64, N = 18432,
  // 144 blocks: two shares against one, which then runs two shares of its own: wide 40 against 50 us, hybrid word 50 against
  // 64 us, mix 52 against 47 us; at K = 4096 28 / 28, 33 / 35 and 27 / 27).  Beyond two thirds of the CUs mid_shares takes one all the same.  A narrow block gains nothing from
  // a second workgroup on its CU.
  const int64_t cus = device_cus();
  const int64_t target = (L.tiles[kWide] > 0 && 2 * blocks >= cus) ? 2 * cus : cus;
  int64_t s = std::max<int64_t>(1, target / std::max<int64_t>(1, blocks));
  s = std::min<int64_t>(s, 8);
  s = std::min<int64_t>(s, std::max(1, min_tiles / 2));
  return (int)s;
}

// How many of the `most` shares that mid_splits allows (and the workspace holds) a call takes: with more than two thirds of the
// CUs busy the shares inside a workgroup do without a pass over partial tiles (wide 4608 x 8160, M = 188, 192 blocks: two
// across the grid 35, three inside 32 us; 6400 x 3856, M = 299, 155 blocks: three across 38, three inside 44).
int mid_shares(const Layout& L, int M, int most) {
  const int64_t blocks = (int64_t)((M + kMidBM - 1) / kMidBM) * ((L.N + kMidBN - 1) / kMidBN);
  return blocks * 3 > 2 * (int64_t)device_cus() ? 1 : most;
}

// Rows of a block of a dense call.  128-row blocks (narrow): where 64-row ones are more than one to a CU and 128-row ones are not, or where
// there are more than two 64-row ones (us with 64 / 128 rows: 4480 x 24294, M = 73, 48 / 35; 5120 x 6064, M = 361, 54 / 48; 2112 x 22144, M = 714,
// 107 / 98; 896 x 18642, M = 139, 1.7 and 1.1 to a CU, 17 / 24; 5120 x 1656, M = 784, 0.7 and 0.4 to a CU, 32 / 47).
static int mid_dense_rows(const Layout& L, int M, int S, bool far) {
  const int64_t cus = device_cus(), n_blocks = (L.N + kMidBN - 1) / kMidBN;
  const int64_t wg64 = (int64_t)((M + kMidBM - 1) / kMidBM) * n_blocks, wg128 = (int64_t)((M + 2 * kMidBM - 1) / (2 * kMidBM)) * n_blocks;
  return mid_has_tall_blocks(L) && (far || (S == 1 && wg64 > cus && (wg128 <= cus || wg64 > 2 * cus))) ? 2 * kMidBM : kMidBM;
}

// What a dense call takes here, by a fit to 832 random calls of 65 to 4096 rows (nine in ten within 13 %): per step of K the longer of a wavefront's
// own time and the time of those that share its SIMD, a start, and the pass over the partial tiles.
double mid_time(const Layout& L, int M) {
  struct Rates {
    double alone, shared, start;
  };
  constexpr Rates narrow64 = {0.35, 0.28, 6.6}, narrow128 = {0.93, 0.50, 8.4}, wide = {0.41, 0.34, 6.3}, mix = {0.40, 0.34, 6.4}, h16 = {0.28, 0.46, 6.9};
  const int S = mid_shares(L, M, mid_splits(L, M)), bm = mid_dense_rows(L, M, S, false);
  const int64_t cus = device_cus(), blocks = (int64_t)((M + bm - 1) / bm) * ((L.N + kMidBN - 1) / kMidBN) * S;
  bool deep = false;
  const int wk = mid_wk(L, bm, false, S, blocks / S, &deep);
  const Rates r = L.h16 ? h16 : (L.tiles[kWide] == 0 ? (bm == kMidBM ? narrow64 : narrow128) : (L.tiles[kNarrow] == 0 ? wide : mix));
  auto steps = [&](int k, int groups) { return (L.tiles[k] + S * wk - 1) / (S * wk) * groups; };
  const double waves = blocks <= 2 * cus ? (double)((blocks + cus - 1) / cus * wk) : ((double)blocks / (double)cus + 0.6) * wk;
  double t = r.start + (steps(kNarrow, kNarrowGroupsPerTile) + steps(kWide, kWideGroupsPerTile)) * std::max(r.alone, r.shared * waves);
  if (S > 1) t += 2.4 + (double)S * M * L.N * 8.0 / 9.0e6;
  return t;
}

int launch_mid(const ccq_weight* w, const Layout& L, const void* x, int M, int64_t ldx, void* y, int64_t ldy, float* partial, int S,
               void* stream) {
  MidArgs a;
  a.codes = static_cast<const uint8_t*>(w->codes);
  a.scales = static_cast<const uint16_t*>(w->scales);
  a.alpha = w->code_alpha;
  a.beta = w->code_beta;
  a.meta = static_cast<const int32_t*>(w->meta);
  a.scale_super = static_cast<const uint16_t*>(w->scale_super);
  a.x = static_cast<const uint16_t*>(x);
  a.y = static_cast<uint16_t*>(y);
  a.partial = partial;
  a.ldx = ldx;
  a.ldy = ldy;
  a.row_tile_bytes = L.row_tile_bytes;
  a.row_tile_scale_halfs = L.row_tile_scale_halfs;
  a.M = M;
  a.N = L.Npad;
  a.g_last = L.G - 1;
  a.n_last = L.N - 1;
  a.row_tiles = L.row_tiles;
  const int n_blocks = (L.N + kMidBN - 1) / kMidBN;
  const bool far = (2 * kMidBM - 1) * ldx * 2 + 2 * kGroup > (int64_t)1 << 32;   // (a 64-row narrow block has the lean schedule only)
  const int bm = mid_dense_rows(L, M, S, far);
  const int m_blocks = (M + bm - 1) / bm;
  a.tiles[0] = L.tiles[0];
  a.tiles[1] = L.tiles[1];
  a.groups_narrow = L.pgroups[kNarrow];
  a.sorted_rows = nullptr;
  a.expert_offsets = nullptr;
  a.codes_stride = a.scales_stride = a.ab_stride = 0;
  for (int k = 0; k < 2; ++k) a.zp[k] = L.zp[k];
  return mid_launch(L, a, 0, bm, far, S, m_blocks, (int64_t)m_blocks * n_blocks, stream);
}

// Grouped GEMM with many rows per expert: the same kernel over
// (row block of the expert, column block, expert); blocks past an expert's rows return at once. K is not cut (no workspace).
// 128-row blocks as soon as an expert has more rows than a 64-row block holds.
static int mid_grouped_block(const Layout& L, bool far, const GroupedRows& rows) { return mid_has_tall_blocks(L) && (far || rows.most > kMidBM) ? 2 * kMidBM : kMidBM; }

// Where many blocks of the grid are past their expert's rows (one expert has most of them), the first blocks of the others, a
// row block count apart, would with an even count share a few of the chip's eight dies (narrow, 8 experts of 7168 x 512, one with
// 2000 rows, seven with 4: sixteen row blocks 93, seventeen 62 us).
static int mid_grouped_row_blocks(int bm, int E, const GroupedRows& rows) {
  const int m = (rows.most + bm - 1) / bm;
  return m % 2 == 0 && 8 * (bm == kMidBM ? rows.blocks64 : rows.blocks128) < (int64_t)7 * m * E ? m + 1 : m;
}

// What a grouped call takes here, as mid_time, by a fit to 565 random calls (nine in ten within 19 %).
double mid_grouped_time(const Layout& L, int E, const GroupedRows& rows) {
  struct Rates {
    double alone, shared;
  };
  constexpr Rates narrow64 = {0.35, 0.33}, narrow128 = {0.85, 0.52}, wide = {0.67, 0.39}, mix = {0.44, 0.39}, h16 = {0.36, 0.54};
  const int bm = mid_grouped_block(L, false, rows);
  const int64_t cus = device_cus(), n_blocks = (L.N + kMidBN - 1) / kMidBN, blocks = n_blocks * (bm == kMidBM ? rows.blocks64 : rows.blocks128);
  const int64_t grid = n_blocks * mid_grouped_row_blocks(bm, E, rows) * E;
  bool deep = false;
  const int wk = mid_wk(L, bm, false, 1, blocks, &deep);
  const Rates r = L.h16 ? h16 : (L.tiles[kWide] == 0 ? (bm == kMidBM ? narrow64 : narrow128) : (L.tiles[kNarrow] == 0 ? wide : mix));
  auto steps = [&](int k, int groups) { return (L.tiles[k] + wk - 1) / wk * groups; };
  const double waves = blocks <= 2 * cus ? (double)((blocks + cus - 1) / cus * wk) : ((double)blocks / (double)cus + 0.52) * wk;
  return 5.6 + (steps(kNarrow, kNarrowGroupsPerTile) + steps(kWide, kWideGroupsPerTile)) * std::max(r.alone, r.shared * waves) + 0.27e-3 * (double)(grid - blocks);
}

int launch_mid_grouped(const ccq_weight* w0, const Layout& L, int E, int64_t codes_stride, int64_t scales_stride, int64_t ab_stride, const void* x,
                       int64_t ldx, const int32_t* sorted_rows, int T, int P, const int32_t* expert_offsets, const GroupedRows& rows, void* y, int64_t ldy,
                       void* stream) {
  if (E < 1 || E > 65535 || rows.most < 1) return CCQ_ERR_UNSUPPORTED;
  MidArgs a;
  a.codes = static_cast<const uint8_t*>(w0->codes);
  a.scales = static_cast<const uint16_t*>(w0->scales);
  a.alpha = w0->code_alpha;
  a.beta = w0->code_beta;
  a.meta = static_cast<const int32_t*>(w0->meta);
  a.scale_super = static_cast<const uint16_t*>(w0->scale_super);
  a.x = static_cast<const uint16_t*>(x);
  a.y = static_cast<uint16_t*>(y);
  a.partial = nullptr;
  a.ldx = ldx;
  a.ldy = ldy;
  a.row_tile_bytes = L.row_tile_bytes;
  a.row_tile_scale_halfs = L.row_tile_scale_halfs;
  a.M = P;
  a.N = L.Npad;
  a.g_last = L.G - 1;
  a.n_last = L.N - 1;
  a.row_tiles = L.row_tiles;
  const bool far = (int64_t)T * ldx * 2 > (int64_t)1 << 32;
  const int bm = mid_grouped_block(L, far, rows);
  const int64_t row_blocks = bm == kMidBM ? rows.blocks64 : rows.blocks128;
  const int m_blocks = mid_grouped_row_blocks(bm, E, rows);
  a.tiles[0] = L.tiles[0];
  a.tiles[1] = L.tiles[1];
  a.groups_narrow = L.pgroups[kNarrow];
  for (int k = 0; k < 2; ++k) a.zp[k] = L.zp[k];
  a.sorted_rows = sorted_rows;
  a.expert_offsets = expert_offsets;
  a.codes_stride = codes_stride;
  a.scales_stride = scales_stride;
  a.ab_stride = ab_stride;
  const int n_blocks = (L.N + kMidBN - 1) / kMidBN;
  return mid_launch(L, a, E, bm, far, 1, m_blocks, n_blocks * row_blocks, stream);
}

}  // namespace ccq

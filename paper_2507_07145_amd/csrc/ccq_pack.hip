// Canonical (paper order) packed weights to device order, on the GPU: the byte permutation of ccq_pack_codes,
// ccq_pack_scales and ccq_pack_scales4, with canonical and device-order arrays both in device memory.
//
// The permutation is a gather of 2- and 4-byte pieces.  On a host core it costs a few instructions per stored byte; on the
// GPU it is one pass over memory that vanishes behind the upload.  One thread per 16-byte chunk of the code stream
// (a lane's entry of a k-tile, so stores are whole and consecutive; the four quarters of a row read one contiguous run),
// then one per (k-tile, row) entry of the scales.  Padded rows and groups are written as zeros: nothing has to be
// cleared first.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ccq_internal.h"

namespace ccq {

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

struct PackArgs {
  const uint8_t* codes;    // canonical, [E][N][row_bytes]
  const uint8_t* scales;   // canonical fp16 [E][N][G], or the fields uint8 [E][N][field_bytes]
  const int32_t* meta;     // packed group -> original group (group maps only)
  uint8_t* codes_out;
  uint8_t* scales_out;
  int64_t code_bytes, scale_bytes;         // of one expert in device order
  int64_t src_code_bytes, src_scale_bytes; // of one expert in canonical order
  int64_t row_bytes, field_bytes;
  int64_t code_items, items;               // 16-byte chunks of the codes; those and the scale entries
  int32_t N, G, chunks, units;             // chunks and scale entries of one row tile
  int32_t groups[2], pgroups_narrow, tiles_narrow;
  int64_t row_tile_scale_halfs;
  int32_t scale_mode;
};

// Canonical group of packed group p of one kind, p below the number of real ones.
template <bool META>
__device__ __forceinline__ int pack_group(const PackArgs& a, int kind, int p) {
  if constexpr (META) return a.meta[(kind == kWide ? a.pgroups_narrow : 0) + p];
  return p;
}

// META: the weights have a group map.  H16: the hybrid word in place of the wide format.
template <bool META, bool H16>
__global__ void __launch_bounds__(256) ccq_pack_kernel(const PackArgs a) {
  const int64_t item = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (item >= a.items) return;
  const int64_t e = blockIdx.y;
  if (item < a.code_items) {
    const int rt = (int)(item / a.chunks), within = (int)(item % a.chunks);
    u32x4 out = {0u, 0u, 0u, 0u};
    if (within < a.tiles_narrow * 64) {
      const int kt = within >> 6, lane = within & 63, kq = lane >> 4, n = rt * kRowsPerTile + (lane & 15);
      if (n < a.N) {
        const uint8_t* row = a.codes + e * a.src_code_bytes + n * a.row_bytes;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int p = kt * kNarrowGroupsPerTile + j;
          if (p < a.groups[kNarrow]) {
            const int g = pack_group<META>(a, kNarrow, p);
            // of the g groups before this one p are narrow
            const uint8_t* src = row + (int64_t)p * kNarrowGroupBytes + (int64_t)(g - p) * kWideGroupBytes + 4 * kq;
            if constexpr (META) {   // wide groups before it leave 2-byte alignment
              const uint16_t* s2 = reinterpret_cast<const uint16_t*>(src);
              out[j] = (uint32_t)s2[0] | ((uint32_t)s2[1] << 16);
            } else {
              out[j] = *reinterpret_cast<const uint32_t*>(src);
            }
          }
        }
      }
    } else {
      constexpr int tile_chunks = (H16 ? kH16TileBytes : kWideTileBytes) / 16;
      const int w = within - a.tiles_narrow * 64;
      const int kt = w / tile_chunks, rem = w % tile_chunks, t = rem >> 6, lane = rem & 63, kq = lane >> 4;
      const int n = rt * kRowsPerTile + (lane & 15);
      if (n < a.N) {
        const uint8_t* row = a.codes + e * a.src_code_bytes + n * a.row_bytes;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int p = kt * kWideGroupsPerTile + j;
          if (p < a.groups[kWide]) {
            const int g = pack_group<META>(a, kWide, p);
            const uint8_t* src = H16 ? row + (int64_t)p * kH16GroupBytes + 2 * (4 * t + kq)
                                     : row + (int64_t)p * kWideGroupBytes + (int64_t)(g - p) * kNarrowGroupBytes + 6 * kq + 2 * t;
            out[j >> 1] |= (uint32_t)*reinterpret_cast<const uint16_t*>(src) << (16 * (j & 1));
          }
        }
      }
    }
    *reinterpret_cast<u32x4*>(a.codes_out + e * a.code_bytes + item * 16) = out;
    return;
  }
  const int64_t s = item - a.code_items;
  const int rt = (int)(s / a.units), within = (int)(s % a.units), tile = within >> 4, r = within & 15, n = rt * kRowsPerTile + r;
  uint16_t* tile_row = reinterpret_cast<uint16_t*>(a.scales_out + e * a.scale_bytes) + rt * a.row_tile_scale_halfs;
  if (a.scale_mode == 1) {   // narrow groups only: four fields of a k-tile in two bytes
    uint32_t v = 0;
    if (n < a.N) {
      const uint8_t* src = a.scales + e * a.src_scale_bytes + n * a.field_bytes;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int p = 4 * tile + j;
        if (p < a.groups[kNarrow]) v |= (((uint32_t)src[p >> 1] >> (4 * (p & 1))) & 0xFu) << (4 * j);
      }
    }
    tile_row[(int64_t)tile * kNarrowTileScaleHalfs4 + r] = (uint16_t)v;
    return;
  }
  const bool wide = tile >= a.tiles_narrow;
  const int kind = wide ? kWide : kNarrow, kt = wide ? tile - a.tiles_narrow : tile, per = wide ? kWideGroupsPerTile : kNarrowGroupsPerTile;
  u32x4 out = {0u, 0u, 0u, 0u};
  if (n < a.N) {
    const uint16_t* src = reinterpret_cast<const uint16_t*>(a.scales + e * a.src_scale_bytes) + (int64_t)n * a.G;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int p = kt * per + j;
      if (j < per && p < a.groups[kind]) out[j >> 1] |= (uint32_t)src[pack_group<META>(a, kind, p)] << (16 * (j & 1));
    }
  }
  if (wide) *reinterpret_cast<u32x4*>(tile_row + (int64_t)a.tiles_narrow * kNarrowTileScaleHalfs + kt * kWideTileScaleHalfs + r * 8) = out;
  else *reinterpret_cast<uint2*>(tile_row + (int64_t)kt * kNarrowTileScaleHalfs + r * 4) = uint2{out.x, out.y};
}

int launch_pack(const Layout& L, int E, const void* codes, const void* scales, const int32_t* meta, void* codes_out, void* scales_out, void* stream) {
  PackArgs a;
  a.meta = meta;
  a.row_bytes = L.h16 ? (int64_t)L.G * kH16GroupBytes : (int64_t)L.groups[kNarrow] * kNarrowGroupBytes + (int64_t)L.groups[kWide] * kWideGroupBytes;
  a.field_bytes = (L.groups[kNarrow] + 1) / 2;
  a.src_code_bytes = a.row_bytes * L.N;
  a.src_scale_bytes = L.scale_mode == 0 ? (int64_t)L.N * L.G * 2 : a.field_bytes * L.N;
  a.code_bytes = L.row_tile_bytes * L.row_tiles;
  a.scale_bytes = L.row_tile_scale_halfs * L.row_tiles * 2;
  a.chunks = (int32_t)(L.row_tile_bytes / 16);
  a.units = 16 * (L.scale_mode == 0 ? L.tiles[kNarrow] + L.tiles[kWide] : L.tiles[kNarrow]);
  a.code_items = (int64_t)a.chunks * L.row_tiles;
  a.items = a.code_items + (int64_t)a.units * L.row_tiles;
  a.N = L.N;
  a.G = L.G;
  for (int k = 0; k < 2; ++k) a.groups[k] = L.groups[k];
  a.pgroups_narrow = L.pgroups[kNarrow];
  a.tiles_narrow = L.tiles[kNarrow];
  a.row_tile_scale_halfs = L.row_tile_scale_halfs;
  a.scale_mode = L.scale_mode;
  const int64_t blocks = (a.items + 255) / 256;
  if (blocks > 0x7FFFFFFF) return CCQ_ERR_UNSUPPORTED;
  for (int e0 = 0; e0 < E; e0 += 65535) {   // grid.y holds at most 65535 experts
    a.codes = static_cast<const uint8_t*>(codes) + e0 * a.src_code_bytes;
    a.scales = static_cast<const uint8_t*>(scales) + e0 * a.src_scale_bytes;
    a.codes_out = static_cast<uint8_t*>(codes_out) + e0 * a.code_bytes;
    a.scales_out = static_cast<uint8_t*>(scales_out) + e0 * a.scale_bytes;
    const dim3 grid((unsigned)blocks, (unsigned)std::min(65535, E - e0));
    if (L.has_map) hipLaunchKernelGGL((ccq_pack_kernel<true, false>), grid, dim3(256), 0, static_cast<hipStream_t>(stream), a);
    else if (L.h16) hipLaunchKernelGGL((ccq_pack_kernel<false, true>), grid, dim3(256), 0, static_cast<hipStream_t>(stream), a);
    else hipLaunchKernelGGL((ccq_pack_kernel<false, false>), grid, dim3(256), 0, static_cast<hipStream_t>(stream), a);
    if (hipGetLastError() != hipSuccess) return CCQ_ERR_HIP;
  }
  return CCQ_OK;
}

}  // namespace ccq

// Launches of the prompt kernel (ccq_block.h): which blocks and K shares a call takes, and whether it takes them at all.
#include <algorithm>

#include "ccq_block.h"

namespace ccq {

// Estimated times in microseconds, fitted to 10800 launches of 832 random calls (65 to 4096 rows, K 512 to 28672, N 1000 to 28672, all
// formats; nine in ten within 8 %).  Per step of K (a 64-weight group) a block alone takes `alone` + `alone_row` mt, and with all CUs at work, where
// the clock falls with the power, the chip takes `all` + `all_row` mt for a block on every CU; 128-row blocks run one or two to a CU.
struct BlockRates {
  double alone, alone_row, all, all_row, one128, two128, all128;
};
constexpr BlockRates kRatesNarrow = {0.08, 0.13, 0.12, 0.178, 0.66, 1.27, 1.74};
constexpr BlockRates kRatesWide = {0.57, 0.08, 0.42, 0.151, 0.86, 1.54, 1.99};
constexpr BlockRates kRatesH16 = {0.64, 0.08, 0.47, 0.151, 0.93, 1.70, 2.02};
constexpr double kCallTime = 9.1, kSecondPart = 5.4;      // of the first and the second part of a call
constexpr double kRoundTime = -3.0, kRoundTimeRow = 0.80; // more per round of blocks: start, and the outputs
constexpr double kPartialRate = 9.9e6;                    // bytes of partial tiles, written and read, per microsecond
constexpr int64_t kPartialRow = (8 << 20) / 32;           // bytes of partial tiles per row at most: the fit has no more

static double part_time(const Layout& L, int M, const BlockPart& p) {
  const double qn = L.tiles[kNarrow] ? 4.0 * ((L.tiles[kNarrow] + p.S - 1) / p.S) : 0.0, qw = L.tiles[kWide] ? 4.0 * ((2 * L.tiles[kWide] + p.S - 1) / p.S) : 0.0;
  const BlockRates &n = kRatesNarrow, &w = L.h16 ? kRatesH16 : kRatesWide;
  auto steps = [&](double BlockRates::*rate) { return qn * (n.*rate) + qw * (w.*rate); };   // all steps of a block
  const int64_t cus = device_cus();
  const int64_t blocks = (int64_t)((M + 32 * p.mt - 1) / (32 * p.mt)) * ((p.n_count + kBlockCols - 1) / kBlockCols) * p.S;
  double t = 0.0;
  if (p.mt > 4) {
    const double alone = steps(&BlockRates::alone) + steps(&BlockRates::alone_row) * p.mt, all = steps(&BlockRates::all) + steps(&BlockRates::all_row) * p.mt;
    const int64_t full = blocks / cus, rest = blocks % cus;
    t = (double)full * std::max(alone, all) + (rest ? std::max(alone, all * (double)rest / (double)cus) : 0.0);
    t += (double)(full + (rest ? 1 : 0)) * (kRoundTime + kRoundTimeRow * p.mt);
  } else {
    const double one = steps(&BlockRates::one128), two = steps(&BlockRates::two128), all = steps(&BlockRates::all128);
    const int64_t full = blocks / (2 * cus), rest = blocks % (2 * cus);
    t = (double)full * std::max(two, all) + (rest ? std::max(rest <= cus ? one : two, all * (double)rest / (double)(2 * cus)) : 0.0);
    t += ((double)full + (rest == 0 ? 0.0 : (rest <= cus ? 0.5 : 1.0))) * (kRoundTime + kRoundTimeRow * p.mt);
  }
  if (p.S > 1) t += (double)p.S * M * p.n_count * 8.0 / kPartialRate;
  return t;
}

static int64_t part_workspace(int M, const BlockPart& p) {
  return p.S > 1 ? (int64_t)p.S * M * ((p.n_count + kRowsPerTile - 1) / kRowsPerTile * kRowsPerTile) * 4 : 0;
}

// The best blocks and shares for a range of columns, with `bytes` of workspace.
static double best_part(const Layout& L, int M, int n_first, int n_count, int64_t bytes, BlockPart* best) {
  const int64_t cus = device_cus();
  const int b = (M + 255) / 256;   // row blocks, and their heights without rows to spare
  const int heights[4] = {4, std::max(5, (M + 32 * b - 1) / (32 * b)), std::max(5, (M + 32 * b + 31) / (32 * (b + 1))), 8};
  double t_best = 1e30;
  for (int h = 0; h < (M > 128 ? 4 : 1); ++h) {
    for (int S : {1, 2, 3, 4, 5, 6, 8}) {
      BlockPart p;
      p.n_first = n_first;
      p.n_count = n_count;
      p.mt = heights[h];
      p.S = S;
      if (S > 1) {
        const int64_t blocks = (int64_t)((M + 32 * p.mt - 1) / (32 * p.mt)) * ((n_count + kBlockCols - 1) / kBlockCols);
        // more shares only while there are CUs for them (128-row blocks: two to a CU); every share has quads of every kind
        if (blocks * S > (p.mt > 4 ? cus : 2 * cus) + 16) break;
        if ((L.tiles[kNarrow] > 0 && L.tiles[kNarrow] < S) || (L.tiles[kWide] > 0 && 2 * L.tiles[kWide] < S)) break;
        if (part_workspace(M, p) > bytes || part_workspace(1, p) > kPartialRow) break;
      }
      const double t = part_time(L, M, p);
      if (t < t_best) {
        t_best = t;
        *best = p;
      }
    }
  }
  return t_best;
}

// What a plan's time may be: the 64-row kernel is taken where it is as good, for small products and short K.  (1032 calls of 65 to 4096 rows against the
// kernels that served them before: 0.82 of the time in the geometric mean, three more than 3 % slower, the worst, hybrid word 1280 x 937, 1273 rows, 22.7 / 20.3 us;
// with the 64-row kernel's time as it is, 25 of the 832 that the times were fitted to.)
static double worth_it(const Layout& L, int M) { return 0.95 * mid_time(L, M) - 1.5; }

// All columns alike, or as many as fill the CUs a whole number of times in tall blocks and the rest, which would leave CUs idle, in whatever
// is best for them (narrow 7168 x 18432, M = 2048, 576 blocks of 256 x 256: 477 us, in three rounds; 512 of them and 128 blocks of
// 128 x 256 in two shares: 424 us).
static BlockPlan make_plan(const Layout& L, int M, int64_t bytes) {
  BlockPlan plan;
  plan.parts = 1;
  plan.time = kCallTime + best_part(L, M, 0, L.N, bytes, &plan.part[0]);
  const int64_t cus = device_cus();
  const int b = (M + 255) / 256, mt = std::max(5, (M + 32 * b - 1) / (32 * b));
  const int64_t row_blocks = (M + 32 * mt - 1) / (32 * mt), n_blocks = (L.N + kBlockCols - 1) / kBlockCols, rounds = row_blocks * n_blocks / cus;
  const int64_t n_full = row_blocks > 0 ? cus * rounds / row_blocks : 0;
  if (M > 128 && n_full > 0 && n_full < n_blocks) {
    BlockPart p[2];
    p[0].n_count = (int)n_full * kBlockCols;
    p[0].mt = mt;
    const double t = kCallTime + kSecondPart + part_time(L, M, p[0]) + best_part(L, M, p[0].n_count, L.N - p[0].n_count, bytes, &p[1]);
    if (t < plan.time) {
      plan.parts = 2;
      plan.time = t;
      plan.part[0] = p[0];
      plan.part[1] = p[1];
    }
  }
  return plan;
}

int64_t block_workspace(int M, const BlockPlan& plan) {
  int64_t need = 0;
  for (int i = 0; i < plan.parts; ++i) need = std::max(need, part_workspace(M, plan.part[i]));
  return need;
}

// With less workspace than a plan asks for, fewer shares are looked at, down to none, and the 64-row kernel takes over where that is the faster: by these
// estimates a call is never slower with more of it.  (One in passes over the rows, each of which decodes all weights again, was up to seven times as slow.)
BlockPlan block_plan(const Layout& L, int M, int64_t bytes) {
  if (M <= 64 || L.K < 512) return BlockPlan{};
  // a call asks several times: the last answers of this thread, functions of these numbers, with all of the workspace and with less
  struct Key {
    int tn = -1, tw = -1, h16 = -1, K = -1, N = -1, M = -1, cus = -1;
    int64_t bytes = -1;
    bool operator==(const Key& o) const {
      return tn == o.tn && tw == o.tw && h16 == o.h16 && K == o.K && N == o.N && M == o.M && cus == o.cus && bytes == o.bytes;
    }
  };
  static thread_local Key last[2];
  static thread_local BlockPlan plan[2];
  Key key{L.tiles[kNarrow], L.tiles[kWide], L.h16 ? 1 : 0, L.K, L.N, M, device_cus(), kPromptPartialMost};
  for (int i = 0; i < 2; ++i) {
    if (!(key == last[i])) {
      plan[i] = make_plan(L, M, key.bytes);
      if (plan[i].time > worth_it(L, M)) plan[i].parts = 0;
      last[i] = key;
    }
    if (block_workspace(M, plan[i]) <= bytes) return plan[i];
    key.bytes = bytes;
  }
  return BlockPlan{};
}

// Of the row counts of one 32-row tile the first one's plan has the most partial tiles per row: a plan's time grows with the rows by its partial tiles
// alone, so those with more of them drop out as the rows grow.  For the same reason, as the 64-row kernel's time grows evenly too, a plan that is not worth it for the
// first and the last of them is so for none.  (What column range the tiles are of moves the padding to whole row tiles by eight shares' at most.)
// Past the rows looked at no K is cut: 128-row blocks (two to a CU), and taller ones, of a single column block fill the chip.
int64_t block_workspace_most(const Layout& L, int M_max) {
  if (M_max <= 64 || L.K < 512) return 0;
  int64_t need = 0;
  const int64_t last = std::min<int64_t>(M_max, ((int64_t)device_cus() + 16) * 128);
  for (int64_t m = 65; m <= last; m += 32) {
    const int first = (int)m, end = (int)std::min(m + 31, last);
    const BlockPlan plan = make_plan(L, first, kPromptPartialMost);
    const int64_t bytes = block_workspace(end, plan);
    if (bytes <= need || (plan.time > worth_it(L, first) && make_plan(L, end, kPromptPartialMost).time > worth_it(L, end))) continue;
    need = std::min(bytes + (int64_t)8 * end * (L.Npad - L.N) * 4, kPromptPartialMost);
  }
  return need;
}

static BlockArgs block_args(const ccq_weight* w, const Layout& L, const void* x, int M, int64_t ldx, void* y, int64_t ldy, float* partial, const BlockPart& p) {
  const int64_t rt0 = p.n_first / kRowsPerTile;
  BlockArgs a;
  a.sorted_rows = a.expert_offsets = nullptr;
  a.codes_stride = a.scales_stride = a.ab_stride = 0;
  a.codes = static_cast<const uint8_t*>(w->codes) + rt0 * L.row_tile_bytes;
  a.scales = w->scales ? static_cast<const uint16_t*>(w->scales) + rt0 * L.row_tile_scale_halfs : nullptr;
  a.alpha = w->code_alpha ? w->code_alpha + p.n_first : nullptr;
  a.beta = w->code_beta ? w->code_beta + p.n_first : nullptr;
  a.meta = static_cast<const int32_t*>(w->meta);
  a.scale_super = w->scale_super ? static_cast<const uint16_t*>(w->scale_super) + p.n_first : nullptr;
  a.x = static_cast<const uint16_t*>(x);
  a.y = static_cast<uint16_t*>(y) + p.n_first;
  a.partial = partial;
  a.ldx = ldx;
  a.ldy = ldy;
  a.row_tile_bytes = L.row_tile_bytes;
  a.row_tile_scale_halfs = L.row_tile_scale_halfs;
  a.M = M;
  a.N = p.n_count;
  a.row_tiles = (p.n_count + kRowsPerTile - 1) / kRowsPerTile;
  a.Npad = a.row_tiles * kRowsPerTile;
  a.quads[kNarrow] = L.tiles[kNarrow];
  a.quads[kWide] = 2 * L.tiles[kWide];
  a.g_last = L.G - 1;
  for (int k = 0; k < 2; ++k) {
    a.sq[k] = a.quads[k] / p.S;
    a.sr[k] = a.quads[k] % p.S;
    a.zp[k] = L.zp[k];
    for (int i = 0; i < 3; ++i) a.off[k][i] = -((k == kNarrow ? kNarrowBases[i] : kWideBases[i]) + L.zp[k]);
  }
  return a;
}

static int launch_part(const ccq_weight* w, const Layout& L, const void* x, int M, int64_t ldx, void* y, int64_t ldy, float* partial, const BlockPart& p,
                       void* stream) {
  const BlockArgs a = block_args(w, L, x, M, ldx, y, ldy, partial, p);
  const int bm = 32 * p.mt;
  const size_t lds = kBlockLds0 + (size_t)2 * bm * kGroup * 2;
  const BlockKernel kern = L.h16 ? block_kernel_h16(L.scale_mode, p.mt)
                                 : (L.tiles[kWide] == 0 ? block_kernel_narrow(L.scale_mode, p.mt)
                                                        : (L.tiles[kNarrow] == 0 ? block_kernel_wide(L.scale_mode, p.mt) : block_kernel_mix(L.scale_mode, p.mt)));
  if (lds > 48 * 1024 && hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) {
    (void)hipGetLastError();
    return CCQ_ERR_HIP;
  }
  const dim3 grid((unsigned)((M + bm - 1) / bm), (unsigned)((p.n_count + kBlockCols - 1) / kBlockCols), (unsigned)p.S);
  hipLaunchKernelGGL(kern, grid, dim3(256), lds, static_cast<hipStream_t>(stream), a);
  return hipGetLastError() == hipSuccess ? CCQ_OK : CCQ_ERR_HIP;
}

int launch_block(const ccq_weight* w, const Layout& L, const void* x, int M, int64_t ldx, void* y, int64_t ldy, void* workspace, const BlockPlan& plan,
                 void* stream) {
  for (int i = 0; i < plan.parts; ++i) {
    const BlockPart& p = plan.part[i];
    // lane offsets have 32 bits; column blocks are a grid dimension
    if ((int64_t)32 * p.mt * ldx * 2 >= (int64_t)1 << 32 || 4 * L.row_tile_bytes >= (int64_t)1 << 31 || (p.n_count + kBlockCols - 1) / kBlockCols > 65535)
      return CCQ_ERR_UNSUPPORTED;
  }
  for (int i = 0; i < plan.parts; ++i) {
    const BlockPart& p = plan.part[i];
    float* partial = p.S > 1 ? static_cast<float*>(workspace) : nullptr;
    int rc = launch_part(w, L, x, M, ldx, y, ldy, partial, p, stream);
    if (rc == CCQ_OK && p.S > 1)
      rc = launch_reduce_splits(partial, static_cast<uint16_t*>(y) + p.n_first, ldy, M, p.n_count, (p.n_count + kRowsPerTile - 1) / kRowsPerTile * kRowsPerTile,
                                p.S, stream);
    if (rc != CCQ_OK) return rc;
  }
  return CCQ_OK;
}

// Grouped calls: blocks of up to 128 rows, and K is not cut.  Times by a fit to 565 random calls (4 to 160 experts, the fullest with 33 to 4000 rows; nine in
// ten within 11 %): per step of K `alone` + `alone_row` times the 32-row tiles of the tallest block, and what the chip takes for all blocks, two to a CU;
// the shorter of the two does not quite hide behind the longer.  Where blocks share CUs, which they do before each CU has one if the grid
// has blocks without rows between them, a block takes 1.4 times as long.
struct GroupedRates {
  double alone, alone_row, all, all_row;
};
constexpr GroupedRates kGroupedNarrow = {0.30, 0.087, 0.47, 0.38}, kGroupedWide = {0.48, 0.088, 0.93, 0.32}, kGroupedH16 = {0.49, 0.105, 1.02, 0.30};

static int grouped_row_blocks(int E, const GroupedRows& r) {
  const int m = (r.most + 127) / 128;
  // An even count of row blocks with many of them without rows leaves the others on a few of the chip's eight dies: an odd one spreads them.
  return m % 2 == 0 && 8 * r.blocks128 < (int64_t)7 * m * E ? m + 1 : m;
}

double block_grouped_time(const Layout& L, int E, const GroupedRows& r) {
  const double cus = device_cus(), n_blocks = (L.N + kBlockCols - 1) / kBlockCols;
  const double blocks = n_blocks * (double)r.blocks128, tiles = n_blocks * (double)r.tiles32, grid = n_blocks * grouped_row_blocks(E, r) * E;
  const double top = std::min(4, (r.most + 31) / 32);
  const GroupedRates &n = kGroupedNarrow, &w = L.h16 ? kGroupedH16 : kGroupedWide;
  auto steps = [&](double GroupedRates::*rate) {
    return (double)(L.tiles[kNarrow] * kNarrowGroupsPerTile) * (n.*rate) + (double)(L.tiles[kWide] * kWideGroupsPerTile) * (w.*rate);
  };
  double alone = steps(&GroupedRates::alone) + steps(&GroupedRates::alone_row) * top;
  if (blocks > cus || (blocks > cus / 2 && grid > 1.1 * blocks)) alone *= 1.42;
  const double all = (steps(&GroupedRates::all) * blocks + steps(&GroupedRates::all_row) * tiles) / (2 * cus);
  return 6.6 + std::max(alone, all) + 0.27 * std::min(alone, all) + 4.1 * blocks / (2 * cus) + 0.14e-3 * (grid - blocks);
}

// Against the 64-row kernel (565 calls: 0.90 of the time in the geometric mean with the rule, 0.89 with the better one each time; eight more than
// 3 % slower, one by 16: mix 896 x 7041, 13 experts with up to 33 rows).
bool block_grouped_is_better(const Layout& L, int E, const GroupedRows& r) {
  return L.K >= 512 && block_grouped_time(L, E, r) < 0.93 * mid_grouped_time(L, E, r);
}

int launch_block_grouped(const ccq_weight* w0, const Layout& L, int E, int64_t codes_stride, int64_t scales_stride, int64_t ab_stride, const void* x,
                         int64_t ldx, const int32_t* sorted_rows, int T, int P, const int32_t* expert_offsets, const GroupedRows& rows, void* y, int64_t ldy,
                         void* stream) {
  const int n_blocks = (L.N + kBlockCols - 1) / kBlockCols;
  const int m_blocks = grouped_row_blocks(E, rows);
  // 32-bit lane offsets reach any activation row and the row tiles of a wavefront, and the grid fits
  if (E < 1 || E > 65535 || n_blocks > 65535 || rows.most < 1 || (int64_t)T * ldx * 2 + 4096 > (int64_t)1 << 32 || 4 * L.row_tile_bytes >= (int64_t)1 << 31)
    return CCQ_ERR_UNSUPPORTED;
  BlockPart p;
  p.n_first = 0;
  p.n_count = L.N;
  p.mt = 4;
  p.S = 1;
  BlockArgs a = block_args(w0, L, x, P, ldx, y, ldy, nullptr, p);
  a.sorted_rows = sorted_rows;
  a.expert_offsets = expert_offsets;
  a.codes_stride = codes_stride;
  a.scales_stride = scales_stride;
  a.ab_stride = ab_stride;
  const BlockKernel kern = L.h16 ? block_grouped_h16(L.scale_mode)
                                 : (L.tiles[kWide] == 0 ? block_grouped_narrow(L.scale_mode)
                                                        : (L.tiles[kNarrow] == 0 ? block_grouped_wide(L.scale_mode) : block_grouped_mix(L.scale_mode)));
  const size_t lds = kBlockLds0 + (size_t)2 * 128 * kGroup * 2;
  hipLaunchKernelGGL(kern, dim3((unsigned)m_blocks, (unsigned)n_blocks, (unsigned)E), dim3(256), lds, static_cast<hipStream_t>(stream), a);
  return hipGetLastError() == hipSuccess ? CCQ_OK : CCQ_ERR_HIP;
}

}  // namespace ccq

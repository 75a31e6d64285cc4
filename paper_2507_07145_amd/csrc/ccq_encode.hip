// The offline quantizer of CCQ on the GPU (gfx950): Alg. 1 (group scale, nearest codeword of the
// convolutional codebook for every N-vector), the least-squares scale of Eq. 4 ("Scale Optimization"),
// and the Code Cluster map of Sec. 3.3 / Eq. 1, for every layout the multiply kernels read.  Output goes
// straight into the device layout that ccq_gemm reads.
//
// Every decision (an argmin, a kept-or-rejected scale) is the one taken in fp64 with separate multiplies and adds in a
// fixed order -- squared errors of a vector are added left to right, the sums of Eq. 4 and of the group error run over
// the 64 weights in index order -- so that the result does not depend on how the work is spread over lanes.
// Contraction into fused multiply-adds is switched off for this file; where one is written out, the product is exact.
// What is searched in fp32 (ccq_search.h, the candidates of the Code Cluster map below) is accepted only where the
// distance to the next best answer exceeds what fp32 can be off by; the rest is searched in fp64 by a whole wavefront.
// Ties go to the numerically lowest code, which is what an exhaustive scan in ascending order returns.
//
// Bound by vector instructions, not by bytes (8192 x 8192 reads 268 MB: 50 us).  The first version searched with one
// state per lane in fp64 (a wavefront per vector, shuffles between the steps): 53 ms narrow, 14 ms wide at that size.
#include <hip/hip_runtime.h>

#include <cmath>

#include "ccq_internal.h"
#include "ccq_search.h"

#pragma clang fp contract(off)

namespace ccq {

// The last unit of a hybrid-word group holds one weight and six zeros of padding, which tie on many paths whatever the
// weight and the scale are.  They are decided once, on the host (h16_tail): the (3,4,2) code of four zeros, and for either
// value of the bit that the first state of the (3,3,2) code passes on, the best states for its two zeros (the lower four
// bits of the code) and what they cost.  `decided` is 0 where rounding could order equal costs differently.
struct H16Tail {
  uint32_t zeros, rest[2];
  float cost[2];
  int32_t decided;
};

struct EncArgs {
  const float* W;       // fp32 [N][ldw]
  int64_t ldw;
  int32_t N, G;        // rows; groups per row (all kinds)
  // the groups of the kind this launch works on (all of them unless the matrix mixes formats): GK groups per row,
  // the p-th of them is original group meta[mbase + p] (p itself without a map), entry pbase + p of a row in the
  // per-(row, group) workspace arrays, and sits at packed position p of the kind's k-tiles, which start
  // kind_code_off bytes / kind_scale_off halfwords into a row tile.  (The map holds whole k-tiles per kind, the
  // workspace arrays only the real groups: with a ragged last narrow tile mbase > pbase for the wide kind.)
  int32_t GK, pbase, mbase;
  int32_t quads;        // ceil(GK / 4): a workgroup takes four groups of sixteen rows
  const int32_t* meta;
  int64_t kind_code_off, kind_scale_off;
  double zp;
  H16Tail tail;         // hybrid word only
  uint8_t* codes;       // device order
  uint16_t* scales;     // device order, fp16 bits
  float* alpha;
  float* beta;
  uint32_t* minmax;     // workspace: smallest and largest (<< 16) unclustered code of a row's four groups, [N][quads] (narrow format only)
  uint16_t* rowscale;   // workspace: fp16 bits of the group scales after the first pass, [N][GK] (narrow format only)
  // compressed scales (Sec. 3.4) only:
  uint16_t* canon_scales;  // workspace: final fp16 group scales, [N][G] (not in device order); NULL = fp16 scales are the output
  uint16_t* ssup;          // output: fp16 super scale per output channel, [N]
  double field_max;        // largest value of a scale field: 15, or 8191 for the hybrid word
  int64_t row_tile_bytes, row_tile_scale_halfs;
};

// ---- fp16 rounding of a non-negative finite double (11-bit significand, minimum normal exponent -14,
// subnormals with quantum 2^-24, round to nearest even), as a double; overflow gives +inf
__device__ __forceinline__ double fp16_round(double x) {
  if (x == 0.0) return 0.0;
  int e;
  (void)frexp(x, &e);  // x = f * 2^e, f in [0.5, 1)
  int q = e - 11;
  if (q < -24) q = -24;
  const double r = nearbyint(ldexp(x, -q));
  const double y = ldexp(r, q);
  return y > 65504.0 ? INFINITY : y;
}
// the scale that is stored: fp16-rounded, and the smallest normal fp16 number when that would be 0 or inf
__device__ __forceinline__ double fp16_scale(double s) {
  const double r = fp16_round(s);
  return (!(r > 0.0) || isinf(r)) ? 0x1p-14 : r;
}
// bit pattern of a non-negative double that is exactly an fp16 number
__device__ __forceinline__ uint16_t fp16_bits(double y) {
  if (y == 0.0) return 0;
  int e;
  const double f = frexp(y, &e);
  const int E = e - 1;
  if (E < -14) return (uint16_t)ldexp(y, 24);
  const uint16_t m = (uint16_t)ldexp(f, 11) & 0x3FFu;
  return (uint16_t)(((E + 15) << 10) | m);
}
__device__ __forceinline__ double fp16_value(uint16_t h) {
  const int e = (h >> 10) & 0x1F, m = h & 0x3FF;
  return e == 0 ? ldexp((double)m, -24) : ldexp((double)(m | 0x400), e - 25);
}

__device__ __forceinline__ double sqerr(double v, double s, double lv) {
  const double d = v - s * lv;
  return d * d;
}

// The exact search: nearest codeword of one N-vector (Alg. 1, the argmin) in fp64, by the 2^L lanes lane & ~(2^L - 1) .. of the
// wavefront, which hold the 2^L states; one step takes the best of the 2^S predecessors of every state.  Every lane of
// that set returns the code.  v[] must be the same in all lanes of the set.
template <int L, int NV, int S>
__device__ __forceinline__ uint32_t nearest_code(const double (&v)[NV], double s, double zp, int lane) {
  constexpr int NS = 1 << L, NT = 1 << S;
  const int st = lane & (NS - 1), base = lane & ~(NS - 1);
  const double lv = (double)st - zp;  // the state's value in the integer domain
  double cost = sqerr(v[0], s, lv);
  uint32_t pre = (uint32_t)st;  // code prefix of the best path that ends in this state
#pragma unroll
  for (int i = 1; i < NV; ++i) {
    const double e = sqerr(v[i], s, lv);
    double best = INFINITY;
    uint32_t bcode = 0xFFFFFFFFu;
#pragma unroll
    for (int h = 0; h < NT; ++h) {
      const int p = base | (h << (L - S)) | (st >> S);  // the predecessors of st: p << S | t = st (mod 2^L)
      const double cp = __shfl(cost, p);
      const uint32_t pp = (uint32_t)__shfl((int)pre, p);
      const double c = cp + e;
      const uint32_t code = (pp << S) | (uint32_t)(st & (NT - 1));
      if (c < best || (c == best && code < bcode)) { best = c; bcode = code; }
    }
    cost = best;
    pre = bcode;
  }
#pragma unroll
  for (int off = NS / 2; off >= 1; off >>= 1) {
    const double oc = __shfl_xor(cost, off);
    const uint32_t op = (uint32_t)__shfl_xor((int)pre, off);
    if (oc < cost || (oc == cost && op < pre)) { cost = oc; pre = op; }
  }
  return pre;
}

// ---- the three kinds of stored code ---------------------------------------------------------------------
enum EncFmt { kEncNarrow = 0, kEncWide = 1, kEncH16 = 2 };

// CPG code units per 64-weight group, WPC weights per unit (a hybrid word is one unit of two codes), 2^(L-1) - 1
template <int FMT> struct EncTraits;
template <> struct EncTraits<kEncNarrow> { static constexpr int CPG = 16, WPC = 4, QMAX = 31; };
template <> struct EncTraits<kEncWide> { static constexpr int CPG = 22, WPC = 3, QMAX = 7; };
template <> struct EncTraits<kEncH16> { static constexpr int CPG = 10, WPC = 7, QMAX = 3; };

// state of weight i of a unit (Table 1: shifts [9,6,3,0], [4,2,0], [13,11,9,6,4,2,0])
template <int FMT>
__device__ __forceinline__ uint32_t unit_state(uint32_t c, int i) {
  if constexpr (FMT == kEncNarrow) return (c >> (9 - 3 * i)) & 63u;
  else if constexpr (FMT == kEncWide) return (c >> (4 - 2 * i)) & 15u;
  else return (c >> (i < 3 ? 13 - 2 * i : 12 - 2 * i)) & 7u;
}

// The lanes that `want` it have their vector searched exactly, as many at a time as the wavefront has sets of 2^L lanes: one
// (narrow), four (wide) or eight (either half of the hybrid word).  Weights with many zeros or few distinct values send a
// large share of their vectors here (half zeros: 14 % of the wide ones, 21 % and 35 % of the halves of the hybrid word).
// 8192 x 8192 with 9 in 10 weights zero, one vector at a time against sets: wide 1.32 -> 0.68 ms, hybrid word 8.98 ->
// 1.48 ms (13.4 -> 2.15 ms with compressed scales); half zeros 2.68 -> 1.00 ms and 5.19 -> 1.00 ms.
template <int L, int NV, int S>
__device__ __forceinline__ uint32_t search_exact(const float* v, double s, double zp, bool want, uint32_t code, int lane) {
  constexpr int kSets = 64 >> L;
  const int set = lane >> L;
  unsigned long long todo = __ballot(want);
  while (todo) {
    const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(todo >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)todo, 0));   // of this lane's vector in todo
    const bool mine = ((todo >> lane) & 1) && rank < kSets;
    int src = 0;   // whose vector this lane's set takes (sets left over repeat the last one)
#pragma unroll
    for (int k = 0; k < kSets; ++k) {
      const int next = __builtin_ctzll(todo);
      if (set >= k) src = next;
      const unsigned long long rest = todo & (todo - 1);
      todo = rest || k == kSets - 1 ? rest : todo;
    }
    double vd[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) vd[i] = (double)__shfl(v[i], src);
    const uint32_t c = nearest_code<L, NV, S>(vd, __shfl(s, src), zp, lane);
    const uint32_t answer = (uint32_t)__shfl((int)c, (rank << L) & 63);
    if (mine) code = answer;
  }
  return code;
}

// One code unit per lane: v[] = its weights, s = the group's scale.  All 64 lanes of the wavefront must be here.
template <int FMT>
__device__ __forceinline__ uint32_t search_unit(const float (&v)[EncTraits<FMT>::WPC], double s, const InvScale& inv, double zp, const H16Tail& tail, int j, bool active,
                                                int lane) {
  constexpr int WPC = EncTraits<FMT>::WPC;
  const float zpf = (float)zp;
  float t[WPC];
#pragma unroll
  for (int i = 0; i < WPC; ++i) t[i] = unit_scale(v[i], inv);
  if constexpr (FMT == kEncNarrow) {
    const FastCode f = fast_narrow(t, zpf);
    return search_exact<6, 4, 3>(v, s, zp, active && !f.sure, f.code, lane);
  } else if constexpr (FMT == kEncWide) {
    const FastCode f = fast_small<4, 3, 2>(t, zpf);
    return search_exact<4, 3, 2>(v, s, zp, active && !f.sure, f.code, lane);
  } else {
    // a (3,3,2) code on the first three weights and a (3,4,2) code on the other four; their bits do not overlap
    const float ta[3] = {t[0], t[1], t[2]}, tb[4] = {t[3], t[4], t[5], t[6]};
    const bool last = j == EncTraits<kEncH16>::CPG - 1 && tail.decided && s == s;
    FastCode fa = fast_small<3, 3, 2>(ta, zpf), fb = fast_small<3, 4, 2>(tb, zpf);
    if (last) {
      fa = fast_first<3, 3, 2>(ta[0], zpf, tail.cost, tail.rest);
      fb.code = tail.zeros;
      fb.sure = true;
    }
    const uint32_t ca = search_exact<3, 3, 2>(v, s, zp, active && !fa.sure, fa.code, lane);
    const uint32_t cb = search_exact<3, 4, 2>(v + 3, s, zp, active && !fb.sure, fb.code, lane);
    return (ca << 9) | cb;
  }
}

// ---- a workgroup's share: sixteen rows (one row tile) x four consecutive groups of the kind, 64 groups in all ----------
// (64 weights and 4 spare, which are zero: what a code reads past the end of its group is the zero padding of Sec. 3.1;
// 68 floats and an odd number of dwords of codes keep lanes that read the same place of different groups apart in LDS)
constexpr int kEncRow = 68;
template <int FMT> constexpr int kEncUnitRow = FMT == kEncNarrow ? 18 : EncTraits<FMT>::CPG;

// Original group of position p of the kind.
__device__ __forceinline__ int enc_group(const EncArgs& a, int p) { return a.meta ? a.meta[a.mbase + p] : p; }

// The 64 groups' weights into LDS, zeros for rows and groups that are not there.
template <int THREADS>
__device__ __forceinline__ void load_groups(const EncArgs& a, int rt, int quad, float* wl, int tid) {
#pragma unroll
  for (int i = 0; i < 1024 / THREADS; ++i) {
    const int f = i * THREADS + tid, row = f >> 6, gj = (f >> 4) & 3, c4 = f & 15;
    const int n = rt * kRowsPerTile + row, p = quad * 4 + gj;
    float4 v = {0.f, 0.f, 0.f, 0.f};
    if (n < a.N && p < a.GK) v = *reinterpret_cast<const float4*>(a.W + (int64_t)n * a.ldw + (int64_t)enc_group(a, p) * kGroup + c4 * 4);
    *reinterpret_cast<float4*>(wl + (row * 4 + gj) * kEncRow + c4 * 4) = v;
  }
  if (tid < 64) *reinterpret_cast<float4*>(wl + tid * kEncRow + 64) = float4{0.f, 0.f, 0.f, 0.f};
}

// Unit j of a group: its weights (a hybrid word's last unit reaches past the spare ones).
template <int FMT>
__device__ __forceinline__ void unit_weights(const float* wg, int j, float (&v)[EncTraits<FMT>::WPC]) {
  constexpr int WPC = EncTraits<FMT>::WPC;
  if constexpr (FMT == kEncNarrow) {
    const float4 w = *reinterpret_cast<const float4*>(wg + 4 * j);
    v[0] = w.x; v[1] = w.y; v[2] = w.z; v[3] = w.w;
  } else {
#pragma unroll
    for (int i = 0; i < WPC; ++i) v[i] = wg[min(WPC * j + i, kGroup)];
  }
}

// All units of a group searched with scale s, LPG lanes per group.
template <int FMT, int LPG>
__device__ __forceinline__ void search_groups(const float* wg, uint16_t* cg, double s, double zp, const H16Tail& tail, bool active, int sub, int lane) {
  constexpr int CPG = EncTraits<FMT>::CPG;
  const InvScale inv = inv_scale(active ? s : 1.0);
#pragma unroll 1
  for (int j0 = 0; j0 < CPG; j0 += LPG) {
    const int j = min(j0 + sub, CPG - 1);
    const bool mine = j0 + sub < CPG;   // (a ragged last round leaves lanes without a unit)
    float v[EncTraits<FMT>::WPC];
    unit_weights<FMT>(wg, j, v);
    const uint32_t c = search_unit<FMT>(v, s, inv, zp, tail, j, active && mine, lane);
    // A vector with a NaN has no nearest code: the exact search returns all ones, which must not reach past the unit's own
    // bits, where the next code lies
    constexpr uint32_t kBits = FMT == kEncWide ? 0xFFu : 0xFFFFu;
    if (mine) cg[j] = (uint16_t)(active ? c & kBits : 0u);
  }
}

// f(w, wq) over the group's weights in index order, wq = the weight's level.
template <int FMT, typename F>
__device__ __forceinline__ void for_weights(const float* wg, const uint16_t* cg, double zp, F f) {
  constexpr int CPG = EncTraits<FMT>::CPG, WPC = EncTraits<FMT>::WPC, TAIL = kGroup - (CPG - 1) * WPC;
#pragma unroll 2
  for (int j = 0; j < CPG - 1; ++j) {
    float v[WPC];
    unit_weights<FMT>(wg, j, v);
    const uint32_t c = cg[j];
#pragma unroll
    for (int i = 0; i < WPC; ++i) f((double)v[i], (double)unit_state<FMT>(c, i) - zp);
  }
  const uint32_t c = cg[CPG - 1];
#pragma unroll
  for (int i = 0; i < TAIL; ++i) f((double)wg[(CPG - 1) * WPC + i], (double)unit_state<FMT>(c, i) - zp);
}

// The codes of the 64 groups into device order.
template <int FMT>
__device__ __forceinline__ void store_units(const EncArgs& a, int rt, int quad, const uint16_t* cl, int tid, int threads) {
  constexpr int CS = kEncUnitRow<FMT>;
  static_assert(FMT != kEncNarrow, "");
  constexpr int kSlots = FMT == kEncWide ? 11 : 10;   // (segment, quarter) pairs: two codes of a quarter, or one word
  for (int i = tid; i < kSlots * 16; i += threads) {
    const int slot = i >> 4, r = i & 15;
    if (rt * kRowsPerTile + r >= a.N) continue;
    uint32_t h[4];
#pragma unroll
    for (int gj = 0; gj < 4; ++gj) {
      const uint16_t* cg = cl + (r * 4 + gj) * CS;
      if constexpr (FMT == kEncWide) {
        const int c = 6 * (slot & 3) + 2 * (slot >> 2);
        h[gj] = (uint32_t)cg[c] | ((uint32_t)cg[c + 1] << 8);
      } else {
        h[gj] = cg[slot];
      }
    }
    uint8_t* tile = a.codes + (int64_t)rt * a.row_tile_bytes + a.kind_code_off + (int64_t)(quad >> 1) * (FMT == kEncWide ? kWideTileBytes : kH16TileBytes);
    *reinterpret_cast<uint2*>(tile + (slot >> 2) * 1024 + ((slot & 3) * 16 + r) * 16 + (quad & 1) * 8) = uint2{h[0] | (h[1] << 16), h[2] | (h[3] << 16)};
  }
}

// The squared error of a group is den (s - s*)^2 above its least, s* = num / den: how much it falls from scale s0 to s1.
__device__ __forceinline__ double error_fall(double den, double s0, double s1, double sbest) { return den * ((s0 - s1) * ((s0 - sbest) + (s1 - sbest))); }
// A fall beyond this (either way) decides which of the two sums of squared errors is the smaller without forming them.  A residual and
// its two terms are below r (amax: no weight is larger), so its square is off by less than 5 2^-53 r^2, a sum of 64 by less than
// (64 5 + 63 64) 2^-53 r^2 < 2^-40 r^2, and the rounding of num moves the fall by less than 2^-40 r^2.  Nearly every group is decided
// (the scale moves by 1e-3 of itself and more); 8192 x 8192: narrow 735 -> 678, wide 352 -> 306, hybrid word 318 -> 271 us.
template <int FMT>
__device__ __forceinline__ double error_doubt(double amax, double s0, double s1, double zp) {
  const double smax = 2.0 * EncTraits<FMT>::QMAX + 1.0;   // the largest state
  const double r = amax + fmax(fabs(zp), fabs(smax - zp)) * fmax(s0, s1);
  return 0x1p-38 * (r * r);
}

// Eq. 4: S = sum(W Wq) / sum(Wq^2), s0 where that is no better, rounded to the scale that is stored.  A fp32 number times a
// level (at most 8 bits) is exact in fp64, so the fused multiply-add rounds once, as the separate multiply and add do.
template <int FMT>
__device__ __forceinline__ double refit_scale(const float* wg, const uint16_t* cg, double s0, double zp) {
  double num = 0.0, den = 0.0;
  for_weights<FMT>(wg, cg, zp, [&](double w, double wq) {
    num = __builtin_fma(w, wq, num);
    den = __builtin_fma(wq, wq, den);
  });
  double s1 = den > 0.0 ? num / den : s0;
  if (s1 > 0.0 && error_fall(den, s0, s1, s1) > error_doubt<FMT>((double)EncTraits<FMT>::QMAX * s0, s0, s1, zp)) return fp16_scale(s1);
  double e1 = 0.0, e0 = 0.0;
  for_weights<FMT>(wg, cg, zp, [&](double w, double wq) {
    const double d1 = w - wq * s1, d0 = w - wq * s0;
    e1 += d1 * d1;
    e0 += d0 * d0;
  });
  if (!(s1 > 0.0) || e1 > e0) s1 = s0;
  return fp16_scale(s1);
}

// Smallest and largest (<< 16) code, narrow format, of each row's four groups under the scales sl, returned to threads 0 .. 15.  Of the second search
// nothing else is wanted, so only vectors that can have one of the two are searched.  cl holds the first search's codes: what such a code costs
// under the new scale is no less than what the nearest one does, so the nearest one's first state, the upper six bits of its code, is no
// further from its weight than the root of that cost.  A vector whose least possible state is above the row's smallest greatest one cannot have
// the row's smallest code, and so for the largest.  About one in eight is left on Gaussian weights; they are listed (in cl) and shared out
// over the workgroup.  (8192 x 8192, first pass: 287 us with all vectors searched, 219.)
template <int LPG>
__device__ __forceinline__ uint32_t code_range(const float* wl, uint16_t* cl, const double* sl, double zp, bool there, bool live, int tid) {
  constexpr int CS = kEncUnitRow<kEncNarrow>, kThreads = 64 * LPG, kMine = 16 / LPG;
  static_assert(64 * CS >= 1024, "the list takes the place of the codes");
  __shared__ uint32_t row_lo[16], row_hi[16], listed;
  const int lane = tid & 63, gl = tid / LPG, sub = tid % LPG;
  if (tid < 16) row_lo[tid] = 0xFFFFu, row_hi[tid] = 0u;
  if (tid == 0) listed = 0;
  __syncthreads();
  const InvScale inv = inv_scale(live ? sl[gl] : 1.0);
  const float zpf = (float)zp;
  int lo[kMine], hi[kMine], least = 63, most = 0;   // a row's smallest greatest state, and its largest least one
#pragma unroll
  for (int i = 0; i < kMine; ++i) {
    const int j = sub + i * LPG;
    float v[4], T = 0.f, u0 = 0.f;
    unit_weights<kEncNarrow>(wl + gl * kEncRow, j, v);
    const uint32_t c = cl[gl * CS + j];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float u = unit_scale(v[k], inv) + zpf, d = (float)unit_state<kEncNarrow>(c, k) - u;
      T = __builtin_fmaf(d, d, T);
      if (k == 0) u0 = u;
    }
    // (u and T are off by a millionth of themselves; NaN and what is far beyond the levels can be anything)
    const bool known = T < 1e6f;
    const float r = __builtin_fmaf(__builtin_amdgcn_sqrtf(T), 1.001f, 0.01f);
    lo[i] = known ? (int)med_(ceilf(u0 - r), 0.f, 63.f) : 0;
    hi[i] = known ? (int)med_(floorf(u0 + r), 0.f, 63.f) : 63;
    if (!live) lo[i] = hi[i] = 0;   // codes of zero
    if (there) least = min(least, hi[i]), most = max(most, lo[i]);
  }
#pragma unroll
  for (int off = 2 * LPG; off >= 1; off >>= 1) {
    least = min(least, __shfl_xor(least, off));
    most = max(most, __shfl_xor(most, off));
  }
  __syncthreads();   // the codes have been read
#pragma unroll
  for (int i = 0; i < kMine; ++i)
    if (there && live && (lo[i] <= least || hi[i] >= most)) cl[atomicAdd(&listed, 1u)] = (uint16_t)(gl * 16 + sub + i * LPG);
  if (there && !live && sub == 0) atomicMin(&row_lo[gl >> 2], 0u);
  __syncthreads();
  const int count = (int)listed;
  const H16Tail none = {};
#pragma unroll 1
  for (int i0 = 0; i0 < count; i0 += kThreads) {
    // (with sixteen lanes per group a wavefront's exact searches, one after the other, are the time: every wavefront takes a few)
    const int i = i0 + (LPG > 4 ? lane * LPG + (tid >> 6) : tid);
    const bool active = i < count;
    const int id = active ? cl[i] : 0, g = id >> 4;
    float v[4];
    unit_weights<kEncNarrow>(wl + g * kEncRow, id & 15, v);
    const double s = sl[g];
    const uint32_t c = search_unit<kEncNarrow>(v, s, inv_scale(active ? s : 1.0), zp, none, 0, active, lane) & 0xFFFFu;
    if (active) {
      atomicMin(&row_lo[g >> 2], c);
      atomicMax(&row_hi[g >> 2], c);
    }
  }
  __syncthreads();
  return tid < 16 ? row_lo[tid] | (row_hi[tid] << 16) : 0u;
}

// First pass, LPG lanes per (row, group): scale = absmax / (2^(L-1) - 1), search, Eq. 4 refit (kept when the error does
// not grow), fp16 rounding, search again with the stored scale.  An all-zero group gets scale 0 and codes 0.  Without
// Code Cluster this is the final result and is written in device order; with it only the scales and the range of the
// codes are wanted by the passes that follow (code_range).
template <int FMT, int LPG>
__global__ void __launch_bounds__(64 * LPG) ccq_encode_groups_kernel(const EncArgs a) {
  constexpr int CS = kEncUnitRow<FMT>;
  __shared__ __attribute__((aligned(16))) float wl[64 * kEncRow];
  __shared__ uint16_t cl[64 * CS];
  __shared__ double sl[FMT == kEncNarrow || LPG > 4 ? 64 : 1];
  const int tid = threadIdx.x, lane = tid & 63, rt = blockIdx.x / a.quads, quad = blockIdx.x % a.quads;
  load_groups<64 * LPG>(a, rt, quad, wl, tid);
  __syncthreads();
  const int gl = tid / LPG, sub = tid % LPG;
  const int n = rt * kRowsPerTile + (gl >> 2), p = quad * 4 + (gl & 3);
  const bool there = n < a.N && p < a.GK;
  const float* wg = wl + gl * kEncRow;
  uint16_t* cg = cl + gl * CS;
  float amax = __builtin_nanf("");   // stays one in a group of nothing else, which then has codes of all ones and the smallest scale
  for (int c4 = sub; c4 < 16; c4 += LPG) {
    const float4 w = *reinterpret_cast<const float4*>(wg + 4 * c4);
    amax = fmaxf(fmaxf(amax, fmaxf(fabsf(w.x), fabsf(w.y))), fmaxf(fabsf(w.z), fabsf(w.w)));
  }
#pragma unroll
  for (int off = LPG / 2; off >= 1; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off));
  const bool live = amax != 0.f;
  const double s0 = (double)amax / (double)EncTraits<FMT>::QMAX;
  search_groups<FMT, LPG>(wg, cg, s0, a.zp, a.tail, live, sub, lane);
  constexpr bool kOneWave = FMT == kEncNarrow || LPG > 4;
  if (kOneWave && sub == 0) sl[gl] = s0;
  __syncthreads();
  double s = 0.0;
  if constexpr (kOneWave) {
    // The sums, one lane per group: sixteen copies would share the CU's fp64 units.  By one wavefront of the workgroup, not the same in all of
    // them, as a wavefront's place decides its SIMD.  (Two lanes per group, 8192 x 8192, against both running the sums: narrow 219 -> 211 us, but
    // wide 287 -> 293, whose workgroups have more to do on either side of it.)
    if ((tid >> 6) == (int)((blockIdx.x * 2654435761u) >> (32 - (LPG == 2 ? 1 : (LPG == 4 ? 2 : 4))))) {
      const double st = sl[lane];
      if (st != 0.0) sl[lane] = refit_scale<FMT>(wl + lane * kEncRow, cl + lane * CS, st, a.zp);
    }
    __syncthreads();
    s = sl[gl];
  } else {
    if (live) s = refit_scale<FMT>(wg, cg, s0, a.zp);
    __syncthreads();
  }
  if constexpr (FMT == kEncNarrow) {
    if (there && sub == 0) a.rowscale[(int64_t)n * a.GK + p] = fp16_bits(s);
    const uint32_t range = code_range<LPG>(wl, cl, sl, a.zp, there, live, tid);
    if (tid < 16 && rt * kRowsPerTile + tid < a.N) a.minmax[(int64_t)(rt * kRowsPerTile + tid) * a.quads + quad] = range;
  } else {
    search_groups<FMT, LPG>(wg, cg, s, a.zp, a.tail, live, sub, lane);
    __syncthreads();
    store_units<FMT>(a, rt, quad, cl, tid, 64 * LPG);
    if (there && sub == 0) {
      if (a.canon_scales) a.canon_scales[(int64_t)n * a.G + a.pbase + p] = fp16_bits(s);
      else
        a.scales[(int64_t)rt * a.row_tile_scale_halfs + a.kind_scale_off + (int64_t)(quad >> 1) * kWideTileScaleHalfs + (gl >> 2) * kWideGroupsPerTile +
                 (quad & 1) * 4 + (gl & 3)] = fp16_bits(s);
    }
  }
}

// Second pass (Sec. 3.3, Eq. 1), one wavefront per output channel: beta = smallest code of the row,
// alpha = (largest - smallest) / 255 (1 when they are equal).
__global__ void __launch_bounds__(256) ccq_encode_cluster_kernel(const EncArgs a) {
  const int n = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (n >= a.N) return;
  uint32_t lo = 0xFFFFu, hi = 0;
  for (int i = lane; i < a.quads; i += 64) {
    const uint32_t m = a.minmax[(int64_t)n * a.quads + i];
    lo = min(lo, m & 0xFFFFu);
    hi = max(hi, m >> 16);
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    lo = min(lo, (uint32_t)__shfl_xor((int)lo, off));
    hi = max(hi, (uint32_t)__shfl_xor((int)hi, off));
  }
  if (lane == 0) {
    a.beta[n] = (float)lo;
    a.alpha[n] = hi > lo ? (float)((double)(hi - lo) / 255.0) : 1.0f;
  }
}

// ---- search over the 256 codes a row's Code Cluster map reaches ---------------------------------------------------
// cost(q) - |t|^2 = |lv(q)|^2 - 2 lv(q) . t is a contraction over the four weights of a vector: MFMA 32x32x16 bf16 with the
// candidates as A and the vectors as B.  Levels are multiples of 0.5 up to 64: exact in bf16; -2 t is cut into three bf16
// numbers (24 bits) and |lv|^2 (at most 16 bits) into two:
//   k-slot    0..3   4..7   8..11   12      13     14 15
//   A         lv     lv     lv      |lv|^2 high, low      0
//   B         the three parts of -2t        1      1      0
// so products are exact and only the fp32 sums round: 16 of them, below |lv|^2 + 2 sum |lv t|.  Per vector the smallest
// value of every block of eight candidates is tracked (best block, second best value); the eight of the best block are
// compared in fp32 as sums of squares; both times the answer is taken only when the next best is further away than
// rounding reaches, and the other vectors are searched in fp64.
// Bound by vector issue, so what is not needed stays out: products in vector registers (four wavefronts per SIMD asked for: with more than 256
// registers allowed the compiler takes accumulator registers and moves every product out, 256 moves per 64 vectors), minima without
// the quieting of their operands, a lane of the map per candidate, its levels from a table.  8192 x 8192, finish pass 425 -> 305 us, 676 ->
// 613 vector instructions per 64 vectors by the last two (1066 at first).
typedef __attribute__((ext_vector_type(8))) __bf16 enc_bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 enc_bf16x2;
typedef __attribute__((ext_vector_type(2))) float enc_f32x2;
typedef __attribute__((ext_vector_type(16))) float enc_f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t enc_u32x4;

__device__ __forceinline__ uint32_t enc_pack_bf16(float lo, float hi) {
  const enc_f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, enc_bf16x2));
}
__device__ __forceinline__ float enc_lo(uint32_t v) { return __builtin_bit_cast(float, v << 16); }
__device__ __forceinline__ float enc_hi(uint32_t v) { return __builtin_bit_cast(float, v & 0xFFFF0000u); }

// code of byte q: round(q alpha + beta) by one FMA against beta + 2^23 (exact: the sum lies in [2^23, 2^24))
__device__ __forceinline__ uint32_t cluster_code(float q, float al, float bem) { return __builtin_bit_cast(uint32_t, __builtin_fmaf(q, al, bem)) & 0x7FFFu; }

struct RowMap {
  enc_u32x4 A[8];   // the candidates, 32 per tile
  const uint32_t* states;   // of all of them, a byte each (LDS, this wavefront's)
  float al, bem, zp, lmax;
};

// A lane works out one candidate of two tiles' 64, and the halves of the wavefront exchange them.
__device__ __forceinline__ void row_map(RowMap& m, float al, float be, float zp, uint32_t* states, int lane) {
  m.al = al;
  m.bem = be + 0x1p23f;
  m.zp = zp;
  m.lmax = fmaxf(zp, 63.f - zp);
  m.states = states;
  const bool upper = lane >= 32;
#pragma unroll
  for (int t = 0; t < 8; t += 2) {
    const uint32_t c = cluster_code((float)(32 * t + lane), al, m.bem);
    float lv[4], n = 0.f;
    uint32_t all = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t st = unit_state<kEncNarrow>(c, i);
      lv[i] = (float)st - zp;
      n = __builtin_fmaf(lv[i], lv[i], n);
      all |= st << (8 * i);
    }
    states[32 * t + lane] = all;
    const uint32_t l01 = enc_pack_bf16(lv[0], lv[1]), l23 = enc_pack_bf16(lv[2], lv[3]);
    const uint32_t nh = enc_pack_bf16(n, 0.f);
    const uint32_t nn = nh | (enc_pack_bf16(n - enc_lo(nh), 0.f) << 16);
    // element 0: what the lower lanes hold, in both halves; 1: what the upper lanes hold
    const auto x01 = __builtin_amdgcn_permlane32_swap(l01, l01, false, false);
    const auto x23 = __builtin_amdgcn_permlane32_swap(l23, l23, false, false);
    const auto xn = __builtin_amdgcn_permlane32_swap(nn, nn, false, false);
#pragma unroll
    for (int h = 0; h < 2; ++h) m.A[t + h] = enc_u32x4{x01[h], x23[h], upper ? xn[h] : x01[h], upper ? 0u : x23[h]};
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ double cluster_cost(uint32_t c, const double (&v)[4], double s, double zp) {
  double cost = sqerr(v[0], s, (double)unit_state<kEncNarrow>(c, 0) - zp);
  cost = cost + sqerr(v[1], s, (double)unit_state<kEncNarrow>(c, 1) - zp);
  cost = cost + sqerr(v[2], s, (double)unit_state<kEncNarrow>(c, 2) - zp);
  cost = cost + sqerr(v[3], s, (double)unit_state<kEncNarrow>(c, 3) - zp);
  return cost;
}

// the smallest value, whose it is, and the second smallest
__device__ __forceinline__ void see_block(float x, int i, float& best, float& second, int& at) {
  at = x < best ? i : at;
  second = __builtin_amdgcn_fmed3f(best, second, x);
  best = fminf(best, x);
}

// One vector per lane, all of the row m is the map of; returns the byte.  All 64 lanes must be here.
__device__ __forceinline__ uint32_t search_cluster(const RowMap& m, const float4 w, double s, double zp, bool active, int lane) {
  const float v[4] = {w.x, w.y, w.z, w.w};
  const InvScale inv = inv_scale(active ? s : 1.0);
  float t[4], x[4], y[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) t[i] = unit_scale(v[i], inv), x[i] = -2.f * t[i];
  const uint32_t h01 = enc_pack_bf16(x[0], x[1]), h23 = enc_pack_bf16(x[2], x[3]);
  y[0] = x[0] - enc_lo(h01), y[1] = x[1] - enc_hi(h01), y[2] = x[2] - enc_lo(h23), y[3] = x[3] - enc_hi(h23);
  const uint32_t m01 = enc_pack_bf16(y[0], y[1]), m23 = enc_pack_bf16(y[2], y[3]);
  const uint32_t l01 = enc_pack_bf16(y[0] - enc_lo(m01), y[1] - enc_hi(m01)), l23 = enc_pack_bf16(y[2] - enc_lo(m23), y[3] - enc_hi(m23));
  // operand of the vectors of lanes 0..31 (k-slots 0..7 in lanes 0..31, 8..15 in lanes 32..63), and of lanes 32..63
  const auto s0 = __builtin_amdgcn_permlane32_swap(h01, l01, false, false);
  const auto s1 = __builtin_amdgcn_permlane32_swap(h23, l23, false, false);
  const auto s2 = __builtin_amdgcn_permlane32_swap(m01, 0x3F803F80u, false, false);
  const auto s3 = __builtin_amdgcn_permlane32_swap(m23, 0u, false, false);
  float best[2], second[2];
  int at[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const enc_u32x4 B = {s0[h], s1[h], s2[h], s3[h]};
    best[h] = second[h] = kFar;
    at[h] = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const enc_f32x16 zero = {};
      const enc_f32x16 d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(enc_bf16x8, m.A[k]), __builtin_bit_cast(enc_bf16x8, B), zero, 0, 0, 0);
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const float b0 = fminf(fminf(d[8 * b], d[8 * b + 1]), d[8 * b + 2]), b1 = fminf(fminf(d[8 * b + 3], d[8 * b + 4]), d[8 * b + 5]);
        const float b2 = fminf(fminf(b0, b1), d[8 * b + 6]);
        see_block(med_(b2, d[8 * b + 7], -kFar), 2 * k + b, best[h], second[h], at[h]);
      }
    }
  }
  // lane l and lane l ^ 32 hold the two halves of a vector's candidates: bring both to the vector's own lane
  const auto cb = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, best[0]), __builtin_bit_cast(uint32_t, best[1]), false, false);
  const auto cs = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, second[0]), __builtin_bit_cast(uint32_t, second[1]), false, false);
  const auto ca = __builtin_amdgcn_permlane32_swap((uint32_t)at[0], (uint32_t)at[1], false, false);
  const uint32_t b0 = cb[0], b1 = cb[1], n0 = cs[0], n1 = cs[1];   // (by value: a bit cast of a vector's element takes element 0)
  const float p0 = __builtin_bit_cast(float, b0), p1 = __builtin_bit_cast(float, b1);
  const bool upper = p1 < p0;   // which half
  const float first = fminf(p0, p1);
  const float next = fminf(fmaxf(p0, p1), fminf(__builtin_bit_cast(float, n0), __builtin_bit_cast(float, n1)));
  const int blk = upper ? (int)ca[1] : (int)ca[0];
  const float tmax = max_abs(t);
  // 16 sums of numbers below 4 lmax^2 + 8 lmax tmax, each off by at most 2^-23 of that; both sides
  bool sure = next - first > 0x1p-18f * (4.f * m.lmax * m.lmax + 8.f * m.lmax * tmax);
  // the best block's candidates: rows 16 (blk % 2) + 4 half + {0..3, 8..11} of tile blk / 2
  const int q0 = 16 * blk + (upper ? 4 : 0);
  const enc_u32x4 near[2] = {*reinterpret_cast<const enc_u32x4*>(m.states + q0), *reinterpret_cast<const enc_u32x4*>(m.states + q0 + 8)};
  float u[4];   // the wanted places among the states: rounded once more than t, which every difference then carries
#pragma unroll
  for (int k = 0; k < 4; ++k) u[k] = t[k] + m.zp;
  Best2 in;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const uint32_t states = near[i >> 2][i & 3];
    float T = 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float d = (float)((states >> (8 * k)) & 255u) - u[k];
      T = __builtin_fmaf(d, d, T);
    }
    in.see(T, i + (i & 4));
  }
  // (2 sum |d| 2^-24 |u| on either side, in search_margin's terms)
  const float apart = search_margin(in.best, tmax) + 0x1p-22f * (tmax + fabsf(m.zp)) * (in.best + 1.f);
  sure = sure && in.gap() > apart && tmax <= kSearchMaxT;
  uint32_t q = (uint32_t)(q0 + in.at) & 255u;
  unsigned long long todo = __ballot(active && !sure);
  while (todo) {   // exactly: four candidates per lane
    const int src = __builtin_ctzll(todo);
    todo &= todo - 1;
    double vd[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) vd[i] = (double)__shfl(v[i], src);
    const double sd = __shfl(s, src);
    double bc = INFINITY;
    uint32_t bq = 0xFFFFFFFFu;
#pragma unroll 1
    for (int k = 0; k < 4; ++k) {
      const double cost = cluster_cost(cluster_code((float)(lane + 64 * k), m.al, m.bem), vd, sd, zp);
      if (cost < bc) { bc = cost; bq = (uint32_t)(lane + 64 * k); }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      const double oc = __shfl_xor(bc, off);
      const uint32_t oq = (uint32_t)__shfl_xor((int)bq, off);
      if (oc < bc || (oc == bc && oq < bq)) { bc = oc; bq = oq; }
    }
    if (lane == src) q = bq;
  }
  return active ? q : 0u;
}

// A workgroup of the passes over the row's map takes four rows x sixteen groups (four narrow k-tiles): a wavefront keeps
// one row's map and walks its groups four at a time, one vector per lane.  Building the map costs about half of what 64
// vectors cost to search: with one k-tile of four rows per wavefront instead the pass took 500 us at 8192 x 8192.
struct ClusterBlock {
  int row, n, rt, tile0;   // this wavefront's row of the workgroup, of the matrix; row tile; first k-tile
};
template <int TILES>
__device__ __forceinline__ ClusterBlock cluster_block(const EncArgs& a) {
  const int per_row = (a.quads + TILES - 1) / TILES, rq = blockIdx.x / per_row;
  ClusterBlock b;
  b.row = threadIdx.x >> 6;
  b.n = rq * 4 + b.row;
  b.rt = rq >> 2;
  b.tile0 = (blockIdx.x % per_row) * TILES;
  return b;
}

// The workgroup's bytes, [k-tile][row][group][16] in LDS, to device order: byte 4 kq + b of group j of a k-tile at
// (kq * 16 + row) * 16 + 4 j + b.  One 16-byte store per thread of a wavefront: (k-tile, kq, row).
template <int TILES>
__device__ __forceinline__ void store_bytes(const EncArgs& a, const ClusterBlock& b, const uint32_t* ql, int lane) {
  const int t = lane >> 4, kq = (lane >> 2) & 3, row = lane & 3, n = b.n - b.row + row;
  if (t >= TILES || n >= a.N || b.tile0 + t >= a.quads) return;
  const uint32_t* src = ql + (t * 4 + row) * 16 + kq;
  *reinterpret_cast<uint4*>(a.codes + (int64_t)b.rt * a.row_tile_bytes + a.kind_code_off + (int64_t)(b.tile0 + t) * kNarrowTileBytes + (kq * 16 + (n & 15)) * 16) =
      uint4{src[0], src[4], src[8], src[12]};
}

// Third pass (narrow format): every vector is searched again over the 256 codes round(q alpha + beta) the row's map can
// reach (never worse than rounding the unconstrained code by Eq. 1, which is one of the candidates), then one more Eq. 4
// refit with the final codes, kept when the error does not grow; its sums run one group per lane.
template <int TILES>
__global__ void __launch_bounds__(256, 4) ccq_encode_finish_narrow_kernel(const EncArgs a) {
  __shared__ __attribute__((aligned(16))) float wl[16 * TILES * kEncRow];
  __shared__ __attribute__((aligned(16))) uint32_t ql[16 * TILES * 4];
  __shared__ __attribute__((aligned(16))) uint32_t states[4 * 256];
  const int lane = threadIdx.x & 63, gj = lane >> 4;
  const ClusterBlock b = cluster_block<TILES>(a);
  if (b.n < a.N) {   // (uniform in the wavefront)
    RowMap m;
    row_map(m, a.alpha[b.n], a.beta[b.n], (float)a.zp, states + 256 * b.row, lane);
#pragma unroll 1
    for (int t = 0; t < TILES; ++t) {
      const int p = (b.tile0 + t) * 4 + gj, slot = (t * 4 + b.row) * 4 + gj;
      float4 w = {0.f, 0.f, 0.f, 0.f};
      double s = 0.0;
      if (p < a.GK) {
        w = *reinterpret_cast<const float4*>(a.W + (int64_t)b.n * a.ldw + (int64_t)enc_group(a, p) * kGroup + (lane & 15) * 4);
        s = fp16_value(a.rowscale[(int64_t)b.n * a.GK + p]);
      }
      const uint32_t q = search_cluster(m, w, s, a.zp, s > 0.0, lane);
      *reinterpret_cast<float4*>(wl + slot * kEncRow + (lane & 15) * 4) = w;
      reinterpret_cast<uint8_t*>(ql)[slot * 16 + (lane & 15)] = (uint8_t)q;
    }
  }
  __syncthreads();
  if (b.row == 3) store_bytes<TILES>(a, b, ql, lane);
  if (b.row != 0) return;
  // lane = slot: k-tile lane / 16, row (lane / 4) % 4, group lane % 4
  const int n = b.n + ((lane >> 2) & 3), tile = b.tile0 + (lane >> 4), p = tile * 4 + (lane & 3);
  if (lane >= 16 * TILES || n >= a.N || p >= a.GK) return;
  const float al = a.alpha[n], bem = a.beta[n] + 0x1p23f;
  double s = fp16_value(a.rowscale[(int64_t)n * a.GK + p]);
  auto for_all = [&](auto f) {
#pragma unroll 1
    for (int j4 = 0; j4 < 4; ++j4) {
      const uint32_t qs = ql[lane * 4 + j4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t c = cluster_code((float)((qs >> (8 * k)) & 255u), al, bem);
        const float4 w = *reinterpret_cast<const float4*>(wl + lane * kEncRow + 16 * j4 + 4 * k);
        f((double)w.x, (double)unit_state<kEncNarrow>(c, 0) - a.zp);
        f((double)w.y, (double)unit_state<kEncNarrow>(c, 1) - a.zp);
        f((double)w.z, (double)unit_state<kEncNarrow>(c, 2) - a.zp);
        f((double)w.w, (double)unit_state<kEncNarrow>(c, 3) - a.zp);
      }
    }
  };
  double num = 0.0, den = 0.0;
  float amax = 0.f;
  for_all([&](double w, double wq) {
    num = __builtin_fma(w, wq, num);   // exact products, as in the first pass
    den = __builtin_fma(wq, wq, den);
    amax = fmaxf(amax, fabsf((float)w));
  });
  const double s2 = den > 0.0 ? num / den : s;
  const double s2h = s2 > 0.0 ? fp16_scale(s2) : s;
  const double fall = error_fall(den, s, s2h, s2), doubt = error_doubt<kEncNarrow>((double)amax, s, s2h, a.zp);
  double e2 = fall > doubt ? -1.0 : 0.0, e1 = fall < -doubt ? -1.0 : 0.0;
  if (!(fabs(fall) > doubt)) for_all([&](double w, double wq) {
    const double d2 = __builtin_fma(-wq, s2h, w), d1 = __builtin_fma(-wq, s, w);   // (an fp16 number times a level is exact too)
    e2 += d2 * d2;
    e1 += d1 * d1;
  });
  if (e2 <= e1) s = s2h;
  if (a.canon_scales) a.canon_scales[(int64_t)n * a.G + a.pbase + p] = fp16_bits(s);
  else
    a.scales[(int64_t)b.rt * a.row_tile_scale_halfs + a.kind_scale_off + (int64_t)tile * kNarrowTileScaleHalfs + (n & 15) * kNarrowGroupsPerTile + (lane & 3)] = fp16_bits(s);
}

// ---- Sec. 3.4 "Scale Compression", encoder side ------------------------------------------------------
// Channel-wise super scale: the largest group scale of the row / the largest field value, rounded to fp16.  (fp16 bit patterns of
// non-negative numbers order like the numbers.)
__global__ void __launch_bounds__(256) ccq_encode_super_kernel(const EncArgs a) {
  __shared__ uint32_t smax[256];
  const int n = blockIdx.x;
  uint32_t hi = 0;
  for (int i = threadIdx.x; i < a.G; i += 256) hi = max(hi, (uint32_t)a.canon_scales[(int64_t)n * a.G + i]);
  smax[threadIdx.x] = hi;
  __syncthreads();
  for (int off = 128; off >= 1; off >>= 1) {
    if ((int)threadIdx.x < off) smax[threadIdx.x] = max(smax[threadIdx.x], smax[threadIdx.x + off]);
    __syncthreads();
  }
  if (threadIdx.x == 0) a.ssup[n] = fp16_bits(fp16_round(fp16_value((uint16_t)smax[0]) / a.field_max));
}

// The group scale becomes the nearest multiple field * s_super, field in 1..field_max (0 only when the scale or the super
// scale is 0).
__device__ __forceinline__ int scale_field(const EncArgs& a, int n, int p, double& se) {
  const double s = fp16_value(a.canon_scales[(int64_t)n * a.G + a.pbase + p]), ssup = fp16_value(a.ssup[n]);
  int k = 0;
  if (ssup > 0.0 && s > 0.0) {
    const double kr = nearbyint(s / ssup);
    k = kr < 1.0 ? 1 : (kr > a.field_max ? (int)a.field_max : (int)kr);
  }
  se = (double)k * ssup;  // the scale the decoder will use
  return k;
}

// Because the scale that is stored has changed, every group's codes are searched once more with it; a group whose scale
// is now 0 keeps its codes.  Wide format and hybrid word: over all codes; the field goes into the spare low nibble of the
// wide group's last byte, or the low 13 bits of the last word (scale mask 0x1FFF of Table 1).
template <int FMT, int LPG>
__global__ void __launch_bounds__(64 * LPG) ccq_encode_compress_kernel(const EncArgs a) {
  constexpr int CS = kEncUnitRow<FMT>, CPG = EncTraits<FMT>::CPG;
  __shared__ __attribute__((aligned(16))) float wl[64 * kEncRow];
  __shared__ uint16_t cl[64 * CS];
  const int tid = threadIdx.x, lane = tid & 63, rt = blockIdx.x / a.quads, quad = blockIdx.x % a.quads;
  load_groups<64 * LPG>(a, rt, quad, wl, tid);
  __syncthreads();
  const int gl = tid / LPG, sub = tid % LPG;
  const int n = rt * kRowsPerTile + (gl >> 2), p = quad * 4 + (gl & 3);
  const bool there = n < a.N && p < a.GK;
  uint16_t* cg = cl + gl * CS;
  double se = 0.0;
  const int k = there ? scale_field(a, n, p, se) : 0;
  search_groups<FMT, LPG>(wl + gl * kEncRow, cg, se, a.zp, a.tail, se > 0.0, sub, lane);
  __syncthreads();
  if (there && sub == 0) {
    if (!(se > 0.0)) {
      const uint8_t* tile = a.codes + (int64_t)rt * a.row_tile_bytes + a.kind_code_off + (int64_t)(quad >> 1) * (FMT == kEncWide ? kWideTileBytes : kH16TileBytes) +
                            ((quad & 1) * 4 + (gl & 3)) * 2;
      for (int j = 0; j < CPG; ++j) {
        if constexpr (FMT == kEncWide) cg[j] = tile[((j % 6) / 2) * 1024 + ((j / 6) * 16 + (gl >> 2)) * 16 + (j & 1)];
        else cg[j] = *reinterpret_cast<const uint16_t*>(tile + (j >> 2) * 1024 + ((j & 3) * 16 + (gl >> 2)) * 16);
      }
    }
    cg[CPG - 1] = (uint16_t)((cg[CPG - 1] & (FMT == kEncWide ? 0xF0u : 0xE000u)) | (uint32_t)k);
  }
  __syncthreads();
  store_units<FMT>(a, rt, quad, cl, tid, 64 * LPG);
}

// Narrow format: over the 256 codes of the row's map; the four fields of a k-tile's groups go into one 16-bit word per
// row (group j in bits 4j..4j+3; groups that pad the last k-tile keep field 0: scale 0).
template <int TILES>
__global__ void __launch_bounds__(256, 4) ccq_encode_compress_narrow_kernel(const EncArgs a) {
  __shared__ __attribute__((aligned(16))) uint32_t ql[16 * TILES * 4];
  __shared__ __attribute__((aligned(16))) uint32_t states[4 * 256];
  const int lane = threadIdx.x & 63, gj = lane >> 4;
  const ClusterBlock b = cluster_block<TILES>(a);
  if (b.n < a.N) {   // (uniform in the wavefront)
    RowMap m;
    row_map(m, a.alpha[b.n], a.beta[b.n], (float)a.zp, states + 256 * b.row, lane);
#pragma unroll 1
    for (int t = 0; t < TILES; ++t) {
      const int tile = b.tile0 + t, p = tile * 4 + gj;
      float4 w = {0.f, 0.f, 0.f, 0.f};
      double se = 0.0;
      int k = 0;
      if (p < a.GK) {
        w = *reinterpret_cast<const float4*>(a.W + (int64_t)b.n * a.ldw + (int64_t)enc_group(a, p) * kGroup + (lane & 15) * 4);
        k = scale_field(a, b.n, p, se);
      }
      uint32_t q = search_cluster(m, w, se, a.zp, se > 0.0, lane);
      if (p < a.GK && !(se > 0.0))
        q = a.codes[(int64_t)b.rt * a.row_tile_bytes + a.kind_code_off + (int64_t)tile * kNarrowTileBytes + (((lane & 15) >> 2) * 16 + (b.n & 15)) * 16 + gj * 4 + (lane & 3)];
      reinterpret_cast<uint8_t*>(ql)[((t * 4 + b.row) * 4 + gj) * 16 + (lane & 15)] = (uint8_t)q;
      const int word = k << (4 * gj);
      const int all = __shfl(word, 0) | __shfl(word, 16) | __shfl(word, 32) | __shfl(word, 48);
      if (lane == 0 && tile < a.quads)
        a.scales[(int64_t)b.rt * a.row_tile_scale_halfs + a.kind_scale_off + (int64_t)tile * kNarrowTileScaleHalfs4 + (b.n & 15)] = (uint16_t)all;
    }
  }
  __syncthreads();
  if (b.row == 3) store_bytes<TILES>(a, b, ql, lane);
}

// Clears `n16` 16-byte units (a kernel, not a memset node: the call may be recorded into a graph).
__global__ void __launch_bounds__(256) ccq_encode_clear_kernel(uint4* p, int64_t n16) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n16) p[i] = uint4{0u, 0u, 0u, 0u};
}

static int64_t round16(int64_t v) { return (v + 15) / 16 * 16; }

// The workspace is laid out as [range of the unclustered codes, first-pass scales (narrow)] [final fp16 scales (compressed
// scales)].  The figure that callers size it by is an older one and stays: room for every unclustered code and a byte
// per narrow group besides, of which only the front is used.
int64_t encode_workspace_bytes(const Layout& L) {
  const int64_t groups = (int64_t)L.N * L.G, narrow = (int64_t)L.N * L.groups[kNarrow];
  int64_t need = 0;
  if (narrow > 0) need += round16(narrow * 16 * 2) + round16(narrow * 2);   // a row's quads are at most its groups: 4 bytes a quad fit
  if (L.scale_mode == 1) need += round16(groups * 2) + round16(narrow);
  return need;
}

// What the zeros at the end of a hybrid-word group cost and are coded as (H16Tail).  The lowest code of those that tie, as
// the exact search takes it; its costs are rounded sums, so ties are only decided here where they are ties under any
// scale: the tied paths add the same square any number of times and otherwise zeros, which gives the same partial sums in
// every order.
static H16Tail h16_tail(double zp) {
  H16Tail t;
  t.decided = 1;
  auto sq = [&](uint32_t st) { return ((double)st - zp) * ((double)st - zp); };
  // of n states in the low bits of a code (after the bits `lead`), the cheapest of the `codes` choices
  auto least = [&](int n, uint32_t codes, uint32_t lead, float* cost_out) {
    double best = INFINITY;
    uint32_t at = 0;
    for (int pass = 0; pass < 2; ++pass)
      for (uint32_t c = 0; c < codes; ++c) {
        double cost = 0.0, one = 0.0;
        bool plain = true;   // a single value besides zero
        for (int i = 0; i < n; ++i) {
          const double e = sq(((lead | c) >> (2 * (n - 1 - i))) & 7u);
          cost += e;
          if (e != 0.0 && one != 0.0 && e != one) plain = false;
          if (e != 0.0) one = e;
        }
        if (pass == 0 && cost < best) { best = cost; at = c; }
        if (pass == 1 && cost == best && c != at) {
          double other = 0.0;
          for (int i = 0; i < n; ++i) other = std::fmax(other, sq(((lead | at) >> (2 * (n - 1 - i))) & 7u));
          if (!plain || one != other) t.decided = 0;
        }
      }
    if (cost_out) *cost_out = (float)best;
    return at;
  };
  t.zeros = least(4, 512u, 0u, nullptr);
  for (uint32_t x = 0; x < 2; ++x) t.rest[x] = least(2, 16u, x << 4, &t.cost[x]);
  return t;
}

// A matrix whose groups, 64 to a workgroup, are at most one workgroup per CU: there the time is one wavefront's, and sixteen
// lanes per group, or one narrow k-tile of the map's passes, leave it a quarter of the vectors.  Against four lanes and
// k-tiles: 256 x 4096 (256 workgroups) half zeros 400 -> 205 us (narrow), 84 -> 59 us (wide), dense 76 -> 69 and 46 -> 44 us;
// 512 x 4096 dense 6 to 17 % slower.
static bool few_blocks(int64_t blocks) { return blocks <= (int64_t)device_cus(); }

// Lanes per group: few of them do the fewest instructions (the sums of Eq. 4 are run by every lane of a group), many give
// a small matrix more wavefronts, each with fewer vectors that it searches exactly one after the other.
template <int FMT>
static void launch_groups(const EncArgs& a, int64_t blocks, hipStream_t st) {
  const dim3 grid((unsigned)blocks);
  if (blocks >= 16 * (int64_t)device_cus()) hipLaunchKernelGGL((ccq_encode_groups_kernel<FMT, 2>), grid, dim3(128), 0, st, a);
  else if (!few_blocks(blocks)) hipLaunchKernelGGL((ccq_encode_groups_kernel<FMT, 4>), grid, dim3(256), 0, st, a);
  else hipLaunchKernelGGL((ccq_encode_groups_kernel<FMT, 16>), grid, dim3(1024), 0, st, a);
}

template <int FMT>
static void launch_compress(const EncArgs& a, int64_t blocks, hipStream_t st) {
  const dim3 grid((unsigned)blocks);
  if (!few_blocks(blocks)) hipLaunchKernelGGL((ccq_encode_compress_kernel<FMT, 4>), grid, dim3(256), 0, st, a);
  else hipLaunchKernelGGL((ccq_encode_compress_kernel<FMT, 16>), grid, dim3(1024), 0, st, a);
}

int launch_encode(const Layout& L, const float* W, int64_t ldw, void* codes, void* scales, float* alpha, float* beta, void* scale_super,
                  const int32_t* meta, void* workspace, void* stream) {
  const int64_t narrow = (int64_t)L.N * L.groups[kNarrow];
  EncArgs a;
  a.tail = H16Tail{};
  a.field_max = L.h16 ? 8191.0 : 15.0;
  a.W = W;
  a.ldw = ldw;
  a.N = L.N;
  a.G = L.G;
  a.meta = L.has_map ? meta : nullptr;
  a.codes = static_cast<uint8_t*>(codes);
  a.scales = static_cast<uint16_t*>(scales);
  a.alpha = alpha;
  a.beta = beta;
  uint8_t* ws = static_cast<uint8_t*>(workspace);
  a.minmax = nullptr;
  a.rowscale = nullptr;
  if (narrow > 0) {
    a.minmax = reinterpret_cast<uint32_t*>(ws);
    ws += round16((int64_t)L.N * L.tiles[kNarrow] * 4);
    a.rowscale = reinterpret_cast<uint16_t*>(ws);
    ws += round16(narrow * 2);
  }
  a.canon_scales = L.scale_mode == 1 ? reinterpret_cast<uint16_t*>(ws) : nullptr;
  a.ssup = static_cast<uint16_t*>(scale_super);
  a.row_tile_bytes = L.row_tile_bytes;
  a.row_tile_scale_halfs = L.row_tile_scale_halfs;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const dim3 block(256);
  if (L.padded()) {
    // rows that pad the last row tile and groups that pad the last k-tile of a kind are written by no kernel below:
    // zero codes and zero scales (both arrays are whole 16-byte units: a row tile's share of either is)
    const int64_t code16 = L.row_tile_bytes * L.row_tiles / 16, scale16 = L.row_tile_scale_halfs * L.row_tiles / 8;
    if (code16 > 0) hipLaunchKernelGGL(ccq_encode_clear_kernel, dim3((unsigned)((code16 + 255) / 256)), block, 0, st, reinterpret_cast<uint4*>(codes), code16);
    if (scale16 > 0 && scales)
      hipLaunchKernelGGL(ccq_encode_clear_kernel, dim3((unsigned)((scale16 + 255) / 256)), block, 0, st, reinterpret_cast<uint4*>(scales), scale16);
  }
  // the narrow groups of every row, then the wide ones (or the hybrid words, which never mix)
  EncArgs an = a, aw = a;
  an.GK = L.groups[kNarrow];
  an.quads = (an.GK + 3) / 4;
  an.pbase = 0;
  an.mbase = 0;
  an.kind_code_off = 0;
  an.kind_scale_off = 0;
  an.zp = (double)L.zp[kNarrow];
  aw.GK = L.groups[kWide];
  aw.quads = (aw.GK + 3) / 4;
  aw.pbase = L.groups[kNarrow];
  aw.mbase = L.pgroups[kNarrow];
  aw.kind_code_off = (int64_t)L.tiles[kNarrow] * kNarrowTileBytes;
  aw.kind_scale_off = L.scale_mode == 1 ? 0 : (int64_t)L.tiles[kNarrow] * kNarrowTileScaleHalfs;
  aw.zp = (double)L.zp[kWide];
  if (L.h16) aw.tail = h16_tail(aw.zp);
  const int64_t blocks_n = (int64_t)L.row_tiles * an.quads, blocks_w = (int64_t)L.row_tiles * aw.quads;
  const bool few_n = few_blocks(blocks_n);   // of the passes over the row's map: one narrow k-tile per wavefront, or four
  const unsigned blocks_m = (unsigned)(((L.N + 3) / 4) * (few_n ? an.quads : (an.quads + 3) / 4));
  if (an.GK > 0) {
    launch_groups<kEncNarrow>(an, blocks_n, st);
    hipLaunchKernelGGL(ccq_encode_cluster_kernel, dim3((unsigned)((L.N + 3) / 4)), block, 0, st, an);
    if (few_n) hipLaunchKernelGGL(ccq_encode_finish_narrow_kernel<1>, dim3(blocks_m), block, 0, st, an);
    else hipLaunchKernelGGL(ccq_encode_finish_narrow_kernel<4>, dim3(blocks_m), block, 0, st, an);
  }
  if (aw.GK > 0) {
    if (L.h16) launch_groups<kEncH16>(aw, blocks_w, st);
    else launch_groups<kEncWide>(aw, blocks_w, st);
  }
  if (L.scale_mode == 1) {
    hipLaunchKernelGGL(ccq_encode_super_kernel, dim3((unsigned)L.N), block, 0, st, a);
    if (an.GK > 0 && few_n) hipLaunchKernelGGL(ccq_encode_compress_narrow_kernel<1>, dim3(blocks_m), block, 0, st, an);
    else if (an.GK > 0) hipLaunchKernelGGL(ccq_encode_compress_narrow_kernel<4>, dim3(blocks_m), block, 0, st, an);
    if (aw.GK > 0) {
      if (L.h16) launch_compress<kEncH16>(aw, blocks_w, st);
      else launch_compress<kEncWide>(aw, blocks_w, st);
    }
  }
  if (hipGetLastError() != hipSuccess) return CCQ_ERR_HIP;
  return CCQ_OK;
}

}  // namespace ccq

// Nearest codeword of one vector (Alg. 1, the argmin) by one lane, together with whether that answer is proven to be the
// one that the search in fp64 with its fixed order of operations gives.  Device code only.
//
// A code is a path s_0, s_1, .. of states; two neighbouring states share L - S bits and nothing else.  The best path is
// therefore found by a dynamic program over the shared bits alone (8 values for L = 6, S = 3; 4 for L = 4, S = 2; 2 for
// L = 3, S = 2): some two hundred operations in one lane instead of one over all 2^L states that fills a wavefront.
//
// Errors are counted in units of the group scale: t = v / s against the levels lv = state - zp (multiples of 0.5).  Along
// the best path the distance to the next best choice is kept for every decision.  With r = 2^-24, t carries at most
// 1.5 r |t| (see unit_scale), every difference lv - t is rounded once more, and a path of cost T = sum d_i^2 (at most four
// terms) is therefore off by at most
//   2 * 1.5 r max|t| * sum|d_i| + 6 r T  <=  3 r max|t| (T + 1) + 6 r T       (sum|d_i| <= 2 sqrt(T) <= T + 1).
// Two paths are in their true order when they differ by more than twice that; the exact search's own rounding (fp64)
// is far inside the slack of `search_margin`.  `sure` says that every decision on the path did, so that every choice the
// exact search takes on its way, ties included, is this one.  The caller hands the others to the exact search: on
// Gaussian weights 1 to 2 in 10,000 (exact ties for the most part: a group's largest weight sits on a level).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace ccq {

__device__ __forceinline__ float search_margin(float T, float tmax) { return 0x1p-24f * (8.f * tmax + 16.f) * (T + 1.f); }
constexpr float kFar = 1e30f;           // a cost that nothing real reaches (sums of it stay finite)
constexpr float kSearchMaxT = 4096.f;   // beyond this the answer is never sure

__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ float med_(float a, float b, float c) { return __builtin_amdgcn_fmed3f(a, b, c); }

// 1 / s as a sum of two fp32 numbers, so that t = v / s is rounded once
struct InvScale {
  float hi, lo;
};
__device__ __forceinline__ InvScale inv_scale(double s) {
  const double i = 1.0 / s;
  InvScale r;
  r.hi = (float)i;
  r.lo = (float)(i - (double)r.hi);
  return r;
}
__device__ __forceinline__ float unit_scale(float v, const InvScale& i) { return fma_(v, i.hi, v * i.lo); }

// Of levels `step` apart the nearest was taken, `off` steps from the wanted place (a place outside the levels counts as
// the outermost level): how much more the next nearest costs, at least.  The place is known to a few units in its last
// place of fp32 (1e-4 of step^2 is more than that comes to).
__device__ __forceinline__ float nearest_gap(float step, float off) { return step * step * (0.9999f - 2.f * fabsf(off)); }

// the smallest two of what was seen, and the index of the smallest
struct Best2 {
  float best = kFar, second = kFar;
  int at = 0;
  __device__ __forceinline__ void see(float x, int i) {
    at = x < best ? i : at;
    second = med_(best, second, x);
    best = fminf(best, x);
  }
  __device__ __forceinline__ float gap() const { return second - best; }
};

// v[i] by selects (values, not places: an index into an array would put the array in memory)
template <int N, typename T>
__device__ __forceinline__ T pick(const T (&v)[N], int i) {
  T c[N];
#pragma unroll
  for (int k = 0; k < N; ++k) c[k] = v[k];
  T r = c[0];
#pragma unroll
  for (int k = 1; k < N; ++k) {
    const bool here = i == k;
    r = here ? c[k] : r;
  }
  return r;
}

struct FastCode {
  uint32_t code;
  bool sure;
};

template <int NV>
__device__ __forceinline__ float max_abs(const float (&t)[NV]) {
  float m = fabsf(t[0]);
#pragma unroll
  for (int i = 1; i < NV; ++i) m = fmaxf(m, fabsf(t[i]));
  return m;
}

// (L=6,N=4,S=3): code = (a, b, c, d, e), three bits each; states (a,b), (b,c), (c,d), (d,e).
// Of the eight values of b only the one whose block of states (8b .. 8b+7) holds t[1] and its two neighbours are looked
// at, the same for c (by t[2]) and d (by t[3]): every other value costs at least the square of the distance from t to
// the nearest state of the blocks left out (8 or more), and the answer is only called sure when the best path is
// cheaper than that.  a and e are free given b and d: the nearest of eight states spaced by eight, and by one.
__device__ __forceinline__ FastCode fast_narrow(const float (&t)[4], float zp) {
  float in[3], apart = kFar;  // block of t[1], t[2], t[3]; distance to the nearest state outside the three blocks
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const float u = t[i + 1] + zp;
    in[i] = med_(floorf(u * 0.125f), 0.f, 7.f);
    const float f = fma_(in[i], -8.f, u);
    apart = fminf(apart, in[i] >= 2.f ? f + 9.f : kFar);
    apart = fminf(apart, in[i] <= 5.f ? 16.f - f : kFar);
  }
  float b[3], a[3], F[3], gapF[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    b[k] = in[0] + (float)(k - 1);
    const float bz = b[k] - zp;
    const float q = med_((bz - t[0]) * -0.125f, 0.f, 7.f);
    a[k] = rintf(q);
    const float d = fma_(a[k], 8.f, bz) - t[0];
    F[k] = d * d;
    gapF[k] = nearest_gap(8.f, a[k] - q);
  }
  F[0] = in[0] < 1.f ? kFar : F[0];
  F[2] = in[0] > 6.f ? kFar : F[2];
  Best2 G[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const float cz = in[1] + ((float)(j - 1) - zp);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const float d = fma_(b[k], 8.f, cz) - t[1];
      G[j].see(fma_(d, d, F[k]), k);
    }
  }
  G[0].best = in[1] < 1.f ? kFar : G[0].best;
  G[2].best = in[1] > 6.f ? kFar : G[2].best;
  Best2 H[3], all;
  float e[3], gapE[3];
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    const float dl = in[2] + (float)(l - 1), dz = dl - zp;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const float d = fma_(in[1] + (float)(j - 1), 8.f, dz) - t[2];
      H[l].see(fma_(d, d, G[j].best), j);
    }
    const float lo = fma_(dl, 8.f, -zp);
    const float q = med_(t[3] - lo, 0.f, 7.f);
    e[l] = rintf(q);
    const float d = (lo + e[l]) - t[3];
    gapE[l] = nearest_gap(1.f, e[l] - q);
    float T = fma_(d, d, H[l].best);
    if (l == 0) T = in[2] < 1.f ? kFar : T;
    if (l == 2) T = in[2] > 6.f ? kFar : T;
    all.see(T, l);
  }
  const int l = all.at;
  const float gaps_l[3] = {fminf(gapE[0], H[0].gap()), fminf(gapE[1], H[1].gap()), fminf(gapE[2], H[2].gap())};
  const int at_l[3] = {H[0].at, H[1].at, H[2].at};
  const int j = pick(at_l, l);
  const float gaps_j[3] = {G[0].second - G[0].best, G[1].gap(), G[2].second - G[2].best};
  const int at_j[3] = {G[0].at, G[1].at, G[2].at};
  const int k = pick(at_j, j);
  const float gap = fminf(fminf(all.gap(), pick(gaps_l, l)), fminf(pick(gaps_j, j), pick(gapF, k)));
  const float tmax = max_abs(t), m = search_margin(all.best, tmax);
  float c = fma_(pick(a, k), 8.f, pick(b, k));
  c = fma_(c, 8.f, in[1] + (float)(j - 1));
  c = fma_(c, 8.f, in[2] + (float)(l - 1));
  c = fma_(c, 8.f, pick(e, l));
  FastCode r;
  r.code = (uint32_t)c & 0x7FFFu;
  r.sure = gap > m && all.best + m < apart * apart * 0.999f && tmax <= kSearchMaxT;
  return r;
}

// The first state of a code with few shared bits: per value o of the bits that it passes on, the nearest state o + NI h.
template <int L, int S>
__device__ __forceinline__ void first_states(float t0, float zp, float (&cost)[1 << (L - S)], float (&gap)[1 << (L - S)], float (&h)[1 << (L - S)]) {
  constexpr int NI = 1 << (L - S), kTop = (1 << S) - 1;
#pragma unroll
  for (int o = 0; o < NI; ++o) {
    const float oz = (float)o - zp;
    const float q = med_((oz - t0) * (-1.f / NI), 0.f, (float)kTop);
    h[o] = rintf(q);
    const float d = fma_(h[o], (float)NI, oz) - t0;
    cost[o] = d * d;
    gap[o] = nearest_gap((float)NI, h[o] - q);
  }
}

// A code whose states after the first are given per value of the passed-on bits, with their cost.
template <int L, int NV, int S>
__device__ __forceinline__ FastCode fast_first(float t0, float zp, const float* rest_cost, const uint32_t* rest) {
  constexpr int NI = 1 << (L - S);
  float M[NI], gap0[NI], h0[NI];
  first_states<L, S>(t0, zp, M, gap0, h0);
  Best2 all;
  uint32_t codes[NI];
#pragma unroll
  for (int o = 0; o < NI; ++o) {
    all.see(M[o] + rest_cost[o], o);
    codes[o] = (((uint32_t)h0[o] * NI + (uint32_t)o) << (S * (NV - 1))) | rest[o];
  }
  FastCode r;
  r.code = pick(codes, all.at) & ((1u << (L + (NV - 1) * S)) - 1u);
  r.sure = fminf(all.gap(), pick(gap0, all.at)) > search_margin(all.best, fabsf(t0)) && fabsf(t0) <= kSearchMaxT;
  return r;
}

// The codes with few shared bits, all values of them: (L=4,N=3,S=2) and the two halves (3,3,2), (3,4,2) of the hybrid word.
template <int L, int NV, int S>
__device__ __forceinline__ FastCode fast_small(const float (&t)[NV], float zp) {
  constexpr int NI = 1 << (L - S);      // values of the shared bits
  constexpr int NM = (1 << S) / NI;     // fresh bits that are not passed on, between the two shared fields of a state
  constexpr int kTop = (1 << S) - 1;
  float M[NI], gap0[NI], h0[NI];
  first_states<L, S>(t[0], zp, M, gap0, h0);
  Best2 mid[NV - 2][NI];
#pragma unroll
  for (int i = 1; i < NV - 1; ++i) {
#pragma unroll
    for (int o = 0; o < NI; ++o)
#pragma unroll
      for (int x = 0; x < NI; ++x)
#pragma unroll
        for (int m = 0; m < NM; ++m) {
          const float d = ((float)((x << S) | (m * NI) | o) - zp) - t[i];
          mid[i - 1][o].see(fma_(d, d, M[x]), x * NM + m);
        }
#pragma unroll
    for (int o = 0; o < NI; ++o) M[o] = mid[i - 1][o].best;
  }
  Best2 all;
  float last[NI], gapT[NI];
#pragma unroll
  for (int x = 0; x < NI; ++x) {  // last state: any fresh bits
    const float lo = (float)(x << S) - zp;
    const float q = med_(t[NV - 1] - lo, 0.f, (float)kTop);
    last[x] = rintf(q);
    const float d = (lo + last[x]) - t[NV - 1];
    gapT[x] = nearest_gap(1.f, last[x] - q);
    all.see(fma_(d, d, M[x]), x);
  }
  int o = all.at;
  float gap = fminf(all.gap(), pick(gapT, o));
  uint32_t code = (uint32_t)pick(last, o);
#pragma unroll
  for (int i = NV - 2; i >= 1; --i) {
    int at[NI];
    float g[NI];
#pragma unroll
    for (int q = 0; q < NI; ++q) {
      at[q] = mid[i - 1][q].at;
      g[q] = mid[i - 1][q].gap();
    }
    gap = fminf(gap, pick(g, o));
    const int xm = pick(at, o);
    code |= (uint32_t)((xm % NM) * NI + o) << (S * (NV - 1 - i));  // the fresh bits of state i
    o = xm / NM;
  }
  gap = fminf(gap, pick(gap0, o));
  code |= ((uint32_t)pick(h0, o) * NI + (uint32_t)o) << (S * (NV - 1));
  const float tmax = max_abs(t);
  FastCode r;
  r.code = code & ((1u << (L + (NV - 1) * S)) - 1u);
  r.sure = gap > search_margin(all.best, tmax) && tmax <= kSearchMaxT;
  return r;
}

}  // namespace ccq

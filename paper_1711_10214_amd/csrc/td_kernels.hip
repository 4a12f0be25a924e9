// Time-domain (classical) ASHRT / AASHRT operator pair, the O(P nx^2 nt)
// reference the Stolt operator is compared against (thesis Chapter 3, the
// ASHRT and AASHRT rows of the Radon-operator table; Chapter 6, equations
// ch6_AASHRT_forward and ch6_AASHRT_adjoint; Chapter 5's speed comparison).
//
// A model sample at apex time tau (samples), apex trace xa and panel p lies
// on the data curve T = n0_p + sqrt(tau^2 + (x - xa)^2 q_p), q_p =
// (dx / (v_p dt))^2, read with linear interpolation: the adjoint gathers
// m[p][xa][tau] = sum_x (1 - f) d[x][i0] + f d[x][i0 + 1] (i0 = floor T,
// f = T - i0, samples outside [0, nt) dropped); the forward is its exact
// transpose written as a gather: d[x][t] = sum_{p, xa, tau} hat(T - t)
// m[p][xa][tau] with hat(s) = max(0, 1 - |s|), over the tau whose curve
// passes within one sample of t (found from the inverse of T).  T is good to
// FP64 rounding of its square (its fractional part is the interpolation
// weight); sums are FP32.  No atomics: every output has one owner.
//
// T depends on the panel and on the distance h = |x - xa| alone, so one set
// of curve times and weights serves every (x, xa) pair at that distance: a
// wave takes consecutive times of K neighbouring traces and walks the
// distances, and at each one uses the weights for up to 2 K pairs (both
// sides).  32 panels of 512 x 128 samples: forward 7140 -> 660 us, adjoint
// 377 -> 150 us against one curve time per pair (and per candidate tau in
// the forward).  The forward is bound by vector instructions (89 % of its
// cycles), under a quarter of them the pairs' products; waves near an apex,
// where many tau fall on one time, take several rounds.  The adjoint has one
// issued 72 % of its cycles; small ones are a chain of latencies, one a distance,
// which several distances at a time overlap (8 panels of 256 x 64: 29 us with one
// curve time per pair, 67 with one distance at a time, 19 with four).
#include "kernels.h"

#include <type_traits>

namespace ashrt {

// (dx / (v dt))^2 from the panel's Stolt bin scale c2 = (v ntp dt / (nxp dx))^2
// (0 for v = 0, which restricts the curve to its apex trace).
__device__ __forceinline__ double td_q(const PanelDev& P, const GatherDev& G) {
  if (P.c2 <= 0.0) return -1.0;
  const double r = (double)G.ntp / (double)G.nxp;
  return r * r / P.c2;
}

constexpr int kTdFwdWaves = 16;  // waves that share a forward tile's panels and distances
constexpr int kTdAdjWaves = 4;   // adjoint waves per workgroup
constexpr int kTdMaxTraces = 4096;  // longest x transform a plan takes

// sqrt(T2) to FP64 rounding: two Newton steps, their residuals in FP64, from an
// FP32 root (good to 1e-15 for a root below that, and 0 for 0).  T2 is below
// 2^26 (callers test it against the record first).
__device__ __forceinline__ double td_root(double T2) {
  const float t = (float)T2, i = __builtin_amdgcn_rsqf(fmaxf(t, 1e-30f));
  const double s0 = (double)(t * i), h = (double)(0.5f * i);
  const double s1 = fma(fma(-s0, s0, T2), h, s0);
  return fma(fma(-s1, s1, T2), h, s1);
}

// n consecutive floats at a 4-byte aligned address, as one load.
template <int N>
__device__ __forceinline__ void td_load(float (&v)[N], const float* row, unsigned off) {
  __builtin_memcpy(v, reinterpret_cast<const char*>(row) + off, 4 * N);
}

// A wave's sums over 64 apex times of K neighbouring apexes of one panel.  H
// distances at a time, so that their roots and loads overlap: the walk is a
// chain of latencies where few waves run.  Pair k of distance h is trace x0 + k
// + h, pair K + k is x0 + k - h (h = 0: only the first half), taken where the
// trace is in the gather and live; lane 2 K j + k looks pair k of the j-th
// distance up, and the ballot is wave-uniform.  Lanes without a curve time in
// the record, and the sample before the record's last, weigh 0; SAFE leaves
// those out, which differs only where a sample is not finite.
template <int K, int H, bool SAFE>
__device__ __forceinline__ void td_adjoint_wave(const TdArgs& A, const PanelDev& P, double q, int nt, int nx, int tau,
                                                int x0, const uint8_t* live, float (&acc)[K]) {
  constexpr unsigned kAll = (unsigned)((1ull << 2 * K * H) - 1);
  static_assert(2 * K * H <= 16, "one lane and one bit a pair");
#pragma unroll
  for (int k = 0; k < K; ++k) acc[k] = 0.f;
  const double t2 = (double)tau * (double)tau;
  const double lim = (double)(nt - P.n0) * (double)(nt - P.n0);
  const int hmax = q < 0.0 ? 0 : max(x0 + K - 1, nx - 1 - x0);
  const int lane = (int)threadIdx.x & 63, lj = lane / (2 * K), lk = lane % K;
  const bool down = lane % (2 * K) >= K;
  const bool mine = lane < 2 * K * H && x0 + lk < nx && (q >= 0.0 || lj == 0), self = down && lj == 0;
  const int xl = x0 + lk + (down ? -lj : lj);
  for (int h0 = 0; h0 <= hmax; h0 += H) {
    const int x = xl + (down ? -h0 : h0);
    bool use = mine && (unsigned)x < (unsigned)nx && !(self && h0 == 0);
    if (A.tmask && use) use = live[x] != 0;
    const unsigned ok = (unsigned)__ballot(use);
    float v[H][2 * K][2], w0[H], w1[H];
    bool on[H], last[H];
    unsigned off[H];
#pragma unroll
    for (int j = 0; j < H; ++j) {
      const double hd = (double)(h0 + j), T2 = q < 0.0 ? t2 : fma(hd * hd, q, t2);
      on[j] = tau < nt && T2 < lim;            // T < nt
      if (j == 0 && !__any(on[0])) return;     // T rises with h
      const double T = td_root(T2), fl = floor(T);
      const int i0 = on[j] ? P.n0 + (int)fl : 0;
      const float f = (float)(T - fl), e = 1.f - f;
      last[j] = i0 > nt - 2;
      on[j] = on[j] && i0 < nt;
      w0[j] = on[j] && !last[j] ? e : 0.f;
      w1[j] = on[j] ? (last[j] ? e : f) : 0.f;
      off[j] = 4u * (unsigned)min(i0, nt - 2);
    }
    const float* const up = A.d + (long long)(x0 + h0) * nt;  // rows x0 + h + k and x0 - h + k
    const float* const dn = A.d + (long long)(x0 - h0) * nt;
    auto load = [&](int j, int k) {
      td_load(v[j][k], (k < K ? up + (long long)(k + j) * nt : dn + (long long)(k - K - j) * nt), off[j]);
    };
    auto add = [&](int j, int k) {
      const float a = SAFE && (!on[j] || last[j]) ? 0.f : v[j][k][0], b = SAFE && !on[j] ? 0.f : v[j][k][1];
      acc[k % K] = fmaf(w1[j], b, fmaf(w0[j], a, acc[k % K]));
    };
    if (ok == kAll) {
#pragma unroll
      for (int i = 0; i < 2 * K * H; ++i) load(i / (2 * K), i % (2 * K));
#pragma unroll
      for (int i = 0; i < 2 * K * H; ++i) add(i / (2 * K), i % (2 * K));
    } else {
#pragma unroll
      for (int i = 0; i < 2 * K * H; ++i)
        if (ok >> i & 1) load(i / (2 * K), i % (2 * K));
#pragma unroll
      for (int i = 0; i < 2 * K * H; ++i)
        if (ok >> i & 1) add(i / (2 * K), i % (2 * K));
    }
  }
}

// Adjoint: a wave owns 64 apex times of K neighbouring apexes of one panel.
template <int K, int H>
__global__ __launch_bounds__(64 * kTdAdjWaves) void k_td_adjoint(TdArgs A) {
  __shared__ uint8_t live[kTdMaxTraces];
  const GatherDev G = A.gd[0];
  const int nt = G.nt, nx = G.nx;
  const int ntt = (nt + 63) / 64, nxt = (nx + K - 1) / K;
  if (A.tmask) {
    for (int x = threadIdx.x; x < nx; x += 64 * kTdAdjWaves) live[x] = A.tmask[x];
    __syncthreads();
  }
  const int lane = (int)threadIdx.x & 63;
  const int id = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * kTdAdjWaves + (threadIdx.x >> 6)));
  if (id >= G.npanel * nxt * ntt) return;
  // early times see more traces inside the record: panels and apexes vary
  // fastest, so that the longest waves start first
  const int tb = id / (G.npanel * nxt), q2 = id - tb * (G.npanel * nxt), x0 = (q2 % nxt) * K, p = q2 / nxt;
  const PanelDev P = A.panels[G.panel_off + p];
  const double q = td_q(P, G);
  const int tau = tb * 64 + lane;
  float acc[K];
#pragma unroll
  for (int k = 0; k < K; ++k) acc[k] = 0.f;
  if (P.n0 < nt) {
    td_adjoint_wave<K, H, false>(A, P, q, nt, nx, tau, x0, live, acc);
    bool fin = true;
#pragma unroll
    for (int k = 0; k < K; ++k) fin = fin && isfinite(acc[k]);
    if (__any(!fin)) td_adjoint_wave<K, H, true>(A, P, q, nt, nx, tau, x0, live, acc);
  }
  if (tau < nt) {
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (x0 + k < nx) A.m[((long long)p * nx + x0 + k) * nt + tau] = acc[k];
  }
}

// One wave's share of a forward tile of 32 times: its two halves take two
// neighbouring distances, and the (panel, distance pair) list is dealt to the
// kTdFwdWaves waves in turn.  The tau of a curve within one sample of
// t are a run of about 2 / slope (slope = dT / dtau <= 1): taken four at a
// time, with weights computed once per (panel, distance), and one four-sample
// load per pair.  SAFE leaves out samples without weight; otherwise they are
// multiplied by zero, which differs only where a sample is not finite.
template <int K, bool SAFE>
__device__ __forceinline__ void td_forward_wave(const TdArgs& A, const GatherDev& G, int tb, int x0, int wave,
                                                float (&acc)[K]) {
  const int nt = G.nt, nx = G.nx;
  const int half = ((int)threadIdx.x >> 5) & 1;
  const int t = tb * 32 + ((int)threadIdx.x & 31);
#pragma unroll
  for (int k = 0; k < K; ++k) acc[k] = 0.f;
  int turn = 0;
  for (int p = 0; p < G.npanel; ++p) {
    const PanelDev P = A.panels[G.panel_off + p];
    if (P.n0 >= nt) continue;
    const double q = td_q(P, G);
    // last distance whose curve starts before the tile's last time + 1
    const double smax = (double)(min(tb * 32 + 31, nt - 1) + 1 - P.n0);
    if (smax <= 0.0) continue;
    int hmax = q < 0.0 ? 0 : max(x0 + K - 1, nx - 1 - x0);
    if (q > 0.0) hmax = (int)fmin((double)hmax, smax / sqrt(q) + 1.0);
    hmax = __builtin_amdgcn_readfirstlane(hmax);
    const float* __restrict__ mp = A.m + (long long)p * nx * nt;
    const int ts = t - P.n0;
    const double s0 = (double)ts, s1 = (double)(ts - 1), s2 = (double)(ts + 1);
    const double s12 = s1 * s1, s22 = s2 * s2;
    int hh = wave - turn;
    if (hh < 0) hh += kTdFwdWaves;
    for (; 2 * hh <= hmax; hh += kTdFwdWaves) {
      const int h = 2 * hh + half;
      const double h2 = q < 0.0 ? 0.0 : (double)h * (double)h * q;
      // tau with t - 1 < T < t + 1 lie in [lo, hi] (FP32 roots are good to
      // 5e-4 here, the margins cover that)
      const bool on = t < nt && ts >= 0 && s22 > h2 && h <= hmax;
      int lo = 0, hi = -1;
      if (on) {
        const float a = (float)(s12 - h2);
        lo = (ts > 1 && a > 0.f) ? max(0, (int)ceilf(__builtin_amdgcn_sqrtf(a) - 2e-3f)) : 0;
        hi = min(nt - 1, (int)floorf(__builtin_amdgcn_sqrtf((float)(s22 - h2)) + 2e-3f));
      }
      // both halves' pairs all inside the gather
      const bool inside = hh > 0 && x0 - 2 * hh - 1 >= 0 && x0 + K - 1 + 2 * hh + 1 < nx && nt >= 4;
      const float* row = mp + (long long)x0 * nt;
      for (int c = lo; c <= hi; c += 4) {
        const int b = max(0, min(c, nt - 4));  // the load stays in the row (nt >= 4)
        float w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          // the weight 1 - |T - t| in FP64, rounded once
          const int tau = b + i;
          const double td = (double)tau;
          const float ww = (float)(1.0 - fabs(td_root(fma(td, td, h2)) - s0));
          w[i] = (tau >= c && tau <= hi) ? fmaxf(ww, 0.f) : 0.f;
        }
        auto add = [&](float& a, const float (&v)[4]) {
#pragma unroll
          for (int i = 0; i < 4; ++i) a = fmaf(w[i], SAFE && !(w[i] > 0.f) ? 0.f : v[i], a);
        };
        if (inside) {
          // byte offsets from the tile's first row (4 nx nt < 2^31)
          const unsigned up = 4u * (unsigned)(h * nt + b), dn = 4u * (unsigned)b - 4u * (unsigned)(h * nt);
          float v[2 * K][4];
#pragma unroll
          for (int k = 0; k < K; ++k) {
            td_load(v[k], row + (long long)k * nt, up);
            td_load(v[K + k], mp + (long long)k * nt, dn + 4u * (unsigned)(x0 * nt));
          }
#pragma unroll
          for (int k = 0; k < 2 * K; ++k) add(acc[k % K], v[k]);
        } else {
#pragma unroll
          for (int k = 0; k < 2 * K; ++k) {
            const int xa = k < K ? x0 + k + h : x0 + k - K - h;
            if (x0 + k % K < nx && xa >= 0 && xa < nx && (h > 0 || k < K)) {
              const float* mr = mp + (long long)xa * nt;
              float v[4];
#pragma unroll
              for (int i = 0; i < 4; ++i) v[i] = mr[min(b + i, nt - 1)];
              add(acc[k % K], v);
            }
          }
        }
      }
    }
    turn = (turn + hmax / 2 + 1) % kTdFwdWaves;
  }
}

// Forward: a workgroup owns 32 times of K neighbouring traces; its waves add
// their sums through LDS in wave order.
template <int K>
__global__ __launch_bounds__(64 * kTdFwdWaves) void k_td_forward(TdArgs A) {
  __shared__ float part[kTdFwdWaves][K][64];
  const GatherDev G = A.gd[0];
  const int nt = G.nt, nx = G.nx;
  const int nxt = (nx + K - 1) / K;
  const int lane = (int)threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  // late times see more traces: start them first
  const int tb = (nt + 31) / 32 - 1 - (int)blockIdx.x / nxt, x0 = ((int)blockIdx.x % nxt) * K;
  float acc[K];
  td_forward_wave<K, false>(A, G, tb, x0, wave, acc);
  bool fin = true;
#pragma unroll
  for (int k = 0; k < K; ++k) fin = fin && isfinite(acc[k]);
  if (__any(!fin)) td_forward_wave<K, true>(A, G, tb, x0, wave, acc);
#pragma unroll
  for (int k = 0; k < K; ++k) part[wave][k][lane] = acc[k];
  __syncthreads();
  for (int i = threadIdx.x; i < K * 32; i += 64 * kTdFwdWaves) {
    const int k = i >> 5, l = i & 31, x = x0 + k, tt = tb * 32 + l;
    if (x >= nx || tt >= nt) continue;
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < kTdFwdWaves; ++w) s += part[w][k][l] + part[w][k][l + 32];
    A.d[(long long)x * nt + tt] = (A.tmask && A.tmask[x] == 0) ? 0.f : s;
  }
}

hipError_t launch_td(const TdArgs& a, bool forward, int nt, int nx, int npanel, hipStream_t s) {
  if (forward) {
    // the widest tile (fewest weight evaluations per pair) that still gives
    // every CU two workgroups, a late and an early one
    const dim3 b(64 * kTdFwdWaves);
    auto tiles = [&](int K) { return (unsigned)((nt + 31) / 32 * ((nx + K - 1) / K)); };
    if (tiles(8) >= 512) hipLaunchKernelGGL(k_td_forward<8>, dim3(tiles(8)), b, 0, s, a);
    else if (tiles(4) >= 512) hipLaunchKernelGGL(k_td_forward<4>, dim3(tiles(4)), b, 0, s, a);
    else hipLaunchKernelGGL(k_td_forward<2>, dim3(tiles(2)), b, 0, s, a);
  } else {
    auto waves = [&](int K) { return (long long)((nt + 63) / 64) * ((nx + K - 1) / K) * npanel; };
    if (waves(1) > 0x7fffff00LL) return hipErrorInvalidValue;
    auto go = [&](auto k, auto h) {
      constexpr int K = decltype(k)::value, H = decltype(h)::value;
      hipLaunchKernelGGL((k_td_adjoint<K, H>), dim3((unsigned)((waves(K) + kTdAdjWaves - 1) / kTdAdjWaves)),
                         dim3(64 * kTdAdjWaves), 0, s, a);
    };
    // 4 apexes a wave share the most weights, once their waves fill the card (7 a
    // SIMD); fewer waves are latency, and 2 apexes with four distances at a time
    // give more of them more in flight (us, 4 and 2 apexes: 512 x 128, 32 panels
    // (8192 waves of 4) 150 and 170; 700 x 150, 17 (7106) 169 and 157; 512 x 128, 8
    // (2048) 62 and 55; 256 x 64, 8 (512) 30 and 19)
    if (waves(4) >= 7168) go(std::integral_constant<int, 4>{}, std::integral_constant<int, 2>{});
    else go(std::integral_constant<int, 2>{}, std::integral_constant<int, 4>{});
  }
  return hipGetLastError();
}

}  // namespace ashrt

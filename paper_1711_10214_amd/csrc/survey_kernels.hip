// Numerical blending and pseudo-deblending of a multi-source survey (thesis
// Chapter 2, equations ch2_blending and pseudodeblending_equ), and the
// source <-> receiver re-sort of a cube.
//
// Blending:  b[r][tau] = sum_s D[s][r][tau - T_s]  (0 <= tau - T_s < nt),
// written as a gather (one owner per record sample, no atomics, sources added
// in index order);
// pseudo-deblending (its adjoint): D~[s][r][t] = b[r][T_s + t], written in
// either the source-major [s][r][t] or the receiver-major [r][s][t] order
// (the latter is the batch of common receiver gathers the separation
// consumes, so no separate sort is needed).
//
// All three move each byte once and are bound by memory: a thread takes four
// consecutive samples with one 16-byte access each way (firing times and odd
// sizes leave them at 4-byte alignment, which the hardware takes), and its
// indices need one 32-bit division.  Blending first lists the sources whose
// shots reach the wave's stretch of the record, a handful, instead of testing
// every source at every sample, and keeps the loads of several in flight (many
// shots over every sample, 200 x 200 x 128 fired 5 samples apart: 24 us with every
// source tested, 76 with one listed source at a time, 12).  128 x 128 x 1024:
// blending 247 -> 25 us, pseudo-deblending 41 -> 20 us, re-sorting 37 -> 19 us
// (4, 5 and 7 TB/s).
#include "kernels.h"

#include <algorithm>

namespace ashrt {

constexpr int kBlendList = 512;           // sources tested at a time
constexpr int kBlendRows = 8;             // most receivers per workgroup

__device__ __forceinline__ float4 load4(const float* p) {
  float4 v;
  __builtin_memcpy(&v, p, 16);
  return v;
}
__device__ __forceinline__ void store4(float* p, float4 v) { __builtin_memcpy(p, &v, 16); }

// Adds the n listed sources' samples to a thread's Q record samples, in list
// order, the loads of U sources in flight.  (A source that does not reach a
// sample adds zero, which leaves the sum as it is.)
template <int Q, int U>
__device__ __forceinline__ void blend_add(float (&acc)[Q], const float* __restrict__ D, int r, int nr, int nt, int tau,
                                          const int* src, const int* at, int n) {
  for (int i = 0; i < n; i += U) {
    float v[U][Q];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = min(i + u, n - 1), t = i + u < n ? tau - at[e] : nt;
      const float* __restrict__ d = D + ((long long)src[e] * nr + r) * nt + t;
#pragma unroll
      for (int k = 0; k < Q; ++k) v[u][k] = 0.f;
      if (Q == 4 && t >= 0 && t + 4 <= nt) {
        __builtin_memcpy(v[u], d, 4 * Q);
      } else if (t > -Q && t < nt) {
#pragma unroll
        for (int k = 0; k < Q; ++k)
          if (t + k >= 0 && t + k < nt) v[u][k] = d[k];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int k = 0; k < Q; ++k) acc[k] += v[u][k];
  }
}

// A wave owns 64 Q record samples of its receivers and lists the sources whose
// shots reach them.
template <int Q, int U>
__global__ __launch_bounds__(kThreads) void k_blend(const float* __restrict__ D, int ns, int nr, int nt,
                                                   const int* __restrict__ fire, float* __restrict__ b, int nrec,
                                                   int rows) {
  constexpr int kWave = 64 * Q, kWaves = kThreads / 64;
  __shared__ int lists[kWaves][2][kBlendList];
  const int lane = (int)threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  int *const src = lists[wave][0], *const at = lists[wave][1];
  const long long lo = ((long long)blockIdx.x * kWaves + wave) * kWave, hi = min(nrec - lo, (long long)kWave);
  if (hi <= 0) return;                     // samples lo .. lo + hi - 1
  const int left = (int)hi - Q * lane;     // of the lane's samples tau, tau + 1, ...
  const int tau = (int)lo + (left > 0 ? Q * lane : 0);
  for (int s0 = 0; s0 < ns; s0 += kBlendList) {
    // of the sources s0 .. s0 + kBlendList - 1, in index order
    int f[kBlendList / 64], n = 0;
#pragma unroll
    for (int u = 0; u < kBlendList / 64; ++u) f[u] = fire[min(s0 + 64 * u + lane, ns - 1)];
#pragma unroll
    for (int u = 0; u < kBlendList / 64; ++u) {
      const int s = s0 + 64 * u + lane;
      const bool in = s < ns && f[u] < lo + hi && (long long)f[u] + nt > lo;
      const unsigned long long m = __ballot(in);
      if (in) {
        const int off = n + __popcll(m & ((1ull << lane) - 1));
        src[off] = s;
        at[off] = f[u];
      }
      n += __popcll(m);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    for (int rb = (int)blockIdx.y; left > 0 && rb * rows < nr; rb += gridDim.y) {
      for (int r = rb * rows; r < min(nr, (rb + 1) * rows); ++r) {
        float* __restrict__ out = b + (long long)r * nrec + tau;
        float acc[Q];
#pragma unroll
        for (int k = 0; k < Q; ++k) acc[k] = s0 && k < left ? out[k] : 0.f;
        blend_add<Q, U>(acc, D, r, nr, nt, tau, src, at, n);
        if (left >= Q) {
          __builtin_memcpy(out, acc, 4 * Q);
        } else {
#pragma unroll
          for (int k = 0; k < Q; ++k)
            if (k < left) out[k] = acc[k];
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
}

// Rows of nt samples: inner rows j = j0 .. nj - 1 of each outer index o; quads
// of samples per row.  Returns false past the end.
__device__ __forceinline__ bool quad_of(int j0, int nj, int nt, int* j, int* t) {
  const unsigned q = ((unsigned)nt + 3) / 4;
  const unsigned i = blockIdx.x * blockDim.x + threadIdx.x;
  const unsigned k = i / q;
  *t = 4 * (int)(i - k * q);
  *j = j0 + (int)k;
  return k < (unsigned)(nj - j0);
}

__global__ __launch_bounds__(kThreads) void k_deblend(const float* __restrict__ b, int ns, int nr, int nt,
                                                     const int* __restrict__ fire, int nrec, float* __restrict__ out,
                                                     int receiver_major, int j0) {
  int j, t;
  if (!quad_of(j0, receiver_major ? ns : nr, nt, &j, &t)) return;
  const int no = receiver_major ? nr : ns, nj = receiver_major ? ns : nr;
  for (int o = blockIdx.y; o < no; o += gridDim.y) {
    const int s = receiver_major ? j : o, r = receiver_major ? o : j;
    const int f = fire[s];
    const long long tau = (long long)f + t;
    const float* __restrict__ p = b + (long long)r * nrec + tau;
    float* __restrict__ q = out + ((long long)o * nj + j) * nt + t;
    if (t + 4 <= nt && tau >= 0 && tau + 4 <= nrec) {
      store4(q, load4(p));
    } else {
      for (int k = 0; k < 4 && t + k < nt; ++k) q[k] = (tau + k >= 0 && tau + k < nrec) ? p[k] : 0.f;
    }
  }
}

__global__ __launch_bounds__(kThreads) void k_resort(const float* __restrict__ in, int na, int nb, int nt,
                                                    float* __restrict__ out, int j0) {
  int a, t;
  if (!quad_of(j0, na, nt, &a, &t)) return;
  for (int bb = blockIdx.y; bb < nb; bb += gridDim.y) {  // out[bb][a][t] = in[a][bb][t]
    const float* __restrict__ p = in + ((long long)a * nb + bb) * nt + t;
    float* __restrict__ q = out + ((long long)bb * na + a) * nt + t;
    if (t + 4 <= nt) {
      store4(q, load4(p));
    } else {
      for (int k = 0; t + k < nt; ++k) q[k] = p[k];
    }
  }
}

// Runs f(grid, j0) over nj rows of nt samples in quads by no outer indices:
// one launch, or slices of j where the index would pass 32 bits.
template <class F>
static hipError_t quad_launch(int nj, int nt, int no, F&& f) {
  const long long q = ((long long)nt + 3) / 4;
  const int step = (int)std::min<long long>(nj, std::max(1LL, 0x7fffff00LL / q));
  for (int j0 = 0;; j0 += step) {
    const long long n = std::min(step, nj - j0) * q;
    f(dim3((unsigned)((n + kThreads - 1) / kThreads), (unsigned)std::min(no, 65535)), j0);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || nj - j0 <= step) return e;
  }
}

hipError_t launch_blend(const float* D, int ns, int nr, int nt, const int* fire, float* b, int nrec, hipStream_t s) {
  // four samples a thread once that gives 1024 workgroups, else one; receivers
  // share a workgroup's source list while enough workgroups remain
  auto tiles = [&](int q) { return ((long long)nrec + q * kThreads - 1) / (q * kThreads); };
  const bool wide = tiles(4) * nr >= 1024;
  const long long n = tiles(wide ? 4 : 1);
  const int rows = (int)std::max(1LL, std::min<long long>(kBlendRows, n * nr / 1024));
  const dim3 grid((unsigned)n, (unsigned)std::min((nr - 1) / rows + 1, 65535));
  if (wide) hipLaunchKernelGGL((k_blend<4, 4>), grid, dim3(kThreads), 0, s, D, ns, nr, nt, fire, b, nrec, rows);
  else hipLaunchKernelGGL((k_blend<1, 8>), grid, dim3(kThreads), 0, s, D, ns, nr, nt, fire, b, nrec, rows);
  return hipGetLastError();
}

hipError_t launch_deblend(const float* b, int ns, int nr, int nt, const int* fire, int nrec, float* out, int rmaj,
                          hipStream_t s) {
  return quad_launch(rmaj ? ns : nr, nt, rmaj ? nr : ns, [&](dim3 g, int j0) {
    hipLaunchKernelGGL(k_deblend, g, dim3(kThreads), 0, s, b, ns, nr, nt, fire, nrec, out, rmaj, j0);
  });
}

hipError_t launch_resort(const float* in, int na, int nb, int nt, float* out, hipStream_t s) {
  return quad_launch(na, nt, nb, [&](dim3 g, int j0) {
    hipLaunchKernelGGL(k_resort, g, dim3(kThreads), 0, s, in, na, nb, nt, out, j0);
  });
}

}  // namespace ashrt

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
// shots reach the workgroup's stretch of the record, a handful, instead of
// testing every source at every sample.  128 x 128 x 1024: blending 247 ->
// 28 us, pseudo-deblending 41 -> 20 us, re-sorting 37 -> 19 us (3.4, 5 and 7 TB/s).
#include "kernels.h"

#include <algorithm>

namespace ashrt {

constexpr int kBlendTile = 4 * kThreads;  // record samples per workgroup
constexpr int kBlendList = 1024;          // sources tested at a time
constexpr int kBlendRows = 8;             // most receivers per workgroup

__device__ __forceinline__ float4 load4(const float* p) {
  float4 v;
  __builtin_memcpy(&v, p, 16);
  return v;
}
__device__ __forceinline__ void store4(float* p, float4 v) { __builtin_memcpy(p, &v, 16); }

__global__ __launch_bounds__(kThreads) void k_blend(const float* __restrict__ D, int ns, int nr, int nt,
                                                   const int* __restrict__ fire, float* __restrict__ b, int nrec,
                                                   int rows) {
  __shared__ int src[kBlendList], at[kBlendList];
  __shared__ int wsum[kThreads / 64];
  const int lo = (int)blockIdx.x * kBlendTile, hi = min(nrec - lo, kBlendTile);  // samples lo .. lo + hi - 1
  const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
  const int left = hi - 4 * (int)threadIdx.x;  // of the thread's samples tau, tau + 1, ...
  const int tau = lo + (left > 0 ? 4 * (int)threadIdx.x : 0);
  for (int s0 = 0; s0 < ns; s0 += kBlendList) {
    // the sources s0 .. s0 + kBlendList - 1 that reach the tile, in index order
    int n = 0;
    for (int c = s0; c < min(ns, s0 + kBlendList); c += kThreads) {
      const int s = c + (int)threadIdx.x;
      const int f = s < ns ? fire[s] : 0;
      const bool in = s < min(ns, s0 + kBlendList) &&
                      (long long)f < (long long)lo + hi && (long long)f + nt > (long long)lo;
      const unsigned long long m = __ballot(in);
      if (lane == 0) wsum[wave] = __popcll(m);
      __syncthreads();
      int off = n + __popcll(m & ((1ull << lane) - 1));
      int all = 0;
      for (int w = 0; w < kThreads / 64; ++w) {
        if (w < wave) off += wsum[w];
        all += wsum[w];
      }
      if (in) {
        src[off] = s;
        at[off] = f;
      }
      n += all;
      __syncthreads();
    }
    for (int rb = (int)blockIdx.y; left > 0 && rb * rows < nr; rb += gridDim.y)
    for (int r = rb * rows; r < min(nr, (rb + 1) * rows); ++r) {
      float* __restrict__ out = b + (long long)r * nrec + tau;
      if (left >= 4) {
        float4 acc = s0 ? load4(out) : make_float4(0.f, 0.f, 0.f, 0.f);
        for (int i = 0; i < n; ++i) {
          const int t = tau - at[i];
          const float* __restrict__ d = D + ((long long)src[i] * nr + r) * nt + t;
          if (t >= 0 && t + 4 <= nt) {
            const float4 v = load4(d);
            acc = make_float4(acc.x + v.x, acc.y + v.y, acc.z + v.z, acc.w + v.w);
          } else if (t > -4 && t < nt) {
            if (t >= 0) acc.x += d[0];
            if (t + 1 >= 0 && t + 1 < nt) acc.y += d[1];
            if (t + 2 >= 0 && t + 2 < nt) acc.z += d[2];
            if (t + 3 >= 0 && t + 3 < nt) acc.w += d[3];
          }
        }
        store4(out, acc);
      } else {
        for (int k = 0; k < left; ++k) {
          float acc = s0 ? out[k] : 0.f;
          for (int i = 0; i < n; ++i) {
            const int t = tau + k - at[i];
            if (t >= 0 && t < nt) acc += D[((long long)src[i] * nr + r) * nt + t];
          }
          out[k] = acc;
        }
      }
    }
    __syncthreads();
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
  // receivers share a workgroup's source list while enough workgroups remain
  const long long tiles = (nrec + (long long)kBlendTile - 1) / kBlendTile;
  const int rows = (int)std::max(1LL, std::min<long long>(kBlendRows, tiles * nr / 1024));
  hipLaunchKernelGGL(k_blend, dim3((unsigned)tiles, (unsigned)std::min((nr - 1) / rows + 1, 65535)), dim3(kThreads), 0, s,
                     D, ns, nr, nt, fire, b, nrec, rows);
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

// HIP kernels of the robust inversion (thesis Chapter 4, "Robust Radon
// transform"): CGLS vector updates in FP32 with FP64 inner products and step
// scalars kept on the device, the IRLS residual and model weights, and the
// median absolute deviation by radix selection on float bit patterns.
//
// All kernels take per-gather work lists so one launch serves a whole batch.
// Reductions are deterministic: each work item writes one partial, and the
// partials of a gather are summed in a fixed tree order.
#include "block_reduce.h"
#include "kernels.h"

namespace ashrt {

// ------------------------------------------------------------ partial reductions


__global__ __launch_bounds__(kThreads) void k_reduce_part(RedArgs A) {
  __shared__ double sh[kThreads / 64];
  const int it = blockIdx.x;
  const VecItem w = load_const(A.items + it);
  const GatherDev G = load_const(A.gd + w.g);
  const uint8_t* tm = A.tmask ? A.tmask + G.mask_off : nullptr;
  double a = 0.0, b = 0.0;
  const double eps = A.sc ? A.sc[w.g * kNScal + SC_EPS_R] : 0.0;
  long long i0 = threadIdx.x;
  if ((A.op == RED_SUMSQ || A.op == RED_ABSMAX) && ((w.start | w.len) & 3) == 0) {
    const float4* x4 = reinterpret_cast<const float4*>(A.x + w.start);
    // the loads of kBatch iterations are issued before any is used
    constexpr int kBatch = 4;
    const int n4 = (int)(w.len >> 2);
    for (int base = threadIdx.x; base < n4; base += kBatch * kThreads) {
      float4 q[kBatch];
#pragma unroll
      for (int k = 0; k < kBatch; ++k) q[k] = x4[min(base + k * kThreads, n4 - 1)];
#pragma unroll
      for (int k = 0; k < kBatch; ++k) {
        if (base + k * kThreads >= n4) break;
        const float4 v = q[k];
        if (A.op == RED_SUMSQ) {
          a += (double)v.x * v.x + (double)v.y * v.y + (double)v.z * v.z + (double)v.w * v.w;
        } else {
          a = fmax(a, (double)fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
        }
      }
    }
    i0 = w.len;  // done
  }
  for (long long i = i0; i < w.len; i += kThreads) {
    const long long o = w.start + i;
    const double v = (double)A.x[o];
    if (A.op == RED_SUMSQ) {
      a += v * v;
    } else if (A.op == RED_ABSMAX) {
      a = fmax(a, fabs(v));
    } else if (A.op == RED_ABSSUM) {
      a += fabs(v);
    } else {
      bool live = true;
      if (tm) {
        const unsigned x = (unsigned)(o - G.d_off) / (unsigned)G.nt;  // nx nt < 2^31
        live = tm[x] != 0;
      }
      if (!live) continue;
      if (A.op == RED_ABSMAX_LIVE) {
        a = fmax(a, fabs(v));
      } else {  // RED_MISFIT: sum |r|^p and the Huber (p = 1) or LS (p = 2) objective
        const double av = fabs(v);
        if (A.p == 1) {
          a += av;
          b += (eps > 0.0) ? ((av <= eps) ? av * av / (2.0 * eps) : av - 0.5 * eps) : av;
        } else {
          a += v * v;
          b += 0.5 * v * v;
        }
      }
    }
  }
  double ra, rb = 0.0;
  if (A.op == RED_ABSMAX || A.op == RED_ABSMAX_LIVE) {
    ra = block_max(a, sh);
  } else {
    ra = block_sum(a, sh);
    if (A.op == RED_MISFIT) rb = block_sum(b, sh);
  }
  if (threadIdx.x == 0) {
    A.part[2 * it] = ra;
    A.part[2 * it + 1] = rb;
  }
}

// One workgroup per gather: combine the partials of its items in a fixed order
// and store into the scalar slots (dst0, dst1; -1 = skip).  is_max selects max.

__global__ __launch_bounds__(kThreads) void k_reduce_fin(FinArgs A) {
  __shared__ double sh[kThreads / 64];
  const int g = blockIdx.x;
  if (g >= A.ngather) return;
  const GatherDev G = load_const(A.gd + g);
  const int lo = A.is_model ? G.mit_lo : G.dit_lo;
  const int hi = A.is_model ? G.mit_hi : G.dit_hi;
  double a = 0.0, b = 0.0;
  for (int i = lo + threadIdx.x; i < hi; i += kThreads) {
    if (A.is_max) {
      a = fmax(a, A.part[2 * i]);
    } else {
      a += A.part[2 * i];
      b += A.part[2 * i + 1];
    }
  }
  double ra, rb = 0.0;
  if (A.is_max) {
    ra = block_max(a, sh);
  } else {
    ra = block_sum(a, sh);
    rb = block_sum(b, sh);
  }
  if (threadIdx.x == 0) {
    if (A.dst0 >= 0) A.sc[g * kNScal + A.dst0] = ra;
    if (A.dst1 >= 0) A.sc[g * kNScal + A.dst1] = rb;
    if (A.rep) {
      A.rep[g].misfit[A.outer] = ra;
      A.rep[g].huber[A.outer] = rb;
      if (!isfinite(ra) || !isfinite(rb)) A.sc[g * kNScal + SC_NONFINITE] = 1.0;
    }
  }
}

// ------------------------------------------------------------ element-wise
// Bound by memory: 16-byte accesses, and each thread issues the loads of kBatch
// of them before it uses any.  The FISTA step of 25 M values (5 arrays): 76 us,
// 6.6 TB/s out of memory and the last-level cache; all element-wise passes of a
// run of 10 + 20 iterations 1.88 ms, 2.20 with 4-byte accesses.
template <int OP>
__device__ __forceinline__ float ew_one(const EwArgs& A, float c, float c2, bool live, float x, float y, float z,
                                        float& zo) {
  if constexpr (OP == EW_MUL) return x * z;
  if constexpr (OP == EW_COPY) return x;
  if constexpr (OP == EW_FILL) return A.value;
  if constexpr (OP == EW_WR_INIT) return live ? (A.x ? x : 1.0f) : 0.f;
  if constexpr (OP == EW_WR_UPDATE) return live ? ((c > 0.f) ? 1.0f / sqrtf(fmaxf(fabsf(x), c)) : 1.0f) : 0.f;
  if constexpr (OP == EW_WR_MASK) return live ? 1.0f : 0.f;
  if constexpr (OP == EW_WM_UPDATE) return (c > 0.f) ? sqrtf(fmaxf(fabsf(x), c)) : 1.0f;
  if constexpr (OP == EW_SCALE_RSQRT) return x * c;
  if constexpr (OP == EW_FISTA) {
    const float v = fmaf(c, x, y);
    const float a = fabsf(v) - c2;
    const float mn = a > 0.f ? copysignf(a, v) : 0.f;
    const float mo = zo;
    zo = mn;
    return fmaf(A.value, mn - mo, mn);
  }
}

template <int OP>
__global__ __launch_bounds__(kThreads) void k_elementwise(EwArgs A) {
  constexpr bool RX = OP != EW_FILL && OP != EW_WR_MASK, RZ = OP == EW_MUL, FISTA = OP == EW_FISTA;
  constexpr bool MASK = OP == EW_WR_INIT || OP == EW_WR_UPDATE || OP == EW_WR_MASK;
  const VecItem w = load_const(A.items + blockIdx.x);
  const GatherDev G = load_const(A.gd + w.g);
  float c = 0.f, c2 = 0.f;
  if constexpr (OP == EW_WR_UPDATE || OP == EW_WM_UPDATE) c = (float)A.sc[w.g * kNScal + A.coef];
  if constexpr (OP == EW_SCALE_RSQRT) {
    const double ss = A.sc[w.g * kNScal + A.coef];
    c = ss > 0.0 ? (float)(1.0 / sqrt(ss)) : 0.f;
  }
  if constexpr (FISTA) {
    c = (float)A.sc[w.g * kNScal + A.coef];
    c2 = (float)A.sc[w.g * kNScal + A.coef + 1];
  }
  const uint8_t* tm = MASK && A.tmask ? A.tmask + G.mask_off : nullptr;
  const unsigned rel0 = (unsigned)(w.start - G.d_off);  // data vectors: sample in the gather (nx nt < 2^31)
  auto live = [&](int i) { return !tm || tm[(rel0 + (unsigned)i) / (unsigned)G.nt] != 0; };
  const bool hx = RX && (OP != EW_WR_INIT || A.x);
  float* const y = A.y + w.start;
  float* const zo = A.z_out + w.start;
  const float* const x = A.x + w.start;
  const float* const z = A.z + w.start;
  const int n = (int)w.len;
  uintptr_t al = (uintptr_t)y | (uintptr_t)(w.len * 4);
  if (hx) al |= (uintptr_t)x;
  if (RZ) al |= (uintptr_t)z;
  if (FISTA) al |= (uintptr_t)zo;
  if ((al & 15) == 0) {
    constexpr int kBatch = 4;
    const int n4 = n >> 2;
    for (int base = threadIdx.x; base < n4; base += kBatch * kThreads) {
      float4 xv[kBatch], yv[kBatch], zv[kBatch];
#pragma unroll
      for (int b = 0; b < kBatch; ++b) {
        const int i = min(base + b * kThreads, n4 - 1);
        xv[b] = yv[b] = zv[b] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (hx) xv[b] = reinterpret_cast<const float4*>(x)[i];
        if constexpr (RZ) zv[b] = reinterpret_cast<const float4*>(z)[i];
        if constexpr (FISTA) {
          yv[b] = reinterpret_cast<const float4*>(y)[i];
          zv[b] = reinterpret_cast<const float4*>(zo)[i];
        }
      }
#pragma unroll
      for (int b = 0; b < kBatch; ++b) {
        const int i = base + b * kThreads;
        if (i >= n4) break;
        float4 o = zv[b], r;
        r.x = ew_one<OP>(A, c, c2, !MASK || live(4 * i), xv[b].x, yv[b].x, zv[b].x, o.x);
        r.y = ew_one<OP>(A, c, c2, !MASK || live(4 * i + 1), xv[b].y, yv[b].y, zv[b].y, o.y);
        r.z = ew_one<OP>(A, c, c2, !MASK || live(4 * i + 2), xv[b].z, yv[b].z, zv[b].z, o.z);
        r.w = ew_one<OP>(A, c, c2, !MASK || live(4 * i + 3), xv[b].w, yv[b].w, zv[b].w, o.w);
        reinterpret_cast<float4*>(y)[i] = r;
        if constexpr (FISTA) reinterpret_cast<float4*>(zo)[i] = o;
      }
    }
  } else {
    for (int i = threadIdx.x; i < n; i += kThreads) {
      float o = FISTA ? zo[i] : 0.f;
      const float r = ew_one<OP>(A, c, c2, !MASK || live(i), hx ? x[i] : 0.f, FISTA ? y[i] : 0.f, RZ ? z[i] : 0.f, o);
      y[i] = r;
      if constexpr (FISTA) zo[i] = o;
    }
  }
}

// ------------------------------------------------------------ per-gather scalar steps


__global__ void k_scalar(ScalArgs A) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= A.ngather) return;
  double* s = A.sc + g * kNScal;
  switch (A.step) {
    case ST_EPS_M:
      s[SC_EPS_M] = A.b_m * s[SC_MMAX] / 100.0;
      if (A.rep) A.rep[g].eps_m[A.outer] = s[SC_EPS_M];
      break;
    case ST_EPS_R: {
      double e;
      if (A.freeze && s[SC_FROZEN_SET] != 0.0) {
        e = s[SC_EPS_FROZEN];
      } else {
        e = fmax(A.b_r * s[SC_MAD] / 0.6745, A.floor_rel * s[SC_DMAX]);
        if (A.freeze) {
          s[SC_EPS_FROZEN] = e;
          s[SC_FROZEN_SET] = 1.0;
        }
      }
      s[SC_EPS_R] = e;
      if (A.rep) A.rep[g].eps_r[A.outer] = e;
      break;
    }
    case ST_REPORT_INNER:
      if (A.rep) A.rep[g].inner[A.outer] = s[SC_NINNER];
      break;
    case ST_FISTA: {
      const double lf = 2.0 * A.safety * sqrt(fmax(s[SC_POW_SS], 0.0));
      const double mu = A.mu_abs > 0.0 ? A.mu_abs : A.mu_rel * 2.0 * s[SC_MMAX];
      s[SC_LIP] = lf;
      s[SC_MU] = mu;
      s[SC_FSTEP] = lf > 0.0 ? 2.0 / lf : 0.0;
      s[SC_FTHR] = lf > 0.0 ? mu / lf : 0.0;
      break;
    }
    default:
      break;
  }
}

// ------------------------------------------------------------ radix select
//
// Order statistics of the live residual samples by three histogram passes
// over the float bit pattern mapped to an order-preserving unsigned key
// (11, 11, 10 bits).  The two middle ranks floor((n-1)/2) and floor(n/2) are
// selected together so the median of an even count is the mean of the two
// middle values; while their prefixes agree one histogram serves both.  Stage
// 0 selects on r, stage 1 on |r - median(r)|.
__device__ __forceinline__ unsigned float_key(float f) {
  const unsigned b = __float_as_uint(f);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float key_float(unsigned k) {
  const unsigned b = (k & 0x80000000u) ? (k & 0x7fffffffu) : ~k;
  return __uint_as_float(b);
}


// Digits of the three passes.
constexpr int kSelShift[3] = {21, 10, 0};
constexpr int kSelWidth[3] = {11, 11, 10};

// kSelSplit workgroups per data-vector item; each thread issues the loads
// of four samples before it bins them.
constexpr int kSelSplit = 2;
__global__ __launch_bounds__(kThreads) void k_sel_hist(SelArgs A) {
  __shared__ unsigned h[2][kSelBins];
  const int b = blockIdx.x;
  for (int i = threadIdx.x; i < 2 * kSelBins; i += kThreads) (&h[0][0])[i] = 0u;
  __syncthreads();
  const int it = b / kSelSplit, part = b - it * kSelSplit;
  const VecItem w = load_const(A.items + it);
  const GatherDev G = load_const(A.gd + w.g);
  const unsigned hmask = (A.shift + A.width >= 32) ? 0u : (0xffffffffu << (A.shift + A.width));
  const unsigned p0 = A.st[w.g].prefix[0] & hmask, p1 = A.st[w.g].prefix[1] & hmask;
  const unsigned dmask = (1u << A.width) - 1u;
  const uint8_t* tm = A.tmask ? A.tmask + G.mask_off : nullptr;
  const double med = A.stage ? A.sc[w.g * kNScal + SC_MED] : 0.0;
  const long long lo = w.start + w.len * part / kSelSplit;
  const int n = (int)(w.start + w.len * (part + 1) / kSelSplit - lo);
  const unsigned rel0 = (unsigned)(lo - G.d_off);  // sample index in the gather (nx nt < 2^31)
  for (int base = threadIdx.x; base < n; base += 4 * kThreads) {
    float v[4];
    int live[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = A.x[lo + min(base + u * kThreads, n - 1)];
    if (tm) {
#pragma unroll
      for (int u = 0; u < 4; ++u) live[u] = tm[(rel0 + (unsigned)min(base + u * kThreads, n - 1)) / (unsigned)G.nt];
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u) live[u] = 1;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (base + u * kThreads >= n || live[u] == 0) continue;
      float x = v[u];
      if (A.stage) x = (float)fabs((double)x - med);
      const unsigned key = float_key(x);
      const unsigned dg = (key >> A.shift) & dmask;
      if ((key & hmask) == p0) atomicAdd(&h[0][dg], 1u);
      else if ((key & hmask) == p1) atomicAdd(&h[1][dg], 1u);
    }
  }
  __syncthreads();
  unsigned* gh = A.hist + (long long)w.g * 2 * kSelBins;
  for (int i = threadIdx.x; i < 2 * kSelBins; i += kThreads) {
    const unsigned c = (&h[0][0])[i];
    if (c) atomicAdd(&gh[i], c);
  }
}

// The two ranks of a selection over n samples.
__device__ __forceinline__ unsigned sel_rank(double n, int s) {
  const unsigned nn = (unsigned)n;
  return nn ? (nn - 1u + s) / 2u : 0u;
}

// Median of the two selected keys (in FP64), 0 without samples.
__device__ __forceinline__ double sel_median(const unsigned prefix[2], double n) {
  return n > 0.0 ? 0.5 * ((double)key_float(prefix[0]) + (double)key_float(prefix[1])) : 0.0;
}

// Thread t of NT holds c = the counts of its bins: the count before them,
// among all threads.  Two barriers; wsum: NT / 64 words of LDS.
template <int NT>
__device__ __forceinline__ unsigned count_before(unsigned c, unsigned* wsum) {
  const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
  unsigned v = c;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const unsigned o = __shfl_up(v, off);
    if (lane >= off) v += o;
  }
  if (lane == 63) wsum[wave] = v;
  __syncthreads();
  unsigned before = v - c;
  for (int k = 0; k < wave; ++k) before += wsum[k];
  __syncthreads();
  return before;
}

// One workgroup per gather and histogram pass: find the digit holding each
// rank, fix it in the prefix, subtract the counts below, and clear the
// histogram for the next pass.  The first pass starts from the ranks and the
// last writes the median to sc[g][dst].
__global__ __launch_bounds__(kThreads) void k_sel_pick(SelArgs A, double* sc, int dst) {
  constexpr int PER = kSelBins / kThreads;  // bins per thread
  __shared__ unsigned wsum[kThreads / 64], prefix[2], kk[2];
  const int g = blockIdx.x;
  const double n = sc[g * kNScal + SC_NLIVE];
  const bool first = A.shift + A.width == 32, last = A.shift == 0;
  if (threadIdx.x < 2) {
    prefix[threadIdx.x] = first ? 0u : A.st[g].prefix[threadIdx.x];
    kk[threadIdx.x] = first ? sel_rank(n, threadIdx.x) : A.st[g].kk[threadIdx.x];
  }
  unsigned* gh = A.hist + (long long)g * 2 * kSelBins;
  unsigned c[2][PER], sum[2] = {0u, 0u};
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      unsigned* const hb = gh + s * kSelBins + threadIdx.x * PER + i;
      c[s][i] = *hb;
      *hb = 0u;
      sum[s] += c[s][i];
    }
  __syncthreads();
  const int h1 = prefix[0] == prefix[1] ? 0 : 1;  // histogram of the second rank
  const unsigned k0 = kk[0], k1 = kk[1];
  const unsigned b0 = count_before<kThreads>(sum[0], wsum), b1 = h1 ? count_before<kThreads>(sum[1], wsum) : b0;
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const bool second = s == 1 && h1 == 1;
    unsigned run = second ? b1 : b0;
    const unsigned k = s == 0 ? k0 : k1;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const unsigned n1 = second ? c[1][i] : c[0][i];
      if (k >= run && k < run + n1) {
        prefix[s] |= (unsigned)(threadIdx.x * PER + i) << A.shift;
        kk[s] = k - run;
      }
      run += n1;
    }
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    A.st[g].prefix[threadIdx.x] = prefix[threadIdx.x];
    A.st[g].kk[threadIdx.x] = kk[threadIdx.x];
  }
  if (last && threadIdx.x == 0) sc[g * kNScal + dst] = sel_median(prefix, n);
}

// Median and median absolute deviation of a gather of at most kSelSmall
// samples: one workgroup holds the samples in registers and the histograms in
// LDS through all six passes.  256 x 64 samples: one launch of 33 us in place of
// sixteen of 71 together.  Larger gathers would leave their samples to one CU
// (1024 x 256: 1 MB), so they take k_sel_hist and k_sel_pick.
constexpr int kSelSmallThreads = 1024;
__global__ __launch_bounds__(kSelSmallThreads) void k_sel_small(SelArgs A, double* sc, int dst_med, int dst_mad) {
  constexpr int NT = kSelSmallThreads, U = kSelSmall / NT, PER = kSelBins / NT;
  static_assert(U <= 32, "one live bit each");
  // four copies of the first histogram, lanes taking turns: residuals crowd
  // into few bins, and equal addresses of a wave are added one by one
  __shared__ uint4 h0[kSelBins];
  __shared__ unsigned h1[kSelBins], wsum[NT / 64], prefix[2], kk[2];
  unsigned* const hc = reinterpret_cast<unsigned*>(h0) + (threadIdx.x & 3);
  const int g = blockIdx.x;
  const GatherDev G = load_const(A.gd + g);
  const int n = G.nx * G.nt;
  const double nlive = sc[g * kNScal + SC_NLIVE];
  const uint8_t* tm = A.tmask ? A.tmask + G.mask_off : nullptr;
  float v[U];
  unsigned live = 0u;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int i = (int)threadIdx.x + u * NT;
    v[u] = 0.f;
    if (i < n) {
      v[u] = A.x[G.d_off + i];
      if (!tm || tm[i / G.nt] != 0) live |= 1u << u;
    }
  }
  double med = 0.0;
  for (int stage = 0; stage < 2; ++stage) {
    if (threadIdx.x < 2) {
      prefix[threadIdx.x] = 0u;
      kk[threadIdx.x] = sel_rank(nlive, threadIdx.x);
    }
    for (int pass = 0; pass < 3; ++pass) {
      const int shift = kSelShift[pass], width = kSelWidth[pass];
      const unsigned hmask = shift + width >= 32 ? 0u : 0xffffffffu << (shift + width);
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        h0[threadIdx.x * PER + i] = make_uint4(0u, 0u, 0u, 0u);
        h1[threadIdx.x * PER + i] = 0u;
      }
      __syncthreads();
      const unsigned p0 = prefix[0] & hmask, p1 = prefix[1] & hmask;
      const unsigned k0 = kk[0], k1 = kk[1];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (!(live >> u & 1u)) continue;
        const float x = stage ? (float)fabs((double)v[u] - med) : v[u];
        const unsigned key = float_key(x), dg = (key >> shift) & ((1u << width) - 1u);
        if ((key & hmask) == p0) atomicAdd(hc + 4 * dg, 1u);
        else if ((key & hmask) == p1) atomicAdd(&h1[dg], 1u);
      }
      __syncthreads();
      unsigned c[2][PER], before[2];
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const uint4 q = h0[threadIdx.x * PER + i];
        c[0][i] = (q.x + q.y) + (q.z + q.w);
        c[1][i] = p0 == p1 ? c[0][i] : h1[threadIdx.x * PER + i];
      }
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        unsigned sum = 0u;
#pragma unroll
        for (int i = 0; i < PER; ++i) sum += c[s][i];
        before[s] = s && p0 == p1 ? before[0] : count_before<NT>(sum, wsum);
      }
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const unsigned k = s ? k1 : k0;
        unsigned run = before[s];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
          if (k >= run && k < run + c[s][i]) {
            prefix[s] |= (unsigned)(threadIdx.x * PER + i) << shift;
            kk[s] = k - run;
          }
          run += c[s][i];
        }
      }
      __syncthreads();
    }
    const double r = sel_median(prefix, nlive);
    if (stage == 0) med = r;
    if (threadIdx.x == 0) sc[g * kNScal + (stage ? dst_mad : dst_med)] = r;
    __syncthreads();  // the prefixes are read
  }
}

// Live sample count per gather: (# live traces) * nt.
__global__ __launch_bounds__(kThreads) void k_count_live(const GatherDev* gd, int ngather,
                                                         const uint8_t* tmask, double* sc) {
  __shared__ double sh[kThreads / 64];
  const int g = blockIdx.x;
  if (g >= ngather) return;
  const GatherDev G = load_const(gd + g);
  double c = 0.0;
  for (int x = threadIdx.x; x < G.nx; x += kThreads) c += (tmask ? (tmask[G.mask_off + x] != 0) : 1) ? 1.0 : 0.0;
  const double r = block_sum(c, sh);
  if (threadIdx.x == 0) sc[g * kNScal + SC_NLIVE] = r * (double)G.nt;
}

// CG initialisation / update over model-vector items (see CgArgs).
// Per-gather sum of per-tile partials in a fixed order: four interleaved
// thread-strided partial sums per thread (loads in flight), then block_sum.
constexpr int kSumThreads = 1024;
__global__ __launch_bounds__(kSumThreads) void k_sum_items(const GatherDev* gd, int ngather, const double* part,
                                                           int is_model, double* sc, int dst) {
  __shared__ double sh[kSumThreads / 64];
  const int g = blockIdx.x;
  if (g >= ngather) return;
  const GatherDev G = load_const(gd + g);
  const int lo = is_model ? G.xm_lo : G.xd_lo;
  const int hi = is_model ? G.xm_hi : G.xd_hi;
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
  int i = lo + (int)threadIdx.x;
  for (; i + 3 * kSumThreads < hi; i += 4 * kSumThreads) {
    a0 += part[i];
    a1 += part[i + kSumThreads];
    a2 += part[i + 2 * kSumThreads];
    a3 += part[i + 3 * kSumThreads];
  }
  for (; i < hi; i += kSumThreads) a0 += part[i];
  const double r = block_sum((a0 + a1) + (a2 + a3), sh);
  if (threadIdx.x == 0) sc[(long long)g * kNScal + dst] = r;
}

__global__ __launch_bounds__(kThreads) void k_cg(CgArgs A) {
  __shared__ double sh[kThreads / 64];
  const int it = blockIdx.x;
  const VecItem w = load_const(A.items + it);
  const GatherDev G = load_const(A.gd + w.g);
  double* const sc = A.sc + (long long)w.g * kNScal;
  if (A.init) {
    if (it != G.mit_lo) return;
    double gsum = 0.0;
    if (A.part_gamma) {
      double part = 0.0;
      for (int i = G.xm_lo + (int)threadIdx.x; i < G.xm_hi; i += kThreads) part += A.part_gamma[i];
      gsum = block_sum(part, sh);
    }
    if (threadIdx.x == 0) {
      sc[SC_GAMMA0] = A.part_gamma ? gsum : sc[SC_GNEW];
      sc[SC_DONE] = 0.0;
      sc[SC_NINNER] = 0.0;
    }
    return;
  }
  const float alpha = sc[SC_DONE] != 0.0 ? 0.f : (float)sc[SC_ALPHA];
  float* __restrict__ u = A.u + w.start;
  const float* __restrict__ p = A.pdir + w.start;
  const int n = (int)w.len;
  if ((((uintptr_t)u | (uintptr_t)p | (uintptr_t)(w.len * 4)) & 15) == 0 && n > 0) {
    float4* u4 = reinterpret_cast<float4*>(u);
    const float4* p4 = reinterpret_cast<const float4*>(p);
    // the loads of kBatch loop iterations are issued before any is used
    // (indices past the item clamped for the loads, skipped for the stores)
    constexpr int kBatch = 4;
    const int n4 = n >> 2;
    for (int base = threadIdx.x; base < n4; base += kBatch * kThreads) {
      float4 pv[kBatch], uv[kBatch];
#pragma unroll
      for (int b = 0; b < kBatch; ++b) {
        const int i = min(base + b * kThreads, n4 - 1);
        pv[b] = p4[i];
        uv[b] = u4[i];
      }
#pragma unroll
      for (int b = 0; b < kBatch; ++b) {
        const int i = base + b * kThreads;
        if (i >= n4) break;
        u4[i] = make_float4(fmaf(alpha, pv[b].x, uv[b].x), fmaf(alpha, pv[b].y, uv[b].y),
                            fmaf(alpha, pv[b].z, uv[b].z), fmaf(alpha, pv[b].w, uv[b].w));
      }
    }
  } else {
    for (int i = threadIdx.x; i < n; i += kThreads) u[i] = fmaf(alpha, p[i], u[i]);
  }
}

// Clear n 32-bit words (a fill kernel rather than a memset, so the call can
// sit inside a captured graph).
__global__ void k_zero_words(unsigned* p, long long n) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
    p[i] = 0u;
}

// ------------------------------------------------------------ launchers
static inline int grid_of(int n) { return n < 1 ? 1 : n; }

hipError_t launch_reduce_part(const RedArgs& a, hipStream_t s) {
  if (a.nitems <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_reduce_part, dim3(grid_of(a.nitems)), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_reduce_fin(const FinArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_reduce_fin, dim3(grid_of(a.ngather)), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_elementwise(const EwArgs& a, hipStream_t s) {
  if (a.nitems <= 0) return hipSuccess;
#define EW_CASE(OP) \
  case OP: hipLaunchKernelGGL(k_elementwise<OP>, dim3(a.nitems), dim3(kThreads), 0, s, a); break
  switch (a.op) {
    EW_CASE(EW_MUL);
    EW_CASE(EW_COPY);
    EW_CASE(EW_FILL);
    EW_CASE(EW_WR_INIT);
    EW_CASE(EW_WR_UPDATE);
    EW_CASE(EW_WM_UPDATE);
    EW_CASE(EW_WR_MASK);
    EW_CASE(EW_SCALE_RSQRT);
    EW_CASE(EW_FISTA);
    default: return hipErrorInvalidValue;
  }
#undef EW_CASE
  return hipGetLastError();
}
hipError_t launch_scalar(const ScalArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_scalar, dim3((a.ngather + 63) / 64), dim3(64), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_zero_words(void* p, long long n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  long long blocks = (n + kThreads - 1) / kThreads;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_zero_words, dim3((unsigned)blocks), dim3(kThreads), 0, s, (unsigned*)p, n);
  return hipGetLastError();
}
hipError_t launch_sum_items(const GatherDev* gd, int ngather, const double* part, int is_model, double* sc,
                            int dst, hipStream_t s) {
  if (ngather <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_sum_items, dim3(ngather), dim3(kSumThreads), 0, s, gd, ngather, part, is_model, sc, dst);
  return hipGetLastError();
}

hipError_t launch_cg(const CgArgs& a, hipStream_t s) {
  if (a.nitems <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_cg, dim3(grid_of(a.nitems)), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_count_live(const GatherDev* gd, int ngather, const uint8_t* tmask, double* sc,
                             hipStream_t s) {
  hipLaunchKernelGGL(k_count_live, dim3(grid_of(ngather)), dim3(kThreads), 0, s, gd, ngather, tmask, sc);
  return hipGetLastError();
}

// Median of the live samples of a.x into sc[g][dst_med] and the median of their
// absolute deviations from it into sc[g][dst_mad].  The histogram must be zero
// on entry and is left zero.
hipError_t launch_select_median_mad(SelArgs a, bool small, double* sc, int dst_med, int dst_mad, hipStream_t s) {
  if (small) {
    hipLaunchKernelGGL(k_sel_small, dim3(a.ngather), dim3(kSelSmallThreads), 0, s, a, sc, dst_med, dst_mad);
    return hipGetLastError();
  }
  for (a.stage = 0; a.stage < 2; ++a.stage) {
    for (int pass = 0; pass < 3; ++pass) {
      a.shift = kSelShift[pass];
      a.width = kSelWidth[pass];
      if (a.nitems > 0) hipLaunchKernelGGL(k_sel_hist, dim3(grid_of(a.nitems * kSelSplit)), dim3(kThreads), 0, s, a);
      hipLaunchKernelGGL(k_sel_pick, dim3(a.ngather), dim3(kThreads), 0, s, a, sc, a.stage ? dst_mad : dst_med);
    }
  }
  return hipGetLastError();
}

}  // namespace ashrt

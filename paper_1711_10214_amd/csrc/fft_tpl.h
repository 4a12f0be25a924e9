// Compile-time-length Stockham FFT in LDS for 256-thread workgroups.
//
// N = 2^a or 3*2^a.  Passes: one radix-3 pass if 3 | N, then radix-8 passes,
// then one radix-4 or radix-2 pass for the leftover power of two.  Pass i
// with radix R and span Ns (product of the earlier radices) maps
//   v_r = x[j + r N/R] * w^(r (j mod Ns)),  w = exp(-+2 pi i / (Ns R)),
//   y[(j div Ns) Ns R + (j mod Ns) + r Ns] = DFT_R(v)_r .
// Elements live at padded LDS positions fft_pad(i) = i + i/16 (one 8-byte
// gap every 128 bytes), which makes the strided writes of the first passes
// hit distinct banks; a padded transform occupies fft_padlen(N) slots.
// Each pass reads its butterflies into registers, waits at a barrier, and
// writes the outputs in place.
//
// Twiddles.  A radix-8 butterfly of v_r w^r is three radix-2 stages whose
// twiddles are w^4, then w^2, then w and w e^(-i pi/4), up to a factor -i
// that only swaps components.  Each is stored as (cos, sin), and a + w b and
// a - w b take six FMAs: two a component for the first, and the second is
// 2 a minus the first.  That is 72 instructions per twiddled radix-8 butterfly
// where multiplying the inputs by w .. w^7 formed by recurrence took 112, with
// fewer roundings on the way (no powers, one FMA where a multiply and an add
// were).  On the 1024 x 256, 32-panel gather the forward row kernel went from
// 48.3 to 45.4 us, the model x kernels from 28.3 to 27.1 and 31.2 to 30.1 us,
// and the operator's error against FP64 from 3.7e-7 to 2.5e-7.  No value passes
// |a| + |b|, so the transforms take the whole FP32 range (the same six
// instructions as c (b.x - tan b.y) with tabulated tangents are as fast and
// reach 2.1e-7, but their quarter turns overflow from 2^100 on).
// A per-length "pass table" built in FP64 on the host holds, for pass i and
// jm = 0..Ns-1,
//   radix 8: (w^4, w^2)[Ns], (w, w e^(-i pi/4))[Ns];  radix 4: (w^2, w)[Ns];
//   radix 2: w[Ns]          (16-byte records, w = exp(-2 pi i jm / (Ns R))).
#pragma once

#include <hip/hip_runtime.h>

#include "ashrt_internal.h"
#include "fft_lds.h"

namespace ashrt {

constexpr int ilog2c(int n) { return n <= 1 ? 0 : 1 + ilog2c(n / 2); }

__host__ __device__ constexpr int fft_pad(int i) { return i + (i >> 4); }
__host__ __device__ constexpr int fft_padlen(int n) { return n + (n >> 4); }

// True when fft_pad(x + r S) == fft_pad(x) + fft_pad(r S) for every r < R
// and every x congruent mod 16 to q QS + m (q >= 0, 0 <= m < M): no step r S
// carries out of x's low four bits.  A butterfly's R padded addresses are
// then one base plus compile-time offsets, which the LDS instructions take
// as immediates instead of a shift and two adds per element.
constexpr bool pad_linear(int S, int R, int QS, int M) {
  for (int q = 0; q < 16; ++q)
    for (int m = 0; m < M && m < 16; ++m)
      for (int r = 0; r < R; ++r)
        if (((q * QS + m) & 15) + ((r * S) & 15) >= 16) return false;
  return true;
}

// fft_pad(x + c) for a constant c >= 0 from p = fft_pad(x) and lo = x & 15:
// the step adds c + c/16 slots, and one more when x's low four bits carry
// (a compare against a constant instead of a shift and two adds).
__device__ __forceinline__ int pad_step(int p, int lo, int c) {
  return p + c + (c >> 4) + ((c & 15) != 0 && lo >= 16 - (c & 15) ? 1 : 0);
}

// Index of logical element i of a buffer written by an FFT of compile-time
// length N (padded) or by the generic runtime FFT (N == 0, unpadded).
template <int N>
__device__ __forceinline__ int px(int i) {
  if constexpr (N > 0) return fft_pad(i);
  else return i;
}

// The thread index as a fresh value that the compiler cannot relate to any
// other use of threadIdx.x.  Every pass derives its LDS indices from its own
// copy.  With the plain index, the compiler built the address of element
// j + 384 once, as (j | 384), inside the 96-lane guard of pass 1 of the
// 768-point transform (where the bits are disjoint), and reused it in the
// 192-lane radix-4 pass, where lanes 128..191 then read the wrong element.
__device__ __forceinline__ int pass_tid() {
  int t = (int)threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

template <int N>
struct FftPlan {
  static constexpr bool three = (N % 3) == 0;
  static constexpr int M = three ? N / 3 : N;
  static constexpr int L = ilog2c(M);
  static constexpr int n8 = L / 3;
  static constexpr int rem = L % 3;
  static constexpr int npass = (three ? 1 : 0) + n8 + (rem ? 1 : 0);
  static constexpr int radix(int i) {
    return (three && i == 0) ? 3 : (i < (three ? 1 : 0) + n8 ? 8 : (rem == 1 ? 2 : 4));
  }
  static constexpr int ns(int i) {
    int s = 1;
    for (int k = 0; k < i; ++k) s *= radix(k);
    return s;
  }
  // float2 entries of pass i's twiddles (pass 0 has none) and their offset
  static constexpr int twlen(int i) { return i == 0 ? 0 : ns(i) * (radix(i) / 2); }
  static constexpr int twoff(int i) {
    int o = 0;
    for (int k = 0; k < i; ++k) o += twlen(k);
    return o;
  }
  static constexpr int twsize() { return twoff(npass); }
};

// LDS slots of the staged twiddles in front of an FFT buffer, an even count
// (what follows stays 16-byte aligned): the pass table without the last pass
// (the x transforms) or the last two (the row transforms), whose twiddles
// depend on the thread alone and stay in registers, or the plain n-entry
// table of the generic runtime FFT (key 0).
inline __host__ __device__ int fft_tw_slots(int key, int n);
inline __host__ __device__ int fft_row_tw_slots(int key, int n);

// Host and device: pass-table length for a runtime N of a supported size
// (0 for lengths handled by the generic runtime FFT).
// Lengths with a compile-time FFT (others use the runtime-generic fft_lds).
#define ASHRT_TPL_SIZES(X) X(128) X(192) X(256) X(384) X(512) X(768) X(1024) X(1536) X(2048) X(3072) X(4096)

inline __host__ __device__ int fft_tpl_twsize(int n) {
#define ASHRT_TW_CASE(S) \
  if (n == S) return FftPlan<S>::twsize();
  ASHRT_TPL_SIZES(ASHRT_TW_CASE)
#undef ASHRT_TW_CASE
  return 0;
}

inline __host__ __device__ int fft_tpl_twstaged(int n) {
#define ASHRT_TW_CASE(S) \
  if (n == S) return FftPlan<S>::twoff(FftPlan<S>::npass - 1);
  ASHRT_TPL_SIZES(ASHRT_TW_CASE)
#undef ASHRT_TW_CASE
  return 0;
}

inline __host__ __device__ int fft_tw_slots(int key, int n) { return key > 0 ? (fft_tpl_twstaged(key) + 1) & ~1 : n; }
inline __host__ __device__ int fft_row_tw_slots(int key, int n) {
#define ASHRT_TW_CASE(S) \
  if (key == S) return (FftPlan<S>::twoff(FftPlan<S>::npass - 2) + 1) & ~1;
  ASHRT_TPL_SIZES(ASHRT_TW_CASE)
#undef ASHRT_TW_CASE
  return n;
}

// One butterfly's twiddles as (cos, sin) pairs: radix 8 (w^4, w^2, w,
// w e^(-i pi/4)), radix 4 (w^2, w), radix 2 (w).
template <int R>
struct Tw {
  float2 w[R / 2];
  __device__ __forceinline__ void load(const float2* tab, int Ns, int jm) {
    if constexpr (R == 2) {
      w[0] = tab[jm];
    } else {
#pragma unroll
      for (int q = 0; q < R / 4; ++q) {
        const float4 v = reinterpret_cast<const float4*>(tab)[q * Ns + jm];
        w[2 * q] = make_float2(v.x, v.y);
        w[2 * q + 1] = make_float2(v.z, v.w);
      }
    }
  }
};

// (a, b) <- (a + z b, a - z b) with z = w (ROT = 0) or -i w (ROT = 1); the
// inverse transform takes the conjugate of z.
template <bool INV, int ROT>
__device__ __forceinline__ void bfly_tw(float2& a, float2& b, float2 w) {
  const float zx = ROT == 0 ? w.x : w.y, zi = ROT == 0 ? w.y : -w.x, zy = INV ? -zi : zi;
  const float2 p = make_float2(fmaf(-zy, b.y, fmaf(zx, b.x, a.x)), fmaf(zy, b.x, fmaf(zx, b.y, a.y)));
  b = make_float2(fmaf(2.f, a.x, -p.x), fmaf(2.f, a.y, -p.y));
  a = p;
}
// The same for z = 1, -i (conjugated when INV), without multiplications.
template <bool INV, int ROT>
__device__ __forceinline__ void bfly_one(float2& a, float2& b) {
  const float2 p = ROT == 0 ? b : (INV ? make_float2(-b.y, b.x) : make_float2(b.y, -b.x));
  b = csub(a, p);
  a = cadd(a, p);
}

// In place: v_r -> DFT_R(v_r w^r).
template <int R, bool INV>
__device__ __forceinline__ void dft_tw(float2 (&v)[R], const Tw<R>& w) {
  if constexpr (R == 2) {
    bfly_tw<INV, 0>(v[0], v[1], w.w[0]);
  } else if constexpr (R == 4) {
    bfly_tw<INV, 0>(v[0], v[2], w.w[0]);
    bfly_tw<INV, 0>(v[1], v[3], w.w[0]);
    bfly_tw<INV, 0>(v[0], v[1], w.w[1]);  // outputs 0, 2
    bfly_tw<INV, 1>(v[2], v[3], w.w[1]);  // outputs 1, 3
    const float2 y2 = v[1];
    v[1] = v[2];
    v[2] = y2;
  } else {
#pragma unroll
    for (int r = 0; r < 4; ++r) bfly_tw<INV, 0>(v[r], v[r + 4], w.w[0]);
    bfly_tw<INV, 0>(v[0], v[2], w.w[1]);  // even inputs: E0 (0), E2 (2)
    bfly_tw<INV, 1>(v[4], v[6], w.w[1]);  //              E1 (4), E3 (6)
    bfly_tw<INV, 0>(v[1], v[3], w.w[1]);  // odd inputs:  O0 (1), O2 (3)
    bfly_tw<INV, 1>(v[5], v[7], w.w[1]);  //              O1 (5), O3 (7)
    bfly_tw<INV, 0>(v[0], v[1], w.w[2]);  // outputs 0, 4
    bfly_tw<INV, 1>(v[2], v[3], w.w[2]);  // outputs 2, 6
    bfly_tw<INV, 0>(v[4], v[5], w.w[3]);  // outputs 1, 5
    bfly_tw<INV, 1>(v[6], v[7], w.w[3]);  // outputs 3, 7
    const float2 y4 = v[1], y1 = v[4], y6 = v[3], y3 = v[6];
    v[1] = y1;
    v[3] = y3;
    v[4] = y4;
    v[6] = y6;
  }
}

// DFT of eight inputs, in place; HALF: inputs 4 .. 7 are zero (and not read).
template <bool INV, bool HALF = false>
__device__ __forceinline__ void dft8(float2 (&v)[8]) {
  constexpr float h = 0.70710678118654752440f;
  if constexpr (HALF) {
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r + 4] = v[r];
  } else {
#pragma unroll
    for (int r = 0; r < 4; ++r) bfly_one<INV, 0>(v[r], v[r + 4]);
  }
  bfly_one<INV, 0>(v[0], v[2]);
  bfly_one<INV, 1>(v[4], v[6]);
  bfly_one<INV, 0>(v[1], v[3]);
  bfly_one<INV, 1>(v[5], v[7]);
  bfly_one<INV, 0>(v[0], v[1]);
  bfly_one<INV, 1>(v[2], v[3]);
  bfly_tw<INV, 0>(v[4], v[5], make_float2(h, -h));
  bfly_tw<INV, 1>(v[6], v[7], make_float2(h, -h));
  const float2 y4 = v[1], y1 = v[4], y6 = v[3], y3 = v[6];
  v[1] = y1;
  v[3] = y3;
  v[4] = y4;
  v[6] = y6;
}

template <int R, bool INV>
__device__ __forceinline__ void dft_r(float2 (&v)[R]) {
  if constexpr (R == 8) dft8<INV>(v);
  else butterfly<R, INV>(v);
}

// One pass's twiddles of a batch of NBN / N length-N transforms by NT
// threads, for the butterflies threadIdx.x + i NT: they depend on the thread
// alone, so a kernel loads them once and uses them for every transform.
template <int N, int NT, int NBN, int PASS>
struct PassTw {
  static constexpr int R = FftPlan<N>::radix(PASS);
  static constexpr int Ns = FftPlan<N>::ns(PASS);
  static constexpr int MAXB = (NBN / R + NT - 1) / NT;
  Tw<R> w[MAXB];
  __device__ __forceinline__ void load(const float2* __restrict__ tab) {
#pragma unroll
    for (int i = 0; i < MAXB; ++i)
      w[i].load(tab + FftPlan<N>::twoff(PASS), Ns, (int)((threadIdx.x + i * NT) % (N / R)) % Ns);
  }
  // Waits for the loads and keeps the values in registers: without this the
  // compiler may load them again at every use.
  __device__ __forceinline__ void pin() {
#pragma unroll
    for (int i = 0; i < MAXB; ++i)
#pragma unroll
      for (int q = 0; q < R / 2; ++q) asm volatile("" : "+v"(w[i].w[q].x), "+v"(w[i].w[q].y));
  }
};

// The register twiddles of a transform: its last pass (FIRST = npass - 1) or
// its last two (FIRST = npass - 2), the earlier passes reading LDS.
template <int N, int NT, int NBN = N, int REGS = 1>
struct RegTw {
  static constexpr int L = FftPlan<N>::npass - 1;
  static constexpr int FIRST = L + 1 - REGS;
  static_assert(FIRST >= 1, "the first pass has no twiddles");
  static_assert(FftPlan<N>::ns(L) * FftPlan<N>::radix(L) == N, "the last pass spans N");
  PassTw<N, NT, NBN, L> last;
  PassTw<N, NT, NBN, FIRST> prev;  // FIRST == L: unused
  __device__ __forceinline__ void load(const float2* __restrict__ tab) {
    last.load(tab);
    if constexpr (REGS == 2) prev.load(tab);
  }
  __device__ __forceinline__ void pin() {
    last.pin();
    if constexpr (REGS == 2) prev.pin();
  }
};

// Pair layout of a length-N spectrum whose bins 0 and N/2 are not needed:
// pair k (1 <= k < N/2) holds bin k at float2 slot 2k and bin N-k at slot
// 2k+1, so a map that touches both mirror bins of k reads 16 bytes at once.
// The pairs occupy the first N float2 slots of the transform's buffer.
template <int N>
__device__ __forceinline__ float2 pair_get(const float2* buf, int i) {
  if (i == 0 || i == N / 2) return make_float2(0.f, 0.f);
  return i < N / 2 ? buf[2 * i] : buf[2 * (N - i) + 1];
}

template <int N>
__device__ __forceinline__ void pair_put(float2* buf, int o, float2 v) {
  if (o == 0 || o == N / 2) return;
  if (o < N / 2) buf[2 * o] = v;
  else buf[2 * (N - o) + 1] = v;
}

// One pass of a batch of nb transforms (nb * N <= NBN) at buf + b*bstride,
// run by a workgroup of NT threads.  IO = 1: this pass reads its input from
// the pair layout; IO = 2: it writes its output in the pair layout (bins 0
// and N/2 dropped; one transform: pair 0 and slots N .. N+7 are zeroed); IO = 3: inputs at index >= nvalid are taken as zero (and
// never read); IO = 4: outputs at index >= nvalid are dropped; IO = 0:
// padded layout both ways.  Reads complete before the barrier and writes
// follow it, so the layouts may share memory.
// lw: the last passes' twiddles in registers (RegTw).
template <int N, int PASS, int NBN, bool INV, int NT, int IO, class LW>
__device__ __forceinline__ void tpl_pass(float2* buf, int nb, int bstride, const float2* twp, int nvalid,
                                         const LW& lw) {
  using P = FftPlan<N>;
  constexpr int R = P::radix(PASS);
  constexpr int Ns = P::ns(PASS);
  constexpr int B = N / R;
  constexpr int TW = P::twoff(PASS);
  constexpr int MAXB = (NBN / R + NT - 1) / NT;
  // reads x[j + r B], j < B; writes y[jq Ns R + jm + r Ns], jm < Ns
  constexpr bool RLIN = IO != 1 && pad_linear(B, R, 0, B);
  constexpr bool WLIN = IO != 2 && IO != 4 && pad_linear(Ns, R, Ns * R, Ns);
  // one transform whose butterflies split evenly over the NT threads of the
  // workgroup: every id below is a butterfly, so no lane test is needed
  constexpr bool FULL = NBN == N && B % NT == 0;
  float2 v[MAXB][R];
  int dst[MAXB], bq[MAXB];
  const int total = B * nb;
  const int tid = pass_tid();
#pragma unroll
  for (int i = 0; i < MAXB; ++i) {
    const int id = tid + i * NT;
    dst[i] = -1;
    if (FULL || id < total) {
      // one transform (NBN == N) has b = 0; indices are non-negative, so
      // unsigned division by the compile-time B and Ns is a shift or mul_hi
      const int b = NBN == N ? 0 : (int)((unsigned)id / (unsigned)B);
      const int j = id - b * B;
      const int jq = (int)((unsigned)j / (unsigned)Ns);
      const int jm = j - jq * Ns;
      const float2* src = buf + b * bstride;
      const float2* s0 = src + fft_pad(j);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if constexpr (IO == 1 && R % 2 == 0) {
          // B R = N and j < B: element j + r B lies below N/2 exactly when
          // r < R/2, so each read is one of two bases plus a constant
          // (elements 0 and N/2, for j = 0, read a valid slot and are zeroed)
          if (r < R / 2) {
            const float2 x = src[2 * j + 2 * r * B];
            v[i][r] = (r == 0 && j == 0) ? make_float2(0.f, 0.f) : x;
          } else {
            const float2 x = src[2 * (N - j) + 1 - 2 * r * B];
            v[i][r] = (r == R / 2 && j == 0) ? make_float2(0.f, 0.f) : x;
          }
        } else if constexpr (IO == 1) v[i][r] = pair_get<N>(src, j + r * B);
        else if constexpr (IO == 3 && RLIN) v[i][r] = (j + r * B < nvalid) ? s0[fft_pad(r * B)] : make_float2(0.f, 0.f);
        else if constexpr (IO == 3) v[i][r] = (j + r * B < nvalid) ? src[fft_pad(j + r * B)] : make_float2(0.f, 0.f);
        else if constexpr (RLIN) v[i][r] = s0[fft_pad(r * B)];
        else v[i][r] = src[fft_pad(j + r * B)];
      }
      if constexpr (Ns > 1) {
        Tw<R> w;
        if constexpr (PASS == P::npass - 1) w = lw.last.w[i];
        else if constexpr (PASS >= LW::FIRST) w = lw.prev.w[i];
        else w.load(twp + TW, Ns, jm);
        dft_tw<R, INV>(v[i], w);
      } else {
        dft_r<R, INV>(v[i]);
      }
      bq[i] = jq * Ns * R + jm;
      // padded layout: dst is the padded address of bq, and bq keeps only
      // its low four bits when the steps r Ns need them
      if constexpr (IO == 2 || IO == 4) {
        dst[i] = b * bstride;
      } else {
        dst[i] = b * bstride + fft_pad(bq[i]);
        bq[i] &= 15;
      }
    }
  }
  __syncthreads();
  if constexpr (IO == 2) {
    // pair 0 (bins 0 and N) and pairs N/2 .. N/2 + 3 (slots N .. N + 7, in
    // the padding) are left zero: a map reading taps there gets zeros
    static_assert(N >= 128, "pair output needs eight padding slots");
    if (tid < 10) buf[tid < 2 ? tid : N + tid - 2] = make_float2(0.f, 0.f);
  }
#pragma unroll
  for (int i = 0; i < MAXB; ++i) {
    if (FULL || dst[i] >= 0) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if constexpr (IO == 2 && R % 2 == 0 && Ns * R == N) {
          // last pass: bq = jm < Ns, so output jm + r Ns lies below N/2
          // exactly when r < R/2 (outputs 0 and N/2, for jm = 0, are dropped)
          if (r < R / 2) {
            if (r != 0 || bq[i] != 0) buf[dst[i] + 2 * bq[i] + 2 * r * Ns] = v[i][r];
          } else {
            if (r != R / 2 || bq[i] != 0) buf[dst[i] + 2 * (N - bq[i]) + 1 - 2 * r * Ns] = v[i][r];
          }
        } else if constexpr (IO == 2) {
          pair_put<N>(buf + dst[i], bq[i] + r * Ns, v[i][r]);
        } else if constexpr (IO == 4) {
          if (bq[i] + r * Ns < nvalid) buf[dst[i] + fft_pad(bq[i] + r * Ns)] = v[i][r];
        } else if constexpr (WLIN) {
          buf[dst[i] + fft_pad(r * Ns)] = v[i][r];
        } else {
          buf[pad_step(dst[i], bq[i], r * Ns)] = v[i][r];
        }
      }
    }
  }
  __syncthreads();
}

// PAIRS_IN: the first pass reads the pair layout; PAIRS_OUT: the last pass
// writes it.
// Passes PASS .. END-1 (END defaults to all of them).  MASK_IN: the first
// pass reads only indices < nvalid (the rest is zero); MASK_OUT: the last
// pass writes only indices < nvalid.
template <int N, int PASS, int NBN, bool INV, int NT, bool PAIRS_IN = false, bool PAIRS_OUT = false,
          int END = FftPlan<N>::npass, bool MASK_IN = false, bool MASK_OUT = false, class LW>
__device__ __forceinline__ void tpl_passes(float2* buf, int nb, int bstride, const float2* twp, int nvalid,
                                           const LW& lw) {
  if constexpr (PASS < END) {
    constexpr bool last = PASS == FftPlan<N>::npass - 1;
    constexpr int IO = (PAIRS_IN && PASS == 0)   ? 1
                       : (PAIRS_OUT && last)     ? 2
                       : (MASK_IN && PASS == 0)  ? 3
                       : (MASK_OUT && last)      ? 4
                                                 : 0;
    static_assert(!(PAIRS_IN && PAIRS_OUT && FftPlan<N>::npass == 1), "pair input and output need two passes");
    static_assert(!(MASK_IN && MASK_OUT && FftPlan<N>::npass == 1), "masked input and output need two passes");
    tpl_pass<N, PASS, NBN, INV, NT, IO>(buf, nb, bstride, twp, nvalid, lw);
    tpl_passes<N, PASS + 1, NBN, INV, NT, PAIRS_IN, PAIRS_OUT, END, MASK_IN, MASK_OUT>(buf, nb, bstride, twp, nvalid,
                                                                                      lw);
  }
}

// Full transform(s) of inputs that are zero at index >= nvalid (MASK_IN:
// those slots are never read, so they need not be filled) or of which only
// outputs < nvalid are wanted (MASK_OUT: the others are not written).
template <int N, int NBN, bool INV, bool MASK_IN, bool MASK_OUT, int NT = kThreads, class LW>
__device__ __forceinline__ void fft_tpl_masked(float2* buf, int nb, int bstride, const float2* twp, int nvalid,
                                               const LW& lw) {
  tpl_passes<N, 0, NBN, INV, NT, false, false, FftPlan<N>::npass, MASK_IN, MASK_OUT>(buf, nb, bstride, twp, nvalid,
                                                                                    lw);
}

// One transform of length N whose output is left in the pair layout.
template <int N, bool INV, int NT, class LW>
__device__ __forceinline__ void fft_tpl_to_pairs(float2* buf, const float2* twp, const LW& lw) {
  tpl_passes<N, 0, N, INV, NT, false, true>(buf, 1, fft_padlen(N), twp, N, lw);
}

// First-pass inputs of a length-N transform held in registers: the
// butterfly with id = threadIdx.x + i NT takes x[id + r N/R0], r < R0 (R0 the
// first radix), so a caller can load them straight from global memory.
// HALF (radix-8 first passes): rows at most N/2 long, the default padding;
// the inputs r >= R0/2 are zero, and neither held, loaded nor added.
template <int N, int NT, bool HALF>
struct FftRegsIn {
  static constexpr int R = FftPlan<N>::radix(0);
  static constexpr int B = N / R;
  static constexpr int MAXB = (B + NT - 1) / NT;
  static constexpr int RIN = HALF ? R / 2 : R;
  static_assert(FftPlan<N>::npass >= 2, "register input needs a later pass to write the pair layout");
  static_assert(!HALF || R == 8, "half inputs need a radix-8 first pass");
  float2 v[MAXB][RIN];
  // x[t] = src[t] for t < nt, zero after (HALF: nt <= N/2)
  __device__ __forceinline__ void load(const float2* __restrict__ src, int nt) {
    const int tid = pass_tid();
#pragma unroll
    for (int i = 0; i < MAXB; ++i) {
      const int id = tid + i * NT;
#pragma unroll
      for (int r = 0; r < RIN; ++r) {
        const int t = id + r * B;
        v[i][r] = ((B % NT == 0 || id < B) && t < nt) ? src[t] : make_float2(0.f, 0.f);
      }
    }
  }
};

// Transform whose first pass takes its inputs from registers (no twiddles
// there: its span is 1) and whose output is left in the pair layout, in two
// calls: regs_pass0 (the caller must have finished every read of buf; the
// registers are free again when it returns) and rest_to_pairs.
template <int N, bool INV, int NT, bool HALF>
__device__ __forceinline__ void fft_tpl_regs_pass0(float2* buf, const FftRegsIn<N, NT, HALF>& in) {
  using I = FftRegsIn<N, NT, HALF>;
  const int tid = pass_tid();
#pragma unroll
  for (int i = 0; i < I::MAXB; ++i) {
    const int id = tid + i * NT;
    if (I::B % NT == 0 || id < I::B) {
      float2 v[I::R];
#pragma unroll
      for (int r = 0; r < I::RIN; ++r) v[r] = in.v[i][r];
      if constexpr (HALF) dft8<INV, true>(v);
      else dft_r<I::R, INV>(v);
      constexpr bool LIN = pad_linear(1, I::R, I::R, 1);
      const int p0 = fft_pad(id * I::R), lo = (id * I::R) & 15;
#pragma unroll
      for (int r = 0; r < I::R; ++r) {
        if constexpr (LIN) buf[p0 + r] = v[r];
        else buf[pad_step(p0, lo, r)] = v[r];
      }
    }
  }
  __syncthreads();
}

template <int N, bool INV, int NT, class LW>
__device__ __forceinline__ void fft_tpl_rest_to_pairs(float2* buf, const float2* twp, const LW& lw) {
  tpl_passes<N, 1, N, INV, NT, false, true>(buf, 1, fft_padlen(N), twp, N, lw);
}

// Outputs of a length-N transform's last pass held in registers: the
// butterfly with id = threadIdx.x + i NT (id < N/RL, RL the last radix) holds
// output element id + r N/RL in v[i][r], so a caller can store them
// straight to global memory.
template <int N, int NT>
struct FftRegsOut {
  static constexpr int L = FftPlan<N>::npass - 1;
  static constexpr int R = FftPlan<N>::radix(L);
  static constexpr int B = N / R;
  static constexpr int MAXB = (B + NT - 1) / NT;
  static_assert(L >= 1 && FftPlan<N>::ns(L) == B, "the last pass spans N/R");
  float2 v[MAXB][R];
};

// Passes FIRST .. last of a transform (FIRST reading the pair layout when
// PAIRS_IN, for FIRST == 0) whose last pass leaves its outputs in
// registers; buf may be reused once every thread has passed a barrier after
// this returns.
template <int N, bool INV, int NT, int FIRST, bool PAIRS_IN, class LW>
__device__ __forceinline__ void fft_tpl_passes_to_regs(float2* buf, const float2* twp, const LW& lw,
                                                       FftRegsOut<N, NT>& out) {
  using O = FftRegsOut<N, NT>;
  static_assert(!PAIRS_IN || FIRST == 0, "only the first pass reads pairs");
  tpl_passes<N, FIRST, N, INV, NT, PAIRS_IN, false, O::L>(buf, 1, fft_padlen(N), twp, N, lw);
  const int tid = pass_tid();
#pragma unroll
  for (int i = 0; i < O::MAXB; ++i) {
    const int id = tid + i * NT;
    if (O::B % NT == 0 || id < O::B) {
      constexpr bool LIN = pad_linear(O::B, O::R, 0, O::B);
      const float2* s0 = buf + fft_pad(id);
#pragma unroll
      for (int r = 0; r < O::R; ++r) out.v[i][r] = LIN ? s0[fft_pad(r * O::B)] : buf[fft_pad(id + r * O::B)];
      dft_tw<O::R, INV>(out.v[i], lw.last.w[i]);
    }
  }
}

// Transform whose input is read from the pair layout (bins 0 and N/2 taken
// as zero) and whose last pass leaves its outputs in registers.
template <int N, bool INV, int NT, class LW>
__device__ __forceinline__ void fft_tpl_from_pairs_to_regs(float2* buf, const float2* twp, const LW& lw,
                                                           FftRegsOut<N, NT>& out) {
  fft_tpl_passes_to_regs<N, INV, NT, 0, true>(buf, twp, lw, out);
}

}  // namespace ashrt

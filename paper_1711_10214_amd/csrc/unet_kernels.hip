// HIP kernels of the warm-start U-Net for gfx950.
//
// 3x3 convolutions (forward and input-gradient) and their weight gradients
// run on the BF16 matrix cores, v_mfma_f32_16x16x32_bf16: a wave multiplies
// a 16 x 32 BF16 tile A by a 32 x 16 tile B into a 16 x 16 FP32 tile.
// Lane l supplies A[l % 16][8 (l / 16) + i] and B[8 (l / 16) + i][l % 16]
// (i = 0..7, eight consecutive BF16 values = 16 bytes) and receives
// D[4 (l / 16) + i][l % 16] (i = 0..3).
//
// Forward convolution: A = packed weights (rows = output channels, k =
// (tap, input channel)), B = the input tile staged in LDS as [row][col][ci]
// (so eight consecutive channels of one tap are one 16-byte read), D =
// output channels x pixels, written as four consecutive channels of one
// pixel (NHWC).  The input-gradient is the same kernel on the gradient of
// the output's pre-activation with the transposed, tap-flipped weights; its
// epilogue routes the result to the tensors the forward input was built
// from (ConvRoute).  Launches with few workgroups split the channel chunks
// over workgroups and finish in k_conv_finish.
// Weight gradient: A = output gradient, B = input, k = pixels, both staged
// [pixel][channel] and read with the LDS transpose read; workgroups split
// the pixels and write FP32 partials that one kernel for all layers sums in
// a fixed order.
#include "unet_internal.h"

#include <type_traits>

namespace unet {

typedef __bf16 bf16x8 __attribute__((__vector_size__(8 * sizeof(__bf16))));
typedef float f32x4 __attribute__((__vector_size__(4 * sizeof(float))));

__device__ __forceinline__ float bf2f(uint32_t h) { return __uint_as_float(h << 16); }

// Two FP32 -> BF16 bit pairs, round to nearest even (v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint32_t f2bf2(float lo, float hi) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){lo, hi}, bf16x2));
}

__device__ __forceinline__ uint4 pack8(const float v[8]) {
  return make_uint4(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]), f2bf2(v[4], v[5]), f2bf2(v[6], v[7]));
}

__device__ __forceinline__ void unpack8(uint4 q, float v[8]) {
  v[0] = bf2f(q.x & 0xFFFFu);
  v[1] = bf2f(q.x >> 16);
  v[2] = bf2f(q.y & 0xFFFFu);
  v[3] = bf2f(q.y >> 16);
  v[4] = bf2f(q.z & 0xFFFFu);
  v[5] = bf2f(q.z >> 16);
  v[6] = bf2f(q.w & 0xFFFFu);
  v[7] = bf2f(q.w >> 16);
}

// ReLU derivative from the stored (post-ReLU) BF16 output: 1 where it is > 0.
__device__ __forceinline__ bool relu_on(uint32_t h) { return (h & 0x8000u) == 0 && (h & 0x7FFFu) != 0; }

__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Stages a ROWS x COLS pixel tile of 8 NG channels of a convolution's input
// into LDS as [pixel][channel], pixel stride PS BF16 values, in two calls:
// fetch issues the global loads into registers (so that they fly under the
// multiplies of the tile before) and store rounds and writes them.  A task is
// one pixel's group of 8 channels; a thread's tasks all have the same channel
// group and lie 256 / NG pixels apart, so their indices are found once per
// workgroup (init) and their LDS places are constants apart: with the indices
// recomputed per chunk by run-time divisions the convolutions were bound by
// integer arithmetic (24 M VALU instructions in 22 M CU cycles at 4 x 1024 x 256
// pixels, 16 channels).  Outside the image and beyond the real channels the
// tile is zero.  MODE: ConvIn::modeA (a pooled A has no skip); FP32 inputs are
// at the same resolution and alone.  Ca and Cb are multiples of 8 unless Ca == 1
// (the FP32 network input).
template <bool AF32, int MODE, int NG, int ROWS, int COLS, int PS>
struct TileStage {
  static constexpr int N = ROWS * COLS * NG;
  static constexpr int S = (N + 255) / 256;
  static_assert(256 % NG == 0 && S <= 32, "tasks of a thread share a channel group; one bit each");
  static_assert(!AF32 || MODE == 0, "FP32 inputs are at the same resolution");
  int po[S];              // pixel offset of each task from the tile's first pixel
  int ph[MODE == 1 ? S : 1];  // the same in the half-resolution A
  long long org, orgA;    // the tile's first pixel and its A pixel (of the batch's pixels in order)
  unsigned ok;            // bit u: task u lies in the image
  float4 f0[AF32 ? S : 1], f1[AF32 ? S : 1];
  uint4 q[AF32 ? 1 : S];

  __device__ __forceinline__ void init(const ConvIn& I, int b, int y0, int x0) {
    const int pix0 = (int)threadIdx.x / NG;
    ok = 0;
    org = ((long long)b * I.H + y0) * I.W + x0;
    if constexpr (MODE == 0) orgA = org;
    if constexpr (MODE == 1) orgA = ((long long)b * (I.H >> 1) + (y0 >> 1)) * (I.W >> 1) + (x0 >> 1);
    if constexpr (MODE == 2) orgA = ((long long)b * (2 * I.H) + 2 * y0) * (2 * I.W) + 2 * x0;
#pragma unroll
    for (int u = 0; u < S; ++u) {
      const int pix = pix0 + u * (256 / NG);
      const int r = pix / COLS, x = pix - r * COLS;
      const int yy = y0 + r, xx = x0 + x;
      const bool in = pix < ROWS * COLS && yy >= 0 && yy < I.H && xx >= 0 && xx < I.W;
      ok |= in ? 1u << u : 0u;
      po[u] = (MODE == 2 ? 4 * r * I.W + 2 * x : r * I.W + x);
      if constexpr (MODE == 1) ph[u] = ((yy >> 1) - (y0 >> 1)) * (I.W >> 1) + ((xx >> 1) - (x0 >> 1));
    }
  }

  // channels [c0, c0 + 8 NG)
  __device__ __forceinline__ void fetch(const ConvIn& I, int c0) {
    const int c = c0 + ((int)threadIdx.x % NG) * 8;
    const bool inA = c < I.Ca;
    if constexpr (AF32) {
      const float* p = static_cast<const float*>(I.A) + orgA * I.Ca + c;
#pragma unroll
      for (int u = 0; u < S; ++u) {
        f0[u] = f1[u] = make_float4(0.f, 0.f, 0.f, 0.f);
        if ((ok >> u & 1u) && inA) {
          const float* t = p + (long long)po[u] * I.Ca;
          if (I.Ca == 1) {
            f0[u].x = *t;
          } else {
            f0[u] = *reinterpret_cast<const float4*>(t);
            f1[u] = *reinterpret_cast<const float4*>(t + 4);
          }
        }
      }
    } else if constexpr (MODE == 2) {
      const uint16_t* p = static_cast<const uint16_t*>(I.A) + orgA * I.Ca + c;
      const long long row = 2LL * I.W * I.Ca;
#pragma unroll
      for (int u = 0; u < S; ++u) {
        q[u] = make_uint4(0u, 0u, 0u, 0u);
        if ((ok >> u & 1u) && inA) {
          float v[8], t[8];
          const uint16_t* s = p + (long long)po[u] * I.Ca;
          const uint4 h[4] = {*reinterpret_cast<const uint4*>(s), *reinterpret_cast<const uint4*>(s + I.Ca),
                              *reinterpret_cast<const uint4*>(s + row),
                              *reinterpret_cast<const uint4*>(s + row + I.Ca)};
          unpack8(h[0], v);
#pragma unroll
          for (int k = 1; k < 4; ++k) {
            unpack8(h[k], t);
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] += t[i];
          }
#pragma unroll
          for (int i = 0; i < 8; ++i) v[i] *= 0.25f;
          q[u] = pack8(v);
        }
      }
    } else {
      const uint16_t* p = inA ? static_cast<const uint16_t*>(I.A) + orgA * I.Ca + c : I.Bs + org * I.Cb + (c - I.Ca);
      const int C = inA ? I.Ca : I.Cb;
      const bool live = c < I.Ca + I.Cb;
#pragma unroll
      for (int u = 0; u < S; ++u) {
        q[u] = make_uint4(0u, 0u, 0u, 0u);
        if ((ok >> u & 1u) && live) {
          int o = po[u];
          if constexpr (MODE == 1) {
            const int h = ph[u];
            o = inA ? h : o;
          }
          q[u] = *reinterpret_cast<const uint4*>(p + (long long)o * C);
        }
      }
    }
  }

  __device__ __forceinline__ void store(uint16_t* dst) const {
    uint16_t* d = dst + ((int)threadIdx.x / NG) * PS + ((int)threadIdx.x % NG) * 8;
#pragma unroll
    for (int u = 0; u < S; ++u) {
      if (N % 256 != 0 && u == S - 1 && (int)threadIdx.x + u * 256 >= N) continue;
      uint4 w;
      if constexpr (AF32) {
        const float v[8] = {f0[u].x, f0[u].y, f0[u].z, f0[u].w, f1[u].x, f1[u].y, f1[u].z, f1[u].w};
        w = pack8(v);
      } else {
        w = q[u];
      }
      *reinterpret_cast<uint4*>(d + u * (256 / NG) * PS) = w;
    }
  }
};

// ------------------------------------------------------------ routed epilogue
// float4 store or accumulate of four consecutive channels, each zeroed where
// the activation m (four BF16 values, or null: none) is not positive.
__device__ __forceinline__ void put4(float* p, const uint16_t* m, float v0, float v1, float v2, float v3, bool add) {
  if (m) {
    const uint2 h = *reinterpret_cast<const uint2*>(m);
    if (!relu_on(h.x & 0xFFFFu)) v0 = 0.f;
    if (!relu_on(h.x >> 16)) v1 = 0.f;
    if (!relu_on(h.y & 0xFFFFu)) v2 = 0.f;
    if (!relu_on(h.y >> 16)) v3 = 0.f;
  }
  float4 o = make_float4(v0, v1, v2, v3);
  if (add) {
    const float4 q = *reinterpret_cast<const float4*>(p);
    o.x += q.x;
    o.y += q.y;
    o.z += q.z;
    o.w += q.w;
  }
  *reinterpret_cast<float4*>(p) = o;
}

// The value held by lane l ^ 1 (DPP quad permutation 1, 0, 3, 2).
__device__ __forceinline__ float lane_pair_swap(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, false));
}

// Epilogue of an input-gradient convolution (see ConvRoute): lane (sub, n16)
// holds channels co0 + 16 mi + 4 sub + [0, 4) of the pixels (y0 + rr, tx0 + 16
// ni + n16).  An upsampled A (UP, mode 1) sums each 2 x 2 pixel block, (g00 +
// g01) + (g10 + g11): the two columns by a lane exchange, then the wave's two
// rows; the even lanes store the first column tile's sums and the odd lanes
// the second's (16-channel tiles lie wholly in A or in B there, Ca being a
// multiple of 16).  UP is a template parameter so that the other input
// gradients do not carry its registers.
template <int MT, int NTL, int RW, bool UP>
__device__ __forceinline__ void route_store(const ConvArgs& a, f32x4 (&acc)[RW][MT][NTL], int b, int y0, int tx0,
                                            int co0) {
  const ConvRoute& R = a.rt;
  const int H = a.in.H, W = a.in.W;
  const int lane = (int)threadIdx.x & 63;
  const int sub = lane >> 4, n16 = lane & 15;
  if constexpr (UP) {
    static_assert(RW == 2 && NTL == 2, "a wave holds whole 2 x 2 blocks of two column tiles");
    const int Hh = H >> 1, Wh = W >> 1;
    const bool odd = n16 & 1;
    const int yh = y0 >> 1, xh = (tx0 + (odd ? 16 : 0) + n16) >> 1;
#pragma unroll
    for (int mi = 0; mi < MT; ++mi) {
      const int co = co0 + mi * 16 + sub * 4;
      if (co0 + mi * 16 >= R.Ca) continue;
      float t[NTL][4];
#pragma unroll
      for (int ni = 0; ni < NTL; ++ni)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float r0 = acc[0][mi][ni][i] + lane_pair_swap(acc[0][mi][ni][i]);
          const float r1 = acc[1][mi][ni][i] + lane_pair_swap(acc[1][mi][ni][i]);
          t[ni][i] = r0 + r1;
        }
      if (yh < Hh && xh < Wh) {
        const long long oa = (((long long)b * Hh + yh) * Wh + xh) * R.Ca + co;
        put4(R.gA + oa, R.mA ? R.mA + oa : nullptr, odd ? t[1][0] : t[0][0], odd ? t[1][1] : t[0][1],
             odd ? t[1][2] : t[0][2], odd ? t[1][3] : t[0][3], R.accA != 0);
      }
    }
  }
#pragma unroll
  for (int mi = 0; mi < MT; ++mi) {
    const int co = co0 + mi * 16 + sub * 4;
    if (co >= R.Ca + R.Cb) continue;
    if (UP && co < R.Ca) continue;  // stored above
#pragma unroll
    for (int rr = 0; rr < RW; ++rr) {
      const int y = y0 + rr;
      if (y >= H) continue;
#pragma unroll
      for (int ni = 0; ni < NTL; ++ni) {
        const int x = tx0 + ni * 16 + n16;
        if (x >= W) continue;
        const f32x4 o = acc[rr][mi][ni];
        if (co >= R.Ca) {
          const long long ob = (((long long)b * H + y) * W + x) * R.Cb + (co - R.Ca);
          put4(R.gB + ob, R.mB ? R.mB + ob : nullptr, o[0], o[1], o[2], o[3], R.accB != 0);
        } else if (R.modeA == 0) {
          const long long oa = (((long long)b * H + y) * W + x) * R.Ca + co;
          put4(R.gA + oa, R.mA ? R.mA + oa : nullptr, o[0], o[1], o[2], o[3], R.accA != 0);
        } else {
          // mode 2 (pooled A): an upsampled A (mode 1) always launches with UP
          // set, or split with the route left to k_conv_finish
          const int H2 = 2 * H, W2 = 2 * W;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const long long oa = (((long long)b * H2 + 2 * y + (q >> 1)) * W2 + 2 * x + (q & 1)) * R.Ca + co;
            put4(R.gA + oa, R.mA ? R.mA + oa : nullptr, 0.25f * o[0], 0.25f * o[1], 0.25f * o[2], 0.25f * o[3],
                 R.accA != 0);
          }
        }
      }
    }
  }
}

// LDS pixel stride of a conv tile in BF16 values.  A fragment read takes 16
// consecutive pixels' 16-byte groups, and the hardware serves lanes 0-3, 12-15
// of one group together with lanes 4-11 of the next: strides of 2 mod 4 groups
// keep the 16 of them on different banks for any first pixel.
constexpr int conv_ps(int CC) { return CC == 32 ? 48 : CC; }

// ------------------------------------------------------------ 3x3 convolution
// Grid: (row tiles x column tiles, output-channel tiles of 16 MT, batch x
// ksplit).  Wave w computes output rows RW w .. RW w + RW - 1 of the tile: MT x
// NTL MFMA tiles (16 MT channels x 16 NTL columns) of each.  The taps are
// unrolled, every LDS offset a constant, and the next chunk's tile is loaded
// while this one multiplies.  Whatever the tile, an output value adds the same
// products in the same order (chunks, then taps, 32 at a time), so the rounded
// activations do not depend on it.
// Level-0 and level-1 input gradients are bound by their FP32 tensors (16 -> 16
// channels at 4 x 1024 x 256 pixels: 167 MB in 35 us), the others by the LDS and
// L1 reads of the fragments (64 -> 64 at 4 x 256 x 64: 15 us for 4 us of products).
template <bool AF32, bool OUTF32, int MODE, int CC, int MT, int NTL, int RW, bool UP>
__global__ __launch_bounds__(256) void k_conv3(ConvArgs a) {
  constexpr int TW = 16 * NTL, TW2 = TW + 2, TH = 4 * RW, PS = conv_ps(CC), NG = CC / 8;
  constexpr int TPK = 32 / CC, KS = (9 + TPK - 1) / TPK;  // taps per k-step, k-steps per chunk
  constexpr int PF = 3;                                   // weight fragments held: this k-step's and the next two
  static_assert(TPK > 1 || KS % PF == 0, "the fragment rotation restarts with each chunk");
  __shared__ __attribute__((aligned(16))) uint16_t sX[(TH + 2) * TW2 * PS];
  const int H = a.in.H, W = a.in.W;
  const int tiles_x = (W + TW - 1) / TW;
  const int ty0 = ((int)blockIdx.x / tiles_x) * TH;
  const int tx0 = ((int)blockIdx.x % tiles_x) * TW;
  const int co0 = (int)blockIdx.y * 16 * MT, b = (int)blockIdx.z % a.B, ks = (int)blockIdx.z / a.B;
  const int wave = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63;
  const int sub = lane >> 4, n16 = lane & 15;
  const ConvPack& P = a.pk;
  const int y0 = ty0 + RW * wave;

  f32x4 acc[RW][MT][NTL];
#pragma unroll
  for (int rr = 0; rr < RW; ++rr)
#pragma unroll
    for (int mi = 0; mi < MT; ++mi)
#pragma unroll
      for (int ni = 0; ni < NTL; ++ni) acc[rr][mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};

  // LDS offset of this lane's tap of k-step kc from its first pixel; tap past the ninth: no product
  const uint16_t* const bx = sX + (RW * wave * TW2 + n16) * PS + (sub * 8) % CC;
  auto tap_off = [&](int kc) {
    if constexpr (TPK == 1) {
      return ((kc / 3) * TW2 + kc % 3) * PS;
    } else {
      const int t = kc * TPK + (sub * 8) / CC, tt = t < 9 ? t : 0;
      return ((tt / 3) * TW2 + tt % 3) * PS;
    }
  };

  // packed weights of output channel co0 + 16 mi + n16: the k-steps of the
  // whole reduction are consecutive blocks of 32
  const uint16_t* wrow[MT];
  const int cc_lo = ks * P.ncc / a.ksplit, cc_hi = (ks + 1) * P.ncc / a.ksplit;
#pragma unroll
  for (int mi = 0; mi < MT; ++mi)
    wrow[mi] = a.Wp + ((long long)(co0 + mi * 16 + n16) * P.ncc + cc_lo) * (KS * 32) + sub * 8;
  uint4 wq[PF][MT];
#pragma unroll
  for (int s = 0; s < PF - 1; ++s)
#pragma unroll
    for (int mi = 0; mi < MT; ++mi) wq[s][mi] = *reinterpret_cast<const uint4*>(wrow[mi] + s * 32);

  TileStage<AF32, MODE, NG, TH + 2, TW2, PS> st;
  st.init(a.in, b, ty0 - 1, tx0 - 1);
  st.fetch(a.in, cc_lo * CC);
  for (int cc = cc_lo; cc < cc_hi; ++cc) {
    st.store(sX);
    __syncthreads();
    const bool more = TPK == 1 && cc + 1 < cc_hi;  // channel counts below 32 are one chunk
    if (more) st.fetch(a.in, (cc + 1) * CC);
#pragma unroll
    for (int kc = 0; kc < KS; ++kc) {
      if (kc + PF - 1 < KS || more) {
#pragma unroll
        for (int mi = 0; mi < MT; ++mi)
          wq[(kc + PF - 1) % PF][mi] = *reinterpret_cast<const uint4*>(wrow[mi] + (kc + PF - 1) * 32);
      }
      const int to = tap_off(kc);
      const bool none = kc * TPK + (sub * 8) / CC >= 9;
#pragma unroll
      for (int rr = 0; rr < RW; ++rr) {
        bf16x8 bf[NTL];
#pragma unroll
        for (int ni = 0; ni < NTL; ++ni) {
          uint4 q = *reinterpret_cast<const uint4*>(bx + to + (rr * TW2 + ni * 16) * PS);
          if (TPK > 1 && kc == KS - 1 && none) q = make_uint4(0u, 0u, 0u, 0u);
          bf[ni] = __builtin_bit_cast(bf16x8, q);
        }
#pragma unroll
        for (int mi = 0; mi < MT; ++mi)
#pragma unroll
          for (int ni = 0; ni < NTL; ++ni)
            acc[rr][mi][ni] = mfma(__builtin_bit_cast(bf16x8, wq[kc % PF][mi]), bf[ni], acc[rr][mi][ni]);
      }
    }
    if (more) {
#pragma unroll
      for (int mi = 0; mi < MT; ++mi) wrow[mi] += KS * 32;
      __syncthreads();
    }
  }

  if (!UP && a.ksplit > 1) {  // the upsampled route is launched unsplit
    // raw partial sums of this split; the finishing kernel applies the epilogue
#pragma unroll
    for (int rr = 0; rr < RW; ++rr) {
      const int y = y0 + rr;
      if (y >= H) continue;
#pragma unroll
      for (int mi = 0; mi < MT; ++mi) {
        const int co = co0 + mi * 16 + sub * 4;
#pragma unroll
        for (int ni = 0; ni < NTL; ++ni) {
          const int x = tx0 + ni * 16 + n16;
          if (x >= W) continue;
          const long long off = ((((long long)ks * a.B + b) * H + y) * W + x) * P.Coutp + co;
          *reinterpret_cast<float4*>(a.kpart + off) =
              make_float4(acc[rr][mi][ni][0], acc[rr][mi][ni][1], acc[rr][mi][ni][2], acc[rr][mi][ni][3]);
        }
      }
    }
    return;
  }
  if constexpr (OUTF32) {
    // FP32 outputs are input gradients, always routed (launch_conv3)
    route_store<MT, NTL, RW, UP>(a, acc, b, y0, tx0, co0);
  } else {
#pragma unroll
    for (int mi = 0; mi < MT; ++mi) {
      const int co = co0 + mi * 16 + sub * 4;
      if (co >= P.Cout) continue;
      float4 bias = make_float4(0.f, 0.f, 0.f, 0.f);
      if (a.bias) bias = make_float4(a.bias[co], a.bias[co + 1], a.bias[co + 2], a.bias[co + 3]);
#pragma unroll
      for (int rr = 0; rr < RW; ++rr) {
        const int y = y0 + rr;
        if (y >= H) continue;
#pragma unroll
        for (int ni = 0; ni < NTL; ++ni) {
          const int x = tx0 + ni * 16 + n16;
          if (x >= W) continue;
          float o[4] = {acc[rr][mi][ni][0] + bias.x, acc[rr][mi][ni][1] + bias.y, acc[rr][mi][ni][2] + bias.z,
                        acc[rr][mi][ni][3] + bias.w};
          if (a.relu) {
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = fmaxf(o[i], 0.f);
          }
          const long long off = (((long long)b * H + y) * W + x) * P.Cout + co;
          *reinterpret_cast<uint2*>(static_cast<uint16_t*>(a.out) + off) =
              make_uint2(f2bf2(o[0], o[1]), f2bf2(o[2], o[3]));
        }
      }
    }
  }
}

// Finish a convolution split over its channel chunks: S(pixel, co) = the
// ksplit partials added in split order, then the epilogue of k_conv3 for
// that value: bias, ReLU and a BF16 store, or (OUTF32) the route to A and the
// skip (see ConvRoute).  Four channels a thread.  An upsampled A takes
// its 2 x 2 block sums as (S00 + S01) + (S10 + S11) in a second index range
// over A's pixels.
__device__ __forceinline__ float4 ksum4(const ConvArgs& a, long long pix, int co) {
  const long long stride = (long long)a.B * a.in.H * a.in.W * a.pk.Coutp;
  float4 t = *reinterpret_cast<const float4*>(a.kpart + pix * a.pk.Coutp + co);
  for (int k = 1; k < a.ksplit; ++k) {
    const float4 q = *reinterpret_cast<const float4*>(a.kpart + k * stride + pix * a.pk.Coutp + co);
    t.x += q.x;
    t.y += q.y;
    t.z += q.z;
    t.w += q.w;
  }
  return t;
}

template <bool OUTF32>
__global__ __launch_bounds__(256) void k_conv_finish(ConvArgs a) {
  const int H = a.in.H, W = a.in.W;
  const long long npix = (long long)a.B * H * W;
  const ConvRoute& R = a.rt;
  const bool up = OUTF32 && R.modeA == 1;
  // range 1: every output pixel's channel groups (without the A channels of
  // an upsampled route); range 2: the A pixels of an upsampled route
  const int c_lo = up ? R.Ca : 0, ng1 = (a.pk.Cout - c_lo) >> 2;
  const long long n1 = npix * ng1;
  const long long n2 = up ? npix / 4 * (R.Ca >> 2) : 0;
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n1 + n2; i += (long long)gridDim.x * 256) {
    if (i < n1) {
      const long long pix = i / ng1;
      const int co = c_lo + 4 * (int)(i - pix * ng1);
      const float4 t = ksum4(a, pix, co);
      if constexpr (!OUTF32) {
        float o[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if (a.bias) o[k] += a.bias[co + k];
          if (a.relu) o[k] = fmaxf(o[k], 0.f);
        }
        *reinterpret_cast<uint2*>(static_cast<uint16_t*>(a.out) + pix * a.pk.Cout + co) =
            make_uint2(f2bf2(o[0], o[1]), f2bf2(o[2], o[3]));
      } else if (co >= R.Ca) {
        const long long ob = pix * R.Cb + (co - R.Ca);
        put4(R.gB + ob, R.mB ? R.mB + ob : nullptr, t.x, t.y, t.z, t.w, R.accB != 0);
      } else if (R.modeA == 0) {
        const long long oa = pix * R.Ca + co;
        put4(R.gA + oa, R.mA ? R.mA + oa : nullptr, t.x, t.y, t.z, t.w, R.accA != 0);
      } else {
        const long long b = pix / ((long long)H * W);
        const int rem = (int)(pix - b * H * W), y = rem / W, x = rem - y * W;
        const int H2 = 2 * H, W2 = 2 * W;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const long long oa = ((b * H2 + 2 * y + (q >> 1)) * W2 + 2 * x + (q & 1)) * R.Ca + co;
          put4(R.gA + oa, R.mA ? R.mA + oa : nullptr, 0.25f * t.x, 0.25f * t.y, 0.25f * t.z, 0.25f * t.w,
               R.accA != 0);
        }
      }
    } else {
      const long long j = i - n1;
      const int ngA = R.Ca >> 2;
      const long long ph = j / ngA;  // A pixel (b, yh, xh)
      const int co = 4 * (int)(j - ph * ngA);
      const int Hh = H >> 1, Wh = W >> 1;
      const long long b = ph / ((long long)Hh * Wh);
      const int rem = (int)(ph - b * Hh * Wh), yh = rem / Wh, xh = rem - yh * Wh;
      const long long p00 = (b * H + 2 * yh) * W + 2 * xh;
      const float4 s00 = ksum4(a, p00, co), s01 = ksum4(a, p00 + 1, co);
      const float4 s10 = ksum4(a, p00 + W, co), s11 = ksum4(a, p00 + W + 1, co);
      put4(R.gA + ph * R.Ca + co, R.mA ? R.mA + ph * R.Ca + co : nullptr, (s00.x + s01.x) + (s10.x + s11.x),
           (s00.y + s01.y) + (s10.y + s11.y), (s00.z + s01.z) + (s10.z + s11.z), (s00.w + s01.w) + (s10.w + s11.w),
           R.accA != 0);
    }
  }
}

// ------------------------------------------------------------ weight gradient
// One launch for all layers of an output-channel tile COT (16, 32 or 64): a
// workgroup takes an input-channel chunk, an output-channel tile and every
// nsplit-th pixel tile of one layer.  Layer by layer, the small ones needed
// hundreds of pixel splits to fill the card, and their partials, 342 MB at 4 x
// 1024 x 256 pixels, base 16, cost as much as the products.
// The 9 taps x NI input tiles go to the waves in turn (unit u to wave u mod 4).
// Both operands are staged in LDS pixel-major with channels contiguous (one
// 16-byte store per 8 channels of a pixel, the tap shift being an address
// offset) and read as MFMA fragments with the gfx950 LDS transpose read: for
// each group of 16 lanes, lane 4 r + q loads four consecutive channels 4 q +
// [0, 4) of pixel r, and lane c receives channel c of pixels 0..3.  k-group s
// of a row takes its pixels 4 s + [0, 4) and 16 + 4 s + [0, 4) (any bijection
// does, the same for both operands): 32 lanes then read eight consecutive
// pixels, which strides of an odd number of 32-byte units keep on different
// banks.  All layers 303 us and the reduction 42 (485 and 96 layer by layer).
typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef short v8i16 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) v4i16 lds_v4i16;

// The 8 pixels p and p + step of this lane's k-group.
__device__ __forceinline__ bf16x8 tr_frag(const uint16_t* p, int step) {
  const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)((__attribute__((address_space(3))) uint16_t*)p));
  const v4i16 hi =
      __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)((__attribute__((address_space(3))) uint16_t*)(p + step)));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// LDS pixel stride of C channels in BF16 values: an odd number of 32-byte units.
constexpr int wg_ps(int C) { return C % 32 == 0 ? C + 16 : C; }

template <bool AF32, int MODE, int COT, int NI>
__device__ __forceinline__ void wgrad_item(const WgradArgs& a, int cc, int co0, int split, uint16_t* lds) {
  constexpr int MT = COT / 16;
  constexpr int NG = COT / 8;            // 8-channel groups of the output gradient
  constexpr int ZP = wg_ps(COT);
  constexpr int XW = kWgTW + 2, XR = kWgTH + 2;
  constexpr int XP = wg_ps(16 * NI);
  constexpr int UNITS = 9 * NI, US = (UNITS + 3) / 4;
  uint16_t* const sZ = lds;
  uint16_t* const sX = lds + kWgTH * kWgTW * ZP;
  const int H = a.in.H, W = a.in.W;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
  const int sub = lane >> 4, n16 = lane & 15;
  const int tiles_x = (W + kWgTW - 1) / kWgTW, tiles_y = (H + kWgTH - 1) / kWgTH;
  const int T = a.B * tiles_x * tiles_y;
  // this lane's transpose-read offsets: pixel n16 / 4 of its k-group, channel quad n16 % 4
  const int kp = 4 * sub + (n16 >> 2), cq = 4 * (n16 & 3);

  f32x4 acc[US][MT];
#pragma unroll
  for (int s = 0; s < US; ++s)
#pragma unroll
    for (int mi = 0; mi < MT; ++mi) acc[s][mi] = f32x4{0.f, 0.f, 0.f, 0.f};
  // bias partial: thread t always stages channel group t % NG
  float bsum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  // the next tile's loads are issued before this tile's multiplies
  TileStage<true, 0, NG, kWgTH, kWgTW, ZP> sz;   // output gradient (of the pre-activation), [pixel][co]
  TileStage<AF32, MODE, 2 * NI, XR, XW, XP> sx;  // input tile with a one-pixel halo, [pixel][ci]
  ConvIn gz{};
  gz.A = a.gY;
  gz.Ca = a.Cout;
  gz.H = H;
  gz.W = W;
  auto fetch = [&](int t) {
    const int b = t / (tiles_x * tiles_y);
    const int rem = t - b * tiles_x * tiles_y;
    const int ty0 = (rem / tiles_x) * kWgTH, tx0 = (rem % tiles_x) * kWgTW;
    sz.init(gz, b, ty0, tx0);
    sz.fetch(gz, co0);
    sx.init(a.in, b, ty0 - 1, tx0 - 1);
    sx.fetch(a.in, cc * a.CCw);
  };
  fetch(split);  // split < T: the host takes at most T splits
  for (int t = split; t < T; t += a.nsplit) {
#pragma unroll
    for (int u = 0; u < sz.S; ++u) {
      bsum[0] += sz.f0[u].x;
      bsum[1] += sz.f0[u].y;
      bsum[2] += sz.f0[u].z;
      bsum[3] += sz.f0[u].w;
      bsum[4] += sz.f1[u].x;
      bsum[5] += sz.f1[u].y;
      bsum[6] += sz.f1[u].z;
      bsum[7] += sz.f1[u].w;
    }
    sz.store(sZ);
    sx.store(sX);
    __syncthreads();
    if (t + a.nsplit < T) fetch(t + a.nsplit);
    for (int row = 0; row < kWgTH; ++row) {
      bf16x8 af[MT];
#pragma unroll
      for (int mi = 0; mi < MT; ++mi) af[mi] = tr_frag(sZ + (row * kWgTW + kp) * ZP + mi * 16 + cq, 16 * ZP);
#pragma unroll
      for (int s = 0; s < US; ++s) {
        const int u = wave + 4 * s;
        if (4 * s + 3 >= UNITS && u >= UNITS) continue;
        const int kk = u / NI, ni = u - kk * NI, dy = kk / 3, dx = kk - dy * 3;
        const bf16x8 bf = tr_frag(sX + ((row + dy) * XW + kp + dx) * XP + ni * 16 + cq, 16 * XP);
#pragma unroll
        for (int mi = 0; mi < MT; ++mi) acc[s][mi] = mfma(af[mi], bf, acc[s][mi]);
      }
    }
    __syncthreads();
  }

#pragma unroll
  for (int s = 0; s < US; ++s) {
    const int u = wave + 4 * s;
    if (u >= UNITS) continue;
    const int kk = u / NI, ci = cc * a.CCw + (u - kk * NI) * 16 + n16;
#pragma unroll
    for (int mi = 0; mi < MT; ++mi)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int co = co0 + mi * 16 + sub * 4 + i;
        if (co < a.Cout && ci < a.Cipw)
          a.part[(((long long)split * a.Cout + co) * 9 + kk) * a.Cipw + ci] = acc[s][mi][i];
      }
  }
  // bias partial of this split (channel chunk 0 only): the threads of one
  // channel group are added in thread order
  if (cc == 0) {
    float* red = reinterpret_cast<float*>(lds);  // the loop ended with a barrier
#pragma unroll
    for (int i = 0; i < 8; ++i) red[threadIdx.x * 8 + i] = bsum[i];
    __syncthreads();
    const int c = (int)threadIdx.x;
    if (c < COT && co0 + c < a.Cout) {
      float sum = 0.f;
      for (int k = c >> 3; k < 256; k += NG) sum += red[k * 8 + (c & 7)];
      a.bpart[(long long)split * a.Cout + co0 + c] = sum;
    }
  }
}

template <int COT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_wgrad(WgradAll A) {
  constexpr int SZ = kWgTH * kWgTW * wg_ps(COT) + (kWgTH + 2) * (kWgTW + 2) * wg_ps(32);
  static_assert(SZ * 2 >= 256 * 8 * 4, "the bias partials reuse the tiles");
  __shared__ __attribute__((aligned(16))) uint16_t lds[SZ];
  int l = 0;
  while ((int)blockIdx.x >= A.wg[l + 1]) ++l;
  const WgradArgs& a = A.L[l];
  int i = (int)blockIdx.x - A.wg[l];
  const int split = i % a.nsplit;
  i /= a.nsplit;
  const int cc = i % a.nccw, co0 = (i / a.nccw) * COT;
  // the last chunk of a padded count with at most 16 real channels stages and multiplies only those
  const bool half = a.Cin - cc * a.CCw <= 16;
  if (a.af32) {  // the network's single-channel input
    wgrad_item<true, 0, COT, 1>(a, cc, co0, split, lds);
  } else if (a.in.modeA == 0) {
    if (half) wgrad_item<false, 0, COT, 1>(a, cc, co0, split, lds);
    else wgrad_item<false, 0, COT, 2>(a, cc, co0, split, lds);
  } else if (a.in.modeA == 1) {
    if (half) wgrad_item<false, 1, COT, 1>(a, cc, co0, split, lds);
    else wgrad_item<false, 1, COT, 2>(a, cc, co0, split, lds);
  } else {
    if (half) wgrad_item<false, 2, COT, 1>(a, cc, co0, split, lds);
    else wgrad_item<false, 2, COT, 2>(a, cc, co0, split, lds);
  }
}

// Sum the pixel-split partials of every layer (see RedAll) into the
// canonical weight gradients [Cout][Cin][3][3] and the bias gradients.  A
// workgroup takes E consecutive elements of one layer (E = 64: each wave
// load is 64 consecutive floats; E = 16 for layers with many splits, so that
// no thread walks a long chain of them) and 256 / E thread groups over the
// splits (split sp -> group sp mod G); the G partial sums of an element are
// added in group order, so the result does not depend on timing.
__global__ __launch_bounds__(256) void k_wgrad_reduce(RedAll a) {
  __shared__ float s[16 * 17 > 4 * 65 ? 16 * 17 : 4 * 65];
  const int b = (int)blockIdx.x;
  int l = 0;
  while (b >= a.wg[l + 1]) ++l;
  const RedLayer& L = a.L[l];
  const int E = L.e, G = 256 / E;
  const int te = (int)threadIdx.x % E, g = (int)threadIdx.x / E;
  const int nw = L.Cout * L.Cin * 9, n = nw + L.Cout;
  const int jl = (b - a.wg[l]) * E + te;
  float acc = 0.f;
  int co = 0, kk = 0, ci = 0;
  if (jl < nw) {
    // neighbouring elements are neighbouring ci: coalesced partial reads
    co = jl / (9 * L.Cin);
    const int r = jl - co * 9 * L.Cin;
    kk = r / L.Cin;
    ci = r - kk * L.Cin;
    const long long stride = (long long)L.Cout * 9 * L.Cipw;
    const float* p = L.part + ((long long)co * 9 + kk) * L.Cipw + ci;
#pragma unroll 8
    for (int sp = g; sp < L.nsplit; sp += G) acc += p[sp * stride];
  } else if (jl < n) {
#pragma unroll 8
    for (int sp = g; sp < L.nsplit; sp += G) acc += L.bpart[(long long)sp * L.Cout + (jl - nw)];
  }
  s[g * (E + 1) + te] = acc;
  __syncthreads();
  if (g == 0 && jl < n) {
    float t = 0.f;
    for (int q = 0; q < G; ++q) t += s[q * (E + 1) + te];
    if (jl < nw) L.grad[((long long)co * L.Cin + ci) * 9 + kk] = t;
    else L.gb[jl - nw] = t;
  }
}

// out[seg ne + e] = sum over the rows k of segment seg (rows seg R ..
// min(seg R + R, nblk) - 1) of part[k ne + e]: 64 consecutive elements per
// workgroup (one per lane: each wave load is 64 consecutive floats) and
// the four waves over the segment's rows (row k -> wave (k - seg R) mod 4),
// the waves' sums added in wave order (deterministic).
__global__ __launch_bounds__(256) void k_sum_rows(const float* __restrict__ part, int nblk, int ne, int R,
                                                 float* __restrict__ out) {
  __shared__ float s[4][65];
  const int te = (int)threadIdx.x & 63, g = (int)threadIdx.x >> 6;
  const int seg = (int)blockIdx.y, e = (int)blockIdx.x * 64 + te;
  const int k0 = seg * R, k1 = min(k0 + R, nblk);
  float acc = 0.f;
  if (e < ne)
    for (int k = k0 + g; k < k1; k += 4) acc += part[(long long)k * ne + e];
  s[g][te] = acc;
  __syncthreads();
  if (g == 0 && e < ne) out[(long long)seg * ne + e] = ((s[0][te] + s[1][te]) + s[2][te]) + s[3][te];
}

// out[e] = sum over k < nblk of part[k ne + e], in two fixed-order stages:
// segments of kSumRowsSeg rows into scratch (ceil(nblk / kSumRowsSeg) rows
// of ne), then those rows.
constexpr int kSumRowsSeg = 64;
static void sum_parts(const float* part, int nblk, int ne, float* scratch, float* out, hipStream_t s) {
  const unsigned gx = (unsigned)((ne + 63) / 64);
  const int nseg = (nblk + kSumRowsSeg - 1) / kSumRowsSeg;
  hipLaunchKernelGGL(k_sum_rows, dim3(gx, (unsigned)nseg), dim3(256), 0, s, part, nblk, ne, kSumRowsSeg, scratch);
  hipLaunchKernelGGL(k_sum_rows, dim3(gx, 1), dim3(256), 0, s, (const float*)scratch, nseg, ne, nseg, out);
}

// ------------------------------------------------------------ heads
constexpr int kHeadRowTiles = 5;  // 16-row tiles of the P + 1 <= 65 head-gradient rows

// Head weights are the same for every thread: read through the constant
// address space they come as scalar loads and operands (as LDS broadcasts their
// reads bound the kernel).
typedef const __attribute__((address_space(4))) float cfloat;
__device__ __forceinline__ cfloat* as_const(const float* p) { return (cfloat*)(unsigned long long)p; }

// One row of the model head: bias + w . h.
template <int C1>
__device__ __forceinline__ float head_row(cfloat* w, float bias, const float (&h)[C1]) {
  float s = bias;
#pragma unroll
  for (int c = 0; c < C1; ++c) s = fmaf(w[c], h[c], s);
  return s;
}

// The weight head: w [C1], then its bias.
template <int C1>
__device__ __forceinline__ float head_sigmoid(cfloat* w, const float (&h)[C1]) {
  return 1.0f / (1.0f + __expf(-head_row<C1>(w, w[C1], h)));
}

template <int C1>
__device__ __forceinline__ void head_input(const uint16_t* hp, float (&h)[C1]) {
#pragma unroll
  for (int c = 0; c < C1; c += 8) {
    float v[8];
    unpack8(*reinterpret_cast<const uint4*>(hp + c), v);
#pragma unroll
    for (int i = 0; i < 8; ++i) h[c + i] = v[i];
  }
}

// One pixel per thread: y_m = Wm h + bm (P channels, planar output), y_w =
// sigmoid(Ww h + bw), in FP32; C1 = 8, 16 or 32.  Bound by its output.
template <int C1>
__global__ __launch_bounds__(256) void k_head_fwd(HeadArgs a) {
  const int P = a.P;
  cfloat* const Wm = as_const(a.Wm);
  const long long HW = (long long)a.H * a.W, npix = a.B * HW;
  const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= npix) return;
  float h[C1];
  head_input<C1>(a.h + p * C1, h);
  const long long b = p / HW, yx = p - b * HW;
  float* ym = a.y_m + b * P * HW + yx;
#pragma unroll 2
  for (int co = 0; co < P; ++co) ym[co * HW] = head_row<C1>(Wm + co * C1, Wm[P * C1 + co], h);
  a.y_w[p] = head_sigmoid<C1>(as_const(a.Ww), h);
}

// The heads' outputs (as k_head_fwd has them; they stay in registers: written
// and read back they were 268 MB at 4 x 1024 x 256 pixels and 32 channels),
// loss terms, gradient of the head input's pre-activation (FP32 NHWC: the
// head input is a ReLU output) and per-block partial sums of the
// head-parameter gradient and of the two squared errors.
// One 256-pixel block per workgroup.  Dynamic LDS: gy [256][P+1] (column
// P: the gradient gz of the weight head's logit), h [256][C1+1] (column C1:
// 1); the waves' partials of the parameter gradient
// reuse it from the start once those are read.  Every head parameter's
// block gradient is one entry of sum_t gy[t] h[t]^T, a (P+1) x (C1+1)
// outer-product sum (Wm, bm; Ww, bw), computed on the FP32 matrix cores,
// each wave over a quarter of the block's pixels, and added over the waves
// in wave order.  110 us at that size (152 with the separate forward pass),
// about 65 of them vector instructions: the head both ways is 1024 FMAs a pixel.
template <int C1>
__global__ __launch_bounds__(256) void k_head_bwd(LossArgs a) {
  extern __shared__ __attribute__((aligned(16))) float sh[];
  __shared__ double sred[2][4];
  const HeadArgs& d = a.hd;
  const int P = d.P, tid = (int)threadIdx.x;
  const int GP = P + 1, HC = C1 + 1;
  float* sgy = sh;
  float* shh = sgy + 256 * GP;
  cfloat* const Wm = as_const(d.Wm);  // [P][C1], then bm [P]
  cfloat* const Ww = as_const(d.Ww);  // [C1], then bw
  const long long HW = (long long)d.H * d.W, npix = d.B * HW;
  const float inv_m = 1.0f / (float)((double)npix * P), inv_w = 1.0f / (float)npix;
  // parameter-gradient block sums on the FP32 matrix cores
  // (v_mfma_f32_16x16x4_f32: lane l supplies A[l % 16][l / 16] and
  // B[l / 16][l % 16] and receives D[4 (l / 16) + i][l % 16]):
  // D[r][c] = sum_t gy[t][r] h[t][c], r < P + 1, c < C1 + 1, in 16 x 16
  // tiles; wave w takes pixels 64 w .. 64 w + 63 (16 k-steps of 4)
  constexpr int TC = (C1 + 1 + 15) / 16;
  const int TR = (GP + 15) / 16;  // <= kHeadRowTiles: checked by the launcher
  const int wave = tid >> 6, lane = tid & 63, kq = lane >> 4, l16 = lane & 15;
  f32x4 acc[kHeadRowTiles][TC];
#pragma unroll
  for (int i = 0; i < kHeadRowTiles; ++i)
#pragma unroll
    for (int j = 0; j < TC; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  double lm = 0.0, lw = 0.0;
  const long long p = (long long)blockIdx.x * 256 + tid;
  if (p < npix) {
    float h[C1];
    head_input<C1>(d.h + p * C1, h);
    const float yw = head_sigmoid<C1>(Ww, h), dw = yw - a.t_w[p];
    lw = (double)dw * (double)dw;
    const float gz = 2.0f * a.lam_w * dw * inv_w * yw * (1.0f - yw);
    sgy[tid * GP + P] = gz;
    // g_h[c] = Ww[c] gz + sum over co of Wm[co][c] gy[co], co ascending
    float s[C1];
#pragma unroll
    for (int c = 0; c < C1; ++c) s[c] = Ww[c] * gz;
    const long long b = p / HW, yx = p - b * HW;
    const float* tm = a.t_m + b * P * HW + yx;
    constexpr int UT = 16;  // targets in flight
    for (int c0 = 0; c0 < P; c0 += UT) {
      float t[UT];
#pragma unroll
      for (int k = 0; k < UT; ++k) t[k] = c0 + k < P ? tm[(c0 + k) * HW] : 0.f;
#pragma unroll
      for (int k = 0; k < UT; ++k) {
        if (c0 + k >= P) continue;
        cfloat* const w = Wm + (c0 + k) * C1;
        const float df = head_row<C1>(w, Wm[P * C1 + c0 + k], h) - t[k];
        lm += (double)df * (double)df;
        const float gy = 2.0f * df * inv_m;
        sgy[tid * GP + c0 + k] = gy;
#pragma unroll
        for (int c = 0; c < C1; ++c) s[c] = fmaf(w[c], gy, s[c]);
      }
    }
    // the head input is a ReLU output: store the gradient of its pre-activation
#pragma unroll
    for (int c = 0; c < C1; ++c) {
      if (!(h[c] > 0.f)) s[c] = 0.f;
      shh[tid * HC + c] = h[c];
    }
    shh[tid * HC + C1] = 1.f;
#pragma unroll
    for (int c = 0; c < C1; c += 4)
      *reinterpret_cast<float4*>(a.g_h + p * C1 + c) = make_float4(s[c], s[c + 1], s[c + 2], s[c + 3]);
  } else {
    for (int co = 0; co < GP; ++co) sgy[tid * GP + co] = 0.f;
    for (int c = 0; c < HC; ++c) shh[tid * HC + c] = 0.f;
  }
  __syncthreads();
  for (int ks = 0; ks < 16; ++ks) {
    const int t = 64 * wave + 4 * ks + kq;
    float hb[TC];
#pragma unroll
    for (int ct = 0; ct < TC; ++ct) hb[ct] = 16 * ct + l16 < HC ? shh[t * HC + 16 * ct + l16] : 0.f;
#pragma unroll
    for (int rt = 0; rt < kHeadRowTiles; ++rt) {
      if (rt >= TR) continue;
      const float ga = 16 * rt + l16 < GP ? sgy[t * GP + 16 * rt + l16] : 0.f;
#pragma unroll
      for (int ct = 0; ct < TC; ++ct) acc[rt][ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(ga, hb[ct], acc[rt][ct], 0, 0, 0);
    }
  }
  __syncthreads();  // gy and h are read: their space takes the wave partials
  float* red = sh;   // [wave][TR][TC][16 x 16]
#pragma unroll
  for (int rt = 0; rt < kHeadRowTiles; ++rt) {
    if (rt >= TR) continue;
#pragma unroll
    for (int ct = 0; ct < TC; ++ct)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        red[((wave * TR + rt) * TC + ct) * 256 + (4 * kq + i) * 16 + l16] = acc[rt][ct][i];
  }
  __syncthreads();
  // entry e of the partial layout [Wm P x C1][bm P][Ww C1][bw] -> (r, c),
  // the four waves' sums added in wave order
  for (int e = tid; e < a.ne; e += 256) {
    int r, c;
    if (e < P * C1) {
      r = e / C1;
      c = e - r * C1;
    } else if (e < P * C1 + P) {
      r = e - P * C1;
      c = C1;
    } else {
      r = P;
      c = e - P * C1 - P;  // C1 for bw
    }
    const int o = ((r >> 4) * TC + (c >> 4)) * 256 + (r & 15) * 16 + (c & 15);
    float sum = 0.f;
    for (int w = 0; w < 4; ++w) sum += red[w * TR * TC * 256 + o];
    a.hpart[(long long)blockIdx.x * a.ne + e] = sum;
  }
  // block sums of the squared errors (fixed order)
  for (int off = 32; off > 0; off >>= 1) {
    lm += __shfl_down(lm, off);
    lw += __shfl_down(lw, off);
  }
  if ((tid & 63) == 0) {
    sred[0][tid >> 6] = lm;
    sred[1][tid >> 6] = lw;
  }
  __syncthreads();
  if (tid == 0) {
    a.lpart[2 * blockIdx.x] = sred[0][0] + sred[0][1] + sred[0][2] + sred[0][3];
    a.lpart[2 * blockIdx.x + 1] = sred[1][0] + sred[1][1] + sred[1][2] + sred[1][3];
  }
}

// loss = sum_m / Nm + lam_w sum_w / Nw over the block partials (one block).
__global__ __launch_bounds__(256) void k_loss_reduce(const double* __restrict__ lpart, int nblk, double Nm,
                                                    double Nw, double lam_w, double* loss) {
  __shared__ double s[2][256];
  double a = 0.0, b = 0.0;
  for (int k = threadIdx.x; k < nblk; k += 256) {
    a += lpart[2 * k];
    b += lpart[2 * k + 1];
  }
  s[0][threadIdx.x] = a;
  s[1][threadIdx.x] = b;
  __syncthreads();
  if (threadIdx.x == 0) {
    double ta = 0.0, tb = 0.0;
    for (int k = 0; k < 256; ++k) {
      ta += s[0][k];
      tb += s[1][k];
    }
    *loss = ta / Nm + lam_w * tb / Nw;
  }
}

// ------------------------------------------------------------ parameters
__global__ __launch_bounds__(256) void k_pack(PackAll a) {
  for (int e = (int)(blockIdx.x * blockDim.x + threadIdx.x); e < a.start[a.n]; e += (int)(gridDim.x * blockDim.x)) {
    int l = 0;
    while (e >= a.start[l + 1]) ++l;
    const PackArgs& L = a.L[l];
    const int nf = L.f.Coutp * L.f.ncc * L.f.KKp * L.f.CC;
    const bool fw = e - a.start[l] < nf;
    const ConvPack& P = fw ? L.f : L.t;
    const int i = fw ? e - a.start[l] : e - a.start[l] - nf;
    int r = i;
    const int c = r % P.CC;
    r /= P.CC;
    const int kk = r % P.KKp;
    r /= P.KKp;
    const int cc = r % P.ncc;
    const int co = r / P.ncc;
    const int ci = cc * P.CC + c;
    float v = 0.f;
    if (co < P.Cout && ci < P.Cin && kk < 9) {
      // forward: W[co][ci][kk]; transposed: output = forward input channel
      // co, input = forward output channel ci, taps flipped
      v = fw ? L.W[((long long)co * P.Cin + ci) * 9 + kk] : L.W[((long long)ci * P.Cout + co) * 9 + (8 - kk)];
    }
    (fw ? L.Wp : L.Wtp)[i] = (uint16_t)f2bf2(v, 0.f);
  }
}

__global__ __launch_bounds__(256) void k_adamw(float* __restrict__ th, const float* __restrict__ g,
                                              float* __restrict__ m, float* __restrict__ v, long long n, float lr,
                                              float b1, float b2, float eps, float wd, float bc1, float bc2) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float mh = mi / bc1, vh = vi / bc2;
    th[i] = th[i] * (1.f - lr * wd) - lr * mh / (sqrtf(vh) + eps);
  }
}


// ------------------------------------------------------------ launchers
static inline unsigned grid_for(long long n, int per = 256, int cap = 8192) {
  long long g = (n + per - 1) / per;
  return (unsigned)(g < 1 ? 1 : (g > cap ? cap : g));
}

// Workgroups below which a convolution launch splits its channel chunks
// (such launches leave CUs idle while each workgroup walks every chunk).
constexpr long long kConvSplitGroups = 512;

// Channel-chunk split of a launch (1: none), by the workgroups of 4 rows x 32
// columns x 64 channels (64 x 16 for at most 16 channels) that it has without.
// The split decides the order in which an output's products are added, so it
// goes by the sizes alone and not by the tile that is launched.  The host sizes
// the partial buffer with this same function.
int conv_ksplit(const ConvPack& pk, int B, int H, int W, bool up) {
  const bool narrow = !up && pk.Coutp <= 16;
  const long long groups = (long long)((H + 3) / 4) * ((W + (narrow ? 63 : 31)) / (narrow ? 64 : 32)) *
                           ((pk.Coutp + 63) / 64) * B;
  if (groups >= kConvSplitGroups) return 1;
  return (int)std::min<long long>(pk.ncc, (kConvSplitGroups + groups - 1) / groups);
}

// MFMA tile of a launch: waves of 2 rows by 32 columns by 32 output channels
// (64 columns where 16 channels are all).  Each weight fragment that comes
// through the L1 then serves four products; one row halves that, and 64
// channels cost the registers of a third wave per SIMD.  All convolutions of a
// gradient step at 4 x 1024 x 256 pixels, base 16: 860 us, one row 1010, 64
// channels 920; the 32 x 16-channel tiles 54 us with 64 columns, 56 with 32.
template <bool AF32, bool OUTF32, int MODE, int CC, bool UP>
static hipError_t conv3_pick(const ConvArgs& a, hipStream_t s) {
  constexpr int RW = 2;
  auto go = [&](auto mt) {
    constexpr int MT = decltype(mt)::value, NTL = MT == 1 && !UP ? 4 : 2;
    const int tiles = ((a.in.H + 4 * RW - 1) / (4 * RW)) * ((a.in.W + 16 * NTL - 1) / (16 * NTL));
    const dim3 grid(tiles, a.pk.Coutp / (16 * MT), a.B * a.ksplit);
    hipLaunchKernelGGL((k_conv3<AF32, OUTF32, MODE, CC, MT, NTL, RW, UP>), grid, dim3(256), 0, s, a);
    return hipGetLastError();
  };
  const int m16 = a.pk.Coutp / 16;
  if (m16 % 2 == 0) return go(std::integral_constant<int, 2>{});
  if (m16 % 3 == 0) return go(std::integral_constant<int, 3>{});
  return go(std::integral_constant<int, 1>{});
}

hipError_t launch_conv3(const ConvArgs& args, bool af32, bool outf32, hipStream_t s) {
  ConvArgs a = args;
  a.ksplit = std::max(1, a.ksplit);  // the kernel divides by it
  const bool up = outf32 && a.rt.gA && a.rt.modeA == 1;
  // FP32 outputs are input gradients: FP32 input, routed; an FP32 forward
  // input is the network's single channel
  if (outf32 && (!af32 || !a.rt.gA)) return hipErrorInvalidValue;
  if (af32 && !outf32 && a.pk.CC != 8) return hipErrorInvalidValue;
  if (a.ksplit > 1 && (!a.kpart || a.ksplit > a.pk.ncc)) return hipErrorInvalidValue;
  const bool unsplit_up = up && a.ksplit == 1;
  const int mode = a.in.modeA;
  hipError_t e = hipErrorInvalidValue;
#define UNET_CONV_CC(C)                                                                   \
  if (a.pk.CC == C) {                                                                     \
    if (unsplit_up) e = conv3_pick<true, true, 0, C, true>(a, s);                         \
    else if (outf32) e = conv3_pick<true, true, 0, C, false>(a, s);                       \
    else if (!af32 && mode == 0) e = conv3_pick<false, false, 0, C, false>(a, s);         \
    else if (!af32 && mode == 2) e = conv3_pick<false, false, 2, C, false>(a, s);         \
  }
  UNET_CONV_CC(8)
  UNET_CONV_CC(16)
  UNET_CONV_CC(32)
#undef UNET_CONV_CC
  // an upsampled A comes with its skip, at least 24 channels together
  if (!af32 && mode == 1 && a.pk.CC == 32) e = conv3_pick<false, false, 1, 32, false>(a, s);
  if (af32 && !outf32) e = conv3_pick<true, false, 0, 8, false>(a, s);
  if (e != hipSuccess) return e;
  if (a.ksplit > 1) {
    const long long npix = (long long)a.B * a.in.H * a.in.W;
    const long long n = npix * (a.pk.Cout >> 2);  // an upper bound of both index ranges
    if (outf32) hipLaunchKernelGGL(k_conv_finish<true>, dim3(grid_for(n)), dim3(256), 0, s, a);
    else hipLaunchKernelGGL(k_conv_finish<false>, dim3(grid_for(n)), dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

// output-channel tile of the weight gradient: 16, 32 or 64 (no idle tiles
// for 16- and 32-channel layers)
int wgrad_cot(int Cout) { return Cout <= 16 ? 16 : (Cout <= 32 ? 32 : 64); }

// The layers of one output-channel tile (wgrad_cot of each is cot).
hipError_t launch_wgrad(const WgradAll& a, int cot, hipStream_t s) {
  if (a.n < 1) return hipSuccess;
  for (int l = 0; l < a.n; ++l)
    if (a.L[l].af32 && a.L[l].Cin > 16) return hipErrorInvalidValue;
  const dim3 grid((unsigned)a.wg[a.n]);
  if (cot == 16) hipLaunchKernelGGL(k_wgrad<16>, grid, dim3(256), 0, s, a);
  else if (cot == 32) hipLaunchKernelGGL(k_wgrad<32>, grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL(k_wgrad<64>, grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_wgrad_reduce(const RedAll& a, hipStream_t s) {
  if (a.wg[a.n] < 1) return hipSuccess;
  hipLaunchKernelGGL(k_wgrad_reduce, dim3((unsigned)a.wg[a.n]), dim3(256), 0, s, a);
  return hipGetLastError();
}

size_t head_bwd_lds(int P, int C1) {
  // the four waves' 16 x 16 tiles of the (P + 1) x (C1 + 1) entries
  const size_t red = (size_t)4 * ((P + 16) / 16) * ((C1 + 16) / 16) * 256;
  return std::max((size_t)(256 * (P + 1) + 256 * (C1 + 1)), red) * 4;
}

hipError_t launch_head_fwd(const HeadArgs& a, hipStream_t s) {
  const long long npix = (long long)a.B * a.H * a.W;
  const dim3 grid((unsigned)((npix + 255) / 256));
  if (a.C1 == 8) hipLaunchKernelGGL(k_head_fwd<8>, grid, dim3(256), 0, s, a);
  else if (a.C1 == 16) hipLaunchKernelGGL(k_head_fwd<16>, grid, dim3(256), 0, s, a);
  else if (a.C1 == 32) hipLaunchKernelGGL(k_head_fwd<32>, grid, dim3(256), 0, s, a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_head_bwd(const LossArgs& a, int nblk, float* ghead, double* loss, double lam_w, hipStream_t s) {
  const long long npix = (long long)a.hd.B * a.hd.H * a.hd.W;
  if ((a.hd.P + 1 + 15) / 16 > kHeadRowTiles) return hipErrorInvalidValue;
  const size_t lds = head_bwd_lds(a.hd.P, a.hd.C1);
  if (a.hd.C1 == 8) hipLaunchKernelGGL(k_head_bwd<8>, dim3(nblk), dim3(256), lds, s, a);
  else if (a.hd.C1 == 16) hipLaunchKernelGGL(k_head_bwd<16>, dim3(nblk), dim3(256), lds, s, a);
  else if (a.hd.C1 == 32) hipLaunchKernelGGL(k_head_bwd<32>, dim3(nblk), dim3(256), lds, s, a);
  else return hipErrorInvalidValue;
  sum_parts((const float*)a.hpart, nblk, a.ne, a.hpart + (long long)nblk * a.ne, ghead, s);
  hipLaunchKernelGGL(k_loss_reduce, dim3(1), dim3(256), 0, s, (const double*)a.lpart, nblk,
                     (double)npix * a.hd.P, (double)npix, lam_w, loss);
  return hipGetLastError();
}

hipError_t launch_pack(const PackAll& a, hipStream_t s) {
  hipLaunchKernelGGL(k_pack, dim3(grid_for(a.start[a.n])), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_adamw(float* th, const float* g, float* m, float* v, long long n, float lr, float b1, float b2,
                        float eps, float wd, float bc1, float bc2, hipStream_t s) {
  hipLaunchKernelGGL(k_adamw, dim3(grid_for(n)), dim3(256), 0, s, th, g, m, v, n, lr, b1, b2, eps, wd, bc1, bc2);
  return hipGetLastError();
}


hipError_t unet_kernels_init() {
  hipError_t e = hipSuccess;
  const void* fns[3] = {reinterpret_cast<const void*>(&k_head_bwd<8>), reinterpret_cast<const void*>(&k_head_bwd<16>),
                        reinterpret_cast<const void*>(&k_head_bwd<32>)};
  for (const void* f : fns) {
    e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 150 * 1024);
    if (e != hipSuccess) return e;
  }
  return e;
}

}  // namespace unet

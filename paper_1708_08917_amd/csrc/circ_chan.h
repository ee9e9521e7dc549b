// Transforms down the channel axis of NCHW images (CONV layers): rows of K channels, consecutive rows
// (pixels) adjacent in memory, consecutive elements of a row one image plane apart.
//
// Lanes run along the pixels, so the elements a thread needs for its sub-transform of the first pass
// (n = R2 n1 + n2, all n1) are R1 coalesced loads of its column, and the time samples it holds after the second pass
// of the inverse are coalesced stores: the forward transform starts in registers straight from memory and the
// inverse ends there.  Against a tile staged in LDS on both sides this saves a pass over LDS and
// a barrier in front of the first butterfly (and the table of row addresses with its own barrier), and all
// loads of a thread are in flight together: 21,632 rows of 96 (13x13 images) 10.8 -> 8.0 us forward, 11.6 ->
// 9.0 us inverse; 100,352 rows of 64 (28x28) 12.4 -> 11.2 us forward (52 MB: 4.7 TB/s, a large copy reaches 5.2).
//
// A column is two pixels (rows 2u, 2u + 1) packed into one complex sequence.  PAIR: the image has an even
// number of pixels, so that a column's two values are one aligned access.  first: workgroups of earlier launches of
// the same transform (a launch has fewer than 2^32 threads).
#pragma once

#include <hip/hip_runtime.h>

#include "circ_kernels.h"

namespace circ {

// inter-pass twiddles of one thread: W_K^(f1 n2), f1 = 1..R1-1, as (cos, sin)
template <int K>
__device__ __forceinline__ void chan_twiddles(float2 (&w)[radix1_of(K)], int n2) {
#pragma unroll
  for (int f1 = 1; f1 < radix1_of(K); ++f1) {
    if constexpr (kTwN % K == 0) w[f1] = reinterpret_cast<const float2*>(kTw.cs)[f1 * n2 * (kTwN / K)];
    else w[f1] = reinterpret_cast<const float2*>(kRoots<K>.cs)[f1 * n2];
  }
}

// First pass of thread (column, n2): R1-point transform, twiddles, exchange layout of fft_lds_pass2.
template <int K, bool INV>
__device__ __forceinline__ void chan_pass1(float (&re)[radix1_of(K)], float (&im)[radix1_of(K)], const float2 (&w)[radix1_of(K)],
                                           float2* z, int PP, int col, int n2) {
  constexpr int R1 = radix1_of(K), R2 = radix2_of(K);
  FftReg<R1, INV>::run(re, im);
#pragma unroll
  for (int f1 = 0; f1 < R1; ++f1) {
    float vr = re[f1], vi = im[f1];
    if (f1 > 0) {
      const float c = w[f1].x, s = INV ? w[f1].y : -w[f1].y;
      const float xr = c * vr - s * vi;
      vi = c * vi + s * vr;
      vr = xr;
    }
    z[(R2 * f1 + n2) * PP + col] = make_float2(vr, vi);
  }
}

// out[f*out_fstride + rid]: bins 0..K/2 of row rid.  P columns per workgroup (a power of two), P * R2 threads.
// HMODE: 0, or kHalfRows (with kHalfBf16): 16-bit images, the spectra stay fp32.
template <int K, int HMODE, bool PAIR>
__global__ __launch_bounds__(512) void rfft_chan_kernel(const void* __restrict__ in, float2* __restrict__ out, RowMap map,
                                                        long long nrows, long long out_fstride, int P, unsigned first) {
  constexpr int R1 = radix1_of(K), R2 = radix2_of(K);
  constexpr bool HALF = (HMODE & kHalfRows) != 0, BF = (HMODE & kHalfBf16) != 0;
  extern __shared__ __attribute__((aligned(16))) float2 chan_z[];
  const int PP = P + 1, lgP = __ffs(P) - 1, tid = threadIdx.x, col = tid & (P - 1), n2 = tid >> lgP;
  const long long t0 = (long long)(blockIdx.x + first) * 2 * P, rid = t0 + 2 * col;
  const long long e0 = row_base(map, min(rid, nrows - (PAIR ? 2 : 1))) + n2 * map.es;
  const long long e1 = PAIR ? e0 + 1 : row_base(map, min(rid + 1, nrows - 1)) + n2 * map.es;   // (rows past the end repeat the last one)
  const long long step = R2 * map.es;
  float re[R1], im[R1];
  if constexpr (HALF) {
    const unsigned short* xh = static_cast<const unsigned short*>(in);
    unsigned raw[R1];
#pragma unroll
    for (int n1 = 0; n1 < R1; ++n1) {
      if constexpr (PAIR) raw[n1] = *reinterpret_cast<const unsigned*>(xh + e0 + n1 * step);
      else raw[n1] = unsigned(xh[e0 + n1 * step]) | (unsigned(xh[e1 + n1 * step]) << 16);
    }
#pragma unroll
    for (int n1 = 0; n1 < R1; ++n1) {
      const float2 v = unpack_pair16<BF>(raw[n1]);
      re[n1] = v.x;
      im[n1] = v.y;
    }
  } else {
    const float* xf = static_cast<const float*>(in);
#pragma unroll
    for (int n1 = 0; n1 < R1; ++n1) {
      if constexpr (PAIR) {
        const float2 v = *reinterpret_cast<const float2*>(xf + e0 + n1 * step);
        re[n1] = v.x;
        im[n1] = v.y;
      } else {
        re[n1] = xf[e0 + n1 * step];
        im[n1] = xf[e1 + n1 * step];
      }
    }
  }
  float2 w[R1];
  chan_twiddles<K>(w, n2);
  chan_pass1<K, false>(re, im, w, chan_z, PP, col, n2);
  __syncthreads();
  // (as fft_lds_pass2_inplace, spelled out: with that function in common the compiler gives rfft_kernel more registers,
  // 116 instead of 94 at K = 192, which cost that kernel a wave per SIMD and a fourth of its speed)
  fft_lds_pass2<K, false>(chan_z, PP, col, n2, R2, [&](int f, float2 v) { chan_z[fft_pos<K>(f) * PP + col] = v; });
  __syncthreads();
  rfft_store_tile<K, 0>(chan_z, P, lgP, tid, blockDim.x, t0, nrows, out, out_fstride, 1.0f, 0);
}

// Inverse: rows from bins 0..K/2, + bias[rid / bias_div][n], ReLU.  SPAIR: even plane pitch and a 16-byte aligned
// spectrum (both bins of a column in one load).
template <int K, int HMODE, bool PAIR, bool SPAIR>
__global__ __launch_bounds__(512) void irfft_chan_kernel(const float2* __restrict__ in, void* __restrict__ out, RowMap map,
                                                         long long nrows, long long in_fstride, int P, const float* __restrict__ bias,
                                                         long long bias_div, int relu, unsigned first) {
  constexpr int R1 = radix1_of(K), R2 = radix2_of(K);
  constexpr bool HALF = (HMODE & kHalfRows) != 0, BF = (HMODE & kHalfBf16) != 0;
  extern __shared__ __attribute__((aligned(16))) float2 chan_z[];
  const int PP = P + 1, lgP = __ffs(P) - 1, tid = threadIdx.x, col = tid & (P - 1), n2 = tid >> lgP;
  const long long rid = (long long)(blockIdx.x + first) * 2 * P + 2 * col;
  const long long r0 = min(rid, nrows - 1), r1 = min(rid + 1, nrows - 1);
  // Z = Ya + i Yb on all K bins (Hermitian symmetry): bin f > K/2 comes from bin K - f
  float re[R1], im[R1];
  float4 y[R1];
#pragma unroll
  for (int n1 = 0; n1 < R1; ++n1) {
    const int f = R2 * n1 + n2;
    const long long o = (long long)(2 * f <= K ? f : K - f) * in_fstride;
    if constexpr (SPAIR) {
      y[n1] = *reinterpret_cast<const float4*>(in + o + min(rid, nrows - 2));
    } else {
      const float2 a = in[o + r0], b = in[o + r1];
      y[n1] = make_float4(a.x, a.y, b.x, b.y);
    }
  }
  float2 w[R1];
  chan_twiddles<K>(w, n2);
#pragma unroll
  for (int n1 = 0; n1 < R1; ++n1) {
    const int f = R2 * n1 + n2;
    if (f == 0 || 2 * f == K) {                    // DC and Nyquist bins of a real signal are real
      re[n1] = y[n1].x;
      im[n1] = y[n1].z;
    } else {
      const float s = 2 * f < K ? 1.f : -1.f;
      re[n1] = y[n1].x - s * y[n1].w;
      im[n1] = y[n1].z + s * y[n1].y;
    }
  }
  chan_pass1<K, true>(re, im, w, chan_z, PP, col, n2);
  __syncthreads();
  if (n2 >= R1 || rid >= nrows) return;
  const int f1 = n2;                               // this thread's samples: n = f1 + R1 f2
  const long long e0 = row_base(map, r0), e1 = PAIR ? e0 + 1 : row_base(map, r1);
  const float* b0 = bias ? bias + (long long)(unsigned(r0) / unsigned(bias_div)) * K : nullptr;
  const float* b1 = PAIR || !bias ? b0 : bias + (long long)(unsigned(r1) / unsigned(bias_div)) * K;
  const bool two = rid + 1 < nrows;
  fft_lds_pass2<K, true>(chan_z, PP, col, f1, R2, [&](int n, float2 v) {
    if (bias) {
      v.x += b0[n];
      v.y += b1[n];
    }
    if (relu) {
      v.x = fmaxf(v.x, 0.f);
      v.y = fmaxf(v.y, 0.f);
    }
    const long long o = n * map.es;
    if constexpr (HALF) {
      unsigned short* yh = static_cast<unsigned short*>(out);
      const unsigned h = pack_pair16<BF>(v.x, v.y);
      if constexpr (PAIR) {
        *reinterpret_cast<unsigned*>(yh + e0 + o) = h;
      } else {
        yh[e0 + o] = (unsigned short)(h & 0xffffu);
        if (two) yh[e1 + o] = (unsigned short)(h >> 16);
      }
    } else {
      float* yf = static_cast<float*>(out);
      if constexpr (PAIR) {
        *reinterpret_cast<float2*>(yf + e0 + o) = v;
      } else {
        yf[e0 + o] = v.x;
        if (two) yf[e1 + o] = v.y;
      }
    }
  });
}

}  // namespace circ

// In-register FFT of R points (any R) and the split K = R1 * R2 of the two-pass transforms: the
// arithmetic core of every transform in the library.
// Plain C++ apart from the __device__ / __forceinline__ markers: tests/test_fftreg_host.py compiles
// it for the CPU and checks every size the kernels use against the definition of the transform.
#pragma once

#include <cmath>

#include "circ_twiddle.h"

namespace circ {

constexpr int ilog2(int v) { return v <= 1 ? 0 : 1 + ilog2(v >> 1); }
constexpr bool is_pow2_c(int v) { return v > 0 && (v & (v - 1)) == 0; }
// K = R1 * R2 with R1 <= R2.  Powers of two: R2 <= 2 * R1; for odd log2 K the longer sub-transform
// is the second one: the first pass then has R2 = 2*R1 short sub-transforms (plus the twiddles) per
// column, which keep every thread of a 16-threads-per-column kernel busy, and the second pass R1
// long ones without twiddles (fused kernel, K = 128: 1.25 + 0.47 us per chunk with the longer one
// first, about 0.4 us less this way).  Other sizes: the factor pair closest to the square root
// (96 = 8 * 12, 100 = 10 * 10, 384 = 16 * 24).
constexpr int radix1_of(int K) {
  if (is_pow2_c(K)) return K / (1 << ((ilog2(K) + 1) / 2));
  int best = 1;
  for (int d = 2; d * d <= K; ++d)
    if (K % d == 0) best = d;
  return best;
}
constexpr int radix2_of(int K) { return K / radix1_of(K); }

constexpr int smallest_odd_factor(int R) {
  for (int d = 3; d * d <= R; d += 2)
    if (R % d == 0) return d;
  return R;
}

// ---- in-register FFT of R points, natural order in and out ---------------------------
// Even R: the radix-2 recursion of Sec. 4.1 (two transforms of R/2 points and one butterfly
// level).  Odd R = p * M, p its smallest prime factor: p transforms of M points over the
// subsequences x[p*n + s], then X[f + M*m] = sum_s (E_s[f] W_R^(s f)) W_p^(s m): the same
// recursion with p-point butterflies.  The p-point butterfly pairs s with p - s:
// with a_s = T_s + T_(p-s), b_s = T_s - T_(p-s), X_m and X_(p-m) are
// (T_0 + sum_s cos(2 pi s m / p) a_s) -/+ i (sum_s sin(2 pi s m / p) b_s)  (forward; inverse: +/-).
// All twiddles are compile-time constants.
template <int R, bool INV>
struct FftReg {
  template <int M>
  static __device__ __forceinline__ void combine(float (&re)[R], float (&im)[R],
                                                 const float (&er)[R / 2], const float (&ei)[R / 2],
                                                 const float (&pr)[R / 2], const float (&pi)[R / 2]) {
    if constexpr (M < R / 2) {
      float tr, ti;
      if constexpr (M == 0) {
        tr = pr[M];
        ti = pi[M];
      } else if constexpr (4 * M == R) {           // twiddle = -i (forward) or +i (inverse)
        tr = INV ? -pi[M] : pi[M];
        ti = INV ? pr[M] : -pr[M];
      } else {
        constexpr float c = tw_cos(M, R);
        constexpr float s = INV ? tw_sin(M, R) : -tw_sin(M, R);   // twiddle = c + i*s
        tr = c * pr[M] - s * pi[M];
        ti = c * pi[M] + s * pr[M];
      }
      re[M] = er[M] + tr;
      im[M] = ei[M] + ti;
      re[M + R / 2] = er[M] - tr;
      im[M + R / 2] = ei[M] - ti;
      combine<M + 1>(re, im, er, ei, pr, pi);
    }
  }

  // odd R: outputs f, f + M, ..., f + (p-1)*M from the p sub-transforms' values at f
  template <int P, int M, int F>
  static __device__ __forceinline__ void combine_odd(float (&re)[R], float (&im)[R], const float (&sr)[P][M],
                                                     const float (&si)[P][M]) {
    if constexpr (F < M) {
      float tr[P], ti[P];
      tr[0] = sr[0][F];
      ti[0] = si[0][F];
      odd_twiddle<P, M, F, 1>(tr, ti, sr, si);
      constexpr int H = (P - 1) / 2;
      float ar[H + 1], ai[H + 1], br[H + 1], bi[H + 1];
#pragma unroll
      for (int s = 1; s <= H; ++s) {
        ar[s] = tr[s] + tr[P - s];
        ai[s] = ti[s] + ti[P - s];
        br[s] = tr[s] - tr[P - s];
        bi[s] = ti[s] - ti[P - s];
      }
      float x0r = tr[0], x0i = ti[0];
#pragma unroll
      for (int s = 1; s <= H; ++s) {
        x0r += ar[s];
        x0i += ai[s];
      }
      re[F] = x0r;
      im[F] = x0i;
      odd_outputs<P, M, F, 1>(re, im, tr[0], ti[0], ar, ai, br, bi);
      combine_odd<P, M, F + 1>(re, im, sr, si);
    }
  }
  template <int P, int M, int F, int S>
  static __device__ __forceinline__ void odd_twiddle(float (&tr)[P], float (&ti)[P], const float (&sr)[P][M],
                                                     const float (&si)[P][M]) {
    if constexpr (S < P) {
      if constexpr (F == 0) {
        tr[S] = sr[S][F];
        ti[S] = si[S][F];
      } else {
        constexpr float c = tw_cos(S * F, R);
        constexpr float s = INV ? tw_sin(S * F, R) : -tw_sin(S * F, R);
        tr[S] = c * sr[S][F] - s * si[S][F];
        ti[S] = c * si[S][F] + s * sr[S][F];
      }
      odd_twiddle<P, M, F, S + 1>(tr, ti, sr, si);
    }
  }
  template <int P, int M, int F, int MM>
  static __device__ __forceinline__ void odd_outputs(float (&re)[R], float (&im)[R], float t0r, float t0i,
                                                     const float (&ar)[(P - 1) / 2 + 1], const float (&ai)[(P - 1) / 2 + 1],
                                                     const float (&br)[(P - 1) / 2 + 1], const float (&bi)[(P - 1) / 2 + 1]) {
    constexpr int H = (P - 1) / 2;
    if constexpr (MM <= H) {
      float cr = t0r, ci = t0i, qr = 0.f, qi = 0.f;
      odd_terms<P, MM, 1>(cr, ci, qr, qi, ar, ai, br, bi);
      // forward: X_m = C - i Q, X_(p-m) = C + i Q; inverse: the other way round
      if constexpr (INV) {
        re[F + M * MM] = cr - qi;
        im[F + M * MM] = ci + qr;
        re[F + M * (P - MM)] = cr + qi;
        im[F + M * (P - MM)] = ci - qr;
      } else {
        re[F + M * MM] = cr + qi;
        im[F + M * MM] = ci - qr;
        re[F + M * (P - MM)] = cr - qi;
        im[F + M * (P - MM)] = ci + qr;
      }
      odd_outputs<P, M, F, MM + 1>(re, im, t0r, t0i, ar, ai, br, bi);
    }
  }
  template <int P, int MM, int S>
  static __device__ __forceinline__ void odd_terms(float& cr, float& ci, float& qr, float& qi,
                                                   const float (&ar)[(P - 1) / 2 + 1], const float (&ai)[(P - 1) / 2 + 1],
                                                   const float (&br)[(P - 1) / 2 + 1], const float (&bi)[(P - 1) / 2 + 1]) {
    if constexpr (S <= (P - 1) / 2) {
      constexpr float c = tw_cos((S * MM) % P, P), s = tw_sin((S * MM) % P, P);
      cr = fmaf(c, ar[S], cr);
      ci = fmaf(c, ai[S], ci);
      qr = fmaf(s, br[S], qr);
      qi = fmaf(s, bi[S], qi);
      odd_terms<P, MM, S + 1>(cr, ci, qr, qi, ar, ai, br, bi);
    }
  }

  static __device__ __forceinline__ void run(float (&re)[R], float (&im)[R]) {
    if constexpr (R % 2 == 0) {
      float er[R / 2], ei[R / 2], pr[R / 2], pi[R / 2];
#pragma unroll
      for (int i = 0; i < R / 2; ++i) {
        er[i] = re[2 * i];
        ei[i] = im[2 * i];
        pr[i] = re[2 * i + 1];
        pi[i] = im[2 * i + 1];
      }
      FftReg<R / 2, INV>::run(er, ei);
      FftReg<R / 2, INV>::run(pr, pi);
      combine<0>(re, im, er, ei, pr, pi);
    } else {
      constexpr int P = smallest_odd_factor(R), M = R / P;
      float sr[P][M], si[P][M];
#pragma unroll
      for (int s = 0; s < P; ++s) {
#pragma unroll
        for (int n = 0; n < M; ++n) {
          sr[s][n] = re[P * n + s];
          si[s][n] = im[P * n + s];
        }
        FftReg<M, INV>::run(sr[s], si[s]);
      }
      combine_odd<P, M, 0>(re, im, sr, si);
    }
  }
};

template <bool INV>
struct FftReg<1, INV> {
  static __device__ __forceinline__ void run(float (&)[1], float (&)[1]) {}
};

// ---- in-register FFT of K real values, K = 2, 4, 8, 16, 32 -----------------------------------------
// Half spectrum as K floats: comp 0: bin 0, comp 1: bin K/2, comps 2f and 2f+1: re, im of bin f.
// Decimation in time by four: real transforms of the Q = K/4 long subsequences x[4n + m], twiddles W_K^(f m), and 4-point
// butterflies over m, of which bin f < Q/2 gives the bins f, f + Q, K/2 - f and Q - f (the last two as conjugates); the
// inverse is the same flow backwards.  At most two roundings by twiddles on the way of a value at K = 32 (W_8 and
// W_32), where a half-length complex transform and its separation into even and odd parts have three and one more
// butterfly level: root mean square error 6.3e-8 forward, 6.6e-8 inverse against 7.7e-8 and 7.8e-8 in that form and
// 6.9e-8 and 7.2e-8 of the two-pass transform of two packed rows (K = 32; fewer additions than either).
template <int K>
struct RealFft {
  static constexpr int H = K / 2, Q = K / 4;

  static __device__ __forceinline__ void forward(const float (&v)[K], float (&out)[K]) {
    if constexpr (K == 2) {
      out[0] = v[0] + v[1];
      out[1] = v[0] - v[1];
    } else if constexpr (K == 4) {
      const float a = v[0] + v[2], b = v[1] + v[3];
      out[0] = a + b;
      out[1] = a - b;
      out[2] = v[0] - v[2];
      out[3] = v[3] - v[1];
    } else {
      float s[4][Q], a[4][Q];
#pragma unroll
      for (int m = 0; m < 4; ++m) {
#pragma unroll
        for (int n = 0; n < Q; ++n) s[m][n] = v[4 * n + m];
        RealFft<Q>::forward(s[m], a[m]);
      }
      const float e = a[0][0] + a[2][0], o = a[1][0] + a[3][0];
      out[0] = e + o;
      out[1] = e - o;
      out[2 * Q] = a[0][0] - a[2][0];
      out[2 * Q + 1] = a[3][0] - a[1][0];
      // bin Q/2 of the subsequences is real, its twiddles eighth roots: bins Q/2 and Q/2 + Q
      constexpr float r = tw_cos(1, 8);
      const float x = r * (a[1][1] - a[3][1]), y = r * (a[1][1] + a[3][1]);
      out[Q] = a[0][1] + x;
      out[Q + 1] = -(a[2][1] + y);
      out[3 * Q] = a[0][1] - x;
      out[3 * Q + 1] = a[2][1] - y;
      bins<1>(a, out);
    }
  }

  // sum convention (no 1/K)
  static __device__ __forceinline__ void inverse(const float (&in)[K], float (&v)[K]) {
    if constexpr (K == 2) {
      v[0] = in[0] + in[1];
      v[1] = in[0] - in[1];
    } else if constexpr (K == 4) {
      const float a = in[0] + in[1], b = in[0] - in[1];
      v[0] = fmaf(2.f, in[2], a);
      v[2] = fmaf(-2.f, in[2], a);
      v[1] = fmaf(-2.f, in[3], b);
      v[3] = fmaf(2.f, in[3], b);
    } else {
      float s[4][Q], a[4][Q];
      const float e = in[0] + in[1], o = in[0] - in[1];
      a[0][0] = fmaf(2.f, in[2 * Q], e);
      a[2][0] = fmaf(-2.f, in[2 * Q], e);
      a[1][0] = fmaf(-2.f, in[2 * Q + 1], o);
      a[3][0] = fmaf(2.f, in[2 * Q + 1], o);
      constexpr float r2 = 2.f * tw_cos(1, 8);
      const float ar = in[Q], ai = in[Q + 1], br = in[3 * Q], bi = in[3 * Q + 1];
      a[0][1] = 2.f * (ar + br);
      a[1][1] = r2 * ((ar - ai) - (br + bi));
      a[2][1] = 2.f * (bi - ai);
      a[3][1] = r2 * ((br - bi) - (ar + ai));
      inverse_bins<1>(in, a);
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        RealFft<Q>::inverse(a[m], s[m]);
#pragma unroll
        for (int n = 0; n < Q; ++n) v[4 * n + m] = s[m][n];
      }
    }
  }

 private:
  template <int F>
  static __device__ __forceinline__ void bins(const float (&a)[4][Q], float (&out)[K]) {
    if constexpr (2 * F < Q) {
      float tr[4], ti[4];
      tr[0] = a[0][2 * F];
      ti[0] = a[0][2 * F + 1];
      twiddle<F, 1>(tr[1], ti[1], a[1]);
      twiddle<F, 2>(tr[2], ti[2], a[2]);
      twiddle<F, 3>(tr[3], ti[3], a[3]);
      const float sr = tr[0] + tr[2], si = ti[0] + ti[2], dr = tr[0] - tr[2], di = ti[0] - ti[2];
      const float ur = tr[1] + tr[3], ui = ti[1] + ti[3], vr = tr[1] - tr[3], vi = ti[1] - ti[3];
      out[2 * F] = sr + ur;
      out[2 * F + 1] = si + ui;
      out[2 * (F + Q)] = dr + vi;
      out[2 * (F + Q) + 1] = di - vr;
      out[2 * (H - F)] = sr - ur;
      out[2 * (H - F) + 1] = ui - si;
      out[2 * (Q - F)] = dr - vi;
      out[2 * (Q - F) + 1] = -(di + vr);
      bins<F + 1>(a, out);
    }
  }
  template <int F, int M>                              // W_K^(F M) times bin F
  static __device__ __forceinline__ void twiddle(float& tr, float& ti, const float (&a)[Q]) {
    constexpr float c = tw_cos(F * M, K), s = tw_sin(F * M, K);
    tr = c * a[2 * F] + s * a[2 * F + 1];
    ti = c * a[2 * F + 1] - s * a[2 * F];
  }
  template <int F>
  static __device__ __forceinline__ void inverse_bins(const float (&in)[K], float (&a)[4][Q]) {
    if constexpr (2 * F < Q) {
      const float y0r = in[2 * F], y0i = in[2 * F + 1], y1r = in[2 * (F + Q)], y1i = in[2 * (F + Q) + 1];
      const float y2r = in[2 * (H - F)], y2i = -in[2 * (H - F) + 1], y3r = in[2 * (Q - F)], y3i = -in[2 * (Q - F) + 1];
      const float sr = y0r + y2r, si = y0i + y2i, dr = y0r - y2r, di = y0i - y2i;
      const float ur = y1r + y3r, ui = y1i + y3i, vr = y1r - y3r, vi = y1i - y3i;
      a[0][2 * F] = sr + ur;
      a[0][2 * F + 1] = si + ui;
      inverse_twiddle<F, 1>(a[1], dr - vi, di + vr);
      inverse_twiddle<F, 2>(a[2], sr - ur, si - ui);
      inverse_twiddle<F, 3>(a[3], dr + vi, di - vr);
      inverse_bins<F + 1>(in, a);
    }
  }
  template <int F, int M>
  static __device__ __forceinline__ void inverse_twiddle(float (&a)[Q], float tr, float ti) {
    constexpr float c = tw_cos(F * M, K), s = tw_sin(F * M, K);
    a[2 * F] = c * tr - s * ti;
    a[2 * F + 1] = c * ti + s * tr;
  }
};

}  // namespace circ

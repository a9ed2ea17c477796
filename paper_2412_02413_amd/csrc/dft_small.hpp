// In-register DFTs of any length R up to 32 whose prime factors are at most 13, kernel
// e^{S 2 pi i n k / R} (S = +1 or -1), natural order in and out.  The lateral grids of 32 k
// columns need lengths 2 .. 32 (even) and 9 .. 15 beside the 8- and 16-point transforms that
// have codelets of their own.
//
// Composite lengths split as R = P Q (n = Q n1 + n2, k = k1 + P k2): P-point transforms over
// n1, twiddles e^{S 2 pi i n2 k1 / R}, Q-point transforms over n2, with P = 4 where 4 divides
// R, else 2, else the smallest prime factor.  An odd prime P pairs the inputs n and P - n: with
// s_n, d_n their sum and difference, X_k and X_{P-k} are A_k +- i S B_k, A_k = x_0 + sum cos s_n
// and B_k = sum sin d_n, real-by-complex products only: (P - 1)^2 FMAs and multiplies besides
// the additions, which at P = 13 (about 190 operations) is still close to the 144 of the
// 16-point codelet.  Every index is a compile-time constant, so all values stay in registers
// and the constants become literals.
#pragma once
#include <hip/hip_runtime.h>

namespace pam {

// cos and sin of 2 pi n / d, evaluated at compile time: reduced with exact integers to an eighth
// turn, then the Taylor series.
constexpr double kTau = 6.283185307179586476925286766559;
constexpr double taylor(double x, double term, int first) {   // sum of the alternating series from x^first / first!
  double sum = term;
  for (int k = first + 1; k < first + 24; k += 2) {
    term *= -x * x / (k * (k + 1));
    sum += term;
  }
  return sum;
}
constexpr double turn_cos(long n, long d) {
  n = ((n % d) + d) % d;
  if (2 * n > d) n = d - n;                                   // cos is even
  if (4 * n > d) return -turn_cos(d - 2 * n, 2 * d);          // cos x = -cos(pi - x)
  if (8 * n > d) return taylor(kTau * (d - 4 * n) / (4 * d), kTau * (d - 4 * n) / (4 * d), 1);   // sin(pi/2 - x)
  return taylor(kTau * n / d, 1.0, 0);
}
constexpr double turn_sin(long n, long d) { return turn_cos(4 * n - d, 4 * d); }   // cos(x - pi/2)

template <int R>
struct TurnTable {   // cos and sin of 2 pi k / R
  float c[R] = {}, s[R] = {};
  constexpr TurnTable() {
    for (int k = 0; k < R; ++k) {
      c[k] = (float)turn_cos(k, R);
      s[k] = (float)turn_sin(k, R);
    }
  }
};

constexpr int dft_factor(int r) {
  if (r % 4 == 0) return 4;
  for (int p = 2; p <= 13; ++p)
    if (r % p == 0) return p;
  return r;
}

// v[O + ST n], n < R, in place
template <int S, int R, int O = 0, int ST = 1, int N>
__device__ __forceinline__ void dft_small(float2 (&v)[N]) {
  static_assert(O + ST * (R - 1) < N, "range");
  if constexpr (R == 2) {
    const float2 a = v[O], b = v[O + ST];
    v[O] = make_float2(a.x + b.x, a.y + b.y);
    v[O + ST] = make_float2(a.x - b.x, a.y - b.y);
  } else if constexpr (R == 4) {
    const float2 x0 = v[O], x1 = v[O + ST], x2 = v[O + 2 * ST], x3 = v[O + 3 * ST];
    const float2 a0 = make_float2(x0.x + x2.x, x0.y + x2.y), a1 = make_float2(x0.x - x2.x, x0.y - x2.y);
    const float2 b0 = make_float2(x1.x + x3.x, x1.y + x3.y), d = make_float2(x1.x - x3.x, x1.y - x3.y);
    const float2 b1 = S > 0 ? make_float2(-d.y, d.x) : make_float2(d.y, -d.x);
    v[O] = make_float2(a0.x + b0.x, a0.y + b0.y);
    v[O + ST] = make_float2(a1.x + b1.x, a1.y + b1.y);
    v[O + 2 * ST] = make_float2(a0.x - b0.x, a0.y - b0.y);
    v[O + 3 * ST] = make_float2(a1.x - b1.x, a1.y - b1.y);
  } else if constexpr (dft_factor(R) == R) {
    constexpr TurnTable<R> T{};
    constexpr int H = (R - 1) / 2;
    const float2 x0 = v[O];
    float2 s[H], d[H], sum = x0;
#pragma unroll
    for (int n = 0; n < H; ++n) {
      const float2 a = v[O + ST * (n + 1)], b = v[O + ST * (R - 1 - n)];
      s[n] = make_float2(a.x + b.x, a.y + b.y);
      d[n] = make_float2(a.x - b.x, a.y - b.y);
      sum = make_float2(sum.x + s[n].x, sum.y + s[n].y);
    }
    v[O] = sum;
#pragma unroll
    for (int k = 1; k <= H; ++k) {
      float2 A = x0, B = make_float2(0.f, 0.f);
#pragma unroll
      for (int n = 0; n < H; ++n) {
        const int m = (n + 1) * k % R;
        A = make_float2(fmaf(T.c[m], s[n].x, A.x), fmaf(T.c[m], s[n].y, A.y));
        B = n == 0 ? make_float2(T.s[m] * d[n].x, T.s[m] * d[n].y)
                   : make_float2(fmaf(T.s[m], d[n].x, B.x), fmaf(T.s[m], d[n].y, B.y));
      }
      // A + i S B at k, A - i S B at R - k
      v[O + ST * (S > 0 ? k : R - k)] = make_float2(A.x - B.y, A.y + B.x);
      v[O + ST * (S > 0 ? R - k : k)] = make_float2(A.x + B.y, A.y - B.x);
    }
  } else {
    constexpr int P = dft_factor(R), Q = R / P;
    constexpr TurnTable<R> T{};
    float2 t[Q][P];
#pragma unroll
    for (int n2 = 0; n2 < Q; ++n2) {
      float2 u[P];
#pragma unroll
      for (int n1 = 0; n1 < P; ++n1) u[n1] = v[O + ST * (Q * n1 + n2)];
      dft_small<S, P>(u);
#pragma unroll
      for (int k1 = 0; k1 < P; ++k1) {
        const int m = n2 * k1 % R;
        const float c = T.c[m], sn = S > 0 ? T.s[m] : -T.s[m];
        t[n2][k1] = m == 0           ? u[k1]
                    : 4 * m == R     ? (S > 0 ? make_float2(-u[k1].y, u[k1].x) : make_float2(u[k1].y, -u[k1].x))
                                     : make_float2(fmaf(c, u[k1].x, -sn * u[k1].y), fmaf(c, u[k1].y, sn * u[k1].x));
      }
    }
#pragma unroll
    for (int k1 = 0; k1 < P; ++k1) {
      float2 w[Q];
#pragma unroll
      for (int n2 = 0; n2 < Q; ++n2) w[n2] = t[n2][k1];
      dft_small<S, Q>(w);
#pragma unroll
      for (int k2 = 0; k2 < Q; ++k2) v[O + ST * (k1 + P * k2)] = w[k2];
    }
  }
}

}  // namespace pam

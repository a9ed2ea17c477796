// K3 for FP32 operands, every lateral size N = 32 .. 512 in steps of 32: the inverse lateral
// transform as a 16 x N/16 FFT on the vector ALUs.
//
// Same factorisation as k3_factored.hpp (q = (N/16) q1 + q2, x = x1 + 16 x2):
//   stage 1  Y(x1, q2)  = sum_q1 A((N/16) q1 + q2) e^{2 pi i q1 x1 / 16}
//   twiddle  Y'(x1, q2) = Y(x1, q2) e^{2 pi i q2 x1 / N}
//   stage 3  p(x1 + 16 x2) = sum_q2 Y'(x1, q2) e^{2 pi i q2 x2 / (N/16)}
// but each small transform is a radix-4 FFT held in one lane's registers instead of a
// DFT-GEMM on the matrix cores.  On gfx950 the FP32 matrix product runs at twice the
// vector FMA rate and does not overlap vector work, while the GEMM form executes 256 flops
// per complex output against about 11 vector operations per point and stage for the FFT,
// so for FP32 operands the vector FFT is the faster form.  (The 16-bit forms keep the
// matrix cores, whose rate is eight times higher and which overlap vector work.)
//
// N = 256.  A wave holds four depths, one per group of 16 lanes (g = lane / 16), and lane j
// of a group holds column q2 = j of stage 1 and column x1 = j of stage 3, i.e. its pixels
// are x = j + 16 x2, x2 = 0..15.  Per bin and sub-aperture:
//   A(16 m + j) = H G for m = 0..15 from the staged row j (K2's [q2][q1] order),
//   16-point FFT over m, twiddle, transpose through the group's LDS block (row x1),
//   16-point FFT over q2: the 16 fields of the lane's pixels.
// The fold into the per-pixel sums is that of k3ff.  A workgroup is 4 waves = 16 depths of
// one frame, staging each bin's coefficients and kz row in LDS (double-buffered, one
// barrier per bin) exactly as k3ff does, so the workspace layout and K2 are shared.
// With COH (n_sub = 1) the adjacent-pixel pair sums come from lanes j ^ 1 (column
// partner) and g ^ 1, i.e. lane ^ 16 (depth partner).
//
// Other N <= 256: stage 3 has K = N / 16 < 16 points (dft_small.hpp, codelets at 8 and 16).
// A group then holds DG depths of CW = 16 / DG >= K stage-1 columns each: lane j is (depth
// j / CW, column q2 = j % CW), columns K .. CW - 1 idle; in stage 3 lane j = x1 runs DG
// transforms of K points, one per depth, and its pixels are (depth d, x = j + 16 x2), d < DG,
// x2 < K.  N = 128: two depths of 8 columns, 192: one of 12, 96: two of 6, 64: four of 4.
// A wave holds 4 DG depths and a workgroup 16 DG.
//
// N > 256 splits the sum by the parity e of q as k3ff does:
// p(x) = P_0(x mod N/2) + e^{2 pi i x / N} P_1(x mod N/2), P_e the transform of A(2 q' + e)
// over N/2 = 16 K points (K = 16 at N = 512, 12 at 384, ...).  The lane groups of a wave
// become (depth, e) = (g / 2, g % 2), so a wave holds two depths and a workgroup eight.  Lane
// (g, j) takes its inputs from staged row 2 j + e (q = 2 K m + 2 j + e, K2's order for
// N / 16 = 2 K rows); after stage 3 the lanes g and g ^ 1 (lane ^ 16) exchange P_0 and P_1 of
// their columns x' = j + 16 x2, and group e forms pixel x' + e N/2 as P_0 +- w P_1 with
// w = e^{2 pi i x' / N} (a K x 16 table in LDS).
//
// The sizes without a codelet ran as dense DFT-GEMMs on the FP32 matrix cores before (4 N
// flops per complex output against about 11 operations per point and stage): 4.14 -> 0.58 ms for
// 4 frames of 301 x 192 pixels and 691 bins (the idle stage-1 lanes, 4 of 16 here, are
// what it lacks to the rate of N = 256).
#pragma once
#include <utility>

#include "dft_small.hpp"
#include "k3_factored.hpp"

namespace pam {

constexpr int kFtWaves = 4;                    // waves per workgroup
constexpr int kFtTr = 16 * kFfRow;             // float2 per lane group's transpose block [16 x1][kFfRow]

// Shape of the transform at N columns.
template <int NN>
struct FtShape {
  static_assert(NN % 32 == 0 && NN >= 32 && NN <= 512, "lateral sizes 32 .. 512 in steps of 32");
  static constexpr int R = NN > 256 ? 2 : 1;                       // parities of q transformed apart
  static constexpr int K = NN / 16 / R;                            // stage-3 points
  static constexpr int DG = K <= 2 ? 8 : (K <= 4 ? 4 : (K <= 8 ? 2 : 1));   // depths per lane group
  static constexpr int CW = 16 / DG;                               // stage-1 columns (lanes) per depth
};
// depths per workgroup: 16 DG, 8 where a wave holds both parities
template <int NN>
__host__ __device__ constexpr int ft_depths() { return 16 * FtShape<NN>::DG / FtShape<NN>::R; }
inline int ft_depths_of(int n) { return n > 256 ? 8 : (n > 128 ? 16 : (n > 64 ? 32 : (n > 32 ? 64 : 128))); }

// The 16-byte pieces of a bin's staged inputs, 256 per pass (one per thread): one pass up to
// N = 128 (which three sub-apertures fill exactly), two up to 256, two parts of two passes
// beyond.  Separate members (not an array) so that they stay in registers.
template <int NSUB, int NN>
struct FtPiece {
  typedef FfRows<NSUB, NN / 16> P;
  static constexpr int R = FtShape<NN>::R;
  uint4 v0, v1, v2, v3;
  int d0, d1, d2, d3;
  __device__ FtPiece(int tid) {
    d0 = P::where(tid);
    d1 = NN > 128 ? P::where(tid + 256) : -1;
    d2 = R > 1 ? P::where(tid + 512) : -1;
    d3 = R > 1 ? P::where(tid + 768) : -1;
  }
  // pieces 0, 1 (part 0) and, beyond N = 256, pieces 2, 3 (part 1): the kernel moves the two
  // parts at different points of a bin so that only two are in registers at a time
  __device__ __forceinline__ void load(const K3Args& a, int f, int b, int tid, int part) {
    if (part == 0) {
      if (d0 >= 0) v0 = P::fetch(a, f, b, tid);
      if (NN > 128 && d1 >= 0) v1 = P::fetch(a, f, b, tid + 256);
    } else if (R > 1) {
      if (d2 >= 0) v2 = P::fetch(a, f, b, tid + 512);
      if (d3 >= 0) v3 = P::fetch(a, f, b, tid + 768);
    }
  }
  __device__ __forceinline__ void store(float2* stage, int part) const {
    if (part == 0) {
      if (d0 >= 0) *reinterpret_cast<uint4*>(stage + d0) = v0;
      if (NN > 128 && d1 >= 0) *reinterpret_cast<uint4*>(stage + d1) = v1;
    } else if (R > 1) {
      if (d2 >= 0) *reinterpret_cast<uint4*>(stage + d2) = v2;
      if (d3 >= 0) *reinterpret_cast<uint4*>(stage + d3) = v3;
    }
  }
};

__device__ __forceinline__ float2 f2add(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 f2sub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 f2iadd(float2 a, float2 b) { return make_float2(a.x - b.y, a.y + b.x); }  // a + i b
__device__ __forceinline__ float2 f2isub(float2 a, float2 b) { return make_float2(a.x + b.y, a.y - b.x); }  // a - i b

// In-register inverse 16-point DFT, natural order in and out:
//   v[k] <- sum_n v[n] e^{+2 pi i n k / 16}.
// Radix 4 x 4 with n = 4 n1 + n2 and k = k1 + 4 k2: 4-point transforms over n1, then for
// each k1 the 4-point transform over n2 of y_n2 = W^(n2 k1) T[n2][k1], W = e^{2 pi i / 16}.
// The twiddled inputs of that second transform are written as y = c (x + i t x), c and t
// the cosine and tangent of the twiddle angle, so that the rotation costs two FMAs and its
// cosine folds into the butterfly's FMAs; y1 +- y3 = c1 (u1 +- (c3 / c1) u3) shares the
// factor c1.  A twiddled column then takes 22 operations instead of 28 (20 instead of 24 at
// k1 = 2).  Every tangent and cosine ratio used lies within [-2.42, 2.42].
__device__ __forceinline__ float2 tan_rot(float2 x, float t) {   // x + i t x
  return make_float2(fmaf(-t, x.y, x.x), fmaf(t, x.x, x.y));
}
// second-stage column with general twiddles W^k1, W^2k1, W^3k1 (k1 = 1 or 3):
// y0 = x0, yj = cj uj with uj = xj + i tj xj; r = c3 / c1
__device__ __forceinline__ void idft4_tw(float2& x0, float2& x1, float2& x2, float2& x3, float c1, float t1, float c2,
                                         float t2, float t3, float r) {
  const float2 u1 = tan_rot(x1, t1), u2 = tan_rot(x2, t2), u3 = tan_rot(x3, t3);
  const float2 a0 = make_float2(fmaf(c2, u2.x, x0.x), fmaf(c2, u2.y, x0.y));      // y0 + y2
  const float2 a1 = make_float2(fmaf(-c2, u2.x, x0.x), fmaf(-c2, u2.y, x0.y));    // y0 - y2
  const float2 v = make_float2(fmaf(r, u3.x, u1.x), fmaf(r, u3.y, u1.y));         // (y1 + y3) / c1
  const float2 w = make_float2(fmaf(-r, u3.x, u1.x), fmaf(-r, u3.y, u1.y));       // (y1 - y3) / c1
  x0 = make_float2(fmaf(c1, v.x, a0.x), fmaf(c1, v.y, a0.y));
  x2 = make_float2(fmaf(-c1, v.x, a0.x), fmaf(-c1, v.y, a0.y));
  x1 = make_float2(fmaf(-c1, w.y, a1.x), fmaf(c1, w.x, a1.y));                   // a1 + i (y1 - y3)
  x3 = make_float2(fmaf(c1, w.y, a1.x), fmaf(-c1, w.x, a1.y));                   // a1 - i (y1 - y3)
}
// in(n2) is called when inputs n2, n2 + 4, n2 + 8 and n2 + 12 are needed, out(k1) when outputs k1, k1 + 4, k1 + 8 and
// k1 + 12 are in v.
template <typename In, typename Out>
__device__ __forceinline__ void idft16(float2 (&v)[16], In&& in, Out&& out) {
  constexpr float C1 = 0.92387953251128674f;   // cos(pi / 8)
  constexpr float S1 = 0.38268343236508977f;   // sin(pi / 8) = cos(3 pi / 8)
  constexpr float R2 = 0.70710678118654752f;   // cos(pi / 4)
  constexpr float T1 = 0.41421356237309505f;   // tan(pi / 8)
  constexpr float T3 = 2.41421356237309505f;   // tan(3 pi / 8)
  float2 T[4][4];
#pragma unroll
  for (int n2 = 0; n2 < 4; ++n2) {
    in(n2);
    const float2 a0 = f2add(v[n2], v[8 + n2]), a1 = f2sub(v[n2], v[8 + n2]);
    const float2 b0 = f2add(v[4 + n2], v[12 + n2]), b1 = f2sub(v[4 + n2], v[12 + n2]);
    T[n2][0] = f2add(a0, b0);
    T[n2][2] = f2sub(a0, b0);
    T[n2][1] = f2iadd(a1, b1);
    T[n2][3] = f2isub(a1, b1);
  }
  // k1 = 0: no twiddles
  {
    const float2 a0 = f2add(T[0][0], T[2][0]), a1 = f2sub(T[0][0], T[2][0]);
    const float2 b0 = f2add(T[1][0], T[3][0]), b1 = f2sub(T[1][0], T[3][0]);
    v[0] = f2add(a0, b0);
    v[8] = f2sub(a0, b0);
    v[4] = f2iadd(a1, b1);
    v[12] = f2isub(a1, b1);
  }
  out(0);
  // k1 = 1: W^1 (pi / 8), W^2 (pi / 4), W^3 (3 pi / 8)
  idft4_tw(T[0][1], T[1][1], T[2][1], T[3][1], C1, T1, R2, 1.0f, T3, S1 / C1);
  v[1] = T[0][1];
  v[5] = T[1][1];
  v[9] = T[2][1];
  v[13] = T[3][1];
  out(1);
  // k1 = 2: W^2 (pi / 4), W^4 = i, W^6 (3 pi / 4); y1 +- y3 = R2 (u1 -+ u3)
  {
    const float2 x0 = T[0][2], x2 = T[2][2];
    const float2 a0 = make_float2(x0.x - x2.y, x0.y + x2.x);                   // y0 + i x2
    const float2 a1 = make_float2(x0.x + x2.y, x0.y - x2.x);                   // y0 - i x2
    const float2 u1 = make_float2(T[1][2].x - T[1][2].y, T[1][2].y + T[1][2].x);   // (1 + i) x1
    const float2 u3 = make_float2(T[3][2].x + T[3][2].y, T[3][2].y - T[3][2].x);   // (1 - i) x3 = -(-1 + i) x3
    const float2 s = f2sub(u1, u3), d = f2add(u1, u3);                          // (y1 + y3), (y1 - y3) over R2
    v[2] = make_float2(fmaf(R2, s.x, a0.x), fmaf(R2, s.y, a0.y));
    v[10] = make_float2(fmaf(-R2, s.x, a0.x), fmaf(-R2, s.y, a0.y));
    v[6] = make_float2(fmaf(-R2, d.y, a1.x), fmaf(R2, d.x, a1.y));
    v[14] = make_float2(fmaf(R2, d.y, a1.x), fmaf(-R2, d.x, a1.y));
  }
  out(2);
  // k1 = 3: W^3 (3 pi / 8), W^6 (3 pi / 4), W^9 (9 pi / 8)
  idft4_tw(T[0][3], T[1][3], T[2][3], T[3][3], S1, T3, -R2, -1.0f, T1, -C1 / S1);
  v[3] = T[0][3];
  v[7] = T[1][3];
  v[11] = T[2][3];
  v[15] = T[3][3];
  out(3);
}

// An LDS address the compiler cannot see through: accesses at constant offsets from it keep this base, so that pairs of
// 8-byte accesses merge into one instruction (their offsets are 8 bits wide; from a shared base they do not fit).
typedef float f2v __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) f2v lds_f2;
typedef __attribute__((address_space(3))) v4f lds_f4;
__device__ __forceinline__ float2 get2(const lds_f2* p) {
  const f2v v = *p;
  return make_float2(v.x, v.y);
}
__device__ __forceinline__ void put2(lds_f2* p, float2 v) { *p = f2v{v.x, v.y}; }
__device__ __forceinline__ lds_f2* lds_base(float2* p) {
  unsigned a = (unsigned)(uintptr_t)(lds_f2*)p;
  asm volatile("" : "+v"(a));
  return (lds_f2*)(uintptr_t)a;
}

// Stage 3 with the twiddles folded into the transform (16 and 8 points).  The twiddle of input n is
// w_n = c_n (1 + i t_n), c_n and t_n the cosine and tangent of 2 pi n x1 / 16 K, x1 the lane's row.  u_n = y_n + i t_n y_n
// costs two FMAs; the cosines enter the butterflies' FMAs as ratios, so a butterfly of scaled inputs takes as many
// operations as one of plain inputs: with s_n2 = c_n2 the scale of column n2 of the first stage,
//   a = u_n2 +- (c_{8+n2} / c_n2) u_{8+n2}, b = u_{4+n2} +- (c_{12+n2} / c_{4+n2}) u_{12+n2},
//   T = a +- (c_{4+n2} / c_n2) (i) b,
// and s_n2 multiplies the second stage's constant twiddles.  144 + 30 operations at 16 points instead of 144 + 64.
// The constants depend on the lane's row only: float4s k at c[16 k] (ft_table on the host).  A cosine of zero (n x1 a
// quarter turn of 16 K: (8, 8) at K = 16, (4, 8) at K = 8) is stored as 2^-30, its tangent as 2^30: the product is exact.
__device__ __forceinline__ void bfly_scaled(float2& x0, float2& x1, float2& x2, float2& x3, float al, float be, float ga) {
  const float2 a0 = make_float2(fmaf(al, x2.x, x0.x), fmaf(al, x2.y, x0.y));
  const float2 a1 = make_float2(fmaf(-al, x2.x, x0.x), fmaf(-al, x2.y, x0.y));
  const float2 b0 = make_float2(fmaf(ga, x3.x, x1.x), fmaf(ga, x3.y, x1.y));
  const float2 b1 = make_float2(fmaf(-ga, x3.x, x1.x), fmaf(-ga, x3.y, x1.y));
  x0 = make_float2(fmaf(be, b0.x, a0.x), fmaf(be, b0.y, a0.y));
  x2 = make_float2(fmaf(-be, b0.x, a0.x), fmaf(-be, b0.y, a0.y));
  x1 = make_float2(fmaf(-be, b1.y, a1.x), fmaf(be, b1.x, a1.y));       // a1 + i be b1
  x3 = make_float2(fmaf(be, b1.y, a1.x), fmaf(-be, b1.x, a1.y));
}
// the column of twiddles i c2 and (1 +- i) in the second stage: y0 + i c2 x2, y1 +- y3 = cr ((1 + i) x1 -+ rho (1 - i) x3)
__device__ __forceinline__ void idft4_quarter(float2& x0, float2& x1, float2& x2, float2& x3, float c2, float cr, float rho) {
  const float2 a0 = make_float2(fmaf(-c2, x2.y, x0.x), fmaf(c2, x2.x, x0.y));
  const float2 a1 = make_float2(fmaf(c2, x2.y, x0.x), fmaf(-c2, x2.x, x0.y));
  const float2 u1 = make_float2(x1.x - x1.y, x1.y + x1.x);             // (1 + i) x1
  const float2 u3 = make_float2(x3.x + x3.y, x3.y - x3.x);             // (1 - i) x3
  const float2 v = make_float2(fmaf(-rho, u3.x, u1.x), fmaf(-rho, u3.y, u1.y));
  const float2 w = make_float2(fmaf(rho, u3.x, u1.x), fmaf(rho, u3.y, u1.y));
  x0 = make_float2(fmaf(cr, v.x, a0.x), fmaf(cr, v.y, a0.y));
  x2 = make_float2(fmaf(-cr, v.x, a0.x), fmaf(-cr, v.y, a0.y));
  x1 = make_float2(fmaf(-cr, w.y, a1.x), fmaf(cr, w.x, a1.y));
  x3 = make_float2(fmaf(cr, w.y, a1.x), fmaf(-cr, w.x, a1.y));
}
template <int NSUB>
__device__ __forceinline__ void idft16_tw(float2 (&p)[NSUB][16], const lds_f4* c) {
  constexpr float T1 = 0.41421356237309505f;   // tan(pi / 8)
  constexpr float T3 = 2.41421356237309505f;   // tan(3 pi / 8)
  // c[2 n2]: tangents of n2, 4 + n2, 8 + n2, 12 + n2; c[2 n2 + 1]: the column's three ratios and one of s1 s2 rho C1 s1;
  // c[8], c[9]: R2 s2, (S1 / C1) rho, R2 s1, S1 s1 | (-C1 / S1) rho.  Every sub-aperture's column takes the constants
  // while they are in registers; the next column's load during its butterflies.
  float q[4];
  v4f t = c[0], r = c[16];
#pragma unroll
  for (int n2 = 0; n2 < 4; ++n2) {
    const v4f tn = c[32 * (n2 + 1)], rn = c[32 * (n2 + 1) + 16];
    q[n2] = r[3];
#pragma unroll
    for (int i = 0; i < NSUB; ++i) {
      float2(&v)[16] = p[i];
      if (n2 > 0) v[n2] = tan_rot(v[n2], t[0]);
      v[4 + n2] = tan_rot(v[4 + n2], t[1]);
      v[8 + n2] = tan_rot(v[8 + n2], t[2]);
      v[12 + n2] = tan_rot(v[12 + n2], t[3]);
      // x_k1 at v[4 k1 + n2]: the order idft4 of (n2, 4 + n2, 8 + n2, 12 + n2) gives
      bfly_scaled(v[n2], v[4 + n2], v[8 + n2], v[12 + n2], r[0], r[1], r[2]);
    }
    t = tn;
    r = rn;
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int i = 0; i < NSUB; ++i) {
    float2(&v)[16] = p[i];
    // second stage over n2 for each k1, in place in v[4 k1 ..]
    bfly_scaled(v[0], v[1], v[2], v[3], q[1], q[0], q[2]);
    idft4_tw(v[4], v[5], v[6], v[7], q[3], T1, t[0], 1.0f, T3, t[1]);
    idft4_quarter(v[8], v[9], v[10], v[11], q[1], t[2], q[2]);
    idft4_tw(v[12], v[13], v[14], v[15], t[3], T3, -t[0], -1.0f, T1, r[0]);
    // v[4 k1 + k2] holds output k1 + 4 k2
#pragma unroll
    for (int k1 = 0; k1 < 4; ++k1)
#pragma unroll
      for (int k2 = k1 + 1; k2 < 4; ++k2) {
        const float2 x = v[4 * k1 + k2];
        v[4 * k1 + k2] = v[4 * k2 + k1];
        v[4 * k2 + k1] = x;
      }
  }
}
// 8 points at v[O ..]: first stage of two inputs n2, 4 + n2; second stage k1 = 0 and k1 = 1 (twiddles W8^n2)
template <int O>
__device__ __forceinline__ void idft8_tw(float2 (&v)[16], const v4f (&c)[4]) {
  // c: t1 t2 t3 t4 | t5 t6 t7 al0 | al1 al2 al3 s1 | s2 rho R2 s1 -
  const float al[4] = {c[1][3], c[2][0], c[2][1], c[2][2]};
  const float t[8] = {0.f, c[0][0], c[0][1], c[0][2], c[0][3], c[1][0], c[1][1], c[1][2]};
  float2 a[4], b[4];
#pragma unroll
  for (int n2 = 0; n2 < 4; ++n2) {
    const float2 x = n2 > 0 ? tan_rot(v[O + n2], t[n2]) : v[O], y = tan_rot(v[O + 4 + n2], t[4 + n2]);
    a[n2] = make_float2(fmaf(al[n2], y.x, x.x), fmaf(al[n2], y.y, x.y));
    b[n2] = make_float2(fmaf(-al[n2], y.x, x.x), fmaf(-al[n2], y.y, x.y));
  }
  bfly_scaled(a[0], a[1], a[2], a[3], c[3][0], c[2][3], c[3][1]);
  idft4_quarter(b[0], b[1], b[2], b[3], c[3][0], c[3][2], c[3][1]);
#pragma unroll
  for (int k2 = 0; k2 < 4; ++k2) {
    v[O + 2 * k2] = a[k2];
    v[O + 2 * k2 + 1] = b[k2];
  }
}

// y w with the roundings written out (the compiler is free to contract a plain product either way)
__device__ __forceinline__ float2 twiddled(float2 y, float2 w) {
  return make_float2(fmaf(y.x, w.x, -(y.y * w.y)), fmaf(y.y, w.x, y.x * w.y));
}

// Whether stage 3 of N columns takes its twiddles itself (else they multiply the stage-1 outputs), and the size of the
// table in LDS: [10 or 4 float4][16 rows], or [16 x1][16 j] factors.  The pair sums (COH) keep the plain twiddles: they
// become BF16 features, where a last-bit difference moves the network's output by a BF16 rounding.
template <int NN, bool COH = false>
__host__ __device__ constexpr bool ft_folded() { return !COH && (FtShape<NN>::K == 16 || FtShape<NN>::K == 8); }
template <int NN, bool COH = false>
__host__ __device__ constexpr int ft_stage_tw() { return !ft_folded<NN, COH>() ? 256 : (FtShape<NN>::K == 16 ? 320 : 128); }

// LDS: staged bins [2][ff_stage_rows], the stage-3 constants or stage twiddles, (N > 256) combination
// twiddles [2 e][16 x2][16 j], transpose blocks [4 waves][4 groups][kFtTr].
template <int NN, bool COH = false>
__host__ __device__ constexpr int ft_twiddles() { return ft_stage_tw<NN, COH>() + (NN > 256 ? 512 : 0); }
template <int NSUB, int NN = 256, bool COH = false>
inline size_t k3fft_lds() {
  return (size_t)(2 * ff_stage_rows<NSUB, NN / 16>() + ft_twiddles<NN, COH>() + kFtWaves * 4 * kFtTr) * sizeof(float2);
}

// The K-point transforms of stage 3 for every sub-aperture, depth D's at p[i][D CW ..]; c: the lane's constants (folded
// forms).
template <int NN, bool FOLDED, int NSUB, int... D>
__device__ __forceinline__ void stage3(float2 (&p)[NSUB][16], const lds_f4* c, std::integer_sequence<int, D...>) {
  constexpr int K = FtShape<NN>::K;
  if constexpr (K == 16 && FOLDED) {
    idft16_tw(p, c);
  } else if constexpr (K == 16) {
#pragma unroll
    for (int i = 0; i < NSUB; ++i) idft16(p[i], [](int) {}, [](int) {});
  } else if constexpr (K == 8) {
    const v4f cc[4] = {c[0], c[16], c[32], c[48]};
#pragma unroll
    for (int i = 0; i < NSUB; ++i) (idft8_tw<8 * D>(p[i], cc), ...);
  } else {
#pragma unroll
    for (int i = 0; i < NSUB; ++i) (dft_small<1, K, D * FtShape<NN>::CW>(p[i]), ...);
  }
}

// kz(q) = kz(N - q), so the propagator of a column's m = 9 .. 15 is that of another column's 15 - m at the same
// depth.  N <= 256 (q = K m + q2): N - q = K (15 - m) + (K - q2), column K - q2 of the same CW lanes; column 0 pairs
// with itself as H[16 - m] (the caller's case).  N > 256 (q = 2 K m + 2 j + e): columns K - j in the even-q rows,
// K - 1 - j in the odd-q rows.  This returns the partner column's value: a DPP rotation of the row of 16 lanes by n
// (lane i takes lane i - n) and a mirror of the row (15 - i) or of its halves (7 - i), so lane i receives lane
// 15 - n - i or 7 - n - i; rows 0, 2 (even q) and 1, 3 (odd q) rotate apart through the row mask.
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}
template <int NN>
__device__ __forceinline__ float partner_column(float v) {
  typedef FtShape<NN> F;
  constexpr int K = F::K;
  if constexpr (F::R == 2) {
    constexpr int even = (15 - K) & 15, odd = (16 - K) & 15;
    const int x = __builtin_bit_cast(int, v);
    int t = x;
    if constexpr (even > 0) t = __builtin_amdgcn_update_dpp(t, x, 0x120 + even, 0x5, 0xF, false);
    if constexpr (odd > 0) t = __builtin_amdgcn_update_dpp(t, x, 0x120 + odd, 0xA, 0xF, false);
    return dpp_mov<0x140>(__builtin_bit_cast(float, t));
  } else if constexpr (F::CW == 16) {
    return dpp_mov<0x140>(dpp_mov<0x120 + ((15 - K) & 15)>(v));
  } else if constexpr (F::CW == 8) {
    return dpp_mov<0x141>(dpp_mov<0x120 + ((7 - K) & 15)>(v));
  } else if constexpr (F::CW == 4) {
    return dpp_mov<0x6C>(v);                     // quad permutation [0, 3, 2, 1]
  } else {
    return v;                                    // K = 2: column 1 pairs with itself
  }
}

// Bound: the vector ALUs' issue (about 1,470 instructions per wave and bin at N = 256 and three sub-apertures), as long
// as the LDS instructions keep out of each other's way.  A wave issues 89 of those a bin, and in bursts (sixteen row
// writes, eight row reads, eight coefficient reads in a row) they stall both waves of a SIMD in the LDS queue, so they
// are spread over the arithmetic, held in place by scheduling barriers: coefficients in two halves, the previous
// sub-aperture's row reads between the columns of stage 1, row writes after each column of its second stage, and the
// stage-3 constants read once a bin for all sub-apertures.  64 frames of the benchmark array (512 x 256, 768 bins): 17.1
// ms with twiddles multiplied between the stages, 17.5 with them folded but the LDS instructions in bursts, 15.7 so.
// One frame of 1,024 x 512 pixels and 3,072 bins: 6.37 -> 5.55 ms; 4 of 301 x 192 and 691: 0.578 -> 0.535.
// The mirrored propagator values through LDS instead of two DPP moves and a select (42 vector instructions fewer)
// measured the same at N = 256 and 6 % slower at 512.
//
// Two workgroups per CU (at most 256 VGPRs a lane).  At N = 512 with three sub-apertures this spills a few values per bin
// to scratch, which measures faster (about 1.4x) than one workgroup per CU without spills.
//
// EARLY: with one sub-aperture (up to 256 columns) the next bin's inputs are stored and the bin's barrier passed before
// stage 3, which ends their registers there; with three it measured 1 % slower at 512 columns.
// LEAN (with the pair sums): EARLY and the twiddles read where they are used, 164 registers instead of 194, so that three
// workgroups fit a CU.  64 frames of the benchmark array 8.67 -> 7.76 ms, 24 frames in two bin splits 3.35 -> 3.05, and
// over workgroups per CU 1.17 to 1.21 times as fast at three and 1.09 to 1.14 beyond four; but up to two it is 0.90 to
// 0.96 (16 frames 2.28 ms against 2.45), and at four, which it runs as three and one, 1.03 with 8 bins a workgroup, 0.99
// with 24 and 0.95 with 55, so those launches keep the other form.
template <int NSUB, bool COH = false, int NN = 256, bool LEAN = false>
__global__ __launch_bounds__(256, 2) void k3fft(K3Args a0, K3Groups grp) {
  static_assert(!COH || (NSUB == 1 && NN == 256), "pair cross-spectra come with the full-aperture sums at N = 256");
  constexpr int NP = AccCount<NSUB>::pairs;
  constexpr int N = NN;
  constexpr int R = FtShape<NN>::R, K = FtShape<NN>::K, DG = FtShape<NN>::DG, CW = FtShape<NN>::CW;
  constexpr int PX = DG * K;                                       // pixels per lane
  constexpr bool FOLDED = ft_folded<NN, COH>();
  constexpr bool EARLY = NSUB == 1 && R == 1 && (!COH || LEAN);
  constexpr bool SPREAD = !COH || LEAN;
  constexpr int ROWS = NN / 16;
  extern __shared__ float2 lds_ft[];
  float2* stage = lds_ft;                                          // [2][ff_stage_rows]
  float2* twl = lds_ft + 2 * ff_stage_rows<NSUB, ROWS>();          // stage-3 constants or twiddles (+ [2 e][16 x2][16 j])
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int g = lane >> 4, j = lane & 15;
  const int e = R == 2 ? (g & 1) : 0;                              // parity of q (N > 256)
  float2* tr = twl + ft_twiddles<NN, COH>() + (w * 4 + g) * kFtTr;     // this group's transpose block
  // stage-1 column of this lane (idle lanes repeat the last one) and its staged row
  const int col = K == CW ? j % CW : min(j % CW, K - 1);
  const int srow = R == 1 ? col : 2 * col + e;
  K3Args a = a0;
  const WgFF wg(a, wg_group(a, grp));
  const int f = wg.f;
  // first depth of the lane's pixels, and the depth of its stage-1 column
  const int depth = wg.dt * ft_depths<NN>() + (R == 1 ? (4 * w + g) * DG : 2 * w + (g >> 1));
  const int depth1 = depth + j / CW;
  const double z = depth1 < a.n_z ? a.z[depth1] : 0.0;

  // stage-3 constants or twiddles e^{2 pi i q2 x1 / 16 K}, and (N > 256) the combination twiddles
  // e^{2 pi i (j + 16 x2 + e N/2) / N}, the e = 1 half the negated e = 0 half (FP32 tables built in FP64)
  constexpr int TW = ft_stage_tw<NN, COH>();
  for (int k = tid; k < TW; k += 256) twl[k] = a.ff_tw_vec[k];
  if constexpr (R == 2) {
    const float2 t = a.ff_tw2_vec[tid];
    twl[TW + tid] = t;
    twl[TW + 256 + tid] = make_float2(-t.x, -t.y);
  }

  float accS[NSUB][PX];
  float accC[NP > 0 ? NP : 1][PX];
  float accG[COH ? 4 : 1][PX];
#pragma unroll
  for (int x2 = 0; x2 < PX; ++x2) {
#pragma unroll
    for (int i = 0; i < NSUB; ++i) accS[i][x2] = 0.f;
#pragma unroll
    for (int p = 0; p < (NP > 0 ? NP : 1); ++p) accC[p][x2] = 0.f;
#pragma unroll
    for (int q = 0; q < (COH ? 4 : 1); ++q) accG[q][x2] = 0.f;
  }

  lds_f2* const tcol = lds_base(tr + j);                            // column j of the transpose block
  lds_f2* const trow = lds_base(tr + j * kFfRow);                   // row j
  lds_f2* const grow = lds_base(stage + srow * kFfRow);             // staged coefficients of the lane's row
  lds_f2* const twj = lds_base(twl + (FOLDED ? 2 : 1) * j);   // this row's constants or this column's twiddles
  const lds_f4* const twc4 = (const lds_f4*)twj;
  lds_f2* const twc = R == 2 ? lds_base(twl + TW + 256 * e + j) : twj;

  FtPiece<NSUB, NN> pc(tid);
  if (wg.b_begin < wg.b_end) {
#pragma unroll
    for (int part = 0; part < R; ++part) {
      pc.load(a, f, wg.b_begin, tid, part);
      pc.store(stage, part);
    }
  }
  __syncthreads();
  for (int b = wg.b_begin; b < wg.b_end; ++b) {
    const bool more = b + 1 < wg.b_end;
    float2* nxt = stage + ((b + 1 - wg.b_begin) & 1) * ff_stage_rows<NSUB, ROWS>();   // free since the last barrier
    if (more) pc.load(a, f, b + 1, tid, 0);
    const float2* st = stage + ((b - wg.b_begin) & 1) * ff_stage_rows<NSUB, ROWS>();
    const double* kzr = reinterpret_cast<const double*>(st + NSUB * ROWS * kFfRow) + srow * kFfRow;
    // propagator at q = K m + col or 2 K m + 2 col + e (Eq. 2): phase in FP64 reduced to [-1/2, 1/2] cycle, hardware
    // sin/cos; evanescent values replaced in a branch only lanes holding any take.  A lane computes H[0..8] and takes
    // the other seven from its partner column (partner_column above).
    constexpr int MD = 9;   // values computed directly
    float2 H[16];
#pragma unroll
    for (int m = 0; m < MD; ++m) {
      const double ph = z * kzr[m];
      const float r = (float)(ph - rint(ph));
      H[m] = make_float2(__builtin_amdgcn_cosf(r), __builtin_amdgcn_sinf(r));
    }
    if (a.ev_bin[b]) {
#pragma unroll
      for (int m = 0; m < MD; ++m)
        if (kzr[m] < 0.0) H[m] = propagator(z, kzr[m], a.zero_evanescent);
    }
    {
      const bool self = col == 0 && e == 0;
#pragma unroll
      for (int m = MD; m < 16; ++m) {
        const float2 o = make_float2(partner_column<NN>(H[15 - m].x), partner_column<NN>(H[15 - m].y));
        H[m] = self ? H[16 - m] : o;
      }
    }
    // Stage 1 and the transpose sub-aperture by sub-aperture (one's row reads are in flight during the next one's stage
    // 1), then stage 3 of all of them, so that each constant is read once a bin.
    float2 p[NSUB][16];
    // S_i and C_ij sums over the bins (Eq. 4): sum |p_i|^2, sum Re(p_i conj p_j)
    auto add_s = [&](int i) {
#pragma unroll
      for (int px = 0; px < PX; ++px) {
        const float2 v = p[i][px / K * CW + px % K];               // of depth px / K
        accS[i][px] = fmaf(v.x, v.x, fmaf(v.y, v.y, accS[i][px]));
      }
    };
    auto add_c = [&](int c, int i, int j2) {
#pragma unroll
      for (int px = 0; px < PX; ++px) {
        const float2 v = p[i][px / K * CW + px % K], u = p[j2][px / K * CW + px % K];
        accC[c][px] = fmaf(v.x, u.x, fmaf(v.y, u.y, accC[c][px]));
      }
    };
    // half h of row x1 = j of the transpose block
    auto rows = [&](float2 (&v)[16], int h) {
#pragma unroll
      for (int k = 4 * h; k < 4 * h + 4; ++k) {
        const v4f yy = *(lds_f4*)(trow + 2 * k);
        v[2 * k] = make_float2(yy.x, yy.y);
        v[2 * k + 1] = make_float2(yy.z, yy.w);
      }
    };
    // A column's twiddles stay in registers for the bin, also where a few spill (24 at 32 lateral
    // samples: 152 us against 163 for 16 frames with them read at their use; 64: 281 / 299; 416:
    // 3029 / 3160; 448 even).  With 15 points in stage 3 69 spill and reading them wins: 3452 -> 3230.
    constexpr bool TWREG = !FOLDED && !LEAN && (NSUB < 3 || K < 15);
    float2 tw[TWREG ? 16 : 1];
    if constexpr (TWREG) {
#pragma unroll
      for (int x1 = 1; x1 < 16; ++x1) tw[x1] = get2(twj + x1 * 16);
    }
    v4f ga[4], gb[4];
    auto coeffs = [&](int i, int h, v4f (&g)[4]) {                 // staged pairs 2 k + h: inputs 4 k + 2 h, 4 k + 2 h + 1
#pragma unroll
      for (int k = 0; k < 4; ++k)
        g[k] = *(lds_f4*)(grow + ((b - wg.b_begin) & 1) * ff_stage_rows<NSUB, ROWS>() + i * ROWS * kFfRow + 4 * k + 2 * h);
    };
#pragma unroll
    for (int i = 0; i < NSUB; ++i) {
      coeffs(i, 0, ga);
      idft16(p[i], [&](int n2) {
        if (n2 & 1) return;
        if (n2 == 0) coeffs(i, 1, gb);
        if constexpr (SPREAD) __builtin_amdgcn_sched_barrier(0);
        if (n2 == 2 && i > 0) rows(p[i - 1], 0);
        v4f (&g)[4] = n2 ? gb : ga;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int m = 4 * k + n2;
          p[i][m] = cmul(H[m], make_float2(g[k].x, g[k].y));
          p[i][m + 1] = cmul(H[m + 1], make_float2(g[k].z, g[k].w));
        }
      }, [&](int k1) {                                             // Y(x1, q2 = j), x1 = 0..15
        if (k1 == 0) {
          if (i > 0) rows(p[i - 1], 1);
          __builtin_amdgcn_wave_barrier();
        }
#pragma unroll
        for (int x1 = k1; x1 < 16; x1 += 4) {
          if constexpr (FOLDED) put2(tcol + x1 * kFfRow, p[i][x1]);
          else if constexpr (!TWREG) put2(tcol + x1 * kFfRow, twiddled(p[i][x1], get2(twj + x1 * 16)));
          else put2(tcol + x1 * kFfRow, x1 == 0 ? p[i][x1] : twiddled(p[i][x1], tw[x1]));
        }
        if constexpr (SPREAD) __builtin_amdgcn_sched_barrier(0);
      });
      __builtin_amdgcn_wave_barrier();
      if (R == 2 && i == 0 && more) {
        pc.store(nxt, 0);
        pc.load(a, f, b + 1, tid, 1);
      }
    }
    if constexpr (EARLY) {
      if (more) pc.store(nxt, R - 1);
      __syncthreads();
    }
    rows(p[NSUB - 1], 0);
    rows(p[NSUB - 1], 1);
    stage3<NN, FOLDED>(p, twc4, std::make_integer_sequence<int, DG>());    // depth d: p(j + 16 x2) in p[i][d CW + x2]
    // the fields are final here (sunk to the fold, the last butterflies or the combination would keep their inputs live)
    if constexpr (R == 2) {
      // p(x' + e N/2) = P_0(x') + w P_1(x'), x' = j + 16 x2, w = e^{2 pi i (x' + e N/2) / N}: the even row of
      // each row pair (e = 0) holds P_0(x'), the odd row P_1(x'), and one row swap hands both to both rows
#pragma unroll
      for (int x2 = 0; x2 < K; ++x2) {
        const float2 w2 = get2(twc + x2 * 16);
#pragma unroll
        for (int i = 0; i < NSUB; ++i) {
          const float2 re = rows_even_odd(p[i][x2].x), im = rows_even_odd(p[i][x2].y);   // (P_0, P_1) parts
          p[i][x2] = make_float2(fmaf(w2.x, re.y, fmaf(-w2.y, im.y, re.x)), fmaf(w2.x, im.y, fmaf(w2.y, re.y, im.x)));
          asm volatile("" : "+v"(p[i][x2].x), "+v"(p[i][x2].y));
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < NSUB; ++i)
#pragma unroll
        for (int d = 0; d < DG; ++d)
#pragma unroll
          for (int k = 0; k < K; ++k) asm volatile("" : "+v"(p[i][d * CW + k].x), "+v"(p[i][d * CW + k].y));
    }
#pragma unroll
    for (int i = 0; i < NSUB; ++i) add_s(i);
    if constexpr (NSUB == 3) {
      add_c(0, 0, 1);
      add_c(1, 1, 2);
      add_c(2, 2, 0);
    } else if constexpr (NSUB == 2) {
      add_c(0, 0, 1);
    }
    if constexpr (COH) {
#pragma unroll
      for (int px = 0; px < PX; ++px) {
        const float pr = p[0][px].x, pi = p[0][px].y;
        const float lr = lane_xor1(pr), li = lane_xor1(pi);
        const float zr = lane_xor16(pr), zi = lane_xor16(pi);
        accG[0][px] = fmaf(pr, lr, fmaf(pi, li, accG[0][px]));
        accG[1][px] = fmaf(pi, lr, fmaf(-pr, li, accG[1][px]));
        accG[2][px] = fmaf(pr, zr, fmaf(pi, zi, accG[2][px]));
        accG[3][px] = fmaf(pi, zr, fmaf(-pr, zi, accG[3][px]));
      }
    }
    if constexpr (!EARLY) {
      if (more) pc.store(nxt, R - 1);
      __syncthreads();
    }
  }
  constexpr int NA = COH ? 5 : AccCount<NSUB>::total;
  const size_t plane = (size_t)a.n_z * N;
  float* base = a.accum + ((size_t)wg.sp * a.F + f) * NA * plane;
#pragma unroll
  for (int k = 0; k < PX; ++k) {
    // pixel of register k: (depth + k / K, j + 16 (k % K) + e N/2)
    const int d = depth + k / K;
    if (d >= a.n_z) continue;
    float* dst = base + (size_t)d * N + j + 16 * (k % K) + (N / 2) * e;
#pragma unroll
    for (int i = 0; i < NSUB; ++i) dst[i * plane] = accS[i][k];
#pragma unroll
    for (int q = 0; q < NP; ++q) dst[(NSUB + q) * plane] = accC[q][k];
    if constexpr (COH) {
#pragma unroll
      for (int q = 0; q < 4; ++q) dst[(1 + q) * plane] = accG[q][k];
    }
  }
}

}  // namespace pam

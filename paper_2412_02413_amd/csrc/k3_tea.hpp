// Frequency-domain delay-and-sum fields with the cross-spectra epilogue (FD-TEA-TAX).
//
// The paper's comparison beamformer in its frequency-domain form (Appendix, "PAM with
// DAX and TAX"): the monochromatic field at pixel r is the element spectra advanced by
// their travel times from r,
//     p_i(r, w) = sum_l a_i[l] X_l(w) exp(+i w tau_l(r)),   tau_l(r) = |r - r_l| / c,
// the Fourier transform of the delay-and-sum of Eq. 6 (unit distance weights).  The
// sums over w of |p_i|^2 and Re(p_i^* p_j) then give the NCC, TAX weight and image
// exactly as for the angular-spectrum fields (K4).
//
// Elements sit on grid columns (col0 + step l), so the phasor depends on a pixel column x
// and an element only through x - step l: with x = r + step t (r < step), the pixels of one
// depth and residue r form a Toeplitz product over D = t - l.  Its T + L - 1 phasors are
// made once per (depth, residue, bin) - phase k u in FP64 (u = distance fs / (n_t c), cycles
// per bin index) reduced to [-1/2, 1/2] cycle, hardware sine and cosine - instead of once per
// (pixel, element, bin), and what remains is four FMAs per (pixel, element, bin): the vector
// FMA rate is the bound.
//
// Work split.  A lane holds four consecutive pixels t = 4 q .. 4 q + 3, so four elements
// need seven phasors per lane, three of them left from the four before: four 8-byte LDS reads
// per 64 FMAs.  Elements run in units of eight.  The table is stored as four planes (D mod 4), so that lanes
// of consecutive q read consecutive values.  The element spectra are uniform over the
// workgroup and come through scalar loads; the sub-aperture of a unit is a scalar branch.  A
// wave covers 64 lanes' worth of (depth, residue) rows (several where a row has few pixels,
// part of one where it has more than 256) with its own table, so there is no workgroup
// barrier.  u is kept beside the table in FP64: an FP32 delay would leave phase errors of
// ~2e-5 cycle at 8 MHz.
//
// One frame of 512 x 256 pixels, 128 elements and 768 bins: 7.3 ms with one thread a pixel making every
// (pixel, element, bin) phasor, 1.54 ms here (67 TFLOP/s of the 78.6 of unpacked vector FMAs; spectra and sub-aperture
// sets through vector loads instead of scalar ones: 1.9 ms).  A launch that leaves SIMDs with one wave or none is bound by
// latency instead: 4 frames of 34 x 288 pixels, 190 elements and 13 bins took 182 us (one thread a pixel 148) with every
// unit waiting for its own spectra, code and phasors and 118 with the first two asked for ahead; one of 5 x 224
// zero-stuffed 16.4 -> 12.0 with fewer rows a wave.
#pragma once
#include <algorithm>
#include <type_traits>

#include "kernels.hpp"

namespace pam {

constexpr int TEA_WAVES = 4;       // waves per workgroup
constexpr int TEA_PX = 4;          // pixels per lane

struct TeaArgs {
  const float2* spectra;   // [F][n_sel][L] (K1)
  const int32_t* ksel;     // [n_sel] bin index k on the call's record-length grid
  const int32_t* units;    // [(L + 7) / 8] unit codes
  const double* z;         // [n_z] depths
  float* accum;            // [n_split][F][n_acc][n_z][N]
  double dx;               // grid spacing
  double cyc;              // fs / (n_t c): phase cycles per bin index per metre of path
  int32_t L, N, n_z, n_sel, F, n_split, bins_per_split;
  int32_t n_acc;           // accumulator planes per frame: more than this kernel writes on a plan with pair sums
  int32_t col0, step;      // grid column of element l: col0 + step l
  // the split of a depth's pixels into lanes (tea_shape)
  int32_t T, Q, rows, chunks, PL, n_wg;
};

// T pixels per (depth, residue) row; Q lanes of four pixels a row (at most 64) and `chunks` such pieces a row;
// `rows` rows per wave; PL values per plane of a row's phasor table; n_wg workgroups per frame and bin split.
inline void tea_shape(TeaArgs& a) {
  a.T = (a.N + a.step - 1) / a.step;
  const int q = (a.T + TEA_PX - 1) / TEA_PX;
  a.Q = q < 64 ? q : 64;
  a.chunks = (q + 63) / 64;
  a.rows = 64 / a.Q;
  a.PL = a.Q + 2 * ((a.L + 7) / 8);
  // a launch of less than a wave per SIMD (1,024) packs fewer rows into a wave: each row's table is that wave's own work
  const long long row_waves = (long long)a.n_z * a.step * a.chunks * a.F * a.n_split;
  a.rows = (int)std::max(1ll, std::min((long long)a.rows, row_waves / 1024));
  const long long waves = ((long long)a.n_z * a.step + a.rows - 1) / a.rows * a.chunks;
  a.n_wg = (int)((waves + TEA_WAVES - 1) / TEA_WAVES);
}
// bytes of LDS per workgroup: u (FP64) and the phasors of every wave's rows (at most 48 KiB, 512 elements on 512
// columns)
inline size_t tea_lds(const TeaArgs& a) { return (size_t)TEA_WAVES * a.rows * 4 * a.PL * (sizeof(double) + sizeof(float2)); }

// Element j of four times the four pixels' phasors w[3 + i - j], the seven of them split as lo = w[0..3] and
// hi = w[4..6].
__device__ __forceinline__ void tea_mac(float2 (&p)[TEA_PX], float2 x, int j, const float2 (&lo)[4], const float2 (&hi)[4]) {
#pragma unroll
  for (int i = 0; i < TEA_PX; ++i) {
    const float2 e = 3 + i - j < 4 ? lo[(3 + i - j) & 3] : hi[(3 + i - j) & 3];
    p[i].x = fmaf(x.x, e.x, fmaf(-x.y, e.y, p[i].x));
    p[i].y = fmaf(x.x, e.y, fmaf(x.y, e.x, p[i].y));
  }
}

// The spectra of a unit's eight elements, uniform over the workgroup and read through the scalar cache (the constant
// address space; nothing writes them while the kernel runs).  The last unit of a bin may read up to seven values past
// it: the next bin's, or after the last bin the workspace region that follows the spectra.
typedef float __attribute__((address_space(4))) scalar_float;
typedef int32_t __attribute__((address_space(4))) scalar_int;
__device__ __forceinline__ void tea_load(float (&x)[16], const scalar_float* X) {
#pragma unroll
  for (int j = 0; j < 16; ++j) x[j] = X[j];
}

// Unit codes (tea_unit_code on the host): bits 24 and up name the sub-aperture that alone holds all eight elements, or
// kTeaNone or kTeaMixed; bits 3 j + i say whether element j is in sub-aperture i.  Elements past the last are in none.
constexpr int kTeaNone = 3, kTeaMixed = 4;
inline int tea_unit_code(const int* sets, int n) {    // the sets (bit i: in sub-aperture i) of the unit's n elements
  int code = 0;
  bool same = true;
  for (int j = 0; j < 8; ++j) {
    const int b = j < n ? sets[j] : 0;
    code |= b << (3 * j);
    same = same && b == sets[0];
  }
  const int one = !same ? kTeaMixed : (sets[0] == 0 ? kTeaNone : (sets[0] == 1 ? 0 : (sets[0] == 2 ? 1 : (sets[0] == 4 ? 2 : kTeaMixed))));
  return code | one << 24;
}

// MIXED: some unit belongs to more than one sub-aperture (the plan knows), so the loop has the branch per element
template <int NSUB, bool MIXED>
__global__ __launch_bounds__(64 * TEA_WAVES) void k3_tea(TeaArgs a) {
  constexpr int NP = AccCount<NSUB>::pairs;
  extern __shared__ double lds_tea[];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int bid = blockIdx.x;
  const int sp = bid % a.n_split; bid /= a.n_split;
  const int wg = bid % a.n_wg; bid /= a.n_wg;
  const int f = bid;
  const int b_begin = sp * a.bins_per_split;
  const int b_end = min(a.n_sel, b_begin + a.bins_per_split);
  const int units = (a.L + 7) / 8, entries = 4 * a.PL;              // units of eight elements; phasors of a row
  const scalar_int* codes = (const scalar_int*)a.units;
  const int wave = wg * TEA_WAVES + w, chunk = wave % a.chunks;
  const int row0 = wave / a.chunks * a.rows, n_rows = a.n_z * a.step;   // (depth, residue) rows of this wave
  double* u = lds_tea + (size_t)w * a.rows * entries;
  float2* E = reinterpret_cast<float2*>(lds_tea + (size_t)TEA_WAVES * a.rows * entries) + (size_t)w * a.rows * entries;

  // The scalar loads of a bin's spectra are a serial chain of 64-byte lines that this XCD's L2 has not seen; one vector
  // load a bin, a lane a line, brings the next bin's lines in (up to 512 elements) while this one's products run.
  const auto touch = [&](int b) {
    const size_t line = ((size_t)f * a.n_sel + b) * a.L + min(8 * lane, a.L - 1);
    return b_begin < b_end ? a.spectra[line].x : 0.f;
  };
  const float first = touch(b_begin);

  // plane p, position n of a row: D = 4 n + p - (8 units - 1) + first pixel of the chunk
  for (int s = lane; s < a.rows * entries; s += 64) {
    const int row = row0 + s / entries, e = s % entries;
    const int D = 4 * (e % a.PL) + e / a.PL - (8 * units - 1) + 64 * TEA_PX * chunk;
    const double z = row < n_rows ? a.z[row / a.step] : 0.0;
    const double x = (double)(row % a.step - a.col0 + a.step * D) * a.dx;
    u[s] = sqrt(x * x + z * z) * a.cyc;
  }

  asm volatile("" ::"v"(first));
  const int slot = lane / a.Q;                                      // lanes past the wave's rows repeat row 0
  const bool lane_live = slot < a.rows && row0 + slot < n_rows;
  const int q = lane % a.Q;
  const int t0 = TEA_PX * (64 * chunk + q);
  const float2* Eq = E + (lane_live ? slot : 0) * entries + q;

  float accS[NSUB][TEA_PX], accC[NP > 0 ? NP : 1][TEA_PX];
#pragma unroll
  for (int i = 0; i < TEA_PX; ++i) {
#pragma unroll
    for (int s = 0; s < NSUB; ++s) accS[s][i] = 0.f;
#pragma unroll
    for (int c = 0; c < (NP > 0 ? NP : 1); ++c) accC[c][i] = 0.f;
  }

  for (int b = b_begin; b < b_end; ++b) {
    const double k = (double)a.ksel[b];
    const float ahead = touch(min(b + 1, b_end - 1));
    for (int s = lane; s < a.rows * entries; s += 64) {
      const double ph = k * u[s];
      const float r = (float)(ph - rint(ph));
      E[s] = make_float2(__builtin_amdgcn_cosf(r), __builtin_amdgcn_sinf(r));
    }
    __builtin_amdgcn_wave_barrier();
    const scalar_float* X = (const scalar_float*)(a.spectra + ((size_t)f * a.n_sel + b) * a.L);
    float2 p[NSUB][TEA_PX];
#pragma unroll
    for (int s = 0; s < NSUB; ++s)
#pragma unroll
      for (int i = 0; i < TEA_PX; ++i) p[s][i] = make_float2(0.f, 0.f);
    float x[16], xn[16];                                            // this unit's spectra, the next one's
    tea_load(x, X);
    int code = codes[0], code_n = 0;                                // this unit's code, the next one's
    // mac(j, x_j, lo, hi) for the unit's elements.  The next unit's spectra and code are asked for once this unit's
    // phasors are here: scalar and LDS loads share a counter, so asked for before them, every unit would wait for both.
    auto unit = [&](int un, auto&& mac) {
      const float2* Ep = Eq + 2 * (units - 1 - un);
      float2 e0[4], e1[4], e2[4];                                   // positions q + B, q + B + 1, q + B + 2
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        e0[c] = Ep[c * a.PL];
        e1[c] = Ep[c * a.PL + 1];
        e2[c] = c < 3 ? Ep[c * a.PL + 2] : e1[c];
      }
      mac(0, 0, make_float2(x[0], x[1]), e1, e2);
      __builtin_amdgcn_sched_barrier(0);
      tea_load(xn, X + 16 * min(un + 1, units - 1));
      code_n = codes[min(un + 1, units - 1)];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 1; j < 4; ++j) mac(j, j, make_float2(x[2 * j], x[2 * j + 1]), e1, e2);
#pragma unroll
      for (int j = 0; j < 4; ++j) mac(4 + j, j, make_float2(x[8 + 2 * j], x[8 + 2 * j + 1]), e0, e1);
#pragma unroll
      for (int j = 0; j < 16; ++j) x[j] = xn[j];
    };
    for (int un = 0; un < units;) {
      if (MIXED && (code >> 24) == kTeaMixed) {
        unit(un, [&](int j8, int j, float2 xj, const float2 (&lo)[4], const float2 (&hi)[4]) {
#pragma unroll
          for (int s = 0; s < NSUB; ++s)
            if (code >> (3 * j8 + s) & 1) tea_mac(p[s], xj, j, lo, hi);
        });
        ++un;
        code = code_n;
        continue;
      }
      bool done = false;
#pragma unroll
      for (int s = 0; s < NSUB; ++s)
        if ((code >> 24) == s) {                                    // a run of units that sub-aperture s alone holds
          do {
            unit(un, [&](int, int j, float2 xj, const float2 (&lo)[4], const float2 (&hi)[4]) {
              tea_mac(p[s], xj, j, lo, hi);
            });
            code = code_n;
          } while (++un < units && code >> 24 == s);
          done = true;
        }
      if (!done) {                                                  // no sub-aperture holds any of the eight
        ++un;
        tea_load(x, X + 16 * min(un, units - 1));
        code = codes[min(un, units - 1)];
      }
    }
    __builtin_amdgcn_wave_barrier();                                // the table is free for the next bin
    asm volatile("" ::"v"(ahead));                                  // the touched lines are here by now
#pragma unroll
    for (int i = 0; i < TEA_PX; ++i) {
#pragma unroll
      for (int s = 0; s < NSUB; ++s) accS[s][i] = fmaf(p[s][i].x, p[s][i].x, fmaf(p[s][i].y, p[s][i].y, accS[s][i]));
      if constexpr (NSUB == 3) {
        accC[0][i] = fmaf(p[0][i].x, p[1][i].x, fmaf(p[0][i].y, p[1][i].y, accC[0][i]));
        accC[1][i] = fmaf(p[1][i].x, p[2][i].x, fmaf(p[1][i].y, p[2][i].y, accC[1][i]));
        accC[2][i] = fmaf(p[2][i].x, p[0][i].x, fmaf(p[2][i].y, p[0][i].y, accC[2][i]));
      } else if constexpr (NSUB == 2) {
        accC[0][i] = fmaf(p[0][i].x, p[1][i].x, fmaf(p[0][i].y, p[1][i].y, accC[0][i]));
      }
    }
  }
  if (!lane_live) return;
  const size_t plane = (size_t)a.n_z * a.N;
  const int row = row0 + slot;
  float* dst = a.accum + ((size_t)sp * a.F + f) * a.n_acc * plane + (size_t)(row / a.step) * a.N + row % a.step;
#pragma unroll
  for (int i = 0; i < TEA_PX; ++i) {
    if (t0 + i >= a.T || row % a.step + a.step * (t0 + i) >= a.N) continue;
#pragma unroll
    for (int s = 0; s < NSUB; ++s) dst[s * plane + a.step * (t0 + i)] = accS[s][i];
#pragma unroll
    for (int c = 0; c < NP; ++c) dst[(NSUB + c) * plane + a.step * (t0 + i)] = accC[c][i];
  }
}

// Few elements: one thread a pixel makes its own phasors, with the delays in registers.  A row's table holds 4 PL phasors
// however few pixels and elements the row has, so below some number of elements it costs more than it saves: of
// 4 frames of 151 x 512 pixels and 205 bins, one element zero-stuffed takes 672 us with the table (12 phasors for each
// one-pixel row) and 77 here, two 375 and 99, four 232 and 144; padded (rows of 512 pixels in two tables of 264) two take
// 129 and 99, three 134 and 120; 3 frames of 317 x 384, 205 bins and six elements zero-stuffed 303 and 184.  Timed both
// ways over 176 drawn calls of up to eight elements, this form is 1.05 to 1.65 times as fast where a depth's pixels times
// elements are at most 3.1 of its table phasors and 0.6 to 1.1 beyond 3.3 (calls above 30 us), so the line lies at 3.2;
// seven elements get there at most.
constexpr int kTeaFew = 7;
inline bool tea_few(const TeaArgs& a) {              // (a's shape set)
  return a.L <= kTeaFew && 5ll * a.L * a.N <= 16ll * a.step * a.chunks * 4 * a.PL;
}
template <int NSUB>
__global__ __launch_bounds__(64 * TEA_WAVES) void k3_tea_few(TeaArgs a) {
  constexpr int NP = AccCount<NSUB>::pairs;
  int bid = blockIdx.x;
  const int sp = bid % a.n_split; bid /= a.n_split;
  const int wg = bid % a.n_wg; bid /= a.n_wg;
  const int f = bid;
  const int b_begin = sp * a.bins_per_split;
  const int b_end = min(a.n_sel, b_begin + a.bins_per_split);
  const int n_pix = a.n_z * a.N, pix = wg * 64 * TEA_WAVES + (int)threadIdx.x;
  const int d = min(pix, n_pix - 1) / a.N, j = min(pix, n_pix - 1) - d * a.N;
  const int code = *(const scalar_int*)a.units;                     // membership bits of the one unit
  double u[kTeaFew];
#pragma unroll
  for (int l = 0; l < kTeaFew; ++l) {
    const double x = (double)(j - a.col0 - a.step * l) * a.dx, z = a.z[d];
    u[l] = l < a.L ? sqrt(x * x + z * z) * a.cyc : 0.0;
  }
  float accS[NSUB], accC[NP > 0 ? NP : 1];
#pragma unroll
  for (int s = 0; s < NSUB; ++s) accS[s] = 0.f;
#pragma unroll
  for (int c = 0; c < (NP > 0 ? NP : 1); ++c) accC[c] = 0.f;
  // four bins at a time, so that their spectra are asked for together and their phasors overlap; the rest one by one
  const auto bins = [&](auto count, int b0) {
    constexpr int BC = decltype(count)::value;
    double k[BC];
    const scalar_float* X[BC];
    float2 p[NSUB][BC];
#pragma unroll
    for (int c = 0; c < BC; ++c) {
      k[c] = (double)((const scalar_int*)a.ksel)[b0 + c];
      X[c] = (const scalar_float*)(a.spectra + ((size_t)f * a.n_sel + b0 + c) * a.L);
#pragma unroll
      for (int s = 0; s < NSUB; ++s) p[s][c] = make_float2(0.f, 0.f);
    }
#pragma unroll
    for (int l = 0; l < kTeaFew; ++l) {
      if (l >= a.L) break;
      float2 v[BC];
#pragma unroll
      for (int c = 0; c < BC; ++c) v[c] = make_float2(X[c][2 * l], X[c][2 * l + 1]);
#pragma unroll
      for (int c = 0; c < BC; ++c) {
        const double ph = k[c] * u[l];
        const float r = (float)(ph - rint(ph));
        v[c] = cmul(v[c], make_float2(__builtin_amdgcn_cosf(r), __builtin_amdgcn_sinf(r)));
      }
#pragma unroll
      for (int s = 0; s < NSUB; ++s)
        if (code >> (3 * l + s) & 1)
#pragma unroll
          for (int c = 0; c < BC; ++c) p[s][c] = cadd(p[s][c], v[c]);
    }
#pragma unroll
    for (int c = 0; c < BC; ++c) {
#pragma unroll
      for (int s = 0; s < NSUB; ++s) accS[s] = fmaf(p[s][c].x, p[s][c].x, fmaf(p[s][c].y, p[s][c].y, accS[s]));
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        const float2 v = p[q][c], w = p[NSUB == 3 ? (q + 1) % 3 : NSUB - 1][c];
        accC[q] = fmaf(v.x, w.x, fmaf(v.y, w.y, accC[q]));
      }
    }
  };
  int b = b_begin;
  for (; b + 4 <= b_end; b += 4) bins(std::integral_constant<int, 4>(), b);
  for (; b < b_end; ++b) bins(std::integral_constant<int, 1>(), b);
  if (pix >= n_pix) return;
  float* dst = a.accum + ((size_t)sp * a.F + f) * a.n_acc * n_pix + pix;
#pragma unroll
  for (int s = 0; s < NSUB; ++s) dst[(size_t)s * n_pix] = accS[s];
#pragma unroll
  for (int c = 0; c < NP; ++c) dst[(size_t)(NSUB + c) * n_pix] = accC[c];
}

}  // namespace pam

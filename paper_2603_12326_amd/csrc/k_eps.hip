// FP64 dielectric matrix, its inverse diagonal and the loss (Eq. eps_LFE,
// Eq. eps_noLFE).
//
// eps_GG' = delta_GG' - v_G v_G' chi0_GG' with v_G = sqrt(4 pi)/|q+G| (the
// symmetrised Coulomb factor of Eq. RPA).  [eps^-1]_GG for every G comes from
// an in-place Gauss-Jordan inversion with partial pivoting on column moduli
// |re| + |im|.  Rows are not swapped: step k picks pivot row p_k among the rows
// not yet used, and at the end [eps^-1]_kk = B[p_k][k'] where k' is the step at
// which row k served as pivot.
#include <limits.h>

#include <algorithm>
#include <utility>

#include "common.h"

namespace qcx {

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

// Upper-triangle pair index p -> (G, G'), G <= G', row-major.  Row g starts
// at s(g) = g n - g (g - 1) / 2; the quadratic is inverted in double and the
// rounding fixed by at most a step either way.
__device__ inline void pair_decode(int p, int n_g, int& G, int& Gp) {
  auto start = [&](long gg) { return gg * n_g - gg * (gg - 1) / 2; };
  const double b = 2.0 * n_g + 1.0;
  int g = (int)floor(0.5 * (b - sqrt(fmax(b * b - 8.0 * p, 0.0))));
  g = max(0, min(g, n_g - 1));
  while (g > 0 && start(g) > p) --g;
  while (g + 1 < n_g && start(g + 1) <= p) ++g;
  G = g;
  Gp = g + (int)(p - start(g));
}

// mode 0: eps; mode 1: chi0
__global__ void k_assemble(AsmArgs a, Chi0Geom g, int mode, cplx* __restrict__ out) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long)g.n_w * g.n_pairs) return;
  const int j = (int)(i / g.n_pairs), p = (int)(i % g.n_pairs);
  int G, Gp;
  pair_decode(p, g.n_g, G, Gp);
  double Xr = 0.0, Xi = 0.0, Yr = 0.0, Yi = 0.0;
  if (p < a.n_pairs64) {
    for (int ks = 0; ks < a.ks64; ++ks) {
      const double* x0 = a.XY + ((size_t)ks * a.n_rowsp64 + 2 * j) * a.n_colp64 + 2 * p;
      const double* x1 = x0 + a.n_colp64;
      Xr += x0[0];
      Xi += x0[1];
      Yr += x1[0];
      Yi += x1[1];
    }
  } else if (a.C64) {
    const int b = p - g.p0;
    const size_t r0 = (size_t)(2 * j) * 2, r1 = r0 + 2;
    Xr = a.C64[(r0 + 0) * g.n_bulkp + b];
    Xi = a.C64[(r0 + 1) * g.n_bulkp + b];
    Yr = a.C64[(r1 + 0) * g.n_bulkp + b];
    Yi = a.C64[(r1 + 1) * g.n_bulkp + b];
  } else {
    const int b = p - g.p0;
    for (int ks = 0; ks < a.ks; ++ks) {
      const size_t r0 = ((size_t)ks * g.n_rowsp + 2 * j) * 2;  // row 2j: Re W
      const size_t r1 = r0 + 2;                                 // row 2j+1: Im W
      Xr += (double)a.C[(r0 + 0) * g.n_bulkp + b];
      Xi += (double)a.C[(r0 + 1) * g.n_bulkp + b];
      Yr += (double)a.C[(r1 + 0) * g.n_bulkp + b];
      Yi += (double)a.C[(r1 + 1) * g.n_bulkp + b];
    }
  }
  if (G == Gp) {  // P_t(G, G) = |R_t(G)|^2 is real
    Xi = 0.0;
    Yi = 0.0;
  }
  cplx cab = {a.pref * (Xr - Yi), a.pref * (Xi + Yr)};  // chi0_{G G'}
  cplx cba = {a.pref * (Xr + Yi), a.pref * (Yr - Xi)};  // chi0_{G' G}
  const size_t base = (size_t)j * g.n_g * g.n_g;
  if (mode == 0) {
    const double vv = a.vq[G] * a.vq[Gp];
    cab = {(G == Gp ? 1.0 : 0.0) - vv * cab.re, -vv * cab.im};
    cba = {(G == Gp ? 1.0 : 0.0) - vv * cba.re, -vv * cba.im};
  }
  out[base + (size_t)G * g.n_g + Gp] = cab;
  if (G != Gp) out[base + (size_t)Gp * g.n_g + G] = cba;
}

// 1/a = conj(a) / |a|^2 with a first scaled by the binary exponent of
// max(|re|, |im|) (exact), so that |a|^2 neither underflows nor overflows for
// any finite nonzero a; zero and non-finite a take the plain formula (they
// are reported as singular pivots).
__device__ inline cplx cinv(cplx a) {
  const double s = fmax(fabs(a.re), fabs(a.im));
  if (!(s > 0.0 && s < INFINITY)) {
    const double d = 1.0 / (a.re * a.re + a.im * a.im);
    return {a.re * d, -a.im * d};
  }
  int e;
  (void)frexp(s, &e);
  const double x = ldexp(a.re, -e), y = ldexp(a.im, -e);
  const double d = 1.0 / (x * x + y * y);
  return {ldexp(x * d, -e), ldexp(-y * d, -e)};
}

// A pivot of modulus zero, or a non-finite one (NaN or infinite entries, e.g.
// eta = 0 with w on a transition energy), makes the matrix count as singular.
__device__ inline bool bad_pivot(cplx v) {
  const double m = fabs(v.re) + fabs(v.im);
  return !(m > 0.0 && m < INFINITY);
}

// An empty asm statement makes x opaque, so that choosing one element of a
// register array by a run-time index (a == pa, b == jt / 16) stays a choice
// between values instead of becoming an indexed load that would move the
// whole array to scratch memory.
__device__ inline cplx opaque(cplx x) {
  asm volatile("" : "+v"(x.re), "+v"(x.im));
  return x;
}

__device__ inline double readlane_d(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), lane);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Element pa (wave-uniform) of a per-lane register array, as held by lane pl:
// one scalar branch per slot, so that only the readlanes of slot pa run and
// they read the registers in place (no VALU copy of the chosen element).
template <int RP>
__device__ inline cplx readlane_slot(const cplx (&c)[RP], int pa, int pl) {
  cplx r = {0.0, 0.0};
#pragma unroll
  for (int a = 0; a < RP; ++a)
    if (a == pa) r = {readlane_d(c[a].re, pl), readlane_d(c[a].im, pl)};
  return r;
}

// Maximum of a 32-bit value over the wave: DPP butterflies inside each row of
// 16 lanes, then the four row results by readlane.  Needs every lane active.
__device__ inline unsigned wave_max_u32(unsigned x) {
  auto step = [&](auto ctrl) {
    constexpr int c = decltype(ctrl)::value;
    const unsigned o = (unsigned)__builtin_amdgcn_update_dpp((int)x, (int)x, c, 0xF, 0xF, false);
    x = o > x ? o : x;
  };
  step(std::integral_constant<int, 0xB1>{});   // quad_perm [1,0,3,2]
  step(std::integral_constant<int, 0x4E>{});   // quad_perm [2,3,0,1]
  step(std::integral_constant<int, 0x141>{});  // row_half_mirror
  step(std::integral_constant<int, 0x140>{});  // row_mirror
  unsigned r = 0u;
#pragma unroll
  for (int row = 0; row < 4; ++row) {
    const unsigned o = (unsigned)__builtin_amdgcn_readlane((int)x, 16 * row);
    r = o > r ? o : r;
  }
  return r;
}

// 1/a as cinv, with 1/|a|^2 of the scaled a (in [1/4, 2)) from a
// single-precision estimate refined by two Newton steps in FP64 (24 -> 48 ->
// 96 bits: within an ulp of the FP64 reciprocal), a shorter chain of
// dependent instructions than the IEEE division.
__device__ inline cplx cinv_nr(cplx a) {
  const double s = fmax(fabs(a.re), fabs(a.im));
  if (!(s > 0.0 && s < INFINITY)) {
    const double d = 1.0 / (a.re * a.re + a.im * a.im);
    return {a.re * d, -a.im * d};
  }
  int e;
  (void)frexp(s, &e);
  const double x = ldexp(a.re, -e), y = ldexp(a.im, -e);
  const double d = x * x + y * y;
  double r = (double)__builtin_amdgcn_rcpf((float)d);
  r = fma(r, fma(-d, r, 1.0), r);
  r = fma(r, fma(-d, r, 1.0), r);
  return {ldexp(x * r, -e), ldexp(-y * r, -e)};
}

// 1/a by |a|^2 and the hardware reciprocal refined by two Newton steps where
// |a|^2 is far from the ends of the range, cinv_nr elsewhere.
__device__ inline cplx cinv_pivot(cplx a) {
  const double d = fma(a.re, a.re, a.im * a.im);
  if (!(d > 0x1p-900 && d < 0x1p900)) return cinv_nr(a);
  double r = __builtin_amdgcn_rcp(d);
  r = fma(r, fma(-d, r, 1.0), r);
  r = fma(r, fma(-d, r, 1.0), r);
  return {a.re * r, -a.im * r};
}

// The pivot of a column c (row l + 64 a in slot a of lane l): the live row
// (bit a of live) of largest modulus |re| + |im| to 8 mantissa bits, then the
// smaller row; a NaN counts above infinity.  Each lane keeps its best element,
// so the pivot is read from lane p % 64 without a look at its slot.  Writes
// u_i = (c_i - [i == p]) / piv to uc[64 RP] and returns p; wk = piv + 1.
template <int RP>
__device__ __forceinline__ int gj_choose(const cplx (&c)[RP], unsigned live, int l, cplx* uc, cplx& wk,
                                         bool& singular) {
  unsigned best = 0u;
  cplx bv = {0.0, 0.0};
#pragma unroll
  for (int a = 0; a < RP; ++a) {
    const double mag = fabs(c[a].re) + fabs(c[a].im);
    const unsigned hi = (unsigned)((unsigned long long)__double_as_longlong(mag) >> 32);
    const unsigned on = (unsigned)__builtin_amdgcn_sbfe((int)live, a, 1);
    const unsigned key = ((hi & 0x7FFFF000u) | (unsigned)(0xFFF - (l + 64 * a))) & on;
    const bool g = key > best;
    best = g ? key : best;
    bv.re = g ? c[a].re : bv.re;
    bv.im = g ? c[a].im : bv.im;
  }
  best = wave_max_u32(best);
  const int p = __builtin_amdgcn_readfirstlane(0xFFF - (int)(best & 0xFFFu));
  const cplx pv = {readlane_d(bv.re, p & 63), readlane_d(bv.im, p & 63)};
  const cplx inv = cinv_pivot(pv);
#pragma unroll
  for (int a = 0; a < RP; ++a) {
    const int i = l + 64 * a;
    cplx x = c[a];
    x.re -= i == p ? 1.0 : 0.0;
    uc[i] = cmul(x, inv);
  }
  if (bad_pivot(pv)) singular = true;
  wk = {pv.re + 1.0, pv.im};
  return p;
}

// Register-resident Gauss-Jordan for n <= 64 RP and n <= 16 CP with 16 waves:
// lane l of wave v owns rows l + 64 a and columns v + 16 b, so column k lives
// in wave k % 16 alone.  Step k applies m <- m - u w^T with the pivot folded
// into u: u_i = c_i / piv (u_p = (piv - 1) / piv) and w = row p as it stands
// except w_k = piv + 1, where c = column k and piv = m[p][k].  This is the
// Gauss-Jordan sweep (row p / piv, column k -c / piv, pivot 1 / piv, the rest
// m - c row_p / piv) with no per-element fix-ups.
//
// One barrier per step.  Between two barriers the wave that owns column k + 1
// runs the chain that bounds the step: read p and u, update column k + 1,
// choose its pivot and publish u and p through LDS (gj_choose).  It runs that
// chain before any of its other columns, while the other waves do their FMAs.
// Every wave then reads row p of its columns from lane p % 64 with readlane (scalar registers, no LDS
// traffic: the LDS pipe is shared by all 16 waves); the row slot p / 64 is
// dispatched once per step by a scalar branch, so the readlanes take the
// registers in place instead of a VALU copy of the chosen slot.  u and p are
// double-buffered by the parity of k; u is zero past row n; used-row marks
// live in registers.
// What bounds it is the issue of the FMAs and readlanes (1.5 us per step at
// n = 113, 0.66 us with the chain alone).
// Body of one 1024-thread block: matrix A (n x n, only read), diagonal of the
// inverse into drow[n]; a zero pivot sets *sing to at most widx.
template <int RP, int CP>
__device__ __forceinline__ void gj_reg_body(const cplx* __restrict__ A, int n,
                                            cplx* __restrict__ drow, int* sing, int widx) {
  constexpr int NW = 16;
  __shared__ cplx ucol[2][64 * RP];
  __shared__ int prow[2], sor[64 * RP];
  const int tid = threadIdx.x, l = tid & 63;
  const int v = __builtin_amdgcn_readfirstlane(tid >> 6);
  cplx m[RP][CP];
#pragma unroll
  for (int a = 0; a < RP; ++a)
#pragma unroll
    for (int b = 0; b < CP; ++b) {
      const int i = l + 64 * a, j = v + NW * b;
      m[a][b] = (i < n && j < n) ? A[(size_t)i * n + j] : cplx{0.0, 0.0};
    }
  for (int e = tid; e < 2 * 64 * RP; e += 1024) (&ucol[0][0])[e] = {0.0, 0.0};
  __syncthreads();
  unsigned live = 0;       // bit a: row l + 64 a has not served as a pivot yet
#pragma unroll
  for (int a = 0; a < RP; ++a) live |= l + 64 * a < n ? 1u << a : 0u;
  bool singular = false;
  cplx wk = {0.0, 0.0};    // piv + 1 of the column this wave owns next

  // Owner wave of column kc (current values c): choose the pivot, publish u
  // into buffer pb, p and sor[p].
  auto choose = [&](const cplx (&c)[RP], int kc, int pb) __attribute__((always_inline)) {
    const int p = gj_choose<RP>(c, live, l, ucol[pb], wk, singular);
    if (l == 0) {
      prow[pb] = p;
      sor[p] = kc;
    }
  };

  if (v == 0) {
    cplx c[RP];
#pragma unroll
    for (int a = 0; a < RP; ++a) c[a] = m[a][0];
    choose(c, 0, 0);
  }
  // Step k = 16 kb + kk; with kb, t and the row slot unrolled every register
  // index is static.  The owner of column k + 1 (slot kb, or kb + 1 when
  // kk = 15) updates it and chooses before its other columns.
#pragma unroll
  for (int kb = 0; kb < CP; ++kb) {
    for (int kk = 0; kk < NW; ++kk) {
      const int k = NW * kb + kk;
      if (k >= n) break;
      const int par = k & 1;
      // the owner of column k + 1 runs at raised wave priority until it has
      // published, so that its chain is issued ahead of the other waves' FMAs
      if (v == (k + 1) % NW) __builtin_amdgcn_s_setprio(3);
      __syncthreads();  // u, p of column k published
      const int p = __builtin_amdgcn_readfirstlane(prow[par]);
      const int pl = p & 63, pa = p >> 6;
      cplx u[RP];
#pragma unroll
      for (int a = 0; a < RP; ++a) u[a] = ucol[par][l + 64 * a];
      if (l == pl) live &= ~(1u << pa);
      const int k1 = k + 1;
      const bool owner1 = k1 < n && v == k1 % NW;  // owns column k + 1
      const bool next = kk == NW - 1;               // column k + 1 in slot kb + 1
      // m[.][b] -= u w^T for one column
      auto update = [&](int b, cplx w) __attribute__((always_inline)) {
#pragma unroll
        for (int a = 0; a < RP; ++a) {
          m[a][b].re = fma(-u[a].re, w.re, m[a][b].re);
          m[a][b].re = fma(u[a].im, w.im, m[a][b].re);
          m[a][b].im = fma(-u[a].re, w.im, m[a][b].im);
          m[a][b].im = fma(-u[a].im, w.re, m[a][b].im);
        }
      };
      if (owner1) {
        auto update_choose = [&](int b) __attribute__((always_inline)) {
          cplx c[RP];
#pragma unroll
          for (int a = 0; a < RP; ++a) c[a] = m[a][b];
          update(b, readlane_slot<RP>(c, pa, pl));  // column k + 1 is never column k
#pragma unroll
          for (int a = 0; a < RP; ++a) c[a] = m[a][b];
          choose(c, k1, par ^ 1);
        };
        if (!next)
          update_choose(kb);
        else
          update_choose(kb + 1 < CP ? kb + 1 : CP - 1);  // k1 < n keeps kb + 1 < CP
      }
      __builtin_amdgcn_s_setprio(0);
      cplx wr[CP];  // row p of this wave's columns (lane pl), wave-uniform
      // pa is wave-uniform: one scalar branch per row slot, and inside it
      // the readlanes take the registers in place (no VALU copies)
#pragma unroll
      for (int a = 0; a < RP; ++a)
        if (a == pa) {
#pragma unroll
          for (int b = 0; b < CP; ++b) wr[b] = {readlane_d(m[a][b].re, pl), readlane_d(m[a][b].im, pl)};
        }
      if (v == kk) wr[kb] = wk;  // owner of column k: w_k = piv + 1
#pragma unroll
      for (int t = 0; t < CP; ++t) {
        const int b = (kb + t) % CP;
        const bool done = owner1 && ((t == 0 && !next) || (t == 1 && next));
        if (v + NW * b < n && !done) update(b, wr[b]);
      }
    }
  }
  __syncthreads();
  // [eps^-1]_kk sits at row piv[k] (the row whose sor is k) and column sor[k]
#pragma unroll
  for (int a = 0; a < RP; ++a) {
    const int i = l + 64 * a;
    if (i >= n) continue;
    const int k = sor[i], jt = sor[k];
    if (jt % NW != v) continue;
#pragma unroll
    for (int b = 0; b < CP; ++b)
      if (b == jt / NW) drow[k] = opaque(m[a][b]);
  }
  if (singular) atomicMin(sing, widx);
}

// Blocked Gauss-Jordan over several workgroups per matrix for n > 128; the
// matrix stays in global memory and is swept in panels of MB columns.  One
// workgroup per matrix left most of the chip idle below 256 matrices, and its
// updates waited on one L2 round trip after the other (n = 259, 175 matrices:
// 0.5 ms of pivot steps, 1.3 ms of updates).  With a block per column tile the
// updates fill the chip and the pivot steps, 1.9 us each (instruction issue of
// the 16 waves of a sweep), bound it: 175 matrices of 259 1.09 ms (1.89 before),
// 44 0.58 (1.72), 875 6.7 (9.7); 500 x 128 5.4 (11.6); 749 x 512 75 (87);
// 953 x 16 6.4 (63), 953 x 256 76 (93).
//
// T[:, j] += Z Y[:, j] on the tile of MB columns j = jt .., by one block of NT
// threads: Z = swept panel k0 .. with 1 subtracted at (p_a, a), Y the panel's
// pivot rows before the update (staged in y).  FP64 MFMA on 16 x 16 blocks,
// Re T += Re Z Re Y - Im Z Im Y, Im T += Re Z Im Y + Im Z Re Y; each wave takes
// its Z fragments and its T block straight from L2 into registers.
// MFMA layouts: A 16x4, lane l holds A[l%16][l/16]; B 4x16, lane l holds
// B[l/16][l%16]; D 16x16, lane l holds D[4r + l/16][l%16], r = 0..3.
// The pivot record of a matrix is S[4 k] = pivot row of step k, S[4 i + 1] =
// step of pivot row i (-1: none yet), kept where its diagonal will go.
template <int MB, int NT>
__device__ __forceinline__ void gj_update(cplx* y, int* piv, const cplx* src, cplx* A, int n, const int* S,
                                          int k0, int jt) {
  constexpr int CT = MB / 16;
  const int tid = threadIdx.x, l = tid & 63, li = l & 15, lk = l >> 4;
  const int v = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int mb = min(MB, n - k0);
  const cplx* T = k0 ? A : src;
  for (int e = tid; e < MB * MB; e += NT) {
    const int a = e / MB, j = jt + e % MB;
    const int pa = a < mb ? S[4 * (k0 + a)] : -1;
    y[e] = (a < mb && j < n) ? T[(size_t)pa * n + j] : cplx{0.0, 0.0};
    if (e % MB == 0) piv[a] = pa;
  }
  __syncthreads();
  const int n_u = (n + 15) / 16 * CT;
  for (int u = v; u < n_u; u += NT / 64) {
    const int i0 = u / CT * 16, c0 = u % CT * 16, j = jt + c0 + li;
    cplx z[MB / 4];
#pragma unroll
    for (int s = 0; s < MB / 4; ++s) {
      const int a = 4 * s + lk, i = i0 + li;
      z[s] = (i < n && a < mb) ? A[(size_t)i * n + k0 + a] : cplx{0.0, 0.0};
    }
    cplx t[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = i0 + 4 * r + lk;
      t[r] = (i < n && j < n) ? T[(size_t)i * n + j] : cplx{0.0, 0.0};
    }
    f64x4 re = {0.0, 0.0, 0.0, 0.0}, im = re;  // T is added once, at the end
#pragma unroll
    for (int s = 0; s < MB / 4; ++s) {
      const int a = 4 * s + lk;
      const cplx b = y[a * MB + c0 + li];
      if (piv[a] == i0 + li) z[s].re -= 1.0;
      re = __builtin_amdgcn_mfma_f64_16x16x4f64(z[s].re, b.re, re, 0, 0, 0);
      im = __builtin_amdgcn_mfma_f64_16x16x4f64(z[s].re, b.im, im, 0, 0, 0);
      re = __builtin_amdgcn_mfma_f64_16x16x4f64(-z[s].im, b.im, re, 0, 0, 0);
      im = __builtin_amdgcn_mfma_f64_16x16x4f64(z[s].im, b.re, im, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = i0 + 4 * r + lk;
      if (i < n && j < n) A[(size_t)i * n + j] = cplx{t[r].re + re[r], t[r].im + im[r]};
    }
  }
}

template <int RP, int CP, int NW>
struct GjTile {
  static constexpr int MB = NW * CP, NT = 64 * NW;
  struct Lds {
    cplx y[MB * MB];
    cplx ucol[2][64 * RP];
    int piv[MB];
    int prow[2];
  };

  // The pivot steps of panel s0 .. on its own columns (column s0 + NW b + v in
  // slot b of wave v, row l + 64 a in lane l), steps as in gj_reg_body.
  static __device__ __forceinline__ void sweep(Lds& L, const cplx* src, cplx* A, int n,
                                               int* S, int s0, int* sing, int widx) {
    const int tid = threadIdx.x, l = tid & 63;
    const int v = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ms = min(MB, n - s0);
    const cplx* T = s0 ? A : src;
    unsigned live = 0;
    bool singular = false;
    cplx wk = {0.0, 0.0};
    if (s0 == 0)
      for (int i = tid; i < n; i += NT) S[4 * i + 1] = -1;
#pragma unroll
    for (int a = 0; a < RP; ++a) {
      const int i = l + 64 * a;
      if (i < n && (s0 == 0 || S[4 * i + 1] < 0)) live |= 1u << a;
    }
    cplx m[RP][CP];
#pragma unroll
    for (int b = 0; b < CP; ++b)
#pragma unroll
      for (int a = 0; a < RP; ++a) {
        const int i = l + 64 * a, c = v + NW * b;
        m[a][b] = (i < n && c < ms) ? T[(size_t)i * n + s0 + c] : cplx{0.0, 0.0};
      }
    for (int e = tid; e < 2 * 64 * RP; e += NT) (&L.ucol[0][0])[e] = {0.0, 0.0};
    __syncthreads();
    auto choose = [&](const cplx (&c)[RP], int kc, int pb) __attribute__((always_inline)) {
      const int p = gj_choose<RP>(c, live, l, L.ucol[pb], wk, singular);
      if (l == 0) {
        L.prow[pb] = p;
        L.piv[kc] = p;  // the record in S after the sweep: no global store waits at a barrier
      }
    };
    if (v == 0) {
      cplx c[RP];
#pragma unroll
      for (int a = 0; a < RP; ++a) c[a] = m[a][0];
      choose(c, 0, 0);
    }
#pragma unroll
    for (int kb = 0; kb < CP; ++kb) {
      for (int kk = 0; kk < NW; ++kk) {
        const int k = NW * kb + kk;
        if (k >= ms) break;
        const int par = k & 1;
        if (v == (k + 1) % NW) __builtin_amdgcn_s_setprio(3);
        __syncthreads();  // u, p of step k published
        const int p = __builtin_amdgcn_readfirstlane(L.prow[par]);
        const int pl = p & 63, pa = p >> 6;
        if (l == pl) live &= ~(1u << pa);
        // Row p of this wave's columns, wave-uniform, by one scalar branch on its
        // slot, and u read once for all of them (the LDS pipe is shared by every
        // wave): 259 x 44 matrices 633 -> 576 us, 953 x 16 10.1 -> 6.4 ms.  Not
        // where it spills (eight row slots: 500 x 128 5.4 -> 5.8 ms) or where the
        // unrolled columns outgrow the instruction cache (CP = 4: 1.09 -> 1.12).
        constexpr bool ONCE = CP < 4 && RP != 8;
        const cplx w0 = wk;  // owner of column k: w_k = piv + 1
        cplx wr[CP];
        auto row = [&](int b) __attribute__((always_inline)) {
          cplx c[RP];
#pragma unroll
          for (int a = 0; a < RP; ++a) c[a] = m[a][b];
          wr[b] = readlane_slot<RP>(c, pa, pl);
        };
        if constexpr (ONCE) {
#pragma unroll
          for (int a = 0; a < RP; ++a)
            if (a == pa) {
#pragma unroll
              for (int b = 0; b < CP; ++b) wr[b] = {readlane_d(m[a][b].re, pl), readlane_d(m[a][b].im, pl)};
            }
          if (v == kk) wr[kb] = w0;
        }
        auto axpy = [&](int a, int b, cplx u) __attribute__((always_inline)) {
          m[a][b].re = fma(-u.re, wr[b].re, m[a][b].re);
          m[a][b].re = fma(u.im, wr[b].im, m[a][b].re);
          m[a][b].im = fma(-u.re, wr[b].im, m[a][b].im);
          m[a][b].im = fma(-u.im, wr[b].re, m[a][b].im);
        };
        auto column = [&](int b) __attribute__((always_inline)) {
#pragma unroll
          for (int a = 0; a < RP; ++a) axpy(a, b, L.ucol[par][l + 64 * a]);
        };
        auto step1 = [&](int b) __attribute__((always_inline)) {
          if constexpr (!ONCE) row(b);
          column(b);
          cplx c[RP];
#pragma unroll
          for (int a = 0; a < RP; ++a) c[a] = m[a][b];
          choose(c, k + 1, par ^ 1);
          if constexpr (ONCE) wr[b] = {0.0, 0.0};  // done
        };
        const bool next = kk == NW - 1, owner1 = k + 1 < ms && v == (k + 1) % NW;
        if (owner1) {
          if (!next)
            step1(kb);
          else
            step1(kb + 1 < CP ? kb + 1 : CP - 1);  // k + 1 < ms keeps kb + 1 < CP
        }
        __builtin_amdgcn_s_setprio(0);
        if constexpr (ONCE) {
#pragma unroll
          for (int a = 0; a < RP; ++a) {
            const cplx u = L.ucol[par][l + 64 * a];
#pragma unroll
            for (int b = 0; b < CP; ++b) axpy(a, b, u);
          }
        } else {
#pragma unroll
          for (int b = 0; b < CP; ++b) {
            if (owner1 && b == (next ? kb + 1 : kb)) continue;  // done
            if (v == kk && b == kb)
              wr[b] = w0;
            else
              row(b);
            column(b);
          }
        }
      }
    }
#pragma unroll
    for (int b = 0; b < CP; ++b)
#pragma unroll
      for (int a = 0; a < RP; ++a) {
        const int i = l + 64 * a, c = v + NW * b;
        if (i < n && c < ms) A[(size_t)i * n + s0 + c] = m[a][b];
      }
    if (tid < ms) {
      S[4 * (s0 + tid)] = L.piv[tid];
      S[4 * L.piv[tid] + 1] = s0 + tid;
    }
    if (singular) atomicMin(sing, widx);
  }

  // Block y of a matrix in launch p (-1: the first sweep only).  Launch p gives
  // every other column tile its update by panel p, one block per tile, and the
  // block of tile p + 1 then sweeps its columns, the next panel: one launch per
  // panel in a matrix's chain.
  static __device__ __forceinline__ void run(const cplx* src, cplx* A, int n, cplx* drow,
                                             int* sing, int widx, int p, int y) {
    __shared__ Lds L;
    const int n_t = (n + MB - 1) / MB;
    int* S = reinterpret_cast<int*>(drow);
    if (p >= n_t) return;
    if (y > (p < 0 ? 0 : n_t - 2)) return;
    const int t = p + 1 + y < n_t ? p + 1 + y : p + 1 + y - n_t;  // the next panel's tile first
    if (p >= 0) {
      gj_update<MB, NT>(L.y, L.piv, src, A, n, S, MB * p, MB * t);
      if (t != p + 1) return;
      __syncthreads();  // the tile's columns in memory
    }
    sweep(L, src, A, n, S, MB * (p + 1), sing, widx);
  }
};

// The panel of 2 MB columns k0 .. by one block: its two halves swept in turn,
// each half's update given to the other, so that it holds what 2 MB single
// steps leave there.
template <int RP, int CP, int NW>
__device__ __forceinline__ void gj_panel2(const cplx* src, cplx* A, int n, cplx* drow, int* sing, int widx,
                                          int k0) {
  using G = GjTile<RP, CP, NW>;
  __shared__ typename G::Lds L;
  int* S = reinterpret_cast<int*>(drow);
  if (k0 >= n) return;
  G::sweep(L, src, A, n, S, k0, sing, widx);
  if (k0 + G::MB >= n) return;
  __syncthreads();  // the first half and its pivots in memory
  gj_update<G::MB, G::NT>(L.y, L.piv, src, A, n, S, k0, k0 + G::MB);
  __syncthreads();
  G::sweep(L, src, A, n, S, k0 + G::MB, sing, widx);
  __syncthreads();
  gj_update<G::MB, G::NT>(L.y, L.piv, A, A, n, S, k0 + G::MB, k0);
}

// diag of the inverse from the swept matrix: [eps^-1]_kk sits at row piv[k],
// column sor[k]; the pivot record in the diagonal's own storage is replaced
__device__ __forceinline__ void gj_gather(const cplx* A, int n, cplx* drow) {
  __shared__ int ps[2 * 1024];
  const int* S = reinterpret_cast<const int*>(drow);
  for (int k = threadIdx.x; k < n; k += blockDim.x) {
    ps[2 * k] = S[4 * k];
    ps[2 * k + 1] = S[4 * k + 1];
  }
  __syncthreads();
  for (int k = threadIdx.x; k < n; k += blockDim.x) drow[k] = A[(size_t)ps[2 * k] * n + ps[2 * k + 1]];
}

template <int RP, int CP>
__global__ void __launch_bounds__(1024) k_gj_reg(const cplx* __restrict__ eps, int n,
                                                 cplx* __restrict__ diag, int* sing, int w_base) {
  gj_reg_body<RP, CP>(eps + (size_t)blockIdx.x * n * n, n, diag + (size_t)blockIdx.x * n, sing,
                      w_base + (int)blockIdx.x);
}

// The job of a block in a multi-item launch: blocks [block0, block0 +
// n_w) of a launch belong to job j (jobs sorted by block0).
__device__ inline GjJob find_job(const GjJob* __restrict__ jobs, int n_jobs, int block, int& w) {
  int j = 0;
  while (j + 1 < n_jobs && block >= jobs[j + 1].block0) ++j;
  w = block - jobs[j].block0;
  return jobs[j];
}

template <int RP, int CP>
__global__ void __launch_bounds__(1024) k_gj_reg_jobs(const GjJob* __restrict__ jobs, int n_jobs) {
  int w;
  const GjJob J = find_job(jobs, n_jobs, blockIdx.x, w);
  gj_reg_body<RP, CP>(J.eps + (size_t)w * J.n * J.n, J.n, J.diag + (size_t)w * J.n, J.sing, w);
}

// launch of panel p over n_w matrices (grid x, rounded up to 8 so that the
// blocks of a matrix share an XCD) and their tiles (grid y)
template <int RP, int CP, int NW>
__global__ void __launch_bounds__(64 * NW) k_gj_tile(const cplx* src, cplx* A, int n, int n_w,
                                                     cplx* diag, int* sing, int w_base, int p) {
  const int w = blockIdx.x;
  if (w >= n_w) return;
  GjTile<RP, CP, NW>::run(src + (size_t)w * n * n, A + (size_t)w * n * n, n, diag + (size_t)w * n,
                          sing, w_base + w, p, blockIdx.y);
}

template <int RP, int CP, int NW>
__global__ void __launch_bounds__(64 * NW) k_gj_tile_jobs(const GjJob* __restrict__ jobs, int n_jobs,
                                                          int n_blocks, int p) {
  if ((int)blockIdx.x >= n_blocks) return;
  int w;
  const GjJob J = find_job(jobs, n_jobs, blockIdx.x, w);
  cplx* A = J.eps + (size_t)w * J.n * J.n;
  GjTile<RP, CP, NW>::run(A, A, J.n, J.diag + (size_t)w * J.n, J.sing, w, p, blockIdx.y);
}

// The two launches per panel where the chip is full of matrices: their panels,
// then the updates of every other tile by small blocks, those of a matrix
// neighbours on one XCD (its Z stays in that L2).
template <int RP>
__global__ void __launch_bounds__(1024) k_gj_panel2(const cplx* src, cplx* A, int n, cplx* diag, int* sing,
                                                    int w_base, int k0) {
  const size_t w = blockIdx.x;
  gj_panel2<RP, 1, 16>(src + w * n * n, A + w * n * n, n, diag + w * n, sing, w_base + (int)w, k0);
}

template <int RP>
__global__ void __launch_bounds__(1024) k_gj_panel2_jobs(const GjJob* __restrict__ jobs, int n_jobs, int k0) {
  int w;
  const GjJob J = find_job(jobs, n_jobs, blockIdx.x, w);
  cplx* A = J.eps + (size_t)w * J.n * J.n;
  gj_panel2<RP, 1, 16>(A, A, J.n, J.diag + (size_t)w * J.n, J.sing, w, k0);
}

__device__ __forceinline__ bool gj_tile_of(int n_t, int n_w, int p, int& w, int& t) {
  const int r = blockIdx.x / 8;
  w = r / (n_t - 1) * 8 + blockIdx.x % 8;
  t = r % (n_t - 1);
  t += t >= p;
  return w < n_w;
}

__global__ void __launch_bounds__(256) k_gj_update(const cplx* src, cplx* A, int n, int n_w, const cplx* diag,
                                                   int p) {
  __shared__ cplx y[32 * 32];
  __shared__ int piv[32];
  int w, t;
  if (!gj_tile_of((n + 31) / 32, n_w, p, w, t)) return;
  gj_update<32, 256>(y, piv, src + (size_t)w * n * n, A + (size_t)w * n * n, n,
                     reinterpret_cast<const int*>(diag + (size_t)w * n), 32 * p, 32 * t);
}

__global__ void __launch_bounds__(256) k_gj_update_jobs(const GjJob* __restrict__ jobs, int n_jobs, int max_n,
                                                        int n_w, int p) {
  __shared__ cplx y[32 * 32];
  __shared__ int piv[32];
  int b, w, t;
  if (!gj_tile_of((max_n + 31) / 32, n_w, p, b, t)) return;
  const GjJob J = find_job(jobs, n_jobs, b, w);
  if (32 * max(p, t) >= J.n) return;
  cplx* A = J.eps + (size_t)w * J.n * J.n;
  gj_update<32, 256>(y, piv, A, A, J.n, reinterpret_cast<const int*>(J.diag + (size_t)w * J.n), 32 * p, 32 * t);
}

__global__ void __launch_bounds__(256) k_gj_gather(const cplx* A, int n, cplx* diag) {
  gj_gather(A + (size_t)blockIdx.x * n * n, n, diag + (size_t)blockIdx.x * n);
}

__global__ void __launch_bounds__(256) k_gj_gather_jobs(const GjJob* __restrict__ jobs, int n_jobs) {
  int w;
  const GjJob J = find_job(jobs, n_jobs, blockIdx.x, w);
  gj_gather(J.eps + (size_t)w * J.n * J.n, J.n, J.diag + (size_t)w * J.n);
}

__global__ void k_nolfe(const cplx* eps, int n, int n_w, cplx* diag, int* sing, int w_base) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long)n * n_w) return;
  const int j = (int)(i / n), G = (int)(i % n);
  const cplx e = eps[((size_t)j * n + G) * n + G];
  if (bad_pivot(e)) atomicMin(sing, w_base + j);
  diag[i] = cinv(e);
}

__global__ void k_loss(const cplx* diag, int n, int n_w, double* loss, cplx* epsM) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long)n * n_w) return;
  const cplx d = diag[i];
  loss[i] = -d.im;
  if (epsM && i % n == 0) epsM[i / n] = cinv(d);
}

// noLFE loss of Eq. (eps_noLFE) for a list of G from diagonal-only partial
// sums: chi0_GG = pref (Xr + i Yr) with Xr, Yr the Re W and Im W rows of the
// G-th diagonal pair (P_t(G, G) = |R_t(G)|^2 is real), eps_GG = 1 - v_G^2
// chi0_GG, loss = Im(-1 / eps_GG) = Im eps_GG / |eps_GG|^2.  Partials come
// from the bulk (a.C, [ks][n_rowsp][2][n_bulkp]) or the FP64 pairs kernel
// (a.XY, [ks64][n_rowsp64][n_colp64]); column b of chunk G-index b.
__global__ void k_diag_loss(AsmArgs a, Chi0Geom g, int n_g, int n_w, double* __restrict__ loss,
                            cplx* __restrict__ inv, int ldl, int g0) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long)n_w * n_g) return;
  const int j = (int)(i / n_g), b = (int)(i % n_g);
  const int parts = a.parts == 1 ? 1 : 2;
  double Xr = 0.0, Yr = 0.0;
  if (a.XY) {
    for (int ks = 0; ks < a.ks64; ++ks) {
      const double* x0 = a.XY + ((size_t)ks * a.n_rowsp64 + 2 * j) * a.n_colp64 + parts * b;
      Xr += x0[0];
      Yr += x0[a.n_colp64];
    }
  } else {
    for (int ks = 0; ks < a.ks; ++ks) {
      const size_t r0 = ((size_t)ks * g.n_rowsp + 2 * j) * parts;
      Xr += (double)a.C[r0 * g.n_bulkp + b];
      Yr += (double)a.C[(r0 + parts) * g.n_bulkp + b];
    }
  }
  const double vv = a.vq[b] * a.vq[b];
  const double er = 1.0 - vv * a.pref * Xr, ei = -vv * a.pref * Yr;
  const double d2 = er * er + ei * ei;
  loss[(size_t)j * ldl + g0 + b] = ei / d2;
  if (inv) inv[(size_t)j * ldl + g0 + b] = {er / d2, -ei / d2};  // 1 / eps_GG
}

__global__ void k_rho_export(const cplx* R, size_t ldt, int n_g, int n_t, cplx* out) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long)n_g * n_t) return;
  const int t = (int)(i / n_g), g = (int)(i % n_g);
  out[i] = R[(size_t)g * ldt + t];
}

}  // namespace

void launch_eps_assemble(const AsmArgs& a, const Chi0Geom& g, cplx* eps, hipStream_t st) {
  const long total = (long)g.n_w * g.n_pairs;
  hipLaunchKernelGGL(k_assemble, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, a, g, 0,
                     eps);
}

void launch_chi0_export(const AsmArgs& a, const Chi0Geom& g, cplx* chi, hipStream_t st) {
  const long total = (long)g.n_w * g.n_pairs;
  hipLaunchKernelGGL(k_assemble, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, a, g, 1,
                     chi);
}

int gj_class(int n_g) {
  if (n_g <= 64) return 0;
  if (n_g <= 128) return 1;
  if (n_g <= 192) return 2;
  if (n_g <= 256) return 3;
  if (n_g <= 320) return 4;
  if (n_g <= 512) return 5;
  if (n_g <= 768) return 6;
  if (n_g <= 1024) return 7;
  return 8;  // beyond the inversion kernels: callers reject n_g > 1024
}

namespace {

// the launches of one class of tiled inversions: single (jobs null) or multi-item
struct GjRun {
  const cplx* src;
  cplx* eps;
  int n, n_w;  // the largest size, matrices
  cplx* diag;
  int *sing, w_base;
  const GjJob* jobs;
  int n_jobs;
  int n_all;  // matrices of the whole call, of which this launch may be a chunk
};

void gj_gather(const GjRun& r, hipStream_t st) {
  if (r.jobs)
    hipLaunchKernelGGL(k_gj_gather_jobs, dim3(r.n_w), dim3(256), 0, st, r.jobs, r.n_jobs);
  else
    hipLaunchKernelGGL(k_gj_gather, dim3(r.n_w), dim3(256), 0, st, r.eps, r.n, r.diag);
}

template <int RP, int CP, int NW>
void gj_tiles(const GjRun& r, hipStream_t st) {
  constexpr int MB = NW * CP;
  const int n_t = (r.n + MB - 1) / MB, bx = (r.n_w + 7) / 8 * 8;
  for (int p = -1; p < n_t; ++p) {
    const dim3 g(bx, p < 0 ? 1 : n_t - 1), b(64 * NW);
    if (r.jobs)
      hipLaunchKernelGGL((k_gj_tile_jobs<RP, CP, NW>), g, b, 0, st, r.jobs, r.n_jobs, r.n_w, p);
    else
      hipLaunchKernelGGL((k_gj_tile<RP, CP, NW>), g, b, 0, st, r.src, r.eps, r.n, r.n_w, r.diag, r.sing,
                         r.w_base, p);
  }
  gj_gather(r, st);
}

template <int RP>
void gj_panels(const GjRun& r, hipStream_t st) {
  const int n_t = (r.n + 31) / 32, ub = (r.n_w + 7) / 8 * 8 * (n_t - 1);
  for (int p = 0; p < n_t; ++p) {
    if (r.jobs) {
      hipLaunchKernelGGL(k_gj_panel2_jobs<RP>, dim3(r.n_w), dim3(1024), 0, st, r.jobs, r.n_jobs, 32 * p);
      hipLaunchKernelGGL(k_gj_update_jobs, dim3(ub), dim3(256), 0, st, r.jobs, r.n_jobs, r.n, r.n_w, p);
    } else {
      hipLaunchKernelGGL(k_gj_panel2<RP>, dim3(r.n_w), dim3(1024), 0, st, r.src, r.eps, r.n, r.diag, r.sing,
                         r.w_base, 32 * p);
      hipLaunchKernelGGL(k_gj_update, dim3(ub), dim3(256), 0, st, r.src, r.eps, r.n, r.n_w, r.diag, p);
    }
  }
  gj_gather(r, st);
}

// Which form.  One launch per panel (gj_tiles) keeps a matrix's chain short:
// the next panel is swept beside the other tiles' updates.  It wins while the
// sweeps leave compute units free for those; past that its 1024-thread update
// blocks, one per compute unit, are the bound, and smaller ones win: 8 waves
// holding four columns each up to n = 320, above it panels and updates in two
// launches (gj_panels).  Measured, us (gj_tiles | the other): n = 180, 160
// matrices 412 | 423, 200 524 | 458; n = 259, 128 matrices 910 | 936, 160 1113 |
// 1029; n = 500, 128 5392 | 5931, 192 8110 | 8154, 256 10781 | 10123; n = 749, 96
// 15930 | 16257, 128 21367 | 20545; n = 800, 32 8051 | 8476, 48 12247 | 10989;
// n = 953, 16 6369 | 8101, 32 15677 | 14724, 64 31903 | 23775.
void gj_tiles(int cls, const GjRun& r, hipStream_t st) {
  // Up to n = 320 both forms give the same bits.  Above, their rounding differs,
  // so the whole call decides: the results of a call that runs in chunks are
  // those of one that does not.
  const bool few = (cls <= 4 ? r.n_w : r.n_all) <= (cls == 7 ? 32 : cls == 6 ? 96 : cls == 5 ? 192 : 128);
  switch (cls) {
    case 2: return few ? gj_tiles<3, 2, 16>(r, st) : gj_tiles<3, 4, 8>(r, st);
    case 3: return few ? gj_tiles<4, 2, 16>(r, st) : gj_tiles<4, 4, 8>(r, st);
    case 4: return few ? gj_tiles<5, 2, 16>(r, st) : gj_tiles<5, 4, 8>(r, st);
    case 5: return few ? gj_tiles<8, 2, 16>(r, st) : gj_panels<8>(r, st);
    case 6: return few ? gj_tiles<12, 2, 16>(r, st) : gj_panels<12>(r, st);
    case 7: return few ? gj_tiles<16, 1, 16>(r, st) : gj_panels<16>(r, st);
    default: return;  // callers keep n_g <= 1024 (class 7); nothing is launched beyond
  }
}

}  // namespace

void launch_gj_diag(const cplx* src, cplx* eps, int n_g, int n_w, cplx* diag, int* sing, hipStream_t st,
                    int w_base, int n_all) {
  const dim3 g(n_w), b(1024);
  const int cls = gj_class(n_g);
  if (cls == 0)
    hipLaunchKernelGGL((k_gj_reg<1, 4>), g, b, 0, st, src, n_g, diag, sing, w_base);
  else if (cls == 1)
    hipLaunchKernelGGL((k_gj_reg<2, 8>), g, b, 0, st, src, n_g, diag, sing, w_base);
  else
    gj_tiles(cls, GjRun{src, eps, n_g, n_w, diag, sing, w_base, nullptr, 0, std::max(n_w, n_all)}, st);
}

void launch_gj_jobs(int cls, const GjJob* jobs, int n_jobs, int n_blocks, int max_n, hipStream_t st) {
  const dim3 g(n_blocks), b(1024);
  if (cls == 0)
    hipLaunchKernelGGL((k_gj_reg_jobs<1, 4>), g, b, 0, st, jobs, n_jobs);
  else if (cls == 1)
    hipLaunchKernelGGL((k_gj_reg_jobs<2, 8>), g, b, 0, st, jobs, n_jobs);
  else
    gj_tiles(cls, GjRun{nullptr, nullptr, max_n, n_blocks, nullptr, nullptr, 0, jobs, n_jobs, n_blocks}, st);
}

void launch_nolfe_diag(const cplx* eps, int n_g, int n_w, cplx* diag, int* sing, hipStream_t st,
                       int w_base) {
  const long total = (long)n_g * n_w;
  hipLaunchKernelGGL(k_nolfe, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, eps, n_g,
                     n_w, diag, sing, w_base);
}

void launch_loss(const cplx* diag, int n_g, int n_w, double* loss, cplx* epsM, hipStream_t st) {
  const long total = (long)n_g * n_w;
  hipLaunchKernelGGL(k_loss, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, diag, n_g,
                     n_w, loss, epsM);
}

void launch_diag_loss(const AsmArgs& a, const Chi0Geom& g, int n_g, int n_w, double* loss,
                      cplx* inv, int ldl, int g0, hipStream_t st) {
  const long total = (long)n_g * n_w;
  hipLaunchKernelGGL(k_diag_loss, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, a, g,
                     n_g, n_w, loss, inv, ldl, g0);
}

void launch_rho_export(const cplx* R, size_t ldt, int n_g, int n_t, cplx* out, hipStream_t st) {
  const long total = (long)n_g * n_t;
  hipLaunchKernelGGL(k_rho_export, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, R, ldt,
                     n_g, n_t, out);
}

}  // namespace qcx

// Kernels of the energy-panel route of chi0 (Eq. (RPA) at finite eta, see
// panel_plan.h): with W_t(w) = sum_i c_{a,i}(w) T_i(y_t) on the panel a of
// transition t,
//   sum_t W_t(w) P_t(G, G') = sum_a sum_i c_{a,i}(w) S_{a,i}(G, G'),
//   S_{a,i}(G, G') = sum_{t in a} T_i(y_t) P_t(G, G'),
// so the N_T transitions enter once with 16 (FP64: 32) rows instead of once
// with 2 N_w rows, and the frequencies enter through a product whose depth is
// the number of panel terms instead of N_T.
#include <algorithm>
#include <vector>

#include "panel.h"

namespace qcx {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

// The reduced-precision modes hold every operand in 24 bits of FP32's range:
// basis functions and densities enter the moments as FP32, on FP32 MFMA; the
// moments and the coefficients enter the product over panels as three bf16
// planes, x = p0 + p1 + p2, each the bf16 nearest to what is left, with the six
// products of planes down to 2^-16 of the first.  Two fp16 planes (22 bits, one
// power-of-two scale per row of G) took 0.3 ms less for 113 G, 65,536
// transitions and 400 frequencies (1.7 against 2.0 ms), but have an absolute
// floor: where the densities of a row span three orders of magnitude the
// absorptive part far from every pole came out 3e-4 off (directly 1.4e-6).
constexpr int NS = 3;  // planes
__device__ inline uint16_t b_bits(float x) { return __builtin_bit_cast(uint16_t, (__bf16)x); }
__device__ inline float b_val(uint16_t b) { return __uint_as_float((unsigned)b << 16); }

template <class F>
__device__ inline void split_b(F x, uint16_t (&o)[NS]) {
#pragma unroll
  for (int p = 0; p < NS; ++p) {
    o[p] = b_bits((float)x);
    x -= (F)b_val(o[p]);
  }
}

// ------------------------------------------------------------------- sorting
// panel of energy D on its side: the number of edges at or below D (a NaN
// counts none, so every index is valid whatever the energies hold)
__device__ inline int panel_of(const PanelSort& s, int t, double D) {
  const int side = t >= s.n_t / 2;
  const double* e = s.edge + (side ? s.P0 - 1 : 0);
  int lo = 0, hi = (side ? s.P - s.P0 : s.P0) - 1;
  while (lo < hi) {
    const int m = (lo + hi) >> 1;
    if (e[m] <= D)
      lo = m + 1;
    else
      hi = m;
  }
  return lo + (side ? s.P0 : 0);
}

__global__ void __launch_bounds__(256) k_pan_hist(PanelSort s) {
  extern __shared__ int h[];
  for (int p = threadIdx.x; p < s.P; p += 256) h[p] = 0;
  __syncthreads();
  const int t1 = min(s.n_t, (int)(blockIdx.x + 1) * s.per);
  for (int t = blockIdx.x * s.per + threadIdx.x; t < t1; t += 256) {
    const int p = panel_of(s, t, s.dt[t]);
    s.pidx[t] = p;
    atomicAdd(&h[p], 1);  // integer counts: any order gives the same
  }
  __syncthreads();
  for (int p = threadIdx.x; p < s.P; p += 256) s.hist[(size_t)blockIdx.x * s.P + p] = h[p];
}

// Counts of the blocks -> first rank of each block in each panel, first step
// of each panel, and the entries: those of ch transitions first (their waves
// run longest, so they start first), then what is left of each panel.  One
// block; latency-bound (the loads over the blocks go eight at a time).
__global__ void __launch_bounds__(1024) k_pan_scan(PanelSort s) {
  extern __shared__ int cnt[];
  __shared__ int ws[3][16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int full = 0;
  for (int p = tid; p < s.P; p += 1024) {
    int run = 0;
    for (int b = 0; b < s.nb; b += 8) {
      int v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = b + i < s.nb ? s.hist[(size_t)(b + i) * s.P + p] : 0;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        if (b + i < s.nb) s.hist[(size_t)(b + i) * s.P + p] = run;
        run += v[i];
      }
    }
    cnt[p] = run;
    full += run / s.ch;
  }
#pragma unroll
  for (int d = 32; d; d >>= 1) full += __shfl_xor(full, d);
  if (lane == 0) ws[0][wave] = full;
  __syncthreads();
  int tot[3] = {0, 0, 0};  // steps, full entries, rests before this pass
#pragma unroll
  for (int w = 0; w < 16; ++w) tot[2] += ws[0][w];
  __syncthreads();
  for (int base = 0; base < s.P; base += 1024) {
    const int p = base + tid;
    const int c = p < s.P ? cnt[p] : 0;
    const int mine[3] = {(c + kPanStep - 1) / kPanStep, c / s.ch, c % s.ch > 0};
    int in[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {  // inclusive sums over the wave, then the block
      in[k] = mine[k];
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int a = __shfl_up(in[k], d);
        if (lane >= d) in[k] += a;
      }
      if (lane == 63) ws[k][wave] = in[k];
    }
    __syncthreads();
    int at[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      at[k] = tot[k] + in[k] - mine[k];
#pragma unroll
      for (int w = 0; w < 16; ++w) {
        if (w < wave) at[k] += ws[k][w];
        tot[k] += ws[k][w];
      }
    }
    if (p < s.P) {
      s.pstart[p] = at[0];
      const int per = s.ch / kPanStep;
      for (int k = 0; k < mine[1]; ++k) s.act[at[1] + k] = make_int4(p, at[0] + k * per, s.ch, 0);
      if (mine[2]) s.act[at[2]] = make_int4(p, at[0] + mine[1] * per, c % s.ch, 0);
    }
    __syncthreads();
  }
  if (tid == 0) {
    s.n_act[0] = tot[2];
    s.n_act[1] = tot[0];
  }
}

// Stable scatter: within a panel the transitions keep their order, so the
// sums do not depend on the launch.
__global__ void __launch_bounds__(256) k_pan_scatter(PanelSort s) {
  extern __shared__ int run[];
  __shared__ __attribute__((aligned(16))) int key[256];
  for (int p = threadIdx.x; p < s.P; p += 256) run[p] = s.hist[(size_t)blockIdx.x * s.P + p];
  const int t1 = min(s.n_t, (int)(blockIdx.x + 1) * s.per);
  for (int t0 = blockIdx.x * s.per; t0 < t1; t0 += 256) {
    const int t = t0 + threadIdx.x;
    const int p = t < t1 ? s.pidx[t] : -1 - (int)threadIdx.x;  // no two idle keys alike
    key[threadIdx.x] = p;
    __syncthreads();
    int before = 0, all = 0;
    for (int j = 0; j < 256; j += 4) {
      const int4 k4 = *reinterpret_cast<const int4*>(&key[j]);
      const int k[4] = {k4.x, k4.y, k4.z, k4.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int e = k[i] == p;
        all += e;
        before += e & (j + i < (int)threadIdx.x);
      }
    }
    const int r = t < t1 ? run[p] + before : 0;
    __syncthreads();
    if (t < t1) {
      if (before == 0) run[p] += all;
      const int q = s.pstart[p] * kPanStep + r;
      s.pos[t] = q;
      s.Ds[q] = s.dt[t];
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------ basis functions
// y and the factor of the basis at energy D
__device__ inline double panel_y(const PanelDesc& d, double D, double& f) {
  if (d.kind == 0) {
    f = 1.0;
    return (D - d.c) * d.s;
  }
  const double u = d.s / (D - d.c);
  f = u;
  return 2.0 * u - 1.0;
}

// An entry's positions go round kTabSplit blocks (grid y): the longest entries
// (1024 positions and more) set the time.
constexpr int kTabSplit = 4;
__global__ void __launch_bounds__(256) k_pan_tab(PanelSort s, float4* __restrict__ T) {
  const int a = blockIdx.x;
  if (a >= s.n_act[0]) return;
  const int4 pd = s.act[a];
  const PanelDesc d = s.desc[pd.x];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = lane & 15;
  const int steps = (pd.z + kPanStep - 1) / kPanStep;
  for (int st = wave + 4 * blockIdx.y; st < steps; st += 4 * kTabSplit) {
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int q = st * kPanStep + 8 * (lane >> 4) + j;
      double x = 0.0;
      if (q < pd.z) {
        double f;
        const double y = panel_y(d, s.Ds[(size_t)pd.y * kPanStep + q], f);
        double t0 = f, t1 = f * y;  // T_i by its recurrence
        for (int n = 0; n < i; ++n) {
          const double t2 = 2.0 * y * t1 - t0;
          t0 = t1;
          t1 = t2;
        }
        x = t0;
      }
      v[j] = (float)x;
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
      T[((size_t)(pd.y + st) * 2 + h) * 64 + lane] = make_float4(v[4 * h], v[4 * h + 1], v[4 * h + 2], v[4 * h + 3]);
  }
}

__global__ void __launch_bounds__(256) k_pan_tab64(PanelSort s, double* __restrict__ T64) {
  const int a = blockIdx.x;
  if (a >= s.n_act[0]) return;
  const int4 pd = s.act[a];
  const PanelDesc d = s.desc[pd.x];
  const int n = (pd.z + kPanStep - 1) / kPanStep * kPanStep;
  const int m = threadIdx.x & 3;  // terms 8m .. 8m + 7
  for (int q = (threadIdx.x >> 2) + 64 * blockIdx.y; q < n; q += 64 * kTabSplit) {
    const size_t p = (size_t)pd.y * kPanStep + q;
    double o[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (q < pd.z) {
      double f;
      const double y = panel_y(d, s.Ds[p], f);
      double t0 = f, t1 = f * y;
      for (int k = 0; k < 8 * m; ++k) {
        const double t2 = 2.0 * y * t1 - t0;
        t0 = t1;
        t1 = t2;
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        o[k] = t0;
        const double t2 = 2.0 * y * t1 - t0;
        t0 = t1;
        t1 = t2;
      }
    }
    double2* w = reinterpret_cast<double2*>(T64 + p * kPanelTerms64 + 8 * m);
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = make_double2(o[2 * k], o[2 * k + 1]);
  }
}

// -------------------------------------------------------------------- packing
// A block moves PP_N times 32 transitions x 64 rows of R through LDS: reads
// along t, writes along g at the transition's position.  Blocks past the
// transitions clear the padded positions of one entry each.
constexpr int PP_T = 32, PP_G = 64, PP_N = 4;
__global__ void __launch_bounds__(256) k_pan_pack(PanelSort s, PanelPack p, int n_tb) {
  __shared__ cplx tile[PP_T][PP_G + 1];
  __shared__ cplx r0[PP_T];
  if ((int)blockIdx.x >= n_tb) {
    const int a = blockIdx.x - n_tb;
    if (blockIdx.y || a >= s.n_act[0]) return;
    const int4 pd = s.act[a];
    const int n = (pd.z + kPanStep - 1) / kPanStep * kPanStep;
    for (int q = pd.z; q < n; ++q) {
      const size_t r = (size_t)pd.y * kPanStep + q;
      if (p.R32)
        for (int i = threadIdx.x; i < p.ld32; i += 256) p.R32[r * p.ld32 + i] = make_float2(0.f, 0.f);
      if (p.R64)
        for (int i = threadIdx.x; i < p.ld64; i += 256) p.R64[r * p.ld64 + i] = cplx{0.0, 0.0};
      if (p.W64)
        for (int i = threadIdx.x; i < p.ldw; i += 256) p.W64[r * p.ldw + i] = cplx{0.0, 0.0};
      if (p.A64)
        for (int i = threadIdx.x; i < p.lda64; i += 256) p.A64[r * p.lda64 + i] = 0.0;
    }
    return;
  }
  const int g0 = blockIdx.y * PP_G, gg = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int i = 0; i < PP_N; ++i) {
    const int t0 = (blockIdx.x * PP_N + i) * PP_T;
    if (t0 >= s.n_t) break;
    if (i) __syncthreads();
    for (int e = threadIdx.x; e < PP_T * PP_G; e += 256) {
      const int g = g0 + e / PP_T, t = t0 + e % PP_T;
      tile[e % PP_T][e / PP_T] = (g < p.n_g && t < s.n_t) ? p.R[(size_t)g * p.ldt + t] : cplx{0.0, 0.0};
    }
    if (p.W64 && threadIdx.x < PP_T)
      r0[threadIdx.x] = t0 + (int)threadIdx.x < s.n_t ? p.R[t0 + threadIdx.x] : cplx{0.0, 0.0};
    __syncthreads();
    const int g = g0 + gg;
#pragma unroll
    for (int k = 0; k < PP_T / 4; ++k) {
      const int tt = wv + 4 * k, t = t0 + tt;
      if (t >= s.n_t) break;
      const size_t r = (size_t)s.pos[t];
      const cplx v = tile[tt][gg];
      if (p.R32 && g >= p.g_lo && g - p.g_lo < p.ld32)
        p.R32[r * p.ld32 + g - p.g_lo] = make_float2((float)v.re, (float)v.im);
      if (p.R64 && g < p.ld64) p.R64[r * p.ld64 + g] = v;
      if (p.W64 && g < p.ldw) p.W64[r * p.ldw + g] = cmulc(r0[tt], v);
      if (p.A64 && g < p.lda64) p.A64[r * p.lda64 + g] = v.re * v.re + v.im * v.im;
    }
  }
}

// -------------------------------------------------------------------- moments
// One wave = one entry x 8 G x 16 G' on v_mfma_f32_16x16x4_f32 (A 16x4: lane
// holds A[l % 16][l / 16]; B 4x16: B[l / 16][l % 16]; D: D[4 (l / 16) + r][l %
// 16]).  Per step of 32 positions a lane holds R of its G' (lane % 16) at its 8
// positions (8 (lane / 16) ..) in registers, which are its K slots of the
// step's eight MFMAs; the 8 rows of G go through the wave's own LDS (each is
// read by all lanes of a position group); the pair products are formed in FP32
// and are the B operand, the Chebyshev functions the A operand (16 terms).  No
// barriers: the LDS is private to the wave.  Bound by the FP32 MFMAs and the
// forming of the products, whose times add up (113 G, 65,536 transitions: 395
// us, of which the MFMAs are 200 and the vector instructions 100; forming the
// products of one or two G ahead changed nothing).
constexpr int PB_G = kPanBinRows;

// store terms 4 q .. 4 q + 3 (q = lane / 16) of one column
__device__ __forceinline__ void pan_store(uint2* __restrict__ S, size_t tile0, int col, int q, const f32x4& v) {
  uint16_t o[4][NS];
#pragma unroll
  for (int r = 0; r < 4; ++r) split_b(v[r], o[r]);
  const size_t fr = (tile0 + (col >> 5)) * NS;
#pragma unroll
  for (int p = 0; p < NS; ++p) {
    uint2 w;
    w.x = o[0][p] | ((uint32_t)o[1][p] << 16);
    w.y = o[2][p] | ((uint32_t)o[3][p] << 16);
    S[((fr + p) * 64 + (col & 31) + 32 * (q >> 1)) * 2 + (q & 1)] = w;
  }
}

// wave w of the launch -> item: entry a, task.  Entries are dealt to the XCDs
// in turn (workgroup i runs on XCD i % 8), so the rows of an entry are read
// into one L2 only.  A launch holds a few rounds of resident blocks; items
// beyond it go to the blocks of its end first (round 1 counts backwards),
// whose first items are the short ones.
__device__ inline void pan_task(int n_task, int wave, int round, int& a, int& task) {
  const int x = blockIdx.x & 7, nb = gridDim.x >> 3, b = blockIdx.x >> 3;
  const int i = (round * nb + (round & 1 ? nb - 1 - b : b)) * 4 + wave;
  a = 8 * (i / n_task) + x;
  task = i % n_task;
}

__global__ void __launch_bounds__(256, 2) k_pan_bin(PanelSort s, const float4* __restrict__ T, PanelBin b) {
  __shared__ __attribute__((aligned(16))) f32x2 sG[4][PB_G][34];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n_act = s.n_act[0];
  const int n = lane & 15, kg = lane >> 4;
  const int g4 = 4 * (lane & 1), tt = lane >> 1;
  const unsigned og = tt * b.ld32 + g4, oh = 8 * kg * b.ld32 + n;
  const size_t row_step = (size_t)kPanStep * b.ld32;
  for (int round = 0;; ++round) {
    int a, task;
    pan_task(b.n_task, wave, round, a, task);
    if (a >= n_act) break;
    const int4 pd = s.act[a];
    const int2 tk = b.tasks[task];
    const int steps = (pd.z + kPanStep - 1) / kPanStep;
    // addresses: a part common to the wave and the lane's own 32-bit offset
    const float2* Ru = b.R32 + (size_t)pd.y * row_step;
    const float4* Tu = T + (size_t)pd.y * 2 * 64;
    float4 gn[2];
    float2 hn[8];
    float4 tn[2];
    auto fetch = [&](int st) {
      const float2* r = Ru + st * row_step;
      const float4* src = reinterpret_cast<const float4*>(r + tk.x + og);
      gn[0] = src[0];
      gn[1] = src[1];
#pragma unroll
      for (int j = 0; j < 8; ++j) hn[j] = (r + tk.y + (size_t)j * b.ld32)[oh];
#pragma unroll
      for (int p = 0; p < 2; ++p) tn[p] = (Tu + ((size_t)st * 2 + p) * 64)[lane];
    };
    fetch(0);
    f32x4 ar[PB_G], ai[PB_G];
#pragma unroll
    for (int g = 0; g < PB_G; ++g) ar[g] = ai[g] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int st = 0; st < steps; ++st) {
      float2 h[8];
      __builtin_amdgcn_wave_barrier();
      sG[wave][g4 + 0][tt] = f32x2{gn[0].x, gn[0].y};
      sG[wave][g4 + 1][tt] = f32x2{gn[0].z, gn[0].w};
      sG[wave][g4 + 2][tt] = f32x2{gn[1].x, gn[1].y};
      sG[wave][g4 + 3][tt] = f32x2{gn[1].z, gn[1].w};
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int j = 0; j < 8; ++j) h[j] = hn[j];
      const float t[8] = {tn[0].x, tn[0].y, tn[0].z, tn[0].w, tn[1].x, tn[1].y, tn[1].z, tn[1].w};
      if (st + 1 < steps) fetch(st + 1);
#pragma unroll
      for (int g = 0; g < PB_G; ++g) {
        const f32x4* rg = reinterpret_cast<const f32x4*>(&sG[wave][g][8 * kg]);
        f32x4 sr = {0.f, 0.f, 0.f, 0.f}, si = sr;  // the step's sums, then onto the entry's
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const f32x4 x = rg[j];
          const float2 y0 = h[2 * j], y1 = h[2 * j + 1];  // conj(x) y
          sr = __builtin_amdgcn_mfma_f32_16x16x4f32(t[2 * j], x.x * y0.x + x.y * y0.y, sr, 0, 0, 0);
          si = __builtin_amdgcn_mfma_f32_16x16x4f32(t[2 * j], x.x * y0.y - x.y * y0.x, si, 0, 0, 0);
          sr = __builtin_amdgcn_mfma_f32_16x16x4f32(t[2 * j + 1], x.z * y1.x + x.w * y1.y, sr, 0, 0, 0);
          si = __builtin_amdgcn_mfma_f32_16x16x4f32(t[2 * j + 1], x.z * y1.y - x.w * y1.x, si, 0, 0, 0);
        }
        ar[g] += sr;
        ai[g] += si;
      }
    }
    const size_t tile0 = (size_t)a * (2 * b.nbp / 32);
    const int Gp = tk.y + n;
#pragma unroll
    for (int g = 0; g < PB_G; ++g) {
      const int G = tk.x + g;
      if (G > Gp || Gp >= b.n_gl) continue;
      const long pb = (long)G * b.n_gl - (long)G * (G - 1) / 2 + (Gp - G) - b.b0;
      pan_store(b.S, tile0, (int)pb, kg, ar[g]);
      pan_store(b.S, tile0, b.nbp + (int)pb, kg, ai[g]);
    }
  }
}

// FP64 moments of the columns of a table: one wave = one active panel x 32
// columns on v_mfma_f64_16x16x4f64 (A 16x4: lane holds A[l % 16][l / 16]; B
// 4x16: B[l / 16][l % 16]; D: D[4 r + l / 16][l % 16]).  Fragment f of A holds
// terms 2 m + f, fragment c of B columns 2 n + c, so that a lane loads both of
// its values at once.  SPLIT: the four waves of a block share a panel and its
// columns, every fourth group of 16 positions each, and add up through LDS.
template <bool SPLIT>
__global__ void __launch_bounds__(256) k_pan_bin64(PanelSort s, const double* __restrict__ T64,
                                                   const double* __restrict__ X, int ldx, int n_task,
                                                   int n_col, double* __restrict__ S64, int lds) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int a, task;
  if constexpr (SPLIT) {
    const int i = blockIdx.x >> 3;
    a = 8 * (i / n_task) + (int)(blockIdx.x & 7);
    task = i % n_task;
  } else {
    pan_task(n_task, wave, 0, a, task);
  }
  if (a >= s.n_act[0]) return;
  const int4 pd = s.act[a];
  const int n = lane & 15, kg = lane >> 4, c0 = 32 * task + 2 * n;
  const size_t p0 = (size_t)pd.y * kPanStep + kg;
  const double* Tp = T64 + p0 * kPanelTerms64 + 2 * n;
  const double* Xp = X + p0 * ldx + c0;
  f64x4 acc[2][2];
#pragma unroll
  for (int f = 0; f < 2; ++f)
#pragma unroll
    for (int c = 0; c < 2; ++c) acc[f][c] = f64x4{0.0, 0.0, 0.0, 0.0};
  // padded positions hold zeros, so whole groups of 16 may be taken
  const int n16 = (pd.z + 15) / 16;
  double2 tn[4], xn[4];
  auto fetch = [&](int q) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      tn[u] = *reinterpret_cast<const double2*>(Tp + (size_t)(16 * q + 4 * u) * kPanelTerms64);
      xn[u] = *reinterpret_cast<const double2*>(Xp + (size_t)(16 * q + 4 * u) * ldx);
    }
  };
  constexpr int QS = SPLIT ? 4 : 1;
  const int q0 = SPLIT ? wave : 0;
  if (q0 < n16) fetch(q0);
  for (int q = q0; q < n16; q += QS) {
    double2 t[4], x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      t[u] = tn[u];
      x[u] = xn[u];
    }
    if (q + QS < n16) fetch(q + QS);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(t[u].x, x[u].x, acc[0][0], 0, 0, 0);
      acc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(t[u].x, x[u].y, acc[0][1], 0, 0, 0);
      acc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(t[u].y, x[u].x, acc[1][0], 0, 0, 0);
      acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(t[u].y, x[u].y, acc[1][1], 0, 0, 0);
    }
  }
  if constexpr (SPLIT) {
    // wave w adds and stores element r = w of every fragment
    __shared__ double part[4][16][64];
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) part[wave][4 * r + 2 * f + c][lane] = acc[f][c][r];
    __syncthreads();
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      double v[2] = {0.0, 0.0};
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int w = 0; w < 4; ++w) v[c] += part[w][4 * wave + 2 * f + c][lane];
      double* o = S64 + ((size_t)a * kPanelTerms64 + 2 * (4 * wave + kg) + f) * lds + c0;
      if (c0 + 1 < n_col)
        *reinterpret_cast<double2*>(o) = make_double2(v[0], v[1]);
      else if (c0 < n_col)
        *o = v[0];
    }
    return;
  }
#pragma unroll
  for (int f = 0; f < 2; ++f)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      double* o = S64 + ((size_t)a * kPanelTerms64 + 2 * (4 * r + kg) + f) * lds + c0;
      if (c0 + 1 < n_col)
        *reinterpret_cast<double2*>(o) = make_double2(acc[f][0][r], acc[f][1][r]);
      else if (c0 < n_col)
        *o = acc[f][0][r];
    }
}

// FP64 moments of pairs: one wave = one active panel x 2 G x 16 G'; lane n
// holds R of G' (one position per MFMA K slot), the G rows are broadcast
// loads; products in FP64.  Bound by the loads' latency, then by the moments
// written (620 MB for 89 G): two G rows leave room for four waves per SIMD with
// two steps of loads in flight, 478 us there; four rows with one step in flight
// (one wave per SIMD) 794, at two waves 588 to 626; one row 523, three 530.
constexpr int PQ_G = kPanBin64Rows;
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4)))
k_pan_bin64_pairs(PanelSort s, const double* __restrict__ T64, PanelBin64 b) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int a, task;
  pan_task(b.n_task, wave, 0, a, task);
  if (a >= s.n_act[0]) return;
  const int4 pd = s.act[a];
  const int2 tk = b.tasks[task];
  const int n = lane & 15, kg = lane >> 4;
  const size_t p0 = (size_t)pd.y * kPanStep + kg;
  const double* Tp = T64 + p0 * kPanelTerms64 + 2 * n;
  const cplx* Rh = b.R64 + p0 * b.ld64 + tk.y + n;
  const cplx* Rg = b.R64 + p0 * b.ld64 + tk.x;
  f64x4 acc[PQ_G][2][2];  // [G][term parity][part]
#pragma unroll
  for (int g = 0; g < PQ_G; ++g)
#pragma unroll
    for (int f = 0; f < 2; ++f) acc[g][f][0] = acc[g][f][1] = f64x4{0.0, 0.0, 0.0, 0.0};
  // padded positions hold zeros: whole pairs of steps
  const int n4 = (pd.z + 7) / 8 * 2;
  struct In {
    double2 t;
    cplx h, g[PQ_G];
  } in[2];
  auto fetch = [&](int q, In& x) {
    x.t = *reinterpret_cast<const double2*>(Tp + (size_t)4 * q * kPanelTerms64);
    x.h = Rh[(size_t)4 * q * b.ld64];
#pragma unroll
    for (int g = 0; g < PQ_G; ++g) x.g[g] = Rg[(size_t)4 * q * b.ld64 + g];
  };
  fetch(0, in[0]);
  fetch(1, in[1]);
  for (int q0 = 0; q0 < n4; q0 += 2)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const double2 t = in[u].t;
      cplx P[PQ_G];
#pragma unroll
      for (int g = 0; g < PQ_G; ++g) P[g] = cmulc(in[u].g[g], in[u].h);
      if (q0 + 2 < n4) fetch(q0 + 2 + u, in[u]);
#pragma unroll
      for (int g = 0; g < PQ_G; ++g) {
        acc[g][0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(t.x, P[g].re, acc[g][0][0], 0, 0, 0);
        acc[g][0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(t.x, P[g].im, acc[g][0][1], 0, 0, 0);
        acc[g][1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(t.y, P[g].re, acc[g][1][0], 0, 0, 0);
        acc[g][1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(t.y, P[g].im, acc[g][1][1], 0, 0, 0);
      }
    }
  const int Gp = tk.y + n;
#pragma unroll
  for (int g = 0; g < PQ_G; ++g) {
    const int G = tk.x + g;
    if (G > Gp || Gp >= b.n_g) continue;
    const long pb = (long)G * b.n_g - (long)G * (G - 1) / 2 + (Gp - G) - b.b0;
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        *reinterpret_cast<double2*>(b.S64 + ((size_t)a * kPanelTerms64 + 2 * (4 * r + kg) + f) * b.lds +
                                    2 * pb) = make_double2(acc[g][f][0][r], acc[g][f][1][r]);
  }
}

// --------------------------------------------------------------- coefficients
struct cd {
  double re, im;
};
__device__ inline cd cd_mul(cd a, cd b) { return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }
__device__ inline cd cd_inv(cd a) {  // |a| of order one or above here
  const double r = 1.0 / (a.re * a.re + a.im * a.im);
  return {a.re * r, -a.im * r};
}
__device__ inline cd cd_sqrt(cd a) {  // principal branch
  const double m = hypot(a.re, a.im);
  const double x = sqrt(0.5 * (m + fabs(a.re)));
  if (!(x > 0.0)) return {0.0, 0.0};
  const double y = 0.5 * a.im / x;
  return a.re >= 0.0 ? cd{x, y} : cd{fabs(y), copysign(x, a.im)};
}

// series of 1 / (x - D + i eta) on a panel: coefficient i is
// (i ? 2 : 1) amp q^i in the panel's basis
__device__ inline void panel_series(const PanelDesc& d, double x, double eta, cd& amp, cd& q) {
  cd z;
  cd f;
  if (d.kind == 0) {
    z = {(x - d.c) * d.s, eta * d.s};
    f = {d.s, 0.0};
  } else {
    const cd iz = cd_inv({(x - d.c) / d.s, eta / d.s});  // 1 / zeta, |zeta| < 1
    z = {2.0 * iz.re - 1.0, 2.0 * iz.im};
    f = {-2.0 * iz.re / d.s, -2.0 * iz.im / d.s};
  }
  const cd s = cd_mul(cd_sqrt({z.re - 1.0, z.im}), cd_sqrt({z.re + 1.0, z.im}));
  q = cd_inv({z.re + s.re, z.im + s.im});
  amp = cd_mul(f, cd_inv(s));
}

__global__ void __launch_bounds__(256) k_pan_coef(PanelSort s, const double* __restrict__ w, int n_w,
                                                  double eta, int row0, int n_rb,
                                                  uint4* __restrict__ A) {
  const int a = blockIdx.y;
  if (a >= s.n_act[0]) return;
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n_rb * 64) return;
  const int lane = i & 63, rb = i >> 6;
  const int row = row0 + 32 * rb + (lane & 31), j = row >> 1;
  uint16_t v[NS][8];
  cd amp{0.0, 0.0}, q{0.0, 0.0};
  if (j < n_w) {
    const int p = s.act[a].x;
    panel_series(s.desc[p], p >= s.P0 ? -w[j] : w[j], eta, amp, q);
    if (lane >> 5) {  // terms 8 ..
      const cd q2 = cd_mul(q, q), q4 = cd_mul(q2, q2);
      amp = cd_mul(amp, cd_mul(q4, q4));
    }
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    uint16_t o[NS];
    split_b((k || (lane >> 5) ? 2.0 : 1.0) * ((row & 1) ? amp.im : amp.re), o);
#pragma unroll
    for (int p = 0; p < NS; ++p) v[p][k] = o[p];
    amp = cd_mul(amp, q);
  }
#pragma unroll
  for (int p = 0; p < NS; ++p) {
    uint4 o;
    o.x = v[p][0] | ((uint32_t)v[p][1] << 16);
    o.y = v[p][2] | ((uint32_t)v[p][3] << 16);
    o.z = v[p][4] | ((uint32_t)v[p][5] << 16);
    o.w = v[p][6] | ((uint32_t)v[p][7] << 16);
    A[(((size_t)a * n_rb + rb) * NS + p) * 64 + lane] = o;
  }
}

__global__ void __launch_bounds__(256) k_pan_coef64(PanelSort s, const double* __restrict__ w, int n_w,
                                                    double eta, int ldm, double* __restrict__ K) {
  const int a = blockIdx.y;
  if (a >= s.n_act[0]) return;
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (2 * j >= ldm) return;
  cd amp{0.0, 0.0}, q{0.0, 0.0};
  if (j < n_w) {
    const int p = s.act[a].x;
    panel_series(s.desc[p], p >= s.P0 ? -w[j] : w[j], eta, amp, q);
  }
  double* o = K + (size_t)a * kPanelTerms64 * ldm + 2 * j;
  for (int i = 0; i < kPanelTerms64; ++i) {
    const double f = i ? 2.0 : 1.0;
    *reinterpret_cast<double2*>(o + (size_t)i * ldm) = make_double2(f * amp.re, f * amp.im);
    amp = cd_mul(amp, q);
  }
}

// ------------------------------------------------------------------- response
// C = A S on v_mfma_f32_32x32x16_bf16, both operands in fragment order (one
// active panel = one K step of 16 terms).  A block of 4 waves owns AF x 32
// rows x 256 columns: each wave all rows and 64 columns (AF x 2 accumulators
// of 16 registers, two waves per SIMD from two blocks).  An entry's six products
// are summed apart and enter the accumulators once, rounded to nearest (six
// MFMAs straight into them: the loss of 113 G 1.6e-6 off instead of 2.3e-7).  The 1 KB fragments of
// a step are copied straight into LDS one step ahead, two stages (39 KB each
// for AF = 5, so that two blocks fit a CU); a step's 60 MFMAs per wave outlast
// the copies.
typedef __attribute__((address_space(3))) void* lds_ptr_t;
template <int AF>
struct GemmStage {
  float4 a[AF * NS * 64];
  float4 b[8 * NS * 64];
};

template <int AF>
__device__ __forceinline__ void pan_gemm_tile(const PanelSort& s, const PanelGemm& g,
                                              GemmStage<AF>& s0, GemmStage<AF>& s1) {
  using L = GemmStage<AF>;
  const int lane = threadIdx.x & 63, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nct = 2 * g.nbp / 32;
  const int n_mt = g.n_rb / AF, n_nt = (nct + 7) / 8;
  // blocks that share a column tile are neighbours on one XCD
  const int total = n_mt * n_nt * g.ks, per_x = (total + 7) / 8;
  const int logical = (blockIdx.x % 8) * per_x + blockIdx.x / 8;
  if ((int)(blockIdx.x / 8) >= per_x || logical >= total) return;
  const int mt = logical % n_mt, nt = (logical / n_mt) % n_nt, z = logical / (n_mt * n_nt);
  const int n_act = s.n_act[0];
  const int per = (n_act + g.ks - 1) / g.ks, a0 = z * per;
  const int steps = max(0, min(per, n_act - a0));

  constexpr int NCH = (AF + 8) * NS;          // fragments of a step
  constexpr int NCP = (NCH + 3) / 4;          // copies per wave and step
  const float4* src[NCP];
  size_t stride[NCP];
  int dst[NCP];  // fragment slot: A slots first
#pragma unroll
  for (int i = 0; i < NCP; ++i) {
    int c = wave + 4 * i;
    if (c >= NCH) c -= NCH;
    dst[i] = c;
    if (c < AF * NS) {
      src[i] = reinterpret_cast<const float4*>(g.A) + (((size_t)a0 * g.n_rb + mt * AF) * NS + c) * 64 + lane;
      stride[i] = (size_t)g.n_rb * NS * 64;
    } else {
      const int f = c - AF * NS, ct = min(nt * 8 + f / NS, nct - 1);
      src[i] = reinterpret_cast<const float4*>(g.S) + (((size_t)a0 * nct + ct) * NS + f % NS) * 64 + lane;
      stride[i] = (size_t)nct * NS * 64;
    }
  }
  auto stage = [&](int st, L& d) {
#pragma unroll
    for (int i = 0; i < NCP; ++i) {
      float4* to = dst[i] < AF * NS ? d.a + 64 * dst[i] : d.b + 64 * (dst[i] - AF * NS);
      __builtin_amdgcn_global_load_lds((const void*)(src[i] + stride[i] * st), (lds_ptr_t)to, 16, 0, 0);
    }
  };

  f32x16 acc[AF][2];
#pragma unroll
  for (int f = 0; f < AF; ++f)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[f][0][r] = acc[f][1][r] = 0.f;

  auto compute = [&](const L& cur) {
    bf16x8 B[2][NS];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int p = 0; p < NS; ++p)
        B[c][p] = __builtin_bit_cast(bf16x8, cur.b[((2 * wave + c) * NS + p) * 64 + lane]);
#pragma unroll
    for (int f = 0; f < AF; ++f) {
      f32x16 t[2];
#pragma unroll
      for (int r = 0; r < 16; ++r) t[0][r] = t[1][r] = 0.f;
#pragma unroll
      for (int p = NS - 1; p >= 0; --p) {  // the small products first
        const bf16x8 A = __builtin_bit_cast(bf16x8, cur.a[(f * NS + p) * 64 + lane]);
#pragma unroll
        for (int q = NS - 1 - p; q >= 0; --q)
#pragma unroll
          for (int c = 0; c < 2; ++c) t[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A, B[c][q], t[c], 0, 0, 0);
      }
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[f][c][r] += t[c][r];
    }
  };
  // this wave's copies have landed and its reads are done, then everyone's
  auto barrier = [] { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
  auto one = [&](int st, const L& cur, L& nxt) {
    if (st + 1 < steps) stage(st + 1, nxt);
    compute(cur);
    __builtin_amdgcn_sched_barrier(0);
    barrier();
  };
  if (steps > 0) {
    stage(0, s0);
    barrier();
    for (int st = 0; st < steps; st += 2) {
      one(st, s0, s1);
      if (st + 1 < steps) one(st + 1, s1, s0);
    }
  }
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int ct = nt * 8 + 2 * wave + c;
    if (ct >= nct) continue;
    const int part = 32 * ct / g.nbp, b = 32 * ct - part * g.nbp + (lane & 31);
    if (b >= g.nb) continue;
#pragma unroll
    for (int f = 0; f < AF; ++f)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = g.row0 + (mt * AF + f) * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
        g.C[(((size_t)z * g.c_rows + row) * 2 + part) * g.n_bulkp + g.b0 + b] = acc[f][c][r];
      }
  }
}

template <int AF>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_pan_gemm(PanelSort s, PanelGemm g) {
  __shared__ GemmStage<AF> s0, s1;
  pan_gemm_tile<AF>(s, g, s0, s1);
}

unsigned pan_grid(const PanelSort& s, int n_task) {
  const long pa = (s.max_act + 7) / 8;  // entries per XCD at most
  return (unsigned)(8 * ((pa * n_task + 3) / 4));
}
unsigned pan_active(const PanelSort& s) { return (unsigned)s.max_act; }

}  // namespace

void pan_sort_geom(PanelSort& s) {
  // blocks of at least 1024 transitions: the scan walks one count per block
  s.nb = std::max(1, std::min(512, s.n_t / 1024));
  s.per = (s.n_t + s.nb - 1) / s.nb;
  // entries of about a 128th of the transitions, 1024 (32 steps) to 16384: the
  // FP32 sums of one entry stay within 16384 transitions, as the direct sum's do
  const int c = (s.n_t + 127) / 128;
  s.ch = std::max(1024, std::min(16384, (c + kPanStep - 1) / kPanStep * kPanStep));
  s.max_act = std::min(s.P, s.n_t) + s.n_t / s.ch + 1;
  s.cap = s.n_t / kPanStep + std::min(s.P, s.n_t) + 1;
}

void launch_pan_sort(const PanelSort& s, hipStream_t st) {
  const size_t lds = sizeof(int) * s.P;
  hipLaunchKernelGGL(k_pan_hist, dim3(s.nb), dim3(256), lds, st, s);
  hipLaunchKernelGGL(k_pan_scan, dim3(1), dim3(1024), lds, st, s);
  hipLaunchKernelGGL(k_pan_scatter, dim3(s.nb), dim3(256), lds, st, s);
}

void launch_pan_tab(const PanelSort& s, float4* T, hipStream_t st) {
  hipLaunchKernelGGL(k_pan_tab, dim3(pan_active(s), kTabSplit), dim3(256), 0, st, s, T);
}
void launch_pan_tab64(const PanelSort& s, double* T64, hipStream_t st) {
  hipLaunchKernelGGL(k_pan_tab64, dim3(pan_active(s), kTabSplit), dim3(256), 0, st, s, T64);
}

void launch_pan_pack(const PanelSort& s, const PanelPack& p, hipStream_t st) {
  const int n_tb = (s.n_t + PP_T * PP_N - 1) / (PP_T * PP_N);
  int w = p.R32 ? p.g_lo + p.ld32 : 0;
  if (p.R64) w = std::max(w, p.ld64);
  if (p.W64) w = std::max(w, p.ldw);
  if (p.A64) w = std::max(w, p.lda64);
  hipLaunchKernelGGL(k_pan_pack, dim3((unsigned)n_tb + pan_active(s), (unsigned)((w + PP_G - 1) / PP_G)),
                     dim3(256), 0, st, s, p, n_tb);
}

// tiles of G rows [g_first, g_last) that hold pairs G <= G'
static void tile_list(int n_g, int g_first, int g_last, int rows, std::vector<int>& tasks) {
  tasks.clear();
  for (int g = g_first / rows * rows; g < g_last; g += rows)
    for (int h = std::max(g, g_first) / 16 * 16; h < n_g; h += 16) {
      tasks.push_back(g);
      tasks.push_back(h);
    }
}
void pan_bin_tasks(int n_gl, int g_first, int g_last, std::vector<int>& tasks) {
  tile_list(n_gl, g_first, g_last, PB_G, tasks);
}
void pan_bin64_tasks(int n_g, int g_first, int g_last, std::vector<int>& tasks) {
  tile_list(n_g, g_first, g_last, PQ_G, tasks);
}

void launch_pan_bin(const PanelSort& s, const float4* T, const PanelBin& b, hipStream_t st) {
  // four and a half rounds of two blocks per CU at most: enough for the
  // hardware to even out the items' lengths, without the thousands of empty
  // blocks of a grid sized for the largest possible number of entries
  hipLaunchKernelGGL(k_pan_bin, dim3(std::min(2304u, pan_grid(s, b.n_task))), dim3(256), 0, st, s, T, b);
}

void launch_pan_bin64(const PanelSort& s, const double* T64, const double* X, int ldx, int n_col,
                      double* S64, int lds, hipStream_t st) {
  const int n_task = (n_col + 31) / 32;
  // where the blocks of one entry each fit a few rounds of the chip (head and
  // wings), the longest entry's chain of loads is the time: split it
  const long split = 8L * ((pan_active(s) + 7) / 8) * n_task;
  if (split <= 16384)
    hipLaunchKernelGGL(k_pan_bin64<true>, dim3((unsigned)split), dim3(256), 0, st, s, T64, X, ldx, n_task,
                       n_col, S64, lds);
  else
    hipLaunchKernelGGL(k_pan_bin64<false>, dim3(pan_grid(s, n_task)), dim3(256), 0, st, s, T64, X, ldx, n_task,
                       n_col, S64, lds);
}

void launch_pan_bin64_pairs(const PanelSort& s, const double* T64, const PanelBin64& b, hipStream_t st) {
  hipLaunchKernelGGL(k_pan_bin64_pairs, dim3(pan_grid(s, b.n_task)), dim3(256), 0, st, s, T64, b);
}

void launch_pan_coef(const PanelSort& s, const double* w, int n_w, double eta, int row0, int n_rb,
                     uint4* A, hipStream_t st) {
  const dim3 grid((unsigned)((n_rb * 64 + 255) / 256), pan_active(s));
  hipLaunchKernelGGL(k_pan_coef, grid, dim3(256), 0, st, s, w, n_w, eta, row0, n_rb, A);
}

void launch_pan_coef64(const PanelSort& s, const double* w, int n_w, double eta, int ldm, double* K,
                       hipStream_t st) {
  hipLaunchKernelGGL(k_pan_coef64, dim3((unsigned)((ldm / 2 + 255) / 256), pan_active(s)), dim3(256), 0,
                     st, s, w, n_w, eta, ldm, K);
}

int pan_gemm_blocks(const PanelGemm& g) {
  return (g.n_rb / g.af) * ((2 * g.nbp / 32 + 7) / 8);
}

// the tile height that costs least: padded rows, and per tile the operand
// columns that every tile stages again (about a third of a row block's time)
int pan_row_frags(int n_rows) {
  int best = 1;
  double cost = 1e300;
  for (int af = 5; af >= 1; --af) {
    const int rows = (n_rows + 32 * af - 1) / (32 * af) * (32 * af);
    const double c = rows * (1.0 + 0.35 / af);
    if (c < cost) {
      cost = c;
      best = af;
    }
  }
  return best;
}

void launch_pan_gemm(const PanelSort& s, const PanelGemm& g, hipStream_t st) {
  const int total = pan_gemm_blocks(g) * g.ks;
  const dim3 grid((unsigned)(8 * ((total + 7) / 8)));
  switch (g.af) {
    case 1: hipLaunchKernelGGL(k_pan_gemm<1>, grid, dim3(256), 0, st, s, g); return;
    case 2: hipLaunchKernelGGL(k_pan_gemm<2>, grid, dim3(256), 0, st, s, g); return;
    case 3: hipLaunchKernelGGL(k_pan_gemm<3>, grid, dim3(256), 0, st, s, g); return;
    case 4: hipLaunchKernelGGL(k_pan_gemm<4>, grid, dim3(256), 0, st, s, g); return;
    default: hipLaunchKernelGGL(k_pan_gemm<5>, grid, dim3(256), 0, st, s, g); return;
  }
}

}  // namespace qcx

// Response of Eq. (RPA) through energy panels (internal launchers): the
// transitions are sorted by panel, summed against the panel's Chebyshev
// functions once for all frequencies (the moments S), and the response at
// every frequency is a matrix product of the series coefficients with S.
// panel_plan.h defines the panels.
#pragma once

#include "common.h"
#include "panel_plan.h"

namespace qcx {

constexpr int kPanStep = 32;      // positions per step; panels start on a step
constexpr int kPanPlane = 16 * 2 * 3;  // bytes of the 16 terms of a moment or coefficient in its planes
constexpr int kPanMax = 8192;     // panels of both sides

// The transitions of one context in panel order (device arrays).  Panels
// that hold transitions are listed in energy order, resonant side first, as
// n_act entries of at most ch transitions each (a dense panel takes several,
// which keeps the sums of one entry short and the work even); entry a holds
// positions [32 act[a].y, 32 act[a].y + act[a].z) of panel act[a].x, the last
// one of a panel padded to whole steps.  Only the device knows n_act; the
// host sizes for max_act.
struct PanelSort {
  int n_t, P, P0;           // transitions; panels, of these resonant
  int nb, per;              // blocks of the counting sort, transitions each
  int ch, max_act;          // transitions per entry, entries at most
  const PanelDesc* desc;    // [P]
  const double* edge;       // [P0 - 1] resonant, then [P - P0 - 1] anti-resonant
  const double* dt;         // [n_t] transition energies
  int* pidx;                // [n_t] panel of each transition
  int* hist;                // [nb][P] counts, then first ranks
  int* pstart;              // [P] first step of each panel
  int* pos;                 // [n_t] position of each transition
  double* Ds;               // [32 cap] energies in panel order
  int4* act;                // [max_act] {panel, first step, transitions, 0}
  int* n_act;               // {entries, steps}
  int cap;                  // steps the arrays hold: n_t / 32 + min(P, n_t) + 1
};
void pan_sort_geom(PanelSort& s);  // nb, per, ch, max_act, cap from n_t and P
void launch_pan_sort(const PanelSort& s, hipStream_t st);

// Chebyshev functions at the sorted energies: FP32, 2 KB per step, lane l
// holding function l % 16 at the positions 8 (l / 16) .. + 7 as two float4; or
// FP64 rows T64[position][32].
void launch_pan_tab(const PanelSort& s, float4* T, hipStream_t st);
void launch_pan_tab64(const PanelSort& s, double* T64, hipStream_t st);

// Sorted copies of the pair densities R[g][t], zero in padded positions; any
// subset (null: not written).
struct PanelPack {
  const cplx* R;
  size_t ldt;
  int n_g, g_lo;        // rows of R; first row of the bulk
  float2* R32;          // [position][ld32]: R of rows g_lo .. as FP32
  int ld32;
  cplx* R64;            // [position][ld64]: R of rows 0 ..
  int ld64;
  cplx* W64;            // [position][ldw]: conj(R_0) R_g (head and wings)
  int ldw;
  double* A64;          // [position][lda64]: |R_g|^2
  int lda64;
};
void launch_pan_pack(const PanelSort& s, const PanelPack& p, hipStream_t st);

// Moments of a range of pairs (G, G') as three bf16 planes in the B-operand
// order of v_mfma_f32_32x32x16_bf16: [active][column tile of 32][plane][64 lanes][8].
// Columns: (Re, Im) part x nbp pairs (a multiple of 128), pair b of the range
// at column part * nbp + b - b0.
struct PanelBin {
  const float2* R32;
  int ld32;
  int n_gl;             // bulk rows
  const int2* tasks;    // {first G, first G'} of 8 x 16 tiles, local rows
  int n_task;
  long b0;              // first pair of the range (upper-triangle index of local rows)
  int nbp;
  uint2* S;
};
void pan_bin_tasks(int n_gl, int g_first, int g_last, std::vector<int>& tasks);
void launch_pan_bin(const PanelSort& s, const float4* T, const PanelBin& b, hipStream_t st);
// FP64 moments S64[32 active + i][lds]: of the columns of a table X[position][ldx]
// (n_col doubles, multiple of 32 readable), or of pairs (columns 2 (b - b0) + part)
void launch_pan_bin64(const PanelSort& s, const double* T64, const double* X, int ldx, int n_col,
                      double* S64, int lds, hipStream_t st);
struct PanelBin64 {
  const cplx* R64;
  int ld64, n_g;
  const int2* tasks;    // {first G, first G'} of 4 x 16 tiles
  int n_task;
  long b0;
  double* S64;
  int lds;
};
void pan_bin64_tasks(int n_g, int g_first, int g_last, std::vector<int>& tasks);
void launch_pan_bin64_pairs(const PanelSort& s, const double* T64, const PanelBin64& b, hipStream_t st);

// Series coefficients of 1 / (x_j - D + i eta), x = w (resonant panels) or -w:
// bf16 planes in the A-operand order of v_mfma_f32_32x32x16_bf16,
// [active][n_rb row blocks of 32][plane][64][8], rows row0 .. of (Re, Im) per
// frequency; or FP64 rows K[32 active + i][ldm].
void launch_pan_coef(const PanelSort& s, const double* w, int n_w, double eta, int row0, int n_rb,
                     uint4* A, hipStream_t st);
void launch_pan_coef64(const PanelSort& s, const double* w, int n_w, double eta, int ldm, double* K,
                       hipStream_t st);

// C[((z rows + row) 2 + part) n_bulkp + b] = sum over the active panels of
// split z and their 16 terms of A[row][.] S[.][col]; rows = 32 n_rb of them
// starting at row0 of the buffer, af (1 .. 5) row blocks per tile (divides n_rb)
struct PanelGemm {
  const uint4* A;
  const uint4* S;
  int n_rb, af;
  int nbp, nb;             // padded and real pairs of the range (columns: Re, then Im)
  long b0;                 // first pair of the range in C
  int ks, row0, c_rows;
  int n_bulkp;
  float* C;
};
int pan_gemm_blocks(const PanelGemm& g);  // tiles of one split
int pan_row_frags(int n_rows);  // row blocks per tile for n_rows rows
void launch_pan_gemm(const PanelSort& s, const PanelGemm& g, hipStream_t st);

// ------------------------------------------------------------ host (qcx_panel.hip)
// Buffers of a context's panel runs.
struct PanelBuf {
  DevBuf desc, ints, Ds, T, T64, R, W, S, S64, A, K, tasks;
  std::vector<DevBuf*> all() {
    return {&desc, &ints, &Ds, &T, &T64, &R, &W, &S, &S64, &A, &K, &tasks};
  }
};

// The panels of one frequency list and broadening (both sides), kept while
// the list stays the same.
struct PanelSet {
  std::vector<double> w;
  double eta = -1.0;
  bool ok = false;
  int P0 = 0;
  std::vector<char> table;  // PanelDesc[2 P0], then the edges of both sides
  bool uploaded = false;    // the owner's buffer holds the table
  void plan(const std::vector<double>& w_ha, double eta_ha);
};

// One response through panels: pair densities R[g][t] (stride ldt) with
// energies dt, frequencies w (host and device copies, Hartree), to the bulk
// partials C (FP32 / split-BF16) and the FP64 partials XY that the assembly
// reads.  pan_job_plan decides the geometry, pan_job_reserve the buffers and
// the uploads; the enqueue functions launch kernels only.
struct PanelJob {
  int n_t, n_g, n_w, prec;
  bool hw64;            // head and wings (pairs (0, G')) in FP64
  bool diag;            // only the squares |R_g|^2 (launch_diag_loss), FP64
  double eta;
  // geometry
  PanelSort s;
  bool bulk;                       // a bulk below FP64 (pairs of the rows g_lo ..)
  int g_lo, n_gl, ld32;            // bulk rows
  int n_ps64;                      // FP64 pairs (0: none)
  int ld64;
  std::vector<PanelRange> ranges, ranges64;
  std::vector<int> tasks;          // {G, G'} of all ranges, bulk then FP64
  int row_chunk;                   // row blocks of coefficients held at once
  Chi0Geom g;                      // what the assembly reads of C
  Geom64 g64;                      // and of XY
  size_t c_floats, xy_doubles;     // sizes of C and XY
};
PanelWork pan_work(const PanelJob& j);
// false: sum the transitions directly (too many panels, or the direct sum is the
// cheaper one)
// (force: whenever possible, as the remainder of a job that pays)
bool pan_job_plan(PanelJob& j, const PanelSet& set, bool force = false);
// bytes by which the buffers of a planned job would grow
size_t pan_job_grows(const PanelJob& j, const PanelSet& set, PanelBuf& b);
// reserve the buffers of a planned job and bind its device views; the caller
// then uploads desc, edge and tasks
hipError_t pan_job_reserve(PanelJob& j, const PanelSet& set, PanelBuf& b);
// sort, basis functions, FP64 coefficients; then, per list of pair densities,
// packing, moments and response
void pan_enqueue_sort(const PanelJob& j, const PanelBuf& b, const double* d_w, hipStream_t st);
void pan_enqueue_response(const PanelJob& j, const PanelBuf& b, const cplx* R, size_t ldt, const double* d_w,
                          float* C, double* XY, hipStream_t st);

}  // namespace qcx

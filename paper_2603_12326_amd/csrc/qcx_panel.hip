// Host side of the panel route of chi0 (panel.h): when it is taken, its
// geometry, buffers and launches.
#include "ctx.h"
#include "kk.h"
#include "panel.h"

namespace qcx {

namespace {
// moments S of one range of pairs, and coefficients of one range of rows
constexpr size_t kPanMoments = (size_t)4 << 30, kPanCoefs = (size_t)2 << 30;
}  // namespace

PanelWork pan_work(const PanelJob& j) {
  return {j.prec == QCX_FP64, j.prec == QCX_FP32, j.diag, j.n_t, j.n_g, j.n_w};
}

void PanelSet::plan(const std::vector<double>& w_ha, double eta_ha) {
  if (eta == eta_ha && w == w_ha) return;
  w = w_ha;
  eta = eta_ha;
  uploaded = false;
  std::vector<double> x = w_ha;
  std::sort(x.begin(), x.end());
  std::vector<double> edge, me;
  std::vector<PanelDesc> desc, md;
  ok = panel_side(x, eta, kPanMax / 2, edge, desc);
  P0 = (int)desc.size();
  if (!ok) return;
  panel_mirror(edge, desc, me, md);
  const size_t nd = P0 * sizeof(PanelDesc), ne = edge.size() * sizeof(double);
  table.resize(2 * (nd + ne));
  memcpy(table.data(), desc.data(), nd);
  memcpy(table.data() + nd, md.data(), nd);
  if (ne) {
    memcpy(table.data() + 2 * nd, edge.data(), ne);
    memcpy(table.data() + 2 * nd + ne, me.data(), ne);
  }
}

bool pan_job_plan(PanelJob& j, const PanelSet& set, bool force) {
  if (!set.ok || !(force || panels_pay(pan_work(j), set.P0))) return false;
  const int P0 = set.P0;
  PanelSort& s = j.s;
  s = PanelSort{};
  s.n_t = j.n_t;
  s.P0 = P0;
  s.P = 2 * P0;
  pan_sort_geom(s);
  if (s.max_act > 65535) return false;  // the coefficients' grid has a row per entry
  j.tasks.clear();
  j.ranges.clear();
  j.ranges64.clear();
  const bool fp64 = j.prec == QCX_FP64;
  const int parts = j.diag ? 1 : 2;
  const int n_pairs = j.diag ? j.n_g : j.n_g * (j.n_g + 1) / 2;
  Chi0Geom& g = j.g;
  g = Chi0Geom{};
  g.n_g = j.n_g;
  g.n_t = j.n_t;
  g.n_w = j.n_w;
  g.n_rows = 2 * j.n_w;
  g.n_pairs = n_pairs;
  const bool wings = !fp64 && j.hw64;
  g.p0 = fp64 ? n_pairs : wings ? j.n_g : 0;
  g.n_bulk = n_pairs - g.p0;
  g.n_bulkp = (int)roundup(std::max(g.n_bulk, 1), 128);
  g.ksplit = 1;
  j.c_floats = j.xy_doubles = 0;
  j.g_lo = wings ? 1 : 0;
  j.n_gl = j.n_g - j.g_lo;
  j.row_chunk = 0;
  j.bulk = g.n_bulk > 0;
  if (j.bulk) {
    const int af = pan_row_frags(g.n_rows);
    g.n_rowsp = (int)roundup(g.n_rows, 32 * af);
    g.c_rows = g.n_rowsp;
    j.ld32 = (int)roundup(j.n_gl, 16);
    const size_t per_pair = (size_t)s.max_act * kPanPlane * 2;  // moments of two parts
    panel_ranges(j.n_gl, kPanBinRows, (long)(kPanMoments / per_pair), false, j.ranges);
    for (PanelRange& r : j.ranges) {
      std::vector<int> t;
      pan_bin_tasks(j.n_gl, r.g0, r.g1, t);
      r.task0 = (int)j.tasks.size() / 2;
      r.n_task = (int)t.size() / 2;
      j.tasks.insert(j.tasks.end(), t.begin(), t.end());
    }
    // Splits: two blocks per CU in one round where the tiles are few, entries
    // per split within the FP32 accumulation limit of 1024 steps, and enough
    // of them for the accuracy: the rounding of the sums grows with the root of
    // the entries per split and is the largest error of this route.  The split
    // mode takes two at least (2e-7 against the direct sum's 6e-7 to 1.5e-6),
    // the FP32 mode one per 56 panels of a side and eight at least: rms error
    // of chi0 at 113 G with two | eight splits, 16,000 transitions 1.8e-7 |
    // 1.05e-7 (direct 7.2e-7), 65,536 2.1e-7 | 1.05e-7 (direct 1.5e-6); the
    // most accurate direct sum met (40 G, 64 splits) has 1.25e-7.  Where they
    // would take more than the direct sum's partials may (8 GiB) the FP32 mode
    // sums directly.
    const int tiles = (g.n_rowsp / (32 * af)) * ((2 * g.n_bulkp / 32 + 7) / 8);
    const size_t split = sizeof(float) * g.c_rows * 2 * (size_t)g.n_bulkp;
    const int least = j.prec == QCX_FP32 ? std::max(8, (P0 + 55) / 56) : 2;
    if (j.prec == QCX_FP32 && least * split > (size_t)8 << 30) return false;
    int ks = std::max(least, std::min(8, 512 / std::max(1, tiles)));
    ks = std::max(ks, (s.max_act + 1023) / 1024);
    g.ksplit = ks;
    j.c_floats = (size_t)ks * g.c_rows * 2 * g.n_bulkp;
    const size_t per_rb = (size_t)s.max_act * kPanPlane * 32;
    j.row_chunk = (int)std::max<size_t>(1, kPanCoefs / (per_rb * af)) * af;
    j.row_chunk = std::min(j.row_chunk, g.n_rowsp / 32);
  }
  j.n_ps64 = fp64 ? n_pairs : wings ? j.n_g : 0;
  if (j.n_ps64) {
    Geom64& q = j.g64;
    q = Geom64{};
    q.n_g = j.n_g;
    q.n_w = j.n_w;
    q.n_t = j.n_t;
    q.n_ps = j.n_ps64;
    q.n_rowsp = kk_ldm(j.n_w);
    q.n_colp = (int)roundup(parts * j.n_ps64, 128);
    j.ld64 = (int)roundup(j.n_g, 32);
    const size_t per_col = (size_t)s.max_act * kPanelTerms64 * sizeof(double);
    if (fp64)
      panel_ranges(j.n_g, j.diag ? 128 : kPanBin64Rows, (long)(kPanMoments / (per_col * parts)), j.diag, j.ranges64);
    else
      j.ranges64.push_back({0, j.n_g, 0, 0, 0, j.n_g, j.n_g});
    for (PanelRange& r : j.ranges64) {
      if (!fp64 || j.diag) continue;
      std::vector<int> t;
      pan_bin64_tasks(j.n_g, r.g0, r.g1, t);
      r.task0 = (int)j.tasks.size() / 2;
      r.n_task = (int)t.size() / 2;
      j.tasks.insert(j.tasks.end(), t.begin(), t.end());
    }
    const int tiles = kk_tiles(j.n_w, parts * j.n_ps64);
    int ks = std::max(1, std::min({24, 512 / std::max(1, tiles), std::max(1, P0 * 2 / 8)}));
    const size_t split = (size_t)q.n_rowsp * q.n_colp;
    while (ks > 1 && ks * split * sizeof(double) > ((size_t)512 << 20)) --ks;
    q.ksplit = ks;
    q.chunk_t = 0;
    j.xy_doubles = (size_t)ks * split;
  }
  return true;
}

// Bytes of every buffer of a job, in the order of PanelBuf::all().
static std::vector<size_t> job_bytes(const PanelJob& j, const PanelSet& set) {
  const PanelSort& s = j.s;
  const size_t pos = (size_t)s.cap * kPanStep;
  const size_t ints = 2 * (size_t)s.n_t + (size_t)s.nb * s.P + s.P + 4 * (size_t)s.max_act + 64;
  size_t r = 0, wg = 0, mom = 0, mom64 = 0;
  if (j.bulk) r = pos * j.ld32 * sizeof(float2);
  for (const PanelRange& x : j.ranges)
    mom = std::max(mom, (size_t)s.max_act * kPanPlane * 2 * x.nbp);
  for (const PanelRange& x : j.ranges64)
    mom64 = std::max(mom64, (size_t)s.max_act * kPanelTerms64 * roundup((j.diag ? 1 : 2) * x.nb, 128));
  if (j.n_ps64) wg = pos * j.ld64 * (j.diag ? sizeof(double) : sizeof(cplx));
  return {set.table.size(),
          sizeof(int) * ints,
          sizeof(double) * pos,
          j.bulk ? (size_t)s.cap * 2 * 1024 : 0,
          j.n_ps64 ? pos * kPanelTerms64 * sizeof(double) : 0,
          r,
          wg,
          mom,
          mom64 * sizeof(double),
          j.bulk ? (size_t)s.max_act * j.row_chunk * kPanPlane * 32 : 0,
          j.n_ps64 ? (size_t)s.max_act * kPanelTerms64 * kk_ldm(j.n_w) * sizeof(double) : 0,
          sizeof(int) * std::max<size_t>(1, j.tasks.size())};
}

size_t pan_job_grows(const PanelJob& j, const PanelSet& set, PanelBuf& b) {
  const std::vector<size_t> need = job_bytes(j, set);
  const std::vector<DevBuf*> bufs = b.all();
  size_t grow = 0;
  for (size_t i = 0; i < bufs.size(); ++i)
    if (need[i] + 64 > bufs[i]->bytes) grow += need[i] + 64 - bufs[i]->bytes;
  return grow;
}

hipError_t pan_job_reserve(PanelJob& j, const PanelSet& set, PanelBuf& b) {
  const std::vector<size_t> need = job_bytes(j, set);
  const std::vector<DevBuf*> bufs = b.all();
  for (size_t i = 0; i < bufs.size(); ++i)
    if (need[i]) {
      // the uploads ask for 64 bytes of slack
      const hipError_t e = bufs[i]->reserve(need[i] + 64);
      if (e != hipSuccess) return e;
    }
  PanelSort& s = j.s;
  s.desc = b.desc.as<PanelDesc>();
  s.edge = reinterpret_cast<const double*>(s.desc + s.P);
  s.Ds = b.Ds.as<double>();
  int* p = b.ints.as<int>();
  s.act = reinterpret_cast<int4*>(p);
  p += 4 * (size_t)s.max_act;
  s.n_act = p;
  p += 16;
  s.pstart = p;
  p += s.P;
  s.hist = p;
  p += (size_t)s.nb * s.P;
  s.pidx = p;
  p += s.n_t;
  s.pos = p;
  return hipSuccess;
}

void pan_enqueue_sort(const PanelJob& j, const PanelBuf& b, const double* d_w, hipStream_t st) {
  const PanelSort& s = j.s;
  launch_pan_sort(s, st);
  if (j.bulk) launch_pan_tab(s, b.T.as<float4>(), st);
  if (j.n_ps64) {
    launch_pan_tab64(s, b.T64.as<double>(), st);
    launch_pan_coef64(s, d_w, j.n_w, j.eta, kk_ldm(j.n_w), b.K.as<double>(), st);
  }
}

void pan_enqueue_response(const PanelJob& j, const PanelBuf& b, const cplx* R, size_t ldt, const double* d_w,
                          float* C, double* XY, hipStream_t st) {
  const PanelSort& s = j.s;
  const int parts = j.diag ? 1 : 2;
  PanelPack p{};
  p.R = R;
  p.ldt = ldt;
  p.n_g = j.n_g;
  p.g_lo = j.g_lo;
  if (j.bulk) {
    p.R32 = b.R.as<float2>();
    p.ld32 = j.ld32;
  }
  if (j.n_ps64) {
    if (j.diag) {
      p.A64 = b.W.as<double>();
      p.lda64 = j.ld64;
    } else if (j.prec != QCX_FP64) {
      p.W64 = b.W.as<cplx>();
      p.ldw = j.ld64;
    } else {
      p.R64 = b.W.as<cplx>();
      p.ld64 = j.ld64;
    }
  }
  launch_pan_pack(s, p, st);
  const int2* tasks = b.tasks.as<int2>();
  if (j.bulk) {
    const int n_rb = j.g.n_rowsp / 32;
    bool coefs = false;  // one range of rows: its coefficients serve every range of pairs
    for (const PanelRange& r : j.ranges) {
      PanelBin pb{};
      pb.R32 = b.R.as<float2>();
      pb.ld32 = j.ld32;
      pb.n_gl = j.n_gl;
      pb.tasks = tasks + r.task0;
      pb.n_task = r.n_task;
      pb.b0 = r.b0;
      pb.nbp = r.nbp;
      pb.S = b.S.as<uint2>();
      launch_pan_bin(s, b.T.as<float4>(), pb, st);
      for (int rb0 = 0; rb0 < n_rb; rb0 += j.row_chunk) {
        PanelGemm q{};
        q.A = b.A.as<uint4>();
        q.S = b.S.as<uint4>();
        q.n_rb = std::min(j.row_chunk, n_rb - rb0);
        q.af = pan_row_frags(j.g.n_rows);
        q.nbp = r.nbp;
        q.nb = r.nb;
        q.b0 = r.b0;
        q.ks = j.g.ksplit;
        q.row0 = 32 * rb0;
        q.c_rows = j.g.n_rowsp;
        q.n_bulkp = j.g.n_bulkp;
        q.C = C;
        if (!coefs || j.row_chunk < n_rb)
          launch_pan_coef(s, d_w, j.n_w, j.eta, 32 * rb0, q.n_rb, b.A.as<uint4>(), st);
        coefs = true;
        launch_pan_gemm(s, q, st);
      }
    }
  }
  for (const PanelRange& r : j.ranges64) {
    const int cols = parts * r.nb, lds = (int)roundup(cols, 128);
    double* S64 = b.S64.as<double>();
    if (j.prec != QCX_FP64) {
      launch_pan_bin64(s, b.T64.as<double>(), b.W.as<double>(), 2 * j.ld64, cols, S64, lds, st);
    } else if (j.diag) {
      launch_pan_bin64(s, b.T64.as<double>(), b.W.as<double>() + r.g0, j.ld64, cols, S64, lds, st);
    } else {
      PanelBin64 pb{};
      pb.R64 = b.W.as<cplx>();
      pb.ld64 = j.ld64;
      pb.n_g = j.n_g;
      pb.tasks = tasks + r.task0;
      pb.n_task = r.n_task;
      pb.b0 = r.b0;
      pb.S64 = S64;
      pb.lds = lds;
      launch_pan_bin64_pairs(s, b.T64.as<double>(), pb, st);
    }
    const Geom64& q = j.g64;
    launch_kk_transform({b.K.as<double>(), kk_ldm(j.n_w), S64, lds, cols, kPanelTerms64, s.n_act, 2 * j.n_w,
                         q.ksplit, XY + parts * r.b0, q.n_colp, (size_t)q.n_rowsp * q.n_colp},
                        st);
  }
}

}  // namespace qcx

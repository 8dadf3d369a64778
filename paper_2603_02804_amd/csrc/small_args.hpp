// small_args.hpp -- argument records of the coefficient, assembly and
// reduction kernels, the host code that fills them from a plan, and the job
// records of merged mixed-batch launches.
#pragma once
#include <stdint.h>

#include <algorithm>

#include "kargs.hpp"

namespace qf {

// Coefficient rows: the 2x2 matrix of a gate (per-gate paths), or the RZ RY RZ split
// with the RY as shears or as a scaled rotation (see apply_rot in device.hpp).
enum RunForm : int { kFormMatrix = 0, kFormShear = 1, kFormScaled = 2 };
inline int run_form(int R) { return R <= 4 ? kFormScaled : kFormShear; }

// Least cosine of a scaled rotation: t = tan f stays below 2^25 and the growth of four
// below 2^100.  The cosine moves by less than half an ulp of 1, the rounding of the
// rotated amplitudes.
constexpr double kMinCos = 1.0 / (1 << 25);
// Rows of the epoch tables whose scales' roundings carry over to the next (see table_body).
constexpr int kCarryRows = 8;

// Coefficient, reduction and gradient arguments carry the real type of the call:
// float on the fused and per-gate paths, double on the complex128 validation path.
template <class Real>
struct CoefArgsT {
  Tabs T;
  const Real* theta;
  const Real* x;
  Real* csh;
  Real* cps;
  double* dsh;     // shared runs' double rows (fused paths)
  int F, n_sh, n_ps, B;
  int form;        // row format: RunForm
};
using CoefArgs = CoefArgsT<float>;

struct EventArgs {
  Tabs T;
  const TabRec* trecs;
  const ThrBase* tbases;
  const TabEvent* tevs;
  const CzGroup* czg;
  const int32_t* tcor;
  const double* dsh;
  float* tab;
  float* tco;
  double* gvec;    // or null: no backward follows
  const float* theta;
  int n_tab, NT, form, n_sh;
  const float* csh;
  const float* cps;
  float* esh;
  float* eps;
  int n_ev_sh, n_ev_ps, B, n_ps;
};

template <class Real>
struct ReduceEArgsT {
  const Real* partE;
  Real* E;
  int nb, sample0, parts, K;
  int wide;        // a workgroup per sample instead of a thread per sum
};
using ReduceEArgs = ReduceEArgsT<float>;

// Column sums of the functionals of passes [p0, p0 + np) in chunks of their rows.
struct FsumArgs {
  Tabs T;
  const float* partF;
  double* fsum;
  int p0, np, nb, tiles, groups, chunks;
};

struct AssembleArgs {
  Tabs T;
  const float* theta;
  const float* x;
  const float* partF;
  const double* fsum;
  const double* gvec;
  float* Gr;
  int p0, np, nb, sample0, tiles, n_angle, F;
  int groups;      // workgroups per pass for the shared runs (kAssembleRuns each)
  int chunks;      // partial sums of fsum, 0: the rows of partF
  int ps0, nps;    // entries of T.ps_pass in the segment
};

template <class Real>
struct ReduceGArgsT {
  Tabs T;
  const Real* Gr;
  Real* dtheta;
  Real* dx;
  int nb, sample0, n_angle, P, F, accumulate;
  // dtheta blocks: each sums cols angles over the micro-batch with kSmallThreads / cols
  // sample lanes (lane j takes samples j, j + lanes, ...), then a fixed tree over the lanes
  int cols, th_blocks;
  // (the dx pointer of a mixed batch is only known at call time: items are counted regardless)
  long long dx_items() const { return (long long)nb * F; }
};
using ReduceGArgs = ReduceGArgsT<float>;

constexpr int kSmallThreads = 256;

inline unsigned blocks_for(long long n, int t = kSmallThreads) {
  return (unsigned)std::max<long long>(1, (n + t - 1) / t);
}

template <class Real>
inline CoefArgsT<Real> make_coef_args_t(const PlanCore& c, const PlanPtrs& d, const Real* theta, const Real* x,
                                        Real* csh, Real* cps, double* dsh = nullptr) {
  CoefArgsT<Real> a;
  a.T = d.tabs;
  a.theta = theta;
  a.x = x;
  a.csh = csh;
  a.cps = cps;
  a.F = c.C.F;
  a.n_sh = c.S.n_coef_shared;
  a.n_ps = c.S.n_coef_ps;
  a.B = c.B;
  a.dsh = dsh;
  a.form = c.per_gate ? kFormMatrix : run_form(c.S.R);
  return a;
}

inline CoefArgs make_coef_args(const PlanCore& c, const PlanPtrs& d, const float* theta, const float* x,
                               const CoefPtrs& cp) {
  return make_coef_args_t<float>(c, d, theta, x, const_cast<float*>(cp.csh), const_cast<float*>(cp.cps),
                                 cp.dsh);
}

template <class Real>
inline long long coef_items(const CoefArgsT<Real>& a) { return a.n_sh + (long long)a.n_ps * a.B; }

inline EventArgs make_event_args(const PlanCore& c, const PlanPtrs& d, const CoefPtrs& cp, const float* theta) {
  EventArgs a;
  a.T = d.tabs;
  a.trecs = d.trecs;
  a.tbases = d.tbases;
  a.tevs = d.tevs;
  a.czg = d.czg;
  a.tcor = d.tcor;
  a.dsh = cp.dsh;
  a.tab = cp.tab;
  a.tco = cp.tco;
  a.n_tab = (int)c.S.tabs.size();
  a.NT = c.S.NT;
  a.form = run_form(c.S.R);
  a.gvec = cp.gvec;
  a.theta = theta;
  a.n_sh = c.S.n_coef_shared;
  a.csh = cp.csh;
  a.cps = cp.cps;
  a.esh = const_cast<float*>(cp.esh);
  a.eps = const_cast<float*>(cp.eps);
  a.n_ev_sh = c.S.n_ev_shared;
  a.n_ev_ps = c.S.n_ev_ps;
  a.B = c.B;
  a.n_ps = c.S.n_coef_ps;
  return a;
}

// Phase events, then (each from the next whole block) one thread per entry of the epoch
// tables and one per shared run, for its gates' generators.
inline long long event_rows(const EventArgs& a) { return a.n_ev_sh + (long long)a.n_ev_ps * a.B; }
inline long long event_blocks(const EventArgs& a) {
  const long long tab = (long long)a.n_tab * a.NT;
  return (event_rows(a) + kSmallThreads - 1) / kSmallThreads + (tab + kSmallThreads - 1) / kSmallThreads +
         (a.gvec ? (a.n_sh + kSmallThreads - 1) / kSmallThreads : 0);
}

template <class Real>
inline ReduceEArgsT<Real> make_reduce_E_args(const PlanCore& c, int nb, int sample0, int parts, const Real* partE,
                                             Real* E) {
  ReduceEArgsT<Real> a;
  a.partE = partE;
  a.E = E;
  a.nb = nb;
  a.sample0 = sample0;
  a.parts = parts;
  a.K = c.C.K;
  // few partial sums: a thread each keeps many samples in one workgroup (65,536 samples of
  // 9 qubits); many: 1,024 of a 20-qubit sample took 305 us as one serial chain per thread
  a.wide = parts > 16 ? 1 : 0;
  return a;
}
// (a circuit without observables: one idle workgroup, an empty grid is a launch error)
template <class Real>
inline long long reduce_E_blocks(const ReduceEArgsT<Real>& a) {
  return a.wide ? a.nb : (long long)blocks_for((long long)a.nb * a.K);
}

inline FsumArgs make_fsum_args(const PlanCore& c, const PlanPtrs& d, int seg, int nb, const float* partF,
                               double* fsum) {
  FsumArgs a;
  a.T = d.tabs;
  a.partF = partF;
  a.fsum = fsum;
  a.p0 = c.seg_begin[seg];
  a.np = c.seg_begin[seg + 1] - a.p0;
  a.nb = nb;
  a.tiles = c.tiles;
  a.groups = c.fsum_groups;
  a.chunks = c.fsum_chunks;
  return a;
}
inline long long fsum_blocks(const FsumArgs& a) { return (long long)a.np * a.groups * a.chunks; }

constexpr int kAssembleRuns = 21;   // runs per workgroup: 63 columns of functionals

inline AssembleArgs make_assemble_args(const PlanCore& c, const PlanPtrs& d, int seg, int nb, int sample0,
                                       const float* theta, const float* x, const float* partF, const double* fsum,
                                       const double* gvec, float* Gr) {
  AssembleArgs a;
  a.T = d.tabs;
  a.theta = theta;
  a.x = x;
  a.partF = partF;
  a.Gr = Gr;
  a.p0 = c.seg_begin[seg];
  a.np = c.seg_begin[seg + 1] - a.p0;
  a.nb = nb;
  a.sample0 = sample0;
  a.tiles = c.tiles;
  a.n_angle = c.n_angle;
  a.F = c.C.F;
  a.fsum = fsum;
  a.gvec = gvec;
  a.groups = (c.S.max_slots + kAssembleRuns - 1) / kAssembleRuns;
  a.chunks = c.fsum_chunks;
  const auto lo = std::lower_bound(c.ps_pass.begin(), c.ps_pass.end(), a.p0);
  a.ps0 = (int)(lo - c.ps_pass.begin());
  a.nps = (int)(std::lower_bound(lo, c.ps_pass.end(), a.p0 + a.np) - lo);
  return a;
}
inline long long assemble_blocks(const AssembleArgs& a) {
  return (long long)a.np * a.groups + (long long)a.nb * a.nps;
}

template <class Real>
inline ReduceGArgsT<Real> make_reduce_grads_args(const PlanCore& c, const PlanPtrs& d, int nb, int sample0,
                                                 const Real* Gr, Real* dtheta, Real* dx, bool accumulate) {
  ReduceGArgsT<Real> a;
  a.T = d.tabs;
  a.Gr = Gr;
  a.dtheta = dtheta;
  a.dx = dx;
  a.nb = nb;
  a.sample0 = sample0;
  a.n_angle = c.n_angle;
  a.P = c.C.P;
  a.F = c.C.F;
  a.accumulate = accumulate ? 1 : 0;
  // wide blocks of angles when there are many (coalesced rows of Gr), more sample
  // lanes per angle when there are few
  int cols = 1;
  while (cols < 64 && cols < a.P) cols *= 2;
  // per-sample runs are added over the samples here: at most 64 per lane if the block allows
  if (!c.ps_runs.empty() || c.per_gate)
    while (cols > 1 && (long long)nb * cols > 64ll * kSmallThreads) cols /= 2;
  a.cols = cols;
  a.th_blocks = (a.P + cols - 1) / cols;
  return a;
}

// Blocks of kSmallThreads threads: th_blocks for dtheta, then one thread per
// (sample, input) for dx.
template <class Real>
inline long long reduce_grads_blocks(const ReduceGArgsT<Real>& a) {
  const long long nx = a.dx_items();
  return (long long)a.th_blocks + (nx + kSmallThreads - 1) / kSmallThreads;
}
// LDS of the reduction kernels: one double per thread.
inline size_t reduce_shmem() { return sizeof(double) * kSmallThreads; }

// ---------------------------------------------------------------- mixed batches
// Caller buffers of one circuit of a mixed batch, refreshed on every call.
struct CircPtrs {
  const float* theta;
  const float* x;
  float* E;
  const float* dE;
  float* dtheta;
  float* dx;
};

// A pass launch of one circuit inside a merged launch.  Workspace addresses are
// stored as offsets from the batch workspace base (never 0: the first bytes of
// the workspace are reserved), null stays null; dE comes from CircPtrs.
struct PassJob {
  KArgs A;
  int32_t circ;
  int32_t pass;       // pass index in the circuit's plan (host checks only)
};

enum SmallKind : int32_t { SJ_COEF = 0, SJ_EVENT = 1, SJ_REDUCE_E = 2, SJ_ASSEMBLE = 3, SJ_REDUCE_G = 4,
                           SJ_FSUM = 5 };

// A small-kernel launch of one circuit inside a merged launch: same address
// convention; theta, x, E, dtheta and dx come from CircPtrs.
struct SmallJob {
  int32_t kind;
  int32_t circ;
  union {
    CoefArgs coef;
    EventArgs ev;
    ReduceEArgs re;
    AssembleArgs as;
    FsumArgs fs;
    ReduceGArgs rg;
  } u;
};

}  // namespace qf

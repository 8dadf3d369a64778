// small_kernels.hpp -- device code of the coefficient, gradient-assembly and
// reduction kernels (the 2x2 run algebra in double precision), shared by the
// single-plan kernels, the merged mixed-batch kernels and the complex128
// validation path.
#pragma once
#include <hip/hip_runtime.h>

#include "small_args.hpp"

namespace qf {

struct D2 {
  double r[4], i[4];   // row-major 2x2 complex
};

__device__ inline D2 d2_mul(const D2& a, const D2& b) {
  D2 c;
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      double re = 0, im = 0;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        re += a.r[2 * r + k] * b.r[2 * k + q] - a.i[2 * r + k] * b.i[2 * k + q];
        im += a.r[2 * r + k] * b.i[2 * k + q] + a.i[2 * r + k] * b.r[2 * k + q];
      }
      c.r[2 * r + q] = re;
      c.i[2 * r + q] = im;
    }
  return c;
}

__device__ inline D2 d2_eye() {
  D2 u;
  for (int i = 0; i < 4; ++i) u.r[i] = u.i[i] = 0;
  u.r[0] = u.r[3] = 1;
  return u;
}

__device__ inline D2 d2_rot(int kind, double phi) {
  double s, c;
  sincos(0.5 * phi, &s, &c);
  D2 u;
  for (int i = 0; i < 4; ++i) u.r[i] = u.i[i] = 0;
  if (kind == QF_RX) { u.r[0] = c; u.i[1] = -s; u.i[2] = -s; u.r[3] = c; }
  else if (kind == QF_RY) { u.r[0] = c; u.r[1] = -s; u.r[2] = s; u.r[3] = c; }
  else { u.r[0] = c; u.i[0] = -s; u.r[3] = c; u.i[3] = s; }
  return u;
}

__device__ inline D2 d2_pauli(int kind) {
  D2 p;
  for (int i = 0; i < 4; ++i) p.r[i] = p.i[i] = 0;
  if (kind == QF_RX) { p.r[1] = 1; p.r[2] = 1; }
  else if (kind == QF_RY) { p.i[1] = -1; p.i[2] = 1; }
  else { p.r[0] = 1; p.r[3] = -1; }
  return p;
}

__device__ inline D2 d2_dag(const D2& a) {
  D2 d;
  d.r[0] = a.r[0]; d.i[0] = -a.i[0];
  d.r[1] = a.r[2]; d.i[1] = -a.i[2];
  d.r[2] = a.r[1]; d.i[2] = -a.i[1];
  d.r[3] = a.r[3]; d.i[3] = -a.i[3];
  return d;
}

template <class Real>
__device__ inline double gate_angle(const Tabs& T, const GateRec& g, const Real* theta, const Real* x, int F,
                                    int sample) {
  if (g.theta_idx <= -2) return T.consts[-2 - g.theta_idx];   // fixed angle of an internal gate
  return g.theta_idx >= 0 ? (double)theta[g.theta_idx] : (double)x[(size_t)sample * F + g.input_idx];
}

// RZ(a) RY(b) RZ(c) split of an SU(2) matrix V (V00 = e^{-i(a+c)/2} cos(b/2),
// V10 = e^{i(a-c)/2} sin(b/2)).  Returns cos(b/2), sin(b/2), u = e^{-ia/2},
// v = e^{-ic/2} and z = u^2 = e^{-ia}.
struct ZYZ {
  double cb, sb, ur, ui, vr, vi, zr, zi;
};

__device__ inline ZYZ zyz_split(const D2& V) {
  ZYZ o;
  const double a0 = sqrt(V.r[0] * V.r[0] + V.i[0] * V.i[0]);
  const double b0 = sqrt(V.r[2] * V.r[2] + V.i[2] * V.i[2]);
  const double nrm = sqrt(a0 * a0 + b0 * b0);
  o.cb = a0 / nrm;
  o.sb = b0 / nrm;
  double Ar = 1, Ai = 0, Br = 1, Bi = 0;
  if (a0 > 1e-300) { Ar = V.r[0] / a0; Ai = V.i[0] / a0; }
  if (b0 > 1e-300) { Br = V.r[2] / b0; Bi = V.i[2] / b0; }
  // b = 0 or pi leaves only a + c or a - c given: c = 0.  A run of RY gates followed by RZ
  // gates then has its whole RZ in a for every angle, which its missing X functional needs
  // (kEpochNoX): shared out evenly, RY(0) RZ(1.1) had 0.1294 for a gradient of 0.2499.
  if (b0 <= 1e-300) { Br = Ar; Bi = -Ai; }
  if (a0 <= 1e-300) { Ar = Br; Ai = -Bi; }
  o.zr = Ar * Br + Ai * Bi;        // A conj(B)
  o.zi = Ai * Br - Ar * Bi;
  // u = e^{i arg(z) / 2}, arg in (-pi, pi], by half angles of the unit z
  double s, c;
  if (o.zr >= 0) {
    c = sqrt(0.5 * (1.0 + o.zr));
    s = o.zi / (2.0 * c);
  } else {
    const double m = sqrt(0.5 * (1.0 - o.zr));
    c = fabs(o.zi) / (2.0 * m);
    s = copysign(m, o.zi);
  }
  o.ur = c;
  o.ui = s;
  o.vr = Ar * c + Ai * s;          // A conj(u)
  o.vi = Ai * c - Ar * s;
  return o;
}

template <class Real>
__device__ inline D2 run_matrix(const Tabs& T, const RunRec& rr, const Real* theta, const Real* x, int F,
                                int sample) {
  D2 U = d2_eye();
  for (int i = 0; i < rr.gate_count; ++i) {
    const GateRec g = T.gates[T.run_gates[rr.gate_begin + i]];
    U = d2_mul(d2_rot(g.kind, gate_angle(T, g, theta, x, F, sample)), U);
  }
  return U;
}

// Run coefficients, f = b/2 of the RZ(a) RY(b) RZ(c) split.
//   kFormShear   [cos f, sin f, u, v, tan(f/2), 0]
//   kFormScaled  [cos f, sin f, u, v, t = tan f, tan(f/2)]
//   kFormMatrix  the 2x2 matrix row-major (one-gate runs of the per-gate paths)
// Shared runs of the split forms also leave as doubles (dsh) u, v and the scale that
// an unscaled rotation owes: 1/sqrt(1 + t^2) of the float t, so that no norm is lost.
template <class Real>
__device__ inline void coef_body(const CoefArgsT<Real>& a, long long idx) {
  if (idx >= a.n_sh + (long long)a.n_ps * a.B) return;
  int r, sample;
  Real* out;
  if (idx < a.n_sh) {
    r = a.T.coef_runs_sh[idx];
    sample = 0;
    out = a.csh + 8 * idx;
  } else {
    const long long j = idx - a.n_sh;
    sample = (int)(j / a.n_ps);
    const int i = (int)(j - (long long)sample * a.n_ps);
    r = a.T.coef_runs_ps[i];
    out = a.cps + 8 * j;
  }
  const D2 U = run_matrix(a.T, a.T.runs[r], a.theta, a.x, a.F, sample);
  if (a.form != kFormMatrix) {
    const ZYZ z = zyz_split(U);
    // f in [0, pi/2]
    double scale = 1.0;
    Real t, half = 0;
    if (a.form == kFormScaled) {
      half = (Real)(z.sb / (1.0 + z.cb));
      t = (Real)(z.sb / fmax(z.cb, kMinCos));
      scale = 1.0 / sqrt(1.0 + (double)t * (double)t);
    } else {
      t = (Real)(z.sb / (1.0 + z.cb));
    }
    out[0] = (Real)z.cb; out[1] = (Real)z.sb;
    out[2] = (Real)z.ur; out[3] = (Real)z.ui;
    out[4] = (Real)z.vr; out[5] = (Real)z.vi;
    out[6] = t;
    out[7] = half;
    if (idx < a.n_sh) {
      double* d = a.dsh + kDshRow * idx;
      d[0] = z.ur; d[1] = z.ui;
      d[2] = z.vr; d[3] = z.vi;
      d[4] = scale;
    }
  } else {
    for (int i = 0; i < 4; ++i) {
      out[2 * i] = (Real)U.r[i];
      out[2 * i + 1] = (Real)U.i[i];
    }
  }
}

// The factor of a shared phase event, u(prev run) * v(next run) from the double rows,
// rounded once.
__device__ inline float2 shared_event(const double* dsh, const EventRec& e) {
  double wr = 1.0, wi = 0.0;
  const int ref[2] = {e.prev_ref, e.next_ref};
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    if (ref[k] == INT32_MIN) continue;
    const double* d = dsh + kDshRow * (long long)ref[k] + 2 * k;
    const double tr = wr * d[0] - wi * d[1];
    wi = wr * d[1] + wi * d[0];
    wr = tr;
  }
  return make_float2((float)wr, (float)wi);
}

// The scale that a row of the epoch tables owes: of its shared runs' rotations, and of
// the rounded norms of the shared phases that the pass kernel applies itself.  left: the
// product of their cosines, rounded as the pass kernel compares it.
__device__ inline bool turns_twice(double left) { return (float)left < 1.f / kMaxGrowth; }
__device__ inline double row_scale(const EventArgs& a, const TabRec* r, double* left) {
  double scale = 1.0;
#pragma unroll
  for (int j = 0; j < kMaxR; ++j)
    if (r->ref[j] != INT32_MIN) scale *= a.dsh[kDshRow * (long long)r->ref[j] + 4];
  *left = scale;
  if (turns_twice(scale)) {   // 1/(1 + h^2) of h = tan(f/2) each
    double halves = 1.0;
    for (int j = 0; j < kMaxR; ++j)
      if (r->ref[j] != INT32_MIN) {
        const double h = a.csh[8 * (long long)r->ref[j] + 7];
        halves *= 1.0 + h * h;
      }
    scale = 1.0 / halves;
  }
  for (int i = 0; i < r->cor_count; ++i) {
    const float2 w = shared_event(a.dsh, a.T.events[a.tcor[r->cor_first + i]]);
    scale /= sqrt((double)w.x * w.x + (double)w.y * w.y);
  }
  return scale;
}

// One entry of the epoch tables (TabRec): the factor that thread t of the row's layout
// owes when the epoch's exchange sends its amplitudes, formed in double precision and
// rounded once; and, by the first threads, the row's run coefficients.  The
// scale's own rounding would change all amplitudes alike, with the same sign in many rows
// (1/sqrt(2) of a CNOT's quarter turn: -1.7e-8): every row also owes what that of the rows
// before it left, from the last multiple of kCarryRows on.  A workgroup's rows lie in one
// such window; its first threads form the window's scales and, behind them in scales, the
// products of cosines.
__device__ inline void table_body(const EventArgs& a, int blk, int thread, double* scales) {
  const long long idx = (long long)blk * kSmallThreads + thread;
  const int row = (int)(idx / a.NT), t = (int)(idx - (long long)row * a.NT);
  const int window = (int)((long long)blk * kSmallThreads / a.NT) / kCarryRows * kCarryRows;
  if (thread < kCarryRows && window + thread < a.n_tab)
    scales[thread] = row_scale(a, a.trecs + window + thread, scales + kCarryRows + thread);
  __syncthreads();
  if (row >= a.n_tab) return;
  const TabRec* r = a.trecs + row;
  const uint32_t x = a.tbases[(size_t)r->layout * a.NT + t].log;
  uint32_t par = 0;
  for (int i = 0; i < r->czg_count; ++i) {
    const CzGroup g = a.czg[r->czg_first + i];
    par ^= x & (x >> g.shift) & g.mask;
  }
  double wr = __popc(par) & 1 ? -1.0 : 1.0, wi = 0.0;
  // four events at a time: their records are read together, then their factors
  for (int i0 = 0; i0 < r->tev_count; i0 += 4) {
    TabEvent e[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) e[i] = a.tevs[r->tev_first + min(i0 + i, r->tev_count - 1)];
    double f[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool on = i0 + i < r->tev_count, u = on && e[i].prev_ref != INT32_MIN, v = on && e[i].next_ref != INT32_MIN;
      const double* du = a.dsh + kDshRow * (long long)(u ? e[i].prev_ref : 0);
      const double* dv = a.dsh + kDshRow * (long long)(v ? e[i].next_ref : 0) + 2;
      f[i][0] = u ? du[0] : 1.0;
      f[i][1] = u ? du[1] : 0.0;
      f[i][2] = v ? dv[0] : 1.0;
      f[i][3] = v ? dv[1] : 0.0;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      // conjugate where the event's qubit is 1
      const double c = (x >> e[i].q) & 1 ? -1.0 : 1.0;
#pragma unroll
      for (int k = 0; k < 4; k += 2) {
        const double ur = f[i][k], ui = c * f[i][k + 1];
        const double tr = wr * ur - wi * ui;
        wi = wr * ui + wi * ur;
        wr = tr;
      }
    }
  }
  // (the scale itself is rounded before it turns, so that its remainder is known)
  double carry = 1.0, scale = 1.0;
  for (int q = window; q <= row; ++q) {
    const double owed = carry * scales[q - window];
    scale = (double)(float)owed;
    carry = owed / scale;
  }
  a.tab[2 * idx] = (float)(scale * wr);
  a.tab[2 * idx + 1] = (float)(scale * wi);
  if (t < kTabCoefs) {
    const int j = t & 7;
    const bool present = j < kMaxR && r->ref[j] != INT32_MIN;
    const double left = scales[kCarryRows + row - window];
    float v = present ? a.csh[8 * (long long)r->ref[j] + (t >= kTabSine ? 1 : turns_twice(left) ? 7 : 6)] : 0.f;
    if (t == kTabLeft && a.form == kFormScaled) v = (float)left;
    a.tco[(long long)row * kTabCoefs + t] = v;
  }
}

// Gradients of the gates of run r from the functionals F = Im<lambda|P_q|psi>
// (P = X, Y, Z) taken at the cut right after the run's RY (zyz = 1) or right
// after the whole run (zyz = 0).  dL/dtheta_g = 1/2 Im<lambda|G|psi>, with G the
// generator of gate g carried to the cut: G = K P_g K^dagger (K = gates of the
// run after g), conjugated by RZ(a)^dagger for the zyz cut.  Writing
// G = n_x X + n_y Y + n_z Z gives dL/dtheta_g = 1/2 (n . F).
//
// run_generators calls put(gate's out_idx, 1/2 n) for every gate of the run.
template <class Real, class Put>
__device__ inline void run_generators(const Tabs& T, int r, const Real* theta, const Real* x, int F, int sample,
                                      int zyz, Put put) {
  const RunRec rr = T.runs[r];
  double zr = 1, zi = 0;
  if (zyz) {
    const ZYZ z = zyz_split(run_matrix(T, rr, theta, x, F, sample));
    zr = z.zr;
    zi = z.zi;
  }
  D2 K = d2_eye();
  for (int i = rr.gate_count - 1; i >= 0; --i) {
    const GateRec g = T.gates[T.run_gates[rr.gate_begin + i]];
    const D2 G = d2_mul(d2_mul(K, d2_pauli(g.kind)), d2_dag(K));
    put(g.out_idx, 0.5 * (zr * G.r[2] - zi * G.i[2]), 0.5 * (zr * G.i[2] + zi * G.r[2]), 0.5 * G.r[0]);
    K = d2_mul(K, d2_rot(g.kind, gate_angle(T, g, theta, x, F, sample)));
  }
}

template <class Real>
__device__ inline void run_grads(const Tabs& T, int r, const Real* theta, const Real* x, int F, int sample,
                                 double fx, double fy, double fz, Real* Grow, int zyz) {
  run_generators(T, r, theta, x, F, sample, zyz, [&](int g, double nx, double ny, double nz) {
    Grow[g] = (Real)(nx * fx + ny * fy + nz * fz);
  });
}

// The generators of a shared run's gates, once per call.
__device__ inline void gvec_body(const EventArgs& a, int idx) {
  if (idx >= a.n_sh) return;
  // (a shared run has no input angles: the inputs are never read)
  run_generators(a.T, a.T.coef_runs_sh[idx], a.theta, a.theta, 0, 0, 1,
                 [&](int g, double nx, double ny, double nz) {
                   double* o = a.gvec + 3ll * g;
                   o[0] = nx;
                   o[1] = ny;
                   o[2] = nz;
                 });
}

// Phase event coefficients w = u(prev run) * v(next run); the blocks after the events'
// form the epoch tables.
__device__ inline void event_body(const EventArgs& a, int blk, int thread, double* red) {
  const long long rows = a.n_ev_sh + (long long)a.n_ev_ps * a.B;
  const int ev_blocks = (int)((rows + kSmallThreads - 1) / kSmallThreads);
  if (blk >= ev_blocks) {
    const int tab_blocks = (int)(((long long)a.n_tab * a.NT + kSmallThreads - 1) / kSmallThreads);
    blk -= ev_blocks;
    if (blk < tab_blocks) table_body(a, blk, thread, red);
    else gvec_body(a, (blk - tab_blocks) * kSmallThreads + thread);
    return;
  }
  const long long idx = (long long)blk * kSmallThreads + thread;
  if (idx >= rows) return;
  if (idx < a.n_ev_sh) {
    const float2 w = shared_event(a.dsh, a.T.events[idx]);
    a.esh[2 * idx] = w.x;
    a.esh[2 * idx + 1] = w.y;
    return;
  }
  const long long j = idx - a.n_ev_sh;
  const int sample = (int)(j / a.n_ev_ps);
  const EventRec e = a.T.events[a.n_ev_sh + (int)(j - (long long)sample * a.n_ev_ps)];
  float* out = a.eps + 2 * j;
  auto row = [&](int ref) {
    return ref >= 0 ? a.csh + 8 * (long long)ref : a.cps + 8 * ((long long)sample * a.n_ps + (-1 - ref));
  };
  float wr = 1.f, wi = 0.f;
  if (e.prev_ref != INT32_MIN) {
    const float* p = row(e.prev_ref);
    const float ur = p[2], ui = p[3];
    const float tr = wr * ur - wi * ui, ti = wr * ui + wi * ur;
    wr = tr; wi = ti;
  }
  if (e.next_ref != INT32_MIN) {
    const float* p = row(e.next_ref);
    const float vr = p[4], vi = p[5];
    const float tr = wr * vr - wi * vi, ti = wr * vi + wi * vr;
    wr = tr; wi = ti;
  }
  out[0] = wr;
  out[1] = wi;
}

// Sum of the four lanes of a column (thread 64 lane + column) in a fixed order, valid
// in lane 0's threads; red: kSmallThreads doubles of LDS.
__device__ inline double lane_sum4(double acc, int t, double* red) {
  __syncthreads();
  red[t] = acc;
  __syncthreads();
  return t < 64 ? (red[t] + red[t + 64]) + (red[t + 128] + red[t + 192]) : 0.0;
}

// The gradient of a shared run's gate is linear in the functionals, with the same
// generator for every sample: the functionals are added over samples and tiles first,
// and the 2x2 algebra runs once per gate instead of once per gate and sample.  Bound by
// reading the functionals once.  When per-sample gradients were formed and added by one
// workgroup per group of angles, 65,536 samples of a 9-qubit layer took 3.8 ms of a 5.3 ms
// step (now 1.1 ms in all), and 12 qubits x 100 layers x 1,024 samples 200 us of 3.1 ms.
//
// Column sums: workgroup (pass, 64 columns, chunk of rows), four row lanes per column.
__device__ inline void fsum_body(const FsumArgs& a, int blk, int t, double* red) {
  const int c = blk % a.chunks, q = blk / a.chunks;
  const int g = q % a.groups, p = a.p0 + q / a.groups;
  const int ncol = 3 * a.T.passes[p].n_slots, col = g * 64 + (t & 63);
  if (g * 64 >= ncol) return;
  const long long rows = (long long)a.nb * a.tiles;
  const long long r1 = rows * (c + 1) / a.chunks;
  const float* base = a.partF + (long long)a.nb * a.T.partF_off[p];
  double acc = 0;
  if (col < ncol) {
#pragma unroll 8
    for (long long r = rows * c / a.chunks + (t >> 6); r < r1; r += 4) acc += base[r * ncol + col];
  }
  acc = lane_sum4(acc, t, red);
  if (t < 64 && col < ncol) {
    const int rb0 = a.T.pass_run_begin[a.p0];
    const long long stride = 3ll * (a.T.pass_run_begin[a.p0 + a.np] - rb0);
    a.fsum[c * stride + 3ll * (a.T.pass_run_begin[p] - rb0) + col] = acc;
  }
}

// Per-gate gradients of a segment.  The first np * groups workgroups take kAssembleRuns
// runs of a pass each: shared runs, summed over the micro-batch, into row 0 of Gr.  The
// others take one (sample, pass) each: its per-sample runs, into the sample's row.
__device__ inline void assemble_body(const AssembleArgs& a, int blk, int t, double* red) {
  const int col = t & 63, lane = t >> 6;
  const int n_shared = a.np * a.groups;
  if (blk < n_shared) {
    const int p = a.p0 + blk / a.groups, s0 = (blk % a.groups) * kAssembleRuns;
    const int ns = a.T.passes[p].n_slots;
    if (s0 >= ns) return;
    const int rb = a.T.pass_run_begin[p];
    const int n = min(kAssembleRuns, ns - s0);
    double acc = 0;
    if (col < 3 * n) {
      if (a.chunks > 0) {
        const int rb0 = a.T.pass_run_begin[a.p0];
        const long long stride = 3ll * (a.T.pass_run_begin[a.p0 + a.np] - rb0);
        const double* src = a.fsum + 3ll * (rb - rb0 + s0) + col;
#pragma unroll 4
        for (int c = lane; c < a.chunks; c += 4) acc += src[c * stride];
      } else {
        const float* src = a.partF + (long long)a.nb * a.T.partF_off[p] + 3 * s0 + col;
        const int rows = a.nb * a.tiles;
#pragma unroll 4
        for (int r = lane; r < rows; r += 4) acc += src[(long long)r * 3 * ns];
      }
    }
    acc = lane_sum4(acc, t, red);
    __syncthreads();
    if (t < 64) red[t] = acc;
    __syncthreads();
    if (t >= n) return;
    const RunRec rr = a.T.runs[a.T.pass_runs[rb + s0 + t]];
    if (rr.coef < 0) return;
    for (int i = 0; i < rr.gate_count; ++i) {
      const int g = a.T.gates[a.T.run_gates[rr.gate_begin + i]].out_idx;
      const double* v = a.gvec + 3ll * g;
      a.Gr[g] = (float)(v[0] * red[3 * t] + v[1] * red[3 * t + 1] + v[2] * red[3 * t + 2]);
    }
    return;
  }
  const int s = (blk - n_shared) / a.nps, e = a.ps0 + (blk - n_shared) % a.nps;
  const int p = a.T.ps_pass[e], r0 = a.T.ps_begin[e], r1 = a.T.ps_begin[e + 1];
  const int ns = a.T.passes[p].n_slots;
  const float* base = a.partF + (long long)a.nb * a.T.partF_off[p] + (long long)s * a.tiles * 3 * ns;
  for (int q0 = r0; q0 < r1; q0 += kAssembleRuns) {
    const int n = min(kAssembleRuns, r1 - q0);
    double acc = 0;
    if (col < 3 * n) {
      const float* src = base + 3 * a.T.runs[a.T.ps_runs[q0 + col / 3]].slot + col % 3;
#pragma unroll 4
      for (int i = lane; i < a.tiles; i += 4) acc += src[(long long)i * 3 * ns];
    }
    acc = lane_sum4(acc, t, red);
    __syncthreads();
    if (t < 64) red[t] = acc;
    __syncthreads();
    if (t < n)
      run_grads(a.T, a.T.ps_runs[q0 + t], a.theta, a.x, a.F, a.sample0 + s, red[3 * t], red[3 * t + 1],
                red[3 * t + 2], a.Gr + (long long)s * a.n_angle, 1);
  }
}

// theta: sum over the gates sharing the angle, and over the micro-batch for the gates of
// per-sample runs (a shared run's gradient is summed already); x: sum
// over the gates sharing the input, per sample.  Block blk < th_blocks owns
// angles [blk * cols, (blk + 1) * cols): thread t takes angle t % cols and sample
// lane t / cols, sums its samples (lane, lane + lanes, ...) in order, and the
// lanes are added by a fixed pairwise tree in LDS (red: kSmallThreads doubles), so
// the result does not depend on scheduling.  The later blocks form dx, one thread
// per (sample, input).
template <class Real>
__device__ inline void reduce_grads_body(const ReduceGArgsT<Real>& a, int blk, int t, double* red) {
  if (blk < a.th_blocks) {
    const int cols = a.cols, lanes = kSmallThreads / cols;
    const int col = t % cols, lane = t / cols;
    const int p = blk * cols + col;
    double acc = 0;
    if (p < a.P) {
      const int r0 = a.T.th_ref_begin[p], r1 = a.T.th_ref_begin[p + 1];
      for (int i = r0; i < r1; ++i) {
        const int g = a.T.th_refs[i];
        if (g < 0) {
          if (lane == 0) acc += a.Gr[-1 - g];
        } else {
#pragma unroll 4
          for (int s = lane; s < a.nb; s += lanes) acc += a.Gr[(long long)s * a.n_angle + g];
        }
      }
    }
    red[t] = acc;
    __syncthreads();
    for (int half = lanes / 2; half >= 1; half /= 2) {
      if (lane < half) red[t] += red[t + half * cols];
      __syncthreads();
    }
    if (lane == 0 && p < a.P) {
      const double sum = red[col];
      a.dtheta[p] = a.accumulate ? a.dtheta[p] + (Real)sum : (Real)sum;
    }
    return;
  }
  const long long j = (long long)(blk - a.th_blocks) * kSmallThreads + t;
  if (!a.dx || j >= (long long)a.nb * a.F) return;
  const int s = (int)(j / a.F), f = (int)(j - (long long)s * a.F);
  double acc = 0;
  for (int i = a.T.in_ref_begin[f]; i < a.T.in_ref_begin[f + 1]; ++i)
    acc += a.Gr[(long long)s * a.n_angle + a.T.in_refs[i]];
  a.dx[(long long)(a.sample0 + s) * a.F + f] = (Real)acc;
}

// Expectations from their partial sums.  wide: one workgroup per sample, `lanes` partial
// sums at a time for each of the K observables (cols, a power of two), added by a fixed
// tree; else one thread per sum.
template <class Real>
__device__ inline void reduce_E_body(const ReduceEArgsT<Real>& a, int blk, int t, double* red) {
  if (!a.wide) {
    const long long idx = (long long)blk * kSmallThreads + t;
    if (idx >= (long long)a.nb * a.K) return;
    const int s = (int)(idx / a.K), k = (int)(idx - (long long)s * a.K);
    double acc = 0;
    for (int i = 0; i < a.parts; ++i) acc += a.partE[((long long)s * a.parts + i) * a.K + k];
    a.E[(long long)(a.sample0 + s) * a.K + k] = (Real)acc;
    return;
  }
  int cols = 1;
  while (cols < a.K) cols *= 2;
  const int lanes = kSmallThreads / cols, k = t % cols, lane = t / cols;
  const Real* src = a.partE + (long long)blk * a.parts * a.K;
  double acc = 0;
  if (k < a.K) {
#pragma unroll 4
    for (int i = lane; i < a.parts; i += lanes) acc += src[(long long)i * a.K + k];
  }
  red[t] = acc;
  __syncthreads();
  for (int half = lanes / 2; half >= 1; half /= 2) {
    if (lane < half) red[t] += red[t + half * cols];
    __syncthreads();
  }
  if (lane == 0 && k < a.K) a.E[(long long)(a.sample0 + blk) * a.K + k] = (Real)red[t];
}

}  // namespace qf

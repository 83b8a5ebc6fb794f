// kernels_fast.hip -- the throughput path of the explicit-Euler rollout (the
// configurations of Sec. IV with dead time and rolling resistance, and the
// lead-vehicle extension of Sec. VIII), FP64 and FP32-compensated, for one
// scenario or a batch of scenarios in one launch.
//
// Three stages:
//  1. prep: per sample, load (or draw) the parameters, derive the constants
//     of eq. (4)-(6), predict the number of steps to the stop from a
//     closed-form approximation of the braking phases, and classify the
//     sample (friction-limited or not).  Writes a 64-byte job record and a
//     sort key; counts keys in an LDS histogram.
//  2. counting sort of the keys: samples with the same predicted length land
//     in the same wavefront, longest first, so a wavefront's lanes finish
//     together and long wavefronts start early.
//     (Up to SORT1_MAX samples one workgroup sorts.)
//  3. rollout: each lane integrates one sample.  Steps run in blocks without
//     per-step tests (K steps; 16, then 4 as the wavefront nears its limits,
//     then single steps), in none of which a running lane can reach the horizon
//     or pass its command switch (the switch is the dead time, plus the
//     sample's own perception delay when the scenario has one, and then the sort
//     groups equal switch steps).  A lane may stop, or pass the obstacle, inside
//     a block: both are found at the block's end and the lane's end is
//     recomputed by replaying the block from its start, saved in LDS, while the
//     other lanes go on.  Inside a block the step takes the cheapest form that
//     gives bit-identical results in the current phase: dead time (a = 0),
//     generic, never-limited (max(a, alim) = a) or friction-limited
//     (max(a, alim) = alim for good, actuator update dead).  The grid is one
//     pass over the samples, or persistent: each wavefront takes its first chunk
//     of 64 sorted samples by its place and claims further ones through an
//     atomic counter (longest first, dynamically balanced).
#include <hip/hip_runtime.h>

#include <type_traits>
#include <vector>

#include "aeb_common.h"
#include "aeb_runtime.h"
#include "fast_path.h"
#include "rollout_steps.h"
#include "tune.h"

namespace aeb {

namespace {

// The step and block helpers of the FP64 integration are always inlined: an
// out-of-line call takes the lane state by reference, which puts it in
// scratch memory (the compiler declined to inline the largest forms).
#define HOT __device__ __attribute__((always_inline)) inline

// sort keys: 2 classes x 4,096 length levels (with perception 64 coarse length
// bins x 64 levels of length and command step); with the controller 64 decision
// ticks x 2 classes x 128 length levels (the sort's kernels take the key count
// as a template argument: their per-bin loops cost latency on small launches)
constexpr int NBINS = 8192;
constexpr int NBINS_CTL = 16384;
// The sort's kernels (prep, scan, scatter) run in workgroups of one wavefront
// per SIMD: beside a running integration kernel (four wavefronts per SIMD)
// each CU has room for one such workgroup, so the next launch's preparation
// overlaps the current integration when launches are pipelined on two streams.
constexpr int PREP_BLOCK = 256;
constexpr int PREP_SAMPLES = 4096;                     // samples per scatter block
constexpr int PREP_PER = PREP_SAMPLES / PREP_BLOCK;    // samples per scatter thread
// The drawing prep kernel takes one sample per thread, and its key histogram
// is a kernel of its own.  (A loop over several samples per thread, to share
// a block histogram's flush, let the compiler hoist the constants of the
// draws' log, sqrt, sine and cosine out of the loop and hold them in
// registers: 231 VGPRs, two wavefronts per SIMD, against 113 without it; and
// a block histogram per 256 samples costs more than the draws save.)  The
// plain method's prep, which draws nothing, keeps PREP_PER samples per thread
// with the histogram fused in (k_prep_cols).
inline unsigned prep_grid(int64_t n) {
  return static_cast<unsigned>((n + PREP_BLOCK - 1) / PREP_BLOCK);
}
template <bool DEVRNG>
constexpr int prep_threads() { return PREP_BLOCK; }

// Closed-form estimate of the stopping time (s): dead time at zero brake,
// first-order ramp of the brake to the friction limit (or to the command),
// then constant deceleration; drag taken at a third of the squared speed.
__device__ inline float predict_stop_time(float v0, float kd, float c, float alim, float tau,
                                          float acmd, float td) {
  const float amag = -acmd;  // command magnitude
  if (!(amag > 0.0f)) return INFINITY;
  float v1 = v0 - (c + kd * v0 * v0) * td;
  if (v1 <= 0.0f) return td;
  if (alim > acmd) {  // limited: the ramp stops at alim
    const float lim = -alim;
    const float ratio = alim / acmd;  // in (0, 1)
    const float ss = -tau * log1pf(-ratio);
    const float dv = amag * ss - tau * lim + (c + kd * v1 * v1 * 0.5f) * ss;
    const float v2 = v1 - dv;
    if (v2 <= 0.0f) return td + ss * (v1 / fmaxf(v1 - v2, 1e-6f));
    const float den = lim + c + kd * v2 * v2 * (1.0f / 3.0f);
    if (!(den > 0.0f)) return INFINITY;
    return td + ss + v2 / den;
  }
  const float den = amag + c + kd * v1 * v1 * (1.0f / 3.0f);
  if (!(den > 0.0f)) return INFINITY;
  return td + (v1 + amag * tau) / den;
}

// Predicted stop time under the closed-loop controller with a stationary
// obstacle, for the sort only (noise left out): constant speed until the
// first decision with TTC below ttc_warn, then the partial command (after
// the dead time and, roughly, the actuator lag) until the first decision with
// TTC below ttc_brake, then the full command as in predict_stop_time.
// Decisions fall on the controller's tick grid (period per); *t_full gets
// the predicted time of the full-braking decision.
__device__ inline float predict_ctl_stop_time(float v0, float gap, float tw, float tb, float aw,
                                              float per, float dead, float kd, float c,
                                              float alim, float tau, float acmd,
                                              float* t_full) {
  *t_full = 0.0f;
  if (!(v0 > 0.0f)) return dead;
  auto tick = [&](float t) { return ceilf(fmaxf(t, 0.0f) / per) * per; };
  float t_b, v_b;
  if (!(tw > tb)) {
    // no partial stage: full braking from the first decision below ttc_brake
    t_b = tick(gap / v0 - tb);
    v_b = v0;
  } else {
    const float t_w = tick(gap / v0 - tw);
    const float delay = dead + tau;
    const float g0 = gap - v0 * (t_w + delay);  // gap when the partial braking bites
    if (g0 <= tb * v0) {
      t_b = tick(gap / v0 - tb);
      v_b = v0;
    } else {
      // gap g0 - v0 s + aw s^2 / 2 reaches tb (v0 - aw s): smallest root
      float sroot;
      if (aw < 1e-6f) {
        sroot = (g0 - tb * v0) / v0;
      } else {
        const float bq = v0 - tb * aw;
        const float disc = bq * bq - 2.0f * aw * (g0 - tb * v0);
        // the partial braking alone stops the vehicle first
        *t_full = t_w + delay + v0 / aw;
        if (!(disc >= 0.0f) || bq <= 0.0f) return *t_full;
        sroot = (bq - sqrtf(disc)) / aw;
        if (sroot * aw >= v0) return *t_full;
      }
      t_b = tick(t_w + delay + sroot);
      v_b = fmaxf(v0 - aw * (t_b - t_w - delay), 0.0f);
    }
  }
  *t_full = t_b;
  return t_b + predict_stop_time(v_b, kd, c, alim, tau, acmd, dead);
}

// The actuator's stage values of one RK4 step from a1, and its end value.
struct RkAct {
  double a2, a3, a4, end;
};
__device__ inline RkAct rk4_act(double a1, double kt, double dt, double h2, double h6, double cmd);
constexpr int ACT_HDR = 8;    // doubles in front of the actuator table's entries: `fix`
constexpr int ACT_PAD = 64;   // entries written past the last step or `fix`

// Inputs of the prep stage: one scenario (uniform) or a batch table.
struct PrepArgs {
  aeb_scenario s;          // single scenario
  ParamSrc src;            // its parameter columns (plain method)
  int64_t n;               // samples in the launch
  int nd, nmax;            // single scenario's step counts
  float cap;               // step count that maps to the last sort bin
  const aeb_scenario* scns;  // batch: scenarios
  const ScnDev* tab;         // batch: per-scenario constants and offsets
  int n_scn;
  int32_t* nds;              // per-sample command step (launches with perception), else null
  int ctl;                   // closed-loop controller (single scenario)
  double* weight;            // single scenario: importance-sampling weights out (or null)
  const BatchHdr* hdr;       // batch on device tables: n, cap and n_scn from here (else null)
  double* act;               // single scenario: the actuator table to fill (or null)
};

// One sample: its parameters (drawn, or loaded from the plain method's
// columns), its job record and its sort key.
// (i: global index; j, local: its scenario and its index there)
template <bool DEVRNG, bool BATCH>
HOT uint32_t prep_sample(const PrepArgs& a, int64_t i, uint32_t j, int64_t local, float capf,
                         Job* jobs, LeadJob* leads) {
  const aeb_scenario& s = BATCH ? a.scns[j] : a.s;
  const int nd = BATCH ? a.tab[j].nd : a.nd;
  const int nmax = BATCH ? a.tab[j].nmax : a.nmax;
  double v0, mu, mass, sg, cg, cda, crr, tau, gap, lead, trig, lw;
  if (DEVRNG) {
    Sample q = draw_sample(s, static_cast<uint64_t>(local));
    v0 = q.v0; mu = q.mu; mass = q.mass; sg = q.sin_grade; cg = q.cos_grade;
    cda = q.cda; crr = q.crr; tau = q.tau; gap = q.gap; lead = q.lead_decel;
    trig = q.trigger;
    lw = q.log_w;
  } else {
    v0 = a.src.v0[i]; mu = a.src.mu[i]; mass = a.src.mass[i]; sg = a.src.sin_g[i];
    cg = a.src.cos_g[i]; cda = a.src.cda[i]; crr = a.src.crr[i]; tau = a.src.tau[i];
    gap = a.src.gap[i]; lead = a.src.lead[i];
    trig = a.src.trig ? a.src.trig[i] : 0.0;
    lw = a.src.logw ? a.src.logw[i] : 0.0;
  }
  // the importance-sampling weight goes straight to the sample's output
  double* wout = BATCH ? a.tab[j].out.weight : a.weight;
  if (wout) wout[local] = exp(lw);
  // with perception every sample has its own command step
  int ndl = nd;
  if (a.nds) {
    ndl = static_cast<int>(command_step(s, trig, nmax));
    a.nds[i] = ndl;
  }
  const Consts k = derive(s, mu, mass, sg, cg, cda, crr);
  Job J;
  J.v0 = v0;
  J.nkd = -k.kd;
  J.c = k.c;
  J.alim = k.alim;
  J.kt = s.integrator == AEB_RK4 ? 1.0 / tau : s.dt / tau;  // Euler: dt/tau; RK4: 1/tau
  J.gap = gap;
  // |acc| <= min(|a_cmd|, |alim|) + kd vmax^2 + |c|, with vmax the largest
  // speed the sample can reach (only a downhill pull can raise it)
  const double creach = k.c < 0.0 ? -k.c : 0.0;
  const double vmax = fabs(v0) + s.horizon * creach;
  const double brake = fmin(fabs(s.a_cmd), fabs(k.alim));
  J.dmax = (brake + fabs(k.kd) * vmax * vmax + fabs(k.c)) * 1.0001 + 1e-9;
  // That supposes a brake between zero and its command over every step, and the
  // Euler kernels' steady forms one that approaches the command from one side:
  // an Euler step of at most one time constant, an RK4 step (whose mean brake
  // stays there while it is stable, to 2.785) of at most 2.5.  Columns may hold
  // other time constants, and so may RK4's draws: no bound then, so that the
  // sample's wavefront takes single steps in the generic form, with every test,
  // for as long as the sample runs.
  const bool rk4 = s.integrator == AEB_RK4;
  const double z = rk4 ? J.kt * s.dt : J.kt;
  if (!(z >= 0.0 && z <= (rk4 ? 2.5 : 1.0))) J.dmax = INFINITY;
  // classify and predict
  const bool limited = !(k.alim < s.a_cmd - 1e-6);
  float td = static_cast<float>(ndl) * static_cast<float>(s.dt);
  if (a.ctl && s.obstacle == AEB_OBS_LEAD) {
    // approach until the full-brake threshold, for the sort only: a lead
    // braking at `lead` from the ego's speed (closing speed lead t, gap
    // closed by lead t^2 / 2)
    const float T = static_cast<float>(s.ttc_brake), G = static_cast<float>(gap);
    const float A = static_cast<float>(lead);
    td += A > 0.0f ? sqrtf(T * T + 2.0f * G / A) - T : static_cast<float>(s.horizon);
  }
  float t, t_full = -1.0f;
  if (a.ctl && s.obstacle != AEB_OBS_LEAD)
    t = predict_ctl_stop_time(static_cast<float>(v0), static_cast<float>(gap),
                              static_cast<float>(s.ttc_warn), static_cast<float>(s.ttc_brake),
                              -static_cast<float>(s.a_warn), static_cast<float>(s.ctl_period),
                              static_cast<float>(ndl) * static_cast<float>(s.dt),
                              static_cast<float>(k.kd), static_cast<float>(k.c),
                              static_cast<float>(k.alim), static_cast<float>(tau),
                              static_cast<float>(s.a_cmd), &t_full);
  else
    t = predict_stop_time(static_cast<float>(v0), static_cast<float>(k.kd),
                          static_cast<float>(k.c), static_cast<float>(k.alim),
                          static_cast<float>(tau), static_cast<float>(s.a_cmd), td);
  float steps = t / static_cast<float>(s.dt);
  if (!(steps < static_cast<float>(nmax))) steps = static_cast<float>(nmax);
  if (!(steps > 0.0f)) steps = 0.0f;
  J.pred = steps;
  J.scn = j;
  jobs[i] = J;
  if (leads) leads[i].decel = lead;
  const uint32_t u = static_cast<uint32_t>(fminf(steps, capf) * (4096.0f / (capf + 1.0f)));
  const uint32_t ud = 4095u - (u > 4095u ? 4095u : u);  // longest first
  // within a coarse length bin: finer length; with perception 8 finer length
  // levels, then the command step in 16-step bins, so a wavefront's lanes
  // end close together and switch the command within a few steps of each
  // other (each distinct switch step cuts the wavefront's blocks)
  const uint32_t fine =
      a.nds ? (((ud >> 3) & 7u) << 3) | ((static_cast<uint32_t>(ndl) >> 4) & 7u) : ud & 63u;
  uint32_t key = (limited ? 0u : 4096u) | (ud & ~63u) | fine;
  // with a lead vehicle: first how far into the run the ego gets out of its
  // reach, in eighths (a wavefront drops the lead once it is out of reach of
  // all its lanes): the lead brakes at once, the ego after the dead time and
  // the actuator's lag, and then gains by what it brakes harder; the last
  // eighth holds those that never do
  if (s.obstacle == AEB_OBS_LEAD && !a.ctl) {
    const float al = static_cast<float>(lead), lag = td + static_cast<float>(tau);
    const float gain = -static_cast<float>(fmax(s.a_cmd, k.alim) - k.c) - al;
    const float part = gain > 0.0f ? (lag + al * lag / gain) / t : 1.0f;
    const uint32_t e = part < 0.875f ? static_cast<uint32_t>(fmaxf(part, 0.0f) * 8.0f) : 7u;
    key = ((7u - e) << 10) | (limited ? 0u : 512u) | (ud >> 3);
  }
  // with the controller: first the tick of the predicted full-braking
  // decision (modulo 64, latest first), so a wavefront's lanes reach the
  // thresholds, where the noise can decide and the whole wavefront draws
  // it, at the same ticks; then the class and the length in 128 levels, so
  // that they also stop close together (each lane's stop takes the
  // wavefront down the block ladder)
  if (t_full >= 0.0f) {
    const uint32_t tk =
        static_cast<uint32_t>(t_full / static_cast<float>(s.ctl_period) + 0.5f) & 63u;
    key = ((63u - tk) << 8) | (limited ? 0u : 128u) | (ud >> 5);
  }
  return key;
}

// The actuator table (ActTab) of a scenario with a CONST time constant, by one
// lane: a serial chain of about twenty operations per step (50 ns) over the
// steps of the horizon or until the actuator stands still (32 time constants
// or so), beside the prep of the samples.  In groups of FG steps, tested once
// each: entries past the last step are never read, and entries past `fix` all
// equal it.
__device__ inline void fill_act(const aeb_scenario& s, int nd, int nmax, double* act) {
  constexpr int FG = 16;
  static_assert(ACT_PAD >= 3 * FG, "a group past the last step, and two past `fix`");
  const double dt = s.dt, cmd = s.a_cmd, kt = 1.0 / s.tau.p0;  // as in the job records
  const double h2 = 0.5 * dt, h6 = dt / 6.0;
  const int n = nd < nmax ? nmax - nd : 0;  // braking steps
  double* tb = act + ACT_HDR;
  double a = 0.0;
  auto entry = [&](int i) {
    const RkAct r = rk4_act(a, kt, dt, h2, h6, cmd);
    tb[4 * i] = a;
    tb[4 * i + 1] = r.a2;
    tb[4 * i + 2] = r.a3;
    tb[4 * i + 3] = r.a4;
    return r.end;
  };
  int i = 0;
  bool still = false;
  while (i < n && !still) {
    double before = a;
#pragma unroll
    for (int j = 0; j < FG; ++j) {
      before = a;
      a = entry(i + j);
    }
    i += FG;
    still = a == before;  // a step that changes nothing: none later does
  }
  // the reads that start at `fix`: a block and the entries loaded ahead of it
  for (int j = 0; j < 2 * FG; ++j) entry(i + j);
  *reinterpret_cast<int*>(act) = i;
}

template <bool DEVRNG, bool BATCH>
__global__ __launch_bounds__(prep_threads<DEVRNG>()) void k_prep(PrepArgs a, Job* jobs,
                                                                 LeadJob* leads, uint32_t* keys) {
  constexpr int NT = prep_threads<DEVRNG>();
  // a recorded mix reads its sizes from the device header
  const int64_t n_all = a.hdr ? a.hdr->total : a.n;
  const float capf = a.hdr ? a.hdr->cap : a.cap;
  const int n_scn = a.hdr ? a.hdr->n_scn : a.n_scn;
  if (!BATCH) {
    int64_t blk = blockIdx.x;
    if (a.act) {  // the first block fills the actuator table
      if (blk == 0) {
        if (threadIdx.x == 0) fill_act(a.s, a.nd, a.nmax, a.act);
        return;
      }
      --blk;
    }
    const int64_t i = blk * NT + threadIdx.x;
    if (i < n_all) keys[i] = prep_sample<DEVRNG, false>(a, i, 0u, i, capf, jobs, leads);
    return;
  }
  // A batch: the launch covers an index space where every scenario starts on
  // a multiple of 64, so each wavefront holds samples of one scenario, found
  // from the wavefront's first index: its table entry and scenario are then
  // uniform (scalar loads, no per-lane copies of the scenario in registers).
  const int64_t pw = static_cast<int64_t>(blockIdx.x) * NT +
                     __builtin_amdgcn_readfirstlane(threadIdx.x & ~63u);
  int lo = 0, hi = n_scn - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (a.tab[mid].poff <= pw)
      lo = mid;
    else
      hi = mid - 1;
  }
  const uint32_t j = static_cast<uint32_t>(lo);
  const int64_t off = a.tab[j].off;
  const int64_t n_j = (lo + 1 < n_scn ? a.tab[lo + 1].off : n_all) - off;
  const int64_t local = pw - a.tab[j].poff + (threadIdx.x & 63);
  if (local < n_j) keys[off + local] = prep_sample<DEVRNG, true>(a, off + local, j, local, capf,
                                                                  jobs, leads);
}

// The plain method's prep (parameters from the columns: no draws, so nothing
// for the compiler to hoist): PREP_PER samples per thread with the key
// histogram in LDS, flushed with one atomic per key the block holds, so no
// separate histogram pass.
template <int NB>
__global__ __launch_bounds__(PREP_BLOCK) void k_prep_cols(PrepArgs a, Job* jobs, LeadJob* leads,
                                                          uint32_t* keys, uint32_t* ghist) {
  __shared__ uint32_t hist[NB];
  for (int j = threadIdx.x; j < NB; j += PREP_BLOCK) hist[j] = 0;
  __syncthreads();
  const int64_t base_i = static_cast<int64_t>(blockIdx.x) * PREP_SAMPLES;
  for (int r = 0; r < PREP_PER; ++r) {
    const int64_t i = base_i + r * PREP_BLOCK + threadIdx.x;
    if (i >= a.n) break;
    const uint32_t key = prep_sample<false, false>(a, i, 0u, i, a.cap, jobs, leads);
    keys[i] = key;
    atomicAdd(&hist[key], 1u);
  }
  __syncthreads();
  for (int j = threadIdx.x; j < NB; j += PREP_BLOCK)
    if (hist[j]) atomicAdd(&ghist[j], hist[j]);
}

// Key histogram: per block of PREP_SAMPLES keys in LDS, then one global
// atomic per key the block holds.
template <int NB>
__global__ __launch_bounds__(PREP_BLOCK) void k_hist(const uint32_t* keys, int64_t n,
                                                     uint32_t* ghist, const BatchHdr* hdr) {
  if (hdr) n = hdr->total;
  __shared__ uint32_t hist[NB];
  for (int j = threadIdx.x; j < NB; j += PREP_BLOCK) hist[j] = 0;
  __syncthreads();
  uint32_t key[PREP_PER];
  const int64_t base_i = static_cast<int64_t>(blockIdx.x) * (PREP_BLOCK * PREP_PER);
#pragma unroll
  for (int r = 0; r < PREP_PER; ++r) {
    const int64_t i = base_i + r * PREP_BLOCK + threadIdx.x;
    key[r] = i < n ? keys[i] : NB;
  }
#pragma unroll
  for (int r = 0; r < PREP_PER; ++r)
    if (key[r] < NB) atomicAdd(&hist[key[r]], 1u);
  __syncthreads();
  for (int j = threadIdx.x; j < NB; j += PREP_BLOCK)
    if (hist[j]) atomicAdd(&ghist[j], hist[j]);
}

// exclusive scan of the key histogram into bucket offsets (one block); also
// clears the integration kernel's chunk counter
template <int NB>
__global__ __launch_bounds__(PREP_BLOCK) void k_scan(uint32_t* hist, unsigned long long* counter) {
  if (threadIdx.x == 0) *counter = 0ull;
  __shared__ uint32_t part[PREP_BLOCK];
  constexpr int PER = NB / PREP_BLOCK;
  uint32_t loc[PER];
  uint32_t sum = 0;
  for (int j = 0; j < PER; ++j) {
    loc[j] = hist[threadIdx.x * PER + j];
    sum += loc[j];
  }
  part[threadIdx.x] = sum;
  __syncthreads();
  for (int off = 1; off < PREP_BLOCK; off <<= 1) {
    uint32_t v = threadIdx.x >= static_cast<unsigned>(off) ? part[threadIdx.x - off] : 0u;
    __syncthreads();
    part[threadIdx.x] += v;
    __syncthreads();
  }
  uint32_t base = part[threadIdx.x] - sum;
  for (int j = 0; j < PER; ++j) {
    hist[threadIdx.x * PER + j] = base;
    base += loc[j];
  }
}

// Placement: each block ranks its samples per key in LDS, reserves one range
// per key with a single global atomic, then writes the permutation.
template <int NB>
__global__ __launch_bounds__(PREP_BLOCK) void k_scatter(const uint32_t* keys, int64_t n,
                                                        uint32_t* offs, uint32_t* perm,
                                                        const BatchHdr* hdr) {
  if (hdr) n = hdr->total;
  __shared__ uint32_t cnt[NB];
  for (int j = threadIdx.x; j < NB; j += PREP_BLOCK) cnt[j] = 0;
  __syncthreads();
  uint32_t key[PREP_PER], rank[PREP_PER];
  const int64_t base_i = static_cast<int64_t>(blockIdx.x) * (PREP_BLOCK * PREP_PER);
  // every key load in flight before the first LDS rank
#pragma unroll
  for (int r = 0; r < PREP_PER; ++r) {
    const int64_t i = base_i + r * PREP_BLOCK + threadIdx.x;
    key[r] = i < n ? keys[i] : 0u;
  }
#pragma unroll
  for (int r = 0; r < PREP_PER; ++r) {
    const int64_t i = base_i + r * PREP_BLOCK + threadIdx.x;
    rank[r] = i < n ? atomicAdd(&cnt[key[r]], 1u) : 0u;
  }
  __syncthreads();
  // the range reservations, 16 keys of the thread at a time: every atomic of
  // a group is in flight before the first result is read (one after another
  // they set the kernel's time on small launches)
  constexpr int G = 16;
  static_assert(NB % (G * PREP_BLOCK) == 0, "key count");
  for (int j0 = threadIdx.x; j0 < NB; j0 += G * PREP_BLOCK) {
    uint32_t c[G], o[G];
#pragma unroll
    for (int q = 0; q < G; ++q) c[q] = cnt[j0 + q * PREP_BLOCK];
#pragma unroll
    for (int q = 0; q < G; ++q) {
      o[q] = 0u;
      if (c[q]) o[q] = atomicAdd(&offs[j0 + q * PREP_BLOCK], c[q]);
    }
#pragma unroll
    for (int q = 0; q < G; ++q) cnt[j0 + q * PREP_BLOCK] = o[q];
  }
  __syncthreads();
  for (int r = 0; r < PREP_PER; ++r) {
    const int64_t i = base_i + r * PREP_BLOCK + threadIdx.x;
    if (i < n) perm[cnt[key[r]] + rank[r]] = static_cast<uint32_t>(i);
  }
}

// The whole sort of a small launch in one workgroup: histogram, scan and
// placement in LDS, each thread's keys and ranks in registers.  One launch
// instead of four (clear, histogram, scan, placement), whose fixed costs set the
// time at such sizes: 25,000 keys 12 us against 19 us of kernels and the gaps
// between them, 1,000 keys 3.7 us (the call with four launches 290 and 284 us, with
// one 272 and 266).  Up to SORT1_MAX keys: beyond, the separate kernels spread
// over the chip.
constexpr int SORT1_T = 1024;
constexpr int SORT1_PER = 32;
constexpr int64_t SORT1_MAX = static_cast<int64_t>(SORT1_T) * SORT1_PER;

// SPT: samples per thread
template <int NB, int SPT>
__global__ __launch_bounds__(SORT1_T) void k_sort1(const uint32_t* keys, int64_t n, uint32_t* perm,
                                                   unsigned long long* counter,
                                                   const BatchHdr* hdr) {
  if (hdr) n = hdr->total;
  __shared__ uint32_t cnt[NB];
  __shared__ uint32_t wsum[SORT1_T / 64];
  const int t = threadIdx.x;
  if (t == 0) *counter = 0ull;
  uint32_t key[SPT], rank[SPT];
  // every key load in flight before the first LDS rank
#pragma unroll
  for (int r = 0; r < SPT; ++r) {
    const int64_t i = static_cast<int64_t>(r) * SORT1_T + t;
    key[r] = i < n ? keys[i] : 0u;
  }
  for (int j = t; j < NB; j += SORT1_T) cnt[j] = 0;
  __syncthreads();
  // Adds of one wavefront to one counter run one after the other.  Where a launch
  // has few keys (parameters that do not vary, a horizon that ends every sample)
  // that set the sort's time: lanes that share a key then add once (rollout of
  // 32,768 samples of one key 139 -> 120 us, the separate kernels 128; of two keys
  // 110 -> 103, 106).  Taken where two keys cover half of a wavefront's first
  // samples: more keys are counted faster one by one.
  unsigned long long left = __ballot(t < n);
  const unsigned long long first = left;
  for (int q = 0; q < 2 && left; ++q)
    left &= ~__ballot(key[0] == __shfl(key[0], __ffsll(static_cast<long long>(left)) - 1));
  const bool few = 2 * __popcll(left) <= __popcll(first);
  if (few) {
    const unsigned long long below = (1ull << (t & 63)) - 1ull;
#pragma unroll
    for (int r = 0; r < SPT; ++r) {
      bool mine = static_cast<int64_t>(r) * SORT1_T + t < n;
      rank[r] = 0u;
      for (int q = 0; q < 2; ++q) {
        const unsigned long long who = __ballot(mine);
        if (who == 0) break;
        const int from = __ffsll(static_cast<long long>(who)) - 1;
        const unsigned long long same =
            __ballot(mine && key[r] == static_cast<uint32_t>(__shfl(key[r], from)));
        uint32_t base = 0;
        if ((t & 63) == from)
          base = atomicAdd(&cnt[key[r]], static_cast<uint32_t>(__popcll(same)));
        base = __shfl(base, from);
        if (same >> (t & 63) & 1) {
          rank[r] = base + static_cast<uint32_t>(__popcll(same & below));
          mine = false;
        }
      }
      if (mine) rank[r] = atomicAdd(&cnt[key[r]], 1u);
    }
  } else {
#pragma unroll
    for (int r = 0; r < SPT; ++r) {
      const int64_t i = static_cast<int64_t>(r) * SORT1_T + t;
      rank[r] = i < n ? atomicAdd(&cnt[key[r]], 1u) : 0u;
    }
  }
  __syncthreads();
  // exclusive scan of the counts, PER consecutive bins per thread
  constexpr int PER = NB / SORT1_T;
  uint32_t loc[PER], sum = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    loc[j] = cnt[t * PER + j];
    sum += loc[j];
  }
  uint32_t inc = sum;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t v = __shfl_up(inc, o);
    if ((t & 63) >= o) inc += v;
  }
  if ((t & 63) == 63) wsum[t >> 6] = inc;
  __syncthreads();
  uint32_t base = inc - sum;
  for (int w = 0; w < (t >> 6); ++w) base += wsum[w];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    cnt[t * PER + j] = base;
    base += loc[j];
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < SPT; ++r) {
    const int64_t i = static_cast<int64_t>(r) * SORT1_T + t;
    rank[r] = i < n ? cnt[key[r]] + rank[r] : ~0u;
  }
  // The permutation by way of LDS, in the counters' place, and from there in
  // whole lines: one CU takes a cycle per line of a scattered store (25,000 keys
  // placed by scattered stores 18 us, so 12).
  uint16_t* stage = reinterpret_cast<uint16_t*>(cnt);
  constexpr uint32_t STAGE = 2 * NB;
  static_assert(SORT1_MAX <= 65536, "a sample's index fits 16 bits");
  for (uint32_t lo = 0; lo < n; lo += STAGE) {
    __syncthreads();
#pragma unroll
    for (int r = 0; r < SPT; ++r) {
      if (rank[r] - lo < STAGE && rank[r] != ~0u)
        stage[rank[r] - lo] = static_cast<uint16_t>(r * SORT1_T + t);
    }
    __syncthreads();
    for (uint32_t j = t; j < STAGE && lo + j < n; j += SORT1_T) perm[lo + j] = stage[j];
  }
}

__global__ void k_zero(uint32_t* p, int64_t n) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0u;
}

// ---------------------------------------------------------------------------
// FP64 block forms.  All four give the canonical step's x and v bit for bit:
//   G: abe = max(a, alim); acc = fma(-kd, v v, abe) - c; x, v, a fma updates
//   F: never limited (alim < a_cmd): max(a, alim) = a
//   C: limited for good (a <= alim < a_cmd): abe = alim, a no longer read
//   D: dead time (cmd = 0, a = 0): abe = 0 exactly, a stays 0
// ---------------------------------------------------------------------------
struct St64 {
  double x, v, a;
};

// lead vehicle and the running minimum of the clearance (gap + x_lead) - x
struct Ld64 {
  double xl, vl, gmin;
};

// ---------------------------------------------------------------------------
// Classical RK4 (Sec. IV-D) in the same forms, no fused operations, the
// command held over the step.  Stage derivative of the speed:
//   (max(a, alim) - kd v v) - c, written (m + (-kd) (v v)) - c (the same bits);
// the position's stages are the stage speeds.  Job.kt holds 1/tau here.
// ---------------------------------------------------------------------------
template <int FORM>
__device__ inline double rk_dv(const Job& J, double v, double a) {
  double m;
  if (FORM == FORM_G)
    m = fmax(a, J.alim);
  else if (FORM == FORM_F)
    m = a;
  else if (FORM == FORM_C)
    m = J.alim;
  else
    m = 0.0;  // dead time: a = 0 exactly and max(0, alim) = 0
  return (m + J.nkd * (v * v)) - J.c;
}

// (k1 + 2 k2 + 2 k3 + k4): the doubled stages come in by fused multiply-adds,
// the same bits as a product and a sum, since doubling is exact; two operations
// less in each of the three sums.
__device__ inline double rk_sum(double k1, double k2, double k3, double k4) {
  return fma(2.0, k3, fma(2.0, k2, k1)) + k4;
}

__device__ inline RkAct rk4_act(double a1, double kt, double dt, double h2, double h6,
                                double cmd) {
  RkAct r;
  const double k1 = (cmd - a1) * kt;
  r.a2 = a1 + h2 * k1;
  const double k2 = (cmd - r.a2) * kt;
  r.a3 = a1 + h2 * k2;
  const double k3 = (cmd - r.a3) * kt;
  r.a4 = a1 + dt * k3;
  const double k4 = (cmd - r.a4) * kt;
  r.end = a1 + h6 * rk_sum(k1, k2, k3, k4);
  return r;
}

// TAB: the actuator's stage values come from tb (see ActTab) and the lane's own
// actuator is left alone.
template <int FORM, bool TAB = false>
__device__ inline void rk4_step(St64& s, const Job& J, double dt, double h2, double h6,
                                double cmd, const double* tb = nullptr) {
  constexpr bool ACT = FORM == FORM_G || FORM == FORM_F;  // the actuator is read
  const double v1 = s.v;
  double a1 = s.a;
  RkAct act{a1, a1, a1, a1};
  if (ACT && TAB) {
    a1 = tb[0];
    act = RkAct{tb[1], tb[2], tb[3], s.a};
  } else if (ACT) {
    act = rk4_act(a1, J.kt, dt, h2, h6, cmd);
  }
  const double k1v = rk_dv<FORM>(J, v1, a1);
  const double v2 = v1 + h2 * k1v;
  const double k2v = rk_dv<FORM>(J, v2, act.a2);
  const double v3 = v1 + h2 * k2v;
  const double k3v = rk_dv<FORM>(J, v3, act.a3);
  const double v4 = v1 + dt * k3v;
  const double k4v = rk_dv<FORM>(J, v4, act.a4);
  s.x = s.x + h6 * rk_sum(v1, v2, v3, v4);
  s.v = v1 + h6 * rk_sum(k1v, k2v, k3v, k4v);
  if (ACT) s.a = act.end;
}

// Kernel tag of explicit Euler in the unfused form (the paper's rule of no
// fused operations): every a*b + c below a rounded product, then a rounded sum.
constexpr int EULER_NOFMA = 2;

// a*b + c: one fused multiply-add, or (unfused) a rounded product and a
// rounded sum (the build contracts nothing implicitly).  The canonical step's
// (abe - kd v v) and vl - dt al equal abe + (-kd)(v v) and vl + (-dt) al bit
// for bit (negation is exact), so one form serves both.
template <bool NF>
__device__ inline double mad(double a, double b, double c) {
  return NF ? a * b + c : fma(a, b, c);
}

// The actuator's trajectory when every sample of the launch has the same
// actuator time constant and command step (a CONST tau, no perception, no
// controller): it is then the same for all of them, so the prep launch's first
// block runs it once and the integration reads the values (scalar loads)
// instead of updating every lane's actuator: 19 of 51 operations of an RK4 step.
// Entry i holds step nd + i: the actuator at the step's start and its three
// later stage values.  Entries repeat from `fix` on, where a step leaves the
// actuator's bits as they are.  RK4 only: of an Euler step it would save 2 of 7
// operations and add a load that comes too late (350,000 samples 0.46 against
// 0.42 ms, 12,000 0.26 against 0.13).
struct ActTab {
  const double* __restrict__ tb;  // null: no table
  int fix, nd;
  HOT const double* at(int k) const { return tb + int64_t(4) * min(k - nd, fix); }
};

// TAB: the actuator from tb (K steps of entries), J's own left alone
template <int FORM, int K, bool LEAD, int INTEG = AEB_EULER, bool TAB = false>
HOT void block64(St64& s, Ld64& l, const Job& J, double al, double dt, double cmd,
                 const double* tb = nullptr) {
  constexpr bool NF = INTEG == EULER_NOFMA;
  if (INTEG == AEB_RK4) {
    const double h2 = 0.5 * dt, h6 = dt / 6.0;
    if (TAB) {
      // entries two steps at a time, loaded two steps ahead: a scalar load
      // takes longer than one step of a wavefront alone on its SIMD
      double e[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) e[q] = tb[q];
#pragma unroll
      for (int j = 0; j < K; j += 2) {
        double f[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) f[q] = tb[4 * (j + 2) + q];
        __builtin_amdgcn_sched_barrier(0);
        rk4_step<FORM, true>(s, J, dt, h2, h6, cmd, e);
        asm volatile("" : "+v"(s.x));
        rk4_step<FORM, true>(s, J, dt, h2, h6, cmd, e + 4);
        asm volatile("" : "+v"(s.x));
#pragma unroll
        for (int q = 0; q < 8; ++q) e[q] = f[q];
      }
      static_assert(!TAB || K % 2 == 0, "step pairs");
      return;
    }
#pragma unroll
    for (int j = 0; j < K; ++j) {
      rk4_step<FORM>(s, J, dt, h2, h6, cmd);
      // each step's position sum at its step (see run_steady)
      asm volatile("" : "+v"(s.x));
    }
    return;
  }
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const double q = s.v * s.v;
    double acc;
    if (FORM == FORM_G) {
      acc = mad<NF>(J.nkd, q, fmax(s.a, J.alim)) - J.c;
      s.a = mad<NF>(J.kt, cmd - s.a, s.a);
    } else if (FORM == FORM_F) {
      acc = mad<NF>(J.nkd, q, s.a) - J.c;
      s.a = mad<NF>(J.kt, cmd - s.a, s.a);
    } else if (FORM == FORM_C) {
      acc = mad<NF>(J.nkd, q, J.alim) - J.c;
    } else {  // FORM_D
      acc = mad<NF>(J.nkd, q, 0.0) - J.c;
    }
    s.x = mad<NF>(dt, s.v, s.x);
    s.v = mad<NF>(dt, acc, s.v);
    if (LEAD) {
      l.xl = mad<NF>(dt, l.vl, l.xl);
      l.vl = fmax(mad<NF>(-dt, al, l.vl), 0.0);
      l.gmin = fmin(l.gmin, (J.gap + l.xl) - s.x);
    }
    // unfused: each step's position sum happens at its step (else the
    // compiler defers the sums and holds every step's product in a register)
    if (NF) asm volatile("" : "+v"(s.x));
    if (NF && LEAD) {  // likewise the lead vehicle's state, and no step interleaved with the next
      asm volatile("" : "+v"(l.xl), "+v"(l.vl), "+v"(l.gmin), "+v"(s.v));
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

template <bool LEAD, int INTEG = AEB_EULER>
HOT void step64(St64& s, Ld64& l, const Job& J, double al, double dt, double cmd) {
  constexpr bool NF = INTEG == EULER_NOFMA;
  if (INTEG == AEB_RK4) {
    rk4_step<FORM_G>(s, J, dt, 0.5 * dt, dt / 6.0, cmd);
    return;
  }
  const double q = s.v * s.v;
  const double acc = mad<NF>(J.nkd, q, fmax(s.a, J.alim)) - J.c;
  s.a = mad<NF>(J.kt, cmd - s.a, s.a);
  s.x = mad<NF>(dt, s.v, s.x);
  s.v = mad<NF>(dt, acc, s.v);
  if (LEAD) {
    l.xl = mad<NF>(dt, l.vl, l.xl);
    l.vl = fmax(mad<NF>(-dt, al, l.vl), 0.0);
  }
}

// Scenario constants a lane works with: uniform kernel arguments for one
// scenario, the scenario table in a batch.
struct Ctx {
  double dt, a_cmd;
  int nd, nmax, impact_exit;
  OutCols out;
  const ScnDev* tab;
  const int32_t* nds;  // per-sample command steps (perception), else null
  CtlArgs ca;          // the closed-loop controller (kernels instantiated for it)
  const BatchHdr* hdr; // a recorded mix: the launch's sample count (else null)
  // profiling (timing enabled): the sum over chunks of the steps the
  // wavefront ran times its sample slots (the steps output sums the useful
  // ones: lane efficiency is their ratio), else null
  unsigned long long* lanes;
};

// Lane accounting of one chunk: the wavefront ran k steps for spw sample
// slots (one atomic per chunk, from its first lane).
__device__ inline void count_lanes(unsigned long long* lanes, int k, int spw) {
  if ((threadIdx.x & 63) == 0)
    atomicAdd(lanes, static_cast<unsigned long long>(k) * static_cast<unsigned long long>(spw));
}

struct LaneScn {
  double dt, a_cmd;
  int nd, nmax;
};

template <bool BATCH>
__device__ inline LaneScn lane_scn(const Ctx& c, const Job& J, bool valid, uint32_t g) {
  LaneScn r;
  if (BATCH) {
    const ScnDev& t = c.tab[J.scn];
    r.dt = t.dt;
    r.a_cmd = t.a_cmd;
    r.nd = t.nd;
    r.nmax = t.nmax;
  } else {
    r.dt = c.dt;
    r.a_cmd = c.a_cmd;
    r.nd = c.nd;
    r.nmax = c.nmax;
  }
  if (c.nds && valid) r.nd = c.nds[g];
  return r;
}

// A uniform value passed through an identity DPP move (quad_perm [0,1,2,3]):
// the same bits, which the compiler then keeps in a vector register as a lane
// value.  Measured on the compensated FP32 kernel with a stationary obstacle:
// its scenario constants and limits as lane values (as in a batch) take 79
// VGPRs instead of 85, six wavefronts per SIMD instead of five, and the
// single-scenario launch runs 5-6 % faster.
__device__ inline int lane_value(int x) {
  return __builtin_amdgcn_update_dpp(0, x, 0xe4, 0xf, 0xf, false);
}

__device__ inline double lane_value(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = lane_value(static_cast<int>(b)), hi = lane_value(static_cast<int>(b >> 32));
  return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned>(lo));
}

__device__ inline LaneScn lane_values(LaneScn r) {
  r.dt = lane_value(r.dt);
  r.a_cmd = lane_value(r.a_cmd);
  r.nd = lane_value(r.nd);
  r.nmax = lane_value(r.nmax);
  return r;
}

// Output columns and the sample's index in them (read only at the store, so
// that the pointers are not held through the integration).
template <bool BATCH>
__device__ inline OutCols lane_out(const Ctx& c, const Job& J, uint32_t g, int64_t& local) {
  if (BATCH) {
    const ScnDev& t = c.tab[J.scn];
    local = static_cast<int64_t>(g) - t.off;
    return t.out;
  }
  local = g;
  return c.out;
}

// Largest step index a block may end on without a per-step test: a block
// never straddles the command switch nd and ends before the last step
// nmax - 1 (the horizon test fires after that step).  The launch-wide
// limit of a wavefront is the minimum over its active lanes; it only grows
// as k passes a lane's nd or lanes finish, so it is refreshed once k reaches it.
__device__ inline int lane_lim(int k, int nd, int nmax) {
  return k < nd ? min(nd, nmax - 1) : nmax - 1;
}

// Minimum over the wavefront (every lane active), left in every lane: DPP row
// shifts of 1, 2, 4, 8 lanes give each row's minimum in its lane 15, the row
// broadcasts of lanes 15 and 31 carry it to lane 63.  Register moves, no LDS.
template <int CTRL, int ROW_MASK>
__device__ inline int dpp_min(int x) {
  return min(x, __builtin_amdgcn_update_dpp(INT_MAX, x, CTRL, ROW_MASK, 0xf, false));
}

__device__ inline int wave_min(int x) {
  x = dpp_min<0x111, 0xf>(x);  // row_shr:1
  x = dpp_min<0x112, 0xf>(x);  // row_shr:2
  x = dpp_min<0x114, 0xf>(x);  // row_shr:4
  x = dpp_min<0x118, 0xf>(x);  // row_shr:8
  x = dpp_min<0x142, 0xa>(x);  // row_bcast:15 into rows 1 and 3
  x = dpp_min<0x143, 0xc>(x);  // row_bcast:31 into rows 2 and 3
  return __builtin_amdgcn_readlane(x, 63);
}

// varnd: nd or nmax differ between lanes (a batch, or per-sample command steps)
__device__ inline int wave_lim(bool varnd, bool active, int k, int nd, int nmax) {
  // nd, nmax are uniform: say so, so that the tests on the limit are scalar
  if (!varnd) return __builtin_amdgcn_readfirstlane(lane_lim(k, nd, nmax));
  return wave_min(active ? lane_lim(k, nd, nmax) : INT_MAX);
}

// claim the next 64 sorted positions for this wavefront
__device__ inline int64_t claim(unsigned long long* counter) {
  unsigned long long base = 0;
  if ((threadIdx.x & 63) == 0) base = atomicAdd(counter, 64ull);
  const unsigned lo = __builtin_amdgcn_readfirstlane(static_cast<unsigned>(base));
  const unsigned hi = __builtin_amdgcn_readfirstlane(static_cast<unsigned>(base >> 32));
  return static_cast<int64_t>((static_cast<unsigned long long>(hi) << 32) | lo);
}

// The next 64 sorted positions of a wavefront.  First pass: the wavefront's
// own slice of its workgroup's range.  Later passes of a persistent launch:
// chunks claimed from the counter beyond the range the whole grid covered in
// its first pass (so the launch does not start with every wavefront
// contending for one atomic); a one-pass launch stops after the first.
__device__ inline int64_t next_chunk(unsigned long long* counter, int persistent, int pass,
                                     int64_t n) {
  if (pass == 0)
    return static_cast<int64_t>(blockIdx.x) * blockDim.x +
           __builtin_amdgcn_readfirstlane(threadIdx.x & ~63u);
  if (!persistent) return n;
  return claim(counter) + static_cast<int64_t>(gridDim.x) * blockDim.x;
}

// Lane sets of a wavefront, one bit per lane.  The flags of the integration
// (who is active, passed the obstacle, stopped, ...) are such sets: uniform
// values in scalar registers, combined by scalar instructions, so the block
// loops' tests and branches are scalar.  (As per-lane flags they took vector
// registers and some 50 instructions and half a dozen dependent branches per
// block, about 540 cycles where one wavefront runs alone on its SIMD.)
using lanes_t = unsigned long long;
HOT lanes_t ballot(bool b) { return __builtin_amdgcn_ballot_w64(b); }
HOT bool in(lanes_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }
// After a branch that lanes take differently: no instruction, but the lanes
// join here and not in a block further on, where the compiler would take every
// value that arrives over several edges (the lane sets, the step index) for
// one that differs between lanes, and put it in vector registers.
HOT void lanes_join() { __builtin_amdgcn_wave_barrier(); }

// Lane state and lane sets of the FP64 integration.
struct Wave64 {
  St64 s;
  Ld64 l;               // lead vehicle
  int on1, on2, stage;  // controller: first steps of its two commands (INT_MAX: none), stage
  double margin;        // lead vehicle: the running minimum when the lane ended
  // still running; passed the obstacle; passed it inside a block, and stopped
  // inside a block (both still to be replayed); friction-limited for good;
  // never limited; can become limited
  lanes_t active, collided, pend, stopped, clamped, free_lane, limited;
  // lead vehicle: lanes within the bounds of out_of_reach; lanes whose lead was dropped
  lanes_t tame, dropped;
};

// Block start states, kept in LDS for the replays.  Slot 0: the start of the
// lanes' current block, written at every block.  When a lane passes the
// obstacle or stops inside a block its entry is copied: slot 1 keeps the
// block it ended in, slot 2 (stationary obstacle) the block where a lane that
// runs on passed the obstacle.  Each lane reads and writes its own entries
// only, so no barrier is needed.  In registers these states took 16 VGPRs of
// every lane for the whole integration; here they cost two or four LDS writes
// per block.
constexpr int ROLL_MAX = 256;  // largest workgroup of the integration kernels
enum { SAV_CUR = 0, SAV_END = 1, SAV_PASS = 2 };
template <int OBS>
struct Saves64 {
  static constexpr int SLOTS = OBS == AEB_OBS_STATIONARY ? 3 : 2;
  static constexpr int NL = OBS == AEB_OBS_LEAD ? ROLL_MAX : 1;
  double x[SLOTS][ROLL_MAX], v[SLOTS][ROLL_MAX], a[SLOTS][ROLL_MAX];
  double xl[2][NL], vl[2][NL], gmin[2][NL];
  int k[SLOTS][ROLL_MAX], e[SLOTS][ROLL_MAX];  // first step of the block, and its end
};

template <int OBS>
HOT void save_start(const Wave64& L, Saves64<OBS>& S) {
  const int t = threadIdx.x;
  S.x[SAV_CUR][t] = L.s.x;
  S.v[SAV_CUR][t] = L.s.v;
  S.a[SAV_CUR][t] = L.s.a;
  if (OBS == AEB_OBS_LEAD) {
    S.xl[SAV_CUR][t] = L.l.xl;
    S.vl[SAV_CUR][t] = L.l.vl;
    S.gmin[SAV_CUR][t] = L.l.gmin;
  }
}

template <int OBS>
HOT void keep_start(Saves64<OBS>& S, int slot, int k, int B) {
  const int t = threadIdx.x;
  S.x[slot][t] = S.x[SAV_CUR][t];
  S.v[slot][t] = S.v[SAV_CUR][t];
  S.a[slot][t] = S.a[SAV_CUR][t];
  if (OBS == AEB_OBS_LEAD) {
    S.xl[slot][t] = S.xl[SAV_CUR][t];
    S.vl[slot][t] = S.vl[SAV_CUR][t];
    S.gmin[slot][t] = S.gmin[SAV_CUR][t];
  }
  S.k[slot][t] = k;
  S.e[slot][t] = k + B;
}

// What happened to the lanes in the block of B steps from step k: passed the
// obstacle, or stopped.  A lane that stopped does not test its end position
// (it may have moved back since): the replay of its block tests every step.
// With a lead vehicle a lane below zero clearance was reached before any stop
// in the block, since after a stop the clearance only grows.
// (DROP: the lead no longer matters, see out_of_reach)
template <int OBS, bool DROP>
HOT void block_events(Wave64& L, Saves64<OBS>& S, const Job& J, int k, int B, int impact_exit) {
  constexpr bool LEAD = OBS == AEB_OBS_LEAD;
  lanes_t stop = ballot(L.s.v <= 0.0) & L.active;
  lanes_t hit = 0;
  if (OBS == AEB_OBS_STATIONARY) hit = ballot(L.s.x > J.gap) & L.active & ~stop & ~L.collided;
  if (LEAD && !DROP) {
    hit = ballot(L.l.gmin < 0.0) & L.active;
    stop &= ~hit;
  }
  // (the sets change outside the lanes' branches, so that they stay scalar)
  L.collided |= hit;
  L.pend |= hit;
  L.stopped |= stop;
  const bool ends = LEAD || impact_exit;
  L.active &= ~(stop | (ends ? hit : 0ull));
  if (hit | stop) {
    if (in(hit)) keep_start<OBS>(S, ends ? SAV_END : SAV_PASS, k, B);
    if (in(stop)) {
      keep_start<OBS>(S, SAV_END, k, B);
      if (LEAD) L.margin = L.l.gmin;
    }
    lanes_join();
  }
}

// The lane's brake command at step kk (constant inside every block: blocks
// end at every command switch), and the first step with any command.
template <bool CTL>
__device__ inline double lane_cmd(const Wave64& L, const LaneScn& c, double a_warn, int kk) {
  if (!CTL) return kk >= c.nd ? c.a_cmd : 0.0;
  return kk >= L.on2 ? c.a_cmd : (kk >= L.on1 ? a_warn : 0.0);
}

template <bool CTL>
__device__ inline int first_cmd(const Wave64& L, const LaneScn& c) {
  return CTL ? min(L.on1, L.on2) : c.nd;
}

// Controller block limit of a lane: its next command switch, and the last step.
__device__ inline int ctl_lim(const Wave64& L, int k, int nmax) {
  // the earlier of the switches still ahead (either may be unset, INT_MAX)
  int sw = INT_MAX;
  if (L.on1 > k) sw = L.on1;
  if (L.on2 > k) sw = min(sw, L.on2);
  return min(sw, nmax - 1);
}

// The lanes whose speed cannot rise over the next block (nor over any later
// block under the same command): the brake is at or above its command and
// falls toward it, so max(a, alim) does not rise, drag only slows, and what is
// left of the acceleration is below zero by far more than any rounding.  A
// stop inside the block then shows at the block's end (speed still at or below
// zero), so such a lane may stop anywhere inside a block.  kt in steps: dt/tau.
HOT lanes_t falling(const Wave64& L, const Job& J, double cmd, double ktdt) {
  return ballot(J.nkd <= 0.0 && ktdt >= 0.0 && ktdt <= 1.0 && cmd <= L.s.a + 1e-9 &&
                fmax(L.s.a, J.alim) - J.c < -1e-3);
}

// The lanes that the lead vehicle cannot matter to any more: the ego is slower
// than the lead and brakes harder than it for the rest of the run, so the
// clearance only grows until the ego stands, and it is already above its
// running minimum.  No impact can follow, the margin is final, and the lead's
// state is not read again.  The ego's brake only falls (fall: the lanes of
// `falling`) and drag only slows, so its acceleration stays at or below
// max(a, alim) - c; the lead's is -al until it stands, at which point the
// slower ego has stopped.  The bounds leave room for rounding: in each step
// the speed difference grows by at least 1e-12 m/s and the clearance by
// 1e-9 m, several units in the last place of speeds below 1e3 m/s and
// positions below 1e6 m (tested once per lane: see `tame` in the kernel).
HOT lanes_t out_of_reach(const Wave64& L, const Job& J, double al, double dt, lanes_t fall) {
  const double idt = 1.0 / dt;
  const double ea = fmax(1e-6, 1e-12 * idt), ev = fmax(1e-6, 1e-9 * idt);
  return fall & L.tame &
         ballot(fmax(L.s.a, J.alim) - J.c < -al - ea && L.s.v < L.l.vl - ev &&
                (J.gap + L.l.xl) - L.s.x > L.l.gmin + 1e-6);
}

// B steps of one form from step k, in pieces of at most 16 (entries of the
// actuator table are contiguous over a piece), the actuator taken over from the
// table at the end so that tests, saves and checked steps find it in the lane.
template <int FORM, int B, bool LEAD, int INTEG, bool TAB>
HOT void steps64(Wave64& L, const Job& J, double al, double dt, double cmd, int k,
                 const ActTab& at) {
  if (!TAB || (FORM != FORM_F && FORM != FORM_G)) {
    block64<FORM, B, LEAD, INTEG>(L.s, L.l, J, al, dt, cmd);
    return;
  }
  constexpr int P = B < 16 ? B : 16;
#pragma unroll
  for (int q = 0; q < B / P; ++q)
    block64<FORM, P, LEAD, INTEG, true>(L.s, L.l, J, al, dt, cmd, at.at(k + q * P));
  static_assert(!TAB || B % P == 0, "whole pieces");
  L.s.a = *at.at(k + B);
}

// wnd: the smallest nd of the wavefront's lanes (the whole block is dead time
// for every lane when k + B <= wnd).  TOP: a block of the top level, where the
// steady forms are the runs' business and only the dead time and the generic
// form are left.
template <int OBS, int B, int INTEG, bool CTL, bool TOP, bool TAB, bool DROP>
HOT void run_block64(Wave64& L, Saves64<OBS>& S, const Job& J, double al, const LaneScn& c, int k,
                     int wnd, int impact_exit, double a_warn, double& xmax, const ActTab& at) {
  constexpr bool LEAD = OBS == AEB_OBS_LEAD && !DROP;
  const double cmd = lane_cmd<CTL>(L, c, a_warn, k);
  save_start<OBS>(L, S);
  if (k + B <= wnd) {
    steps64<FORM_D, B, LEAD, INTEG, TAB>(L, J, al, c.dt, cmd, k, at);
  } else if (!TOP && (L.active & ~L.clamped) == 0) {
    steps64<FORM_C, B, LEAD, INTEG, TAB>(L, J, al, c.dt, cmd, k, at);
  } else if (!TOP && (L.active & ~L.free_lane) == 0) {
    steps64<FORM_F, B, LEAD, INTEG, TAB>(L, J, al, c.dt, cmd, k, at);
  } else {
    steps64<FORM_G, B, LEAD, INTEG, TAB>(L, J, al, c.dt, cmd, k, at);
    L.clamped |= L.limited & ballot(k + B > first_cmd<CTL>(L, c) && L.s.a <= J.alim);
  }
  block_events<OBS, DROP>(L, S, J, k, B, impact_exit);
  if (INTEG == AEB_RK4) xmax = fmax(xmax, in(L.active) ? L.s.x : xmax);
}

// Whether a K-step block (no lane of the wavefront past its limit) is the
// right one: no active lane can stop inside it (speed above thr), or those
// that can fall throughout it and another lane is still at least a block away
// from its stop.
HOT bool long_block(const Wave64& L, double thr, lanes_t fall) {
  const lanes_t low = ballot(L.s.v <= thr) & L.active;
  if (low == 0) return true;
  return (low & ~fall) == 0 && (ballot(L.s.v > 2.0 * thr) & L.active) != 0;
}

// Consecutive K-step blocks in one steady form (every active lane friction-
// limited for good, or every one never limited), until the block limit wl or
// until shorter blocks are the better choice.  Returns the step index after
// the last block.
template <int OBS, int K, int FORM, int INTEG, bool TAB, bool DROP>
HOT int run_steady(Wave64& L, Saves64<OBS>& S, const Job& J, double al, double dt, double cmd,
                   int k, int wl, double thr, lanes_t fall, int impact_exit, double& xmax,
                   const ActTab& at, bool may_drop) {
  constexpr bool LEAD = OBS == AEB_OBS_LEAD && !DROP;
  bool more;
  do {
    k = __builtin_amdgcn_readfirstlane(k);
    save_start<OBS>(L, S);
    // in 16-step pieces whose position is pinned in a register at the end of
    // each: with no obstacle nothing inside the run reads the position, and
    // the compiler would otherwise hold every step's speed for a position
    // update sunk to the end of the run (hundreds of registers)
#pragma unroll
    for (int q = 0; q < K / 16; ++q) {
      steps64<FORM, 16, LEAD, INTEG, TAB>(L, J, al, dt, cmd, k + 16 * q, at);
      asm volatile("" : "+v"(L.s.x));
    }
    if (K % 16 != 0) block64<FORM, K % 16, LEAD, INTEG>(L.s, L.l, J, al, dt, cmd);
    static_assert(!TAB || K % 16 == 0, "whole pieces");
    block_events<OBS, DROP>(L, S, J, k, K, impact_exit);
    if (INTEG == AEB_RK4) xmax = fmax(xmax, in(L.active) ? L.s.x : xmax);
    k += K;
    more = k + K <= wl && L.active != 0 && long_block(L, thr, fall);
    if (LEAD && may_drop)  // every lane out of the lead's reach: the caller drops it
      more = more && (L.active & ~out_of_reach(L, J, al, dt, fall)) != 0;
  } while (more);
  return k;
}

template <int OBS, int K, bool BATCH, int INTEG = AEB_EULER, bool CTL = false, bool TAB = false>
__global__ __launch_bounds__(ROLL_MAX) void k_roll_fp64(const Job* __restrict__ jobs,
                                                        const LeadJob* __restrict__ leads,
                                                        const uint32_t* __restrict__ perm,
                                                        int64_t n, Ctx ctx,
                                                        unsigned long long* counter,
                                                        int persistent,
                                                        const double* __restrict__ act) {
  ActTab at{nullptr, 0, 0};
  if (TAB) at = ActTab{act + ACT_HDR, *reinterpret_cast<const int*>(act), ctx.nd};
  if (ctx.hdr) n = ctx.hdr->total;  // a recorded mix: its size from the device header
  // block ladder: K steps, then KM, then KS, then single checked steps.  A
  // level runs while every lane that could stop inside the block (speed below
  // the level's bound) is one whose speed can only fall, so that its stop
  // shows at the block's end and is found by replaying that block.  K-step
  // blocks go on past such lanes while another lane is still at least a block
  // away from its stop (a wavefront whose lanes stop far apart stays in the
  // long blocks); once every lane is near, KM-step blocks, so that little runs
  // past the last stop.  (A ladder that left the long blocks at the first
  // lane's stop ran the spread of a wavefront's stops in short blocks and
  // checked steps: 25,000 samples 191 us against 107, 200,000 with perception
  // 390 against 300, 1,048,576, whose wavefronts stop together, 1.00 against
  // 0.98 ms.)
  constexpr int KS = 4;
  constexpr int KM = K > 16 ? 16 : KS;
  // with the controller, decisions every few tens of steps leave short
  // remainders: a 2-step level before the single steps
  constexpr int K2 = CTL ? 2 : KS;
  constexpr bool LEAD = OBS == AEB_OBS_LEAD;
  __shared__ Saves64<OBS> sav;
  for (int pass = 0;; ++pass) {
    const int64_t base = next_chunk(counter, persistent, pass, n);
    if (base >= n) break;
    const int64_t pos = base + (threadIdx.x & 63);
    const bool valid = pos < n;
    const uint32_t g = valid ? perm[pos] : 0u;
    Job J;
    if (valid) {
      J = jobs[g];
    } else {
      J = Job{1.0, 0.0, 0.0, -1.0, 0.5, 1e30, 1.0, 0.0f, 0u};
    }
    const double al = (LEAD && valid) ? leads[g].decel : 0.0;
    const LaneScn c = lane_scn<BATCH>(ctx, J, valid, g);
    const bool varnd = BATCH || ctx.nds;
    // every lane is in its dead time for blocks ending at or before wnd (with
    // the controller: until its first command, known once decided)
    int wnd = CTL ? INT_MAX
                  : __builtin_amdgcn_readfirstlane(varnd ? wave_min(valid ? c.nd : INT_MAX) : c.nd);
    // v above these cannot reach 0 within a block (|dv/dt| <= dmax)
    const double thr_k = static_cast<double>(K) * c.dt * J.dmax;
    const double thr_m = static_cast<double>(KM) * c.dt * J.dmax;
    const double thr_s = static_cast<double>(KS) * c.dt * J.dmax;
    const double thr_2 = static_cast<double>(K2) * c.dt * J.dmax;
    // the smallest block level and its stopping bound
    constexpr int KMIN = K2 < KS ? K2 : KS;
    const double thr_min = K2 < KS ? thr_2 : thr_s;
    const double ktdt = INTEG == AEB_RK4 ? J.kt * c.dt : J.kt;
    Wave64 L;
    L.on1 = L.on2 = INT_MAX;
    L.stage = 0;
    L.s = St64{0.0, J.v0, 0.0};
    L.l = Ld64{0.0, LEAD ? J.v0 : 0.0, J.gap};
    L.margin = J.gap;
    L.active = ballot(valid);
    L.collided = L.pend = L.stopped = L.clamped = L.dropped = 0;
    // (the horizon in seconds bounds both vehicles' travel)
    L.tame = LEAD ? ballot(al >= 0.0 && fabs(J.v0) < 1e3 && fabs(J.gap) < 1e5 &&
                           fabs(J.v0) * (c.nmax * c.dt) < 5e5)
                  : 0;
    // never limited: a >= a_cmd - (rounding) > alim, so max(a, alim) = a; and
    // limited for good once a <= alim: a never climbs above max(a, a_cmd) <
    // alim.  Both need an actuator that approaches its command from one side,
    // RK4's stages included: a step of at most one time constant (beyond it
    // an RK4 lane keeps the generic form, and an Euler lane the single steps).
    const bool smooth = ktdt >= 0.0 && ktdt <= 1.0;
    L.free_lane = ballot(smooth && J.alim < c.a_cmd - 1e-6);
    L.limited = ballot(smooth && J.alim > c.a_cmd + 1e-9);
    int end = 0, steps = 0;
    double dist = __builtin_nan("");  // until the lane's end is found
    // RK4's last step may move the position back (stage speeds below zero as
    // the vehicle stops): the margin then comes from the largest position,
    // tracked at block ends and over checked steps (before a stop the position
    // rises)
    double xmax = 0.0;
    float vimp = 0.0f;
    int k = 0, wl = -1;
    // controller: the next decision step and the decisions taken (uniform)
    int ktick = 0;
    uint32_t tick = 0;
    // a run of steady blocks, and one block of a level; with a lead vehicle in
    // two forms, with it and without
    auto run = [&](auto form, bool dropped, double cmd, int kk, int lim, lanes_t f) {
      constexpr int FORM = decltype(form)::value;
      if (LEAD && dropped)
        return run_steady<OBS, K, FORM, INTEG, TAB, LEAD>(L, sav, J, al, c.dt, cmd, kk, lim,
                                                          thr_k, f, ctx.impact_exit, xmax, at,
                                                          false);
      // (past the command of every lane, so a lane's speed falls for good)
      return run_steady<OBS, K, FORM, INTEG, TAB, false>(
          L, sav, J, al, c.dt, cmd, kk, lim, thr_k, f, ctx.impact_exit, xmax, at,
          !CTL && (L.active & ~ballot(kk >= c.nd)) == 0);
    };
    auto block = [&](auto len, auto top, bool dropped, int kk) {
      constexpr int B = decltype(len)::value;
      constexpr bool TOP = decltype(top)::value;
      if (LEAD && dropped)
        run_block64<OBS, B, INTEG, CTL, TOP, TAB, LEAD>(L, sav, J, al, c, kk, wnd,
                                                        ctx.impact_exit, ctx.ca.a_warn, xmax, at);
      else
        run_block64<OBS, B, INTEG, CTL, TOP, TAB, false>(
            L, sav, J, al, c, kk, wnd, ctx.impact_exit, ctx.ca.a_warn, xmax, at);
    };
    // every lane has ended by its step nmax (the horizon test fires at k + 1 = nmax)
    while (L.active) {
      // the step index is the same in every lane: keep it (and the branches on it) scalar
      k = __builtin_amdgcn_readfirstlane(k);
      if (CTL) {
        if (k == ktick) {
          // decision on the state after k steps; a raised stage's command
          // starts nd steps later.  Once every active lane is at the full
          // stage no decision can change anything: decisions stop, and so do
          // the block limits at decision steps.
          if ((ballot(L.stage < 2) & L.active) == 0) {
            ktick = INT_MAX;
          } else {
            if (in(L.active) && L.stage < 2) {
              const double gt = LEAD ? (J.gap + L.l.xl) - L.s.x : (J.gap + 0.0) - L.s.x;
              const double cl = LEAD ? L.s.v - L.l.vl : L.s.v - 0.0;
              // the noise is drawn only where it can change the decision,
              // estimated in single precision with an error box, and
              // evaluated exactly only where the box straddles a threshold
              int want = ctl_screen(ctx.ca, L.stage, gt, cl);
              if (want < 0) {
                const U2 u = uniform2(ctx.ca.seed, ctx.ca.sid, g, AEB_SLOT_CONTROL, tick);
                want = ctl_fast(ctx.ca, L.stage, gt, cl, u);
                if (want < 0) want = ctl_exact(ctx.ca, u, gt, cl);
              }
              if (want > L.stage) {
                if (want == 2)
                  L.on2 = k + c.nd;
                else
                  L.on1 = k + c.nd;
                L.stage = want;
              }
            }
            lanes_join();
            ++tick;
            // past the last step no decision can act
            const int64_t nk = static_cast<int64_t>(ktick) + ctx.ca.period;
            ktick = nk < c.nmax ? static_cast<int>(nk) : INT_MAX;
          }
          wnd = wave_min(valid ? min(L.on1, L.on2) : INT_MAX);
          wl = -1;
        }
        if (k >= wl) wl = min(ktick, wave_min(in(L.active) ? ctl_lim(L, k, c.nmax) : INT_MAX));
      } else if (!varnd || k >= wl) {
        wl = wave_lim(varnd, in(L.active), k, c.nd, c.nmax);
      }
      // lanes that could stop inside a K-step block need speeds that fall
      lanes_t fall = ~0ull;
      if (ballot(L.s.v <= thr_k) & L.active)
        fall = falling(L, J, lane_cmd<CTL>(L, c, ctx.ca.a_warn, k), ktdt);
      // every lane out of the lead's reach (past the command): drop the lead
      if (LEAD && !CTL && L.dropped == 0 && k >= wnd) {
        const double cmd = lane_cmd<CTL>(L, c, ctx.ca.a_warn, k);
        const lanes_t f = falling(L, J, cmd, ktdt) & ballot(k >= c.nd);
        if ((L.active & ~out_of_reach(L, J, al, c.dt, f)) == 0) L.dropped = L.active;
      }
      const bool drop = LEAD && L.dropped != 0;
      if (k + K <= wl && long_block(L, thr_k, fall)) {
        // past every lane's dead time, in a form no later block changes:
        // a run of blocks without the per-block bookkeeping
        const bool past = k + K > wnd;
        if (past && (L.active & ~L.clamped) == 0) {
          // (a clamped lane's speed falls whenever its acceleration without
          // drag is below zero)
          const lanes_t f = ballot(J.nkd <= 0.0 && J.alim - J.c < -1e-3);
          k = run(std::integral_constant<int, FORM_C>(), drop, 0.0, k, wl, f);
        } else if (past && (L.active & ~L.free_lane) == 0) {
          const double cmd = lane_cmd<CTL>(L, c, ctx.ca.a_warn, k);
          const lanes_t f = falling(L, J, cmd, ktdt);
          k = run(std::integral_constant<int, FORM_F>(), drop, cmd, k, wl, f);
        } else if (past && (L.active & ~(L.clamped | L.free_lane)) == 0) {
          // both kinds: the generic form, whose step serves either
          const double cmd = lane_cmd<CTL>(L, c, ctx.ca.a_warn, k);
          const lanes_t f = falling(L, J, cmd, ktdt);
          k = run(std::integral_constant<int, FORM_G>(), drop, cmd, k, wl, f);
        } else {
          block(std::integral_constant<int, K>(), std::true_type(), drop, k);
          k += K;
        }
      } else if (KM > KS && k + KM <= wl && (ballot(L.s.v <= thr_m) & L.active & ~fall) == 0) {
        block(std::integral_constant<int, KM>(), std::false_type(), drop, k);
        k += KM;
      } else if (k + KS <= wl && (ballot(L.s.v <= thr_s) & L.active & ~fall) == 0) {
        block(std::integral_constant<int, KS>(), std::false_type(), drop, k);
        k += KS;
      } else if (K2 < KS && k + K2 <= wl && (ballot(L.s.v <= thr_2) & L.active & ~fall) == 0) {
        block(std::integral_constant<int, K2>(), std::false_type(), drop, k);
        k += K2;
      } else {
        // checked single steps, in a loop of their own for as long as no
        // block level fits (a lane within the smallest level's stopping
        // bound, or the block limit closer than that level) and no decision
        // step or block limit is reached
        do {
          const double cmd = lane_cmd<CTL>(L, c, ctx.ca.a_warn, k);
          bool clamp = false, impact = false, done = false;
          if (in(L.active)) {
            if (LEAD && drop)
              step64<false, INTEG>(L.s, L.l, J, al, c.dt, cmd);
            else
              step64<LEAD, INTEG>(L.s, L.l, J, al, c.dt, cmd);
            if (INTEG == AEB_RK4) xmax = fmax(xmax, L.s.x);
            clamp = k >= first_cmd<CTL>(L, c) && L.s.a <= J.alim;
            if (LEAD && drop) {
              // no impact can follow
            } else if (LEAD) {
              const double gk = (J.gap + L.l.xl) - L.s.x;
              L.l.gmin = fmin(L.l.gmin, gk);
              impact = gk < 0.0;
            } else if (OBS == AEB_OBS_STATIONARY) {
              impact = L.s.x > J.gap;
            }
            if (impact && !in(L.collided))
              vimp = static_cast<float>(LEAD ? L.s.v - L.l.vl : L.s.v);
            if (impact && (LEAD || ctx.impact_exit))
              end = AEB_END_IMPACT;
            else if (L.s.v <= 0.0)
              end = AEB_END_STOP;
            else if (k + 1 >= c.nmax)
              end = AEB_END_HORIZON;
            done = end != 0;
            if (done) {
              steps = k + 1;
              dist = L.s.x;
              if (LEAD) L.margin = L.l.gmin;
            }
          }
          lanes_join();
          L.clamped |= L.limited & ballot(clamp);
          if (OBS != AEB_OBS_NONE) L.collided |= ballot(impact);
          L.active &= ~ballot(done);
          k += 1;
        } while (k < wl && !(CTL && k == ktick) && L.active != 0 &&
                 (k + KMIN > wl || (ballot(L.s.v <= thr_min) & L.active & ~fall) != 0));
      }
    }
    // replay the block in which each pending lane passed the obstacle, and the
    // block in which each stopped lane stopped.  Inside the first every speed
    // stays positive, so the position rises (and with a lead vehicle the
    // running minimum of the clearance can only fall); inside the second the
    // speed only falls and the position rises until the stop.  A chunk of RB
    // steps that ends inside the block therefore holds the event exactly when
    // its end state shows it; chunks without one are skipped whole, the one
    // holding it runs step by step.  The generic form is the canonical step,
    // so the replay reproduces the block's states bit for bit.
    auto replay = [&](lanes_t who, int slot, bool to_stop) {
      const int t = threadIdx.x;
      bool go = in(who);
      St64 r{0.0, 0.0, 0.0};
      Ld64 rl{};
      int kr = 0, se = 0;
      if (go) {
        r = St64{sav.x[slot][t], sav.v[slot][t], sav.a[slot][t]};
        if (LEAD) rl = Ld64{sav.xl[SAV_END][t], sav.vl[SAV_END][t], sav.gmin[SAV_END][t]};
        kr = sav.k[slot][t];
        se = sav.e[slot][t];
      }
      // a stopped lane may also have passed the obstacle in the same block
      bool seek = OBS != AEB_OBS_NONE && (!to_stop || !in(L.collided));
      // a dropped lead is not reached (and its saved state stands still)
      if (LEAD) seek = !in(L.dropped);
      bool passed = false;
      constexpr int RB = 8;
      if (K > RB) {
        // the command is constant over a block
        const double cmd = lane_cmd<CTL>(L, c, ctx.ca.a_warn, kr);
        bool skip = go;
        for (int it = 0; it < K / RB; ++it) {
          skip = skip && kr + RB <= se;
          if (ballot(skip) == 0) break;
          if (skip) {
            St64 q = r;
            Ld64 ql = rl;
            block64<FORM_G, RB, LEAD, INTEG>(q, ql, J, al, c.dt, cmd);
            const bool over = seek && (LEAD ? ql.gmin < 0.0 : q.x > J.gap);
            if (over || (to_stop && q.v <= 0.0)) {
              skip = false;
            } else {
              r = q;
              rl = ql;
              kr += RB;
            }
          }
        }
      }
      if (INTEG == AEB_RK4 && to_stop && go) xmax = fmax(xmax, r.x);
      // the event recurs within the block
      for (int it = 0; it <= K; ++it) {
        if (ballot(go) == 0) break;
        if (go) {
          const double cmd = lane_cmd<CTL>(L, c, ctx.ca.a_warn, kr);
          step64<LEAD, INTEG>(r, rl, J, al, c.dt, cmd);
          ++kr;
          if (INTEG == AEB_RK4 && to_stop) xmax = fmax(xmax, r.x);
          bool impact = false;
          if (LEAD) {
            const double gk = (J.gap + rl.xl) - r.x;
            rl.gmin = fmin(rl.gmin, gk);
            impact = seek && gk < 0.0;
          } else if (OBS == AEB_OBS_STATIONARY) {
            impact = seek && r.x > J.gap;
          }
          if (impact) {
            passed = true;
            seek = false;
            vimp = static_cast<float>(LEAD ? r.v - rl.vl : r.v);
            if (LEAD || ctx.impact_exit) {
              end = AEB_END_IMPACT;
              steps = kr;
              dist = r.x;
              xmax = r.x;
              L.margin = rl.gmin;
              go = false;
            }
            if (!to_stop) go = false;
          }
          if (to_stop && go && r.v <= 0.0) {
            end = AEB_END_STOP;
            steps = kr;
            dist = r.x;
            go = false;
          }
        }
      }
      lanes_join();
      if (OBS != AEB_OBS_NONE) L.collided |= ballot(passed);
      // (unreachable: a broken replay is visible; dist is still what it began with)
      if (go) vimp = __builtin_nanf("");
    };
    if (OBS != AEB_OBS_NONE && L.pend)
      replay(L.pend, OBS == AEB_OBS_STATIONARY && !ctx.impact_exit ? SAV_PASS : SAV_END, false);
    if (L.stopped) replay(L.stopped, SAV_END, true);
    if (ctx.lanes) count_lanes(ctx.lanes, k, 64);
    if (valid) {
      double margin = L.margin;
      if (!LEAD) {
        const double mg = J.gap - (INTEG == AEB_RK4 ? xmax : dist);
        margin = mg < J.gap ? mg : J.gap;
      }
      int64_t i;
      const OutCols o = lane_out<BATCH>(ctx, J, g, i);
      o.dist[i] = dist;
      o.margin[i] = margin;
      o.steps[i] = steps;
      o.status[i] = static_cast<uint8_t>(end | (in(L.collided) ? AEB_COLLIDED : 0));
      o.vimp[i] = in(L.collided) ? vimp : 0.0f;
    }
  }
}

// ---------------------------------------------------------------------------
// Two samples per lane (explicit Euler, fused form, no obstacle or a
// stationary one, no controller): lane l of a wavefront integrates the
// sorted positions base + l and base + 64 + l of a 128-sample chunk, so a
// wavefront's block bookkeeping, ladder and replay serve twice the samples
// and every block interleaves two independent dependency chains.  The forms and
// block limits are those of k_roll_fp64, taken over both samples of every lane.
// The ladder leaves a level as soon as a sample could stop inside its block, so
// stops fall on checked steps and only crossings are replayed.  Each sample's
// steps are the canonical step's, bit for bit.
// ---------------------------------------------------------------------------
// state and flags of one of a lane's samples
struct Lane64x2 {
  St64 s, sv;  // state, and start state of the block where the obstacle was passed
  Ld64 l;
  int sk, se;  // step index at that block start, and at its end
  bool active, collided, pend, clamped, free_lane, limited;
};

template <int FORM, int K>
HOT void block64x2(St64 (&s)[2], const Job (&J)[2], double dt0, double dt1, double cmd0,
                   double cmd1) {
  Ld64 l{};
#pragma unroll
  for (int j = 0; j < K; ++j) {
    block64<FORM, 1, false, AEB_EULER>(s[0], l, J[0], 0.0, dt0, cmd0);
    block64<FORM, 1, false, AEB_EULER>(s[1], l, J[1], 0.0, dt1, cmd1);
    // each step's position sums happen at their step (else the compiler
    // defers them and holds the speeds of many steps in registers)
    asm volatile("" : "+v"(s[0].x), "+v"(s[1].x));
  }
}

template <int OBS, int B>
HOT void run_block64x2(Lane64x2 (&L)[2], const Job (&J)[2], const LaneScn (&c)[2], int k, int wnd,
                       int impact_exit) {
  double cmd[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    cmd[q] = k >= c[q].nd ? c[q].a_cmd : 0.0;
    if (OBS != AEB_OBS_NONE && !L[q].collided) {
      L[q].sv = L[q].s;
      L[q].sk = k;
      L[q].se = k + B;
    }
  }
  St64 s[2] = {L[0].s, L[1].s};
  if (k + B <= wnd) {
    block64x2<FORM_D, B>(s, J, c[0].dt, c[1].dt, cmd[0], cmd[1]);
  } else if (__all((!L[0].active || L[0].clamped) && (!L[1].active || L[1].clamped))) {
    block64x2<FORM_C, B>(s, J, c[0].dt, c[1].dt, cmd[0], cmd[1]);
  } else if (__all((!L[0].active || L[0].free_lane) && (!L[1].active || L[1].free_lane))) {
    block64x2<FORM_F, B>(s, J, c[0].dt, c[1].dt, cmd[0], cmd[1]);
  } else {
    block64x2<FORM_G, B>(s, J, c[0].dt, c[1].dt, cmd[0], cmd[1]);
#pragma unroll
    for (int q = 0; q < 2; ++q)
      L[q].clamped = L[q].clamped || (L[q].limited && k + B > c[q].nd && s[q].a <= J[q].alim);
  }
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    L[q].s = s[q];
    if (OBS == AEB_OBS_STATIONARY && L[q].active && !L[q].collided && L[q].s.x > J[q].gap) {
      L[q].collided = true;
      L[q].pend = true;
      if (impact_exit) L[q].active = false;
    }
  }
}

// runs of steady blocks for both samples of every lane (see run_steady)
template <int OBS, int K, int FORM>
HOT int run_steady_x2(Lane64x2 (&L)[2], const Job (&J)[2], const LaneScn (&c)[2], double cmd0,
                      double cmd1, int k, int wl, const double (&thr)[2], int impact_exit) {
  St64 s[2] = {L[0].s, L[1].s};
  do {
    const St64 b0 = s[0], b1 = s[1];
#pragma unroll
    for (int q = 0; q < K / 16; ++q) {
      block64x2<FORM, 16>(s, J, c[0].dt, c[1].dt, cmd0, cmd1);
      asm volatile("" : "+v"(s[0].x), "+v"(s[1].x));
    }
    if (K % 16 != 0) block64x2<FORM, K % 16>(s, J, c[0].dt, c[1].dt, cmd0, cmd1);
    if (OBS == AEB_OBS_STATIONARY) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        if (L[q].active && !L[q].collided && s[q].x > J[q].gap) {
          L[q].sv = q == 0 ? b0 : b1;
          L[q].sk = k;
          L[q].se = k + K;
          L[q].collided = true;
          L[q].pend = true;
          if (impact_exit) L[q].active = false;
        }
      }
    }
    k += K;
  } while (k + K <= wl && __any(L[0].active || L[1].active) &&
           !__any((L[0].active && s[0].v <= thr[0]) || (L[1].active && s[1].v <= thr[1])));
  L[0].s = s[0];
  L[1].s = s[1];
  return k;
}

// the next 128 sorted positions of a wavefront (see next_chunk)
__device__ inline int64_t next_chunk2(unsigned long long* counter, int persistent, int pass,
                                      int64_t n) {
  if (pass == 0)
    return 2 * (static_cast<int64_t>(blockIdx.x) * blockDim.x +
                __builtin_amdgcn_readfirstlane(threadIdx.x & ~63u));
  if (!persistent) return n;
  unsigned long long b = 0;
  if ((threadIdx.x & 63) == 0) b = atomicAdd(counter, 128ull);
  const unsigned lo = __builtin_amdgcn_readfirstlane(static_cast<unsigned>(b));
  const unsigned hi = __builtin_amdgcn_readfirstlane(static_cast<unsigned>(b >> 32));
  return static_cast<int64_t>((static_cast<unsigned long long>(hi) << 32) | lo) +
         2 * static_cast<int64_t>(gridDim.x) * blockDim.x;
}

template <int OBS, int K, bool BATCH>
__global__ __launch_bounds__(256) void k_roll_fp64x2(const Job* __restrict__ jobs,
                                                     const uint32_t* __restrict__ perm,
                                                     int64_t n, Ctx ctx,
                                                     unsigned long long* counter,
                                                     int persistent) {
  if (ctx.hdr) n = ctx.hdr->total;  // a recorded mix: its size from the device header
  constexpr int KS = 4;
  constexpr int KM = K > 16 ? 16 : KS;
  for (int pass = 0;; ++pass) {
    const int64_t base = next_chunk2(counter, persistent, pass, n);
    if (base >= n) break;
    bool valid[2];
    uint32_t g[2];
    Job J[2];
    LaneScn c[2];
    Lane64x2 L[2];
    double thr_k[2], thr_m[2], thr_s[2], dist[2], margin[2];
    float vimp[2];
    int end[2], steps[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int64_t pos = base + 64 * q + (threadIdx.x & 63);
      valid[q] = pos < n;
      g[q] = valid[q] ? perm[pos] : 0u;
      J[q] = valid[q] ? jobs[g[q]] : Job{1.0, 0.0, 0.0, -1.0, 0.5, 1e30, 1.0, 0.0f, 0u};
      c[q] = lane_scn<BATCH>(ctx, J[q], valid[q], g[q]);
      thr_k[q] = static_cast<double>(K) * c[q].dt * J[q].dmax;
      thr_m[q] = static_cast<double>(KM) * c[q].dt * J[q].dmax;
      thr_s[q] = static_cast<double>(KS) * c[q].dt * J[q].dmax;
      L[q].s = St64{0.0, J[q].v0, 0.0};
      L[q].l = Ld64{0.0, 0.0, J[q].gap};
      L[q].sv = L[q].s;
      L[q].sk = L[q].se = 0;
      L[q].active = valid[q];
      L[q].collided = L[q].pend = L[q].clamped = false;
      L[q].free_lane = J[q].alim < c[q].a_cmd - 1e-6;
      L[q].limited = J[q].alim > c[q].a_cmd + 1e-9;
      dist[q] = __builtin_nan("");  // until its end is found
      margin[q] = J[q].gap;
      vimp[q] = 0.0f;
      end[q] = steps[q] = 0;
    }
    const bool varnd = BATCH || ctx.nds;
    int wnd = __builtin_amdgcn_readfirstlane(
        varnd ? wave_min(min(valid[0] ? c[0].nd : INT_MAX, valid[1] ? c[1].nd : INT_MAX))
              : c[0].nd);
    int k = 0, wl = -1;
    for (;;) {
      k = __builtin_amdgcn_readfirstlane(k);
      if (!__any(L[0].active || L[1].active)) break;
      if (!varnd) {
        wl = __builtin_amdgcn_readfirstlane(lane_lim(k, c[0].nd, c[0].nmax));
      } else if (k >= wl) {
        const int l0 = L[0].active ? lane_lim(k, c[0].nd, c[0].nmax) : INT_MAX;
        const int l1 = L[1].active ? lane_lim(k, c[1].nd, c[1].nmax) : INT_MAX;
        wl = wave_min(min(l0, l1));
      }
      if (k + K <= wl && !__any((L[0].active && L[0].s.v <= thr_k[0]) ||
                                (L[1].active && L[1].s.v <= thr_k[1]))) {
        const bool past = k + K > wnd;
        if (past && __all((!L[0].active || L[0].clamped) && (!L[1].active || L[1].clamped))) {
          k = run_steady_x2<OBS, K, FORM_C>(L, J, c, 0.0, 0.0, k, wl, thr_k, ctx.impact_exit);
        } else if (past && __all((!L[0].active || L[0].free_lane) &&
                                 (!L[1].active || L[1].free_lane))) {
          const double cmd0 = k >= c[0].nd ? c[0].a_cmd : 0.0;
          const double cmd1 = k >= c[1].nd ? c[1].a_cmd : 0.0;
          k = run_steady_x2<OBS, K, FORM_F>(L, J, c, cmd0, cmd1, k, wl, thr_k, ctx.impact_exit);
        } else {
          run_block64x2<OBS, K>(L, J, c, k, wnd, ctx.impact_exit);
          k += K;
        }
      } else if (KM > KS && k + KM <= wl &&
                 !__any((L[0].active && L[0].s.v <= thr_m[0]) ||
                        (L[1].active && L[1].s.v <= thr_m[1]))) {
        run_block64x2<OBS, KM>(L, J, c, k, wnd, ctx.impact_exit);
        k += KM;
      } else if (k + KS <= wl && !__any((L[0].active && L[0].s.v <= thr_s[0]) ||
                                        (L[1].active && L[1].s.v <= thr_s[1]))) {
        run_block64x2<OBS, KS>(L, J, c, k, wnd, ctx.impact_exit);
        k += KS;
      } else {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          if (!L[q].active) continue;
          const double cmd = k >= c[q].nd ? c[q].a_cmd : 0.0;
          step64<false, AEB_EULER>(L[q].s, L[q].l, J[q], 0.0, c[q].dt, cmd);
          if (k >= c[q].nd) L[q].clamped = L[q].clamped || (L[q].limited && L[q].s.a <= J[q].alim);
          const bool impact = OBS == AEB_OBS_STATIONARY && L[q].s.x > J[q].gap;
          if (impact && !L[q].collided) {
            L[q].collided = true;
            vimp[q] = static_cast<float>(L[q].s.v);
          }
          if (impact && ctx.impact_exit) {
            L[q].active = false;
            end[q] = AEB_END_IMPACT;
            steps[q] = k + 1;
            dist[q] = L[q].s.x;
          }
          if (L[q].active) {
            if (L[q].s.v <= 0.0) {
              L[q].active = false;
              end[q] = AEB_END_STOP;
              steps[q] = k + 1;
              dist[q] = L[q].s.x;
            } else if (k + 1 >= c[q].nmax) {
              L[q].active = false;
              end[q] = AEB_END_HORIZON;
              steps[q] = k + 1;
              dist[q] = L[q].s.x;
            }
          }
        }
        k += 1;
      }
    }
    // replay the block in which each pending sample passed the obstacle (see
    // k_roll_fp64), one sample of the lane after the other
    if (OBS == AEB_OBS_STATIONARY) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        if (!__any(L[q].pend)) continue;
        St64 r = L[q].sv;
        Ld64 rl{};
        int kr = L[q].sk;
        constexpr int RB = 8;
        const double cmd = kr >= c[q].nd ? c[q].a_cmd : 0.0;
        if (K > RB) {
          bool skip = L[q].pend;
          for (int it = 0; it < K / RB; ++it) {
            skip = skip && kr + RB <= L[q].se;
            if (!__any(skip)) break;
            if (skip) {
              St64 t = r;
              block64<FORM_G, RB, false, AEB_EULER>(t, rl, J[q], 0.0, c[q].dt, cmd);
              if (t.x > J[q].gap) {
                skip = false;
              } else {
                r = t;
                kr += RB;
              }
            }
          }
        }
        for (int it = 0; it <= K; ++it) {
          if (!__any(L[q].pend)) break;
          if (L[q].pend) {
            const double cm = kr >= c[q].nd ? c[q].a_cmd : 0.0;
            step64<false, AEB_EULER>(r, rl, J[q], 0.0, c[q].dt, cm);
            ++kr;
            if (r.x > J[q].gap) {
              L[q].pend = false;
              vimp[q] = static_cast<float>(r.v);
              if (ctx.impact_exit) {
                end[q] = AEB_END_IMPACT;
                steps[q] = kr;
                dist[q] = r.x;
              }
            }
          }
        }
        if (L[q].pend) vimp[q] = __builtin_nanf("");  // unreachable; makes a broken replay visible
      }
    }
    if (ctx.lanes) count_lanes(ctx.lanes, k, 128);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (!valid[q]) continue;
      const double mg = J[q].gap - dist[q];
      margin[q] = mg < J[q].gap ? mg : J[q].gap;
      int64_t i;
      const OutCols o = lane_out<BATCH>(ctx, J[q], g[q], i);
      o.dist[i] = dist[q];
      o.margin[i] = margin[q];
      o.steps[i] = steps[q];
      o.status[i] = static_cast<uint8_t>(end[q] | (L[q].collided ? AEB_COLLIDED : 0));
      o.vimp[i] = L[q].collided ? vimp[q] : 0.0f;
    }
  }
}

// ---------------------------------------------------------------------------
// FP32 compensated block forms.  State: speed (a float, or with SPLIT a float
// base plus an in-block increment carried exactly at block ends), actuator
// deviation e = a - cmd, in-block position sum p and a Kahan pair X that
// absorbs p at every block end.  Forms as in FP64:
//   G: m = max(e + (a_cmd - c), alim - c), e decays;  F: m = e + (a_cmd - c);
//   C: m = alim - c;  D: m = max(-c, alim - c) (e = 0 during the dead time).
// ---------------------------------------------------------------------------
struct L32 {
  float dt, nkd, nkt, alc, tb, td, tdm, ejump, thr, gapf;
};

// A lane whose speed is not split holds it whole in vi, with vb = 0: the sum
// vb + vi is then vi itself and the step's update of vi the plain one, so the
// split step serves both kinds of lanes in one wavefront (running each form
// under its lane mask made the one wavefront that holds both the longest of
// small launches: 25,000 samples 166 us); only the flush tells them apart.
struct St32 {
  float vb, vi, e, p;
  Kahan32 X;
};

template <bool SPLIT>
__device__ inline float speed32(const St32& s) {
  return SPLIT ? s.vb + s.vi : s.vi;
}

template <int FORM, int K, bool SPLIT>
__device__ inline void block32(St32& s, const L32& c, float tk) {
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const float v = speed32<SPLIT>(s);
    const float q = v * v;
    float m;
    if (FORM == FORM_G)
      m = fmaxf(s.e + tk, c.alc);
    else if (FORM == FORM_F)
      m = s.e + tk;
    else if (FORM == FORM_C)
      m = c.alc;
    else
      m = c.tdm;
    const float acc = fmaf(c.nkd, q, m);
    s.p = fmaf(c.dt, v, s.p);
    s.vi = fmaf(c.dt, acc, s.vi);
    if (FORM == FORM_G || FORM == FORM_F) s.e = fmaf(c.nkt, s.e, s.e);
  }
}

// Every 64 steps (by step index, so the rounding of a lane never depends on
// how its wavefront grouped the steps) the speed base absorbs its increment
// and the position's block sum goes into the Kahan pair.
constexpr int FLUSH = 64;

__device__ inline void flush32(St32& s, bool split) {
  if (split) {
    const float t = s.vb + s.vi;
    s.vi = s.vi - (t - s.vb);
    s.vb = t;
  }
  s.X.add(s.p);
  s.p = 0.0f;
}

__device__ inline void step32(St32& s, const L32& c, bool braking) {
  const float v = speed32<true>(s);
  const float q = v * v;
  const float m = fmaxf(s.e + (braking ? c.tb : c.td), c.alc);
  const float acc = fmaf(c.nkd, q, m);
  s.p = fmaf(c.dt, v, s.p);
  s.vi = fmaf(c.dt, acc, s.vi);
  s.e = fmaf(c.nkt, s.e, s.e);
}

// Without compensation the speed's rounding grows with the step count; a
// lane predicted to run longer than this carries it.
constexpr double SPLIT_STEPS = 6000.0;

// Speed compensation is a per-lane property (its predicted length), so a
// lane's arithmetic never depends on its wavefront.
template <int FORM, int K>
HOT void block32_any(St32& s, const L32& c, float tk, lanes_t splits) {
  if (splits == 0)
    block32<FORM, K, false>(s, c, tk);
  else
    block32<FORM, K, true>(s, c, tk);
}

// Lane state and lane sets of the compensated FP32 integration (see Wave64).
struct Wave32 {
  St32 s;
  lanes_t active, crossed, pend, stopped, clamped, free_lane;
};

// Block start states in LDS, as Saves64.
template <int OBS>
struct Saves32 {
  static constexpr int SLOTS = OBS == AEB_OBS_STATIONARY ? 3 : 2;
  float vb[SLOTS][ROLL_MAX], vi[SLOTS][ROLL_MAX], e[SLOTS][ROLL_MAX], p[SLOTS][ROLL_MAX];
  float hi[SLOTS][ROLL_MAX], lo[SLOTS][ROLL_MAX];
  int k[2][ROLL_MAX], end[2][ROLL_MAX];  // of slots SAV_END, SAV_PASS
};

template <int OBS>
HOT void save_start32(const Wave32& L, Saves32<OBS>& S) {
  const int t = threadIdx.x;
  S.vb[SAV_CUR][t] = L.s.vb;
  S.vi[SAV_CUR][t] = L.s.vi;
  S.e[SAV_CUR][t] = L.s.e;
  S.p[SAV_CUR][t] = L.s.p;
  S.hi[SAV_CUR][t] = L.s.X.hi;
  S.lo[SAV_CUR][t] = L.s.X.lo;
}

template <int OBS>
HOT void keep_start32(Saves32<OBS>& S, int slot, int k, int B) {
  const int t = threadIdx.x;
  S.vb[slot][t] = S.vb[SAV_CUR][t];
  S.vi[slot][t] = S.vi[SAV_CUR][t];
  S.e[slot][t] = S.e[SAV_CUR][t];
  S.p[slot][t] = S.p[SAV_CUR][t];
  S.hi[slot][t] = S.hi[SAV_CUR][t];
  S.lo[slot][t] = S.lo[SAV_CUR][t];
  S.k[slot - 1][t] = k;
  S.end[slot - 1][t] = k + B;
}

// What happened to the lanes in the block of B steps from step k (see
// block_events of the FP64 kernel).
template <int OBS>
HOT void block_events32(Wave32& L, Saves32<OBS>& S, const L32& c, int k, int B,
                        int impact_exit) {
  const lanes_t stop = ballot(speed32<true>(L.s) <= 0.0f) & L.active;
  lanes_t hit = 0;
  if (OBS == AEB_OBS_STATIONARY)
    hit = ballot((L.s.X.hi - L.s.X.lo) + L.s.p > c.gapf) & L.active & ~stop & ~L.crossed;
  L.crossed |= hit;
  L.pend |= hit;
  L.stopped |= stop;
  L.active &= ~(stop | (impact_exit ? hit : 0ull));
  if (hit | stop) {
    if (OBS == AEB_OBS_STATIONARY && in(hit))
      keep_start32<OBS>(S, impact_exit ? SAV_END : SAV_PASS, k, B);
    if (in(stop)) keep_start32<OBS>(S, SAV_END, k, B);
    lanes_join();
  }
}

// The lanes whose speed cannot rise over the next block (see falling of the
// FP64 kernel): the actuator's deviation from the command decays from above,
// so the brake term m only falls, and m is below zero.  With the speed split
// into base and increment the flush may move the read speed by the rounding of
// the increment; the bound on m keeps each step's change well above that.
HOT lanes_t falling32(const St32& s, const L32& c, float tk) {
  return ballot(c.nkd <= 0.0f && c.nkt <= 0.0f && c.nkt >= -1.0f && s.e >= 0.0f &&
                fmaxf(s.e + tk, c.alc) < -1e-2f);
}

template <int OBS, int B, bool TOP>
HOT void run_block32(Wave32& L, Saves32<OBS>& S, const L32& c, bool split, lanes_t splits, int nd,
                     int k, int wnd, int impact_exit) {
  save_start32<OBS>(L, S);
  // blocks never straddle nd: the lane's target is fixed for the block
  const float tk = k >= nd ? c.tb : c.td;
  if (k + B <= wnd) {
    block32_any<FORM_D, B>(L.s, c, tk, splits);
  } else if (!TOP && (L.active & ~L.clamped) == 0) {
    block32_any<FORM_C, B>(L.s, c, tk, splits);
  } else if (!TOP && (L.active & ~L.free_lane) == 0) {
    block32_any<FORM_F, B>(L.s, c, tk, splits);
  } else {
    block32_any<FORM_G, B>(L.s, c, tk, splits);
    L.clamped |= ballot(k + B > nd && L.s.e + c.tb <= c.alc);
  }
  if ((k + B) % FLUSH == 0) flush32(L.s, split);
  block_events32<OBS>(L, S, c, k, B, impact_exit);
}

// (see long_block of the FP64 kernel; thr: the speed above which no lane can
// stop inside the block)
HOT bool long_block32(const Wave32& L, float thr, lanes_t fall) {
  const float v = speed32<true>(L.s);
  const lanes_t low = ballot(v <= thr) & L.active;
  if (low == 0) return true;
  return (low & ~fall) == 0 && (ballot(v > 2.0f * thr) & L.active) != 0;
}

// K-step pieces of a run between its tests: two, unrolled, for a wavefront with
// split speeds in a batched launch, whose wavefronts are long and many, so that
// the tests' share is worth a longer replay of the block with the crossing or the
// stop (1,000 uneven scenarios, most of their steps split: kernel 30.1 ms with
// one, 29.6 with two); one elsewhere (1,048,576 samples of one scenario 0.551 ms,
// 0.565 with two; 200,000 0.150 and 0.159).
template <int K, bool BATCH>
constexpr int run_pieces() { return BATCH && K == FLUSH ? 2 : 1; }

// Whether U pieces from step k stay below the block limit wl with every stop
// inside them found at their end: asked before each of a run's rounds, the first
// included.
template <int K, int U>
HOT bool run_fits32(const Wave32& L, const L32& c, int k, int wl, lanes_t fall) {
  return k + U * K <= wl && long_block32(L, U * c.thr, fall);
}

// Consecutive K-step blocks in one steady form, SPLIT if any lane's speed is
// split, U of them between tests (as run_steady of the FP64 kernel), with the
// flush at every flush point.  The caller has asked run_fits32 of the first U.
// (Two blocks per round of tests, the second in a rolled loop: no faster for one
// wavefront on its SIMD, and 35 more VGPRs.)
template <int OBS, int K, int FORM, bool SPLIT, int U>
HOT int run_steady32(Wave32& L, Saves32<OBS>& S, const L32& c, float tk, bool split, int k,
                     int wl, lanes_t fall, int impact_exit) {
  do {
    k = __builtin_amdgcn_readfirstlane(k);
    save_start32<OBS>(L, S);
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int q = 0; q < K / 16; ++q) {
        block32<FORM, 16, SPLIT>(L.s, c, tk);
        asm volatile("" : "+v"(L.s.p));  // no position update sunk to the end of the run
      }
      if (K == FLUSH || (k + K) % FLUSH == 0) flush32(L.s, SPLIT && split);
    }
    block_events32<OBS>(L, S, c, k, U * K, impact_exit);
    k += U * K;
  } while (L.active != 0 && run_fits32<K, U>(L, c, k, wl, fall));
  return k;
}

template <int OBS, int K, bool BATCH>
__global__ __launch_bounds__(ROLL_MAX) void k_roll_fp32c(const Job* __restrict__ jobs,
                                                         const uint32_t* __restrict__ perm,
                                                         int64_t n, Ctx ctx, double band_abs,
                                                         double band_rel, uint32_t* fix,
                                                         unsigned long long* counter,
                                                         int persistent) {
  if (ctx.hdr) n = ctx.hdr->total;  // a recorded mix: its size from the device header
  // the block ladder of the FP64 kernel, blocks starting on multiples of their length
  constexpr int KS = 4;
  constexpr int KM = K >= 64 ? 16 : KS;  // middle level of the block ladder
  static_assert(FLUSH % K == 0 && K % KM == 0 && KM % KS == 0,
                "flush points must fall on block ends");
  __shared__ Saves32<OBS> sav;
  for (int pass = 0;; ++pass) {
    const int64_t base = next_chunk(counter, persistent, pass, n);
    if (base >= n) break;
    const int64_t pos = base + (threadIdx.x & 63);
    const bool valid = pos < n;
    const uint32_t g = valid ? perm[pos] : 0u;
    Job J;
    if (valid) {
      J = jobs[g];
    } else {
      J = Job{1.0, 0.0, 0.0, -1.0, 0.5, 1e30, 1.0, 0.0f, 0u};
    }
    // the scenario's constants and limits as lane values, also for one scenario
    // (the limits then take the per-lane path: the same values in every lane)
    const LaneScn sc = BATCH ? lane_scn<BATCH>(ctx, J, valid, g)
                             : lane_values(lane_scn<BATCH>(ctx, J, valid, g));
    const int nd = sc.nd, nmax = sc.nmax;
    const int wnd = __builtin_amdgcn_readfirstlane(wave_min(valid ? nd : INT_MAX));
    L32 c;  // (the speed read below is base + increment; the increment is 0 without compensation)
    c.dt = static_cast<float>(sc.dt);
    c.nkd = static_cast<float>(J.nkd);
    c.nkt = static_cast<float>(-J.kt);
    c.alc = static_cast<float>(J.alim - J.c);
    c.tb = static_cast<float>(sc.a_cmd - J.c);
    c.td = static_cast<float>(0.0 - J.c);
    c.tdm = fmaxf(c.td, c.alc);
    c.ejump = static_cast<float>(-sc.a_cmd);
    c.thr = static_cast<float>(static_cast<double>(K) * sc.dt * J.dmax);
    c.gapf = static_cast<float>(J.gap);
    const float thr_m = static_cast<float>(static_cast<double>(KM) * sc.dt * J.dmax);
    const float thr_s = static_cast<float>(static_cast<double>(KS) * sc.dt * J.dmax);
    const double band = band_abs + band_rel * fabs(J.gap);
    const bool split = J.pred > SPLIT_STEPS;  // per lane
    const lanes_t splits = ballot(split);
    Wave32 L;
    const float v0f = static_cast<float>(J.v0);
    L.s.vb = split ? v0f : 0.0f;
    L.s.vi = split ? static_cast<float>(J.v0 - static_cast<double>(v0f)) : v0f;
    L.s.e = 0.0f;
    L.s.p = 0.0f;
    L.active = ballot(valid);
    L.crossed = L.pend = L.stopped = L.clamped = 0;
    L.free_lane = ballot(J.alim < sc.a_cmd - 1e-6);
    const int impact_exit = ctx.impact_exit;
    bool boundary = false;
    int end = 0, steps = 0;
    // (until the lane's end, or its impact, is found: a broken replay is visible)
    double dist = __builtin_nan("");
    float vimp = __builtin_nanf("");
    int k = 0, wl = -1;
    while (L.active) {
      // the step index is the same in every lane: keep it (and the branches on it) scalar
      k = __builtin_amdgcn_readfirstlane(k);
      if (k >= wl) wl = wave_lim(true, in(L.active), k, nd, nmax);
      // the command switches on at step nd: e = a - cmd jumps by -a_cmd.  Blocks
      // never straddle nd, so every lane passes through k == nd at a loop top.
      L.s.e += k == nd ? c.ejump : 0.0f;
      const float v_now = speed32<true>(L.s);
      const float tk = k >= nd ? c.tb : c.td;
      lanes_t fall = ~0ull;
      if (ballot(v_now <= c.thr) & L.active) fall = falling32(L.s, c, tk);
      // blocks start on multiples of their length, so flush points fall on block ends
      if (k % K == 0 && k + K <= wl && long_block32(L, c.thr, fall)) {
        // past every lane's dead time, in a form no later block changes: a run
        // of blocks
        const lanes_t f = falling32(L.s, c, tk);
        const bool no_split = (splits & L.active) == 0;
        // (one piece fits: just tested; U of them before a run with split speeds)
        constexpr int U = run_pieces<K, BATCH>();
        const bool past =
            k + K > wnd && (no_split || U == 1 || run_fits32<K, U>(L, c, k, wl, f));
        const bool steady_c = past && (L.active & ~L.clamped) == 0;
        const bool steady_f = past && !steady_c && (L.active & ~L.free_lane) == 0;
        const bool steady_g = past && (L.active & ~(L.clamped | L.free_lane)) == 0;
        // (calls, not a lambda that captures k: 1,048,576 samples without an
        // obstacle 0.493 against 0.528 ms)
        if (steady_c && no_split) {
          k = run_steady32<OBS, K, FORM_C, false, 1>(L, sav, c, tk, split, k, wl, f,
                                                     impact_exit);
        } else if (steady_f && no_split) {
          k = run_steady32<OBS, K, FORM_F, false, 1>(L, sav, c, tk, split, k, wl, f,
                                                     impact_exit);
        } else if (steady_c) {
          k = run_steady32<OBS, K, FORM_C, true, U>(L, sav, c, tk, split, k, wl, f,
                                                     impact_exit);
        } else if (steady_f) {
          k = run_steady32<OBS, K, FORM_F, true, U>(L, sav, c, tk, split, k, wl, f,
                                                     impact_exit);
        } else if (steady_g && (no_split || U == 1)) {
          // both kinds: the generic form, whose step serves either
          k = run_steady32<OBS, K, FORM_G, true, 1>(L, sav, c, tk, split, k, wl, f,
                                                     impact_exit);
        } else if (steady_g) {
          k = run_steady32<OBS, K, FORM_G, true, U>(L, sav, c, tk, split, k, wl, f,
                                                     impact_exit);
        } else {
          run_block32<OBS, K, U == 1>(L, sav, c, split, splits & L.active, nd, k, wnd,
                                      impact_exit);
          k += K;
        }
      } else if (KM > KS && k % KM == 0 && k + KM <= wl &&
                 (ballot(v_now <= thr_m) & L.active & ~fall) == 0) {
        run_block32<OBS, KM, false>(L, sav, c, split, splits & L.active, nd, k, wnd, impact_exit);
        k += KM;
      } else if (k % KS == 0 && k + KS <= wl &&
                 (ballot(v_now <= thr_s) & L.active & ~fall) == 0) {
        run_block32<OBS, KS, false>(L, sav, c, split, splits & L.active, nd, k, wnd, impact_exit);
        k += KS;
      } else {
        bool clamp = false, cross = false, done = false;
        if (in(L.active)) {
          const float vb = v_now;
          step32(L.s, c, k >= nd);
          if ((k + 1) % FLUSH == 0) flush32(L.s, split);
          clamp = k >= nd && L.s.e + c.tb <= c.alc;
          const float v = speed32<true>(L.s);
          if (OBS == AEB_OBS_STATIONARY && !in(L.crossed) &&
              (L.s.X.hi - L.s.X.lo) + L.s.p > c.gapf) {
            cross = true;
            vimp = v;
            if (impact_exit) {
              end = AEB_END_IMPACT;
              const double x = L.s.X.value(L.s.p);
              const double step_len = static_cast<double>(c.dt) * static_cast<double>(vb);
              boundary = fabs(x - J.gap) < band || fabs(J.gap - (x - step_len)) < band;
            }
          }
          if (end == 0) {
            if (v <= 0.0f)
              end = AEB_END_STOP;
            else if (k + 1 >= nmax)
              end = AEB_END_HORIZON;
          }
          done = end != 0;
          if (done) {
            steps = k + 1;
            dist = L.s.X.value(L.s.p);
          }
        }
        lanes_join();
        L.clamped |= ballot(clamp);
        if (OBS == AEB_OBS_STATIONARY) L.crossed |= ballot(cross);
        L.active &= ~ballot(done);
        k += 1;
      }
    }
    // replay the blocks in which lanes passed the obstacle, and those in which
    // they stopped (see the FP64 kernel): chunks of RB steps that hold no event
    // whole, then single steps with every test.  The crossing recurs within the
    // block (at its last step at the latest, where the block-end test fired).
    auto replay = [&](lanes_t who, int slot, bool to_stop) {
      const int t = threadIdx.x;
      bool go = in(who);
      St32 r = L.s;
      int kr = 0, se = 0;
      if (go) {
        r.vb = sav.vb[slot][t];
        r.vi = sav.vi[slot][t];
        r.e = sav.e[slot][t];
        r.p = sav.p[slot][t];
        r.X.hi = sav.hi[slot][t];
        r.X.lo = sav.lo[slot][t];
        kr = sav.k[slot - 1][t];
        se = sav.end[slot - 1][t];
      }
      // a stopped lane may also have passed the obstacle in the same block
      bool seek = OBS == AEB_OBS_STATIONARY && (!to_stop || !in(L.crossed));
      bool passed = false;
      constexpr int RB = 8;
      if (K > RB) {
        const float tk = kr >= nd ? c.tb : c.td;  // one target over a block
        bool skip = go;
        for (int it = 0; it < run_pieces<K, BATCH>() * K / RB; ++it) {
          skip = skip && kr % RB == 0 && kr + RB <= se;
          if (ballot(skip) == 0) break;
          if (skip) {
            St32 q = r;
            block32<FORM_G, RB, true>(q, c, tk);
            if ((kr + RB) % FLUSH == 0) flush32(q, split);
            if ((seek && (q.X.hi - q.X.lo) + q.p > c.gapf) ||
                (to_stop && speed32<true>(q) <= 0.0f)) {
              skip = false;
            } else {
              r = q;
              kr += RB;
            }
          }
        }
      }
      for (int it = 0; it < run_pieces<K, BATCH>() * K; ++it) {
        if (ballot(go) == 0) break;
        if (go) {
          const float vb = speed32<true>(r);
          step32(r, c, kr >= nd);
          ++kr;
          if (kr % FLUSH == 0) flush32(r, split);
          const float v = speed32<true>(r);
          if (seek && (r.X.hi - r.X.lo) + r.p > c.gapf) {
            passed = true;
            seek = false;
            vimp = v;
            if (impact_exit) {
              end = AEB_END_IMPACT;
              steps = kr;
              dist = r.X.value(r.p);
              const double step_len = static_cast<double>(c.dt) * static_cast<double>(vb);
              boundary = fabs(dist - J.gap) < band || fabs(J.gap - (dist - step_len)) < band;
              go = false;
            }
            if (!to_stop) go = false;
          }
          if (to_stop && go && v <= 0.0f) {
            end = AEB_END_STOP;
            steps = kr;
            dist = r.X.value(r.p);
            go = false;
          }
        }
      }
      lanes_join();
      if (OBS == AEB_OBS_STATIONARY) L.crossed |= ballot(passed);
    };
    if (OBS == AEB_OBS_STATIONARY && L.pend)
      replay(L.pend, impact_exit ? SAV_END : SAV_PASS, false);
    if (L.stopped) replay(L.stopped, SAV_END, true);
    bool collided = in(L.crossed);
    if (OBS == AEB_OBS_STATIONARY && !impact_exit) {
      // the flag is decided in FP64 on the compensated distance
      collided = dist > J.gap;
      boundary = fabs(J.gap - dist) < band;
      if (collided != in(L.crossed)) vimp = 0.0f;
    } else if (OBS == AEB_OBS_STATIONARY && !in(L.crossed)) {
      boundary = J.gap - dist < band;
    }
    if (ctx.lanes) count_lanes(ctx.lanes, k, 64);
    if (valid) {
      const double mg = J.gap - dist;
      int64_t i;
      const OutCols o = lane_out<BATCH>(ctx, J, g, i);
      o.dist[i] = dist;
      o.margin[i] = mg < J.gap ? mg : J.gap;
      o.steps[i] = steps;
      o.status[i] = static_cast<uint8_t>(end | (collided ? AEB_COLLIDED : 0) |
                                         (boundary ? AEB_BOUNDARY : 0));
      o.vimp[i] = collided ? vimp : 0.0f;
      if (boundary && fix) {
        const uint32_t slot = atomicAdd(fix, 1u);
        fix[1 + slot] = g;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// FP32 compensated form with a lead vehicle.  The clearance is integrated
// directly, c' = c + dt (v_lead - v), as an in-block sum plus a Kahan pair,
// so no two large positions are ever subtracted; both speeds are a float
// base plus an in-block increment.  A lane's clearance after a step is read
// after that step's flush (every 64 steps by index) in every path, and its
// running minimum is the margin.  A crossing inside a block (minimum below
// zero) is replayed from the block's start state; the rollout ends there.
// ---------------------------------------------------------------------------
struct Ld32 {
  float vb, vi;  // lead speed: base + increment (read clamped at 0)
  float pg;      // in-block clearance sum
  Kahan32 G;     // clearance
  float gmin;    // running minimum of the clearance after each step
};

__device__ inline float lead_speed(const Ld32& l) { return fmaxf(l.vb + l.vi, 0.0f); }
__device__ inline float clearance(const Ld32& l) { return (l.G.hi - l.G.lo) + l.pg; }

__device__ inline void flush32l(St32& s, Ld32& l) {
  flush32(s, true);
  const float t = l.vb + l.vi;
  l.vi = l.vi - (t - l.vb);
  l.vb = t;
  l.G.add(l.pg);
  l.pg = 0.0f;
}

// one step of ego and lead (the ego's form as in block32, speed always split)
template <int FORM>
__device__ inline void step32l(St32& s, Ld32& l, const L32& c, float tk, float al) {
  const float v = s.vb + s.vi;
  const float vl = lead_speed(l);
  const float q = v * v;
  float m;
  if (FORM == FORM_G)
    m = fmaxf(s.e + tk, c.alc);
  else if (FORM == FORM_F)
    m = s.e + tk;
  else if (FORM == FORM_C)
    m = c.alc;
  else
    m = c.tdm;
  const float acc = fmaf(c.nkd, q, m);
  s.p = fmaf(c.dt, v, s.p);
  l.pg = fmaf(c.dt, vl - v, l.pg);
  l.vi = fmaf(-c.dt, al, l.vi);
  s.vi = fmaf(c.dt, acc, s.vi);
  if (FORM == FORM_G || FORM == FORM_F) s.e = fmaf(c.nkt, s.e, s.e);
}

template <int FORM, int K>
HOT void block32l(St32& s, Ld32& l, const L32& c, float tk, float al, bool flush_end) {
  float ghl = l.G.hi - l.G.lo;
#pragma unroll
  for (int j = 0; j < K; ++j) {
    step32l<FORM>(s, l, c, tk, al);
    if (j == K - 1 && flush_end) {
      flush32l(s, l);
      ghl = l.G.hi - l.G.lo;
    }
    l.gmin = fminf(l.gmin, ghl + l.pg);
  }
}

// Lane state and lane sets (see Wave64; ended: ended inside a block, to be replayed).
struct Wave32L {
  St32 s;
  Ld32 l;
  lanes_t active, ended, clamped, free_lane, tame, dropped;
};

// Block start states in LDS, as Saves64: every lane ends in its last block.
struct Saves32L {
  float f[2][12][ROLL_MAX];
  int k[ROLL_MAX], end[ROLL_MAX];
};

HOT void save_start32l(const Wave32L& L, Saves32L& S) {
  const int t = threadIdx.x;
  S.f[SAV_CUR][0][t] = L.s.vb;
  S.f[SAV_CUR][1][t] = L.s.vi;
  S.f[SAV_CUR][2][t] = L.s.e;
  S.f[SAV_CUR][3][t] = L.s.p;
  S.f[SAV_CUR][4][t] = L.s.X.hi;
  S.f[SAV_CUR][5][t] = L.s.X.lo;
  S.f[SAV_CUR][6][t] = L.l.vb;
  S.f[SAV_CUR][7][t] = L.l.vi;
  S.f[SAV_CUR][8][t] = L.l.pg;
  S.f[SAV_CUR][9][t] = L.l.G.hi;
  S.f[SAV_CUR][10][t] = L.l.G.lo;
  S.f[SAV_CUR][11][t] = L.l.gmin;
}

// The lanes that ended in the block of B steps from step k: reached the lead
// (its replay finds which came first), or stopped.
template <bool DROP>
HOT void block_events32l(Wave32L& L, Saves32L& S, int k, int B) {
  lanes_t over = ballot(L.s.vb + L.s.vi <= 0.0f) & L.active;
  if (!DROP) over |= ballot(L.l.gmin < 0.0f) & L.active;
  L.ended |= over;
  L.active &= ~over;
  if (over) {
    if (in(over)) {
      const int t = threadIdx.x;
#pragma unroll
      for (int q = 0; q < 12; ++q) S.f[SAV_END][q][t] = S.f[SAV_CUR][q][t];
      S.k[t] = k;
      S.end[t] = k + B;
    }
    lanes_join();
  }
}

// The lanes out of the lead's reach (see out_of_reach of the FP64 kernel).  The
// step's rounding is that of the two increments, below 4 * 2^-24 * 64 dt
// (dmax + al) <= 1.6e-3 dt for the rates `tame` admits, against a gain of at
// least 1e-2 dt in the speed difference; the clearance is read to a few units in
// its last place.
HOT lanes_t out_of_reach32(const Wave32L& L, const L32& c, float tk, float al, lanes_t fall) {
  const float g = clearance(L.l);
  return fall & L.tame &
         ballot(fmaxf(L.s.e + tk, c.alc) < -al - 1e-2f &&
                L.s.vb + L.s.vi < lead_speed(L.l) - 1e-2f &&
                g > L.l.gmin + (1e-3f + 1e-6f * fabsf(g)));
}

// B steps of one form with the lead, or without it (DROP), pieces of 16 with the
// position's sum pinned at the end of each (see run_steady32)
template <int FORM, int B, bool DROP>
HOT void steps32l(Wave32L& L, const L32& c, float tk, float al, bool flush_end) {
  constexpr int P = B < 16 ? B : 16;
#pragma unroll
  for (int q = 0; q < B / P; ++q) {
    const bool fl = flush_end && q == B / P - 1;
    if (DROP) {
      block32<FORM, P, true>(L.s, c, tk);
      if (fl) flush32(L.s, true);
    } else {
      block32l<FORM, P>(L.s, L.l, c, tk, al, fl);
    }
    asm volatile("" : "+v"(L.s.p));
  }
}

template <int B, bool TOP, bool DROP>
HOT void run_block32l(Wave32L& L, Saves32L& S, const L32& c, float al, int nd, int k, int wnd) {
  save_start32l(L, S);
  const float tk = k >= nd ? c.tb : c.td;
  const bool fl = (k + B) % FLUSH == 0;
  if (k + B <= wnd) {
    steps32l<FORM_D, B, DROP>(L, c, tk, al, fl);
  } else if (!TOP && (L.active & ~L.clamped) == 0) {
    steps32l<FORM_C, B, DROP>(L, c, tk, al, fl);
  } else if (!TOP && (L.active & ~L.free_lane) == 0) {
    steps32l<FORM_F, B, DROP>(L, c, tk, al, fl);
  } else {
    steps32l<FORM_G, B, DROP>(L, c, tk, al, fl);
    L.clamped |= ballot(k + B > nd && L.s.e + c.tb <= c.alc);
  }
  block_events32l<DROP>(L, S, k, B);
}

HOT bool long_block32l(const Wave32L& L, float thr, lanes_t fall) {
  const float v = L.s.vb + L.s.vi;
  const lanes_t low = ballot(v <= thr) & L.active;
  if (low == 0) return true;
  return (low & ~fall) == 0 && (ballot(v > 2.0f * thr) & L.active) != 0;
}

template <int K, int FORM, bool DROP>
HOT int run_steady32l(Wave32L& L, Saves32L& S, const L32& c, float tk, float al, int k, int wl,
                      lanes_t fall) {
  bool more;
  do {
    k = __builtin_amdgcn_readfirstlane(k);
    save_start32l(L, S);
    steps32l<FORM, K, DROP>(L, c, tk, al, K == FLUSH || (k + K) % FLUSH == 0);
    block_events32l<DROP>(L, S, k, K);
    k += K;
    more = k + K <= wl && L.active != 0 && long_block32l(L, c.thr, fall);
    if (!DROP)  // every lane out of the lead's reach: the caller drops it
      more = more && (L.active & ~out_of_reach32(L, c, tk, al, fall)) != 0;
  } while (more);
  return k;
}

template <int K, bool BATCH>
__global__ __launch_bounds__(ROLL_MAX) void k_roll_fp32c_lead(const Job* __restrict__ jobs,
                                                         const LeadJob* __restrict__ leads,
                                                         const uint32_t* __restrict__ perm,
                                                         int64_t n, Ctx ctx, double band_abs,
                                                         double band_rel, uint32_t* fix,
                                                         unsigned long long* counter,
                                                         int persistent) {
  if (ctx.hdr) n = ctx.hdr->total;  // a recorded mix: its size from the device header
  // the block ladder of the FP64 kernel, blocks starting on multiples of their length
  constexpr int KS = 4;
  constexpr int KM = K >= 64 ? 16 : KS;  // middle level of the block ladder
  static_assert(FLUSH % K == 0 && K % KM == 0 && KM % KS == 0,
                "flush points must fall on block ends");
  __shared__ Saves32L sav;
  for (int pass = 0;; ++pass) {
    const int64_t base = next_chunk(counter, persistent, pass, n);
    if (base >= n) break;
    const int64_t pos = base + (threadIdx.x & 63);
    const bool valid = pos < n;
    const uint32_t g = valid ? perm[pos] : 0u;
    Job J;
    if (valid) {
      J = jobs[g];
    } else {
      J = Job{1.0, 0.0, 0.0, -1.0, 0.5, 1e30, 1.0, 0.0f, 0u};
    }
    const float al = valid ? static_cast<float>(leads[g].decel) : 0.0f;
    const LaneScn sc = BATCH ? lane_scn<BATCH>(ctx, J, valid, g)
                             : lane_values(lane_scn<BATCH>(ctx, J, valid, g));
    const int nd = sc.nd, nmax = sc.nmax;
    const int wnd = __builtin_amdgcn_readfirstlane(wave_min(valid ? nd : INT_MAX));
    L32 c;
    c.dt = static_cast<float>(sc.dt);
    c.nkd = static_cast<float>(J.nkd);
    c.nkt = static_cast<float>(-J.kt);
    c.alc = static_cast<float>(J.alim - J.c);
    c.tb = static_cast<float>(sc.a_cmd - J.c);
    c.td = static_cast<float>(0.0 - J.c);
    c.tdm = fmaxf(c.td, c.alc);
    c.ejump = static_cast<float>(-sc.a_cmd);
    c.thr = static_cast<float>(static_cast<double>(K) * sc.dt * J.dmax);
    c.gapf = static_cast<float>(J.gap);
    const float thr_m = static_cast<float>(static_cast<double>(KM) * sc.dt * J.dmax);
    const float thr_s = static_cast<float>(static_cast<double>(KS) * sc.dt * J.dmax);
    const double band = band_abs + band_rel * fabs(J.gap);
    Wave32L L;
    L.s.vb = static_cast<float>(J.v0);
    L.s.vi = static_cast<float>(J.v0 - static_cast<double>(L.s.vb));
    L.s.e = 0.0f;
    L.s.p = 0.0f;
    L.l.vb = L.s.vb;
    L.l.vi = L.s.vi;
    L.l.pg = 0.0f;
    L.l.G.hi = c.gapf;
    L.l.G.lo = static_cast<float>(static_cast<double>(c.gapf) - J.gap);
    L.l.gmin = clearance(L.l);
    L.active = ballot(valid);
    L.ended = L.clamped = L.dropped = 0;
    L.free_lane = ballot(J.alim < sc.a_cmd - 1e-6);
    L.tame = ballot(al >= 0.0f && J.dmax + al < 100.0);
    bool boundary = false, collided = false;
    int end = 0, steps = 0;
    double dist = __builtin_nan("");  // until the lane's end is found
    float vimp = 0.0f;
    float gm_end = L.l.gmin;  // running minimum of the clearance when the lane ended
    int k = 0, wl = -1;
    auto run = [&](auto form, bool drop, float tk, int kk, int lim, lanes_t f) {
      constexpr int FORM = decltype(form)::value;
      return drop ? run_steady32l<K, FORM, true>(L, sav, c, tk, al, kk, lim, f)
                  : run_steady32l<K, FORM, false>(L, sav, c, tk, al, kk, lim, f);
    };
    auto block = [&](auto len, auto top, bool drop, int kk) {
      constexpr int B = decltype(len)::value;
      constexpr bool TOP = decltype(top)::value;
      if (drop)
        run_block32l<B, TOP, true>(L, sav, c, al, nd, kk, wnd);
      else
        run_block32l<B, TOP, false>(L, sav, c, al, nd, kk, wnd);
    };
    while (L.active) {
      k = __builtin_amdgcn_readfirstlane(k);
      if (k >= wl) wl = wave_lim(true, in(L.active), k, nd, nmax);
      L.s.e += k == nd ? c.ejump : 0.0f;
      const float v_now = L.s.vb + L.s.vi;
      const float tk = k >= nd ? c.tb : c.td;
      lanes_t fall = ~0ull;
      if (ballot(v_now <= c.thr) & L.active) fall = falling32(L.s, c, tk);
      // past the command of every lane, each speed that falls does so for good
      const lanes_t past_nd = ballot(k >= nd);
      if (L.dropped == 0 && k >= wnd &&
          (L.active & ~out_of_reach32(L, c, tk, al, falling32(L.s, c, tk) & past_nd)) == 0)
        L.dropped = L.active;
      const bool drop = L.dropped != 0;
      if (k % K == 0 && k + K <= wl && long_block32l(L, c.thr, fall)) {
        // (see the kernel without a lead)
        const bool past = k + K > wnd && (L.active & ~past_nd) == 0;
        const lanes_t f = falling32(L.s, c, tk);
        if (past && (L.active & ~L.clamped) == 0) {
          k = run(std::integral_constant<int, FORM_C>(), drop, tk, k, wl, f);
        } else if (past && (L.active & ~L.free_lane) == 0) {
          k = run(std::integral_constant<int, FORM_F>(), drop, tk, k, wl, f);
        } else if (past && (L.active & ~(L.clamped | L.free_lane)) == 0) {
          k = run(std::integral_constant<int, FORM_G>(), drop, tk, k, wl, f);
        } else {
          block(std::integral_constant<int, K>(), std::true_type(), drop, k);
          k += K;
        }
      } else if (KM > KS && k % KM == 0 && k + KM <= wl &&
                 (ballot(v_now <= thr_m) & L.active & ~fall) == 0) {
        block(std::integral_constant<int, KM>(), std::false_type(), drop, k);
        k += KM;
      } else if (k % KS == 0 && k + KS <= wl &&
                 (ballot(v_now <= thr_s) & L.active & ~fall) == 0) {
        block(std::integral_constant<int, KS>(), std::false_type(), drop, k);
        k += KS;
      } else {
        bool clamp = false, done = false;
        if (in(L.active)) {
          const float gp = clearance(L.l);
          bool impact = false;
          if (drop) {
            step32(L.s, c, k >= nd);
            if ((k + 1) % FLUSH == 0) flush32(L.s, true);
          } else {
            step32l<FORM_G>(L.s, L.l, c, tk, al);
            if ((k + 1) % FLUSH == 0) flush32l(L.s, L.l);
            const float gk = clearance(L.l);
            L.l.gmin = fminf(L.l.gmin, gk);
            impact = gk < 0.0f;
            if (impact)
              boundary =
                  fabs(static_cast<double>(gp)) < band || fabs(static_cast<double>(gk)) < band;
          }
          clamp = k >= nd && L.s.e + c.tb <= c.alc;
          const float v = L.s.vb + L.s.vi;
          if (impact) {
            collided = true;
            vimp = v - lead_speed(L.l);
            end = AEB_END_IMPACT;
          } else if (v <= 0.0f) {
            end = AEB_END_STOP;
          } else if (k + 1 >= nmax) {
            end = AEB_END_HORIZON;
          }
          done = end != 0;
          if (done) {
            steps = k + 1;
            dist = L.s.X.value(L.s.p);
            gm_end = L.l.gmin;
          }
        }
        lanes_join();
        L.clamped |= ballot(clamp);
        L.active &= ~ballot(done);
        k += 1;
      }
    }
    // replay the block in which each ended lane reached the lead or stopped: the
    // same steps, chunks of RB without either whole, then one at a time with the
    // clearance read after each (post-flush); a dropped lead is not reached, and
    // its running minimum stands
    if (L.ended) {
      const int t = threadIdx.x;
      bool go = in(L.ended);
      const bool seek = !in(L.dropped);
      St32 r = L.s;
      Ld32 rl = L.l;
      int kr = 0, se = 0;
      if (go) {
        r.vb = sav.f[SAV_END][0][t];
        r.vi = sav.f[SAV_END][1][t];
        r.e = sav.f[SAV_END][2][t];
        r.p = sav.f[SAV_END][3][t];
        r.X.hi = sav.f[SAV_END][4][t];
        r.X.lo = sav.f[SAV_END][5][t];
        rl.vb = sav.f[SAV_END][6][t];
        rl.vi = sav.f[SAV_END][7][t];
        rl.pg = sav.f[SAV_END][8][t];
        rl.G.hi = sav.f[SAV_END][9][t];
        rl.G.lo = sav.f[SAV_END][10][t];
        rl.gmin = sav.f[SAV_END][11][t];
        kr = sav.k[t];
        se = sav.end[t];
        gm_end = rl.gmin;
      }
      constexpr int RB = 8;
      if (K > RB) {
        const float tk = kr >= nd ? c.tb : c.td;  // one target over a block
        bool skip = go;
        for (int it = 0; it < K / RB; ++it) {
          skip = skip && kr % RB == 0 && kr + RB <= se;
          if (ballot(skip) == 0) break;
          if (skip) {
            St32 q = r;
            Ld32 ql = rl;
            block32l<FORM_G, RB>(q, ql, c, tk, al, (kr + RB) % FLUSH == 0);
            if ((seek && ql.gmin < 0.0f) || q.vb + q.vi <= 0.0f) {
              skip = false;
            } else {
              r = q;
              rl = ql;
              kr += RB;
            }
          }
        }
      }
      for (int it = 0; it <= K; ++it) {
        if (ballot(go) == 0) break;
        if (go) {
          const float gprev = clearance(rl);
          step32l<FORM_G>(r, rl, c, kr >= nd ? c.tb : c.td, al);
          ++kr;
          if (kr % FLUSH == 0) flush32l(r, rl);
          const float gk = clearance(rl);
          rl.gmin = fminf(rl.gmin, gk);
          const float v = r.vb + r.vi;
          if (seek && gk < 0.0f) {
            go = false;
            collided = true;
            vimp = v - lead_speed(rl);
            end = AEB_END_IMPACT;
            boundary =
                fabs(static_cast<double>(gprev)) < band || fabs(static_cast<double>(gk)) < band;
          } else if (v <= 0.0f) {
            go = false;
            end = AEB_END_STOP;
          }
          if (!go) {
            steps = kr;
            dist = r.X.value(r.p);
            if (seek) gm_end = rl.gmin;
          }
        }
      }
    }
    if (!collided) boundary = static_cast<double>(gm_end) < band;
    if (ctx.lanes) count_lanes(ctx.lanes, k, 64);
    if (valid) {
      int64_t i;
      const OutCols o = lane_out<BATCH>(ctx, J, g, i);
      o.dist[i] = dist;
      o.margin[i] = static_cast<double>(gm_end);
      o.steps[i] = steps;
      o.status[i] = static_cast<uint8_t>(end | (collided ? AEB_COLLIDED : 0) |
                                         (boundary ? AEB_BOUNDARY : 0));
      o.vimp[i] = collided ? vimp : 0.0f;
      if (boundary && fix) {
        const uint32_t slot = atomicAdd(fix, 1u);
        fix[1 + slot] = g;
      }
    }
  }
}

}  // namespace

// The block path counts steps in int and tests k + (block length) and
// k + (command delay): the horizon and the dead time together stay this far
// below 2^31 (longer runs take the checked FP64 kernel, which counts in 64 bits).
bool block_steps_ok(const aeb_scenario& s) {
  return horizon_steps(s) + dead_steps(s) <= BLOCK_STEP_MAX;
}

bool fast_path_applies(const aeb_scenario& s, int precision) {
  if (!block_steps_ok(s)) return false;
  // the controller: FP64 only (explicit Euler, fused or unfused, or RK4)
  if (control_on(s)) return precision == AEB_FP64;
  if (precision == AEB_FP64) return s.obstacle != AEB_OBS_LEAD || s.integrator != AEB_RK4;
  if (s.integrator != AEB_EULER) return false;
  return precision == AEB_FP32C || precision == AEB_FP32C_FIXUP;
}

namespace {

// Launch shape of the integration kernel from the tuning table: workgroup
// size, and either one pass over ceil(n / block) workgroups or a persistent
// grid of `waves_per_simd` wavefronts per SIMD claiming work from the counter.
struct Shape {
  unsigned grid, block;
  int persistent;
};

// spt: samples per lane of the kernel launched (a one-pass grid covers
// n / spt lanes)
// A persistent launch of fewer chunks than the grid has wavefronts would run
// them all at once, some SIMDs one more than others; with as many wavefronts per
// SIMD as there are whole chunks for (at least 2), the shortest chunks, which
// are left over, go to the SIMDs that are done first.  FP64, kernel with 4 and
// with 3: 200,000 samples 0.258 and 0.237 ms, with a lead 0.432 and 0.346, RK4
// 1.50 and 1.29; 160,000 with 4 and with 2: 0.209 and 0.198.  Not under the
// controller, whose wavefronts wait on their draws: 200,000 samples 0.485 and
// 0.523; and only the built-in shapes (spread): one that was set or tuned starts
// the wavefronts that it says.
Shape shape(const TuneCfg& t, int64_t n, int spt, bool spread) {
  static int cus = 0;
  if (cus == 0) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
      cus = 256;
  }
  Shape sh;
  sh.block = static_cast<unsigned>(t.block);
  const int64_t per = static_cast<int64_t>(t.block) * spt;
  const int64_t need = (n + per - 1) / per;
  if (t.waves_per_simd > 0) {
    const int64_t simds = static_cast<int64_t>(cus) * 4, chunks = (n + 64 * spt - 1) / (64 * spt);
    int64_t waves = t.waves_per_simd;
    if (spread && waves > 2 && chunks < waves * simds)
      waves = chunks / simds > 2 ? chunks / simds : 2;
    const int64_t grid = simds * waves * 64 / t.block;
    sh.grid = static_cast<unsigned>(need < grid ? need : grid);
    sh.persistent = 1;
  } else {
    sh.grid = static_cast<unsigned>(need);
    sh.persistent = 0;
  }
  return sh;
}

struct Bufs {
  Job* jobs;
  LeadJob* leads;
  uint32_t* keys;
  uint32_t* perm;
  int32_t* nds;
  uint32_t* fix;  // FP32C fix-up list: count, then sample indices
  uint32_t* hist;
  unsigned long long* counter;
  ScnDev* tab;
  aeb_scenario* scns;
};

// scratch: jobs | leads | keys | perm | command steps | fix-up list |
// histogram | counter | scenario tables
size_t bufs_layout(int64_t n, int n_scn, bool lead, char* base, Bufs* b) {
  auto up = [](size_t x) { return (x + 255) & ~size_t(255); };
  const size_t off_jobs = 0;
  const size_t off_leads = up(off_jobs + sizeof(Job) * n);
  const size_t off_keys = up(off_leads + (lead ? sizeof(LeadJob) * n : 0));
  const size_t off_perm = up(off_keys + sizeof(uint32_t) * n);
  const size_t off_nds = up(off_perm + sizeof(uint32_t) * n);
  const size_t off_fix = up(off_nds + sizeof(int32_t) * n);
  const size_t off_hist = up(off_fix + sizeof(uint32_t) * (n + 1));
  const size_t off_cnt = up(off_hist + sizeof(uint32_t) * NBINS_CTL);
  const size_t off_tab = up(off_cnt + sizeof(unsigned long long));
  const size_t off_scn = up(off_tab + sizeof(ScnDev) * n_scn);
  const size_t total = up(off_scn + sizeof(aeb_scenario) * n_scn);
  if (b) {
    b->jobs = reinterpret_cast<Job*>(base + off_jobs);
    b->leads = lead ? reinterpret_cast<LeadJob*>(base + off_leads) : nullptr;
    b->keys = reinterpret_cast<uint32_t*>(base + off_keys);
    b->perm = reinterpret_cast<uint32_t*>(base + off_perm);
    b->nds = reinterpret_cast<int32_t*>(base + off_nds);
    b->fix = reinterpret_cast<uint32_t*>(base + off_fix);
    b->hist = reinterpret_cast<uint32_t*>(base + off_hist);
    b->counter = reinterpret_cast<unsigned long long*>(base + off_cnt);
    b->tab = reinterpret_cast<ScnDev*>(base + off_tab);
    b->scns = reinterpret_cast<aeb_scenario*>(base + off_scn);
  }
  return total;
}

// sort the prepared keys into the permutation (and zero the claim counter)
// (hdr: a recorded mix, n its capacity and the actual count on the device)
// (hist: the key histogram still to be taken; the plain method's prep takes it)
template <int NB = NBINS>
void sort_keys(const Bufs& b, int64_t n, hipStream_t st, const BatchHdr* hdr = nullptr,
               bool hist = true) {
  if (n <= SORT1_MAX) {
    // (the unrolled samples past n cost: 1,000 samples 6.3 us with 32 a thread)
    if (n <= SORT1_T * 8)
      hipLaunchKernelGGL((k_sort1<NB, 8>), dim3(1), dim3(SORT1_T), 0, st, b.keys, n, b.perm,
                         b.counter, hdr);
    else
      hipLaunchKernelGGL((k_sort1<NB, SORT1_PER>), dim3(1), dim3(SORT1_T), 0, st, b.keys, n,
                         b.perm, b.counter, hdr);
    return;
  }
  const unsigned pblk = static_cast<unsigned>((n + PREP_SAMPLES - 1) / PREP_SAMPLES);
  if (hist)
    hipLaunchKernelGGL(k_hist<NB>, dim3(pblk), dim3(PREP_BLOCK), 0, st, b.keys, n, b.hist, hdr);
  hipLaunchKernelGGL(k_scan<NB>, dim3(1), dim3(PREP_BLOCK), 0, st, b.hist, b.counter);
  hipLaunchKernelGGL(k_scatter<NB>, dim3(pblk), dim3(PREP_BLOCK), 0, st, b.keys, n, b.hist,
                     b.perm, hdr);
}

template <int OBS, int K, bool BATCH, int INTEG = AEB_EULER, bool CTL = false>
void go64(const Shape& sh, const Bufs& b, int64_t n, const Ctx& ctx, hipStream_t st) {
  hipLaunchKernelGGL((k_roll_fp64<OBS, K, BATCH, INTEG, CTL>), dim3(sh.grid), dim3(sh.block), 0,
                     st, b.jobs, b.leads, b.perm, n, ctx, b.counter, sh.persistent, nullptr);
}

// the RK4 integration on the launch's actuator table
template <int OBS>
void go64_act(const Shape& sh, const Bufs& b, int64_t n, const Ctx& ctx, const double* act,
              hipStream_t st) {
  hipLaunchKernelGGL((k_roll_fp64<OBS, 16, false, AEB_RK4, false, true>), dim3(sh.grid),
                     dim3(sh.block), 0, st, b.jobs, b.leads, b.perm, n, ctx, b.counter,
                     sh.persistent, act);
}

// The middle of a distribution, and its share above x (truncation left out).
double middle(const aeb_dist& d) {
  if (d.kind == AEB_DIST_UNIFORM) return 0.5 * (d.p0 + d.p1);
  if (d.kind == AEB_DIST_TRUNC_NORMAL) return std::fmin(std::fmax(d.p0, d.lo), d.hi);
  return d.p0;
}
double share_above(const aeb_dist& d, double x) {
  if (d.kind == AEB_DIST_CONST || !(d.p1 > (d.kind == AEB_DIST_UNIFORM ? d.p0 : 0.0)))
    return d.p0 > x ? 1.0 : 0.0;
  if (d.kind == AEB_DIST_UNIFORM) return std::fmin(std::fmax((d.p1 - x) / (d.p1 - d.p0), 0.0), 1.0);
  return 0.5 * std::erfc((x - d.p0) / (d.p1 * std::sqrt(2.0)));
}

// Whether the actuator table gains more than its fill takes, for a scenario with
// a CONST time constant.  The fill is a serial chain, 65 ns a step, of which the
// first 75 us run beside the prep, to the last braking step or until the actuator
// stands still, which at a step of z time constants takes ln(2^53 z) / z steps.
// The table saves a wavefront's actuator for as long as it is live: to the
// stop, or about four time constants where friction limits the brake.  A SIMD with
// w wavefronts saves 25 w + 16 ns a step.  The stop is reckoned at the middles of
// the distributions.  Rollout calls of the paper's preset, plain form and table, ms:
// 131,072 samples, tau 0.15 s 1.36 and 1.27, tau 0.5 s 1.45 and 1.73, tau 1 s and a
// horizon of 30 s 1.54 and 2.96; 350,000, tau 0.5 s 3.04 and 2.78, 30 s 3.05 and
// 3.09, tau 2.5 s, 60 s 4.16 and 6.77; 1,048,576, tau 0.15 s 7.61 and 5.70, tau 1 s,
// 30 s 9.16 and 8.72, tau 2.5 s, 60 s 11.4 and 12.1.  Friction about N(0.7, 0.1), which
// limits half the samples: 100,000 1.16 and 1.27, 200,000 1.78 and 1.66.
bool act_pays(const aeb_scenario& s, int64_t n) {
  auto drawn = [&](const aeb_dist& d, int slot) -> const aeb_dist& {
    return (s.is_mask >> slot) & 1 ? s.proposal[slot] : d;
  };
  const aeb_dist& mu = drawn(s.mu, AEB_SLOT_MU);
  const double tau = s.tau.p0, z = s.dt / tau;
  const double nmax = static_cast<double>(horizon_steps(s));
  const double nd = static_cast<double>(dead_steps(s));
  const double fill = std::fmin(nmax - nd, std::fmax(36.74 + std::log(z), 1.0) / z);
  const double v = middle(drawn(s.v0, AEB_SLOT_V0));
  const double grade = middle(drawn(s.grade, AEB_SLOT_GRADE));
  const Consts k = derive(s, middle(mu), middle(drawn(s.mass, AEB_SLOT_MASS)), std::sin(grade),
                          std::cos(grade), middle(drawn(s.cda, AEB_SLOT_CDA)),
                          middle(drawn(s.crr, AEB_SLOT_CRR)));
  const double slow = -std::fmax(s.a_cmd, k.alim) + k.c + k.kd * v * v / 3.0;
  const double stop = slow > 0.0 ? v / slow + tau : s.horizon;
  // the friction coefficient at which the limit is the command
  const double amag = -s.a_cmd, reach = s.g - amag * s.h_cog / s.wheelbase;
  const double free = amag <= 0.0 ? 1.0 : reach > 0.0 ? share_above(mu, amag / reach) : 0.0;
  const double live = free * stop + (1.0 - free) * std::fmin(stop, 4.0 * tau);
  const double steps = std::fmin(nmax - nd, live / s.dt);
  const double w = std::fmax(2.0, static_cast<double>(n) / 65536.0);
  return 65.0 * fill - 75000.0 < (25.0 * w + 16.0) * steps;
}

// Bytes of the actuator table (ActTab) of a launch of n samples, 0 where it is
// not used.  One actuator for all samples: RK4 with a CONST time constant (host
// columns may hold any), no perception, no controller.  From ACT_MIN samples:
// below, a SIMD has a wavefront or two, whose speed is a serial chain that the
// actuator's operations only accompany (preset of the paper, rollout with and
// without it: 65,536 samples 1.25 and 1.02 ms, 100,000 1.29 and 1.36, 350,000
// 2.30 and 2.78, 1,048,576 5.8 and 7.7), and where it pays (act_pays).  The table
// takes the space of the command steps and the fix-up list, which such a launch
// leaves unused (8 bytes a sample); a horizon that needs more keeps the plain form.
constexpr int64_t ACT_MIN = 98304;
size_t act_bytes(const aeb_scenario& s, int64_t n) {
  if (s.integrator != AEB_RK4 || s.tau.kind != AEB_DIST_CONST || perception_on(s) ||
      control_on(s) || n < ACT_MIN || !act_pays(s, n))
    return 0;
  const size_t steps = static_cast<size_t>(horizon_steps(s));
  const size_t room = 8 * static_cast<size_t>(n);
  if (steps >= room) return 0;
  const size_t b = sizeof(double) * (ACT_HDR + 4 * (steps + ACT_PAD));
  return b <= room ? b : 0;
}

template <int OBS, int K, bool BATCH>
void go64x2(const Shape& sh, const Bufs& b, int64_t n, const Ctx& ctx, hipStream_t st) {
  hipLaunchKernelGGL((k_roll_fp64x2<OBS, K, BATCH>), dim3(sh.grid), dim3(sh.block), 0, st, b.jobs,
                     b.perm, n, ctx, b.counter, sh.persistent);
}

template <int OBS, bool BATCH>
void go64x2k(int k, const Shape& sh, const Bufs& b, int64_t n, const Ctx& ctx, hipStream_t st) {
  if (k == 16)
    go64x2<OBS, 16, BATCH>(sh, b, n, ctx, st);
  else if (k == 64)
    go64x2<OBS, 64, BATCH>(sh, b, n, ctx, st);
  else if (k == 128)
    go64x2<OBS, 128, BATCH>(sh, b, n, ctx, st);
  else
    go64x2<OBS, 32, BATCH>(sh, b, n, ctx, st);
}

template <int OBS, bool BATCH>
void go64k(int k, const Shape& sh, const Bufs& b, int64_t n, const Ctx& ctx, hipStream_t st) {
  if (k == 16)
    go64<OBS, 16, BATCH>(sh, b, n, ctx, st);
  else if (k == 64)
    go64<OBS, 64, BATCH>(sh, b, n, ctx, st);
  else if (k == 128)
    go64<OBS, 128, BATCH>(sh, b, n, ctx, st);
  else
    go64<OBS, 32, BATCH>(sh, b, n, ctx, st);
}

template <int OBS, bool BATCH>
void go32k(int k, const Shape& sh, const Bufs& b, int64_t n, const Ctx& ctx, double band_abs,
           double band_rel, uint32_t* fix, hipStream_t st) {
  if (k == 16)
    hipLaunchKernelGGL((k_roll_fp32c<OBS, 16, BATCH>), dim3(sh.grid), dim3(sh.block), 0, st,
                       b.jobs, b.perm, n, ctx, band_abs, band_rel, fix, b.counter, sh.persistent);
  else if (k == 64)
    hipLaunchKernelGGL((k_roll_fp32c<OBS, 64, BATCH>), dim3(sh.grid), dim3(sh.block), 0, st,
                       b.jobs, b.perm, n, ctx, band_abs, band_rel, fix, b.counter, sh.persistent);
  else
    hipLaunchKernelGGL((k_roll_fp32c<OBS, 32, BATCH>), dim3(sh.grid), dim3(sh.block), 0, st,
                       b.jobs, b.perm, n, ctx, band_abs, band_rel, fix, b.counter, sh.persistent);
}

// With timing enabled, the lane accounting of the launch that follows
// (zeroed first, by a kernel so that the sequence stays recordable).
inline void arm_lanes(Ctx& ctx, hipStream_t st) {
  ctx.lanes = timing_lanes();
  if (ctx.lanes)
    hipLaunchKernelGGL(k_zero, dim3(1), dim3(64), 0, st, reinterpret_cast<uint32_t*>(ctx.lanes),
                       int64_t(2));
}

template <bool BATCH>
int integrate(const aeb_scenario& s0, int precision, const Bufs& b, int64_t n, const Ctx& ctx_in,
              const ParamSrc* src, hipStream_t st, const double* act = nullptr) {
  const int obs = s0.obstacle;
  Ctx ctx = ctx_in;
  const int form = precision == AEB_FP64 ? AEB_FP64 : AEB_FP32C;
  const TuneCfg t = tune_get(form, obs);
  const bool builtin = tune_is_builtin(form, obs, t);
  const Shape sh = shape(t, n, 1, builtin && (BATCH || !control_on(s0)));
  if (!BATCH && control_on(s0)) {
    // the controller decides every ctl_period and blocks stay within a
    // decision period: the top level is a block size that divides the period
    // where one is built (50 steps: 20 and 10 Hz at 1 ms; 40: 25 Hz), else 48
    // (a 50-step period would take a 48-step and a 2-step block); FP64 only
    const int64_t per = ctl_args(s0).period;
    arm_lanes(ctx, st);
    timing_begin(st);
    if (s0.integrator == AEB_RK4)
      go64<AEB_OBS_STATIONARY, 16, false, AEB_RK4, true>(sh, b, n, ctx, st);
    else if (s0.nofma && obs == AEB_OBS_LEAD)  // the unfused form
      per % 50 == 0   ? go64<AEB_OBS_LEAD, 50, false, EULER_NOFMA, true>(sh, b, n, ctx, st)
      : per % 40 == 0 ? go64<AEB_OBS_LEAD, 40, false, EULER_NOFMA, true>(sh, b, n, ctx, st)
                      : go64<AEB_OBS_LEAD, 48, false, EULER_NOFMA, true>(sh, b, n, ctx, st);
    else if (s0.nofma)
      per % 50 == 0   ? go64<AEB_OBS_STATIONARY, 50, false, EULER_NOFMA, true>(sh, b, n, ctx, st)
      : per % 40 == 0 ? go64<AEB_OBS_STATIONARY, 40, false, EULER_NOFMA, true>(sh, b, n, ctx, st)
                      : go64<AEB_OBS_STATIONARY, 48, false, EULER_NOFMA, true>(sh, b, n, ctx, st);
    else if (obs == AEB_OBS_LEAD)
      per % 50 == 0   ? go64<AEB_OBS_LEAD, 50, false, AEB_EULER, true>(sh, b, n, ctx, st)
      : per % 40 == 0 ? go64<AEB_OBS_LEAD, 40, false, AEB_EULER, true>(sh, b, n, ctx, st)
                      : go64<AEB_OBS_LEAD, 48, false, AEB_EULER, true>(sh, b, n, ctx, st);
    else
      per % 50 == 0   ? go64<AEB_OBS_STATIONARY, 50, false, AEB_EULER, true>(sh, b, n, ctx, st)
      : per % 40 == 0 ? go64<AEB_OBS_STATIONARY, 40, false, AEB_EULER, true>(sh, b, n, ctx, st)
                      : go64<AEB_OBS_STATIONARY, 48, false, AEB_EULER, true>(sh, b, n, ctx, st);
    timing_end(st);
    AEB_HIP(hipGetLastError());
    return AEB_OK;
  }
  if (precision == AEB_FP64 && s0.integrator == AEB_RK4) {
    // an RK4 step costs about eight Euler steps: short blocks keep the tail small
    arm_lanes(ctx, st);
    timing_begin(st);
    if (!BATCH && act)
      obs == AEB_OBS_STATIONARY ? go64_act<AEB_OBS_STATIONARY>(sh, b, n, ctx, act, st)
                                : go64_act<AEB_OBS_NONE>(sh, b, n, ctx, act, st);
    else if (obs == AEB_OBS_STATIONARY)
      go64<AEB_OBS_STATIONARY, 16, BATCH, AEB_RK4>(sh, b, n, ctx, st);
    else
      go64<AEB_OBS_NONE, 16, BATCH, AEB_RK4>(sh, b, n, ctx, st);
    timing_end(st);
    AEB_HIP(hipGetLastError());
    return AEB_OK;
  }
  if (precision == AEB_FP64 && s0.nofma) {
    // the unfused form: 128-step blocks, the launch shape of the table
    arm_lanes(ctx, st);
    timing_begin(st);
    if (obs == AEB_OBS_STATIONARY)
      go64<AEB_OBS_STATIONARY, 128, BATCH, EULER_NOFMA>(sh, b, n, ctx, st);
    else if (obs == AEB_OBS_LEAD)
      go64<AEB_OBS_LEAD, 128, BATCH, EULER_NOFMA>(sh, b, n, ctx, st);
    else
      go64<AEB_OBS_NONE, 128, BATCH, EULER_NOFMA>(sh, b, n, ctx, st);
    timing_end(st);
    AEB_HIP(hipGetLastError());
    return AEB_OK;
  }
  if (precision == AEB_FP64 && t.spt == 2 && obs != AEB_OBS_LEAD) {
    // two samples per lane (the tuned FP64 shape)
    const Shape sh2 = shape(t, n, 2, builtin);
    arm_lanes(ctx, st);
    timing_begin(st);
    if (obs == AEB_OBS_STATIONARY)
      go64x2k<AEB_OBS_STATIONARY, BATCH>(t.k, sh2, b, n, ctx, st);
    else
      go64x2k<AEB_OBS_NONE, BATCH>(t.k, sh2, b, n, ctx, st);
    timing_end(st);
    AEB_HIP(hipGetLastError());
    return AEB_OK;
  }
  if (precision == AEB_FP64) {
    arm_lanes(ctx, st);
    timing_begin(st);
    if (obs == AEB_OBS_STATIONARY)
      go64k<AEB_OBS_STATIONARY, BATCH>(t.k, sh, b, n, ctx, st);
    else if (obs == AEB_OBS_LEAD)
      go64k<AEB_OBS_LEAD, BATCH>(t.k, sh, b, n, ctx, st);
    else
      go64k<AEB_OBS_NONE, BATCH>(t.k, sh, b, n, ctx, st);
    timing_end(st);
    AEB_HIP(hipGetLastError());
    return AEB_OK;
  }
  uint32_t* fix = nullptr;
  if (precision == AEB_FP32C_FIXUP) {
    if (BATCH) return fail(AEB_EINVAL, "the FP64 fix-up mode is not available for batches");
    fix = b.fix;
    hipLaunchKernelGGL(k_zero, dim3(1), dim3(64), 0, st, fix, int64_t(1));
  }
  // The form's stated distance tolerance is 1e-4 relative; at the obstacle the
  // distance is the gap, so outcomes within 1 mm + 1e-4 of the gap of the
  // boundary are flagged (and, in the fix-up mode, recomputed in FP64): as
  // long as the distance error stays below that band, every flag outside it
  // equals the FP64 one.
  const double band_abs = 1e-3, band_rel = 1e-4;
  arm_lanes(ctx, st);
  timing_begin(st);
  if (obs == AEB_OBS_LEAD) {
    if (t.k == 16)
      hipLaunchKernelGGL((k_roll_fp32c_lead<16, BATCH>), dim3(sh.grid), dim3(sh.block), 0, st,
                         b.jobs, b.leads, b.perm, n, ctx, band_abs, band_rel, fix, b.counter,
                         sh.persistent);
    else if (t.k == 64)
      hipLaunchKernelGGL((k_roll_fp32c_lead<64, BATCH>), dim3(sh.grid), dim3(sh.block), 0, st,
                         b.jobs, b.leads, b.perm, n, ctx, band_abs, band_rel, fix, b.counter,
                         sh.persistent);
    else
      hipLaunchKernelGGL((k_roll_fp32c_lead<32, BATCH>), dim3(sh.grid), dim3(sh.block), 0, st,
                         b.jobs, b.leads, b.perm, n, ctx, band_abs, band_rel, fix, b.counter,
                         sh.persistent);
  } else if (obs == AEB_OBS_STATIONARY)
    go32k<AEB_OBS_STATIONARY, BATCH>(t.k, sh, b, n, ctx, band_abs, band_rel, fix, st);
  else
    go32k<AEB_OBS_NONE, BATCH>(t.k, sh, b, n, ctx, band_abs, band_rel, fix, st);
  timing_end(st);
  AEB_HIP(hipGetLastError());
  if (fix) return launch_fixup(s0, src, ctx.out, fix, st);
  return AEB_OK;
}

}  // namespace

size_t rollout_scratch_bytes(const aeb_scenario& s, int64_t n) {
  return bufs_layout(n, 0, s.obstacle == AEB_OBS_LEAD, nullptr, nullptr);
}

int launch_rollout_fast_into(const aeb_scenario& s, const ParamSrc* src, int precision,
                             const OutCols& out, int64_t n, void* scratch_base, hipStream_t st) {
  const int64_t nd = dead_steps(s), nmax = horizon_steps(s);
  if (!block_steps_ok(s))
    return fail(AEB_EINVAL, "horizon plus dead time beyond 2^31 - 4096 steps on the block path");
  const bool lead = s.obstacle == AEB_OBS_LEAD;
  Bufs b;
  bufs_layout(n, 0, lead, static_cast<char*>(scratch_base), &b);
  double* act = !src && act_bytes(s, n) > 0 ? reinterpret_cast<double*>(b.nds) : nullptr;
  const unsigned pblk = prep_grid(n) + (act ? 1 : 0);
  const bool ctl = control_on(s);
  const int nb = ctl ? NBINS_CTL : NBINS;
  // a small launch's sort takes its own histogram
  const bool small = n <= SORT1_MAX;
  if (!small) hipLaunchKernelGGL(k_zero, dim3(nb / 256), dim3(256), 0, st, b.hist, int64_t(nb));
  PrepArgs pa{};
  pa.s = s;
  pa.src = src ? *src : ParamSrc{};
  pa.n = n;
  pa.nd = static_cast<int>(nd);
  pa.nmax = static_cast<int>(nmax);
  pa.cap = static_cast<float>(nmax);
  pa.nds = perception_on(s) ? b.nds : nullptr;
  pa.ctl = ctl ? 1 : 0;
  pa.weight = out.weight;
  pa.act = act;
  const unsigned cblk = static_cast<unsigned>((n + PREP_SAMPLES - 1) / PREP_SAMPLES);
  if (src && small)
    hipLaunchKernelGGL((k_prep<false, false>), dim3(pblk), dim3(PREP_BLOCK), 0, st, pa, b.jobs,
                       b.leads, b.keys);
  else if (src && ctl)
    hipLaunchKernelGGL(k_prep_cols<NBINS_CTL>, dim3(cblk), dim3(PREP_BLOCK), 0, st, pa, b.jobs,
                       b.leads, b.keys, b.hist);
  else if (src)
    hipLaunchKernelGGL(k_prep_cols<NBINS>, dim3(cblk), dim3(PREP_BLOCK), 0, st, pa, b.jobs,
                       b.leads, b.keys, b.hist);
  else
    hipLaunchKernelGGL((k_prep<true, false>), dim3(pblk), dim3(PREP_BLOCK), 0, st, pa, b.jobs,
                       b.leads, b.keys);
  if (ctl)
    sort_keys<NBINS_CTL>(b, n, st, nullptr, !src);
  else
    sort_keys(b, n, st, nullptr, !src);
  Ctx ctx{};
  ctx.dt = s.dt;
  ctx.a_cmd = s.a_cmd;
  ctx.nd = static_cast<int>(nd);
  ctx.nmax = static_cast<int>(nmax);
  ctx.impact_exit = s.impact_exit;
  ctx.out = out;
  ctx.tab = nullptr;
  ctx.nds = pa.nds;
  ctx.ca = ctl_args(s);
  return integrate<false>(s, precision, b, n, ctx, src, st, act);
}

int launch_rollout_fast(const aeb_scenario& s, const ParamSrc* src, int precision,
                        const OutCols& out, int64_t n, hipStream_t st) {
  void* base = pool_block(rollout_scratch_bytes(s, n), st);
  if (!base) return AEB_ENOMEM;
  return launch_rollout_fast_into(s, src, precision, out, n, base, st);
}

size_t batch_scratch_bytes(int64_t total, int n_scn, bool lead) {
  return bufs_layout(total, n_scn, lead, nullptr, nullptr);
}

int fill_batch_table(const aeb_scenario* scns, int n_scn, const OutCols* outs, ScnDev* tab,
                     int64_t* total_out, int64_t* cap_out) {
  int64_t total = 0, cap = 1, padded = 0;
  for (int j = 0; j < n_scn; ++j) {
    const int64_t nd = dead_steps(scns[j]), nmax = horizon_steps(scns[j]);
    if (!block_steps_ok(scns[j]))
      return fail(AEB_EINVAL, "horizon plus dead time beyond 2^31 - 4096 steps on the block path");
    tab[j].dt = scns[j].dt;
    tab[j].a_cmd = scns[j].a_cmd;
    tab[j].nd = static_cast<int>(nd);
    tab[j].nmax = static_cast<int>(nmax);
    tab[j].off = total;
    tab[j].poff = padded;
    tab[j].out = outs[j];
    total += scns[j].n_samples;
    padded += (scns[j].n_samples + 63) & ~int64_t(63);
    if (nmax > cap) cap = nmax;
  }
  if (total > 0xffffffffLL) return fail(AEB_EINVAL, "a batch holds at most 2^32 - 1 samples");
  *total_out = total;
  *cap_out = cap;
  return AEB_OK;
}

int launch_batch_fast_into(const aeb_scenario* scns, int n_scn, int precision,
                           const ScnDev* tab, int64_t total, int64_t cap, void* scratch_base,
                           hipStream_t st) {
  const bool lead = scns[0].obstacle == AEB_OBS_LEAD;
  Bufs b;
  bufs_layout(total, n_scn, lead, static_cast<char*>(scratch_base), &b);
  AEB_HIP(hipMemcpyAsync(b.tab, tab, sizeof(ScnDev) * n_scn, hipMemcpyHostToDevice, st));
  AEB_HIP(hipMemcpyAsync(b.scns, scns, sizeof(aeb_scenario) * n_scn, hipMemcpyHostToDevice, st));
  // the prep's index space: each scenario padded to a multiple of 64 samples
  const int64_t padded = tab[n_scn - 1].poff + ((scns[n_scn - 1].n_samples + 63) & ~int64_t(63));
  const unsigned pblk = prep_grid(padded);
  if (total > SORT1_MAX)
    hipLaunchKernelGGL(k_zero, dim3(NBINS / 256), dim3(256), 0, st, b.hist, int64_t(NBINS));
  PrepArgs pa{};
  pa.n = total;
  pa.cap = static_cast<float>(cap);
  pa.scns = b.scns;
  pa.tab = b.tab;
  pa.n_scn = n_scn;
  bool perc = false;
  for (int j = 0; j < n_scn; ++j) perc = perc || perception_on(scns[j]);
  pa.nds = perc ? b.nds : nullptr;
  hipLaunchKernelGGL((k_prep<true, true>), dim3(pblk), dim3(PREP_BLOCK), 0, st, pa, b.jobs,
                     b.leads, b.keys);
  sort_keys(b, total, st);
  Ctx ctx{};
  ctx.impact_exit = scns[0].impact_exit;
  ctx.tab = b.tab;
  ctx.nds = pa.nds;
  return integrate<true>(scns[0], precision, b, total, ctx, nullptr, st);
}

int launch_batch_fast_dev(const aeb_scenario& kind, bool perception, int precision,
                          const BatchHdr* hdr, const ScnDev* tab, const aeb_scenario* scns,
                          int cap_scn, int64_t cap_total, void* scratch_base, hipStream_t st) {
  const bool lead = kind.obstacle == AEB_OBS_LEAD;
  Bufs b;
  bufs_layout(cap_total, 0, lead, static_cast<char*>(scratch_base), &b);
  // the prep's index space for any mix within the capacity (each scenario
  // padded to a multiple of 64 samples)
  const unsigned pblk = prep_grid(cap_total + 63 * static_cast<int64_t>(cap_scn));
  if (cap_total > SORT1_MAX)
    hipLaunchKernelGGL(k_zero, dim3(NBINS / 256), dim3(256), 0, st, b.hist, int64_t(NBINS));
  PrepArgs pa{};
  pa.n = cap_total;
  pa.cap = 1.0f;
  pa.scns = scns;
  pa.tab = tab;
  pa.n_scn = cap_scn;
  pa.nds = perception ? b.nds : nullptr;
  pa.hdr = hdr;
  hipLaunchKernelGGL((k_prep<true, true>), dim3(pblk), dim3(PREP_BLOCK), 0, st, pa, b.jobs,
                     b.leads, b.keys);
  sort_keys(b, cap_total, st, hdr);
  Ctx ctx{};
  ctx.impact_exit = kind.impact_exit;
  ctx.tab = tab;
  ctx.nds = pa.nds;
  ctx.hdr = hdr;
  return integrate<true>(kind, precision, b, cap_total, ctx, nullptr, st);
}

int launch_batch_fast(const aeb_scenario* scns, int n_scn, int precision, const OutCols* outs,
                      hipStream_t st) {
  std::vector<ScnDev> tab(n_scn);
  int64_t total = 0, cap = 1;
  int rc = fill_batch_table(scns, n_scn, outs, tab.data(), &total, &cap);
  if (rc != AEB_OK) return rc;
  const bool lead = scns[0].obstacle == AEB_OBS_LEAD;
  void* base = pool_block(batch_scratch_bytes(total, n_scn, lead), st);
  if (!base) return AEB_ENOMEM;
  rc = launch_batch_fast_into(scns, n_scn, precision, tab.data(), total, cap, base, st);
  if (rc != AEB_OK) return rc;
  // the tables are copied from pageable host memory: keep them valid until
  // the copies have run
  AEB_HIP(hipStreamSynchronize(st));
  return AEB_OK;
}

}  // namespace aeb

// kernels_reduce.hip -- statistics of one batch of rollout outputs (Sec. VI):
// counts and P(collision | H0) (eq. (20)), moments of the stopping distance
// (Table I), the collision-risk curve and exact minimum safe headways
// (Sec. VI-C), and margin statistics.
//
// Sums run in a fixed order (each block a fixed slice, a fixed tree inside the
// block, blocks summed in index order), so repeated calls give identical
// bits.  Order statistics are exact: a histogram over 4,096 value bins
// spanning each array's finite range (plus one bin for the censored +inf
// values) finds the bin holding a target's rank; the bin's elements are
// collected and the rank selected among them in LDS (a radix select over an
// order-preserving map of the FP64 bit patterns).  A bin with more than 8,192
// elements falls back to a radix select over the whole array (8 passes of 8
// bits; the sets of a batch that need it go through the passes together).
#include <hip/hip_runtime.h>

#include <cmath>
#include <atomic>
#include <cstring>
#include <vector>

#include "aeb_runtime.h"

namespace aeb {

namespace {

constexpr int RB = 256;          // threads per reduction block
constexpr int EB = 1024;         // threads per block of the element passes
constexpr int CP = 4;            // elements per thread loaded together
constexpr int MAX_T = AEB_MAX_RISK + AEB_MAX_MARGIN_Q;
constexpr int NVB = 4096;        // value bins of the selection histograms (+1 overflow)
constexpr int CAP = 8192;        // candidates a target's bin may hold for the LDS sort
constexpr int FB = 1024;         // threads of the finalize / bin-search blocks
// block histogram row: distance value bins | margin value bins | risk-grid ranks
constexpr int HG = 2 * (NVB + 1);             // offset of the risk-grid part
constexpr int HW = HG + AEB_MAX_GRID + 1;     // row width
// importance-sampling accumulators: four words per risk-grid rank bin, plus
// bins for the collided samples and for all samples
constexpr int WACC = (AEB_MAX_GRID + 3) * 4;

struct Partial {
  long long ncol, nstop, nimp, nhor, nbnd;
  double sum, dmin, dmax, msum, mmin, mmax;
  float vmax;
  float pad;
  double wmax;     // largest importance-sampling weight
  long long wbad;  // weights that are not finite and >= 0
};

// Selection progress: the value bin holding each target's rank and the rank
// inside the bin, the candidates collected, the binning of each array.
struct Sel {
  int fallback, pad;
  int bin[MAX_T];          // -1: answered without candidates
  unsigned rank_in_bin[MAX_T];
  unsigned bin_count[MAX_T];
  double vmin[2], scale[2];
  int wshift[2];  // fixed-point exponents of w and w^2 (importance-sampling sums)
};

// Radix-select state of the fallback path.
struct SelState {
  unsigned long long prefix[MAX_T];
  unsigned long long rank[MAX_T];
};

__host__ __device__ inline size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

// Scratch layout of one reduction: stats, selection state and the bin totals
// (selection bins and risk-grid ranks) first (zeroed by one launch), then the
// block partials, the block histograms, the candidates and the radix-select
// state.
struct RLayout {
  long long chunk, chunk2;
  int nb, nb2, T;
  unsigned ccap;  // candidates kept per target: min(n, CAP) (a bin holds at most n)
  size_t off_sel, off_zero_end, off_var, off_bh, off_bt, off_wa, off_bo, off_cand, off_ss, off_sh,
      total;
};

__host__ __device__ inline RLayout layout(long long n, int T) {
  RLayout L;
  // element passes: 4,096 elements per block of 1,024 threads (measured faster
  // than smaller blocks or slices: fewer partials, block histograms and
  // per-block fixed costs)
  L.chunk = EB * CP;
  L.chunk2 = EB * CP;
  L.nb = static_cast<int>((n + L.chunk - 1) / L.chunk);
  L.nb2 = static_cast<int>((n + L.chunk2 - 1) / L.chunk2);
  L.T = T;
  const int tc = L.T > 0 ? L.T : 1;
  L.off_sel = align256(sizeof(aeb_stats));
  L.off_bt = align256(L.off_sel + sizeof(Sel));
  L.off_wa = align256(L.off_bt + sizeof(unsigned) * HW);
  L.off_zero_end = align256(L.off_wa + sizeof(unsigned long long) * WACC);
  L.off_var = align256(L.off_zero_end + sizeof(Partial) * L.nb);
  L.off_bh = align256(L.off_var + sizeof(double) * (L.nb > L.nb2 ? L.nb : L.nb2));
  L.off_bo = align256(L.off_bh + sizeof(unsigned) * HW * L.nb2);
  L.off_cand = align256(L.off_bo + sizeof(unsigned) * tc * L.nb2);
  L.ccap = static_cast<unsigned>(n < CAP ? (n > 0 ? n : 1) : CAP);
  L.off_ss = align256(L.off_cand + sizeof(unsigned long long) * tc * L.ccap);
  L.off_sh = align256(L.off_ss + sizeof(SelState));
  L.total = align256(L.off_sh + sizeof(unsigned) * tc * 256);
  return L;
}

// One output set of a segmented reduction: its columns, its scratch (the
// layout below), where its statistics go, and its place among the launch's
// element-pass blocks and bin-totals rows.
struct RSeg {
  OutCols out;
  long long n;
  char* base;      // the set's scratch (RLayout of n)
  aeb_stats* st;   // its statistics (device)
  int nb;          // element-pass blocks of the set
  int blk0;        // its first block among the launch's element-pass blocks
  int row0;        // its first row of the bin-totals grid
  int pad;
};

// The sets of one launch sequence: a single set by value, or a device table
// with the set of every element-pass block and every bin-totals row.
// Grids cover a capacity of sets, blocks and rows; the table says how many
// sets this launch has (a recorded graph replays with other counts) and maps
// the blocks and rows beyond them to -1, and those blocks return at once.
struct RSegs {
  RSeg one;
  const RSeg* tab;    // null: the single set `one`
  const int* bmap;    // set of each element-pass block (-1: none)
  const int* rmap;    // set of each bin-totals row (-1: none)
  const int* count;   // sets of the launch (device)
};

__device__ inline int seg_count(const RSegs& S) { return S.tab ? *S.count : 1; }

// The set by value: a pointer or reference that may point at the kernel
// argument `one` makes the compiler copy the argument to per-lane scratch.
__device__ inline RSeg seg_at(const RSegs& S, int j) { return S.tab ? S.tab[j] : S.one; }

// The set of element-pass block `gb` and the block's index inside it; false
// for a block beyond the launch's sets.
__device__ inline bool seg_of_block(const RSegs& S, int gb, int& local, RSeg& g) {
  if (!S.tab) {
    local = gb;
    g = S.one;
    return gb < S.one.nb;
  }
  const int j = S.bmap[gb];
  if (j < 0) return false;
  g = S.tab[j];
  local = gb - g.blk0;
  return true;
}

// What a reduction computes: risk levels and margin quantile levels, and the
// risk-curve grid (the request of the C ABI, by value).
struct RReq {
  int n_risk, n_mq, ng, pad;
  double risk[AEB_MAX_RISK];
  double mq[AEB_MAX_MARGIN_Q];
  double glo, gstep, ginv;
};

// Selection targets of a set of n samples: target t < n_risk is H(risk[t]),
// the element of 0-based rank n - floor(r n) - 1 of the censored distances;
// target n_risk + j the margin quantile at mq[j], the element of rank
// floor(p n) (floors of binary64 products, as the host computes them).
__device__ inline int sel_kind(const RReq& q, int t) { return t >= q.n_risk ? 1 : 0; }

__device__ inline unsigned long long sel_rank(const RReq& q, long long n, int t) {
  const double nd = static_cast<double>(n);
  if (t < q.n_risk) {
    const long long m = static_cast<long long>(floor(q.risk[t] * nd));
    return static_cast<unsigned long long>(n - m - 1);
  }
  return static_cast<unsigned long long>(static_cast<long long>(floor(q.mq[t - q.n_risk] * nd)));
}

// order-preserving map of binary64 onto uint64
__device__ inline unsigned long long ordered(double d) {
  unsigned long long u = static_cast<unsigned long long>(__double_as_longlong(d));
  return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

__device__ inline double unordered(unsigned long long u) {
  u = (u >> 63) ? (u & 0x7fffffffffffffffull) : ~u;
  return __longlong_as_double(static_cast<long long>(u));
}

__device__ inline double censored(const double* dist, const uint8_t* status, long long i) {
  return (status[i] & 3) == AEB_END_STOP ? dist[i] : INFINITY;
}

// value bin: monotone in v; +inf goes to the overflow bin NVB
__device__ inline int value_bin(double v, double vmin, double scale) {
  if (!(v < INFINITY)) return NVB;
  double f = (v - vmin) * scale;
  int b = f > 0.0 ? static_cast<int>(f) : 0;
  return b < NVB ? b : NVB - 1;
}

// number of grid headways strictly below d, H0_j = lo + j * step (j < ng):
// an arithmetic guess corrected with exact comparisons against the same
// expression, so the count is exact
__device__ inline int grid_rank(double d, double lo, double step, double inv_step, int ng) {
  if (!(d > lo)) return 0;
  if (!(d < INFINITY)) return ng;
  double g = (d - lo) * inv_step;
  int j = g < static_cast<double>(ng) ? static_cast<int>(g) : ng;
  // count = first j with H0_j >= d
  while (j > 0 && !(lo + static_cast<double>(j - 1) * step < d)) --j;
  while (j < ng && lo + static_cast<double>(j) * step < d) ++j;
  return j;
}

template <int NT, typename T, typename Op>
__device__ inline T block_reduce(T v, T* sh, Op op) {
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int w = NT / 2; w > 0; w >>= 1) {
    if (static_cast<int>(threadIdx.x) < w) sh[threadIdx.x] = op(sh[threadIdx.x], sh[threadIdx.x + w]);
    __syncthreads();
  }
  T r = sh[0];
  __syncthreads();
  return r;
}

// exclusive scan of one value per thread over a block of NT threads: a
// shuffle scan inside each wavefront, then the wavefronts' totals through LDS
// (two barriers; a scan of all NT values in LDS takes 20 and 2 us at 1,024
// threads, and a reduction makes up to a dozen of them one after the other)
template <int NT>
__device__ inline unsigned long long block_exscan(unsigned long long v, unsigned long long* sh) {
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  unsigned long long inc = v;
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned long long t = __shfl_up(inc, o);
    if (l >= o) inc += t;
  }
  if (l == 63) sh[w] = inc;
  __syncthreads();
  unsigned long long base = 0;
  for (int q = 0; q < NT / 64; ++q) base += q < w ? sh[q] : 0ull;
  __syncthreads();
  return base + inc - v;
}

// A 64-bit value moved between lanes by a data-parallel-primitives (DPP)
// modifier; lanes without a source lane under the row and bank masks get `id`.
template <int CTRL, int ROW_MASK, int BANK_MASK>
__device__ inline unsigned long long dpp64(unsigned long long v, unsigned long long id) {
  const unsigned lo = static_cast<unsigned>(__builtin_amdgcn_update_dpp(
      static_cast<int>(static_cast<unsigned>(id)), static_cast<int>(static_cast<unsigned>(v)), CTRL,
      ROW_MASK, BANK_MASK, false));
  const unsigned hi = static_cast<unsigned>(__builtin_amdgcn_update_dpp(
      static_cast<int>(static_cast<unsigned>(id >> 32)), static_cast<int>(static_cast<unsigned>(v >> 32)),
      CTRL, ROW_MASK, BANK_MASK, false));
  return (static_cast<unsigned long long>(hi) << 32) | lo;
}

__device__ inline unsigned long long bits64(double v) {
  return static_cast<unsigned long long>(__double_as_longlong(v));
}
__device__ inline unsigned long long bits64(long long v) { return static_cast<unsigned long long>(v); }
__device__ inline double from_bits(unsigned long long u, double) {
  return __longlong_as_double(static_cast<long long>(u));
}
__device__ inline long long from_bits(unsigned long long u, long long) {
  return static_cast<long long>(u);
}

template <int CTRL, int ROW_MASK, int BANK_MASK, typename T>
__device__ inline T dpp(T v, T id) {
  return from_bits(dpp64<CTRL, ROW_MASK, BANK_MASK>(bits64(v), bits64(id)), v);
}

// Reduction of one value per lane over a wavefront (every lane active): an
// inclusive scan by DPP row shifts of 1, 2, 4, 8 lanes inside each row of 16,
// then row broadcasts of lane 15 and lane 31, leaves the total in lane 63,
// which is read back for every lane.  A fixed association order, so repeated
// calls give the same bits; register moves only, no memory round trips.
template <typename T, typename Op>
__device__ inline T wave_reduce(T v, Op op) {
  const T id = Op::template ident<T>();
  v = op(v, dpp<0x111, 0xf, 0xf>(v, id));  // row_shr:1
  v = op(v, dpp<0x112, 0xf, 0xf>(v, id));  // row_shr:2
  v = op(v, dpp<0x114, 0xf, 0xf>(v, id));  // row_shr:4
  v = op(v, dpp<0x118, 0xf, 0xf>(v, id));  // row_shr:8
  v = op(v, dpp<0x142, 0xa, 0xf>(v, id));  // row_bcast:15 into rows 1 and 3
  v = op(v, dpp<0x143, 0xc, 0xf>(v, id));  // row_bcast:31 into rows 2 and 3
  const unsigned long long u = bits64(v);
  const unsigned lo = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(static_cast<unsigned>(u)), 63));
  const unsigned hi = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(static_cast<unsigned>(u >> 32)), 63));
  return from_bits((static_cast<unsigned long long>(hi) << 32) | lo, v);
}

struct AddOp {
  template <typename T>
  __device__ T operator()(T a, T b) const { return a + b; }
  template <typename T>
  __device__ static T ident() { return T(0); }
};
struct MinOp {
  __device__ double operator()(double a, double b) const { return b < a ? b : a; }
  template <typename T>
  __device__ static T ident() { return INFINITY; }
};
struct MaxOp {
  __device__ double operator()(double a, double b) const { return b > a ? b : a; }
  template <typename T>
  __device__ static T ident() { return -INFINITY; }
};

__device__ inline void combine(Partial& a, const Partial& b) {
  a.ncol += b.ncol;
  a.nstop += b.nstop;
  a.nimp += b.nimp;
  a.nhor += b.nhor;
  a.nbnd += b.nbnd;
  a.sum += b.sum;
  a.dmin = b.dmin < a.dmin ? b.dmin : a.dmin;
  a.dmax = b.dmax > a.dmax ? b.dmax : a.dmax;
  a.msum += b.msum;
  a.mmin = b.mmin < a.mmin ? b.mmin : a.mmin;
  a.mmax = b.mmax > a.mmax ? b.mmax : a.mmax;
  a.vmax = b.vmax > a.vmax ? b.vmax : a.vmax;
  a.wmax = b.wmax > a.wmax ? b.wmax : a.wmax;
  a.wbad += b.wbad;
}

__device__ inline Partial identity_partial() {
  Partial p;
  p.ncol = p.nstop = p.nimp = p.nhor = p.nbnd = 0;
  p.sum = p.msum = 0.0;
  p.dmin = p.mmin = INFINITY;
  p.dmax = p.mmax = -INFINITY;
  p.vmax = 0.0f;
  p.pad = 0.0f;
  p.wmax = 0.0;
  p.wbad = 0;
  return p;
}

// every field reduced over the wavefront by the fixed butterfly
__device__ inline Partial wave_combine(const Partial& a) {
  Partial p;
  p.ncol = wave_reduce(a.ncol, AddOp());
  p.nstop = wave_reduce(a.nstop, AddOp());
  p.nimp = wave_reduce(a.nimp, AddOp());
  p.nhor = wave_reduce(a.nhor, AddOp());
  p.nbnd = wave_reduce(a.nbnd, AddOp());
  p.sum = wave_reduce(a.sum, AddOp());
  p.dmin = wave_reduce(a.dmin, MinOp());
  p.dmax = wave_reduce(a.dmax, MaxOp());
  p.msum = wave_reduce(a.msum, AddOp());
  p.mmin = wave_reduce(a.mmin, MinOp());
  p.mmax = wave_reduce(a.mmax, MaxOp());
  p.vmax = static_cast<float>(wave_reduce(static_cast<double>(a.vmax), MaxOp()));
  p.pad = 0.0f;
  p.wmax = wave_reduce(a.wmax, MaxOp());
  p.wbad = wave_reduce(a.wbad, AddOp());
  return p;
}

// the block's wavefront partials (in LDS) combined by wavefront 0, lane w
// holding wavefront w's partial; every lane of wavefront 0 gets the result
template <int NW>
__device__ inline Partial block_combine(const Partial* wp) {
  const int l = threadIdx.x;
  return wave_combine(l < NW ? wp[l] : identity_partial());
}

// Pass 1 over element-pass block bx of set g (a workgroup of EB threads).
__device__ inline void pass1_blk(const RSeg& g, int bx) {
  const OutCols o = g.out;
  const long long n = g.n;
  const long long chunk = static_cast<long long>(EB) * CP;
  Partial* part = reinterpret_cast<Partial*>(g.base + layout(n, 0).off_zero_end);
  __shared__ Partial wp[EB / 64];
  const long long lo = static_cast<long long>(bx) * chunk;
  const long long hi = lo + chunk < n ? lo + chunk : n;
  long long ncol = 0, nstop = 0, nimp = 0, nhor = 0, nbnd = 0, wbad = 0;
  double sum = 0.0, dmin = INFINITY, dmax = -INFINITY, msum = 0.0, mmin = INFINITY,
         mmax = -INFINITY, wmax = 0.0;
  float vmax = 0.0f;
  if (o.weight) {  // importance-sampling weights: their range and validity
    for (long long i = lo + threadIdx.x; i < hi; i += EB) {
      const double w = o.weight[i];
      if (w >= 0.0 && w < INFINITY)
        wmax = w > wmax ? w : wmax;
      else
        ++wbad;
    }
  }
  // CP elements per thread are loaded before any is used (chunk = CP * EB)
  for (long long i0 = lo; i0 < hi; i0 += static_cast<long long>(EB) * CP) {
    uint8_t sv[CP];
    double dv[CP], mv[CP];
    float vv[CP];
#pragma unroll
    for (int p = 0; p < CP; ++p) {
      const long long i = i0 + p * EB + threadIdx.x;
      sv[p] = 0;
      dv[p] = mv[p] = 0.0;
      vv[p] = 0.0f;
      if (i < hi) {
        sv[p] = o.status[i];
        dv[p] = o.dist[i];
        mv[p] = o.margin[i];
        vv[p] = o.vimp[i];
      }
    }
#pragma unroll
    for (int p = 0; p < CP; ++p) {
    if (i0 + p * EB + threadIdx.x >= hi) break;
    const uint8_t st = sv[p];
    if (st & AEB_BOUNDARY) ++nbnd;
    const double d = dv[p];
    const double m = mv[p];
    const int end = st & 3;
    if (st & AEB_COLLIDED) {
      ++ncol;
      const float vi = vv[p];
      vmax = vi > vmax ? vi : vmax;
    }
    if (end == AEB_END_STOP) {
      ++nstop;
      sum += d;
      dmin = d < dmin ? d : dmin;
      dmax = d > dmax ? d : dmax;
    } else if (end == AEB_END_IMPACT) {
      ++nimp;
    } else if (end == AEB_END_HORIZON) {
      ++nhor;
    }
    msum += m;
    mmin = m < mmin ? m : mmin;
    mmax = m > mmax ? m : mmax;
    }
  }
  // wavefront partials, then the block's waves combined in index order
  Partial p;
  p.ncol = ncol;
  p.nstop = nstop;
  p.nimp = nimp;
  p.nhor = nhor;
  p.nbnd = nbnd;
  p.sum = sum;
  p.dmin = dmin;
  p.dmax = dmax;
  p.msum = msum;
  p.mmin = mmin;
  p.mmax = mmax;
  p.vmax = vmax;
  p.pad = 0.0f;
  p.wmax = wmax;
  p.wbad = wbad;
  p = wave_combine(p);
  if ((threadIdx.x & 63) == 0) wp[threadIdx.x >> 6] = p;
  __syncthreads();
  if (threadIdx.x < 64) {
    const Partial q = block_combine<EB / 64>(wp);
    if (threadIdx.x == 0) part[bx] = q;
  }
}

__global__ __launch_bounds__(EB) void k_pass1(RSegs S) {
  int bx;
  RSeg g;
  if (!seg_of_block(S, blockIdx.x, bx, g)) return;  // beyond the launch's sets (the whole block)
  pass1_blk(g, bx);
}

// Combine the block partials in a fixed order (thread t takes partials
// t, t+FB, ... in order, then a fixed tree).
__device__ inline void fin1_set(const RSeg& g) {
  const int weighted = g.out.weight ? 1 : 0;
  const long long n = g.n;
  const RLayout RL = layout(n, 0);
  const Partial* part = reinterpret_cast<const Partial*>(g.base + RL.off_zero_end);
  const int nb = RL.nb;
  aeb_stats* st = g.st;
  Sel* sel = reinterpret_cast<Sel*>(g.base + RL.off_sel);
  __shared__ Partial wp[FB / 64];
  Partial p = identity_partial();
  for (int b = threadIdx.x; b < nb; b += FB) combine(p, part[b]);
  p = wave_combine(p);
  if ((threadIdx.x & 63) == 0) wp[threadIdx.x >> 6] = p;
  __syncthreads();
  if (threadIdx.x >= 64) return;
  const Partial q = block_combine<FB / 64>(wp);
  const long long ncol = q.ncol, nstop = q.nstop, nimp = q.nimp, nhor = q.nhor, nbnd = q.nbnd;
  const double sum = q.sum, dmin = q.dmin, dmax = q.dmax, msum = q.msum, mmin = q.mmin,
               mmax = q.mmax;
  const double vmax = q.vmax;
  if (threadIdx.x == 0) {
    st->n = n;
    st->n_collide = ncol;
    st->n_stop = nstop;
    st->n_impact = nimp;
    st->n_horizon = nhor;
    st->n_boundary = nbnd;
    st->p_collision = static_cast<double>(ncol) / static_cast<double>(n);
    st->mean_dist = nstop > 0 ? sum / static_cast<double>(nstop) : NAN;
    st->dist_min = nstop > 0 ? dmin : NAN;
    st->dist_max = nstop > 0 ? dmax : NAN;
    st->sd_dist = NAN;
    st->margin_min = mmin;
    st->margin_mean = msum / static_cast<double>(n);
    st->v_impact_max = static_cast<float>(vmax);
    // value bins span the finite range of each selected array
    sel->vmin[0] = nstop > 0 ? dmin : 0.0;
    sel->scale[0] = (nstop > 0 && dmax > dmin) ? static_cast<double>(NVB) / (dmax - dmin) : 0.0;
    sel->vmin[1] = mmin;
    sel->scale[1] = mmax > mmin ? static_cast<double>(NVB) / (mmax - mmin) : 0.0;
    // fixed point of the weighted sums: value * 2^shift as a 128-bit integer,
    // with n * max value * 2^shift < 2^126 (no sum can overflow)
    int ln = 0;
    while ((1ll << ln) < n) ++ln;
    int e1 = 0, e2 = 0;
    frexp(q.wmax, &e1);
    frexp(q.wmax * q.wmax, &e2);
    sel->wshift[0] = q.wmax > 0.0 ? 126 - ln - e1 : 0;
    sel->wshift[1] = q.wmax > 0.0 ? 126 - ln - e2 : 0;
    st->weighted = weighted ? (q.wbad > 0 ? -1 : 1) : 0;
  }
}

__global__ __launch_bounds__(FB) void k_fin1(RSegs S) {
  if (static_cast<int>(blockIdx.x) >= seg_count(S)) return;
  fin1_set(seg_at(S, blockIdx.x));
}

// Sum of squared deviations for the sd, and block-private histograms (LDS,
// written out without atomics): value bins of the arrays that have targets,
// and the number of risk-grid headways below each censored distance.
__device__ inline void pass2_blk(const RSeg& g, int bx, int need_d, int need_m, const RReq& rq,
                                 int hw) {
  const OutCols o = g.out;
  const long long n = g.n;
  const long long chunk = static_cast<long long>(EB) * CP;
  const RLayout RL = layout(n, 0);
  const aeb_stats* st = g.st;
  const Sel* sel = reinterpret_cast<const Sel*>(g.base + RL.off_sel);
  unsigned* bhist = reinterpret_cast<unsigned*>(g.base + RL.off_bh);
  double* part = reinterpret_cast<double*>(g.base + RL.off_var);
  const double glo = rq.glo, gstep = rq.gstep, ginv = rq.ginv;
  const int ng = rq.ng;
  __shared__ double shd[EB / 64];
  __shared__ unsigned h[HW];
  for (int j = threadIdx.x; j < hw; j += EB) h[j] = 0;
  __syncthreads();
  const double mean = st->mean_dist;
  const double vmin0 = sel->vmin[0], sc0 = sel->scale[0];
  const double vmin1 = sel->vmin[1], sc1 = sel->scale[1];
  const long long lo = static_cast<long long>(bx) * chunk;
  const long long hi = lo + chunk < n ? lo + chunk : n;
  double ss = 0.0;
  // CP elements per thread are loaded before any is used (chunk2 = CP * EB)
  for (long long i0 = lo; i0 < hi; i0 += static_cast<long long>(EB) * CP) {
    uint8_t sv[CP];
    double dv[CP], mv[CP];
#pragma unroll
    for (int p = 0; p < CP; ++p) {
      const long long i = i0 + p * EB + threadIdx.x;
      sv[p] = 0;
      dv[p] = mv[p] = 0.0;
      if (i < hi) {
        sv[p] = o.status[i];
        dv[p] = o.dist[i];
        mv[p] = o.margin[i];
      }
    }
#pragma unroll
    for (int p = 0; p < CP; ++p) {
      if (i0 + p * EB + threadIdx.x >= hi) break;
      const bool stop = (sv[p] & 3) == AEB_END_STOP;
      const double d = dv[p];
      if (stop) {
        const double e = d - mean;
        ss += e * e;
      }
      if (need_d) atomicAdd(&h[value_bin(stop ? d : INFINITY, vmin0, sc0)], 1u);
      if (need_m) atomicAdd(&h[(NVB + 1) + value_bin(mv[p], vmin1, sc1)], 1u);
      if (ng >= 2) atomicAdd(&h[HG + grid_rank(stop ? d : INFINITY, glo, gstep, ginv, ng)], 1u);
    }
  }
  ss = wave_reduce(ss, AddOp());
  if ((threadIdx.x & 63) == 0) shd[threadIdx.x >> 6] = ss;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = shd[0];
    for (int w = 1; w < EB / 64; ++w) t += shd[w];
    part[bx] = t;
  }
  unsigned* out = bhist + static_cast<size_t>(bx) * hw;
  for (int j = threadIdx.x; j < hw; j += EB) out[j] = h[j];
}

__global__ __launch_bounds__(EB) void k_pass2(RSegs S, int need_d, int need_m, RReq rq,
                                              int hw) {
  int bx;
  RSeg g;
  if (!seg_of_block(S, blockIdx.x, bx, g)) return;  // beyond the launch's sets (the whole block)
  pass2_blk(g, bx, need_d, need_m, rq, hw);
}

// ---- importance-sampling sums: exact 128-bit fixed point ----
// A nonnegative value as the integer floor(value * 2^shift) in two words
// (the scaling by a power of two and the split are exact in binary64).
__device__ inline void to_fixed(double v, int shift, unsigned long long& hi,
                                unsigned long long& lo) {
  const double t = ldexp(v, shift);
  const double h = floor(ldexp(t, -64));
  hi = static_cast<unsigned long long>(h);
  lo = static_cast<unsigned long long>(t - ldexp(h, 64));
}

// acc[0] low word, acc[1] high word; integer adds in any order give the
// same total, so the sums do not depend on scheduling
__device__ inline void add_fixed(unsigned long long* acc, unsigned long long hi,
                                 unsigned long long lo) {
  if (lo) {
    const unsigned long long old = atomicAdd(&acc[0], lo);
    if (old + lo < old) atomicAdd(&acc[1], 1ull);
  }
  if (hi) atomicAdd(&acc[1], hi);
}

__device__ inline double from_fixed(unsigned long long hi, unsigned long long lo, int shift) {
  return ldexp(static_cast<double>(hi), 64 - shift) + ldexp(static_cast<double>(lo), -shift);
}

// Per block (the histogram pass's slices): for each risk-grid rank bin the
// sums of w and w^2, then bins for the collided samples and for all samples;
// four words per bin (w low, w high, w^2 low, w^2 high), merged into the
// zeroed global accumulators.
__global__ __launch_bounds__(EB) void k_wpass(RSegs S, RReq rq) {
  int bx;
  RSeg g;
  if (!seg_of_block(S, blockIdx.x, bx, g)) return;  // beyond the launch's sets (the whole block)
  const OutCols o = g.out;
  const long long n = g.n;
  const long long chunk = static_cast<long long>(EB) * CP;
  const RLayout RL = layout(n, 0);
  const Sel* sel = reinterpret_cast<const Sel*>(g.base + RL.off_sel);
  unsigned long long* gacc = reinterpret_cast<unsigned long long*>(g.base + RL.off_wa);
  const double glo = rq.glo, gstep = rq.gstep, ginv = rq.ginv;
  const int ng = rq.ng;
  if (!o.weight) return;  // a set without weights (uniform over the block)
  __shared__ unsigned long long acc[WACC];
  const int G = ng >= 2 ? ng + 1 : 0;  // rank bins 0..ng
  const int nacc = (G + 2) * 4;
  for (int j = threadIdx.x; j < nacc; j += EB) acc[j] = 0ull;
  __syncthreads();
  const int s1 = sel->wshift[0], s2 = sel->wshift[1];
  const long long lo = static_cast<long long>(bx) * chunk;
  const long long hi = lo + chunk < n ? lo + chunk : n;
  for (long long i = lo + threadIdx.x; i < hi; i += EB) {
    const double w = o.weight[i];
    if (!(w >= 0.0 && w < INFINITY)) continue;  // reported through the statistics' flag
    const uint8_t st = o.status[i];
    const double d = o.dist[i];
    unsigned long long h1, l1, h2, l2;
    to_fixed(w, s1, h1, l1);
    to_fixed(w * w, s2, h2, l2);
    if (G) {
      const int b = grid_rank((st & 3) == AEB_END_STOP ? d : INFINITY, glo, gstep, ginv, ng);
      add_fixed(&acc[4 * b], h1, l1);
      add_fixed(&acc[4 * b + 2], h2, l2);
    }
    if (st & AEB_COLLIDED) {
      add_fixed(&acc[4 * G], h1, l1);
      add_fixed(&acc[4 * G + 2], h2, l2);
    }
    add_fixed(&acc[4 * (G + 1)], h1, l1);
  }
  __syncthreads();
  for (int j = threadIdx.x; j < nacc / 2; j += EB) {
    const unsigned long long l = acc[2 * j], h = acc[2 * j + 1];
    if (l | h) add_fixed(&gacc[2 * j], h, l);
  }
}

// The weighted estimates from the accumulated sums (one thread, in a fixed
// order): suffix sums over the rank bins from the top give sum w [D > H0_j].
__global__ void k_wfin(RSegs S, int ng) {
  if (static_cast<int>(blockIdx.x) >= seg_count(S)) return;
  const RSeg g = seg_at(S, blockIdx.x);
  if (!g.out.weight) return;
  const long long n = g.n;
  const RLayout RL = layout(n, 0);
  const Sel* sel = reinterpret_cast<const Sel*>(g.base + RL.off_sel);
  const unsigned long long* gacc = reinterpret_cast<const unsigned long long*>(g.base + RL.off_wa);
  aeb_stats* st = g.st;
  if (threadIdx.x != 0) return;
  const int G = ng >= 2 ? ng + 1 : 0;
  const double nd = static_cast<double>(n);
  const int s1 = sel->wshift[0], s2 = sel->wshift[1];
  if (st->weighted != 1) {
    st->p_collision_w = st->p_collision_se = st->weight_mean = NAN;
    for (int j = 0; j < ng; ++j) st->risk_pw[j] = st->risk_se[j] = NAN;
    return;
  }
  auto se_of = [&](double p, double m2) {
    const double v = m2 / nd - p * p;
    return n > 1 ? sqrt((v > 0.0 ? v : 0.0) / (nd - 1.0)) : NAN;
  };
  unsigned long long a_l = 0, a_h = 0, b_l = 0, b_h = 0;  // suffix sums of w and w^2
  for (int b = G - 1; b >= 1; --b) {
    const unsigned long long* c = gacc + 4 * b;
    const unsigned long long al = a_l + c[0];
    a_h += c[1] + (al < a_l ? 1ull : 0ull);
    a_l = al;
    const unsigned long long bl = b_l + c[2];
    b_h += c[3] + (bl < b_l ? 1ull : 0ull);
    b_l = bl;
    const double p = from_fixed(a_h, a_l, s1) / nd;
    st->risk_pw[b - 1] = p;
    st->risk_se[b - 1] = se_of(p, from_fixed(b_h, b_l, s2));
  }
  const unsigned long long* c = gacc + 4 * G;
  const double pc = from_fixed(c[1], c[0], s1) / nd;
  st->p_collision_w = pc;
  st->p_collision_se = se_of(pc, from_fixed(c[3], c[2], s2));
  st->weight_mean = from_fixed(gacc[4 * (G + 1) + 1], gacc[4 * (G + 1)], s1) / nd;
}

// Bin totals of the block-private histograms: a 2-D grid, each thread sums
// BT_ROWS blocks' counts of one bin (adjacent threads, adjacent bins) and adds
// them to the zeroed totals (integer adds: order-free).
constexpr int BT_ROWS = 16;
__global__ __launch_bounds__(256) void k_bin_totals(RSegs S, int hw) {
  if (S.tab && S.rmap[blockIdx.y] < 0) return;
  const RSeg& g = S.tab ? S.tab[S.rmap[blockIdx.y]] : S.one;
  const int row = S.tab ? static_cast<int>(blockIdx.y) - g.row0 : static_cast<int>(blockIdx.y);
  const RLayout RL = layout(g.n, 0);
  const unsigned* bhist = reinterpret_cast<const unsigned*>(g.base + RL.off_bh);
  unsigned* btot = reinterpret_cast<unsigned*>(g.base + RL.off_bt);
  const int nb = RL.nb2;
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= hw) return;
  const int b0 = row * BT_ROWS;
  const int b1 = b0 + BT_ROWS < nb ? b0 + BT_ROWS : nb;
  unsigned c = 0;
  for (int b = b0; b < b1; ++b) c += bhist[static_cast<size_t>(b) * hw + j];
  if (c) atomicAdd(&btot[j], c);
}

// Block 0: the sd and the risk curve.  Block 1 + t: find the value bin
// holding target t's rank.
__device__ inline void fin2_blk(const RSeg& g, int bx, const RReq& rq, int hw) {
  const int T1 = 1 + rq.n_risk + rq.n_mq;
  const long long n = g.n;
  const int ng = rq.ng;
  const RLayout RL = layout(n, T1 - 1);
  const double* part = reinterpret_cast<const double*>(g.base + RL.off_var);
  const int nb = RL.nb2;
  aeb_stats* st = g.st;
  Sel* sel = reinterpret_cast<Sel*>(g.base + RL.off_sel);
  const unsigned* btot = reinterpret_cast<const unsigned*>(g.base + RL.off_bt);
  const unsigned* bhist = reinterpret_cast<const unsigned*>(g.base + RL.off_bh);
  unsigned* boff = reinterpret_cast<unsigned*>(g.base + RL.off_bo);
  __shared__ double shd[FB];
  __shared__ unsigned long long shu[FB];
  __shared__ int s_bin;
  if (bx == 0) {
    double ss = 0.0;
    for (int b = threadIdx.x; b < nb; b += FB) ss += part[b];
    ss = block_reduce<FB>(ss, shd, AddOp());
    if (threadIdx.x == 0)
      st->sd_dist = st->n_stop > 1 ? sqrt(ss / static_cast<double>(st->n_stop - 1)) : NAN;
    // risk curve: #{D > H0_j} = n - #{D with at most j headways below it}
    const unsigned* gh = btot + HG;
    constexpr int PER = (AEB_MAX_GRID + FB - 1) / FB;
    unsigned long long loc = 0;
    for (int q = 0; q < PER; ++q) {
      const int j = threadIdx.x * PER + q;
      if (j < ng) loc += gh[j];
    }
    unsigned long long before = block_exscan<FB>(loc, shu);
    for (int q = 0; q < PER; ++q) {
      const int j = threadIdx.x * PER + q;
      if (j < ng) {
        before += gh[j];
        const long long above = n - static_cast<long long>(before);
        st->risk_count[j] = above;
        st->risk_p[j] = static_cast<double>(above) / static_cast<double>(n);
      }
    }
    return;
  }
  const int t = bx - 1;
  if (t >= (rq.n_risk + rq.n_mq)) return;
  if (threadIdx.x == 0) s_bin = -1;
  const unsigned* tot = btot + (sel_kind(rq, t) ? (NVB + 1) : 0);
  constexpr int PER = (NVB + 1 + FB - 1) / FB;
  unsigned cnt[PER];
  unsigned long long loc = 0;
  for (int q = 0; q < PER; ++q) {
    const int j = threadIdx.x * PER + q;
    cnt[q] = j <= NVB ? tot[j] : 0u;
    loc += cnt[q];
  }
  const unsigned long long r = sel_rank(rq, n, t);
  unsigned long long before = block_exscan<FB>(loc, shu);
  if (r >= before && r < before + loc) {
    for (int q = 0; q < PER; ++q) {
      const int j = threadIdx.x * PER + q;
      if (j > NVB) break;
      if (r < before + cnt[q]) {
        sel->rank_in_bin[t] = static_cast<unsigned>(r - before);
        sel->bin_count[t] = cnt[q];
        if (j == NVB) {  // the rank falls among the censored (+inf) samples
          sel->bin[t] = -1;
          if (t < rq.n_risk) st->headway[t] = INFINITY;
        } else if (cnt[q] > CAP) {
          sel->bin[t] = -1;
          atomicOr(&sel->fallback, 1);
        } else {
          sel->bin[t] = j;
          s_bin = j;
        }
        break;
      }
      before += cnt[q];
    }
  }
  __syncthreads();
  // where each histogram block's elements of the bin go among the candidates:
  // an exclusive scan of the block histograms' counts of that bin, so the
  // collection needs no global atomics (it uses the histogram pass's blocks)
  const int j = s_bin;
  if (j < 0) return;
  const int col = (sel_kind(rq, t) ? (NVB + 1) : 0) + j;
  unsigned long long carry = 0;
  for (int b0 = 0; b0 < nb; b0 += FB) {
    const int b = b0 + static_cast<int>(threadIdx.x);
    const unsigned long long c = b < nb ? bhist[static_cast<size_t>(b) * hw + col] : 0ull;
    const unsigned long long ex = block_exscan<FB>(c, shu);
    if (b < nb) boff[static_cast<size_t>(t) * nb + b] = static_cast<unsigned>(carry + ex);
    if (threadIdx.x == FB - 1) shu[0] = ex + c;  // the tile's total
    __syncthreads();
    carry += shu[0];
    __syncthreads();
  }
}

__global__ __launch_bounds__(FB) void k_fin2(RSegs S, RReq rq, int hw) {
  const int T1 = 1 + rq.n_risk + rq.n_mq;
  if (static_cast<int>(blockIdx.x / T1) >= seg_count(S)) return;
  fin2_blk(seg_at(S, blockIdx.x / T1), blockIdx.x % T1, rq, hw);
}

// Collect the keys of every element in a target's bin: block b of the
// histogram pass's decomposition writes its elements from the offset the bin
// search computed for it, ranked inside the block by LDS counters.
__device__ inline void collect_blk(const RSeg& g, int bx, const RReq& rq) {
  const OutCols o = g.out;
  const long long n = g.n;
  const long long chunk = static_cast<long long>(EB) * CP;
  const RLayout RL = layout(n, rq.n_risk + rq.n_mq);
  const Sel* sel = reinterpret_cast<const Sel*>(g.base + RL.off_sel);
  const unsigned* boff = reinterpret_cast<const unsigned*>(g.base + RL.off_bo);
  unsigned long long* cand = reinterpret_cast<unsigned long long*>(g.base + RL.off_cand);
  const int nbk = RL.nb2;
  const unsigned ccap = RL.ccap;
  __shared__ int tb[MAX_T], tk[MAX_T];
  __shared__ unsigned lc[MAX_T], lbase[MAX_T];
  __shared__ double vmin[2], scale[2];
  const int T = (rq.n_risk + rq.n_mq);
  if (static_cast<int>(threadIdx.x) < T) {
    tb[threadIdx.x] = sel->bin[threadIdx.x];
    tk[threadIdx.x] = sel_kind(rq, threadIdx.x);
    lc[threadIdx.x] = 0u;
    lbase[threadIdx.x] =
        tb[threadIdx.x] >= 0 ? boff[static_cast<size_t>(threadIdx.x) * nbk + bx] : 0u;
  }
  if (threadIdx.x < 2) {
    vmin[threadIdx.x] = sel->vmin[threadIdx.x];
    scale[threadIdx.x] = sel->scale[threadIdx.x];
  }
  __syncthreads();
  const long long lo = static_cast<long long>(bx) * chunk;
  const long long hi = lo + chunk < n ? lo + chunk : n;
  // each pass loads CP elements per thread before using any of them
  for (long long i0 = lo; i0 < hi; i0 += static_cast<long long>(EB) * CP) {
    uint8_t stt[CP];
    double dv[CP], mv[CP];
#pragma unroll
    for (int p = 0; p < CP; ++p) {
      const long long i = i0 + p * EB + threadIdx.x;
      stt[p] = 0;
      dv[p] = mv[p] = 0.0;
      if (i < hi) {
        stt[p] = o.status[i];
        dv[p] = o.dist[i];
        mv[p] = o.margin[i];
      }
    }
#pragma unroll
    for (int p = 0; p < CP; ++p) {
      const bool ok = i0 + p * EB + threadIdx.x < hi;
      const double dc = (stt[p] & 3) == AEB_END_STOP ? dv[p] : INFINITY;
      const double m = mv[p];
      const int bd = value_bin(dc, vmin[0], scale[0]);
      const int bm = value_bin(m, vmin[1], scale[1]);
      // most wavefronts hold no element of any target's bin: one test first
      bool any = false;
#pragma unroll
      for (int t = 0; t < MAX_T; ++t)
        if (t < T) any = any || (tb[t] >= 0 && (tk[t] ? bm : bd) == tb[t]);
      if (!(ok && any)) continue;
      for (int t = 0; t < T; ++t) {
        const int b = tk[t] ? bm : bd;
        if (tb[t] >= 0 && b == tb[t]) {
          const unsigned slot = lbase[t] + atomicAdd(&lc[t], 1u);
          if (slot < ccap) cand[t * ccap + slot] = ordered(tk[t] ? m : dc);
        }
      }
    }
  }
}

__global__ __launch_bounds__(EB) void k_collect(RSegs S, RReq rq) {
  int bx;
  RSeg g;
  if (!seg_of_block(S, blockIdx.x, bx, g)) return;  // beyond the launch's sets (the whole block)
  collect_blk(g, bx, rq);
}

// One block per target: the element of rank r among the bin's candidates by
// a most-significant-digit radix select in LDS, starting at the first byte
// in which the candidates differ (they share the bin's leading bits).
template <int NT>
__device__ inline void pick_tgt(const RSeg& g, int t, const RReq& rq) {
  static_assert(NT >= 256 && NT % 64 == 0, "a thread per digit bin at least");
  const int T = rq.n_risk + rq.n_mq;
  const RLayout RL = layout(g.n, T);
  const Sel* sel = reinterpret_cast<const Sel*>(g.base + RL.off_sel);
  const unsigned long long* cand = reinterpret_cast<const unsigned long long*>(g.base + RL.off_cand);
  const unsigned ccap = RL.ccap;
  aeb_stats* st = g.st;
  __shared__ unsigned long long key[CAP];
  __shared__ unsigned hist[256];
  __shared__ unsigned long long wlo[NT / 64], whi[NT / 64];
  __shared__ unsigned long long s_prefix;
  __shared__ unsigned s_rank;
  // the host reads the fallback flag through the statistics' reserved word
  if (t == 0 && threadIdx.x == 0) st->reserved = sel->fallback;
  if (t >= (rq.n_risk + rq.n_mq) || sel->bin[t] < 0) return;
  // every element of the bin was collected (the bin holds at most CAP)
  const unsigned m = sel->bin_count[t] < ccap ? sel->bin_count[t] : ccap;
  unsigned long long lo = ~0ull, hi = 0ull;
  for (unsigned j = threadIdx.x; j < m; j += NT) {
    const unsigned long long k = cand[t * ccap + j];
    key[j] = k;
    lo = k < lo ? k : lo;
    hi = k > hi ? k : hi;
  }
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned long long a = __shfl_xor(lo, o), b = __shfl_xor(hi, o);
    lo = a < lo ? a : lo;
    hi = b > hi ? b : hi;
  }
  if ((threadIdx.x & 63) == 0) {
    wlo[threadIdx.x >> 6] = lo;
    whi[threadIdx.x >> 6] = hi;
  }
  __syncthreads();
  lo = wlo[0];
  hi = whi[0];
  for (int w = 1; w < NT / 64; ++w) {
    lo = wlo[w] < lo ? wlo[w] : lo;
    hi = whi[w] > hi ? whi[w] : hi;
  }
  const unsigned long long diff = lo ^ hi;
  const int first = diff ? __clzll(static_cast<long long>(diff)) / 8 : 8;  // first differing byte
  if (threadIdx.x == 0) {
    s_prefix = first == 0 ? 0ull : (lo & (~0ull << (64 - 8 * first)));
    s_rank = sel->rank_in_bin[t];
  }
  __syncthreads();
  for (int pass = first; pass < 8; ++pass) {
    const int shift = 56 - 8 * pass;
    const unsigned long long mask = pass == 0 ? 0ull : (~0ull << (64 - 8 * pass));
    const unsigned long long pre = s_prefix;
    if (threadIdx.x < 256) hist[threadIdx.x] = 0;  // 256 digit bins
    __syncthreads();
    for (unsigned j = threadIdx.x; j < m; j += NT) {
      const unsigned long long k = key[j];
      if ((k & mask) == pre) atomicAdd(&hist[(k >> shift) & 255ull], 1u);
    }
    __syncthreads();
    if (threadIdx.x < 64) {
      // wave 0: digit whose cumulative count passes the rank (4 bins per lane)
      const int l = threadIdx.x;
      unsigned c[4], tot = 0;
      for (int q = 0; q < 4; ++q) {
        c[q] = hist[4 * l + q];
        tot += c[q];
      }
      unsigned inc = tot;  // inclusive scan over lanes
      for (int o = 1; o < 64; o <<= 1) {
        const unsigned v = __shfl_up(inc, o);
        if (l >= o) inc += v;
      }
      const unsigned r = s_rank;
      unsigned before = inc - tot;
      if (r >= before && r < inc) {
        for (int q = 0; q < 4; ++q) {
          if (r < before + c[q]) {
            s_prefix = pre | (static_cast<unsigned long long>(4 * l + q) << shift);
            s_rank = r - before;
            break;
          }
          before += c[q];
        }
      }
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double v = unordered(first == 8 ? lo : s_prefix);
    if (t < rq.n_risk)
      st->headway[t] = v;
    else
      st->margin_q[t - rq.n_risk] = v;
  }
}

__global__ __launch_bounds__(RB) void k_pick(RSegs S, RReq rq) {
  const int T = rq.n_risk + rq.n_mq;
  if (static_cast<int>(blockIdx.x / T) >= seg_count(S)) return;
  pick_tgt<RB>(seg_at(S, blockIdx.x / T), blockIdx.x % T, rq);
}

// ---- small sets: the sequence in one workgroup per set ----
// Every pass over a set of at most SMALL_N samples (one element-pass block)
// run by one workgroup of EB threads with the same per-block arithmetic and
// the same combination order as the separate kernels, so the statistics are
// the same bits; the zeroing, the bin totals and the radix select (integer or
// exact work) are done the workgroup's way.  Three kernels replace nine
// launches (for such sets the launches, not the elements, set the time): the
// first runs through the bin search, the second collects the candidates (one
// kernel for both would keep too many values live for the registers of 1,024
// threads), the third selects, a workgroup per target.  The kernels take any number of blocks per set,
// one after another, but beyond one block the separate kernels, whose blocks
// run side by side, are faster (measured: 0.20 against 0.12 ms per call at
// 25,000 samples).
constexpr long long SMALL_N = static_cast<long long>(EB) * CP;

__global__ __launch_bounds__(EB) void k_small(RSegs S, RReq rq, int hw, int need_d,
                                              int need_m) {
  if (static_cast<int>(blockIdx.x) >= seg_count(S)) return;
  const RSeg g = seg_at(S, blockIdx.x);
  const int T = rq.n_risk + rq.n_mq;
  const RLayout RL = layout(g.n, 0);
  {
    unsigned* a = reinterpret_cast<unsigned*>(g.base + RL.off_sel);
    const long long na = static_cast<long long>((RL.off_zero_end - RL.off_sel) / 4);
    for (long long i = threadIdx.x; i < na; i += EB) a[i] = 0u;
    unsigned* b = reinterpret_cast<unsigned*>(g.st);
    for (int i = threadIdx.x; i < static_cast<int>(sizeof(aeb_stats) / 4); i += EB) b[i] = 0u;
  }
  __syncthreads();
  for (int bx = 0; bx < RL.nb; ++bx) {
    pass1_blk(g, bx);
    __syncthreads();
  }
  fin1_set(g);
  __syncthreads();
  for (int bx = 0; bx < RL.nb2; ++bx) {
    pass2_blk(g, bx, need_d, need_m, rq, hw);
    __syncthreads();
  }
  if (hw > 0) {
    const unsigned* bhist = reinterpret_cast<const unsigned*>(g.base + RL.off_bh);
    unsigned* btot = reinterpret_cast<unsigned*>(g.base + RL.off_bt);
    for (int j = threadIdx.x; j < hw; j += EB) {
      unsigned c = 0;
      for (int b = 0; b < RL.nb2; ++b) c += bhist[static_cast<size_t>(b) * hw + j];
      btot[j] = c;
    }
  }
  __syncthreads();
  for (int j = 0; j <= T; ++j) {
    fin2_blk(g, j, rq, hw);
    __syncthreads();
  }
}

__global__ __launch_bounds__(EB) void k_small_collect(RSegs S, RReq rq) {
  if (static_cast<int>(blockIdx.x) >= seg_count(S)) return;
  const RSeg g = seg_at(S, blockIdx.x);
  const RLayout RL = layout(g.n, 0);
  for (int bx = 0; bx < RL.nb2; ++bx) {
    collect_blk(g, bx, rq);
    __syncthreads();
  }
}

// ---- fallback: most-significant-digit radix select, 8 passes of 8 bits ----
// The sets whose selection asks for it, FB_SETS of them per launch sequence
// (by value in the kernel arguments): every kernel covers all of them, so a
// batch with many such sets costs one sequence of 17 short launches per FB_SETS
// and not one per set, and then two small copies per set.  26 sets of 100,000 samples (a sweep's scenarios in which most
// samples collide share one margin bin): 0.35 ms against 20 ms one set after the
// other with two wavefronts per SIMD at work on one of 36.
constexpr int FB_SETS = FALLBACK_SETS;
struct FbSet {
  const double* dist;
  const uint8_t* status;
  const double* margin;
  long long n;
  SelState* ss;
  unsigned* hist;  // T x 256 counters
  aeb_stats* st;
};
struct FbSets {
  FbSet s[FB_SETS];
};

// a set's targets, and its counters cleared
__global__ __launch_bounds__(RB) void k_select_init(FbSets F, RReq rq) {
  const FbSet& g = F.s[blockIdx.x];
  const int T = rq.n_risk + rq.n_mq;
  for (int j = threadIdx.x; j < T * 256; j += RB) g.hist[j] = 0;
  if (static_cast<int>(threadIdx.x) < T) {
    g.ss->prefix[threadIdx.x] = 0;
    g.ss->rank[threadIdx.x] = sel_rank(rq, g.n, threadIdx.x);
  }
}

// Digit counts of the elements that share each target's prefix, a workgroup
// per EB x CP elements of a set (blockIdx.y), counted in LDS.
__global__ __launch_bounds__(EB) void k_select_hist(FbSets F, RReq rq, int pass) {
  const FbSet& g = F.s[blockIdx.y];
  const long long lo = static_cast<long long>(blockIdx.x) * (EB * CP);
  if (lo >= g.n) return;
  const int T = rq.n_risk + rq.n_mq;
  __shared__ unsigned hist[MAX_T * 256];
  __shared__ unsigned long long pre[MAX_T];
  for (int j = threadIdx.x; j < T * 256; j += EB) hist[j] = 0;
  if (static_cast<int>(threadIdx.x) < T) pre[threadIdx.x] = g.ss->prefix[threadIdx.x];
  __syncthreads();
  const int shift = 56 - 8 * pass;
  const unsigned long long mask = pass == 0 ? 0ull : (~0ull << (64 - 8 * pass));
  unsigned long long kd[CP], km[CP];
#pragma unroll
  for (int p = 0; p < CP; ++p) {
    const long long i = lo + p * EB + threadIdx.x;
    kd[p] = km[p] = 0;
    if (i < g.n) {
      kd[p] = ordered(censored(g.dist, g.status, i));
      km[p] = ordered(g.margin[i]);
    }
  }
#pragma unroll
  for (int p = 0; p < CP; ++p) {
    const bool ok = lo + p * EB + threadIdx.x < g.n;
    for (int t = 0; t < T; ++t) {
      const unsigned long long key = t >= rq.n_risk ? km[p] : kd[p];
      const bool mine = ok && (key & mask) == (pre[t] & mask);
      const unsigned d = static_cast<unsigned>((key >> shift) & 255ull);
      // the leading digits agree over most wavefronts: one add for all of them
      const unsigned long long who = __ballot(mine);
      if (who == 0) continue;
      const unsigned d0 = __shfl(d, __ffsll(static_cast<long long>(who)) - 1);
      if (__ballot(mine && d != d0) == 0) {
        if ((threadIdx.x & 63) == 0) atomicAdd(&hist[t * 256 + d0], __popcll(who));
      } else if (mine) {
        atomicAdd(&hist[t * 256 + d], 1u);
      }
    }
  }
  __syncthreads();
  for (int j = threadIdx.x; j < T * 256; j += EB)
    if (hist[j]) atomicAdd(&g.hist[j], hist[j]);
}

// Each target's digit: one wavefront per target, four digits per lane; the
// counters are cleared for the next pass.  After the last one the prefix is
// the element.
__global__ __launch_bounds__(64) void k_select_step(FbSets F, RReq rq, int pass) {
  const FbSet& g = F.s[blockIdx.y];
  const int t = blockIdx.x, l = threadIdx.x;
  unsigned* h = g.hist + t * 256;
  unsigned long long c[4], tot = 0;
  for (int q = 0; q < 4; ++q) {
    c[q] = h[4 * l + q];
    tot += c[q];
    h[4 * l + q] = 0;
  }
  unsigned long long inc = tot;  // inclusive scan over the lanes
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned long long v = __shfl_up(inc, o);
    if (l >= o) inc += v;
  }
  const unsigned long long r = g.ss->rank[t];
  unsigned long long before = inc - tot;
  if (!(r >= before && r < inc)) return;  // the one lane that holds the rank
  for (int q = 0; q < 4; ++q) {
    if (r < before + c[q]) {
      const unsigned long long pre =
          g.ss->prefix[t] | (static_cast<unsigned long long>(4 * l + q) << (56 - 8 * pass));
      g.ss->rank[t] = r - before;
      g.ss->prefix[t] = pre;
      if (pass == 7) {
        if (t < rq.n_risk)
          g.st->headway[t] = unordered(pre);
        else
          g.st->margin_q[t - rq.n_risk] = unordered(pre);
      }
      break;
    }
    before += c[q];
  }
}

}  // namespace

namespace {

// zero each set's selection state, bin totals and weighted accumulators, and
// its statistics (fill kernels: no memset nodes in recorded graphs)
__global__ void k_zero_sets(RSegs S) {
  if (static_cast<int>(blockIdx.y) >= seg_count(S)) return;
  const RSeg g = seg_at(S, blockIdx.y);
  const RLayout RL = layout(g.n, 0);
  unsigned* a = reinterpret_cast<unsigned*>(g.base + RL.off_sel);
  const long long na = static_cast<long long>((RL.off_zero_end - RL.off_sel) / 4);
  unsigned* b = reinterpret_cast<unsigned*>(g.st);
  const long long nw = static_cast<long long>(sizeof(aeb_stats) / 4);
  const long long stride = static_cast<long long>(gridDim.x) * blockDim.x;
  for (long long i = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x; i < na; i += stride)
    a[i] = 0u;
  for (long long i = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x; i < nw; i += stride)
    b[i] = 0u;
}

// the statistics written to pinned host memory by the kernel itself
constexpr int OUT_BLOCKS = 10;
__global__ __launch_bounds__(RB) void k_stats_out(const aeb_stats* st, aeb_stats* host) {
  static_assert(sizeof(aeb_stats) % sizeof(unsigned long long) == 0, "whole words");
  const unsigned long long* a = reinterpret_cast<const unsigned long long*>(st);
  unsigned long long* b = reinterpret_cast<unsigned long long*>(host);
  const int n = static_cast<int>(sizeof(aeb_stats) / sizeof(unsigned long long));
  for (int i = blockIdx.x * RB + threadIdx.x; i < n; i += OUT_BLOCKS * RB) b[i] = a[i];
}

int n_targets(const aeb_reduce_req& req) { return req.n_risk + req.n_margin_q; }

RReq rreq_of(const aeb_reduce_req& req) {
  RReq q;
  std::memset(&q, 0, sizeof(q));
  q.n_risk = req.n_risk;
  q.n_mq = req.n_margin_q;
  q.ng = req.n_grid;
  for (int j = 0; j < req.n_risk; ++j) q.risk[j] = req.risk[j];
  for (int j = 0; j < req.n_margin_q; ++j) q.mq[j] = req.margin_q[j];
  q.glo = req.grid_lo;
  q.gstep = q.ng >= 2 ? (req.grid_hi - req.grid_lo) / static_cast<double>(q.ng - 1) : 0.0;
  q.ginv = q.ng >= 2 ? 1.0 / q.gstep : 0.0;
  return q;
}

// Table of a segmented launch, laid out for a capacity of sets, element-pass
// blocks and bin-totals rows: the launch's set count, the sets, the set of
// every block and row (-1 past the launch's), then (device only) the sets'
// statistics.
struct TLayout {
  int cap, tb, tr;
  size_t off_seg, off_bmap, off_rmap, host_bytes, off_stats, total;
};

TLayout tlayout_of(int cap, int tb, int tr) {
  TLayout T;
  T.cap = cap;
  T.tb = tb;
  T.tr = tr;
  T.off_seg = 256;
  T.off_bmap = align256(T.off_seg + sizeof(RSeg) * cap);
  T.off_rmap = align256(T.off_bmap + sizeof(int) * tb);
  T.host_bytes = T.off_rmap + sizeof(int) * tr;
  T.off_stats = align256(T.host_bytes);
  T.total = align256(T.off_stats + sizeof(aeb_stats) * cap);
  return T;
}

// exactly the given sets
TLayout tlayout(int nseg, const int64_t* ns) {
  int tb = 0, tr = 0;
  for (int j = 0; j < nseg; ++j) {
    const RLayout L = layout(ns[j], 0);
    tb += L.nb;
    tr += (L.nb2 + BT_ROWS - 1) / BT_ROWS;
  }
  return tlayout_of(nseg, tb, tr);
}

// any cap sets of cap_samples samples in all: every set adds at most one
// partly filled block and one partly filled row
TLayout tlayout_cap(int cap, int64_t cap_samples) {
  const long long chunk = static_cast<long long>(EB) * CP;
  const int tb = static_cast<int>(cap_samples / chunk) + cap;
  return tlayout_of(cap, tb, tb / BT_ROWS + cap);
}

// Fill the host side of the table for the sets (which must fit T); returns
// whether any set carries importance-sampling weights.
bool fill_table(const TLayout& T, const OutCols* outs, const int64_t* ns, int nseg,
                char* const* bases, char* table_dev, char* hb) {
  *reinterpret_cast<int*>(hb) = nseg;
  RSeg* seg = reinterpret_cast<RSeg*>(hb + T.off_seg);
  int* bmap = reinterpret_cast<int*>(hb + T.off_bmap);
  int* rmap = reinterpret_cast<int*>(hb + T.off_rmap);
  aeb_stats* dst = reinterpret_cast<aeb_stats*>(table_dev + T.off_stats);
  bool weighted = false;
  int blk = 0, row = 0;
  for (int j = 0; j < nseg; ++j) {
    const RLayout L = layout(ns[j], 0);
    std::memset(&seg[j], 0, sizeof(RSeg));
    seg[j].out = outs[j];
    seg[j].n = ns[j];
    seg[j].base = bases[j];
    seg[j].st = dst + j;
    seg[j].nb = L.nb;
    seg[j].blk0 = blk;
    seg[j].row0 = row;
    for (int b = 0; b < L.nb; ++b) bmap[blk + b] = j;
    const int rows = (L.nb2 + BT_ROWS - 1) / BT_ROWS;
    for (int r = 0; r < rows; ++r) rmap[row + r] = j;
    blk += L.nb;
    row += rows;
    weighted = weighted || outs[j].weight != nullptr;
  }
  for (int b = blk; b < T.tb; ++b) bmap[b] = -1;
  for (int r = row; r < T.tr; ++r) rmap[r] = -1;
  return weighted;
}

RSegs table_segs(const TLayout& T, const char* db) {
  RSegs S;
  std::memset(&S, 0, sizeof(S));
  S.tab = reinterpret_cast<const RSeg*>(db + T.off_seg);
  S.bmap = reinterpret_cast<const int*>(db + T.off_bmap);
  S.rmap = reinterpret_cast<const int*>(db + T.off_rmap);
  S.count = reinterpret_cast<const int*>(db);
  return S;
}

// The launch sequence over the sets of S (grids from the totals).
int enqueue_sets(const RSegs& S, int nseg, int tb, int tr, bool weighted, int64_t max_n,
                 const aeb_reduce_req& req, hipStream_t st) {
  // nseg, tb, tr: the grids' capacity of sets, element-pass blocks and rows;
  // max_n: no set holds more samples
  const RReq q = rreq_of(req);
  const int T = n_targets(req);
  const int ng = req.n_grid;
  // block histograms: the value bins only when some target needs them
  const int hw0 = ng >= 2 ? HG + ng + 1 : (T > 0 ? HG : 0);
  if (!weighted && max_n <= SMALL_N) {
    // every set small: one workgroup per set runs the whole sequence
    hipLaunchKernelGGL(k_small, dim3(nseg), dim3(EB), 0, st, S, q, hw0, req.n_risk > 0 ? 1 : 0,
                       req.n_margin_q > 0 ? 1 : 0);
    if (T > 0) {
      hipLaunchKernelGGL(k_small_collect, dim3(nseg), dim3(EB), 0, st, S, q);
      hipLaunchKernelGGL(k_pick, dim3(nseg * T), dim3(RB), 0, st, S, q);
    }
    AEB_HIP(hipGetLastError());
    return AEB_OK;
  }
  hipLaunchKernelGGL(k_zero_sets, dim3(32, nseg), dim3(256), 0, st, S);
  hipLaunchKernelGGL(k_pass1, dim3(tb), dim3(EB), 0, st, S);
  hipLaunchKernelGGL(k_fin1, dim3(nseg), dim3(FB), 0, st, S);
  const int hw = hw0;
  hipLaunchKernelGGL(k_pass2, dim3(tb), dim3(EB), 0, st, S, req.n_risk > 0 ? 1 : 0,
                     req.n_margin_q > 0 ? 1 : 0, q, hw);
  if (hw > 0)
    hipLaunchKernelGGL(k_bin_totals, dim3((hw + 255) / 256, tr), dim3(256), 0, st, S, hw);
  hipLaunchKernelGGL(k_fin2, dim3(nseg * (1 + T)), dim3(FB), 0, st, S, q, hw);
  if (weighted) {
    hipLaunchKernelGGL(k_wpass, dim3(tb), dim3(EB), 0, st, S, q);
    hipLaunchKernelGGL(k_wfin, dim3(nseg), dim3(64), 0, st, S, ng);
  }
  if (T > 0) {
    hipLaunchKernelGGL(k_collect, dim3(tb), dim3(EB), 0, st, S, q);
    hipLaunchKernelGGL(k_pick, dim3(nseg * T), dim3(RB), 0, st, S, q);
  }
  AEB_HIP(hipGetLastError());
  return AEB_OK;
}

}  // namespace

size_t reduce_scratch_bytes(int64_t n, const aeb_reduce_req& req) {
  return layout(n, n_targets(req)).total;
}

size_t reduce_scratch_bytes_cap(int cap_sets, int64_t cap_samples, const aeb_reduce_req& req) {
  // a set's scratch is a fixed part, parts per element-pass block and the
  // candidate lists (min(n, CAP) per target), each rounded up to 256 bytes:
  // bound the blocks by cap_samples / chunk + cap_sets and the candidates
  // by min(cap_samples, cap_sets * CAP)
  const int T = n_targets(req);
  const int tc = T > 0 ? T : 1;
  const RLayout one = layout(1, T);
  const long long chunk = static_cast<long long>(EB) * CP;
  const size_t blocks = static_cast<size_t>(cap_samples / chunk) + cap_sets + 1;
  const size_t per_block = sizeof(Partial) + sizeof(double) + sizeof(unsigned) * HW +
                           sizeof(unsigned) * tc;
  const size_t cand = static_cast<size_t>(cap_samples < static_cast<int64_t>(cap_sets) * CAP
                                              ? cap_samples
                                              : static_cast<int64_t>(cap_sets) * CAP);
  return static_cast<size_t>(cap_sets) * (one.total + 8 * 256) + blocks * per_block +
         cand * sizeof(unsigned long long) * tc;
}

namespace {

int enqueue_one(const OutCols& out, int64_t n, const aeb_reduce_req& req, void* scratch_base,
                hipStream_t st) {
  const RLayout L = layout(n, n_targets(req));
  RSegs S;
  std::memset(&S, 0, sizeof(S));
  S.one.out = out;
  S.one.n = n;
  S.one.base = static_cast<char*>(scratch_base);
  S.one.st = reinterpret_cast<aeb_stats*>(scratch_base);
  S.one.nb = L.nb;
  const int rc = enqueue_sets(S, 1, L.nb, (L.nb2 + BT_ROWS - 1) / BT_ROWS, out.weight != nullptr,
                              n, req, st);
  return rc;
}

}  // namespace

int reduce_enqueue(const OutCols& out, int64_t n, const aeb_reduce_req& req, void* scratch_base,
                   aeb_stats* host_out, hipStream_t st) {
  const int rc = enqueue_one(out, n, req, scratch_base, st);
  if (rc != AEB_OK) return rc;
  // (host_out is the caller's: a copy takes any memory)
  AEB_HIP(hipMemcpyAsync(host_out, scratch_base, sizeof(aeb_stats), hipMemcpyDeviceToHost, st));
  return AEB_OK;
}

size_t reduce_table_bytes(int nseg, const int64_t* ns) { return tlayout(nseg, ns).total; }

size_t reduce_table_bytes_cap(int cap_sets, int64_t cap_samples) {
  return tlayout_cap(cap_sets, cap_samples).total;
}

aeb_stats* reduce_table_stats(void* table_dev, int nseg, const int64_t* ns) {
  return reinterpret_cast<aeb_stats*>(static_cast<char*>(table_dev) + tlayout(nseg, ns).off_stats);
}

aeb_stats* reduce_table_stats_cap(void* table_dev, int cap_sets, int64_t cap_samples) {
  return reinterpret_cast<aeb_stats*>(static_cast<char*>(table_dev) +
                                      tlayout_cap(cap_sets, cap_samples).off_stats);
}

int reduce_enqueue_sets(const OutCols* outs, const int64_t* ns, int nseg,
                        const aeb_reduce_req& req, char* const* bases, void* table_dev,
                        void* table_host, aeb_stats* host_out, hipStream_t st) {
  if (nseg < 1) return fail(AEB_EINVAL, "reduction of no output sets");
  const TLayout T = tlayout(nseg, ns);
  char* db = static_cast<char*>(table_dev);
  char* hb = static_cast<char*>(table_host);
  const bool weighted = fill_table(T, outs, ns, nseg, bases, db, hb);
  int64_t max_n = 0;
  for (int j = 0; j < nseg; ++j) max_n = ns[j] > max_n ? ns[j] : max_n;
  AEB_HIP(hipMemcpyAsync(db, hb, T.host_bytes, hipMemcpyHostToDevice, st));
  const int rc = enqueue_sets(table_segs(T, db), T.cap, T.tb, T.tr, weighted, max_n, req, st);
  if (rc != AEB_OK) return rc;
  AEB_HIP(hipMemcpyAsync(host_out, db + T.off_stats, sizeof(aeb_stats) * nseg,
                         hipMemcpyDeviceToHost, st));
  return AEB_OK;
}

int reduce_fill_sets_cap(const OutCols* outs, const int64_t* ns, int nseg, int cap_sets,
                         int64_t cap_samples, char* const* bases, void* table_dev,
                         void* table_host) {
  int64_t tot = 0;
  for (int j = 0; j < nseg; ++j) tot += ns[j];
  if (nseg < 1 || nseg > cap_sets || tot > cap_samples)
    return fail(AEB_EINVAL, "output sets beyond the recorded reduction's capacity");
  (void)fill_table(tlayout_cap(cap_sets, cap_samples), outs, ns, nseg, bases,
                   static_cast<char*>(table_dev), static_cast<char*>(table_host));
  return AEB_OK;
}

int reduce_enqueue_sets_cap(int cap_sets, int64_t cap_samples, const aeb_reduce_req& req,
                            bool weighted, void* table_dev, const void* table_host,
                            aeb_stats* host_out, hipStream_t st) {
  const TLayout T = tlayout_cap(cap_sets, cap_samples);
  char* db = static_cast<char*>(table_dev);
  AEB_HIP(hipMemcpyAsync(db, table_host, T.host_bytes, hipMemcpyHostToDevice, st));
  const int rc = enqueue_sets(table_segs(T, db), T.cap, T.tb, T.tr, weighted, cap_samples, req,
                              st);
  if (rc != AEB_OK) return rc;
  AEB_HIP(hipMemcpyAsync(host_out, db + T.off_stats, sizeof(aeb_stats) * cap_sets,
                         hipMemcpyDeviceToHost, st));
  return AEB_OK;
}

static std::atomic<unsigned long long> g_fallbacks{0};

unsigned long long reduce_fallback_count() { return g_fallbacks.load(); }

int reduce_fallback(const Fallback* f, int count, const aeb_reduce_req& req, hipStream_t st) {
  // targets whose value bin held more than CAP candidates: radix select
  g_fallbacks.fetch_add(static_cast<unsigned long long>(count));
  const RReq q = rreq_of(req);
  const int T = n_targets(req);
  for (int j0 = 0; j0 < count; j0 += FB_SETS) {
    const int c = count - j0 < FB_SETS ? count - j0 : FB_SETS;
    FbSets F;
    std::memset(&F, 0, sizeof(F));
    int64_t max_n = 0;
    for (int j = 0; j < c; ++j) {
      const Fallback& a = f[j0 + j];
      const RLayout L = layout(a.n, T);
      char* base = static_cast<char*>(a.scratch);
      F.s[j] = FbSet{a.out.dist, a.out.status, a.out.margin, a.n,
                     reinterpret_cast<SelState*>(base + L.off_ss),
                     reinterpret_cast<unsigned*>(base + L.off_sh), a.dstats};
      max_n = a.n > max_n ? a.n : max_n;
    }
    const unsigned nb = static_cast<unsigned>((max_n + EB * CP - 1) / (EB * CP));
    hipLaunchKernelGGL(k_select_init, dim3(c), dim3(RB), 0, st, F, q);
    for (int pass = 0; pass < 8; ++pass) {
      hipLaunchKernelGGL(k_select_hist, dim3(nb, c), dim3(EB), 0, st, F, q, pass);
      hipLaunchKernelGGL(k_select_step, dim3(T, c), dim3(64), 0, st, F, q, pass);
    }
    AEB_HIP(hipGetLastError());
    // the order statistics are all that changed
    for (int j = 0; j < c; ++j) {
      const Fallback& a = f[j0 + j];
      AEB_HIP(hipMemcpyAsync(a.host->headway, a.dstats->headway, sizeof(a.host->headway),
                             hipMemcpyDeviceToHost, st));
      AEB_HIP(hipMemcpyAsync(a.host->margin_q, a.dstats->margin_q, sizeof(a.host->margin_q),
                             hipMemcpyDeviceToHost, st));
    }
  }
  AEB_HIP(hipStreamSynchronize(st));
  for (int j = 0; j < count; ++j) f[j].host->reserved = 0;
  return AEB_OK;
}

int launch_reduce(const OutCols& out, int64_t n, const aeb_reduce_req& req, aeb_stats* host_out,
                  hipStream_t st) {
  void* base = pool_block(reduce_scratch_bytes(n, req), st);
  if (!base) return AEB_ENOMEM;
  // The statistics come by way of the library's pinned memory, written by a
  // kernel: a copy to pageable memory starts only once the kernels are done, and
  // a copy engine has a start of its own (25,000 samples, rollout and reduction:
  // 275 us with the copy, 256 with a copy to pinned memory, 242 so).
  aeb_stats* pin = pool_stats();
  int rc;
  if (pin) {
    rc = enqueue_one(out, n, req, base, st);
    if (rc != AEB_OK) return rc;
    hipLaunchKernelGGL(k_stats_out, dim3(OUT_BLOCKS), dim3(RB), 0, st,
                       static_cast<const aeb_stats*>(base), pin);
    AEB_HIP(hipGetLastError());
  } else {
    rc = reduce_enqueue(out, n, req, base, host_out, st);
    if (rc != AEB_OK) return rc;
  }
  AEB_HIP(hipStreamSynchronize(st));
  if (pin) *host_out = *pin;
  const int fallback = host_out->reserved;
  host_out->reserved = 0;
  if (!fallback) return AEB_OK;
  const Fallback f{out, n, base, static_cast<aeb_stats*>(base), host_out};
  return reduce_fallback(&f, 1, req, st);
}

int launch_batch_reduce(const OutCols* outs, const int64_t* ns, int nseg,
                        const aeb_reduce_req& req, aeb_stats* host_out, hipStream_t st) {
  // consecutive sets in groups of at most GROUP_BYTES of set scratch (or one
  // larger set): one launch sequence per group, all groups on one pool block
  constexpr size_t GROUP_BYTES = size_t(256) << 20;
  constexpr int GROUP_SETS = 4096;
  std::vector<int> first{0};
  size_t need = 0;
  {
    size_t acc = 0;
    int cnt = 0;
    for (int j = 0; j < nseg; ++j) {
      const size_t b = align256(reduce_scratch_bytes(ns[j], req));
      if (cnt > 0 && (acc + b > GROUP_BYTES || cnt == GROUP_SETS)) {
        first.push_back(j);
        acc = 0;
        cnt = 0;
      }
      acc += b;
      ++cnt;
    }
    first.push_back(nseg);
    for (size_t g = 0; g + 1 < first.size(); ++g) {
      const int a = first[g], c = first[g + 1] - first[g];
      size_t bytes = align256(reduce_table_bytes(c, ns + a));
      for (int j = a; j < a + c; ++j) bytes += align256(reduce_scratch_bytes(ns[j], req));
      need = bytes > need ? bytes : need;
    }
  }
  char* pool = static_cast<char*>(pool_block(need, st));
  if (!pool) return AEB_ENOMEM;
  std::vector<char> host;
  std::vector<char*> bases;
  for (size_t g = 0; g + 1 < first.size(); ++g) {
    const int a = first[g], c = first[g + 1] - first[g];
    const size_t tbytes = align256(reduce_table_bytes(c, ns + a));
    host.assign(tbytes, 0);
    bases.clear();
    char* p = pool + tbytes;
    for (int j = a; j < a + c; ++j) {
      bases.push_back(p);
      p += align256(reduce_scratch_bytes(ns[j], req));
    }
    int rc = reduce_enqueue_sets(outs + a, ns + a, c, req, bases.data(), pool, host.data(),
                                 host_out + a, st);
    if (rc != AEB_OK) return rc;
    AEB_HIP(hipStreamSynchronize(st));
    aeb_stats* dst = reduce_table_stats(pool, c, ns + a);
    FallbackList fb;
    for (int j = 0; j < c; ++j) {
      aeb_stats& h = host_out[a + j];
      if (!h.reserved) continue;
      rc = fb.add(Fallback{outs[a + j], ns[a + j], bases[j], dst + j, &h}, req, st);
      if (rc != AEB_OK) return rc;
    }
    rc = fb.run(req, st);
    if (rc != AEB_OK) return rc;
  }
  return AEB_OK;
}

}  // namespace aeb

// The integration kernels' own source on the CPU (hip/hip_runtime.h here): the
// scenarios of each file as one batched launch against each scenario's launch
// alone, bit for bit.  Arguments: a kernel ("fp64", "fp64x2" or "fp32c") and
// files of aeb_scenario records.  Prints a line per file; the exit status is 0
// if every launch ended, none took a step past its horizon and none differed.
// A kernel named with a "!" gets job records whose bound on the speed's change is
// 20 m/s^2 whatever the actuator: blocks may then hold events that their replay
// does not find, and the exit status is 0 if samples are marked with a distance
// that is no number, and none is left without an end and without that mark.
#include <hip/hip_runtime.h>

#include "kernels_fast.hip"

#include <cstdio>
#include <string>

namespace aeb {
int fail(int code, const std::string&) { return code; }
void timing_begin(hipStream_t) {}
void timing_end(hipStream_t) {}
unsigned long long* timing_lanes() { return nullptr; }
TuneCfg tune_get(int, int) { return TuneCfg{}; }
void* scratch_slot(int, size_t, hipStream_t) { return nullptr; }
int launch_fixup(const aeb_scenario&, const ParamSrc*, const OutCols&, const uint32_t*,
                 hipStream_t) {
  return AEB_OK;
}
int64_t horizon_steps(const aeb_scenario& s) { return std::llround(s.horizon / s.dt); }
int64_t dead_steps(const aeb_scenario& s) { return std::llround(s.dead_time / s.dt); }
}  // namespace aeb

using namespace aeb;

namespace {

enum Kernel { FP64, FP64X2, FP32C };
bool g_wrong_bound = false;
constexpr long long LIMIT = 400000;  // wave operations of one wavefront

struct Out {
  std::vector<double> dist, margin;
  std::vector<uint8_t> status;
  std::vector<int32_t> steps;
  std::vector<float> vimp;
  explicit Out(size_t n) : dist(n, -1.0), margin(n, -1.0), status(n, 99), steps(n, -1), vimp(n, -1.0f) {}
  OutCols cols() {
    return OutCols{dist.data(), status.data(), steps.data(), margin.data(), vimp.data(), nullptr};
  }
  bool same(const Out& o, size_t i) const {
    return !std::memcmp(&dist[i], &o.dist[i], 8) && !std::memcmp(&margin[i], &o.margin[i], 8) &&
           status[i] == o.status[i] && steps[i] == o.steps[i] &&
           !std::memcmp(&vimp[i], &o.vimp[i], 4);
  }
};

// one launch; false if a wavefront does not end
template <bool BATCH, int OBS, int INTEG>
bool launch(const std::vector<aeb_scenario>& scns, std::vector<Out>& outs, Kernel kern) {
  constexpr bool LEAD = OBS == AEB_OBS_LEAD, EULER = INTEG == AEB_EULER;
  const int m = static_cast<int>(scns.size());
  std::vector<ScnDev> tab(m);
  std::vector<OutCols> cols;
  for (Out& o : outs) cols.push_back(o.cols());
  int64_t n = 0, cap = 0;
  fill_batch_table(scns.data(), m, cols.data(), tab.data(), &n, &cap);
  std::vector<Job> jobs(n);
  std::vector<LeadJob> leads(n);
  std::vector<uint32_t> keys(n), perm(n);
  std::vector<int32_t> nds(n);
  PrepArgs pa{};
  pa.s = scns[0];
  pa.n = n;
  pa.cap = static_cast<float>(cap);
  pa.scns = scns.data();
  pa.tab = tab.data();
  pa.n_scn = m;
  pa.nd = tab[0].nd;
  pa.nmax = tab[0].nmax;
  for (const aeb_scenario& s : scns)
    if (perception_on(s)) pa.nds = nds.data();
  for (int j = 0; j < m; ++j)
    for (int64_t i = 0; i < static_cast<int64_t>(scns[j].n_samples); ++i)
      keys[tab[j].off + i] = prep_sample<true, BATCH>(pa, tab[j].off + i, j, i, pa.cap,
                                                      jobs.data(), leads.data());
  for (Job& J : jobs)
    if (g_wrong_bound) J.dmax = 20.0;
  for (int64_t i = 0; i < n; ++i) perm[i] = static_cast<uint32_t>(i);
  std::stable_sort(perm.begin(), perm.end(),
                   [&](uint32_t a, uint32_t b) { return keys[a] < keys[b]; });
  Ctx ctx{};
  ctx.impact_exit = scns[0].impact_exit;
  ctx.nds = pa.nds;
  if (BATCH) {
    ctx.tab = tab.data();
  } else {
    ctx.dt = scns[0].dt;
    ctx.a_cmd = scns[0].a_cmd;
    ctx.nd = pa.nd;
    ctx.nmax = pa.nmax;
    ctx.out = cols[0];
  }
  unsigned long long counter = 0;
  const int64_t per = kern == FP64X2 ? 128 : 64;
  const unsigned waves = static_cast<unsigned>((n + per - 1) / per);
  wave::block_dim = dim3(64);
  wave::grid_dim = dim3(waves);
  for (unsigned w = 0; w < waves; ++w) {
    wave::block_idx = dim3(w);
    const bool ended = wave::run(
        [&] {
          if (kern == FP64)
            k_roll_fp64<OBS, EULER ? 128 : 16, BATCH, INTEG>(
                jobs.data(), leads.data(), perm.data(), n, ctx, &counter, 0, nullptr);
          else if constexpr (EULER && LEAD)
            k_roll_fp32c_lead<64, BATCH>(jobs.data(), leads.data(), perm.data(), n, ctx, 1e-3,
                                         1e-4, nullptr, &counter, 0);
          else if constexpr (EULER)
            kern == FP64X2
                ? k_roll_fp64x2<OBS, 64, BATCH>(jobs.data(), perm.data(), n, ctx, &counter, 0)
                : k_roll_fp32c<OBS, 64, BATCH>(jobs.data(), perm.data(), n, ctx, 1e-3, 1e-4,
                                               nullptr, &counter, 0);
        },
        LIMIT);
    if (!ended) return false;
  }
  return true;
}

template <bool BATCH>
bool launch(const std::vector<aeb_scenario>& s, std::vector<Out>& o, Kernel kern) {
  if (s[0].integrator == AEB_RK4)
    return s[0].obstacle == AEB_OBS_NONE ? launch<BATCH, AEB_OBS_NONE, AEB_RK4>(s, o, kern)
                                         : launch<BATCH, AEB_OBS_STATIONARY, AEB_RK4>(s, o, kern);
  if (s[0].obstacle == AEB_OBS_LEAD) return launch<BATCH, AEB_OBS_LEAD, AEB_EULER>(s, o, kern);
  return s[0].obstacle == AEB_OBS_NONE ? launch<BATCH, AEB_OBS_NONE, AEB_EULER>(s, o, kern)
                                       : launch<BATCH, AEB_OBS_STATIONARY, AEB_EULER>(s, o, kern);
}

std::vector<aeb_scenario> load(const char* path) {
  std::vector<aeb_scenario> scns;
  aeb_scenario s;
  std::FILE* f = std::fopen(path, "rb");
  while (f && std::fread(&s, sizeof(s), 1, f) == 1) scns.push_back(s);
  if (f) std::fclose(f);
  return scns;
}

bool check(const char* path, Kernel kern) {
  const std::vector<aeb_scenario> scns = load(path);
  if (scns.empty()) return false;
  std::vector<Out> all;
  for (const aeb_scenario& x : scns) all.emplace_back(x.n_samples);
  bool ended = launch<true>(scns, all, kern);
  if (g_wrong_bound) {
    long long marked = 0, lost = 0;
    for (const Out& o : all)
      for (size_t i = 0; i < o.dist.size(); ++i) {
        marked += std::isnan(o.dist[i]);
        lost += (o.status[i] & 3) == 0 && !std::isnan(o.dist[i]);
      }
    std::printf("%s: ended %d, marked %lld, lost %lld\n", path, ended, marked, lost);
    return ended && marked > 0 && lost == 0;
  }
  long long differ = 0, past = 0;
  for (size_t j = 0; j < scns.size(); ++j) {
    std::vector<Out> alone;
    alone.emplace_back(scns[j].n_samples);
    ended = launch<false>({scns[j]}, alone, kern) && ended;
    for (size_t i = 0; i < scns[j].n_samples; ++i) {
      differ += !alone[0].same(all[j], i);
      past += all[j].steps[i] > horizon_steps(scns[j]);
    }
  }
  std::printf("%s: ended %d, differ %lld, past the horizon %lld\n", path, ended, differ, past);
  return ended && differ == 0 && past == 0;
}

}  // namespace

int main(int argc, char** argv) {
  if (argc < 3) return 2;
  std::string k = argv[1];
  if (k == "shape" && argc == 9) {
    const TuneCfg t{std::atoi(argv[4]), std::atoi(argv[5]), std::atoi(argv[6]), std::atoi(argv[7])};
    const Shape sh = shape(t, std::atoll(argv[8]), t.spt,
                           tune_is_builtin(std::atoi(argv[2]), std::atoi(argv[3]), t));
    std::printf("%u\n", sh.grid * sh.block / 64);
    return 0;
  }
  if (k == "act") {
    for (int a = 2; a < argc; ++a)
      for (const aeb_scenario& s : load(argv[a]))
        std::printf("%d\n", act_bytes(s, static_cast<int64_t>(s.n_samples)) > 0);
    return 0;
  }
  g_wrong_bound = k.back() == '!';
  if (g_wrong_bound) k.pop_back();
  const Kernel kern = k == "fp64" ? FP64 : k == "fp64x2" ? FP64X2 : FP32C;
  bool ok = true;
  for (int a = 2; a < argc; ++a) ok = check(argv[a], kern) && ok;
  return ok ? 0 : 1;
}

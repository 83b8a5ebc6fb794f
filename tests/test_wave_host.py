"""The integration kernels' control flow on the CPU: their own source on 64
emulated lanes (wave64/).  A scenario's samples in a batched launch, whatever
wavefronts they share, equal its launch alone bit for bit, every launch ends,
and none runs past a block limit (a horizon, a command switch)."""
import os
import subprocess

import pytest

from paper_2604_27193_amd import workloads as W

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("wave") / "roll_check")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-ffp-contract=off",
                        "-I", os.path.join(HERE, "wave64"), "-I", os.path.join(ROOT, "include"),
                        "-I", os.path.join(ROOT, "paper_2604_27193_amd", "csrc"),
                        os.path.join(HERE, "wave64", "roll_check.cpp"), "-o", out],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return out


def limited_and_not(other=None, **over):
    """32 friction-limited samples and 32 never limited, in one wavefront; none
    long enough for split speeds.  `other`: overrides of the second scenario."""
    over.setdefault("v0", ("trunc_normal", 18.0, 1.0, 15.0, 21.0))
    a = W.single(32, seed=9, mu=("const", 0.45), **over)
    return [a, dict(a, scenario_id=1, mu=("const", 0.85), **(other or {}))]


# each pair of limits leaves both remainders of the 128 steps that two blocks take
LIMITS = {f"horizon_{h}": limited_and_not(horizon=h * 1e-3) for h in (1300, 1364, 1500, 1564)}
LIMITS.update({f"command_{t}": limited_and_not({"dead_time": t}) for t in
               (0.26, 0.34, 0.46, 0.6, 0.66, 0.75)})
LIMITS["steps"] = limited_and_not({"dt": 2e-3}, horizon=1.5)
# no lane can stop: downhill beyond what the brake holds
for _h in (1500, 1564):
    LIMITS[f"downhill_{_h}"] = limited_and_not(horizon=_h * 1e-3, grade=("const", -0.3),
                                               a_cmd=-2.0)
    LIMITS[f"downhill_{_h}"][0]["mu"] = ("const", 0.15)
LIMITS["perception"] = [dict(W.perception(n, seed=6, scenario_id=j), mu=("uniform", 0.35, 1.0),
                             v0=("trunc_normal", 18.0, 1.0, 15.0, 21.0))
                        for j, n in enumerate((40, 65, 23))]
OBSTACLES = {"none": {"obstacle": "none"}, "stationary": {}, "exit": {"impact_exit": True},
             "lead": {"obstacle": "lead", "lead_decel": ("normal", 3.0, 0.5)}}


@pytest.mark.parametrize("obstacle", sorted(OBSTACLES))
@pytest.mark.parametrize("kernel", ["fp32c", "fp64", "fp64x2"])
def test_batch_equals_alone(exe, tmp_path, kernel, obstacle):
    from paper_2604_27193_amd import binding
    if kernel == "fp64x2" and obstacle == "lead":
        pytest.skip("two samples per lane: no lead vehicle")
    files = []
    for name, scns in LIMITS.items():
        files.append(tmp_path / name)
        files[-1].write_bytes(b"".join(bytes(binding.scenario(dict(d, **OBSTACLES[obstacle])))
                                       for d in scns))
    r = subprocess.run([exe, kernel, *map(str, files)], capture_output=True, text=True,
                       timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


# One sample per scenario, so that alone each runs in a wavefront of its own;
# actuator steps from a quarter of the time constant to beyond where the update
# diverges (parameter columns may hold any; explicit Euler's draws are refused).
def stiff(**over):
    d = dict(v0=("uniform", 0.5, 2.5), mu=("uniform", 0.3, 1.0), gap=("uniform", 0.1, 0.5),
             grade=("normal", 0.0, 0.1))
    d.update(over)
    return [W.single(1, seed=5, scenario_id=j, **d) for j in range(64)]


STIFF = {"euler": stiff(horizon=0.4, tau=("uniform", 4e-4, 4e-3)),
         "euler_diverging": stiff(horizon=0.3, tau=("uniform", 3e-4, 2e-3),
                                  v0=("uniform", 1.0, 10.0)),
         "rk4": stiff(horizon=1.5, dt=5e-3, integrator="rk4", tau=("uniform", 1.9e-3, 2e-2)),
         "rk4_diverging": stiff(horizon=1.0, dt=5e-3, integrator="rk4",
                                tau=("uniform", 1.3e-3, 3e-3), v0=("uniform", 1.0, 10.0))}


@pytest.mark.parametrize("kernel,obstacle", [("fp64", "none"), ("fp64", "exit"), ("fp64", "lead"),
                                             ("fp64x2", "none"), ("fp64x2", "stationary"),
                                             ("fp32c", "none"), ("fp32c", "stationary"),
                                             ("fp32c", "lead")])
def test_stiff_actuator(exe, tmp_path, kernel, obstacle):
    """A sample's result does not depend on its wavefront, however long its step
    is against its actuator's time constant."""
    from paper_2604_27193_amd import binding
    files = []
    for name, scns in STIFF.items():
        if name.startswith("rk4") and (kernel != "fp64" or obstacle == "lead"):
            continue
        files.append(tmp_path / name)
        files[-1].write_bytes(b"".join(bytes(binding.scenario(dict(d, **OBSTACLES[obstacle])))
                                       for d in scns))
    r = subprocess.run([exe, kernel, *map(str, files)], capture_output=True, text=True,
                       timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.parametrize("obstacle", ["none", "stationary"])
def test_broken_replay_is_visible(exe, tmp_path, obstacle):
    """Where a block's replay does not find the stop that the block showed (forced
    by job records with a wrong bound, under which the steady forms of stiff
    actuators run), the sample's distance is no number: it is not left without an
    end, nor given another block's."""
    from paper_2604_27193_amd import binding
    path = tmp_path / "diverging"
    path.write_bytes(b"".join(bytes(binding.scenario(
        W.single(64, seed=5, scenario_id=j, horizon=0.6, v0=("uniform", v, 6.0 * v),
                 mu=("uniform", 0.3, 1.0), gap=("uniform", 0.5, 20.0),
                 grade=("normal", 0.0, 0.1), tau=("uniform", 4e-4, 9e-4),
                 **OBSTACLES[obstacle]))) for j, v in enumerate((0.5, 1.0, 2.0, 5.0))))
    r = subprocess.run([exe, "fp32c!", str(path)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


# (samples, time constant, horizon, step, overrides): calls measured at least 2 %
# faster on the actuator table, and at least 2 % slower
MU = {m: {"mu": ("normal", m, 0.1)} for m in (0.6, 0.7)}
SLOW, HARD = {"v0": ("normal", 10.0, 2.0)}, {"a_cmd": -8.0}
RARE = {"proposal": {"v0": ("normal", 36.0, 2.0), "mu": ("normal", 0.55, 0.1)}}
TABLE = [(98304, 0.05, 10, 1e-3, {}), (98304, 0.15, 10, 1e-3, {}), (131072, 0.15, 10, 1e-3, {}),
         (131072, 0.15, 10, 5e-4, {}), (200000, 0.15, 10, 1e-3, {}),
         (200000, 0.15, 10, 2e-3, {}), (200000, 2.5, 10, 1e-3, {}), (350000, 0.15, 10, 1e-3, {}),
         (350000, 0.3, 10, 1e-3, {}), (350000, 0.5, 10, 1e-3, {}), (350000, 2.5, 10, 1e-3, {}),
         (1048576, 0.15, 10, 1e-3, {}), (1048576, 0.5, 30, 1e-3, {}),
         (1048576, 0.5, 30, 5e-4, {}), (1048576, 1.0, 30, 1e-3, {}),
         (1048576, 2.5, 10, 1e-3, {}), (200000, 0.15, 10, 1e-3, MU[0.7]),
         (350000, 0.15, 10, 1e-3, MU[0.7]), (1048576, 0.15, 10, 1e-3, MU[0.6]),
         (350000, 1.0, 10, 1e-3, MU[0.6]), (1048576, 1.0, 10, 1e-3, MU[0.6]),
         (1048576, 0.15, 10, 1e-3, RARE), (350000, 0.15, 10, 1e-3, SLOW),
         (1048576, 0.15, 10, 1e-3, SLOW), (1048576, 0.15, 10, 1e-3, HARD)]
PLAIN = [(98304, 0.3, 10, 1e-3, {}), (98304, 0.5, 10, 1e-3, {}), (98304, 2.5, 10, 1e-3, {}),
         (131072, 0.3, 10, 1e-3, {}), (131072, 0.5, 10, 1e-3, {}), (131072, 0.5, 30, 1e-3, {}),
         (131072, 1.0, 30, 1e-3, {}), (131072, 2.5, 10, 1e-3, {}), (200000, 0.5, 30, 1e-3, {}),
         (200000, 1.0, 30, 1e-3, {}), (350000, 0.5, 30, 5e-4, {}), (350000, 1.0, 30, 1e-3, {}),
         (350000, 2.5, 60, 1e-3, {}), (1048576, 2.5, 60, 1e-3, {}),
         (100000, 0.15, 10, 1e-3, MU[0.6]), (100000, 0.15, 10, 1e-3, MU[0.7]),
         (200000, 0.15, 10, 1e-3, MU[0.6]), (100000, 1.0, 10, 1e-3, MU[0.6]),
         (200000, 1.0, 10, 1e-3, MU[0.6]), (100000, 0.15, 10, 1e-3, RARE),
         (100000, 0.15, 10, 1e-3, SLOW), (200000, 0.15, 10, 1e-3, SLOW),
         (100000, 0.15, 10, 1e-3, HARD), (200000, 0.15, 10, 1e-3, HARD),
         (350000, 0.15, 10, 1e-3, HARD)]


def test_actuator_table_only_where_it_pays(exe, tmp_path):
    from paper_2604_27193_amd import binding
    path = tmp_path / "scenarios"
    path.write_bytes(b"".join(bytes(binding.scenario(W.paper_preset(
        n, tau=("const", tau), horizon=float(h), dt=dt, **over)))
        for n, tau, h, dt, over in TABLE + PLAIN))
    r = subprocess.run([exe, "act", str(path)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
    got = [int(x) for x in r.stdout.split()]
    want = [1] * len(TABLE) + [0] * len(PLAIN)
    assert got == want, [c for c, g, w in zip(TABLE + PLAIN, got, want) if g != w]


# precision, obstacle, k, block, waves per SIMD, samples per thread, samples ->
# wavefronts started on 1,024 SIMDs
SHAPES = [((0, 1, 128, 256, 4, 1, 1 << 20), 4096), ((0, 1, 128, 256, 4, 1, 200_000), 3072),
          ((0, 1, 128, 256, 4, 1, 100_000), 1564), ((0, 0, 64, 256, 4, 1, 160_000), 2048),
          # set or tuned: what they say, as far as there are chunks
          ((0, 1, 128, 256, 8, 1, 1 << 20), 8192), ((0, 1, 128, 256, 8, 1, 200_000), 3128),
          ((0, 1, 64, 256, 4, 1, 200_000), 3128), ((0, 2, 128, 64, 3, 1, 160_000), 2500),
          ((0, 1, 128, 256, 1, 1, 200_000), 1024), ((0, 1, 128, 256, 3, 2, 300_000), 2344),
          ((1, 1, 64, 256, 4, 1, 200_000), 3128), ((1, 1, 64, 256, 0, 1, 200_000), 3128)]


@pytest.mark.parametrize("args,waves", SHAPES)
def test_launch_shape(exe, args, waves):
    r = subprocess.run([exe, "shape", *map(str, args)], capture_output=True, text=True)
    assert r.returncode == 0 and int(r.stdout) == waves

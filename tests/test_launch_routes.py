"""Which decisions take two launches, the update and then the step without it,
and how wide the second one is (CPU: the driver in tests/c_abi/launch_routes.c
stands in for the HIP runtime's launch calls)."""
import os
import shutil
import subprocess

import pytest

import test_gpu_split as gpu
from paper_2508_01744_amd import _build, make_config

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
RULES = dict(prune_rule=15, heuristics=gpu.RULES)
REFINE = dict(prune_rule=1, refine=dict(refine_period=50, refine_stride=10, refine_half=10, refine_mature=100, refine_min_n=4))

pytestmark = pytest.mark.skipif(shutil.which("gcc") is None, reason="gcc not found")


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    """routes([(B, K, d, options, decisions before, dump)]): per entry the
    (threads per workgroup, workgroups) of each launch of that decision."""
    assert os.path.exists(_build.LIB), "run __graft_entry__.build()"
    exe = str(tmp_path_factory.mktemp("routes") / "launch_routes")
    subprocess.run(["gcc", "-std=c11", "-O1", "-Wall", "-rdynamic", "-D__HIP_PLATFORM_AMD__", "-I", _build.INCLUDE,
                    "-I", os.path.join(ROCM, "include"), os.path.join(HERE, "c_abi", "launch_routes.c"), _build.LIB,
                    "-L", os.path.join(ROCM, "lib"), "-lamdhip64", "-Wl,-rpath," + os.path.dirname(_build.LIB),
                    "-Wl,-rpath," + os.path.join(ROCM, "lib"), "-o", exe], check=True)

    def run(entries):
        lines = [f"{bytes(make_config(B, K, d, **opts)).hex()} {t} {int(dump)}\n" for B, K, d, opts, t, dump in entries]
        out = subprocess.run([exe], input="".join(lines), capture_output=True, text=True, timeout=120, check=True).stdout
        got = [[tuple(int(v) for v in launch.split("x")) for launch in line.split()] for line in out.splitlines()]
        assert len(got) == len(entries)
        return got

    return run


def test_gpu_cases_take_two_launches(routes):
    """Every case of the GPU comparison splits in its large batch, at its plain
    steps and, by the dump's own rule, at those with the dump; never in its small
    one, nor without a reward to fold in."""
    entries, want = [], []
    for B, K, d, name in gpu.CASES:
        opts = dict(alpha0=0.5, **gpu.OPTIONS[name])
        for n, t, dump in ((B, 15, False), (B, 17, True), (B, 0, False), (gpu.FEW, 15, False), (gpu.FEW, 17, True)):
            entries.append((n, K, d, opts, t, dump))
            want.append(2 if n == B and t and gpu._split(B, K, d, opts, dump) else 1)
    assert len(gpu.CASES) >= 36
    for entry, launches, n in zip(entries, routes(entries), want):
        assert len(launches) == n, entry
        assert launches[-1][1] == entry[0]   # the step: one workgroup per instance


@pytest.mark.parametrize("d,K,opts,dump,least", [
    (16, 128, dict(prune_rule=1), False, 8192), (16, 54, {}, False, 8192),      # instances bind: 256 MB are less
    (16, 53, {}, False, 8331), (16, 27, {}, False, 16353),                      # 256 MB bind
    (32, 96, dict(prune_rule=1), False, 16384), (32, 7, {}, False, 17120),
    (8, 128, dict(prune_rule=1), False, 23832), (8, 186, dict(prune_rule=1), False, 16401),   # d = 8, one wavefront: 512 MB
    (8, 187, dict(prune_rule=1), False, 65250), (8, 256, dict(prune_rule=1), False, 47663),   # four: 2 GB
    (8, 139, {}, False, 21946), (8, 140, {}, False, 43578), (8, 256, {}, False, 23832),   # no arm goes: 1 GB from 24 KB on
    (8, 256, RULES, False, 11916), (8, 600, RULES, False, 20337),               # the rules' own limit of widths
    (8, 256, dict(prune_rule=1), True, 11916),                                  # with the dump: 512 MB
    (16, 128, REFINE, False, 21025), (16, 128, REFINE, True, None),             # and none up to 16 KB
])
def test_smallest_batch_of_two_launches(routes, d, K, opts, dump, least):
    if least is None:
        assert len(routes([(1 << 20, K, d, opts, 2, dump)])[0]) == 1
        return
    below, at = routes([(least - 1, K, d, opts, 2, dump), (least, K, d, opts, 2, dump)])
    assert (len(below), len(at)) == (1, 2)


def test_width_of_the_second_launch(routes):
    """One wavefront up to 32 KB of records per instance, 96 KB with rules 2-8,
    four beyond; by the theta copy's bytes once instances may exploit."""
    ph = dict(prune_rule=1, exploit=dict(ph_delta=0.05, ph_lambda=2.0, ph_window=8, ph_min_rounds=10))
    entries = [(1 << 17, K, d, o, t, False) for d, K, o, t in (
        (16, 53, {}, 2), (16, 54, {}, 2), (16, 161, RULES, 2), (16, 162, RULES, 2), (32, 14, {}, 2), (32, 15, {}, 2),
        (16, 128, ph, 9), (16, 128, ph, 10))]
    assert [(len(r), r[-1][0]) for r in routes(entries)] == [(2, w) for w in (64, 256, 64, 256, 64, 256, 256, 64)]

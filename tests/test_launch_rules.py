"""The launch rules (csrc/launch_rules.hpp) on the CPU: compiled into a small host
program and asked which workgroup shape a call takes."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NAMES = {(4, 1): "narrow", (8, 1): "wide", (4, 2): "half", (2, 4): "quarter", (1, 8): "eighth"}

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ is not installed")


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    """rules(lines) -> the shape's name (k lines: a bool) per line of launch_rules.cpp's input."""
    exe = tmp_path_factory.mktemp("rules") / "launch_rules"
    res = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror",
                          os.path.join(ROOT, "tests", "launch_rules.cpp"), "-o", str(exe)],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr

    def ask(lines):
        run = subprocess.run([str(exe)], input="\n".join(lines), capture_output=True, text=True, timeout=60)
        assert run.returncode == 0
        got = [NAMES[tuple(map(int, l.split()))] if " " in l else l == "1" for l in run.stdout.splitlines()]
        assert len(got) == len(lines)
        return got
    return ask


def _line(d, N, bh, causal=False, fp8=False, bf16=False):
    return f"b {d} {N} {bh}" if bf16 else f"f {d} {N} {bh} {int(causal)} {int(fp8)}"


def _grid():
    for d in (64, 128):
        for N in (128, 256, 384, 512, 640, 768, 1024, 1152, 1664, 2048, 2176, 3968, 4096, 8192, 14080, 32768):
            for bh in (*range(1, 70), 96, 128, 192, 257, 384, 512, 768, 1290, 3072, 6144):
                yield d, N, bh


def test_shapes_divide_the_rows(rules):
    """Every launch covers N exactly: 256-query workgroups only where 256 divides N, and
    no shape that does not exist (FP8 P/V at d = 128 has no eight-way split)."""
    points = [(d, N, bh, dict(causal=c, fp8=f)) for d, N, bh in _grid() for c in (False, True) for f in (False, True)]
    points += [(d, N, bh, dict(bf16=True)) for d, N, bh in _grid()]
    for (d, N, bh, o), name in zip(points, rules([_line(d, N, bh, **o) for d, N, bh, o in points])):
        assert name != "wide" or N % 256 == 0, (d, N, bh, o)
        assert name != "eighth" or not (o.get("bf16") or (o.get("fp8") and d == 128)), (d, N, bh, o)
        assert name != "quarter" or not o.get("bf16"), (d, N, bh, o)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("fp8", [False, True])
def test_kernels_built_are_the_kernels_launched(rules, d, causal, fp8):
    """A kernel is built for exactly the shapes that the rule returns for some grid."""
    launched = set(rules([_line(dd, N, bh, causal, fp8) for dd, N, bh in _grid() if dd == d]))
    built = rules([f"k {d} {int(causal)} {int(fp8)} {qg} {ks}" for qg, ks in NAMES])
    assert launched == {name for name, b in zip(NAMES.values(), built) if b}


def _check(rules, points):
    """points: (d, N, workgroups of 128 queries, options, the shape measured fastest)"""
    got = rules([_line(d, N, U * 128 // N, **o) for d, N, U, o, _ in points])
    for (d, N, U, o, want), name in zip(points, got):
        assert name == want, (d, N, U, o, name)


def test_fp8_short_rows(rules):
    """FP8 P/V at d = 128, rows under 1024: a second round is not worth a key split (it
    took 8 to 17 % longer than the unsplit launch); long rows keep it."""
    _check(rules, [(128, 256, 576, dict(fp8=True), "wide"), (128, 256, 768, dict(fp8=True), "wide"),
                   (128, 512, 704, dict(fp8=True), "wide"), (128, 768, 702, dict(fp8=True), "wide"),
                   (128, 1024, 704, dict(fp8=True), "half"), (128, 4096, 768, dict(fp8=True), "half"),
                   (128, 256, 512, dict(fp8=True, causal=True), "wide"), (128, 512, 512, dict(fp8=True, causal=True), "wide"),
                   (128, 512, 288, dict(fp8=True, causal=True), "half"), (128, 4096, 512, dict(fp8=True, causal=True), "half"),
                   (128, 384, 513, dict(fp8=True), "half")])


def test_causal_short_rows(rules):
    """Causal rows under 512 keys: the merge of a split costs more than the steps it saves
    (it took 7 to 9 % longer at N 128); from 512 on few workgroups split."""
    narrow = [(d, N, U, dict(causal=True, fp8=f), "narrow") for d, N, U, f in
              ((128, 128, 2, False), (128, 128, 16, False), (128, 256, 32, False), (128, 384, 48, False),
               (64, 128, 32, False), (64, 256, 64, False), (64, 384, 96, False), (64, 128, 16, True), (64, 256, 32, True))]
    _check(rules, narrow + [(64, 1664, 416, dict(causal=True), "half"), (128, 4096, 512, dict(causal=True), "half"),
                            (64, 4096, 512, dict(causal=True, fp8=True), "half")])


ROUTES = {"plain": dict(), "causal": dict(causal=True), "fp8": dict(fp8=True), "causal fp8": dict(causal=True, fp8=True),
          "bf16": dict(bf16=True)}
# Keys from which a kernel's main loop runs, whatever its ring: 10 unsplit steps of 64 (BF16:
# of 32), 6 tiles (BF16: of 64) in two key groups, 9 stages of 2 tiles, 6 stages of 4 tiles.
MAIN_LOOP = {"narrow": 640, "wide": 640, "half": 768, "quarter": 2304, "eighth": 3072}
MAIN_LOOP_BF16 = {"narrow": 320, "wide": 320, "half": 384}


@pytest.mark.parametrize("route", ROUTES)
@pytest.mark.parametrize("d", [64, 128])
def test_gpu_tables_reach_every_kernel(rules, route, d):
    """The shapes of the GPU sweeps (tests/test_gpu_shape_sweep.py, test_gpu_bf16.py) launch
    every workgroup shape that the rules can launch on this route, each with its main loop,
    so that a later rule cannot take a kernel out of the tests."""
    from test_gpu_bf16 import BOUNDARY_SHAPES
    from test_gpu_shape_sweep import SHAPES, SPLIT_SHAPES
    opts = ROUTES[route]
    grid = [(N, bh) for dd, N, bh in _grid() if dd == d]
    reachable = {}
    for (N, bh), name in zip(grid, rules([_line(d, N, bh, **opts) for N, bh in grid])):
        reachable[name] = max(N, reachable.get(name, 0))
    table = [(N, B * H) for B, H, N, dd in (BOUNDARY_SHAPES if route == "bf16" else SHAPES + SPLIT_SHAPES) if dd == d]
    tested = {}
    for (N, bh), name in zip(table, rules([_line(d, N, bh, **opts) for N, bh in table])):
        tested[name] = max(N, tested.get(name, 0))
    assert set(tested) == set(reachable)
    loop = MAIN_LOOP_BF16 if route == "bf16" else MAIN_LOOP
    for name, longest in reachable.items():
        assert tested[name] >= min(loop[name], longest), (name, tested[name])


@pytest.mark.parametrize("d", [64, 128])
def test_gpu_grids_reach_every_kernel(rules, d):
    """The grids of the GPU test that runs every exponential density (which the guarded
    and causal routes have too) take all five workgroup shapes."""
    from test_gpu_shape_sweep import GRIDS
    N, grids = GRIDS[d]
    for opts in (dict(), dict(causal=True)):
        assert set(rules([_line(d, N, bh, **opts) for bh in grids])) == set(NAMES.values())

"""The host planner's choices at the benchmarked shapes (no GPU): the planner
source is compiled with its kernel launchers stubbed out (tests/planner) and
asked for the plan of each descriptor. These pin the execution paths that the
measurements in the design notes were taken on, and check that every plan
fits one compute unit's LDS and the chip's resident workgroup slots."""
import json
import random
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_10805_amd", "csrc")
LDS_FLOATS = 160 * 1024 // 4


def lds_wgs(floats):
    """Workgroups per CU an LDS size allows: 128 granules of 1280 bytes per CU
    (measured on MI355X: three workgroups of 53760 bytes fit, of 53888 two)."""
    return 128 // -(-floats // 320)


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("needs g++")
    exe = str(tmp_path_factory.mktemp("planner") / "plan_dump")
    subprocess.run([gxx, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-x", "c++",
                    os.path.join(ROOT, "tests", "planner", "plan_dump.cpp"), "-o", exe,
                    "-L", "/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib"], check=True,
                   capture_output=True)

    def plan(B, C, H, W, k, L, dtype=0):
        out = subprocess.run([exe], input=f"{B} {C} {H} {W} {k} {L} {dtype}\n", capture_output=True, text=True,
                             check=True, timeout=60).stdout
        return json.loads(out.strip().splitlines()[-1])
    return plan


def test_headline_workload_plan(planner):
    """B64 C96 56x56 k5 L3 fp32: the forward holds one plane per workgroup in
    one round of 4x4 tiles, levels >= 3 sharing level 1's round; the backward
    is the gradient pass (one resident plane, one block round) plus dx by the
    forward with rotated taps; no workspace for the forward."""
    p = planner(64, 96, 56, 56, 5, 3)
    assert p["fwd_mode"] == "resident" and p["fwd_PP"] == 1 and p["fwd_one_round"] == 1
    assert p["fwd_merge_deep"] == 1
    # 14 output tiles per row, laid out over 16 lanes (one round, four wavefronts either way)
    assert p["fwd_tiles_x"] == 14 and p["fwd_tiles_xl"] == 16
    assert p["fwd_ws"] == 0
    assert p["grad_pass"] == 1 and p["grad_levels"] == 3 and p["grad_coarse"] == 0
    assert p["grad_PP"] == 1 and p["grad_rounds"] == 1
    # four workgroups per CU fit in LDS
    assert lds_wgs(p["fwd_lds_floats"]) >= 4


@pytest.mark.parametrize("C,H,L,fwd_mode", [(96, 56, 5, "resident"), (192, 28, 4, "resident"),
                                            (192, 28, 5, "split"), (384, 14, 3, "resident"),
                                            (384, 14, 4, "split"), (768, 7, 3, "tiny")])
def test_convnext_stage_modes(planner, C, H, L, fwd_mode):
    p = planner(128, C, H, H, 5, L)
    assert p["fwd_mode"] == fwd_mode


def test_tile_row_padding_keeps_the_busy_wavefronts(planner):
    """Padding tile rows to 8 lanes is skipped where it would put work on more
    wavefronts: 12 x 12 planes have 3 tiles per row (at L = 4, 16 planes: 144
    tiles on three wavefronts; padded, more)."""
    p = planner(128, 192, 12, 12, 5, 4)
    assert p["fwd_mx_rounds"] == 0 and p["fwd_one_round"] == 1
    assert p["fwd_tiles_xl"] == p["fwd_tiles_x"] == 3
    p = planner(64, 192, 28, 28, 5, 1)
    assert p["fwd_tiles_xl"] == 8


def test_small_planes_take_mixed_rounds(planner):
    """Planes of at most 16 x 16 run the forward with mixed task rounds: at
    14 x 14 L = 1, eight planes' 128 output tiles and 128 level-1 tiles fill
    one round of 256 lanes; the split 14 x 14 L = 4 forward's level-1 pass is
    the same plan. Larger planes keep the fused kernel."""
    p = planner(128, 384, 14, 14, 5, 1)
    assert p["fwd_mode"] == "resident" and p["fwd_mx_rounds"] == 1 and p["fwd_PP"] == 8
    assert sorted(map(tuple, p["fwd_mx_seg"][0])) == [(1, 0, 0, 128)] + [(2, 1, q, 32) for q in range(4)]
    p = planner(128, 384, 14, 14, 5, 4)
    assert p["fwd_mode"] == "split" and p["fwd_mx_rounds"] == 1
    for H, L in [(56, 3), (28, 3), (20, 3)]:
        assert planner(64, 96, H, H, 5, L)["fwd_mx_rounds"] == 0


def test_gradient_pass_level1_tiles_and_shed(planner):
    """The gradient pass takes level 1 in 2 x 2 site tiles where the smaller
    footprint fits three workgroups per CU (B64 C192 28 x 28 L1: four planes
    in 13440 floats instead of five in 16800), not where it would trade
    workgroups for planes (B128 C384 12 x 12 L2 keeps ten planes at three per
    CU). A single level above m = 2 goes to the coarse sub-problem from
    18432 planes on (28 x 28 L3: B128 C192 yes, B64 C192 no)."""
    p = planner(64, 192, 28, 28, 5, 1)
    assert p["grad_PP"] == 4 and lds_wgs(p["grad_lds_floats"]) == 3
    p = planner(128, 384, 12, 12, 5, 2)
    assert p["grad_PP"] == 10 and lds_wgs(p["grad_lds_floats"]) == 3
    p = planner(128, 192, 28, 28, 5, 3)
    assert p["grad_levels"] == 2 and p["grad_coarse"] == 1
    p = planner(64, 192, 28, 28, 5, 3)
    assert p["grad_levels"] == 3 and p["grad_coarse"] == 0


@pytest.fixture(scope="module")
def mixed_check(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("needs g++")
    exe = str(tmp_path_factory.mktemp("mixed") / "mixed_check")
    subprocess.run([gxx, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-x", "c++",
                    os.path.join(ROOT, "tests", "planner", "mixed_check.cpp"), "-o", exe,
                    "-L", "/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib"], check=True,
                   capture_output=True)
    return exe


def test_mixed_round_plans_hold_their_invariants(mixed_check):
    """Every mixed-round plan over 3000 seeded random small-plane problems
    (and the ConvNeXt-T 14 x 14 stage) keeps what the kernel relies on: whole
    (level, band) groups per round before the output rounds, every tile and
    group covered once, at most 256 tasks a round, every window and write-back
    inside its array and the LDS (tests/planner/mixed_check.cpp)."""
    rng = random.Random(7)
    lines = [f"{rng.randint(1, 140)} {rng.randint(1, 400)} {rng.randint(9, 16)} {rng.randint(9, 16)} "
             f"{rng.choice([1, 3, 5, 7, 9])} {rng.randint(1, 8)} {rng.randint(0, 2)}" for _ in range(3000)]
    lines += [f"128 384 14 14 {k} {L} 0" for k in (3, 5, 7, 9) for L in range(1, 6)]
    out = subprocess.run([mixed_check], input="\n".join(lines) + "\n", capture_output=True, text=True,
                         check=True, timeout=120).stdout.split("\n")[:len(lines)]
    fails = [(l, o) for l, o in zip(lines, out) if not (o.startswith("ok") or o == "fused")]
    assert not fails, fails[:5]
    assert sum(o.startswith("ok") for o in out) > 1000


@pytest.fixture(scope="module")
def phase_check(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("needs g++")
    exe = str(tmp_path_factory.mktemp("phase") / "phase_check")
    subprocess.run([gxx, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-x", "c++",
                    os.path.join(ROOT, "tests", "planner", "phase_check.cpp"), "-o", exe,
                    "-L", "/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib"], check=True,
                   capture_output=True)
    return exe


def test_polyphase_plans_hold_their_invariants(phase_check):
    """Every polyphase plan (whole plane, regions, kernel gradients) over 3000
    seeded random problems stays inside its arrays and the LDS and covers the
    plane and the batch (tests/planner/phase_check.cpp)."""
    rng = random.Random(11)
    size = lambda hi: int(round(2 ** rng.uniform(2, hi)))  # noqa: E731
    lines = [f"{size(8.5) - 3} {size(10) - 3} {size(8.5) - 3} {size(8.5)} {rng.choice([3, 5])} {rng.randint(1, 5)} "
             f"{rng.randint(0, 2)}" for _ in range(3000)]
    lines += [f"{B} {C} {n} {n} {k} {L} {t}" for B, C, n in ((64, 96, 56), (128, 384, 14), (70000, 1, 8), (16, 64, 224))
              for k in (3, 5) for L in range(1, 6) for t in range(3)]
    out = subprocess.run([phase_check], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True,
                         timeout=120).stdout.split("\n")[:len(lines)]
    fails = [(l, o) for l, o in zip(lines, out) if not o.startswith("ok")]
    assert not fails, fails[:5]
    assert all(sum(o.split()[i] == "1" for o in out) > 800 for i in (1, 2, 3))


@pytest.fixture(scope="module")
def phase_routes(tmp_path_factory):
    """(B, C, H, W, k, L, dtype) tuples -> [(forward route, PP, batches, last,
    gradient route, PP, batches, last)], see tests/planner/phase_routes.cpp."""
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("needs g++")
    exe = str(tmp_path_factory.mktemp("routes") / "phase_routes")
    subprocess.run([gxx, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-x", "c++",
                    os.path.join(ROOT, "tests", "planner", "phase_routes.cpp"), "-o", exe,
                    "-L", "/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib"], check=True,
                   capture_output=True)

    def run(specs):
        lines = [" ".join(map(str, (*s[:6], ("f32", "bf16", "f16").index(s[6])))) for s in specs]
        out = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True,
                             timeout=60).stdout.strip().split("\n")
        return [tuple(map(int, line.split())) for line in out]

    return run


def test_gpu_tests_of_the_polyphase_kernels_reach_them(phase_routes):
    """The problems that tests/test_gpu_phase.py lists for their plans have them."""
    pytest.importorskip("torch")
    from tests import test_gpu_phase as gpu

    for (spec, fwd, grad), r in zip(gpu.GROUPS, phase_routes([g[0] for g in gpu.GROUPS])):
        assert r[:4] == (1, *fwd), (spec, r)
        assert r[4:] == ((1, *grad) if grad else (0, 0, 0, 0)), (spec, r)
    assert all(r[0] == (2 if s[2] > 100 else 1) for s, r in zip(gpu.STAGES, phase_routes(gpu.STAGES)))
    assert all(r[0] == 2 for r in phase_routes(gpu.REGIONS))
    # every stage count, kernel size and type somewhere, in the forward and the gradients
    reached = {(s[4], s[5], s[6]) for s, f, g in gpu.GROUPS}
    assert {(k, L) for k, L, t in reached if t != "f32"} == {(k, L) for k in (3, 5) for L in range(1, 6)}
    assert {(k, L) for k, L, t in reached if t == "f32"} == {(k, L) for k in (3, 5) for L in range(1, 4)}


# on both sides of every line of the gradient rule; the times are at the rule
@pytest.mark.parametrize("spec,phase", [
    ((64, 768, 7, 7, 5, 1, "bf16"), 0), ((128, 768, 7, 7, 5, 1, "bf16"), 1), ((32, 768, 7, 7, 3, 1, "f16"), 1),
    ((64, 768, 8, 8, 5, 1, "f16"), 1), ((64, 384, 10, 10, 5, 5, "bf16"), 0), ((32, 384, 14, 14, 5, 5, "bf16"), 1),
    ((128, 384, 14, 14, 3, 5, "f16"), 1), ((16, 96, 56, 56, 5, 4, "bf16"), 0), ((32, 96, 64, 64, 5, 4, "bf16"), 1),
    ((16, 64, 48, 48, 5, 5, "f16"), 1), ((64, 96, 56, 56, 5, 3, "f32"), 0)])
def test_where_the_gradient_pass_is_polyphase(phase_routes, spec, phase):
    assert phase_routes([spec])[0][4] == phase


# on both sides of every line of the forward rule; the times are at the rule
@pytest.mark.parametrize("spec,route", [
    ((8, 64, 116, 116, 5, 2, "f32"), 2), ((8, 64, 128, 128, 3, 3, "f32"), 2), ((8, 64, 134, 134, 5, 2, "f32"), 0),
    ((8, 64, 169, 169, 5, 3, "f32"), 2), ((8, 64, 170, 170, 3, 2, "f32"), 2), ((8, 64, 116, 170, 5, 2, "f32"), 2),
    ((8, 64, 60, 170, 5, 3, "f32"), 2), ((16, 64, 224, 224, 5, 3, "f32"), 0), ((16, 64, 100, 100, 5, 2, "f32"), 0),
    ((16, 96, 72, 72, 5, 4, "f32"), 0), ((16, 64, 224, 224, 5, 3, "bf16"), 2),
    ((18, 136, 69, 102, 5, 3, "f32"), 0), ((1, 64, 169, 169, 3, 2, "f32"), 0), ((2, 64, 128, 128, 3, 2, "f32"), 2),
    ((128, 144, 119, 119, 3, 3, "f32"), 2), ((8, 512, 171, 171, 3, 2, "f32"), 0), ((16, 768, 266, 68, 5, 2, "f32"), 2),
    ((8, 256, 171, 171, 5, 2, "f32"), 2), ((8, 768, 113, 113, 5, 3, "f32"), 2),
    ((12, 768, 164, 164, 5, 1, "bf16"), 0), ((4, 768, 164, 164, 5, 1, "bf16"), 2), ((12, 768, 171, 171, 3, 1, "f16"), 2),
    # float32, L = 1
    ((8, 512, 63, 63, 5, 1, "f32"), 1), ((100, 256, 13, 13, 5, 1, "f32"), 1), ((64, 256, 16, 16, 5, 1, "f32"), 0),
    ((48, 435, 99, 99, 3, 1, "f32"), 2), ((16, 96, 111, 155, 5, 1, "f32"), 0),
    ((1, 144, 224, 224, 5, 1, "f32"), 0), ((4, 144, 224, 224, 5, 1, "f32"), 2), ((1, 144, 148, 148, 5, 1, "f32"), 0),
    ((1, 144, 148, 148, 3, 1, "f32"), 2), ((26, 40, 168, 168, 3, 1, "f32"), 0), ((4, 64, 80, 120, 5, 1, "f32"), 2),
    ((16, 64, 64, 64, 5, 1, "f32"), 0), ((64, 96, 64, 64, 5, 1, "f32"), 1), ((16, 64, 56, 56, 3, 1, "f32"), 0),
    ((64, 96, 16, 16, 5, 1, "f32"), 0), ((64, 192, 12, 16, 5, 1, "f32"), 1), ((128, 435, 14, 12, 5, 1, "f32"), 1),
    # few batches
    ((8, 64, 56, 56, 5, 1, "f16"), 1), ((4, 96, 64, 64, 5, 3, "f16"), 0), ((16, 96, 64, 64, 5, 3, "f16"), 1),
    ((16, 64, 56, 56, 5, 5, "bf16"), 0), ((48, 64, 56, 56, 5, 5, "bf16"), 1), ((1, 64, 56, 56, 5, 3, "bf16"), 1),
    ((16, 64, 48, 48, 5, 3, "f32"), 0), ((24, 64, 48, 48, 5, 3, "f32"), 1), ((2, 16, 32, 32, 5, 1, "f32"), 1),
    # fewer planes per CU than the vector plan
    ((32, 96, 72, 72, 5, 2, "f32"), 1), ((32, 96, 72, 72, 5, 3, "f32"), 0), ((32, 96, 72, 72, 3, 2, "f32"), 0),
    ((32, 96, 64, 64, 3, 2, "f32"), 1), ((32, 96, 64, 64, 3, 3, "f32"), 0), ((32, 128, 50, 70, 3, 3, "f32"), 0),
    # float32, k = 5, L = 2 and 3
    ((64, 96, 56, 56, 5, 3, "f32"), 0), ((64, 96, 48, 48, 5, 3, "f32"), 1), ((32, 128, 55, 57, 5, 3, "f32"), 1),
    ((64, 96, 60, 60, 5, 2, "f32"), 1), ((64, 192, 28, 28, 5, 3, "f32"), 0), ((32, 128, 63, 95, 5, 3, "f32"), 1),
    ((64, 256, 20, 20, 5, 2, "f32"), 1), ((64, 256, 20, 20, 5, 3, "f32"), 0),
    ((128, 384, 14, 14, 5, 2, "f32"), 1), ((128, 435, 14, 12, 5, 2, "f32"), 0), ((200, 512, 17, 17, 5, 2, "f32"), 1),
    ((100, 64, 65, 65, 5, 2, "f32"), 1), ((48, 435, 65, 65, 3, 2, "f32"), 0),
    ((24, 96, 30, 25, 5, 3, "f32"), 0), ((100, 48, 30, 30, 5, 3, "f32"), 1),
    ((64, 96, 14, 14, 5, 2, "f32"), 0), ((64, 256, 14, 14, 5, 2, "f32"), 1), ((64, 256, 14, 14, 3, 2, "f32"), 0),
    # float32, k = 3
    ((64, 192, 28, 28, 3, 3, "f32"), 1), ((64, 192, 32, 32, 3, 2, "f32"), 0), ((32, 128, 35, 90, 3, 2, "f32"), 0),
    ((64, 128, 40, 40, 3, 2, "f32"), 1), ((32, 128, 55, 57, 3, 3, "f32"), 1), ((32, 128, 63, 95, 3, 3, "f32"), 0)])
def test_where_the_forward_is_polyphase(phase_routes, spec, route):
    assert phase_routes([spec])[0][0] == route


def test_odd_shape_block_rounds(planner):
    """63 x 95 planes have 384 4x4 blocks: the gradient pass takes them in
    two rounds over one resident plane."""
    p = planner(32, 128, 63, 95, 5, 3)
    assert p["grad_pass"] == 1 and p["grad_PP"] == 1 and p["grad_rounds"] == 2


def test_large_planes_take_the_region_path(planner):
    """Planes larger than one CU's LDS run in region tiles; their backward is
    the gradient pass over the tiles plus the rotated forward for dx (64 x 64
    regions: 56 x 56 tiles at k = 3, 5, 48 x 48 at k = 7, 9), and the fused
    region backward when there is no level (L = 0)."""
    p = planner(16, 64, 224, 224, 5, 3)
    assert p["fwd_mode"] == "region" and p["fwd_ws"] > 0 and p["bwd_ws"] > 0
    assert p["bwd_mode"] == "region" and p["bwd_region_grad"] == 1
    assert planner(8, 32, 512, 512, 3, 3)["bwd_region_grad"] == 1
    assert planner(8, 128, 128, 128, 5, 1)["bwd_region_grad"] == 1
    assert planner(1, 1, 300, 300, 7, 4)["bwd_region_grad"] == 1
    assert planner(1, 2, 130, 126, 9, 3)["bwd_region_grad"] == 1
    assert planner(1, 2, 130, 126, 5, 0)["bwd_region_grad"] == 0  # no level: the fused region backward


def test_lds_granule_model():
    assert lds_wgs(53760 // 4) == 3 and lds_wgs(53888 // 4) == 2 and lds_wgs(81920 // 4) == 2
    assert lds_wgs(40960 // 4) == 4 and lds_wgs(9656) == 4


@pytest.mark.parametrize("B,C,H,W,k,L", [(64, 96, 56, 56, 5, 3), (128, 192, 28, 28, 5, 2), (128, 384, 14, 14, 5, 1),
                                         (32, 128, 63, 95, 5, 5), (8, 64, 100, 100, 3, 2), (64, 96, 40, 40, 7, 4)])
def test_plans_fit_the_chip(planner, B, C, H, W, k, L):
    """Every resident plan fits one CU's LDS, and the gradient pass is one
    round of resident workgroups (at most three per CU on 256 CUs)."""
    p = planner(B, C, H, W, k, L)
    if p["fwd_mode"] in ("resident", "split"):
        assert 0 < p["fwd_lds_floats"] <= LDS_FLOATS
        assert p["fwd_nb"] % p["fwd_PP"] == 0
    if p["grad_pass"]:
        assert 0 < p["grad_lds_floats"] <= LDS_FLOATS
        wgs = min(3, lds_wgs(p["grad_lds_floats"]))
        assert p["grad_nchunks"] * C <= max(256 * wgs, C)

"""Arithmetic that the kernels and launchers share with the host, run on the CPU in small C++ programs."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2511_02647_amd", "csrc")


def run(tmp_path, name, stdin=""):
    exe = str(tmp_path / name)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I" + CSRC, "-o", exe, os.path.join(ROOT, "tests", "host", name + ".cpp")])
    p = subprocess.run([exe], input=stdin, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=60)
    assert p.returncode == 0, p.stdout
    return p.stdout


def test_routes_of_calls(tmp_path):
    """Which launches calls take, and what they hand them: workspaces, lists of tiles (tests/host/routes.cpp)."""
    hipcc = "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    exe = str(tmp_path / "routes")
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-w", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                           "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-o", exe, os.path.join(CSRC, "api.hip"),
                           "-x", "hip", os.path.join(ROOT, "tests", "host", "routes.cpp")])
    p = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=60)
    assert p.returncode == 0 and "clean" in p.stdout, p.stdout


def test_halves_of_a_listed_tile_stay_inside_it(tmp_path):
    assert "clean" in run(tmp_path, "half_tile")


def test_the_layouts_of_the_gpu_tests_take_the_launches_they_name(tmp_path):
    """On the 256 CUs of the device the tests run on; every launch at every padded head dimension that has it is among them."""
    import test_gpu_general_shapes as g
    want, shapes = [], []

    def add(what, dtype, D, Hq, Hkv, causal, sync, lens):
        want.append(what)
        shapes.append("%s %d %d %d %d %d 0 256 %s" % (dtype, D, Hq, Hkv, causal, sync, " ".join(map(str, lens))))

    for launch, sync, causal, lens, Hq, Hkv, dims in g.LAUNCHES:
        for D in dims:
            add(launch, "bf16", D, Hq, Hkv, causal, sync, lens)
    for name, (lens, Hq, Hkv) in g.PLAN_LAYOUTS.items():
        for D in (64, 128):
            add({"eight-short": "eight", "split-long": "split"}.get(name, name), "bf16", D, Hq, Hkv, 1, 1, lens)
    for D in (8, 40, 72, 96, 120, 160, 256):
        for sync in (0, 1):
            for name in ("short", "long"):
                add("split" if D <= 128 else "four-ordered", "bf16", D, *g.BF16_LAYOUTS[name][1:], 1, sync, g.BF16_LAYOUTS[name][0])
            add("four", "bf16", D, *g.BF16_LAYOUTS["four"][1:], 1, sync, g.BF16_LAYOUTS["four"][0])
    for D in (8, 40, 64, 88, 128, 136, 256):
        for name, (lens, Hq, Hkv) in g.LAYOUTS.items():
            add("shared" if name == "shared" else "keys", "f32", D, Hq, Hkv, 1, 1, lens)
    for layout, name, sync in (("eight", "eight", 1), ("eight-pairs", "eight-pairs", 1), ("local-pairs", "eight-pairs", 0)):
        lens, Hq, Hkv = g.HIDDEN_LAYOUTS[layout]
        add(name, "bf16", 72, Hq, Hkv, 1, sync, lens)
    got = run(tmp_path, "launch_choice", "\n".join(shapes)).split()
    assert len(got) == len(want)
    assert not [(s, w, x) for s, w, x in zip(shapes, want, got) if w != x]
    padded = lambda D: D if D in (64, 128) else -(-D // 32) * 32 + 1000    # 1000: weights at full precision
    reached = {(launch, padded(D)) for launch, _, _, _, _, _, dims in g.LAUNCHES for D in dims}
    assert reached >= {(l, d) for l in ("four", "eight", "eight-pairs", "split") for d in (64, 128, 1032, 1064, 1096, 1128)}
    assert reached >= {("four-ordered", d) for d in (64, 128, 1032, 1064, 1096, 1128, 1160, 1192, 1224, 1256)}
    assert reached >= {("four", d) for d in (1160, 1192, 1224, 1256)}


def test_chunk_length_of_wide_sync_blocks_is_that_of_the_full_search(tmp_path):
    assert "clean" in run(tmp_path, "wide_chunks")


def test_pairs_are_taken_in_one_round_of_workgroups_only(tmp_path):
    """At 256 and 272 pairs, with and without a keep-list, local and sync; the GPU test of pairs has layouts that take them."""
    import test_gpu_general_shapes as g
    shapes = ["128 32 8 1 1 %d 256 %s" % (keep, " ".join(["512"] * 4 if one else ["516"] * 4)) for keep in (0, 1) for one in (1, 0)]
    shapes += ["128 16 8 1 0 0 256 1019 1019 1019 1019", "128 16 2 1 0 0 256 2239 2239"]
    for lens, Hq, Hkv in g.PAIRS.values():
        shapes += ["%d %d %d 1 1 %d 256 %s" % (D, Hq, Hkv, keep, " ".join(map(str, lens))) for D in g.PAIRS_DIMS for keep in (0, 1)]
    got = [l.split() for l in run(tmp_path, "launch_taken", "\n".join(shapes)).splitlines()]
    assert [taken == "eight-pairs" for _, taken, _ in got[:6]] == [True, False, True, False, True, False]
    assert all(choice == "eight-pairs" for choice, _, _ in got[:6])
    assert all(taken == "eight-pairs" for _, taken, _ in got[6:])


def test_dense_layouts_apart_are_read_where_they_are_by_the_launches_they_name(tmp_path):
    """Every launch that the rule has read matrices apart, at both head dimensions, and one layout that is copied first."""
    import test_gpu_parity as g
    shapes = ["%d %d %d %d 1 0 256 %s" % (D, Hq, Hkv, causal, " ".join(map(str, lens))) for _, causal, lens, Hq, Hkv, D in g.APART]
    got = [l.split()[1:] for l in run(tmp_path, "launch_taken", "\n".join(shapes)).splitlines()]
    want = [["four", "copied"] if launch == "copied" else [launch, "apart"] for launch, *_ in g.APART]
    assert not [(s, w, x) for s, w, x in zip(shapes, want, got) if w != x] and len(got) == len(want)
    assert {(launch, D) for launch, _, _, _, _, D in g.APART} >= {(l, D) for l in ("four", "eight", "eight-pairs", "split") for D in (64, 128)}

"""The launch rules' choices (host code only; no GPU).

A rule picks a kernel or a tile from the sizes of a launch.  The lattices here
were timed with every choice (in the comments, microseconds on an MI355X); the
rule takes the fastest, or one within the 5% that separates a choice from
noise.  tests/launch_rules/rules.cpp prints the choices; it is compiled for
the host from the sources of the library."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1708_09689_amd", "csrc")


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    cxx = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(cxx):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("rules") / "rules")
    cmd = [cxx, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
           os.path.join(ROOT, "tests", "launch_rules", "rules.cpp"), "-o", exe]
    done = subprocess.run(cmd, capture_output=True, text=True)
    assert done.returncode == 0, done.stderr

    def ask(line):
        out = subprocess.run([exe], input=line + "\n", capture_output=True, text=True)
        assert out.returncode == 0, line
        return tuple(int(v) for v in out.stdout.split())

    return ask


# staged tile of a launch without a shape of its own: (elements per lane, lanes)
TILES = [
    # rows that fill long tiles, walks enough for 512-lane workgroups
    ("ti 0 256 256 64 4 plain", (2, 512)),     # 503 short, 472 long, 444 long with 512 lanes
    ("ti 0 64 64 64 32 step", (2, 512)),       # 326, 304, 292
    ("ti 1 256 256 64 4 step", (4, 256)),      # 320, 275, 288
    ("ti 0 64 64 64 8 step", (2, 256)),        # 83, 71, 73
    # a last round of 512-lane workgroups that is mostly idle
    ("ti 0 72 64 64 32 step", (2, 256)),       # 379, 376, 413
    ("ti 0 264 256 64 4 plain", (2, 256)),     # 522, 502, 543
    # rows that leave long tiles half empty
    ("ti 0 17 300 60 16 step", (1, 256)),      # 210, 235, 342
    ("ti 0 33 200 50 8 plain", (1, 256)),      # 93, 118, 153
    ("ti 1 65 65 65 8 step", (2, 256)),        # 61, 73, 91
    ("weyl 0 130 130 60 4 plain", (1, 256)),   # 72, 87, 122
    # rows much shorter than any tile: a long one is empty lanes only
    ("graphene4 0 8 200000 1 1 step", (1, 256)),
    ("graphene4 0 512 512 1 32 step", (2, 512)),   # 330, -, 276
]


@pytest.mark.parametrize("launch,choice", TILES)
def test_tile_of_a_staged_launch(rules, launch, choice):
    assert rules("tile " + launch) == choice


# walks of a staged launch on the short tile: (planes per walk, 1 along y).
# 96 and 128 workgroups per XCD: three and four per CU.
WALKS = [
    ("weyl 1 65 65 65 16 128", (22, 0)),      # 22 planes 45.0, 13 planes 49.9
    ("weyl 1 130 130 60 4 128", (20, 0)),     # 20 planes 42.8, 12 planes 47.2
    ("weyl 1 100 90 40 8 128", (14, 0)),      # 14 planes 30.4, 8 planes 35.5
    ("ti 0 36 166 43 2 96", (15, 0)),         # 15 planes 31.7, 11 planes 37.6
    ("weyl 0 10 118 74 8 96", (13, 0)),       # fewer chunks fill it: 13 planes 24.4, 11 planes 26.2
    ("ti 0 40 40 40 8 64", (8, 0)),           # adjoint steps: more chunks gain, gradient 1383 against 1510 in 14
    ("ti 1 57 83 46 8 96", (23, 0)),          # series steps: 23 planes 62.1, 46 planes 66.3
    ("ti 0 240 240 6 32 64", (30, 1)),        # along y 346, along z 402
]


@pytest.mark.parametrize("launch,choice", WALKS)
def test_walks_of_a_staged_launch(rules, launch, choice):
    assert rules("walk " + launch) == choice


# adjoint steps: kernel and elements per lane of the launch shape -> 0 direct, 1
# staged with the run-time epilogue (slower than direct), 2 with its own
ADJOINTS = [
    ("ti 0 64 64 64 8 0 0", 2), ("ti 0 64 64 64 8 0 2", 2), ("ti 0 64 64 64 8 2 1", 2), ("ti 0 64 64 64 8 2 2", 2),
    ("ti 0 64 64 64 8 1 2", 0), ("ti 0 16 16 16 8 0 2", 0), ("ti 0 16 16 16 8 2 2", 2),
    ("weyl 0 64 64 64 16 0 2", 0), ("weyl 0 64 64 64 16 2 2", 2), ("graphene4 0 512 512 1 8 0 2", 2),
    # rows that leave the tiles mostly empty: direct by default
    ("ti 0 3 300 300 8 0 0", 0), ("ti 0 6 191 115 2 0 0", 0), ("ti 0 17 300 60 4 0 0", 2), ("ti 0 12 100 100 4 0 0", 2),
    ("graphene2 0 8 80000 1 1 0 0", 0), ("graphene2 0 30 20000 1 1 0 0", 2), ("ti 0 6 191 115 2 2 0", 2),
    ("ti 1 64 64 64 8 0 4", 0), ("ti 1 64 64 64 8 2 4", 1),
]


@pytest.mark.parametrize("launch,route", ADJOINTS)
def test_route_of_an_adjoint_step(rules, launch, route):
    assert rules("adjoint " + launch) == (route,)


# batches of cubes: (staged, longer tile)
BATCHES = [
    ((4, 1, 16), [64] * 12, (1, 1)),            # short 957, long 872
    ((4, 0, 8), [32] * 64, (1, 1)),             # 667, 609
    ((4, 1, 4), [32] * 64, (1, 0)),             # 184, 253: rows of half a long tile
    ((4, 1, 1), [32] * 64, (1, 0)),             # 143, 235
    ((4, 1, 4), [65] * 16, (1, 0)),             # 509, 586
    ((4, 1, 8), [33] * 40, (1, 0)),             # 371, 423
    ((4, 0, 2), [65] * 16, (1, 0)),             # 501, 565
    ((4, 1, 4), [96] * 4, (1, 0)),              # 315, 371: too few walks
    ((2, 1, 1), [95] * 27, (1, 0)),             # 534, 869
    ((4, 0, 1), [27, 62, 71, 85], (1, 0)),      # direct 179, staged 119
    ((4, 0, 4), [45] * 2, (1, 0)),              # direct 76, staged 67
    ((4, 0, 1), [64] * 3, (0, 0)),              # direct 78, staged 86
    ((4, 0, 1), [96], (0, 0)),                  # direct 77, staged 121
    ((4, 1, 1), [128], (0, 0)),                 # direct 92, staged 169
]


@pytest.mark.parametrize("kind,lengths,choice", BATCHES)
def test_default_shape_of_a_batch(rules, kind, lengths, choice):
    line = "batch {} {} {} ".format(*kind) + " ".join(map(str, lengths)) + " 0"
    assert rules(line) == choice


# rotations: one thread per entry (1) or matrix instructions (0)
ROTATIONS = [
    ("0 200000 1 1 0", 1),      # entries 2.4, matrix instructions 7.1
    ("0 1400000 2 2 1", 1),     # 2.7 times as fast
    ("1 1400000 8 1 0", 1),     # 1.7 times
    ("0 1400000 8 1 0", 0),     # matrix instructions 1.6 times as fast
    ("0 1400000 8 1 1", 0),     # 85, 69
    ("0 200000 8 4 1", 1),      # 12.5, 15.3
    ("1 600000 1 64 1", 1),     # 131, 164
    ("0 600000 1 64 1", 0),     # matrix instructions 1.1 times as fast
    ("0 3000 2 1 0", 1),        # 1.9, 2.6
    ("0 30000 4 8 1", 1),       # 1.2 times
    ("0 200000 8 8 0", 0),      # matrix instructions 1.9 times as fast
    ("0 30000 16 2 1", 1),      # 3.4, 4.5
    ("0 30000 16 1 1", 0),      # equal at this size, matrix instructions at others
    ("0 30000 64 1 1", 0),      # 1.2 times as fast
    ("0 1382400 32 32 1", 0),   # 396 against 1515
]


@pytest.mark.parametrize("launch,entry", ROTATIONS)
def test_kernel_of_a_rotation(rules, launch, entry):
    assert rules("rotate " + launch) == (entry,)

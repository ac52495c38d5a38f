"""Launch shapes that the library chooses by itself, on the host: ``ns_api.hip``
linked with ``launch_rules.cpp``, which reports what a call would launch on a
device of 256 compute units.  The GPU tests compare kernels that give the same
bits, so only this tells which of them ran."""
import os
import random
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FP64, FP32 = 0, 1


@pytest.fixture(scope="module")
def chosen(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    tmp = tmp_path_factory.mktemp("rules")
    objs = []
    for name, src in (("api.o", os.path.join(ROOT, "paper_1709_09713_amd", "csrc", "ns_api.hip")),
                      ("rules.o", os.path.join(HERE, "launch_rules.cpp"))):
        obj = str(tmp / name)
        subprocess.check_call([HIPCC, "-x", "hip", "--offload-host-only", "--offload-arch=gfx950", "-O1", "-std=c++17",
                               "-fPIC", "-w", "-I" + os.path.join(ROOT, "include"), "-c", src, "-o", obj])
        objs.append(obj)
    exe = str(tmp / "rules")
    subprocess.check_call(["g++", "-o", exe, *objs])

    def run(calls):
        """(planes of a brick or 0, tile, z-chunk, partials fit) per (precision, grid)"""
        text = "".join(f"{q} {n[0]} {n[1]} {n[2]}\n" for q, n in calls)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True, timeout=60).stdout
        return [tuple(int(x) for x in line.split()) for line in out.splitlines()]

    return run


def test_bricks(chosen):
    want = [((FP64, (5, 5, 5)), 2), ((FP64, (8, 5, 8)), 2), ((FP64, (7, 9, 6)), 2), ((FP64, (16, 16, 16)), 2),
            ((FP64, (24, 24, 24)), 2), ((FP64, (31, 33, 12)), 2), ((FP64, (2048, 5, 5)), 0), ((FP64, (32, 32, 32)), 4),
            ((FP64, (33, 32, 32)), 4), ((FP64, (40, 40, 40)), 4), ((FP64, (44, 44, 44)), 0), ((FP64, (64, 40, 28)), 0),
            ((FP64, (16, 165, 5)), 4), ((FP32, (16, 16, 16)), 2), ((FP32, (32, 32, 32)), 4), ((FP32, (48, 48, 48)), 4),
            ((FP32, (50, 50, 50)), 0), ((FP32, (16, 165, 5)), 4)]
    got = chosen([c for c, _ in want])
    assert [g[0] for g in got] == [w for _, w in want]


def test_tiles_of_the_march(chosen):
    """FP64: 16x8 in three groups on grids of about one block a compute unit,
    else 32x8.  FP32 storage: three groups where measured faster."""
    sides = range(44, 161)
    f64 = {n: g[1] for n, g in zip(sides, chosen([(FP64, (n, n, n)) for n in sides]))}
    assert all(f64[n] == 8 for n in (48, 56, 64, 80)) and all(f64[n] == 9 for n in (88, 96, 128, 160))
    assert set(f64.values()) == {8, 9}
    f32 = {n: g[1] for n, g in zip(sides, chosen([(FP32, (n, n, n)) for n in sides]))}
    three = [n for n in sides if f32[n] == 9]
    assert three == [*range(49, 97), *range(113, 117), *range(121, 125)]
    assert all(f32[n] in (-1, 0) for n in sides if n not in three)


def test_partials_fit_the_workspace(chosen):
    rng = random.Random(5)
    grids = [tuple(rng.choice((rng.randint(5, 12), rng.randint(5, 70), rng.randint(5, 300))) for _ in range(3))
             for _ in range(4000)]
    assert all(g[3] == 1 for q in (FP64, FP32) for g in chosen([(q, n) for n in grids]))

"""The rules that choose a GEMM kernel, on the host: the shapes that were
measured on both sides of a rule go to the faster one, and the shapes of the
GPU tests to the kernels that those tests are for."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    from paper_2503_23144_amd import build, lrcc
    d = str(tmp_path_factory.mktemp("plans"))
    lib_dir, lib = os.path.split(lrcc.LIB_PATH)
    subprocess.run([build.HIPCC, "-x", "hip", "--cuda-host-only", "-std=c++17", "-I" + os.path.join(ROOT, "include"),
                    "-I" + build.SRC, "-c", os.path.join(ROOT, "tests", "gemm_plans.cpp"), "-o", d + "/plans.o"],
                   check=True, capture_output=True, timeout=120)
    subprocess.run([build.HIPCC, "-o", d + "/plans", d + "/plans.o", "-L" + lib_dir, "-l:" + lib,
                    "-Wl,-rpath," + lib_dir], check=True, capture_output=True, timeout=120)

    def run(queries):
        r = subprocess.run([d + "/plans"], input="\n".join(queries) + "\n", capture_output=True, text=True, timeout=60)
        assert r.returncode == 0
        return [[float(x) for x in line.split()] for line in r.stdout.splitlines()]

    return run


# (fp64, ta, tb, m, n, k), us on the tiled kernel, us on the wavefront kernel
MEASURED = [((1, 0, 0, 4000, 3900, 3000), 6740, 6135), ((1, 0, 0, 4000, 3900, 600), 1381, 1410),
            ((1, 0, 1, 9000, 1700, 3000), 6225, 6970), ((1, 1, 0, 9784, 612, 25), 42.7, 62.2),
            ((1, 0, 1, 3500, 3500, 600), 1004, 1162), ((1, 0, 1, 686, 799, 9669), 775, 950),
            ((1, 1, 0, 1798, 884, 45), 21.0, 27.9), ((1, 0, 0, 3000, 3000, 3000), 3822, 3582),
            ((1, 0, 0, 438, 1284, 330), 61.4, 55.0), ((1, 0, 1, 1548, 229, 499), 88.9, 48.0),
            ((1, 1, 0, 7784, 36, 306), 57.7, 30.9), ((0, 0, 0, 388, 4541, 736), 98.3, 133.0),
            ((0, 0, 0, 7015, 55, 11561), 325.7, 468.6), ((0, 1, 0, 8614, 42, 7382), 273.1, 371.3),
            ((0, 1, 0, 2290, 121, 11254), 220.4, 269.1), ((0, 0, 1, 868, 2006, 1826), 222.4, 162.5),
            ((0, 0, 1, 3564, 144, 4693), 217.8, 177.9), ((0, 0, 1, 7930, 268, 1318), 225.3, 186.1)]


def test_measured_products_take_the_faster_kernel(plans):
    for (q, tiled, wave), p in zip(MEASURED, plans(["w " + " ".join(map(str, q)) for q, _, _ in MEASURED])):
        assert (p[0] >= 0) == (wave < tiled), q


def test_gpu_test_shapes_cover_every_variant(plans):
    from test_gpu_gemm_paths import test_gemm_few_tiles_matches_host as few
    shapes = next(m for m in few.pytestmark if m.name == "parametrize" and m.args[0] == "m,n,k").args[1]
    for fp64 in (1, 0):
        seen = plans([f"w {fp64} {ta} {tb} {m} {n} {k}" for m, n, k in shapes for ta, tb in
                      ((0, 0), (0, 1), (1, 0), (1, 1))])
        assert {int(p[0]) for p in seen} == {0, 1, 2, 3, 4}
        assert {int(p[0]) for p in seen if p[1] > 1} >= {0, 2}

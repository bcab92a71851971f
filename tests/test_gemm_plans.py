"""The rules that choose a GEMM kernel, on the host: the shapes that were
measured on both sides of a rule go to the faster one, and the shapes of the
GPU tests to the kernels that those tests are for; and the memory that its
packed operands give back."""
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


STATIC, CONTEXT = 256 << 20, 1280 << 20  # bytes that lrcc_gemm_noalloc and a context have for packed operands


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_large_fp32_products_fit_their_memory(plans, ta, tb):
    """A product too large for the packed operands is cut into blocks of rows,
    columns or depth; the memory does not take it off the BF16 kernel."""
    sizes = [1024, 1536, 2048, 3072, 4096, 6144, 8192, 12288, 18432, 32768]
    shapes = [(m, n, k) for m in sizes for n in sizes for k in (512, 1024, 2048, 3072, 6144, 12288)]
    shapes += [(18000, 3000, 3000), (3200, 3200, 3072), (4000, 4000, 3000), (5000, 5000, 3000), (6000, 6000, 6000),
               (8192, 8192, 3072), (30000, 30000, 3072), (12500, 12600, 1100)]
    free = [p[0] for p in plans([f"s {ta} {tb} {m} {n} {k} {1 << 50}" for m, n, k in shapes])]
    assert sum(free) > 300 and all(free[-8:])
    for budget in (STATIC, CONTEXT):
        for s, f, (use, splits, mc, nc, kl, total) in zip(shapes, free, plans([f"s {ta} {tb} {m} {n} {k} {budget}"
                                                                               for m, n, k in shapes])):
            m, n, k = s
            assert use == f, (s, budget)
            if not use:
                continue
            assert 0 < total <= budget, (s, budget)
            assert 0 < mc <= m and 0 < nc <= n and 0 < kl <= k, (s, budget)
            assert kl / splits <= 3072 and (kl == k or kl % 32 == 0), (s, budget)
            rows = lambda x: -(-x // 128) * 128  # noqa: E731
            packed = (rows(mc) + rows(nc)) * -(-kl // 32) * 32 * 18 + (splits * mc * nc * 8 if splits > 1 else 0)
            assert packed < total <= packed + 4096, (s, budget)


def test_small_budgets_and_products_are_left_to_fp32(plans):
    for q in ("0 1 2000 2000 2000 1000000", "0 1 100 100 100 1000000000", "0 1 5000 5000 255 1000000000",
              "0 1 16 20000 20000 1000000000", "0 1 0 10 10 1000000000"):
        assert plans(["s " + q])[0][0] == 0, q


def test_gpu_test_shapes_take_the_bf16_kernel(plans):
    import test_gpu_gemm_calls as calls
    import test_gpu_gemm_split_range as rng
    params = lambda f: next(m for m in f.pytestmark if m.args[0] == "m,n,k").args[1]  # noqa: E731
    shapes = [(2040, 2048, 2001), (4096, 2048, 1100)] + params(rng.test_large_values_in_split_and_blocked_products)
    blocked = params(calls.test_blocks_of_the_operands_match_64_bits)
    for ta, tb in ((0, 0), (0, 1), (1, 0), (1, 1)):
        got = plans([f"s {ta} {tb} {m} {n} {k} {STATIC}" for m, n, k in shapes + blocked])
        assert all(p[0] for p in got)
        kinds = {(p[2] < m, p[3] < n, p[4] < k) for p, (m, n, k) in zip(got, shapes + blocked)}
        assert {(True, True, False), (True, False, True), (False, False, False)} <= kinds, kinds


def test_a_failing_allocation_asks_once_for_what_can_yield(plans):
    assert plans(["y"]) == [[1.0]]

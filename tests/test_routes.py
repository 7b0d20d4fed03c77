"""The host-side launch rules (paper_2403_04206_amd/csrc/grawa_route.h, no GPU dependency) at sizes that no test can
allocate: a small program prints what the rules give."""
import os
import shutil
import subprocess
from decimal import Decimal, getcontext

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("route") / "route_driver")
    res = subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-I",
                          os.path.join(ROOT, "paper_2403_04206_amd", "csrc"), os.path.join(ROOT, "tests", "route_driver.cpp"),
                          "-o", out], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    return lambda *args, read=int: [[read(v) for v in line.split()] for line in
                          subprocess.run([out] + [str(a) for a in args], capture_output=True, text=True,
                                         check=True).stdout.splitlines()]


def test_row_split_grid_within_the_launch_limit(driver):
    P = [1, 256, 257, (1 << 26) - 1, 1 << 26, (1 << 26) + 1, (1 << 30) - 256, 1 << 30, (1 << 30) + 1, (1 << 31) + 5, (1 << 32) - 512]
    cells = sorted({(p + 255) // 256 for p in P})
    rows = driver("split", *cells)
    for n in cells:
        launches = [r for r in rows if r[0] == n]
        assert all(blocks >= 1 and blocks * threads < 1 << 32 for _, _, blocks, threads in launches)
        assert [r[1] for r in launches] == [sum(r[2] for r in launches[:i]) for i in range(len(launches))]   # no gap
        assert sum(r[2] for r in launches) == n          # every cell once
        assert len(launches) == 1 or n > 1 << 18



def test_no_arrivals_with_many_layers(driver):
    # one arrival per layer on one address: bounded by a rule on the layer count, whatever else the problem is
    assert driver("model", 1, 62, 100, 101, 161, 291, 100000) == [[1, 1], [62, 1], [100, 1], [101, 0], [161, 0], [291, 0], [100000, 0]]


def test_estimate_launch(driver):
    cases = [(K, L, T) for K in (1, 3, 8, 15, 16, 17, 64, 1024) for L in (1, 60, 511, 512, 513, 5000, 1 << 20)
             for T in (1, 128, 129, 1024, 1025, 50000)]
    for (K, L, T, rows, threads, most) in driver("estimate", *[v for c in cases for v in c]):
        assert 64 <= threads <= 1024 and threads % 64 == 0 and 1 <= rows <= K
        assert rows == 1 or rows * L <= (512 if T <= most else 4096)
        assert most == (128 if K * L <= 512 else 1024)
        assert T > most or (rows - 1) * (threads // 64) < K              # no row of blocks without a worker
        assert L * threads < 1 << 32


def test_weights_in_the_pull(driver):
    # every block adds the tiles of its layers: bounded by the blocks alone where there are few workers
    on = [(1, 2560), (2, 2560), (4, 2560), (8, 1280), (15, 682)]
    off = [(1, 2561), (1, 10240), (2, 2561), (2, 5120), (3, 2561), (4, 2561), (8, 1281), (15, 683), (16, 1)]
    assert all(r[2] == 1 for r in driver("tiles", *[v for c in on for v in c]))
    assert all(r[2] == 0 for r in driver("tiles", *[v for c in off for v in c]))


def test_no_route_without_a_kernel(driver):
    # the rule that sends a call to the weights-in-the-pull form knows no other counts than its dispatch
    have = dict(driver("counts", *range(1, 1025)))
    assert [k for k in have if have[k]] == list(range(1, 16))
    assert all(r[2] == have[r[0]] for r in driver("tiles", *[v for k in range(1, 1025) for v in (k, 1)]))


def test_forms_of_rows_off_the_grid(driver):
    plain, wide, burst = range(3)
    rows = {(k, sgd): tuple(rest) for k, sgd, *rest in driver("offgrid", *range(1, 1025))}
    assert all(has for _, _, _, has in rows.values())     # every count has a kernel of the form that the rule names
    for (k, sgd), (form, groups, merge, _) in rows.items():
        if k > 71:
            assert form == plain
        elif k <= 5 or (sgd and 12 <= k <= 23):
            assert form == wide and merge == (sgd and k <= 5)
        else:
            assert form == burst and (groups, merge) == ((2, 1) if k <= 9 else (4, 1) if k <= 15 else (4, 0) if k <= 23 else (8, 0))


def test_bursts_without_the_step_begin_where_no_cache_holds_the_array(driver):
    rows = driver("offgrid_large", *[v for k in range(1, 72) for sgd in (0, 1) for mb in (128, 129, 320, 321) for v in (k, sgd, mb)])
    for k, sgd, mb, yes in rows:
        assert yes == (mb > (320 if not sgd and (6 <= k <= 11 or k >= 24) else 128))


def test_local_steps_off_the_grid(driver):
    # steps that follow each other find part of x in the cache: without the center they stream only where it is larger than that
    from_mb = {(bf16, center, scored): mb for bf16, center, scored, mb in driver("rowstep")}
    assert from_mb == {(0, 0, 0): 0, (0, 0, 1): 320, (0, 1, 0): 0, (0, 1, 1): 0,
                       (1, 0, 0): 0, (1, 0, 1): -1, (1, 1, 0): 128, (1, 1, 1): 0}


def test_scored_step_by_layers(driver):
    M = 1 << 20
    ask = lambda *case: driver("layers", *case)[0][4]
    assert [ask(1, 1, 1024 * tiles, tiles) for tiles in (1, 7, 8, 10, 40)] == [1, 1, 0, 0, 0]             # longest layer
    assert [ask(1, 600, p, 7) for p in (3 * M, 3 * M + 1, 4 * M, 4 * M + 1)] == [1, 1, 1, 0]               # elements
    assert [ask(1, 600, p, 8) for p in (3 * M, 3 * M + 1, 4 * M, 4 * M + 1)] == [0, 1, 1, 0]
    assert [ask(1, 600, p, t) for p, t in ((4 * M, 10), (4 * M, 11))] == [1, 0]
    assert [ask(k, L, 1000, 7) for k, L in ((1, 2560), (64, 40), (1, 2561))] == [1, 1, 0]                  # blocks
    assert [ask(1, L, 4 * M, 10) for L in (640, 641)] == [1, 0]
    # products beyond 32 bits
    assert ask(1024, 1 << 30, 1 << 31, 1) == 0 and ask(1024, 1, 1 << 31, 1 << 21) == 0


def test_sums_left_to_the_next_launch(driver):
    later = lambda *case: driver("fold", *case)[0][0]
    # never what a block takes by layers
    assert [later(4, 59, 270000, t) for t in (7, 8)] == [0, 1]
    assert [later(4, 400, 1 << 20, t) for t in (7, 8)] == [0, 1] and [later(4, 100, 1 << 20, t) for t in (10, 11)] == [0, 1]
    M = 1 << 17                                                                                            # blocks of 1024 columns
    assert [later(1, 1, 1024 * n, n) for n in (M, M + 1)] == [1, 0] and [later(8, 1, 1024 * n, n) for n in (M // 8, M // 8 + 1)] == [1, 0]
    assert later(1024, 1, (1 << 32) - 512, 1 << 22) == 0
    assert [later(4, L, 1 << 23, 40) for L in (2048, 2049)] == [1, 0]                                     # layers
    assert [later(64, L, 1 << 20, 40) for L in (320, 321)] == [1, 0] and later(1024, 21, 100000, 40) == 0      # sums
    # one longer than a wave adds
    assert [later(8, L, 1 << 21, t) for L, t in ((128, 512), (129, 512), (128, 513), (129, 513))] == [1, 1, 1, 0]
    for tiny in ((70, 700, 7700, 1), (2, 5000, 15000, 2), (100, 250, 250 * 7, 1), (35, 31, 614550, 601), (40, 31, 1050666, 1027),
                 (3, 2101, 1051701, 1026), (5, 4101, 1057876, 1027)):
        assert later(*tiny) == 0, tiny               # what the GPU tests of the estimate's own launch take


def test_weights_from_estimates_in_the_pull(driver):
    yes = lambda *case: driver("fold", *case)[0][1]
    assert [yes(4, 9, 270000, t) for t in (128, 129)] == [1, 0] and [yes(15, 3, 40000, t) for t in (34, 35)] == [1, 0]
    assert yes(1, 1, 512 * 1024, 512) == 1 and yes(1, 1, 513 * 1024, 513) == 0
    assert yes(16, 1, 20000, 20) == 0 and [yes(8, 10, 256 * n, 60) for n in (1280, 1281)] == [1, 0]


def test_folding_of_long_layers(driver):
    # the launch of the weights adds them itself; and what many workers have beyond 8000 tiles, a launch before it
    for case, yes in (((64, 1, 126000, 124), 1), ((64, 1, 128000, 125), 0), ((33, 1, 250000, 243), 0), ((33, 1, 250000, 242), 1), ((32, 1, 1 << 19, 512), 1),
                      ((8, 1, 1 << 22, 4096), 1), ((9, 1, 1 << 20, 1024), 0), ((8, 2, 1 << 23, 4097), 0), ((1, 1, 1 << 20, 1024), 1)):
        assert driver("fold", *case)[0][2] == yes, case


def test_blocks_that_fold_in_the_step(driver):
    # all sums have a wave or block; the columns of every row stay on the XCDs (8 blocks apart) that they have without them, or, with the center, on one
    cases = [(K, L, t, c, group, z) for K in (1, 2, 7, 40, 41, 64, 1024) for L in (1, 20, 1024) for t in (1, 512, 513) for c in (0, 1)
             for group in (1, 9, 199, 200, 201, 255, 300, 4096, 50000) for z in (1, 3) if z == 1 or group == 4096]
    for K, L, t, c, group, z, blocks, rows in driver("fold_blocks", *[v for case in cases for v in case]):
        want = K * L if t > 512 else -(-K * L // 4)
        assert (blocks > 0) != (rows > 0) and (rows == 0 or z == 1) and rows + K <= 65535
        assert blocks * K * z >= want or rows * group >= want
        assert (group + blocks) % 8 == 0 if c and K <= 40 and group >= 200 else blocks % 8 == 0
    assert [r[6:] for r in driver("fold_blocks", 64, 1, 300, 0, 300, 1, 4, 60, 40, 0, 300, 1, 4, 60, 40, 1, 300, 1, 40, 1, 300, 1, 304, 1)] == \
        [[0, 1], [16, 0], [20, 0], [0, 1]]


def test_folding_for_the_model_level(driver):
    cases = [(4, 256, 17, 4), (4, 256, 17, 5), (4, 257, 17, 4), (16, 64, 512, 1), (16, 64, 513, 1), (17, 2, 30, 1), (1024, 1, 10, 0), (1025, 1, 10, 0)]
    assert [r[0] for r in driver("fold_model", *[v for c in cases for v in c])] == [1, 0, 0, 1, 0, 0, 1, 0]


def test_columns_of_g_read_through_the_caches(driver):
    cases = [(k, p, e) for k in (1, 2, 3, 7, 64, 1000, 1024) for p in (1, 255, 60000, 1 << 20, (1 << 32) - 1) for e in (2, 4)]
    for k, p, e, cols in driver("cachedg", *[v for c in cases for v in c]):
        assert 1 <= cols <= p and cols * k * e <= 224 << 20
        assert cols == p or (cols + 1) * k * e > 224 << 20


def test_power_of_gamma(driver):
    # 1 - gamma^t of the running estimate, gamma a float32 up to the last one below 1: at most four units of the last place
    getcontext().prec = 60
    cases = [(float(np.float32(g)), t) for g in (1e-30, 0.1, 0.5, 0.9, 0.99, 0.999, 1 - 2.0 ** -20, 1 - 2.0 ** -24)
             for t in (1, 2, 3, 4, 5, 7, 10, 16, 31, 100, 1000, 4097)]
    got = driver("power", *[v for g, t in cases for v in (repr(g), t)], read=float.fromhex)
    for (g, t), (read, value) in zip(cases, got):
        assert read == g
        exact = 1 - Decimal(g) ** t
        assert abs(Decimal(value) / exact - 1) <= Decimal(4 * 2.0 ** -53), (g, t)


def test_plain_form_counts(driver):
    # each count the rule names has a kernel: 1..15 and 17..32 (16 has its own form), and 32 only on few cells
    rows = driver("plain", *[v for k in (1, 23, 24, 32, 33, 64) for n in (1, 800, 801, 1 << 24) for v in (k, n)])
    assert [r[2] for r in rows] == [1] * 8 + [1, 1, 0, 0] * 2 + [0] * 8


def test_a_missing_kernel_is_an_error():
    src = open(os.path.join(ROOT, "paper_2403_04206_amd", "csrc", "grawa_pull.hip")).read()
    for name, counts in (("dispatch_cp_off_grid", "GRAWA_OFF_GRID_EACH"), ("dispatch_cp_off_grid", "GRAWA_OFF_GRID_EIGHTHS"),
                         ("dispatch_cp_tiles", "GRAWA_TILES_COUNTS")):
        body = src[src.index("static hipError_t %s(" % name):]
        body = body[:body.index("\n}\n")]
        assert counts in body and "return hipErrorInvalidValue;" in body

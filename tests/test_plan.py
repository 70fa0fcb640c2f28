"""The FFT form's work decomposition (host code, no GPU): tests/host/plan_print.cpp, linked to
libbfly.so, prints the planner's ranges for banks and block counts too large to search here."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    from paper_1802_01685_amd import build as B
    if not any(c and os.path.exists(c) for c in
               (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc"))):
        pytest.skip("no ROCm toolchain")
    out = tmp_path_factory.mktemp("plan")
    obj, exe = str(out / "plan_print.o"), str(out / "plan_print")
    src = os.path.join(ROOT, "tests", "host", "plan_print.cpp")
    for cmd in ([B._hipcc(), *B.COMMON, *B.DEVICE, "-c", src, "-o", obj],
                [B._hipcc(), *B.DEVICE, obj, B.LIB, f"-Wl,-rpath,{os.path.dirname(B.LIB)}",
                 "-o", exe]):
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-3000:]

    def run(*shapes, args=()):
        text = "".join(" ".join(str(v) for v in s) + "\n" for s in shapes)
        r = subprocess.run([exe, *args], input=text, capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, r.stderr[-3000:]
        return [tuple(int(v) for v in line.split()) for line in r.stdout.splitlines()]

    return run


def test_items_fit_a_launch(plan):
    """Batches of many blocks: a work-group of 512 threads per item stays below HIP's 2^32
    threads, and the ranges remain a multiple of 8 (each XCD sweeps its own)."""
    shapes = [(n_bins, n_fdot, L, blocks, 256, tails, 1)
              for n_bins, n_fdot, L in ((240, 3000, 2000), (256, 1024, 64), (2880, 3000, 2000),
                                        (9, 70000, 4096))
              for blocks in (35000, 131072, 500000, 1000000) for tails in (0, 1)]
    for s, (ranges, items) in zip(shapes, plan(*shapes)):
        assert items * 512 < 2 ** 32, (s, ranges, items)
        assert ranges % 8 == 0 and 8 <= ranges <= s[0], (s, ranges)


# bins, templates per bin, L, blocks, t_block: the ranges within 5% of the fastest of 8, 16, 24, 32,
# 40, 48, 64, 96, 128, ... 512, in the single pass of a tail search on an MI355X
TAIL_PLANS = {
    (16, 64, 600, 200, 1): {16},
    (16, 64, 600, 1000, 1): {8, 16},
    (502, 1, 1024, 300, 1): {8, 16, 24, 32, 40, 48},
    (300, 5, 1024, 100, 1): {24, 40},
    (64, 30, 2000, 40, 1): {64},
    (66, 89, 512, 300, 1): {8, 24, 40},
    (48, 200, 1024, 5, 1): {48},
    (249, 9, 37, 40, 1): {24, 64},
    (256, 256, 4096, 30, 1): {256},
    (64, 64, 4096, 120, 1): {8, 16, 24, 32, 40, 48, 64},
    (240, 300, 2000, 42, 1): {24, 48, 240},
    (64, 512, 2000, 2, 1): {64},
    (24, 100, 2000, 48, 1): {8, 24},
    (16, 16, 600, 1000, 1): {8},
    (240, 3000, 2000, 11, 1): {40, 240},
    (512, 16, 2000, 15, 1): {32, 64, 96, 128, 192, 256},
    (64, 30, 2000, 40, 16): {24, 32, 64},
    (99, 16, 600, 80, 16): {32, 40, 56, 64},
    (96, 3, 512, 40, 16): {24, 48},
}


# the same in plain searches
SEARCH_PLANS = {
    (200, 10, 1024, 14, 1): {72},
    (16, 64, 600, 200, 1): {16},
    (96, 3, 512, 40, 1): {24, 32},
    (64, 30, 2000, 40, 256): {64},
    (128, 40, 4096, 28, 1): {64, 128},
    (256, 256, 4096, 31, 1): {256},
    (240, 3000, 2000, 42, 1): {48, 240},
}


@pytest.mark.parametrize("tails", [0, 1])
def test_plans_near_the_fastest(plan, tails):
    fastest = TAIL_PLANS if tails else SEARCH_PLANS
    got = {s: r for s, (r, _) in zip(fastest, plan(*[s[:4] + (256, tails, s[4]) for s in fastest]))}
    assert {s: r for s, r in got.items() if r not in fastest[s]} == {}


def test_plan_refuses_short_series_first(plan):
    """bf_plan's argument checks come before the device is asked for (exit status 2 otherwise)."""
    assert plan() == []


def test_small_fp32_searches_take_the_small_tile(plan, monkeypatch):
    """The 1 x 1 tile of 128 offsets up to a few work items per CU (the shapes of
    test_gpu_small_tile, the shortest among them, whose item counts are those of the 2 x 4 tile),
    the 2 x 4 tile of 512 beyond and where BF_TILE asks for it: in the first eight large searches
    it took at least 1.3 times less time in k_main."""
    banks = [(16, 16, 512), (3, 40, 37), (5, 7, 200), (9, 33, 97), (1, 70, 16)]
    small = [b + (W, 256) for b in banks for W in (1, 127, 128, 129, 513, 1537)]
    large = [(4, 8, 37, 60000, 256), (4, 8, 256, 200000, 256), (16, 16, 64, 60000, 256),
             (36, 3, 64, 133760, 256), (36, 3, 128, 200000, 256), (3, 100, 64, 200000, 256),
             (1, 20, 128, 200000, 256), (4, 8, 512, 200000, 256), (256, 256, 4096, 126977, 256),
             (64, 64, 2000, 126001, 256)]
    monkeypatch.delenv("BF_TILE", raising=False)
    assert plan(*small, args=("tiles",)) == [(1, 1, 128)] * len(small)
    assert plan(*large, args=("tiles",)) == [(2, 4, 512)] * len(large)
    monkeypatch.setenv("BF_TILE", "2x4")
    assert plan(*small, args=("tiles",)) == [(2, 4, 512)] * len(small)


def test_ranges_cut_bins_where_that_is_faster(plan):
    """Searches of one series on an MI355X in which ranges that cut bins took at least 1.1 times as
    long as whole bins (their parts of bins meet in atomics), and in which
    they took at most 0.8 times as long."""
    # bins, templates per bin, L, offsets, CUs
    slower = [(255, 4, 512, 4373), (64, 16, 512, 4373), (510, 2, 2000, 7001), (64, 16, 600, 19401),
              (100, 10, 600, 19401), (60, 9, 600, 19401), (300, 16, 1024, 38977),
              (700, 3, 1024, 38977), (600, 1, 1024, 38977)]
    faster = [(9, 97, 512, 4373), (5, 300, 600, 19401), (1, 600, 2000, 7001), (48, 200, 4096, 28673),
              (16, 64, 2000, 7001), (40, 100, 512, 4373)]
    cuts = [r[0] for r in plan(*[s + (256,) for s in slower + faster], args=("cuts",))]
    assert cuts[:len(slower)] == [0] * len(slower)
    assert all(c > s[0] for c, s in zip(cuts[len(slower):], faster))

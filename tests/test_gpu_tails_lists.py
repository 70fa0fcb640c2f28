"""FFT tail searches whose pair lists hold most of the bank (BF_TAILS_MARGIN above every exact
threshold lists every template): lists, sigma and counts equal those of two passes bit for bit,
for one template, few groups of 64 templates, more groups than shards, lists too long to be worth
it (those get the whole pass) and a batch in which one series alone lists nothing."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from synth import BankParams, white_noise  # noqa: E402
from tests.test_gpu_tails import _tails_run  # noqa: E402

pytestmark = pytest.mark.gpu


def _bank(grid, L):
    return BankParams(fs=float(L), L=L, n_f0=grid[0], n_fdot=grid[1], f0_min=0.04 * L,
                      f0_max=0.4 * L, fdot_min=-0.2 * L, fdot_max=0.2 * L)


@pytest.mark.parametrize("grid,L,lengths,margin", [
    ((1, 1), 64, [64], "1.1"), ((1, 19), 600, [700] * 3 + [16000], "1.1"),
    ((13, 5), 55, [65], "1.1"), ((54, 3), 256, [460] * 700, "1.0"),
    ((40, 420), 512, [9000], "1.1"), ((16, 64), 600, [3000] * 90, "1.05"),
    ((16, 64), 600, [3000] * 90, "0.99"), ((9, 100), 1024, [30000, 1024, 1500], "1.0")])
def test_lists_equal_two_passes(grid, L, lengths, margin, monkeypatch):
    from paper_1802_01685_amd import bfly as bf
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    xs = [white_noise(n, 17 * i + n).astype(np.float32) for i, n in enumerate(lengths)]
    if len(xs) > 1:
        xs[1][:] = 1.0     # every window degenerate
    bank = bf.bank_create(_bank(grid, L), "fft")
    want_out, want = _tails_run(bf, bank, xs, 3.5, {"BF_TAILS_TWO_PASS": "1"}, monkeypatch)
    got_out, got = _tails_run(bf, bank, xs, 3.5, {"BF_TAILS_MARGIN": margin}, monkeypatch)
    for i in range(len(xs)):
        assert want[i]["n"] == got[i]["n"]
        for key in ("sigma", "tau", "k", "rho", "counts"):
            assert np.array_equal(np.asarray(want[i][key]).view(np.uint8),
                                  np.asarray(got[i][key]).view(np.uint8)), (i, key)
        for key in want_out[i]:
            assert np.array_equal(want_out[i][key].view(np.uint8),
                                  got_out[i][key].view(np.uint8)), (i, key)


@pytest.mark.parametrize("grid,L,n,series", [((1, 19), 600, 7000, 150),
                                             ((5, 63), 4096, 11617, 40),
                                             ((16, 64), 600, 3000, 400)])
def test_long_lists_keep_the_chip_busy(grid, L, n, series, monkeypatch):
    """The tails of a bank listed whole take no more than four times the whole tails pass (which
    candidate lists without room select): each pair is the same transform, at most twice as long
    for its block's reload, and as much again for other kernels and the clock's noise.  Lists
    handed to a few work-groups took 20 to 47 times as long."""
    from paper_1802_01685_amd import bfly as bf
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    bank = bf.bank_create(_bank(grid, L), "fft")
    gen = torch.Generator(device="cuda").manual_seed(2)
    xs = [torch.randn(n, generator=gen, device="cuda") for _ in range(series)]
    prm = bf.make_params(t_block=64)
    outs = [bf.alloc_outputs(bank, n, prm, "cuda") for _ in xs]
    tails = [bf.alloc_tails(bank, 4096, "cuda") for _ in xs]
    ws = torch.empty(bf.tails_workspace_bytes(bank, [n] * series, prm), dtype=torch.uint8,
                     device="cuda")

    def tail_stage(env):
        with monkeypatch.context() as m:
            for k, v in env.items():
                m.setenv(k, v)
            best = float("inf")
            for i in range(5):
                bf.set_timing(i > 0)
                bf.search_tails(bank, xs, 6.0, 4096, prm, outs=outs, tails=tails, workspace=ws)
                torch.cuda.synchronize()
                bf.set_timing(False)
                if i:
                    best = min(best, bf.kernel_times()[0]["finalize"])
            return best

    whole = tail_stage({"BF_TAILS_MARGIN": "1.1", "BF_TAILS_CAND_CAP": "0"})
    lists = tail_stage({"BF_TAILS_MARGIN": "1.1"})
    print(f"{grid} x {series}: lists {lists:.3f} ms, whole pass {whole:.3f} ms")
    assert lists <= 4.0 * whole

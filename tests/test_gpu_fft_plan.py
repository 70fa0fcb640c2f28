"""FFT searches whose work ranges cut f0 bins (few blocks against few bins), against the same
search with decimated spectrograms, whose ranges hold whole bins: maxima, argmax, histogram and
spectrum equal bit for bit, the spectrogram's row blocks equal their maxima; and every offset
against the FP64 oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import bfly_oracle as O  # noqa: E402
from synth import BankParams, white_noise  # noqa: E402
from tests.parity_util import check_against_oracle, to_np  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid", [(8, 64), (3, 200), (1, 257), (16, 16), (9, 97)])
@pytest.mark.parametrize("lengths", [[3000], [9001, 700, 20000]])
def test_ranges_that_cut_bins(grid, lengths):
    from paper_1802_01685_amd import bfly as bf
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    p = BankParams(fs=600.0, L=600, n_f0=grid[0], n_fdot=grid[1], f0_min=20.0, f0_max=250.0,
                   fdot_min=-100.0, fdot_max=120.0)
    xs = [white_noise(n, n).astype(np.float32) for n in lengths]
    xs[0][1500] = np.nan
    xt = [torch.from_numpy(x).cuda() for x in xs]
    bank = bf.bank_create(p, "fft")
    cut = [to_np(o) for o in bf.search_batch(bank, xt, bf.make_params())]
    whole = [to_np(o) for o in bf.search_batch(bank, xt, bf.make_params(t_block=4))]
    for x, a, b in zip(xs, cut, whole):
        for k in ("max_abs", "argmax", "hist", "spectrum", "n_degenerate"):
            assert np.array_equal(a[k].view(np.uint8), b[k].view(np.uint8)), k
        W = a["spec"].shape[1]
        pad = np.zeros((grid[0], -(-W // 4) * 4), np.float32)
        pad[:, :W] = a["spec"]
        assert np.array_equal(pad.reshape(grid[0], -1, 4).max(2), b["spec"])
        x64 = x.astype(np.float64)
        check_against_oracle(x64, p, a, O.search(x64, p), "fft", f"cut/{grid}/{len(x)}")


@pytest.mark.parametrize("grid", [(32, 2100), (16, 4200)])
def test_ranges_of_a_long_search(grid):
    """More than 64 items per work-group: the ranges shrink towards 4096 templates.  The maxima,
    argmax and spectra are those of the two half banks, whose plans differ, bit for bit."""
    from paper_1802_01685_amd import bfly as bf
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = 4200 * (8193 - 64)
    gen = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn(n, generator=gen, device="cuda")
    got = []
    for index, count in ((0, 1), (0, 2), (1, 2)):
        p = BankParams(fs=64.0, L=64, n_f0=grid[0], n_fdot=grid[1], f0_min=2.0, f0_max=25.0,
                       fdot_min=-10.0, fdot_max=10.0, shard_index=index, shard_count=count)
        bank = bf.bank_create(p, "fft")
        params = bf.make_params(t_block=4096)
        if count == 1:
            ranges, items = bf.plan(bank, [n])
            assert ranges >= 16 and items == 4200 * ranges
        out = bf.alloc_outputs(bank, n, params, x.device, want=("max_abs", "argmax", "spectrum"))
        bf.search_segment(bank, x, params, out=out)
        torch.cuda.synchronize()
        got.append(out)
        del bank
    whole, lo, hi = got
    upper = hi["max_abs"] > lo["max_abs"]
    assert torch.equal(whole["max_abs"], torch.where(upper, hi["max_abs"], lo["max_abs"]))
    assert torch.equal(whole["argmax"], torch.where(upper, hi["argmax"], lo["argmax"]))
    assert torch.equal(whole["spectrum"], torch.cat([lo["spectrum"], hi["spectrum"]]))


@pytest.mark.parametrize("grid,lengths", [((8, 64), [3000]), ((3, 200), [3000, 9001]),
                                          ((1, 512), [700]), ((9, 97), [9001, 700, 20000]),
                                          ((1, 2051), [3000]), ((48, 200), [20000])])
def test_plan_reports_ranges_that_cut_bins(grid, lengths):
    """bf_plan gives the ranges of the search with default parameters: more than there are bins
    where they cut bins, a multiple of 8, and the results are those of whole bins (t_block = 4)."""
    from paper_1802_01685_amd import bfly as bf
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    p = BankParams(fs=600.0, L=600, n_f0=grid[0], n_fdot=grid[1], f0_min=20.0, f0_max=250.0,
                   fdot_min=-100.0, fdot_max=120.0)
    xt = [torch.from_numpy(white_noise(n, n).astype(np.float32)).cuda() for n in lengths]
    bank = bf.bank_create(p, "fft")
    ranges, items = bf.plan(bank, lengths)
    assert ranges > grid[0] and ranges % 8 == 0
    assert items == ranges * sum(-(-(n - p.L + 1) // (8193 - p.L)) for n in lengths)
    cut = [to_np(o) for o in bf.search_batch(bank, xt, bf.make_params())]
    whole = [to_np(o) for o in bf.search_batch(bank, xt, bf.make_params(t_block=4))]
    for a, b in zip(cut, whole):
        for k in ("max_abs", "argmax", "hist", "spectrum", "n_degenerate"):
            assert np.array_equal(a[k].view(np.uint8), b[k].view(np.uint8)), k

"""Prefix sums over the edges of their chunks of 2,048 samples.  Integer-valued samples with a
mean well inside one standard deviation keep every sum exact and the subtracted level at 0, so
the windows of a series and of the same series without its first s samples must agree bit for
bit wherever the chunk edges fall; and every window agrees with the FP64 oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import bfly_oracle as O  # noqa: E402
from synth import BankParams, white_noise  # noqa: E402
from tests.parity_util import check_against_oracle, to_np  # noqa: E402

pytestmark = pytest.mark.gpu
P = BankParams(fs=128.0, L=48, n_f0=3, n_fdot=4, f0_min=3.0, f0_max=40.0, fdot_min=-30.0,
               fdot_max=25.0)


@pytest.fixture(scope="module")
def bf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1802_01685_amd import bfly
    return bfly


def _series(n):
    x = np.rint(3.0 * white_noise(n, n)).astype(np.float32)
    x[[i for i in (2047, 6144) if i < n]] = np.inf
    x[[i for i in (2200, 4095, 4096) if i < n]] = np.nan
    return x


@pytest.mark.parametrize("norm", ["centred", "raw"])
@pytest.mark.parametrize("n", [48, 2047, 2048, 2049, 4096, 8200])
def test_chunk_edges(bf, n, norm):
    x32 = _series(n)
    bank = bf.bank_create(P, "fp32")
    prm = bf.make_params(norm=norm)
    g = to_np(bf.search_segment(bank, torch.from_numpy(x32).cuda(), prm))
    x64 = x32.astype(np.float64)
    check_against_oracle(x64, P, g, O.search(x64, P, norm=norm), "fp32", f"chunks/{n}", norm=norm)
    for s in (1, 700, 2047, 2048, 3000):
        if s + P.L > n:
            continue
        h = to_np(bf.search_segment(bank, torch.from_numpy(x32[s:].copy()).cuda(), prm))
        assert np.array_equal(h["max_abs"], g["max_abs"][s:]), s
        assert np.array_equal(h["argmax"], g["argmax"][s:]), s
        assert np.array_equal(h["spec"], g["spec"][:, s:]), s


def test_long_series_alone_and_in_a_batch(bf):
    """300,001 samples: 147 chunks."""
    bank = bf.bank_create(P, "fp32")
    xs = [torch.from_numpy(_series(n)).cuda() for n in (60, 300001, 2049)]
    alone = to_np(bf.search_segment(bank, xs[1], bf.make_params()))
    mixed = to_np(bf.search_batch(bank, xs, bf.make_params())[1])
    torch.cuda.synchronize()
    for k in alone:
        assert np.array_equal(alone[k].view(np.uint8), mixed[k].view(np.uint8)), k
    x64 = xs[1].cpu().numpy().astype(np.float64)
    check_against_oracle(x64, P, alone, O.search(x64, P), "fp32", "long")

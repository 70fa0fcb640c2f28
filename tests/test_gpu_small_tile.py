"""FP32 searches too small for the 2 x 4 tile run a 1 x 1 tile (128 offsets, 32 templates): the
results equal the 2 x 4 tile's bit for bit at the edges of both, with bins that share and that
straddle template tiles, an L of an odd number of chunks, and degenerate windows."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import bfly_oracle as O  # noqa: E402
from synth import BankParams, white_noise  # noqa: E402
from tests.parity_util import check_against_oracle, to_np  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bank", [(16, 16, 512), (3, 40, 37), (5, 7, 200), (9, 33, 97), (1, 70, 16)])
@pytest.mark.parametrize("W", [1, 127, 128, 129, 513, 1537])
def test_equals_default_tile(bank, W, monkeypatch):
    from paper_1802_01685_amd import bfly as bf
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n_f0, n_fdot, L = bank
    p = BankParams(fs=float(L), L=L, n_f0=n_f0, n_fdot=n_fdot, f0_min=0.05 * L, f0_max=0.4 * L,
                   fdot_min=-0.2 * L, fdot_max=0.2 * L)
    n = W + L - 1
    x32 = white_noise(n, n).astype(np.float32)
    if W > 500:
        x32[n // 2] = np.nan
    bk = bf.bank_create(p, "fp32")
    x = torch.from_numpy(x32).cuda()
    prm = bf.make_params(t_block=1 if W % 2 else 5, hist_bins=32)
    small_items = bf.plan(bk, [n])[1]
    g = to_np(bf.search_segment(bk, x, prm))
    monkeypatch.setenv("BF_TILE", "2x4")
    assert small_items > bf.plan(bk, [n])[1] or W <= 128
    h = to_np(bf.search_segment(bk, x, prm))
    for k in g:
        assert np.array_equal(g[k].view(np.uint8), h[k].view(np.uint8)), k
    x64 = x32.astype(np.float64)
    check_against_oracle(x64, p, g, O.search(x64, p, hist_bins=32), "fp32", f"{bank}/{W}",
                         t_block=prm.t_block)

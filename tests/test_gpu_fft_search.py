"""The FFT form's search kernel at the edges of its output levels: block positions come in
levels of 1024, the last of which may be held by few waves or by a single offset.  Every offset
against the FP64 oracle, on a bank whose bins hold an odd number of templates."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import bfly_oracle as O  # noqa: E402
from synth import BankParams, white_noise  # noqa: E402
from tests.parity_util import check_against_oracle, check_hist, to_np, TOL  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [4096, 3073, 3072, 2049, 2048, 1025, 1024, 8])
@pytest.mark.parametrize("extra", [0, 1, 1500])
def test_output_levels(L, extra):
    """One whole block, one offset of a second block, and a partial second block."""
    from paper_1802_01685_amd import bfly as bf
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    p = BankParams(fs=float(L), L=L, n_f0=3, n_fdot=5, f0_min=0.05 * L, f0_max=0.3 * L,
                   fdot_min=-0.2 * L, fdot_max=0.1 * L)
    n = 8192 + extra
    x32 = white_noise(n, 100 + L + extra).astype(np.float32)
    x32[n // 2] = np.nan
    prm = bf.make_params(hist_bins=64)
    g = to_np(bf.search_segment(bf.bank_create(p, "fft"), torch.from_numpy(x32).cuda(), prm))
    x64 = x32.astype(np.float64)
    orc = O.search(x64, p, hist_bins=64)
    check_against_oracle(x64, p, g, orc, "fft", f"levels/{L}/{extra}")
    check_hist(g, orc["m"], orc["degen"], TOL["fft"], 64, 0.0, 1.0, f"levels/{L}/{extra}")

"""Tail search with some templates below their predicted bound: those alone are searched again
(the FFT form lists all their blocks, the direct forms run their tiles of 64 templates), and the
result is that of two passes bit for bit.  A margin near 1 splits the templates about evenly
between the two routes; the last tile is partial and tiles straddle the f0 bins."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from synth import BankParams, white_noise  # noqa: E402
from tests.test_gpu_tails import _tails_run  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fft", "f16f6", "f16f8", "fp32", "bf16x3", "f16x2", "fp8"])
@pytest.mark.parametrize("margin", ["0.97", "1.0", "1.02"])
def test_templates_below_their_bound(prec, margin, monkeypatch):
    from paper_1802_01685_amd import bfly as bf
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    p = BankParams(fs=512.0, L=512, n_f0=20, n_fdot=13, f0_min=20.0, f0_max=200.0,
                   fdot_min=-100.0, fdot_max=100.0)
    xs = [white_noise(n, n).astype(np.float32) for n in (9000, 2500)]
    bank = bf.bank_create(p, prec)
    want_out, want = _tails_run(bf, bank, xs, 3.5, {"BF_TAILS_TWO_PASS": "1"}, monkeypatch)
    got_out, got = _tails_run(bf, bank, xs, 3.5, {"BF_TAILS_MARGIN": margin}, monkeypatch)
    for i in range(2):
        assert want[i]["n"] == got[i]["n"] > 0
        for key in ("sigma", "tau", "k", "rho", "counts"):
            assert np.array_equal(np.asarray(want[i][key]).view(np.uint8),
                                  np.asarray(got[i][key]).view(np.uint8)), (i, key)
        for key in want_out[i]:
            assert np.array_equal(want_out[i][key].view(np.uint8),
                                  got_out[i][key].view(np.uint8)), (i, key)

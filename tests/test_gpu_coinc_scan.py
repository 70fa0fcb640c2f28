"""Coincidence over offset counts at the edges of the bucket scan's rounds (8,192 entries), with
tails at the first, the last and the rounds' border offsets, against pairwise loops."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from synth import BankParams  # noqa: E402

pytestmark = pytest.mark.gpu
P = BankParams(fs=64.0, L=16, n_f0=5, n_fdot=4, f0_min=2.0, f0_max=20.0, fdot_min=-5.0,
               fdot_max=5.0)


@pytest.mark.parametrize("W", [1, 8191, 8192, 8193, 16385, 40000])
@pytest.mark.parametrize("dtau", [0, 3, 9000])
def test_scan_rounds(W, dtau):
    from paper_1802_01685_amd import bfly as bf
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(W + dtau)
    edge = [t for t in (0, 8190, 8191, 8192, 16383, 16384, W - 1) if 0 <= t < W]
    sides = []
    for n in (150, 130):
        tau = np.concatenate([edge, rng.integers(0, W, n)]).astype(np.int32)
        k = rng.integers(0, P.K, tau.size).astype(np.int32)
        sides.append((tau, k))
    bank = bf.bank_create(P, "fp32")
    f0 = bank.grid()[0]
    cuda = [{"tau": torch.from_numpy(t).cuda(), "k": torch.from_numpy(k).cuda(),
             "n_tails": torch.tensor([t.size], device="cuda")} for t, k in sides]
    df = 4.6
    got = bf.coincidence(bank, cuda[0], cuda[1], W, dtau, df)
    (ta, ka), (tb, kb) = sides
    near = (np.abs(ta[:, None].astype(int) - tb) <= dtau) & (np.abs(f0[ka][:, None] - f0[kb]) <= df)
    assert int(got["n_pairs"]) == int(near.sum())
    for key, k, hit in (("counts_a", ka, near.any(1)), ("counts_b", kb, near.any(0))):
        want = np.bincount(k[hit] // P.n_fdot, minlength=P.n_f0)
        assert np.array_equal(got[key].cpu().numpy(), want), key

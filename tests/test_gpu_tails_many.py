"""FFT tail searches of very many short series: what is done per series around the contraction
stays small beside it."""
import pytest

torch = pytest.importorskip("torch")

from synth import BankParams  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def stages():
    """Stage times of 4,000 series of 128 samples against 64 templates of 64 taps, with a kappa so
    high and a kept bound so low that nothing is listed: the tails pass has nothing to do."""
    from paper_1802_01685_amd import bfly as bf
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    p = BankParams(fs=64.0, L=64, n_f0=8, n_fdot=8, f0_min=3.0, f0_max=25.0, fdot_min=-10.0,
                   fdot_max=10.0)
    bank = bf.bank_create(p, "fft")
    gen = torch.Generator(device="cuda").manual_seed(4)
    n, series = 128, 4000
    xs = list(torch.randn((series, n), generator=gen, device="cuda"))
    prm = bf.make_params()
    outs = [bf.alloc_outputs(bank, n, prm, "cuda") for _ in xs]
    tails = [bf.alloc_tails(bank, 16, "cuda") for _ in xs]
    ws = torch.empty(bf.tails_workspace_bytes(bank, [n] * series, prm), dtype=torch.uint8,
                     device="cuda")
    best = {}
    with pytest.MonkeyPatch.context() as m:
        m.setenv("BF_TAILS_MARGIN", "0.05")
        for i in range(6):
            bf.set_timing(i > 0)
            bf.search_tails(bank, xs, 1000.0, 16, prm, outs=outs, tails=tails, workspace=ws)
            torch.cuda.synchronize()
            bf.set_timing(False)
            if i:
                t = bf.kernel_times()[0]
                best = {k: min(v, best.get(k, v)) for k, v in t.items()}
    assert all(int(t["n_tails"]) == 0 for t in tails)
    print({k: round(v, 3) for k, v in best.items()})
    return best


def test_idle_tails_pass(stages):
    """The stage after the contraction reads each series' sums once and leaves the tails pass at
    once: less than the contraction, which transforms all 256,000 pairs.  With every work-group of
    the tails pass looking through all the series it took many times as long."""
    assert stages["finalize"] < stages["main"]


@pytest.mark.parametrize("L,series", [(64, 700), (600, 90), (4096, 9)])
def test_predictor_of_many_series(L, series):
    """A series' part of the workspace, the predictor's lag sums, cosine transform and bounds and
    the pair lists among it, comes out the same bit for bit alone and in a batch, where one
    work-group forms several or all of the series' frequencies."""
    from paper_1802_01685_amd import bfly as bf
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    p = BankParams(fs=float(L), L=L, n_f0=4, n_fdot=9, f0_min=0.05 * L, f0_max=0.4 * L,
                   fdot_min=-0.2 * L, fdot_max=0.2 * L)
    bank = bf.bank_create(p, "fft")
    gen = torch.Generator(device="cuda").manual_seed(L)
    n = 3 * L
    x = torch.randn(n, generator=gen, device="cuda")
    prm = bf.make_params()
    # 256 more series add 256 table entries (of 256 to 511 bytes each) and parts (whole 256 bytes)
    size = [bf.tails_workspace_bytes(bank, [n] * k, prm) for k in (1, 257)]
    part = (size[1] - size[0]) // 256 // 256 * 256 - 256

    def parts(k):
        ws = torch.zeros(bf.tails_workspace_bytes(bank, [n] * k, prm), dtype=torch.uint8,
                         device="cuda")
        bf.search_tails(bank, [x] * k, 3.0, 1 << 12, prm, workspace=ws)
        torch.cuda.synchronize()
        return ws[ws.numel() - k * part:].reshape(k, part)

    one = parts(1)
    assert one.any()
    assert torch.equal(parts(series), one.expand(series, part))

"""FFT searches through the server whose ticks hold more work items than its fixed grid has
work-groups (two per CU): the work-groups take further items from a counter per XCD, which every
tick's table upload clears.  Ticks of changing size replay the same graphs; every request equals a
direct search bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from synth import BankParams, white_noise  # noqa: E402
from tests.test_gpu_serving import _direct, _same, _wait  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid,lengths", [
    ((64, 6), [262000, 41000, 300, 79000, 238300, 20000]),
    ((97, 3), [262000, 256, 63000, 265000]),
    ((5, 40), [1373000, 50000, 1388900])])     # ranges no multiple of 8: 865 and 875 items
def test_ticks_beyond_the_grid(grid, lengths):
    from paper_1802_01685_amd import bfly as bf
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    p = BankParams(fs=1024.0, L=256, n_f0=grid[0], n_fdot=grid[1], f0_min=20.0, f0_max=400.0,
                   fdot_min=-300.0, fdot_max=300.0)
    bank = bf.bank_create(p, "fft")
    prm = bf.make_params(hist_bins=64)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    ranges, items = bf.plan(bank, [lengths[0]])
    assert items > 2 * cus and ranges <= grid[0]   # whole bins: the plan is the server's too
    xs = [white_noise(n, 5 + n).astype(np.float32) for n in lengths]
    want = [_direct(bf, bank, x, prm) for x in xs]
    srv = bf.server_create(bank, hbm_budget_bytes=2 << 30, max_slots=8, ticks_in_flight=2,
                           params=prm)
    for one_by_one in (True, False, False, True):
        tickets = []
        for x in xs:
            tickets.append(bf.submit(srv, x))
            if one_by_one:
                _wait(bf, srv, tickets[-1:])
        _wait(bf, srv, tickets)
        for i, t in enumerate(tickets):
            _same(bf.fetch(srv, t, lengths[i]), want[i], (grid, i, one_by_one))
    bf.server_destroy(srv)

"""GPU parity of the launch choices that depend on sizes: each kernel variant
at the edges of its range, against the CPU oracle (bit for bit)."""
import numpy as np
import pytest

from paper_1310_3437_amd import inputs as I
from tests.test_gpu_parity import run_parity
from tests.test_gpu_screen import dense_gas

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [63, 65536, 65537, 200_001])
def test_state_read_out(kmc, n):
    """Direct read-out up to 65536 particles, the gather above; on the initial
    state (an exact copy) and on a state in cell order, a ragged last wave."""
    w = I.c1_small(n=n, steps=2)
    sim = kmc.Sim(w.boxes, w.state, device="cuda:0", seed=w.seed)
    assert np.array_equal(sim.state().cpu().numpy(), w.state)
    sim.close()
    for block in (64, 1024):
        _, exact = run_parity(kmc, w, 2, block_size=block)
        assert exact


@pytest.mark.parametrize("D,dt", [(0.05, 0.005), (0.05, 0.02), (0.08, 0.02), (0.1, 0.05)])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_half_search_extra_pairs(kmc, D, dt, precision):
    """About 2, 7, 18 and 70 acceptable partners per particle: lanes beyond
    their four pairs, waves beyond their list of extra pairs (windows marked
    for the re-search), the re-search of single particles and of the whole
    step when most of them need it."""
    w = dense_gas(n=20_011, D=D, dt=dt)
    _, exact = run_parity(kmc, w, 2, precision=precision)
    assert exact

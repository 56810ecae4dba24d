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


@pytest.mark.parametrize("D,dt", [(0.05, 0.005), (0.05, 0.02), (0.1, 0.05)])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_full_search_many_partners(kmc, D, dt, precision):
    """Pruning by the best key so far: about 2, 7 and 70 acceptable partners
    per particle, one kind and two kinds of different size, every tile shape."""
    w = dense_gas(n=20_011, D=D, dt=dt)
    for tile in (0, 1, 2):
        _, exact = run_parity(kmc, w, 2, precision=precision, search_mode=kmc.KMC_SEARCH_FULL, tile=tile)
        assert exact
    w.species = np.random.default_rng(3).integers(0, 2, w.n).astype(np.uint8)
    w.radius, w.mass = (0.5 * D, 0.3 * D), (1.0, 3.0)
    _, exact = run_parity(kmc, w, 2, precision=precision, search_mode=kmc.KMC_SEARCH_FULL,
                          kinds=(w.species, w.radius, w.mass))
    assert exact


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_full_search_equal_and_near_equal_keys(kmc, precision):
    """One particle among rings of partners whose keys are equal (the smaller
    id wins) or one ulp apart, more of them than the deferred slots, so that
    the screen cannot tell them apart and the particle is searched again."""
    h, D = 0.1, 0.09
    s = np.zeros((6, 60 * 40))
    k = 0
    rng = np.random.default_rng(8)
    for c in range(60):
        # partners of a resting particle move past it along +x at the same
        # distance of closest approach, each at its own place on the circle
        cx, cy, cz = 0.15 + h * (c % 5) * 1.8, 0.15 + h * (c // 5 % 4) * 1.8, 0.15 + h * (c // 20) * 1.8
        s[0:3, k] = cx, cy, cz
        k += 1
        for e in range(39):
            a = 2 * np.pi * rng.random()
            r = 0.04 if e % 3 else 0.04 * (1.0 + 2.0 ** -52 * e)
            s[0:3, k] = cx - 0.01, cy + r * np.cos(a), cz + r * np.sin(a)
            s[3, k] = 1.0
            k += 1
    s = s[:, rng.permutation(k)]
    box = I.Box(n=k, lo=(0, 0, 0), hi=(1, 1, 1), ncell=(10, 10, 10), periodic=(True,) * 3, D2=D * D, dt=0.05)
    w = I.Workload("rings", [box], s, 1)
    for mode in (kmc.KMC_SEARCH_FULL, kmc.KMC_SEARCH_HALF):
        _, exact = run_parity(kmc, w, 1, precision=precision, search_mode=mode)
        assert exact

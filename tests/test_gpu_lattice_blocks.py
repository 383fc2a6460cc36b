"""The lattice's rescaling on both sides of 8 192 chunks (4 096 cells each), below
which a block takes one chunk and above which eight, at chunk counts per image that
these do not divide; and what it takes where every cell of a small lattice is
occupied.  Against the oracle's definition, bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2305_07454_amd import gen

from _parity import assert_exact, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cv():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_07454_amd import cvetl
    cvetl.lib()
    oracle.lib()
    return cvetl


def _lattice(n_lat, n_lon, n_t, fill, seed=1):
    rng = np.random.default_rng(seed)
    lat = np.zeros((n_t, 2, n_lat, n_lon), np.float32)
    vol = np.where(rng.random((n_t, n_lat, n_lon)) < fill, rng.integers(1, 50, (n_t, n_lat, n_lon)), 0)
    lat[:, 1] = vol
    lat[:, 0] = np.where(vol > 0, rng.uniform(-3, 40, vol.shape), 0)
    return gen.GridSpec(36.0, -95.8, 0.02, 0.02, n_lat, n_lon, gen.T0_MS, 900_000, n_t), lat


@pytest.mark.parametrize("n_lat,n_lon,n_t", [(10, 10, 8_191), (10, 10, 8_192), (17, 241, 4_096), (5, 7_373, 819), (5, 7_373, 820)])
@pytest.mark.parametrize("fill", [0.01, 1.0])
def test_normalize_blocks(cv, n_lat, n_lon, n_t, fill):
    import torch
    print(f"[lattice blocks] {n_lat}x{n_lon}x{n_t} fill={fill}", flush=True)
    grid, lat = _lattice(n_lat, n_lon, n_t, fill)
    en, emm = oracle.lattice_normalize(lat)
    t, mm = cv.cv_lattice_normalize(torch.from_numpy(lat).cuda(), grid)
    assert_exact("normalized", host(t).view(np.uint32).ravel(), en.view(np.uint32).ravel())
    assert_exact("min/max", host(mm).view(np.uint32).ravel(), emm.view(np.uint32).ravel())


def test_full_small_lattice_takes_no_chain_of_chunks(cv):
    """24 full images of 200 x 200 cells, 8 MB: three launches of about 6 us, and 50 us
    or more where a wave takes one chunk after the other."""
    import torch
    grid, lat = _lattice(200, 200, 24, 1.0)
    src = torch.from_numpy(lat).cuda()
    t = src.clone()
    cv.cv_lattice_normalize(t, grid)
    took = []
    for _ in range(9):
        t.copy_(src)
        torch.cuda.synchronize()
        cv.cv_timing_reset()
        cv.cv_timing_enable(True)
        cv.cv_lattice_normalize(t, grid)
        torch.cuda.synchronize()
        cv.cv_timing_enable(False)
        took.append(1e3 * cv.cv_timing_read("lattice_norm")[0])
    print(f"[lattice blocks] {sorted(took)[4]:.1f} us", flush=True)
    assert sorted(took)[4] < 45.0

"""The lattice normalisation at the edges of its chunks (4 096 cells, stretches
of 64), with images on and off 16-byte boundaries, and with a workspace that
holds the chunks' extrema but not their occupancy words.  Against the oracle's
definition, bit for bit."""
import ctypes

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


@pytest.mark.parametrize("n_lat,n_lon", [(1, 1), (1, 63), (64, 64), (64, 65), (3, 4096), (5, 4097), (128, 2048)])
@pytest.mark.parametrize("n_dir,n_t,offset", [(0, 1, 0), (0, 70, 1), (3, 5, 0), (2, 3, 3)])
def test_normalize_chunks(cv, n_lat, n_lon, n_dir, n_t, offset):
    import torch
    print(f"[lattice chunks] {n_lat}x{n_lon} n_dir={n_dir} n_t={n_t} offset={offset}", flush=True)
    rng = np.random.default_rng(n_lat * n_lon + n_dir)
    grid = gen.GridSpec(36.0, -95.8, 0.02, 0.02, n_lat, n_lon, gen.T0_MS, 900_000, n_t)
    D = n_dir + 1 if n_dir else 1
    cells = n_lat * n_lon
    lat = np.zeros((n_t, 2 * D, cells), np.float32)
    vol = (rng.random((n_t, D, cells)) < 0.02) * rng.integers(1, 50, (n_t, D, cells))
    vol[..., -1] = rng.integers(0, 2, (n_t, D))
    if D > 1:
        vol[:, 1] = 0  # a sector with no occupied cell
    lat[:, 1::2] = vol
    lat[:, 0::2] = np.where(vol > 0, rng.uniform(-3, 40, vol.shape), 0).astype(np.float32)
    lat = lat.reshape(n_t, 2 * D, n_lat, n_lon)
    en, emm = oracle.lattice_normalize(lat)
    need = cv._size(cv.lib().cv_lattice_normalize_workspace_size, n_t, ctypes.byref(cv._spec_struct(grid)), n_dir)
    chunks = n_t * D * -(-cells // 4096)
    parts = -(-16 * chunks // 256) * 256
    assert parts < need
    for size in (need, parts):
        buf = torch.empty(lat.size + 4, device="cuda")
        t = buf[offset:offset + lat.size].view(lat.shape)
        t.copy_(torch.from_numpy(lat))
        mm = torch.empty(4 * D, device="cuda")
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        st = cv.lib().cv_lattice_normalize(cv._ptr(t), n_t, ctypes.byref(cv._spec_struct(grid)), n_dir, cv._ptr(mm),
                                           cv._ptr(ws), size, cv._stream())
        assert st == 0
        assert_exact("normalized", host(t).view(np.uint32).ravel(), en.view(np.uint32).ravel())
        assert_exact("min/max", host(mm).view(np.uint32).ravel(), emm.view(np.uint32).ravel())

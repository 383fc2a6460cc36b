"""How many radix passes a sort ran, read from its workspace: none for whole journeys
in near order, else what the key's bits need."""
import numpy as np
import pytest

from paper_2305_07454_amd import gen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cv():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_07454_amd import cvetl
    cvetl.lib()
    return cvetl


def _files(n, per):
    rng = np.random.default_rng(n)
    j = np.arange(n) // per
    jid = rng.permutation(int(j[-1]) + 1)[j] * 5
    return (jid, gen.T0_MS + 1000 * (np.arange(n) % per), rng.uniform(36, 40, n), rng.uniform(-95, -90, n),
            np.zeros(n, np.float32))


@pytest.mark.parametrize("n", [70_000, 700_000, 2_200_000])
def test_sort_passes(cv, n):
    print(f"[sort passes] n={n}", flush=True)
    cols = _files(n, 500)
    mj = n // 500 + 10
    ws = cv.workspace(cv._size(cv.lib().cv_sort_workspace_size, n, mj))
    _, _, r = cv.cv_sort_records(cv.to_device(cols), max_journeys=mj, ws=ws)
    assert r["status"] == 0 and cv.cv_sort_passes(ws) == 0
    order = np.random.default_rng(1).permutation(n)
    _, _, r = cv.cv_sort_records(cv.to_device(tuple(c[order] for c in cols)), max_journeys=mj, ws=ws)
    bits, first = r["key_bits"], r["flags"]
    assert cv.cv_sort_passes(ws) == 1 + -(-(bits - first) // 8)
    assert cv.lib().cv_sort_passes(None, cv._ptr(ws), None) == cv.CV_ERR_INVALID_ARGUMENT
    assert cv.lib().cv_sort_passes(cv._ptr(ws), None, None) == cv.CV_ERR_INVALID_ARGUMENT

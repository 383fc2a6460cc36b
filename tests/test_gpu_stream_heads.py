"""The batch's journeys of a serving push, numbered in one pass over tiles of
4 096 sorted records: pushes at the edges of tiles, of the waves' 1 024 records and
of rows of 64, with one journey, one per record, and starts at every offset.
Journeys and their record counts equal numpy's over all pushes."""
import numpy as np
import pytest

from paper_2305_07454_amd import gen

from _parity import host, u32

pytestmark = pytest.mark.gpu

SIZES = [1, 63, 65, 1_023, 1_025, 4_095, 4_096, 4_097, 8_193, 70_001]


@pytest.fixture(scope="module")
def cv():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_07454_amd import cvetl
    cvetl.lib()
    return cvetl


@pytest.mark.parametrize("pattern", ["one", "each", "few", "mixed", "least"])
def test_journeys_of_a_push(cv, pattern):
    print(f"[stream heads] {pattern}", flush=True)
    rng = np.random.default_rng(3)
    total = sum(SIZES)
    grid = gen.GRIDS["c1"]
    st = cv.Stream(grid, total, 1 << 17, max(SIZES))
    ids = []
    for k, n in enumerate(SIZES):
        jid = dict(one=np.full(n, 5), each=rng.permutation(n) + 1_000_000 * k, few=rng.integers(0, 70, n),
                   mixed=np.where(rng.random(n) < 0.5, 9, rng.integers(0, n + 1, n)),
                   least=np.where(rng.random(n) < 0.5, -2 ** 63, rng.integers(-40, 40, n)))[pattern].astype(np.int64)
        cols = (jid, gen.T0_MS + 1000 * k + rng.integers(0, 900, n), rng.uniform(36, 40, n), rng.uniform(-95, -90, n),
                rng.integers(0, 40, n).astype(np.float32))
        st.push(cv.to_device(cols))
        ids.append(jid)
    uid, count = np.unique(np.concatenate(ids), return_counts=True)
    j = st.flush(len(uid), 1 << 17)[0]
    assert np.array_equal(host(j["journey_id"]), uid)
    assert np.array_equal(u32(host(j["n_points"])).astype(np.int64), count)

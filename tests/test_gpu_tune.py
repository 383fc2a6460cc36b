"""The tuner's sweep of tile shapes: input that says nothing of them is refused."""
import numpy as np
import pytest

from test_gpu_sort_passes import _files, cv  # noqa: F401

pytestmark = pytest.mark.gpu


def test_tuner_refuses_idle_passes(cv):  # noqa: F811
    from paper_2305_07454_amd import tune
    shape = cv.cv_tuning_get("sort_shape")
    try:
        with pytest.raises(ValueError):
            tune.sweep_sort_shapes(cv.to_device(_files(2_200_000, 500)), None, reps=1, log=lambda m: None)
        with pytest.raises(ValueError):
            tune.sweep_sort_shapes(cv.to_device(_files(70_000, 500)), None, reps=1, log=lambda m: None)
        cols = _files(2_200_000, 500)
        order = np.random.default_rng(1).permutation(len(cols[0]))
        res = tune.sweep_sort_shapes(cv.to_device(tuple(c[order] for c in cols)), None, reps=2, log=lambda m: None)
        assert len(res) == cv.cv_tuning_get("sort_shapes") and all(r["sort_ms"] > 0 for r in res)
    finally:
        cv.cv_tuning_set("sort_shape", shape)

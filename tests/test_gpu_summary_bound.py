"""The journey summary on both sides of 25 x 2^20 records, from where a wave walks 64
windows of records instead of 16: compared with numpy, exactly."""
import pytest

from test_gpu_summary_split import _case, _check, cv  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [25 << 20, (25 << 20) + 1])
@pytest.mark.parametrize("mean", [40, 5_000])
def test_summary_windows(cv, n, mean):  # noqa: F811
    import torch
    print(f"[summary bound] n={n} mean={mean}", flush=True)
    cols, feat, head = _case(mean, n, mean)
    got, r = cv.cv_journey_summary(cv.to_device(tuple(cols)), {k: torch.from_numpy(v).cuda() for k, v in feat.items()},
                                   capacity=int(head.sum()))
    _check(cv, cols, feat, head, got, r["count"])

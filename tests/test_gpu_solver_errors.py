"""What the multiple-flow-direction solvers report and return at the ends of
their inputs' range, whichever of them serves a call."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

fr = pytest.importorskip("paper_2606_12800_amd")


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    fr.load_library()
    yield


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def relnorm(a, b):
    return float(np.linalg.norm(a.astype(np.float64) - b) / np.linalg.norm(b))


@pytest.mark.parametrize("tilt,path", [(0.0, "engine"), (2.0, "row_sweep")])
def test_rain_beyond_float32(tilt, path):
    """Float64 rain that float32 water cannot hold is an error, the largest that it can is not."""
    print(f"rain beyond float32, {path}", flush=True)
    z = synth.dem(81, 70, 130, tilt=tilt)
    zt = dev(z)
    code = fr.receivers(zt, "mfd")
    rain = np.zeros(z.shape)
    low = np.unravel_index(np.argmin(z), z.shape)
    rain[low] = np.finfo(np.float32).max
    q, _, _ = fr.accumulate(code, zt, dev(rain), "mfd", torch.float32)
    assert fr.served_by() == path
    assert q[low].item() == np.finfo(np.float32).max
    rain[low] = 1e39
    with pytest.raises(fr.FlowRouteError) as e:
        fr.accumulate(code, zt, dev(rain), "mfd", torch.float32)
    assert e.value.code == fr.ERR_NONFINITE
    q, _, _ = fr.accumulate(code, zt, dev(rain), "mfd", torch.float64)
    assert q[low].item() == 1e39

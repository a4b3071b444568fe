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


@pytest.mark.parametrize("path", ["engine", "sweep"])
@pytest.mark.parametrize("rule", ["d8", "mfd"])
def test_overflow_stays_downstream(rule, path):
    """Float64 sums beyond its range are infinite there and where the values go, and no neighbour that takes nothing
    from such a cell is touched."""
    print(f"overflow {rule} {path}", flush=True)
    nr, nc = 70, 130
    # Steps: neighbours of one height exchange nothing.
    z = np.floor(12 * synth.dem(82, nr, nc, tilt=0.0)).astype(np.float32)
    x = np.ones(z.shape)
    x.ravel()[np.argsort(synth.uniform(83, synth.STREAM_NOISE, z.size))[:2000]] = 1.5e308
    zt, xt = dev(z), dev(x)
    with np.errstate(over="ignore", invalid="ignore"):
        if rule == "d8":
            code = oracle.receivers(z)
            back = oracle.adjoint_single(code, x, z=z)
        else:
            code, frac = oracle.mfd_fractions(z, 1.1)
            back = oracle.adjoint_mfd(z, x, 1.1)
            q = x.copy().ravel()
            for i in np.argsort(-z.ravel(), kind="stable"):
                for k, (dr, dc) in enumerate(oracle.OFFSETS):
                    if (int(code.ravel()[i]) >> k) & 1:
                        q[i + dr * nc + dc] += frac.reshape(-1, 8)[i, k] * q[i]
            q = q.reshape(z.shape)
    assert np.isinf(back).sum() > 20 and np.isfinite(back).sum() > 1000
    with fr.accumulate_path(path):
        got = [(fr.adjoint(dev(code), xt, zt if rule == "mfd" else None, rule), back)]
        if rule == "mfd":
            assert np.isinf(q).sum() > 20 and np.isfinite(q).sum() > 1000
            got.append((fr.accumulate(dev(code), zt, xt, "mfd", torch.float64)[0], q))
    for g, want in got:
        g = g.cpu().numpy()
        ok = np.isfinite(want)
        assert np.array_equal(np.isfinite(g), ok)
        assert not np.isnan(g).any()
        assert np.max(np.abs(g[ok] / want[ok] - 1)) <= 1e-10

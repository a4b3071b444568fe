"""Multiple flow directions on slopes at both ends of float32's range, against
the float64 oracle with the bars of test_gpu_parity.py (float32 within 1e-6 in
the 2-norm): flats at elevation 0 that the epsilon filling raises in steps of
1.4e-45, cells beside -3.4e38, drops that float32 cannot hold, and slopes of
one cell more than 2^126 apart."""
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


def terrain(kind):
    if kind == "zeros":
        return oracle.fill_depressions(np.zeros((7, 7), dtype=np.float32))
    if kind == "zeros_large":
        return oracle.fill_depressions(np.zeros((200, 300), dtype=np.float32))
    z = synth.dem(71, 150, 210, tilt=0.0)
    if kind == "integers":
        return oracle.fill_depressions(np.floor(6 * z).astype(np.float32))
    if kind == "sea":
        # Zeros below the median height: subnormal drops beside ordinary ones.
        return oracle.fill_depressions(np.where(z < np.median(z), 0, z).astype(np.float32))
    hole = synth.uniform(72, synth.STREAM_NOISE, z.size).reshape(z.shape) < 0.02
    if kind == "nodata":
        return np.where(hole, np.float32(-np.finfo(np.float32).max), z).astype(np.float32)
    # Peaks and holes whose drop is above float32's largest value.
    peak = synth.uniform(73, synth.STREAM_NOISE, z.size).reshape(z.shape) < 0.02
    z = np.where(hole, np.float32(-3e38), z)
    return np.where(peak, np.float32(3e38), z).astype(np.float32)


KINDS = ["zeros", "zeros_large", "integers", "sea", "nodata", "peaks"]


@pytest.mark.parametrize("p", [0.1, 1.1, 4.0])
@pytest.mark.parametrize("kind", KINDS)
def test_peel_slopes(kind, p):
    print(f"slopes {kind} p {p}", flush=True)
    z = terrain(kind)
    rain = synth.rain(71, *z.shape) + np.float32(2.0**-24)
    zt, rt = dev(z), dev(rain)
    with fr.accumulate_path("engine"):
        code = fr.receivers(zt, "mfd")
        q, _, mass = fr.accumulate(code, zt, rt, "mfd", torch.float32, mass=True, p=p)
        rbar = fr.adjoint(code, rt, zt, "mfd", p=p)
    assert relnorm(q.cpu().numpy(), oracle.accumulate_mfd(z, rain, p)) <= 1e-6
    total = float(rain.astype(np.float64).sum())
    assert mass[0].item() == pytest.approx(total, rel=1e-6)
    assert relnorm(rbar.cpu().numpy(), oracle.adjoint_mfd(z, rain.astype(np.float64), p)) <= 1e-6


@pytest.mark.parametrize("kind", KINDS)
def test_workflow_and_batch_slopes(kind):
    """The automatic choice, the gradient layer and a batch on the same grids."""
    print(f"workflow slopes {kind}", flush=True)
    z = terrain(kind)
    rain = synth.rain(71, *z.shape) + np.float32(2.0**-24)
    zt = dev(z)
    rt = dev(rain).requires_grad_(True)
    q = fr.FlowAccumulate.apply(rt, zt, "mfd")
    ref = oracle.accumulate_mfd(z, rain, 1.1)
    assert relnorm(q.detach().cpu().numpy(), ref) <= 1e-6
    (grad,) = torch.autograd.grad(q, rt, torch.ones_like(q))
    assert relnorm(grad.cpu().numpy(), oracle.adjoint_mfd(z, np.ones(z.shape), 1.1)) <= 1e-6
    tile = {"z": zt, "rule": "mfd", "rain": dev(rain), "q": torch.empty_like(zt)}
    fr.Batch([tile]).run()
    assert relnorm(tile["q"].cpu().numpy(), ref) <= 1e-6


def ramp(kind, nr=90, nc=200):
    """Every row lies below the one before it: no cell sends water up."""
    u = synth.uniform(74, synth.STREAM_NOISE, nr * nc).reshape(nr, nc)
    r = np.arange(nr)[:, None]
    if kind == "subnormal":
        return ((4 * (nr - r) + np.floor(3 * u)) * 2.0**-149).astype(np.float32)
    z = 0.01 * (nr - r) + 0.004 * u
    if kind == "sea":  # ordinary slopes that run out into subnormal ones
        return np.where(r < 60, z, (4 * (nr - r) + np.floor(3 * u)) * 2.0**-149).astype(np.float32)
    if kind == "nodata":
        return np.where(r == nr - 1, np.float32(-np.finfo(np.float32).max), z).astype(np.float32)
    # A drop above float32's largest value from row 39 to row 40.
    high, low = 3e38 * (1 - 1e-3 * r - 1e-4 * u), -3e38 * (1 + 1e-3 * r + 1e-4 * u)
    return np.where(r < 40, high, low).astype(np.float32)


@pytest.mark.parametrize("up", [False, True])
@pytest.mark.parametrize("p", [0.1, 1.1, 4.0])
@pytest.mark.parametrize("kind", ["subnormal", "sea", "nodata", "peaks"])
def test_row_sweep_slopes(kind, p, up):
    print(f"row sweep slopes {kind} p {p}", flush=True)
    z = ramp(kind)
    z = np.ascontiguousarray(z[::-1]) if up else z
    rain = synth.rain(75, *z.shape) + np.float32(2.0**-24)
    zt, rt = dev(z), dev(rain)
    code = fr.receivers(zt, "mfd")
    q, _, mass = fr.accumulate(code, zt, rt, "mfd", torch.float32, mass=True, p=p)
    assert fr.served_by() == "row_sweep"
    rbar = fr.adjoint(code, rt, zt, "mfd", p=p)
    assert fr.served_by() == "row_sweep"
    assert relnorm(q.cpu().numpy(), oracle.accumulate_mfd(z, rain, p)) <= 1e-6
    assert mass[0].item() == pytest.approx(float(rain.astype(np.float64).sum()), rel=1e-6)
    assert relnorm(rbar.cpu().numpy(), oracle.adjoint_mfd(z, rain.astype(np.float64), p)) <= 1e-6


@pytest.mark.parametrize("p", [0.5, 1.1, 2.0, 60.0, 3000.0])
def test_float64_fractions(p):
    """Peaks with rain 1 over three pits each (one straight, two diagonal) whose only water is the peak's share, drops
    over 40 binary orders (large powers: shares over 60): the shares against extended precision.  With u = 2^-53 a slope is within 2 u (its division
    and sqrt 2), its power within 2 p u and pow's own 2 u, their sum within 2 u of that, reciprocal and product within
    u each: 2 (2 p + 2) + 4 units, whatever the slopes' ratio."""
    n = 128
    u = synth.uniform(76, synth.STREAM_NOISE, 3 * n * n).reshape(3, n, n)
    drop = np.exp2(-40.0 * u if p < 10 else 120 - 60 * u / p).astype(np.float32)
    if p >= 10:
        drop[1:] *= np.float32(2**0.5)
    z = np.full((4 * n, 4 * n), 10, dtype=np.float32)
    z[1::4, 1::4] = 0
    at = [(0, 1), (2, 0), (2, 2)]
    for d, (r, c) in zip(drop, at):
        z[r::4, c::4] = -d
    rain = np.zeros(z.shape)
    rain[1::4, 1::4] = 1
    zt = dev(z)
    with fr.accumulate_path("engine"):
        q, _, _ = fr.accumulate(fr.receivers(zt, "mfd"), zt, dev(rain), "mfd", torch.float64, p=p)
    q = q.cpu().numpy()
    s = drop.astype(np.longdouble)
    s[1:] /= np.sqrt(np.longdouble(2))
    w = (s / s.max(0)) ** np.longdouble(p)
    want = w / w.sum(0)
    got = np.stack([q[r::4, c::4] for r, c in at]).astype(np.longdouble)
    err = float(np.max(np.abs(got - want) / want))
    print(f"p {p}: largest relative error {err:.2e}", flush=True)
    assert err <= (2 * (2 * p + 2) + 4) * 2.0**-53

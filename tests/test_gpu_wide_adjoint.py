"""Adjoint of single receivers on wide grids (from 20000 columns, of fewer than
512 rows from 28672): the wavefront sweep where water runs along the columns,
the peeling solver where it does not or where two passes leave cells, against
the oracle with the bars of test_gpu_parity.py (float32 within 1e-6 in the
2-norm, float64 within 1e-10 of the largest value)."""
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


def check(z, rule, dtype, served):
    code = oracle.receivers(z, oracle.D8 if rule == "d8" else oracle.D4)
    qbar = synth.rain(91, *z.shape).astype(np.float64) - 0.5
    want = oracle.adjoint_single(code, qbar, z=z)
    got = fr.adjoint(dev(code), dev(qbar).to(dtype), None, rule)
    assert fr.served_by() == served
    again = fr.adjoint(dev(code), dev(qbar).to(dtype), None, rule)
    assert torch.equal(got, again)
    err = got.cpu().numpy().astype(np.float64) - want
    if dtype == torch.float32:
        assert np.linalg.norm(err) <= 1e-6 * np.linalg.norm(want)
    else:
        assert np.max(np.abs(err)) <= 1e-10 * np.abs(want).max()


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("rule", ["d8", "d4"])
@pytest.mark.parametrize("nr,nc,tilt,served", [(512, 19999, 2.0, "engine"), (512, 20000, 2.0, "sweep"),
                                               (512, 20000, 0.0, "engine"), (511, 20000, 2.0, "engine"),
                                               (70, 28672, 2.0, "sweep"), (1, 28701, 2.0, "engine")])
def test_wide_adjoint(nr, nc, tilt, served, rule, dtype):
    print(f"adjoint {nr}x{nc} tilt {tilt} {rule} {dtype}", flush=True)
    z = synth.dem(91, nr, nc, tilt=tilt)
    check(z, rule, dtype, served)
    if served == "sweep":
        check(np.ascontiguousarray(z[::-1]), rule, dtype, served)


def test_wide_adjoint_with_turns():
    """A canyon that runs down, sideways and up the grid again, six times: more turns than two passes take."""
    nr, nc = 600, 20003
    z = (10.0 * np.arange(nr)[:, None] + synth.uniform(92, synth.STREAM_NOISE, nr * nc).reshape(nr, nc)).astype(np.float32)
    k = 0
    for leg in range(6):
        c = 9000 + 4 * leg
        rows = range(5, nr - 5) if leg % 2 == 0 else range(nr - 6, 4, -1)
        for r in rows:
            z[r, c] = -1 - 1e-3 * k
            k += 1
        if leg < 5:
            for s in (1, 2, 3):
                z[rows[-1], c + s] = -1 - 1e-3 * k
                k += 1
    print("adjoint of a canyon with turns", flush=True)
    check(z, "d8", torch.float32, "engine")

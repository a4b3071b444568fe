"""Receivers at the edges of their strips of rows (4 to 32 rows, by the grid's
size) and the single-receiver row sweeps at the edges of their tiles (256
columns; 16 to 256 rows, by the grid's shape), against the oracle: codes and
cell counts exactly, float32 water within 1e-6 (2-norm)."""
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


# 4 rows a strip, 8 (over 4 x 2048 rows of one strip), 16, 32; each with a remainder of 1 and less one.
@pytest.mark.parametrize("nr,nc", [(1, 1), (3, 5), (4, 1024), (5, 1025), (7, 2047), (8193, 9), (8199, 12), (16385, 7),
                                   (32769, 5), (65537, 4), (65599, 3)])
def test_receiver_strips(nr, nc):
    print(f"receivers {nr}x{nc}", flush=True)
    z = synth.dem(61, nr, nc, tilt=0.01)
    for rule, r in (("d8", oracle.D8), ("d4", oracle.D4)):
        assert np.array_equal(fr.receivers(dev(z), rule).cpu().numpy(), oracle.receivers(z, r))


# Tile heights 16 (of a few tiles), 32, 64 and 128, remainders of one row and column.
@pytest.mark.parametrize("nr,nc", [(97, 257), (1281, 3329), (2561, 2049), (5249, 1025), (8193, 257)])
def test_row_sweep_tiles(nr, nc):
    print(f"row sweeps {nr}x{nc}", flush=True)
    z = synth.dem(62, nr, nc)
    rain = synth.rain(62, nr, nc)
    code = oracle.receivers(z)
    q, cnt = oracle.accumulate_single(code, rain, z=z)
    with fr.accumulate_path("auto"):
        got, gcnt, _ = fr.accumulate(dev(code), None, dev(rain), "d8", torch.float32, counts=True)
        assert fr.served_by() == "rows"
    assert np.array_equal(gcnt.cpu().numpy().astype(np.int64), cnt.astype(np.int64))
    got = got.cpu().numpy().astype(np.float64)
    assert np.linalg.norm(got - q) / np.linalg.norm(q) <= 1e-6


@pytest.mark.parametrize("nr,nc", [(97, 257), (1281, 3329), (2561, 2049), (5249, 1025), (8193, 257)])
def test_row_sweep_tiles_per_cell(nr, nc):
    """Float32 water of single receivers: within 1e-6 in every cell, float64 within 1e-10."""
    print(f"row sweeps {nr}x{nc} per cell", flush=True)
    z = synth.dem(62, nr, nc)
    rain = synth.rain(62, nr, nc) + np.float32(2.0**-24)
    code = oracle.receivers(z)
    q, _ = oracle.accumulate_single(code, rain, z=z)
    for dtype, bar in ((torch.float32, 1e-6), (torch.float64, 1e-10)):
        got = fr.accumulate(dev(code), None, dev(rain), "d8", dtype)[0].cpu().numpy().astype(np.float64)
        assert np.max(np.abs(got - q) / q) <= bar

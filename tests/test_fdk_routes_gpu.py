"""FDK's routes against the oracle's FP64 FDK: the filter's matrix product at
the edges of its tiles (columns per wave and workgroup, rows), wider panels by
direct sums, the bricked backprojection with eight and sixteen layers, rows
loaded singly and in fours, ragged volumes that reach past the panel on every
side, windows too large for LDS, and a filter in place."""
import numpy as np
import pytest

from paper_2512_21180_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    from paper_2512_21180_amd import cbct
    return torch, cbct


def _geo(n_ang, nu, nv, nx, ny, nz, vox, off_u=0.0, off_v=0.0, width=409.6):
    return W.geometry(n_ang, nu, nv, width / nu, width / nu, nx, ny, nz, vox, off_u=off_u, off_v=off_v)


CASES = [
    _geo(5, 37, 19, 20, 18, 9, 8.0),                         # one thread per voxel
    _geo(3, 128, 21, 24, 20, 8, 6.0),                        # filter: 64 rows of 128 columns
    _geo(7, 129, 11, 24, 20, 8, 6.0, off_u=60.0),            # 32 rows, a wave with one column
    _geo(3, 257, 17, 24, 20, 8, 6.0, off_u=115.0),           # 16 rows, waves past the panel
    _geo(4, 512, 9, 24, 20, 8, 6.0, off_u=115.0),            # the widest product
    _geo(3, 515, 9, 24, 20, 8, 6.0),                         # direct sums
    _geo(300, 96, 40, 180, 165, 45, 2.5, off_u=60.0),        # bricks of eight, two window tables
    _geo(6, 101, 88, 180, 170, 83, 2.5, off_u=-60.0, off_v=30.0),   # sixteen layers, rows singly
    _geo(6, 64, 30, 200, 200, 70, 3.4),                      # volume wider than the panel all round
    _geo(6, 256, 200, 180, 170, 83, 2.0, width=150.0),       # near windows above the LDS buffer
]



@pytest.mark.parametrize("window", ["ramlak", "hann"])
@pytest.mark.parametrize("k", range(len(CASES)))
def test_fdk_routes(dev, oracle, k, window):
    torch, cbct = dev
    g = CASES[k]
    print(f"[fdk] route {k} {window}", flush=True)
    p = np.random.default_rng(k).uniform(0.0, 2.0, W.sino_shape(g)).astype(np.float32)
    geo = cbct.Geometry(g)
    work = torch.tensor(p, device="cuda")
    got = cbct.fdk(geo, work, work=work, window=window)    # the filter in place
    # FP32 sums over a row (filter) and over the angles (backprojection)
    ref = oracle.fdk_filter(g, p.astype(np.float64), window)
    f = work.double().cpu().numpy()
    assert np.linalg.norm(f - ref) <= 2e-6 * np.linalg.norm(ref)
    ref = oracle.fdk_backproject(g, ref)
    got = got.double().cpu().numpy()
    # white noise makes the interpolation's FP32 position (a few 1e-5 pixel) the largest term
    assert np.linalg.norm(got - ref) <= 3e-5 * np.linalg.norm(ref)
    again = cbct.fdk(geo, torch.tensor(p, device="cuda"), window=window)
    assert torch.equal(again, torch.from_numpy(got).float().cuda())

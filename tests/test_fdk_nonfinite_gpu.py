"""An infinite or undefined pixel in FDK's filter: the ramp's even offsets are
zero, so under Ram-Lak such a pixel leaves the columns an even distance away
finite, whichever kernel filters (up to 512 columns and enough rows the
matrix product, else direct sums); under the Hann window it takes its row.
Other rows are untouched."""
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


# (angles, columns, rows): 64, 32 and 16 rows a workgroup, and direct sums
@pytest.mark.parametrize("n_ang,nu,nv", [(64, 100, 70), (40, 201, 60), (40, 300, 40), (3, 520, 8), (2, 100, 8)])
@pytest.mark.parametrize("window", ["ramlak", "hann"])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_nonfinite_pixel(dev, oracle, n_ang, nu, nv, window, value):
    torch, cbct = dev
    print(f"[fdk] {value} in {n_ang} x {nv} x {nu}, {window}", flush=True)
    g = W.geometry(n_ang, nu, nv, 300.0 / nu, 300.0 / nu, 12, 12, 8, 5.0)
    p = np.random.default_rng(nu).uniform(0.0, 2.0, W.sino_shape(g)).astype(np.float32)
    clean = p.copy()
    at = [(0, 0, 7), (n_ang - 1, nv - 1, nu - 1), (1, nv // 2, 0), (1, nv // 2, 30)]
    for a, v, u in at:
        p[a, v, u] = value
    geo = cbct.Geometry(g)
    work = torch.tensor(p, device="cuda")
    cbct.fdk(geo, work, work=work, window=window)
    got = work.double().cpu().numpy()
    hit = {(a, v) for a, v, _ in at}
    cols = np.arange(nu)
    with np.errstate(invalid="ignore"):
        ref = oracle.fdk_filter(g, clean.astype(np.float64), window)
    bound = 1e-5 * np.abs(ref).max()
    for a in range(n_ang):
        for v in range(nv):
            if (a, v) not in hit:
                continue
            bad = np.zeros(nu, dtype=bool)
            for qa, qv, u in at:
                if (qa, qv) == (a, v):
                    bad |= (cols == u) | ((cols - u) % 2 == 1) if window == "ramlak" else True
            assert not np.isfinite(got[a, v, bad]).any()
            assert np.isfinite(got[a, v, ~bad]).all()
    # the rows without such a pixel: as without any
    keep = np.ones((n_ang, nv), dtype=bool)
    for a, v in hit:
        keep[a, v] = False
    assert np.abs(got[keep] - ref[keep]).max() <= bound

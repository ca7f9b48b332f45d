"""The scatter integration's routes against the oracle: packed densities or
the caller's volumes, records in one chunk or several, ragged pixel tiles,
rays parallel to an axis, records outside the volume, and a captured call
(which takes the route without the library's buffer)."""
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


def _inputs(nu, nv, n, nvox=(41, 41, 30)):
    g = W.geometry(4, nu, nv, 400.0 / nu, 300.0 / nv, *nvox, 6.0)
    rho = np.abs(np.random.default_rng(n).standard_normal((2,) + nvox[::-1])).astype(np.float32)
    rho[1] *= 0.1
    r = np.random.default_rng(nu)
    rec = np.zeros((n, 8), dtype=np.float32)
    rec[:, :3] = r.uniform(-0.45, 0.45, (n, 3)) * (np.array(nvox) * 6.0)
    rec[0, :2] = (30.0, 0.0)            # d_y = 0 toward the middle column of an odd panel
    rec[1, :3] = (200.0, 11.0, 7.0)     # outside, its rays pass through
    rec[2, :3] = (-200.0, 11.0, 7.0)    # outside, between volume and panel
    d = r.standard_normal((n, 3))
    rec[:, 3:6] = d / np.linalg.norm(d, axis=1, keepdims=True)
    rec[:, 6] = r.uniform(25.0, 115.0, n)
    rec[:, 7] = r.uniform(0.05, 1.0, n)
    rec[3, 7] = 0.0
    return g, rho, rec


# 41 x 41 x 30 voxels: packed from 3152 record-pixel pairs on, chunks from 32 records on
@pytest.mark.parametrize("nu,nv,n", [(9, 7, 20), (9, 7, 45), (17, 33, 6), (33, 17, 300), (8, 8, 31)])
def test_integrate_routes(dev, oracle, nu, nv, n):
    torch, cbct = dev
    print(f"[scatter] route {nu}x{nv}, {n} records", flush=True)
    g, rho, rec = _inputs(nu, nv, n)
    xs = W.scatter_tables()
    geo, X = cbct.Geometry(g), cbct.ScatterTables(xs, "cuda")
    rho_g, rec_g = torch.tensor(rho, device="cuda"), torch.tensor(rec, device="cuda")
    img = cbct.scatter_integrate(geo, rho_g, X, 0, rec_g)
    xs32 = {k: (np.asarray(v, dtype=np.float32).astype(np.float64) if k in ("mu", "icdf", "dens")
                else v) for k, v in xs.items()}
    ref = oracle.scatter_integrate(g, rho[0].astype(np.float64).ravel(),
                                   rho[1].astype(np.float64).ravel(), xs32, 0,
                                   rec.astype(np.float64))
    got = img.double().cpu().numpy()
    # FP32 marches of some 60 segments: the tolerances of the integration's parity test
    assert np.linalg.norm(got - ref) <= 1e-4 * np.linalg.norm(ref)
    assert np.max(np.abs(got - ref)) <= 5e-4 * np.max(ref)
    assert torch.equal(img, cbct.scatter_integrate(geo, rho_g, X, 0, rec_g))


def test_integrate_captured(dev):
    torch, cbct = dev
    print("[scatter] captured", flush=True)
    g, rho, rec = _inputs(33, 17, 300)
    geo, X = cbct.Geometry(g), cbct.ScatterTables(W.scatter_tables(), "cuda")
    rho_g, rec_g = torch.tensor(rho, device="cuda"), torch.tensor(rec, device="cuda")
    ref = cbct.scatter_integrate(geo, rho_g, X, 0, rec_g)
    out = torch.empty_like(ref)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        cbct.scatter_integrate(geo, rho_g, X, 0, rec_g, out=out)
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.linalg.norm(out - ref) <= 1e-5 * torch.linalg.norm(ref)
        ref2 = cbct.scatter_integrate(geo, rho_g, X, 0, rec_g)
        assert torch.equal(ref, ref2)

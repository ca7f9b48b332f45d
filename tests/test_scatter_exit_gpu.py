"""A march of the scatter integration that leaves the volume counts nothing
behind its exit face, from packed densities or from the caller's volumes (as
under stream capture)."""
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


def _records(n, seed, span):
    r = np.random.default_rng(seed)
    rec = np.zeros((n, 8), dtype=np.float32)
    rec[:, :3] = r.uniform(-1.0, 1.0, (n, 3)) * np.array(span)
    d = r.standard_normal((n, 3)) - np.array([1.5, 0.0, 0.0])
    rec[:, 3:6] = d / np.linalg.norm(d, axis=1, keepdims=True)
    rec[:, 6] = r.uniform(25.0, 115.0, n)
    rec[:, 7] = r.uniform(0.05, 1.0, n)
    return rec


def _captured(torch, cbct, geo, rho, X, rec, ref):
    out = torch.empty_like(ref)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        cbct.scatter_integrate(geo, rho, X, 0, rec, out=out)
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        yield out


def test_nothing_behind_the_exit_face(dev, oracle):
    """Rays from the middle leave through x = lo, towards the panel, and some
    through the z faces.  The faces they do not cross are dense beyond
    measure: a march that ran on past its exit into the opposite face's voxel
    would show it, however short the step."""
    torch, cbct = dev
    print("[scatter] exit face", flush=True)
    # 0.7 mm voxels: face positions that FP32 rounds
    g = W.geometry(4, 48, 48, 6.0, 6.0, 61, 61, 61, 0.7)
    rho = np.full((2, 61, 61, 61), 0.5, dtype=np.float32)
    rho[1] = 0.1
    rho[:, :, :, -1] = 1e7          # behind every record
    rec = _records(24, 3, (3.0, 3.0, 3.0))
    geo, X = cbct.Geometry(g), cbct.ScatterTables(W.scatter_tables(), "cuda")
    rho_g, rec_g = torch.tensor(rho, device="cuda"), torch.tensor(rec, device="cuda")
    xs = W.scatter_tables()
    xs32 = {k: (np.asarray(v, dtype=np.float32).astype(np.float64) if k in ("mu", "icdf", "dens")
                else v) for k, v in xs.items()}
    ref = oracle.scatter_integrate(g, rho[0].astype(np.float64).ravel(),
                                   rho[1].astype(np.float64).ravel(), xs32, 0,
                                   rec.astype(np.float64))
    img = cbct.scatter_integrate(geo, rho_g, X, 0, rec_g)
    # the tolerances of the integration's parity test
    assert np.max(np.abs(img.double().cpu().numpy() - ref)) <= 5e-4 * np.max(ref)
    for out in _captured(torch, cbct, geo, rho_g, X, rec_g, img):
        got = out.double().cpu().numpy()
        assert np.max(np.abs(got - ref)) <= 5e-4 * np.max(ref)

"""Adjoints of few bricks, whose angles are gathered in ranges: against the
oracle at angle counts around the ranges' edges (one range, two, uneven ones,
eight), and stacks, the batched call and 16-bit volumes against single calls."""
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


@pytest.mark.parametrize("n_ang", [31, 32, 33, 50, 130])
def test_ranges_of_angles(dev, oracle, n_ang):
    torch, cbct = dev
    print(f"[adjoint ranges] {n_ang} angles", flush=True)
    g = W.geometry(n_ang, 40, 30, 6.0, 6.0, 27, 30, 22, 5.0, off_u=30.0)
    geo = cbct.Geometry(g)
    y = np.random.default_rng(n_ang).standard_normal((3,) + W.sino_shape(g)).astype(np.float32)
    yg = torch.tensor(y, device="cuda")
    one = [cbct.adjoint(geo, yg[c].contiguous()) for c in range(3)]
    for c in range(3):
        ref = oracle.adjoint(g, y[c].astype(np.float64))
        got = one[c].double().cpu().numpy()
        assert np.linalg.norm(got - ref) <= 1e-5 * np.linalg.norm(ref)
    assert torch.equal(cbct.adjoint(geo, yg), torch.stack(one))
    other = cbct.Geometry(W.geometry(9, 40, 30, 6.0, 6.0, 12, 30, 22, 5.0))
    z = torch.randn(other.sino_shape, device="cuda")
    got = cbct.batch_adjoint([geo, other, geo], [yg[0].contiguous(), z, yg[1].contiguous()])
    assert torch.equal(got[0], one[0]) and torch.equal(got[2], one[1])
    assert torch.equal(got[1], cbct.adjoint(other, z))
    b = cbct.adjoint(geo, yg[2].to(torch.bfloat16).contiguous())
    wide = cbct.adjoint(geo, yg[2].to(torch.bfloat16).float().contiguous())
    assert b.dtype == torch.bfloat16 and torch.equal(b, wide.to(torch.bfloat16))


@pytest.mark.parametrize("nu,nv,width,n,vox", [(256, 64, 200.0, 37, 12.0), (256, 200, 200.0, 32, 8.0),
                                               (160, 96, 200.0, 27, 16.0), (300, 200, 300.0, 22, 10.0),
                                               (400, 32, 300.0, 39, 10.0), (256, 128, 200.0, 17, 12.0)])
def test_long_runs_and_large_windows(dev, oracle, nu, nv, width, n, vox):
    """Pixels far finer than voxels: runs of more than 32 rows per voxel, and
    panel windows of 61 to 64 KB (with the list of angles and the column
    ranges a workgroup takes up to 67 KB) or above, where the bricks give way
    to one thread per voxel."""
    torch, cbct = dev
    print(f"[adjoint] large windows {nu}x{nv}", flush=True)
    g = W.geometry(4, nu, nv, width / nu, width / nu, n, n, n // 2, vox)
    geo = cbct.Geometry(g)
    y = np.random.default_rng(nu).standard_normal(W.sino_shape(g)).astype(np.float32)
    got = cbct.adjoint(geo, torch.tensor(y, device="cuda")).double().cpu().numpy()
    ref = oracle.adjoint(g, y.astype(np.float64))
    assert np.linalg.norm(got - ref) <= 1e-5 * np.linalg.norm(ref)

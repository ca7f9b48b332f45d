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

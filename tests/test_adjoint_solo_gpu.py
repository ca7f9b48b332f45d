"""Adjoints that take every angle by itself (windows that leave no room beside
them for the list of angles, and scans of few angles) against the oracle, and
in a batch that takes another scan's angles one by one too, with its bits."""
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


def _geo(n_ang, nu, nv, nx, ny, nz, vox, off_u=0.0):
    return W.geometry(n_ang, nu, nv, 409.6 / nu, 409.6 / nu, nx, ny, nz, vox, off_u=off_u)


# name: (geometry, layers per wave)
GEOS = {
    "tall window, 16 layers": (_geo(8, 275, 200, 113, 111, 105, 4.25, 60.0), 4),
    "wide window, 8 layers": (_geo(8, 274, 235, 73, 72, 70, 5.9, 60.0), 2),
    "wide window, 4 layers": (_geo(8, 427, 260, 54, 46, 35, 5.53), 1),
    "one angle": (_geo(1, 128, 100, 60, 57, 43, 3.0), 1),
    "two angles, 16 layers": (_geo(2, 150, 110, 128, 125, 97, 2.0), 4),
    "three angles, 8 layers": (_geo(3, 128, 128, 64, 63, 61, 4.0, 20.0), 2),
}


@pytest.mark.parametrize("name", GEOS)
def test_angles_one_by_one(dev, oracle, name):
    torch, cbct = dev
    g, kv = GEOS[name]
    print(f"[adjoint solo] {name}", flush=True)
    geo = cbct.Geometry(g)
    assert geo.plan_info()["adj_kv"] == kv
    y = W.random_sino(g, 7)
    yg = torch.tensor(y, dtype=torch.float32, device="cuda")
    one = cbct.adjoint(geo, yg)
    ref = oracle.adjoint(g, yg.double().cpu().numpy())
    got = one.double().cpu().numpy()
    # the projector pair's parity bar
    assert np.linalg.norm(got - ref) <= 1e-5 * np.linalg.norm(ref)
    assert np.max(np.abs(got - ref)) <= 2e-5 * np.max(np.abs(ref))
    other = cbct.Geometry(_geo(37, 200, 150, 100, 90, 60, 4.0, 30.0))
    z = torch.tensor(W.random_sino(other.params, 8), dtype=torch.float32, device="cuda")
    a, b = cbct.batch_adjoint([geo, other], [yg, z])
    assert torch.equal(a, one)
    assert torch.equal(b, cbct.adjoint(other, z))


@pytest.mark.parametrize("channels", [2, 3, 4])
def test_channels_of_two_angles(dev, channels):
    """Channels gathered together take their angles as a group, a single call one by one."""
    torch, cbct = dev
    print(f"[adjoint solo] {channels} channels", flush=True)
    geo = cbct.Geometry(GEOS["two angles, 16 layers"][0])
    y = torch.tensor(np.random.default_rng(channels).standard_normal((channels,) + geo.sino_shape),
                     dtype=torch.float32, device="cuda")
    ref = torch.stack([cbct.adjoint(geo, y[c].contiguous()) for c in range(channels)])
    assert ref.abs().max() > 0
    assert torch.equal(cbct.adjoint(geo, y), ref)

"""Channels gathered together run in shorter bricks than a call of their own:
where a run of rows is longer than its support (coarse panel pixels, or the
panel's edge inside a brick) each run still starts at the same row, so every
channel is bitwise equal to a single call."""
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


# all with bricks of sixteen layers, at least 1024 of them, and runs of at most eight rows
GEOS = {
    "pixels of two voxels": W.geometry(24, 128, 128, 3.2, 3.2, 128, 128, 128, 1.0),
    "pixels of three voxels": W.geometry(24, 90, 50, 5.13, 5.13, 128, 128, 64, 1.07, off_v=3.3),
    "past the panel": W.geometry(31, 128, 14, 3.9, 3.9, 128, 125, 67, 1.03, off_u=40.0),
    "panel edge, fine rows": W.geometry(11, 200, 40, 1.2, 1.2, 128, 125, 67, 2.0, off_v=-9.0),
    "runs of seven": W.geometry(11, 100, 90, 2.4, 1.2, 128, 125, 67, 2.0, off_u=20.0),
    "beside the source": W.geometry(8, 50, 60, 16.0, 8.6, 128, 128, 64, 1.0, sid=103.0, sdd=400.0),
}


@pytest.mark.parametrize("name", GEOS)
def test_four_channels_equal_single_calls(dev, name):
    torch, cbct = dev
    g = GEOS[name]
    print(f"[adjoint edges] {name}", flush=True)
    geo = cbct.Geometry(g)
    p = geo.plan_info()
    assert p["adj_kv"] == 4 and p["nt_max"] <= 8
    y = torch.tensor(np.random.default_rng(5).standard_normal((4,) + W.sino_shape(g)),
                     dtype=torch.float32, device="cuda")
    ref = torch.stack([cbct.adjoint(geo, y[c].contiguous()) for c in range(4)])
    assert ref.abs().max() > 0
    got = cbct.adjoint(geo, y)
    assert torch.equal(got, ref), int((got != ref).sum())
    got = torch.stack(list(cbct.batch_adjoint([geo] * 4, [y[c].contiguous() for c in range(4)])))
    assert torch.equal(got, ref)

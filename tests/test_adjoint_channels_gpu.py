"""Channel stacks of one geometry through the adjoint: gathered in fours and
twos (the rest singly), each channel bitwise equal to a call of its own, by
cbct_adjoint on a stack and by the batched call on separate tensors; one
geometry per brick height, at sizes with partial bricks on every side."""
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


GEOS = {
    "tall bricks": W.geometry(37, 120, 70, 3.2, 3.2, 161, 157, 83, 2.0, off_u=60.0),
    "short bricks": W.geometry(9, 64, 40, 6.4, 6.4, 130, 131, 21, 3.0),
    "long runs": W.geometry(11, 300, 260, 1.0, 1.0, 120, 116, 40, 2.5),       # one channel at a time
    "few bricks": W.geometry(11, 64, 40, 6.4, 6.4, 40, 41, 30, 6.0),          # likewise
}


@pytest.mark.parametrize("name", GEOS)
@pytest.mark.parametrize("channels", [2, 3, 4, 7])
def test_channels_equal_single_calls(dev, name, channels):
    torch, cbct = dev
    g = GEOS[name]
    print(f"[adjoint channels] {name} x {channels}", flush=True)
    geo = cbct.Geometry(g)
    y = torch.tensor(np.random.default_rng(channels).standard_normal((channels,) + W.sino_shape(g)),
                     dtype=torch.float32, device="cuda")
    ref = torch.stack([cbct.adjoint(geo, y[c].contiguous()) for c in range(channels)])
    assert ref.abs().max() > 0
    assert torch.equal(cbct.adjoint(geo, y), ref)
    other = cbct.Geometry(GEOS["few bricks"])
    z = torch.randn(other.sino_shape, device="cuda")
    got = cbct.batch_adjoint([geo, other] + [geo] * (channels - 1),
                             [y[0].contiguous(), z] + [y[c].contiguous() for c in range(1, channels)])
    assert torch.equal(got[1], cbct.adjoint(other, z))
    assert torch.equal(torch.stack([got[0]] + list(got[2:])), ref)

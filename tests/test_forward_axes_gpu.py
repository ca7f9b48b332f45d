"""Projections whose rays all sample one axis (one copy of the volume is made
instead of two), both, or none of whose rays meet the volume, singly and in a
batch, against the oracle."""
import math

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


def _geo(angles, origin=(0.0, 0.0, 0.0), nu=70):
    return W.geometry(len(angles), nu, 45, 3.0, 3.0, 41, 37, 30, 2.9, angles=angles, origin=origin)


GEOS = {
    "x planes": _geo([0.0, math.pi]),
    "y planes": _geo([0.5 * math.pi]),
    "both": _geo([0.25 * math.pi, 1.0]),
    "missed": _geo([0.0, 0.5 * math.pi], origin=(0.0, 0.0, 400.0)),
}


@pytest.mark.parametrize("dtype", ["float32", "bfloat16"])
def test_axes(dev, oracle, dtype):
    torch, cbct = dev
    geos = {k: cbct.Geometry(g) for k, g in GEOS.items()}
    vols = {k: torch.tensor(W.random_volume(g, 3), dtype=getattr(torch, dtype), device="cuda")
            for k, g in GEOS.items()}
    one = {}
    for k, g in GEOS.items():
        print(f"[forward axes] {k} {dtype}", flush=True)
        assert geos[k].plan_info()["fwd_tiled"]
        one[k] = cbct.forward(geos[k], vols[k])
        ref = oracle.forward(g, vols[k].double().cpu().numpy())
        got = one[k].double().cpu().numpy()
        if k == "missed":
            assert not ref.any() and not got.any()
        else:
            # FP32 sums of 41 samples; 16-bit results are rounded once (2^-9 at most)
            tol = 2e-6 if dtype == "float32" else 2.0 ** -9
            assert np.linalg.norm(got - ref) <= tol * np.linalg.norm(ref)
    outs = cbct.batch_forward(list(geos.values()), list(vols.values()))
    for k, o in zip(GEOS, outs):
        assert torch.equal(o, one[k]), k

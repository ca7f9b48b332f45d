"""Forward plans of eight, four, two and one ray per thread: each against the
oracle, on ragged tiles of both widths, and the same bits in a batch of all."""
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
    8: W.geometry(40, 257, 230, 1.0, 1.0, 40, 37, 33, 4.0, off_u=11.0),
    4: W.geometry(7, 90, 67, 3.0, 3.0, 41, 37, 33, 4.0),
    2: W.geometry(8, 67, 49, 4.0, 4.0, 60, 57, 43, 2.0),
    1: W.geometry(8, 67, 49, 4.0, 8.0, 60, 57, 43, 2.2),
}


@pytest.mark.parametrize("dtype", ["float32", "float16"])
def test_rays_per_thread(dev, oracle, dtype):
    torch, cbct = dev
    geos = [cbct.Geometry(g) for g in GEOS.values()]
    vols = [torch.tensor(W.random_volume(g, 5), dtype=getattr(torch, dtype), device="cuda")
            for g in GEOS.values()]
    one = []
    for (r, g), geo, x in zip(GEOS.items(), geos, vols):
        print(f"[forward rays] {r} {dtype}", flush=True)
        assert geo.plan_info()["fwd_tiled"] and geo.plan_info()["rays_per_thread"] == r
        one.append(cbct.forward(geo, x))
        ref = oracle.forward(g, x.double().cpu().numpy())
        got = one[-1].double().cpu().numpy()
        # FP32 sums of 60 samples; 16-bit results are rounded once (2^-12 at most)
        tol = 2e-6 if dtype == "float32" else 2.0 ** -11
        assert np.linalg.norm(got - ref) <= tol * np.linalg.norm(ref)
    for a, b in zip(one, cbct.batch_forward(geos, vols)):
        assert torch.equal(a, b)

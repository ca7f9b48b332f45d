"""Poisson counts of the polychromatic simulator at bin numbers around the
workgroup sizes, ragged element counts, and means over the sampler's whole
range (zero, inversion, the edge at ten, large means, its largest): equal to
the oracle's counts on the same line integrals."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    from paper_2512_21180_amd import cbct
    return torch, cbct


@pytest.mark.parametrize("bins,n,nv,nu", [(1, 3, 5, 13), (16, 5, 7, 31), (17, 5, 7, 31), (32, 4, 8, 32)])
def test_counts_over_bins_and_means(dev, oracle, bins, n, nv, nu):
    torch, cbct = dev
    print(f"[poly] {bins} bins", flush=True)
    r = np.random.default_rng(bins)
    pw = r.uniform(0.0, 12.0, (n, nv, nu)).astype(np.float32)
    pb = r.uniform(0.0, 3.0, (n, nv, nu)).astype(np.float32)
    pw[0, 0, :4] = (0.0, 800.0, 740.0, -2.0)       # transparent, opaque, denormal means, gain
    i0 = np.exp(r.uniform(np.log(1.0), np.log(3e5), (bins, nv, nu))).astype(np.float32)
    i0[0, 0, 4:9] = (0.0, 10.0, 10.000001, 9.999999, 5e7)
    pw[0, 0, 4:9], pb[0, 0, 4:9] = 0.0, 0.0
    mw, mb = r.uniform(0.2, 1.0, bins), r.uniform(0.2, 1.0, bins)
    resp = r.uniform(0.0, 20.0, bins)
    y, s, c = cbct.sim_poly(torch.tensor(pw, device="cuda"), torch.tensor(pb, device="cuda"), mw, mb,
                            resp, torch.tensor(i0, device="cuda"), 99, 3, signal=True, counts=True)
    yr, sr, cr = oracle.sim_poly(pw.astype(np.float64), pb.astype(np.float64), mw, mb, resp,
                                 i0.astype(np.float64), 99, 3)
    assert int((c.cpu().numpy() != cr).sum()) == 0
    np.testing.assert_allclose(s.cpu().numpy().astype(np.float64), sr, rtol=2.4e-7, atol=0)

"""Kernels at the edges of their tiles and ranges, GPU (C-ABI) against the oracle.

Tolerances: float64 sums of at most 2^21 terms of one sign or of a transform's outputs, compared to
1e-12 relative (eps x sqrt(terms) is 3e-13); integers and counts exactly."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import field as fld, power  # noqa: E402
from paper_0906_4548_amd import inputs  # noqa: E402
from tests.gpu_common import oracle_params, gpu_params, rel_l2, to_dev  # noqa: E402


@pytest.fixture(scope="module")
def dgp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0906_4548_amd import dgp as mod
    mod._lib.load()
    return mod


# one bin, a bin count that is no multiple of a wavefront, and the largest; meshes from one row tile
# (8^3: 40 rows in a 256-row tile) to several tiles per workgroup
@pytest.mark.parametrize("n,batch,nbins", [(8, 3, 64), (8, 1, 128), (16, 2, 1), (32, 1, 65), (64, 1, 128), (128, 2, 7)])
def test_power_spectrum_bins_and_gradient(dgp, n, batch, nbins):
    box, op = 2.0 * n, oracle_params()
    f = np.stack([inputs.gaussian_field(n, box, 70 + b, slope=-1.0) for b in range(batch)])
    g = np.random.default_rng(n + nbins).standard_normal((batch, nbins))
    with dgp.Plan(n, box, batch=batch) as plan:
        p = gpu_params(dgp)
        pk, cnt = plan.power_spectrum(p, to_dev(f), nbins=nbins)
        pc, _ = plan.power_spectrum(p, to_dev(f), of_c=True, nbins=nbins)
        gf = torch.zeros((batch, n, n, n), dtype=torch.float64, device="cuda")
        plan.power_spectrum_backward(p, to_dev(f), g, gf)
    for b in range(batch):
        ref, cnt_ref, _ = power.power_spectrum(f[b], box, nbins)
        refc, _, _ = power.power_spectrum(fld.c_from_u(f[b], box, op), box, nbins)
        assert np.array_equal(cnt, cnt_ref)
        assert np.allclose(pk[b], ref, rtol=1e-12, atol=0) and np.allclose(pc[b], refc, rtol=1e-12, atol=0)
        assert rel_l2(gf[b].cpu().numpy(), power.power_spectrum_grad(f[b], g[b], box, nbins)) <= 1e-12

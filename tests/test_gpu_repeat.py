"""A solve's answer does not depend on what its plan solved before (GPU).

The plan learns how many passes to enqueue before the host looks at the control blocks; the passes'
results, residuals and decisions are the same wherever those looks fall."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_0906_4548_amd import inputs  # noqa: E402
from tests.gpu_common import gpu_params, to_dev  # noqa: E402


@pytest.fixture(scope="module")
def dgp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0906_4548_amd import dgp as mod
    mod._lib.load()
    return mod


# every mesh size up to 128^3 (the pass is decided by the next pass's launch up to 64^3, by a launch of
# its own above and at the end of a chunk), both precisions, chunks cut differently by check_every
@pytest.mark.parametrize("n,batch", [(8, 3), (16, 2), (32, 1), (64, 1), (64, 3), (128, 1)])
@pytest.mark.parametrize("prec", [0, 1])
def test_solve_bits_do_not_depend_on_the_chunks(dgp, n, batch, prec):
    box = 2.0 * n
    d = to_dev(np.stack([inputs.lognormal_delta(n, box, 0.9, 20 + b) for b in range(batch)]))
    runs = []
    with dgp.Plan(n, box, batch=batch, precision=prec) as plan:
        # a first solve (chunks of two, then by the observed convergence), a second one (the learned
        # count), one after a solve of another length, one with a host look after every pass
        for check_every in (4, 4, None, 4, 1):
            u = torch.zeros_like(d)
            if check_every is None:
                # (a shorter float32 phase would be cut short by the next solve's first chunk)
                plan.solve_field(gpu_params(dgp, tol=1e-2 if prec == 0 else 1e-12), d, u)
                continue
            _, info = plan.solve_field(gpu_params(dgp, tol=1e-10, check_every=check_every), d, u)
            hist = [plan.history(b) for b in range(batch)]
            runs.append((u.cpu().numpy(), info, hist))
    u0, i0, h0 = runs[0]
    for u, info, hist in runs[1:]:
        for b in range(batch):
            assert np.array_equal(u[b], u0[b])
            for k in ("status", "iters", "resid", "resid_min", "eps", "bad_fraction", "mean_u"):
                assert info[b][k] == i0[b][k], (k, info[b][k], i0[b][k])
            if prec == 0:
                assert info[b]["passes"] == i0[b]["passes"]
            for x, y in zip(hist[b], h0[b]):
                assert np.array_equal(x, y)

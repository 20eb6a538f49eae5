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


def _sort_loads():
    """(name, mesh, positions) of loads around the tile sort's rules, 2^18 to 2^20 particles."""
    rng = np.random.default_rng(5)
    np_ = 2 ** 20 + 37
    lat = inputs.zeldovich_load(104, 128.0, 8)[0]
    yield "small mesh", 64, lat[:, :np_].copy()
    yield "lattice order, ragged", 128, 2.0 * lat[:, :np_]
    yield "float32", 128, (2.0 * lat[:, :np_]).astype(np.float32)
    yield "random order", 128, rng.uniform(0.0, 256.0, (3, np_))
    # compact chunks deposited directly beside sorted ones
    mixed = 2.0 * lat[:, :np_]
    mixed[:, :300000] = 3.0 + rng.uniform(0.0, 8.0, (3, 300000))
    yield "compact and spread chunks", 128, mixed
    # one tile holding most particles (several work items), over the periodic corner, in random order
    dense = (rng.normal(0.0, 6.0, (3, np_)) + 1.0) % 256.0
    yield "dense periodic corner", 128, np.where(dense >= 256.0, 0.0, dense)
    yield "just below the rule", 128, 2.0 * lat[:, :2 ** 18 - 1]
    yield "at the rule", 128, 2.0 * lat[:, :2 ** 18]


@pytest.mark.timeout(600)
def test_deposit_tile_sort_bit_exact(dgp):
    from oracle import pm
    for name, n, pos in _sort_loads():
        print(name, flush=True)
        box = 2.0 * n
        ref = pm.cic_deposit_fixed(pos.astype(np.float64), n, box)
        with dgp.Plan(n, box) as plan:
            g = torch.zeros(n ** 3, dtype=torch.int64, device="cuda")
            for _ in range(2):   # the second pass over a workspace that the first one used
                plan.deposit(to_dev(pos, torch.float32 if pos.dtype == np.float32 else torch.float64), g)
            assert np.array_equal(g.cpu().numpy().reshape(n, n, n), ref), name


# both sides of the chunk rule (2^18 particles), ragged, compact and spread chunks
@pytest.mark.parametrize("np_,block,nc", [(2 ** 18 - 1, 8, 3), (2 ** 18 + 13, 8, 3), (2 ** 18 + 13, 0, 2), (300, 0, 1)])
def test_interp_mesh_gradient_chunks(dgp, np_, block, nc):
    from oracle import adjoint
    n, box = 32, 64.0
    side = 72
    pos = inputs.zeldovich_load(side, box, 12, rms_disp=0.8, block=block)[0][:, :np_].copy()
    g = np.random.default_rng(np_).standard_normal((nc, np_))
    mesh = np.random.default_rng(3).standard_normal((nc, n, n, n))
    _, ref = adjoint.interp_backward(mesh, pos, g, box)
    with dgp.Plan(n, box) as plan:
        gm = torch.zeros((nc, n, n, n), dtype=torch.float64, device="cuda")
        plan.interp_backward(None, to_dev(pos), to_dev(g), None, gm)
    assert rel_l2(gm.cpu().numpy(), ref) <= 1e-12


# batches whose elements share a workgroup's plane or leave it ragged; every element alone runs the same
# arithmetic (float64: last-place rounding; mixed: the float64 polish from float32 iterates that agree)
@pytest.mark.parametrize("n,batch", [(8, 3), (16, 11), (32, 7), (64, 3), (128, 2)])
@pytest.mark.parametrize("prec", [0, 1])
def test_solve_batch_elements_and_source_mean(dgp, n, batch, prec):
    box, op = 2.0 * n, oracle_params()
    d = np.stack([inputs.lognormal_delta(n, box, 0.8, 40 + b) for b in range(batch)])
    p = gpu_params(dgp, tol=1e-10)
    u = torch.zeros((batch, n, n, n), dtype=torch.float64, device="cuda")
    with dgp.Plan(n, box, batch=batch, precision=prec) as plan:
        _, info = plan.solve_field(p, to_dev(d), u)
    for b in range(batch):
        u1 = torch.zeros((1, n, n, n), dtype=torch.float64, device="cuda")
        with dgp.Plan(n, box, precision=prec) as plan:
            _, one = plan.solve_field(p, to_dev(d[b:b + 1]), u1)
        assert one[0]["passes"] == info[b]["passes"] and one[0]["status"] == info[b]["status"]
        assert rel_l2(u[b].cpu().numpy(), u1[0].cpu().numpy()) <= (1e-12 if prec == 0 else 1e-9)
        _, ref = fld.solve(d[b], box, op, fixed_iters=0)
        assert abs(info[b]["eps"] - ref.eps) <= 1e-12 * ref.eps


# the row groups of 512^3: raw transforms and the power spectrum against torch, the solve's own fields
# through their copies in and out (the same iterates from a warm start; a rolled input, also spherical)
def test_row_groups_512(dgp):
    n, box = 512, 1024.0
    gen = torch.Generator(device="cuda").manual_seed(5)
    f = torch.randn((n, n, n), dtype=torch.float64, device="cuda", generator=gen) * 0.1
    ref = torch.fft.rfftn(f, dim=(1, 2, 0))
    spec = torch.zeros((n // 2 + 1, n, n), dtype=torch.complex128, device="cuda")

    def rel(x, y):
        return float((x - y).norm() / y.norm())
    for prec, tol in ((0, 1e-13), (1, 1e-5)):
        with dgp.Plan(n, box, precision=prec) as plan:
            plan.fft_forward(f, spec)
            assert rel(spec, ref) <= tol
            back = torch.zeros_like(f)
            plan.fft_inverse(spec, back)
            assert rel(back, f) <= tol
    w = torch.full((n // 2 + 1, 1, 1), 2.0, dtype=torch.float64, device="cuda")
    w[0] = w[-1] = 1.0
    m = torch.fft.fftfreq(n, 1.0 / n, dtype=torch.float64, device="cuda")
    k2 = m[:n // 2 + 1, None, None] ** 2 + m[None, :, None] ** 2 + m[None, None, :] ** 2
    total = float((w * ref.abs() ** 2 * ((k2 >= 1) & (k2 < (n // 2) ** (12 / 7)))).sum())   # six bins of seven
    del ref, spec, k2, w
    with dgp.Plan(n, box) as plan:
        pk, cnt = plan.power_spectrum(gpu_params(dgp), f, nbins=7)
        got = float(np.sum((pk * cnt)[..., :6])) * n ** 6 / box ** 3
        assert abs(got - total) <= 1e-11 * total
        u2, u1 = torch.zeros_like(f), torch.zeros_like(f)
        plan.solve_field(gpu_params(dgp, tol=0.0, max_iter=2), f, u2)
        plan.solve_field(gpu_params(dgp, tol=0.0, max_iter=1), f, u1)
        plan.solve_field(gpu_params(dgp, tol=0.0, max_iter=1, init=dgp.INIT_WARM), f, u1)
        assert rel(u1, u2) <= 1e-12
        roll = ((1, 6, 3), (0, 1, 2))
        fr = f.roll(*roll).contiguous()
        for kw in ({"tol": 0.0, "max_iter": 2}, {"spherical": 1, "init": dgp.INIT_ZERO}):
            plan.solve_field(gpu_params(dgp, **kw), f, u1)
            plan.solve_field(gpu_params(dgp, **kw), fr, u2)
            assert rel(u2, u1.roll(*roll)) <= 1e-12


# gathers and the deposit's adjoint by chunks: compact (staged in LDS) and spread (direct) ones, a ragged
# last chunk, one particle
@pytest.mark.parametrize("np_,block", [(1, 0), (255, 8), (2 ** 14 + 3, 8), (2 ** 14 + 3, 0)])
@pytest.mark.parametrize("fp32", [False, True])
def test_gather_chunks(dgp, np_, block, fp32):
    from oracle import adjoint, pm
    n, box, side = 32, 64.0, 32
    pos = inputs.zeldovich_load(side, box, 12, rms_disp=0.8, block=block)[0][:, :np_].copy()
    pos = pos.astype(np.float32) if fp32 else pos
    ref_pos = pos.astype(np.float64)
    g = np.random.default_rng(np_).standard_normal((3, np_))
    mesh = np.random.default_rng(3).standard_normal((3, n, n, n))
    with dgp.Plan(n, box) as plan:
        tp = torch.from_numpy(pos).cuda()
        out = torch.zeros((3, np_), dtype=torch.float64, device="cuda")
        plan.interp(to_dev(mesh), tp, out)
        gp = torch.zeros((3, np_), dtype=torch.float64, device="cuda")
        plan.interp_backward(to_dev(mesh), tp, to_dev(g), gp, None)
    ref = pm.cic_interpolate(mesh, ref_pos, box)
    refp, _ = adjoint.interp_backward(mesh, ref_pos, g, box)
    assert rel_l2(out.cpu().numpy(), ref) <= 1e-12
    assert rel_l2(gp.cpu().numpy(), refp) <= 1e-12

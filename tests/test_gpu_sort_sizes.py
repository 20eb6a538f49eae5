"""The deposit's tile sort over its range of meshes, chunks and orders (GPU against the oracle, bit for bit).

test_gpu_edges.py covers 128^3; here are the tile grids of 256^3 and 512^3 (whose chunks hold 2048
particles), chunks of more tiles than a workgroup counts beside sorted ones, a non-finite position in a
sorted chunk, graph replays, and the entry point without a plan, which never sorts."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import pm  # noqa: E402
from paper_0906_4548_amd import inputs  # noqa: E402
from tests.gpu_common import to_dev  # noqa: E402


@pytest.fixture(scope="module")
def dgp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0906_4548_amd import dgp as mod
    mod._lib.load()
    return mod


def _dtype(fp32):
    return torch.float32 if fp32 else torch.float64


def _lattice(n, np_):
    """np_ particles of a lattice-order Zel'dovich load, the box of an n^3 mesh of cell 2."""
    side = int(np.ceil(np_ ** (1 / 3)))
    return inputs.zeldovich_load(side, 2.0 * n, 31, rms_disp=2.5)[0][:, :np_].copy()


def _loads(n):
    rng = np.random.default_rng(n)
    box, np_ = 2.0 * n, 2 ** 18 + 4099
    yield "lattice", _lattice(n, np_)
    yield "random", rng.uniform(0.0, box, (3, np_))
    # rows along axis 2 that cross the periodic corner of axes 0 and 1
    rows = np.stack([rng.normal(0.0, 3.0, np_), rng.normal(0.0, 3.0, np_), rng.uniform(0.0, box, np_)]) % box
    yield "corner rows", np.where(rows >= box, 0.0, rows)
    mixed = _lattice(n, np_)
    mixed[:, :100000] = rng.uniform(0.0, box, (3, 100000))          # chunks over the whole mesh
    mixed[:, 100000:160000] = 5.0 + rng.uniform(0.0, 9.0, (3, 60000))   # compact chunks
    yield "random, compact and lattice chunks", mixed


@pytest.mark.timeout(600)
@pytest.mark.parametrize("n", [256, 512])
@pytest.mark.parametrize("fp32", [False, True])
def test_tile_sort_large_meshes_bit_exact(dgp, n, fp32):
    box = 2.0 * n
    with dgp.Plan(n, box) as plan:
        g = torch.zeros(n ** 3, dtype=torch.int64, device="cuda")
        for name, pos in _loads(n):
            print(n, fp32, name, flush=True)
            pos = pos.astype(np.float32 if fp32 else np.float64)
            pos = np.where(pos >= box, 0.0, pos).astype(pos.dtype)
            ref = pm.cic_deposit_fixed(pos, n, box).reshape(-1)
            plan.deposit(to_dev(pos, _dtype(fp32)), g)
            idx = torch.nonzero(g).reshape(-1)
            vals = g[idx].cpu().numpy()
            ref_idx = np.flatnonzero(ref)
            assert np.array_equal(idx.cpu().numpy(), ref_idx), name
            assert np.array_equal(vals, ref[ref_idx]), name
            del idx, ref


@pytest.mark.parametrize("fp32", [False, True])
def test_nonfinite_position_in_a_sorted_chunk(dgp, fp32):
    n, box = 128, 256.0
    pos = _lattice(n, 2 ** 18 + 5).astype(np.float32 if fp32 else np.float64)
    with dgp.Plan(n, box) as plan:
        d = torch.zeros(n ** 3, dtype=torch.float64, device="cuda")
        for bad in (np.nan, np.inf):
            broken = pos.copy()
            broken[2, 70001] = bad
            plan.deposit(to_dev(broken, _dtype(fp32)), None, d)
            assert bool(torch.all(torch.isnan(d)))
        plan.deposit(to_dev(pos, _dtype(fp32)), None, d)   # the flag is the call's own
        assert bool(torch.all(torch.isfinite(d)))


def test_sorted_deposit_equals_the_call_without_a_plan(dgp):
    n, box = 128, 256.0
    pos = to_dev(_lattice(n, 2 ** 19 + 77))
    g0, g1 = (torch.zeros(n ** 3, dtype=torch.int64, device="cuda") for _ in range(2))
    d0, d1 = (torch.zeros(n ** 3, dtype=torch.float64, device="cuda") for _ in range(2))
    with dgp.Plan(n, box) as plan:
        plan.deposit(pos, g0, d0)
        torch.cuda.synchronize()
    p = [ctypes.c_void_p(t.data_ptr()) for t in (pos, g1, d1)]
    assert dgp._lib.load().dgp_deposit_noalloc(n, box, p[0], 0, pos.shape[1], p[1], p[2], dgp._stream()) == 0
    torch.cuda.synchronize()
    assert torch.equal(g0, g1) and torch.equal(d0, d1)


def test_sorted_deposit_in_a_graph(dgp):
    """Replays of a captured deposit on changing positions, with eager work in between."""
    n, box = 128, 256.0
    pos = to_dev(_lattice(n, 2 ** 18 + 1000))
    shifts = [0.0, 17.3, 101.9, 0.4]
    g, ge = (torch.zeros(n ** 3, dtype=torch.int64, device="cuda") for _ in range(2))
    d, de = (torch.zeros(n ** 3, dtype=torch.float64, device="cuda") for _ in range(2))
    buf = pos.clone()
    with dgp.Plan(n, box) as plan, dgp.Plan(n, box) as eager:
        plan.deposit(buf, g, d)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            plan.deposit(buf, g, d)
        for s in shifts:
            x = torch.remainder(pos + s, box)
            buf.copy_(torch.where(x >= box, x - box, x))
            graph.replay()
            eager.deposit(buf, ge, de)
            torch.cuda.synchronize()
            assert torch.equal(g, ge) and torch.equal(d, de)
            assert int(g.sum()) > 0

"""GPU: the matrix passes with several wavefronts per slice (images of few
slices) against the one-wave walk bit for bit, and against numpy within the
rounding bound of an ascending sum; sizes around the rule's lines, ragged and
empty last slices, rows of 1 to some hundred entries, 16-bit and 32-bit
column indices, shared offsets with and without clamping."""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def amg():
    import paper_2511_21268_amd as m
    assert torch.cuda.is_available()
    m.lib()
    return m


def _arrays(A):
    A = sp.csr_matrix(A)
    A.sort_indices()
    return A.indptr.astype(np.int64), A.indices.astype(np.int32), A.data.astype(np.float64)


def _random_spd(n, per_row, seed, far=False):
    """Ragged rows: random symmetric couplings over a dominant diagonal; far:
    the first and last unknowns coupled (a column gap of n - 1)."""
    r = np.random.default_rng(seed)
    m = n * per_row // 2
    i, j = r.integers(0, n, m), r.integers(0, n, m)
    i[: m // 4] = i[: m // 4] // 7          # some rows much longer than others
    if far:
        i, j = np.append(i, 0), np.append(j, n - 1)
    C = sp.coo_matrix((r.uniform(-1, -0.1, len(i)), (i, j)), shape=(n, n)).tocsr()
    C = C + C.T
    C.setdiag(0.0)
    C.eliminate_zeros()
    return C + sp.diags(np.asarray(abs(C).sum(axis=1)).ravel() + 1.0)


CASES = {
    "stencil-2d-p2-1slice": ("iga", 2, 2, 7), "stencil-2d-p2": ("iga", 2, 2, 32), "stencil-3d-p3": ("iga", 3, 3, 16),
    "stencil-3d-p4-last-slice-1-row": ("iga", 3, 4, 15), "stencil-3d-p2-255": ("iga", 3, 2, 25),
    "ragged-1": ("rnd", 1, 0, 0), "ragged-65": ("rnd", 65, 9, 1), "ragged-16383": ("rnd", 16383, 40, 2),
    "ragged-16385": ("rnd", 16385, 40, 3), "ragged-long": ("rnd", 700, 500, 4), "far-70000": ("far", 70000, 24, 5),
}


@pytest.mark.parametrize("name", CASES)
def test_split_pass_equals_one_wave(amg, name):
    kind, a, b, c = CASES[name]
    print(f"case split {name}", flush=True)
    if kind == "iga":
        rp, ci, v, _ = amg.iga_poisson(a, b, c, want_F=False)
        K = sp.csr_matrix((v, ci, rp), shape=(len(rp) - 1, len(rp) - 1))
    else:
        K = _random_spd(a, b, c, far=kind == "far")
    n = K.shape[0]
    x = np.random.default_rng(9).standard_normal(n)
    ctx = amg.Context(*_arrays(K))
    y = ctx.spmv(torch.from_numpy(x).cuda()).cpu().numpy()
    # an ascending FMA chain of w terms: |error| <= w u / (1 - w u) sum |k_ij x_j|
    w = int(np.diff(K.indptr).max())
    u = 2.0 ** -53
    bound = 2.0 * (w + 1) * u * (abs(K) @ np.abs(x))     # twice: numpy's own sum rounds too
    assert np.all(np.abs(y - K @ x) <= bound)
    # the same rows in an image of 1,200 slices or more, one wave per slice:
    # copies of K ending in whole slices, each with a chain of 1 to 64 more
    # unknowns that joins it to the next copy's (so that it coarsens)
    pad = 64 - n % 64
    chain = sp.diags([np.full(pad, 3.0), np.full(pad - 1, -1.0), np.full(pad - 1, -1.0)], [0, -1, 1])
    Kp = sp.block_diag([K, chain], format="lil")
    Kp[n - 1, n] = Kp[n, n - 1] = -0.5
    Kp = Kp.tocsr()
    m = n + pad
    times = -(-1200 * 64 // m)
    i = np.arange(1, times) * m
    link = sp.coo_matrix((np.full(2 * len(i), -0.25), (np.append(i - 1, i + n), np.append(i + n, i - 1))),
                         shape=(m * times, m * times))
    xp = np.append(x, np.ones(pad))
    small = amg.Context(*_arrays(Kp)).spmv(torch.from_numpy(xp).cuda()).cpu().numpy()[:n]
    big = amg.Context(*_arrays(sp.block_diag([Kp] * times, format="csr") + link))
    yb = big.spmv(torch.from_numpy(np.tile(xp, times)).cuda()).cpu().numpy()
    for k in (0, times // 2, times - 1):
        assert np.array_equal(yb[k * m:k * m + n], small), k


@pytest.mark.parametrize("n", [64, 64 * 255, 64 * 256, 64 * 1199, 64 * 1200])
def test_split_rule_lines(amg, n):
    """Both sides of every line of the rule, on a banded matrix whose result is
    exact in floating point (small integers)."""
    print(f"case split rule n={n}", flush=True)
    band = [np.full(n - k, -1.0) for k in range(1, 41)]
    K = sp.diags([np.full(n, 100.0)] + band + band, [0] + list(range(1, 41)) + list(range(-1, -41, -1)), format="csr")
    x = np.random.default_rng(n).integers(-50, 50, n).astype(np.float64)
    ctx = amg.Context(*_arrays(K))
    y = ctx.spmv(torch.from_numpy(x).cuda()).cpu().numpy()
    assert np.array_equal(y, K @ x)


@pytest.mark.parametrize("d,p,n", [(3, 3, 14), (3, 2, 33), (2, 3, 61), (3, 5, 9), (3, 3, 40)])
@pytest.mark.parametrize("fp32", [0, 1])
def test_block_split_equals_one_lane(amg, d, p, n, fp32):
    """The block V-cycle on the lanes-per-row images (one wave or several per
    slice, loads ahead) against the one-lane-per-row kernels: the V-cycle has the
    same bits, so the first iterate u = alpha z differs by alpha's dots only."""
    print(f"case block split d={d} p={p} n={n} fp32={fp32}", flush=True)
    rp, ci, v, _ = amg.iga_poisson(d, p, n, want_F=False)
    ctx = amg.Context(rp, ci, v, nrhs=16, itmax=1, **(dict(vcycle_fp32=1, krylov=1) if fp32 else {}))
    lpr, threads = ctx.batched_variant()
    F = torch.from_numpy(np.random.default_rng(n).standard_normal((16, len(rp) - 1))).cuda().t()
    got = ctx.solve_batched(F)["U"]
    ctx.set_batched_variant(1, 256)
    ref = ctx.solve_batched(F)["U"]
    print(f"  lanes per row {lpr}", flush=True)
    # two sums of N products each: 2 N u on sums of absolute terms at most about
    # ten times their value
    assert torch.linalg.norm(got - ref) <= 20 * len(rp) * 2.0 ** -53 * torch.linalg.norm(ref)

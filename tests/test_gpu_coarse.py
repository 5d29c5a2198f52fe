"""GPU: the coarsest-level solve (products with the inverse factor in four
segments per row) at the edges of its segments, row groups and tiles, on
single-level systems, whose V-cycle is that solve; the restriction inside the kernel
and the 16-column kernel on a two-level system, bit for bit."""
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


def _band(n):
    """Diagonally dominant band matrix: eigenvalues in [1, 7]."""
    k = min(3, n - 1)
    off = [np.full(n - t, -0.5) for t in range(1, k + 1)]
    K = sp.diags([np.full(n, 4.0)] + off + off, [0] + list(range(1, k + 1)) + list(range(-1, -k - 1, -1))).tocsr()
    K.sort_indices()
    return K


def _context(amg, K, **kw):
    return amg.Context(K.indptr.astype(np.int64), K.indices.astype(np.int32), K.data, **kw)


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 63, 64, 65, 255, 256, 257, 1025, 2000])
def test_single_level_solve(amg, n):
    print(f"case coarse n={n}", flush=True)
    K = _band(n)
    ctx = _context(amg, K, max_coarse=2000)
    assert ctx.nlevels == 1
    F = np.random.default_rng(n).standard_normal((3, n))
    z = [ctx.vcycle(torch.from_numpy(f).cuda()).cpu().numpy() for f in F]
    # the factor's, the inverse's and the product's errors: a few n u cond, cond 7
    for f, x in zip(F, z):
        ref = np.linalg.solve(K.toarray(), f)
        assert np.linalg.norm(x - ref) <= 20 * (n + 10) * 2.0 ** -53 * 7 * np.linalg.norm(ref)
    # solves: one preconditioned step reaches the tolerance (no bit equality on a
    # single level: its (r, z) comes from the element-parallel dot kernels)
    Ft = torch.from_numpy(F).cuda()
    out = ctx.solve_batched(Ft.t(), tol=1e-10)
    for j in range(3):
        one = ctx.solve(Ft[j], tol=1e-10)
        assert one["iters"] == out["iters"][j] == 1
        # two solutions with residuals of at most 1e-10 |f|, cond 7
        assert torch.linalg.norm(one["u"] - out["U"][:, j]) <= 14e-10 * torch.linalg.norm(one["u"])


@pytest.mark.parametrize("n", [201, 403, 799])
@pytest.mark.parametrize("fp32", [0, 1])
def test_two_level_restriction(amg, n, fp32):
    """The coarse kernel restricts the fine residual itself in the single
    V-cycle, a kernel of its own does in the 16-column one: the same bits (FP64),
    iterates of the same solve."""
    print(f"case coarse restriction n={n} fp32={fp32}", flush=True)
    ctx = _context(amg, _band(n), **(dict(vcycle_fp32=1, krylov=1) if fp32 else {}))
    assert ctx.nlevels == 2
    F = torch.from_numpy(np.random.default_rng(n).standard_normal((2, n))).cuda()
    out = ctx.solve_batched(F.t(), tol=1e-8)
    for j in range(2):
        one = ctx.solve(F[j], tol=1e-8)
        assert one["status"] == 0 and one["iters"] == out["iters"][j]
        if not fp32:
            assert torch.equal(one["u"], out["U"][:, j].contiguous())


@pytest.mark.parametrize("n", [65, 150, 1000])
def test_residual_of_an_ill_conditioned_coarsest_matrix(amg, n):
    """Condition 1e12, smooth solutions: the residual of the solve is that of
    products with the triangular inverses (n u sqrt(cond)), not of one with the
    inverse matrix (u cond: 7e-5 |f| at n = 150)."""
    print(f"case coarse residual n={n}", flush=True)
    one = np.ones(n - 1)
    d = np.full(n, 2.0)
    d[0] = d[-1] = 1.0
    K = sp.diags([d + 4e-12, -one, -one], [0, 1, -1]).tocsr()
    ctx = _context(amg, K, max_coarse=2000)
    assert ctx.nlevels == 1
    F = K @ np.random.default_rng(n).standard_normal((n, 3))
    # both products' and the factor's errors: 4 n u sqrt(cond) (|f| + |K| |z|)
    tol = 4 * n * 2.0 ** -53 * 1e6
    Ft = torch.from_numpy(np.ascontiguousarray(F.T)).cuda()
    for j in range(3):
        z = ctx.vcycle(Ft[j]).cpu().numpy()
        res, scale = np.linalg.norm(K @ z - F[:, j]), np.linalg.norm(F[:, j]) + 4 * np.linalg.norm(z)
        print(f"  residual {res / scale:.1e}, bound {tol:.1e}", flush=True)
        assert res <= tol * scale
    if n <= 150:    # the bound times |F|'s share of the scale is below 1e-6
        assert list(ctx.solve_batched(Ft.t(), tol=1e-6)["iters"]) == [1, 1, 1]
        assert ctx.solve(Ft[0], tol=1e-6)["iters"] == 1

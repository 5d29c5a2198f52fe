"""GPU: the device-filled matrix images (entries from the device copy of the
matrix, or uploaded in pieces of 4M entries) in every layout: shared offsets,
sorted windows, 16-bit and 32-bit columns, ragged last slices.  The matrices
and vectors hold small integers, so K x is exact in any order of the sum."""
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


def _matrix(kind, n):
    if kind == "planes":                     # box stencil of m^3 points: slices across lines and planes
        D = sp.diags([np.ones(n - abs(k)) for k in range(-2, 3)], range(-2, 3))
        A = -sp.kron(sp.kron(D, D), D).tocsr()
        A.setdiag(200.0)
        return A
    if kind == "band":                       # 41 diagonals: shared offsets
        k = np.arange(1, 41)
        return sp.diags([np.full(n, 100.0)] + [np.full(n - s, -1.0) for s in k] * 2, [0, *k, *-k], format="csr")
    r = np.random.default_rng(n)
    m = n * 35
    i, j = r.integers(0, n, m), r.integers(0, n, m)
    i[: m // 8] //= 9                        # some rows much longer than others
    if kind == "far":                        # a column gap of n - 1
        i, j = np.append(i[::9], 0), np.append(j[::9], n - 1)
    C = sp.coo_matrix((-r.integers(1, 4, len(i)).astype(np.float64), (i, j)), shape=(n, n)).tocsr()
    C = C + C.T
    C.setdiag(0.0)
    C.eliminate_zeros()
    return (C + sp.diags(np.asarray(abs(C).sum(axis=1)).ravel() + 1.0)).tocsr()


# 70,001 rows: 5.7M (band) and about 4.8M (ragged) entries, two pieces
@pytest.mark.parametrize("kind,n", [("band", 90), ("band", 4097), ("band", 70001), ("ragged", 130), ("ragged", 70001),
                                    ("far", 70001), ("planes", 13), ("planes", 17)])
@pytest.mark.parametrize("kw", [{}, {"setup_device": 1}, {"slice_offsets": 0}, {"smoother": 2},
                                {"nrhs": 16}], ids=str)
def test_images_hold_the_matrix(amg, kind, n, kw):
    print(f"case images {kind} n={n} {kw}", flush=True)
    K = _matrix(kind, n)
    K.sort_indices()
    ctx = amg.Context(K.indptr.astype(np.int64), K.indices.astype(np.int32), K.data, **kw)
    n = K.shape[0]
    if kind == "planes" and "nrhs" in kw:    # every slice has an offset list, across the planes too
        assert ctx.format(0)["shared_slices"] == (n + 63) // 64
    x = np.random.default_rng(1).integers(-50, 50, n).astype(np.float64)
    y = ctx.spmv(torch.from_numpy(x).cuda()).cpu().numpy()
    assert np.array_equal(y, K @ x)
    if kw.get("smoother") == 2:
        return
    # K P inside the V-cycle against the same V-cycle without it (the coarse
    # correction added first): a few sums of the row lengths' terms apart
    r = torch.from_numpy(np.random.default_rng(2).standard_normal(n)).cuda()
    z = ctx.vcycle(r)
    ctx.set_fused_post(False)
    ref = ctx.vcycle(r)
    w = int(np.diff(K.indptr).max())
    assert torch.linalg.norm(z - ref) <= 100 * (w + 10) * 2.0 ** -53 * torch.linalg.norm(ref)


@pytest.mark.parametrize("half", [1, 8, 49, 50, 70])
def test_device_setup_either_side_of_the_lanes_rule(amg, half):
    """3 to 141 entries a row, 16 or 64 lanes a row: aggregates, prolongator and
    coarse matrix of the host set-up, bit for bit."""
    print(f"case device set-up band {half}", flush=True)
    n = 6000
    r = np.random.default_rng(half)
    off = [r.uniform(-1.0, -0.1, n - s) for s in range(1, half + 1)]
    k = np.arange(1, half + 1)
    K = sp.diags([np.full(n, 2.0 * half + 1.0)] + off * 2, [0, *k, *-k], format="csr")
    K.sort_indices()
    arrays = (K.indptr.astype(np.int64), K.indices.astype(np.int32), K.data)
    dev, host = amg.Context(*arrays, setup_device=1), amg.Context(*arrays, host_only=True)
    for l in range(host.nlevels - 1):
        for a, b in zip(dev.aggregates(l), host.aggregates(l)):
            assert np.array_equal(a, b)
        for a, b in zip(dev.coarse_matrix(l + 1), host.coarse_matrix(l + 1)):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("row", [0, 31, 2999])
@pytest.mark.parametrize("fault", ["range", "order", "nan", "diag", "values"])
@pytest.mark.parametrize("half", [8, 60])
def test_device_check_refuses_what_the_host_refuses(amg, half, fault, row):
    """One fault in one row (16 or 64 lanes a row): the host's code and message."""
    print(f"case check {half} {fault} {row}", flush=True)
    n = 3000
    k = np.arange(1, half + 1)
    K = sp.diags([np.full(n, 200.0)] + [np.full(n - s, -1.0) for s in k] * 2, [0, *k, *-k], format="csr")
    K.sort_indices()
    rp, ci, v = K.indptr.astype(np.int64), K.indices.astype(np.int32), K.data.copy()
    a, b = rp[row], rp[row + 1]
    if fault == "range":
        ci[b - 1] = n
    elif fault == "order":
        ci[a + 1] = ci[a]
    elif fault == "nan":
        v[a] = np.nan
    elif fault == "diag":
        v[a + int(np.searchsorted(ci[a:b], row))] = -1.0
    else:
        v[a + (1 if ci[a] == row else 0)] = -1.5
    errors = []
    for kw in ({"setup_device": 1}, {"host_only": True}):
        with pytest.raises(amg.AmgError) as e:
            amg.Context(rp, ci, v, **kw)
        errors.append(str(e.value))
    assert errors[0] == errors[1]


@pytest.mark.parametrize("d,p,n,nrhs", [(2, 1, 1100, 16), (3, 2, 65, 1)])
def test_device_setup_past_one_grid(amg, d, p, n, nrhs):
    """More rows than one pass of the grid holds (16 lanes: 2^20 rows, 64 lanes:
    2^18), and more slices than one launch of the fill (65,536): the host
    set-up's hierarchy bit for bit, and the block kernels' first iterate on the
    lanes-per-row images against one lane per row."""
    print(f"case device set-up past one grid d={d} p={p} n={n}", flush=True)
    rp, ci, v, _ = amg.iga_poisson(d, p, n, want_F=False)
    dev = amg.Context(rp, ci, v, setup_device=1, nrhs=nrhs, itmax=1)
    host = amg.Context(rp, ci, v, host_only=True)
    assert dev.nlevels == host.nlevels
    for l in range(host.nlevels - 1):
        for a, b in zip(dev.aggregates(l), host.aggregates(l)):
            assert np.array_equal(a, b)
        for a, b in zip(dev.coarse_matrix(l + 1), host.coarse_matrix(l + 1)):
            assert np.array_equal(a, b)
    K = sp.csr_matrix((v, ci, rp))
    x = np.random.default_rng(1).standard_normal(len(rp) - 1)
    y = dev.spmv(torch.from_numpy(x).cuda()).cpu().numpy()
    w = int(np.diff(rp).max())
    # ascending sums of w products on both sides
    assert np.all(np.abs(y - K @ x) <= 2 * (w + 1) * 2.0 ** -53 * (abs(K) @ np.abs(x)))
    if nrhs == 1:
        return
    F = torch.from_numpy(np.random.default_rng(n).standard_normal((16, len(rp) - 1))).cuda().t()
    got = dev.solve_batched(F)["U"]
    dev.set_batched_variant(1, 256)
    ref = dev.solve_batched(F)["U"]
    # two sums of N products each: 2 N u on sums of absolute terms at most about
    # ten times their value
    assert torch.linalg.norm(got - ref) <= 20 * len(rp) * 2.0 ** -53 * torch.linalg.norm(ref)

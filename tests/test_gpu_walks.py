"""GPU: every walk of an image gives the same bits: x windows, one wavefront per
slice, several."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def amg():
    import paper_2511_21268_amd as m
    assert torch.cuda.is_available()
    m.lib()
    return m


@pytest.mark.parametrize("d,p,n", [(3, 3, 16), (2, 5, 40), (2, 2, 61)])
def test_x_window_option_reaches_small_images(amg, d, p, n):
    """Images below the several-wavefronts rule start without windows, so that
    the option's two values are two walks there (one wavefront per slice
    through the windows, several with gathers): operator and V-cycle bit for
    bit, through FP32 values and Chebyshev passes too."""
    print(f"case x window d={d} p={p} n={n}", flush=True)
    rp, ci, v, _ = amg.iga_poisson(d, p, n, want_F=False)
    x = torch.from_numpy(np.random.default_rng(3).standard_normal(len(rp) - 1)).cuda()
    for kw in ({}, {"vcycle_fp32": 1, "krylov": 1}, {"smoother": 2}):
        ctx = amg.Context(rp, ci, v, **kw)
        assert ctx.option(amg.amg.AMG_OPT_X_WINDOW) == 0
        start = ctx.spmv(x), ctx.vcycle(x)
        for on in (1, 0):
            ctx.set_x_window(on)
            assert ctx.option(amg.amg.AMG_OPT_X_WINDOW) == on
            assert torch.equal(ctx.spmv(x), start[0]) and torch.equal(ctx.vcycle(x), start[1]), (kw, on)


FORMS = {
    "fp64": {}, "fp32": dict(vcycle_fp32=1, krylov=1), "learned": dict(smoother=1),
    "learned32": dict(smoother=1, vcycle_fp32=1, krylov=1), "chebyshev": dict(smoother=2), "paper": None,
    "batched": dict(nrhs=16), "batched32": dict(nrhs=16, vcycle_fp32=1, krylov=1),
}


def _same(a, b):
    return torch.equal(a["u" if "u" in a else "U"], b["u" if "u" in b else "U"]) and np.array_equal(a["iters"], b["iters"])


# finest images of 77 (8 wavefronts), 562 and 993 (4) slices
@pytest.mark.parametrize("d,p,n", [(3, 3, 16), (3, 2, 33), (2, 4, 250)])
@pytest.mark.parametrize("form", FORMS)
def test_several_wavefronts_equal_one(amg, form, d, p, n):
    """AMG_OPT_SPLIT: operator, V-cycle and whole solves bit for bit, through
    every pass (plain, fused post-smoothing, residual of the polynomial steps,
    Chebyshev, 16 columns; FP64 and FP32, dots included)."""
    print(f"case walks {form} d={d} p={p} n={n}", flush=True)
    from paper_2511_21268_amd import learned
    kw = FORMS[form]
    rp, ci, v, _ = amg.iga_poisson(d, p, n, want_F=False)
    ctx = amg.Context(rp, ci, v, itmax=40, **(amg.paper_default(p) if kw is None else kw))
    if form.startswith("learned"):
        assert any(learned.apply_learned(ctx)[0])
    N = len(rp) - 1
    F = torch.from_numpy(np.random.default_rng(n).standard_normal((16, N))).cuda()
    if form.startswith("batched"):
        # 16-column passes of the coarse levels; the level-0 images have windows
        ctx.set_block_window(0)
        if ctx.batched_variant()[0] == 1:
            pytest.skip("one lane per row was faster on this system")
        calls = [lambda: ctx.solve_batched(F.t(), tol=1e-6, check=False)]
    else:
        calls = [lambda: ctx.spmv(F[0]), lambda: ctx.vcycle(F[1]), lambda: ctx.solve(F[2], tol=1e-6, check=False)]
    got = {}
    for on in (1, 0):
        ctx.set_split(on)
        assert ctx.option(amg.amg.AMG_OPT_SPLIT) == on
        got[on] = [c() for c in calls]
    for a, b in zip(got[1], got[0]):
        assert torch.equal(a, b) if isinstance(a, torch.Tensor) else _same(a, b)

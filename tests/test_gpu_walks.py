"""GPU: which kernels walk an image, and that every walk of it gives the same
bits: x windows, one wavefront per slice, several."""
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


def _kernels(call):
    """Names of the GPU kernels that a call launches."""
    from torch.profiler import ProfilerActivity, profile
    call()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    return " ".join(e.name for e in prof.events())


@pytest.mark.parametrize("d,p,n", [(3, 3, 16), (2, 5, 40), (2, 2, 61)])
def test_x_window_option_reaches_small_images(amg, d, p, n):
    """Images below the several-wavefronts rule: with the option on the passes
    walk the windows (one wavefront per slice), without it they do not; it
    starts off there."""
    print(f"case x window route d={d} p={p} n={n}", flush=True)
    rp, ci, v, _ = amg.iga_poisson(d, p, n, want_F=False)
    ctx = amg.Context(rp, ci, v)
    x = torch.from_numpy(np.random.default_rng(3).standard_normal(len(rp) - 1)).cuda()
    out = []
    for on, walk, other in ((None, "k_split", "k_sell"), (1, "k_sell", "k_split"), (0, "k_split", "k_sell")):
        if on is not None:
            ctx.set_x_window(on)
        assert ctx.option(amg.amg.AMG_OPT_X_WINDOW) == (on or 0)
        names = _kernels(lambda: ctx.spmv(x))
        assert walk in names and other not in names, names
        out.append(ctx.spmv(x))
    assert torch.equal(out[0], out[1]) and torch.equal(out[0], out[2])

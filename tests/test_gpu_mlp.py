"""GPU: the smoother network's forward and gradient kernels at the edges of
their tiles (16 samples forward, 64 backward), of the workspace rule (one block
of sums below 76 samples, at most 512) and at large batches, against FP64."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _reference(w, X, T):
    """FP64 forward, loss, gradient and the gradient's sums of absolute terms."""
    parts, at = [], 0
    for rows, cols in ((64, 8), (64, 1), (64, 64), (64, 1), (4, 64), (4, 1)):
        parts.append(w[at:at + rows * cols].reshape(rows, cols))
        at += rows * cols
    W1, b1, W2, b2, W3, b3 = parts
    h1 = np.tanh(X @ W1.T + b1.T)
    h2 = np.tanh(h1 @ W2.T + b2.T)
    Y = h2 @ W3.T + b3.T
    scale = 2.0 / T.size

    def grad(dy, W2, W3, t1, t2, X, h1, h2):
        d2 = (dy @ W3) * t2
        d1 = (d2 @ W2) * t1
        return np.concatenate([a.ravel() for a in (d1.T @ X, d1.sum(0), d2.T @ h1, d2.sum(0), dy.T @ h2, dy.sum(0))])

    g = grad(scale * (Y - T), W2, W3, 1 - h1 ** 2, 1 - h2 ** 2, X, h1, h2)
    top = abs(h2) @ abs(W3).T + abs(b3).T + abs(T)
    ga = grad(scale * top, abs(W2), abs(W3), 1.0, 1.0, abs(X), abs(h1), abs(h2))
    return h1, h2, Y, top, ((Y - T) ** 2).mean(), g, ga


@pytest.mark.parametrize("B", [1, 15, 16, 17, 63, 64, 65, 75, 76, 129, 1000, 16384, 40000])
def test_mlp_batches(B):
    print(f"case mlp B={B}", flush=True)
    from paper_2511_21268_amd import amg
    from paper_2511_21268_amd.learned import Trainer
    L = amg.lib()
    tr = Trainer(seed=B)
    r = np.random.default_rng(B)
    X, T = (r.standard_normal((B, k)).astype(np.float32) for k in (8, 4))
    # weights at an odd BF16 position: no alignment beyond their own type
    shifted = torch.empty(amg.MLP_NPARAM + 1, dtype=torch.int16, device="cuda")[1:]
    shifted.copy_(tr.w)
    # guard values past every output
    guard = 64
    act, Y = (torch.full((B * k + guard,), 7.0, device="cuda") for k in (amg.MLP_NACT, 4))
    work = torch.full((B * amg.MLP_NDEL + guard,), 7.0, device="cuda")
    g, loss = torch.full((amg.MLP_NPARAM + guard,), 7.0, device="cuda"), torch.full((1 + guard,), 7.0, device="cuda")
    Xd, Td = torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda()
    p = lambda t: C.c_void_p(t.data_ptr())  # noqa: E731
    st = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    amg._check(L.amg_mlp_forward(p(shifted), p(Xd), B, p(Y), p(act), st))
    amg._check(L.amg_mlp_backward(p(shifted), p(Xd), p(act), p(Y), p(Td), B, p(work), p(g), p(loss), st))
    torch.cuda.synchronize()
    for t, n in ((act, B * amg.MLP_NACT), (Y, B * 4), (work, B * amg.MLP_NDEL), (g, amg.MLP_NPARAM), (loss, 1)):
        assert bool((t[n:] == 7.0).all())
    w = tr.w.view(torch.bfloat16).double().cpu().numpy()
    h1, h2, Yr, top, lr, gr, ga = _reference(w, X.astype(np.float64), T.astype(np.float64))
    # chains of at most 65 terms per layer, tanh within 4 units, then at most
    # 128 samples per block, 32 partial sums per thread and 16 threads: below
    # 3 * (65 + 4) + 180 = 387 roundings of 2^-24 on the sums of absolute terms
    u = 2.0 ** -24
    got = act[:B * amg.MLP_NACT].cpu().numpy().reshape(B, 2, 64)
    assert np.all(abs(got[:, 0] - h1) <= 20 * u * (1 + abs(X).sum(1, keepdims=True)))
    assert np.all(abs(Y[:B * 4].cpu().numpy().reshape(B, 4) - Yr) <= 387 * u * (top + 64))
    assert np.all(abs(g[:amg.MLP_NPARAM].cpu().numpy() - gr) <= 387 * u * (ga + ga.max()))
    assert abs(float(loss[0]) - lr) <= 387 * u * float((top ** 2).mean())


def _loss(tr, X, T):
    """Loss, gradient and outputs of one forward and backward pass."""
    from paper_2511_21268_amd import amg
    Xd, Td = torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda()
    act = torch.empty(len(X), amg.MLP_NACT, device="cuda")
    Y = tr.forward(Xd, act)
    return tr.backward(Xd, act, Y, Td), tr.grad.cpu().numpy(), Y.cpu().numpy()


@pytest.mark.parametrize("B", [1, 58, 76, 1000, 16384, 20001])
@pytest.mark.parametrize("fault,expect", [("inf", np.inf), ("square", np.inf), ("sum", np.inf), ("nan", np.nan),
                                          ("inf nan", np.nan)])
def test_loss_of_a_diverged_training(B, fault, expect):
    """Targets that are infinite, whose squares or whose sum of squares
    overflow, or NaN, at the batch's start, middle or end: the loss is that of
    the ascending FP32 sum."""
    print(f"case mlp loss {fault} B={B}", flush=True)
    from paper_2511_21268_amd.learned import Trainer
    tr = Trainer(seed=1)
    r = np.random.default_rng(B)
    X = r.standard_normal((B, 8)).astype(np.float32)
    for at in {0, B // 2, B - 1}:
        T = r.standard_normal((B, 4)).astype(np.float32)
        if fault == "sum":
            T[:] = 1.2e19 if B == 1 else 3.7e38 ** 0.5 / B ** 0.5      # squares add up past 3.4e38
        else:
            T[at] = {"inf": np.inf, "square": 1e25, "nan": np.nan, "inf nan": np.inf}[fault]
        if fault == "inf nan":
            T[B - 1 - at, 3] = np.nan
        loss = _loss(tr, X, T)[0]
        assert np.array_equal(loss, expect, equal_nan=True), (at, loss)


@pytest.mark.parametrize("B", [1, 7, 16, 58, 64, 65, 75, 76, 129, 1000, 16384, 40000])
def test_loss_is_the_ascending_chain(B):
    """One definition for every batch size: l = fma(e, e, l) in FP32 over the
    outputs in order, divided by their number.  One block walks the chain
    itself; several form it from segments, which differ from it where a segment
    starts next to a binade's end and in the final roundings (16 units of 2^-24)."""
    print(f"case mlp loss chain B={B}", flush=True)
    from paper_2511_21268_amd.learned import Trainer
    r = np.random.default_rng(B)
    X, T = (r.standard_normal((B, k)).astype(np.float32) for k in (8, 4))
    loss, _, Y = _loss(Trainer(seed=2), X, T)
    l = np.float32(0.0)
    for e in (Y - T).ravel():
        l = np.float32(np.float64(e) * np.float64(e) + np.float64(l))   # exact product, one FP64 sum
    chain = float(l / np.float32(4 * B))
    # equal but for the FP64 sum's own rounding before the FP32 one (a tie, rarely)
    assert abs(loss - chain) <= (1 if B < 76 else 16) * 2.0 ** -24 * chain


@pytest.mark.parametrize("B", [58, 64, 100, 1000])
def test_gradient_of_infinite_weights(B):
    """An infinite output weight: where the sum over the samples is infinite it
    stays so, also in batches that do not fill their last tile (a tile's rows
    past the batch hold zeros, and inf * 0 is NaN)."""
    print(f"case mlp infinite weight B={B}", flush=True)
    from paper_2511_21268_amd.learned import Trainer
    tr = Trainer(seed=3)
    w = tr.w.view(torch.bfloat16)
    b2, W3 = 64 * 8 + 64 + 64 * 64, 64 * 8 + 64 + 64 * 64 + 64
    w[W3 + 7] = float("inf")
    w[b2 + 7] = 0.75                                       # hidden unit 7 positive for every sample
    w[64 * 8 + 64 + 7 * 64: 64 * 8 + 64 + 8 * 64] *= 0.01
    r = np.random.default_rng(B)
    X, T = (r.standard_normal((B, k)).astype(np.float32) for k in (8, 4))
    _, g, _ = _loss(tr, X, T)
    with np.errstate(all="ignore"):
        gr = _reference(w.double().cpu().numpy(), X.astype(np.float64), T.astype(np.float64))[5]
    at = b2 + 7                                            # sum of inf * (1 - h2^2) over the samples
    assert gr[at] == np.inf and g[at] == np.inf, (gr[at], g[at])
    assert g[W3 + 7] == np.inf == gr[W3 + 7]


@pytest.mark.parametrize("B", [1 << 27, (1 << 27) + 5, 1 << 28])
def test_forward_of_more_samples_than_one_launch_holds(B):
    """The launch limit is 2^32 threads, 16 a sample (13 GB of inputs and
    outputs at 2^28): the last samples' outputs are those of a small batch."""
    print(f"case mlp forward B={B}", flush=True)
    from paper_2511_21268_amd.learned import Trainer
    tr = Trainer(seed=4)
    tail = torch.randn(40, 8, generator=torch.Generator().manual_seed(1)).cuda()
    X = torch.zeros(B, 8, device="cuda")
    X[-40:] = tail
    X[:40] = tail
    Y, small = tr.forward(X), tr.forward(tail)
    assert torch.equal(Y[-40:], small) and torch.equal(Y[:40], small)
    assert bool((Y[40:-40] == Y[50]).all())

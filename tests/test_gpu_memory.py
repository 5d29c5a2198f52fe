"""GPU: set-ups with little device memory.  The card is filled by one
allocation and a smaller one on top of it leaves what a case asks for."""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _hubs(n, every, links):
    """Every `every`th unknown coupled to `links` others: images several times
    the matrix's size (a long row pads its slice), levels that fill in."""
    r = np.random.default_rng(0)
    h, t = np.repeat(np.arange(0, n, every), links), r.integers(0, n, n // every * links + links)[: len(range(0, n, every)) * links]
    C = sp.coo_matrix((np.ones(len(h)), (h, t)), shape=(n, n)).tocsr()
    C = C + C.T + sp.diags([np.ones(n - 1)] * 2, [1, -1])
    C.setdiag(0.0)
    C.eliminate_zeros()
    C.data[:] = -0.5
    K = (C + sp.diags(np.asarray(abs(C).sum(axis=1)).ravel() + 1.0)).tocsr()
    K.sort_indices()
    return K.indptr.astype(np.int64), K.indices.astype(np.int32), K.data


class Card:
    """Leaves a given amount of device memory free."""

    ROOM = 6 << 30

    def __init__(self):
        self.hold = torch.empty(self.free() - self.ROOM, dtype=torch.uint8, device="cuda")
        self.rest = None

    @staticmethod
    def free():
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        return torch.cuda.mem_get_info()[0]

    def leave(self, amount):
        self.rest = None
        n = self.free() - int(amount)
        assert n > 0
        self.rest = torch.empty(n, dtype=torch.uint8, device="cuda")


@pytest.fixture(scope="module")
def scarce():
    """The matrix, its context's size and result, and the filled card."""
    import paper_2511_21268_amd as amg
    arrays = _hubs(150000, 32, 512)
    x = torch.randn(150000, generator=torch.Generator().manual_seed(1), dtype=torch.float64).cuda()
    for _ in range(2):                                   # the first loads code, too
        before = Card.free()
        ctx = amg.Context(*arrays)
        z = ctx.vcycle(x)
        size = before - Card.free()
        ctx.close()
    other = amg.Context(*amg.iga_poisson(2, 2, 40, want_F=False)[:3])
    xo = x[:1600].contiguous()
    other.vcycle(xo)
    card = Card()
    yield amg, arrays, x, z, size, card, lambda: other.vcycle(xo)
    card.rest = card.hold = None
    torch.cuda.empty_cache()


@pytest.mark.parametrize("device", [0, 1])
def test_a_failed_set_up_leaves_no_error_behind(scarce, device):
    """Later calls of the library and of torch succeed."""
    amg, arrays, x, z, size, card, other = scarce
    print(f"case stale error device={device}", flush=True)
    for share in (0.05, 0.3, 0.9):
        card.leave(share * size)
        with pytest.raises(amg.AmgError):
            amg.Context(*arrays, setup_device=device)
        other()
        assert float((x + 1.0).sum()) == float((x + 1.0).sum())


def test_a_fault_is_named_without_memory_for_the_check(scarce):
    """No room for the device's copy of K: the host checks the entries."""
    amg, arrays, x, z, size, card, other = scarce
    print("case check on the host", flush=True)
    card.leave(4 * len(arrays[1]))
    bad = arrays[2].copy()
    bad[0] = np.nan
    messages = []
    for kw in ({"setup_device": 1}, {"host_only": True}):
        with pytest.raises(amg.AmgError) as e:
            amg.Context(arrays[0], arrays[1], bad, **kw)
        messages.append(str(e.value))
    assert messages[0] == messages[1]
    other()


# 20 bytes an entry: less than the copies of the level matrices (12 bytes for
# each of 3.7 entries), and far less than the products' work space
@pytest.mark.parametrize("spare", [20, 30, 50, 70])
@pytest.mark.parametrize("device", [0, 1])
def test_copies_and_idle_blocks_go_before_the_images_fail(scarce, spare, device):
    amg, arrays, x, z, size, card, _ = scarce
    print(f"case scarce memory spare={spare} B/entry device={device}", flush=True)
    card.leave(size + spare * len(arrays[1]))
    ctx = amg.Context(*arrays, setup_device=device)
    # the products of host and device have the same bits, and so the images
    assert torch.equal(ctx.vcycle(x), z)
    ctx.close()


@pytest.mark.parametrize("device", [0, 1])
def test_images_without_memory_are_out_of_memory(scarce, device):
    """The images do not fit: AMG_ERR_OOM, with the products on either side."""
    amg, arrays, x, z, size, card, _ = scarce
    print(f"case no memory device={device}", flush=True)
    for share in (0.6, 0.75, 0.9):
        card.leave(share * size)
        with pytest.raises(amg.AmgError) as e:
            amg.Context(*arrays, setup_device=device)
        assert e.value.status == -4, (share, str(e.value))

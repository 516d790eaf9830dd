"""What a call reads back on the host (ranks, energies, norms) is its own,
whatever became of the calls before it on the same thread or runs inside it.

Results are compared with the same call made alone: bit-identical, since the
kernels sum in a fixed order.
"""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def tk():
    import paper_1901_06043_amd as tk
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    tk.lib()
    return tk


class HookedAllocator:
    """The library's blocks from PyTorch's allocator; `hook(i)` is asked before
    the i-th block and refuses it by returning False."""

    def __init__(self, tk, hook=None):
        self.tk, self.hook, self.calls, self.blocks = tk, hook, 0, {}

    def __enter__(self):
        def alloc(nbytes, ctx, stream):
            i = self.calls
            self.calls += 1
            if self.hook is not None and self.hook(i) is False:
                return None
            block = torch.empty(int(nbytes), dtype=torch.uint8, device="cuda")
            self.blocks[block.data_ptr()] = block
            return block.data_ptr()

        # (blocks are kept until the end: the streams that use them are not PyTorch's)
        fields = self.tk._Allocator._fields_
        self.table = self.tk._Allocator(fields[0][1](alloc), fields[1][1](lambda p, ctx, stream: None), None)
        assert self.tk.lib().tucker_set_allocator(ctypes.byref(self.table)) == 0
        return self

    def __exit__(self, *exc):
        assert self.tk.lib().tucker_set_allocator(None) == 0
        torch.cuda.synchronize()


def tensor(seed, dims, scale=1.0):
    rng = np.random.default_rng(seed)
    return torch.from_numpy(scale * rng.standard_normal(list(reversed(dims)))).cuda()


def told(t):
    return t.ranks, t.discarded, t.norm2


DIMS, RANKS = [40, 36, 70], [9, 8, 7]


def test_early_return_leaves_no_writes(tk):
    """Given ranks, an allocation refused in the middle while the stream is
    busy: the call waits for what it enqueued, and the next calls of the thread
    on another stream read their own results."""
    x, y = tensor(1, DIMS), tensor(2, [50, 31, 33], 3.0)
    alone = tk.sthosvd_ranks(y, [5, 6, 7])
    b = tk.Batch([x, y], 1e-1)
    b.run()
    items = [told(b.item(i)) for i in range(2)]
    torch.cuda.synchronize()
    with HookedAllocator(tk) as a:
        tk.sthosvd_ranks(x, RANKS).free()
        total = a.calls
    busy = torch.randn(8192, 8192, device="cuda")
    sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for refused in (total // 2, total - 1):  # in the second step and at the last product
        with HookedAllocator(tk, lambda i: i != refused):
            with torch.cuda.stream(sa):
                for _ in range(10):
                    busy @ busy
            with pytest.raises(tk.TuckerError) as e:
                tk.sthosvd_ranks(x, RANKS, stream=sa)
            assert e.value.name == "ENOMEM"
            assert sa.query()
        b.run(stream=sb)
        assert [told(b.item(i)) for i in range(2)] == items
        assert told(tk.sthosvd_ranks(y, [5, 6, 7], stream=sb)) == told(alone)


@pytest.mark.parametrize("given", [True, False])
def test_allocator_that_calls_the_library(tk, given):
    """A compression and a batch item inside the allocator's callback leave the
    outer call's results alone."""
    x, y = tensor(3, DIMS), tensor(4, [50, 31, 33], 3.0)

    def run():
        return told(tk.sthosvd_ranks(x, RANKS) if given else tk.sthosvd(x, 0.3))

    alone = run()
    b = tk.Batch([x, y], 1e-1)
    inner = []

    def hook(i):
        if inner and inner[-1] is None:  # the callback's own blocks
            return True
        inner.append(None)
        torch.cuda.synchronize()
        b.run()
        inner[-1] = (told(tk.sthosvd_ranks(y, [5, 6, 7])), told(b.item(1)))
        return True

    with HookedAllocator(tk, hook):
        assert run() == alone
    assert len(inner) > 8 and all(v == inner[0] for v in inner)


def test_item_after_replay_on_the_null_stream(tk):
    """A captured run replayed on the null stream behind other work: an item
    taken right after it is the replay's, as the ranks of the whole batch are."""
    x, other = tensor(5, [30, 40, 50]), tensor(6, [30, 40, 50], 2.0)
    other[:, :, 10:] *= 1e-6
    ref = tk.Batch([other.clone()], 1e-2)
    ref.run()
    want, core = told(ref.item(0)), ref.item(0).core.clone()
    b = tk.Batch([x], 1e-2)
    b.run()
    assert told(b.item(0)) != want
    busy = torch.randn(8192, 8192, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        b.run()
    first = x.clone()
    for src in (other, first, other):
        for _ in range(10):
            busy @ busy
        x.copy_(src)
        g.replay()
        t = b.item(0)
        if src is other:
            assert told(t) == want
            assert torch.equal(t.core, core)
        else:
            assert told(t) != want
        assert b.ranks()[0] == t.ranks

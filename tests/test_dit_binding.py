"""Host side of the block binding (dit.py) on the CPU: the library is replaced
by one that records its arguments, so that what is checked is which memory a
call is handed."""
import threading

import pytest

from paper_2607_28144_amd import _lib

torch = pytest.importorskip("torch")

S, S_CTX, C, F, HEADS = 8, 4, 512, 64, 4


class Recorder:
    """The block call of the library: notes each call's workspace, with
    `inside` run while the call is under way."""

    def __init__(self, inside=None):
        self.calls, self.inside, self.lock = [], inside, threading.Lock()

    def regenvc_dit_block_fwd(self, *args):
        with self.lock:
            self.calls.append((args[14], args[15]))
        if self.inside is not None:
            self.inside()
        return _lib.OK

    def regenvc_dit_block_workspace(self, S, S_ctx, C, heads, F, n_cu, out):
        out._obj.value = 256 * S
        return _lib.OK


@pytest.fixture
def block(monkeypatch):
    from paper_2607_28144_amd import dit

    class Props:
        multi_processor_count = 256
    monkeypatch.setattr(torch.cuda, "get_device_properties", lambda device: Props)
    monkeypatch.setattr(dit, "_vec", lambda t, *a: t.data_ptr())
    monkeypatch.setattr(dit, "_stream", lambda device: None)
    blk = object.__new__(dit.DitBlock)  # no parameters: a device is needed for those
    blk.C, blk.F, blk.heads, blk._ws, blk._need, blk._c = C, F, HEADS, {}, {}, _lib.DitParams()

    def use(lib):
        monkeypatch.setattr(_lib, "load", lambda: lib)
        return lib

    def call(S=S):
        x, e = torch.zeros(S, C), torch.zeros(C)
        ctx = torch.zeros(S_CTX, HEADS, C // HEADS, dtype=torch.bfloat16)
        return blk.forward(x, e, ctx, ctx, (1, 1, S))
    return blk, use, call


def test_calls_under_way_at_once_share_no_workspace(block):
    """Two threads inside forward() of one block at the same time (each would
    enqueue on its own stream): disjoint workspaces."""
    _, use, call = block
    both = threading.Barrier(2, timeout=30)
    lib = use(Recorder(inside=both.wait))
    threads = [threading.Thread(target=call) for _ in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    (a, n), (b, m) = lib.calls
    assert n == m == 256 * S
    assert a + n <= b or b + m <= a


def test_no_workspace_is_held_between_calls(block):
    """Calls at many token counts: nothing but sizes is kept."""
    blk, use, call = block
    lib = use(Recorder())
    for s in range(1, 30):
        call(s)
    assert [n for _, n in lib.calls] == [256 * s for s in range(1, 30)]
    assert blk._ws == {} and all(isinstance(v, int) for v in blk._need.values())

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


class NoRoom:
    """torch.empty for a device whose memory holds no byte buffer above `limit`."""

    def __init__(self, limit):
        self.limit, self.empty = limit, torch.empty

    def __call__(self, *size, dtype=None, device=None, **kw):
        if dtype == torch.uint8 and size[0] > self.limit:
            raise torch.OutOfMemoryError("no room")
        return self.empty(*size, dtype=dtype, **kw)


def test_block_without_room_for_partial_sums_runs_in_the_least_workspace(block, monkeypatch):
    _, use, call = block
    lib = use(Recorder())
    lib.regenvc_dit_block_workspace_least = lambda *a: setattr(a[-1]._obj, "value", 256) or _lib.OK
    monkeypatch.setattr(torch, "empty", NoRoom(1000))
    call()
    assert [n for _, n in lib.calls] == [256]


def test_linear_and_convolution_without_room_for_partial_sums_do_not_split(monkeypatch):
    """A call that can run without its workspace is not refused for want of it."""
    from paper_2607_28144_amd import dit, vae
    given = []

    class Lib:
        def regenvc_linear_fwd_ws(self, *args):
            given.append(args[-3:-1])
            return _lib.OK

        def regenvc_vae_conv3d_fwd(self, *args):
            given.append(args[-3:-1])
            return _lib.OK
    monkeypatch.setattr(_lib, "load", lambda: Lib())
    monkeypatch.setattr(torch, "empty", NoRoom(1000))
    for m in (dit, vae):
        monkeypatch.setattr(m, "_stream", lambda device: None)
    monkeypatch.setattr(dit, "_rows", lambda t, *a: t.stride(0))
    monkeypatch.setattr(dit, "linear_workspace_bytes", lambda *a: 4096)
    monkeypatch.setattr(vae, "_check", lambda *a: None)
    monkeypatch.setattr(vae, "conv3d_workspace_bytes", lambda *a: 4096)
    dit.linear_fwd(torch.zeros(4, 64, dtype=torch.bfloat16), torch.zeros(16, 64, dtype=torch.bfloat16))
    vae.conv3d(torch.zeros(1, 2, 3, 64, dtype=torch.bfloat16), torch.zeros(64, 3, 3, 3, 64, dtype=torch.bfloat16),
               torch.zeros(64, dtype=torch.bfloat16), [_lib.VaeTile(0, 2, 0, 3, 0, 2, 0, 3)], 2, 3)
    assert given == [(None, 0), (None, 0)]

"""GPU parity of the spatially split VAE tile (include/regenvc_vae.h) against
the fp64 oracle (oracle/vae.py) on the same seeded bf16 inputs.

Each stage is checked on the GPU's own bf16 input to it, so that every bound
is the per-element one of a single rounding: a convolution output satisfies
|gpu - ref| <= 2^-8 |ref| + 2 * 2^-20 * sum |x||w| (fp32 accumulation over
the 27 Cin taps; SiLU's slope is below 1.1), the blend 2^-8 |ref| + 1e-6.
The end-to-end result (all stages on the GPU) is compared with the oracle's
stack on the whole plane -- equal in exact arithmetic when the halo covers
band + layers -- within two bf16 steps of each value plus 2^-8 of the RMS,
room for the rare rounding flips that carry from one layer into the next.
"""
import ctypes

import numpy as np
import pytest

from oracle import vae as ovae
from oracle.dit import widen
from paper_2607_28144_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

ULP = 2.0 ** -8
ACC = 2.0 ** -20


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_28144_amd import vae  # noqa: F401  (fails loudly if the library is missing)
    yield
    torch.cuda.synchronize()


def kern():
    from paper_2607_28144_amd import vae
    return vae


def dev_bits(bits):
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).view(torch.bfloat16).cuda()


def host(t):
    return t.float().cpu().numpy().astype(np.float64)


def check_bound(name, got, ref, tol):
    err = np.abs(got - ref)
    over = int(np.count_nonzero(err > tol))
    print(f"[vae] {name}: max|d|={err.max():.3e} rms={np.sqrt((err * err).mean()):.3e} "
          f"max err/bound={float((err / tol).max()):.3f} over={over}/{err.size}", flush=True)
    assert np.all(np.isfinite(got)) and over == 0, name


def region(t):
    return (t.reg_y0, t.reg_y1), (t.reg_x0, t.reg_x1)


def conv_ref(x, w_bits, b_bits, silu):
    """Oracle convolution of bf16-valued x (one region) and its bound."""
    W, B = widen(w_bits), widen(b_bits)
    y = ovae.conv3d_causal(x, W, B)
    slack = 2 * ACC * ovae.conv3d_causal(np.abs(x), np.abs(W), np.zeros_like(B))
    if silu:
        y = ovae.silu(y)
        slack = 1.1 * slack
    return y, ULP * np.abs(y) + slack + 1e-6


def stagewise(name, T, H, W, C, ty, tx, halo, band, tiles_to_check, seed):
    x, convs = synth.vae_inputs(seed, T, H, W, C)
    X = widen(x)
    tiles, Hr, Wr = kern().split(H, W, ty, tx, halo)
    tl = list(tiles)
    dx = dev_bits(x)
    dconvs = [(dev_bits(w), dev_bits(b)) for w, b in convs]
    y1 = kern().conv3d(dx, *dconvs[0], tl, Hr, Wr, silu=True)
    y2 = kern().conv3d(y1, *dconvs[1], tl, Hr, Wr, plane_hw=(H, W))
    out = kern().blend(y2, tl, H, W, band)
    torch.cuda.synchronize()
    g1, g2 = host(y1), host(y2)
    for i in tiles_to_check:
        (r0, r1), (c0, c1) = region(tl[i])
        h, w = r1 - r0, c1 - c0
        ref, tol = conv_ref(X[:, r0:r1, c0:c1], *convs[0], True)
        check_bound(f"{name} tile {i} conv 1 (SiLU)", g1[i, :, :h, :w], ref, tol)
        ref, tol = conv_ref(g1[i, :, :h, :w], *convs[1], False)
        check_bound(f"{name} tile {i} conv 2", g2[i, :, :h, :w], ref, tol)
    ref = np.zeros((T, H, W, C))
    for i, t in enumerate(tl):
        (r0, r1), (c0, c1) = region(t)
        wgt = np.outer(ovae.ramp(H, (t.core_y0, t.core_y1), (r0, r1), band),
                       ovae.ramp(W, (t.core_x0, t.core_x1), (c0, c1), band))
        ref[:, r0:r1, c0:c1] += wgt[None, :, :, None] * g2[i, :, :r1 - r0, :c1 - c0]
    check_bound(f"{name} blend", host(out), ref, ULP * np.abs(ref) + 1e-6)
    return X, convs, dx, dconvs, tl, Hr, Wr, y1, y2, out


def test_small_plane_every_tile_and_the_whole_plane():
    """3 frames of 12 x 16, 64 channels, 2 x 2 tiles, halo 4 >= band 2 + 2
    layers: every tile's stages, the blend, and the blended result against
    the oracle's stack on the whole plane."""
    X, convs, *_, out = stagewise("small", 3, 12, 16, 64, 2, 2, 4, 2, range(4), 71)
    full = ovae.stack(X, convs)
    got = host(out)
    check_bound("small end to end vs whole plane", got, full,
                2 * ULP * np.abs(full) + ULP * float(np.sqrt((full * full).mean())))


def test_window_latent_tile_of_an_eight_way_split():
    """The decoder stage at the window's latent resolution: 7 frames of
    60 x 104, 384 channels, split 2 x 4 (one tile per GPU of the node), halo
    4, band 2.  Tiles 1 (top row, inner column) and 4 (bottom-left) are
    checked stage by stage; one tile launched alone (one GPU's share) gives
    bitwise the batched launch's values when K is not split, and passes the
    same per-element bounds in its split-K form (the single tile's 64 row
    tiles run as 4 K ranges each); the blend is checked everywhere."""
    T, H, W, C = 7, 60, 104, 384
    X, convs, dx, dconvs, tl, Hr, Wr, y1, y2, out = stagewise("window", T, H, W, C, 2, 4, 4, 2, (1, 4), 72)
    assert kern().conv3d_workspace_bytes(T, Hr, Wr, 1, C, C, dx.device) > 0  # the single tile splits K
    assert kern().conv3d_workspace_bytes(T, Hr, Wr, 8, C, C, dx.device) == 0  # the batch does not
    one1 = kern().conv3d(dx, *dconvs[0], [tl[1]], Hr, Wr, silu=True, split_k=False)
    one2 = kern().conv3d(one1, *dconvs[1], [tl[1]], Hr, Wr, plane_hw=(H, W), split_k=False)
    sk1 = kern().conv3d(dx, *dconvs[0], [tl[1]], Hr, Wr, silu=True)
    sk2 = kern().conv3d(sk1, *dconvs[1], [tl[1]], Hr, Wr, plane_hw=(H, W))
    torch.cuda.synchronize()
    (r0, r1), (c0, c1) = region(tl[1])
    h, w = r1 - r0, c1 - c0
    assert torch.equal(one1[0, :, :h, :w], y1[1, :, :h, :w])
    assert torch.equal(one2[0, :, :h, :w], y2[1, :, :h, :w])
    g1 = host(sk1)[0, :, :h, :w]
    ref, tol = conv_ref(X[:, r0:r1, c0:c1], *convs[0], True)
    check_bound("window tile 1 split-K conv 1 (SiLU)", g1, ref, tol)
    ref, tol = conv_ref(g1, *convs[1], False)
    check_bound("window tile 1 split-K conv 2", host(sk2)[0, :, :h, :w], ref, tol)


@pytest.mark.parametrize("Cin,most", [(64, 3), (192, 8)])
def test_split_k_every_range_count(Cin, most):
    """Small convolutions in the split-K form with workspaces that allow 2,
    3 and 8 K ranges (and none): each against the oracle's per-element
    bound, on a 1 x 2 split (two tiles, 128 channels out).  A range has at
    least 8 steps of 64, so 64 channels in (27 steps) are cut into 3 ranges at most and 192 (81) into 8."""
    T, H, W, Cout = 3, 9, 14, 128
    rng = np.random.default_rng(74)
    x = synth.normal_bf16(rng, (T, H, W, Cin))
    wb = synth.normal_bf16(rng, (Cout, 3, 3, 3, Cin), float(1.0 / np.sqrt(27 * Cin)))
    bb = synth.normal_bf16(rng, (Cout,), 0.02)
    X = widen(x)
    tiles, Hr, Wr = kern().split(H, W, 1, 2, 3)
    tl = list(tiles)
    M = len(tl) * T * Hr * Wr
    dx, dw, db = dev_bits(x), dev_bits(wb), dev_bits(bb)
    from paper_2607_28144_amd import _lib
    lib = _lib.load()
    plan = _lib.TilePlan()
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    arr = (_lib.VaeTile * len(tl))(*tl)
    for ranges in (0, 2, 3, 8):
        out = torch.empty((len(tl), T, Hr, Wr, Cout), dtype=torch.bfloat16, device=dx.device)
        nbytes = ranges * M * Cout * 4
        _lib.check(lib.regenvc_vae_conv3d_plan_query(T, Hr, Wr, len(tl), Cin, Cout, n_cu, nbytes, ctypes.byref(plan)),
                   "plan query")
        assert plan.k_ranges == max(1, min(ranges, most))
        ws = torch.empty(max(nbytes, 256), dtype=torch.uint8, device=dx.device) if ranges else None
        st = lib.regenvc_vae_conv3d_fwd(dx.data_ptr(), 1, dw.data_ptr(), db.data_ptr(), 1, out.data_ptr(), T, H, W,
                                        Cin, Cout, arr, len(tl), Hr, Wr, ws.data_ptr() if ws is not None else None,
                                        nbytes, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        _lib.check(st, "regenvc_vae_conv3d_fwd")
        torch.cuda.synchronize()
        g = host(out)
        for i in range(len(tl)):
            (r0, r1), (c0, c1) = region(tl[i])
            ref, tol = conv_ref(X[:, r0:r1, c0:c1], wb, bb, True)
            check_bound(f"split-K {ranges} ranges, tile {i}", g[i, :, :r1 - r0, :c1 - c0], ref, tol)


# (T, H, W, Cin, Cout) and its plan on 256 compute units (rows, channels and
# waves of a tile, K ranges): every tile, whole and split, with ragged last rows and channels; and weight
# rows whose offsets need 64 bits.  test_tile_plan.py holds the plan to these
# and the list to every kernel.
CONV_PLANS = [
    (1, 17, 19, 64, 64, (128, 128, 4, 3)), (2, 97, 101, 64, 64, (128, 128, 4, 1)), (3, 90, 61, 64, 64, (128, 128, 4, 1)),
    (5, 71, 73, 256, 192, (128, 192, 4, 1)), (7, 34, 34, 384, 384, (128, 192, 4, 2)), (3, 34, 53, 256, 192, (128, 192, 4, 5)),
    (7, 75, 67, 64, 192, (192, 192, 4, 1)), (2, 47, 61, 256, 320, (192, 192, 4, 4)),
    (7, 83, 93, 64, 192, (256, 192, 4, 1)), (3, 90, 61, 192, 192, (256, 192, 4, 3)),
    (7, 90, 101, 128, 256, (256, 256, 4, 1)), (5, 61, 59, 256, 256, (256, 256, 4, 3)),
    (7, 34, 35, 192, 384, (128, 128, 4, 1)),
    (1, 2, 3, 155392, 64, (128, 128, 4, 8)),
]


@pytest.mark.parametrize("silu", [False, True])
@pytest.mark.parametrize("T,H,W,Cin,Cout,plan", CONV_PLANS)
def test_conv_tiles(T, H, W, Cin, Cout, plan, silu):
    """One region, the whole plane: against the same sums in float64 (one
    matrix product per tap), each element within one rounding of its value
    and 2^-19 of the sum of magnitudes."""
    g = torch.Generator(device="cuda").manual_seed(T * H + Cin)
    x = torch.randn(T, H, W, Cin, generator=g, device="cuda").bfloat16()
    w = (torch.randn(Cout, 3, 3, 3, Cin, generator=g, device="cuda") / (27 * Cin) ** 0.5).bfloat16()
    b = (torch.randn(Cout, generator=g, device="cuda") * 0.02).bfloat16()
    tiles, Hr, Wr = kern().split(H, W, 1, 1, 0)
    from test_tile_plan import conv_plan
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    assert n_cu != 256 or conv_plan(T, H, W, Cin, Cout) == plan
    # the plan as it is, and where that splits K also without
    got = [kern().conv3d(x, w, b, list(tiles), Hr, Wr, silu=silu)[0].double()]
    if plan[3] > 1:
        got.append(kern().conv3d(x, w, b, list(tiles), Hr, Wr, silu=silu, split_k=False)[0].double())

    def taps(x, w, b):
        p = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1, 2, 0))
        out = b.expand(T * H * W, -1).clone()
        for dt in range(3):
            for dy in range(3):
                for dx in range(3):
                    a = p[dt:dt + T, dy:dy + H, dx:dx + W].reshape(T * H * W, Cin)
                    out += torch.mm(a, w[:, dt, dy, dx].t().contiguous())
        return out.view(T, H, W, Cout)
    ref = taps(x.double(), w.double(), b.double())
    slack = 2.0 ** -19 * taps(x.double().abs(), w.double().abs(), b.double().abs())
    if silu:  # its slope is at most 1.1
        ref, slack = ref * torch.sigmoid(ref), 1.1 * slack + 1e-6
    tol = ULP * ref.abs() + slack
    worst = max(float(((g - ref).abs() / tol).max()) for g in got)
    print(f"[vae] conv {T}x{H}x{W} {Cin}->{Cout} silu={silu} on {plan}: max err/bound {worst:.3f}", flush=True)
    assert worst <= 1.0


def test_plain_crop_and_single_tile():
    """band 0 (plain crop to the cores) and a 1 x 1 split (no halo at all: the
    stack on the whole plane) against the oracle."""
    T, H, W, C = 2, 10, 12, 64
    x, convs = synth.vae_inputs(73, T, H, W, C)
    X = widen(x)
    dconvs = [(dev_bits(w), dev_bits(b)) for w, b in convs]
    for ty, tx, halo, band in [(1, 1, 0, 0), (2, 3, 2, 0)]:
        got = host(kern().split_stack(dev_bits(x), dconvs, ty, tx, halo, band))
        torch.cuda.synchronize()
        full = ovae.stack(X, convs)
        check_bound(f"split {ty}x{tx} halo {halo} band {band} vs whole plane", got, full,
                    2 * ULP * np.abs(full) + ULP * float(np.sqrt((full * full).mean())))

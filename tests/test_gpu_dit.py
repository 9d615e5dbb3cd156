"""GPU parity of the diffusion-transformer block kernels and of the block
forward (include/regenvc_dit.h) against the fp64 block oracle (oracle/dit.py)
on the same seeded bf16 inputs.

Per-kernel bounds follow from the arithmetic: the kernels accumulate in fp32
(error well below 2^-20 of sum |a_k w_k| for these K) and round bf16 outputs
once (at most 2^-8 of the value), so a bf16 output must satisfy
|gpu - ref| <= 2^-8 |ref| + 2 * 2^-20 * sum_k |a_k||w_k| (plus a GELU slope
of at most 1.13, and 1e-6 for the fp32 exponential); float32 outputs
(gated residual, modulation vectors) carry only the accumulation term and
float32 rounding.

The composed block differs from the oracle through bf16 rounding flips: a
value whose fp32 and fp64 forms straddle a bf16 rounding boundary is stored
one bf16 step apart, and the following layers carry the step on (the
attention's bf16 weights and the 8960-deep feed-forward sum many of them).
How far two correct bf16 implementations drift apart this way is measured,
not guessed: the tests run the oracle a second time with every value
perturbed by 1e-5 (relative, seeded) just before each bf16 rounding -- any
perturbation that small gives the same spread, about 1.1e-3 relative RMS
after one step and 2e-3 after four -- and hold the GPU to twice that
spread per step in relative RMS and in max error (relative to max|x|).  A
dropped 0.02 bias in any branch moves the stream by ~9e-3 of its RMS.
"""
import numpy as np
import pytest

from oracle import dit as odit
from paper_2607_28144_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

ULP = 2.0 ** -8
ACC = 2.0 ** -20


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_28144_amd import dit  # noqa: F401  (fails loudly if the library is missing)
    yield
    torch.cuda.synchronize()


def kern():
    from paper_2607_28144_amd import dit
    return dit


def dev_bits(bits):
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).view(torch.bfloat16).cuda()


def host(t):
    return t.float().cpu().numpy().astype(np.float64)


def check_bound(name, got, ref, tol):
    err = np.abs(got - ref)
    ratio = float((err / tol).max())
    over = int(np.count_nonzero(err > tol))
    print(f"[dit] {name}: max|d|={err.max():.3e} rms={np.sqrt((err * err).mean()):.3e} "
          f"max err/bound={ratio:.3f} over={over}/{err.size}", flush=True)
    assert np.all(np.isfinite(got)), f"{name}: non-finite output"
    assert over == 0, f"{name}: {over} elements over the bound (worst err/bound {ratio:.3f})"


def bits(rng, shape, scale=1.0):
    return synth.normal_bf16(rng, shape, scale)


@pytest.mark.parametrize("M,N,K", [(300, 256, 1536), (1000, 1536, 1536), (577, 4608, 1536), (333, 1536, 8960),
                                   (10920, 1536, 1536), (500, 400, 512), (289, 272, 64)])
def test_linear_epilogues(M, N, K):
    """Whole-width tiles stage their output through LDS; a last tile column
    narrower than 256 channels (N = 400, 272) stores straight from the
    accumulators."""
    rng = np.random.default_rng(M + N + K)
    a, w, b = bits(rng, (M, K)), bits(rng, (N, K), 0.02), bits(rng, (N,), 0.02)
    gate = rng.standard_normal(N).astype(np.float32)
    x0 = rng.standard_normal((M, N)).astype(np.float32)
    A, Wt, B = odit.widen(a), odit.widen(w), odit.widen(b)
    y = odit.gemm(A, Wt, B)
    slack = 2 * ACC * (np.abs(A) @ np.abs(Wt).T)
    da, dw, db = dev_bits(a), dev_bits(w), dev_bits(b)
    out = kern().linear_fwd(da, dw, db, "bias")
    out_g = kern().linear_fwd(da, dw, db, "bias_gelu")
    xr = torch.from_numpy(x0).cuda()
    kern().linear_fwd(da, dw, db, "gated_residual", gate=torch.from_numpy(gate).cuda(), out=xr)
    torch.cuda.synchronize()
    check_bound(f"linear bias M={M} N={N} K={K}", host(out), y, ULP * np.abs(y) + slack)
    g = odit.gelu_tanh(y)
    check_bound(f"linear bias+gelu M={M} N={N} K={K}", host(out_g), g, ULP * np.abs(g) + 1.13 * slack + 1e-6)
    xref = x0.astype(np.float64) + gate.astype(np.float64) * y
    check_bound(f"linear gated residual M={M} N={N} K={K}", host(xr), xref,
                np.abs(gate) * slack + 2.0 ** -22 * (np.abs(x0) + np.abs(gate * y)) + 1e-7)


# ragged last rows and channels, the shortest K, and K splits with uneven ranges
@pytest.mark.parametrize("M,N,K", [(1, 16, 64), (65, 1552, 128), (513, 1536, 192),
                                   (5461, 272, 64), (300, 4624, 1536), (1365, 1536, 1536),
                                   (1001, 8960, 1536), (5460, 1552, 1536),
                                   (1365, 8976, 1536),
                                   (5460, 1536, 1536),
                                   (2731, 1552, 1536), (2001, 1536, 8960),
                                   (1365, 1552, 8960), (64, 1536, 8960), (700, 1536, 8896)])
def test_linear_tiles(M, N, K):
    test_linear_epilogues(M, N, K)


# (M, N, K, epilogue) and its plan on 256 compute units (rows, channels and
# waves of a tile, K ranges): every tile with every epilogue that it is chosen
# for, and split over K; last rows and channels ragged.  test_tile_plan.py holds the plan to these
# and the list to every kernel.
LINEAR_PLANS = [
    (1, 16, 64, 0, (64, 128, 4, 1)), (65, 1552, 128, 1, (64, 128, 4, 1)), (513, 1536, 192, 2, (64, 128, 4, 1)),
    (64, 1536, 8960, 0, (64, 128, 4, 8)), (1, 16, 1536, 2, (64, 128, 4, 3)),
    (5461, 272, 64, 0, (128, 128, 4, 1)), (5461, 272, 64, 1, (128, 128, 4, 1)), (1365, 1536, 1536, 2, (128, 128, 4, 1)),
    (700, 1536, 8896, 1, (128, 128, 4, 3)), (2731, 16, 4096, 0, (128, 128, 4, 8)),
    (2731, 1552, 1536, 0, (128, 192, 4, 1)), (10921, 272, 1024, 1, (128, 192, 4, 1)), (10921, 272, 1024, 2, (128, 192, 4, 1)),
    (1001, 1536, 8960, 0, (128, 192, 4, 4)), (2001, 1536, 8960, 0, (128, 192, 4, 2)), (65, 8976, 8896, 2, (128, 192, 4, 5)),
    (1001, 8960, 1536, 0, (160, 256, 4, 1)), (5461, 1552, 320, 1, (160, 256, 4, 1)), (5461, 1552, 1024, 2, (160, 256, 4, 1)),
    (129, 8976, 8896, 0, (160, 256, 4, 7)), (1365, 1552, 8960, 1, (160, 256, 4, 4)),
    (5461, 1040, 1536, 0, (192, 192, 4, 1)), (5460, 1536, 1536, 1, (192, 192, 4, 1)), (10921, 528, 8896, 2, (192, 192, 4, 1)),
    (1365, 1536, 8960, 2, (192, 192, 4, 4)), (257, 4624, 8896, 0, (192, 192, 4, 5)),
    (10921, 1040, 1024, 0, (256, 256, 4, 1)), (1365, 8960, 1536, 1, (256, 256, 4, 1)), (10920, 1024, 8960, 2, (256, 256, 4, 1)),
    (4097, 1040, 8896, 1, (256, 256, 4, 3)),
    (10921, 1040, 64, 0, (256, 256, 8, 1)), (10921, 1040, 512, 2, (256, 256, 8, 1)), (1365, 8976, 1536, 2, (256, 256, 8, 1)),
    (10921, 1536, 64, 0, (288, 256, 8, 1)), (10921, 1536, 128, 1, (288, 256, 8, 1)), (10921, 1536, 320, 2, (288, 256, 8, 1)),
]


@pytest.mark.parametrize("M,N,K,epi,plan", LINEAR_PLANS)
def test_linear_on_every_tile(M, N, K, epi, plan):
    """Against float64 on the GPU, within the bounds of the module."""
    from test_tile_plan import linear_plan
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    assert n_cu != 256 or linear_plan(M, N, K, epi) == plan
    r = torch.Generator(device="cuda").manual_seed(M + N + K)
    rand = lambda *n: torch.randn(*n, generator=r, device="cuda")  # noqa: E731
    a, w, b, gate = rand(M, K).bfloat16(), (rand(N, K) * 0.02).bfloat16(), (rand(N) * 0.02).bfloat16(), rand(N)
    x0 = rand(M, N) if epi == 2 else None
    y = torch.mm(a.double(), w.double().t().contiguous()) + b.double()
    slack = 2 * ACC * torch.mm(a.double().abs(), w.double().abs().t().contiguous())
    if epi == 2:
        got = kern().linear_fwd(a, w, b, "gated_residual", gate=gate, out=x0.clone())
        g = gate.double()
        ref, tol = x0.double() + g * y, g.abs() * slack + 2.0 ** -22 * (x0.double().abs() + (g * y).abs()) + 1e-7
    elif epi == 1:
        got = kern().linear_fwd(a, w, b, "bias_gelu")
        ref = 0.5 * y * (1 + torch.tanh((2 / torch.pi) ** 0.5 * (y + 0.044715 * y ** 3)))
        tol = ULP * ref.abs() + 1.13 * slack + 1e-6
    else:
        got = kern().linear_fwd(a, w, b)
        ref, tol = y, ULP * y.abs() + slack
    worst = float(((got.double() - ref).abs() / tol).max())
    print(f"[dit] linear {M}x{N}x{K} epilogue {epi} on {plan}: max err/bound {worst:.3f}", flush=True)
    assert worst <= 1.0


def test_linear_wide_row_stride():
    """Rows so far apart that a tile's offsets leave 32 bits: 64-bit addresses
    on 128 x 128 tiles, the contiguous call on 64 x 128.  Both add the steps of
    K one after another, in the same order."""
    M, N, K, ld = 300, 272, 192, 1 << 23
    rng = np.random.default_rng(5)
    a, w = bits(rng, (M, K)), bits(rng, (N, K), 0.02)
    wide = torch.zeros((M - 1) * ld + K, dtype=torch.bfloat16, device="cuda")
    da = wide.as_strided((M, K), (ld, 1))
    da.copy_(dev_bits(a))
    dw = dev_bits(w)
    got = kern().linear_fwd(da, dw)
    assert torch.equal(got, kern().linear_fwd(da.contiguous(), dw))


@pytest.mark.parametrize("N,rows", [(1536, (1, 1365, 2731, 5461, 8193)),   # seven tiles between them and the epilogues
                                    (1552, (1, 1365, 2731, 5461, 8193))])  # 160 x 256 and ragged channels
@pytest.mark.parametrize("epi", [0, 1, 2])
def test_rows_come_out_alike_without_a_split(N, rows, epi):
    """Without a workspace a row is bitwise the same in a call of any number of
    rows, on whatever tile."""
    import ctypes
    from paper_2607_28144_amd import _lib
    M, K, lib = 10921, 512, _lib.load()
    r = torch.Generator(device="cuda").manual_seed(N)
    rand = lambda *n: torch.randn(*n, generator=r, device="cuda")  # noqa: E731
    a, w, b, gate, x0 = rand(M, K).bfloat16(), (rand(N, K) * 0.02).bfloat16(), rand(N).bfloat16(), rand(N), rand(M, N)

    def call(m):
        out = x0[:m].clone() if epi == 2 else torch.empty(m, N, dtype=torch.bfloat16, device="cuda")
        _lib.check(lib.regenvc_linear_fwd(a.data_ptr(), K, w.data_ptr(), b.data_ptr(), gate.data_ptr() if epi == 2 else None,
                                          out.data_ptr(), N, m, N, K, epi,
                                          ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)), "regenvc_linear_fwd")
        return out
    whole = call(M)
    for m in rows:
        assert torch.equal(call(m), whole[:m]), m


def test_linear_split_workspace_sizes():
    """The split-K form under a workspace that is missing, too small for any
    split, enough for some and enough for all ranges."""
    import ctypes
    from paper_2607_28144_amd import _lib
    M, N, K = 300, 1536, 8960
    rng = np.random.default_rng(6)
    a, w = bits(rng, (M, K)), bits(rng, (N, K), 0.02)
    y = odit.gemm(odit.widen(a), odit.widen(w), np.zeros(N))
    slack = 2 * ACC * (np.abs(odit.widen(a)) @ np.abs(odit.widen(w)).T)
    da, dw = dev_bits(a), dev_bits(w)
    full = kern().linear_workspace_bytes(M, N, K, "bias", da.device)
    plane = M * N * 4
    assert full >= 2 * plane
    lib = _lib.load()
    for need in (0, 256, 2 * plane, 3 * plane + 256, full):
        ws = torch.full((max(need, 1) + 512,), 0x7F, dtype=torch.uint8, device="cuda")
        out = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
        st = lib.regenvc_linear_fwd_ws(da.data_ptr(), K, dw.data_ptr(), None, None, out.data_ptr(), N, M, N, K, 0,
                                       ws.data_ptr() if need else None, need,
                                       ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        _lib.check(st, "regenvc_linear_fwd_ws")
        torch.cuda.synchronize()
        assert bool((ws[need:] == 0x7F).all()), "written past the workspace"
        check_bound(f"linear split, workspace {need}", host(out), y, ULP * np.abs(y) + slack)


def test_linear_without_bias_or_gate_into_a_strided_output():
    """No bias, no gate (1), the output a column slice of a wider buffer."""
    rng = np.random.default_rng(5)
    M, N, K = 400, 512, 1536
    a, w = bits(rng, (M, K)), bits(rng, (N, K), 0.02)
    wide = torch.zeros((M, N + 256), dtype=torch.float32, device="cuda")
    kern().linear_fwd(dev_bits(a), dev_bits(w), None, "gated_residual", out=wide[:, 128:128 + N])
    torch.cuda.synchronize()
    y = odit.gemm(odit.widen(a), odit.widen(w))
    slack = 2 * ACC * (np.abs(odit.widen(a)) @ np.abs(odit.widen(w)).T)
    got = host(wide)
    check_bound("linear plain into a column slice", got[:, 128:128 + N], y, slack + 1e-7)
    assert np.all(got[:, :128] == 0) and np.all(got[:, 128 + N:] == 0)


def test_layer_norm_both_forms():
    rng = np.random.default_rng(6)
    rows, C = 777, 1536
    x = (rng.standard_normal((rows, C)) * 3 + 0.5).astype(np.float32)
    shift, scale = rng.standard_normal(C).astype(np.float32), rng.standard_normal(C).astype(np.float32)
    w, b = bits(rng, (C,)), bits(rng, (C,))
    dx = torch.from_numpy(x).cuda()
    y1 = kern().layer_norm_fwd(dx, shift=torch.from_numpy(shift).cuda(), scale=torch.from_numpy(scale).cuda())
    y2 = kern().layer_norm_fwd(dx, w=dev_bits(w), b=dev_bits(b))
    torch.cuda.synchronize()
    ln = odit.layer_norm(x.astype(np.float64))
    r1 = odit.modulate(ln, shift.astype(np.float64), scale.astype(np.float64))
    r2 = ln * odit.widen(w) + odit.widen(b)
    check_bound("layer norm, modulated", host(y1), r1, ULP * np.abs(r1) + 1e-5 * (1 + np.abs(ln) * (1 + np.abs(scale))))
    check_bound("layer norm, affine", host(y2), r2, ULP * np.abs(r2) + 1e-5 * (1 + np.abs(ln * odit.widen(w))))


def test_rms_norm_in_place():
    rng = np.random.default_rng(7)
    rows, C = 555, 1536
    x, w = bits(rng, (rows, C), 2.0), synth.f32_to_bf16_bits(1 + 0.1 * rng.standard_normal(C).astype(np.float32))
    dx = dev_bits(x)
    kern().rms_norm_fwd(dx, dev_bits(w), out=dx)
    torch.cuda.synchronize()
    ref = odit.rms_norm(odit.widen(x), odit.widen(w))
    check_bound("rms norm in place", host(dx), ref, ULP * np.abs(ref) + 1e-5 * (1 + np.abs(ref)))


def test_modulation_vectors():
    rng = np.random.default_rng(8)
    C = 1536
    w, b = bits(rng, (6 * C, C), 0.02), bits(rng, (6 * C,), 0.02)
    e = rng.standard_normal(C).astype(np.float32)
    out = kern().modulation(dev_bits(w).view(6 * C, C), dev_bits(b), torch.from_numpy(e).cuda())
    torch.cuda.synchronize()
    ref = odit.modulation(e.astype(np.float64), odit.widen(w), odit.widen(b)).reshape(-1)
    s = odit.silu(e.astype(np.float64))
    check_bound("adaLN modulation", out.cpu().numpy().astype(np.float64), ref,
                2 * ACC * (np.abs(odit.widen(w)) @ np.abs(s)) + 1e-7)


def test_modulation_vectors_any_width():
    """Widths that are not a multiple of 8 (and a row count that is not a
    multiple of the rows per wave) take the scalar form of the kernel; the
    vector form's partial last group of rows is covered by 6 x 1536 - 4 rows."""
    rng = np.random.default_rng(9)
    for rows, C in [(21, 100), (6 * 1536 - 4, 1536)]:
        w, b = bits(rng, (rows, C), 0.02), bits(rng, (rows,), 0.02)
        e = rng.standard_normal(C).astype(np.float32)
        out = kern().modulation(dev_bits(w).view(rows, C), dev_bits(b), torch.from_numpy(e).cuda())
        torch.cuda.synchronize()
        s = odit.silu(e.astype(np.float64))
        ref = odit.gemm(s[None, :], odit.widen(w), odit.widen(b)).reshape(-1)
        check_bound(f"adaLN modulation rows={rows} C={C}", out.cpu().numpy().astype(np.float64), ref,
                    2 * ACC * (np.abs(odit.widen(w)) @ np.abs(s)) + 1e-7)


# ------------------------------------------------------------------ the block
def device_block(params):
    return kern().DitBlock({n: dev_bits(v) for n, v in params.items()})


def rel_errors(got, ref):
    d = got - ref
    return float(np.sqrt((d * d).mean() / (ref * ref).mean())), float(np.abs(d).max() / np.abs(ref).max())


def jittered_oracle(seed: int, rel: float = 1e-5):
    """A copy of the block oracle whose every bf16 storage point rounds the
    value times (1 + rel * N(0, 1)): a second correct bf16 implementation,
    differing from the first only in last bits before each rounding."""
    import types
    src = open(odit.__file__).read()
    mod = types.ModuleType("oracle._dit_jittered")
    mod.__package__ = "oracle"
    mod.__file__ = odit.__file__
    exec(compile(src, odit.__file__ + " (jittered)", "exec"), mod.__dict__)
    rng = np.random.default_rng(seed)
    exact = mod.round_bf16
    mod.round_bf16 = lambda x: exact(np.asarray(x) * (1.0 + rel * rng.standard_normal(np.shape(x))))
    return mod


def block_errors(name, got, ref, ref2):
    """GPU vs oracle, held to twice the oracle's own spread (ref2: the
    jittered oracle)."""
    rms, mx = rel_errors(got, ref)
    rms2, mx2 = rel_errors(ref2, ref)
    print(f"[dit] {name}: max|dx|={np.abs(got - ref).max():.3e} (max|x|={np.abs(ref).max():.3e}) "
          f"rms|dx|/rms|x|={rms:.3e} max|dx|/max|x|={mx:.3e}; bf16 spread of the oracle: rms {rms2:.3e} "
          f"max {mx2:.3e}", flush=True)
    assert np.all(np.isfinite(got))
    assert rms <= 2 * rms2 and mx <= 2 * mx2 + 1e-4, name


def test_block_four_steps_every_row():
    """A 7 x 6 x 8 latent window (336 tokens), 12 heads x 128, 64 context
    tokens, four denoising steps: every row of the residual stream."""
    params = synth.dit_params(11)
    x, e, kc, vc = synth.dit_inputs(12, 7 * 6 * 8, 64)
    blk = device_block(params)
    dx = torch.from_numpy(x).cuda()
    dk, dv = dev_bits(kc), dev_bits(vc)
    ref = x.astype(np.float64)
    ref2 = ref.copy()
    jit = jittered_oracle(1)
    for s in range(4):
        blk.forward(dx, torch.from_numpy(e[s]).cuda(), dk, dv, (7, 6, 8))
        ref = odit.block(ref, e[s], params, kc, vc, (7, 6, 8))
        ref2 = jit.block(ref2, e[s], params, kc, vc, (7, 6, 8))
        torch.cuda.synchronize()
        block_errors(f"block step {s + 1}, 336 tokens", dx.cpu().numpy().astype(np.float64), ref, ref2)


def test_block_workspace_without_room_for_partial_sums():
    """A block call is taken from the attention calls' share of the scratch
    (one byte less is refused) to the queried size, and writes no byte behind
    what it was given: every row against the oracle at three sizes."""
    S, S_ctx, C, F, align = 336, 64, 1536, 8960, lambda b: (b + 255) // 256 * 256
    params = synth.dit_params(11)
    x, e, kc, vc = synth.dit_inputs(12, S, S_ctx, steps=1)
    blk = device_block(params)
    dk, dv, de = dev_bits(kc), dev_bits(vc), torch.from_numpy(e[0]).cuda()
    from paper_2607_28144_amd import attn_plan
    n_cu = torch.cuda.get_device_properties(dk.device).multi_processor_count
    plans = [attn_plan(1, 12, S, n, 128, n_cu) for n in (S, S_ctx)]
    least = (align(6 * C * 4) + align(S * C * 2) * 2 + align(S * 3 * C * 2) + align(S * F * 2) +
             align(max(p["workspace_bytes"] for p in plans)))
    full = blk.workspace_bytes(S, S_ctx, dk.device)
    assert least == blk.workspace_bytes(S, S_ctx, dk.device, least=True) < full
    ref = odit.block(x.astype(np.float64), e[0], params, kc, vc, (7, 6, 8))
    ref2 = jittered_oracle(1).block(x.astype(np.float64), e[0], params, kc, vc, (7, 6, 8))
    for size in (least, align((least + full) // 2), full):
        ws = torch.full((full + 256,), 0x5A, dtype=torch.uint8, device="cuda")
        blk._ws = {(dk.device.index, S, S_ctx): ws[:size]}
        dx = torch.from_numpy(x).cuda()
        blk.forward(dx, de, dk, dv, (7, 6, 8))
        torch.cuda.synchronize()
        assert bool((ws[size:] == 0x5A).all()), "written past the workspace"
        block_errors(f"block, workspace of {size} bytes", dx.cpu().numpy().astype(np.float64), ref, ref2)
    blk._ws = {(dk.device.index, S, S_ctx): ws[:least - 1]}
    with pytest.raises(RuntimeError, match="workspace"):
        blk.forward(dx, de, dk, dv, (7, 6, 8))


def test_block_window_shape_one_step_sampled_rows():
    """The workload's window: 10920 tokens (7 x 30 x 52), 12 heads x 128,
    512 context tokens, one step; sampled rows of the residual stream against
    the oracle (whose self-attention still sees every key)."""
    params = synth.dit_params(21)
    S = 7 * 30 * 52
    x, e, kc, vc = synth.dit_inputs(22, S, 512, steps=1)
    blk = device_block(params)
    dx = torch.from_numpy(x).cuda()
    blk.forward(dx, torch.from_numpy(e[0]).cuda(), dev_bits(kc), dev_bits(vc), (7, 30, 52))
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([[0, 1, 255, 256, 1559, 1560, S // 2, S - 2, S - 1],
                                     np.random.default_rng(23).choice(S, 64, replace=False)]))
    ref = odit.block(x.astype(np.float64), e[0], params, kc, vc, (7, 30, 52), rows=rows)
    ref2 = jittered_oracle(2).block(x.astype(np.float64), e[0], params, kc, vc, (7, 30, 52), rows=rows)
    block_errors("block window one step (sampled rows)", dx.cpu().numpy().astype(np.float64)[rows], ref, ref2)


def test_block_on_two_streams_at_once():
    """One block, two inputs, each stepped on a stream of its own without
    waiting for the other: bitwise the outputs of the calls one by one."""
    S, S_ctx, grid = 336, 64, (7, 6, 8)
    blk = device_block(synth.dit_params(11))
    x, e, kc, vc = synth.dit_inputs(12, S, S_ctx, steps=2)
    dk, dv, de = dev_bits(kc), dev_bits(vc), [torch.from_numpy(v).cuda() for v in e]
    xs = [torch.from_numpy(x).cuda(), torch.from_numpy(x[::-1].copy()).cuda()]
    ref = [t.clone() for t in xs]
    for r in ref:
        for _ in range(4):
            for v in de:
                blk.forward(r, v, dk, dv, grid)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in xs]
    for _ in range(4):
        for v in de:
            for t, s in zip(xs, streams):
                with torch.cuda.stream(s):
                    blk.forward(t, v, dk, dv, grid)
    torch.cuda.synchronize()
    for t, r in zip(xs, ref):
        assert torch.equal(t, r)


def test_block_and_split_linear_in_a_graph():
    """A block step and a linear layer with K split, captured (their
    workspaces come from the graph's pool): replays with eager calls between
    them give the eager results, bitwise."""
    S, S_ctx, grid = 336, 64, (7, 6, 8)
    blk = device_block(synth.dit_params(11))
    x, e, kc, vc = synth.dit_inputs(12, S, S_ctx, steps=1)
    dk, dv, de, x0 = dev_bits(kc), dev_bits(vc), torch.from_numpy(e[0]).cuda(), torch.from_numpy(x).cuda()
    rng = np.random.default_rng(9)
    a, w = dev_bits(bits(rng, (300, 8960))), dev_bits(bits(rng, (1536, 8960), 0.02))
    assert kern().linear_workspace_bytes(300, 1536, 8960, "bias", a.device) > 0

    def step(t):
        return blk.forward(t, de, dk, dv, grid), kern().linear_fwd(a, w)
    ref = step(x0.clone())
    t = x0.clone()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        t.copy_(x0)
        got = step(t)
    for _ in range(4):
        graph.replay()
        eager = step(x0.clone())
        torch.cuda.synchronize()
        for g, q, r in zip(got, eager, ref):
            assert torch.equal(g, r) and torch.equal(q, r)

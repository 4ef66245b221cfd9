"""GPU parity: the HIP library (through its C ABI) against the CPU oracle, element by
element, on seeded inputs that span several tiles and ragged tails."""
import types

import numpy as np
import pytest
import torch

import paper_2605_18739_amd as nv
from paper_2605_18739_amd import workloads as wl
from tests.parity import assert_gemm_close, assert_q_equal, dev_bf16, host_q

pytestmark = pytest.mark.gpu


def say(msg):
    print(msg, flush=True)


# ------------------------------------------------------------------ quantize

def _quant_case(oracle, xb, what, **kw):
    say(f"[quantize] {what} shape={xb.shape}")
    oq = oracle.quantize(xb)
    gq = nv.nvfp4_quantize(dev_bf16(xb))
    assert_q_equal(gq, oq, what)
    return oq, gq


def test_quantize_config1(oracle):
    cfg = wl.config1()
    _quant_case(oracle, cfg["A"], "config1 A")
    _quant_case(oracle, cfg["W"], "config1 W")


@pytest.mark.parametrize("R,C", [(1, 16), (3, 48), (257, 272), (64, 4096), (1000, 1040)])
def test_quantize_ragged_shapes(oracle, R, C):
    g = np.random.default_rng(R * 7 + C)
    x = g.standard_normal((R, C)).astype(np.float32) * np.float32(10.0 ** g.uniform(-3, 3))
    _quant_case(oracle, wl.to_bf16_bits(x), f"ragged {R}x{C}")


def test_quantize_outliers_small_weights_and_gradients(oracle):
    _quant_case(oracle, wl.activation_with_outliers(300, 3072, 1, 0), "outlier activations")
    _quant_case(oracle, wl.normal((256, 3072), 0.02, 1, 1), "weights sigma 0.02")
    _quant_case(oracle, wl.normal((128, 14336), 1e-3, 4, 2), "gradients sigma 1e-3")


def test_quantize_degenerate(oracle):
    z = np.zeros((8, 64), np.float32)
    _quant_case(oracle, wl.to_bf16_bits(z), "all zero")
    z[3, 17] = -0.0
    z[5, 40] = 3.0            # one non-zero element: every other block is all zero
    _quant_case(oracle, wl.to_bf16_bits(z), "single element")
    z[:] = 1.0
    _quant_case(oracle, wl.to_bf16_bits(z), "constant")
    big = np.full((4, 32), 3.0e38, np.float32)
    big[0, :16] = 1e-30       # block scale underflows to 0
    _quant_case(oracle, wl.to_bf16_bits(big), "huge and tiny")


def test_quantize_tie_heavy(oracle):
    """amax = 5.25 gives s_g = 2^-9 exactly; small-integer multiples of 2^-k then land
    on rounding midpoints all the time, which exercises the exact slow path."""
    g = np.random.default_rng(17)
    x = g.integers(-40, 41, size=(128, 256)).astype(np.float32) * np.float32(0.125)
    x[x > 5.25] = 5.25
    x[x < -5.25] = -5.25
    x[7, 100] = 5.25
    _quant_case(oracle, wl.to_bf16_bits(x), "tie heavy s_g=2^-9")
    x2 = g.integers(-21, 22, size=(64, 128)).astype(np.float32)
    x2[0, 0] = 21.0           # s_g = 21/2688 = 2^-7
    _quant_case(oracle, wl.to_bf16_bits(x2), "integers s_g=2^-7")


def test_quantize_given_scale_and_stride(oracle):
    g = np.random.default_rng(23)
    xb = wl.to_bf16_bits(g.standard_normal((100, 200)).astype(np.float32))   # padded rows: ld = 200, C = 176
    x = dev_bf16(xb)
    view = x[:, :176]
    oq = oracle.quantize(np.ascontiguousarray(xb[:, :176]))
    assert_q_equal(nv.nvfp4_quantize(view), oq, "strided")
    for gs in (2.0 ** -9, 0.0011, 0.02):
        gsd = torch.tensor([gs], dtype=torch.float32, device="cuda")
        oq = oracle.quantize(np.ascontiguousarray(xb[:, :176]), global_scale_in=gs)
        assert_q_equal(nv.nvfp4_quantize(view, global_scale_in=gsd), oq, f"given scale {gs}")


@pytest.mark.parametrize("R,C,ld", [(1, 16, 24), (700, 16, 24), (333, 48, 56), (129, 1008, 1016), (1000, 3088, 3104), (65, 4096, 4104)])
@pytest.mark.parametrize("search", [False, True])
def test_quantize_padded_rows_of_many_widths(oracle, R, C, ld, search):
    """Rows cut out of a wider buffer: the kernels find a block's row by dividing by the width (one block, powers of two, odd)."""
    xb = wl.to_bf16_bits(np.random.default_rng(R + C).standard_normal((R, ld)).astype(np.float32))
    want = oracle.quantize(np.ascontiguousarray(xb[:, :C]), four_over_six=search)
    view = dev_bf16(xb)[:, :C]
    assert_q_equal(nv.nvfp4_quantize_4over6(view) if search else nv.nvfp4_quantize(view), want, f"{R}x{C} of {ld}")


@pytest.mark.parametrize("R,C,ld", [(1100, 4112, 4120), (2100, 4112, 4120), (5836, 4112, 4128), (5837, 4112, 4128)])
def test_quantize_padded_rows_of_several_turns_a_lane(oracle, R, C, ld):
    """Padded rows of 257 blocks each: with 1024 workgroups a lane of the search comes to its second turn at 262 144 blocks and one of the plain
    rule at 524 288; 1.5 M blocks (between the last two) is where the plain rule goes from four blocks to a lane to two."""
    say(f"[quantize] {R}x{C} of {ld}")
    xb = wl.to_bf16_bits(np.random.default_rng(R).standard_normal((R, ld)).astype(np.float32))
    xc = np.ascontiguousarray(xb[:, :C])
    view = dev_bf16(xb)[:, :C]
    want = oracle.quantize(xc)
    plain = nv.nvfp4_quantize(view)
    assert_q_equal(plain, want, "plain")
    assert_q_equal(nv.nvfp4_quantize(view, global_scale_in=plain.global_scale), want, "given scale")
    assert_q_equal(nv.nvfp4_quantize_4over6(view), oracle.quantize(xc, four_over_six=True), "search")


@pytest.mark.parametrize("offset", [0.0, 2.0 ** -23, -2.0 ** -23, 2.0 ** -19, -2.0 ** -19, -2.0 ** -17, 2.0 ** -16])
def test_quantize_tensor_scales_on_and_beside_ties(oracle, offset):
    """Given scales (bf16 number) / (odd number below 128), and the same a little off: elements and block maxima of
    bf16 numbers next to the midpoints, through the row, column, tile and scale-search encoders."""
    g = np.random.default_rng(97)
    T = np.array([0.25, 0.75, 1.25, 1.75, 2.5, 3.5, 5.0])
    for c in (1, 3, 5, 7, 21, 35, 49, 91, 105, 51, 93, 17, 31):
        gs = np.float32(float(g.integers(128, 256)) / c * (1.0 + offset) * 2.0 ** -9)
        say(f"[near ties] scale {gs!r}")
        sb = wl.bf16_bits_to_f32(wl.to_bf16_bits(g.integers(8, 16, (128, 16)) * 2.0 ** g.integers(-13, 4, (128, 16)).astype(np.float32)))
        x = T[g.integers(0, 7, (128, 16, 16))] * sb[:, :, None] * gs * g.choice([-1.0, 1.0], (128, 16, 16))
        top = np.where(g.random((128, 16)) < 0.5, 6.0, 6.0 * (1.0 + 1.0 / 16))          # maxima on a block scale / on a midpoint
        x[:, :, 3] = top * sb * gs
        xb = wl.to_bf16_bits(x.reshape(128, 256).astype(np.float32))
        gsd = torch.tensor([gs], dtype=torch.float32, device="cuda")
        xd = dev_bf16(xb)
        assert_q_equal(nv.nvfp4_quantize(xd, global_scale_in=gsd), oracle.quantize(xb, global_scale_in=gs), f"rows {gs!r}")
        assert_q_equal(nv.nvfp4_quantize_4over6(xd, global_scale_in=gsd), oracle.quantize(xb, global_scale_in=gs, four_over_six=True), f"search {gs!r}")
        xt = np.ascontiguousarray(xb.T)
        assert_q_equal(nv.nvfp4_quantize(dev_bf16(xt), block_axis=1, global_scale_in=gsd), oracle.quantize(xt, block_axis=1, global_scale_in=gs), f"columns {gs!r}")
        got, want = nv.nvfp4_quantize_2d(xd, global_scale_in=gsd), oracle.quantize_2d(xb, global_scale_in=gs)
        assert_q_equal(got[0], want[0], f"tiles {gs!r}")
        assert_q_equal(got[1], want[1], f"tiles transposed {gs!r}")


@pytest.mark.parametrize("R,C", [(16, 8), (48, 24), (128, 256), (400, 520), (1024, 3072)])
def test_quantize_transposed(oracle, R, C):
    g = np.random.default_rng(R + C)
    xb = wl.to_bf16_bits(g.standard_normal((R, C)).astype(np.float32) * np.float32(0.3))
    say(f"[quantize^T] {R}x{C}")
    oq = oracle.quantize(xb, block_axis=1)
    gq = nv.nvfp4_quantize(dev_bf16(xb), block_axis=1)
    assert gq.rows == C and gq.K == R
    assert_q_equal(gq, oq, f"transposed {R}x{C}")


def test_quantize_random_sweep(oracle):
    """Seeded sweep over shapes, leading dimensions, value distributions (Gaussian at many
    magnitudes, coarse grids full of rounding ties, heavy tails, mostly-zero tensors), both block
    axes, the plain rule and the scale search: every byte equals the oracle's."""
    g = np.random.default_rng(4242)
    for case in range(48):
        axis = int(g.integers(0, 2))
        if axis == 0:
            R, C = int(g.integers(1, 500)), 16 * int(g.integers(1, 66))
        else:
            R, C = 16 * int(g.integers(1, 40)), 8 * int(g.integers(1, 130))
        kind = case % 6
        if kind == 0:
            x = g.standard_normal((R, C)) * 10.0 ** g.uniform(-6, 6)
        elif kind == 1:                                       # a grid of 1/8 steps under a power-of-two tensor scale
            x = g.integers(-42, 43, size=(R, C)) * 0.125
            x.flat[0] = 5.25
        elif kind == 2:                                       # heavy tails
            x = g.standard_cauchy((R, C)).clip(-1e4, 1e4)
        elif kind == 3:                                       # mostly zeros, signed zeros included
            x = np.where(g.random((R, C)) < 0.9, 0.0, g.standard_normal((R, C)))
            x = np.where(g.random((R, C)) < 0.05, -0.0, x)
        elif kind == 4:                                       # channels of very different size
            x = g.standard_normal((R, C)) * 2.0 ** g.integers(-12, 13, size=(1, C))
        else:                                                 # values that are exactly representable
            x = g.choice([0.5, 1, 1.5, 2, 3, 4, 6], size=(R, C)) * g.choice([-1.0, 1.0], size=(R, C)) * 2.0 ** g.integers(-3, 4, size=(R, 1))
        pad = 8 * int(g.integers(0, 3))
        xb = wl.to_bf16_bits(np.asarray(x, np.float32))
        full = np.zeros((R, C + pad), np.uint16)
        full[:, :C] = xb
        view = dev_bf16(full)[:, :C]
        search = axis == 0 and case % 2 == 1
        say(f"[quantize] sweep {case}: {R}x{C} ld={C + pad} axis={axis} kind={kind} search={search}")
        if search:
            got = nv.nvfp4_quantize_4over6(view)
            want = oracle.quantize(xb, four_over_six=True)
        else:
            got = nv.nvfp4_quantize(view, block_axis=axis)
            want = oracle.quantize(xb, block_axis=axis)
        assert_q_equal(got, want, f"sweep {case}")


def test_quantize_more_than_2_to_31_elements(oracle):
    """A tensor past 2^31 elements (4.3 GB of bf16): every index in the kernels is 64-bit.  The tensor
    is drawn on the device; rows around the 2^31-element mark, the first and last rows and seeded
    ones are checked against the oracle, which gets the tensor scale the way the kernel finds it
    (from the one largest element, planted in the last row)."""
    R, C = 66000, 32768
    assert R * C > 2 ** 31
    say(f"[quantize] {R}x{C} = {R * C / 2 ** 30:.2f} Gi elements")
    x = torch.empty((R, C), dtype=torch.bfloat16, device="cuda")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(31)
    for r0 in range(0, R, 4000):
        r1 = min(R, r0 + 4000)
        x[r0:r1] = torch.randn((r1 - r0, C), generator=gen, device="cuda").to(torch.bfloat16)
    x[R - 1, C - 1] = 77.0                          # larger than any N(0,1) draw
    for axis in (0, 1):
        say(f"[quantize] {R}x{C} block_axis={axis}")
        q = nv.nvfp4_quantize(x, block_axis=axis)
        torch.cuda.synchronize()
        gs = oracle.global_scale(wl.to_bf16_bits(np.array([[77.0]], np.float32)))
        assert np.float32(q.global_scale.cpu().numpy()[0]).view(np.uint32) == np.float32(gs).view(np.uint32)
        g = np.random.default_rng(axis)
        if axis == 0:
            rows = np.unique(np.concatenate([[0, 1, 65535, 65536, 65537, R - 2, R - 1], g.integers(0, R, 8)]))
            xb = nv.bits_from_bf16(x[torch.as_tensor(rows, device="cuda")])
            want = oracle.quantize(xb, global_scale_in=gs)
            sel = torch.as_tensor(rows, device="cuda")
            assert (q.codes[sel].cpu().numpy() == want.codes).all()
            assert (q.scales[sel].cpu().numpy() == want.scales).all()
        else:
            # blocks run along the rows: output row = input column; check whole output rows
            cols = np.unique(np.concatenate([[0, 1, C - 1], g.integers(0, C, 5)]))
            sel = torch.as_tensor(cols, device="cuda")
            xb = nv.bits_from_bf16(x[:R - R % 16][:, sel].t().contiguous())
            want = oracle.quantize(xb, global_scale_in=gs)
            assert (q.codes[sel].cpu().numpy() == want.codes).all()
            assert (q.scales[sel].cpu().numpy() == want.scales).all()
        del q
    del x
    torch.cuda.empty_cache()


def test_quantize_one_launch_path_with_and_without_the_grid_wide_wait(oracle):
    """Tensors that fit on the chip are quantized by one launch whose workgroups exchange their maxima through
    a bounded grid-wide wait.  With the bound set to zero from the host every workgroup gives up at once and
    derives the tensor maximum from the tensor itself: same bytes, every kernel still ends normally.  Sizes: one
    workgroup; many workgroups, one block per lane with a ragged tail; several register slots; register and
    LDS slots together (more than 20 blocks per lane on 256 workgroups)."""
    g = np.random.default_rng(2024)
    cases = [(40, 208), (1000, 1040), (3520, 3072), (22000, 2048)]
    tensors = []
    for R, C in cases:
        x = g.standard_normal((R, C)).astype(np.float32)
        x[g.integers(0, R), g.integers(0, C)] = 300.0          # the tensor maximum sits in ONE workgroup's slice
        tensors.append(wl.to_bf16_bits(x))
    want = [(oracle.quantize(b), oracle.quantize(b, four_over_six=True)) for b in tensors]
    kb = wl.to_bf16_bits(wl.bf16_bits_to_f32(wl.kv_tensor(300, 24, 128, 8, 1)).reshape(7200, 128) + np.float32(1.5))
    want_k = _oracle_k_path(oracle, kb)
    for limit in (None, 0):
        say(f"[one launch] wait bound {'default' if limit is None else limit}")
        nv.nvfp4_set_one_launch(nv.ONE_LAUNCH_ALWAYS)          # at these sizes the default rule would partly take two passes
        if limit is not None:
            nv.nvfp4_set_sync_spin_limit(limit)
        try:
            for b, (w6, w46) in zip(tensors, want):
                assert_q_equal(nv.nvfp4_quantize(dev_bf16(b)), w6, f"plain {b.shape} limit {limit}")
                assert_q_equal(nv.nvfp4_quantize_4over6(dev_bf16(b)), w46, f"search {b.shape} limit {limit}")
            gq, gm = nv.nvfp4_kv_quant_k(dev_bf16(kb).reshape(300, 24, 128))
            assert (nv.bits_from_bf16(gm) == want_k[0]).all()
            assert_q_equal(gq, want_k[1], f"smoothed keys limit {limit}")
        finally:
            nv.nvfp4_set_sync_spin_limit()                     # back to the default bound
            nv.nvfp4_set_one_launch()                          # and to the default rule


def test_one_launch_and_two_pass_forms_return_the_same_bytes(oracle):
    """Which form a tensor that fits on the chip takes is a matter of speed (nvfp4_set_one_launch): always, never
    and the default rule give the oracle's bytes for the plain rule, the scale search, the smoothed keys and the
    all-to-all packer, at a small, a middle and a large size."""
    for T, H, d in ((40, 4, 64), (4620, 24, 128), (14000, 24, 128)):
        kb = wl.kv_tensor(T, H, d, 31, T).reshape(T * H, d)
        want, want46 = oracle.quantize(kb), oracle.quantize(kb, four_over_six=True)
        want_mean, want_k = _oracle_k_path(oracle, kb)
        kv = dev_bf16(kb).reshape(T, H, d)
        for mode in (nv.ONE_LAUNCH_ALWAYS, nv.ONE_LAUNCH_NEVER, nv.ONE_LAUNCH_AUTO):
            say(f"[one launch] mode {mode}, {T}x{H}x{d}")
            nv.nvfp4_set_one_launch(mode)
            try:
                assert_q_equal(nv.nvfp4_kv_quant(kv), want, f"plain, mode {mode}")
                assert_q_equal(nv.nvfp4_kv_quant_4over6(kv), want46, f"search, mode {mode}")
                gq, gm = nv.nvfp4_kv_quant_k(kv)
                assert (nv.bits_from_bf16(gm) == want_mean).all()
                assert_q_equal(gq, want_k, f"smoothed keys, mode {mode}")
                codes, scales, gs = host_q(nv.nvfp4_quantize_for_all_to_all(kv, 2))
                slabs = lambda a: a.reshape(T, 2, H // 2, -1).transpose(1, 0, 2, 3).reshape(T * H, -1)
                assert (codes == slabs(want.codes)).all() and (scales == slabs(want.scales)).all(), f"all-to-all, mode {mode}"
            finally:
                nv.nvfp4_set_one_launch()


@pytest.mark.parametrize("magnitude", [1e-33, 1e-36, 3e-39, 1e30, 3e37])
def test_quantize_tensor_scales_outside_the_fp32_safe_range(oracle, magnitude):
    """Tensors whose scale amax / 2688 lies below 2^-100 or above 2^100 (the reciprocal 1 / (6 s_g) and the products
    s_b s_g leave the normal fp32 range there, bf16 subnormals included): every route through the quantizers -- one
    launch, streaming with a padded row stride, a given scale, blocks along the rows, the scale search, 16 x 16
    tiles -- still returns the oracle's bytes."""
    g = np.random.default_rng(int(-np.log10(magnitude)) + 100)
    R, C = 96, 208
    xb = wl.to_bf16_bits(g.standard_normal((R, C)).astype(np.float32) * np.float32(magnitude))
    say(f"[quantize] magnitude {magnitude}: one launch")
    want = oracle.quantize(xb)
    assert_q_equal(nv.nvfp4_quantize(dev_bf16(xb)), want, f"one launch {magnitude}")
    assert_q_equal(nv.nvfp4_quantize_4over6(dev_bf16(xb)), oracle.quantize(xb, four_over_six=True), f"search {magnitude}")
    full = np.zeros((R, C + 16), np.uint16)
    full[:, :C] = xb
    view = dev_bf16(full)[:, :C]
    say(f"[quantize] magnitude {magnitude}: streaming, padded rows")
    assert_q_equal(nv.nvfp4_quantize(view), want, f"strided {magnitude}")
    assert_q_equal(nv.nvfp4_quantize_4over6(view), oracle.quantize(xb, four_over_six=True), f"strided search {magnitude}")
    gs = float(want.global_scale) * 1.5
    gsd = torch.tensor([gs], dtype=torch.float32, device="cuda")
    if np.isfinite(np.float32(gs)) and np.float32(gs) > 0:
        say(f"[quantize] magnitude {magnitude}: given scale")
        assert_q_equal(nv.nvfp4_quantize(dev_bf16(xb), global_scale_in=gsd),
                       oracle.quantize(xb, global_scale_in=float(np.float32(gs))), f"given scale {magnitude}")
    say(f"[quantize] magnitude {magnitude}: blocks along the rows")
    assert_q_equal(nv.nvfp4_quantize(dev_bf16(xb), block_axis=1), oracle.quantize(xb, block_axis=1), f"transposed {magnitude}")


def test_binding_refuses_tensors_it_cannot_marshal():
    x = torch.zeros((32, 64), dtype=torch.bfloat16, device="cuda")
    for bad in (x.float(), x.t(), x[0], x[:, ::2]):
        with pytest.raises(AssertionError):
            nv.nvfp4_quantize(bad, out=nv.NVFP4Tensor(32, 64))
    for bad in (x.view(2, 16, 64).float(), x.view(2, 16, 64)[:, :, :32], x):
        with pytest.raises(AssertionError):
            nv.nvfp4_kv_quant(bad, out=nv.NVFP4Tensor(32, 64))
    q = nv.nvfp4_quantize(x)
    with pytest.raises((AttributeError, TypeError)):
        nv.nvfp4_gemm(q, (q.codes, q.scales), Y=torch.empty((32, 32), device="cuda"))
    with pytest.raises(nv.NVFP4Error):                                   # refused by the library, nothing launched
        nv.nvfp4_gemm(q, nv.nvfp4_quantize(x[:, :32]), Y=torch.empty((32, 32), device="cuda"))
    with pytest.raises(nv.NVFP4Error):
        nv.nvfp4_quantize(x, workspace=torch.empty(16, dtype=torch.uint8, device="cuda"))


def _pool_of(t):
    """The stream whose pool a tensor's memory belongs to."""
    return next(s["stream"] for s in torch.cuda.memory_snapshot() if s["address"] <= t.data_ptr() < s["address"] + s["total_size"])


def test_calls_on_another_stream_allocate_from_its_pool():
    """stream= another stream than the current one: outputs and workspaces come from that stream's pool (no block that
    the current stream still uses, none that it is handed back too early), the results are the same, and the current
    stream stays what it is.  With buffers given, or with the current stream itself, nothing changes pools."""
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    x = torch.randn((256, 512), generator=g, device="cuda").to(torch.bfloat16)
    kv = x.view(256, 4, 128)
    a, b = x[:128].contiguous(), torch.randn((256, 128), generator=g, device="cuda").to(torch.bfloat16)
    q = nv.nvfp4_quantize(x)
    t = nv.nvfp4_lora_down(x, a)
    qk, mean = nv.nvfp4_kv_quant_k(kv)
    calls = [lambda **kw: nv.nvfp4_quantize(x, **kw), lambda **kw: nv.nvfp4_quantize(x, block_axis=1, **kw), lambda **kw: nv.nvfp4_gemm(q, q, **kw),
             lambda **kw: nv.nvfp4_gemm_scale_out(q, q, **kw), lambda **kw: nv.nvfp4_lora_down(x, a, **kw), lambda **kw: nv.nvfp4_gemm_lora(q, q, t, b, 0.5, **kw),
             lambda **kw: nv.nvfp4_gemm_act_quant(q, q, **kw), lambda **kw: nv.nvfp4_kv_quant(kv, **kw), lambda **kw: nv.nvfp4_quantize_4over6(x, **kw),
             lambda **kw: nv.nvfp4_kv_quant_4over6(kv, **kw), lambda **kw: nv.nvfp4_quantize_for_all_to_all(kv, 2, **kw),
             lambda **kw: nv.nvfp4_quantize_rht(x, 0x5A3C, **kw), lambda **kw: nv.nvfp4_quantize_2d(x, **kw), lambda **kw: nv.nvfp4_kv_quant_k(kv, **kw),
             lambda **kw: nv.nvfp4_kv_dequant_gather([(qk, mean, 256)], 4, 128, **kw), lambda **kw: nv.nvfp4_kv_dequant(q, 256, 1, 512, **kw)]

    def tensors(result):
        flat = result if isinstance(result, tuple) else (result,)
        return [u for r in flat for u in ((r.codes, r.scales, r.global_scale) if isinstance(r, nv.NVFP4Tensor) else (r,))]

    torch.cuda.synchronize()
    here, side = torch.cuda.current_stream(), torch.cuda.Stream()
    assert side.cuda_stream != here.cuda_stream
    for call in calls:
        want = tensors(call(stream=here))
        got = tensors(call(stream=side))
        raw = tensors(call(stream=types.SimpleNamespace(cuda_stream=side.cuda_stream)))     # anything that names a stream
        assert torch.cuda.current_stream() == here
        assert {_pool_of(u) for u in want} == {here.cuda_stream} and {_pool_of(u) for u in got + raw} == {side.cuda_stream}
        torch.cuda.synchronize()
        for u, v, w in zip(want, got, raw):
            assert torch.equal(u.view(torch.uint8), v.view(torch.uint8)) and torch.equal(u.view(torch.uint8), w.view(torch.uint8))
    # only the workspace is missing: it comes from the other stream's pool as well
    out = nv.NVFP4Tensor(512, 256, "cuda")
    size = nv.nvfp4_workspace_bytes(nv.OP_QUANTIZE, 256, 512)
    fresh = torch.cuda.Stream()
    torch.cuda.synchronize()
    assert nv.nvfp4_quantize(x, block_axis=1, out=out, stream=fresh) is out
    assert sum(s["total_size"] for s in torch.cuda.memory_snapshot() if s["stream"] == fresh.cuda_stream) >= size
    assert _pool_of(out.codes) == here.cuda_stream
    torch.cuda.synchronize()


@pytest.mark.parametrize("rows", [255, 256, 16383, 16384, 16385, 65537, 70000])
def test_row_encoders_of_every_grid(oracle, rows):
    """16 blocks a row: one block a lane below 1024 workgroups of 256 (16 384 rows), then up to four a lane, then more workgroups."""
    say(f"[quantize] {rows} rows of 256")
    xb = wl.normal((rows, 256), 1.0, 29, rows)
    x = dev_bf16(xb)
    nv.nvfp4_set_one_launch(nv.ONE_LAUNCH_NEVER)
    try:
        assert_q_equal(nv.nvfp4_quantize(x), oracle.quantize(xb), "plain")
        assert_q_equal(nv.nvfp4_quantize_4over6(x), oracle.quantize(xb, four_over_six=True), "search")
        want_mean, want = _oracle_k_path(oracle, xb)
        got, mean = nv.nvfp4_kv_quant_k(x.reshape(rows, 1, 256))
    finally:
        nv.nvfp4_set_one_launch()
    assert (nv.bits_from_bf16(mean) == want_mean).all()
    assert_q_equal(got, want, "smoothed")


def test_quantize_is_deterministic():
    xb = wl.activation_with_outliers(512, 3072, 1, 0)
    x = dev_bf16(xb)
    a, b = host_q(nv.nvfp4_quantize(x)), host_q(nv.nvfp4_quantize(x))
    assert (a[0] == b[0]).all() and (a[1] == b[1]).all() and a[2] == b[2]


# ------------------------------------------------------------------------ KV

@pytest.mark.parametrize("T,H,d", [(1, 1, 16), (33, 24, 128), (257, 3, 64)])
def test_kv_round_trip(oracle, T, H, d):
    say(f"[kv] T={T} H={H} d={d}")
    kb = wl.kv_tensor(T, H, d, 3, 0)
    oq = oracle.quantize(kb.reshape(T * H, d))
    kv = dev_bf16(kb)
    gq = nv.nvfp4_kv_quant(kv)
    assert_q_equal(gq, oq, "kv quant")
    back = nv.nvfp4_kv_dequant(gq, T, H, d)
    want = oracle.dequant_bf16(oq).reshape(T, H, d)
    got = nv.bits_from_bf16(back)
    bad = np.argwhere(got != want)
    assert bad.size == 0, f"kv dequant: {len(bad)} differ, first {bad[0]} gpu {got[tuple(bad[0])]:#x} oracle {want[tuple(bad[0])]:#x}"


def test_kv_dequant_awkward_scales(oracle):
    """Global scales with full 24-bit mantissas and subnormal block scales: the single
    rounding to bf16 must match the oracle's."""
    g = np.random.default_rng(5)
    rows, d = 64, 128
    codes = g.integers(0, 256, size=(rows, d // 2)).astype(np.uint8)
    scales = g.integers(0, 127, size=(rows, d // 16)).astype(np.uint8)
    for gs in (np.float32(1.0 / 2688), np.float32(0.0123456789), np.float32(3.3e-5), np.float32(1.0)):
        oq = oracle.Q(codes, scales, gs)
        want = oracle.dequant_bf16(oq)
        t = nv.NVFP4Tensor.from_host(codes, scales, gs)
        got = nv.bits_from_bf16(nv.nvfp4_kv_dequant(t, rows, 1, d)).reshape(rows, d)
        assert (got == want).all(), f"gs={gs}"


# ---------------------------------------------------------------------- GEMM

def _nan_filled(M, N, dtype):
    """An output buffer in which an unwritten element is visible: every element starts as NaN."""
    return torch.full((M, N), float("nan"), dtype=dtype, device="cuda")


def _gemm_case(oracle, ab, wb, what, rows=None, check_bf16=True):
    say(f"[gemm] {what} A{ab.shape} W{wb.shape}")
    oa, ow = oracle.quantize(ab), oracle.quantize(wb)
    ga, gw = nv.nvfp4_quantize(dev_bf16(ab)), nv.nvfp4_quantize(dev_bf16(wb))
    assert_q_equal(ga, oa, what + " A")
    assert_q_equal(gw, ow, what + " W")
    Y, S = oracle.gemm(oa, ow, rows=rows)
    y32 = nv.nvfp4_gemm(ga, gw, nv.OUT_F32, Y=_nan_filled(ga.rows, gw.rows, torch.float32))
    torch.cuda.synchronize()
    assert bool(torch.isfinite(y32).all()), f"{what}: part of the fp32 output was never written"
    y = y32.cpu().numpy()
    ysel = y if rows is None else y[rows]
    fro, worst = assert_gemm_close(ysel, Y, S, what)
    say(f"        rel fro {fro:.2e}  worst err/S {worst:.2e}")
    if check_bf16:
        y16 = nv.nvfp4_gemm(ga, gw, nv.OUT_BF16, Y=_nan_filled(ga.rows, gw.rows, torch.bfloat16))
        # bf16 output is the fp32 result rounded once, bit for bit (a tile left unwritten stays NaN and differs)
        assert (nv.bits_from_bf16(y16) == nv.bits_from_bf16(y32.to(torch.bfloat16))).all()
    return y32


def test_gemm_config1(oracle):
    cfg = wl.config1()
    _gemm_case(oracle, cfg["A"], cfg["W"], "config1")


@pytest.mark.parametrize("M,N,K", [(1, 4, 64), (100, 136, 192), (130, 260, 128), (300, 520, 64),
                                   (513, 1028, 320),
                                   (1100, 2048, 320),      # 128x128 tiles, odd number of 64-k steps
                                   # shapes that only the 64x64 tile takes: K not a multiple of 64 (16, 48, 80: one block,
                                   # a partial step, one step and a bit), N not a multiple of 8, several tiles each way
                                   (5, 12, 16), (130, 260, 48), (257, 132, 208), (64, 68, 1040), (300, 264, 80)])
def test_gemm_ragged_tiles(oracle, M, N, K):
    say(f"[gemm] ragged {M}x{N}x{K}: {nv.nvfp4_gemm_plan(M, N, K)}")
    g = np.random.default_rng(M + N + K)
    ab = wl.to_bf16_bits(g.standard_normal((M, K)).astype(np.float32))
    wb = wl.to_bf16_bits((g.standard_normal((N, K)) * 0.02).astype(np.float32))
    _gemm_case(oracle, ab, wb, f"ragged {M}x{N}x{K}")


@pytest.mark.parametrize("M,N,K", [(1, 8, 64), (63, 72, 128), (64, 64, 512), (65, 56, 576),       # whole units; 8 waves / 4 waves
                                   (130, 136, 640), (70, 200, 1600),                                # 5 units; 12 and a half
                                   (63, 68, 112), (33, 60, 144), (66, 132, 496), (40, 76, 1040)])   # scales off the dword grid, partial units
def test_gemm_tile_that_cuts_k_between_its_waves(oracle, M, N, K):
    g = np.random.default_rng(M * N + K)
    assert nv.nvfp4_gemm_plan(M, N, K)[0][0] in ("64x64", "generic")
    ab = wl.to_bf16_bits(g.standard_normal((M, K)).astype(np.float32))
    wb = wl.to_bf16_bits((g.standard_normal((N, K)) * 0.02).astype(np.float32))
    _gemm_case(oracle, ab, wb, f"K cut between waves {M}x{N}x{K}")


@pytest.mark.parametrize("M,N,K", [(40, 67, 80), (65, 129, 64), (70, 190, 208), (33, 5, 128), (3, 1, 16)])
def test_gemm_widths_that_are_no_multiple_of_4(oracle, M, N, K):
    """Odd widths in a padded Y, both output types: the last columns of a row are stored one by one and the padding is
    left alone."""
    g = np.random.default_rng(M * N + K)
    ab = wl.to_bf16_bits(g.standard_normal((M, K)).astype(np.float32))
    wb = wl.to_bf16_bits((g.standard_normal((N, K)) * 0.02).astype(np.float32))
    ga, gw = nv.nvfp4_quantize(dev_bf16(ab)), nv.nvfp4_quantize(dev_bf16(wb))
    Y, S = oracle.gemm(oracle.quantize(ab), oracle.quantize(wb))
    for pad in (4, 8):
        ldy = (N + 3) // 4 * 4 + pad
        y32, y16 = (torch.full((M, ldy), -7.0, dtype=t, device="cuda") for t in (torch.float32, torch.bfloat16))
        nv.nvfp4_gemm(ga, gw, nv.OUT_F32, Y=y32[:, :N])
        nv.nvfp4_gemm(ga, gw, nv.OUT_BF16, Y=y16[:, :N])
        assert_gemm_close(y32[:, :N].cpu().numpy(), Y, S, f"width {N}, ldy {ldy}")
        assert (nv.bits_from_bf16(y16) == nv.bits_from_bf16(y32.to(torch.bfloat16))).all()
        assert bool((y32[:, N:] == -7.0).all())


def test_gemm_random_shapes(oracle):
    """Seeded sweep over shapes that land on every tile kind of the launch plan, with ragged M and
    N tails, odd numbers of 64-k steps and multi-launch plans."""
    g = np.random.default_rng(20260518)
    kinds = set()
    shapes = [(int(g.integers(1, 900)), 8 * int(g.integers(1, 260)), 64 * int(g.integers(1, 9))) for _ in range(10)]
    shapes += [(1290, 2056, 192), (2400, 2304, 64), (4600, 1800, 320), (9000, 4104, 64), (17000, 3080, 64)]
    # whole waves of 256x256 tiles plus one or two more launches: rows below the last full wave, the tail
    # of a tile row, a main launch that ends with a whole tile row, and both kinds of leftover
    shapes += [(5489, 2928, 768), (6418, 7544, 512), (7226, 7000, 1856), (7040, 5296, 2368)]
    for M, N, K in shapes:
        plan = nv.nvfp4_gemm_plan(M, N, K)
        kinds.update(t for t, _ in plan)
        ab = wl.to_bf16_bits(g.standard_normal((M, K)).astype(np.float32))
        wb = wl.to_bf16_bits((g.standard_normal((N, K)) * 0.02).astype(np.float32))
        rows = None if M * N * K < 3e9 else np.unique(np.concatenate([g.integers(0, M, 200), [0, M - 1]]))
        _gemm_case(oracle, ab, wb, f"sweep {M}x{N}x{K} {plan}", rows=rows, check_bf16=False)
    assert kinds >= {"64x64", "128x128", "256x192", "256x256"}, kinds
    assert [len(nv.nvfp4_gemm_plan(*shp)) for shp in shapes[-4:]] == [2, 2, 2, 3]
    assert nv.nvfp4_gemm_plan(7226, 7000, 1856)[0][1] % 256 != 0       # 27 whole tile rows of 28 tiles


@pytest.mark.parametrize("M,N", [(300100, 264), (72, 300104)])
def test_gemm_operand_of_2_gib(oracle, M, N):
    """An operand of more than 2 GiB of codes (K = 14336: about 299 thousand rows per launch) is cut
    into row chunks; rows on both sides of the cut, the first and last rows and seeded ones are
    checked against the oracle.  The NVFP4 operands are drawn on the device (any code and any
    normal scale byte is a valid tensor)."""
    K = 14336
    say(f"[gemm] {M}x{N}x{K}: {nv.nvfp4_gemm_plan(M, N, K)}")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N)

    def draw(rows):
        codes = torch.randint(0, 256, (rows, K // 2), dtype=torch.uint8, device="cuda", generator=gen)
        scales = torch.randint(40, 72, (rows, K // 16), dtype=torch.uint8, device="cuda", generator=gen)
        gs = torch.tensor([2.0 ** -9], dtype=torch.float32, device="cuda")
        return nv.NVFP4Tensor(rows, K, "cuda", codes, scales, gs)

    A, W = draw(M), draw(N)
    assert max(M, N) * (K // 2) > 2 ** 31
    y = nv.nvfp4_gemm(A, W, nv.OUT_F32)
    torch.cuda.synchronize()
    g = np.random.default_rng(M)
    cut = 299264                                   # rows per launch at this K
    big = max(M, N)
    pick = np.unique(np.concatenate([[0, 1, cut - 1, cut, cut + 1, big - 1], g.integers(0, big, 6)]))
    sel = torch.as_tensor(pick, device="cuda")

    def host(t, idx=None):
        c, sc = (t.codes, t.scales) if idx is None else (t.codes[idx], t.scales[idx])
        return oracle.Q(c.cpu().numpy(), sc.cpu().numpy(), np.float32(2.0 ** -9))

    if M > N:
        Y, S = oracle.gemm(host(A, sel), host(W))
        got = y[sel].cpu().numpy()
    else:
        Y, S = oracle.gemm(host(A), host(W, sel))
        got = y[:, sel].cpu().numpy()
    fro, worst = assert_gemm_close(got, Y, S, f"chunked {M}x{N}x{K}")
    say(f"        rel fro {fro:.2e}  worst err/S {worst:.2e}")
    del A, W, y
    torch.cuda.empty_cache()


@pytest.mark.parametrize("M,N,K", [(5, 8, 16), (7, 12, 48), (9, 4, 80)])
def test_gemm_small_k_untiled(oracle, M, N, K):
    g = np.random.default_rng(M * N * K)
    ab = wl.to_bf16_bits(g.standard_normal((M, K)).astype(np.float32))
    wb = wl.to_bf16_bits(g.standard_normal((N, K)).astype(np.float32))
    _gemm_case(oracle, ab, wb, f"64x64 tile alone {M}x{N}x{K}", check_bf16=(N % 4 == 0))


def test_gemm_unit_scales_is_bit_exact(oracle):
    """Block scales 1, tensor scales 1: every partial sum is a small multiple of 1/4, so
    FP32 accumulation in any order is exact and the GPU must match the oracle bit for bit."""
    g = np.random.default_rng(4)
    mags = np.array([0, .5, 1, 1.5, 2, 3, 4, 6])

    def unit(rows, K):
        v = mags[g.integers(0, 8, size=(rows, K))] * g.choice([-1.0, 1.0], size=(rows, K))
        v[:, 0::16] = 6.0
        v[0, 1] = 2688.0
        return wl.to_bf16_bits(v.astype(np.float32))

    ab, wb = unit(192, 256), unit(160, 256)
    oa, ow = oracle.quantize(ab), oracle.quantize(wb)
    assert oa.global_scale == 1 and ow.global_scale == 1
    Y, _ = oracle.gemm(oa, ow)
    ga, gw = nv.nvfp4_quantize(dev_bf16(ab)), nv.nvfp4_quantize(dev_bf16(wb))
    y = nv.nvfp4_gemm(ga, gw, nv.OUT_F32).cpu().numpy().astype(np.float64)
    # [0, 0] holds 2688 * 2688 plus quarters: more than 24 bits, the only inexact element
    y[0, 0] = Y[0, 0] = 0.0
    assert (y == Y).all()


def test_gemm_scale_linearity_and_determinism(oracle):
    cfg = wl.config1()
    ga, gw = nv.nvfp4_quantize(dev_bf16(cfg["A"])), nv.nvfp4_quantize(dev_bf16(cfg["W"]))
    y1 = nv.nvfp4_gemm(ga, gw).clone()
    y2 = nv.nvfp4_gemm(ga, gw)
    assert torch.equal(y1, y2)
    ga.global_scale.mul_(0.5)
    y3 = nv.nvfp4_gemm(ga, gw)
    assert torch.equal(y3, y1 * 0.5)


def test_gemm_backward_operands(oracle):
    """dgrad dX = dY W and wgrad dW = dY^T X with every operand re-quantized along its own K."""
    M, N, K = 272, 320, 192          # X [M,K], W [N,K], dY [M,N]
    g = np.random.default_rng(31)
    xb = wl.activation_with_outliers(M, K, 4, 0)
    wb = wl.normal((N, K), 0.02, 4, 1)
    dyb = wl.normal((M, N), 1e-3, 4, 2)
    x, w, dy = dev_bf16(xb), dev_bf16(wb), dev_bf16(dyb)
    # dgrad: A = dY [M, K'=N] (blocks along N), W' = W^T [K, K'=N] (blocks along W's row axis)
    o_dy, o_wt = oracle.quantize(dyb), oracle.quantize(np.ascontiguousarray(wb.T))
    g_dy, g_wt = nv.nvfp4_quantize(dy), nv.nvfp4_quantize(w, block_axis=1)
    assert_q_equal(g_wt, o_wt, "W^T")
    Y, S = oracle.gemm(o_dy, o_wt)
    assert_gemm_close(nv.nvfp4_gemm(g_dy, g_wt).cpu().numpy(), Y, S, "dgrad")
    # wgrad: A = dY^T [N, K'=M], W' = X^T [K, K'=M]
    o_dyt, o_xt = oracle.quantize(np.ascontiguousarray(dyb.T)), oracle.quantize(np.ascontiguousarray(xb.T))
    g_dyt, g_xt = nv.nvfp4_quantize(dy, block_axis=1), nv.nvfp4_quantize(x, block_axis=1)
    assert_q_equal(g_dyt, o_dyt, "dY^T")
    assert_q_equal(g_xt, o_xt, "X^T")
    Y, S = oracle.gemm(o_dyt, o_xt)
    assert_gemm_close(nv.nvfp4_gemm(g_dyt, g_xt).cpu().numpy(), Y, S, "wgrad")


# ------------------------------------------------------------ four over six

def _assert_search_equal(oracle, xb, what, gs=None):
    say(f"[4over6] {what} {xb.shape}")
    want = oracle.quantize(xb, four_over_six=True, global_scale_in=gs)
    gst = None if gs is None else torch.tensor([gs], dtype=torch.float32, device="cuda")
    got = nv.nvfp4_quantize_4over6(dev_bf16(xb), global_scale_in=gst)
    assert_q_equal(got, want, what)
    return want


def test_quantize_four_over_six(oracle):
    """Scale search (Appendix, Eq. 12-13): bytes identical to the oracle's, on data where the
    choice goes both ways, on ragged shapes, on tie-heavy and degenerate blocks."""
    cfg = wl.config2(seed=3, M=300)
    q = _assert_search_equal(oracle, cfg["A"], "activations with outliers")
    plain = oracle.quantize(cfg["A"])
    changed = (q.scales != plain.scales).mean()
    say(f"        blocks that switch to the 4-target scale: {changed:.3f}")
    assert 0.05 < changed < 0.95
    _assert_search_equal(oracle, wl.normal((257, 272), 0.02, 3, 1), "small weights, ragged")
    _assert_search_equal(oracle, wl.normal((64, 4096), 1e-3, 3, 2), "gradients")
    _assert_search_equal(oracle, wl.normal((1, 16), 1.0, 3, 3), "one block")
    _assert_search_equal(oracle, cfg["A"], "given scale", gs=0.01)
    g = np.random.default_rng(46)
    # blocks where both candidates reconstruct equally well (a lone maximum, exact grids, zeros):
    # the decision falls to the exact comparison, and equality keeps the 6-target scale
    x = np.zeros((64, 256), np.float32)
    x[:, ::16] = (g.integers(1, 200, size=(64, 16)) * 0.25).astype(np.float32)          # one non-zero per block
    x[5] = 0.0
    x[6, :128] = np.tile(np.array([0, .5, 1, 1.5, 2, 3, 4, 6, -6, -4, -3, -2, -1.5, -1, -.5, 0], np.float32), 8)
    x[0, 0] = 2688.0
    _assert_search_equal(oracle, wl.to_bf16_bits(x), "equal-error blocks")
    # values on a coarse grid: many exact ties between the two candidates' errors
    y = (g.integers(-12, 13, size=(128, 512)) * 0.5).astype(np.float32)
    y[0, 0] = 2688.0 / 64
    _assert_search_equal(oracle, wl.to_bf16_bits(y), "coarse grid")
    _assert_search_equal(oracle, wl.to_bf16_bits(np.zeros((16, 64), np.float32)), "all zero")


def test_four_over_six_errors_that_tie_in_exact_arithmetic(oracle):
    """Blocks whose two candidates have EQUAL squared error in exact arithmetic (grid-like values, block scales in the
    ratio 3 : 2) while the tensor scale has a full mantissa: the comparison then hangs on how the fp64 sums round, each
    multiplication, subtraction and addition on its own, and a fused multiply-add anywhere in it changes the answer.
    The first block is one that a randomized comparison against the oracle turned up; the rest are of its kind."""
    bits = [0xbe40, 0x3d80, 0x3e40, 0xbd80, 0x3f10, 0x0, 0xbf00, 0x3f70, 0xbf88, 0x3ec0, 0xbf30, 0xbfe0, 0x3fa8, 0x3f50, 0x3d80, 0x3d80]
    xb = np.zeros((2, 16), np.uint16)
    xb[0] = bits
    xb[1, 0] = 0x409C                                   # 4.875: the tensor scale 4.875 / 2688
    want = _assert_search_equal(oracle, xb, "the block that was found")
    assert want.scales[0, 0] == 0x77                    # the 4-target scale: its fp64 sum comes out one ulp smaller
    _assert_search_equal(oracle, xb, "the same, scale given", gs=float(want.global_scale))
    g = np.random.default_rng(755)
    for amax in (4.875, 7.3125, 2.40625, 13.25):
        x = (g.integers(-30, 31, size=(256, 512)) / 16.0).astype(np.float32)
        x[g.random((256, 512)) < 0.15] = 0.0
        x[0, 0] = amax
        xb = wl.to_bf16_bits(x)
        want = _assert_search_equal(oracle, xb, f"sixteenths, amax {amax}")
        _assert_search_equal(oracle, xb, f"sixteenths, amax {amax}, scale given", gs=float(want.global_scale))


def test_kv_quant_four_over_six(oracle):
    T, H, d = 129, 24, 128
    kb = wl.kv_tensor(T, H, d, 4, 0)
    say(f"[4over6] KV {kb.shape}")
    want = oracle.quantize(kb.reshape(T * H, d), four_over_six=True)
    kv = dev_bf16(kb.reshape(T * H, d)).reshape(T, H, d)
    got = nv.nvfp4_kv_quant_4over6(kv)
    assert_q_equal(got, want, "KV 4over6")
    # and the cache reads back through the ordinary dequantizer, bit for bit
    back = nv.nvfp4_kv_dequant(got, T, H, d)
    assert (nv.bits_from_bf16(back).reshape(T * H, d) == oracle.dequant_bf16(want)).all()
    # the search never loses to the plain rule (squared error per block, fp64)
    x = wl.bf16_bits_to_f32(kb.reshape(T * H, d)).astype(np.float64)
    e46 = ((x - oracle.dequant_f64(want)) ** 2).sum()
    e6 = ((x - oracle.dequant_f64(oracle.quantize(kb.reshape(T * H, d)))) ** 2).sum()
    say(f"        squared error with search / plain: {e46 / e6:.4f}")
    assert e46 <= e6


# ----------------------------------------------------------- LoRA side branch

def _lora_case(oracle, M, N, K, scale, what, rows=None):
    say(f"[lora] {what} {M}x{N}x{K}")
    r = nv.LORA_RANK
    xb = wl.activation_with_outliers(M, K, 28, 0)
    wb = wl.normal((N, K), 0.02, 28, 1)
    ab = wl.normal((r, K), 0.02, 28, 2)
    bb = wl.normal((N, r), 0.05, 28, 3)
    # down projection on the unquantized activations: bf16 result, equal to the fp64 chain's
    # rounding almost everywhere and never more than one bf16 ulp (plus fp32 accumulation) away
    t = nv.nvfp4_lora_down(dev_bf16(xb), dev_bf16(ab))
    torch.cuda.synchronize()
    tb = nv.bits_from_bf16(t)
    want_t = oracle.lora_down(xb, ab)
    tv, wv = wl.bf16_bits_to_f32(tb).astype(np.float64), wl.bf16_bits_to_f32(want_t).astype(np.float64)
    bound = (np.abs(wl.bf16_bits_to_f32(xb)).astype(np.float64) @ np.abs(wl.bf16_bits_to_f32(ab)).astype(np.float64).T)
    assert (np.abs(tv - wv) <= 2.0 ** -7 * np.abs(wv) + 2.0 ** -15 * bound).all()
    assert (tb != want_t).mean() < 0.02
    # fused GEMM: quantized product + scale * T B^T, against the oracle fed the T the GPU produced
    oa, ow = oracle.quantize(xb), oracle.quantize(wb)
    ga, gw = nv.nvfp4_quantize(dev_bf16(xb)), nv.nvfp4_quantize(dev_bf16(wb))
    Y, S = oracle.gemm_lora(oa, ow, tb, bb, scale, rows=rows)
    y32 = nv.nvfp4_gemm_lora(ga, gw, t, dev_bf16(bb), scale, nv.OUT_F32)
    torch.cuda.synchronize()
    got = y32.cpu().numpy()
    fro, worst = assert_gemm_close(got if rows is None else got[rows], Y, S, what)
    say(f"        rel fro {fro:.2e}  worst err/S {worst:.2e}")
    y16 = nv.nvfp4_gemm_lora(ga, gw, t, dev_bf16(bb), scale, nv.OUT_BF16)
    assert (nv.bits_from_bf16(y16) == nv.bits_from_bf16(y32.to(torch.bfloat16))).all()
    # the branch really contributes, and a zero adapter gives the plain GEMM bit for bit
    plain = nv.nvfp4_gemm(ga, gw, nv.OUT_F32)
    assert not torch.equal(plain, y32)
    zero = nv.nvfp4_gemm_lora(ga, gw, t, torch.zeros_like(dev_bf16(bb)), scale, nv.OUT_F32)
    assert torch.equal(zero, plain)


def test_gemm_lora_small_and_ragged(oracle):
    _lora_case(oracle, 100, 136, 192, 1.0, "one ragged tile")
    _lora_case(oracle, 300, 520, 64, 0.5, "several tiles, one k step")
    _lora_case(oracle, 520, 400, 320, 2.0, "several tiles, five k steps")


@pytest.mark.parametrize("M,N,K", [(1, 8, 64), (65, 72, 128), (40, 264, 448), (130, 200, 512),     # the phase on wave 1, 1, 4, 4 of eight
                                   (63, 136, 576), (100, 80, 1024), (70, 64, 2112)])                # wave 1, 0, 1 of four; long K
def test_gemm_lora_on_the_tile_that_cuts_k_between_its_waves(oracle, M, N, K):
    _lora_case(oracle, M, N, K, 0.7, f"lora, K cut between waves {M}x{N}x{K}")


@pytest.mark.parametrize("M,K", [(1, 16), (127, 48), (130, 208), (300, 272), (129, 1040)])     # ranges that end inside a 64-k step
def test_lora_down_partial_steps(oracle, M, K):
    xb, ab = wl.normal((M, K), 1.0, M, K), wl.normal((nv.LORA_RANK, K), 0.02, M, K + 1)
    x = torch.full((M, K + 8), float("nan"), dtype=torch.bfloat16, device="cuda")             # what lies behind a row is not read as part of it
    x[:, :K] = dev_bf16(xb)
    tv = wl.bf16_bits_to_f32(nv.bits_from_bf16(nv.nvfp4_lora_down(x[:, :K], dev_bf16(ab)))).astype(np.float64)
    wv = wl.bf16_bits_to_f32(oracle.lora_down(xb, ab)).astype(np.float64)
    bound = np.abs(wl.bf16_bits_to_f32(xb)).astype(np.float64) @ np.abs(wl.bf16_bits_to_f32(ab)).astype(np.float64).T
    assert (np.abs(tv - wv) <= 2.0 ** -7 * np.abs(wv) + 2.0 ** -15 * bound).all()              # one bf16 step and the fp32 sums


@pytest.mark.parametrize("M,N,K,tiles", [
    (911, 8248, 192, ["256x192"]), (911, 8248, 320, ["256x192"]), (1338, 8104, 64, ["256x256"]), (1338, 8104, 192, ["256x256"]),
    (1100, 2048, 320, ["128x128"]), (2000, 1536, 64, ["128x128"]),
    (4500, 4104, 64, ["256x192", "128x128"]), (3332, 7016, 192, ["256x256", "128x128"]), (5889, 8200, 64, ["256x256", "64x64"]),
    (2321, 6728, 768, ["256x192", "64x64"])])
def test_gemm_lora_on_every_tile_and_leftover_rectangle(oracle, M, N, K, tiles):
    """The launch plan of the plain GEMM, each tile shape with its LoRA phase: single launches of few steps, and leftover
    rectangles of both kinds; ragged both ways."""
    assert [t for t, _ in nv.nvfp4_gemm_plan(M, N, K)] == tiles
    rows = np.unique(np.concatenate([np.random.default_rng(3).integers(0, M, 60), np.arange(256, M, 256), np.arange(255, M, 256), [0, M - 1]])).astype(np.int64)
    _lora_case(oracle, M, N, K, 0.5, f"lora {tiles}", rows=rows)


@pytest.mark.parametrize("M,N,K", [(520, 400, 320), (1000, 3072, 3072), (2000, 1536, 1536), (3520, 1024, 3072), (2321, 6728, 768)])
def test_gemm_lora_with_an_adapter_of_zeros_is_the_plain_gemm(M, N, K):
    """Bit for bit, on values whose fp32 sums depend on their order (heavy tails)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(M)

    def heavy(rows):
        x = torch.randn((rows, K), generator=g, device="cuda")
        return nv.nvfp4_quantize((x * torch.exp(3.0 * torch.randn((rows, K), generator=g, device="cuda"))).to(torch.bfloat16))

    a, w = heavy(M), heavy(N)
    t = torch.randn((M, nv.LORA_RANK), generator=g, device="cuda").to(torch.bfloat16)
    b = torch.zeros((N, nv.LORA_RANK), dtype=torch.bfloat16, device="cuda")
    for dtype in (nv.OUT_F32, nv.OUT_BF16):
        assert torch.equal(nv.nvfp4_gemm_lora(a, w, t, b, 0.5, dtype), nv.nvfp4_gemm(a, w, dtype))


def test_gemm_lora_projection_shape(oracle):
    """The DiT projection with its adapter (rank 128, alpha 128): sampled rows against the oracle."""
    M = wl.TOKENS_INFER
    rows = _sample_rows(M, 64, 5)
    _lora_case(oracle, M, wl.D_MODEL, wl.D_MODEL, 1.0, "projection 3520x3072x3072", rows=rows)


# ------------------------------------------------------- all-to-all send buffers

@pytest.mark.parametrize("T,H,d,P", [(5, 4, 16, 1), (33, 24, 128, 4), (220, 24, 128, 8), (7, 6, 64, 3)])
def test_quantize_for_all_to_all(oracle, T, H, d, P):
    """Appendix "Sequence Parallelism Inference", Eq. 11: NVFP4 along d, rows regrouped into one
    contiguous slab per destination.  The bytes are the oracle's, permuted by plain indexing."""
    say(f"[a2a] {T}x{H}x{d} over {P} peers")
    xb = wl.kv_tensor(T, H, d, 27, T)
    want = oracle.quantize(xb.reshape(T * H, d))
    got = nv.nvfp4_quantize_for_all_to_all(dev_bf16(xb.reshape(T * H, d)).reshape(T, H, d), P)
    codes, scales, gs = host_q(got)
    Hp = H // P
    perm = lambda a: a.reshape(T, P, Hp, -1).transpose(1, 0, 2, 3).reshape(T * H, -1)
    assert gs.view(np.uint32) == np.float32(want.global_scale).view(np.uint32)
    assert (codes == perm(want.codes)).all() and (scales == perm(want.scales)).all()
    # slab p is what device p receives: heads p*Hp.. of every local token, ready for the plain dequantizer
    p = P - 1
    slab = nv.NVFP4Tensor(T * Hp, d, "cuda", got.codes[p * T * Hp:(p + 1) * T * Hp], got.scales[p * T * Hp:(p + 1) * T * Hp], got.global_scale)
    back = nv.bits_from_bf16(nv.nvfp4_kv_dequant(slab, T, Hp, d)).reshape(T, Hp, d)
    ref = oracle.dequant_bf16(want).reshape(T, H, d)[:, p * Hp:(p + 1) * Hp]
    assert (back == ref).all()


@pytest.mark.parametrize("mode", [1, 2])            # one launch, two passes
@pytest.mark.parametrize("T,H,d,P", [(1, 1, 16, 1), (9, 7, 48, 7), (31, 15, 80, 5), (100, 22, 96, 2), (64, 16, 64, 4)])
def test_all_to_all_slabs_of_odd_widths_in_both_forms(oracle, T, H, d, P, mode):
    """Widths and head counts that are no powers of two: the slab order divides by each of them."""
    xb = wl.kv_tensor(T, H, d, 28, T).reshape(T * H, d)
    want = oracle.quantize(xb)
    nv.nvfp4_set_one_launch(mode)
    try:
        codes, scales, _ = host_q(nv.nvfp4_quantize_for_all_to_all(dev_bf16(xb).reshape(T, H, d), P))
    finally:
        nv.nvfp4_set_one_launch()
    perm = lambda a: a.reshape(T, P, H // P, -1).transpose(1, 0, 2, 3).reshape(T * H, -1)
    assert (codes == perm(want.codes)).all() and (scales == perm(want.scales)).all()


# ----------------------------------------------------- random Hadamard transform

@pytest.mark.parametrize("R,C,mask", [(16, 8, 0), (48, 24, 0xFFFF), (128, 256, 0x9A3C), (400, 520, 0x0F5A), (1024, 3072, 0x6D21)])
def test_quantize_rht(oracle, R, C, mask):
    """Weight-gradient operand: Hadamard transform along the contraction axis, then the transposed
    quantizer (Sec. 2.2).  Bytes identical to the oracle's transform followed by its quantizer."""
    say(f"[rht] {R}x{C} mask {mask:#06x}")
    xb = wl.activation_with_outliers(R, C, 25, R) if C >= 256 else wl.normal((R, C), 1.0, 25, R)
    want = oracle.quantize(oracle.rht_rows(xb, mask), block_axis=1)
    got = nv.nvfp4_quantize_rht(dev_bf16(xb), mask)
    assert_q_equal(got, want, "rht")
    # a workspace that holds the partial maxima only: the encoding pass tests every group again instead of being told
    small = torch.empty(nv.nvfp4_workspace_bytes(nv.OP_QUANTIZE, R, C), dtype=torch.uint8, device="cuda")
    assert small.numel() < nv.nvfp4_workspace_bytes(nv.OP_QUANTIZE_RHT, R, C)
    assert_q_equal(nv.nvfp4_quantize_rht(dev_bf16(xb), mask, workspace=small), want, "rht, small workspace")
    gs = torch.tensor([0.0125], dtype=torch.float32, device="cuda")
    got = nv.nvfp4_quantize_rht(dev_bf16(xb), mask, global_scale_in=gs)
    assert_q_equal(got, oracle.quantize(oracle.rht_rows(xb, mask), block_axis=1, global_scale_in=0.0125), "rht, given scale")


def test_quantize_rht_groups_of_every_exponent_spread(oracle):
    """The transform runs in fp32 where that is exact (a group's non-zero magnitudes within 12 binades, away from
    the ends of the exponent range), as two fp32 halves up to 25 binades, and in fp64 elsewhere; the groups that need
    the slower forms are listed per workgroup and worked off in rounds.  Groups on both sides of every condition: spreads of
    0..40 binades, all-zero groups, groups of zeros and one value, signed zeros, magnitudes near 2^-120 and 2^120
    (alone: the tensor scale is shared), exact cancellations (equal values with alternating signs)."""
    g = np.random.default_rng(77)
    R, C = 256, 272                    # a full tile of columns and a ragged one; most groups of a tile need the slower forms
    x = g.standard_normal((R, C)).astype(np.float64)
    spread = g.integers(0, 41, size=(R // 16, 1, C))                    # per group of 16 rows and column
    expo = -(g.random((R // 16, 16, C)) * (spread + 1)).astype(np.int64)
    x = (x.reshape(R // 16, 16, C) * 2.0 ** expo).reshape(R, C)
    x[0:16, 0:8] = 0.0
    x[16:32, 0:8] = 0.0
    x[20, 3] = 1.5
    x[32:48, 0:8] = -0.0
    x[48:64, 0:8] = 0.75 * (1 - 2 * (np.arange(16) % 2))[:, None]       # cancels in most outputs
    x[64:80, 0:8] = 3.0
    for scale, tag in ((1.0, "unit"), (2.0 ** -118, "tiny"), (2.0 ** 112, "huge")):
        xb = wl.to_bf16_bits((x * scale).astype(np.float32))
        for mask in (0x0000, 0xA53C):
            say(f"[rht] spreads, {tag} magnitudes, mask {mask:#06x}")
            want = oracle.quantize(oracle.rht_rows(xb, mask), block_axis=1)
            assert_q_equal(nv.nvfp4_quantize_rht(dev_bf16(xb), mask), want, f"rht spreads {tag} {mask:#x}")
            small = torch.empty(nv.nvfp4_workspace_bytes(nv.OP_QUANTIZE, R, C), dtype=torch.uint8, device="cuda")
            assert_q_equal(nv.nvfp4_quantize_rht(dev_bf16(xb), mask, workspace=small), want, f"rht spreads {tag} {mask:#x}, small workspace")


def test_quantize_rht_random_sweep(oracle):
    """Seeded sweep over shapes (ragged tile edges in both directions), sign masks and value distributions for the
    Hadamard quantizer: Gaussian, a few huge rows, sparse with whole groups of zeros, grid values whose sums cancel
    and land on bf16 ties, magnitudes that differ by many binades inside a group."""
    g = np.random.default_rng(4242)
    for case in range(16):
        R, C = 16 * int(g.integers(1, 40)), 8 * int(g.integers(1, 90))
        mask = int(g.integers(0, 1 << 16))
        kind = case % 4
        x = g.standard_normal((R, C))
        if kind == 1:
            x[g.choice(R, max(1, R // 50), replace=False)] *= 300.0
        elif kind == 2:
            x = np.where(g.random((R, C)) < 0.7, 0.0, x)
            x[: 16 * (R // 32)] = 0.0
        elif kind == 3:
            x = g.integers(-6, 7, size=(R, C)) * 2.0 ** g.integers(-20, 4, size=(R, C))
        xb = wl.to_bf16_bits(np.asarray(x, np.float32))
        say(f"[rht] sweep {case}: {R}x{C} mask {mask:#06x} kind={kind}")
        want = oracle.quantize(oracle.rht_rows(xb, mask), block_axis=1)
        assert_q_equal(nv.nvfp4_quantize_rht(dev_bf16(xb), mask), want, f"rht sweep {case}")


def test_wgrad_with_rht(oracle):
    """dW = dY^T X with both operands transformed by the same signs: the GEMM equals the oracle's on
    the oracle's transformed operands; both quantized products approximate the unquantized one (the
    transform is orthogonal), their errors are reported."""
    M, N, K = 512, 144, 272
    g = np.random.default_rng(26)
    x = g.standard_normal((M, K)).astype(np.float32)
    x[g.choice(M, 5, replace=False)] *= 40.0                      # a few outlier tokens
    xb = wl.to_bf16_bits(x)
    dyb = wl.normal((M, N), 1e-3, 26, 1)
    mask = 0xB7C5
    o_dy = oracle.quantize(oracle.rht_rows(dyb, mask), block_axis=1)
    o_x = oracle.quantize(oracle.rht_rows(xb, mask), block_axis=1)
    g_dy, g_x = nv.nvfp4_quantize_rht(dev_bf16(dyb), mask), nv.nvfp4_quantize_rht(dev_bf16(xb), mask)
    assert_q_equal(g_dy, o_dy, "dY")
    assert_q_equal(g_x, o_x, "X")
    Y, S = oracle.gemm(o_dy, o_x)
    got = nv.nvfp4_gemm(g_dy, g_x).cpu().numpy()
    assert_gemm_close(got, Y, S, "wgrad with RHT")
    exact = wl.bf16_bits_to_f32(dyb).astype(np.float64).T @ wl.bf16_bits_to_f32(xb).astype(np.float64)
    plain, _ = oracle.gemm(oracle.quantize(dyb, block_axis=1), oracle.quantize(xb, block_axis=1), want_abs=False)
    e_rht, e_plain = np.linalg.norm(Y - exact), np.linalg.norm(plain - exact)
    say(f"        wgrad error vs unquantized product: with RHT {e_rht:.3e}, without {e_plain:.3e}")
    assert e_rht < 0.2 * np.linalg.norm(exact) and e_plain < 0.2 * np.linalg.norm(exact)


# ------------------------------------------------- 2-D block scaling (weights)

@pytest.mark.parametrize("R,C", [(16, 16), (48, 272), (256, 256), (1040, 528), (3072, 1024)])
def test_quantize_2d_weights(oracle, R, C):
    """One scale per 16x16 tile (Sec. 2.2 training recipe): both operands byte-identical to the oracle's."""
    say(f"[2d] {R}x{C}")
    wb = wl.normal((R, C), 0.02, 23, R + C)
    want, want_t = oracle.quantize_2d(wb)
    got, got_t = nv.nvfp4_quantize_2d(dev_bf16(wb))
    assert_q_equal(got, want, "W")
    assert_q_equal(got_t, want_t, "W^T")
    only, none = nv.nvfp4_quantize_2d(dev_bf16(wb), transposed=False)
    assert none is None
    assert_q_equal(only, want, "W without the transposed operand")


def test_quantize_2d_serves_fprop_and_dgrad(oracle):
    """The reason for 2-D scaling: dgrad multiplies by exactly the weights fprop used.  fprop
    Y = X W^T uses W [N, K]; dgrad dX = dY W uses W^T [K, N]: both from one quantization."""
    M, N, K = 160, 272, 192
    xb = wl.activation_with_outliers(M, K, 24, 0)
    wb = wl.normal((N, K), 0.02, 24, 1)
    dyb = wl.normal((M, N), 1e-3, 24, 2)
    ow, owt = oracle.quantize_2d(wb)
    gw, gwt = nv.nvfp4_quantize_2d(dev_bf16(wb))
    assert_q_equal(gw, ow, "W")
    assert_q_equal(gwt, owt, "W^T")
    ox, ody = oracle.quantize(xb), oracle.quantize(dyb)
    gx, gdy = nv.nvfp4_quantize(dev_bf16(xb)), nv.nvfp4_quantize(dev_bf16(dyb))
    Y, S = oracle.gemm(ox, ow)
    assert_gemm_close(nv.nvfp4_gemm(gx, gw).cpu().numpy(), Y, S, "fprop on 2-D weights")
    Y, S = oracle.gemm(ody, owt)
    assert_gemm_close(nv.nvfp4_gemm(gdy, gwt).cpu().numpy(), Y, S, "dgrad on the same weights")
    # given scale, strided input
    big = torch.zeros((N, K + 64), dtype=torch.bfloat16, device="cuda")
    big[:, :K] = dev_bf16(wb)
    gs = torch.tensor([0.003], dtype=torch.float32, device="cuda")
    a, at = nv.nvfp4_quantize_2d(big[:, :K], global_scale_in=gs)
    b, bt = oracle.quantize_2d(wb, global_scale_in=0.003)
    assert_q_equal(a, b, "strided, given scale")
    assert_q_equal(at, bt, "strided, given scale, transposed")


# ------------------------------------------- smoothed keys, gathered reconstruction

def _oracle_k_path(oracle, kb2d):
    mean, xbar = oracle.kv_smooth(kb2d)
    return mean, oracle.quantize(xbar, four_over_six=True)


@pytest.mark.parametrize("T,H,d", [(1, 1, 16), (37, 24, 128), (130, 3, 64), (9, 5, 256), (3, 2, 1024)])
def test_kv_quant_k_smoothing(oracle, T, H, d):
    """Keys as the paper caches them (Sec. 3.2, Eq. 6 + scale search): means, codes, scales and
    tensor scale identical to the oracle's; reconstruction with the means identical too."""
    say(f"[kv-k] {T}x{H}x{d}")
    g = np.random.default_rng(T + d)
    x = wl.bf16_bits_to_f32(wl.kv_tensor(T, H, d, 8, 0)).reshape(T * H, d)
    x = x + g.uniform(-6, 6, size=(T * H, 1)).astype(np.float32)        # a per-row offset for the smoothing to remove
    kb = wl.to_bf16_bits(x)
    want_mean, want_q = _oracle_k_path(oracle, kb)
    got_q, got_mean = nv.nvfp4_kv_quant_k(dev_bf16(kb).reshape(T, H, d))
    torch.cuda.synchronize()
    assert (nv.bits_from_bf16(got_mean) == want_mean).all()
    assert_q_equal(got_q, want_q, "smoothed keys")
    back = nv.nvfp4_kv_dequant_gather([(got_q, got_mean, T)], H, d)
    assert (nv.bits_from_bf16(back).reshape(T * H, d) == oracle.dequant_bf16(want_q, want_mean)).all()


@pytest.mark.parametrize("d", [16, 32, 64, 128, 256, 512, 1024])
def test_kv_quant_k_row_means_on_and_beside_bf16_midpoints(oracle, d):
    """Rows whose exact mean is a midpoint between two bf16 numbers, or lies off it by t / d for t from far below what
    an fp32 sum resolves (2^-40 of the mean) to far above, either way: the means are the exact ones rounded once, in both
    forms of the call.  a, b: neighbouring bf16 numbers; a row is {2a, 2b, t, 0} and pairs {a, b}, in any order."""
    g = np.random.default_rng(d)
    rows = []
    for k in range(-44, -4):
        for sign in (-1.0, 0.0, 1.0):
            lead, scale = float(g.integers(128, 255)), 2.0 ** float(g.integers(-20, 20)) * float(g.choice([-1.0, 1.0]))
            t = sign * float(g.integers(128, 256)) * 2.0 ** k
            x = np.array([2 * lead, 2 * lead + 2, t, 0.0] + [lead, lead + 1] * ((d - 4) // 2))
            rows.append(g.permutation(x * scale))
    x = np.array(rows)
    kb = wl.to_bf16_bits(x.astype(np.float32))
    assert (wl.bf16_bits_to_f32(kb).astype(np.float64) == x).all()                 # every value is a bf16 number
    want_mean, want = _oracle_k_path(oracle, kb)
    kv = dev_bf16(kb).reshape(len(rows), 1, d)
    for mode in (nv.ONE_LAUNCH_ALWAYS, nv.ONE_LAUNCH_NEVER):
        nv.nvfp4_set_one_launch(mode)
        try:
            gq, gm = nv.nvfp4_kv_quant_k(kv)
        finally:
            nv.nvfp4_set_one_launch()
        assert (nv.bits_from_bf16(gm) == want_mean).all(), f"means, mode {mode}"
        assert_q_equal(gq, want, f"mode {mode}")


def test_kv_cache_random_sweep(oracle):
    """Seeded sweep over cache shapes and value distributions: plain values, the scale search, the
    smoothed keys and their reconstruction, all byte for byte against the oracle."""
    g = np.random.default_rng(777)
    for case in range(24):
        d = 16 * 2 ** int(g.integers(0, 7))                  # 16 .. 1024 (the smoothed path needs d / 16 a power of two)
        T, H = int(g.integers(1, 60)), int(g.integers(1, 9))
        kind = case % 4
        x = g.standard_normal((T * H, d))
        if kind == 0:
            x = x * g.uniform(0.5, 4, size=(T * H, 1)) + g.uniform(-8, 8, size=(T * H, 1))
        elif kind == 1:                                       # offsets that dwarf the signal
            x = x * 2.0 ** -6 + g.choice([-96.0, 0.75, 40.0], size=(T * H, 1))
        elif kind == 2:                                       # grid values: ties in the mean and in the codes
            x = g.integers(-24, 25, size=(T * H, d)) * 0.25
        else:                                                 # sparse rows, some all zero
            x = np.where(g.random((T * H, d)) < 0.8, 0.0, x)
            x[:: 5] = 0.0
        kb = wl.to_bf16_bits(np.asarray(x, np.float32))
        say(f"[kv] sweep {case}: {T}x{H}x{d} kind={kind}")
        kv = dev_bf16(kb).reshape(T, H, d)
        assert_q_equal(nv.nvfp4_kv_quant(kv), oracle.quantize(kb), f"kv sweep {case} plain")
        assert_q_equal(nv.nvfp4_kv_quant_4over6(kv), oracle.quantize(kb, four_over_six=True), f"kv sweep {case} search")
        want_mean, want_q = _oracle_k_path(oracle, kb)
        got_q, got_mean = nv.nvfp4_kv_quant_k(kv)
        assert (nv.bits_from_bf16(got_mean) == want_mean).all(), f"kv sweep {case} means"
        assert_q_equal(got_q, want_q, f"kv sweep {case} smoothed")
        back = nv.nvfp4_kv_dequant_gather([(got_q, got_mean, T)], H, d)
        assert (nv.bits_from_bf16(back).reshape(T * H, d) == oracle.dequant_bf16(want_q, want_mean)).all()


def test_kv_quant_k_degenerate_rows(oracle):
    T, H, d = 8, 4, 128
    x = np.zeros((T * H, d), np.float32)
    x[1] = 3.25                                    # constant row: nothing left after smoothing
    x[2, ::2], x[2, 1::2] = 1.0, -1.0              # zero mean
    x[3, 0] = 1000.0                               # one outlier drags the mean
    x[4] = np.linspace(-4, 4, d, dtype=np.float32)
    kb = wl.to_bf16_bits(x)
    want_mean, want_q = _oracle_k_path(oracle, kb)
    got_q, got_mean = nv.nvfp4_kv_quant_k(dev_bf16(kb).reshape(T, H, d))
    assert (nv.bits_from_bf16(got_mean) == want_mean).all()
    assert_q_equal(got_q, want_q, "degenerate rows")
    # all-zero cache: scale 1, zero codes, zero means
    z = wl.to_bf16_bits(np.zeros((T * H, d), np.float32))
    zq, zm = nv.nvfp4_kv_quant_k(dev_bf16(z).reshape(T, H, d))
    assert_q_equal(zq, oracle.quantize(z, four_over_six=True), "zero cache")
    assert (nv.bits_from_bf16(zm) == 0).all()


def test_kv_quant_k_wide_exponent_range(oracle):
    """Elements up to 2^36 apart in one row: the difference to the row mean is far from exact in
    fp32 for many of them, the rounded result must still be the single rounding of the exact one."""
    T, H, d = 16, 8, 128
    g = np.random.default_rng(77)
    e = g.integers(-18, 19, size=(T * H, d))
    x = (np.ldexp(1.0 + g.integers(0, 128, size=e.shape) / 128.0, e) * g.choice([-1.0, 1.0], size=e.shape)).astype(np.float32)
    x[::3] = np.abs(x[::3])                         # rows with a mean of the size of their largest element
    kb = wl.to_bf16_bits(x)
    want_mean, want_q = _oracle_k_path(oracle, kb)
    say(f"[kv-k] wide exponent range {T}x{H}x{d}")
    got_q, got_mean = nv.nvfp4_kv_quant_k(dev_bf16(kb).reshape(T, H, d))
    assert (nv.bits_from_bf16(got_mean) == want_mean).all()
    assert_q_equal(got_q, want_q, "wide exponent range")


def test_kv_dequant_gather_window(oracle):
    """A sink chunk plus a sliding window of chunks of different lengths, keys smoothed and values
    plain, reconstructed by one launch each: every byte equals the per-chunk oracle output."""
    H, d = 24, 128
    lens = [880, 1, 37, 880, 300, 19, 23]
    k_chunks, v_chunks, want_k, want_v = [], [], [], []
    for i, T in enumerate(lens):
        kb = wl.kv_tensor(T, H, d, 9, 2 * i).reshape(T * H, d)
        vb = wl.kv_tensor(T, H, d, 9, 2 * i + 1).reshape(T * H, d)
        if i == 2:
            kb = wl.to_bf16_bits(wl.bf16_bits_to_f32(kb) * 50.0)       # chunks differ in scale
        if i == 5:                                                     # a chunk far below and one far above the range in which
            kb = wl.to_bf16_bits(wl.bf16_bits_to_f32(kb) * np.float32(2.0 ** -100))   # the mean is added back in fp32
        if i == 6:
            kb = wl.to_bf16_bits(wl.bf16_bits_to_f32(kb) * np.float32(2.0 ** 90))
            kb[5 * H:7 * H] = 0                                        # rows of zeros: mean zero, scale bytes zero
        m, q = _oracle_k_path(oracle, kb)
        want_k.append(oracle.dequant_bf16(q, m))
        want_v.append(oracle.dequant_bf16(oracle.quantize(vb)))
        gq, gm = nv.nvfp4_kv_quant_k(dev_bf16(kb).reshape(T, H, d))
        k_chunks.append((gq, gm, T))
        v_chunks.append((nv.nvfp4_kv_quant(dev_bf16(vb).reshape(T, H, d)), None, T))
    say(f"[kv-gather] {len(lens)} chunks, {sum(lens)} tokens")
    kk = nv.bits_from_bf16(nv.nvfp4_kv_dequant_gather(k_chunks, H, d)).reshape(-1, d)
    vv = nv.bits_from_bf16(nv.nvfp4_kv_dequant_gather(v_chunks, H, d)).reshape(-1, d)
    assert (kk == np.concatenate(want_k)).all()
    assert (vv == np.concatenate(want_v)).all()
    # mixed list (smoothed and plain chunks in one call), and the single-chunk call equals nvfp4_kv_dequant
    mixed = nv.bits_from_bf16(nv.nvfp4_kv_dequant_gather([k_chunks[0], v_chunks[1], k_chunks[4]], H, d)).reshape(-1, d)
    assert (mixed == np.concatenate([want_k[0], want_v[1], want_k[4]])).all()
    one = nv.nvfp4_kv_dequant_gather([v_chunks[3]], H, d)
    assert (nv.bits_from_bf16(one) == nv.bits_from_bf16(nv.nvfp4_kv_dequant(v_chunks[3][0], lens[3], H, d))).all()


# --------------------------------------------------- fused activation + quantize

def _gelu64(y):
    """tanh-form GELU in fp64 (numpy), only to judge the kernel's fp32 evaluation on its own inputs.
    0.5 (1 + tanh u) is written as e / (e + 1), e = exp(2u): the same function, but accurate for very negative
    y, where 1 + tanh(u) in floating point keeps only a digit or two (at y = -7 the textbook form is off by
    5 % in fp64; the results there are ~1e-15 and no tolerance of the parity tests sees them)."""
    e = np.exp(np.minimum(2.0 * np.sqrt(2.0 / np.pi) * (y + 0.044715 * y ** 3), 80.0))
    return y * e / (e + 1.0)


def _act_quant_case(oracle, M, N, K, given_scale, what, max_flips=0.001):
    say(f"[act-quant] {what} {M}x{N}x{K} given_scale={given_scale}")
    g = np.random.default_rng(M + N)
    ab = wl.activation_with_outliers(M, K, 2, 0)
    wb = wl.normal((N, K), 0.02, 2, 1)
    ga, gw = nv.nvfp4_quantize(dev_bf16(ab)), nv.nvfp4_quantize(dev_bf16(wb))
    oa, ow = oracle.quantize(ab), oracle.quantize(wb)
    h = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    gs = torch.tensor([0.004], dtype=torch.float32, device="cuda") if given_scale else None
    out = nv.nvfp4_gemm_act_quant(ga, gw, nv.ACT_GELU_TANH, global_scale_in=gs, h_bf16=h)
    torch.cuda.synchronize()
    hb = nv.bits_from_bf16(h)
    # (1) the packed output is exactly the quantizer applied to the H this GEMM produced
    oq = oracle.quantize(hb, global_scale_in=0.004 if given_scale else None)
    assert_q_equal(out, oq, what + " fused vs quantize(H)")
    # (2) H itself is the activation of the GEMM, within bf16 rounding of the fp64 chain
    Y, S = oracle.gemm(oa, ow)
    want = wl.bf16_bits_to_f32(oracle.gelu_tanh_bf16(Y)).astype(np.float64)
    got = wl.bf16_bits_to_f32(hb).astype(np.float64)
    tol = 2.0 ** -7 * np.abs(want) + 2.0 ** -15 * S + 1e-30      # one bf16 ulp + GEMM bound
    assert (np.abs(got - want) <= tol).all()
    flips = (got != want).mean()
    assert flips < max_flips                                      # and it is the same bf16 almost everywhere
    # (2b) the activation itself, on the accumulators this kernel produced (the plain GEMM call runs the same
    # launch plan): H is the bf16 nearest to gelu(y) up to the few fp32 ulps of the kernel's evaluation, for
    # negative y as well (relative, where a form that subtracts two nearly equal numbers would lose all digits)
    y32 = nv.nvfp4_gemm(ga, gw, nv.OUT_F32).cpu().numpy().astype(np.float64)
    g64 = _gelu64(y32)
    # half a bf16 ulp plus the fp32 evaluation error: the exponent 2u log2(e) reaches ~75 in magnitude at
    # y = -8, so its fp32 rounding alone moves exp(2u) by up to ~2e-5 relative; 2^-14 covers it
    near = np.abs(got - g64) <= (2.0 ** -8 + 2.0 ** -14) * np.abs(g64) + 1e-30
    deep = y32 < -8.0            # results below ~1e-13: the hardware exponential flushes towards zero there
    assert (near | deep).all(), f"{what}: activation off by more than half a bf16 ulp at y = {y32[~(near | deep)][:4]}"
    assert (np.abs(got[deep]) <= 1e-12).all()
    act_flips = (got != wl.bf16_bits_to_f32(oracle.gelu_tanh_bf16(y32)).astype(np.float64))[y32 > -5.0].mean()
    say(f"        bf16 H differs from the fp64 chain on {flips:.2%} of the outputs, from bf16(gelu(own y)) on {act_flips:.3%}")
    assert act_flips < 1e-4
    # (3) without the optional H buffer the bytes are the same
    out2 = nv.nvfp4_gemm_act_quant(ga, gw, nv.ACT_GELU_TANH, global_scale_in=gs)
    a, b = host_q(out), host_q(out2)
    assert (a[0] == b[0]).all() and (a[1] == b[1]).all() and a[2] == b[2]


@pytest.mark.parametrize("given_scale", [False, True])
def test_gemm_act_quant(oracle, given_scale):
    for M, N, K, tile in ((200, 272, 256, "64x64"), (520, 1040, 128, "64x64"), (1100, 2048, 192, "128x128"), (2100, 2064, 256, "128x128"),
                          (1500, 6000, 192, "256x192"), (4200, 3072, 128, "256x256"), (40, 48, 48, "generic")):
        assert [t for t, _ in nv.nvfp4_gemm_plan(M, N, K)] == [tile]
        _act_quant_case(oracle, M, N, K, given_scale, f"{tile} tiles")
    # whole waves of 256x256 tiles, then the tail of a tile row on 64x64 tiles and the rows below on
    # 128x128 tiles: three launches share the output pitch and the table of partial maxima
    assert len(nv.nvfp4_gemm_plan(7040, 5296, 2368)) == 3
    # (the fp32 accumulation error grows with K against the fixed bf16 ulp, so more results land on the
    # other side of a rounding boundary than at K = 256: 0.15 % here)
    _act_quant_case(oracle, 7040, 5296, 2368, given_scale, "three launches", max_flips=0.005)


@pytest.mark.parametrize("M,N,K", [(520, 1040, 128), (1100, 2048, 192), (4200, 3072, 128), (300, 272, 80)])
def test_gemm_scale_out_feeds_the_given_scale_quantizers(oracle, M, N, K):
    """nvfp4_gemm_scale_out: bf16 Y bit for bit what nvfp4_gemm gives, and the tensor scale of Y from the GEMM's
    epilogue equal to the oracle's amax / 2688 of those bits.  The calls that quantize Y afterwards take the scale as
    given (one read of Y each) and return the oracle's bytes along both axes and with the scale search.  Tiled
    shapes of every size, and an odd shape that only the 64x64 tile takes."""
    say(f"[gemm+scale] {M}x{N}x{K}: {nv.nvfp4_gemm_plan(M, N, K)}")
    g = np.random.default_rng(M + N + K)
    ga = nv.nvfp4_quantize(dev_bf16(wl.to_bf16_bits(g.standard_normal((M, K)).astype(np.float32))))
    gw = nv.nvfp4_quantize(dev_bf16(wl.to_bf16_bits((g.standard_normal((N, K)) * 0.02).astype(np.float32))))
    y_ref = nv.nvfp4_gemm(ga, gw, nv.OUT_BF16)
    y = _nan_filled(M, N, torch.bfloat16)
    scale = torch.full((1,), float("nan"), dtype=torch.float32, device="cuda")
    nv.nvfp4_gemm_scale_out(ga, gw, Y=y, scale_out=scale)
    torch.cuda.synchronize()
    yb = nv.bits_from_bf16(y)
    assert (yb == nv.bits_from_bf16(y_ref)).all(), "Y differs from nvfp4_gemm's"
    want_gs = oracle.global_scale(yb)
    assert np.float32(scale.item()).view(np.uint32) == np.float32(want_gs).view(np.uint32), "tensor scale of Y"
    assert_q_equal(nv.nvfp4_quantize(y, global_scale_in=scale), oracle.quantize(yb), "rows, given scale")
    assert_q_equal(nv.nvfp4_quantize_4over6(y, global_scale_in=scale), oracle.quantize(yb, four_over_six=True), "search")
    if True:
        Mt = M - M % 16                                   # blocks along the rows need whole groups of 16 rows
        assert_q_equal(nv.nvfp4_quantize(y[:Mt], block_axis=1, global_scale_in=scale),
                       oracle.quantize(yb[:Mt], block_axis=1, global_scale_in=float(want_gs)), "columns, given scale")


@pytest.mark.parametrize("M,N,K", [(33, 4, 128), (100, 12, 64), (70, 3076, 96), (65, 67, 80), (1, 1, 16)])
def test_gemm_scale_out_sees_the_columns_behind_the_last_whole_vector(oracle, M, N, K):
    """Widths that are no multiple of 8 in a padded Y, the largest value in the last column: Y and its scale as always,
    the padding left alone."""
    g = np.random.default_rng(M + N + K)
    w = g.standard_normal((N, K)) * 0.02
    w[-1] *= 50.0
    ga = nv.nvfp4_quantize(dev_bf16(wl.to_bf16_bits(g.standard_normal((M, K)).astype(np.float32))))
    gw = nv.nvfp4_quantize(dev_bf16(wl.to_bf16_bits(w.astype(np.float32))))
    y = torch.full((M, (N + 7) // 8 * 8 + 8), -7.0, dtype=torch.bfloat16, device="cuda")
    _, scale = nv.nvfp4_gemm_scale_out(ga, gw, Y=y[:, :N])
    ref = torch.full_like(y, -7.0)
    nv.nvfp4_gemm(ga, gw, nv.OUT_BF16, Y=ref[:, :N])
    yb = nv.bits_from_bf16(y)
    assert (yb == nv.bits_from_bf16(ref)).all() and bool((y[:, N:] == -7.0).all())
    assert int(y[:, :N].float().abs().max(0).values.argmax()) == N - 1
    want = oracle.global_scale(np.ascontiguousarray(yb[:, :N]))
    assert np.float32(scale.item()).view(np.uint32) == np.float32(want).view(np.uint32)


# -------------------------------------------------------- full benchmark sizes

def test_full_size_projection_config2(oracle):
    """A[3520,3072], W[3072,3072]: codes and scales in full and the WHOLE output matrix against the
    oracle, in the launch configuration bench.py times."""
    cfg = wl.config2()
    _gemm_case(oracle, cfg["A"], cfg["W"], "config2")


@pytest.mark.parametrize("M,N,K,tile", [(4100, 8200, 128, "256x192"),      # ragged M and N tails
                                        (8200, 8192, 192, "256x256"),      # odd number of 64-k steps
                                        (3520, 3072, 320, "256x192"),      # the projection shape, 5 steps
                                        (911, 8248, 64, "256x192"),        # single step
                                        (700, 1544, 64, "128x128")])
def test_gemm_large_tile_paths(oracle, M, N, K, tile):
    """Shapes that take the larger tiles."""
    assert nv.nvfp4_gemm_plan(M, N, K)[0][0] == tile
    g = np.random.default_rng(M + K)
    ab = wl.activation_with_outliers(M, K, 7, 0)
    wb = wl.normal((N, K), 0.02, 7, 1)
    edge = [0, 127, 128, 255, 256, M - 257, M - 256, M - 1]
    rows = np.unique(np.concatenate([edge, g.integers(0, M, 20)])).astype(np.int64)
    _gemm_case(oracle, ab, wb, f"large tile {M}x{N}x{K}", rows=rows)


@pytest.mark.parametrize("K", [128, 256, 384, 448, 640])
def test_gemm_several_tiles_per_workgroup(oracle, K):
    """More 256-row tiles than compute units, several rounds of workgroups; the K values give every
    combination of even / odd counts of 64-k steps, 128-k copy steps and 256-k scale groups.
    One sampled row in every band of 256 rows, plus the band edges."""
    M, N = 4400, 8192
    g = np.random.default_rng(K)
    ab = wl.activation_with_outliers(M, K, 11, 0)
    wb = wl.normal((N, K), 0.02, 11, 1)
    bands = np.arange(0, M, 256)
    rows = np.unique(np.concatenate([bands, np.minimum(bands + g.integers(1, 256, bands.size), M - 1),
                                     [255, 256, M - 1]])).astype(np.int64)
    _gemm_case(oracle, ab, wb, f"several tiles per workgroup {M}x{N}x{K}", rows=rows)


def test_gemm_subnormal_and_extreme_block_scales(oracle):
    """Raw operands with every E4M3 scale byte 0x00..0x7E (subnormal scales included)."""
    g = np.random.default_rng(99)
    M, N, K = 512, 768, 256
    def raw(rows):
        codes = g.integers(0, 256, size=(rows, K // 2)).astype(np.uint8)
        scales = g.integers(0, 127, size=(rows, K // 16)).astype(np.uint8)
        scales[:, ::3] = g.integers(0, 9, size=scales[:, ::3].shape)       # many subnormal / zero scales
        return codes, scales
    ca, sa = raw(M)
    cw, sw = raw(N)
    gsa, gsw = np.float32(2.0 ** -8), np.float32(1.5 * 2.0 ** -9)
    Y, S = oracle.gemm(oracle.Q(ca, sa, gsa), oracle.Q(cw, sw, gsw))
    y = nv.nvfp4_gemm(nv.NVFP4Tensor.from_host(ca, sa, gsa), nv.NVFP4Tensor.from_host(cw, sw, gsw)).cpu().numpy()
    assert_gemm_close(y, Y, S, "raw scales")


# The remaining benchmark configurations at full size, in the launch configurations bench.py
# times: codes / scales / KV bytes in full, GEMM outputs on sampled rows the oracle computes.

def _sample_rows(M, n=512, seed=0, band=256):
    """Rows of a full-size output that the oracle computes: the first and the last row of EVERY band of
    `band` rows (the tallest tile of any launch plan, so every row of tiles of every launch is compared),
    the rows around the first and last band edges, and n seeded rows."""
    first = np.arange(0, M, band)
    last = np.minimum(first + band - 1, M - 1)
    edge = [0, 127, 128, 255, 256, M - 257, M - 256, M - 1]
    picks = np.concatenate([first, last, edge, np.random.default_rng(seed).integers(0, M, n)])
    return np.unique(picks[(picks >= 0) & (picks < M)]).astype(np.int64)


def test_ffn_step_replays_from_a_hip_graph():
    """The entry points allocate nothing, synchronise nothing and clear no memory with memset
    nodes, so a caller may capture them: one FFN step (quantize, up projection with GELU and
    re-quantization, down projection) captured once and replayed several times, with eager
    work and synchronisations in between, gives the eager result bit for bit every time."""
    M, D, F = 520, 1024, 2048
    g = np.random.default_rng(11)
    A = dev_bf16(wl.to_bf16_bits(g.standard_normal((M, D)).astype(np.float32)))
    W1 = nv.nvfp4_quantize(dev_bf16(wl.to_bf16_bits((g.standard_normal((F, D)) * 0.02).astype(np.float32))))
    W2 = nv.nvfp4_quantize(dev_bf16(wl.to_bf16_bits((g.standard_normal((D, F)) * 0.02).astype(np.float32))))
    qA, qH = nv.NVFP4Tensor(M, D, "cuda"), nv.NVFP4Tensor(M, F, "cuda")
    Y = torch.empty((M, D), dtype=torch.bfloat16, device="cuda")
    ws_q = torch.empty(nv.nvfp4_workspace_bytes(nv.OP_QUANTIZE, M, D), dtype=torch.uint8, device="cuda")
    ws_g = torch.empty(nv.nvfp4_workspace_bytes(nv.OP_GEMM_ACT_QUANT, M, F, 0), dtype=torch.uint8, device="cuda")

    def step():
        nv.nvfp4_quantize(A, out=qA, workspace=ws_q)
        nv.nvfp4_gemm_act_quant(qA, W1, nv.ACT_GELU_TANH, out=qH, workspace=ws_g)
        nv.nvfp4_gemm(qH, W2, nv.OUT_BF16, Y=Y)

    step()                                          # eager: also the first use of every kernel variant
    torch.cuda.synchronize()
    want, want_codes = Y.clone(), qH.codes.clone()
    say("[graph] capture")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        step()
    torch.cuda.synchronize()
    for rep in range(4):
        Y.zero_()
        qH.codes.zero_()
        A2 = (A.float() * 0.5).to(torch.bfloat16)   # unrelated eager work between the replays
        torch.cuda.synchronize()
        say(f"[graph] replay {rep}")
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y, want) and torch.equal(qH.codes, want_codes), f"replay {rep}"
        del A2


def test_one_launch_quantizer_replayed_from_a_graph_on_changing_data(oracle):
    """The one-launch quantizer tells the maxima of this launch from those of earlier ones by an epoch.  A
    captured launch is replayed with identical kernel arguments, so the epoch is counted on the device: every
    replay below quantizes NEW contents of the same buffer (tensor maximum moved to another workgroup's slice,
    larger, then much smaller than before), with eager calls of the same entry points in between, and must
    return the oracle's bytes each time.  Plain rule, scale search, smoothed keys and the allocation-free entry."""
    g = np.random.default_rng(404)
    R, C = 3000, 1040                                   # several register slots on 256 workgroups, ragged tail
    x = torch.empty((R, C), dtype=torch.bfloat16, device="cuda")
    kv = torch.empty((200, 24, 128), dtype=torch.bfloat16, device="cuda")
    q6, q46 = nv.NVFP4Tensor(R, C, "cuda"), nv.NVFP4Tensor(R, C, "cuda")
    qk, qn = nv.NVFP4Tensor(200 * 24, 128, "cuda"), nv.NVFP4Tensor(200 * 24, 128, "cuda")
    mean = torch.empty(200 * 24, dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(max(nv.nvfp4_workspace_bytes(nv.OP_QUANTIZE, R, C), nv.nvfp4_workspace_bytes(nv.OP_KV_QUANT_K, 200, 24, 128)),
                     dtype=torch.uint8, device="cuda")

    def fill(rep):
        xs = g.standard_normal((R, C)).astype(np.float32) * np.float32([1.0, 3.0, 0.01, 40.0][rep])
        xs[g.integers(0, R), g.integers(0, C)] = np.float32([50.0, 900.0, 0.5, 7000.0][rep])
        ks = wl.bf16_bits_to_f32(wl.kv_tensor(200, 24, 128, 8, rep)) * np.float32([1.0, 0.02, 30.0, 4.0][rep]) + np.float32(0.75)
        xb, kb = wl.to_bf16_bits(xs), wl.to_bf16_bits(ks.astype(np.float32))
        x.copy_(dev_bf16(xb))
        kv.copy_(dev_bf16(kb).reshape(200, 24, 128))
        return xb, kb.reshape(4800, 128)

    def step():
        nv.nvfp4_quantize(x, out=q6, workspace=ws)
        nv.nvfp4_quantize_4over6(x, out=q46, workspace=ws)
        nv.nvfp4_kv_quant_k(kv, out=qk, row_mean=mean, workspace=ws)
        nv.nvfp4_kv_quant_noalloc(kv, out=qn)

    nv.nvfp4_set_one_launch(nv.ONE_LAUNCH_ALWAYS)       # (the default rule would take two passes for some of these sizes)
    fill(0)
    step()                                              # eager: first use of every kernel variant
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        step()
    torch.cuda.synchronize()
    for rep in range(4):
        xb, kb = fill(rep)
        other = nv.nvfp4_quantize(dev_bf16(xb[:500]))   # eager launches between the replays use the same slots in turn
        torch.cuda.synchronize()
        say(f"[graph] one-launch quantizer, replay {rep}")
        graph.replay()
        torch.cuda.synchronize()
        assert_q_equal(q6, oracle.quantize(xb), f"plain, replay {rep}")
        assert_q_equal(q46, oracle.quantize(xb, four_over_six=True), f"search, replay {rep}")
        want_mean, want_k = _oracle_k_path(oracle, kb)
        assert (nv.bits_from_bf16(mean) == want_mean).all(), f"row means, replay {rep}"
        assert_q_equal(qk, want_k, f"smoothed keys, replay {rep}")
        assert_q_equal(qn, oracle.quantize(kb), f"allocation-free entry, replay {rep}")
        del other
    nv.nvfp4_set_one_launch()                           # back to the default rule


def test_full_size_ffn_pair_config3(oracle):
    cfg = wl.config3()
    M, D, F = wl.TOKENS_INFER, wl.D_MODEL, wl.D_FFN
    say("[config3] quantize A, W1, W2")
    oa, ow1, ow2 = oracle.quantize(cfg["A"]), oracle.quantize(cfg["W1"]), oracle.quantize(cfg["W2"])
    ga = nv.nvfp4_quantize(dev_bf16(cfg["A"]))
    gw1 = nv.nvfp4_quantize(dev_bf16(cfg["W1"]))
    gw2 = nv.nvfp4_quantize(dev_bf16(cfg["W2"]))
    assert_q_equal(ga, oa, "A")
    assert_q_equal(gw1, ow1, "W1")
    assert_q_equal(gw2, ow2, "W2")
    say("[config3] up projection + GELU + re-quantize (scale from amax)")
    h = _nan_filled(M, F, torch.bfloat16)
    gh = nv.nvfp4_gemm_act_quant(ga, gw1, nv.ACT_GELU_TANH, h_bf16=h)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(h).all()), "part of H was never written"
    hb = nv.bits_from_bf16(h)
    oh = oracle.quantize(hb)
    assert_q_equal(gh, oh, "fused H")            # fused bytes == quantizer applied to the H the GPU produced
    rows = _sample_rows(M, 512, 3)
    Y1, S1 = oracle.gemm(oa, ow1, rows=rows)
    want = wl.bf16_bits_to_f32(oracle.gelu_tanh_bf16(Y1)).astype(np.float64)
    got = wl.bf16_bits_to_f32(hb[rows]).astype(np.float64)
    assert (np.abs(got - want) <= 2.0 ** -7 * np.abs(want) + 2.0 ** -15 * S1 + 1e-30).all()
    say("[config3] single-pass variant with the same scale gives the same bytes")
    gs = gh.global_scale.clone()
    gh2 = nv.nvfp4_gemm_act_quant(ga, gw1, nv.ACT_GELU_TANH, global_scale_in=gs)
    a, b = host_q(gh), host_q(gh2)
    assert (a[0] == b[0]).all() and (a[1] == b[1]).all() and a[2] == b[2]
    say("[config3] down projection")
    Y2, S2 = oracle.gemm(oh, ow2, rows=rows)
    y32 = nv.nvfp4_gemm(gh, gw2, nv.OUT_F32, Y=_nan_filled(M, D, torch.float32))
    assert bool(torch.isfinite(y32).all()), "part of the down projection was never written"
    fro, worst = assert_gemm_close(y32.cpu().numpy()[rows], Y2, S2, "down projection")
    say(f"        rel fro {fro:.2e}  worst err/S {worst:.2e}  ({len(rows)} rows)")
    y16 = nv.nvfp4_gemm(gh, gw2, nv.OUT_BF16, Y=_nan_filled(M, D, torch.bfloat16))
    assert (nv.bits_from_bf16(y16) == nv.bits_from_bf16(y32.to(torch.bfloat16))).all()


def test_full_size_kv_cache_config4(oracle):
    cfg = wl.config4()
    T, H, d = wl.KV_TOKENS, wl.KV_HEADS, wl.KV_DIM
    for name in ("K", "V"):
        say(f"[config4] {name}")
        oq = oracle.quantize(cfg[name].reshape(T * H, d))
        gq = nv.nvfp4_kv_quant(dev_bf16(cfg[name]))
        assert_q_equal(gq, oq, name)
        back = nv.bits_from_bf16(nv.nvfp4_kv_dequant(gq, T, H, d)).reshape(T * H, d)
        want = oracle.dequant_bf16(oq)
        assert (back == want).all()
        x = wl.bf16_bits_to_f32(cfg[name]).astype(np.float64).reshape(T * H, d)
        xh = wl.bf16_bits_to_f32(back).astype(np.float64)
        rel = np.linalg.norm(x - xh) / np.linalg.norm(x)
        say(f"        round-trip relative Frobenius error {rel:.4f} (reported, no closed form)")
        assert 0.02 < rel < 0.2
        # storage: 9/16 byte per element against 2 in bf16
        assert (gq.codes.numel() + gq.scales.numel()) * 16 == 9 * T * H * d
    say("[config4] K with the four-over-six scale search")
    oq = oracle.quantize(cfg["K"].reshape(T * H, d), four_over_six=True)
    gq = nv.nvfp4_kv_quant_4over6(dev_bf16(cfg["K"]))
    assert_q_equal(gq, oq, "K 4over6")
    back = nv.bits_from_bf16(nv.nvfp4_kv_dequant(gq, T, H, d)).reshape(T * H, d)
    x = wl.bf16_bits_to_f32(cfg["K"]).astype(np.float64).reshape(T * H, d)
    rel46 = np.linalg.norm(x - wl.bf16_bits_to_f32(back).astype(np.float64)) / np.linalg.norm(x)
    say(f"        round-trip relative Frobenius error with the search {rel46:.4f}")
    assert rel46 < rel          # rel: the plain rule on V above; K and V are drawn alike
    say("[config4] K with smoothing and the scale search, reconstructed as a window of 21 chunks")
    Tc = 880
    chunks, want = [], []
    for c in range(T // Tc):
        kb = cfg["K"][c * Tc:(c + 1) * Tc].reshape(Tc * H, d)
        m, q = _oracle_k_path(oracle, kb)
        want.append(oracle.dequant_bf16(q, m))
        gq, gm = nv.nvfp4_kv_quant_k(dev_bf16(kb).reshape(Tc, H, d))
        assert (nv.bits_from_bf16(gm) == m).all()
        assert_q_equal(gq, q, f"K chunk {c}")
        chunks.append((gq, gm, Tc))
    got = nv.bits_from_bf16(nv.nvfp4_kv_dequant_gather(chunks, H, d)).reshape(T * H, d)
    assert (got == np.concatenate(want)).all()


def test_full_size_training_triplet_config5(oracle):
    cfg = wl.config5()
    Mt, D, F = wl.TOKENS_TRAIN, wl.D_MODEL, wl.D_FFN
    x, w, dy = dev_bf16(cfg["X"]), dev_bf16(cfg["W"]), dev_bf16(cfg["dY"])
    q = {}
    for name, bits, t in (("X", cfg["X"], x), ("W", cfg["W"], w), ("dY", cfg["dY"], dy)):
        for axis in (0, 1):
            say(f"[config5] quantize {name} axis {axis}")
            oq = oracle.quantize(bits, block_axis=axis)
            gq = nv.nvfp4_quantize(t, block_axis=axis)
            assert_q_equal(gq, oq, f"{name} axis {axis}")
            q[(name, axis)] = (oq, gq)
    for what, a, b in (("fprop X W^T", ("X", 0), ("W", 0)),          # [Mt, F], K = D
                       ("dgrad dY W", ("dY", 0), ("W", 1)),          # [Mt, D], K = F
                       ("wgrad dY^T X", ("dY", 1), ("X", 1))):       # [F, D],  K = Mt
        (oa, ga), (ob, gb) = q[a], q[b]
        rows = _sample_rows(oa.rows, 512, 5)
        say(f"[config5] {what}: {oa.rows}x{ob.rows}x{oa.K}")
        Y, S = oracle.gemm(oa, ob, rows=rows)
        y = nv.nvfp4_gemm(ga, gb, nv.OUT_F32, Y=_nan_filled(ga.rows, gb.rows, torch.float32))
        assert bool(torch.isfinite(y).all()), f"{what}: part of the output was never written"
        fro, worst = assert_gemm_close(y[torch.from_numpy(rows).cuda()].cpu().numpy(), Y, S, what)
        say(f"        rel fro {fro:.2e}  worst err/S {worst:.2e}  ({len(rows)} rows)")
        del y


def test_full_size_training_recipe_config5(oracle):
    """The later rows at the training layer's sizes, in the launch configurations the benchmark times:
    2-D weight scaling with the transposed operand, the Hadamard-transformed weight-gradient operands,
    the scale search on activations, and the all-to-all send buffers of one device's share of the
    attention window.  Every byte against the oracle."""
    cfg = wl.config5()
    say("[config5] 2-D scaling of W and W^T")
    want, want_t = oracle.quantize_2d(cfg["W"])
    got, got_t = nv.nvfp4_quantize_2d(dev_bf16(cfg["W"]))
    assert_q_equal(got, want, "W")
    assert_q_equal(got_t, want_t, "W^T")
    del got, got_t, want, want_t
    mask = 0x6D21
    for name in ("X", "dY"):
        say(f"[config5] Hadamard transform + transposed quantizer of {name}")
        want = oracle.quantize(oracle.rht_rows(cfg[name], mask), block_axis=1)
        got = nv.nvfp4_quantize_rht(dev_bf16(cfg[name]), mask)
        assert_q_equal(got, want, name)
        del got, want
    say("[config5] scale search on X")
    assert_q_equal(nv.nvfp4_quantize_4over6(dev_bf16(cfg["X"])), oracle.quantize(cfg["X"], four_over_six=True), "X 4over6")
    T, H, d, P = wl.KV_TOKENS // 4, wl.KV_HEADS, wl.KV_DIM, 4
    say(f"[config4] all-to-all send buffers {T}x{H}x{d} over {P} peers")
    xb = wl.config4()["K"][:T].reshape(T * H, d)
    want = oracle.quantize(xb)
    codes, scales, gs = host_q(nv.nvfp4_quantize_for_all_to_all(dev_bf16(xb).reshape(T, H, d), P))
    perm = lambda a: a.reshape(T, P, H // P, -1).transpose(1, 0, 2, 3).reshape(T * H, -1)
    assert gs.view(np.uint32) == np.float32(want.global_scale).view(np.uint32)
    assert (codes == perm(want.codes)).all() and (scales == perm(want.scales)).all()

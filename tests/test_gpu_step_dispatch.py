"""Layer-by-layer parity (tests/layerwise.py, bars of tests/test_gpu_layerwise.py) of small modules whose shapes sit at the
edges of the rules that choose a kernel: partly filled channel groups, remainders of tiles, the ends of a rule's range."""
import numpy as np
import pytest

import fdg_workloads as W
from fdg_workloads import Layer, ModuleSpec
from tests import test_gpu_kernels as TK
from tests import test_gpu_layerwise as LT

pytestmark = pytest.mark.gpu

H = dict(momentum=0.9, weight_decay=5e-4, bn_eps=1e-5, bn_momentum=0.1, lr=0.01)


def check(name, spec):
    print(f"case {name} layer by layer", flush=True)
    plain = []
    LT._judge(LT._run(spec, seed=1, steps_after_warmup=2, plain=plain), name)
    LT._judge_plain(plain, name)


# A module with narrow 3x3 kernels keeps its batch-norm sums in eight copies, which the batch-norm kernels fold by workgroup:
# 1, 2, 4 and 8 channel groups a workgroup, one of them partly filled (24, 40 and 72 channels), one and two normalised operands
COPIES = {
    "copies preact": [Layer(W.BASIC_PREACT, 16, 16, 1), Layer(W.BASIC_PREACT, 16, 24, 1), Layer(W.BASIC_PREACT, 24, 8, 1),
                      Layer(W.BASIC_PREACT, 8, 72, 1)],
    "copies postact": [Layer(W.BASIC_POSTACT, 16, 40, 2), Layer(W.BASIC_POSTACT, 40, 8, 1), Layer(W.BASIC_POSTACT, 8, 72, 1),
                       Layer(W.BASIC_POSTACT, 72, 16, 1), Layer(W.BASIC_POSTACT, 16, 16, 1)],
}


@pytest.mark.parametrize("name", sorted(COPIES))
def test_sums_in_copies(name):
    check(name, ModuleSpec(6, 16, 23, 21, COPIES[name], delay=1, is_bottom=False, beta=0.5, name=name, **H))


# The streams between layers are written only in the forms (fp32, bf16) that the next layer reads, a trace makes every layer
# write its fp32 form: the same bits either way, whatever follows what
STREAMS = {
    "post": [Layer(W.STEM, 3, 16, 1), Layer(W.BASIC_POSTACT, 16, 32, 2), Layer(W.BASIC_PREACT, 32, 32, 1),
             Layer(W.BASIC_PREACT, 32, 64, 2), Layer(W.BASIC_POSTACT, 64, 64, 1), Layer(W.BOTTLENECK_POSTACT, 64, 64, 1)],
    "pre": [Layer(W.STEM, 3, 16, 1), Layer(W.BASIC_PREACT, 16, 32, 1), Layer(W.BASIC_PREACT, 32, 32, 1),
            Layer(W.BASIC_POSTACT, 32, 32, 1), Layer(W.INVERTED_RESIDUAL, 32, 32, 1), Layer(W.INVERTED_RESIDUAL, 32, 16, 2)],
}


@pytest.mark.parametrize("name", sorted(STREAMS))
@pytest.mark.parametrize("replay", [False, True])
def test_streams_with_and_without_a_trace(name, replay):
    import torch as t
    from paper_1906_09108_amd import FdgModule
    spec = ModuleSpec(4, 3, 16, 16, STREAMS[name], delay=1, is_bottom=True, beta=0.5, name=name, **H)
    results = []
    for traced in (False, True):
        m = FdgModule(spec, save_mode=1 if replay else 0)
        m.set_params(W.make_params(spec, 0, perturb_bn=True))
        if traced:
            m.trace_attach()
        for it in range(3):
            y = m.forward(t.from_numpy(W.make_input(spec, it, 0)).cuda())
            if it >= 1:
                m.backward_delayed(t.from_numpy(W.make_grad_out(spec, it - 1, 0)).cuda())
                m.update(spec.lr)
        results.append((y.cpu().numpy(), m.get_grads(), m.get_params(), m.get_bn_running()))
        m.close()
    for a, b in zip(*results):
        assert np.isfinite(a).all() and np.array_equal(a, b)


# A thread makes 2 x 2 cells of a depthwise convolution and walks segments of 8 cells for its weight gradient: odd heights and
# widths, single rows and columns, one cell more and less than a segment, a partly filled block of 8 channel groups
@pytest.mark.parametrize("case", [(2, 1, 17, 72, 1), (3, 17, 1, 8, 2), (2, 8, 8, 64, 1), (2, 15, 16, 72, 2), (5, 7, 15, 136, 1), (1, 2, 2, 8, 2)])
def test_depthwise_edges(case):
    TK.test_depthwise_convolution_kernels(case)


# The weight gradient's chunks: a segment to a lane with the scratch it asks for, longer ones with less (a chunk per 256 cells is
# enough, less is refused); single-pixel images, rows a cell longer than a segment, more segments than chunks
@pytest.mark.parametrize("case", [(1024, 1, 1, 64, 1), (40, 3, 9, 72, 1), (600, 2, 2, 16, 2), (64, 33, 33, 128, 1)])
def test_depthwise_weight_gradient_at_scratch_limits(case):
    import torch as t
    from paper_1906_09108_amd import kernels as K
    n, h, w, c, s = case
    print("depthwise scratch", case, flush=True)
    ho, wo = (h - 1) // s + 1, (w - 1) // s + 1
    rng = np.random.default_rng(19)
    x, dy = (TK.bf16_round(rng.standard_normal(sh).astype(np.float32)) for sh in ((n, c, h, w), (n, c, ho, wo)))
    xd, dyd = TK.to_dev_nhwc_b16(x), TK.to_dev_nhwc_b16(dy)
    ref = TK.K32.dwconv_bwd_weight(x, dy, 3, s, 1)
    segments, groups = n * ho * -(-wo // 8), -(-c // 64)
    full, least = (min(-(-1024 // groups), k) for k in (-(-segments // 32), -(-n * ho * wo // 256)))
    assert K.fdgk_dwconv3_wgrad_scratch_bytes(n, h, w, c, s) == full * 36 * c
    for chunks in sorted({full, (full + least) // 2, least}):
        scratch = t.full((chunks * 9 * c,), float("nan"), device="cuda")
        dw = t.full((c, 9), float("nan"), device="cuda")
        K.fdgk_dwconv3_wgrad(xd, dyd, dw, scratch, n, h, w, c, s)
        assert TK.rel(dw.cpu().numpy().reshape(c, 1, 3, 3), ref) <= TK.F32_TOL, chunks
    with pytest.raises(RuntimeError):
        K.fdgk_dwconv3_wgrad(xd, dyd, dw, t.empty(least * 9 * c - 1, device="cuda"), n, h, w, c, s)


# A tap outside the image is left out, not multiplied by zero: an infinite weight, activation or gradient reaches the results
# that it reaches in the definition and no others
@pytest.mark.parametrize("where", ["weights", "activations", "gradients"])
@pytest.mark.parametrize("case", [(2, 5, 11, 72, 1), (2, 6, 9, 16, 2), (1, 8, 8, 16, 1), (2, 7, 18, 16, 2)])
def test_infinities_at_the_border_of_a_depthwise_convolution(case, where):
    import torch as t
    from paper_1906_09108_amd import kernels as K
    n, h, w, c, s = case
    print("depthwise infinities", case, where, flush=True)
    ho, wo = (h - 1) // s + 1, (w - 1) // s + 1
    rng = np.random.default_rng(17)
    x, wgt, dy = (TK.bf16_round(rng.standard_normal(sh).astype(np.float32)) for sh in ((n, c, h, w), (c, 1, 3, 3), (n, c, ho, wo)))
    marked = {"weights": wgt, "activations": x, "gradients": dy}[where]
    rows, cols = (sorted({0, z // 2, z - 1}) for z in marked.shape[2:])
    for k, (i, j) in enumerate((i, j) for i in rows for j in cols):      # a corner, an edge or the middle in channel k of image 0
        marked[0 if where != "weights" else k, k if where != "weights" else 0, i, j] = np.inf if k % 2 else -np.inf
    xd, dyd = TK.to_dev_nhwc_b16(x), TK.to_dev_nhwc_b16(dy)
    wt = t.from_numpy(np.ascontiguousarray(wgt.reshape(c, 9).T)).to(t.bfloat16).cuda()
    y, dx = (t.empty(sh, dtype=t.bfloat16, device="cuda") for sh in ((n, ho, wo, c), (n, h, w, c)))
    dw = t.empty((c, 9), device="cuda")
    scratch = t.empty(K.fdgk_dwconv3_wgrad_scratch_bytes(n, h, w, c, s) // 4, device="cuda")
    K.fdgk_dwconv3_fwd(xd, wt, y, n, h, w, c, s)
    K.fdgk_dwconv3_dgrad(dyd, wt, dx, n, h, w, c, s)
    K.fdgk_dwconv3_wgrad(xd, dyd, dw, scratch, n, h, w, c, s)
    with np.errstate(invalid="ignore"):
        pairs = {"forward": (TK.nhwc_to_nchw(y), TK.K32.dwconv_fwd(x, wgt, s, 1), TK.B16_TOL),
                 "data gradient": (TK.nhwc_to_nchw(dx), TK.K32.dwconv_bwd_data(dy, wgt, x.shape, s, 1), TK.B16_TOL),
                 "weight gradient": (dw.cpu().numpy().reshape(c, 1, 3, 3), TK.K32.dwconv_bwd_weight(x, dy, 3, s, 1), TK.F32_TOL)}
    for name, (got, ref, tol) in pairs.items():
        ok = np.isfinite(ref)
        assert np.array_equal(np.where(ok, 0, got), np.where(ok, 0, ref), equal_nan=True), name
        assert np.isfinite(got[ok]).all() and np.abs(got[ok] - ref[ok]).max() <= tol * np.abs(ref[ok]).max(), name


# Classes on 16 lanes or a wave to a row, and 16 classes to a step of the gradient: at, below and above those counts
@pytest.mark.parametrize("case", [(70, 2, 2, 24, 15), (3, 1, 1, 8, 16), (65, 2, 2, 16, 17), (17, 1, 2, 40, 65), (5, 1, 1, 8, 1)])
def test_head_edges(case):
    TK.test_head_kernels_one_by_one(case)


# 64 -> 64 channel weight gradients: one tile per workgroup and one row, several tiles with a ragged last one (two buffers), an
# image too wide for two buffers, the same with more tiles than workgroups, the widest images the kernel takes and one column
# more.  The kernel alone, to the bound of 32-bit sums: through a whole block a pre-activation that two orders of a sum put on
# either side of zero moves a gradient of so few pixels by more than the kernel's own error.
@pytest.mark.parametrize("case,narrow", [((3, 1, 7, 64, 64, 3, 1), True), ((4, 9, 21, 64, 64, 3, 1), True),
                                         ((23, 47, 50, 64, 64, 3, 1), True), ((2, 3, 170, 64, 64, 3, 1), True),
                                         ((2, 130, 160, 64, 64, 3, 1), True), ((1, 3, 286, 64, 64, 3, 1), True),
                                         ((1, 3, 287, 64, 64, 3, 1), False)])
def test_weight_gradient_of_64_channels(case, narrow):
    from paper_1906_09108_amd import kernels as K
    TK.test_conv_wgrad(case)
    assert (K.fdgk_last_kernel() == "conv_wgrad_narrow64_kernel") == narrow, K.fdgk_last_kernel()


# The slices of one weight gradient are added up by the next, of the same and of another width; with a few images and, where the
# next has fewer tiles than it takes workgroups to add them up, with one
@pytest.mark.parametrize("n,h,w", [(8, 21, 19), (1, 12, 11)])
@pytest.mark.parametrize("name", ["64 64", "32 64", "64 32"])
def test_slices_of_an_earlier_weight_gradient(name, n, h, w):
    first, second = (int(c) for c in name.split())
    layers = [Layer(W.BASIC_POSTACT, first, first, 1), Layer(W.BASIC_POSTACT, first, second, 1), Layer(W.BASIC_POSTACT, second, second, 1)]
    check(f"slices {name} n{n}", ModuleSpec(n, first, h, w, layers, delay=1, is_bottom=False, beta=0.5, name=f"slices {name}", **H))


# 1x1 layers of few output channels behind a long contraction and of 72 .. 120 input channels: both ends of the ranges on either
# side of the tiles a rule asks for, a ragged last tile of pixels, channel counts that fill no tile, stride 2.  With each the
# kernels that forward and data gradient run.
GENERIC64, GENERIC = "conv_gather_kernel<128, 64, 2, 2>", "conv_gather_kernel<128, 128, 2, 2>"
PIPE, THIN64, THIN96, PAIR = "conv_gather_pipe_kernel<128, 4, false>", *(f"conv_gather_dma_pair_kernel<{k}>" for k in ("64, 3", "96, 4", "128, 2"))
THIN = [((9, 43, 43, 128, 40, 1, 1), THIN64, GENERIC), ((9, 43, 43, 192, 64, 1, 1), THIN64, PIPE),
        ((8, 45, 45, 128, 64, 1, 1), GENERIC64, PIPE), ((9, 43, 43, 128, 72, 1, 1), THIN96, GENERIC),
        ((9, 43, 43, 128, 104, 1, 1), GENERIC, GENERIC), ((8, 46, 46, 384, 96, 1, 1), THIN96, PAIR),
        ((37, 23, 23, 72, 264, 1, 1), PAIR, GENERIC), ((33, 23, 23, 72, 152, 1, 1), GENERIC, GENERIC),
        ((21, 31, 31, 120, 264, 1, 1), PAIR, GENERIC), ((9, 85, 85, 128, 64, 1, 2), THIN64, PIPE),
        ((9, 43, 43, 64, 128, 1, 1), PIPE, THIN64)]


@pytest.mark.parametrize("case,forward,dgrad", THIN)
def test_thin_1x1_layers(case, forward, dgrad):
    from paper_1906_09108_amd import kernels as K
    TK.test_conv_fwd(case)
    assert K.fdgk_last_kernel() == forward
    TK.test_conv_dgrad(case)
    assert K.fdgk_last_kernel() == dgrad
    TK.test_conv_wgrad(case)


# One round of workgroups means longer sums: the 1x1 weight gradient against 64 bits on long lists of pixels.  The error of fp32
# sums grows with the pixels of one sum; on the generic kernel, with 1024 workgroups, one sum each, it is 1.42e-7, 1.53e-7 and 1.79e-7
# here, with 512 it was 1.59e-7, 1.78e-7 and 2.10e-7.  Bounds: 4 % above the former.  Unit stride, as a list and as images, on the
# kernel that runs such layers in a network; stride 2 on the generic one
TWO_SUMS, RAGGED = "conv_wgrad_kernel<128, 128, two sums>", "conv_wgrad128w8_kernel<5, flat, ragged>"


@pytest.mark.parametrize("case, bound, kernel", [
    ((1, 131072, 1, 384, 64, 1, 1), 1.48e-7, RAGGED), ((1, 134912, 1, 448, 64, 1, 1), 1.59e-7, RAGGED),
    ((1, 401408, 1, 72, 136, 1, 1), 1.86e-7, RAGGED), ((128, 32, 32, 384, 64, 1, 1), 1.48e-7, RAGGED),
    ((31, 68, 64, 448, 64, 1, 1), 1.59e-7, RAGGED), ((128, 56, 56, 72, 136, 1, 1), 1.86e-7, RAGGED),
    ((128, 64, 64, 384, 64, 1, 2), 1.48e-7, TWO_SUMS), ((31, 136, 128, 448, 64, 1, 2), 1.59e-7, TWO_SUMS),
    ((128, 112, 112, 72, 136, 1, 2), 1.86e-7, TWO_SUMS),
])
def test_weight_gradient_of_1x1_layers_against_64_bits(case, bound, kernel):
    import torch as t
    from paper_1906_09108_amd import kernels as K
    n, h, w, ci, co, k, s = case
    pixels = n * (h // s) * (w // s)
    g = t.Generator(device="cuda")
    g.manual_seed(3)
    x = t.randn(n, h, w, ci, generator=g, device="cuda").relu().bfloat16()
    dy = t.randn(pixels, co, generator=g, device="cuda").bfloat16()
    scratch = t.empty(K.fdgk_conv_wgrad_scratch_bytes(*case) // 4, device="cuda")
    dw = t.empty(co, ci, device="cuda")
    K.fdgk_conv_wgrad(x, dy, dw, scratch, *case, overwrite=True)
    ran = K.fdgk_last_kernel()
    ref = dy.cpu().double().T @ x[:, ::s, ::s].reshape(pixels, ci).cpu().double()
    err = float((dw.cpu().double() - ref).norm() / ref.norm())
    print(f"1x1 weight gradient {case}: {err:.3e}", flush=True)
    assert ran == kernel
    assert err <= bound


# The bytes that timing records charge are those of the tensors a launch is given: a gradient that arrives gated needs no gate, the
# forms of the stream that nobody reads are not written, a batch norm without an activation behind it reads no gate
@pytest.mark.parametrize("name", ["basic", "projecting", "inverted", "inverted with sums"])
def test_bytes_of_the_timing_records(name):
    import torch as t
    from paper_1906_09108_amd import FdgModule
    if name == "basic":
        spec = ModuleSpec(8, 16, 16, 16, [Layer(W.BASIC_POSTACT, 16, 16, 1)] * 2, delay=0, beta=0.5, name=name, **H)
        e, w = 8 * 16 * 16 * 16, 2 * 16 * 9 * 16
        # conv2 of the upper block (bf16 in; gate, batch-norm input, fp32 out); its conv1 (fp32 gradient and batch-norm input in,
        # bf16 out; gated fp32 shortcut, gate and batch-norm input of the block below, fp32 out); the lower block's, fed from above
        expected = {"conv_dgrad": e * ((2 + 8) + (8 + 6 + 4 + 4) + (8 + 4 + 4) + (8 + 4 + 4)) + 4 * w, "bn_bwd": e * (8 + 8 + 2)}
    elif name == "projecting":
        spec = ModuleSpec(2, 128, 8, 8, [Layer(W.BASIC_POSTACT, 128, 128, 2)], delay=0, beta=0.5, name=name, **H)
        e, o, w, wp = 2 * 64 * 128, 2 * 16 * 128, 128 * 9 * 128, 128 * 128
        # conv2 (bf16 in, gate and batch-norm input, bf16 out), then conv1 and the projection in one launch (fp32 out)
        expected = {"conv_dgrad": 2 * o + 2 * w + o * (2 + 2 + 2) + 2 * (o + o) + 2 * (w + wp) + 4 * e}
    elif name == "inverted":
        spec = ModuleSpec(2, 16, 8, 8, [Layer(W.INVERTED_RESIDUAL, 16, 16, 1)], delay=0, beta=0.5, name=name, **H)
        m = 2 * 8 * 8
        # the closing batch norm and the one after the depthwise convolution in two passes; the first one's sums come out of the
        # depthwise data gradient, so only its apply pass runs
        expected = {"bn_bwd": m * 16 * (6 + 6 + 2) + m * 96 * (8 + 8 + 2) + m * 96 * (4 + 2 + 2)}
    else:
        spec = ModuleSpec(2, 64, 8, 8, [Layer(W.INVERTED_RESIDUAL, 64, 64, 1)], delay=0, beta=0.5, name=name, **H)
        m, w = 2 * 8 * 8, 64 * 384
        # projecting convolution (bf16 in; gate and batch-norm input, fp32 out), expanding one (bf16 in, fp32 shortcut, fp32 out);
        # both batch norms of 384 channels have their sums already
        expected = {"conv_dgrad": 2 * m * 64 + 2 * w + m * 384 * (2 + 2 + 4) + 2 * m * 384 + 2 * w + m * 64 * (4 + 4),
                    "bn_bwd": m * 64 * (6 + 6 + 2) + 2 * m * 384 * (4 + 2 + 2)}
    mod = FdgModule(spec)
    mod.set_params(W.make_params(spec, 0))
    mod.profile_enable(True)
    x, g = (t.from_numpy(f(spec, 0, 0)).cuda() for f in (W.make_input, W.make_grad_out))
    mod.forward(x)
    mod.backward_delayed(g, t.empty_like(x))
    got = {}
    for r in mod.profile_read():
        got[r["name"]] = got.get(r["name"], 0) + r["bytes"]
    mod.close()
    for k, v in expected.items():
        assert got[k] == v, (k, got[k], v)

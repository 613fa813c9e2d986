"""Kernels chosen by a rule on sizes, at the edges of that rule and at shapes that divide into none of their tiles: the parity
checks of tests/test_gpu_kernels.py (same oracle, same bars), with the kernel that ran named."""
import numpy as np
import pytest

import fdg_workloads as W
from fdg_workloads import Layer, ModuleSpec
from tests import layerwise as LW
from tests import test_gpu_kernels as TK
from tests import test_gpu_layerwise as LT
from tests import test_gpu_step_dispatch as TD

pytestmark = pytest.mark.gpu


# 64 -> 64 channels over at least 65536 pixels: whole rows of one image to a tile.  Rows that fill a tile, rows that leave a part
# of it, a last tile of one row, images lower than a tile, more rounds of loads for the patch; below and beside the rule: the
# kernel that ran before
@pytest.mark.parametrize("case, kernel", [
    ((16, 64, 64, 64, 64, 3, 1), "conv_narrow64_kernel"),
    ((17, 63, 63, 64, 64, 3, 1), "conv_narrow64_kernel"),
    ((22, 55, 56, 64, 64, 3, 1), "conv_narrow64_kernel"),
    ((69, 31, 31, 64, 64, 3, 1), "conv_narrow64_kernel"),
    ((520, 16, 8, 64, 64, 3, 1), "conv_narrow64_kernel"),
    ((1366, 3, 16, 64, 64, 3, 1), "conv_narrow_kernel<64, 2, 2, 4>"),   # 48 pixels an image: less than half a tile
    ((8, 88, 94, 64, 64, 3, 1), "conv_narrow_kernel<64, 2, 2, 4>"),     # the patch takes more rounds than there are
    ((15, 64, 64, 64, 64, 3, 1), "conv_narrow_kernel<64, 2, 2, 2>"),
])
def test_64_channels_over_many_pixels(case, kernel):
    from paper_1906_09108_amd import kernels as K
    for check in (TK.test_conv_fwd, TK.test_conv_dgrad, TK.test_data_gradient_that_feeds_the_layer_below):
        check(case)
        assert K.fdgk_last_kernel() == kernel


# Wide 3x3 convolutions of few tiles: the contraction in parts, added up by a launch of its own that does the output stage.  Whole
# parts and parts of two lengths, ragged pixel and channel tiles, a partly filled last channel block, both tile widths; forward, and
# the data gradients with gate and sums, with an addend, and plain, as a step of a module makes them
@pytest.mark.parametrize("kind, c_in, c_out, n, h, w, delay, kernel", [
    (W.BASIC_PREACT, 640, 640, 5, 7, 9, 1, "conv_patch_kernel<160, 160, 5> in parts"),
    (W.BASIC_PREACT, 584, 640, 3, 9, 17, 1, "conv_patch_kernel<160, 192, 5> in parts"),
    (W.BASIC_POSTACT, 640, 640, 9, 16, 8, 1, "conv_patch_kernel<160, 160, 5> in parts"),
    (W.BASIC_PREACT, 568, 584, 2, 5, 30, 1, "conv_patch_kernel<128, 192, 5, true> in parts"),
    (W.BASIC_PREACT, 512, 512, 4, 8, 8, 1, "conv_patch_kernel<128, 160, 5> in parts"),
    (W.BASIC_PREACT, 512, 512, 17, 8, 8, 1, "conv_patch_kernel<128, 160, 5>"),   # 36 tiles: eight blocks in fewer than eight parts
    (W.BASIC_PREACT, 640, 640, 17, 12, 12, 0, "conv_patch_kernel<160, 160, 5> in parts"),   # 80 tiles: three parts fill a round,
    (W.BASIC_PREACT, 640, 640, 17, 12, 12, 1, "conv_patch_kernel<160, 160, 5>"),   # and half a round, where two streams run, is full
])
def test_contraction_in_parts(kind, c_in, c_out, n, h, w, delay, kernel):
    from paper_1906_09108_amd import FdgModule, kernels as K
    import torch as t
    spec = ModuleSpec(n, c_in, h, w, [Layer(kind, c_in, c_out, 1)], delay=delay, is_bottom=False, beta=0.5, name="parts", **TD.H)
    TD.check(f"parts {c_in}>{c_out} {n}x{h}x{w}", spec)
    m = FdgModule(spec)
    m.set_params(W.make_params(spec, 0))
    x = t.zeros((n, c_in, h, w), device="cuda")
    m.forward(x, None, m.new_output())
    t.cuda.synchronize()
    assert K.fdgk_last_kernel() == kernel
    m.close()


# One split added to what dw held, without scratch: the sum that the same launch writes over dw, plus dw, rounded once
@pytest.mark.parametrize("case, kernel", [
    ((8, 7, 7, 160, 160, 1, 1), "conv_wgrad128w8_kernel<5, flat, ragged>"),
    ((5, 7, 9, 136, 152, 3, 1), "conv_wgrad128w8_kernel<5, flat, ragged>"),
    ((1, 16, 16, 64, 128, 3, 1), "conv_wgrad128w8_kernel<5, paired>"),
    ((1, 16, 16, 256, 160, 3, 2), "conv_wgrad_tall_kernel<4, columns>"),
])
def test_one_split_added_to_the_weight_gradient(case, kernel):
    from paper_1906_09108_amd import kernels as K
    import torch as t
    n, h, w, ci, co, k, s = case
    gen = t.Generator(device="cuda")
    gen.manual_seed(0)
    ho, wo = (h - 1) // s + 1, (w - 1) // s + 1
    x, dy = (t.randn(m, generator=gen, device="cuda").to(t.bfloat16) for m in (n * h * w * ci, n * ho * wo * co))
    held = t.randn(co * k * k * ci, generator=gen, device="cuda")
    written, added = t.empty_like(held), held.clone()
    K.fdgk_conv_wgrad(x, dy, written, None, n, h, w, ci, co, k, s, overwrite=True)
    assert K.fdgk_last_kernel() == kernel
    K.fdgk_conv_wgrad(x, dy, added, None, n, h, w, ci, co, k, s)
    assert K.fdgk_last_kernel() == kernel
    assert t.equal(added, held + written)


# A chain's top module keeps no history, but where two and more modules run beside it, it fills half a round as they do (64 tiles: two
# parts would not pay), and a whole one again once the chain is gone
@pytest.mark.parametrize("modules", [2, 3])
def test_contraction_in_parts_of_a_chain(modules):
    from paper_1906_09108_amd import FdgChain, binding
    import torch as t
    common = dict(n=32, h_in=8, w_in=8, num_classes=10, **TD.H)
    wide = Layer(W.BASIC_PREACT, 640, 640, 1)
    layers = [[Layer(W.STEM, 3, 16, 1), Layer(W.BASIC_PREACT, 16, 640, 1)], [wide], [wide, Layer(W.HEAD_PREACT, 640)]]
    if modules == 2:
        del layers[1]
    specs = [ModuleSpec(c_in=ls[0].c_in, layers=ls, delay=2 * (modules - 1 - k), is_bottom=k == 0, beta=0.5 if k < modules - 1 else 1.0,
                        name=f"module {k}", **common) for k, ls in enumerate(layers)]
    chain = FdgChain(specs)
    for m, sp in zip(chain.modules, specs):
        m.set_params(W.make_params(sp, 0))
    top = chain.modules[-1]
    x, labels = t.randn((32, 3, 8, 8), device="cuda"), t.zeros(32, device="cuda", dtype=t.int32)

    def parts(step):
        top.profile_enable(True)
        step()
        t.cuda.synchronize()
        kernels = [r["kernel"] for r in top.profile_read() if r["name"] in ("conv_fwd", "conv_dgrad") and "conv_patch_kernel" in r["kernel"]]
        assert kernels
        return ["in parts" in k for k in kernels]

    assert set(parts(lambda: [chain.step(x, labels, 0.01) for _ in range(modules + 1)])) == {modules == 2}
    binding.load().fdg_chain_destroy(chain.handle)
    chain.handle = None
    assert all(parts(lambda: top.forward(t.randn((32, 640, 8, 8), device="cuda"), labels, top.new_output())))
    chain.close()


# Inverted residual blocks: data gradients of the 1x1 layers that end in a gate and sums (every instantiation: 64 channels and a partly
# filled block of 72 into the expanded tensor; 384, 576 and 432 channels down to 64, 96 and 72), the depthwise kernels with sums (a
# partly filled block of channels, odd images, both strides, more and fewer cells than a round takes), blocks that feed the one below
@pytest.mark.parametrize("channels, n, h, w", [
    ([(64, 64, 1), (64, 96, 1), (96, 96, 1)], 3, 13, 11),
    ([(64, 72, 2), (72, 72, 1), (72, 64, 2)], 2, 19, 23),
    ([(24, 40, 1), (40, 64, 2), (64, 64, 1)], 5, 9, 12),
    ([(96, 96, 1)], 1, 6, 6),
])
def test_inverted_blocks_with_sums(channels, n, h, w):
    layers = [Layer(W.INVERTED_RESIDUAL, ci, co, s) for ci, co, s in channels]
    spec = ModuleSpec(n, channels[0][0], h, w, layers, delay=1, is_bottom=False, beta=0.5, name="inverted", **TD.H)
    print(f"case inverted {channels} {n}x{h}x{w}", flush=True)
    LT._judge(LT._run(spec, seed=1, steps_after_warmup=2), f"inverted {channels[0][0]}-{channels[-1][1]} {n}x{h}x{w}")


# 64 -> 128 channels at stride 2: the data gradient's parity classes on the 1x1 kernels' loop (even and odd images, a last class
# of a single column, 72 and 96 channels), the weight gradient with two taps to a block (widths that divide 64; others: the
# generic kernel), and in a module the projection beside them and the sums of the layer below
@pytest.mark.parametrize("case, dgrad, wgrad", [
    ((3, 16, 16, 64, 128, 3, 2), "conv_gather_dma_pair_kernel<64, 3, classes>", "conv_wgrad128w8_kernel<5, paired>"),
    ((2, 64, 64, 64, 256, 3, 2), "conv_gather_dma_pair_kernel<64, 3, classes>", "conv_wgrad128w8_kernel<5, paired>"),
    ((5, 9, 14, 64, 128, 3, 2), "conv_gather_dma_pair_kernel<64, 3, classes>", "conv_wgrad_kernel<128, 128, 2, 2, 1>"),
    ((4, 7, 2, 72, 128, 3, 2), "conv_gather_dma_pair_kernel<96, 4, classes>", "conv_wgrad_kernel<128, 128, 2, 2, 1>"),
    ((2, 10, 6, 96, 192, 1, 2), "conv_gather_dma_pair_kernel<96, 4, classes>", "conv_wgrad_kernel<128, 128, two sums>"),
    ((4, 8, 8, 64, 128, 3, 1), None, "conv_wgrad128w8_kernel<5, paired>"),
])
def test_stride_2_into_few_channels(case, dgrad, wgrad):
    from paper_1906_09108_amd import kernels as K
    import torch as t
    n, h, w, ci, co, k, s = case
    if dgrad:
        TK.test_conv_dgrad(case)
        z = [t.zeros(c, device="cuda", dtype=t.bfloat16) for c in (n * h * w * co, ci * k * k * co)]
        K.fdgk_conv_dgrad(z[0], z[1], None, None, t.empty(n * h * w * ci, device="cuda"), None, n, h, w, ci, co, k, s)
        assert K.fdgk_last_kernel() == dgrad
    TK.test_conv_wgrad(case)
    assert K.fdgk_last_kernel() == wgrad


@pytest.mark.parametrize("c, n, h, w", [(64, 4, 14, 16), (64, 3, 9, 11), (96, 2, 6, 7)])
def test_projecting_block_that_feeds_the_one_below(c, n, h, w):
    layers = [Layer(W.BASIC_POSTACT, c, c, 1), Layer(W.BASIC_POSTACT, c, 2 * c, 2), Layer(W.BASIC_POSTACT, 2 * c, 2 * c, 1)]
    TD.check(f"projecting {c} {n}x{h}x{w}", ModuleSpec(n, c, h, w, layers, delay=1, is_bottom=False, beta=0.5, name="projecting", **TD.H))


# Weight gradients of unit stride whose pixels fill no whole chunk of 64 or whose channels no whole tile of 128: one chunk and a pixel,
# a last chunk of one row, more chunks than stages, sums folded more than once, both tiles ragged, 1x1, images of one row; scratch and
# none (test_conv_wgrad runs both); shapes just outside keep their kernels
@pytest.mark.parametrize("case, kernel", [
    ((5, 1, 13, 136, 128, 3, 1), "conv_wgrad128w8_kernel<5, flat, ragged>"),
    ((3, 7, 7, 128, 256, 3, 1), "conv_wgrad128w8_kernel<5, flat, ragged>"),
    ((9, 14, 14, 320, 200, 3, 1), "conv_wgrad128w8_kernel<5, flat, ragged>"),
    ((37, 14, 14, 256, 136, 1, 1), "conv_wgrad128w8_kernel<5, flat, ragged>"),
    ((50, 8, 9, 128, 128, 3, 1), "conv_wgrad128w8_kernel<5, flat, ragged>"),
    ((7, 28, 28, 160, 320, 3, 1), "conv_wgrad128w8_kernel<5, flat, ragged>"),
    ((3, 15, 15, 128, 256, 3, 1), "conv_wgrad_kernel<128, 128, 2, 2, 1>"),     # the validity of a pixel repeats too late
    ((4, 4, 4, 128, 120, 3, 1), "conv_wgrad_kernel<128, 128, 2, 2, 1>"),       # fewer than 128 channels
    ((1, 7, 9, 128, 128, 3, 1), "conv_wgrad_kernel<128, 128, 2, 2, 1>"),       # less than a chunk
    ((16, 14, 14, 128, 256, 3, 1), "conv_wgrad128w8_kernel<5, flat>"),
    # 1x1 of fewer than 128 channels on a side: one chunk and a pixel, any image width, a partly filled tile on either side or both,
    # 32 channels and just below, folds in the middle and at the end of a split; without scratch and at stride 2 the generic kernel
    ((5, 1, 13, 32, 40, 1, 1), "conv_wgrad128w8_kernel<5, flat, ragged>"),
    ((2, 31, 31, 32, 192, 1, 1), "conv_wgrad_kernel<128, 32, 4, 1, 1>"),       # smaller blocks, from 200 to 8192 pixels
    ((9, 31, 31, 32, 192, 1, 1), "conv_wgrad128w8_kernel<5, flat, ragged>"),
    ((1, 1, 199, 64, 40, 1, 1), "conv_wgrad128w8_kernel<5, flat, ragged>"),
    ((1, 8, 25, 64, 64, 1, 1), "conv_wgrad_kernel<32, 32, 1, 1, 4>"),
    ((8, 32, 32, 40, 64, 1, 1), "conv_wgrad_kernel<32, 32, 1, 1, 4>"),
    ((3, 2731, 1, 64, 64, 1, 1), "conv_wgrad128w8_kernel<5, flat, ragged>"),
    ((19, 15, 15, 576, 96, 1, 1), "conv_wgrad128w8_kernel<5, flat, ragged>"),
    ((64, 16, 16, 64, 384, 1, 1), "conv_wgrad128w8_kernel<5, flat, ragged>"),
    ((5, 64, 1, 64, 96, 1, 1), "conv_wgrad128w8_kernel<5, flat, ragged>"),     # one column
    ((4, 16, 16, 24, 144, 1, 1), "conv_wgrad_kernel<128, 32, 4, 1, 1>"),
    ((8, 16, 16, 64, 384, 1, 2), "conv_wgrad_kernel<128, 128, two sums>"),
])
def test_ragged_weight_gradients(case, kernel):
    from paper_1906_09108_amd import kernels as K
    TK.test_conv_wgrad(case)
    assert K.fdgk_last_kernel() == kernel


# One round of 128-pixel tiles, and one more tile than that: tiles of 256 pixels, which leave half the chip idle
@pytest.mark.parametrize("case, kernel", [
    ((128, 8, 8, 128, 512, 3, 1), "conv_patch_kernel<128, 160, 5>"),
    ((257, 8, 8, 64, 256, 3, 1), "conv_patch256_kernel<128, 320, 3>"),
    ((33, 31, 32, 136, 136, 3, 1), "conv_patch256_kernel<128, 384, 3, true>"),
])
def test_tiles_of_256_pixels(case, kernel):
    from paper_1906_09108_amd import kernels as K
    TK.test_conv_fwd(case)
    assert K.fdgk_last_kernel() == kernel
    TK.test_conv_dgrad(case)


# Weight gradients of 160 output channels on blocks of 128 columns of the (tap, channel) axis: columns that fill whole tiles and not, a
# unit's tap changing within a tile, strides, 1x1, images narrower than a chunk, fewer chunks than stages, chunks in odd and even
# number; without scratch (test_conv_wgrad runs both) and outside the rule the kernels that ran before
@pytest.mark.parametrize("case, kernel", [
    ((1, 8, 8, 160, 160, 3, 1), "conv_wgrad_tall_kernel<4, columns>"),
    ((7, 16, 16, 160, 160, 3, 1), "conv_wgrad_tall_kernel<4, columns>"),
    ((5, 32, 32, 160, 160, 3, 1), "conv_wgrad_tall_kernel<4, columns>"),
    ((64, 16, 16, 24, 160, 3, 1), "conv_wgrad_tall_kernel<4, columns>"),
    ((4, 32, 32, 160, 320, 3, 2), "conv_wgrad_tall_kernel<4, columns>"),
    ((8, 16, 16, 160, 320, 1, 2), "conv_wgrad_tall_kernel<4, columns>"),
    ((512, 4, 8, 16, 160, 3, 1), "conv_wgrad_tall_kernel<4, columns>"),
    ((511, 4, 8, 16, 160, 3, 1), "conv_wgrad_kernel<128, 32, 4, 1, 1>"),      # 16 channels over fewer than 16384 pixels
    ((21, 28, 28, 16, 160, 3, 1), "conv_wgrad_tall_kernel<4, columns, flat>"),   # pixels that fill no whole chunk
    ((60, 15, 22, 40, 160, 3, 1), "conv_wgrad_kernel<128, 128, 2, 2, 1>"),       # the validity of a pixel repeats too late
    ((301, 7, 9, 40, 320, 3, 1), "conv_wgrad_tall_kernel<4, columns, flat>"),
    ((342, 48, 1, 16, 160, 3, 1), "conv_wgrad_tall_kernel<4, columns, flat>"),   # rows of one pixel
    ((2, 64, 64, 160, 160, 3, 1), "conv_wgrad_dma_kernel<3>"),               # rows longer than a chunk
    ((4, 32, 32, 8, 160, 3, 1), "conv_wgrad_kernel<128, 32, 4, 1, 1>"),      # fewer than 16 channels
])
def test_weight_gradients_over_columns(case, kernel):
    from paper_1906_09108_amd import kernels as K
    n, h, w, ci, co, k, s = case
    TK.test_conv_wgrad(case)
    import torch as t
    z = [t.zeros(c, device="cuda", dtype=t.bfloat16) for c in (n * h * w * ci, n * ((h - 1) // s + 1) * ((w - 1) // s + 1) * co)]
    dw, scratch = t.empty(co * k * k * ci, device="cuda"), t.empty(K.fdgk_conv_wgrad_scratch_bytes(n, h, w, ci, co, k, s) // 4, device="cuda")
    K.fdgk_conv_wgrad(*z, dw, scratch, n, h, w, ci, co, k, s, overwrite=True)
    assert K.fdgk_last_kernel() == kernel


# Scratch for the splits of a weight gradient is optional.  The kernels that took layers over from the generic one run them only with
# room for their splits (one tile after the other took up to twenty times as long, in sums as many times longer); a byte too few
# counts as none, a layer of one split needs none
@pytest.mark.parametrize("case, without, within", [
    ((8, 32, 32, 64, 128, 3, 2), "conv_wgrad_kernel<128, 128, 2, 2, 1>", "conv_wgrad128w8_kernel<5, paired>"),
    ((8, 16, 16, 64, 256, 3, 1), "conv_wgrad_kernel<128, 128, 2, 2, 1>", "conv_wgrad128w8_kernel<5, paired>"),
    ((21, 14, 14, 136, 160, 3, 1), "conv_wgrad_kernel<128, 128, 2, 2, 1>", "conv_wgrad128w8_kernel<5, flat, ragged>"),
    ((8, 28, 28, 192, 160, 1, 1), "conv_wgrad_kernel<128, 128, two sums>", "conv_wgrad128w8_kernel<5, flat, ragged>"),
    ((8, 16, 16, 64, 384, 1, 1), "conv_wgrad_kernel<128, 128, two sums>", "conv_wgrad128w8_kernel<5, flat, ragged>"),
    ((3, 7, 7, 128, 256, 3, 1), "conv_wgrad128w8_kernel<5, flat, ragged>", "conv_wgrad128w8_kernel<5, flat, ragged>"),
])
def test_weight_gradients_without_room_for_their_splits(case, without, within):
    from paper_1906_09108_amd import kernels as K
    import torch as t
    n, h, w, ci, co, k, s = case
    TK.test_conv_wgrad(case)
    z = [t.zeros(c, device="cuda", dtype=t.bfloat16) for c in (n * h * w * ci, n * ((h - 1) // s + 1) * ((w - 1) // s + 1) * co)]
    dw, room = t.empty(co * k * k * ci, device="cuda"), K.fdgk_conv_wgrad_scratch_bytes(n, h, w, ci, co, k, s) // 4
    for scratch, kernel in ((None, without), (t.empty(co * k * k * ci - 1, device="cuda"), without), (t.empty(room, device="cuda"), within)):
        K.fdgk_conv_wgrad(*z, dw, scratch, n, h, w, ci, co, k, s, overwrite=True)
        assert K.fdgk_last_kernel() == kernel


# The validity of a pixel under a tap repeats after a number of chunks: workgroups with fewer chunks than that, with exactly as many
# and with several times as many
@pytest.mark.parametrize("case", [(9, 6, 6, 512, 512, 3, 1), (16, 6, 6, 512, 512, 3, 1), (37, 6, 6, 512, 512, 3, 1), (24, 6, 12, 640, 512, 3, 1)])
def test_weight_gradients_whose_pixels_repeat(case):
    from paper_1906_09108_amd import kernels as K
    TK.test_conv_wgrad(case)
    assert K.fdgk_last_kernel().startswith("conv_wgrad128w8_kernel<5, flat")


# Kernels that took layers over from the generic one split their pixels less, and no sum is to lose digits to that: the error against
# 64 bits is no larger than the generic kernel's on the same operands.  Those were measured once and are the bounds: workgroups of
# two to five chunks, of more than a fold each, parts added up one after the other and in pairs; the ragged, thin and paired forms
def check_weight_gradient_against_64_bits(case, bound, kernel):
    from paper_1906_09108_amd import kernels as K
    import torch as t
    n, h, w, ci, co, k, s = case
    ho, wo = (h - 1) // s + 1, (w - 1) // s + 1
    g = t.Generator(device="cuda")
    g.manual_seed(11)
    x = t.randn(n, h, w, ci, generator=g, device="cuda").relu().bfloat16()
    dy = t.randn(n * ho * wo, co, generator=g, device="cuda").bfloat16()
    scratch = t.empty(K.fdgk_conv_wgrad_scratch_bytes(*case) // 4, device="cuda")
    dw = t.empty(co, k, k, ci, device="cuda")
    K.fdgk_conv_wgrad(x, dy, dw, scratch, *case, overwrite=True)
    ran = K.fdgk_last_kernel()
    xp, dyt = t.nn.functional.pad(x, (0, 0, k // 2, k // 2, k // 2, k // 2)).double(), dy.double().t().contiguous()
    num = den = 0.0
    for r in range(k):
        for q in range(k):
            ref = dyt @ xp[:, r:r + (ho - 1) * s + 1:s, q:q + (wo - 1) * s + 1:s].reshape(n * ho * wo, ci)
            num, den = num + float((dw[:, r, q].double() - ref).square().sum()), den + float(ref.square().sum())
    err = (num / den) ** 0.5
    print(f"weight gradient {case}: {err:.3e} (bound {bound:.3e}) {ran}", flush=True)
    assert ran == kernel and err <= bound


@pytest.mark.parametrize("case, bound", [
    ((2, 7, 7, 512, 512, 3, 1), 3.45e-8), ((5, 7, 7, 320, 320, 3, 1), 4.77e-8), ((5, 7, 7, 256, 1024, 1, 1), 5.07e-8), ((37, 14, 14, 128, 512, 1, 1), 9.88e-8),
    ((19, 14, 14, 512, 512, 3, 1), 1.063e-7), ((128, 8, 8, 96, 576, 1, 1), 9.57e-8), ((5, 26, 37, 64, 320, 1, 1), 9.52e-8), ((16, 14, 14, 384, 64, 1, 1), 9.43e-8),
    ((128, 32, 32, 96, 480, 1, 1), 1.382e-7),
])
def test_ragged_weight_gradients_against_64_bits(case, bound):
    check_weight_gradient_against_64_bits(case, bound, "conv_wgrad128w8_kernel<5, flat, ragged>")


@pytest.mark.parametrize("case, bound", [((4, 16, 16, 64, 256, 3, 2), 4.97e-8), ((9, 64, 64, 64, 128, 3, 2), 1.034e-7), ((64, 16, 16, 64, 128, 3, 1), 1.072e-7)])
def test_paired_weight_gradients_against_64_bits(case, bound):
    check_weight_gradient_against_64_bits(case, bound, "conv_wgrad128w8_kernel<5, paired>")


# Blocks of 128 columns hold a sum as long as its split: by rows and flat, splits of four chunks, one round of workgroups and two
@pytest.mark.parametrize("case, bound, form", [
    ((4, 16, 16, 136, 160, 3, 2), 5.02e-8, "columns"), ((4, 16, 16, 192, 480, 3, 2), 4.93e-8, "columns"),
    ((64, 32, 32, 96, 640, 3, 1), 2.73e-7, "columns"), ((64, 32, 32, 120, 160, 3, 1), 1.73e-7, "columns"),
    ((64, 28, 28, 104, 320, 3, 1), 1.82e-7, "columns, flat"), ((128, 24, 24, 16, 160, 3, 1), 1.83e-7, "columns, flat"),
])
def test_weight_gradients_over_columns_against_64_bits(case, bound, form):
    check_weight_gradient_against_64_bits(case, bound, f"conv_wgrad_tall_kernel<4, {form}>")


# The output stages that gate by a ReLU6 and take the sums of the batch-norm backward behind it, with about a third of the gate shut
# from below, a third clamped at 6 and values just below 6: the gradient is zero where the activation is clamped, and only there
def relu6_operands(shape, r):
    z = r.standard_normal(shape).astype(np.float32) * 7 + 3
    gate = TK.bf16_round(np.clip(z, 0, 6))
    gate[gate == 6] = np.where(r.random(int((gate == 6).sum())) < 0.1, np.float32(5.96875), np.float32(6))   # the bf16 below 6
    bnx = TK.bf16_round(r.standard_normal(shape) * (0.5 + r.random((1, shape[1], 1, 1))) + r.standard_normal((1, shape[1], 1, 1)))
    shut, clamped = gate == 0, gate == 6
    assert shut.mean() > 0.2 and clamped.mean() > 0.2 and (gate == 5.96875).any()
    return gate, bnx, shut | clamped


def check_gated_with_sums(dx32, ref, closed, bnx, sums, c):
    from paper_1906_09108_amd import kernels as K
    import torch as t
    got = TK.nhwc_to_nchw(dx32)
    assert TK.rel(got, ref * ~closed) <= TK.F32_TOL
    assert np.all(got[closed] == 0) and np.mean(got[~closed] != 0) > 0.99
    g, x = dx32.to(t.float64).reshape(-1, c).cpu().numpy(), bnx.transpose(0, 2, 3, 1).reshape(-1, c).astype(np.float64)
    total = K.fdgk_sums_read(sums, c)
    assert TK.rel(total[:c], g.sum(0)) <= 1e-5 and TK.rel(total[c:], (g * x).sum(0)) <= 1e-5


# every instantiation: 64 and a partly filled block of 72 channels into 128 and more, 128 and more into up to 64 and up to 96; ragged
# pixels, several tiles; with and without an addend
@pytest.mark.parametrize("case, kernel", [
    ((3, 7, 9, 200, 64, 1, 1), "conv_gather_dma_pair_kernel<128, 2, feeding>"), ((5, 16, 16, 384, 72, 1, 1), "conv_gather_dma_pair_kernel<128, 2, feeding>"),
    ((2, 13, 11, 64, 384, 1, 1), "conv_gather_dma_pair_kernel<64, 3, feeding>"), ((4, 9, 12, 40, 128, 1, 1), "conv_gather_dma_pair_kernel<64, 3, feeding>"),
    ((3, 10, 13, 96, 576, 1, 1), "conv_gather_dma_pair_kernel<96, 4, feeding>"), ((1, 5, 5, 72, 192, 1, 1), "conv_gather_dma_pair_kernel<96, 4, feeding>"),
])
def test_data_gradient_behind_a_relu6(case, kernel):
    from paper_1906_09108_amd import kernels as K
    import torch as t
    n, h, w, ci, co, k, s = case
    print("dgrad behind a ReLU6", case, flush=True)
    x, wt, dy, ho, wo = TK._conv_data(case, 31)
    r = np.random.default_rng(32)
    gate, bnx, closed = relu6_operands(x.shape, r)
    ref = TK.K32.conv_bwd_data(dy, wt, x.shape, 1, 0).astype(np.float64)
    add = r.standard_normal(ref.shape).astype(np.float32) * 0.5
    dyd, wtd = TK.to_dev_nhwc_b16(dy), t.from_numpy(wt.transpose(1, 2, 3, 0).copy()).to(t.bfloat16).contiguous().cuda()
    for addend, gated, hi in ((None, True, 6.0), (add, True, 6.0), (add, True, 0.0), (add, False, 0.0)):
        sums, dx32 = K.new_sums(ci), t.full((n, h, w, ci), float("nan"), device="cuda")
        K.fdgk_conv_dgrad_with_sums(dyd, wtd, None if addend is None else TK.to_dev_nhwc_f32(addend), TK.to_dev_nhwc_b16(gate) if gated else None,
                                    hi, TK.to_dev_nhwc_b16(bnx), sums, dx32, None, n, h, w, ci, co)
        assert K.fdgk_last_kernel() == kernel
        shut = closed if hi else (gate <= 0) & gated     # no upper end: only what is not positive
        check_gated_with_sums(dx32, ref + (0 if addend is None else addend), shut, bnx, sums, ci)


@pytest.mark.parametrize("case", [(3, 9, 11, 72, 1), (2, 16, 16, 192, 1), (1, 1, 1, 8, 1), (3, 9, 11, 72, 2), (2, 16, 16, 192, 2), (40, 31, 30, 64, 1)])
def test_depthwise_kernels_with_sums(case):
    from paper_1906_09108_amd import kernels as K
    import torch as t
    n, h, w, c, s = case
    print("depthwise with sums", case, flush=True)
    ho, wo = (h - 1) // s + 1, (w - 1) // s + 1
    r = np.random.default_rng(33)
    x, dy = (TK.bf16_round(r.standard_normal(sh).astype(np.float32)) for sh in ((n, c, h, w), (n, c, ho, wo)))
    wgt = TK.bf16_round((r.standard_normal((c, 1, 3, 3)) * np.sqrt(2.0 / 9)).astype(np.float32))
    wt = t.from_numpy(np.ascontiguousarray(wgt.reshape(c, 9).T)).to(t.bfloat16).cuda()
    y, plain = (t.empty((n, ho, wo, c), dtype=t.bfloat16, device="cuda") for _ in range(2))
    sums = K.new_sums(c)
    K.fdgk_dwconv3_fwd(TK.to_dev_nhwc_b16(x), wt, plain, n, h, w, c, s)
    K.fdgk_dwconv3_fwd_sums(TK.to_dev_nhwc_b16(x), wt, y, sums, n, h, w, c, s)
    assert t.equal(y, plain)
    yd, total = y.to(t.float64).reshape(-1, c).cpu().numpy(), K.fdgk_sums_read(sums, c)
    assert TK.rel(total[:c], yd.sum(0)) <= 1e-5 and TK.rel(total[c:], (yd * yd).sum(0)) <= 1e-5
    if x.size < 100:     # too few cells for a share of them to be clamped
        return
    gate, bnx, closed = relu6_operands(x.shape, r)
    dx, sums = t.full((n, h, w, c), float("nan"), device="cuda"), K.new_sums(c)
    K.fdgk_dwconv3_dgrad_sums(TK.to_dev_nhwc_b16(dy), wt, TK.to_dev_nhwc_b16(gate), 6.0, TK.to_dev_nhwc_b16(bnx), dx, sums, n, h, w, c, s)
    check_gated_with_sums(dx, TK.K32.dwconv_bwd_data(dy, wgt, x.shape, s, 1).astype(np.float64), closed, bnx, sums, c)


def clamped_params(spec, theta):
    """theta with the batch norms of the expanded tensors at 4 x + 3: about a fifth of the ReLU6 outputs is 0 and a fifth 6."""
    theta, expanded, at = theta.copy(), {6 * L.c_in for L in spec.layers}, 0
    for _, shape, role in W.param_shapes(spec):
        if role in ("gamma", "beta") and shape[0] in expanded:
            theta[at:at + shape[0]] = 4 if role == "gamma" else 3
        at += int(np.prod(shape))
    return theta


# Two inverted blocks whose batch norms push a good part of their ReLU6 outputs to the clamp, layer by layer
@pytest.mark.parametrize("stride", [1, 2])
def test_inverted_blocks_at_the_clamp(stride, monkeypatch):
    layers = [Layer(W.INVERTED_RESIDUAL, 64, 64, 1), Layer(W.INVERTED_RESIDUAL, 64, 96, stride)]
    spec = ModuleSpec(3, 64, 12, 13, layers, delay=1, is_bottom=False, beta=0.5, name="clamped", **TD.H)
    make = W.make_params
    monkeypatch.setattr(W, "make_params", lambda sp, seed, **kw: clamped_params(sp, make(sp, seed, **kw)))
    LT._judge(LT._run(spec, seed=1, steps_after_warmup=2), f"clamped stride {stride}")


# The second sum of a batch-norm backward, sum g (x - mean), against 64 bits, with batch means of up to 64 standard deviations: from the
# launches that take it where the gradient is made, given the forward sums.  The pass of its own that they replace is off by 1.2e-7 ..
# 1.6e-7 at these sizes, whatever the mean; sums of g x from which mean * sum g is subtracted later by 1.5e-7, 5e-7, 2e-6 and 1e-5 at means
# of 1, 4, 16 and 64
BIASED = {
    "depthwise": ((32, 16, 16, 192), lambda K, r, x, gt, st, dx, b: K.fdgk_dwconv3_dgrad_sums(
        r(32, 16, 16, 192), r(9, 192), gt, 6.0, x, dx, st, 32, 16, 16, 192, 1, bnx_sums=b)),
    "depthwise stride 2": ((32, 16, 16, 72), lambda K, r, x, gt, st, dx, b: K.fdgk_dwconv3_dgrad_sums(
        r(32, 8, 8, 72), r(9, 72), gt, 6.0, x, dx, st, 32, 16, 16, 72, 2, bnx_sums=b)),
    "1x1 up": ((32, 16, 16, 384), lambda K, r, x, gt, st, dx, b: K.fdgk_conv_dgrad_with_sums(
        r(32, 16, 16, 64), r(384, 64), None, gt, 6.0, x, st, dx, None, 32, 16, 16, 384, 64, bnx_sums=b)),
    "1x1 to 64": ((32, 16, 16, 64), lambda K, r, x, gt, st, dx, b: K.fdgk_conv_dgrad_with_sums(
        r(32, 16, 16, 384), r(64, 384), None, None, 0.0, x, st, dx, None, 32, 16, 16, 64, 384, bnx_sums=b)),
    "1x1 to 96": ((32, 16, 16, 96), lambda K, r, x, gt, st, dx, b: K.fdgk_conv_dgrad_with_sums(
        r(32, 16, 16, 576), r(96, 576), None, None, 0.0, x, st, dx, None, 32, 16, 16, 96, 576, bnx_sums=b)),
    "pair": ((32, 32, 32, 64), lambda K, r, x, gt, st, dx, b: K.fdgk_conv_dgrad_thin_pair(
        r(32, 16, 16, 128), r(64, 9, 128), r(32, 16, 16, 128), r(64, 128), gt, x, st, dx, None, 32, 32, 32, 64, 128, bnx_sums=b)),
    "pair to 96": ((32, 16, 16, 96), lambda K, r, x, gt, st, dx, b: K.fdgk_conv_dgrad_thin_pair(
        r(32, 8, 8, 192), r(96, 9, 192), r(32, 8, 8, 192), r(96, 192), gt, x, st, dx, None, 32, 16, 16, 96, 192, bnx_sums=b)),
}


@pytest.mark.parametrize("mean", [0.0, 4.0, 64.0])
@pytest.mark.parametrize("name", sorted(BIASED))
def test_batch_norm_sums_around_the_mean(name, mean):
    from paper_1906_09108_amd import kernels as K
    import torch as t
    shape, launch = BIASED[name]
    c, m = shape[3], shape[0] * shape[1] * shape[2]
    g = t.Generator(device="cuda")
    g.manual_seed(5)
    r = lambda *sh: t.randn(*sh, generator=g, device="cuda").bfloat16()
    x = (t.randn(*shape, generator=g, device="cuda") + mean).bfloat16()
    gate = (t.randn(*shape, generator=g, device="cuda") * 3 + 2).clamp(0, 6).bfloat16()
    forward, sums, dx = K.new_sums(c), K.new_sums(c), t.empty(*shape, device="cuda")
    K.fdgk_bn_stats(x, forward, m, c)
    launch(K, r, x, gate, sums, dx, forward)
    batch_mean = t.from_numpy(K.fdgk_sums_read(forward, c)[:c] / m).cuda()
    ref = (dx.double().reshape(m, c) * (x.double().reshape(m, c) - batch_mean)).sum(0)
    total = t.from_numpy(K.fdgk_sums_read(sums, c)).cuda()
    err = float((total[c:] - batch_mean * total[:c] - ref).norm() / ref.norm())
    print(f"{name}, mean {mean}: {err:.2e}", flush=True)
    assert err <= 1.6e-7


# The same through a module: the lower block's last batch norm, whose sums the block above takes.  Its input has means of up to a hundred
# standard deviations (the depthwise convolution's batch norm at 0.05 x + 3); what is left is fp32 rounding of the gradient itself
def test_scale_gradient_of_a_biased_batch_norm():
    from paper_1906_09108_amd import FdgModule
    import torch as t
    spec = ModuleSpec(8, 64, 16, 16, [Layer(W.INVERTED_RESIDUAL, 64, 64, 1)] * 2, delay=0, is_bottom=False, beta=0.5, name="biased", **TD.H)
    theta, at, where, seen = W.make_params(spec, 0), 0, {}, 0
    for name, shape, role in W.param_shapes(spec):
        if role == "gamma":
            where[seen], seen = at, seen + 1
        if role in ("gamma", "beta") and seen == 2:
            theta[at:at + shape[0]] = 0.05 if role == "gamma" else 3
        at += int(np.prod(shape))
    m = FdgModule(spec)
    m.set_params(theta)
    m.trace_attach()
    m.forward(t.from_numpy(W.make_input(spec, 0, 0)).cuda())
    m.backward_delayed(t.from_numpy(W.make_grad_out(spec, 0, 0)).cuda(), t.empty(spec.input_shape(), device="cuda"))
    g, x = m.trace_read(1, 1)[0].astype(np.float64), m.saved_read(0, 0, LW.BN_INPUT[W.INVERTED_RESIDUAL]["bn3"]).astype(np.float64)
    got = m.get_grads()[where[2]:where[2] + 64]
    m.close()
    mean, std = x.mean((0, 2, 3), keepdims=True), np.sqrt(x.var((0, 2, 3), keepdims=True) + TD.H["bn_eps"])
    assert np.median(np.abs(mean) / std) > 10
    ref = (g * (x - mean) / std).sum((0, 2, 3))
    err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    print(f"scale gradient: {err:.2e}", flush=True)
    assert err <= 1e-6


# The two data gradients of a projecting block of 40 .. 96 channels in one launch: gated, with the sums of the fp32 values, and plain
@pytest.mark.parametrize("case", [(3, 9, 11, 64, 128), (4, 16, 14, 64, 64), (2, 7, 2, 72, 128), (5, 8, 8, 96, 192), (2, 5, 6, 40, 192)])
def test_data_gradients_of_a_thin_projecting_block(case):
    from paper_1906_09108_amd import kernels as K
    import torch as t
    n, h, w, ci, co = case
    print("thin pair", case, flush=True)
    x, wt, dy, ho, wo = TK._conv_data((n, h, w, ci, co, 3, 2), 41)
    _, wt2, dy2, _, _ = TK._conv_data((n, h, w, ci, co, 1, 2), 42)
    r = np.random.default_rng(43)
    ref = (TK.K32.conv_bwd_data(dy, wt, x.shape, 2, 1).astype(np.float64) + TK.K32.conv_bwd_data(dy2, wt2, x.shape, 2, 0).astype(np.float64))
    gate = TK.bf16_round(np.maximum(r.standard_normal(ref.shape), 0))
    bnx = TK.bf16_round(r.standard_normal(ref.shape) + 3 * r.standard_normal((1, ci, 1, 1)))
    w1, w2 = (t.from_numpy(a.transpose(1, 2, 3, 0).copy()).to(t.bfloat16).contiguous().cuda() for a in (wt, wt2))
    xd, forward = TK.to_dev_nhwc_b16(bnx), K.new_sums(ci)
    K.fdgk_bn_stats(xd, forward, n * h * w, ci)
    for bnx_sums in (None, forward):
        sums, dx32, dx16 = K.new_sums(ci), t.full((n, h, w, ci), float("nan"), device="cuda"), t.zeros((n, h, w, ci), device="cuda", dtype=t.bfloat16)
        K.fdgk_conv_dgrad_thin_pair(TK.to_dev_nhwc_b16(dy), w1, TK.to_dev_nhwc_b16(dy2), w2, TK.to_dev_nhwc_b16(gate), xd, sums, dx32, dx16,
                                    n, h, w, ci, co, bnx_sums=bnx_sums)
        check_gated_with_sums(dx32, ref, gate <= 0, bnx, sums, ci)
        assert TK.rel(TK.nhwc_to_nchw(dx16), ref * (gate > 0)) <= TK.B16_TOL
    K.fdgk_conv_dgrad_thin_pair(TK.to_dev_nhwc_b16(dy), w1, TK.to_dev_nhwc_b16(dy2), w2, None, None, None, dx32, None, n, h, w, ci, co)
    assert TK.rel(TK.nhwc_to_nchw(dx32), ref) <= TK.F32_TOL


# A projecting block takes the sums of the layer below where that layer reads them in a pass of its own: a stem, a block of channels
# that the narrow kernels do not run, 64 channels over many pixels; not where they would send it to a slower kernel
@pytest.mark.parametrize("below, c, n, h, w, feeds", [
    ([], 64, 2, 10, 12, True), ([Layer(W.BASIC_POSTACT, 96, 96, 1)], 96, 2, 6, 7, True), ([Layer(W.BASIC_POSTACT, 64, 64, 1)], 64, 3, 9, 11, False),
    ([Layer(W.BASIC_POSTACT, 64, 64, 1)], 64, 33, 64, 64, True),
])
def test_what_a_projecting_block_feeds(below, c, n, h, w, feeds):
    from paper_1906_09108_amd import FdgModule
    import torch as t
    layers = ([] if below else [Layer(W.STEM, 3, c, 1)]) + below + [Layer(W.BASIC_POSTACT, c, 2 * c, 2)]
    spec = ModuleSpec(n, layers[0].c_in, h, w, layers, delay=0, is_bottom=not below, beta=0.5, name="feeds", **TD.H)
    if n * h * w < 1000:
        TD.check(f"projecting above {len(below)} {c}", spec)
    m = FdgModule(spec)
    m.set_params(W.make_params(spec, 0))
    m.trace_attach()
    m.forward(t.randn(*spec.input_shape(), device="cuda"))
    m.backward_delayed(t.randn(*spec.output_shape(), device="cuda"), None if spec.is_bottom else t.empty(spec.input_shape(), device="cuda"))
    t.cuda.synchronize()
    assert m.trace_read(1, 1)[1] == feeds
    m.close()

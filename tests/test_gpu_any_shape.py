"""Kernels for shapes outside the fixed tables: image sizes and channel
counts of any kind, single layers against the oracle (2e-2 max-rel in bf16,
1e-4 in fp32, as every single-layer run), at the sizes where a tile, a strip
or a chunk ends."""
import numpy as np
import pytest
import torch

import paper_2004_09910_amd as tgp
from gpu_util import (check_network, check_stage, gpu_network, gpu_stage, oracle_network,
                      oracle_stage, say)
from paper_2004_09910_amd.harness import Session
from workloads import specs
from workloads.specs import (BF16, CONV1X1, CONV3X3, DWCONV3X3, FP32, PRO_MAXPOOL2, Layer,
                             Net)
from workloads.synth import EXACT, NORMAL

pytestmark = pytest.mark.gpu


def one_layer(L, h, w):
    return Net("one", (L,), L.cin, h, w)


def run_and_check(L, h, w, dtype, B, m, what, **kw):
    say(what)
    net = one_layer(L, h, w)
    got = gpu_stage(net, dtype, B, m, 0, (1,), 1, **kw)
    ref = oracle_stage(net, dtype, 0, 1, got["xv"], got["G"])
    check_stage(got, ref, dtype, what, NORMAL)
    got["sess"].close()
    return got


@pytest.mark.parametrize("cin,cout,h,w,B,m", [
    (8, 8, 1, 1, 1, 1),          # one pixel, half a 16-channel chunk
    (24, 40, 17, 33, 4, 2),      # a last chunk of 8 channels, ragged units
    (72, 136, 13, 9, 2, 1),      # past one 64-channel item and one 128-channel tile
    (16, 8, 3, 130, 2, 2),       # column strips
    (40, 64, 2, 600, 1, 1),      # many strips, two rows
    (64, 64, 57, 56, 4, 2),      # 64-multiples at a width of no table
    (64, 192, 40, 61, 14, 2),    # the rectangular-stage weight gradient, odd units
    (264, 16, 7, 7, 2, 2),       # many chunks, few pixels
    (64, 72, 27, 8, 64, 1),      # a full slot of 27 one-unit rows in the weight gradient
])
def test_conv3x3_any_shape(cin, cout, h, w, B, m):
    run_and_check(Layer(CONV3X3, cin, cout), h, w, BF16, B, m,
                  f"conv3x3 {cin}->{cout} @{h}x{w} B={B} m={m}")


@pytest.mark.parametrize("cfg", range(7))
def test_conv3x3_tile_configurations(cfg):
    """Each configuration of the rectangular-tile kernel, forced, with ragged
    tiles on both sides; all sum in one order, so their bits agree."""
    net = one_layer(Layer(CONV3X3, 40, 72), 21, 37)
    base = gpu_stage(net, BF16, 2, 1, 0, (1,), 1)
    tgp.debug_set_fwd_variant(501 + cfg)
    try:
        got = run_and_check(Layer(CONV3X3, 40, 72), 21, 37, BF16, 2, 1, f"tile cfg {cfg}")
    finally:
        tgp.debug_set_fwd_variant(0)
    assert torch.equal(got["y"], base["y"]) and torch.equal(got["dx"], base["dx"])


def test_conv3x3_any_shape_groups_are_bitwise():
    """A group of nine micro-batches (launches of eight and one) gives the
    bits of one micro-batch per launch."""
    net = one_layer(Layer(CONV3X3, 48, 80), 19, 23)
    one = gpu_stage(net, BF16, 9, 9, 0, (1,), 1)
    grp = gpu_stage(net, BF16, 9, 9, 0, (1,), 1, lanes=9, group=9, serial=True)
    assert torch.equal(one["y"], grp["y"]) and torch.equal(one["dx"], grp["dx"])
    for a, b in zip(one["grads"][0], grp["grads"][0]):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("h,w", [(45, 61), (10, 20), (7, 33)])
def test_wgrad_padding_keeps_infinities_apart(h, w):
    """Input pixels of the last row and column pair with no output at filter
    row 0 / column 0: an infinity there must not reach those taps through the
    zero padding (the per-tap kernel; the rectangular stages below)."""
    net = one_layer(Layer(CONV3X3, 64, 128, relu=False), h, w)
    sess = Session(net, BF16)
    sess.plan(3, 1, specs.CKPT_NEVER)
    torch.manual_seed(3)
    x = torch.randn(3, h, w, 64, device="cuda").bfloat16()
    dy = torch.randn(3, h, w, 128, device="cuda").bfloat16()
    y = torch.empty_like(dy)
    out = []
    for v in (0.0, float("inf")):
        x[:, -1, :, 5] = v
        x[:, :, -1, 5] = v
        sess.stage_step(1, x, y, dy, None, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        out.append(sess.params[0]["dw"].clone())          # cout, kh, kw, cin
    assert torch.equal(out[0][:, 0, 0, 5], out[1][:, 0, 0, 5])
    assert torch.equal(out[0][..., :5], out[1][..., :5])
    assert not torch.isfinite(out[1][:, 2, 2, 5]).any()
    sess.close()


def kernels_of(call):
    """Names of the kernels that `call` launches."""
    tgp.profile_enable(True)
    try:
        tgp.profile_read()
        call()
        torch.cuda.synchronize()
        return {k["name"] for k in tgp.profile_read()}
    finally:
        tgp.profile_enable(False)


@pytest.mark.parametrize("cin,cout,h,w,b,name", [
    (24, 16, 6, 4, 10, "conv_gen_wgrad<1,4>"),    # a chain of ten samples
    (72, 40, 5, 17, 3, "conv_gen_wgrad<2,2>"),    # 255 pixels
    (72, 40, 8, 16, 2, "conv_wgrad_tile"),        # two samples
    (72, 40, 8, 8, 4, "conv_wgrad_tile"),         # 256 pixels
    (520, 472, 4, 4, 4, "conv_wgrad_tile"),       # 72 items
    (8, 16, 15, 16, 1, "conv_wgrad_tile"),        # one range: two stages of rows
])
def test_wgrad_of_few_pixels(cin, cout, h, w, b, name):
    """Layers of fewer than 256 pixels, whose weight gradient has one K range:
    both sides of the line, against the oracle."""
    what = f"conv3x3 {cin}->{cout} @{h}x{w}x{b}"
    names = kernels_of(lambda: run_and_check(Layer(CONV3X3, cin, cout), h, w, BF16, b, 1, what))
    assert [n for n in names if "wgrad" in n] == [name], names


@pytest.mark.parametrize("cin,cout,h,w,b,tile", [
    (64, 192, 40, 61, 7, True),
    (64, 192, 40, 61, 6, False),      # few products
    (128, 512, 15, 10, 24, False),    # rows of 10 pixels in units of 8
    (128, 512, 15, 14, 16, True),
])
def test_wgrad_kernel_of_a_shape(cin, cout, h, w, b, tile):
    names = kernels_of(lambda: run_and_check(Layer(CONV3X3, cin, cout), h, w, BF16, 2 * b, 2,
                                             f"wgrad {cin}->{cout} @{h}x{w}x{b}"))
    assert ("conv_wgrad_tile" in names) == tile, names


@pytest.mark.parametrize("cin,cout,h,w,b", [
    (128, 128, 100, 100, 4),     # strips of 24 pixels, the last of 4
    (64, 72, 40, 52, 2),         # of 16, the last of 4; a second channel item of 8
    (48, 48, 86, 86, 2),         # of 32, the last of 22
    (64, 64, 49, 49, 21),        # of 32, the last of 17
    (40, 24, 5, 9, 2),           # two units a row, the second of one pixel
])
def test_wgrad_tile_clears_the_padding_of_every_unit(cin, cout, h, w, b):
    """The rectangular-stage weight gradient: the last column's input pixels
    pair with no output at column tap 0, nor the last row's at row tap 0, so an
    infinity there must not reach those taps, whatever unit of a strip the
    image ends in."""
    net = one_layer(Layer(CONV3X3, cin, cout, relu=False), h, w)
    sess = Session(net, BF16)
    sess.plan(b, 1, specs.CKPT_NEVER)
    torch.manual_seed(3)
    x = torch.randn(b, h, w, cin, device="cuda").bfloat16()
    dy = torch.randn(b, h, w, cout, device="cuda").bfloat16()
    y = torch.empty_like(dy)

    def step(xs):
        names = kernels_of(lambda: sess.stage_step(1, xs, y, dy, None,
                                                   torch.cuda.current_stream().cuda_stream))
        assert "conv_wgrad_tile" in names, names
        return sess.params[0]["dw"].clone()                   # cout, kh, kw, cin

    for edge, tap in ((np.s_[:, :, -1, 5], np.s_[:, :, 0, 5]), (np.s_[:, -1, :, 5], np.s_[:, 0, :, 5])):
        x0, x1 = x.clone(), x.clone()
        x0[edge] = 0.0
        x1[edge] = float("inf")
        d0, d1 = step(x0), step(x1)
        assert torch.equal(d0[tap], d1[tap])
        assert torch.equal(d0[..., :5], d1[..., :5]) and torch.equal(d0[..., 6:], d1[..., 6:])
        assert not torch.isfinite(d1[:, 1, 1, 5]).any()
    sess.close()


@pytest.mark.parametrize("c,h,w,relu,bias", [
    (24, 9, 13, True, True),       # 3 packs: 255 threads, partly filled rows
    (192, 28, 28, True, True),     # 24 packs, several strips and chunks
    (2000, 3, 5, False, True),     # 250 packs: one column a block
    (2056, 3, 5, True, True),      # past 256 packs: the per-element kernels
    (40, 40, 30, False, False),
    (192, 100, 56, True, True),    # past 128 blocks of eight rows
])
def test_depthwise_any_channels(c, h, w, relu, bias):
    run_and_check(Layer(DWCONV3X3, c, c, relu=relu, bias=bias), h, w, BF16, 4, 2,
                  f"depthwise {c} @{h}x{w}")


@pytest.mark.parametrize("dtype,c,h,w", [(BF16, 192, 18, 14), (BF16, 24, 34, 22), (FP32, 12, 10, 6),
                                         (FP32, 100, 40, 30)])
def test_bias_sums_any_channels(dtype, c, h, w):
    """ReLU backward with its bias sums, and its pooled form inside a
    partition, where the channel packs divide no block; exact inputs."""
    cin = 64 if dtype == BF16 else 8
    net = Net("two", (Layer(CONV3X3, cin, c), Layer(CONV3X3, c, 64, prologue=PRO_MAXPOOL2)), cin,
              h, w)
    got = gpu_stage(net, dtype, 4, 2, 0, (2,), 1, family=EXACT)
    ref = oracle_stage(net, dtype, 0, 2, got["xv"], got["G"], family=EXACT, certify=True)
    check_stage(got, ref, dtype, f"bias sums c={c} {h}x{w}", EXACT)
    got["sess"].close()


@pytest.mark.parametrize("dtype,kind,c,h,w", [
    (BF16, CONV1X1, 16, 130, 151),      # two packs: rounds of 128 rows
    (BF16, CONV1X1, 2048, 72, 73),      # one row at a time, past ten
    (FP32, CONV1X1, 1024, 50, 51),      # not past ten
])
def test_bias_sums_of_many_rows(dtype, kind, c, h, w):
    """The block counts of the ReLU backward with its bias sums; exact inputs."""
    net = one_layer(Layer(kind, 8, c), h, w)
    got = gpu_stage(net, dtype, 2, 2, 0, (1,), 1, family=EXACT)
    ref = oracle_stage(net, dtype, 0, 1, got["xv"], got["G"], family=EXACT, certify=True)
    check_stage(got, ref, dtype, f"bias sums c={c} {h}x{w}", EXACT)
    got["sess"].close()


@pytest.mark.parametrize("dtype,cin,c,h,w,pool,at_once", [
    (BF16, 8, 24, 128, 80, False, True),     # room for 8 blocks of 85 rows
    (BF16, 8, 24, 128, 80, True, True),
    (BF16, 8, 24, 100, 110, False, False),   # for 56
    (BF16, 8, 24, 20, 30, False, False),     # few rows a block also with 8
    (BF16, 8, 2000, 4, 6, False, True),      # one row a block at a time, no room
    (FP32, 8, 12, 128, 80, True, True),
])
def test_bias_sums_in_the_slot_or_at_once(dtype, cin, c, h, w, pool, at_once):
    """Bias sums of channels that are no power of two, kept for the accumulation or
    summed in the same pass where the layer's room is too small: exact inputs,
    one micro-batch a launch and a group with the same bits."""
    layers = (Layer(CONV1X1, cin, c),)
    if pool:
        layers += (Layer(CONV1X1, c, 8, prologue=PRO_MAXPOOL2),)
    net = Net("bias", layers, cin, h, w)
    out = []
    names = kernels_of(lambda: out.append(gpu_stage(net, dtype, 4, 2, 0, (len(layers),), 1,
                                                    family=EXACT)))
    one = out[0]
    assert ("pool_relu_backward_bias" if pool else "relu_backward_bias") in names, names
    assert ("reduce_now" in names) == at_once, names
    ref = oracle_stage(net, dtype, 0, len(layers), one["xv"], one["G"], family=EXACT, certify=True)
    check_stage(one, ref, dtype, f"bias sums {cin}->{c} {h}x{w}", EXACT)
    grp = gpu_stage(net, dtype, 4, 2, 0, (len(layers),), 1, lanes=2, group=2, serial=True,
                    family=EXACT)
    for a, b in zip(one["grads"][0], grp["grads"][0]):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("c,h,w", [(192, 14, 14), (64, 9, 7), (48, 11, 5)])
def test_masked_depthwise_gradient_past_the_last_column(c, h, w):
    """Two cells whose depthwise data gradient stores the ReLU backward of the
    1x1 layer below with blocks that end past the image."""
    net = specs.amoeba_cells(2, c, 8)
    net = Net("cells", net.layers, c, h, w)
    got = gpu_stage(net, BF16, 4, 2, 0, (4,), 1, family=EXACT)
    ref = oracle_stage(net, BF16, 0, 4, got["xv"], got["G"], family=EXACT, certify=True)
    check_stage(got, ref, BF16, f"cells c={c} {h}x{w}", EXACT)
    got["sess"].close()


@pytest.mark.parametrize("dtype,kind,cin,cout,h,w,B,m", [
    (FP32, CONV3X3, 1, 1, 1, 1, 1, 1),
    (FP32, CONV3X3, 3, 5, 7, 9, 4, 2),          # K = 27, scalar loads
    (FP32, CONV3X3, 16, 16, 32, 32, 4, 2),      # the K step split over four waves
    (FP32, CONV3X3, 72, 100, 40, 36, 2, 1),     # 64 x 32 and 64 x 64 tiles, ragged channels
    (FP32, CONV3X3, 20, 68, 90, 61, 4, 2),
    (FP32, CONV1X1, 130, 70, 11, 13, 2, 1),
    (FP32, CONV1X1, 8, 24, 100, 90, 2, 2),      # 32 x 128 tiles
    (BF16, CONV3X3, 3, 64, 33, 29, 4, 2),       # an image layer
    (BF16, CONV3X3, 64, 3, 20, 12, 2, 1),
    (BF16, CONV3X3, 5, 7, 9, 11, 2, 2),
    (BF16, CONV3X3, 12, 20, 17, 5, 2, 1),       # multiples of 4, not of 8
    (BF16, CONV1X1, 1, 1, 5, 3, 2, 1),
    (BF16, CONV1X1, 36, 28, 19, 21, 4, 2),
])
def test_float32_matrix_convolutions(dtype, kind, cin, cout, h, w, B, m):
    run_and_check(Layer(kind, cin, cout), h, w, dtype, B, m,
                  f"{'fp32' if dtype == FP32 else 'bf16'} kind {kind} {cin}->{cout} @{h}x{w}")


def test_float32_matrix_convolutions_groups_are_bitwise():
    net = one_layer(Layer(CONV3X3, 12, 36), 19, 23)
    one = gpu_stage(net, FP32, 6, 6, 0, (1,), 1)
    grp = gpu_stage(net, FP32, 6, 6, 0, (1,), 1, lanes=6, group=6, serial=True)
    assert torch.equal(one["y"], grp["y"]) and torch.equal(one["dx"], grp["dx"])
    for a, b in zip(one["grads"][0], grp["grads"][0]):
        np.testing.assert_array_equal(a, b)


def test_slices_reduced_at_once_groups_are_bitwise():
    """A float32 layer whose slices are too many to keep: they are summed after
    the launch, for one micro-batch and for a group.  (No ReLU: among four
    million outputs one lies within float32 rounding of zero.)"""
    layer = Layer(CONV3X3, 128, 128, relu=False)
    one = run_and_check(layer, 122, 120, FP32, 2, 2, "conv3x3 128 @122x120 fp32")
    grp = gpu_stage(one_layer(layer, 122, 120), FP32, 2, 2, 0, (1,), 1, lanes=2, group=2, serial=True)
    assert torch.equal(one["y"], grp["y"]) and torch.equal(one["dx"], grp["dx"])
    for a, b in zip(one["grads"][0], grp["grads"][0]):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("dtype,h,w,B,m", [(BF16, 3, 5, 6, 3), (BF16, 40, 60, 2, 1),
                                           (FP32, 130, 90, 2, 2)])
def test_loss_of_odd_sizes(dtype, h, w, B, m):
    """One-channel outputs whose micro-batch slices are not 16-byte aligned,
    and more elements than one round of the loss's blocks."""
    cin = 64 if dtype == BF16 else 4
    net = one_layer(Layer(CONV1X1, cin, 1, relu=False), h, w)
    got = gpu_network(net, dtype, B, m, 1, 0)
    check_network(got, oracle_network(net, dtype, B), dtype, f"loss {h}x{w} B={B} m={m}")
    got["sess"].close()


@pytest.mark.parametrize("c,h,w,B,m,lanes", [
    (64, 46, 50, 2, 2, 1),        # 72 blocks, the last one ragged
    (128, 97, 96, 2, 2, 2),       # past 512 blocks of 2048: some take a second round
])
def test_loss_of_wide_outputs(c, h, w, B, m, lanes):
    """The loss and its gradient where a micro-batch has many elements, alone
    and in one launch of two."""
    net = one_layer(Layer(CONV1X1, 8, c, relu=False), h, w)
    got = gpu_network(net, BF16, B, m, 1, 0, lanes=lanes)
    check_network(got, oracle_network(net, BF16, B), BF16, f"loss c={c} {h}x{w} B={B} m={m}")
    got["sess"].close()


@pytest.mark.parametrize("cin,cout,h,w,B,m", [
    (8, 8, 1, 1, 1, 1),
    (24, 40, 17, 33, 4, 2),       # one partial stage
    (72, 200, 13, 9, 2, 1),       # a second stage of 8 channels, ragged channel tiles
    (264, 64, 7, 7, 2, 2),        # the deep ring
    (64, 32, 40, 30, 4, 2),       # 32-channel tiles
    (192, 136, 60, 50, 4, 1),     # 128 x 128 tiles
])
def test_conv1x1_any_channels(cin, cout, h, w, B, m):
    run_and_check(Layer(CONV1X1, cin, cout), h, w, BF16, B, m,
                  f"conv1x1 {cin}->{cout} @{h}x{w} B={B} m={m}")


@pytest.mark.parametrize("cfg", range(5))
def test_conv1x1_tile_configurations(cfg):
    """Each tile of the 1x1 kernel, forced, with ragged tiles on both sides;
    the sums run in one order, so their bits agree, in groups too."""
    net = one_layer(Layer(CONV1X1, 72, 136), 11, 17)
    base = gpu_stage(net, BF16, 3, 3, 0, (1,), 1, lanes=3, group=3, serial=True)
    tgp.debug_set_fwd_variant(601 + cfg)
    try:
        got = run_and_check(Layer(CONV1X1, 72, 136), 11, 17, BF16, 3, 3, f"1x1 tile cfg {cfg}")
    finally:
        tgp.debug_set_fwd_variant(0)
    assert torch.equal(got["y"], base["y"]) and torch.equal(got["dx"], base["dx"])


@pytest.mark.parametrize("cin,cout,h,w,B,m", [
    (1, 8, 1, 1, 1, 1),
    (1, 72, 9, 5, 2, 2),          # one block of 16 terms, a second channel tile
    (3, 64, 33, 47, 6, 2),        # two blocks; rows no multiple of a tile
    (4, 24, 130, 70, 2, 1),       # three blocks, two tiles of terms; several ranges
    (7, 136, 31, 3, 15, 3),       # all 63 terms
    (3, 16, 150, 110, 2, 1),      # two items a wave
])
def test_conv3x3_few_input_channels(cin, cout, h, w, B, m):
    run_and_check(Layer(CONV3X3, cin, cout), h, w, BF16, B, m,
                  f"conv3x3 {cin}->{cout} @{h}x{w} B={B} m={m}")


@pytest.mark.parametrize("dt", [BF16, FP32])
@pytest.mark.parametrize("cin,cout,h,w,B,m", [
    (8, 1, 1, 1, 1, 1),
    (64, 1, 29, 31, 6, 2),
    (256, 3, 17, 40, 6, 3),       # bias sums of rows of three
    (16, 4, 70, 66, 4, 1),
    (256, 2, 60, 51, 2, 1),       # data gradient in four pixels a thread
])
def test_conv1x1_few_output_channels(dt, cin, cout, h, w, B, m):
    run_and_check(Layer(CONV1X1, cin, cout, relu=False), h, w, dt, B, m,
                  f"conv1x1 {cin}->{cout} @{h}x{w} B={B} m={m}")


@pytest.mark.parametrize("cin,cout,h,w", [(512, 64, 13, 11), (1024, 192, 5, 7), (2048, 64, 16, 16)])
def test_conv3x3_shares_of_a_long_sum(cin, cout, h, w):
    """Layers of long sums and few pixels, whose sums are split over blocks, and
    their data gradients (sums over 64 and 192: not split): against the oracle,
    and the same bits in a group as one by one."""
    net = one_layer(Layer(CONV3X3, cin, cout), h, w)
    got = run_and_check(Layer(CONV3X3, cin, cout), h, w, BF16, 3, 3, f"conv3x3 {cin}->{cout} @{h}x{w}")
    grp = gpu_stage(net, BF16, 3, 3, 0, (1,), 1, lanes=3, group=3, serial=True)
    assert torch.equal(got["y"], grp["y"]) and torch.equal(got["dx"], grp["dx"])
    back = run_and_check(Layer(CONV3X3, cout, cin), h, w, BF16, 2, 1, f"conv3x3 {cout}->{cin} @{h}x{w}")
    back["sess"].close()


@pytest.mark.parametrize("dtype,kind,cin,cout,h,w", [
    (BF16, CONV3X3, 512, 128, 20, 20),    # shares of the sum
    (BF16, CONV3X3, 1024, 256, 14, 14),
    (BF16, CONV3X3, 128, 128, 48, 48),    # whole rows or rectangles, by the launch
    (BF16, CONV3X3, 64, 192, 45, 61),
    (BF16, CONV3X3, 40, 72, 21, 37),
    (BF16, CONV3X3, 3, 64, 33, 29),
    (BF16, CONV1X1, 256, 256, 28, 28),
    (BF16, CONV1X1, 192, 136, 30, 25),
    (BF16, DWCONV3X3, 192, 192, 14, 14),
    (FP32, CONV3X3, 16, 40, 32, 32),
])
def test_outputs_do_not_depend_on_the_micro_batch_size(dtype, kind, cin, cout, h, w):
    """A sample's output and input gradient have the same bits alone and among
    four samples: the order of every sum is fixed by the per-sample shape."""
    net = one_layer(Layer(kind, cin, cout), h, w)
    one = gpu_stage(net, dtype, 4, 4, 0, (1,), 1)
    four = gpu_stage(net, dtype, 4, 1, 0, (1,), 1)
    assert torch.equal(one["y"], four["y"]) and torch.equal(one["dx"], four["dx"])


def test_conv3x3_small_and_large_launches_agree():
    """The whole-row kernel's widths: a launch of few samples takes the
    rectangular tiles, one of many the whole rows, with the same bits."""
    net = one_layer(Layer(CONV3X3, 64, 64), 96, 96)
    one = gpu_stage(net, BF16, 6, 6, 0, (1,), 1, lanes=6)
    grp = gpu_stage(net, BF16, 6, 6, 0, (1,), 1, lanes=6, group=6, serial=True)
    assert torch.equal(one["y"], grp["y"]) and torch.equal(one["dx"], grp["dx"])


@pytest.mark.parametrize("cin,cout,h,w,split", [
    (768, 64, 10, 10, True),      # four shares of 12 stages
    (512, 192, 5, 9, True),       # two of 16
    (448, 64, 9, 10, False),      # two would have 14
    (2048, 128, 34, 36, True),    # past 1024 pixels: the longest sums only
    (1408, 128, 34, 36, False),
])
def test_conv3x3_where_a_sum_is_split(cin, cout, h, w, split):
    """Both sides of the lines for split sums: against the oracle, one by one and
    as a group of two with the same bits."""
    layer = Layer(CONV3X3, cin, cout)
    what = f"conv3x3 {cin}->{cout} @{h}x{w}"
    out = []
    names = kernels_of(lambda: out.append(run_and_check(layer, h, w, BF16, 2, 2, what)))
    assert any(n.startswith("conv3x3_tile") and n.endswith("4,split>") for n in names) == split, names
    grp = gpu_stage(one_layer(layer, h, w), BF16, 2, 2, 0, (1,), 1, lanes=2, group=2, serial=True)
    assert torch.equal(out[0]["y"], grp["y"]) and torch.equal(out[0]["dx"], grp["dx"])


@pytest.mark.parametrize("c,hw,b,m,lanes,wt", [
    (128, 96, 1, 2, 1, False),   # every launch of the plan is small: the forward weights serve
    (128, 96, 1, 2, 2, False),   # the largest small launch
    (128, 96, 1, 4, 4, True),    # a launch of all four lanes takes the whole rows
    (64, 96, 8, 1, 1, True),
])
def test_transposed_weights_only_where_a_launch_reads_them(c, hw, b, m, lanes, wt):
    net = one_layer(Layer(CONV3X3, c, c), hw, hw)
    what = f"conv3x3 {c} @{hw}x{hw}x{b} m={m}"
    names = kernels_of(lambda: run_and_check(net.layers[0], hw, hw, BF16, b * m, m, what,
                                             lanes=lanes, group=lanes, serial=True))
    assert ("wtransform" in names) == wt, names


@pytest.mark.parametrize("cin,h,w", [(64, 40, 33), (128, 47, 31), (192, 64, 32), (256, 37, 45)])
def test_conv1x1_register_weights(cin, h, w):
    """The 1x1 kernel with its weights in registers, with and without a ragged
    last tile, one micro-batch a launch and a group (several tiles a block):
    each against the oracle and the same bits."""
    one = run_and_check(Layer(CONV1X1, cin, 256), h, w, BF16, 14, 14, f"conv1x1 {cin}->256 one by one")
    grp = run_and_check(Layer(CONV1X1, cin, 256), h, w, BF16, 14, 14, f"conv1x1 {cin}->256 group",
                        lanes=14, group=14, serial=True)
    assert torch.equal(one["y"], grp["y"]) and torch.equal(one["dx"], grp["dx"])


@pytest.mark.parametrize("cin,h,w", [(64, 128, 128), (128, 128, 128), (192, 96, 96), (256, 96, 96),
                                     (64, 127, 129), (256, 97, 95)])
def test_conv1x1_register_weights_long_runs(cin, h, w):
    """Launches of so many tiles that each block's ring reaches its steady state,
    where the wait for a stage counts the stores of the tiles between (whole
    64-pixel tiles), and ragged ones, where it does not: the bits of the tiled
    1x1 kernel, which sums in the same order, and torch's values."""
    m = 16
    sess = Session(one_layer(Layer(CONV1X1, cin, 256), h, w), BF16, init="device")
    sess.plan(m, m, specs.CKPT_NEVER, lanes=m)
    torch.manual_seed(cin)
    x = torch.randn(m, h, w, cin, device="cuda").bfloat16()

    def forward():
        y = torch.zeros(m, h, w, 256, dtype=torch.bfloat16, device="cuda")
        sess.plan(m, m, specs.CKPT_NEVER, lanes=m)
        names = kernels_of(lambda: tgp.stage_forward_n(
            sess.h, 1, 1, [False] * m, [x[i].data_ptr() for i in range(m)],
            [y[i].data_ptr() for i in range(m)], torch.cuda.current_stream().cuda_stream))
        return y, names

    got, names = forward()
    assert names == {"conv1x1_res"}, names
    tgp.debug_set_fwd_variant(601)
    try:
        ref, names = forward()
    finally:
        tgp.debug_set_fwd_variant(0)
    assert all(n.startswith("conv1x1_tile") for n in names), names
    assert torch.equal(got, ref)
    # rounded to bf16: 2^-9 of the value; float32 sums of up to 256 terms of at most
    # about 70 in all: 256 2^-24 70 = 1e-3
    w = sess.params[0]["w"].reshape(256, cin).float()
    want = (x.reshape(-1, cin).float() @ w.t()).relu()
    assert torch.allclose(got.reshape(-1, 256).float(), want, rtol=2.0 ** -8, atol=1e-3)
    sess.close()


@pytest.mark.parametrize("cin,cout,h,w,b,other", [
    (16, 520, 2, 2, 64, 1),       # 9 samples a tile, ragged channels
    (40, 328, 5, 7, 37, 1),       # the last row block ends in a sample
    (520, 24, 1, 8, 40, 1),       # one row a sample; its data gradient in few chunks
    (512, 512, 4, 3, 41, 2),      # split sums
    (24, 640, 8, 8, 30, 1),
])
def test_conv3x3_tiles_across_samples(cin, cout, h, w, b, other):
    """Images of at most 64 pixels: a tile covers several samples with a zero row
    between.  Against the oracle, and bit for bit the one-sample tiles (forced)."""
    layer, net = Layer(CONV3X3, cin, cout), one_layer(Layer(CONV3X3, cin, cout), h, w)
    out = []
    names = kernels_of(lambda: out.append(run_and_check(layer, h, w, BF16, b, 1,
                                                        f"conv3x3 {cin}->{cout} @{h}x{w}x{b}")))
    assert any(",tall" in n for n in names), names
    tgp.debug_set_fwd_variant(501 + other)
    try:
        names = kernels_of(lambda: out.append(gpu_stage(net, BF16, b, 1, 0, (1,), 1)))
    finally:
        tgp.debug_set_fwd_variant(0)
    assert not any(",tall" in n for n in names), names
    assert torch.equal(out[0]["y"], out[1]["y"]) and torch.equal(out[0]["dx"], out[1]["dx"])


@pytest.mark.parametrize("dtype,kind,cin,cout,h,w,b", [
    (BF16, CONV3X3, 40, 72, 21, 37, 2),      # rectangular tiles
    (BF16, CONV3X3, 40, 328, 5, 7, 37),      # tiles across samples
    (BF16, CONV3X3, 512, 64, 10, 10, 2),     # split sums
    (BF16, CONV3X3, 3, 40, 17, 19, 2),       # an image layer
    (BF16, CONV3X3, 12, 20, 17, 5, 2),       # float32 matrix unit
    (FP32, CONV3X3, 20, 68, 17, 13, 2),
    (BF16, CONV1X1, 72, 136, 11, 17, 2),
    (BF16, CONV1X1, 64, 256, 9, 7, 2),       # weights in registers
    (FP32, CONV1X1, 130, 70, 5, 7, 2),
    (BF16, DWCONV3X3, 24, 24, 19, 13, 2),
])
def test_infinities_reach_only_what_they_pair_with(dtype, kind, cin, cout, h, w, b):
    """An infinity in the input (the output gradient) of sample 0, in a corner or
    inside, changes only the outputs (input gradients) of its 3 x 3 neighbourhood
    or, in a 1x1 layer, its pixel."""
    net = one_layer(Layer(kind, cin, cout, relu=False), h, w)
    sess = Session(net, dtype, init="device")
    sess.plan(b, 1, specs.CKPT_NEVER)
    torch.manual_seed(5)
    td = torch.bfloat16 if dtype == BF16 else torch.float32
    x = torch.randn(b, h, w, cin, device="cuda").to(td)
    dy = torch.randn(b, h, w, cout, device="cuda").to(td)

    def step(xs, dys):
        y, dx = torch.empty_like(dy), torch.empty_like(x)
        sess.stage_step(1, xs, y, dys, dx, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        return y, dx

    y0, dx0 = step(x, dy)
    r = 0 if kind == CONV1X1 else 1
    for ph, pw in ((h - 1, w - 1), (0, w // 2), (h // 2, 0)):
        x1, dy1 = x.clone(), dy.clone()
        x1[0, ph, pw, cin - 1] = float("inf")
        dy1[0, ph, pw, cout - 1] = float("inf")
        y1, dx1 = step(x1, dy1)
        for a, c in ((y0, y1), (dx0, dx1)):
            near = torch.zeros(b, h, w, dtype=torch.bool, device="cuda")
            near[0, max(ph - r, 0):ph + r + 1, max(pw - r, 0):pw + r + 1] = True
            assert torch.equal(a[~near], c[~near])
            assert not torch.isfinite(c[0, ph, pw]).all()
    sess.close()


def test_threads_launch_side_by_side():
    """Two networks on two threads and streams, of layers whose launches choose
    among configurations: the bits of one after the other."""
    import threading
    made = []
    for cin, cout, h, w, kind in ((40, 72, 21, 37, CONV3X3), (72, 136, 30, 25, CONV1X1)):
        sess = Session(one_layer(Layer(kind, cin, cout), h, w), BF16, init="device")
        sess.plan(2, 1, specs.CKPT_NEVER)
        x = torch.randn(2, h, w, cin, device="cuda").bfloat16()
        dy = torch.randn(2, h, w, cout, device="cuda").bfloat16()
        made.append((sess, x, dy, torch.empty_like(dy), torch.empty_like(x), torch.cuda.Stream()))
    torch.cuda.synchronize()

    def run(k):
        sess, x, dy, y, dx, st = made[k]
        for _ in range(50):
            sess.stage_step(1, x, y, dy, dx, st.cuda_stream)

    def results():
        torch.cuda.synchronize()
        return [t.clone() for s, _, _, y, dx, _ in made for t in (y, dx, s.params[0]["dw"])]

    run(0)
    run(1)
    alone = results()
    for _, _, _, y, dx, _ in made:
        y.zero_(), dx.zero_()
    torch.cuda.synchronize()
    threads = [threading.Thread(target=run, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for a, b in zip(alone, results()):
        assert torch.equal(a, b)
    for m in made:
        m[0].close()


def test_sums_kept_or_run_at_once_have_the_same_bits():
    """Eight layers whose slices and bias sums fit what the plan of one lane has
    left, but not all of them with two lanes and sixteen micro-batches."""
    net = Net("eight", (Layer(CONV1X1, 656, 656),) * 8, 656, 16, 16)
    one, two = [], []
    alone = kernels_of(lambda: one.append(gpu_stage(net, BF16, 16, 16, 0, (8,), 1)))
    group = kernels_of(lambda: two.append(gpu_stage(net, BF16, 16, 16, 0, (8,), 1, lanes=2, group=2,
                                                    serial=True)))
    assert "reduce_now" not in alone and "reduce_now" in group, (alone, group)
    assert torch.equal(one[0]["y"], two[0]["y"]) and torch.equal(one[0]["dx"], two[0]["dx"])
    for k in one[0]["grads"]:
        for a, b in zip(one[0]["grads"][k], two[0]["grads"][k]):
            np.testing.assert_array_equal(a, b)

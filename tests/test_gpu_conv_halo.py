"""GPU parity of the convolutions that hold their input windows in LDS (bf16) against the oracle:
block shapes, channel counts that are not multiples of 32 or 64, output channels off every vector
width, ragged reduction steps, unpadded and grouped layers, tiles that cross images, whole-image
tiles, padded first layers, data gradients at stride 2; the weight gradients over windows; and
layers that stay on the general kernels."""
import numpy as np
import pytest
import torch

from paper_1704_04560_amd import mtx
from paper_1704_04560_amd import workloads as wl
from tests.test_gpu_train_step import run_case

pytestmark = pytest.mark.gpu

# name: input shape, layers, shards, shard batch, the launches (site, layer, tile rows) expected
CASES = {
    # 16 channels, scalar stores (20 and 18 outputs), 5x5 windows; groups of 24 channels whose 27
    # granules leave a ragged k step
    "narrow": ((3, 41, 53), (wl.conv(16, 3, pad=1, relu=True), wl.conv(20, 5, pad=2, relu=True),
                             wl.conv(48, 1, relu=True), wl.conv(18, 3, pad=1, groups=2, relu=True),
                             wl.maxpool(3, 2), wl.fc(5)),
               3, 8, {("fwd", 1, 32), ("fwd", 3, 32)}),
    # 72 channels, unpadded (the data gradient's windows reach over the whole border), 56 outputs
    "unpadded": ((3, 37, 43), (wl.conv(16, 3, pad=1, relu=True), wl.conv(72, 3, relu=True),
                               wl.conv(56, 3, pad=1, relu=True), wl.maxpool(2, 2), wl.fc(4)),
                 2, 17, {("fwd", 1, None), ("dgrad", 1, None), ("fwd", 2, None), ("dgrad", 2, None)}),
    # 96-row tiles
    "rows96": ((16, 37, 43), (wl.conv(92, 3, relu=True), wl.conv(16, 2), wl.maxpool(3, 3), wl.fc(4)),
               4, 21, {("fwd", 0, 96), ("dgrad", 1, 96)}),
    # 8 x 8 images: every tile crosses images; 2x2 and 7x7 kernels, more padding than the window
    # needs
    "small": ((8, 8, 8), (wl.conv(40, 2, relu=True), wl.conv(32, 7, pad=3, relu=True),
                          wl.conv(48, 3, pad=4), wl.fc(3)), 2, 520,
              {("fwd", 0, 64), ("dgrad", 1, 64), ("fwd", 2, 64), ("dgrad", 2, 32)}),
    # 13 x 13 images, one per block: 192 and 384 rows in eight waves, 192 in four
    "image": ((64, 13, 13), (wl.conv(192, 3, pad=1, relu=True), wl.conv(384, 3, pad=1, groups=2),
                             wl.fc(3)), 2, 200,
              {("fwd", 0, 192), ("fwd", 1, 192), ("dgrad", 1, 96)}),
    # 1x1 data gradients: scalar stores off the fragments, groups
    "pointwise": ((3, 33, 31), (wl.conv(20, 3, pad=1, relu=True), wl.conv(72, 1, relu=True),
                                wl.conv(48, 1, groups=3, relu=True), wl.maxpool(3, 2), wl.fc(3)), 2, 32,
                  {("dgrad", 1, 32), ("dgrad", 2, 32)}),
    # data gradients at stride 2: odd sizes, scalar stores, 2x2, 5x5 and 7x7 kernels, groups, both
    # block shapes
    "stride2": ((3, 33, 30), (wl.conv(24, 3, pad=1, relu=True), wl.conv(64, 3, stride=2, pad=1, relu=True),
                              wl.maxpool(2, 2), wl.fc(3)), 2, 30, {("dgrad", 1, 64)}),
    "stride2g": ((3, 33, 30), (wl.conv(64, 3, pad=1, relu=True),
                               wl.conv(128, 3, stride=2, pad=1, groups=2, relu=True),
                               wl.maxpool(2, 2), wl.fc(3)), 2, 48, {("dgrad", 1, 64)}),
    "stride2k2": ((3, 14, 18), (wl.conv(20, 3, pad=1, relu=True), wl.conv(64, 2, stride=2, relu=True),
                                wl.fc(3)), 2, 120, {("dgrad", 1, 64)}),
    "stride2k5": ((3, 27, 24), (wl.conv(72, 3, pad=1), wl.conv(64, 5, stride=2, pad=2, relu=True),
                                wl.maxpool(2, 2), wl.fc(3)), 2, 40, {("dgrad", 1, 128)}),
    "stride2k7": ((3, 21, 23), (wl.conv(12, 3, pad=1, relu=True), wl.conv(64, 7, stride=2, pad=3, relu=True),
                                wl.maxpool(2, 2), wl.fc(3)), 2, 70, {("dgrad", 1, 64)}),
    # padded first layers: stride 4 with rows past a tile's end, 8-channel pixels, odd channels
    "first": ((3, 51, 47), (wl.conv(70, 11, stride=4, pad=2, relu=True), wl.maxpool(3, 2), wl.fc(4)),
              3, 80, {("fwd", 0, None)}),
    "first3": ((3, 33, 31), (wl.conv(20, 3, pad=1, relu=True), wl.maxpool(3, 2), wl.fc(3)), 2, 60,
               {("fwd", 0, 32)}),
    "first5": ((5, 40, 42), (wl.conv(24, 5, stride=2, relu=True), wl.maxpool(2, 2), wl.fc(3)), 2, 95,
               {("fwd", 0, 32)}),
    "wide": ((64, 13, 13), (wl.conv(256, 3, pad=1, relu=True), wl.conv(384, 3, pad=1), wl.fc(3)), 1,
             200, {("fwd", 1, 384), ("dgrad", 1, 256)}),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_window_convolutions_match_oracle(name):
    shape, layers, R, Nb, expected = CASES[name]
    net = wl.Net("halo-" + name, shape, layers, wl.BF16, "normal")
    model = mtx.Model(shape, wl.layer_tuples(net), wl.BF16, R, Nb, seed=1)
    x, y = wl.make_batch(net, R * Nb, seed=1)
    model.train_step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), 0.01, 0.9)
    torch.cuda.synchronize()
    seen = {(l["site"], l["layer"]): l["tile_rows"] for l in mtx.mtx_get_launches(model.handle)
            if l["flags"] & mtx.MTX_GEMM_HALO}
    print(f"[launches] {name}: {seen}", flush=True)
    model.close()
    for site, layer, rows in expected:
        assert (site, layer) in seen and rows in (None, seen[(site, layer)]), (site, layer, rows, seen)
    run_case("halo-" + name, net, R, Nb, 1, 3, 0.01, 0.9)


def test_window_convolution_keeps_infinities_apart():
    """One infinite input value: only the outputs whose window holds it may differ from a run
    with that value zero (the zero weights of padded reduction granules meet zero inputs)."""
    # 24 channels x 9 taps leave a padded granule
    layers = (wl.conv(24, 1), wl.conv(16, 3, pad=1), wl.fc(3))
    net = wl.Net("halo-inf", (24, 50, 50), layers, wl.BF16, "normal")
    x, y = wl.make_batch(net, 24, seed=2)
    outs = []
    for value in (0.0, np.inf):
        x[3, 2, 20, 30] = value
        model = mtx.Model(net.in_shape, wl.layer_tuples(net), wl.BF16, 2, 12, seed=1)
        model.train_step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), 0.0, 0.0)
        assert any(l["flags"] & mtx.MTX_GEMM_HALO and l["site"] == "fwd"
                   for l in mtx.mtx_get_launches(model.handle))
        outs.append(model.layer_output(1).reshape(24, 16, 50, 50))
        model.close()
    differ = np.argwhere(outs[0] != outs[1])
    assert len(differ)
    assert (differ[:, 0] == 3).all()
    assert (np.abs(differ[:, 2] - 20) <= 1).all() and (np.abs(differ[:, 3] - 30) <= 1).all()


# name: input shape, layers, shards, shard batch, the layers whose weight gradient takes windows
WGRAD_CASES = {
    # channel counts on 2- and 8-byte loads, a 2x2 kernel, groups, 32-channel output tiles
    "odd": ((3, 33, 31), (wl.conv(15, 3, pad=1, relu=True), wl.conv(20, 3, pad=1, relu=True),
                          wl.conv(36, 5, pad=2, groups=2, relu=True), wl.conv(12, 2),
                          wl.maxpool(3, 3), wl.fc(3)), 4, 20, {2, 3}),
    # a first layer of 8 channels with a 7x7 kernel, stride 2 (both on the implicit GEMM: too few
    # channels and tiles), an unpadded 5x5 layer
    "strided": ((8, 24, 24), (wl.conv(16, 7, pad=3, relu=True), wl.conv(136, 3, stride=2, pad=1, relu=True),
                              wl.conv(64, 5, relu=True), wl.maxpool(2, 2), wl.fc(5)), 32, 5, {2}),
    # stride 2 and 7x7 kernels, output tiles of 32 and 64 channels
    "s2k3": ((16, 32, 32), (wl.conv(64, 3, stride=2, pad=1, relu=True), wl.fc(3)), 16, 24, {0}),
    "s2k5": ((16, 32, 32), (wl.conv(16, 5, stride=2, pad=2, relu=True), wl.fc(3)), 16, 24, {0}),
    "s2k7": ((16, 24, 24), (wl.conv(128, 7, stride=2, pad=3, relu=True), wl.fc(3)), 8, 16, {0}),
    "k7": ((16, 12, 12), (wl.conv(16, 7, pad=3, relu=True), wl.fc(3)), 8, 32, {0}),
    # padded first layers: output tiles of 64 and 32 channels
    "firstw": ((3, 33, 31), (wl.conv(60, 3, pad=1, relu=True), wl.maxpool(3, 2), wl.fc(3)), 8, 64, {0}),
    "firstw2": ((5, 32, 32), (wl.conv(20, 4, pad=2, relu=True), wl.maxpool(3, 2), wl.fc(3)), 8, 100, {0}),
    # ... on the implicit GEMM
    "first32": ((3, 33, 31), (wl.conv(20, 3, pad=1, relu=True), wl.maxpool(3, 2), wl.fc(3)), 4, 40, set()),
    "first64": ((5, 41, 43), (wl.conv(76, 3, stride=2, relu=True), wl.maxpool(2, 2), wl.fc(3)), 2, 95, set()),
    "first2": ((3, 40, 42), (wl.conv(36, 2, stride=2, relu=True), wl.maxpool(2, 2), wl.fc(3)), 2, 120, set()),
    # one split: the rows are written straight into gradient rows that start off 16 bytes
    "direct": ((3, 8, 8), (wl.bn(), wl.conv(128, 3, pad=1, relu=True), wl.conv(256, 3, pad=1), wl.fc(3)),
               64, 2, {2}),
}


@pytest.mark.parametrize("name", sorted(WGRAD_CASES))
def test_window_weight_gradients_match_oracle(name):
    shape, layers, R, Nb, expected = WGRAD_CASES[name]
    net = wl.Net("halo-wgrad-" + name, shape, layers, wl.BF16, "normal")
    model = mtx.Model(shape, wl.layer_tuples(net), wl.BF16, R, Nb, seed=1)
    x, y = wl.make_batch(net, R * Nb, seed=1)
    model.train_step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), 0.01, 0.9)
    torch.cuda.synchronize()
    seen = {l["layer"]: (l["tile_rows"], l["splits"]) for l in mtx.mtx_get_launches(model.handle)
            if l["flags"] & mtx.MTX_GEMM_HALO and l["site"] == "wgrad"}
    print(f"[launches] {name}: {seen}", flush=True)
    model.close()
    assert expected <= set(seen), (expected, seen)
    run_case("halo-wgrad-" + name, net, R, Nb, 1, 3, 0.01, 0.9)


# name: input shape, layers, shards, shard batch, the launches (site, layer) that stay off the windows
OTHERWISE = {
    # a layer that closes its images to 1 x 1: 49 taps of its data gradient for one inside dy
    "closing": ((3, 7, 7), (wl.conv(128, 3, pad=1, relu=True), wl.conv(128, 7, relu=True), wl.fc(3)),
                4, 256, {("dgrad", 1)}),
    # 8 input channels in 64-row blocks at stride 2, and in the weight gradient's 16-channel fragments
    "stride2c8": ((3, 22, 22), (wl.conv(8, 3, pad=1, relu=True), wl.conv(192, 3, stride=2, pad=1, relu=True),
                                wl.maxpool(2, 2), wl.fc(3)), 8, 40, {("dgrad", 1), ("wgrad", 1)}),
    # wide images: most of a weight gradient's window is loaded without the prefetch
    "wide52": ((3, 52, 52), (wl.conv(64, 3, pad=1, relu=True), wl.conv(32, 3, relu=True), wl.maxpool(4, 4),
                             wl.fc(3)), 2, 30, {("wgrad", 1)}),
}


@pytest.mark.parametrize("name", sorted(OTHERWISE))
def test_layers_with_little_to_gain_stay_on_the_general_kernels(name):
    shape, layers, R, Nb, expected = OTHERWISE[name]
    net = wl.Net("halo-not-" + name, shape, layers, wl.BF16, "normal")
    model = mtx.Model(shape, wl.layer_tuples(net), wl.BF16, R, Nb, seed=1)
    x, y = wl.make_batch(net, R * Nb, seed=1)
    model.train_step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), 0.01, 0.9)
    torch.cuda.synchronize()
    seen = {(l["site"], l["layer"]) for l in mtx.mtx_get_launches(model.handle)
            if l["flags"] & mtx.MTX_GEMM_HALO}
    model.close()
    assert not expected & seen, (expected, seen)
    run_case("halo-not-" + name, net, R, Nb, 1, 3, 0.01, 0.9)


def test_padding_reads_zeros_in_every_channel():
    """1 x 1 images of 2112 channels under a 2 x 2 kernel with three positions of padding, on the
    four-wave block: 264 granules per position, more than the block has threads.  Four of 36
    outputs have a tap inside the image; all others are the bias."""
    B, C, OC = 1024, 2112, 192
    net = wl.Net("halo-zero", (C, 1, 1), (wl.conv(OC, 2, pad=3), wl.fc(3)), wl.BF16, "normal")
    model = mtx.Model(net.in_shape, wl.layer_tuples(net), wl.BF16, 2, B // 2, seed=1)
    rng = np.random.default_rng(3)
    w, _ = model.get_params()
    bias = rng.standard_normal(OC).astype(np.float32)
    w[C * OC * 4:C * OC * 4 + OC] = bias
    model.set_params(w)
    x, y = wl.make_batch(net, B, seed=3)
    model.train_step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), 0.0, 0.0)
    tiles = [(l["tile_rows"], l["tile_cols"]) for l in mtx.mtx_get_launches(model.handle)
             if l["flags"] & mtx.MTX_GEMM_HALO and l["site"] == "fwd"]
    out = model.layer_output(0).reshape(B, OC, 6, 6)
    model.close()
    assert tiles == [(192, 176)]

    def bf16(a):
        return torch.from_numpy(np.ascontiguousarray(a)).bfloat16().double()

    expected = bf16(bias).view(1, OC, 1, 1).repeat(B, 1, 6, 6)
    taps = bf16(w[:C * OC * 4].reshape(OC, C, 2, 2))
    for u in range(2):
        for v in range(2):
            expected[:, :, 3 - u, 3 - v] = (bf16(x.reshape(B, C)) @ taps[:, :, u, v].t()
                                            + torch.from_numpy(bias).double())
    got = torch.from_numpy(out).double()
    inside = np.zeros((6, 6), bool)
    inside[2:4, 2:4] = True
    assert bool((got[:, :, ~inside] == expected[:, :, ~inside]).all())
    # a rounding to bf16 (2^-9) of a sum of 2112 products in 32 bits (2112 roundings of 2^-24 of
    # magnitudes that add up to less than 100)
    error = (got - expected).abs()[:, :, inside]
    assert (error <= expected.abs()[:, :, inside] * 2.0 ** -8 + 2112 * 100 * 2.0 ** -24).all()

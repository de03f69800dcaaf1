"""The convolutions over windows held in LDS against the general kernels, bit for bit: a layer takes the
windows in a launch of many images and the implicit GEMM (or the col product) in one of few, and an
image's output and data gradient must not depend on which.  And the weight gradients over windows
against 64-bit sums of the same products.

Both tests know the output gradient of the layer under test exactly: the class biases (60, 0) saturate the
softmax to (1, 0), every label is 1, so the class gradients are (1, -1) / shard batch and the gradient
that reaches the layer is the difference of the two class weights, rounded once."""
import numpy as np
import pytest
import torch

from paper_1704_04560_amd import mtx
from paper_1704_04560_amd import workloads as wl

pytestmark = pytest.mark.gpu

FEW = 5


def _model(net, R, Nb, change=lambda w: None):
    """The same weights whatever R is, with the class biases above."""
    model = mtx.Model(net.in_shape, wl.layer_tuples(net), wl.BF16, R, Nb, seed=4)
    w, _ = model.get_params()
    w[-2:] = (60.0, 0.0)
    change(w)
    model.set_params(w)
    return model


def _step(model, x):
    """A step that leaves the weights as they are; its launches."""
    labels = torch.ones(model.B, dtype=torch.int32, device="cuda")
    model.train_step(x.cuda(), labels, 0.0, 0.0)
    torch.cuda.synchronize()
    return {(l["site"], l["layer"]): l for l in mtx.mtx_get_launches(model.handle)}


# name: channels, height, width, outputs, kernel, stride, padding, groups, images, what takes the windows
BITS = {
    "3x3": (64, 16, 16, 64, 3, 1, 1, 1, 300, ("fwd", "dgrad")),
    "5x5 groups": (64, 14, 14, 64, 5, 1, 2, 2, 260, ("fwd", "dgrad")),
    "ragged": (24, 19, 23, 40, 3, 1, 1, 1, 260, ("fwd", "dgrad")),
    "7x7": (16, 20, 20, 16, 7, 1, 3, 1, 200, ("fwd", "dgrad")),
    "2x2 unpadded": (64, 22, 22, 128, 2, 1, 0, 1, 200, ("fwd", "dgrad")),
    "8-byte rows": (28, 21, 20, 24, 3, 1, 1, 1, 200, ("dgrad",)),
    "2-byte rows": (32, 21, 20, 50, 3, 1, 1, 1, 300, ("fwd",)),
    "13x13 groups": (64, 13, 13, 192, 3, 1, 1, 2, 260, ("fwd", "dgrad")),
    "13x13, 11 fragments": (64, 13, 13, 384, 3, 1, 1, 1, 200, ("fwd",)),
    "13x13, 11 fragments, back": (384, 13, 13, 64, 3, 1, 1, 1, 200, ("dgrad",)),
    "22x22, 11 fragments": (32, 22, 22, 192, 3, 1, 1, 1, 150, ("fwd",)),
    "12x15, 384 rows": (64, 12, 15, 384, 2, 1, 1, 1, 400, ("fwd",)),
    "8x11, 256 rows, back": (256, 8, 11, 32, 3, 1, 1, 1, 400, ("dgrad",)),
    "1x1": (256, 32, 32, 64, 1, 1, 0, 1, 100, ("dgrad",)),
    "stride 2": (64, 17, 16, 64, 3, 2, 1, 1, 300, ("dgrad",)),
    "stride 2 5x5": (20, 19, 22, 64, 5, 2, 2, 1, 300, ("dgrad",)),
    "stride 2 7x7": (48, 21, 23, 64, 7, 2, 3, 1, 200, ("dgrad",)),
    "stride 2 groups": (256, 12, 12, 128, 3, 2, 1, 2, 200, ("dgrad",)),
}


@pytest.mark.parametrize("name", list(BITS))
def test_window_convolutions_give_the_general_kernels_bits(name):
    c, h, w, out, k, stride, pad, groups, images, sites = BITS[name]
    # a 1 x 1 layer of 8 channels below; each of an image's 8 channels is one somewhere and zero
    # elsewhere, so that its weight gradient is the data gradient at those 8 positions
    layers = (wl.conv(c, 1, relu=True),
              wl.conv(out, k, stride=stride, pad=pad, groups=groups, relu=True), wl.fc(2))
    net = wl.Net("bits", (8, h, w), layers, wl.BF16, "normal")
    rng = np.random.default_rng(7)
    ones = np.zeros((images, 8, h * w), np.float32)
    for i in range(images):
        ones[i, np.arange(8), rng.choice(h * w, 8, replace=False)] = 1.0
    ones = torch.from_numpy(ones.reshape(images, 8, h, w))
    dense = torch.from_numpy(rng.standard_normal((images, 8, h, w)).astype(np.float32))
    biases = rng.standard_normal(c).astype(np.float32)
    got = []
    for n in (images, FEW):
        print(f"[bits] {name}: {n} images", flush=True)
        model = _model(net, n, 1, lambda w: w.__setitem__(slice(8 * c, 9 * c), biases))
        plans = _step(model, ones[:n])
        for site in sites:
            p = plans[(site, 1)]
            assert bool(p["flags"] & mtx.MTX_GEMM_HALO) == (n == images), (site, n, p)
            assert p["splits"] == 1, (site, n, p)
        dx = model.grads.view(n, model.ld)[:FEW, :c * 8].cpu().numpy()
        _step(model, dense[:n])
        y = model.layer_output(1).reshape(n, -1)[:FEW]
        model.close()
        got.append((y, dx))
    (y0, dx0), (y1, dx1) = got
    if "fwd" in sites:
        assert np.count_nonzero(y0) > y0.size // 8
        assert np.array_equal(y0.view(np.uint32), y1.view(np.uint32))
    if "dgrad" in sites:
        assert np.count_nonzero(dx0) > dx0.size // 8
        assert np.array_equal(dx0.view(np.uint32), dx1.view(np.uint32))


# first layers over a padded input: channels, height, width, outputs, kernel, stride, padding, images
FIRST = [(3, 32, 32, 64, 3, 1, 1, 64), (3, 115, 115, 96, 11, 4, 0, 100), (5, 40, 42, 24, 5, 2, 0, 190)]


@pytest.mark.parametrize("c,h,w,out,k,stride,pad,images", FIRST)
def test_padded_first_layers_give_the_general_kernels_bits(c, h, w, out, k, stride, pad, images):
    layers = (wl.conv(out, k, stride=stride, pad=pad, relu=True), wl.maxpool(2, 2), wl.fc(2))
    net = wl.Net("bits-first", (c, h, w), layers, wl.BF16, "normal")
    x = torch.from_numpy(np.random.default_rng(8).standard_normal((images, c, h, w)).astype(np.float32))
    got = []
    for n in (images, FEW):
        print(f"[bits] first {k}x{k}: {n} images", flush=True)
        model = _model(net, n, 1)
        p = _step(model, x[:n])[("fwd", 0)]
        assert bool(p["flags"] & mtx.MTX_GEMM_HALO) == (n == images) and p["splits"] == 1, (n, p)
        got.append(model.layer_output(0).reshape(n, -1)[:FEW].view(np.uint32))
        model.close()
    assert np.array_equal(got[0], got[1])


# channels, height, width, outputs, kernel, stride, padding, groups, shards, shard batch: output tiles of 32
# and 64 channels, 16-byte, 8-byte and single loads, strides, a last tile that is not full
SUMS = [(64, 16, 16, 64, 3, 1, 1, 1, 16, 64), (16, 32, 32, 16, 5, 2, 2, 1, 8, 64),
        (16, 24, 24, 128, 7, 2, 3, 1, 4, 64), (96, 17, 15, 64, 2, 1, 0, 1, 8, 64),
        (40, 13, 13, 72, 5, 1, 2, 2, 4, 64), (20, 23, 21, 36, 5, 1, 2, 2, 4, 64),
        (58, 19, 17, 62, 5, 1, 2, 2, 4, 64), (64, 19, 17, 60, 3, 1, 1, 1, 8, 64)]


@pytest.mark.parametrize("c,h,w,out,k,stride,pad,groups,R,Nb", SUMS)
def test_window_weight_gradients_are_32_bit_sums(c, h, w, out, k, stride, pad, groups, R, Nb):
    layers = (wl.conv(c, 1, relu=True),
              wl.conv(out, k, stride=stride, pad=pad, groups=groups, relu=True), wl.fc(2))
    net = wl.Net("sums", (8, h, w), layers, wl.BF16, "normal")
    x = torch.from_numpy(np.random.default_rng(9).standard_normal((R * Nb, 8, h, w)).astype(np.float32))
    print(f"[sums] {c} -> {out}, {k} x {k}, stride {stride}", flush=True)
    model = _model(net, R, Nb)
    weights, _ = model.get_params()
    p = _step(model, x)[("wgrad", 1)]
    assert p["flags"] & mtx.MTX_GEMM_HALO, p
    oh, ow = (h + 2 * pad - k) // stride + 1, (w + 2 * pad - k) // stride + 1
    n1, nw = c * 8 + c, out * (c // groups) * k * k
    rows = torch.from_numpy(model.grads_host()[:, n1:n1 + nw + out]).double()
    a = torch.from_numpy(model.layer_output(0)).double().view(R, Nb, c, h, w)
    y = torch.from_numpy(model.layer_output(1)).double().view(R, Nb, out, oh, ow)
    model.close()
    classes = torch.from_numpy(weights[-2 * out * oh * ow - 2:-2].copy()).bfloat16().float().view(2, -1)
    dy = ((classes[0] - classes[1]) / Nb).bfloat16().double().view(1, 1, out, oh, ow) * (y > 0)
    # a product goes through a rounding for each 32 positions after its own, which are random; a
    # position left out or taken twice would show as 1 / sqrt(positions)
    bound = 4 * 2.0 ** -24 * (Nb * oh * ow / 32) ** 0.5
    for r in (0, R - 1):
        cols = torch.nn.functional.unfold(a[r], k, padding=pad, stride=stride)
        cols = cols.view(Nb, groups, -1, oh * ow).permute(1, 2, 0, 3).reshape(groups, -1, Nb * oh * ow)
        d = dy[r].view(Nb, groups, -1, oh * ow).permute(1, 2, 0, 3)
        d = d.reshape(groups, -1, Nb * oh * ow)
        expected = torch.cat([(d @ cols.transpose(1, 2)).flatten(), d.sum(2).flatten()])
        for lo, hi in ((0, nw), (nw, nw + out)):
            error = (rows[r, lo:hi] - expected[lo:hi]).norm() / expected[lo:hi].norm()
            print(f"[sums] shard {r}: error {error.item():.2e} of {bound:.2e}", flush=True)
            assert error <= bound, (r, lo)

"""mtx_init_model_static: a model whose workspace is the library's static device array, for
callers that cannot allocate device memory.  Its steps must give exactly what the same model with
a caller workspace (mtx_init_model) gives: the same kernels run in the same order.  Two models in
a row, the second with a smaller batch, so that the second reuses the array the first wrote."""
import numpy as np
import pytest
import torch

from paper_1704_04560_amd import mtx
from paper_1704_04560_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _same(a, b, what):
    assert np.array_equal(np.asarray(a).view(np.uint32), np.asarray(b).view(np.uint32)), what


def _pair(net, R, Nb, seed, steps):
    layers = wl.layer_tuples(net)
    print(f"[case] static workspace {net.name} B={R * Nb} R={R}", flush=True)
    ref = mtx.Model(net.in_shape, layers, net.dtype, R, Nb, seed=seed)
    st = mtx.Model(net.in_shape, layers, net.dtype, R, Nb, seed=seed, static_workspace=True)
    assert st.workspace is None
    la, lb = torch.zeros(1, device="cuda"), torch.zeros(1, device="cuda")
    for step in range(steps):
        x, y = wl.make_batch(net, R * Nb, seed=seed * 10 + step)
        xd, yd = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
        ref.train_step(xd, yd, 0.01, 0.9, la)
        st.train_step(xd, yd, 0.01, 0.9, lb)
        torch.cuda.synchronize()
        wa, va = ref.get_params()
        wb, vb = st.get_params()
        _same(wa, wb, f"w step {step}")
        _same(va, vb, f"v step {step}")
        _same(ref.grads_host(), st.grads_host(), f"grads step {step}")
        _same(ref.grad_avg.cpu().numpy(), st.grad_avg.cpu().numpy(), f"average step {step}")
        assert la.item() == lb.item(), step
        for i in range(len(layers)):  # outputs in the static array are the last step's
            _same(ref.layer_output(i), st.layer_output(i), f"layer {i} output step {step}")
    ref.close()
    st.close()


def test_static_workspace_steps_match_the_caller_workspace_twice_the_second_smaller():
    _pair(wl.LENET, 4, 64, 3, 2)   # the LeNet workload: 43 MB of its 64 MiB
    _pair(wl.LENET, 2, 8, 4, 2)    # smaller, reusing the array the first model wrote
    _pair(wl.MLP, 2, 32, 5, 2)


def test_static_workspace_matches_where_only_the_general_kernels_fit_it():
    """162 images of a shard: the convolutions over LDS windows fit 64 MiB; 163: their partial sums do
    not, the implicit GEMMs' do, and both kinds of model run those."""
    layers = (wl.conv(64, 5, pad=2, relu=True), wl.maxpool(2, 2), wl.fc(5))
    net = wl.Net("static-edge", (32, 16, 16), layers, wl.BF16, "normal")
    for Nb, windows in ((162, True), (163, False)):
        _pair(net, 2, Nb, 6, 2)
        m = mtx.Model(net.in_shape, wl.layer_tuples(net), net.dtype, 2, Nb)
        assert m.ws_bytes <= 64 << 20
        x, y = wl.make_batch(net, 2 * Nb, seed=1)
        m.train_step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), 0.01, 0.9)
        torch.cuda.synchronize()
        taken = any(l["flags"] & mtx.MTX_GEMM_HALO for l in mtx.mtx_get_launches(m.handle))
        m.close()
        assert taken == windows, Nb


def test_static_workspace_alternating_models():
    """Two static models on one device, steps alternating (not overlapping): each step
    re-establishes its own part of the shared array."""
    net = wl.LENET
    layers = wl.layer_tuples(net)
    a = mtx.Model(net.in_shape, layers, net.dtype, 4, 16, seed=7, static_workspace=True)
    b = mtx.Model(net.in_shape, layers, net.dtype, 2, 4, seed=8, static_workspace=True)
    ra = mtx.Model(net.in_shape, layers, net.dtype, 4, 16, seed=7)
    rb = mtx.Model(net.in_shape, layers, net.dtype, 2, 4, seed=8)
    xa, ya = (torch.from_numpy(t).cuda() for t in wl.make_batch(net, 64, seed=1))
    xb, yb = (torch.from_numpy(t).cuda() for t in wl.make_batch(net, 8, seed=2))
    for _ in range(2):
        for m, x, y in ((a, xa, ya), (b, xb, yb), (ra, xa, ya), (rb, xb, yb)):
            m.train_step(x, y, 0.01, 0.9)
            torch.cuda.synchronize()
    _same(a.get_params()[0], ra.get_params()[0], "model a")
    _same(b.get_params()[0], rb.get_params()[0], "model b")
    for m in (a, b, ra, rb):
        m.close()


def test_static_workspace_rejects_networks_that_do_not_fit():
    net = wl.CIFAR  # B = 512: about 600 MB of workspace
    layers = wl.layer_tuples(net)
    with pytest.raises(mtx.MtxError) as e:
        mtx.Model(net.in_shape, layers, net.dtype, 8, 64, seed=0, static_workspace=True)
    assert e.value.code == mtx.MTX_ENOMEM and "static workspace" in str(e.value)

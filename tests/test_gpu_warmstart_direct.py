"""The matrix-core forms of the FP32 convolutions and weight gradients at the
edges of their tiles, against the FP64 oracle: channels that fill no group of
16 or no stage of 128, more than 128 rows, windows of 32, 64 (the wider tile)
and 128 positions (the generic form), a patch that makes the embedding's
reduction odd, positions that end inside a tile.  Tolerances as for the other
sizes of the same sums: 1e-5 of the largest output, 2e-4 of a layer's gradient
norm."""
import numpy as np
import pytest

from oracle import nn as onn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfgd, n", [
    (dict(window=12, patch=3, width=20, hidden=1, nx=5, ny=1), 5),      # 4 positions a window, 20 in all
    (dict(window=64, patch=2, width=33, hidden=2, nx=3, ny=2), 3),      # 32 positions a window
    (dict(window=64, patch=1, width=40, hidden=2, nx=5, ny=2), 3),      # 64
    (dict(window=128, patch=1, width=24, hidden=1, nx=5, ny=2), 2),     # 128
    (dict(window=16, patch=2, width=150, hidden=2, nx=5, ny=3), 19),    # two row blocks, two channel stages
    (dict(window=48, patch=4, width=36, hidden=2, nx=5, ny=2), 7),      # 12 positions: not in a tile
])
def test_forward_and_gradient(cfgd, n):
    import torch
    from paper_2102_00514_amd import warmstart as W
    net = W.WarmStartNet(W.config(max_batch=n + 3, **cfgd), stream=torch.cuda.current_stream().cuda_stream, seed=4)
    rng = np.random.default_rng(5)
    x = rng.uniform(-1, 1, (2 * n, 2 * cfgd["ny"], cfgd["window"])).astype(np.float32)
    lab = (rng.standard_normal((2 * n, cfgd["window"], cfgd["nx"])) * 2 + 0.5).astype(np.float32)
    idx = rng.permutation(2 * n)[:n].astype(np.int32)
    dx, dl, di = (torch.from_numpy(v).cuda() for v in (x, lab, idx))
    out = torch.empty((n, cfgd["window"], cfgd["nx"]), dtype=torch.float32, device="cuda")
    for seed in (6, 7):    # the second parameters replace the first ones' packed copy
        theta = net.params() + (0.05 * np.random.default_rng(seed).standard_normal(net.n_params)).astype(np.float32)
        net.set_params(theta)
        t64 = net.params().astype(np.float64)
        ref, cache = onn.forward(t64, x[idx].astype(np.float64), cfgd)
        one, zero = np.ones(cfgd["nx"]), np.zeros(cfgd["nx"])
        net.predict(dx.data_ptr(), 2 * n, di.data_ptr(), n, out.data_ptr())
        want = onn.outputs_to_states(ref, zero, one, cfgd)
        assert np.abs(out.cpu().numpy() - want).max() < 1e-5 * np.abs(want).max()
        g, loss = net.gradient(dx.data_ptr(), dl.data_ptr(), 2 * n, di.data_ptr(), n)
        tgt = onn.states_to_outputs(lab[idx].astype(np.float64), zero, one, cfgd)
        assert abs(loss - onn.loss(ref, tgt)) < 1e-5 * onn.loss(ref, tgt)
        gref = onn.backward(t64, cache, ref, tgt, cfgd)
        pos = 0
        for shapes in onn.layer_shapes(cfgd):
            for s in shapes:
                sl = slice(pos, pos + int(np.prod(s)))
                pos = sl.stop
                assert np.linalg.norm(g[sl] - gref[sl]) < 2e-4 * np.linalg.norm(gref[sl]), (shapes, s)
    net.close()


@pytest.mark.parametrize("max_batch, n", [(600, 512), (600, 587), (1100, 1024)])
def test_gradient_of_a_batch_below_max_batch(max_batch, n):
    """Default network: batches that have more chunks than max_batch has, and
    one with several stages to a chunk and a last chunk cut short.

    Tolerance: rounding moves a gradient of these sizes by 5e-7 of its norm, a
    ReLU input that changes sign by it by up to 8e-5 (an FP32 evaluation on the
    CPU against the FP64 one), and a few of the 5 to 10 million inputs may do so:
    1e-3.  A chunk left out or added twice would be 1/128 or more."""
    import torch
    from paper_2102_00514_amd import warmstart as W
    cfgd = dict(window=64, patch=4, width=128, hidden=4, nx=5, ny=2)
    net = W.WarmStartNet(W.config(max_batch=max_batch, **cfgd), stream=torch.cuda.current_stream().cuda_stream, seed=4)
    rng = np.random.default_rng(n)
    x = rng.uniform(-1, 1, (n, 4, 64)).astype(np.float32)
    lab = (rng.standard_normal((n, 64, 5)) * 2 + 0.5).astype(np.float32)
    idx = rng.permutation(n).astype(np.int32)
    dx, dl, di = (torch.from_numpy(v).cuda() for v in (x, lab, idx))
    g, loss = net.gradient(dx.data_ptr(), dl.data_ptr(), n, di.data_ptr(), n)
    t64 = net.params().astype(np.float64)
    ref, cache = onn.forward(t64, x[idx].astype(np.float64), cfgd)
    tgt = onn.states_to_outputs(lab[idx].astype(np.float64), np.zeros(5), np.ones(5), cfgd)
    assert abs(loss - onn.loss(ref, tgt)) < 1e-5 * onn.loss(ref, tgt)
    gref = onn.backward(t64, cache, ref, tgt, cfgd)
    pos = 0
    for shapes in onn.layer_shapes(cfgd):
        for s in shapes:
            sl = slice(pos, pos + int(np.prod(s)))
            pos = sl.stop
            assert np.linalg.norm(g[sl] - gref[sl]) < 1e-3 * np.linalg.norm(gref[sl]), (shapes, s)
    net.close()

"""Calls of the warm-start network captured into a graph of the caller's: a
replay runs with the parameters that the handle holds at that time, however
they got there (ws_set_params, an eager training step, a replayed one), and
eager calls after a replayed training step run with its parameters.  The
reference is a handle that was given those parameters and made the same call:
equal bit for bit, since the same kernels run on the same values."""
import numpy as np
import pytest

from paper_2102_00514_amd import workloads as wl

pytestmark = pytest.mark.gpu

# the one-kernel inference with the matrix-core convolutions, and the generic forms of both
CONFIGS = [dict(window=64, patch=4, width=128, hidden=2, nx=5, ny=2),
           dict(window=48, patch=4, width=36, hidden=1, nx=5, ny=2)]


def _setup(cfgd):
    import torch
    from paper_2102_00514_amd import warmstart as W
    s = torch.cuda.Stream()
    pb = wl.concat_tracks([wl.ct_bearings(T, seed=40 + T) for T in (130, 48, 7)], "graph")
    y = torch.from_numpy(np.ascontiguousarray(pb.y)).cuda()

    def new(theta):
        net = W.WarmStartNet(W.config(max_batch=8, **cfgd), stream=s.cuda_stream, params=theta)
        net.set_tracks(pb.offsets)
        return net

    theta = W.init_params(W.config(max_batch=8, **cfgd), seed=3)
    rng = np.random.default_rng(8)
    thetas = [theta + (0.05 * rng.standard_normal(theta.size)).astype(np.float32) for _ in range(3)]
    mean = torch.zeros((pb.n_slots, 5), dtype=torch.float64, device="cuda")

    def trajectory(net, mfma):
        net.trajectory(y.data_ptr(), mean.data_ptr(), mfma=mfma)
        torch.cuda.synchronize()
        return mean.cpu().numpy().copy()

    n = 6
    x = torch.from_numpy(rng.uniform(-1, 1, (n, 4, cfgd["window"])).astype(np.float32)).cuda()
    lab = torch.from_numpy(rng.standard_normal((n, cfgd["window"], 5)).astype(np.float32)).cuda()
    idx = torch.arange(n, dtype=torch.int32, device="cuda")

    def step(net):
        net.train_step(x.data_ptr(), lab.data_ptr(), n, idx.data_ptr(), n, lr=0.05)

    torch.cuda.synchronize()
    return torch, s, new, thetas, y, mean, trajectory, step


@pytest.mark.parametrize("cfgd", CONFIGS, ids=("fused", "generic"))
@pytest.mark.parametrize("mfma", (False, True), ids=("fp32", "bf16"))
def test_replay_uses_the_current_parameters(cfgd, mfma):
    torch, s, new, thetas, y, mean, trajectory, step = _setup(cfgd)
    net = new(thetas[0])
    trajectory(net, mfma)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        net.trajectory(y.data_ptr(), mean.data_ptr(), mfma=mfma)

    def replay():
        mean.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        return mean.cpu().numpy().copy()

    for theta in thetas:
        net.set_params(theta)
        got = replay()
        assert np.array_equal(got, trajectory(new(theta), mfma))
    step(net)
    got = replay()
    want = trajectory(new(net.params()), mfma)
    assert np.array_equal(got, want) and not np.array_equal(got, trajectory(new(thetas[-1]), mfma))


@pytest.mark.parametrize("cfgd", CONFIGS, ids=("fused", "generic"))
def test_eager_calls_after_a_replayed_training_step(cfgd):
    torch, s, new, thetas, y, mean, trajectory, step = _setup(cfgd)
    net = new(thetas[0])
    step(net)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        step(net)
    before = net.params()
    for _ in range(3):
        for mfma in (False, True):
            trajectory(net, mfma)
        g.replay()
        torch.cuda.synchronize()
        theta = net.params()
        assert not np.array_equal(theta, before)
        before = theta
        for mfma in (False, True):
            assert np.array_equal(trajectory(net, mfma), trajectory(new(theta), mfma))

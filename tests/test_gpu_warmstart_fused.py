"""The one-kernel inference form of the warm-start network (ws_trajectory_mfma
at widths 128 and 256 with whole windows in 128 positions) at the edges of its
tiles, against the FP64 oracle with BF16-rounded operands.

Gates in units of the output scale: an operand within an FP32 ulp of a
bfloat16 rounding boundary may round the other way and move a few outputs by
up to 2^-8 of an activation, so the mean is held to 5e-5, the largest to 5e-2
and the share beyond 1e-3 to 1 % (a wrong fragment, tap or window edge moves
outputs by order one)."""
import numpy as np
import pytest

from oracle import nn as onn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfgd, lengths", [
    # one short track: a single window in a tile of eight
    (dict(window=64, patch=4, width=128, hidden=4, nx=5, ny=2), [1]),
    # ragged tracks whose windows overlap, tail of the last tile
    (dict(window=64, patch=4, width=128, hidden=4, nx=5, ny=2), [64, 65, 63, 700, 129]),
    # no residual layer; one window per tile of 128 positions
    (dict(window=128, patch=1, width=128, hidden=0, nx=5, ny=2), [128, 200, 7]),
    # reduction of the embedding longer than the width (two column blocks), 36 head rows
    (dict(window=32, patch=4, width=128, hidden=2, nx=9, ny=17), [32, 33, 400]),
    # reduction that is no multiple of 16, width 256, dilation up to half a window
    (dict(window=24, patch=3, width=256, hidden=3, nx=3, ny=1), [24, 23, 300, 1]),
])
def test_fused_inference_matches_oracle(cfgd, lengths):
    import torch
    from paper_2102_00514_amd import warmstart as W
    rng = np.random.default_rng(11)
    offsets = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    y = rng.uniform(-np.pi, np.pi, (int(offsets[-1]), cfgd["ny"]))
    mu = rng.standard_normal(cfgd["nx"]).astype(np.float32)
    sigma = rng.uniform(0.5, 2.0, cfgd["nx"]).astype(np.float32)
    net = W.WarmStartNet(W.config(max_batch=4, **cfgd), stream=torch.cuda.current_stream().cuda_stream)
    net.set_normalization(mu, sigma)
    net.set_tracks(offsets)
    dy = torch.from_numpy(y).cuda()
    x = onn.features(y, offsets, cfgd)
    for seed in (1, 2):   # the second parameters replace the first ones' packed copy
        theta = onn.init_params(np.random.default_rng(seed), cfgd)
        theta += (0.1 * np.random.default_rng(seed + 9).standard_normal(theta.size)).astype(np.float32) * (theta == 0)
        net.set_params(theta)
        got = torch.full((int(offsets[-1]) + len(lengths), cfgd["nx"]), float("nan"), dtype=torch.float64,
                         device="cuda")
        net.trajectory(dy.data_ptr(), got.data_ptr(), mfma=True)
        got = got.cpu().numpy()
        out, _ = onn.forward(theta.astype(np.float64), x, cfgd, operand_round=onn.bf16_round)
        ref = onn.trajectory(onn.outputs_to_states(out, mu.astype(np.float64), sigma.astype(np.float64), cfgd),
                             offsets, cfgd)
        scale = sigma * max(1.0, float(np.sqrt(np.mean(out ** 2))))
        d = np.abs(got - ref) / scale
        assert np.all(np.isfinite(got))
        assert d.mean() < 5e-5 and d.max() < 5e-2 and np.mean(d > 1e-3) < 1e-2, (d.mean(), d.max())
    net.close()

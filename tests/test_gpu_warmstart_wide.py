"""ws_trajectory_mfma where the embedding has more columns than the width, or
the head many rows: the forms that run them outside the one kernel, and column
blocks inside it.  Same oracle and gates as the one-kernel form."""
import pytest

from tests import test_gpu_warmstart_fused as fused

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfgd, lengths", [
    # embedding outside: pairs that fill four column blocks, pairs that would be split, longer than a block
    (dict(window=64, patch=16, width=128, hidden=1, nx=2, ny=16), [64, 65, 190]),
    (dict(window=48, patch=12, width=128, hidden=1, nx=2, ny=11), [48, 50, 97]),
    (dict(window=1024, patch=256, width=128, hidden=1, nx=1, ny=2), [1024, 1500, 3]),
    # 257 blocks: two column blocks in the kernel, the last one cut short
    (dict(window=64, patch=8, width=128, hidden=0, nx=2, ny=12), [64 * 4100]),
    # head outside, alone and with the embedding, no residual layer between them; width 256
    (dict(window=64, patch=8, width=128, hidden=1, nx=20, ny=2), [64, 70]),
    (dict(window=64, patch=16, width=128, hidden=0, nx=6, ny=16), [64, 200]),
    (dict(window=64, patch=16, width=256, hidden=1, nx=6, ny=16), [64, 65]),
])
def test_wide_embedding_and_head(cfgd, lengths):
    fused.test_fused_inference_matches_oracle(cfgd, lengths)

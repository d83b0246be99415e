"""Input layer through LDS tiles: 64 and 128 columns a workgroup, last tiles partly outside the batch, block sizes with a kernel of their own
and without; masked and out-of-range categories."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2406_00766_amd import workloads as W
from tests.test_gpu_parity import check_all

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,S,K,B", [
    (64, 256, 32, 150), (64, 256, 32, 256), (64, 256, 32, 290),     # 2048 input blocks: 128 columns, the last tile whole and cut
    (64, 256, 32, 100), (20, 64, 32, 70),                           # 64 columns
    (24, 128, 64, 97), (12, 60, 20, 65), (12, 12, 12, 130),
])
def test_input_tiles_match_oracle(D, S, K, B):
    w = W.rat_spn(D, 2, 4, S, K, B, 96, n_cats=11)
    print(f"case input tiles D={D} S={S} K={K} B={B}", flush=True)
    rng = np.random.default_rng(7)
    mask = (rng.random(w.x.shape) < 0.2).astype(np.uint8)
    x = w.x.copy()
    x[3, 0] = w.n_cats + 2; mask[3, 0] = 0                         # a sample of probability 0
    check_all(w.with_batch(x), mask)

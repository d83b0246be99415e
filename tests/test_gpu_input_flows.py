"""Input-layer flows summed per category (k_input_bwd_sorted): both sides of the lines between 256, 512 and 1024 threads, batches of more than
one slab with a ragged last one, tiles of more quads than one round of loads takes, as many categories as the scan holds; masked and
out-of-range categories."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2406_00766_amd import workloads as W
from tests.test_gpu_parity import check_all

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,B,n_cats", [
    (32, 128, 256), (32, 129, 256),                              # a tile of 16 KB, one of 20: 256 and 512 threads
    (32, 384, 100), (32, 385, 200),                              # 48 and 52 KB: 512 and 1024
    (32, 512, 256), (32, 520, 140), (64, 300, 128),              # the largest slab, two slabs of which the last has 32 or 64 columns
    (65, 256, 128),                                              # 4160 quads, 4096 a round
    (16, 900, 256), (128, 128, 256), (128, 150, 100),            # 1024 threads: the longest slab, the widest; a second slab of 32 columns
    (16, 100, 1023), (32, 330, 1024), (64, 70, 513),
])
def test_flows_per_category_match_oracle(K, B, n_cats):
    w = W.rat_spn(8, 1, 2, K, K, B, 97, n_cats=n_cats)
    print(f"case input flows K={K} B={B} n_cats={n_cats}", flush=True)
    rng = np.random.default_rng(11)
    mask = (rng.random(w.x.shape) < 0.2).astype(np.uint8)
    x = w.x.copy()
    x[:, 1] = n_cats - 1                                           # one category for all samples
    x[3, 0] = w.n_cats + 2; mask[3, 0] = 0                         # a sample of probability 0
    check_all(w.with_batch(x), mask)

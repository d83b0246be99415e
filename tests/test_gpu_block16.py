"""Blocks of 16 nodes against the oracle, at the sizes where their kernels change: a row's neighbours dealt to four waves or
not, last batches of four neighbours partly empty, batches that end in half a round of 64 samples, a parameter block's
pairs split over waves."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2406_00766_amd import workloads as W
from tests.test_gpu_parity import check_all

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("make", [
    lambda: W.hmm(4, 16, 7, 16, 1, 91),                            # one neighbour per row, one sample
    lambda: W.hclt(9, 80, 16, 33, 92, n_cats=6),                   # five neighbours, Bs = 64
    lambda: W.hmm(6, 128, 20, 16, 65, 93, alpha_trans=0.1),        # eight: the first row that is dealt out; tied pairs, Bs = 96
    lambda: W.hmm(3, 272, 20, 16, 32, 94, alpha_trans=0.05),       # seventeen: one wave has five of them, Bs = 32
    lambda: W.sum_layer(9, 512, 16, 130, 95, keep=0.4, n_cats=9),  # ragged rows, one wave per tile, Bs = 160
    lambda: W.pd(3, 1, 64, 16, 97, 96, n_cats=4, keep=0.5),        # blocks fed by several layers: flows added to
    lambda: W.hmm(24, 16, 9, 16, 40, 97),                          # two parameter blocks, 23 pairs: split over waves
])
def test_blocks_of_16_match_oracle(make):
    w = make()
    print(f"case block16 {w.name}", flush=True)
    rng = np.random.default_rng(9)
    mask = (rng.random(w.x.shape) < 0.15).astype(np.uint8)
    x = w.x.copy()
    if w.B > 4:
        x[3, 0] = w.n_cats + 2; mask[3, 0] = 0                     # a sample of probability 0
    check_all(w.with_batch(x), mask)

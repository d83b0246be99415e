"""Input layer through LDS tiles: 64 and 128 columns a workgroup, last tiles partly outside the batch, block sizes with a kernel of their own
and without, in a launch of its own (on the transposed batch) and in the one that begins the pass (on the batch itself), on both sides of the
line between them; masked and out-of-range categories.  The kernels are asserted."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2406_00766_amd import binding as pcb
from paper_2406_00766_amd import workloads as W
from tests.refs import kernels, launches
from tests.test_gpu_dataflow import Dag
from tests.test_gpu_parity import check_all

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,S,K,B,kernel", [
    (64, 256, 32, 150, "k_input_fwd_tile<32, 128>"), (64, 256, 32, 256, "k_input_fwd_tile<32, 128>"),   # 2048 input blocks: the last tile
    (64, 256, 32, 290, "k_input_fwd_tile<32, 128>"),                                                    # whole and cut
    (65, 256, 32, 90, "k_input_fwd_tile<32, 64>"), (65, 256, 64, 200, "k_input_fwd_tile<64, 64>"),      # 4160 workgroups of 64 columns
    (64, 256, 32, 100, "k_begin_forward<32>"), (64, 256, 64, 200, "k_begin_forward<64>"),               # 4096
    (20, 64, 32, 70, "k_begin_forward<32>"), (24, 128, 64, 97, "k_begin_forward<64>"),
    (12, 60, 20, 65, "k_input_fwd_tile<0, 64>"), (12, 12, 12, 130, "k_input_fwd_tile<0, 64>"),
])
def test_input_tiles_match_oracle(D, S, K, B, kernel):
    w = W.rat_spn(D, 2, 4, S, K, B, 96, n_cats=11)
    print(f"case input tiles D={D} S={S} K={K} B={B}", flush=True)
    assert kernels(w, 0)[0] == kernel
    rng = np.random.default_rng(7)
    mask = (rng.random(w.x.shape) < 0.2).astype(np.uint8)
    x = w.x.copy()
    x[3, 0] = w.n_cats + 2; mask[3, 0] = 0                         # a sample of probability 0
    check_all(w.with_batch(x), mask)


def test_largest_batch_is_within_the_limit_of_a_grid():
    """512 blocks of 4 nodes and the most samples of a call: 2^24 workgroups of 256 threads, where HIP takes fewer than 2^32 threads in a dimension of a
    grid.  The launches are captured and dropped; the addresses name no memory."""
    d = Dag(4)
    w = d.workload(d.sum([d.product([d.input() for _ in range(512)])], n_real=1), 1, 98)
    h = pcb.pc_compile(w)
    print("case largest batch of small blocks", flush=True)
    somewhere, B = 1 << 40, 1 << 21
    found = launches(lambda stream: pcb.pc_forward(h, somewhere, somewhere, somewhere, None, B, somewhere, pcb.pc_workspace_bytes(h, B), somewhere, stream))
    pcb.pc_destroy(h)
    assert [k[0] for k in found].count("k_input_fwd_tile<0, 64>") == 1
    for k in found: assert all(n * t < 1 << 32 for n, t in zip(k[1:4], (k[4], 1, 1))), k

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
    (65, 96, 32, 390, "k_input_fwd_tile<32, 128>"), (65, 192, 64, 330, "k_input_fwd_tile<64, 64>"),     # 780 blocks, four beyond whole eights
    (27, 128, 32, 70, "k_begin_forward<32>"), (21, 192, 64, 97, "k_begin_forward<64>"), (65, 96, 32, 1600, "k_input_fwd_tile<32, 128>"),
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


def forward_launches(w):
    c = pcb.Circuit(w)
    c.set_batch(w.x)

    def call(stream):
        with torch.cuda.stream(stream): c.forward()
    found = launches(call)
    c.close()
    return found


@pytest.mark.parametrize("D,K,B,kernel", [
    (3, 32, 150, "k_begin_forward<32>"), (10, 64, 70, "k_begin_forward<64>"), (17, 32, 65, "k_begin_forward<32>"),
    (1, 20, 300, "k_input_fwd_tile<0, 64>"), (7, 12, 65, "k_input_fwd_tile<0, 64>"), (9, 12, 200, "k_input_fwd_tile<0, 64>"),
    (16, 12, 129, "k_input_fwd_tile<0, 64>"),
])
def test_every_workgroup_has_a_tile(D, K, B, kernel):
    """Numbers of input blocks that are no multiple of the number of XCDs."""
    w = W.hmm(D, K, 11, K, B, 97)
    print(f"case few input blocks D={D} K={K} B={B}", flush=True)
    assert kernels(w, 0)[0] == kernel
    Bs = -(-B // 32) * 32
    tiles = D * -(-Bs // 64)
    first = forward_launches(w)[kernel.startswith("k_input")]
    if kernel.startswith("k_begin"): tiles += Bs // 32 + -(-K * Bs // 4096)   # the transposed batch, the null block's rows
    assert first[0] == kernel and first[1] * first[2] == tiles
    check_all(w, (np.random.default_rng(8).random(w.x.shape) < 0.2).astype(np.uint8))

"""How the parameter flows of tied models are dealt to waves and workgroups: as many as its chunks allow where a model is small, a
fixed order where it has many blocks.  The launches are asserted."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2406_00766_amd import binding as pcb
from paper_2406_00766_amd import workloads as W
from tests.refs import launches
from tests.test_gpu_parity import check_all, gpu_run

pytestmark = pytest.mark.gpu


def param_workgroups(w):
    """Workgroups of the launch that takes the parameter flows."""
    c = pcb.Circuit(w)
    c.set_batch(w.x)
    c.forward()

    def call(stream):
        with torch.cuda.stream(stream): c.backward()
    found = [k[1] for k in launches(call) if k[0].startswith("k_param_flow")]
    c.close()
    assert len(found) == 1
    return found[0]


@pytest.mark.parametrize("T,H,K,B,waves", [
    (4, 352, 32, 100, 4), (16, 352, 32, 120, 4), (3, 480, 32, 64, 1), (4, 480, 32, 64, 4),   # 132 and 240 blocks; two pairs each, one at T = 3
    (4, 352, 32, 20, 1), (4, 512, 32, 100, 1),                                              # two chunks a block; 272 blocks
    (4, 704, 64, 64, 4),                                                                    # 132 blocks of 64 x 64: one workgroup each
])
def test_many_tied_blocks_repeat_bit_for_bit(T, H, K, B, waves):
    w = W.hmm(T, H, 20, K, B, 99, alpha_trans=0.1)
    print(f"case ordered parameter flows T={T} H={H} K={K} B={B}", flush=True)
    assert param_workgroups(w) == (w.n_param_blocks * waves + 3) // 4
    check_all(w, (np.random.default_rng(5).random(w.x.shape) < 0.2).astype(np.uint8))
    runs = [gpu_run(w) for _ in range(3)]
    for r in runs[1:]: assert np.array_equal(r["theta_flow"], runs[0]["theta_flow"])
    for r in runs: r["circuit"].close()


@pytest.mark.parametrize("T,H,B,workgroups", [
    (8, 32, 20, 2), (16, 32, 1, 4), (8, 64, 32, 8),                      # one chunk a pair: as many waves as pairs,
    (64, 32, 30, 12),                                                    # up to 24 a block
    (16, 32, 128, 8), (16, 64, 100, 30), (64, 96, 60, 69), (16, 32, 512, 32),   # two chunks a wave; four; 64 waves a block
])
def test_chunks_dealt_to_waves_match_oracle(T, H, B, workgroups):
    w = W.hmm(T, H, 20, 32, B, 100, alpha_trans=0.1)
    print(f"case chunks dealt to waves T={T} H={H} B={B}", flush=True)
    assert param_workgroups(w) == workgroups
    check_all(w, (np.random.default_rng(6).random(w.x.shape) < 0.2).astype(np.uint8))


@pytest.mark.parametrize("T,H,K,B,workgroups", [
    (4, 64, 64, 128, 2 * 4), (4, 128, 128, 100, 2 * 4),                  # two chunks each while there are few workgroups
    (64, 128, 64, 100, 6 * 42), (64, 256, 128, 70, 6 * 42),              # 42 pairs and 168 or 126 chunks a block: a workgroup a pair
    (16, 256, 64, 300, 20 * 25), (16, 512, 128, 100, 20 * 12), (16, 512, 128, 300, 20 * 24),   # few a block: two chunks at K = 64, five at 128
    (40, 128, 64, 512, 6 * 52),                                          # more than 32: eight (421 a block)
])
def test_chunks_dealt_to_workgroups_match_oracle(T, H, K, B, workgroups):
    w = W.hmm(T, H, 20, K, B, 102, alpha_trans=0.1)
    print(f"case chunks dealt to workgroups T={T} H={H} K={K} B={B}", flush=True)
    assert param_workgroups(w) == workgroups
    check_all(w, (np.random.default_rng(7).random(w.x.shape) < 0.2).astype(np.uint8))

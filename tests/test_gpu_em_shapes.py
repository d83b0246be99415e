"""EM step at the sizes where its kernels change: rows held in registers or read twice, tables held by workgroups of 256, 512
and 1024 threads or shared out, against the oracle's update."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import pc_oracle as orc
from paper_2406_00766_amd import binding as pcb
from paper_2406_00766_amd import workloads as W
from tests.test_gpu_dataflow import Dag

pytestmark = pytest.mark.gpu


def mixture(K, n, n_real=1, unused=0):
    """One sum block over n products of one input; parameter blocks that no edge uses, at the end."""
    d = Dag(K)
    i = d.input()
    root = d.sum([d.product([i]) for _ in range(n)], n_real=n_real)
    d.n_params += unused
    return d.workload(root, 4, 87)


@pytest.mark.parametrize("make", [
    lambda: W.rat_spn(32, 2, 4, 256, 32, 20, 81, n_cats=6),        # the root's row: 256 blocks, more than registers hold
    lambda: W.hmm(3, 2048, 20, 32, 20, 82),                        # rows of 64 blocks, tied
    lambda: W.hclt(64, 64, 64, 20, 83, n_cats=401),                # tables of 401 x 64: 512 threads
    lambda: W.hclt(64, 64, 64, 20, 84, n_cats=1000),               # 1024 threads
    lambda: W.hclt(64, 64, 64, 20, 85, n_cats=1030),               # shared out
    lambda: W.hmm(4, 16, 2000, 8, 40, 86),                         # few tables of 2000 x 8: shared out
    lambda: mixture(32, 256),                                      # the longest row that one wave takes, and nothing else
    lambda: mixture(32, 257, n_real=3, unused=2),                  # the shortest in segments: the last one is one block
    lambda: mixture(6, 342, n_real=6),                             # the same in accesses of one column
    lambda: mixture(1, 262145),                                    # more than 1024 x 256 accesses: segments longer than registers
])
def test_em_kernel_shapes(make):
    w = make()
    print(f"case em {w.name}", flush=True)
    c = pcb.Circuit(w)
    rng = np.random.default_rng(8)
    c.theta_flow.copy_(torch.from_numpy((rng.random(w.theta.size) * (w.theta.ravel() > 0)).astype(np.float32)))
    c.table_flow.copy_(torch.from_numpy(rng.random(w.tables.size).astype(np.float32)))
    tf, gf = (t.double().cpu().numpy() for t in (c.theta_flow, c.table_flow))
    ref_th, ref_tb = orc.em_step(w, w.theta, w.tables, tf.reshape(w.theta.shape), gf.reshape(w.tables.shape), step=0.4, pseudocount=0.05)
    c.em_step(0.4, 0.05)
    torch.cuda.synchronize()
    assert np.allclose(c.theta.cpu().numpy().reshape(w.theta.shape), ref_th, rtol=1e-4, atol=1e-9)
    assert np.allclose(c.tables.cpu().numpy().reshape(w.tables.shape), ref_tb, rtol=1e-4, atol=1e-9)
    assert float(c.theta_flow.abs().max()) == 0.0 and float(c.table_flow.abs().max()) == 0.0
    c.close()


def test_rows_of_many_blocks_are_shared_out():
    """One row of 10000 blocks: theta and flows are read and written (the flows read twice) at a tenth of the copy rate (5.5 TB/s)
    or better; 20 us for the launches."""
    w = mixture(32, 10000)
    print(f"case em {w.name}", flush=True)
    c = pcb.Circuit(w)
    c.em_step(0.1, 0.01)
    pcb.pc_profile_enable(c.handle, True)
    c.em_step(0.1, 0.01)
    us = 1e3 * pcb.pc_profile_read(c.handle)["em"][1]
    print(f"  {us:.0f} us", flush=True)
    assert us < 20 + 1e6 * 5 * 4 * w.theta.size / 0.55e12
    c.close()

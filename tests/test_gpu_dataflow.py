"""Narrow layers run as dataflow launches (all of them in one launch per direction): against the oracle where the kernels'
shapes change -- neighbour chunks per wave, several batches of chunks, lists longer than a record, a cut in the middle of
the circuit, a single sample, masked and out-of-range values -- and from the profile, that those layers shared a launch."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2406_00766_amd import binding as pcb
from paper_2406_00766_amd import workloads as W
from tests.test_gpu_parity import check_all

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("make", [
    lambda: W.hmm(9, 32, 20, 32, 1, 71),                       # one chunk of 32 neighbour nodes per row, one sample
    lambda: W.hclt(40, 128, 64, 33, 72, n_cats=16),            # four chunks
    lambda: W.hmm(5, 256, 40, 128, 70, 73),                    # eight
    lambda: W.hmm(4, 512, 30, 64, 40, 74, alpha_trans=0.1),    # sixteen: two per wave
    lambda: W.hmm(3, 1184, 30, 32, 20, 75, alpha_trans=0.05),  # 37: three batches, the last one partly empty
    lambda: W.sum_layer(11, 64, 32, 50, 76, keep=0.6, n_cats=9),   # product blocks of eleven children
    lambda: W.hclt(300, 64, 32, 300, 77, n_cats=8),            # wide layers below the cut, children on both sides of it
    lambda: W.random_circuit(5, 6, 5, 64, 45, 78),             # skip connections, ties, unused blocks
])
def test_dataflow_layers_match_oracle(make):
    w = make()
    print(f"case dataflow {w.name}", flush=True)
    rng = np.random.default_rng(7)
    mask = (rng.random(w.x.shape) < 0.15).astype(np.uint8)
    x = w.x.copy()
    if w.B > 4:
        x[3, 0] = w.n_cats + 2; mask[3, 0] = 0                 # a sample of probability 0
    w = w.with_batch(x)
    check_all(w, mask)
    c = pcb.Circuit(w)
    c.set_batch(w.x)
    pcb.pc_profile_enable(c.handle, True)
    c.forward(); c.backward()
    prof = pcb.pc_profile_read(c.handle)
    n_sum = sum(pcb.pc_get_layer(c.handle, i).kind == 2 for i in range(c.sizes.n_layers))
    assert prof["sum_fwd"][0] < n_sum and prof["sum_bwd_child"][0] < n_sum
    c.close()

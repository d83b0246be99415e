"""Sum layers of few tiles and long rows: their reductions are split over up to sixteen waves, by a rule on chunks of 32
neighbour nodes.  Against the oracle on both sides of that rule's lines, both directions, one and several table groups."""
import pytest

torch = pytest.importorskip("torch")

from paper_2406_00766_amd import binding as pcb
from paper_2406_00766_amd import workloads as W
from tests.refs import kernels
from tests.test_gpu_dataflow import Dag
from tests.test_gpu_parity import check_all

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,widths,B,waves", [
    (32, [15] * 3, 20, (4, 2)), (32, [16] * 16, 33, (8, 8)), (32, [31] * 9, 1, (8, 4)), (32, [33] * 33, 40, (16, 16)),
    (64, [8] * 7, 50, (8, 4)), (64, [17] * 17, 3, (16, 16)), (128, [4] * 4, 60, (8, 8)), (128, [9] * 9, 20, (16, 16)),
    (32, [3, 20, 37], 70, (16, 2)), (64, [2, 18], 1, (16, 4)), (128, [9, 1, 2], 33, (16, 4)),   # several groups in a launch
    (32, [40] * 64, 200, (8, 8)),                                                               # tiles enough: fewer waves again
])
def test_split_reductions_match_oracle(K, widths, B, waves):
    """Waves that share a tile forward and backward.  Sum blocks over products of thirteen inputs (too many for a dataflow launch), one single-child product over each, a root."""
    d = Dag(K)
    inputs = [d.input() for _ in range(13)]
    products = [d.product(inputs) for _ in range(max(widths))]
    sums = [d.sum(products[:n]) for n in widths]
    w = d.workload(d.sum([d.product([s]) for s in sums], n_real=1), B, 91)
    print(f"case split K={K} widths={widths[:3]}x{len(widths)} B={B}", flush=True)
    for direction, n in enumerate(waves):
        assert kernels(w, direction)[2] == f"k_sum_mfma<{K}, 1, {n}, {'true' if direction else 'false'}>"
    check_all(w)


@pytest.mark.parametrize("K,width,B,parts", [
    (32, 63, 20, False), (32, 64, 20, True), (32, 81, 70, True),       # 81 chunks in ten parts of nine: the last is empty
    (64, 40, 33, True), (128, 17, 100, True), (32, 300, 1, True),
    (32, 64, 1024, True), (32, 64, 1025, False), (128, 16, 256, True), (128, 16, 257, False),   # 32 tiles and more
])
@pytest.mark.parametrize("scratch", [False, True])
def test_root_in_parts_matches_oracle(K, width, B, parts, scratch):
    """A root over many products of thirteen inputs, its row in parts of several workgroups; a sample of probability 0."""
    d = Dag(K)
    tables = [[d.input() for _ in range(13)] for _ in range(3)]
    w = d.workload(d.sum([d.product(tables[i % 3][:13 - i % 2]) for i in range(width)], n_real=1), B, 92)
    if scratch:
        w = pcb.pc_order_for_scratch(w)
    print(f"case root in parts K={K} width={width} B={B} scratch={scratch}", flush=True)
    assert (kernels(w, 0)[2] == f"k_sum_mfma<{K}, 1, 4, false, false, 3>") == parts
    x = w.x.copy()
    x[0, 0] = w.n_cats + 2
    check_all(w.with_batch(x))


@pytest.mark.parametrize("K,width,B", [(32, 81, 70), (64, 40, 33), (128, 17, 100)])
@pytest.mark.parametrize("scratch", [False, True])
def test_flows_outlive_the_next_forward_pass(K, width, B, scratch):
    """The parts of a root's row lie where no node buffer is: a forward pass leaves the flows of the batch before."""
    d = Dag(K)
    tables = [[d.input() for _ in range(13)] for _ in range(3)]
    w = d.workload(d.sum([d.product(tables[i % 3][:13 - i % 2]) for i in range(width)], n_real=1), B, 93)
    if scratch:
        w = pcb.pc_order_for_scratch(w)
    print(f"case flows outlive K={K} width={width} B={B} scratch={scratch}", flush=True)
    assert kernels(w, 0)[2] == f"k_sum_mfma<{K}, 1, 4, false, false, 3>"
    c = pcb.Circuit(w)
    c.set_batch(w.x)
    c.forward(); c.backward()
    F = c.node_buffers()[1]
    if scratch: F = F[:(1 + (w.type != W.PRODUCT).sum()) * K]          # product rows are not kept
    before = F.clone()
    assert before.abs().sum() > 0
    c.forward()
    assert torch.equal(F, before)
    c.close()

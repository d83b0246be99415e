"""Narrow layers run as dataflow launches (all of them in one launch per direction): against the oracle where the kernels'
shapes change -- neighbour chunks per wave, several batches of chunks, lists longer than a record, a cut in the middle of
the circuit, a single sample, masked and out-of-range values -- and from the profile, that those layers shared a launch."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2406_00766_amd import binding as pcb
from paper_2406_00766_amd import workloads as W
from tests.refs import kernels
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


@pytest.mark.parametrize("K,H,B,waves,tiles,chunks", [
    (64, 64, 512, 2, 1, 1), (64, 64, 513, 2, 2, 1),            # two chunks: 128 tasks of 16 rows in a layer, then 32 rows
    (32, 128, 256, 4, 1, 1), (32, 128, 257, 4, 2, 1),          # four chunks
    (64, 256, 128, 8, 1, 1), (64, 256, 129, 8, 2, 1),          # eight
    (64, 512, 64, 8, 1, 2), (64, 512, 65, 8, 2, 2),            # sixteen: two per wave
    (128, 640, 16, 8, 1, 4), (128, 640, 65, 8, 2, 4),          # twenty: up to four per wave
])
def test_tile_shapes_match_oracle(K, H, B, waves, tiles, chunks):
    """HMMs on both sides of the line between row tiles of 16 and 32, for every number of waves from two on and chunks per wave."""
    w = W.hmm(4, H, 30, K, B, 90, alpha_trans=0.2)
    print(f"case tile shape K={K} H={H} B={B}", flush=True)
    assert kernels(w, 0)[4] == f"k_flow<{waves}, {tiles}, {chunks}, false, false>"
    assert kernels(w, 1)[4] == f"k_flow<{waves}, {tiles}, {chunks}, true, false>"
    check_all(w)


class Dag(W._Builder):
    """Block DAGs written out by hand: every edge of a sum block has a parameter block of its own."""
    n_params = 0

    def input(self):
        n = sum(t == W.INPUT for t in self.type)
        return self.add(W.INPUT, var=n, table=n)

    def product(self, children):
        p = self.add(W.PRODUCT)
        for c in children:
            self.link(p, c)
        return p

    def sum(self, children, n_real=None):
        s = self.add(W.SUM, n_real=n_real)
        for c in children:
            self.link(s, c, self.n_params)
            self.n_params += 1
        return s

    def workload(self, root, B, seed, n_cats=5, table_alpha=1.0):
        rng = np.random.Generator(np.random.PCG64(seed))
        K, n = self.K, sum(t == W.INPUT for t in self.type)
        theta = np.zeros((self.n_params + 1, K, K), dtype=np.float32)
        for s in range(len(self.type)):
            if self.type[s] == W.SUM:
                ids, rows = self.params[s], self.n_real[s]
                w = W._f32_floor(W._dirichlet_rows(rng, 1.0, (rows, len(ids) * K)))
                for j, p in enumerate(ids):
                    theta[p + 1, :rows] = w[:, j * K:(j + 1) * K]
        tables = np.ascontiguousarray(np.stack([W._f32_floor(W._dirichlet_rows(rng, table_alpha, (K, n_cats))).T for _ in range(n)]))
        return W._make(f"dag_{seed}", self, root, self.n_params, n, n_cats, n, theta, tables, rng.integers(0, n_cats, size=(B, n)), {})


def parallel_lines(B):
    """Five lines of four sum blocks, each over one product of the block before and eight inputs, that meet in one product."""
    d = Dag(32)
    ends = [d.input() for _ in range(5)]
    for _ in range(4):
        ends = [d.sum([d.product([s] + [d.input() for _ in range(8)])]) for s in ends]
    return d.workload(d.sum([d.product(ends)], n_real=1), B, 97)


@pytest.mark.parametrize("make,B,tiles,exact", [
    (lambda B: W.hclt(16, 32, 32, B, 96, n_cats=8), 100, 1, False), (lambda B: W.hclt(16, 32, 32, B, 96, n_cats=8), 300, 2, False),
    (parallel_lines, 192, 1, True), (parallel_lines, 193, 2, True),      # 120 and 140 tasks of 16 rows
])
def test_rows_of_one_block_match_oracle(make, B, tiles, exact):
    """One wave per task (rows of one neighbour block of 32 nodes, several blocks a layer): row tiles of 16 and 32, products of
    few children and of nine."""
    w = make(B)
    print(f"case one wave {w.name} B={B}", flush=True)
    for direction, e in ((0, exact), (1, False)):
        want = f"k_flow<1, {tiles}, 1, {'true' if direction else 'false'}, {'true' if e else 'false'}>"
        assert [k for k in kernels(w, direction) if k.startswith(("k_sum", "k_flow", "k_chain"))].count(want) > 2
    check_all(w)


@pytest.mark.parametrize("make,tiles", [
    (lambda: W.pd(4, 3, 128, 64, 33, 98, keep=1.0, n_cats=8), 2), (lambda: W.rat_spn(24, 2, 4, 128, 64, 1, 99, n_cats=8), 1),
])
def test_long_rows_of_products_with_many_children_match_oracle(make, tiles):
    """More than sixteen chunks a row over products of nine inputs and more: two chunks per wave at once (four spill registers)."""
    w = make()
    print(f"case long rows {w.name}", flush=True)
    assert f"k_flow<8, {tiles}, 2, false, true>" in kernels(w, 0)
    check_all(w)


@pytest.mark.parametrize("K,B", [(32, 20), (64, 1)])
def test_root_below_the_dataflow_layers(K, B):
    """A root over a product of thirteen inputs (its layer is not one for a dataflow launch) beside a deeper chain that nothing
    reads (its layers are): ll still comes from the root, and the chain's flows are 0."""
    d = Dag(K)
    inputs = [d.input() for _ in range(14)]
    root = d.sum([d.product(inputs[:13])], n_real=1)
    s = inputs[13]
    for _ in range(4):
        s = d.sum([d.product([s])])
    w = d.workload(root, B, 79)
    print(f"case shallow root K={K} B={B}", flush=True)
    check_all(w)
    c = pcb.Circuit(w)
    c.set_batch(w.x)
    c.ll.fill_(float("nan"))
    pcb.pc_profile_enable(c.handle, True)
    ll = c.forward()
    assert not torch.isnan(ll).any()
    assert pcb.pc_profile_read(c.handle)["sum_fwd"][0] < 4                 # four sum layers, the upper three in one launch
    c.close()


@pytest.mark.parametrize("K,H,B", [(32, 32, 1), (64, 512, 40)])     # one wave per task, eight waves that meet in LDS
def test_wait_that_is_given_up_is_visible(K, H, B):
    """A wait given up (limit 0: at the first value that is not there yet) leaves NaN, never a finite wrong result, and the
    handle's next call returns the error; forward and backward, each on a handle of its own."""
    w = W.hmm(24, H, 20, K, B, 80)
    print(f"case wait limit K={K} H={H} B={B}", flush=True)

    def refused(call):
        with pytest.raises(pcb.PcError) as e:
            call()
        assert e.value.status_name == "PC_ERR_HIP"

    other_handle = pcb.Circuit(w)
    c = pcb.Circuit(w)
    c.set_batch(w.x)
    ref = c.forward().clone()
    pcb.pc_set_wait_limit(c.handle, 0)
    c.forward()
    torch.cuda.synchronize()
    same = c.ll == ref
    assert torch.isnan(c.ll[~same]).all() and not same.all()
    refused(c.forward)
    refused(lambda: c.em_step(0.1, 0.0))
    c.close()

    c = pcb.Circuit(w)
    c.set_batch(w.x)
    c.forward(); c.backward()
    torch.cuda.synchronize()
    F_ref, table_ref = c.node_buffers()[1].clone(), c.table_flow.clone()
    c.table_flow.zero_()
    pcb.pc_set_wait_limit(c.handle, 0)
    c.backward()
    torch.cuda.synchronize()
    F = c.node_buffers()[1]
    other = F[:, :B] != F_ref[:, :B]
    assert other.any() and torch.isnan(F[:, :B][other]).all()
    assert torch.isnan(c.table_flow[~torch.isclose(c.table_flow, table_ref, rtol=1e-4, atol=0)]).all() and torch.isnan(c.table_flow).any()
    refused(lambda: c.em_step(0.1, 0.0))
    refused(c.backward)
    other_handle.set_batch(w.x)                                # the error is the handle's own
    assert torch.equal(other_handle.forward(), ref)
    other_handle.close(); c.close()


def test_more_handles_than_fault_words():
    w = W.hmm(3, 32, 5, 32, 1, 82)
    handles = [pcb.pc_compile(w) for _ in range(1027)]
    c = pcb.Circuit(w)                                          # one whose word is its own
    c.set_batch(w.x)
    ref = c.forward().clone()
    for h in handles:
        pcb.pc_destroy(h)
    assert torch.equal(c.forward(), ref)
    c.close()


@pytest.mark.parametrize("K,n_in,n_sum", [(32, 9, 0), (32, 12, 0), (128, 12, 0), (64, 7, 5)])
def test_products_of_many_children_keep_their_precision(K, n_in, n_sum):
    """Products of nine to twelve children with log-probabilities of some -80 nats, the next sum layer's values against the same
    sums in 64 bits from the children's rows as stored.  With the products exact to their last bit, what is left is: the
    exponential's argument (below 32, half an ulp 9.5e-7, times ln 2 0.7e-6), its v rounded once (below 8 nats: 2.4e-7), one ulp
    of the exponential (1.2e-7) and of the logarithm (an argument below 16: 9.5e-7 ln 2 = 0.7e-6), the products' sum (a few
    6e-8) and the result's own rounding (below 8: 2.4e-7) -- 2.2e-6, bound 4e-6.  Products summed in fp32 miss it: -80 x 3 alone
    is rounded to 1.5e-5."""
    d = Dag(K)
    kids = [d.input() for _ in range(n_in)] + [d.sum([d.product([d.input()])]) for _ in range(n_sum)]
    mid = d.sum([d.product(kids)])
    root = d.sum([d.product([mid])], n_real=1)
    B = 40
    w = d.workload(root, B, 81)
    rng = np.random.default_rng(5)
    t = np.exp(-80 + rng.uniform(-1, 1, size=w.tables.shape))
    t[:, -1] = 1.0 - t[:, :-1].sum(axis=1)
    w.tables = t.astype(np.float32)
    th = (0.97 * np.eye(K) + 0.03 / K).astype(np.float32)               # node i is nearly child i
    for s in range(len(d.type)):
        if d.type[s] == W.SUM and s != root:
            w.theta[d.params[s][0] + 1] = th
    w = w.with_batch(rng.integers(0, w.n_cats - 1, size=w.x.shape))
    print(f"case precise products K={K} {n_in}+{n_sum}", flush=True)
    c = pcb.Circuit(w)
    c.set_batch(w.x)
    pcb.pc_profile_enable(c.handle, True)
    c.forward()
    assert pcb.pc_profile_read(c.handle)["sum_fwd"][0] == 1              # one dataflow launch
    l, _, R = (t[:, :B].double().cpu().numpy() for t in c.node_buffers())
    rows = lambda u: R[u + 1] + l[(u + 1) * K:(u + 2) * K]
    p = sum(rows(u) for u in kids)
    top = p.max(axis=0)
    ref = top + np.log(th.astype(np.float64) @ np.exp(p - top))
    err = np.abs(rows(mid) - ref).max()
    print(f"  largest error {err:.2e}")
    assert err < 4e-6
    c.close()


@pytest.mark.parametrize("K,B", [(128, 65536), (16, 262144), (32, 33), (32, 65536), (64, 65536)])
def test_null_block_is_filled_by_many_workgroups(K, B):
    """The null block's K x B zeros are written whatever the workspace held, and the launches beside the layers take no longer
    than 20 us and the time of these zeros at a tenth of the copy rate (5.5 TB/s), the three input blocks of K x B values with them
    where the launch that begins the pass writes those as well."""
    w = W.hmm(3, K, 5, K, 64, 83)
    w = w.with_batch(np.tile(w.x, (-(-B // 64), 1))[:B])
    print(f"case null block K={K} B={B}", flush=True)
    c = pcb.Circuit(w)
    c.set_batch(w.x)
    c.forward()                                                 # (first launches load the kernels)
    c._ws.fill_(0xFF)                                           # NaN everywhere
    pcb.pc_profile_enable(c.handle, True)
    ll = c.forward()
    prof = pcb.pc_profile_read(c.handle)
    joined = pcb.pc_get_kernel(c.handle, 0, 0, B).startswith("k_begin_forward")
    begin = prof["input_fwd"] if joined else prof["misc"]
    assert begin[0] >= 1 and joined == (K in (32, 64))
    us = 1e3 * (prof["misc"][1] + (prof["input_fwd"][1] if joined else 0.0))
    l, _, R = c.node_buffers()
    assert (l[:K] == 0).all() and (R[0] == 0).all()
    assert torch.equal(ll, ll[:64].repeat(-(-B // 64))[:B]) and torch.isfinite(ll).all()
    print(f"  {us:.0f} us", flush=True)
    assert us < 20 + 1e6 * 4 * K * B * (4 if joined else 1) / 0.55e12
    c.close()


def test_published_blocks_are_filled_by_many_workgroups():
    """Seventeen blocks of 1 MiB: the launch that writes them takes no longer than a launch that writes nothing (6.3 us between
    two events, here 7) and its bytes at half the copy rate (5.5 TB/s); the shortest of ten."""
    w = W.hmm(16, 128, 50, 128, 64, 84)
    w = w.with_batch(np.tile(w.x, (32, 1)))
    c = pcb.Circuit(w)
    c.set_batch(w.x)
    ref = c.forward().clone()
    us = []
    for _ in range(10):
        pcb.pc_profile_enable(c.handle, True)
        c.forward()
        us.append(1e3 * pcb.pc_profile_read(c.handle)["misc"][1])
    print(f"case fills {min(us):.1f} us", flush=True)
    assert torch.equal(c.ll, ref) and torch.equal(ref, ref[:64].repeat(32))
    assert min(us) < 7 + 1e6 * 4 * 17 * 128 * w.B / 2.75e12
    c.close()


def layered(K, n_sum, n_prod, depth, B, seed):
    """Levels of n_sum sum blocks, each of which feeds n_prod products (with an input of their own) that the whole next level reads."""
    d = Dag(K)
    level = [d.sum([d.product([d.input()])]) for _ in range(n_sum)]
    for _ in range(depth):
        products = [d.product([s, d.input()]) for s in level for _ in range(n_prod)]
        level = [d.sum(products) for _ in range(n_sum)]
    root = d.sum([d.product([s]) for s in level], n_real=1)
    return d.workload(root, B, seed)


@pytest.mark.parametrize("K,n_sum,n_prod,B,merged", [
    (32, 1, 8, 30, True), (32, 1, 30, 30, False), (32, 1, 30, 300, False), (64, 4, 2, 30, True), (128, 1, 24, 60, False),
])
def test_sum_blocks_that_feed_many_products(K, n_sum, n_prod, B, merged):
    """A dataflow task of the backward pass takes the product parents of its sum blocks one after the other: where a sum block has
    many, these layers keep their own launches in that direction (six levels, and the read-out's product), whatever the forward
    pass does; against the oracle."""
    w = layered(K, n_sum, n_prod, 6, B, 85)
    print(f"case many readers K={K} {n_sum} x {n_prod} B={B}", flush=True)
    check_all(w)
    c = pcb.Circuit(w)
    c.set_batch(w.x)
    pcb.pc_profile_enable(c.handle, True)
    c.forward()
    c.backward()
    prof = pcb.pc_profile_read(c.handle)
    assert prof["sum_fwd"][0] == 1 if K == 32 else prof["sum_fwd"][0] >= 1
    assert prof["sum_bwd_child"][0] < 3 if merged else prof["sum_bwd_child"][0] >= 6
    c.close()


@pytest.mark.parametrize("T,K,B,merged", [(16, 32, 512, True), (16, 32, 16384, False), (3, 128, 4096, False), (16, 128, 4096, False),
                                          (3, 64, 512, True)])
def test_layers_of_many_column_tiles_keep_their_launches(T, K, B, merged):
    """Narrow circuits at large batches: 2048 tiles a layer take longer as tasks than as launches.  Equal samples have equal
    log-likelihoods wherever they stand in the batch, and those of the same batch in small parts."""
    w = W.hmm(T, K, 50, K, 64, 86)
    big = w.with_batch(np.tile(w.x, (B // 64, 1)))
    print(f"case many tiles T={T} K={K} B={B}", flush=True)
    c = pcb.Circuit(w)
    c.set_batch(w.x)
    ref = c.forward().double().cpu()
    c.set_batch(big.x)
    pcb.pc_profile_enable(c.handle, True)
    ll = c.forward().double().cpu()
    assert pcb.pc_profile_read(c.handle)["sum_fwd"][0] == (1 if merged else T)
    assert torch.equal(ll, ll[:64].repeat(B // 64))
    assert ((ll[:64] - ref).abs() <= 1e-6 * ref.abs() + 4e-6).all()      # results are held to some 1e-6 (pc.h), R is exact
    c.close()

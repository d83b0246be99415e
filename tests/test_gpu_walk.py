"""Chains of single blocks walked with a wave per column: both sides of the batch sizes where the kernel changes, more links than a
lane holds rows of (64), weights that change with every link, and the pass of pc_forward_static in one launch, where the circuit is nothing but
a chain; kernels asserted, those of a static pass from a capture of it."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import pc_oracle as orc
from paper_2406_00766_amd import binding as pcb
from paper_2406_00766_amd import workloads as W
from tests.refs import kernels, launches
from tests.test_gpu_dataflow import Dag
from tests.test_gpu_parity import assert_logprob_close, check_all, check_repeated

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,T,B,reps,names", [
    (32, 3, 64, 32, ("k_chain<false>", "k_chain<true>")), (32, 3, 64, 33, ("k_chain_wide<false>", "k_chain_wide<true>")),
    (64, 16, 16, 256, ("k_walk64<false>", "k_walk64<true>")), (64, 16, 16, 258, ("k_flow<", "k_flow<")),
    (32, 70, 33, 1, ("k_chain<false>", "k_chain<true>")), (64, 67, 9, 1, ("k_walk64<false>", "k_walk64<true>")),
])
def test_walked_chains_match_oracle(K, T, B, reps, names):
    w = W.hmm(T, K, 30, K, B, 96, alpha_trans=0.3)
    print(f"case walk K={K} T={T} B={B} x {reps}", flush=True)
    for direction in (0, 1):
        assert any(k.startswith(names[direction]) for k in kernels(w, direction, B * reps))
    check_repeated(w, reps, (np.random.default_rng(8).random(w.x.shape) < 0.2).astype(np.uint8))


@pytest.mark.parametrize("K,B,name", [(32, 256, "k_chain<"), (32, 257, "k_chain_wide<"), (64, 256, "k_walk64<"), (64, 257, "k_flow<")])
def test_chains_of_many_weights(K, B, name):
    d = Dag(K)
    s = d.sum([d.product([d.input()])])
    for _ in range(9): s = d.sum([d.product([s, d.input()])])
    w = d.workload(d.sum([d.product([s, d.input()])], n_real=1), B, 97)
    print(f"case many weights K={K} B={B}", flush=True)
    for direction in (0, 1): assert any(k.startswith(name) for k in kernels(w, direction))
    check_all(w)


def static_kernels(c):
    ll = torch.empty(c.B, device="cuda")
    return [k[0] for k in launches(lambda stream: pcb.pc_forward_static(c.handle, c.theta, c.tables, c.x, c.mask, c.B, ll, stream))]


@pytest.mark.parametrize("K,T,B", [(32, 16, 1), (32, 130, 3), (64, 64, 2), (64, 65, 300), (32, 5, 511)])
def test_static_pass_in_one_launch(K, T, B):
    """The same numbers as pc_forward, with masked variables, a category out of range and nothing read from the workspace."""
    w = W.hmm(T, K, 30, K, B, 98, alpha_trans=0.3)
    x, mask = w.x.copy(), (np.random.default_rng(9).random(w.x.shape) < 0.3).astype(np.uint8)
    if B > 2: x[2, T - 1] = -7; mask[2, T - 1] = 0
    c = pcb.Circuit(w)
    c.set_batch(x, mask)
    ref = c.forward().clone()
    ll = torch.full_like(ref, float("nan"))
    print(f"case static walk K={K} T={T} B={B}", flush=True)
    pcb.pc_forward_static(c.handle, c.theta, c.tables, c.x, c.mask, B, ll)
    torch.cuda.synchronize()
    assert torch.equal(ll, ref) and (B <= 2 or ll[2] == -float("inf")) and torch.isfinite(ll).sum() >= B - 1
    assert static_kernels(c) == [f"k_walk_pass<{K}>"]
    c.close()


@pytest.mark.parametrize("kind,one", [("untied", True), ("shared_input", False), ("bare_sum", False), ("unused_input", False), ("wait_limit", False)])
@pytest.mark.parametrize("K,T,B", [(32, 70, 5), (64, 67, 33), (32, 9, 256)])
def test_static_pass_of_chains_and_others_matches_oracle(K, T, B, kind, one):
    """Weights that change with every link, also where a lane's rows run out; circuits that a chain's walk from the tables does not cover."""
    d = Dag(K)
    first = d.input()
    s = d.sum([d.product([first])])
    for i in range(T - 2):
        if kind == "bare_sum" and i == 2: s = d.sum([d.product([s])])
        else: s = d.sum([d.product([s, first if kind == "shared_input" and i == 2 else d.input()])])
    if kind == "unused_input": d.input()
    w = d.workload(d.sum([d.product([s, d.input()])], n_real=1), B, 101)
    mask = (np.random.default_rng(10).random(w.x.shape) < 0.2).astype(np.uint8)
    w.x[1, 0] = w.n_cats; mask[1, 0] = 0
    print(f"case static pass {kind} K={K} T={T} B={B}", flush=True)
    c = pcb.Circuit(w)
    c.set_batch(w.x, mask)
    if kind == "wait_limit": pcb.pc_set_wait_limit(c.handle, 1 << 21)
    ll = torch.full((B,), float("nan"), device="cuda")
    pcb.pc_forward_static(c.handle, c.theta, c.tables, c.x, c.mask, B, ll)
    assert_logprob_close(ll.double().cpu().numpy(), orc.forward(w, w.theta, w.tables, w.x, mask)[1], "ll")
    found = static_kernels(c)
    assert (found == [f"k_walk_pass<{K}>"]) == one and (one or len(found) > 1)
    c.close()


@pytest.mark.parametrize("K,T,B,untied,names,workgroups,threads", [
    (32, 5, 512, False, "k_chain", 256, 64), (32, 5, 513, False, "k_chain", 136, 128), (32, 5, 1025, False, "k_chain", 132, 256),
    (64, 7, 256, False, "k_walk64", 256, 64), (64, 7, 257, False, "k_walk64", 144, 128), (64, 7, 513, False, "k_walk64", 136, 256),
    (64, 5, 225, False, "k_walk64", 256, 64), (64, 7, 256, True, "k_walk64", 256, 64), (32, 7, 256, True, "k_chain", 128, 64),
])
def test_workgroups_of_walks(K, T, B, untied, names, workgroups, threads):
    """A wave to a workgroup while there are no more of them than CUs, then two, then four."""
    if untied:
        d = Dag(K)
        s = d.sum([d.product([d.input()])])
        for _ in range(T - 2): s = d.sum([d.product([s, d.input()])])
        w = d.workload(d.sum([d.product([s, d.input()])], n_real=1), B, 99)
    else:
        w = W.hmm(T, K, 30, K, B, 99, alpha_trans=0.3)
    print(f"case workgroups of walks K={K} T={T} B={B} untied={untied}", flush=True)
    c = pcb.Circuit(w)
    c.set_batch(w.x)
    c.forward()
    for bwd in (False, True):
        def call(stream):
            with torch.cuda.stream(stream): c.backward() if bwd else c.forward()
        assert (f"{names}<{str(bwd).lower()}>", workgroups, 1, 1, threads) in launches(call)
    c.close()
    check_all(w)


def test_short_chains_of_64_leave_the_walk_at_2048():
    for T, B, name in ((7, 2048, "k_walk64<"), (7, 2049, "k_flow<"), (8, 2049, "k_walk64<")):
        assert any(k.startswith(name) for k in kernels(W.hmm(T, 64, 30, 64, 2, 99), 0, B)), (T, B)

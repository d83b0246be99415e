"""Chains of single blocks of 32 and 64 nodes, walked layer by layer (k_chain and k_walk64, a wave per column; k_chain_wide, one per sixteen):
against the oracle with one link and many, one sample to several waves, masked and impossible values; HMMs of several blocks and circuits
that are almost chains, which are not theirs.  The kernels are asserted."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2406_00766_amd import workloads as W
from tests.refs import kernels
from tests.test_gpu_dataflow import Dag
from tests.test_gpu_parity import check_all

pytestmark = pytest.mark.gpu


def chains(w):
    """Whether the forward and the backward pass walk a chain."""
    return tuple(any(k.startswith(("k_chain", "k_walk64")) for k in kernels(w, direction)) for direction in (0, 1))


@pytest.mark.parametrize("K,H,T,B", [
    (32, 32, 16, 1), (32, 32, 2, 40), (32, 32, 9, 17), (64, 64, 12, 1), (64, 64, 3, 100), (32, 64, 10, 33), (32, 64, 7, 512), (32, 32, 40, 129),
])
def test_chains_match_oracle(K, H, T, B):
    w = W.hmm(T, H, 30, K, B, 94, alpha_trans=0.3)
    print(f"case chain K={K} H={H} T={T} B={B}", flush=True)
    rng = np.random.default_rng(7)
    mask = (rng.random(w.x.shape) < 0.2).astype(np.uint8)
    x = w.x.copy()
    if B > 4:
        x[3, 0] = w.n_cats + 2; mask[3, 0] = 0                 # a sample of probability 0
    assert chains(w) == (K == H, K == H)
    check_all(w.with_batch(x), mask)


@pytest.mark.parametrize("kind", ["untied", "narrowing", "shared_input", "skip", "two_inputs", "unused_sum", "deep_beside_root"])
@pytest.mark.parametrize("K,B", [(32, 37), (64, 20)])
def test_almost_chains_match_oracle(kind, K, B):
    """Chains with parameters of their own in every layer, and structures that a chain's conditions have to tell from one."""
    d = Dag(K)
    new = lambda: d.input()
    s, wide = [d.sum([d.product([new()])])], K == 32
    for k in range(5):
        first = new()
        if kind == "two_inputs" and k == 2: p = [d.product([s[0], first, new()])]
        elif kind == "skip" and k == 3: p = [d.product([s[0], first]), d.product([s0, new()])]   # reads a layer further down
        elif wide and kind in ("narrowing", "shared_input") and k < 3: p = [d.product([s[0], first]), d.product([s[-1], first if kind == "shared_input" else new()])]
        else: p = [d.product([s[0], first])] + [d.product([t]) for t in s[1:]]
        s0 = s[0]
        s = [d.sum(p) for _ in range(2 if wide and kind in ("narrowing", "shared_input") and k < 2 else 1)]
        if kind == "unused_sum" and k == 2: d.sum(p)
    root = d.sum([d.product([s[0], new()])], n_real=1)
    if kind == "deep_beside_root":
        t = d.sum([d.product([s[0]])])
        for _ in range(4): t = d.sum([d.product([t])])
    print(f"case almost a chain {kind} K={K} B={B}", flush=True)
    w = d.workload(root, B, 95)
    a_chain = kind == "untied" or (kind in ("narrowing", "shared_input") and not wide)   # (at K = 64 these two are not built)
    assert chains(w) == (a_chain, a_chain or kind == "two_inputs")      # (two inputs: no matter to flows)
    check_all(w)

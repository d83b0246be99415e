"""CPU checks of the library: it loads, exports what include/pc.h declares, and its host compiler
produces tables that equal the compile oracle's bit for bit (no GPU needed for these calls)."""
import os
import re
import subprocess
import sys

import numpy as np
import pytest

from oracle import compile_oracle as co
from paper_2406_00766_amd import binding as pcb
from paper_2406_00766_amd import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "pc.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(pc_[a-z0-9_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = pcb.lib()
    names = declared_symbols()
    assert {"pc_compile", "pc_forward", "pc_backward", "pc_em_step", "pc_destroy", "pc_last_error"} <= set(names)
    for name in names:
        assert hasattr(lib, name), name
    assert sorted(pcb.EXPORTS) == names


def assert_tables_equal(handle, w):
    ref = co.compile_tables(w)
    got = pcb.compiled_tables(handle)
    assert len(got) == len(ref["layers"])
    for a, b in zip(got, ref["layers"]):
        assert (a["kind"], a["depth"]) == (b["kind"], b["depth"])
        for key in ("fwd", "bwd"):
            assert len(a[key]) == len(b[key]), (a["kind"], a["depth"], key)
            for ga, gb in zip(a[key], b[key]):
                for xa, xb in zip(ga, gb):
                    xb = np.asarray(xb).reshape(xa.shape) if xa.size == np.asarray(xb).size else xb
                    assert xa.dtype == np.int32 and np.array_equal(xa, xb)
    s = pcb.pc_get_sizes(handle)
    assert s.n_rows == ref["n_rows"] and s.K == w.K


CASES = [lambda: W.reduced(i) for i in range(1, 6)] + \
        [lambda: W.config(1), lambda: W.config(1, K=16), lambda: W.config(2, draw=False),
         lambda: W.config(2, K=32, draw=False), lambda: W.config(4, draw=False), lambda: W.config(4, K=32, draw=False),
         lambda: W.hmm(4, 6, 5, 3, 2, 7), lambda: W.pd(3, 1, 4, 1, 2, 8, n_cats=3, keep=0.5),
         lambda: W.rat_spn(16, 2, 2, 8, 4, 2, 14, n_cats=3, draw=False),
         lambda: W.sum_layer(5, 64, 8, 3, 15, keep=0.3, draw=False)] + \
        [(lambda s=s, K=K: W.random_circuit(4, 5, 5, K, 3, 100 + s)) for s in range(6) for K in (1, 4, 32)]


@pytest.mark.parametrize("make", CASES)
def test_host_compile_matches_oracle_bit_for_bit(make):
    w = make()
    h = pcb.pc_compile(w, host_only=True)
    try:
        assert_tables_equal(h, w)
    finally:
        pcb.pc_destroy(h)


@pytest.mark.parametrize("idx", [3, 5])
def test_host_compile_large_configs(idx):
    w = W.config(idx, draw=False)
    h = pcb.pc_compile(w, host_only=True)
    try:
        assert_tables_equal(h, w)
    finally:
        pcb.pc_destroy(h)


RING = """
import resource
import numpy as np
from paper_2406_00766_amd import binding as pcb
from paper_2406_00766_amd import workloads as W
N, K = 16000, 4
b = W._Builder(K)
pairs = {i: [b.add(W.INPUT, var=0, table=0) for _ in range(2)] for i in [*range(0, N, 2), *range(1, N, 2)]}
root = b.add(W.SUM, n_real=1)
for i in range(N):
    p = b.add(W.PRODUCT)
    for c in pairs[i] + pairs[(i + 1) % N]:
        b.link(p, c)
    b.link(root, p, i)
w = W._make("ring", b, root, N, 1, 2, 1, np.zeros((1, K, K), np.float32), np.zeros((1, 2, K), np.float32), np.zeros((1, 1), np.int32), {})
before = resource.getrusage(resource.RUSAGE_SELF).ru_maxrss
pcb.pc_destroy(pcb.pc_compile(w, host_only=True))
print(resource.getrusage(resource.RUSAGE_SELF).ru_maxrss - before)
"""


def test_memory_of_compilation_grows_with_the_circuit():
    """16 000 pairs of input blocks, each in two products, neighbours in a ring: two sets of 8000 classes of equal parents, but only
    16 000 of their 64 M pairs are products.  The compiler's tables for these blocks and edges take a few MB."""
    out = subprocess.run([sys.executable, "-c", RING], cwd=ROOT, check=True, capture_output=True, text=True).stdout
    assert int(out) < 64 * 1024                                # KiB


STARVED = """
import resource
import numpy as np
from paper_2406_00766_amd import binding as pcb
from paper_2406_00766_amd import workloads as W
N, K = 150000, 2
b = W._Builder(K)
s = b.add(W.INPUT, var=0, table=0)
for i in range(N):
    p, t = b.add(W.PRODUCT), b.add(W.SUM, n_real=1 if i == N - 1 else None)
    b.link(p, s)
    b.link(t, p, i)
    s = t
w = W._make("line", b, s, N, 1, 2, 1, np.zeros((1, K, K), np.float32), np.zeros((1, 2, K), np.float32), np.zeros((1, 1), np.int32), {})
pcb.pc_destroy(pcb.pc_compile(W.hmm(2, 2, 3, 2, 1, 0), host_only=True))
now = 1024 * int([line.split()[1] for line in open("/proc/self/status") if line.startswith("VmSize")][0])
resource.setrlimit(resource.RLIMIT_AS, (now + (16 << 20), now + (16 << 20)))
try:
    pcb.pc_compile(w, host_only=True)
except pcb.PcError as e:
    print(e)
"""


def test_compilation_that_runs_out_of_memory_is_an_error():
    """A chain of 300 000 blocks with 16 MiB of address space left: an error status, not the end of the process."""
    r = subprocess.run([sys.executable, "-c", STARVED], cwd=ROOT, capture_output=True, text=True)
    assert r.returncode == 0 and "PC_ERR_ARG: out of host memory" in r.stdout, (r.returncode, r.stdout, r.stderr)


def test_kernel_of_a_layer():
    """pc_get_kernel needs no GPU: the rules on sizes, and its errors."""
    h = pcb.pc_compile(W.hmm(4, 32, 5, 32, 1, 0, draw=False), host_only=True)
    assert [pcb.pc_get_kernel(h, li, 0, 7) for li in range(3)] == ["k_begin_forward<32>", "k_prod_fwd", "k_chain<false>"]
    assert [pcb.pc_get_kernel(h, li, 1, 7) for li in range(3)] == ["k_input_bwd", "k_prod_bwd", "k_chain<true>"]
    assert pcb.pc_get_kernel(h, 2, 0, 16384) == "k_sum_mfma<32, 1, 1, false>"
    pcb.pc_set_wait_limit(h, 5)                                # launches that wait only
    assert pcb.pc_get_kernel(h, 2, 0, 7) == "k_flow<1, 1, 1, false, false>"
    for bad in ((9, 0, 1), (-1, 0, 1), (0, 2, 1), (0, 0, 0), (0, 0, (1 << 21) + 1)):
        with pytest.raises(pcb.PcError) as e:
            pcb.pc_get_kernel(h, *bad)
        assert e.value.status_name == "PC_ERR_ARG"
    pcb.pc_destroy(h)


@pytest.mark.parametrize("K,S,B,kernel", [
    (32, 64, 480, "k_prod_fwd"), (64, 128, 480, "k_prod_fwd"),                     # two classes a set: four of a tile's sixteen products
    (32, 96, 480, "k_prod_tile<16, 4>"), (64, 192, 480, "k_prod_tile<8, 4>"),
    (32, 256, 32, "k_prod_tile<16, 2>"), (32, 256, 64, "k_prod_tile<16, 4>"), (64, 256, 128, "k_prod_tile<8, 4>"),
])
def test_kernel_of_leaf_products(K, S, B, kernel):
    w = W.rat_spn(96, 4, 4, S, K, 1, 5, n_cats=3, draw=False)
    h = pcb.pc_compile(w, host_only=True)
    assert pcb.pc_get_kernel(h, 1, 0, B) == kernel
    pcb.pc_destroy(h)


def test_group_tolerance_and_max_groups_are_honoured():
    w = W.reduced(5)
    for G, tol in [(1, 0), (2, 100), (8, 0), (8, 1000)]:
        w.max_groups, w.tol_permille = G, tol
        h = pcb.pc_compile(w, host_only=True)
        try:
            assert_tables_equal(h, w)
        finally:
            pcb.pc_destroy(h)


def _expect(w, status_name):
    with pytest.raises(pcb.PcError) as e:
        h = pcb.pc_compile(w, host_only=True)
        pcb.pc_destroy(h)
    assert e.value.status_name == status_name, str(e.value)


def test_error_paths():
    w = W.hmm(3, 2, 3, 2, 1, 52)
    prod1 = [b for b in range(w.n_blocks) if w.type[b] == W.PRODUCT and w.child_ptr[b + 1] - w.child_ptr[b] == 1][0]
    bad = w.with_batch(w.x); bad.child = w.child.copy(); bad.child[w.child_ptr[prod1]] = w.root_block
    _expect(bad, "PC_ERR_CYCLE")
    s = int(np.nonzero(w.type == W.SUM)[0][0])
    bad = w.with_batch(w.x); bad.child = w.child.copy()
    bad.child[w.child_ptr[s]] = int(np.nonzero(w.type == W.INPUT)[0][0])
    _expect(bad, "PC_ERR_NOT_ALTERNATING")
    bad = w.with_batch(w.x); bad.K = 0
    _expect(bad, "PC_ERR_ARG")
    bad = w.with_batch(w.x); bad.root_block = int(np.nonzero(w.type == W.PRODUCT)[0][0])
    _expect(bad, "PC_ERR_ARG")
    bad = w.with_batch(w.x); bad.param_blk = w.param_blk.copy()
    bad.param_blk[w.child_ptr[w.root_block]] = w.n_param_blocks
    _expect(bad, "PC_ERR_ARG")
    # partial tying: the root borrows one of the transition blocks
    bad = w.with_batch(w.x); bad.param_blk = w.param_blk.copy()
    bad.param_blk[w.child_ptr[w.root_block]] = 0
    _expect(bad, "PC_ERR_TIE")
    # duplicate (parent, child) pair
    w2 = W.hmm(3, 4, 3, 2, 1, 53)
    s = int(np.nonzero(w2.type == W.SUM)[0][0])
    bad = w2.with_batch(w2.x); bad.child = w2.child.copy()
    bad.child[w2.child_ptr[s] + 1] = bad.child[w2.child_ptr[s]]
    _expect(bad, "PC_ERR_NOT_BLOCK_SPARSE")
    # node offsets beyond int32
    big = w.with_batch(w.x); big.K = 1 << 30
    _expect(big, "PC_ERR_TOO_LARGE")


def test_host_only_handle_refuses_device_work():
    w = W.hmm(3, 2, 3, 2, 1, 52)
    h = pcb.pc_compile(w, host_only=True)
    try:
        assert pcb.pc_workspace_bytes(h, 5) > 0
        with pytest.raises(pcb.PcError) as e:
            pcb.pc_forward(h, 1, 1, 1, None, 5, 1, 1 << 40, 1, stream=0)
        assert e.value.status_name == "PC_ERR_STATE"
    finally:
        pcb.pc_destroy(h)


def test_batch_size_limits():
    w = W.hmm(3, 2, 3, 2, 1, 52)
    h = pcb.pc_compile(w, host_only=True)
    try:
        assert pcb.pc_workspace_bytes(h, 2097152) > 0              # PC_MAX_BATCH itself is fine
        for bad, status in ((0, "PC_ERR_ARG"), (-3, "PC_ERR_ARG"), (2097153, "PC_ERR_TOO_LARGE")):
            with pytest.raises(pcb.PcError) as e:
                pcb.pc_workspace_bytes(h, bad)
            assert e.value.status_name == status
    finally:
        pcb.pc_destroy(h)


@pytest.mark.parametrize("make", [lambda: W.hmm(4, 32, 5, 32, 1, 7), lambda: W.hclt(9, 64, 64, 1, 9, n_cats=6),
                                  lambda: W.hmm(5, 8, 9, 2, 1, 13)])
@pytest.mark.parametrize("B", [1, 33, 512])
def test_workspace_holds_the_node_and_block_buffers_and_nothing_else(make, B):
    """l, F, N; R and the block maxima; the batch, transposed -- each rounded up to 256 bytes.  (A byte more would refuse
    circuits that just fit PC_STATIC_SCRATCH_BYTES, and workspaces sized before.)"""
    w = make()
    h = pcb.pc_compile(w, host_only=True)
    Bs = (B + 31) // 32 * 32
    up = lambda n: (n + 255) // 256 * 256
    assert pcb.pc_workspace_bytes(h, B) == 3 * up((w.n_blocks + 1) * w.K * Bs * 4) + 2 * up((w.n_blocks + 1) * Bs * 4) + up(w.n_vars * Bs * 4)
    pcb.pc_destroy(h)

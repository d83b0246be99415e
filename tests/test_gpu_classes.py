"""Product layers over input blocks in classes of equal parents -- forward in tiles of products, backward class by class -- against the
oracle: every block size, tiles of both sizes and cut ones, sets of classes of different sizes, their blocks in turn, and a block of a
class with a parent further up as well.  The kernels that the cases are there for are asserted."""
import pytest

torch = pytest.importorskip("torch")

from paper_2406_00766_amd import workloads as W
from tests.refs import kernels
from tests.test_gpu_dataflow import Dag
from tests.test_gpu_parity import check_all

pytestmark = pytest.mark.gpu


def pairs(K, B, m, p, seed, above):
    """Two sets of p classes of m input blocks (or of p[0], p[1] classes of m[0], m[1]), one product per pair of classes, sums over some
    of the products.  Of different sets the blocks stand in turn, one of every class of the one and of the other, so do they in the products' rows.
    above: an input of the first class is read by a product further up as well, which parts its class in two."""
    d = Dag(K)
    if isinstance(p, tuple):
        sets = [[[] for _ in range(n)] for n in p]
        for k in range(max(m)):
            for s in range(2):
                for c in sets[s]:
                    if k < m[s]: c.append(d.input())
    else:
        sets = [[[d.input() for _ in range(m)] for _ in range(p)] for _ in range(2)]
    left, right = sets
    products = [d.product(a + b) for a in left for b in right]
    sums = [d.sum(products[i::4]) for i in range(4)]
    top = d.sum([d.product([sums[0], left[0][1]]) if above else d.product([sums[0]]), d.product([sums[1]])])
    root = d.sum([d.product([s]) for s in [top, sums[2], sums[3]]], n_real=1)
    return d.workload(root, B, seed)


@pytest.mark.parametrize("K,B,m,p,tile", [
    (32, 1000, 9, 8, "k_prod_tile<16, 2>"), (32, 1010, 5, 17, "k_prod_tile<16, 4>"), (32, 1350, 13, 7, "k_prod_tile<16, 2>"),
    (64, 961, 7, 8, "k_prod_tile<8, 4>"), (64, 1000, 5, 9, "k_prod_tile<8, 4>"), (64, 417, 5, 17, "k_prod_tile<8, 4>"),
    # sets of different sizes, blocks in turn: 6 x 3 classes, 7 x 2, 18 x 11, 17 x 14 (cut tiles on one side and on both)
    (32, 3700, (6, 4), (6, 3), "k_prod_tile<16, 4>"), (64, 4800, (3, 9), (7, 2), "k_prod_tile<8, 4>"),
    (32, 350, (7, 5), (18, 11), "k_prod_tile<16, 2>"), (64, 500, (4, 5), (17, 14), "k_prod_tile<8, 4>"),
])
def test_tiles_of_products_match_oracle(K, B, m, p, tile):
    w = pairs(K, B, m, p, 92, False)
    print(f"case tiles K={K} B={B} m={m} p={p}", flush=True)
    assert kernels(w, 0)[1] == tile and kernels(w, 1)[1] == "k_class_bwd"
    check_all(w)


@pytest.mark.parametrize("K,B,m,p,kernel", [
    (32, 1000, 9, 8, "k_class_bwd"), (32, 1010, 5, 17, "k_class_bwd"), (32, 1350, 13, 7, "k_class_bwd"), (64, 961, 7, 8, "k_class_bwd"),
    (64, 1000, 5, 9, "k_class_bwd"), (32, 33, 9, 8, "k_class_bwd"), (128, 170, 9, 8, "k_class_bwd"), (16, 1000, 9, 8, "k_class_bwd"),
    (8, 90, 9, 8, "k_class_bwd"), (20, 100, 11, 8, "k_class_bwd"),
    (32, 1000, 3, 8, "k_class_bwd"),                           # products of six children, summed in fp32
    (32, 1, 5, 8, "k_prod_bwd"), (64, 40, 6, 5, "k_prod_bwd"), # rows of a dataflow part
])
def test_classes_of_inputs_match_oracle(K, B, m, p, kernel):
    """Class by class backward, added to the flow of a block that has a parent further up as well; no tiles forward: products of three
    classes, one of them that block alone."""
    w = pairs(K, B, m, p, 92, True)
    print(f"case classes K={K} B={B} m={m} p={p}", flush=True)
    assert kernels(w, 0)[1] == "k_prod_fwd" and kernels(w, 1)[1] == kernel
    check_all(w)


def test_rat_spn_with_classes_matches_oracle():
    w = W.rat_spn(45, 2, 1, 256, 32, 515, 93)                  # leaf regions of 11 and 12 variables
    print(f"case classes {w.name}", flush=True)
    assert kernels(w, 0)[1] == "k_prod_tile<16, 2>" and kernels(w, 1)[1] == "k_class_bwd"
    check_all(w)

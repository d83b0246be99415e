"""Product layers over input blocks in classes of equal parents -- forward in tiles of products, backward class by class -- against the
oracle: every block size, tiles of both sizes and cut ones, a block of a class with a parent further up as well."""
import pytest

torch = pytest.importorskip("torch")

from paper_2406_00766_amd import workloads as W
from tests.test_gpu_dataflow import Dag
from tests.test_gpu_parity import check_all

pytestmark = pytest.mark.gpu


def pairs(K, B, m, seed, p=8):
    """Two sets of p classes of m input blocks, one product per pair of classes, sums over some of the products; an input of the
    first class is read by a product further up as well."""
    d = Dag(K)
    left, right = ([[d.input() for _ in range(m)] for _ in range(p)] for _ in range(2))
    products = [d.product(a + b) for a in left for b in right]
    sums = [d.sum(products[i::4]) for i in range(4)]
    top = d.sum([d.product([sums[0], left[0][1]]), d.product([sums[1]])])
    root = d.sum([d.product([s]) for s in [top, sums[2], sums[3]]], n_real=1)
    return d.workload(root, B, seed)


@pytest.mark.parametrize("K,B,m,p", [
    (32, 1000, 9, 8), (32, 1010, 5, 17), (32, 1350, 13, 7), (64, 961, 7, 8), (64, 1000, 5, 9),     # tiles of 2 x 2 and 4 x 4, cut ones
    (32, 33, 9, 8), (32, 1, 5, 8), (64, 40, 6, 5), (128, 170, 9, 8), (16, 1000, 9, 8), (8, 90, 9, 8), (20, 100, 11, 8),   # none
    (32, 1000, 3, 8),                                          # products of six children, summed in fp32
])
def test_classes_of_inputs_match_oracle(K, B, m, p):
    w = pairs(K, B, m, 92, p)
    print(f"case classes K={K} B={B} m={m} p={p}", flush=True)
    check_all(w)


def test_rat_spn_with_classes_matches_oracle():
    w = W.rat_spn(45, 2, 1, 256, 32, 515, 93)                  # leaf regions of 11 and 12 variables
    print(f"case classes {w.name}", flush=True)
    check_all(w)

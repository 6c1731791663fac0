"""fp32 calls with many blocks of tokens and query rows, under every option and with elements beyond the largest bf16 (the checks of
test_gpu_score_split): those of the direct kernels' upper end, and those of the six-product kernels by longer slices, whose merge kernel tells
which of the two a call took."""
import math

import pytest
import torch

from paper_2410_01518_amd import infinipot as ip
from tests import gpu_util as gu
from tests import test_gpu_score_split as base

pytestmark = pytest.mark.gpu


# several rounds of the direct kernels' grid
@pytest.mark.parametrize("units,G,P,n,d,options", [
    (12, 8, 128, 700, 128, ""), (13, 8, 129, 650, 64, "kcat"), (12, 16, 64, 705, 128, "kcat window"), (14, 4, 100, 2100, 64, "lse window"),
    (24, 5, 61, 1100, 128, "lse"), (65, 2, 17, 8200, 64, "window")])
def test_scores(units, G, P, n, d, options):
    base.test_scores(units, G, P, n, d, options)


@pytest.mark.parametrize("kind", ["large keys", "large queries", "infinite keys"])
@pytest.mark.parametrize("units,G,P,n,d,options", [(12, 8, 128, 700, 128, ""), (13, 8, 129, 650, 64, "kcat window"), (14, 4, 100, 2100, 64, "lse window")])
def test_elements_beyond_the_largest_bf16(units, G, P, n, d, options, kind):
    base.test_elements_beyond_the_largest_bf16(units, G, P, n, d, options, kind)


def _by_longer_slices(options, check, *args):
    stages = gu.stages_run(lambda: check(*args))
    assert "score_unit" not in stages and ("score_merge" in stages) == ("lse" not in options)


# The longer slices: row blocks of 32 (two to eight side by side; one row more than four, five, seven and eight of them, two and three sweeps of
# 256); one token more than a slice, a stage of 64 and a tile of 32, one less; two to four slices, last ones of one token
@pytest.mark.parametrize("units,G,P,n,d,options", [
    (256, 1, 33, 833, 128, ""), (256, 1, 97, 321, 128, ""), (140, 3, 43, 289, 128, ""), (100, 1, 225, 257, 128, ""), (60, 1, 97, 513, 128, "kcat"),
    (85, 1, 257, 257, 128, "kcat"), (60, 1, 225, 257, 64, "kcat"), (200, 8, 32, 257, 64, "kcat"), (130, 8, 36, 513, 64, "kcat"),
    (64, 8, 33, 1025, 128, ""), (60, 9, 57, 1409, 128, "kcat window"), (140, 4, 33, 833, 64, "window"), (90, 3, 86, 575, 128, "window"),
    (129, 2, 129, 256, 128, "lse"), (255, 5, 26, 511, 128, "lse"), (85, 4, 64, 769, 128, "lse window")])
def test_scores_by_longer_slices(units, G, P, n, d, options):
    _by_longer_slices(options, base.test_scores, units, G, P, n, d, options)


@pytest.mark.parametrize("kind", ["large keys", "large queries", "infinite keys"])
@pytest.mark.parametrize("units,G,P,n,d,options", [(100, 8, 32, 600, 128, "kcat"), (140, 5, 60, 333, 128, ""), (110, 4, 64, 449, 64, "kcat window"),
                                                   (90, 2, 97, 449, 128, "lse window")])
def test_elements_beyond_the_largest_bf16_by_longer_slices(units, G, P, n, d, options, kind):
    _by_longer_slices(options, base.test_elements_beyond_the_largest_bf16, units, G, P, n, d, options, kind)


def test_a_row_none_of_whose_visible_keys_is_finite_adds_nothing_by_longer_slices():
    _by_longer_slices("", base.test_a_row_none_of_whose_visible_keys_is_finite_adds_nothing, 100, 8, 32, 600, 128, 32, 1)


# 81 to 127 units of 64 elements with more than 6000 tokens times blocks of 256 rows: beyond these the unit kernel is the quicker one, with
# logits good to 2^-16 of sum |q k|.  The six products leave 2e-7 to 4e-7 in the 2-norm and 1.3e-6 at most, the unit kernel 1e-5 and
# 3.4e-5: four times the former is asked for.
@pytest.mark.parametrize("units,G,P,n", [(81, 4, 64, 6001), (100, 4, 16, 7000), (127, 1, 33, 6016), (96, 5, 60, 3001)])
def test_long_rows_below_half_of_the_chip_to_fp32_accuracy(units, G, P, n):
    print(f"long rows {units} {G} {P} {n}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    K = torch.empty((1, units, 1, n, 64), device="cuda").normal_(generator=g)
    Q = torch.empty((1, units, G, P, 64), device="cuda").normal_(generator=g)
    shape = ip.make_shape(Q, K, None, k=n, T=0, pool_w=1)
    scores = torch.empty((1, units, 1, n), device="cuda")
    assert ip.ccd_score(shape, Q, K, None, scores, ip.alloc_workspace(shape)) == ip.CCD_OK
    for i in range(0, units, 20):
        x = torch.matmul(Q[0, i].reshape(G * P, 64).double(), K[0, i, 0].double().t().contiguous()) / math.sqrt(64)
        ref, got = torch.softmax(x, -1).sum(0), scores[0, i, 0].double()
        assert float((got - ref).norm() / ref.norm()) < 1.6e-6 and float(((got - ref).abs() / ref).max()) < 5.2e-6

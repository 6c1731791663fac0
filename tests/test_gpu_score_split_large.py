"""fp32 calls with too many blocks of tokens and query rows for the direct kernels: the six-product kernels by token slices, under every
option and with elements beyond the largest bf16 (the checks of test_gpu_score_split)."""
import pytest

from tests import test_gpu_score_split as base

pytestmark = pytest.mark.gpu


# more than 8192 blocks of 32 x 32, or 16384 with two blocks of rows
@pytest.mark.parametrize("units,G,P,n,d,options", [
    (12, 8, 128, 700, 128, ""), (13, 8, 129, 650, 64, "kcat"), (12, 16, 64, 705, 128, "kcat window"), (14, 4, 100, 2100, 64, "lse window"),
    (24, 5, 61, 1100, 128, "lse"), (65, 2, 17, 8200, 64, "window")])
def test_scores(units, G, P, n, d, options):
    base.test_scores(units, G, P, n, d, options)


@pytest.mark.parametrize("kind", ["large keys", "large queries", "infinite keys"])
@pytest.mark.parametrize("units,G,P,n,d,options", [(12, 8, 128, 700, 128, ""), (13, 8, 129, 650, 64, "kcat window"), (14, 4, 100, 2100, 64, "lse window")])
def test_elements_beyond_the_largest_bf16(units, G, P, n, d, options, kind):
    base.test_elements_beyond_the_largest_bf16(units, G, P, n, d, options, kind)

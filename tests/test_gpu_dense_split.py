"""Dense logistic gradient with the minibatch rows split between row groups: blocks of 32, 64 and 128 float4 columns at
their edges, the last columns of ragged rows, and the unsplit kernel next to the rule, against the oracle."""
import pytest

from paper_1901_08227_amd import binding as B
from test_gpu_step import _dense_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,M,batch", [(127, 3, 70), (129, 2, 17), (2044, 4, 64), (2052, 5, 33), (4099, 16, 64),
                                       (10007, 8, 67), (12289, 3, 16), (12292, 11, 15), (8200, 9, 300)])
def test_columns_and_rows_at_the_edges(d, M, batch):
    _dense_case(M, 96, d, batch, 4, B.NORM_SUB, 2, seed=d, l2=1e-3)

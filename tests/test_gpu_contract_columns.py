"""GPU parity of contractions in tiles of 80 columns whose second operand runs
along the columns in whole 16-byte units (20 or 40 of them, so that some lanes
have no unit of their own), with and without splits of the sum.  Integer
values: the results equal the oracle bit for bit."""
import pytest

from gpu_util import F32, F64
from test_gpu_contract_direct import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [F32, F64], ids=["f32", "f64"])
@pytest.mark.parametrize("m,n,k", [(2048, 80, 1024), (2048, 160, 1024), (3068, 400, 256)])
def test_columns_in_whole_units(dtype, m, n, k):
    _check((0, 2), (1, 2), (0, 1), {0: m, 1: n, 2: k}, dtype, -0.5, 2.0, 11)

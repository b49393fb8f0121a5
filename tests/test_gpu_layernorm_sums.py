"""LayerNorm backward below 2048 columns: one to four chunks per thread in the workgroup's column sums, and numbers of partial rows
that leave none, one, three and seven of a thread's for the last steps of their sum."""
import pytest

from test_gpu_kernels import BF16, F32
from test_gpu_kernels import test_layernorm_forward_backward as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("rows,h", [(1, 8), (5, 512), (69, 520), (257, 1016), (500, 1024), (511, 1032), (1009, 1536), (450, 1544), (2049, 2040)])
def test_backward_column_sums(dtype, rows, h):
    check(dtype, rows, h)

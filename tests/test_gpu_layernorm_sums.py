"""LayerNorm backward below 2048 columns: one to four chunks per thread in the workgroup's column sums, and numbers of partial rows
of which a thread of the last sum has from none to all of the last seven (those that it adds four, two and one at a time)."""
import pytest

from test_gpu_kernels import BF16, F32
from test_gpu_kernels import test_layernorm_forward_backward as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("rows,h", [(1, 8), (5, 512), (69, 520), (257, 1016), (500, 1024), (511, 1032), (1009, 1536), (450, 1544), (2049, 2040)])
def test_backward_column_sums(dtype, rows, h):
    check(dtype, rows, h)


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("rows,h", [(177, 264), (330, 1032), (625, 520)])
def test_steps_of_the_last_sum(dtype, rows, h):
    """45, 83 and 157 partial rows: three or two, six or five, eight and two or one of a thread (threads 16 partial rows apart)."""
    check(dtype, rows, h)

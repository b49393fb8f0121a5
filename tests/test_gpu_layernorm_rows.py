"""LayerNorm backward at the row lengths where its launch shape changes: threads per row (256, 320, 384, 512, 1024),
rows per workgroup, and rows of a step, with one row, fewer rows than a workgroup takes, and several ragged steps."""
import pytest

from test_gpu_kernels import BF16, F32
from test_gpu_kernels import test_layernorm_forward_backward as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("rows,h", [(1, 2056), (5, 2560), (383, 2560), (385, 2056), (1535, 2560), (1537, 2552), (2305, 2560), (1, 2568),
                                    (1538, 3072), (385, 3072), (300, 3080)])
def test_backward_where_the_launch_shape_changes(dtype, rows, h):
    check(dtype, rows, h)

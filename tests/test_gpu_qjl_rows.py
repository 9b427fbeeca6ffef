"""GPU parity of the QJL-corrected attention at every size of its row group: one to four query rows per KV head use one
matrix-core operand per 32 coordinates, five to eight use two, and nine are two groups.  Lengths of one token, a tile and
one more, and a few steps; bar and oracle as in test_gpu_qjl.py."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from test_gpu_qjl import run_decode_qjl_case  # noqa: E402


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("bits,rows", [(1, 8), (1.5, 1), (2, 5), (2.5, 8), (3, 3), (3, 7), (3, 9), (4, 8)])
def test_decode_qjl_rows(d, bits, rows):
    run_decode_qjl_case(d, bits, 3, 2 * rows, 2, 1, [1, 65, 700], seed=int(40 + d + 10 * bits + rows))


@pytest.mark.parametrize("d,rows", [(64, 1), (64, 2), (64, 3), (128, 1), (128, 2), (256, 1), (256, 2)])
def test_decode_qjl_rows_of_the_plan_without_joint_tables(d, rows):
    """4 bits: one row alone at d = 64, two of them and everything at d = 128 padded to four, nothing padded at d = 256."""
    run_decode_qjl_case(d, 4, 3, 2 * rows, 2, 1, [1, 65, 700], seed=int(90 + d + rows))

"""GPU parity of the matrix-core score pass at the sizes where its operands change shape: every plan with joint tables (the
two-class ones cut two code streams into quarters), each head dimension (22, 43 and 86 triplets, none a multiple of four),
one to eight query rows per KV head, and lengths around a block of 16 keys and a tile.  Bar and oracle as in
test_gpu_parity.py."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from test_gpu_parity import run_decode_case  # noqa: E402


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("bits", [1, 1.5, 2, 2.5, 3])
def test_scores_of_every_joint_plan(d, bits):
    run_decode_case(d, bits, 4, 16, 2, 1, [15, 17, 64, 193], "bf16", seed=int(d + 10 * bits))


@pytest.mark.parametrize("rows", [1, 2, 3, 5])
@pytest.mark.parametrize("d,bits", [(64, 3), (128, 2.5), (256, 1.5)])
def test_scores_of_every_row_group(d, bits, rows):
    run_decode_case(d, bits, 2, 2 * rows, 2, 1, [33, 130], "bf16", seed=int(d + rows))


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("rows", [1, 2, 4])
def test_plan_without_joint_tables_small_row_groups(d, rows):
    """At 4 bits a row group may be padded to two or four rows; the padding rows leave no trace."""
    run_decode_case(d, 4, 2, 2 * rows, 2, 1, [129, 700], "bf16", seed=int(d + rows), want_scores=False)

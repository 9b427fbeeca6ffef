"""GPU parity of the merge where the number of partial results per row crosses what a wavefront has in flight: 8, 9, 32, 33, a
wavefront's 64, 65 and 200 partials (a block of 512 tokens, 256 at d = 256, is one partial of a single pair), with a native-precision
window, over fp32 values, and from the many-row kernel's splits.  Bar and oracle as in test_gpu_parity.py."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from test_gpu_hybrid import run_hybrid_case  # noqa: E402
from test_gpu_paged import run_paged_hybrid_case  # noqa: E402
from test_gpu_parity import run_decode_case  # noqa: E402


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("partials", [8, 9, 32, 33, 64, 65, 200])
def test_merge_of_many_partials(d, partials):
    block = 512 if d <= 128 else 256
    run_decode_case(d, 3, 1, 2, 1, 1, [block * partials - 5], "bf16", seed=d + partials, want_scores=False)


def test_merge_of_many_partials_fp32():
    run_decode_case(128, 3, 1, 1, 1, 1, [256 * 65 + 3], "fp32", seed=77, want_scores=False)


@pytest.mark.parametrize("d,tokens", [(64, 512 * 33), (128, 512 * 9 - 100), (128, 512 * 70), (256, 256 * 33)])
def test_merge_of_many_partials_with_a_window(d, tokens):
    run_paged_hybrid_case(d, 3, 1, 4, 1, 1, [tokens], [40], 48, "bf16", seed=d)


@pytest.mark.parametrize("d,tokens", [(64, 512 * 33), (128, 512 * 9 - 100), (256, 256 * 33)])
def test_merge_of_many_partials_with_a_window_of_fp32_keys(d, tokens):
    run_paged_hybrid_case(d, 3, 1, 4, 1, 1, [tokens], [40], 48, "fp32", seed=d + 1)


@pytest.mark.parametrize("v_dtype,k_dtype", [("fp32", "fp32"), ("fp32", "bf16"), ("bf16", "bf16"), ("bf16", "fp32")])
@pytest.mark.parametrize("d,tokens", [(64, 512 * 33), (128, 512 * 9 - 100), (128, 512 * 33), (256, 256 * 33)])
@pytest.mark.parametrize("want_scores", [False, True])
def test_merge_of_many_partials_with_a_window_of_each_type(v_dtype, k_dtype, d, tokens, want_scores):
    run_hybrid_case(d, 3, 1, 2, 1, 1, [tokens], [70], 80, v_dtype, seed=d + 2, want_scores=want_scores, k_dtype=k_dtype)


def test_merge_of_many_splits():
    run_decode_case(128, 3, 1, 1, 1, 40, [5000], "bf16", seed=78, want_scores=False)


def test_merge_of_more_splits_than_lanes():
    run_decode_case(128, 3, 1, 1, 1, 200, [40000], "bf16", seed=79, want_scores=False)

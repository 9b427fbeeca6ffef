"""GPU parity of the division of a decode call's steps over the workgroups: fewer steps than wavefronts, workgroups whose
share spans several (sequence, KV head, row group) pairs and pairs that span several workgroups, empty sequences at the
start, between and at the end, exactly 64 sequences (one per lane), one more, and more than two rounds of lanes.  Bar and
oracle as in test_gpu_parity.py."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from test_gpu_parity import run_decode_case  # noqa: E402


def _lens(n, seed, top):
    r = np.random.default_rng(seed)
    lens = r.integers(0, top, size=n)
    lens[r.random(n) < 0.3] = 0
    return [int(x) for x in lens]


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("d,bits,n_qh,n_kv,lens", [
    (128, 3, 4, 1, [1]),                                  # one step for 256 workgroups
    (128, 3, 6, 2, [0, 0, 0]),                            # nothing at all
    (64, 2, 4, 2, [0, 700, 0, 0, 64, 129, 0]),
    (128, 2.5, 24, 3, [5000, 0, 1, 127, 128, 2049]),      # 8 query rows; one sequence holds most of the steps
    (256, 4, 4, 2, _lens(64, 1, 200) + [77]),
    (64, 3, 2, 2, _lens(64, 2, 400)),
    (64, 1.5, 10, 1, _lens(130, 3, 150) + [0, 0]),        # two row groups
])
def test_decode_work_split(d, bits, n_qh, n_kv, lens, dtype):
    run_decode_case(d, bits, len(lens), n_qh, n_kv, 1, lens, dtype, seed=int(len(lens) + d), want_scores=dtype == "fp32")

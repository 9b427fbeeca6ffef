"""GPU parity of the many-row kernel where its work is cut small: splits of one tile, tiles that do not divide by the splits, numbers
of workgroups that do not divide by the accelerator dies, sequences shorter than the splits are many, and queries of either
type that start where only words are aligned (the kernel rotates them itself).  Bar and oracle as in test_gpu_parity.py."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import oracle  # noqa: E402
from gpu_util import DEV, cache_from_records, check_out, sign_bits_dev, to_dev  # noqa: E402
from paper_2605_21226_amd import binding, synth  # noqa: E402
from test_gpu_parity import make_inputs, oracle_attention_all, run_decode_case  # noqa: E402


@pytest.mark.parametrize("d,bits", [(64, 4), (128, 2.5)])
@pytest.mark.parametrize("n_kv,n_q,lens", [(1, 33, [64 * 5]), (3, 40, [64 * 7 + 1, 64]), (5, 130, [700, 0, 64 * 11]), (1, 300, [3000])])
def test_decode_many_rows_small_splits(d, bits, n_kv, n_q, lens):
    run_decode_case(d, bits, len(lens), n_kv, n_kv, n_q, lens, "bf16", seed=d + n_q, want_scores=False)


# sequences of different lengths in more than one round of workgroups, whose order is spread over the dies by pairs or by units; and in one
# round with more than 16 tiles a split
RAGGED = [190, 64, 0, 65, 1, 130, 20, 333, 5, 128]
SPREAD = [(8, 33, RAGGED * 4), (3, 40, RAGGED * 10), (9, 300, RAGGED * 2), (24, 33, [2000, 70, 0, 1100, 300, 64, 1, 700]),
          (2, 40, [6000] + RAGGED * 4)]


@pytest.mark.parametrize("d,bits", [(64, 3), (128, 4)])
@pytest.mark.parametrize("n_kv,n_q,lens", SPREAD)
def test_decode_many_rows_spread_over_the_dies(d, bits, n_kv, n_q, lens):
    run_decode_case(d, bits, len(lens), n_kv, n_kv, n_q, lens, "bf16", seed=d + n_q, want_scores=False)


@pytest.mark.parametrize("d,n_qh,n_q", [(64, 2, 70), (64, 6, 65), (128, 4, 19), (128, 2, 131)])
@pytest.mark.parametrize("q_dtype", ["bf16", "fp32"])
def test_decode_many_rows_query_types_and_alignment(d, n_qh, n_q, q_dtype):
    n_kv, T, bits = 2, 200, 3
    cb, plan = binding.octopus_build_codebooks(d, bits), oracle.make_plan(d, bits)
    keys, vals, signs = make_inputs(31, 1, n_kv, T, d, "bf16")
    records = np.stack([np.stack([oracle.encode(plan, keys[0, :, h].astype(np.float64), signs[h]) for h in range(n_kv)])])
    cap = 256
    v = np.zeros((1, n_kv, cap, d), dtype=np.float32)
    v[:, :, :T] = vals
    q = synth.queries(31, synth.Workload("t", 1, n_qh, n_kv, d, T, bits, q_dtype, n_q=n_q))
    flat = to_dev(q, q_dtype)
    words = 4 // flat.element_size()
    shifted = torch.empty(flat.numel() + words, dtype=flat.dtype, device=DEV)[words:].view(flat.shape)
    shifted.copy_(flat)
    assert shifted.data_ptr() % 16 == 4
    scale = 1.0 / np.sqrt(d)
    ws = torch.empty(binding.octopus_attn_decode_workspace(cb, 1, n_qh, n_kv, n_q, T), dtype=torch.uint8, device=DEV)
    out = torch.full((1, n_q, n_qh, d), float("nan"), dtype=torch.float32, device=DEV)
    binding.octopus_attn_decode(cb, shifted, sign_bits_dev(signs), cache_from_records(cb, records, cap), cap, to_dev(v, "bf16"),
                                torch.tensor([T], dtype=torch.int32, device=DEV), T, scale, out, ws)
    torch.cuda.synchronize()
    ref, _ = oracle_attention_all(plan, records, signs, q, v, [T], scale)
    got = out.cpu().numpy()
    for h in range(n_qh):
        for qi in range(n_q):
            check_out(got[0, qi, h], ref[0, qi, h])

"""GPU parity of the many-row kernel where max_len (by which a call is cut into splits) is far above the sequences' lengths: programs
that pass their capacity, ragged batches.  A split past a sequence's last tile leaves nothing in the workspace and the merge reads
nothing of it; the workspace starts as NaNs.  Bar and oracle as in test_gpu_parity.py."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import oracle  # noqa: E402
from gpu_util import DEV, cache_from_records, check_out, sign_bits_dev, to_dev  # noqa: E402
from paper_2605_21226_amd import binding, synth  # noqa: E402
from test_gpu_parity import make_inputs, oracle_attention_all  # noqa: E402


@pytest.mark.parametrize("d,bits", [(64, 4), (128, 2.5)])
@pytest.mark.parametrize("n_kv,n_q,lens,max_len", [(1, 40, [150], 16384), (2, 300, [64, 0, 65, 1], 8192), (1, 200, [129], 60000),
                                                   (1, 600, [200, 3], 4096)])
def test_splits_past_the_last_tile_cost_nothing(d, bits, n_kv, n_q, lens, max_len):
    n_seq, T, cap = len(lens), max(lens), -(-max_len // 64) * 64
    cb, plan = binding.octopus_build_codebooks(d, bits), oracle.make_plan(d, bits)
    keys, vals, signs = make_inputs(41, n_seq, n_kv, T, d, "bf16")
    records = np.stack([np.stack([oracle.encode(plan, keys[s, :, h].astype(np.float64), signs[h]) for h in range(n_kv)]) for s in range(n_seq)])
    q = synth.queries(41, synth.Workload("t", n_seq, n_kv, n_kv, d, T, bits, "bf16", n_q=n_q))
    v = np.zeros((n_seq, n_kv, cap, d), dtype=np.float32)
    v[:, :, :T] = vals
    scale = 1.0 / np.sqrt(d)
    ws = torch.full((binding.octopus_attn_decode_workspace(cb, n_seq, n_kv, n_kv, n_q, max_len),), 255, dtype=torch.uint8, device=DEV)
    out = torch.full((n_seq, n_q, n_kv, d), float("nan"), dtype=torch.float32, device=DEV)
    binding.octopus_attn_decode(cb, to_dev(q, "bf16"), sign_bits_dev(signs), cache_from_records(cb, records, cap), cap, to_dev(v, "bf16"),
                                torch.tensor(lens, dtype=torch.int32, device=DEV), max_len, scale, out, ws)
    torch.cuda.synchronize()
    ref, _ = oracle_attention_all(plan, records, signs, q, v, lens, scale)
    got = out.cpu().numpy()
    for s in range(n_seq):
        for qi in range(n_q):
            for h in range(n_kv):
                if lens[s] == 0:
                    assert np.all(got[s, qi, h] == 0.0)
                else:
                    check_out(got[s, qi, h], ref[s, qi, h])
    written = int((ws[:ws.numel() // 4 * 4].view(torch.int32) != -1).sum())
    assert written <= n_q * n_kv * sum(-(-x // 64) for x in lens) * (d + 2)   # (a tile is a split of its own at most)

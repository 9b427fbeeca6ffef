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


@pytest.mark.parametrize("n_seq,extra", [(64, []), (64, [130]), (63, [513]), (62, [513, 1]), (40, [1100, 0, 512])])
def test_decode_division_by_blocks_and_past_it(n_seq, extra):
    """Four KV heads, a block = four steps of 128 tokens: 256 blocks (a workgroup each), one sequence more (an even division),
    sequences of two and three blocks, the last ones short."""
    run_decode_case(64, 3, n_seq + len(extra), 4, 4, 1, [int(x) for x in 1 + np.arange(n_seq) * 37 % 300] + extra, "bf16",
                    seed=n_seq + len(extra), want_scores=False)


def test_short_call_gives_every_block_a_workgroup():
    """32 short sequences, one KV head of eight rows: the partial results lie at slots (workgroup + pair), so the slots written
    say which workgroups took part."""
    from gpu_util import DEV
    from paper_2605_21226_amd import binding
    d, rows, lens = 128, 8, [int(x) for x in 5 + np.arange(32) * 61 % 367]
    lens[7] = 0
    cb = binding.octopus_build_codebooks(d, 3)
    cache = torch.zeros(binding.octopus_cache_bytes(cb, 32, 1, 384), dtype=torch.uint8, device=DEV)
    v = torch.zeros((32, 1, 384, d), dtype=torch.bfloat16, device=DEV)
    q = torch.zeros((32, 1, rows, d), dtype=torch.bfloat16, device=DEV)
    out = torch.zeros((32, 1, rows, d), dtype=torch.float32, device=DEV)
    signs = torch.zeros(d // 8, dtype=torch.uint8, device=DEV)
    ws = torch.full((binding.octopus_attn_decode_workspace(cb, 32, rows, 1, 1, 384),), 255, dtype=torch.uint8, device=DEV)
    binding.octopus_attn_decode(cb, q, signs, cache, 384, v, torch.tensor(lens, dtype=torch.int32, device=DEV), 384, 0.1, out, ws)
    torch.cuda.synchronize()
    rotated = 32 * rows * 132 * 4                         # rotated queries come first: 132 floats a row at this head dimension
    assert rotated % 256 == 0
    ml = ws.cpu().numpy()[rotated:rotated + 256 * rows * 8].view(np.float32).reshape(-1, rows, 2)
    written = np.flatnonzero(~np.isnan(ml[:, 0, 0]))
    pairs = [s for s in range(32) if lens[s]]             # one block each; workgroup b has the b-th of them
    assert list(written) == [b + s for b, s in enumerate(pairs)]


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("n_kv,lens", [
    (4, [20000, 15000, 300, 0, 70, 129]),                 # fewer pairs than workgroups, some short beside the others
    (2, [100] * 40 + [60000] + [64] * 25),                # ... and more than 64 sequences
    (8, [512] * 24),                                      # whole blocks, fewer than workgroups, the bound by rests past them
    (3, [30000, 14500, 1]),
])
def test_decode_division_with_short_pairs(n_kv, lens, dtype):
    run_decode_case(64, 3, len(lens), n_kv, n_kv, 1, lens, dtype, seed=len(lens), want_scores=False)

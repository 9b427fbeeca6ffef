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
    say which workgroups took part.  (Into an output that is not 16-byte aligned: else the kernel writes it without partial results.)"""
    from gpu_util import DEV
    from paper_2605_21226_amd import binding
    d, rows, lens = 128, 8, [int(x) for x in 5 + np.arange(32) * 61 % 367]
    lens[7] = 0
    cb = binding.octopus_build_codebooks(d, 3)
    cache = torch.zeros(binding.octopus_cache_bytes(cb, 32, 1, 384), dtype=torch.uint8, device=DEV)
    v = torch.zeros((32, 1, 384, d), dtype=torch.bfloat16, device=DEV)
    q = torch.zeros((32, 1, rows, d), dtype=torch.bfloat16, device=DEV)
    out = torch.zeros(32 * rows * d + 4, dtype=torch.float32, device=DEV)[1:-3].view(32, 1, rows, d)
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
    (4, [60000, 37400, 832]),                             # shares of three rounds (d = 64, bf16: 512 tokens each)
    (4, [60000, 37400, 768]),                             # ... and just under
    (5, [70001]),
])
def test_decode_division_with_short_pairs(n_kv, lens, dtype):
    run_decode_case(64, 3, len(lens), n_kv, n_kv, 1, lens, dtype, seed=len(lens), want_scores=False)


# Calls of at most 256 (sequence, KV head, row group) pairs and one or two rounds of steps (1024 tokens; 512 at d = 256; over
# fp32 values 256) write their output without a merge; one token or one pair more, and they don't.
@pytest.mark.parametrize("d,bits,n_qh,n_kv,lens,dtype", [
    (128, 3, 16, 2, [1024, 0, 1, 513, 512], "bf16"),
    (128, 3, 16, 2, [1025, 0, 1, 513, 512], "bf16"),
    (64, 4, 6, 2, [0, 1000, 129, 0], "bf16"),              # (no joint tables: one round)
    (64, 4, 6, 2, [0, 500, 129, 0], "bf16"),
    (64, 2, 24, 1, [300, 0, 70], "bf16"),                  # three row groups
    (256, 2.5, 4, 2, [512, 0, 257], "bf16"),
    (128, 3, 8, 2, [256, 0, 65, 1], "fp32"),
    (128, 3, 8, 2, [257, 0, 65, 1], "fp32"),
    (64, 3, 8, 8, [int(x) for x in np.arange(32) * 13 % 200], "bf16"),
    (64, 3, 8, 8, [int(x) for x in np.arange(33) * 13 % 200], "bf16"),
    (64, 3, 2, 2, [0, 0, 0], "bf16"),
])
def test_decode_without_a_merge(d, bits, n_qh, n_kv, lens, dtype):
    run_decode_case(d, bits, len(lens), n_qh, n_kv, 1, lens, dtype, seed=int(len(lens) + d), want_scores=False)


def test_output_that_is_not_16_byte_aligned():
    """The outputs of a short call into an aligned tensor and into one four bytes further: the same to rounding."""
    from gpu_util import DEV
    from paper_2605_21226_amd import binding
    d, n_kv, rows, lens = 128, 2, 4, [300, 0, 77]
    gen = torch.Generator().manual_seed(23)
    cb = binding.octopus_build_codebooks(d, 3)
    cache = torch.zeros(binding.octopus_cache_bytes(cb, 3, n_kv, 320), dtype=torch.uint8, device=DEV)
    signs = torch.randint(0, 256, (n_kv, d // 8), generator=gen, dtype=torch.uint8).to(DEV)
    binding.octopus_encode(cb, torch.randn((3, 300, n_kv, d), generator=gen).to(DEV, torch.bfloat16), signs, cache, 320)
    v = torch.randn((3, n_kv, 320, d), generator=gen).to(DEV, torch.bfloat16)
    q = torch.randn((3, 1, n_kv * rows, d), generator=gen).to(DEV, torch.bfloat16)
    ws = torch.empty(binding.octopus_attn_decode_workspace(cb, 3, n_kv * rows, n_kv, 1, 300), dtype=torch.uint8, device=DEV)
    n = 3 * n_kv * rows * d
    outs = []
    for shift in (0, 1):
        ws.fill_(255)
        out = torch.full((n + 4,), float("nan"), dtype=torch.float32, device=DEV)[shift:shift + n].view(3, 1, n_kv * rows, d)
        binding.octopus_attn_decode(cb, q, signs, cache, 320, v, torch.tensor(lens, dtype=torch.int32, device=DEV), 300, 0.09, out, ws)
        outs.append(out.cpu())
        assert bool((ws == 255).all()) == (shift == 0)   # no partial results where nothing reads them
    assert not outs[0][1].any() and torch.isfinite(outs[0]).all()
    assert torch.allclose(outs[0], outs[1], rtol=1e-6, atol=1e-6)


# Many sequences, some of them empty, more than one per lane: up to 256 pairs by the decode kernel alone, 258 and 260 through the merge.
RAGGED = [int(x) for x in (40 + np.arange(128) * 29 % 171) * (np.arange(128) % 5 > 0)]


@pytest.mark.parametrize("n_seq,n_kv", [(128, 2), (100, 2), (65, 4)])
def test_many_sequences_with_and_without_a_merge(n_seq, n_kv):
    run_decode_case(64, 3, n_seq, n_kv, n_kv, 1, RAGGED[:n_seq], "bf16", seed=31 + n_seq, want_scores=False)


@pytest.mark.parametrize("n_seq,n_kv", [(90, 2), (43, 6)])
def test_many_sequences_over_pages_values_and_the_residual(n_seq, n_kv):
    from test_gpu_paged import run_paged_decode_case, run_paged_qjl_decode_case, run_paged_vq_decode_case
    from test_gpu_qjl import run_decode_qjl_case
    from test_gpu_values import run_decode_vq_case
    lens, n_qh = RAGGED[:n_seq], 4 * n_kv
    run_paged_decode_case(64, 3, n_seq, n_qh, n_kv, 1, lens, seed=37)
    run_decode_vq_case(64, 3, 3, 32, n_seq, n_qh, n_kv, 1, lens, seed=38, want_scores=False)
    run_paged_vq_decode_case(64, 2, 2, 16, n_seq, n_qh, n_kv, 1, lens, seed=39)
    run_decode_qjl_case(64, 3, n_seq, n_qh, n_kv, 1, lens, seed=40, want_scores=False)
    run_paged_qjl_decode_case(64, 2, n_seq, n_qh, n_kv, 1, lens, seed=41)


# The kernels that accumulate on the vector units, calls of one to two rounds of steps (256 tokens each) per workgroup: blocks of two
# rounds, but an even division where the pairs are equal and a power of two.
@pytest.mark.parametrize("n_kv,lens", [
    (8, [6000, 4167, 0, 70]),
    (5, [20000]),
    (1, [40000] + [500] * 66),                            # more than 64 sequences
    (8, [6000, 6000]),                                    # (even)
    (4, [8192, 8192, 8192, 8191]),                        # ... and one token short of it: 256 blocks of two rounds
    (4, [8192, 8192, 8192, 8193]),                        # one token too many
])
def test_decode_by_blocks_of_two_rounds(n_kv, lens):
    run_decode_case(64, 3, len(lens), n_kv, n_kv, 1, lens, "fp32", seed=len(lens) + 7, want_scores=False)


def test_quantised_values_by_blocks_of_two_rounds():
    from test_gpu_values import run_decode_vq_case
    run_decode_vq_case(64, 3, 3, 16, 2, 8, 8, 1, [6000, 4167], seed=43, want_scores=True)


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("lens", [[300], [20000, 100], [5000, 3000, 70]])
def test_infinity_in_the_last_value_row(d, lens):
    """Its channel is infinite, the others are what they are without it: partial results that a batch of them has too many do not count.
    (fp32 values: their weights are not split.)"""
    from gpu_util import DEV
    from paper_2605_21226_amd import binding
    gen = torch.Generator().manual_seed(51)
    n, n_kv, rows, top = len(lens), 2, 2, max(lens)
    cap = (top + 63) // 64 * 64
    cb = binding.octopus_build_codebooks(d, 3)
    signs = torch.randint(0, 256, (n_kv, d // 8), generator=gen, dtype=torch.uint8).to(DEV)
    cache = torch.zeros(binding.octopus_cache_bytes(cb, n, n_kv, cap), dtype=torch.uint8, device=DEV)
    binding.octopus_encode(cb, torch.randn((n, top, n_kv, d), generator=gen).to(DEV), signs, cache, cap)
    v = torch.randn((n, n_kv, cap, d), generator=gen).to(DEV)
    q = torch.randn((n, 1, n_kv * rows, d), generator=gen).to(DEV)
    ws = torch.empty(binding.octopus_attn_decode_workspace(cb, n, n_kv * rows, n_kv, 1, top), dtype=torch.uint8, device=DEV)
    outs = []
    for x in (1.0, float("inf")):
        for s, length in enumerate(lens):
            v[s, :, length - 1, 5] = x
        out = torch.zeros((n, 1, n_kv * rows, d), device=DEV)
        binding.octopus_attn_decode(cb, q, signs, cache, cap, v, torch.tensor(lens, dtype=torch.int32, device=DEV), top, 0.1, out, ws)
        outs.append(out.cpu().numpy())
    assert np.all(np.isposinf(outs[1][..., 5])) and np.all(np.isfinite(outs[0]))
    others = np.arange(d) != 5
    assert np.array_equal(outs[0][..., others], outs[1][..., others])

"""The entry point that allocates nothing (octopus_attn_decode_static: the library's static scratch array in place of
a caller workspace), through the C ABI, against octopus_attn_decode on the same inputs: two calls in a row, the second
with a smaller input, and the refusal of shapes beyond the array."""
import numpy as np
import pytest

import oracle
from paper_2605_21226_amd import binding, layout, synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from gpu_util import (DEV, cache_from_records, check_out, check_scores, record_gammas, score_floor, sign_bits_dev,  # noqa: E402
                      to_dev)
from test_gpu_parity import make_inputs, oracle_attention_all  # noqa: E402


def run_case(seed, n_seq, n_kv, g, n_tok, lens, d=128, bits=3, dtype="bf16"):
    cb = binding.octopus_build_codebooks(d, bits)
    plan = oracle.make_plan(d, bits)
    cap = -(-n_tok // 64) * 64
    keys, vals, signs = make_inputs(seed, n_seq, n_kv, n_tok, d, dtype)
    rec = np.stack([np.stack([oracle.encode(plan, keys[s, :, h].astype(np.float64), signs[h]) for h in range(n_kv)])
                    for s in range(n_seq)])
    cache = cache_from_records(cb, rec, cap)
    v = np.zeros((n_seq, n_kv, cap, d), dtype=np.float32)
    v[:, :, :n_tok] = vals
    rng = np.random.default_rng(seed + 77)
    q = rng.standard_normal((n_seq, 1, n_kv * g, d)).astype(np.float32)
    if dtype == "bf16":
        q = synth.round_to_bf16(q)
    scale = 1.0 / np.sqrt(d)
    q_dev, v_dev, s_dev = to_dev(q, dtype), to_dev(v, dtype), sign_bits_dev(signs)
    lens_dev = torch.tensor(lens, dtype=torch.int32, device=DEV)
    max_len = int(max(lens))
    outs, scores = [], []
    for static in (False, True):
        out = torch.full((n_seq, 1, n_kv * g, d), float("nan"), dtype=torch.float32, device=DEV)
        sc = torch.full((n_seq, 1, n_kv * g, cap), float("nan"), dtype=torch.float32, device=DEV)
        if static:
            binding.octopus_attn_decode_static(cb, q_dev, s_dev, cache, cap, v_dev, lens_dev, max_len, scale, out, sc)
        else:
            ws = torch.empty(binding.octopus_attn_decode_workspace(cb, n_seq, n_kv * g, n_kv, 1, max_len),
                             dtype=torch.uint8, device=DEV)
            binding.octopus_attn_decode(cb, q_dev, s_dev, cache, cap, v_dev, lens_dev, max_len, scale, out, ws, sc)
        torch.cuda.synchronize()
        outs.append(out.cpu().numpy())
        scores.append(sc.cpu().numpy())
    # same kernels, same launch shapes: the two entry points agree bit for bit ...
    assert np.array_equal(outs[0], outs[1])
    assert np.array_equal(np.nan_to_num(scores[0], nan=-1.0), np.nan_to_num(scores[1], nan=-1.0))
    # ... and with the oracle to the bar of every other decode test
    ref_out, ref_scores = oracle_attention_all(plan, rec, signs, q.astype(np.float64), v.astype(np.float64), lens, scale)
    for s in range(n_seq):
        L = int(lens[s])
        for h in range(n_kv * g):
            check_out(outs[1][s, 0, h], ref_out[s, 0, h])
            check_scores(scores[1][s, 0, h, :L], ref_scores[(s, h // g)][0, h % g])


def test_static_scratch_matches_workspace_entry_point_twice_second_call_smaller():
    run_case(21, 3, 2, 4, 700, [700, 333, 64])
    run_case(22, 1, 1, 4, 150, [150])


def test_static_scratch_refuses_shapes_beyond_the_array():
    cb = binding.octopus_build_codebooks(64, 4)
    # 24 heads x 3600 query rows against 75,600 tokens: the partials of the many-row kernel exceed 32 MiB
    need = binding.octopus_attn_decode_workspace(cb, 1, 24, 24, 3600, 75648)
    assert need > binding.STATIC_SCRATCH_BYTES
    q = torch.zeros((1, 3600, 24, 64), dtype=torch.bfloat16, device=DEV)
    v = torch.zeros((1, 24, 75648, 64), dtype=torch.bfloat16, device=DEV)
    cache = torch.zeros(binding.octopus_cache_bytes(cb, 1, 24, 75648), dtype=torch.uint8, device=DEV)
    out = torch.zeros((1, 3600, 24, 64), dtype=torch.float32, device=DEV)
    lens = torch.tensor([75600], dtype=torch.int32, device=DEV)
    signs = torch.zeros(24 * 8, dtype=torch.uint8, device=DEV)
    with pytest.raises(binding.OctopusError) as err:
        binding.octopus_attn_decode_static(cb, q, signs, cache, 75648, v, lens, 75600, 0.125, out)
    assert err.value.code == binding.ESCRATCH


@pytest.mark.parametrize("d,rows,padded,n_seq", [(128, 1, 4, 400), (128, 2, 4, 300)])
@pytest.mark.parametrize("want_scores", [False, True])
def test_static_scratch_serves_shapes_whose_padded_row_groups_exceed_it(d, rows, padded, n_seq, want_scores):
    """At 4 bits row groups of one and two are padded at d = 128; where the padded partials exceed the static array and the documented ones do not,
    the call runs the kernels of the smallest row group.  Mostly empty sequences, 96 of them with tokens; against the call
    with a workspace (padded groups) and, for four sequences, the oracle."""
    n_kv, max_len = 8, 384

    def scratch(group):    # partial results, both rotations of the queries, window partials (up to the rounding of each)
        return (group * 4 * (2048 + n_seq * n_kv) * (4 * d + 8) + n_seq * n_kv * group * (4 * (d + 4) + 4 * d) +
                n_seq * n_kv * rows * (4 * d + 8))
    assert scratch(rows) + 4096 < binding.STATIC_SCRATCH_BYTES < scratch(padded)
    cb = binding.octopus_build_codebooks(d, 4)
    plan = oracle.make_plan(d, 4)
    need = binding.octopus_attn_decode_workspace(cb, n_seq, n_kv * rows, n_kv, 1, max_len)
    rng = np.random.default_rng(d + rows)
    lens = np.zeros(n_seq, dtype=np.int32)
    busy = rng.permutation(n_seq)[:96]
    lens[busy] = rng.integers(1, max_len + 1, size=96)
    keys = torch.randn((96, max_len, n_kv, d), generator=torch.Generator().manual_seed(d + rows)).to(torch.bfloat16)
    signs = synth.sign_vectors(d + rows, n_kv, d)
    s_dev = sign_bits_dev(signs)
    part = torch.zeros(binding.octopus_cache_bytes(cb, 96, n_kv, max_len), dtype=torch.uint8, device=DEV)
    binding.octopus_encode(cb, keys.to(DEV), s_dev, part, max_len)
    cache = torch.zeros(binding.octopus_cache_bytes(cb, n_seq, n_kv, max_len), dtype=torch.uint8, device=DEV).view(n_seq, -1)
    cache[torch.from_numpy(busy).to(DEV)] = part.view(96, -1)
    v = torch.zeros((n_seq, n_kv, max_len, d), dtype=torch.bfloat16, device=DEV)
    v[torch.from_numpy(busy).to(DEV)] = torch.from_numpy(rng.standard_normal((96, n_kv, max_len, d)).astype(np.float32)).to(DEV, torch.bfloat16)
    q = torch.from_numpy(rng.standard_normal((n_seq, 1, n_kv * rows, d)).astype(np.float32)).to(DEV, torch.bfloat16)
    lens_dev = torch.from_numpy(lens).to(DEV)
    scale = 1.0 / np.sqrt(d)
    outs, scores = [], []
    for static in (False, True):
        out = torch.full((n_seq, 1, n_kv * rows, d), float("nan"), dtype=torch.float32, device=DEV)
        sc = torch.full((n_seq, 1, n_kv * rows, max_len), float("nan"), dtype=torch.float32, device=DEV) if want_scores else None
        if static:
            binding.octopus_attn_decode_static(cb, q, s_dev, cache, max_len, v, lens_dev, max_len, scale, out, sc)
        else:
            ws = torch.empty(need, dtype=torch.uint8, device=DEV)
            binding.octopus_attn_decode(cb, q, s_dev, cache, max_len, v, lens_dev, max_len, scale, out, ws, sc)
        torch.cuda.synchronize()
        outs.append(out.cpu().numpy())
        scores.append(None if sc is None else sc.cpu().numpy())
    assert not outs[1][lens == 0].any()
    # the same sums of fp32 products over d terms and at most 384 tokens, in another order
    assert np.max(np.abs(outs[1] - outs[0])) <= 1e-4 * np.max(np.abs(outs[0]))
    if want_scores:
        assert np.array_equal(np.isnan(scores[0]), np.isnan(scores[1]))
        assert np.nanmax(np.abs(scores[1] - scores[0])) <= 1e-4 * np.nanmax(np.abs(scores[0]))
    for i in (0, 31, 63, 95):
        s, n = int(busy[i]), int(lens[busy[i]])
        for h in range(n_kv):
            k = keys[i, :n, h].to(torch.float64).numpy()
            rec = layout.cache_to_records(part.view(96, -1)[i].cpu().numpy(), 1, n_kv, max_len, cb.plan.granules,
                                          cb.plan.record_bytes, n)[0][0, h]
            assert oracle.classify(plan, k, signs[h], rec, tol=1e-6)[2] == 0
            qq = q[s, 0, h * rows:(h + 1) * rows].cpu().to(torch.float64).numpy()
            ref_sc, ref_o, _ = oracle.attention(plan, rec, signs[h], qq, v[s, h, :n].cpu().to(torch.float64).numpy(), scale)
            for r in range(rows):
                check_out(outs[1][s, 0, h * rows + r], ref_o[r])
                if want_scores:
                    check_scores(scores[1][s, 0, h * rows + r, :n], ref_sc[r],
                                 score_floor(qq[r], record_gammas(rec), scale))

"""GPU parity of the hybrid cache: octopus_attn_decode_hybrid (compressed tokens + a native-precision window)
against the oracle's dense definition over the reconstructed keys stacked on the window's keys; scores and
outputs to the 1e-3 bar of the plain decoder."""
import numpy as np
import pytest

import oracle
from paper_2605_21226_amd import binding, synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from gpu_util import DEV, cache_from_records, check_out, check_scores, sign_bits_dev, to_dev  # noqa: E402
from test_gpu_parity import make_inputs  # noqa: E402


def run_hybrid_case(d, bits, n_seq, n_qh, n_kv, n_q, lens, win_lens, w_capacity, dtype, seed, want_scores=True,
                    t_capacity=None, k_dtype=None):
    """k_dtype: type of the window's keys, where it is not the queries' and values' `dtype`"""
    k_dtype = k_dtype or dtype
    cb = binding.octopus_build_codebooks(d, bits)
    plan = oracle.make_plan(d, bits)
    tot = [int(a) + int(b) for a, b in zip(lens, win_lens)]
    T = max(max(tot), 1)
    cap = t_capacity or -(-T // 64) * 64
    keys, vals, signs = make_inputs(seed, n_seq, n_kv, T, d, dtype)          # keys [n_seq, T, n_kv, d]
    records = np.zeros((n_seq, n_kv, max(max(lens), 1), plan.record_bytes), dtype=np.uint8)
    k_win = np.zeros((n_seq, n_kv, w_capacity, d), dtype=np.float32)
    for s in range(n_seq):
        L, W = int(lens[s]), int(win_lens[s])
        for h in range(n_kv):
            if L:
                records[s, h, :L] = oracle.encode(plan, keys[s, :L, h].astype(np.float64), signs[h])
            k_win[s, h, :W] = keys[s, L:L + W, h]
    if k_dtype != dtype:
        k_win = to_dev(k_win, k_dtype).float().cpu().numpy()
    wl = synth.Workload("t", n_seq, n_qh, n_kv, d, T, bits, dtype, n_q=n_q)
    q = synth.queries(seed, wl)
    v = np.zeros((n_seq, n_kv, cap, d), dtype=np.float32)
    v[:, :, :T] = vals
    scale = 1.0 / np.sqrt(d)
    cache = cache_from_records(cb, records, cap)
    max_len = max(int(x) for x in lens)
    ws = torch.empty(binding.octopus_attn_decode_workspace(cb, n_seq, n_qh, n_kv, n_q, max_len), dtype=torch.uint8,
                     device=DEV)
    out = torch.full((n_seq, n_q, n_qh, d), float("nan"), dtype=torch.float32, device=DEV)
    scores = (torch.full((n_seq, n_q, n_qh, cap), float("nan"), dtype=torch.float32, device=DEV) if want_scores else None)
    lens_dev = torch.tensor(np.asarray(lens), dtype=torch.int32, device=DEV)
    win_dev = torch.tensor(np.asarray(win_lens), dtype=torch.int32, device=DEV)
    binding.octopus_attn_decode_hybrid(cb, to_dev(q, dtype), sign_bits_dev(signs), cache, cap, to_dev(v, dtype), lens_dev,
                                       max_len, to_dev(k_win, k_dtype), win_dev, scale, out, ws, scores)
    torch.cuda.synchronize()
    out = out.cpu().numpy()
    scores = scores.cpu().numpy() if want_scores else None
    g = n_qh // n_kv
    worst_s = worst_o = 0.0
    for s in range(n_seq):
        L, W = int(lens[s]), int(win_lens[s])
        for h in range(n_kv):
            if L + W == 0:
                assert np.all(out[s, :, h * g:(h + 1) * g] == 0.0)
                continue
            qq = q[s, :, h * g:(h + 1) * g, :].reshape(-1, d).astype(np.float64)
            ref_s, ref_o = oracle.attention_hybrid(plan, records[s, h, :L], signs[h], k_win[s, h, :W], qq,
                                                   v[s, h, :L + W].astype(np.float64), scale)
            ref_s, ref_o = ref_s.reshape(n_q, g, L + W), ref_o.reshape(n_q, g, d)
            for qi in range(n_q):
                for j in range(g):
                    if want_scores:
                        worst_s = max(worst_s, check_scores(scores[s, qi, h * g + j, :L + W], ref_s[qi, j]))
                    worst_o = max(worst_o, check_out(out[s, qi, h * g + j], ref_o[qi, j]))
        if want_scores:
            assert np.all(np.isnan(scores[s, :, :, L + W:]))
    print(f"[hybrid] d={d} b={bits} lens={list(lens)} window={list(win_lens)}: worst score err {worst_s:.3g} x tol, "
          f"worst out err {worst_o:.3g}")


@pytest.mark.parametrize("bits", [2, 3, 4])
def test_hybrid_gqa_window_32_d128(bits):
    run_hybrid_case(128, bits, 3, 8, 2, 1, [1000, 77, 0], [32, 32, 20], 32, "bf16", seed=int(1400 + 10 * bits))


def test_hybrid_degenerate_windows():
    # empty windows (the plain result), nothing compressed, nothing at all, a window longer than one chunk
    run_hybrid_case(128, 3, 4, 4, 2, 1, [300, 0, 0, 130], [0, 40, 0, 150], 160, "bf16", seed=1450)


def test_hybrid_fp32_everything_d64_and_d256():
    run_hybrid_case(64, 4, 2, 3, 3, 2, [200, 65], [16, 7], 16, "fp32", seed=1460)
    run_hybrid_case(256, 2.5, 2, 4, 2, 1, [513, 64], [32, 1], 32, "bf16", seed=1461)


def test_hybrid_many_query_rows_uses_the_matrix_core_kernel():
    run_hybrid_case(128, 3, 2, 8, 2, 16, [513, 130], [48, 5], 64, "bf16", seed=1470, want_scores=False)


def test_hybrid_window_clipped_at_capacity():
    # 60 compressed + a window of 10 declared, capacity 64: only 4 window tokens fit behind the compressed ones
    d = 128
    cb = binding.octopus_build_codebooks(d, 3)
    plan = oracle.make_plan(d, 3)
    keys, vals, signs = make_inputs(1480, 1, 1, 64, d, "bf16")
    rec = oracle.encode(plan, keys[0, :60, 0].astype(np.float64), signs[0])[None, None]
    k_win = np.zeros((1, 1, 16, d), dtype=np.float32)
    k_win[0, 0, :4] = keys[0, 60:64, 0]
    wl = synth.Workload("t", 1, 2, 1, d, 64, 3, "bf16", n_q=1)
    q = synth.queries(1480, wl)
    cache = cache_from_records(cb, rec, 64)
    ws = torch.empty(binding.octopus_attn_decode_workspace(cb, 1, 2, 1, 1, 60), dtype=torch.uint8, device=DEV)
    out = torch.zeros((1, 1, 2, d), dtype=torch.float32, device=DEV)
    lens = torch.tensor([60], dtype=torch.int32, device=DEV)
    win = torch.tensor([10], dtype=torch.int32, device=DEV)
    v_dev = to_dev(vals, "bf16")
    binding.octopus_attn_decode_hybrid(cb, to_dev(q, "bf16"), sign_bits_dev(signs), cache, 64, v_dev, lens, 60,
                                       to_dev(k_win, "bf16"), win, 0.1, out, ws)
    torch.cuda.synchronize()
    _, ref_o = oracle.attention_hybrid(plan, rec[0, 0], signs[0], k_win[0, 0, :4], q[0, 0].astype(np.float64),
                                       vals[0, 0, :64].astype(np.float64), 0.1)
    for j in range(2):
        check_out(out.cpu().numpy()[0, 0, j], ref_o[j])


@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (128, "bf16"), (256, "bf16"), (128, "fp32")])
@pytest.mark.parametrize("w", [1, 8, 16, 24, 33, 64, 72])
def test_infinity_in_the_last_value_row_of_a_window(d, dtype, w):
    """Its channel is infinite (a weight of at least exp(-60) times infinity), the others are what they are without it: rows that
    a batch of value rows has too many do not count."""
    gen = torch.Generator().manual_seed(w)
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    cb = binding.octopus_build_codebooks(d, 3)
    signs = torch.randint(0, 256, (1, d // 8), generator=gen, dtype=torch.uint8).to(DEV)
    cache = torch.zeros(binding.octopus_cache_bytes(cb, 1, 1, 256), dtype=torch.uint8, device=DEV)
    binding.octopus_encode(cb, torch.randn((1, 100, 1, d), generator=gen).to(DEV, t), signs, cache, 256)
    v = torch.randn((1, 1, 256, d), generator=gen).to(DEV, t)
    k_win = torch.randn((1, 1, 80, d), generator=gen).to(DEV, t)
    q = torch.randn((1, 1, 2, d), generator=gen).to(DEV, t)
    lens, win = (torch.tensor([n], dtype=torch.int32, device=DEV) for n in (100, w))
    ws = torch.empty(binding.octopus_attn_decode_workspace(cb, 1, 2, 1, 1, 100), dtype=torch.uint8, device=DEV)
    outs = []
    for x in (1.0, float("inf")):
        v[0, 0, 100 + w - 1, 5] = x
        out = torch.zeros((1, 1, 2, d), device=DEV)
        binding.octopus_attn_decode_hybrid(cb, q, signs, cache, 256, v, lens, 100, k_win, win, 0.1, out, ws)
        outs.append(out.cpu().numpy()[0, 0])
    assert np.all(np.isposinf(outs[1][:, 5])) and np.all(np.isfinite(outs[0]))
    others = np.arange(d) != 5
    assert np.array_equal(outs[0][:, others], outs[1][:, others])

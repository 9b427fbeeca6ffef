"""The encoder looks at four candidates per triplet where the winner of Alg. 1's nine is known to be among them: for the
library's own direction levels.  Here that claim is checked for every piece of the square, in 64 bits, and the levels the
library takes it for; on the GPU the four-candidate kernels are compared with the nine-candidate ones code for code."""
import ctypes

import numpy as np
import pytest

from paper_2605_21226_amd import binding, layout

torch = pytest.importorskip("torch")


def _books(bd):
    return binding.octopus_build_codebooks(128, {1: 1, 3: 2, 4: 3, 5: 4}[bd])


def _corner_levels(cb):
    fn = getattr(binding.load(), "_ZN7octopus13corner_levelsERK17octopus_codebooks")
    fn.restype = ctypes.c_bool
    return fn(ctypes.byref(cb))


def _unit(xi, eta):
    r = 1 - np.abs(xi) - np.abs(eta)
    a = np.where(r < 0, np.where(xi >= 0, 1, -1) * (1 - np.abs(eta)), xi)
    b = np.where(r < 0, np.where(eta >= 0, 1, -1) * (1 - np.abs(xi)), eta)
    return np.stack([a, b, r], -1) / np.sqrt(a * a + b * b + r * r)[..., None]


def _clip(poly, f):
    """The part of a convex polygon where the linear function f is not negative."""
    out = []
    for a, b in zip(poly, poly[1:] + poly[:1]):
        fa, fb = f(a), f(b)
        if fa >= 0:
            out.append(a)
        if (fa > 0 > fb) or (fa < 0 < fb):
            out.append(a + fa / (fa - fb) * (b - a))
    return out


def test_the_winner_is_one_of_four():
    """One direction bit: one level on either side of an axis, so the corner in the quadrant that the signs of x and y name is the only
    candidate of the encoder's (brackets, from 3 bits on: test_encoder_brackets.py).  Bound: two scores of a unit triplet are off by at
    most 3 roundings of 2^-24 each plus 3 * 2^-24 of either table entry, and the point by 3e-7 in xi and eta (levels up to 0.6 apart):
    under 1e-6 together.  Every other candidate has to lose by 2.5e-6 on the whole of a face's part (the difference is linear there:
    its vertices decide)."""
    near_axis = 1e-5
    c = np.array(_books(1).c_xi[0][:2], dtype=np.float64)
    n = _unit(c[:, None] + 0 * c, c[None, :] + 0 * c[:, None])
    rect = [np.array(p) for p in ((0.0, 0.0), (1.0, 0.0), (1.0, 1.0), (0.0, 1.0))]
    checked, least = 0, np.inf
    for upper in (True, False):
        poly = _clip(rect, (lambda v: 1 - v[0] - v[1]) if upper else (lambda v: v[0] + v[1] - 1))
        for f in ([lambda v: v[0] - near_axis, lambda v: v[1] - near_axis] if upper else
                  [lambda v: 1 - v[1] - near_axis, lambda v: 1 - v[0] - near_axis]):
            poly = _clip(poly, f)
        pts = np.array([[v[0], v[1], 1 - v[0] - v[1]] if upper else [1 - v[1], 1 - v[0], 1 - v[0] - v[1]] for v in poly])
        pts /= np.linalg.norm(pts, axis=1, keepdims=True)
        for e in ((0, 0), (0, 1), (1, 0)):
            least = min(least, (pts @ (n[1, 1] - n[e])).min())
            checked += 1
    print(f"{checked} candidates, least margin {least:.3g}")
    assert checked == 6 and least >= 2.5e-6


def test_levels_the_four_candidates_are_taken_for():
    for d in (64, 128, 256):
        for bits in (1, 1.5, 2, 2.5, 3, 4):
            assert _corner_levels(binding.octopus_build_codebooks(d, bits))
    cb = _books(4)
    cb.c_xi[0][9] *= 1.000001
    assert not _corner_levels(cb)            # one level moved
    cb.c_xi[0][6] *= 1.000001
    assert not _corner_levels(cb)            # both sides moved
    cb = _books(4)
    cb.c_rho[0][3] = 1.0
    assert not _corner_levels(cb)            # a norm level outside [0, 1)
    assert not _corner_levels(binding.octopus_build_codebooks_pair(128, 2, 2))


def _special_keys(n, n_kv, d, gen):
    """Random keys with rows of zeros, one-hot and two-hot rows, constant rows, signs, half zeros, small integers, tiny and huge
    norms, NaN and infinity between them."""
    k = torch.randn((1, n, n_kv, d), generator=gen)
    k[0, 1::16] = 0
    k[0, 2::16] = 0
    for t in range(2, n, 16):
        k[0, t, :, (t * 7) % d] = 1.5
    k[0, 3::16] = 0
    for t in range(3, n, 16):
        k[0, t, :, (t * 5) % d] = 1.0
        k[0, t, :, (t * 3 + 1) % d] = -1.0
    k[0, 4::16] *= 1e-25
    k[0, 5::16] *= 1e25
    k[0, 6::16] = 1.0
    k[0, 7::64, :, 3] = float("nan")
    k[0, 23::64, :, 3] = float("inf")
    k[0, 8::16] = torch.sign(k[0, 8::16])
    k[0, 9::16, :, ::2] = 0
    k[0, 10::16] = torch.round(k[0, 10::16])
    k[0, 11::16, :, :d // 2] = k[0, 11::16, :, d // 2:].clone()
    return k


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("d,bits", [(64, 1), (128, 1.5), (256, 2), (64, 2.5), (128, 3), (64, 4), (256, 4)])
def test_four_candidates_give_the_codes_of_nine(d, bits, dtype):
    """The same keys with the library's codebooks and with the top norm level raised to 1 (nine candidates): norms and direction
    codes agree bit for bit."""
    n, n_kv, start = 531, 2, 13
    gen = torch.Generator().manual_seed(17)
    keys = _special_keys(n, n_kv, d, gen).to("cuda", dtype)
    signs = torch.randint(0, 256, (n_kv, d // 8), generator=gen, dtype=torch.uint8).cuda()
    cap = (n + start + 63) // 64 * 64
    at = torch.tensor([start], dtype=torch.int32, device="cuda")
    codes = []
    for nine in (False, True):
        cb = binding.octopus_build_codebooks(d, bits)
        if nine:
            for c in range(cb.plan.n_class):
                cb.c_rho[c][(1 << cb.plan.b_nrm[c]) - 1] = 1.0
        assert _corner_levels(cb) != nine
        cache = torch.zeros(binding.octopus_cache_bytes(cb, 1, n_kv, cap), dtype=torch.uint8, device="cuda")
        binding.octopus_encode(cb, keys, signs, cache, cap, at)
        torch.cuda.synchronize()
        rec, _ = layout.cache_to_records(cache.cpu().numpy(), 1, n_kv, cap, cb.plan.granules, cb.plan.record_bytes)
        codes.append(rec[..., :4 + cb.plan.dir_bytes])
    assert np.array_equal(codes[0], codes[1])


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("d,bits", [(64, 1), (64, 1.5), (64, 4), (128, 1), (128, 2), (128, 2.5), (128, 3), (128, 4), (256, 1.5), (256, 3), (256, 4)])
def test_appended_keys_have_the_records_of_a_prefill(d, bits, dtype):
    """One call over 300 tokens x 4 KV heads (tiles) and the same tokens one, two and seven at a time (a wavefront per key): the
    same bytes, past the capacity nothing is written."""
    n, n_kv, start = 300, 4, 13
    gen = torch.Generator().manual_seed(19)
    keys = _special_keys(n, n_kv, d, gen).to("cuda", dtype)
    signs = torch.randint(0, 256, (n_kv, d // 8), generator=gen, dtype=torch.uint8).cuda()
    cb = binding.octopus_build_codebooks(d, bits)
    cap = (n + start + 63) // 64 * 64
    caches = [torch.zeros(binding.octopus_cache_bytes(cb, 1, n_kv, cap), dtype=torch.uint8, device="cuda") for _ in range(2)]
    binding.octopus_encode(cb, keys, signs, caches[0], cap, torch.tensor([start], dtype=torch.int32, device="cuda"))
    t, sizes = 0, (1, 2, 7)
    while t < n:
        m = min(sizes[t % 3], n - t)
        binding.octopus_encode(cb, keys[:, t:t + m], signs, caches[1], cap, torch.tensor([start + t], dtype=torch.int32, device="cuda"))
        t += m
    binding.octopus_encode(cb, keys[:, :2], signs, caches[1], cap, torch.tensor([cap], dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    assert torch.equal(caches[0], caches[1])


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("d,bits", [(64, 3), (128, 1.5), (128, 4), (256, 2.5)])
def test_norm_of_a_key_with_nans(d, bits, dtype):
    """A key with one NaN: its norm is that NaN, sign and payload, quieted, from the tile kernel with four and with nine candidates
    and from the append kernel.  Several NaNs: the same one everywhere."""
    n, n_kv = 300, 4
    gen = torch.Generator().manual_seed(29)
    keys = torch.randn((1, n, n_kv, d), generator=gen).to(dtype)
    if dtype == torch.bfloat16:
        nans, raw, quiet = [0x7FC0, 0xFFC0, 0x7FC5, 0xFFC3, 0x7F81, 0xFF82], keys.view(torch.int16), lambda x: (x | 0x40) << 16
    else:
        nans, raw, quiet = [0x7FC00000, 0xFFC00000, 0x7FC12345, 0xFFC54321, 0x7F800001, 0xFF812345], keys.view(torch.int32), lambda x: x | 0x400000
    top = 1 << (15 if dtype == torch.bfloat16 else 31)
    expected = np.zeros((n_kv, n), dtype=np.uint32)
    for t in range(n):
        for h in range(n_kv):
            for j in range(1 if t % 2 else 3):
                x = nans[(t // 2 + h + j) % 6]
                raw[0, t, h, (13 * t + 37 * j + 5 * h) % d] = x - 2 * top if x >= top else x
                expected[h, t] = quiet(x)
    keys = keys.cuda()
    signs = torch.randint(0, 256, (n_kv, d // 8), generator=gen, dtype=torch.uint8).cuda()
    words = []
    for nine, single in ((False, False), (True, False), (False, True)):
        cb = binding.octopus_build_codebooks(d, bits)
        if nine:
            for c in range(cb.plan.n_class):
                cb.c_rho[c][(1 << cb.plan.b_nrm[c]) - 1] = 1.0
        cache = torch.zeros(binding.octopus_cache_bytes(cb, 1, n_kv, 320), dtype=torch.uint8, device="cuda")
        for t in range(n if single else 1):
            at = torch.tensor([t], dtype=torch.int32, device="cuda")
            binding.octopus_encode(cb, keys[:, t:t + 1] if single else keys, signs, cache, 320, at)
        torch.cuda.synchronize()
        rec, _ = layout.cache_to_records(cache.cpu().numpy(), 1, n_kv, 320, cb.plan.granules, cb.plan.record_bytes)
        words.append(np.ascontiguousarray(rec[0, :, :n, :4]).view(np.uint32)[..., 0])
        assert np.array_equal(words[-1][:, 1::2], expected[:, 1::2])
        assert np.array_equal(words[-1], words[0])

"""The encoder finds the bracket of a coordinate by rounding a polynomial of it, whose steps lie beside the levels, not on them.  The
winner of Alg. 1's nine candidates is one of such a bracket's four corners all the same: checked here for every piece of the square,
in 64 bits.  On the GPU: plans whose last triplet is one coordinate, where the four candidates are not looked at."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2605_21226_amd import binding, layout
from test_encoder_corners import _books, _clip, _corner_levels, _special_keys, _unit

torch = pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = next((c for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")) if c and os.path.exists(c)), None)


@pytest.fixture(scope="module")
def kernel_brackets(tmp_path_factory):
    """{direction bits: (near_axis, steps)} of the encoder's own code, compiled for the CPU: fp32 with the fused multiply-add."""
    if HIPCC is None:
        pytest.skip("hipcc not found")
    exe = str(tmp_path_factory.mktemp("host") / "bracket_driver")
    res = subprocess.run([HIPCC, "-O2", "-std=c++17", "--offload-arch=gfx950", "--offload-host-only", "-x", "hip", "-I" + os.path.join(ROOT, "include"),
                          "-I" + os.path.join(ROOT, "paper_2605_21226_amd", "csrc"), "-Wno-unused-command-line-argument",
                          os.path.join(ROOT, "tests", "host", "bracket_driver.cpp"), "-o", exe], capture_output=True, text=True, timeout=600)
    assert res.returncode == 0, res.stderr[-4000:]
    res = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout + res.stderr
    found = {}
    for line in res.stdout.splitlines():
        bd, near_axis, at_zero, at_one, rises, *steps = line.split()
        half = 1 << (int(bd) - 1)
        assert (int(at_zero), int(at_one), int(rises)) == (0, half - 2, 1) and len(steps) == half - 2
        found[int(bd)] = (float(near_axis), [float(x) for x in steps])
    return found


@pytest.mark.parametrize("bd", [3, 4, 5])
def test_the_winner_is_a_corner_of_the_rounded_bracket(bd, kernel_brackets):
    """Bound: two scores of a unit triplet are off by under 1e-6 together, as in test_encoder_corners.py (the reciprocal's unit in the last
    place moves the point by 2e-7 and the steps by as much); every other candidate has to lose by 2.5e-6."""
    k, half = 1 << bd, 1 << (bd - 1)
    c = np.array(_books(bd).c_xi[0][:k], dtype=np.float64)
    n = _unit(c[:, None] + 0 * c, c[None, :] + 0 * c[:, None])
    mids = 0.5 * (c[1:] + c[:-1])
    near_axis, steps = kernel_brackets[bd]
    edges = [0.0] + steps + [1.0]
    assert len(edges) == half and np.abs(np.array(edges[1:-1]) - c[half + 1:k - 1]).max() < 0.003
    checked, least = 0, np.inf

    def pieces(j):   # (a little past the steps, which the kernel computes in fp32)
        lo, hi = max(edges[j] - 1e-6, 0.0), min(edges[j + 1] + 1e-6, 1.0)
        cuts = [lo] + [m for m in mids if lo < m < hi] + [hi]
        return zip(cuts[:-1], cuts[1:])
    for jx in range(half - 1):
        for jy in range(half - 1):
            corners = {(half + jx + a, half + jy + b) for a in (0, 1) for b in (0, 1)}
            for x0, x1 in pieces(jx):
                for y0, y1 in pieces(jy):
                    sx, sy = np.searchsorted(mids, [0.5 * (x0 + x1), 0.5 * (y0 + y1)])
                    assert sx - half - jx in (0, 1) and sy - half - jy in (0, 1)     # the seed is an end of the bracket
                    nine = {(min(max(sx + a, 0), k - 1), min(max(sy + b, 0), k - 1)) for a in (-1, 0, 1) for b in (-1, 0, 1)}
                    rect = [np.array(p) for p in ((x0, y0), (x1, y0), (x1, y1), (x0, y1))]
                    for upper in (True, False):
                        poly = _clip(rect, (lambda v: 1 - v[0] - v[1]) if upper else (lambda v: v[0] + v[1] - 1))
                        for f in ([lambda v: v[0] - near_axis, lambda v: v[1] - near_axis] if upper else
                                  [lambda v: 1 - v[1] - near_axis, lambda v: 1 - v[0] - near_axis]):
                            poly = _clip(poly, f)
                        if not poly:
                            continue
                        pts = np.array([[v[0], v[1], 1 - v[0] - v[1]] if upper else [1 - v[1], 1 - v[0], 1 - v[0] - v[1]]
                                        for v in poly])
                        pts /= np.linalg.norm(pts, axis=1, keepdims=True)
                        for e in nine - corners:
                            least = min(least, max((pts @ (n[t] - n[e])).min() for t in corners))
                            checked += 1
    print(f"{checked} candidates, least margin {least:.3g}")
    assert checked and least >= 2.5e-6


@pytest.mark.parametrize("bd", [1, 3, 4, 5])
def test_the_winner_of_a_lone_coordinate(bd):
    """(x, 0, 0): of the nine the outermost level of x wins, with the lower of the two levels next to eta = 0, whose score is the
    same bit for bit (the table's entries are)."""
    k, half = 1 << bd, 1 << (bd - 1)
    c = np.array(_books(bd).c_xi[0][:k], dtype=np.float64)
    n = _unit(c[:, None] + 0 * c, c[None, :] + 0 * c[:, None])
    sy = int(np.sum(0.5 * (c[1:] + c[:-1]) < 0.0))
    assert sy == half - 1
    for sign, sx in ((1, k - 1), (-1, 0)):
        order = [(min(max(sx + a, 0), k - 1), min(max(sy + b, 0), k - 1)) for a in (-1, 0, 1) for b in (-1, 0, 1)]
        scores = np.array([sign * n[e][0] for e in order])
        assert order[int(np.argmax(scores > scores.max() - 1e-9))] == (sx, half - 1)
        others = [s for e, s in zip(order, scores) if not (e[0] == sx and e[1] in (half - 1, half))]
        assert not others or max(others) < scores.max() - 1e-3


@pytest.mark.gpu
@pytest.mark.parametrize("d,bits", [(64, 1.5), (64, 3), (64, 4), (256, 1), (256, 3), (128, 4), (128, 2)])
@pytest.mark.parametrize("n", [531, 3])   # tiles, a wavefront per key
def test_special_keys_have_the_codes_of_nine_candidates(d, bits, n):
    gen = torch.Generator().manual_seed(23)
    keys = _special_keys(n if n > 64 else 96, 2, d, gen)[:, :n if n > 64 else 96].to("cuda", torch.bfloat16)
    signs = torch.randint(0, 256, (2, d // 8), generator=gen, dtype=torch.uint8).cuda()
    cap, codes = 576, []
    for nine in (False, True):
        cb = binding.octopus_build_codebooks(d, bits)
        if nine:
            for c in range(cb.plan.n_class):
                cb.c_rho[c][(1 << cb.plan.b_nrm[c]) - 1] = 1.0
        assert _corner_levels(cb) != nine
        cache = torch.zeros(binding.octopus_cache_bytes(cb, 1, 2, cap), dtype=torch.uint8, device="cuda")
        step = keys.shape[1] if nine or n > 64 else n
        for t in range(0, keys.shape[1], step):
            binding.octopus_encode(cb, keys[:, t:t + step], signs, cache, cap, torch.tensor([t], dtype=torch.int32, device="cuda"))
        torch.cuda.synchronize()
        rec, _ = layout.cache_to_records(cache.cpu().numpy(), 1, 2, cap, cb.plan.granules, cb.plan.record_bytes)
        codes.append(rec[..., :4 + cb.plan.dir_bytes])
    assert np.array_equal(codes[0], codes[1])

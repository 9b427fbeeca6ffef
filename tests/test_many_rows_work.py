"""The division of the many-row kernel's work over workgroups and accelerator dies, on the CPU by the kernel's own code: every piece once,
the blocks of a unit together, and the dies evenly loaded where sequences differ or max_len is far above them."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = next((c for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")) if c and os.path.exists(c)), None)


@pytest.fixture(scope="module")
def work(tmp_path_factory):
    if HIPCC is None:
        pytest.skip("hipcc not found")
    exe = str(tmp_path_factory.mktemp("host") / "mq_work_driver")
    csrc = os.path.join(ROOT, "paper_2605_21226_amd", "csrc")
    res = subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "--offload-host-only", "-x", "hip", "-I" + os.path.join(ROOT, "include"),
                          "-I" + csrc, "-Wno-unused-command-line-argument", os.path.join(ROOT, "tests", "host", "mq_work_driver.cpp"), "-o", exe],
                         capture_output=True, text=True, timeout=600)
    assert res.returncode == 0, res.stderr[-4000:]

    def ask(*args):
        res = subprocess.run([exe] + [str(x) for x in args], capture_output=True, text=True, timeout=120)
        assert res.returncode == 0, res.stderr
        return np.array([[int(x) for x in line.split()] for line in res.stdout.splitlines()])
    return ask


@pytest.mark.parametrize("spread", [0, 1])
@pytest.mark.parametrize("n_seq,n_kv,splits,blocks", [(1, 1, 1, 1), (1, 1, 7, 1), (1, 1, 23, 11), (2, 1, 125, 2), (3, 1, 5, 4), (1, 8, 4, 8), (9, 1, 1, 3),
                                                      (3, 8, 3, 3), (2, 24, 3, 3), (5, 9, 2, 2), (20, 2, 16, 1), (5, 1, 8, 2), (3, 3, 31, 1), (7, 4, 6, 2)])
def test_every_piece_once(work, n_seq, n_kv, splits, blocks, spread):
    w = work(n_seq, n_kv, splits, blocks, spread)
    n, pairs = n_seq * n_kv * splits * blocks, n_seq * n_kv
    assert len(w) == n and len({tuple(x) for x in w[:, 1:]}) == n
    assert np.all(w.max(0)[1:] == (pairs - 1, splits - 1, blocks - 1))
    per_die = np.bincount(w[:, 0], minlength=8)
    assert per_die.max() == -(-n // 8)
    dies_of_a_unit = {}
    for die, pair, split, _ in w:
        dies_of_a_unit.setdefault((pair, split), set()).add(die)
    assert sum(len(d) - 1 for d in dies_of_a_unit.values()) <= 7   # (a border between two dies parts one unit at most)


@pytest.mark.parametrize("tiles,n_kv,splits,blocks", [
    ([69, 4], 24, 3, 3),                        # one long sequence, one short: every die has its share of the long one
    ([256] + [2] * 15, 2, 16, 1),
    ([125, 60, 30, 10], 8, 5, 2),
    ([63] * 4 + [3] * 4, 4, 4, 4),
    ([125] + [20] * 15, 1, 17, 1),
    ([4] * 8, 8, 32, 1),                        # max_len far above: the first splits of each pair have the tiles
    ([8] * 2, 4, 40, 2),
    ([1] * 64, 1, 4, 2),
])
def test_dies_are_evenly_loaded(work, tiles, n_kv, splits, blocks):
    """Tiles of the busiest die against the mean (in a row, a die had whole sequences: up to the number of dies)."""
    assert work("spreads", len(tiles), n_kv, splits, blocks, 64 * max(max(tiles), splits * 16))[0, 0] == 1
    load = np.zeros(8)
    for die, pair, split, _ in work(len(tiles), n_kv, splits, blocks, 1):
        t = tiles[pair // n_kv]
        load[die] += t // splits + (split < t % splits)
    print(f"busiest die {load.max() / load.mean():.3f} of the mean")
    assert load.max() <= 1.15 * load.mean()


def test_calls_that_are_spread(work):
    """Several sequences in more than one round of workgroups, or with many tiles each; not one sequence, not short splits in one round."""
    assert work("spreads", 2, 24, 3, 3, 4376)[0, 0] == 1 and work("spreads", 8, 4, 2, 4, 6000)[0, 0] == 1
    assert work("spreads", 1, 24, 3, 30, 4376)[0, 0] == 0 and work("spreads", 5, 2, 12, 2, 3697)[0, 0] == 0

"""Which block of query rows the host picks, on the CPU: the calls of the GPU tests of the 256-row blocks at head dimension 128
do take them, and the shapes that are faster with blocks of 128 rows keep those."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = next((c for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")) if c and os.path.exists(c)), None)

WIDE = (9, 8, 8, 385, 130)       # the shape test_gpu_many_rows.py runs at every width, contiguous and paged


@pytest.fixture(scope="module")
def shapes(tmp_path_factory):
    if HIPCC is None:
        pytest.skip("hipcc not found")
    exe = str(tmp_path_factory.mktemp("host") / "shape_driver")
    csrc = os.path.join(ROOT, "paper_2605_21226_amd", "csrc")
    res = subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "-x", "hip", "-I" + os.path.join(ROOT, "include"),
                          "-I" + csrc, "-Wno-unused-command-line-argument", os.path.join(csrc, "octopus_host.cpp"),
                          os.path.join(ROOT, "tests", "host", "shape_driver.cpp"), "-o", exe],
                         capture_output=True, text=True, timeout=600)
    assert res.returncode == 0, res.stderr[-4000:]

    def ask(kind, d, bits, n_seq, n_qh, n_kv, n_q, max_len):
        args = [str(x) for x in (int(kind), d, bits, n_seq, n_qh, n_kv, n_q, max_len)]
        res = subprocess.run([exe] + args, capture_output=True, text=True, timeout=60)
        assert res.returncode == 0, res.stdout + res.stderr
        return tuple(int(x) for x in res.stdout.split())
    return ask


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("bits", [1, 1.5, 2, 2.5, 3, 4])
def test_calls_with_blocks_of_256_rows(shapes, bits, paged):
    assert shapes(paged, 128, bits, *WIDE)[0] == 256
    assert shapes(paged, 128, bits, 1, 8, 8, 130, 25600)[0] == 256
    assert shapes(paged, 64, bits, 1, 1, 1, 192, 1000)[0] == 256


@pytest.mark.parametrize("bits", [1, 1.5, 2, 2.5, 3, 4])
def test_calls_with_blocks_of_512_rows(shapes, bits):
    """Many rows at d = 64, and the shapes of the GPU tests of these blocks; where 256 rows leave fewer rounds they stay."""
    assert shapes(False, 64, bits, 9, 8, 8, 1100, 130)[:3] == (512, 3, 1)
    assert shapes(PAGED_WINDOW, 64, bits, 9, 8, 8, 1100, 130)[:3] == (512, 3, 1)
    assert shapes(False, 64, bits, 1, 24, 24, 800, 3000)[:3] == (512, 2, 5)
    assert shapes(False, 64, bits, 1, 24, 24, 3600, 75600)[0] == 512
    assert shapes(False, 64, bits, 9, 8, 8, 385, 130)[0] == 256 and shapes(False, 64, bits, 33, 8, 8, 256, 130)[0] == 256


def test_calls_with_blocks_of_128_rows(shapes):
    for n_seq, n_qh, n_kv, n_q, max_len in [(1, 4, 1, 59, 4245), (1, 8, 1, 64, 16384), (2, 1, 1, 128, 64), (1, 2, 2, 140, 5000)]:
        assert shapes(False, 128, 3, n_seq, n_qh, n_kv, n_q, max_len)[0] == 128
    assert shapes(False, 64, 3, 1, 1, 1, 191, 1000)[0] == 128


def test_row_groups_of_plans_without_joint_tables(shapes):
    """At 4 bits small groups are padded at d = 128: the row group is part of what the GPU tests of it run."""
    assert [shapes(False, 128, 4, 2, 2 * r, 2, 1, 700)[0] for r in (1, 2, 4, 8)] == [4, 4, 4, 8]
    assert [shapes(False, 64, 4, 2, 2 * r, 2, 1, 700)[0] for r in (1, 2, 4, 8)] == [1, 2, 4, 8]
    assert [shapes(False, 256, 4, 2, 2 * r, 2, 1, 700)[0] for r in (1, 2, 4, 8)] == [1, 2, 4, 8]


BF16, PAGED, FP32, VQ8, VQ4, QJL, WINDOW, SHIFTED, PAGED_VQ8, PAGED_QJL, PAGED_WINDOW = 0, 1, 2, 3, 4, 5, 6, 7, 13, 15, 16


@pytest.mark.parametrize("kind,d,bits,round_tokens,long_steps", [
    (BF16, 128, 3, 512, False), (PAGED, 128, 3, 512, False), (BF16, 64, 1.5, 512, False), (BF16, 256, 2.5, 256, False),
    (VQ8, 128, 3, 512, False), (PAGED_VQ8, 64, 2, 512, False), (VQ4, 128, 3, 256, True), (FP32, 128, 3, 256, True),
    (FP32, 256, 2, 256, True), (QJL, 128, 3, 512, True), (PAGED_QJL, 64, 2, 512, True), (BF16, 64, 4, 512, True), (PAGED, 128, 4, 512, True)])
def test_which_calls_are_served_without_a_merge(shapes, kind, d, bits, round_tokens, long_steps):
    """Up to two rounds of steps and 256 (sequence, KV head, row group) pairs; one round where steps are long and the pairs are at most
    half the workgroups.  One token or one pair more, and the partial results are merged."""
    few = 1 if long_steps else 2
    # (eight query rows per KV head: one row group, whatever the kernel)
    for n_seq, rounds in ((1, few), (64, few), (65, 2), (128, 2)):
        assert shapes(kind, d, bits, n_seq, 16, 2, 1, rounds * round_tokens)[3] == 0
        assert shapes(kind, d, bits, n_seq, 16, 2, 1, 64)[3] == 0
        assert shapes(kind, d, bits, n_seq, 16, 2, 1, rounds * round_tokens + 1)[3] == 1
    assert shapes(kind, d, bits, 129, 16, 2, 1, 64)[3] == 1
    # 24 rows per KV head: three row groups, 252 and 258 pairs
    assert [shapes(kind, d, bits, n, 48, 2, 1, 64)[1::2] for n in (42, 43)] == [(3, 0), (3, 1)]


def test_calls_that_are_always_merged(shapes):
    for kind in (WINDOW, PAGED_WINDOW, SHIFTED):
        assert shapes(kind, 128, 3, 1, 8, 2, 1, 64)[3] == 1
    for kind in (BF16, PAGED):
        assert shapes(kind, 128, 3, 1, 8, 8, 130, 100)[3] == 1           # blocks of many query rows


@pytest.mark.parametrize("d", [64, 128])
def test_splits_of_many_query_rows(shapes, d):
    """Short calls are cut until most compute units have a workgroup, never finer than tiles; the workspace keeps its documented size
    (the call is refused otherwise)."""
    for n_seq, n_qh, n_kv, n_q, max_len in [(1, 32, 8, 36, 2908), (1, 8, 8, 646, 1335), (1, 64, 8, 56, 378), (1, 1, 1, 33, 64), (3, 4, 2, 40, 129)]:
        rows, groups, splits, merged = shapes(False, d, 3, n_seq, n_qh, n_kv, n_q, max_len)
        assert merged == 1 and 1 <= splits <= -(-max_len // 64)
        assert shapes(True, d, 3, n_seq, n_qh, n_kv, n_q, max_len) == (rows, groups, splits, merged)
    rows, groups, splits, _ = shapes(False, d, 4, 1, 32, 8, 36, 2908)
    assert 128 <= 8 * groups * splits <= 256 * (2 if d == 64 else 1)


def test_more_splits_than_lanes_where_few_heads_have_long_contexts(shapes):
    """The shape of the GPU test with more partials per row than a wavefront has lanes; a second round of them has to pay."""
    assert shapes(False, 128, 3, 1, 1, 1, 200, 40000)[:3] == (128, 2, 125)
    assert shapes(False, 64, 3, 1, 1, 1, 300, 10000)[2] <= 64 and shapes(False, 128, 3, 1, 1, 1, 35, 8000)[2] <= 64

"""Kernels whose inner loops have to stay in registers, by what the compiler reports of the built library: scratch memory per
lane.  A change that makes them spill costs tens of per cent and no parity test sees it."""
import os
import re

import pytest

pytest.importorskip("msgpack")

from kernel_resources import kernels  # noqa: E402
from paper_2605_21226_amd import binding  # noqa: E402


@pytest.fixture(scope="module")
def library():
    if not os.path.exists(binding.LIB_PATH):
        pytest.skip("liboctopus.so is not built")
    return kernels(binding.LIB_PATH)


def _decode(library, d, scores, qjl):
    """{((b_dir, b_nrm, b_dir, b_nrm), query rows, paged): scratch bytes per lane} of decode_kernel_mfma."""
    pat = re.compile(rf"18decode_kernel_mfmaINS_5PlanTILi{d}ELi(\d)ELi(\d)ELi(\d)ELi(\d)EEELi(\d)ELb{scores:d}ELb{qjl:d}ELb(\d)E")
    found = {}
    for name, k in library.items():
        m = pat.search(name)
        if m:
            n = [int(x) for x in m.groups()]
            found[(tuple(n[:4]), n[4], n[5])] = k[".private_segment_fixed_size"]
    return found


def test_residual_kernels_at_256_do_not_spill(library):
    """Five bit widths (4 bits scores on the vector units), four row groups, contiguous and paged; 12 bytes are a lane's
    three loop-invariant words."""
    joint = {k: v for k, v in _decode(library, 256, True, True).items() if k[0][0] < 5}
    assert len(joint) == 5 * 4 * 2
    assert {k: v for k, v in joint.items() if v > 12} == {}


@pytest.mark.parametrize("d", [64, 128])
def test_kernels_without_residual_do_not_spill(library, d):
    """Every plan with joint tables (two direction codes and a norm code of at most ten bits), one to eight query rows."""
    joint = {k: v for k, v in _decode(library, d, False, False).items() if all(2 * k[0][c] + k[0][c + 1] <= 10 for c in (0, 2))}
    assert len(joint) >= 5 * 4 * 2
    assert {k: v for k, v in joint.items() if v} == {}


def test_encoders_do_not_spill(library):
    """encode_kernel with four and with nine candidates, every rounding variant and pair, and the append kernel.  The pair of 3 + 5 bits
    over fp32 keys keeps three words of a lane outside its loops, 1.5 bits at d = 256 with the residual and nine candidates two (97.1 us
    of 16 Ki keys x 8 KV heads without them, 97.4 with)."""
    found = {name: k[".private_segment_fixed_size"] for name, k in library.items() if re.search(r"1[37]encode_(few_)?kernel", name)}
    assert sum("encode_few_kernel" in n for n in found) == 18 * 2 and len(found) == 36 + 200
    words = {"13encode_kernelINS_5PlanTILi128ELi3ELi5ELi0ELi0EEELb0ELb0ELb0ELb0E": 12,
             "13encode_kernelINS_5PlanTILi256ELi3ELi1ELi1ELi1EEELb1ELb1ELb0ELb0E": 8}
    assert {n: v for n, v in found.items() if v > max([b for part, b in words.items() if part in n], default=0)} == {}


def test_many_row_kernels_do_not_spill(library):
    """decode_kernel_mq: 128 and 256 query rows at d = 64 and 128, 512 at d = 64; a spill of 100 registers took 1.7 - 2.8 times as long."""
    found = {name: k[".private_segment_fixed_size"] for name, k in library.items() if "16decode_kernel_mq" in name}
    assert len(found) == 6 * 2 + 6 * 3
    assert {n: v for n, v in found.items() if v} == {}


def test_merge_kernels_do_not_spill(library):
    """merge_kernel: three head dimensions, with and without two-round blocks and each kind of window, 8 or 32 partials in flight; in
    scratch memory 32 of them were slower than 8."""
    found = {name: k[".private_segment_fixed_size"] for name, k in library.items() if "12merge_kernel" in name}
    assert len(found) == 3 * 6 * 2
    assert {n: v for n, v in found.items() if v} == {}


def test_scratch_of_the_heaviest_kernels_over_quantised_values(library):
    """Groups of 16, or eight rows, of 1 - 2 bit keys at d = 256 keep hundreds of bytes of a lane in scratch; together no more than
    before the maxima over a wavefront were taken for all rows at once."""
    pat = re.compile(r"decode_kernel_vq_mfmaINS_5PlanTILi256ELi[13]ELi1E\w*ELi(4ELi\dELi16|8ELi\dELi32)E")
    found = [k[".private_segment_fixed_size"] for name, k in library.items() if pat.search(name)]
    assert len(found) == 17 and sum(found) <= 10948

"""The documented workspace size of a decode call is part of its interface (callers allocate by it, and the call without a
workspace refuses shapes by it): it stays what it was whichever kernel, row group or split count serves the call."""
import pytest

from paper_2605_21226_amd import binding


@pytest.mark.parametrize("d,bits,shape,want", [
    (128, 3, (16, 32, 8, 1, 32768), 37007616),
    (128, 4, (1, 1, 1, 1, 64), 22016),
    (256, 2.5, (32, 16, 8, 1, 65536), 40685824),
    (128, 3, (1, 32, 8, 509, 15877), 161491456),
    (64, 4, (1, 24, 24, 3600, 75600), 285508864),
])
def test_documented_workspace(d, bits, shape, want):
    cb = binding.octopus_build_codebooks(d, bits)
    assert binding.octopus_attn_decode_workspace(cb, *shape) == want

"""Maxima over a wavefront are inline assembly whose lane permutes read a register two wait states after it was written at the
earliest; the compiler counts no waits there.  Read in the built library: the two wait states before every such instruction are
waits or the maxima of other values, so that no copy or reload can have come between."""
import os
import re
import shutil
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

import pytest

pytest.importorskip("msgpack")

from kernel_resources import _code_objects  # noqa: E402
from paper_2605_21226_amd import binding  # noqa: E402

OBJDUMP = next((c for c in ("/opt/rocm/llvm/bin/llvm-objdump", shutil.which("llvm-objdump")) if c and os.path.exists(c)), None)


def _unsafe(lines):
    """(maxima, those not preceded by two such wait states)."""
    count, bad = 0, []
    for i, line in enumerate(lines):
        m = re.match(r"v_max_f32_dpp (v\d+), (v\d+), (v\d+) ", line)
        if not m:
            continue
        count += 1
        waits, j = 0, i - 1
        while waits < 2 and j >= 0:
            nop = re.match(r"s_nop (\d+)", lines[j])
            other = re.match(r"v_max_f32_dpp (v\d+),", lines[j])
            if not nop and (not other or other.group(1) in m.groups()):
                bad.append((lines[j], line))
                break
            waits += int(nop.group(1)) + 1 if nop else 1
            j -= 1
        if waits < 2 and j < 0:
            bad.append(("", line))
    return count, bad


def test_the_scan():
    ok = ["s_nop 1", "v_max_f32_dpp v1, v1, v1 row_shr:1", "v_max_f32_dpp v2, v2, v2 row_shr:1", "s_nop 0", "v_max_f32_dpp v1, v1, v1 row_shr:2"]
    assert _unsafe(ok) == (3, [])
    assert len(_unsafe(ok[:3] + ok[4:])[1]) == 1                              # one wait state short
    assert len(_unsafe(ok[:3] + ["v_mov_b32_e32 v1, v9"] + ok[3:])[1]) == 1   # a copy in between
    assert len(_unsafe(ok[1:2])[1]) == 1


def test_permutes_of_the_built_library():
    if not os.path.exists(binding.LIB_PATH) or OBJDUMP is None:
        pytest.skip("liboctopus.so is not built, or no llvm-objdump")
    with open(binding.LIB_PATH, "rb") as f:
        objects = list(_code_objects(f.read()))

    def scan(elf):
        with tempfile.NamedTemporaryFile(suffix=".co") as f:
            f.write(elf)
            f.flush()
            text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", f.name], capture_output=True, text=True, timeout=300, check=True).stdout
        return _unsafe([line.split("//")[0].strip() for line in text.split("\n") if line.startswith("\t")])
    with ThreadPoolExecutor(max_workers=min(8, os.cpu_count())) as pool:
        found = list(pool.map(scan, objects))
    assert sum(n for n, _ in found) > 10000
    bad = [x for _, b in found for x in b]
    assert not bad, f"{len(bad)}, for instance {bad[:4]}"

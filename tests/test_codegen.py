"""A check on the generated code.  The compiler has placed the spill of a value that is
the same in every lane at the head of a block, in front of the instruction that gives the
lanes of a divergent branch back (s_or_b64 exec, exec, ..): the lanes that were off did
not store it, and a later reload brought what lay there.  A response came out scaled by
16.  No kernel may hold that pattern."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

FILES = ["kernels_gemm", "kernels_tiny", "kernels_layer"]


def spills_before_exec(lines):
    """(function, line, instruction) of every scratch access between a block's label and
    the restore of exec that opens the block."""
    found, fn, seen = [], None, None
    for no, line in enumerate(lines, 1):
        m = re.match(r"(_Z\w+):", line)
        if m:
            fn = m.group(1)
        if line.startswith(".LBB"):
            seen = []
        elif seen is not None:
            if re.match(r"\ts_or_b64 exec, exec", line):
                found += seen
                seen = None
            elif re.match(r"\ts_(cbranch|branch|endpgm)", line):
                seen = None
            elif "scratch_" in line:
                seen.append((fn, no, line.strip()))
    return found


def test_the_pattern_is_recognised():
    code = ["_Zk:", ".LBB0_1:", "\tscratch_store_dword off, v3, off", "\ts_or_b64 exec, exec, s[4:5]",
            "\tscratch_load_dword v3, off, off", ".LBB0_2:", "\tscratch_store_dword off, v4, off",
            "\ts_cbranch_scc1 .LBB0_1"]
    assert spills_before_exec(code) == [("_Zk", 3, "scratch_store_dword off, v3, off")]


@pytest.mark.slow
def test_no_spill_in_front_of_an_exec_restore(tmp_path):
    from paper_2203_09621_amd import build

    def assembly(name):
        out = tmp_path / (name + ".s")
        subprocess.run([build.hipcc(), *build._flags(), "--cuda-device-only", "-S",
                        os.path.join(build.CSRC, name + ".hip"), "-o", str(out)],
                       check=True, capture_output=True)
        with open(out) as fh:
            return fh.readlines()

    with ThreadPoolExecutor(max_workers=len(FILES)) as ex:
        for name, lines in zip(FILES, ex.map(assembly, FILES)):
            assert any("s_endpgm" in line for line in lines)
            assert spills_before_exec(lines) == [], name

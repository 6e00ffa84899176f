"""Where the compiler keeps registers in scratch memory, looked at in the assembly of the sources (no GPU): a store at
the head of a block where parted lanes meet again, ahead of the instruction that brings them back (s_or_b64 exec), leaves
the registers of the lanes that sat out behind; read back later they hold anything, addresses included.  (V > 16384 with
top-k: wrong sets A, and a memory fault.)"""
import os
import re
import subprocess

import pytest

from paper_2502_06352_amd import build


def _lost_stores(text):
    """function -> scratch instructions that stand ahead of the s_or_b64 exec of their block"""
    found, name, block = {}, None, []

    def end():
        back = next((i for i, t in enumerate(block) if t.startswith("s_or_b64 exec, exec,")), 0)
        lost = [t for t in block[:back] if t.startswith("scratch_")]
        if lost:
            found.setdefault(name, []).extend(lost)
        block.clear()

    for line in text.splitlines():
        t = line.strip()
        if re.match(r"\.LBB|; %bb\.", line):
            end()
        elif re.match(r"_Z\w+:", line):
            end()
            name = line.split(":")[0]
        elif t and t[0] not in ";.":
            block.append(t)
            if t.startswith("s_endpgm"):
                end()
    return found


SOURCES = ["lpp_verify.hip", "lpp_knn.hip", "lpp_attention.hip"]


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    d = tmp_path_factory.mktemp("asm")
    runs = [subprocess.Popen([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + build.FLAGS +
                             ["-w", "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, "--cuda-device-only", "-S",
                              os.path.join(build.CSRC, n), "-o", str(d / n)], stderr=subprocess.DEVNULL) for n in SOURCES]
    assert [r.wait() for r in runs] == [0] * len(SOURCES)
    return {n: (d / n).read_text() for n in SOURCES}


@pytest.mark.parametrize("source", SOURCES)
def test_no_register_is_spilled_for_some_of_its_lanes(source, assembly):
    assert assembly[source].count("s_endpgm") > 5
    assert _lost_stores(assembly[source]) == {}


def test_a_lost_store_is_found():
    head = "_Zf:\n; %bb.0:\n\ts_and_saveexec_b64 s[0:1], vcc\n\ts_cbranch_execz .LBB0_2\n; %bb.1:\n\tds_read_b32 v1, v0\n"
    lost, back = "\tscratch_store_dword off, v2, off offset:4\n", "\ts_or_b64 exec, exec, s[0:1]\n"
    assert _lost_stores(head + ".LBB0_2:\n" + lost + back + "\ts_endpgm\n") == {"_Zf": [lost.strip()]}
    assert _lost_stores(head + ".LBB0_2:\n" + back + lost + "\ts_endpgm\n") == {}

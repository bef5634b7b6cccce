"""The device assembly of the library's kernels, read for one fault of code generation that no value on the host shows."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

from paper_1912_08756_amd import build


def _early_copies(listing):
    """Joins of a divergent region (targets of its branch around it) at which vector registers are written between the label and
    the instruction that brings the region's other lanes back.  Lane writes of scalars (v_writelane) ignore the lane mask."""
    lines = listing.split("\n")
    joins = {m[1] for m in (re.search(r"s_cbranch_execz (\.LBB\S+)", l) for l in lines) if m}
    kernel, label, early, found = None, None, None, []
    for line in lines:
        m = re.match(r"(_Z\S+):", line)
        if m:
            kernel, early = m[1], None
            continue
        m = re.match(r"(\.LBB\S+):", line)
        if m:
            label, early = m[1], [] if m[1] in joins else None
            continue
        t = line.strip()
        if early is None or not t or t[0] in ";.":
            continue
        if t.startswith("s_or_b64 exec, exec"):
            if early:
                found.append((kernel, label, early))
            early = None
        elif re.match(r"s_(andn2_saveexec|and_saveexec|cbranch|branch|endpgm|setpc|barrier|(xor|mov|andn2)_b64 exec)", t):
            early = None
        elif re.match(r"(v_|scratch_load|ds_read|global_load|buffer_load)", t) and not t.startswith("v_writelane"):
            early.append(t.split(";")[0].strip())
    return found


def test_the_reader_finds_a_copy_before_the_lanes_are_back():
    text = """
_Zk:
\ts_and_saveexec_b64 s[0:1], vcc
\ts_cbranch_execz .LBB0_2
; %%bb.1:
\tglobal_store_dword v[0:1], v2, off
.LBB0_2:
\tv_writelane_b32 v9, s3, 1
%s\ts_or_b64 exec, exec, s[0:1]
\ts_endpgm
"""
    assert _early_copies(text % "") == []
    assert _early_copies(text % "\tv_mov_b32_e32 v5, v6\n") == [("_Zk", ".LBB0_2", ["v_mov_b32_e32 v5, v6"])]


def test_no_kernel_copies_registers_before_a_branch_s_lanes_are_back(tmp_path):
    """At its register limit the compiler splits a value's range at the join of a divergent region and may put the copy in front of
    the instruction that restores the lane mask: lanes that skipped the region keep what stood there before, addresses among
    it (encode_wave_kernel once: only wavefronts with missing items went astray)."""
    def listing(src):
        out = str(tmp_path / (src + ".s"))
        subprocess.run(["hipcc"] + build.FLAGS + ["--cuda-device-only", "-S", os.path.join(build.CSRC, src), "-o", out],
                       check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL, timeout=600)
        with open(out) as f:
            return f.read()
    kernels = 0
    with ThreadPoolExecutor(max_workers=6) as ex:
        for src, text in zip(build.SOURCES, ex.map(listing, build.SOURCES)):
            kernels += text.count("s_endpgm")
            assert _early_copies(text) == [], src
    assert kernels > 100

"""The assembly of the library's kernels, for one way the compiler has gone
wrong with regions of uniform branches left unstructured (a build flag here):
a flag that only the lanes of a divergent region set was kept as a lane mask of
all ones, so that after the region every lane took the flag's branch.  (The
join had merged a store at the end of the region with the same store after it;
63 lanes stored to undefined addresses.)  Such a mask is moved to all ones
under a narrowed exec and, unmasked, chooses the lanes once exec is whole."""
import importlib.util
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def unmasked(lines):
    """Positions where a region ends and a mask set to -1 within it decides."""
    found = []
    for i, line in enumerate(lines):
        if not re.match(r"\ts_or_b64 exec, exec, s\[", line):
            continue
        for use in lines[i + 1:i + 4]:
            m = re.match(r"\ts_and_saveexec_b64 s\[\d+:\d+\], (s\[\d+:\d+\])|\ts_and_b64 vcc, exec, (s\[\d+:\d+\])", use)
            if not m:
                continue
            mask = m.group(1) or m.group(2)
            last = next((ln for ln in reversed(lines[max(i - 400, 0):i]) if mask in ln), "")
            if last.startswith(f"\ts_mov_b64 {mask}, -1"):
                found.append(i)
            break
    return found


def functions(text):
    name, body = None, []
    for line in text.splitlines():
        m = re.match(r"(_Z\w+):", line)
        if m:
            name, body = m.group(1), []
        elif line.startswith(".Lfunc_end") and name:
            yield name, body
            name = None
        elif name:
            body.append(line)


def test_the_pattern_is_found():
    bad = ["\ts_and_saveexec_b64 s[26:27], vcc", "\tv_mov_b32_e32 v2, v3", "\ts_mov_b64 s[24:25], -1",
           "\tv_mov_b64_e32 v[0:1], s[18:19]", ".LBB0_1:", "\ts_or_b64 exec, exec, s[26:27]",
           "\ts_and_saveexec_b64 s[0:1], s[24:25]"]
    assert unmasked(bad) == [5]
    good = bad[:4] + ["\ts_and_b64 s[24:25], s[24:25], exec"] + bad[4:]
    assert unmasked(good) == []


@pytest.mark.parametrize("source", ["gp_device.hip", "gp_mutate.hip"])
def test_no_kernel_has_it(tmp_path, source):
    spec = importlib.util.spec_from_file_location("gp_build", os.path.join(ROOT, "paper_2110_11226_amd", "build.py"))
    build = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(build)
    if not shutil.which("hipcc") and not os.path.exists("/opt/rocm/bin/hipcc"):
        pytest.skip("no hipcc")
    out = tmp_path / "kernels.txt"
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC", "-Rpass-analysis=kernel-resource-usage")]
    subprocess.run([build.hipcc(), *flags, "-I", os.path.join(ROOT, "include"), "--cuda-device-only", "-S", "-o", str(out),
                    os.path.join(build.CSRC, source)], check=True, capture_output=True)
    n = 0
    for name, body in functions(out.read_text()):
        n += 1
        assert not unmasked(body), name
    assert n >= 4

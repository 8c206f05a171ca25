"""The evaluation kernel's interpreter: its generated sources, and its handler
table as assembled (every handler at its multiple of the stride)."""
import importlib.util
import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2110_11226_amd", "csrc")


def generator():
    spec = importlib.util.spec_from_file_location("gen_eval_asm", os.path.join(CSRC, "gen_eval_asm.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def test_headers_are_what_the_generator_writes(tmp_path, monkeypatch):
    monkeypatch.chdir(tmp_path)
    generator().main()
    for name in ("gp_eval_asm.h", "gp_eval_code.h"):
        assert (tmp_path / name).read_text() == open(os.path.join(CSRC, name)).read()


@pytest.mark.parametrize("freg", [0, 2, 8, "adjoint"])
@pytest.mark.parametrize("rows", [1, 2, 4])
def test_every_handler_lies_at_its_offset(tmp_path, rows, freg):
    clang = "/opt/rocm/lib/llvm/bin/clang"
    if not os.path.exists(clang) or not shutil.which("nm"):
        pytest.skip("no assembler")
    mod = generator()
    gen = mod.AdjGen(rows) if freg == "adjoint" else mod.Gen(rows, freg)
    text = "\n".join(ln.replace(".L", "L").replace("%=", "x") for ln in gen.text())
    src, obj = tmp_path / "t.s", tmp_path / "t.o"
    src.write_text('.amdgcn_target "amdgcn-amd-amdhsa--gfx950"\n.text\n.p2align 8\n' + text + "\n")
    subprocess.run([clang, "-c", "-target", "amdgcn-amd-amdhsa", "-mcpu=gfx950", str(src), "-o", str(obj)], check=True)
    at = {}
    for ln in subprocess.run(["nm", str(obj)], check=True, capture_output=True, text=True).stdout.splitlines():
        m = re.match(r"([0-9a-f]+) \w Lh(\d+)_x$", ln)
        if m:
            at[int(m.group(2))] = int(m.group(1), 16)
    assert sorted(at) == list(range(gen.adj["count"] if freg == "adjoint" else gen.sec["count"]))
    assert all(at[i] == at[0] + mod.STRIDE * i for i in at)

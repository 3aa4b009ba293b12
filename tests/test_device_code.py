"""What the built library's gfx950 code has to hold whichever way the compiler orders it: read from its own disassembly."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2502_09888_amd import build as hb

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled kernel name: [instruction, ...]} of libclimber.so"""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    d = tmp_path_factory.mktemp("code")
    shutil.copy(hb.LIB if os.path.exists(hb.LIB) else hb.build(), d / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=d, check=True, capture_output=True)
    out = {}
    for f in sorted(os.listdir(d)):
        if not f.endswith("gfx950"):
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", f], cwd=d, check=True, capture_output=True, text=True).stdout
        for line in text.splitlines():
            m = re.match(r"[0-9a-f]+ <(\S+)>:", line)
            if m:
                code = out.setdefault(m.group(1), [])
            elif line.startswith("\t"):
                code.append(line.split("//")[0].strip())
    return out


def test_bias_attention_waits_for_its_lds_reads_before_a_ring_stage_is_filled_again(kernels):
    # Keys and values from the cache: the copies of a later tile are issued behind a barrier that all copies so far are waited for at,
    # into the stage whose keys were read right before it: every wave has to wait for those reads as well, in the same place.  (From
    # rows, the fifth template argument, the value fragments' own assembly waits for them.)
    seen = 0
    for name, code in kernels.items():
        if not re.search(r"attn_bias_kernelILi\dE(Lb[01]E){3}Lb0E", name):
            continue
        for i, ins in enumerate(code):
            if ins != "s_barrier":
                continue
            waits = []
            for prev in reversed(code[max(0, i - 40):i]):
                if prev.startswith(("s_cbranch", "s_branch", "s_barrier")):
                    break
                if prev.startswith("s_waitcnt"):
                    waits.append(prev)
                    if "vmcnt(0)" in prev:
                        break
            if any("vmcnt(0)" in w for w in waits):
                seen += 1
                assert any("lgkmcnt(0)" in w for w in waits), (name, i, waits)
    assert seen > 0


def test_inline_assembly_of_several_instructions_keeps_its_inputs():
    # an output that an earlier instruction writes may share its register with an input that a later one reads, where the compiler knows
    # both to have one value, unless it is marked as an early clobber
    seen = 0
    for f in sorted(os.listdir(hb.CSRC)):
        if not f.endswith((".hip", ".h")):
            continue
        text = re.sub(r"//[^\n]*", "", open(os.path.join(hb.CSRC, f)).read())
        macros = dict(re.findall(r"#define (CLIMBER_\w+) (\".*\")$", text, flags=re.M))
        for m in re.finditer(r"\basm\b(?: volatile)?\s*\(", text):
            end, depth = m.end(), 1
            while depth:
                depth += {"(": 1, ")": -1}.get(text[end], 0)
                end += 1
            block = text[m.end():end - 1]
            for name, value in macros.items():
                block = block.replace(name, value)
            template, *operands = re.split(r"\s:\s", block)
            if template.count("\\n") == 0 or len(operands) < 2:
                continue
            seen += 1
            outs = re.findall(r'"([=+][^"]*)"', operands[0])
            assert outs and all("&" in o for o in outs), (f, " ".join(block.split())[:120])
    assert seen >= 3

"""What the compiler made of the kernels, from the built library's own gfx950 code object (no GPU)."""
import os
import re
import shutil
import subprocess

import pytest

LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "lib", "llvm", "bin")


@pytest.fixture(scope="module")
def code_object(tmp_path_factory):
    from paper_2505_13765_amd import build

    if build.stale():
        build.build(True)
    where = tmp_path_factory.mktemp("code_object")
    lib = shutil.copy(build.LIB, where / "lib.so")
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", str(lib)], check=True, capture_output=True)
    (code,) = [f for f in os.listdir(where) if "gfx950" in f]
    return str(where / code)


@pytest.fixture(scope="module")
def assembly(code_object):
    out = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", "--no-show-raw-insn", "--no-leading-addr", "--symbolize-operands", code_object],
                         check=True, capture_output=True, text=True).stdout
    return out.splitlines()


def writes_before_lanes_are_back(lines):
    """Places (kernel, instruction) where a block that a wave jumps to without a lane (s_cbranch_execz, a loop's last lane leaving) writes vector
    registers or memory before it takes its lanes back (s_or_b64 exec).  The compiler's register allocator has put copies of live values
    there, in kernels whose spilled scalars are read back at the top of such a block: the copies then happen in none of the lanes."""
    targets, name, per_kernel = {}, None, {}
    for line in lines:
        m = re.match(r"^(?:[0-9a-f]+ )?<(_Z\w+)>:", line)
        if m:
            name = m.group(1)
            per_kernel[name] = []
            targets[name] = set()
        elif name:
            per_kernel[name].append(line.strip())
            m = re.search(r"s_cbranch_execz (?:<)?(L\d+)", line)
            if m:
                targets[name].add(m.group(1))
    found = []
    for name, body in per_kernel.items():
        looking, written = False, []
        for line in body:
            m = re.match(r"^(?:[0-9a-f]+ )?<(L\d+)>:", line)
            if m:
                looking, written = m.group(1) in targets[name], []
                continue
            op = line.split(" ")[0].split("\t")[0]
            if not looking or not op:
                continue
            if re.match(r"s_or_b64\s+exec, exec|s_(or|andn2)_saveexec", line):
                found += [(name, w) for w in written]
                looking = False
            elif op.startswith(("ds_", "global_", "scratch_", "buffer_", "flat_")) or (
                    op.startswith("v_") and not op.startswith(("v_readlane", "v_writelane", "v_readfirstlane", "v_cmp"))):
                written.append(line)
            elif op.startswith(("s_cbranch", "s_branch", "s_endpgm")) or re.search(r"\bexec\b", line):
                looking = False
    return found, sum(len(t) for t in targets.values())


def test_no_block_writes_vectors_before_its_lanes_are_back(assembly):
    found, targets = writes_before_lanes_are_back(assembly)
    assert targets > 1000, "the disassembly was not understood"
    assert not found, found


def test_the_scan_finds_such_a_write():
    planted = ["<_Z1kv>:", "\ts_cbranch_execz L0", "\tv_add_u32_e32 v1, 1, v1", "<L0>:", "\tv_readlane_b32 s0, v9, 3", "\tv_mov_b32_e32 v7, 1",
               "\ts_or_b64 exec, exec, s[8:9]", "\ts_endpgm"]
    assert writes_before_lanes_are_back(planted) == ([("_Z1kv", "v_mov_b32_e32 v7, 1")], 1)
    planted[5], planted[6] = planted[6], planted[5]
    assert writes_before_lanes_are_back(planted)[0] == []


def vector_spills(code_object, pattern):
    notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", code_object], check=True, capture_output=True, text=True).stdout
    kernels = re.findall(r"\.name:\s+(_Z\S+).*?\.vgpr_spill_count:\s+(\d+)", notes, flags=re.S)
    return {n: int(k) for n, k in kernels if re.search(pattern, n)}


def test_groups_of_one_utterance_keep_their_weights_in_registers(code_object):
    """No vector register of the instances that calls of up to 8 utterances take lies in scratch memory (mode 1: the last template argument)."""
    spills = vector_spills(code_object, r"wind_group_(f32_)?kernelI\w*?Li1EEEv")
    assert len(spills) == 15 and not any(spills.values()), spills


def test_groups_of_larger_vocabularies_keep_their_weights_in_registers(code_object):
    """128 to 512 units: no vector register in scratch memory.  640 units: nine, which the kernel's description states."""
    spills = vector_spills(code_object, r"wind_group_vocab_kernelI")
    assert len(spills) == 5
    assert {int(re.search(r"kernelILi(\d)E", n).group(1)): k for n, k in spills.items() if k} in ({}, {5: 9}), spills

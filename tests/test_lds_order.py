"""Values that the lanes of a wave hand each other through the LDS without a barrier: the compiler has to keep the accesses in order.  It does across a
fence, and need not where it can tell two addresses or two types apart.  Looked for in its own optimised code, on every path (loops
included); no GPU."""
import functools
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _unfenced(function, first, second):
    """Lines that match `second` and are reached from one that matches `first` without a fence between.  `function`: the lines of its body."""
    entry = re.match(r"([\w.$-]+):|", function[0])[1] or ""
    blocks, successors, name = {entry: []}, {}, entry
    for line in function:
        label = re.match(r"([\w.$-]+):", line)
        if label:
            name = label[1]
            blocks[name] = []
        blocks[name].append(line)
    for name, lines in blocks.items():
        successors[name] = [s for line in lines for s in re.findall(r"label %([\w.$-]+)", line)]
    found, dirty, todo = set(), {entry: False}, [entry]
    while todo:
        name = todo.pop()
        state = dirty[name]
        for line in blocks[name]:
            if re.match(r"\s+fence ", line):
                state = False
            if state and re.search(second, line):
                found.add(line.strip())
            if re.search(first, line):
                state = True
        for s in successors[name]:
            if s not in dirty or state > dirty[s]:
                dirty[s] = state
                todo.append(s)
    return sorted(found)


@functools.lru_cache(maxsize=None)
def _device_code(source):
    """Optimised device code of a source: kernel name -> lines."""
    from paper_2108_08842_amd import build
    if shutil.which(build.hipcc_path()) is None:
        pytest.skip("no hipcc")
    text = subprocess.run([build.hipcc_path(), "--offload-arch=gfx950", "-O3", "-std=c++17", "--offload-device-only", "-S", "-emit-llvm", "-Xclang", "-target-feature",
                           "-Xclang", "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(build.PKG, "csrc"),
                           os.path.join(build.PKG, "csrc", source), "-o", "-"], check=True, capture_output=True, text=True).stdout
    return {m[1]: m[2].split("\n") for m in re.finditer(r"^define [^\n]*amdgpu_kernel [^\n]*@(\w+)\([^\n]*\n(.*?)^}", text, re.S | re.M)}


def _kernels(source, name):
    found = {k: lines for k, lines in _device_code(source).items() if f"{len(name)}{name}" in k}
    assert found, name
    return found


def test_the_search_itself():
    loop = ["entry:", "  br label %head", "head:", "  store i32 1, ptr addrspace(3) %a", "  %x = load float, ptr addrspace(3) %b", "  br i1 %c, label %head, label %out", "out:", "  ret void"]
    first, second = r"= load float, ptr addrspace\(3\)", r"store i32 .*, ptr addrspace\(3\)"
    fence = "  fence syncscope(\"wavefront\") release"
    assert len(_unfenced(loop, first, second)) == 1              # around the loop
    assert len(_unfenced(loop, second, first)) == 1              # straight on
    assert _unfenced([*loop[:3], fence, *loop[3:]], first, second) == [] and _unfenced([*loop[:4], fence, *loop[4:]], second, first) == []


def test_sign_words_of_the_next_sender_wait_for_the_last_reads():
    # k_dec_lo15_last: a wave's sign words are read (whole numbers; all else there is floats) up to the end of a sender, then written for the next one
    for name, lines in _kernels("eden_kernels_lo15.hip", "k_dec_lo15_last").items():
        assert any(re.search(r"= load (i32|i64|<\d+ x i32>), ptr addrspace\(3\)", line) for line in lines), name
        assert _unfenced(lines, r"= load (i32|i64|<\d+ x i32>), ptr addrspace\(3\)", r"store (i32|i64|<\d+ x i32>) .*, ptr addrspace\(3\)") == [], name


def test_sums_of_the_kept_values_wait_for_the_sender_before():
    # k_sparse_scatter_list: a sum that one lane has added to may be added to by another lane for the next sender
    for name, lines in _kernels("eden_kernels_sparse.hip", "k_sparse_scatter_list").items():
        assert any(re.search(r"store float .*, ptr addrspace\(3\)", line) for line in lines), name
        assert _unfenced(lines, r"store float .*, ptr addrspace\(3\)", r"= load float, ptr addrspace\(3\)") == [], name


def test_sign_words_are_read_in_the_type_they_are_written_in():
    # k_dec_lo14_last and its matrix-core forms: of the LDS's whole numbers none is read as half of what was stored
    for name, lines in _kernels("eden_kernels_lo14.hip", "k_dec_lo14_last").items():
        assert not any(re.search(r"= load i16, ptr addrspace\(3\)", line) for line in lines), name

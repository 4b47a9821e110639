"""The first layer's kernel: lanes read picture rows that other lanes of their wave have put into LDS.  Between such a store and the matrix instructions
that use what was read there has to be a wavefront fence on every path (from the source's intermediate code, where fences still stand)."""
import os
import re
import subprocess

from paper_2006_11735_amd import build

CSRC = os.path.join(os.path.dirname(os.path.abspath(build.__file__)), "csrc")


def blocks_of(body):
    """{label: [instructions]} and {label: successors} of a function's text; the first block's label is None."""
    blocks, cur = {None: []}, None
    for line in body.splitlines():
        m = re.match(r"^([\w.]+):", line)
        if m:
            cur = m.group(1)
            blocks[cur] = []
        elif line.startswith("  "):
            blocks[cur].append(line.strip())
    succ = {k: re.findall(r"label %([\w.]+)", " ".join(t for t in b if re.match(r"br |switch |label |i\d+ -?\d+, label", t))) for k, b in blocks.items()}
    return blocks, succ


def test_rows_are_fenced_before_they_are_multiplied(tmp_path):
    out = tmp_path / "stem.ll"
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + build.FLAGS + ["--cuda-device-only", "-S", "-emit-llvm", "-o", str(out),
                                                                                     os.path.join(CSRC, "conv_stem.hip")], check=True, capture_output=True)
    kernels = re.findall(r"^define [^\n]*amdgpu_kernel[^\n]*@(\w*conv_stem_pool_kernel\w*)\([^\n]*\n(.*?)^}", out.read_text(), re.S | re.M)
    assert len(kernels) == 12                    # one or two chunks, seven or eight rows, three ways to requantise
    for name, body in kernels:
        blocks, succ = blocks_of(body)
        begin, todo = {None: set()}, [None]
        products = fences = stores = 0
        while todo:
            at = todo.pop()
            open_stores = set(begin[at])
            for k, t in enumerate(blocks[at]):
                if re.match(r"store i32 .*addrspace\(3\)", t):
                    open_stores.add((at, k))
                    stores += 1
                elif 'fence syncscope("wavefront' in t or 'fence syncscope("workgroup' in t:
                    open_stores.clear()
                    fences += 1
                elif "llvm.amdgcn.mfma" in t and "call" in t:
                    products += 1
                    assert not open_stores, (name, t, sorted(blocks[a][i] for a, i in open_stores))
            for to in succ[at]:
                if to not in begin or not open_stores <= begin[to]:
                    begin[to] = begin.get(to, set()) | open_stores
                    todo.append(to)
        assert products >= 16 and stores >= 16 and fences >= 1, name

"""The order of the chain kernel's copies into LDS and its reads, from the assembly of the source as it is built: a copy counts as done for the
whole workgroup when its wave has waited for all of its loads (vmcnt(0)) and a barrier has followed."""
import os
import re
import subprocess

from paper_2006_11735_amd import build

CSRC = os.path.join(os.path.dirname(os.path.abspath(build.__file__)), "csrc")


def blocks_of(lines):
    """Basic blocks of a kernel: [instructions], [successors' indexes]."""
    blocks, label_at, cur = [[]], {}, []
    for line in lines:
        m = re.match(r"^(\.LBB\w+):", line)
        if m:
            if blocks[-1]:
                blocks.append([])
            label_at[m.group(1)] = len(blocks) - 1
            continue
        text = line.split(";")[0].strip()
        if not text or text.startswith(".") or text.endswith(":"):
            continue
        blocks[-1].append(text)
        if re.match(r"s_c?branch|s_endpgm", text):
            blocks.append([])
    succ = []
    for i, b in enumerate(blocks):
        last = b[-1] if b else ""
        to = [label_at[w] for w in last.split() if w in label_at] if "branch" in last else []
        if not last.startswith(("s_branch", "s_endpgm")) and i + 1 < len(blocks):
            to.append(i + 1)
        succ.append(to)
    return blocks, succ


def in_cycles(succ):
    """The blocks that can come round to themselves."""
    def reach(start):
        seen, todo = set(), list(succ[start])
        while todo:
            b = todo.pop()
            if b not in seen:
                seen.add(b)
                todo += succ[b]
        return seen
    return {i for i in range(len(succ)) if i in reach(i)}


def unordered_copies(blocks, succ):
    """For every block the state it may begin with: {(copy, whether its wave has waited for it)} of the copies that are not done for everybody."""
    def step(state, text, at):
        if text.startswith("buffer_load") and text.endswith(" lds"):
            return state | {(at, False)}
        if text.startswith("s_waitcnt") and re.search(r"vmcnt\(0\)", text):
            return frozenset((c, True) for c, _ in state)
        if text.startswith("s_barrier"):
            return frozenset((c, w) for c, w in state if not w)
        return state
    begin = [frozenset()] * len(blocks)
    todo = [0]
    reached = {0}
    while todo:
        i = todo.pop()
        state = begin[i]
        for k, text in enumerate(blocks[i]):
            state = step(state, text, (i, k))
        for j in succ[i]:
            if j not in reached or not state <= begin[j]:
                reached.add(j)
                begin[j] = begin[j] | state
                todo.append(j)
    return begin, step


def test_copies_are_done_before_they_are_read(tmp_path):
    out = tmp_path / "chain.s"
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + build.FLAGS + ["--cuda-device-only", "-S", "-o", str(out), os.path.join(CSRC, "conv_chain.hip")],
                   check=True, capture_output=True)
    kernels = re.findall(r"^(_Z\w*conv_chain_kernel\w*):(.*?)^\s*\.section", out.read_text(), re.S | re.M)
    assert len(kernels) == 2
    for name, text in kernels:
        blocks, succ = blocks_of(text.splitlines())
        loop = in_cycles(succ)
        begin, step = unordered_copies(blocks, succ)
        copies = {(i, k) for i, b in enumerate(blocks) for k, t in enumerate(b) if t.startswith("buffer_load") and t.endswith(" lds")}
        assert sum(1 for i, _ in copies if i in loop) >= 5 and sum(1 for i, _ in copies if i not in loop) >= 16, name
        reads = 0
        for i in loop:
            state = begin[i]
            for k, t in enumerate(blocks[i]):
                # the layers run in a loop: what was copied before it is there when it begins ...
                if t.startswith("ds_read_b128"):
                    reads += 1
                    early = sorted(blocks[c[0]][c[1]] for c, _ in state if c[0] not in loop)
                    assert not early, (name, t, early)
                # ... and what a layer copies, for the one after the next, before the next layer begins
                if (i, k) in copies:
                    assert (i, k) not in {c for c, _ in state}, (name, t)
                state = step(state, t, (i, k))
        assert reads >= 36, name

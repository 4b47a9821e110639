"""The waits of the 3x3 kernel that keeps its weights in registers, from the assembly of the source as it is built: what its counted waits count on has been issued on every
path, and its products, which the compiler does not know for products, have the wait states that the compiler gives them elsewhere.  None of it shows in outputs but now
and then."""
import os
import re
import subprocess

import pytest

from paper_2006_11735_amd import build
from test_chain_waits import CSRC, blocks_of

PRODUCTS = 36                                          # of a round: 18 K fragments, two halves of the channels
SUM_STATES, SOURCE_STATES = 12, 2                      # wait states that the compiler puts between this product and a reader or writer of its sums, between a vector
                                                       # instruction and the product that reads its result


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    out = tmp_path_factory.mktemp("keep") / "keep.s"
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + build.FLAGS + ["--cuda-device-only", "-S", "-o", str(out), os.path.join(CSRC, "conv_keep.hip")],
                   check=True, capture_output=True)
    found = re.findall(r"^(_Z\w*conv_keep_kernel\w*):(.*?)^\s*\.section", out.read_text(), re.S | re.M)
    assert len(found) == 4
    return [(name, *blocks_of(text.splitlines())) for name, text in found]


def is_copy(t):
    return t.startswith("buffer_load") and t.endswith(" lds")


def is_request(t):
    return t.startswith(("buffer_", "global_", "flat_", "scratch_"))


def reach(succ, start, stop=lambda b: False):
    """The blocks that can follow block start, none of them behind one that stops the way"""
    seen, todo = set(), list(succ[start])
    while todo:
        b = todo.pop()
        if b not in seen:
            seen.add(b)
            if not stop(b):
                todo += succ[b]
    return seen


def fewest_younger(blocks, succ, copies):
    """{rounds: the fewest requests that a way from a copy, past no other copy, to the barrier that ends its tile issues}"""
    least, fewest = {}, {}
    todo = [(i, k + 1, 0, 0) for i, k in copies]
    while todo:
        i, k, products, n = todo.pop()
        for t in blocks[i][k:]:
            if is_copy(t) or products > 8 * PRODUCTS:
                break
            if t.startswith("s_barrier"):
                assert products % PRODUCTS == 0
                fewest[products // PRODUCTS] = min(n, fewest.get(products // PRODUCTS, n))
                break
            products += t.startswith("v_mfma")
            n += is_request(t)
        else:
            for j in succ[i]:
                if n < least.get((j, products), n + 1):
                    least[j, products] = n
                    todo.append((j, 0, products, n))
    return fewest


def test_a_tiles_rows_have_landed_before_its_barrier(kernels):
    for name, blocks, succ in kernels:
        has = {what: {i for i, b in enumerate(blocks) if any(t.startswith(what) for t in b)} for what in ("v_mfma", "s_barrier")}
        after_products = set().union(*(reach(succ, i) for i in has["v_mfma"]))
        copies = [(i, k) for i, b in enumerate(blocks) for k, t in enumerate(b) if is_copy(t) and i in after_products and reach(succ, i) & has["v_mfma"]]
        assert copies, name
        fewest = fewest_younger(blocks, succ, copies)
        assert set(range(1, 9)) <= set(fewest), name
        # the tile's own waits stand where nothing but its barrier can follow; for one, two, three and more rounds, in the order of their counts
        waits = set()
        for i in after_products - has["v_mfma"]:
            ends = i in has["s_barrier"]
            follow = reach(succ, i, has["s_barrier"].__contains__)
            if ends or (follow & has["s_barrier"] and not follow & has["v_mfma"]):
                waits |= {int(n) for n in re.findall(r"vmcnt\((\d+)\)", "\n".join(blocks[i]).split("s_barrier")[0])}
        waits = sorted(waits)
        assert len(waits) == 4, (name, waits)
        for rounds in range(1, 9):
            assert waits[min(rounds, 4) - 1] <= fewest[rounds], (name, rounds, waits, fewest)


def registers(text):
    """The vector and accumulation registers that an instruction names"""
    out = set()
    for kind, first, last, one in re.findall(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
        out |= {(kind, int(one))} if one else {(kind, r) for r in range(int(first), int(last) + 1)}
    return out


def states_of(t):
    return int(t.split()[1]) + 1 if t.startswith("s_nop") else 1


def operands(t):
    return [o.strip() for o in t.split(None, 1)[1].split(", ")]


def followers(blocks, succ, i, k, states):
    """(wait states between, instruction) of the instructions within so many of instruction k of block i, on every way; a product ends a way where the caller says so"""
    todo, least = [(i, k + 1, 0)], {}
    while todo:
        b, at, n = todo.pop()
        for t in blocks[b][at:]:
            if n >= states or (yield n, t):
                break
            n += states_of(t)
        else:
            for j in succ[b]:
                if n < least.get(j, states):
                    least[j] = n
                    todo.append((j, 0, n))


def hazards(blocks, succ):
    found = []
    for i, b in enumerate(blocks):
        for k, t in enumerate(b):
            if not t.startswith("v_"):
                continue
            product = t.startswith("v_mfma")
            mine = operands(t)
            sums = registers(mine[0])
            walk = followers(blocks, succ, i, k, SUM_STATES if product else SOURCE_STATES)
            ends = None
            while True:
                try:
                    n, u = walk.send(ends)
                except StopIteration:
                    break
                ends = False
                if u.startswith("v_mfma"):
                    theirs = operands(u)
                    if product and theirs[0] == mine[0] and theirs[3] in (mine[0], mine[3]):      # the sum's next product, or the next round's first
                        bad, ends = registers(theirs[1] + " " + theirs[2]) & sums, True
                    else:
                        bad = registers(u) & sums
                else:
                    # (what a product adds to is read late: nobody may write it meanwhile)
                    bad = product and registers(u) & (sums | registers(mine[3]))
                if bad:
                    found.append((t, n, u))
    return found


def test_sums_and_sources_have_their_wait_states(kernels):
    for name, blocks, succ in kernels:
        assert sum(t.startswith("v_mfma") for b in blocks for t in b) == 2 * PRODUCTS, name
        assert not hazards(blocks, succ), (name, hazards(blocks, succ)[:3])

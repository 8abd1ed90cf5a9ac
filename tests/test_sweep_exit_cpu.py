"""How a workgroup of the one-launch sweeps leaves. The last workgroup out
readies the control words for the next sweep while wavefronts of other
workgroups may still wait and give up. What the kernels do with the flag is read
from their source, and every interleaving of it is played through: the next
sweep must not find a flag that it takes for its own."""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1503_01287_amd", "csrc")
KERNELS = [("k_sweep.hip", "k_sweep"), ("k_vanka.hip", "k_vanka_sweep")]


def protocol(name, kernel):
    """(steps after the loop over tiles, the flag is cleared at the end, it
    names its sweep)."""
    text = open(os.path.join(CSRC, name)).read()
    body = text[text.index(f" {kernel}(const"):]
    body = body[:re.search(r"^}", body, re.M).start()]
    tail = body[body.index("while (t < a.n"):]
    tail = tail[re.search(r"^    }$", tail, re.M).end():]  # the loop's brace stands at the function's own indentation
    steps = [k for _, k in sorted((tail.index(s), k) for s, k in (("__syncthreads()", "barrier"), ("(exits, 1)", "count"))
                                  if s in tail)]
    stored = re.findall(r"agent_store\(gave_up, ([^;]*)\);", text)
    tested = re.findall(r"bad = agent_load\(gave_up\) ([^;]*);", text)
    assert stored and tested and "count" in steps
    cleared = "agent_store(gave_up, 0)" in tail
    numbered = all("sweep" in s for s in stored if s != "0") and all(t.startswith("==") and "sweep" in t for t in tested)
    if numbered:  # a new number every sweep, taken from the word that the last workgroup writes
        assert re.search(r"sweep = static_cast<unsigned>\(\*turn\) \+ 1u", body)
        assert "agent_store(turn, static_cast<int>(sweep))" in tail
    return steps, cleared, numbered


def next_sweep_is_clear(steps, cleared, numbered, groups=2, waves=2):
    """Every wavefront may give up in its last tile; wavefront 0 counts its
    workgroup out."""
    plan = [["give up", *[k for k in steps if k == "barrier" or w == 0]] for _ in range(groups) for w in range(waves)]
    seen, todo = set(), [((0,) * len(plan), 0, 0)]
    while todo:
        state = todo.pop()
        if state in seen:
            continue
        seen.add(state)
        at, out, flag = state
        if all(a == len(p) for a, p in zip(at, plan)):
            if flag == 2 or (flag and not numbered):  # (this sweep is number 1, the next one 2)
                return False
            continue
        for k, p in enumerate(plan):
            if at[k] == len(p):
                continue
            move, o, f = {k}, out, flag
            if p[at[k]] == "barrier":  # all wavefronts of the workgroup pass it together
                move = {q for q in range(len(plan)) if q // waves == k // waves}
                if any(at[q] == len(plan[q]) or plan[q][at[q]] != "barrier" for q in move):
                    continue
            elif p[at[k]] == "count":
                o += 1
                f = 0 if cleared and o == groups else f
            else:
                f = 1
            todo.append((tuple(a + (q in move) for q, a in enumerate(at)), o, f))
    return True


def test_the_model_tells_the_protocols_apart():
    assert next_sweep_is_clear(["barrier", "count"], True, False)
    assert next_sweep_is_clear(["count"], False, True)
    assert not next_sweep_is_clear(["count"], True, False)
    assert not next_sweep_is_clear(["count", "barrier"], True, False)
    assert not next_sweep_is_clear(["count"], False, False)


@pytest.mark.parametrize("name,kernel", KERNELS)
def test_a_sweep_leaves_nothing_to_the_next(name, kernel):
    assert next_sweep_is_clear(*protocol(name, kernel))

"""How a workgroup of the one-launch sweeps leaves. The last workgroup out
clears the control words for the next sweep, so no wavefront of the launch may
write one after that. The order of the steps after the loop over tiles is read
from the kernels' source and every interleaving of it is played through."""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1503_01287_amd", "csrc")
STEPS = {"__syncthreads()": "barrier", "atomicAdd(exits, 1)": "count"}


def steps_after_the_loop(name, kernel):
    text = open(os.path.join(CSRC, name)).read()
    body = text[text.index(f" {kernel}(const"):]
    end = re.search(r"^}", body, re.M).start()
    # the loop over tiles ends with a brace at the function's own indentation
    tail = body[:end][body[:end].index("while (t < a.n"):]
    tail = tail[re.search(r"^    }$", tail, re.M).end():]
    found = sorted((tail.index(s), k) for s, k in STEPS.items() if s in tail)
    assert [k for _, k in found].count("count") == 1
    return [k for _, k in found]


def ends_clear(steps, groups=2, waves=2):
    """Wavefronts may still give up (write the flag) in their last tile;
    wavefront 0 counts its workgroup out, the last one clears the flag."""
    plan = [["give up", *[k for k in steps if k == "barrier" or w == 0]] for _ in range(groups) for w in range(waves)]
    seen, todo = set(), [((0,) * len(plan), 0, 0)]
    while todo:
        state = todo.pop()
        if state in seen:
            continue
        seen.add(state)
        at, out, flag = state
        if all(a == len(p) for a, p in zip(at, plan)):
            if flag:
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
                f = 0 if o == groups else f
            else:
                f = 1
            todo.append((tuple(a + (q in move) for q, a in enumerate(at)), o, f))
    return True


def test_the_model_tells_the_orders_apart():
    assert ends_clear(["barrier", "count"])
    assert not ends_clear(["count"])
    assert not ends_clear(["count", "barrier"])


@pytest.mark.parametrize("name,kernel", [("k_sweep.hip", "k_sweep"), ("k_vanka.hip", "k_vanka_sweep")])
def test_workgroups_leave_as_a_whole(name, kernel):
    assert ends_clear(steps_after_the_loop(name, kernel))

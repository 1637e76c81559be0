"""How the workgroups of the construction's search that stands behind one that was given up part (construct_again_kernel): all orders of what
they do, in a model of the words they leave in memory, and the way out of the kernel that the model counts on."""
import os
import re

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
NOT_BEGUN, BEGUN, LEFT = range(3)


def explore(others, steps, left_when_done=True):
    """Every state that the first workgroup and `others` reach with `steps` + 1 exchanges.  Returns how often it ended, and the states in
    which nobody can go on; asserts that the first is by itself once it goes on alone.

    A state: the words of the two sets (0: as cleared, which is bit 63 set, else 1 + the bit written), the workgroups' state words, and
    where everyone is: ("out",) not begun, ("publish", t), ("look", t), ("gave up",), ("done",), ("gone",), of the first also ("alone", i):
    it has asked the first i others, and ("wait", i)."""
    n = others + 1
    bit = lambda t: (t >> 1) & 1
    start = (((None,) * n,) * 2, (NOT_BEGUN,) * n, (("publish", 0),) + (("out",),) * others)

    def present(words, t):
        return all((1 if w is None else w) == bit(t) for w in words[t & 1])

    def put(row, i, v):
        return row[:i] + (v,) + row[i + 1:]

    def moves(s):
        words, state, where = s
        for i in range(n):
            at = where[i]
            go = lambda to, words=words, state=state: (words, state, put(where, i, to))
            if at[0] == "out":                               # it may also never find room while the others are there
                if state[i] == NOT_BEGUN:
                    yield go(("publish", 0), state=put(state, i, BEGUN))
                else:
                    yield go(("gone",))
            elif at[0] == "publish":
                t = at[1]
                yield go(("look", t), words=put(words, t & 1, put(words[t & 1], i, bit(t))))
            elif at[0] == "look":
                t = at[1]
                if present(words, t):
                    yield go(("publish", t + 1) if t < steps else ("done",))
                else:
                    yield go(("gave up",))                   # its patience ends at any time
            elif i > 0 and at[0] in ("gave up", "done"):
                yield go(("gone",), state=put(state, i, LEFT) if at[0] == "gave up" or left_when_done else state)
            elif at[0] == "gave up":
                yield go(("alone", 1))
            elif at[0] == "alone":
                k = at[1]
                if k == n:
                    assert all(w == ("gone",) or (w == ("out",) and state[j] != NOT_BEGUN) for j, w in enumerate(where) if j), s
                    yield go(("done",))
                elif state[k] == NOT_BEGUN:
                    yield go(("alone", k + 1), state=put(state, k, LEFT))
                else:
                    yield go(("wait", k))
            elif at[0] == "wait" and state[at[1]] == LEFT:
                yield go(("alone", at[1] + 1))

    seen, todo, ended, stuck = {start}, [start], 0, []
    while todo:
        s = todo.pop()
        successors = list(moves(s))
        if not successors:
            over = s[2][0] == ("done",) and all(w == ("gone",) for w in s[2][1:])
            ended += over
            if not over:
                stuck.append(s)
        for m in successors:
            if m not in seen:
                seen.add(m)
                todo.append(m)
    return ended, stuck


@pytest.mark.parametrize("steps", [0, 1, 2, 5])
@pytest.mark.parametrize("others", [1, 2, 3])
def test_every_order_ends(others, steps):
    ended, stuck = explore(others, steps)
    assert ended > 0 and not stuck, stuck[:3]


@pytest.mark.parametrize("steps", [0, 1, 3])
def test_the_model_finds_the_wait_for_one_that_is_done(steps):
    """One that leaves without a word when all steps are done is waited for without end by the first, if that has given up."""
    _, stuck = explore(2, steps, left_when_done=False)
    assert stuck and all(where[0][0] == "wait" and ("gone",) in where[1:] for _, _, where in stuck)


def test_one_way_out_for_those_that_began():
    with open(os.path.join(HERE, "..", "paper_2604_17789_amd", "csrc", "construct.hip")) as f:
        source = f.read()
    kernel = source[source.index("void construct_again_kernel("):]
    kernel = re.sub(r"//[^\n]*", "", kernel[:kernel.index("\n}\n")])
    begun = kernel[kernel.index("if (!goes) return;") + len("if (!goes) return;"):]
    assert re.findall(r"[^;{}]*;\s*return\b", begun) == re.findall(r"[^;{}]*__hip_atomic_store\(state \+ blockIdx\.x, kLeft, __ATOMIC_RELEASE[^;{}]*;\s*return\b", begun)
    assert len(re.findall(r"\breturn;", begun)) == 1

"""The count of a bottom-up invocation's scanned edges, which decides for the
whole team whether the query goes on bottom-up: every workgroup has to read
the same value, also where consecutive bottom-up invocations are separated by
their closing barrier alone.  All interleavings of a small team are explored
with the word indexes that the source uses."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
QUERY = os.path.join(ROOT, "paper_1607_05707_amd", "csrc", "irgl_query.h")

TEAM, INVOCATIONS = 2, 6


def _index(pattern, text):
    """The index expression of the count in the statement `pattern` names
    (None: no such statement; 0 where the count is one word)."""
    m = re.search(pattern, text)
    return None if m is None else (lambda rot, e=m.group(1) or "0": eval(e, {"rot": rot}))


def _protocol():
    text = open(QUERY).read()
    word = r"&ctrl->bu_scan(?:\[([^\]]*)\])?"
    clear = _index(r"atomic_store\(" + word, text)
    add = _index(r"add_block_total<B>\(r\.edges - edges_before, " + word, text)
    read = _index(r"atomic_load\(" + word, text)
    assert add and read
    return clear, add, read


def _steps(clear, add, read, wg):
    """A workgroup's accesses in order: (what, invocation, word)."""
    out = []
    for rot in range(INVOCATIONS):
        if wg == 0 and clear:
            out.append(("clear", rot, clear(rot)))
        out += [("add", rot, add(rot)), ("barrier", rot, None), ("read", rot, read(rot))]
    return out


def test_every_workgroup_reads_the_same_count():
    clear, add, read = _protocol()
    steps = [_steps(clear, add, read, wg) for wg in range(TEAM)]
    amount = [[10 ** (2 * wg) * (rot + 1) for rot in range(INVOCATIONS)] for wg in range(TEAM)]
    total = [sum(a[rot] for a in amount) for rot in range(INVOCATIONS)]
    todo = [((0,) * TEAM, (0, 0, 0), (0,) * TEAM)]  # positions, words, each workgroup's last read
    seen = set(todo)
    while todo:
        pos, words, last = todo.pop()
        for wg in range(TEAM):
            if pos[wg] == len(steps[wg]):
                continue
            what, rot, word = steps[wg][pos[wg]]
            w, mine = list(words), list(last)
            if what == "barrier":  # passed once every workgroup has come to it
                arrived = [[i for i, s in enumerate(steps[o]) if s[:2] == ("barrier", rot)][0] for o in range(TEAM)]
                if any(pos[o] < arrived[o] for o in range(TEAM)):
                    continue
            elif what == "clear":
                w[word] = 0
            elif what == "add":
                w[word] += amount[wg][rot]
            else:
                got = w[word] - (0 if clear else last[wg])
                assert got == total[rot], f"workgroup {wg} reads {got} for {total[rot]} in invocation {rot}"
                mine[wg] = w[word]
            state = (pos[:wg] + (pos[wg] + 1,) + pos[wg + 1:], tuple(w), tuple(mine))
            if state not in seen:
                seen.add(state)
                todo.append(state)

"""The workgroup samplers' shared counters, checked in the kernels' sources on the CPU.

A counter in LDS is reset by thread 0, added to by all waves and read by all waves.
Between any two of these that are not of the same kind there has to be a barrier on
every path (a thread's own reads and resets apart): a wave that is late would else
read what comes next, and the waves would disagree on how far a loop goes or whether
the next barrier is reached at all.

The check walks the statements of a kernel: both ways of every branch, loops with any
number of iterations, with break, continue and return, local lambdas where they are
called.  It knows nothing of conditions that go together."""
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2101_06192_amd", "csrc")
COUNTERS = ("s_item", "s_u", "s_c", "s_cnt", "s_set", "s_ext")
BARRIERS = ("__syncthreads", "lds_barrier")


def _source(name):
    with open(os.path.join(CSRC, name)) as f:
        text = f.read()
    text = re.sub(r"//[^\n]*|/\*.*?\*/", " ", text, flags=re.S)
    return "\n".join(line for line in text.splitlines() if not line.lstrip().startswith("#"))


def _closing(text, i):
    """Index of the bracket that closes the one at text[i]."""
    pair = {"(": ")", "{": "}", "[": "]"}
    depth, o, c = 0, text[i], pair[text[i]]
    for j in range(i, len(text)):
        depth += (text[j] == o) - (text[j] == c)
        if depth == 0:
            return j
    raise AssertionError("unbalanced source")


class _Parser:
    """Statements as tuples: ("do", text), ("lambda", name, body), ("if", condition, then,
    otherwise), ("loop", head, body), ("block", statements), ("jump", word)."""

    def __init__(self, text):
        self.t, self.i = text, 0

    def space(self):
        while self.i < len(self.t) and self.t[self.i].isspace():
            self.i += 1

    def word(self, *words):
        self.space()
        for w in words:
            if re.match(rf"{w}\b", self.t[self.i:]):
                self.i += len(w)
                return w
        return None

    def bracket(self, opening):
        self.space()
        assert self.t[self.i] == opening, self.t[self.i:self.i + 40]
        end = _closing(self.t, self.i)
        inner = self.t[self.i + 1:end]
        self.i = end + 1
        return inner

    def statement(self):
        self.space()
        if self.t[self.i] == "{":
            return ("block", _Parser(self.bracket("{")).all())
        if self.word("if"):
            cond, then = self.bracket("("), self.statement()
            return ("if", cond, then, self.statement() if self.word("else") else ("block", []))
        if self.word("for", "while"):
            return ("loop", self.bracket("("), self.statement())
        if self.word("do"):
            body = self.statement()
            assert self.word("while")
            head = self.bracket("(")
            self.space()
            self.i += 1  # ;
            return ("block", [body, ("loop", head, body)])
        jump = self.word("break", "continue", "return")
        if jump:
            self.i = self.t.index(";", self.i) + 1
            return ("jump", jump)
        start = self.i
        while self.t[self.i] != ";":
            self.i = _closing(self.t, self.i) + 1 if self.t[self.i] in "({[" else self.i + 1
        text = self.t[start:self.i]
        self.i += 1
        named = re.match(r"auto (\w+) = \[&\]", text)
        if named:
            at = text.index("{", _closing(text, text.index("(", named.end())) if "(" in text else 0)
            return ("lambda", named.group(1), ("block", _Parser(text[at + 1:_closing(text, at)]).all()))
        return ("do", text)

    def all(self):
        out = []
        while True:
            self.space()
            if self.i >= len(self.t):
                return out
            out.append(self.statement())


# a state: for every counter what has happened to it since the last barrier; None: not reached
def _join(a, b):
    if a is None or b is None:
        return b if a is None else a
    return {k: a.get(k, frozenset()) | b.get(k, frozenset()) for k in {*a, *b}}


CLASHES = [{"read", "reset"}, {"read", "add"}, {"reset", "add"}, {"own read", "add"}]


class _Walk:
    def __init__(self):
        self.lambdas, self.found, self.calling = {}, set(), []

    def event(self, state, counter, kind, text):
        state = dict(state)
        state[counter] = seen = state.get(counter, frozenset()) | {kind}
        for clash in CLASHES:
            if clash <= seen and kind in clash:
                self.found.add((counter, " / ".join(sorted(clash)), " ".join(text.split())[:70]))
        return state

    def text(self, state, text, lead):
        """One expression or simple statement, its parts in order."""
        if state is None or "__shared__" in text:
            return state
        names = "|".join(map(re.escape, (*COUNTERS, *self.lambdas, *BARRIERS)))
        for m in re.finditer(rf"(&?)\b({names})\b(\s*=(?!=))?", text):
            ref, name, assigned = m.groups()
            if name in BARRIERS:
                state = {}
            elif name in self.lambdas:
                if text[m.end():m.end() + 1] == "(" and name not in self.calling:
                    self.calling.append(name)
                    out, _, _, ret = self.run(self.lambdas[name], state, lead)
                    state = _join(out, ret)
                    self.calling.pop()
            elif ref:
                state = self.event(state, name, "add", text)
            elif assigned:
                state = self.event(state, name, "reset" if lead else "add", text)
            else:
                state = self.event(state, name, "own read" if lead else "read", text)
        return state

    def run(self, node, state, lead=False):
        """States after the node: falling through, at break, at continue, at return."""
        if state is None:
            return None, None, None, None
        kind = node[0]
        if kind == "do":
            return self.text(state, node[1], lead), None, None, None
        if kind == "lambda":
            self.lambdas[node[1]] = node[2]
            return state, None, None, None
        if kind == "jump":
            return tuple(None if node[1] != w else state for w in ("", "break", "continue", "return"))
        if kind == "block":
            b = c = r = None
            for child in node[1]:
                state, b1, c1, r1 = self.run(child, state, lead)
                b, c, r = _join(b, b1), _join(c, c1), _join(r, r1)
            return state, b, c, r
        if kind == "if":
            state = self.text(state, node[1], lead)
            x = self.run(node[2], state, lead or "tid == 0" in node[1])
            y = self.run(node[3], state, lead)
            return tuple(map(_join, x, y))
        assert kind == "loop"
        endless = not node[1].replace(";", "").strip()
        ret = leave = None
        while True:
            state = self.text(state, node[1], lead)
            f, b, c, r = self.run(node[2], state, lead)
            leave, ret = _join(leave, b), _join(ret, r)
            again = _join(state, _join(f, c))
            if again == state:
                return (leave if endless else _join(state, leave)), None, None, ret
            state = again


def clashes(text):
    """What the check finds in the kernels of a source."""
    found = set()
    for m in re.finditer(r"__global__", text):
        start = text.index("{", _closing(text, text.index("(", text.index("_kernel", m.start()))))
        walk = _Walk()
        walk.run(("block", _Parser(text[start + 1:_closing(text, start)]).all()), {})
        found |= walk.found
    return sorted(found)


def test_the_check_finds_what_it_is_for():
    kernel = "__global__ void a_kernel(int x) { __shared__ unsigned s_c; %s }"
    fill = "if (tid == 0) s_c = 0; __syncthreads(); wave_append(list, &s_c); __syncthreads(); n = s_c;"
    for body, bad in ((fill, False),
                      (fill + fill, True),
                      (fill + "__syncthreads();" + fill, False),
                      ("for (;;) { %s if (n == 0) break; }" % fill, True),
                      ("for (;;) { %s if (n == 0) break; __syncthreads(); }" % fill, False),
                      ("if (tid == 0) s_c = 0; while (x > 0) { f(); __syncthreads(); } g(&s_c);", True),
                      ("auto h = [&]() { __syncthreads(); }; if (tid == 0) s_c = 0; h(); g(&s_c);", False),
                      ("if (tid == 0) { s_c = 0; n = s_c; }", False)):
        assert bool(clashes(kernel % body)) == bad, body


@pytest.mark.parametrize("source", ["wilson_jump.hip", "wilson_tile.hip", "wilson_hub.hip",
                                    "wilson_lds.hip", "wilson_hyb.hip"])
def test_barriers_between_uses_of_a_counter(source):
    assert clashes(_source(source)) == []

"""The hand-over of windows whose workgroup stopped waiting (sc_gsc_fast.hip, next_left): a model of its steps, every one atomic, with all
orders of all workgroups tried.  Whatever the order, every window is written exactly once, and only when the rows of all before it are published."""
import pytest

ROWS, READY, LEFT = "rows", "ready", "left"


class Model:
    """windows: per window 's' for whole chunks, decided by the workgroup of its slot, or 'L' for one long chunk, decided by a workgroup of its own."""

    def __init__(self, windows):
        self.kind = windows
        procs = []
        for w, k in enumerate(windows):
            procs.append(("publish", w) if k == "s" else ("wait", w))
            if k == "L":
                procs.append(("decide", w))
        self.start = (False, (frozenset(),) * len(windows), (0,) * len(windows), tuple(procs))

    def free(self, words, w):       # a marked window can be taken
        return LEFT in words[w] and (self.kind[w] == "s" or READY in words[w])

    def steps(self, state):
        head_left, words, written, procs = state

        def at(t, i, v):
            return t[:i] + (v,) + t[i + 1:]

        def known(w):
            return all(ROWS in words[v] for v in range(w))

        for i, (step, *a) in enumerate(procs):
            def to(*nxt, head_left=head_left, words=words, written=written):
                return (head_left, words, written, at(procs, i, nxt))

            def word(w, add=(), drop=()):
                return at(words, w, (words[w] | set(add)) - set(drop))

            w = a[0] if a else None
            if step == "publish":
                yield to("wait", w, words=word(w, [ROWS]))
            elif step == "decide":
                yield to("clusters", w, words=word(w, [ROWS]))
            elif step == "clusters":
                yield to("look", words=word(w, [READY]))
            elif step == "look":                            # after all that it has published has arrived
                yield to(*(("search", 0) if head_left else ("end",)))
            elif step == "wait":
                if known(w) and (self.kind[w] == "s" or READY in words[w]):
                    looks = self.kind[w] == "s" and w + 1 < len(self.kind)      # (nobody waits for the rows of the last one)
                    yield to(*(("look",) if looks else ("end",)), written=at(written, w, written[w] + 1))
                yield to("mark", w)                         # stops waiting, at any moment
            elif step == "mark":
                yield to("tell", words=word(w, [LEFT]))
            elif step == "tell":
                yield to("search", 0, head_left=True)
            elif step == "search":
                if w == len(self.kind) or ROWS not in words[w]:
                    yield to("end")
                else:
                    yield to(*(("claim", w) if self.free(words, w) else ("search", w + 1)))
            elif step == "claim":
                yield to(*(("write", w) if LEFT in words[w] else ("search", w + 1)), words=word(w, (), [LEFT]))
            elif step == "write":
                assert known(w)
                yield to("search", w + 1, written=at(written, w, written[w] + 1))


@pytest.mark.parametrize("windows", ["s", "sss", "ssss", "L", "Ls", "sL", "LL", "sLs"])
def test_every_window_is_written_once(windows):
    m = Model(windows)
    seen, todo, ends = {m.start}, [m.start], 0
    while todo:
        state = todo.pop()
        following = list(m.steps(state))
        if not following:
            ends += 1
            assert all(p == ("end",) for p in state[3]) and all(n == 1 for n in state[2]), state
        for nxt in following:
            if nxt not in seen:
                seen.add(nxt)
                todo.append(nxt)
    assert ends > 0

"""The hand-over between a decode launch's merging wavefronts and its chunks (csrc/decode_merge.h), as a model: every order in which
the steps of the chunks' wavefronts and of one block's merging wavefront can take place, the merging wavefront giving up at any of
its looks.  No order stops short, merges twice or leaves a word behind.  (The kernels themselves: test_gpu_decode_merge.py.)"""
import pytest

DONE = ("done", 0, 0)


def _next(state):
    """All states that one more step leads to.  Per slot: has the chunk said that it ends soon, has the merging wavefront given it
    up, has its partial landed; the hand-over word; merges so far; (step, slot, what it knows) of each chunk and of the merger."""
    soon, given, landed, ready, merges, chunks, merger = state
    n = len(soon)
    put = lambda t, i, v: t[:i] + (v,) + t[i + 1:]

    def after(soon=soon, given=given, landed=landed, ready=ready, merges=merges, chunk=None, merger=merger):
        return soon, given, landed, ready, merges, chunks if chunk is None else put(chunks, *chunk), merger

    def look(k):        # state words first, then the partials
        return soon[k] if k < n else landed[k - n]

    def put_back(k):
        return {"soon": put(soon, k, 0), "given": put(given, k, 0), "landed": put(landed, k, 0)}

    for i, (step, k, late) in enumerate(chunks):
        if step == "tiles":
            yield after(soon=put(soon, i, 1), chunk=(i, ("store", 0, given[i])))       # one atomic: its bit, and the other's
        elif step == "store":
            yield after(landed=put(landed, i, 1), chunk=(i, ("landed", 0, late)))
        elif step == "landed":
            yield after(chunk=(i, ("word", 0, 0) if late else DONE))
        elif step == "word":
            yield after(chunk=(i, ("look", 0, 0) if ready else DONE))
        elif step == "look" and k < 2 * n:
            yield after(chunk=(i, ("look", k + 1, 0) if look(k) else DONE))
        elif step == "look":
            yield after(ready=0, chunk=(i, ("put back", 0, 0))) if ready else after(chunk=(i, DONE))
        elif step == "put back":
            yield after(chunk=(i, ("put back", k + 1, 0)), **put_back(k)) if k < n else after(merges=merges + 1, chunk=(i, DONE))
    step, k, first = merger
    if step == "wait":
        yield after(merger=("give up", 0, 0))
        if all(soon):
            yield after(merger=("partials", 0, 0))
    elif step == "partials":
        if k == n:
            yield after(merger=("put back", 0, 0))
        elif landed[k]:
            yield after(merger=("partials", k + 1, 0))
    elif step == "give up":      # first: the slots whose chunks came first
        yield (after(given=put(given, k, 1), merger=("give up", k + 1, first | soon[k] << k)) if k < n
               else after(merger=("first", 0, first)))
    elif step == "first":
        if k == n:
            yield after(ready=1, merger=("look", 0, 0))
        elif landed[k] or not first >> k & 1:
            yield after(merger=("first", k + 1, first))
    elif step == "look" and k < 2 * n:
        yield after(merger=("look", k + 1, 0) if look(k) else DONE)
    elif step == "look":
        yield after(ready=0, merger=("put back", 0, 0)) if ready else after(merger=DONE)
    elif step == "put back":
        yield after(merger=("put back", k + 1, 0), **put_back(k)) if k < n else after(merges=merges + 1, merger=DONE)


@pytest.mark.parametrize("n", [1, 2, 3])
def test_every_order_merges_once_and_leaves_nothing(n):
    start = ((0,) * n, (0,) * n, (0,) * n, 0, 0, (("tiles", 0, 0),) * n, ("wait", 0, 0))
    seen, todo, ends = {start}, [start], set()
    while todo:
        state = todo.pop()
        more = set(_next(state))
        if not more:
            ends.add(state)
        todo += more - seen
        seen |= more
    assert ends == {((0,) * n, (0,) * n, (0,) * n, 0, 1, (DONE,) * n, DONE)}

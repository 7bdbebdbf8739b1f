"""The exchange of maxima between the workgroups of one launch (csrc/ssg_meet.h), a model of it, run through every interleaving at small
sizes on the CPU: where a workgroup overwrites its share of the tensor afterwards, as the Adam step does, and where the source stays
and another launch may write over the words.

A share is two cells, read and written one at a time.  A workgroup reads its share, leaves its maximum in its word, and looks at the
words until it has all maxima; at any time it may give up on one that is missing, form it from the share's cells and look again:
what it formed counts only if the word is still not there, and is then left there.  With all maxima it overwrites its share.  No
workgroup need have started before another one gives up or has ended."""
import pytest

CELLS = 2


def explore(count, reads, in_place=True, lost_words=False):
    """Every outcome of `count` workgroups: the set of the maxima they ended with.  reads(k): the cells (share, index) that
    workgroup k reads for its own maximum, later ones for another's.  in_place: shares are overwritten; lost_words: another launch
    writes over words at any time."""
    true = {(k, c): 1 + CELLS * k + c for k in range(count) for c in range(CELLS)}
    written = 1000                                            # a new code under the old scale: larger than any true value
    # a workgroup: (stage, position in the stage, running maximum, which share it forms, maxima it has, its result)
    start = tuple(("read", 0, 0, k, (None,) * count, None) for k in range(count))
    first = (start, (None,) * count, frozenset())             # workgroups, words, overwritten cells
    seen, todo, results = {first}, [first], set()

    def successors(state):
        groups, words, new = state
        for k, (stage, at, top, j, have, result) in enumerate(groups):
            def to(g, w=words, n=new):
                return groups[:k] + (g,) + groups[k + 1:], w, n
            if stage in ("read", "form"):
                cells = reads(j)
                if at < len(cells):
                    value = written if cells[at] in new else true[cells[at]]
                    yield to((stage, at + 1, max(top, value), j, have, None))
                elif stage == "read":
                    yield to(("look", 0, 0, k, have, None), words[:k] + (top,) + words[k + 1:])
                else:                                         # look again: what was formed counts only if there is nothing
                    late = words[j]
                    got = have[:j] + (top if late is None else late,) + have[j + 1:]
                    yield to(("leave" if late is None else "look", 0, top, j, got, None))
            elif stage == "leave":
                yield to(("look", 0, 0, k, have, None), words[:j] + (top,) + words[j + 1:])
            elif stage == "look":
                missing = [i for i in range(count) if have[i] is None]
                if not missing:
                    yield to(("write", 0, 0, k, have, max(have)))
                for i in missing:
                    if words[i] is not None:
                        yield to(("look", 0, 0, k, have[:i] + (words[i],) + have[i + 1:], None))
                    else:
                        yield to(("form", 0, 0, i, have, None))
            elif stage == "write" and at < CELLS:
                yield to((stage, at + 1, 0, k, have, result), words, new | {(k, at)} if in_place else new)
        for i in range(count):
            if lost_words and words[i] is not None and any(g[0] != "write" for g in groups):
                yield groups, words[:i] + (None,) + words[i + 1:], new

    while todo:
        state = todo.pop()
        following = list(successors(state))
        if not following:
            assert all(g[0] == "write" for g in state[0]), "a workgroup that never ends"
            results.add(tuple(g[5] for g in state[0]))
        for s in following:
            if s not in seen:
                seen.add(s)
                todo.append(s)
    return results, max(true.values())


def own_cells(k):
    return [(k, c) for c in range(CELLS)]


@pytest.mark.parametrize("count", [2, 3])
def test_every_workgroup_gets_the_maximum(count):
    results, top = explore(count, own_cells)
    assert results == {(top,) * count}


def test_words_of_the_ring_may_be_lost_where_the_source_stays():
    results, top = explore(2, own_cells, in_place=False, lost_words=True)
    assert results == {(top,) * 2}


def test_losing_words_where_shares_are_overwritten_is_found():
    """Why launches that overwrite their shares have words of their own: in the ring, where another launch can take a word away,
    a maximum would be formed from new codes."""
    results, top = explore(2, own_cells, lost_words=True)
    assert any(r != (top,) * 2 for r in results)


def test_reading_a_cell_of_another_share_is_found():
    """Where the last workgroup reads the first one's cell too (what stood in for elements beyond the tensor's end once), a late
    workgroup meets new codes: the search has to see it."""
    results, top = explore(3, lambda k: own_cells(k) + ([(0, 0)] if k == 2 else []))
    assert any(r != (top,) * 3 for r in results)

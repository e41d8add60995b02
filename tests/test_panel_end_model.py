"""Model of how a panel without pivoting ends (k_fast_commit<false>): the workgroups of a shift
read the panel state word by word, accept their column and count themselves in; the last to
arrive writes the state, word by word.  Every interleaving is walked; a workgroup must see the
state of before or of after (done) as a whole, since from a mixture it would accept columns of
the panel before it again.  Counting only the workgroups that have a column, as was done once,
lets the others of a ragged panel read while the state is being written."""
import itertools

import pytest

OLD = dict(k0=0, kb=2, done=0)      # the panel at column 2 ...
N = 3                               # ... of which one column is left, of two a panel holds
NEW = dict(k0=2, kb=1, done=1)


def column_of(view):
    """First column a workgroup takes the panel to start at; None: it leaves at once."""
    k0 = view["k0"] + view["kb"]
    return None if view["done"] or k0 >= N else k0


def outcomes(counted, order):
    """Columns that the workgroups take for the panel's first, over all interleavings of a
    workgroup with a column and one without; `order` is how the last arrival writes."""
    seen = set()
    words = ("k0", "kb", "done")

    def walk(mem, pos, views, count, writer):
        moved = False
        for g in (0, 1):
            if pos[g] < len(words):                       # reads one word
                w = words[pos[g]]
                v = dict(views[g], **{w: mem[w]})
                p = tuple(x + (i == g) for i, x in enumerate(pos))
                walk(mem, p, tuple(v if i == g else x for i, x in enumerate(views)), count, writer)
                moved = True
            elif pos[g] == len(words):                    # acts on what it read, arrives
                start = column_of(views[g])
                seen.add(start)
                p = tuple(x + (i == g) for i, x in enumerate(pos))
                arrives = start is not None and (g == 0 or counted == 2)
                c = count + arrives
                walk(mem, p, views, c, 0 if arrives and c == counted else writer)
                moved = True
        if writer is not None and writer < len(order):    # the last arrival writes one word
            m = dict(mem, **{order[writer]: NEW[order[writer]]})
            walk(m, pos, views, count, writer + 1)
            moved = True
        return moved

    walk(dict(OLD), (0, 0), ({}, {}), 0, None)
    return seen


@pytest.mark.parametrize("order", list(itertools.permutations(("k0", "kb", "done"))))
def test_all_workgroups_counted_see_one_state(order):
    assert outcomes(2, order) <= {2, None}


def test_counting_only_workgroups_with_a_column_mixes_states():
    assert any(outcomes(1, o) - {2, None} for o in itertools.permutations(("k0", "kb", "done")))

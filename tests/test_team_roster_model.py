"""Model of how the workgroups of a pivoting panel sign in (k_bk_team): every interleaving of
their steps is walked, with more workgroups than the team needs, some of which start only when
the others have ended.  The panel must be run either by a whole team, each rank once, or by the
first workgroup alone; and whatever has started must be able to end without the rest."""
import pytest

# a workgroup: (step, rank, size it saw); steps: new, close (the last of the team), post (writes
# the size it closed with), poll, give (the first one closes for itself), end
NEW = ("new", -1, 0)


def moves(state, need, gather):
    """Successors of a state: (workgroup, state)."""
    (count, closed, size), wgs = state
    for g, (step, r, s) in enumerate(wgs):
        def to(w, shared=(count, closed, size)):
            return g, (shared, wgs[:g] + (w,) + wgs[g + 1:])
        if step == "new":
            shared = (count + 1, closed, size)
            if closed or count >= need:
                yield to(("end", -1, 0), shared)
            elif count == need - 1 and gather:
                yield to(("close", count, 0), shared)
            else:
                yield to(("poll", count, 0), shared)
        elif step == "close":
            yield to(("post" if not closed else "poll", r, need), (count, True, size))
        elif step == "post":
            yield to(("end" if s == 1 else "poll", r, s), (count, closed, s))
        elif step == "poll":
            if size:
                yield to(("end", r, size))
            elif r == 0:
                yield to(("give", r, 0))       # it may run out of polls at any time
        elif step == "give":
            if closed:
                yield to(("poll", r, 0), (count, True, size))
            else:
                yield to(("post", r, 1), (count, True, size))


def reachable(need, grid, gather):
    start = ((0, False, 0), (NEW,) * grid)
    seen, todo = {start}, [start]
    while todo:
        x = todo.pop()
        for _, y in moves(x, need, gather):
            if y not in seen:
                seen.add(y)
                todo.append(y)
    return seen


def can_end(state, need, gather, memo):
    """Whether the workgroups that have started can all end by themselves."""
    live = [g for g, w in enumerate(state[1]) if w[0] not in ("new", "end")]
    if not live:
        return True
    if state not in memo:
        memo[state] = False
        memo[state] = any(can_end(y, need, gather, memo) for g, y in moves(state, need, gather) if g in live)
    return memo[state]


@pytest.mark.parametrize("gather", [True, False])
@pytest.mark.parametrize("need,grid", [(1, 1), (1, 3), (2, 2), (2, 3), (3, 3), (3, 4)])
def test_whole_team_or_first_workgroup_alone(need, grid, gather):
    memo, ends = {}, set()
    for state in reachable(need, grid, gather):
        assert can_end(state, need, gather, memo)
        wgs = state[1]
        if all(w[0] == "end" for w in wgs):
            run = sorted((r, s) for _, r, s in wgs if 0 <= r < s)   # a rank past the size leaves
            assert run in ([(0, 1)], [(r, need) for r in range(need)])
            ends.add(len(run))
    assert ends == ({1, need} if gather else {1})

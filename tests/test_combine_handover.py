"""The hand-over of the cross-work-group combine, as a model on the CPU.

The last work-group waits a bounded number of looks for the others' partials;
then it marks the slots of those that are missing and leaves, and the
work-group that counts the last mark off combines.  The model takes
every memory operation of that protocol as one step and tries every order in
which the steps of all work-groups can happen: each must end, with one result,
folded from all partials, and a workspace of zeros.  Protocols with one step
left out or out of place must fail the same check, so that it is known to look.
"""
import pytest

MARK = 1


def _partial(i):
    return 10 + i


def _word(i):
    return ("word", i)


def _waiter(last, rounds, wrong):
    """The last work-group: a generator of memory operations, sent their results."""
    for _ in range(rounds + 1):
        seen = []
        for i in range(last):
            seen.append((yield ("load", _word(i))))
        if all(w > MARK for w in seen):
            yield ("result", tuple(seen) + (_partial(last),))
            for i in range(last):
                yield ("store", _word(i), 0)
            return
    if wrong != "own partial late":
        yield ("store", _word(last), _partial(last))
    marks = 0
    for i in range(last):
        w = yield ("load", _word(i))
        if w > MARK:
            continue
        if wrong == "mark by a store":
            yield ("store", _word(i), MARK)
        elif not (yield ("cas", _word(i), w, MARK)):
            continue
        marks += 1
    left = yield ("add", -(last if wrong == "all counted" else marks))
    if wrong == "own partial late":
        yield ("store", _word(last), _partial(last))
    if left == 0:
        yield from _finish(last)


def _arriver(index, last, wrong):
    if wrong == "look and store":
        found = yield ("load", _word(index))
        yield ("store", _word(index), _partial(index))
    else:
        found = yield ("swap", _word(index), _partial(index))
    if found == MARK and (yield ("add", 1)) == 0:
        yield from _finish(last)


def _finish(last):
    seen = []
    for i in range(last + 1):
        seen.append((yield ("load", _word(i))))
    yield ("result", tuple(seen))
    for i in range(last + 1):
        yield ("store", _word(i), 0)


def _step(op, memory, pending, results):
    """One operation on (memory, pending, results): the new ones and its own result."""
    m, out = dict(memory), None
    if op[0] == "load":
        out = m.get(op[1], 0)
    elif op[0] == "store":
        m[op[1]] = op[2]
    elif op[0] == "swap":
        out, m[op[1]] = m.get(op[1], 0), op[2]
    elif op[0] == "cas":
        out = m.get(op[1], 0) == op[2]
        if out:
            m[op[1]] = op[3]
    elif op[0] == "add":
        pending += op[1]
        out = pending
    else:
        results = results + (op[1],)
    return frozenset((k, v) for k, v in m.items() if v), pending, results, out


def _explore(count, rounds, wrong=None):
    """Every order of steps from the start; the bad ends met.  A work-group's
    state is the list of results its operations have had."""
    last = count - 1
    make = [(lambda i=i: _arriver(i, last, wrong)) for i in range(last)] + [lambda: _waiter(last, rounds, wrong)]
    want = (tuple(_partial(i) for i in range(count)),)
    ops = {}

    def next_op(g, past):
        if (g, past) not in ops:
            run = make[g]()
            try:
                op = next(run)
                for r in past:
                    op = run.send(r)
            except StopIteration:
                op = None
            ops[g, past] = op
        return ops[g, past]

    start = (frozenset(), 0, (), ((),) * count)
    todo, met, bad = [start], {start}, []
    while todo:
        memory, pending, results, past = todo.pop()
        ready = [(g, op) for g in range(count) if (op := next_op(g, past[g])) is not None]
        if not ready and (results != want or pending != 0 or memory):
            bad.append((sorted(memory, key=str), pending, results))
        for g, op in ready:
            m, p, res, out = _step(op, memory, pending, results)
            nxt = (m, p, res, past[:g] + (past[g] + (out,),) + past[g + 1:])
            if nxt not in met:
                met.add(nxt)
                todo.append(nxt)
    return bad, len(met)


@pytest.mark.parametrize("count, rounds", [(2, 0), (2, 1), (2, 3), (3, 0), (3, 1), (4, 0)])
def test_every_order_ends_with_one_result_and_a_clear_workspace(count, rounds):
    bad, states = _explore(count, rounds)
    assert not bad, bad[:3]
    assert states > 10


@pytest.mark.parametrize("wrong", ["own partial late", "mark by a store", "all counted", "look and store"])
def test_a_step_out_of_place_is_found(wrong):
    bad, _ = _explore(3, 0, wrong)
    assert bad

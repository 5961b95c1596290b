"""The order of the resident CG's device-coherent stores, as a model on the CPU:
every state that two workgroups can reach when a workgroup's stores arrive in
any order between its waits (stores to one word stay in order).  Nobody may
take a slot or a z that an earlier meeting left, and nobody may wait for ever.
Two workgroups are enough: what one of them takes from another depends on that
pair's stores, and further ones only make both wait longer.  The slots' number
and how far ahead a slot is emptied are read from the kernel's source."""
import os
import re

import pytest

SOURCE = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                      "paper_1812_08942_amd", "csrc", "gr_sgd.hip")
ITERATIONS = 4


def _constant(text, name):
    if name.isdigit():
        return int(name)
    return int(re.search(r"constexpr int %s = (\d+);" % name, text).group(1))


def _of_the_kernel():
    with open(SOURCE) as f:
        text = f.read()
    ahead = re.findall(r"st_agent\(at\(epoch \+ (\w+), blockIdx\.x\) \+ lane, kResEmpty\)", text)
    assert len(ahead) == 1  # one place that empties
    return _constant(text, "kResEpochs"), _constant(text, ahead[0])


def _program(epochs, ahead, early):
    """A workgroup's steps: ("put", word, value), ("take", word, value) of the
    other's word, ("wait",).  early: z is asked for before the second meeting
    is complete, as the waves that do not collect it do."""
    ops, e = [], 0

    def publish():
        ops.append(("put", ("slot", e % epochs), e))

    def collect():
        ops.append(("take", ("slot", e % epochs), e))
        ops.append(("put", ("slot", (e + ahead) % epochs), None))

    publish()  # the mean of b
    collect()
    e = 1
    ops.append(("put", ("z", 1), "start"))
    publish()  # r.z and b.b
    collect()
    ops.append(("take", ("z", 1), "start"))
    for it in range(ITERATIONS):
        e += 1
        ops.append(("wait",))
        publish()  # p.q
        collect()
        ops.append(("put", ("z", it % 2), it))
        ops.append(("put", ("z", (it + 1) % 2), None))
        e += 1
        publish()  # r.z and r.r
        if early:
            ops.append(("take", ("z", it % 2), it))
        collect()
        if not early:
            ops.append(("take", ("z", it % 2), it))
    e += 1
    ops.append(("wait",))
    publish()  # the mean of y
    collect()
    return tuple(ops)


def _faults(epochs, ahead, early):
    """What can go wrong: a set of ("stale", word, wanted, taken) and
    ("stuck", ...); empty for a sound protocol."""
    ops = _program(epochs, ahead, early)
    words = tuple([("slot", k) for k in range(epochs)] + [("z", 0), ("z", 1)])
    at = {w: k for k, w in enumerate(words)}
    # per workgroup: its next step, its words as they have arrived, its
    # stores on the way
    first = ((0, (None,) * len(words), ()),) * 2
    seen, todo, faults = {first}, [first], set()
    while todo:
        state = todo.pop()
        nexts = []
        for me in (0, 1):
            pc, mem, sent = state[me]

            def became(pc, mem, sent):
                mine = (pc, mem, sent)
                nexts.append((mine, state[1]) if me == 0 else (state[0], mine))

            for i, (w, v) in enumerate(sent):
                if all(x[0] != w for x in sent[:i]):  # one word's stores in order
                    became(pc, mem[:at[w]] + (v,) + mem[at[w] + 1:], sent[:i] + sent[i + 1:])
            if pc == len(ops):
                continue
            op = ops[pc]
            if op[0] == "put":
                became(pc + 1, mem, sent + ((op[1], op[2]),))
            elif op[0] == "wait":
                if not sent:
                    became(pc + 1, mem, sent)
            else:
                there = state[1 - me][1][at[op[1]]]
                if there is not None:
                    if there != op[2]:
                        faults.add(("stale", op[1][0], op[2], there))
                    became(pc + 1, mem, sent)
        if not nexts and any(s[0] < len(ops) for s in state):
            faults.add(("stuck", state[0][0], state[1][0]))
        for s in nexts:
            if s not in seen:
                seen.add(s)
                todo.append(s)
    return faults


@pytest.mark.parametrize("early", [False, True])
def test_no_stale_value_is_taken(early):
    epochs, ahead = _of_the_kernel()
    assert _faults(epochs, ahead, early) == set()


def test_the_model_sees_a_slot_emptied_too_late_and_too_early():
    # two epochs ahead: no wait lies between a product's emptying and the
    # next product's use of the slot
    assert any(f[0] == "stale" and f[1] == "slot" for f in _faults(4, 2, False))
    # four ahead is the slot just taken, which the other may not have read
    assert any(f[0] == "stuck" for f in _faults(4, 4, False))

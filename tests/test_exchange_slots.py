"""CPU model of the slots through which a plane's work-groups exchange p and the next
column in the eigensolver's reduction when they share one L2.

A slot is its own flag: it holds "unset" until its value of the step is published, and a
reader loads until nothing it needs is unset.  Slots rotate over three steps.  During step k
each slot of step k + 1 is set back by its writer before that writer publishes step k, and a
work-group that has nothing to publish at step k + 1 leaves before it reads step k.

The model runs every wave as a sequence of single stores and loads under random schedules
(stores become visible in program order, as the waits in the kernel make them) and fails when
a value of another step is read or when nothing can move.  Two slots instead of three,
setting back after publishing, and work-groups that stay to read must each fail."""
import random

import pytest


def _steps(F, W, waves, w, v, n_slots, set_back_first, leave):
    """Events of wave v of work-group w: ("s", slot, value), ("read", slots, k), ("b",)."""
    nwv, gw = W * waves, w * waves + v
    own = list(range(gw, F, nwv))
    last_wg = max([j for u in range(waves) for j in range(w * waves + u, F, nwv)], default=-1)
    ev = []
    for kb in range(1, F):
        k = kb - 1
        back = [("s", ("p", (k + 1) % n_slots, j), None) for j in own if j > kb]
        back += [("s", ("c", (k + 1) % n_slots), None) for j in own if j == kb + 1]
        out = [("s", ("p", k % n_slots, j), k) for j in own if j >= kb]
        out += [("s", ("c", k % n_slots), k) for j in own if j == kb]
        ev += back + out if set_back_first else out + back
        if leave and last_wg <= kb and kb + 1 < F:
            return ev
        need = [("p", k % n_slots, j) for j in range(kb, F)] + [("c", k % n_slots)]
        ev += [("read", need[v::waves], k), ("b",)]
    return ev


def _run(F, W, seed, n_slots=3, set_back_first=True, leave=True, waves=2):
    rng = random.Random(seed)
    ids = [(w, v) for w in range(W) for v in range(waves)]
    evs = {i: _steps(F, W, waves, *i, n_slots, set_back_first, leave) for i in ids}
    pos = {i: 0 for i in ids}
    part = {i: 0 for i in ids}                  # loads of the current poll already done
    bars = {i: 0 for i in ids}
    at = {i: False for i in ids}                # waits at its barrier
    mem = {}
    bias = {i: rng.choice((1, 1, 8)) for i in ids}       # some waves run slower
    idle = 0
    while True:
        live = [i for i in ids if pos[i] < len(evs[i])]
        if not live:
            return True
        if idle > 4000:
            return False                        # nothing can move
        i = rng.choices(live, [1.0 / bias[j] for j in live])[0]
        idle += 1
        e = evs[i][pos[i]]
        if e[0] == "s":
            mem[e[1]] = e[2]
        elif e[0] == "read":
            got = mem.get(e[1][part[i]]) if e[1] else e[2]
            if got is None:                     # still unset: poll again from the start
                part[i] = 0
                continue
            if got != e[2]:
                return False
            part[i] += 1
            if part[i] < len(e[1]):
                continue
            part[i] = 0
        else:                                   # the work-group's barrier
            if not at[i]:
                at[i], bars[i] = True, bars[i] + 1
            if any(bars[(i[0], v)] < bars[i] for v in range(waves)):
                continue
            at[i] = False
        pos[i] += 1
        idle = 0


@pytest.mark.parametrize("F,W", [(6, 2), (9, 2), (9, 3), (13, 3)])
def test_three_slots_are_safe(F, W):
    assert all(_run(F, W, seed) for seed in range(300))


@pytest.mark.parametrize("mistake", [dict(n_slots=2), dict(set_back_first=False), dict(leave=False)])
def test_mistakes_are_seen(mistake):
    assert not all(_run(13, 3, seed, **mistake) for seed in range(300))

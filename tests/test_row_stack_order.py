"""Launches of several small layers, a workgroup per (layer, row), beside each other and beside other work: whether every workgroup comes to
its end on a chip that has room for few of them at once.  The rule that places a workgroup is the library's (row_stack_plan.h, compiled
for the host); the chip is a model: workgroups go to the XCDs by turns, an XCD starts those of a launch in their order, launches of several
streams in any order, each as soon as there is room, and a workgroup ends when the one it waits for has ended."""
import ctypes as C
import os
import random

import pytest

from paper_2101_05453_amd import build as libbuild

XCDS = 8


@pytest.fixture(scope="module")
def place():
    if not os.path.exists(libbuild.HOSTMATH_LIB):
        libbuild.build_hostmath()
    L = C.CDLL(libbuild.HOSTMATH_LIB)
    L.hm_row_stack_place.argtypes = [C.c_int32] * 4 + [C.c_void_p]

    def call(block, rows, dirs, order):
        out = (C.c_int32 * 4)()
        L.hm_row_stack_place(block, rows, dirs, order, out)
        return tuple(out)

    return call


def links_by_start(place, rows, dirs):
    started = {}

    def start(block):
        chain = place(block, rows, dirs, 0)[0]
        order = started[chain] = started.get(chain, -1) + 1
        _, d, row, layer = place(block, rows, dirs, order)
        return layer, d, row

    return start


def links_by_index(place, rows, dirs):
    def start(block):
        _, d, row, _ = place(block, rows, dirs, 0)
        return block // rows, d, row

    return start


def run(place, launches, room, rng, way):
    """launches: (layers, rows, dirs), layers of one direction.  Whether all end."""
    queues = [[] for _ in range(XCDS)]  # of each XCD: of each launch, the workgroups still to start
    starts, ended, running = [], set(), [[] for _ in range(XCDS)]
    for i, (L, rows, dirs) in enumerate(launches):
        first = rng.randrange(XCDS)
        blocks = list(range(L * rows * dirs))
        for x in range(XCDS):
            queues[x].append([b for b in blocks if (b + first) % XCDS == x])
        starts.append(way(place, rows, dirs))
    while any(q for x in queues for q in x) or any(running):
        moved = False
        for x in rng.sample(range(XCDS), XCDS):
            waiting = [i for i, q in enumerate(queues[x]) if q]
            if waiting and len(running[x]) < room:
                i = rng.choice(waiting)
                layer, d, row = starts[i](queues[x][i].pop(0))
                running[x].append((i, layer, d, row))
                moved = True
            for w in list(running[x]):
                i, layer, d, row = w
                dirs = launches[i][2]
                if layer < dirs or (i, layer - dirs, d, row) in ended:
                    running[x].remove(w)
                    assert w not in ended
                    ended.add(w)
                    moved = True
        if not moved:
            return False
    assert len(ended) == sum(L * rows * dirs for L, rows, dirs in launches)  # every (layer, row) by one workgroup
    return True


@pytest.mark.parametrize("room", [1, 2, 5])
def test_every_workgroup_ends(place, room):
    rng = random.Random(room)
    for _ in range(150):
        launches = []
        for _ in range(rng.randint(1, 6)):
            dirs = rng.randint(1, 2)
            L = rng.randint(2, 6 // dirs)
            launches.append((L, rng.randint(1, 256 // (L * dirs)), dirs))
        assert run(place, launches, room, rng, links_by_start), launches


def test_links_by_the_index_alone_do_not(place):
    """The model tells the difference."""
    rng = random.Random(7)
    assert not all(run(place, [(3, 4, 1), (3, 4, 1)], 1, rng, links_by_index) for _ in range(50))


@pytest.mark.parametrize("rows,dirs", [(1, 1), (85, 1), (3, 2), (42, 2)])
def test_places(place, rows, dirs):
    seen = set()
    for block in range(3 * rows * dirs):
        chain, d, row, layer = place(block, rows, dirs, block // (rows * dirs))
        assert 0 <= row < rows and 0 <= d < dirs and chain == d * rows + row and layer % dirs == d
        seen.add((layer, row))
    assert len(seen) == 3 * rows * dirs and {l for l, _ in seen} == set(range(3 * dirs))

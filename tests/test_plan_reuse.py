"""Sizes of packed layers asked for again, by other threads and beyond the number of plans
a thread keeps: always those of a first call."""

import threading

import pytest

import paper_2111_11581_amd as B


def _layers():
    out = []
    for i in range(60):
        reg = (B.ROW, B.COL, B.PUNCHED)[i % 3]
        cin, cout = 16 + 4 * (i % 7), 32 + 16 * (i % 5)
        sch = dict(rows=cout, cols=cin * 9, bh=16, bw=(16, 32)[i % 2], regularity=reg, rate=2 + i % 3, khw=9)
        conv = B.ConvShape(1, cin, 14 + i % 4, 14, 3, 3, 1 + i % 2, 1 + i % 2, 1, 1)
        out += [(sch, conv, B.BF16), (sch, conv, B.F32), (sch, None, B.BF16)]
    return out


def _sizes(layer):
    sch, conv, dt = layer
    return B.bsp_packed_sizes(B.Scheme(*sch.values()), conv, dt)


def test_repeated_plans_are_those_of_a_first_call():
    try:
        B.lib()
    except ImportError as e:
        pytest.skip(str(e))
    layers = _layers()
    first = {}

    def fresh(i):   # a thread of its own keeps no plan
        first[i] = _sizes(layers[i])

    for i in range(0, len(layers), 7):
        t = threading.Thread(target=fresh, args=(i,))
        t.start()
        t.join()
    bad = []

    def walk(order):
        for _ in range(2):
            for i in order:
                got = _sizes(layers[i])
                if i in first and got != first[i]:
                    bad.append((i, got, first[i]))

    ts = [threading.Thread(target=walk, args=(o,)) for o in (range(len(layers)), range(len(layers) - 1, -1, -1))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad, bad[:3]
    # per-block counts are the caller's array: another content, another plan
    sch = B.Scheme(32, 144, 16, 16, B.COL, 2, 1)
    conv = B.ConvShape(1, 16, 14, 14, 3, 3, 1, 1, 1, 1)
    uniform = B.bsp_packed_sizes(sch, conv, B.BF16)
    sch.set_counts([[2] * 9, [3] * 9])
    few = B.bsp_packed_sizes(sch, conv, B.BF16)
    sch.set_counts([[8] * 9, [8] * 9])
    assert few != uniform and B.bsp_packed_sizes(sch, conv, B.BF16)[1] == uniform[1] == 144

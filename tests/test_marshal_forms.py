"""The flat marshalling of a batch against the graph-by-graph one, over the
forms that a graph's rows and labels may take."""
import ctypes

import numpy as np
import pytest

import mcs_instances as mi


def _seen(graphs):
    """What the library reads of an mcs_graph array."""
    out = []
    for g in graphs:
        rw = 1 if g.n <= 64 else (g.n + 63) // 64
        words = [g.adj[k] for k in range(max(g.n, 0) * rw)] if 0 <= g.n <= 254 else None
        out.append((g.n, g.directed, words, [g.label[k] for k in range(g.n)] if g.label else None))
    return out


def _graph(n, rows=None, label=None, directed=False):
    g = {"n": n, "directed": directed, "rows": [0] * n if rows is None else rows}
    return {**g, "label": label}


FORMS = [
    _graph(0), _graph(1), _graph(64, [0] * 63 + [1 << 63]), _graph(65, [1 << 64] + [0] * 64),
    _graph(128), _graph(129), mi.er_graph(254, 0.1, 1, True, True), mi.er_graph(192, 0.1, 2),
    _graph(3, [2]), _graph(70, [5]), _graph(2, [2, 1, 7, 9]),           # rows short and over
    _graph(3, (2, 1, 0)), _graph(3, np.array([2, 1, 0])), _graph(3, np.array([2, 1, 0], np.uint64)),
    _graph(2, [1 << 64, -1]), _graph(66, [-1] + [1 << 200] * 65), _graph(2, [2.0, 1.9]),
    _graph(2, [True, np.bool_(True)]), _graph(2, b"\x02\x01"), _graph("3", [2, 1, 0]),
    _graph(0, label=[]), _graph(3, label=(1, 2, -3)), _graph(3, label=np.array([7, 8, 9])),
    _graph(3, label=[1.7, True, np.int8(3)]), _graph(2, label=[5, 6, 7]), _graph(255), _graph(-2, []),
    {"n": 2, "rows": [2, 1]}, _graph(2, [2, 1], directed=1), _graph(2, [2, 1], directed="yes"),
]


@pytest.mark.parametrize("alone", [True, False])
def test_flat_marshalling_is_the_general_one(alone):
    from paper_1908_06418_amd import _Marshal
    pairs = [(a, b) for a, b in zip(FORMS, FORMS[1:] + FORMS[:1])]
    for batch in ([[p] for p in pairs] if alone else [pairs, pairs[:14], [q for q in pairs if q[0]["n"] in (0, 1, 3)]]):
        m = _Marshal(batch)
        m._keep = getattr(m, "_keep", [])
        want = [(m._graph(g), m._graph(h)) for g, h in batch]
        assert _seen(m.G[:len(batch)]) == _seen([g for g, _ in want])
        assert _seen(m.H[:len(batch)]) == _seen([h for _, h in want])
        assert m.sizes == [max(1, min(g.n, h.n)) for g, h in want]


@pytest.mark.parametrize("bad", [_graph(2, ["x", 1]), _graph(2, None, [2 ** 31, 0]),
                                 _graph(2, None, ["a", 0]), _graph("n", []),
                                 {"rows": [], "label": None}, {"n": 1, "label": None}])
def test_what_was_refused_is_refused(bad):
    from paper_1908_06418_amd import _Marshal
    ref = _Marshal([])
    ref._keep = []
    with pytest.raises(Exception) as a:
        ref._graph(bad)
    with pytest.raises(Exception) as b:
        _Marshal([(mi.er_graph(5, 0.5, 1), bad)])
    assert a.type is b.type


def test_result_room_is_one_buffer_per_side():
    from paper_1908_06418_amd import _Results
    r = _Results([3, 1, 2])
    base = ctypes.addressof(r.map_h)
    assert [ctypes.addressof(r.res[i].map_h.contents) - base for i in range(3)] == [0, 12, 16]
    for i, (size, first) in enumerate(((3, 0), (0, 3), (1, 4))):
        r.res[i].size, r.res[i].optimal, r.res[i].nodes = size, i % 2, 10 ** 12 + i
        r.res[i].t_best_s, r.res[i].t_proof_s = 0.5, 1.5
        for j in range(size):
            r.res[i].map_g[j], r.res[i].map_h[j] = first + j, 100 + first + j
    got = r.results()
    assert [x.mapping for x in got] == [[(0, 100), (1, 101), (2, 102)], [], [(4, 104)]]
    assert [(x.size, x.optimal, x.nodes) for x in got] == \
        [(3, False, 10 ** 12), (0, True, 10 ** 12 + 1), (1, False, 10 ** 12 + 2)]
    assert all((x.t_best_s, x.t_proof_s) == (0.5, 1.5) for x in got)

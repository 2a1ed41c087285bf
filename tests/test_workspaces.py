"""CPU tests of the workspace queries: a workspace sized for the largest call
a program makes serves its smaller ones, so no query falls as a size grows."""
import ctypes
import itertools

import pytest

import paper_2409_08975_amd as tcb

# around the sizes where a layout changes: tiles, window searches, table sizes
EDGES = sorted({max(0, e + d)
                for e in [0, 2048, 4096, 131072, 5 << 16, 6 << 16, 7 << 16, 8 << 16, 9 << 16, 12 << 16, 1 << 20,
                          2**21 * 4 // 5, 2**22 * 4 // 5, 10**7, 10**8, 2**27 * 4 // 5, 2**28 * 4 // 5, 3 * 10**8,
                          2**31 - 2000]
                for d in (-1025, -513, -1, 0, 1, 2, 255, 513, 767, 1025)})
SAMPLES = [1, 1000, 65536, 786431, 786432, 786433, 10**6, 2**22 + 1, 2**23 + 1, 2**24, 2**25 - 1, 2**25, 2**25 + 1,
           10**8]


def _query(name, *args):
    b = ctypes.c_size_t(0)
    assert getattr(tcb.lib(), name)(*args, ctypes.byref(b)) == 0, (name, args)
    return b.value


def _never_falls(values, at):
    top = 0
    for v, a in zip(values, at):
        assert v >= top, a
        top = v


@pytest.mark.parametrize("n", [1, 300, 10**6])
def test_graph_workspace_by_edges(n):
    _never_falls([_query("tc_graph_workspace_bytes", n, m) for m in EDGES], EDGES)


@pytest.mark.parametrize("m", [1, 10**6, 1700000, 3 * 10**8])
def test_graph_workspace_by_vertices(m):
    at = [1, 2, 100, 460, 461, 1000, 10**6, 2**31 - 1]
    _never_falls([_query("tc_graph_workspace_bytes", n, m) for n in at], at)


def test_weights_workspace():
    for nd in range(1, 9):
        _never_falls([_query("tc_weights_batch_workspace_bytes", m, nd) for m in EDGES], EDGES)
    for m in EDGES:
        _never_falls([_query("tc_weights_workspace_bytes", m)] +
                     [_query("tc_weights_batch_workspace_bytes", m, nd) for nd in range(1, 9)], range(9))


@pytest.mark.parametrize("nm", [1, 6, 16])
def test_sampler_workspace(nm):
    for nd in range(1, 9):
        _never_falls([_query("tc_batch_workspace_bytes", k, nd, nm) for k in SAMPLES], SAMPLES)
    for k in SAMPLES:
        _never_falls([_query("tc_sample_workspace_bytes", k, nm)] +
                     [_query("tc_batch_workspace_bytes", k, nd, nm) for nd in range(1, 9)], range(9))


def test_other_workspaces():
    for name in ("tc_features_workspace_bytes", "tc_proposal_workspace_bytes", "tc_proposal_window_workspace_bytes"):
        _never_falls([_query(name, m) for m in EDGES], EDGES)
    for k, nd in itertools.product(SAMPLES, (1, 2, 8)):
        _never_falls([_query("tc_batch_workspace_bytes", k, nd, nm) for nm in range(1, 17)], range(1, 17))

"""GPU tests of calls on either side of a rule that chooses how they run: the
same results whichever way they go."""
import numpy as np
import pytest

import synthgraph as sg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tcb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2409_08975_amd as tcb
    tcb.lib()
    return tcb


@pytest.fixture(scope="module")
def torch_mod():
    import torch
    return torch


def _same(torch, a, b, names=("cnt", "hits", "estimate", "status", "xmax", "e1", "e2", "e3", "X", "P")):
    for name in names:
        u, v = getattr(a, name), getattr(b, name)
        assert (u is None) == (v is None)
        assert u is None or torch.equal(u.view(torch.uint8), v.view(torch.uint8)), name


@pytest.mark.parametrize("k", [40, 700, 3000])
@pytest.mark.parametrize("dplus", [0, 2**33])
def test_long_list_queue_by_blocks(tcb, torch_mod, k, dplus):
    """Queues of items with lists past 1,024 entries: one item a claim, and
    with 16 blocks tickets of sixteen, four and one."""
    rng = np.random.default_rng(3)
    src = [0] * 8 + [1] + [2] * 8 + [0] * 700 + [1] * 1100
    dst = [1] * 8 + [2] + [3] * 8 + [3] * 1800
    t = list(range(1, 9)) + [10] + list(range(11, 19)) + (100 + rng.integers(0, 4000, size=1800)).tolist()
    ut = torch_mod.from_numpy
    G = tcb.tc_build_graph(4, ut(np.array(src, np.int32)).cuda(), ut(np.array(dst, np.int32)).cuda(),
                           ut(np.array(t, np.int64)).cuda(), check=True)
    W = tcb.tc_path_weights(G, 5000 + dplus)
    spine, lists = [(0, 1), (1, 2), (2, 3)], [(0, 3), (1, 3), (0, 3)]
    motifs = [spine + lists, spine + lists[1:], spine + lists[:-1]]
    a = tcb.tc_sample_estimate(G, W, motifs, k, 5, per_sample=True)
    b = tcb.tc_batch_estimate(G, [W], motifs, k, 5, per_sample=True, tuning=tcb.make_tuning(wide_blocks=16))[0]
    _same(torch_mod, a, b)
    assert int(a.status) == 0 and int(a.hits[0]) > 0


@pytest.mark.parametrize("k", [786431, 786432, 2 * 786432 + 5])
def test_sample_order_by_outputs(tcb, torch_mod, k):
    """The same sums and per-sample outputs whichever of them are asked for:
    none or one array (long chunks in rank order), or several (not), and in
    chunks of 2^16."""
    torch, g = torch_mod, sg.gen_tiny()
    ut = torch.from_numpy
    G = tcb.tc_build_graph(g.n, ut(g.src).cuda(), ut(g.dst).cuda(), ut(g.t).cuda())
    Ws = tcb.tc_path_weights_batch(G, [3600, 40000])
    h = torch.randint(1, 9, (g.m,), dtype=torch.int32, device="cuda")
    sets = Ws + [tcb.tc_proposal_weights(G, Ws[1], h)]
    for names in (["M4-0"], ["S5-paw", "M4-1"]):
        motifs = [sg.MOTIFS[x] for x in names]
        want = tcb.tc_batch_estimate(G, sets, motifs, k, 11, per_sample=True, tuning=tcb.make_tuning(chunk_log2=16))
        for keep in ((), ("P",), ("X",), ("e1", "e2", "e3"), ("P", "X"), ("e1", "e2", "e3", "X", "P")):
            outs = [tcb.new_result(len(motifs), k, "cuda", per_sample=True) for _ in sets]
            for o in outs:
                for x in ("e1", "e2", "e3", "X", "P"):
                    if x not in keep:
                        setattr(o, x, None)
            for a, b in zip(tcb.tc_batch_estimate(G, sets, motifs, k, 11, outs=outs), want):
                _same(torch, a, b, ("cnt", "hits", "estimate", "status", "xmax") + keep)


@pytest.mark.parametrize("m", [5 << 16, (6 << 16) + 1, (7 << 16) + 1, (1 << 19) + 1, 9 << 16, (9 << 16) + 1])
@pytest.mark.parametrize("cls", [(1, 0, 2, 1), (0, 0, 1, 3), (2, 1, 0, 0)])
def test_windows_by_class_and_count(tcb, torch_mod, m, cls):
    """One to three deltas of a class give the same words whether the edges
    are searched one by one or the merge passes run: each set of a call of
    three equals its own call, and the columns equal ranks of composite keys."""
    from test_gpu_kernels import test_direct_windows_match_general_definition as against_ranks
    torch = torch_mod
    against_ranks(tcb, torch, m, cls)
    gen = torch.Generator(device="cuda").manual_seed(m)
    src, dst = (torch.randint(0, 5000, (m,), device="cuda", generator=gen).int() for _ in "ab")
    t = torch.randint(0, 10**6, (m,), device="cuda", generator=gen)
    G = tcb.tc_build_graph(5000, src, dst, t, check=True)
    deltas = [4000, 7, 90000]
    assert tcb.tc_path_weights_batch(G, deltas * 2, cls=cls)[5].total() == tcb.tc_path_weights(G, 90000, cls=cls).total()
    for d, w in zip(deltas, tcb.tc_path_weights_batch(G, deltas, cls=cls)):
        one = tcb.tc_path_weights(G, d, cls=cls)
        for name, x in w.arrays().items():
            assert torch.equal(x, one.arrays()[name]), name
        assert torch.equal(w.view("prec", torch.int64, 4 * m), one.view("prec", torch.int64, 4 * m))


@pytest.mark.parametrize("n,m", [(1, 1700001), (2, 1700001), (460, 1700001), (461, 1700001), (612, 3000001)])
def test_run_table_by_vertices(tcb, torch_mod, n, m):
    """Graphs of few vertices, whose runs are inserted one by one, and the
    first that are grouped: every run is found and no other key is there."""
    from test_gpu_kernels import test_pair_table_finds_every_run as finds_every_run
    finds_every_run(tcb, torch_mod, n, m)

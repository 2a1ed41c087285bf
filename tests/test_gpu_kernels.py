"""GPU tests of single kernel branches at the sizes where they change: tile
remainders, the first size on either side of a dispatch rule, and inputs
that only one branch sees."""
import math

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


def _philox(seed, stream, i):
    c, k = [i & 0xFFFFFFFF, i >> 32, 0, stream], [seed & 0xFFFFFFFF, seed >> 32]
    for _ in range(10):
        p0, p1 = 0xD2511F53 * c[0], 0xCD9E8D57 * c[2]
        c = [(p1 >> 32) ^ c[1] ^ k[0], p1 & 0xFFFFFFFF, (p0 >> 32) ^ c[3] ^ k[1], p0 & 0xFFFFFFFF]
        k = [(k[0] + 0x9E3779B9) & 0xFFFFFFFF, (k[1] + 0xBB67AE85) & 0xFFFFFFFF]
    return c


@pytest.mark.parametrize("n,batch", [(1, 32), (33, 32), (70001, 65536), (1500007, 1 << 20)])
def test_train_equals_single_steps(tcb, torch_mod, n, batch):
    """An epoch equals, bit for bit, one gradient and one Adam step per batch
    over the labels in the epoch's Philox order formed here in Python
    integers: one tile, a ragged tile, more tiles than wavefronts, and label
    indices whose product with the multiplier passes 2^32."""
    torch = torch_mod
    seed, lr = 0x123456789, 1e-3
    rng = np.random.default_rng(n)
    F = torch.from_numpy(sg.random_bf16_bits(n, (5000, 8)).view(np.int16)).cuda()
    P = sg.random_params(n)
    rows = rng.integers(0, 5000, size=n).astype(np.int32)
    X = sg.random_counts(n, n).view(np.int64)
    p1, o1 = torch.from_numpy(P.copy()).cuda(), torch.zeros(2 * tcb.MLP_PARAMS, device="cuda")
    p2, o2 = p1.clone(), o1.clone()
    rd, Xd = torch.from_numpy(rows).cuda(), torch.from_numpy(X).cuda()
    tcb.tc_mlp_train(p1, o1, F, rd, Xd, batch, 1, lr, seed)
    x0, x1, x2, x3 = _philox(seed, 0x4D4C5000, 0)
    mul = 1 + ((x1 << 32) | x0) % (n - 1) if n > 1 else 1
    while math.gcd(mul, n) != 1:
        mul = mul + 1 if mul + 1 < n else 1
    add = ((x3 << 32) | x2) % n
    order = (mul * torch.arange(n, device="cuda") + add) % n
    for step, start in enumerate(range(0, n, batch), 1):
        i = order[start:start + batch]
        g, _ = tcb.tc_mlp_grad(p2, F, rd[i].contiguous(), Xd[i].contiguous())
        tcb.tc_mlp_adam(p2, o2, g, step, lr)
    assert torch.equal(p1, p2) and torch.equal(o1, o2)


@pytest.mark.parametrize("n", [1, 31, 33, 2048 * 32 * 4 + 5])
def test_mlp_forward_tiles_and_special_values(tcb, torch_mod, n):
    """Network scores over one ragged tile up to more tiles than the launch
    has wavefronts with all their prefetched tiles, with infinite and NaN
    features among the rows: a ReLU takes NaN to 0, so the scores agree with
    a float64 network that does the same, NaN for NaN."""
    torch = torch_mod
    bits = sg.random_bf16_bits(n, (n, 8))
    special = [0x7F80, 0xFF80, 0x7FC0, 0x0000, 0x8000]
    for k, b in enumerate(special):
        if 3 * k < n:
            bits[3 * k, k] = b
    P = sg.random_params(7)
    g = tcb.tc_mlp_forward(torch.from_numpy(P).cuda(),
                           torch.from_numpy(bits.view(np.int16)).cuda()).cpu().numpy()

    def bf(x):  # bfloat16 rounding of float64 values (via float32)
        return torch.from_numpy(x).float().to(torch.bfloat16).double().numpy()

    with np.errstate(all="ignore"):
        f = (bits.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
        w1, b1, w2 = bf(P[:512].astype(np.float64)).reshape(64, 8), P[512:576], bf(P[576:4672].astype(np.float64))
        b2, w3, b3 = P[4672:4736], bf(P[4736:4800].astype(np.float64)), P[4800]
        relu = lambda z: bf(np.where(z > 0, z, 0.0))  # noqa: E731
        h1 = relu((f[:, None, :] * w1).sum(2) + b1) if n < 100 else relu(f @ w1.T + b1)
        h2 = relu(h1 @ w2.reshape(64, 64).T + b2)
        want = 1.0 / (1.0 + np.exp(-(h2 @ w3 + b3)))
    assert np.array_equal(np.isnan(g), np.isnan(want))
    ok = ~np.isnan(want)
    # a bfloat16 ulp of one hidden activation is 2^-8 of it
    assert np.max(np.abs(g[ok] - want[ok])) <= 4e-3


@pytest.mark.parametrize("m,delta", [(1, 5), (7, 0), (2048, 40), (2049, 3), (6000, 10**9)])
def test_features_long_runs_and_tiles(tcb, torch_mod, m, delta):
    """Edge features on five vertices (pair runs of hundreds of entries and
    equal times, both directions of every pair) at the scan's tile edges:
    float32 evaluation and one bfloat16 rounding, so within 2^-8."""
    from test_gpu_parity import build_both
    G, og = build_both(tcb, torch_mod, sg.gen_micro(m, n=5, m=m, t_span=200))
    F = tcb.tc_edge_features(G, tcb.tc_path_weights(G, delta)).cpu().numpy().view(np.uint16)
    got = (F.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    want = og.features(og.weights(delta))
    assert np.all(np.abs(got - want) <= 2.0**-8 * np.abs(want) + 1e-6)


@pytest.mark.parametrize("m", [2047, 2049, 131073, 2999999, 3000001])
@pytest.mark.parametrize("n,t_bits", [(1, 40), (3, 33), (1 << 11, 22), (1 << 12, 36), (50000, 46), (50000, 55),
                                      (1 << 26, 60)])
def test_build_orders(tcb, torch_mod, m, n, t_bits):
    """The three orders against torch sorts of the same keys: tile
    remainders of both tile sizes, one and several digits per sort, and time
    ranges below 32 bits, packed beside the vertex word and too wide for it."""
    torch = torch_mod
    gen = torch.Generator(device="cuda").manual_seed(m + n)
    src = torch.randint(0, n, (m,), device="cuda", generator=gen).int()
    dst = (torch.randint(0, n, (m,), device="cuda", generator=gen).int() // 2)
    # repeated times, around zero, both ends of the range present
    t = torch.randint(0, 1 << t_bits, (m,), device="cuda", generator=gen)
    t[: m // 2] = t[m - m // 2:]
    t[0], t[-1] = 0, (1 << t_bits) - 1
    t -= 1 << (t_bits - 1)
    g = tcb.tc_build_graph(n, src, dst, t, check=True).arrays()
    by_t = torch.sort(t, stable=True)[1]

    def order(*keys):  # stable, most significant key last
        o = by_t
        for k in keys:
            o = o[torch.sort(k[o], stable=True)[1]]
        return o

    for name, o, key, other in (("out", order(src), src, dst), ("in", order(dst), dst, src)):
        far = "dst" if name == "out" else "src"
        near = "src" if name == "out" else "dst"
        assert torch.equal(g[name + "_eid"].long(), o)
        assert torch.equal(g[f"{name}_{near}"], key[o]) and torch.equal(g[f"{name}_{far}"], other[o])
        assert torch.equal(g[name + "_t"], t[o])
        off = torch.searchsorted(key[o].long(), torch.arange(n + 1, device="cuda"))
        assert torch.equal(g[name + "_off"].long(), off)
    o = order(dst, src)
    assert torch.equal(g["pair_eid"].long(), o) and torch.equal(g["pair_dst"], dst[o])
    assert torch.equal(g["pair_t"], t[o])


@pytest.mark.parametrize("n,m", [(40, 900001), (5000, 1700000), (1 << 20, 13500000), (1 << 20, 14000003),
                                 (1 << 22, 28000001)])
def test_pair_table_finds_every_run(tcb, torch_mod, n, m):
    """Every run of the pair index is found in the run table by linear
    probing from its home slot, and no other key is in it: few and many runs
    per segment, segments of both sizes, loads up to 0.8 (runs that do not
    fit their segment)."""
    torch = torch_mod
    gen = torch.Generator(device="cuda").manual_seed(n)
    src = torch.randint(0, n, (m,), device="cuda", generator=gen).int()
    dst = torch.randint(0, n, (m,), device="cuda", generator=gen).int()
    t = torch.randint(0, 1000, (m,), device="cuda", generator=gen)
    G = tcb.tc_build_graph(n, src, dst, t, check=True)
    lg = G.c.pair_hash_log2
    cap = 1 << lg
    tab = G.view("pair_hash", torch.int64, 2 * cap).view(cap, 2)
    run = tab[:, 1]
    start, end = run & 0xFFFFFFFF, (run >> 32) & 0xFFFFFFFF
    a = G.arrays()
    ps = src[a["pair_eid"].long()].long()
    key = (ps << 32) | a["pair_dst"].long()
    want_start = torch.nonzero(torch.cat([torch.ones(1, dtype=torch.bool, device="cuda"),
                                          key[1:] != key[:-1]])).flatten()
    want_end = torch.cat([want_start[1:], torch.tensor([m], device="cuda")])
    used = torch.nonzero(tab[:, 0] != -1).flatten()
    assert used.numel() == want_start.numel()
    o = torch.sort(start[used])[1]
    used = used[o]
    assert torch.equal(start[used], want_start) and torch.equal(end[used], want_end)
    assert torch.equal(tab[used, 0], key[want_start])
    # a search from the home slot reaches the run: no empty slot on the way
    # (0x9E3779B97F4A7C15 as a signed word; the product wraps)
    home = (key[want_start] * -7046029254386353131) >> (64 - lg)
    home = home & (cap - 1)
    empty = torch.cumsum(torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"),
                                    (tab[:, 0] == -1).long()]), 0)
    on_way = empty[used] - empty[home] + torch.where(used < home, empty[-1], 0)
    assert int(on_way.abs().max()) == 0


@pytest.mark.parametrize("m", [1, 255, 2049, 786432, 786433])
@pytest.mark.parametrize("cls", [(1, 0, 2, 1), (2, 1, 1, 0), (0, 0, 1, 3), (2, 2, 0, 0), (1, 2, 2, 3)])
def test_direct_windows_match_general_definition(tcb, torch_mod, m, cls):
    """Windows, scan and total on both sides of the size where the per-edge
    searches give way to the merge passes, for closed, open, before, after
    and absent sides and two deltas, against ranks of composite keys."""
    torch = torch_mod
    n = 300
    gen = torch.Generator(device="cuda").manual_seed(m)
    src = torch.randint(0, n, (m,), device="cuda", generator=gen).int()
    dst = torch.randint(0, n, (m,), device="cuda", generator=gen).int()
    t = torch.randint(0, max(2, m // 3), (m,), device="cuda", generator=gen)
    G = tcb.tc_build_graph(n, src, dst, t, check=True)
    a = {k: v.long() for k, v in G.arrays().items()}
    T = 4 * m + 8
    keys = {1: a["in_dst"] * T + a["in_t"] + m, 2: a["out_src"] * T + a["out_t"] + m}
    deltas = [m // 7, 3]
    for d, W in zip(deltas, tcb.tc_path_weights_batch(G, deltas, cls=cls)):
        w = W.arrays()
        prod = torch.ones(m, dtype=torch.int64, device="cuda")
        for mode, after, v, lo, ln in ((cls[0], cls[1], a["out_src"], w["lo_in"], w["a"]),
                                       (cls[2], cls[3], a["out_dst"], w["lo_out"], w["b"])):
            if mode == 0:
                assert int(lo.abs().max()) == 0 and bool((ln == 1).all())
                continue
            at = v * T + a["out_t"] + m
            if after & 1:
                first = torch.searchsorted(keys[mode], at, right=bool(after & 2))
                end = torch.searchsorted(keys[mode], at + d, right=True)
            else:
                first = torch.searchsorted(keys[mode], at - d)
                end = torch.searchsorted(keys[mode], at, right=not after & 2)
            # an open window of delta 0 is empty: its first position is past the tie
            assert torch.equal(lo.long(), first) and torch.equal(ln.long(), end - first)
            prod *= ln.long()
        S = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), torch.cumsum(prod, 0)])
        assert torch.equal(w["S"], S) and W.status() == 0


@pytest.mark.parametrize("n_ad,n_bd,tail,span", [
    (511, 2000, 3, 4000),      # a bridged middle list between the longest LDS lists
    (512, 2000, 3, 4000),      # one entry past them
    (1024, 511, 4, 700),       # the first list is the longer one; ties
    (1025, 64, 2, 3000),       # two lists: the first in the second's place
    (3, 1100, 5, 50),          # many equal times, short neighbours
    (129, 1025, 7, 10**6),     # seven lists: totals past 2^32, products past 2^64
    (257, 2049, 2, 900),       # the last list is the longer one
    (64, 1024, 5, 2000), (65, 128, 6, 300), (255, 256, 4, 5000),  # the shorter passes
])
@pytest.mark.parametrize("dplus", [0, 2**33])
def test_chain_counts_by_list_shape(tcb, torch_mod, n_ad, n_bd, tail, span, dplus):
    """Chain counts where the list lengths choose how a level runs: the
    planted spine A->B->C->D, then `tail` lists alternating A->D and B->D.
    Every sum and every per-sample count equals the oracle's, for windows with
    32-bit keys and (dplus) with 64-bit ones."""
    from test_gpu_parity import build_both, check_sample
    rng = np.random.default_rng(n_ad * 7 + n_bd)
    src = [0] * 8 + [1] + [2] * 8 + [0] * n_ad + [1] * n_bd
    dst = [1] * 8 + [2] + [3] * 8 + [3] * (n_ad + n_bd)
    t = list(range(1, 9)) + [10] + list(range(11, 19)) + (100 + rng.integers(0, span, size=n_ad + n_bd)).tolist()
    g = sg.TemporalGraph(4, np.array(src, np.int32), np.array(dst, np.int32), np.array(t, np.int64))
    G, og = build_both(tcb, torch_mod, g)
    delta = 100 + span + dplus
    Wt, ow = tcb.tc_path_weights(G, delta), og.weights(delta)
    lists = [(0, 3) if r % 2 == 0 else (1, 3) for r in range(tail)]
    spine = [(0, 1), (1, 2), (2, 3)]
    R, E = check_sample(tcb, G, Wt, og, ow, [spine + lists, spine + lists[1:], spine + lists[:-1]], 300, seed=4,
                        per_sample=True)
    assert E.status == 0 and int(E.hits[0]) > 0


@pytest.mark.parametrize("k", [786431, 786432, 786433, 1 << 20, 3145727, 3145728 + 77])
@pytest.mark.parametrize("i0", [0, 2**32 - 5])
def test_rank_ordered_samples_equal_small_chunks(tcb, torch_mod, k, i0):
    """Chunks long enough to be put in rank order give every per-sample output
    and every sum of 2^16-sample chunks, which are not; the sums of squares
    agree to the rounding of k additions in another order."""
    torch = torch_mod
    g = sg.gen_tiny()
    ut = torch.from_numpy
    G = tcb.tc_build_graph(g.n, ut(g.src).cuda(), ut(g.dst).cuda(), ut(g.t).cuda())
    Ws = tcb.tc_path_weights_batch(G, [3600, 40000])
    motifs = [sg.MOTIFS["M4-0"], sg.MOTIFS["S5-paw"], sg.MOTIFS["M4-1"]]
    a = tcb.tc_batch_estimate(G, Ws, motifs, k, 7, 2, i0, per_sample=True)
    b = tcb.tc_batch_estimate(G, Ws, motifs, k, 7, 2, i0, per_sample=True,
                              tuning=tcb.make_tuning(chunk_log2=16))
    for x, y in zip(a, b):
        for name in ("cnt", "hits", "estimate", "status", "e1", "e2", "e3", "X"):
            u, v = getattr(x, name), getattr(y, name)
            assert torch.equal(u.view(torch.uint8), v.view(torch.uint8)), name
    h = torch.randint(1, 9, (g.m,), dtype=torch.int32, device="cuda")
    q = tcb.tc_proposal_weights(G, Ws[1], h)
    one = tcb.tc_sample_estimate(G, q, motifs, k, 7, 2, i0, moments=True)
    parts = [tcb.tc_sample_estimate(G, q, motifs, min(1 << 19, k - c), 7, 2, i0 + c, moments=True)
             for c in range(0, k, 1 << 19)]
    assert one.counts() == [sum(c) for c in zip(*(p.counts() for p in parts))]
    m2 = sum(p.m2.double() for p in parts)
    assert torch.all((one.m2 - m2).abs() <= 2 * k * 2.0**-53 * m2)

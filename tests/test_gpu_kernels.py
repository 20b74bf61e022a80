"""Edges of single kernels against the oracle: tile remainders, the smallest
and largest sizes of a dispatch rule's ranges, ties and value ranges."""
import numpy as np
import pytest

gpu = pytest.mark.gpu


def _log(msg):
    print(f"[gpu-kernels] {msg}", flush=True)


@gpu
@pytest.mark.parametrize("E,P", [(1, 1), (5, 5), (64, 64), (63, 9), (65, 13), (128, 64), (255, 15), (512, 64),
                                 (513, 1), (520, 65), (2048, 32)])
@pytest.mark.parametrize("values", ["zeros", "ties", "wide", "past_key"])
def test_place_edges(E, P, values):
    """LPT at full ranks, one expert per rank, odd expert counts and equal
    loads; loads whose layer sum passes the sorted key's range (2^50 and
    more) and more than 64 ranks take the general steps."""
    import oracle as O
    import paper_2608_12146_amd as rp
    _log(f"place E={E} P={P} {values}")
    rng = np.random.default_rng([11, E, P])
    L = 3
    hi = {"zeros": 1, "ties": 4, "wide": 1 << 30, "past_key": 1 << 52}[values]
    agg = rng.integers(0, hi, size=(L, E), dtype=np.int64)
    if values == "past_key":
        agg[:, 0] = 1 << 52
    prob = rp.Problem(1, L, E, 1, P, 1, 1, [0], 1 << 20, [4096], [1])
    slot, load, _ = rp.place_experts(prob, agg)
    o_slot, o_load = O.place(agg, P)
    assert np.array_equal(slot.cpu().numpy(), o_slot)
    assert np.array_equal(load.cpu().numpy(), o_load)


@gpu
@pytest.mark.parametrize("E,P", [(8190, 30), (8192, 64), (13312, 64), (13504, 32)])
@pytest.mark.parametrize("low", [0, 50, 52])
def test_place_many_heavy_experts(E, P, low):
    """Loads of 2^low and up to 2^52 (2^30 with low = 0) for as many experts
    as the LDS holds: capped at 2^50 each, 8192 of them sum to 2^63."""
    import oracle as O
    import paper_2608_12146_amd as rp
    _log(f"place E={E} P={P} loads from 2^{low}")
    rng = np.random.default_rng([22, E, low])
    agg = rng.integers(1 << low, (1 << 52 if low else 1 << 30) + 1, size=(2, E), dtype=np.int64)
    agg[1] = 1 << low
    prob = rp.Problem(1, 2, E, 1, P, 1, 1, [0], 1 << 20, [4096], [1])
    slot, load, _ = rp.place_experts(prob, agg)
    o_slot, o_load = O.place(agg, P)
    assert np.array_equal(slot.cpu().numpy(), o_slot)
    assert np.array_equal(load.cpu().numpy(), o_load)


@gpu
@pytest.mark.parametrize("P", [1, 2, 4, 6, 8, 16, 32, 64, 128])
@pytest.mark.parametrize("L,G,D,R,N", [(1, 1, 1, 1, 1), (1, 2, 3, 5, 40), (3, 1, 4, 17, 257), (5, 3, 7, 9, 130),
                                       (17, 2, 8, 33, 1025), (9, 1, 8, 400, 3300)])
@pytest.mark.parametrize("big", [False, True])
def test_score_edges(P, L, G, D, R, N, big):
    """Scores, costs and diagnostics with one layer per piece and many, row
    groups in a wave, ragged counts and single members, one row-shard to more
    than the list path's LDS holds; big: layer totals of 2^32 and more.
    Layouts: feasible ones, one with an empty cell, one with ids out of range."""
    import oracle as O
    import paper_2608_12146_amd as rp
    _log(f"score P={P} L={L} G={G} D={D} R={R} N={N} big={big}")
    rng = np.random.default_rng([12, P, L, N])
    t = rng.integers(1, 50, size=N).astype(np.int32)
    # (2^53 bounds the scores: few large entries, no fractional bits)
    q = rng.integers(0, 60, size=(N, L, P)).astype(np.int32)
    if big:
        q[:, 0, 0] += (1 << 32) // (2 * N) if N > 2 else 1 << 30
    cap = int(t.sum()) + 1
    g = (np.arange(D) * G // D).astype(np.int32)
    kw = dict(n_samples=N, n_layers=L, n_experts=P, top_k=1, n_ranks=P, n_dp=D, n_edp=G, dp_to_edp=g, capacity=cap,
              alpha_fp=np.array([3, 1]), beta_fp=np.array([0, 1]), frac_bits=0, min_rows=1)
    lays = np.stack([rng.permutation(np.arange(N) % (R * D)) for _ in range(5)]).astype(np.int32)
    lays[3] = np.minimum(lays[3], max(0, R * D - 2))
    lays[4, 0], lays[4, N // 2] = R * D, -1
    load = rng.integers(1, 1000, size=(L, P)).astype(np.int64)
    out = rp.eval_objective(rp.Problem.from_dict(kw), t, q, R, lays, rank_load=load, want_J=True, want_diag=True)
    pb = O.Problem.from_dict(kw)
    for m in range(len(lays)):
        st, s, J, dg = O.score(pb, t, q, R, lays[m], rank_load=load, want_J=True, want_diag=True)
        assert int(out["status"][m]) == st
        assert out["scores"][m].cpu().tolist() == s.tolist()
        assert out["J"][m].cpu().tolist() == J.tolist()
        if st == 0:  # sums of at most L R G doubles in another order
            np.testing.assert_allclose(out["diag"][m].cpu().numpy(), dg, rtol=1e-11, atol=0)


@gpu
@pytest.mark.parametrize("N,L,P,D,G,R,n", [(64, 64, 64, 1, 1, 64, 70000), (64, 1, 6, 1, 1, 64, 262200),
                                             ((1 << 20) + 3, 1, 4, 4, 2, 8, 66)])
def test_score_pieces(N, L, P, D, G, R, n):
    """More layouts than one launch takes: row pieces past 2^32 threads (70000
    layouts x 64 row-shards x 16 pieces), row-shards past them on the general
    kernel (6 ranks), and sample lists past 2^26 entries."""
    import torch
    import oracle as O
    import paper_2608_12146_amd as rp
    _log(f"score pieces N={N} L={L} P={P} R={R} layouts={n}")
    rng = np.random.default_rng([24, N])
    t = rng.integers(1, 50, size=N).astype(np.int32)
    q = rng.integers(0, 60, size=(N, L, P)).astype(np.int32)
    g = (np.arange(D) * G // D).astype(np.int32)
    kw = dict(n_samples=N, n_layers=L, n_experts=P, top_k=1, n_ranks=P, n_dp=D, n_edp=G, dp_to_edp=g,
              capacity=int(t.sum()), alpha_fp=np.array([3]), beta_fp=np.array([0]), frac_bits=0, min_rows=1)
    base = np.stack([rng.permutation(np.arange(N) % (R * D)) for _ in range(3)]).astype(np.int32)
    which = rng.integers(0, 3, size=n)
    lays = torch.as_tensor(base, device="cuda")[torch.as_tensor(which, device="cuda")].contiguous()
    out = rp.eval_objective(rp.Problem.from_dict(kw), t, q, R, lays, want_J=True)
    want = [O.score(O.Problem.from_dict(kw), t, q, R, x, want_J=True) for x in base]
    assert not out["status"].any()
    assert np.array_equal(out["scores"].cpu().numpy(), np.stack([w[1] for w in want])[which])
    assert np.array_equal(out["J"].cpu().numpy(), np.stack([w[2] for w in want])[which])


def _pack_case(N, D, G, cap, lengths, L=2, P=4, seed=5):
    rng = np.random.default_rng([13, N, D, seed])
    q = rng.integers(0, 1000, size=(N, L, P)).astype(np.int32)
    kw = dict(n_samples=N, n_layers=L, n_experts=P, top_k=1, n_ranks=P, n_dp=D, n_edp=G,
              dp_to_edp=(np.arange(D) * G // D).astype(np.int32), capacity=cap, alpha_fp=np.array([4096]),
              beta_fp=np.array([1]), frac_bits=2, min_rows=1)
    return np.asarray(lengths, dtype=np.int32), q, kw


def _check_pack(t, q, kw, width, trials=5, pop=9, seed=77):
    import oracle as O
    import paper_2608_12146_amd as rp
    want = O.pack_rows(O.Problem.from_dict(kw), t, q, seed, trials, width, pop)
    try:
        got = rp.pack_rows(rp.Problem.from_dict(kw), t, q, seed, trials, width, pop)
    except rp.RoutepackError as e:
        assert e.code == want["rc"]
        return None
    assert want["rc"] == 0 and got["r_star"] == want["r_star"]
    assert (got["r_lb"], got["n_distinct"], got["n_trials_ok"]) == (want["r_lb"], want["n_distinct"],
                                                                   want["n_trials_ok"])
    assert np.array_equal(got["population"].cpu().numpy(), want["population"])
    assert np.array_equal(got["scores"].cpu().numpy(), want["scores"])
    return want


@gpu
@pytest.mark.parametrize("width", [1, 2, 5, 17, 62])
@pytest.mark.parametrize("K,N", [(1, 1), (1, 9), (31, 63), (32, 65), (33, 200), (63, 64), (64, 700), (65, 1000),
                                 (512, 1500), (2048, 2500), (2050, 2300)])
def test_pack_cell_counts(K, N, width):
    """Best-fit seeds with one row of keys, full and part-filled last rows,
    the last sorted cell count and the first past it, at narrow and wide
    choices; equal lengths occur throughout (ties by members, then cell)."""
    _log(f"pack K={K} N={N} width={width}")
    rng = np.random.default_rng([14, K, N])
    t = rng.integers(1, 40, size=N)
    D = 2 if K % 2 == 0 else 1
    kw_cap = max(int(-(-t.sum() // K) * 1.08) + 2, int(t.max()))
    t, q, kw = _pack_case(N, D, 1, kw_cap, t, L=1)
    kw["min_rows"] = K // D
    _check_pack(t, q, kw, width)


@gpu
@pytest.mark.parametrize("seed", range(12))
def test_pack_tight_cells(seed):
    """Cells filled to the cap: trials that find no cell, row counts that
    FFD raises, rows of keys that fill up and are spread again."""
    _log(f"pack tight {seed}")
    rng = np.random.default_rng([15, seed])
    n_cells, per = int(rng.integers(20, 200)), int(rng.integers(2, 12))
    cap = 600
    cuts = [np.diff(np.concatenate([[0], np.sort(rng.choice(np.arange(1, cap), per - 1, replace=False)), [cap]]))
            for _ in range(n_cells)]
    t = rng.permutation(np.concatenate(cuts))
    if seed % 3 == 0:  # many short samples: one row of keys takes most placements
        t = np.concatenate([t, np.ones(500, dtype=t.dtype)])
    D = int(rng.choice([1, 2, 4]))
    t, q, kw = _pack_case(len(t), D, 1, cap, t)
    _check_pack(t, q, kw, int(rng.choice([1, 3, 4, 8])))


@gpu
@pytest.mark.parametrize("L,P,D,G,R", [(1, 4, 1, 1, 15), (2, 4, 4, 2, 4), (31, 8, 3, 1, 16), (32, 16, 5, 3, 7),
                                       (33, 16, 4, 1, 17), (64, 64, 2, 1, 9), (5, 12, 4, 2, 40), (3, 48, 8, 8, 9),
                                       (65, 4, 4, 1, 9), (24, 16, 2, 2, 140), (7, 6, 4, 2, 8), (2, 128, 2, 1, 6),
                                       (2, 4, 8, 8, 70)])
@pytest.mark.parametrize("width", [1, 4])
@pytest.mark.parametrize("ties", [False, True])
def test_pack_pairing_shapes(L, P, D, G, R, width, ties):
    """EDPAwarePair with half and whole waves of layers, batches cut short,
    W in LDS and in memory, one row-shard per lane and several, shards of
    unequal size, and the shapes beyond the batched kernels (65 layers, 560
    row-shards, 6 or 128 ranks); ties: few distinct rows, so equal increases
    and equal peaks decide by index."""
    _log(f"pairing L={L} P={P} D={D} G={G} R={R} width={width} ties={ties}")
    N = R * D * 2 + 3
    rng = np.random.default_rng([16, L, P, R])
    t = np.full(N, 10) if ties else rng.integers(1, 40, size=N)
    t, q, kw = _pack_case(N, D, G, int(-(-t.sum() // (R * D)) * 1.6) + 40, t, L=L, P=P)
    if ties:
        q[:] = q[rng.integers(0, 2, size=N)]
    kw["min_rows"] = R
    kw["dp_to_edp"] = np.sort(np.concatenate([np.arange(G), rng.integers(0, G, size=D - G)])).astype(np.int32)
    _check_pack(t, q, kw, width, trials=4)


@gpu
@pytest.mark.parametrize("L,P,D,G,R", [(1, 1, 1, 1, 1), (1, 4, 2, 1, 6), (3, 16, 4, 2, 5), (2, 6, 3, 3, 7)])
@pytest.mark.parametrize("load", [(1 << 31) - 1, 1 << 31, 1 << 33, 1 << 37])
def test_pack_large_loads(L, P, D, G, R, load):
    """Cell sums and row-shard loads on both sides of 2^31.  `load` is the
    largest layer total, which bounds a load in the first shape; in the others
    a row-shard's capacity times the largest entry per token is smaller."""
    _log(f"pack loads up to {load} L={L} P={P} D={D} G={G} R={R}")
    N = 5 * R * D + (1 if R > 1 else 0)
    rng = np.random.default_rng([23, L, P, load & 0xFFFF])
    t, q, kw = _pack_case(N, D, G, 9, np.ones(N), L=L, P=P)
    share = min(load // N, (1 << 31) - 1)
    q[:] = rng.integers(0, max(1, share // P // 2), size=q.shape)
    q[:, 0, :] = 0
    q[:, 0, 0] = share  # layer 0: all on rank 0, its total made exact on sample 0
    q[0, 0, 0] += min(load - share * N, (1 << 31) - 1 - share)
    assert q.min() >= 0 and q[:, 0].sum(dtype=np.int64) == min(load, N * ((1 << 31) - 1))
    kw.update(min_rows=R, frac_bits=0, alpha_fp=np.array([1]), beta_fp=np.array([0]))
    assert _check_pack(t, q, kw, 3) is not None


@gpu
@pytest.mark.parametrize("K,N", [(1, 5), (64, 65), (65, 130), (128, 900), (200, 200), (4096, 4300)])
@pytest.mark.parametrize("scale", [1, 1 << 22])
def test_pack_first_fit(K, N, scale):
    """FixedRowFFD over one chunk of cells, a part-filled last chunk and the
    most chunks, with a cap below and above 2^31 (x_length and x_paired
    only)."""
    _log(f"first fit K={K} N={N} scale={scale}")
    rng = np.random.default_rng([17, K, N])
    t = np.sort(rng.integers(1, 400, size=N))[::-1]
    t = rng.permutation(t)
    cap = max(int(-(-t.sum() // K) * 1.02) + 1, int(t.max())) * scale
    t, q, kw = _pack_case(N, 1, 1, cap, t * scale, L=1)
    q[:] = rng.integers(0, 9, size=q.shape)
    kw.update(min_rows=K, frac_bits=0, alpha_fp=np.array([1]), beta_fp=np.array([0]))
    _check_pack(t, q, kw, 1, trials=2)


@gpu
@pytest.mark.parametrize("P,L", [(2, 3), (4, 1), (8, 33), (16, 20), (64, 5)])
@pytest.mark.parametrize("shards", ["one", "interleaved", "runs"])
def test_anneal_start_state(P, L, shards):
    """Two levels from a population of distinct and repeated layouts whose
    shards hold adjacent slots, none adjacent, or runs of slots: every W row,
    J and pool of the start state enters the trace."""
    import oracle as O
    import paper_2608_12146_amd as rp
    _log(f"anneal start P={P} L={L} {shards}")
    D, R = 6, 7
    rng = np.random.default_rng([18, P, L])
    N = 4 * R * D + 5
    t = rng.integers(1, 60, size=N)
    G = {"one": 1, "interleaved": 2, "runs": 3}[shards]
    t, q, kw = _pack_case(N, D, G, int(-(-t.sum() // (R * D)) * 1.5) + 40, t, L=L, P=P)
    kw["min_rows"] = R
    kw["dp_to_edp"] = np.array({"one": [0] * 6, "interleaved": [0, 1] * 3, "runs": [2, 2, 0, 1, 1, 0]}[shards],
                               dtype=np.int32)
    pb, prob = O.Problem.from_dict(kw), rp.Problem.from_dict(kw)
    pk = O.pack_rows(pb, t, q, 3, 8, 4, 20)
    assert pk["rc"] == 0
    pop = pk["population"].copy()
    rows = rng.permutation(R)  # the rows in another order: further distinct layouts
    pop[5:9] = rows[pop[5:9] // D] * D + pop[5:9] % D
    temps = np.array([1e-2, 1e-3])
    o = O.anneal(pb, t, q, pk["r_star"], pop, temps, 48, 9)
    g = rp.anneal(prob, t, q, pk["r_star"], pop, temps, 48, 9)
    assert np.array_equal(g["trace"].cpu().numpy(), o["trace"])
    assert np.array_equal(g["population"].cpu().numpy(), o["population"])
    assert np.array_equal(g["best_layout"].cpu().numpy(), o["best_layout"])


@gpu
def test_anneal_many_row_shards():
    """Start rows of 32800 distinct members with 512 row-shards each, 2^24 and
    more in one call, on the general kernel (2 ranks)."""
    import oracle as O
    import paper_2608_12146_amd as rp
    pop, N = 32800, 512
    _log(f"anneal {pop} members of {N} row-shards")
    rng = np.random.default_rng([25, pop])
    t, q, kw = _pack_case(N, 1, 1, 60, rng.integers(1, 60, size=N), L=1, P=2)
    layouts = rng.permuted(np.tile(np.arange(N, dtype=np.int32), (pop, 1)), axis=1)
    temps = np.array([1e-2, 1e-3])
    o = O.anneal(O.Problem.from_dict(kw), t, q, N, layouts, temps, 4, 9)
    g = rp.anneal(rp.Problem.from_dict(kw), t, q, N, layouts, temps, 4, 9)
    assert o["rc"] == 0 and o["trace"][..., 6].sum() > 0
    for k in ("trace", "parents", "population", "best_layout"):
        assert np.array_equal(g[k].cpu().numpy(), o[k])


@gpu
@pytest.mark.parametrize("pop", [1, 3, 1023, 1025, 2050, 7372, 7373, 9557, 9558])
def test_level_end_populations(pop, monkeypatch):
    """Resampling after each level of the per-level kernel with one member, a
    ragged share per thread, and the populations at which the weights' prefix
    and the hand-over tables leave LDS."""
    import oracle as O
    import paper_2608_12146_amd as rp
    _log(f"level end pop={pop}")
    monkeypatch.setenv("ROUTEPACK_ANNEAL_KERNEL", "chain")
    rng = np.random.default_rng([21, pop])
    t = rng.integers(1, 60, size=24)
    t, q, kw = _pack_case(24, 4, 1, int(-(-t.sum() // 8) * 1.6) + 60, t, L=2, P=4)
    kw["min_rows"] = 2
    pb, prob = O.Problem.from_dict(kw), rp.Problem.from_dict(kw)
    pk = O.pack_rows(pb, t, q, 3, 8, 4, pop)
    assert pk["rc"] == 0
    temps = np.array([1e-1, 1e-2, 1e-3])
    o = O.anneal(pb, t, q, pk["r_star"], pk["population"], temps, 8, 9, t_next=1e-4)
    g = rp.anneal(prob, t, q, pk["r_star"], pk["population"], temps, 8, 9, t_next=1e-4)
    assert g["level_kernel"] == "chain"
    for k in ("parents", "trace", "population", "best_layout"):
        assert np.array_equal(g[k].cpu().numpy(), o[k])


@gpu
@pytest.mark.parametrize("kernel", ["chain_run", "chain"])
@pytest.mark.parametrize("cap,stages", [(512, 1), (500, 2)])
def test_accept_temperatures(cap, stages, kernel, monkeypatch):
    """The accept test's single-precision bracket: temperatures from which
    every uphill move is taken to those from which none is, and those at and
    past the ends of single precision, where z underflows or overflows there."""
    import oracle as O
    import paper_2608_12146_amd as rp
    _log(f"accept cap={cap} stages={stages} {kernel}")
    monkeypatch.setenv("ROUTEPACK_ANNEAL_KERNEL", kernel)
    rng = np.random.default_rng([22, cap])
    t = rng.integers(1, 60, size=160)
    t, q, kw = _pack_case(160, 4, 1, cap, t, L=5, P=8)
    kw["min_rows"] = 4
    if stages == 2:
        kw.update(alpha_fp=np.array([4096, 2048]), beta_fp=np.array([0, 1]))
    pb, prob = O.Problem.from_dict(kw), rp.Problem.from_dict(kw)
    pk = O.pack_rows(pb, t, q, 3, 8, 4, 64)
    assert pk["rc"] == 0
    temps = np.array([1e300, 4e38, 3e38, 1e20, 10.0, 1.0, 0.3, 0.1, 3e-2, 1e-2, 3e-3, 1e-3, 1e-4, 1e-6, 1e-20, 1e-37,
                      1.2e-38, 1e-39, 1e-45, 1e-300])
    o = O.anneal(pb, t, q, pk["r_star"], pk["population"], temps, 300, 9)
    assert o["rc"] == 0
    g = rp.anneal(prob, t, q, pk["r_star"], pk["population"], temps, 300, 9)
    assert g["level_kernel"] == kernel
    rate = o["trace"][..., 6].sum(axis=1) / o["trace"][..., 7].sum(axis=1)
    assert rate[0] > 0.99 and rate[-1] < 0.2 and np.any((rate > 0.3) & (rate < 0.7))
    for k in ("parents", "trace", "population", "best_layout"):
        assert np.array_equal(g[k].cpu().numpy(), o[k])


@gpu
@pytest.mark.parametrize("P,L,shards", [(4, 5, 2), (8, 31, 1), (16, 40, 2), (32, 3, 1), (64, 6, 1)])
@pytest.mark.parametrize("offset", [0, 1])
def test_q_alignment(P, L, shards, offset):
    """The whole path on a q that starts 4 bytes past a 16-byte boundary, which
    the kernels without 16-byte loads take: window bounds, cell sums, scores,
    the annealing's start rows and their rewrite to chunks."""
    import torch
    import oracle as O
    import paper_2608_12146_amd as rp
    _log(f"q alignment P={P} L={L} shards={shards} offset={offset}")
    D, R = 4, 5
    rng = np.random.default_rng([26, P, L])
    t = rng.integers(1, 60, size=R * D * 4 + 3)
    t, q, kw = _pack_case(len(t), D, shards, int(-(-t.sum() // (R * D)) * 1.5) + 40, t, L=L, P=P)
    kw["min_rows"] = R
    flat = torch.empty(q.size + 4, dtype=torch.int32, device="cuda")
    qd = flat[offset:offset + q.size].view(q.shape)
    assert flat.data_ptr() % 16 == 0
    qd.copy_(torch.as_tensor(q))
    pb, prob = O.Problem.from_dict(kw), rp.Problem.from_dict(kw)
    o = O.pack_rows(pb, t, q, 3, 8, 4, 12)
    g = rp.pack_rows(prob, t, qd, 3, 8, 4, 12)
    assert o["rc"] == 0 and g["r_star"] == o["r_star"]
    assert np.array_equal(g["population"].cpu().numpy(), o["population"])
    assert np.array_equal(g["scores"].cpu().numpy(), o["scores"])
    ev = rp.eval_objective(prob, t, qd, g["r_star"], g["population"], want_J=True)
    assert np.array_equal(ev["scores"].cpu().numpy(), o["scores"])
    for m in range(len(o["population"])):
        assert np.array_equal(ev["J"][m].cpu().numpy(),
                              O.score(pb, t, q, o["r_star"], o["population"][m], want_J=True)[2])
    temps = np.array([1e-1, 1e-2, 1e-3])
    oa = O.anneal(pb, t, q, o["r_star"], o["population"], temps, 64, 9)
    ga = rp.anneal(prob, t, qd, o["r_star"], o["population"], temps, 64, 9)
    assert ga["level_kernel"] in ("chain", "chain_run")
    for k in ("trace", "parents", "population", "best_layout"):
        assert np.array_equal(ga[k].cpu().numpy(), oa[k])


@gpu
@pytest.mark.parametrize("N,D,R,shards", [(200, 4, 2, 1), (203, 2, 2, 1), (600, 4, 2, 1), (900, 4, 7, 2), (37, 4, 3, 1),
                                          (29, 2, 3, 1), (31, 2, 2, 2)])
def test_anneal_pool_room(N, D, R, shards):
    """64 ranks: the pool's spare room (N / 4 places, a multiple of 8) under
    hot levels of relocations -- blocks that fit and grow in place, the room
    running out and the pool packed again, cells above and below 32 members,
    blocks larger than the room (cells of a quarter of the samples) and, below
    32 samples, no room at all."""
    import oracle as O
    import paper_2608_12146_amd as rp
    _log(f"pool room N={N} D={D} R={R} shards={shards}")
    rng = np.random.default_rng([20, N, D])
    t = rng.integers(1, 60, size=N)
    t, q, kw = _pack_case(N, D, shards, int(-(-t.sum() // (R * D)) * 1.6) + 60, t, L=33, P=64)
    kw["min_rows"] = R
    pb, prob = O.Problem.from_dict(kw), rp.Problem.from_dict(kw)
    pk = O.pack_rows(pb, t, q, 3, 8, 4, 12)
    assert pk["rc"] == 0
    temps = np.array([3.0, 1.0, 0.1, 1e-2, 1e-3, 1e-4])
    o = O.anneal(pb, t, q, pk["r_star"], pk["population"], temps, 200, 9)
    g = rp.anneal(prob, t, q, pk["r_star"], pk["population"], temps, 200, 9)
    assert g["level_kernel"] == "chain"
    assert o["trace"][..., 6].sum() > 100 * 12  # accepted moves
    assert np.array_equal(g["trace"].cpu().numpy(), o["trace"])
    assert np.array_equal(g["population"].cpu().numpy(), o["population"])
    assert np.array_equal(g["best_layout"].cpu().numpy(), o["best_layout"])


@gpu
@pytest.mark.parametrize("K,N,fill", [(1, 3, 0.5), (64, 64, 0.9), (65, 200, 0.99), (128, 129, 1.0), (300, 900, 0.97),
                                      (4096, 4500, 0.9), (4097, 4300, 0.9)])
@pytest.mark.parametrize("scale", [1, 1 << 23])
def test_fixed_bin_chunks(K, N, fill, scale):
    """The search over part-filled chunks of cells, equal lengths, dead ends
    and backtracking over blocks of samples, the most chunked cells and the
    first count past them, with a cap below and above 2^31."""
    import oracle.fixedbin as F
    import paper_2608_12146_amd as rp
    _log(f"fixed bin K={K} N={N} fill={fill} scale={scale}")
    rng = np.random.default_rng([19, K, N])
    for rep in range(3):
        t = rng.integers(1, 60, size=N) if rep else np.repeat(rng.integers(1, 60, size=(N + 2) // 3), 3)[:N]
        cap = max(int(t.max()), int(t.sum() / (K * fill)) + 1)
        t, cap = (t * scale).astype(np.int32), cap * scale
        prob = rp.Problem(N, 0, 1, 1, 1, 1, 1, [0], cap, [1], [0])
        got = rp.fixed_bin_search(prob, t, K, 3000)
        want = F.search(t, cap, K, 3000)
        assert got[:2] == want[:2]
        assert (got[2] is None) == (want[2] is None)
        if got[2] is not None:
            assert np.array_equal(got[2].cpu().numpy(), want[2])


@gpu
@pytest.mark.parametrize("K,N,fill,hi", [(8, 24, 0.999, 200), (20, 60, 0.999, 1000), (30, 129, 0.9999, 300),
                                         (65, 200, 0.999, 5000), (130, 500, 0.9995, 300)])
@pytest.mark.parametrize("wide", [False, True])
def test_fixed_bin_backtracking(K, N, fill, hi, wide):
    """Searches that go back and forth for thousands of nodes: within one chunk
    of cells, over the ends of the blocks of samples and over chunks, with a
    cap below and above 2^31."""
    import oracle.fixedbin as F
    import paper_2608_12146_amd as rp
    _log(f"fixed bin backtracking K={K} N={N} wide={wide}")
    rng = np.random.default_rng([K, N])
    t = rng.integers(max(1, hi // 8), hi, size=N)
    cap = max(int(t.max()), int(t.sum() / (K * fill)) + 1)
    scale = (2**31 - 1) // int(t.max()) if wide else 1
    t, cap = (t * scale).astype(np.int32), cap * scale
    assert (cap >= 2**31) == wide
    prob = rp.Problem(N, 0, 1, 1, 1, 1, 1, [0], cap, [1], [0])
    got, want = rp.fixed_bin_search(prob, t, K, 20000), F.search(t, cap, K, 20000)
    assert want[1] > 10 * N and got[:2] == want[:2]
    assert (got[2] is None) == (want[2] is None)
    if got[2] is not None:
        assert np.array_equal(got[2].cpu().numpy(), want[2])

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

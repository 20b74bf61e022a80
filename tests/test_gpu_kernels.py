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

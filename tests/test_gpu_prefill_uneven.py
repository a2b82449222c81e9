"""Batches whose bounds promise many tiles while one short run of queries walks a long context: the tiles of that one are shared
out, the partial results go to the first units of the workspace, and a merge launch of fewer workgroups than tiles puts
them together.  Against the oracle at the attention tolerance, with the default workspace, with room for few partial results
(where a coarser cut than the best one is all that fits), and with none (nothing is split there)."""
import numpy as np
import pytest

from tests import helpers as H
from tests.test_gpu_parity import FA, SA, Layer

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    from paper_2604_07394_amd import binding
    return binding


@pytest.fixture(scope="module")
def ctxs(F):
    c = F.flux_create(0, 0), F.flux_create(0, 1)
    yield c
    for x in c:
        F.flux_destroy(x)


# kib: a workspace that holds no more units than the coarser cut needs (8 per sequence for padding among them; a unit is 128 rows
# of head dimension + 2 floats, behind 16 bytes per tile and the 8 MB and a page that other calls use)
@pytest.mark.parametrize("past,new,modes,hq,hkv,d,kib,coarser", [
    # 480 tiles by the bounds, lists of 85 blocks: 528 parts of 16 blocks by default, 368 units hold 344 of 29
    ([5400, 0, 300], [20, 2500, 100], [FA, FA, SA], 8, 8, 64, 20352, True),
    # 492, 110: 24 parts of one tile per head, which the fewest units that let a call split hold as well
    ([0, 0, 7000], [1300, 1250, 20], [FA, SA, FA], 16, 4, 128, 13952, False),
    # 140 tiles of a sequence, 128 workgroups merge them: 420 parts of 37 blocks by default, 344 units hold 280 of 57
    ([6000] + [900] * 7, [1100] + [30] * 7, [FA] + [SA, FA] * 3 + [FA], 16, 4, 128, 30592, True),
])
def test_one_long_list_among_many_tiles(F, ctxs, past, new, modes, hq, hkv, d, kib, coarser):
    lay = Layer(F, ctxs[0], 4000 + hq + d, len(new), hq, hkv, d, max(p + n for p, n in zip(past, new)) + 7, 16, 500, scales=True, block=1)
    _, kb, vb = lay.new_tokens(past)
    lay.append(kb, vb, past)
    qb, kb, vb = lay.new_tokens(new)
    lay.append(kb, vb, new)
    got, ref = lay.prefill(qb, new, modes)
    H.assert_close(got, ref, "uneven prefill")
    again, _ = lay.prefill(qb, new, modes, want_ref=False)
    assert np.array_equal(got, again)
    small = F.flux_create(0, kib << 10)
    results = []
    for c in (small, ctxs[1]):
        lay.ctx = c
        results.append(lay.prefill(qb, new, modes, want_ref=False)[0])
        H.assert_close(results[-1], ref, "uneven prefill")
        assert F.flux_last_device_status(c) == 0
    F.flux_destroy(small)
    assert not np.array_equal(got, results[1])                              # (it was split)
    assert not np.array_equal(results[0], results[1])                       # ... and where there is little room for parts as well
    assert np.array_equal(got, results[0]) != coarser
    assert F.flux_last_device_status(ctxs[0]) == 0

"""Batches whose bounds promise many tiles while one short run of queries walks a long context: the tiles of that one are shared
out, the partial results go to the first units of the workspace, and a merge launch of fewer workgroups than tiles puts
them together.  Against the oracle at the attention tolerance, with the default workspace, with room for few partial results, and
with none (nothing is split there)."""
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
    c = F.flux_create(0, 0), F.flux_create(0, 16 << 20), F.flux_create(0, 1)
    yield c
    for x in c:
        F.flux_destroy(x)


@pytest.mark.parametrize("past,new,modes,hq,hkv,d", [
    ([5400, 0, 300], [20, 2500, 100], [FA, FA, SA], 8, 8, 64),              # 480 tiles by the bounds, lists of 85 blocks
    ([0, 0, 7000], [1300, 1250, 20], [FA, SA, FA], 16, 4, 128),             # 492, 110
    ([6000] + [900] * 7, [1100] + [30] * 7, [FA] + [SA, FA] * 3 + [FA], 16, 4, 128),   # 140 tiles of a sequence, 128 workgroups merge them
])
def test_one_long_list_among_many_tiles(F, ctxs, past, new, modes, hq, hkv, d):
    lay = Layer(F, ctxs[0], 4000 + hq + d, len(new), hq, hkv, d, max(p + n for p, n in zip(past, new)) + 7, 16, 500, scales=True, block=1)
    _, kb, vb = lay.new_tokens(past)
    lay.append(kb, vb, past)
    qb, kb, vb = lay.new_tokens(new)
    lay.append(kb, vb, new)
    got, ref = lay.prefill(qb, new, modes)
    H.assert_close(got, ref, "uneven prefill")
    again, _ = lay.prefill(qb, new, modes, want_ref=False)
    assert np.array_equal(got, again)
    results = []
    for c in ctxs[1:]:
        lay.ctx = c
        results.append(lay.prefill(qb, new, modes, want_ref=False)[0])
        assert np.abs(results[-1] - ref).max() <= H.MAX_ABS
    assert not np.array_equal(got, results[1])                              # (it was split)
    for c in ctxs:
        assert F.flux_last_device_status(c) == 0

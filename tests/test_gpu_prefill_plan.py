"""Prefill launches that are planned on the device: tiles whose rows come from all heads of a group, ragged batches worked
off longest first, and (queries behind a cached context) tiles whose keys are shared out over several workgroups and
merged.  Against the oracle at the attention tolerance, and against the same call on a context whose workspace has no
room for partial results (nothing is split there; results differ in bits exactly where something was).  Both sides round every weight to bf16 (relative 2^-9), each against
softmax references of its own, so two correct results differ by at most 2 * 2^-9 * max|v - o| (3.5e-2 for values of up to 9)
in the worst case; the bound asserted is the attention tolerance of 1e-2."""
import numpy as np
import pytest
import torch

from oracle import flux_oracle as O
from paper_2604_07394_amd import synth
from tests import helpers as H
from tests.test_gpu_parity import Layer, FA, SA, cu, u8

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    from paper_2604_07394_amd import binding
    return binding


@pytest.fixture(scope="module")
def ctxs(F):
    c = F.flux_create(0, 0), F.flux_create(0, 1)            # the default workspace, and the smallest
    yield c
    for x in c:
        F.flux_destroy(x)


@pytest.mark.parametrize("past,new,modes,hq,hkv,d,n_sink,window,block", [
    ([3000], [1], [FA], 4, 1, 128, 16, 500, 1),             # one row of one token
    ([2113], [33], [FA], 7, 1, 128, 16, 500, 1),            # 231 rows: a tile and a ragged one, a group that divides neither
    ([1024, 1025], [31, 32], [FA, FA], 1, 1, 64, 16, 500, 1),   # 17 blocks: the shortest list that splits; group of one
    ([1500, 40, 5000, 0], [130, 40, 64, 1], [FA, FA, SA, FA], 8, 2, 64, 70, 2100, 1),   # ragged, split and whole tiles mixed
    ([3000, 3500, 2800], [512, 40, 30], [FA, FA, FA], 32, 8, 128, 16, 500, 1),   # 384 tiles by the bounds, 152 in fact
    ([4000, 2500], [17, 200], [SA, FA], 20, 1, 128, 64, 2048, 64),   # more rows of a token than columns of an MFMA, block rule
    ([1800, 1700, 1600], [5, 0, 300], [SA, SA, FA], 6, 3, 128, 0, 1200, 1),   # no new tokens in one; KV heads that do not divide 8
    ([2000] * 3 + [0] * 20, [3] * 3 + [50] * 20, [FA, SA] * 11 + [FA], 4, 2, 64, 5, 1300, 16),
])
def test_planned_prefill(F, ctxs, past, new, modes, hq, hkv, d, n_sink, window, block):
    batch = len(new)
    lay = Layer(F, ctxs[0], 3000 + hq + d, batch, hq, hkv, d, max(p + n for p, n in zip(past, new)) + 7, n_sink, window, scales=True, block=block)
    lay.cache.k.fill_(float("nan"))
    lay.cache.v.fill_(float("nan"))
    if sum(past):
        _, kb, vb = lay.new_tokens(past)
        lay.append(kb, vb, past)
    qb, kb, vb = lay.new_tokens(new)
    lay.append(kb, vb, new)
    got, ref = lay.prefill(qb, new, modes)
    H.assert_close(got, ref, "planned prefill")
    again, _ = lay.prefill(qb, new, modes, want_ref=False)
    assert np.array_equal(got, again)
    # bounds larger than needed, bf16 output
    t = sum(new)
    out16 = torch.zeros(t, hq, d, dtype=torch.bfloat16, device="cuda")
    F.flux_attn_prefill(ctxs[0], F.attn_cfg(hq, hkv, d, n_sink, window, 0.0, 0, block if block > 1 else 0), H.bits_to_torch(qb), cu(new), max(new),
                        max(lay.lens), lay.cache, u8(modes), out16)
    torch.cuda.synchronize()
    assert torch.equal(out16, torch.from_numpy(got).cuda().to(torch.bfloat16))
    loose, _ = lay.prefill(qb, new, modes, max_q_len=max(new) + 150, want_ref=False)
    assert np.abs(loose - ref).max() <= H.MAX_ABS
    lay.ctx = ctxs[1]
    whole, _ = lay.prefill(qb, new, modes, want_ref=False)
    assert np.abs(whole - got).max() <= H.MAX_ABS
    assert not np.array_equal(whole, got)                    # (every case splits: its sums are taken in another order)
    for c in ctxs:
        assert F.flux_last_device_status(c) == 0


@pytest.mark.parametrize("past,new,modes,hq,hkv,d,n_sink,window", [
    ([3000], [40], [SA], 8, 2, 128, 16, 128),               # may split by its bounds, but the window's list is short
    ([3000, 2900, 3001], [40, 1, 90], [SA, SA, SA], 4, 4, 64, 16, 300),
    ([640], [512], [FA], 32, 8, 128, 16, 128),              # 128 tiles of 18 blocks: not worth it
    ([0] * 9, [70] * 9, [FA, SA] * 4 + [FA], 8, 2, 64, 3, 40),   # sequences all alike
    ([0] * 5, [300, 1, 777, 0, 64], [FA, SA, FA, FA, SA], 14, 7, 128, 3, 40),
    ([0] * 4, [513, 400, 3, 1026], [FA, SA, FA, FA], 28, 4, 128, 3, 40),   # 1008 tiles of one head each
    ([0] * 24, [100, 128, 97, 100] * 6, [FA] * 24, 14, 2, 64, 3, 40),      # 672, every sequence one per head
    ([0] * 6, [385, 400, 512, 386, 420, 500], [FA] * 6, 12, 3, 128, 3, 40),   # as many tiles each, other lists: ranked
    ([0] * 8, [900] * 8, [FA] * 8, 16, 16, 64, 3, 40),       # all alike, 16 KV heads, several rounds
    ([0] * 40, [17] * 40, [SA, FA] * 20, 32, 2, 128, 3, 8),  # short: packed, group of 16
    ([90] * 33, [5] * 33, [FA] * 33, 20, 5, 64, 3, 40),      # behind a context: packed, KV heads that do not divide 8
])
def test_calls_that_split_nothing(F, ctxs, past, new, modes, hq, hkv, d, n_sink, window):
    """Bit-identical to the call that has no room to split, also after a call on the same context that did."""
    batch = len(new)
    lay = Layer(F, ctxs[0], 3200 + hq + d, batch, hq, hkv, d, max(p + n for p, n in zip(past, new)), n_sink, window, scales=True)
    if sum(past):
        _, kb, vb = lay.new_tokens(past)
        lay.append(kb, vb, past)
    qb, kb, vb = lay.new_tokens(new)
    lay.append(kb, vb, new)
    lay.prefill(qb, new, [FA] * batch, want_ref=False)
    got, ref = lay.prefill(qb, new, modes)
    H.assert_close(got, ref, "nothing split")
    lay.ctx = ctxs[1]
    whole, _ = lay.prefill(qb, new, modes, want_ref=False)
    assert np.array_equal(whole, got)
    for c in ctxs:
        assert F.flux_last_device_status(c) == 0


@pytest.mark.parametrize("n,hq,hkv,n_sink,window,peak", [
    (620, 6, 2, 0, 7, 1.0),                                 # rows of a wave whose windows begin in different key blocks
    (400, 8, 1, 0, 7, 1.0),
    (500, 4, 2, 300, 64, 40.0),                             # some rows' weights leave the guarded range, others' do not
])
def test_a_row_does_not_depend_on_the_rows_of_its_wave(F, ctxs, n, hq, hkv, n_sink, window, peak):
    """The launch shape of long prompts (rows of all heads of a group share a wave) against the ordinary one (rows of one
    head): the same bits, also where some rows of a wave move their softmax reference and others do not."""
    lay = Layer(F, ctxs[0], 3300 + n, 1, hq, hkv, 128, 32768, n_sink, window, scales=True)
    qb, kb, vb = lay.new_tokens([n])
    if peak != 1.0:
        q = O.bf16_to_f64(qb).astype(np.float32)
        q[::7] *= peak
        qb = synth.f32_to_bf16_bits(q)
    lay.append(kb, vb, [n])
    for mode in (FA, SA):
        got, ref = lay.prefill(qb, [n], [mode])
        H.assert_close(got, ref, "ordinary launch shape")
        wide, _ = lay.prefill(qb, [n], [mode], max_q_len=32768, want_ref=False)
        assert np.array_equal(wide, got)


def test_batches_past_the_planned_size_and_bad_lengths(F, ctxs):
    """65 sequences are not planned; 64 are.  A sequence with more query rows than cached positions is cut and reported."""
    for batch in (64, 65):
        new = [1 + (7 * i) % 90 for i in range(batch)]
        lay = Layer(F, ctxs[0], 3100 + batch, batch, 4, 2, 64, 128, 3, 40)
        modes = [i % 2 for i in range(batch)]
        qb, kb, vb = lay.new_tokens(new)
        lay.append(kb, vb, new)
        got, ref = lay.prefill(qb, new, modes)
        H.assert_close(got, ref, f"{batch} sequences")
    assert F.flux_last_device_status(ctxs[0]) == 0
    lay.cache.kv_len[3] = 2                                  # (its first 2 of 22 rows are computed; the others are not touched)
    keep = torch.full((sum(new), 4, 64), 7.0, dtype=torch.float32, device="cuda")
    small = F.KVCache(lay.cache.k[:8], lay.cache.v[:8], lay.cache.kv_len[:8])
    F.flux_attn_prefill(ctxs[0], lay.cfg, H.bits_to_torch(qb), cu(new[:8]), max(new[:8]), 128, small, u8([FA] * 8), keep)
    torch.cuda.synchronize()
    at = sum(new[:3])
    assert (keep[at:at + 2] != 7.0).any() and (keep[at + 2:at + new[3]] == 7.0).all()
    assert F.flux_last_device_status(ctxs[0]) == F.FLUX_DEV_BAD_LENGTH

"""Decode calls where the ranges of workgroups meet the lists in every way: one list per workgroup, lists cut into fours and
eights, ranges that begin and end inside lists, whole lists inside a range, lists that go on over several ranges, empty caches
and more sequences than lanes.  Against the oracle at the attention tolerance; the fused step, the call without a context
(its merge is a launch of its own) and a replayed graph give the same bits."""
import math

import numpy as np
import pytest
import torch

from oracle import flux_oracle as O
from paper_2604_07394_amd import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu

FA, SA = 1, 0


@pytest.mark.parametrize("hq,hkv,d,lens", [
    (8, 4, 64, [(i * 379) % 1500 for i in range(70)]),        # equal ranges over more than 64 sequences, some empty
    (40, 2, 64, [4000, 0, 1, 3100, 2050]),                    # by eight blocks; two query blocks per KV head
    (2, 1, 64, [(i * 131) % 97 if i % 5 else 0 for i in range(2048)]),   # 32 sequences per lane, all that the table in LDS holds
    (2, 1, 64, [(i * 131) % 97 if i % 5 else 0 for i in range(2049)]),   # ... and more
    (4, 2, 128, [0] * 30 + [900] + [0] * 200 + [40, 3000] + [0] * 60),   # runs of empty caches between lists
    (8, 8, 128, [20000, 40, 17000, 90, 33, 64, 15000, 300]),  # ranges that begin behind the last block of a short list
    (8, 8, 64, [20000, 40, 17000, 90, 33, 64, 15000, 300]),   # ... and 64 lists of head dimension 64: 512 of them
    (4, 4, 128, [900, 340, 1200] * 22),                       # 264 lists: 512 equal ranges
    (4, 4, 128, [900, 340, 1200] * 21),                       # 252: 256 of them
    (4, 4, 128, [256] * 65),                                  # more than 64 sequences: by eight, one workgroup each
    (4, 4, 128, [(37 * i) % 480 + 1 for i in range(66)]),     # 264 lists of up to 16 blocks: one workgroup each
    (8, 8, 64, [(97 * i) % 740 + 1 for i in range(60)]),      # 480 of up to 24: the same
    (8, 8, 64, [(97 * i) % 740 + 1 for i in range(40)]),      # 320 of them: equal ranges
    (8, 8, 64, [(97 * i) % 1000 + 1 for i in range(32)]),     # 256 of up to 32: one each
    (8, 8, 128, [(97 * i) % 760 + 1 for i in range(32)]),     # 256 of up to 24: one each
    (8, 8, 128, [700] * 64),                                  # 512 lists of one length, one workgroup each
    (8, 8, 128, [800] * 64),                                  # ... one range each
    (8, 8, 128, [800] * 32 + [0]),                            # 256 of them, and an empty sequence: 256 ranges
    (8, 8, 128, [800] * 32 + [801]),                          # (one length: as many blocks)
    (4, 2, 64, [5001, 0] * 8),                                # 16 lists of one length, 16 ranges each
    (16, 16, 64, [1024] * 4),                                 # by four: as many as there may be (of four waves under the loosest bound)
    (16, 16, 64, [1024] * 4 + [1]),                           # ... and one list more: by eight, equal ranges under the loosest bound
    (16, 16, 64, [1500, 100, 1490, 70, 40, 1400, 0, 33]),     # half of the lists shorter than a range
    # eight waves: every list of up to eight blocks, one of nine (by four), more merged rows than are taken by four, as many
    # workgroups and sequences as there may be, and one more; counts on one word (up to 128 workgroups) and on 32
    (4, 4, 128, [256, 224, 1]),
    (4, 4, 128, [256, 257, 1]),
    (32, 2, 128, [4000, 33]),
    (32, 8, 128, [4095]),
    (32, 8, 128, [4096]),
    (32, 8, 128, [16383]),
    (32, 8, 128, [16384]),
    (8, 8, 64, [(37 * i) % 255 + 1 for i in range(16)]),
    (8, 8, 64, [(37 * i) % 255 + 1 for i in range(17)]),
    (8, 8, 64, [(37 * i) % 255 + 1 for i in range(64)]),
    (8, 8, 64, [(37 * i) % 255 + 1 for i in range(65)]),
    (16, 1, 128, [(37 * i) % 40 + 1 for i in range(504)]),    # as many rows as the small region holds
    (1, 1, 64, [(37 * i) % 255 for i in range(512)]),
    (1, 1, 64, [(37 * i) % 255 for i in range(513)]),
    (6, 2, 128, [33000]),                                     # 32 columns of heads, parts in several runs of the merge
    (32, 2, 128, [9000, 8000, 700]),                          # 16 heads per KV head: no waves to share the runs
    (7, 1, 64, [70000, 3]),                                   # one pair over nearly all ranges
])
def test_ranges_and_lists(hq, hkv, d, lens):
    from paper_2604_07394_amd import binding as F
    ctx = F.flux_create(0)
    b, n_sink, window, seed = len(lens), 8, 3000, 800 + hq
    modes = [FA if i % 3 != 1 else SA for i in range(b)]
    kb = synth.normal_bf16(seed, synth.stream_id(synth.STREAM_K), (sum(lens) + b, hkv, d))
    vb = synth.normal_bf16(seed, synth.stream_id(synth.STREAM_V), (sum(lens) + b, hkv, d))
    qb = synth.normal_bf16(seed, synth.stream_id(synth.STREAM_QDEC), (b, hq, d))
    cfg = F.attn_cfg(hq, hkv, d, n_sink, window, 0.0, 1)
    t, cap = sum(lens), max(lens) + 1
    room = max(2 * cap, 20000) if b * hkv <= 200 else cap + 2000
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32, device="cuda")
    md = torch.tensor(modes, dtype=torch.uint8, device="cuda")
    q, kn, vn = H.bits_to_torch(qb), H.bits_to_torch(kb[t:]), H.bits_to_torch(vb[t:])
    cache = F.KVCache.empty(b, hkv, room, d)
    cache.k.fill_(float("nan"))
    cache.v.fill_(float("nan"))
    F.flux_kv_append(ctx, cache, hkv, d, H.bits_to_torch(kb[:t]), H.bits_to_torch(vb[:t]), cu, t, max(lens))
    out = torch.full((b, hq, d), float("nan"), dtype=torch.float32, device="cuda")
    F.flux_attn_decode(ctx, cfg, q, max(lens), cache, md, out)            # (an empty cache yields zeros)
    torch.cuda.synchronize()
    assert torch.isfinite(out).all()
    assert all(n > 0 or not out[i].any() for i, n in enumerate(lens))
    F.flux_attn_decode_append(ctx, cfg, q, kn, vn, cap, cache, md, out)
    torch.cuda.synchronize()
    assert cache.kv_len.tolist() == [n + 1 for n in lens]
    kf, vf, qf = O.bf16_to_f64(kb), O.bf16_to_f64(vb), O.bf16_to_f64(qb)
    at = 0
    for i, n in enumerate(lens):
        if b < 10 or i % (7 if b < 300 else 101) == 0 or n > 800:
            k1, v1 = np.concatenate([kf[at:at + n], kf[t + i:t + i + 1]]), np.concatenate([vf[at:at + n], vf[t + i:t + i + 1]])
            H.assert_close(out[i].cpu().numpy(), O.attention(qf[i:i + 1], k1, v1, modes[i], n_sink, window)[0], f"sequence {i} of {n + 1} keys")
        at += n
    again = torch.empty_like(out)
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    # the bound moves the cut (grid, waves of a workgroup, blocks that it takes): the call without a context gives the bits of the
    # call with one at every bound, and two cuts of a list differ by what either may be off (see the test of the error below)
    for bound in (cap, cap + 255, room):
        same = torch.full_like(out, float("nan"))
        F.flux_attn_decode(ctx, cfg, q, bound, cache, md, same)
        again.fill_(float("nan"))
        F.flux_attn_decode_static(cfg, q, bound, cache, md, again, status)
        torch.cuda.synchronize()
        assert torch.equal(again, same) and int(status[0]) == 0
        assert bound > cap or torch.equal(same, out)
        assert ((same - out).double().flatten(1).norm(dim=1) <= 4 * 2.0 ** -16 * out.double().flatten(1).norm(dim=1)).all()
    g = torch.cuda.CUDAGraph()
    s = torch.cuda.Stream()
    with torch.cuda.graph(g, stream=s):
        cache.kv_len.sub_(1)
        F.flux_attn_decode_append(ctx, cfg, q, kn, vn, cap, cache, md, again, stream=s)
    for _ in range(4):
        again.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(again, out) and cache.kv_len.tolist() == [n + 1 for n in lens]
    assert F.flux_last_device_status(ctx) == 0
    F.flux_destroy(ctx)


# 16 query heads per KV head of 128: the rows of 512 workgroups do not fit the small region.  Where the host's bounds allow 1024
# units of 256 keys they go to the partials (which a workspace of the reported size has just the room for), otherwise 256
# workgroups share the keys out.  The last case has its keys in the sequences at the end, behind empty ones.
@pytest.mark.parametrize("hq,hkv,lens,bounds", [
    (16, 1, [16300] * 8, (16301, 32768)),                     # 256 equal ranges / 512 workgroups by eight blocks, in the partials
    (32, 2, [8100] * 8, (8101, 16384)),
    (64, 4, [32768], (32769, 65536)),
    (16, 1, [16300, 700, 0, 33, 9000, 1, 128, 4000], (16301, 32768)),   # equal ranges
    (16, 1, [100 + i % 29 for i in range(505)], (129, 300)),  # more lists than workgroups whose rows fit
    (16, 1, [0] * 384 + [512] * 128, (512, 600)),
])
def test_rows_of_sixteen_heads(hq, hkv, lens, bounds):
    from paper_2604_07394_amd import binding as F
    b, d, cap = len(lens), 128, max(max(bounds), max(lens) + 1)
    g = torch.Generator(device="cuda").manual_seed(hq + b)
    k, v = (torch.empty(b, hkv, cap, d, dtype=torch.bfloat16, device="cuda").normal_(generator=g) for _ in range(2))
    q = torch.empty(b, hq, d, dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    cache = F.KVCache(k, v, torch.tensor(lens, dtype=torch.int32, device="cuda"))
    md = torch.full((b,), FA, dtype=torch.uint8, device="cuda")
    cfg = F.attn_cfg(hq, hkv, d, 8, 3000, 0.0, 1)
    rows = sorted({lens.index(n) for n in lens})[:3] + [b - 1]
    want = {i: O.attention(q[i:i + 1].double().cpu().numpy(), k[i, :, :lens[i]].transpose(0, 1).double().cpu().numpy(),
                           v[i, :, :lens[i]].transpose(0, 1).double().cpu().numpy(), FA, 8, 3000)[0] for i in rows if lens[i] > 0}
    for bound in bounds:
        ctx = F.flux_create(0, F.flux_workspace_needed(cfg, b, bound))
        outs = []
        for turn in range(3):
            out = torch.full((b, hq, d), float("nan"), dtype=torch.float32, device="cuda")
            if turn < 2:
                F.flux_attn_decode(ctx, cfg, q, bound, cache, md, out)
            else:
                F.flux_attn_decode_static(cfg, q, bound, cache, md, out)
            torch.cuda.synchronize()
            outs.append(out)
        assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
        assert all(n > 0 or not outs[0][i].any() for i, n in enumerate(lens))
        for i in want:
            H.assert_close(outs[0][i].cpu().numpy(), want[i], f"sequence {i} under bound {bound}")
        assert F.flux_last_device_status(ctx) == 0
        F.flux_destroy(ctx)


@pytest.mark.parametrize("hq,hkv,d,n,batch", [(32, 8, 128, 4224, 8), (4, 1, 128, 32768, 2), (28, 4, 128, 2112, 16), (8, 2, 64, 700, 3), (16, 1, 64, 250, 2)])
def test_the_error_of_a_list_is_that_of_its_sums(hq, hkv, d, n, batch):
    """However a list is cut, its weights reach the result to 2^-16 (two bf16 terms, the second rounded from what eight bits
    leave) and scores and sums are fp32.  The sum over keys of weight errors is against one of the weights themselves, both
    with V's random signs: 2^-16 of the result at the most where they all lie on one side, and as much again for the scores'
    exponents (2^-22 of a score of some 5 * log2(e), and the sums).  Weights of one bf16 term lie ten times above the bound."""
    from paper_2604_07394_amd import binding as F
    g = torch.Generator(device="cuda").manual_seed(n)
    k, v = (torch.empty(batch, hkv, n, d, dtype=torch.bfloat16, device="cuda").normal_(generator=g) for _ in range(2))
    q = torch.empty(batch, hq, d, dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    out = torch.full((batch, hq, d), float("nan"), dtype=torch.float32, device="cuda")
    ctx = F.flux_create(0)
    F.flux_attn_decode(ctx, F.attn_cfg(hq, hkv, d, 0, 1, 0.0, 1), q, n, F.KVCache(k, v, torch.full((batch,), n, dtype=torch.int32, device="cuda")),
                       torch.full((batch,), FA, dtype=torch.uint8, device="cuda"), out)
    torch.cuda.synchronize()
    for b in (0, batch - 1):
        s = (q[b].double().cpu().view(hkv, -1, d) @ k[b].double().cpu().transpose(1, 2)) * d ** -0.5
        want = (torch.softmax(s, -1) @ v[b].double().cpu()).view(hq, d)
        err = float((out[b].cpu().double() - want).norm() / want.norm())
        print(f"rel-L2 {err:.2e}")
        assert err <= 2 * 2.0 ** -16
    F.flux_destroy(ctx)


def test_an_infinite_value_row_stays_infinite():
    """A row of V that holds an infinity gives that infinity, whatever bits its weight has (one key: a weight of exactly 1;
    32 equal keys: 1 each; 64 keys of different weights)."""
    from paper_2604_07394_amd import binding as F
    ctx = F.flux_create(0)
    for n in (32, 64):
        k = torch.zeros(1, 1, n, 64, dtype=torch.bfloat16, device="cuda")
        if n == 64:
            k.normal_(generator=torch.Generator(device="cuda").manual_seed(1))
        v = torch.ones(1, 1, n, 64, dtype=torch.bfloat16, device="cuda")
        v[0, 0, 5, 3], v[0, 0, 9, 4] = float("inf"), -float("inf")
        out = torch.zeros(1, 4, 64, dtype=torch.float32, device="cuda")
        F.flux_attn_decode(ctx, F.attn_cfg(4, 1, 64, 0, 1, 0.0, 1), torch.ones(1, 4, 64, dtype=torch.bfloat16, device="cuda"), n,
                           F.KVCache(k, v, torch.tensor([n], dtype=torch.int32, device="cuda")), torch.ones(1, dtype=torch.uint8, device="cuda"), out)
        torch.cuda.synchronize()
        assert torch.isposinf(out[:, :, 3]).all() and torch.isneginf(out[:, :, 4]).all()
        out[:, :, 3:5] = 1.0
        assert torch.allclose(out, torch.ones_like(out), atol=1e-5)
    F.flux_destroy(ctx)


def test_an_infinite_value_row_stays_infinite_down_to_the_smallest_weight():
    """... and however small its weight is, as long as that is a normal number: sequence i has one key 64 * (8 + i / 16) / 8 below
    the others (weights of 2^-92 to 2^-125, with and without bits below the upper eight)."""
    from paper_2604_07394_amd import binding as F
    b, n, d = 46, 64, 64
    below = 8 + torch.arange(b, device="cuda") / 16
    k = torch.zeros(b, 1, n, d, dtype=torch.bfloat16, device="cuda")
    k[:, 0, 5] = -below[:, None].to(torch.bfloat16)
    v = torch.ones(b, 1, n, d, dtype=torch.bfloat16, device="cuda")
    v[:, 0, 5, 3] = float("inf")
    out = torch.zeros(b, 4, d, dtype=torch.float32, device="cuda")
    # scale: 1 / 8, or what makes the weights of whole keys powers of two
    for scale in (0.0, math.log(2) / 6):
        ctx = F.flux_create(0)
        F.flux_attn_decode(ctx, F.attn_cfg(4, 1, d, 0, 1, scale, 1), torch.ones(b, 4, d, dtype=torch.bfloat16, device="cuda"), n,
                           F.KVCache(k, v, torch.full((b,), n, dtype=torch.int32, device="cuda")), torch.ones(b, dtype=torch.uint8, device="cuda"), out)
        torch.cuda.synchronize()
        weight = -64 * below * (scale or 0.125) / math.log(2)
        assert torch.isposinf(out[weight > -126, :, 3]).all(), weight[~torch.isposinf(out[:, :, 3]).all(1)]
        out[:, :, 3] = 1.0
        assert torch.allclose(out, torch.ones_like(out), atol=1e-5)
        F.flux_destroy(ctx)


@pytest.mark.parametrize("fp32", [0, 1])
@pytest.mark.parametrize("lens", [[0], [0] * 70, [0] * 300 + [5], [0, 0, 700, 0] * 8, [3000] + [0] * 63, [0] * 64 + [3000]])
def test_every_empty_cache_yields_zeros(lens, fp32):
    """The rows of sequences without keys are shared out over the workgroups: all of them are written, by calls with and
    without a context, where other workgroups have keys to stream and where nobody has."""
    from paper_2604_07394_amd import binding as F
    b, hq, hkv, d, cap = len(lens), 6, 2, 64, 3072
    g = torch.Generator(device="cuda").manual_seed(b)
    k, v = (torch.empty(b, hkv, cap, d, dtype=torch.bfloat16, device="cuda").normal_(generator=g) for _ in range(2))
    q = torch.empty(b, hq, d, dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    cache = F.KVCache(k, v, torch.tensor(lens, dtype=torch.int32, device="cuda"))
    md = torch.tensor([FA if i % 2 else SA for i in range(b)], dtype=torch.uint8, device="cuda")
    ctx, cfg = F.flux_create(0), F.attn_cfg(hq, hkv, d, 8, 3000, 0.0, fp32)
    outs = []
    for call in ("context", "static"):
        out = torch.full((b, hq, d), float("nan"), dtype=torch.float32 if fp32 else torch.bfloat16, device="cuda")
        if call == "context":
            F.flux_attn_decode(ctx, cfg, q, cap, cache, md, out)
        else:
            F.flux_attn_decode_static(cfg, q, cap, cache, md, out)
        torch.cuda.synchronize()
        assert torch.isfinite(out.float()).all()
        assert all(n > 0 or not out[i].any() for i, n in enumerate(lens)) and all(n == 0 or out[i].any() for i, n in enumerate(lens))
        outs.append(out)
    assert torch.equal(*outs)
    assert F.flux_last_device_status(ctx) == 0
    F.flux_destroy(ctx)


def test_more_than_a_million_lists_with_few_keys():
    """Above 2^20 lists nothing is rounded up, so that the live ones may have fewer blocks than there are workgroups: 256 of
    them would hold empty ranges between the blocks of a list, which nobody counts."""
    from paper_2604_07394_amd import binding as F
    b, h, d, cap = 131073, 8, 64, 200
    live = {0: 130, 1: 1, 77777: 200, b - 1: 65}
    k, v = (torch.empty(4, h, cap, d, dtype=torch.bfloat16, device="cuda").normal_(generator=torch.Generator(device="cuda").manual_seed(i)) for i in range(2))
    cache = F.KVCache(k[:1].expand(b, h, cap, d), v[:1].expand(b, h, cap, d), torch.zeros(b, dtype=torch.int32, device="cuda"))
    q = torch.zeros(b, h, d, dtype=torch.bfloat16, device="cuda").normal_(generator=torch.Generator(device="cuda").manual_seed(2))
    cfg = F.attn_cfg(h, h, d, 0, 1, 0.0, 1)
    ctx = F.flux_create(0, F.flux_workspace_needed(cfg, b, cap))
    md = torch.ones(b, dtype=torch.uint8, device="cuda")
    out = torch.full((b, h, d), float("nan"), dtype=torch.float32, device="cuda")
    for lens in (live, {5: 33}, {i: 190 for i in range(0, b, 3000)}):
        cache.kv_len.zero_()
        cache.kv_len[torch.tensor(list(lens), device="cuda")] = torch.tensor(list(lens.values()), dtype=torch.int32, device="cuda")
        for _ in range(2):
            out.fill_(float("nan"))
            F.flux_attn_decode(ctx, cfg, q, cap, cache, md, out)
            torch.cuda.synchronize()
            assert torch.isfinite(out).all() and int((out.abs().sum((1, 2)) > 0).sum()) == len(lens)
            for i, n in lens.items():
                s = (q[i].double().cpu()[:, None] @ k[0, :, :n].double().cpu().transpose(1, 2))[:, 0] * d ** -0.5
                H.assert_close(out[i].cpu().numpy(), (torch.softmax(s, -1)[:, None] @ v[0, :, :n].double().cpu())[:, 0].numpy(), f"sequence {i}")
    assert F.flux_last_device_status(ctx) == 0
    F.flux_destroy(ctx)

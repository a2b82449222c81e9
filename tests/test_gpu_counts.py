"""The workgroups of a launch find out which of them is the last by counting themselves.  Appends, on one word or on
several: lengths and rows of calls on both sides of every step (64 and 65 workgroups, one more and one less than a multiple
of the 16 words, 4096 and 4097), twice in a row on the same counters, another size between them.  Router: a word a sequence."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    from paper_2604_07394_amd import binding
    return binding


@pytest.fixture(scope="module")
def ctx(F):
    c = F.flux_create(0, 0)
    yield c
    F.flux_destroy(c)


# one workgroup per 16 tokens at 2 KV heads of 64
@pytest.mark.parametrize("wgs,batch", [(1, 1), (64, 3), (65, 1), (79, 5), (80, 1), (81, 130), (513, 1), (513, 129), (4096, 2), (4097, 1)])
def test_the_last_workgroup_moves_the_lengths(F, ctx, wgs, batch):
    hkv, d, t = 2, 64, 16 * wgs - 3
    lens = [t // batch] * (batch - 1)
    lens.append(t - sum(lens))
    cu = torch.tensor([sum(lens[:i]) for i in range(batch + 1)], dtype=torch.int32, device="cuda")
    one = torch.arange(batch + 1, dtype=torch.int32, device="cuda")
    cache = F.KVCache.empty(batch, hkv, 2 * max(lens) + 1, d)
    g = torch.Generator(device="cuda").manual_seed(wgs)
    x = [torch.randn(t, hkv, d, device="cuda", generator=g).to(torch.bfloat16) for _ in range(4)]
    for turn in range(2):
        F.flux_kv_append(ctx, cache, hkv, d, x[2 * turn], x[2 * turn + 1], cu, t, max(lens))
        if turn == 0:
            F.flux_kv_append(ctx, cache, hkv, d, x[0], x[1], one, batch, 1)
    torch.cuda.synchronize()
    assert cache.kv_len.tolist() == [2 * n + 1 for n in lens]
    for i, n in enumerate(lens):
        off = sum(lens[:i])
        for c, first, second in ((cache.k, x[0], x[2]), (cache.v, x[1], x[3])):
            assert torch.equal(c[i, :, :n], first[off:off + n].transpose(0, 1))
            assert torch.equal(c[i, :, n], first[i])
            assert torch.equal(c[i, :, n + 1:2 * n + 1], second[off:off + n].transpose(0, 1))
    assert F.flux_last_device_status(ctx) == 0


@pytest.mark.parametrize("batch", [1, 24, 25, 64])
def test_every_sequence_of_a_router_call_gets_its_head(F, ctx, batch):
    """Up to 24 sequences have their counters on lines of their own, more share lines: both give every sequence the logits
    that it gets in a call of its own, twice in a row."""
    hidden, inner, n = 512, 64, 70
    g = torch.Generator(device="cuda").manual_seed(batch)
    x = torch.randn(batch * n, hidden, device="cuda", generator=g).to(torch.bfloat16)
    w1 = (torch.randn(inner, hidden, device="cuda", generator=g) * 0.02).to(torch.bfloat16)
    w2 = (torch.randn(2, inner, device="cuda", generator=g) * 0.02).to(torch.bfloat16)
    cu = torch.arange(0, batch * n + 1, n, dtype=torch.int32, device="cuda")
    mode = torch.full((2, batch), 7, dtype=torch.uint8, device="cuda")
    logits = torch.full((3, batch, 2), float("nan"), dtype=torch.float32, device="cuda")
    for turn in range(2):
        F.flux_router(ctx, x, cu, batch, hidden, 16, w1, None, w2, None, inner, mode[turn], logits[turn])
    alone = torch.zeros(1, dtype=torch.uint8, device="cuda")
    for b in range(batch):
        F.flux_router(ctx, x[b * n:], cu[:2], 1, hidden, 16, w1, None, w2, None, inner, alone, logits[2, b])
    torch.cuda.synchronize()
    assert torch.equal(logits[0], logits[2]) and torch.equal(logits[1], logits[2])
    assert torch.equal(mode[0], mode[1]) and torch.equal(mode[0].bool(), logits[0, :, 0] >= logits[0, :, 1])

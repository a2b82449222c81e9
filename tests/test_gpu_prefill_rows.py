"""Launches of few tiles give every wave 16 query rows instead of 32: parity with the fp64 oracle at the edges of the
64-row tiles, and bit for bit the results of the 128-row tiles (which the block-sparse form with everything kept uses)."""
import numpy as np
import pytest
import torch

from oracle import flux_oracle as O
from paper_2604_07394_amd import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu

FA, SA = 1, 0


@pytest.fixture(scope="module")
def F():
    from paper_2604_07394_amd import binding
    return binding


@pytest.fixture(scope="module")
def ctx(F):
    c = F.flux_create(0, 0)
    yield c
    F.flux_destroy(c)


def i32(x):
    return torch.tensor(x, dtype=torch.int32, device="cuda")


def u8(x):
    return torch.tensor(x, dtype=torch.uint8, device="cuda")


# heads, head size, new tokens and cached positions before them; the last four lie on both sides of the rule's
# bounds (14 and 15 tiles of 128 rows x 32 heads of a whole prompt, 8 and 9 behind a context)
@pytest.mark.parametrize("hq,hkv,d,n,past", [(8, 2, 64, 1, 0), (8, 2, 128, 16, 0), (7, 1, 128, 63, 0), (8, 2, 64, 64, 0), (4, 4, 128, 65, 3),
                                             (8, 8, 128, 127, 500), (20, 1, 64, 129, 63), (8, 2, 128, 200, 64), (32, 8, 128, 1792, 0),
                                             (32, 8, 128, 1793, 0), (32, 8, 128, 1024, 700), (32, 8, 128, 1030, 700)])
def test_rows_of_small_tiles(F, ctx, hq, hkv, d, n, past):
    total = past + n
    qb = synth.normal_bf16(700 + n, synth.stream_id(synth.STREAM_Q), (n, hq, d))
    kb = synth.normal_bf16(700 + n, synth.stream_id(synth.STREAM_K), (total, hkv, d))
    vb = synth.normal_bf16(700 + n, synth.stream_id(synth.STREAM_V), (total, hkv, d))
    cache = F.KVCache.empty(1, hkv, total + 5, d)
    F.flux_kv_append(ctx, cache, hkv, d, H.bits_to_torch(kb), H.bits_to_torch(vb), i32([0, total]), total, total)
    q, cu = H.bits_to_torch(qb), i32([0, n])
    window = 50 if n <= 200 else 2000                          # (a window that cuts the prompt moves the bound)
    cfg = F.attn_cfg(hq, hkv, d, 10, window, 0.0, 1)
    out = torch.full((n, hq, d), float("nan"), dtype=torch.float32, device="cuda")
    rows = range(n) if n <= 200 else (0, 15, 16, 63, 64, n // 2, n - 2, n - 1)
    k, v = O.bf16_to_f64(kb), O.bf16_to_f64(vb)
    for mode in (FA, SA):
        F.flux_attn_prefill(ctx, cfg, q, cu, n, total, cache, u8([mode]), out)
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        want = np.stack([O.attention(O.bf16_to_f64(qb[r:r + 1]), k[:past + r + 1], v[:past + r + 1], mode, 10, window)[0] for r in rows])
        H.assert_close(got[list(rows)], want, f"mode {mode}")
        if mode == FA:
            nb = -(-total // 64)
            keep = torch.ones(1, 1, nb, nb, dtype=torch.uint8, device="cuda")
            wide = torch.full_like(out, float("nan"))
            F.flux_attn_prefill_blocksparse(ctx, cfg, q, cu, n, total, cache, u8([SA]), keep, 1, nb, nb, wide)
            torch.cuda.synchronize()
            assert np.array_equal(wide.cpu().numpy(), got)
    assert F.flux_last_device_status(ctx) == 0

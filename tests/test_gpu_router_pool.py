"""flux_router on either side of the pools that one, two and sixteen row splits hold (128 rows each), sequences that end inside a
round of 16 rows, hidden sizes that end inside a workgroup's 128 columns.  Oracle at 1e-6, the router's tolerance (fp32 sums of
bf16 numbers; logits of order 0.1)."""
import numpy as np
import pytest
import torch

from oracle import flux_oracle as O
from paper_2604_07394_amd import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pool", [1, 63, 64, 65, 128, 129, 1024])
@pytest.mark.parametrize("hidden", [128, 136, 1000])
def test_router_pools_of_whole_splits(pool, hidden):
    from paper_2604_07394_amd import binding as F

    inner, lens = 24, [1, 15, 16, 17, max(1, 2 * pool - 1), 2 * pool, 2 * pool + 1, 2 * pool + 300]
    rng = np.random.default_rng(1000 * pool + hidden)
    xb = synth.f32_to_bf16_bits(rng.standard_normal((sum(lens), hidden)).astype(np.float32))
    w1b = synth.f32_to_bf16_bits((rng.standard_normal((inner, hidden)) * 0.02).astype(np.float32))
    w2b = synth.f32_to_bf16_bits((rng.standard_normal((2, inner)) * 0.02).astype(np.float32))
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32, device="cuda")
    mode = torch.full((len(lens),), 9, dtype=torch.uint8, device="cuda")
    logits = torch.full((len(lens), 2), float("nan"), dtype=torch.float32, device="cuda")
    ctx = F.flux_create(0)
    F.flux_router(ctx, H.bits_to_torch(xb), cu, len(lens), hidden, pool, H.bits_to_torch(w1b), None, H.bits_to_torch(w2b), None, inner, mode, logits)
    torch.cuda.synchronize()
    F.flux_destroy(ctx)
    x, w1, w2 = O.bf16_to_f64(xb), O.bf16_to_f64(w1b), O.bf16_to_f64(w2b)
    off = 0
    for b, n in enumerate(lens):
        ref, dec = O.router(x[off:off + n], pool, w1, None, w2, None)
        off += n
        assert np.abs(logits[b].cpu().numpy() - ref).max() < 1e-6, (b, n)
        assert abs(ref[0] - ref[1]) < 1e-6 or int(mode[b]) == dec, (b, n)

"""The LSE merge at the edges of its passes over the slots (4 or 8 at a time)
against the fp64 oracle, with empty slots.  fp32 results within 1e-5 (the fp32
bound of the other tests); bf16 results within half an ulp of their value
(2^-8 relative) on top."""
import numpy as np
import pytest
import torch

import oracle
from tests import _descs
from tests._gpu import HAVE_GPU, api, to64

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not HAVE_GPU, reason="needs a GPU")]


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("part,out_dt", [(torch.float32, torch.float32), (torch.float32, torch.bfloat16),
                                         (torch.bfloat16, torch.bfloat16)])
@pytest.mark.parametrize("slots", [1, 3, 4, 5, 8, 9, 17])
def test_slot_counts(slots, part, out_dt, hd):
    n, H = 37, 3
    d = _descs.desc(cu_q=(0, n), kind=(1,), kv_first=(0,), kv_count=(slots,), cu_k=tuple(range(slots + 1)),
                    block_index=tuple(range(slots))[::-1], num_slots=slots)
    g = torch.Generator().manual_seed(slots * 10 + hd)
    o = torch.randn((slots, n, H, hd), generator=g).to(part)
    lse = 3 * torch.randn((slots, n, H), generator=g)
    lse[torch.rand(lse.shape, generator=g) < 0.2] = -float("inf")   # empty blocks, some rows with none at all
    lse[:, 5] = -float("inf")
    o[torch.isneginf(lse)] = 0
    out = torch.full((n, H, hd), float("nan"), dtype=out_dt, device="cuda")
    got = torch.full((n, H), float("nan"), device="cuda")
    api.lse_merge(api.SegDesc.of(d), o.cuda(), lse.cuda(), out, got)
    for h in range(H):
        ro, rl = oracle.lse_merge(o[:, :, h].double().numpy(), lse[:, :, h].double().numpy())
        gl = to64(got)[:, h]
        assert np.array_equal(np.isneginf(gl), np.isneginf(rl))
        fin = np.isfinite(rl)
        np.testing.assert_allclose(gl[fin], rl[fin], rtol=0, atol=1e-5)
        np.testing.assert_allclose(to64(out)[:, h], ro, rtol=2.0 ** -8 if out_dt == torch.bfloat16 else 0, atol=1e-5)


@pytest.mark.parametrize("part", [torch.float32, torch.bfloat16])
def test_bits_do_not_depend_on_the_launch(part):
    """A shard of 6 slots beside one of 16 (which sets how many partials a pass loads) and by itself."""
    n, H, hd = 37, 3, 128
    g = torch.Generator(device="cuda").manual_seed(86)
    o = torch.randn((16, 2 * n, H, hd), generator=g, device="cuda").to(part)
    lse = 3 * torch.randn((16, 2 * n, H), generator=g, device="cuda")
    two = _descs.desc(cu_q=(0, n, 2 * n), kind=(1, 1), kv_first=(0, 6), kv_count=(6, 16), cu_k=tuple(range(23)),
                      block_index=tuple(range(6)) + tuple(range(16)), num_slots=16)
    one = _descs.desc(cu_q=(0, n), kind=(1,), kv_first=(0,), kv_count=(6,), cu_k=tuple(range(7)),
                      block_index=tuple(range(6)), num_slots=16)
    res = []
    for d, rows in ((two, 2 * n), (one, n)):
        out = torch.empty((rows, H, hd), dtype=torch.float32, device="cuda")
        got = torch.empty((rows, H), device="cuda")
        api.lse_merge(api.SegDesc.of(d), o[:, :rows].contiguous(), lse[:, :rows].contiguous(), out, got)
        res.append((out, got))
    for a, b in zip(*res):
        assert torch.equal(a[:n], b)

"""The fp32 forward at the edges of its tiles (32 query rows, 32-key blocks
dealt to 4 waves: a wave without a block, with one, with two) against the
fp64 oracle.  Tolerance 1e-5 on O and LSE, the fp32 bound of the other tests."""
import pytest
import torch

from tests import _descs
from tests._gpu import HAVE_GPU, api
from tests.test_gpu_parity import run_and_compare

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not HAVE_GPU, reason="needs a GPU")]


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("lq", [1, 31, 32, 33, 64, 65, 97])
def test_tile_edges(lq, hd):
    # one whole segment of lq rows, and a shard of lq rows against blocks around a block and a full deal
    blocks = (1, 32, 33, 127, 128, 129, 160, 255, 256, 257, 289, 513)
    cu_k = [0, lq]
    for n in blocks:
        cu_k.append(cu_k[-1] + n)
    d = _descs.desc(cu_q=(0, lq, 2 * lq), kind=(0, 1), kv_first=(0, 1), kv_count=(1, len(blocks)), cu_k=cu_k,
                    block_index=(0,) + tuple(range(len(blocks))), num_slots=len(blocks))
    run_and_compare(d, 3, hd, torch.float32, 900 + lq + hd, backward=False)


def test_more_tiles_than_the_grid():
    """A launch has at most 2^20 workgroups, further tiles are taken in turn: 33 one-token segments of 16,384
    heads are 540,672 items of two tiles.  With one key, O is V's row and the LSE the scaled score."""
    n, H, hd = 33, 16384, 64
    g = torch.Generator(device="cuda").manual_seed(89)
    q, k, v = (torch.randn((n, H, hd), generator=g, device="cuda") for _ in range(3))
    cu = tuple(range(n + 1))
    d = _descs.desc(cu_q=cu, kind=(0,) * n, kv_first=cu[:-1], kv_count=(1,) * n, cu_k=cu, block_index=(0,) * n, num_slots=0)
    out, lse = torch.full_like(q, float("nan")), torch.full((n, H), float("nan"), device="cuda")
    api.attn_fwd(api.SegDesc.of(d), q, k, v, 0.125, out, lse)
    assert torch.equal(out, v)
    assert (lse - 0.125 * (q.double() * k.double()).sum(-1)).abs().max().item() <= 1e-5


@pytest.mark.parametrize("hd", [64, 128])
def test_bits_do_not_depend_on_the_launch(hd):
    """A segment alone (30 tiles) and among 40 more of its length (1230 tiles): the same bits."""
    n, m, H = 300, 41, 3
    g = torch.Generator(device="cuda").manual_seed(85)
    q, k, v = (torch.randn((n * m, H, hd), generator=g, device="cuda") for _ in range(3))
    res = []
    for s in (m, 1):
        cu = tuple(n * i for i in range(s + 1))
        d = _descs.desc(cu_q=cu, kind=(0,) * s, kv_first=tuple(range(s)), kv_count=(1,) * s, cu_k=cu,
                        block_index=(0,) * s, num_slots=0)
        res.append(api.attn_fwd(api.SegDesc.of(d), q[:n * s], k[:n * s], v[:n * s], hd ** -0.5)[:2])
    for many, one in zip(*res):
        assert torch.equal(many[:n], one)

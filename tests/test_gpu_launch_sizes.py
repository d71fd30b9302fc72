"""Launches of few and of many items (forward and backward) at the edges of
their tiles against the fp64 oracle, and the same segment's results in both: a
launch's size decides how its items are handed out (one round or queues, dK/dV
and dQ in one launch or two, one or two workgroups per compute unit), never how
an item is computed.  Bounds as in the other parity tests."""
import pytest
import torch

from tests import _descs
from tests._gpu import HAVE_GPU
from tests.test_gpu_parity import run_and_compare

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not HAVE_GPU, reason="needs a GPU")]

WHOLE = (1, 31, 33, 64, 65, 127, 128, 129, 255, 257)   # rows = keys: tile, row-group and step edges


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("heads", [1, 9, 40])
def test_tile_edges(heads, hd):
    # the whole segments, then a shard of 130 rows against blocks of 32, 0, 97 and 385 keys
    blocks = (32, 0, 97, 385)
    cu_q, cu_k = [0], [0]
    for n in WHOLE:
        cu_q.append(cu_q[-1] + n)
        cu_k.append(cu_k[-1] + n)
    cu_q.append(cu_q[-1] + 130)
    for n in blocks:
        cu_k.append(cu_k[-1] + n)
    w = len(WHOLE)
    d = _descs.desc(cu_q=cu_q, kind=(0,) * w + (1,), kv_first=tuple(range(w + 1)), kv_count=(1,) * w + (len(blocks),),
                    cu_k=cu_k, block_index=(0,) * w + tuple(range(len(blocks))), num_slots=len(blocks))
    run_and_compare(d, heads, hd, torch.bfloat16, 60 + heads + hd)


@pytest.mark.parametrize("heads", [2, 20, 30, 160])
def test_one_long_segment(heads):
    # one segment: 3 tiles of 256 rows, the last one ragged; several 128-key tiles.  The backward's dK/dV
    # and dQ run in one launch, in a single round (2, 20 and 30 heads), then in rounds.
    d = _descs.desc(cu_q=(0, 523), kind=(0,), kv_first=(0,), kv_count=(1,), cu_k=(0, 523), block_index=(0,), num_slots=0)
    run_and_compare(d, heads, 128, torch.bfloat16, 70 + heads)


def test_scores_jump_across_parts():
    """Keys that beat the running maximum far beyond the fast path's bound, each in another 32-key block."""
    from tests._gpu import api, to64
    import numpy as np
    import oracle
    n, hd = 300, 128
    g = torch.Generator().manual_seed(81)
    q, k, v = (torch.randn((n, 1, hd), generator=g).to(torch.bfloat16) for _ in range(3))
    for i, f in ((10, 8), (40, 16), (75, 32), (110, 64), (200, 96), (290, 128)):
        k[i] *= f
    d = _descs.desc(cu_q=(0, n), kind=(0,), kv_first=(0,), kv_count=(1,), cu_k=(0, n), block_index=(0,), num_slots=0)
    out, lse, _, _ = api.attn_fwd(api.SegDesc.of(d), q.cuda(), k.cuda(), v.cuda(), hd ** -0.5)
    ref = oracle.packed_forward(d, *(t.double().numpy() for t in (q, k, v)), hd ** -0.5)
    assert np.abs(to64(out) - ref["out"]).max() <= 2e-2
    assert np.abs(to64(lse) - ref["lse"]).max() <= 1e-3


def test_profiled_backward_has_the_same_bits():
    """With profiling on, dK/dV and dQ run as two launches: the same items, the same results."""
    from tests._gpu import api
    d = _descs.mixed_small()
    H, hd = 40, 128
    desc = api.SegDesc.of(d)
    g = torch.Generator().manual_seed(82)
    tq, tk = d["cu_seqlens_q"][-1], d["cu_seqlens_k"][-1]
    q, k, v, do = (torch.randn((n, H, hd), generator=g).to(torch.bfloat16).cuda() for n in (tq, tk, tk, tq))
    out, lse, op, lp = api.attn_fwd(desc, q, k, v, hd ** -0.5)
    api.lse_merge(desc, op, lp, out, lse)
    one = api.attn_bwd(desc, q, k, v, out, lse, do, hd ** -0.5)
    api.profile_reset()
    api.profile_enable(True)
    try:
        two = api.attn_bwd(desc, q, k, v, out, lse, do, hd ** -0.5)
    finally:
        api.profile_enable(False)
    assert api.profile_read(api.ZL_K_BWD_DQ)[1] == 1 and api.profile_read(api.ZL_K_BWD_DKDV)[1] == 1
    api.profile_reset()
    for a, b in zip(one, two):
        assert torch.equal(a, b)


@pytest.mark.parametrize("hd", [64, 128])
def test_long_dq_items_first(hd):
    """A shard of few rows against many blocks, in several rounds: its dQ items are the longest, so the
    backward's one launch starts with them."""
    cu_k = (0, 130, 230, 360, 490, 520, 584)
    d = _descs.desc(cu_q=(0, 40, 104), kind=(1, 0), kv_first=(0, 5), kv_count=(5, 1), cu_k=cu_k,
                    block_index=(0, 1, 2, 3, 4, 0), num_slots=5)
    run_and_compare(d, 100, hd, torch.bfloat16, 90 + hd)


def test_two_workgroups_per_cu():
    """d = 64 with more than four rounds of long items (1040 of 1601 keys): the forward runs two
    workgroups per compute unit.  64 rows of every head against the oracle."""
    from tests._gpu import api, to64
    import numpy as np
    import oracle
    n, H, hd = 1601, 149, 64
    g = torch.Generator().manual_seed(83)
    q, k, v = (torch.randn((n, H, hd), generator=g).to(torch.bfloat16) for _ in range(3))
    d = _descs.desc(cu_q=(0, n), kind=(0,), kv_first=(0,), kv_count=(1,), cu_k=(0, n), block_index=(0,), num_slots=0)
    out, lse, _, _ = api.attn_fwd(api.SegDesc.of(d), q.cuda(), k.cuda(), v.cuda(), hd ** -0.5)
    rows = np.concatenate([np.arange(0, 48), np.arange(n - 16, n)])
    out, lse = to64(out), to64(lse)
    for h in range(H):
        o, l = oracle.attend(q[rows, h].double().numpy(), k[:, h].double().numpy(), v[:, h].double().numpy(), hd ** -0.5)
        assert np.abs(out[rows, h] - o).max() <= 2e-2
        assert np.abs(lse[rows, h] - l).max() <= 1e-3


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("n,others", [(448, 12), (300, 40), (1601, 14)])
def test_bits_do_not_depend_on_the_launch(n, others, hd):
    """A segment alone (its items fit one round with compute units to spare) and among `others` more of
    its length (several rounds): the same outputs and gradients, bit for bit."""
    from tests._gpu import api
    H, scale = 12, hd ** -0.5
    g = torch.Generator(device="cuda").manual_seed(84)
    q, k, v, do = (torch.randn((n * (1 + others), H, hd), generator=g, device="cuda").to(torch.bfloat16) for _ in range(4))
    res = []
    for m in (1 + others, 1):
        cu = tuple(n * i for i in range(m + 1))
        desc = api.SegDesc.of(_descs.desc(cu_q=cu, kind=(0,) * m, kv_first=tuple(range(m)), kv_count=(1,) * m, cu_k=cu,
                                          block_index=(0,) * m, num_slots=0))
        t = [x[:n * m] for x in (q, k, v, do)]
        out, lse, _, _ = api.attn_fwd(desc, *t[:3], scale)
        res.append((out, lse) + tuple(api.attn_bwd(desc, *t[:3], out, lse, t[3], scale)))
    for name, many, one in zip(("out", "lse", "dq", "dk", "dv"), *res):
        assert torch.equal(many[:n], one), name


@pytest.mark.parametrize("heads", [3, 40])
def test_dq_in_place_of_q_or_dout(heads):
    """dq written over q or over dout: the gradients of the call with memory of its own, bit for bit."""
    from tests._gpu import api
    n, hd = 1200, 128
    d = _descs.desc(cu_q=(0, n), kind=(0,), kv_first=(0,), kv_count=(1,), cu_k=(0, n), block_index=(0,), num_slots=0)
    desc = api.SegDesc.of(d)
    g = torch.Generator(device="cuda").manual_seed(87)
    q, k, v, do = (torch.randn((n, heads, hd), generator=g, device="cuda").to(torch.bfloat16) for _ in range(4))
    out, lse, _, _ = api.attn_fwd(desc, q, k, v, hd ** -0.5)
    ref = api.attn_bwd(desc, q, k, v, out, lse, do, hd ** -0.5)
    for name in ("q", "dout"):
        for call in ("bwd", "noalloc"):
            a, b = q.clone(), do.clone()
            dq = a if name == "q" else b
            if call == "bwd":
                got = api.attn_bwd(desc, a, k, v, out, lse, b, hd ** -0.5, dq=dq)
            else:
                got = api.attn_bwd_noalloc(desc, a, k, v, out, lse, b, hd ** -0.5, dq, torch.empty_like(k), torch.empty_like(v))
            for t, x, y in zip(("dq", "dk", "dv"), got, ref):
                assert torch.equal(x, y), (name, call, t)

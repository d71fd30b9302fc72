"""Launches of few and of many items (forward and backward) at the edges of
their tiles against the fp64 oracle, and the same segment's results in both: a
launch's size decides how its items are handed out (one round or queues, dK/dV
and dQ in one launch or two, one or two workgroups per compute unit), never how
an item is computed.  Bounds as in the other parity tests."""
import numpy as np
import pytest
import torch

import oracle
from tests import _descs
from tests._gpu import HAVE_GPU, api, to64
from tests._route import DQ_FIRST, HALVES, ONE_LAUNCH, TWO_PER_CU, route
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
    # 1 head: halves throughout, one backward launch; 9: halves, dK/dV and dQ apart; 40: whole tiles in rounds
    assert route(d, heads, hd, api.ZL_OP_FWD) == (HALVES if heads < 40 else 0)
    assert route(d, heads, hd, api.ZL_OP_BWD) & (HALVES | ONE_LAUNCH) == {1: HALVES | ONE_LAUNCH, 9: HALVES, 40: ONE_LAUNCH}[heads]
    run_and_compare(d, heads, hd, torch.bfloat16, 60 + heads + hd)


@pytest.mark.parametrize("heads", [2, 20, 30, 160])
def test_one_long_segment(heads):
    # one segment: 3 tiles of 256 rows, the last one ragged; several 128-key tiles.  The backward's dK/dV
    # and dQ run in one launch, in a single round (2, 20 and 30 heads), then in rounds.
    d = _descs.desc(cu_q=(0, 523), kind=(0,), kv_first=(0,), kv_count=(1,), cu_k=(0, 523), block_index=(0,), num_slots=0)
    run_and_compare(d, heads, 128, torch.bfloat16, 70 + heads)


def test_scores_jump_across_parts():
    """Keys that beat the running maximum far beyond the fast path's bound, each in another 32-key block."""
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


@pytest.mark.parametrize("H", [3, 80])   # one round, and 1040 items in rounds
def test_profiled_backward_has_the_same_bits(H):
    """With profiling on, dK/dV and dQ run as two launches: the same items, the same results."""
    d = _descs.mixed_small()
    hd = 128
    assert route(d, H, hd, api.ZL_OP_BWD) & ONE_LAUNCH
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
    assert route(d, 140, hd, api.ZL_OP_BWD) == ONE_LAUNCH | DQ_FIRST
    run_and_compare(d, 140, hd, torch.bfloat16, 90 + hd)


def test_two_workgroups_per_cu():
    """d = 64 with more than four rounds of long items: the forward runs two workgroups per compute unit.
    Rows of every tile (the last one has 29) and head against the oracle, every row written."""
    n, H, hd = 3101, 80, 64
    g = torch.Generator().manual_seed(83)
    q, k, v = (torch.randn((n, H, hd), generator=g).to(torch.bfloat16) for _ in range(3))
    d = _descs.desc(cu_q=(0, n), kind=(0,), kv_first=(0,), kv_count=(1,), cu_k=(0, n), block_index=(0,), num_slots=0)
    assert route(d, H, hd, api.ZL_OP_FWD) & TWO_PER_CU
    out = torch.full((n, H, hd), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((n, H), float("nan"), device="cuda")
    api.attn_fwd(api.SegDesc.of(d), q.cuda(), k.cuda(), v.cuda(), hd ** -0.5, out, lse)
    assert torch.isfinite(out).all() and torch.isfinite(lse).all()
    rows = np.array([r for t in range(0, n, 256) for r in (t, t + 31, t + 160, t + 255) if r < n] + [n - 1])
    out, lse = to64(out[rows]), to64(lse[rows])
    for h in range(H):
        o, l = oracle.attend(q[rows, h].double().numpy(), k[:, h].double().numpy(), v[:, h].double().numpy(), hd ** -0.5)
        assert np.abs(out[:, h] - o).max() <= 2e-2
        assert np.abs(lse[:, h] - l).max() <= 1e-3


@pytest.mark.parametrize("part", [torch.float32, torch.bfloat16])
def test_two_workgroups_per_cu_shard(part):
    """The same launch with SHARD items (partials, and ring steps): 420 heads against 4 of them by themselves,
    which run one workgroup per compute unit, bit for bit."""
    nq, blocks, H, few, hd = 650, (2600, 2649), 420, 4, 64
    g = torch.Generator(device="cuda").manual_seed(88)
    q, k, v = (torch.randn((m, H, hd), generator=g, device="cuda").to(torch.bfloat16)
               for m in (nq, sum(blocks), sum(blocks)))
    d = _descs.desc(cu_q=(0, nq), kind=(1,), kv_first=(0,), kv_count=(2,), cu_k=(0, blocks[0], sum(blocks)),
                    block_index=(1, 0), num_slots=2)
    step = [_descs.desc(cu_q=(0, nq), kind=(1,), kv_first=(0,), kv_count=(1,), cu_k=(0, b), block_index=(0,), num_slots=1)
            for b in blocks]
    for x in (d, *step):
        assert route(x, H, hd, api.ZL_OP_FWD) & TWO_PER_CU and not route(x, few, hd, api.ZL_OP_FWD) & TWO_PER_CU
    res = []
    for h in (H, few):
        qh, kh, vh = (t[:, :h].contiguous() for t in (q, k, v))
        _, _, o, l = api.attn_fwd(api.SegDesc.of(d), qh, kh, vh, hd ** -0.5, part_dtype=part)
        out, lse = torch.empty_like(qh), torch.empty((nq, h), device="cuda")
        acc = torch.empty((nq, h, hd), device="cuda"), torch.empty((nq, h), device="cuda")
        row = 0
        for i, b in enumerate(blocks):
            api.attn_fwd_step(api.SegDesc.of(step[i]), qh, kh[row:row + b], vh[row:row + b], hd ** -0.5, out, lse, *acc,
                              api.ZL_STEP_FIRST if i == 0 else api.ZL_STEP_LAST)
            row += b
        res.append((o, l, out, lse))
    o, l, out, lse = res[0]
    assert all(torch.isfinite(t).all() for t in res[0])
    for a, b in zip((o[:, :, :few], l[:, :, :few], out[:, :few], lse[:, :few]), res[1]):
        assert torch.equal(a, b)
    for h in (0, few, H - 1):
        ro, rl = oracle.attend(*(t[:, h].double().cpu().numpy() for t in (q, k, v)), hd ** -0.5)
        assert np.abs(to64(out[:, h]) - ro).max() <= 2e-2 and np.abs(to64(lse[:, h]) - rl).max() <= 1e-3


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("n,others", [(448, 12), (300, 40), (1601, 24)])
def test_bits_do_not_depend_on_the_launch(n, others, hd):
    """A segment alone (its items fit one round with compute units to spare) and among `others` more of
    its length (several rounds): the same outputs and gradients, bit for bit."""
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
    """dq written over q or over dout, and each gradient over out: the gradients of the call with memory of its
    own, bit for bit."""
    n, hd = 1200, 128
    d = _descs.desc(cu_q=(0, n), kind=(0,), kv_first=(0,), kv_count=(1,), cu_k=(0, n), block_index=(0,), num_slots=0)
    desc = api.SegDesc.of(d)
    g = torch.Generator(device="cuda").manual_seed(87)
    q, k, v, do = (torch.randn((n, heads, hd), generator=g, device="cuda").to(torch.bfloat16) for _ in range(4))
    out, lse, _, _ = api.attn_fwd(desc, q, k, v, hd ** -0.5)
    ref = api.attn_bwd(desc, q, k, v, out, lse, do, hd ** -0.5)
    for grad, over in (("dq", "q"), ("dq", "dout"), ("dq", "out"), ("dk", "out"), ("dv", "out")):
        for call in (api.attn_bwd, api.attn_bwd_noalloc):
            t = {"q": q.clone(), "dout": do.clone(), "out": out.clone()}
            to = {x: torch.empty_like(q) for x in ("dq", "dk", "dv")}
            to[grad] = t[over]
            got = call(desc, t["q"], k, v, t["out"], lse, t["dout"], hd ** -0.5, **to)
            for name, x, y in zip(("dq", "dk", "dv"), got, ref):
                assert torch.equal(x, y), (grad, over, call.__name__, name)

"""The work that users of this package have it do, as measurable cases.

A case is one pass of one layer's attention work through the public binding
(``paper_2608_01150_amd.api``), as a training or sampling program calls it
for a packed batch.  Shapes follow Wan's token arithmetic as the rest of the
repository uses it: 448 / 1560 / 3600 / 8160 tokens for a 256p / 480p / 720p /
1080p image, 32,760 for an 81-frame 480p video, 75,600 for a 720p one; 12
heads (Wan2.1-1.3B) or 40 (Wan2.1-14B) of 128.

Kinds of pass (``kind``):
  forward   attn_fwd of WHOLE segments (sampling, or a validation run in fp32)
  train     attn_fwd, lse_merge when a shard is there, attn_bwd
  ring      a shard's blocks arrive one per ring step: attn_fwd_step for each,
            then attn_bwd_step for each; the images ride along in the first
  gather    a shard against its gathered K/V: attn_fwd_step (first and last),
            then attn_bwd_noalloc into the caller's gradients
  merge     lse_merge of partials that are there already
  ulysses   the four staging calls around the two all-to-alls of one layer
"""
from __future__ import annotations

import math

import torch

from paper_2608_01150_amd import api

WHOLE, SHARD = 0, 1


def _case(name, kind, heads=12, dim=128, dtype="bf16", shard=0, blocks=0, block_len=0, wholes="", part="fp32",
          amp=1, group=0):
    """shard: query rows of the one SHARD segment (0: none) against `blocks`
    K/V blocks of block_len rows; wholes: lengths of the WHOLE segments as
    "LxN" terms joined by "+"; part: dtype of the shard's partials; amp: Q and
    K of the first WHOLE segment are multiplied by it; group: Ulysses ranks."""
    c = {"kind": kind, "heads": heads, "dim": dim, "dtype": dtype, "shard": shard, "blocks": blocks,
         "block_len": block_len, "wholes": wholes, "part": part, "amp": amp, "group": group}
    return c if name is None else {"name": name, **c}


def listed():
    return [
        # Sampling or evaluating one 256p image: the smallest call a model layer makes.
        _case("image256p-fwd", "forward", wholes="448x1"),
        # One 480p image on a GPU, forward and backward: a small training step.
        _case("image480p-train", "train", wholes="1560x1"),
        # The image-only batch: sixteen 480p images in one launch.
        _case("images16-train", "train", wholes="1560x16"),
        # The mixed image-video batch of the benchmark (its video's Q and K are x4).
        _case("mixed-video-train", "train", heads=40, wholes="32760x1+3600x2+1560x8", amp=4),
        # One GPU's share of a 720p video at CP=8 with six image fillers, in one coalesced launch.
        _case("shard720p-cp8-train", "train", heads=40, shard=9450, blocks=8, block_len=9450, wholes="1560x6"),
        # One GPU's share of a 480p video at CP=8, partials kept in bf16: few rows, many blocks.
        _case("shard480p-cp8-bf16part-train", "train", shard=4095, blocks=8, block_len=4095, wholes="1560x4",
              part="bf16"),
        # A 480p video at CP=4 whose blocks travel round a ring.
        _case("ring480p-cp4-train", "ring", shard=8190, blocks=4, block_len=8190, wholes="1560x2"),
        # The same video at CP=8 with gathered K/V, and the backward that allocates nothing.
        _case("gather480p-cp8-train", "gather", shard=4095, blocks=1, block_len=32760, wholes="1560x2"),
        # Merging a 720p shard's eight partials into the exact output.
        _case("merge720p-cp8", "merge", heads=40, shard=9450, blocks=8, block_len=9450),
        # Staging of the mixed batch for a Ulysses group of eight.
        _case("ulysses8-mixed", "ulysses", heads=40, wholes="32760x1+3600x2+1560x8", group=8),
        # Head dimension 64, the other one the library takes, with lengths that fit no tile.
        _case("dim64-ragged-train", "train", heads=24, dim=64, wholes="4173x1+1021x6"),
        # A 480p image in fp32, as a validation run against the bf16 path does it.
        _case("image480p-fp32-fwd", "forward", dtype="fp32", wholes="1560x1"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    most = {key: max(work(c)[key] for c in listed()) for key in ("bytes", "flops")}
    while True:
        c = _draw(rng)
        if all(work(c)[key] <= most[key] for key in most):
            return c


def _draw(rng):
    kind = rng.choice(["forward", "forward32", "train", "train", "train64", "shard", "shard16", "ring", "gather",
                       "merge", "ulysses"])
    heads = rng.choice([12, 40])
    if kind == "forward":
        return _case(None, "forward", heads=heads, wholes="%dx%d" % (_log(rng, 100, 8160), rng.randint(1, 4)))
    if kind == "forward32":
        return _case(None, "forward", heads=rng.choice([2, 12]), dim=rng.choice([64, 128]), dtype="fp32",
                     wholes="%dx%d" % (_log(rng, 64, 2000), rng.randint(1, 3)))
    if kind in ("train", "train64"):
        n = _log(rng, 1, 16)
        w = "%dx%d" % (_log(rng, 200, 3600), n)
        if rng.random() < 0.5:
            w = "%dx1+" % _log(rng, 3600, 32760) + w
        if kind == "train64":
            return _case(None, "train", heads=rng.choice([12, 24]), dim=64, wholes=w)
        return _case(None, "train", heads=heads, wholes=w, amp=rng.choice([1, 4]))
    lq, nb = _log(rng, 1000, 9450), rng.choice([2, 4, 8])
    w = "%dx%d" % (_log(rng, 200, 3600), rng.randint(1, 6))
    if kind in ("shard", "shard16"):
        return _case(None, "train", heads=heads, shard=lq, blocks=nb, block_len=lq + rng.randint(0, 40), wholes=w,
                     part="bf16" if kind == "shard16" else "fp32")
    if kind == "ring":
        return _case(None, "ring", shard=lq, blocks=rng.choice([2, 4]), block_len=lq + rng.randint(0, 40), wholes=w)
    if kind == "gather":
        return _case(None, "gather", shard=lq, blocks=1, block_len=lq * nb + rng.randint(0, 40), wholes=w)
    if kind == "merge":
        return _case(None, "merge", heads=heads, dim=rng.choice([64, 128]), shard=lq, blocks=rng.choice([2, 3, 8, 16]),
                     block_len=lq, part=rng.choice(["fp32", "bf16"]))
    return _case(None, "ulysses", heads=heads, dim=rng.choice([64, 128]), group=rng.choice([2, 4]),
                 wholes="%dx1+%dx%d" % (_log(rng, 2000, 32760), _log(rng, 200, 3600), rng.randint(1, 8)))


def _wholes(case):
    out = []
    for term in case["wholes"].split("+"):
        if term:
            length, n = term.split("x")
            out += [int(length)] * int(n)
    return out


def _segments(case):
    """[(kind, query rows, [K/V range lengths])], the shard first."""
    segs = [(SHARD, case["shard"], [case["block_len"]] * case["blocks"])] if case["shard"] else []
    return segs + [(WHOLE, n, [n]) for n in _wholes(case)]


def _desc(segs):
    cu_q, cu_k, kind, first, count, index = [0], [0], [], [], [], []
    slots = 0
    for k, lq, ranges in segs:
        kind.append(k)
        cu_q.append(cu_q[-1] + lq)
        first.append(len(cu_k) - 1)
        count.append(len(ranges))
        for b, lk in enumerate(ranges):
            cu_k.append(cu_k[-1] + lk)
            index.append(b if k == SHARD else 0)
        if k == SHARD:
            slots = max(slots, len(ranges))
    return api.SegDesc(cu_q, kind, first, count, cu_k, index, slots)


def _dtype(name):
    return torch.bfloat16 if name == "bf16" else torch.float32


def _randn(gen, dtype, *shape):
    return torch.randn(shape, generator=gen, dtype=torch.float32, device="cuda").to(dtype)


def _ulysses_rows(case):
    """cu_rank [group][n + 1]: each sequence split over the group in shards that differ by at most one row."""
    g = case["group"]
    cu = [[0] for _ in range(g)]
    for n in _wholes(case):
        for j in range(g):
            cu[j].append(cu[j][-1] + n * (j + 1) // g - n * j // g)
    return cu


def _ring_parts(case):
    """Per ring step: its segments (the images ride along in step 0)."""
    wholes = [(WHOLE, n, [n]) for n in _wholes(case)]
    return [[(SHARD, case["shard"], [case["block_len"]])] + (wholes if b == 0 else [])
            for b in range(case["blocks"])]


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    h, d, dt = case["heads"], case["dim"], _dtype(case["dtype"])
    s = {"case": case, "scale": 1.0 / math.sqrt(d)}
    if case["kind"] == "ulysses":
        cu = _ulysses_rows(case)
        t_loc, t_full, hl = cu[0][-1], sum(c[-1] for c in cu), h // case["group"]
        s.update(cu=cu, q=_randn(gen, dt, t_loc, h, d), k=_randn(gen, dt, t_loc, h, d), v=_randn(gen, dt, t_loc, h, d),
                 recv=_randn(gen, dt, t_full, hl, 3, d), full=_randn(gen, dt, t_full, hl, d),
                 back=_randn(gen, dt, case["group"], t_loc, hl, d))
        return s
    segs = _segments(case)
    tq, tk = sum(x[1] for x in segs), sum(sum(x[2]) for x in segs)
    s["desc"] = _desc(segs)
    if case["kind"] == "merge":
        s.update(o_part=_randn(gen, _dtype(case["part"]), case["blocks"], tq, h, d),
                 # LSEs of blocks of equal length differ by a few tenths; some rows more
                 lse_part=math.log(case["block_len"]) + _randn(gen, torch.float32, case["blocks"], tq, h),
                 out=torch.empty((tq, h, d), dtype=dt, device="cuda"), lse=torch.empty((tq, h), device="cuda"))
        return s
    q, k, v = _randn(gen, dt, tq, h, d), _randn(gen, dt, tk, h, d), _randn(gen, dt, tk, h, d)
    if case["amp"] != 1:
        first = _wholes(case)[0]
        q0, k0 = case["shard"], case["blocks"] * case["block_len"]
        q[q0:q0 + first] *= case["amp"]
        k[k0:k0 + first] *= case["amp"]
    s.update(q=q, k=k, v=v)
    if case["kind"] == "forward":
        return s
    s["do"] = _randn(gen, dt, tq, h, d)
    if case["kind"] == "train":
        return s
    out, lse = torch.empty_like(q), torch.empty((tq, h), device="cuda")
    dq = torch.empty_like(q)
    s.update(out=out, lse=lse, dq=dq)
    if case["kind"] == "gather":
        s.update(dk=torch.empty_like(k), dv=torch.empty_like(v))
        return s
    # ring: each step's K/V is a tensor of its own, as it arrives
    n, bl = case["shard"], case["block_len"]
    s["acc"] = (torch.empty((n, h, d), device="cuda"), torch.empty((n, h), device="cuda"),
                torch.empty((n, h, d), device="cuda"))
    s["steps"] = []
    last = case["blocks"] - 1
    for b, segs in enumerate(_ring_parts(case)):
        rows = tq if b == 0 else n
        kb, vb = (torch.cat([t[b * bl:(b + 1) * bl], t[case["blocks"] * bl:]]) if b == 0
                  else t[b * bl:(b + 1) * bl].clone() for t in (k, v))
        s["steps"].append((_desc(segs), rows, kb, vb, torch.empty_like(kb), torch.empty_like(vb),
                           (api.ZL_STEP_FIRST if b == 0 else 0) | (api.ZL_STEP_LAST if b == last else 0)))
    return s


def run(s):
    case, scale = s["case"], s["scale"]
    kind = case["kind"]
    if kind == "ulysses":
        g, h = case["group"], case["heads"]
        send = api.ulysses_pack_qkv(g, s["q"], s["k"], s["v"])
        q, k, v = api.ulysses_unpack_qkv(g, s["cu"], s["recv"], h)
        osend = api.ulysses_pack_out(g, s["cu"], s["full"], h)
        local = api.ulysses_unpack_out(g, s["back"], h)
        return {"send": send, "q": q, "k": k, "v": v, "osend": osend, "local": local}
    if kind == "merge":
        api.lse_merge(s["desc"], s["o_part"], s["lse_part"], s["out"], s["lse"])
        return {"out": s["out"], "lse": s["lse"]}
    if kind == "forward":
        out, lse, _, _ = api.attn_fwd(s["desc"], s["q"], s["k"], s["v"], scale)
        return {"out": out, "lse": lse}
    if kind == "train":
        desc, q, k, v = s["desc"], s["q"], s["k"], s["v"]
        out, lse, o_part, lse_part = api.attn_fwd(desc, q, k, v, scale, part_dtype=_dtype(case["part"]))
        if case["shard"]:
            api.lse_merge(desc, o_part, lse_part, out, lse)
        dq, dk, dv = api.attn_bwd(desc, q, k, v, out, lse, s["do"], scale)
        return {"out": out, "lse": lse, "dq": dq, "dk": dk, "dv": dv}
    q, do, out, lse, dq = s["q"], s["do"], s["out"], s["lse"], s["dq"]
    if kind == "gather":
        both = api.ZL_STEP_FIRST | api.ZL_STEP_LAST
        api.attn_fwd_step(s["desc"], q, s["k"], s["v"], scale, out, lse, None, None, both)
        api.attn_bwd_noalloc(s["desc"], q, s["k"], s["v"], out, lse, do, scale, dq, s["dk"], s["dv"])
        return {"out": out, "lse": lse, "dq": dq, "dk": s["dk"], "dv": s["dv"]}
    o_acc, lse_acc, dq_acc = s["acc"]
    for desc, n, k, v, _, _, flags in s["steps"]:
        api.attn_fwd_step(desc, q[:n], k, v, scale, out[:n], lse[:n], o_acc, lse_acc, flags)
    for desc, n, k, v, dk, dv, flags in s["steps"]:
        api.attn_bwd_step(desc, q[:n], k, v, out[:n], lse[:n], do[:n], scale, dq[:n], dk, dv, dq_acc, flags)
    return {"out": out, "lse": lse, "dq": dq, "dk": [x[4] for x in s["steps"]], "dv": [x[5] for x in s["steps"]]}


def work(case):
    h, d = case["heads"], case["dim"]
    e = 2 if case["dtype"] == "bf16" else 4
    if case["kind"] == "ulysses":
        cu = _ulysses_rows(case)
        t_loc, t_full = cu[0][-1], sum(c[-1] for c in cu)
        # each of the four calls reads and writes its rows once
        return {"bytes": 2 * e * d * (3 * t_loc * h + 4 * t_full * (h // case["group"]) + t_loc * h), "flops": 0}
    segs = _segments(case)
    tq, tk = sum(x[1] for x in segs), sum(sum(x[2]) for x in segs)
    if case["kind"] == "merge":
        pe = 2 if case["part"] == "bf16" else 4
        return {"bytes": tq * h * (case["blocks"] * (d * pe + 4) + d * e + 4), "flops": 0}
    pairs = sum(lq * sum(ranges) for _, lq, ranges in segs)
    qb, kb, lb = tq * h * d * e, tk * h * d * e, tq * h * 4
    if case["kind"] == "forward":
        return {"bytes": 2 * qb + 2 * kb + lb, "flops": 4 * d * h * pairs}
    # forward S, PV; backward S again, dP, dV, dK, dQ: 14 d per pair
    return {"bytes": 2 * qb + 2 * kb + lb + 4 * qb + 4 * kb + lb, "flops": 14 * d * h * pairs}


def tolerance(case):
    if case["kind"] == "ulysses":
        return "exact"
    if case["dtype"] == "fp32":
        return {"rel": 1e-5}
    return {"rel": 1e-2}


def _attend(q, k, v, scale, do=None):
    """One head of one segment in fp64, in blocks of rows: (out, lse) and, with do, (dq, dk, dv)."""
    o, ls = torch.empty_like(q), torch.empty(q.shape[0], dtype=q.dtype, device=q.device)
    kt = k.t().contiguous()
    if do is not None:
        dq, dk, dv, vt = torch.empty_like(q), torch.zeros_like(k), torch.zeros_like(v), v.t().contiguous()
    step = max(256, min(8192, (1 << 27) // max(1, k.shape[0])))
    for a in range(0, q.shape[0], step):
        qa = q[a:a + step]
        s = (qa @ kt).mul_(scale)
        l = torch.logsumexp(s, 1)
        p = s.sub_(l[:, None]).exp_()
        o[a:a + step], ls[a:a + step] = p @ v, l
        if do is not None:
            da = do[a:a + step]
            dv += p.t().contiguous() @ da
            ds = (da @ vt).sub_((da * o[a:a + step]).sum(1, keepdim=True)).mul_(p).mul_(scale)
            dq[a:a + step] = ds @ k
            dk += ds.t().contiguous() @ qa
    return (o, ls) if do is None else (o, ls, dq, dk, dv)


def exact(case, seed):
    if case["kind"] == "ulysses":  # copies: compared bit for bit
        return None
    s = prepare(case, seed)
    if case["kind"] == "merge":
        lp = s["lse_part"].double()
        lse = torch.logsumexp(lp, 0)
        out = torch.zeros(s["out"].shape, dtype=torch.float64, device="cuda")
        for b in range(case["blocks"]):
            out += torch.exp(lp[b] - lse)[..., None] * s["o_part"][b].double()
        return {"out": out, "lse": lse}
    q, k, v, do = s["q"], s["k"], s["v"], s.get("do")
    bwd = do is not None
    f64 = lambda t: torch.empty(t.shape, dtype=torch.float64, device="cuda")  # noqa: E731
    out, lse = f64(q), torch.empty(q.shape[:2], dtype=torch.float64, device="cuda")
    dq, dk, dv = (f64(q), f64(k), f64(v)) if bwd else (None, None, None)
    a = b = 0
    for _, lq, ranges in _segments(case):
        lk = sum(ranges)
        for h in range(case["heads"]):
            one = lambda t, i, n: t[i:i + n, h].double().contiguous()  # noqa: E731
            r = _attend(one(q, a, lq), one(k, b, lk), one(v, b, lk), s["scale"], one(do, a, lq) if bwd else None)
            out[a:a + lq, h], lse[a:a + lq, h] = r[0], r[1]
            if bwd:
                dq[a:a + lq, h], dk[b:b + lk, h], dv[b:b + lk, h] = r[2:]
        a, b = a + lq, b + lk
    if not bwd:
        return {"out": out, "lse": lse}
    if case["kind"] == "ring":
        n, bl = case["blocks"], case["block_len"]
        parts = lambda t: [torch.cat([t[:bl], t[n * bl:]])] + [t[i * bl:(i + 1) * bl] for i in range(1, n)]  # noqa: E731
        dk, dv = parts(dk), parts(dv)
    return {"out": out, "lse": lse, "dq": dq, "dk": dk, "dv": dv}

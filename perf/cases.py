"""The work a program has this library do, as timed cases: decode steps over
contiguous and paged caches, prompts, and the baselines they are compared
with, at the shapes of gva_inputs.WORKLOADS and generic ones around them.

Each case goes through the calls such a program makes: it lays out caches,
plan, workspace and marshalled calls once (prepare), then makes one pass
(run).  A decode step appends the current token's row and attends in
gva_decode_step; a prompt (or a chunk of one) appends its rows with
gva_append_kv and attends with gva.prefill.

Values, queries and positional keys are N(0, 1) and the maps N(0, 1/d_v), as
in gva_inputs.  Ragged lengths are fixed quantiles of their distribution,
dealt to the sequences in an order of the seed's, so every seed has the same
work.
"""

import math

import torch

from paper_2609_13285_amd import gva

_DT = {"bf16": torch.bfloat16, "f32": torch.float32}


def _case(name, kind, dtype="bf16", *, batch, t_max, heads, groups, d_v, d_c=None, d_r=16, lens="full",
          len_min=0, n_new=0, page_rows=0):
    c = {"kind": kind, "dtype": dtype, "batch": batch, "t_max": t_max, "heads": heads, "groups": groups,
         "d_v": d_v, "d_c": d_v if d_c is None else d_c, "d_r": d_r, "lens": lens, "len_min": len_min,
         "n_new": n_new, "page_rows": page_rows}
    return dict(c, name=name) if name else c


def listed():
    return [
        # One sequence of 256 rows in fp32: the smallest call, as when a
        # program is brought up or checked in fp32.
        _case("step_tiny_f32", "step", "f32", batch=1, t_max=256, heads=8, groups=2, d_v=64),
        # fp32 storage for a small batch of mid-length sequences (350M head
        # shapes, lengths from half to all of 4096 rows).
        _case("step_f32_b8_t4k", "step", "f32", batch=8, t_max=4096, heads=16, groups=4, d_v=64, lens="half"),
        # The 350M model's decode step: eight sequences of 2048 rows.
        _case("step_350m_b8_t2k", "step", batch=8, t_max=2048, heads=16, groups=4, d_v=64),
        # A large serving batch at full context: the bandwidth workload.
        _case("step_b32_t8k", "step", batch=32, t_max=8192, heads=32, groups=8, d_v=128),
        # A few very long contexts (64K to 128K rows).
        _case("step_long_b4_t128k", "step", batch=4, t_max=131072, heads=32, groups=8, d_v=128, d_r=32,
              lens="half"),
        # A mixed serving batch: 128 to 32K rows, eight heads per value group.
        _case("step_ragged_b64_t32k", "step", batch=64, t_max=32768, heads=16, groups=2, d_v=128, lens="log",
              len_min=128),
        # A paged serving batch of unequal lengths, pages of 64 rows.
        _case("paged_b48_t8k", "paged", batch=48, t_max=8192, heads=32, groups=8, d_v=128, lens="log",
              len_min=256, page_rows=64),
        # One long prompt from empty caches.
        _case("prompt_8k", "prompt", batch=1, t_max=8192, heads=32, groups=8, d_v=128, n_new=8192),
        # A chunk of a prompt per sequence after 4.6K and 6.7K cached rows,
        # the wider positional slice.
        _case("prompt_chunk_500", "prompt", batch=2, t_max=8192, heads=32, groups=8, d_v=128, d_r=24, lens="half",
              n_new=500),
        # Four 2048-token prompts at the 350M head shapes.
        _case("prompt_350m_b4_t2k", "prompt", batch=4, t_max=2048, heads=16, groups=4, d_v=64, n_new=2048),
        # The matched grouped-query prompt that GVA is compared with.
        _case("gqa_prompt_4k", "gqa_prompt", batch=1, t_max=4096, heads=32, groups=8, d_v=128, d_r=0, n_new=4096),
        # The ordinary-RoPE contrast: keys reconstructed at every step.
        _case("rope_b8_t8k", "rope", batch=8, t_max=8192, heads=32, groups=8, d_v=128, d_r=0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "f32", "f32", "paged", "prompt", "prompt", "prompt", "gqa_prompt",
                       "rope"])
    groups = rng.choice([1, 2, 4, 8])
    hpg = rng.choice([1, 2, 4, 4, 8])
    d_v = rng.choice([64, 128])
    d_r = rng.choice([0, 8, 16, 16, 24, 32, 64])
    shape = dict(heads=groups * hpg, groups=groups, d_v=d_v, d_r=d_r)
    if kind == "f32":
        # up to 64 MB of cached rows
        batch = _log_int(rng, 1, 16)
        t = _log_int(rng, 64, min(8192, max(64, (64 << 20) // (batch * groups * d_v * 4))))
        return _case(None, "step", "f32", batch=batch, t_max=(t + 15) // 16 * 16,
                     lens=rng.choice(["full", "half", "log"]), len_min=min(t, 33), **shape)
    if kind in ("step", "paged"):
        # up to 512 MB of cached rows
        batch = _log_int(rng, 1, 64)
        t = _log_int(rng, 128, min(131072, max(128, (512 << 20) // (batch * groups * d_v * 2))))
        page = rng.choice([32, 64, 256]) if kind == "paged" else 16
        page = 32 if t < 256 and kind == "paged" else page
        t = (t + page - 1) // page * page
        if kind == "paged" and t // page > gva.GVA_MAX_PAGES:
            t = page * gva.GVA_MAX_PAGES
        d_c = rng.choice([d_v, d_v, 64, 128])
        return _case(None, kind, batch=batch, t_max=t, d_c=d_c, lens=rng.choice(["full", "half", "log"]),
                     len_min=min(t, 65), page_rows=page if kind == "paged" else 0, **shape)
    if kind == "rope":
        hpg = rng.choice([1, 2, 4] if d_v == 128 else [1, 2, 4, 8])
        batch = _log_int(rng, 1, 16)
        t = _log_int(rng, 128, 65536 // batch)
        return _case(None, kind, batch=batch, t_max=(t + 15) // 16 * 16, heads=groups * hpg, groups=groups, d_v=d_v,
                     d_r=0, lens=rng.choice(["full", "half"]))
    # prompts: new rows after a prefix, within the work of one 8192-token
    # prompt of 32 heads (a 4096-token one for the baseline, half of it)
    top = 4096 if kind == "gqa_prompt" else 8192
    n = _log_int(rng, 48, top)
    prefix = rng.choice([0, 0, _log_int(rng, 1, 8192)])
    batch = rng.randint(1, 4)
    heads = groups * hpg
    while batch > 1 and batch * n * (n / 2 + prefix) * heads > 32 * top * top / 2:
        batch -= 1
    if batch * n * (n / 2 + prefix) * heads > 32 * top * top / 2:
        prefix = 0
        hpg = min(hpg, max(1, 32 // groups))
    if kind == "gqa_prompt":
        d_r = 0
    return _case(None, kind, batch=batch, t_max=(n + prefix + 15) // 16 * 16, heads=groups * hpg, groups=groups,
                 d_v=d_v, d_r=d_r, lens="half" if prefix >= n else "full", n_new=n)


def _lengths(c):
    """The case's lengths, shortest first."""
    B, T = c["batch"], c["t_max"]
    if c["lens"] == "full":
        return [T if c["n_new"] == 0 else max(c["n_new"], T - 5)] * B
    if c["lens"] == "half":          # quantiles of U[T/2, T]
        return [max(c["n_new"], min(T, round(T * (0.5 + (i + 0.5) / (2 * B))))) for i in range(B)]
    lo, hi = math.log(max(1, c["len_min"])), math.log(T)       # quantiles of the log-uniform distribution
    return [max(1, min(T, round(math.exp(lo + (i + 0.5) / B * (hi - lo))))) for i in range(B)]


def _inputs(c, seed):
    """Every tensor of one pass, row-major, on the GPU."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    dt = _DT[c["dtype"]]
    B, T, H, G, N = c["batch"], c["t_max"], c["heads"], c["groups"], c["n_new"]
    dv, dc, dr = c["d_v"], c["d_c"], c["d_r"]

    def normal(*shape, std=1.0, dtype=dt):
        x = torch.randn(shape, generator=g, dtype=torch.float32, device="cuda")
        return (x if std == 1.0 else x.mul_(std)).to(dtype)

    lens = torch.tensor(_lengths(c), dtype=torch.int32, device="cuda")
    x = {"lens": lens[torch.randperm(B, generator=g, device="cuda")].contiguous()}
    x["v"] = normal(B, G, T, dv)
    x["kr"] = normal(B, T, dr)
    if c["kind"] == "gqa_prompt":
        x["k"] = normal(B, G, T, dv)
        x["q"] = normal(B, N, H, dv, dtype=torch.float32)
        return x
    x["m"] = normal(H, dv, dc, std=1.0 / math.sqrt(dv))
    if c["kind"] == "prompt":
        x["q"] = normal(B, N, H, dc + dr)
        x["v_new"] = normal(B * N, G, dv)
        x["kr_new"] = normal(B * N, dr)
    else:
        x["q"] = normal(B, H, dc + dr)
        x["v_new"] = normal(B, G, dv)
        x["kr_new"] = normal(B, dr)
    return x


def _dims(c):
    return gva.make_dims(c["batch"], c["heads"], c["groups"], c["d_v"], c["d_c"], c["d_r"], c["t_max"], c["dtype"])


def prepare(case, seed):
    c, d, x = case, _dims(case), _inputs(case, seed)
    B, H, N, dv = c["batch"], c["heads"], c["n_new"], c["d_v"]
    f32 = dict(dtype=torch.float32, device="cuda")
    s = {"kind": c["kind"], "dims": d, "q": x["q"], "lens": x["lens"]}
    v, kr = gva.tiled(x["v"]), gva.tiled(x["kr"]) if c["d_r"] else x["kr"]
    if c["kind"] == "prompt":
        # the prompt's rows sit behind each sequence's cached prefix
        s.update(m=x["m"], v=v, kr=kr, v_new=x["v_new"], kr_new=x["kr_new"],
                 seq=torch.arange(B, dtype=torch.int32, device="cuda").repeat_interleave(N).contiguous(),
                 pos=(x["lens"].unsqueeze(1) - N + torch.arange(N, dtype=torch.int32, device="cuda")).reshape(-1)
                 .to(torch.int32).contiguous())
        return s
    if c["kind"] == "gqa_prompt":
        s.update(v=v, k=gva.tiled(x["k"]), o=torch.empty(B, N, H, dv, **f32), lse=torch.empty(B, N, H, **f32))
        return s
    # a decode loop marshals its calls once and re-issues them
    S, rows = gva.plan_for(d, x["lens"])
    kr_new = x["kr_new"] if c["d_r"] else None
    if c["kind"] == "step":
        o, lse = torch.empty(B, H, dv, **f32), torch.empty(B, H, **f32)
        ws = gva.workspace_for(d, S, rows)
        s["calls"] = [gva.prepare(gva.gva_decode_step, d, x["q"], x["m"], v, kr, x["lens"], S, o, lse, workspace=ws,
                                  v_new=x["v_new"], kr_new=kr_new, split_rows=rows)]
        s.update(out={"o": o, "lse": lse, "v": v, "kr": kr}, keep=(x, ws))
        return s
    bufs = gva.DecodeBuffers(d, S)
    s["out"] = {"o": bufs.o if S > 1 else bufs.o_part.view(B, H, dv),
                "lse": bufs.lse if S > 1 else bufs.lse_part.view(B, H)}
    s["keep"] = [x, bufs, v, kr]
    if c["kind"] == "paged":
        # pages of the pool in a random order
        mp = c["t_max"] // c["page_rows"]
        pg = gva.make_paging(d, c["page_rows"], B * mp)
        gen = torch.Generator(device="cuda")
        gen.manual_seed(int(seed) + 1)
        table = torch.randperm(B * mp, generator=gen, device="cuda").to(torch.int32).reshape(B, mp).contiguous()
        vp, kp = gva.to_pages(v, kr, table, pg)
        fused = gva.gva_prefer_fused(d, S, rows)
        query = dict(q=x["q"], m=x["m"])
        calls = []
        if not fused:
            qa, qr = torch.empty(B, H, dv, **f32), torch.empty(B, H, c["d_r"], **f32)
            calls.append(gva.prepare(gva.gva_absorb_query, d, x["q"], x["m"], x["lens"], qa, qr))
            query = dict(q_abs=qa, q_rot=qr if c["d_r"] else None)
        calls.append(gva.prepare(gva.gva_paged_decode_attention, d, pg, vp, kp, table, x["lens"], S, bufs.o_part,
                                 bufs.lse_part, v_new=x["v_new"], kr_new=kr_new, split_rows=rows, **query))
        s["out"].update(v=vp, kr=kp)
        s["keep"] += [table, query]
    else:
        calls = [gva.prepare(gva.gva_rope_decode_attention, d, x["q"], x["m"], v, x["lens"], S, bufs.o_part,
                             bufs.lse_part, split_rows=rows)]
    if S > 1:
        calls.append(gva.prepare(gva.gva_combine, d, bufs.o_part, bufs.lse_part, S, bufs.o, bufs.lse))
    s["calls"] = calls
    return s


def run(state):
    s = state
    if s["kind"] == "prompt":
        gva.gva_append_kv(s["dims"], s["v"], s["kr"], s["v_new"], s["kr_new"], s["seq"], s["pos"])
        o, lse = gva.prefill(s["dims"], s["q"], s["m"], s["v"], s["kr"], s["lens"])
        return {"o": o, "lse": lse, "v": s["v"], "kr": s["kr"]}
    if s["kind"] == "gqa_prompt":
        gva.gva_gqa_prefill_attention(s["dims"], s["q"].shape[1], s["q"], s["k"], s["v"], s["lens"], s["o"], s["lse"])
        return {"o": s["o"], "lse": s["lse"]}
    for call in s["calls"]:
        call()
    return s["out"]


def _pairs(c):
    """(query, visible row) pairs of one head."""
    L, n = _lengths(c), max(1, c["n_new"])
    return sum(n * (x - n) + n * (n + 1) // 2 for x in L)


def work(case):
    c = case
    e = 2 if c["dtype"] == "bf16" else 4
    B, H, G, n = c["batch"], c["heads"], c["groups"], max(1, c["n_new"])
    dv, dc, dr = c["d_v"], c["d_c"], c["d_r"]
    rows = sum(_lengths(c))
    out = B * n * H * (dv + 1) * 4
    pairs = _pairs(c) * H
    if c["kind"] == "gqa_prompt":
        return {"bytes": rows * 2 * G * dv * e + B * n * H * dv * 4 + out, "flops": 4 * dv * pairs}
    read = rows * (G * dv + dr) * e + H * dv * dc * e + B * n * H * (dc + dr) * e
    if c["kind"] == "rope":
        return {"bytes": read + out, "flops": 2 * (dv * dc + dc + dv) * pairs}
    new = 2 * B * n * (G * dv + dr) * e                # the new rows: read, and stored in the caches
    return {"bytes": read + new + out, "flops": 2 * (2 * dv + dr) * pairs + 2 * B * n * H * dv * dc}


def tolerance(case):
    # About four times what each path measured off a 64-bit evaluation (rel):
    # fp32 steps 1.8e-7 to 3e-7; bf16 steps, whose queries and weights are
    # bf16 high + low pairs, 2.5e-6 to 2.8e-6; prompts, with fp16 weights,
    # 5e-5 to 1.3e-4 (the baseline 1.7e-4); the contrast path, whose
    # query-map product is rounded to bf16, 1.7e-3.
    return {"prompt": {"rel": 6e-4}, "gqa_prompt": {"rel": 7e-4}, "rope": {"rel": 7e-3}}.get(
        case["kind"], {"rel": 1.2e-5} if case["dtype"] == "bf16" else {"rel": 1.5e-6})


def _rotate(x, pos, base=10000.0):
    """x [..., D] rotated in interleaved pairs at positions pos [...]."""
    D = x.shape[-1]
    if D == 0:
        return x
    theta = base ** (-torch.arange(0, D, 2, dtype=torch.float64, device=x.device) / D)
    a = pos.double().unsqueeze(-1) * theta
    x0, x1 = x[..., 0::2], x[..., 1::2]
    return torch.stack((x0 * a.cos() - x1 * a.sin(), x0 * a.sin() + x1 * a.cos()), -1).flatten(-2)


def exact(case, seed):
    c, x = case, _inputs(case, seed)
    B, H, G, n = c["batch"], c["heads"], c["groups"], max(1, c["n_new"])
    dv, dc, dr, hpg = c["d_v"], c["d_c"], c["d_r"], c["heads"] // c["groups"]
    dt = _DT[c["dtype"]]
    lens = x["lens"].tolist()
    o = torch.zeros(B, n, H, dv, dtype=torch.float64, device="cuda")
    lse = torch.zeros(B, n, H, dtype=torch.float64, device="cuda")
    gqa, rope = c["kind"] == "gqa_prompt", c["kind"] == "rope"
    q = x["q"].reshape(B, n, H, -1)
    width = dv if gqa else dc + dr
    for b, L in enumerate(lens):
        at = torch.arange(L - n, L, device="cuda")
        kr = x["kr"][b, :L].double()
        v_rows = x["v"][b, :, :L].double()
        if not gqa and not rope:                       # the new rows, rotated and rounded once
            v_rows[:, L - n:] = x["v_new"].reshape(B, n, G, dv)[b].double().transpose(0, 1)
            kr[L - n:] = _rotate(x["kr_new"].reshape(B, n, dr)[b].double(), at).to(dt).double()
        for h in range(H):
            v = v_rows[h // hpg]
            qh = q[b, :, h].double()
            if gqa:
                keys = x["k"][b, h // hpg, :L].double()
            else:
                keys = v @ x["m"][h].double()
                if rope:
                    keys = _rotate(keys, torch.arange(L, device="cuda"))
                    qh = _rotate(qh, at)
                else:
                    keys = torch.cat((keys, kr), -1)
                    qh = torch.cat((qh[:, :dc], _rotate(qh[:, dc:], at)), -1)
            keys = keys.t().contiguous()
            for i in range(0, n, 2048):
                sc = qh[i:i + 2048] @ keys / math.sqrt(width)
                hidden = torch.arange(L, device="cuda") > at[i:i + 2048].unsqueeze(1)
                sc.masked_fill_(hidden, -math.inf)
                lse[b, i:i + 2048, h] = torch.logsumexp(sc, -1)
                o[b, i:i + 2048, h] = torch.softmax(sc, -1) @ v
    out = {"o": o, "lse": lse}
    if c["kind"] != "prompt" and not gqa:
        out = {"o": o[:, 0], "lse": lse[:, 0]}
    if not gqa and not rope:
        out.update(v=None, kr=None)
    return out

"""The calls whose speed matters to a program that serves with this library,
each through the public binding: decode attention from one short sequence to a
full batch, chunked prefill from one prompt to a prefill-heavy step, the mixed
step (append, then attention over chunks and decode rows) and the scheduler.

``listed()`` names the fixed cases and ``draw(rng)`` gives another one of the
same ranges.  A case holds plain values; its context and chunk lengths follow
from those values alone (``lens`` seeds them), so its work is known without its
inputs, while every number in the inputs, and the place of every page, comes
from the seed that ``prepare`` takes.
"""
import math
import random

import numpy as np
import torch

from paper_2504_09345_amd import binding as pb

PAGE = 16


# --- the cases ---------------------------------------------------------------

def _decode(name, dtype="bf16", H_q=32, H_kv=8, D=128, B=1, ctx=("uniform", 1, 1), append=False, lens=1):
    kind, lo, hi = ctx[0], ctx[-2], ctx[-1]
    return dict(name=name, kind="decode", dtype=dtype, H_q=H_q, H_kv=H_kv, D=D, B=B, ctx=kind, ctx_lo=lo,
                ctx_hi=hi, ctx_median=ctx[1] if kind == "lognormal" else 0, append=append, lens=lens)


def _varlen(name, dtype="bf16", H_q=32, H_kv=8, D=128, chunks=1, chunk=(1, 1), prior=(0, 0), B=0, ctx=(1, 1),
            append=False, lens=1):
    return dict(name=name, kind="varlen", dtype=dtype, H_q=H_q, H_kv=H_kv, D=D, chunks=chunks,
                chunk_lo=chunk[0], chunk_hi=chunk[1], prior_lo=prior[0], prior_hi=prior[1], B=B,
                ctx="uniform", ctx_lo=ctx[0], ctx_hi=ctx[1], ctx_median=0, append=append, lens=lens)


def _sched(name, slots=256, steps=32, prompt=(98, 450), gen=256, lens=1):
    return dict(name=name, kind="sched", slots=slots, steps=steps, prompt_avg=prompt[0], prompt_max=prompt[1],
                gen_max=gen, lens=lens)


def listed():
    return [
        # one user, a short conversation: the new token's K/V go into the cache,
        # then it attends, through the entry that allocates nothing (the launch
        # and its latency are all there is)
        _decode("step-b1-ctx200", B=1, ctx=("uniform", 200, 200), append=True),
        # a lightly loaded server: few sequences of ordinary length
        _decode("decode-b8", B=8, ctx=("uniform", 512, 2048)),
        # the benchmark's batch (Mixtral-8x7B heads, 256 sequences)
        _decode("decode-mixtral-256", B=256, ctx=("uniform", 512, 2048)),
        # DBRX / Mixtral-8x22B heads, lognormal contexts, a large batch
        _decode("decode-dbrx-512", H_q=48, B=512, ctx=("lognormal", 1024, 128, 8192)),
        # a few very long contexts: every sequence is cut over many workgroups
        _decode("decode-long-b4", B=4, ctx=("uniform", 8192, 32768)),
        # the other head dim, a wide group
        _decode("decode-d64-b128", H_q=64, D=64, B=128, ctx=("uniform", 512, 2048)),
        # the other data type
        _decode("decode-fp32-b64", dtype="fp32", B=64, ctx=("uniform", 256, 2048)),
        # one prompt of odd length arrives alone: the time to its first token
        _varlen("prefill-1x700", chunks=1, chunk=(700, 700)),
        # a prefill-heavy step, the largest listed work
        _varlen("prefill-16x2048", chunks=16, chunk=(2048, 2048), prior=(0, 2048)),
        # chunks with the other head dim, ragged
        _varlen("prefill-d64-4", D=64, chunks=4, chunk=(200, 400), prior=(0, 1024)),
        # the mixed step of continuous batching: 8 prompt chunks and 512 decode
        # rows; their K/V are appended, then one varlen call attends
        _varlen("mixed-8x512-512", chunks=8, chunk=(512, 512), prior=(0, 1536), B=512, ctx=(256, 4096), append=True),
        # the scheduler that feeds those calls: 32 consecutive steps on 256
        # batch slots with short-chat arrivals
        _sched("sched-256"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    lens = rng.randrange(1 << 20)
    r = rng.random()
    if r < 0.12:
        mix = rng.choice([((98, 450), 32), ((98, 450), 128), ((98, 450), 256), ((926, 1843), 128), ((128, 410), 512)])
        c = _sched("", slots=_log_int(rng, 8, 4096), steps=rng.randint(8, 32), prompt=mix[0], gen=mix[1], lens=lens)
        del c["name"]
        return c
    H_kv = rng.choice([1, 2, 4, 8, 8, 8])
    H_q = H_kv * rng.choice([1, 2, 4, 4, 6, 8])
    D = rng.choice([64, 128, 128])
    dtype = rng.choice(["bf16", "bf16", "bf16", "bf16", "fp32"])
    heads = dict(dtype=dtype, H_q=H_q, H_kv=H_kv, D=D)
    token_bytes = 2 * H_kv * D * (2 if dtype == "bf16" else 4)
    if r < 0.6:
        mean = _log_int(rng, 20, 20000)
        B = max(1, min(_log_int(rng, 1, 512), int(8e8 / (mean * token_bytes))))
        c = _decode("", B=B, ctx=("uniform", max(1, mean // 3), mean + mean // 2), append=rng.random() < 0.3, lens=lens,
                    **heads)
    else:
        chunk, prior = _log_int(rng, 17, 2048), rng.choice([0, 0, _log_int(rng, 16, 4096)])
        # what the chunks cost is bounded by their (row, key) pairs
        pairs = 4e8 if dtype == "bf16" and D == 128 else 8e6 * 64 / D * (2 if dtype == "bf16" else 1)
        chunks = min(_log_int(rng, 1, 16), int(pairs * 8 / H_q / (chunk * (chunk / 2 + prior))))
        if chunks < 1:
            chunks, chunk, prior = 1, rng.randint(17, 300), 0
        B = 0 if r < 0.82 else min(_log_int(rng, 1, 256), int(4e8 / (2000 * token_bytes)))
        c = _varlen("", chunks=chunks, chunk=(max(2, chunk - chunk // 4), chunk), prior=(prior // 2, prior), B=B,
                    ctx=(1, 2000), append=rng.random() < 0.3, lens=lens, **heads)
    del c["name"]
    return c


# --- lengths and work --------------------------------------------------------

def _lengths(case):
    """(context length, query rows) of each sequence."""
    r = random.Random(case["lens"])
    ctx, rows = [], []
    if case["kind"] == "varlen":
        for _ in range(case["chunks"]):
            rows.append(r.randint(case["chunk_lo"], case["chunk_hi"]))
            ctx.append(rows[-1] + r.randint(case["prior_lo"], case["prior_hi"]))
    for _ in range(case["B"]):
        rows.append(1)
        if case["ctx"] == "lognormal":
            ctx.append(min(case["ctx_hi"], max(case["ctx_lo"], round(case["ctx_median"] * math.exp(r.gauss(0, 1))))))
        else:
            ctx.append(r.randint(case["ctx_lo"], case["ctx_hi"]))
    return ctx, rows


def work(case):
    if case["kind"] == "sched":
        # per slot and step: id, order, finish length and context read; context
        # and row prefix written
        return {"bytes": 24.0 * case["slots"] * case["steps"], "flops": 0.0}
    ctx, rows = _lengths(case)
    es = 2 if case["dtype"] == "bf16" else 4
    H_q, H_kv, D = case["H_q"], case["H_kv"], case["D"]
    nbytes = 2 * sum(ctx) * H_kv * D * es + 2 * sum(rows) * H_q * D * es
    nbytes += 4 * sum((c + PAGE - 1) // PAGE for c in ctx) + 4 * len(ctx)
    if case["append"]:
        nbytes += 4 * sum(rows) * H_kv * D * es  # new K and V, read and written
    pairs = sum(L * (C - L) + L * (L + 1) // 2 for C, L in zip(ctx, rows))
    return {"bytes": float(nbytes), "flops": 4.0 * D * H_q * pairs}


def tolerance(case):
    if case["kind"] == "sched":
        return "exact"
    # Measured against explicit splits of the same batches (sums in another
    # order): bf16 outputs differ by up to 1.1e-4 in the 2-norm and by one
    # rounding step (2^-7 of a value) at most, fp32 outputs by up to 3.6e-7 and
    # 1.7e-6.  Four times that for fp32; for bf16 about the output rounding's
    # own share (1.7e-3 against float64), which chunks with P in fp16 need.
    return {"rel": 2e-3, "max": 1.6e-2} if case["dtype"] == "bf16" else {"rel": 1.5e-6, "max": 8e-6}


# --- inputs ------------------------------------------------------------------

def _prepare_attention(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    H_q, H_kv, D = case["H_q"], case["H_kv"], case["D"]
    ctx, rows = _lengths(case)
    B, T = len(ctx), sum(rows)
    npages = [(c + PAGE - 1) // PAGE for c in ctx]
    need, width = sum(npages), max(npages)
    num_pages = max(need + 1, math.ceil(1.25 * need))

    def normal(*shape):
        return torch.randn(shape, dtype=dt, device="cuda", generator=g)

    perm = torch.randperm(num_pages, device="cuda", generator=g).to(torch.int32).cpu().numpy()
    table = np.full((B, width), perm[need], np.int32)  # unused entries: a page nobody owns
    at = 0
    for b, n in enumerate(npages):
        table[b, :n] = perm[at:at + n]
        at += n
    st = dict(case=case, q=normal(T, H_q, D), k=normal(num_pages, H_kv, PAGE, D), v=normal(num_pages, H_kv, PAGE, D),
              bt=torch.from_numpy(table).cuda(), cl=torch.tensor(ctx, dtype=torch.int32, device="cuda"))
    st["out"] = torch.empty_like(st["q"])
    st["scale"] = 1.0 / math.sqrt(D)
    starts = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    st["qsl"] = torch.from_numpy(starts).cuda()
    st["ctx"], st["rows"], st["table"], st["starts"] = ctx, rows, table, starts
    varlen = case["kind"] == "varlen"
    if case["append"]:
        st["k_new"], st["v_new"] = normal(T, H_kv, D), normal(T, H_kv, D)
    # a decode step with its append goes through the entry without a workspace
    st["noalloc"] = not varlen and case["append"]
    if varlen or st["noalloc"]:
        st["dims"] = pb.make_dims(st["q"], st["k"], st["bt"], max(ctx), num_q_rows=T, max_q_len=max(rows))
    else:
        st["dims"] = pb.make_dims(st["q"], st["k"], st["bt"], max(ctx))
    if not st["noalloc"]:
        st["ws"] = torch.empty(max(1, pb.pa_workspace_size(st["dims"])), dtype=torch.uint8, device="cuda")
    return st


_SCHED = ("free_pages", "hdr", "queue_seq", "queue_tok", "queue_fin", "slot_seq", "slot_order", "slot_fin",
          "context_lens", "block_table")


def _prepare_sched(case, seed):
    """A scheduler in mid-service: most slots decoding somewhere in their
    generation, a short queue, and the arrivals of the coming steps on the
    device."""
    rng = np.random.default_rng([seed, case["lens"]])
    S, steps, gen = case["slots"], case["steps"], case["gen_max"]
    median = case["prompt_avg"] / math.exp(0.32)

    def requests(n):
        p = np.clip(np.rint(median * np.exp(0.8 * rng.standard_normal(n))), 1, case["prompt_max"]).astype(np.int32)
        return p, p + rng.integers(1, gen, size=n, endpoint=True).astype(np.int32)

    MP = (case["prompt_max"] + gen + PAGE - 1) // PAGE
    P = int(S * (case["prompt_avg"] + gen / 2) / PAGE) + 2 * MP  # short of every slot at full length
    Q = 4 * S + 64
    live = rng.random(S) < 0.9
    prompt, fin = requests(S)
    ctx = np.where(live, rng.integers(prompt, fin, endpoint=True), 0).astype(np.int32)
    held = (ctx + PAGE - 1) // PAGE
    while held.sum() > P - MP:  # what the pool holds
        i = rng.choice(np.flatnonzero(live))
        live[i], ctx[i], held[i] = False, 0, 0
    perm = rng.permutation(P).astype(np.int32)
    table = np.zeros((S, MP), np.int32)
    at = 0
    for s in np.flatnonzero(held):
        table[s, :held[s]] = perm[at:at + held[s]]
        at += held[s]
    free = np.zeros(P, np.int32)
    free[:P - at] = perm[at:]
    nq = S // 4
    qp, qf = requests(nq)
    queue = np.zeros((3, Q), np.int32)
    queue[0, :nq], queue[1, :nq], queue[2, :nq] = np.arange(S, S + nq), qp, qf
    order = rng.permutation(S).astype(np.int32)
    host = dict(free_pages=free, hdr=np.array([P - at, S, 0, nq], np.int32), queue_seq=queue[0], queue_tok=queue[1],
                queue_fin=queue[2], slot_seq=np.where(live, np.arange(S), -1).astype(np.int32), slot_order=order,
                slot_fin=fin.astype(np.int32), context_lens=ctx, block_table=table)
    flat = torch.from_numpy(np.concatenate([host[n].reshape(-1) for n in _SCHED])).cuda()
    cur, arrays, at = torch.empty_like(flat), {}, 0
    for n in _SCHED:
        arrays[n] = cur[at:at + host[n].size].view(host[n].shape)
        at += host[n].size
    st = dict(case=case, start=flat, cur=cur, arrays=arrays, c=pb.make_sched_state(arrays), n_real=8 * S)
    nid, st["new"] = 2 * S, []
    for _ in range(steps):
        n = int(rng.poisson(2 * S / gen))
        p, f = requests(n)
        st["new"].append([torch.from_numpy(x.astype(np.int32)).cuda() for x in (np.arange(nid, nid + n), p, f)])
        nid += n
    # a ring of output buffers, one per step in flight to the rest of the program
    st["qsl"] = torch.zeros((steps, S + 1), dtype=torch.int32, device="cuda")
    st["fin"] = torch.zeros((steps, S), dtype=torch.int32, device="cuda")
    st["info"] = torch.zeros((steps, 8), dtype=torch.int32, device="cuda")
    return st


def prepare(case, seed):
    return _prepare_sched(case, seed) if case["kind"] == "sched" else _prepare_attention(case, seed)


# --- one pass ----------------------------------------------------------------

def run(st):
    if st["case"]["kind"] == "sched":
        st["cur"].copy_(st["start"])
        for i, (ids, prompts, fins) in enumerate(st["new"]):
            pb.pa_schedule_step(st["c"], st["n_real"], ids, prompts, fins, ids.numel(), st["qsl"][i], st["fin"][i],
                                st["info"][i])
        return dict(state=st["cur"], rows=st["qsl"], finished=st["fin"], info=st["info"])
    args = (st["q"], st["k"], st["v"], st["bt"], st["cl"])
    varlen = st["case"]["kind"] == "varlen"
    res = dict(out=st["out"])
    if st["case"]["append"]:
        pb.pa_kv_append(st["k_new"], st["v_new"], st["bt"], st["cl"], st["k"], st["v"], st["dims"],
                        query_start_loc=st["qsl"] if varlen else None)
        res.update(k=st["k"], v=st["v"])
    if st["noalloc"]:
        pb.paged_attn_varlen_noalloc(*args, st["qsl"], st["scale"], st["out"], st["dims"])
    elif varlen:
        pb.paged_attn_varlen(*args, st["qsl"], st["scale"], st["out"], st["dims"], workspace=st["ws"])
    else:
        pb.paged_attn(*args, st["scale"], st["out"], st["dims"], workspace=st["ws"])
    return res


# --- the same in 64 bits -----------------------------------------------------

def exact(case, seed):
    """What ``run`` returns for these inputs, from plain torch in float64."""
    if case["kind"] == "sched":
        return None
    st = _prepare_attention(case, seed)
    H_q, H_kv, D = case["H_q"], case["H_kv"], case["D"]
    s, k, v = H_q // H_kv, st["k"], st["v"]
    if case["append"]:
        pos, page = [], []
        for b, (C, L) in enumerate(zip(st["ctx"], st["rows"])):
            p = np.arange(C - L, C)
            pos.append(p % PAGE)
            page.append(st["table"][b, p // PAGE])
        page = torch.from_numpy(np.concatenate(page).astype(np.int64)).cuda()
        pos = torch.from_numpy(np.concatenate(pos)).cuda()
        k[page, :, pos] = st["k_new"]
        v[page, :, pos] = st["v_new"]
    out = torch.empty(st["q"].shape, dtype=torch.float64, device="cuda")
    for b, (C, L) in enumerate(zip(st["ctx"], st["rows"])):
        pages = st["bt"][b, :(C + PAGE - 1) // PAGE].long()
        r0 = int(st["starts"][b])
        visible = torch.arange(C, device="cuda")[None, :] <= torch.arange(C - L, C, device="cuda")[:, None]
        for g in range(H_kv):
            kd = k[pages, g].reshape(-1, D)[:C].double()
            vd = v[pages, g].reshape(-1, D)[:C].double()
            qd = st["q"][r0:r0 + L, g * s:(g + 1) * s].double().transpose(0, 1).reshape(s * L, D)
            x = torch.matmul(qd, kd.t().contiguous()).view(s, L, C) * st["scale"]
            w = torch.softmax(x.masked_fill_(~visible, -math.inf), dim=-1).view(s * L, C)
            out[r0:r0 + L, g * s:(g + 1) * s] = torch.matmul(w, vd).view(s, L, D).transpose(0, 1)
    res = dict(out=out)
    if case["append"]:
        res.update(k=k, v=v)
    return res

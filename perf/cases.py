"""Performance cases: what a serving program asks of this library.

Two kinds of call:

* ``layer``: one transformer layer's attention within a step, the call that
  runs once per layer: ``kv_append`` of the step's new keys and values, then
  the attention call, with the step's metadata and launch plan on the device
  already (a program builds and uploads them once per step and uses them in
  every layer).
* ``step``: a whole one-layer step through the staged path: the pool
  operations, metadata and plan in one library call, their upload, append,
  attention, and the rollback that ends the step.

Sequences are requests over cached prefixes: ``prefix`` tokens shared (over
``prefixes`` different prefixes, each twice as long as the one before, the
shorter ones the more popular), then ``ctx_lo .. ctx_hi`` cached tokens of the
request's own, then ``q_lo .. q_hi`` new tokens.  Lengths come from the case
(``lens``), so every seed of a case does the same work; token ids, block
placement, queries, keys and values come from the seed.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2605_11232_amd import binding as B
from paper_2605_11232_amd import runtime, synth

BS = 16               # tokens per cache block
PREFIX_SEQ = 1 << 40  # ids of the sequences that put the prefixes into the cache
DTYPE = {"bf16": torch.bfloat16, "f32": torch.float32}
SIZE = {"bf16": 2, "f32": 4}
KIND = {"prefill": B.KIND_PREFILL, "mixed": B.KIND_PREFILL, "decode": B.KIND_DECODE,
        "verify": B.KIND_VERIFY}
MIXED_CHUNK = 512     # tokens of a mixed launch's prefill chunks

# a drawn case costs no more than the largest listed ones
MOST_FLOPS, MOST_BYTES, MOST_F32_FLOPS = 1.3e12, 1.3e9, 1.2e10


def _case(name, kind, seqs, prefix, ctx, q, heads=(32, 8, 128), dtype="bf16", call="layer",
          prefixes=1, noalloc=False, lens=1):
    return {"name": name, "call": call, "kind": kind, "dtype": dtype, "hq": heads[0],
            "hkv": heads[1], "d": heads[2], "seqs": seqs, "prefix": prefix, "prefixes": prefixes,
            "ctx_lo": ctx[0], "ctx_hi": ctx[1], "q_lo": q[0], "q_hi": q[1], "noalloc": noalloc,
            "lens": lens}


def listed():
    return [
        # four short float32 requests on a cached prefix: the smallest call, the
        # configuration that exactness is checked on
        _case("tiny_f32", "prefill", 4, 128, (0, 0), (32, 64), (8, 2, 64), "f32"),
        # float32 prefill of a model's own head shape: a reference run at ordinary lengths
        _case("f32_prefill", "prefill", 8, 512, (0, 0), (64, 256), dtype="f32"),
        # an interactive server with few requests in flight: latency of one layer,
        # through the entry point for callers that cannot allocate
        _case("decode_few", "decode", 4, 2048, (256, 1152), (1, 1), noalloc=True),
        # the batch decode of the benchmark: 256 requests on one policy prefix
        _case("decode_batch", "decode", 256, 2048, (256, 1152), (1, 1)),
        # long private contexts that share nothing: all of the cache is read
        _case("decode_long", "decode", 24, 0, (8192, 20480), (1, 1), (64, 8, 128)),
        # a decode step with its host side: 64 requests
        _case("decode_step", "decode", 64, 2048, (256, 1152), (1, 1), call="step"),
        # one case arrives: its evidence against the cached policy prefix
        _case("prefill_one", "prefill", 1, 2048, (0, 0), (389, 389)),
        # the benchmark's prefill: 64 requests on one cached prefix
        _case("prefill_batch", "prefill", 64, 2048, (0, 0), (256, 1024)),
        # whole prompts with nothing cached (how a prefix gets into the cache)
        _case("prefill_long", "prefill", 3, 0, (0, 0), (4000, 12000), (28, 4, 128)),
        # a smaller model: head_dim 64
        _case("prefill_d64", "prefill", 24, 1024, (0, 0), (128, 512), (32, 8, 64)),
        # chunked prefill and decode in one launch over four prefixes (the benchmark's)
        _case("mixed_batch", "mixed", 512, 1024, (256, 1152), (1, 1), (28, 4, 128), prefixes=4),
        # speculative verification on a very long prefix (the benchmark's)
        _case("verify_batch", "verify", 32, 16384, (4096, 4096), (5, 5), (64, 8, 128)),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice(["decode", "decode", "decode", "prefill", "prefill", "prefill", "verify",
                       "mixed", "f32", "step"])
    lens = rng.randrange(1 << 20)
    heads = rng.choice([(32, 8, 128), (32, 8, 128), (28, 4, 128), (64, 8, 128), (32, 8, 64)])
    prefix = rng.choice([0, _log(rng, 64, 8192), _log(rng, 512, 8192)])
    if what == "f32":
        heads = rng.choice([(8, 2, 64), (8, 2, 128), (32, 8, 128)])
        prefix, lo = rng.choice([0, _log(rng, 32, 512)]), _log(rng, 1, 128)
        if rng.random() < 0.3:
            c = _case("", "decode", _log(rng, 1, 16), prefix, (lo, 4 * lo), (1, 1), heads, "f32",
                      lens=lens)
        else:
            c = _case("", "prefill", _log(rng, 1, 8), prefix, (0, 0), (lo, 2 * lo), heads, "f32",
                      lens=lens)
    elif what == "decode":
        lo = _log(rng, 1, 8192)
        c = _case("", "decode", _log(rng, 1, 256), prefix, (lo, int(lo * rng.uniform(1, 4))),
                  (1, 1), heads, noalloc=rng.random() < 0.25, lens=lens)
    elif what == "prefill":
        lo = _log(rng, 1, 2048)
        c = _case("", "prefill", _log(rng, 1, 64), prefix, (0, rng.choice([0, 512])),
                  (lo, int(lo * rng.uniform(1, 4))), heads, lens=lens)
    elif what == "verify" or (what == "step" and rng.random() < 0.3):
        lo, nq = _log(rng, 16, 4096), rng.randint(2, 8)
        c = _case("", "verify", _log(rng, 1, 32), 2 * prefix, (lo, int(lo * rng.uniform(1, 2))),
                  (nq, nq), heads, call="step" if what == "step" else "layer", lens=lens)
    elif what == "step":
        lo = _log(rng, 16, 4096)
        c = _case("", "decode", _log(rng, 1, 256), prefix, (lo, int(lo * rng.uniform(1, 4))),
                  (1, 1), heads, call="step", lens=lens)
    else:
        lo = _log(rng, 64, 512)
        c = _case("", "mixed", _log(rng, 16, 512), _log(rng, 64, 1024), (lo, 4 * lo), (1, 1),
                  heads, prefixes=rng.randint(1, 4), lens=lens)
    del c["name"]
    most = MOST_F32_FLOPS if c["dtype"] == "f32" else MOST_FLOPS
    while c["seqs"] > 1:
        w = work(c)
        if w["flops"] <= most and w["bytes"] <= MOST_BYTES:
            break
        c["seqs"] = max(1, c["seqs"] * 3 // 4)
    return c


def _shape(c):
    """(prefix lengths, [(prefix id, own cached tokens, new tokens) per sequence])."""
    r = random.Random(c["lens"])
    plens = [c["prefix"] << p for p in range(c["prefixes"])]
    weights = [1.0 / (p + 1) ** 1.1 for p in range(c["prefixes"])]
    seqs = []
    for i in range(c["seqs"]):
        p = r.choices(range(c["prefixes"]), weights)[0]
        if c["kind"] == "mixed" and i % 8 == 0:
            seqs.append((p, r.choice([0, MIXED_CHUNK]), MIXED_CHUNK))
        else:
            seqs.append((p, r.randint(c["ctx_lo"], c["ctx_hi"]), r.randint(c["q_lo"], c["q_hi"])))
    r.shuffle(seqs)
    return plens, seqs


def work(c):
    plens, seqs = _shape(c)
    hq, hkv, d, s = c["hq"], c["hkv"], c["d"], SIZE[c["dtype"]]
    cached = flops = table = T = 0
    for p in {p for p, _, _ in seqs}:
        cached += plens[p] // BS * BS
    for p, ctx, q in seqs:
        L = plens[p] + ctx + q
        T += q
        cached += plens[p] % BS + ctx
        table += -(-L // BS) + 2
        flops += 4 * d * hq * (q * (L - q) + q * (q + 1) // 2)
    kv_row = 2 * hkv * d * s
    # cached keys and values read, new ones read and stored, q in, out and lse out
    bytes_ = (cached + 2 * T) * kv_row + 2 * T * hq * d * s + 4 * T * hq + 4 * (table + T)
    return {"bytes": bytes_, "flops": flops}


def _tokens(rng, n):
    return rng.integers(0, synth.TOKEN_VOCAB, size=n, dtype=np.int32)


def _state(c, seed, pending):
    """The device's cache, the pool with every request admitted and, for a layer, the
    step's metadata and plan on the device.  pending=False leaves a step's new tokens
    to the step itself."""
    rng = np.random.default_rng([seed, 1])
    gen = torch.Generator(device="cuda").manual_seed(seed)
    plens, seqs = _shape(c)
    n, hq, hkv, d, dt = len(seqs), c["hq"], c["hkv"], c["d"], DTYPE[c["dtype"]]
    lens = [plens[p] + ctx + q for p, ctx, q in seqs]
    T = sum(q for _, _, q in seqs)
    max_blocks = max(-(-x // BS) for x in lens)
    nb = (sum(-(-x // BS) for x in plens) + 32
          + sum(-(-lens[i] // BS) - plens[p] // BS for i, (p, _, _) in enumerate(seqs)))
    pool = B.Pool(nb, BS, rng.permutation(nb).astype(np.int32))
    prefixes = [_tokens(rng, x) for x in plens]
    for p, toks in enumerate(prefixes):
        if len(toks):
            pool.add(PREFIX_SEQ + p, toks)
            pool.free(PREFIX_SEQ + p)
    late = c["kind"] in ("decode", "verify")  # new tokens extend a live request
    extend = []
    for i, (p, ctx, q) in enumerate(seqs):
        body = _tokens(rng, ctx + q)
        pool.add(i, np.concatenate([prefixes[p], body[:ctx] if late else body]))
        extend.append(body[ctx:])
    if late and pending:
        for i in range(n):
            pool.extend(i, extend[i])

    def values(*shape):
        return torch.randn(shape, dtype=dt, device="cuda", generator=gen)

    st = {"case": c, "pool": pool, "lens": lens,
          "k_cache": values(nb, hkv, d // 32, BS, 32), "v_cache": values(nb, hkv, d, BS),
          "q": values(T, hq, d), "k_new": values(T, hkv, d), "v_new": values(T, hkv, d),
          "out": torch.empty((T, hq, d), dtype=dt, device="cuda"),
          "lse": torch.empty((T, hq), dtype=torch.float32, device="cuda")}
    ids, q_lens = list(range(n)), [q for _, _, q in seqs]
    kind, n_q = KIND[c["kind"]], q_lens[0] if c["kind"] == "verify" else 1
    code = B.PA_BF16 if c["dtype"] == "bf16" else B.PA_F32
    if pending:
        md = pool.metadata(ids, q_lens, max_blocks)
        plan, info = B.plan(kind, n_q, md["seq_lens"], md["cu_seqlens_q"], hq, hkv, d, BS, code,
                            block_table=md["block_table"])
        dev = {k: torch.from_numpy(np.array(v)).cuda() for k, v in md.items()}
        st.update(kind=kind, info=info, plan=torch.from_numpy(np.array(plan)).cuda(),
                  slots=dev["slot_mapping"], block_table=dev["block_table"],
                  seq_lens=dev["seq_lens"], cu=dev["cu_seqlens_q"],
                  ws=torch.empty(int(info.workspace_bytes), dtype=torch.uint8, device="cuda")
                  if info.workspace_bytes else None)
    if c["call"] == "step" and not pending:
        cfg = synth.AttnConfig("step", c["dtype"], hq, hkv, d, BS, 0)
        words = runtime.plan_words_bound(cfg, n, T, max_blocks)
        off = np.concatenate([[0], np.cumsum(q_lens)])
        none, zero = np.zeros(0, np.int32), np.zeros(n, np.int32)
        st.update(
            kind=kind, n_q=n_q, code=code, turn=0, ws=None, inputs=B.LaunchInputs(ids, q_lens),
            stagings=[runtime.Staging("cuda", n, max_blocks, T, words) for _ in range(2)],
            pre=B.PackedOps([B.OP_EXTEND] * n, ids, off, np.concatenate(extend), zero),
            post=B.PackedOps([B.OP_TRUNCATE] * n, ids, np.zeros(n + 1, np.int32), none,
                             [x - q for x, q in zip(lens, q_lens)]))
    return st


def prepare(c, seed):
    return _state(c, seed, pending=c["call"] != "step")


def _step(st):
    """One serving step through a staging buffer, the other one still in use by the step before."""
    c, pool = st["case"], st["pool"]
    sg = st["stagings"][st["turn"]]
    st["turn"] ^= 1
    inp = st["inputs"]
    sg.wait()
    info = pool.prepare_launch(st["pre"], inp, sg.buffers, st["kind"], st["n_q"], c["hq"],
                               c["hkv"], c["d"], st["code"], info=sg.info)
    if info.workspace_bytes and (st["ws"] is None or st["ws"].numel() < info.workspace_bytes):
        st["ws"] = torch.empty(int(info.workspace_bytes), dtype=torch.uint8, device="cuda")
    B.stage_upload(sg.dev, sg.host, 4 * (sg.plan_off + int(info.plan_words)))
    sg.ready.record()
    sg.used = True
    bt, sl, cu, slots = sg.device_views(inp.n, inp.total_q)
    B.kv_append(st["k_new"], st["v_new"], slots, st["k_cache"], st["v_cache"])
    B.attention(st["kind"], st["q"], st["k_cache"], st["v_cache"], bt, sl, cu, sg.plan[1], info,
                st["ws"] if info.workspace_bytes else None, st["out"], st["lse"])
    pool.apply_packed(st["post"])


def run(st):
    if st["case"]["call"] == "step":
        _step(st)
    else:
        B.kv_append(st["k_new"], st["v_new"], st["slots"], st["k_cache"], st["v_cache"])
        if st["case"]["noalloc"] and st["info"].workspace_bytes <= B.NOALLOC_WORKSPACE_BYTES:
            B.attention_decode_noalloc(st["q"], st["k_cache"], st["v_cache"], st["block_table"],
                                       st["seq_lens"], st["cu"], st["plan"], st["info"],
                                       st["out"], st["lse"])
        else:
            B.attention(st["kind"], st["q"], st["k_cache"], st["v_cache"], st["block_table"],
                        st["seq_lens"], st["cu"], st["plan"], st["info"], st["ws"], st["out"],
                        st["lse"])
    return {"out": st["out"], "lse": st["lse"], "k_cache": st["k_cache"],
            "v_cache": st["v_cache"]}


def tolerance(c):
    # bf16: the output's own rounding (2^-9 of each value) and that of the probabilities
    # in the value product, 2.3e-3 measured against exact(); float32: sums in another
    # order, 4.7e-7 measured
    return {"rel": 1e-2, "max": 0.1} if c["dtype"] == "bf16" else {"rel": 2e-6, "max": 4e-5}


def exact(c, seed):
    """The same outputs in 64 bits: the new rows scattered into the cache, and softmax
    attention of every sequence over its keys and values read through the block table."""
    st = _state(c, seed, pending=True)  # a step's tables too: its tokens appended
    hq, hkv, d = c["hq"], c["hkv"], c["d"]
    G = hq // hkv
    kc, vc = st["k_cache"], st["v_cache"]
    off = torch.arange(BS, device="cuda")
    pos = (off & ~12) | ((off & 4) << 1) | ((off & 8) >> 1)  # a key's place in its block
    slots = st["slots"].long()
    T = slots.numel()
    kc[slots // BS, :, :, pos[slots % BS], :] = st["k_new"].view(T, hkv, d // 32, 32)
    vc[slots // BS, :, :, slots % BS] = st["v_new"]
    out = torch.empty((T, hq, d), dtype=torch.float64, device="cuda")
    lse = torch.empty((T, hq), dtype=torch.float64, device="cuda")
    cu = st["cu"].tolist()
    for r, L in enumerate(st["lens"]):
        blocks = st["block_table"][r, :-(-L // BS)].long()
        k = kc[blocks][:, :, :, pos].double().permute(1, 2, 4, 0, 3)  # [hkv, d / 32, 32, nb, bs]
        kt = k.reshape(hkv, d, -1)[:, :, :L].contiguous()
        v = vc[blocks].double().permute(1, 0, 3, 2).reshape(hkv, -1, d)[:, :L].contiguous()
        n = cu[r + 1] - cu[r]
        rows = max(1, (1 << 27) // (hq * L))  # queries at once: scores of at most 1 GiB
        for i in range(0, n, rows):
            m = min(rows, n - i)
            q = st["q"][cu[r] + i:cu[r] + i + m].double() * d ** -0.5
            q = q.view(m, hkv, G, d).permute(1, 0, 2, 3).reshape(hkv, m * G, d).contiguous()
            s = torch.bmm(q, kt).view(hkv, m, G, L)
            last = torch.arange(L - n + i, L - n + i + m, device="cuda")
            hidden = torch.arange(L, device="cuda") > last[:, None]
            s.masked_fill_(hidden[None, :, None, :], -math.inf)
            z = torch.logsumexp(s, dim=3)
            p = s.sub_(z[..., None]).exp_().view(hkv, m * G, L)
            o = torch.bmm(p, v).view(hkv, m, G, d).permute(1, 0, 2, 3)
            out[cu[r] + i:cu[r] + i + m] = o.reshape(m, hq, d)
            lse[cu[r] + i:cu[r] + i + m] = z.permute(1, 0, 2).reshape(m, hq)
    return {"out": out, "lse": lse, "k_cache": kc, "v_cache": vc}

"""The calls a program makes of this framework, as timed cases: the decode step of one attention layer, the
prefill step that builds its packed cache, and the set-up of a request.

A case is a dict of plain values:
  kind       "decode" (one single-query attention call), "append" (a generated token is stored, then the call),
             "prefill" (reorder + quantize of a dense or ragged source), "paged" (the same from a paged cache),
             "request" (chunk-level search, plan, cache, reorder + quantize: what happens once per request and layer)
  batch, q_heads, kv_heads, head_dim, chunk, group     the geometry of the layer
  tokens     context tokens of the longest sequence; shortest: of the shortest one (equal: a batch in lockstep)
  lengths    which lengths a ragged batch has between the two
  mix        percent of the chunks kept at FP16/INT8/INT4/INT2
  appended   generated tokens the call attends to ("append"); page: tokens per page ("paged")

K has four outlier channels per kv head, K, V and q are Gaussian, the bitwidths of the chunks are shuffled and
shared by the heads of a sequence, as in workloads.py.
"""
import math
import random

import numpy as np
import torch

import paper_2503_23294_amd as ck

BITS = (16, 8, 4, 2)            # the order of `mix`
EMBED_DIM = 768                 # width of the retrieval encoder's embeddings
MIX_FEW = "10/0/30/60"          # few chunks matter to a query
MIX_LONG = "5/0/25/70"          # the mix of the 128K-token workload
MIX_GQA = "15/0/35/50"
MIX_INT8 = "5/15/30/50"         # four classes


def _case(name, kind, batch, q_heads, kv_heads, tokens, mix, **more):
    case = {"name": name, "kind": kind, "batch": batch, "q_heads": q_heads, "kv_heads": kv_heads, "head_dim": 128,
            "chunk": 256, "group": 32, "tokens": tokens, "shortest": tokens, "lengths": 0, "mix": mix, "appended": 0, "page": 0}
    case.update(more)
    return case


def listed():
    return [
        # a short prompt on few heads: launches and latency
        _case("decode_2k_8h", "decode", 1, 8, 8, 2048, MIX_FEW, chunk=128),
        # a 7B-class layer (one query head per kv head) at 32K
        _case("decode_32k_32h", "decode", 1, 32, 32, 32768, MIX_FEW),
        # a 13B-class layer at 128K: the largest multi-head context
        _case("decode_128k_40h", "decode", 1, 40, 40, 131072, MIX_LONG, chunk=512, group=64),
        # an 8B-class grouped-query layer, a small batch in lockstep
        _case("decode_64k_gqa4_b4", "decode", 4, 32, 8, 65536, MIX_GQA),
        # the same layer serving eight requests of unlike, odd lengths
        _case("decode_ragged_gqa4_b8", "decode", 8, 32, 8, 130001, "33/0/33/34", shortest=8193, lengths=5),
        # four classes with INT8 chunks
        _case("decode_64k_gqa4_int8_b4", "decode", 4, 32, 8, 65536, MIX_INT8, group=64),
        # a 70B-class layer: eight query heads per kv head
        _case("decode_128k_gqa8_b4", "decode", 4, 64, 8, 131072, MIX_GQA),
        # sixteen query heads per kv head, ragged, odd lengths
        _case("decode_ragged_gqa16_b8", "decode", 8, 64, 4, 65535, MIX_GQA, shortest=4097, lengths=16, group=64),
        # a step of a running generation: store the new token, attend to 16K of context and 300 generated tokens
        _case("append_16k_gqa8_b8", "append", 8, 64, 8, 16384, MIX_GQA, appended=300),
        # prefill of the 13B-class layer: the largest pass over memory
        _case("prefill_128k_40h", "prefill", 1, 40, 40, 131072, MIX_LONG, chunk=512, group=64),
        # prefill out of a serving engine's paged cache, sixteen tokens a page
        _case("paged16_ragged_gqa8_b4", "paged", 4, 64, 8, 65536, MIX_GQA, shortest=8191, lengths=3, page=16),
        # a request comes in: 32-token chunks (the paper's size), odd lengths
        _case("request_32k_gqa4_b2", "request", 2, 32, 8, 32775, "", shortest=20001, lengths=1, chunk=32),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode"] * 5 + ["append", "prefill", "paged", "request"])
    head_dim = rng.choice([128, 128, 128, 64])
    kv_heads = rng.choice([1, 2, 4, 8, 8, 8, 16, 32, 40])
    rep = rng.choice([1, 1, 2, 3, 4, 4, 5, 6, 7, 8, 8, 10, 12, 16]) if kv_heads <= 8 else rng.choice([1, 1, 2])
    batch = rng.choice([1, 1, 2, 3, 4, 8])
    # no more fp16 source than the largest listed case has
    most = min(131072, 40 * 131072 * 128 // (batch * kv_heads * head_dim))
    if kind == "request":
        most = min(most, 40000)
    tokens = _log_uniform(rng, 1024, most)
    ragged = batch > 1 and rng.random() < 0.5
    return {"kind": kind, "batch": batch, "q_heads": kv_heads * rep, "kv_heads": kv_heads, "head_dim": head_dim,
            "chunk": rng.choice([32, 64, 128, 256, 512]), "group": rng.choice([32, 64] if head_dim == 64 else [32, 64, 128]),
            "tokens": tokens, "shortest": max(1, _log_uniform(rng, max(1, tokens // 16), tokens)) if ragged else tokens,
            "lengths": rng.randrange(1000), "mix": rng.choice([MIX_FEW, MIX_LONG, MIX_GQA, MIX_INT8]),
            "appended": rng.randrange(1, 600) if kind == "append" else 0,
            "page": rng.choice([16, 32, 64, 100, 256]) if kind == "paged" else 0}


def _lengths(case):
    rng, n = random.Random(case["lengths"]), case["batch"]
    if case["shortest"] == case["tokens"]:
        return [case["tokens"]] * n
    inner = [rng.randint(case["shortest"], case["tokens"]) for _ in range(n - 2)]
    seqs = ([case["tokens"], case["shortest"]] + inner)[:n]
    rng.shuffle(seqs)
    return seqs


def _shares(case):
    return [int(x) / 100 for x in case["mix"].split("/")]


def _class_chunks(case, chunks):
    """How many of a sequence's chunks are kept at each of BITS."""
    count = [int(round(s * chunks)) for s in _shares(case)[:-1]]
    while sum(count) > chunks:
        count[count.index(max(count))] -= 1
    return count + [chunks - sum(count)]


def _chunk_bits(case, seed):
    rng = np.random.default_rng([250323294, 7, int(seed)])
    out = []
    for t in _lengths(case):
        bits = np.repeat(np.array(BITS, dtype=np.uint8), _class_chunks(case, t // case["chunk"]))
        rng.shuffle(bits)
        out.append(bits)
    return out


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(1000003 * int(seed) + 17)


def _keys_values(case, gen):
    """K and V of all sequences, one behind the other, each [kv_heads, T, head_dim] (fp16, flat)."""
    rows = sum(_lengths(case)) * case["kv_heads"]
    d = case["head_dim"]
    k = torch.empty(rows * d, dtype=torch.float16, device="cuda").normal_(generator=gen)
    v = torch.empty(rows * d, dtype=torch.float16, device="cuda").normal_(generator=gen)
    outliers = torch.rand(case["kv_heads"], d, device="cuda", generator=gen).argsort(dim=1)[:, :4]
    factor = torch.ones(case["kv_heads"], 1, d, dtype=torch.float16, device="cuda").scatter_(2, outliers[:, None], 10.0)
    at = 0
    for t in _lengths(case):
        n = case["kv_heads"] * t * d
        k[at:at + n].view(case["kv_heads"], t, d).mul_(factor)
        at += n
    return k, v


def _inputs(case, seed):
    """What exact() needs as well: sources, query, appended rows, all from the seed."""
    gen = _generator(seed)
    k, v = _keys_values(case, gen)
    q = torch.empty(case["batch"], case["q_heads"], case["head_dim"], dtype=torch.float16, device="cuda").normal_(generator=gen)
    new = torch.empty(2, case["appended"], case["batch"], case["kv_heads"], case["head_dim"], dtype=torch.float16,
                      device="cuda").normal_(generator=gen)
    return k, v, q, new


def _shape(case):
    return ck.make_shape(case["batch"], case["q_heads"], case["kv_heads"], case["head_dim"], case["chunk"], case["group"])


def _fill(cache, case, k, v):
    """The prefill call: a dense [B, Hkv, T, D] source for a batch in lockstep, else sequences back to back."""
    if case["shortest"] == case["tokens"]:
        shape = (case["batch"], case["kv_heads"], case["tokens"], case["head_dim"])
        ck.cocktail_reorder_quantize(cache, k.view(shape), v.view(shape))
    else:
        ck.cocktail_reorder_quantize(cache, k, v, ragged=True)


def _pages(case, k, v, gen):
    """The same tokens in pages of a pool, in random order: K pool, V pool, page table."""
    ps, h, d = case["page"], case["kv_heads"], case["head_dim"]
    need = [-(-t // ps) for t in _lengths(case)]
    ids = torch.rand(sum(need), device="cuda", generator=gen).argsort()
    table = torch.zeros(case["batch"], max(need), dtype=torch.int32, device="cuda")
    pools = [torch.zeros(sum(need), h, ps, d, dtype=torch.float16, device="cuda") for _ in range(2)]
    for pool, flat in zip(pools, (k, v)):
        at = page = 0
        for b, t in enumerate(_lengths(case)):
            padded = torch.zeros(h, need[b] * ps, d, dtype=torch.float16, device="cuda")
            padded[:, :t] = flat[at:at + h * t * d].view(h, t, d)
            pool[ids[page:page + need[b]]] = padded.view(h, need[b], ps, d).permute(1, 0, 2, 3)
            table[b, :need[b]] = ids[page:page + need[b]].to(torch.int32)
            at, page = at + h * t * d, page + need[b]
    return pools[0], pools[1], table


def _kept(chunks):
    """How many of a sequence's chunks the search of a request keeps at each of BITS: few are relevant to the query."""
    few, some = max(1, chunks * 6 // 100), chunks * 14 // 100
    return [few, 0, some, chunks - few - some]


def _embeddings(case, gen):
    """Query and chunk embeddings with cosines clear of the two thresholds (range 0 to 0.8: 0.48 and 0.72), in random order."""
    counts = [t // case["chunk"] for t in _lengths(case)]
    q = torch.randn(case["batch"], EMBED_DIM, device="cuda", generator=gen)
    parts = []
    for b, n in enumerate(counts):
        high, _, mid, low = _kept(n)
        cos = torch.cat([torch.linspace(0.8, 0.74, high), torch.linspace(0.5, 0.7, mid), torch.linspace(0.0, 0.46, low)]).cuda()
        cos = cos[torch.rand(n, device="cuda", generator=gen).argsort()][:, None]
        along = q[b] / q[b].norm()
        c = torch.randn(n, EMBED_DIM, device="cuda", generator=gen)
        c -= (c @ along)[:, None] * along
        c /= c.norm(dim=1, keepdim=True)
        length = 10 + 20 * torch.rand(n, 1, device="cuda", generator=gen)
        parts.append(length * (cos * along + (1 - cos * cos).sqrt() * c))
    return q, torch.cat(parts), counts


def prepare(case, seed):
    dev = torch.device("cuda:0")
    state = {"case": case, "shape": _shape(case)}
    if case["kind"] == "request":
        gen = _generator(seed)
        state["kv"] = _keys_values(case, gen)
        state["emb"] = _embeddings(case, gen)
        return state
    k, v, q, new = _inputs(case, seed)
    bits = np.concatenate(_chunk_bits(case, seed)) if sum(_lengths(case)) >= case["chunk"] else np.zeros(0, np.uint8)
    capacity = (case["appended"] + 255) // 256 * 256 if case["kind"] == "append" else 0
    plan = ck.cocktail_plan(state["shape"], _lengths(case), bits, ck.cocktail_default_workers(state["shape"]),
                            append_capacity=capacity)
    cache = state["cache"] = ck.PackedCache(plan, dev)
    if case["kind"] == "prefill":
        state["kv"] = (k, v)
    elif case["kind"] == "paged":
        state["pages"] = _pages(case, k, v, _generator(seed + 1))
    else:
        _fill(cache, case, k, v)
        state["q"] = q
        if case["kind"] == "append":
            for i in range(case["appended"] - 1):
                ck.cocktail_append_fp16(cache, new[0, i], new[1, i])
            state["new"] = (new[0, -1].clone(), new[1, -1].clone())
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "request":
        q, c, counts = state["emb"]
        bits, scores = ck.cocktail_chunk_bitwidths(q, c, counts)
        plan = ck.cocktail_plan(state["shape"], _lengths(case), bits.cpu().numpy(),
                                ck.cocktail_default_workers(state["shape"]))
        cache = ck.PackedCache(plan, q.device)
        _fill(cache, case, *state["kv"])
        return {"scores": scores, "bits": bits, "perm": plan.perm, "k": cache.k, "v": cache.v}
    cache = state["cache"]
    if case["kind"] == "prefill":
        _fill(cache, case, *state["kv"])
        return {"k": cache.k, "v": cache.v}
    if case["kind"] == "paged":
        ck.cocktail_reorder_quantize_paged(cache, *state["pages"])
        return {"k": cache.k, "v": cache.v}
    if case["kind"] == "append":
        ck.cocktail_append_fp16(cache, *state["new"], position=case["appended"] - 1)
    out, lse = ck.cocktail_decode_attention(cache, state["q"])
    return {"out": out, "lse": lse}


def _packed_bytes(case):
    """K and V bytes of the packed cache: codes, and an fp16 scale and zero per group."""
    d, total = case["head_dim"], 0
    row = {b: d * b // 8 + (4 * d // case["group"] if b < 16 else 0) for b in BITS}
    for t in _lengths(case):
        chunks = t // case["chunk"]
        per = _kept(chunks) if case["kind"] == "request" else _class_chunks(case, chunks)
        total += sum(n * case["chunk"] * row[b] for n, b in zip(per, BITS)) + (t - chunks * case["chunk"]) * row[16]
    return 2 * case["kv_heads"] * total


def work(case):
    d, rows = case["head_dim"], sum(_lengths(case))
    packed, source = _packed_bytes(case), 4 * case["kv_heads"] * rows * d
    if case["kind"] in ("prefill", "paged"):
        return {"bytes": packed + source, "flops": 0}
    if case["kind"] == "request":
        chunks = sum(t // case["chunk"] for t in _lengths(case))
        return {"bytes": packed + source + 4 * EMBED_DIM * (chunks + case["batch"]) + 5 * chunks, "flops": 6 * EMBED_DIM * chunks}
    heads = case["batch"] * case["q_heads"]
    attended = rows + case["batch"] * case["appended"]
    return {"bytes": packed + 4 * case["batch"] * case["appended"] * case["kv_heads"] * d + heads * (4 * d + 4)
            + (4 * case["batch"] * case["kv_heads"] * d if case["kind"] == "append" else 0),
            "flops": 4 * attended * case["q_heads"] * d}


def tolerance(case):
    # the packed cache, the partition and the search results are integers and correctly rounded numbers
    if case["kind"] in ("prefill", "paged", "request"):
        return "exact"
    # measured against 64 bits: 2-norm 1.9e-4 to 2.6e-4, worst value 4e-4 to 1.2e-3 of the rms (`out` is rounded to fp16
    # after a sum whose weights may be fp16 operands)
    return {"rel": 1e-3, "max": 5e-3}


def _dequantized(x, bits, group):
    """x: fp16 [T, D], bits: per token.  The values of the packed cache in 64 bits."""
    t, d = x.shape
    g = x.float().view(t, d // group, group)
    mn, mx = g.amin(dim=2, keepdim=True), g.amax(dim=2, keepdim=True)
    qmax = (2.0 ** bits.double() - 1)[:, None, None]
    scale = ((mx - mn).double() / qmax).float().half()
    inv = torch.where(scale == 0, 0.0, (1.0 / scale.double()).float())
    code = torch.minimum(((g - mn) * inv).round().double(), qmax)
    deq = (mn.double() + code * scale.double()).view(t, d)
    return torch.where((bits == 16)[:, None], x.double(), deq)


def exact(case, seed):
    if case["kind"] in ("prefill", "paged"):
        return None
    if case["kind"] == "request":
        gen = _generator(seed)
        _keys_values(case, gen)
        q, c, counts = _embeddings(case, gen)
        q = q.double().repeat_interleave(torch.tensor(counts, device="cuda"), dim=0)
        scores = torch.nn.functional.cosine_similarity(q, c.double(), dim=1)
        return {"scores": scores, "bits": None, "perm": None, "k": None, "v": None}
    k, v, q, new = _inputs(case, seed)
    d, h = case["head_dim"], case["kv_heads"]
    rep = case["q_heads"] // h
    out = torch.empty(q.shape, dtype=torch.float64, device="cuda")
    lse = torch.empty(q.shape[:2], dtype=torch.float64, device="cuda")
    at = 0
    for b, (t, cb) in enumerate(zip(_lengths(case), _chunk_bits(case, seed))):
        bits = np.full(t, 16, dtype=np.int64)
        bits[:cb.size * case["chunk"]] = np.repeat(cb, case["chunk"])
        bits = torch.from_numpy(bits).cuda()
        for i in range(h):
            ks, vs = (_dequantized(x[at:at + t * d].view(t, d), bits, case["group"]) for x in (k, v))
            at += t * d
            ks, vs = torch.cat([ks, new[0, :, b, i].double()]), torch.cat([vs, new[1, :, b, i].double()])
            s = q[b, i * rep:(i + 1) * rep].double() @ ks.t() / math.sqrt(d)
            lse[b, i * rep:(i + 1) * rep] = torch.logsumexp(s, dim=1)
            out[b, i * rep:(i + 1) * rep] = torch.softmax(s, dim=1) @ vs
    return {"out": out, "lse": lse}

"""Performance cases: the work a user of this library has it do, and how one pass of each is run.

Four kinds of case, each through the public entry points of the package:

  extend    one serving step of one layer: cp_write_kv (append the new K/V to the paged cache), then
            cp_extend_attention (the new rows attend to the cached prefix and to their own keys)
  distance  cp_context_distance: all pairwise distances of n retrieved contexts
  index     a context index from a batch of retrievals: distinct contexts, GPU distances, clustering, aligned
            contexts, search paths, execution order
  dedup     the turns of one conversation through the de-duplication of retrieved text (host data)

listed() gives the fixed cases, draw() more of the same ranges.
"""
import itertools
import math
import random

import numpy as np
import torch

import paper_2511_03475_amd as cp

HEAD_DIM, PAGE = 128, 16
LARGEST_FLOPS = 1.41e14          # of one extend pass: the 128k-token prefill below
LARGEST_POOL_TOKENS = 400_000    # cached and new tokens of one extend pass
HEADS = ((8, 2), (32, 8), (64, 8))   # (query, KV) heads of the configurations and tests


def listed():
    return [
        # one short request on a small model: nothing but launches and latency
        extend("tiny_extend", 8, 2, 1, 512, 128),
        # retrieval-augmented batch: 6 of 8 context blocks of 1024 tokens cached, a 256-token question
        extend("rag_fixed", 32, 8, 8, 6144, 2304),
        # one layer of a large model at 32k context, three quarters of it cached
        extend("long_context_32k", 64, 8, 4, 24576, 8192),
        # a whole 128k-token prompt, nothing cached: the largest prefill
        extend("ctx128k_zero_reuse", 32, 8, 1, 0, 131072),
        # fully cached contexts, only the question is new: few rows over a long prefix
        extend("short_extend", 32, 8, 32, 10240, 128),
        # continuous batching: most requests decode one token, a few bring a chunk of their prompt;
        # lengths odd and ragged
        dict(name="mixed_batch", kind="extend", q_heads=32, kv_heads=8, batch=40, lens="mixed", lens_seed=11,
             max_prefix=12000, max_extend=2000, decoding=32),
        # decoding: one new token per request, bound by reading the cache once
        extend("decode_b32_p10k", 32, 8, 32, 10240, 1),
        # decoding a single long conversation: the cache of one request has to fill the device
        extend("decode_b1_p128k", 32, 8, 1, 131071, 1),
        # speculative decoding: 16 draft tokens per request are checked at once
        extend("decode_b32_p10k_e16", 32, 8, 32, 10240, 16),
        # distance matrix of a large batch of retrievals, top 15 of 2000 blocks
        dict(name="distance_n8192", kind="distance", n=8192, k_min=15, k_max=15, stride=16, blocks=2000),
        # context index of 2000 retrievals, from the block ids to the execution order
        dict(name="index_n2000", kind="index", n=2000, k_min=15, k_max=15, stride=16, blocks=2000),
        # 40 turns of one conversation, 12 retrieved text blocks each
        dict(name="dedup_40_turns", kind="dedup", turns=40, per_turn=12, blocks=200, lines=200, modulus=8),
    ]


def extend(name, q_heads, kv_heads, batch, prefix, new):
    """An extend case in which every request has the same lengths."""
    return dict(name=name, kind="extend", q_heads=q_heads, kv_heads=kv_heads, batch=batch, lens="equal",
                prefix=prefix, extend=new)


def log_int(rng, lo, hi):
    """Whole number from lo to hi, spread evenly over the logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    kind = rng.choice(("prefill", "prefill", "ragged", "mixed", "decode", "decode", "distance", "index", "dedup"))
    if kind == "distance":
        k = rng.randint(5, 15)
        return dict(kind="distance", n=log_int(rng, 200, 8192), k_min=rng.choice((k, 1)), k_max=k, stride=16,
                    blocks=log_int(rng, 500, 4000))
    if kind == "index":
        k = rng.randint(8, 15)
        return dict(kind="index", n=log_int(rng, 100, 2000), k_min=rng.choice((k, 4)), k_max=k, stride=16,
                    blocks=log_int(rng, 500, 4000))
    if kind == "dedup":
        return dict(kind="dedup", turns=rng.randint(2, 40), per_turn=rng.randint(3, 15), blocks=rng.randint(40, 300),
                    lines=log_int(rng, 20, 200), modulus=rng.choice((4, 8, 16)))
    while True:
        q_heads, kv_heads = rng.choice(HEADS)
        case = dict(kind="extend", q_heads=q_heads, kv_heads=kv_heads)
        if kind == "prefill":       # equal lengths, from a short question to a whole prompt
            new = log_int(rng, 100, 131072)
            prefix = rng.choice((0, log_int(rng, 100, 120000), log_int(rng, 100, 120000)))
            case.update(batch=log_int(rng, 1, 32), lens="equal", prefix=prefix, extend=new)
        elif kind == "ragged":      # every request with lengths of its own
            case.update(batch=log_int(rng, 3, 48), lens="ragged", lens_seed=rng.randrange(1 << 30),
                        max_prefix=log_int(rng, 500, 30000), max_extend=log_int(rng, 100, 10000))
        elif kind == "mixed":       # decoding requests next to chunks of prompts
            batch = rng.randint(4, 48)
            case.update(batch=batch, lens="mixed", lens_seed=rng.randrange(1 << 30),
                        max_prefix=log_int(rng, 500, 20000), max_extend=log_int(rng, 200, 4000),
                        decoding=batch - rng.randint(1, max(1, batch // 4)))
        else:                       # decoding, one token or a few drafts each
            case.update(batch=log_int(rng, 1, 64), lens="equal", prefix=log_int(rng, 100, 131071),
                        extend=rng.choice((1, 1, rng.randint(2, 16))))
        prefixes, extends = lengths(case)
        if sum(prefixes) + sum(extends) <= LARGEST_POOL_TOKENS and work(case)["flops"] <= LARGEST_FLOPS:
            return case


def lengths(case):
    """Cached and new tokens of every request."""
    n = case["batch"]
    if case["lens"] == "equal":
        return [case["prefix"]] * n, [case["extend"]] * n
    rng = random.Random(case["lens_seed"])
    prefixes = [log_int(rng, 50, case["max_prefix"]) for _ in range(n)]
    extends = [log_int(rng, 20, case["max_extend"]) for _ in range(n)]
    if case["lens"] == "mixed":
        extends = [1 if i < case["decoding"] else e for i, e in enumerate(extends)]
        both = list(zip(prefixes, extends))
        rng.shuffle(both)
        prefixes, extends = [p for p, _ in both], [e for _, e in both]
    return prefixes, extends


def work(case):
    if case["kind"] == "extend":
        prefixes, extends = lengths(case)
        new, cached = sum(extends), sum(prefixes)
        pairs = sum(e * p + e * (e + 1) // 2 for p, e in zip(prefixes, extends))
        row = HEAD_DIM * 2
        # query and result, new K and V in and into the cache, cached K and V
        return {"bytes": row * (2 * new * case["q_heads"] + 2 * case["kv_heads"] * (2 * new + cached)),
                "flops": 4.0 * HEAD_DIM * case["q_heads"] * pairs}
    if case["kind"] == "dedup":
        # the text of all turns is read once (about 45 bytes a line)
        return {"bytes": case["turns"] * min(case["per_turn"], case["blocks"]) * case["lines"] * 45, "flops": 0}
    n = case["n"]
    # ids in, every distance out once; for the index also once through the clustering
    if case["kind"] == "distance":
        return {"bytes": 4 * n * case["stride"] + 4 * n * n, "flops": 0}
    return {"bytes": 4 * n * case["stride"] + 2 * 4 * n * n, "flops": 0}


def tolerance(case):
    if case["kind"] == "extend":
        # bf16 query, probabilities and result: 0.0021-0.0029 (largest 0.04) from fp64, of which rounding the
        # result alone makes 0.0017.  The whole values are the bits of the cache.
        return {"rel": 1e-2, "max": 0.2}
    if case["kind"] == "distance":
        # exact integers, combined in three 32-bit operations: 2.2e-8 (largest 6.9e-8) from fp64
        return {"rel": 1e-7, "max": 4e-7}
    return "exact"


def normal(g, *shape):
    """N(0, 1) rounded once to bf16."""
    out = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    flat, step = out.view(-1), 1 << 27
    for at in range(0, flat.numel(), step):
        part = flat[at:at + step]
        part.copy_(torch.randn(part.numel(), generator=g, device="cuda"))
    return out


def contexts(case, seed):
    """Retrieved block ids in rank order, drawn without replacement with weight rank^-1.1."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    weight = -1.1 * torch.log(torch.arange(1, case["blocks"] + 1, device="cuda", dtype=torch.float64))
    ids = []
    for at in range(0, case["n"], 2048):
        u = torch.rand((min(2048, case["n"] - at), case["blocks"]), generator=g, device="cuda", dtype=torch.float64)
        ids.append(torch.topk(weight - torch.log(-torch.log(u.clamp_min(1e-300))), case["k_max"], dim=1).indices)
    ids = torch.cat(ids).to(torch.int32)
    lens = torch.randint(case["k_min"], case["k_max"] + 1, (case["n"],), generator=g, device="cuda", dtype=torch.int32)
    out = torch.full((case["n"], case["stride"]), -1, dtype=torch.int32, device="cuda")
    out[:, :case["k_max"]] = torch.where(torch.arange(case["k_max"], device="cuda") < lens[:, None], ids, -1)
    return out, lens


def conversation(case, seed):
    """Text blocks whose lines are random words, with sections that several blocks share, and the
    blocks that each turn retrieves (heavy-tailed popularity)."""
    rng = np.random.default_rng(seed)
    letters = np.frombuffer(b"abcdefghijklmnopqrstuvwxyz", dtype=np.uint8)
    words = [letters[rng.integers(0, 26, size=n)].tobytes() for n in rng.integers(2, 10, size=4000)]

    def text_lines(count):
        counts = rng.integers(4, 13, size=count)
        pick = iter(rng.integers(0, len(words), size=int(counts.sum())).tolist())
        return [b" ".join(words[w] for w in itertools.islice(pick, int(c))) + b"\n" for c in counts]

    sections = [text_lines(int(n)) for n in rng.integers(3, 9, size=10)]
    blocks = []
    for b in range(case["blocks"]):
        own, lines = text_lines(case["lines"]), []
        while len(lines) < case["lines"]:
            if rng.random() < 0.09:
                lines += sections[int(rng.integers(0, len(sections)))]
            else:
                lines.append(own[len(lines)])
        text = b"".join(lines)
        blocks.append(text[:-1] if b % 3 == 0 else text)   # some end without a newline
    p = np.arange(1, case["blocks"] + 1) ** -1.1
    size = min(case["per_turn"], case["blocks"])
    turns = [rng.choice(case["blocks"], size=size, replace=False, p=p / p.sum()).tolist() for _ in range(case["turns"])]
    return [(ids, [blocks[i] for i in ids]) for ids in turns]


def prepare(case, seed):
    if case["kind"] == "dedup":
        return {"kind": "dedup", "turns": conversation(case, seed), "modulus": case["modulus"],
                "room": 3 * case["turns"] * case["per_turn"] * (case["lines"] // 2 + 16)}
    if case["kind"] == "index":      # block ids come from the retriever, in host memory
        ids, lens = contexts(case, seed)
        return {"kind": "index", "ids": ids.cpu().numpy(), "lens": lens.cpu().numpy()}
    if case["kind"] == "distance":
        ids, lens = contexts(case, seed)
        n = case["n"]
        return {"kind": "distance", "ids": ids, "lens": lens, "n": n, "stride": case["stride"],
                "dist": torch.empty((n, n), dtype=torch.float32, device="cuda")}
    g = torch.Generator(device="cuda").manual_seed(seed)
    q_heads, kv_heads = case["q_heads"], case["kv_heads"]
    prefixes, extends = lengths(case)
    pages = [(p + e + PAGE - 1) // PAGE for p, e in zip(prefixes, extends)]
    total, new = sum(pages), sum(extends)
    places = np.random.default_rng(seed).permutation(total)   # pages anywhere in the pool
    table = np.full((case["batch"], max(pages)), -1, dtype=np.int32)
    at = 0
    for r, n in enumerate(pages):
        table[r, :n] = places[at:at + n]
        at += n
    shape = cp.Shape(case["batch"], q_heads, kv_heads, HEAD_DIM, PAGE, total, max(pages), prefixes, extends,
                     1.0 / math.sqrt(HEAD_DIM))
    size = cp.cp_workspace_bytes(shape)
    q = normal(g, new, q_heads, HEAD_DIM)
    as_device = lambda a: torch.tensor(a, dtype=torch.int32, device="cuda")  # noqa: E731
    return {"kind": "extend", "q": q, "k": normal(g, new, kv_heads, HEAD_DIM), "v": normal(g, new, kv_heads, HEAD_DIM),
            "pool": normal(g, total, 2, kv_heads, PAGE, HEAD_DIM), "out": torch.empty_like(q), "shape": shape,
            "table": torch.from_numpy(table).cuda(), "prefix": as_device(prefixes), "extend": as_device(extends),
            "space": torch.empty(max(size, 256), dtype=torch.uint8, device="cuda"), "size": size}


def run(state):
    if state["kind"] == "extend":
        s, stream = state, torch.cuda.current_stream()
        cp.cp_write_kv(s["k"], s["v"], s["pool"], s["table"], s["prefix"], s["extend"], stream, s["shape"])
        cp.cp_extend_attention(s["q"], s["k"], s["v"], s["pool"], s["table"], s["prefix"], s["extend"], s["out"],
                               stream, s["shape"], s["space"], s["size"])
        return {"out": s["out"], "cache": s["pool"].view(torch.int16)}
    if state["kind"] == "distance":
        s = state
        cp.cp_context_distance(s["ids"], s["lens"], s["n"], s["stride"], 0.001, s["dist"], torch.cuda.current_stream())
        return {"dist": s["dist"]}
    if state["kind"] == "index":
        return index_pass(state["ids"], state["lens"])
    talk, kept, found = cp.Conversation(state["modulus"]), [], []
    for ids, texts in state["turns"]:
        parts, n = talk.turn(ids, texts)
        kept.append(n)
        found.append(parts)
    talk.close()
    # -2: the whole block is a reference; otherwise begin, end and referenced block of each piece
    flat = [x for parts in found for what, x in parts for x in ((-2,) if what == "block" else itertools.chain(*x))]
    return {"kept": np.array(kept, dtype=np.int64), "pieces": padded(flat, state["room"])}


def padded(values, room):
    """The values in an array whose size does not depend on the seed."""
    out = np.full(max(room, len(values)), -3, dtype=np.int32)
    out[:len(values)] = values
    return out


def index_pass(ids, lens):
    n, stride = ids.shape
    first_of, m = cp.cp_index_distinct(ids, lens)
    rows = np.zeros(m, np.int64)
    rows[first_of[::-1]] = np.arange(n)[::-1]      # first row of every distinct context
    device_ids, device_lens = torch.from_numpy(ids[rows]).cuda(), torch.from_numpy(lens[rows]).cuda()
    dist = torch.empty((m, m), dtype=torch.float32, device="cuda")
    cp.cp_context_distance(device_ids, device_lens, m, stride, 0.001, dist, torch.cuda.current_stream())
    index = cp.ContextIndex(ids, lens, 0.001, dist=dist.cpu().numpy())
    paths = [index.path(i) for i in range(n)]
    aligned = [index.aligned(i) for i in range(n)]
    order = cp.cp_index_schedule(paths)
    index.close()
    return {"order": np.array(order, dtype=np.int32), "aligned": padded(list(itertools.chain(*aligned)), n * stride),
            "paths": padded(list(itertools.chain(*paths)), n * 128),
            "depths": np.array([len(p) for p in paths], dtype=np.int32)}

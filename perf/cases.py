"""The work a user of this library has it do, as measured cases.

A serving program builds the index of its stores (one large common store,
project stores of every size, growing project stores), then drafts at every
decoding step: it retrieves the continuations of each sequence's context from
the stores, folds them into a draft tree and accepts the longest path; the
target model's attention over that tree is the library's too.  Batches run
from one sequence (the paper decodes at batch size 1) to a full serving batch.

Each case is one kind of call at one size; draw() gives more sizes of the same
kinds.  Stores are seeded stand-ins for code: template n-grams drawn with Zipf
reuse, 10% of the tokens replaced at random, files of 500 tokens joined by 0.
"""
from __future__ import annotations

import numpy as np
import torch

import paper_2502_17139_amd as fc

VOCAB = 32256
FILE_LEN = 500
NOISE = 0.1
CTX_LEN = 16
N_MAX, N_MIN = 16, 2
HEAD_DIM = fc.FC_TREE_ATTN_HEAD_DIM


# ------------------------------------------------------------------ cases --

def listed() -> list:
    return [
        # drafting, one step of a full serving batch on the largest stores:
        # retrieval, tree, acceptance (the benchmark's headline workload)
        dict(name="draft_1024_on_1B", kind="draft", batch=1024, project=10_000_000, general=1_000_000_000,
             tables="records", k=5000, m=10, c=64, alpha=1),
        # the same step of a medium batch on a project and a mid-sized common store
        dict(name="draft_256_on_100M", kind="draft", batch=256, project=2_000_000, general=100_000_000,
             tables="records", k=5000, m=10, c=64, alpha=1),
        # one sequence being decoded: the smallest call, where latency counts
        dict(name="draft_1_on_10M", kind="draft", batch=1, project=1_000_000, general=10_000_000, tables="records",
             k=5000, m=10, c=64, alpha=1),
        # stores as Store(tokens) makes them, without the optional tables (a
        # project store rebuilt often is not worth a 4 GB table), odd sizes,
        # longer continuations, a weight per store
        dict(name="draft_77_no_tables", kind="draft", batch=77, project=333_333, general=30_000_001, tables="none",
             k=1500, m=16, c=48, alpha=2),
        # decode-trace replay with the CACHE: every per-step decision on the GPU
        dict(name="replay_128_cache", kind="replay", streams=128, length=2048, steps=64, project=2_000_000,
             general=50_000_000, k=5000, m=10, c=64, cache=20),
        # index of the common store, built offline
        dict(name="index_1B", kind="build", n=1_000_000_000, templates=2_000_000, zipf=1.1),
        # index of one large project store
        dict(name="index_10M", kind="build", n=10_019_999, templates=2_000, zipf=1.2),
        # one index per repository, all in one call
        dict(name="index_64_repos", kind="repos", repos=64, min_files=20, max_files=4000),
        # a project store that grows by the files just written
        dict(name="extend_10M_by_20_files", kind="extend", n_old=10_000_000, new_files=20, keep_inverse=True),
        # the optional tables of a store (first token, two tokens, records, sample)
        dict(name="tables_100M", kind="tables", n=100_000_000, vocab=VOCAB),
        # the target model's attention over a batch of trees
        dict(name="attention_64_trees", kind="attention", batch=64, rows=65, heads=32, kv_heads=32, prefix=2048,
             ragged=False),
        # and over the one tree of a single decoded sequence, grouped key heads
        dict(name="attention_1_tree", kind="attention", batch=1, rows=65, heads=32, kv_heads=8, prefix=3000,
             ragged=True),
    ]


def _log_int(rng, lo: int, hi: int) -> int:
    """An integer spread evenly over the logarithm of [lo, hi]."""
    return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng) -> dict:
    kind = rng.choice(["draft", "draft", "draft", "replay", "build", "build", "repos", "extend", "tables", "attention",
                       "attention"])
    if kind == "draft":
        k = rng.choice([500, 1000, 1501, 3000, 5000])
        return dict(kind=kind, batch=_log_int(rng, 1, 1024), project=_log_int(rng, 50_000, 10_000_000),
                    general=_log_int(rng, 1_000_000, 100_000_000), tables=rng.choice(["records", "records", "none"]),
                    k=k, m=rng.choice([10, 8, 5]) if k > 3000 else rng.choice([10, 7, 16]),
                    c=rng.choice([64, 32, 48, 100]), alpha=rng.choice([1, 1, 2]))
    if kind == "replay":
        return dict(kind=kind, streams=_log_int(rng, 4, 128), length=2048, steps=rng.randint(16, 64),
                    project=_log_int(rng, 100_000, 5_000_000), general=_log_int(rng, 1_000_000, 50_000_000), k=5000,
                    m=10, c=64, cache=rng.choice([-1, 5, 20]))
    if kind == "build":
        n = _log_int(rng, 20_000, 200_000_000)
        return dict(kind=kind, n=n, templates=max(100, n // rng.choice([500, 5000])), zipf=rng.choice([1.1, 1.2]))
    if kind == "repos":
        return dict(kind=kind, repos=_log_int(rng, 3, 128), min_files=rng.randint(1, 30),
                    max_files=_log_int(rng, 100, 4000))
    if kind == "extend":
        return dict(kind=kind, n_old=_log_int(rng, 100_000, 50_000_000), new_files=_log_int(rng, 1, 400),
                    keep_inverse=rng.random() < 0.7)
    if kind == "tables":
        return dict(kind=kind, n=_log_int(rng, 200_000, 100_000_000), vocab=rng.choice([VOCAB, 16_000, 8_191]))
    heads = rng.choice([16, 32, 40])
    return dict(kind=kind, batch=_log_int(rng, 1, 48), rows=rng.choice([65, 65, 33, 49, 101]), heads=heads,
                kv_heads=rng.choice([heads, heads, 8]), prefix=_log_int(rng, 100, 4096), ragged=rng.random() < 0.6)


# ----------------------------------------------------------------- inputs --

def _gen(seed: int, role: int) -> torch.Generator:
    g = torch.Generator(device="cuda")
    g.manual_seed((seed * 1_000_003 + role) & 0x7FFFFFFFFFFF)
    return g


class _Pool:
    """Templates of 4 to 32 tokens and their Zipf table."""

    def __init__(self, seed: int, role: int, templates: int, zipf: float, vocab: int = VOCAB):
        g = _gen(seed, role)
        self.vocab = vocab
        self.len = torch.randint(4, 33, (templates,), generator=g, device="cuda")
        self.off = torch.cumsum(self.len, 0) - self.len
        total = int(self.off[-1] + self.len[-1])
        self.tok = torch.randint(1, vocab, (total,), generator=g, device="cuda", dtype=torch.int32)
        w = torch.arange(1, templates + 1, dtype=torch.float64).pow(-zipf)
        cum = torch.cumsum(w, 0)
        self.cum = (cum / cum[-1]).cuda()

    def text(self, g: torch.Generator, n: int) -> torch.Tensor:
        """n tokens (uint16): templates one after another, noise, a 0 after every FILE_LEN tokens."""
        out = torch.empty(n, dtype=torch.int16, device="cuda")
        step = 1 << 25
        for a in range(0, n, step):
            c = min(step, n - a)
            draws = c // 16 + 64
            while True:
                u = torch.rand(draws, generator=g, device="cuda", dtype=torch.float64)
                t = torch.searchsorted(self.cum, u).clamp_(max=self.len.numel() - 1)
                ln = self.len[t]
                end = torch.cumsum(ln, 0)
                if int(end[-1]) >= c:
                    break
                draws *= 2
            src = torch.repeat_interleave(self.off[t] - (end - ln), ln)[:c] + torch.arange(c, device="cuda")
            tok = self.tok[src]
            noise = torch.rand(c, generator=g, device="cuda") < NOISE
            tok = torch.where(noise, torch.randint(1, self.vocab, (c,), generator=g, device="cuda",
                                                   dtype=torch.int32), tok)
            out[a:a + c] = tok.to(torch.int16)
        out[FILE_LEN::FILE_LEN + 1] = 0
        return out.view(torch.uint16)


def _windows(text: torch.Tensor, count: int, g: torch.Generator) -> torch.Tensor:
    """count windows of CTX_LEN tokens at random places inside files (int16)."""
    files = max(1, text.numel() // (FILE_LEN + 1))
    room = min(FILE_LEN, text.numel()) - CTX_LEN
    at = (torch.randint(0, files, (count,), generator=g, device="cuda") * (FILE_LEN + 1) +
          torch.randint(0, room + 1, (count,), generator=g, device="cuda"))
    return text.view(torch.int16)[at[:, None] + torch.arange(CTX_LEN, device="cuda")]


def _two_stores(case, seed):
    """Project and common store with their pools (the common one far more varied)."""
    pools = (_Pool(seed, 1, max(100, case["project"] // 5000), 1.2), _Pool(seed, 2, max(1000, case["general"] // 500), 1.1))
    texts = [p.text(_gen(seed, 10 + i), n) for i, (p, n) in enumerate(zip(pools, (case["project"], case["general"])))]
    return pools, texts


def _stores(texts, tables: str):
    if tables == "none":
        return [fc.Store(t) for t in texts]
    return [fc.Store(t, pair_vocab=VOCAB, records=True) for t in texts]


def _contexts(pools, texts, batch: int, seed: int) -> torch.Tensor:
    """70% of the contexts from the project's code, the rest from the common store's; half are windows of the stores
    themselves and half unseen text of the same kind."""
    g = _gen(seed, 20)
    parts = []
    for i, share in ((0, (batch * 7 + 9) // 10), (1, batch - (batch * 7 + 9) // 10)):
        seen = (share + 1) // 2
        if seen:
            parts.append(_windows(texts[i], seen, g))
        if share - seen:
            fresh = pools[i].text(_gen(seed, 30 + i), max(FILE_LEN, (share - seen) * (FILE_LEN + 1)))
            parts.append(_windows(fresh, share - seen, g))
    ctx = torch.cat(parts)
    ctx = ctx[torch.randperm(batch, generator=g, device="cuda")]
    return ctx.contiguous().view(torch.uint16)


_SIGNED = {torch.uint16: torch.int16, torch.uint32: torch.int32}


def _clear(outputs: dict) -> dict:
    """Output buffers as a program keeps them, zeroed once: slots past a query's kept ones are never written."""
    for t in outputs.values():
        t.view(_SIGNED.get(t.dtype, t.dtype)).zero_()
    return outputs


def _plain(*outputs: dict) -> dict:
    """The buffers of all calls under one roof, unsigned words shown as signed ones (the same bits)."""
    return {f: t.view(_SIGNED.get(t.dtype, t.dtype)) for o in outputs for f, t in o.items()}


def _random_trees(batch: int, rows: int, seed: int) -> dict:
    """Draft trees of 3/4 to all of `rows` rows in preorder, at most 10 deep: num_nodes, pos_ids, mask."""
    r = np.random.RandomState(seed & 0x7FFFFFFF)
    nodes = r.randint(max(1, rows * 3 // 4), rows + 1, batch).astype(np.int32)
    depth = np.zeros((batch, rows), np.int32)
    mask = np.zeros((batch, rows, rows), np.int32)
    path = np.zeros((batch, 11), np.int64)  # the current row at each depth
    every = np.arange(batch)
    mask[:, 0, 0] = 1
    for i in range(1, rows):
        d = 1 + (r.random_sample(batch) * np.minimum(depth[:, i - 1] + 1, 10)).astype(np.int64)
        mask[:, i] = mask[every, path[every, d - 1]]
        mask[:, i, i] = 1
        depth[:, i] = d
        path[every, d] = i
    past = np.arange(rows)[None, :] >= nodes[:, None]
    depth[past] = 0
    mask[past] = 0
    return dict(num_nodes=torch.from_numpy(nodes).cuda(), pos_ids=torch.from_numpy(depth).cuda(),
                mask=torch.from_numpy(mask).cuda())


# ---------------------------------------------------------------- prepare --

def _prepare_draft(case, seed):
    pools, texts = _two_stores(case, seed)
    ctx = _contexts(pools, texts, case["batch"], seed)
    stores = _stores(texts, case["tables"])
    B, S, k, m, c = case["batch"], 2, case["k"], case["m"], case["c"]
    s = dict(kind="draft", stores=stores, ctx=ctx, k=k, m=m, c=c, alpha=(case["alpha"], 1))
    s["r"] = _clear(fc.retrieve_outputs(B, S, k, m, "cuda"))
    s["t"] = _clear(fc.tree_outputs(B, c, "cuda"))
    s["a"] = _clear(fc.accept_outputs(B, m, "cuda"))
    s["rws"] = torch.empty(fc.fc_retrieve_workspace_bytes(B, S, N_MAX, N_MIN, k, m), dtype=torch.uint8, device="cuda")
    s["tws"] = torch.empty(max(fc.fc_build_tree_workspace_bytes(B), 1), dtype=torch.uint8, device="cuda")
    # what the target model answers after each row: the text that a sequence goes on with, here a file of its pool
    truth = pools[0].text(_gen(seed, 40), B * 64).view(B, 64)
    s["target"] = torch.empty((B, c + 1), dtype=torch.int32, device="cuda")
    _draft(s)
    # half of the sequences go on along the first path of their tree, the others with unseen text
    start = torch.zeros(B, dtype=torch.int32, device="cuda")
    fc.fc_targets_from_truth(truth, start, s["t"], out=s["target"])
    par, tok = s["t"]["parent"].to(torch.int64), s["t"]["node_tok"]
    rows = torch.arange(c + 1, device="cuda").expand(B, c + 1)
    first = torch.full((B, c + 2), c + 1, dtype=torch.int64, device="cuda")
    first.scatter_reduce_(1, torch.where(par >= 0, par, c + 1), rows, "amin")
    child = first[:, :c + 1]
    follow = torch.where(child <= c, torch.gather(tok, 1, child.clamp(max=c)), s["target"])
    s["target"][::2] = follow[::2]
    s["result"] = _plain(s["r"], s["t"], s["a"])
    return s


def _prepare_replay(case, seed):
    pools, texts = _two_stores(case, seed)
    stores = _stores(texts, "records")
    files = -(-case["length"] // FILE_LEN)
    n = case["streams"] * files * (FILE_LEN + 1)
    truth = pools[0].text(_gen(seed, 50), n + 1).view(torch.int16)[:n].view(-1, FILE_LEN + 1)
    # streams are files without their separators
    truth = truth[:, :FILE_LEN].clamp(min=1).reshape(case["streams"], -1)[:, :case["length"]]
    engine = fc.ReplayEngine(stores, truth.contiguous().view(torch.uint16), n_max=N_MAX, n_min=N_MIN, k=case["k"],
                             m=case["m"], c=case["c"], alpha=(1, 1), lru=32, ctx_len=CTX_LEN,
                             max_steps=case["steps"], cache_l=None if case["cache"] < 0 else case["cache"])
    return dict(kind="replay", engine=engine, steps=case["steps"])


def _prepare_build(case, seed):
    n = case["n"]
    tokens = _Pool(seed, 1, case["templates"], case["zipf"]).text(_gen(seed, 10), n)
    ws = torch.empty(fc.fc_datastore_build_workspace_bytes(n), dtype=torch.uint8, device="cuda")
    sa = torch.zeros(n, dtype=torch.int32, device="cuda").view(torch.uint32)
    return dict(kind="build", tokens=tokens, sa=sa, ws=ws, result=sa.view(torch.int32))


def _prepare_repos(case, seed):
    r = np.random.RandomState(seed & 0x7FFFFFFF)
    # sizes spread evenly over their logarithm, in any order
    files = r.permutation(np.exp(np.linspace(np.log(case["min_files"]), np.log(case["max_files"]),
                                             case["repos"])).round().astype(np.int64))
    off = np.zeros(case["repos"] + 1, np.uint64)
    off[1:] = np.cumsum(files * (FILE_LEN + 1) - 1)
    n = int(off[-1])
    # repositories share a template pool (common library code); each ends without a separator
    flat = _Pool(seed, 1, 2000, 1.2).text(_gen(seed, 10), int(files.sum()) * (FILE_LEN + 1)).view(torch.int16)
    keep = torch.ones(flat.numel(), dtype=torch.bool, device="cuda")
    keep[torch.from_numpy(np.cumsum(files) * (FILE_LEN + 1) - 1).cuda()] = False
    tokens = flat[keep].contiguous().view(torch.uint16)
    ws = torch.empty(fc.fc_datastore_build_batched_workspace_bytes(n, case["repos"]), dtype=torch.uint8, device="cuda")
    sa = torch.zeros(n, dtype=torch.int32, device="cuda").view(torch.uint32)
    return dict(kind="repos", tokens=tokens, off=off, sa=sa, ws=ws, result=sa.view(torch.int32))


def _prepare_extend(case, seed):
    n_new = case["new_files"] * (FILE_LEN + 1)
    n = case["n_old"] + n_new
    tokens = _Pool(seed, 1, max(100, case["n_old"] // 5000), 1.2).text(_gen(seed, 10), n)
    old_sa = fc.fc_datastore_build(tokens[n_new:].clone())
    old_isa = None
    if case["keep_inverse"]:
        inv = torch.empty(case["n_old"], dtype=torch.int32, device="cuda")
        inv[old_sa.view(torch.int32).to(torch.int64)] = torch.arange(case["n_old"], dtype=torch.int32, device="cuda")
        old_isa = inv.view(torch.uint32)
    ws = torch.empty(fc.fc_datastore_extend_workspace_bytes(n, n_new, case["keep_inverse"]), dtype=torch.uint8,
                     device="cuda")
    new = lambda: torch.zeros(n, dtype=torch.int32, device="cuda").view(torch.uint32)  # noqa: E731
    s = dict(kind="extend", tokens=tokens, n_new=n_new, old_sa=old_sa, old_isa=old_isa, sa=new(),
             isa=new() if case["keep_inverse"] else None, ws=ws)
    s["result"] = [t.view(torch.int32) for t in (s["sa"], s["isa"]) if t is not None]
    return s


def _prepare_tables(case, seed):
    n, V = case["n"], case["vocab"]
    tokens = _Pool(seed, 1, max(100, n // 500), 1.1, V).text(_gen(seed, 10), n)
    sa = fc.fc_datastore_build(tokens)
    u32 = lambda size: torch.zeros(size, dtype=torch.int32, device="cuda").view(torch.uint32)  # noqa: E731
    s = dict(kind="tables", tokens=tokens, sa=sa, n=n, vocab=V, bucket=u32(fc.FC_BUCKETS),
             pair=u32(fc.fc_pair_table_entries(V)),
             rec=torch.zeros(fc.fc_record_bytes(n), dtype=torch.uint8, device="cuda"),
             top=torch.zeros(-(-n // 256) * 32, dtype=torch.uint8, device="cuda"))
    s["result"] = [s["bucket"].view(torch.int32), s["pair"].view(torch.int32), s["rec"].view(torch.int32),
                   s["top"].view(torch.int32)]
    return s


def _attention_inputs(case, seed):
    B, R, H, Hkv, P = (case[f] for f in ("batch", "rows", "heads", "kv_heads", "prefix"))
    g = _gen(seed, 60)
    # projections of normalised activations: about normal; queries sharp enough that some keys dominate
    rnd = lambda *shape: torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32).to(torch.bfloat16)  # noqa: E731
    s = dict(q=rnd(B, R, H, HEAD_DIM), k_tree=rnd(B, R, Hkv, HEAD_DIM), v_tree=rnd(B, R, Hkv, HEAD_DIM),
             k_cache=rnd(B, P, Hkv, HEAD_DIM), v_cache=rnd(B, P, Hkv, HEAD_DIM))
    if case["ragged"]:
        s["prefix_len"] = torch.randint(P * 3 // 4, P + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
    else:
        s["prefix_len"] = torch.full((B,), P, dtype=torch.int32, device="cuda")
    s["tree"] = _random_trees(B, R, seed)
    return s


def _prepare_attention(case, seed):
    s = _attention_inputs(case, seed)
    return dict(kind="attention", out=torch.zeros(s["q"].shape, dtype=torch.float32, device="cuda"), **s)


def prepare(case: dict, seed: int):
    return globals()["_prepare_" + case["kind"]](case, seed)


# -------------------------------------------------------------------- run --

def _draft(s):
    r = fc.fc_retrieve(s["stores"], s["ctx"], n_max=N_MAX, n_min=N_MIN, k=s["k"], m=s["m"], out=s["r"],
                       workspace=s["rws"])
    t = fc.fc_build_tree(r["taken"], r["cont_len"], r["cont_tok"], s["ctx"], c=s["c"], alpha=s["alpha"], out=s["t"],
                         workspace=s["tws"])
    fc.fc_verify_accept(t, s["target"], m=s["m"], out=s["a"])
    return s.get("result")


def run(s):
    kind = s["kind"]
    if kind == "draft":
        return _draft(s)
    if kind == "replay":
        engine = s["engine"]
        out = engine.run(limit=s["steps"])
        out.update({f: engine.t[f].view(_SIGNED.get(engine.t[f].dtype, engine.t[f].dtype))
                    for f in fc.TREE_FIELDS + fc.ACCEPT_FIELDS})  # the last step's trees and accepted paths
        return out
    if kind == "build":
        fc.fc_datastore_build(s["tokens"], sa_out=s["sa"], workspace=s["ws"])
    elif kind == "repos":
        fc.fc_datastore_build_batched(s["tokens"], s["off"], sa_out=s["sa"], workspace=s["ws"])
    elif kind == "extend":
        fc.fc_datastore_extend(s["tokens"], s["n_new"], s["old_sa"], s["old_isa"], sa_out=s["sa"], isa_out=s["isa"],
                               workspace=s["ws"])
    elif kind == "tables":
        fc.fc_store_prepare(s["tokens"], s["sa"], bucket_out=s["bucket"])
        fc.fc_store_prepare_pairs(s["tokens"], s["sa"], s["vocab"], pair_out=s["pair"])
        fc.fc_store_prepare_records(s["tokens"], s["sa"], rec_out=s["rec"])
        fc.fc_store_prepare_top(s["rec"], s["n"], top_out=s["top"])
    else:
        return fc.fc_tree_attention(s["q"], s["k_tree"], s["v_tree"], s["k_cache"], s["v_cache"], s["prefix_len"],
                                    s["tree"], out=s["out"])
    return s["result"]


# ------------------------------------------------------------------- work --

def _draft_bytes(batch: int, k: int, m: int, c: int) -> float:
    """One step: the context and ranges, the kept slots (about a fifth of the cap on average: few contexts are as
    frequent as the cap allows) read from the store, written, read by the tree; the tree's rows and mask; the accepted
    path."""
    kept = 0.2 * k
    return batch * (2 * CTX_LEN + 32 + kept * (4 + 2 * m) + kept * (6 + 2 * m) + kept * (1 + 2 * m) + 8 +
                    16 * (c + 1) + 4 * (c + 1) ** 2 + 4 * (c + 1) + 4 * (m + 3))


def work(case: dict) -> dict:
    kind = case["kind"]
    if kind == "draft":
        return {"bytes": _draft_bytes(case["batch"], case["k"], case["m"], case["c"]), "flops": 0}
    if kind == "replay":
        return {"bytes": case["steps"] * _draft_bytes(case["streams"], case["k"], case["m"], case["c"]), "flops": 0}
    if kind == "build":
        return {"bytes": 6.0 * case["n"], "flops": 0}
    if kind == "repos":
        mean = (case["max_files"] - case["min_files"]) / np.log(case["max_files"] / case["min_files"])
        return {"bytes": 6.0 * case["repos"] * float(mean) * (FILE_LEN + 1), "flops": 0}
    if kind == "extend":
        n = case["n_old"] + case["new_files"] * (FILE_LEN + 1)
        return {"bytes": (16.0 if case["keep_inverse"] else 8.0) * n + 2.0 * n, "flops": 0}
    if kind == "tables":
        n = case["n"]
        return {"bytes": 6.0 * n + 4.0 * fc.FC_BUCKETS + 4.0 * case["vocab"] * (case["vocab"] + 1) + 64.0 * n + n / 8,
                "flops": 0}
    B, R, H, Hkv, P = (case[f] for f in ("batch", "rows", "heads", "kv_heads", "prefix"))
    P = P * (0.875 if case["ragged"] else 1.0)
    n = R * 0.875
    byts = B * (R * H * HEAD_DIM * 6 + (P + n) * Hkv * HEAD_DIM * 4 + 4 * R * R + 4 * R)
    return {"bytes": byts, "flops": 4.0 * B * H * n * (P + n) * HEAD_DIM}


# -------------------------------------------------------------- tolerance --

def tolerance(case: dict):
    if case["kind"] != "attention":
        return "exact"  # whole numbers throughout
    # bf16 products (rotated queries and keys and the weights rounded to 8 bits of mantissa), 32-bit sums
    return {"rel": 1e-2, "max": 0.1}


def exact(case: dict, seed: int):
    if case["kind"] != "attention":
        return None
    s = _attention_inputs(case, seed)
    B, R, H, D = s["q"].shape
    Hkv = s["k_tree"].shape[2]
    n_of, p_of = s["tree"]["num_nodes"].tolist(), s["prefix_len"].tolist()
    inv = 10000.0 ** (-2.0 * torch.arange(D // 2, dtype=torch.float64, device="cuda") / D)

    def rotate(x, pos):  # [rows][heads][D]
        ang = pos.to(torch.float64)[:, None] * inv
        co, si = ang.cos()[:, None, :], ang.sin()[:, None, :]
        a, b = x[..., :D // 2], x[..., D // 2:]
        return torch.cat([a * co - b * si, b * co + a * si], -1)

    out = torch.zeros((B, R, H, D), dtype=torch.float64, device="cuda")
    for b in range(B):
        n, p = n_of[b], p_of[b]
        pos = p + s["tree"]["pos_ids"][b, :n]
        q = rotate(s["q"][b, :n].double(), pos)
        kk = torch.cat([s["k_cache"][b, :p].double(), rotate(s["k_tree"][b, :n].double(), pos)])
        vv = torch.cat([s["v_cache"][b, :p], s["v_tree"][b, :n]]).double()
        hidden = torch.cat([torch.zeros((n, p), dtype=torch.bool, device="cuda"), s["tree"]["mask"][b, :n, :n] != 1], 1)
        for g in range(Hkv):
            qg = q[:, g * (H // Hkv):(g + 1) * (H // Hkv)].permute(1, 0, 2).reshape(-1, D)
            sc = (qg @ kk[:, g].t().contiguous()) / D ** 0.5
            sc = sc.view(H // Hkv, n, p + n).masked_fill(hidden, float("-inf"))
            og = torch.softmax(sc, -1).reshape(-1, p + n) @ vv[:, g].contiguous()
            out[b, :n, g * (H // Hkv):(g + 1) * (H // Hkv)] = og.view(H // Hkv, n, D).permute(1, 0, 2)
    return out

"""The calls a program makes of this library, sized as its users size them, for timing.

Every case is one pass through the public entry points (the C ABI of include/copse.h through the
`paper_2104_09583_amd.copse` binding):

  evaluate  the server classifies `groups` encrypted query groups with a resident model and takes the
            result ciphertexts out as bytes (copse_evaluate for one group, copse_evaluate_batch for more);
  wire      the same for one group that arrives as bytes: import, evaluate, export;
  query     the data owner encrypts one group of feature vectors and takes the ciphertexts out as bytes;
  labels    the data owner takes in a result's bytes and decrypts the labels.

The forest shapes are those of the repository's workloads (`synth.WORKLOADS`, `synth.TABLE6`) or smaller;
the encrypted 64-tree model of the headline benchmark is 45 GiB and minutes of encryption, so encrypted
models here are the 8-tree forest, which runs the same kernels.  What a serving process makes once and
keeps for its life (the context, one data owner's keys, the encoded model) is made once per process here
too; the queries, their encryption and everything that follows come from the seed.
"""
from __future__ import annotations

import ctypes
import functools
import math

import numpy as np

from paper_2104_09583_amd import copse, synth

CHAINS = {"16k": synth.CHAIN_16K, "32k8": synth.CHAIN_32K_P8, "32k16": synth.CHAIN_32K_P16}


def _case(name, path="evaluate", chain="32k8", trees=16, depth=5, split=0.7, features=16, precision=8, classes=4,
          forest=2, groups=1, queries=0, encrypted=False, fold=False, n1_r=0, n1_l=0, replicate=False, pad=0):
    """queries: per group, 0 for as many as the layout holds; pad > 0: private result with that many padding
    labels; replicate: the server replicates the features."""
    return dict(name=name, path=path, chain=chain, trees=trees, depth=depth, split=split, features=features,
                precision=precision, classes=classes, forest=forest, groups=groups, queries=queries,
                encrypted=encrypted, fold=fold, n1_r=n1_r, n1_l=n1_l, replicate=replicate, pad=pad)


def listed():
    return [
        # the smallest call: one complete tree, one query, the small ring; latency and launches
        _case("single_1x3_16k", chain="16k", trees=1, depth=3, split=1.0, features=4, classes=2, forest=1, queries=1,
              fold=True),
        # one interactive query against the 16-tree forest: the library's own latency workload
        _case("single_16x5", queries=1, n1_r=16),
        # one query of 16-bit features against a tiny two-tree forest: the comparison is most of it
        _case("single_2x5_p16", chain="32k16", trees=2, depth=5, features=2, precision=16, classes=3, forest=11,
              queries=1),
        # one query against a model that is encrypted too
        _case("single_enc_8x4", chain="32k16", trees=8, depth=4, forest=5, queries=1, encrypted=True),
        # a few groups that happened to queue up together: an odd batch
        _case("three_16x5", groups=3, n1_r=16),
        # an odd batch of 16-bit queries, the last block of each group left empty
        _case("five_8x4_p16", chain="32k16", trees=8, depth=4, features=32, precision=16, classes=10, forest=7,
              groups=5, queries=3),
        # the throughput workload: 256 queries against 32 trees in one call of 16 groups
        _case("batch16_32x6", trees=32, depth=6, classes=8, forest=3, groups=16, n1_l=16),
        # the throughput of an encrypted model: 16 groups in one call
        _case("batch16_enc_8x4", chain="32k16", trees=8, depth=4, forest=5, groups=16, encrypted=True),
        # the private options together: features replicated by the server, results shuffled and padded
        _case("pair_replicated_8x4", chain="32k16", trees=8, depth=4, forest=5, groups=2, replicate=True, pad=21),
        # a request as it reaches a server: bytes in, evaluation, bytes out
        _case("wire_16x5", path="wire", queries=1, n1_r=16),
        # the client's side of that request: encrypt and serialise a full group, decrypt the answer
        _case("query_16x5", path="query", n1_r=16),
        _case("labels_16x5", path="labels", n1_r=16),
    ]


def draw(rng):
    """One more case: the forest's size over its logarithm, odd group counts, precisions and query counts."""
    def log_int(lo, hi):
        return min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))

    path = rng.choice(["evaluate"] * 9 + ["wire", "query", "labels"])
    chain = rng.choice(["16k", "32k8", "32k8", "32k8", "32k16", "32k16"])
    encrypted = path == "evaluate" and chain != "16k" and rng.random() < 0.3
    replicate = path == "evaluate" and chain == "32k16" and not encrypted and rng.random() < 0.3
    depth = rng.randint(2, 3 if chain == "16k" else 4 if encrypted else 6)
    trees = log_int(1, 4 if chain == "16k" else 8 if encrypted else 24)
    # the longer chain has one level more: 16-bit features, or the replication product
    precision = rng.randint(9, 16) if chain == "32k16" and not replicate else rng.randint(3, 8)
    groups = log_int(1, 16 if trees * 2 ** depth <= 400 else 8) if path == "evaluate" else 1
    return _case("", path=path, chain=chain, trees=trees, depth=depth, features=rng.randint(2, 32),
                 precision=precision, classes=rng.randint(2, 10), forest=rng.randrange(1000), groups=groups,
                 queries=rng.randint(0, 4), encrypted=encrypted, fold=chain == "16k", replicate=replicate,
                 pad=rng.choice([0, 0, 0, rng.randint(1, 60)]))


# ---------------------------------------------------------------- what a process makes once and keeps
def _text(c):
    shape = synth.ForestShape(c["trees"], c["depth"], c["split"], c["features"], c["precision"], c["classes"])
    return synth.gen_forest_text(shape, c["forest"])


def _compiled(c):
    return copse.forest_compile_ex(_text(c), c["features"], c["precision"], CHAINS[c["chain"]]["log_n"], fold=c["fold"],
                                   n1_R=c["n1_r"], n1_L=c["n1_l"], server_replication=c["replicate"],
                                   privacy_seed=b"\x29" * 32 if c["pad"] else None, n_pad=c["pad"])


@functools.lru_cache(maxsize=None)
def _owner(chain):
    """The context and one data owner's keys (full, and as the server holds them): every rotation that the
    compiler's splits of these forests use, so that all resident models share one key set."""
    ctx = copse.Context(**CHAINS[chain])
    top = 256 if chain == "16k" else 1024
    rots = sorted(set(range(1, 32)) | {40, 56} | set(range(16, min(640, top), 16)) | set(range(32, top, 32)))
    keys = ctx.keygen(synth.crypto_seed("perf-" + chain), rots)
    return ctx, keys, ctx.export_eval(keys)


@functools.lru_cache(maxsize=16)
def _model(items):
    c = dict(items)
    ctx, keys, _ = _owner(c["chain"])
    comp, meta = _compiled(c)
    seed = synth.crypto_seed("perf-model")
    return ctx.model_encode(comp, keys, True, seed) if c["encrypted"] else ctx.model_encode(comp), meta


def _resident(c):
    shape = {k: v for k, v in c.items() if k not in ("name", "path", "groups", "queries")}
    return _model(tuple(sorted(shape.items())))


# ---------------------------------------------------------------- one case
def _features(c, meta, seed, group):
    n = min(c["queries"] or meta.queries_per_ct, meta.queries_per_ct)
    return synth.gen_queries(n, c["features"], c["precision"], 1000 * seed + group)


def _export(ctx, cts):
    """The ciphertexts' bytes, in the library's wire format (64-bit words)."""
    need = ctypes.c_size_t()
    copse.check(copse.lib().copse_cts_export(ctx.ptr, cts.ptr, None, 0, ctypes.byref(need)))
    buf = np.empty(need.value, dtype=np.uint64)
    copse.check(copse.lib().copse_cts_export(ctx.ptr, cts.ptr, buf.ctypes.data_as(ctypes.POINTER(ctypes.c_uint64)),
                                             buf.size, ctypes.byref(need)))
    return buf.view(np.int64)


def _import(ctx, buf):
    h = ctypes.c_void_p()
    copse.check(copse.lib().copse_cts_import(ctx.ptr, buf.ctypes.data_as(ctypes.POINTER(ctypes.c_uint64)), buf.size,
                                             ctypes.byref(h)))
    return copse.Cts(h, ctx)


def prepare(case, seed):
    ctx, keys, server_keys = _owner(case["chain"])
    if case["path"] == "query":
        meta = _compiled(case)[1]   # the data owner knows the public facts, not the model
        return dict(case=case, ctx=ctx, keys=keys, meta=meta, features=_features(case, meta, seed, 0),
                    seed=synth.crypto_seed(f"perf-{seed}"))
    model, meta = _resident(case)
    features = [_features(case, meta, seed, g) for g in range(case["groups"])]
    queries = [ctx.query_encrypt(keys, meta, f, synth.crypto_seed(f"perf-{seed}"), group=g)
               for g, f in enumerate(features)]
    st = dict(case=case, ctx=ctx, model=model, server_keys=server_keys, queries=queries)
    if case["path"] == "wire":
        st["queries"] = None
        st["bytes"] = _export(ctx, queries[0])
    elif case["path"] == "labels":
        return dict(case=case, ctx=ctx, keys=keys, meta=meta, n=len(features[0]),
                    bytes=_export(ctx, ctx.evaluate(model, server_keys, queries[0])))
    return st


def run(st):
    ctx, path = st["ctx"], st["case"]["path"]
    if path == "query":
        return _export(ctx, ctx.query_encrypt(st["keys"], st["meta"], st["features"], st["seed"]))
    if path == "labels":
        return ctx.decrypt_labels(st["keys"], st["meta"], _import(ctx, st["bytes"]), st["n"])
    if path == "wire":
        return _export(ctx, ctx.evaluate(st["model"], st["server_keys"], _import(ctx, st["bytes"])))
    if len(st["queries"]) == 1:
        return _export(ctx, ctx.evaluate(st["model"], st["server_keys"], st["queries"][0]))
    return [_export(ctx, r) for r in ctx.evaluate_batch(st["model"], st["server_keys"], st["queries"])]


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    """bytes: the query planes, the model, the keys' rows at the levels of use and the results, each once;
    flops: 8 per modular product of the circuit's transforms, key switches and diagonal products."""
    meta = _compiled(case)[1]
    ch = CHAINS[case["chain"]]
    N, L, alpha, p, G = 1 << ch["log_n"], ch["n_data_primes"] - 1, ch["alpha"], case["precision"], case["groups"]
    row, ntt = 8 * N, N // 2 * ch["log_n"]
    fresh, result = p * 2 * (L + 1) * row, 2 * row
    enc = 3 * (L + 1) * ntt + 2 * (L + 1) * N   # one encryption: three transforms, two products a limb
    if case["path"] == "query":
        return {"bytes": fresh + 2 * (L + 1) * row, "flops": 8.0 * (p * enc + fresh / row * ntt)}
    if case["path"] == "labels":
        return {"bytes": result + row, "flops": 8.0 * (4 * ntt + N)}
    total = dict(bytes=float(G * (fresh + result)), mul=0.0)

    def switch(level, inputs, keys, outputs):
        """ModUp of `inputs`, `outputs` inner products with `keys` distinct keys, ModDown of `outputs`."""
        nl, ext, D = level + 1, level + 1 + alpha, -(-(level + 1) // alpha)
        total["bytes"] += keys * 2.0 * D * ext * row
        total["mul"] += inputs * (D * ext * ntt + (D * ext - nl) * alpha * N)
        total["mul"] += outputs * (2 * D * ext * N + 2 * ext * ntt + 2 * nl * (alpha + 2) * N)

    def product(level, n, rows, n1, many, babies=True):
        """`many` matrix products of n diagonals over rows nonzero entries that share their baby steps."""
        nz = many * (n if case["encrypted"] else n * (1.0 - (1.0 - 1.0 / n) ** rows))
        n1 = n1 or 1 << math.ceil(math.log2(max(1.0, math.sqrt(n))))
        giants = -(-n // n1)
        switch(level, G, min(n1, n) - 1, G * (min(n1, n) - 1))
        polys = 2 if case["encrypted"] else 1
        total["bytes"] += nz * polys * (level + 1) * row
        total["mul"] += nz * G * (level + 1) * N * (3 if case["encrypted"] else 2)
        if case["encrypted"]:
            switch(level, G * giants * many, 1, G * giants * many)
        switch(level, G * (giants - 1) * many, giants - 1, G * many)

    level = L
    if case["replicate"]:
        Gp, G = G, G * p
        product(level, case["features"], meta.m + meta.b + meta.q - 2, 0, 1)
        G, level = Gp, level - 1
    total["bytes"] += p * (2 if case["encrypted"] else 4) * (level + 1) * row
    if case["encrypted"]:
        switch(level, G * p, 1, G * p)
    total["mul"] += G * p * 4 * (level + 1) * (N + ntt)
    rounds = max(1, math.ceil(math.log2(p)))
    for r in range(rounds):
        level -= 1
        switch(level, G * 2 * p / rounds, 1, G * 2 * p / rounds)
    level -= 1
    if not case["fold"]:
        product(level, meta.q, meta.m + meta.b - 1, case["n1_r"], 1)
        level -= 1
    n = meta.q if case["fold"] else meta.b
    product(level, n, meta.m, case["n1_l"], meta.d)
    total["bytes"] += meta.d * level * row
    for _ in range(math.ceil(math.log2(meta.d))):
        level -= 1
        switch(max(level, 0), G * meta.d / 2.0, 1, G * meta.d / 2.0)
    if case["path"] == "wire":
        total["mul"] += (fresh + result) / row * ntt
    return {"bytes": total["bytes"], "flops": 8.0 * total["mul"]}


def exact(case, seed):
    """The labels by walking the trees.  Ciphertexts are whole numbers fixed bit for bit by the scheme, with
    no rounding that a wider type would take away, so they have no such value."""
    if case["path"] != "labels" or case["pad"]:
        return None   # (a private result's slots are shuffled by the model owner's secret permutation)
    meta = _compiled(case)[1]
    text = _text(case).splitlines()[1:]
    X = _features(case, meta, seed, 0).astype(np.int64)
    bits = np.zeros((len(X), meta.m), dtype=np.uint8)
    leaf = 0

    def walk(tokens, hit):
        """Consumes one subtree; marks its leaf slot for the queries that reach it."""
        nonlocal leaf
        if next(tokens) == "L":
            next(tokens)
            bits[:, leaf] = hit
            leaf += 1
            return
        f, t = int(next(tokens)), int(next(tokens))
        true = X[:, f] < t
        walk(tokens, hit & ~true)
        walk(tokens, hit & true)

    for line in text:
        walk(iter(line.split()), np.ones(len(X), dtype=bool))
    return bits

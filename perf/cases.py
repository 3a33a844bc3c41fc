"""Workloads for measuring the library through its public calls.

A case is a dict of plain values; its "kind" names the work of one pass:

  detect    the decision for one batch of host-to-device payloads: detect()
  send      the transfer around a decision already made: send_plan(), pack_misses() at
            the sender, restore_blocks() at the receiver
  identify  free-time identification of the allocations of a batch: identify_weights(), or
            identify_leaves() where "leaves" is true
  writes    the first-write rule over the recorded writes of many allocations:
            first_writes()
  turnover  a model comes to a table of identifiers and goes again: lookup() of its
            digests, insert() of the new ones, touch() of all, erase() of the new ones
  bounded   a table held at its size by LRU eviction: insert() of a model used once,
            touch() of a model in use, evict() down to the size, export() of the set
  remap     tasks come and go on the address-remap map: update() (some tasks unloaded,
            others loaded in their place), translate() of the pointers of remoted calls,
            update() back, export()

Payload lengths, write logs and address spaces have the shapes that workloads/ and bench.py
use: one random buffer, ResNet-50's and a 7B decoder's tensors, many small copies with
log-uniform sizes, tasks that load such models into 1 TB spaces of their own. A case fixes
how many of everything there are (payload lengths, writes of each allocation, model of each
task); the seed draws the contents: bytes, what is held, repeated or changed, addresses.
Every output is a whole number or bytes, so two correct implementations agree exactly.
"""

import math

import numpy as np
import torch

import paper_2607_23115_amd as g

LEAF = 4096
KiB, MiB = 1 << 10, 1 << 20
DEVICE = "cuda"


def listed():
    return [
        # The smallest decision: one 16 MiB copy, a quarter of its blocks new. Bound by
        # latency, as every copy call that a task makes on its own is.
        {"name": "detect_copy_16m", "kind": "detect", "shape": "copy", "bytes": 16 * MiB, "block": 64 * KiB,
         "held": 0.75, "repeat": 0.0, "skew": 0, "others": 10_000},
        # A small model loaded as one batch: ResNet-50's 161 fp16 tensors, half of them held.
        {"name": "detect_resnet50", "kind": "detect", "shape": "resnet50", "block": 64 * KiB, "held": 0.5,
         "repeat": 0.0, "skew": 0, "others": 100_000},
        # The headline: a 7B decoder's fp16 weights, one tensor in ten new, in a table that
        # also holds the identifiers of many other models.
        {"name": "detect_decoder7b", "kind": "detect", "shape": "decoder", "layers": 32, "d": 4096, "ffn": 11008,
         "vocab": 32000, "block": MiB, "held": 0.9, "repeat": 0.0, "skew": 0, "others": 1_000_000},
        # Many small copies in one batch, a fifth of the full leaves repeated, nothing held yet.
        {"name": "detect_copies_100k", "kind": "detect", "shape": "copies", "n": 100_000, "lo": 256, "hi": 64 * KiB,
         "block": 4 * KiB, "held": 0.0, "repeat": 0.2, "skew": 0, "others": 100_000},
        # Sending small copies that do not start aligned: a third held by the receiver.
        {"name": "send_copies_20k", "kind": "send", "shape": "copies", "n": 20_000, "lo": 256, "hi": 64 * KiB,
         "block": 4 * KiB, "held": 0.33, "repeat": 0.2, "skew": 4, "others": 1000},
        # Sending a decoder shard (8 of 32 layers): one tensor in ten travels, the receiver
        # rebuilds all of it.
        {"name": "send_decoder_shard", "kind": "send", "shape": "decoder", "layers": 8, "d": 4096, "ffn": 11008,
         "vocab": 32000, "block": MiB, "held": 0.9, "repeat": 0.0, "skew": 0, "others": 1000},
        # Free time of a decoder shard: which allocations still hold what was written,
        # located to the leaf.
        {"name": "identify_leaves", "kind": "identify", "shape": "decoder", "layers": 6, "d": 4096, "ffn": 11008,
         "vocab": 32000, "block": MiB, "skew": 0, "leaves": True, "changed": 0.1, "per_region": 9},
        # Free time of many small buffers: allocations of a few payloads each.
        {"name": "identify_copies", "kind": "identify", "shape": "copies", "n": 30_000, "lo": 256, "hi": 64 * KiB,
         "block": 4 * KiB, "skew": 0, "leaves": False, "changed": 0.05, "per_region": 8},
        # Write logs of 4,096 allocations of up to 64 recorded writes.
        {"name": "first_writes_4096", "kind": "writes", "allocations": 4096, "most": 64},
        # One 7B decoder's 12,917 digests come to a table of a million identifiers and go.
        {"name": "turnover_decoder", "kind": "turnover", "resident": 1_000_000, "model": 12_917, "held": 0.6},
        # The large shared table of a long-lived server: 20 M identifiers at load 0.6, a
        # 20,000-block model used once and pushed out, the identifier set exported.
        {"name": "bounded_20m", "kind": "bounded", "resident": 20_000_000, "model": 20_000, "in_use": 200_000},
        # The address map of 256 tasks: one task replaced and put back, a million pointers.
        {"name": "remap_256_tasks", "kind": "remap", "tasks": 256, "swap": 1, "pointers": 1 << 20},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_payloads(rng, most_bytes):
    """Payload lengths of one of the shapes: at most about most_bytes in all."""
    shape = rng.choice(["copy", "copies", "copies", "decoder"])
    if shape == "copy":
        c = {"shape": shape, "bytes": _log(rng, 64 * KiB, min(most_bytes, 1 << 30)),
             "block": rng.choice([4, 16, 64, 256]) * KiB}
    elif shape == "copies":
        c = {"shape": shape, "n": _log(rng, 16, 100_000), "lo": _log(rng, 64, 1024), "hi": _log(rng, 8 * KiB, 128 * KiB),
             "block": rng.choice([4, 4, 8, 16]) * KiB}
        while c["n"] > 16 and _volume(c)[0] > most_bytes:
            c["n"] = c["n"] // 2
    else:
        d = 64 * rng.randrange(8, 65)
        c = {"shape": shape, "layers": _log(rng, 1, 32), "d": d, "ffn": int(d * rng.choice([2.6875, 3.5, 4])),
             "vocab": _log(rng, 8000, 64000), "block": rng.choice([64, 256, 1024, 2048]) * KiB}
        while c["layers"] > 1 and _volume(c)[0] > most_bytes:
            c["layers"] = c["layers"] // 2
    c["skew"] = rng.choice([0, 0, 0, 4, 8, rng.randrange(1, 256)])
    return c


def draw(rng):
    kind = rng.choice(["detect", "detect", "detect", "send", "send", "identify", "writes", "turnover", "bounded",
                       "remap"])
    if kind == "detect":
        c = _draw_payloads(rng, 8 << 30)
        c.update(held=round(rng.uniform(0, 1), 3), repeat=rng.choice([0.0, 0.0, 0.05, 0.2]),
                 others=_log(rng, 1000, 4_000_000))
        if c["shape"] == "decoder":
            c["repeat"] = 0.0
    elif kind == "send":
        c = _draw_payloads(rng, 3 << 30)
        c.update(held=round(rng.uniform(0, 1), 3), repeat=rng.choice([0.0, 0.05, 0.2]), others=1000)
        if c["shape"] == "decoder":
            c["repeat"] = 0.0
    elif kind == "identify":
        c = _draw_payloads(rng, 6 << 30)
        c.update(leaves=rng.choice([False, True]), changed=round(rng.uniform(0, 0.5), 3),
                 per_region=rng.randrange(1, 17))
    elif kind == "writes":
        most = _log(rng, 2, 2048)
        c = {"allocations": max(2, min(_log(rng, 16, 32_768), 600_000 // most)), "most": most}
    elif kind == "turnover":
        c = {"resident": _log(rng, 1000, 20_000_000), "model": _log(rng, 16, 400_000),
             "held": round(rng.uniform(0, 1), 3)}
    elif kind == "bounded":
        n = _log(rng, 1000, 16_000_000)
        c = {"resident": n, "model": _log(rng, 16, max(32, n // 20)), "in_use": _log(rng, 16, max(32, n // 4))}
    else:
        tasks = _log(rng, 2, 512)
        c = {"tasks": tasks, "swap": min(tasks, _log(rng, 1, 24)), "pointers": _log(rng, 64, 4 << 20)}
    return dict(kind=kind, **c)


# --------------------------------------------------------------------------- #
# Payloads
# --------------------------------------------------------------------------- #
def _resnet50_elements():
    """Element counts of ResNet-50's 161 parameter tensors, in module order."""
    n = [64 * 3 * 49, 64, 64]
    cin = 64
    for count, w in ((3, 64), (4, 128), (6, 256), (3, 512)):
        for b in range(count):
            n += [w * cin, w, w, w * w * 9, w, w, 4 * w * w, 4 * w, 4 * w]
            if b == 0:
                n += [4 * w * cin, 4 * w, 4 * w]
            cin = 4 * w
    return n + [1000 * 2048, 1000]


def _decoder_elements(layers, d, ffn, vocab):
    """Element counts of a decoder's tensors: embedding, per layer two norms, four
    attention and three MLP matrices, final norm, head."""
    layer = [d, d * d, d * d, d * d, d * d, d, ffn * d, ffn * d, d * ffn]
    return [vocab * d] + layer * layers + [d, vocab * d]


def _shape_rng():
    """What belongs to the case rather than to the seed is drawn from here."""
    return np.random.default_rng(20)


def _lengths(case):
    if case["shape"] == "copy":
        return np.array([case["bytes"]], np.uint64)
    if case["shape"] == "resnet50":
        return 2 * np.array(_resnet50_elements(), np.uint64)
    if case["shape"] == "decoder":
        return 2 * np.array(_decoder_elements(case["layers"], case["d"], case["ffn"], case["vocab"]), np.uint64)
    lo, hi = math.log(case["lo"]), math.log(case["hi"])
    return np.floor(np.exp(_shape_rng().uniform(lo, hi, case["n"]))).astype(np.uint64)


def _volume(case):
    """(payload bytes, blocks) of a case."""
    n = _lengths(case)
    return int(n.sum()), int((-(-n.astype(np.int64) // case["block"])).sum())


def _arena(case, seed):
    """(arena, offsets, lengths): the payloads in device memory, each `skew` bytes past a
    multiple of 256. Tensors hold fp16 normals, other buffers random bytes; a share
    `repeat` of the full 4 KiB leaves repeats another one."""
    rng = np.random.default_rng([seed, 1])
    lengths = _lengths(case)
    padded = (lengths + np.uint64(255)) // np.uint64(256) * np.uint64(256)
    offsets = np.concatenate([[0], np.cumsum(padded)[:-1]]).astype(np.uint64)
    total = int(padded.sum())
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    if case["shape"] in ("resnet50", "decoder"):
        arena = torch.empty(total // 2, dtype=torch.float16, device=DEVICE).normal_(0.0, 0.02, generator=gen)
    else:
        arena = torch.empty(total // 8, dtype=torch.int64, device=DEVICE).random_(generator=gen)
        arena ^= torch.empty_like(arena).random_(generator=gen) << 1  # random_() leaves the top bit clear
    if case.get("repeat"):
        words = arena.view(torch.int64)
        per = (lengths // np.uint64(LEAF)).astype(np.int64)
        k = np.arange(int(per.sum())) - np.repeat(np.cumsum(per) - per, per)
        full = np.repeat(offsets.astype(np.int64), per) + LEAF * k
        order = rng.permutation(full.size)
        n = int(case["repeat"] * full.size)
        if n and full.size > n:
            to = torch.from_numpy(full[order[:n]] // 8).to(DEVICE)
            at = torch.from_numpy(full[order[n + rng.integers(0, full.size - n, n)]] // 8).to(DEVICE)
            row = torch.arange(LEAF // 8, device=DEVICE)
            words[to[:, None] + row] = words[at[:, None] + row]
    arena = arena.view(torch.uint8)
    if case["skew"]:
        moved = torch.zeros(total + 256, dtype=torch.uint8, device=DEVICE)
        moved[case["skew"]:case["skew"] + total] = arena
        arena, offsets = moved, offsets + np.uint64(case["skew"])
    return arena, offsets, lengths


def _u64(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.uint64).view(np.int64)).to(DEVICE)


def _random_u64(rng, n):
    return rng.integers(0, 1 << 64, n, dtype=np.uint64)


def _random_keys(seed, n):
    """n random 64-bit keys, made on the GPU."""
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    a = torch.empty(n, dtype=torch.int64, device=DEVICE).random_(generator=gen)
    return a ^ (torch.empty_like(a).random_(generator=gen) << 1)


def _capacity(n):
    cap = 16
    while 0.65 * cap < n:
        cap *= 2
    return cap


def _decided(case, seed, holder_of=None):
    """The batch, a table that holds some of its blocks, and a Detect for it. Table values
    are the held blocks' offsets in the holder's arena, or their addresses where holder_of
    makes that arena (of the payload's)."""
    rng = np.random.default_rng([seed, 2])
    arena, offsets, lengths = _arena(case, seed)
    batch = g.Batch.from_arena(arena, offsets, lengths, case["block"])
    digests = g.fp_chunks(batch)
    blocks = np.diff(batch.host_first.astype(np.int64))
    first = np.repeat(batch.host_first[:-1].astype(np.int64), blocks)
    at = np.repeat(offsets.astype(np.int64), blocks) + (np.arange(batch.n_blocks) - first) * case["block"]
    if case["shape"] in ("resnet50", "decoder"):  # whole tensors are held
        mask = np.repeat(rng.random(batch.n_seg) < case["held"], blocks)
    else:
        mask = rng.random(batch.n_blocks) < case["held"]
    held = np.flatnonzero(mask)
    holder = None if holder_of is None else holder_of(arena)
    table = g.Cache(_capacity(case["others"] + held.size + 1))
    table.insert(_random_keys(seed + 7919, case["others"]), torch.arange(case["others"], device=DEVICE))
    if held.size:
        pick = torch.from_numpy(held).to(DEVICE)
        base = 0 if holder is None else holder.data_ptr()
        table.insert(digests[pick].contiguous(), torch.from_numpy(at[held] + base).to(DEVICE))
    out = g.Detect(batch)
    for t in (out.digests, out.status, out.ref, out.miss_idx, out.counters):
        t.zero_()
    return batch, table, out, holder, (arena, offsets, lengths)


# --------------------------------------------------------------------------- #
# Preparation
# --------------------------------------------------------------------------- #
def _prepare_detect(case, seed):
    batch, table, out, _, _ = _decided(case, seed)
    return {"batch": batch, "table": table, "out": out}


def _prepare_send(case, seed):
    batch, table, out, holder, (arena, offsets, lengths) = _decided(case, seed, torch.clone)
    g.detect(batch, table, out)
    into = torch.zeros_like(arena)
    dst = g.Batch.from_arena(into, offsets, lengths, case["block"])
    # the sender's buffer is large enough for a batch of which nothing is held
    packed = torch.zeros(int(((lengths + np.uint64(15)) // np.uint64(16)).sum()) * 16 + 16 * batch.n_blocks,
                         dtype=torch.uint8, device=DEVICE)
    return {"batch": batch, "dst": dst, "into": into, "holder": holder, "digests": out.digests, "status": out.status,
            "ref": out.ref, "ws": g.workspace(batch.n_blocks), "packed": packed}


def _prepare_identify(case, seed):
    rng = np.random.default_rng([seed, 3])
    arena, offsets, lengths = _arena(case, seed)
    batch = g.Batch.from_arena(arena, offsets, lengths, case["block"])
    recorded, leaves = g.fp_chunks(batch, with_leaves=True)
    changed = np.flatnonzero((rng.random(lengths.size) < case["changed"]) & (lengths > 0))
    at = offsets[changed] + (rng.random(changed.size) * lengths[changed]).astype(np.uint64)
    arena[torch.from_numpy(at.astype(np.int64)).to(DEVICE)] ^= 1
    regions = np.append(np.arange(0, lengths.size, case["per_region"]), lengths.size)
    n = batch.n_blocks * (batch.leaves_per_block if case["leaves"] else 1)
    return {"batch": batch, "recorded": leaves if case["leaves"] else recorded, "regions": _u64(regions),
            "leaves": case["leaves"], "ws": g.workspace(n + batch.n_seg)}


def _prepare_writes(case, seed):
    """Allocation r at (r + 1) << 36 of 4 KiB to 16 MiB, each with 1 to `most` writes in time
    order: two in ten repeat an earlier write, three in ten cover all of it, the others a
    part."""
    rng = np.random.default_rng([seed, 4])
    n_alloc = case["allocations"]
    counts = _shape_rng().integers(1, case["most"] + 1, n_alloc)
    sizes = np.floor(np.exp(rng.uniform(math.log(4 * KiB), math.log(16 * MiB), n_alloc))).astype(np.int64)
    first = np.concatenate([[0], np.cumsum(counts)])
    alloc = np.repeat(np.arange(n_alloc), counts)
    j = np.arange(first[-1]) - first[alloc]
    size = sizes[alloc]
    ends = np.sort((rng.random((j.size, 2)) * (size[:, None] + 1)).astype(np.int64), axis=1)
    u = rng.random(j.size)
    whole = (u >= 0.2) & (u < 0.5)
    ends[whole, 0], ends[whole, 1] = 0, size[whole]
    source = np.where((u < 0.2) & (j > 0), first[alloc] + (rng.random(j.size) * j).astype(np.int64), np.arange(j.size))
    while np.any(source[source] != source):
        source = source[source]
    ends = ends[source]
    addr = ((alloc + 1).astype(np.uint64) << np.uint64(36)) + ends[:, 0].astype(np.uint64)
    out = g.first_writes_outputs(j.size, n_alloc)
    for t in out:
        t.zero_()
    return {"addr": _u64(addr), "length": _u64(ends[:, 1] - ends[:, 0]), "first": _u64(first), "out": out,
            "ws": g.first_writes_workspace(j.size, n_alloc)}


def _prepare_turnover(case, seed):
    n, m = case["resident"], case["model"]
    keys = _random_keys(seed, n + m)
    n_held = int(case["held"] * min(m, n))
    model = torch.cat([keys[:n_held], keys[n:n + m - n_held]])
    gen = torch.Generator(device=DEVICE).manual_seed(seed + 1)
    model = model[torch.randperm(m, generator=gen, device=DEVICE)].contiguous()
    table = g.Cache(_capacity(n + m))
    table.insert(keys[:n].contiguous(), torch.arange(n, device=DEVICE))
    new = keys[n:n + m - n_held].contiguous()
    return {"table": table, "model": model, "new": new, "vals": torch.arange(new.numel(), device=DEVICE),
            "bound": n, "ws": g.workspace(m), "status": torch.zeros(m, dtype=torch.uint8, device=DEVICE),
            "ref": torch.zeros(m, dtype=torch.int64, device=DEVICE)}


def _prepare_bounded(case, seed):
    n, m = case["resident"], case["model"]
    keys = _random_keys(seed, n + m)
    gen = torch.Generator(device=DEVICE).manual_seed(seed + 1)
    table = g.Cache(_capacity(n + m))
    table.insert(keys[:n].contiguous(), torch.arange(n, device=DEVICE))
    table.touch(keys[:n].contiguous(), torch.randint(1, 100_000, (n,), generator=gen, device=DEVICE))
    use = torch.randint(0, n, (case["in_use"],), generator=gen, device=DEVICE)
    return {"table": table, "new": keys[n:].contiguous(), "vals": torch.arange(m, device=DEVICE), "size": n,
            "in_use": keys[use].contiguous(), "ws": g.workspace(m), "maint": table.maint_workspace()}


def _task_spaces(case, seed):
    """Intervals (start, length, target) of each task: the tensors of its model (a decoder,
    ResNet-50 or a 2,000-tensor set) packed from a random base of its own 1 TB space, each
    onto the shareable copy of the same tensor. `swap` more tasks wait to be loaded."""
    rng = np.random.default_rng([seed, 5])
    wide = np.exp(_shape_rng().uniform(math.log(MiB), math.log(200 * MiB), 2000)).astype(np.uint64)
    sizes = [2 * np.array(_decoder_elements(32, 4096, 11008, 32000), np.uint64),
             2 * np.array(_resnet50_elements(), np.uint64), wide]
    rounded = [(s + np.uint64(511)) // np.uint64(512) * np.uint64(512) for s in sizes]
    packed = [np.concatenate([[0], np.cumsum(s)[:-1]]).astype(np.uint64) for s in rounded]
    n = case["tasks"] + case["swap"]
    kind = _shape_rng().integers(0, 3, n)
    base = (np.arange(n, dtype=np.uint64) << np.uint64(40)) + (
        rng.integers(0, 1 << 18, n).astype(np.uint64) << np.uint64(21))
    return [(packed[k] + b, sizes[k], packed[k] + np.uint64(0x7000_0000_0000 + (int(k) << 40)))
            for k, b in zip(kind, base)], rng


def _joined(tasks):
    return tuple(_u64(np.concatenate([t[i] for t in tasks])) for i in range(3))


def _prepare_remap(case, seed):
    tasks, rng = _task_spaces(case, seed)
    n = case["tasks"]
    out_tasks = np.arange(case["swap"])
    gone, come = _joined([tasks[i] for i in out_tasks]), _joined(tasks[n:])
    live = [tasks[i] for i in range(n) if i not in set(out_tasks.tolist())]
    count = sum(t[0].size for t in tasks[:n])
    cap = 1 << (count + come[0].numel()).bit_length()
    table = g.Remap(cap)
    start, length, target = _joined(live) if live else gone
    table.update(add_start=start, add_len=length, add_target=target)
    if live:
        table.update(add_start=gone[0], add_len=gone[1], add_target=gone[2])
    # pointers: nine in ten inside a tensor, the rest anywhere in a task's space
    starts = np.concatenate([t[0] for t in live + tasks[n:]])
    lens = np.concatenate([t[1] for t in live + tasks[n:]])
    p = case["pointers"]
    pick = rng.integers(0, starts.size, p)
    inside = starts[pick] + (rng.random(p) * lens[pick].astype(np.float64)).astype(np.uint64)
    anywhere = _random_u64(rng, p) % np.uint64(len(tasks) << 40)
    addr = np.where(rng.random(p) < 0.9, inside, anywhere)
    most = max(gone[0].numel(), come[0].numel())
    counts = [torch.zeros(4, dtype=torch.int64, device=DEVICE) for _ in range(2)]
    return {"map": table, "gone": gone, "come": come, "addr": _u64(addr), "count": count, "counts": counts,
            "out": torch.zeros(p, dtype=torch.int64, device=DEVICE), "ws": table.update_workspace(most, most)}


def prepare(case, seed):
    state = {"detect": _prepare_detect, "send": _prepare_send, "identify": _prepare_identify,
             "writes": _prepare_writes, "turnover": _prepare_turnover, "bounded": _prepare_bounded,
             "remap": _prepare_remap}[case["kind"]](case, seed)
    state["kind"] = case["kind"]
    return state


# --------------------------------------------------------------------------- #
# One pass
# --------------------------------------------------------------------------- #
def _run_detect(s):
    out = g.detect(s["batch"], s["table"], s["out"])
    return out.digests, out.status, out.ref, out.miss_idx, out.counters


def _run_send(s):
    records, totals = g.send_plan(s["batch"], s["digests"], s["status"], s["ref"], s["ws"])
    g.pack_misses(s["batch"], records, s["packed"])
    g.restore_blocks(s["dst"], records, s["packed"], s["ref"])
    return records, totals, s["packed"].view(torch.int64), s["into"].view(torch.int64)


def _run_identify(s):
    call = g.identify_leaves if s["leaves"] else g.identify_weights
    return call(s["batch"], s["recorded"], s["regions"], s["ws"])


def _run_writes(s):
    return g.first_writes(s["addr"], s["length"], s["first"], out=s["out"], ws=s["ws"])


def _run_turnover(s):
    t = s["table"]
    status, ref = t.lookup(s["model"], s["status"], s["ref"], s["ws"])
    n_new = t.insert(s["new"], s["vals"], s["ws"])
    touched = t.touch(s["model"], epoch=5)
    counts = t.erase(s["new"])
    t.set_key_bound(s["bound"])  # the table is back at its size
    return status, ref, n_new, touched, counts


def _run_bounded(s):
    """The inserted model is never touched, so it is the oldest and eviction removes it: the
    table ends each pass as it began."""
    t, size = s["table"], s["size"]
    n_new = t.insert(s["new"], s["vals"], s["ws"])
    touched = t.touch(s["in_use"], epoch=100_000)
    evicted, counts = t.evict(size, s["maint"])
    keys, vals, stamps, count = t.export(s["maint"])
    # the valid entries: what was inserted was evicted, `size` remain
    return n_new, touched, evicted[:s["new"].numel()], counts, keys[:size], vals[:size], stamps[:size], count


def _run_remap(s):
    m, gone, come, n = s["map"], s["gone"], s["come"], s["count"]
    loaded, counts1 = m.update(gone[0], gone[1], *come, counts=s["counts"][0], ws=s["ws"])
    out = m.translate(s["addr"], s["out"])
    back, counts2 = m.update(come[0], come[1], *gone, counts=s["counts"][1], ws=s["ws"])
    start, length, target, count = m.export()
    return loaded, counts1, out, back, counts2, start[:n], length[:n], target[:n], count


def run(state):
    return {"detect": _run_detect, "send": _run_send, "identify": _run_identify, "writes": _run_writes,
            "turnover": _run_turnover, "bounded": _run_bounded, "remap": _run_remap}[state["kind"]](state)


# --------------------------------------------------------------------------- #
# What a pass cannot do without
# --------------------------------------------------------------------------- #
def work(case):
    """Bytes of one pass: every input read once and every output written once. The
    operations are integer ones and are not counted."""
    kind = case["kind"]
    if kind in ("detect", "send", "identify"):
        data, blocks = _volume(case)
        payloads = case["n"] if case["shape"] == "copies" else _lengths(case).size
        about = 24 * payloads  # descriptors
        if kind == "detect":  # digest, status, ref, index and the table's slot of each block
            return {"bytes": data + about + (8 + 1 + 8 + 8 + 16) * blocks, "flops": 0}
        if kind == "send":  # the plan's inputs and records; misses packed, everything restored
            miss = (1 - case["held"]) * (1 - case["repeat"]) * data
            return {"bytes": about + (17 + 3 * 40) * blocks + 2 * miss + 2 * data, "flops": 0}
        slots = blocks * (case["block"] // LEAF if case["leaves"] else 1)
        return {"bytes": data + about + 9 * slots + 8 * payloads, "flops": 0}
    if kind == "writes":  # the log; a piece for about every other write
        n = case["allocations"] * (case["most"] + 1) / 2
        return {"bytes": 16 * n + 24 * n / 2 + 17 * case["allocations"], "flops": 0}
    if kind == "turnover":  # each key and its slot once a call
        m = case["model"]
        new = m - int(case["held"] * min(m, case["resident"]))
        return {"bytes": m * (8 + 16 + 9) + new * (16 + 16) + m * (8 + 16) + new * (8 + 16), "flops": 0}
    if kind == "bounded":  # the table read and written by evict, read by export, the set written
        cap, n = _capacity(case["resident"] + case["model"]), case["resident"]
        return {"bytes": 3 * 24 * cap + 24 * n + 40 * case["model"] + 24 * case["in_use"], "flops": 0}
    # remap: the map read and written by each update, an interval looked up for each pointer
    n = case["tasks"] * 817 + 0.0  # mean tensors of a task over the three models
    return {"bytes": 2 * 2 * 24 * n + (8 + 8) * case["pointers"] + 2 * 24 * n, "flops": 0}


def tolerance(case):
    return "exact"

"""GPU parity of free-time weight identification (Sec. 4.1.1): block matches, each
payload's first changed block and each allocation's verdict equal the oracle's, and
the byte-level truth (which payloads were changed after being written)."""

import numpy as np
import pytest
import torch

import oracle
import paper_2607_23115_amd as g
import workloads as W
from gpu_util import host_threads, keys_to_device, say, to_device, u64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible GPU")
    torch.cuda.init()


def run_identify(arena, offs, lens, block, recorded, region_first):
    batch = g.Batch.from_arena(to_device(arena), offs, lens, block)
    m, f, w = g.identify_weights(batch, keys_to_device(recorded), region_first)
    torch.cuda.synchronize()
    return m.cpu().numpy(), u64(f), w.cpu().numpy()


@pytest.mark.parametrize("block", [4096, 65536, 1 << 20, 2 << 20])
def test_identify_random_regions(block):
    rng = np.random.default_rng(800 + block.bit_length())
    lens = [int(x) for x in rng.integers(0, 4 * block, 60)] + [0, 1, 4096, block]
    rng.shuffle(lens)
    written = [np.frombuffer(rng.bytes(n), np.uint8).copy() for n in lens]
    current = [w.copy() for w in written]
    changed = set()
    for i, c in enumerate(current):
        if c.size and rng.random() < 0.25:  # in-place updates after the write
            for _ in range(int(rng.integers(1, 4))):
                c[int(rng.integers(0, c.size))] ^= 1 << int(rng.integers(0, 8))
            changed.add(i)
    cuts = sorted(set(int(x) for x in rng.integers(0, len(lens) + 1, 12)))
    region_first = np.array([0] + cuts + [len(lens)], np.uint64)
    recorded, _ = oracle.batch_digests(written, block)
    arena, offs, lens_a = W.pack(current)
    say("identify block", block, "payloads", len(lens), "regions", region_first.size - 1)
    m, f, w = run_identify(arena, offs, lens_a, block, recorded, region_first)
    em, ef, ew = oracle.identify_weights(recorded, current, block, region_first)
    assert np.array_equal(m, em) and np.array_equal(f, ef) and np.array_equal(w, ew)
    # byte-level truth: a payload shows a difference iff it was changed
    assert {i for i in range(len(lens)) if f[i] != oracle.NO_DIFF} == {i for i in changed if current[i].size}


def test_identify_unaligned_and_empty_regions():
    rng = np.random.default_rng(850)
    block = 65536
    written = [np.frombuffer(rng.bytes(int(n)), np.uint8).copy() for n in rng.integers(1, 200000, 30)]
    current = [w.copy() for w in written]
    current[4][100] ^= 1
    current[17][-1] ^= 0x80
    region_first = np.array([0, 0, 5, 5, 12, 20, 30, 30], np.uint64)
    recorded, _ = oracle.batch_digests(written, block)
    arena, offs, lens = W.pack(current, skew=3)
    say("identify unaligned")
    m, f, w = run_identify(arena, offs, lens, block, recorded, region_first)
    em, ef, ew = oracle.identify_weights(recorded, current, block, region_first)
    assert np.array_equal(m, em) and np.array_equal(f, ef) and np.array_equal(w, ew)
    assert w.tolist() == [0, 0, 0, 1, 0, 1, 0]


@pytest.mark.timeout(900)
def test_identify_decoder7b_full():
    """Allocations = embedding, each layer, head; the payload is the base weights as
    written, the device holds the rank-16-updated layers: exactly those 3 layers'
    allocations are not weights, and every block of their 7 matrices changed."""
    threads = host_threads()
    dec = W.Decoder()
    block = W.DECODER_BLOCK
    say("identify decoder7b generate")
    arena, offs, lens = dec.arena(perturbed=True, threads=threads)
    current = [arena[int(o):int(o) + int(n)] for o, n in zip(offs, lens)]
    recorded, _ = oracle.batch_digests(current, block, threads=threads)
    first = oracle.geometry(lens, block)[0]
    for i in dec.perturbed:
        bd, _ = oracle.payload_digests(dec.base(i), block)
        recorded[int(first[i]):int(first[i + 1])] = bd
    # allocation boundaries: [embed], [layer l tensors] x 32, [final norm, lm head]
    region_first = np.array([0] + [1 + 9 * l for l in range(33)] + [len(lens)], np.uint64)
    say("identify decoder7b gpu", int(lens.sum()), "bytes")
    m, f, w = run_identify(arena, offs, lens, block, recorded, region_first)
    em, ef, ew = oracle.identify_weights(recorded, current, block, region_first, threads=threads)
    assert np.array_equal(m, em) and np.array_equal(f, ef) and np.array_equal(w, ew)
    bad_regions = {int(l) + 1 for l in dec.perturbed_layers}
    assert {r for r in range(w.size) if w[r] == 0} == bad_regions
    assert all(f[i] == 0 for i in dec.perturbed)


@pytest.mark.parametrize("block", [4096, 1 << 20])
def test_identify_payloads_changed_throughout(block):
    """Payloads whose every leaf changed (a layer rewritten in place) next to unchanged and
    partly changed ones, payload boundaries inside waves: leaf matches, first changed
    leaves and verdicts equal the oracle's; and a 256 MiB payload changed throughout is
    compared within a small multiple of the time of an unchanged one (with one atomic per
    changed leaf on the payload's word it took 15x as long)."""
    rng = np.random.default_rng(9100 + block.bit_length())
    lens = [3 << 20, 5000, 1 << 20, 4096, 777, 2 << 20]
    written = [np.frombuffer(rng.bytes(n), np.uint8).copy() for n in lens]
    current = [np.frombuffer(rng.bytes(n), np.uint8).copy() if i % 2 == 0 else w.copy()
               for i, (n, w) in enumerate(zip(lens, written))]
    current[3][100] ^= 1
    region_first = np.array([0, 2, 4, len(lens)], np.uint64)
    _, rec = oracle.batch_digests(written, block, with_leaves=True)
    arena, offs, lens_a = W.pack(current)
    batch = g.Batch.from_arena(to_device(arena), offs, lens_a, block)
    say("identify changed throughout", block)
    m, f, w = g.identify_leaves(batch, keys_to_device(rec.reshape(-1)), region_first)
    torch.cuda.synchronize()
    em, ef, ew = oracle.identify_leaves(rec, current, block, region_first)
    assert np.array_equal(m.cpu().numpy(), em)
    assert np.array_equal(u64(f), ef)
    assert np.array_equal(w.cpu().numpy(), ew)
    if block != 4096:
        return
    big = torch.randint(0, 256, (256 << 20,), dtype=torch.uint8, device="cuda")
    other = torch.randint(0, 256, (256 << 20,), dtype=torch.uint8, device="cuda")
    cur = g.Batch.from_arena(big, [0], [big.numel()], block)
    times = {}
    for label, src in (("changed", other), ("same", big)):
        rb = g.Batch.from_arena(src, [0], [src.numel()], block)
        leaves = torch.empty(rb.n_blocks * rb.leaves_per_block, dtype=torch.int64, device="cuda")
        g.fp_chunks(rb, leaf_out=leaves)
        ws = g.workspace(leaves.numel() + 1)
        for _ in range(3):
            g.identify_leaves(cur, leaves, [0, 1], ws=ws)
        torch.cuda.synchronize()
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(5):
            g.identify_leaves(cur, leaves, [0, 1], ws=ws)
        b.record()
        torch.cuda.synchronize()
        times[label] = a.elapsed_time(b) / 5
    assert times["changed"] < 3 * times["same"] + 0.05, times


@pytest.mark.parametrize("shape,block", [("one wave", 65536), ("few", 16384), ("few", 2 << 20), ("small payloads", 4096),
                                         ("small payloads", 65536), ("large payloads", 1 << 20),
                                         ("large payloads", 4096)])
def test_identify_matches_the_digests_of_both_states(shape, block):
    """The comparison runs inside the fingerprint kernels: in every launch they choose (one
    and four waves per workgroup, two lanes per leaf with a four-lane end, whole blocks) the
    matches, first differences and verdicts are those of the digests before and after."""
    rng = np.random.default_rng([block, len(shape)])
    lens = {"one wave": rng.integers(0, 5000, 40), "few": rng.integers(0, 40 * 4096, 300),
            "small payloads": rng.integers(0, 6 * 4096, 40_000 if block == 4096 else 9000),
            "large payloads": rng.integers(0, 64 << 20, 12)}[shape].astype(np.uint64)
    offs = np.concatenate([[0], np.cumsum((lens + np.uint64(15)) // np.uint64(16) * np.uint64(16))[:-1]]).astype(np.uint64)
    arena = torch.randint(0, 256, (int(offs[-1] + lens[-1]) + 16,), dtype=torch.uint8, device="cuda")
    batch = g.Batch.from_arena(arena, offs, lens, block)
    lpb = batch.leaves_per_block
    say("identify both states", shape, block, "slots", batch.n_blocks * lpb)
    blocks0, leaves0 = g.fp_chunks(batch, with_leaves=True)
    change = np.flatnonzero((rng.random(lens.size) < 0.3) & (lens > 0))
    at = (offs[change] + (rng.random(change.size) * lens[change]).astype(np.uint64)).astype(np.int64)
    arena[torch.from_numpy(at).cuda()] ^= 1
    blocks1, leaves1 = g.fp_chunks(batch, with_leaves=True)
    regions = np.append(np.arange(0, lens.size, 7), lens.size).astype(np.uint64)
    first = batch.host_first.astype(np.int64)
    for got, before, after, per in ((g.identify_weights(batch, blocks0, regions), blocks0, blocks1, 1),
                                    (g.identify_leaves(batch, leaves0, regions), leaves0, leaves1, lpb)):
        torch.cuda.synchronize()
        same = (u64(before) == u64(after)).reshape(-1)
        want = np.full(lens.size, oracle.NO_DIFF, np.uint64)
        bad = np.flatnonzero(~same)
        seg = np.searchsorted(first, bad // per, side="right") - 1
        for s in np.unique(seg):
            want[s] = bad[seg == s][0] - first[s] * per
        verdict = [int(np.all(want[a:b] == oracle.NO_DIFF)) for a, b in zip(regions[:-1].astype(int), regions[1:].astype(int))]
        assert np.array_equal(got[0].cpu().numpy().reshape(-1) != 0, same)
        assert np.array_equal(u64(got[1]), want)
        assert got[2].cpu().numpy().tolist() == verdict
    assert np.array_equal(np.flatnonzero(want != oracle.NO_DIFF), change)


@pytest.mark.parametrize("block,n", [(256 << 10, 3000), (512 << 10, 2100), (1 << 20, 1100), (4 << 20, 300),
                                     (16 << 20, 150), (16 << 20, 700)])
def test_identify_leaves_of_short_blocks(block, n):
    """Payloads far shorter than their blocks between some of several blocks, in every unit
    size of the launch for such batches: the matches (also of slots that hold no leaf, where
    the recorded digests name one), first differences and verdicts are those of the digests."""
    rng = np.random.default_rng([9300, block, n])
    lens = rng.choice([0, 1, 4095, 4097, 20_000, 127 * 4096, 128 * 4096, 128 * 4096 + 1, block - 1, block, block + 1,
                       2 * block + 5000], n, p=[.1, .1, .2, .2, .3] + [.1 / 7] * 7).astype(np.uint64)
    offs = np.concatenate([[0], np.cumsum((lens + np.uint64(15)) // np.uint64(16) * np.uint64(16))[:-1]]).astype(np.uint64)
    arena = torch.randint(0, 256, (int(offs[-1] + lens[-1]) + 16,), dtype=torch.uint8, device="cuda")
    batch = g.Batch.from_arena(arena, offs, lens, block)
    per, first = batch.leaves_per_block, batch.host_first.astype(np.int64)
    say("identify leaves of short blocks", block, n, "slots", batch.n_blocks * per)
    _, recorded = g.fp_chunks(batch, with_leaves=True)
    change = np.flatnonzero((rng.random(n) < 0.3) & (lens > 0))
    at = (offs[change] + (rng.random(change.size) * lens[change]).astype(np.uint64)).astype(np.int64)
    arena[torch.from_numpy(at).cuda()] ^= 1
    _, current = g.fp_chunks(batch, with_leaves=True)
    stray = torch.from_numpy(rng.integers(0, batch.n_blocks * per, 25)).cuda()  # mostly slots without a leaf
    recorded[stray] ^= 77
    regions = np.append(np.arange(0, n, 7), n).astype(np.uint64)
    match, first_diff, weight = g.identify_leaves(batch, recorded, regions)
    same = recorded == current
    assert torch.equal(match.reshape(-1) != 0, same.reshape(-1))
    bad = torch.nonzero(~same.reshape(-1)).reshape(-1).cpu().numpy()
    seg = np.searchsorted(first, bad // per, side="right") - 1
    want = np.full(n, oracle.NO_DIFF, np.uint64)
    np.minimum.at(want, seg, (bad - first[seg] * per).astype(np.uint64))
    assert np.array_equal(u64(first_diff), want)
    assert weight.cpu().numpy().tolist() == [int(np.all(want[a:b] == oracle.NO_DIFF))
                                             for a, b in zip(regions[:-1].astype(int), regions[1:].astype(int))]


def test_identify_leaves_cost_follows_the_leaves():
    """5,000 payloads of 12 KB in 16 MiB blocks, 15,000 leaves in 20 M slots: locating changes
    to the leaf costs less than comparing whole blocks (0.7 times); with a workgroup for every
    64 slots it cost 13 times as much. The bound lies between."""
    n, block = 5000, 16 << 20
    arena = torch.randint(0, 256, (n * 12_288,), dtype=torch.uint8, device="cuda")
    batch = g.Batch.from_arena(arena, np.arange(n, dtype=np.uint64) * np.uint64(12_288), np.full(n, 12_000, np.uint64), block)
    blocks, leaves = g.fp_chunks(batch, with_leaves=True)
    regions = np.array([0, n], np.uint64)
    ws = g.workspace(leaves.numel() + n)
    say("identify leaves cost")

    def cost(call, recorded):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        best = float("inf")
        for _ in range(4):
            a.record()
            call(batch, recorded, regions, ws)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    whole, located = cost(g.identify_weights, blocks), cost(g.identify_leaves, leaves)
    assert located < 3 * whole, (whole, located)


def test_identify_leaves_beyond_one_launch():
    """262,145 payloads of a few bytes in 16 MiB blocks, 2^30 leaf slots and 4,096 more: one
    workgroup for every 64 of them is more than one launch holds. The largest and the last
    payloads differ, and one in the part of the second launch."""
    rng = np.random.default_rng(9200)
    n, block, per = (1 << 18) + 1, 16 << 20, 4096
    lens = rng.integers(1, 60, n).astype(np.uint64)
    offs = np.arange(n, dtype=np.uint64) * np.uint64(64)
    arena = torch.randint(0, 256, (64 * n,), dtype=torch.uint8, device="cuda")
    batch = g.Batch.from_arena(arena, offs, lens, block)
    say("identify leaves beyond one launch", batch.n_blocks * per)
    _, recorded = g.fp_chunks(batch, with_leaves=True)
    change = np.array([0, int(lens.argmax()), 131_073, n - 2, n - 1])
    arena[torch.from_numpy(64 * change).cuda()] ^= 1
    regions = np.append(np.arange(0, n, 1000), n).astype(np.uint64)
    match, first_diff, weight = g.identify_leaves(batch, recorded, regions)
    want = np.full(n, oracle.NO_DIFF, np.uint64)
    want[change] = 0
    assert np.array_equal(u64(first_diff), want)
    match = match.reshape(n, per)
    assert np.array_equal(match[:, 0].cpu().numpy() == 0, want == 0) and bool((match[:, 1:] == 1).all())
    assert weight.cpu().numpy().tolist() == [int((want[a:b] != 0).all()) for a, b in
                                             zip(regions[:-1].astype(int), regions[1:].astype(int))]

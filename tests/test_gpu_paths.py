"""Bit-exact parity with the oracle where a path changes form: staging of few
segments, remainders and edges of the kernels' tiles.
"""
import time

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2008_10596_amd import ckpt as K
from tests.gpu_common import assert_dense, check_full, check_restored, d2h, host, log, random_allocs, register_all

pytestmark = pytest.mark.gpu

MiB = 1 << 20


@pytest.mark.parametrize("sizes, zero", [
    ([MiB, MiB], (0,)),                          # two segments, the first all ZERO
    ([MiB, MiB], ()),
    ([MiB + 17, 900000, 5], ()),                 # short tails: segments shorter than their slot
    ([MiB // 2, MiB, MiB, MiB // 2, MiB], (1,)),   # four segments, less than four slots of bytes
    ([100] * 1000, ()),                          # many short chunks: 4 segments, 112 KB
])
def test_few_segments_stay_in_their_staging(sizes, zero):
    """Fewer serialized bytes than four segment slots: every segment of a
    drain and of a refill (with an increment staged behind it) lies inside the
    staging, and results equal the oracle's."""
    C = 4096
    log("%d allocations, zero %s" % (len(sizes), zero))
    tensors = random_allocs(sizes, seed=71, zero=zero)
    ctx = K.Context(chunk_bytes=C, segment_mib=1)
    register_all(ctx, tensors)
    img = ctx.checkpoint()
    ref = O.checkpoint([host(t) for t in tensors], C)
    check_full(img, ref, tensors, C)
    tensors[-1][:3] = 9
    d = ctx.checkpoint(mode=K.CKPT_INCREMENTAL, base=img)
    dsts = [torch.full_like(t, 0x5A) for t in tensors]
    rc, rep = ctx.restore(img, dsts, delta=d)
    assert rc == K.CKPT_OK and rep["n_bad"] == 0
    check_restored(dsts, tensors)
    for x in (d, img, ctx):
        x.close()


@pytest.mark.parametrize("n, C", [(1, 4096), (15, 4096), (16, 4096), (17, 4096), (1024, 4096), (1025, 4096),
                                  (16500, 1024), (40000, 16), (70, 4112), (70, 65536), (9, 262144)])
def test_gather_tiles_and_pieces(n, C):
    """The gather at the edges of its tiles (16 to 1024 chunks) and pieces
    (4 KiB), to device staging and straight to host memory: DATA equals the
    oracle's for a full image and for an increment from the allocations."""
    log("gather of %d chunks of %d" % (n, C))
    tensors = random_allocs([(n - n // 3) * C - C // 2 - 7, n // 3 * C + 1], seed=72)
    tensors[0][:n // 5 * C] = 0
    ref = O.checkpoint([host(t) for t in tensors], C)
    base = None
    for flags in (0, K.CKPT_DRAIN_DIRECT):
        ctx = K.Context(chunk_bytes=C, flags=flags)
        register_all(ctx, tensors)
        img = ctx.checkpoint()
        check_full(img, ref, tensors, C)
        if base is None:
            base = img
        else:
            img.close()
    tensors[0][::7 * C] += 1
    tensors[1][-1:] += 1
    dref = O.delta([host(t) for t in tensors], C, ref["crc"])
    d = ctx.checkpoint(mode=K.CKPT_INCREMENTAL, base=base)
    assert np.array_equal(d.dirty_ids, dref["dirty_ids"]) and np.array_equal(d.data, dref["delta"])
    for x in (d, base, ctx):
        x.close()


@pytest.mark.parametrize("C", [16, 1024, 4096, 65536])
def test_every_tail_length(C):
    """Chunks ending 0..15 bytes after a 16-byte piece, alone and behind a full
    chunk, in every pass: pack, hash, restore; the restore writes no byte past
    a destination's end."""
    sizes = [r for r in range(1, 33)] + [C + r for r in range(16)]
    tensors = random_allocs(sizes, seed=73, zero=(3, 40))
    ctx = K.Context(chunk_bytes=C)
    register_all(ctx, tensors)
    img = ctx.checkpoint()
    ref = O.checkpoint([host(t) for t in tensors], C)
    check_full(img, ref, tensors, C)
    for t in tensors[::3]:
        t[-1:] += 1
    dref = O.delta([host(t) for t in tensors], C, ref["crc"])
    d = ctx.checkpoint(mode=K.CKPT_INCREMENTAL, base=img)
    assert np.array_equal(d.crc, dref["crc"]) and np.array_equal(d.flags, dref["flags"])
    assert np.array_equal(d.dirty_ids, dref["dirty_ids"]) and np.array_equal(d.data, dref["delta"])
    pools = [torch.full((s + 32,), 0x5A, dtype=torch.uint8, device="cuda") for s in sizes]
    rc, rep = ctx.restore(img, [p[:s] for p, s in zip(pools, sizes)], delta=d)
    assert rc == K.CKPT_OK and rep["n_bad"] == 0
    for p, t, s in zip(pools, tensors, sizes):
        assert torch.equal(p[:s], t) and bool((p[s:] == 0x5A).all())
    for x in (d, img, ctx):
        x.close()


@pytest.mark.parametrize("C", [4112, 5120, 8192, 16384, 65536, 262144])
def test_long_chunks_that_turn_non_zero(C):
    """One wave per chunk of several batches: chunks (full and short) whose
    first non-zero byte is at the edges of pieces, rounds and batches, or that
    are all ZERO; over the pack, the dense image, the hash pass and the
    restore."""
    log("long chunks, C=%d" % C)
    at = sorted({p for e in (0, 16, 1024, 4096, 8192, C) for p in (e - 1, e, e + 1) if 0 <= p < C} | {C // 2, C - 17})
    tails = [1, 15, 16, 1023, 1040, 4096, 4097, C - 1]
    tensors = []
    for first in at:                       # a ZERO chunk, one non-zero from `first` on, a short one
        t = torch.zeros(2 * C + tails[len(tensors) % len(tails)], dtype=torch.uint8, device="cuda")
        t[C + first:C + first + 1 + len(tensors) % 3] = 0x80 + len(tensors)
        if len(tensors) % 2:
            t[-1] = 5
        tensors.append(t)
    tensors += random_allocs([3 * C, C + 33], seed=74)
    ctx = K.Context(chunk_bytes=C, flags=K.CKPT_KEEP_DENSE)
    register_all(ctx, tensors)
    img = ctx.checkpoint()
    ref = O.checkpoint([host(t) for t in tensors], C)
    check_full(img, ref, tensors, C)
    p, nb = img.dense_ptr
    assert_dense(d2h(p, nb), ref["dense"][:nb], [t.numel() for t in tensors], C, ref["flags"])
    tensors[0].zero_()
    tensors[1][-1:] += 1
    dref = O.delta([host(t) for t in tensors], C, ref["crc"])
    d = ctx.checkpoint(mode=K.CKPT_INCREMENTAL, base=img)
    assert np.array_equal(d.crc, dref["crc"]) and np.array_equal(d.flags, dref["flags"])
    assert np.array_equal(d.dirty_ids, dref["dirty_ids"]) and np.array_equal(d.data, dref["delta"])
    dsts = [torch.full_like(t, 0x5A) for t in tensors]
    rc, rep = ctx.restore(img, dsts, delta=d)
    assert rc == K.CKPT_OK and rep["n_bad"] == 0
    check_restored(dsts, tensors)
    for x in (d, img, ctx):
        x.close()


@pytest.mark.parametrize("n, big", [(1, 0), (1, 1), (63, 0), (64, 1), (65, 1), (128, 0), (129, 1), (700, 1)])
def test_table_tiles_and_long_rows(n, big):
    """The table's scan in tiles of 64 rows and its map in pieces of long rows
    (over 4096 chunks, cut at 16384), at their edges: plain call, replayed
    graph, allocation-free call and server give the oracle's image."""
    C = 16
    log("table of %d rows, long rows %d" % (n, big))
    rng = np.random.default_rng(n)
    sizes = [int(x) for x in rng.integers(1, 200, n)]
    sizes[n // 3] = 0 if n > 64 else 1      # one empty allocation (two would share address 0)
    if big:
        for k, chunks in zip((0, n // 2, n - 1), (4096, 4097, 2 * 16384 + 1)):
            sizes[k] = chunks * C - 5
    tensors = random_allocs(sizes, seed=75, zero=(n // 3,))
    ref = O.checkpoint([host(t) for t in tensors], C)
    for flags in (0, K.CKPT_GRAPH):
        ctx = K.Context(chunk_bytes=C, flags=flags)
        register_all(ctx, tensors)
        for _ in range(2):
            img = ctx.checkpoint()
            check_full(img, ref, tensors, C)
            img.close()
        ctx.close()
    ctx = K.Context(chunk_bytes=C)
    register_all(ctx, tensors)
    N, D = ctx.noalloc_sizes()
    dense = torch.zeros(max(D, 16), dtype=torch.uint8, device="cuda")
    crc = torch.zeros(max(N, 1), dtype=torch.int32, device="cuda")
    fl = torch.zeros(max(N, 1), dtype=torch.uint8, device="cuda")
    ctx.checkpoint_noalloc(crc, fl, dense=dense)
    assert np.array_equal(host(crc).view(np.uint32)[:N], ref["crc"]) and np.array_equal(host(fl)[:N], ref["flags"])
    assert_dense(host(dense)[:D], ref["dense"][:D], sizes, C, ref["flags"])
    ctx.close()
    srv = K.Server(chunk_bytes=C, staging_budget=64 * MiB)
    res = srv.wait(srv.submit(K.CKPT_REQ_CHECKPOINT, tensors))
    assert res["status"] == K.CKPT_OK
    check_full(res["image"], ref, tensors, C)
    res["image"].close()
    srv.close()


@pytest.mark.parametrize("n", [1, 4095, 4096, 4097, 3 * 4096 + 17, 2048 * 4096, 2048 * 4096 + 3])
def test_selection_tiles(n):
    """The selection at the edges of its tiles (4096 items) and of the forms
    that add up the tiles' totals (2048 tiles): serialized offsets, dirty ids
    and restores of a base with an increment, against the oracle."""
    C = 16
    log("selection over %d chunks" % n)
    tensors = random_allocs([n * C - 3] if n < 100 else [n // 3 * C - 1, 5 * C, (n - n // 3 - 5) * C], seed=76)
    tensors[0][::3 * C] = 0
    tensors[-1][: n // 7 * C] = 0
    ctx = K.Context(chunk_bytes=C)
    register_all(ctx, tensors)
    img = ctx.checkpoint()
    ref = O.checkpoint([host(t) for t in tensors], C)
    check_full(img, ref, tensors, C)
    tensors[0][::11 * C] += 1
    tensors[-1][-1:] += 1
    dref = O.delta([host(t) for t in tensors], C, ref["crc"])
    d = ctx.checkpoint(mode=K.CKPT_INCREMENTAL, base=img)
    assert np.array_equal(d.dirty_ids, dref["dirty_ids"]) and np.array_equal(d.data, dref["delta"])
    dsts = [torch.full_like(t, 0x5A) for t in tensors]
    rc, rep = ctx.restore(img, dsts, delta=d)
    assert rc == K.CKPT_OK and rep["n_bad"] == 0
    check_restored(dsts, tensors)
    for x in (d, img, ctx):
        x.close()


@pytest.mark.parametrize("total, zero", [(MiB, ()), (15 * MiB, (0, 1)), (16 * MiB, ()), (16 * MiB + 4096, (1,)), (40 * MiB, (0,))])
def test_drains_without_staging(total, zero):
    """Full checkpoints of at most one segment store to the image's pinned
    memory, small ones (16 MiB) before their serialized size is known; an
    increment's delta of up to 1 MiB does too, larger ones are staged; all
    ZERO.  Budgets refuse as a staged drain does."""
    C = 4096
    log("drain of %d bytes, zero %s" % (total, zero))
    sizes = [total // 2, total // 4 - 5, total - total // 2 - total // 4 - 11]
    tensors = random_allocs(sizes, seed=77, zero=zero)
    ctx = K.Context(chunk_bytes=C)
    register_all(ctx, tensors)
    img = ctx.checkpoint()
    ref = O.checkpoint([host(t) for t in tensors], C)
    check_full(img, ref, tensors, C)
    for n in (1, 255, 256, 257, 600):        # dirty chunks: up to and past 1 MiB of delta
        tensors[2][:min(n * C, tensors[2].numel())] += 1
        dref = O.delta([host(t) for t in tensors], C, ref["crc"])
        d = ctx.checkpoint(mode=K.CKPT_INCREMENTAL, base=img)
        assert np.array_equal(d.dirty_ids, dref["dirty_ids"]) and np.array_equal(d.data, dref["delta"])
        assert np.array_equal(d.crc, dref["crc"]) and np.array_equal(d.flags, dref["flags"])
        d.close()
    for t in tensors:
        t.zero_()
    d = ctx.checkpoint(mode=K.CKPT_INCREMENTAL, base=img)      # dirty ids without DATA
    dref = O.delta([host(t) for t in tensors], C, ref["crc"])
    assert np.array_equal(d.dirty_ids, dref["dirty_ids"]) and d.data.size == 0
    allzero = ctx.checkpoint()
    assert allzero.info()["serialized_bytes"] == 0 and (allzero.flags == 3).all()
    dense = sum(-(-s // 16) * 16 for s in sizes)
    for x in (d, allzero, img, ctx):
        x.close()
    tensors = random_allocs(sizes, seed=78)
    for budget, ok in ((2 * dense, True), (2 * dense - 16, False)):
        ctx = K.Context(chunk_bytes=C, staging_budget=budget)
        register_all(ctx, tensors)
        if ok:
            ctx.checkpoint().close()
        else:
            with pytest.raises(K.CkptError) as e:
                ctx.checkpoint()
            assert e.value.status == K.CKPT_E_BUDGET
        ctx.close()


@pytest.mark.parametrize("segment_mib", [0, 1, 0xFFFFFFFF])
def test_restore_refuses_flags_that_do_not_match(segment_mib):
    """Flags that select other than the serialized bytes: the restore is
    refused, and none of that image's chunks is written; read from the
    image's memory, in segments and in one pass."""
    C = 4096
    tensors = random_allocs([3 * MiB, 777, 2 * MiB + 5], seed=79)
    tensors[0][: 4 * C] = 0
    ctx = K.Context(chunk_bytes=C, segment_mib=segment_mib)
    register_all(ctx, tensors)
    img = ctx.checkpoint()
    before = [t.clone() for t in tensors]
    tensors[1][:] += 1
    d = ctx.checkpoint(mode=K.CKPT_INCREMENTAL, base=img)
    for image, g in ((img, 1), (img, 9), (d, int(d.dirty_ids[0]))):
        dsts = [torch.full_like(t, 0x5A) for t in tensors]
        image.flags[g] ^= 1                 # one chunk more, or less, than DATA holds
        with pytest.raises(K.CkptError) as e:
            ctx.restore(img, dsts, delta=d)
        image.flags[g] ^= 1
        assert e.value.status == K.CKPT_E_INVAL
        if image is img:
            assert all(bool((t == 0x5A).all()) for t in dsts)
        else:                               # the base was written, its increment not
            check_restored(dsts, before)
    dsts = [torch.full_like(t, 0x5A) for t in tensors]
    rc, rep = ctx.restore(img, dsts, delta=d)
    assert rc == K.CKPT_OK
    check_restored(dsts, tensors)
    for x in (d, img, ctx):
        x.close()


def test_restore_of_a_batch_s_images():
    """Images of one batch share a pinned block (their CRC and flag arrays
    start anywhere in it): restores of each, plain and through the server."""
    C = 4096
    sets = [random_allocs([C * (i + 1) + i, 5000 + i], seed=80 + i) for i in range(5)]
    ctxs = []
    for t in sets:
        ctxs.append(K.Context(chunk_bytes=C))
        register_all(ctxs[-1], t)
    imgs = K.checkpoint_batch(ctxs)
    srv = K.Server(chunk_bytes=C, staging_budget=64 * MiB)
    for ctx, img, t in zip(ctxs, imgs, sets):
        dsts = [torch.full_like(x, 0x5A) for x in t]
        rc, rep = ctx.restore(img, dsts)
        assert rc == K.CKPT_OK
        check_restored(dsts, t)
        dsts = [torch.full_like(x, 0x5A) for x in t]
        assert srv.wait(srv.submit(K.CKPT_REQ_RESTORE, dsts, image=img))["status"] == K.CKPT_OK
        check_restored(dsts, t)
    srv.close()
    for x in imgs + ctxs:
        x.close()


@pytest.mark.parametrize("aux", [1, 2, 5])
def test_server_finishes_and_refills_side_by_side(aux):
    """A burst of checkpoints and restores, with images that hold nothing
    (all ZERO), one byte, a chunk less and more than a tile of the selection:
    every image equals the plain path's, whatever number of workers finish them."""
    C = 4096
    sets = [random_allocs(s, seed=200 + i, zero=z) for i, (s, z) in enumerate([
        ([3 * C, 5000], (0, 1)), ([1], ()), ([C], ()), ([255 * C, 7], ()), ([256 * C], (0,)), ([257 * C + 1, 16], ()),
        ([2 * MiB, 100, 3 * MiB + 5], (1,)), ([9 * MiB], ())])]
    plain = []
    for t in sets:
        with K.Context(chunk_bytes=C) as ctx:
            register_all(ctx, t)
            plain.append(ctx.checkpoint())
    srv = K.Server(chunk_bytes=C, staging_budget=256 * MiB, aux_threads=aux, step_bytes=4 * MiB)
    for _ in range(3):
        dsts = [[torch.full_like(x, 0x5A) for x in t] for t in sets]
        tickets = []
        for t, d, img in zip(sets, dsts, plain):
            tickets.append((srv.submit(K.CKPT_REQ_CHECKPOINT, t), img))
            tickets.append((srv.submit(K.CKPT_REQ_RESTORE, d, image=img), None))
        for ticket, want in tickets:
            r = srv.wait(ticket)
            assert r["status"] == K.CKPT_OK
            if want:
                for k in ("crc", "flags", "data"):
                    assert np.array_equal(getattr(r["image"], k), getattr(want, k)), k
                r["image"].close()
        for d, t in zip(dsts, sets):
            check_restored(d, t)
    srv.close()
    for x in plain:
        x.close()


@pytest.mark.parametrize("rows, chunks, C, block, waves", [
    (1, 1, 4096, 1024, 1), (64, 200, 4096, 1024, 1), (65, 200, 4096, 1024, 1),   # rows that fit the arguments, or not
    (3, 8191, 4096, 1024, 1), (64, 8192, 4096, 1024, 1), (7, 8193, 4096, 1024, 1),   # chunks that do, or not
    (40, 3000, 1024, 1024, 1), (64, 700, 16384, 1024, 1), (64, 700, 65536, 256, 4), (33, 2000, 4096, 64, 1),
])
def test_noalloc_tables_in_arguments(rows, chunks, C, block, waves):
    """The allocation-free pass with its table in the kernel's arguments and
    with a laid-out one, at the edges of both, an empty row between: packed,
    against a base, and hash-only, equal to the oracle's."""
    rng = np.random.default_rng(rows * 1000 + chunks)
    filled = max(rows - 1, 1)   # and one empty row: only one allocation can be at address 0
    cuts = np.sort(rng.choice(np.arange(1, chunks), filled - 1, replace=False)) if filled > 1 else np.zeros(0, int)
    sizes = [int(p) * C - int(rng.integers(0, C)) for p in np.diff(np.concatenate([[0], cuts, [chunks]]))]
    if rows > 1:
        sizes.insert(rows // 2, 0)
    tensors = random_allocs(sizes, seed=rows + chunks, zero=(rows // 3,))
    ref = O.checkpoint([host(t) for t in tensors], C)
    ctx = K.Context(chunk_bytes=C, block_threads=block, waves_per_chunk=waves)
    register_all(ctx, tensors)
    N, D = ctx.noalloc_sizes()
    assert N == chunks
    dense = torch.zeros(max(D, 16), dtype=torch.uint8, device="cuda")
    crc = torch.zeros(N, dtype=torch.int32, device="cuda")
    fl = torch.zeros(N, dtype=torch.uint8, device="cuda")
    ctx.checkpoint_noalloc(crc, fl, dense=dense)
    assert np.array_equal(host(crc).view(np.uint32), ref["crc"]) and np.array_equal(host(fl), ref["flags"])
    assert_dense(host(dense)[:D], ref["dense"][:D], sizes, C, ref["flags"])
    base = crc.clone()
    base[::3] += 1
    dirty = np.zeros(N, bool)
    dirty[::3] = True
    for mode in (K.CKPT_FULL, K.CKPT_INCREMENTAL):
        crc.zero_()
        fl.fill_(0x55)
        ctx.checkpoint_noalloc(crc, fl, dense=dense if mode == K.CKPT_FULL else None, base_crc=base, mode=mode)
        assert np.array_equal(host(crc).view(np.uint32), ref["crc"])
        got = host(fl)
        assert np.array_equal((got & 1) != 0, (ref["flags"] & 1) != 0)
        assert np.array_equal((got & 2) != 0, dirty)
    ctx.close()


@pytest.mark.parametrize("filled", [1, 100, 511, 512, 513, 4000])
def test_small_drains_keep_little_more_than_they_hold(filled):
    """A drain of 16 MiB with few non-ZERO chunks: the image is the oracle's,
    and its pinned memory follows what it holds (an eighth of the dense bytes
    is 512 chunks)."""
    C = 4096
    tensors = random_allocs([16 * MiB], seed=90, zero=(0,))
    tensors[0].view(-1, C)[:filled] = random_allocs([filled * C], seed=91)[0].view(-1, C)
    ctx = K.Context(chunk_bytes=C)
    register_all(ctx, tensors)
    ctx.checkpoint().close()
    before = K.host_memory()[0]
    img = ctx.checkpoint()
    check_full(img, O.checkpoint([host(t) for t in tensors], C), tensors, C)
    held = K.host_memory()[0] - before
    # the pool's slack: a quarter, and 4 MiB, of each of DATA and the CRC and flag block
    assert held <= (filled * C if filled <= 512 else 16 * MiB) * 5 // 4 + 16 * MiB // C * 5 + 2 * 6 * MiB
    dsts = [torch.full_like(t, 0x5A) for t in tensors]
    assert ctx.restore(img, dsts)[0] == K.CKPT_OK
    check_restored(dsts, tensors)
    img.close()
    ctx.close()


@pytest.mark.parametrize("C, waves", [(4112, 1), (8192, 1), (65536, 1), (262144, 1), (65536, 4)])
@pytest.mark.parametrize("rows", [6, 70])
def test_packs_above_4_KiB_store_zero_chunks(C, waves, rows):
    """Chunks above 4 KiB are stored whatever they hold: a dense buffer that
    held other bytes (the caller's, or the context's staging) has zeros where
    the memory has, and the whole dense image is the oracle's."""
    sizes = [2 * C, C + 33, 3 * C - 5, 1, C - 16, 2 * C + 1024] + [k % 5 * C + 7 * k + 1 for k in range(rows - 6)]
    tensors = random_allocs(sizes, seed=92, zero=(0, 1, 3))
    tensors[2][C:] = 0
    ref = O.checkpoint([host(t) for t in tensors], C)
    assert (ref["flags"] & 1).any()
    ctx = K.Context(chunk_bytes=C, waves_per_chunk=waves, flags=K.CKPT_NO_DRAIN)
    register_all(ctx, tensors)
    N, D = ctx.noalloc_sizes()
    dense = torch.full((D,), 0x5A, dtype=torch.uint8, device="cuda")
    crc = torch.zeros(N, dtype=torch.int32, device="cuda")
    fl = torch.zeros(N, dtype=torch.uint8, device="cuda")
    ctx.checkpoint_noalloc(crc, fl, dense=dense)
    assert np.array_equal(host(crc).view(np.uint32), ref["crc"]) and np.array_equal(host(fl), ref["flags"])
    assert np.array_equal(host(dense), ref["dense"][:D])
    saved = [t.clone() for t in tensors]
    for t in tensors:
        t.fill_(0x77)
    ctx.checkpoint().close()             # the staging holds other bytes now
    for t, x in zip(tensors, saved):
        t.copy_(x)
    img = ctx.checkpoint()
    assert np.array_equal(d2h(*img.dense_ptr), ref["dense"][:D])
    img.close()
    ctx.close()


@pytest.mark.parametrize("drain", [True, False])
def test_graph_replays_between_increments(drain):
    """A context that replays its captured graph and takes increments in
    between, against the graph's images and against increments: each equals
    the oracle's, and so do batches led by a context with a log of its own."""
    C = 4096
    tensors = random_allocs([MiB + 5, 70000, 4096], seed=93, zero=(1,))
    other = random_allocs([300000], seed=94)
    ctx = K.Context(chunk_bytes=C, flags=K.CKPT_GRAPH | (0 if drain else K.CKPT_NO_DRAIN))
    second = K.Context(chunk_bytes=C)
    register_all(ctx, tensors)
    register_all(second, other)
    base = base_crc = None
    for i in range(8):
        tensors[i % 3][i:i + 40] += 1
        ref = O.checkpoint([host(t) for t in tensors], C)
        if i % 4 == 3:
            img, b = K.checkpoint_batch([ctx, second])
            assert np.array_equal(b.crc, O.checkpoint([host(t) for t in other], C)["crc"])
            b.close()
        else:
            img = ctx.checkpoint()
        assert np.array_equal(img.crc, ref["crc"]) and np.array_equal(img.flags, ref["flags"])
        if drain:
            assert np.array_equal(img.data, ref["serialized"])
        if base is not None:
            base.close()
        base, base_crc = img, ref["crc"]
        for k in range(i % 3 + 1):                 # an odd and an even number of increments
            tensors[0][4096 * k + i] += 1
            dref = O.delta([host(t) for t in tensors], C, base_crc)
            d = ctx.checkpoint(mode=K.CKPT_INCREMENTAL, base=base)
            assert np.array_equal(d.crc, dref["crc"]) and np.array_equal(d.dirty_ids, dref["dirty_ids"])
            if drain:
                assert np.array_equal(d.data, dref["delta"])
            base.close()
            base, base_crc = d, dref["crc"]
    for x in (base, ctx, second):
        x.close()


@pytest.mark.parametrize("rows", [3, 64, 65])
def test_captured_noalloc_pass_reads_the_log_at_replay(rows):
    """An allocation-free pass captured into a graph, replayed with eager work
    between: after an allocation was exchanged for another (of the same size,
    then of a smaller one), the replay covers the one that is live then."""
    C = 4096
    sizes = [5 * C + 17 * k + 1 for k in range(rows)]
    tensors = random_allocs(sizes, seed=95, zero=(1,))
    ctx = K.Context(chunk_bytes=C, flags=K.CKPT_STREAM_ORDERED)
    register_all(ctx, tensors)
    N, D = ctx.noalloc_sizes()
    dense = torch.zeros(D, dtype=torch.uint8, device="cuda")
    crc = torch.zeros(N, dtype=torch.int32, device="cuda")
    fl = torch.zeros(N, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ctx.checkpoint_noalloc(crc, fl, dense=dense, stream=torch.cuda.current_stream())
    kept = []
    for i, size in enumerate([None, sizes[0], sizes[0], 2 * C + 5, None]):
        if size:
            kept.append(tensors.pop(0))      # its memory stays: a stale table would read it
            ctx.unregister(kept[-1])
            tensors.append(random_allocs([size], seed=96 + i)[0])
            ctx.register(tensors[-1])
        tensors[-1][3 + i:40] += 1
        for x in (dense, crc, fl):
            x.fill_(0x11)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        ref = O.checkpoint([host(t) for t in tensors], C)
        n = ref["n_chunks"]
        assert n <= N
        assert np.array_equal(host(crc).view(np.uint32)[:n], ref["crc"]) and np.array_equal(host(fl)[:n], ref["flags"])
        now = [t.numel() for t in tensors]
        bytes_ = sum(-(-s // 16) * 16 for s in now)
        assert_dense(host(dense)[:bytes_], ref["dense"][:bytes_], now, C, ref["flags"])
    del graph
    ctx.close()


@pytest.mark.parametrize("C, n, longest", [(8192, 1500, 8192), (1 << 20, 1500, 300000), (1 << 28, 300, 5 * MiB),
                                           (1 << 30, 40, 3 * MiB + 7)])
def test_gather_of_short_chunks_under_a_large_chunk_size(C, n, longest):
    """Allocations much shorter than a chunk, a few long ones among them:
    increments, direct drains and the server's images are the oracle's, and an
    increment of short allocations takes as long as with 4 KiB chunks."""
    log("%d short allocations, C=%d" % (n, C))
    sizes = [100 + 37 * k % 900 for k in range(n)]
    for k in (0, n // 2, n - 1):
        sizes[k] = longest
    sizes[n // 3] = 4097
    tensors = random_allocs(sizes, seed=97, zero=(5,))
    ref = O.checkpoint([host(t) for t in tensors], C)
    ctx = K.Context(chunk_bytes=C, flags=K.CKPT_DRAIN_DIRECT)
    register_all(ctx, tensors)
    img = ctx.checkpoint()
    check_full(img, ref, tensors, C)
    for t in tensors[::2]:
        t[-1:] += 1
    dref = O.delta([host(t) for t in tensors], C, ref["crc"])
    for flags in (0, K.CKPT_DRAIN_DIRECT):
        with K.Context(chunk_bytes=C, flags=flags) as other:
            register_all(other, tensors)
            d = other.checkpoint(mode=K.CKPT_INCREMENTAL, base=img)
            assert np.array_equal(d.dirty_ids, dref["dirty_ids"]) and np.array_equal(d.data, dref["delta"])
            d.close()
    srv = K.Server(chunk_bytes=C, staging_budget=64 * MiB)
    res = srv.wait(srv.submit(K.CKPT_REQ_CHECKPOINT, tensors))
    assert res["status"] == K.CKPT_OK
    check_full(res["image"], O.checkpoint([host(t) for t in tensors], C), tensors, C)
    for x in (res["image"], srv, img, ctx):
        x.close()
    short = [t for t in tensors if t.numel() < 1000]
    best = []
    for chunk in (4096, C):
        with K.Context(chunk_bytes=chunk) as c:
            register_all(c, short)
            base = c.checkpoint()
            for t in short:
                t += 1
            times = []
            for _ in range(10):
                t0 = time.perf_counter()
                c.checkpoint(mode=K.CKPT_INCREMENTAL, base=base).close()
                times.append(time.perf_counter() - t0)
            base.close()
            best.append(min(times))
    log("  increment of %d short allocations: %.0f us, with 4 KiB chunks %.0f us" % (len(short), best[1] * 1e6, best[0] * 1e6))
    assert best[1] < 5 * best[0] + 200e-6


@pytest.mark.parametrize("C", [16, 1008, 1024, 1040, 2048, 2064])
@pytest.mark.parametrize("zero", [0, 1])
def test_tiles_of_short_chunks(C, zero):
    """Chunks on both sides of the sizes at which the tile changes, in numbers
    around two tiles of 32 and of 64 for every workgroup, and many more than a
    group of results; random, and ZERO but for a chunk here and there: snapshot,
    refill and the allocation-free pass are the oracle's."""
    grid = torch.cuda.get_device_properties(0).multi_processor_count
    for n in (1, 63, 65, 64 * grid - 1, 64 * grid + 1, 128 * grid, 128 * grid + 33, 200 * grid + 7):
        t = random_allocs([n * C - min(C - 1, 5)], seed=98 + n)[0]
        if zero:
            keep = t[:: 37 * C].clone()
            t.zero_()
            t[:: 37 * C] = keep
        ref = O.checkpoint([host(t)], C)
        ctx = K.Context(chunk_bytes=C)
        ctx.register(t)
        img = ctx.checkpoint()
        check_full(img, ref, [t], C)
        dst = torch.full_like(t, 0x5A)
        assert ctx.restore(img, [dst])[0] == K.CKPT_OK and torch.equal(dst, t)
        N, D = ctx.noalloc_sizes()
        dense = torch.zeros(D, dtype=torch.uint8, device="cuda")
        crc = torch.zeros(N, dtype=torch.int32, device="cuda")
        fl = torch.zeros(N, dtype=torch.uint8, device="cuda")
        ctx.checkpoint_noalloc(crc, fl, dense=dense)
        assert np.array_equal(host(crc).view(np.uint32), ref["crc"]) and np.array_equal(host(fl), ref["flags"])
        assert np.array_equal(host(dense)[:t.numel()], host(t))
        img.close()
        ctx.close()

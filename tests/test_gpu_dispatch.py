"""Kernel variants chosen by size, each at the edges of its range, against the
oracle's decode of the same bytes."""
import numpy as np
import pytest

import oracle.zfo as zo
from paper_2602_08190_amd import datagen as g
from paper_2602_08190_amd import zf

import helpers as H
from conftest import gpu_available
from test_gpu_parity import check, decode_image, decode_staged, log, torch

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def cus():
    return torch().cuda.get_device_properties(0).multi_processor_count


def ans_mix(n_chunks, size, exact=False):
    """n_chunks ANS chunks of about (or exactly) `size` bytes: incompressible bytes (half a
    word a step and lane), one symbol (no words), flags, text, bytes that
    switch between rare and frequent (bursts of 64 words a step), and lengths
    around the 16-step blocks."""
    r = g.rng(n_chunks + size)
    parts = []
    for i in range(n_chunks):
        n = size if exact else max(1, size + int(r.integers(-70, 70)))
        k = i % 5
        if k == 0:
            parts.append(np.frombuffer(r.bytes(n), np.uint8))
        elif k == 1:
            parts.append(np.full(n, i % 256, np.uint8))
        elif k == 2:
            parts.append(r.choice(np.frombuffer(b"ANR", np.uint8), size=n, p=[0.2, 0.7, 0.1]))
        elif k == 3:
            parts.append(np.frombuffer(b"the quick brown fox. " * (n // 21 + 1), np.uint8)[:n])
        else:
            burst = (np.arange(n) // 64) % 8 == 0
            parts.append(np.where(burst, r.integers(0, 256, size=n), 7).astype(np.uint8))
    ce = [len(p) for p in parts]
    x = np.concatenate(parts)
    return zf.Column.compress(x, zf.ANS, chunk_elems=ce), x


@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("size", [90, 1100])
def test_ans_at_the_fused_models_limit(over, size):
    # work of 8 whole chunks per compute unit takes the fused model, one chunk
    # more the other
    n = 8 * cus() + over
    log("ans", n, "chunks of", size)
    col, x = ans_mix(n, size, exact=True)
    check([col], decode_image([col]), [x])


@pytest.mark.parametrize("size", [5000, 40000])
def test_ans_long_chunks(size):
    # thousands of words a chunk: the ring goes round many times
    col, x = ans_mix(15, size)
    check([col], decode_image([col]), [x])
    check([col], decode_image([col], persistent=True), [x])


@pytest.mark.parametrize("d", [-1, 0, 1])
def test_smallest_units(d):
    # columns of one smallest unit of each kind (2048 values, 256 elements,
    # 1,024 bytes of text, 8 KiB of plain copy) and a few, give or take one
    # value, planned with the default tiles
    cols, xs = [], []
    for k in (1, 3, 40):
        nb, ne, nt = 2048 * k + d, 256 * k + d, 1024 * k + d
        r = g.rng(100 * k + d)
        xs += [r.integers(-5, 10 ** 6, size=nb).astype(np.int32), r.integers(-5, 10 ** 6, size=nb),
               g.fixed16_column(nb, 30, k), r.integers(0, 7, size=nb).astype(np.int32), r.integers(0, 7, size=nb),
               g.decimal_column(nb, k, 100, 10 ** 6), g.sorted_runs_column(ne, 3, k),
               g.sorted_runs_column(ne, 3, k, dtype=np.int64), g.key_column(ne, k), g.orderkey_column(ne, k),
               g.text_column(nt, k), g.text_column(nt, k), g.text_column(nt, k),
               np.frombuffer(r.bytes(8192 * k + d), np.uint8)]
        codecs = [zf.FOR_BP, zf.FOR_BP, zf.DICT_BP, zf.DICT_BP, zf.DICT_BP, zf.F2I_BP, zf.RLE_DELTA_BP, zf.DELTA_BP,
                  zf.DSTRIDE_BP, zf.DSTREE, zf.SDICT_BP, zf.SDICT_COL, zf.SDICT_COL_ANS, zf.PLAIN]
        cols += [zf.Column.compress(x, c) for x, c in zip(xs[-14:], codecs)]
    check(cols, decode_image(cols), xs)
    for slot in (1 << 14, 1 << 20):
        outs, _ = decode_staged(cols, slot_bytes=slot)
        check(cols, outs, xs)


def f2i_bits(cols, outs, xs):
    for c, o, x in zip(cols, outs, xs):
        assert np.array_equal(o.view(np.uint64), x.view(np.uint64))
        assert np.array_equal(zo.decode(c.bytes()).view(np.uint64), x.view(np.uint64))


@pytest.mark.parametrize("n", [1, 127, 2048, 2049, 7001])
def test_f2i_exceptions_in_place(n):
    # exceptions nowhere, everywhere, at the ends of blocks and steps, in pairs
    r = g.rng(n)
    i = np.arange(n)
    cols, xs = [], []
    for where in (i < 0, i >= 0, i % 2 == 1, i % 128 == 127, (i % 2048 == 0) | (i % 2048 == 2047) | (i == n - 1),
                  r.random(n) < 0.1, (i // 3) % 5 == 2):
        x = r.integers(1, 10 ** 6, size=n) / 100.0
        x = np.where(where, r.random(n) * 1e-3, x)
        xs.append(x)
        cols.append(zf.Column.compress(x, zf.F2I_BP, chunk_elems=[n] if n < 5000 else [2047, 2051, n - 4098]))
    f2i_bits(cols, decode_image(cols), xs)
    f2i_bits(cols, decode_image(cols, persistent=True), xs)


@pytest.mark.parametrize("bits", [20, 53, 61])
def test_f2i_quotients_of_every_exponent(bits):
    # d / 10^e for every e, d up to 2^bits in magnitude, exact powers among
    # them: the same doubles as IEEE division
    cols, xs = [], []
    for e in range(19):
        r = g.rng(100 * bits + e)
        d = r.integers(-(1 << bits), 1 << bits, size=3 * 2048)
        d[:64] = [s * (1 << min(k, bits)) for k in range(32) for s in (1, -1)]
        x = d.astype(np.float64) / np.float64(10 ** e)
        xs.append(x)
        cols.append(zf.Column.compress(x, zf.F2I_BP))
    f2i_bits(cols, decode_image(cols), xs)
    f2i_bits(cols, decode_image(cols, persistent=True), xs)


@pytest.mark.parametrize("n_entries", [1, 3, 255, 256, 257, 1024, 1025])
def test_dict_views(n_entries):
    # dictionaries up to 4 KiB (gathered from LDS) and past it, whose sizes
    # end inside a 16-byte load; chunks off the output's 16-byte grid
    r = g.rng(n_entries)
    cols, xs = [], []
    for kind in ("i4", "i8", "c16"):
        n = 2 * 2048 + 333
        d = g.fixed16_dictionary(n_entries, 7) if kind == "c16" else \
            np.arange(n_entries).astype(kind) * 1000003 - 5
        code = np.concatenate([np.arange(n_entries), r.integers(0, n_entries, size=n)])
        xs.append(d[code])
        m = len(code)
        cols.append(zf.Column.compress(xs[-1], zf.DICT_BP, chunk_elems=[2049, 1, 2, m - 2052]))
    check(cols, decode_image(cols), xs)


@pytest.mark.parametrize("dtype", [np.int32, np.int64])
@pytest.mark.parametrize("unit", [64, 2048, 2049, 8192])
def test_spans_of_the_run_map(dtype, unit):
    # runs that start, end and lie across the 2048-element spans of the run
    # map, units of one span and around it, 64 groups' records and more in a
    # unit, a run longer than 2^26, chunks off the output's 16-byte grid
    r = g.rng(unit)
    runs = [np.full(5, 2048), np.full(300, 1), np.full(3, 2047), np.full(7, 2049), np.full(65 * 64, 1),
            r.integers(1, 5000, size=40), r.integers(1, 4, size=9000)]
    x = g.column_from_runs(np.concatenate(runs).astype(np.int64), 3, dtype)
    keys = g.orderkey_column(150_001, 4, dtype=dtype)
    ce = lambda n: [1, 3, 5, n // 2, n - n // 2 - 9]  # noqa: E731
    xs = [x, x, keys, g.key_column(60_007, 5, dtype=dtype), np.arange(70_001).astype(dtype) * 3]
    codecs = [zf.RLE_DELTA_BP, zf.DELTA_BP, zf.DSTREE, zf.DSTRIDE_BP, zf.DELTA_BP]
    cols = [zf.Column.compress(v, c, chunk_elems=ce(len(v))) for v, c in zip(xs, codecs)]
    check(cols, decode_image(cols, tiles={"GP": dict(unit=unit)}), xs)
    check(cols, decode_image(cols), xs)
    if unit == 8192 and dtype == np.int32:
        big = np.repeat(np.array([7, -3, 9], dtype), [(1 << 26) + 5, 3, 700])
        col = zf.Column.compress(big, zf.RLE_DELTA_BP, chunk_elems=[len(big)])
        out, = decode_image([col])
        assert np.array_equal(out, big)


def lz_containers():
    """Streams for the workgroup LZ77 kernel: batches of 64 matches of 33 and
    36 bytes (more pieces than a wave lists), a group of 512 sequences that
    all take two extension words, literal runs of 1 to 5,000 bytes, matches of
    every length 4..70, overlapping and long ones, empty sequences, batches
    that are not flat, chunks of 1..67 bytes and of 64 KiB."""
    r = g.rng(42)
    out = []

    def add(seqs, plain):
        nlit = sum(s[0] for s in seqs)
        out.append((H.lz_stream(seqs, r.bytes(nlit), plain), plain, zf.LZ77))

    def total(seqs):
        return sum(a + b for a, b, _ in seqs)
    for ml in (33, 36):
        seqs = [(4096, 0, 0)] + [(0, 0, 0)] * 63 + [(0, ml, int(r.integers(ml + 64 * ml, 4000))) for _ in range(640)]
        add(seqs, total(seqs))
    seqs = [(900, 0, 0)] + [(0, 0, 0)] * 63 + [(7 + i % 3, 34 + i % 5, 1 + (i * 7) % 6) for i in range(600)]
    add(seqs, total(seqs))
    seqs = [(n, 0, 0) for n in (1, 2, 3, 4, 5, 31, 32, 33, 255, 256, 257, 1023, 1025, 5000)]
    add(seqs, total(seqs))
    seqs = [(3000, 0, 0)] + [(0, 0, 0)] * 63 + [(i % 4, 4 + i % 67, 2900 - i % 60) for i in range(500)]
    add(seqs, total(seqs))
    for n in list(range(1, 68)) + [65535, 65536]:
        for gen in (H.random_lz, H.flat_lz):
            seqs, lits = gen(r, n)
            out.append((H.lz_stream(seqs, lits, n), n, zf.LZ77))
    seqs, lits = H.flat_lz(r, 40_000, empty_every=3)
    out.append((H.lz_stream(seqs, lits, 40_000), 40_000, zf.LZ77))
    return out


def test_lz_chunk_kernel_streams():
    chunks = lz_containers()
    log("lz chunk kernel,", len(chunks), "streams")
    blob = H.container(zf.BYTES, chunks)
    col = zf.Column.from_bytes(blob)
    check([col], decode_image([col]))
    check([col], decode_image([col], tiles={"LZ77": dict(unit=4)}))


@pytest.mark.parametrize("kind", ["zeros", "random", "dates", "period"])
@pytest.mark.parametrize("ce", [8192, 16384])
def test_lz_chunk_kernel_columns(kind, ce):
    n = 100_003
    x = {"zeros": np.zeros(n, np.int32), "random": np.frombuffer(g.rng(1).bytes(4 * n), np.int32),
         "dates": g.sorted_runs_column(n, 8, 3), "period": np.resize(np.arange(25, dtype=np.int32), n)}[kind]
    col = zf.Column.compress(x, zf.LZ77, chunk_elems=[1, ce] + [ce - 1] * (n // ce - 1) + [n - 1 - ce - (ce - 1) * (n // ce - 1)]
                             if kind != "zeros" else [ce] * (n // ce) + [n % ce])
    check([col], decode_image([col]), [x])


def test_lz_past_the_chunk_kernels_limit():
    # more tiny chunks than the workgroup kernel takes: the one-wave kernel
    n = 5 * 4 * cus() + 7
    x = g.text_column(20 * n, 9)
    col = zf.Column.compress(x, zf.LZ77, chunk_elems=[20] * n)
    check([col], decode_image([col]), [x])


@pytest.mark.parametrize("pinned", [True, False, None])
@pytest.mark.parametrize("slot", [1 << 12, 100_001, 1 << 22])
def test_staged_copies(pinned, slot):
    # transfers by the copy kernel (every column pinned), by copy commands
    # (none pinned, or one that is not), over one to many batches, three calls
    # in a row into other outputs
    xs = [g.uniform_i32(20_000, 5, 1 << 14, 1), g.fixed16_column(7_003, 300, 2), g.text_column(60_001, 3),
          g.text_column(44_444, 4), g.sorted_runs_column(30_011, 8, 5), np.zeros(0, np.int32)]
    codecs = [zf.FOR_BP, zf.DICT_BP, zf.SDICT_COL_ANS, zf.LZ77, zf.RLE_DELTA_BP, zf.FOR_BP]
    cols = [zf.Column.compress(x, c, chunk_bytes=(1 << 12, 1 << 14), seed=i,
                               pinned=(i != 2 if pinned is None else pinned))
            for i, (x, c) in enumerate(zip(xs, codecs))]
    plan = zf.Plan(cols, slot_bytes=slot)
    for timing in (False, True, False):
        outs = zf.empty_outputs(cols)
        plan.transfer_and_decompress(outs, timing=timing)
        t = plan.sync()
        if timing:
            assert t["wall_ms"] > 0 and t["h2d_ms"] > 0 and t["plain_bytes"] == sum(x.nbytes for x in xs)
        check(cols, [o.cpu().numpy() for o in outs], xs)


@pytest.mark.parametrize("first", [0, 1])
def test_staged_copies_of_long_ranges(first):
    # a batch of one long range goes by a copy command, the others by the
    # copy kernel, the dictionary with the first batch whichever that is
    xs = [np.frombuffer(g.rng(7).bytes(33 << 20), np.uint8), g.fixed16_column(70_003, 300, 2),
          g.text_column(300_001, 3)]
    codecs = [zf.PLAIN, zf.DICT_BP, zf.SDICT_COL]
    if first:
        xs, codecs = xs[::-1], codecs[::-1]
    cols = [zf.Column.compress(x, c, seed=i, pinned=True) for i, (x, c) in enumerate(zip(xs, codecs))]
    plan = zf.Plan(cols, slot_bytes=34 << 20, order=1)
    for _ in range(2):
        outs = zf.empty_outputs(cols)
        plan.transfer_and_decompress(outs)
        plan.sync()
        for o, x in zip(outs, xs):
            assert np.array_equal(o.cpu().numpy().reshape(-1).view(np.uint8), x.reshape(-1).view(np.uint8))


@pytest.mark.parametrize("n_cols", [1, 32, 33, 70])
@pytest.mark.parametrize("chain", [zf.LZ77, zf.ANS, zf.SDICT_COL_ANS, None])
def test_forked_launches_and_output_pointers(n_cols, chain):
    # output pointers with the launch (up to 32 columns) or in the table, and
    # kinds beside a chain of whole-chunk units on a second stream: two sets of
    # outputs in turn without a wait between, then a captured decode replayed
    T = torch()
    kinds = [(zf.FOR_BP, lambda i: g.uniform_i32(3_001 + i, 5, 1 << 14, i)),
             (zf.RLE_DELTA_BP, lambda i: g.sorted_runs_column(2_011 + i, 8, i)),
             (zf.DICT_BP, lambda i: g.fixed16_column(1_003 + i, 30, i))]
    xs, cols = [], []
    for i in range(n_cols):
        if chain is not None and i % 4 == 0:
            x, c = g.text_column(5_003 + i, i), chain
        else:
            c, make = kinds[i % 3]
            x = make(i)
        xs.append(x)
        cols.append(zf.Column.compress(x, c, chunk_bytes=(1 << 10, 1 << 12), seed=i))
    plan = zf.Plan(cols, device=0)
    img = zf.upload_image(plan, cols)
    a, b = zf.empty_outputs(cols), zf.empty_outputs(cols)
    for outs in (a, b, a):
        plan.decompress_async(img, img.numel(), outs)
    plan.sync()
    check(cols, [o.cpu().numpy() for o in a], xs)
    check(cols, [o.cpu().numpy() for o in b], xs)
    graph = T.cuda.CUDAGraph()
    s = T.cuda.Stream()
    s.wait_stream(T.cuda.current_stream())
    with T.cuda.graph(graph, stream=s):
        plan.decompress_async(img, img.numel(), b, stream=s)
    for k in range(3):
        for o in b:
            o.zero_()
        graph.replay()
        T.cuda.synchronize()
        check(cols, [o.cpu().numpy() for o in b], xs)


def test_ans_chunks_of_one_byte():
    # a byte that holds the whole model, first, last and between, at lengths
    # around the lanes and steps and off the 16-byte grid; then states and
    # words that no encoder writes: the oracle's verdict
    lens = [1, 15, 63, 64, 65, 1023, 1024, 1025, 5000, 70_000]
    vals = [0, 3, 77, 252, 255]
    parts = [np.full(n, vals[i % 5], np.uint8) for i, n in enumerate(lens * 2)]
    x = np.concatenate(parts)
    col = zf.Column.compress(x, zf.ANS, chunk_elems=[len(p) for p in parts])
    check([col], decode_image([col]), [x])
    n = 1000
    b = zo.encode(np.full(n, 77, np.uint8), zo.ANS)
    c = zo.chunks(b)[0]
    s0 = bytes(b[c["comp_off"]:c["comp_off"] + c["comp_len"]])
    for lane, state, words in ((0, 65537, []), (63, 1, []), (7, 1, [0]), (7, 1, [1]), (5, 65536, [0]),
                               (9, 1 << 31, []), (64, 0, [5] * 700)):
        s = np.frombuffer(s0 + np.array(words, np.uint16).tobytes(), np.uint8).copy()
        s[4:8] = np.frombuffer(np.uint32(len(words)).tobytes(), np.uint8)
        for j in range(64):
            if j == lane or lane == 64:
                s[528 + 4 * j:532 + 4 * j] = np.frombuffer(np.uint32(state).tobytes(), np.uint8)
        blob = H.container(zf.BYTES, [(s.tobytes(), n, zf.ANS)])
        try:
            want = zo.decode(blob)
        except zo.OracleError:
            want = None
        try:
            out, = decode_image([zf.Column.from_bytes(blob)])
        except zf.ZfError as e:
            assert e.status == zf.E_CORRUPT
            out = None
        log("ans of one byte: lane", lane, "state", state, len(words), "words:", "refused" if want is None else "taken")
        assert (want is None) == (out is None)
        assert want is None or np.array_equal(out, want)


@pytest.mark.parametrize("copies", [1, 6])
@pytest.mark.parametrize("kinds", ["few", "many", "chain"])
def test_staged_launches(kinds, copies):
    # batches of up to five launches go one by one, of more as a graph, those
    # with a chain beside other kinds on two streams; output pointers of up to
    # 32 columns with the launches; two sets of outputs in turn
    n, r = 5_003, g.rng(copies)
    make = [(zf.FOR_BP, lambda i: r.integers(0, 10 ** 6, size=n + i).astype(np.int32)),
            (zf.RLE_DELTA_BP, lambda i: g.sorted_runs_column(n + i, 8, i)),
            (zf.DICT_BP, lambda i: g.fixed16_column(n + i, 30, i))]
    if kinds != "few":
        make += [(zf.FOR_BP, lambda i: r.integers(0, 10 ** 6, size=n + i)),
                 (zf.DICT_BP, lambda i: r.integers(0, 7, size=n + i)),
                 (zf.RLE_DELTA_BP, lambda i: g.sorted_runs_column(n + i, 8, i, dtype=np.int64)),
                 (zf.F2I_BP, lambda i: g.decimal_column(n + i, i, 100, 10 ** 6))]
    if kinds == "chain":
        make += [(zf.ANS, lambda i: g.text_column(n + i, i)), (zf.LZ77, lambda i: g.text_column(n + i, i))]
    xs, cols = [], []
    for i in range(copies):
        for codec, m in make:
            xs.append(m(i))
            cols.append(zf.Column.compress(xs[-1], codec, pinned=True))
    for slot in (1 << 16, 1 << 24):
        plan = zf.Plan(cols, slot_bytes=slot)
        a, b = zf.empty_outputs(cols), zf.empty_outputs(cols)
        for outs in (a, b, a):
            plan.transfer_and_decompress(outs, timing=False)
        plan.sync()
        check(cols, [o.cpu().numpy() for o in a], xs)
        check(cols, [o.cpu().numpy() for o in b], xs)


@pytest.mark.parametrize("dtype", [np.int32, np.int64])
@pytest.mark.parametrize("run", [1, 4, 5, 8, 9, 40, 700, 5000])
def test_carried_windows(dtype, run):
    # run lengths on both sides of the carrying rule (36 bytes a run), units
    # that cut groups, chunks of odd lengths off the 128-byte grid, chunks
    # shorter than a window; outputs not a multiple of a line long
    r = g.rng(run)
    for unit in (64, 500, 4096):
        xs, cols = [], []
        for n in (1, 31, 257, 1023, 12_345, 70_001):
            lens = r.integers(1, 2 * run, size=n // run + 2) if run > 1 else r.integers(1, 3, size=n + 2)
            x = np.repeat(r.integers(-2 ** 31, 2 ** 31, size=len(lens)), lens).astype(dtype)[:n]
            xs.append(x)
            n = len(x)
            ce = None if n < 2000 else [777, 1, n // 2, n - n // 2 - 778]
            cols.append(zf.Column.compress(x, zf.RLE_DELTA_BP, chunk_elems=ce))
        tiles = {k: dict(unit=unit, waves_per_block=4) for k in ("RLE32", "RLE64")}
        check(cols, decode_image(cols, tiles=tiles), xs)
        check(cols, decode_image(cols, persistent=True, tiles=tiles), xs)


@pytest.mark.parametrize("run", [1, 3, 4, 5, 8, 40, 700])
def test_carried_windows_of_progressions(run):
    # DeltaStride and its tree on both sides of the carrying rule, int64 and
    # int32, units that cut groups, chunks off the 128-byte grid
    r = g.rng(100 + run)
    for dtype in (np.int32, np.int64):
        xs, cols = [], []
        for n in (1, 33, 1023, 20_011):
            parts, at = [], 0
            while sum(map(len, parts)) < n:
                k = int(r.integers(1, 2 * run)) if run > 1 else 1
                at += int(r.integers(1, 50))
                parts.append(at + np.arange(k))
                at += k
            x = np.concatenate(parts)[:n].astype(dtype)
            for codec in (zf.DSTRIDE_BP, zf.DSTREE):
                xs.append(x)
                ce = None if n < 2000 else [777, 1, n // 2, n - n // 2 - 778]
                cols.append(zf.Column.compress(x, codec, chunk_elems=ce))
        for unit in (64, 500, 4096):
            tiles = {k: dict(unit=unit, waves_per_block=4) for k in ("RLE32", "RLE64", "TREE")}
            check(cols, decode_image(cols, tiles=tiles), xs)
            check(cols, decode_image(cols, persistent=True, tiles=tiles), xs)

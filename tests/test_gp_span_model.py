"""A CPU model of the Group-Parallel decode wave as the kernels run it
(csrc/kernels.hpp: unit_rle, unit_tree_starts, unit_tree, expand_runs), over
product-encoded RLE, Delta, DeltaStride and DeltaStride-tree streams, both
widths, for the units the planner cuts (zf_chunk_units) and output addresses on
and off the 16- and 128-byte grids.

It follows the kernels step by step, 64 lanes at a time: the window of group
records, one per lane, and when it is read again; the words of a lane's field
through a view that ends with the group's; the run lengths' scan; the map of a
2048-element span, a word per lane, and the run of an element from the word's
count and the bits up to the element; the lane reads that fetch a run's value;
the windows of 64 x 16 bytes, carried from group to group or not by the
kernels' rule; the stores of whole windows, whole lines, 16 bytes and elements.
It asserts what the kernels rely on: a record read lies in the window, a fetched
run is one of the group's, 16-byte stores are aligned, and a unit writes each of
its elements once and no other.  Parity with the oracle then shows the algorithm
right independent of the GPU."""
import struct

import numpy as np
import pytest

import oracle.zfo as zo
from paper_2602_08190_amd import datagen as g
from paper_2602_08190_amd import zf

LANE = np.arange(64, dtype=np.int64)
U64 = np.uint64


def popc(x):
    return np.array([bin(int(v)).count("1") for v in x], np.int64)


class Wave:
    """One wave over one unit [e0, e1) of a chunk's stream s; output element p
    lies at address base + es * p."""

    def __init__(self, s, es, e0, e1, base, out):
        self.s, self.es, self.e0, self.e1, self.base, self.out = s, es, e0, e1, base, out
        self.M = U64((1 << (8 * es)) - 1)
        self.R = 16 // es
        self.open = np.zeros((self.R, 64), U64)

    # ---- the window of group records
    def rec_load(self, at, size, g0, ng):
        self.g0 = g0
        self.rec = [struct.unpack_from("<%dI" % (size // 4), self.s, at + size * min(g0 + l, ng - 1)) for l in range(64)]

    def rec_word(self, k, i):
        assert 0 <= i < 64, "a record outside the window"
        return self.rec[i][k]

    def rec_has(self, g):
        return (g - self.g0) % 2**32 <= 61

    # ---- a lane's packed field
    def field(self, at, end, j, w, wide):
        """Field j (per lane) of width w at byte `at`; dwords past `end` are zero."""
        n = 3 if wide else 2
        o = at + 4 * ((j * w) >> 5)
        v = [0] * 64
        for lane in range(64):
            x = 0
            for d in range(n):
                b = int(o[lane]) + 4 * d
                if 0 <= b and b + 4 <= end:
                    x |= struct.unpack_from("<I", self.s, b)[0] << (32 * d)
            v[lane] = (x >> (int(j[lane]) * w & 31)) & ((1 << w) - 1)
        return np.array(v, U64)

    def scan(self, x):
        return np.cumsum(x.astype(U64), dtype=U64) & self.M

    def lengths(self, r, last):
        wide = bool((r >> U64(26)).any())
        incl = np.cumsum(r, dtype=U64)
        total = int(incl[last]) if wide else int(incl[last]) & 0xFFFFFFFF
        return incl & U64(0xFFFFFFFF), total

    # ---- stores
    def put(self, p, x):
        assert self.e0 <= p < self.e1, "a store outside the unit"
        assert self.out[p] is None, "an element stored twice"
        self.out[p] = int(x)

    def put16(self, p, val, lane):
        a = self.base + self.es * p
        assert a % 16 == 0, "a 16-byte store off its grid"
        for i in range(self.R):
            self.put(p + i, val[i, lane])

    # ---- expansion of one group
    def expand(self, carry, lo_off, next_off, act, start, v, stride):
        R, es = self.R, self.es
        WIN, SPAN, LINE = 64 * R, 2048, 128 // es
        ua, ub = self.e0, self.e1
        ia, ib = max(ua, lo_off), min(ub, next_off)
        if ia >= ib:
            return
        cnt = int(act.sum())
        lo = ua if carry else ia
        w0 = lo - ((self.base + es * lo) & (127 if carry else 15)) // es
        sh = (R * LANE) & 31
        upto = (2 << sh) - 1
        for S in range(w0 + (ia - w0) // WIN * WIN, ib, SPAN):
            words = np.zeros(64, np.int64)
            for j in np.flatnonzero(act):
                rel = (int(start[j]) - S) % 2**32
                if rel < SPAN:
                    words[rel >> 5] |= 1 << (rel & 31)
            c = popc(words)
            before = np.cumsum(c) - c + int((act & (start.astype(np.int64) < S)).sum()) - 1
            for W in range(S, min(S + SPAN, ib), WIN):
                word = ((W - S) // 8 + ((R * LANE) >> 5) * 4) // 4
                b = words[word]
                run = before[word] + popc(b & upto)
                p = W + R * LANE
                val = np.zeros((R, 64), U64)
                for i in range(R):
                    if i:
                        run = run + ((b >> (sh + i)) & 1)
                    used = (p + i >= ia) & (p + i < ib)
                    assert ((run >= 0) & (run < cnt))[used].all(), "a run outside the group"
                    src = run & 63
                    x = v[src]
                    if stride is not None:
                        d = stride[src] if isinstance(stride, np.ndarray) else np.full(64, U64(stride))
                        x = x + d * ((p + i) % 2**32).astype(U64)
                    val[i] = x & self.M
                if carry and W < ia:
                    for i in range(R):
                        val[i] = np.where(p + i < ia, self.open[i], val[i])
                if carry and not (W + WIN <= ib or ib == ub):
                    self.open = val
                    continue
                whole = carry and W >= lo and W + WIN <= ib
                for lane in range(64):
                    q = int(p[lane])
                    line = q - ((R * lane) & (LINE - 1))
                    if whole or (carry and line >= lo and line + LINE <= ib):
                        assert (self.base + es * line) % 128 == 0, "a whole line off its grid"
                        self.put16(q, val, lane)
                    elif q >= lo and q + R <= ib:
                        self.put16(q, val, lane)
                    else:
                        for i in range(R):
                            if lo <= q + i < ib:
                                self.put(q + i, val[i, lane])


def run_rle(w, codec, n, g0):
    """unit_rle: RLE_DELTA_BP, DELTA_BP and DSTRIDE_BP."""
    s, wide = w.s, w.es == 8
    DS = codec == zf.DSTRIDE_BP
    nr, ng, roff = struct.unpack_from("<III", s, 0)
    U = lambda x: U64(x) & w.M  # noqa: E731
    w.rec_load(16, 32, g0, ng)

    def load(gr):
        i = gr - w.g0
        G = dict(goff=w.rec_word(0, i), next=w.rec_word(0, i + 1) if gr + 1 < ng else n)
        G["base"] = U(w.rec_word(4, i) | w.rec_word(5, i) << 32)
        G["dmin"] = U(w.rec_word(6, i) | w.rec_word(7, i) << 32)
        G["cnt"] = cnt = min(64, nr - gr * 64)
        r1, r2 = w.rec_word(1, i), w.rec_word(2, i)
        wd = (r2 >> 8) & 0xFF if DS else 0
        at, G["w"] = (r1 + 8, r2 & 0xFF) if DS else (r2, r1)
        end = at + 4 * (((cnt - 1) * G["w"] + 31) // 32)
        dend = end + 4 * ((cnt * wd + 31) // 32)
        assert dend <= len(s)
        k = gr * 64 + LANE
        G["r"] = np.array([1 if codec == zf.DELTA_BP else
                           struct.unpack_from("<I", s, roff + 4 * int(x))[0] if x < nr else 0 for x in k], U64)
        G["f"] = w.field(at, end, np.maximum(LANE - 1, 0), G["w"], wide)
        if DS:
            G["d"] = w.field(end, dend, LANE, wd, wide)
            G["gmin"] = U(struct.unpack_from("<Q", s, r1)[0])
        return G

    if codec == zf.DELTA_BP:
        for gr in range(g0, ng, 4):
            if gr - w.g0 > 63 - 4:
                w.rec_load(16, 32, gr, ng)
            for k, G in enumerate([load(min(gr + k, ng - 1)) for k in range(4)]):
                assert gr + k < ng and G["goff"] + G["cnt"] == G["next"]
                delta = np.where(LANE > 0, G["dmin"] + G["f"], G["base"])
                v = w.scan(np.where(LANE < G["cnt"], delta, U64(0)))
                for lane in range(G["cnt"]):
                    if w.e0 <= G["goff"] + lane < w.e1:
                        w.put(G["goff"] + lane, v[lane])
                if G["next"] >= w.e1:
                    return
    carry = (not DS or wide) and n // 5 >= nr
    gr, cur = g0, load(g0)
    while True:
        more = cur["next"] < w.e1
        if more:
            if not w.rec_has(gr):
                w.rec_load(16, 32, gr, ng)
            nxt = load(gr + 1)
        act = LANE < cur["cnt"]
        r = np.where(act, cur["r"], U64(0))
        incl, total = w.lengths(r, cur["cnt"] - 1)
        assert cur["goff"] + total == cur["next"]
        start = (U64(cur["goff"]) + incl - r) & U64(0xFFFFFFFF)
        if DS:
            stride = np.where(act, (cur["dmin"] + cur["d"]) & w.M, U64(0))
            f = np.where(act, (stride * r) & w.M, U64(0))
            gap = np.where(act & (LANE >= 1), (cur["gmin"] + cur["f"]) & w.M, U64(0))
            st = (cur["base"] + (w.scan(f) - f) + w.scan(gap)) & w.M
            v = (st - stride * start) & w.M
        else:
            stride = None
            v = w.scan(np.where(act, np.where(LANE > 0, cur["dmin"] + cur["f"], cur["base"]), U64(0)))
        w.expand(carry, cur["goff"], cur["next"], act, start, v, stride)
        if not more:
            return carry
        gr, cur = gr + 1, nxt


def run_tree_starts(w, n, g0):
    """unit_tree_starts: the starts of a DSTREE chunk (n of them)."""
    s = w.s
    Q, ng = struct.unpack_from("<II", s, 8)
    w.rec_load(32, 32, g0, ng)

    def load(gr):
        i = gr - w.g0
        poff, widths = w.rec_word(1, i), w.rec_word(2, i)
        cnt = min(64, Q - 64 * gr)
        wv, wl = widths & 0xFF, (widths >> 8) & 0xFF
        vend = poff + 4 * ((cnt * wv + 31) // 32)
        lend = vend + 4 * ((cnt * wl + 31) // 32)
        assert lend <= len(s)
        return dict(goff=w.rec_word(0, i), next=w.rec_word(0, i + 1) if gr + 1 < ng else n, cnt=cnt,
                    base=U64(w.rec_word(4, i) | w.rec_word(5, i) << 32) & w.M,
                    v=(U64(w.rec_word(6, i) | w.rec_word(7, i) << 32) + w.field(poff, vend, LANE, wv, w.es == 8)) & w.M,
                    r=U64(w.rec_word(3, i)) + w.field(vend, lend, LANE, wl, False))

    gr, cur = g0, load(g0)
    while True:
        more = cur["next"] < w.e1
        if more:
            if not w.rec_has(gr):
                w.rec_load(32, 32, gr, ng)
            nxt = load(gr + 1)
        act = LANE < cur["cnt"]
        vj = np.where(act, cur["v"], U64(0))
        r = np.where(act, cur["r"], U64(0))
        incl, total = w.lengths(r, cur["cnt"] - 1)
        assert cur["goff"] + total == cur["next"]
        start = U64(cur["goff"]) + incl - r
        f = (vj * r) & w.M
        first = (cur["base"] + (w.scan(f) - f) + vj) & w.M
        w.expand(False, cur["goff"], cur["next"], act, start, (first - vj * start) & w.M, vj)
        if not more:
            return
        gr, cur = gr + 1, nxt


def run_tree(w, n, g0, S):
    """unit_tree: the output of a DSTREE chunk from its starts S."""
    s = w.s
    R, ng = struct.unpack_from("<II", s, 0)
    d = U64(struct.unpack_from("<Q", s, 16)[0]) & w.M
    b_off = struct.unpack_from("<I", s, 24)[0]
    w.rec_load(b_off, 16, g0, ng)

    def load(gr):
        i = gr - w.g0
        poff, wc, cmin = (w.rec_word(k, i) for k in (1, 2, 3))
        cnt = min(64, R - 64 * gr)
        end = poff + 4 * ((cnt * wc + 31) // 32)
        assert end <= len(s)
        return dict(goff=w.rec_word(0, i), next=w.rec_word(0, i + 1) if gr + 1 < ng else n, cnt=cnt,
                    st=np.array([S[64 * gr + k] if k < cnt else 0 for k in range(64)], U64),
                    r=U64(cmin) + w.field(poff, end, LANE, wc, False))

    carry = w.es == 8 and n // 5 >= R
    gr, cur = g0, load(g0)
    while True:
        more = cur["next"] < w.e1
        if more:
            if not w.rec_has(gr):
                w.rec_load(b_off, 16, gr, ng)
            nxt = load(gr + 1)
        act = LANE < cur["cnt"]
        r = np.where(act, cur["r"], U64(0))
        incl, total = w.lengths(r, cur["cnt"] - 1)
        assert cur["goff"] + total == cur["next"]
        start = U64(cur["goff"]) + incl - r
        w.expand(carry, cur["goff"], cur["next"], act, start, (cur["st"] - d * start) & w.M, d)
        if not more:
            return carry
        gr, cur = gr + 1, nxt


def blocks(n, seed, run, dtype):
    """Blocks of consecutive values, mean length `run`, jumps between them."""
    r = g.rng(seed)
    lens = r.integers(1, 2 * run, size=2 * n // run + 4)
    starts = np.cumsum(lens + r.integers(1, 50, size=len(lens)))
    return np.concatenate([np.arange(k) + s for k, s in zip(lens, starts)])[:n].astype(dtype)


def runs(lens, seed, dtype):
    r = g.rng(seed)
    return np.repeat(r.integers(-2**31, 2**31, size=len(lens)), lens).astype(dtype)


MIXED = np.concatenate([np.full(4, 2048), np.full(130, 1), np.full(3, 2047), np.full(3, 2049), np.full(70, 3)])
SHORT = np.concatenate([np.full(65 * 70, 1), np.full(90, 2), np.full(5, 300)])
CASES = {
    "rle32 short": (zf.RLE_DELTA_BP, lambda: g.sorted_runs_column(6000, 3, 5)),
    "rle32 long": (zf.RLE_DELTA_BP, lambda: runs(g.rng(1).integers(1, 90, size=200), 2, np.int32)),
    "rle32 mixed": (zf.RLE_DELTA_BP, lambda: runs(MIXED, 3, np.int32)),
    "rle32 many groups": (zf.RLE_DELTA_BP, lambda: runs(SHORT, 4, np.int32)),
    "rle64 at the rule": (zf.RLE_DELTA_BP, lambda: runs(np.full(900, 5), 5, np.int64)),
    "rle64 long": (zf.RLE_DELTA_BP, lambda: g.sorted_runs_column(9000, 40, 5).astype(np.int64) * 3_000_000_001),
    "delta32": (zf.DELTA_BP, lambda: np.cumsum(g.rng(6).integers(-5, 9, size=9000)).astype(np.int32)),
    "delta64": (zf.DELTA_BP, lambda: np.cumsum(g.rng(7).integers(-5, 1 << 40, size=2500))),
    "stride32": (zf.DSTRIDE_BP, lambda: g.key_column(6000, 8, dtype=np.int32)),
    "stride64": (zf.DSTRIDE_BP, lambda: blocks(6000, 9, 30, np.int64)),
    "stride64 short": (zf.DSTRIDE_BP, lambda: g.rng(4).integers(-2**63, 2**63 - 1, size=900, dtype=np.int64)),
    "stride64 wrap": (zf.DSTRIDE_BP, lambda: (np.arange(3000, dtype=np.int64) * 977 + np.iinfo(np.int64).max - 3000)
                      .astype(np.uint64).astype(np.int64)),
    "tree32": (zf.DSTREE, lambda: g.orderkey_column(7000, 3)),
    "tree64": (zf.DSTREE, lambda: g.orderkey_column(7000, 4, dtype=np.int64)),
    "tree64 short": (zf.DSTREE, lambda: blocks(2000, 5, 2, np.int64)),
}


@pytest.mark.parametrize("name", CASES)
def test_span_model(name):
    codec, make = CASES[name]
    x = make()
    es, n = x.dtype.itemsize, len(x)
    cuts = [n // 3 + 7, n // 3 - 5, n - 2 * (n // 3) - 2]
    col = zf.Column.compress(x, codec, chunk_elems=cuts, pinned=False)
    blob = bytes(col.bytes())
    assert np.array_equal(zo.decode(col.bytes()), x)
    M = (1 << (8 * es)) - 1
    for ci, c in enumerate(zo.chunks(col.bytes())):
        s = blob[c["comp_off"]:c["comp_off"] + c["comp_len"]]
        m, at = c["n_elems"], c["plain_off"] // es
        want = [int(t) & M for t in x[at:at + m]]
        for unit, bases in ((64, (es,)), (500, (0, 128 - es)), (2048, (16 + es, 64)), (4096, (0, es))):
            tiles = {k: {"unit": unit} for k in ("RLE32", "RLE64", "TREE")}
            units = zf.chunk_units(col, ci, tiles=tiles)
            S = None
            if codec == zf.DSTREE:
                R = struct.unpack_from("<I", s, 0)[0]
                S = [None] * R
                for _, g0, e0, e1 in [u for u in units if u[0] != "TREE"]:
                    run_tree_starts(Wave(s, es, e0, e1, 256, S), R, g0)
                assert None not in S
                units = [u for u in units if u[0] == "TREE"]
            for base in bases:
                out = [None] * m
                for _, g0, e0, e1 in units:
                    w = Wave(s, es, e0, e1, 4096 + base, out)
                    if codec == zf.DSTREE:
                        run_tree(w, m, g0, S)
                    else:
                        run_rle(w, codec, m, g0)
                assert out == want, (name, ci, unit, base)


def test_long_runs_take_the_wide_scan():
    w = Wave(b"", 4, 0, 1, 0, [])
    r = np.zeros(64, U64)
    r[:40] = 1 << 27                       # their sum needs more than 32 bits
    assert w.lengths(r, 39)[1] == 40 << 27
    r[:40] = (1 << 26) - 1                 # the longest that a 32-bit scan adds up
    r[40:] = (1 << 26) - 1
    assert w.lengths(r, 63)[1] == 64 * ((1 << 26) - 1) < 2**32


def test_the_model_sees_a_wrong_carry():
    # an open window dropped between groups is noticed
    x = runs(np.full(200, 40), 5, np.int32)
    col = zf.Column.compress(x, zf.RLE_DELTA_BP, chunk_elems=[len(x)], pinned=False)
    c = zo.chunks(col.bytes())[0]
    s = bytes(col.bytes())[c["comp_off"]:c["comp_off"] + c["comp_len"]]
    out = [None] * len(x)
    w = Wave(s, 4, 0, len(x), 4096 + 4, out)
    expand = w.expand

    def dropping(*a):
        w.open = np.zeros((w.R, 64), U64)
        expand(*a)
    w.expand = dropping
    run_rle(w, zf.RLE_DELTA_BP, len(x), 0)
    assert out != [int(t) & 0xFFFFFFFF for t in x]

"""Corrupt LZ77 streams whose fault the host cannot see, through the kernel
that decodes a chunk in a workgroup's LDS (no tile set) and the one-wave kernel:
the oracle refuses every one, and so does the device."""
import struct

import numpy as np
import pytest

import oracle.zfo as zo
from paper_2602_08190_amd import zf

import helpers as H
from conftest import gpu_available
from test_gpu_parity import _expect_corrupt, check, decode_image, log

N_SEQ = 1300   # three groups of 512 sequences, the last one part full
BAD_AT = [0, 63, 64, 200, 511, 512, 600, 1023, 1024, 1299]


def sequences():
    """Literals first, then short matches; every seventh sequence takes one
    extension word and every eleventh two."""
    seqs = [(300, 0, 0)]
    for i in range(1, N_SEQ):
        ll, ml = i % 4, 4 + i % 9
        if i % 7 == 0:
            ll = 7 + i % 5
        if i % 11 == 0:
            ll, ml = 8, 34 + i % 3
        seqs.append((ll, ml, 1 + (i * 37) % 290))
    return seqs


def stream(seqs, plain=None, lit_more=0, ext_more=0):
    """The stream of the sequences, its literal array and its extension words
    longer or shorter than they use; sizes as the header's."""
    lits = bytes(i * 31 % 251 for i in range(sum(s[0] for s in seqs)))
    total = sum(s[0] + s[1] for s in seqs)
    s = H.lz_stream(seqs, lits, total if plain is None else plain)
    nseq, nlit, next_, p = struct.unpack_from("<IIII", s)
    body = s[16:]
    offs, rest = body[:2 * nseq], body[2 * nseq:]
    ext, rest = rest[:2 * next_], rest[2 * next_:]
    tags, lit = rest[:nseq], rest[nseq:]
    lit = lit + bytes(lit_more) if lit_more > 0 else lit[:nlit + lit_more]
    ext = ext + bytes(2 * ext_more) if ext_more > 0 else ext[:2 * (next_ + ext_more)]
    return struct.pack("<IIII", nseq, nlit + lit_more, next_ + ext_more, p) + offs + ext + tags + lit, p


def faults():
    good = sequences()
    total = sum(a + b for a, b, _ in good)
    out = []
    for at in BAD_AT:
        ll, ml, off = good[at]
        pos = sum(a + b for a, b, _ in good[:at])

        def with_(seq):
            return good[:at] + [seq] + good[at + 1:]
        out.append((f"{at}: an offset past the bytes before it",
                    stream(with_((ll, max(ml, 4), pos + ll + 1)), plain=total + max(ml, 4) - ml)))
        out.append((f"{at}: an offset of zero", stream(with_((ll, max(ml, 4), 0)), plain=total + max(ml, 4) - ml)))
        out.append((f"{at}: an offset without a match", stream(with_((ll, 0, 5)), plain=total - ml)))
        out.append((f"{at}: a match past the end", stream(with_((ll, 60000, 1)), plain=total)))
        out.append((f"{at}: literals past the end", stream(with_((60000, ml, max(off, 1 if ml else 0))), plain=total,
                                                           lit_more=ll - 60000)))
    out.append(("a byte too few", stream(good, plain=total + 1)))
    out.append(("a byte too many", stream(good, plain=total - 1)))
    for d in (-900, -300, -2, -1, 1, 500):
        out.append((f"{d} literals", stream(good, lit_more=d)))
    for d in (-100, -2, -1, 1, 2, 300):
        out.append((f"{d} extension words", stream(good, ext_more=d)))
    out.append(("no sequences", stream([], plain=5)))
    return out


def test_the_oracle_refuses_them():
    blob = H.container(zf.BYTES, [(*stream(sequences()), zf.LZ77)])
    x = zo.decode(blob)
    assert len(x) == sum(a + b for a, b, _ in sequences())
    for name, (s, plain) in faults():
        with pytest.raises(zo.OracleError):
            zo.decode(H.container(zf.BYTES, [(s, plain, zf.LZ77)]))
        zf.Column.from_bytes(H.container(zf.BYTES, [(s, plain, zf.LZ77)]), pinned=False)   # the host takes it


@pytest.mark.gpu
@pytest.mark.skipif(not gpu_available(), reason="needs a GPU")
@pytest.mark.parametrize("tiles", [{}, {"LZ77": dict(unit=8)}], ids=["workgroup", "wave"])
def test_the_device_refuses_them(tiles):
    good, plain = stream(sequences())
    col = zf.Column.from_bytes(H.container(zf.BYTES, [(good, plain, zf.LZ77)] * 3))
    check([col], decode_image([col], tiles=tiles))
    for name, (s, n) in faults():
        log("lz corrupt:", name, tiles)
        _expect_corrupt([zf.Column.from_bytes(H.container(zf.BYTES, [(s, n, zf.LZ77)]))], tiles=tiles)
        blob = H.container(zf.BYTES, [(good, plain, zf.LZ77)] * 2 + [(s, n, zf.LZ77), (good, plain, zf.LZ77)])
        _expect_corrupt([zf.Column.from_bytes(blob)], tiles=tiles)

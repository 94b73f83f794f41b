"""Kernel variants chosen by size, each at the edges of its range, against the
oracle's decode of the same bytes."""
import numpy as np
import pytest

from paper_2602_08190_amd import datagen as g
from paper_2602_08190_amd import zf

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

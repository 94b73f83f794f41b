"""Which kernels a decode launches: the tile shapes a caller sets reach their
kernels, and the kernels chosen by size are left where the rule says so."""
import numpy as np
import pytest

from paper_2602_08190_amd import datagen as g
from paper_2602_08190_amd import zf

from conftest import gpu_available
from test_gpu_dispatch import ans_mix
from test_gpu_parity import check, log, torch

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def kernel_names(p):
    """Names of the library's kernels that a profile holds, and all its keys."""
    keys = [e.key for e in p.key_averages()]
    names = {k.split("(")[0].split("<")[0].split("::")[-1] for k in keys if "zf::" in k}
    if not any(n.startswith("k_decode") for n in names):
        pytest.skip("the profiler recorded no kernels here")
    return names, keys


def launched(cols, xs, staged=False, **kw):
    """Names of the kernels of one decode, which is checked, and whether it
    issued copies from the host."""
    T = torch()
    plan = zf.Plan(cols, device=0, **kw)
    outs = zf.empty_outputs(cols)
    img = None if staged else zf.upload_image(plan, cols)
    T.cuda.synchronize()
    act = T.profiler.ProfilerActivity
    with T.profiler.profile(activities=[act.CUDA]) as p:
        if staged:
            plan.transfer_and_decompress(outs)
        else:
            plan.decompress_async(img, img.numel(), outs)
        plan.sync()
        T.cuda.synchronize()
    check(cols, [o.cpu().numpy() for o in outs], xs)
    names, keys = kernel_names(p)
    return names, any("HtoD" in k for k in keys)


@pytest.mark.parametrize("waves", [None, 1, 7, 16])
def test_ans_workgroups_the_caller_sets(waves):
    # chunks whose rings go round many times, in workgroups of one to 16 waves
    # (16: more than 64 KiB of LDS; 16 and 7: the last workgroup part empty)
    for size, n in ((5000, 33), (40000, 17)):
        col, x = ans_mix(n, size)
        log("ans", n, "chunks of", size, "waves", waves)
        tiles = {"ANS": dict(waves_per_block=waves)} if waves else {}
        names, _ = launched([col], [x], tiles=tiles)
        assert names == {"k_decode_ans" if waves else "k_decode_ans_fused"}


def test_ans_unit_alone_keeps_the_fused_model():
    col, x = ans_mix(9, 3000)
    names, _ = launched([col], [x], tiles={"ANS": dict(unit=1)})
    assert names == {"k_decode_ans_fused"}


@pytest.mark.parametrize("symbols", [1, 2, 3, 5, 63, 64, 65, 255, 256])
def test_ans_models_in_workgroups(symbols):
    # the slot table of the model that several waves a compute unit keep: bytes
    # whose slots begin at every place in a lane's four, equal and steep counts,
    # bytes with one slot, alphabets that begin and end anywhere
    r = g.rng(symbols)
    parts = []
    for k in range(6):
        alphabet = np.sort(r.permutation(256)[:symbols]).astype(np.uint8)
        p = np.ones(symbols) if k == 0 else r.random(symbols) ** (2 * k) + 1e-4
        parts.append(r.choice(alphabet, size=1500 + 701 * k, p=p / p.sum()))
    x = np.concatenate(parts)
    col = zf.Column.compress(x, zf.ANS, chunk_elems=[len(p) for p in parts])
    names, _ = launched([col], [x], tiles={"ANS": dict(waves_per_block=4)})
    assert names == {"k_decode_ans"}


@pytest.mark.parametrize("persistent", [False, True])
def test_staged_copies_beside_the_persistent_kernel(persistent):
    # a copy kernel that wants a compute unit's LDS would wait for the persistent
    # kernel to end: that plan's copies are commands, of dictionaries too
    xs = [g.text_column(90_001, 3), g.fixed16_column(7_003, 300, 2), g.text_column(60_001, 5),
          g.uniform_i32(20_000, 5, 1 << 14, 1)]
    codecs = [zf.LZ77, zf.DICT_BP, zf.SDICT_COL_ANS, zf.FOR_BP]
    cols = [zf.Column.compress(x, c, chunk_bytes=(1 << 12, 1 << 14), seed=i, pinned=True)
            for i, (x, c) in enumerate(zip(xs, codecs))]
    for slot in (1 << 14, 1 << 22):
        names, commands = launched(cols, xs, staged=True, slot_bytes=slot, persistent=persistent)
        assert ("k_copy" in names) == (not persistent)
        assert commands == persistent


def big_text(mib, codec, seed):
    """mib MiB of one MiB of text over and over, in chunks of a MiB."""
    x = np.tile(g.text_column(1 << 20, seed), mib)
    return x, zf.Column.compress(x, codec, chunk_elems=[1 << 20] * mib, pinned=False)


@pytest.mark.parametrize("parts,hot", [
    ([(511, zf.SDICT_COL)], False), ([(512, zf.SDICT_COL)], True),
    ([(600, zf.SDICT_COL_ANS)], False), ([(832, zf.SDICT_COL_ANS)], True),
    ([(300, zf.SDICT_COL), (500, zf.SDICT_COL_ANS)], True),
    ([(1024, zf.SDICT_BP), (20, zf.SDICT_COL)], False)])
def test_sdict_workgroups_by_bytes_over_column_dictionaries(parts, hot):
    # the 16-wave workgroups that share a copy of a column dictionary's hottest
    # records, on both sides of their lines; own dictionaries do not count
    T = torch()
    log("sdict", parts)
    xs, cols = zip(*[big_text(m, c, i) for i, (m, c) in enumerate(parts)])
    plan = zf.Plan(list(cols), device=0)
    img = zf.upload_image(plan, list(cols))
    outs = zf.empty_outputs(list(cols))
    act = T.profiler.ProfilerActivity
    with T.profiler.profile(activities=[act.CUDA]) as p:
        plan.decompress_async(img, img.numel(), outs)
        plan.sync()
        T.cuda.synchronize()
    for x, o in zip(xs, outs):
        assert bool((o.view(-1, 1 << 20) == T.from_numpy(x[:1 << 20]).cuda()).all())
    names, _ = kernel_names(p)
    assert ("k_decode_sdict_hot" in names) == hot
    assert ("k_decode_sdict" in names) != hot


@pytest.mark.parametrize("size,n,chunked", [(1000, 3, False), (4608, 5, False), (4609, 5, True), (7000, 767, True),
                                            (7000, 1024, False), (65536, 5, True), (65536, 2304, True),
                                            (65536, 2400, False)])
def test_lz_chunk_kernel_by_bytes_and_count(size, n, chunked):
    # short chunks and many stay with the one-wave kernel, which is faster there
    x = np.tile(g.text_column(min(size * n, 1 << 20), size), -(-size * n // (1 << 20)))[:size * n]
    x = np.resize(x, size * n)
    log("lz", n, "chunks of", size)
    col = zf.Column.compress(x, zf.LZ77, chunk_elems=[size] * n)
    T = torch()
    plan = zf.Plan([col], device=0)
    img = zf.upload_image(plan, [col])
    outs = zf.empty_outputs([col])
    act = T.profiler.ProfilerActivity
    with T.profiler.profile(activities=[act.CUDA]) as p:
        plan.decompress_async(img, img.numel(), outs)
        plan.sync()
        T.cuda.synchronize()
    assert bool((outs[0] == T.from_numpy(x).cuda()).all())
    names, _ = kernel_names(p)
    assert names == {"k_decode_lz_chunk" if chunked else "k_decode_lz"}


@pytest.mark.parametrize("per_cu,more,size,kernel", [
    (18, 0, 70, "k_decode_ans"), (18, 1, 5000, "k_decode_ans_small"), (25, 0, 130, "k_decode_ans_small"),
    (25, 1, 90, "k_decode_ans"), (54, 1, 65, "k_decode_ans_small")])
def test_ans_layouts_by_rounds(per_cu, more, size, kernel):
    # the layout that lets 25 chunks run per compute unit instead of 18, where
    # that saves a round; its ring goes round many times in chunks of 5,000
    n = per_cu * torch().cuda.get_device_properties(0).multi_processor_count + more
    col, x = ans_mix(n, size, exact=True)
    log("ans", n, "chunks of", size)
    names, _ = launched([col], [x])
    assert names == {kernel}


@pytest.mark.parametrize("symbols", [1, 2, 3, 5, 63, 64, 65, 255, 256])
def test_ans_models_of_the_small_layout(symbols):
    r = g.rng(1000 + symbols)
    n = 19 * torch().cuda.get_device_properties(0).multi_processor_count
    parts = []
    for k in range(n):
        alphabet = np.sort(r.permutation(256)[:symbols]).astype(np.uint8)
        p = r.random(symbols) ** (1 + k % 7) + 1e-4
        parts.append(r.choice(alphabet, size=400, p=p / p.sum()))
    x = np.concatenate(parts)
    col = zf.Column.compress(x, zf.ANS, chunk_elems=[400] * n)
    names, _ = launched([col], [x])
    assert names == {"k_decode_ans_small"}

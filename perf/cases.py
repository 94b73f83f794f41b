"""Performance cases: columns and tables decoded through zf's public calls.

A case names a column family (or a whole table, or the cost model), its size
and its options.  ``prepare`` draws the values on the GPU from the seed,
compresses them on the host and builds what a program holds before it decodes:
the plan, the compressed image in device memory (or pinned columns) and the
output buffers.  ``run`` is one call.
"""
import math

import numpy as np
import torch

from paper_2602_08190_amd import zf

DEV = "cuda"
MIB = 1 << 20
# plain bytes of a column's chunks (log-uniform between the two); None: the
# codec's default, 1 MiB (LZ77: 64 KiB)
CHUNKS = {"default": None, "16K": (16 << 10, 16 << 10), "64K": (64 << 10, 64 << 10),
          "256K": (256 << 10, 256 << 10), "16K-64K": (16 << 10, 64 << 10), "16K-256K": (16 << 10, 256 << 10),
          "uneven": (16 << 10, 4 << 20)}


# ------------------------------------------------------------------ cases
def listed():
    return [
        # a lookup that touches one small chunk: nothing but launches and latency
        {"name": "for_i32_small", "family": "for", "bits": 32, "n": 10_007, "width": 12, "chunk": "default"},
        # money columns: int64 cents
        {"name": "for_i64", "family": "for", "bits": 64, "n": 12_500_003, "width": 24, "chunk": "uneven"},
        # prices stored as doubles with two decimal places
        {"name": "f2i_f64", "family": "f2i", "n": 16_777_259, "places": 2, "specials": 0, "chunk": "default"},
        # date-like columns, runs of 8 on average, 64 KiB chunks
        {"name": "rle_i32", "family": "rle", "bits": 32, "n": 33_554_467, "run": 8, "chunk": "64K"},
        # sparse order keys through the two-stage DeltaStride tree
        {"name": "dstree_i32", "family": "dstree", "bits": 32, "n": 33_554_393, "chunk": "default"},
        # comment text as LZ77, 64 KiB chunks (the codec's largest)
        {"name": "lz77_text", "family": "lz", "n": 128 * MIB + 77, "chunk": "default"},
        # a skewed flag column through ANS, 64 KiB chunks
        {"name": "ans_flags", "family": "ans", "n": 128 * MIB + 13, "skew": 0.5, "chunk": "64K"},
        # a comment column: String-dictionary over one dictionary | bit-packing | ANS
        {"name": "sdict_col_ans_text", "family": "sdict", "codec": "SDICT_COL_ANS", "n": 256 * MIB + 31,
         "chunk": "default"},
        # one row group of a 16-column table: many kinds, little work for each
        {"name": "table_row_group", "family": "table", "rows": 20_011, "mode": "image", "slot": 0},
        # a table scan from device memory
        {"name": "table_scan", "family": "table", "rows": 1_500_007, "mode": "image", "slot": 0},
        # a table read from pinned host memory: copies overlapped with decodes
        {"name": "table_staged", "family": "table", "rows": 500_009, "mode": "staged", "slot": 8 * MIB},
        # one minibatch of the cost model's training: scores, loss and gradient
        {"name": "cost_model_step", "family": "mlp", "n": 2048},
    ]


def draw(rng):
    """One more case, sizes log-uniform from a few thousand values up."""
    def size(lo, hi):
        return int(math.exp(rng.uniform(math.log(lo), math.log(hi)))) | rng.randrange(2)

    chunk = rng.choice(["default", "uneven", "64K", "256K"])
    family = rng.choice(["for", "for", "dict", "f2i", "rle", "delta", "dstride", "dstree", "lz", "ans", "sdict",
                         "sdict", "table", "table", "mlp"])
    bits = rng.choice([32, 64])
    if family == "for":
        return {"family": family, "bits": bits, "n": size(3000, 30_000_000), "width": rng.randrange(1, bits - 1),
                "chunk": chunk}
    if family == "dict":
        kind = rng.choice(["i32", "i64", "char16"])
        return {"family": family, "kind": kind, "n": size(3000, 15_000_000),
                "distinct": size(2, 20_000 if kind != "char16" else 2000), "chunk": chunk}
    if family == "f2i":
        return {"family": family, "n": size(3000, 16_000_000), "places": rng.randrange(0, 5),
                "specials": rng.choice([0, 0, 1000]), "chunk": chunk}
    if family == "rle":
        return {"family": family, "bits": bits, "n": size(3000, 30_000_000), "run": size(2, 600), "chunk": chunk}
    if family == "delta":
        return {"family": family, "bits": bits, "n": size(3000, 30_000_000), "chunk": chunk}
    if family in ("dstride", "dstree"):
        return {"family": family, "bits": bits, "n": size(3000, 30_000_000), "chunk": chunk}
    if family == "lz":
        return {"family": family, "n": size(20_000, 128 * MIB), "chunk": rng.choice(["default", "16K-64K"])}
    if family == "ans":
        return {"family": family, "n": size(20_000, 128 * MIB), "skew": rng.choice([0.34, 0.5, 0.8, 0.96, 0.0]),
                "chunk": rng.choice(["64K", "16K", "16K-256K"])}
    if family == "sdict":
        return {"family": family, "codec": rng.choice(["SDICT_BP", "SDICT_ANS", "SDICT_COL", "SDICT_COL_ANS"]),
                "n": size(20_000, 250 * MIB), "chunk": chunk}
    if family == "table":
        return {"family": family, "rows": size(2000, 1_200_000), "mode": rng.choice(["image", "staged"]),
                "slot": rng.choice([0, 4 * MIB])}
    return {"family": "mlp", "n": size(8, 16_000)}


# ----------------------------------------------------------------- values
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _ints(n, lo, hi, g, dtype=torch.int64):
    return torch.randint(lo, hi, (n,), generator=g, device=DEV, dtype=torch.int64).to(dtype)


def _int_type(bits):
    return torch.int32 if bits == 32 else torch.int64


def _run_lengths(n, mean, g):
    """Geometric run lengths that cover at least n values."""
    k = int(n / mean * 1.1) + 64
    r = torch.empty(k, device=DEV).geometric_(min(1.0, 1.0 / mean), generator=g).to(torch.int64)
    r[-1] += n
    return r


def _dates(n, mean, g, dtype):
    r = _run_lengths(n, mean, g)
    v = torch.arange(r.numel(), device=DEV) % 2557
    return torch.repeat_interleave(v, r)[:n].to(dtype)


def _order_keys(n, g, dtype):
    """The first 8 keys of every 32, 1% of them deleted."""
    m = int(n * 1.02) + 4096
    i = torch.arange(m, device=DEV)
    keys = 1 + 32 * (i // 8) + i % 8
    return keys[torch.rand(m, generator=g, device=DEV) >= 0.01][:n].to(dtype)


def _block_keys(n, g, dtype):
    """Blocks of consecutive keys, mean length 8, jumps of 1 to 64 between them."""
    r = _run_lengths(n, 8, g)
    ends = torch.cumsum(r, 0)
    starts = ends - r + torch.cumsum(_ints(r.numel(), 1, 65, g), 0)
    i = torch.arange(n, device=DEV)
    b = torch.searchsorted(ends, i, right=True)
    return (starts[b] + i - (ends - r)[b]).to(dtype)


def _words(k, lo, hi, width, g):
    """k random words of lo..hi letters, zero padded to width; their lengths."""
    length = _ints(k, lo, hi + 1, g)
    letters = _ints(k * width, 97, 123, g, torch.uint8).reshape(k, width)
    return letters * (torch.arange(width, device=DEV) < length[:, None]).to(torch.uint8), length


def _text(n, g):
    """n bytes of Zipf(1.1) words from a vocabulary of 10,000, a space after
    each, a line end after one in ten."""
    k = 10_000
    words, length = _words(k, 3, 10, 12, g)
    p = np.arange(1, k + 1, dtype=np.float64) ** -1.1
    cdf = torch.from_numpy(np.cumsum(p / p.sum())).to(DEV)
    m = n // 4 + 64  # words have at least three letters
    w = torch.searchsorted(cdf, torch.rand(m, generator=g, device=DEV, dtype=torch.float64)).clamp_(max=k - 1)
    size = length[w] + 1
    end = torch.cumsum(size, 0)
    m = int(torch.searchsorted(end, torch.tensor(n, device=DEV))) + 1
    w, size, end = w[:m], size[:m], end[:m]
    sep = torch.where(torch.rand(m, generator=g, device=DEV) < 0.1, 10, 32).to(torch.uint8)
    out = torch.empty(n, dtype=torch.uint8, device=DEV)
    step = 1 << 25
    for a in range(0, n, step):
        i = torch.arange(a, min(n, a + step), device=DEV)
        t = torch.searchsorted(end, i, right=True)
        c = i - (end - size)[t]
        out[a:a + step] = torch.where(c == length[w[t]], sep[t], words[w[t], c.clamp(max=11)])
    return out


def _flags(n, skew, g):
    """'A', 'N', 'R': 'N' with probability skew, the others sharing the rest."""
    u = torch.rand(n, generator=g, device=DEV)
    a = (1.0 - skew) / 2
    return torch.where(u < a, 65, torch.where(u < a + skew, 78, 82)).to(torch.uint8)


def _decimals(n, places, specials, g):
    x = _ints(n, 90_000, 10_500_000, g).to(torch.float64) / float(10 ** places)
    if specials:
        # values without a short decimal form, stored raw
        pool = torch.tensor([-0.0, 1.0 / 3.0, math.pi, math.e, 1e15 / 7.0], dtype=torch.float64, device=DEV)
        k = min(specials, n)
        x[torch.arange(k, device=DEV) * (n // k)] = pool[_ints(k, 0, 5, g)]
    return x


def _char16(n, k, g):
    return _words(k, 5, 15, 16, g)[0][_ints(n, 0, k, g)]


def _column(case, seed):
    """(values on the GPU, codec) of a single-column case."""
    g, f, n = _gen(seed), case["family"], case["n"]
    if f == "for":
        lo = 10 ** 6 if case["width"] < 30 else -(1 << (case["width"] - 1))
        return _ints(n, lo, lo + (1 << case["width"]), g, _int_type(case["bits"])), zf.FOR_BP
    if f == "dict":
        k = case["distinct"]
        if case["kind"] == "char16":
            return _char16(n, k, g), zf.DICT_BP
        t = torch.int32 if case["kind"] == "i32" else torch.int64
        return _ints(k, -(1 << 30), 1 << 30, g, t)[_ints(n, 0, k, g)], zf.DICT_BP
    if f == "f2i":
        return _decimals(n, case["places"], case["specials"], g), zf.F2I_BP
    if f == "rle":
        return _dates(n, case["run"], g, _int_type(case["bits"])), zf.RLE_DELTA_BP
    if f == "delta":
        return torch.cumsum(_ints(n, 0, 64, g), 0).to(_int_type(case["bits"])), zf.DELTA_BP
    if f == "dstride":
        return _block_keys(n, g, _int_type(case["bits"])), zf.DSTRIDE_BP
    if f == "dstree":
        return _order_keys(n, g, _int_type(case["bits"])), zf.DSTREE
    if f == "lz":
        return _text(n, g), zf.LZ77
    if f == "ans":
        return (_flags(n, case["skew"], g) if case["skew"] else _text(n, g)), zf.ANS
    return _text(n, g), getattr(zf, case["codec"])


def _table(case, seed):
    """[(values, codec)] of a 16-column table: six int32 keys, three int64
    cents, three dates, three CHAR(16) flags and a comment."""
    g, n = _gen(seed), case["rows"]
    cols = [(_ints(n, 10 ** 6, 10 ** 6 + (1 << w), g, torch.int32), zf.FOR_BP) for w in (12, 16, 20, 24, 25)]
    cols.append((_ints(n, -(1 << 30), 1 << 30, g, torch.int32), zf.FOR_BP))
    cols += [(_ints(n, 100, 10 ** 7, g), zf.FOR_BP) for _ in range(3)]
    cols += [(_dates(n, run, g, torch.int32), zf.RLE_DELTA_BP) for run in (8, 64, 512)]
    cols += [(_char16(n, 25, g), zf.DICT_BP) for _ in range(3)]
    cols.append((_text(75 * n, g), zf.SDICT_COL_ANS))
    return cols


def _mlp_inputs(case, seed):
    """Parameters (the usual scaled normal initialisation), standardised
    statistics, measured outputs and their log times."""
    g, n = _gen(seed), case["n"]

    def normal(*shape):
        return torch.randn(*shape, generator=g, device=DEV)
    params = torch.cat([(normal(64, 32) * (2 / 32) ** 0.5).flatten(), 0.1 * normal(64),
                        (normal(64, 64) * (2 / 64) ** 0.5).flatten(), 0.1 * normal(64),
                        (normal(24, 64) * (1 / 64) ** 0.5).flatten(), 0.1 * normal(24)])
    return params, normal(n, 32), _ints(n, 0, 24, g, torch.int32), normal(n)


# ---------------------------------------------------------------- passes
def prepare(case, seed):
    if case["family"] == "mlp":
        params, x, k, t = _mlp_inputs(case, seed)
        n = case["n"]
        return {"mode": "mlp", "params": params, "x": x, "k": k, "t": t,
                "y": torch.empty(n, zf.MLP_OUT, device=DEV), "grad": torch.empty(zf.MLP_PARAMS, device=DEV),
                "loss": torch.empty(1, device=DEV),
                "work": torch.empty(zf.mlp_grad_work_bytes(n) // 4, device=DEV)}
    table = case["family"] == "table"
    staged = table and case["mode"] == "staged"
    values = _table(case, seed) if table else [_column(case, seed)]
    chunk = CHUNKS["uneven" if table else case["chunk"]]
    cols = [zf.Column.compress(v.cpu().numpy(), codec, chunk_bytes=chunk, seed=i, pinned=staged)
            for i, (v, codec) in enumerate(values)]
    del values
    plan = zf.Plan(cols, **({"slot_bytes": case["slot"]} if table and case["slot"] else {}))
    state = {"mode": "staged" if staged else "image", "cols": cols, "plan": plan, "outs": zf.empty_outputs(cols)}
    if not staged:
        state["image"] = zf.upload_image(plan, cols)
    return state


def run(state):
    if state["mode"] == "mlp":
        zf.mlp_forward(state["params"], state["x"], state["y"])
        zf.mlp_grad(state["params"], state["x"], state["k"], state["t"], state["grad"], state["loss"], state["work"])
        return {"y": state["y"], "grad": state["grad"], "loss": state["loss"]}
    if state["mode"] == "staged":
        state["plan"].transfer_and_decompress(state["outs"], timing=False)
    else:
        state["plan"].decompress_async(state["image"], state["image"].numel(), state["outs"])
    return state["outs"]


def work(case):
    """Compressed bytes read and plain bytes written (from the families'
    usual sizes), or the network's multiply-adds."""
    f = case["family"]
    if f == "mlp":
        macs = 32 * 64 + 64 * 64 + 64 * 24
        n = case["n"]
        # scores, then a forward pass and both products of the backward pass
        return {"bytes": 4 * (n * (32 + 24 + 2) + 2 * zf.MLP_PARAMS), "flops": 2 * n * (4 * macs - 32 * 64)}
    if f == "table":
        plain = case["rows"] * (6 * 4 + 3 * 8 + 3 * 4 + 3 * 16 + 75)
        comp = case["rows"] * ((12 + 16 + 20 + 24 + 25 + 31 + 3 * 24 + 3 * 5) / 8 + 0.7 + 14)
        return {"bytes": int(plain + comp), "flops": 0}
    n = case["n"]
    if f == "for":
        return {"bytes": n * (case["bits"] + case["width"]) // 8, "flops": 0}
    if f == "dict":
        es = {"i32": 4, "i64": 8, "char16": 16}[case["kind"]]
        return {"bytes": int(n * (es + math.ceil(math.log2(case["distinct"])) / 8)), "flops": 0}
    if f == "f2i":
        return {"bytes": 11 * n, "flops": n}
    if f == "rle":
        return {"bytes": int(n * (case["bits"] / 8 + 4.6 / case["run"])), "flops": 0}
    if f == "delta":
        return {"bytes": int(n * (case["bits"] / 8 + 1.3)), "flops": 0}
    if f == "dstride":
        return {"bytes": int(n * (case["bits"] / 8 + 0.8)), "flops": 0}
    if f == "dstree":
        return {"bytes": int(n * (case["bits"] / 8 + 0.14)), "flops": 0}
    ratio = {"lz": 2.0, "ans": 4.0, "SDICT_BP": 2.1, "SDICT_ANS": 2.3, "SDICT_COL": 4.0,
             "SDICT_COL_ANS": 5.4}[case["codec"] if f == "sdict" else f]
    return {"bytes": int(n * (1 + 1 / ratio)), "flops": 0}


def exact(case, seed):
    """The decoded values themselves; the network in 64 bits."""
    if case["family"] == "table":
        return [v for v, _ in _table(case, seed)]
    if case["family"] != "mlp":
        return [_column(case, seed)[0]]
    p, x, k, t = (v.double() if v.is_floating_point() else v for v in _mlp_inputs(case, seed))
    p.requires_grad_(True)
    w1, b1, w2, b2, w3, b3 = torch.split(p, [2048, 64, 4096, 64, 1536, 24])
    h = torch.relu(x @ w1.reshape(64, 32).t() + b1)
    h = torch.relu(h @ w2.reshape(64, 64).t() + b2)
    y = h @ w3.reshape(24, 64).t() + b3
    loss = ((y[torch.arange(x.shape[0], device=DEV), k.long()] - t) ** 2).mean()
    grad, = torch.autograd.grad(loss, p)
    return {"y": y.detach(), "grad": grad, "loss": loss.detach().reshape(1)}

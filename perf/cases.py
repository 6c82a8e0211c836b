"""The calls that this framework is measured on.

A case is one use of the public entry points (`Plan`, `Batch`, `decode_blob`,
`encode`) on a seeded synthetic stream. The kinds are

  decode    a plan's stream is resident on the device; a pass is Plan.decode
  adaptive  the same with per-symbol tables: Plan.decode_adaptive
  packed    the packed split metadata is resident; a pass unpacks the records on
            the device and decodes (a client that keeps the container's section)
  batch     many independent streams of mixed shapes: Batch.decode
  whole     container bytes on the host to symbols on the host: Blob.from_bytes and
            decode_blob (plan, allocation, upload, decode, copy back)
  encode    symbols on the host to container bytes on the host: encode, to_bytes

Sizes follow the benchmark's workloads (the 1 MiB Laplace stream of 256 splits, the
256 MiB Zipf stream of 65536, its combinations to few splits, the 16-table adaptive
stream, the mixed batch) and the serving corpus's smallest stream, 64 KiB. Symbols
are drawn by table from a 2^16-entry inverse CDF.
"""

import math
import os
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import torch

import paper_2306_12141_amd as rc
from paper_2306_12141_amd.batch import Batch

KIB, MIB = 1 << 10, 1 << 20


def listed():
    return [
        # The serving corpus's smallest stream at its stored 1 KiB per split: the call
        # whose launch and set-up cost as much as its decoding.
        _decode("decode_64k_w32", n=64 * KIB, lanes=32, bits=11, splits=64, dist="laplace", param=4.0),
        # The benchmark's small configuration: 1 MiB, 256 splits, fewer units than the
        # chip has SIMDs.
        _decode("decode_1m_w32", n=MIB, lanes=32, bits=11, splits=256, dist="laplace", param=4.0),
        # An ordinary 16-bit image plane of odd size, 4096 values, ragged last group.
        _decode("decode_1500007_u16_w64", n=1500007, lanes=64, bits=12, splits=367, dist="laplace", param=24.0,
                alphabet=4096),
        # A large stream combined to 256 splits for a client of little parallelism.
        _decode("decode_64m_w32_few", n=64 * MIB, lanes=32, bits=12, splits=256, dist="zipf", param=1.1),
        # The headline: 256 MiB at 65536 splits, W = 64.
        _decode("decode_256m_w64", n=256 * MIB, lanes=64, bits=12, splits=65536, dist="zipf", param=1.1),
        # The finest quantisation (two-level tables).
        _decode("decode_64m_w64_n16", n=64 * MIB, lanes=64, bits=16, splits=16384, dist="zipf", param=1.1),
        # Large 16-bit data at W = 32.
        _decode("decode_32m_u16_w32", n=32 * MIB, lanes=32, bits=12, splits=8192, dist="laplace", param=24.0,
                alphabet=4096),
        # Per-symbol tables, as for image latents under a hyperprior.
        dict(_decode("adaptive_32m_w32", n=32 * MIB, lanes=32, bits=9, splits=8192, dist="tables", param=16.0,
                     alphabet=64), kind="adaptive"),
        # A W = 32 stream at full parallelism whose client unpacks the stored metadata.
        dict(_decode("packed_64m_w32", n=64 * MIB, lanes=32, bits=12, splits=16384, dist="zipf", param=1.1),
             kind="packed"),
        # The mixed batch: 4 KiB .. 16 MiB streams, 8- and 16-bit, one launch per table class.
        dict(name="batch_60", kind="batch", count=60, lo=4 * KIB, hi=16 * MIB, split_bytes=8 * KIB),
        # One whole call on host data: a container arrives, its symbols are wanted.
        dict(_decode("whole_4m_w32", n=4 * MIB, lanes=32, bits=11, splits=1024, dist="laplace", param=4.0),
             kind="whole"),
        # The other direction on host data.
        dict(_decode("encode_1m_w32", n=MIB, lanes=32, bits=11, splits=256, dist="laplace", param=4.0),
             kind="encode"),
    ]


def draw(rng):
    kind = rng.choice(["decode"] * 6 + ["adaptive", "packed", "batch", "whole", "encode"])
    if kind == "batch":
        return dict(kind=kind, count=rng.randint(12, 60), lo=4 * KIB, hi=_log_int(rng, 256 * KIB, 16 * MIB),
                    split_bytes=rng.choice([2 * KIB, 8 * KIB, 16 * KIB]))
    top = {"decode": 128 * MIB, "packed": 64 * MIB, "adaptive": 32 * MIB, "whole": 4 * MIB, "encode": MIB}[kind]
    wide = kind in ("decode", "packed", "whole") and rng.random() < 0.3   # 16-bit symbols
    n = _log_int(rng, 64 * KIB, top // 2 if wide else top)
    per_split = _log_int(rng, 1024, 16 * KIB)
    splits = max(1, n // per_split)
    if kind == "decode" and rng.random() < 0.35:   # combined for a client of less parallelism
        splits = max(1, n // (256 * KIB), min(splits, _log_int(rng, 64, 4096)))
    case = _decode(None, n=n, lanes=rng.choice([32, 64]), bits=rng.choice([10, 11, 12, 12, 14, 16]), splits=splits,
                   dist=rng.choice(["laplace", "zipf", "uniform"]), param=0.0, alphabet=4096 if wide else 256)
    if case["dist"] == "laplace":
        case["param"] = round(rng.uniform(1.0, 32.0), 3)
    elif case["dist"] == "zipf":
        case["param"] = round(rng.uniform(0.8, 1.5), 3)
    if wide:
        case["bits"] = max(case["bits"], 12)
    if kind == "adaptive":
        case.update(bits=rng.choice([9, 10]), dist="tables", param=16.0, alphabet=64)
    if kind == "decode" and not wide and rng.random() < 0.15:
        case["partitioned"] = True       # the conventional sub-sequences
    case["kind"] = kind
    del case["name"]
    return case


def _decode(name, n, lanes, bits, splits, dist, param, alphabet=256):
    return dict(name=name, kind="decode", n=n, lanes=lanes, bits=bits, splits=splits, dist=dist, param=param,
                alphabet=alphabet, partitioned=False)


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# ------------------------------------------------------------------ inputs


def _laplace(alphabet, scale):
    k = np.arange(alphabet, dtype=np.float64)
    w = np.exp(-np.abs(k - alphabet / 2) / scale)
    return w / w.sum()


def _pmf(dist, param, alphabet, rng):
    if dist == "laplace":
        return _laplace(alphabet, param)
    if dist == "uniform":
        return np.full(alphabet, 1.0 / alphabet)
    p = np.arange(1, alphabet + 1, dtype=np.float64) ** (-param)
    return rng.permutation(p / p.sum())


def _edges(pmf):
    c = np.rint(np.cumsum(pmf) * 65536.0).astype(np.int64)
    c[-1] = 65536
    return np.diff(np.concatenate([[0], c]))


def _draws(rng, n):
    return rng.integers(0, 65536, n, dtype=np.uint16)


def _symbols(case, seed):
    rng = np.random.default_rng(seed)
    dtype = np.uint8 if case["alphabet"] <= 256 else np.uint16
    counts = _edges(_pmf(case["dist"], case["param"], case["alphabet"], rng))
    return np.repeat(np.arange(case["alphabet"], dtype=dtype), counts)[_draws(rng, case["n"])]


def _tables(case):
    """16 discrete Laplace tables with scales from 0.5 to 16, and their frequencies summing to 2^bits."""
    counts = [_edges(_laplace(case["alphabet"], 0.5 * 32.0 ** (t / 15.0))) for t in range(16)]
    freq = np.stack([rc.quantize(np.maximum(c, 1), case["bits"]) for c in counts])
    return counts, freq


def _adaptive_symbols(case, seed):
    """Symbols and their table index: constant over blocks of 256, with a jitter of one."""
    rng = np.random.default_rng(seed)
    n = case["n"]
    counts, _ = _tables(case)
    base = np.repeat(rng.integers(0, 16, -(-n // 256), dtype=np.int8), 256)[:n]
    index = np.clip(base + rng.integers(-1, 2, n, dtype=np.int8), 0, 15).astype(np.uint8)
    inverse = np.concatenate([np.repeat(np.arange(case["alphabet"], dtype=np.uint8), c) for c in counts])
    return inverse[(index.astype(np.uint32) << 16) | _draws(rng, n)], index


def _batch_streams(case, seed):
    """The case's stream shapes, each with its own symbols by the seed."""
    rng = np.random.default_rng(case["count"])
    out = []
    for i in range(case["count"]):
        size = int(math.exp(rng.uniform(math.log(case["lo"]), math.log(case["hi"]))))
        wide = rng.random() < 0.25
        dist = ("laplace", "zipf", "uniform")[rng.integers(0, 3)]
        param = rng.uniform(1.0, 32.0) if dist == "laplace" else rng.uniform(0.8, 1.5)
        bits = 12 if wide else int(rng.integers(10, 13))
        out.append(dict(n=max(64, size // (2 if wide else 1)), lanes=32, bits=bits, dist=dist, param=float(param),
                        alphabet=4096 if wide else 256, splits=max(1, size // case["split_bytes"]),
                        partitioned=False, seed=(seed << 8) + i))
    return out


def _encode(case, symbols):
    f = rc.encode_partitioned if case["partitioned"] else rc.encode
    kw = {"partitions": case["splits"]} if case["partitioned"] else {"splits": case["splits"]}
    return f(symbols, lanes=case["lanes"], quant_bits=case["bits"], alphabet=case["alphabet"], **kw)


def _map(f, items):
    with ThreadPoolExecutor(max_workers=min(8, len(os.sched_getaffinity(0)))) as ex:
        return list(ex.map(f, items))


# ------------------------------------------------------------------ the cases


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        streams = _batch_streams(case, seed)
        batch = Batch(_map(lambda s: _encode(s, _symbols(s, s["seed"])), streams))
        ws, out, err = batch.allocate()
        batch.upload(ws)
        views = [out[o:o + n] for o, n in (batch.output_range(i) for i in range(batch.count))]
        return dict(kind=kind, batch=batch, ws=ws, out=out, err=err, views=views)
    if kind == "adaptive":
        symbols, index = _adaptive_symbols(case, seed)
        blob = rc.encode_adaptive(symbols, _tables(case)[1], index, lanes=case["lanes"], quant_bits=case["bits"],
                                  splits=case["splits"], alphabet=case["alphabet"])
        return dict(_resident(kind, rc.Plan(blob)), index=torch.from_numpy(index).cuda())
    symbols = _symbols(case, seed)
    if kind == "encode":
        # The message buffer that the container is put into; its tail stays zero.
        return dict(kind=kind, case=case, symbols=symbols, message=np.zeros(2 * symbols.nbytes + MIB, dtype=np.uint8))
    blob = _encode(case, symbols)
    if kind == "whole":
        return dict(kind=kind, data=blob.to_bytes())
    return _resident(kind, rc.Plan(blob, packed_target=0 if kind == "packed" else None))


def _resident(kind, plan):
    ws = plan.allocate_workspace()
    plan.upload(ws)
    return dict(kind=kind, plan=plan, ws=ws, out=plan.allocate_output(),
                err=torch.zeros(1, dtype=torch.int32, device="cuda"))


def run(state):
    kind = state["kind"]
    if kind == "encode":
        data = _encode(state["case"], state["symbols"]).to_bytes()
        state["message"][:len(data)] = np.frombuffer(data, dtype=np.uint8)
        return {"container": state["message"], "bytes": len(data)}
    if kind == "whole":
        return rc.decode_blob(rc.Blob.from_bytes(state["data"]))
    if kind == "batch":
        state["batch"].decode(state["ws"], state["out"], state["err"])
        return {"symbols": state["views"], "error": state["err"]}
    plan, ws, out, err = state["plan"], state["ws"], state["out"], state["err"]
    if kind == "packed":
        plan.unpack(ws)
    if kind == "adaptive":
        plan.decode_adaptive(ws, state["index"], out, err)
    else:
        plan.decode(ws, out, err)
    return {"symbols": out, "error": err}


def exact(case, seed):
    """The symbols that were encoded: the coding is lossless."""
    kind = case["kind"]
    if kind == "encode":
        return None      # container bytes: no computed numbers
    if kind == "batch":
        syms = _map(lambda s: _symbols(s, s["seed"]), _batch_streams(case, seed))
        return {"symbols": [torch.from_numpy(s.view(np.uint8)) for s in syms], "error": torch.zeros(1, dtype=torch.int32)}
    symbols = _adaptive_symbols(case, seed)[0] if kind == "adaptive" else _symbols(case, seed)
    if kind == "whole":
        return symbols, 0
    return {"symbols": torch.from_numpy(symbols.view(np.uint8)), "error": torch.zeros(1, dtype=torch.int32)}


def work(case):
    """Symbols out, bitstream, split records, table and index in; a product and a sum per symbol."""
    if case["kind"] == "batch":
        parts = [work(dict(s, kind="decode")) for s in _batch_streams(case, 0)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    n, lanes, splits = case["n"], case["lanes"], case["splits"]
    rng = np.random.default_rng(0)
    if case["kind"] == "adaptive":
        pmfs = [_laplace(case["alphabet"], 0.5 * 32.0 ** (t / 15.0)) for t in range(16)]
    else:
        pmfs = [_pmf(case["dist"], case["param"], case["alphabet"], rng)]
    bits = sum(float(-(p[p > 0] * np.log2(p[p > 0])).sum()) for p in pmfs) / len(pmfs)
    symbol_bytes = 1 if case["alphabet"] <= 256 else 2
    moved = n * symbol_bytes + n * bits / 8
    if case["kind"] == "adaptive":
        moved += n
    moved += splits * (2.4 * lanes if case["kind"] in ("packed", "whole", "encode") else 4 * lanes + 16)
    return {"bytes": int(moved), "flops": int(2 * n)}

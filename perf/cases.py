"""The work this decoder is timed on: whole archives, batches of archives and
byte ranges of a resident archive, decoded on the device, and the host encode,
each through the package's public entry points.

A case is a dict of plain values.  Its "path" names the call:

  archive   Decoder.decode_all of one resident archive into a kept output with
            a kept workspace ("static": decode_all_static, the form for callers
            that cannot allocate device memory)
  batch     Batch.decode of many archives, the launch sequence replayed as a
            captured graph (AX_OPT_GRAPH), as bench.py --workload batch runs it
  read      Decoder.decode_range of one range (a closed-loop reader)
  serve     RangePlan.decode of many ranges at once (one admitted batch of the
            serving loop)
  encode    the host encode of one input

Inputs are the generators of synth/ (DNA, English-like text, protein
sequences, FASTQ-like reads) and encoder parameters are those that bench.py,
studies.py and the tests use.
"""
import concurrent.futures as cf
import math

import numpy as np
import torch

import paper_2608_10188_amd as ax
import synth

KIB, MIB = 1 << 10, 1 << 20

# Compression ratio of each input kind with the default parameters (measured,
# rounded): archive bytes in work() are estimated with it.
RATIO = {"dna": 2.55, "text": 5.2, "protein": 2.1, "reads": 1.76, "mixed": 3.0}

# Encoder parameters a case may set, with aceapex_encode's defaults.
PARAMS = {"block_size": 16384, "min_match": 4, "no_rep": 0, "rans_min_syms_per_lane": 32}


def listed():
    return [
        # the smallest archive of the batch workload (64 KiB, four blocks): a
        # call whose time is launches and latency
        {"name": "dna_64k", "path": "archive", "kind": "dna", "n": 64 * KIB},
        # a small ragged text through the allocation-free entry point
        {"name": "text_1m_static", "path": "archive", "kind": "text", "n": 1_000_003, "static": True},
        # the parity workload's size, an ordinary archive
        {"name": "dna_4m", "path": "archive", "kind": "dna", "n": 4 * MIB},
        # the headline workload's size, 15,500 blocks
        {"name": "dna_254m", "path": "archive", "kind": "dna", "n": 15500 * 16384},
        # deep match chains (thousands of levels), nearly every byte copied
        {"name": "text_80m", "path": "archive", "kind": "text", "n": 80 * MIB},
        # deep and shallow chains mixed, a quarter of the bytes copied; ragged
        {"name": "reads_32m", "path": "archive", "kind": "reads", "n": 32 * MIB - 77},
        # few matches; smaller blocks and the longer minimum match of the sweep
        {"name": "protein_4m_b8k", "path": "archive", "kind": "protein", "n": 4 * MIB - 1, "block_size": 8192,
         "min_match": 8},
        # the smallest blocks, the history-free encoding, few rANS lanes; ragged
        {"name": "dna_16m_b4k", "path": "archive", "kind": "dna", "n": 16 * MIB + 12345, "block_size": 4096,
         "no_rep": 1, "rans_min_syms_per_lane": 128},
        # a batch of the batch workload's size distribution (capped), 60 % DNA and 40 % text
        {"name": "batch_40", "path": "batch", "kind": "mixed", "count": 40, "cap": 4 * MIB},
        # one 16 KiB read of a resident archive, the latency a reader sees
        {"name": "read_16k", "path": "read", "kind": "dna", "n": 32 * MIB, "len": 16 * KIB},
        # a served batch of the mixed request sizes (16 KiB to 1 MiB)
        {"name": "serve_32_mixed", "path": "serve", "kind": "dna", "n": 32 * MIB, "count": 32, "len_min": 16 * KIB,
         "len_max": 1 * MIB},
        # preparing an archive on the host
        {"name": "encode_dna_4m", "path": "encode", "kind": "dna", "n": 4 * MIB},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["archive"] * 6 + ["batch", "read", "serve", "encode"])
    if path == "batch":
        return {"path": path, "kind": "mixed", "count": rng.randint(2, 40), "cap": _log_uniform(rng, 100_000, 4 * MIB)}
    if path == "read":
        n = _log_uniform(rng, 1 * MIB, 32 * MIB)
        return {"path": path, "kind": rng.choice(["dna", "dna", "reads"]), "n": n,
                "len": min(n, _log_uniform(rng, 1, 1 * MIB))}
    if path == "serve":
        lo = _log_uniform(rng, 64, 16 * KIB)
        return {"path": path, "kind": "dna", "n": _log_uniform(rng, 4 * MIB, 32 * MIB), "count": rng.randint(2, 64),
                "len_min": lo, "len_max": _log_uniform(rng, lo, 1 * MIB)}
    if path == "encode":
        return {"path": path, "kind": rng.choice(["dna", "text"]), "n": _log_uniform(rng, 4 * KIB, 4 * MIB)}
    kind = rng.choice(["dna", "dna", "dna", "text", "text", "reads", "protein"])
    hi = {"dna": 128 * MIB, "text": 48 * MIB, "reads": 24 * MIB, "protein": 4 * MIB}[kind]
    case = {"path": path, "kind": kind, "n": _log_uniform(rng, 3000, hi),
            "block_size": rng.choice([16384, 16384, 16384, 8192, 4096]),
            "min_match": rng.choice([4, 4, 4, 6, 8, 12, 32]), "no_rep": rng.choice([0, 0, 0, 1]),
            "rans_min_syms_per_lane": rng.choice([32, 32, 128])}
    if case["n"] <= 2 * MIB:
        case["static"] = rng.choice([True, False])
    return case


def _input(kind, n, seed):
    if kind == "dna" and n > 16 * MIB:  # the same bytes' shape, generated in parallel
        return synth.dna_segmented(n, seed, seg=16 * MIB, threads=8)
    return synth.GENERATORS[kind](n, seed)


def _encode(x, case, threads=0):
    return ax.encode(x, threads=threads, **{k: case[k] for k in PARAMS if k in case})


def _decoder(arc, dev):
    return ax.Decoder(arc, torch.from_numpy(arc).to(dev))


def _batch_archive(item):
    kind, n, seed = item
    return ax.encode(synth.GENERATORS[kind](n, seed), threads=1)


def _batch_plan(case):
    """Sizes and kinds of a batch case's archives (the case's own, whatever the seed)."""
    sizes, kinds = synth.batch_plan(case["count"], 4)
    return [min(int(n), case["cap"]) for n in sizes], kinds


def _serve_lens(case):
    """Request lengths of a serve case (log-uniform; the case's own, whatever the seed)."""
    return synth.trace(case["count"], 55, 1 << 30, 16384, 1000.0, case["len_min"], case["len_max"])[2]


def prepare(case, seed):
    path = case["path"]
    if path == "encode":
        return {"path": path, "x": synth.GENERATORS[case["kind"]](case["n"], seed), "case": dict(case)}
    dev = torch.device("cuda:0")
    if path == "batch":
        sizes, kinds = _batch_plan(case)
        items = [("dna" if k == 0 else "text", n, seed * 1000 + i)
                 for i, (n, k) in enumerate(zip(sizes, kinds))]
        with cf.ThreadPoolExecutor(max_workers=8) as pool:
            arcs = list(pool.map(_batch_archive, items))
        outs = [torch.zeros(n, dtype=torch.uint8, device=dev) for _, n, _ in items]
        batch = ax.Batch([_decoder(a, dev) for a in arcs], outs)
        batch.set_option(ax.OPT_GRAPH, 1)
        return {"path": path, "batch": batch, "work": batch.workspace(), "outs": outs}
    n = case["n"]
    arc = _encode(_input(case["kind"], n, seed), case)
    dec = _decoder(arc, dev)
    if path == "archive":
        st = {"path": path, "dec": dec, "out": torch.zeros(max(16, n), dtype=torch.uint8, device=dev), "n": n,
              "static": bool(case.get("static"))}
        if not st["static"]:
            st["work"] = dec.workspace()
        return st
    dec.build_index()
    if path == "read":
        rng = np.random.default_rng(seed)
        off, length = int(rng.integers(0, n - case["len"] + 1)), case["len"]
        work = torch.empty(max(256, dec.range_workspace(off, length)), dtype=torch.uint8, device=dev)
        return {"path": path, "dec": dec, "off": off, "len": length, "work": work,
                "out": torch.zeros(length, dtype=torch.uint8, device=dev)}
    _, offs, _ = synth.trace(case["count"], seed, n, 16384, 1000.0, 1, 1)
    lens = _serve_lens(case)
    offs = np.minimum(offs, n - lens)
    plan = ax.RangePlan(dec, max_blocks=int(dec.info.n_blocks), max_tokens=max(1, int(dec.info.n_matches)))
    work = torch.empty(plan.workspace_bytes, dtype=torch.uint8, device=dev)
    outs = [torch.zeros(int(v), dtype=torch.uint8, device=dev) for v in lens]
    return {"path": path, "plan": plan, "offs": offs, "lens": lens, "work": work, "outs": outs}


def run(state):
    path = state["path"]
    if path == "archive":
        if state["static"]:
            return state["dec"].decode_all_static(state["out"])[: state["n"]]
        return state["dec"].decode_all(out=state["out"], work=state["work"])
    if path == "batch":
        return state["batch"].decode(work=state["work"])
    if path == "read":
        return state["dec"].decode_range(state["off"], state["len"], state["out"], state["work"])
    if path == "serve":
        state["plan"].decode(state["offs"], state["lens"], state["outs"], state["work"])
        return state["outs"]
    arc = _encode(state["x"], state["case"])
    out = np.zeros(2 * state["x"].size + 4096, np.uint8)  # the archive, in a buffer of one size for every input
    out[: arc.size] = arc
    return [out, arc.size]


def work(case):
    """Output bytes written once and archive bytes read once (for an encode:
    the input read, the archive written).  No floating-point work."""
    path = case["path"]
    if path == "batch":
        n = sum(_batch_plan(case)[0])
    elif path == "read":
        n = case["len"]
    elif path == "serve":
        n = int(_serve_lens(case).sum())
    else:
        n = case["n"]
    return {"bytes": n + int(n / RATIO[case["kind"]]), "flops": 0}

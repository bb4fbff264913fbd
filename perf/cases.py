"""Performance cases: the work that a program using this framework has it do.

Each case is one call (or the few calls that belong together) through the
package's public entry points on seeded synthetic banks made on the GPU: banks
with the length and residue distributions of ``synth``, planted homologs so
that hits, gapped scores and alignments meet real similarity, repeat-carrying
banks, and fragment banks as six-frame translation leaves them.

The library writes hits, matches and alignments in no particular order, so
``run`` puts them into a fixed order the way a program that joins them would:
hits and matches sorted by their sequence pair and positions, alignments by the
hit that produced them.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_0804_3643_amd import binding as B
from paper_0804_3643_amd import params, synth

DEV = "cuda"
PAD, PAD_LEN = synth.PAD_CODE, synth.PAD_LEN
MEAN_LEN = 298          # residues of a protein, on average
FRAG_LEN = 16           # residues of a translated fragment, on average
PAIRS = 1.9e-4          # share of (word of bank 1, word of bank 2) pairs that share a seed key
HITS = 1.7e-3           # share of scored pairs that reach S1
PASS = 0.1              # share of hits that pass the gapped filter
TUNED = {"item_cols": [2048, 8192, 16384, 16384], "xcd_queues": 8, "gapped_threads": 512}
SCORES = 512            # ungapped scores of BLOSUM62 lie below 44 * 11 + 1


# --------------------------------------------------------------------------- the cases

def listed():
    return [
        # Stage 0 of a database: a bank of 300,000 proteins indexed once (the second bank of configuration 2).
        {"name": "index_bank", "op": "index", "n": 300_000, "kind": "protein"},
        # Six-frame translation of a nucleotide bank (TPLAST-N): 300 sequences of 50-200 kb, 37 Mnt.
        {"name": "translate_dna", "op": "translate", "n": 300, "lo": 50_000, "hi": 200_000},
        # The smallest online query: one request of 3 proteins against a resident bank (serving), where
        # launches and latency count.
        {"name": "search_one", "op": "search", "requests": 1, "per": 3, "n2": 100_000},
        # A served batch: 3 requests of 150 proteins merged, against a resident bank of 1M proteins.
        {"name": "search_batch", "op": "search", "requests": 3, "per": 150, "n2": 1_000_000},
        # A whole small bank-versus-bank search, replayed as a graph (configuration 0).
        {"name": "pipeline_small", "op": "pipeline", "n1": 200, "n2": 2_000, "kind": "protein", "tuned": False},
        # A whole search on banks with low-complexity repeats (configuration 2 at a quarter of its size).
        {"name": "pipeline_skewed", "op": "pipeline", "n1": 5_000, "n2": 75_000, "kind": "repeat", "tuned": True},
        # Ungapped extension of bank against bank: configuration 1, 10,000 x 100,000 proteins.
        {"name": "extend_large", "op": "extend", "n1": 10_000, "n2": 100_000, "kind": "protein", "units": 1,
         "tuned": True},
        # The same stage against translated fragments (TPLAST-N), many short sequences.
        {"name": "extend_fragments", "op": "extend", "n1": 1_001, "n2": 1_500_000, "kind": "fragment", "units": 1,
         "tuned": False},
        # The same stage with a matrix in finer units (BLOSUM62 in sixths of a bit), whose entries are wider.
        {"name": "extend_matrix", "op": "extend", "n1": 1_500, "n2": 30_000, "kind": "protein", "units": 3,
         "tuned": False},
        # Small gapped filter on the hits of a search, with the reference parameters.
        {"name": "gapped_hits", "op": "gapped", "n1": 1_500, "n2": 40_000, "window": 64, "band": 16, "gap_open": 11,
         "gap_extend": 1},
        # The same filter with a narrower band and window, for a quicker and stricter search.
        {"name": "gapped_narrow", "op": "gapped", "n1": 500, "n2": 30_011, "window": 40, "band": 10, "gap_open": 10,
         "gap_extend": 2},
        # Stage 3.2: full gapped alignment of the hits that passed, one search's worth.
        {"name": "align_hits", "op": "align", "n1": 1_000, "n2": 30_000},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["index", "translate", "search", "pipeline", "extend", "extend", "gapped", "align"])
    if op == "index":
        kind = rng.choice(["protein", "protein", "repeat", "fragment"])
        n = _log(rng, 100, 300_000)
        return {"op": op, "n": n * 5 if kind == "fragment" else n, "kind": kind}
    if op == "translate":
        lo = _log(rng, 300, 50_000)
        return {"op": op, "n": max(1, int(_log(rng, 100_000, 37_000_000) / (2.5 * lo))), "lo": lo, "hi": 4 * lo}
    if op == "search":
        n2 = _log(rng, 20_000, 1_000_000)
        return {"op": op, "requests": rng.randint(1, 5), "per": _log(rng, 1, 90), "n2": n2}
    if op == "gapped":
        n1 = _log(rng, 30, 1_500)
        band, window = rng.choice([(16, 64), (16, 64), (16, 50), (10, 40), (6, 32)])
        op1, ex1 = rng.choice([(11, 1), (11, 1), (10, 2), (9, 2), (12, 1)])
        n2 = _log(rng, 3_000, 15_000 if band < 16 else 40_000)
        return {"op": op, "n1": min(n1, 500) if band < 16 else n1, "n2": n2, "window": window, "band": band,
                "gap_open": op1, "gap_extend": ex1}
    if op == "align":
        return {"op": op, "n1": _log(rng, 30, 1_000), "n2": _log(rng, 1_000, 30_000)}
    kind = rng.choice(["protein", "protein", "repeat", "fragment"])
    n1, n2 = _log(rng, 60, 5_000), _log(rng, 1_000, 75_000)
    case = {"op": op, "n1": n1, "n2": n2 * 10 if kind == "fragment" else n2, "kind": kind,
            "tuned": rng.random() < 0.5}
    if op == "extend":
        case["units"] = 3 if rng.random() < 0.2 and n1 * n2 <= 45_000_000 else 1
    return case


# --------------------------------------------------------------------------- inputs

_CUM = torch.tensor(np.cumsum(synth.BACKGROUND / synth.BACKGROUND.sum()), dtype=torch.float32)


def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1_000_003 + stream) & 0x7FFFFFFFFFFFFFFF)
    return g


def _shuffled(codes, start, lens, seed, stream, pad=PAD_LEN):
    """The sequences in an order drawn from the seed.  A case's sequences are the same for every seed, so that its
    results have the same sizes, and each seed deals them to other places."""
    perm = torch.randperm(lens.numel(), device=DEV, generator=_gen(seed, stream))
    to = torch.empty_like(start)
    to[0] = pad
    to[1:] = pad + torch.cumsum(lens[perm] + pad, 0)
    row = torch.repeat_interleave(torch.arange(lens.numel(), device=DEV), lens[perm])
    j = torch.arange(row.numel(), device=DEV) - (to[row] - pad - pad * row)
    out = torch.full_like(codes, PAD)
    out[to[row] + j] = codes[start[perm[row]] + j]
    return out, to, lens[perm]


def _residues(n, g):
    u = torch.rand(n, device=DEV, generator=g)
    return torch.bucketize(u, _CUM.to(DEV), right=True).clamp_(max=19).to(torch.uint8)


def _lengths(n, g, kind):
    if kind == "fragment":  # open reading stretches between stops: geometric
        u = torch.rand(n, device=DEV, generator=g).clamp_(min=1e-7)
        return (torch.log(u) / math.log(1 - 1 / FRAG_LEN)).to(torch.int64).clamp_(0, 399) + 1
    z = torch.randn(n, device=DEV, generator=g)
    return torch.exp(math.log(300.0) - 0.18 + 0.6 * z).round_().to(torch.int64).clamp_(50, 1000)


def _bank(n, stream, kind="protein", pool=0):
    """codes uint8 (padded layout), seq_start int64[n + 1], lengths int64[n] on the GPU."""
    g = _gen(n, stream)
    lens = _lengths(n, g, kind)
    start = torch.empty(n + 1, dtype=torch.int64, device=DEV)
    start[0] = PAD_LEN
    start[1:] = PAD_LEN + torch.cumsum(lens + PAD_LEN, 0)
    codes = torch.full((int(start[-1]),), PAD, dtype=torch.uint8, device=DEV)
    flat = _residues(int(lens.sum()), g)
    at = torch.repeat_interleave(torch.arange(n, device=DEV, dtype=torch.int32), lens)
    codes[torch.arange(flat.numel(), device=DEV) + PAD_LEN * (at.to(torch.int64) + 1)] = flat
    if kind == "repeat":  # 5% of the sequences carry a run over 2, 3 or 4 letters, other ones in the two banks
        k = max(1, n // 20)
        who = torch.randperm(n, device=DEV, generator=g)[:k]
        run = torch.minimum(torch.randint(100, 401, (k,), device=DEV, generator=g), lens[who])
        off = (torch.rand(k, device=DEV, generator=g) * (lens[who] - run + 1)).to(torch.int64)
        which = torch.randint(0, 3, (k,), device=DEV, generator=g)
        row = torch.repeat_interleave(torch.arange(k, device=DEV), run)
        j = torch.arange(row.numel(), device=DEV) - torch.repeat_interleave(torch.cumsum(run, 0) - run, run)
        first = torch.tensor([0, 2, 5], device=DEV)[which[row]] + 9 * pool
        letter = first + (torch.rand(row.numel(), device=DEV, generator=g) * (2 + which[row])).to(torch.int64)
        codes[start[who[row]] + off[row] + j] = letter.to(torch.uint8)
    return codes, start, lens


def _plant(src, dst, share, stream):
    """Writes homologs of bank ``src``'s sequences over ``share`` of bank ``dst``'s (30-60% identity, a gap of a few
    letters in each)."""
    (ca, sa, la), (cb, sb, lb) = src, dst
    g = _gen(lb.numel(), stream)
    k = max(1, int(share * lb.numel()))
    d = torch.randperm(lb.numel(), device=DEV, generator=g)[:k]
    s = torch.randint(0, la.numel(), (k,), device=DEV, generator=g)
    n = torch.minimum(la[s] - 4, lb[d]).clamp_(min=0)
    row = torch.repeat_interleave(torch.arange(k, device=DEV), n)
    j = torch.arange(row.numel(), device=DEV) - torch.repeat_interleave(torch.cumsum(n, 0) - n, n)
    ident = 0.3 + 0.3 * torch.rand(k, device=DEV, generator=g)
    cut = (torch.rand(k, device=DEV, generator=g) * n).to(torch.int64)
    gap = torch.randint(0, 5, (k,), device=DEV, generator=g)
    res = ca[sa[s[row]] + j + torch.where(j >= cut[row], gap[row], 0)]
    keep = torch.rand(row.numel(), device=DEV, generator=g) < ident[row]
    cb[sb[d[row]] + j] = torch.where(keep, res, _residues(row.numel(), g))


def _pair(seed, n1, n2, kind="protein"):
    a = _bank(n1, 1, "repeat" if kind == "repeat" else "protein", 0)
    b = _bank(n2, 2, kind, 1)
    if kind != "fragment":
        _plant(a, b, 0.005, 3)
    return _shuffled(*a, seed, 4), _shuffled(*b, seed, 5)


def _index_bank(case, seed):
    return _shuffled(*_bank(case["n"], 1, case["kind"]), seed, 4)


def _matrix(units):
    if units == 1:
        return None
    return (units * synth._b62_in_alphabet_order()).astype(np.int8)


def _order(rows, columns):
    """Row order by the given (column, size) pairs, all of one record."""
    key = torch.zeros(rows.shape[0], dtype=torch.int64, device=rows.device)
    for c, size in columns:
        key.mul_(size).add_(rows[:, c])
    return torch.sort(key)


def _hit_columns(st, scores=0):
    cols = [(0, st["n1"]), (1, 1024), (2, st["n2"]), (3, 1024)]
    return cols + [(4, scores)] if scores else cols


def prepare(case, seed):
    op = case["op"]
    if op == "index":
        codes, start, _ = _index_bank(case, seed)
        ib, wb = B.index_bytes(codes.numel(), start.numel() - 1)
        return {"op": op, "codes": codes, "start": start, "out": torch.empty(ib, dtype=torch.uint8, device=DEV),
                "ws": torch.empty(wb, dtype=torch.uint8, device=DEV)}
    if op == "translate":
        dna, start = _dna(case, seed)
        return {"op": op, "tr": B.Translator(dna, start)}
    if op == "search":
        return _prepare_search(case, seed)
    a, b = _pair(seed, case["n1"], case["n2"], case.get("kind", "protein"))
    st = {"op": op, "n1": case["n1"], "n2": case["n2"]}
    tuning = TUNED if case.get("tuned") else None
    if op == "pipeline":
        ia, ib = B.build_index(a[0], a[1]), B.build_index(b[0], b[1])
        _, n_ext, items = B.ungapped_workspace_bytes(ia, ib, tuning=tuning)
        st["pipe"] = B.Pipeline(a[0], a[1], b[0], b[1], params.S1, params.S2, items, B.default_capacity(n_ext),
                                tuning=tuning)
        return st
    ia, ib = B.build_index(a[0], a[1]), B.build_index(b[0], b[1])
    if op == "extend":
        u = case["units"]
        st["scores"] = SCORES * u
        st["ext"] = B.Extender(ia, ib, params.S1 * u, matrix=_matrix(u), tuning=tuning)
        return st
    hits, _ = B.ungapped_extend(ia, ib, params.S1)
    hits = hits[_order(hits, _hit_columns(st))[1]].contiguous()
    st.update(ia=ia, ib=ib, hits=hits)
    if op == "gapped":
        st["g"] = {k: case[k] for k in ("window", "band", "gap_open", "gap_extend")}
        st["out"] = (torch.empty(hits.shape[0], dtype=torch.int32, device=DEV),
                     torch.empty(hits.shape[0], dtype=torch.uint8, device=DEV))
        return st
    st["gscore"], st["passed"] = B.gapped_filter(ia, ib, hits, params.S2)
    st["aligner"] = B.Aligner(ia, ib, hits.shape[0])
    return st


def _dna(case, seed):
    g = _gen(case["n"], 1)
    lens = torch.randint(case["lo"], case["hi"] + 1, (case["n"],), device=DEV, generator=g)
    start = torch.zeros(case["n"] + 1, dtype=torch.int64, device=DEV)
    start[1:] = torch.cumsum(lens, 0)
    u = torch.rand(int(start[-1]), device=DEV, generator=g)  # 40% G + C
    dna = torch.bucketize(u, torch.tensor([0.3, 0.5, 0.7], device=DEV), right=True).to(torch.uint8)
    return _shuffled(dna, start, lens, seed, 4, pad=0)[:2]


def _prepare_search(case, seed):
    b = _bank(case["n2"], 2)
    n = case["requests"] * case["per"]
    a = _bank(n, 1)
    _plant(b, a, 0.1, 3)
    a, b = _shuffled(*a, seed, 4), _shuffled(*b, seed, 5)
    ib = B.build_index(b[0], b[1])
    _, n_ext, items = B.ungapped_workspace_bytes(B.build_index(a[0], a[1]), ib)
    s = B.Searcher(ib, a[0].numel(), n, items, B.default_capacity(n_ext), params.S1, params.S2)
    seg = torch.arange(0, n + 1, case["per"], dtype=torch.int32)
    pinned = [t.cpu().pin_memory() for t in (a[0], a[1], seg)]
    return {"op": "search", "n1": n, "n2": case["n2"], "s": s, "host": pinned, "segments": case["requests"]}


# --------------------------------------------------------------------------- one pass

def run(st):
    op = st["op"]
    if op == "index":
        ix = B.build_index(st["codes"], st["start"], workspace=st["ws"], out_buf=st["out"])
        return {"key_off": ix.key_off(), "occ": ix.occ(), "occ_seq": ix.occ_seq()}
    if op == "translate":
        codes, starts, frag = st["tr"].run()
        return {"codes": codes, "seq_start": starts, "frag": frag}
    if op == "search":
        s, (codes, starts, seg) = st["s"], st["host"]
        s.codes[:codes.numel()].copy_(codes, non_blocking=True)
        s.starts[:starts.numel()].copy_(starts, non_blocking=True)
        s.seg_first[:seg.numel()].copy_(seg, non_blocking=True)
        s.enqueue(codes.numel(), st["n1"], n_seg=st["segments"])
        r = s.result()
        m = s.matches[:r["n_matches"]]
        return {"n_ext": r["n_ext"], "n_hits": r["n_hits"], "segments": s.seg_off[:st["segments"] + 1],
                "matches": m[_order(m, _hit_columns(st))[1]]}
    if op == "pipeline":
        p = st["pipe"]
        p.launch()
        r = p.result()
        hits, gscore, passed = p.outputs(r["n_hits"])
        # a hit with its score in one sorted word
        key, order = _order(hits, _hit_columns(st, SCORES))
        return {"n_ext": r["n_ext"], "hits": key, "gscore": gscore[order], "passed": passed[order]}
    if op == "extend":
        hits, n_ext = st["ext"].run()
        return {"n_ext": n_ext, "hits": _order(hits, _hit_columns(st, st["scores"]))[0]}
    if op == "gapped":
        gscore, passed = B.gapped_filter(st["ia"], st["ib"], st["hits"], params.S2, out=st["out"], **st["g"])
        return {"gscore": gscore, "passed": passed}
    rec, cover = st["aligner"].run(st["hits"], st["gscore"], st["passed"])
    return {"records": rec[torch.sort(rec[:, 13])[1]], "cover": cover}


# --------------------------------------------------------------------------- what a pass cannot do without

def _residues_of(n, kind="protein"):
    return n * (FRAG_LEN if kind == "fragment" else MEAN_LEN)


def _words_of(n, kind="protein"):
    # words of 4 letters inside a sequence; a geometric length of mean 16 leaves 13.2 of them
    return n * (13.2 if kind == "fragment" else MEAN_LEN - 3)


def work(case):
    """Bytes: each input read once, each output written once.  Operations: 88 per scored pair (44 additions, 44
    maxima), 8 per cell of the gapped filter's bands, 7 per cell of an alignment's rectangles."""
    op = case["op"]
    if op == "index":
        k = case["kind"]
        return {"bytes": _residues_of(case["n"], k) + PAD_LEN * case["n"] + 8 * case["n"] + 8 * _words_of(case["n"], k)
                + 8 * B.NKEYS, "flops": 0}
    if op == "translate":
        nt = case["n"] * (case["lo"] + case["hi"]) / 2
        frags = 2 * nt * 0.059  # six frames of nt / 3 codons, a stop at 6.3% of them
        return {"bytes": nt + 2 * nt * 0.937 + 40 * frags, "flops": 0}
    n1 = case["requests"] * case["per"] if op == "search" else case["n1"]
    k2 = case.get("kind", "protein")
    pairs = PAIRS * _words_of(n1) * _words_of(case["n2"], k2)
    hits = HITS * pairs
    banks = _residues_of(n1) + PAD_LEN * n1 + _residues_of(case["n2"], k2) + PAD_LEN * case["n2"]
    if op == "extend":
        return {"bytes": banks + 8 * (_words_of(n1) + _words_of(case["n2"], k2)) + 20 * hits, "flops": 88 * pairs}
    if op == "align":
        return {"bytes": banks + 25 * hits + 56 * 0.7 * PASS * hits + 4 * hits, "flops": 7 * 9.0e4 * 0.7 * PASS * hits}
    # cells of one band, edges clipped by the window
    w, bd = case.get("window", 64), case.get("band", 16)
    cells = sum(min(w, i + bd) - max(1, i - bd) + 1 for i in range(1, w + 1))
    gapped = 8 * 2 * cells * 0.85 * hits  # windows clipped at sequence ends
    if op == "gapped":
        return {"bytes": min(banks, 4 * w * hits) + 25 * hits, "flops": gapped}
    if op == "search":
        return {"bytes": banks + 8 * _words_of(case["n2"], k2) + 45 * hits, "flops": 88 * pairs + gapped}
    return {"bytes": banks + 25 * hits, "flops": 88 * pairs + gapped}


# --------------------------------------------------------------------------- 64-bit results

_CLASS2 = [1 if c in "GPATSNHQEDRK" else 0 for c in synth.ALPHABET]
_CLASS3 = [next(k for k, s in enumerate(("A", "C", "FYW", "G", "IV", "ML", "NH", "P", "QED", "RK", "TS")) if c in s)
           for c in synth.ALPHABET]
_CODONS = "KNKNTTTTRSRSIIMIQHQHPPPPRRRRLLLLEDEDAAAAGGGGVVVV*Y*YSSSS*CWCLFLF"  # AAA, AAC, ... TTT


def exact(case, seed):
    """Every output is a whole number; the stages that plain torch computes in good time are given here."""
    if case["op"] == "index":
        return _exact_index(*_index_bank(case, seed))
    if case["op"] == "translate" and case["n"] <= 2000:
        return _exact_translate(*_dna(case, seed))
    return None


def _exact_index(codes, start, lens):
    c = codes.to(torch.int64)
    t = [c[i:c.numel() - 3 + i] for i in range(4)]
    at = torch.nonzero(torch.stack([x < 20 for x in t]).all(0)).reshape(-1)
    w = [x[at] for x in t]
    c2, c3 = torch.tensor(_CLASS2, device=DEV), torch.tensor(_CLASS3, device=DEV)
    key = ((w[0] * 2 + c2[w[1]]) * 11 + c3[w[2]]) * 20 + w[3]
    order = torch.sort(key, stable=True)[1]
    off = torch.zeros(B.NKEYS + 1, dtype=torch.int64, device=DEV)
    off[1:] = torch.cumsum(torch.bincount(key, minlength=B.NKEYS), 0)
    occ = at[order]
    return {"key_off": off, "occ": occ.to(torch.int32),
            "occ_seq": (torch.searchsorted(start[:-1].contiguous(), occ, right=True) - 1).to(torch.int32)}


def _exact_translate(dna, start):
    aa = torch.tensor([synth.ALPHABET.find(x) for x in _CODONS], device=DEV)
    codes, frags = [], []
    for d, (s, e) in enumerate(zip(start[:-1].tolist(), start[1:].tolist())):
        fwd = dna[s:e].to(torch.int64)
        for frame in range(6):
            x = (fwd if frame < 3 else (3 - fwd).flip(0))[frame % 3:]
            x = x[:x.numel() // 3 * 3].reshape(-1, 3)
            p = aa[x[:, 0] * 16 + x[:, 1] * 4 + x[:, 2]]
            live = p >= 0
            before = torch.cat([live.new_zeros(1), live[:-1]])
            first = torch.nonzero(live & ~before).reshape(-1)
            codes.append(torch.where(live, p, -1))
            codes.append(p.new_full((1,), -1))  # a frame ends its last fragment
            frags.append(torch.stack([torch.full_like(first, d), torch.full_like(first, frame), first], 1))
    flat = torch.cat(codes)
    live = flat >= 0
    first = live & ~torch.cat([live.new_zeros(1), live[:-1]])
    seq = torch.cumsum(first, 0)[live]                      # 1-based fragment of each residue
    pos = torch.arange(seq.numel(), device=DEV) + PAD_LEN * seq
    n = int(seq[-1]) if seq.numel() else 0
    out = torch.full((seq.numel() + PAD_LEN * (n + 1),), PAD, dtype=torch.uint8, device=DEV)
    out[pos] = flat[live].to(torch.uint8)
    begin = torch.cat([pos[first[live]], torch.tensor([out.numel()], device=DEV)])
    return {"codes": out, "seq_start": begin, "frag": torch.cat(frags).to(torch.int32)}

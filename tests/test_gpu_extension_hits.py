"""GPU tests of the ungapped extension where hits are many: banks that share
low-complexity words, and low thresholds.  The hits equal the oracle's (exactly,
whole numbers) however often the staging areas fill, a buffer that is too small is
filled and not passed, and the time does not leave the pairs' own."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import coracle as C
from oracle import plast_oracle as O
from paper_0804_3643_amd import synth

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

# Words that banks a and b are brought to with runs of one letter, another one in each, and the kernel that must run
# (0: matrix cores, 3: an item per wavefront, in binary16).
PATHS = {"wave": (0, 0, 3), "wave_many_rows": (12_000, 2_600_000, 3), "matrix": (120_000, 2_700_000, 0)}


@pytest.fixture(scope="module")
def B():
    from paper_0804_3643_amd import binding
    binding.load()
    return binding


def _filled(seqs, words, letter):
    n = max(0, -(-(words - sum(max(0, len(s) - 3) for s in seqs)) // 4997))
    return synth.Bank.from_seqs(list(seqs) + [np.full(5000, synth.encode(letter)[0], np.uint8)] * n)


def _banks(path, a, b):
    return _filled(a, PATHS[path][0], "M"), _filled(b, PATHS[path][1], "K")


def _extend(B, ia, ib, s1, path, **kw):
    """The hits and pairs of a call, whose workspace header says which kernel ran and how many items it has in all and as
    large ones."""
    e = B.Extender(ia, ib, s1, **kw)
    hits, n_ext = e.run()
    head = e.ws[64:76].view(torch.int32).tolist()
    assert head[2] == PATHS[path][2], head
    return hits, n_ext, head[0], head[1]


def _indexes(B, *banks):
    return [B.build_index(*B.bank_to_device(b, "cuda")) for b in banks]


# Two words of one seed key: a pair scores 42 at least from the word alone, or 22.
RICH, POOR = "WCWW", "WLFW"


def _word_seqs(rng, n, word=RICH):
    """n sequences around a word, up to 30 letters on each side."""
    w = synth.encode(word)
    return [np.concatenate([rng.integers(0, 20, i), w, rng.integers(0, 20, j)]).astype(np.uint8)
            for i, j in rng.integers(0, 31, (n, 2))]


# The counts of columns around a group and a staging area, and keys of several items.
@pytest.mark.parametrize("rows,cols", [(1, 64), (1, 257), (4, 64), (4, 65), (4, 640), (9, 700), (40, 1300), (70, 5000),
                                       (3, 6000), (5, 4200), (33, 500), (64, 520)])
@pytest.mark.parametrize("path", PATHS)
def test_every_pair_a_hit(B, path, rows, cols):
    rng = np.random.default_rng(rows + cols)
    a, b = _banks(path, _word_seqs(rng, rows), _word_seqs(rng, cols))
    ia, ib = _indexes(B, a, b)
    ref, ref_ext = C.ungapped_hits(a, b, 42, matrix=O.BLOSUM62)
    for tuning in (None, {"item_cols": [512] * 4, "xcd_queues": 8}):
        hits, n_ext, items, large = _extend(B, ia, ib, 42, path, tuning=tuning)
        assert n_ext == ref_ext and len(ref) >= rows * cols
        if path == "wave_many_rows":  # the word's key has large items where 16384 pairs fit one
            assert (large > 0) == (min(rows, 32) * min(cols, 512 if tuning else 4096) >= 16384) and large < items
        assert np.array_equal(B.canonical_hits(hits), ref)


@pytest.mark.parametrize("order", ["first", "last", "mixed"])
@pytest.mark.parametrize("path", PATHS)
def test_hits_in_part_of_a_key(B, path, order):
    """Columns (in position order) that are all hits, then hardly any, or the other way round."""
    rng = np.random.default_rng(5)
    rich, poor = _word_seqs(rng, 2500), _word_seqs(rng, 2500, POOR)
    cols = {"first": rich + poor, "last": poor + rich, "mixed": [s for p in zip(rich, poor) for s in p]}[order]
    a, b = _banks(path, _word_seqs(rng, 50), cols)
    ia, ib = _indexes(B, a, b)
    ref, ref_ext = C.ungapped_hits(a, b, 42, matrix=O.BLOSUM62)
    hits, n_ext, _, _ = _extend(B, ia, ib, 42, path, tuning={"item_cols": [4096] * 4, "xcd_queues": 8})
    assert n_ext == ref_ext and 125_000 <= len(ref) < 150_000
    assert np.array_equal(B.canonical_hits(hits), ref)


@pytest.mark.parametrize("capacity", [0, 1, 300, 50_000])
@pytest.mark.parametrize("path", PATHS)
def test_capacity_is_kept(B, path, capacity):
    """All hits are counted, the first ``capacity`` places hold hits, and nothing is written past them."""
    rng = np.random.default_rng(9)
    a, b = _banks(path, _word_seqs(rng, 60), _word_seqs(rng, 2000))
    ia, ib = _indexes(B, a, b)
    ref, _ = C.ungapped_hits(a, b, 42, matrix=O.BLOSUM62)
    e = B.Extender(ia, ib, 42, capacity=capacity + 4096)
    e.hits.fill_(-7)
    n_hits, n_ext = ctypes.c_int64(0), ctypes.c_int64(0)
    rc = B.load().plast_ungapped_extend(ctypes.byref(ia.view), ctypes.byref(ib.view), ctypes.byref(e.params),
                                        B.MODES["batched"], B._ptr(e.ws), e.ws.numel(), B._ptr(e.hits), capacity,
                                        ctypes.byref(n_hits), ctypes.byref(n_ext), B._stream(None))
    assert rc == B.E_CAPACITY and n_hits.value == len(ref)
    got = e.hits.cpu().numpy()
    assert (got[capacity:] == -7).all()
    kept = {tuple(r) for r in got[:capacity].tolist()}
    assert len(kept) == capacity and kept <= {tuple(r) for r in ref.tolist()}


def _proteins(rng, n, runs=0.0):
    """n proteins; in a share of them a run of 200 letters over two."""
    p = synth.BACKGROUND / synth.BACKGROUND.sum()
    seqs = [rng.choice(20, size=int(k), p=p).astype(np.uint8) for k in rng.integers(200, 401, n)]
    for s in seqs[:round(runs * n)]:
        s[:200] = rng.choice([0, 2], 200)
    return seqs


def _kernel_ms(B, ia, ib, s1, reps=5):
    e = B.Extender(ia, ib, s1)
    e.run()
    e.run()
    B.timing_enable(True)
    t = []
    for _ in range(reps):
        e.run()
        t.append(B.timing_read()["ungapped_ms"])
    B.timing_enable(False)
    return min(t)


# Times the kernel's time on ordinary proteins at the default threshold that a lower threshold, or runs over the same two
# letters in both banks, may take.  Measured: 1.4, 2.6, 4.6, 7.9 and 2.4, the pairs and writing the hits; 10, 10, 11, 24
# and 16 where an atomic on the one counter serves a few hundred hits at most, or one wavefront has all of a key's columns.
@pytest.mark.parametrize("n1,n2,s1,runs,times", [(200, 10_000, 25, 0.0, 3.0), (500, 20_000, 20, 0.0, 6.0), (200, 10_000, 12, 0.0, 8.0),
                                                 (200, 10_000, 38, 0.1, 12.0), (500, 20_000, 38, 0.05, 8.0)])
def test_time_with_many_hits(B, n1, n2, s1, runs, times):
    rng = np.random.default_rng(3)
    usual = _indexes(B, *(synth.Bank.from_seqs(_proteins(rng, n)) for n in (n1, n2)))
    ia, ib = _indexes(B, *(synth.Bank.from_seqs(_proteins(rng, n, runs)) for n in (n1, n2)))
    assert _kernel_ms(B, ia, ib, s1) < times * _kernel_ms(B, *usual, 38)

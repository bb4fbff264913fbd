"""GPU tests of the ungapped extension's kernels: an item per wavefront (small
banks), an item per workgroup on the VALU, and the matrix cores.  The hits equal
the oracle's (exactly, whole numbers) at the edges of their tiles, of their
staging areas and of their number formats, and equal the PLAIN schedule's."""
import numpy as np
import pytest
import torch

from oracle import coracle as C
from oracle import plast_oracle as O
from paper_0804_3643_amd import synth

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

# Codes that banks a and b are brought to with empty sequences (20 codes each): the kernel is chosen by them.
PATHS = {"wave": (0, 0), "valu": (100_000, 2_600_000), "matrix": (110_000, 2_600_000)}


@pytest.fixture(scope="module")
def B():
    from paper_0804_3643_amd import binding
    binding.load()
    return binding


def _word_bank(rng, n, lo=0, hi=30):
    """n sequences around the word WCWW, 0 to 30 letters on each side of it (scans that stay inside and that leave the
    sequence)."""
    word = synth.encode("WCWW")
    seqs = []
    for _ in range(n):
        a, b = rng.integers(lo, hi + 1, 2)
        seqs.append(np.concatenate([rng.integers(0, 20, a), word, rng.integers(0, 20, b)]).astype(np.uint8))
    return synth.Bank.from_seqs(seqs)


def _padded(bank, codes):
    n = max(0, (codes - bank.codes.shape[0]) // synth.PAD_LEN + 1)
    return synth.Bank(np.concatenate([bank.codes, np.full(n * synth.PAD_LEN, synth.PAD_CODE, np.uint8)]),
                      np.concatenate([bank.seq_start, bank.seq_start[-1] + synth.PAD_LEN * np.arange(1, n + 1)]))


def _check(B, path, b1, b2, s1, matrix=None, tuning=None):
    b1, b2 = _padded(b1, PATHS[path][0]), _padded(b2, PATHS[path][1])
    ia, ib = (B.build_index(*B.bank_to_device(b, "cuda")) for b in (b1, b2))
    ref, ref_ext = C.ungapped_hits(b1, b2, s1, matrix=O.BLOSUM62 if matrix is None else matrix)
    hits, n_ext = B.ungapped_extend(ia, ib, s1, matrix=matrix, tuning=tuning)
    assert n_ext == ref_ext
    assert np.array_equal(B.canonical_hits(hits), ref)
    plain, _ = B.ungapped_extend(ia, ib, s1, mode="plain", matrix=matrix)
    assert np.array_equal(B.canonical_hits(plain), ref)
    return ref


@pytest.mark.parametrize("rows", [1, 4, 5, 8, 9, 31, 32, 33, 40, 63, 64, 65, 72, 73, 97, 130])
@pytest.mark.parametrize("path", PATHS)
def test_row_edges(B, rows, path):
    rng = np.random.default_rng(rows)
    b1, b2 = _word_bank(rng, rows), _word_bank(rng, 300)
    assert len(_check(B, path, b1, b2, 34)) > 0


@pytest.mark.parametrize("cols", [1, 31, 32, 33, 127, 128, 129, 255, 257, 600])
@pytest.mark.parametrize("path", ["wave", "matrix"])
def test_column_edges(B, cols, path):
    rng = np.random.default_rng(1000 + cols)
    b1, b2 = _word_bank(rng, 70), _word_bank(rng, cols)
    assert len(_check(B, path, b1, b2, 34, tuning={"item_cols": [512] * 4, "xcd_queues": 8})) > 0


@pytest.mark.parametrize("s1", [-3, 0, 1, 20, 39, 10 ** 6])
@pytest.mark.parametrize("path", PATHS)
def test_thresholds(B, s1, path):
    """From every pair a hit (the staging areas overflow) to none."""
    rng = np.random.default_rng(7)
    b1, b2 = _word_bank(rng, 100), _word_bank(rng, 400)
    ref = _check(B, path, b1, b2, s1)
    assert (len(ref) == 0) == (s1 == 10 ** 6)


@pytest.mark.parametrize("kind", ["plus15", "extremes", "asymmetric", "sixteen", "halves", "wide"])
@pytest.mark.parametrize("path", PATHS)
def test_matrices(B, kind, path):
    """Entries at the edge of the 6-bit format (15 and -15), orientation, the first value past it, and entries that
    need 16-bit integers."""
    rng = np.random.default_rng(11)
    m = {"plus15": np.full((20, 20), 15),
         "extremes": rng.choice([-15, 15], (20, 20)),
         "asymmetric": rng.integers(-15, 16, (20, 20)),
         "sixteen": np.where(np.eye(20) > 0, 16, rng.integers(-15, 16, (20, 20))),
         "wide": rng.integers(-100, 101, (20, 20)),
         "halves": np.where(np.eye(20) > 0, 7, -np.tri(20, dtype=int) * 3 + 1)}[kind].astype(np.int8)
    b1, b2 = _word_bank(rng, 90), _word_bank(rng, 200)
    ref = _check(B, path, b1, b2, 60 if kind != "plus15" else 300, matrix=m)
    assert len(ref) > 0
    if kind == "plus15":
        assert ref[:, 4].max() == 44 * 15


@pytest.mark.parametrize("seed", range(4))
@pytest.mark.parametrize("path", PATHS)
def test_heavy_keys(B, seed, path):
    """Banks over few letters: keys of many sizes, several items and groups a key, several queues."""
    rng = np.random.default_rng(40 + seed)
    b1 = synth.random_bank(rng, 120, 20, 90, 3 + seed)
    b2 = synth.random_bank(rng, 400, 4, 120, 3 + seed)
    m = O.BLOSUM62.astype(np.int8) if seed % 2 else None
    _check(B, path, b1, b2, 45, matrix=m, tuning={"item_cols": [1024, 512, 2048, 16384], "xcd_queues": 8 if seed < 2 else 1})


@pytest.mark.parametrize("entry,s1", [(46, 1), (46, 2023), (46, 2024), (46, 2025), (47, 2068), (-46, 700), (-47, 700)])
@pytest.mark.parametrize("path", ["wave", "valu"])
def test_largest_entries_in_binary16(B, entry, s1, path):
    """Entries all 46 (the best is 2024, every integer below it exact in binary16) or 47 (16-bit integers), at the
    thresholds around the best, and random signs of them."""
    rng = np.random.default_rng(13)
    m = (np.full((20, 20), entry) if entry > 0 else rng.choice([-entry, entry], (20, 20))).astype(np.int8)
    b1, b2 = _word_bank(rng, 90), _word_bank(rng, 200)
    ref = _check(B, path, b1, b2, s1, matrix=m)
    assert (len(ref) > 0) == (s1 <= 44 * abs(entry))


@pytest.mark.parametrize("codes", [4_400_000, 4_600_000])
def test_columns_shared_between_xcds(B, codes):
    """Bank b below and past the size from which every XCD takes an eighth of a key's columns (512 codes a key): keys of
    fewer columns than XCDs, of one item and of several, and of more than 8 rows."""
    rng = np.random.default_rng(19)
    b1 = synth.random_bank(rng, 40, 5, 60, 5)
    b2 = synth.Bank.from_seqs([rng.integers(0, 5 if i % 3 else 20, n).astype(np.uint8)
                               for i, n in enumerate(rng.integers(0, 80, 3000))])
    b2 = _padded(b2, codes)
    ia, ib = B.build_index(*B.bank_to_device(b1, "cuda")), B.build_index(*B.bank_to_device(b2, "cuda"))
    hits, _ = B.ungapped_extend(ia, ib, 25, tuning={"item_cols": [512, 512, 512, 512]})
    ref, _ = C.ungapped_hits(b1, b2, 25, matrix=O.BLOSUM62)
    assert len(ref) > 1000 and np.array_equal(B.canonical_hits(hits), ref)

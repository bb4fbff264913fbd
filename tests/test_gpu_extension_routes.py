"""GPU tests of the ungapped extension's kernels on banks brought to their sizes with
words, not with empty sequences, so that the rules on words choose the kernel named; the
workspace's header says that it ran.  The cases, and the oracle that they are compared
with, are those of the kernels' edge tests."""
import numpy as np
import pytest
import torch

import test_gpu_extension_kernels as K
from oracle import coracle as C
from oracle import plast_oracle as O
from paper_0804_3643_amd import synth

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

# Words of banks a and b, which runs of one letter bring them to (another one in each bank), and the kernels that may run:
# 0 matrix cores, 1 and 2 an item per workgroup (binary16, int16), 3 and 4 an item per wavefront.
PATHS = {"valu": ((90_000, "M"), (2_800_000, "P")), "matrix": ((110_000, "M"), (2_800_000, "P")),
         "shared": ((0, "M"), (4_600_000, "P"))}


def _padded(bank, fill):
    words, letter = fill
    have = np.maximum(np.diff(bank.seq_start) - synth.PAD_LEN - 3, 0).sum()
    n = max(0, -(-(words - int(have)) // 4997))
    run = np.concatenate([np.full(5000, synth.encode(letter)[0], np.uint8),
                          np.full(synth.PAD_LEN, synth.PAD_CODE, np.uint8)])
    return synth.Bank(np.concatenate([bank.codes, np.tile(run, n)]),
                      np.concatenate([bank.seq_start, bank.seq_start[-1] + run.size * np.arange(1, n + 1)]))


class _Seen:
    """The binding, whose batched calls note the kernel that ran."""

    def __init__(self, binding):
        self._b, self.kernels = binding, []

    def __getattr__(self, name):
        return getattr(self._b, name)

    def ungapped_extend(self, ia, ib, s1, mode="batched", **kw):
        e = self._b.Extender(ia, ib, s1, mode=mode, **kw)
        out = e.run()
        if mode == "batched":
            self.kernels.append(e.ws[64:76].view(torch.int32).tolist()[2])
        return out


@pytest.fixture
def B(monkeypatch):
    from paper_0804_3643_amd import binding
    binding.load()
    monkeypatch.setattr(K, "PATHS", PATHS)
    monkeypatch.setattr(K, "_padded", _padded)
    return _Seen(binding)


def _ran(B, path, matrix_cores=True):
    allowed = {"valu": {1, 2}, "matrix": {0} if matrix_cores else {1, 2}, "shared": {3, 4}}[path]
    assert B.kernels and set(B.kernels) <= allowed, (path, B.kernels)


@pytest.mark.parametrize("rows", [1, 4, 8, 9, 31, 32, 33, 63, 64, 65, 72, 73, 130])
@pytest.mark.parametrize("path", PATHS)
def test_row_edges(B, rows, path):
    K.test_row_edges(B, rows, path)
    _ran(B, path)


@pytest.mark.parametrize("cols", [1, 31, 32, 33, 127, 128, 129, 257, 600])
@pytest.mark.parametrize("path", PATHS)
def test_column_edges(B, cols, path):
    K.test_column_edges(B, cols, path)
    _ran(B, path)


@pytest.mark.parametrize("s1", [1, 20, 39, 10 ** 6])
@pytest.mark.parametrize("path", PATHS)
def test_thresholds(B, s1, path):
    K.test_thresholds(B, s1, path)
    _ran(B, path)


@pytest.mark.parametrize("kind", ["plus15", "extremes", "asymmetric", "sixteen", "halves", "wide"])
@pytest.mark.parametrize("path", PATHS)
def test_matrices(B, kind, path):
    K.test_matrices(B, kind, path)
    _ran(B, path, kind not in ("sixteen", "wide"))


@pytest.mark.parametrize("seed", range(4))
@pytest.mark.parametrize("path", PATHS)
def test_heavy_keys(B, seed, path):
    K.test_heavy_keys(B, seed, path)
    _ran(B, path)


@pytest.mark.parametrize("rows,cols", [(3, 6000), (20, 5000), (64, 2600)])
def test_columns_shared_between_xcds(B, rows, cols):
    """Small and large items of a bank b of which every XCD takes an eighth: keys of fewer columns than XCDs and of
    several items; and the first ones of the list are the large ones."""
    rng = np.random.default_rng(rows)
    b1 = _padded(K._word_bank(rng, rows), (12_000, "M"))
    b2 = _padded(K._word_bank(rng, cols), PATHS["shared"][1])
    ia, ib = (B.build_index(*B.bank_to_device(b, "cuda")) for b in (b1, b2))
    e = B.Extender(ia, ib, 34, tuning={"item_cols": [1024, 4096, 8192, 16384], "xcd_queues": 8})
    hits, n_ext = e.run()
    ref, ref_ext = C.ungapped_hits(b1, b2, 34, matrix=O.BLOSUM62)
    assert n_ext == ref_ext and len(ref) >= rows * cols and np.array_equal(B.canonical_hits(hits), ref)
    items, large, kernel = e.ws[64:76].view(torch.int32).tolist()
    assert kernel == 3 and (large > 0) == (min(rows, 32) * min(cols, 4096) >= 16384) and large < items

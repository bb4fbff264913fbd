"""GPU test of the gapped filter at every band: the packed kernel has band 16 alone,
the general one is compiled for the even bands and masks the outermost cells of the
ones between; scores equal the oracle's exactly, with gaps cheap enough that the best
paths run along the band's edges."""
import numpy as np
import pytest
import torch

from oracle import coracle as C
from paper_0804_3643_amd import synth

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.fixture(scope="module")
def B():
    from paper_0804_3643_amd import binding
    binding.load()
    return binding


@pytest.fixture(scope="module")
def banks():
    """Homologs with long gaps (shifts around every band's edge), and short sequences whose ends clip the windows."""
    rng = np.random.default_rng(77)
    a, b = [], []
    for i in range(60):
        s = rng.integers(0, 20, 90).astype(np.uint8)
        gap = i % 20
        cut = int(rng.integers(24, 60))
        t = np.concatenate([s[:cut], s[cut + gap:]]) if i % 2 else np.concatenate([s[:cut], rng.integers(0, 20, gap).astype(np.uint8), s[cut:]])
        keep = rng.random(len(t)) < 0.9
        b.append(np.where(keep, t, rng.integers(0, 20, len(t))).astype(np.uint8))
        a.append(s)
    for n in list(range(4, 24)) + [64, 65, 80]:
        s = rng.integers(0, 20, n).astype(np.uint8)
        a.append(s)
        b.append(s.copy())
    return synth.Bank.from_seqs(a), synth.Bank.from_seqs(b)


@pytest.mark.parametrize("band", range(17))
@pytest.mark.parametrize("window,gap_open,gap_extend", [(64, 2, 1), (37, 11, 1), (5, 0, 1), (64, 3, 0)])
def test_every_band(B, banks, band, window, gap_open, gap_extend):
    b1, b2 = banks
    ia, ib = (B.build_index(*B.bank_to_device(b, "cuda")) for b in banks)
    hits, _ = B.ungapped_extend(ia, ib, 20)
    h = hits.cpu().numpy().astype(np.int64)
    assert len(h) > 500
    par = dict(window=window, band=band, gap_open=gap_open, gap_extend=gap_extend)
    gs, ps = B.gapped_filter(ia, ib, hits, 40, **par)
    ref = C.gapped_scores(b1, b2, h, **par)
    assert np.array_equal(gs.cpu().numpy().astype(np.int64), ref)
    assert np.array_equal(ps.cpu().numpy().astype(bool), ref >= 40)


@pytest.mark.parametrize("n", [1, 2, 3, 1000, 16383, 16384, 16385, 40000])
@pytest.mark.parametrize("window,gap_open,gap_extend,threads", [(64, 2, 1, 256), (63, 11, 1, 128), (17, 3, 0, 512),
                                                                (1, 0, 1, 256)])
def test_few_hits_and_many(B, banks, n, window, gap_open, gap_extend, threads):
    """Around the number of hits up to which a hit takes half a wavefront instead of a lane; some name no sequence."""
    b1, b2 = banks
    ia, ib = (B.build_index(*B.bank_to_device(b, "cuda")) for b in banks)
    hits, _ = B.ungapped_extend(ia, ib, 20)
    rng = np.random.default_rng(n)
    h = hits.cpu().numpy()[rng.integers(0, hits.shape[0], n)]
    par = dict(window=window, gap_open=gap_open, gap_extend=gap_extend)
    ref = C.gapped_scores(b1, b2, h.astype(np.int64), **par)
    bad = (rng.random(n) < 0.01) & (np.arange(n) > 0)
    h[bad, rng.integers(0, 4)] = -1
    ref[bad] = -1
    gs, ps = B.gapped_filter(ia, ib, torch.from_numpy(h).cuda(), 40, tuning={"gapped_threads": threads}, **par)
    assert np.array_equal(gs.cpu().numpy().astype(np.int64), ref)
    assert np.array_equal(ps.cpu().numpy().astype(bool), ref >= 40)

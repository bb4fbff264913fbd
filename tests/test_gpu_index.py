"""GPU tests of the index build at the edges of its tiles (32 positions a lane,
2048 a wavefront, 8192 a workgroup): key_off, occ and occ_seq equal the oracle's."""
import sys

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


@pytest.mark.parametrize("shift", [0, 1, 4])
@pytest.mark.parametrize("n_padded", [60, 2047, 2048, 2049, 2080, 8191, 8192, 8193, 10240, 65535, 70001])
def test_index_at_the_edges_of_tiles(B, n_padded, shift):
    """Banks that end around a lane's, a tile's and a workgroup's last position,
    of random letters and of one letter (a lane's 32 words all in one bucket),
    with the codes on 16-byte, 4-byte and odd addresses."""
    rng = np.random.default_rng(n_padded)
    for letters, cuts in ((20, 5), (1, 0)):
        print("[gpu-test] index n_padded %d shift %d letters %d" % (n_padded, shift, letters), flush=True)
        sys.stdout.flush()
        room = n_padded - 20 * (cuts + 2)  # letters of cuts + 1 sequences
        if room < cuts + 1:
            cuts, room = 0, n_padded - 40
        at = np.sort(rng.integers(0, room + 1, cuts))
        lens = np.diff(np.concatenate([[0], at, [room]]))
        bank = synth.Bank.from_seqs([rng.integers(0, letters, n).astype(np.uint8) for n in lens])
        assert int(bank.seq_start[-1]) == n_padded
        codes, st = B.bank_to_device(bank, "cuda")
        moved = torch.empty(codes.numel() + shift, dtype=torch.uint8, device="cuda")[shift:]
        moved.copy_(codes)
        ix = B.build_index(moved, st)
        k, s, p = C.build_index(bank)
        occ_seq = ix.occ_seq().cpu().numpy().astype(np.int64)
        occ = ix.occ().cpu().numpy().astype(np.int64)
        assert np.array_equal(ix.key_off().cpu().numpy(), k)
        assert np.array_equal(occ_seq, s)
        assert np.array_equal(occ - bank.seq_start[occ_seq], p)


@pytest.mark.parametrize("code", [21, 127, 128, 148, 255])
def test_index_refuses_codes_that_are_no_letters(B, code):
    """Beside residues and in a separator run, the first and last byte of a
    dword of codes."""
    bank = synth.random_bank(np.random.default_rng(3), 40, 100, 200)
    codes, st = B.bank_to_device(bank, "cuda")
    for at in (20, 23, 2047, 2048, int(bank.seq_start[1]) - 1, codes.numel() - 1):
        bad = codes.clone()
        bad[at] = code
        with pytest.raises(B.PlastError) as e:
            B.build_index(bad, st)
        assert e.value.code == B.E_ALPHABET

"""CPU tests of the rules by which the BATCHED schedule chooses the kernel of the
ungapped extension: they look at words, whatever the number of separators between
them, and a bank's words are those of its sequences."""
import os
import subprocess

import numpy as np
import pytest

from paper_0804_3643_amd import synth

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_0804_3643_amd", "csrc")
WAVE, GROUP, MATRIX = range(3)


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("route")
    src, exe = d / "route.cpp", d / "route"
    src.write_text("""
#include <stdio.h>
#include "ungapped_route.h"
int main() {  // lines of: codes and sequences of bank a, of bank b, whether the matrix cores hold the scores, threshold
  long long ca, cb;
  int na, nb, m, s1;
  while (scanf("%lld %d %lld %d %d %d", &ca, &na, &cb, &nb, &m, &s1) == 6) {
    const bool low = plast::low_threshold(s1, 116);  // BLOSUM62's diagonal
    const double a = plast::bank_words(ca, na), b = plast::bank_words(cb, nb);
    printf("%.0f %.0f %d %d\\n", a, b, (int)plast::ungapped_route(a, b, cb, m != 0, low), (int)plast::columns_shared(cb, 512) + 2 * plast::columns_shared(cb, 8) + 4 * plast::columns_shared(cb, 7));
  }
}
""")
    subprocess.check_call(["g++", "-std=c++17", "-I" + CSRC, str(src), "-o", str(exe)])

    def ask(*rows):
        text = "".join("%d %d %d %d %d %d\n" % (*r, *((38,) if len(r) == 5 else ())) for r in rows)
        out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(int(x) for x in line.split()) for line in out.splitlines()]
    return ask


def _bank(words, length):
    """Codes and sequences of a bank of sequences of a length, of about so many words."""
    n = max(1, round(words / (length - 3)))
    return n * length + 20 * (n + 1), n


def test_words_of_a_bank(rules):
    rng = np.random.default_rng(1)
    for lo, hi in ((3, 30), (50, 400), (0, 3)):
        bank = synth.random_bank(rng, 100, lo, hi)
        lens = np.diff(bank.seq_start) - 20
        got = rules((bank.codes.size, lens.size, 20, 0, 1))[0]
        assert got[:2] == (max(int(lens.sum()) - 3 * lens.size, 0), 0)
        if lo == 3:
            assert got[0] == np.maximum(lens - 3, 0).sum()


@pytest.mark.parametrize("length1", [16, 60, 300])
@pytest.mark.parametrize("words1,words2,expected", [
    (2_000, 3_000_000, WAVE), (60_000, 3_000_000, WAVE), (60_000, 9_000_000, WAVE),     # few pairs, few rows
    (90_000, 9_000_000, GROUP), (120_000, 9_000_000, MATRIX),                             # 10 and 14 rows a key
    (90_000, 28_000_000, MATRIX), (60_000, 28_000_000, WAVE),                             # a large bank b
    (60_000, 200_000_000, MATRIX), (30_000, 200_000_000, WAVE),                           # a larger one
    (300_000, 600_000, WAVE), (300_000, 1_000_000, WAVE), (300_000, 2_000_000, MATRIX)])  # few columns a key
def test_route_by_words(rules, length1, words1, words2, expected):
    """The same kernel for as many words in fragments, short sequences and proteins."""
    a, b = _bank(words1, length1), _bank(words2, 300)
    held, other = rules((*a, *b, 1), (*a, *b, 0))
    assert held[2] == expected
    assert other[2] == (GROUP if expected == MATRIX else expected)


@pytest.mark.parametrize("words1,words2,expected", [
    (60_000, 3_000_000, GROUP), (300_000, 600_000, GROUP), (60_000, 600_000, GROUP),  # rows and pairs enough
    (60_000, 300_000, WAVE), (8_000, 30_000_000, WAVE),                               # few pairs, few rows
    (120_000, 9_000_000, MATRIX), (90_000, 9_000_000, GROUP)])                        # as at any threshold
def test_route_at_low_thresholds(rules, words1, words2, expected):
    a, b = _bank(words1, 300), _bank(words2, 300)
    got = [r[2] for r in rules(*((*a, *b, 1, s1) for s1 in (-5, 1, 20, 21, 38)))]
    assert got[:3] == [expected] * 3 and got[3] == got[4] == rules((*a, *b, 1))[0][2]
    if expected != GROUP or words2 == 9_000_000:
        assert got[3] == expected


def test_shared_columns(rules):
    sizes = (3_200_000, 4_400_000, 4_600_000, 32_000_000, 64_000_000, 64_000_001, 318_000_000)
    # bits: launches of 512, 8 and 7 workgroups, the last of which would leave an eighth of the columns out
    assert [r[3] for r in rules(*((1000, 3, c, c // 318, 1) for c in sizes))] == [0, 0, 3, 3, 3, 0, 0]

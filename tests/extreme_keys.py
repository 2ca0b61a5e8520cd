"""Bootstrapping keys and inputs at the edges of the blind rotation's exactness
argument: words of the largest magnitude whose low parts (the split of
csrc/fft.h) are at their ends, met by digits at theirs.

The first two CMux steps are arranged.  With a body of 0 and a mask word of 2^31
the first step sees (X^1024 - 1) B = -2 MU in every coefficient, three digits of
-64; its key gives A the same value MU in every coefficient, so that the second
step has six digit polynomials of -64 throughout and an extreme key.  The later
steps meet extreme keys with digits that look random."""
import os
import re

import numpy as np

N, n, ELL, BG_BIT = 1024, 630, 3, 7
MU = 0xC0810000  # -2 MU = -64 (2^25 + 2^18 + 2^11): digits (-64, -64, -64)
HALF = 1 << 31   # a mask word of 2^31 rotates by 1024, i.e. negates

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_12761_amd", "csrc")
KEY_SHIFT = int(re.search(r"constexpr int KEY_SHIFT = (\d+);", open(os.path.join(CSRC, "fft.h")).read()).group(1))


def split(word):
    """(hi, lo) with word = 2^KEY_SHIFT hi + lo as a signed number, lo in [-2^(KEY_SHIFT-1), 2^(KEY_SHIFT-1))."""
    k = (word & 0xFFFFFFFF) - ((word & HALF) << 1)
    lo = ((k + (1 << (KEY_SHIFT - 1))) % (1 << KEY_SHIFT)) - (1 << (KEY_SHIFT - 1))
    return (k - lo) >> KEY_SHIFT, lo


_E = 1 << (KEY_SHIFT - 1)
POS_LOW = (HALF - 1) // (2 * _E) * 2 * _E + _E  # largest positive word with lo = -E: the largest hi
POS_HIGH = POS_LOW - 1                          # lo = E - 1
NEG_HIGH = HALF + _E - 1                        # -2^31 + E - 1: lo = E - 1, the smallest hi
NEG_LOW = HALF + _E                             # lo = -E
assert [split(w)[1] for w in (POS_LOW, POS_HIGH, NEG_HIGH, NEG_LOW)] == [-_E, _E - 1, _E - 1, -_E]
assert split(POS_LOW)[0] == -split(NEG_HIGH)[0] == HALF >> KEY_SHIFT


def _constant(w):
    return np.full(N, w, np.uint32)


def _wave(f, plus, minus):
    """Words whose signs (and low parts) follow one frequency of the transform."""
    s = np.cos(np.pi * (2 * f + 1) * np.arange(N) / N)
    return np.where(s >= 0, plus, minus).astype(np.uint32)


# name -> words of the key rows' A and B polynomials
CASES = {
    "lows down": (_constant(POS_LOW), _constant(POS_LOW)),
    "lows up": (_constant(NEG_HIGH), _constant(NEG_HIGH)),
    "A down B up": (_constant(POS_LOW), _constant(NEG_HIGH)),
    "A up B down": (_constant(NEG_HIGH), _constant(POS_LOW)),
    "hi apart": (_constant(POS_LOW), _constant(NEG_LOW)),
    "wave 0": (_wave(0, POS_HIGH, NEG_LOW), _wave(0, NEG_HIGH, POS_LOW)),
    "wave 301": (_wave(301, POS_HIGH, NEG_LOW), _wave(301, NEG_HIGH, POS_LOW)),
    "wave 511": (_wave(511, POS_LOW, NEG_HIGH), _wave(511, POS_LOW, NEG_HIGH)),
}


def keys(name):
    """bk [630][6][2][1024]: the arranged first step, then the case's words, negated from step to step."""
    words = np.stack(CASES[name])
    bk = np.broadcast_to(words, (n, 2 * ELL, 2, N)).copy()
    bk[2::2] = (0 - bk[2::2].astype(np.int64)).astype(np.uint32)
    bk[0] = 0
    bk[0, ELL, 0, 0] = (0 - (MU >> 6)) & 0xFFFFFFFF  # digit -64 of B's first row: A += -64 (-MU / 64) = MU
    return bk


def rows():
    """Inputs [5][631]: both arranged steps and then none (every later mask word
    0); both, then random words; a second step with half the coefficients at
    digits of 0; two without arranged steps."""
    import synth
    r = synth.uniform_ciphertexts(78, "extreme digits", (5,))
    r[:3, n] = 0
    r[:2, :2] = HALF
    r[0, 2:n] = 0
    r[2, 0], r[2, 1] = HALF, 1 << 30
    return r

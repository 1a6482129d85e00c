"""The autotuner's choice from its timings: an entry governs calls alone and
lists, so a unit that is faster in one and slower in the other is not entered."""
from paper_2506_03747_amd.autotune import choose

OWN = (1.0, 3.0)


def test_choice_weighs_calls_alone_and_lists():
    A, B, C = (1, 4, 4), (1, 4, 2), (1, 2, 2)
    assert choose(OWN, {}) is None
    assert choose(OWN, {A: (0.9, 3.5), B: (1.2, 2.0)}) is None          # a gain in one, a loss in the other
    assert choose(OWN, {A: (0.99, 2.97), B: (1.01, 3.0)}) is None       # nothing beyond the noise
    assert choose(OWN, {A: (0.9, 3.03), B: (1.5, 2.0)}) == A
    assert choose(OWN, {A: (0.9, 2.9), B: (1.01, 2.0), C: (0.8, 3.2)}) == B

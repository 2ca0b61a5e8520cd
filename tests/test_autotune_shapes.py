"""The autotuner's list of launch shapes: each entry launches something else than
every other (the tuning knobs as include/vlp.h states them)."""
from paper_2506_12761_amd import autotune


def _launches(shape):
    """(kernel's wavefronts per rotation, rotations per workgroup, rotations per
    CU a round is sized for, most gates of a key-switching tile)."""
    r, w, b, k = shape
    br = {0: ("automatic",), 1: (1, w, w * b), 2: (6 if w == 1 else 3, min(w, 2), w * b), 4: (6, 1, b)}[r]
    return br + (min(k, 256),)


def test_no_two_shapes_launch_the_same():
    assert len({_launches(s) for s in autotune.SHAPES}) == len(autotune.SHAPES)


def test_every_kernel_and_the_default_are_among_them():
    got = {_launches(s) for s in autotune.SHAPES}
    assert ("automatic", 256) in got and ("automatic", 128) in got
    assert {s[0] for s in autotune.SHAPES} == {0, 1, 2, 4}
    assert {(1, 4, 4), (1, 8, 8), (3, 2, 4), (6, 1, 1)} <= {g[:3] for g in got if len(g) == 4}

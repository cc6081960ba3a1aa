"""What the tuner keeps: the current value unless another is faster by more than
the timings of one launch differ among themselves; a knob whose kernels did not
run keeps its value."""
from paper_2202_02840_amd import autotune as at


def test_choice():
    assert at.choose({0: 1.01, 4: 1.0, 8: 1.3}, 0) == 0
    assert at.choose({0: 1.05, 4: 1.0, 8: 1.3}, 0) == 4
    assert at.choose({0: 1.05, 4: 1.0, 8: 1.3}, 16) == 4
    assert at.choose({1: 0.0, 2: 0.0, 4: 0.0}, 4) == 4


def test_candidates_hold_the_defaults():
    assert set(at.CANDIDATES) == set(at.DEFAULT)
    for knob, cands in at.CANDIDATES.items():
        assert at.DEFAULT[knob] in cands, knob
        assert len(set(cands)) == len(cands)
    assert all(isinstance(k, tuple) for k in at.KERNEL.values())

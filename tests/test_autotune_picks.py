"""What the autotuner times is what a unit length sets.  Short walks over pairs are
cut into 64 units or units of 16 steps, so at 14 to 18 photons every candidate
splits the sampler's minors alike and the shortest is the pick; at 27 and 28
photons nearly every item of an FP64 batch goes over the pair walk, which splits
itself, and lengths tuned on none are the default."""
import pytest

from paper_2309_07027_amd import binding as B

pytestmark = pytest.mark.gpu

DEFAULT = 512


def test_candidates_that_split_alike_share_a_rate():
    print("case autotune minors", flush=True)
    B.autotune(14, 18, precision=B.BBFG_MINORS)
    assert [B.batch_unit_length(n, precision=B.BBFG_MINORS) for n in range(14, 19)] == [64] * 5


def test_a_size_whose_items_all_go_over_pairs_keeps_the_default():
    print("case autotune without items", flush=True)
    B.autotune(34, 35)
    assert [B.batch_unit_length(n) for n in (34, 35)] == [DEFAULT] * 2

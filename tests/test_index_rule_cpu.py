"""When the index builder spreads its first round over the whole chip (two launches more): by how much there is to compare,
not by the number of sequences alone (radix_debug_index_first_round, the function the builder calls)."""
import os

import pytest

from paper_2601_15013_amd import binding


@pytest.fixture(scope="module")
def rule():
    if not os.path.exists(binding.LIB_PATH):
        from paper_2601_15013_amd import build
        build.build()
    return binding.load_library().radix_debug_index_first_round


@pytest.mark.parametrize("B,length", [(1, 100000), (16, 8192), (17, 8), (17, 64), (17, 2500), (20, 32), (24, 40), (32, 300), (48, 40),
                                      (48, 450), (64, 40)])
def test_little_to_compare_stays_in_one_kernel(rule, B, length):
    assert rule(B, B * length) == 0


@pytest.mark.parametrize("B,length", [(24, 2400), (48, 1200), (64, 700), (128, 24), (512, 6), (2048, 512), (65535, 1)])
def test_much_to_compare_takes_the_chip(rule, B, length):
    assert rule(B, B * length) == 1


def test_more_work_never_goes_back_to_one_workgroup(rule):
    for B in (17, 18, 33, 34, 50, 66, 82, 100):
        lengths = [rule(B, B * n) for n in (1, 8, 64, 256, 512, 1024, 4096, 16384)]
        assert lengths == sorted(lengths)
    for n in (1, 64, 1024):
        per_batch = [rule(B, B * n) for B in range(1, 200)]
        assert per_batch == sorted(per_batch)


def test_bad_sizes_are_refused(rule):
    assert rule(0, 5) == -2 and rule(5, 0) == -2 and rule(1 << 28, 2**31 - 1) == 1

"""The keyed mix of the symmetry check (dpo_pair.h) on the CPU: what is paired
sums to zero under every key, and unpaired entries do so under few, also when
they lie next to each other or the key makes a factor trivial."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("mix") / "pair_mix")
    r = subprocess.run(["g++", "-std=c++17", "-O2", os.path.join(HERE, "host", "pair_mix.cpp"), "-I",
                        os.path.join(ROOT, "paper_2201_02789_amd", "csrc"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0
    return [x.split() for x in r.stdout.splitlines()]


def test_paired_entries_and_loops_sum_to_zero(lines):
    assert not [x for x in lines if x[0] == "PAIRED"]


def test_one_entry_without_its_reverse_is_never_missed(lines):
    some = [x for x in lines if x[2] in ("single", "twice", "cycle3")]
    assert len(some) > 30
    for bits, key, name, miss, keys in some:
        assert int(miss) == 0, (bits, key, name, miss)


def test_sets_of_unpaired_entries_are_missed_by_few_keys(lines):
    """Two odd words give 2^(2 N - 2) values of h: 8-bit words may miss at 16
    times 2^-14.  16-bit words must miss more rarely than any one coincidence of
    a word (2^-16) would, by a factor of 16.  32-bit words, given one such
    coincidence, may not miss 2^-12 of the keys."""
    for bits, key, name, miss, keys in lines:
        share = int(miss) / int(keys)
        limit = {"8": 2 ** -10, "16": 2 ** -20, "32": 2 ** -12}[bits]
        assert share <= limit, (bits, key, name, miss, keys)

"""Variant grouping where its paths change, against the oracle: a variant that
most cases share (counted through the block cache), variants of 254, 255 and
256 cases (the count digit's last exact value), several thousand variants of
255 cases or more (ordered by pairs), more than 16384 of them (byte passes),
lengths around the 1024-event hash window, no cases at all."""
import numpy as np
import pytest
import torch

from paper_2204_04898_amd import pm4g
from tests.gpu_util import check_variants, note

pytestmark = pytest.mark.gpu


def _from_sequences(seqs, counts, seed):
    """A shuffled log in which sequence k occurs in counts[k] cases."""
    rng = np.random.default_rng(seed)
    which = rng.permutation(np.repeat(np.arange(len(seqs)), counts))
    L = np.array([len(s) for s in seqs])[which]
    flat = np.concatenate([np.asarray(s) for s in seqs])
    off = np.cumsum([0] + [len(s) for s in seqs])[:-1]
    case = np.repeat(np.arange(len(which)), L)
    pos = np.arange(len(case)) - np.repeat(np.cumsum(L) - L, L)
    act = flat[np.repeat(off[which], L) + pos]
    rows = rng.permutation(len(case))
    return case[rows].astype(np.int32), act[rows].astype(np.int32), pos[rows].astype(np.int64)


def test_one_variant_in_most_cases():
    rng = np.random.default_rng(1)
    seqs = [[0, 1, 2]] + [rng.integers(0, 9, 5).tolist() for _ in range(3000)]
    note("variant paths: one frequent variant")
    check_variants(*_from_sequences(seqs, [90_000] + [1] * 3000, 2), 9)


def test_counts_around_the_digit_bound():
    seqs = [[i % 8, i // 8, 7] for i in range(40)]
    note("variant paths: counts 1..600")
    check_variants(*_from_sequences(seqs, [253, 254, 255, 256, 257, 1, 2, 600, 255, 254] * 4, 3), 8)


@pytest.mark.parametrize("V", [1023, 1025, 6000])
def test_many_frequent_variants(V):
    rng = np.random.default_rng(V)
    seqs = [[i % 512, i // 512] for i in range(V)]
    note(f"variant paths: {V} variants of 255 cases or more")
    check_variants(*_from_sequences(seqs, rng.integers(255, 262, V), V), 512)


def test_more_than_16384_frequent_variants():
    V = 16400
    seqs = [[i % 512, i // 512] for i in range(V)]
    counts = 255 + (np.arange(V) * 7919 % 5)
    note(f"variant paths: {V} variants of 255 cases or more")
    check_variants(*_from_sequences(seqs, counts, 4), 512)


@pytest.mark.parametrize("n", [1023, 1024, 1025, 2049, 5000])
def test_long_cases(n):
    rng = np.random.default_rng(n)
    base = rng.integers(0, 5, n).tolist()
    other = list(base)
    other[n // 2] ^= 1
    note(f"variant paths: cases of {n} events")
    check_variants(*_from_sequences([base, other, base[:-1], [1]], [3, 2, 2, 70], 5), 6)


def test_no_cases():
    z = torch.zeros(0, dtype=torch.int32, device="cuda:0")
    v = pm4g.pm4g_variants(z, z, z.long(), 3)
    assert int(v["n_variants"].item()) == 0 and int(v["var_off"][0].item()) == 0 and int(v["status"].item()) == 0

"""Identities the kernels rest on, checked on the CPU by brute force.

Nothing here calls the library or the oracle.  The rank formula and the exchange + bitonic
rounds of the kernels for more than 169 rows are statements about sorted sequences, tried on
every 0/1 input of small sizes (comparator networks and min/max formulas that are right on all
0/1 inputs are right on all inputs) and on random integers with many ties at the sizes the
kernels use.  The single pass's rule for the copy that feeds the median, and the condition
under which its output stands, are modelled on small vectors.
"""
import itertools
import os
import sys

import numpy as np
import pytest


def rank_from_halves(A, B):
    """Rank H-1 (0-based) of the union of two ascending sequences of H values each."""
    H = len(A)
    best = min(A[H - 1], B[H - 1])
    for m in range(H - 1):
        best = min(best, max(A[m], B[H - 2 - m]))
    return best


@pytest.mark.parametrize("H", [1, 2, 3, 4, 5, 6, 7])
def test_rank_of_two_sorted_halves_all_zero_one_inputs(H):
    for bits in itertools.product((0, 1), repeat=2 * H):
        A, B = sorted(bits[:H]), sorted(bits[H:])
        assert rank_from_halves(A, B) == sorted(bits)[H - 1], bits


@pytest.mark.parametrize("H", [96, 112, 128])
def test_rank_of_two_sorted_halves_with_spare_wires(H):
    # f values on 2H wires: the spare wires at the end, H-1-(f-1)/2 of them smallest, the rest
    # largest, put the median of the f values at rank H-1
    rng = np.random.default_rng(H)
    for f in (H + 1, H + 2, 2 * H - 3, 2 * H - 1):
        if f % 2 == 0:
            f += 1
        for _ in range(200):
            v = rng.integers(1, 9, size=f).tolist()
            low = H - 1 - (f - 1) // 2
            wires = v + [0] * low + [10 ** 6] * (2 * H - f - low)
            A, B = sorted(wires[:H]), sorted(wires[H:])
            assert rank_from_halves(A, B) == sorted(v)[(f - 1) // 2], (H, f)


def bitonic_rounds(k):
    P = len(k)
    apart = P // 2
    while apart >= 1:
        for i in range(P):
            if (i & apart) == 0 and k[i] > k[i + apart]:
                k[i], k[i + apart] = k[i + apart], k[i]
        apart //= 2
    return k


def split_and_sort(A, B, P):
    """What the two waves do after sorting their halves A and B of H values: minima and maxima of
    A[m] against B[H-1-m], each padded to P wires and run through the bitonic rounds."""
    H = len(A)
    lo = [min(A[m], B[H - 1 - m]) for m in range(H)]          # rises, then falls
    hi = [0] * H
    for m in range(H):
        hi[H - 1 - m] = max(A[m], B[H - 1 - m])               # falls, then rises
    lo_sorted = bitonic_rounds([-1] * (P - H) + lo)[P - H:]    # smallest key in front
    hi_sorted = bitonic_rounds(hi + [10 ** 9] * (P - H))[:H]   # largest key behind
    return lo_sorted + hi_sorted


@pytest.mark.parametrize("H,P", [(1, 1), (2, 2), (3, 4), (4, 4), (5, 8), (6, 8), (7, 8), (8, 8)])
def test_exchange_and_bitonic_rounds_sort_all_zero_one_inputs(H, P):
    for bits in itertools.product((0, 1), repeat=2 * H):
        A, B = sorted(bits[:H]), sorted(bits[H:])
        assert split_and_sort(A, B, P) == sorted(bits), bits


@pytest.mark.parametrize("H", [96, 112, 128])
def test_exchange_and_bitonic_rounds_sort_at_the_kernels_sizes(H):
    rng = np.random.default_rng(1000 + H)
    for _ in range(60):
        v = rng.integers(0, 12, size=2 * H).tolist()
        assert split_and_sort(sorted(v[:H]), sorted(v[H:]), 128) == sorted(v)


def _single_pass_model(copies, wave):
    """The single pass's choice of the copy that feeds the median, modelled on small vectors:
    per stretch of `wave` coordinates the first copy of the largest class of copies identical on
    that stretch feeds; `differs[b]` says whether some stretch fed a copy that differed from copy
    b there.  -> (fed vector, differs, winner by plurality with the lowest index on ties)."""
    r, n = copies.shape
    fed = np.zeros(n, dtype=copies.dtype)
    differs = [False] * r
    for c0 in range(0, n, wave):
        seg = copies[:, c0:c0 + wave]
        same = [[bool((seg[a] == seg[b]).all()) for b in range(r)] for a in range(r)]
        sizes = [sum(row) for row in same]
        pick = sizes.index(max(sizes))
        fed[c0:c0 + wave] = seg[pick]
        for b in range(r):
            differs[b] = differs[b] or not same[pick][b]
    same_all = [[bool((copies[a] == copies[b]).all()) for b in range(r)] for a in range(r)]
    counts = [sum(row) for row in same_all]
    winner = counts.index(max(counts))
    return fed, differs, winner, counts[winner]


@pytest.mark.parametrize("r", [3, 5, 7])
def test_wave_local_choice_feeds_the_winner_or_says_so(r):
    # (1) if no stretch fed a copy that differed from the winner there, the fed vector is the
    # winner's; (2) a winner with a strict majority of the copies is never differed from
    rng = np.random.default_rng(r)
    stood = redone = 0
    for _ in range(6000):
        n, wave = 12, 4
        n_kinds = int(rng.integers(1, r + 1))
        kinds = rng.integers(0, 2, size=(n_kinds, n))
        # kinds that agree on most stretches: start from one vector, change a few words
        kinds[1:] = kinds[0]
        for k in range(1, n_kinds):
            for c in rng.integers(0, n, size=int(rng.integers(1, 3))):
                kinds[k, c] = rng.integers(2, 5)
        copies = kinds[rng.integers(0, n_kinds, size=r)]
        fed, differs, winner, count = _single_pass_model(copies, wave)
        if not differs[winner]:
            assert (fed == copies[winner]).all()
            stood += 1
        else:
            redone += 1
        if 2 * count > r:
            assert not differs[winner]
    assert stood > 0 and redone > 0


# ------------------------------------------------------------------- three-way merge

sys.path.insert(0, os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                                "paper_2010_04902_amd", "csrc"))
import gen_selnet  # noqa: E402


@pytest.mark.parametrize("sizes", [(1, 1, 1), (2, 1, 1), (3, 3, 3), (4, 3, 2), (5, 5, 1), (7, 6, 6),
                                   (9, 9, 7), (9, 9, 9), (13, 4, 2), (27, 11, 11), (27, 27, 27)])
def test_three_way_merge_all_zero_one_inputs(sizes):
    # a merge is right iff it is right on sorted 0/1 lists, i.e. for every number of zeros in each;
    # every block order too, because the merge numbers its lists by length
    for order in sorted(set(itertools.permutations(sizes))):
        starts = [sum(order[:k]) for k in range(3)]
        sorters = []
        out = gen_selnet.merge_three(sorters, *[list(range(s, s + m)) for s, m in zip(starts, order)])
        assert out == list(range(sum(sizes)))
        zeros = np.array(list(itertools.product(*[range(m + 1) for m in order])))
        v = np.concatenate([(np.arange(m)[None, :] >= zeros[:, k:k + 1]) for k, m in enumerate(order)],
                           axis=1).astype(np.uint8)
        for wires in sorters:
            v[:, list(wires)] = np.sort(v[:, list(wires)], axis=1)
        assert np.array_equal(v, np.sort(v, axis=1)), order


def _merges_in_use():
    """Sizes of the blocks of every merge that the generated networks are made of."""
    merges = set()

    def descend(sizes):
        if len(sizes) > 1 and tuple(sizes) not in merges:
            merges.add(tuple(sizes))
            for m in sizes:
                descend(gen_selnet.best_split(m)[1])

    for f in set(gen_selnet.SIZES) | set(gen_selnet.STREAMED_SIZES):
        descend(gen_selnet.median_blocks(f))
    for f in gen_selnet.SORT_SIZES:
        descend(gen_selnet.best_split(f)[1])
    return sorted(merges, key=lambda m: (sum(m), m))


@pytest.mark.parametrize("sizes", _merges_in_use(), ids=str)
def test_every_merge_of_the_generated_networks_on_all_zero_one_inputs(sizes):
    # with sorted blocks merged rightly at every level the whole network sorts
    starts = [sum(sizes[:k]) for k in range(len(sizes))]
    sorters = []
    out = gen_selnet.merge_blocks(sorters, [list(range(s, s + m)) for s, m in zip(starts, sizes)])
    assert out == list(range(sum(sizes)))
    zeros = np.array(list(itertools.product(*[range(m + 1) for m in sizes])))
    v = [(i >= zeros[:, k]).astype(np.uint8) for k, m in enumerate(sizes) for i in range(m)]
    for wires in sorters:
        if len(wires) == 2:
            (a, b), x = wires, [v[w] for w in wires]
            v[a], v[b] = x[0] & x[1], x[0] | x[1]
        else:
            (a, b, c), x = wires, [v[w] for w in wires]
            v[a], v[b], v[c] = x[0] & x[1] & x[2], (x[0] & x[1]) | (x[2] & (x[0] | x[1])), x[0] | x[1] | x[2]
    total = sum(sizes) - zeros.sum(axis=1)  # ones
    for i in range(sum(sizes)):
        assert np.array_equal(v[i], (i >= sum(sizes) - total).astype(np.uint8)), i


def test_sorters_and_their_comparators_agree():
    # the comparators of a three-wire sorter give the outputs that are needed, for every subset
    for mask in range(1, 8):
        outputs = (bool(mask & 1), bool(mask & 2), bool(mask & 4))
        for values in itertools.product(range(3), repeat=3):
            got = gen_selnet.apply_network(gen_selnet.comparators((0, 1, 2), outputs), values)
            for w in range(3):
                assert not outputs[w] or got[w] == sorted(values)[w], (outputs, values)


@pytest.mark.parametrize("full_sort,sizes", [(False, gen_selnet.STREAMED_SIZES),
                                             (True, gen_selnet.SORT_SIZES)])
def test_every_changed_wire_is_pinned_before_the_next_file(full_sort, sizes):
    for f in sizes:
        most = gen_selnet.SORTERS_BETWEEN_PINS.get(f) if full_sort else None
        changed, run, longest, total = set(), 0, 0, 0
        for step in gen_selnet.streamed_sorters(f, full_sort):
            if step[0] == "sort":
                run += 1
                total += 1
                longest = max(longest, run)
                changed |= {w for w, needed in zip(step[1], step[2]) if needed}
            elif step[0] == "pin":
                assert step[1] in changed, (f, step)
                changed.remove(step[1])
                if not changed:
                    run = 0
            else:  # the next file's share, or the end
                assert not changed, (f, step, changed)
                run = 0
        assert total == len(gen_selnet.sorters_for(f, full_sort)), f
        assert longest == most if most else longest > 0, (f, longest)

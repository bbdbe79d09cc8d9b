"""GPU parity: the HIP path through the C-ABI against the CPU oracle, bit for bit.

Vote and odd-count median are pure selection, so the bar is exact equality of every output
word (winner indices, pair bits, median bit patterns).
"""
import itertools
import math

import numpy as np
import pytest
import torch

import paper_2010_04902_amd as B
import synth
from oracle import byz_oracle as O
from oracle import c_oracle as C
from tests import workloads as W

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
MOLS, RAM, FRC = B.BYZ_SCHEME_MOLS, B.BYZ_SCHEME_RAMANUJAN, B.BYZ_SCHEME_FRC

REVERSED = {"kind": "reversed", "c": 100.0}
ALIE = {"kind": "alie", "z": 1.0}
CONST = {"kind": "constant", "value": 1e3}
MIXED = {"kind": "mixed", "z": 1.0, "value": 1e3, "file_scales": True}


SINGLE, REDONE, REVOTED, TWO_STEP = (B.BYZ_PATH_SINGLE_PASS, B.BYZ_PATH_MEDIAN_REDONE,
                                     B.BYZ_PATH_REVOTED, B.BYZ_PATH_TWO_STEP)


def _check_all(X, rows_np, d, f, r, expect_path=None, tag=""):
    """Runs vote, median-on-winners and aggregate on the GPU and compares with the oracle."""
    Xh = X.detach().cpu().numpy()
    rows_dev = torch.tensor(rows_np.reshape(-1), dtype=torch.int32, device=DEV)
    wrep_o, wrow_o, neq_o = C.vote(Xh, rows_np, d)
    out_o = C.median(Xh, wrow_o, d)

    wrep, wrow, neq = B.byz_vote(X, d, rows_dev, f, r)
    torch.cuda.synchronize()
    assert np.array_equal(wrep.cpu().numpy(), wrep_o), tag
    assert np.array_equal(wrow.cpu().numpy(), wrow_o), tag
    assert np.array_equal(W.bits(neq), neq_o), tag

    out_m = B.byz_median(X, d, wrow)
    torch.cuda.synchronize()
    assert np.array_equal(W.bits(out_m), W.bits(out_o)), tag

    for flags in (B.BYZ_AGG_EARLY_MAJORITY, 0):
        out, wrep2, ws = B.byz_aggregate_opts(X, d, rows_dev, f, r, flags)
        torch.cuda.synchronize()
        assert np.array_equal(W.bits(out), W.bits(out_o)), (tag, flags)
        assert np.array_equal(wrep2.cpu().numpy(), wrep_o), (tag, flags)
        path = B.byz_aggregate_path(ws)
        if flags == 0:
            # without early-majority mode the copies are never compared a second time
            assert path in (SINGLE, REDONE, TWO_STEP), (tag, path)
            if expect_path is not None:
                assert path == expect_path, (tag, path)
        else:
            assert path in (SINGLE, REDONE, REVOTED, REDONE | REVOTED, TWO_STEP), (tag, path)
    out, wrep2, ws = B.byz_aggregate(X, d, rows_dev, f, r)
    torch.cuda.synchronize()
    assert np.array_equal(W.bits(out), W.bits(out_o)), tag
    assert np.array_equal(wrep2.cpu().numpy(), wrep_o), tag
    # trimmed mean in the single pass: same bits as vote followed by byz_trimmed_mean (both
    # follow one rounding contract; byz_trimmed_mean itself is checked against the fp64 oracle)
    trim = min(2, (f - 1) // 2)
    out_t2 = B.byz_trimmed_mean(X, d, wrow, trim)
    for flags in (B.BYZ_AGG_TRIM(trim), B.BYZ_AGG_TRIM(trim) | B.BYZ_AGG_EARLY_MAJORITY):
        out_t, wrep3, _ = B.byz_aggregate_opts(X, d, rows_dev, f, r, flags)
        torch.cuda.synchronize()
        assert np.array_equal(W.bits(out_t), W.bits(out_t2)), (tag, flags)
        assert np.array_equal(wrep3.cpu().numpy(), wrep_o), (tag, flags)
        # ... and, on its own account, within the rounding contract's bound of the fp64 oracle's
        # trimmed mean of the oracle's winners
        _assert_trimmed_mean_close(out_t, Xh, wrow_o, d, trim, (tag, flags))
    return out_o, wrep_o, path


SMALL_D = [1, 2, 3, 5, 63, 64, 255, 1000, 4099, 70001]


@pytest.mark.parametrize("scheme,a,b,q,attack", [
    (MOLS, 5, 3, 3, REVERSED), (MOLS, 5, 3, 4, ALIE), (MOLS, 7, 3, 5, REVERSED),
    (RAM, 5, 5, 6, MIXED), (MOLS, 7, 3, 6, ALIE), (RAM, 3, 3, 2, CONST), (MOLS, 7, 5, 5, MIXED),
    (RAM, 5, 3, 3, CONST), (FRC, 15, 3, 4, REVERSED), (FRC, 25, 5, 7, MIXED),
    # Ramanujan Case 2 (m > s): f = m*s = 15, 21, 35
    (RAM, 3, 5, 2, CONST), (RAM, 3, 7, 2, ALIE), (RAM, 5, 7, 6, MIXED),
    # r = 7 and r = 5 with f > 64 (Sec. 4.2.1, Eq. 6, Case 2): (K,f,l,r) = (49,49,7,7), (49,63,9,7),
    # (25,65,13,5)
    (RAM, 7, 7, 5, MIXED), (RAM, 7, 9, 4, ALIE), (RAM, 5, 13, 4, REVERSED)])
def test_small_sizes_all_layouts(scheme, a, b, q, attack):
    # sizes below one tile, several tiles and ragged tails; row pitches that give 16-byte,
    # 8-byte and 4-byte aligned rows
    for i, d in enumerate(SMALL_D):
        for ld in sorted({d, d + (-d) % 2, synth.padded_ld(d, 4), synth.padded_ld(d, 64)}):
            w = W.make(scheme, a, b, q, d, attack, seed=100 + i, ld=ld, device=DEV)
            out_o, wrep_o, _ = _check_all(w.X, w.file_rows, d, w.f, w.r, tag=(d, ld))


def test_all_honest_reproduces_the_honest_median():
    w = W.make(MOLS, 5, 3, 0, 5000, REVERSED, seed=1, device=DEV)
    out_o, wrep_o, _ = _check_all(w.X, w.file_rows, w.d, w.f, w.r, expect_path=SINGLE)
    assert (wrep_o == 0).all()
    honest = np.median(w.G.cpu().numpy(), axis=0)
    assert np.array_equal(W.bits(out_o), W.bits(honest))


def test_unaligned_base_pointer():
    # a view that starts 4 bytes into an allocation: only dword alignment is guaranteed
    w = W.make(MOLS, 5, 3, 4, 3001, ALIE, seed=2, device=DEV)
    R, ld = w.X.shape
    buf = torch.empty(R * ld + 1, dtype=torch.float32, device=DEV)
    Xs = buf[1:].view(R, ld)
    Xs.copy_(w.X)
    assert Xs.data_ptr() % 8 == 4
    _check_all(Xs, w.file_rows, w.d, w.f, w.r, expect_path=SINGLE)


def test_generic_shapes_without_a_generated_network():
    # f = 27 (Ramanujan s=3, m=9) and f = 33 (s=3, m=11): no single pass; vote kernel, then the
    # median on the next generated network with spare wires
    for (a, b, q) in [(3, 9, 2), (3, 11, 2)]:
        w = W.make(RAM, a, b, q, 2222, CONST, seed=3, device=DEV)
        assert not B.byz_aggregate_has_single_pass(w.f, w.r)
        _check_all(w.X, w.file_rows, w.d, w.f, w.r, expect_path=TWO_STEP)
    # byz_median alone for assorted odd f, including rows used more than once
    rng = np.random.default_rng(5)
    X = torch.randn(70, 1500, device=DEV)
    for f in [1, 3, 5, 7, 9, 11, 13, 15, 21, 25, 31, 35, 49, 63]:
        idx = rng.integers(0, 70, size=f).astype(np.int32)
        out = B.byz_median(X, 1500, torch.tensor(idx, device=DEV))
        torch.cuda.synchronize()
        assert np.array_equal(W.bits(out), W.bits(O.median(X.cpu().numpy(), idx, 1500)))


def _plant(X, rows_np, j, k, coords, value):
    for c in coords:
        X[int(rows_np[j, k]), c] = value


def test_copy_that_matches_on_the_probe_sample_but_differs_elsewhere():
    # The streaming pass compares every pair of copies everywhere, and each wave feeds the median
    # from a copy of the class that is largest on its own coordinates.  So a changed word costs
    # nothing while its file keeps a strict majority, whichever copy it is in; only a file
    # without one can make the pass feed values of a copy that loses the vote, and then the
    # median over the winners is redone.  The copies are never compared again.  The changed
    # words sit off the 16 runs of 16 coordinates that early-majority mode's probe samples.
    d = 100_000
    w = W.make(MOLS, 5, 3, 0, d, REVERSED, seed=4, device=DEV)
    stride = (d - 16) // 15  # start of run u is u * stride
    unsampled = [c for c in (17, stride - 1, d - 17, d // 2 + 19) if (c % stride) >= 16]
    assert unsampled
    # one changed word in replica 1 or 2 (first, middle, last coordinate region): the true
    # classes {0,2},{1} resp. {0,1},{2} are known after the pass, replica 0 fed the network
    # everywhere and is the winner -> no further pass
    for k, c in [(1, unsampled[0]), (2, unsampled[1]), (1, d - 1), (2, d // 2 + 19)]:
        X1 = w.X.clone()
        _plant(X1, w.file_rows, 5, k, [c], 9.0)
        out_o, wrep_o, _ = _check_all(X1, w.file_rows, d, w.f, w.r, expect_path=SINGLE, tag=(k, c))
        assert wrep_o[5] == 0
    # one changed word in replica 0: classes {0},{1,2}, winner replica 1.
    # The wave that holds the word feeds from replica 1 there, the others from replica 0, which
    # equals the winner on their coordinates -> the output stands
    X2 = w.X.clone()
    _plant(X2, w.file_rows, 8, 0, unsampled[:1], -3.0)
    out_o, wrep_o, _ = _check_all(X2, w.file_rows, d, w.f, w.r, expect_path=SINGLE)
    assert wrep_o[8] == 1
    # no majority: replicas 1 and 2 carry the same false vector except for one word off the
    # sample.  The three copies are distinct, replica 0 wins the tie (Sec. 2), but nearly every
    # wave saw {1,2} as the largest class and fed their values -> median redone.  With the
    # false vectors in replicas 0 and 1 instead, replica 0 both wins and is what the waves fed.
    for pair, want, winner in [((1, 2), REDONE, 0), ((0, 1), SINGLE, 0)]:
        Xs = w.X.clone()
        for k in pair:
            Xs[int(w.file_rows[8, k])] = -50.0 * w.G[8]
        _plant(Xs, w.file_rows, 8, pair[1], unsampled[:1], -3.0)
        out_o, wrep_o, _ = _check_all(Xs, w.file_rows, d, w.f, w.r, expect_path=want, tag=pair)
        assert wrep_o[8] == winner
    # early-majority mode reads replicas 0 and 1 of such a file: a changed word in replica 2 is
    # never seen (and cannot matter); in replica 1 it makes the two copies differ, all three
    # copies of that one file are compared, replica 0 turns out to be the winner and is what
    # the wave with the word fed (first of two unequal copies): no median; in replica 0 the
    # winner is replica 1, that wave fed replica 0, and the median is redone as well.
    # (_check_all has compared the outputs above.)
    rows_dev = torch.tensor(w.file_rows.reshape(-1), dtype=torch.int32, device=DEV)
    for k, want in [(2, SINGLE), (1, REVOTED), (0, REVOTED | REDONE)]:
        Xe = w.X.clone()
        _plant(Xe, w.file_rows, 8, k, unsampled[:1], -3.0)
        _, _, ws = B.byz_aggregate_opts(Xe, d, rows_dev, w.f, w.r, B.BYZ_AGG_EARLY_MAJORITY)
        torch.cuda.synchronize()
        assert B.byz_aggregate_path(ws) == want, (k, want)
    # replicas 0 and 2 of file 3 both deviate (identically) in a few words: the true classes are
    # {0,2},{1}, and replica 0, which every wave fed, is a winner
    X3 = w.X.clone()
    for k in (0, 2):
        _plant(X3, w.file_rows, 3, k, unsampled, 7.0)
    out_o, wrep_o, _ = _check_all(X3, w.file_rows, d, w.f, w.r, expect_path=SINGLE)
    assert wrep_o[3] == 0
    # replicas 0 and 2 deviate differently: three distinct copies, replica 0 wins the tie and
    # is what every wave fed (first of the largest class everywhere)
    X4 = X3.clone()
    _plant(X4, w.file_rows, 3, 2, unsampled[:1], 8.0)
    out_o, wrep_o, _ = _check_all(X4, w.file_rows, d, w.f, w.r, expect_path=SINGLE)
    assert wrep_o[3] == 0
    # replica 0 differs at one coordinate that early-majority mode's probe samples
    X5 = w.X.clone()
    _plant(X5, w.file_rows, 5, 0, [5 * stride + 3], 9.0)
    out_o, wrep_o, _ = _check_all(X5, w.file_rows, d, w.f, w.r, expect_path=SINGLE)
    assert wrep_o[5] == 1
    # r = 5: replica 0 of a file has a changed word while two Byzantine copies agree
    # with each other: 1 + 2 + 2 -> the lowest honest replica left wins; the wave with the word
    # sees {1,2} first among the classes of two and feeds replica 1, the others feed replica 0,
    # which equals it there
    w5 = W.make(RAM, 5, 5, 0, d, REVERSED, seed=5, device=DEV)
    Y = w5.X.clone()
    _plant(Y, w5.file_rows, 6, 0, unsampled[:1], 5.0)
    for k in (3, 4):
        Y[int(w5.file_rows[6, k])] = -100.0 * w5.G[6]
    out_o, wrep_o, _ = _check_all(Y, w5.file_rows, d, w5.f, w5.r, expect_path=SINGLE)
    assert wrep_o[6] == 1
    # 1 + 2 + 2 the other way round: replicas 0 and 1 false and equal, 2 honest with a word of
    # its own, 3 and 4 honest: classes {0,1},{2},{3,4}, replica 0 wins the tie; the waves fed
    # the honest copies, which are three of five wherever the word is not -> median redone
    Y3 = w5.X.clone()
    for k in (0, 1):
        Y3[int(w5.file_rows[6, k])] = -100.0 * w5.G[6]
    _plant(Y3, w5.file_rows, 6, 2, unsampled[:1], 5.0)
    out_o, wrep_o, _ = _check_all(Y3, w5.file_rows, d, w5.f, w5.r, expect_path=REDONE)
    assert wrep_o[6] == 0
    # the same with the off-sample word in replica 2 instead: nothing to redo
    Y2 = w5.X.clone()
    _plant(Y2, w5.file_rows, 6, 2, unsampled[:1], 5.0)
    for k in (3, 4):
        Y2[int(w5.file_rows[6, k])] = -100.0 * w5.G[6]
    out_o, wrep_o, _ = _check_all(Y2, w5.file_rows, d, w5.f, w5.r, expect_path=SINGLE)
    assert wrep_o[6] == 0


def test_no_majority_and_ties():
    d = 3000
    # r = 3, all three copies different -> replica 0 wins
    w = W.make(MOLS, 5, 3, 0, d, REVERSED, seed=6, device=DEV)
    X = w.X.clone()
    X[int(w.file_rows[4, 1])] *= 2.0
    X[int(w.file_rows[4, 2])] *= 3.0
    out_o, wrep_o, _ = _check_all(X, w.file_rows, d, w.f, w.r)
    assert wrep_o[4] == 0
    # r = 5: every equality pattern of five copies on one file each (52 set partitions > 25
    # files, so three rounds), values differing everywhere
    w5 = W.make(RAM, 5, 5, 0, d, REVERSED, seed=7, device=DEV)

    def partitions(n):
        def rec(prefix, mx):
            if len(prefix) == n:
                yield list(prefix)
                return
            for lab in range(mx + 2):
                yield from rec(prefix + [lab], max(mx, lab))
        return list(rec([0], 0))
    parts = partitions(5)
    assert len(parts) == 52
    for start in range(0, 52, 25):
        X = w5.X.clone()
        chunk = parts[start:start + 25]
        for j, labels in enumerate(chunk):
            for k, lab in enumerate(labels):
                X[int(w5.file_rows[j, k])] = w5.G[j] * float(1 + lab)
        out_o, wrep_o, _ = _check_all(X, w5.file_rows, d, w5.f, w5.r, tag=start)
        for j, labels in enumerate(chunk):
            counts = [labels.count(x) for x in labels]
            assert wrep_o[j] == counts.index(max(counts))


def test_special_values_nan_inf_signed_zero():
    d = 4096
    w = W.make(MOLS, 5, 3, 4, d, ALIE, seed=8, device=DEV)
    X = w.X.clone()
    Xi = X.view(torch.int32)
    rng = np.random.default_rng(9)
    patterns = np.array([0x7FC00000, 0xFFC00000, 0x7F800000, 0xFF800000, 0x80000000, 0x00000000,
                         0x7FC00001, 0x00000001, 0x80000001], dtype=np.uint32).view(np.int32)
    # honest copies stay bitwise identical: write the same special word into all honest copies
    for _ in range(600):
        j = int(rng.integers(0, w.f))
        c = int(rng.integers(0, d))
        p = int(patterns[rng.integers(0, len(patterns))])
        for k in range(w.r):
            if int(w.file_workers[j, k]) not in w.byz:
                Xi[int(w.file_rows[j, k]), c] = p
    # a column where most files hold a NaN / zeros of both signs
    for j in range(w.f):
        for k in range(w.r):
            Xi[int(w.file_rows[j, k]), 11] = int(patterns[j % 2])
            Xi[int(w.file_rows[j, k]), 12] = int(patterns[4 + (j % 2)])
    _check_all(X, w.file_rows, d, w.f, w.r)
    # raw random bit patterns, each file's copies identical
    U = torch.randint(-2**31, 2**31 - 1, (w.f, d), dtype=torch.int64, device=DEV).to(torch.int32)
    Xr = torch.empty_like(X).view(torch.int32)
    for j in range(w.f):
        for k in range(w.r):
            Xr[int(w.file_rows[j, k])] = U[j]
    _check_all(Xr.view(torch.float32), w.file_rows, d, w.f, w.r, expect_path=SINGLE)


def test_argument_errors():
    w = W.make(MOLS, 5, 3, 3, 100, REVERSED, seed=10, device=DEV)
    rows_dev = torch.tensor(w.file_rows.reshape(-1), dtype=torch.int32, device=DEV)
    # the library rejects these before any launch; the row table is long enough for each so
    # that the binding's own length check does not fire first
    rows_long = torch.zeros(257 * 9, dtype=torch.int32, device=DEV)
    for (f, r, code) in [(25, 4, -1), (25, 1, -1), (0, 3, -1), (257, 3, -1), (25, 9, -1)]:
        with pytest.raises(B.ByzError) as e:
            B.byz_vote(w.X, 100, rows_long, f, r)
        assert e.value.code == code
    with pytest.raises(ValueError):
        B.byz_vote(w.X, 100, rows_dev, 65, 3)  # 75-entry table, the call would read 195
    with pytest.raises(ValueError):
        B.byz_aggregate(w.X, 100, rows_dev, 81, 3)
    with pytest.raises(B.ByzError) as e:
        B.byz_vote(w.X, 101, rows_dev, 25, 3)  # d > ld
    assert e.value.code == -1
    with pytest.raises(B.ByzError) as e:
        B.byz_median(w.X, 100, rows_dev[:24])  # even f
    assert e.value.code == -2
    for bad in (4, 0x100, B.BYZ_AGG_TRIM(13)):  # unknown bit, b without the flag, 2b >= f
        with pytest.raises(B.ByzError) as e:
            B.byz_aggregate_opts(w.X, 100, rows_dev, 25, 3, bad)
        assert e.value.code == -1
    small = torch.empty(64, dtype=torch.uint8, device=DEV)
    with pytest.raises(B.ByzError) as e:
        B.byz_aggregate(w.X, 100, rows_dev, 25, 3, workspace=small)
    assert e.value.code == -3
    # d = 0: every copy is trivially equal
    wrep, wrow, neq = B.byz_vote(w.X, 0, rows_dev, 25, 3)
    torch.cuda.synchronize()
    assert (wrep == 0).all() and (neq == 0).all()
    out, wrep2, _ = B.byz_aggregate(w.X, 0, rows_dev, 25, 3)
    torch.cuda.synchronize()
    assert out.numel() == 0 and (wrep2 == 0).all()


@pytest.mark.parametrize("scheme,a,b,q", [(MOLS, 5, 3, 4), (MOLS, 7, 3, 5), (RAM, 5, 5, 6)])
def test_probe_sample_shift(scheme, a, b, q):
    # BYZ_AGG_PROBE_SHIFT moves the coordinates the single pass samples first: the output and
    # the winners never change; for which inputs byz_aggregate has to redo the median does
    d = 70_001
    w = W.make(scheme, a, b, q, d, ALIE, seed=77, ld=synth.padded_ld(d, 4), device=DEV)
    rows_dev = torch.tensor(w.file_rows.reshape(-1), dtype=torch.int32, device=DEV)
    Xh = w.X.cpu().numpy()
    wrep_o, wrow_o, _ = C.vote(Xh, w.file_rows, d)
    out_o = C.median(Xh, wrow_o, d)
    shifts = (0, 1, 2, 7, 255, 12345, 40000, 65535)
    for s in shifts:
        for extra in (0, B.BYZ_AGG_EARLY_MAJORITY):
            out, wrep, ws = B.byz_aggregate_opts(w.X, d, rows_dev, w.f, w.r, B.BYZ_AGG_PROBE_SHIFT(s) | extra)
            torch.cuda.synchronize()
            assert np.array_equal(W.bits(out), W.bits(out_o)), (s, extra)
            assert np.array_equal(wrep.cpu().numpy(), wrep_o), (s, extra)
            assert B.byz_aggregate_path(ws) == SINGLE, (s, extra)
    # One honest copy differs in a single word.  With shift 0 that word is one of the sampled
    # ones (run 3, word 5 of the 16 runs (d - 16) / 15 apart), other shifts sample elsewhere.
    # Nothing depends on that, nor on which copy it is: the file keeps a majority of two, every
    # wave feeds a copy that equals it on the wave's coordinates, and the output stands.
    clean = [j for j in range(w.f) if not any(int(x) in w.byz for x in w.file_workers[j])]
    c_star = 3 * ((d - 16) // 15) + 5
    for k in (1, 0):
        P = w.X.clone()
        P[int(w.file_rows[clean[0], k]), c_star] += 1.0
        Ph = P.cpu().numpy()
        wrep_p, wrow_p, neq_p = C.vote(Ph, w.file_rows, d)
        out_p = C.median(Ph, wrow_p, d)
        assert neq_p[clean[0]] != 0 and wrep_p[clean[0]] == (1 if k == 0 else 0)
        for s in shifts:
            out, wrep, ws = B.byz_aggregate_opts(P, d, rows_dev, w.f, w.r, B.BYZ_AGG_PROBE_SHIFT(s))
            torch.cuda.synchronize()
            assert np.array_equal(W.bits(out), W.bits(out_p)), s
            assert np.array_equal(wrep.cpu().numpy(), wrep_p), s
            assert B.byz_aggregate_path(ws) == SINGLE, (k, s)


def test_generator_same_bytes_on_cpu_and_gpu():
    for fs in (False, True):
        Gc = synth.honest_gradients(9, 5000, 77, step=3, device="cpu", file_scales=fs)
        Gg = synth.honest_gradients(9, 5000, 77, step=3, device=DEV, file_scales=fs)
        assert np.array_equal(W.bits(Gc), W.bits(Gg))
    assert np.array_equal(W.bits(synth.alie_vector(Gc, 1.5)), W.bits(synth.alie_vector(Gg, 1.5)))


def test_largest_shapes_f63_r7():
    # Ramanujan s=7, m=9 (Case 2): K=49 workers, f=63 files, r=7 (largest r), l=9: 21 pair bits
    # per file, seven copies of a file in flight in the single pass
    w = W.make(RAM, 7, 9, 6, 1537, MIXED, seed=12, device=DEV)
    assert (w.K, w.f, w.l, w.r) == (49, 63, 9, 7) and B.byz_aggregate_has_single_pass(63, 7)
    _check_all(w.X, w.file_rows, w.d, w.f, w.r, expect_path=SINGLE)
    # every copy of one file different (seven singletons), 3-3-1 and 2-2-2-1 splits on others
    X = w.X.clone()
    for j, labels in enumerate([[0, 1, 2, 3, 4, 5, 6], [1, 0, 1, 0, 1, 0, 2], [0, 0, 1, 1, 2, 2, 3],
                                [3, 2, 2, 1, 1, 1, 0]]):
        for k, lab in enumerate(labels):
            X[int(w.file_rows[j, k])] = w.G[j] * float(1 + lab)
    out_o, wrep_o, _ = _check_all(X, w.file_rows, w.d, w.f, w.r, expect_path=SINGLE)
    assert wrep_o[:4].tolist() == [0, 0, 0, 3]
    # the same splits where the copies differ in one word off the probe's sample only: the probe
    # sees seven equal copies; the wave that holds the word sees the true classes and feeds from
    # the first of the largest, which is the winner (file 3: replicas 3, 4, 5 agree); the
    # other waves feed replica 0, which equals the winner on their coordinates -> nothing redone
    X2 = w.X.clone()
    hidden = w.d // 2 + 37
    for j, labels in enumerate([[0, 1, 2, 3, 4, 5, 6], [1, 0, 1, 0, 1, 0, 2], [0, 0, 1, 1, 2, 2, 3],
                                [3, 2, 2, 1, 1, 1, 0]]):
        for k, lab in enumerate(labels):
            X2[int(w.file_rows[j, k])] = w.G[j]
            X2[int(w.file_rows[j, k]), hidden] = float(lab)
    out_o, wrep_o, _ = _check_all(X2, w.file_rows, w.d, w.f, w.r, expect_path=SINGLE)
    assert wrep_o[:4].tolist() == [0, 0, 0, 3]
    # seven distinct copies of file 3, told apart by two words in different waves' ranges: at the
    # first, replica 0 stands alone against six equal copies, so that wave feeds replica 1, but
    # with seven singletons replica 0 wins the tie (Sec. 2) -> median redone
    X3 = w.X.clone()
    far = 11
    for k in range(7):
        X3[int(w.file_rows[3, k])] = w.G[3]
        X3[int(w.file_rows[3, k]), hidden] = float(k > 0)
        X3[int(w.file_rows[3, k]), far] = float(max(0, k - 1))
    out_o, wrep_o, _ = _check_all(X3, w.file_rows, w.d, w.f, w.r, expect_path=REDONE)
    assert wrep_o[3] == 0


def test_hip_graph_capture_and_replay():
    # the entry points enqueue kernels only (no memset, no allocation, no sync), so a caller
    # can capture them; every replay must give the eager result, with eager work in between
    w = W.make(MOLS, 5, 3, 4, 200_003, ALIE, seed=13, ld=200_064, device=DEV)
    rows_dev = torch.tensor(w.file_rows.reshape(-1), dtype=torch.int32, device=DEV)
    out_e, wrep_e, _ = B.byz_aggregate(w.X, w.d, rows_dev, w.f, w.r)
    torch.cuda.synchronize()
    Xs = w.X.clone()  # static input buffer of the graph
    out = torch.empty(w.d, dtype=torch.float32, device=DEV)
    wrep = torch.empty(w.f, dtype=torch.int32, device=DEV)
    ws = torch.empty(B.byz_aggregate_workspace_bytes(w.f, w.r), dtype=torch.uint8, device=DEV)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        B.byz_aggregate(Xs, w.d, rows_dev, w.f, w.r, out=out, winner_replica=wrep, workspace=ws)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.byz_aggregate(Xs, w.d, rows_dev, w.f, w.r, out=out, winner_replica=wrep, workspace=ws)
    # second input: replicas 1 and 2 of a file hold a false vector, equal but for one word off
    # the probe's sample: no majority, replica 0 wins the tie, the waves fed the other two (the
    # median is redone)
    X2 = w.X.clone()
    X2[int(w.file_rows[3, 1]), :w.d] = -50.0 * w.G[3]
    X2[int(w.file_rows[3, 2])] = X2[int(w.file_rows[3, 1])]
    X2[int(w.file_rows[3, 2]), 12345] = 7.0
    out_e2, wrep_e2, ws_e2 = B.byz_aggregate(X2, w.d, rows_dev, w.f, w.r)
    torch.cuda.synchronize()
    for rep, (src, want_out, want_rep) in enumerate([(w.X, out_e, wrep_e), (X2, out_e2, wrep_e2),
                                                     (w.X, out_e, wrep_e), (X2, out_e2, wrep_e2)]):
        Xs.copy_(src)
        out.zero_()
        wrep.fill_(-1)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int32), want_out.view(torch.int32)), rep
        assert torch.equal(wrep, want_rep), rep
        # eager work between replays
        chk, _, _ = B.byz_aggregate(src, w.d, rows_dev, w.f, w.r)
        torch.cuda.synchronize()
        assert torch.equal(chk.view(torch.int32), want_out.view(torch.int32))
    assert wrep_e2[3].item() == 0 and B.byz_aggregate_path(ws_e2) == REDONE


def test_read_rows_reference_kernel():
    # the access-pattern reference kernel XORs the rows it reads; without the store it leaves
    # the output alone
    rng = np.random.default_rng(6)
    for (n_rows, d, ld) in [(1, 4, 4), (5, 1000, 1003), (6, 1027, 1028), (7, 70001, 70004), (75, 5003, 5003)]:
        Xh = rng.integers(0, 2 ** 32, size=(n_rows + 1, ld), dtype=np.uint64).astype(np.uint32)
        X = torch.tensor(Xh.view(np.float32), device=DEV)
        out = torch.full((d,), 7.0, dtype=torch.float32, device=DEV)
        B.byz_calibration_read_rows(X, d, n_rows, out, 0)
        torch.cuda.synchronize()
        assert (out == 7.0).all()
        B.byz_calibration_read_rows(X, d, n_rows, out, 1)
        torch.cuda.synchronize()
        n4 = d // 4 * 4
        want = np.bitwise_xor.reduce(Xh[:n_rows, :n4], axis=0)
        assert np.array_equal(W.bits(out)[:n4], want), (n_rows, d)
        assert (out[n4:] == 7.0).all()
    with pytest.raises(B.ByzError):
        B.byz_calibration_read_rows(X, 3, 1, out, 1)  # d < 4
    with pytest.raises(ValueError):
        B.byz_calibration_read_rows(X, 8, 500, out, 1)  # more rows than the matrix has


def test_measurement_aids():
    src = torch.randn(1 << 20, device=DEV)
    dst = torch.zeros_like(src)
    B.byz_calibration_copy(src, dst)
    torch.cuda.synchronize()
    assert torch.equal(src, dst)
    w = W.make(MOLS, 5, 3, 3, 50_000, REVERSED, seed=14, device=DEV)
    rows_dev = torch.tensor(w.file_rows.reshape(-1), dtype=torch.int32, device=DEV)
    B.byz_profile_enable(2)
    for _ in range(3):
        B.byz_aggregate(w.X, w.d, rows_dev, w.f, w.r)
    ms = B.byz_profile_collect(8)
    B.byz_profile_enable(0)
    assert len(ms) == 2 and all(0 < t < 50 for t in ms)
    assert B.byz_profile_collect(8) == []


def test_profiled_kernel_is_named():
    # the kernel the events stand around: short rows, rows without room for slots, early-majority mode, files
    # split over two waves, vote on its own
    for f, r, d, flags, want in ((25, 3, 5000, 0, "short_pass_kernel"), (25, 3, 1100000, 0, "fused_kernel"),
                                 (25, 3, 5000, B.BYZ_AGG_EARLY_MAJORITY, "fused_kernel"),
                                 (171, 3, 1 << 18, 0, "fused_halves_kernel"), (171, 3, 5000, 0, "vote_pairs_kernel"),
                                 (27, 3, 5000, 0, "vote_pairs_kernel")):
        X = torch.zeros((f * r, d), device=DEV)
        rows = torch.arange(f * r, dtype=torch.int32, device=DEV)
        B.byz_profile_enable(1)
        assert B.byz_profile_kernel() == ""
        B.byz_aggregate_opts(X, d, rows, f, r, flags)
        name, ms = B.byz_profile_kernel(), B.byz_profile_collect(1)
        B.byz_profile_enable(0)
        assert name == want and len(ms) == 1, (f, r, d, flags, name)


def test_profiled_kernel_of_rows_that_one_block_holds():
    # the longest such row and the first that isn't one, by its threads and by the words in all
    for f, r, d, flags, want in ((25, 3, 1003, 0, "one_block_kernel"), (25, 3, 1024, 0, "one_block_kernel"),
                                 (25, 3, 1025, 0, "short_pass_kernel"), (25, 5, 393, 0, "one_block_kernel"),
                                 (25, 5, 394, 0, "short_pass_kernel"),
                                 (25, 3, 655, B.BYZ_AGG_TRIM(2), "one_block_kernel"),
                                 (25, 3, 656, B.BYZ_AGG_TRIM(2), "short_pass_kernel"),
                                 (25, 3, 1003, B.BYZ_AGG_EARLY_MAJORITY, "fused_kernel"),
                                 (35, 5, 64, 0, "short_pass_kernel")):
        X = torch.zeros((f * r, d), device=DEV)
        rows = torch.arange(f * r, dtype=torch.int32, device=DEV)
        B.byz_profile_enable(1)
        assert B.byz_profile_kernel() == ""
        B.byz_aggregate_opts(X, d, rows, f, r, flags)
        name, ms = B.byz_profile_kernel(), B.byz_profile_collect(1)
        B.byz_profile_enable(0)
        assert name == want and len(ms) == 1, (f, r, d, flags, name)


def _assert_trimmed_mean_close(out, Xh, idx_np, d, b, tag):
    """`out` (GPU, fp32) against the fp64 oracle's trimmed mean of the rows idx_np of Xh.

    Tolerance from the arithmetic: n-1 fp32 additions and one division, each with relative
    rounding error u = 2^-24 on partial sums bounded by sum|x|  =>  |err| <= n * u * max|kept|
    (first order; the factor 1.5 covers the second-order terms and the final conversion)."""
    idx_np = np.ascontiguousarray(idx_np, dtype=np.int32)
    want = C.trimmed_mean(Xh, idx_np, d, b)
    f = len(idx_np)
    n = f - 2 * b
    keys = O.order_key(Xh.view(np.uint32)[idx_np][:, :d])
    srt = np.take_along_axis(Xh[idx_np][:, :d], np.argsort(keys, axis=0, kind="stable"), axis=0)
    with np.errstate(invalid="ignore"):
        kept_abs = np.abs(srt[b:f - b].astype(np.float64))
    kept_max = kept_abs.max(axis=0)
    tol = 1.5 * n * 2.0 ** -24 * kept_max + 1e-44
    got = out.cpu().numpy().astype(np.float64)
    finite = np.isfinite(want)
    # where the fp32 partial sums may overflow (sum|x| near FLT_MAX) the contract gives +-inf
    # while the fp64 oracle stays finite: not compared
    no_overflow = kept_abs.sum(axis=0) < 1e38
    ok = finite & no_overflow
    assert (np.abs(got[ok] - want[ok]) <= tol[ok]).all(), tag
    # non-finite results (kept infinities / NaNs) must agree in kind
    assert np.array_equal(np.isnan(got[~finite]), np.isnan(want[~finite])), tag
    assert np.array_equal(got[~finite & ~np.isnan(want)], want[~finite & ~np.isnan(want)]), tag


def _trimmed_mean_check(X, idx_np, d, b, tag):
    """GPU byz_trimmed_mean (fp32, ascending sequential sum) against the fp64 oracle."""
    idx_dev = torch.tensor(idx_np, dtype=torch.int32, device=DEV)
    out = B.byz_trimmed_mean(X, d, idx_dev, b)
    torch.cuda.synchronize()
    _assert_trimmed_mean_close(out, X.detach().cpu().numpy(), idx_np, d, b, tag)
    return out


@pytest.mark.parametrize("scheme,a,b,q,attack", [(MOLS, 5, 3, 4, ALIE), (MOLS, 7, 3, 5, REVERSED),
                                                 (RAM, 3, 3, 2, CONST), (RAM, 3, 5, 2, CONST)])
def test_trimmed_mean_on_the_vote_winners(scheme, a, b, q, attack):
    for i, d in enumerate([1, 3, 4, 5, 257, 4099, 70001]):
        w = W.make(scheme, a, b, q, d, attack, seed=300 + i, ld=synth.padded_ld(d, 4) + 4 * (i % 2),
                   device=DEV)
        rows_dev = torch.tensor(w.file_rows.reshape(-1), dtype=torch.int32, device=DEV)
        _, wrow, _ = B.byz_vote(w.X, d, rows_dev, w.f, w.r)
        torch.cuda.synchronize()
        idx = wrow.cpu().numpy()
        for trim in sorted({0, 1, min(w.cmax, (w.f - 1) // 2), (w.f - 1) // 2}):
            out = _trimmed_mean_check(w.X, idx, d, trim, (d, trim))
            if trim == (w.f - 1) // 2:  # keeps one value: the median itself
                med = B.byz_median(w.X, d, wrow)
                torch.cuda.synchronize()
                assert torch.equal(out, med) or torch.equal(out + 0.0, med + 0.0)
    for bad_b in (-1, (w.f + 1) // 2):
        with pytest.raises(B.ByzError) as e:
            B.byz_trimmed_mean(w.X, w.d, wrow, bad_b)
        assert e.value.code == -1


def test_trimmed_mean_special_values():
    d, f = 2048, 25
    rng = np.random.default_rng(31)
    U = rng.integers(0, 2**32, size=(f, d), dtype=np.uint64).astype(np.uint32)  # raw bit patterns
    X = torch.tensor(U.view(np.int32), device=DEV).view(torch.float32)
    idx = np.arange(f, dtype=np.int32)
    for b in (0, 3, 12):
        _trimmed_mean_check(X, idx, d, b, b)


@pytest.mark.parametrize("scheme,a,b,q,attack", [
    (RAM, 5, 13, 5, MIXED),      # Ramanujan Case 2, f = 65, r = 5: first size past one lane per file
    (MOLS, 9, 3, 4, ALIE),       # F_9: f = 81
    (MOLS, 11, 3, 4, REVERSED),  # f = 121
    (MOLS, 13, 3, 3, CONST),     # F_13: f = 169
    (RAM, 3, 47, 2, ALIE),       # f = 141: the 169-wire network with spare wires
    (RAM, 3, 85, 2, ALIE)])      # f = 255, the largest odd f
def test_more_than_64_files(scheme, a, b, q, attack):
    # pair bits in several 64-file groups; median and trimmed mean on the 81-, 121- and 169-wire
    # register networks, with spare wires where f lies between two sizes, and on the two-wave
    # kernels past 169
    for i, d in enumerate([1, 5, 64, 65, 1000, 4099]):
        ld = d if i % 2 == 0 else synth.padded_ld(d, 4) + 4
        w = W.make(scheme, a, b, q, d, attack, seed=700 + i, ld=ld, device=DEV)
        assert w.f > 64
        out_o, wrep_o, _ = _check_all(w.X, w.file_rows, d, w.f, w.r, tag=(w.f, d))
        idx = np.array([w.file_rows[j, wrep_o[j]] for j in range(w.f)], dtype=np.int32)
        for trim in (0, w.cmax, (w.f - 1) // 2):
            _trimmed_mean_check(w.X, idx, d, trim, (w.f, d, trim))


def test_more_than_64_rows_of_raw_bit_patterns():
    # byz_median / byz_trimmed_mean alone on random words (NaNs, infinities, signed zeros, many
    # equal keys through repeated rows)
    rng = np.random.default_rng(77)
    d = 1500
    U = rng.integers(0, 2**32, size=(300, d), dtype=np.uint64).astype(np.uint32)
    U[:, :200] &= np.uint32(0x80000003)  # few distinct values: ties everywhere
    X = torch.tensor(U.view(np.int32), device=DEV).view(torch.float32)
    # 171 ... 255: the two-wave kernels, every size of their halves at both ends of its range
    for f in (65, 67, 127, 129, 171, 191, 193, 223, 225, 255):
        idx = rng.integers(0, 300, size=f).astype(np.int32)
        out = B.byz_median(X, d, torch.tensor(idx, device=DEV))
        torch.cuda.synchronize()
        assert np.array_equal(W.bits(out), W.bits(C.median(U, idx, d))), f
        for b in (0, 7, (f - 1) // 2):
            _trimmed_mean_check(X, idx, d, b, (f, b))
    for f, b in ((256, 100), (256, 0), (256, 127), (170, 84), (200, 1)):  # even f: trimmed mean only
        idx = rng.integers(0, 300, size=f).astype(np.int32)
        _trimmed_mean_check(X, idx, d, b, (f, b))
    for f in (257, 1000):
        with pytest.raises(B.ByzError) as e:
            B.byz_median(X, d, torch.zeros(f, dtype=torch.int32, device=DEV))
        assert e.value.code == -1


def test_more_than_169_rows_random_sizes():
    # the two-wave kernels (rows split over two waves that sort a half each): random f in
    # 170..256 (every size of the halves, spare wires of both kinds), d from one coordinate to
    # several blocks with ragged tails, row pitches, raw bit patterns with ties and signed zeros
    # as well as normal data; median for odd f, trimmed mean with b = 0, random, largest
    rng = np.random.default_rng(169)
    for case in range(36):
        f = int(rng.integers(170, 257))
        d = int(rng.choice([rng.integers(1, 70), rng.integers(70, 700), rng.integers(700, 9000)]))
        ld = d + int(rng.integers(0, 7))
        n_rows = f + int(rng.integers(0, 40))
        U = rng.integers(0, 2**32, size=(n_rows, ld), dtype=np.uint64).astype(np.uint32)
        if case % 3 == 0:
            U[:, : d // 2] &= np.uint32(0x80000007)
        if case % 3 == 1:
            U = rng.standard_normal((n_rows, ld)).astype(np.float32).view(np.uint32)
        X = torch.tensor(U.view(np.int32), device=DEV).view(torch.float32)
        idx = rng.integers(0, n_rows, size=f).astype(np.int32)
        if f % 2 == 1:
            out = B.byz_median(X, d, torch.tensor(idx, device=DEV))
            torch.cuda.synchronize()
            assert np.array_equal(W.bits(out), W.bits(C.median(U, idx, d))), (case, f, d, ld)
        for b in sorted({0, int(rng.integers(0, (f + 1) // 2)), (f - 1) // 2}):
            _trimmed_mean_check(X, idx, d, b, (case, f, d, ld, b))


@pytest.mark.parametrize("f", [3, 16, 17, 32, 33, 48, 49, 64, 65, 80, 81, 96, 97, 112, 113, 128])
def test_gram_distances_at_tile_edges_and_for_inputs_that_are_not_finite(f):
    # every number of row tiles, one row more or less; d around the 32 coordinates a wave multiplies
    # at a time, the span of a wave and of a block, all within one step of a wave.  Distances
    # against fp64: at most 32 rounded sums of a wave and the waves of a block on top of each other,
    # far from adding up (three times the largest error seen is 40): |err| <= 64 * 2^-24 * (G_ii + G_jj).
    rng = np.random.default_rng(f)
    idx = torch.tensor(rng.permutation(f).astype(np.int32), device=DEV)
    order = idx.cpu().numpy()
    for d in (1, 31, 33, 129, 1026, 20011):
        Xh = np.ascontiguousarray((rng.standard_normal((f, d + 1)) * rng.uniform(0.01, 3, (f, 1))).astype(np.float32))
        X = torch.tensor(Xh, device=DEV)
        _, _, _, dist = B.byz_multi_krum(X, d, idx, 0, 1)
        torch.cuda.synchronize()
        V = Xh[order, :d].astype(np.float64)
        G = V @ V.T
        n = np.diag(G)
        want = np.maximum(n[:, None] + n[None, :] - 2 * G, 0)
        np.fill_diagonal(want, 0)
        assert (np.abs(dist.cpu().numpy() - want) <= 64 * 2.0 ** -24 * (n[:, None] + n[None, :])).all(), (f, d)
    # infinities, NaNs and a value whose square overflows: same kinds as fp64 products of fp32
    # range (the huge value's square is infinite in fp32, its products with 0 are 0)
    for what in (np.inf, -np.inf, np.nan, np.float32(3.4e38)):
        Y = Xh.copy()
        Y[:, 777] = 0.0
        Y[order[1], 777] = what
        _, _, _, dist = B.byz_multi_krum(torch.tensor(Y, device=DEV), d, idx, 0, 1)
        torch.cuda.synchronize()
        got = dist.cpu().numpy()
        W64 = Y[order, :d].astype(np.float64)
        with np.errstate(all="ignore"):
            P = np.array([[np.float32(np.float32(W64[i, 777]) * np.float32(W64[j, 777])) for j in range(f)]
                          for i in range(f)]).astype(np.float64)
            W64[:, 777] = 0
            G = W64 @ W64.T + P
            n = np.diag(G)
            want = n[:, None] + n[None, :] - 2 * G
            want[want < 0] = 0
        np.fill_diagonal(want, 0)
        assert np.array_equal(np.isnan(got), np.isnan(want)), (f, what)
        assert np.array_equal(np.isinf(got), np.isinf(want)), (f, what)
        scale = (n[:, None] + n[None, :])
        ok = np.isfinite(scale)  # the diagonal of the row itself is 0 whatever it holds
        assert (np.abs(got - want)[ok] <= 64 * 2.0 ** -24 * scale[ok]).all(), (f, what)


def _krum_distances(Xh, d, order):
    X = torch.tensor(Xh, device=DEV)
    _, _, _, dist = B.byz_multi_krum(X, d, torch.tensor(order, device=DEV), 0, 1)
    torch.cuda.synchronize()
    return dist.cpu().numpy()


@pytest.mark.parametrize("f", [3, 16, 17, 33, 49, 65, 81, 97, 113, 128])
def test_gram_products_are_rounded_once(f):
    # one coordinate, one row of zeros: the distance from it to row i is the fp32 rounding of the
    # square of row i's value, to the bit, whatever the size of the square (down to subnormal ones)
    rng = np.random.default_rng(f)
    for scale in (1.0, 1e15, 1e-18, 1e-20):
        Xh = ((1 + rng.random((f, 1))) * scale).astype(np.float32)
        Xh[f // 2] = 0.0
        got = _krum_distances(Xh, 1, np.arange(f, dtype=np.int32))[f // 2]
        assert np.array_equal(got, (Xh[:, 0] * Xh[:, 0]).astype(np.float64)), (f, scale)


@pytest.mark.parametrize("f,d", [(9, 300007), (16, 1048601), (3, 1600013), (25, 300007), (33, 140011), (49, 140011),
                                 (65, 140011), (81, 140011), (100, 140011), (128, 140011)])
def test_gram_of_long_rows(f, d):
    # every number of row tiles with two or three steps of a wave one after the other, f <= 16 also
    # with two stretches of 32 coordinates a step, and a ragged end; rows far apart in size, one
    # around 1e-18, row pitch that is no multiple of a cache line and rows on cache lines.
    # |err| <= 2 L 2^-24 (G_ii + G_jj), L = _gram_additions; a stretch left out is 32 / d of that and more.
    rng = np.random.default_rng(f * 1000003 + d)
    order = rng.permutation(f).astype(np.int32)
    for ld in (d + 2, (d + 31) // 32 * 32):
        Xh = rng.standard_normal((f, ld), dtype=np.float32)
        Xh *= rng.uniform(0.01, 3, (f, 1)).astype(np.float32)
        Xh[order[0]] *= np.float32(1e-18)
        got = _krum_distances(Xh, d, order)
        V = torch.tensor(Xh, device=DEV)[torch.tensor(order, device=DEV).long(), :d].double()
        G = (V @ V.T.contiguous()).cpu().numpy()
        n = np.diag(G)
        want = np.maximum(n[:, None] + n[None, :] - 2 * G, 0)
        np.fill_diagonal(want, 0)
        assert (np.abs(got - want) <= 2 * _gram_additions(d) * 2.0 ** -24 * (n[:, None] + n[None, :])).all(), (f, d, ld)
    # an infinity (times the others' zeros a NaN) and a NaN in the last step of a wave
    for what in (np.inf, np.nan):
        Xh[:, d - 5] = 0.0
        Xh[order[1], d - 5] = what
        got = _krum_distances(Xh, d, order)
        assert np.isnan(got[1, [0] + list(range(2, f))]).all(), (f, what)
        rest = np.ix_([0] + list(range(2, f)), [0] + list(range(2, f)))
        assert np.isfinite(got[rest]).all(), (f, what)


@pytest.mark.parametrize("f,d,ld", [(9, 6000001, 6000032), (25, 6000001, 6000032), (33, 6000001, 6000032),
                                    (33, 6000001, 6000001), (65, 3000001, 3000032), (97, 3000001, 3000001)])
def test_gram_of_long_rows_does_not_drift(f, d, ld):
    # the distance from a row of zeros to a row of values between 1 and 2 is that row's sum of squares.
    # Runs of at most 128 products whose roundings go either way: at most 2^-24 sqrt(128) of a run, over
    # sqrt(runs) of them together and as many blocks rounded once, four times that for 2 f rows; one
    # running sum per wave is 1.5 to 4e-8 too low
    X = torch.rand((f, ld), generator=torch.Generator(device=DEV).manual_seed(f), device=DEV) + 1
    X[f // 2] = 0.0
    want = np.array([float((X[j, :d].double() ** 2).sum()) for j in range(f)])
    _, _, _, dist = B.byz_multi_krum(X, d, torch.arange(f, dtype=torch.int32, device=DEV), 0, 1)
    torch.cuda.synchronize()
    got = dist[f // 2].cpu().numpy()
    runs = d / 128
    bound = 4 * 2.0 ** -24 * (math.sqrt(128 / runs) + 1 / math.sqrt(512))
    with np.errstate(invalid="ignore"):
        off = np.delete(np.abs(got / want - 1), f // 2)
    assert off.max() <= bound, (f, d, off.max(), bound)


@pytest.mark.parametrize("f,d", [(3, 31), (16, 4001), (16, 1048601), (25, 140011), (32, 262177), (25, 262177), (33, 50021),
                                 (48, 140011), (49, 50021), (64, 140011), (80, 50021), (96, 140011), (112, 50021),
                                 (128, 50021), (128, 140011), (33, 4194337), (49, 4194337)])
def test_gram_of_whole_numbers_is_exact(f, d):
    # entries -1, 0 and 1: every product and every sum is a whole number below 2^24, so the distances
    # are exact in whatever order they are added, and one coordinate left out or taken twice shows.
    # Rows on cache lines and off them (ordinary loads, blocks in another order, longer stretches a
    # step above 4 M coordinates), the table in reverse order, guard words behind the rows
    order = np.arange(f, dtype=np.int32)[::-1].copy()
    g = torch.Generator(device=DEV).manual_seed(f * 7 + d)
    for ld in ((d + 31) // 32 * 32, (d + 31) // 32 * 32 + 7, (d + 31) // 32 * 32 + 16):
        X = torch.randint(-1, 2, (f, ld), generator=g, device=DEV, dtype=torch.int8).float()
        X[:, d:] = 3.0
        G = torch.zeros((f, f), dtype=torch.float64, device=DEV)
        for c in range(0, d, 1 << 19):
            V = X[:, c:min(d, c + (1 << 19))].flip(0).double()
            G += V @ V.T.contiguous()
        n = G.diagonal()
        want = n[:, None] + n[None, :] - 2 * G
        _, _, _, dist = B.byz_multi_krum(X, d, torch.tensor(order, device=DEV), 0, 1)
        torch.cuda.synchronize()
        assert torch.equal(dist, want), (f, d, ld)
        # a matrix that starts off a cache line
        if d < 300000:
            Y = torch.zeros(f * ld + 1, device=DEV)
            Y[1:] = X.reshape(-1)
            _, _, _, dist = B.byz_multi_krum(Y[1:].reshape(f, ld), d, torch.tensor(order, device=DEV), 0, 1)
            torch.cuda.synchronize()
            assert torch.equal(dist, want), (f, d, ld)


@pytest.mark.parametrize("f", [33, 36, 37, 50, 52, 53, 56, 57, 68, 69, 84, 85, 100, 104, 105, 108, 109, 116, 120, 121, 124, 125])
def test_gram_of_rows_in_groups_of_four(f):
    # every number of groups behind the row tiles, full and with one row, and the first f without: whole
    # numbers are exact, and a row of the last four that repeats row 1, 17 or its neighbour has the
    # repeated row's distances to the bit (the groups' matrix instructions add in the tiles' order)
    rng = np.random.default_rng(f)
    order = np.arange(f, dtype=np.int32)
    for d, ld in ((1, 3), (35, 64), (1027, 1056), (20011, 20011), (150011, 150016)):
        Xh = rng.integers(-1, 2, size=(f, ld)).astype(np.float32)
        got = _krum_distances(Xh, d, order)
        G = Xh[:, :d] @ Xh[:, :d].T
        n = np.diag(G)
        assert np.array_equal(got, (n[:, None] + n[None, :] - 2 * G).astype(np.float64)), (f, d)
        Xh = rng.standard_normal((f, ld)).astype(np.float32)
        last, same = f - 1 - int(rng.integers(0, 3)), int(rng.choice([1, 17, f - 5]))
        Xh[last] = Xh[same]
        got = _krum_distances(Xh, d, order)
        assert got[last, same] == 0 and np.array_equal(got, got.T), (f, d)
        rest = np.delete(order, [last, same])
        assert np.array_equal(got[last, rest], got[same, rest]), (f, d, last, same)


def _bulyan_order(dist, c):
    """Bulyan's first phase on given distances: terms added one by one in ascending order, lowest index on ties."""
    f = len(dist)
    left, order = list(range(f)), []
    for _ in range(f - 2 * c):
        scores = []
        for i in left:
            near = sorted(dist[i, j] for j in left if j != i)[:max(0, len(left) - c - 2)]
            total = 0.0
            for v in near:
                total += v
            scores.append((total, i))
        best = min(scores)[1]
        order.append(best)
        left.remove(best)
    return order


@pytest.mark.parametrize("f,c", [(3, 0), (7, 1), (18 + 1, 1), (19, 0), (35, 1), (35, 2), (51, 1), (63, 0), (63, 13), (65, 1),
                                 (67, 1), (67, 0), (69, 1), (83, 1), (127, 0), (127, 1), (127, 31)])
def test_bulyan_selection_on_the_returned_distances(f, c):
    # f - c - 2 terms around whole stretches of sixteen, 64 and the widest; whole numbers, so that equal
    # distances and equal scores abound, and ordinary rows; an infinite row comes last
    rng = np.random.default_rng(f * 100 + c)
    for kind in range(3):
        Xh = rng.integers(-1, 2, size=(f, 40)).astype(np.float32) if kind == 0 else \
            rng.standard_normal((f, 40)).astype(np.float32)
        if kind == 2:
            Xh[f // 2, 3] = 3e30  # its distances are infinite
        out, sel, order, dist = B.byz_bulyan(torch.tensor(Xh, device=DEV), 40, torch.arange(f, dtype=torch.int32, device=DEV), c)
        torch.cuda.synchronize()
        want = _bulyan_order(dist.cpu().numpy(), c)
        assert order.cpu().tolist() == want, (f, c, kind)
        assert sorted(np.nonzero(sel.cpu().numpy())[0].tolist()) == sorted(want), (f, c, kind)


@pytest.mark.parametrize("f,c", [(7, 0), (7, 1), (49, 8), (63, 0), (65, 1), (83, 20), (127, 0), (127, 31)])
def test_bulyan_selection_among_infinite_scores(f, c):
    # finite rows whose squared norm is beyond fp32: distances to them are infinite, and with more than c + 1 of
    # them so are the scores of all vectors left in some round.  A vector is chosen once all the same; lowest
    # index among equal scores.  c + 2 such rows, every second row and all of them
    rng = np.random.default_rng(f * 100 + c)
    d = 131
    idx = torch.arange(f, dtype=torch.int32, device=DEV)
    for far in (np.arange(c + 2) * (f // (c + 2)), np.arange(0, f, 2), np.arange(f)):
        Xh = rng.standard_normal((f, d)).astype(np.float32)
        Xh[far, far] = 3e30
        out, sel, order, dist = B.byz_bulyan(torch.tensor(Xh, device=DEV), d, idx, c)
        torch.cuda.synchronize()
        assert not np.isnan(dist.cpu().numpy()).any()
        want = _bulyan_order(dist.cpu().numpy(), c)
        assert order.cpu().tolist() == want, (f, c, len(far))
        assert np.nonzero(sel.cpu().numpy())[0].tolist() == sorted(want), (f, c, len(far))
    # NaN distances (rows that hold a NaN; two finite rows with such a norm in one column): the order is not
    # specified, a vector is still chosen once
    for kind in range(3):
        Xh = rng.standard_normal((f, d)).astype(np.float32)
        if kind == 0:
            Xh[0, 5] = np.nan
        elif kind == 1:
            Xh[:, 7] = np.nan
        else:
            Xh[[1, f - 1], 9] = 3e30
        out, sel, order, dist = B.byz_bulyan(torch.tensor(Xh, device=DEV), d, idx, c)
        torch.cuda.synchronize()
        chosen = order.cpu().tolist()
        assert np.isnan(dist.cpu().numpy()).any() and len(set(chosen)) == f - 2 * c, (f, c, kind, chosen)
        assert np.nonzero(sel.cpu().numpy())[0].tolist() == sorted(chosen), (f, c, kind)


NETWORKS = (9, 15, 21, 25, 31, 35, 41, 49, 57, 63, 65, 73, 81, 97, 109, 121, 137, 153, 169)


@pytest.mark.parametrize("below,wires", list(zip((0,) + NETWORKS, NETWORKS)))
def test_networks_with_most_and_least_spare_wires(below, wires):
    # every generated network at the ends of its range of f (no spare wire, most of them): median
    # and trimmed mean on raw bit patterns with ties, NaNs and signed zeros and on normal data, d
    # from one coordinate to more than a block with a ragged tail, odd row pitch
    rng = np.random.default_rng(wires)
    for f in sorted({below + 1, below + 2, wires}):
        for d in (1, 5, 63, 1027):
            U = rng.integers(0, 2**32, size=(f + 3, d + 3), dtype=np.uint64).astype(np.uint32)
            U[:, : d // 3] &= np.uint32(0x80000007)
            U[:, 2 * d // 3 :] = rng.standard_normal((f + 3, d + 3 - 2 * d // 3)).astype(np.float32).view(np.uint32)
            X = torch.tensor(U.view(np.int32), device=DEV).view(torch.float32)
            idx = rng.integers(0, f + 3, size=f).astype(np.int32)
            if f % 2 == 1:
                out = B.byz_median(X, d, torch.tensor(idx, device=DEV))
                torch.cuda.synchronize()
                assert np.array_equal(W.bits(out), W.bits(C.median(U, idx, d))), (f, d)
            for b in sorted({0, f // 3, (f - 1) // 2}):
                _trimmed_mean_check(X, idx, d, b, (f, d, b))


@pytest.mark.parametrize("below,wires", [p for p in zip((0,) + NETWORKS, NETWORKS) if p[1] <= 97])
def test_median_of_long_rows_on_and_off_cache_lines(below, wires):
    # above 131072 coordinates rows that do not start on cache lines take four words per thread (from
    # 2^20 on above 35 wires) or another order of the blocks; the last vector overlaps its neighbour
    # and the last group of blocks is not whole.  Pitch off the lines, matrix off the lines, both on
    rng = np.random.default_rng(wires)
    for f, d in [(below + 1, 131077), (wires, 131074), (wires, 262147)] + ([(wires, 1048583)] if wires in (41, 49) else []):
        f += 1 - f % 2
        X = torch.empty(f * ((d + 31) // 32 * 32 + 33) + 1, device=DEV).normal_(generator=torch.Generator(device=DEV).manual_seed(f))
        idx = rng.permutation(f).astype(np.int32)
        idx_dev = torch.tensor(idx, device=DEV)
        for start, ld in ((0, (d + 31) // 32 * 32), (0, (d + 31) // 32 * 32 + 33), (1, (d + 31) // 32 * 32)):
            M = X[start:start + f * ld].reshape(f, ld)
            out = torch.full((d + 8,), 7.0, device=DEV)
            B.byz_median(M, d, idx_dev, out=out)
            torch.cuda.synchronize()
            want = M[:, :d].sort(dim=0).values[(f - 1) // 2]
            assert torch.equal(out[:d], want) and bool((out[d:] == 7.0).all()), (f, d, start, ld)


def test_trimmed_mean_of_few_long_rows():
    # fewer than nine rows on the nine-wire network: four words per thread above 262144 coordinates,
    # the last vector overlaps its neighbour; raw bit patterns with ties, odd pitch
    rng = np.random.default_rng(8)
    for f in range(1, 9):
        for d in (262144, 262145, 262150, 300003):
            U = rng.integers(0, 2**32, size=(f + 1, d + 3), dtype=np.uint64).astype(np.uint32)
            U[:, : d // 3] &= np.uint32(0x80000007)
            U[:, d // 2 :] = rng.standard_normal((f + 1, d + 3 - d // 2)).astype(np.float32).view(np.uint32)
            X = torch.tensor(U.view(np.int32), device=DEV).view(torch.float32)
            for b in sorted({0, (f - 1) // 2}):
                _trimmed_mean_check(X, rng.permutation(f + 1)[:f].astype(np.int32), d, b, (f, d, b))


@pytest.mark.parametrize("f,r", [(49, 5), (9, 7)])
def test_vote_where_the_files_are_no_longer_dealt_out(f, r):
    # 449 to 452 blocks of rows: around the number from which five and seven copies are left to whole
    # blocks; one word of one copy differs, in the first, the last whole and the ragged vector
    for d in (449 * 1024 + 3, 450 * 1024, 450 * 1024 + 5, 452 * 1024 + 1):
        g = torch.Generator(device=DEV).manual_seed(d)
        X = torch.randn(f, 1, d, device=DEV, generator=g).expand(f, r, d).reshape(f * r, d).contiguous()
        rows = torch.arange(f * r, dtype=torch.int32, device=DEV)
        want = np.zeros(f, dtype=np.int64)
        for j, k, c in ((0, 0, 0), (f // 2, r - 1, d // 1024 * 1024 - 1), (f - 1, 1, d - 1)):
            X[j * r + k, c] += 1
            want[j] = sum(1 << i for i, p in enumerate(itertools.combinations(range(r), 2)) if k in p)
        wrep, wrow, neq = B.byz_vote(X, d, rows, f, r)
        torch.cuda.synchronize()
        assert np.array_equal(neq.cpu().numpy(), want), d
        best = [1 if j == 0 else 0 for j in range(f)]
        assert wrep.cpu().tolist() == best and wrow.cpu().tolist() == [j * r + best[j] for j in range(f)], d


def _rows_on_and_off_lines(n, d, seed):
    # [n, d] values in rows that start on cache lines, and off them by pitch and by the matrix's start
    ld = (d + 31) // 32 * 32
    gen = torch.Generator(device=DEV).manual_seed(seed)
    buf = torch.empty(n * (ld + 33) + 1, device=DEV).normal_(generator=gen)
    for start, pitch in ((0, ld), (1, ld + 33)):
        yield buf[start:start + n * pitch].reshape(n, pitch)


@pytest.mark.parametrize("f,r,vec", [(25, 3, 4), (49, 3, 4), (49, 7, 2), (81, 3, 2), (121, 3, 1), (169, 3, 1),
                                     (25, 5, 4), (35, 5, 4), (49, 5, 4)])
def test_long_single_passes_on_and_off_cache_lines(f, r, vec):
    # more than 2048 blocks, dealt out to the XCDs by whole groups of neighbours, the last group not
    # whole and the last vector overlapping; five copies also around the length from which a thread takes
    # four words.  A false copy of every third file, in its last word.
    sizes = [2048 * 256 * vec + 1, 2048 * 256 * vec + 8 * 64 * 256 * vec + 77]
    if r == 5:
        sizes = [(15 << 16) - 1, 15 << 16, sizes[0]]
    for d in sizes:
        for X in _rows_on_and_off_lines(f * r, d, f * r + d % 911):
            for j in range(f):
                X[j * r + 1:(j + 1) * r] = X[j * r]
                if j % 3 == 0:
                    X[j * r + j % r, d - 1] += 1.0
            rows = torch.arange(f * r, dtype=torch.int32, device=DEV)
            first = torch.tensor([1 if j % 3 == 0 and j % r == 0 else 0 for j in range(f)], device=DEV)
            ranks = X.index_select(0, torch.arange(f, device=DEV) * r + first)[:, :d].sort(dim=0).values
            for flags, b in ((0, -1), (B.BYZ_AGG_TRIM(4), 4), (B.BYZ_AGG_EARLY_MAJORITY, -1)):
                out = torch.full((d + 8,), 7.0, device=DEV)
                _, wrep, _ = B.byz_aggregate_opts(X, d, rows, f, r, flags, out=out)
                torch.cuda.synchronize()
                want = ranks[(f - 1) // 2]
                if b >= 0:
                    want = torch.zeros(d, device=DEV)
                    for v in ranks[b:f - b]:
                        want += v
                    want /= torch.tensor(float(f - 2 * b), device=DEV)
                assert torch.equal(out[:d], want) and bool((out[d:] == 7.0).all()), (f, r, d, X.shape[1], flags)
                assert torch.equal(wrep.long(), first), (f, r, d, X.shape[1], flags)
            del ranks


@pytest.mark.parametrize("f", [25, 35, 49])
def test_early_majority_trimmed_mean_of_long_rows_of_five_copies(f):
    # two words a thread at every length, also where other calls take four; an odd last vector
    r, b, rows = 5, f // 8, torch.arange(f * 5, dtype=torch.int32, device=DEV)
    for d in (15 << 16, (1 << 20) + 1):
        X = torch.randn(f, 1, d + 1, device=DEV, generator=torch.Generator(device=DEV).manual_seed(d))
        want = torch.zeros(d, device=DEV)
        for v in X[:, 0, :d].sort(dim=0).values[b:f - b]:
            want += v
        want /= torch.tensor(float(f - 2 * b), device=DEV)
        X = X.expand(f, r, d + 1).reshape(f * r, d + 1).contiguous()
        X[3 * r + 4, d - 1] += 1.0
        out, wrep, _ = B.byz_aggregate_opts(X, d, rows, f, r, B.BYZ_AGG_EARLY_MAJORITY | B.BYZ_AGG_TRIM(b))
        torch.cuda.synchronize()
        assert torch.equal(out, want) and wrep.cpu().tolist() == [0] * f, (f, d)


@pytest.mark.parametrize("f", [9, 15])
def test_long_single_passes_of_few_files(f):
    # up to 15 files of three copies keep the plain order of the blocks up to 8192 of them: the last such
    # launch and the first in groups of neighbours, the group and the last vector not whole
    r, rows, b = 3, torch.arange(f * 3, dtype=torch.int32, device=DEV), 2
    for d in (2049 * 1024 - 1, 8192 * 1024, 8192 * 1024 + 77):
        X = torch.randn(f, 1, d + 1, device=DEV, generator=torch.Generator(device=DEV).manual_seed(d))
        ranks = X[:, 0, :d].sort(dim=0).values
        X = X.expand(f, r, d + 1).reshape(f * r, d + 1).contiguous()
        X[0, d - 1] += 1.0
        X[r * f - 1, 1] -= 2.0
        first = [1] + [0] * (f - 1)
        for flags in (0, B.BYZ_AGG_TRIM(b), B.BYZ_AGG_EARLY_MAJORITY):
            out = torch.full((d + 8,), 7.0, device=DEV)
            _, wrep, _ = B.byz_aggregate_opts(X, d, rows, f, r, flags, out=out)
            torch.cuda.synchronize()
            want = ranks[(f - 1) // 2]
            if flags == B.BYZ_AGG_TRIM(b):
                want = torch.zeros(d, device=DEV)
                for v in ranks[b:f - b]:
                    want += v
                want /= torch.tensor(float(f - 2 * b), device=DEV)
            assert torch.equal(out[:d], want) and bool((out[d:] == 7.0).all()), (f, d, flags)
            assert wrep.cpu().tolist() == first, (f, d, flags)


@pytest.mark.parametrize("f", [9, 49, 81, 97, 127, 171, 207, 255])
def test_sorts_of_long_rows_on_and_off_cache_lines(f):
    # above 131072 coordinates neighbouring blocks go to one XCD where rows don't start on cache lines:
    # trimmed mean, median of more than 169 rows, mean around the median; a last group that is not whole
    for d in (131073, 131072 + 8 * 64 * 64 + 77):
        for X in _rows_on_and_off_lines(f, d, f + d):
            idx = torch.randperm(f, generator=torch.Generator().manual_seed(f)).to(torch.int32).to(DEV)
            ranks = X[:, :d].sort(dim=0).values
            b = f // 4
            want = torch.zeros(d, device=DEV)
            for v in ranks[b:f - b]:
                want += v
            want /= torch.tensor(float(f - 2 * b), device=DEV)
            calls = [(lambda o: B.byz_trimmed_mean(X, d, idx, b, out=o), want),
                     (lambda o: B.byz_median(X, d, idx, out=o), ranks[(f - 1) // 2])]
            if f <= 128:  # one value around the median is the median
                calls.append((lambda o: B.byz_mean_around_median(X, d, idx, 1, out=o), ranks[(f - 1) // 2]))
            for n, (call, expected) in enumerate(calls):
                out = torch.full((d + 8,), 7.0, device=DEV)
                call(out)
                torch.cuda.synchronize()
                assert torch.equal(out[:d], expected) and bool((out[d:] == 7.0).all()), (f, d, X.shape[1], n)


def test_mean_around_median_alone():
    # byz_mean_around_median = the second phase of Bulyan on rows of the caller's choice: every
    # network size of that kernel and the sizes between (spare wires), d from one word to many
    # blocks, beta = 1 (the median, bit for bit), a random beta, beta = f (plain mean);
    # normal data and small integers (ties in the window rule)
    rng = np.random.default_rng(183)
    for f in (1, 3, 9, 13, 15, 25, 27, 49, 51, 63, 81, 99, 121, 127):
        d = int(rng.choice([rng.integers(1, 4), rng.integers(4, 300), rng.integers(300, 20000)]))
        ld = d + int(rng.integers(0, 5))
        Xh = np.zeros((f + 3, ld), dtype=np.float32)
        Xh[:, :d] = rng.standard_normal((f + 3, d)).astype(np.float32) * rng.uniform(0.1, 30.0, size=(f + 3, 1))
        Xh[:, : d // 3] = rng.integers(-3, 4, size=(f + 3, d // 3)).astype(np.float32)
        X = torch.tensor(Xh, device=DEV)
        idx = rng.permutation(f + 3)[:f].astype(np.int32)
        idx_dev = torch.tensor(idx, device=DEV)
        chosen = np.arange(f, dtype=np.int32)
        vmax = np.abs(Xh[idx][:, :d].astype(np.float64)).max(axis=0)
        for beta in sorted({1, int(rng.integers(1, f + 1)), f}):
            out = B.byz_mean_around_median(X, d, idx_dev, beta)
            torch.cuda.synchronize()
            out_o = C.mean_around_median(Xh, idx, chosen, d, beta)
            tol = 1.5 * beta * 2.0 ** -24 * vmax + 1e-44
            assert (np.abs(out.cpu().numpy().astype(np.float64) - out_o) <= tol).all(), (f, d, beta)
            if beta == 1:
                assert np.array_equal(W.bits(out), W.bits(B.byz_median(X, d, idx_dev))), (f, d)
    X = torch.zeros((130, 8), device=DEV)
    for n, beta, code in [(4, 1, -2), (5, 0, -1), (5, 6, -1), (129, 1, -1)]:
        with pytest.raises(B.ByzError) as e:
            B.byz_mean_around_median(X, 8, torch.arange(n, dtype=torch.int32, device=DEV), beta)
        assert e.value.code == code, (n, beta)


@pytest.mark.parametrize("f", [1, 3, 5, 9, 15, 33, 35, 49, 65, 101, 127])
def test_window_around_the_median_on_special_values(f):
    # the window's start is found by halving the candidates where the tests are in order, and by counting the failed
    # ones in the waves that have a NaN or an infinite median: words as of the rule (the window's first position is the
    # number of failed tests behind the lowest candidate), fp32 additions in ascending order.  Waves of ordinary
    # values, of ties, of values whose differences overflow, of infinities, of NaNs; every length of a halving.
    rng = np.random.default_rng(f)
    d = 64 * 9 + 37
    Xh = rng.standard_normal((f, d)).astype(np.float32)
    Xh[:, 64:128] = rng.integers(-2, 3, size=(f, 64))
    Xh[:, 128:192] = rng.choice(np.float32([3e38, -3e38, 1.0, 2e38]), size=(f, 64))
    for w, special in ((3, [np.inf, 0.0, 1.0]), (4, [-np.inf, np.inf, 0.5]), (5, [np.nan, 1.0, 2.0, 3.0]),
                       (6, [np.nan, np.inf, -np.inf, 0.0]), (7, [np.inf, np.inf, 2.0])):
        Xh[:, 64 * w:64 * w + 64] = rng.choice(np.float32(special), size=(f, 64))
    Xh[f // 2, 64 * 8 + 5] = -np.float32(np.nan)
    X = torch.tensor(Xh, device=DEV)
    idx = torch.arange(f, dtype=torch.int32, device=DEV)
    order = np.argsort(O.order_key(Xh.view(np.uint32)), axis=0, kind="stable")
    v = np.take_along_axis(Xh, order, axis=0)
    h, at = (f - 1) // 2, np.arange(d)
    for beta in sorted({b for b in (1, 2, 3, 7, 8, h, h + 1, f - 2, f - 1, f) if 1 <= b <= f}):
        first = max(0, h - beta + 1)
        start = np.full(d, first)
        with np.errstate(invalid="ignore", over="ignore"):
            for s in range(first, h):
                if s + beta <= f - 1:
                    start += ~((v[h] - v[s]) <= (v[s + beta] - v[h]))
            acc = np.zeros(d, dtype=np.float32)
            for t in range(beta):
                acc = acc + v[start + t, at]
            want = acc / np.float32(beta)
        got = B.byz_mean_around_median(X, d, idx, beta).cpu().numpy()
        same = (got.view(np.uint32) == want.view(np.uint32)) | (np.isnan(got) & np.isnan(want))
        assert same.all(), (f, beta, np.flatnonzero(~same)[:5])


@pytest.mark.parametrize("f, r", [(9, 3), (15, 3), (21, 3), (25, 3), (25, 5)])
def test_aggregation_in_one_block(f, r):
    # rows short enough for one block vote, choose and, where the fed copy was not the winner's, redo the output in one
    # kernel: the smallest row, whole waves and one word more and less, the last length of the rule (five sixteenths or
    # three sixteenths of 2^18 words in all, 1024 coordinates at most) and the first behind it.
    rng = np.random.default_rng(f * r)
    rows = rng.permutation(f * r + 2)[:f * r].reshape(f, r).astype(np.int32)
    rows_dev = torch.tensor(rows.reshape(-1), device=DEV)
    for trim in (0, f // 4):
        most = min(1024, ((3 if trim or r == 5 else 5) << 14) // (f * r))
        for d in sorted({4, 5, 63, 64, 65, 255, most - 1, most, most + 1}):
            for split in (False, True):
                G = rng.standard_normal((f, d)).astype(np.float32)
                Xh = np.zeros((f * r + 2, d + 3), dtype=np.float32)
                for j in range(f):
                    Xh[rows[j], :d] = G[j]
                    if split and j % 3 == 0:  # no majority; most of the copies are alike but for a word each
                        for k in range(r // 2 + 1):
                            Xh[rows[j, r - 1 - k], :d] = -2.0
                            Xh[rows[j, r - 1 - k], (11 * j + k) % d] = k
                    elif j % 4 == 1:
                        Xh[rows[j, int(rng.integers(r))], int(rng.integers(d))] += 1.0
                X = torch.tensor(Xh, device=DEV)
                out = torch.full((d + 4,), 7.0, device=DEV)
                flags = B.BYZ_AGG_TRIM(trim) if trim else 0
                _, wrep, ws = B.byz_aggregate_opts(X, d, rows_dev, f, r, flags, out=out)
                out_o, wrep_o, _ = C.aggregate(Xh, rows, d)
                assert np.array_equal(wrep.cpu().numpy(), wrep_o), (trim, d, split)
                if trim:
                    wrow = torch.tensor(rows[np.arange(f), wrep_o], device=DEV)
                    out_o = B.byz_trimmed_mean(X, d, wrow, trim).cpu().numpy()
                assert np.array_equal(W.bits(out[:d]), out_o.view(np.uint32)), (trim, d, split)
                assert bool((out[d:] == 7.0).all()), (trim, d, split)
                if not split:
                    assert B.byz_aggregate_path(ws) == B.BYZ_PATH_SINGLE_PASS, (trim, d)


@pytest.mark.parametrize("f, r, trim", [(9, 3, 0), (9, 3, 2), (15, 3, 0), (21, 3, 0), (25, 3, 0), (25, 3, 6), (25, 5, 0),
                                        (25, 5, 6)])
def test_output_redone_in_one_block(f, r, trim):
    # false copies that differ in a word each: the waves without such a word feed one of them, the vote goes to an honest
    # one, and the path says so (the differing words lie in two waves at most, so rows of four waves and more are redone)
    gen = torch.Generator(device=DEV).manual_seed(f * r)
    rows = torch.arange(f * r, dtype=torch.int32, device=DEV)
    most = min(1024, ((3 if trim or r == 5 else 5) << 14) // (f * r))
    for d in (255, most - 1, most):
        X = torch.empty((f, d), device=DEV).normal_(generator=gen).repeat_interleave(r, dim=0)
        for j in range(0, f, 3):
            for k in range(r // 2 + 1):
                X[j * r + r - 1 - k] = -2.0
                X[j * r + r - 1 - k, (11 * j + k) % d] = float(k)
        out, wrep, ws = B.byz_aggregate_opts(X, d, rows, f, r, B.BYZ_AGG_TRIM(trim) if trim else 0)
        assert B.byz_aggregate_path(ws) == B.BYZ_PATH_MEDIAN_REDONE, d
        assert int(wrep.max()) == 0, d  # a tie of three, or two alike of five
        won = rows[::r].contiguous()
        want = B.byz_trimmed_mean(X, d, won, trim) if trim else B.byz_median(X, d, won)
        assert torch.equal(out.view(torch.int32), want.view(torch.int32)), d


@pytest.mark.parametrize("f, r, d, trim", [(9, 3, 4 * 2048 * 256 + 3, 0), (25, 3, 4 * 2048 * 256 + 1029, 5),
                                           (25, 5, 4 * 2048 * 256 + 1, 0), (49, 3, 4 * 2048 * 256, 0),
                                           (49, 3, 4 * 2048 * 256 + 5, 8), (81, 3, 2048 * 256 + 1, 0),
                                           (121, 3, 2048 * 256 + 63, 20), (65, 5, 2048 * 256 - 1, 0),
                                           (9, 3, 4 * 2048 * 256, 2), (25, 5, 4 * 2048 * 256 - 3, 5),
                                           (49, 7, 131072, 8), (49, 7, 131073, 8), (121, 3, 768 * 256, 0),
                                           (121, 3, 768 * 256 + 1, 0), (169, 3, 768 * 256, 20), (169, 3, 768 * 256 + 1, 0)])
def test_output_redone_in_rounds(f, r, d, trim):
    # longer calls decide in the blocks that redo the output up to 2048 of them (768 for more than 81 files, 131072
    # coordinates for the trimmed mean of 49), and in a kernel of their own beyond: one word or one block past the line, or on
    # it.  In every third file the honest copies win (tie of three, or two alike of five) while the waves see the false
    # ones alike.
    gen = torch.Generator(device=DEV).manual_seed(f + d)
    X = torch.empty((f * r, d), device=DEV)
    rows = np.arange(f * r, dtype=np.int32).reshape(f, r)
    for j in range(f):
        X[j * r].normal_(generator=gen)
        for k in range(1, r):
            X[j * r + k] = X[j * r]
        if j % 3 == 0:
            for k in range(r // 2 + 1):  # replicas 1, 2 (and 3): alike but for a word each
                X[j * r + 1 + k] = -2.0
                X[j * r + 1 + k, (j * 65537 + 31 * k) % d] = k
    rows_dev = torch.tensor(rows.reshape(-1), device=DEV)
    out = torch.full((d + 8,), 7.0, device=DEV)
    _, wrep, ws = B.byz_aggregate_opts(X, d, rows_dev, f, r, B.BYZ_AGG_TRIM(trim) if trim else 0, out=out)
    assert B.byz_aggregate_path(ws) == B.BYZ_PATH_MEDIAN_REDONE
    assert not wrep.cpu().numpy().any()
    winners = torch.tensor(rows[:, 0].copy(), device=DEV)
    want = B.byz_trimmed_mean(X, d, winners, trim) if trim else B.byz_median(X, d, winners)
    assert torch.equal(out[:d].view(torch.int32), want.view(torch.int32))
    assert bool((out[d:] == 7.0).all())


def _gram_additions(d):
    """Most fp32 additions behind one entry of a partial Gram matrix: a run of at most 128 products, the
    runs of a wave (at least four waves in each of 512 blocks, 96 products or more each), then one
    rounding of the block's sum."""
    return 129 + -(-d // (512 * 4 * 96))


def _multi_krum_check(X, idx_np, d, c, m, tag):
    """GPU Multi-Krum against the fp64 oracle.

    Tolerances from the arithmetic: a Gram entry is accumulated in fp32 with at most L additions
    (_gram_additions), then in fp64, so
    |dG_ij| <= L * 2^-24 * (G_ii + G_jj) / 2 and |dD_ij| <= 2 * L * 2^-24 * (G_ii + G_jj).
    A score adds at most f distances.  The selection is compared where the oracle's scores are
    further from the cut than twice that; the mean is checked against the oracle's mean
    (fp32 sequential sum: m * 2^-24 * max|x|)."""
    idx_dev = torch.tensor(idx_np, dtype=torch.int32, device=DEV)
    out, sel, scores, dist = B.byz_multi_krum(X, d, idx_dev, c, m)
    torch.cuda.synchronize()
    Xh = X.detach().cpu().numpy()
    mean_o, sel_o, scores_o, dist_o = O.multi_krum(Xh, idx_np, d, c, m)
    f = len(idx_np)
    L = _gram_additions(d)
    norms = np.diag(dist_o * 0) + np.array([float(np.dot(Xh[j, :d].astype(np.float64), Xh[j, :d].astype(np.float64))) for j in idx_np])
    tol_d = 2.0 * L * 2.0 ** -24 * (norms[:, None] + norms[None, :]) + 1e-300
    dist_g = dist.cpu().numpy()
    assert (np.abs(dist_g - dist_o) <= tol_d).all(), tag
    assert (np.diag(dist_g) == 0).all() and np.array_equal(dist_g, dist_g.T), tag
    tol_s = f * tol_d.max()
    assert (np.abs(scores.cpu().numpy() - scores_o) <= tol_s).all(), tag
    sel_g = sel.cpu().numpy()
    assert sel_g.sum() == m, tag
    cut = np.sort(scores_o)[m - 1]
    assert (sel_g[scores_o < cut - 2 * tol_s] == 1).all(), tag
    assert (sel_g[scores_o > cut + 2 * tol_s] == 0).all(), tag
    # the test inputs keep the scores far from the cut, so both sides select the same rows
    assert np.array_equal(sel_g, sel_o), tag
    rows = Xh[idx_np[sel_o == 1]][:, :d].astype(np.float64)
    tol_m = 1.5 * m * 2.0 ** -24 * np.abs(rows).max(axis=0) + 1e-44
    assert (np.abs(out.cpu().numpy().astype(np.float64) - mean_o) <= tol_m).all(), tag
    return sel_g, sel_o


@pytest.mark.parametrize("scheme,a,b,q,attack", [(MOLS, 5, 3, 4, ALIE), (MOLS, 7, 3, 5, REVERSED),
                                                 (RAM, 5, 5, 6, MIXED), (RAM, 3, 3, 1, CONST),
                                                 (RAM, 3, 5, 2, CONST), (RAM, 7, 9, 6, CONST)])
def test_multi_krum_on_the_vote_winners(scheme, a, b, q, attack):
    for i, d in enumerate([1, 3, 255, 256, 257, 5000, 70001, 300001]):
        w = W.make(scheme, a, b, q, d, attack, seed=400 + i, ld=synth.padded_ld(d, 4) + 4 * (i % 2),
                   device=DEV)
        rows_dev = torch.tensor(w.file_rows.reshape(-1), dtype=torch.int32, device=DEV)
        wrep, wrow, _ = B.byz_vote(w.X, d, rows_dev, w.f, w.r)
        torch.cuda.synchronize()
        idx = wrow.cpu().numpy()
        c = min(w.cmax, (w.f - 3) // 2)
        for m in sorted({1, w.f - c}):
            sel_g, sel_o = _multi_krum_check(w.X, idx, d, c, m, (d, m))
        if d >= 5000 and attack["kind"] in ("reversed", "constant") and c == w.cmax:
            # the distorted winners (far-away payloads) are exactly the ones left out
            lost = [j for j in range(w.f) if int(w.file_workers[j, wrep[j].item()]) in w.byz]
            assert [j for j in range(w.f) if sel_g[j] == 0] == lost
    rows_dev = None
    for (c, m) in [(-1, 1), ((w.f - 1) // 2, 1), (2, 0), (2, w.f - 1)]:  # f < 2c + 3, m outside [1, f - c]
        with pytest.raises(B.ByzError) as e:
            B.byz_multi_krum(w.X, w.d, wrow, c, m)
        assert e.value.code == -1


def _bulyan_check(X, idx_np, d, c, tag, big=False, exact_order=False):
    """GPU Bulyan against the fp64 oracle.

    Distances: tolerance of the Multi-Krum check (L fp32 additions behind a Gram entry).  Phase 1
    is a chain of argmin decisions on fp64 scores computed from those distances: the order
    chosen must equal the oracle's whenever, in every round, the oracle's best score is further
    than twice the score tolerance from its second best; in any case each GPU pick must be
    within that tolerance of the round's best oracle score (a valid pick).  Phase 2 is always
    compared (fp32 sequential sum of beta values: 1.5 * beta * 2^-24 * max|x|): with the oracle's
    output when both chose the same vectors, else with the oracle's second phase run on the
    vectors the GPU chose.  (The second phase's window rule assumes finite values; a non-finite
    value makes the distances of phase 1 NaN, for which the rule is not defined, so no input
    reaches phase 2 with one.)
    Returns True if the GPU chose the oracle's vectors in the oracle's order."""
    idx_dev = torch.tensor(idx_np, dtype=torch.int32, device=DEV)
    out, sel, order, dist = B.byz_bulyan(X, d, idx_dev, c)
    torch.cuda.synchronize()
    Xh = X.detach().cpu().numpy()
    f = len(idx_np)
    theta, beta = f - 2 * c, f - 4 * c
    out_o, chosen_o, dist_o = (C.bulyan if big else O.bulyan)(Xh, idx_np, d, c)
    L = _gram_additions(d)
    norms = np.array([float(np.dot(Xh[j, :d].astype(np.float64), Xh[j, :d].astype(np.float64))) for j in idx_np])
    tol_d = 2.0 * L * 2.0 ** -24 * (norms[:, None] + norms[None, :]) + 1e-300
    dist_g = dist.cpu().numpy()
    assert (np.abs(dist_g - dist_o) <= tol_d).all(), tag
    tol_s = f * tol_d.max()
    order_g = [int(x) for x in order.cpu().numpy()]
    sel_g = sel.cpu().numpy()
    assert len(order_g) == theta and len(set(order_g)) == theta, tag
    assert sorted(order_g) == [i for i in range(f) if sel_g[i] == 1], tag
    # replay the rounds along the GPU's picks with the oracle's distances
    remaining = list(range(f))
    decisive = True
    for pick in order_g:
        k = max(len(remaining) - c - 2, 0)
        scores = {i: sum(sorted(dist_o[i, j] for j in remaining if j != i)[:k]) for i in remaining}
        ranked = sorted(remaining, key=lambda i: (scores[i], i))
        assert scores[pick] <= scores[ranked[0]] + 2 * tol_s, (tag, pick)
        if len(ranked) > 1 and scores[ranked[1]] - scores[ranked[0]] <= 2 * tol_s and k > 0:
            decisive = False
        remaining.remove(pick)
    if decisive or exact_order:
        assert order_g == chosen_o, tag
    same_order = order_g == chosen_o
    if not same_order:
        # Only a near-tie of the oracle's own fp64 scores (within twice the stated score
        # tolerance, asserted above: `decisive` is False here) lets the fp32 Gram matrix decide
        # a round the other way.  Every pick was checked to be valid; phase 2 then runs on
        # another chosen set, so it is compared with the oracle's phase 2 on that set.
        assert not decisive, tag
        out_o = C.mean_around_median(Xh, idx_np, np.array(order_g, dtype=np.int32), d, beta)
    chosen = np.array(order_g, dtype=np.int32)
    vmax = np.abs(Xh[idx_np[chosen]][:, :d].astype(np.float64)).max(axis=0)
    tol_m = 1.5 * beta * 2.0 ** -24 * vmax + 1e-44
    assert (np.abs(out.cpu().numpy().astype(np.float64) - out_o) <= tol_m).all(), tag
    return same_order


@pytest.mark.parametrize("scheme,a,b,q,attack", [(MOLS, 5, 3, 4, ALIE), (MOLS, 7, 3, 5, REVERSED),
                                                 (RAM, 5, 5, 6, MIXED), (RAM, 3, 3, 1, CONST),
                                                 (RAM, 3, 5, 2, CONST), (RAM, 3, 9, 2, ALIE)])
def test_bulyan_on_the_vote_winners(scheme, a, b, q, attack):
    # per-file gradient scales make the honest vectors' scores differ by far more than the fp32
    # Gram error, so the order chosen is decided and compared exactly in most cases
    attack = dict(attack, file_scales=True)
    compared = []
    for i, d in enumerate([1, 3, 4, 257, 5000, 70001]):
        w = W.make(scheme, a, b, q, d, attack, seed=500 + i, ld=synth.padded_ld(d, 4) + 4 * (i % 2),
                   device=DEV)
        rows_dev = torch.tensor(w.file_rows.reshape(-1), dtype=torch.int32, device=DEV)
        wrep, wrow, _ = B.byz_vote(w.X, d, rows_dev, w.f, w.r)
        torch.cuda.synchronize()
        idx = wrow.cpu().numpy()
        for c in sorted({0, 1, (w.f - 3) // 4}):
            compared.append(_bulyan_check(w.X, idx, d, c, (w.f, d, c)))
    # the inputs are built so that near-ties are rare: almost every case follows the oracle's
    # order (the others were compared on the GPU's own valid picks)
    assert sum(compared) >= len(compared) - 2, compared
    for c in (-1, (w.f - 3) // 4 + 1):  # f < 4c + 3
        with pytest.raises(B.ByzError) as e:
            B.byz_bulyan(w.X, w.d, wrow, c)
        assert e.value.code == -1
    with pytest.raises(B.ByzError) as e:  # even f
        B.byz_bulyan(w.X, w.d, wrow[:w.f - 1], 0)
    assert e.value.code == -2


def test_bulyan_ties_and_identical_vectors():
    # identical vectors: all distances 0, picks in index order, output = the vector; and a case
    # with exact ties in the window rule (integers around the median)
    d, f = 300, 25
    base = torch.randn(1, d, device=DEV)
    X = base.repeat(f, 1).contiguous()
    idx = np.arange(f, dtype=np.int32)
    out, sel, order, dist = B.byz_bulyan(X, d, torch.tensor(idx, device=DEV), 4)
    torch.cuda.synchronize()
    assert order.cpu().tolist() == list(range(f - 8)) and (dist == 0).all()
    # nine equal values added in fp32 and divided by nine: within a few ulp of the value
    assert (out - base[0]).abs().max().item() <= 9 * 2.0 ** -24 * base.abs().max().item()
    # every vector is one distinct small integer (equal in all coordinates): distances, scores
    # and the fp32 Gram are exact, equal scores abound (lowest index wins), and the window
    # around the median meets equal distances on both sides (the lower value is taken)
    vals = np.array([3, -2, 7, 0, 1, -1, 5, 2, -3, 4, 6, -4, 8, -5, 9], dtype=np.float32)
    Y = torch.tensor(np.repeat(vals[:, None], 16, axis=1), device=DEV)
    assert _bulyan_check(Y, np.arange(15, dtype=np.int32), 16, 2, "integer ties", exact_order=True)
    assert _bulyan_check(Y, np.arange(15, dtype=np.int32), 16, 3, "integer ties", exact_order=True)
    # the same two situations past 64 vectors (rounds on rows in LDS, winner across two waves)
    f = 81
    X = base.repeat(f, 1).contiguous()
    out, sel, order, dist = B.byz_bulyan(X, d, torch.arange(f, dtype=torch.int32, device=DEV), 10)
    torch.cuda.synchronize()
    assert order.cpu().tolist() == list(range(f - 20)) and (dist == 0).all()
    assert (out - base[0]).abs().max().item() <= 41 * 2.0 ** -24 * base.abs().max().item()
    rng = np.random.default_rng(85)
    vals = rng.permutation(np.arange(-42, 43)).astype(np.float32)  # 85 distinct integers
    Y = torch.tensor(np.repeat(vals[:, None], 16, axis=1), device=DEV)
    for c in (0, 3, 20):
        assert _bulyan_check(Y, np.arange(85, dtype=np.int32), 16, c, ("integer ties", c), exact_order=True)


def _tolerant_check(X, rows_np, d, f, r, atol, rtol, tag):
    rows_dev = torch.tensor(rows_np.reshape(-1), dtype=torch.int32, device=DEV)
    wrep, wrow, far = B.byz_vote_tolerant(X, d, rows_dev, f, r, atol, rtol)
    torch.cuda.synchronize()
    wrep_o, wrow_o, far_o = C.vote_tolerant(X.detach().cpu().numpy(), rows_np, d, atol, rtol)
    # the decision is taken in fp32 on both sides: every word must agree
    assert np.array_equal(W.bits(far), far_o), tag
    assert np.array_equal(wrep.cpu().numpy(), wrep_o), tag
    assert np.array_equal(wrow.cpu().numpy(), wrow_o), tag
    return wrep_o, far_o


@pytest.mark.parametrize("scheme,a,b,q", [(MOLS, 5, 3, 4), (RAM, 5, 5, 6), (RAM, 7, 7, 3),
                                          (MOLS, 9, 3, 4)])
def test_tolerant_vote(scheme, a, b, q):
    # honest copies of a file differ by relative rounding noise, Byzantine copies are far away
    rng = np.random.default_rng(900 + a)
    for i, d in enumerate([1, 2, 3, 5, 64, 1000, 4099, 70001]):
        ld = d if i % 2 == 0 else synth.padded_ld(d, 4) + 4
        w = W.make(scheme, a, b, q, d, REVERSED, seed=800 + i, ld=ld, device=DEV)
        X = w.X.clone()
        noise = torch.tensor(rng.standard_normal((X.shape[0], d)).astype(np.float32), device=DEV)
        X[:, :d] *= (1.0 + 2e-7 * noise)
        for atol, rtol in [(1e-6, 1e-5), (0.0, 1e-6), (0.0, 3e-7), (1e-7, 0.0), (0.0, 0.0)]:
            wrep_o, far_o = _tolerant_check(X, w.file_rows, d, w.f, w.r, atol, rtol, (d, atol, rtol))
        # with the widest tolerance honest copies are close to each other and the vote behaves
        # as Sec. 2 says: a file is lost iff at least r' of its copies are Byzantine
        wrep_o, _ = _tolerant_check(X, w.file_rows, d, w.f, w.r, 1e-6, 1e-5, d)
        lost = [j for j in range(w.f) if int(w.file_workers[j, wrep_o[j]]) in w.byz]
        assert len(lost) == w.cmax
    # noise right at the tolerance: many element-wise decisions fall within an ulp of the bound
    w = W.make(MOLS, 5, 3, 0, 3, REVERSED, seed=77, device=DEV)
    for trial in range(20):
        X = w.X.clone()
        noise = torch.tensor(rng.standard_normal((X.shape[0], 3)).astype(np.float32), device=DEV)
        X[:, :3] *= (1.0 + 1e-6 * noise)
        _, far_o = _tolerant_check(X, w.file_rows, 3, w.f, w.r, 0.0, 2e-6, trial)
    assert 0 < np.count_nonzero(far_o) < w.f  # the last trial has both outcomes


def test_tolerant_vote_special_values_and_errors():
    d = 2048
    w = W.make(MOLS, 5, 3, 4, d, ALIE, seed=81, device=DEV)
    X = w.X.clone()
    Xi = X.view(torch.int32)
    rng = np.random.default_rng(82)
    patterns = np.array([0x7FC00000, 0xFFC00000, 0x7F800000, 0xFF800000, 0x80000000, 0x00000000,
                         0x00000001, 0x80000001, 0x7F7FFFFF], dtype=np.uint32).view(np.int32)
    for _ in range(800):
        row = int(rng.integers(0, X.shape[0]))
        c = int(rng.integers(0, d))
        Xi[row, c] = int(patterns[rng.integers(0, len(patterns))])
    for atol, rtol in [(0.0, 0.0), (1e-3, 1e-3), (float("inf"), 0.0)]:
        _tolerant_check(X, w.file_rows, d, w.f, w.r, atol, rtol, (atol, rtol))
    rows_dev = torch.tensor(w.file_rows.reshape(-1), dtype=torch.int32, device=DEV)
    for atol, rtol in [(-1.0, 0.0), (0.0, -1e-3), (float("nan"), 0.0)]:
        with pytest.raises(B.ByzError) as e:
            B.byz_vote_tolerant(X, d, rows_dev, w.f, w.r, atol, rtol)
        assert e.value.code == -1
    wrep, wrow, far = B.byz_vote_tolerant(X, 0, rows_dev, w.f, w.r, 0.0, 0.0)
    torch.cuda.synchronize()
    assert (wrep == 0).all() and (far == 0).all()


@pytest.mark.parametrize("l", [5, 7, 9])
def test_hip_graph_capture_of_the_other_entry_points(l):
    # vote (exact and tolerant), trimmed mean, Multi-Krum and Bulyan also enqueue kernels only;
    # f = 49 has four row tiles in the Gram kernel, f = 81 six, the wide selection kernel, which asks for
    # more than 64 KiB of LDS, and the 81-wire second phase of Bulyan
    w = W.make(MOLS, l, 3, 3, 50_001, dict(REVERSED, file_scales=True), seed=14, device=DEV)
    rows_dev = torch.tensor(w.file_rows.reshape(-1), dtype=torch.int32, device=DEV)
    c = 2

    def run(X):
        wrep, wrow, neq = B.byz_vote(X, w.d, rows_dev, w.f, w.r)
        trep, trow, far = B.byz_vote_tolerant(X, w.d, rows_dev, w.f, w.r, 1e-6, 1e-5)
        tm = B.byz_trimmed_mean(X, w.d, wrow, c)
        mk, sel, scores, dist = B.byz_multi_krum(X, w.d, wrow, c, w.f - c)
        bu, bsel, order, bdist = B.byz_bulyan(X, w.d, trow, c)
        return [wrep, neq, trep, far, tm, mk, sel, bu, bsel, order]

    X2 = w.X.clone()
    X2[int(w.file_rows[2, 1])] *= 3.0
    X2[int(w.file_rows[2, 2])] *= 3.0   # two equal wrong copies win file 2
    eager = [[t.clone() for t in run(X)] for X in (w.X, X2)]
    torch.cuda.synchronize()
    assert eager[0][0][2].item() == 0 and eager[1][0][2].item() == 1
    Xs = w.X.clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        run(Xs)  # warm-up outside the capture (first-call set-up of the library and of torch)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        outs = run(Xs)
    for rep, which in enumerate([0, 1, 0, 1]):
        Xs.copy_((w.X, X2)[which])
        for t in outs:
            t.zero_()
        graph.replay()
        torch.cuda.synchronize()
        for got, want in zip(outs, eager[which]):
            assert torch.equal(got.view(torch.int32), want.view(torch.int32)), (rep, which)
        again = run((w.X, X2)[which])  # eager work between replays
        torch.cuda.synchronize()
        for got, want in zip(again, eager[which]):
            assert torch.equal(got.view(torch.int32), want.view(torch.int32))


SINGLE_PASS_SHAPES = ((9, 3), (15, 3), (21, 3), (25, 3), (25, 5), (35, 5), (49, 3), (49, 5), (49, 7), (63, 7),
                      (65, 5), (81, 3), (121, 3), (169, 3))


def _median_and_trimmed_mean(winners, b):
    """Of distinct finite values: the middle row of the sorted ones; the kept ones added in order."""
    v = winners.sort(dim=0).values
    f = v.shape[0]
    total = torch.zeros(v.shape[1], device=v.device)
    for i in range(b, f - b):
        total += v[i]
    trimmed = total.cpu().numpy() / np.float32(f - 2 * b)
    return W.bits(v[(f - 1) // 2].contiguous()), trimmed.view(np.uint32)


@pytest.mark.parametrize("f,r", SINGLE_PASS_SHAPES)
def test_single_pass_around_every_change_of_width(f, r):
    # every single-pass shape, median and trimmed mean, with and without the early majority, where the
    # number of words per thread changes: one block of 256 threads, one block of the wide form, the
    # longest row that runs one word per thread; above 131072 coordinates the median and the trimmed
    # mean behind the decision run four words too.  First with tampered copies that are outvoted,
    # then with a file without a majority whose winner every stretch around one word outnumbers, so
    # that the kernels behind the decision write the output
    assert B.byz_aggregate_has_single_pass(f, r)
    wide = (2 if r >= 5 else 4) if f <= 49 else (2 if f <= 81 else 1)
    short = 65536 if f <= 25 and r == 5 else 131072
    rows = torch.arange(f * r, dtype=torch.int32, device=DEV)
    b = max(1, f // 8)
    for d in sorted({255, 256, 257, 256 * wide, 256 * wide + 1, short, short + 1, 131072, 131079}):
        g = torch.Generator(device=DEV).manual_seed(f * 10 + r + d)
        X = torch.randn(f, 1, d + 3, device=DEV, generator=g).expand(f, r, d + 3).reshape(f * r, d + 3).contiguous()
        X[0] += 1.0                        # file 0: the first copy differs everywhere
        X[r + r - 1, d - 1] -= 2.0         # file 1: the last copy differs in the last word
        winner = [1] + [0] * (f - 1)
        for majority in (True, False):
            if not majority:               # the middle file: every copy differs from every other in a word of its own
                j = f // 2
                for k in range(r):
                    X[j * r + k, d // 2 + k] = 9.0 + k
                X[j * r, d - 2] = -9.0
            won = torch.stack([X[q * r + winner[q], :d] for q in range(f)])
            want = _median_and_trimmed_mean(won, b)
            for flags in (0, B.BYZ_AGG_TRIM(b), B.BYZ_AGG_EARLY_MAJORITY, B.BYZ_AGG_TRIM(b) | B.BYZ_AGG_EARLY_MAJORITY):
                out = torch.full((d + 8,), 7.0, device=DEV)
                _, wrep, ws = B.byz_aggregate_opts(X, d, rows, f, r, flags, out=out)
                torch.cuda.synchronize()
                tag = (f, r, d, majority, flags)
                assert wrep.cpu().tolist() == winner, tag
                assert np.array_equal(W.bits(out[:d].contiguous()), want[1 if flags & B.BYZ_AGG_TRIMMED_MEAN else 0]), tag
                assert bool((out[d:] == 7.0).all()), tag
                if flags & B.BYZ_AGG_EARLY_MAJORITY == 0:
                    assert B.byz_aggregate_path(ws) == (SINGLE if majority else REDONE), tag


@pytest.mark.parametrize("f,r", SINGLE_PASS_SHAPES)
def test_short_rows_where_the_blocks_or_the_kernels_change(f, r):
    # the longest row of every form of the two-kernel call and the shortest of the next one: blocks of 256 and
    # 512 threads of one word, the wider blocks of up to 49 files, the four kernels; a tampered copy that
    # is outvoted, told by the last word, then a file without a majority
    slots = 4096 // ((f * {3: 8, 5: 16, 7: 32}[r] + 127) // 128 * 4)
    sizes = [slots * 256, slots * 512] if f >= 21 else [131072]
    if 21 <= f <= 49:
        sizes += [slots * 1024] + ([slots * 2048] if r == 3 and f <= 25 else [])
    rows = torch.arange(f * r, dtype=torch.int32, device=DEV)
    b = max(1, f // 8)
    for d in sorted({1003} | {n + e for n in sizes for e in (0, 1)}):
        g = torch.Generator(device=DEV).manual_seed(f * 10 + r + d)
        X = torch.randn(f, 1, d + 2, device=DEV, generator=g).expand(f, r, d + 2).reshape(f * r, d + 2).contiguous()
        X[0, d - 1] += 1.0
        X[r * f - 1, 0] -= 2.0
        winner = [1] + [0] * (f - 1)
        for majority in (True, False):
            if not majority:
                for k in range(r):
                    X[f // 2 * r + k, d // 2 + k] = 9.0 + k
                X[f // 2 * r, d - 2] = -9.0
            want = _median_and_trimmed_mean(torch.stack([X[q * r + winner[q], :d] for q in range(f)]), b)
            for trim in (0, 1):
                out = torch.full((d + 8,), 7.0, device=DEV)
                ws = torch.randint(0, 256, (B.byz_aggregate_workspace_bytes(f, r),), dtype=torch.uint8, device=DEV)
                _, wrep, _ = B.byz_aggregate_opts(X, d, rows, f, r, B.BYZ_AGG_TRIM(b) if trim else 0, out=out, workspace=ws)
                torch.cuda.synchronize()
                tag = (f, r, d, majority, trim)
                assert B.byz_aggregate_path(ws) == (SINGLE if majority else REDONE), tag
                assert wrep.cpu().tolist() == winner, tag
                assert np.array_equal(W.bits(out[:d].contiguous()), want[trim]), tag
                assert bool((out[d:] == 7.0).all()), tag


@pytest.mark.parametrize("d", [524288, 524289, 698368, 698369])
def test_short_rows_around_one_block_a_cu(d):
    # the median of (25,3) takes four kernels between 256 and 341 blocks of 2048 words and two on either side
    f, r, rows = 25, 3, torch.arange(75, dtype=torch.int32, device=DEV)
    X = torch.randn(f, 1, d + 1, device=DEV, generator=torch.Generator(device=DEV).manual_seed(d))
    X = X.expand(f, r, d + 1).reshape(f * r, d + 1).contiguous()
    X[0, d - 1] += 1.0
    for majority in (True, False):
        if not majority:
            for k in range(r):
                X[r * 12 + k, d // 2 + k] = 9.0 + k
            X[r * 12, d - 2] = -9.0
        keep = torch.arange(f, device=DEV) * r
        keep[0] += 1
        want = X.index_select(0, keep)[:, :d].sort(dim=0).values[f // 2]
        out, wrep, ws = B.byz_aggregate(X, d, rows, f, r)
        torch.cuda.synchronize()
        assert torch.equal(out, want) and wrep.cpu().tolist() == [1] + [0] * 24, (d, majority)
        assert B.byz_aggregate_path(ws) == (SINGLE if majority else REDONE), (d, majority)


@pytest.mark.parametrize("f", [171, 191, 193, 223, 225, 255])
def test_pass_over_files_split_over_two_waves(f):
    # most and fewest spare wires of every size of the halves, the shortest rows that take it and a ragged
    # end; files of both waves tampered with: copies that are outvoted, told by one word, then a file of each
    # wave without a majority, whose winner the stretch around one word outnumbers: only then the median is
    # redone, and one word fewer takes vote and median one after the other, which redo nothing
    r, rows, b = 3, torch.arange(f * 3, dtype=torch.int32, device=DEV), f // 8
    for d in ((1 << 18) - 1, 1 << 18, (1 << 18) + 37):
        g = torch.Generator(device=DEV).manual_seed(f + d)
        X = torch.randn(f, 1, d + 2, device=DEV, generator=g).expand(f, r, d + 2).reshape(f * r, d + 2).contiguous()
        X[0] += 1.0
        X[3 * 130, d - 1] += 1.0
        X[3 * f - 1, 5] -= 2.0
        winner = [0] * f
        winner[0] = winner[130] = 1
        for majority in (True, False):
            if not majority:
                for j in (7, f - 20):
                    for k in range(r):
                        X[3 * j + k, d // 2 + k] = 9.0 + k
                    X[3 * j, d - 2] = -9.0
            want = _median_and_trimmed_mean(torch.stack([X[3 * q + winner[q], :d] for q in range(f)]), b)
            for trim in (0, 1):
                out = torch.full((d + 8,), 7.0, device=DEV)
                ws = torch.randint(0, 256, (B.byz_aggregate_workspace_bytes(f, r),), dtype=torch.uint8, device=DEV)
                _, wrep, _ = B.byz_aggregate_opts(X, d, rows, f, r, B.BYZ_AGG_TRIM(b) if trim else 0, out=out, workspace=ws)
                torch.cuda.synchronize()
                tag = (f, d, majority, trim)
                redone = d >= 1 << 18 and not majority
                assert B.byz_aggregate_path(ws) == (TWO_STEP | REDONE if redone else TWO_STEP), tag
                assert wrep.cpu().tolist() == winner, tag
                assert np.array_equal(W.bits(out[:d].contiguous()), want[trim]), tag
                assert bool((out[d:] == 7.0).all()), tag


def _hidden_pattern_case(rng, scheme, a, b, d, tag, seen):
    """Random equality patterns among the copies of random files, the classes one changed word apart at random
    coordinates, in both modes against the oracle; the path codes go into seen."""
    w = W.make(scheme, a, b, 0, d, REVERSED, seed=int(rng.integers(1 << 30)), device=DEV)
    X = w.X.clone()
    for j in rng.permutation(w.f)[:int(rng.integers(1, max(2, w.f // 2)))]:
        n_classes = int(rng.integers(1, w.r + 1))
        labels = rng.integers(0, n_classes, size=w.r)
        where = rng.integers(0, d, size=n_classes)
        for k in range(w.r):
            if labels[k] or rng.integers(2):
                X[int(w.file_rows[j, k]), int(where[labels[k]])] += float(1 + labels[k])
    rows_dev = torch.tensor(w.file_rows.reshape(-1), dtype=torch.int32, device=DEV)
    Xh = X.cpu().numpy()
    wrep_o, wrow_o, _ = C.vote(Xh, w.file_rows, d)
    out_o = C.median(Xh, wrow_o, d)
    ws = torch.empty(B.byz_aggregate_workspace_bytes(w.f, w.r), dtype=torch.uint8, device=DEV)
    for flags in (0, B.BYZ_AGG_EARLY_MAJORITY):
        out, wrep, _ = B.byz_aggregate_opts(X, d, rows_dev, w.f, w.r, flags, workspace=ws)
        path = B.byz_aggregate_path(ws)
        seen.add((flags, path))
        assert np.array_equal(W.bits(out), W.bits(out_o)), (tag, scheme, a, b, d, flags, path)
        assert np.array_equal(wrep.cpu().numpy(), wrep_o), (tag, scheme, a, b, d, flags, path)


def test_hidden_equality_patterns_of_wide_files():
    # r = 3 ... 13: random equality patterns among the copies of random files, the classes one
    # changed word apart at random coordinates (the comparison over all of d is what finds
    # them): with and without a majority, ties between classes, the first copy inside and
    # outside the winning class; both modes, and every path code has to turn up
    rng = np.random.default_rng(5)
    shapes = [(RAM, 5, 5), (RAM, 3, 5), (RAM, 3, 7), (RAM, 5, 7), (RAM, 7, 7), (RAM, 7, 9),
              (RAM, 5, 13), (MOLS, 7, 5), (MOLS, 9, 5), (MOLS, 5, 3), (MOLS, 13, 3), (FRC, 25, 5)]
    seen = set()
    for case in range(90):
        scheme, a, b = shapes[case % len(shapes)]
        d = int(rng.choice([rng.integers(300, 3000), rng.integers(3000, 90000)]))
        _hidden_pattern_case(rng, scheme, a, b, d, case, seen)
    assert {p for fl, p in seen if fl == 0} >= {B.BYZ_PATH_SINGLE_PASS, B.BYZ_PATH_MEDIAN_REDONE,
                                                B.BYZ_PATH_TWO_STEP}, seen
    assert {p for fl, p in seen if fl} >= {B.BYZ_PATH_SINGLE_PASS, B.BYZ_PATH_REVOTED,
                                           B.BYZ_PATH_REVOTED | B.BYZ_PATH_MEDIAN_REDONE}, seen


def test_hidden_equality_patterns_of_rows_past_the_short_form():
    # the same at lengths where the blocks' findings have no slots left and are merged in shared words: just past
    # every shape's reach, and (25,3) where it takes four kernels in between
    rng = np.random.default_rng(6)
    seen = set()
    cases = [(MOLS, 5, 3, 524_289), (MOLS, 5, 3, 1_048_577), (RAM, 5, 5, 262_145), (RAM, 5, 7, 208_897), (MOLS, 7, 3, 262_145),
             (MOLS, 7, 5, 149_505), (RAM, 7, 7, 79_873), (RAM, 7, 9, 32_769), (RAM, 5, 13, 57_857), (MOLS, 9, 3, 87_041),
             (MOLS, 11, 3, 65_537), (MOLS, 13, 3, 47_617), (RAM, 3, 3, 131_073), (RAM, 3, 5, 131_073)]
    for case, (scheme, a, b, d) in enumerate(cases + cases):
        _hidden_pattern_case(rng, scheme, a, b, d + case // len(cases) * 7, case, seen)
    assert {p for fl, p in seen if fl == 0} == {B.BYZ_PATH_SINGLE_PASS, B.BYZ_PATH_MEDIAN_REDONE}, seen


@pytest.mark.parametrize("scheme,a,b,q,d", [(MOLS, 5, 3, 4, 300_007), (MOLS, 5, 3, 4, 1_050_001), (RAM, 7, 7, 5, 80_001)])
def test_repeated_calls_on_one_workspace_never_change(scheme, a, b, q, d):
    # what the waves publish through atomics (pair bits, which copies were fed) may arrive in
    # any order: the same call forty times on one workspace, on an input that takes the single
    # pass and on one that sends it past it, has to give the same words, winners and path.  The
    # first size writes to slots instead (but in early-majority mode), the others are past them
    w = W.make(scheme, a, b, q, d, ALIE, seed=91, ld=synth.padded_ld(d, 64), device=DEV)
    rows_dev = torch.tensor(w.file_rows.reshape(-1), dtype=torch.int32, device=DEV)
    split = w.X.clone()
    for j in range(w.f):
        ks = [k for k in range(w.r) if int(w.file_workers[j, k]) in w.byz]
        if len(ks) >= 2:
            for i, k in enumerate(ks):
                split[int(w.file_rows[j, k]), d // 2 + 7 + 64 * i] += 1.0
    seen_paths = set()
    for X in (w.X, split):
        for flags in (0, B.BYZ_AGG_EARLY_MAJORITY, B.BYZ_AGG_TRIM(w.cmax)):
            ws = torch.empty(B.byz_aggregate_workspace_bytes(w.f, w.r), dtype=torch.uint8, device=DEV)
            out0, wrep0, _ = B.byz_aggregate_opts(X, d, rows_dev, w.f, w.r, flags, workspace=ws)
            path0 = B.byz_aggregate_path(ws)
            seen_paths.add(path0)
            out0, wrep0 = out0.clone(), wrep0.clone()
            if flags & B.BYZ_AGG_TRIMMED_MEAN == 0:
                out_o, wrep_o, _ = C.aggregate(X.cpu().numpy(), w.file_rows, d)
                assert np.array_equal(W.bits(out0), W.bits(out_o)), flags
                assert np.array_equal(wrep0.cpu().numpy(), wrep_o), flags
            out, wrep = torch.empty_like(out0), torch.empty_like(wrep0)
            for it in range(40):
                B.byz_aggregate_opts(X, d, rows_dev, w.f, w.r, flags, out=out, winner_replica=wrep,
                                     workspace=ws)
                assert B.byz_aggregate_path(ws) == path0, (flags, it)
                assert torch.equal(out.view(torch.int32), out0.view(torch.int32)), (flags, it)
                assert torch.equal(wrep, wrep0), (flags, it)
    assert SINGLE in seen_paths and REDONE in seen_paths, seen_paths


def _keep_busy(scratch, times=100):
    for _ in range(times):  # 50 us each at least
        scratch.mul_(1.0)


@pytest.mark.parametrize("as_handle", [False, True])
def test_row_tables_are_checked_on_the_stream_of_the_call(as_handle):
    # vote and median of its winners on a busy side stream, nothing on the current one: the check of the winner
    # table has to come behind the vote.  The memory new tables get holds rows outside the matrix.  Then a table
    # that the current stream is still making, for a call on the side stream.
    f, r, d = 25, 3, 4099
    w = W.make(MOLS, 5, 3, 3, d, REVERSED, seed=3, device=DEV)
    rows = torch.tensor(w.file_rows.reshape(-1), dtype=torch.int32, device=DEV)
    side = torch.cuda.Stream()
    on = side.cuda_stream if as_handle else side
    wrep0, wrow0, neq0 = B.byz_vote(w.X, d, rows, f, r)
    want = B.byz_median(w.X, d, wrow0)
    scratch = torch.ones(1 << 26, device=DEV)
    backwards = torch.arange(f * r, dtype=torch.int32, device=DEV)
    for it in range(3):
        junk = [torch.full((f,), -7 + 1000 * (it % 2), dtype=torch.int32, device=DEV) for _ in range(64)]
        torch.cuda.synchronize()
        del junk
        with torch.cuda.stream(side):
            _keep_busy(scratch)
        wrep, wrow, _ = B.byz_vote(w.X, d, rows, f, r, stream=on)
        out = B.byz_median(w.X, d, wrow, stream=on)
        side.synchronize()
        assert torch.equal(wrow, wrow0) and torch.equal(out.view(torch.int32), want.view(torch.int32)), it
        _keep_busy(scratch)
        table = (f * r - 1 - backwards)[:f]
        out = B.byz_median(w.X, d, table, stream=on)
        side.synchronize()
        assert torch.equal(out.view(torch.int32), B.byz_median(w.X, d, table.clone()).view(torch.int32)), it
    # a table that was refused is looked at again, whoever wrote it in the meantime
    table = torch.full((f,), f * r, dtype=torch.int32, device=DEV)
    with pytest.raises(ValueError, match="names rows"):
        B.byz_median(w.X, d, table, stream=on)
    B.byz_calibration_copy(torch.zeros(4 * ((f + 3) // 4), dtype=torch.int32, device=DEV)[:f // 4 * 4], table[:f // 4 * 4])
    with pytest.raises(ValueError, match="names rows 0..%d" % (f * r)):
        B.byz_median(w.X, d, table, stream=on)


def test_tensors_of_a_call_on_another_stream_share_no_memory_with_the_current_one():
    # what a call allocates while its stream is busy is neither what work still queued on the current stream
    # reads, nor given away when it is dropped before the call has run
    d = 70001
    X = torch.randn(25, d, device=DEV)
    idx = torch.arange(25, dtype=torch.int32, device=DEV)
    want = B.byz_median(X, d, idx)
    scratch = torch.ones(1 << 26, device=DEV)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    for on in (side, side.cuda_stream):
        source = torch.ones(d, device=DEV)
        _keep_busy(scratch)
        copy, at = source + 0, source.data_ptr()
        del source
        out = B.byz_median(X, d, idx, stream=on)
        assert out.data_ptr() != at
        torch.cuda.synchronize()
        assert bool((copy == 1.0).all()) and torch.equal(out, want)
        with torch.cuda.stream(side):
            _keep_busy(scratch)
        out = B.byz_median(X, d, idx, stream=on)
        at = out.data_ptr()
        del out
        assert all(torch.empty(d, device=DEV).data_ptr() != at for _ in range(2))
        torch.cuda.synchronize()


def test_workspaces_of_calls_on_a_busy_stream():
    # Multi-Krum, Bulyan and the aggregation keep working in workspaces they allocated and dropped while the
    # current stream fills everything it can get of that size
    f, d = 25, 4099
    X = torch.randn(f, d, device=DEV)
    idx = torch.arange(f, dtype=torch.int32, device=DEV)
    w = W.make(MOLS, 5, 3, 3, d, ALIE, seed=5, device=DEV)
    rows = torch.tensor(w.file_rows.reshape(-1), dtype=torch.int32, device=DEV)
    scratch = torch.ones(1 << 26, device=DEV)
    side = torch.cuda.Stream()
    calls = [(lambda s: B.byz_multi_krum(X, d, idx, 5, 15, stream=s), B.byz_multi_krum_workspace_bytes(f)),
             (lambda s: B.byz_bulyan(X, d, idx, 5, stream=s), B.byz_bulyan_workspace_bytes(f)),
             (lambda s: B.byz_aggregate(w.X, d, rows, w.f, w.r, stream=s)[:2], B.byz_aggregate_workspace_bytes(w.f, w.r))]
    for call, nbytes in calls:
        want = call(None)
        for on in (side, side.cuda_stream):
            torch.cuda.synchronize()
            with torch.cuda.stream(side):
                _keep_busy(scratch)
            got = call(on)
            junk = [torch.full((nbytes,), 255, dtype=torch.uint8, device=DEV) for _ in range(4)]
            torch.cuda.synchronize()
            assert all(torch.equal(a, b) for a, b in zip(got, want)), (nbytes, on)
            del junk


def test_random_shapes_sizes_and_layouts():
    # a seeded sweep over assignments (every kernel family: generated, padded and 169-wire
    # networks, single pass and two-step, more than 64 files, r = 3, 5, 7), sizes, row pitches,
    # attacks and planted single-word differences; everything against the C oracle
    import math
    rng = np.random.default_rng(2010)
    shapes = [(MOLS, 5, 3), (MOLS, 7, 3), (MOLS, 7, 5), (RAM, 5, 5), (RAM, 3, 3), (RAM, 5, 3),
              (RAM, 7, 3), (RAM, 3, 5), (RAM, 3, 7), (RAM, 5, 7), (RAM, 7, 7), (RAM, 3, 9),
              (RAM, 3, 11), (RAM, 5, 9), (RAM, 5, 13), (MOLS, 9, 3), (MOLS, 11, 3), (MOLS, 13, 3),
              (MOLS, 9, 5), (FRC, 15, 3), (FRC, 25, 5), (FRC, 27, 3), (RAM, 3, 47), (RAM, 3, 85),
              (RAM, 7, 9)]
    attacks = [REVERSED, ALIE, CONST, MIXED]
    for case in range(150):
        scheme, a, b = shapes[rng.integers(len(shapes))]
        asg = B.byz_build_assignment(scheme, a, b)
        d = int(rng.choice([rng.integers(1, 20), rng.integers(20, 3000), rng.integers(3000, 60000)]))
        ld = d + int(rng.integers(0, 9))
        q = int(rng.integers(0, max(1, asg.K // 3)))
        while math.comb(asg.K, q) > 2_000_000:
            q -= 1
        attack = attacks[rng.integers(len(attacks))]
        w = W.make(scheme, a, b, q, d, attack, seed=int(rng.integers(1 << 30)), ld=ld, device=DEV)
        X = w.X.clone()
        for _ in range(int(rng.integers(0, 4))):
            X[int(w.file_rows[rng.integers(w.f), rng.integers(w.r)]), int(rng.integers(d))] += 1.0
        tag = (case, scheme, a, b, q, d, ld, attack["kind"])
        rows_dev = torch.tensor(w.file_rows.reshape(-1), dtype=torch.int32, device=DEV)
        Xh = X.cpu().numpy()
        wrep_o, wrow_o, neq_o = C.vote(Xh, w.file_rows, d)
        out_o = C.median(Xh, wrow_o, d)
        wrep, wrow, neq = B.byz_vote(X, d, rows_dev, w.f, w.r)
        assert np.array_equal(wrep.cpu().numpy(), wrep_o) and np.array_equal(W.bits(neq), neq_o), tag
        assert np.array_equal(W.bits(B.byz_median(X, d, wrow)), W.bits(out_o)), tag
        for flags in (0, B.BYZ_AGG_EARLY_MAJORITY):
            out, wrep2, _ = B.byz_aggregate_opts(X, d, rows_dev, w.f, w.r, flags)
            assert np.array_equal(W.bits(out), W.bits(out_o)), (tag, flags)
            assert np.array_equal(wrep2.cpu().numpy(), wrep_o), (tag, flags)
        trim = int(rng.integers(0, (w.f + 1) // 2))
        _trimmed_mean_check(X, wrow_o, d, trim, tag)
        out_t, _, _ = B.byz_aggregate_opts(X, d, rows_dev, w.f, w.r, B.BYZ_AGG_TRIM(trim))
        assert np.array_equal(W.bits(out_t), W.bits(B.byz_trimmed_mean(X, d, wrow, trim))), tag
        _tolerant_check(X, w.file_rows, d, w.f, w.r, 1e-6, 1e-5, tag)


@pytest.mark.parametrize("f", [3, 25, 26, 31, 32, 33, 40, 41, 64, 65, 96, 97, 128])
def test_multi_krum_mean_of_short_and_long_rows(f):
    # rows of up to 3 * 2^17 coordinates (fewer for many vectors, above all off the cache lines) are averaged in blocks
    # that choose for themselves: one word more and less than a block and than that limit, more chosen rows than are in
    # flight at once and fewer, rows off the cache lines.  Choice and mean from the scores the call returned: m lowest,
    # lower index first; fp32 additions in ascending index order.  NaN compares with nothing: every vector is chosen.
    rng = np.random.default_rng(f)
    off = 3 << 17 if f <= 25 else (5 << 16 if f <= 40 else 1 << 18)
    on = 3 << 17 if f <= 96 else 5 << 16
    for d, ld, nan in [(1, 6, False), (3, 8, False), (4, 9, False), (255, 260, False), (257, 262, True), (off, off + 5, False),
                       (off + 1, off + 6, False), (on, on, False), (on + 1, on + 32, False)]:
        X = torch.empty((f + 2, ld), device=DEV).normal_(generator=torch.Generator(device=DEV).manual_seed(f * 1000 + d % 997))
        idx = rng.permutation(f + 2)[:f].astype(np.int32)
        if nan:
            X[int(idx[f // 2]), 7] = float("nan")
        c = (f - 3) // 2
        for m in {1, f - c}:
            out = torch.full((d + 8,), 7.0, device=DEV)
            _, sel, scores, _ = B.byz_multi_krum(X, d, torch.tensor(idx, device=DEV), c, m, out=out)
            torch.cuda.synchronize()
            sc = scores.cpu().numpy()
            with np.errstate(invalid="ignore"):
                rank = [sum((sc[k] < sc[i]) or (sc[k] == sc[i] and k < i) for k in range(f)) for i in range(f)]
            want_sel = np.array([r < m for r in rank])
            assert np.array_equal(sel.cpu().numpy().astype(bool), want_sel), (f, d, m)
            acc = torch.zeros(d, device=DEV)
            for i in np.flatnonzero(want_sel):
                acc += X[int(idx[i]), :d]
            want = (acc / torch.tensor(float(want_sel.sum()), device=DEV)).cpu().numpy()
            assert np.array_equal(out[:d].cpu().numpy(), want, equal_nan=True), (f, d, m)
            assert bool((out[d:] == 7.0).all()), (f, d, m)


@pytest.mark.parametrize("f, c, m, d, ld", [(9, 2, 7, 22400003, 22400003), (16, 2, 14, 8400001, 8400032),
                                            (25, 5, 20, 5600001, 5600064), (32, 4, 28, 3800035, 3800035),
                                            (33, 5, 28, 5600002, 5600003), (49, 8, 41, 3900031, 3900064),
                                            (56, 8, 48, 3200033, 3200064), (64, 10, 54, 2800037, 2800040)])
def test_multi_krum_mean_taken_with_the_distances(f, c, m, d, ld):
    # rows long enough that the choice is guessed from a sample and averaged in the pass over all rows: guess right;
    # wrong, as a chosen row differs from what the sample shows in one word; wrong and infinite; not made, as rows are
    # alike; not made, as the output is one of the rows.  The words are those of one addition after the other
    # whichever way they came.
    gen = torch.Generator(device=DEV).manual_seed(f)
    X = torch.empty((f + 1, ld), device=DEV)
    idx = np.random.default_rng(f).permutation(f + 1)[:f].astype(np.int32)
    idx_dev = torch.tensor(idx, device=DEV)
    for kind in ("right", "wrong", "infinite", "alike", "in place"):
        for t, i in enumerate(idx):
            X[int(i)].normal_(generator=gen)
            if kind != "alike":
                X[int(i)].mul_(1.0 + 0.05 * t)
        first = int(idx[0])  # the smallest row, chosen unless the word is seen
        if kind == "wrong":
            X[first, d - 1] = 1e6
        elif kind == "infinite":
            X[first, d - 1] = float("inf")
        out = X[first] if kind == "in place" else torch.full((d + 8,), 7.0, device=DEV)
        kept = X[:, d - 1].clone()
        before = X[first].clone()
        _, sel, scores, _ = B.byz_multi_krum(X, d, idx_dev, c, m, out=out)
        torch.cuda.synchronize()
        sc = scores.cpu().numpy()
        with np.errstate(invalid="ignore"):
            rank = [sum((sc[k] < sc[i]) or (sc[k] == sc[i] and k < i) for k in range(f)) for i in range(f)]
        want_sel = np.array([r < m for r in rank])
        assert np.array_equal(sel.cpu().numpy().astype(bool), want_sel), (f, kind)
        assert want_sel[0] == (kind not in ("wrong", "infinite")) or kind in ("alike", "infinite"), (f, kind)
        acc = torch.zeros(d, device=DEV)
        for i in np.flatnonzero(want_sel):
            acc += (before if kind == "in place" and int(idx[i]) == first else X[int(idx[i])])[:d]
        want = acc / torch.tensor(float(want_sel.sum()), device=DEV)
        n = d - 8 if kind == "in place" else d  # (two threads write the last words of an odd row)
        assert bool(((out[:n] == want[:n]) | (torch.isnan(out[:n]) & torch.isnan(want[:n]))).all()), (f, kind)
        if kind != "in place":
            assert bool((out[d:] == 7.0).all()) and torch.equal(X[:, d - 1], kept), (f, kind)


@pytest.mark.parametrize("f, d, ld", [(25, 4000003, 4000003), (33, 4400003, 4400003), (40, 3700001, 3700002),
                                      (49, 3000001, 3000001), (49, 4300001, 4300003), (56, 2600003, 2600064),
                                      (56, 2600003, 2600005), (64, 2300001, 2300001), (64, 4300001, 4300001)])
def test_multi_krum_distances_do_not_depend_on_how_many_are_chosen(f, d, ld):
    # the order of the additions behind a distance follows from f, d, ld and the alignment: the same bits whether the
    # mean of many rows is taken in the pass over all of them or the mean of one row behind it, one or two stretches
    # at a time off the cache lines and on them
    X = torch.empty((f, ld), device=DEV).normal_(generator=torch.Generator(device=DEV).manual_seed(f))
    X.mul_(torch.linspace(0.5, 2.0, f, device=DEV).view(f, 1))
    idx = torch.arange(f, dtype=torch.int32, device=DEV)
    _, _, scores, dist = B.byz_multi_krum(X, d, idx, 0, 1)
    _, _, scores_m, dist_m = B.byz_multi_krum(X, d, idx, 0, f)
    assert torch.equal(dist.view(torch.int64), dist_m.view(torch.int64))
    assert torch.equal(scores.view(torch.int64), scores_m.view(torch.int64))


def _guess_of(workspace, f):
    """The vectors whose mean Multi-Krum's pass over all rows has taken, one bit each: the word before the partial sums."""
    nt = (f + 15) // 16
    at = B.byz_multi_krum_workspace_bytes(f) - 4 * 512 * (nt * (nt + 1) // 2) * 256 - 8
    return int(workspace[at:at + 8].cpu().numpy().view(np.uint64)[0])


@pytest.mark.parametrize("f, c, m, off", [(9, 2, 7, 3), (16, 2, 14, 0), (25, 5, 20, 0), (32, 4, 28, 1), (33, 5, 28, 0),
                                          (49, 8, 40, 3), (56, 8, 48, 1), (64, 10, 54, 5), (64, 10, 54, 0)])
def test_multi_krum_guess_is_made_where_it_is_sure(f, c, m, off):
    # which way a call on long rows goes: the mean taken with the distances (guess right), taken again (wrong), or not
    # guessed at, and one coordinate below the rule's first length no guess at all; the words are the same, those of
    # the distances too
    gen = torch.Generator(device=DEV).manual_seed(f)
    d = max(-(-350000000 // (f + m)), -(-((1 << 26) if f <= 32 else (3 << 25)) // (m - 2 - f // 4)))
    X = torch.empty((f, (d + 127) // 64 * 64 + off), device=DEV)
    idx = torch.arange(f, dtype=torch.int32, device=DEV)
    ws = torch.empty(B.byz_multi_krum_workspace_bytes(f), dtype=torch.uint8, device=DEV)
    out = torch.empty(d, device=DEV)

    def call(n):
        ws.fill_(0xA5)
        _, sel, scores, dist = B.byz_multi_krum(X, n, idx, c, m, out=out, workspace=ws)
        chosen = sum(1 << i for i, v in enumerate(sel.cpu().tolist()) if v)
        guess = _guess_of(ws, f)
        acc = torch.zeros(n, device=DEV)
        for i in range(f):
            if (chosen >> i) & 1:
                acc += X[i, :n]
        want = acc / torch.tensor(float(m), device=DEV)
        assert torch.equal(out[:n].view(torch.int32), want.view(torch.int32)), (f, n)
        _, _, scores_one, dist_one = B.byz_multi_krum(X, n, idx, c, 1, out=out, workspace=ws)
        assert torch.equal(scores, scores_one) and torch.equal(dist, dist_one), (f, n)
        return guess, chosen

    for i in range(f):
        X[i].normal_(generator=gen).mul_(1.0 + 0.05 * i)
    guess, chosen = call(d)
    assert guess == chosen == (1 << m) - 1
    assert call(d - 1) == (0xA5A5A5A5A5A5A5A5, chosen)
    X[0, d - 1] = 1e6  # not in the sample
    guess, chosen = call(d)
    assert guess == (1 << m) - 1 and chosen == (1 << (m + 1)) - 2
    X[0].copy_(X[1])  # every vector alike but for their last word
    for i in range(1, f):
        X[i].copy_(X[0])
        X[i, d - 1] = float(i)
    assert call(d)[0] == 0
    for i in range(f):  # one distribution, whose scores differ by less than a sample can tell
        X[i].normal_(generator=gen)
    assert call(d)[0] == 0


def test_multi_krum_guess_knows_uneven_coordinates():
    # coordinates of very different scale, as the layers of a network have: a few of them make the scores, and a sample tells
    # little.  A guess by a fixed margin of 0.2 % is made, and wrong, in nine calls of ten.
    f, c, m, d = 25, 5, 20, 7800000
    idx = torch.arange(f, dtype=torch.int32, device=DEV)
    ws = torch.empty(B.byz_multi_krum_workspace_bytes(f), dtype=torch.uint8, device=DEV)
    X = torch.empty((f, d), device=DEV)
    wrong = 0
    for seed in range(8):
        gen = torch.Generator(device=DEV).manual_seed(seed)
        scale = torch.rand(f, generator=gen, device=DEV) * 0.2 + 0.9
        uneven = torch.randn(d, generator=gen, device=DEV).mul_(2.0).exp_()
        for i in range(f):
            X[i].normal_(generator=gen).mul_(uneven).mul_(scale[i])
        _, sel, _, _ = B.byz_multi_krum(X, d, idx, c, m, workspace=ws)
        chosen = sum(1 << i for i, v in enumerate(sel.cpu().tolist()) if v)
        wrong += _guess_of(ws, f) not in (0, chosen)
    assert wrong <= 1  # one in forty is to be expected


def test_multi_krum_and_bulyan_for_every_f():
    # every f from 3 to 64 and a spread of the wider ones (all tile counts and staging shapes of
    # the Gram kernel, one and two distances per lane in the row sort, Bulyan's rounds in
    # registers and in LDS, every network size of its second phase incl. the spare-wire cases),
    # random d, row pitch, c and m; per-row scales keep
    # the scores apart, so selections are compared exactly
    rng = np.random.default_rng(64)
    compared = []
    for f in list(range(3, 65)) + [65, 66, 80, 81, 84, 85, 96, 97, 112, 113, 121, 123, 127, 128]:
        d = int(rng.choice([rng.integers(1, 10), rng.integers(10, 600), rng.integers(600, 40000)]))
        ld = d + int(rng.integers(0, 6))
        Xh = np.zeros((f + 2, ld), dtype=np.float32)
        Xh[:, :d] = (rng.standard_normal((f + 2, d)) * rng.uniform(0.5, 2.0, size=(f + 2, 1))).astype(np.float32)
        idx = rng.permutation(f + 2)[:f].astype(np.int32)
        c = int(rng.integers(0, (f - 3) // 2 + 1))
        n_far = int(rng.integers(0, c + 1))
        Xh[idx[:n_far], :d] = (30.0 * rng.standard_normal((n_far, d))).astype(np.float32)
        X = torch.tensor(Xh, device=DEV)
        m = int(rng.integers(1, f - c + 1))
        _multi_krum_check(X, idx, d, c, m, (f, d, ld, c, m))
        if f % 2 == 1:
            cb = int(rng.integers(0, (f - 3) // 4 + 1))
            compared.append(_bulyan_check(X, idx, d, cb, (f, d, ld, cb)))
    assert sum(compared) >= len(compared) - 2, compared
    # one vector too many
    X = torch.zeros((B.BYZ_MAX_F_KRUM + 1, 8), device=DEV)
    too_many = torch.arange(B.BYZ_MAX_F_KRUM + 1, dtype=torch.int32, device=DEV)
    for call in (lambda: B.byz_multi_krum(X, 8, too_many, 1, 1), lambda: B.byz_bulyan(X, 8, too_many, 1)):
        with pytest.raises(B.ByzError) as e:
            call()
        assert e.value.code == -1

"""Build step: writes the compare-exchange lists the median kernels unroll.

The coordinate-wise median of f values (Sec. 2 and Sec. 6.1 of the ByzShield
paper: the aggregation applied to the f vote winners) is computed per thread
by a fixed network held in registers.  This script derives the network;
nothing is typed in by hand.

gfx950 has minimum, median and maximum of three operands as single
instructions, so putting three wires in order costs three instructions, as
much per wire as a two-wire comparator costs (two instructions) while it
settles log2(6)/3 instead of 1/2 bit per instruction.  The networks are built
for that machine:

  1. Sort: the wires are split into two or three blocks, each sorted
     recursively, and the sorted blocks merged.  Which split, by counting
     instructions of every candidate (`best_split`).
  2. Two sorted lists are merged by Batcher's odd-even merge.
  3. Three sorted lists A, B, C are merged three ways: D merges the elements
     0, 3, 6, .. of each list, E the elements 1, 4, 7, .., F the elements
     2, 5, 8, .. .  On 0/1 inputs, with z zeros a list gives ceil(z/3),
     ceil((z-1)/3), ceil((z-2)/3) of them to D, E, F, so the zeros of D
     exceed those of F by x <= 3 and those of E exceed those of F by y <= x:
     ten cases.  In the order D0 E0 F0 D1 E1 F1 .. sorting the triples
     (F[i-1], E[i], D[i+1]) settles every case but x = 2, y = 1, and the pairs
     (F[i], D[i+1]) after it settle that one.
  4. Walking backwards from the wanted outputs, outputs that cannot influence
     them are dropped (the median needs one wire).

81 wires cost 998 instructions to sort (Batcher's sort of two-wire
comparators: 1720) and 646 to select the median (1324).

The programs are written with BYZ_S_SORT3(i,j,k,lo,mid,hi) (three wires, which
of the outputs are needed), BYZ_S_CE(i,j) (two wires, both outputs),
BYZ_S_CE_LO(i,j) (min -> wire i) and BYZ_S_CE_HI(i,j) (max -> wire j).
"""
import functools
import os
import sys

DEPTHS = (1, 2, 3, 4, 5, 8, 20)  # prefetch distances the streamed programs carry load steps for


def _merge(wires):
    n = len(wires)
    if n == 2:
        return [(wires[0], wires[1])]
    ces = _merge(wires[0::2]) + _merge(wires[1::2])
    ces += [(wires[i], wires[i + 1]) for i in range(1, n - 1, 2)]
    return ces


def _sort(wires):
    n = len(wires)
    if n == 1:
        return []
    return _sort(wires[:n // 2]) + _sort(wires[n // 2:]) + _merge(wires)


def batcher_sort(n):
    """Comparators (i, j), i < j: min goes to wire i, max to wire j.  n a power of two.  The
    two-wire reference the host-side tests hold the networks below against."""
    assert n >= 1 and n & (n - 1) == 0
    return _sort(list(range(n)))


END = None  # stands for a value above every key, behind the end of a list


def _put_in_order(sorters, columns):
    """Sorts what the places `columns` (pairs of a list and an index, first place first) hold:
    appends the sorter and moves the wires; the lowest wire takes the lowest value."""
    wires = sorted(c[i] for c, i in columns if c[i] is not END)
    if len(wires) > 1:
        sorters.append(tuple(wires))
    wires += [END] * (len(columns) - len(wires))
    for (c, i), w in zip(columns, wires):
        c[i] = w


def merge_two(sorters, a, b):
    """Merges two sorted lists of wires; -> the sorted list.  Appends the sorters it takes."""
    if not a or not b:
        return list(a) + list(b)
    if len(a) == len(b) == 1:
        out = [a[0], b[0]]
        _put_in_order(sorters, [(out, 0), (out, 1)])
        return out
    d = merge_two(sorters, a[0::2], b[0::2])
    e = merge_two(sorters, a[1::2], b[1::2])
    n = max(len(d), len(e) + 1)
    d += [END] * (n - len(d))
    e += [END] * (n - len(e))
    for i in range(n - 1):
        _put_in_order(sorters, [(e, i), (d, i + 1)])
    return [x for pair in zip(d, e) for x in pair][:len(a) + len(b)]


def merge_three(sorters, a, b, c):
    """Merges three sorted lists of wires (item 3 above)."""
    a, b, c = sorted((a, b, c), key=len, reverse=True)
    if not c:
        return merge_two(sorters, a, b)
    if len(a) == 1:
        out = [a[0], b[0], c[0]]
        _put_in_order(sorters, [(out, 0), (out, 1), (out, 2)])
        return out
    d, e, f = (merge_three(sorters, a[k::3], b[k::3], c[k::3]) for k in range(3))
    n = len(d) + 1
    for part in (d, e, f):
        part += [END] * (n - len(part))
    for i in range(n):
        triple = [(f, i - 1)] if i > 0 else []
        triple.append((e, i))
        if i + 1 < n:
            triple.append((d, i + 1))
        _put_in_order(sorters, triple)
    for i in range(n - 1):
        _put_in_order(sorters, [(f, i), (d, i + 1)])
    return [x for row in zip(d, e, f) for x in row][:len(a) + len(b) + len(c)]


def merge_blocks(sorters, blocks):
    return (merge_two if len(blocks) == 2 else merge_three)(sorters, *blocks)


def _consecutive(sizes):
    starts = [sum(sizes[:k]) for k in range(len(sizes))]
    return [list(range(s, s + m)) for s, m in zip(starts, sizes)]


@functools.lru_cache(None)
def merge_cost(sizes):
    """Instructions it takes to merge sorted blocks of these sizes."""
    sorters = []
    merge_blocks(sorters, _consecutive(sizes))
    return sum(len(s) for s in sorters)


@functools.lru_cache(None)
def best_split(n):
    """-> (instructions, block sizes) of the cheapest sort of n wires found: blocks of equal size
    (one more in the first ones), or equal ones and a smaller or larger last one."""
    if n <= 3:
        return (n if n > 1 else 0), (1,) * n
    best = None
    for k in (2, 3):
        q, rem = divmod(n, k)
        candidates = {(q + 1,) * rem + (q,) * (k - rem)}
        for a in range(max(1, q - 6), q + 14):
            last = n - a * (k - 1)
            if last >= 1:
                candidates.add(tuple(sorted((a,) * (k - 1) + (last,), reverse=True)))
        for sizes in sorted(candidates, reverse=True):  # of equals, the smallest last block
            cost = sum(best_split(m)[0] for m in sizes) + merge_cost(sizes)
            if best is None or cost < best[0]:
                best = (cost, sizes)
    return best


def _sort_wires(sorters, wires):
    if len(wires) == 1:
        return wires
    sizes = best_split(len(wires))[1]
    return merge_blocks(sorters, [_sort_wires(sorters, [wires[i] for i in part])
                                  for part in _consecutive(sizes)])


def _needed_part(sorters, needed):
    """Drops what cannot influence the wires `needed`; -> [(wires, which outputs are needed)]."""
    needed, kept = set(needed), []
    for wires in reversed(sorters):
        outputs = tuple(w in needed for w in wires)
        if any(outputs):
            kept.append((wires, outputs))
            needed.update(wires)
    kept.reverse()
    return kept


def _sort_blocks(f, sizes):
    sorters = []
    out = merge_blocks(sorters, [_sort_wires(sorters, part) for part in _consecutive(sizes)])
    assert out == list(range(f))  # every sorter leaves sorted wires alone
    return sorters


def _shares(f, sorters):
    """Per sorter, the file whose value completes its inputs, if wire j's value comes with file j."""
    ready, share = list(range(f)), []
    for wires, _ in sorters:
        t = max(ready[w] for w in wires)
        share.append(t)
        for w in wires:
            ready[w] = t
    return share


def most_live(f, sorters):
    """Most wires alive at once when every sorter runs as soon as the file that completes it is in."""
    dropped = [0] * f
    for (_, outputs), t in zip(sorters, _shares(f, sorters)):
        dropped[t] += outputs.count(False)
    live = peak = 0
    for n in dropped:
        peak = max(peak, live + 1)
        live += 1 - n
    return peak


# block sizes tried for a median's last merge, besides the remainder
BLOCKS = (3, 5, 7, 9, 11, 13, 15, 17, 18, 19, 21, 25, 27, 30, 33, 36, 39, 43, 45, 51, 54, 57, 63, 81)


def _median_part(f, sizes):
    return _needed_part(_sort_blocks(f, sizes), [(f - 1) // 2])


@functools.lru_cache(None)
def median_blocks(f):
    """Sizes of the blocks the median of f wires merges last, decided by what is left after
    dropping, an instruction counting as much as half a live wire: fewer live wires are fewer
    registers (25 files in the single pass: 9 + 9 + 7 needs 23 keys at a time, 9 + 8 + 8 all 25,
    which costs a quarter of the resident waves)."""
    candidates = {best_split(f)[1]}
    if f >= 4:
        for a in BLOCKS:
            for b in BLOCKS:
                if b <= a and a < f <= 3 * a and 0 <= f - a - b <= b:
                    candidates.add(tuple(m for m in (a, b, f - a - b) if m))
    best = None
    for sizes in sorted(candidates):
        sorters = _median_part(f, sizes)
        score = op_count(sorters) + 2 * most_live(f, sorters)
        if best is None or score < best[0]:
            best = (score, sizes)
    return best[1]


@functools.lru_cache(None)
def sorters_for(f, full_sort=False):
    """The network on wires 0..f-1 as sorters (wires ascending, which outputs are needed): after
    it wire i holds the element of rank i, or (full_sort false) wire (f-1)/2 the median."""
    if full_sort:
        return _needed_part(_sort_blocks(f, best_split(f)[1]), range(f))
    return _median_part(f, median_blocks(f))


def comparators(wires, outputs):
    """A sorter as two-wire comparators (i, j, need_lo, need_hi)."""
    if len(wires) == 2:
        return [wires + outputs]
    (a, b, c), (lo, mid, hi) = wires, outputs
    if not mid and not hi:
        return [(b, c, True, False), (a, b, True, False)]
    if not lo and not mid:
        return [(a, b, False, True), (b, c, False, True)]
    return [(a, b, True, True), (b, c, True, hi), (a, b, lo, mid)]


def op_count(sorters):
    """Instructions of a network: one per needed output."""
    return sum(sum(outputs) for _, outputs in sorters)


def best_network(f, full_sort=False):
    """-> (comparators (i, j, need_lo, need_hi) on wires 0..f-1, median wire)."""
    ops = [ce for wires, outputs in sorters_for(f, full_sort) for ce in comparators(wires, outputs)]
    return ops, (f - 1) // 2


def apply_network(ops, values):
    """Reference execution on a Python list (used by the host-side tests)."""
    v = list(values)
    for (i, j, lo, hi) in ops:
        a, b = v[i], v[j]
        if lo:
            v[i] = a if a <= b else b
        if hi:
            v[j] = b if a <= b else a
    return v


def emit(f, path):
    ops, wire = best_network(f)
    with open(path, "w") as fh:
        fh.write("// generated by gen_selnet.py: median selection network, f = %d, "
                 "%d two-wire comparators\n" % (f, len(ops)))
        for (i, j, lo, hi) in ops:
            name = "BYZ_CE" if (lo and hi) else ("BYZ_CE_LO" if lo else "BYZ_CE_HI")
            fh.write("%s(%d,%d)\n" % (name, i, j))
        fh.write("BYZ_MEDIAN_WIRE(%d)\n" % wire)
    return len(ops)


# Sorting programs whose long shares are pinned every so many sorters, not only at their end.  The
# share of the last of 169 files holds 608 sorters; left to itself the compiler draws them together
# until the single pass needs more than the 256 registers of two waves per SIMD and spills 18 (4 M
# coordinates of 169 x 3 copies, trimmed mean: 1429 us, early-majority mode 1182).  With pins it takes
# 247 and spills none: 1314 / 1093; every 16, 32 or 48 sorters is the same to 0.2 %.
SORTERS_BETWEEN_PINS = {169: 48}


def streamed_sorters(f, full_sort=False):
    """The network of best_network(f, full_sort), ordered for a kernel that receives wire j's value
    when it loads file j: every sorter is placed right after the last file it depends on.

    Returns a list of ("load", depth, j) / ("step", j) / ("use", j) / ("sort", wires, outputs) /
    ("pin", w) / ("median", w) steps; ("step", j) marks the start of file j's share of the
    program and ("pin", w) follows the sorters of that share for every wire they changed (a
    kernel may pin its instruction schedule there; the sorting programs of SORTERS_BETWEEN_PINS have
    them inside long shares too): the loads of file j+depth are issued before
    use(j), so that the next file(s) are in flight while file j's compares and the sorters it
    unblocks execute.  Load steps are listed for every depth in DEPTHS; a consumer follows one
    of them.
    """
    sorters = sorters_for(f, full_sort)
    when = _shares(f, sorters)
    prog = [("load", depth, j) for depth in DEPTHS for j in range(min(depth, f))]
    for j in range(f):
        prog.append(("step", j))
        # a kernel prefetching `depth` files ahead issues the ("load", depth, .) steps only
        for depth in DEPTHS:
            if j + depth < f:
                prog.append(("load", depth, j + depth))
        prog.append(("use", j))
        touched, since = [], 0
        for (wires, outputs), t in zip(sorters, when):
            if t == j:
                if full_sort and since == SORTERS_BETWEEN_PINS.get(f):
                    prog += [("pin", w) for w in touched]
                    touched, since = [], 0
                prog.append(("sort", wires, outputs))
                since += 1
                for w, needed in zip(wires, outputs):
                    if needed and w not in touched:
                        touched.append(w)
        # wires that changed in file j's share: a kernel may force them to be computed here
        for w in touched:
            prog.append(("pin", w))
    prog.append(("sorted", f) if full_sort else ("median", (f - 1) // 2))
    return prog


def streamed_program(f, full_sort=False):
    """The same steps with every sorter as its two-wire comparators, ("ce", i, j, lo, hi)."""
    prog = []
    for step in streamed_sorters(f, full_sort):
        prog += [("ce",) + ce for ce in comparators(*step[1:])] if step[0] == "sort" else [step]
    return prog


def run_streamed(prog, values, depth=1):
    """Reference execution of a streamed program on a Python list (host-side tests)."""
    v = [None] * len(values)
    loaded = set()
    for step in prog:
        if step[0] == "load":
            if step[1] == depth:
                loaded.add(step[2])
        elif step[0] in ("step", "pin"):
            pass
        elif step[0] == "use":
            assert step[1] in loaded
            v[step[1]] = values[step[1]]
        elif step[0] == "ce":
            _, i, j, lo, hi = step
            a, b = v[i], v[j]
            assert a is not None and b is not None
            if lo:
                v[i] = a if a <= b else b
            if hi:
                v[j] = b if a <= b else a
        elif step[0] == "sorted":
            return v
        else:
            return v[step[1]]


def sorter_line(wires, outputs):
    if len(wires) == 3:
        return "BYZ_S_SORT3(%d,%d,%d,%d,%d,%d)\n" % (wires + outputs)
    name = "BYZ_S_CE" if all(outputs) else ("BYZ_S_CE_LO" if outputs[0] else "BYZ_S_CE_HI")
    return "%s(%d,%d)\n" % ((name,) + wires)


def emit_streamed(f, path, full_sort=False):
    """Writes the program; -> instructions of the network after the last file is in."""
    text = {"load": "BYZ_S_LOAD%d(%d)\n", "step": "BYZ_S_STEP(%d)\n", "pin": "BYZ_S_PIN(%d)\n",
            "use": "BYZ_S_USE(%d)\n", "sorted": "BYZ_S_SORTED(%d)\n", "median": "BYZ_S_MEDIAN(%d)\n"}
    last_share = 0
    with open(path, "w") as fh:
        fh.write("// generated by gen_selnet.py: %s network for f = %d interleaved with the "
                 "file loop\n" % ("sorting" if full_sort else "median", f))
        for step in streamed_sorters(f, full_sort):
            if step[0] == "sort":
                fh.write(sorter_line(*step[1:]))
                last_share += sum(step[2])
            else:
                fh.write(text[step[0]] % step[1:])
            if step[0] == "use":
                last_share = 0
    return last_share


SIZES = (3, 5, 7)  # medians of fewer rows than the streamed programs start at
# sizes with a median program: the paper's file counts (l^2 for MOLS and Ramanujan Case 1, m*s for
# Case 2) and sizes between them, so that any other f has at most a fifth of spare wires
STREAMED_SIZES = (9, 15, 21, 25, 31, 35, 41, 49, 57, 63, 65, 73, 81, 97, 109, 121, 137, 153, 169)
# full-sort programs (trimmed mean, second phase of Bulyan); 96, 112 and 128 wires sort each half
# of the rows in the median and the trimmed mean of more than 169 rows
SORT_SIZES = (9, 15, 21, 25, 31, 35, 41, 49, 57, 63, 65, 73, 81, 96, 97, 109, 112, 121, 128, 137,
              153, 169)


def main(outdir):
    os.makedirs(outdir, exist_ok=True)
    for f in SIZES:
        n_ce = emit(f, os.path.join(outdir, "selnet_%d.inc" % f))
        print("selnet f=%d: %d comparators" % (f, n_ce))
    # chains "if constexpr (F == f) { #include <program for f> } else ..." over the streamed sizes
    for stem, sizes in (("selnet_stream", STREAMED_SIZES), ("selnet_sort_stream", SORT_SIZES)):
        with open(os.path.join(outdir, stem + "_dispatch.inc"), "w") as fh:
            fh.write("// generated by gen_selnet.py: picks the streamed program for template parameter F\n")
            for n, f in enumerate(sizes):
                fh.write("%sif constexpr (F == %d) {\n#include \"%s_%d.inc\"\n}" %
                         ("" if n == 0 else " else ", f, stem, f))
            fh.write(" else {\n    static_assert(F < 0, \"no streamed network generated for this f\");\n}\n")
    for f in STREAMED_SIZES:
        tail = emit_streamed(f, os.path.join(outdir, "selnet_stream_%d.inc" % f))
        print("selnet_stream f=%d: %d instructions, %d after the last file"
              % (f, op_count(sorters_for(f)), tail))
    for f in SORT_SIZES:
        tail = emit_streamed(f, os.path.join(outdir, "selnet_sort_stream_%d.inc" % f), True)
        print("selnet_sort_stream f=%d: %d instructions, %d after the last file"
              % (f, op_count(sorters_for(f, True)), tail))


if __name__ == "__main__":
    main(sys.argv[1] if len(sys.argv) > 1 else
         os.path.join(os.path.dirname(os.path.abspath(__file__)), "generated"))

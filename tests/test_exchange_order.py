"""What the workgroups of a whole-iteration kernel exchange while they run: every read sees the version it means to see, whatever
the workgroups' relative speed.

The steps of a workgroup and the barriers between them are taken from the kernel's source in their order; steps between two barriers count as
unordered (different waves make them).  Across workgroups a step is ordered behind another one only by what the kernel waits for: partial
logits with the iteration's ticket (all workgroups of a worker) and arrivals (the same workgroup of all workers).  In that partial order a read has to
lie behind the write of its version and ahead of the write that replaces it."""
import itertools
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2009_05766_amd", "csrc")
STEPS = {
    "arrive": r"fetch_add\(p\.rows_count",
    "post": r"__hip_atomic_store\((?:p\.)?words",
    "poll": r">> 32\) == ticket",
    "await": r"await_arrivals\(p\.rows_count",
    "read rows": r"\bxp\[v\] = __hip_atomic_load\(at_bytes\(Xcur|\brequest_peer\(strip\);",
    "write rows": r"store_row\(at_bytes\(Xnext, own|__hip_atomic_store\(at_bytes\(Xnext, w1_next",
    "read first bias": r"MAX_C\] = .*p\.x_first|\? (?:Xcur \+ tiled_offset|at_bytes\(Xcur \+ shift)",
    "read bias copy": r"p\.biases \+ \(\(\(size_t\)cur",
    "write bias copy": r"p\.biases \+ \(\(\(size_t\)nxt",
    "write bias": r"store_row\((?:Xnext \+ bias_own|at_bytes\(Xnext, b2_at)",
}


def _segments(source):
    """Step -> number of barriers of the iteration's loop above it (-1: above the loop)."""
    loop = source.index("    for (int it = 0; it < ")
    barriers = [m.start() for m in re.finditer(r"^        __syncthreads\(\);", source, re.M) if m.start() > loop]
    assert re.search(r"stores_arrived\(\);[^\n]*\n        __syncthreads\(\);\n[^\n]*fetch_add\(p\.rows_count", source), "arrival behind the stores"
    found = {}
    for step, pattern in STEPS.items():
        at = [m.start() for m in re.finditer(pattern, source)]
        assert len(at) == 1, (step, at)
        found[step] = -1 if at[0] < loop else sum(b < at[0] for b in barriers)
    return found, len(barriers) + 1


def _conflicts(found, n_segments, workers, parts, iters):
    """Pairs (read, write) of one cell that nothing puts into the order they need."""
    groups = list(itertools.product(range(workers), range(parts)))
    when = lambda step, it: found[step] if found[step] < 0 else it * n_segments + found[step]      # place in the workgroup's own sequence
    behind = {}                                                          # (group, place) -> (group, place) of which it is waited for there
    for (i, s), it in itertools.product(groups, range(iters)):
        behind.setdefault((i, s, when("poll", it)), []).extend((i, q, when("post", it)) for q in range(parts))
        if it > 0:
            behind.setdefault((i, s, when("await", it)), []).extend((j, s, when("arrive", it)) for j in range(workers))
    last = iters * n_segments

    # known[g][place][h]: the latest place of h that is complete before g leaves `place`.  A segment's steps are complete behind it only, but a step
    # that was waited for is; what was complete ahead of it is everything known in the segments above it.
    known = {g: {p: {} for p in range(-2, last + 1)} for g in groups}

    def at(g, place):                                                    # known to g when it begins the segment `place`
        return known[g][place - 1] if place >= 0 else {}
    changed = True
    while changed:
        changed = False
        for g in groups:
            for p in range(-1, last + 1):
                merged = dict(known[g][p - 1])
                for (j, q, place) in behind.get((*g, p), []):
                    for h, v in at((j, q), place).items():
                        merged[h] = max(merged.get(h, -2), v)
                    if (j, q) != g:
                        merged[(j, q)] = max(merged.get((j, q), -2), place - 1)
                merged[g] = p
                if merged != known[g][p]:
                    known[g][p] = merged
                    changed = True
    ordered = lambda a, pa, b, pb: (pa < pb) if a == b else at(b, pb).get(a, -2) >= pa

    writes, reads = {}, []                                               # cell -> [(version, group, place)]; (cell, version, group, place)
    for i, s in groups:
        g = (i, s)
        for it in range(iters):
            writes.setdefault(("rows", (it + 1) % 2, i, s), []).append((it + 1, g, when("write rows", it)))
            writes.setdefault(("copy", (it + 1) % 2, i, s), []).append((it + 1, g, when("write bias copy", it)))
            if s == parts - 1:
                writes.setdefault(("bias", (it + 1) % 2, i), []).append((it + 1, g, when("write bias", it)))
            for m in range(workers):
                reads.append((("rows", it % 2, m, s), it, g, when("read rows", it)))
                if it == 0:
                    reads.append((("bias", 0, m), 0, g, when("read first bias", 0)))
                else:
                    reads.append((("copy", it % 2, m, s), it, g, when("read bias copy", it)))
        reads.append((("bias", 0, i), 0, g, -1))                         # its own, above the loop
        reads.append((("rows", 0, i, s), 0, g, -1))
    bad = []
    for cell, version, g, place in reads:
        for w_version, h, w_place in writes.get(cell, []):
            fine = ordered(h, w_place, g, place) if w_version <= version else ordered(g, place, h, w_place)
            if not fine:
                bad.append((cell, version, g, w_version, h))
    # partial logits: the words of iteration it are read before those of it + 2 replace them
    for (i, s), q, it in itertools.product(groups, range(parts), range(iters - 2)):
        if not ordered((i, q), when("poll", it), (i, s), when("post", it + 2)):
            bad.append((("words", it % 2, i, s), it, (i, q), it + 2, (i, s)))
    return bad


@pytest.mark.parametrize("name", ["k_sliced_iter.hip", "k_resident_mlp.hip"])
@pytest.mark.parametrize("workers,parts,iters", [(2, 1, 5), (2, 2, 5), (3, 3, 4)])
def test_reads_see_their_version(name, workers, parts, iters):
    with open(os.path.join(CSRC, name)) as f:
        found, n_segments = _segments(f.read())
    assert _conflicts(found, n_segments, workers, parts, iters) == []


@pytest.mark.parametrize("change", [{"read first bias": 1}, {"write rows": 0}, {"await": 2}])
def test_the_order_is_needed(change):
    """The same check on a sequence with one step moved: the peer's first bias asked for behind the partial logits, rows written ahead of the wait
    for arrivals, that wait beside the reads."""
    with open(os.path.join(CSRC, "k_sliced_iter.hip")) as f:
        found, n_segments = _segments(f.read())
    assert _conflicts({**found, **change}, n_segments, 2, 2, 4) != []

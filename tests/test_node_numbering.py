"""The numbering of a unit's nodes, on the host.

The kernels that refine below the roots append a unit's nodes in whatever order
they come to them, with their depth, and one pass numbers them at the end: the
starts of each depth as a 128-bit mask, a node's place by the population counts
of the depths above and of the starts before its own, its first child the node
of the depth below that starts where it does, its parent the last node of the
depth above that starts at or before it.  This model of that pass, fed with the
nodes of random trees in random order, must give the table of a sequential
breadth-first build: the same (start, length, first child, parent, child count)
at every index; slots of 1 to 128 tokens, chains down to depth 127 among them."""
import random


def _decide(a, n, rnd, chain):
    if n == 2:
        return [(0, 1), (1, 1)]
    if chain is not None:                       # peel one token: 0 from the left, 1 from the right
        return [(0, 1), (1, n - 1)] if chain == 0 else [(0, n - 1), (n - 1, 1)]
    if rnd.random() < 0.7:
        x = rnd.randint(1, n - 1)
        return [(0, x), (x, n - x)]
    p = rnd.randint(0, n - 1)                   # an extracted token
    kids = [(0, p)] if p > 0 else []
    kids.append((p, 1))
    if p + 1 < n:
        kids.append((p + 1, n - p - 1))
    return kids


def _breadth_first(n, rnd, stop, chain):
    """The table of a breadth-first build; ``stop``: the share of nodes left unrefined."""
    nodes = [dict(a=0, n=n, child=-1, parent=-1, nch=0, depth=0)]
    head = 0
    while head < len(nodes):
        nd = nodes[head]
        if nd["n"] >= 2 and rnd.random() >= stop:
            kids = _decide(nd["a"], nd["n"], rnd, chain)
            nd.update(child=len(nodes), nch=len(kids))
            nodes += [dict(a=nd["a"] + ka, n=kn, child=-1, parent=head, nch=0, depth=nd["depth"] + 1) for ka, kn in kids]
        head += 1
    return nodes


def _number(appended):
    """(depth, start) ranks from one mask of starts per depth."""
    depths = max(x["depth"] for x in appended) + 1
    mask = [0] * (depths + 1)
    for x in appended:
        assert not mask[x["depth"]] >> x["a"] & 1          # the nodes of a depth are disjoint
        mask[x["depth"]] |= 1 << x["a"]
    count = lambda m: bin(m).count("1")                     # noqa: E731
    first = [0]
    for m in mask:
        first.append(first[-1] + count(m))
    below = lambda d, p: count(mask[d] & ((1 << p) - 1))    # noqa: E731
    out = [None] * len(appended)
    for x in appended:
        d, a = x["depth"], x["a"]
        i = first[d] + below(d, a)
        assert out[i] is None
        out[i] = (a, x["n"], first[d + 1] + below(d + 1, a) if x["nch"] else -1,
                  first[d - 1] + below(d - 1, a + 1) - 1 if d else -1, x["nch"])
    return out


def _check(n, rnd, stop, chain=None):
    table = _breadth_first(n, rnd, stop, chain)
    appended = [dict(a=x["a"], n=x["n"], depth=x["depth"], nch=x["nch"]) for x in table]
    rnd.shuffle(appended)
    assert _number(appended) == [(x["a"], x["n"], x["child"], x["parent"], x["nch"]) for x in table]
    assert len(table) <= 2 * n - 1
    return max(x["depth"] for x in table)


def test_ranks_by_depth_and_start_are_breadth_first():
    rnd = random.Random(1)
    for _ in range(400):
        _check(rnd.randint(1, 128), rnd, rnd.choice([0.0, 0.0, 0.2, 0.5]))
    for n in (1, 2, 3, 16, 17, 32, 33, 64, 65, 127, 128):
        _check(n, rnd, 0.0)


def test_chains_reach_the_greatest_depth():
    rnd = random.Random(2)
    for side in (0, 1):
        assert _check(128, rnd, 0.0, chain=side) == 127

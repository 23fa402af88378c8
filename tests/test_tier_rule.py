"""The tier path's rule for "the cost matrix is a tree of tiers" (each row
against the row of its set's lowest rank, then labels and counts) against the
definition (ranks within each cost form a partition), over every small matrix."""
import itertools


def _rule(C):
    R = len(C)
    rows = []
    for i in range(R):
        costs = sorted({C[i][j] for j in range(R) if j != i})
        rows.append([(c, frozenset([i] + [j for j in range(R) if j != i and C[i][j] <= c])) for c in costs])
    for i in range(R):
        for c, near in rows[i][:-1]:
            x = min(near)
            if x != i and frozenset([x] + [j for j in range(R) if j != x and C[x][j] <= c]) != near:
                return False
    for c in sorted({c for row in rows for c, _ in row})[:-1]:
        sets = [([frozenset([i])] + [s for cost, s in rows[i] if cost <= c])[-1] for i in range(R)]
        low = [min(s) for s in sets]
        if any(low[low[i]] != low[i] or low.count(low[i]) != len(sets[i]) for i in range(R)):
            return False
    return True


def _is_tree(C):
    R = len(C)
    for c in {C[i][j] for i in range(R) for j in range(R) if i != j}:
        near = [frozenset(j for j in range(R) if j == i or C[i][j] <= c) for i in range(R)]
        if any(near[j] != near[i] for i in range(R) for j in near[i]):
            return False
    return True


def test_rule_is_the_definition():
    trees = 0
    for R, values in ((2, 4), (3, 4), (4, 2)):
        for e in itertools.product(range(values), repeat=R * (R - 1)):
            it = iter(e)
            C = [[0 if i == j else next(it) for j in range(R)] for i in range(R)]
            assert _rule(C) == _is_tree(C), C
            trees += _is_tree(C)
    assert trees > 20  # both outcomes occur


def test_rule_on_four_ranks_with_three_costs():
    for n, e in enumerate(itertools.product(range(3), repeat=12)):
        if n % 7:
            continue
        it = iter(e)
        C = [[0 if i == j else next(it) for j in range(4)] for i in range(4)]
        assert _rule(C) == _is_tree(C), C

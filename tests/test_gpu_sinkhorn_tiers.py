"""The tier path of taot_sinkhorn_batched (a shared cost matrix whose entries
are the tiers of a tree) against the fp64 oracle, at the edges of its rule:
what it takes agrees with the oracle to the rounding of fp32, what it leaves
to the other kernels within their tolerance."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2608_03676_amd as taot
from helpers import potentials_check, sinkhorn_check

pytestmark = pytest.mark.gpu

# An entry of the plan is a product of three fp64 factors, each off by at most
# a few ten 2^-52 after the iterations these tests run, rounded once to fp32.
TIER_RTOL = 2.0 ** -24 * 1.01


def _tree_cost(R, sizes, costs, diag=0.0, perm=None):
    """C of nested groups: costs[l] inside a group of sizes[l] ranks, costs[-1] beyond."""
    r = np.arange(R) if perm is None else perm
    C = np.full((R, R), costs[-1], np.float32)
    for size, c in sorted(zip(sizes, costs), reverse=True):
        C[(r // size)[:, None] == (r // size)[None, :]] = c
    np.fill_diagonal(C, diag)
    return C


def _marginals(rng, R, B, surplus=0.0):
    """Disjoint supports, integer supplies; demand total = supply total * (1 + surplus)."""
    a, b = np.zeros((B, R), np.float32), np.zeros((B, R), np.float32)
    for p in range(B):
        nh = int(rng.integers(1, max(2, R // 3 + 1)))
        nc = int(rng.integers(1, R - nh + 1))
        at = rng.permutation(R)
        a[p, at[:nh]] = rng.integers(1, 4000, size=nh)
        total = int(a[p].sum() * (1 + surplus))
        b[p, at[nh:nh + nc]] = rng.multinomial(total, np.full(nc, 1.0 / nc))
        if not b[p].any():
            b[p, at[nh]] = total
    return a, b


def _run(a, b, C, eps, iters, flags=0):
    dev = torch.device("cuda:0")
    out = taot.sinkhorn_batched(*(torch.from_numpy(np.ascontiguousarray(x)).to(dev) for x in (a, b, C)), eps, iters, flags)
    torch.cuda.synchronize()
    return [x.cpu().numpy() for x in (out.T, out.f, out.g, out.status)]


def _check(a, b, C, eps, iters, tier, flags=0):
    eps = float(np.float32(eps))  # the value the call takes: costs of 200 eps amplify its rounding
    T, f, g, st = _run(a, b, C, eps, iters, flags)
    a64, b64 = a.astype(np.float64), b.astype(np.float64)
    ref = O.sinkhorn(a64, b64, C.astype(np.float64), eps, iters, colcap=not (flags & taot.SK_NO_COLCAP))
    potentials_check(f, g, ref.f, ref.g, eps, iters)
    if tier:
        tiny = np.abs(ref.T) < 2.0 ** -120  # fp32 results near the denormals round by an absolute step
        assert np.all(np.abs(T - ref.T)[~tiny] <= TIER_RTOL * np.abs(ref.T)[~tiny] * (1 + iters * 1e-3))
        assert np.all(np.abs(T)[tiny] <= 2.0 ** -119)
    sinkhorn_check(T, ref.T, a64, b64)
    return T, st


@pytest.mark.parametrize("R,sizes,costs", [
    (2, (8,), (1.0, 4.0)),                      # one leaf of two ranks
    (8, (8,), (1.0, 4.0)),                      # one leaf: a constant off the diagonal
    (9, (8,), (1.0, 4.0)),                      # a leaf of one rank beside a full one
    (17, (8, 16), (1.0, 3.0, 8.0)),             # a rack of one rank
    (60, (3, 12, 24), (1.0, 2.0, 5.0, 9.0)),    # four tiers, odd fan-outs
    (64, (1,), (1.0, 1.0)),                     # no groups at all: one leaf
    (100, (8, 32), (-2.0, 3.0, 8.0)),           # ragged racks, a negative cost
    (128, (8, 32), (1.0, 3.0, 8.0)),            # the largest R of the one-block prepass
    (129, (8, 32), (1.0, 3.0, 8.0)),
    (256, (4, 32), (1.0, 3.0, 8.0)),            # 64 slots: a wave
    (256, (2, 32), (1.0, 3.0, 8.0)),            # 128 slots: two to a lane
    (257, (8, 64), (1.0, 4.0, 12.0)),           # the first R of eight-wave groups; a leaf of one rank
    (320, (2, 4, 32), (1.0, 2.0, 4.0, 9.0)),    # 256 slots: four to a lane
    (1100, (8, 64), (1.0, 4.0, 12.0)),          # more rows than the tree block has threads
    (2048, (8, 64, 512), (1.0, 4.0, 7.0, 12.0)),
])
@pytest.mark.parametrize("shuffled", [False, True])
def test_tree_costs(R, sizes, costs, shuffled, gpu):
    rng = np.random.default_rng(R + len(sizes))
    C = _tree_cost(R, sizes, costs, perm=rng.permutation(R) if shuffled else None)
    a, b = _marginals(rng, R, 3)
    for eps, iters in ((0.08, 40), (0.7, 1), (0.3, 2)):
        print(f"[tiers] R={R} sizes={sizes} shuffled={shuffled} eps={eps}", flush=True)
        _check(a, b, C, eps, iters, tier=True)


@pytest.mark.parametrize("B", [1024, 1025, 1033])
@pytest.mark.parametrize("R,sizes", [(20, (8, 16)), (130, (2, 32))])
def test_batches_of_eight_to_a_group(B, R, sizes, gpu):
    """Around the batch size where eight problems share a workgroup (a ragged
    last group), with up to 32 slots (two problems to a wave) and more; among
    them problems the tier kernel leaves to others."""
    rng = np.random.default_rng(B + R)
    C = _tree_cost(R, sizes, (1.0, 3.0, 8.0))
    a, b = _marginals(rng, R, B)
    a[5] = 0.0                      # zero mass
    b[6, 0] = a[6, 0] = 7.0         # a rank on both sides
    a[B - 1, :] = np.nan            # invalid
    good = [p for p in range(B) if p not in (5, B - 1)]
    T, f, g, st = _run(a, b, C, 0.2, 30)
    ref = O.sinkhorn(a[good].astype(np.float64), b[good].astype(np.float64), C.astype(np.float64), 0.2, 30)
    sinkhorn_check(T[good], ref.T, a[good].astype(np.float64), b[good].astype(np.float64))
    st = st.view(np.uint32)
    assert st[5] == taot.ST_ZERO_MASS and st[B - 1] == taot.ST_BAD_INPUT and not st[good].any()
    assert not T[5].any() and not T[B - 1].any()


@pytest.mark.parametrize("R", [247, 248, 249, 255])
def test_groups_of_eight_around_64_kib_of_lds(R, gpu):
    """Eight problems' LDS just below and above 64 KiB: at R = 248 the dynamic
    part alone is below, with the kernel's own variables it is above."""
    rng = np.random.default_rng(R)
    C = _tree_cost(R, (8, 32), (1.0, 3.0, 8.0))
    a, b = _marginals(rng, R, 1025)
    T, f, g, st = _run(a, b, C, 0.2, 20)
    at = [0, 511, 1023, 1024]
    a64, b64 = a[at].astype(np.float64), b[at].astype(np.float64)
    ref = O.sinkhorn(a64, b64, C.astype(np.float64), 0.2, 20)
    sinkhorn_check(T[at], ref.T, a64, b64)
    assert not st.any()


@pytest.mark.parametrize("case", ["five tiers", "not nested", "not symmetric", "one entry", "range", "diagonal range", "slots"])
def test_other_costs_are_left(case, gpu):
    rng = np.random.default_rng(3)
    R, eps = 96, 0.1
    C = _tree_cost(R, (4, 16, 48), (1.0, 2.0, 4.0, 6.0))
    if case == "five tiers":
        C = _tree_cost(R, (2, 4, 16, 48), (0.5, 1.0, 2.0, 4.0, 6.0))
    elif case == "not nested":  # a ring: equal rows counts, no groups
        d = np.abs(np.arange(R)[:, None] - np.arange(R)[None, :])
        C = np.minimum(np.minimum(d, R - d), 4).astype(np.float32)
    elif case == "not symmetric":
        C[np.triu_indices(R, 1)] += np.float32(0.25) * (C[np.triu_indices(R, 1)] > 5)
    elif case == "one entry":
        C[70, 3] = 4.0
    elif case == "range":
        eps = 0.024  # 5 / 0.024 > 200
    elif case == "diagonal range":
        C[11, 11] = -21.0
    else:  # one, four and four address bits: 512 slots
        R = 400
        C = _tree_cost(R, (2, 4, 40), (1.0, 2.0, 4.0, 6.0))
    a, b = _marginals(rng, R, 4)
    _check(a, b, C, eps, 60, tier=False)


def _near_tree(rng, R, levels, changed):
    """Nested random groups of shuffled ranks; then `changed` entries at other tiers, half of them on one side only."""
    C = np.full((R, R), float(levels), np.float32)
    key = np.zeros(R, int)
    for l in range(levels - 1, 0, -1):
        key = key * 3 + rng.integers(0, 3, size=R)
        C[key[:, None] == key[None, :]] = l
    for _ in range(changed):
        i, j = rng.choice(R, 2, replace=False)
        C[i, j] = rng.integers(1, levels + 1)
        if rng.random() < 0.5:
            C[j, i] = C[i, j]
    np.fill_diagonal(C, 0.0)
    return C


@pytest.mark.parametrize("R", [3, 5, 9, 40, 70, 300, 1100])
def test_near_trees(R, gpu):
    """Trees and matrices one or two entries away from one, which only a look
    at every entry tells apart: all agree with the oracle."""
    rng = np.random.default_rng(R)
    for k in range(24 if R < 100 else 6):
        levels = int(rng.integers(2, 5))
        C = _near_tree(rng, R, levels, k % 3)
        a, b = _marginals(rng, R, 2)
        _check(a, b, C, 0.1, 12, tier=False)


def test_problems_that_are_left_beside_solved_ones(gpu):
    """In one call over a tree: every third problem has a rank on both sides;
    the register, wide and streamed kernels then run on the lists that the
    prepass leaves, in batches of one and of eight problems to a group."""
    rng = np.random.default_rng(12)
    for R, B in ((64, 9), (130, 1030), (300, 9), (1100, 5)):
        C = _tree_cost(R, (8, 64), (1.0, 3.0, 8.0))
        a, b = _marginals(rng, R, B)
        for p in range(0, B, 3):
            b[p, int(a[p].argmax())] = 3.0
        at = list(range(0, B, 1 if B < 100 else 41))
        T = _run(a, b, C, 0.2, 25)[0]
        a64, b64 = a[at].astype(np.float64), b[at].astype(np.float64)
        ref = O.sinkhorn(a64, b64, C.astype(np.float64), 0.2, 25)
        sinkhorn_check(T[at], ref.T, a64, b64)


def test_marginals_that_are_left(gpu):
    """Overlapping supports, more demand than supply (the scalings drift by
    the ratio in every iteration), tiny and huge marginals."""
    rng = np.random.default_rng(4)
    R = 48
    C = _tree_cost(R, (8, 16), (1.0, 3.0, 8.0))
    a, b = _marginals(rng, R, 4)
    b[:, :3] += 5.0
    _check(a, b, C, 0.2, 30, tier=False)
    for surplus in (0.001, 0.5, 30.0):
        a, b = _marginals(rng, R, 4, surplus)
        _check(a, b, C, 0.2, 60, tier=surplus < 0.5)
    a, b = _marginals(rng, R, 2)
    tiny = a.copy()
    tiny[:, a.argmax(1)[0]] = np.float32(2.0 ** -65)
    _check(tiny, b, C, 0.2, 20, tier=False)
    _check(a * np.float32(2.0 ** 40), b * np.float32(2.0 ** 40), C, 0.2, 20, tier=True)


def test_outputs_and_flags(gpu):
    """Without the column cap, without a plan, and the same bits on every run
    and in whichever batch a problem stands."""
    rng = np.random.default_rng(6)
    R = 72
    C = _tree_cost(R, (8, 24), (1.0, 3.0, 8.0), diag=0.5)
    a, b = _marginals(rng, R, 1030)
    _check(a[:3], b[:3], C, 0.1, 50, tier=True, flags=taot.SK_NO_COLCAP)
    dev = torch.device("cuda:0")
    ta, tb, tc = (torch.from_numpy(x).to(dev) for x in (a, b, C))
    all1 = taot.sinkhorn_batched(ta, tb, tc, 0.1, 50)
    all2 = taot.sinkhorn_batched(ta, tb, tc, 0.1, 50)
    few = taot.sinkhorn_batched(ta[:40].contiguous(), tb[:40].contiguous(), tc, 0.1, 50)
    noT = taot.Flow(None, torch.empty_like(ta), torch.empty_like(ta), torch.empty(1030, dtype=torch.int32, device=dev))
    taot.sinkhorn_batched(ta, tb, tc, 0.1, 50, out=noT)
    for x in ("T", "f", "g"):
        assert torch.equal(getattr(all1, x), getattr(all2, x)), x
        assert torch.equal(getattr(all1, x)[:40], getattr(few, x)), x
    assert torch.equal(noT.f, all1.f) and torch.equal(noT.g, all1.g)

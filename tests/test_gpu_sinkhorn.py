"""GPU parity of taot_sinkhorn_batched with the fp64 oracle at the same
iteration count: relative L1 <= 1e-4, column error <= 1e-5 * mass, row error
within 1e-5 * mass of the oracle's own fixed-N residual."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2608_03676_amd as taot
import workloads as W
from helpers import off_tree, oracle_inputs, potentials_check, sinkhorn_check

pytestmark = pytest.mark.gpu


def _gpu_sinkhorn(a, b, C, eps, iters, flags=0):
    dev = torch.device("cuda:0")
    out = taot.sinkhorn_batched(torch.from_numpy(np.ascontiguousarray(a, np.float32)).to(dev),
                                torch.from_numpy(np.ascontiguousarray(b, np.float32)).to(dev),
                                torch.from_numpy(np.ascontiguousarray(C, np.float32)).to(dev),
                                eps, iters, flags)
    torch.cuda.synchronize()
    return (out.T.cpu().numpy(), out.f.cpu().numpy(), out.g.cpu().numpy(),
            out.status.cpu().numpy().view(np.uint32))


def _check_against_oracle(a32, b32, C32, eps, iters, flags=0):
    a = a32.astype(np.float64)
    b = b32.astype(np.float64)
    T, f, g, st = _gpu_sinkhorn(a32, b32, C32, eps, iters, flags)
    ref = O.sinkhorn(a, b, C32.astype(np.float64), eps, iters, colcap=not (flags & taot.SK_NO_COLCAP))
    rels = sinkhorn_check(T, ref.T, a, b)
    worst = potentials_check(f, g, ref.f, ref.g, eps, iters)
    print(f"  potentials: max |d(f+g)| {worst[0]:.2e} eps, max |df|, |dg| {worst[1]:.2e} eps", flush=True)
    return T, st, rels


@pytest.mark.parametrize("cfg,problems", [(0, [0]), (1, list(range(58))), (2, list(range(0, 384, 24))),
                                          (3, [0, 1, 2, 977, 1951])])
@pytest.mark.parametrize("flags,tree", [(0, True), (0, False), (taot.SK_NO_REGISTER, True)])
def test_workloads(cfg, problems, flags, tree, gpu):
    """Default flags take the tier path for the workloads' costs and the
    register-resident path for costs that are no tree; SK_NO_REGISTER takes
    the LDS-resident one."""
    w = W.WORKLOADS[cfg]
    print(f"[sinkhorn parity] workload {cfg} problems {problems} flags {flags} tree {tree}", flush=True)
    _, L = oracle_inputs(w, problems)
    C = W.cost_matrix(w) if tree else off_tree(W.cost_matrix(w))
    _, st, rels = _check_against_oracle(L.excess.astype(np.float32), L.spare.astype(np.float32), C, w.eps,
                                        w.iters, flags)
    assert np.all(st == 0)
    print(f"max relL1 {max(rels):.2e}")


@pytest.mark.parametrize("seed", range(3))
@pytest.mark.parametrize("tree", [True, False])
def test_mixed_size_classes_in_one_batch(seed, tree, gpu):
    """One batch whose problems fall into different kernel classes: hot-set
    sizes 1..70 and cold-set sizes 1..250 (register classes and the fallback;
    all on the tier path with the tree's costs)."""
    rng = np.random.default_rng(50 + seed)
    R, B = 256, 24
    a = np.zeros((B, R), np.float32)
    b = np.zeros((B, R), np.float32)
    for p in range(B):
        nh = int(rng.integers(1, 71))
        nc = int(rng.integers(1, min(250, R - nh) + 1))
        perm = rng.permutation(R)
        a[p, perm[:nh]] = rng.integers(1, 3000, size=nh)
        b[p, perm[nh:nh + nc]] = rng.multinomial(int(a[p].sum()), np.full(nc, 1.0 / nc))
    C = W.cost_matrix_for(R, ("three_tier", 1.0, 3.0, 8.0, 32))
    _check_against_oracle(a, b, C if tree else off_tree(C), 0.08, 300)


@pytest.mark.parametrize("flags,tree", [(0, True), (0, False), (taot.SK_NO_REGISTER, True)])
def test_workload4(flags, tree, gpu):
    """R = 1024 (about 85 hot and 940 cold ranks): by default the tier path
    for its costs, and for costs that are no tree the wide register kernel,
    which holds the block in one workgroup's registers; with SK_NO_REGISTER
    it is streamed through device memory."""
    w = W.WORKLOADS[4]
    print(f"[sinkhorn parity] workload 4 problem 0 flags {flags} tree {tree}", flush=True)
    _, L = oracle_inputs(w, [0])
    C = W.cost_matrix(w) if tree else off_tree(W.cost_matrix(w))
    _, st, rels = _check_against_oracle(L.excess.astype(np.float32), L.spare.astype(np.float32), C, w.eps, w.iters,
                                        flags)
    assert np.all(st == (taot.ST_STREAMED if flags else 0))


@pytest.mark.parametrize("R", [300, 1100])
@pytest.mark.parametrize("tree", [True, False])
def test_wide_shapes(R, tree, gpu):
    """Problems for the wide register kernel (65..96 hot ranks, or more than
    256 cold ranks), one per columns-per-lane class, with eps small enough to
    trigger the log-domain updates; beside them one problem too large for it
    (streamed) in the same batch.  With the tree's costs the tier path solves
    them all and reports the same classes."""
    rng = np.random.default_rng(R)
    if R == 300:
        shapes = [(65, 200), (80, 220), (96, 204), (40, 257), (8, 290)]
    else:
        shapes = [(1, 300), (50, 400), (96, 500), (33, 640), (70, 700), (90, 830), (60, 897), (96, 960), (20, 1000)]
    B = len(shapes)
    a = np.zeros((B, R), np.float32)
    b = np.zeros((B, R), np.float32)
    for p, (nh, nc) in enumerate(shapes):
        perm = rng.permutation(R)
        a[p, perm[:nh]] = rng.integers(1, 4000, size=nh)
        b[p, perm[nh:nh + nc]] = rng.multinomial(int(a[p].sum()), np.full(nc, 1.0 / nc)) + 1
    C = W.cost_matrix_for(R, ("three_tier", 1.0, 3.0, 8.0, 32))
    C = C if tree else off_tree(C)
    for eps, iters in ((0.5, 3), (0.08, 120)):
        print(f"[sinkhorn parity] wide shapes R={R} eps={eps} tree={tree}", flush=True)
        _, st, _ = _check_against_oracle(a, b, C, eps, iters)
        streamed = [nc > 960 for _, nc in shapes]
        assert np.array_equal(st == taot.ST_STREAMED, np.array(streamed)), st


def test_forced_stream_matches_lds_path(gpu):
    """The streamed and the LDS-resident kernels run the same arithmetic in the
    same order, only the plan block lives elsewhere: their plans are identical."""
    w = W.WORKLOADS[2]
    _, L = oracle_inputs(w, [7, 8, 9])
    C = W.cost_matrix(w)
    a, b = L.excess.astype(np.float32), L.spare.astype(np.float32)
    T1, st1, _ = _check_against_oracle(a, b, C, w.eps, w.iters, taot.SK_NO_REGISTER)
    T2, st2, _ = _check_against_oracle(a, b, C, w.eps, w.iters, taot.SK_FORCE_STREAM)
    assert np.all(st1 == 0) and np.all(st2 == taot.ST_STREAMED)
    assert T1.tobytes() == T2.tobytes()


def _random_case(rng, R, overlap=False, integer=True):
    a = np.zeros(R, np.float32)
    b = np.zeros(R, np.float32)
    hot = rng.choice(R, size=max(1, R // 4), replace=False)
    cold = rng.choice(R, size=max(1, R // 2), replace=False) if overlap else np.setdiff1d(np.arange(R), hot)
    if cold.size == 0:
        cold = hot
    if integer:
        a[hot] = rng.integers(1, 5000, size=hot.size)
        b[cold] = rng.multinomial(int(a.sum()), np.full(cold.size, 1.0 / cold.size))
    else:
        a[hot] = rng.uniform(0.5, 20.0, size=hot.size)
        b[cold] = rng.uniform(0.5, 20.0, size=cold.size)
    return a, b


@pytest.mark.parametrize("R", [1, 2, 5, 16, 33, 100, 256, 300])
@pytest.mark.parametrize("overlap", [False, True])
def test_random(R, overlap, gpu):
    rng = np.random.default_rng(R + 1000 * overlap)
    B = 3
    cases = [_random_case(rng, R, overlap, integer=(p != 2)) for p in range(B)]
    a = np.stack([c[0] for c in cases])
    b = np.stack([c[1] for c in cases])
    C = rng.uniform(0.0, 3.0, (R, R)).astype(np.float32)
    for eps, iters in ((0.5, 1), (0.2, 7), (0.08, 150)):
        _check_against_oracle(a, b, C, eps, iters)


def test_per_problem_cost_and_no_colcap(gpu):
    rng = np.random.default_rng(11)
    R, B = 48, 4
    cases = [_random_case(rng, R) for _ in range(B)]
    a = np.stack([c[0] for c in cases])
    b = np.stack([c[1] for c in cases])
    C = rng.uniform(0.0, 4.0, (B, R, R)).astype(np.float32)
    dev = torch.device("cuda:0")
    for flags in (0, taot.SK_NO_COLCAP):
        out = taot.sinkhorn_batched(torch.from_numpy(a).to(dev), torch.from_numpy(b).to(dev),
                                    torch.from_numpy(C).to(dev), 0.1, 80, flags)
        torch.cuda.synchronize()
        ref = O.sinkhorn(a.astype(float), b.astype(float), C.astype(float), 0.1, 80,
                         colcap=not flags)
        sinkhorn_check(out.T.cpu().numpy(), ref.T, a.astype(float), b.astype(float))


def test_degenerate(gpu):
    R = 8
    C = np.ones((R, R), np.float32)
    a = np.zeros((4, R), np.float32)
    b = np.zeros((4, R), np.float32)
    b[0, 1] = 3.0                    # zero supply
    a[1, 2] = 3.0                    # zero demand
    a[2, 0], b[2, 3] = np.nan, 1.0   # bad supply
    a[3, 0], b[3, 3] = 2.0, 2.0      # fine problem next to the bad ones
    T, f, g, st = _gpu_sinkhorn(a, b, C, 0.5, 10)
    assert st[0] == taot.ST_ZERO_MASS and st[1] == taot.ST_ZERO_MASS and st[2] == taot.ST_BAD_INPUT
    assert st[3] == 0
    assert not T[:3].any() and np.all(np.isneginf(f[:3])) and np.all(np.isneginf(g[:3]))
    np.testing.assert_allclose(T[3, 0, 3], 2.0, rtol=1e-6)
    Cb = C.copy()
    Cb[0, 5] = np.inf
    _, _, _, st = _gpu_sinkhorn(a[3:], b[3:], Cb, 0.5, 10)
    assert st[0] == taot.ST_BAD_INPUT


@pytest.mark.parametrize("R,where", [(8, (5, 1)), (8, (3, 3)), (300, (299, 7)), (1100, (1099, 1098))])
@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_nonfinite_cost_anywhere(R, where, bad, gpu):
    """A NaN or infinity in any entry of C marks the problem BAD_INPUT with a
    zero plan and -inf potentials, as in the oracle, also in a row or column
    the iterate never reads (here the entry's row is not hot, or it is the
    diagonal).  With per-problem costs only the problem whose matrix holds it
    is marked; the others are planned as usual (register, wide and streamed
    classes at R = 8 / 300 / 1100)."""
    rng = np.random.default_rng(R)
    B = 3
    a = np.zeros((B, R), np.float32)
    b = np.zeros((B, R), np.float32)
    for p in range(B):
        a[p, :2] = rng.integers(5000, 20000, size=2)    # hot ranks 0 and 1
        # cold ranks 2 .. R-2, demand about the supply; the last rank is neither
        b[p, 2:R - 1] = rng.multinomial(int(a[p].sum()), np.full(R - 3, 1.0 / (R - 3))) + 1
    C = W.cost_matrix_for(R, ("three_tier", 1.0, 3.0, 8.0, 32)) if R > 8 else \
        rng.uniform(0.5, 2.0, (R, R)).astype(np.float32)
    i, j = where
    assert a[0, i] == 0  # a row the iterate does not read
    Cs = C.copy()
    Cs[i, j] = bad
    eps, iters = 0.1, 20
    T, f, g, st = _gpu_sinkhorn(a, b, Cs, eps, iters)
    ref = O.sinkhorn(a.astype(float), b.astype(float), Cs.astype(float), eps, iters)
    assert np.all(ref.status == O.ST_BAD_INPUT)
    assert np.all(st == taot.ST_BAD_INPUT), st
    assert not T.any() and np.all(np.isneginf(f)) and np.all(np.isneginf(g))
    # per-problem costs: only problem 1's matrix holds the bad entry
    Cp = np.stack([C, C, C])
    Cp[1, i, j] = bad
    T, f, g, st = _gpu_sinkhorn(a, b, Cp, eps, iters)
    ref = O.sinkhorn(a.astype(float), b.astype(float), Cp.astype(float), eps, iters)
    assert list(ref.status) == [0, O.ST_BAD_INPUT, 0]
    assert st[1] == taot.ST_BAD_INPUT and st[0] & taot.ST_BAD_INPUT == 0 and st[2] & taot.ST_BAD_INPUT == 0, st
    assert not T[1].any() and np.all(np.isneginf(f[1])) and np.all(np.isneginf(g[1]))
    keep = [0, 2]
    sinkhorn_check(T[keep], ref.T[keep], a[keep].astype(float), b[keep].astype(float))
    potentials_check(f[keep], g[keep], ref.f[keep], ref.g[keep], eps, iters)


@pytest.mark.parametrize("tree", [True, False])
def test_deterministic(tree, gpu):
    w = W.WORKLOADS[3]
    _, L = oracle_inputs(w, [3, 4])
    C = W.cost_matrix(w) if tree else off_tree(W.cost_matrix(w))
    a, b = L.excess.astype(np.float32), L.spare.astype(np.float32)
    T1 = _gpu_sinkhorn(a, b, C, w.eps, w.iters)[0]
    T2 = _gpu_sinkhorn(a, b, C, w.eps, w.iters)[0]
    assert T1.tobytes() == T2.tobytes()


@pytest.mark.parametrize("nh,nc", [(49, 129), (56, 200), (57, 256), (64, 193), (64, 256)])
@pytest.mark.parametrize("tree", [True, False])
def test_two_wave_rows(nh, nc, tree, gpu):
    """Hot sets of 49..64 ranks with more than 128 cold ranks: the row block is
    split over two waves that exchange column sums (the tier path takes the
    tree's costs but at the smallest eps).  Small eps drives the scalings out
    of range, so both log-domain absorptions run as well."""
    rng = np.random.default_rng(nh * 1000 + nc)
    R = nh + nc
    B = 3
    a = np.zeros((B, R), np.float32)
    b = np.zeros((B, R), np.float32)
    for p in range(B):
        perm = rng.permutation(R)
        a[p, perm[:nh]] = rng.integers(1, 4000, size=nh)
        b[p, perm[nh:]] = rng.multinomial(int(a[p].sum()), np.full(nc, 1.0 / nc)) + 1
    C = W.cost_matrix_for(R, ("three_tier", 1.0, 3.0, 8.0, 32))
    C = C if tree else off_tree(C)
    for eps, iters in ((0.5, 3), (0.08, 200), (0.02, 120)):
        print(f"[sinkhorn parity] two-wave nh={nh} nc={nc} eps={eps} tree={tree}", flush=True)
        _check_against_oracle(a, b, C, eps, iters)


def test_folded_shapes(gpu):
    """Every one-wave shape of the two-wave kernel (SK_WAVES_1), whose single
    problems fold their columns over the half-waves: 1..8 columns per lane
    (cold ranks up to 32 per column, exact multiples and ragged), every
    chunk count the layout holds (ragged hot ranks), and past it the
    two-wave problems (more than 48 hot and 128 cold ranks)."""
    rng = np.random.default_rng(23)
    R = 320
    shapes = []
    for cpl in range(1, 9):
        for c8 in range(1, 9):
            nc = 32 * cpl - (int(rng.integers(1, 31)) if c8 % 2 else 0)
            nh = 8 * c8 - int(rng.integers(0, 8))
            shapes.append((nh, nc))
    B = len(shapes)
    a = np.zeros((B, R), np.float32)
    b = np.zeros((B, R), np.float32)
    for p, (nh, nc) in enumerate(shapes):
        perm = rng.permutation(R)
        a[p, perm[:nh]] = rng.integers(1, 4000, size=nh)
        b[p, perm[nh:nh + nc]] = rng.multinomial(int(a[p].sum()), np.full(nc, 1.0 / nc)) + 1
    C = W.cost_matrix_for(R, ("three_tier", 1.0, 3.0, 8.0, 32))
    for eps, iters in ((0.08, 200), (0.02, 120)):
        print(f"[sinkhorn parity] folded shapes eps={eps}", flush=True)
        _check_against_oracle(a, b, C, eps, iters, taot.SK_WAVES_1)


@pytest.mark.parametrize("flags,tree", [(0, True), (0, False), (taot.SK_WAVES_1, True)])
def test_register_shapes(flags, tree, gpu):
    """One problem of every register class (1, 2 or 4 columns per lane x 1..8
    chunks of 8 hot ranks) in one batch.  By default a small batch spreads
    each problem over up to four waves (one-chunk problems share a workgroup,
    one wave each); SK_WAVES_1 takes the shapes of large batches (one wave per
    problem where its rows fit, else two).  With default flags the tier path
    takes the tree's costs but at the smallest eps.  Small eps drives the scalings out
    of range, so the log-domain updates run too."""
    rng = np.random.default_rng(7 + flags)
    R = 320
    shapes = [(nh, nc) for lo, hi in ((1, 64), (65, 128), (129, 256))
              for c8 in range(1, 9)
              for nh, nc in [(8 * c8 - int(rng.integers(0, 8)), int(rng.integers(lo, hi + 1)))]]
    B = len(shapes)
    a = np.zeros((B, R), np.float32)
    b = np.zeros((B, R), np.float32)
    for p, (nh, nc) in enumerate(shapes):
        perm = rng.permutation(R)
        a[p, perm[:nh]] = rng.integers(1, 4000, size=nh)
        b[p, perm[nh:nh + nc]] = rng.multinomial(int(a[p].sum()), np.full(nc, 1.0 / nc)) + 1
    C = W.cost_matrix_for(R, ("three_tier", 1.0, 3.0, 8.0, 32))
    C = C if tree else off_tree(C)
    for eps, iters in ((0.5, 3), (0.08, 200), (0.02, 120)):
        print(f"[sinkhorn parity] register shapes flags={flags} tree={tree} eps={eps}", flush=True)
        _check_against_oracle(a, b, C, eps, iters, flags)


@pytest.mark.parametrize("B", [1024, 1100])
def test_large_batch_of_register_problems(B, gpu):
    """Shared costs that are no tree and default flags, up to and past the
    batch in which every problem can hold four waves (16 per compute unit):
    hot sets of 1..70 and cold sets of 1..180 ranks, in one call."""
    rng = np.random.default_rng(B)
    R = 256
    a = np.zeros((B, R), np.float32)
    b = np.zeros((B, R), np.float32)
    for p in range(B):
        nh, nc = int(rng.integers(1, 71)), int(rng.integers(1, 181))
        perm = rng.permutation(R)
        a[p, perm[:nh]] = rng.integers(1, 3000, size=nh)
        b[p, perm[nh:nh + nc]] = rng.multinomial(int(a[p].sum()), np.full(nc, 1.0 / nc))
    C = off_tree(W.cost_matrix_for(R, ("three_tier", 1.0, 3.0, 8.0, 32)))
    T, f, g, st = _gpu_sinkhorn(a, b, C, 0.08, 100)
    assert np.all(st == 0)
    at = list(range(0, B, 37)) + [B - 1]
    a64, b64 = a[at].astype(np.float64), b[at].astype(np.float64)
    ref = O.sinkhorn(a64, b64, C.astype(np.float64), 0.08, 100)
    sinkhorn_check(T[at], ref.T, a64, b64)
    potentials_check(f[at], g[at], ref.f, ref.g, 0.08, 100)

"""The walk kernel at its edges against the oracle, element by element: every
tile width (by the number of features), one sample and sizes around a tile and
a block's range, subsets read through the index and as multiplicities (with
repeated samples), one tree to many groups, columns whose threshold count
passes what the packed words hold, and unaligned rank columns."""
import numpy as np
import pytest

import oracle
from gpu_helpers import dev, np_, random_trees, u32
from paper_2311_06952_amd import synth

pytestmark = pytest.mark.gpu


def _check(mh, ds, ods, feat, tau, D, idx=None):
    want = oracle.fitness(ods, feat, tau, D, idx=idx, n_min=2, alpha=0.5)
    for static in (False, True):
        got = mh.fitness_eval(ds, dev(feat), dev(tau), D, idx=None if idx is None else dev(idx),
                              n_min=2, alpha=0.5, static=static)
        for k in range(2):
            np.testing.assert_array_equal(u32(got[k]), want[k])
        for k in (2, 3):
            np.testing.assert_array_equal(np_(got[k]), want[k])


# (n, F, K, D, P): tiles of 1,024, 512, 256 and 128 samples
@pytest.mark.parametrize("n,F,K,D,P", [
    (1, 24, 2, 6, 3), (63, 24, 3, 6, 65), (1023, 24, 2, 7, 5), (1025, 24, 4, 6, 33),
    (513, 25, 3, 6, 17), (1537, 48, 2, 8, 4), (255, 49, 3, 6, 41), (1281, 128, 2, 6, 19),
    (127, 129, 3, 6, 70), (641, 255, 2, 10, 3), (70_003, 5, 2, 6, 300)])
def test_walk_tile_edges(mh_mod, n, F, K, D, P):
    X, y = synth.random_small(n + F, n, F, K, levels=None if n % 2 else 30)
    ods = oracle.dataset_from_X(X, y, K)
    ds = mh_mod.dataset(X, y, K)
    rng = np.random.default_rng(n)
    feat, tau = random_trees(rng, P, D, F, ods.n_unique)
    _check(mh_mod, ds, ods, feat, tau, D)


@pytest.mark.parametrize("share", [0.1, 0.249, 0.25, 0.9, 3.0])
def test_walk_subsets(mh_mod, share):
    """Below a quarter of the samples the subset is gathered; from there on it
    is counted, repeated samples as often as they are named."""
    n, F, K, D = 4001, 9, 3, 7
    X, y = synth.random_small(7, n, F, K)
    ods = oracle.dataset_from_X(X, y, K)
    ds = mh_mod.dataset(X, y, K)
    rng = np.random.default_rng(3)
    feat, tau = random_trees(rng, 21, D, F, ods.n_unique)
    idx = rng.integers(0, n, size=int(n * share)).astype(np.uint32)
    _check(mh_mod, ds, ods, feat, tau, D, idx=idx)


@pytest.mark.parametrize("share", [0.25, 0.95, 3.0])
def test_walk_large_subsets(mh_mod, share):
    """From 2^20 gathered ranks on the subset is counted into multiplicities."""
    n, F, K, D = 130_000, 9, 3, 6
    X, y = synth.random_small(8, n, F, K)
    ods = oracle.dataset_from_X(X, y, K)
    ds = mh_mod.dataset(X, y, K)
    rng = np.random.default_rng(4)
    feat, tau = random_trees(rng, 5, D, F, ods.n_unique)
    idx = rng.integers(0, n, size=int(n * share)).astype(np.uint32)
    _check(mh_mod, ds, ods, feat, tau, D, idx=idx)


# at most as many nodes as columns: only the columns split on are staged (tiles
# of every width; one tree; trees without a split)
@pytest.mark.parametrize("n,F,K,D,P,nosplit", [
    (5000, 120, 3, 2, 40, 0.15), (1999, 255, 2, 1, 255, 0.15), (130, 90, 3, 4, 6, 0.1),
    (3001, 100, 4, 5, 1, 0.15), (70_001, 85, 2, 3, 2, 0.3), (900, 81, 3, 2, 5, 1.0),
    (2500, 200, 3, 1, 47, 0.0)])
def test_walk_selected_columns(mh_mod, n, F, K, D, P, nosplit):
    X, y = synth.random_small(n + F, n, F, K, levels=None if n % 2 else 30)
    ods = oracle.dataset_from_X(X, y, K)
    ds = mh_mod.dataset(X, y, K)
    rng = np.random.default_rng(n)
    feat, tau = random_trees(rng, P, D, F, ods.n_unique, p_nosplit=nosplit)
    _check(mh_mod, ds, ods, feat, tau, D)
    idx = rng.integers(0, n, size=n // 2).astype(np.uint32)
    _check(mh_mod, ds, ods, feat, tau, D, idx=idx)


@pytest.mark.parametrize("ld", [1301, 1304])
def test_walk_many_thresholds(mh_mod, ld):
    """Columns cut out of an encoding of more values than the packed words
    hold, with rank columns that are and are not multiples of 16 bytes."""
    import torch
    n, F, K, D, P = 1300, 6, 3, 6, 11
    rng = np.random.default_rng(ld)
    nu = np.array([2**24, 700, 2**25, 2**24 - 1, 5, 2**24 - 2], np.uint32)
    ranks = np.stack([rng.integers(0, v, size=n) for v in nu]).astype(np.uint32)
    y = rng.integers(0, K, size=n).astype(np.uint8)
    ods = oracle.Dataset(ranks, nu, y, K)
    padded = torch.zeros((F, ld), dtype=torch.int32, device="cuda")
    padded[:, :n] = dev(ranks)
    feat, tau = random_trees(rng, P, D, F, nu)
    for few in (False, True):  # with and without the wide columns
        if few:
            nu = np.minimum(nu, 2**24 - 2).astype(np.uint32)
            ranks = np.minimum(ranks, nu[:, None] - 1).astype(np.uint32)
            padded[:, :n] = dev(ranks)
            ods = oracle.Dataset(ranks, nu, y, K)
        ds = mh_mod.Dataset(padded, dev(y), dev(nu), n, F, K)
        _check(mh_mod, ds, ods, feat, tau, D)


def test_walk_wide_ranks(mh_mod):
    """2^24 samples: thresholds of 32 bits, over a subset and over all."""
    n, F, K, D, P = 2**24, 2, 2, 6, 9
    rng = np.random.default_rng(5)
    ranks = np.stack([rng.permutation(n), rng.integers(0, 1000, size=n)]).astype(np.uint32)
    nu = np.array([n, 1000], np.uint32)
    y = (ranks[0] % 3 == 0).astype(np.uint8)
    ods = oracle.Dataset(ranks, nu, y, K)
    ds = mh_mod.Dataset(dev(ranks), dev(y), dev(nu), n, F, K)
    feat, tau = random_trees(rng, P, D, F, nu)
    idx = rng.integers(0, n, size=3001).astype(np.uint32)
    _check(mh_mod, ds, ods, feat, tau, D, idx=idx)
    _check(mh_mod, ds, ods, feat[:1], tau[:1], D)


@pytest.fixture(scope="module")
def mh_mod():
    import paper_2311_06952_amd as m
    return m


def _near_limit_counts(n, tau, K=3):
    """Leaf counts of a depth-6 tree over samples i < n with rank i % 64 and
    label (i // 64) % 3."""
    rows, tail = divmod(n, 64)
    per_class = np.array([len(range(k, rows, K)) for k in range(K)], dtype=np.int64)
    counts = np.zeros((64, K), dtype=np.int64)
    for r in range(64):
        t = 1
        for _ in range(6):
            t = 2 * t if r < tau[t - 1] else 2 * t + 1
        counts[t - 64] += per_class
        if r < tail:
            counts[t - 64, rows % K] += 1
    return counts


@pytest.mark.parametrize("n", [2**32 - 4, 2**32 - 1021])
def test_walk_sample_counts_near_the_32_bit_limit(n):
    """The last ranges and tiles end within a tile of 2^32 samples (rows of
    whole 16-byte chunks, and an odd row)."""
    import torch

    import paper_2311_06952_amd as mh
    ranks = torch.arange(64, dtype=torch.int32, device="cuda").repeat(1 << 26)[:n].view(1, n)
    labels = torch.arange(3, dtype=torch.uint8, device="cuda").repeat_interleave(64)
    labels = labels.repeat((1 << 32) // 192 + 1)[:n]
    ds = mh.Dataset(ranks, labels, torch.tensor([64], dtype=torch.int32, device="cuda"), n, 1, 3)
    tau = np.random.default_rng(3).integers(0, 65, 63).astype(np.int32)
    feat = torch.ones((1, 63), dtype=torch.uint8, device="cuda")
    counts, correct, _, _ = mh.fitness_eval(ds, feat, torch.as_tensor(tau).cuda(), 6)
    got = counts.cpu().numpy().view(np.uint32).astype(np.int64)[0]
    del ranks, labels, ds
    torch.cuda.empty_cache()
    np.testing.assert_array_equal(got, _near_limit_counts(n, tau))
    assert int(correct.cpu().numpy().view(np.uint32)[0]) == got.max(axis=1).sum()


@pytest.mark.parametrize("static", [False, True])
def test_walk_subset_near_the_32_bit_limit(static):
    """A subset that names 2^20 samples 4,096 times, but for the last five."""
    import torch

    import paper_2311_06952_amd as mh
    n, n_sub = 1 << 20, 2**32 - 5
    ranks = (torch.arange(n, dtype=torch.int32, device="cuda") % 64).view(1, n).contiguous()
    labels = (torch.arange(n, dtype=torch.int32, device="cuda") // 64 % 3).to(torch.uint8)
    ds = mh.Dataset(ranks, labels, torch.tensor([64], dtype=torch.int32, device="cuda"), n, 1, 3)
    idx = torch.arange(n, dtype=torch.int32, device="cuda").repeat(4096)[:n_sub]
    tau = np.random.default_rng(4).integers(0, 65, 63).astype(np.int32)
    feat = torch.ones((1, 63), dtype=torch.uint8, device="cuda")
    counts, _, _, _ = mh.fitness_eval(ds, feat, torch.as_tensor(tau).cuda(), 6, idx=idx,
                                      static=static)
    got = counts.cpu().numpy().view(np.uint32).astype(np.int64)[0]
    del idx
    torch.cuda.empty_cache()
    want = 4095 * _near_limit_counts(n, tau) + _near_limit_counts(n - 5, tau)
    np.testing.assert_array_equal(got, want)


# The form of the walk by shape and by kind of call (all samples; a random half,
# counted in the call's own scratch or gathered in a caller's; every sample three
# times over): tiles, direct or weights.  One tree to a group's remainder, four
# and eight chains, counts in LDS and (many classes at depth 9 and 10) in memory.
@pytest.mark.parametrize("n,F,K,P,D,forms", [
    (1, 49, 2, 1, 6, ("direct", "direct", "direct")),
    (255, 100, 2, 7, 6, ("direct", "direct", "direct")),
    (257, 200, 3, 8, 5, ("direct", "direct", "direct")),
    (4097, 255, 4, 33, 1, ("direct", "direct", "direct")),
    (1500, 120, 254, 5, 10, ("direct", "direct", "direct")),
    (2000, 90, 200, 13, 9, ("direct", "direct", "direct")),
    (70_001, 130, 2, 3, 7, ("tiles", "direct", "weights")),
    (3000, 60, 2, 65, 6, ("tiles", "tiles", "weights")),
    (513, 128, 20, 70, 7, ("tiles", "direct", "direct")),
])
def test_walk_forms(mh_mod, monkeypatch, capfd, n, F, K, P, D, forms):
    monkeypatch.setenv("MHDEOCT_DEBUG", "1")
    ctx = mh_mod.Context(0)
    X, y = synth.random_small(n + F, n, F, K, levels=None if n % 2 else 30)
    ods = oracle.dataset_from_X(X, y, K)
    ds = mh_mod.dataset(X, y, K, ctx=ctx)
    rng = np.random.default_rng(n + P)
    feat, tau = random_trees(rng, P, D, F, ods.n_unique)
    half = rng.integers(0, n, size=n // 2 + 1).astype(np.uint32)
    thrice = np.tile(np.arange(n, dtype=np.uint32), 3)
    for idx, form in zip((None, half, thrice), forms):
        want = oracle.fitness(ods, feat, tau, D, idx=idx, n_min=2, alpha=0.5)
        for static in (False, True):
            capfd.readouterr()
            got = mh_mod.fitness_eval(ds, dev(feat), dev(tau), D, ctx=ctx,
                                      idx=None if idx is None else dev(idx),
                                      n_min=2, alpha=0.5, static=static)
            line = [e for e in capfd.readouterr().err.splitlines() if e.startswith("k_walk")]
            assert len(line) == 1
            assert ("k_walk_direct" in line[0]) == (form == "direct") or static
            assert ("weights" in line[0]) == (form == "weights" and not static)
            for k in range(2):
                np.testing.assert_array_equal(u32(got[k]), want[k])
            for k in (2, 3):
                np.testing.assert_array_equal(np_(got[k]), want[k])
    # entries past n are left out
    bad = np.concatenate([half, np.array([n, 2**32 - 1], np.uint32)])
    want = oracle.fitness(ods, feat, tau, D, idx=half, n_min=2, alpha=0.5)
    for static in (False, True):
        got = mh_mod.fitness_eval(ds, dev(feat), dev(tau), D, idx=dev(bad), ctx=ctx,
                                  n_min=2, alpha=0.5, static=static)
        np.testing.assert_array_equal(u32(got[0]), want[0])
    ctx.close()


def test_walk_weights_of_a_run(mh_mod, monkeypatch, capfd):
    """A run counts its subset once for all generations; the next run's subset
    replaces it, also one that is gathered."""
    n, F, K, D, prm = 4001, 9, 3, 7, (21, 40, 0.5, 0.7, 5, 1, 0.0)
    monkeypatch.setenv("MHDEOCT_DEBUG", "1")
    ctx = mh_mod.Context(0)
    X, y = synth.random_small(11, n, F, K)
    ods = oracle.dataset_from_X(X, y, K)
    ds = mh_mod.dataset(X, y, K, ctx=ctx)
    rng = np.random.default_rng(12)
    for size in (12_003, 11_000, 50, 12_003):
        idx = rng.integers(0, n, size=size).astype(np.uint32)
        want = oracle.deoct(ods, D, oracle.de_params(*prm), idx=idx, with_pop=True)
        capfd.readouterr()
        got = mh_mod.subtree_solve(ds, D, mh_mod.de_params(*prm), idx=dev(idx), ctx=ctx,
                                   with_pop=True)
        lines = [e for e in capfd.readouterr().err.splitlines() if e.startswith("k_walk")]
        assert len(lines) == 42  # the first population, 40 trials and the best tree
        assert all(("weights" in e) == (size > 50) for e in lines)
        for key in ("feat", "tau", "label", "pop", "pop_cost"):
            np.testing.assert_array_equal(got[key], want[key])
        assert got["correct"] == want["correct"] and got["cost"] == want["cost"]
    ctx.close()

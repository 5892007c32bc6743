"""GPU parity of the whole-run kernel with tiles staged every generation by four
groups per block against the oracle: best tree, cost and the final population
bit for bit; and several problems of very different sizes in one launch."""
import numpy as np
import pytest

import oracle
from paper_2311_06952_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mh():
    import paper_2311_06952_amd as m
    return m


def _check(mh, ctx, X, y, K, D, prm):
    want = oracle.deoct(oracle.dataset_from_X(X, y, K), D, oracle.de_params(*prm), with_pop=True)
    got = mh.subtree_solve(mh.dataset(X, y, K, ctx=ctx), D, mh.de_params(*prm), ctx=ctx,
                           with_pop=True)
    for key in ("feat", "tau", "label", "pop", "pop_cost"):
        np.testing.assert_array_equal(got[key], want[key])
    assert got["correct"] == want["correct"] and got["cost"] == want["cost"]


# whole records below 16 features, the compact form from there on; blocks
# without a tile, with one group busy, with a ragged last round
@pytest.mark.parametrize("D,P,K,n,F", [
    (1, 3, 2, 5, 2), (1, 65, 3, 9000, 17), (2, 64, 4, 3000, 15), (2, 200, 2, 20_000, 16),
    (3, 5, 3, 64, 16), (3, 64, 5, 17_000, 3), (3, 128, 3, 40_000, 20), (3, 256, 2, 33_000, 9),
    (3, 129, 7, 6_000, 18), (3, 100, 2, 2_000, 39)])
def test_four_staged_groups(mh, monkeypatch, D, P, K, n, F):
    from paper_2311_06952_amd import capi
    monkeypatch.setenv("MHDEOCT_PERSIST", "1")
    monkeypatch.setenv("MHDEOCT_PERSIST_RESIDENT", "0")
    monkeypatch.setenv("MHDEOCT_PERSIST_HALVES", "4")
    X, y = synth.random_small(D * 1000 + P, n, F, K, levels=50 if K == 5 else None)
    ctx = capi.Context(0)
    _check(mh, ctx, X, y, K, D, (P, 7, -1.0 if K > 3 else 0.5, 0.7, 77 + D, 2, 0.5))
    ctx.close()


def test_four_staged_groups_by_size(mh):
    """More tiles than the LDS of the chip holds: taken without being asked for."""
    from paper_2311_06952_amd import capi
    X, y = synth.random_small(5, 175_000, 20, 3)
    ctx = capi.Context(0)
    _check(mh, ctx, X, y, 3, 3, (9, 3, 0.5, 0.9, 3, 1, 0.0))
    ctx.close()


@pytest.mark.parametrize("share", [0.004, 0.31, 0.97])
def test_problems_of_unequal_size(mh, monkeypatch, share):
    """The blocks of a launch follow the problems' tiles: the left child of the
    first split holds about this share of the samples."""
    from paper_2311_06952_amd import capi
    monkeypatch.setenv("MHDEOCT_PERSIST", "1")
    monkeypatch.setenv("MHDEOCT_PERSIST_RESIDENT", "0")
    n, F, K, D = 16_000, 5, 3, 4
    rng = np.random.default_rng(int(share * 1000))
    X = rng.normal(size=(n, F)).astype(np.float32)
    cut = np.quantile(X[:, 0], share)
    y = np.where(X[:, 0] < cut, 2, (X[:, 1] > 0.3).astype(int)).astype(np.uint8)
    y[rng.random(n) < 0.05] = 1
    prm = (40, 12, 0.5, 0.8, 11, 1, 0.0)
    want = oracle.mh_train(oracle.dataset_from_X(X, y, K), D, 1, oracle.de_params(*prm))
    ctx = capi.Context(0)
    got = mh.mh_train(mh.dataset(X, y, K, ctx=ctx), D, 1, mh.de_params(*prm), batched=True, ctx=ctx)
    ctx.close()
    for key in ("feat", "tau", "label"):
        np.testing.assert_array_equal(got[key], want[key])
    assert got["correct"] == want["correct"] and got["cost"] == want["cost"]


# (D, P, K, n, F): a run that is resident when nothing is asked for, and one of
# four staged groups
@pytest.mark.parametrize("D,P,K,n,F", [(3, 100, 2, 2000, 4), (2, 9, 3, 175_000, 20)])
@pytest.mark.parametrize("switch,value,groups", [
    ("MHDEOCT_PERSIST_HALVES", "1", 1), ("MHDEOCT_PERSIST_HALVES", "2", 2),
    ("MHDEOCT_PERSIST_BLOCKS_PER_CU", "1", 2)])
def test_asked_groups_and_blocks_run(mh, monkeypatch, capfd, switch, value, groups, D, P, K, n, F):
    """Groups or blocks per CU that are asked for are those that run."""
    from paper_2311_06952_amd import capi
    monkeypatch.setenv(switch, value)
    monkeypatch.setenv("MHDEOCT_DEBUG", "1")
    X, y = synth.random_small(D * 100 + P, n, F, K)
    ctx = capi.Context(0)
    capfd.readouterr()
    _check(mh, ctx, X, y, K, D, (P, 3, 0.5, 0.9, 3, 1, 0.0))
    err = capfd.readouterr().err
    ctx.close()
    assert "k_deoct_resident" not in err
    assert f"k_deoct_persist<{D},{(P + 63) // 64},{groups}," in err


@pytest.mark.parametrize("D,P,K,n,F,form", [
    (3, 100, 2, 2000, 4, "k_deoct_resident<"), (2, 9, 3, 175_000, 20, "k_deoct_persist<2,1,4,")])
def test_tuner_times_the_form_of_its_own_choice(mh, monkeypatch, capfd, D, P, K, n, F, form):
    """Twelve candidates, one of them the form that runs when nothing is tuned
    (0 blocks per CU); later runs take the winner's form."""
    from paper_2311_06952_amd import capi
    monkeypatch.setenv("MHDEOCT_DEBUG", "1")
    X, y = synth.random_small(D * 100 + P, n, F, K)
    ctx = capi.Context(0)
    ds = mh.dataset(X, y, K, ctx=ctx)
    capfd.readouterr()
    tuned = mh.autotune(ds, D, mh.de_params(P, 5, 0.5, 0.9, 3), generations=5, ctx=ctx)
    lines = [e for e in capfd.readouterr().err.splitlines() if e.startswith("k_deoct")]
    own = [e for e in lines if e.startswith(form)]
    assert len(tuned["ms"]) == 12
    # each candidate runs four times; four groups are asked for at 1, 2 and 4 blocks too
    assert len(own) == (4 if "resident" in form else 16)
    assert len(lines) == 36
    prm = (P, 5, 0.5, 0.9, 8, 1, 0.0)
    _check(mh, ctx, X, y, K, D, prm)
    err = capfd.readouterr().err
    ctx.close()
    if tuned["persist"] == 0:
        assert "k_deoct" not in err
    elif tuned["persist_blocks_per_cu"] == 0:
        assert form in err
    else:
        assert f"k_deoct_persist<{D},{(P + 63) // 64},{tuned['halves']}," in err


@pytest.mark.parametrize("D,D_MH", [(4, 2), (5, 3)])
@pytest.mark.parametrize("share", [0.004, 0.31, 0.97])
@pytest.mark.parametrize("resident", ["0", "1"])
def test_runs_of_unequal_problems(mh, monkeypatch, capfd, resident, share, D, D_MH):
    """Several problems of very different sizes in one launch of the staged
    whole-run kernel and, its blocks scaled down to the CUs, of the resident
    one."""
    from paper_2311_06952_amd import capi
    monkeypatch.setenv("MHDEOCT_PERSIST", "1")
    monkeypatch.setenv("MHDEOCT_PERSIST_RESIDENT", resident)
    monkeypatch.setenv("MHDEOCT_DEBUG", "1")
    n, F, K = 120_000, 5, 3
    rng = np.random.default_rng(int(share * 1000) + D_MH)
    X = rng.normal(size=(n, F)).astype(np.float32)
    cut = np.quantile(X[:, 0], share)
    y = np.where(X[:, 0] < cut, 2, (X[:, 1] > 0.3).astype(int)).astype(np.uint8)
    y[rng.random(n) < 0.05] = 1
    prm = (20, 6, 0.5, 0.8, 11, 1, 0.0)
    want = oracle.mh_train(oracle.dataset_from_X(X, y, K), D, D_MH, oracle.de_params(*prm))
    ctx = capi.Context(0)
    ds = mh.dataset(X, y, K, ctx=ctx)
    capfd.readouterr()
    got = mh.mh_train(ds, D, D_MH, mh.de_params(*prm), batched=True, ctx=ctx)
    err = capfd.readouterr().err
    ctx.close()
    runs = [int(e.split()[1]) for e in err.splitlines() if e.startswith("k_deoct_resident")]
    assert bool(runs) == (resident == "1" and D_MH == 3)
    if runs and share > 0.3:  # (their own best numbers of blocks add up to more than the CUs)
        assert max(runs) >= 3
    assert len(runs) + err.count("k_deoct_persist") == D - 1
    for key in ("feat", "tau", "label"):
        np.testing.assert_array_equal(got[key], want[key])
    assert got["correct"] == want["correct"] and got["cost"] == want["cost"]


@pytest.mark.parametrize("halves,ms", [("", 20), ("2", 2000)])
def test_four_groups_give_up_sooner(mh, monkeypatch, capfd, halves, ms):
    """Blocks of four groups that fill a CU can be kept from starting by waves
    of another stream: they wait for each other 20 ms, not 2 s."""
    from paper_2311_06952_amd import capi
    if halves:
        monkeypatch.setenv("MHDEOCT_PERSIST_HALVES", halves)
    monkeypatch.setenv("MHDEOCT_DEBUG", "1")
    X, y = synth.random_small(5, 175_000, 20, 3)
    ctx = capi.Context(0)
    capfd.readouterr()
    _check(mh, ctx, X, y, 3, 3, (9, 3, 0.5, 0.9, 3, 1, 0.0))
    err = capfd.readouterr().err
    ctx.close()
    assert f"waits up to {ms} ms" in err

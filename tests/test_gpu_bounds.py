"""The bounded search against the evaluation of every configuration (GPU, through the C ABI).

Large spaces are evaluated by a search that decides units, strips, columns and configurations by
bounds; smaller ones evaluate every configuration, which the oracle checks elsewhere.  Here a random
space is given enough hardware samples that it takes the search, and each sample's groups are
compared bit for bit (bucket tables, best, weight samples) with the same samples in spaces small
enough to be evaluated in full, whose groups and ids are the same up to their base.  Which way each
space went is asserted.  The exact staircases, whose candidate pass is the search's in either, are
compared with the oracle's.
"""

import copy

import numpy as np
import pytest

from oracle import oracle as O
from paper_2503_19050_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "a GPU is required"
    torch.cuda.init()
    return torch


BOUNDED, BOUNDED_ALPHA = 1.3e8, 6.3e8   # configurations from which the search runs, and some more
ORACLE = 3_000_000                      # configurations of a group whose staircase the oracle forms
FULL = 1.0e8                            # and below which every configuration is evaluated


def _space(seed, R, n_alpha, factors):
    """A random model and space with R ratios and groups large enough for the search, and enough
    hardware samples: budgets from far too small to roomy, factors seeded, all 1, up to 50, up to 2^12
    (where the slope bound is off) or one of 2^17 (where bounds on the objective are off)."""
    rng = np.random.default_rng(seed)
    wl = W.random_space(seed)
    grid = [0.0] if rng.random() < 0.7 else [0.04]
    wl["space"]["ratios"] = sorted(grid + list(rng.uniform(0.05, 1.0, R - 1)))
    if rng.random() < 0.5:
        wl["space"]["ratios"][-1] = 1.0
    wl["space"]["n_buckets"] = int(rng.choice([1, 7, 33, 64]))
    wl["space"]["l_rule"] = W.L_BALANCED
    wl["model"]["n_layers"] = {2: 400, 3: 160, 4: 60, 5: 24, 6: 12}.get(R, 5 if R < 11 else 2)
    if R <= 4:
        wl["space"].update(n_devices=2, global_batch=32, mb=[1, 2, 4, 8])
    wl["space"].pop("alphas", None)
    if n_alpha:
        wl["space"]["alphas"] = [float(x) for x in rng.choice([0.0, 1.0, 0.5, 0.03, 0.9, 0.999999], n_alpha)]
    one = copy.deepcopy(wl)
    one["hws"] = one["hws"][:1]
    o = O.Oracle(one)
    if o.n_configs == 0 or o.n_configs / o.n_groups < (31000 if n_alpha else 8500) or not 3e5 < o.n_configs < 5e7:
        return None
    n_hw = int((BOUNDED_ALPHA if n_alpha else BOUNDED) // o.n_configs) + 1
    wl["hws"] = []
    for i in range(n_hw):
        hw = W.hw_sample(seed * 1000 + i, {"mem_bytes": 10.0 ** rng.uniform(6.0, 10.0)})
        if factors == "unit":
            hw["phi"] = [[1.0] * 4 for _ in range(16)]
        elif factors == "large":
            hw["phi"] = [[1.0 + 49.0 * rng.random() for _ in range(4)] for _ in range(16)]
        elif factors == "wide":
            hw["phi"] = [[2.0 ** (12.0 * rng.random()) for _ in range(4)] for _ in range(16)]
        elif factors == "huge":
            hw["phi"][int(rng.choice([13, 15, 5, 12]))][int(rng.choice([0, 2, 3]))] = 2.0 ** 17
        wl["hws"].append(hw)
    return wl, o.n_configs, o.n_groups


def _results(S, n_alpha):
    S.eval()
    ids, objs, masks = S.buckets()
    best = S.best_array()
    out = {"ids": ids, "objs": objs, "masks": masks, "best": best["id"].copy(), "bobj": best["obj"].copy()}
    if n_alpha:
        from paper_2503_19050_amd import mist
        raw = (mist.Result * (S.n_groups * n_alpha))()
        assert S.L.mist_get_alpha(S.h, 0, S.n_groups, raw) == 0
        al = np.ctypeslib.as_array(raw)
        out["aid"], out["aobj"] = al["id"].copy(), al["obj"].copy()
    return out


def _check_stairs(S, wl, n1, g1):
    """The exact staircases of a few groups, of different machines, against the oracle's."""
    S.eval_pareto_exact()
    n = 0
    for g in range(S.n_groups // 26, S.n_groups, max(1, S.n_groups // 13)):
        if S.group_key(g)["size"] > ORACLE:
            continue
        h = g // g1
        want = O.Oracle(dict(wl, hws=[wl["hws"][h]])).pareto_exact(g - h * g1)
        got = S.pareto_exact(g)
        assert [r["id"] for r in got] == [int(i) + h * n1 for i in want["id"]], g
        assert [r["obj"] for r in got] == want["obj"].tolist() and [r["mem"] for r in got] == want["mem"].tolist(), g
        n += 1
    return n


@pytest.mark.parametrize("R, n_alpha, factors", [
    (2, 0, "seeded"), (3, 0, "large"), (4, 0, "unit"), (5, 0, "huge"), (5, 0, "seeded"), (6, 0, "large"),
    (7, 0, "seeded"), (9, 0, "unit"), (11, 0, "seeded"), (16, 0, "large"),
    (4, 1, "seeded"), (5, 3, "large"), (6, 16, "seeded"), (7, 4, "wide"), (9, 8, "huge"), (11, 2, "unit"),
])
def test_search_equals_full_evaluation(R, n_alpha, factors, torch_cuda):
    from paper_2503_19050_amd import mist
    found = stairs = 0
    for seed in range(7000 + 100 * R, 7100 + 100 * R):
        made = _space(seed, R, n_alpha, factors)
        if made is None:
            continue
        wl, n1, g1 = made
        print("bounds: R", R, "seed", seed, "hw", len(wl["hws"]), "configurations per hw", n1, flush=True)
        S = mist.from_workload(wl)
        assert S.searched()
        got = _results(S, n_alpha)
        stairs += _check_stairs(S, wl, n1, g1)
        S.close()
        part = max(1, int(FULL // n1) if n1 < FULL else 1)
        none = np.uint64(mist.MIST_NONE)
        for h in range(0, len(wl["hws"]), part):
            sub = dict(wl, hws=wl["hws"][h:h + part])
            g0, base = h * g1, np.uint64(h * n1)
            F = mist.from_workload(sub)
            assert not F.searched()
            want = _results(F, n_alpha)
            n = F.n_groups
            F.close()
            shift = lambda x: np.where(x == none, none, x + base)  # noqa: E731
            assert np.array_equal(got["objs"][g0:g0 + n], want["objs"])
            assert np.array_equal(got["ids"][g0:g0 + n], shift(want["ids"]))
            assert np.array_equal(got["masks"][g0:g0 + n], want["masks"])
            assert np.array_equal(got["best"][g0:g0 + n], shift(want["best"]))
            assert np.array_equal(got["bobj"][g0:g0 + n], want["bobj"])
            if n_alpha:
                at = slice(g0 * n_alpha, (g0 + n) * n_alpha)
                assert np.array_equal(got["aobj"][at], want["aobj"])
                assert np.array_equal(got["aid"][at], shift(want["aid"]))
        found += 1
        if found == 2:
            break
    assert found == 2 and stairs > 0

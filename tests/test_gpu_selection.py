"""Top_maxO where the ranking needs more than the upper half of the keys, and
around the sizes of the selection's pools, against the oracle bit for bit
(norms given, so both sides hold identical float64 keys)."""
import numpy as np
import pytest

from gpu_util import assert_step_matches, require_gpu
from oracle import Controller as Oracle

pytestmark = pytest.mark.gpu


def run(U, base, max_o, alpha=1.1, budget=0, lock_len=2):
    torch = require_gpu()
    from paper_2606_00539_amd import Controller

    ora = Oracle(U, window=5, max_o=max_o, lock_len=lock_len, eps=1e-12,
                 budget_mode=budget)
    dn = torch.empty(U, dtype=torch.float64, device="cuda")
    with Controller(U, 5, max_o, lock_len, 1e-12, np.zeros(U + 1), [], [],
                    budget_mode=budget) as ctl:
        for t, n in enumerate(base, start=1):
            dn.copy_(torch.from_numpy(n))
            ctl.step_from_norms(dn, alpha, 1.5)
            ref = ora.step(n, alpha, 1.5)
            assert_step_matches(ctl.query(), ref, rtol=1e-14, what=f"U={U} t={t}")


@pytest.mark.parametrize("U", [200, 1000, 3000])
@pytest.mark.parametrize("spread", [1e-9, 1e-13])
@pytest.mark.parametrize("budget", [0, 1])
def test_near_ties_at_the_cut(U, spread, budget):
    """150 units spike with risks a relative `spread` apart (equal in the upper
    32 bits of the keys), some of them exactly equal; the cut falls among them.
    200 and 1000 units: the single-workgroup step; 150 candidates: past the
    directly counted pools."""
    print(f"near ties U={U} spread={spread} budget={budget}", flush=True)
    rng = np.random.default_rng(U)
    base = np.exp(rng.normal(scale=0.01, size=(9, U)))
    near = rng.permutation(U)[:150]
    base[:, near] = base[:, near[:1]]
    base[6, near] *= 6.0 * (1.0 + spread * rng.integers(0, 40, 150))
    base[6, near[:10]] *= 2.0
    run(U, base, max_o=64, budget=budget)


@pytest.mark.parametrize("pool", [16383, 16384, 16385])
def test_pools_at_the_lds_capacity(pool):
    """As many candidates as the selection holds in LDS, one fewer and one more
    (ranked from memory then), distinct and tied risks at the cut."""
    print(f"selection pool of {pool}", flush=True)
    U = 17000
    rng = np.random.default_rng(pool)
    base = np.exp(rng.normal(scale=0.01, size=(8, U)))
    hot = rng.permutation(U)[:pool]
    base[6, hot] *= 6.0
    base[7, hot[:200]] = base[7, hot[0]]
    run(U, base, max_o=100, lock_len=0)


@pytest.mark.parametrize("U,max_o", [(42, 0), (5000, 0), (300000, 64)])
def test_every_unit_triggers(U, max_o):
    """alpha = 0.4: every unit is a candidate; 300,000 units are more K2
    workgroups than the selection has threads."""
    print(f"every unit triggers U={U}", flush=True)
    rng = np.random.default_rng(U)
    run(U, np.exp(rng.normal(scale=0.05, size=(4, U))), max_o=max_o, alpha=0.4)


@pytest.mark.parametrize("U", [1500, 6000])
def test_few_candidates_among_many_workgroups(U):
    """Units summed by a wavefront (40 items each: four units to a K2
    workgroup) or a whole workgroup (600 items): candidates in scattered
    workgroups, more of these than the selection has threads."""
    torch = require_gpu()
    from paper_2606_00539_amd import Controller

    for parts in (40, 600):
        if U * parts > 2_000_000:
            continue
        print(f"selection from partials U={U} parts={parts}", flush=True)
        rng = np.random.default_rng(U + parts)
        ora = Oracle(U, window=5, max_o=32, lock_len=2, eps=1e-12)
        with Controller(U, 5, 32, 2, 1e-12, np.zeros(U + 1, np.int64), [], []) as ctl:
            ctl.bind_partials(np.arange(U + 1, dtype=np.int64) * parts)
            for t in range(1, 9):
                # partials that are powers of four: sums and roots without rounding doubt
                scale = np.where(rng.random(U) < (0.05 if t == 7 else 0.0), 2.0 ** rng.integers(2, 6, U), 1.0)
                part = np.repeat((scale * scale).astype(np.float32), parts)
                ctl.step_from_partials(torch.from_numpy(part).to("cuda"), 1.1, 1.5)
                ref = ora.step(np.sqrt(scale * scale * parts), 1.1, 1.5)
                assert_step_matches(ctl.query(), ref, rtol=1e-14, what=f"parts={parts} t={t}")


@pytest.mark.parametrize("U,parts", [(1, 1), (1024, 10), (1024, 11), (1025, 1), (32, 320),
                                     (32, 321), (33, 100), (8, 1280), (8, 1281), (9, 600),
                                     (1, 10240), (1, 10241)])
def test_one_and_two_launch_steps(U, parts):
    """Around the limits of the single-workgroup step from partials: a unit by
    one thread, a wavefront and a workgroup, in one launch and in two.  Units
    of differing sizes, random partials: norms within float64 rounding of the
    sums in another order, decisions the oracle's."""
    torch = require_gpu()
    from paper_2606_00539_amd import Controller

    print(f"step from partials U={U} parts={parts}", flush=True)
    rng = np.random.default_rng(U * 7 + parts)
    sizes = np.full(U, parts)
    if U > 1:                      # the same total: one unit gives, another takes
        sizes[0] -= parts // 3
        sizes[-1] += parts // 3
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    max_o = max(1, U // 4)
    ora = Oracle(U, window=5, max_o=max_o, lock_len=2, eps=1e-12)
    with Controller(U, 5, max_o, 2, 1e-12, np.zeros(U + 1, np.int64), [], []) as ctl:
        ctl.bind_partials(off)
        for t in range(1, 9):
            scale = np.where(rng.random(U) < (0.5 if t == 7 else 0.0), 30.0 + 10 * rng.random(U),
                             1.0)
            part = ((0.999 + 0.002 * rng.random(int(off[-1]))) *
                    np.repeat(scale, sizes)).astype(np.float32)
            ctl.step_from_partials(torch.from_numpy(part).to("cuda"), 1.1, 1.5)
            sums = [part[off[b]:off[b + 1]].astype(np.float64).sum() for b in range(U)]
            ref = ora.step(np.sqrt(np.array(sums)), 1.1, 1.5)
            # float64 sums of up to 10,241 positive terms in two orders: 2 n 2^-53
            assert_step_matches(ctl.query(), ref, rtol=1e-11, what=f"t={t}")


# Sparse pools over more K2 workgroups of 256 units than the selection has threads
# (two, four and five to a thread, the last one ragged): scattered candidates and
# neighbouring ones, up to one and several rounds of threads.
@pytest.mark.parametrize("U,pool,together", [
    (262145, 300, False), (262145, 1025, True), (300000, 1000, False), (524289, 2500, True),
    (700001, 9000, False), (1048577, 1, False), (1048577, 16384, True)])
def test_sparse_pool_of_many_units(U, pool, together):
    print(f"sparse pool U={U} pool={pool} together={together}", flush=True)
    rng = np.random.default_rng(U + pool)
    base = np.exp(rng.normal(scale=0.01, size=(3, U)))
    hot = np.arange(U - pool, U) if together else rng.permutation(U)[:pool]
    base[1:, hot] *= 3.0 + rng.random((2, pool))
    run(U, base, max_o=max(0, pool // 3), alpha=1.2)


# Every candidate tied, exactly or within the keys' lower halves, and half of them
# non-finite: in registers, in LDS and in memory, cut within the tie.
@pytest.mark.parametrize("U", [130, 1000, 3000, 16385, 42496])
@pytest.mark.parametrize("kind", ["equal", "near", "infinite", "half"])
def test_ties_over_the_whole_pool(U, kind):
    print(f"whole pool tied U={U} {kind}", flush=True)
    rng = np.random.default_rng(U)
    base = np.ones((4, U))
    if kind == "near":
        base[2:] *= 1.0 + 1e-14 * rng.integers(0, 5, (2, U))
    elif kind == "infinite":
        base[2:] = np.inf
    elif kind == "half":
        base *= np.exp(rng.normal(scale=0.05, size=(4, U)))
        base[2:, rng.permutation(U)[:U // 2]] = np.inf
    for max_o in (1, U // 3, U - 1):
        run(U, base, max_o=max_o, alpha=0.4)

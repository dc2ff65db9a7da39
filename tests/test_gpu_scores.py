"""Per-plan scores where the kernels' pieces change, against the fp64 oracle:
ranges that do not begin at a multiple of 64 outputs, and per-backend pressure
by the kernel of four levels at a time (levels about the staged 4 and 8, DAGs
about the unrolled 8, 16, 24 and 32 nodes, tables too large for LDS, word and
byte rows, 64-bit plan indices, bad row ids).

Tolerance: fp32 products, sums and maxima of at most 32 rounded terms are
within 2 N 2^-24 <= 3.9e-6 of the fp64 values; feasibility bits are exact."""
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as orc  # noqa: E402
from paper_2607_02942_amd import dyplan as D  # noqa: E402
from paper_2607_02942_amd import workload as wl  # noqa: E402

from test_gpu_parity import assert_scores, run_score  # noqa: E402
from test_gpu_range_sweep import problem  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    D.lib()
    torch.cuda.set_device(0)
    yield


@pytest.mark.parametrize("radix", [[5, 4, 1], [3, 5, 4, 7], [6, 7, 12], [2, 3, 255], [97], [9, 31, 2], [9, 31, 3]])
@pytest.mark.parametrize("K", [1, 4, 5, 8])
def test_range_scores_at_any_begin(radix, K):
    rng = np.random.default_rng([len(radix), K])
    prob = problem(rng, radix, K, True)
    total = prob.n_plans()
    with D.Plan(prob) as plan:
        for begin, count in ((0, total), (1, total - 1), (63 % total, total - 63 % total), (total // 3, 1),
                             (total // 2, total // 3 + 1)):
            count = max(1, min(count, total - begin))
            got = run_score(plan, D.range_source(0, begin, count), count, K)
            assert_scores(got, orc.score_range(prob, begin, count), f"{radix} K {K} [{begin}+{count}]")


@pytest.mark.parametrize("K", [1, 4, 7, 8, 9, 32])
@pytest.mark.parametrize("n,R", [(1, 7), (2, 5), (8, 6), (9, 6), (16, 5), (17, 6), (24, 36), (25, 4), (32, 3), (20, 80),
                                 (30, 250)])
def test_class_rows(n, R, K):
    rng = np.random.default_rng([n, R, K])
    prob = problem(rng, [R] * n, K, False, edge_p=0.3)
    assert not (prob.rho == prob.rho[:, :1]).all()
    m = 300
    rows = rng.integers(0, R, (m, n)).astype(np.uint8)
    want = orc.score_rows(prob, rows)
    for stride in (n, (n + 3) // 4 * 4, n + 1):
        buf = np.zeros((m, stride), np.uint8)
        buf[:, :n] = rows
        d = torch.from_numpy(buf).cuda()
        with D.Plan(prob) as plan:
            got = run_score(plan, D.rows_source(0, d, m, stride), m, K)
        assert_scores(got, want, f"{n} nodes, {R}, K {K}, stride {stride}")


def test_class_ranges_and_bad_rows():
    rng = np.random.default_rng(4)
    prob = problem(rng, [4, 1, 6, 5, 3, 7], 6, False)
    total = prob.n_plans()
    with D.Plan(prob) as plan:
        for begin, count in ((0, total), (77, total - 100), (total - 1, 1)):
            got = run_score(plan, D.range_source(0, begin, count), count, 6)
            assert_scores(got, orc.score_range(prob, begin, count), f"[{begin}+{count}]")
        rows = np.zeros((70, 6), np.uint8)
        rows[33, 2] = 6  # an id past the node's radix: NaN scores, no feasible level
        c, cp, dem, feas = run_score(plan, D.rows_source(0, torch.from_numpy(rows).cuda(), 70, 6), 70, 6)
    assert np.isnan(c[33]) and np.isnan(cp[33]).all() and np.isnan(dem[33]) and feas[33] == 0
    ok = np.arange(70) != 33
    assert np.isfinite(c[ok]).all() and np.isfinite(cp[ok]).all()
    # 64-bit plan indices
    big = problem(rng, [40] * 8, 3, False)
    begin = 40 ** 8 - 999
    with D.Plan(big) as plan:
        got = run_score(plan, D.range_source(0, begin, 900), 900, 3)
    rows = np.stack([orc.decode(big, begin + i) for i in range(900)]).astype(np.uint8)
    assert_scores(got, orc.score_rows(big, rows), "64-bit indices")


def test_class_feasibility_on_the_bound():
    # every plan's CP_k equals the bound at level 0: fp64 decides each
    prob = problem(np.random.default_rng(8), [3, 4, 2, 3], 3, False)
    prob = dataclasses.replace(prob, tau=np.full_like(prob.tau, np.float32(0.1)),
                               rho=np.array([[0.0, 0.0], [0.2, 0.0], [0.5, 0.1]], np.float32))
    total = prob.n_plans()
    cps = orc.cp0_values(prob, 0, total)
    prob.slo = float(np.float32(cps.max()))
    with D.Plan(prob) as plan:
        got = run_score(plan, D.range_source(0, 0, total), total, 3)
    assert_scores(got, orc.score_range(prob, 0, total), "bound")

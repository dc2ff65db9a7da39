"""Per-plan scores where the kernels' pieces change, against the fp64 oracle:
ranges that begin anywhere.

Tolerance: fp32 products, sums and maxima of at most 32 rounded terms are
within 2 N 2^-24 <= 3.9e-6 of the fp64 values; feasibility bits are exact."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as orc  # noqa: E402
from paper_2607_02942_amd import dyplan as D  # noqa: E402

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


@pytest.mark.parametrize("radix", [[5, 4, 1], [3, 5, 4, 7], [6, 7, 12], [2, 3, 255], [97]])
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

"""GPU parity of the range sweep that folds the last three nodes into tables.

Against the fp64 oracle, at the sizes where its pieces change: one to four
nodes (folded nodes missing), the last unrolled head and the first looped one,
one implementation and the most a node can have, one and 32 levels, ranges
that cut heads at both ends, one workgroup and several, several sinks, no edge
between the last two nodes, unequal pressure, levels nothing meets.  Selections
are decided in 64 bits, so the bar is equality.
"""
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as orc  # noqa: E402
from paper_2607_02942_amd import dyplan as D  # noqa: E402
from paper_2607_02942_amd import workload as wl  # noqa: E402

from test_gpu_objective import assert_obj_choices  # noqa: E402
from test_gpu_parity import assert_choices, run_score, stream  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    D.lib()
    torch.cuda.set_device(0)
    yield


def problem(rng, radix, K, uniform, edge_p=0.4, tau_zero=False):
    n, R = len(radix), max(radix)
    edges = [(i, j) for i in range(n) for j in range(i + 1, n) if rng.random() < edge_p]
    tau = rng.lognormal(0.0, 0.7, (n, R)).astype(np.float32)
    if tau_zero:
        tau[rng.random((n, R)) < 0.5] = 0.0
    rho = np.sort(rng.uniform(0.0, 0.9, K))[:, None] * (np.ones((1, 2)) if uniform else rng.uniform(0.3, 1.0, (1, 2)))
    prob = wl.Problem(n_nodes=n, edges=np.array(edges, np.int32).reshape(-1, 2), radix=np.array(radix, np.int32),
                      p=rng.uniform(0.3, 1.0, (n, R)).astype(np.float32), tau=tau,
                      size=np.ones((n, R), np.float32), backend=rng.integers(0, 2, (n, R)).astype(np.int32),
                      w=rng.uniform(0.0, 1.0, n).astype(np.float32), rho=rho.astype(np.float32), slo=0.0)
    # (for spaces beyond counting, the middle of a random sample's path lengths)
    ids = [rng.integers(0, r, 999) for r in radix]
    f = []
    for v in range(n):
        pr = [u for u, w in edges if w == v]
        f.append(tau[v, ids[v]] + (np.max([f[u] for u in pr], axis=0) if pr else 0.0))
    prob.slo = float(np.float32(np.median(np.max(f, axis=0)) * rng.uniform(0.6, 1.6)))
    return prob


SHAPES = {
    "one": [7], "two": [5, 9], "three": [4, 1, 6], "four": [1, 3, 8, 5], "tools": [1, 1, 6, 1, 7, 1, 5, 1],
    "wide_y": [3, 4, 255], "wide_x": [3, 255, 4], "wide_w": [2, 255, 3, 4], "wide_head": [255, 2, 3, 4],
    "head8": [2, 3, 2, 2, 3, 2, 2, 2, 3, 4, 5], "head9": [2, 3, 2, 2, 2, 3, 2, 2, 2, 3, 4, 5],
    "deep": [2] * 18, "six": [12] * 6, "big_table": [3, 2, 60, 40, 55, 3],
}


@pytest.mark.parametrize("mode", ["level", "class", "objective"])
@pytest.mark.parametrize("shape", sorted(SHAPES))
def test_shapes(shape, mode):
    rng = np.random.default_rng([sorted(SHAPES).index(shape), len(mode)])
    radix = SHAPES[shape]
    for trial in range(4):
        K = [1, 32, 5, 7][trial]
        prob = problem(rng, radix, K, mode != "class", edge_p=[0.4, 0.0, 1.0, 0.5][trial], tau_zero=trial == 3)
        total = prob.n_plans()
        begin = int(rng.integers(0, max(1, total // 3))) if trial else 0
        count = int(rng.integers(1, total - begin + 1)) if trial else total
        srcs = [D.range_source(0, begin, count), D.range_source(0, total - 1, 1)]
        ctx = f"{shape} {mode} trial {trial} [{begin}+{count}]"
        if mode == "objective":
            obj = wl.paper_objective(prob, levels=np.sort(rng.uniform(0, 4, K)), lambda_l=[0.05, 0.0, 0.4, 2.0][trial],
                                     lambda_c=[0.01, 0.5, -0.1, 0.0][trial],
                                     is_tool=(rng.random(len(radix)) < 0.3).astype(np.int32))
            with D.Plan((prob, obj)) as plan:
                got = plan.select(srcs, stream=stream())
            for g, s in zip(got, srcs):
                assert_obj_choices(g, orc.obj_select_range(prob, obj, s.begin, s.count), ctx)
        else:
            with D.Plan(prob) as plan:
                got = plan.select(srcs, stream=stream())
            for g, s in zip(got, srcs):
                assert_choices(g, orc.select_range(prob, s.begin, s.count), ctx)


@pytest.mark.parametrize("mode", ["level", "class", "objective"])
@pytest.mark.parametrize("shape", ["narrow", "wide"])
def test_most_nodes(shape, mode):
    # 32 nodes: the launch with the most LDS (recurrence columns for the sweep
    # and the seeding, every table at its largest)
    rng = np.random.default_rng([32, len(shape), len(mode)])
    radix = [1] * 18 + [2] * 11 + [3, 4, 2] if shape == "narrow" else [1] * 17 + [2] * 13 + [255, 3]
    K = 32 if shape == "narrow" else 4
    prob = problem(rng, radix, K, mode != "class", edge_p=0.1)
    total = prob.n_plans()
    srcs = [D.range_source(0, 0, 3001), D.range_source(0, total - 4099, 4099), D.range_source(0, total // 3, 1500)]
    obj = wl.paper_objective(prob, levels=np.sort(rng.uniform(0, 4, K))) if mode == "objective" else None
    with D.Plan((prob, obj) if obj else prob) as plan:
        got = plan.select(srcs, stream=stream())
    for g, s in zip(got, srcs):
        if obj:
            assert_obj_choices(g, orc.obj_select_range(prob, obj, s.begin, s.count), f"{shape} {mode}")
        else:
            assert_choices(g, orc.select_range(prob, s.begin, s.count), f"{shape} {mode}")


@pytest.mark.parametrize("mode", ["level", "class", "objective"])
def test_mixed_batch_repeats(mode):
    # sources of different depths and sizes in one launch, some cut, one of
    # several workgroups; repeated calls list the same candidates
    rng = np.random.default_rng(5)
    shapes = [[7], [5, 9], [6, 5, 4], [12] * 5, [2] * 15, [9, 8, 7, 6, 5, 4, 3], [20, 20, 20, 20, 5]]
    probs = [problem(rng, r, 4, mode != "class") for r in shapes]
    objs = [wl.paper_objective(p) for p in probs]
    srcs, want = [], []
    for j, p in enumerate(probs):
        total = p.n_plans()
        b = int(rng.integers(0, total))
        for begin, count in ((0, total), (b, total - b)):
            srcs.append(D.range_source(j, begin, count))
            want.append(orc.obj_select_range(p, objs[j], begin, count) if mode == "objective"
                        else orc.select_range(p, begin, count))
    items = list(zip(probs, objs)) if mode == "objective" else probs
    cands = []
    with D.Plan(items) as plan:
        for call in range(3):
            got = plan.select(srcs, stream=stream())
            cands.append(plan.stats().candidates)
            for q, (g, w) in enumerate(zip(got, want)):
                (assert_obj_choices if mode == "objective" else assert_choices)(g, w, f"{mode} call {call} source {q}")
    assert len(set(cands)) == 1, cands


def test_class_levels_out_of_order():
    # durations of a later level below those of an earlier one, and levels
    # whose bound no plan meets: each level's own sweep finds its choice
    rng = np.random.default_rng(17)
    for trial in range(6):
        prob = problem(rng, [6, 5, 7, 4, 6], 6, False)
        rho = rng.uniform(0.0, 0.95, (6, 2)).astype(np.float32)
        rho[2] = 0.0
        rho[4] = 0.995
        prob = dataclasses.replace(prob, rho=rho)
        total = prob.n_plans()
        with D.Plan(prob) as plan:
            got = plan.select([D.range_source(0, 0, total)], stream=stream())[0]
        assert_choices(got, orc.select_range(prob, 0, total), f"trial {trial}")


@pytest.mark.parametrize("slo", [0.0, 3.0e38, float("inf")])
@pytest.mark.parametrize("uniform", [True, False])
def test_extreme_bounds(slo, uniform):
    prob = dataclasses.replace(problem(np.random.default_rng(3), [5, 6, 4, 3, 5], 4, uniform), slo=slo)
    total = prob.n_plans()
    with D.Plan(prob) as plan:
        got = plan.select([D.range_source(0, 0, total), D.range_source(0, 17, 1000)], stream=stream())
    assert_choices(got[0], orc.select_range(prob, 0, total), "whole")
    assert_choices(got[1], orc.select_range(prob, 17, 1000), "part")


def test_all_zero_durations_and_factors():
    # every plan on one bin; factors of 0 (a plan of corr 0 is chosen)
    prob = problem(np.random.default_rng(9), [4, 5, 6, 3], 3, True)
    for p, w, tau in ((0.0, 1.0, 0.0), (0.5, 1.0, 0.0), (0.0, 1.0, 1.0)):
        q = dataclasses.replace(prob, p=np.full_like(prob.p, p), w=np.full_like(prob.w, w),
                                tau=np.full_like(prob.tau, tau), slo=10.0)
        total = q.n_plans()
        with D.Plan(q) as plan:
            got = plan.select([D.range_source(0, 0, total)], stream=stream())[0]
        assert_choices(got, orc.select_range(q, 0, total), f"p {p} tau {tau}")


@pytest.mark.parametrize("mode", ["level", "class"])
def test_overflow_then_other_sources(mode):
    # equal plans overflow a list of 16 (decided exhaustively), near-equal ones
    # are retried on the seeds kept; what the calls after it see is clean
    rng = np.random.default_rng(41)
    tied = problem(rng, [6, 5, 7, 4, 6], 3, mode != "class")
    tied = dataclasses.replace(tied, p=np.full_like(tied.p, 0.8), tau=np.ones_like(tied.tau), slo=1e6)
    near = problem(rng, [8, 8, 8, 8, 8], 3, mode != "class")
    near = dataclasses.replace(near, p=(0.8 + 1e-6 * rng.random(near.p.shape)).astype(np.float32), slo=1e6)
    low = problem(rng, [6, 5, 7, 4, 6], 3, mode != "class")
    low = dataclasses.replace(low, p=low.p * np.float32(0.1))
    probs = [tied, near, low]
    want = [orc.select_range(p, 0, p.n_plans()) for p in probs]
    with D.Plan(probs) as plan:
        plan.set_option(D.DY_OPT_CAND_CAPACITY, 16)
        for order in ([0, 1, 2], [2, 2, 2], [1, 0, 2], [2, 1, 0], [2, 2, 2]):
            got = plan.select([D.range_source(j, 0, probs[j].n_plans()) for j in order], stream=stream())
            for g, j in zip(got, order):
                assert_choices(g, want[j], f"{mode} {order} problem {j}")


@pytest.mark.parametrize("mode", ["level", "class", "objective"])
@pytest.mark.parametrize("radix,count,generated", [
    ([12] * 7 + [2, 1, 2], 1 << 24, 1), ([12] * 7 + [2, 1, 2], (1 << 24) - 1, 0), ([12] * 7 + [5, 1, 1], 1 << 24, 0),
    ([3] * 14 + [8, 4, 4], 1 << 24, 1), ([3] * 14 + [3, 1, 43], 1 << 24, 0), ([12] * 7, 1 << 24, 0)])
def test_generated_where_little_is_folded(radix, count, generated, mode):
    # the route at the edges of its rule, against the library's sweep (exact choices)
    prob = problem(np.random.default_rng(8), radix, 3, mode != "class")
    item = (prob, wl.paper_objective(prob)) if mode == "objective" else prob
    src = [D.range_source(0, 12345, count)]
    got = []
    for jit in (1, 0):
        with D.Plan(item) as plan:
            plan.set_option(D.DY_OPT_JIT, jit)
            got.append([plan.select(src, stream=stream())[0] for _ in range(3)])
            assert plan.stats().generated_jobs == (generated if jit else 0)
    for g in got[0] + got[1]:
        assert repr(g) == repr(got[1][0])  # (NaN where infeasible)


def test_recovered_overflow_of_a_generated_sweep_leaves_no_seeds():
    # a generated sweep samples into every seed slot; its list overflows and the
    # library's sweep recovers it.  The next source in the same job slot has
    # lower factors: a seed left behind would shut out all of its plans
    rng = np.random.default_rng(23)
    high = problem(rng, [12] * 6, 3, True)
    low = dataclasses.replace(high, p=high.p * np.float32(0.1))
    total = high.n_plans()
    want_high, want_low = orc.select_range(high, 0, total), orc.select_range(low, 0, total)
    rows = np.stack([rng.integers(0, 12, 20000) for _ in range(6)], axis=1).astype(np.uint8)
    want_rows = orc.select_rows(low, rows)
    d = torch.from_numpy(rows).cuda()
    with D.Plan([high, low]) as plan:
        plan.set_option(D.DY_OPT_JIT, 2)
        whole = [D.range_source(j, 0, total) for j in range(2)]
        plan.select([whole[0]], stream=stream())
        assert plan.stats().generated_jobs == 1 and plan.stats().candidates > 16  # overflows a list of 16
        plan.set_option(D.DY_OPT_CAND_CAPACITY, 16)
        for jit, src, want in ((2, whole[1], want_low), (2, D.rows_source(1, d, 20000, 6), want_rows),
                               (0, D.rows_source(1, d, 20000, 6), want_rows), (0, whole[1], want_low)):
            plan.set_option(D.DY_OPT_JIT, 2)
            assert_choices(plan.select([whole[0]], stream=stream())[0], want_high, "recovered")
            st = plan.stats()
            assert st.generated_jobs == 1 and st.fallbacks == 0 and st.candidates <= 16
            plan.set_option(D.DY_OPT_JIT, jit)
            assert_choices(plan.select([src], stream=stream())[0], want, f"after it, jit {jit} kind {src.kind}")


def test_candidates_beyond_32_bits():
    # 2^32 plans, every one a candidate: a 32-bit count of them is 0 again
    n = 8
    prob = problem(np.random.default_rng(2), [16] * n, 1, True)
    prob = dataclasses.replace(prob, w=np.zeros(n, np.float32), slo=1e9)
    assert prob.n_plans() == 1 << 32
    with D.Plan(prob) as plan:
        got = plan.select([D.range_source(0, 0, 1 << 32)], stream=stream())[0]
        assert plan.stats().fallbacks == 1
    assert_choices(got, orc.select_range(prob, 0, 1), "equal plans: the first is chosen")


@pytest.mark.parametrize("mode", ["level", "class", "objective"])
@pytest.mark.parametrize("stride", [256, 4096, 65536])
def test_padded_tables(stride, mode):
    # the row stride of the tables may be far above the radices
    rng = np.random.default_rng([stride, len(mode)])
    plain = problem(rng, [6, 5, 7, 4, 3], 3, mode != "class")

    def pad(a):
        b = np.zeros((a.shape[0], stride), a.dtype)
        b[:, :a.shape[1]] = a
        return b
    prob = dataclasses.replace(plain, p=pad(plain.p), tau=pad(plain.tau), size=pad(plain.size),
                               backend=pad(plain.backend))
    total = plain.n_plans()
    objs = [wl.paper_objective(p) if mode == "objective" else None for p in (plain, prob)]
    check, oracle = ((assert_obj_choices, lambda b, c: orc.obj_select_range(plain, objs[0], b, c))
                     if mode == "objective" else (assert_choices, lambda b, c: orc.select_range(plain, b, c)))
    items = [p if o is None else (p, o) for p, o in zip((plain, prob), objs)]
    for probs in (items[1:], items):
        srcs = [D.range_source(j, b, total - b) for j in range(len(probs)) for b in (0, 777)]
        with D.Plan(probs) as plan:
            got = plan.select(srcs, stream=stream())
        for g, s in zip(got, srcs):
            check(g, oracle(s.begin, s.count), f"{mode} stride {stride} [{s.begin}+{s.count}]")


def test_weights_beyond_fp32():
    # durations of zero leave the weights lambda_ld L_k unbounded: at the last
    # level the product exceeds the largest fp32, and J_k = U all the same
    rng = np.random.default_rng(12)
    prob = problem(rng, [6, 5, 7, 4], 1, True)
    prob = dataclasses.replace(prob, tau=np.zeros_like(prob.tau))
    obj = wl.paper_objective(prob, levels=(0.0, 1e10, 1e25), lambda_ld=1e20)
    total = prob.n_plans()
    srcs = [D.range_source(0, 0, total), D.range_source(0, 100, total - 100)]
    with D.Plan((prob, obj)) as plan:
        for climb in (1, 2):
            plan.set_option(D.DY_OPT_CLIMB, climb)
            got = plan.select(srcs, stream=stream())
            for g, s in zip(got, srcs):
                assert_obj_choices(g, orc.obj_select_range(prob, obj, s.begin, s.count), f"[{s.begin}+{s.count}]")
        rows = rng.integers(0, [6, 5, 7, 4], (5000, 4)).astype(np.uint8)
        d = torch.from_numpy(rows).cuda()
        got = plan.select([D.rows_source(0, d, 5000, 4)], stream=stream())[0]
        assert_obj_choices(got, orc.obj_select_rows(prob, obj, rows), "rows")
        for src, n in ((srcs[1], total - 100), (D.rows_source(0, d, 5000, 4), 5000)):
            u, j, _, _ = run_score(plan, src, n, 3)
            assert (j == u[:, None]).all()  # J_k = U, exactly


@pytest.mark.parametrize("mode", ["level", "class", "objective"])
def test_other_sources_on_another_stream(mode):
    # calls of at most 64 sources return on the results' arrival, and the next
    # call uploads other sources on another stream: the surplus workgroups of
    # the first launch (sources of one workgroup beside one of many) must not
    # take the second's descriptors for theirs
    rng = np.random.default_rng([64, len(mode)])
    big = problem(rng, [12] * 7, 2, mode != "class")
    small = [problem(rng, [4, 3, 5], 5, mode != "class") for _ in range(40)]
    probs = [big] + small
    objs = [wl.paper_objective(p) for p in probs]
    order = [list(range(41)), list(range(40, -1, -1))]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    with D.Plan(list(zip(probs, objs)) if mode == "objective" else probs) as plan:
        first = {}
        for call in range(60):
            js = order[call % 2]
            got = plan.select([D.range_source(j, 0, probs[j].n_plans()) for j in js], stream=streams[call % 2])
            for j, g in zip(js, got):
                assert repr(first.setdefault(j, g)) == repr(g), f"call {call} problem {j}"
    for j in range(1, 41):
        if mode == "objective":
            assert_obj_choices(first[j], orc.obj_select_range(probs[j], objs[j], 0, 60), f"problem {j}")
        else:
            assert_choices(first[j], orc.select_range(probs[j], 0, 60), f"problem {j}")


@pytest.mark.parametrize("mode", ["level", "class", "objective"])
@pytest.mark.parametrize("radix", [[5], [3, 4], [3, 1, 4], [2, 3, 2, 3]])
def test_every_range_of_a_space(radix, mode):
    # seeds are constructed in parts of a range; one constructed outside it would
    # shut out its plans
    rng = np.random.default_rng([len(radix), len(mode), 3])
    prob = problem(rng, radix, 3, mode != "class")
    total = prob.n_plans()
    obj = wl.paper_objective(prob) if mode == "objective" else None
    srcs = [D.range_source(0, b, c) for b in range(total) for c in range(1, total - b + 1)]
    with D.Plan((prob, obj) if obj else prob) as plan:
        got = plan.select(srcs, stream=stream())
    for g, s in zip(got, srcs):
        if obj:
            assert_obj_choices(g, orc.obj_select_range(prob, obj, s.begin, s.count), f"{radix} [{s.begin}+{s.count}]")
        else:
            assert_choices(g, orc.select_range(prob, s.begin, s.count), f"{radix} [{s.begin}+{s.count}]")


@pytest.mark.parametrize("mode", ["level", "objective"])
def test_seeds_of_a_range_that_ends_inside_the_space(mode):
    # ranges whose first and last plan part at neighbouring ids: the seeds lie in
    # the large parts below, not next to the ends (tens of thousands of candidates)
    rng = np.random.default_rng(71)
    prob = problem(rng, [12] * 11, 3, True)
    obj = wl.paper_objective(prob) if mode == "objective" else None
    with D.Plan((prob, obj) if obj else prob) as plan:
        plan.set_option(D.DY_OPT_CAND_CAPACITY, 1 << 26)
        for begin, count in ((1 << 33, 1 << 24), ((1 << 33) - 5, 1 << 20), (12 ** 9 - 40, 12 ** 7)):
            plan.select([D.range_source(0, begin, count)], stream=stream())
            assert plan.stats().candidates < 10000, (begin, count, plan.stats().candidates)


@pytest.mark.parametrize("K", [9, 17, 32])
@pytest.mark.parametrize("near", [0.0, 1e-4])
def test_class_levels_that_share_candidates(K, near):
    # levels seeded in several rounds; equal levels, whose sweeps are left out
    # (their candidates are another level's), in spaces of several workgroups
    rng = np.random.default_rng([K, int(near > 0)])
    prob = problem(rng, [12] * 6, K, False)
    rho = np.sort(rng.uniform(0.0, 0.9, K)).astype(np.float32)
    rho[1::3] = rho[0::3][:len(rho[1::3])]
    prob = dataclasses.replace(prob, rho=np.stack([rho, rho * np.float32(0.5)], axis=1))
    if near:  # many plans about the best
        prob = dataclasses.replace(prob, p=(0.8 + near * rng.random(prob.p.shape)).astype(np.float32))
    total = prob.n_plans()
    srcs = [D.range_source(0, 0, total), D.range_source(0, 100003, total - 200000)]
    with D.Plan(prob) as plan:
        for call in range(2):
            got = plan.select(srcs, stream=stream())
            for g, s in zip(got, srcs):
                assert_choices(g, orc.select_range(prob, s.begin, s.count), f"K {K} [{s.begin}+{s.count}] call {call}")


def test_overflows_of_every_kind_in_one_call():
    # sources that end exhaustively after one more sweep (equal plans), after
    # three (per-backend pressure, a generated sweep's), that are recovered, and
    # that never overflow, in one call; each is decided once
    rng = np.random.default_rng(77)
    radix, probs = [6, 5, 7, 4, 6], []
    for uniform in (True, False):
        tied = problem(rng, radix, 3, uniform)
        probs.append(dataclasses.replace(tied, p=np.full_like(tied.p, 0.8), tau=np.ones_like(tied.tau), slo=1e6))
    probs += [dataclasses.replace(problem(rng, [8] * 5, 3, True), slo=1e6), problem(rng, [3, 2], 3, True)]
    want = [orc.select_range(p, 0, p.n_plans()) for p in probs]
    for jit in (0, 2):
        with D.Plan(probs) as plan:
            plan.set_option(D.DY_OPT_CAND_CAPACITY, 16)
            plan.set_option(D.DY_OPT_JIT, jit)
            for call in range(2):
                got = plan.select([D.range_source(j, 0, p.n_plans()) for j, p in enumerate(probs)], stream=stream())
                assert plan.stats().fallbacks == 6  # two sources of three levels
                for g, w in zip(got, want):
                    assert_choices(g, w, f"jit {jit} call {call}")


def test_smaller_call_between_an_overflow_and_a_larger_call():
    # the eighth source of a call ends exhaustively; a call of two sources comes
    # between it and others of eight, whose last job slot must not see what it left
    rng = np.random.default_rng(88)
    low = problem(rng, [6, 5, 7, 4, 6], 3, True)
    low = dataclasses.replace(low, p=low.p * np.float32(0.1), slo=1e6)
    tied = [dataclasses.replace(low, p=np.full_like(low.p, p), tau=np.ones_like(low.tau)) for p in (0.9, 0.1)]
    probs, total = [low] + tied, low.n_plans()
    want = [orc.select_range(p, 0, total) for p in probs]
    rows = np.stack([rng.integers(0, r, 5000) for r in low.radix], axis=1).astype(np.uint8)
    want_rows = orc.select_rows(low, rows)
    d = torch.from_numpy(rows).cuda()
    with D.Plan(probs) as plan:
        plan.set_option(D.DY_OPT_JIT, 0)
        plan.set_option(D.DY_OPT_CAND_CAPACITY, 16)

        def ranges(js):
            got = plan.select([D.range_source(j, 0, total) for j in js], stream=stream())
            for g, j in zip(got, js):
                assert_choices(g, want[j], f"{js} problem {j}")
        for last in ("rows", "tied"):
            ranges([0] * 7 + [1])
            assert plan.stats().fallbacks == 3
            ranges([0, 0])
            if last == "tied":
                ranges([0] * 7 + [2])
            else:
                for g in plan.select([D.rows_source(0, d, 5000, 5)] * 8, stream=stream()):
                    assert_choices(g, want_rows, "rows")

"""Batches and serving at their limits, through the C ABI on MI355X: the grid of the
direct path's shared launch, and HBM budgets around one tile of the planned class."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pa():
    from paper_1805_02372_amd import pa as _pa
    return _pa


def test_direct_batch_beyond_one_grid(pa):
    """1,100 direct jobs of 8,192 workgroups each: together more work-items than
    the 2^32 that a launch may have along one dimension, so the jobs are launched
    one by one (1,000 fit one launch)."""
    from gpu_util import to_dev, from_dev, describe
    import torch
    n, m = 50, 1 << 24
    p = synth.random_problem(np.random.default_rng(3), n, m)
    s, k = to_dev(p.seed), to_dev(p.key)
    ref = oracle.hash_words(p.seed, n, m, p.key)
    dref = to_dev(ref)
    c = pa.pa_create(0, 0, None)
    try:
        for count in (1000, 1100):
            outs = torch.full((count, m // 64), -1, dtype=torch.int64, device="cuda:0")
            torch.cuda.synchronize()
            print(f"{count} jobs", flush=True)
            st, per = pa.pa_hash_batch(c, [(s, k, outs[i], n, m) for i in range(count)], pa.PA_PREC_DIRECT)
            torch.cuda.synchronize()
            assert st == pa.PA_OK and per == [pa.PA_OK] * count, pa.pa_strerror(st)
            assert bool((outs == dref[None, :]).all()), describe(from_dev(outs[count - 1]), ref, m)
            launches = pa.pa_last_stats(c)["launches"]
            assert launches == (1 if count == 1000 else count), launches
            del outs
    finally:
        pa.pa_destroy(c)


# One FP32 tile of this shape's planned class (3 2^20 points and their bit planes)
# is more than 24 MiB; 2^21 points fit.
TIGHT = (3_664_349, 1_086_326)


def _direct(pa, ctx, s, k, n, m):
    from gpu_util import empty_dev, from_dev
    import torch
    out = empty_dev(synth.words_for(m))
    assert pa.pa_hash(ctx, s, n, m, k, out, pa.PA_PREC_DIRECT) == pa.PA_OK
    torch.cuda.synchronize()
    return from_dev(out)[:synth.words_for(m)]


@pytest.mark.parametrize("prec", ["fp32", "fp64", "ntt"])
@pytest.mark.parametrize("others", [[], [(300_000, 70_001), (1_500_000, 150_000), TIGHT]])
def test_batch_budget_below_the_planned_tile(pa, prec, others):
    """A budget that does not hold one tile of a group's class: its jobs run on
    shorter classes.  With several groups, one that finds the memory taken waits
    for the group beside it."""
    from gpu_util import to_dev, from_dev, empty_dev, describe
    import torch
    flags = {"fp32": pa.PA_PREC_FP32_SEG, "fp64": pa.PA_PREC_FP64, "ntt": pa.PA_PREC_NTT}[prec]
    rng = np.random.default_rng(24)
    budget = 24 << 20
    assert pa.pa_plan_query(*TIGHT, pa.PA_PREC_FP32_SEG)["fft_len"] * 8 >= budget
    c = pa.pa_create(0, budget, None)
    try:
        jobs = []
        for n, m in [TIGHT] + others:
            p = synth.random_problem(rng, n, m)
            jobs.append((to_dev(p.seed), to_dev(p.key), empty_dev(synth.words_for(m)), n, m))
        for _ in range(2):   # again with the workspaces that the first call left
            print(f"batch of {len(jobs)}, {prec}", flush=True)
            st, per = pa.pa_hash_batch(c, jobs, flags)
            torch.cuda.synchronize()
            assert st == pa.PA_OK and per == [pa.PA_OK] * len(jobs), (pa.pa_strerror(st), per)
            s = pa.pa_last_stats(c)
            assert s["tiles"] >= len(jobs) and s["fallback_tiles"] == 0 and s["model_bytes"] > 0, s
            for js, jk, jo, n, m in jobs:
                a, b = from_dev(jo)[:synth.words_for(m)], _direct(pa, c, js, jk, n, m)
                assert np.array_equal(a, b), describe(a, b, m)
                jo.fill_(-1)
            torch.cuda.synchronize()
    finally:
        pa.pa_destroy(c)


def test_serving_budget_below_the_planned_tile(pa):
    """The same for requests: admitted at a class whose tile fits the budget, and
    run on a shorter one where the launch does not find the memory."""
    from gpu_util import to_dev, from_dev, empty_dev, describe
    import torch
    n, m = TIGHT
    rng = np.random.default_rng(25)
    c = pa.pa_create(0, 24 << 20, None)
    try:
        seed = synth.gen_bits(rng, n + m - 1)
        ds = to_dev(seed)
        sid = pa.pa_seed_register(c, ds, n + m - 1)
        keys = [to_dev(synth.gen_bits(rng, n)) for _ in range(5)]
        outs = [empty_dev(synth.words_for(m)) for _ in keys]
        tickets = []
        for k, o in zip(keys, outs):
            st, t = pa.pa_submit(c, sid, n, m, k, o)
            assert st == pa.PA_OK, pa.pa_strerror(st)
            tickets.append(t)
        got = [pa.pa_wait(c, t) for t in tickets]
        torch.cuda.synchronize()
        assert got == [pa.PA_OK] * len(keys), [pa.pa_strerror(x) for x in got]
        assert pa.pa_serve_stats(c)["tiles"] >= len(keys)
        for k, o in zip(keys, outs):
            a, b = from_dev(o)[:synth.words_for(m)], _direct(pa, c, ds, k, n, m)
            assert np.array_equal(a, b), describe(a, b, m)
    finally:
        pa.pa_destroy(c)


@pytest.mark.parametrize("call", ["hash", "batch"])
def test_fallback_budget_below_one_fp64_tile(pa, call):
    """A budget that holds the FP32 tiles but not one FP64 tile of their class:
    the failed job is rebuilt in FP64 on shorter classes.  All ones: every output
    is n mod 2."""
    from gpu_util import to_dev, from_dev, empty_dev
    import torch
    n, m = TIGHT
    rng = np.random.default_rng(26)
    c = pa.pa_create(0, 40 << 20, None)
    try:
        s, k = to_dev(synth.pattern_bits("ones", n + m - 1)), to_dev(synth.pattern_bits("ones", n))
        o = empty_dev(synth.words_for(m))
        p = synth.random_problem(rng, 200_000, 50_000)
        o2 = empty_dev(synth.words_for(p.m))
        if call == "hash":
            assert pa.pa_hash(c, s, n, m, k, o, pa.PA_PREC_FP32_SEG) == pa.PA_OK
        else:
            st, per = pa.pa_hash_batch(c, [(s, k, o, n, m), (to_dev(p.seed), to_dev(p.key), o2, p.n, p.m)],
                                       pa.PA_PREC_FP32_SEG)
            assert st == pa.PA_OK and per == [pa.PA_OK] * 2
        torch.cuda.synchronize()
        stats = pa.pa_last_stats(c)
        assert stats["fallback_tiles"] > 0, stats
        assert np.array_equal(synth.bits_to_array(from_dev(o), m), np.full(m, n & 1, np.uint8)), stats
        if call == "batch":
            assert np.array_equal(from_dev(o2)[:synth.words_for(p.m)], oracle.hash_words(p.seed, p.n, p.m, p.key))
        assert pa.pa_hash(c, s, n, m, k, o, pa.PA_PREC_FP32_SEG | pa.PA_NO_FALLBACK) == pa.PA_EPRECISION
    finally:
        pa.pa_destroy(c)


def _job(pa, rng, n, m):
    from gpu_util import to_dev, empty_dev
    p = synth.random_problem(rng, n, m)
    return to_dev(p.seed), to_dev(p.key), empty_dev(synth.words_for(m)), n, m


def test_certificates_fit_beside_a_full_workspace(pa, monkeypatch):
    """A batch whose tiles fill the budget to the last few kilobytes: the workspace
    leaves room for their certificates."""
    import torch
    from gpu_util import from_dev
    rng = np.random.default_rng(27)
    c = pa.pa_create(0, 24 << 20, None)
    try:
        monkeypatch.setenv("PA_ONLY_LEN", str(1 << 12))
        batch = [_job(pa, rng, 60_000, 5_000) for _ in range(100)]
        print("100 jobs of tiles of 2^12", flush=True)
        st, _ = pa.pa_hash_batch(c, batch, pa.PA_PREC_FP32_SEG)
        torch.cuda.synchronize()
        assert st == pa.PA_OK and pa.pa_last_stats(c)["tiles"] * (8 << 12) > 24 << 20, pa.pa_strerror(st)
        for s, k, o, n, m in batch[:2] + batch[-2:]:
            assert np.array_equal(from_dev(o)[:synth.words_for(m)], _direct(pa, c, s, k, n, m))
    finally:
        pa.pa_destroy(c)


def test_full_budget_leaves_room_for_another_class(pa, monkeypatch):
    """A batch whose tiles fill the budget to the last few kilobytes, then a hash of a
    class whose tables are not there yet: it runs on its own class."""
    import torch
    rng = np.random.default_rng(27)
    c = pa.pa_create(0, 24 << 20, None)
    try:
        monkeypatch.setenv("PA_ONLY_LEN", str(1 << 12))
        batch = [_job(pa, rng, 60_000, 5_000) for _ in range(100)]
        st, _ = pa.pa_hash_batch(c, batch, pa.PA_PREC_FP32_SEG)
        assert st == pa.PA_OK and pa.pa_last_stats(c)["tiles"] > 1000
        monkeypatch.delenv("PA_ONLY_LEN")
        s, k, o, n, m = _job(pa, rng, 700_000, 200_000)
        want = pa.pa_plan_query(n, m, pa.PA_PREC_FP64)["fft_len"]
        print(f"n={n} m={m} class {want}", flush=True)
        assert pa.pa_hash(c, s, n, m, k, o, pa.PA_PREC_FP64) == pa.PA_OK
        torch.cuda.synchronize()
        assert pa.pa_last_stats(c)["fft_len"] == want, pa.pa_last_stats(c)
        from gpu_util import from_dev
        assert np.array_equal(from_dev(o)[:synth.words_for(m)], _direct(pa, c, s, k, n, m))
    finally:
        pa.pa_destroy(c)


def test_idle_workspaces_are_given_back(pa, monkeypatch):
    """A batch of two groups leaves a workspace with each of its two streams; a batch
    of one group that needs most of the budget still runs in one go."""
    import torch
    from gpu_util import from_dev
    rng = np.random.default_rng(28)
    c = pa.pa_create(0, 64 << 20, None)
    try:
        two = [_job(pa, rng, 200_000, 60_000) for _ in range(9)] + [_job(pa, rng, 20_000, 3_000) for _ in range(40)]
        st, _ = pa.pa_hash_batch(c, two, pa.PA_PREC_FP64)
        assert st == pa.PA_OK and pa.pa_last_stats(c)["launches"] == 6, pa.pa_last_stats(c)
        monkeypatch.setenv("PA_ONLY_LEN", str(1 << 18))
        one = [_job(pa, rng, 200_000, 60_000) for _ in range(13)]   # a tile of 4 MB each
        print("13 jobs of one tile of 2^18", flush=True)
        st, _ = pa.pa_hash_batch(c, one, pa.PA_PREC_FP64)
        torch.cuda.synchronize()
        stats = pa.pa_last_stats(c)
        assert st == pa.PA_OK and stats["tiles"] == 13 and stats["launches"] == 3, stats
        monkeypatch.delenv("PA_ONLY_LEN")
        for s, k, o, n, m in one[:3] + two[:2] + two[-2:]:
            assert np.array_equal(from_dev(o)[:synth.words_for(m)], _direct(pa, c, s, k, n, m)), (n, m)
    finally:
        pa.pa_destroy(c)


def test_groups_of_a_batch_keep_their_workspaces(pa, monkeypatch):
    """A batch of two groups, then one whose first group could use the whole budget: it
    leaves the other group's workspace alone.  Twice the jobs of the first group are two
    runs of tiles at most, the second group stays one; three passes each, and as much
    again for another choice of classes."""
    import torch
    from gpu_util import from_dev
    rng = np.random.default_rng(29)
    c = pa.pa_create(0, 64 << 20, None)
    try:
        two = [_job(pa, rng, 200_000, 60_000) for _ in range(9)] + [_job(pa, rng, 20_000, 3_000) for _ in range(40)]
        st, _ = pa.pa_hash_batch(c, two, pa.PA_PREC_FP64)
        assert st == pa.PA_OK and pa.pa_last_stats(c)["launches"] == 6, pa.pa_last_stats(c)
        more = two + [_job(pa, rng, 200_000, 60_000) for _ in range(9)]
        for _ in range(3):
            st, _ = pa.pa_hash_batch(c, more, pa.PA_PREC_FP64)
            torch.cuda.synchronize()
            stats = pa.pa_last_stats(c)
            assert st == pa.PA_OK and stats["launches"] <= 18, stats
        for s, k, o, n, m in more[:2] + more[20:22] + more[-2:]:
            assert np.array_equal(from_dev(o)[:synth.words_for(m)], _direct(pa, c, s, k, n, m)), (n, m)
    finally:
        pa.pa_destroy(c)


def test_serving_tile_beyond_a_lanes_share(pa):
    """A tile that the budget holds and a serving lane's share of it (a third) does not:
    the request still runs on its planned class."""
    from gpu_util import from_dev
    n, m = 1_436_744, 1_306_539
    plan = pa.pa_plan_query(n, m, pa.PA_PREC_FP32_SEG)
    budget = 24 << 20
    assert budget // 3 < plan["fft_len"] * 8 < budget * 3 // 4, plan
    s, k, o, n, m = _job(pa, np.random.default_rng(30), n, m)
    c = pa.pa_create(0, budget, None)
    try:
        sid = pa.pa_seed_register(c, s, n + m - 1)
        st, t = pa.pa_submit(c, sid, n, m, k, o)
        assert st == pa.PA_OK and pa.pa_wait(c, t) == pa.PA_OK
        stats = pa.pa_serve_stats(c)
        assert stats["tiles"] == plan["chunks"] * plan["windows"], (stats, plan)
        assert np.array_equal(from_dev(o)[:synth.words_for(m)], _direct(pa, c, s, k, n, m))
    finally:
        pa.pa_destroy(c)


def test_serving_lanes_wait_for_each_others_memory(pa):
    """Requests of two classes whose tiles do not fit the budget side by side: each runs
    on its planned class, when the other lane has ended and given its workspace back."""
    from gpu_util import from_dev
    budget = 24 << 20
    rng = np.random.default_rng(31)
    shapes = [(1_436_744, 1_306_539), (1_491_755, 699_609)]
    plans = [pa.pa_plan_query(n, m, pa.PA_PREC_FP32_SEG) for n, m in shapes]
    assert plans[0]["fft_len"] != plans[1]["fft_len"]
    assert all(p["fft_len"] * 8 < budget * 3 // 4 for p in plans) and sum(p["fft_len"] * 8 for p in plans) > budget, plans
    c = pa.pa_create(0, budget, None)
    try:
        s = _job(pa, rng, *shapes[0])[0]
        sid = pa.pa_seed_register(c, s, sum(shapes[0]) - 1)
        reqs = [_job(pa, rng, *shapes[q % 2])[1:] for q in range(12)]
        tickets = []
        for k, o, n, m in reqs:
            st, t = pa.pa_submit(c, sid, n, m, k, o)
            assert st == pa.PA_OK
            tickets.append(t)
        got = [pa.pa_wait(c, t) for t in tickets]
        assert got == [pa.PA_OK] * len(reqs), got
        stats = pa.pa_serve_stats(c)
        assert stats["tiles"] == 6 * sum(p["chunks"] * p["windows"] for p in plans), (stats, plans)
        for k, o, n, m in reqs[:4]:
            assert np.array_equal(from_dev(o)[:synth.words_for(m)], _direct(pa, c, s, k, n, m)), (n, m)
    finally:
        pa.pa_destroy(c)


@pytest.mark.parametrize("call", ["select", "host hash", "seed", "stream", "host batch", "direct batch"])
def test_full_budget_leaves_room_for_other_calls(pa, call, monkeypatch):
    """A batch whose tiles fill the budget to the last few kilobytes, then a call that
    needs device memory for something else than tiles."""
    import torch
    from gpu_util import to_dev, from_dev
    rng = np.random.default_rng(32)
    c = pa.pa_create(0, 24 << 20, None)
    try:
        monkeypatch.setenv("PA_ONLY_LEN", str(1 << 12))
        st, _ = pa.pa_hash_batch(c, [_job(pa, rng, 60_000, 5_000) for _ in range(100)], pa.PA_PREC_FP32_SEG)
        torch.cuda.synchronize()
        assert st == pa.PA_OK and pa.pa_last_stats(c)["tiles"] > 1000
        monkeypatch.delenv("PA_ONLY_LEN")
        n, m = 700_000, 200_000
        p = synth.random_problem(rng, n, m)
        ref = oracle.hash_words(p.seed, n, m, p.key)
        out = np.zeros(synth.words_for(m), np.uint64)
        print(call, flush=True)
        if call == "select":
            idx = [0, 1, 77_777, m - 1]
            st, bits = pa.pa_hash_select(c, to_dev(p.seed), n, m, to_dev(p.key), idx)
            assert st == pa.PA_OK
            assert [int(b) for b in bits] == [int(ref[i >> 6] >> np.uint64(i & 63)) & 1 for i in idx]
            return
        if call == "host hash":
            assert pa.pa_hash(c, p.seed, n, m, p.key, out, pa.PA_PREC_FP64) == pa.PA_OK
        elif call == "host batch":
            st, per = pa.pa_hash_batch(c, [(p.seed, p.key, out, n, m)], pa.PA_PREC_FP64)
            assert st == pa.PA_OK and per == [pa.PA_OK]
        elif call == "direct batch":
            jobs = [_job(pa, rng, 3_000, 100) for _ in range(2_000)]
            st, per = pa.pa_hash_batch(c, jobs, pa.PA_PREC_DIRECT)
            assert st == pa.PA_OK and per == [pa.PA_OK] * len(jobs)
            torch.cuda.synchronize()
            s, k, o, n, m = jobs[-1]
            assert np.array_equal(from_dev(o)[:synth.words_for(m)], _direct(pa, c, s, k, n, m))
            return
        elif call == "seed":
            sid = pa.pa_seed_register(c, to_dev(p.seed), n + m - 1)
            o = to_dev(out)
            st, t = pa.pa_submit(c, sid, n, m, to_dev(p.key), o)
            assert st == pa.PA_OK and pa.pa_wait(c, t) == pa.PA_OK
            out = from_dev(o)
        else:
            st, s = pa.pa_stream_open(c, n, m, pa.PA_PREC_FP64)
            assert st == pa.PA_OK
            assert pa.pa_stream_feed(s, p.key, 0, n, p.seed) == pa.PA_OK
            assert pa.pa_stream_close(s, out) == pa.PA_OK
        assert np.array_equal(out[:synth.words_for(m)], ref[:synth.words_for(m)])
    finally:
        pa.pa_destroy(c)


def test_a_group_waits_rather_than_run_in_pieces(pa, monkeypatch):
    """A batch of one group takes nearly the whole budget; of the next batch's two groups
    the second finds room for a few tiles only and waits for the first.  Two or three
    runs of tiles in all, three passes each."""
    import torch
    from gpu_util import from_dev
    rng = np.random.default_rng(33)
    c = pa.pa_create(0, 64 << 20, None)
    try:
        monkeypatch.setenv("PA_ONLY_LEN", str(1 << 18))
        st, _ = pa.pa_hash_batch(c, [_job(pa, rng, 200_000, 60_000) for _ in range(16)], pa.PA_PREC_FP64)
        assert st == pa.PA_OK
        monkeypatch.delenv("PA_ONLY_LEN")
        two = [_job(pa, rng, 200_000, 60_000) for _ in range(9)] + [_job(pa, rng, 20_000, 3_000) for _ in range(40)]
        for _ in range(3):
            st, _ = pa.pa_hash_batch(c, two, pa.PA_PREC_FP64)
            torch.cuda.synchronize()
            stats = pa.pa_last_stats(c)
            assert st == pa.PA_OK and stats["launches"] <= 9, stats
        for s, k, o, n, m in two[:2] + two[-2:]:
            assert np.array_equal(from_dev(o)[:synth.words_for(m)], _direct(pa, c, s, k, n, m)), (n, m)
    finally:
        pa.pa_destroy(c)

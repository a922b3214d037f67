"""GPU parity of single paths of the kernels at the sizes where each can go wrong
(edges of its range, remainders, the largest values), against the oracle.

Every quantity is an integer and must match exactly.
"""
import numpy as np
import pytest

import oracle
from oracle import ALPHA_INF
from test_gpu_opt import check as check_opt
from test_gpu_simulate import (ISJL_VARIANTS, assert_same, check_copies, compute_units,  # noqa: F401
                               dev, gpu_sim, log, plan_links_in_hbm)  # (dev: the fixture)

pytestmark = pytest.mark.gpu


def check(dev, ctx, a, p, o, prefill=False, **kw):
    log(ctx)
    got, gs, gf = gpu_sim(dev, a, p, o, prefill=prefill, **kw)
    ref, rs, rf = oracle.simulate(a, p, o, schedule=True,
                                  flags=oracle.FLAG_PREFILL if prefill else 0, **kw)
    assert_same(ctx, got, ref, gs, rs, gf, rf)
    return got


@pytest.mark.parametrize("policy,n,B,alpha,M_kv,prefill", [
    ("fcfs", 1000, 1000, ALPHA_INF, 0, False),
    ("isjl", 1000, 1000, ALPHA_INF, 1 << 40, False),  # a budget that no 32-bit sum reaches
    ("ljf", 1000, 1000, 5, (1 << 31) + 7, False),
    ("isjl", 500, 500, 1 << 10, (1 << 29) + 12345, False),
    ("sjf", 120, 100, ALPHA_INF, (1 << 26), False),
    ("fcfs", 1000, 1000, ALPHA_INF, (1 << 29) + 77, True),
    ("isjl", 130, 128, 2, 1 << 33, True),
])
def test_largest_reservations_and_footprints(dev, policy, n, B, alpha, M_kv, prefill):
    """Jobs just below 2^20 tokens on up to 1,000 workers: reservations and footprint
    sums near 2^30, the range that the 32-bit span sums are exact over."""
    rng = np.random.default_rng(n + B)
    size = (2, n)
    a = np.sort(rng.integers(0, 40, size=size), axis=1).astype(np.int32)
    if prefill:
        o = rng.integers(1, 60, size=size).astype(np.int32)
        p = ((1 << 20) - 1 - o - rng.integers(0, 300, size=size)).astype(np.int32)
    else:
        o = rng.integers(1, 3000, size=size).astype(np.int32)
        p = ((1 << 20) - 1 - o - rng.integers(0, 3, size=size)).astype(np.int32)
        p[1] = p[1] // 64  # a shorter instance beside it, where the starts spread further
    check(dev, f"{policy} n={n} B={B} M={M_kv} prefill={prefill}", a, p, o, prefill=prefill,
          policy=policy, B=B, alpha=alpha, M_kv=M_kv, cost_c=3, cost_tau=2)


@pytest.mark.parametrize("n,top,alphas", [
    (1, 9, (0, 3)), (2, 255, (0, 1, 254, ALPHA_INF)), (3, 255, (0, 100, ALPHA_INF)),
    (5, 60, (0, 7, 59)), (7, 24, (1, 23)), (8, 1, (0, 4)), (8, 3, (0, 2, 5)),
    (8, 16, (0, 1, 2, 4, 11, 19, ALPHA_INF)),
])
def test_two_worker_optima(dev, n, top, alphas):
    """The two-worker table of the exact optimum: one class of identical jobs to eight
    different ones, tables from a few entries to beyond the largest that it keeps
    (the search takes those), instances with a release (not its kind) among them."""
    rng = np.random.default_rng(100 * n + top)
    size = (70, n)
    z = np.zeros(size, np.int32)
    o = rng.integers(1, top + 1, size=size).astype(np.int32)
    o[::7] = rng.integers(1, top + 1, size=(10, 1))  # identical jobs
    if n == 8 and top == 16:
        o[3] = 13 + np.arange(8)
    a = z.copy()
    a[5::9, -1] = 3
    for alpha in alphas:
        for M in (0, max(2, (3 * top) // 2)):
            check_opt(dev, f"n={n} top={top} alpha={alpha} M={M}", a, z, o, B=2, alpha=alpha,
                      M_kv=M)


def test_two_worker_tables_beyond_lds(dev):
    """Eight long jobs of different lengths: 2^8 rows of up to 2,000 entries, more than the
    table keeps, solved by the search beside short instances solved by the table."""
    rng = np.random.default_rng(8)
    o = np.concatenate([rng.integers(120, 136, size=(2, 8)), rng.integers(1, 5, size=(30, 8)),
                        rng.integers(17, 21, size=(4, 8))]).astype(np.int32)
    z = np.zeros_like(o)
    # alpha = 130: the long instances need 256 * (1 + 8 * 131) entries at most; M_kv lets no
    # two long jobs run together, so their search ends at once
    T = check_opt(dev, "long", z, z, o, B=2, alpha=130, M_kv=200)
    assert (T[:2] == o[:2].sum(1)).all()


@pytest.mark.parametrize("policy,alpha,prefill", [
    ("fcfs", ALPHA_INF, False), ("sjf", ALPHA_INF, False), ("ljf", 6, False),
    ("isjl", 40, False), ("isjl", ALPHA_INF, False), ("isjl", 5, True), ("fcfs", ALPHA_INF, True),
])
@pytest.mark.parametrize("n,B", [(1, 1), (63, 5), (65, 64), (1025, 130), (2048, 512),
                                 (2049, 100), (4096, 1000)])
def test_releases_in_another_order(dev, policy, alpha, prefill, n, B):
    """Arrivals not sorted by job index, beside sorted instances of the same launch: shuffled,
    reversed, all equal but one, the last below the largest unsorted arrival (2^20)."""
    rng = np.random.default_rng(n + B)
    size = (7, n)
    a = np.sort(rng.integers(0, 4 * n, size=size), axis=1).astype(np.int32)
    p = rng.integers(0, 40, size=size).astype(np.int32)
    o = rng.integers(1, 60, size=size).astype(np.int32)
    a[1] = rng.permutation(a[1])
    a[2] = a[2][::-1]
    a[3] = 0
    a[3, 0] = 17
    a[4] = rng.integers(0, 3, size=n)  # many releases at once
    a[5, 0] = (1 << 20) - 1
    check(dev, f"{policy} n={n} B={B}", np.ascontiguousarray(a), p, o, prefill=prefill,
          policy=policy, B=B, alpha=alpha, M_kv=[0, 900][n % 2], cost_c=3, cost_tau=2)


@pytest.mark.parametrize("policy,alpha", [("fcfs", ALPHA_INF), ("sjf", ALPHA_INF), ("isjl", 0),
                                          ("isjl", 7), ("isjl", 45), ("isjl", ALPHA_INF)])
@pytest.mark.parametrize("n,B,rate", [(64, 64, 8), (65, 40, 3), (129, 128, 64), (300, 130, 9),
                                      (700, 512, 21), (700, 600, 5)])
def test_runs_of_releases_into_idle_workers(dev, policy, alpha, n, B, rate):
    """Releases while workers are idle: release steps that straddle a chunk of 64 jobs, that end
    in the middle of the free workers or of the KV budget, that meet a completion (of a job
    admitted just before, too), worker 1's start time or A_max = alpha."""
    rng = np.random.default_rng(n + B + rate)
    k = 24
    gap = (rng.random((k, n)) < 1.0 / rate) * rng.integers(1, 4, size=(k, n))
    a = np.cumsum(gap, axis=1).astype(np.int32)
    o = rng.integers(1, 30, size=(k, n)).astype(np.int32)
    long = rng.random((k, n)) < np.linspace(0.05, 1.0, k)[:, None]
    p = np.where(long, rng.integers(20, 120, size=(k, n)), 0).astype(np.int32)
    a[-1] = rng.permutation(a[-1])
    for M in (0, 25 * B, 60 * B):
        check(dev, f"{policy} n={n} B={B} rate={rate} M={M}", a, p, o, policy=policy, B=B,
              alpha=alpha, M_kv=M, cost_c=3, cost_tau=2)


@pytest.mark.parametrize("policy,alpha", [("fcfs", ALPHA_INF), ("sjf", ALPHA_INF),
                                          ("isjl", ALPHA_INF), ("isjl", 1 << 20)])
@pytest.mark.parametrize("n,B", [(90, 2), (200, 64), (260, 65), (500, 200), (900, 300),
                                 (1500, 600)])
def test_fill_sweep_over_many_slots(dev, policy, alpha, n, B):
    """Runs of completions that admit queued jobs, 1 to 16 slots per lane: long runs (every job
    long), runs cut by short jobs, more than 64 completions at one step, more than 64 jobs
    admitted by one run (a long job holding the KV budget back first), releases between."""
    rng = np.random.default_rng(n + B)
    size = (6, n)
    a = np.zeros(size, np.int32)
    a[1] = np.sort(rng.integers(0, 600, size=n))
    p = np.zeros(size, np.int32)
    o = rng.integers(100, 260, size=size).astype(np.int32)
    o[2] = rng.integers(1, 400, size=n)
    o[3] = 50 * rng.integers(1, 4, size=n)  # completions at few distinct steps
    o[4] = rng.integers(3, 9, size=n)
    o[4, ::40] = 5 * B  # jobs that fill most of the budget alone
    a[5] = rng.permutation(np.arange(n) // 7)
    for M in (0, 6 * B, 150 * B):
        check(dev, f"{policy} alpha={alpha} n={n} B={B} M={M}", a, p, o, policy=policy, B=B,
              alpha=alpha, M_kv=M, cost_c=3, cost_tau=2)


@pytest.mark.parametrize("alpha", [3, 40, 200])
@pytest.mark.parametrize("n,B", [(64, 3), (200, 16), (420, 65), (900, 130), (1500, 520),
                                 (1200, 1000), (2500, 60)])
def test_pack_scan_batches(dev, n, B, alpha):
    """Phase ONE's pack scan over batches of 64 candidates: packs that span batches, spare and
    long workers, candidates that fit nowhere (runs of them, to the next batch and to the end of
    the queue), no candidate at all; plan links in LDS."""
    rng = np.random.default_rng(n + B + alpha)
    size = (8, n)
    z = np.zeros(size, np.int32)
    short = rng.integers(1, max(2, alpha // 6 + 1), size=size)
    mid = rng.integers(max(1, alpha // 2), alpha + 1, size=size)
    long = rng.integers(alpha + 1, 5 * alpha + 9, size=size)
    u = rng.random(size)
    share = np.linspace(0.0, 0.9, 8)[:, None]  # of short jobs
    o = np.where(u < share, short, np.where(u < share + 0.05, mid, long)).astype(np.int32)
    o[1, : n - 2] = 1 + np.arange(n - 2) % max(1, alpha)  # two long jobs, the rest pack
    o[1, n - 2:] = 4 * alpha + 1
    a = z.copy()
    a[2:5] = np.sort(rng.integers(0, 9 * alpha, size=(3, n)), axis=1)
    for M in (0, 2 * B * alpha):
        check(dev, f"n={n} B={B} alpha={alpha} M={M}", a, z, o, policy="isjl", B=B, alpha=alpha,
              M_kv=M, cost_c=3, cost_tau=2)


@pytest.mark.parametrize("n", [1, 32, 33, 64, 512, 513, 700, 1024, 1025, 2048, 2049, 4096])
def test_rescoring_halves(dev, n):
    """Re-scoring with one and with two waves per instance: groups across the middle of the sorted
    events (every start or every end at one step, too), idle gaps, a second half with nothing
    active before it, jobs of 65,536 tokens and more beside short ones, violations of every kind."""
    import torch
    import paper_2608_02244_amd as fs
    rng = np.random.default_rng(n)
    k = 9
    size = (k, n)
    a = rng.integers(0, 5, size=size).astype(np.int32)
    p = rng.integers(0, 30, size=size).astype(np.int32)
    o = rng.integers(1, 90, size=size).astype(np.int32)
    s = (a + rng.integers(0, 3 * n + 1, size=size)).astype(np.int32)
    s[1] = 7  # all start together
    s[2] = 200 - (p[2] + o[2])  # all end together
    s[3] = np.where(np.arange(n) % 2, 5, 400)  # two batches with a gap between them
    p[4, : max(1, n // 2)] = 70000  # long jobs
    s[5] = a[5] + rng.integers(0, 4, size=n)  # few distinct starts
    p[6], o[6], s[6] = 0, 1, np.arange(n)  # one at a time
    s[7] = np.sort(s[7])
    s[8] = a[8] + 3 * rng.integers(0, n + 1, size=n)
    for B, alpha, M in ((0, ALPHA_INF, 0), (3, 11, 500), (n, 0, 40 * n)):
        log(f"rescoring n={n} B={B} alpha={alpha} M={M}")
        t = [torch.from_numpy(np.ascontiguousarray(x)).to(dev) for x in (a, p, o, s)]
        m, v = fs.cost_decompose(*t, B=B, alpha=alpha, M_kv=M, cost_c=3, cost_tau=2)
        torch.cuda.synchronize()
        rm, rv = oracle.decompose(a, p, o, s, B=B, alpha=alpha, M_kv=M, cost_c=3, cost_tau=2)
        assert_same(f"rescoring n={n} B={B}", fs.metrics_view(m), rm)
        assert np.array_equal(v.cpu().numpy().astype(np.uint32), rv)


@pytest.mark.parametrize("variant", list(ISJL_VARIANTS))
@pytest.mark.parametrize("B", [16, 100, 200, 500])
@pytest.mark.parametrize("n,lds_waves,hbm_waves", [(2000, 12, 16), (2500, 6, 8)])
def test_plan_links_in_hbm_for_large_batches(dev, n, lds_waves, hbm_waves, B, variant):
    """The plan-queue links move to HBM scratch only where the batch is larger than what the LDS
    lets run at once with them (12 waves per CU at 2,000 jobs, 6 at 2,500, whose bitmap takes two
    words per lane): copies of 8 instances, just above that (all resident at once without them,
    taking the kernels that turn the issue priority) and beyond what is resident without them."""
    rng = np.random.default_rng(B)
    a, p, o = (rng.integers(lo, hi, size=(8, n)).astype(np.int32)
               for lo, hi in ((0, 300), (0, 40), (1, 200)))
    a.sort(axis=1)
    a[7] = rng.permutation(a[7])
    u = o + rng.integers(0, 60, size=o.shape).astype(np.int32)
    kw = dict(B=B, alpha=45, M_kv=70 * B, cost_c=3, cost_tau=2)
    units = compute_units(dev)
    opt, _ = ISJL_VARIANTS[variant]
    assert not plan_links_in_hbm(lds_waves * units, n, **opt, **kw)
    for waves in (lds_waves, hbm_waves):
        copies = waves * units // 8 + 1
        assert plan_links_in_hbm(8 * copies, n, **opt, **kw)
        check_copies(dev, f"links in HBM n={n} B={B} {variant} {8 * copies} instances", a, p, o,
                     u, copies, variant, **kw)


def test_host_arrays_of_every_size_and_thread(dev):
    """Host mode below, at and above the 4 MiB of the pool's arena, from several threads at
    once, against device mode; an invalid table in between is still refused."""
    import threading
    import torch
    import paper_2608_02244_amd as fs
    errors = []

    def work(seed):
        try:
            rng = np.random.default_rng(seed)
            # rows of 1,000 jobs: 250 instances with schedules take 4.96 MB, 200 take 4.02 MB
            for k, n in ((1, 1), (3, 70), (200, 1000), (209, 1000), (250, 1000)):
                a = np.zeros((k, n), np.int32)
                p = rng.integers(0, 20, size=(k, n)).astype(np.int32)
                o = rng.integers(1, 50, size=(k, n)).astype(np.int32)
                kw = dict(B=8, alpha=20, M_kv=300, cost_c=3, cost_tau=2)
                t = [torch.from_numpy(x).to(dev) for x in (a, p, o)]
                for policy in ("isjl", "fcfs"):
                    m, s, f = fs.simulate(a, p, o, policy=policy, schedule=True, **kw)
                    gm, gs, gf = fs.simulate(*t, policy=policy, schedule=True, **kw)
                    assert np.array_equal(m, fs.metrics_view(gm))
                    assert np.array_equal(s, gs.cpu().numpy())
                    assert np.array_equal(f, gf.cpu().numpy())
                    dm, dv = fs.cost_decompose(a, p, o, s, **kw)
                    gdm, gdv = fs.cost_decompose(*t, gs, **kw)
                    assert np.array_equal(dm, fs.metrics_view(gdm))
                    assert np.array_equal(dv, gdv.cpu().numpy().astype(np.uint32))
                bad = o.copy()
                bad[-1, -1] = 0
                with pytest.raises(fs.FschedError) as ei:
                    fs.simulate(a, p, bad, policy="isjl", **kw)
                assert ei.value.code == fs.EINVAL
            q = rng.integers(1, 9, size=(500, 6)).astype(np.int32)
            z = np.zeros_like(q)
            T, st = fs.bruteforce_opt(z, z, q, B=2, alpha=2, schedule=True)
            Tg, sg = fs.bruteforce_opt(*(torch.from_numpy(x).to(dev) for x in (z, z, q)), B=2,
                                       alpha=2, schedule=True)
            assert np.array_equal(T, Tg.cpu().numpy()) and np.array_equal(st, sg.cpu().numpy())
        except Exception as e:  # noqa: BLE001  (reported by the main thread)
            errors.append(repr(e))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    fs.release_cache()


@pytest.mark.parametrize("resume", [False, True])
@pytest.mark.parametrize("B,alpha", [(2, 9), (8, 30), (16, 100), (64, 40), (65, 25), (128, 200)])
def test_plan_runs(dev, B, alpha, resume):
    """Runs of planned starts: every worker busy, worker 1 on its timer, workers idle in DRAIN or
    behind a head that the KV budget holds back (with releases meanwhile), ended by a worker
    without a plan, by the guard or by the budget; several completions at one step."""
    rng = np.random.default_rng(B + alpha)
    n = 300
    size = (24, n)
    short = rng.integers(1, max(2, alpha // 4), size=size)
    grid = (alpha // 5 + 1) * rng.integers(1, 4, size=size)  # many completions at one step
    long = rng.integers(alpha + 1, 6 * alpha + 5, size=size)
    u = rng.random(size)
    share = np.linspace(0.3, 0.95, 24)[:, None]
    o = np.where(u < share, np.where(rng.random(size) < 0.5, short, grid), long).astype(np.int32)
    p = np.zeros(size, np.int32)
    a = np.zeros(size, np.int32)
    a[8:16] = np.sort(rng.integers(0, 4 * alpha, size=(8, n)), axis=1)
    a[16:] = rng.integers(0, 40 * alpha, size=(8, n))
    ref_flags = oracle.FLAG_RESUME_FILL if resume else 0
    for M in (0, 3 * B * alpha, B * alpha, 9 * alpha):
        ctx = f"B={B} alpha={alpha} M={M} resume={resume}"
        log(ctx)
        kw = dict(policy="isjl", B=B, alpha=alpha, M_kv=M, cost_c=3, cost_tau=2)
        got, gs, gf = gpu_sim(dev, a, p, o, resume_fill=resume, **kw)
        ref, rs, rf = oracle.simulate(a, p, o, schedule=True, flags=ref_flags, **kw)
        assert_same(ctx, got, ref, gs, rs, gf, rf)


def test_plan_runs_with_predicted_sizes(dev):
    import torch
    import paper_2608_02244_amd as fs
    rng = np.random.default_rng(3)
    size = (16, 250)
    z = np.zeros(size, np.int32)
    o = np.where(rng.random(size) < 0.8, rng.integers(1, 20, size=size),
                 rng.integers(60, 300, size=size)).astype(np.int32)
    u = (o + (rng.random(size) * o).astype(np.int32)).astype(np.int32)
    for B, M in ((8, 0), (16, 900), (100, 4000)):
        for prefill in (False, True):
            log(f"predicted sizes B={B} M={M} prefill={prefill}")
            p = rng.integers(0, 9, size=size).astype(np.int32) if prefill else z
            kw = dict(B=B, alpha=50, M_kv=M, cost_c=3, cost_tau=2)
            t = [torch.from_numpy(x).to(dev) for x in (z, p, o, u)]
            m, s, f = fs.simulate_robust(*t, schedule=True, prefill=prefill, **kw)
            rm, rs, rf = oracle.simulate_robust(z, p, o, u, schedule=True,
                                                flags=oracle.FLAG_PREFILL if prefill else 0, **kw)
            assert_same(f"B={B} M={M}", fs.metrics_view(m), rm, s.cpu().numpy(), rs,
                        f.cpu().numpy(), rf)


@pytest.mark.parametrize("policy,alpha", [("fcfs", ALPHA_INF), ("sjf", ALPHA_INF), ("isjl", 0),
                                          ("isjl", 12), ("isjl", 60), ("isjl", ALPHA_INF)])
@pytest.mark.parametrize("n,B,rate", [(65, 40, 3), (129, 128, 30), (300, 130, 9), (700, 512, 8),
                                      (900, 1000, 4)])
def test_releases_among_completions_with_prefill(dev, policy, alpha, n, B, rate):
    """Prompts prefilled: runs of releases with completions between them (at the same step too),
    jobs that complete inside the run, the earliest or the latest started job ending in it, the
    largest footprint's holder ending in it, more than 64 completions, workers freed in it."""
    rng = np.random.default_rng(n + B + rate)
    k = 18
    gap = (rng.random((k, n)) < 1.0 / rate) * rng.integers(1, 4, size=(k, n))
    a = np.cumsum(gap, axis=1).astype(np.int32)
    o = rng.integers(1, 30, size=(k, n)).astype(np.int32)
    o[3:6] = rng.integers(8, 14, size=(3, n))  # many completions, few inside a run
    o[6:9] = np.where(rng.random((3, n)) < 0.1, 200, o[6:9])
    o[9] = 10
    o[10] = 1 + np.arange(n) % 40
    p = rng.integers(0, 400, size=(k, n)).astype(np.int32)
    p[1::3] = rng.integers(0, 9, size=p[1::3].shape)
    a[-1] = rng.permutation(a[-1])
    for M in (0, 200 * B, 20 * B + 400):
        check(dev, f"{policy} alpha={alpha} n={n} B={B} M={M}", a, p, o, prefill=True,
              policy=policy, B=B, alpha=alpha, M_kv=M, cost_c=3, cost_tau=2)


def test_releases_among_completions_in_full_blocks(dev):
    """FCFS with one slot per lane, prompts prefilled, in blocks of several instances: each one's
    completions are packed in a place of its own."""
    rng = np.random.default_rng(33)
    k, n = 1100, 150
    a = np.cumsum(rng.integers(0, 3, size=(k, n)), axis=1).astype(np.int32)
    o = np.minimum(8 * (1 - rng.random((k, n))) ** -0.6, 900).astype(np.int32)
    p = rng.integers(1, 1500, size=(k, n)).astype(np.int32)
    for B, M in ((33, 0), (64, 30000)):
        check(dev, f"B={B} M={M}", a, p, o, prefill=True, policy="fcfs", B=B, alpha=64, M_kv=M,
              cost_c=3, cost_tau=2)


@pytest.mark.parametrize("alpha", [1 << 30, (1 << 31) - 1000, (1 << 31) - 2])
@pytest.mark.parametrize("B", [2, 64, 65, 130, 300, 520])
def test_finite_fairness_budgets_up_to_the_largest(dev, B, alpha):
    """A finite alpha beyond every length, up to the largest (2^31 - 2), while the KV budget holds
    Phase TWO back: A_max never passes it, and the step where it would lies beyond 2^31."""
    import torch
    import paper_2608_02244_amd as fs
    rng = np.random.default_rng(B)
    n = B + 40
    size = (6, n)
    a = np.sort(rng.integers(0, 90, size=size), axis=1).astype(np.int32)
    a[0] = 0
    a[1] = rng.permutation(a[1])
    p = rng.integers(0, 30, size=size).astype(np.int32)
    o = rng.integers(1, 60, size=size).astype(np.int32)
    o[2, :: 7] = 900  # jobs that run alone
    u = (o + rng.integers(0, 20, size=size)).astype(np.int32)
    for M in (60, 12 * B + 50):
        kw = dict(B=B, alpha=alpha, M_kv=M, cost_c=3, cost_tau=2)
        for prefill in (False, True):
            check(dev, f"B={B} alpha={alpha} M={M} prefill={prefill}", a, p, o, prefill=prefill,
                  policy="isjl", **kw)
            t = [torch.from_numpy(x).to(dev) for x in (a, p, o, u)]
            m, s, f = fs.simulate_robust(*t, schedule=True, prefill=prefill, **kw)
            rm, rs, rf = oracle.simulate_robust(a, p, o, u, schedule=True,
                                                flags=oracle.FLAG_PREFILL if prefill else 0, **kw)
            assert_same(f"robust B={B} alpha={alpha} M={M} prefill={prefill}", fs.metrics_view(m),
                        rm, s.cpu().numpy(), rs, f.cpu().numpy(), rf)
    q = rng.integers(1, 12, size=(40, 6)).astype(np.int32)
    for Bq in (2, 3):
        check_opt(dev, f"optimum B={Bq} alpha={alpha}", np.zeros_like(q), np.zeros_like(q), q,
                  B=Bq, alpha=alpha, M_kv=14)


@pytest.mark.parametrize("B", [2, 65, 130])
def test_fairness_budget_beyond_the_last_step(dev, B):
    """Releases near the largest makespan (2^31 - 648): min_s + alpha + 1 lies beyond 2^31 for an
    ordinary alpha too.  The schedule is that of the same jobs released at step 0, later."""
    rng = np.random.default_rng(B)
    n, late = 20, (1 << 31) - 648 - 20 * 120 - 10
    o = rng.integers(1, 60, size=(6, n)).astype(np.int32)
    z = np.zeros_like(o)
    kw = dict(policy="isjl", B=B, alpha=4000, M_kv=70, cost_c=0, cost_tau=2)
    for prefill in (False, True):
        log(f"late releases B={B} prefill={prefill}")
        ref, rs, rf = oracle.simulate(z, z, o, schedule=True,
                                      flags=oracle.FLAG_PREFILL if prefill else 0, **kw)
        got, gs, gf = gpu_sim(dev, z + np.int32(late), z, o, prefill=prefill, **kw)
        assert np.array_equal(got["T"], ref["T"] + late)
        assert np.array_equal(gs, rs + late) and np.array_equal(gf, rf + late)
        for f in ("E", "C", "W", "sum_extent", "busy_steps", "peak_kv", "max_active"):
            assert np.array_equal(got[f], ref[f]), f

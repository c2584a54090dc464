"""Pins of the CPU oracle against what the paper and mathematics fix.

Each test names the passage it follows.  None of these needs a GPU.
"""
import json
import os
from math import comb
from types import SimpleNamespace as NS

import numpy as np
import pytest

import oracle
from oracle import pyref
from paper_2404_03226_amd import synth
from invariants import check_schedule

GOLD = os.path.join(os.path.dirname(__file__), "golden")


def gold(name):
    with open(os.path.join(GOLD, name)) as f:
        return json.load(f)


def wl(n, rp, col, n_cpu, n_gpu, dur, est=None):
    dur = np.asarray(dur, np.int32).reshape(n, 2)
    est = dur.copy() if est is None else np.asarray(est, np.int32).reshape(n, 2)
    return NS(n=n, row_ptr=np.asarray(rp, np.int32), col=np.asarray(col, np.int32), dur=dur, est=est,
              n_cpu=n_cpu, n_gpu=n_gpu)


def csr(n, edges):
    rp = np.zeros(n + 1, np.int64)
    for a, _ in edges:
        rp[a + 1] += 1
    np.cumsum(rp, out=rp)
    col = [b for a, b in sorted(edges, key=lambda e: e[0])]
    return rp.astype(np.int32), np.asarray(col, np.int32)


# ------------------------------------------------------------ worked examples

def test_w1_attributes_and_unit_time():
    g = gold("w1_attributes.json")
    ia, ie, U = oracle.attributes(g["n"], g["row_ptr"], g["col"], g["est"], g["n_gpu"])
    assert ia.tolist() == g["ia"] and ie.tolist() == g["ie_auto"] and U == g["unit_time_auto"]
    for u, key in ((4, "ie_after_task1_u4"), (5, "ie_after_task1_u5")):
        _, ie2, U2 = oracle.attributes(g["n"], g["row_ptr"], g["col"], g["est"], g["n_gpu"],
                                       rem=g["rem_after_task1"], unit_time=u)
        assert U2 == u
        # IE is meaningful for unfinished tasks only
        live = g["unfinished_after_task1"]
        assert [ie2[v] for v in live] == [g[key][v] for v in live]


def test_w2_fig1_analogue():
    g = gold("w2_schedule.json")
    w = wl(g["n"], g["row_ptr"], g["col"], g["n_cpu"], g["n_gpu"], np.ones((g["n"], 2)))
    for pol in ("fifo", "inspirit"):
        r = oracle.schedule(w, policy=pol, trace=True)
        assert r["worker"].tolist() == g[pol]["worker"]
        assert r["start"].tolist() == g[pol]["start"]
        assert r["makespan"] == g[pol]["makespan"]
        check_schedule(w, r["worker"], r["start"], r["finish"], r["makespan"])
    assert oracle.schedule(w)["unit_time"] == g["unit_time"]
    tr = oracle.schedule(w, policy="inspirit", trace=True)["trace"]
    assert tr["t"].tolist() == g["inspirit"]["trace_t"]
    assert tr["nready"].tolist() == g["inspirit"]["trace_nready"]
    assert tr["mode"].tolist() == g["inspirit"]["trace_mode"]
    assert tr["cnt"].tolist() == g["inspirit"]["trace_cnt"]
    assert oracle.brute_opt(w) == g["optimal_makespan"]


def test_w3_regulator_table():
    g = gold("w3_regulator.json")
    mode, cnt, peak = oracle.regulate(g["t"], g["N"], g["W"], g["tau_bar"])
    assert mode.tolist() == g["mode"]
    assert cnt.tolist() == g["cnt"]
    assert peak.tolist() == g["peak"]
    reg = pyref.Regulator(g["W"], g["tau_bar"])
    got = []
    for t, N in zip(g["t"], g["N"]):
        reg.observe(t, N)
        got.append((reg.mode, reg.cnt, reg.peak))
    assert got == list(zip(g["mode"], g["cnt"], g["peak"]))


def test_regulator_explicit_parameters_override_defaults():
    # k_inc = 1/1: a rise of 2 over 10 ticks is slow (EFI); of 20 over 10 is fast
    mode, _, _ = oracle.regulate([0, 10, 20], [1, 3, 23], 4, 10, s_inc=1, k_num=1, k_den=1)
    assert mode.tolist() == [0, 1, 0]
    # a window of 5 ignores a change of 4
    mode, _, peak = oracle.regulate([0, 10], [5, 9], 4, 10, s_inc=5)
    assert mode.tolist() == [0, 0] and peak.tolist() == [5, 9]


# ------------------------------------------------------------------ IA / IE

def test_ia_figure_two_dependencies():
    # Section 4.2 figure: A -> B, A -> C; completing A releases two dependencies
    rp, col = csr(3, [(0, 1), (0, 2)])
    ia, _, _ = oracle.attributes(3, rp, col, np.ones((3, 2)), 1)
    assert ia[0] == 2


@pytest.mark.parametrize("N", [2, 3, 7, 20])
def test_complete_dag_source_ability(N):
    # Section 4.3: fully connected DAG with one source; the source's ability
    # counts every other task (exclusive reading: N - 1)
    rp, col = csr(N, [(i, j) for i in range(N) for j in range(i + 1, N)])
    ia, _, _ = oracle.attributes(N, rp, col, np.ones((N, 2)), 1)
    assert ia[0] == N - 1
    assert ia.tolist() == [N - 1 - i for i in range(N)]


def _rand_small(seed, n, p):
    return synth.random_dag(seed, n, n, p, dur_hi=40, n_gpu=1)


@pytest.mark.parametrize("seed", range(8))
def test_ie_limits_in_unit_time(seed):
    # Section 4.2: U too low -> IE tends to zero; U too high -> IE converges
    # to IA (exactly, for successors whose only remaining predecessor is v)
    w = _rand_small(seed, 30, 0.2)
    rp, col = oracle.canon(w.n, w.row_ptr, w.col)
    tau = w.est[:, 1].astype(np.int64)
    rem = np.bincount(col, minlength=w.n)
    prev = None
    for U in [1, 2, 3, 5, 8, 13, 21, 34, 55, 80, 81, 200]:
        ia, ie, _ = oracle.attributes(w.n, rp, col, w.est, 1, unit_time=U)
        for v in range(w.n):
            succ = col[rp[v]:rp[v + 1]]
            if succ.size and U < tau[v] + tau[succ].min():
                assert ie[v] == 0
        if prev is not None:
            assert (ie >= prev).all()  # monotone in U
        prev = ie
    ia, ie, _ = oracle.attributes(w.n, rp, col, w.est, 1, unit_time=10 ** 6)
    sole = np.array([int((rem[col[rp[v]:rp[v + 1]]] == 1).sum()) for v in range(w.n)])
    assert (ie == sole).all()
    assert (ia == np.diff(rp)).all()


def test_ie_equals_ia_on_out_tree_at_large_u():
    # every successor in an out-tree has v as its only predecessor
    edges = [(0, 1), (0, 2), (1, 3), (1, 4), (1, 5), (2, 6)]
    rp, col = csr(7, edges)
    ia, ie, _ = oracle.attributes(7, rp, col, np.full((7, 2), 3), 1, unit_time=1000)
    assert (ia == ie).all()


def test_ie_uses_gpu_column_only_when_gpus_exist():
    # Section 4.3: IE uses GPU times; with no GPU worker the CPU column stands in
    rp, col = csr(2, [(0, 1)])
    est = np.array([[10, 1], [10, 1]])
    _, ie_g, _ = oracle.attributes(2, rp, col, est, 1, unit_time=5)
    _, ie_c, _ = oracle.attributes(2, rp, col, est, 0, unit_time=5)
    assert ie_g[0] == 1 and ie_c[0] == 0


def test_auto_unit_time_maximises_score_over_ladder():
    # brute force over the ladder with the oracle's own IE at fixed U
    for seed in range(6):
        w = _rand_small(seed + 20, 40, 0.15)
        rp, col = oracle.canon(w.n, w.row_ptr, w.col)
        _, _, U = oracle.attributes(w.n, rp, col, w.est, 1)
        scores = {}
        J = 0
        while 2 ** J < 2 * int(w.est[:, 1].max()):
            J += 1
        for j in range(J + 1):
            ia, ie, _ = oracle.attributes(w.n, rp, col, w.est, 1, unit_time=2 ** j)
            scores[2 ** j] = int(((ie > 0) & (ie < ia)).sum())
        best = max(scores.values())
        assert U == max(u for u, s in scores.items() if s == best)


# ------------------------------------------------------------- closed forms

@pytest.mark.parametrize("policy", ["inspirit", "fifo", "ability", "efi"])
def test_chain_picks_fastest_kind(policy):
    n = 12
    rp, col = csr(n, [(i, i + 1) for i in range(n - 1)])
    st = synth.Stream(5, 1)
    dur = st.randint(np.arange(2 * n).reshape(n, 2), 1, 50)
    w = wl(n, rp, col, 3, 2, dur)
    r = oracle.schedule(w, policy=policy)
    assert r["makespan"] == int(dur.min(axis=1).sum())
    check_schedule(w, r["worker"], r["start"], r["finish"], r["makespan"])


@pytest.mark.parametrize("n,W", [(1, 1), (7, 3), (64, 8), (65, 8), (100, 7)])
@pytest.mark.parametrize("policy", ["inspirit", "fifo"])
def test_independent_unit_tasks(n, W, policy):
    w = wl(n, np.zeros(n + 1), [], W, 0, np.ones((n, 2)))
    r = oracle.schedule(w, policy=policy)
    assert r["makespan"] == -(-n // W)


def test_empty_dag():
    w = wl(0, [0], [], 2, 1, np.zeros((0, 2)))
    r = oracle.schedule(w)
    assert r["makespan"] == 0 and r["worker"].size == 0


@pytest.mark.parametrize("seed", range(40))
def test_makespan_not_below_brute_force_optimum(seed):
    n = 3 + seed % 6
    w = synth.random_dag(31, seed, n, 0.3, dur_hi=6, n_cpu=1 + seed % 2, n_gpu=1)
    opt = oracle.brute_opt(w)
    lb = max(int(w.dur.min(axis=1).sum()) // (w.n_cpu + w.n_gpu), int(w.dur.min(axis=1).max()))
    assert opt >= lb
    for pol in ("inspirit", "fifo", "ability", "efi"):
        r = oracle.schedule(w, policy=pol)
        assert r["makespan"] >= opt


def test_brute_force_exact_on_tiny_cases():
    # one task, two kinds: the optimum is the faster kind
    w = wl(1, [0, 0], [], 1, 1, [[7, 3]])
    assert oracle.brute_opt(w) == 3
    # two independent tasks on one CPU + one GPU: one on each kind
    w = wl(2, [0, 0, 0], [], 1, 1, [[4, 5], [4, 5]])
    assert oracle.brute_opt(w) == 5
    # ... unless both fit on the faster kind back to back
    w = wl(2, [0, 0, 0], [], 1, 1, [[9, 2], [9, 2]])
    assert oracle.brute_opt(w) == 4


def test_fifo_pops_in_push_order():
    # Section 4.1: each worker takes its queue head; push order is (ready time, id)
    for seed in range(10):
        w = synth.random_dag(41, seed, 60, 0.06, dur_hi=30, n_cpu=3, n_gpu=1)
        r = oracle.schedule(w, policy="fifo")
        rp, col = oracle.canon(w.n, w.row_ptr, w.col)
        ready = np.zeros(w.n, np.int64)
        src = np.repeat(np.arange(w.n), np.diff(rp))
        np.maximum.at(ready, col, r["finish"][src])
        for wk in range(w.n_cpu + w.n_gpu):
            idx = np.nonzero(r["worker"] == wk)[0]
            by_start = idx[np.argsort(r["start"][idx], kind="stable")]
            keys = list(zip(ready[by_start], by_start))
            assert keys == sorted(keys)


# ------------------------------------------------------------- invariants

@pytest.mark.parametrize("policy", ["inspirit", "fifo", "ability", "efi"])
def test_invariants_on_workloads(policy):
    for w in (synth.cfg1(), synth.cfg2(nb=12), *synth.cfg3(select=[0, 1, 2])):
        r = oracle.schedule(w, policy=policy, variant=oracle.HEAP)
        check_schedule(w, r["worker"], r["start"], r["finish"], r["makespan"])


def test_cfg2_cholesky_counts_closed_form():
    for N in list(range(1, 13)) + [40]:
        rp, col, ty = synth.cholesky_dag(N)
        n_exp = N + 2 * comb(N, 2) + comb(N, 3)
        m_exp = (N - 1) * (2 * N - 1) + 2 * comb(N, 3) + comb(N - 1, 3)
        assert ty.size == n_exp and col.size == m_exp
        assert (np.bincount(ty, minlength=4) == [N, comb(N, 2), comb(N, 2), comb(N, 3)]).all()
        oracle.canon(ty.size, rp, col)  # acyclic, no repeats
    assert synth.cfg2().n == 11480 and synth.cfg2().m == 31980


def _stf_edges(tasks):
    """Dependencies of a sequential task flow derived generically: each task
    lists the tiles it reads and writes; an edge joins the last writer of a
    tile to a later reader or writer of it, and every reader since that write
    to a later writer."""
    last_w, readers, edges = {}, {}, set()
    for t, (rd, wr) in enumerate(tasks):
        for tile in rd | wr:
            if tile in last_w:
                edges.add((last_w[tile], t))
        for tile in wr:
            for r in readers.get(tile, ()):
                if r != t:
                    edges.add((r, t))
        for tile in rd:
            readers.setdefault(tile, set()).add(t)
        for tile in wr:
            last_w[tile] = t
            readers[tile] = set()
    return edges


def test_lu_dag_matches_generic_task_flow():
    # tiled LU without pivoting as tile accesses, in the generator's order
    for nb in range(1, 7):
        tasks = []
        for k in range(nb):
            tasks.append(({(k, k)}, {(k, k)}))                                  # GETRF
            for j in range(k + 1, nb):
                tasks.append(({(k, k), (k, j)}, {(k, j)}))                      # row TRSM
            for i in range(k + 1, nb):
                tasks.append(({(k, k), (i, k)}, {(i, k)}))                      # column TRSM
            for i in range(k + 1, nb):
                for j in range(k + 1, nb):
                    tasks.append(({(i, k), (k, j), (i, j)}, {(i, j)}))          # GEMM
        rp, col, ty = synth.lu_dag(nb)
        got = {(u, int(v)) for u in range(ty.size) for v in col[rp[u]:rp[u + 1]]}
        assert got == _stf_edges(tasks), nb
        assert ty.size == nb * (nb + 1) * (2 * nb + 1) // 6
        oracle.canon(ty.size, rp, col)
    w = synth.lu_workload()
    assert w.n == 22140 and w.m == 63180


def test_cholesky_dag_matches_generic_task_flow():
    for nb in range(1, 7):
        tasks = []
        for k in range(nb):
            tasks.append(({(k, k)}, {(k, k)}))                                  # POTRF
            for i in range(k + 1, nb):
                tasks.append(({(k, k), (i, k)}, {(i, k)}))                      # TRSM
            for i in range(k + 1, nb):
                tasks.append(({(i, k), (i, i)}, {(i, i)}))                      # SYRK
                for j in range(k + 1, i):
                    tasks.append(({(i, k), (j, k), (i, j)}, {(i, j)}))          # GEMM
        rp, col, ty = synth.cholesky_dag(nb)
        got = {(u, int(v)) for u in range(ty.size) for v in col[rp[u]:rp[u + 1]]}
        assert got == _stf_edges(tasks), nb


# ------------------------------------------------- independent transcriptions

@pytest.mark.parametrize("chunk", range(4))
def test_c_plain_heap_and_python_twin_agree(chunk):
    for i in range(chunk * 60, chunk * 60 + 60):
        n = 1 + i % 37
        w = synth.random_dag(7, i, n, 0.05 + (i % 5) * 0.05, n_cpu=1 + i % 3, n_gpu=i % 2, dur_hi=25,
                             est_equal=(i % 3 != 0))
        for pol in ("inspirit", "fifo", "ability", "efi"):
            a = oracle.schedule(w, policy=pol, variant=oracle.PLAIN, trace=True)
            b = oracle.schedule(w, policy=pol, variant=oracle.HEAP)
            c = pyref.schedule(w.n, w.row_ptr, w.col, w.n_cpu, w.n_gpu, w.dur, w.est, policy=pol)
            for k in ("worker", "start", "finish", "ie_at_pop", "mode_at_pop"):
                assert np.array_equal(a[k], b[k]), (i, pol, k)
                assert a[k].tolist() == c[k], (i, pol, k)
            assert a["makespan"] == b["makespan"] == c["makespan"]
            assert [tuple(x) for x in a["trace"].tolist()] == c["trace"]


def test_variants_agree_on_many_releases_in_one_event():
    """Forty tasks that end together and share their eight successors: more
    releases in one event than the DAG has tasks."""
    k, m = 40, 8
    rp, col = csr(k + m, [(a, k + b) for a in range(k) for b in range(m)])
    for ticks in ([3, 3], [3, 5]):
        w = wl(k + m, rp, col, 30, 10, np.tile(ticks, (k + m, 1)))
        for pol in ("inspirit", "fifo", "efi"):
            a, b = oracle.schedule(w, policy=pol), oracle.schedule(w, policy=pol, variant=oracle.HEAP)
            for f in ("worker", "start", "finish", "ie_at_pop", "mode_at_pop"):
                assert np.array_equal(a[f], b[f]), (pol, f)


def test_plain_and_heap_agree_on_cholesky_and_layered():
    for w in (synth.cfg1(), synth.cfg2(nb=20), *synth.cfg3(select=[5, 6])):
        a = oracle.schedule(w, variant=oracle.PLAIN)
        b = oracle.schedule(w, variant=oracle.HEAP)
        for k in ("worker", "start", "finish", "ie_at_pop", "mode_at_pop"):
            assert np.array_equal(a[k], b[k]), k


def test_batch_driver_matches_single_runs():
    ws = synth.cfg3(select=[3, 9, 17])
    b = synth.concat(ws)
    r = oracle.schedule_batch(b, threads=3)
    for i, w in enumerate(ws):
        s = oracle.schedule(w, variant=oracle.HEAP)
        lo, hi = b.task_off[i], b.task_off[i + 1]
        assert r["makespan"][i] == s["makespan"]
        assert np.array_equal(r["start"][lo:hi], s["start"])


# ------------------------------------------------------------- error paths

def test_error_codes():
    one = np.ones((3, 2))
    rp, col = csr(3, [(0, 1), (1, 2), (2, 0)])
    with pytest.raises(oracle.OracleError) as e:
        oracle.schedule(wl(3, rp, col, 1, 0, one))
    assert e.value.code == oracle.E_CYCLE
    for bad_rp, bad_col in (([0, 2, 1, 1], [1, 2]), ([1, 1, 1, 1], [1]), ([0, 1, 1, 1], [5]),
                            ([0, 1, 1, 1], [0])):
        with pytest.raises(oracle.OracleError) as e:
            oracle.schedule(wl(3, bad_rp, bad_col, 1, 0, one))
        assert e.value.code == oracle.E_INVAL
    rp, col = csr(3, [(0, 1)])
    with pytest.raises(oracle.OracleError) as e:
        oracle.schedule(wl(3, rp, col, 1, 0, [[1, 1], [0, 1], [1, 1]]))
    assert e.value.code == oracle.E_RANGE
    with pytest.raises(oracle.OracleError) as e:
        oracle.schedule(wl(3, rp, col, 0, 0, one))
    assert e.value.code == oracle.E_RANGE
    with pytest.raises(oracle.OracleError) as e:
        oracle.schedule(wl(3, rp, col, 1, 0, one), max_events=1)
    assert e.value.code == oracle.E_HANG


def test_duplicate_edges_are_merged():
    rp = [0, 3, 3, 3]
    a = oracle.schedule(wl(3, rp, [1, 1, 2], 1, 1, [[3, 2]] * 3))
    b = oracle.schedule(wl(3, [0, 2, 2, 2], [1, 2], 1, 1, [[3, 2]] * 3))
    assert np.array_equal(a["start"], b["start"])


def test_generators_are_deterministic():
    a, b = synth.cfg1(), synth.cfg1()
    assert np.array_equal(a.col, b.col) and np.array_equal(a.dur, b.dur)
    c = synth.cfg3(select=[7])[0]
    d = synth.cfg3(select=[6, 7])[1]
    assert np.array_equal(c.col, d.col)
    sizes = synth.cfg3_sizes()
    assert sizes.min() >= 200 and sizes.max() <= 20000 and sizes.size == 4096


def _small(name):
    g = gold("w4_w7_small.json")[name]
    n = g["n"]
    dur = g.get("dur", g.get("est"))
    return g, wl(n, g["row_ptr"], g["col"], g.get("n_cpu", 0), g.get("n_gpu", 0), dur,
                 g.get("est", None))


def test_w4_simultaneous_readiness_pushed_in_id_order():
    g, w = _small("w4")
    r = oracle.schedule(w)
    assert r["worker"].tolist() == g["worker"] and r["start"].tolist() == g["start"]
    assert r["makespan"] == g["makespan"]


def test_w5_push_counts_the_running_task():
    g, w = _small("w5")
    for pol in ("inspirit", "fifo"):
        r = oracle.schedule(w, policy=pol)
        assert r["worker"].tolist() == g["worker"] and r["start"].tolist() == g["start"]


def test_w6_ladder_reaches_twice_the_largest_tau():
    g, w = _small("w6")
    ia, ie, U = oracle.attributes(g["n"], g["row_ptr"], g["col"], g["est"], g["n_gpu"])
    assert U == g["unit_time"] and ie.tolist() == g["ie"]


def test_w7_first_rule_is_high_ability():
    g, w = _small("w7")
    r = oracle.schedule(w)
    assert int(r["mode_at_pop"][0]) == g["mode_at_pop_first"]


# ------------------------------------------------------------- HEFT baseline

def _rank_reference(w):
    """Upward rank from its definition, by memoised recursion over successors:
    R(v) = n_cpu * est_cpu(v) + n_gpu * est_gpu(v) + max over successors R(s)."""
    import functools
    import sys
    sys.setrecursionlimit(10000)
    rp, col = oracle.canon(w.n, w.row_ptr, w.col)
    est = np.asarray(w.est, np.int64).reshape(w.n, 2)

    @functools.lru_cache(maxsize=None)
    def R(v):
        succ = col[rp[v]:rp[v + 1]]
        return int(w.n_cpu * est[v, 0] + w.n_gpu * est[v, 1]) + max((R(int(s)) for s in succ), default=0)
    return [R(v) for v in range(w.n)], rp, col


def test_w8_heft_hand_worked():
    g = gold("w8_heft.json")["w8"]
    w = wl(g["n"], g["row_ptr"], g["col"], g["n_cpu"], g["n_gpu"], g["dur"])
    assert _rank_reference(w)[0] == g["rank"]
    for variant in (oracle.PLAIN, oracle.HEAP):
        r = oracle.schedule(w, policy="heft", variant=variant)
        assert r["worker"].tolist() == g["heft"]["worker"] and r["start"].tolist() == g["heft"]["start"]
        assert r["makespan"] == g["heft"]["makespan"]
        assert set(r["mode_at_pop"].tolist()) == {g["heft"]["mode_at_pop"]}
    f = oracle.schedule(w, policy="fifo")
    assert f["start"].tolist() == g["fifo"]["start"] and f["makespan"] == g["fifo"]["makespan"]


@pytest.mark.parametrize("chunk", range(3))
def test_heft_pops_the_highest_rank_of_each_queue(chunk):
    # property of any HEFT schedule: a task is popped from its worker's queue
    # when no task waiting in that queue (pushed, not yet started) has a higher
    # rank, or an equal rank and an earlier readiness time (an earlier push).
    # Ranks come from the definition above, not from the oracle.
    for i in range(chunk * 40, chunk * 40 + 40):
        n = 2 + i % 40
        w = synth.random_dag(21, i, n, 0.05 + (i % 5) * 0.06, n_cpu=1 + i % 3, n_gpu=i % 3, dur_hi=30,
                             est_equal=(i % 2 == 0))
        R, rp, col = _rank_reference(w)
        r = oracle.schedule(w, policy="heft", variant=oracle.HEAP)
        start, finish, worker = r["start"], r["finish"], r["worker"]
        ready = np.zeros(n, np.int64)
        for v in range(n):
            for s in col[rp[v]:rp[v + 1]]:
                ready[s] = max(ready[s], finish[v])
        for v in range(n):
            waiting = [u for u in range(n) if worker[u] == worker[v] and ready[u] <= start[v] <= start[u]]
            assert max(R[u] for u in waiting) == R[v], (i, v)
            assert not any(R[u] == R[v] and ready[u] < ready[v] for u in waiting), (i, v)
        check_schedule(w, worker, start, finish, r["makespan"])


def test_heft_plain_and_heap_agree():
    for i in range(60):
        w = synth.random_dag(23, i, 1 + i % 45, 0.04 + (i % 6) * 0.05, n_cpu=1 + i % 4, n_gpu=i % 3, dur_hi=40,
                             est_equal=(i % 3 != 0))
        a = oracle.schedule(w, policy="heft", variant=oracle.PLAIN)
        b = oracle.schedule(w, policy="heft", variant=oracle.HEAP)
        for k in ("worker", "start", "finish", "ie_at_pop", "mode_at_pop"):
            assert np.array_equal(a[k], b[k]), (i, k)


# ------------------------------------------------- transitive attributes (f1)

def _paths_reference(n, rp, col, tau):
    """IA_T and every EF_v(d) by enumerating all paths out of v (exponential;
    tiny DAGs only) -- no dynamic programming, no topological order."""
    succ = [list(col[rp[v]:rp[v + 1]]) for v in range(n)]
    EF = [dict() for _ in range(n)]

    def walk(v, d, acc):
        acc += int(tau[d])
        if acc > EF[v].get(d, 0):
            EF[v][d] = acc
        for s in succ[d]:
            walk(v, s, acc)
    for v in range(n):
        walk(v, v, 0)
    return EF


def _reach_closure(n, rp, col):
    """D(v) sizes from the boolean closure of (I + A), squared until stable."""
    M = np.eye(n, dtype=bool)
    for v in range(n):
        M[v, col[rp[v]:rp[v + 1]]] = True
    while True:
        M2 = (M.astype(np.int64) @ M.astype(np.int64)) > 0
        if (M2 == M).all():
            return M.sum(axis=1)
        M = M2


@pytest.mark.parametrize("N", [1, 2, 5, 12])
def test_transitive_complete_dag_source_scores_every_task(N):
    # Section 4.3: in a fully connected DAG with one source, the source's
    # inspiring ability equals the number of tasks
    rp, col = csr(N, [(i, j) for i in range(N) for j in range(i + 1, N)])
    ia, _, _, cp = oracle.transitive(N, rp, col, np.ones((N, 2)), 1)
    assert ia[0] == N and ia.tolist() == [N - i for i in range(N)]
    assert cp == N


def test_w9_transitive_hand_worked():
    g = gold("w9_transitive.json")["w9"]
    ia, ie, U, cp = oracle.transitive(g["n"], g["row_ptr"], g["col"], g["est"], g["n_gpu"], unit_time=7)
    assert ia.tolist() == g["ia_t"] and ie.tolist() == g["ie_t_u7"] and U == 7 and cp == g["longest_path"]
    ia, ie, U, _ = oracle.transitive(g["n"], g["row_ptr"], g["col"], g["est"], g["n_gpu"])
    assert U == g["unit_time_auto"] and ie.tolist() == g["ie_t_auto"]


@pytest.mark.parametrize("key", ["w10_tie", "w10_top"])
def test_w10_transitive_ladder_edges(key):
    g = gold("w9_transitive.json")[key]
    _, ie, U, _ = oracle.transitive(g["n"], g["row_ptr"], g["col"], g["est"], g["n_gpu"])
    assert U == g["unit_time_auto"] and ie.tolist() == g["ie_t_auto"]


@pytest.mark.parametrize("seed", range(10))
def test_transitive_matches_path_enumeration(seed):
    w = synth.random_dag(51, seed, 3 + seed % 7, 0.35, n_cpu=1, n_gpu=seed % 2, dur_hi=12, est_equal=False)
    rp, col = oracle.canon(w.n, w.row_ptr, w.col)
    tau = w.est[:, 1 if w.n_gpu else 0]
    EF = _paths_reference(w.n, rp, col, tau)
    assert [len(e) for e in EF] == _reach_closure(w.n, rp, col).tolist()
    cp = max(max(e.values()) for e in EF)
    for U in (1, 5, 13, 30, cp, cp + 7):
        ia, ie, _, cp2 = oracle.transitive(w.n, rp, col, w.est, w.n_gpu, unit_time=U)
        assert cp2 == cp
        assert ia.tolist() == [len(e) for e in EF]
        assert ie.tolist() == [sum(x <= U for x in e.values()) for e in EF], U


def test_transitive_unit_time_limits():
    # Section 4.2: too small a unit time drives IE towards zero; too large a
    # one makes it converge to IA
    for seed in range(6):
        w = synth.random_dag(52, seed, 40, 0.1, n_cpu=2, n_gpu=1, dur_hi=30, est_equal=False)
        rp, col = oracle.canon(w.n, w.row_ptr, w.col)
        _, _, _, cp = oracle.transitive(w.n, rp, col, w.est, 1, unit_time=1)
        prev = None
        for U in sorted({1, 2, 3, 8, 40, 200, max(cp - 1, 1), cp, cp + 1}):
            ia, ie, _, _ = oracle.transitive(w.n, rp, col, w.est, 1, unit_time=U)
            tau = w.est[:, 1]
            assert ((tau > U) <= (ie == 0)).all()  # a task slower than U counts nothing
            if prev is not None:
                assert (ie >= prev).all()
            prev = ie
            if U >= cp:
                assert (ie == ia).all()


def test_transitive_chain_closed_form():
    n = 30
    rp, col = csr(n, [(i, i + 1) for i in range(n - 1)])
    est = synth.Stream(53, 1).randint(np.arange(2 * n).reshape(n, 2), 1, 20).astype(np.int32)
    tau = est[:, 1].astype(np.int64)
    for U in (3, 17, 60, 400):
        ia, ie, _, cp = oracle.transitive(n, rp, col, est, 1, unit_time=U)
        assert ia.tolist() == [n - i for i in range(n)] and cp == tau.sum()
        cum = np.concatenate([[0], np.cumsum(tau)])
        # tasks i..j finish within U of i's start while cum[j+1] - cum[i] <= U
        want = [int(np.searchsorted(cum, cum[i] + U, side="right")) - 1 - i for i in range(n)]
        assert ie.tolist() == want


def test_transitive_out_tree_closed_form():
    # in an out-tree every descendant has a single path from v: EF is the sum
    # of tau along it, and D(v) is v's subtree
    rng = np.random.default_rng(54)
    n = 60
    parent = [-1] + [int(rng.integers(0, v)) for v in range(1, n)]
    rp, col = csr(n, [(parent[v], v) for v in range(1, n)])
    est = rng.integers(1, 15, (n, 2)).astype(np.int32)
    tau = est[:, 1].astype(np.int64)
    depth_sum = np.zeros(n, np.int64)
    for v in range(n):
        depth_sum[v] = tau[v] + (depth_sum[parent[v]] if parent[v] >= 0 else 0)
    anc = [set() for _ in range(n)]
    for v in range(n):
        u = v
        while u >= 0:
            anc[v].add(u)
            u = parent[u]
    U = 25
    ia, ie, _, _ = oracle.transitive(n, rp, col, est, 1, unit_time=U)
    for v in range(n):
        sub = [d for d in range(n) if v in anc[d]]
        assert ia[v] == len(sub)
        # EF_v(d) = depth_sum[d] - depth_sum[v] + tau[v]
        assert ie[v] == sum(depth_sum[d] - depth_sum[v] + tau[v] <= U for d in sub)


def test_transitive_auto_unit_time_maximises_score_over_ladder():
    for seed in range(6):
        w = synth.random_dag(55, seed, 35, 0.12, n_cpu=1, n_gpu=1, dur_hi=25, est_equal=False)
        rp, col = oracle.canon(w.n, w.row_ptr, w.col)
        _, ie_auto, U, cp = oracle.transitive(w.n, rp, col, w.est, 1)
        J = 0
        while 2 ** J < cp:
            J += 1
        scores = {}
        for j in range(J + 1):
            ia, ie, _, _ = oracle.transitive(w.n, rp, col, w.est, 1, unit_time=2 ** j)
            scores[2 ** j] = int(((ie > 0) & (ie < ia)).sum())
        best = max(scores.values())
        assert U == max(u for u, s in scores.items() if s == best)
        assert np.array_equal(ie_auto, oracle.transitive(w.n, rp, col, w.est, 1, unit_time=U)[1])


def test_transitive_longest_path_limit():
    # the longest path must stay below 2^30 ticks
    n = 1100
    rp, col = csr(n, [(i, i + 1) for i in range(n - 1)])
    est = np.full((n, 2), 1 << 20, np.int32)
    with pytest.raises(oracle.OracleError) as e:
        oracle.transitive(n, rp, col, est, 1)
    assert e.value.code == oracle.E_RANGE
    ia, _, _, _ = oracle.transitive(1023, *csr(1023, [(i, i + 1) for i in range(1022)]), est[:1023], 1)
    assert ia[0] == 1023


@pytest.mark.parametrize("chunk", range(2))
def test_transitive_schedule_pops_by_static_keys(chunk):
    # with transitive attributes the keys never change while a task waits:
    # under the ability-only rule a pop takes the waiting task with the
    # largest (IA_T, IE_T), ties to the earlier readiness; attributes come
    # from path enumeration, not from the oracle
    for i in range(chunk * 25, chunk * 25 + 25):
        n = 3 + i % 8
        w = synth.random_dag(56, i, n, 0.3, n_cpu=1 + i % 2, n_gpu=i % 2, dur_hi=15, est_equal=(i % 2 == 0))
        rp, col = oracle.canon(w.n, w.row_ptr, w.col)
        EF = _paths_reference(n, rp, col, w.est[:, 1 if w.n_gpu else 0])
        U = 12
        ia = [len(e) for e in EF]
        ie = [sum(x <= U for x in e.values()) for e in EF]
        for variant in (oracle.PLAIN, oracle.HEAP):
            r = oracle.schedule(w, policy="ability", variant=variant, attr_mode="transitive", unit_time=U)
            start, finish, worker = r["start"], r["finish"], r["worker"]
            assert r["ie_at_pop"].tolist() == ie
            ready = np.zeros(n, np.int64)
            for v in range(n):
                for s in col[rp[v]:rp[v + 1]]:
                    ready[s] = max(ready[s], finish[v])
            for v in range(n):
                waiting = [u for u in range(n) if worker[u] == worker[v] and ready[u] <= start[v] <= start[u]]
                top = max((ia[u], ie[u]) for u in waiting)
                assert (ia[v], ie[v]) == top, (i, v)
                assert not any((ia[u], ie[u]) == top and ready[u] < ready[v] for u in waiting), (i, v)
            check_schedule(w, worker, start, finish, r["makespan"])


def test_transitive_schedule_plain_and_heap_agree():
    for i in range(40):
        w = synth.random_dag(57, i, 2 + i % 40, 0.05 + (i % 5) * 0.05, n_cpu=1 + i % 3, n_gpu=i % 3, dur_hi=30,
                             est_equal=(i % 2 == 0))
        for pol in ("inspirit", "efi"):
            a = oracle.schedule(w, policy=pol, variant=oracle.PLAIN, attr_mode="transitive")
            b = oracle.schedule(w, policy=pol, variant=oracle.HEAP, attr_mode="transitive")
            for k in ("worker", "start", "finish", "ie_at_pop", "mode_at_pop"):
                assert np.array_equal(a[k], b[k]), (i, pol, k)


# ------------------------------------------------------------ data model (f2)

def _data_w(g):
    d = np.asarray(g["dur"], np.int32)
    return NS(n=g["n"], row_ptr=np.asarray(g["row_ptr"], np.int32), col=np.asarray(g["col"], np.int32), dur=d,
              est=d, n_cpu=g["n_cpu"], n_gpu=g["n_gpu"], data_kib=np.asarray(g["data_kib"], np.int32))


@pytest.mark.parametrize("variant", [oracle.PLAIN, oracle.HEAP])
def test_w11_data_model_hand_worked(variant):
    g = gold("w11_data.json")["w11"]
    w = _data_w(g)
    for pol, key, bw in (("locality", "locality", g["data_bw"]), ("efi", "efi", g["data_bw"]),
                         ("locality", "locality_no_data", 0)):
        r = oracle.schedule(w, policy=pol, variant=variant, unit_time=g["unit_time"], data_bw=bw)
        for f in ("worker", "start", "finish"):
            assert r[f].tolist() == g[key][f], (key, f)
        assert r["makespan"] == g[key]["makespan"], key
        # a worker holding a task whose inputs are still moving is busy
        # but not running it, so the non-idling property does not apply
        check_schedule(w, r["worker"], r["start"], r["finish"], r["makespan"], non_idling=bw == 0)
    r = oracle.schedule(w, policy="locality", variant=variant, unit_time=g["unit_time"], data_bw=g["data_bw"])
    assert r["ie_at_pop"].tolist() == g["locality"]["ie_at_pop"]
    assert set(r["mode_at_pop"].tolist()) == {g["locality"]["mode_at_pop"]}


@pytest.mark.parametrize("variant", [oracle.PLAIN, oracle.HEAP])
def test_w12_transfers_overlap_and_are_not_shared(variant):
    g = gold("w11_data.json")["w12"]
    r = oracle.schedule(_data_w(g), policy="fifo", variant=variant, data_bw=g["data_bw"])
    for f in ("worker", "start", "finish"):
        assert r[f].tolist() == g["fifo"][f], f
    assert r["makespan"] == g["fifo"]["makespan"]


def _with_data(w, seed, hi=64):
    w.data_kib = synth.Stream(seed, 9).randint(np.arange(w.n), 0, hi).astype(np.int32)
    return w


@pytest.mark.parametrize("policy", ["inspirit", "fifo", "efi", "locality", "heft"])
def test_data_model_reduces_to_the_plain_model(policy):
    # no transfer ever costs anything when every item is empty, when all
    # workers share one memory node (CPUs only, or a single GPU), so the
    # schedules are those of the model without data
    for i in range(20):
        w = _with_data(synth.random_dag(71, i, 3 + i * 3, 0.12, n_cpu=1 + i % 3, n_gpu=1 + i % 2, dur_hi=30), i)
        base = oracle.schedule(w, policy=policy, variant=oracle.HEAP)
        w0 = NS(**{**vars(w), "data_kib": np.zeros(w.n, np.int32)})
        r = oracle.schedule(w0, policy=policy, variant=oracle.HEAP, data_bw=100)
        assert np.array_equal(r["start"], base["start"]) and np.array_equal(r["worker"], base["worker"]), i
        for n_cpu, n_gpu in ((3, 0), (0, 1)):
            wm = NS(**{**vars(w), "n_cpu": n_cpu, "n_gpu": n_gpu})
            a = oracle.schedule(wm, policy=policy, variant=oracle.HEAP)
            b = oracle.schedule(wm, policy=policy, variant=oracle.HEAP, data_bw=7)
            assert np.array_equal(a["start"], b["start"]) and np.array_equal(a["worker"], b["worker"]), (i, n_cpu)


@pytest.mark.parametrize("policy", ["inspirit", "locality", "fifo"])
def test_data_model_start_covers_input_transfers(policy):
    # every input moved from another memory node costs its ticks after the
    # task became ready: start >= last input's finish + the sum of the remote
    # inputs' transfer ticks (the transfers of one task run back to back)
    for i in range(30):
        bw = 256 + 512 * (i % 4)
        w = _with_data(synth.random_dag(72, i, 5 + i * 2, 0.15, n_cpu=1 + i % 3, n_gpu=1 + i % 3, dur_hi=40,
                                        est_equal=(i % 2 == 0)), 50 + i, hi=200)
        r = oracle.schedule(w, policy=policy, variant=oracle.HEAP, data_bw=bw)
        check_schedule(w, r["worker"], r["start"], r["finish"], r["makespan"], non_idling=False)
        rp, col = oracle.canon(w.n, w.row_ptr, w.col)
        node = np.where(r["worker"] < w.n_cpu, 0, 1 + r["worker"] - w.n_cpu)
        preds = [[] for _ in range(w.n)]
        for u in range(w.n):
            for s in col[rp[u]:rp[u + 1]]:
                preds[s].append(u)
        for v in range(w.n):
            if preds[v]:
                ready = max(r["finish"][u] for u in preds[v])
                x = sum(-(-1024 * int(w.data_kib[u]) // bw) for u in preds[v] if node[u] != node[v])
                assert r["start"][v] >= ready + x, (i, v)


def test_data_model_plain_and_heap_agree():
    for i in range(40):
        w = _with_data(synth.random_dag(73, i, 2 + i * 2, 0.1, n_cpu=1 + i % 4, n_gpu=i % 3, dur_hi=30,
                                        est_equal=(i % 2 == 0)), 90 + i)
        for pol in ("inspirit", "locality"):
            for am in ("direct", "transitive"):
                a = oracle.schedule(w, policy=pol, variant=oracle.PLAIN, data_bw=512, attr_mode=am)
                b = oracle.schedule(w, policy=pol, variant=oracle.HEAP, data_bw=512, attr_mode=am)
                for k in ("worker", "start", "finish", "ie_at_pop", "mode_at_pop"):
                    assert np.array_equal(a[k], b[k]), (i, pol, am, k)


def test_data_model_range_checks():
    w = _with_data(synth.random_dag(74, 0, 6, 0.4, n_cpu=1, n_gpu=1), 1)
    w.data_kib[0] = -1
    with pytest.raises(oracle.OracleError) as e:
        oracle.schedule(w, data_bw=10)
    assert e.value.code == oracle.E_RANGE


@pytest.mark.parametrize("case", ["heft", "transitive", "data", "locality"])
def test_new_policies_never_beat_the_brute_force_optimum(case):
    # any list schedule is a schedule: its makespan is at least the optimum
    # over all schedules (and transfers only add waits to a schedule that
    # stays feasible without them)
    kw = {"heft": dict(policy="heft"), "transitive": dict(attr_mode="transitive"),
          "data": dict(data_bw=256), "locality": dict(policy="locality", data_bw=256)}[case]
    for i in range(12):
        w = synth.random_dag(91, i, 3 + i % 5, 0.35, dur_hi=7, n_cpu=1, n_gpu=1 + i % 2)
        w.data_kib = synth.Stream(92, i).randint(np.arange(w.n), 0, 3).astype(np.int32)
        r = oracle.schedule(w, variant=oracle.HEAP, **kw)
        assert r["makespan"] >= oracle.brute_opt(w), (case, i)

"""Serving-queue policy on the simulation backend (no GPU).

The simulation backend runs the library's own scheduler thread -- admission,
grouping, stream assignment, completion, accounting -- with modelled launch
durations instead of device work, so these tests exercise the same code the
HIP backend uses, minus the launches.  Device-input requests carry fake,
never-dereferenced pointers here.
"""
import ctypes
import threading
import time

import numpy as np
import pytest

import paper_2608_25469_amd as hs

pytestmark = pytest.mark.skipif(not hs.os.path.exists(hs.LIB_PATH), reason="library not built")

FAKE = 0x1000  # never dereferenced by the simulation backend
MS = 1e6       # ns


def dev_req(m, n, cx=False, alpha=1.0, t_arrival_ns=0.0):
    a = complex(alpha)
    prob = hs.Problem(hs.NON_UNIT, hs.C64F if cx else hs.R64F, m, n, a.real, a.imag,
                      ctypes.c_void_p(FAKE), m, ctypes.c_void_p(FAKE), m)
    return hs.Request(prob, hs.INPUT_DEVICE, 0, 0, t_arrival_ns)


def syn_req(m, n, key=1, cx=False, keep=False):
    return hs.request(m, n, 1.0, complex_=cx, key=key, release_on_completion=not keep)


def sim_queue(rate_flops_per_ns=1000.0, fixed_ns=0.0, **kw):
    return hs.Queue(simulated=True, sim_flops_per_ns=rate_flops_per_ns, sim_fixed_ns=fixed_ns, **kw)


def wait_all(q, tickets, timeout_s=20.0):
    return [q.wait(t, timeout_s) for t in tickets]


def test_fifo_admission_under_budget():
    r = dev_req(1024, 1024)               # 1.07e9 flops -> ~1.1 ms at 1 TF/s... scaled below
    fp = hs.request_footprint(r)
    assert fp > 0
    # budget for exactly one request at a time
    with sim_queue(rate_flops_per_ns=200.0, hbm_budget_bytes=int(fp * 1.5)) as q:
        tk = q.submit([dev_req(1024, 1024) for _ in range(5)])
        infos = wait_all(q, tk)
        st = q.stats()
    assert [i["status"] for i in infos] == [0] * 5
    assert all(i["path"] == 2 for i in infos)
    admits = [i["t_admit_ns"] for i in infos]
    dones = [i["t_done_ns"] for i in infos]
    assert admits == sorted(admits)                # arrival order
    for k in range(1, 5):                          # one at a time
        assert admits[k] >= dones[k - 1]
    assert st["bytes_peak"] <= int(fp * 1.5)
    assert st["bytes_peak"] == fp
    assert st["completed"] == 5 and st["failed"] == 0 and st["bytes_in_use"] == 0


def test_too_large_rejected_all_or_nothing():
    big = dev_req(4096, 512)
    fp = hs.request_footprint(big)
    with sim_queue(hbm_budget_bytes=fp - 1) as q:
        with pytest.raises(hs.HsmaError) as e:
            q.submit(big)
        assert e.value.status == 7
        with pytest.raises(hs.HsmaError) as e:
            q.submit([dev_req(32, 32), big])       # nothing of this batch is queued
        assert e.value.status == 7
        st = q.stats()
        assert st["rejected"] == 2 and st["submitted"] == 0
        t = q.submit(dev_req(32, 32))
        q.wait(t, 10)
        assert q.stats()["submitted"] == 1


def test_max_inflight_limit():
    with sim_queue(rate_flops_per_ns=400.0, max_inflight=2, n_streams=8) as q:
        tk = q.submit([dev_req(1024, 1024) for _ in range(6)])
        infos = wait_all(q, tk)
    iv = [(i["t_admit_ns"], i["t_done_ns"]) for i in infos]
    for a, _ in iv:
        live = sum(1 for s, e in iv if s <= a < e)
        assert live <= 2


def test_small_requests_grouped_per_round():
    with sim_queue(rate_flops_per_ns=1.0) as q:
        # one large request first keeps the scheduler busy while the small ones queue up
        tk = q.submit([dev_req(16 + i % 48, 1 + i % 64, cx=bool(i % 3 == 0)) for i in range(50)])
        infos = wait_all(q, tk)
    assert all(i["path"] == 1 for i in infos)
    assert len({i["t_admit_ns"] for i in infos}) == 1      # admitted in one round
    assert len({i["t_done_ns"] for i in infos}) == 1       # one launch


def test_kept_results_hold_budget_until_release():
    r = syn_req(512, 256, keep=True)
    fp = hs.request_footprint(r)
    data = 8 * (512 * 512 + 512 * 256)
    assert fp > data
    with sim_queue(hbm_budget_bytes=int(fp * 1.5)) as q:
        t1, t2 = q.submit([syn_req(512, 256, key=1, keep=True), syn_req(512, 256, key=2, keep=True)])
        i1 = q.wait(t1, 10)
        assert i1["status"] == 0
        assert q.stats()["bytes_in_use"] == data           # result kept, workspace returned
        time.sleep(0.05)
        st, _ = q.poll(t2)
        assert st == 9                                     # still pending: no room
        assert q.stats()["pending"] == 1
        q.release(t1)
        i2 = q.wait(t2, 10)
        assert i2["status"] == 0 and i2["t_admit_ns"] >= i1["t_done_ns"]
        q.release(t2)
        assert q.stats()["bytes_in_use"] == 0
        assert q.poll(t1)[0] == 11                          # released -> not found


def test_release_on_completion_frees_everything():
    with sim_queue() as q:
        tk = q.submit([syn_req(300, 40, key=k) for k in range(8)])
        wait_all(q, tk)
        assert q.stats()["bytes_in_use"] == 0


def test_latency_statistics_match_records():
    with sim_queue(rate_flops_per_ns=2000.0, fixed_ns=20_000.0) as q:
        rng = np.random.default_rng(0)
        reqs = [dev_req(int(m), int(n)) for m, n in zip(rng.integers(8, 600, 40), rng.integers(1, 200, 40))]
        tk = q.submit(reqs)
        infos = wait_all(q, tk)
        st = q.stats()
    lat = np.sort([i["t_done_ns"] - i["t_arrival_ns"] for i in infos])
    assert st["completed"] == 40
    # percentiles come from a histogram with bins 2^(1/64) wide: within 0.6 %
    for q_, key in ((0.5, "p50_ns"), (0.99, "p99_ns")):
        ex = lat[int(q_ * 39 + 0.5)]
        assert abs(st[key] - ex) <= 0.006 * ex, (key, st[key], ex)
    assert st["max_ns"] == lat[-1]
    assert abs(st["mean_ns"] - lat.mean()) <= 1e-6 * lat.mean()
    assert st["solves_per_s"] > 0
    assert all(i["t_arrival_ns"] <= i["t_admit_ns"] <= i["t_done_ns"] for i in infos)


def test_scheduled_arrival_counts_toward_latency():
    with sim_queue() as q:
        t0 = hs.clock_ns()
        t = q.submit(dev_req(32, 32, t_arrival_ns=t0 - 5 * MS))
        i = q.wait(t, 10)
    assert i["t_arrival_ns"] == t0 - 5 * MS
    assert i["t_done_ns"] - i["t_arrival_ns"] >= 5 * MS


def test_validation():
    with sim_queue() as q:
        bad = dev_req(32, 32)
        bad.input = 7
        with pytest.raises(hs.HsmaError) as e:
            q.submit(bad)
        assert e.value.status == 1
        with pytest.raises(hs.HsmaError) as e:
            q.submit(dev_req(0, 5))
        assert e.value.status == 2
        r = dev_req(32, 32)
        r.prob.alpha_im = 1.0
        with pytest.raises(hs.HsmaError) as e:
            q.submit(r)
        assert e.value.status == 1
        r = dev_req(32, 32)
        r.prob.A = None
        with pytest.raises(hs.HsmaError) as e:
            q.submit(r)
        assert e.value.status == 3
        r = dev_req(32, 32)
        r.prob.lda = 16
        with pytest.raises(hs.HsmaError) as e:
            q.submit(r)
        assert e.value.status == 2
        r = syn_req(32, 32)
        r.release_on_completion = 3
        with pytest.raises(hs.HsmaError) as e:
            q.submit(r)
        assert e.value.status == 1
        assert q.poll(12345)[0] == 11
        with pytest.raises(hs.HsmaError) as e:
            q.release(12345)
        assert e.value.status == 11
        assert q.stats()["submitted"] == 0


def test_release_and_wait_while_running():
    with sim_queue(rate_flops_per_ns=5.0) as q:      # 1.3e8 flops -> ~27 ms
        t = q.submit(dev_req(512, 512))
        with pytest.raises(hs.HsmaError) as e:
            q.release(t)
        assert e.value.status == 9
        with pytest.raises(hs.HsmaError) as e:
            q.wait(t, 0.001)
        assert e.value.status == 10
        assert q.wait(t, 20)["status"] == 0


def test_concurrent_submitters():
    with sim_queue(rate_flops_per_ns=50000.0) as q:
        got = [[] for _ in range(4)]

        def worker(k):
            for i in range(50):
                got[k].append(q.submit(dev_req(8 + (i * 7 + k) % 120, 1 + i % 30)))

        ths = [threading.Thread(target=worker, args=(k,)) for k in range(4)]
        for t in ths:
            t.start()
        for t in ths:
            t.join()
        tickets = [t for g in got for t in g]
        assert len(set(tickets)) == 200
        infos = wait_all(q, tickets)
        assert all(i["status"] == 0 for i in infos)
        assert q.stats()["completed"] == 200


def test_destroy_with_unadmittable_pending_returns():
    r = syn_req(512, 256, keep=True)
    fp = hs.request_footprint(r)
    q = sim_queue(hbm_budget_bytes=int(fp * 1.5))
    t1, t2 = q.submit([syn_req(512, 256, key=1, keep=True), syn_req(512, 256, key=2, keep=True)])
    q.wait(t1, 10)
    t0 = time.time()
    q.close()                                            # t2 can never be admitted
    assert time.time() - t0 < 5.0


def test_config_validation():
    h = ctypes.c_void_p()
    cfg = hs.QueueConfig(5, 0, 0, 0, 0, 0.0, 0.0)
    assert hs.lib().hsma_queue_create(ctypes.byref(cfg), ctypes.byref(h)) == 1
    cfg = hs.QueueConfig(hs.BACKEND_SIMULATED, -1, 0, 0, 0, 0.0, 0.0)
    assert hs.lib().hsma_queue_create(ctypes.byref(cfg), ctypes.byref(h)) == 1
    assert hs.lib().hsma_queue_create(ctypes.byref(cfg), None) == 3


def test_blocked_classes_split_by_size_and_data_type():
    """One admission round with a real and a complex request of each blocked
    size class: four class launches on four different streams, each modelled
    as fixed + its own flops / rate, so each request finishes at its own
    class's modelled time (a launch shared by the real and the complex
    request of a class would finish both at the summed time).  The real
    requests have four times the columns, so the two requests of a class
    model the same time and a shared launch would double it: the bound
    (40 % over the model) separates the two with room for a late wake-up of
    the retiring thread on a busy host."""
    rate, fixed = 0.05, 1_000.0
    shapes = [(200, 40, False), (200, 10, True), (600, 40, False), (600, 10, True)]
    with sim_queue(rate_flops_per_ns=rate, fixed_ns=fixed, n_streams=8) as q:
        tk = q.submit([dev_req(m, n, cx=cx) for m, n, cx in shapes])
        infos = wait_all(q, tk)
    assert all(i["status"] == 0 and i["path"] == 2 for i in infos)
    assert len({i["t_admit_ns"] for i in infos}) == 1          # one round
    for (m, n, cx), i in zip(shapes, infos):
        model = fixed + m * m * n * (4.0 if cx else 1.0) / rate
        took = i["t_done_ns"] - i["t_admit_ns"]
        assert model * 0.999 <= took <= 1.4 * model, (m, cx, took, model)


def exact_pct(v, q):
    v = np.sort(np.asarray(v))
    return float(v[int(q * (len(v) - 1) + 0.5)])


def test_latency_histogram_matches_exact_order_statistics():
    """Percentiles from the fixed-size histogram are within 0.6 % of the exact
    order statistics of the same latencies, overall and per size class
    (m <= 64, 64 < m <= 512, m > 512); max and mean are exact."""
    shapes = [(8 + (i * 37) % 1500, 1 + (i * 11) % 40) for i in range(300)]
    with sim_queue(rate_flops_per_ns=2000.0, fixed_ns=20_000.0) as q:
        tk = q.submit([dev_req(m, n) for m, n in shapes])
        infos = wait_all(q, tk)
        st = q.stats()
    lat = np.array([i["t_done_ns"] - i["t_arrival_ns"] for i in infos])
    assert st["all"]["count"] == len(shapes) == st["completed"]
    for q_, key in ((0.5, "p50_ns"), (0.99, "p99_ns")):
        ex = exact_pct(lat, q_)
        assert abs(st["all"][key] - ex) <= 0.006 * ex, (key, st["all"][key], ex)
        assert st[key] == st["all"][key]
    assert st["all"]["max_ns"] == lat.max()
    assert abs(st["all"]["mean_ns"] - lat.mean()) <= 1e-9 * lat.mean()
    cls = np.array([0 if m <= 64 else (1 if m <= 512 else 2) for m, _ in shapes])
    for c, name in enumerate(hs.LATENCY_CLASS_NAMES):
        sub = lat[cls == c]
        got = st["by_class"][name]
        assert got["count"] == len(sub) > 0, name
        for q_, key in ((0.5, "p50_ns"), (0.99, "p99_ns")):
            ex = exact_pct(sub, q_)
            assert abs(got[key] - ex) <= 0.006 * ex, (name, key, got[key], ex)
        assert got["max_ns"] == sub.max()


def test_fire_and_forget_drops_records_but_counts():
    """release_on_completion = 2: the record is gone once the request has
    finished (poll, wait and release give NOT_FOUND), its memory is freed, and
    it still enters the counters and the latency statistics."""
    with sim_queue(rate_flops_per_ns=5000.0) as q:
        reqs = [hs.request(64 + 8 * i, 16, 1.0, key=100 + i, forget=True) for i in range(50)]
        assert all(r.release_on_completion == 2 for r in reqs)
        tk = q.submit(reqs)
        deadline = time.time() + 20
        while q.stats()["completed"] < 50 and time.time() < deadline:
            time.sleep(0.005)
        st = q.stats()
        assert st["completed"] == 50 and st["all"]["count"] == 50
        assert st["bytes_in_use"] == 0 and st["inflight"] == 0
        for t in tk:
            assert q.poll(t)[0] == 11
            with pytest.raises(hs.HsmaError) as e:
                q.release(t)
            assert e.value.status == 11
        with pytest.raises(hs.HsmaError) as e:
            q.wait(tk[0], 1)
        assert e.value.status == 11


def test_stats_window_leaves_out_earlier_arrivals():
    with sim_queue(rate_flops_per_ns=5000.0) as q:
        early = q.submit([dev_req(100, 10) for _ in range(5)])
        wait_all(q, early)
        assert q.stats()["all"]["count"] == 5
        t_from = hs.clock_ns()
        q.stats_reset(t_from)
        st = q.stats()
        assert st["all"]["count"] == 0 and st["completed"] == 5      # counters kept
        # one arrival stamped before the window, three inside it
        tk = q.submit([dev_req(100, 10, t_arrival_ns=t_from - 1e6)] +
                      [dev_req(100, 10) for _ in range(3)])
        wait_all(q, tk)
        st = q.stats()
        assert st["completed"] == 9 and st["all"]["count"] == 3
        assert st["by_class"]["64<m<=512"]["count"] == 3


def test_default_budget_is_32_gib():
    """A synthetic request whose inputs alone exceed 32 GiB is rejected by a
    queue with the default budget, and one just below it is accepted."""
    with sim_queue() as q:
        big = syn_req(65536, 1)            # 8 (m^2 + m) bytes > 32 GiB
        assert hs.request_footprint(big) > 32 * 2**30
        with pytest.raises(hs.HsmaError) as e:
            q.submit(big)
        assert e.value.status == 7
        ok = syn_req(40000, 1)             # about 12 GiB
        assert hs.request_footprint(ok) < 32 * 2**30
        t = q.submit(ok)
        assert q.wait(t, 60)["status"] == 0


def test_footprint_covers_what_a_solve_takes():
    """The budget bounds what is allocated: a request's footprint is at least
    the workspace its solve takes, and, beyond that, no more than descriptors
    (256 bytes an operation) and the share that every request pays."""
    f = hs.lib()["_ZN4hsma13blocked_bytesIdEEmbllib"]   # blocked_bytes<double>
    f.argtypes = [ctypes.c_bool, ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_bool]
    f.restype = ctypes.c_size_t
    chains = 0
    for cx in (False, True):
        for m in (65, 200, 257, 512, 513, 1000, 1024, 2048, 4096, 8192, 16384, 40000):
            for n in (1, 15, 16, 17, 256, 257, 512, 1000, 1024, 1025, 4096):
                ws = f(cx, m, n, 0, False)
                chains += ws > 0
                most = ws + 4096 + 512 + 512 * (m * (2 if cx else 1) // 256 + 2)
                fp = hs.request_footprint(dev_req(m, n, cx))
                assert ws + 4096 <= fp <= most, (m, n, cx, ws, fp)
                data = (16 if cx else 8) * (m * m + m * n)
                assert hs.request_footprint(syn_req(m, n, cx=cx)) == fp + data
    assert chains > 50
    assert hs.request_footprint(dev_req(64, 64)) == 4096

"""One TAS handle shared by two host threads on two HIP streams: every call takes its scratch from the
workspace of its own stream, so the results must be those of the oracle whatever the interleaving."""
import sys
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2105_13336_amd as P  # noqa: E402
from oracle import oracle as O  # noqa: E402
from workloads import make_plans, plans_from_lists, small_random_tas  # noqa: E402


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def with_long_plans(base, which, length):
    """The batch with the plans `which` repeated until they hold `length` intervals (more than the evaluation
    kernel keeps in registers: those plans go to the kernel that is gated by the per-launch flag)."""
    lists = []
    for b in range(base.B):
        t, o, r, k = base.plan(b)
        one = [(int(t[j]), int(o[j]), int(r[j]), int(k[j])) for j in range(len(t))]
        if b in which and one:
            one = (one * (length // len(one) + 1))[:length + b]
        lists.append(one)
    return plans_from_lists(lists)


def test_two_threads_two_streams_one_handle(tuning):
    tuning("eval_segments", 3)          # several segments per plan: per-segment partials live in scratch
    tas = small_random_tas(7001, N=400, T=20011, max_acc=5, timed=True, link_bytes_per_us=400_000)
    batches = [with_long_plans(make_plans(tas, 37, 1, p_swap=0.6), {0, 11, 35}, 2100),
               make_plans(tas, 23, 2, p_swap=0.4)]
    say(f"two threads, two streams: B={[b.B for b in batches]} K={[b.n_intervals for b in batches]}")
    want = []
    for pl in batches:
        r0, p0, a0, m0 = O.eval_plans(tas, pl)
        want.append((r0, p0, a0, m0, O.score_plans(tas, pl, r0, p0, a0), O.score_recompute_plans(tas, pl, r0, p0, a0),
                     O.link_occupancy(tas, pl, reuse=True)))
    h = P.tas_load(tas)
    got, errors = [None, None], []
    start = threading.Barrier(2)

    def worker(k):
        try:
            torch.cuda.set_device(0)
            pl = batches[k]
            B, T, N = pl.B, tas.T, tas.N
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                dp = P.DevicePlans.from_numpy(pl.plan_offsets, pl.iv_tensor, pl.iv_out, pl.iv_in, pl.iv_kind)
                res = torch.empty((B, T), dtype=torch.int64, device="cuda")
                peak = torch.empty(B, dtype=torch.int64, device="cuda")
                arg = torch.empty(B, dtype=torch.int32, device="cuda")
                mn = torch.empty(B, dtype=torch.int64, device="cuda")
                sc = [torch.empty((B, N), dtype=torch.int64, device="cuda") for _ in range(2)]
                wo = [torch.empty((B, N), dtype=torch.int32, device="cuda") for _ in range(2)]
                wi = [torch.empty((B, N), dtype=torch.int32, device="cuda") for _ in range(2)]
                link = torch.empty((B, T), dtype=torch.int32, device="cuda")
                lpk, larg, lover = (torch.empty(B, dtype=torch.int32, device="cuda") for _ in range(3))
                start.wait()
                for _ in range(25):     # enqueue only: nothing here waits for the device
                    P.tensile_eval_plans(h, dp, res, peak, arg, mn, stream=s)
                    P.tensile_score_candidates(h, dp, res, peak, arg, sc[0], wo[0], wi[0], stream=s)
                    P.tensile_score_recompute(h, dp, res, peak, arg, sc[1], wo[1], wi[1], stream=s)   # (first call builds its index)
                    P.tensile_eval_link(h, dp, lpk, link, larg, lover, reuse_host_copies=True, stream=s)
                s.synchronize()
                got[k] = [x.cpu().numpy() for x in (res, peak, arg, mn, sc[0], wo[0], wi[0], sc[1], wo[1], wi[1], link, lpk, larg, lover)]
        except Exception as e:      # noqa: BLE001 - reported below
            errors.append(e)

    threads = [threading.Thread(target=worker, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for k in range(2):
        r0, p0, a0, m0, (s0, o0, i0), (s1, o1, i1), (l0, lp0, la0, lo0) = want[k]
        names = ("resident", "peak", "argmax", "min", "score", "win_out", "win_in", "saving", "rc_out", "rc_in", "link",
                 "link_peak", "link_argmax", "overbooked")
        for name, g, w in zip(names, got[k], (r0, p0, a0, m0, s0, o0, i0, s1, o1, i1, l0, lp0, la0, lo0)):
            assert np.array_equal(g, w), f"thread {k}: {name}"
    h.close()


def test_one_call_steps_of_two_threads_on_one_handle():
    """Evaluation and scoring in one call from two host threads on two streams: what the one kernel hands to the other lives in
    the stream's workspace, which grows from batch to batch."""
    tas = small_random_tas(7003, N=700, T=12_001, max_acc=5, timed=True, link_bytes_per_us=400_000)
    batches = [[make_plans(tas, B, 31 + B, p_swap=0.4) for B in sizes] for sizes in ((5, 300, 40), (270, 9, 600))]
    say("one-call steps on two streams")
    want = [[(*O.eval_plans(tas, pl), O.score_plans(tas, pl, *O.eval_plans(tas, pl)[:3])) for pl in mine] for mine in batches]
    h = P.tas_load(tas)
    got, errors = [[], []], []
    start = threading.Barrier(2)

    def worker(k):
        try:
            torch.cuda.set_device(0)
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                dps = [P.DevicePlans.from_numpy(pl.plan_offsets, pl.iv_tensor, pl.iv_out, pl.iv_in, pl.iv_kind) for pl in batches[k]]
                outs = [[torch.empty(shape, dtype=dt, device="cuda") for shape, dt in
                         (((dp.B, tas.T), torch.int64), ((dp.B,), torch.int64), ((dp.B,), torch.int32), ((dp.B,), torch.int64),
                          ((dp.B, tas.N), torch.int64), ((dp.B, tas.N), torch.int32), ((dp.B, tas.N), torch.int32))] for dp in dps]
                start.wait()
                for _ in range(8):
                    for dp, out in zip(dps, outs):
                        P.tensile_eval_score_plans(h, dp, *out, stream=s)
                s.synchronize()
                got[k] = [[x.cpu().numpy() for x in out] for out in outs]
        except Exception as e:      # noqa: BLE001 - reported below
            errors.append(e)

    threads = [threading.Thread(target=worker, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for k in range(2):
        for b, (r0, p0, a0, m0, scores) in enumerate(want[k]):
            for j, (g, w) in enumerate(zip(got[k][b], (r0, p0, a0, m0, *scores))):
                assert np.array_equal(g, w), f"thread {k}, batch {b}, output {j}"
    h.close()


def test_greedy_next_to_a_batch_on_another_stream():
    """tensile_greedy_plan works on the default stream while a batch is evaluated over and over on another."""
    tas = small_random_tas(7002, N=200, T=9001, max_acc=5, timed=True, link_bytes_per_us=300_000)
    pl = make_plans(tas, 300, 5, p_swap=0.5)
    say("greedy next to a batch")
    h = P.tas_load(tas)
    og = O.greedy(tas, 0, max_iters=40)
    _, p0, a0, _ = O.eval_plans(tas, pl, want_resident=False)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        dp = P.DevicePlans.from_numpy(pl.plan_offsets, pl.iv_tensor, pl.iv_out, pl.iv_in, pl.iv_kind)
        peak = torch.empty(pl.B, dtype=torch.int64, device="cuda")
        arg = torch.empty(pl.B, dtype=torch.int32, device="cuda")
    out = {}

    def planner():
        torch.cuda.set_device(0)
        out["g"] = P.tensile_greedy_plan(h, 0, max_iters=40, capacity=64)

    th = threading.Thread(target=planner)
    th.start()
    for _ in range(200):
        P.tensile_eval_plans(h, dp, None, peak, arg, None, stream=s)
    th.join()
    s.synchronize()
    assert np.array_equal(peak.cpu().numpy(), p0) and np.array_equal(arg.cpu().numpy(), a0)
    for f in ("iv_tensor", "iv_out", "iv_in", "iv_kind", "peak_trace"):
        assert np.array_equal(out["g"][f], og[f]), f
    h.close()

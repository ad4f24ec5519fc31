"""Calls at the limits of what the library asks of the device: memory that cannot be had, batches of millions of plans,
very long sequences, streams that are being captured.  Compared with the CPU oracle, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2105_13336_amd as P  # noqa: E402
from oracle import oracle as O  # noqa: E402
from test_gpu_parity import (check_eval, check_link, check_step, gpu_eval, gpu_score, gpu_score_recompute, gpu_step,  # noqa: E402
                             same_greedy, say, upload)  # noqa: E402
from workloads import make_plans, plans_from_lists, prng, small_random_tas, tas_from_lists  # noqa: E402


@pytest.mark.parametrize("T,B", [(6000, 300), (20011, 600)])
def test_eval_score_without_memory_for_the_block_maxima(T, B, tuning):
    """The call needs scratch only for what the evaluation hands to the scoring; without it the scoring reads the rows,
    and the refused allocation is not reported by this or a later call."""
    tas = small_random_tas(9000 + T, N=200, T=T, max_acc=5, timed=True, link_bytes_per_us=400_000)
    pl = make_plans(tas, B, 3, p_swap=0.4)
    say(f"eval+score without scratch T={T} B={B}")
    h = P.tas_load(tas)
    gpu_eval(h, upload(pl))                    # (what the evaluation itself needs is there)
    tuning("alloc_fail", 1)
    assert check_step(tas, pl, h=h, label="refused") > 0
    assert check_step(tas, pl, h=h, label="granted") > 0
    # a larger batch asks for twice what is there; that refused, for what it needs
    tuning("alloc_fail", 1)
    assert check_step(tas, make_plans(tas, B + B // 2, 4, p_swap=0.4), h=h, label="grown") > 0
    h.close()


def test_a_refused_allocation_is_reported_once(tuning):
    tas = small_random_tas(9001, N=60, T=20011, max_acc=4)
    pl = make_plans(tas, 3, 5, p_swap=0.5)     # few plans: several segments each, whose partial results need scratch
    say("refused allocation in eval_plans")
    h = P.tas_load(tas)
    tuning("eval_segments", 3)
    s = torch.cuda.Stream()
    peak, arg = torch.empty(3, dtype=torch.int64, device="cuda"), torch.empty(3, dtype=torch.int32, device="cuda")
    dp = upload(pl)
    tuning("alloc_fail", 1)
    with pytest.raises(P.TensileError) as e:
        P.tensile_eval_plans(h, dp, None, peak, arg, None, stream=s)
    assert e.value.code == P.binding.TENSILE_E_NOMEM
    P.tensile_eval_plans(h, dp, None, peak, arg, None, stream=s)
    s.synchronize()
    _, p0, a0, _ = gpu_eval(h, dp)
    assert np.array_equal(peak.cpu().numpy(), p0.cpu().numpy()) and np.array_equal(arg.cpu().numpy(), a0.cpu().numpy())
    h.close()


def test_scores_of_eight_million_plans():
    """More plans than a launch of one workgroup each has room for (2^32 threads): sixteen plans, over and over."""
    tas = small_random_tas(9002, N=4, T=12, max_acc=3, timed=True, link_bytes_per_us=400_000)
    pl = make_plans(tas, 16, 7, p_swap=0.5)
    times = (1 << 19) + 1
    r0, p0, a0, m0 = O.eval_plans(tas, pl)
    want = [np.stack(x) for x in zip(O.score_plans(tas, pl, r0, p0, a0), O.score_recompute_plans(tas, pl, r0, p0, a0))]
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    lens = up(np.diff(pl.plan_offsets)).repeat(times)
    dp = P.DevicePlans(torch.cat([lens.new_zeros(1), torch.cumsum(lens, 0)]), *(up(x).repeat(times) for x in (pl.iv_tensor, pl.iv_out, pl.iv_in, pl.iv_kind)))
    say(f"scores of {dp.B} plans, {dp.n_intervals} intervals")
    assert dp.B * 512 >= 1 << 32
    same = lambda got, one: bool((got.view(times, *one.shape) == up(one)).all())
    h = P.tas_load(tas)
    res, peak, arg, mn, *step = gpu_step(h, dp)
    assert same(res, r0) and same(peak, p0) and same(arg, a0) and same(mn, m0)
    for k, got in enumerate((gpu_score(h, dp, res, peak, arg), gpu_score_recompute(h, dp, res, peak, arg), step)):
        for g, w in zip(got, want):
            assert same(g, w[k % 2]), f"call {k}"
    h.close()


@pytest.mark.parametrize("first", ["the two calls", "the one call"])
def test_eval_score_in_a_captured_stream(first):
    """The call enqueues without allocating in a stream that is being captured: after earlier calls of the two parts (the
    scoring then reads the rows) and after one of its own.  Several replays on other plans, eager calls in between."""
    tas = small_random_tas(9003, N=150, T=5003, max_acc=5, timed=True, link_bytes_per_us=400_000)
    B = 40
    batches = [make_plans(tas, B, 20 + k, p_swap=0.5) for k in range(4)]
    K = max(pl.n_intervals for pl in batches)
    say(f"captured eval+score, warmed by {first}")
    h = P.tas_load(tas)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        offs = torch.zeros(B + 1, dtype=torch.int64, device="cuda")
        t, o, r = (torch.zeros(K, dtype=torch.int32, device="cuda") for _ in range(3))
        dp = P.DevicePlans(offs, t, o, r, None)

        def put(pl):
            for dst, src in ((offs, pl.plan_offsets), (t, pl.iv_tensor), (o, pl.iv_out), (r, pl.iv_in)):
                dst[:len(src)].copy_(torch.from_numpy(src))

        def outputs():
            return [torch.full(shape, -3, dtype=dt, device="cuda") for shape, dt in
                    (((B, tas.T), torch.int64), ((B,), torch.int64), ((B,), torch.int32), ((B,), torch.int64),
                     ((B, tas.N), torch.int64), ((B, tas.N), torch.int32), ((B, tas.N), torch.int32))]

        def check(out, pl):
            r0, p0, a0, m0 = O.eval_plans(tas, pl)
            s.synchronize()
            for k, (g, w) in enumerate(zip(out, (r0, p0, a0, m0, *O.score_plans(tas, pl, r0, p0, a0)))):
                assert np.array_equal(g.cpu().numpy(), w), f"output {k}"

        out, eager = outputs(), outputs()
        put(batches[0])
        if first == "the one call":
            P.tensile_eval_score_plans(h, dp, *eager, stream=s)
        else:
            P.tensile_eval_plans(h, dp, *eager[:4], stream=s)
            P.tensile_score_candidates(h, dp, *eager[:3], *eager[4:], stream=s)
        check(eager, batches[0])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        P.tensile_eval_score_plans(h, dp, *out, stream=s)
    with torch.cuda.stream(s):
        for pl in batches + batches[:1]:
            put(pl)
            for x in out:
                x.fill_(-5)
            graph.replay()
            check(out, pl)
            P.tensile_eval_score_plans(h, dp, *eager, stream=s)
            check(eager, pl)
    del graph
    h.close()


def test_an_update_of_the_latencies_that_fails_half_way(tuning):
    """Whichever allocation of the update is refused: what depends on the latencies is refused until an update succeeds,
    the rest works, and a later update leaves nothing of the failure behind."""
    import copy
    tas = small_random_tas(9004, N=200, T=9001, max_acc=5, timed=True, link_bytes_per_us=400_000)
    before = copy.copy(tas)
    before.step_ns, before.link_bytes_per_us = None, 0
    pl = make_plans(tas, 5, 9, p_swap=0.5)
    dp = upload(pl)
    r0, p0, a0, _ = O.eval_plans(tas, pl)
    failed = 0
    for n in range(1, 40):
        h = P.tas_load(before)                 # (no latencies: the tables that need them have never been allocated)
        res, peak, arg, mn = gpu_eval(h, dp)
        s0 = gpu_score_recompute(h, dp, res, peak, arg)
        tuning("alloc_fail", n)
        try:
            P.tensile_tas_update_latencies(h, tas.step_ns, tas.link_bytes_per_us)
        except P.TensileError as e:
            assert e.code == P.binding.TENSILE_E_NOMEM
            failed += 1
        else:
            tuning("alloc_fail", 0)
            h.close()
            break
        say(f"update of the latencies, allocation {n} refused")
        pk = torch.empty(pl.B, dtype=torch.int32, device="cuda")
        for call in (lambda: gpu_score(h, dp, res, peak, arg), lambda: gpu_step(h, dp), lambda: P.tensile_eval_link(h, dp, pk, None),
                     lambda: P.tensile_greedy_plan(h, 0, max_iters=5, capacity=8)):
            with pytest.raises(P.TensileError) as e:
                call()
            assert e.value.code == P.binding.TENSILE_E_INVAL and "update" in str(e.value)
        with pytest.raises(P.TensileError):    # (refused before anything is touched: changes nothing about it)
            P.tensile_tas_update_latencies(h, tas.step_ns, 0)
        check_eval(tas, pl, h=h, label="after a failed update")
        for g, w in zip(gpu_score_recompute(h, dp, res, peak, arg), s0):
            assert torch.equal(g, w)
        P.tensile_tas_update_latencies(h, tas.step_ns, tas.link_bytes_per_us)
        for g, w in zip(gpu_score(h, dp, res, peak, arg), O.score_plans(tas, pl, r0, p0, a0)):
            assert np.array_equal(g.cpu().numpy(), w)
        check_step(tas, pl, h=h)
        check_link(tas, pl, False, h=h)
        same_greedy(P.tensile_greedy_plan(h, 0, max_iters=20, capacity=32), O.greedy(tas, 0, max_iters=20))
        h.close()
    assert failed >= 4


def test_a_sequence_of_more_than_a_thousand_million_steps():
    """So many steps that the candidate index could have more buckets than a launch takes workgroups of its kernels."""
    T = (1 << 30) + 5
    say(f"T={T}")
    #          present          used at            (the gap of tensor 0 around the peak is the one candidate)
    tas = tas_from_lists(T, [10, 7, 3], [0, 500, T - 9], [[9, 1000], [501], [T - 2]])
    h = P.tas_load(tas)
    assert P.tensile_tas_info(h) == (17, 500)
    g = P.tensile_greedy_plan(h, 0, max_iters=3, capacity=4)
    assert [x.tolist() for x in (g["iv_tensor"], g["iv_out"], g["iv_in"])] == [[0], [9], [1000]]
    assert g["peak_trace"].tolist() == [17, 10] and g["final_peak"] == 10
    h.close()


def test_link_scratch_of_very_long_rows():
    """Plans of several passes without rows, more of them than CUs, on rows so long that a scratch row per workgroup is
    kept to one workgroup per CU."""
    T, B = 2_200_001, 530
    tas = small_random_tas(9005, N=60, T=T, max_acc=40, timed=True, link_bytes_per_us=400_000)
    few = make_plans(tas, 3, 11, p_swap=0.9)
    lists = []
    for b, n in ((0, 6150), (1, 12_300), (2, 40)):
        t, o, r, k = few.plan(b)
        one = [(int(t[j]), int(o[j]), int(r[j]), int(k[j])) for j in range(len(t))]
        lists.append((one * (n // len(one) + 1))[:n])
    pl = plans_from_lists(lists)
    _, p0, a0, o0 = O.link_occupancy(tas, pl, reuse=True)
    which = np.arange(B) % 3
    which[3:-3] = 2                            # (the long ones first and last: most plans are short)
    pl = pl.select(which)
    say(f"link scratch T={T} B={B} K={pl.n_intervals}")
    h = P.tas_load(tas)
    dp = upload(pl)
    out = [torch.full((B,), -7, dtype=torch.int32, device="cuda") for _ in range(3)]
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    P.tensile_eval_link(h, dp, out[0], None, out[1], out[2], reuse_host_copies=True)
    torch.cuda.synchronize()
    taken = before - torch.cuda.mem_get_info()[0]
    for g, w in zip(out, (p0, a0, o0)):
        assert np.array_equal(g.cpu().numpy(), w[which])
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert taken <= 1.1 * cus * 4 * (T + tas.N), f"{taken} bytes of scratch"
    h.close()


@pytest.mark.parametrize("T,N,B", [(1, 1, 3), (256, 65, 5), (4096, 512, 4), (4097, 512, 4), (4096, 513, 4), (6001, 129, 256), (6001, 2049, 257), (33_334, 4500, 7), (140_001, 40_000, 3),
                                   (140_002, 70_000, 2), (100_000, 900, 255)])   # (the last: 204 MB of rows)
def test_scores_by_large_and_small_workgroups(T, N, B, tuning):
    """Batches of as many plans as CUs take the large workgroups, one more or little work per plan the small ones: both, forced and
    chosen, over tensors that leave wavefronts without any, that share filter bits (more than 32,768 of them) and rows read past the L2."""
    i = np.arange(N)
    alloc = prng.randint(89, 1, i, 0, max(0, 2 * T // 3 - 2))
    used = np.minimum(T - 1, alloc + 1 + prng.randint(89, 2, i, 0, T // 3))
    sizes = prng.randint(89, 3, i, 1, 1 << 20)
    tas = tas_from_lists(T, sizes.tolist(), alloc.tolist(), [[int(u)] if u > x else [] for x, u in zip(alloc, used)], None,
                         prng.randint(89, 4, np.arange(T), 1, 1000).astype(np.int64), 0, 4_000_000)
    pl = make_plans(tas, min(B, 7), 13, p_swap=0.4)
    which = np.arange(B) % pl.B
    r0, p0, a0, _ = O.eval_plans(tas, pl)
    want = [O.score_plans(tas, pl, r0, p0, a0), O.score_recompute_plans(tas, pl, r0, p0, a0)]
    dp = upload(pl.select(which))
    h = P.tas_load(tas)
    for wide in (0, 1, -1):
        say(f"scores T={T} N={N} B={B} wide={wide}")
        tuning("score_wide", wide)
        res, peak, arg, mn, *step = gpu_step(h, dp)
        for g, w in zip((res, peak, arg), (r0, p0, a0)):
            assert np.array_equal(g[:pl.B].cpu().numpy(), w)
        for k, got in enumerate((gpu_score(h, dp, res, peak, arg), gpu_score_recompute(h, dp, res, peak, arg), step)):
            for g, w in zip(got, want[k % 2]):
                assert bool((g == torch.from_numpy(w).cuda()[which]).all()), f"call {k}, wide={wide}"
    h.close()

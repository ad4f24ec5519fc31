"""Calls at the limits of what the library asks of the device: memory that cannot be had, batches of millions of plans,
very long sequences, streams that are being captured.  Compared with the CPU oracle, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2105_13336_amd as P  # noqa: E402
from test_gpu_parity import check_step, gpu_eval, say, upload  # noqa: E402
from workloads import make_plans, small_random_tas  # noqa: E402


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

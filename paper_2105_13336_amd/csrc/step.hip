// Peak analysis and candidate scores of a batch in one call (the body of the paper's Alg. 3 loop: the memory
// peak analysis of Alg. 1 immediately followed by the choice among the tensors resident at the peak, section
// IV-C): the evaluation kernel and the scoring kernel enqueued back to back.  The evaluation also writes the maximum of
// every 256 steps of its rows, which is nearly all that scoring wants to know of them (score.hip): where the scoring call
// by itself reads every row once, here it reads a 256th of that and the one to three blocks around each plan's peak.
#include "common.h"

namespace tensile {

namespace {

// Whether a capture is under way that an allocation would break.  (A question about the default stream is refused while
// another stream's capture rules out work on it: a capture too.)
bool capturing(hipStream_t stream) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    const hipError_t e = hipStreamIsCapturing(stream, &status);
    if (e != hipSuccess) (void)hipGetLastError();
    return e != hipSuccess || status != hipStreamCaptureStatusNone;
}

}  // namespace

int launch_step(const tensile_tas *tas, Workspace &ws, const tensile_plans *plans, int64_t *resident, int64_t *peak,
                int32_t *argmax, int64_t *min_resident, int64_t *score, int32_t *win_out, int32_t *win_in) {
    EvalArgs ea{};
    ea.T = tas->T; ea.N = tas->N; ea.B = plans->B; ea.o_min = 0; ea.n_intervals = plans->n_intervals;
    ea.plan_offsets = plans->plan_offsets;
    ea.iv_tensor = plans->iv_tensor; ea.iv_out = plans->iv_out; ea.iv_in = plans->iv_in;
    ea.size = tas->d_size.p; ea.size_units = tas->d_size_units.p; ea.size_shift = tas->size_shift;
    ea.MF0 = tas->d_MF0.p; ea.dMF0 = tas->d_dMF0.p; ea.resident = resident;
    // The maxima of the rows' pieces: 1/256 of the rows' bytes.  Without the memory for them scoring reads the rows; so it does
    // while the stream is being captured, unless an earlier call has left enough (an allocation would end the capture, and
    // the call has no other need of one), and on request (tuning knob step_fused: 0).
    const size_t n_max = static_cast<size_t>(plans->B) * ((static_cast<size_t>(tas->T) + kScoreMini - 1) / kScoreMini);
    const bool there = ws.blk_max.p && n_max <= ws.blk_max.n;
    if (tas->N > 0 && g_tuning.step_fused != 0 && (there || !capturing(ws.stream)) &&
        ws.provide(ws.blk_max, n_max, "eval_score_plans: maxima of the rows' pieces") == TENSILE_OK)
        ea.blk_max = ws.blk_max.p;
    const int rc = launch_eval(tas, ws, ea, peak, argmax, min_resident);
    if (rc != TENSILE_OK) return rc;
    return launch_score(tas, ws, tas->index, false, plans, resident, peak, argmax, score, win_out, win_in, ea.blk_max);
}

}  // namespace tensile

using namespace tensile;

extern "C" int tensile_eval_score_plans(const tensile_tas *tas, const tensile_plans *plans, int64_t *resident, int64_t *peak,
                                        int32_t *argmax, int64_t *min_resident, int64_t *score, int32_t *win_out,
                                        int32_t *win_in, void *hip_stream) {
    int rc = check_plans(tas, plans, "eval_score_plans");
    if (rc != TENSILE_OK) return rc;
    if (plans->B == 0) return TENSILE_OK;
    if (!resident || !peak || !argmax || !score) {
        set_error("eval_score_plans: resident, peak, argmax and score are required");
        return TENSILE_E_INVAL;
    }
    rc = check_times(tas, "eval_score_plans");
    if (rc != TENSILE_OK) return rc;
    WorkspaceLock ws = acquire_workspace(tas, static_cast<hipStream_t>(hip_stream));
    return launch_step(tas, *ws, plans, resident, peak, argmax, min_resident, score, win_out, win_in);
}

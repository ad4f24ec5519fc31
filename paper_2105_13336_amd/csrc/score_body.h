// Candidate scoring of one plan (section IV-C of the paper) from block maxima of its footprint row: the device
// functions that the batch kernel and the planner's kernel (both in score.hip) share.  Everything here has internal
// linkage.
#pragma once

#include "common.h"
#include "wave_ops.h"

namespace tensile {

namespace {

constexpr int kMini = kScoreMini;    // steps of a piece: 4 consecutive steps per lane of a wavefront
constexpr int kFilterWords = kScoreFilterWords;
constexpr int kIvU = 4;              // intervals per thread and round of the cancelling pass
constexpr int kWindow = 8192;       // entries of a bucket whose flags are in LDS at a time
constexpr int kStage = kScoreStage;  // tensors whose output one wavefront composes in LDS at a time

typedef long long ll2 __attribute__((ext_vector_type(2)));
typedef int i4 __attribute__((ext_vector_type(4)));

struct ScoreArgs {
    int32_t T, N, B;
    int32_t tspan;               // (batch kernel) tensors per wavefront, a multiple of kScoreStage
    int32_t n_mini;              // pieces of kMini steps: ceil(T / kMini)
    int32_t piece_shift;         // a block of the LDS tables is 2^piece_shift pieces, so that they hold all of ...
    int32_t n_blk;               // ... the n_blk = ceil(n_mini / 2^piece_shift) blocks
    int32_t any_interval;        // an interval of the entry's tensor cancels it wherever it lies
    int64_t n_intervals;
    const int64_t *plan_offsets;
    const int32_t *iv_tensor, *iv_out, *iv_in;
    int32_t bucket_shift, filter_shift, filter_words;
    const int32_t *bucket_off;   // the candidate index, see CandIndex
    const int4 *cand;
    const int32_t *cand_gap;
    const int64_t *cand_size;
    const uint32_t *filter;
    const int32_t *filter_base;
    const int64_t *resident;
    const int64_t *blk_max;      // [B][n_mini] maxima of the rows' pieces, or null: they are taken from the rows
    const int64_t *peak;
    const int32_t *argmax;
    int64_t *score;
    int32_t *win_out, *win_in;
};

// row[0..n) = v with 16-byte stores where the row allows them
template <int kThr, typename E>
__device__ __forceinline__ void fill_row(E *row, int32_t n, E v, int tid) {
    constexpr int kPer = 16 / sizeof(E);
    typedef E vec_t __attribute__((ext_vector_type(kPer)));
    const uintptr_t addr = reinterpret_cast<uintptr_t>(row);
    int32_t head = static_cast<int32_t>(((16 - (addr & 15)) & 15) / sizeof(E));
    if (head > n) head = n;
    if (tid < head) row[tid] = v;
    const int32_t n_vec = (n - head) / kPer;
    vec_t *dst = reinterpret_cast<vec_t *>(row + head);
    vec_t vv;
#pragma unroll
    for (int j = 0; j < kPer; ++j) vv[j] = v;
    for (int32_t k = tid; k < n_vec; k += kThr) dst[k] = vv;
    const int32_t done = head + n_vec * kPer;
    if (done + tid < n) row[done + tid] = v;
}

// Four consecutive steps of the row starting at step t (a multiple of 4; two 16-byte loads when
// the row allows them).  The loads are always issued, at clamped addresses; steps outside
// [0, T) come back as INT64_MIN.
template <bool kVec>
__device__ __forceinline__ void load_quad(const int64_t *MF, int32_t t, int32_t T, int64_t (&x)[4]) {
    if (kVec) {   // T is even here, so an even step t' < T implies t' + 1 < T
        const ll2 lo = *reinterpret_cast<const ll2 *>(MF + (t < T ? t : T - 2));
        const ll2 hi = *reinterpret_cast<const ll2 *>(MF + (t + 2 < T ? t + 2 : T - 2));
        x[0] = lo[0]; x[1] = lo[1]; x[2] = hi[0]; x[3] = hi[1];
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = MF[t + j < T ? t + j : T - 1];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (t + j >= T) x[j] = INT64_MIN;
}

// Inclusive max-scan over the 64 lanes from the high end: lane l receives the maximum of lanes
// l .. 63.  Shifts towards lower lanes inside rows of 16, then the totals of the later rows.
__device__ __forceinline__ int64_t wave_rscan_max(int64_t x, int lane) {
    x = max64(x, dpp_move<0x101, 0xf>(x, INT64_MIN));
    x = max64(x, dpp_move<0x102, 0xf>(x, INT64_MIN));
    x = max64(x, dpp_move<0x104, 0xf>(x, INT64_MIN));
    x = max64(x, dpp_move<0x108, 0xf>(x, INT64_MIN));
    const int64_t r3 = lane_value(x, 48);
    const int64_t r2 = max64(lane_value(x, 32), r3);
    const int64_t r1 = max64(lane_value(x, 16), r2);
    const int64_t later = lane < 16 ? r1 : (lane < 32 ? r2 : (lane < 48 ? r3 : INT64_MIN));
    return max64(x, later);
}

// The maximum over the 64 lanes, in every lane.  Where the lanes' values share their upper halves, as footprints of
// neighbouring steps nearly always do, the lower halves decide: one instruction per step instead of five.
__device__ __forceinline__ int64_t wave_max(int64_t x) {
    const int32_t hi = static_cast<int32_t>(x >> 32);
    if (__builtin_amdgcn_ballot_w64(hi != __builtin_amdgcn_readfirstlane(hi)) == 0) {   // (wave-uniform)
        uint32_t lo = static_cast<uint32_t>(x);
        auto step = [&](uint32_t y) { lo = y > lo ? y : lo; };
        step(__builtin_amdgcn_update_dpp(0, static_cast<int>(lo), 0x111, 0xf, 0xf, true));
        step(__builtin_amdgcn_update_dpp(0, static_cast<int>(lo), 0x112, 0xf, 0xf, true));
        step(__builtin_amdgcn_update_dpp(0, static_cast<int>(lo), 0x114, 0xf, 0xf, true));
        step(__builtin_amdgcn_update_dpp(0, static_cast<int>(lo), 0x118, 0xf, 0xf, true));
        step(__builtin_amdgcn_update_dpp(0, static_cast<int>(lo), 0x142, 0xa, 0xf, true));
        step(__builtin_amdgcn_update_dpp(0, static_cast<int>(lo), 0x143, 0xc, 0xf, true));
        const uint32_t m = __builtin_amdgcn_readlane(static_cast<int>(lo), 63);
        return static_cast<int64_t>((static_cast<uint64_t>(static_cast<uint32_t>(hi)) << 32) | m);
    }
    return last_lane(wave_scan_max(x));
}

// A 16-byte piece of an output row.  Where the rows are read past the L2's allocation (kStream) the store is
// nontemporal too: the lines are not read again by this kernel, and left out of the L2 they leave it to the
// candidate index.
template <bool kStream, typename V>
__device__ __forceinline__ void store_out(V *at, const V v) {
    if constexpr (kStream) __builtin_nontemporal_store(v, at);
    else *at = v;
}

// value of the previous / next lane; the first / last lane receives `edge`
__device__ __forceinline__ int64_t from_prev_lane(int64_t x, int64_t edge) { return dpp_move<0x138, 0xf>(x, edge); }   // wave_shr:1
__device__ __forceinline__ int64_t from_next_lane(int64_t x, int64_t edge) { return dpp_move<0x130, 0xf>(x, edge); }   // wave_shl:1

// A load whose address is the same in every lane, from memory that no kernel writes during this
// launch: through the constant address space it goes to the scalar unit and its result lives in
// scalar registers (as a vector load it would hold one register per lane for as long as the value lives).
template <typename T>
__device__ __forceinline__ T uniform_load(const T *p, int64_t i) {
    typedef const T __attribute__((address_space(4))) *const_ptr;
    return ((const_ptr)p)[i];
}

// Phase timing for tuning, compiled in with -DTENSILE_SCORE_PROF only: thread 0 of every
// workgroup adds the 100 MHz ticks it spent in each phase to g_score_prof.
#ifdef TENSILE_SCORE_PROF
__device__ unsigned long long g_score_prof[16];
#define PROF_START unsigned long long prof_t = wall_clock64()
#define PROF_MARK(k)                                              \
    do {                                                          \
        if (threadIdx.x == 0) {                                   \
            const unsigned long long now_ = wall_clock64();       \
            atomicAdd(&g_score_prof[k], now_ - prof_t);           \
            prof_t = now_;                                        \
        }                                                         \
    } while (0)
#else
#define PROF_START do { } while (0)
#define PROF_MARK(k) do { } while (0)
#endif

// ---- prefix and suffix maxima of the row's blocks -----------------------------------------------------------
// pm[k] = max of the blocks before k, sm[k] = max of the blocks k .. (both -inf where there is none)
template <int kTab>
struct BlockMaxima {
    int64_t pm[kTab + 1], sm[kTab + 1];
};

// From the blocks' maxima themselves, which the caller has put into pm[k + 1] and sm[k] (a barrier ago): wavefront 0
// scans the one array, wavefront 1 the other, in place.  The caller's next barrier ends it.
template <int kTab>
__device__ __forceinline__ void scan_block_maxima(BlockMaxima<kTab> &m, int32_t n_blk, int wave, int lane) {
    if (wave == 0) {
        int64_t run = INT64_MIN;
        if (lane == 0) m.pm[0] = INT64_MIN;
        for (int32_t k0 = 0; k0 < n_blk; k0 += 64) {
            const int32_t k = k0 + lane;
            const int64_t incl = max64(wave_scan_max(k < n_blk ? m.pm[k + 1] : INT64_MIN), run);
            if (k < n_blk) m.pm[k + 1] = incl;
            run = last_lane(incl);
        }
    } else if (wave == 1) {
        int64_t run = INT64_MIN;
        if (lane == 0) m.sm[n_blk] = INT64_MIN;
        for (int32_t top = n_blk; top > 0; top -= 64) {
            const int32_t k = top - 1 - lane;
            const int64_t incl = max64(wave_scan_max(k >= 0 ? m.sm[k] : INT64_MIN), run);
            if (k >= 0) m.sm[k] = incl;
            run = last_lane(incl);
        }
    }
}

// ---- candidates the block maxima leave open ------------------------------------------------------------------
// For an entry (o, q, size) of the bucket with o < t* < q,
//   score = P - max( max MF[0..o], max MF[q..T), P - size ).
// With bo, bq the blocks of o and q, the maximum is at least lo = max( pm[bo], sm[bq + 1], P - size ) and at most
// what it becomes when the whole of the blocks bo and bq counts.  Where the two agree - on the sequences of training
// jobs for 85 to 95 of 100 candidates, because a block far from the peak lies further below it than most tensors are
// large - the row itself is not looked at.  The others are listed with the sides that matter, and the few blocks they
// lie in (one to three of a row, those around the peak) are read.
template <int kUn>
struct OpenList {
    int64_t acc[kUn];            // lo, raised to the true maximum by resolve_open
    int2 oq[kUn];                // o, q; -1 for a side that cannot matter
    int32_t n;
};

struct Classified {
    int64_t lo;
    bool open_o, open_q;
};
template <int kTab>
__device__ __forceinline__ Classified classify(const BlockMaxima<kTab> &m, int block_shift, int2 oq, int64_t without) {
    const int32_t bo = oq.x >> block_shift, bq = oq.y >> block_shift;
    Classified c;
    c.lo = max64(max64(m.pm[bo], m.sm[bq + 1]), without);
    c.open_o = m.pm[bo + 1] > c.lo;
    c.open_q = m.sm[bq] > c.lo;
    return c;
}

// One piece of a row in a wavefront's LDS buffer: its values, per lane (4 steps) the maximum of everything in the block
// before them and after them.
struct SpanBuf {
    int64_t raw[kMini];
    int64_t before[64], after[64];
};

// Raises acc of every listed entry with a side in one of the blocks marked in `need` (one bit per block).  The blocks
// are dealt to the first kBufs wavefronts.
template <bool kVec, int kBufs, int kUn>
__device__ __forceinline__ void resolve_open(const ScoreArgs &a, const int64_t *MF, const uint32_t *need, OpenList<kUn> &open,
                                             const int32_t n_open, SpanBuf *bufs, int wave, int lane) {
    if (wave >= kBufs) return;
    SpanBuf *const buf = bufs + wave;
    const int ps = a.piece_shift;
    static_assert(kMini == 256, "the shifts by 8");
    int ord = 0;
    for (int32_t w = 0; w * 32 < a.n_blk; ++w) {
        uint32_t bits = __builtin_amdgcn_readfirstlane(need[w]);
        while (bits) {   // (wave-uniform)
            const int32_t blk = w * 32 + __builtin_ctz(bits);
            bits &= bits - 1;
            if (ord++ % kBufs != wave) continue;
            const int32_t p0 = blk << ps, p1 = min(p0 + (1 << ps), a.n_mini);
            // forward over the block's pieces for the o sides, then backward for the q sides (one piece: both at once)
            int64_t carry = INT64_MIN;
            for (int pass = 0; pass < 2; ++pass) {
                if (pass == 1 && ps == 0) break;
                carry = INT64_MIN;
                for (int32_t i = 0; i < p1 - p0; ++i) {
                    const int32_t piece = pass == 0 ? p0 + i : p1 - 1 - i;
                    const int32_t t0 = piece * kMini;
                    int64_t x[4];
                    load_quad<kVec>(MF, t0 + 4 * lane, a.T, x);
                    const int64_t m = max64(max64(x[0], x[1]), max64(x[2], x[3]));
                    const int64_t fwd = wave_scan_max(m), bwd = wave_rscan_max(m, lane);
                    const int64_t edge_b = pass == 0 ? carry : INT64_MIN, edge_a = pass == 1 ? carry : INT64_MIN;
                    // (the lanes of a wavefront execute in step and LDS serves a wavefront's accesses in
                    // order, so the buffer needs no barrier: the fences only pin the compiler's order)
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    reinterpret_cast<ll2 *>(buf->raw)[2 * lane] = ll2{x[0], x[1]};
                    reinterpret_cast<ll2 *>(buf->raw)[2 * lane + 1] = ll2{x[2], x[3]};
                    buf->before[lane] = max64(from_prev_lane(fwd, INT64_MIN), edge_b);
                    buf->after[lane] = max64(from_next_lane(bwd, INT64_MIN), edge_a);
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    carry = max64(carry, last_lane(fwd));
                    for (int32_t k = lane; k < n_open; k += 64) {
                        const int2 oq = open.oq[k];
                        if (pass == 0 && (oq.x >> 8) == piece) {      // (a side that does not matter is -1: no piece)
                            const int32_t r = oq.x - t0, l = r >> 2, j = r & 3;
                            int64_t v = max64(buf->before[l], buf->raw[4 * l]);
                            if (j >= 1) v = max64(v, buf->raw[4 * l + 1]);
                            if (j >= 2) v = max64(v, buf->raw[4 * l + 2]);
                            if (j >= 3) v = max64(v, buf->raw[4 * l + 3]);
                            atomicMax(reinterpret_cast<long long *>(open.acc + k), static_cast<long long>(v));
                        }
                        if ((pass == 1 || ps == 0) && (oq.y >> 8) == piece) {
                            const int32_t r = oq.y - t0, l = r >> 2, j = r & 3;
                            int64_t v = max64(buf->after[l], buf->raw[4 * l + 3]);
                            if (j <= 2) v = max64(v, buf->raw[4 * l + 2]);
                            if (j <= 1) v = max64(v, buf->raw[4 * l + 1]);
                            if (j <= 0) v = max64(v, buf->raw[4 * l]);
                            atomicMax(reinterpret_cast<long long *>(open.acc + k), static_cast<long long>(v));
                        }
                    }
                    __builtin_amdgcn_wave_barrier();
                }
            }
        }
    }
}

// ---- the plan's own intervals cancel candidates ---------------------------------------------------------------
// Sets the bit of every entry w_lo .. w_lo + w_n - 1 of the bucket that one of the intervals k0 .. k1-1 cancels: an
// interval inside the gap of an entry of its tensor (any interval of that tensor when a.any_interval).  filter, base: the
// bucket's filter bits over tensors and, per word of them, the first entry of its tensors, both in LDS.  Most intervals
// end at the filter.  For the others the tensor's first entry lies at or after the word's first entry plus the number of
// filter bits set below the tensor's - exactly there as long as none of the word's earlier tensors has several entries,
// else it is searched for.  (A caller's list keeps its intervals in tensor order, and so are the entries: the lanes
// of a wavefront read neighbouring ones.  The hash table this replaced scattered them over four times the lines.)
template <int kThr>
__device__ __forceinline__ void cancel_by_plan(const ScoreArgs &a, const int64_t k0, const int64_t k1, const int4 *entries,
                                               const int32_t n_e, const int32_t w_lo, const int32_t w_n, const uint32_t *filter,
                                               const int32_t *base, uint32_t *cancelled, const int tid) {
    auto cancel = [&](int32_t e) {
        const uint32_t el = static_cast<uint32_t>(e - w_lo);
        if (el < static_cast<uint32_t>(w_n)) atomicOr(&cancelled[el >> 5], 1u << (el & 31));
    };
    for (int64_t kb = k0 + tid; kb < k1; kb += kIvU * kThr) {
        int32_t i[kIvU], o[kIvU], r[kIvU], e[kIvU];
        int4 c[kIvU];
        bool go[kIvU];
#pragma unroll
        for (int u = 0; u < kIvU; ++u) {
            const int64_t k = kb + u * kThr;
            const int64_t kc = k < k1 ? k : k1 - 1;
            i[u] = a.iv_tensor[kc];
            o[u] = a.iv_out[kc];
            r[u] = a.iv_in[kc];
            if (k >= k1) i[u] = -1;
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kIvU; ++u) {
            go[u] = static_cast<uint32_t>(i[u]) < static_cast<uint32_t>(a.N) && o[u] >= 0 && r[u] <= a.T && r[u] > o[u];
            const uint32_t bit = go[u] ? static_cast<uint32_t>(i[u]) >> a.filter_shift : 0u;
            const uint32_t word = filter[bit >> 5];
            go[u] = go[u] && ((word >> (bit & 31)) & 1u);
            e[u] = go[u] ? base[bit >> 5] + __builtin_popcount(word & ((1u << (bit & 31)) - 1)) : 0;
            c[u] = entries[e[u]];                  // (a set bit has an entry: e is one of the word's)
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kIvU; ++u) {
            if (!go[u]) continue;
            if (c[u].x < i[u]) {                   // the first entry of tensor i[u] or a later one, behind e
                int32_t lo = e[u] + 1, hi = base[((static_cast<uint32_t>(i[u]) >> a.filter_shift) >> 5) + 1];
                while (lo < hi) {
                    const int32_t mid = (lo + hi) >> 1;
                    if (entries[mid].x < i[u]) lo = mid + 1;
                    else hi = mid;
                }
                e[u] = lo;
                if (lo < n_e) c[u] = entries[lo];
                else continue;
            }
            while (c[u].x == i[u]) {
                if (a.any_interval || (c[u].y <= o[u] && r[u] <= c[u].z)) cancel(e[u]);
                if (++e[u] >= n_e) break;
                c[u] = entries[e[u]];
            }
        }
    }
}

// (host) the arguments of a scoring pass
inline ScoreArgs make_score_args(const tensile_tas *tas, const CandIndex &ix, bool any_interval, const tensile_plans *plans,
                                 int max_blocks, const int64_t *resident, const int64_t *peak, const int32_t *argmax,
                                 int64_t *score, int32_t *win_out, int32_t *win_in) {
    ScoreArgs a{};
    a.T = tas->T; a.N = tas->N; a.B = plans->B;
    a.n_mini = static_cast<int32_t>((static_cast<int64_t>(tas->T) + kMini - 1) / kMini);
    a.piece_shift = 0;
    while (((static_cast<int64_t>(a.n_mini) + (1 << a.piece_shift) - 1) >> a.piece_shift) > max_blocks) ++a.piece_shift;
    a.n_blk = static_cast<int32_t>((static_cast<int64_t>(a.n_mini) + (1 << a.piece_shift) - 1) >> a.piece_shift);
    a.any_interval = any_interval ? 1 : 0;
    a.n_intervals = plans->n_intervals;
    a.plan_offsets = plans->plan_offsets;
    a.iv_tensor = plans->iv_tensor; a.iv_out = plans->iv_out; a.iv_in = plans->iv_in;
    a.bucket_shift = ix.shift; a.filter_shift = ix.filter_shift; a.filter_words = ix.filter_words;
    a.bucket_off = ix.bucket_off.p;
    a.cand = ix.cand.p; a.cand_gap = ix.cand_gap.p; a.cand_size = ix.cand_size.p;
    a.filter = ix.filter.p; a.filter_base = ix.filter_base.p;
    a.resident = resident; a.peak = peak; a.argmax = argmax;
    a.score = score; a.win_out = win_out; a.win_in = win_in;
    return a;
}

}  // namespace

}  // namespace tensile

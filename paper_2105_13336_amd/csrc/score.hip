// Candidate scoring (section IV-C of the paper): for every plan, how much would
// evicting each tensor that is resident and idle at the peak lower the peak,
// given the earliest swap-out / latest swap-in the host link's speed allows:
//   score = P - max( max MF[0..o], max MF[q..T), P - size ).
//
// Which tensors can be candidates at a peak step t* does not depend on the plan:
// they are the gaps (p, q) of the TAS with a feasible earliest swap-out step o
// (a property of the gap alone: it follows from p, q, the transfer time and the
// cumulative latency) and o < t* < q.  tensile_tas_load files every such gap
// under each bucket of 2^shift steps that (o, q) overlaps, so a plan looks at the
// one bucket of its t* (see CandIndex in common.h).  Everything a plan needs
// beyond its own footprint row and interval list is static and shared by all plans
// with the same bucket.  The recomputation savings (section IV-D) use the same
// kernel on a second index in which every gap is filed with o = p, and any interval
// of a tensor cancels its entries.
//
// Per plan, one workgroup of 256, 512 or 1024 threads (Shape):
//   1. the maxima of the row's blocks of 256 steps (more for rows of over 262,144
//      steps), streamed from the row or taken from the evaluation; then their prefix and suffix
//      maxima (two wavefronts), while the plan's own intervals cancel candidates:
//      an interval inside the gap of an entry of its tensor (Alg. 2 of the paper only
//      takes tensors that are not swapped out yet).  A per-bucket bit filter over
//      tensors, kept in LDS, turns most intervals away and leads the others to their
//      tensor's entries;
//   2. every entry with o < t* < q that is not cancelled is bounded from both sides by
//      the block maxima (score_body.h: classify).  Most are decided by that; the
//      open ones are listed, and the few blocks of the row that they lie in - those
//      around the peak - are read (resolve_open);
//   3. every wavefront composes the output of its own range of tensors, 128 at a time,
//      in LDS (zeros and -1, then the entries, which are stored in tensor order) and writes whole pieces of the rows, so
//      that each output line goes to memory once.  (What step 2 found is not kept but found
//      again: it costs a few LDS reads per entry and no space.)
// Nothing is kept per entry but a bit or two, so a workgroup of 256 or 512 threads needs a third of a CU's LDS or less,
// and the phases of several plans overlap on a CU.
// What bounds it: HBM (rows in unless the evaluation hands over their maxima, output rows out) on long rows, the
// chains of dependent loads of a plan's phases on short ones.  Measured against the kernel before it (one workgroup of 1024
// threads per CU that ran two 64-bit max-scans over every 256 steps of the row and met every candidate's o and q on the way, its
// phases one after the other with nothing beside them): scoring by itself, 16,384 plans of 50,000 steps 2.72 -> 2.6 ms
// (4.9 TB/s of what has to move), 1,024 of 10^6 2.43 -> 2.04 ms; evaluation and scoring in one call, 4,096 plans of 6,000
// steps 243 -> 141 us, 8,192 of 24,000 1.20 -> 0.88 ms, 1,111 ragged ones of 33,331 216 -> 124 us.
// A plan with more open entries than the list holds, or a bucket with more entries than there are flags
// (kWindow), takes the general form: rows cleared first, then the entries in runs of one per thread, written one by one.
#include <type_traits>

#include "score_body.h"

namespace tensile {

namespace {

// The workgroup and its table of block maxima.  In batches of no more plans than CUs, where nothing but a plan's own wavefronts
// covers the chains of its phases: 1024 threads and 1,024 blocks (of as many pieces of 256 steps as it takes).  Scoring by
// itself, against 512 threads (rows up to 131,072 steps) or 256 (longer ones): 256 plans of 24,000 steps 32.7 -> 27.0 us, of
// 50,000 steps 56.8 -> 45.6, 32 of 300,000 steps 161 -> 61, one of 10^6 steps 487 -> 152; evaluation and scoring in one call,
// against 256 threads, 32 plans of 6,000 steps 25.6 -> 21.3; more pieces ahead than two gain nothing.  The rest of the LDS holds
// a copy of the bucket's entries, which the cancelling looks at again and again when a plan's list is in no order (256 ragged,
// shuffled plans of 50,000 steps 56 -> 48 us).  Not where four wavefronts
// have a piece of work each and more would idle (60 tensors, 200 steps: 64 plans 15.9 us with 1024 threads, 15.7 with 256; 534 tensors,
// 1,000 steps: 18.9 and 19.1).  Rows of more bytes
// than the memory-side cache keeps (256 MB) are read past the L2's allocation there: 32 plans of 10^6 steps 236 -> 213 us,
// 256 of 300,000 202 -> 157; with rows that stay in it that costs (256 of 50,000 steps 45.6 and 53.3, 32 of 300,000 61 and 76).
// Larger batches, up to 32,768 steps, when the maxima are given: 256
// threads and 128 blocks, six workgroups per CU, whose chains of short dependent loads cover each other (against 512
// threads, with evaluation: 4,096 plans of 6,000 steps 161 -> 141 us, 8,192 of 24,000 steps 912 -> 876).  Else, up to 131,072
// steps: 512 threads, 512 blocks, three per CU (streaming 4,096 rows of 24,000 steps 336 us, with 256 threads 381; 50,000
// steps 2.62 ms and 2.69).  Longer rows: 256 threads, 1,024 blocks, four per CU, plans dealt to as many workgroups as are
// resident (10^6 steps 2.04 ms; with 512 threads 2.17).
template <int tab, int thr, int eu, int bufs, int entries, bool stream>
struct Shape {
    static constexpr int kTab = tab, kThr = thr, kWaves = thr / 64;
    static constexpr int kBufs = bufs;           // wavefronts that read the row's blocks for the open entries: as many as the LDS has room for
    static constexpr int kEu = eu;               // wavefronts per SIMD that fit
    static constexpr int kEntries = entries;     // entries of the bucket that are copied to the LDS for the cancelling
    static constexpr bool kStream = stream;      // rows read and outputs written past the L2's allocation
};
typedef Shape<128, 256, 6, 3, 0, false> Small;
typedef Shape<512, 512, 6, 5, 0, false> Short;
typedef Shape<1024, 256, 4, 2, 0, true> Long;
typedef Shape<1024, 1024, 4, 16, 4096, false> Wide;
typedef Shape<1024, 1024, 4, 16, 4096, true> WideStream;
constexpr int64_t kWideStreamBytes = int64_t{192} << 20;

struct StageBuf {
    int64_t score[kStage];
    int32_t win[2][kStage];      // win_out, win_in
};

template <class S>
struct ScoreLds {
    union {
        __attribute__((aligned(16))) StageBuf stage[S::kWaves];
        __attribute__((aligned(16))) SpanBuf bufs[S::kBufs];
    };
    BlockMaxima<S::kTab> mx;
    OpenList<S::kThr> open;
    uint64_t cancelled[kWindow / 64];    // one bit per entry of the window
    uint64_t open_bits[kWindow / 64];    // the entry is on the open list, at open_base + its rank within the word
    uint16_t open_base[kWindow / 64];
    uint32_t filter[kFilterWords];
    int32_t filter_base[kFilterWords + 1];
    uint32_t need[S::kTab / 32];         // blocks of the row that open entries lie in
    __attribute__((aligned(16))) int4 entries[S::kEntries ? S::kEntries : 1];   // the bucket's, if that many hold them
};

// Step 1: the maxima of the row's blocks into pm[k + 1] and sm[k].  The blocks are dealt round-robin, so that
// the workgroup reads neighbouring lines at any time, each wavefront kAhead pieces ahead.
template <bool kVec, class S>
__device__ __forceinline__ void stream_block_maxima(const ScoreArgs &a, const int64_t *MF, BlockMaxima<S::kTab> &mx, int wave, int lane) {
    constexpr int kAhead = 2, kWaves = S::kWaves;
    constexpr bool kStream = S::kStream;
    const int ps = a.piece_shift;
    const int32_t mine = wave < a.n_blk ? (a.n_blk - wave + kWaves - 1) / kWaves : 0;   // blocks of this wavefront
    const int32_t n = mine << ps;
    const int32_t T = a.T;
    auto first_step = [&](int32_t i) { return (((wave + (i >> ps) * kWaves) << ps) + (i & ((1 << ps) - 1))) * kMini; };
    // (any order of the 256 steps over the lanes will do here: whole lines per load.  Beyond the row's end the loads are
    // clamped and the values left out.)
    auto load = [&](int32_t i, int64_t (&x)[4]) {
        const int32_t t0 = first_step(i < n ? i : n - 1);
        if constexpr (kVec) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int32_t t = t0 + 128 * j + 2 * lane;
                const ll2 *at = reinterpret_cast<const ll2 *>(MF + (t < T ? t : T - 2));
                ll2 v;
                if constexpr (kStream) v = __builtin_nontemporal_load(at);
                else v = *at;
                x[2 * j] = v[0];
                x[2 * j + 1] = v[1];
            }
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int32_t t = t0 + 64 * j + lane;
                const int64_t *at = MF + (t < T ? t : T - 1);
                if constexpr (kStream) x[j] = __builtin_nontemporal_load(at);
                else x[j] = *at;
            }
        }
    };
    if (n == 0) return;      // (wave-uniform)
    // (a clamped load brings the row's last step or last two once more: a value of the row's last block again, which
    // changes no maximum as long as the piece itself starts inside the row)
    int64_t x[kAhead][4];
#pragma unroll
    for (int d = 0; d < kAhead; ++d) load(d, x[d]);
    int64_t run = INT64_MIN;
    for (int32_t i0 = 0; i0 < n; i0 += kAhead) {
#pragma unroll
        for (int d = 0; d < kAhead; ++d) {
            const int32_t i = i0 + d;
            if (i < n) {     // (wave-uniform)
                const int64_t m = max64(max64(x[d][0], x[d][1]), max64(x[d][2], x[d][3]));
                load(i + kAhead, x[d]);
                const int32_t t0 = first_step(i);
                run = max64(run, t0 < T ? m : INT64_MIN);
                if ((i & ((1 << ps) - 1)) == (1 << ps) - 1) {     // the block's last piece
                    const int64_t v = wave_max(run);
                    const int32_t blk = wave + (i >> ps) * kWaves;
                    if (lane == 0) {
                        mx.pm[blk + 1] = v;
                        mx.sm[blk] = v;
                    }
                    run = INT64_MIN;
                }
            }
        }
    }
}

// Step 1 where the maxima of the row's pieces are known (the evaluation wrote them): the row is not read.
template <class S>
__device__ __forceinline__ void load_block_maxima(const ScoreArgs &a, const int64_t *pieces, BlockMaxima<S::kTab> &mx, int tid) {
    const int ps = a.piece_shift;
    for (int32_t k = tid; k < a.n_blk; k += S::kThr) {
        const int32_t p0 = k << ps, p1 = min(p0 + (1 << ps), a.n_mini);
        int64_t v = pieces[p0];
        for (int32_t p = p0 + 1; p < p1; ++p) v = max64(v, pieces[p]);
        mx.pm[k + 1] = v;
        mx.sm[k] = v;
    }
}

// kVec: the footprint rows are 16-byte aligned and T is even.
// kTable: the maxima of the rows' pieces are given.
template <class S, bool kVec, bool kTable>
__device__ __forceinline__ void score_plan(const ScoreArgs &a, const int32_t b, ScoreLds<S> &L, int32_t &filter_of) {
    constexpr int kThr = S::kThr, kBufs = S::kBufs;
    constexpr bool kBig = S::kStream;
    // (the thread index is made opaque once per plan: everything derived from it is then
    // recomputed where it is used instead of being held in registers across the whole loop)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t tstar = uniform_load(a.argmax, b);
    const int64_t P = uniform_load(a.peak, b);
    const int64_t *MF = a.resident + static_cast<int64_t>(b) * a.T;
    int64_t *score = a.score + static_cast<int64_t>(b) * a.N;
    int32_t *wout = a.win_out ? a.win_out + static_cast<int64_t>(b) * a.N : nullptr;
    int32_t *win = a.win_in ? a.win_in + static_cast<int64_t>(b) * a.N : nullptr;
    PROF_START;
    const bool has_peak = tstar >= 0 && tstar < a.T;     // else not produced by the evaluator: no candidate
    const int32_t bk = has_peak ? tstar >> a.bucket_shift : 0;
    const int32_t e0 = uniform_load(a.bucket_off, bk), n_e = has_peak ? uniform_load(a.bucket_off, bk + 1) - e0 : 0;
    auto clear_rows = [&]() {
        fill_row<kThr, int64_t>(score, a.N, 0, tid);
        if (wout) fill_row<kThr, int32_t>(wout, a.N, -1, tid);
        if (win) fill_row<kThr, int32_t>(win, a.N, -1, tid);
    };
    if (n_e == 0) {                                      // no gap around t* can be swapped in time
        clear_rows();
        return;
    }
    int64_t k0 = uniform_load(a.plan_offsets, b), k1 = uniform_load(a.plan_offsets, b + 1);
    if (k0 < 0) k0 = 0;
    if (k1 > a.n_intervals) k1 = a.n_intervals;
    const int bs = a.piece_shift + 8;
    const int4 *const entries = a.cand + e0;
    const int64_t *const size_of = a.cand_size + e0;

    // ---- 1
    __syncthreads();       // the previous plan has finished with the LDS
    if (filter_of != bk) {
        const uint32_t *src = a.filter + static_cast<int64_t>(bk) * a.filter_words;
        const int32_t *src_base = a.filter_base + static_cast<int64_t>(bk) * (a.filter_words + 1);
        for (int32_t k = tid; k < a.filter_words; k += kThr) L.filter[k] = src[k];
        for (int32_t k = tid; k <= a.filter_words; k += kThr) L.filter_base[k] = src_base[k];
        filter_of = bk;
    }
    for (int32_t k = tid; k < kWindow / 64 && k * 64 < n_e; k += kThr) L.cancelled[k] = 0;
    for (int32_t k = tid; k * 32 < a.n_blk; k += kThr) L.need[k] = 0;
    if (tid == 0) L.open.n = 0;
    const bool copied = n_e <= S::kEntries;
    if constexpr (S::kEntries > 0) {
        if (copied)
            for (int32_t k = tid; k < n_e; k += kThr) L.entries[k] = entries[k];
    }
    if constexpr (kTable) load_block_maxima<S>(a, a.blk_max + static_cast<int64_t>(b) * a.n_mini, L.mx, tid);
    else stream_block_maxima<kVec, S>(a, MF, L.mx, wave, lane);
    PROF_MARK(0);
    __syncthreads();
    PROF_MARK(1);
    scan_block_maxima(L.mx, a.n_blk, wave, lane);
    PROF_MARK(2);
    auto cancel_from = [&](const int4 *list) {
        cancel_by_plan<kThr>(a, k0, k1, list, n_e, 0, n_e < kWindow ? n_e : kWindow, L.filter, L.filter_base, reinterpret_cast<uint32_t *>(L.cancelled), tid);
    };
    if constexpr (S::kEntries > 0) {
        if (copied) cancel_from(L.entries);
        else cancel_from(entries);
    } else {
        cancel_from(entries);
    }
    PROF_MARK(3);
    __syncthreads();
    PROF_MARK(4);

    // an entry: is it a candidate, and what do the block maxima say
    struct Entry {
        bool valid, open;
        Classified c;
    };
    auto look = [&](int32_t k, int32_t in_window, int2 oq, int64_t size) {   // (k < n_e, or valid comes out false)
        Entry e;
        e.valid = k < n_e && oq.x < tstar && tstar < oq.y && !((L.cancelled[in_window >> 6] >> (in_window & 63)) & 1u);
        e.c = classify(L.mx, bs, oq, P - size);
        e.open = e.valid && (e.c.open_o || e.c.open_q);
        return e;
    };
    // puts this wavefront's open entries (64 consecutive entries of the bucket, in order) on the list
    auto list_open = [&](const Entry &e, int2 oq, int32_t in_window) {
        const uint64_t mask = __builtin_amdgcn_ballot_w64(e.open);
        const int32_t word = __builtin_amdgcn_readfirstlane(in_window >> 6);
        if (lane == 0) L.open_bits[word] = mask;
        if (mask == 0) return;
        int32_t base = 0;
        if (lane == 0) {
            base = atomicAdd(&L.open.n, __builtin_popcountll(mask));
            L.open_base[word] = static_cast<uint16_t>(base);
        }
        base = __builtin_amdgcn_readfirstlane(base);
        const int32_t at = base + __builtin_popcountll(mask & ((1ull << lane) - 1));
        if (e.open && at < kThr) {
            L.open.acc[at] = e.c.lo;
            L.open.oq[at] = make_int2(e.c.open_o ? oq.x : -1, e.c.open_q ? oq.y : -1);
            if (e.c.open_o) atomicOr(&L.need[oq.x >> (bs + 5)], 1u << ((oq.x >> bs) & 31));
            if (e.c.open_q) atomicOr(&L.need[oq.y >> (bs + 5)], 1u << ((oq.y >> bs) & 31));
        }
    };
    auto outside_of = [&](const Entry &e, int32_t in_window) {   // the maximum outside the entry's window, at least P - size
        if (!e.open) return e.c.lo;
        const int32_t word = in_window >> 6, bit = in_window & 63;
        return L.open.acc[L.open_base[word] + __builtin_popcountll(L.open_bits[word] & ((1ull << bit) - 1))];
    };

    // ---- 2
    bool general = n_e > kWindow;
    if (!general) {
        for (int32_t kb = 0; kb < n_e; kb += kThr) {
            const int32_t k = kb + tid, kc = k < n_e ? k : n_e - 1;
            if (kb + wave * 64 >= n_e) break;            // (wave-uniform)
            const int4 c = entries[kc];
            const int2 oq = make_int2(c.w, c.z);
            list_open(look(k, kc, oq, size_of[kc]), oq, kb + wave * 64);
        }
        __syncthreads();
        const int32_t n_open = L.open.n;
        general = n_open > kThr;
        if (n_open > 0 && !general) {
            resolve_open<kVec, kBufs>(a, MF, L.need, L.open, n_open, L.bufs, wave, lane);
            __syncthreads();
        }
    }
    PROF_MARK(5);

    // ---- 3
    if (!general) {
        StageBuf &st = L.stage[wave];
        // With 16-byte aligned arrays the chunks start where the plan's rows are aligned too: `shift` tensors later, when
        // N is no multiple of four (the first `shift` tensors are a chunk of their own).
        const bool wide = ((reinterpret_cast<uintptr_t>(a.score) | reinterpret_cast<uintptr_t>(a.win_out) | reinterpret_cast<uintptr_t>(a.win_in)) & 15) == 0;
        const int32_t shift = wide ? static_cast<int32_t>((0u - static_cast<uint32_t>(b) * static_cast<uint32_t>(a.N)) & 3u) : 0;
        const int32_t t_begin = wave == 0 ? (shift ? shift - kStage : 0) : wave * a.tspan + shift;
        const int32_t t_end = min((wave + 1) * a.tspan + shift, a.N);
        if (t_begin >= t_end) return;                    // (wave-uniform: no tensors for this wavefront)
        // the wavefront's entries, 64 at a time: those at hand, examined, and the next ones on their way.  They start
        // with the first entry of the filter word that its first tensor falls into (or some earlier tensor of the word does).
        int32_t k = __builtin_amdgcn_readfirstlane(L.filter_base[(wave * a.tspan) >> (5 + a.filter_shift)]);
        int4 next;
        int64_t next_size;
        auto request = [&](int32_t at) {
            const int32_t kc = at + lane < n_e ? at + lane : n_e - 1;
            next = entries[kc];
            next_size = size_of[kc];
        };
        int32_t tensor, o, q;
        int64_t value;
        bool has;
        auto take_up = [&]() {                           // the requested entries become those at hand; request the next
            const int32_t kk = k + lane;
            const int32_t kc = kk < n_e ? kk : n_e - 1;
            const Entry e = look(kk, kc, make_int2(next.w, next.z), next_size);
            tensor = kk < n_e ? next.x : INT32_MAX;
            o = next.w;
            q = next.z;
            has = e.valid;
            value = P - outside_of(e, kc);
            request(k + 64);
        };
        int32_t pos = 0;                                 // entries at hand that are done
        request(k);
        take_up();
        for (int32_t t0 = t_begin; t0 < t_end; t0 += kStage) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            reinterpret_cast<ll2 *>(st.score)[lane] = ll2{0, 0};
            reinterpret_cast<ll2 *>(st.win)[lane] = ll2{-1, -1};
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            for (;;) {                                   // (wave-uniform)
                const bool take = lane >= pos && tensor < t0 + kStage;
                if (take && has && tensor >= t0) {       // (those below t0 belong to the wavefront before)
                    st.score[tensor - t0] = value;
                    st.win[0][tensor - t0] = o;
                    st.win[1][tensor - t0] = q;
                }
                pos += __builtin_popcountll(__builtin_amdgcn_ballot_w64(take));
                if (pos < 64) break;
                k += 64;
                pos = 0;
                take_up();
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (wide && t0 >= 0 && t0 + kStage <= a.N) {
                store_out<kBig>(reinterpret_cast<ll2 *>(score + t0) + lane, reinterpret_cast<const ll2 *>(st.score)[lane]);
                int32_t *const dst = lane < 32 ? wout : win;     // (32 vectors of four each)
                if (dst) store_out<kBig>(reinterpret_cast<i4 *>(dst + t0) + (lane & 31), reinterpret_cast<const i4 *>(st.win)[lane]);
            } else {
#pragma unroll
                for (int j = 0; j < kStage / 64; ++j) {
                    const int32_t u = j * 64 + lane;
                    if (t0 + u >= 0 && t0 + u < a.N) {
                        score[t0 + u] = st.score[u];
                        if (wout) wout[t0 + u] = st.win[0][u];
                        if (win) win[t0 + u] = st.win[1][u];
                    }
                }
            }
        }
        PROF_MARK(6);
        return;
    }

    // ---- 2 and 3 in the general form
    clear_rows();
    for (int32_t w_lo = 0; w_lo < n_e; w_lo += kWindow) {
        const int32_t w_n = min(kWindow, n_e - w_lo);
        if (w_lo > 0) {                                  // (the first window's flags are there)
            for (int32_t k = tid; k < kWindow / 64; k += kThr) L.cancelled[k] = 0;
            __syncthreads();
            cancel_by_plan<kThr>(a, k0, k1, entries, n_e, w_lo, w_n, L.filter, L.filter_base, reinterpret_cast<uint32_t *>(L.cancelled), tid);
        }
        for (int32_t kb = 0; kb < w_n; kb += kThr) {
            __syncthreads();       // everybody has finished with the list and the blocks of the previous run (and clearing the rows)
            for (int32_t k = tid; k * 32 < a.n_blk; k += kThr) L.need[k] = 0;
            if (tid == 0) L.open.n = 0;
            __syncthreads();
            const int32_t k = w_lo + kb + tid, kc = k < n_e ? k : n_e - 1;
            const int4 c = entries[kc];
            const int2 oq = make_int2(c.w, c.z);
            const Entry e = look(k, kc - w_lo, oq, size_of[kc]);
            if (kb + wave * 64 < w_n) list_open(e, oq, kb + wave * 64);
            __syncthreads();
            const int32_t n_open = L.open.n;             // (at most one per thread)
            if (n_open > 0) {
                resolve_open<kVec, kBufs>(a, MF, L.need, L.open, n_open, L.bufs, wave, lane);
                __syncthreads();
            }
            if (e.valid && kb + tid < w_n) {
                const int32_t tensor = c.x;
                score[tensor] = P - outside_of(e, kb + tid);
                if (wout) wout[tensor] = oq.x;
                if (win) win[tensor] = oq.y;
            }
        }
    }
}

// Workgroup w takes the plans w, w + grid, ...
template <class S, bool kVec, bool kTable>
__global__ __launch_bounds__(S::kThr) __attribute__((amdgpu_waves_per_eu(S::kEu, S::kEu))) void score_kernel(const ScoreArgs a) {
    __shared__ ScoreLds<S> lds;
    int32_t filter_of = -1;      // bucket whose filter is in LDS
    for (int64_t b = blockIdx.x; b < a.B; b += gridDim.x) score_plan<S, kVec, kTable>(a, static_cast<int32_t>(b), lds, filter_of);
}

// ---- one iteration of the planner on the device --------------------------------------------------------
// Alg. 3 analyses the peak again after every tensor it schedules.  The planner's row exists already, so an
// iteration is: take the new interval's bytes out of its window of the row; bring the maxima (and their earliest
// steps) of the 256-step blocks the window touches up to date - the table of block maxima is kept in global
// memory from iteration to iteration: it is the block-level form of the prefix / suffix maxima of the row, of
// which only the window's part changes; find the peak and its earliest step from the table; score the candidates
// from the table's prefix and suffix maxima, as the batch kernel does - the row itself is read only in the few blocks
// that leave a candidate open - and hand the host one record per tensor with a window.  One workgroup, one launch.
// Which candidates the plan has already dealt with is not worked out from the plan's list (the list grows with
// every iteration): a flag per gap and per tensor, set as intervals join, says so.
// (Before: every block of the row with an endpoint of a candidate in it was read and scanned, every iteration.)
struct GreedyStepArgs {
    ScoreArgs s;                 // the scoring pass: one plan
    int64_t *row;                // [T] the plan's footprint, in/out
    int64_t *blk_max;            // [ceil(T / kMini)] maxima of the row's 256-step pieces, in/out
    int32_t *blk_arg;            // [ceil(T / kMini)] earliest step of each piece's maximum, in/out
    uint8_t *gap_taken;          // [gaps] the plan holds an interval inside this gap, in/out
    uint8_t *tensor_taken;       // [N] the plan holds an interval of this tensor, in/out
    int32_t new_gap;             // the new interval's gap, or -1
    const int64_t *size;         // [N]
    int32_t rebuild;             // every piece's maximum is computed afresh (first launch on a row)
    int32_t has_new;             // an interval joins the plan: applied to the row and written to position plan_n
    int32_t new_tensor, new_out, new_in, plan_n;
    int32_t *plan_t, *plan_o, *plan_r;
    int32_t do_score;            // 0: only the header {peak, peak step, 0} is produced
    ScoreHeader *hdr;            // the record for the host (pinned host memory)
    ScoreCand *compact;
    unsigned long long *ready;   // receives ready_value when header and records are visible system-wide
    unsigned long long ready_value;
};

constexpr int kPlanThr = 1024, kPlanWaves = kPlanThr / 64;
constexpr int kPer = 3, kPlanRun = kPer * kPlanThr;   // entries of the bucket per thread, and per run
constexpr int kPlanTab = 1024;
static_assert(kPlanTab <= kPlanThr, "one block of the table per thread");

struct PlanLds {
    union {
        __attribute__((aligned(16))) SpanBuf bufs[kPlanWaves];
        __attribute__((aligned(16))) ScoreCand stage[kPlanRun];   // records on their way to the host
    };
    BlockMaxima<kPlanTab> mx;
    OpenList<kPlanRun> open;
    uint32_t need[kPlanTab / 32];
    int64_t red_v[kPlanWaves];
    int32_t red_t[kPlanWaves];
    int32_t n_stage;
};

// The window of the new interval leaves the row, and the table entries of the blocks it touches (of all blocks on a
// fresh row) are recomputed.  One block per wavefront and round, 4 steps per lane.
template <bool kVec>
__device__ __forceinline__ void patch_row_and_table(const GreedyStepArgs &g, int tid) {
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t T = g.s.T, n_blk = g.s.n_mini;
    int64_t *const row = g.row;
    const int32_t i = g.new_tensor, o = g.new_out, r = g.new_in;
    const bool ok = g.has_new && static_cast<uint32_t>(i) < static_cast<uint32_t>(g.s.N) && o >= 0 && r <= T && r > o;
    if (g.has_new && tid == 0) {   // the plan's own arrays learn of the interval here, and so do the flags
        g.plan_t[g.plan_n] = i;
        g.plan_o[g.plan_n] = o;
        g.plan_r[g.plan_n] = r;
        if (ok) {
            g.tensor_taken[i] = 1;
            if (g.new_gap >= 0) g.gap_taken[g.new_gap] = 1;
        }
    }
    const int64_t sz = ok ? g.size[i] : 0;
    const int32_t win_lo = ok ? o + 1 : 0, win_hi = ok ? r : 0;   // steps win_lo .. win_hi - 1 lose sz bytes
    const bool any = win_hi > win_lo;
    const int32_t kb0 = g.rebuild ? 0 : (any ? win_lo / kMini : 0);
    const int32_t kb1 = g.rebuild ? n_blk : (any ? (win_hi - 1) / kMini + 1 : 0);
    for (int32_t k = kb0 + wave; k < kb1; k += kPlanWaves) {   // (wave-uniform)
        const int32_t t = k * kMini + 4 * lane;
        int64_t x[4];
        load_quad<kVec>(row, t, T, x);    // steps beyond T come back as INT64_MIN and lie outside every window
        bool ch[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            ch[j] = t + j >= win_lo && t + j < win_hi;
            x[j] -= ch[j] ? sz : 0;
        }
#pragma unroll
        for (int j = 0; j < 4; j += 2) {
            if (kVec && ch[j] && ch[j + 1]) {
                *reinterpret_cast<ll2 *>(row + t + j) = ll2{x[j], x[j + 1]};
            } else {
                if (ch[j]) row[t + j] = x[j];
                if (ch[j + 1]) row[t + j + 1] = x[j + 1];
            }
        }
        const int64_t lm = max64(max64(x[0], x[1]), max64(x[2], x[3]));
        int32_t lj = 3;
#pragma unroll
        for (int j = 2; j >= 0; --j)
            if (x[j] == lm) lj = j;
        const int64_t m = last_lane(wave_scan_max(lm));
        const uint64_t holders = __builtin_amdgcn_ballot_w64(lm == m);   // (never empty)
        if (lane == __builtin_ctzll(holders)) {
            g.blk_max[k] = m;
            g.blk_arg[k] = t + lj;
        }
    }
}

template <bool kVec>
__global__ __launch_bounds__(kPlanThr) void greedy_step_kernel(const GreedyStepArgs g) {
    __shared__ PlanLds lds;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    PROF_START;
    const ScoreArgs &a = g.s;
    const int ps = a.piece_shift, bs = ps + 8;
    patch_row_and_table<kVec>(g, tid);
    // other wavefronts of this workgroup read what these stores wrote (table entries now, the row in the scoring pass)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __syncthreads();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");

    // ---- the table into LDS, one block per thread; the peak and its earliest step
    int64_t bv = INT64_MIN;
    int32_t bt = INT32_MAX;
    if (tid < a.n_blk) {
        const int32_t p0 = tid << ps, p1 = min(p0 + (1 << ps), a.n_mini);
        for (int32_t p = p0; p < p1; ++p) {
            const int64_t v = g.blk_max[p];
            const int32_t t = g.blk_arg[p];
            if (v > bv) {        // (in ascending order: the earliest step among equals)
                bv = v;
                bt = t;
            }
        }
        lds.mx.pm[tid + 1] = bv;
        lds.mx.sm[tid] = bv;
    }
    auto better = [&](int64_t ov, int32_t ot) {
        if (ov > bv || (ov == bv && ot < bt)) {
            bv = ov;
            bt = ot;
        }
    };
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) better(__shfl_xor(bv, d, 64), __shfl_xor(bt, d, 64));
    if (lane == 0) {
        lds.red_v[wave] = bv;
        lds.red_t[wave] = bt;
    }
    if (tid * 32 < a.n_blk) lds.need[tid] = 0;
    if (tid == 0) lds.n_stage = lds.open.n = 0;
    __syncthreads();
    bv = lds.red_v[lane & (kPlanWaves - 1)];             // (every wavefront reduces for itself: no barrier)
    bt = lds.red_t[lane & (kPlanWaves - 1)];
#pragma unroll
    for (int d = kPlanWaves / 2; d >= 1; d >>= 1) better(__shfl_xor(bv, d, 64), __shfl_xor(bt, d, 64));
    const int32_t tstar = __builtin_amdgcn_readfirstlane(bt);
    const int64_t P = lane_value(bv, 0);
    PROF_MARK(8);
    if (!g.do_score) {
        if (tid == 0) {
            *g.hdr = ScoreHeader{P, tstar, 0};
            __hip_atomic_store(g.ready, g.ready_value, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        return;
    }
    const int32_t bk = tstar >> a.bucket_shift;
    const int32_t e0 = uniform_load(a.bucket_off, bk), n_e = uniform_load(a.bucket_off, bk + 1) - e0;
    int32_t n_out = 0;     // records handed to the host so far (the same in every thread)
    for (int32_t run_lo = 0; run_lo < n_e; run_lo += kPlanRun) {
        const int32_t n_run = min(kPlanRun, n_e - run_lo);
        if (run_lo > 0) {
            __syncthreads();       // the previous run has finished with the lists and the staging area
            if (tid * 32 < a.n_blk) lds.need[tid] = 0;
            if (tid == 0) lds.n_stage = lds.open.n = 0;
        }
        // this thread's entries: static, requested now, and on their way while two wavefronts scan the table
        int2 oq[kPer];
        int32_t tensor[kPer], gap[kPer];
        int64_t size[kPer];
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int32_t k = j * kPlanThr + tid, e = e0 + run_lo + (k < n_run ? k : n_run - 1);
            const int4 c = a.cand[e];
            oq[j] = make_int2(c.w, c.z);
            tensor[j] = c.x;
            gap[j] = a.cand_gap[e];
            size[j] = a.cand_size[e];
        }
        uint8_t taken[kPer];       // (the flags were set before the first barrier)
#pragma unroll
        for (int j = 0; j < kPer; ++j) taken[j] = a.any_interval ? g.tensor_taken[tensor[j]] : g.gap_taken[gap[j]];
        if (run_lo == 0) scan_block_maxima(lds.mx, a.n_blk, wave, lane);
        __syncthreads();
        PROF_MARK(9);
        // ---- what the table says; the open ones on the list
        int64_t value[kPer];
        int32_t at[kPer];          // place on the open list, -1: none, -2: not a candidate
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const bool valid = j * kPlanThr + tid < n_run && oq[j].x < tstar && tstar < oq[j].y && !taken[j];
            const Classified c = classify(lds.mx, bs, oq[j], P - size[j]);
            value[j] = c.lo;
            at[j] = valid ? -1 : -2;
            const bool open = valid && (c.open_o || c.open_q);
            const uint64_t mask = __builtin_amdgcn_ballot_w64(open);
            if (mask) {            // (wave-uniform)
                int32_t base = 0;
                if (lane == 0) base = atomicAdd(&lds.open.n, __builtin_popcountll(mask));
                base = __builtin_amdgcn_readfirstlane(base);
                if (open) {
                    at[j] = base + __builtin_popcountll(mask & ((1ull << lane) - 1));
                    lds.open.acc[at[j]] = c.lo;
                    lds.open.oq[at[j]] = make_int2(c.open_o ? oq[j].x : -1, c.open_q ? oq[j].y : -1);
                    if (c.open_o) atomicOr(&lds.need[oq[j].x >> (bs + 5)], 1u << ((oq[j].x >> bs) & 31));
                    if (c.open_q) atomicOr(&lds.need[oq[j].y >> (bs + 5)], 1u << ((oq[j].y >> bs) & 31));
                }
            }
        }
        __syncthreads();
        PROF_MARK(10);
        const int32_t n_open = lds.open.n;
        if (n_open > 0) {
            resolve_open<kVec, kPlanWaves>(a, g.row, lds.need, lds.open, n_open, lds.bufs, wave, lane);
            __syncthreads();
        }
        PROF_MARK(11);
        // ---- the records, staged in LDS and sent to the host as whole lines
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const uint64_t mask = __builtin_amdgcn_ballot_w64(at[j] != -2);
            if (mask == 0) continue;
            int32_t base = 0;
            if (lane == 0) base = atomicAdd(&lds.n_stage, __builtin_popcountll(mask));
            base = __builtin_amdgcn_readfirstlane(base);
            if (at[j] != -2)
                lds.stage[base + __builtin_popcountll(mask & ((1ull << lane) - 1))] =
                    ScoreCand{P - (at[j] >= 0 ? lds.open.acc[at[j]] : value[j]), tensor[j], oq[j].x, oq[j].y, gap[j]};
        }
        __syncthreads();
        const int32_t n_st = lds.n_stage;
        const int64_t *src = reinterpret_cast<const int64_t *>(lds.stage);
        int64_t *dst = reinterpret_cast<int64_t *>(g.compact + n_out);
        for (int32_t w = tid; w < 3 * n_st; w += kPlanThr) dst[w] = src[w];
        n_out += n_st;
        PROF_MARK(12);
    }
    // the header travels with the records: one wait for the host's memory instead of two.  The barrier orders every
    // thread's records before thread 0's store of the signal, and that store releases at system scope - which
    // covers what happened before it in other threads too (a system-scope fence in each of the 1024 threads,
    // as it was first written, cost 2 us per iteration more)
    if (tid == 0) *g.hdr = ScoreHeader{P, tstar, n_out};
    __syncthreads();
    if (tid == 0) __hip_atomic_store(g.ready, g.ready_value, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    PROF_MARK(13);
}

}  // namespace

// One iteration of tensile_greedy_plan on the device (see greedy_step_kernel).  pl: the one plan INCLUDING the new
// interval (n_intervals counts it; its slot in the device arrays is written by the kernel).
int launch_greedy_step(const tensile_tas *tas, Workspace &ws, const CandIndex &ix, bool any_interval, const tensile_plans *pl,
                       int64_t *row, const GreedyTables &tables, bool rebuild, const GreedyNew *fresh, bool do_score,
                       ScoreHeader *hdr, ScoreCand *compact, unsigned long long *ready, unsigned long long ready_value) {
    GreedyStepArgs g{};
    g.s = make_score_args(tas, ix, any_interval, pl, kPlanTab, row, nullptr, nullptr, nullptr, nullptr, nullptr);
    g.hdr = hdr; g.compact = compact; g.ready = ready; g.ready_value = ready_value;
    g.row = row; g.blk_max = tables.blk_max; g.blk_arg = tables.blk_arg; g.size = tas->d_size.p;
    g.gap_taken = tables.gap_taken; g.tensor_taken = tables.tensor_taken; g.new_gap = -1;
    g.rebuild = rebuild ? 1 : 0;
    g.do_score = (do_score && tas->N > 0) ? 1 : 0;
    if (fresh) {
        g.has_new = 1;
        g.new_tensor = fresh->tensor; g.new_out = fresh->out; g.new_in = fresh->in; g.plan_n = fresh->position;
        g.new_gap = fresh->gap;
        g.plan_t = fresh->plan_t; g.plan_o = fresh->plan_o; g.plan_r = fresh->plan_r;
    }
    const bool vec16 = tas->T % 2 == 0 && reinterpret_cast<uintptr_t>(row) % 16 == 0;
    if (vec16) hipLaunchKernelGGL(greedy_step_kernel<true>, dim3(1), dim3(kPlanThr), 0, ws.stream, g);
    else hipLaunchKernelGGL(greedy_step_kernel<false>, dim3(1), dim3(kPlanThr), 0, ws.stream, g);
    TS_HIP(hipGetLastError());
    return TENSILE_OK;
}

int launch_score(const tensile_tas *tas, Workspace &ws, const CandIndex &ix, bool any_interval, const tensile_plans *plans,
                 const int64_t *resident, const int64_t *peak, const int32_t *argmax, int64_t *score, int32_t *win_out,
                 int32_t *win_in, const int64_t *blk_max) {
    if (plans->B == 0 || tas->N == 0) return TENSILE_OK;
    const bool vec16 = tas->T % 2 == 0 && reinterpret_cast<uintptr_t>(resident) % 16 == 0;
    // (A launch has room for fewer than 2^32 threads: past kMostBlocks a workgroup takes several plans.)
    constexpr int32_t kMostBlocks = 1 << 22;
    static_assert(int64_t{kMostBlocks} * Short::kThr < int64_t{1} << 32, "threads of a launch");
    const int32_t most = plans->B < kMostBlocks ? plans->B : kMostBlocks;
    auto launch = [&](auto shape) {
        typedef decltype(shape) S;
        ScoreArgs a = make_score_args(tas, ix, any_interval, plans, S::kTab, resident, peak, argmax, score, win_out, win_in);
        a.blk_max = blk_max;
        a.tspan = static_cast<int32_t>(((static_cast<int64_t>(tas->N) + S::kWaves - 1) / S::kWaves + kStage - 1) / kStage * kStage);
        // One workgroup per plan, so that they start as others end; on long rows as many as the device keeps resident (four per
        // CU), the plans dealt evenly among them.  (16,384 plans of 50,000 steps: resident workgroups 2.70 ms, one per plan 2.59;
        // 4,096 of 6,000 steps 167 and 159 us with evaluation; 1,024 of 10^6 steps 2.08 and 2.16 ms.)
        int32_t blocks = most;
        if constexpr (std::is_same<S, Long>::value) {
            const int64_t resident_blocks = 4 * static_cast<int64_t>(tas->num_cus), rounds = (plans->B + resident_blocks - 1) / resident_blocks;
            blocks = static_cast<int32_t>((plans->B + rounds - 1) / rounds);
        }
        if (const int v = g_tuning.score_blocks; v > 0)   // tuning knob: size of the grid (plans are dealt round-robin)
            blocks = v < most ? v : most;
        const dim3 grid(blocks), block(S::kThr);
        if (blk_max) {
            if (vec16) hipLaunchKernelGGL((score_kernel<S, true, true>), grid, block, 0, ws.stream, a);
            else hipLaunchKernelGGL((score_kernel<S, false, true>), grid, block, 0, ws.stream, a);
        } else if constexpr (!std::is_same<S, Small>::value) {     // (Small: with the maxima given only)
            if (vec16) hipLaunchKernelGGL((score_kernel<S, true, false>), grid, block, 0, ws.stream, a);
            else hipLaunchKernelGGL((score_kernel<S, false, false>), grid, block, 0, ws.stream, a);
        }
    };
    const int forced = g_tuning.score_wide;               // tuning knob: 0 / 1 = never / always the large workgroups
    const bool little = tas->N <= Small::kWaves * kStage && tas->T <= 4 * Small::kWaves * kMini;
    if (forced >= 0 ? forced == 1 : plans->B <= tas->num_cus && !little) {
        if (static_cast<int64_t>(plans->B) * tas->T * 8 > kWideStreamBytes) launch(WideStream{});
        else launch(Wide{});
    } else if (blk_max && tas->T <= Small::kTab * kMini) launch(Small{});
    else if (tas->T <= Short::kTab * kMini) launch(Short{});
    else launch(Long{});
    TS_HIP(hipGetLastError());
    return TENSILE_OK;
}

#ifdef TENSILE_SCORE_PROF
extern "C" int tensile_debug_score_prof(unsigned long long *out, int reset) {
    if (out) (void)hipMemcpyFromSymbol(out, HIP_SYMBOL(g_score_prof), sizeof(g_score_prof));
    if (reset) {
        unsigned long long z[16] = {};
        (void)hipMemcpyToSymbol(HIP_SYMBOL(g_score_prof), z, sizeof(z));
    }
    return 0;
}
#endif

}  // namespace tensile

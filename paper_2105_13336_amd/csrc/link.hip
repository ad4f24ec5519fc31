// Occupancy of the host link by the transfers of each plan (section IV-C of the paper, "Swap Event
// Scheduling": data transfers use the PCIe channel exclusively, so only one tensor can be on its way
// at a time; a plan respects that iff no step of its occupancy timeline exceeds one).
//
// A plan stores, for a swap of tensor i, the last resident step o and the step r at which the bytes
// are back.  The transfers are taken in their shortest form: the swap-out ends with step o and
// occupies s..o for the latest s with C[o+1] - C[s] >= x_i, the swap-in ends right before step r and
// occupies s'..r-1 for the latest s' with C[r] - C[s'] >= x_i (C = cumulative operator latency, x_i =
// transfer time; step 0 if the past is too short).  Recomputation intervals use no link.  With host
// copy reuse (section III-C: the copy in host memory stays until the tensor's last access) only the
// earliest swap-out of a tensor within a plan transfers anything.
//
// Two persistent workgroups of 512 threads per CU walk the plans slot, slot + grid, ... (one of 1024 where they are few):
//  * where a transfer that ends with step e begins: most transfers of the sequences of training jobs are shorter than the
//    step they end with, and a byte each says so: the transfer time rounded up and the step's latency rounded down to a
//    common unit.  The others need the last step that starts by the time C[e+1] - x: a table over time (time_step_kernel)
//    brackets it, and C decides between the few steps in the bracket.  Four loads one after the other, however long the
//    transfer and however uneven the latencies.  (Records of the last six latencies per step, one load for transfers of up to
//    six steps and a search through all of C behind them, were as fast on steps of 0.05 to 2 ms and took 20 loads where
//    transfers span tens of steps: 16,384 plans of 4,800 swaps on 50,000 steps of 0.02 to 0.2 ms 3.57 ms, now 1.69; before
//    them a table of 7,167 values of C in LDS took 13 probes for every transfer and kept a second workgroup off the CU.)
//  * the four endpoints of an interval (+1 at s, -1 at o+1, +1 at s', -1 at r) stay in registers, twelve intervals per
//    thread (six with 1024 threads), taken up two at a time with the next two's list entries on their way; a longer plan
//    takes several passes of 6144 intervals, each over all tiles,
//    and the passes add up in the output row (or in a scratch row per workgroup when no rows are
//    wanted): occupancy is additive over the intervals;
//  * per tile of 32,764 steps: scatter into a difference tile in LDS that packs two steps into one 32-bit
//    word (16-bit counters: a pass holds at most 12288 endpoints, so every count and every prefix of
//    counts fits; the adds are done on the whole word, +-1 or +-65536, and the two halves are taken apart
//    after the scatter, which is exact because sums are linear modulo 2^32), barrier; every wavefront sums its
//    part of the tile (one add per word), barrier; then it walks its part 256 steps at a time, four steps per
//    lane: clear, take the halves apart, scan (DPP), reduce (max, earliest argmax, steps occupied twice), and store 16
//    contiguous bytes per lane straight from the registers.  The tile is laid out so that a lane's four steps are
//    16-byte aligned in the plan's output row, whatever T.  The stores are nontemporal: the rows would push the
//    tables out of the L2 (4,096 plans on 24,000 steps 180 -> 147 us);
//  * reuse: the earliest swap-out step per tensor is found in a table in LDS (over the tile, which is
//    idle at that point), 16,384 tensors at a time, for plans of one pass on sequences of up to 65,536
//    tensors, else in one row of N entries per workgroup in global memory, L2 atomics.
// What bounds it: the scattered loads (three per interval at least) and the store of the rows.  Measured with rows of 50,000
// steps, 16,384 plans of 4,800 swaps, steps of 0.05 to 2 ms: 1.46 ms (three or four intervals at a time spill registers).  13
// bytes per interval and 4 per step have to move, 0.78 ms at the rate of a plain kernel; the vector units are busy for
// about as long.  4,096 plans on 6,000 steps 68 us, 256 plans of 60,000 intervals on 10^6 steps 3.9 ms.
#include <type_traits>

#include "common.h"
#include "wave_ops.h"

namespace tensile {

namespace {

constexpr int kCells = 32768;                        // steps the LDS tile has room for
constexpr int kTile = kCells - 4;                    // ... and holds: up to three cells before its first step are unused
constexpr int kTileWords = kCells / 2;               // two 16-bit counters per word: 64 KB
constexpr int kPass = 6144;                          // intervals per pass (at most 2 * kPass endpoints per step: far below 2^15)
constexpr int64_t kMostScratch = int64_t{4} << 30;   // bytes of scratch that two workgroups per CU may take
constexpr int kFirstRounds = 4;                      // reuse: at most this many tables of kTileWords tensors, one after the other
static_assert(2 * kPass < (1 << 15), "16-bit counters");

typedef int i32x4 __attribute__((ext_vector_type(4)));

struct LinkArgs {
    int32_t T, N, B;
    int32_t reuse;
    int64_t n_intervals;
    const int64_t *plan_offsets;
    const int32_t *iv_tensor, *iv_out, *iv_in;
    const uint8_t *iv_kind;        // may be null: every interval is a swap
    const int64_t *C;              // [T+1]
    const int64_t *x;              // [N]
    const uint8_t *lat8, *x8;      // [T], [N] the latencies rounded down and the transfer times rounded up to a common unit
    int32_t search_only;           // (testing aid) the bytes are not used
    const int32_t *time_step;      // the steps under way at the times k << time_shift
    int32_t time_shift;
    int32_t *first_out;            // [grid][N], INT32_MAX everywhere between plans (reuse only)
    int32_t *acc_rows;             // [grid][T] scratch rows for plans of several passes when link == null
    int32_t *link;                 // [B*T] or null
    int32_t *peak, *argmax, *overbooked;   // [B]; the last two may be null
};

// inclusive add-scan over the 64 lanes (32-bit)
__device__ __forceinline__ int32_t wave_scan_add32(int32_t x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, true);
    return x;
}

// Phase timing for tuning, compiled in with -DTENSILE_LINK_PROF only: thread 0 of every workgroup adds the
// 100 MHz ticks it spent in each phase to g_link_prof.
#ifdef TENSILE_LINK_PROF
__device__ unsigned long long g_link_prof[8];
#define LINK_MARK(k)                                              \
    do {                                                          \
        if (threadIdx.x == 0) {                                   \
            const unsigned long long now_ = wall_clock64();       \
            atomicAdd(&g_link_prof[k], now_ - prof_t);            \
            prof_t = now_;                                        \
        }                                                         \
    } while (0)
#else
#define LINK_MARK(k) do { } while (0)
#endif

// kNear: rows of at most 65,534 steps, whose endpoints are kept in 16 bits each.
// kThr: 512, two workgroups per CU, or 1024 and one, mostly for batches of no more plans than CUs, which would leave half of every CU idle
// (256 plans of 60,000 intervals on 10^6 steps: 33 ms with 512 threads and passes added up step by step; 3.96 with 1024 and
// passes added up 16 bytes at a time).
template <int kThr, bool kNear>
__global__ __launch_bounds__(kThr) __attribute__((amdgpu_waves_per_eu(4, 4))) void link_kernel(const LinkArgs a) {
    constexpr int kWaves = kThr / 64, kR = kPass / kThr;   // intervals per thread and pass
    constexpr int kBatch = 2, kBatches = kR / kBatch;      // ... and taken up together
    // the difference tile; between two plans also the table of the earliest swap-out step per tensor (host copy reuse)
    __shared__ __attribute__((aligned(16))) uint32_t delta[kTileWords];
    int32_t *const first_lds = reinterpret_cast<int32_t *>(delta);
    __shared__ int32_t wave_tot[kWaves];
    __shared__ int32_t red_mx[kWaves], red_arg[kWaves], red_over[kWaves];

    for (int u = threadIdx.x; u < kTileWords; u += kThr) delta[u] = 0;
    __syncthreads();

    // C[k] through the uniform base and a 32-bit byte offset (the host keeps T below 2^28): no 64-bit
    // address per probe
    auto c_at = [&](uint32_t k) { return *reinterpret_cast<const int64_t *>(reinterpret_cast<const char *>(a.C) + k * 8u); };
    int32_t *first_out = (a.reuse && a.first_out) ? a.first_out + static_cast<int64_t>(blockIdx.x) * a.N : nullptr;

#ifdef TENSILE_LINK_PROF
    unsigned long long prof_t = wall_clock64();
#endif
    for (int64_t plan = blockIdx.x; plan < a.B; plan += gridDim.x) {
        LINK_MARK(0);
        // the per-lane numbers, derived afresh for every plan from a copy of the thread id that the compiler
        // cannot trace back: otherwise dozens of values computed from it are kept (and spilled) across the kernel
        int tid_now = threadIdx.x;
        asm volatile("" : "+v"(tid_now));
        const int tid = tid_now, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        // (the offsets through the constant address space, i.e. the scalar unit: as a vector load they would queue
        // behind the row stores of the plan before, and the interval loads depend on them)
        typedef const int64_t __attribute__((address_space(4))) *const_i64_ptr;
        int64_t k0 = ((const_i64_ptr)a.plan_offsets)[plan], k1 = ((const_i64_ptr)a.plan_offsets)[plan + 1];
        if (k0 < 0) k0 = 0;
        if (k1 > a.n_intervals) k1 = a.n_intervals;
        if (k1 < k0) k1 = k0;
        auto is_swap = [&](int32_t i, int32_t o, int32_t r, uint32_t kind) {   // an applicable swap interval?
            return kind == 0 && static_cast<uint32_t>(i) < static_cast<uint32_t>(a.N) && o >= 0 && r <= a.T && r > o;
        };
        const int64_t n_pass = k1 > k0 ? (k1 - k0 + kPass - 1) / kPass : 1;
        // Host copy reuse needs the earliest swap-out step of every tensor of the plan: in LDS for a plan of one pass
        // (`uncharged`: one bit per interval of this thread whose swap-out transfers nothing), else in global memory, with L2 atomics.
        const bool reuse_lds = a.reuse && a.N <= kFirstRounds * kTileWords && n_pass == 1;   // (block-uniform)
        uint32_t uncharged = 0;
        if (a.reuse && !reuse_lds) {
            for (int64_t k = k0 + tid; k < k1; k += kThr) {
                const int32_t i = a.iv_tensor[k], o = a.iv_out[k];
                if (is_swap(i, o, a.iv_in[k], a.iv_kind ? a.iv_kind[k] : 0)) atomicMin(&first_out[i], o);
            }
            __threadfence();   // the minima are in L2 before anyone reads them
            __syncthreads();
        } else if (a.reuse && k1 > k0) {
            int32_t i[kR], o[kR];
            const uint32_t len = static_cast<uint32_t>(k1 - k0);
#pragma unroll
            for (int j = 0; j < kR; ++j) {
                const uint32_t k = j * kThr + tid;
                const int64_t kc = k0 + (k < len ? k : 0);
                i[j] = a.iv_tensor[kc];
                o[j] = a.iv_out[kc];
                const int32_t r = a.iv_in[kc];
                const uint32_t kind = a.iv_kind ? a.iv_kind[kc] : 0;
                if (k >= len || !is_swap(i[j], o[j], r, kind)) i[j] = -1;
            }
            for (int32_t base = 0; base < a.N; base += kTileWords) {
                // only the entries this plan touches are set up, and put back to zero afterwards: the rest of the
                // tile is zero already (the scan clears what it reads)
                auto mine = [&](int j) { return static_cast<uint32_t>(i[j] - base) < static_cast<uint32_t>(kTileWords) && i[j] >= 0; };
#pragma unroll
                for (int j = 0; j < kR; ++j)
                    if (mine(j)) first_lds[i[j] - base] = INT32_MAX;
                __syncthreads();
#pragma unroll
                for (int j = 0; j < kR; ++j)
                    if (mine(j)) atomicMin(&first_lds[i[j] - base], o[j]);
                __syncthreads();
#pragma unroll
                for (int j = 0; j < kR; ++j)
                    if (mine(j) && first_lds[i[j] - base] != o[j]) uncharged |= 1u << j;
                __syncthreads();
#pragma unroll
                for (int j = 0; j < kR; ++j)
                    if (mine(j)) first_lds[i[j] - base] = 0;
                __syncthreads();
            }
        }
        int32_t *row = a.link ? a.link + plan * a.T : nullptr;
        // where the passes add up: the output row, else this workgroup's scratch row
        int32_t *acc = row ? row : (n_pass > 1 ? a.acc_rows + static_cast<int64_t>(blockIdx.x) * a.T : nullptr);
        // cells before a tile's first step, so that four cells that one lane takes are 16-byte aligned in the row
        const int32_t pad = acc ? static_cast<int32_t>((reinterpret_cast<uintptr_t>(acc) >> 2) & 3) : 0;
        int32_t best_mx = -1, best_arg = 0, over = 0;   // (over: wave-uniform)

        for (int64_t pass = 0; pass < n_pass; ++pass) {
            const bool only = n_pass == 1, first = pass == 0, last = pass == n_pass - 1;
            // ---- this pass's intervals: their endpoints (steps), UINT32_MAX = none.
            typedef typename std::conditional<kNear, uint16_t, uint32_t>::type Step;
            constexpr int kWords = kNear ? 2 : 4;        // registers of an interval's endpoints: s and o + 1, s' and r
            constexpr uint32_t kNone = static_cast<Step>(~Step(0));
            uint32_t e[kR][kWords];
            int32_t lo_t = INT32_MAX, hi_t = -1;
            const int64_t kb = k0 + pass * kPass;
            const uint32_t len = k1 - kb < kPass ? static_cast<uint32_t>(k1 - kb) : kPass;   // (0 only for an empty plan)
            // a batch of kBatch intervals per thread: its list entries (lanes side by side: every load is whole
            // lines) are requested a batch ahead, at clamped places
            int32_t in_i[kBatch], in_o[kBatch], in_r[kBatch];
            uint32_t in_kind[kBatch];
            auto request = [&](int b) {
#pragma unroll
                for (int j = 0; j < kBatch; ++j) {
                    const uint32_t k = (b * kBatch + j) * kThr + tid;
                    const int64_t kc = kb + (k < len ? k : 0);
                    in_i[j] = a.iv_tensor[kc];
                    in_o[j] = a.iv_out[kc];
                    in_r[j] = a.iv_in[kc];
                    in_kind[j] = a.iv_kind ? a.iv_kind[kc] : 0;
                }
            };
#pragma unroll
            for (int j = 0; j < kR; ++j) {
#pragma unroll
                for (int q = 0; q < kWords; ++q) e[j][q] = UINT32_MAX;
            }
            if (len > 0) request(0);
#pragma unroll
            for (int b = 0; b < kBatches; ++b) {
                if (static_cast<uint32_t>(b) * (kBatch * kThr) >= len) break;       // (block-uniform)
                int32_t iv_i[kBatch], iv_o[kBatch], iv_r[kBatch];
                bool ok[kBatch];
#pragma unroll
                for (int j = 0; j < kBatch; ++j) {
                    const uint32_t k = (b * kBatch + j) * kThr + tid;
                    ok[j] = k < len && is_swap(in_i[j], in_o[j], in_r[j], in_kind[j]);
                    iv_i[j] = ok[j] ? in_i[j] : 0;       // (harmless stand-ins for the loads below)
                    iv_o[j] = ok[j] ? in_o[j] : 0;
                    iv_r[j] = ok[j] ? in_r[j] : 1;
                }
                // the step the transfer ends with, then the one it starts with
                int32_t at[kBatch][2];
                uint32_t x8[kBatch], l8[kBatch][2];
#pragma unroll
                for (int j = 0; j < kBatch; ++j) {
                    at[j][0] = iv_o[j];
                    at[j][1] = iv_r[j] - 1;
                    x8[j] = a.x8[iv_i[j]];
                    l8[j][0] = a.lat8[at[j][0]];
                    l8[j][1] = a.lat8[at[j][1]];
                }
                bool charged[kBatch];
#pragma unroll
                for (int j = 0; j < kBatch; ++j) {
                    charged[j] = !((uncharged >> (b * kBatch + j)) & 1u);
                    if (a.reuse && !reuse_lds)
                        charged[j] = __hip_atomic_load(&first_out[iv_i[j]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == iv_o[j];
                }
                if (b + 1 < kBatches && static_cast<uint32_t>(b + 1) * (kBatch * kThr) < len) request(b + 1);
                LINK_MARK(1);
                // a transfer no longer than the step it ends with starts there
                bool open[kBatch][2], any_open = false;
#pragma unroll
                for (int j = 0; j < kBatch; ++j) {
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        open[j][q] = ok[j] && (x8[j] > l8[j][q] || a.search_only);
                        any_open = any_open || open[j][q];
                    }
                }
                if (__builtin_amdgcn_ballot_w64(any_open) != 0) {
                    // the others with the last step s with C[s] <= v = C[end + 1] - x (step 0 when there is none): one of those
                    // under way between the times before and after v in the table, the wavefront's searches in lockstep
                    int64_t v[kBatch][2];
                    int32_t lo[kBatch][2], hi[kBatch][2];
#pragma unroll
                    for (int j = 0; j < kBatch; ++j) {
                        const int64_t x = open[j][0] || open[j][1] ? a.x[iv_i[j]] : 0;
#pragma unroll
                        for (int q = 0; q < 2; ++q) v[j][q] = (open[j][q] ? c_at(static_cast<uint32_t>(at[j][q]) + 1) : 0) - x;
                    }
#pragma unroll
                    for (int j = 0; j < kBatch; ++j) {
#pragma unroll
                        for (int q = 0; q < 2; ++q) {
                            const int64_t k = v[j][q] > 0 ? v[j][q] >> a.time_shift : 0;
                            lo[j][q] = hi[j][q] = 0;
                            if (open[j][q]) {
                                lo[j][q] = a.time_step[k];
                                hi[j][q] = a.time_step[k + 1];
                            }
                        }
                    }
                    for (;;) {
                        bool unsure = false;
#pragma unroll
                        for (int j = 0; j < kBatch; ++j) unsure = unsure || lo[j][0] < hi[j][0] || lo[j][1] < hi[j][1];
                        if (__builtin_amdgcn_ballot_w64(unsure) == 0) break;
                        int32_t mid[kBatch][2];
                        int64_t c[kBatch][2];
#pragma unroll
                        for (int j = 0; j < kBatch; ++j) {
#pragma unroll
                            for (int q = 0; q < 2; ++q) {
                                mid[j][q] = lo[j][q] + ((hi[j][q] - lo[j][q] + 1) >> 1);
                                c[j][q] = lo[j][q] < hi[j][q] ? c_at(static_cast<uint32_t>(mid[j][q])) : 0;
                            }
                        }
#pragma unroll
                        for (int j = 0; j < kBatch; ++j) {
#pragma unroll
                            for (int q = 0; q < 2; ++q) {
                                if (lo[j][q] < hi[j][q]) {
                                    if (c[j][q] <= v[j][q]) lo[j][q] = mid[j][q];
                                    else hi[j][q] = mid[j][q] - 1;
                                }
                            }
                        }
                    }
#pragma unroll
                    for (int j = 0; j < kBatch; ++j) {
#pragma unroll
                        for (int q = 0; q < 2; ++q)
                            if (open[j][q]) at[j][q] = lo[j][q];
                    }
                }
#pragma unroll
                for (int j = 0; j < kBatch; ++j) {
                    if (ok[j]) {
                        uint32_t (&out)[kWords] = e[b * kBatch + j];
                        auto put = [&](int q, int32_t from, int32_t to) {
                            if constexpr (kNear) {
                                out[q] = static_cast<uint32_t>(from) | (static_cast<uint32_t>(to) << 16);
                            } else {
                                out[2 * q] = static_cast<uint32_t>(from);
                                out[2 * q + 1] = static_cast<uint32_t>(to);
                            }
                        };
                        if (charged[j]) {
                            put(0, at[j][0], iv_o[j] + 1);
                            lo_t = at[j][0] < lo_t ? at[j][0] : lo_t;
                        }
                        put(1, at[j][1], iv_r[j]);
                        lo_t = at[j][1] < lo_t ? at[j][1] : lo_t;
                        hi_t = iv_r[j] > hi_t ? iv_r[j] : hi_t;
                    }
                }
                LINK_MARK(2);
            }

            int32_t carry = 0;
            for (int32_t tile_lo = 0; tile_lo < a.T; tile_lo += kTile) {
                const int32_t tile_hi = a.T - tile_lo < kTile ? a.T : tile_lo + kTile;
                const uint32_t tile_n = static_cast<uint32_t>(tile_hi - tile_lo);
                // ---- scatter (a wavefront none of whose lanes has an endpoint in range skips it)
                const bool mine = hi_t >= tile_lo && lo_t < tile_hi;
                if (__builtin_amdgcn_ballot_w64(mine) != 0) {
#pragma unroll
                    for (int j = 0; j < kR; ++j) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const uint32_t step = kNear ? (q & 1 ? e[j][q / 2] >> 16 : e[j][q / 2] & kNone) : e[j][kNear ? 0 : q];
                            const uint32_t u = step - static_cast<uint32_t>(tile_lo), cell = u + static_cast<uint32_t>(pad);
                            const uint32_t one = (q & 1) ? 0xffffffffu : 1u;          // -1 or +1 ...
                            if (u < tile_n) atomicAdd(&delta[cell >> 1], one << (16 * (cell & 1)));   // ... on the cell's half
                        }
                    }
                }
                __syncthreads();
                LINK_MARK(3);
                // ---- the wavefront's part: 256 cells at a time, four per lane
                const int32_t n_cells = static_cast<int32_t>(tile_n) + pad;
                const int32_t part = (n_cells + kWaves * 256 - 1) / (kWaves * 256) * 256;
                const int32_t u_lo = wave * part, u_hi = min(u_lo + part, n_cells);
                typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
                {
                    uint32_t s = 0;      // both halves of the words at once: neither sum leaves 16 bits
                    for (int32_t u = u_lo; u < u_hi; u += 256) {
                        const u32x2 c = *reinterpret_cast<const u32x2 *>(&delta[(u >> 1) + 2 * lane]);
                        s += c[0] + c[1];
                    }
                    const int32_t lo = static_cast<int16_t>(s & 0xffffu);
                    const int32_t incl = wave_scan_add32(lo + (static_cast<int32_t>(s - static_cast<uint32_t>(lo)) >> 16));
                    if (lane == 63) wave_tot[wave] = incl;
                }
                __syncthreads();
                LINK_MARK(4);
                int32_t run = carry;     // occupancy before the part's next cell (wave-uniform)
#pragma unroll
                for (int w = 0; w < kWaves; ++w) {
                    const int32_t t = __builtin_amdgcn_readfirstlane(wave_tot[w]);
                    run += w < wave ? t : 0;
                    carry += t;
                }
                for (int32_t u = u_lo; u < u_hi; u += 256) {
                    u32x2 *cell = reinterpret_cast<u32x2 *>(&delta[(u >> 1) + 2 * lane]);
                    const u32x2 c = *cell;
                    *cell = u32x2{0, 0};
                    int32_t v[4];
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const int32_t lo = static_cast<int16_t>(c[h] & 0xffffu);
                        v[2 * h] = lo;
                        v[2 * h + 1] = static_cast<int32_t>(c[h] - static_cast<uint32_t>(lo)) >> 16;
                    }
#pragma unroll
                    for (int j = 1; j < 4; ++j) v[j] += v[j - 1];
                    const int32_t incl = wave_scan_add32(v[3]);
                    const int32_t before = run + incl - v[3];
#pragma unroll
                    for (int j = 0; j < 4; ++j) v[j] += before;
                    run += __builtin_amdgcn_readlane(incl, 63);
                    const int32_t t0 = tile_lo - pad + u + 4 * lane;      // (below tile_lo only in the tile's first cells)
                    if (u >= pad && u + 256 <= n_cells) {                 // (uniform) all of the 256 steps exist
                        if (!only) {         // passes of a long plan add up, each step in one lane's hands
                            i32x4 *const sum = reinterpret_cast<i32x4 *>(acc + t0);
                            if (!first) {
                                const i32x4 c4 = *sum;
#pragma unroll
                                for (int j = 0; j < 4; ++j) v[j] += c4[j];
                            }
                            if (!last) {
                                *sum = i32x4{v[0], v[1], v[2], v[3]};
                                continue;
                            }
                        }
                        const int32_t m = max(max(v[0], v[1]), max(v[2], v[3]));
                        if (__builtin_amdgcn_ballot_w64(m > best_mx) != 0) {
                            if (m > best_mx) {
                                best_mx = m;
                                best_arg = t0 + (v[0] == m ? 0 : v[1] == m ? 1 : v[2] == m ? 2 : 3);
                            }
                        }
#pragma unroll
                        for (int j = 0; j < 4; ++j) over += __builtin_popcountll(__builtin_amdgcn_ballot_w64(v[j] >= 2));
                        if (row) __builtin_nontemporal_store(i32x4{v[0], v[1], v[2], v[3]}, reinterpret_cast<i32x4 *>(row + t0));
                        continue;
                    }
                    bool in[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) in[j] = t0 + j >= tile_lo && t0 + j < tile_hi;
                    if (!only) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            if (!first && in[j]) v[j] += acc[t0 + j];
                            if (!last && in[j]) acc[t0 + j] = v[j];
                        }
                        if (!last) continue;   // (block-uniform)
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if (in[j] && v[j] > best_mx) {
                            best_mx = v[j];
                            best_arg = t0 + j;
                        }
                        over += __builtin_popcountll(__builtin_amdgcn_ballot_w64(in[j] && v[j] >= 2));
                        if (row && in[j]) row[t0 + j] = v[j];
                    }
                }
                __syncthreads();       // every part is clear again before the next scatter
                LINK_MARK(5);
            }
        }

        // ---- the plan's result
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            const int32_t omx = __shfl_xor(best_mx, d, 64), oarg = __shfl_xor(best_arg, d, 64);
            if (omx > best_mx || (omx == best_mx && oarg < best_arg)) {
                best_mx = omx;
                best_arg = oarg;
            }
        }
        if (lane == 0) {
            red_mx[wave] = best_mx;
            red_arg[wave] = best_arg;
            red_over[wave] = over;
        }
        if (a.reuse && !reuse_lds) {   // leave the table as it was found
            for (int64_t k = k0 + tid; k < k1; k += kThr) {
                const int32_t i = a.iv_tensor[k], o = a.iv_out[k];
                if (is_swap(i, o, a.iv_in[k], a.iv_kind ? a.iv_kind[k] : 0))
                    __hip_atomic_store(&first_out[i], INT32_MAX, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            __threadfence();   // ... before the next plan's minima arrive
        }
        __syncthreads();
        if (tid == 0) {
            int32_t mx = red_mx[0], arg = red_arg[0], ov = red_over[0];
#pragma unroll
            for (int w = 1; w < kWaves; ++w) {
                if (red_mx[w] > mx || (red_mx[w] == mx && red_arg[w] < arg)) {
                    mx = red_mx[w];
                    arg = red_arg[w];
                }
                ov += red_over[w];
            }
            a.peak[plan] = mx;
            if (a.argmax) a.argmax[plan] = arg;
            if (a.overbooked) a.overbooked[plan] = ov;
        }
        // (red_* are written again only after the barriers of the next plan's tiles)
    }
}

// Without latencies nothing is transferred in measurable time: every output is zero.
__global__ void link_zero_kernel(int64_t n_rows, int32_t *link, int32_t B, int32_t *peak, int32_t *argmax, int32_t *overbooked) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t k = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; k < n_rows; k += stride) link[k] = 0;
    for (int64_t k = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; k < B; k += stride) {
        peak[k] = 0;
        if (argmax) argmax[k] = 0;
        if (overbooked) overbooked[k] = 0;
    }
}

__global__ void link_fill_kernel(int32_t *p, int64_t n, int32_t v) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t k = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; k < n; k += stride) p[k] = v;
}

}  // namespace

int launch_link(const tensile_tas *tas, Workspace &ws, const tensile_plans *plans, bool reuse, int32_t *link, int32_t *peak,
                int32_t *argmax, int32_t *overbooked) {
    const hipStream_t stream = ws.stream;
    const int32_t B = plans->B, T = tas->T;
    if (B == 0) return TENSILE_OK;
    if (T > kLinkMostSteps) { set_error("eval_link: T = %d exceeds 2^28 steps", T); return TENSILE_E_RANGE; }
    if (!tas->timed || tas->N == 0) {
        const int64_t n_rows = link ? static_cast<int64_t>(B) * T : 0;
        hipLaunchKernelGGL(link_zero_kernel, dim3(tas->num_cus * 4), dim3(256), 0, stream, n_rows, link, B, peak, argmax, overbooked);
        TS_HIP(hipGetLastError());
        return TENSILE_OK;
    }
    LinkArgs a{};
    a.T = T; a.N = tas->N; a.B = B; a.reuse = reuse ? 1 : 0;
    a.n_intervals = plans->n_intervals;
    a.plan_offsets = plans->plan_offsets;
    a.iv_tensor = plans->iv_tensor; a.iv_out = plans->iv_out; a.iv_in = plans->iv_in; a.iv_kind = plans->iv_kind;
    a.C = tas->d_C.p; a.x = tas->d_x.p;
    a.lat8 = tas->d_lat8.p; a.x8 = tas->d_x8.p;
    a.search_only = g_tuning.link_packed == 0 ? 1 : 0;   // (testing aid)
    a.time_step = tas->d_time_step.p; a.time_shift = tas->time_shift;
    // scratch per workgroup: the table of plans that the kernel cannot serve from LDS (see reuse_lds there), and the row where
    // the passes of a long plan add up
    const bool needs_first = reuse && (tas->N > kFirstRounds * kTileWords || plans->n_intervals > kPass);
    const bool needs_acc = !link && plans->n_intervals > kPass;
    const int64_t per_group = 4 * ((needs_first ? int64_t{tas->N} : 0) + (needs_acc ? int64_t{T} : 0));
    // One large workgroup per CU when there are no more plans than that - and when the scratch of two per CU would be out of
    // proportion (rows of more than two million steps): a plan is many tiles then, and one workgroup per CU takes plans as
    // fast as two (60,000 intervals on 10^6 steps: 256 plans in one round 3.79 ms, 1,024 with two per CU 15.2).
    const bool wide = B <= tas->num_cus || 2 * tas->num_cus * per_group > kMostScratch;
    const int32_t slots = wide ? tas->num_cus : 2 * tas->num_cus, grid = B < slots ? B : slots;
    if (needs_first) {
        const size_t need = static_cast<size_t>(grid) * static_cast<size_t>(tas->N);
        bool fresh = false;
        const int rc = ws.provide(ws.link_first, need, "eval_link: earliest swap-out table", &fresh);
        if (rc != TENSILE_OK) return rc;
        if (fresh) {   // (the kernel leaves the table as it found it)
            hipLaunchKernelGGL(link_fill_kernel, dim3(tas->num_cus * 4), dim3(256), 0, stream, ws.link_first.p,
                               static_cast<int64_t>(ws.link_first.n), INT32_MAX);
            TS_HIP(hipGetLastError());
        }
        a.first_out = ws.link_first.p;
    }
    if (needs_acc) {   // some plan may need several passes
        const size_t need = static_cast<size_t>(grid) * static_cast<size_t>(T);
        const int rc = ws.provide(ws.link_acc, need, "eval_link: accumulation rows");
        if (rc != TENSILE_OK) return rc;
        a.acc_rows = ws.link_acc.p;
    }
    a.link = link; a.peak = peak; a.argmax = argmax; a.overbooked = overbooked;
    const bool near = T <= 65534;
    auto launch = [&](auto thr) {
        constexpr int kThr = decltype(thr)::value;
        if (near) hipLaunchKernelGGL((link_kernel<kThr, true>), dim3(grid), dim3(kThr), 0, stream, a);
        else hipLaunchKernelGGL((link_kernel<kThr, false>), dim3(grid), dim3(kThr), 0, stream, a);
    };
    if (wide) launch(std::integral_constant<int, 1024>{});
    else launch(std::integral_constant<int, 512>{});
    TS_HIP(hipGetLastError());
    return TENSILE_OK;
}

#ifdef TENSILE_LINK_PROF
extern "C" int tensile_debug_link_prof(unsigned long long *out, int reset) {
    if (out) (void)hipMemcpyFromSymbol(out, HIP_SYMBOL(g_link_prof), sizeof(g_link_prof));
    if (reset) {
        unsigned long long z[8] = {};
        (void)hipMemcpyToSymbol(HIP_SYMBOL(g_link_prof), z, sizeof(z));
    }
    return 0;
}
#endif

}  // namespace tensile

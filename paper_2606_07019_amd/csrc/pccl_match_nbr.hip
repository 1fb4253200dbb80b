// The event-stepped chunk-to-link matching with neighbour-only
// synchronisation: the kernel of every network whose devices each fit one
// wavefront.
//
// Semantics are those of the windowed matcher (pccl_match.hip): at every
// event time links whose transfer ends deliver and become free, every free
// link s->d picks the highest-priority chunk held by s and still needed by d,
// picks of one chunk into one device clash (fastest link, then lowest link
// id, wins), losers pick again, time advances to the next transfer end.
//
// What bounds this work is latency: thousands of dependent steps, each a few
// hundred bytes.  Two things make a step short here.
//
//  1. No grid-wide exchange.  Time is cut into windows [k Tmin, (k+1) Tmin)
//     of the smallest link time.  A transfer started in a window ends after
//     it, so device d can run its events of window k as soon as it knows the
//     transfers that were in flight into the sources of its in-links when
//     window k began: the state of its in-neighbours' in-links, nobody
//     else's.  Each wave publishes one 64-bit entry per in-link and window
//     (tag, chunk, end time); the entry carries its own window number, so a
//     reader polls the very words it needs, and the data arrives with the
//     synchronisation: one store and one load between two dependent windows
//     (0.9 us measured between compute units of different XCDs), where the
//     exchange of all workgroups, the wait for the stores before it and the
//     loads of the entries after it took three round trips, and the slowest
//     wave of the whole grid set the pace of every window.
//     Four copies of the entries alternate by window: before d overwrites
//     the entry of window k - 4 it has seen every reader at window k - 3.
//  2. No scans and no memory accesses inside a window.  Column i of
//     destination d is the i-th chunk d needs, in priority order.  Every
//     in-link keeps its candidates (held by its source, needed by d) as a
//     bit set over d's columns with one or two summary levels, in LDS; an
//     arrival at the source sets a bit.  The best candidate of every link is
//     two or three dependent LDS reads away, for all links at once.  A
//     delivered column is cleared once, in the `live` set that masks every
//     row; rows are not updated, a row word without live bits is dropped
//     from the summary when a pick meets it.
//
// A device with many columns (a switch that relays a large part of the
// chunks) leaves its candidate rows, its chunk table or its column table in
// device memory when they do not fit its share of LDS; the live set and the
// summaries always fit (the host checks the bound).
#include "pccl_internal.h"

namespace pccl {
namespace {

constexpr uint32_t NBR_THREADS = MATCH_THREADS;
constexpr uint32_t NBR_WAVES = NBR_THREADS / 64;
constexpr uint32_t NBR_SPIN_LIMIT = 1u << 24;

// Published entry of an in-link: bit 63 the device is finished (the entry
// holds for every later window), 12 bits window tag, 19 bits chunk rank
// (NBR_IDLE: no transfer in flight), 32 bits end time.
constexpr uint32_t NBR_IDLE = (1u << 19) - 1u;
static_assert(NBR_MAX_CHUNKS < NBR_IDLE, "a chunk rank and the idle mark fit in 19 bits");
constexpr uint64_t NBR_FINAL = 1ull << 63;

__device__ __forceinline__ uint64_t nbr_tag(uint32_t k) { return (uint64_t)(k & 0xFFFu) << 51; }
constexpr uint64_t NBR_TAG_MASK = 0xFFFull << 51;

template <class Op>
__device__ __forceinline__ uint32_t dpp_reduce(uint32_t v, uint32_t id, Op op)
{
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)id, (int)v, 0xb1, 0xf, 0xf, false));   // quad_perm 1,0,3,2
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)id, (int)v, 0x4e, 0xf, 0xf, false));   // quad_perm 2,3,0,1
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)id, (int)v, 0x114, 0xf, 0xf, false));  // row_shr 4
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)id, (int)v, 0x118, 0xf, 0xf, false));  // row_shr 8
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)id, (int)v, 0x142, 0xa, 0xf, false));  // row_bcast 15
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)id, (int)v, 0x143, 0xc, 0xf, false));  // row_bcast 31
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

struct MinOp { __device__ uint32_t operator()(uint32_t a, uint32_t b) const { return min(a, b); } };
struct MaxOp { __device__ uint32_t operator()(uint32_t a, uint32_t b) const { return max(a, b); } };
struct AddOp { __device__ uint32_t operator()(uint32_t a, uint32_t b) const { return a + b; } };

__device__ __forceinline__ uint32_t lane_prefix(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Position of the lowest set bit of a non-zero word.
__device__ __forceinline__ uint32_t low_bit(uint64_t x) { return (uint32_t)__builtin_ctzll(x); }

extern __shared__ __attribute__((aligned(16))) unsigned char nbr_lds[];

// One destination's tables: byte offsets into the workgroup's LDS, and the
// device memory of those that did not fit there (`in_lds` says which did).
constexpr uint32_t IN_ROW = 1, IN_NEED = 2, IN_RANK = 4;
struct Tables {
    uint32_t live_at, top_at, mid_at, row_at, need_at, pre_at, rank_at;
    uint32_t ms, rs;        // strides of mid and row
    uint32_t in_lds;
    uint64_t *g_row;        // [n * mw] candidate rows
    const uint64_t *g_need; // [W] the columns as a chunk bitmap
    const uint32_t *g_pre;  // [W] columns before each word
    const uint32_t *g_rank; // [M] chunk rank of each column

    // [mw] columns still needed
    __device__ uint64_t *live() const { return reinterpret_cast<uint64_t *>(nbr_lds + live_at); }
    // [n] per in-link: which mid words (L3) or row words hold candidates
    __device__ uint64_t *top() const { return reinterpret_cast<uint64_t *>(nbr_lds + top_at); }
    // [n * ms] per in-link: which row words hold candidates (L3 only)
    __device__ uint64_t *mid() const { return reinterpret_cast<uint64_t *>(nbr_lds + mid_at); }
    __device__ uint64_t *row() const { return reinterpret_cast<uint64_t *>(nbr_lds + row_at); }
    __device__ uint64_t *need() const { return reinterpret_cast<uint64_t *>(nbr_lds + need_at); }
    __device__ uint16_t *pre() const { return reinterpret_cast<uint16_t *>(nbr_lds + pre_at); }
    __device__ uint32_t *rank() const { return reinterpret_cast<uint32_t *>(nbr_lds + rank_at); }
    __device__ uint32_t rank_of(uint32_t col) const { return (in_lds & IN_RANK) ? rank()[col] : g_rank[col]; }
};

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The lowest live candidate column of this lane's in-link, NONE32 if none.
// `want`: the lane's link is free.  A row word none of whose bits is live any
// more leaves the summaries.
template <bool L3>
__device__ __forceinline__ uint32_t first_live(const Tables &tb, bool want, uint32_t &words)
{
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t col = NONE32;
    uint64_t tp = want ? tb.top()[lane] : 0ull;
    while (__ballot(tp != 0ull)) {
        if (tp) {
            uint32_t w = low_bit(tp);
            uint64_t m = 0;
            if (L3) {
                m = tb.mid()[lane * tb.ms + w];
                w = w * 64u + low_bit(m);
            }
            uint64_t x;
            const uint64_t lv = tb.live()[w];
            // (rows in device memory are updated by atomics, which the L1
            // cache does not see: they are read past it)
            if (tb.in_lds & IN_ROW) x = tb.row()[lane * tb.rs + w];
            else x = __hip_atomic_load(&tb.g_row[(uint64_t)lane * tb.rs + w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            x &= lv;
            words++;
            if (x) {
                col = w * 64u + low_bit(x);
                tp = 0;
            } else {
                if (L3) {
                    m &= m - 1ull;
                    tb.mid()[lane * tb.ms + (w >> 6)] = m;
                }
                if (!L3 || !m) {
                    tp &= tp - 1ull;
                    tb.top()[lane] = tp;
                }
            }
        }
    }
    return col;
}

// PPL: polled entries per lane.  L3: some destination may have more than
// 4,096 columns (two summary levels).
template <uint32_t PPL, bool L3>
__device__ __forceinline__ void run_dest(const Layout &ly, const Sizes &sz, uint32_t d, uint32_t lds_at, uint32_t room)
{
    Control *ctl = ly.ctl;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t base = ly.in_off[d], n = ly.in_off[d + 1] - base;
    const bool mine = lane < n;
    const unsigned long long log0 = ly.dest_log[d];
    const uint32_t M = ly.dest_cols[d], mw = (M + 63u) >> 6, mm = (mw + 63u) >> 6;
    const uint32_t W = (uint32_t)sz.W;

    // this wave's share of LDS
    Tables tb{};
    {
        uint32_t at = lds_at;
        const uint32_t end = lds_at + room;
        auto take = [&](uint32_t bytes) {
            const uint32_t p = at;
            at += (bytes + 7u) & ~7u;
            return p;
        };
        tb.live_at = take(mw * 8u);
        tb.top_at = take(n * 8u);
        tb.ms = mm | 1u;
        if (L3) tb.mid_at = take(n * tb.ms * 8u);
        tb.g_row = ly.cand + ly.cand_off[d];
        tb.g_need = ly.needs + (uint64_t)d * sz.Wp;
        tb.g_pre = ly.need_pre + (uint64_t)d * sz.Wp;
        tb.g_rank = ly.col_rank + log0;
        tb.rs = mw | 1u;
        if (at + n * tb.rs * 8u <= end) {
            tb.in_lds |= IN_ROW;
            tb.row_at = take(n * tb.rs * 8u);
        } else {
            tb.rs = mw;
        }
        if (M <= 0xFFFFu && at + W * 10u + 8u <= end) {
            tb.in_lds |= IN_NEED;
            tb.need_at = take(W * 8u);
            tb.pre_at = take(W * 2u);
            for (uint32_t i = lane; i < W; i += 64) {
                tb.need()[i] = tb.g_need[i];
                tb.pre()[i] = (uint16_t)tb.g_pre[i];
            }
        }
        if (at + M * 4u <= end) {
            tb.in_lds |= IN_RANK;
            tb.rank_at = take(M * 4u);
            for (uint32_t i = lane; i < M; i += 64) tb.rank()[i] = tb.g_rank[i];
        }
        for (uint32_t i = lane; i < mw; i += 64)
            tb.live()[i] = i + 1 < mw || (M & 63u) == 0 ? NONE64 : (1ull << (M & 63u)) - 1ull;
        // rows and summaries, link by link (64 row words give one summary word)
        for (uint32_t j = 0; j < n; j++) {
            uint64_t tsum = 0;
            for (uint32_t g = 0; g < mm; g++) {
                const uint32_t w = g * 64u + lane;
                uint64_t x = 0;
                if (w < mw) {
                    x = tb.g_row[(uint64_t)j * mw + w];
                    if (tb.in_lds & IN_ROW) tb.row()[j * tb.rs + w] = x;
                }
                const uint64_t s = __ballot(x != 0);
                if (L3) {
                    if (lane == 0) tb.mid()[j * tb.ms + g] = s;
                    if (s) tsum |= 1ull << g;
                } else {
                    tsum = s;
                }
            }
            if (lane == 0) tb.top()[j] = tsum;
        }
        wave_sync();
    }
    // this lane's in-link
    uint32_t tim = 0, lid = 0;
    if (mine) {
        tim = ly.slot_time[base + lane];
        lid = ly.slot_link[base + lane];
    }
    // the entries this lane polls: slot << 8 | in-link they feed (0xFF: only
    // the window tag counts, a reader of d that is no source of d)
    const uint32_t p0 = ly.poll_off[d], np = ly.poll_off[d + 1] - p0;
    uint32_t pol[PPL];
#pragma unroll
    for (uint32_t u = 0; u < PPL; u++) pol[u] = np ? ly.poll[p0 + min(64u * u + lane, np - 1u)] : 0u;

    const uint32_t tmin = sz.tmin;
    const uint64_t L = sz.L;
    uint32_t left = M, fin = 0;
    uint32_t busy_end = 0, busy_rank = NBR_IDLE;  // the transfer in flight on this lane's link
    uint32_t cstar = 0, words = 0;
    uint32_t rounds = 0, clashes = 0;
    unsigned long long log = log0;
    uint64_t t0 = 0;
    uint32_t k = 0;
    bool bad = false;
    for (;; k++, t0 += tmin) {
        uint32_t ra[PPL], ca[PPL];  // arrivals of this window: offset into the window (NONE32: none), column
        uint32_t rb = NONE32;       // the end of this lane's transfer when inside the window
#pragma unroll
        for (uint32_t u = 0; u < PPL; u++) {
            ra[u] = NONE32;
            ca[u] = 0;
        }
        if (k) {
            if (np) {
                // sources: the state at the end of window k - 1; readers of d
                // that are no sources: that they have read window k - 4
                const uint64_t *b1 = ly.pub + (uint64_t)((k - 1u) & 3u) * L, *b3 = ly.pub + (uint64_t)((k - 3u) & 3u) * L;
                const uint64_t tag1 = nbr_tag(k - 1u), tag3 = nbr_tag(k - 3u);
                uint64_t e[PPL];
#pragma unroll
                for (uint32_t u = 0; u < PPL; u++) e[u] = 0;
                uint32_t spins = 0;
                while (true) {
                    bool ok = true;
#pragma unroll
                    for (uint32_t u = 0; u < PPL; u++) {
                        if (64u * u >= np) break;
                        const bool dep = (pol[u] & 0xFFu) == 0xFFu;
                        e[u] = __hip_atomic_load((dep ? b3 : b1) + (pol[u] >> 8), __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
                    }
#pragma unroll
                    for (uint32_t u = 0; u < PPL; u++) {
                        if (64u * u >= np) break;
                        const bool dep = (pol[u] & 0xFFu) == 0xFFu;
                        const uint64_t want = dep ? tag3 : tag1;
                        ok = ok && ((int64_t)e[u] < 0 || (e[u] & NBR_TAG_MASK) == want || (dep && k < 3u));
                    }
                    if (__ballot(!ok) == 0) break;
                    // (another wave's error ends the wait; the spin limit turns
                    // a wait that should not happen into an error)
                    if ((++spins & 15u) == 0) {
                        if (__hip_atomic_load(&ctl->error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                            bad = true;
                            break;
                        }
                        if (spins > NBR_SPIN_LIMIT) {
                            if (lane == 0) {
                                atomicExch(&ctl->abort, 1u);
                                record_error(ctl, ST_EINTERNAL, 3, d, k);
                            }
                            bad = true;
                            break;
                        }
                    }
                }
                if (bad) break;
                if (left && !(t0 >> 32)) {
                    // arrivals inside the window, in d's columns, that d still needs
                    bool in[PPL];
                    bool any = false;
                    const uint32_t t032 = (uint32_t)t0;
#pragma unroll
                    for (uint32_t u = 0; u < PPL; u++) in[u] = false;
#pragma unroll
                    for (uint32_t u = 0; u < PPL; u++) {
                        if (64u * u >= np) break;
                        const uint32_t end = (uint32_t)e[u], r = (uint32_t)(e[u] >> 32) & NBR_IDLE;
                        in[u] = 64u * u + lane < np && r != NBR_IDLE && (pol[u] & 0xFFu) != 0xFFu && end >= t032 &&
                                end - t032 < tmin;
                        any = any || in[u];
                    }
                    if (__ballot(any)) {
                        uint64_t nw[PPL];
                        uint32_t pr[PPL];
#pragma unroll
                        for (uint32_t u = 0; u < PPL; u++) {
                            nw[u] = 0;
                            pr[u] = 0;
                            if (in[u]) {
                                const uint32_t w = ((uint32_t)(e[u] >> 32) & NBR_IDLE) >> 6;
                                if (tb.in_lds & IN_NEED) {
                                    nw[u] = tb.need()[w];
                                    pr[u] = tb.pre()[w];
                                } else {
                                    nw[u] = tb.g_need[w];
                                    pr[u] = tb.g_pre[w];
                                }
                            }
                        }
#pragma unroll
                        for (uint32_t u = 0; u < PPL; u++) {
                            const uint32_t b = (uint32_t)(e[u] >> 32) & 63u;
                            if (in[u] && ((nw[u] >> b) & 1ull)) {
                                ca[u] = pr[u] + (uint32_t)__popcll(nw[u] & ((1ull << b) - 1ull));
                                if ((tb.live()[ca[u] >> 6] >> (ca[u] & 63u)) & 1ull) ra[u] = (uint32_t)e[u] - t032;
                            }
                        }
                    }
                }
            }
            if (busy_rank != NBR_IDLE && !(t0 >> 32) && busy_end - (uint32_t)t0 < tmin) rb = busy_end - (uint32_t)t0;
        }

        // events of the window in time order
        uint32_t newcol = NONE32;  // the column this lane's link committed in this window (at most one: Tmin)
        bool first = k == 0;
        while (true) {
            uint32_t m = rb;
#pragma unroll
            for (uint32_t u = 0; u < PPL; u++) m = min(m, ra[u]);
            const uint32_t t = first ? 0u : dpp_reduce(m, NONE32, MinOp());
            if (t == NONE32) break;
            first = false;
            if (rb == t) {
                busy_rank = NBR_IDLE;
                rb = NONE32;
            }
#pragma unroll
            for (uint32_t u = 0; u < PPL; u++) {
                if (ra[u] == t) {
                    const uint32_t j = pol[u] & 0xFFu, w = ca[u] >> 6;
                    const unsigned long long bit = 1ull << (ca[u] & 63u);
                    if (tb.in_lds & IN_ROW) atomicOr((unsigned long long *)&tb.row()[j * tb.rs + w], bit);
                    else __hip_atomic_fetch_or(&tb.g_row[(uint64_t)j * tb.rs + w], (uint64_t)bit, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
                    if (L3) {
                        atomicOr((unsigned long long *)&tb.mid()[j * tb.ms + (w >> 6)], 1ull << (w & 63u));
                        atomicOr((unsigned long long *)&tb.top()[j], 1ull << (w >> 6));
                    } else {
                        atomicOr((unsigned long long *)&tb.top()[j], 1ull << w);
                    }
                    ra[u] = NONE32;
                }
            }
            // pick rounds
            bool want = mine && busy_rank == NBR_IDLE && newcol == NONE32;
            while (true) {
                const uint32_t col = first_live<L3>(tb, want, words);
                const bool act = col != NONE32;
                if (__ballot(act) == 0) break;
                // clear the picked columns; a lane that finds its column
                // already cleared shares it with another lane
                uint64_t old = 0;
                if (act) old = atomicAnd((unsigned long long *)&tb.live()[col >> 6], ~(1ull << (col & 63u)));
                bool win = act && ((old >> (col & 63u)) & 1ull);
                uint64_t clash = __ballot(act && !win);
                uint64_t losers = clash;
                if (clash) {
                    // fastest link, then lowest id, among the links that picked the column
                    while (clash) {
                        const uint32_t v = (uint32_t)__builtin_amdgcn_readlane((int)col, __builtin_ctzll(clash));
                        const bool in_g = act && col == v;
                        const uint64_t g = __ballot(in_g);
                        const uint32_t tm = dpp_reduce(in_g ? tim : NONE32, NONE32, MinOp());
                        const uint32_t li = dpp_reduce(in_g && tim == tm ? lid : NONE32, NONE32, MinOp());
                        if (in_g) win = tim == tm && lid == li;
                        clash &= ~g;
                    }
                    losers = __ballot(act && !win);
                    clashes += (uint32_t)__popcll(losers);
                }
                rounds++;
                if (win) {
                    newcol = col;
                    const uint64_t end = t0 + t + tim;
                    busy_end = (uint32_t)end;
                    if (end > 0xFFFFFFFFull) {
                        record_error(ctl, ST_ERANGE, tb.rank_of(col), d, 2);
                        busy_end = 0xFFFFFFFFu;
                    }
                    cstar = max(cstar, busy_end);
                }
                if (!losers) break;
                want = act && !win;
            }
        }

        // publish the state at the window's end, then log the commits
        const uint64_t cm = __ballot(newcol != NONE32);
        if (newcol != NONE32) busy_rank = tb.rank_of(newcol);
        left -= (uint32_t)__popcll(cm);
        if (mine)
            __hip_atomic_store(ly.pub + (uint64_t)(k & 3u) * L + base + lane,
                               (left ? 0ull : NBR_FINAL) | nbr_tag(k) | ((uint64_t)busy_rank << 32) | busy_end,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (newcol != NONE32) {
            const unsigned long long q = log + lane_prefix(cm);
            ly.skey[0][q] = ((uint64_t)(busy_end - tim) << 32) | lid;
            ly.sval[0][q] = busy_rank;
        }
        log += (unsigned long long)__popcll(cm);
        // finished: the four copies of the entries all say so, then the wave ends
        if (!left && ++fin == 4u) break;
        // no event can follow the last representable time; by D windows later
        // an overflow met by any other device has been recorded first
        if (left && t0 > 0xFFFFFFFFull + (uint64_t)(sz.D + 4u) * tmin) {
            if (lane == 0) record_error(ctl, ST_EDEADLOCK, left, 0, 0);
            break;
        }
    }
    words = dpp_reduce(words, 0u, AddOp());
    cstar = dpp_reduce(cstar, 0u, MaxOp());
    if (lane == 0) {
        atomicMax(&ctl->cstar, cstar);
        atomicMax(&ctl->windows, (unsigned long long)k + 1ull - (fin ? fin - 1u : 0u));
        if (log != log0) atomicAdd(&ctl->n_log, log - log0);
        if (clashes) atomicAdd(&ctl->clashes, (unsigned long long)clashes);
        if (rounds) atomicAdd(&ctl->rounds, (unsigned long long)rounds);
        if (words) atomicAdd(&ctl->scan_words, (unsigned long long)words);
    }
}

template <uint32_t PPL, bool L3>
__global__ void __launch_bounds__(NBR_THREADS) k_match_nbr(Layout ly, Sizes sz, uint32_t lds_bytes)
{
    Control *ctl = ly.ctl;
    if (__hip_atomic_load(&ctl->error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
    if (ctl->needs_total == 0) return;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), wpb = blockDim.x >> 6;
    const uint32_t *wd = ly.wave_dest + (uint64_t)blockIdx.x * wpb;
    const uint32_t d = (uint32_t)__builtin_amdgcn_readfirstlane((int)wd[wave]);
    if (d == NONE32) return;
    // a device alone in its workgroup has all of its LDS
    uint32_t act = 0;
    for (uint32_t w = 0; w < wpb; w++) act += wd[w] != NONE32 ? 1u : 0u;
    const uint32_t share = act > 1u ? (lds_bytes / wpb) & ~15u : lds_bytes;
    run_dest<PPL, L3>(ly, sz, d, act > 1u ? wave * share : 0u, share);
}

const void *nbr_kernel(bool wide, bool l3)
{
    if (wide)
        return l3 ? reinterpret_cast<const void *>(k_match_nbr<NBR_MAX_POLL / 64u, true>)
                  : reinterpret_cast<const void *>(k_match_nbr<NBR_MAX_POLL / 64u, false>);
    return l3 ? reinterpret_cast<const void *>(k_match_nbr<1, true>) : reinterpret_cast<const void *>(k_match_nbr<1, false>);
}

}  // namespace

int match_nbr_max_grid(int device, int waves_per_block, bool wide, bool l3, size_t dyn_lds)
{
    int per_cu = 0, cus = 0;
    const void *kern = nbr_kernel(wide, l3);
    if (hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn_lds) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, 64 * waves_per_block, dyn_lds) != hipSuccess)
        return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) return 0;
    return per_cu * cus;
}

hipError_t launch_match_nbr(const Layout &ly, const Sizes &sz, hipStream_t st, int grid, int waves_per_block, bool wide,
                            bool l3, size_t dyn_lds)
{
    if (waves_per_block < 1 || waves_per_block > (int)NBR_WAVES) return hipErrorInvalidValue;
    const void *kern = nbr_kernel(wide, l3);
    const hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn_lds);
    if (e != hipSuccess) return e;
    Layout l = ly;
    Sizes s = sz;
    uint32_t b = (uint32_t)dyn_lds;
    void *args[] = {&l, &s, &b};
    return hipLaunchCooperativeKernel(kern, dim3(grid), dim3(64 * waves_per_block), args, (unsigned)dyn_lds, st);
}

}  // namespace pccl

// The event-stepped chunk-to-link matching with neighbour-only
// synchronisation: the kernel of the networks whose devices each fit one
// wavefront and whose link times lie close together (plan_nbr has the rule).
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

// Published entry of an in-link, high word: bit 31 the device is finished
// (the entry holds for every later window), 12 bits window tag, 19 bits chunk
// rank; low word: end time of the transfer in flight, 0 if none (a transfer
// takes at least 1 ns, so it never ends at 0).
constexpr uint32_t NBR_RANK = (1u << 19) - 1u;
static_assert(NBR_MAX_CHUNKS <= NBR_RANK, "a chunk rank fits in 19 bits");
constexpr uint32_t NBR_BEHIND = 0x800u << NBR_TAG_SHIFT;  // top bit of a tag difference
constexpr uint32_t NBR_FINAL = 1u << 31;
__device__ __forceinline__ uint32_t nbr_tag(uint32_t k) { return (k & 0xFFFu) << NBR_TAG_SHIFT; }

__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }
__device__ __forceinline__ uint32_t readlane(uint32_t v, uint32_t l)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)l);
}

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
    uint32_t ms, n;         // stride of mid; in-links, the stride of the rows
    uint32_t in_lds;
    uint64_t *g_row;        // [mw * n] candidate rows, word by word
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
    // [M] low 16 bits of the ranks, which ascend: those of the columns from
    // step[i] on lie above (i + 1) * 65,536
    __device__ uint16_t *rank() const { return reinterpret_cast<uint16_t *>(nbr_lds + rank_at); }
    uint32_t step[3];
};

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A wait that has lasted: another wave's error ends it, and the spin limit
// turns a wait that should not happen into an error.
__device__ __attribute__((noinline)) bool give_up(Control *ctl, uint32_t spins, uint32_t d, uint32_t k)
{
    if (__hip_atomic_load(&ctl->error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return true;
    if (spins <= NBR_SPIN_LIMIT) return false;
    if ((threadIdx.x & 63u) == 0) {
        atomicExch(&ctl->abort, 1u);
        record_error(ctl, ST_EINTERNAL, 3, d, k);
    }
    return true;
}

// The best candidate of a lane's in-link: its column (NONE32 if none), and
// where it was found: the live candidates of its row word and the summary
// words above it.
struct Pick {
    uint32_t col;
    uint64_t x, m, tp;
};

// The lowest live candidate column of this lane's in-link.  `want`: the
// lane's link is free.  A row word none of whose bits is live any more leaves
// the summaries.
template <bool L3, bool ALL>
__device__ __forceinline__ Pick first_live(const Tables &tb, bool want, uint32_t &words)
{
    const uint32_t lane = threadIdx.x & 63u;
    Pick p{NONE32, 0, 0, 0};
    bool go = false;
    if (want) p.tp = tb.top()[lane];
    go = p.tp != 0;
    do {
        if (go) {
            uint32_t w = low_bit(p.tp);
            if (L3) {
                p.m = tb.mid()[lane * tb.ms + w];
                w = w * 64u + low_bit(p.m);
            }
            uint64_t x;
            const uint64_t lv = tb.live()[w];
            // (rows in device memory are updated by atomics, which the L1
            // cache does not see: they are read past it)
            if (ALL || (tb.in_lds & IN_ROW)) x = tb.row()[w * tb.n + lane];
            else x = __hip_atomic_load(&tb.g_row[w * tb.n + lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            p.x = x & lv;
            words++;
            if (p.x) {
                p.col = w * 64u + low_bit(p.x);
                go = false;
            } else {
                if (L3) {
                    p.m &= p.m - 1ull;
                    tb.mid()[lane * tb.ms + (w >> 6)] = p.m;
                }
                if (!L3 || !p.m) {
                    p.tp &= p.tp - 1ull;
                    tb.top()[lane] = p.tp;
                    go = p.tp != 0;
                }
            }
        }
    } while (ballot(go));
    return p;
}

// The picked column leaves the row: its word leaves the summaries when the
// column was its last live candidate, so that the link's next pick does not
// meet an empty word.
template <bool L3>
__device__ __forceinline__ void drop_last(const Tables &tb, const Pick &p)
{
    const uint32_t lane = threadIdx.x & 63u;
    if (p.x & (p.x - 1ull)) return;
    if (L3) {
        const uint64_t m = p.m & (p.m - 1ull);
        tb.mid()[lane * tb.ms + low_bit(p.tp)] = m;
        if (m) return;
    }
    tb.top()[lane] = p.tp & (p.tp - 1ull);
}

// All windows of device d.  PPL: polled entries per lane.  L3: two summary
// levels (more than 4,096 columns).  ALL: every table is in LDS.
template <uint32_t PPL, bool L3, bool ALL>
__device__ __forceinline__ void run_dest(const Layout &ly, const Sizes &sz, const Tables &tb, uint32_t d, uint32_t M, uint32_t np)
{
    Control *ctl = ly.ctl;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t base = ly.in_off[d], n = ly.in_off[d + 1] - base;
    const bool mine = lane < n;
    const unsigned long long log0 = ly.dest_log[d];
    // this lane's in-link
    uint32_t tim = 0, lid = 0;
    if (mine) {
        tim = ly.slot_time[base + lane];
        lid = ly.slot_link[base + lane];
    }
    // the entries this lane polls (a lane past the last one polls that again):
    // their place; whether they feed an in-link (and where its row and summary
    // lie) or only tell how far a reader of d is (`dep`)
    const uint32_t *poll = sz.nbr_prune ? ly.poll_use + ly.poll_off[d] + ly.out_off[d] : ly.poll + ly.poll_off[d];
    const uint32_t W = (uint32_t)sz.W, L = sz.pub_n, tmin = sz.tmin, own = ly.pub_off[d] + lane;
    uint32_t at[PPL], link[PPL];
    bool dep[PPL], data[PPL];
#pragma unroll
    for (uint32_t u = 0; u < PPL; u++) {
        const uint32_t q = np ? poll[min(64u * u + lane, np - 1u)] : 0u;
        at[u] = q >> 8;
        link[u] = q & 0xFFu;
        dep[u] = link[u] == 0xFFu;
        data[u] = 64u * u + lane < np && !dep[u];
        if (!data[u]) link[u] = 0;
    }
    uint32_t left = M, fin = 0, k = 0;
    uint32_t busy_end = 0, busy_rank = 0;  // the transfer in flight on this lane's link (end 0: none)
    uint32_t cstar = 0, words = 0, rounds = 0, clashes = 0;
    unsigned long long log = log0;
    uint64_t t64 = 0;
    for (;; k++, t64 += tmin) {
        // the window is [t0, t0 + lim); past the last representable time lim
        // is 0 (ends below t0, and the 0 of an idle entry, wrap to at least lim)
        const uint32_t t0 = (uint32_t)t64;
        const uint32_t lim = t64 >> 32 ? 0u : (uint32_t)min((uint64_t)tmin, (1ull << 32) - t64);
        uint32_t ra[PPL], ca[PPL];  // arrivals of this window: offset into the window (NONE32: none), column
#pragma unroll
        for (uint32_t u = 0; u < PPL; u++) ra[u] = NONE32;
        if (k && np) {
            // sources: the state at the end of window k - 1; readers of d
            // that are no sources: that they have read window k - 4 (whose
            // entries this window's replace)
            const uint32_t o1 = ((k - 1u) & 3u) * L, o3 = ((k - 3u) & 3u) * L;
            const uint32_t g1 = nbr_tag(k - 1u), g3 = nbr_tag(k - 3u);
            uint64_t e[PPL];
            uint32_t spins = 0;
            bool stuck = false;
            while (true) {
                bool ok = true;
#pragma unroll
                for (uint32_t u = 0; u < PPL; u++) {
                    if (PPL > 2 && 64u * u >= np) break;
                    e[u] = __hip_atomic_load(ly.pub + (at[u] + (dep[u] ? o3 : o1)), __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
                }
#pragma unroll
                for (uint32_t u = 0; u < PPL; u++) {
                    if (PPL > 2 && 64u * u >= np) break;
                    const uint32_t hi = (uint32_t)(e[u] >> 32);
                    // the tag has reached the wanted one (modulo 4,096): a
                    // source is never ahead of it, but a reader that does not
                    // read this device's entries in turn may be
                    ok = ok && ((int32_t)hi < 0 || ((hi - (dep[u] ? g3 : g1)) & NBR_BEHIND) == 0);
                }
                if (ballot(!ok) == 0) break;
                if ((++spins & 15u) == 0 && give_up(ctl, spins, d, k)) {
                    stuck = true;
                    break;
                }
            }
            if (stuck) break;
            bool in[PPL], any = false;
#pragma unroll
            for (uint32_t u = 0; u < PPL; u++) in[u] = false;
#pragma unroll
            for (uint32_t u = 0; u < PPL; u++) {
                if (PPL > 2 && 64u * u >= np) break;
                in[u] = data[u] && (uint32_t)e[u] - t0 < lim;
                any = any || in[u];
            }
            if (left && ballot(any)) {
                // the arrivals in d's columns, those that d still needs
#pragma unroll
                for (uint32_t u = 0; u < PPL; u++) {
                    if (PPL > 2 && 64u * u >= np) break;
                    if (in[u]) {
                        const uint32_t r = (uint32_t)(e[u] >> 32) & NBR_RANK, w = r >> 6, b = r & 63u;
                        uint64_t nw;
                        uint32_t pr;
                        if (ALL || (tb.in_lds & IN_NEED)) {
                            nw = tb.need()[w];
                            pr = tb.pre()[w];
                        } else {
                            nw = tb.g_need[w];
                            pr = tb.g_pre[w];
                        }
                        if ((nw >> b) & 1ull) {
                            ca[u] = pr + (uint32_t)__popcll(nw & ((1ull << b) - 1ull));
                            if ((tb.live()[ca[u] >> 6] >> (ca[u] & 63u)) & 1ull) ra[u] = (uint32_t)e[u] - t0;
                        }
                    }
                }
            }
        }
        // this lane's transfer, when it ends inside the window; at time 0
        // every (idle) link counts as ending there
        uint32_t rb = busy_end - t0 < lim ? busy_end - t0 : NONE32;

        // events of the window in time order
        uint32_t newcol = NONE32;  // the column this lane's link commits in this window (at most one: T >= Tmin)
        while (true) {
            uint32_t m = rb;
#pragma unroll
            for (uint32_t u = 0; u < PPL; u++) m = min(m, ra[u]);
            const uint64_t pend = ballot(m != NONE32);
            if (!pend) break;
            // the earliest: mostly the first pending lane's
            uint32_t t = readlane(m, low_bit(pend));
            if (ballot(m < t)) t = dpp_reduce(m, NONE32, MinOp());
            if (rb == t) {
                busy_end = 0;
                rb = NONE32;
            }
#pragma unroll
            for (uint32_t u = 0; u < PPL; u++) {
                if (PPL > 2 && 64u * u >= np) break;
                if (ra[u] == t) {
                    const uint32_t j = link[u], w = ca[u] >> 6;
                    const unsigned long long bit = 1ull << (ca[u] & 63u);
                    if (ALL || (tb.in_lds & IN_ROW)) atomicOr((unsigned long long *)&tb.row()[w * tb.n + j], bit);
                    else __hip_atomic_fetch_or(&tb.g_row[w * tb.n + j], (uint64_t)bit, __ATOMIC_RELAXED,
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
            // rows in device memory: the arrivals' bits are set before other
            // lanes read them (rows in LDS: a wave's LDS operations are done in
            // order).  No test of where the rows are: it changes the registers
            // of all builds (8x8x4 torus, 2.65 -> 2.71 ms), the wait alone costs
            // nothing measurable.
            if (!ALL) __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
            // pick rounds
            const uint32_t now = t0 + t;
            bool want = mine && busy_end == 0;
            uint64_t losers;
            do {
                const Pick pk = first_live<L3, ALL>(tb, want, words);
                const uint32_t col = pk.col;
                const bool act = col != NONE32;
                const uint64_t actm = ballot(act);
                losers = 0;
                if (actm) {
                    bool win = act;
                    unsigned long long *lw = (unsigned long long *)&tb.live()[col >> 6];
                    const uint64_t bit = 1ull << (col & 63u);
                    if ((actm & (actm - 1ull)) == 0) {
                        if (act) atomicAnd(lw, ~bit);
                    } else {
                        // clear the picked columns; a lane that finds its
                        // column already cleared shares it with another lane
                        if (act) win = (atomicAnd(lw, ~bit) & bit) != 0;
                        uint64_t clash = ballot(act && !win);
                        if (clash) {
                            // fastest link, then lowest id, among the links that picked the column
                            while (clash) {
                                const uint32_t v = readlane(col, low_bit(clash));
                                const bool in_g = col == v;
                                const uint64_t g = ballot(in_g);
                                const uint32_t tm = dpp_reduce(in_g ? tim : NONE32, NONE32, MinOp());
                                const uint32_t li = dpp_reduce(in_g && tim == tm ? lid : NONE32, NONE32, MinOp());
                                if (in_g) win = tim == tm && lid == li;
                                clash &= ~g;
                            }
                            losers = ballot(act && !win);
                            clashes += (uint32_t)__popcll(losers);
                            want = act && !win;
                        }
                    }
                    rounds++;
                    if (win) {
                        newcol = col;
                        busy_end = now + tim;
                        drop_last<L3>(tb, pk);
                    }
                }
            } while (losers);
        }

        // publish the state at the window's end, then log the commits
        if (newcol != NONE32) {
            if (ALL || (tb.in_lds & IN_RANK)) {
                busy_rank = tb.rank()[newcol];
                if (W > 1024u) {
#pragma unroll
                    for (uint32_t i = 0; i < 3; i++) busy_rank += newcol >= tb.step[i] ? 0x10000u : 0u;
                }
            } else {
                busy_rank = tb.g_rank[newcol] & NBR_RANK_MASK;
            }
        }
        const uint64_t cm = ballot(newcol != NONE32);
        if (newcol != NONE32) cstar = max(cstar, busy_end);
        left -= (uint32_t)__popcll(cm);
        if (mine)
            __hip_atomic_store(ly.pub + ((k & 3u) * L + own),
                               ((uint64_t)((left ? 0u : NBR_FINAL) | nbr_tag(k) | busy_rank) << 32) | busy_end,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (newcol != NONE32) {
            const unsigned long long q = log + lane_prefix(cm);
            ly.skey[0][q] = ((uint64_t)(busy_end - tim) << 32) | lid;
            ly.sval[0][q] = busy_rank;
        }
        log += (unsigned long long)__popcll(cm);
        // an end beyond 32 bits ends the synthesis
        if (newcol != NONE32 && busy_end < tim) record_error(ctl, ST_ERANGE, busy_rank, d, 2);
        // finished: the four copies of the entries all say so, then the wave ends
        if (!left && ++fin == 4u) break;
        // no event can follow the last representable time; by D windows later
        // an overflow met by any other device has been recorded first
        if (left && t64 > 0xFFFFFFFFull + (uint64_t)(sz.D + 4u) * tmin) {
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

// Calls f(i, load(i)) for the i < n that are this lane's, eight loads in
// flight together (one memory round trip per 512 elements, not per 64).
template <class Load, class F>
__device__ __forceinline__ void copy_batched(uint32_t n, Load load, F f)
{
    const uint32_t lane = threadIdx.x & 63u;
    for (uint32_t i0 = lane; i0 < n; i0 += 512) {
        decltype(load(0u)) v[8];
#pragma unroll
        for (uint32_t k = 0; k < 8; k++) v[k] = load(min(i0 + 64u * k, n - 1u));
#pragma unroll
        for (uint32_t k = 0; k < 8; k++)
            if (i0 + 64u * k < n) f(i0 + 64u * k, v[k]);
    }
}

// Places device d's tables in the LDS bytes [at, at + room) and fills them.
__device__ __forceinline__ void fill_tables(const Layout &ly, const Sizes &sz, uint32_t d, uint32_t M, uint32_t at, uint32_t room,
                                            Tables &tb)
{
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t n = ly.in_off[d + 1] - ly.in_off[d], W = (uint32_t)sz.W;
    const uint32_t mw = (M + 63u) >> 6, mm = (mw + 63u) >> 6, end = at + room;
    const bool l3 = mm > 1u;
    auto take = [&](uint32_t bytes) {
        const uint32_t p = at;
        at += (bytes + 7u) & ~7u;
        return p;
    };
    tb.live_at = take(mw * 8u);
    tb.top_at = take(n * 8u);
    tb.ms = mm | 1u;
    tb.n = n;
    if (l3) tb.mid_at = take(n * tb.ms * 8u);
    tb.g_row = ly.cand + ly.cand_off[d];
    tb.g_need = ly.needs + (uint64_t)d * sz.Wp;
    tb.g_pre = ly.need_pre + (uint64_t)d * sz.Wp;
    tb.g_rank = ly.col_rank + ly.dest_log[d];
    // the summaries follow the rows: lane j's words of every group
    uint64_t top = 0;
    if (lane < n && mm) {
        const uint64_t *g_mid = tb.g_row + (uint64_t)mw * n + lane;
        for (uint32_t g0 = 0; g0 < mm; g0 += 8) {
            uint64_t v[8];
#pragma unroll
            for (uint32_t k = 0; k < 8; k++) v[k] = g_mid[min(g0 + k, mm - 1u) * n];
#pragma unroll
            for (uint32_t k = 0; k < 8; k++) {
                if (g0 + k >= mm) continue;
                if (l3) {
                    tb.mid()[lane * tb.ms + g0 + k] = v[k];
                    if (v[k]) top |= 1ull << (g0 + k);
                } else {
                    top = v[k];
                }
            }
        }
    }
    if (lane < n) tb.top()[lane] = top;
    if (at + n * mw * 8u <= end) {
        tb.in_lds |= IN_ROW;
        tb.row_at = take(n * mw * 8u);
        copy_batched(n * mw, [&](uint32_t i) { return tb.g_row[i]; }, [&](uint32_t i, uint64_t v) { tb.row()[i] = v; });
    }
    if (M <= 0xFFFFu && at + W * 10u + 8u <= end) {
        tb.in_lds |= IN_NEED;
        tb.need_at = take(W * 8u);
        tb.pre_at = take(W * 2u);
        copy_batched(W, [&](uint32_t i) { return tb.g_need[i]; }, [&](uint32_t i, uint64_t v) { tb.need()[i] = v; });
        copy_batched(W, [&](uint32_t i) { return tb.g_pre[i]; }, [&](uint32_t i, uint32_t v) { tb.pre()[i] = (uint16_t)v; });
    }
    static_assert(NBR_MAX_CHUNKS <= 4u << 16, "ranks have at most two bits above 16");
#pragma unroll
    for (uint32_t i = 0; i < 3; i++) tb.step[i] = (i + 1u) * 1024u < W ? tb.g_pre[(i + 1u) * 1024u] : M;
    if (at + M * 2u <= end) {
        tb.in_lds |= IN_RANK;
        tb.rank_at = take(M * 2u);
        // (a count may lie above the rank)
        copy_batched(M, [&](uint32_t i) { return tb.g_rank[i]; }, [&](uint32_t i, uint32_t v) { tb.rank()[i] = (uint16_t)v; });
    }
    for (uint32_t i = lane; i < mw; i += 64)
        tb.live()[i] = i + 1 < mw || (M & 63u) == 0 ? NONE64 : (1ull << (M & 63u)) - 1ull;
    wave_sync();
}

// Each wave takes the build of run_dest for its device: polled entries per
// lane, summary levels, and whether every table found room in LDS.
template <uint32_t PPL>
__device__ __forceinline__ void run_built(const Layout &ly, const Sizes &sz, const Tables &tb, uint32_t d, uint32_t M, uint32_t np)
{
    if (tb.in_lds != (IN_ROW | IN_NEED | IN_RANK)) {
        if (M > 4096u) run_dest<PPL, true, false>(ly, sz, tb, d, M, np);
        else run_dest<PPL, false, false>(ly, sz, tb, d, M, np);
    } else if (M > 4096u) {
        run_dest<PPL, true, true>(ly, sz, tb, d, M, np);
    } else {
        run_dest<PPL, false, true>(ly, sz, tb, d, M, np);
    }
}

__global__ void __launch_bounds__(NBR_THREADS) k_match_nbr(Layout ly, Sizes sz, uint32_t lds_bytes, uint32_t spread)
{
    if (blockIdx.x % spread) return;
    Control *ctl = ly.ctl;
    if (__hip_atomic_load(&ctl->error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
    if (ctl->needs_total == 0) return;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), wpb = blockDim.x >> 6;
    const uint32_t *wd = ly.wave_dest + (uint64_t)(blockIdx.x / spread) * wpb;
    const uint32_t d = (uint32_t)__builtin_amdgcn_readfirstlane((int)wd[wave]);
    if (d == NONE32) return;
    // a device alone in its workgroup has all of its LDS
    uint32_t act = 0;
    for (uint32_t w = 0; w < wpb; w++) act += wd[w] != NONE32 ? 1u : 0u;
    const uint32_t share = act > 1u ? (lds_bytes / wpb) & ~15u : lds_bytes;
    const uint32_t M = ly.dest_cols[d], np = sz.nbr_prune ? ly.poll_cnt[d] : ly.poll_off[d + 1] - ly.poll_off[d];
    Tables tb{};
    fill_tables(ly, sz, d, M, act > 1u ? wave * share : 0u, share, tb);
    if (np <= 64u) run_built<1>(ly, sz, tb, d, M, np);
    else if (np <= 128u) run_built<2>(ly, sz, tb, d, M, np);
    else run_built<NBR_MAX_POLL / 64u>(ly, sz, tb, d, M, np);
}

}  // namespace

int match_nbr_max_grid(int device, int waves_per_block, size_t dyn_lds)
{
    int per_cu = 0, cus = 0;
    const void *kern = reinterpret_cast<const void *>(k_match_nbr);
    if (hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn_lds) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, 64 * waves_per_block, dyn_lds) != hipSuccess)
        return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) return 0;
    return per_cu * cus;
}

hipError_t launch_match_nbr(const Layout &ly, const Sizes &sz, hipStream_t st, int grid, int waves_per_block,
                            size_t dyn_lds, uint32_t spread)
{
    if (waves_per_block < 1 || waves_per_block > (int)NBR_WAVES) return hipErrorInvalidValue;
    const void *kern = reinterpret_cast<const void *>(k_match_nbr);
    const hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn_lds);
    if (e != hipSuccess) return e;
    Layout l = ly;
    Sizes s = sz;
    uint32_t b = (uint32_t)dyn_lds;
    void *args[] = {&l, &s, &b, &spread};
    return hipLaunchCooperativeKernel(kern, dim3(grid * spread), dim3(64 * waves_per_block), args, (unsigned)dyn_lds, st);
}

}  // namespace pccl

// Setup of one synthesis on the device: conditions from the pre/postcondition
// bitmaps, shortest-path trees from every chunk source, condition distances,
// the priority order, relay devices and the initial holds/needs bitmaps over
// priority-ordered columns.
#include "pccl_internal.h"

namespace pccl {
namespace {

constexpr uint32_t FLAG_POST = 0x80000000u;  // holder_cnt: chunk has a postcondition bit
constexpr uint32_t CNT_MASK = 0x7FFFFFFFu;

// detail codes carried in error_arg[2] for PCCL_EINVAL
enum : uint32_t { BAD_TAIL = 1, BAD_MEMBER = 2, BAD_GROUP = 3, TWO_HOLDERS = 4, NO_HOLDER = 5 };

// The start of a synthesis: the control block, the per-chunk arrays and the
// bitmaps (one launch; a launch costs as much as clearing 16 MB).
__global__ void __launch_bounds__(256) k_reset(Layout ly, Sizes sz)
{
    const uint64_t i0 = (uint64_t)blockIdx.x * 256u + threadIdx.x, step = (uint64_t)gridDim.x * 256u;
    if (i0 == 0) {
        Control c = {};
        c.max_sends = sz.max_sends;
        *ly.ctl = c;
    }
    for (uint64_t i = i0; i < sz.C; i += step) {
        ly.holder_cnt[i] = 0;
        ly.chunk_src[i] = NONE32;
        ly.chunk_dist[i] = 0;
    }
    for (uint64_t i = i0; i < sz.N; i += step) ly.is_src[i] = 0;
    if (sz.sw_cols)
        for (uint64_t i = i0; i < 2ull * MAX_MATCH_GRID; i += step) ly.xslot[i * XSLOT_WORDS] = 0;
    const uint4 z = make_uint4(0, 0, 0, 0);
    const uint64_t bm = (uint64_t)sz.D * sz.Wp / 2;  // rows are whole 1 KiB lines
    for (uint64_t i = i0; i < bm; i += step) {
        reinterpret_cast<uint4 *>(ly.needs)[i] = z;
        if (!sz.cols) reinterpret_cast<uint4 *>(ly.holds)[i] = z;
    }
}

__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Calls f(lane, bit) for every set bit of the 64 words that the lanes of a
// wave hold (word `lane` is lane's x), bits shared out evenly over the lanes:
// a dense word's work is a wave's and not one lane's (8x8 torus, 64 chunks:
// the relay walks 77 -> 11 us).  `list`: room for 4,096 positions in LDS.
template <class F>
__device__ __forceinline__ void for_bits(uint64_t x, uint16_t *list, F f)
{
    const uint32_t lane = threadIdx.x & 63u;
    if (__builtin_amdgcn_ballot_w64(x != 0) == 0) return;
    uint32_t inc = (uint32_t)__popcll(x);
    for (uint32_t o = 1; o < 64; o <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)inc, o);
        if (lane >= o) inc += y;
    }
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
    uint32_t at = inc - (uint32_t)__popcll(x);
    for (; x; x &= x - 1) list[at++] = (uint16_t)(lane * 64u + (uint32_t)__builtin_ctzll(x));
    wave_fence();
    for (uint32_t i = lane; i < total; i += 64) {
        const uint32_t e = list[i];
        f(e >> 6, e & 63u);
    }
    // (the next call's writes come after these reads)
    __builtin_amdgcn_wave_barrier();
}
constexpr uint32_t BIT_LIST = 4096;  // 64 words

// Mask of valid bits in word k of a chunk row.
__device__ inline uint64_t tail_mask(uint64_t k, const Sizes &sz)
{
    if (k + 1 < sz.W || (sz.C & 63u) == 0) return NONE64;
    return (1ull << (sz.C & 63u)) - 1ull;
}

// Conditions (Sec. 4.1): for every set bit of the NPU-centric bitmaps,
// count precondition holders per chunk, mark chunks that are needed
// somewhere and NPUs that hold something, and check that pre/post bits sit on
// members of the chunk's process group.  Grid: x over words, y over NPU rows.
// The per-bit updates are atomics whose results are not used (a second holder
// is found by the per-chunk check), so they are in flight together; with a
// single process group the membership of the row is checked once per word.
__global__ void __launch_bounds__(256) k_conditions(Layout ly, Sizes sz, const uint64_t *pre, const uint64_t *post,
                                                    const uint16_t *cg)
{
    __shared__ uint16_t list[4][BIT_LIST];
    const uint64_t k = (uint64_t)blockIdx.x * 256u + threadIdx.x, k0 = k & ~63ull;
    const uint32_t v = blockIdx.y;
    uint64_t p = 0, q = 0;
    if (k < sz.W) {
        p = pre[(uint64_t)v * sz.W + k];
        q = post[(uint64_t)v * sz.W + k];
    }
    if ((p | q) != 0) {
        const uint64_t tm = tail_mask(k, sz);
        if ((p | q) & ~tm) record_error(ly.ctl, ST_EINVAL, sz.C, v, BAD_TAIL);
        p &= tm;
        q &= tm;
        if (p) ly.is_src[v] = 1u;
        if (!cg && (p | q) && !((ly.group_masks[v >> 6] >> (v & 63)) & 1ull))
            record_error(ly.ctl, ST_EINVAL, (uint32_t)(k * 64 + __builtin_ctzll(p | q)), v, BAD_MEMBER);
    }
    uint16_t *l = list[threadIdx.x >> 6];
    if (cg) {
        for_bits(p | q, l, [&](uint32_t w, uint32_t b) {
            const uint32_t c = (uint32_t)(k0 + w) * 64u + b;
            const uint32_t g = cg[c];
            if (g >= sz.G) record_error(ly.ctl, ST_EINVAL, c, v, BAD_GROUP);
            else if (!((ly.group_masks[(uint64_t)g * sz.WN + (v >> 6)] >> (v & 63)) & 1ull))
                record_error(ly.ctl, ST_EINVAL, c, v, BAD_MEMBER);
        });
    }
    for_bits(p, l, [&](uint32_t w, uint32_t b) {
        const uint32_t c = (uint32_t)(k0 + w) * 64u + b;
        atomicAdd(&ly.holder_cnt[c], 1u);
        ly.chunk_src[c] = v;  // the one holder (several are an error, reported below)
    });
    for_bits(q, l, [&](uint32_t w, uint32_t b) { atomicOr(&ly.holder_cnt[(uint32_t)(k0 + w) * 64u + b], FLAG_POST); });
}

constexpr uint32_t SP_BATCH = 8;  // links whose loads one thread issues together

// The per-chunk check of the conditions (shared out over the workgroups), and
// shortest paths from one NPU per workgroup, those that hold a chunk (Alg. 3
// ShortestPath over the alpha-beta link times): Bellman-Ford relaxation with the distances in
// LDS, then the parent of each device = the smallest-id in-neighbour on a
// shortest path (the tree the pruned BFS of Sec. 4.3 keeps).
__global__ void __launch_bounds__(512) k_shortest_paths(Layout ly, Sizes sz)
{
    extern __shared__ unsigned long long dist[];
    __shared__ uint32_t changed;
    const uint32_t s = blockIdx.x, tid = threadIdx.x;
    for (uint64_t c = (uint64_t)s * blockDim.x + tid; c < sz.C; c += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t h = ly.holder_cnt[c];
        if ((h & FLAG_POST) && !(h & CNT_MASK)) record_error(ly.ctl, ST_EINVAL, (uint32_t)c, 0, NO_HOLDER);
        if ((h & CNT_MASK) > 1u) record_error(ly.ctl, ST_EINVAL, (uint32_t)c, ly.chunk_src[c], TWO_HOLDERS);
    }
    if (!ly.is_src[s]) return;
    for (uint32_t v = tid; v < sz.D; v += blockDim.x) dist[v] = v == s ? 0ull : NONE64;
    __syncthreads();
    for (uint32_t it = 0; it < sz.D; it++) {
        if (tid == 0) changed = 0;
        __syncthreads();
        // eight links per thread loaded together (indices past L reread the
        // last link and are skipped)
        for (uint32_t e0 = tid; e0 < sz.L; e0 += SP_BATCH * blockDim.x) {
            uint32_t ls[SP_BATCH], ld[SP_BATCH], lt[SP_BATCH];
#pragma unroll
            for (uint32_t k = 0; k < SP_BATCH; k++) {
                const uint32_t e = min(e0 + k * blockDim.x, sz.L - 1u);
                ls[k] = ly.lsrc[e];
                ld[k] = ly.ldst[e];
                lt[k] = ly.ltime[e];
            }
#pragma unroll
            for (uint32_t k = 0; k < SP_BATCH; k++) {
                if (e0 + k * blockDim.x >= sz.L) continue;
                const unsigned long long du = dist[ls[k]];
                if (du == NONE64) continue;
                const unsigned long long nd = du + lt[k];
                if (nd < dist[ld[k]]) {
                    atomicMin(&dist[ld[k]], nd);
                    changed = 1;
                }
            }
        }
        __syncthreads();
        const uint32_t again = changed;
        __syncthreads();
        if (!again) break;
    }
    for (uint32_t v = tid; v < sz.D; v += blockDim.x) {
        const unsigned long long dv = dist[v];
        ly.sp_dist[(uint64_t)s * sz.D + v] = dv;
        uint32_t par = NONE32;
        if (v != s && dv != NONE64) {
            const uint32_t i0 = ly.in_off[v], i1 = ly.in_off[v + 1];
            for (uint32_t i = i0; i < i1; i += SP_BATCH) {
                uint32_t su[SP_BATCH], st[SP_BATCH];
#pragma unroll
                for (uint32_t k = 0; k < SP_BATCH; k++) {
                    const uint32_t x = min(i + k, i1 - 1u);
                    su[k] = ly.slot_src[x];
                    st[k] = ly.slot_time[x];
                }
#pragma unroll
                for (uint32_t k = 0; k < SP_BATCH; k++) {
                    if (i + k >= i1) continue;
                    const unsigned long long du = dist[su[k]];
                    if (du != NONE64 && du + st[k] == dv && su[k] < par) par = su[k];
                }
            }
        }
        ly.sp_parent[(uint64_t)s * sz.D + v] = par;
    }
}

// Condition distance = max over destinations of the shortest-path distance
// (Alg. 3); destinations = postcondition and not precondition.
__global__ void __launch_bounds__(256) k_chunk_dist(Layout ly, Sizes sz, const uint64_t *pre, const uint64_t *post)
{
    __shared__ uint16_t list[4][BIT_LIST];
    if (ly.ctl->error) return;
    const uint64_t k = (uint64_t)blockIdx.x * 256u + threadIdx.x, k0 = k & ~63ull;
    const uint32_t v = blockIdx.y;
    uint64_t x = 0;
    if (k < sz.W) x = post[(uint64_t)v * sz.W + k] & ~pre[(uint64_t)v * sz.W + k] & tail_mask(k, sz);
    for_bits(x, list[threadIdx.x >> 6], [&](uint32_t w, uint32_t b) {
        const uint32_t c = (uint32_t)(k0 + w) * 64u + b, s = ly.chunk_src[c];
        const unsigned long long dv = ly.sp_dist[(uint64_t)s * sz.D + v];
        if (dv == NONE64) record_error(ly.ctl, ST_EUNREACHABLE, c, v, s);
        else if (dv >= 0xFFFFFFFFull) record_error(ly.ctl, ST_ERANGE, c, v, 1);
        else atomicMax(&ly.chunk_dist[c], dv);
    });
}

// Switch model: for every limited-switch row and chunk rank, how many of the
// switch's out-links lead to a device that needs the chunk once the needs
// rows are set up (the matching kernel keeps the count as those devices
// receive it, and reads it when the switch takes the chunk into a buffer
// place); for the kernel over columns which ones, as a mask.  One thread per
// (row, chunk): the 64 threads of a wave read the
// same needs word of each out-neighbour.
__global__ void k_adm_counts(Layout ly, Sizes sz)
{
    const uint64_t c = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t row = blockIdx.y;
    if (c >= sz.C) return;
    const uint32_t o0 = ly.sw.b_abs[2 * row], no = ly.sw.b_abs[2 * row + 1];
    uint32_t n = 0;
    uint64_t mask = 0;
    for (uint32_t q = 0; q < no; q++) {
        const uint32_t o = ly.sw.b_out[o0 + q] & 0xFFFFu;
        const uint64_t x = (ly.needs[(uint64_t)o * sz.Wp + (c >> 6)] >> (c & 63u)) & 1ull;
        n += (uint32_t)x;
        mask |= x << (q & 63u);
    }
    // (a column plan's switches have at most 64 out-links)
    if (sz.sw_cols) ly.sw.amask[(uint64_t)row * sz.C + c] = mask;
    else ly.sw.acnt[(uint64_t)row * sz.C + c] = n;
}

// Priority order (distance descending, then the SplitMix64 key ascending,
// then chunk id): one stable sort of the bitwise-not of the distance (high
// word) and the key's high word (low word), from chunk id order, then runs
// of equal sort keys ordered by the key's low word (k_rank).
__global__ void k_keys_hash(Layout ly, Sizes sz, uint64_t seed)
{
    const uint64_t c = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= sz.C) return;
    const uint32_t nd = ~(uint32_t)ly.chunk_dist[c];
    ly.skey[0][c] = ((uint64_t)nd << 32) | (splitmix64_key(seed, c) >> 32);
    ly.sval[0][c] = (uint32_t)c;
}

__device__ inline void set_rank(const Layout &ly, const Sizes &sz, uint32_t r, uint32_t c)
{
    ly.order[r] = c;
    ly.rank[c] = r;
    // (the counts of the array it shares are no longer read)
    if (sz.cols) ly.rank_src[r] = ly.chunk_src[c];
}

// After the sort: ranks.  The first thread of a run of equal sort keys (equal
// distance and key high word; with random keys a run is rare and short)
// orders the run by (key low word, chunk id), in place, and ranks it.
__global__ void k_rank(Layout ly, Sizes sz, uint64_t seed)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= sz.C) return;
    const uint32_t cur = ly.ctl->sort_cur;
    const uint64_t *k = ly.skey[cur];
    uint32_t *v = ly.sval[cur];
    const uint64_t ki = k[i];
    if (i > 0 && k[i - 1] == ki) return;  // ranked by the run's first thread
    uint64_t j = i + 1;
    while (j < sz.C && k[j] == ki) j++;
    // insertion sort; the stable sort left the run in chunk id order
    for (uint64_t a = i + 1; a < j; a++) {
        const uint32_t c = v[a], lo = (uint32_t)splitmix64_key(seed, c);
        uint64_t b = a;
        while (b > i) {
            const uint32_t p = v[b - 1], plo = (uint32_t)splitmix64_key(seed, p);
            if (plo < lo || (plo == lo && p < c)) break;
            v[b] = p;
            b--;
        }
        v[b] = c;
    }
    for (uint64_t a = i; a < j; a++) set_rank(ly, sz, (uint32_t)a, v[a]);
}

// The same for at most SMALL_SORT chunks, in one workgroup and one launch from
// the distances to the ranks: a bitonic sort in LDS by distance descending,
// then the whole SplitMix64 key.
__global__ void __launch_bounds__(1024) k_order_small(Layout ly, Sizes sz, uint64_t seed)
{
    __shared__ uint64_t key[SMALL_SORT];
    __shared__ uint32_t low[SMALL_SORT], val[SMALL_SORT];
    const uint32_t tid = threadIdx.x;
    uint32_t m = 64;
    while (m < sz.C) m <<= 1;
    for (uint32_t c = tid; c < m; c += 1024) {
        uint64_t k = NONE64;
        uint32_t lo = NONE32;
        if (c < sz.C) {
            const uint64_t h = splitmix64_key(seed, c);
            k = ((uint64_t)(~(uint32_t)ly.chunk_dist[c]) << 32) | (h >> 32);
            lo = (uint32_t)h;
        }
        key[c] = k;
        low[c] = lo;
        val[c] = c < sz.C ? c : NONE32;
    }
    bitonic_sort(m, [&](uint32_t a, uint32_t b) {
        return key[a] != key[b] ? key[a] > key[b] : low[a] != low[b] ? low[a] > low[b] : val[a] > val[b];
    }, [&](uint32_t a, uint32_t b) {
        const uint64_t k = key[a];
        key[a] = key[b];
        key[b] = k;
        uint32_t t = low[a];
        low[a] = low[b];
        low[b] = t;
        t = val[a];
        val[a] = val[b];
        val[b] = t;
    });
    for (uint32_t r = tid; r < sz.C; r += 1024) set_rank(ly, sz, r, val[r]);
}

__global__ void k_holds(Layout ly, Sizes sz)
{
    if (ly.ctl->error) return;
    const uint64_t c = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= sz.C) return;
    if ((ly.holder_cnt[c] & CNT_MASK) != 1u) return;
    const uint32_t r = ly.rank[c];
    atomicOr((unsigned long long *)&ly.holds[(uint64_t)ly.chunk_src[c] * sz.Wp + (r >> 6)], 1ull << (r & 63));
}

// needs = destinations plus the relays on their tree paths (the paths the
// pruned BFS keeps, Sec. 4.3): walk parents from each destination up to the
// source.  A walk that meets a bit already set stops there: whoever set it
// is a destination or a walk that continues upward.  Two walks may both
// pass a device before either bit is visible; both then set it (harmless).
__global__ void __launch_bounds__(256) k_needs(Layout ly, Sizes sz, const uint64_t *pre, const uint64_t *post)
{
    __shared__ uint16_t list[4][BIT_LIST];
    if (ly.ctl->error) return;
    const uint64_t k = (uint64_t)blockIdx.x * 256u + threadIdx.x, k0 = k & ~63ull;
    const uint32_t v = blockIdx.y;
    uint64_t x = 0;
    if (k < sz.W) x = post[(uint64_t)v * sz.W + k] & ~pre[(uint64_t)v * sz.W + k] & tail_mask(k, sz);
    for_bits(x, list[threadIdx.x >> 6], [&](uint32_t wo, uint32_t b) {
        const uint32_t c = (uint32_t)(k0 + wo) * 64u + b;
        const uint32_t s = ly.chunk_src[c], r = ly.rank[c];
        const uint64_t bit = 1ull << (r & 63);
        const uint32_t *par = ly.sp_parent + (uint64_t)s * sz.D;
        uint32_t u = v;
        for (uint32_t hop = 0; hop < sz.D && u != s && u < sz.D; hop++) {
            unsigned long long *w = (unsigned long long *)&ly.needs[(uint64_t)u * sz.Wp + (r >> 6)];
            const uint32_t next = par[u];
            // a relay bit another walk already set: that walk covers the rest
            if ((atomicOr(w, bit) & bit) && hop > 0) break;
            u = next;
        }
    });
}

// Candidates of every link at the start (one wave per destination-major
// slot): popcount(holds[src] & needs[dst]) over the rows.  The matching
// kernel keeps this count as an upper bound (arrivals add, the link's own
// commits subtract, a pick round that finds nothing resets it to 0), so a
// freed link whose bound is 0 has no candidate and needs no scan.
__global__ void __launch_bounds__(256) k_link_counts(Layout ly, Sizes sz)
{
    if (ly.ctl->error) return;
    const uint32_t lane = threadIdx.x & 63;
    const uint64_t sl = (uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (sl >= sz.L) return;
    const uint64_t Ws = (sz.W + 1) & ~1ull;
    const uint64_t *h = ly.holds + (uint64_t)ly.slot_src[sl] * sz.Wp;
    const uint64_t *n = ly.needs + (uint64_t)ly.ldst[ly.slot_link[sl]] * sz.Wp;
    uint32_t c = 0;
    for (uint64_t w = 2 * lane; w < Ws; w += 128) {
        const uint4 a = *reinterpret_cast<const uint4 *>(h + w), b = *reinterpret_cast<const uint4 *>(n + w);
        c += __popc(a.x & b.x) + __popc(a.y & b.y) + __popc(a.z & b.z) + __popc(a.w & b.w);
    }
    for (int off = 32; off; off >>= 1) c += (uint32_t)__shfl_xor((int)c, off);
    if (lane == 0) ly.lcnt[sl] = c;
}

// Each destination gets a contiguous segment of the send log, as long as
// the number of deliveries it needs (every delivery is one transfer into it).
__global__ void __launch_bounds__(256) k_needs_count(Layout ly, Sizes sz)
{
    __shared__ unsigned long long part[4];
    const uint32_t d = blockIdx.x, tid = threadIdx.x;
    unsigned long long c = 0;
    if (!ly.ctl->error) {
        const uint64_t *row = ly.needs + (uint64_t)d * sz.Wp;
        for (uint64_t w = tid; w < sz.Wp; w += 256) c += (unsigned long long)__popcll(row[w]);
    }
    for (int off = 32; off; off >>= 1) c += __shfl_xor(c, off);
    if ((tid & 63) == 0) part[tid >> 6] = c;
    __syncthreads();
    if (tid == 0) ly.dest_log[d] = part[0] + part[1] + part[2] + part[3];
}

__global__ void __launch_bounds__(1024) k_log_offsets(Layout ly, Sizes sz)
{
    __shared__ unsigned long long part[1024];
    const uint32_t tid = threadIdx.x;
    const uint32_t per = (sz.D + 1023) / 1024;
    const uint32_t lo = tid * per, hi = min(lo + per, sz.D);
    unsigned long long s = 0;
    for (uint32_t v = lo; v < hi; v++) s += ly.dest_log[v];
    part[tid] = s;
    __syncthreads();
    for (uint32_t off = 1; off < 1024; off <<= 1) {
        unsigned long long x = tid >= off ? part[tid - off] : 0;
        __syncthreads();
        part[tid] += x;
        __syncthreads();
    }
    unsigned long long run = tid ? part[tid - 1] : 0;
    for (uint32_t v = lo; v < hi; v++) {
        const unsigned long long c = ly.dest_log[v];
        ly.dest_log[v] = run;
        run += c;
    }
    if (tid == 1023) ly.ctl->needs_total = part[1023];
}

__global__ void k_init_match(Layout ly, Sizes sz)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < sz.L) {
        ly.busy[i] = 0;
        ly.infl[i] = NONE32;
        ly.cur[i] = 0;
        ly.lflags[i] = 0;
        ly.snap[i] = NONE64;
        ly.snap[sz.L + i] = NONE64;
        ly.snap[2ull * sz.L + i] = NONE64;
    }
    if (i < 2ull * MAX_MATCH_GRID) ly.xslot[i * XSLOT_WORDS] = 0;
    if (i == 0) {
        Control *ctl = ly.ctl;
        ctl->needs_remaining = ctl->needs_total;
        if (!ctl->error && ctl->needs_total > ctl->max_sends)
            record_error(ctl, ST_ENOMEM, (uint32_t)(ctl->needs_total >> 32), (uint32_t)ctl->needs_total, 0);
    }
}

// Inclusive scan of one value per thread over the workgroup (blockDim.x
// threads, whole waves), `part`: a word of LDS per wave.
__device__ __forceinline__ uint32_t block_scan(uint32_t x, uint32_t *part)
{
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    for (uint32_t o = 1; o < 64; o <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)x, o);
        if (lane >= o) x += y;
    }
    if (lane == 63) part[wave] = x;
    __syncthreads();
    for (uint32_t w = 0; w < wave; w++) x += part[w];
    return x;
}

// Neighbour-stepped matcher: the columns of device d are the chunks it needs
// in priority order.  Their number before each word of the needs row, and in
// all: one workgroup per device, four adjacent words per thread (at most
// 2^18 chunks, so one pass), loaded and written as whole 16-byte pieces.
__global__ void __launch_bounds__(1024) k_need_prefix(Layout ly, Sizes sz)
{
    static_assert(NBR_MAX_CHUNKS <= 1024u * 4u * 64u, "four words per thread hold a row");
    __shared__ uint32_t part[16];
    const uint32_t d = blockIdx.x, w = 4u * threadIdx.x;
    const uint64_t *row = ly.needs + (uint64_t)d * sz.Wp;
    uint32_t c[4] = {0, 0, 0, 0};
    const bool in = w < sz.Wp && !ly.ctl->error;  // (words past the last chunk's are zero)
    if (in) {
        const ulonglong2 a = *reinterpret_cast<const ulonglong2 *>(row + w), b = *reinterpret_cast<const ulonglong2 *>(row + w + 2);
        c[0] = (uint32_t)__popcll(a.x);
        c[1] = (uint32_t)__popcll(a.y);
        c[2] = (uint32_t)__popcll(b.x);
        c[3] = (uint32_t)__popcll(b.y);
    }
    const uint32_t n = c[0] + c[1] + c[2] + c[3], inc = block_scan(n, part), p = inc - n;
    if (in)
        *reinterpret_cast<uint4 *>(ly.need_pre + (uint64_t)d * sz.Wp + w) =
            make_uint4(p, p + c[0], p + c[0] + c[1], p + c[0] + c[1] + c[2]);
    if (threadIdx.x == blockDim.x - 1u) ly.dest_cols[d] = inc;
}

// Offsets, column lists and initial candidate rows (one workgroup per
// device).  Every workgroup sums the columns of the devices before its own
// (its send-log segment: a device's transfers are its columns) and their
// candidate words.  Then a thread per needs word writes the ranks of its
// columns, and a wave per 64 columns looks up the chunks' holders and, where
// a holder is the source of an in-link, sets the column's bit in the link's
// row: the 64 columns' words of all rows are put together in LDS and written
// as one piece (rows are stored word by word, in-links adjacent).  A scattered
// atomic per column kept the one workgroup of a rail switch busy for 100 us.
// Behind the rows lie, group by group of 64 row words, the rows' summary
// words (which words hold a bit).
constexpr uint32_t COL_BATCH = 4;   // 64-column groups one wave has in flight
__global__ void __launch_bounds__(1024) k_columns(Layout ly, Sizes sz)
{
    __shared__ uint8_t link_of[MAX_DEVICES_SP];  // in-link of d whose source is the device, 0xFF none
    __shared__ unsigned long long sums[4];       // columns and candidate words: before d, of all
    __shared__ unsigned long long word[16][MAX_IN_LINKS];  // per wave: one row word of every in-link
    __shared__ unsigned long long mid[MAX_IN_LINKS * 64];  // summary words
    const uint32_t d = blockIdx.x, tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    // the published entries start as those of windows -4 to -1
    if (sz.nbr_prune)
        for (uint32_t i = d * 1024u + tid; i < sz.L; i += gridDim.x * 1024u) ly.rel[i] = 0;
    for (uint32_t i = d * 1024u + tid; i < 4u * sz.pub_n; i += gridDim.x * 1024u)
        ly.pub[i] = (uint64_t)((0xFFCu + i / sz.pub_n) << NBR_TAG_SHIFT) << 32;
    if (tid < 4) sums[tid] = 0;
    for (uint32_t v = tid; v < sz.D; v += 1024) link_of[v] = 0xFFu;
    __syncthreads();
    {
        unsigned long long s[4] = {0, 0, 0, 0};
        for (uint32_t v = tid; v < sz.D; v += 1024) {
            const uint32_t m = ly.dest_cols[v];
            const unsigned long long r = cand_size(ly.in_off[v + 1] - ly.in_off[v], m);
            s[0] += v < d ? m : 0u;
            s[1] += v < d ? r : 0ull;
            s[2] += m;
            s[3] += r;
        }
#pragma unroll
        for (uint32_t i = 0; i < 4; i++) {
            for (int o = 32; o; o >>= 1) s[i] += __shfl_xor(s[i], o);
            if (lane == 0) atomicAdd(&sums[i], s[i]);
        }
    }
    __syncthreads();
    const unsigned long long log0 = sums[0], off = sums[1], total = sums[2];
    if (tid == 0) {
        ly.dest_log[d] = log0;
        ly.cand_off[d] = off;
        if (d == 0) {
            Control *ctl = ly.ctl;
            ctl->needs_total = total;
            if (!ctl->error && total > ctl->max_sends)
                record_error(ctl, ST_ENOMEM, (uint32_t)(total >> 32), (uint32_t)total, 0);
            else if (!ctl->error && sums[3] > sz.cand_words)
                record_error(ctl, ST_EINTERNAL, 4, 0, 0);
        }
    }
    const uint32_t M = ly.dest_cols[d];
    if (M == 0 || total > sz.max_sends || sums[3] > sz.cand_words) return;
    const uint32_t base = ly.in_off[d], n = ly.in_off[d + 1] - base, mw = (M + 63u) >> 6, mm = (mw + 63u) >> 6;
    uint64_t *rows = ly.cand + off;
    uint32_t *rank = ly.col_rank + log0;
    const uint64_t *need = ly.needs + (uint64_t)d * sz.Wp;
    const uint32_t *pre = ly.need_pre + (uint64_t)d * sz.Wp;
    for (uint32_t i = tid; i < n * mm; i += 1024) mid[i] = 0ull;
    for (uint32_t j = tid; j < n; j += 1024) link_of[ly.slot_src[base + j]] = (uint8_t)j;
    for (uint32_t w = tid; w < (uint32_t)sz.W; w += 1024) {
        uint32_t c = pre[w];
        for (uint64_t x = need[w]; x; x &= x - 1) rank[c++] = w * 64u + (uint32_t)__builtin_ctzll(x);
    }
    __syncthreads();
    unsigned long long *mine = word[wave];
    for (uint32_t w0 = wave; w0 < mw; w0 += 16 * COL_BATCH) {
        uint32_t r[COL_BATCH], s[COL_BATCH];
#pragma unroll
        for (uint32_t k = 0; k < COL_BATCH; k++) r[k] = rank[min((w0 + 16u * k) * 64u + lane, M - 1u)];
#pragma unroll
        for (uint32_t k = 0; k < COL_BATCH; k++) s[k] = ly.rank_src[r[k]];
#pragma unroll
        for (uint32_t k = 0; k < COL_BATCH; k++) {
            const uint32_t w = w0 + 16u * k;
            if (w >= mw) break;
            const uint32_t j = w * 64u + lane < M && s[k] != NONE32 ? link_of[s[k]] : 0xFFu;
            if (lane < n) mine[lane] = 0ull;
            wave_fence();
            if (j != 0xFFu) atomicOr(&mine[j], 1ull << lane);
            wave_fence();
            if (lane < n) {
                const unsigned long long x = mine[lane];
                rows[(uint64_t)w * n + lane] = x;
                if (x) atomicOr(&mid[(w >> 6) * n + lane], 1ull << (w & 63u));
            }
            wave_fence();
        }
    }
    __syncthreads();
    for (uint32_t i = tid; i < n * mm; i += 1024) rows[(uint64_t)mw * n + i] = mid[i];
}

// Which polled entries matter (run where some device polls many).  A transfer
// of chunk c over link q->u concerns u's out-neighbour d only if d needs c and
// q can offer c to u before d has it: q holds c from the start, or q needs c
// and some in-neighbour of q other than u and d ever holds c (holds it from
// the start or needs it; a device receives a chunk once, so what q had from u
// or d comes too late).  A relay switch polls none of its NPUs' in-links this
// way: what they receive came through it.
//
// First, per column of q: how many in-neighbours of q ever hold the chunk,
// kept above the rank in the column list.
constexpr uint32_t REL_COLS = 256;   // columns a workgroup takes at a time
constexpr uint32_t REL_BATCH = 8;    // in-links whose lookups are in flight together
__global__ void __launch_bounds__(REL_COLS) k_col_counts(Layout ly, Sizes sz)
{
    __shared__ uint32_t src[MAX_IN_LINKS];
    const uint32_t q = blockIdx.x, tid = threadIdx.x, M = ly.dest_cols[q];
    if (blockIdx.y * REL_COLS >= M || ly.ctl->error) return;
    const uint32_t base = ly.in_off[q], n = ly.in_off[q + 1] - base;
    if (tid < n) src[tid] = ly.slot_src[base + tid];
    __syncthreads();
    if (blockIdx.y == 0) {
        // per in-link x->q (a wave each): whether x is fed by q, and by which
        // of q's out-neighbours
        const uint32_t lane = tid & 63u, o0 = ly.out_off[q], m = ly.out_off[q + 1] - o0;
        const uint32_t dst = lane < m ? ly.out_dst[o0 + lane] : NONE32;
        for (uint32_t j = tid >> 6; j < n; j += REL_COLS / 64) {
            const uint32_t b = ly.in_off[src[j]], e = ly.in_off[src[j] + 1];
            const uint32_t s = b + lane < e ? ly.slot_src[b + lane] : NONE32;  // (at most 64 in-links)
            bool f = false;
            for (uint32_t p = 0; p < e - b; p++) f = f || (uint32_t)__builtin_amdgcn_readlane((int)s, (int)p) == dst;
            const uint64_t fm = __builtin_amdgcn_ballot_w64(f && lane < m), bk = __builtin_amdgcn_ballot_w64(s == q);
            if (lane == 0) {
                ly.feeds[base + j] = fm;
                ly.back[base + j] = bk ? 1u : 0u;
            }
        }
    }
    uint32_t *cols = ly.col_rank + ly.dest_log[q];
    for (uint32_t c = blockIdx.y * REL_COLS + tid; c < M; c += gridDim.y * REL_COLS) {
        const uint32_t r = cols[c], h = ly.rank_src[r], w = r >> 6;
        uint32_t cnt = 0;
        for (uint32_t j0 = 0; j0 < n; j0 += REL_BATCH) {
            uint64_t x[REL_BATCH];
#pragma unroll
            for (uint32_t k = 0; k < REL_BATCH; k++) x[k] = ly.needs[(uint64_t)src[min(j0 + k, n - 1u)] * sz.Wp + w];
#pragma unroll
            for (uint32_t k = 0; k < REL_BATCH; k++)
                if (j0 + k < n) cnt += (((x[k] >> (r & 63u)) & 1ull) || src[j0 + k] == h) ? 1u : 0u;
        }
        cols[c] = r | (cnt << NBR_COUNT_SHIFT);
    }
}

// Then, for every in-link q->u and out-link u->d of a device u, whether some
// column of u can come in over the one and concern the other's destination:
// bit rows over 256 columns at a time (offers of the in-links, without and
// with d among the excluded holders; needs of the out-neighbours), and an AND
// per pair of links.
__global__ void __launch_bounds__(REL_COLS) k_relevant(Layout ly, Sizes sz)
{
    constexpr uint32_t NW = REL_COLS / 64;
    __shared__ uint64_t offer[2][MAX_IN_LINKS][NW], wants[MAX_IN_LINKS][NW];
    __shared__ uint64_t feeds[MAX_IN_LINKS];  // per in-link q->u: out-neighbours d with a link d->q
    __shared__ uint32_t src[MAX_IN_LINKS], dst[MAX_IN_LINKS], back[MAX_IN_LINKS], log[MAX_IN_LINKS];
    const uint32_t u = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63u, M = ly.dest_cols[u];
    if (blockIdx.y * REL_COLS >= M || ly.ctl->error) return;
    const uint32_t base = ly.in_off[u], n = ly.in_off[u + 1] - base;
    const uint32_t o0 = ly.out_off[u], m = ly.out_off[u + 1] - o0;
    if (m == 0) return;
    if (tid < n) {
        src[tid] = ly.slot_src[base + tid];
        log[tid] = (uint32_t)ly.dest_log[src[tid]];
        feeds[tid] = ly.feeds[base + tid];
        back[tid] = ly.back[base + tid];
    }
    if (tid < m) dst[tid] = ly.out_dst[o0 + tid];
    __syncthreads();
    const uint32_t *cols = ly.col_rank + ly.dest_log[u];
    for (uint32_t c0 = blockIdx.y * REL_COLS; c0 < M; c0 += gridDim.y * REL_COLS) {
        const uint32_t c = c0 + tid, r = cols[min(c, M - 1u)] & NBR_RANK_MASK, h = ly.rank_src[r], w = r >> 6, b = r & 63u;
        const bool in = c < M;
        for (uint32_t j0 = 0; j0 < n; j0 += REL_BATCH) {
            uint64_t x[REL_BATCH];
            uint32_t pre[REL_BATCH], col[REL_BATCH];
#pragma unroll
            for (uint32_t k = 0; k < REL_BATCH; k++) {
                const uint64_t at = (uint64_t)src[min(j0 + k, n - 1u)] * sz.Wp + w;
                x[k] = ly.needs[at];
                pre[k] = ly.need_pre[at];
            }
#pragma unroll
            for (uint32_t k = 0; k < REL_BATCH; k++) {
                // (for a chunk q does not need the list's first entry, ignored)
                const bool nb = (x[k] >> b) & 1ull;
                col[k] = ly.col_rank[nb ? log[min(j0 + k, n - 1u)] + pre[k] + (uint32_t)__popcll(x[k] & ((1ull << b) - 1ull)) : 0u];
            }
#pragma unroll
            for (uint32_t k = 0; k < REL_BATCH; k++) {
                const uint32_t j = j0 + k;
                if (j >= n) break;
                const bool nb = (x[k] >> b) & 1ull, init = src[j] == h;
                const uint32_t cnt = nb ? col[k] >> NBR_COUNT_SHIFT : 0u;
                const uint64_t a0 = __builtin_amdgcn_ballot_w64(in && (init || cnt > back[j]));
                const uint64_t a1 = __builtin_amdgcn_ballot_w64(in && (init || cnt > back[j] + 1u));
                if (lane == 0) {
                    offer[0][j][wave] = a0;
                    offer[1][j][wave] = a1;
                }
            }
        }
        for (uint32_t k0 = 0; k0 < m; k0 += REL_BATCH) {
            uint64_t x[REL_BATCH];
#pragma unroll
            for (uint32_t k = 0; k < REL_BATCH; k++) x[k] = ly.needs[(uint64_t)dst[min(k0 + k, m - 1u)] * sz.Wp + w];
#pragma unroll
            for (uint32_t k = 0; k < REL_BATCH; k++) {
                if (k0 + k >= m) break;
                const uint64_t v = __builtin_amdgcn_ballot_w64(in && ((x[k] >> b) & 1ull));
                if (lane == 0) wants[k0 + k][wave] = v;
            }
        }
        __syncthreads();
        for (uint32_t j = wave; j < n; j += NW) {
            bool any = false;
            if (lane < m && src[j] != dst[lane]) {  // (not what d itself sends)
                const uint64_t *a = offer[(feeds[j] >> lane) & 1ull][j];
#pragma unroll
                for (uint32_t i = 0; i < NW; i++) any = any || (a[i] & wants[lane][i]) != 0;
            }
            const uint64_t am = __builtin_amdgcn_ballot_w64(any);
            if (am && lane == 0) atomicOr((unsigned long long *)&ly.rel[base + j], (unsigned long long)am);
        }
        __syncthreads();
    }
}

// Each device's list of polled entries: the relevant ones, and one in-link of
// every out-neighbour that reads its entries without being polled itself (a
// wave per device).
__global__ void __launch_bounds__(64) k_poll_lists(Layout ly, Sizes sz)
{
    if (ly.ctl->error) return;
    const uint32_t d = blockIdx.x, lane = threadIdx.x;
    const uint32_t p0 = ly.poll_off[d], np = ly.poll_off[d + 1] - p0, o0 = ly.out_off[d], m = ly.out_off[d + 1] - o0;
    const uint32_t base = ly.in_off[d], n = ly.in_off[d + 1] - base;
    uint32_t *out = ly.poll_use + p0 + o0;
    __shared__ uint32_t polled[MAX_IN_LINKS];  // in-link j's source has a polled entry
    if (lane < n) polled[lane] = 0;
    __syncthreads();
    uint32_t cnt = 0;
    for (uint32_t i0 = 0; i0 < np; i0 += 64) {
        const uint32_t i = i0 + lane, e = ly.poll[p0 + min(i, np - 1u)], j = e & 0xFFu;
        bool keep = false;
        if (i < np && j != 0xFFu) {
            const uint32_t sl = base + j, s = ly.slot_src[sl];
            keep = (ly.rel[ly.in_off[s] + ((e >> 8) - ly.pub_off[s])] >> ly.slot_out[sl]) & 1ull;
            if (keep) polled[j] = 1u;
        }
        const uint64_t km = __builtin_amdgcn_ballot_w64(keep);
        if (keep) out[cnt + (uint32_t)__popcll(km & ((1ull << lane) - 1ull))] = e;
        cnt += (uint32_t)__popcll(km);
    }
    __syncthreads();
    // which out-links' destinations read d's entries
    uint64_t readers = 0;
    for (uint32_t j = 0; j < n; j++) readers |= ly.rel[base + j];
    bool dep = lane < m && ((readers >> lane) & 1ull);
    uint32_t entry = 0;
    if (dep) {
        const uint32_t x = ly.out_dst[o0 + lane], xb = ly.in_off[x], xn = ly.in_off[x + 1] - xb;
        for (uint32_t j = 0; j < n; j++)
            if (polled[j] && ly.slot_src[base + j] == x) dep = false;
        for (uint32_t p = 0; p < xn; p++)
            if (ly.slot_src[xb + p] == d) entry = ((ly.pub_off[x] + p) << 8) | 0xFFu;
    }
    const uint64_t dm = __builtin_amdgcn_ballot_w64(dep);
    if (dep) out[cnt + (uint32_t)__popcll(dm & ((1ull << lane) - 1ull))] = entry;
    cnt += (uint32_t)__popcll(dm);
    if (lane == 0) ly.poll_cnt[d] = cnt;
}

inline uint32_t blocks_for(uint64_t n, uint32_t t) { return (uint32_t)((n + t - 1) / t); }

}  // namespace

hipError_t launch_setup(const Layout &ly, const Sizes &sz, const uint64_t *pre, const uint64_t *post,
                        const uint16_t *chunk_group, uint64_t seed, hipStream_t st)
{
    const uint32_t T = 256;
    const uint64_t C = sz.C, bm = (uint64_t)sz.D * sz.Wp / 2;
    k_reset<<<std::max(1u, std::min(blocks_for(std::max(bm, C), T), 2048u)), T, 0, st>>>(ly, sz);
    const dim3 gw(blocks_for(sz.W ? sz.W : 1, T), sz.N);
    if (sz.W) k_conditions<<<gw, T, 0, st>>>(ly, sz, pre, post, chunk_group);
    k_shortest_paths<<<sz.N, 512, sizeof(unsigned long long) * sz.D, st>>>(ly, sz);
    if (sz.W) k_chunk_dist<<<gw, T, 0, st>>>(ly, sz, pre, post);
    if (C && C <= SMALL_SORT) {
        k_order_small<<<1, 1024, 0, st>>>(ly, sz, seed);
    } else if (C) {
        k_keys_hash<<<blocks_for(C, T), T, 0, st>>>(ly, sz, seed);
        const hipError_t e = radix_sort_pairs(ly, C, 0, 8, sz.max_tiles, true, st);
        if (e != hipSuccess) return e;
        k_rank<<<blocks_for(C, T), T, 0, st>>>(ly, sz, seed);
    }
    if (C && !sz.cols) k_holds<<<blocks_for(C, T), T, 0, st>>>(ly, sz);
    if (sz.W) k_needs<<<gw, T, 0, st>>>(ly, sz, pre, post);
    if (sz.sw_nbt && C) k_adm_counts<<<dim3(blocks_for(C, T), sz.sw_nbt), T, 0, st>>>(ly, sz);
    if (sz.cols) {
        k_need_prefix<<<sz.D, (uint32_t)std::min<uint64_t>(1024, ((sz.W + 3) / 4 + 63) / 64 * 64 + (sz.W ? 0 : 64)), 0, st>>>(ly, sz);
        k_columns<<<sz.D, 1024, 0, st>>>(ly, sz);
        if (sz.nbr_prune && C) {
            const dim3 g(sz.D, std::min(blocks_for(C, REL_COLS), 64u));
            k_col_counts<<<g, REL_COLS, 0, st>>>(ly, sz);
            k_relevant<<<g, REL_COLS, 0, st>>>(ly, sz);
            k_poll_lists<<<sz.D, 64, 0, st>>>(ly, sz);
        }
        return hipGetLastError();
    }
    if (sz.L) k_link_counts<<<blocks_for(sz.L, 4), 256, 0, st>>>(ly, sz);
    k_needs_count<<<sz.D, 256, 0, st>>>(ly, sz);
    k_log_offsets<<<1, 1024, 0, st>>>(ly, sz);
    k_init_match<<<blocks_for(std::max<uint64_t>(sz.L, 4ull * MAX_MATCH_GRID), T), T, 0, st>>>(ly, sz);
    return hipGetLastError();
}

}  // namespace pccl

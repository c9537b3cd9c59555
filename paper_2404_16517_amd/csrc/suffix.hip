// Suffix sorting as repeated sorting of equal-length strings (the paper's
// Section 6 names suffix sorting based on sorting strings of equal length as
// the next application), space-efficiently: the suffixes T[i, N) overlap and
// are never stored.  Prefix doubling over ranks: rank_h(i) is the rank of
// suffix i's h-character prefix among all such prefixes (here the sorted
// position where its group of equal prefixes starts, plus one); the 2h-prefix
// of suffix i is the pair (rank_h(i), rank_h(i + h)) (rank 0 past the text).
// A step's groups are contiguous in the order so far, so the pairs' first
// halves need no sorting: the step sorts each group of two or more suffixes by
// rank_h(i + h) alone and leaves everything that is already distinct where it
// is.  The first step sorts all suffixes by their first K bytes followed by the
// remaining length capped at K (so that a suffix ending inside the window sorts
// before its extensions, whatever bytes follow).
//
// Sorting all N pairs in every step as strings cost 10 full sorts on 8 MB of
// text with one repeated passage of 2,000 bytes (17.0 ms); all steps after the
// second touch only a few thousand suffixes there, and the whole call takes
// 2.2 ms.
#include "sort_core.hpp"

#define SFX_K 6    // first step: K bytes and one length byte
#define SFX_T 64   // members of a group per 8 lanes

// First step: the key of T[i, i+K), zero-padded, then min(K, N - i); the low
// byte 8 marks equal keys as tied.  sa[i] = i.
__global__ void k_sfx_init(const u8 *T, u64 N, u64 *keys, u32 *sa)
{
    const u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    const u64 rem = N - i;
    const u32 take = rem < SFX_K ? (u32)rem : SFX_K;
    keys[i] = (load_be(T, N, i, take) & ~0xFFFFull) | ((u64)take << 8) | 8u;
    sa[i] = (u32)i;
}

// The whole text as the first step's one group, in the list of its size.
__global__ void k_sfx_first(u32 n, SortWs w, u32 block_max, u32 tile)
{
    for (u32 j = 0; j < C_NCTR; j++) w.ctr[j] = 0;
    const Seg g{0, n, 0, 0};
    if (n <= WS_MAX) {
        w.tiny[0] = g;
        w.ctr[C_TINY] = 1;
        w.ctr[C_TINYN] = n;
    } else if (n <= block_max) {
        (n <= BS_SMALL ? w.small : w.mid)[0] = g;
        w.ctr[n <= BS_SMALL ? C_SMALL : C_MID] = 1;
        w.ctr[C_SMALLN] = n;
    } else {
        w.largeA[0] = Seg{0, n, 0, SEG_NOROOT};
        w.ctr[C_LARGE] = 1;
        w.ctr[C_LTILES] = (n + tile - 1) / tile;
        w.ctr[C_LELEM] = n;
    }
}

// Tile counts (SFX_T members each) of the groups to sort; block 0 also resets
// the counters of the lists the step builds.
__global__ void k_sfx_tiles(const Seg *act, u32 nact, u32 *out, u32 *ctr)
{
    const u32 j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < nact) out[j] = (act[j].end - act[j].begin + SFX_T - 1) / SFX_T;
    if (j < C_NCTR) ctr[j] = 0;
}

// The same and the scan of the counts for up to LIST_ONE groups, in one launch
// (the later steps are launches and read-backs more than work).
__global__ __launch_bounds__(LIST_NT) void k_sfx_tiles_one(const Seg *act, u32 nact, u32 *tstart, u32 *ctr)
{
    if (threadIdx.x < C_NCTR) ctr[threadIdx.x] = 0;
    list_tiles(act, nact, SFX_T, tstart);
}

// One doubling step over the groups, eight lanes per 64 members: groups of up
// to eight are sorted by rank(i + h) at once (each lane counts the smaller
// keys), and what stays tied goes to the next list; of larger ones the keys are
// written and the group is routed to the sort of its size.  Bounded by the
// random reads of the ranks.
__global__ __launch_bounds__(256) void k_sfx_step(const Seg *act, const u32 *tstart, u32 nact, const u32 *rank,
                                                  u64 N, u64 h, u32 *sa, SortWs w, SortShape z)
{
    enum { NX = 0, TY, SM, MD, LG, TYN, SMN, LGT, LGN, NXN, CNT };
    __shared__ u32 c[CNT], base[5];
    if (threadIdx.x < CNT) c[threadIdx.x] = 0;
    __syncthreads();
    const u32 t = blockIdx.x * 32 + (threadIdx.x >> 3), gl = threadIdx.x & 7;
    u32 kind = CNT, slot = 0;
    Seg o{0, 0, 0, 0};
    if (t < tstart[nact]) {
        const u32 s = seg_of_tile(tstart, nact, t);
        const Seg g = act[s];
        const u32 m = g.end - g.begin;
        if (m <= 8) {  // (the same for the tile's eight lanes)
            const u32 v = gl < m ? sa[g.begin + gl] : 0u;
            const u32 k = gl < m ? ((u64)v + h < N ? rank[v + h] : 0u) : 0xFFFFFFFFu;  // (ranks are <= N < 2^32 - 1)
            u32 r = 0, eq = 0, eqb = 0;
#pragma unroll
            for (u32 j = 0; j < 8; j++) {
                const u32 y = __shfl(k, j, 8);
                r += (y < k || (y == k && j < gl)) ? 1u : 0u;
                eq += y == k ? 1u : 0u;
                eqb += (y == k && j < gl) ? 1u : 0u;
            }
            if (gl < m) {
                sa[g.begin + r] = v;
                if (eq > 1 && eqb == 0) {  // the first of a tied run
                    kind = NX;
                    o = Seg{g.begin + r, g.begin + r + eq, 0, 0};
                }
            }
        } else {
            const u32 lt = t - tstart[s], p0 = g.begin + lt * SFX_T;
            u32 v[SFX_T / 8];
#pragma unroll
            for (u32 q = 0; q < SFX_T / 8; q++) v[q] = p0 + 8 * q + gl < g.end ? sa[p0 + 8 * q + gl] : 0u;
#pragma unroll
            for (u32 q = 0; q < SFX_T / 8; q++) {
                const u32 p = p0 + 8 * q + gl;
                if (p < g.end) w.keyA[p] = ((u64)((u64)v[q] + h < N ? rank[v[q] + h] : 0u) << 32) | 8u;
            }
            if (lt == 0 && gl == 0) {
                o = Seg{g.begin, g.end, 0, 0};
                kind = m <= WS_MAX ? TY : (m > z.block_max ? LG : (m <= BS_SMALL ? SM : MD));
            }
        }
    }
    const u32 sz = o.end - o.begin;
    if (kind < CNT) {
        slot = atomicAdd(&c[kind], 1u);
        atomicAdd(&c[kind == NX ? NXN : (kind == TY ? TYN : (kind == LG ? LGN : SMN))], sz);
        if (kind == LG) atomicAdd(&c[LGT], (sz + z.tile - 1) / z.tile);
    }
    __syncthreads();
    if (threadIdx.x < CNT && c[threadIdx.x]) {
        const u32 to[CNT] = {C_NEXT, C_TINY, C_SMALL, C_MID, C_LARGE, C_TINYN, C_SMALLN, C_LTILES, C_LELEM, C_NELEM};
        u32 x = 0;
#pragma unroll
        for (u32 q = 0; q < CNT; q++)
            if (threadIdx.x == q) x = to[q];
        const u32 at = atomicAdd(&w.ctr[x], c[threadIdx.x]);
        if (threadIdx.x < 5) base[threadIdx.x] = at;
    }
    __syncthreads();
    if (kind == NX) w.nxt[base[NX] + slot] = o;
    else if (kind == TY) w.tiny[base[TY] + slot] = o;
    else if (kind == SM) w.small[base[SM] + slot] = o;
    else if (kind == MD) w.mid[base[MD] + slot] = o;
    else if (kind == LG) w.largeA[base[LG] + slot] = Seg{o.begin, o.end, o.depth, SEG_NOROOT};
}

// Ranks of every suffix as if it were alone in its group: its position + 1.
__global__ void k_sfx_rank_all(const u32 *sa, u64 N, u32 *rank)
{
    const u64 p = (u64)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < N) rank[sa[p]] = (u32)p + 1;
}

// Ranks of the members of a list's groups: as above, or (TIED) the group's.
template <bool TIED>
__global__ __launch_bounds__(256) void k_sfx_rank(const Seg *list, const u32 *tstart, u32 cnt, const u32 *sa, u32 *rank)
{
    const u32 t = blockIdx.x * 32 + (threadIdx.x >> 3), gl = threadIdx.x & 7;
    if (t >= tstart[cnt]) return;
    const u32 s = seg_of_tile(tstart, cnt, t);
    const Seg g = list[s];
    const u32 p0 = g.begin + (t - tstart[s]) * SFX_T, p1 = g.end < p0 + SFX_T ? g.end : p0 + SFX_T;
    for (u32 p = p0 + gl; p < p1; p += 8) rank[sa[p]] = (TIED ? g.begin : p) + 1;
}

// lcp[k] = lcp of the suffixes at sorted positions k-1 and k, by comparison
// (cost: the sum of the LCPs, the suffixes' D).  Every lane compares its first
// 64 bytes; pairs that agree on those are compared one after the other by the
// whole wavefront, 512 bytes a step, so that one repeated passage does not keep
// a lane busy for its length in 8-byte steps.
__global__ __launch_bounds__(256) void k_sfx_lcp(const u8 *T, u64 N, const u32 *sa, u32 *lcp)
{
    const u64 k = (u64)blockIdx.x * blockDim.x + threadIdx.x;
    const bool on = k > 0 && k < N;
    const u64 a = on ? sa[k - 1] : 0ull, b = on ? sa[k] : 0ull;
    const u64 m = on ? N - (a > b ? a : b) : 0ull;
    u64 l = 0;
    bool open = m > 0;
    while (open && l < 64) {
        const u32 take = (m - l) < 8 ? (u32)(m - l) : 8u;
        const u64 x = load_be(T, N, a + l, take), y = load_be(T, N, b + l, take);
        if (x != y) {
            l += __clzll(x ^ y) >> 3;
            open = false;
        } else {
            l += take;
            open = l < m;
        }
    }
    const u32 lane = threadIdx.x & 63;
    for (u64 left = __ballot(open); left; left &= left - 1) {  // (uniform over the wavefront)
        const int src = __ffsll((unsigned long long)left) - 1;
        const u64 wa = __shfl(a, src, 64), wb = __shfl(b, src, 64), wm = __shfl(m, src, 64);
        for (u64 c = 64;; c += 512) {
            const u64 q = c + 8ull * lane;
            const u32 take = q < wm ? (wm - q < 8 ? (u32)(wm - q) : 8u) : 0u;
            const u64 x = load_be(T, N, wa + q, take), y = load_be(T, N, wb + q, take);
            const u64 stop = __ballot(x != y || take < 8);
            if (stop) {
                const int at = __ffsll((unsigned long long)stop) - 1;
                const u64 r = __shfl(x != y ? q + (__clzll(x ^ y) >> 3) : q + take, at, 64);
                if ((int)lane == src) l = r;
                break;
            }
        }
    }
    if (k < N) lcp[k] = (u32)l;
}

struct SfxWs {
    u32 *rank, *tiles;  // tiles: starts of the tiles of every group of a step
    SortWs sort;
};

static void sfx_layout(u64 N, SfxWs *w, WsArena *a, WsCounter *c)
{
    const u64 groups = N / 2 + 2;
    if (a) {
        w->rank = a->take<u32>(N);
        w->tiles = a->take<u32>(groups);
    } else {
        c->take<u32>(N);
        c->take<u32>(groups);
    }
    sort_ws_layout(N, &w->sort, a, c);
}

extern "C" size_t ss_suffix_sort_workspace(uint64_t N)
{
    WsCounter c;
    SfxWs w;
    sfx_layout(N, &w, nullptr, &c);
    return c.used;
}

extern "C" int ss_suffix_sort(const uint8_t *text, uint64_t N, uint32_t *sa, uint32_t *lcp, uint32_t *steps_host,
                              void *ws, size_t ws_bytes, void *stream)
{
    ss_clear_error();
    if (steps_host) *steps_host = 0;
    if (N >= 0xFFFFFFFFull) {
        ss_set_error("text of %llu bytes beyond the 32-bit index limit", (unsigned long long)N);
        return SS_ERR_TOO_LARGE;
    }
    if (N == 0) return SS_OK;
    if (!text || !sa) {
        ss_set_error("null text or sa");
        return SS_ERR_INVALID_ARG;
    }
    WsArena a(ws, ws_bytes);
    SfxWs w;
    sfx_layout(N, &w, &a, nullptr);
    if (a.overflow || !ws) {
        ss_set_error("workspace too small: need %zu bytes", ss_suffix_sort_workspace(N));
        return SS_ERR_WORKSPACE;
    }
    hipStream_t st = (hipStream_t)stream;
    SortWs &sw = w.sort;
    const SortShape z = sort_shape(N);
    const unsigned g = (unsigned)ceil_div(N, 256);
    SortJob J{text, N, nullptr, sa, sw.lcp_scratch, st, N, N};
    u32 ctr[C_NCTR];
    k_sfx_init<<<g, 256, 0, st>>>(text, N, sw.keyA, sa);
    SS_CHECK_LAUNCH();
    k_sfx_first<<<1, 1, 0, st>>>((u32)N, sw, z.block_max, z.tile);
    SS_CHECK_LAUNCH();
    SS_TRY(sort_keyed(J, sw, ctr));
    u64 h = SFX_K;
    u32 steps = 1, nact = ctr[C_NEXT], elems = ctr[C_NELEM];
    if (nact > 0 && h < N) {
        k_sfx_rank_all<<<g, 256, 0, st>>>(sa, N, w.rank);
        SS_CHECK_LAUNCH();
    }
    while (nact > 0 && h < N) {
        // the groups left (in sw.nxt): their members' ranks, one step over
        // them, and the ranks that the step's order gives (the next turn
        // corrects those of the groups still tied)
        Seg *tmp = sw.act; sw.act = sw.nxt; sw.nxt = tmp;
        const unsigned tg = (unsigned)ceil_div((u64)nact + elems / SFX_T, 32);  // (at most one part tile per group)
        if (nact <= LIST_ONE) {
            k_sfx_tiles_one<<<1, LIST_NT, 0, st>>>(sw.act, nact, w.tiles, sw.ctr);
            SS_CHECK_LAUNCH();
        } else {
            k_sfx_tiles<<<(unsigned)ceil_div(nact, 256), 256, 0, st>>>(sw.act, nact, w.tiles, sw.ctr);
            SS_CHECK_LAUNCH();
            SS_TRY(ss_scan_exclusive<u32>(w.tiles, w.tiles, nact, (u32 *)sw.scan_scratch, st));
        }
        k_sfx_rank<true><<<tg, 256, 0, st>>>(sw.act, w.tiles, nact, sa, w.rank);
        SS_CHECK_LAUNCH();
        k_sfx_step<<<tg, 256, 0, st>>>(sw.act, w.tiles, nact, w.rank, N, h, sa, sw, z);
        SS_CHECK_LAUNCH();
        SS_TRY(sort_keyed(J, sw, ctr));
        if (ctr[C_NEXT] > 0) {
            k_sfx_rank<false><<<tg, 256, 0, st>>>(sw.act, w.tiles, nact, sa, w.rank);
            SS_CHECK_LAUNCH();
        }
        steps++;
        h *= 2;
        nact = ctr[C_NEXT];
        elems = ctr[C_NELEM];
    }
    if (lcp) {
        k_sfx_lcp<<<g, 256, 0, st>>>(text, N, sa, lcp);
        SS_CHECK_LAUNCH();
    }
    if (steps_host) *steps_host = steps;
    return SS_OK;
}

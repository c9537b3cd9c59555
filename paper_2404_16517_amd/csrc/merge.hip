// Front-coding decode and LCP-aware k-way merge of sorted runs (Section 3,
// step 3; the LCP-aware merge building block of Section 2).
//
// Decode.  Within a run, string i equals the first e_i bytes of string i-1
// followed by its literal.  Its bytes [e_i, d_i) are its own literal; bytes
// [e_j, e_i) with j = psv(i) = the nearest earlier position with e_j < e_i are
// string j's literal, and so on down the psv chain to an e = 0 position (every
// run starts with e = 0).  psv is found by a min-tree search: inside each
// 1024-element block on a tree in LDS, else on a binary tree of the block
// minima (climb to the nearest left subtree holding a smaller value, descend to
// its rightmost such block, then its rightmost such 16-element chunk).  Each output 16-byte word then walks
// the chain of its string.
//
// Merge.  The paper merges r runs with an LCP loser tree, one element after
// the other.  Here every element caches its 7 bytes at its group's common
// prefix (found by one scan over the runs) as a 64-bit key, and the runs of a
// group are merged by key in one pass over memory: sampled keys cut the runs
// into tiles of about a thousand outputs (a tile holds all elements with keys
// in one interval, so equal keys never part), and each tile's windows are merged
// in LDS.  Different keys give the LCP of neighbours too.  Only elements whose
// whole keys tie -- equal strings, mostly -- are compared as strings: small
// ties directly, the others by further keys and the segmented sort.
#include <string.h>

#include <algorithm>
#include <vector>

#include <mutex>

#include "sort_core.hpp"

#define PSV_NONE 0xFFFFFFFFu

// ---------------------------------------------------------------- decode

// The format check of the runs; the lengths go out widened for their scan.
__global__ __launch_bounds__(256) void k_check_runs(const u64 *run_off, u32 k, const u32 *e, const u32 *d,
                                                    u32 n, u32 *bad, u64 *len)
{
    const u32 i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0 && (run_off[0] != 0 || run_off[k] != n)) atomicOr(bad, 1u);
    if (i < k) {
        const u64 s = run_off[i];
        if (run_off[i + 1] < s || run_off[i + 1] > n) atomicOr(bad, 1u);
        else if (run_off[i + 1] > s && e[s] != 0) atomicOr(bad, 2u);
    }
    if (i < n) {
        const u32 di = d[i];
        len[i] = di;
        if (e[i] > di) atomicOr(bad, 4u);
        if (i > 0 && e[i] > d[i - 1]) atomicOr(bad, 4u);
    }
}

// p[0..count) = v (a kernel rather than hipMemsetAsync, so that a captured
// graph holds no memset node).
__global__ void k_fill_u32(u32 *p, u32 v, u32 count)
{
    const u32 i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = v;
}

#define PB 1024  // psv block (one workgroup)
#define PC 16    // chunk whose minimum is kept for the far search
#define PCB (PB / PC)

// psv inside each block of PB entries (PSV_NONE if the answer lies before the
// block).  The block minimum goes to leaf P + block of the tree T, the minima
// of its PC-entry chunks to cm[block * PCB ..].  This and the kernels below do
// nothing when `need` is given and points to zero.
__global__ __launch_bounds__(PB) void k_psv_block(const u32 *e, u32 n, u32 *psv, u32 *T, u32 P, u32 *cm,
                                                 u32 *farl, u32 *fcnt, const u32 *need)
{
    if (need && *need == 0) return;
    __shared__ u32 t[2 * PB];  // heap: node x has children 2x, 2x+1; leaves PB..2PB-1
    const u32 b0 = blockIdx.x * PB;
    const u32 i = b0 + threadIdx.x;
    const u32 v = i < n ? e[i] : 0xFFFFFFFFu;
    t[PB + threadIdx.x] = v;
    __syncthreads();
    for (u32 c = PB / 2; c >= 1; c >>= 1) {
        if (threadIdx.x < c) {
            const u32 x = c + threadIdx.x;
            const u32 a = t[2 * x], b = t[2 * x + 1];
            t[x] = a < b ? a : b;
        }
        __syncthreads();
    }
    bool far = false;  // the answer lies before this block: left to k_psv_far
    if (i < n) {
        u32 res = PSV_NONE;
        if (v > 0) {
            u32 x = PB + threadIdx.x;
            bool found = false;
            while (x > 1) {
                if ((x & 1) && t[x - 1] < v) {
                    x = x - 1;
                    found = true;
                    break;
                }
                x >>= 1;
            }
            if (found) {
                while (x < PB) {
                    x = 2 * x + 1;
                    if (t[x] >= v) x--;
                }
                res = b0 + (x - PB);
            }
            far = !found;
        }
        psv[i] = res;
    }
    // this block's far entries, compacted to farl[b0 ..], their count in fcnt[block]
    __shared__ u32 wcnt[PB / 64];
    const u64 fm = __ballot(far);
    const u32 wid = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) wcnt[wid] = (u32)__popcll(fm);
    __syncthreads();
    u32 wb = 0;
    for (u32 q = 0; q < wid; q++) wb += wcnt[q];
    if (far) farl[b0 + wb + (u32)__popcll(fm & lanemask_lt())] = i;
    if (threadIdx.x == 0) {
        u32 tot = 0;
        for (u32 q = 0; q < PB / 64; q++) tot += wcnt[q];
        fcnt[blockIdx.x] = tot;
    }
    if (threadIdx.x == 0) T[P + blockIdx.x] = t[1];
    if (threadIdx.x < PCB) cm[(u64)blockIdx.x * PCB + threadIdx.x] = t[PCB + threadIdx.x];
}

// Internal nodes of the tree T: each workgroup takes up to 512 nodes of one
// level (m nodes, indices m..2m-1) and writes `lv` levels above them.
__global__ __launch_bounds__(256) void k_tree_up(u32 *T, u32 m, u32 lv, const u32 *need)
{
    if (need && *need == 0) return;
    __shared__ u32 s[512];
    const u32 cnt = m < 512 ? m : 512;
    const u32 base = m + blockIdx.x * cnt;
    for (u32 q = threadIdx.x; q < cnt; q += 256) s[q] = T[base + q];
    __syncthreads();
    u32 c = cnt, b = base;
    for (u32 L = 0; L < lv; L++) {
        c >>= 1;
        b >>= 1;
        u32 v = 0;
        if (threadIdx.x < c) {
            const u32 x = s[2 * threadIdx.x], y = s[2 * threadIdx.x + 1];
            v = x < y ? x : y;
        }
        __syncthreads();
        if (threadIdx.x < c) {
            s[threadIdx.x] = v;
            T[b + threadIdx.x] = v;
        }
        __syncthreads();
    }
}

// psv for positions whose answer lies before their block: nearest left
// subtree of T with a smaller minimum, its rightmost such block, that block's
// rightmost such chunk, that chunk's rightmost such entry.
__device__ __forceinline__ void psv_far_one(const u32 *e, const u32 *T, u32 P, const u32 *cm, u32 i, u32 n,
                                            u32 *psv)
{
    const u32 v = e[i];
    u32 x = P + i / PB;
    bool found = false;
    while (x > 1) {
        if ((x & 1) && T[x - 1] < v) {
            x = x - 1;
            found = true;
            break;
        }
        x >>= 1;
    }
    if (!found) return;  // malformed input (no e = 0 before): stays PSV_NONE
    while (x < P) {
        x = 2 * x + 1;
        if (T[x] >= v) x--;
    }
    const u32 blk = x - P;
    const uint4 *c4 = (const uint4 *)(cm + (u64)blk * PCB);  // 256-byte aligned workspace
    uint4 w[PCB / 4];
#pragma unroll
    for (int q = 0; q < PCB / 4; q++) w[q] = c4[q];
    int c = -1;
#pragma unroll
    for (int q = 0; q < PCB / 4; q++) {
        if (w[q].x < v) c = 4 * q;
        if (w[q].y < v) c = 4 * q + 1;
        if (w[q].z < v) c = 4 * q + 2;
        if (w[q].w < v) c = 4 * q + 3;
    }
    // the block minimum is < v, so some chunk qualifies (c >= 0), and that
    // chunk's entries all lie below n (padding entries are all-ones)
    const u32 lo = blk * PB + (u32)c * PC;
    u32 ev[PC];
#pragma unroll
    for (int q = 0; q < PC; q++) ev[q] = (lo + q < n) ? e[lo + q] : 0xFFFFFFFFu;
    u32 r = lo;
#pragma unroll
    for (int q = 0; q < PC; q++)
        if (ev[q] < v) r = lo + (u32)q;
    psv[i] = r;
}

// Workgroup b takes the far entries k_psv_block b left, packed at
// farl[b*PB ..] (fcnt[b] of them); each walk is a chain of dependent loads,
// so packing keeps the walks of a block in as few wavefronts as possible.
__global__ __launch_bounds__(256) void k_psv_far(const u32 *e, const u32 *T, u32 P, const u32 *cm, const u32 *farl,
                                                 const u32 *fcnt, u32 n, u32 *psv, const u32 *need)
{
    if (need && *need == 0) return;
    const u32 cnt = fcnt[blockIdx.x];
    const u32 *lst = farl + (u64)blockIdx.x * PB;
    for (u32 q = threadIdx.x; q < cnt; q += blockDim.x) psv_far_one(e, T, P, cm, lst[q], n, psv);
}

// Tree size (leaves) for n entries.
static u32 psv_leaves(u64 n)
{
    const u64 nb = ceil_div(n, PB);
    u32 P = 1;
    while (P < nb) P <<= 1;
    return P;
}

// psv of every entry of e[0..n) (n >= 1).  T holds 2 * psv_leaves(n) words,
// cm psv_leaves(n) * PCB words (256-byte aligned).  Skipped on the device
// when `need` is given and points to zero.
static int psv_build(const u32 *e, u64 n, u32 *psv, u32 *T, u32 *cm, u32 *farl, u32 *fcnt, hipStream_t st,
                     const u32 *need = nullptr)
{
    if (n == 0) return SS_OK;
    const u32 nb = (u32)ceil_div(n, PB);
    const u32 P = psv_leaves(n);
    if (P > nb) {
        k_fill_u32<<<(unsigned)ceil_div(P - nb, 256), 256, 0, st>>>(T + P + nb, 0xFFFFFFFFu, P - nb);
        SS_CHECK_LAUNCH();
    }
    {
        SS_PROF("k_psv_block", st, (double)n * 8.0);  // e in, psv out
        k_psv_block<<<nb, PB, 0, st>>>(e, (u32)n, psv, T, P, cm, farl, fcnt, need);
    }
    SS_CHECK_LAUNCH();
    for (u32 m = P; m > 1;) {
        u32 lv = 0;
        while (lv < 9 && (m >> lv) > 1) lv++;
        const u32 blocks = m > 512 ? m / 512 : 1;
        k_tree_up<<<blocks, 256, 0, st>>>(T, m, lv, need);
        SS_CHECK_LAUNCH();
        m >>= lv;
    }
    {
        // (far entries only: their value, the tree path, one chunk)
        SS_PROF("k_psv_far", st, 0.0);
        k_psv_far<<<nb, 256, 0, st>>>(e, T, P, cm, farl, fcnt, (u32)n, psv, need);
    }
    SS_CHECK_LAUNCH();
    return SS_OK;
}

#define DC_NT 256
#define DC_SPAN 16384  // output bytes a chunk covers at most (64 per thread)
#define DC_WU 2        // words a thread has in flight
#define DC_MID 32      // bytes between the literals up to which a string's own thread fetches them
// copy words of a chunk: 16-byte words of the span, and two shared ones per piece
#define DC_WORDS (DC_SPAN / 16 + 4 * DC_NT + 2)

// What a decoded string takes from the strings before it, as a scan along the
// front-coded order: the string's first 8 bytes (win, little-endian), and its
// head, the nearest entry with e <= 8 at or before it, whose literal holds all
// its bytes from 8 on (byte k at hsuf + k) and whose first F bytes the string
// shares.  An entry keeps the first p = min(e, 8) bytes of its predecessor's
// window and brings the rest; one with e <= 8 is a new head.
struct DOp {
    u64 win, hsuf;
    u32 F;
    u32 rp;  // bits 0..3: p, bit 4: a head
};

__device__ __forceinline__ u64 low_bytes(u32 k) { return k >= 8 ? ~0ull : ((1ull << (8 * k)) - 1ull); }

// a, then b
__device__ __forceinline__ DOp dop_cat(const DOp &a, const DOp &b)
{
    const bool head = (b.rp & 16u) != 0;
    const u32 pa = a.rp & 15u, pb = b.rp & 15u;
    const u64 keep = low_bytes(pb);
    DOp r;
    r.win = (a.win & keep) | (b.win & ~keep);
    r.hsuf = head ? b.hsuf : a.hsuf;
    r.F = head || b.F < a.F ? b.F : a.F;
    r.rp = ((a.rp | b.rp) & 16u) | (pa < pb ? pa : pb);
    return r;
}

__device__ __forceinline__ DOp dop_shfl_up(const DOp &a, u32 d)
{
    DOp r;
    r.win = __shfl_up(a.win, d, 64);
    r.hsuf = __shfl_up(a.hsuf, d, 64);
    r.F = __shfl_up(a.F, d, 64);
    r.rp = __shfl_up(a.rp, d, 64);
    return r;
}

// Largest i in [0, n) with a[i] <= x (a[0] <= x), by one wavefront: 64 probes
// a step, so four dependent loads serve 16M entries.
__device__ __forceinline__ u32 wave_find(const u64 *a, u32 n, u64 x)
{
    u32 lo = 0, len = n;  // the answer lies in [lo, lo + len)
    const u32 lane = threadIdx.x & 63;
    while (len > 1) {
        const u32 step = (len + 63) / 64;
        const u64 q = (u64)lane * step;
        const bool le = q < len && a[lo + q] <= x;
        const u32 c = (u32)__popcll(__ballot(le));  // (monotone: a prefix of the lanes)
        const u32 k = c ? c - 1 : 0u;
        lo += k * step;
        len = len - k * step < step ? len - k * step : step;
    }
    return lo;
}

// Bytes v (little-endian) or-ed into an LDS buffer at byte position `at`.
__device__ __forceinline__ void buf_or(u64 *buf, u32 at, u64 v)
{
    const u32 r = at & 7u;
    atomicOr((unsigned long long *)&buf[at >> 3], (unsigned long long)(v << (8 * r)));
    if (r) atomicOr((unsigned long long *)&buf[(at >> 3) + 1], (unsigned long long)(v >> (64 - 8 * r)));
}

// Decode: the output [0, out_off[n]) is dealt to the workgroups in contiguous
// ranges, and each walks its range in chunks of at most DC_NT strings and
// DC_SPAN bytes.  A chunk's strings are read once, one per thread, with a scan
// that gives every string its first 8 bytes and its head (DOp); the state
// after a chunk is carried to the next, and only the first string of a range
// is found by walking its psv chain.  Then the chunk is assembled in LDS: a
// string's bytes below 8 come from its window, those from e on from its own
// literal, those below F from its head's (all of an equal string's, as runs of
// equal strings share their head), and only what lies between walks the psv
// chain.  The two literal pieces of every string are cut at the buffer's
// 16-byte words, and the words dealt evenly to the threads, which keep DC_WU
// of them in flight.  What lies between is a few bytes in short strings, which
// the string's thread fetches itself; more than DC_MID are dealt out by words
// as well, a chain walk each (20,000 strings of 5,000 bytes, their LCPs uniform:
// 1520 us a call where one thread fetched all of them, now 242).
//
// The bytes in and out bound it at best; in practice the latency of the loads
// and the vector instructions per word.  2M text strings (132 MB out): 566 us
// with a global search per thread and single bytes moved, each piece by a
// chain walk; 180 us with threads owning 16-byte words of the output (a search,
// up to four pieces and their shifts: 560 instructions a word); 160 us with
// four lanes per string (one load in flight per lane); 103 us in this form.
// Nothing is written unless status is null or 0.
__global__ __launch_bounds__(DC_NT, 5) void k_decode(const u32 *e, const u32 *d, const u64 *suf_off, const u8 *suf,
                                                  const u32 *psv, u32 n, const u64 *out_off, const u32 *status,
                                                  u8 *out)
{
    __shared__ u64 s_src[2 * DC_NT], s_cend;
    __shared__ u16 s_at[2 * DC_NT], s_end[2 * DC_NT], s_base[2 * DC_NT], s_own[DC_WORDS];
    __shared__ u32 s_wsum[DC_NT / 64];
    __shared__ DOp s_tot[DC_NT / 64], s_carry;
    // bytes between a string's literals that are dealt out: from byte s_mk of the
    // string, buffer positions [s_ma, s_mb); s_mid: some string has them
    __shared__ u64 s_mk[DC_NT];
    __shared__ u16 s_ma[DC_NT], s_mb[DC_NT];
    __shared__ u32 s_r0, s_mid;
    __shared__ __attribute__((aligned(16))) u64 buf[DC_SPAN / 8 + 2];
    if (status && *status != 0) return;  // (uniform)
    const u64 total = out_off[n], sufN = suf_off[n];
    const u32 mis = (u32)((uintptr_t)out & 15);
    // this workgroup's range, its bounds on 16-byte words of the output
    u64 per = (total + mis + gridDim.x - 1) / gridDim.x;
    per = (per + 15) & ~15ull;
    u64 c0 = blockIdx.x * per, r1 = c0 + per;
    c0 = c0 > mis ? c0 - mis : 0;
    r1 = r1 - mis < total ? r1 - mis : total;  // (per >= 16 > mis)
    if (c0 >= r1) return;
    const u32 lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    for (u32 w = threadIdx.x; w < DC_SPAN / 8 + 2; w += DC_NT) buf[w] = 0;
    if (wv == 0) {
        const u32 r = wave_find(out_off, n, c0);
        if (lane == 0) {
            // the first string's own state, along its psv chain (its operator
            // applied to that state gives it again)
            DOp c{0ull, 0ull, 0xFFFFFFFFu, 16u};
            u32 j = r, ej = e[r], h = d[r];
            bool found = false;  // the head
            for (;;) {
                const u64 so = suf_off[j];
                if (ej <= 8 && !found) {
                    found = true;
                    c.hsuf = so - ej;
                }
                if (!found) c.F = ej;
                const u32 m = h < 8 ? h : 8u;
                if (ej < m) c.win |= load_le(suf, sufN, so, m - ej) << (8 * ej);
                if (ej == 0) break;
                h = ej;
                j = psv[j];
                ej = e[j];
            }
            s_carry = c;
            s_r0 = r;
            s_mid = 0;
        }
    }
    __syncthreads();
    const u32 t = threadIdx.x;
    u32 ei = 0, di = 0;  // this thread's string of the chunk
    u64 so = 0, oo = 0;
    if (s_r0 + t < n) {
        ei = e[s_r0 + t];
        di = d[s_r0 + t];
        so = suf_off[s_r0 + t];
        oo = out_off[s_r0 + t];
    }
    for (;;) {  // chunks (uniform over the workgroup)
        const u32 r0 = s_r0;
        const u32 ns = n - r0 < DC_NT ? n - r0 : DC_NT;
        DOp o{0ull, 0ull, 0xFFFFFFFFu, 8u};
        if (t < ns) {
            if (t == ns - 1) s_cend = oo + di;
            o.rp = (ei < 8 ? ei : 8u) | (ei <= 8 ? 16u : 0u);
            o.F = ei <= 8 ? 0xFFFFFFFFu : ei;
            o.hsuf = so - ei;
            const u32 m = di < 8 ? di : 8u;
            if (ei < m) o.win = load_le(suf, sufN, so, m - ei) << (8 * ei);
        }
        // The scan over the wavefront: a string's head is the highest lane at
        // or below its own that is one; windows and minima in six steps.
        const u64 heads = __ballot((o.rp & 16u) != 0), upto = heads & (lane == 63 ? ~0ull : (2ull << lane) - 1ull);
        const u32 hl = upto ? 63u - (u32)__clzll(upto) : 0u;  // (0: no head below, minima from lane 0 on)
        DOp inc = o;
        inc.hsuf = __shfl(o.hsuf, hl, 64);
        u32 p = o.rp & 15u;
#pragma unroll
        for (u32 q = 1; q < 64; q <<= 1) {
            const u64 yw = __shfl_up(inc.win, q, 64);
            const u32 yF = __shfl_up(inc.F, q, 64), yp = __shfl_up(p, q, 64);
            if (lane >= q) {
                const u64 keep = low_bytes(p);
                inc.win = (yw & keep) | (inc.win & ~keep);
                p = yp < p ? yp : p;
            }
            if (lane >= hl + q) inc.F = yF < inc.F ? yF : inc.F;
        }
        inc.rp = p | (upto ? 16u : 0u);
        if (lane == 63) s_tot[wv] = inc;
        DOp st = s_carry;
        __syncthreads();
        for (u32 w = 0; w < wv; w++) st = dop_cat(st, s_tot[w]);
        const DOp pre0 = st;  // the state before this wavefront
        st = dop_cat(st, inc);
        // the chunk's end; the string that holds it starts the next chunk
        const u64 cend = s_cend;
        u64 c1 = c0 + DC_SPAN - ((uintptr_t)(out + c0) & 15);
        c1 = c1 < r1 ? c1 : r1;
        c1 = c1 < cend ? c1 : cend;
        {
            const DOp up = dop_shfl_up(st, 1);
            if (t < ns) {
                if (c1 == cend) {
                    if (t == ns - 1) {
                        s_carry = st;
                        s_r0 = r0 + ns;
                    }
                } else if (oo <= c1 && c1 < oo + di) {
                    // the state before the string
                    s_carry.win = lane ? up.win : pre0.win;
                    s_carry.hsuf = lane ? up.hsuf : pre0.hsuf;
                    s_carry.F = lane ? up.F : pre0.F;
                    s_carry.rp = lane ? up.rp : pre0.rp;
                    s_r0 = r0 + t;
                }
            }
        }
        // This thread's string in the chunk.  Its window bytes and what only
        // its psv chain holds go to the buffer (buf[lead] = output byte c0) at
        // once; the piece of its head's literal and the one of its own become
        // copies of as many 16-byte words as they touch.
        const u32 lead = (u32)((uintptr_t)(out + c0) & 15);
        u32 wc0 = 0, wc1 = 0;  // words of the two pieces
        s_ma[t] = s_mb[t] = 0;
        if (t < ns && oo < c1) {
            const u64 k0 = oo < c0 ? c0 - oo : 0ull;  // bytes [k0, kend) lie in the chunk
            const u64 kend = (oo + di < c1 ? oo + di : c1) - oo;
            const u64 rel = oo - c0 + lead;           // byte k is at buffer position k + rel (mod 2^64)
            u64 k = k0;
            if (k < 8 && k < kend) {
                const u64 m = kend < 8 ? kend : 8ull;
                buf_or(buf, (u32)(k + rel), (st.win & low_bytes((u32)m)) >> (8 * k));
                k = m;
            }
            const u64 eb = ei < kend ? ei : kend, fb = st.F < eb ? st.F : eb;
            u64 src = st.hsuf + k, q = k;
            if (k < fb) q = fb;
            s_at[2 * t] = (u16)(k + rel);
            s_end[2 * t] = (u16)(q + rel);
            s_src[2 * t] = src;
            if (q > k) wc0 = (u32)((q + rel + 15) / 16 - (k + rel) / 16);
            k = q;
            if (k + DC_MID < eb) {
                s_mk[t] = k;
                s_ma[t] = (u16)(k + rel);
                s_mb[t] = (u16)(eb + rel);
                s_mid = 1;
                k = eb;
            }
            while (k < eb) {
                u32 h = ei, j = psv[r0 + t], ej = e[j];
                while (ej > k) {
                    h = ej;
                    j = psv[j];
                    ej = e[j];
                }
                const u64 m = h < eb ? h : eb, pos = suf_off[j] - ej;
                for (; k < m; k += 8)
                    buf_or(buf, (u32)(k + rel), load_le(suf, sufN, pos + k, m - k < 8 ? (u32)(m - k) : 8u));
                k = m;
            }
            s_at[2 * t + 1] = (u16)(k + rel);
            s_end[2 * t + 1] = (u16)(kend + rel);
            s_src[2 * t + 1] = so + (k - ei);
            if (k < kend) wc1 = (u32)((kend + rel + 15) / 16 - (k + rel) / 16);
        }
        // every word of every piece gets a place of its own in the copy list
        u32 base = wc0 + wc1;
#pragma unroll
        for (u32 q = 1; q < 64; q <<= 1) {
            const u32 y = __shfl_up(base, q, 64);
            if (lane >= q) base += y;
        }
        if (lane == 63) s_wsum[wv] = base;
        __syncthreads();
        for (u32 w = 0; w < wv; w++) base += s_wsum[w];
        u32 nwords = 0;
        for (u32 w = 0; w < DC_NT / 64; w++) nwords += s_wsum[w];
        base -= wc0 + wc1;
        s_base[2 * t] = (u16)base;
        s_base[2 * t + 1] = (u16)(base + wc0);
        for (u32 q = 0; q < wc0 + wc1; q++) s_own[base + q] = (u16)(2 * t + (q < wc0 ? 0u : 1u));
        // the next chunk's strings, while this one's words are assembled
        u32 ei_n = 0, di_n = 0;
        u64 so_n = 0, oo_n = 0;
        const u32 rn = s_r0 + t;
        if (c1 < r1 && rn < n) {
            ei_n = e[rn];
            di_n = d[rn];
            so_n = suf_off[rn];
            oo_n = out_off[rn];
        }
        __syncthreads();
        const bool mids = s_mid != 0;  // (written before the barrier above, reset after the next)
        // The copies: DC_WU words a thread in flight, each loaded as five
        // 4-byte words and shifted into place (a piece's end words, shared with
        // the pieces beside it, are or-ed in)
        for (u32 g0 = t; g0 < nwords; g0 += DC_WU * DC_NT) {
            u32 x[DC_WU][5], w[DC_WU], b0[DC_WU], b1[DC_WU], r[DC_WU];
            u64 ps[DC_WU];
            bool safe[DC_WU];
#pragma unroll
            for (u32 u = 0; u < DC_WU; u++) {
                const u32 g = g0 + u * DC_NT;
                b0[u] = b1[u] = 0;
                safe[u] = true;
                w[u] = 0;
                r[u] = 0;
                ps[u] = 0;
                if (g < nwords) {
                    const u32 o2 = s_own[g], at = s_at[o2], end = s_end[o2];
                    w[u] = at / 16 + (g - s_base[o2]);
                    b0[u] = 16 * w[u] < at ? at - 16 * w[u] : 0u;             // bytes [b0, b1) of the word
                    b1[u] = end - 16 * w[u] < 16 ? end - 16 * w[u] : 16u;
                    ps[u] = s_src[o2] + (u64)((long long)(16 * w[u]) - (long long)at);  // suf offset of the word's byte 0
                    const u8 *a = suf + ps[u];
                    r[u] = (u32)((uintptr_t)a & 3);
                    safe[u] = (long long)ps[u] >= 4 && ps[u] + 20 <= sufN;
                    const u32 *q = (const u32 *)(a - r[u]);
                    if (safe[u]) {
#pragma unroll
                        for (int y = 0; y < 5; y++) x[u][y] = q[y];
                    }
                }
            }
#pragma unroll
            for (u32 u = 0; u < DC_WU; u++) {
                if (b0[u] >= b1[u]) continue;
                u64 v0 = 0, v1 = 0;
                if (safe[u]) {
#pragma unroll
                    for (int y = 0; y < 4; y++) x[u][y] = __builtin_amdgcn_alignbyte(x[u][y + 1], x[u][y], r[u]);
                    v0 = (u64)x[u][0] | ((u64)x[u][1] << 32);
                    v1 = (u64)x[u][2] | ((u64)x[u][3] << 32);
                } else {  // (near suf's ends)
                    for (u32 y = b0[u]; y < b1[u]; y++) {
                        const u64 z = suf[ps[u] + y];
                        if (y < 8) v0 |= z << (8 * y);
                        else v1 |= z << (8 * (y - 8));
                    }
                }
                if (b1[u] - b0[u] == 16) {
                    *(ulonglong2 *)&buf[2 * w[u]] = make_ulonglong2(v0, v1);
                } else {
                    v0 &= low_bytes(b1[u]) & ~low_bytes(b0[u]);
                    v1 &= (b1[u] > 8 ? low_bytes(b1[u] - 8) : 0ull) & (b0[u] > 8 ? ~low_bytes(b0[u] - 8) : ~0ull);
                    if (v0) atomicOr((unsigned long long *)&buf[2 * w[u]], (unsigned long long)v0);
                    if (v1) atomicOr((unsigned long long *)&buf[2 * w[u] + 1], (unsigned long long)v1);
                }
            }
        }
        __syncthreads();
        if (t == 0) s_mid = 0;
        if (mids) {  // (uniform)
            u32 mbase = s_ma[t] < s_mb[t] ? (s_mb[t] + 15u) / 16 - s_ma[t] / 16 : 0u;
            const u32 own = mbase;
#pragma unroll
            for (u32 q = 1; q < 64; q <<= 1) {
                const u32 y = __shfl_up(mbase, q, 64);
                if (lane >= q) mbase += y;
            }
            if (lane == 63) s_wsum[wv] = mbase;
            __syncthreads();
            u32 nm = 0;
            for (u32 w = 0; w < DC_NT / 64; w++) {
                if (w < wv) mbase += s_wsum[w];
                nm += s_wsum[w];
            }
            s_base[t] = (u16)(mbase - own);
            __syncthreads();
            // two neighbouring words to a thread: they mostly lie in one piece of the
            // chain, which is then found once
            u32 lo = DC_NT, h = 0;  // string, and where its current piece [ej, h) ends
            u64 pos = 0;            // byte k of the piece is at suf + pos + k
            for (u32 g0 = 2 * t; g0 < nm; g0 += g0 & 1 ? 2 * DC_NT - 1 : 1) {
                if (lo == DC_NT || (lo + 1 < DC_NT && s_base[lo + 1] <= g0)) {
                    u32 hi = DC_NT;  // the last string whose words start at or before g0
                    for (lo = 0; hi - lo > 1;) {
                        const u32 mid = (lo + hi) >> 1;
                        if (s_base[mid] <= g0) lo = mid;
                        else hi = mid;
                    }
                    h = 0;
                }
                const u32 at = s_ma[lo], w = at / 16 + (g0 - s_base[lo]);
                u32 x = 16 * w < at ? at : 16 * w;
                const u32 end = s_mb[lo] < 16 * w + 16 ? s_mb[lo] : 16 * w + 16;
                u64 k = s_mk[lo] + (x - at), v0 = 0, v1 = 0;
                while (x < end) {
                    if (k >= h) {  // (byte k < e of the string)
                        h = e[r0 + lo];
                        u32 j = psv[r0 + lo], ej = e[j];
                        while (ej > k) {
                            h = ej;
                            j = psv[j];
                            ej = e[j];
                        }
                        pos = suf_off[j] - ej;
                    }
                    const u32 m = end - x < h - k ? end - x : (u32)(h - k), sh = 8 * (x - 16 * w);
                    u64 a0, a1;
                    win16_finish(suf, win16_issue(suf, sufN, pos + k, m), a0, a1);
                    if (sh >= 64) {
                        v1 |= a0 << (sh - 64);
                    } else {
                        v0 |= a0 << sh;
                        v1 |= (a1 << sh) | (sh ? a0 >> (64 - sh) : 0ull);
                    }
                    x += m;
                    k += m;
                }
                if (v0) atomicOr((unsigned long long *)&buf[2 * w], (unsigned long long)v0);
                if (v1) atomicOr((unsigned long long *)&buf[2 * w + 1], (unsigned long long)v1);
            }
            __syncthreads();
        }
        const u32 span = (u32)(c1 - c0);
        // and out, in aligned 16-byte words; the buffer is cleared behind
        const u32 nw = (span + lead + 15) / 16;
        for (u32 w = t; w < nw; w += DC_NT) {
            const u64 v0 = buf[2 * w], v1 = buf[2 * w + 1];
            buf[2 * w] = 0;
            buf[2 * w + 1] = 0;
            u8 *dst = out + c0 - lead + 16 * w;
            const u32 b0 = w == 0 ? lead : 0u, b1 = span + lead - 16 * w < 16 ? span + lead - 16 * w : 16u;
            if (b1 - b0 == 16) *(ulonglong2 *)dst = make_ulonglong2(v0, v1);
            else
                for (u32 x = b0; x < b1; x++) dst[x] = (u8)((x < 8 ? v0 >> (8 * x) : v1 >> (8 * (x - 8))) & 0xFF);
        }
        c0 = c1;
        if (c0 >= r1) break;
        ei = ei_n;
        di = di_n;
        so = so_n;
        oo = oo_n;
        __syncthreads();  // the tables are rewritten by the next chunk
    }
}

// Workgroups of a decode of at most `cap` bytes: as many as the device holds
// at once (a range's first string costs a search and a chain walk), each at
// least one span.
static unsigned decode_grid(u64 cap)
{
    const u64 g = ceil_div(cap + 15, DC_SPAN), r = resident(k_decode, DC_NT);
    return (unsigned)(g < r ? g : r);
}

// status = 0 (runs well formed, decoded bytes fit), 1 (malformed runs) or 2
// (more decoded bytes than cap).
__global__ void k_decode_status(const u32 *bad, const u64 *out_off, u32 n, u64 cap, u32 *status)
{
    *status = *bad ? 1u : (out_off[n] > cap ? 2u : 0u);
}

// The check flag and the decoded total side by side, for one read-back.
__global__ void k_decode_total(const u64 *total, u32 *bad) { *(u64 *)(bad + 2) = *total; }

struct DecWs {
    u32 *psv, *tree, *cmin, *bad, *far, *fcnt;
    u64 *scratch;
};

static void dec_layout(u64 n, DecWs *w, WsArena *a, WsCounter *c)
{
    const u64 nt = 2 * (u64)psv_leaves(n);
    if (a) {
        w->psv = a->take<u32>(n + 1);
        w->tree = a->take<u32>(nt);
        w->cmin = a->take<u32>(nt / 2 * PCB);
        w->bad = a->take<u32>(4);
        w->far = a->take<u32>(n + 1);
        w->fcnt = a->take<u32>(ceil_div(n, PB) + 1);
        w->scratch = a->take<u64>(ss_scan_scratch_elems<u64>(n + 1));
    } else {
        c->take<u32>(n + 1);
        c->take<u32>(nt);
        c->take<u32>(nt / 2 * PCB);
        c->take<u32>(4);
        c->take<u32>(n + 1);
        c->take<u32>(ceil_div(n, PB) + 1);
        c->take<u64>(ss_scan_scratch_elems<u64>(n + 1));
    }
}

static int decode_impl(u32 k, const u64 *run_off, const u32 *e, const u32 *d, const u64 *suf_off, const u8 *suf,
                       u64 n, u64 *out_off, u8 *out, u64 out_cap, DecWs &w, hipStream_t st)
{
    k_fill_u32<<<1, 64, 0, st>>>(w.bad, 0u, 1);
    SS_CHECK_LAUNCH();
    const u64 grid = ceil_div((n > k ? n : k) + 1, 256);
    k_check_runs<<<(unsigned)grid, 256, 0, st>>>(run_off, k, e, d, (u32)n, w.bad, out_off);
    SS_CHECK_LAUNCH();
    SS_TRY(ss_scan_exclusive<u64>(out_off, out_off, n, w.scratch, st));
    k_decode_total<<<1, 1, 0, st>>>(out_off + n, w.bad);
    SS_CHECK_LAUNCH();
    u32 hw[4];
    SS_TRY(ss_read_u32(w.bad, hw, 4, st));
    const u32 bad = hw[0];
    u64 total;
    memcpy(&total, hw + 2, sizeof(u64));
    if (bad) {
        ss_set_error("malformed front-coded runs (code %u): runs must start with e = 0 and e_i <= d_i, "
                     "e_i <= d_{i-1}", bad);
        return SS_ERR_INVALID_ARG;
    }
    if (total > out_cap) {
        ss_set_error("decoded bytes %llu exceed capacity %llu", (unsigned long long)total,
                     (unsigned long long)out_cap);
        return SS_ERR_CAPACITY;
    }
    if (n == 0 || total == 0) return SS_OK;
    SS_TRY(psv_build(e, n, w.psv, w.tree, w.cmin, w.far, w.fcnt, st));
    k_decode<<<decode_grid(total), DC_NT, 0, st>>>(e, d, suf_off, suf, w.psv, (u32)n, out_off, nullptr, out);
    SS_CHECK_LAUNCH();
    return SS_OK;
}

extern "C" size_t ss_fc_decode_workspace(uint64_t n)
{
    WsCounter c;
    DecWs w;
    dec_layout(n, &w, nullptr, &c);
    return c.used;
}

extern "C" int ss_fc_decode(uint32_t k, const uint64_t *run_off, const uint32_t *fc_lcp, const uint32_t *fc_len,
                            const uint64_t *suf_off, const uint8_t *suf, uint64_t n, uint64_t *out_offsets,
                            uint8_t *out_bytes, uint64_t out_cap, void *ws, size_t ws_bytes, void *stream)
{
    ss_clear_error();
    if (n >= 0xFFFFFFFFull) { ss_set_error("n too large"); return SS_ERR_TOO_LARGE; }
    if (k == 0 || !run_off || !out_offsets || (n > 0 && (!fc_lcp || !fc_len || !suf_off))) {
        ss_set_error("fc_decode: bad arguments");
        return SS_ERR_INVALID_ARG;
    }
    WsArena a(ws, ws_bytes);
    DecWs w;
    dec_layout(n, &w, &a, nullptr);
    if (a.overflow || !ws) {
        ss_set_error("workspace too small: need %zu bytes", ss_fc_decode_workspace(n));
        return SS_ERR_WORKSPACE;
    }
    return decode_impl(k, run_off, fc_lcp, fc_len, suf_off, suf, n, out_offsets, out_bytes, out_cap, w,
                       (hipStream_t)stream);
}

// ------------------------------------------------ allocation-free decode
//
// ss_fc_decode_noalloc keeps its scratch in one static device array per GPU
// (the code object's copy on each device) instead of a caller workspace.  In
// host code the array's name is only a stand-in: its device address is
// looked up once per device with hipGetSymbolAddress (on the call's first
// use of that device, with the device current) and only that address is
// passed to kernels.  Calls on one device share the array: calls that
// overlap on one GPU (different streams, or threads) race.

#define FCD_NOALLOC_SCRATCH_BYTES (36u << 20)
static __device__ __align__(256) unsigned char scratch[FCD_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int FCD_MAX_DEVICES = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[FCD_MAX_DEVICES] = {};

int scratch_address(void **out)
{
    int dev = 0;
    SS_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= FCD_MAX_DEVICES) {
        ss_set_error("device index %d beyond %d", dev, FCD_MAX_DEVICES);
        return SS_ERR_INVALID_ARG;
    }
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            ss_set_error("hipGetSymbolAddress(scratch) failed on device %d: %s", dev, hipGetErrorString(e));
            return SS_ERR_HIP;
        }
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return SS_OK;
}
}  // namespace

extern "C" int ss_fc_decode_noalloc(uint32_t k, const uint64_t *run_off, const uint32_t *fc_lcp,
                                    const uint32_t *fc_len, const uint64_t *suf_off, const uint8_t *suf,
                                    uint64_t n, uint64_t *out_offsets, uint8_t *out_bytes, uint64_t out_cap,
                                    uint32_t *status, void *stream)
{
    ss_clear_error();
    if (n > SS_FC_DECODE_NOALLOC_MAX) {
        ss_set_error("fc_decode_noalloc: n = %llu exceeds the limit of %u entries", (unsigned long long)n,
                     (unsigned)SS_FC_DECODE_NOALLOC_MAX);
        return SS_ERR_TOO_LARGE;
    }
    if (k == 0 || !run_off || !out_offsets || !status || (n > 0 && (!fc_lcp || !fc_len || !suf_off))) {
        ss_set_error("fc_decode_noalloc: bad arguments");
        return SS_ERR_INVALID_ARG;
    }
    if (ss_fc_decode_workspace(n) > FCD_NOALLOC_SCRATCH_BYTES) {  // (cannot happen below the limit)
        ss_set_error("fc_decode_noalloc: scratch too small for n = %llu", (unsigned long long)n);
        return SS_ERR_TOO_LARGE;
    }
    void *base = nullptr;
    SS_TRY(scratch_address(&base));
    hipStream_t st = (hipStream_t)stream;
    WsArena a(base, FCD_NOALLOC_SCRATCH_BYTES);
    DecWs w;
    dec_layout(n, &w, &a, nullptr);
    const u32 *e = fc_lcp, *d = fc_len;
    // w.bad starts at zero on every call (the array keeps the last call's contents)
    k_fill_u32<<<1, 64, 0, st>>>(w.bad, 0u, 1);
    SS_CHECK_LAUNCH();
    const u64 grid = ceil_div((n > k ? n : k) + 1, 256);
    k_check_runs<<<(unsigned)grid, 256, 0, st>>>(run_off, k, e, d, (u32)n, w.bad, out_offsets);
    SS_CHECK_LAUNCH();
    SS_TRY(ss_scan_exclusive<u64>(out_offsets, out_offsets, n, w.scratch, st));
    k_decode_status<<<1, 1, 0, st>>>(w.bad, out_offsets, (u32)n, out_cap, status);
    SS_CHECK_LAUNCH();
    if (n == 0 || out_cap == 0) return SS_OK;
    // the psv chains only read e (any values are safe); bytes are decoded
    // only when the status is 0
    SS_TRY(psv_build(e, n, w.psv, w.tree, w.cmin, w.far, w.fcnt, st));
    k_decode<<<decode_grid(out_cap), DC_NT, 0, st>>>(e, d, suf_off, suf, w.psv, (u32)n, out_offsets, status,
                                                   out_bytes);
    SS_CHECK_LAUNCH();
    return SS_OK;
}

// ----------------------------------------------------------------- merge

// Read access to front-coded strings without decoding them: bytes [k, k+take)
// of string g are gathered piece by piece along its psv chain.
struct FcView {
    const u32 *e, *d, *psv;
    const u64 *suf_off;
    const u8 *suf;
    u64 sufN;
};

// The literal piece of front-coded string g that holds byte k (< d_g): the
// offset in suf of byte k, and how many of the string's bytes from k on lie
// in that literal (the chain element whose e is the first <= k, walking the
// psv chain from g; its literal covers bytes [e_j, e of the element after it
// toward g), or [e_g, d_g) for g itself).
__device__ __forceinline__ void fc_piece(const FcView &V, u32 g, u64 k, u64 *pos, u64 *avail)
{
    u32 j = g;
    u64 h = V.d[g];
    u32 ej = V.e[j];
    while (ej > k) {
        h = ej;
        j = V.psv[j];
        ej = V.e[j];
    }
    *pos = V.suf_off[j] + (k - ej);
    *avail = h - k;
}

// The merge's results: per output, the source (run, position in run), the
// string id, the LCP with the previous output and the string length (src and
// len optional).  sb/sid: the non-empty runs' front-coded starts, ascending,
// and their run numbers.
struct MergeOut {
    const u64 *sb;
    const u32 *sid;
    u32 kne;
    const u32 *fc_id, *fc_len;
    u64 *src;
    u32 *id, *lcp, *len;
};

// (the element's front-coded position g; its LCP is written apart)
__device__ __forceinline__ void merge_emit(const MergeOut &O, u64 x, u32 g)
{
    if (O.src) {
        u32 lo = 0, hi = O.kne;  // largest j with sb[j] <= g
        while (hi - lo > 1) {
            u32 mid = (lo + hi) >> 1;
            if (O.sb[mid] <= g) lo = mid;
            else hi = mid;
        }
        O.src[x] = ((u64)O.sid[lo] << 32) | (u64)(g - O.sb[lo]);
    }
    O.id[x] = O.fc_id[g];
    if (O.len) O.len[x] = O.fc_len[g];
}

// Minimum LCP-with-predecessor over each run except its first element, i.e.
// the LCP of the run's first and last strings: gridDim.y workgroups per run
// (blockIdx.y = part), one atomic each.  The caller gives a run of the average
// size a workgroup per 4096 entries, at most 64 of them: with 245 the atomics
// on one word cost more than they save.  4 runs of 500,000 entries: 18 us with
// one load in flight, 6.4 us with eight (13.8 us with 245 workgroups per run).
// Runs of more than `limit` entries, far above the average, are listed and take
// a launch of their own with 64 workgroups each: one run of 8M among 1,023 of 100
// took 783 us without it.
#define RM_PARTS 64
__global__ __launch_bounds__(256) void k_run_min(const u32 *list, u64 limit, const u64 *run_begin, const u64 *P,
                                                 const u32 *e, u32 *runmin)
{
    __shared__ u32 wmin[4];
    const u32 r = list ? list[blockIdx.x] : blockIdx.x;
    const u64 b = run_begin[r], n = P[r + 1] - P[r];
    if (!list && n > limit) return;  // (uniform)
    const u64 i0 = 1 + (n * blockIdx.y) / gridDim.y, i1 = 1 + (n * (blockIdx.y + 1)) / gridDim.y;
    u32 mn = 0xFFFFFFFFu;
    const u64 end = i1 < n ? i1 : n;
    for (u64 i = i0 + threadIdx.x; i < end; i += 8 * 256) {
        u32 v[8];  // (eight loads in flight; past the end the first again)
#pragma unroll
        for (u32 q = 0; q < 8; q++) v[q] = e[b + (i + q * 256 < end ? i + q * 256 : i)];
#pragma unroll
        for (u32 q = 0; q < 8; q++) mn = v[q] < mn ? v[q] : mn;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const u32 y = __shfl_xor(mn, o, 64);
        mn = y < mn ? y : mn;
    }
    if ((threadIdx.x & 63) == 0) wmin[threadIdx.x >> 6] = mn;
    __syncthreads();
    if (threadIdx.x == 0) {
        u32 m = wmin[0];
        for (int w = 1; w < 4; w++) m = wmin[w] < m ? wmin[w] : m;
        if (m != 0xFFFFFFFFu) atomicMin(&runmin[r], m);
    }
}

// Common prefix length of each group: every string of run r shares
// min(lcp(head of the group's first run, head of r), runmin[r]) bytes with the
// group's first head.  A wavefront per run: heads are whole in their literals
// (e = 0), so 512 bytes of both are compared at once (a thread per run: 31 us
// where the heads share 250 bytes, now 8).
__global__ __launch_bounds__(256) void k_group_depth(const u64 *run_begin, const u64 *P, const u32 *run_group,
                                                     const u32 *rep, u32 k, const u32 *runmin, FcView V, u32 *Cg)
{
    const u32 r = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= k) return;  // (uniform over the wavefront)
    if (P[r + 1] == P[r]) return;
    const u32 g = run_group[r];
    const u32 r0 = rep[g];
    u32 v = runmin[r];
    if (r0 != r) {
        const u32 a = (u32)run_begin[r0], b = (u32)run_begin[r];
        u64 l;
        wave_str_cmp(V.suf, V.sufN, V.suf_off[a], V.d[a], V.suf_off[b], V.d[b], &l);
        v = min(v, (u32)l);
    }
    if ((threadIdx.x & 63) == 0) atomicMin(&Cg[g], v);
}

// ---- the elements' keys by one scan over the runs
//
// Output position x of run r is front-coded entry g = run_begin[r] + x - P[r]
// with LCP e_g to its predecessor (0 at the run start).  Its key is bytes
// [C, C+7) of its string and min(d_g - C, 8), C = the group's common prefix.
// It follows a scan with the operator (p, v): the 7-byte window at C keeps its
// first p bytes from the predecessor's window (p = clamp(e_g - C, 0, 7), none
// at a run start) and takes the rest, v, from the entry's literal.
struct MOp {
    u32 p;
    u64 v;
};

__device__ __forceinline__ MOp mop_id() { return MOp{7u, 0ull}; }

// a, then b
__device__ __forceinline__ MOp mop_cat(MOp a, MOp b)
{
    const u64 keep = b.p ? (~0ull << (64 - 8 * b.p)) : 0ull;
    MOp r;
    r.p = a.p < b.p ? a.p : b.p;
    r.v = (a.v & keep) | (b.v & ~keep);
    return r;
}

__device__ __forceinline__ MOp mop_shfl_up(MOp a, u32 d)
{
    MOp r;
    r.p = __shfl_up(a.p, d, 64);
    r.v = __shfl_up(a.v, d, 64);
    return r;
}

struct MScan {
    const u64 *run_begin, *P;
    const u32 *run_group, *Cg;
    const u32 *bfirst;  // run of every scan block's first element
    u32 k, n_out;
    FcView V;
    u32 *ties;  // set to 1 if two adjacent strings of a run agree on [0, C+7)
};

// The run holding the positions being walked: its output range [pr, pr1),
// front-coded start and group depth, kept in registers.
struct RunCur {
    u32 r;
    u64 pr, pr1, rb;
    u32 C;
};

__device__ __forceinline__ RunCur run_cur(const MScan &S, u32 r)
{
    return RunCur{r, S.P[r], S.P[r + 1], S.run_begin[r], S.Cg[S.run_group[r]]};
}

// advance to the run containing x (x >= the current run's start)
__device__ __forceinline__ void run_seek(const MScan &S, RunCur &c, u64 x)
{
    while (c.pr1 <= x) {
        c.r++;
        c.pr = c.pr1;
        c.pr1 = S.P[c.r + 1];
        c.rb = S.run_begin[c.r];
        c.C = S.Cg[S.run_group[c.r]];
    }
}

__device__ __forceinline__ u32 run_of(const u64 *P, u32 k, u64 x)
{
    u32 lo = 0, hi = k;  // largest j with P[j] <= x
    while (hi - lo > 1) {
        const u32 mid = (lo + hi) >> 1;
        if (P[mid] <= x) lo = mid;
        else hi = mid;
    }
    return lo;
}

// 7 elements per thread: the apply kernel's LDS operators take 28 KB
#define MS_PER 7
#define MS_ITEMS (256 * MS_PER)  // elements per workgroup

// This thread's elements x = x0 + 256 q + threadIdx.x (q < MS_PER; lanes on
// consecutive elements): entry g, run depth C and the in-range / run-start
// bits, from the block's first run and the cursor, which moves only at run
// bounds -- before any load of the elements' data is issued.
struct MElems {
    u32 g[MS_PER], C[MS_PER];
    u32 in, start;  // bit q
};

__device__ __forceinline__ void mscan_locate(const MScan &S, u64 x0, MElems &E)
{
    RunCur c = run_cur(S, S.bfirst[blockIdx.x]);
    E.in = E.start = 0;
#pragma unroll
    for (u32 q = 0; q < MS_PER; q++) {
        const u64 x = x0 + q * 256 + threadIdx.x;
        E.g[q] = 0;  // (a valid entry to load from: the workgroup has elements)
        E.C[q] = 0;
        if (x < S.n_out) {
            run_seek(S, c, x);
            E.g[q] = (u32)(c.rb + (x - c.pr));
            E.C[q] = c.C;
            E.in |= 1u << q;
            if (x == c.pr) E.start |= 1u << q;
        }
    }
}

// The operators of this thread's elements (identity out of range) and their
// LCPs e[q]: the entries' LCPs, lengths and literal offsets are loaded for all
// elements first, then every element's window bytes, then combined.  An
// operator's low byte carries the element's length count min(d - C, 8), so
// that the inclusive operator at x is the element's cached key.
__device__ __forceinline__ void mscan_ops(const MScan &S, const MElems &E, MOp *o, u32 *e)
{
    u32 d[MS_PER];
    u64 so[MS_PER];
#pragma unroll
    for (u32 q = 0; q < MS_PER; q++) {
        e[q] = S.V.e[E.g[q]];
        d[q] = S.V.d[E.g[q]];
        so[q] = S.V.suf_off[E.g[q]];
    }
    u32 p[MS_PER];
    Raw8 lit[MS_PER];
#pragma unroll
    for (u32 q = 0; q < MS_PER; q++) {
        if ((E.start >> q) & 1) e[q] = 0;
        const u32 C = E.C[q];
        p[q] = e[q] > C ? (e[q] - C < 7 ? e[q] - C : 7u) : 0u;
        const u32 from = C + p[q];  // first window byte the entry's literal supplies (>= e)
        const u32 to = d[q] < C + 7 ? d[q] : C + 7;
        const bool want = ((E.in >> q) & 1) && p[q] < 7 && to > from;
        lit[q] = raw8_issue(S.V.suf, S.V.sufN, want ? so[q] + (from - e[q]) : 0ull, want ? to - from : 0u);
    }
#pragma unroll
    for (u32 q = 0; q < MS_PER; q++) {
        const u32 C = E.C[q];
        MOp r;
        r.p = p[q];
        r.v = (d[q] > C ? (d[q] - C < 8 ? d[q] - C : 8u) : 0u) |
              (__builtin_bswap64(raw8_le(S.V.suf, lit[q])) >> (8 * p[q]));
        o[q] = ((E.in >> q) & 1) ? r : mop_id();
    }
}

// Ordered reduction / exclusive scan of one operator per thread over a
// 256-thread workgroup.
__device__ __forceinline__ MOp block_mop_reduce(MOp a)
{
    __shared__ MOp wsum[4];
    const u32 lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (u32 d = 1; d < 64; d <<= 1) {
        const MOp y = mop_shfl_up(a, d);
        if (lane >= d) a = mop_cat(y, a);
    }
    if (lane == 63) wsum[wv] = a;
    __syncthreads();
    MOp t = wsum[0];
    for (u32 w = 1; w < 4; w++) t = mop_cat(t, wsum[w]);
    __syncthreads();
    return t;
}

__device__ __forceinline__ MOp block_mop_exclusive(MOp a, MOp carry)
{
    __shared__ MOp wsum[4];
    const u32 lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    MOp inc = a;
#pragma unroll
    for (u32 d = 1; d < 64; d <<= 1) {
        const MOp y = mop_shfl_up(inc, d);
        if (lane >= d) inc = mop_cat(y, inc);
    }
    if (lane == 63) wsum[wv] = inc;
    MOp ex = mop_shfl_up(inc, 1);
    if (lane == 0) ex = mop_id();
    __syncthreads();
    MOp pre = carry;
    for (u32 w = 0; w < wv; w++) pre = mop_cat(pre, wsum[w]);
    __syncthreads();
    return mop_cat(pre, ex);
}

// Initial values of a merge's counters and minima, and the run of every scan
// block's first element (the run r with P[r] <= x < P[r+1], x = j MS_ITEMS).
__global__ void k_merge_init(const u64 *P, u32 k, u32 nb, u32 *bfirst, u32 *runmin, u32 *Cg, u32 groups, u32 *ties,
                             u32 *ctr)
{
    const u32 j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < k) runmin[j] = 0xFFFFFFFFu;
    if (j < groups) Cg[j] = 0xFFFFFFFFu;
    if (j < C_NCTR) ctr[j] = 0;
    if (j == 0) *ties = 0;
    if (j < nb) {
        u32 lo = 0, hi = k;
        while (hi - lo > 1) {
            const u32 mid = (lo + hi) >> 1;
            if (P[mid] <= (u64)j * MS_ITEMS) lo = mid;
            else hi = mid;
        }
        bfirst[j] = lo;
    }
}

// Phase 1: the operator of every MS_ITEMS-element block.  Its p needs only each
// element's e.  Of its window, byte k (k < 7) is
// the one written by the block's last element with p <= k (a later element
// with a larger p keeps it), and the count byte is the last element's, so at
// most eight literal bytes are read per block instead of every element's.
__global__ __launch_bounds__(256) void k_mscan_reduce(MScan S, MOp *blk)
{
    // per wavefront, per window byte k < 7 and the count (7): last supplier + 1, block-relative (0: none)
    __shared__ u32 s_wl[4][8];
    __shared__ u32 s_p[MS_ITEMS];
    const u64 x0 = (u64)blockIdx.x * MS_ITEMS;
    MElems E;
    mscan_locate(S, x0, E);
    u32 e[MS_PER];
#pragma unroll
    for (u32 q = 0; q < MS_PER; q++) e[q] = S.V.e[E.g[q]];
#pragma unroll
    for (u32 q = 0; q < MS_PER; q++) {
        const u32 i = q * 256 + threadIdx.x;
        const bool st = (E.start >> q) & 1;
        const u32 ee = st ? 0u : e[q], C = E.C[q];
        const u32 p = ee > C ? (ee - C < 7 ? ee - C : 7u) : 0u;
        s_p[i] = ((E.in >> q) & 1) ? p : 0xFFu;  // (0xFF: out of range)
    }
    __syncthreads();
    // this thread's MS_PER consecutive elements, in order
    MOp t = mop_id();
    u32 lastk[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (u32 q = 0; q < MS_PER; q++) {
        const u32 i = threadIdx.x * MS_PER + q;
        const u32 p = s_p[i];
        if (p == 0xFFu) break;  // (out of range from here on)
        t.p = p < t.p ? p : t.p;
#pragma unroll
        for (u32 k = 0; k < 7; k++)
            if (p <= k) lastk[k] = i + 1;
        lastk[7] = i + 1;
    }
    // the last supplier of each byte is the highest lane that has one
    // (a thread's elements follow those of the lanes below it)
#pragma unroll
    for (u32 k = 0; k < 8; k++) {
        const u64 m = __ballot(lastk[k] != 0);
        const u32 v = m ? (u32)__shfl((int)lastk[k], 63 - __clzll(m), 64) : 0u;
        if ((threadIdx.x & 63) == 0) s_wl[threadIdx.x >> 6][k] = v;
    }
    t = block_mop_reduce(t);  // (p; its window is filled below, its barriers complete s_wl)
    u32 last[8];
#pragma unroll
    for (u32 k = 0; k < 8; k++) last[k] = max(max(s_wl[0][k], s_wl[1][k]), max(s_wl[2][k], s_wl[3][k]));
    __shared__ u64 s_v[8];
    if (threadIdx.x < 8) s_v[threadIdx.x] = 0;
    __syncthreads();
    // byte k comes from element last[k] - 1; the thread holding that
    // element's entry loads it
#pragma unroll
    for (u32 q = 0; q < MS_PER; q++) {
        const u32 j = q * 256 + threadIdx.x + 1;
        u32 ks = 0;
#pragma unroll
        for (u32 k = 0; k < 8; k++)
            if (last[k] == j) ks |= 1u << k;
        if (ks) {
            const u32 g = E.g[q], C = E.C[q];
            const u32 ee = ((E.start >> q) & 1) ? 0u : e[q];
            const u32 d = S.V.d[g];
            const u64 so = S.V.suf_off[g];
            if (ks & 0x80u) s_v[7] = d > C ? (d - C < 8 ? d - C : 8u) : 0u;  // the count byte
#pragma unroll
            for (u32 k = 0; k < 7; k++)  // byte at position C + k of the string (its literal starts at e <= C + k)
                if (((ks >> k) & 1) && C + k < d) s_v[k] = (u64)S.V.suf[so + (C + k - ee)] << (8 * (7 - k));
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        u64 v = 0;
#pragma unroll
        for (u32 k = 0; k < 8; k++) v |= s_v[k];
        t.v = v;
        blk[blockIdx.x] = t;
    }
}

// Phase 2: exclusive scan of the block operators (one workgroup of 1024:
// each thread composes a chunk, the chunk composites are scanned by
// wavefront shuffles and one pass over the 16 wavefront totals).
__global__ __launch_bounds__(1024) void k_mscan_top(MOp *blk, u32 nb)
{
    __shared__ MOp wtot[16];
    const u32 per = (nb + 1023) / 1024;
    const u32 c0 = threadIdx.x * per, c1 = (c0 + per < nb) ? c0 + per : nb;
    // (operators loaded eight at a time, ahead of the chain that combines them)
    MOp t = mop_id();
    for (u32 i = c0; i < c1; i += 8) {
        MOp v[8];
#pragma unroll
        for (u32 j = 0; j < 8; j++) v[j] = (i + j < c1) ? blk[i + j] : mop_id();
#pragma unroll
        for (u32 j = 0; j < 8; j++) t = mop_cat(t, v[j]);
    }
    const u32 lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    MOp inc = t;
#pragma unroll
    for (u32 d = 1; d < 64; d <<= 1) {
        const MOp y = mop_shfl_up(inc, d);
        if (lane >= d) inc = mop_cat(y, inc);
    }
    if (lane == 63) wtot[wv] = inc;
    MOp ex = mop_shfl_up(inc, 1);
    if (lane == 0) ex = mop_id();
    __syncthreads();
    MOp pre = mop_id();
    for (u32 w = 0; w < wv; w++) pre = mop_cat(pre, wtot[w]);
    pre = mop_cat(pre, ex);
    for (u32 i = c0; i < c1; i += 8) {
        MOp v[8];
#pragma unroll
        for (u32 j = 0; j < 8; j++) v[j] = (i + j < c1) ? blk[i + j] : mop_id();
#pragma unroll
        for (u32 j = 0; j < 8; j++) {
            if (i + j < c1) blk[i + j] = pre;
            pre = mop_cat(pre, v[j]);
        }
    }
}

// Phase 3: every element's inclusive operator, its key (written with
// consecutive lanes on consecutive elements).
// Keys that fall within a run (runs are sorted by precondition) raise *bad: a
// merge by key would then lose elements, and the groups are sorted as a whole
// instead.
__global__ __launch_bounds__(256, 4) void k_mscan_apply(MScan S, const MOp *blk, u64 *K, u32 *bad)
{
    __shared__ MOp ops[MS_ITEMS];
    const u64 x0 = (u64)blockIdx.x * MS_ITEMS;
    MElems E;
    mscan_locate(S, x0, E);
    MOp o[MS_PER];
    u32 e[MS_PER];
    mscan_ops(S, E, o, e);
#pragma unroll
    for (u32 q = 0; q < MS_PER; q++) ops[q * 256 + threadIdx.x] = o[q];
    __syncthreads();
    MOp t = mop_id();
#pragma unroll
    for (u32 q = 0; q < MS_PER; q++) t = mop_cat(t, ops[threadIdx.x * MS_PER + q]);
    MOp st = block_mop_exclusive(t, blk[blockIdx.x]);
    // adjacent strings of a run that agree on their whole cached key
    bool tie = false;
#pragma unroll
    for (u32 q = 0; q < MS_PER; q++) tie |= ((E.in >> q) & 1) && e[q] >= E.C[q] + 7;
    if (__ballot(tie) && (threadIdx.x & 63) == 0) *S.ties = 1u;
#pragma unroll
    for (u32 q = 0; q < MS_PER; q++) {
        const u32 i = threadIdx.x * MS_PER + q;
        st = mop_cat(st, ops[i]);
        ops[i].v = st.v;
    }
    __syncthreads();
    bool fall = false;
#pragma unroll
    for (u32 q = 0; q < MS_PER; q++) {
        const u32 i = q * 256 + threadIdx.x;
        if (!((E.in >> q) & 1)) break;
        const u64 v = ops[i].v;
        K[x0 + i] = v;
        if (!((E.start >> q) & 1)) fall |= (i ? ops[i - 1].v : blk[blockIdx.x].v) > v;
    }
    if (__ballot(fall) && (threadIdx.x & 63) == 0) *bad = 1u;
}

// ---- merging by key
//
// The non-empty runs, in order, are numbered j = 0, 1, ... over all groups;
// group g has runs [gs[g], gs[g+1]).  Level 0 of a key list is the runs
// themselves (run j at K[ps[j]], ps[j+1] - ps[j] keys); level v + 1 takes every
// S-th key of every run of level v, beginning at positions spread over [0, S)
// by the run's number (samples at the same positions of like runs would come in
// lumps), so that a sample's rank among the samples times S is its rank without
// bias.  A group of
// more than MW_CAP keys in level v is cut into tiles of MW_TILE at keys of its
// merged level v + 1; a smaller one is one tile.  Tile t of group g takes from
// run j the keys in [threshold t, threshold t + 1): their positions are entries
// t and t + 1 of the run's row in the group's bounds matrix.
#define MW_NT 256
#define MW_IPT 9  // (odd shares: the threads' blocked accesses then meet no bank conflicts)
#define MW_CAP (MW_NT * MW_IPT)  // keys a tile can hold
#define MW_TILE 1280             // keys of a tile on average
#define MW_RUNS 2048             // runs of a group merged this way
#define MW_FEW 512               // (a kernel of its own for so many: its windows' bounds take less LDS)
#define MW_RANK 16               // groups of up to so many runs rank their samples directly
#define MW_LEVELS 9

// Sampling step of a group of kg runs.  A threshold cuts every run up to S/2
// from where its samples say, so the sizes of tiles vary by about 0.4 S sqrt(kg)
// about MW_TILE: these steps keep that at 205 or less, a fifth of what a tile has
// to spare (half the steps: 256 runs of 31,250 keys 581 us instead of 556).
__device__ __host__ __forceinline__ u32 mw_step(u32 kg)
{
    return kg <= 64 ? 64u : (kg <= 256 ? 32u : (kg <= 1024 ? 16u : 8u));
}
// Where run r of a group of kg starts sampling, how many samples a run of len
// keys gives, and the sample that threshold t of nt tiles over tot keys takes
// (of ns).
__device__ __host__ __forceinline__ u32 mw_phase(u32 r, u32 kg) { return (2 * r + 1) * mw_step(kg) / (2 * kg); }
__device__ __host__ __forceinline__ u64 mw_samples(u64 len, u32 r, u32 kg)
{
    const u32 S = mw_step(kg);
    return (len + S - 1 - mw_phase(r, kg)) / S;
}
__device__ __forceinline__ u32 mw_cut(u32 t, u32 nt, u32 tot, u32 ns, u32 S)
{
    const u64 x = (u64)t * tot / ((u64)nt * S);
    return x < ns ? (u32)x : ns - 1;
}

struct MwLevel {
    const u64 *K;     // this level's keys
    const u32 *ps;    // start of every run in K (runs + 1)
    const u32 *gs;    // first run of every group (groups + 1)
    const u32 *ts;    // first tile of every group (groups + 1)
    const u32 *bo;    // first bounds entry of every group (groups + 1)
    const u64 *spl;   // merged keys of the next level
    const u32 *sps;   // its run starts: run j's samples begin at sps[j]
    u32 groups;
    u32 *bounds;
    const u32 *bad;   // raised: some run is not sorted (nothing is merged)
};

// largest g in [0, n) with a[g] <= x
__device__ __forceinline__ u32 mw_find(const u32 *a, u32 n, u32 x)
{
    u32 lo = 0, hi = n;
    while (hi - lo > 1) {
        const u32 mid = (lo + hi) >> 1;
        if (a[mid] <= x) lo = mid;
        else hi = mid;
    }
    return lo;
}

// Threshold t (0 < t < nt) of a group.
__device__ __forceinline__ u64 mw_threshold(const MwLevel &M, u32 j0, u32 kg, u32 t, u32 nt)
{
    const u32 s0 = M.sps[j0], ns = M.sps[j0 + kg] - s0, tot = M.ps[j0 + kg] - M.ps[j0];
    return M.spl[s0 + mw_cut(t, nt, tot, ns, mw_step(kg))];
}

// The sampled keys of level v (run j's at out[st[j]]).
__global__ void k_mw_sample(const u64 *K, const u32 *ps, const u32 *gs, u32 groups, u32 kc, const u32 *st, u32 v,
                            u64 *out)
{
    const u32 x = st[0] + blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= st[kc]) return;
    const u32 j = mw_find(st, kc, x);
    const u32 g = mw_find(gs, groups, j);
    const u32 kg = gs[g + 1] - gs[g], S = mw_step(kg), ph = mw_phase(j - gs[g], kg);
    u64 i = x - st[j];
    for (u32 y = 0; y < v; y++) i = i * S + ph;
    out[x] = K[ps[j] + i];
}

// Merged positions of the first-level samples of the groups of up to MW_RANK
// runs: a sample's rank is its own index plus how many samples of each other
// run lie below it (or equal it, in an earlier run).  That is one launch where
// further levels take two more each; what it costs, samples x runs x
// log(samples of a run) probes, is 1/4 of a probe per key and search step at 16
// runs.  4M keys in 16 x 16 runs: 63 us with one search after the other, 33
// us with four side by side.
__global__ __launch_bounds__(256) void k_mw_rank(const u64 *K, const u32 *ps0, const u32 *ps, const u32 *gs,
                                                 u32 groups, u32 kc, u64 *KM, const u32 *bad)
{
    const u32 x = ps[0] + blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= ps[kc]) return;
    if (*bad) return;
    const u32 j = mw_find(ps, kc, x);
    const u32 g = mw_find(gs, groups, j);
    const u32 j0 = gs[g], j1 = gs[g + 1];
    const u32 kg = j1 - j0, S = mw_step(kg);
    if (kg > MW_RANK) return;
    const u64 key = K[ps0[j] + (u64)(x - ps[j]) * S + mw_phase(j - j0, kg)];
    u32 r = ps[j0] + (x - ps[j]);
    for (u32 o = j0; o < j1; o += 4) {  // four searches side by side: each is a chain of loads
        const u64 *k[4];
        u32 lo[4], n[4], most = 0;
#pragma unroll
        for (u32 q = 0; q < 4; q++) {
            // (a run shorter than its first sample's place has none: nothing of it is read)
            const bool on = o + q < j1 && o + q != j && ps[o + q + 1] > ps[o + q];
            const u32 w = on ? o + q : j;
            k[q] = K + ps0[w] + mw_phase(w - j0, kg);
            lo[q] = 0;
            n[q] = on ? ps[w + 1] - ps[w] : 0u;  // samples in doubt: [lo, lo + n)
            most = n[q] > most ? n[q] : most;
        }
        for (; most; most >>= 1) {
            u64 y[4];
#pragma unroll
            for (u32 q = 0; q < 4; q++) y[q] = k[q][n[q] ? (u64)(lo[q] + (n[q] >> 1)) * S : 0];
#pragma unroll
            for (u32 q = 0; q < 4; q++) {
                const u32 h = n[q] >> 1;
                const bool below = n[q] && (o + q < j ? y[q] <= key : y[q] < key);
                lo[q] += below ? h + 1 : 0u;
                n[q] = below ? n[q] - h - 1 : h;
            }
        }
#pragma unroll
        for (u32 q = 0; q < 4; q++) r += lo[q];
    }
    KM[r] = key;
}

// The bounds matrices of a level: row j, entry t of a group = how many keys of
// its run j lie below threshold t (entry 0: none; the last: all).  Consecutive
// lanes search one run for consecutive thresholds, so they read the same lines
// (the launches of a merge of 256 runs of 31,250 keys: 170 us with lanes on
// different runs, 45 us so).
__global__ __launch_bounds__(256) void k_mw_bounds(MwLevel M, u32 total)
{
    const u32 x = blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= total) return;
    if (*M.bad) return;
    const u32 g = mw_find(M.bo, M.groups, x);
    const u32 j0 = M.gs[g], kg = M.gs[g + 1] - j0, nt = M.ts[g + 1] - M.ts[g];
    const u32 j = j0 + (x - M.bo[g]) / (nt + 1), row = (x - M.bo[g]) % (nt + 1);
    const u32 p0 = M.ps[j], len = M.ps[j + 1] - p0;
    u32 r = row == 0 ? 0u : len;
    if (row > 0 && row < nt) {
        const u64 t = mw_threshold(M, j0, kg, row, nt);
        u32 lo = 0, hi = len;  // first position with a key >= t
        while (lo < hi) {
            const u32 mid = (lo + hi) >> 1;
            if (M.K[p0 + mid] < t) lo = mid + 1;
            else hi = mid;
        }
        r = lo;
    }
    M.bounds[x] = r;
}

#define TIE_SMALL 8  // tied segments of up to this many are sorted at once
#define TIE_REC 1u  // a tied segment whose members' entries lie beside the order, and whose results are written

struct MwOut {
    u64 *keys;           // sample levels: the merged keys
    const u32 *Cg;       // the rest: level 0
    const u32 *rrun, *rbeg;  // every non-empty run's number and front-coded start
    const u32 *fc_lcp, *fc_len;
    const u64 *suf_off;
    MergeOut O;
    u32 *order;          // front-coded positions of tied elements, by output position
    Seg *ties;           // runs of outputs with tied keys (C_RNEXT of them)
    Seg *over;           // segments handed to the sort as a whole (C_RTILES of them)
    SortWs s;
    u32 tile, block_max; // of that sort
};

// One segment to the sort of its size, and to the list of what is to be emitted
// (from: the tile it is, or MW_GROUP: a whole group).
#define MW_GROUP 0xFFFFFFFFu
#define MW_EQUAL 0x80000000u  // a tile of one key, in its final order but for ties
__device__ __forceinline__ void mw_route(const MwOut &W, Seg o, u32 from)
{
    const u32 m = o.end - o.begin;
    u32 *ctr = W.s.ctr;
    W.over[atomicAdd(&ctr[C_RTILES], 1u)] = Seg{o.begin, o.end, o.depth, from};
    if (m > W.block_max) {
        W.s.largeA[atomicAdd(&ctr[C_LARGE], 1u)] = Seg{o.begin, o.end, o.depth, o.aux | SEG_NOROOT};
        atomicAdd(&ctr[C_LTILES], (m + W.tile - 1) / W.tile);
        atomicAdd(&ctr[C_LELEM], m);
    } else if (m <= WS_MAX) {
        if (m > 1) W.s.tiny[atomicAdd(&ctr[C_TINY], 1u)] = o;
    } else {
        if (m <= BS_SMALL) W.s.small[atomicAdd(&ctr[C_SMALL], 1u)] = o;
        else W.s.mid[atomicAdd(&ctr[C_MID], 1u)] = o;
        atomicAdd(&ctr[C_SMALLN], m);
    }
    atomicAdd(&ctr[C_NELEM], m);
}

// Merge of one tile: the windows of its runs one after the other in LDS, then
// ceil(log2 runs) levels, each merging neighbouring lists pairwise; a thread
// finds where its outputs start (pair, then merge path) and merges them
// serially, stepping over pair ends.  Keys alone are compared and earlier runs
// win ties, so equal keys stay in (run, position) order.
//
// OUT (level 0): writes the merge's results; keys that differ give the LCPs.
// Runs of outputs with equal keys whose strings go on become segments at depth
// C + 7 if they come from more than one run (within one run their order and
// LCPs stand).  A tile whose windows exceed MW_CAP (many copies of one key, or
// a group with too few samples) becomes one segment for the segmented sort
// (k_mw_over copies its windows), or, if all its keys are one, is in order as it
// is; in a sample level its keys all become its lower threshold, which only makes
// later tiles larger.
//
// Bounded by vector instructions: about 25 per element and level, against 8 B
// in and 8 to 20 B out.  8M keys in 256 runs: 235 us over all levels, where
// eight pairwise levels took 900 us; 16M keys in 16 x 16 runs: 305 us, against
// 670 us of four.
template <bool OUT, u32 RUNS>
__global__ __launch_bounds__(MW_NT) void k_mw_tile(MwLevel M, MwOut W)
{
    __shared__ u64 sk[MW_CAP];
    __shared__ u16 si[MW_CAP];
    constexpr u32 R = RUNS / MW_NT;  // runs per thread, consecutive ones
    __shared__ u32 woff[RUNS + 1], wlo[RUNS];
    __shared__ u32 s_sum[MW_NT / 64], s_lo[MW_NT / 64];
    __shared__ u64 s_prev[MW_NT / 64], s_min[MW_NT / 64];
    __shared__ u32 s_n, s_base, s_big;
    if (*M.bad) return;  // (uniform)
    const u32 t = threadIdx.x, lane = t & 63, wv = t >> 6;
    // consecutive tiles on one XCD (workgroups go round the eight): neighbours
    // share the lines of their windows' ends in its L2
    const u32 per = gridDim.x / 8, tile = blockIdx.x < 8 * per ? (blockIdx.x & 7) * per + (blockIdx.x >> 3) : blockIdx.x;
    const u32 g = mw_find(M.ts, M.groups, tile);
    const u32 j0 = M.gs[g], kg = M.gs[g + 1] - j0;
    const u32 row = tile - M.ts[g], nt1 = M.ts[g + 1] - M.ts[g] + 1;
    const u32 *b = M.bounds + M.bo[g] + row;
    u32 nr[R], inc = 0, sl = 0;
    u64 prev = 0, mn = ~0ull;  // the largest key before the tile, the smallest in it (level 0)
#pragma unroll
    for (u32 q = 0; q < R; q++) {
        const u32 w = R * t + q;
        nr[q] = 0;
        if (w < kg) {
            const u32 lo = b[w * nt1];
            nr[q] = b[w * nt1 + 1] - lo;
            wlo[w] = lo;
            sl += lo;
            inc += nr[q];
            if (OUT) {
                const u64 *k = M.K + M.ps[j0 + w];
                if (lo) { const u64 y = k[lo - 1]; prev = y > prev ? y : prev; }
                if (nr[q]) { const u64 y = k[lo]; mn = y < mn ? y : mn; }
            }
        }
    }
    u32 ex = inc;  // (less its own below)
#pragma unroll
    for (u32 d = 1; d < 64; d <<= 1) {
        const u32 y = __shfl_up(inc, d, 64);
        if (lane >= d) inc += y;
        sl += __shfl_xor(sl, d, 64);
        if (OUT) {
            const u64 a = __shfl_xor(prev, d, 64), b = __shfl_xor(mn, d, 64);
            prev = a > prev ? a : prev;
            mn = b < mn ? b : mn;
        }
    }
    if (lane == 63) {
        s_sum[wv] = inc;
        s_lo[wv] = sl;
        if (OUT) {
            s_prev[wv] = prev;
            s_min[wv] = mn;
        }
    }
    if (t == 0) s_n = s_big = 0;
    __syncthreads();
    ex = inc - ex;
    u32 cnt = 0, before = 0;
#pragma unroll
    for (u32 w = 0; w < MW_NT / 64; w++) {
        if (w < wv) ex += s_sum[w];
        cnt += s_sum[w];
        before += s_lo[w];  // keys of the group before this tile
        if (OUT) {
            prev = s_prev[w] > prev ? s_prev[w] : prev;
            mn = s_min[w] < mn ? s_min[w] : mn;
        }
    }
#pragma unroll
    for (u32 q = 0; q < R; q++) {
        if (R * t + q < kg) woff[R * t + q] = ex;
        ex += nr[q];
    }
    if (t == 0) woff[kg] = cnt;
    if (cnt == 0) return;  // (uniform)
    __syncthreads();
    const u32 X = M.ps[j0] + before;  // the tile's first output (level 0: in output space as well)
    const u32 C = OUT ? W.Cg[g] : 0u;
    // source of window element u: its run (of the group) and position in the run
    auto run_at = [&](u32 u) { return mw_find(woff, kg, u); };
    if (cnt > MW_CAP) {  // (uniform)
        if (!OUT) {
            const u64 low = row ? mw_threshold(M, j0, kg, row, M.ts[g + 1] - M.ts[g]) : 0ull;
            for (u32 e = t; e < cnt; e += MW_NT) W.keys[X + e] = low;
        } else {
            u64 mx = 0;  // its largest key
#pragma unroll
            for (u32 q = 0; q < R; q++)
                if (nr[q]) {
                    const u64 y = M.K[M.ps[j0 + R * t + q] + wlo[R * t + q] + nr[q] - 1];
                    mx = y > mx ? y : mx;
                }
#pragma unroll
            for (u32 d = 1; d < 64; d <<= 1) {
                const u64 y = __shfl_xor(mx, d, 64);
                mx = y > mx ? y : mx;
            }
            if (lane == 0) s_min[wv] = mx;
            __syncthreads();
            if (t == 0) {
                for (u32 w = 0; w < MW_NT / 64; w++) mx = s_min[w] > mx ? s_min[w] : mx;
                W.O.lcp[X] = before ? key_lcp(prev, mn, C) : 0u;
                if (mx != mn) {
                    mw_route(W, Seg{X, X + cnt, C, SEG_INB}, tile);
                } else {
                    const u32 c8 = (u32)(mn & 0xFF);
                    W.over[atomicAdd(&W.s.ctr[C_RTILES], 1u)] = Seg{X, X + cnt, C + c8, tile | MW_EQUAL};
                    atomicAdd(&W.s.ctr[C_NELEM], cnt);
                    if (c8 == 8) {
                        W.ties[atomicAdd(&W.s.ctr[C_RNEXT], 1u)] = Seg{X, X + cnt, C + 7, 0};
                        W.s.ctr[C_TIEBIG] = 1;
                    }
                }
            }
        }
        return;
    }
    for (u32 e = t; e < cnt; e += MW_NT) {
        const u32 r = run_at(e);
        sk[e] = M.K[M.ps[j0 + r] + wlo[r] + (e - woff[r])];
        if (OUT) si[e] = (u16)e;
    }
    __syncthreads();
    const u32 ipt = ((cnt + MW_NT - 1) / MW_NT) | 1u;
    const u32 x0 = t * ipt;
    for (u32 lv = 0; (1u << lv) < kg; lv++) {  // (uniform)
        u64 k[MW_IPT];
        u16 v[MW_IPT];
        // lists of 2^lv windows: bounds of list i
        auto at = [&](u32 i) { const u32 w = i << lv; return woff[w < kg ? w : kg]; };
        if (x0 < cnt) {
            u32 lo = 0, hi = (kg + (2u << lv) - 1) >> (lv + 1);  // largest pair starting at or before x0
            while (hi - lo > 1) {
                const u32 mid = (lo + hi) >> 1;
                if (at(2 * mid) <= x0) lo = mid;
                else hi = mid;
            }
            u32 p = lo;
            u32 pb = at(2 * p), pa = at(2 * p + 1), pe = at(2 * p + 2);
            const u32 d = x0 - pb, na = pa - pb, nb = pe - pa;
            lo = d > nb ? d - nb : 0u;
            hi = d < na ? d : na;
            while (lo < hi) {
                const u32 mid = (lo + hi) >> 1;
                if (sk[pb + mid] <= sk[pa + d - 1 - mid]) lo = mid + 1;
                else hi = mid;
            }
            u32 i = pb + lo, j = pa + d - lo;
            u64 ka = i < pa ? sk[i] : 0ull, kb = j < pe ? sk[j] : 0ull;
#pragma unroll
            for (u32 q = 0; q < MW_IPT; q++) {
                if (q < ipt && x0 + q < cnt) {
                    while (i == pa && j == pe) {  // the next pair
                        p++;
                        pb = pe;
                        pa = at(2 * p + 1);
                        pe = at(2 * p + 2);
                        i = pb;
                        j = pa;
                        ka = i < pa ? sk[i] : 0ull;
                        kb = j < pe ? sk[j] : 0ull;
                    }
                    const bool first = j >= pe || (i < pa && ka <= kb);
                    const u32 src = first ? i : j;
                    k[q] = first ? ka : kb;
                    if (OUT) v[q] = si[src];
                    i += first ? 1u : 0u;
                    j += first ? 0u : 1u;
                    const u32 nx = src + 1;
                    const u64 kn = nx < (first ? pa : pe) ? sk[nx] : 0ull;
                    ka = first ? kn : ka;
                    kb = first ? kb : kn;
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (u32 q = 0; q < MW_IPT; q++)
            if (q < ipt && x0 + q < cnt) {
                sk[x0 + q] = k[q];
                if (OUT) si[x0 + q] = v[q];
            }
        __syncthreads();
    }
    if (!OUT) {
        for (u32 e = t; e < cnt; e += MW_NT) W.keys[X + e] = sk[e];
        return;
    }
    // first of the elements equal to element e (strides that double, then halve:
    // most tied runs are short)
    auto first_equal = [&](u32 e, u64 key) {
        u32 s = 1;
        for (; s <= e && sk[e - s] == key; s <<= 1) e -= s;
        for (s >>= 1; s; s >>= 1)
            if (s <= e && sk[e - s] == key) e -= s;
        return e;
    };
    u32 lasts = 0, it = 0;  // bit per element of this thread: the last of a tied run from several runs
    for (u32 e = t; e < cnt; e += MW_NT, it++) {
        const u64 kb = sk[e];
        const u32 u = si[e], r = run_at(u), i = wlo[r] + (u - woff[r]), G = W.rbeg[j0 + r] + i;
        const u32 x = X + e;
        const u32 c8 = (u32)(kb & 0xFF);
        const u64 ka = e ? sk[e - 1] : prev;
        u32 l;
        bool tied = false;  // with a neighbour
        if (e == 0) {
            l = before ? key_lcp(ka, kb, C) : 0u;
        } else if (ka != kb) {
            l = key_lcp(ka, kb, C);
        } else if (c8 < 8) {
            l = C + c8;
        } else {
            l = W.fc_lcp[G];  // (right if the predecessor is of the same run: then it is entry G - 1)
            tied = true;
        }
        W.O.id[x] = W.O.fc_id[G];
        if (W.O.src) W.O.src[x] = ((u64)W.rrun[j0 + r] << 32) | i;
        if (W.O.len) W.O.len[x] = W.O.fc_len[G];
        W.O.lcp[x] = l;
        const bool next = c8 == 8 && e + 1 < cnt && sk[e + 1] == kb;
        if (tied || next) {
            // the tied run's ends
            const u32 a = first_equal(e, kb);
            u32 y = e, s = 1;
            for (; y + s < cnt && sk[y + s] == kb; s <<= 1) y += s;
            for (s >>= 1; s; s >>= 1)
                if (y + s < cnt && sk[y + s] == kb) y += s;
            if (run_at(si[a]) != run_at(si[y])) {
                // (with what a comparison needs of it, read here where the
                // windows' entries are neighbours)
                W.order[x] = G;
                W.s.keyB[x] = W.suf_off[G];
                W.s.mpr[x] = make_uint2(W.fc_len[G], W.fc_lcp[G]);
                if (e == y) lasts |= 1u << it;
            }
        }
    }
    if (__syncthreads_or(lasts != 0)) {
        for (int pass = 0; pass < 2; pass++) {  // counted, then written
            for (u32 m = lasts; m; m &= m - 1) {
                const u32 e = t + MW_NT * (u32)(__ffs((int)m) - 1);
                const u32 a = first_equal(e, sk[e]);
                const u32 slot = atomicAdd(&s_n, 1u);
                if (pass == 0) {
                    if (e + 1 - a > TIE_SMALL) s_big = 1;
                } else W.ties[s_base + slot] = Seg{X + a, X + e + 1, C + 7, TIE_REC};
            }
            __syncthreads();
            if (pass == 0 && t == 0) {
                s_base = atomicAdd(&W.s.ctr[C_RNEXT], s_n);
                if (s_big) W.s.ctr[C_TIEBIG] = 1;
                s_n = 0;
            }
            __syncthreads();
        }
    }
}

// Groups of more runs than a tile merge takes: all their elements as one
// segment each, the keys where the scan left them (run order is output order).
__global__ __launch_bounds__(256) void k_mw_whole(const u32 *wg, u32 nwg, const u32 *gs, const u32 *ps, u32 kc,
                                                  u32 n_out, MwOut W)
{
    for (u32 x = blockIdx.x * blockDim.x + threadIdx.x; x < n_out; x += gridDim.x * blockDim.x) {
        const u32 j = mw_find(ps, kc, x);
        u32 lo = 0, hi = nwg;  // whether run j's group is one of them
        while (lo < hi) {
            const u32 mid = (lo + hi) >> 1;
            if (gs[wg[mid] + 1] <= j) lo = mid + 1;
            else hi = mid;
        }
        if (lo >= nwg || gs[wg[lo]] > j) continue;
        const u32 g = wg[lo];
        W.order[x] = W.rbeg[j] + (x - ps[j]);
        if (x == ps[gs[g]]) {
            const u32 cnt = ps[gs[g + 1]] - x;
            W.O.lcp[x] = 0;
            mw_route(W, Seg{x, x + cnt, W.Cg[g], 0}, MW_GROUP);
        }
    }
}

// Keys and entries of the tiles that became segments, MW_OVER at a time, into
// the sort's second pair (the first still holds the runs' keys); of those with
// one key the order, which is final but for ties, and the LCPs of strings that
// end in it.  They may hold most of the input (few distinct strings): copying 1M
// copies of one string from 8 runs took the tile's own workgroup 1150 us.
#define MW_OVER 2048
template <u32 RUNS>
__global__ __launch_bounds__(MW_NT) void k_mw_over(MwLevel M, MwOut W, const u32 *tstart, u32 nover)
{
    constexpr u32 R = RUNS / MW_NT;
    __shared__ u32 woff[RUNS + 1], wlo[RUNS], s_sum[MW_NT / 64];
    const u32 t = threadIdx.x, lane = t & 63, wv = t >> 6;
    if (blockIdx.x >= tstart[nover]) return;
    const u32 s = seg_of_tile(tstart, nover, blockIdx.x);
    const Seg o = W.over[s];
    if (o.aux == MW_GROUP) return;  // (uniform, as all of this)
    const u32 tile = o.aux & ~MW_EQUAL, g = mw_find(M.ts, M.groups, tile);
    const u32 j0 = M.gs[g], kg = M.gs[g + 1] - j0;
    const u32 row = tile - M.ts[g], nt1 = M.ts[g + 1] - M.ts[g] + 1;
    const u32 *b = M.bounds + M.bo[g] + row;
    u32 nr[R], inc = 0;
#pragma unroll
    for (u32 q = 0; q < R; q++) {
        const u32 w = R * t + q;
        nr[q] = 0;
        if (w < kg) {
            wlo[w] = b[w * nt1];
            nr[q] = b[w * nt1 + 1] - wlo[w];
            inc += nr[q];
        }
    }
    u32 ex = inc;  // (less its own below)
#pragma unroll
    for (u32 d = 1; d < 64; d <<= 1) {
        const u32 y = __shfl_up(inc, d, 64);
        if (lane >= d) inc += y;
    }
    if (lane == 63) s_sum[wv] = inc;
    __syncthreads();
    ex = inc - ex;
#pragma unroll
    for (u32 w = 0; w < MW_NT / 64; w++)
        if (w < wv) ex += s_sum[w];
#pragma unroll
    for (u32 q = 0; q < R; q++) {
        if (R * t + q < kg) woff[R * t + q] = ex;
        ex += nr[q];
    }
    __syncthreads();
    const u32 cnt = o.end - o.begin, e0 = (blockIdx.x - tstart[s]) * MW_OVER, e1 = cnt < e0 + MW_OVER ? cnt : e0 + MW_OVER;
    for (u32 e = e0 + t; e < e1; e += MW_NT) {
        const u32 r = mw_find(woff, kg, e), i = wlo[r] + (e - woff[r]);
        if (o.aux & MW_EQUAL) {
            W.order[o.begin + e] = W.rbeg[j0 + r] + i;
            if (e) W.O.lcp[o.begin + e] = o.depth;
        } else {
            W.s.keyB[o.begin + e] = M.K[M.ps[j0 + r] + i];
            W.s.valB[o.begin + e] = W.rbeg[j0 + r] + i;
        }
    }
}

// ---- tied keys
//
// Segments of outputs whose strings agree up to the segment's depth, in (run,
// position) order; order[x] = the front-coded entry at output x.  Eight lanes
// per 16 members.

#define TIE_T 16  // members of a segment per eight lanes

// A front-coded entry and what a comparison needs of it.
struct FcEl {
    u32 g, d, e;
    u64 so;
};

__device__ __forceinline__ FcEl fc_el(const FcView &V, u32 g) { return FcEl{g, V.d[g], V.e[g], V.suf_off[g]}; }

__device__ __forceinline__ FcEl fc_el_shfl(const FcEl &a, u32 src)  // within eight lanes
{
    return FcEl{__shfl(a.g, src, 8), __shfl(a.d, src, 8), __shfl(a.e, src, 8), __shfl(a.so, src, 8)};
}

// Three-way comparison of front-coded strings X and Y from byte `from` (they
// agree on [0, from)) by eight lanes with the same arguments, 128 bytes a step;
// *lcp receives their LCP.  A string whose own literal holds the byte (the usual
// case) is read from there without a chain walk, otherwise its piece is found
// along its psv chain.
__device__ __forceinline__ int fc_cmp8(const FcView &V, const FcEl &X, const FcEl &Y, u64 from, u32 gl, u64 *lcp)
{
    const u32 x = X.g, y = Y.g, ex = X.e, ey = Y.e;
    const u64 lx = X.d, ly = Y.d, sx = X.so, sy = Y.so;
    const u64 m = lx < ly ? lx : ly;
    u64 i = from < m ? from : m;
    while (i < m) {
        u64 px, ax, py, ay;  // the pieces that hold byte i
        if (ex <= i) { px = sx + (i - ex); ax = lx - i; }
        else fc_piece(V, x, i, &px, &ax);
        if (ey <= i) { py = sy + (i - ey); ay = ly - i; }
        else fc_piece(V, y, i, &py, &ay);
        u64 run = ax < ay ? ax : ay;
        run = run < m - i ? run : m - i;
        for (u64 c = 0; c < run; c += 128) {
            const u64 q = c + 16 * gl;
            const u32 take = q < run ? (run - q < 16 ? (u32)(run - q) : 16u) : 0u;
            const Win16 ra = win16_issue(V.suf, V.sufN, px + q, take), rb = win16_issue(V.suf, V.sufN, py + q, take);
            u64 a0, a1, b0, b1;
            win16_finish(V.suf, ra, a0, a1);
            win16_finish(V.suf, rb, b0, b1);
            const u64 d0 = a0 ^ b0, d1 = a1 ^ b1;
            u32 f = 0xFFFFFFFFu;  // 2 (first differing byte) + (y smaller)
            if (d0 | d1) {
                const u64 d = d0 ? d0 : d1;
                const u32 at = (u32)(__builtin_ctzll(d) >> 3);
                const u32 av = (u32)((d0 ? a0 : a1) >> (8 * at)) & 0xFFu, bv = (u32)((d0 ? b0 : b1) >> (8 * at)) & 0xFFu;
                f = (16 * gl + (d0 ? 0u : 8u) + at) * 2 + (av < bv ? 0u : 1u);
            }
#pragma unroll
            for (int s = 1; s < 8; s <<= 1) {
                const u32 z = __shfl_xor(f, s, 8);
                f = z < f ? z : f;
            }
            if (f != 0xFFFFFFFFu) {
                *lcp = i + c + (f >> 1);
                return (f & 1) ? 1 : -1;
            }
        }
        i += run;
    }
    *lcp = m;
    return lx < ly ? -1 : (lx > ly ? 1 : 0);
}

// Tile counts (`per` members each) of a list of segments; their comparison words
// (see k_tie_compare) and the counters of the lists the round builds are reset.
__global__ void k_tie_tiles(const Seg *list, u32 cnt, u32 per, u32 *tiles, u64 *cmp, u32 *ctr)
{
    const u32 j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < cnt) {
        tiles[j] = (list[j].end - list[j].begin + per - 1) / per;
        if (cmp) cmp[j] = ~0ull;
    }
    if (ctr && j < C_NCTR) ctr[j] = 0;
}

// Segments of up to TIE_SMALL members (most are two equal strings), eight lanes
// each: every pair is compared, a member's rank is the number before it and its
// LCP the largest with one of those.  (Neighbours of one run -- which share the key, unlike a run end and the next start -- need no comparison:
// their LCP is the run's.)  The tile merge has written the results in (run,
// position) order, so those of members that stay where they are -- all of an
// equal run's -- are final, the others are written again here.  Larger segments
// are passed on to `big` (C_RNEXT of them, C_RELEM elements).
//
// Bounded by the latency of scattered reads (entry, then its length, LCP and
// offset, then the bytes, 128 a step).  The ties of 4M text strings in 16 x 16
// runs took about 1.9 ms inside the former pairwise merge, where one lane's
// comparison held up its wavefront, and about 0.3 ms so.
__global__ __launch_bounds__(256) void k_tie_small(const Seg *list, u32 cnt, FcView V, u32 *order, const u64 *rso,
                                                   const uint2 *rde, MergeOut O, Seg *big, u32 *ctr)
{
    __shared__ u32 s_n, s_el, s_base;
    if (threadIdx.x == 0) s_n = s_el = 0;
    __syncthreads();
    const u32 s = blockIdx.x * 32 + (threadIdx.x >> 3), gl = threadIdx.x & 7;
    Seg g{0, 0, 0, 0};
    if (s < cnt) g = list[s];
    const u32 m = g.end - g.begin;
    u32 slot = 0;
    const bool pass = m > TIE_SMALL && gl == 0;
    if (pass) {
        slot = atomicAdd(&s_n, 1u);
        atomicAdd(&s_el, m);
    }
    __syncthreads();
    if (threadIdx.x == 0 && s_n) {
        s_base = atomicAdd(&ctr[C_RNEXT], s_n);
        atomicAdd(&ctr[C_RELEM], s_el);
    }
    __syncthreads();
    if (pass) big[s_base + slot] = g;
    // (no barrier from here on: a wavefront with long strings holds up no other)
    if (m && m <= TIE_SMALL) {
        FcEl E{0, 0, 0, 0};
        if (gl < m) {
            const u32 p = g.begin + gl;
            if (g.aux & TIE_REC) {
                const uint2 de = rde[p];
                E = FcEl{order[p], de.x, de.y, rso[p]};
            } else {
                E = fc_el(V, order[p]);
            }
        }
        u32 rank = 0, mx = 0;
        for (u32 i = 0; i + 1 < m; i++) {
            const FcEl A = fc_el_shfl(E, i);
            for (u32 j = i + 1; j < m; j++) {
                const FcEl B = fc_el_shfl(E, j);
                u64 l = B.e;
                const bool nb = B.g == A.g + 1 && B.e >= g.depth;
                const bool after = !nb && fc_cmp8(V, A, B, g.depth, gl, &l) > 0;  // i after j
                if (gl == (after ? i : j)) {
                    rank++;
                    mx = (u32)l > mx ? (u32)l : mx;
                }
            }
        }
        if (gl < m) {
            const u32 p = g.begin + rank;
            if (rank) O.lcp[p] = mx;
            if (rank != gl) {
                order[p] = E.g;
                if (g.aux & TIE_REC) merge_emit(O, p, E.g);  // (else: with the larger segment it came from)
            }
        }
    }
}

// Members of larger segments against the segment's first: the minimum over a
// segment of 2 LCP + (equal) says how far all agree and whether all are equal.
__global__ __launch_bounds__(256) void k_tie_compare(const Seg *list, const u32 *tiles, u32 cnt, FcView V,
                                                     const u32 *order, u64 *cmp)
{
    const u32 t = blockIdx.x * 32 + (threadIdx.x >> 3), gl = threadIdx.x & 7;
    if (t >= tiles[cnt]) return;
    const u32 s = seg_of_tile(tiles, cnt, t);
    const Seg g = list[s];
    const u32 p0 = g.begin + (t - tiles[s]) * TIE_T, p1 = g.end < p0 + TIE_T ? g.end : p0 + TIE_T;
    const FcEl F = fc_el(V, order[g.begin]);
    FcEl E[TIE_T / 8];
#pragma unroll
    for (u32 h = 0; h < TIE_T / 8; h++) E[h] = fc_el(V, order[p0 + 8 * h + gl < p1 ? p0 + 8 * h + gl : p0]);
    u64 best = ~0ull;
#pragma unroll
    for (u32 h = 0; h < TIE_T / 8; h++)
        for (u32 q = 0; q < 8 && p0 + 8 * h + q < p1; q++) {
            if (p0 + 8 * h + q == g.begin) continue;
            u64 l;
            const int r = fc_cmp8(V, F, fc_el_shfl(E[h], q), g.depth, gl, &l);
            const u64 w = 2 * l + (r == 0 ? 1u : 0u);
            best = w < best ? w : best;
        }
    // (a segment's tiles meet on its word: only what would change it as it is read
    // is committed; it only ever falls)
    if (gl == 0 && best < __hip_atomic_load(&cmp[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMin((unsigned long long *)&cmp[s], (unsigned long long)best);
}

// The larger segments after their comparison: equal strings are done (LCP =
// length, in order already); of the others the keys at their exact common
// prefix are written and the segment goes to the sort of its size.
__global__ __launch_bounds__(256) void k_tie_keys(const Seg *list, const u32 *tiles, u32 cnt, FcView V,
                                                  const u32 *order, u32 *lcp, const u64 *cmp, SortWs w, SortShape z)
{
    const u32 t = blockIdx.x * 32 + (threadIdx.x >> 3), gl = threadIdx.x & 7;
    if (t >= tiles[cnt]) return;
    const u32 s = seg_of_tile(tiles, cnt, t);
    const Seg g = list[s];
    const u32 m = g.end - g.begin;
    const u32 lt = t - tiles[s];
    const u32 p0 = g.begin + lt * TIE_T, p1 = g.end < p0 + TIE_T ? g.end : p0 + TIE_T;
    const u64 c = cmp[s];
    const u64 dep = c >> 1;
    if (c & 1) {
        for (u32 p = p0 + gl; p < p1; p += 8)
            if (p > g.begin) lcp[p] = (u32)dep;
        return;
    }
    for (u32 p = p0 + gl; p < p1; p += 8) {
        const u32 G = order[p];
        const u64 d = V.d[G];
        u64 v = 0;
        u64 i = dep;
        const u64 e = d < dep + 7 ? d : dep + 7;
        while (i < e) {  // the pieces of [dep, dep + 7)
            u64 pos, av;
            fc_piece(V, G, i, &pos, &av);
            const u32 take = (u32)(av < e - i ? av : e - i);
            v |= load_be(V.suf, V.sufN, pos, take) >> (8 * (i - dep));
            i += take;
        }
        w.keyA[p] = v | (d - dep < 8 ? d - dep : 8ull);
    }
    if (lt == 0 && gl == 0) {
        const Seg o{g.begin, g.end, (u32)dep, 0};
        if (m <= WS_MAX) {
            w.tiny[atomicAdd(&w.ctr[C_TINY], 1u)] = o;
            atomicAdd(&w.ctr[C_TINYN], m);
        } else if (m <= z.block_max) {
            if (m <= BS_SMALL) w.small[atomicAdd(&w.ctr[C_SMALL], 1u)] = o;
            else w.mid[atomicAdd(&w.ctr[C_MID], 1u)] = o;
            atomicAdd(&w.ctr[C_SMALLN], m);
        } else {
            w.largeA[atomicAdd(&w.ctr[C_LARGE], 1u)] = Seg{o.begin, o.end, o.depth, SEG_NOROOT};
            atomicAdd(&w.ctr[C_LTILES], (m + z.tile - 1) / z.tile);
            atomicAdd(&w.ctr[C_LELEM], m);
        }
    }
}

// The results of the tied elements, once their order is final.
__global__ __launch_bounds__(256) void k_tie_emit(const Seg *list, const u32 *tiles, u32 cnt, const u32 *order,
                                                  MergeOut O)
{
    const u32 t = blockIdx.x * 32 + (threadIdx.x >> 3), gl = threadIdx.x & 7;
    if (t >= tiles[cnt]) return;
    const u32 s = seg_of_tile(tiles, cnt, t);
    const Seg g = list[s];
    const u32 p0 = g.begin + (t - tiles[s]) * TIE_T, p1 = g.end < p0 + TIE_T ? g.end : p0 + TIE_T;
    for (u32 p = p0 + gl; p < p1; p += 8) merge_emit(O, p, order[p]);
}

// Host-plan header: [0] check flag, [1] literal-buffer size, [2, 2+k) run
// begins, [2+k, 2+2k) run ends, then the group offsets as packed u32.
__global__ __launch_bounds__(256) void k_merge_header(const u64 *rb, const u64 *re, u32 k, const u32 *go,
                                                      u32 groups, const u32 *bad, const u64 *sufN, u64 *H)
{
    const u64 t = (u64)blockIdx.x * blockDim.x + threadIdx.x;
    if (t == 0) {
        H[0] = bad ? *bad : 0u;
        H[1] = sufN ? *sufN : 0ull;
    }
    if (t < k) {
        H[2 + t] = rb[t];
        H[2 + k + t] = re[t];
    }
    if (t <= groups) ((u32 *)(H + 2 + 2 * (u64)k))[t] = go[t];
}

__global__ __launch_bounds__(256) void k_check_merge_runs(const u64 *rb, const u64 *re, u32 k, u64 n_fc,
                                                          const u32 *e, const u32 *d, u32 *bad)
{
    const u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < k) {
        if (re[i] < rb[i] || re[i] > n_fc) atomicOr(bad, 1u);
        else if (re[i] > rb[i] && e[rb[i]] != 0) atomicOr(bad, 2u);
    }
    if (i < n_fc) {
        if (e[i] > d[i]) atomicOr(bad, 4u);
        if (i > 0 && e[i] > d[i - 1]) atomicOr(bad, 4u);
    }
}

struct MergeWs {
    DecWs dec;
    SortWs sort;  // (its key arrays hold the merge's keys and samples before any tie is sorted)
    u32 *sid, *plan, *Cg, *rgroup, *rep, *runmin, *bfirst, *ties, *order, *tiles;
    Seg *segs, *over, *big;
    MOp *mblk;
    u64 *P, *sb;
};

#define MERGE_MAX_K 65536
// words of the merge plan: per level run starts, tile starts and bounds starts;
// the group starts, runs and their front-coded starts, groups taken whole, long runs
#define MERGE_PLAN(k) ((3 * (size_t)MW_LEVELS + 7) * ((size_t)(k) + 4))

static void merge_layout(u64 n_out, u64 n_fc, u64 k, MergeWs *w, WsArena *a, WsCounter *c)
{
    dec_layout(n_fc, &w->dec, a, c);
    sort_ws_layout(n_out, &w->sort, a, c);
#define MT(field, T, cnt)                       \
    do {                                         \
        if (a) w->field = a->take<T>(cnt);       \
        else c->take<T>(cnt);                    \
    } while (0)
    // host-planned arrays, in one contiguous block (uploaded in one copy)
    MT(P, u64, k + 2); MT(sb, u64, k + 2); MT(sid, u32, k + 2); MT(rgroup, u32, k + 2); MT(rep, u32, k + 2);
    MT(plan, u32, MERGE_PLAN(k));
    MT(Cg, u32, k + 2);
    MT(runmin, u32, k + 2); MT(mblk, MOp, n_out / MS_ITEMS + 2); MT(bfirst, u32, n_out / MS_ITEMS + 2);
    MT(ties, u32, 4);
    MT(order, u32, n_out); MT(segs, Seg, n_out / 2 + 2); MT(tiles, u32, n_out / 2 + 3);
    MT(over, Seg, n_out / (MW_CAP + 1) + k + 2); MT(big, Seg, n_out / TIE_SMALL + 2);
#undef MT
}

// Host arrays to device arrays that lie in one block in this order: staged in
// pinned memory at the same relative offsets and uploaded by one asynchronous
// copy (the staging buffer is reused once the copy has run).  Without pinned
// memory: one copy each, and a wait before the host arrays go away.
struct UpPart {
    void *dst;
    const void *src;
    size_t bytes;
};

static int upload_parts(const UpPart *parts, int np, hipStream_t st)
{
    u8 *base = (u8 *)parts[0].dst;
    const size_t span = (size_t)((u8 *)parts[np - 1].dst - base) + parts[np - 1].bytes;
    void *pin = ss_upload_take(span);
    if (!pin) {
        for (int q = 0; q < np; q++)
            if (parts[q].bytes) SS_HIP(hipMemcpyAsync(parts[q].dst, parts[q].src, parts[q].bytes,
                                                      hipMemcpyHostToDevice, st));
        SS_HIP(hipStreamSynchronize(st));
        return SS_OK;
    }
    for (int q = 0; q < np; q++)
        if (parts[q].bytes) memcpy((u8 *)pin + ((u8 *)parts[q].dst - base), parts[q].src, parts[q].bytes);
    const hipError_t e = hipMemcpyAsync(base, pin, span, hipMemcpyHostToDevice, st);
    ss_upload_release(pin, st);
    if (e != hipSuccess) {
        ss_set_error("plan upload failed: %s", hipGetErrorString(e));
        return SS_ERR_HIP;
    }
    return SS_OK;
}

extern "C" size_t ss_lcp_merge_workspace(uint64_t n_out, uint64_t n_fc, uint32_t k)
{
    WsCounter c;
    MergeWs w;
    merge_layout(n_out, n_fc, k, &w, nullptr, &c);
    return c.used;
}

extern "C" int ss_lcp_merge(uint32_t k, const uint64_t *run_begin, const uint64_t *run_end, uint32_t groups,
                            const uint32_t *group_off, uint64_t n_fc, const uint32_t *fc_lcp, const uint32_t *fc_len,
                            const uint32_t *fc_id, const uint64_t *suf_off, const uint8_t *suf, uint64_t *out_src,
                            uint32_t *out_id, uint32_t *out_lcp, uint32_t *out_len, uint64_t out_cap,
                            uint64_t *n_out_host, void *ws, size_t ws_bytes, void *stream)
{
    ss_clear_error();
    if (n_fc >= 0xFFFFFFFFull) { ss_set_error("n_fc too large"); return SS_ERR_TOO_LARGE; }
    if (k == 0 || k > MERGE_MAX_K || groups == 0 || groups > k || !run_begin || !run_end || !group_off) {
        ss_set_error("lcp_merge: bad arguments (1 <= k <= %d, 1 <= groups <= k)", MERGE_MAX_K);
        return SS_ERR_INVALID_ARG;
    }
    hipStream_t st = (hipStream_t)stream;
    // The format check of the front-coded runs runs on the device before the
    // run bounds are known on the host, so that one read-back serves both.
    // Its flag lives in the decoding part of the workspace, whose placement
    // depends on n_fc only.
    WsArena a0(ws, ws_bytes);
    DecWs d0;
    dec_layout(n_fc, &d0, &a0, nullptr);
    if (a0.overflow || !ws) {
        ss_set_error("workspace too small for %llu front-coded entries", (unsigned long long)n_fc);
        return SS_ERR_WORKSPACE;
    }
    const bool have_fc = fc_lcp && fc_len && fc_id && suf_off;
    if (have_fc) {
        SS_HIP(hipMemsetAsync(d0.bad, 0, sizeof(u32), st));
        k_check_merge_runs<<<(unsigned)ceil_div((n_fc > k ? n_fc : k) + 1, 256), 256, 0, st>>>(
            run_begin, run_end, k, n_fc, fc_lcp, fc_len, d0.bad);
        SS_CHECK_LAUNCH();
    }
    // Everything the host plan needs, packed on the device into one staging
    // array (after the decoding part of the workspace; the merge arrays reuse
    // that space later) and brought back by one copy.
    std::vector<u64> rb(k), re(k);
    std::vector<u32> go(groups + 1);
    const u64 hdr = 2 + 2 * (u64)k + ((u64)groups + 2) / 2;
    u64 *stage = a0.take<u64>(hdr);
    std::vector<u64> H(hdr);
    if (stage) {
        const u64 nt = (u64)k > (u64)groups + 1 ? (u64)k : (u64)groups + 1;
        k_merge_header<<<(unsigned)ceil_div(nt, 256), 256, 0, st>>>(run_begin, run_end, k, group_off, groups,
                                                                    have_fc ? d0.bad : nullptr,
                                                                    have_fc ? suf_off + n_fc : nullptr, stage);
        SS_CHECK_LAUNCH();
        SS_TRY(ss_read_bytes(stage, H.data(), sizeof(u64) * hdr, st));
        memcpy(rb.data(), H.data() + 2, sizeof(u64) * k);
        memcpy(re.data(), H.data() + 2 + k, sizeof(u64) * k);
        memcpy(go.data(), H.data() + 2 + 2 * (u64)k, sizeof(u32) * (groups + 1));
    } else {
        H[0] = H[1] = 0;
        u32 b32 = 0;
        if (have_fc) {
            SS_HIP(hipMemcpyAsync(&b32, d0.bad, sizeof(u32), hipMemcpyDeviceToHost, st));
            SS_HIP(hipMemcpyAsync(&H[1], suf_off + n_fc, sizeof(u64), hipMemcpyDeviceToHost, st));
        }
        SS_HIP(hipMemcpyAsync(rb.data(), run_begin, sizeof(u64) * k, hipMemcpyDeviceToHost, st));
        SS_HIP(hipMemcpyAsync(re.data(), run_end, sizeof(u64) * k, hipMemcpyDeviceToHost, st));
        SS_HIP(hipMemcpyAsync(go.data(), group_off, sizeof(u32) * (groups + 1), hipMemcpyDeviceToHost, st));
        SS_HIP(hipStreamSynchronize(st));
        H[0] = b32;
    }
    const u32 bad = (u32)H[0];
    const u64 sufN = H[1];
    if (go[0] != 0 || go[groups] != k) {
        ss_set_error("group_off must start at 0 and end at k");
        return SS_ERR_INVALID_ARG;
    }
    std::vector<u64> P(k + 1, 0);
    for (u32 j = 0; j < k; j++) {
        if (re[j] < rb[j] || re[j] > n_fc) {
            ss_set_error("run %u = [%llu, %llu) is not inside the %llu front-coded entries", j,
                         (unsigned long long)rb[j], (unsigned long long)re[j], (unsigned long long)n_fc);
            return SS_ERR_INVALID_ARG;
        }
        P[j + 1] = P[j] + (re[j] - rb[j]);
    }
    for (u32 g = 0; g < groups; g++)
        if (go[g + 1] < go[g]) {
            ss_set_error("group_off must be non-decreasing");
            return SS_ERR_INVALID_ARG;
        }
    const u64 n_out = P[k];
    if (n_out_host) *n_out_host = n_out;
    if (n_out == 0) return SS_OK;
    if (n_out > out_cap) {
        ss_set_error("merge output has %llu entries, capacity %llu", (unsigned long long)n_out,
                     (unsigned long long)out_cap);
        return SS_ERR_CAPACITY;
    }
    if (!have_fc || !out_id || !out_lcp) {
        ss_set_error("lcp_merge: null array");
        return SS_ERR_INVALID_ARG;
    }
    if (bad) {
        ss_set_error("malformed front-coded runs (code %u): runs must start with e = 0 and e_i <= d_i, "
                     "e_i <= d_{i-1}", bad);
        return SS_ERR_INVALID_ARG;
    }
    // non-empty runs sorted by front-coded start, to map positions back to runs
    std::vector<u32> order;
    for (u32 j = 0; j < k; j++)
        if (re[j] > rb[j]) order.push_back(j);
    std::sort(order.begin(), order.end(), [&](u32 x, u32 y) { return rb[x] < rb[y]; });
    for (size_t t = 1; t < order.size(); t++)
        if (re[order[t - 1]] > rb[order[t]]) {
            ss_set_error("runs overlap");
            return SS_ERR_INVALID_ARG;
        }
    const u32 kne = (u32)order.size();
    std::vector<u64> sbv(kne);
    std::vector<u32> sidv(kne);
    for (u32 t = 0; t < kne; t++) { sbv[t] = rb[order[t]]; sidv[t] = order[t]; }

    WsArena a(ws, ws_bytes);
    MergeWs w;
    merge_layout(n_out, n_fc, k, &w, &a, nullptr);
    if (a.overflow) {
        ss_set_error("workspace too small: need %zu bytes", ss_lcp_merge_workspace(n_out, n_fc, k));
        return SS_ERR_WORKSPACE;
    }

    const FcView V{fc_lcp, fc_len, w.dec.psv, suf_off, suf, sufN};
    // group of every run, first non-empty run of every group
    std::vector<u32> rg(k), rep(groups, 0);
    for (u32 g = 0; g < groups; g++) {
        bool found = false;
        for (u32 j = go[g]; j < go[g + 1]; j++) {
            rg[j] = g;
            if (!found && re[j] > rb[j]) { rep[g] = j; found = true; }
        }
    }
    // The plan of the merge by key: the non-empty runs, and per level of the
    // key lists their starts, tiles and bounds.
    std::vector<u32> plan;
    struct Lv { size_t ps, ts, bo; u32 tiles, bounds; };
    std::vector<Lv> lv;
    std::vector<u32> gs(groups + 1), whole;
    std::vector<u64> len;  // of every non-empty run in the current level
    std::vector<u32> rrun, rbeg;
    for (u32 g = 0; g < groups; g++) {
        gs[g] = (u32)rrun.size();
        for (u32 j = go[g]; j < go[g + 1]; j++)
            if (re[j] > rb[j]) {
                rrun.push_back(j);
                rbeg.push_back((u32)rb[j]);
                len.push_back(re[j] - rb[j]);
            }
    }
    const u32 kc = (u32)rrun.size();
    gs[groups] = kc;
    u32 nsample = 0;
    bool few = true, ranked = false, leveled = false;
    for (u32 v = 0; v < MW_LEVELS; v++) {
        Lv L{plan.size(), 0, 0, 0, 0};
        u32 at = v < 2 ? 0u : nsample;  // (levels 1, 2, ... lie behind each other in the sample array)
        for (u32 j = 0; j < kc; j++) { plan.push_back(at); at += (u32)len[j]; }
        plan.push_back(at);
        if (v) nsample = at;
        L.ts = plan.size();
        std::vector<u32> bo(groups + 1);
        bool more = false;
        for (u32 g = 0; g < groups; g++) {
            const u32 kg = gs[g + 1] - gs[g];
            u64 tot = 0, ns = 0;
            for (u32 j = gs[g]; j < gs[g + 1]; j++) { tot += len[j]; ns += mw_samples(len[j], j - gs[g], kg); }
            plan.push_back(L.tiles);
            bo[g] = L.bounds;
            u32 nt = 1;
            if (tot > MW_CAP && ns) nt = (u32)ceil_div(tot, MW_TILE);
            // (a bounds matrix of a group must fit two words per key)
            const bool take = kg <= MW_RUNS && (v || (nt + 1) * (u64)kg <= 2 * tot);
            if (v == 0 && tot) few &= !take || kg <= MW_FEW;
            if (v == 1 && tot) (kg <= MW_RANK ? ranked : leveled) = true;
            if (tot == 0 || !take || (v == 1 && kg <= MW_RANK)) {
                if (v == 0 && tot && !take) whole.push_back(g);
                for (u32 j = gs[g]; j < gs[g + 1]; j++) len[j] = 0;
                continue;
            }
            if (tot > MW_CAP) {
                more |= ns > 0;
                for (u32 j = gs[g]; j < gs[g + 1]; j++) len[j] = mw_samples(len[j], j - gs[g], kg);
            } else {
                for (u32 j = gs[g]; j < gs[g + 1]; j++) len[j] = 0;
            }
            L.tiles += nt;
            L.bounds += (nt + 1) * kg;
        }
        plan.push_back(L.tiles);
        L.bo = plan.size();
        bo[groups] = L.bounds;
        plan.insert(plan.end(), bo.begin(), bo.end());
        lv.push_back(L);
        if (!more) break;
    }
    const size_t p_gs = plan.size();
    plan.insert(plan.end(), gs.begin(), gs.end());
    const size_t p_rrun = plan.size();
    plan.insert(plan.end(), rrun.begin(), rrun.end());
    const size_t p_rbeg = plan.size();
    plan.insert(plan.end(), rbeg.begin(), rbeg.end());
    const size_t p_whole = plan.size();
    plan.insert(plan.end(), whole.begin(), whole.end());
    plan.resize(p_whole + groups);
    const u64 rparts = std::min<u64>(ceil_div(n_out, (u64)k * 4096), RM_PARTS);
    const u64 rlimit = rparts < RM_PARTS ? rparts * 32768 : ~0ull;  // (16 steps of a workgroup)
    const size_t p_long = plan.size();
    for (u32 j = 0; j < k; j++)
        if (re[j] - rb[j] > rlimit) plan.push_back(j);
    const u32 nlong = (u32)(plan.size() - p_long);
    // (the samples and their merge share the mismatch words' array, the bounds
    // the boundary list: about n / 7 keys and at most 2 n words)
    if (plan.size() > MERGE_PLAN(k) || 2ull * nsample > n_out) {
        ss_set_error("internal: merge plan exceeds its workspace");
        return SS_ERR_INVALID_ARG;
    }
    for (const Lv &L : lv)
        if (L.bounds > 2 * n_out) {
            ss_set_error("internal: merge bounds exceed their workspace");
            return SS_ERR_INVALID_ARG;
        }
    {
        const UpPart parts[] = {{w.P, P.data(), sizeof(u64) * (k + 1)},
                                {w.sb, sbv.data(), sizeof(u64) * kne},
                                {w.sid, sidv.data(), sizeof(u32) * kne},
                                {w.rgroup, rg.data(), sizeof(u32) * k},
                                {w.rep, rep.data(), sizeof(u32) * groups},
                                {w.plan, plan.data(), sizeof(u32) * plan.size()}};
        SS_TRY(upload_parts(parts, 6, st));
    }
    SortWs &sw = w.sort;
    const u32 nb = (u32)ceil_div(n_out, MS_ITEMS);
    const u32 ni = std::max(std::max(nb, k), std::max(groups, (u32)C_NCTR));
    k_merge_init<<<(unsigned)ceil_div(ni, 256), 256, 0, st>>>(w.P, k, nb, w.bfirst, w.runmin, w.Cg, groups, w.ties,
                                                             sw.ctr);
    SS_CHECK_LAUNCH();
    {
        SS_PROF("k_run_min", st, (double)n_out * 4.0);  // front-coded LCP in
        k_run_min<<<dim3(k, (unsigned)rparts), 256, 0, st>>>(nullptr, rlimit, run_begin, w.P, fc_lcp, w.runmin);
        SS_CHECK_LAUNCH();
        if (nlong) {
            k_run_min<<<dim3(nlong, RM_PARTS), 256, 0, st>>>(w.plan + p_long, rlimit, run_begin, w.P, fc_lcp, w.runmin);
            SS_CHECK_LAUNCH();
        }
    }
    k_group_depth<<<(unsigned)ceil_div(k, 4), 256, 0, st>>>(run_begin, w.P, w.rgroup, w.rep, k, w.runmin, V, w.Cg);
    SS_CHECK_LAUNCH();
    u32 *const unsorted = sw.ctr + C_BADSET;
    u64 *K = sw.keyA, *KS = sw.mword, *KM = sw.mword + nsample;
    u32 *bounds = (u32 *)sw.bnd;
    {
        // front-coded LCP, length, literal offset and up to 7 literal bytes in, LCP once more, key out
        SS_PROF("k_mscan", st, (double)n_out * (28.0 + 8.0));
        const MScan S{run_begin, w.P, w.rgroup, w.Cg, w.bfirst, k, (u32)n_out, V, w.ties};
        k_mscan_reduce<<<nb, 256, 0, st>>>(S, w.mblk);
        SS_CHECK_LAUNCH();
        k_mscan_top<<<1, 1024, 0, st>>>(w.mblk, nb);
        SS_CHECK_LAUNCH();
        k_mscan_apply<<<nb, 256, 0, st>>>(S, w.mblk, K, unsorted);
    }
    SS_CHECK_LAUNCH();
    const u32 *pl = w.plan, *gsd = pl + p_gs;
    const u32 nl = (u32)lv.size() - 1;  // sample levels
    if (nl && nsample) {
        for (u32 v = 1; leveled && v <= nl; v++) {
            const u32 tot = plan[lv[v].ps + kc] - plan[lv[v].ps];
            if (!tot) continue;
            k_mw_sample<<<(unsigned)ceil_div(tot, 256), 256, 0, st>>>(K, pl + lv[0].ps, gsd, groups, kc, pl + lv[v].ps,
                                                                     v, KS);
            SS_CHECK_LAUNCH();
        }
        if (ranked) {
            const u32 tot = plan[lv[1].ps + kc];
            k_mw_rank<<<(unsigned)ceil_div(tot, 256), 256, 0, st>>>(K, pl + lv[0].ps, pl + lv[1].ps, gsd, groups, kc,
                                                                        KM, unsorted);
            SS_CHECK_LAUNCH();
        }
    }
    const MergeOut O{w.sb, w.sid, kne, fc_id, fc_len, out_src, out_id, out_lcp, out_len};
    const SortShape z = sort_shape(n_out);
    const MwOut W{KM, w.Cg, pl + p_rrun, pl + p_rbeg, fc_lcp, fc_len, suf_off, O, w.order, w.segs, w.over, sw, z.tile, z.block_max};
    auto level = [&](u32 v) {
        const Lv &L = lv[v];
        return MwLevel{v ? KS : K, pl + L.ps, gsd, pl + L.ts, pl + L.bo, KM, v < nl ? pl + lv[v + 1].ps : pl + L.ps,
                       groups, bounds, unsorted};
    };
    for (u32 v = nl + 1; v-- > 0;) {
        const Lv &L = lv[v];
        if (!L.tiles) continue;
        const MwLevel M = level(v);
        k_mw_bounds<<<(unsigned)ceil_div(L.bounds, 256), 256, 0, st>>>(M, L.bounds);
        SS_CHECK_LAUNCH();
        if (v) {
            if (few) k_mw_tile<false, MW_FEW><<<L.tiles, MW_NT, 0, st>>>(M, W);
            else k_mw_tile<false, MW_RUNS><<<L.tiles, MW_NT, 0, st>>>(M, W);
        } else {
            // key, id, LCP bytes in; id and LCP out
            SS_PROF("k_mw_tile", st, (double)n_out * 20.0);
            if (few) k_mw_tile<true, MW_FEW><<<L.tiles, MW_NT, 0, st>>>(M, W);
            else k_mw_tile<true, MW_RUNS><<<L.tiles, MW_NT, 0, st>>>(M, W);
        }
        SS_CHECK_LAUNCH();
    }
    const u64 wb = ceil_div(n_out, 256);
    auto take_whole = [&](u32 cnt) -> int {
        k_mw_whole<<<(unsigned)(wb < 4096 ? wb : 4096), 256, 0, st>>>(pl + p_whole, cnt, gsd, pl + lv[0].ps, kc,
                                                                      (u32)n_out, W);
        SS_CHECK_LAUNCH();
        return SS_OK;
    };
    if (!whole.empty()) SS_TRY(take_whole((u32)whole.size()));
    u32 ctr[C_NCTR];
    SS_TRY(ss_read_u32(sw.ctr, ctr, C_NCTR, st));
    if (ctr[C_BADSET]) {
        // runs that are not sorted: every group as one segment
        whole.clear();
        for (u32 g = 0; g < groups; g++)
            if (gs[g + 1] > gs[g]) whole.push_back(g);
        const UpPart parts[] = {{w.plan + p_whole, whole.data(), sizeof(u32) * whole.size()}};
        SS_TRY(upload_parts(parts, 1, st));
        k_fill_u32<<<1, 64, 0, st>>>(sw.ctr, 0u, C_NCTR);
        SS_CHECK_LAUNCH();
        SS_TRY(take_whole((u32)whole.size()));
        SS_TRY(ss_read_u32(sw.ctr, ctr, C_NCTR, st));
    }
    const u32 nover = ctr[C_RTILES], eover = ctr[C_NELEM];
    u32 nact = ctr[C_RNEXT];
    const bool small_only = !nover && !ctr[C_TIEBIG];  // then the first round is the last: its counters aren't read
    if (!nact && !nover) return SS_OK;
    const SortJob J{nullptr, 0, nullptr, w.order, out_lcp, st, n_out, n_out};
    // (lists of segments, in tiles of `per` members)
    auto tile_list = [&](const Seg *l, u32 cnt, u32 per, u64 *cmp, u32 *c) -> int {
        k_tie_tiles<<<(unsigned)ceil_div(cnt, 256), 256, 0, st>>>(l, cnt, per, w.tiles, cmp, c);
        SS_CHECK_LAUNCH();
        return ss_scan_exclusive<u32>(w.tiles, w.tiles, cnt, (u32 *)sw.scan_scratch, st);
    };
    if (nover) {
        // segments too large for a tile: sorted by key, their ties join the others
        SS_TRY(tile_list(w.over, nover, MW_OVER, nullptr, nullptr));
        const unsigned og = (unsigned)(nover + eover / MW_OVER);
        if (few) k_mw_over<MW_FEW><<<og, MW_NT, 0, st>>>(level(0), W, w.tiles, nover);
        else k_mw_over<MW_RUNS><<<og, MW_NT, 0, st>>>(level(0), W, w.tiles, nover);
        SS_CHECK_LAUNCH();
        k_fill_u32<<<1, 64, 0, st>>>(sw.ctr + C_NELEM, 0u, 1);
        SS_CHECK_LAUNCH();
        SS_TRY(sort_keyed(J, sw, ctr));
        if (ctr[C_NEXT])
            SS_HIP(hipMemcpyAsync(w.segs + nact, sw.nxt, sizeof(Seg) * ctr[C_NEXT], hipMemcpyDeviceToDevice, st));
        nact += ctr[C_NEXT];
    }
    // Tied keys.  Strings are compared without decoding them, along psv chains
    // over the whole front-coded array.  A comparison starts at byte C + 7 or
    // later of its group and a chain walk for byte i only at an entry with e >
    // i: none takes place, and no chains are built, unless adjacent strings of
    // a run share C + 7 bytes.
    if (nact) SS_TRY(psv_build(fc_lcp, n_fc, w.dec.psv, w.dec.tree, w.dec.cmin, w.dec.far, w.dec.fcnt, st, w.ties));
    auto tile_grid = [](u32 cnt, u32 el) { return (unsigned)ceil_div((u64)cnt + el / TIE_T, 32); };
    // rounds: the list's small segments end; its large ones go to `big` -- the
    // first round's stay there for the final emission -- and their ties, after
    // a sort by the next keys, make the next list
    const Seg *list = w.segs;
    u32 nbig0 = 0, ebig0 = 0;
    for (bool first = true; nact; first = false) {
        Seg *big = first ? w.big : w.segs;
        k_fill_u32<<<1, 64, 0, st>>>(sw.ctr, 0u, C_NCTR);
        SS_CHECK_LAUNCH();
        {
            SS_PROF("k_tie_small", st, (double)nact * 48.0);  // of two: entry, its LCP, length, offset; LCP out; not the bytes
            k_tie_small<<<(unsigned)ceil_div(nact, 32), 256, 0, st>>>(list, nact, V, w.order, sw.keyB, sw.mpr, O, big,
                                                                     sw.ctr);
        }
        SS_CHECK_LAUNCH();
        if (small_only) break;
        SS_TRY(ss_read_u32(sw.ctr, ctr, C_NCTR, st));
        const u32 nbig = ctr[C_RNEXT], ebig = ctr[C_RELEM];
        if (!nbig) break;
        if (first) {
            nbig0 = nbig;
            ebig0 = ebig;
        }
        SS_TRY(tile_list(big, nbig, TIE_T, sw.mword, sw.ctr));
        const unsigned tg = tile_grid(nbig, ebig);
        {
            SS_PROF("k_tie_compare", st, (double)ebig * 20.0);  // entry, its LCP, length, offset; not the bytes
            k_tie_compare<<<tg, 256, 0, st>>>(big, w.tiles, nbig, V, w.order, sw.mword);
        }
        SS_CHECK_LAUNCH();
        k_tie_keys<<<tg, 256, 0, st>>>(big, w.tiles, nbig, V, w.order, out_lcp, sw.mword, sw, z);
        SS_CHECK_LAUNCH();
        SS_TRY(sort_keyed(J, sw, ctr));
        nact = ctr[C_NEXT];
        Seg *tmp = sw.act; sw.act = sw.nxt; sw.nxt = tmp;
        list = sw.act;
    }
    if (nbig0) {
        SS_TRY(tile_list(w.big, nbig0, TIE_T, nullptr, nullptr));
        k_tie_emit<<<tile_grid(nbig0, ebig0), 256, 0, st>>>(w.big, w.tiles, nbig0, w.order, O);
        SS_CHECK_LAUNCH();
    }
    if (nover) {
        SS_TRY(tile_list(w.over, nover, TIE_T, nullptr, nullptr));
        k_tie_emit<<<tile_grid(nover, eover), 256, 0, st>>>(w.over, w.tiles, nover, w.order, O);
        SS_CHECK_LAUNCH();
    }
    return SS_OK;
}

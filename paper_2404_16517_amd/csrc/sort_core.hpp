// Segmented string sort machinery (workspace layout and the round driver).
#pragma once
#include "common.hpp"

// A contiguous range [begin, end) of sorted positions whose strings share a
// known prefix of `depth` bytes.  aux: bits 0..5 = leading key bits that earlier
// radix levels have used up, bit 6 = compute the common-prefix skip first, bit 7
// = the segment's keys and payload are in the B arrays (radix levels alternate
// between A and B; everything final is in A), bits 8..31 = the radix segment of
// the round it descends from (whose varying key bits are known; SEG_NOROOT: not).
struct Seg {
    u32 begin, end, depth, aux;
};
enum { SEG_SKIP = 64, SEG_INB = 128, SEG_ROOT = 8 };  // (SEG_ROOT: shift)
#define SEG_NOROOT 0xFFFFFF00u

// counters: list lengths, and the tile / element totals of the lists being
// built (so that grids are known without reading the lists back)
enum {
    C_SMALL = 0, C_LARGE = 1, C_NEXT = 2, C_IDENT = 3, C_BND = 4,
    C_LTILES = 5, C_SMALLN = 6, C_NTILES = 7, C_ITILES = 8, C_LELEM = 9, C_NELEM = 12, C_TINY = 13,
    C_TINYN = 14, C_BADSET = 15, C_MID = 16,
    C_RNEXT = 17, C_RTILES = 18, C_RELEM = 19,  // what k_resolve leaves of the C_NEXT segments
    C_TIEBIG = 20,  // (merge) some tied segment has more than TIE_SMALL members
    C_WG = 21,  // radix segments left to one workgroup each (device-driven sorts)
    C_NCTR = 22
};
// ctr[10..11]: 64-bit sum of size * skip over the routed segments

#define WS_MAX 128   // segments of up to this many strings: one wavefront each, in registers
#define BS_IPT 8     // elements per thread in the block sort
#define BS_SMALL 512  // ... segments of up to this many: one wavefront each
#define BS_MID 2048   // ... and up to this many: four wavefronts

__device__ __forceinline__ u32 seg_of_tile(const u32 *tstart, u32 nseg, u32 t)
{
    // largest s with tstart[s] <= t (tstart has nseg+1 entries, strictly
    // increasing).  Every segment has a tile, so s <= t, and all but
    // extra = tstart[nseg] - nseg segments have one, so s >= t - extra: with
    // many small segments (one tile each) the search is short.
    const u32 extra = tstart[nseg] - nseg;
    u32 lo = t > extra ? t - extra : 0u;
    u32 hi = (t < nseg - 1 ? t : nseg - 1) + 1;
    while (hi - lo > 1) {
        u32 mid = (lo + hi) >> 1;
        if (tstart[mid] <= t) lo = mid;
        else hi = mid;
    }
    return lo;
}

// Exclusive scan of the tile counts of nseg segments by one workgroup of
// LIST_NT threads (tstart[nseg] = total, which is returned).
#define LIST_NT 1024
#define LIST_ONE 4096  // lists of up to so many segments: one workgroup (three launches take longer)
__device__ __forceinline__ u32 list_tiles(const Seg *segs, u32 nseg, u32 tile, u32 *tstart)
{
    __shared__ u32 wsum[LIST_NT / 64];
    const u32 lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    u32 carry = 0;
    for (u32 b = 0; b < nseg; b += LIST_NT) {
        const u32 j = b + threadIdx.x;
        const u32 v = j < nseg ? (segs[j].end - segs[j].begin + tile - 1) / tile : 0u;
        u32 x = v;
#pragma unroll
        for (u32 o = 1; o < 64; o <<= 1) {
            const u32 y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63) wsum[wv] = x;
        __syncthreads();
        u32 tot = 0;
        x += carry - v;
#pragma unroll
        for (u32 w = 0; w < LIST_NT / 64; w++) {
            if (w < wv) x += wsum[w];
            tot += wsum[w];
        }
        if (j < nseg) tstart[j] = x;
        carry += tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) tstart[nseg] = carry;
    return carry;
}

// LDS slot of element i where threads own runs of 8 (a pad each: no bank conflicts)
__device__ __forceinline__ u32 bs_at(u32 i) { return i + i / BS_IPT; }

struct SortWs {
    u64 *keyA, *keyB, *mword;  // mword, mpr: each member's first mismatch with its segment's first string
    uint2 *mpr;
    u32 *valB, *lcp_scratch;
    Seg *act, *nxt, *tiny, *small, *mid, *ident, *largeA, *largeB, *wgl;
    uint2 *bnd;
    u32 *skipv;
    u64 *smin, *smax;
    u64 *rmask, *dig;  // per radix segment of a round its varying key bits; per radix segment its digit
    u64 *split;  // splitters of the segments that a level divides by them (see SPLIT_MIN)
    u8 *scat;
    u8 *kinds;  // per radix segment and digit: what the bucket became
    u32 *tstart, *hist;
    u64 *scan_scratch;
    u64 *dscan, *hscan;  // state of the device-length scans: of lists, of histograms
    u32 *ctr;
    u32 *hdr;    // list lengths of the current round and level (device)
};

struct SortJob {
    const u8 *bytes;
    u64 N;
    const u64 *off;
    u32 *vals;  // payload: input indices
    u32 *lcp;   // LCP output
    hipStream_t stream;
    u64 n_first;  // strings in the first round's segments (for byte accounting)
    u64 n_total;  // strings of the whole sort (bounds every list)
    // First-round seed (null: none): the mismatch records of the first
    // round's one segment, used in place of the workspace's when *seed_ok.
    u64 *seed_word;
    uint2 *seed_pos;
    const u32 *seed_ok;
};

void sort_ws_layout(u64 n, SortWs *w, WsArena *a, WsCounter *c);
// Host-driven rounds from nact segments in w.act covering `atiles` element
// tiles (of sort_shape's et; their count, tiles and strings also in the counters).
int sort_rounds(const SortJob &J, SortWs &w, u32 nact, u32 atiles, bool whole = false);
// Elements per workgroup of the element-wise kernels, tile of the radix passes
// and the size up to which segments are sorted in LDS, for a sort of n strings.
struct SortShape {
    u32 et, tile, block_max;
};
SortShape sort_shape(u64 n);
// The sorts of one round over segments whose 64-bit keys (in w.keyA) the caller
// computed and which it put into w.tiny, w.small, w.mid and w.largeA (counts
// and totals in the counters): each is sorted stably by key.  Runs of
// equal keys whose low byte is 8 are appended to w.nxt.  h receives the
// counters afterwards; J.lcp is written with values of no meaning.
int sort_keyed(const SortJob &J, SortWs &w, u32 *h);

// Segmented MSD radix string sort with LCP by-product (gfx950).
//
// Sorting the local string array is the first step of the paper's merge sort
// (Section 3, "Initialization"); the LCP array is its by-product.  This is a
// GPU-native design, not the paper's CPU algorithm:
//
//   * The sorted array is a set of contiguous SEGMENTS whose strings share a
//     known prefix of `depth` bytes.  Segment boundaries are final.
//   * Each ROUND takes the unresolved segments and
//       1. skips their common prefix: every string is compared with the
//          segment's first string from `depth` on and the minimum LCP is added
//          to `depth` (deep shared prefixes cost one read of D bytes, not one
//          radix pass per 7 bytes);
//       2. loads a 64-bit key per string: the next 7 bytes big-endian plus the
//          remaining length capped at 8, so that integer order is string order
//          over that window, end-of-string below every byte;
//       3. sorts each segment by (key, input index): segments larger than the
//          LDS cutover go through MSD radix levels over digits of their varying
//          key bits (histogram, global scan, stable scatter); segments of up to
//          128 strings are sorted by one wavefront each with a bitonic network
//          in registers; the others by one workgroup each with a merge sort in
//          LDS;
//       4. where neighbours' keys differ the LCP is final and is written; runs
//          of equal keys whose strings continue become next round's segments
//          at depth + 7; runs of equal keys whose strings end are equal
//          strings (LCP = length, order = input index).
#include <string.h>

#include "common.hpp"
#include <map>
#include <mutex>

#include "sort_core.hpp"

#define NT 256
#define ETILE 2048  // elements per workgroup in element-wise round kernels (fewer in small sorts)
#define RX_PF 8     // 256-element chunks a radix pass loads ahead

// Headers that the round and level kernels read their list lengths from
// (copied from the counters by k_round_begin / k_level_begin, so that the
// counters can be reset for the lists being built): hdr[H_ACT] active
// segments, hdr[H_LARGE] radix segments of the current level, hdr[H_HIST]
// their histogram length (256 per tile).
enum { H_ACT = 0, H_LARGE = 1, H_HIST = 2, H_REMAIN = 3, H_NHDR = 4 };
// ------------------------------------------------------------ wave helpers

// Wave-aggregated atomic add of per-lane values.
__device__ __forceinline__ void wave_add(u32 v, u32 *counter)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if (__lane_id() == 0 && v) atomicAdd(counter, v);
}

template <class T, int NTB = NT>
__device__ __forceinline__ T block_min(T v)
{
    __shared__ T red[NTB / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        T y = __shfl_xor(v, o, 64);
        v = y < v ? y : v;
    }
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    T r = red[0];
    for (int w = 1; w < NTB / 64; w++) r = red[w] < r ? red[w] : r;
    __syncthreads();
    return r;
}

template <class T>
__device__ __forceinline__ T block_max(T v)
{
    __shared__ T red[NT / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        T y = __shfl_xor(v, o, 64);
        v = y > v ? y : v;
    }
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    T r = red[0];
    for (int w = 1; w < NT / 64; w++) r = red[w] > r ? red[w] : r;
    __syncthreads();
    return r;
}

// ------------------------------------------------------------ tile lists

// Every kernel below reads the length of the list it works on from device
// memory and takes its items in a grid-stride loop, so one launch shape
// serves any length: the host either sizes the grid from counts it read back,
// or launches a fixed grid without reading anything back.

#define GSTRIDE(j, count) for (u32 j = blockIdx.x * blockDim.x + threadIdx.x; j < (count); j += gridDim.x * blockDim.x)

// Tile loop of the heavier kernels: with LOOP, a grid-stride loop over `count`
// tiles (fixed grids); without, exactly one tile per workgroup, t = blockIdx.x
// (grids sized from counts read back) -- the loop then runs once and compiles
// away, keeping the kernel's registers as they were.
#define TILE_LOOP(t, count) \
    for (u32 t = blockIdx.x; LOOP ? (t < (count)) : (t == blockIdx.x); t += LOOP ? gridDim.x : 1u)

// ---- radix digits
//
// A level's digit is made of the next W varying bits of the segment's keys, in
// up to three pieces of neighbouring bits (for letters: five bits of one byte and
// three of the next), or, where these would reach less far, of the next W bits
// whether they vary or not.  Bits that all keys of the round's segment share
// order nothing, so digits order like keys; and a level uses up at least W of
// the 64 bits, so there are at most 64 / W levels.  Which bits vary is found
// where the keys are made (k_keys); segments whose keys come from elsewhere
// take every bit as varying.  (Digits at byte boundaries have 26 values for
// letters: 100,000 D/N strings took two levels and 176 us, now one and 129; 16M
// in 16 sets three levels, now two.)
//
// Packed: piece q's shift in bits 10q..10q+5 and length in 10q+6..10q+9, then
// (30..36) the key bits used up after this level, then (37..42) its lowest bit.
template <u32 W>
struct Digits {
    static constexpr u32 NB = 1u << W;                 // buckets of a level
    static constexpr u32 LEVELS = (64 + W - 1) / W;    // most levels of one key
    static constexpr u32 DPT = NB / 256;               // digits per thread of a 256-thread workgroup
};

//
// narrow: no more bits than leave buckets of about NARROW_TO strings, if all bits
// vary freely (at least three).  Segments of some thousand strings then end as
// buckets of some hundred, which the block sort takes faster than the wave sort
// takes the fifty of a full digit, and the scatter writes longer runs.  Where
// the strings are skewed it can cost another level of launches, so only levels of
// NARROW_MIN strings and more do it: 16M D/N strings in 16 sets 5410 -> 5300 us,
// 512 sets 964 -> 924, but 200,000 text strings 589 -> 661, 1M D/N 264 -> 272.  Text
// strings without and with it: 1M 853 and 951, 2M 1044 and 1038, 2.5M 1169 and
// 1157, 3M 1240 and 1205, 6M 1844 and 1729; D/N strings: 2M 378 and 384, 3M 446
// and 431, 4M 566 and 541, 6M 712 and 710.
#define NARROW_TO 512
#define NARROW_MIN 2000000
__device__ __forceinline__ u64 digit_spec(const Seg &g, const u64 *rmask, u32 W, bool narrow)
{
    if (narrow) {
        const u32 b = 32 - (u32)__clz((int)((g.end - g.begin - 1) / NARROW_TO));
        W = b < 3 ? 3u : (b < W ? b : W);
    }
    const u32 used = g.aux & 63, root = g.aux >> SEG_ROOT;
    const u64 mask = (root == (SEG_NOROOT >> SEG_ROOT) ? ~0ull : rmask[root]) & (~0ull >> used);
    if (!mask) return 64ull << 30;  // (one key in the whole segment)
    const u32 top = 63 - (u32)__clzll(mask);
    u64 m = mask, spec = 0;
    u32 bits = 0, low = top + 1;
#pragma unroll
    for (u32 q = 0; q < 3; q++) {
        if (!m || bits == W) break;
        const u32 hi = 63 - (u32)__clzll(m);
        const u64 inv = ~(m << (63 - hi));
        const u32 ones = inv ? (u32)__clzll(inv) : 64u, take = ones < W - bits ? ones : W - bits;
        low = hi + 1 - take;
        spec |= (u64)(low | (take << 6)) << (10 * q);
        bits += take;
        m &= low ? ~0ull >> (64 - low) : 0ull;
    }
    u32 next = m ? 64 - (u32)__clzll(m) : 0u;  // bits [0, next) are left
    if (next && top + 1 - next < W) {
        low = top + 1 - W;  // (not below 0: bits below the pieces are left)
        if (top + 1 < W) low = 0;
        spec = (u64)(low | ((top + 1 - low) << 6));
        m = low ? mask & (~0ull >> (64 - low)) : 0ull;
        next = m ? 64 - (u32)__clzll(m) : 0u;
    }
    return spec | ((u64)(64 - next) << 30) | ((u64)low << 37);
}

struct Digit {
    u32 s[3], m[3], o[3];  // shift, mask, place in the digit
    u32 used, low;
};

__device__ __forceinline__ Digit digit_unpack(u64 spec)  // the same for the whole wavefront
{
    spec = ((u64)__builtin_amdgcn_readfirstlane((u32)(spec >> 32)) << 32) | (u32)__builtin_amdgcn_readfirstlane((u32)spec);
    Digit D;
    u32 at = 0;
#pragma unroll
    for (int q = 2; q >= 0; q--) {
        const u32 f = (u32)(spec >> (10 * q)) & 0x3FFu;
        D.s[q] = f & 63;
        D.m[q] = (1u << (f >> 6)) - 1u;
        D.o[q] = at;
        at += f >> 6;
    }
    D.used = (u32)(spec >> 30) & 127u;
    D.low = (u32)(spec >> 37) & 63u;
    return D;
}

__device__ __forceinline__ u32 digit_of(u64 k, const Digit &D)
{
    u32 d = 0;
#pragma unroll
    for (int q = 0; q < 3; q++) d |= ((u32)(k >> D.s[q]) & D.m[q]) << D.o[q];
    return d;
}

// ---- digits by splitters
//
// Where one workgroup takes what the levels over the whole device leave
// (k_radix_wg), these must leave no long segment, whatever its keys: bits would
// keep strings that share most of a key together (2M strings, 95 % of them
// sharing six bytes: 15.4 ms, with all levels over the device 1.4).  So segments
// of more than SPLIT_MIN strings with more than SPLIT_SKEW of a sample of 1024 in
// one digit of bits are divided by up to SPLITS of their own keys, every eighth of
// the sorted sample: digit 2 i + 1 is the i-th of them, 2 i what lies before it.
// A bucket between two then has a 50th of the segment or so, and one of a key is
// done.  (Without skew bits divide finer: 520,000 random strings 304 us, by
// splitters 434.)
#define SPLIT_MIN 131072
#define SPLITS 127  // (a table has one entry more)
#define SPLIT_SAMPLE 1024
#define SPLIT_SKEW 128
#define SPLIT_LIST 80  // segments of a level: sorts that get here hold at most 4097 times 2048 strings
#define SPLIT_FLAG (1ull << 63)  // in a segment's digit: by the splitters of this index

__device__ __forceinline__ u32 split_digit(const u64 *tab, u64 k)  // tab: ascending, past the last ~0
{
    u32 i = 0;
#pragma unroll
    for (u32 d = 64; d; d >>= 1) i += tab[i + d - 1] < k ? d : 0u;
    return 2 * i + (tab[i] == k ? 1u : 0u);
}

// Key k with its digit replaced by d.
__device__ __forceinline__ u64 digit_put(u64 k, u32 d, const Digit &D)
{
#pragma unroll
    for (int q = 0; q < 3; q++)
        k = (k & ~((u64)D.m[q] << D.s[q])) | ((u64)((d >> D.o[q]) & D.m[q]) << D.s[q]);
    return k;
}

// Whether segment [b, e) of keys is to be divided by splitters instead of the
// digit D, and if so these into tab; by a workgroup of SPLIT_SAMPLE.
__device__ __forceinline__ bool split_choose(const u64 *keys, u32 b, u32 e, const Digit &D, u64 *tab)
{
    __shared__ u64 sk[SPLIT_SAMPLE];
    __shared__ u32 s_kept[2], h[256];
    const u32 t = threadIdx.x, m = e - b, step = m / SPLIT_SAMPLE;
    if (t < 256) h[t] = 0;
    // (somewhere in the t-th part of the segment: inputs repeat at even distances)
    const u64 key = keys[b + (u32)((u64)m * t / SPLIT_SAMPLE) + ((t * 2654435761u) >> 8) % step];
    sk[t] = key;
    __syncthreads();
    atomicAdd(&h[digit_of(key, D)], 1u);
    __syncthreads();
    if (!__syncthreads_or(t < 256 && h[t] > SPLIT_SKEW)) return false;  // (its barrier: h is free again)
    for (u32 k = 2; k <= SPLIT_SAMPLE; k <<= 1)
        for (u32 j = k >> 1; j; j >>= 1) {
            __syncthreads();
            const u32 y = t ^ j;
            if (y > t) {
                const u64 x0 = sk[t], x1 = sk[y];
                if ((x0 > x1) == ((t & k) == 0)) {
                    sk[t] = x1;
                    sk[y] = x0;
                }
            }
        }
    __syncthreads();
    constexpr u32 EVERY = SPLIT_SAMPLE / (SPLITS + 1);
    const u64 mine = t < SPLITS ? sk[(t + 1) * EVERY] : ~0ull;
    const bool keep = t < SPLITS && (t == 0 || mine != sk[t * EVERY]);
    const u64 m64 = __ballot(keep);
    if (t < 128 && (t & 63) == 0) s_kept[t >> 6] = (u32)__popcll(m64);
    __syncthreads();
    if (t < 128) {
        if (keep) tab[(t >= 64 ? s_kept[0] : 0u) + (u32)__popcll(m64 & lanemask_lt())] = mine;
        if (t >= s_kept[0] + s_kept[1]) tab[t] = ~0ull;
    }
    __syncthreads();  // (the next segment)
    return true;
}

// k_tile_counts and its scan for up to LIST_ONE segments.
__global__ __launch_bounds__(LIST_NT) void k_list_tiles(const Seg *segs, const u32 *nsegp, u32 tile, u32 *tstart)
{
    list_tiles(segs, *nsegp, tile, tstart);
}

// k_round_begin, k_round_tiles and the scan for up to LIST_ONE segments.
__global__ __launch_bounds__(LIST_NT) void k_round_start(const Seg *segs, u32 *ctr, u32 *hdr, u32 from, u32 tile,
                                                         u32 *tstart, u32 *skipv, u64 *vary, u32 block_max)
{
    const u32 nseg = ctr[from];
    __syncthreads();
    if (threadIdx.x == 0) hdr[H_ACT] = nseg;
    if (threadIdx.x < C_NCTR && threadIdx.x != C_BADSET) ctr[threadIdx.x] = 0;
    for (u32 j = threadIdx.x; j < nseg; j += LIST_NT) {
        skipv[j] = 0xFFFFFFFFu;
        if (segs[j].end - segs[j].begin > block_max) vary[segs[j].begin] = 0;
    }
    list_tiles(segs, nseg, tile, tstart);
}

// k_level_begin, k_level_tiles and the scan for up to LIST_ONE segments: one
// launch, where four to six took longer than the level's work on small inputs
// (sorting 100,000 D/N strings, two levels: 218 us with them, 199 us so).
//
// WG: segments of up to wg_max strings are taken out and listed in wl (see
// k_radix_wg).
// Those of more than SPLIT_MIN whose keys are skewed get splitters.
template <bool WG>
__global__ __launch_bounds__(LIST_NT) void k_level_start(Seg *segs, u32 *ctr, u32 *hdr, u32 nb, u32 tile,
                                                         u32 *tstart, u64 *smin, u64 *smax, u64 *hscan,
                                                         const u64 *rmask, u64 *dig, bool narrow, Seg *wl,
                                                         u32 wg_max, const u64 *keyA, const u64 *keyB, u64 *split)
{
    u32 nseg = ctr[C_LARGE];
    scan_state_zero(hscan);
    __syncthreads();
    if (WG) {
        __shared__ u32 s_keep;
        if (threadIdx.x == 0) s_keep = 0;
        for (u32 b = 0; b < nseg; b += LIST_NT) {
            const u32 j = b + threadIdx.x;
            Seg x = {0, 0, 0, 0};
            if (j < nseg) x = segs[j];
            __syncthreads();  // (kept segments go to places already read)
            const bool keep = x.end - x.begin > wg_max;
            const u64 mk = __ballot(keep), ml = __ballot(j < nseg && !keep);
            u32 ak = 0, al = 0;
            if (__lane_id() == 0) {
                if (mk) ak = atomicAdd(&s_keep, (u32)__popcll(mk));
                if (ml) al = atomicAdd(&ctr[C_WG], (u32)__popcll(ml));
            }
            ak = __shfl(ak, 0, 64);
            al = __shfl(al, 0, 64);
            if (keep) segs[ak + (u32)__popcll(mk & lanemask_lt())] = x;
            else if (j < nseg) wl[al + (u32)__popcll(ml & lanemask_lt())] = x;
        }
        __syncthreads();
        nseg = s_keep;
    }
    __shared__ u32 s_nbig, s_big[SPLIT_LIST];  // segments to be divided by splitters
    if (WG && threadIdx.x == 0) s_nbig = 0;
    __syncthreads();
    for (u32 j = threadIdx.x; j < nseg; j += LIST_NT) {
        smin[j] = ~0ull;
        smax[j] = 0;
        if (WG && segs[j].end - segs[j].begin > SPLIT_MIN) {
            const u32 x = atomicAdd(&s_nbig, 1u);
            if (x < SPLIT_LIST) s_big[x] = j;
        }
        dig[j] = digit_spec(segs[j], rmask, (u32)__ffs((int)nb) - 1, narrow);
    }
    if (WG) {
        __syncthreads();
        static_assert(LIST_NT == SPLIT_SAMPLE, "a sample per thread");
        const u32 nbig = s_nbig < SPLIT_LIST ? s_nbig : SPLIT_LIST;
        for (u32 x = 0; x < nbig; x++) {  // (uniform)
            const u32 j = s_big[x];
            const Seg g = segs[j];
            const Digit D = digit_unpack(digit_spec(g, rmask, (u32)__ffs((int)nb) - 1, narrow));
            if (split_choose((g.aux & SEG_INB) ? keyB : keyA, g.begin, g.end, D, split + (SPLITS + 1) * x) &&
                threadIdx.x == 0)
                dig[j] = SPLIT_FLAG | x;
        }
    }
    const u32 tiles = list_tiles(segs, nseg, tile, tstart);
    if (threadIdx.x == 0) {
        hdr[H_LARGE] = nseg;
        hdr[H_HIST] = nb * tiles;
        ctr[C_LARGE] = 0;
        ctr[C_LTILES] = 0;
        ctr[C_LELEM] = 0;
    }
}

__global__ void k_tile_counts(const Seg *segs, const u32 *nsegp, u32 tile, u32 *out, u64 *dscan)
{
    const u32 nseg = *nsegp;
    if (blockIdx.x == 0) scan_state_zero(dscan);
    GSTRIDE(j, nseg) out[j] = (segs[j].end - segs[j].begin + tile - 1) / tile;
}

// Start of a round: the active list's length (counter `from`) goes to the
// header, the counters of the lists the round builds are reset.
__global__ void k_round_begin(u32 *ctr, u32 *hdr, u32 from)
{
    if (threadIdx.x == 0) hdr[H_ACT] = ctr[from];
    __syncthreads();
    if (threadIdx.x < C_NCTR && threadIdx.x != C_BADSET) ctr[threadIdx.x] = 0;
}

// Tile counts of the active segments for a round; also resets the segments'
// skip minima and, for those that may take radix levels, the varying bits of
// their keys (kept where the segment begins in the second key array).
__global__ void k_round_tiles(const Seg *segs, const u32 *nsegp, u32 tile, u32 *out, u32 *skipv, u64 *dscan,
                              u64 *vary, u32 block_max)
{
    const u32 nseg = *nsegp;
    if (blockIdx.x == 0) scan_state_zero(dscan);
    GSTRIDE(j, nseg) {
        out[j] = (segs[j].end - segs[j].begin + tile - 1) / tile;
        skipv[j] = 0xFFFFFFFFu;
        if (segs[j].end - segs[j].begin > block_max) vary[segs[j].begin] = 0;
    }
}

// Start of a radix level: the radix list's length and its histogram length
// go to the header, the counters of the next level's radix list are reset.
__global__ void k_level_begin(u32 *ctr, u32 *hdr, u32 nb, u64 *hscan)
{
    scan_state_zero(hscan);
    if (threadIdx.x == 0) {
        hdr[H_LARGE] = ctr[C_LARGE];
        hdr[H_HIST] = nb * ctr[C_LTILES];
        ctr[C_LARGE] = 0;
        ctr[C_LTILES] = 0;
        ctr[C_LELEM] = 0;
    }
}

// Tile counts of the radix segments of a level; also resets their key minima
// and maxima.
__global__ void k_level_tiles(const Seg *segs, const u32 *nsegp, u32 tile, u32 *out, u64 *smin, u64 *smax,
                              u64 *dscan, const u64 *rmask, u64 *dig, u32 W, bool narrow)
{
    const u32 nseg = *nsegp;
    if (blockIdx.x == 0) scan_state_zero(dscan);
    GSTRIDE(j, nseg) {
        out[j] = (segs[j].end - segs[j].begin + tile - 1) / tile;
        smin[j] = ~0ull;
        smax[j] = 0;
        dig[j] = digit_spec(segs[j], rmask, W, narrow);
    }
}

// ------------------------------------------------------------ round kernels

#define SKB 16      // strings per wavefront batch in the skip kernel
#define SKC_LONG 17  // 16-byte chunks per string of a long window (covers >= 257 bytes)
#define SKC_SHORT 5  // ... of a short window (covers >= 65 bytes)
#define SKR 5120     // LDS bytes per wavefront: five 1 KiB transfer rows
#define SKFS 256     // words (8 bytes) of the segment's first string staged in LDS

typedef __attribute__((address_space(3))) void lds_void;

// 8 bytes (little-endian) at any byte offset of LDS, from aligned words.
__device__ __forceinline__ u64 lds_le8(const u8 *R, u32 a)
{
    const u32 *p = (const u32 *)(R + (a & ~3u));
    const u32 r = a & 3u;
    u64 v = (u64)p[0] | ((u64)p[1] << 32);
    if (r) v = (v >> (8 * r)) | ((u64)p[2] << (64 - 8 * r));
    return v;
}

__device__ __forceinline__ u64 mask_le(u64 v, u32 take) { return take >= 8 ? v : (v & ((1ull << (8 * take)) - 1ull)); }

// Copy the window chunks of the batch's strings into the wavefront's LDS rows:
// chunk c of string s (16 bytes at the string's 16-aligned window start wa[s]
// plus 16c, relative to `bytes`) goes to R + 16 (CH s + c); wn[s] chunks are
// copied (0 for a window reaching outside the byte array, which is compared
// from global memory instead).
template <int CH>
__device__ __forceinline__ void skip_copy(const u8 *bytes, u8 *R, u32 lane, const u64 *wa, const u32 *wn)
{
    constexpr int T = (SKB * CH + 63) / 64;
    u64 ad[T];
    bool ok[T];
#pragma unroll
    for (int t = 0; t < T; t++) {  // every address first: the copies then issue back to back
        u32 slot = 64 * t + lane;
        asm volatile("" : "+v"(slot));  // recomputed per window rather than held in registers
        const u32 s = slot / CH, c = slot % CH;
        ad[t] = wa[s & 15] + 16u * c;
        ok[t] = s < SKB && c < wn[s & 15];
    }
#pragma unroll
    for (int t = 0; t < T; t++)
        if (ok[t]) __builtin_amdgcn_global_load_lds((const void *)(bytes + ad[t]), (lds_void *)(R + 1024 * t), 16, 0, 0);
}

// First mismatch of a member with the first string in [x, lim): each of the
// member's four lanes compares words q, q+4, q+8, ... (8 bytes each) of the
// window.  Returns the position (~0 if none) after a minimum over the four.
// Positions are string-relative (strings are shorter than 2^32 bytes).
template <int CH>
__device__ __forceinline__ u32 skip_cmp(const u8 *bytes, u64 N, const u8 *R, const u64 *fsw, u32 s, u32 q,
                                        u32 x, u32 lim, u32 sh, bool edge, u64 o, u64 fo, u32 depth)
{
    constexpr int WPL = (16 * CH + 31) / 32;  // words per lane
    const u32 rl = lim - x;                    // window bytes to compare (<= 16 CH)
    const u32 k0 = (x - depth) >> 3;           // first-string word of the window start
    const u32 rb = 16 * CH * s + sh;           // LDS offset of the window start
    u32 best = 0xFFFFFFFFu;
#pragma unroll 3
    for (int k = 0; k < WPL; k++) {
        const u32 w = q + 4 * k;
        const u32 rel = 8 * w;
        const u32 take = rel < rl ? ((rl - rel) < 8 ? rl - rel : 8u) : 0u;
        u64 wa = 0, wb = 0;
        if (take) {
            wa = edge ? load_le(bytes, N, o + x + rel, take) : mask_le(lds_le8(R, rb + rel), take);
            const u32 kw = k0 + w;
            wb = kw < SKFS ? mask_le(fsw[kw], take) : load_le(bytes, N, fo + x + rel, take);
        }
        const u64 d = wa ^ wb;
        const u32 mp = d ? rel + (u32)(__builtin_ctzll(d) >> 3) : 0xFFFFFFFFu;
        best = mp < best ? mp : best;
    }
#pragma unroll
    for (int o2 = 1; o2 < 4; o2 <<= 1) {
        const u32 y = __shfl_xor(best, o2, 64);
        best = y < best ? y : best;
    }
    return best == 0xFFFFFFFFu ? best : x + best;
}

// Minimum LCP of every member with the segment's first string, from `depth`.
// Each wavefront takes its members 16 at a time, four lanes per member: the
// window of every member (a short one of >= 65 bytes, or a long one of >= 257
// bytes once most members of the previous batch reached past 48 bytes) is
// copied from global memory into LDS by the transfer unit, then the four lanes
// compare it, 8 bytes at a time, against the first string's bytes
// [depth, depth + 2048) in LDS.  Members not resolved inside their window
// continue with the next one.  Before that, one lane per member, members are
// compared over 16 bytes as long as most of them differ there: only those that
// do not are taken by windows (512 sets of random strings: 473 -> 340 us).  Each
// member also leaves its first mismatch
// position, its remaining length there (capped at 8) and its 8 bytes there
// (mword, mpr), from which k_keys builds its key without reading the string
// again.
//
// SEED (the first round of a seeded sort, one segment from depth 0 in input
// order): when *seed_ok, mword and mpr arrive holding every member's record
// as far as an earlier pass over the first bytes found it; a member whose
// mpr.y is SEED_OPEN agreed with the first string up to mpr.x and is compared
// from there, every other one is done without reading its string.
#define SEED_OPEN 0xFFFFFFFFu
// (the grid-stride form keeps its loop state live as well: five workgroups
// per compute unit give it the registers to do so without spilling)
template <bool LOOP, bool SEED = false, int NTB = NT>
__global__ __launch_bounds__(NTB, (LOOP ? 5 : 6) * (NT / NTB)) void k_skip(const Seg *segs, const u32 *tstart, const u32 *nsegp, u32 et,
                                             const u8 *bytes, u64 N, const u64 *off,
                                             const u32 *perm, u32 *skipv, u64 *mword, uint2 *mpr,
                                             const u32 *seed_ok = nullptr)
{
    __shared__ u64 fsw[SKFS];
    __shared__ __attribute__((aligned(16))) u8 rows[(NTB / 64) * SKR];
    __shared__ u64 wwa[NTB / 64][SKB];  // per wavefront: window start of each member
    __shared__ u32 wwn[NTB / 64][SKB];  // ... and its chunk count
    __shared__ u64 lof[NTB / 64][64];   // per wavefront: the open members' offsets, lengths
    __shared__ u32 lln[NTB / 64][64];   // ... and which of the 64 they are
    __shared__ u8 lst[NTB / 64][64];
    const u32 nseg = *nsegp;
    const u32 ntiles = LOOP ? tstart[nseg] : 0u;
    const bool sok = SEED && *seed_ok != 0;  // uniform
    TILE_LOOP(t, ntiles) {  // (uniform over the workgroup)
    const u32 sg = seg_of_tile(tstart, nseg, t);
    const Seg g = segs[sg];
    if (!(g.aux & SEG_SKIP)) continue;  // uniform over the workgroup
    const u32 lt = t - tstart[sg];
    const u32 b0 = g.begin + lt * et;
    const u32 b1 = min(g.end, b0 + et);
    if (SEED && sok) {
        // the tile's records, one member per thread: when the seed resolved
        // every member, their minimum is the tile's part of the skip and no
        // string is read (a tile with an open member takes the loop below)
        u32 sb = 0xFFFFFFFFu;
        bool open = false;
#pragma unroll 8
        for (u32 k = 0; k < et / NTB; k++) {
            const u32 i = b0 + k * NTB + threadIdx.x;
            if (i < b1) {
                const uint2 sp = mpr[i];
                open |= sp.y == SEED_OPEN;
                const u32 c = sp.x > g.depth ? sp.x - g.depth : 0u;
                sb = c < sb ? c : sb;
            }
        }
        if (!__syncthreads_or(open)) {  // (uniform)
            const u32 bm = block_min<u32, NTB>(sb);
            if (threadIdx.x == 0) atomicMin(&skipv[sg], bm);
            continue;
        }
    }
    const u32 f = perm[g.begin];
    const u64 fo = off[f];
    const u32 fl = (u32)(off[f + 1] - fo);
    const u32 depth = g.depth;
    const u32 fd = fl > depth ? fl - depth : 0;  // first-string bytes from depth
    for (u32 q = threadIdx.x; q < SKFS; q += NTB) {
        const u32 k = 8 * q;
        fsw[q] = k < fd ? load_le(bytes, N, fo + depth + k, (fd - k) < 8 ? fd - k : 8u) : 0ull;
    }
    __syncthreads();
    const u32 lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const u32 sl = lane >> 2, q = lane & 3;  // this lane's member of the batch, its quarter
    u8 *R = rows + wv * SKR;
    const u64 babs = (u64)(uintptr_t)bytes;
    bool longw = false;  // window size of the next batch (uniform over the wavefront)
    u32 trial = !SEED && NTB > 64 ? SKB : 0u;  // members of the next 64 that are tried by 16 bytes first (likewise)
    u32 best = 0xFFFFFFFFu;
    for (u32 base = b0 + wv * 64; base < b1; base += NTB) {
        // one member per lane: what it is, and whether its bytes have to be compared from x
        const u32 i = base + lane;
        const bool valid = i < b1;
        u64 o = 0;
        u32 len = 0, m = 0, x = depth, res = 0xFFFFFFFFu;
        bool open = valid;
        if (SEED && sok && valid) {
            const uint2 sp = mpr[i];
            x = sp.x;
            if (sp.y != SEED_OPEN) {
                open = false;
                res = x;
            }
        }
        if (open) {
            const u32 p = perm[i];
            o = off[p];
            len = (u32)(off[p + 1] - o);
            m = len < fl ? len : fl;
            if (x >= m) {
                open = false;
                res = m;
                if (m <= depth) {  // nothing to compare: the member ends at or before depth
                    const u32 rem = len - m;
                    const u32 tk = rem < 8 ? rem : 8u;
                    mword[i] = load_be(bytes, N, o + m, tk);
                    mpr[i] = make_uint2(m, tk);
                }
            }
        }
        for (u32 from = 0; from < trial;) {
            if (open && lane >= from && lane < trial) {
                const u32 rem0 = len - depth;
                const Win16 c = win16_issue(bytes, N, o + depth, rem0 < 16 ? rem0 : 16u);
                u64 a0, a1;
                win16_finish(bytes, c, a0, a1);
                const u64 d0 = a0 ^ fsw[0], d1 = a1 ^ fsw[1];
                u32 r = d0 ? (u32)(__builtin_ctzll(d0) >> 3) : (d1 ? 8 + (u32)(__builtin_ctzll(d1) >> 3) : 16u);
                if (r < 16 || m - depth <= 16) {  // (zeros stand for bytes past an end)
                    r = r < m - depth ? r : m - depth;
                    const u32 rem = rem0 - r, tk = rem < 8 ? rem : 8u;
                    u64 mw;
                    if (r <= 8) mw = mask_le(r == 8 ? a1 : (r ? (a0 >> (8 * r)) | (a1 << (64 - 8 * r)) : a0), tk);
                    else mw = load_le(bytes, N, o + depth + r, tk);
                    mword[i] = __builtin_bswap64(mw);
                    mpr[i] = make_uint2(depth + r, tk);
                    res = depth + r;
                    open = false;
                }
            }
            // the tile's first try is of a few members; the rest follow if most of those are done
            if (trial != SKB || from || 2 * __popcll(__ballot(valid && !open && lane < SKB)) < SKB) break;
            from = SKB;
            trial = 64;
        }
        if (res != 0xFFFFFFFFu) {
            const u32 c = res > depth ? res - depth : 0u;
            best = c < best ? c : best;
        }
        const u64 U = __ballot(open);
        const u32 nu = (u32)__popcll(U);
        u32 near = (u32)__popcll(__ballot(valid)) - nu;  // members that differ within 16 bytes
        if (open) {
            const u32 at = (u32)__popcll(U & lanemask_lt());
            lof[wv][at] = o;
            lln[wv][at] = len;
            lst[wv][at] = (u8)lane;
        }
        for (u32 k = 0; k < nu; k += SKB) {  // 16 of the open ones, four lanes each
            const bool has = k + sl < nu;
            const u32 at = has ? k + sl : 0u, ib = base + lst[wv][at];
            const u64 ob = lof[wv][at];
            const u32 lenb = lln[wv][at], mb = lenb < fl ? lenb : fl;
            u32 xb = SEED && sok ? mpr[ib].x : depth + (lst[wv][at] < trial ? 16u : 0u), resb = mb;
            bool act = has;
            while (__ballot(act)) {  // uniform over the wavefront
                const u32 CH = longw ? SKC_LONG : SKC_SHORT;
                const u64 A0 = (babs + ob + xb) & ~15ull;
                const u32 sh = (u32)((babs + ob + xb) & 15);
                const u32 cov = 16 * CH - sh;                         // window bytes from xb
                const u32 wend = lenb - xb < cov ? lenb : xb + cov;   // copied: [xb, wend)
                const u32 lim = mb - xb < cov ? mb : xb + cov;        // compared: [xb, lim)
                const u32 nch = act ? (sh + (wend - xb) + 15) / 16 : 0u;
                // a window reaching outside the byte array is compared from global memory
                const bool edge = act && (A0 < babs || A0 + 16ull * nch > babs + N);
                if (q == 0) {  // (read back below by the same wavefront: LDS keeps its order)
                    wwa[wv][sl] = A0 - babs;
                    wwn[wv][sl] = edge ? 0u : nch;
                }
                u32 mis;
                if (longw) {
                    skip_copy<SKC_LONG>(bytes, R, lane, wwa[wv], wwn[wv]);
                    mis = skip_cmp<SKC_LONG>(bytes, N, R, fsw, sl, q, xb, act ? lim : xb, sh, edge, ob, fo, depth);
                } else {
                    skip_copy<SKC_SHORT>(bytes, R, lane, wwa[wv], wwn[wv]);
                    mis = skip_cmp<SKC_SHORT>(bytes, N, R, fsw, sl, q, xb, act ? lim : xb, sh, edge, ob, fo, depth);
                }
                if (act) {
                    u32 r = mis;
                    if (r == 0xFFFFFFFFu && lim >= mb) r = mb;
                    if (r != 0xFFFFFFFFu) {
                        // the member's 8 bytes at its mismatch, from the window when it holds them
                        const u32 rem = lenb - r;
                        const u32 tk = rem < 8 ? rem : 8u;
                        if (q == 0) {
                            u64 mw = 0;
                            if (tk)
                                mw = (!edge && r + tk <= wend) ? mask_le(lds_le8(R, 16 * CH * sl + sh + (r - xb)), tk)
                                                               : load_le(bytes, N, ob + r, tk);
                            mword[ib] = __builtin_bswap64(mw);
                            mpr[ib] = make_uint2(r, tk);
                        }
                        resb = r;
                        act = false;
                    } else {
                        xb += cov & ~7u;
                    }
                }
            }
            // most of the batch reaching past 48 bytes from depth: long windows next
            longw = __popcll(__ballot(has && q == 0 && resb >= depth + 48)) >= SKB / 2;
            near += (u32)__popcll(__ballot(has && q == 0 && resb < depth + 16));
            if (has && q == 0) best = resb - depth < best ? resb - depth : best;
        }
        trial = !SEED && NTB > 64 && near >= 32 ? 64u : 0u;
    }
    const u32 bm = block_min<u32, NTB>(best);  // (ends with a barrier: fsw and the rows are free again)
    if (threadIdx.x == 0) atomicMin(&skipv[sg], bm);
    }
}

template <bool LOOP, int NTB = NT>
__global__ __launch_bounds__(NTB) void k_keys(const Seg *segs, const u32 *tstart, const u32 *nsegp, u32 et,
                                             const u8 *bytes, u64 N, const u64 *off,
                                             const u32 *perm, const u32 *skipv, const u64 *mword,
                                             const uint2 *mpr, u64 *keys, u64 *vary, u32 block_max)
{
    __shared__ u64 fw;  // key of the segment's first string
    __shared__ u64 red[NTB / 64];
    const u32 nseg = *nsegp;
    const u32 ntiles = LOOP ? tstart[nseg] : 0u;
    TILE_LOOP(t, ntiles) {
    const u32 s = seg_of_tile(tstart, nseg, t);
    const Seg g = segs[s];
    const u32 lt = t - tstart[s];
    const u32 b0 = g.begin + lt * et;
    const u32 b1 = min(g.end, b0 + et);
    if (!(g.aux & SEG_SKIP)) {
        const u64 d = g.depth;
        for (u32 i = b0 + threadIdx.x; i < b1; i += NTB) {
            const u32 p = perm[i];
            const u64 o = off[p], l = off[p + 1] - o;
            keys[i] = make_key(bytes, N, o, l, d);
        }
        continue;  // (uniform over the workgroup)
    }
    // A member agrees with the segment's first string up to its mismatch
    // position pos >= d, so its key at d is the first string's bytes [d, pos)
    // followed by its own bytes from pos (mword).
    const u64 d = (u64)g.depth + skipv[s];
    if (threadIdx.x == 0) {
        const u32 f = perm[g.begin];
        const u64 fo = off[f], fl = off[f + 1] - fo;
        const u64 r = fl - d;  // the first string is a member: fl >= d
        fw = load_be(bytes, N, fo + d, r < 7 ? (u32)r : 7u) | (r < 8 ? r : 8ull);
    }
    __syncthreads();
    const bool radix = g.end - g.begin > block_max;  // (uniform) the bits where keys differ are wanted
    u64 diff = 0;
    for (u32 i = b0 + threadIdx.x; i < b1; i += NTB) {
        const uint2 pr = mpr[i];
        const u32 k = pr.x - (u32)d;  // bytes shared with the first string beyond d
        u64 data = fw;
        if (k < 7) {
            const u64 keep = k ? (~0ull << (64 - 8 * k)) : 0ull;
            data = (fw & keep) | (mword[i] >> (8 * k));
        }
        const u32 cnt = pr.y + k < 8 ? pr.y + k : 8u;
        const u64 key = (data & ~0xFFull) | cnt;
        keys[i] = key;
        diff |= key ^ fw;
    }
    if (radix) {
        u32 lo = (u32)diff, hi = (u32)(diff >> 32);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            lo |= __shfl_xor(lo, o, 64);
            hi |= __shfl_xor(hi, o, 64);
        }
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ((u64)hi << 32) | lo;
    }
    __syncthreads();  // (also: fw is rewritten by the next tile)
    if (radix && threadIdx.x == 0) {
        u64 v = red[0];
        for (int w = 1; w < NTB / 64; w++) v |= red[w];
        if (v) atomicOr((unsigned long long *)&vary[g.begin], (unsigned long long)v);
    }
    }
}

// Apply the skip, route each active segment to the LDS list or the radix list.
// The lists' lengths and totals are counted in LDS and added by one atomic per
// counter and 256 segments: one per wavefront made 446K small segments queue
// on the few counters for 246 us; 11K of them now take 5 us.
__global__ __launch_bounds__(256) void k_classify(const Seg *act, const u32 *nactp, const u32 *skipv, u32 small_max,
                                                  u32 tile, Seg *tiny, Seg *small, Seg *mid, Seg *large,
                                                  u32 *ctr, const u64 *vary, u64 *rmask)
{
    enum { TY = 0, SM, MD, LG, TYN, SMN, LGT, LGN, CNT };  // list lengths, then their totals
    __shared__ u32 c[CNT], base[4];
    __shared__ u64 sk;  // sum of size * skip
    const u32 nact = *nactp;
    for (u32 j0 = blockIdx.x * blockDim.x; j0 < nact; j0 += gridDim.x * blockDim.x) {
    if (threadIdx.x < CNT) c[threadIdx.x] = 0;
    if (threadIdx.x == CNT) sk = 0;
    __syncthreads();
    const u32 j = j0 + threadIdx.x;
    const bool valid = j < nact;
    Seg g = {0, 0, 0, 0};
    u64 skn = 0;
    bool root = false;  // the varying bits of its keys are known
    if (valid) {
        g = act[j];
        if (g.aux & SEG_SKIP) {
            g.depth += skipv[j];
            skn = (u64)(g.end - g.begin) * skipv[j];
        }
        root = g.aux & SEG_SKIP;
        g.aux = 0;
    }
    const u32 sz = g.end - g.begin;
    const u32 kind = !valid ? (u32)CNT : (sz <= WS_MAX ? (u32)TY : (sz > small_max ? (u32)LG : (sz <= BS_SMALL ? (u32)SM : (u32)MD)));
    u32 slot = 0;
#pragma unroll
    for (u32 k = 0; k < 4; k++) {
        const u64 m = __ballot(kind == k);
        if (!m) continue;  // (uniform over the wavefront)
        u32 v = kind == k ? sz : 0u, t = kind == k ? (sz + tile - 1) / tile : 0u, at = 0;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            v += __shfl_xor(v, o, 64);
            if (k == LG) t += __shfl_xor(t, o, 64);
        }
        if (__lane_id() == 0) {
            at = atomicAdd(&c[k], (u32)__popcll(m));
            atomicAdd(&c[k == TY ? TYN : (k == LG ? LGN : SMN)], v);
            if (k == LG) atomicAdd(&c[LGT], t);
        }
        at = __shfl(at, 0, 64);
        if (kind == k) slot = at + (u32)__popcll(m & lanemask_lt());
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) skn += __shfl_xor(skn, o, 64);
    if (__lane_id() == 0 && skn) atomicAdd((unsigned long long *)&sk, (unsigned long long)skn);
    __syncthreads();
    if (threadIdx.x < CNT && c[threadIdx.x]) {
        const u32 to[CNT] = {C_TINY, C_SMALL, C_MID, C_LARGE, C_TINYN, C_SMALLN, C_LTILES, C_LELEM};
        u32 w = 0;
#pragma unroll
        for (u32 q = 0; q < CNT; q++)
            if (threadIdx.x == q) w = to[q];
        const u32 at = atomicAdd(&ctr[w], c[threadIdx.x]);
        if (threadIdx.x < 4) base[threadIdx.x] = at;
    }
    if (threadIdx.x == CNT && sk) atomicAdd((unsigned long long *)&ctr[10], (unsigned long long)sk);
    __syncthreads();
    if (kind == TY) tiny[base[TY] + slot] = g;
    else if (kind == SM) small[base[SM] + slot] = g;
    else if (kind == MD) mid[base[MD] + slot] = g;
    else if (kind == LG) {
        const u32 at = base[LG] + slot;
        g.aux = root ? at << SEG_ROOT : SEG_NOROOT;
        large[at] = g;
        rmask[at] = vary[g.begin];
    }
    __syncthreads();  // the counters are reset for the next segments
    }
}

#define RS_BUF 256    // runs a workgroup collects before it updates the counters
#define RS_MAX 16     // runs of up to this many tied strings are compared directly
#define RS_CMP 1024   // ... over this many bytes past their common prefix

// Runs of tied strings that a round hands to the next, most of them two or
// three equal strings: eight lanes per run compare every member with the
// first, 64 bytes a step.  Equal strings end here (LCP = length; they are in
// input order already), two unequal ones too; a longer run with unequal
// members goes on from its exact common prefix (no skip needed), and runs too
// long or tied for too long go on as they are.  `in` (count *nin) to `out`,
// whose counters (C_NEXT, C_NTILES, C_NELEM) are zero before.
//
// Bounded by the latency of scattered reads: two lines per string.  A round's
// skip, keys, routing and sort took 1.1 ms for 446K such runs (4M text
// strings); this takes 199 us (227 with three updates of the counters per 32 runs:
// they queue where the chip's L2s meet).
__global__ __launch_bounds__(256) void k_resolve(const Seg *in, const u8 *bytes, u64 N, const u64 *off,
                                                 u32 *vals, u32 *lcp, Seg *out, u32 *ctr, u32 et)
{
    __shared__ Seg buf[RS_BUF];  // what goes on, until it is worth an update of the counters
    __shared__ u32 s_cnt, s_tiles, s_elems, s_base;
    const u32 nin = ctr[C_NEXT];
    u32 held = 0;  // entries of buf: counted by the barrier itself, so that every thread decides alike
    auto flush = [&]() {  // (by the whole workgroup, after a barrier)
        if (threadIdx.x == 0) {
            s_base = atomicAdd(&ctr[C_RNEXT], held);
            static_assert(C_RTILES % 2 == 0 && C_RELEM == C_RTILES + 1, "both counters in one 8-byte word");
            atomicAdd((unsigned long long *)&ctr[C_RTILES], ((unsigned long long)s_elems << 32) | s_tiles);
        }
        __syncthreads();
        for (u32 k = threadIdx.x; k < held; k += 256) out[s_base + k] = buf[k];
        __syncthreads();
        if (threadIdx.x == 0) s_cnt = s_tiles = s_elems = 0;
        __syncthreads();
        held = 0;
    };
    if (threadIdx.x == 0) s_cnt = s_tiles = s_elems = 0;
    __syncthreads();
    for (u32 s0 = blockIdx.x * 32; s0 < nin; s0 += gridDim.x * 32) {  // (uniform over the workgroup)
    const u32 s = s0 + (threadIdx.x >> 3), gl = threadIdx.x & 7;
    bool keep = false;
    Seg g = {0, 0, 0, 0};
    if (s < nin) {
        g = in[s];
        const u32 m = g.end - g.begin;
        if (m > RS_MAX) {
            keep = true;
        } else {
            // every member's index, offset and length first, two per lane
            u32 pm[2], lm[2];
            u64 om[2];
#pragma unroll
            for (int h = 0; h < 2; h++) {
                const u32 j = gl + 8 * h;
                pm[h] = j < m ? vals[g.begin + j] : 0u;
            }
#pragma unroll
            for (int h = 0; h < 2; h++) {
                om[h] = off[pm[h]];
                lm[h] = (u32)(off[pm[h] + 1] - om[h]);
            }
            const u32 p0 = __shfl(pm[0], 0, 8), l0 = __shfl(lm[0], 0, 8);
            const u64 o0 = __shfl(om[0], 0, 8);
            bool same = true, open = false;
            u32 dmin = 0xFFFFFFFFu;
            u64 oj = 0;
            u32 pj = 0, lj = 0;
            for (u32 j = 1; j < m && !open; j++) {  // (the same for the run's eight lanes)
                pj = __shfl(j < 8 ? pm[0] : pm[1], j & 7, 8);
                oj = __shfl(j < 8 ? om[0] : om[1], j & 7, 8);
                lj = __shfl(j < 8 ? lm[0] : lm[1], j & 7, 8);
                const u32 lim = l0 < lj ? l0 : lj;
                u32 pos = g.depth, mis = 0xFFFFFFFFu;
                while (pos < lim && mis == 0xFFFFFFFFu && pos - g.depth < RS_CMP) {
                    const u32 q = pos + 8 * gl;
                    const u32 take = q < lim ? (lim - q < 8 ? lim - q : 8u) : 0u;
                    const Raw8 ra = raw8_issue(bytes, N, o0 + q, take), rb = raw8_issue(bytes, N, oj + q, take);
                    const u64 d = raw8_le(bytes, ra) ^ raw8_le(bytes, rb);
                    u32 f = d ? q + (u32)(__builtin_ctzll(d) >> 3) : 0xFFFFFFFFu;
#pragma unroll
                    for (int x = 1; x < 8; x <<= 1) {
                        const u32 y = __shfl_xor(f, x, 8);
                        f = y < f ? y : f;
                    }
                    mis = f;
                    pos += 64;
                }
                open = mis == 0xFFFFFFFFu && pos < lim;
                const u32 l = mis == 0xFFFFFFFFu ? lim : mis;
                same = same && mis == 0xFFFFFFFFu && l0 == lj;
                dmin = l < dmin ? l : dmin;
            }
            if (open) {
                keep = true;
            } else if (same) {
                for (u32 j = 1 + gl; j < m; j += 8) lcp[g.begin + j] = l0;
            } else if (m == 2) {
                if (gl == 0) {
                    lcp[g.begin + 1] = dmin;
                    const bool first = dmin == l0 || (dmin < lj && bytes[o0 + dmin] < bytes[oj + dmin]);
                    if (!first) {
                        vals[g.begin] = pj;
                        vals[g.begin + 1] = p0;
                    }
                }
            } else {
                keep = true;
                g.depth = dmin;
                g.aux = 0;
            }
        }
    }
    if (keep && gl == 0) {
        buf[atomicAdd(&s_cnt, 1u)] = g;
        atomicAdd(&s_tiles, (g.end - g.begin + et - 1) / et);
        atomicAdd(&s_elems, g.end - g.begin);
    }
    // (s_cnt itself may not be read for this: a wavefront that is ahead adds to it
    // again before a late one has read it, and only some would enter the flush)
    held += (u32)__syncthreads_count(keep && gl == 0);
    if (held > RS_BUF - 32) flush();
    }
    if (held) flush();
}

// ------------------------------------------------------------ radix passes
//
// A radix level sorts a segment by one digit of the 64-bit key, W = 8 or 11 bits
// wide: which bits, the segment's keys decide (Digits, above), so a key takes at
// most eight or six levels and mostly one to three.  The histograms have 2^W
// buckets.

// Lanes of this wave holding the same W-bit digit (restricted to `valid`).
template <u32 W>
__device__ __forceinline__ u64 match_digit_w(u32 digit, bool valid)
{
    u64 m = __ballot(valid);
#pragma unroll
    for (int b = 0; b < (int)W; b++) {
        u64 bb = __ballot((digit >> b) & 1);
        m &= ((digit >> b) & 1) ? bb : ~bb;
    }
    return m;
}

// A level's digit of a segment, by bits or (SP: where segments may have them) by
// splitters, which are read into LDS.  set() is called by the whole workgroup,
// after a barrier that ends the use of the last; the digit is used after another.
template <bool SP>
struct LevelDigit {
    Digit D;
    const u64 *tab;
    bool by;
    __device__ __forceinline__ void set(u64 spec, const u64 *split)
    {
        D = digit_unpack(spec);
        by = SP && (spec & SPLIT_FLAG);
        if (SP && by) {
            __shared__ u64 lds[SPLITS + 1];
            tab = lds;
            const u64 *src = split + (SPLITS + 1) * (u64)(u32)spec;
            for (u32 i = threadIdx.x; i < SPLITS + 1; i += blockDim.x) lds[i] = src[i];
        }
    }
    __device__ __forceinline__ u32 operator()(u64 k) const { return SP && by ? split_digit(tab, k) : digit_of(k, D); }
};

// Per-tile histogram of the segment's current digit, digit-major per
// segment: hist[NB*tstart[s] + d*T_s + lt].  Also the segment's min and max key.
//
// Bounded by its 8 B per key (27 us for 16M) and the vector unit.  One LDS add
// per key, whatever the digits: finding the lanes that share a digit first, to
// add once for all of them, costs more than even 64 adds on one word (16M keys
// in 16 segments 54 us a level, now 41).
template <bool LOOP, u32 W>
__global__ __launch_bounds__(NT) void k_hist(const Seg *segs, const u32 *tstart, const u32 *nsegp, u32 tile,
                                             const u64 *keyA, const u64 *keyB, u32 *hist, u64 *smin, u64 *smax,
                                             const u64 *dig, const u64 *split)
{
    constexpr u32 NB = Digits<W>::NB;
    __shared__ u32 h[NB];
    LevelDigit<LOOP && W == 8> digit;
    const u32 nseg = *nsegp;
    const u32 ntiles = LOOP ? tstart[nseg] : 0u;
    TILE_LOOP(t, ntiles) {
    const u32 s = seg_of_tile(tstart, nseg, t);
    const Seg g = segs[s];
    const u64 *keys = (g.aux & SEG_INB) ? keyB : keyA;
    const u32 T = tstart[s + 1] - tstart[s];
    const u32 lt = t - tstart[s];
    digit.set(dig[s], split);
    const u32 b0 = g.begin + lt * tile;
    const u32 b1 = min(g.end, b0 + tile);
    for (u32 d = threadIdx.x; d < NB; d += NT) h[d] = 0;
    __syncthreads();
    u64 mn = ~0ull, mx = 0;
    for (u32 c0 = b0; c0 < b1; c0 += RX_PF * NT) {
        // RX_PF chunks' keys loaded before any is counted
        u64 kq[RX_PF];
#pragma unroll
        for (u32 q = 0; q < RX_PF; q++) {
            const u32 i = c0 + q * NT + threadIdx.x;
            kq[q] = i < b1 ? keys[i] : 0;
        }
#pragma unroll
        for (u32 q = 0; q < RX_PF; q++) {
            const u32 c = c0 + q * NT;
            if (c >= b1) break;  // (uniform)
            const bool valid = c + threadIdx.x < b1;
            const u64 k = kq[q];
            if (valid) {
                mn = k < mn ? k : mn;
                mx = k > mx ? k : mx;
                atomicAdd(&h[digit(k)], 1u);
            }
        }
    }
    __syncthreads();
    for (u32 d = threadIdx.x; d < NB; d += NT) hist[NB * tstart[s] + d * T + lt] = h[d];
    mn = block_min(mn);
    mx = block_max(mx);  // (ends with a barrier: h is free again)
    if (threadIdx.x == 0) {
        atomicMin((unsigned long long *)&smin[s], (unsigned long long)mn);
        atomicMax((unsigned long long *)&smax[s], (unsigned long long)mx);
    }
    }
}

struct EmitOut {
    Seg *tiny, *small, *mid, *large_next, *next, *ident;
    uint2 *bnd;
    u32 *ctr;
    u8 *scat;
    u8 *kinds;
    u32 small_max;
    u32 tile;
    u32 et;
};

enum { K_NONE = 0, K_SMALL, K_LARGE, K_NEXT, K_IDENT, K_TINY, K_MID, K_KINDS };

// What digit d of radix segment s becomes: an entry for one of the lists
// (kind, seg) and/or a bucket boundary (sb, depth) for the LCP pass.
struct EmitItem {
    u32 kind;
    Seg ns;
    bool bnd;
    uint2 bv;
};

// ... once the segment is known not to share the whole digit (start: members in
// lower buckets; used: the key bits that all its members share; c8: the keys' last
// byte, if that is all 64).
__device__ __forceinline__ EmitItem emit_bucket(const Seg &g, u32 used, u32 c8, u32 start, u32 cnt, u32 small_max)
{
    EmitItem it{K_NONE, Seg{0, 0, 0, 0}, false, make_uint2(0, 0)};
    const u32 cf = (g.aux & SEG_INB) ? 0u : (u32)SEG_INB;  // the scatter writes the other arrays
    const u32 sb = g.begin + start, se = sb + cnt;
    it.bnd = cnt > 0 && start > 0;
    it.bv = make_uint2(sb, g.depth);
    it.ns = Seg{sb, se, g.depth, cf};
    if (cnt >= 2) {
        if (used == 64) {
            // no varying bit is left: the bucket's keys are equal in all 64
            // bits, and their last byte counts the strings' bytes
            if (c8 == 8) { it.kind = K_NEXT; it.ns = Seg{sb, se, g.depth + 7, SEG_SKIP}; }
            else { it.kind = K_IDENT; it.ns = Seg{sb, se, g.depth + c8, 0}; }
        } else if (cnt <= WS_MAX) {
            it.kind = K_TINY;
        } else if (cnt <= small_max) {
            it.kind = cnt <= BS_SMALL ? K_SMALL : K_MID;
        } else {
            it.kind = K_LARGE;
            it.ns.aux = used | cf | (g.aux & SEG_NOROOT);
        }
    }
    return it;
}

// A segment of one key (all 8 bytes): it continues in the next round, or its
// strings are equal.
__device__ __forceinline__ EmitItem emit_whole(const Seg &g, u64 key)
{
    const u32 cnt = (u32)(key & 0xFF);
    if (cnt == 8) return EmitItem{K_NEXT, Seg{g.begin, g.end, g.depth + 7, SEG_SKIP}, false, make_uint2(0, 0)};
    return EmitItem{K_IDENT, Seg{g.begin, g.end, g.depth + cnt, 0}, false, make_uint2(0, 0)};
}

template <u32 W>
__device__ __forceinline__ EmitItem emit_item(const Seg *segs, const u32 *tstart, const u32 *hist, const u64 *smin,
                                              const u64 *smax, const u64 *dig, const u64 *split, const EmitOut &o,
                                              u32 s, u32 d, bool *scat)
{
    constexpr u32 NB = Digits<W>::NB;
    EmitItem it{K_NONE, Seg{0, 0, 0, 0}, false, make_uint2(0, 0)};
    const Seg g = segs[s];
    const u64 spec = dig[s];
    const Digit D = digit_unpack(spec);
    const bool by = spec & SPLIT_FLAG;
    const u32 rt = g.aux & SEG_NOROOT;
    const u32 pf = g.aux & SEG_INB;  // where the segment's data is now
    const u64 mn = smin[s], mx = smax[s];
    // next-round and equal-string runs (and singletons) end in A: the settle
    // pass copies them there; the other kinds carry their buffer flag
    if (mn == mx) {
        *scat = false;
        return d == 0 ? emit_whole(g, mn) : it;
    }
    const u32 fd = (u32)__clzll(mn ^ mx);  // leading bits that all keys share
    if (!by && fd > 63 - D.low) {
        // the whole digit is common to the segment: no scatter needed
        *scat = false;
        if (d == 0) { it.kind = K_LARGE; it.ns = Seg{g.begin, g.end, g.depth, fd | pf | rt}; }
        return it;
    }
    *scat = true;
    const u32 ts = tstart[s];
    const u32 T = tstart[s + 1] - ts;
    const u32 e = NB * ts + d * T;
    const u32 base = hist[NB * ts];
    u32 used = D.used, c8 = (u32)digit_put(mn, d, D) & 0xFFu;
    if (by) {
        used = d & 1 ? 64u : g.aux & 63u;
        c8 = d & 1 ? (u32)split[(SPLITS + 1) * (u64)(u32)spec + (d >> 1)] & 0xFFu : 0u;
    }
    return emit_bucket(g, used, c8, hist[e] - base, hist[e + T] - hist[e], o.small_max);
}

// Segments per workgroup in k_emit: two of 256 digits (an item per thread and
// segment), or one of 2048.  Eight made fewer global atomics, but a chain of
// scattered reads per thread and too few workgroups (suffix sorting of 8 MB
// 2068 us, with two 2000, with one 2018).
template <u32 W>
struct EmitShape {
    static constexpr u32 SPG = Digits<W>::DPT == 1 ? 2 : 1;
    static constexpr u32 EPB = SPG * Digits<W>::DPT;  // items per thread
};

// The items of a workgroup into their lists: counted in LDS, one global atomic
// per list, then written.  Before it, emit_zero; it ends with a barrier.
struct EmitLds {
    u32 count[K_KINDS], slot[K_KINDS], sum[7], base[K_KINDS];
};

__device__ __forceinline__ void emit_zero(EmitLds &L)
{
    if (threadIdx.x < K_KINDS) { L.count[threadIdx.x] = 0; L.slot[threadIdx.x] = 0; }
    if (threadIdx.x < 7) L.sum[threadIdx.x] = 0;
}

template <u32 EPB>
__device__ __forceinline__ void emit_push(const EmitItem (&it)[EPB], const EmitOut &o, EmitLds &L)
{
    const u32 tx = threadIdx.x;
    __syncthreads();
#pragma unroll
    for (u32 q = 0; q < EPB; q++) {
        const EmitItem &x = it[q];
        const u32 cnt = x.ns.end - x.ns.begin;
        if (x.bnd) atomicAdd(&L.count[0], 1u);
        if (x.kind) atomicAdd(&L.count[x.kind], 1u);
        if (x.kind == K_SMALL || x.kind == K_MID) atomicAdd(&L.sum[0], cnt);
        if (x.kind == K_LARGE) { atomicAdd(&L.sum[1], (cnt + o.tile - 1) / o.tile); atomicAdd(&L.sum[2], cnt); }
        if (x.kind == K_NEXT) { atomicAdd(&L.sum[3], (cnt + o.et - 1) / o.et); atomicAdd(&L.sum[4], cnt); }
        if (x.kind == K_IDENT) atomicAdd(&L.sum[5], (cnt + o.et - 1) / o.et);
        if (x.kind == K_TINY) atomicAdd(&L.sum[6], cnt);
    }
    __syncthreads();
    // (a thread per counter: one after the other they took most of the kernel on
    // small inputs)
    static_assert(K_KINDS == 7, "counters of the lists");
    if (tx < 14) {
        u32 to = C_BND;
        to = tx == K_SMALL ? (u32)C_SMALL : tx == K_LARGE ? (u32)C_LARGE : tx == K_NEXT ? (u32)C_NEXT : to;
        to = tx == K_IDENT ? (u32)C_IDENT : tx == K_TINY ? (u32)C_TINY : tx == K_MID ? (u32)C_MID : to;
        to = tx == 7 ? (u32)C_SMALLN : tx == 8 ? (u32)C_LTILES : tx == 9 ? (u32)C_LELEM : to;
        to = tx == 10 ? (u32)C_NTILES : tx == 11 ? (u32)C_NELEM : tx == 12 ? (u32)C_ITILES : tx == 13 ? (u32)C_TINYN : to;
        const u32 v = tx < 7 ? L.count[tx] : L.sum[tx - 7];
        if (v) {
            const u32 at = atomicAdd(&o.ctr[to], v);
            if (tx < 7) L.base[tx] = at;
        }
    }
    __syncthreads();
#pragma unroll
    for (u32 q = 0; q < EPB; q++) {
        const EmitItem &x = it[q];
        if (x.bnd) o.bnd[L.base[0] + atomicAdd(&L.slot[0], 1u)] = x.bv;
        if (x.kind) {
            const u32 a = L.base[x.kind] + atomicAdd(&L.slot[x.kind], 1u);
            Seg *dst = x.kind == K_TINY ? o.tiny : x.kind == K_SMALL ? o.small : x.kind == K_MID ? o.mid
                     : x.kind == K_LARGE ? o.large_next : x.kind == K_NEXT ? o.next : o.ident;
            dst[a] = x.ns;
        }
    }
    __syncthreads();  // the LDS counters are reset for the next group
}

// Digit counts from the scanned histogram and emission of the sub-segments.
// A workgroup takes SPG segments (thread x = digits x + 256 r, r < DPT).
template <bool LOOP, u32 W>
__global__ __launch_bounds__(256) void k_emit(const Seg *segs, const u32 *tstart, const u32 *nsegp,
                                              const u32 *hist, const u64 *smin, const u64 *smax,
                                              const u64 *dig, const u64 *split, EmitOut o)
{
    constexpr u32 NB = Digits<W>::NB, DPT = Digits<W>::DPT, SPG = EmitShape<W>::SPG, EPB = EmitShape<W>::EPB;
    __shared__ EmitLds L;
    const u32 nseg = *nsegp;
    const u32 ngrp = LOOP ? (nseg + SPG - 1) / SPG : 0u;
    TILE_LOOP(grp, ngrp) {
    emit_zero(L);
    EmitItem it[EPB];
#pragma unroll
    for (u32 q = 0; q < EPB; q++) {
        const u32 s = grp * SPG + q / DPT;
        const u32 d = threadIdx.x + 256u * (q % DPT);
        it[q].kind = K_NONE;
        it[q].bnd = false;
        if (s >= nseg) continue;
        bool sc = false;
        it[q] = emit_item<W>(segs, tstart, hist, smin, smax, dig, split, o, s, d, &sc);
        if (d == 0) o.scat[s] = sc ? 1 : 0;
        o.kinds[NB * s + d] = (u8)it[q].kind;
    }
    emit_push(it, o, L);
    }
}

// Stable scatter of (key, payload) by the current digit into the other pair
// of arrays (A -> B or B -> A, by the segment's flag), SC_ITEMS elements at a
// time: every wavefront ranks its 512 by digit (the first lane of each digit
// counts all its peers, and the steps' counts follow one another without a
// barrier, as LDS serves a wavefront in order), one scan over digits and
// wavefronts gives each element its place in the chunk sorted by digit, the
// chunk is put in that order in LDS and written from there, so that neighbouring
// lanes write neighbouring elements of a bucket.
//
// Bounded by its 24 B per element (81 us for 16M at the copy's rate).  16M keys
// in 16 segments, about 200 buckets each: 222 us a level when every thread wrote
// its element where it belongs and the wavefronts took turns at each 256, now
// 103; 26 buckets took 112 then.  1024 elements a chunk: 4 % longer sorts.
#define SC_PER 8  // elements per thread and chunk
template <u32 W, u32 NTB = NT>
struct ScatterLds {
    static constexpr u32 ITEMS = SC_PER * NTB;  // elements of a chunk
    static constexpr bool HALF = W > 8;  // counts (at most ITEMS) in 16 bits, two to a word
    static constexpr u32 CW = HALF ? Digits<W>::NB / 2 : Digits<W>::NB;
    u64 sk[ITEMS];
    u32 sv[ITEMS];
    u32 cnt[NTB / 64][CW];    // per wavefront and digit: elements so far, then their place in the chunk
    u32 gofs[Digits<W>::NB];  // output position of a bucket's element, less its place in the chunk
    u32 wsum[NTB / 64];
};

// Elements [b0, b1) by digit(key); run: see k_scatter (the first 256 threads').
template <u32 W, u32 NTB = NT, class DG>
__device__ __forceinline__ void scatter_range(ScatterLds<W, NTB> &L, const DG &digit, const u64 *ksrc,
                                              const u32 *vsrc, u64 *kdst, u32 *vdst, u32 b0, u32 b1,
                                              u32 (&run)[Digits<W>::DPT])
{
    constexpr u32 DPT = Digits<W>::DPT, NW = NTB / 64, CW = ScatterLds<W, NTB>::CW, SC_ITEMS = ScatterLds<W, NTB>::ITEMS;
    constexpr bool HALF = ScatterLds<W, NTB>::HALF;
    const bool dt = NTB == 256 || threadIdx.x < 256;  // owns digits
    const u32 wid = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (u32 c0 = b0; c0 < b1; c0 += SC_ITEMS) {
        const u32 m = b1 - c0 < SC_ITEMS ? b1 - c0 : SC_ITEMS;
        u64 kq[SC_PER];
        u32 vq[SC_PER], pos[SC_PER];
#pragma unroll
        for (u32 q = 0; q < SC_PER; q++) {
            const u32 i = (wid * SC_PER + q) * 64 + lane;
            kq[q] = 0;
            vq[q] = 0;
            if (i < m) {
                kq[q] = ksrc[c0 + i];
                vq[q] = vsrc[c0 + i];
            }
        }
        for (u32 d = threadIdx.x; d < NW * CW; d += NTB) (&L.cnt[0][0])[d] = 0;
        __syncthreads();
#pragma unroll
        for (u32 q = 0; q < SC_PER; q++) {
            const bool valid = (wid * SC_PER + q) * 64 + lane < m;
            const u32 d = digit(kq[q]);
            const u64 peers = match_digit_w<W>(d, valid);
            const u32 rank = (u32)__popcll(peers & lanemask_lt());
            u32 old = 0;
            if (valid && rank == 0) {
                const u32 np = (u32)__popcll(peers);
                if (HALF) old = (atomicAdd(&L.cnt[wid][d >> 1], np << (16 * (d & 1))) >> (16 * (d & 1))) & 0xFFFFu;
                else old = atomicAdd(&L.cnt[wid][d], np);
            }
            const int leader = valid ? __ffsll((unsigned long long)peers) - 1 : (int)lane;
            pos[q] = __shfl(old, leader, 64) + rank;
        }
        __syncthreads();
        {
            u32 c[NW][DPT], sum = 0;
#pragma unroll
            for (u32 r = 0; r < DPT; r++)
#pragma unroll
                for (u32 w = 0; w < NW; w++) {
                    const u32 d = threadIdx.x * DPT + r;
                    c[w][r] = !dt ? 0u : HALF ? (L.cnt[w][d >> 1] >> (16 * (d & 1))) & 0xFFFFu : L.cnt[w][d];
                    sum += c[w][r];
                }
            u32 x = sum;
#pragma unroll
            for (u32 o = 1; o < 64; o <<= 1) {
                const u32 y = __shfl_up(x, o, 64);
                if (lane >= o) x += y;
            }
            if (lane == 63) L.wsum[wid] = x;
            __syncthreads();
            x -= sum;
#pragma unroll
            for (u32 w = 0; w < NW; w++)
                if (w < wid) x += L.wsum[w];
            u32 pk[NW];  // (16 bits: this thread's even digit, for the odd one's word)
#pragma unroll
            for (u32 r = 0; r < DPT; r++) {
                if (!dt) break;
                const u32 d = threadIdx.x * DPT + r, x0 = x;
                L.gofs[d] = run[r] - x0;
#pragma unroll
                for (u32 w = 0; w < NW; w++) {
                    if (!HALF) L.cnt[w][d] = x;
                    else if (r & 1) L.cnt[w][d >> 1] = pk[w] | (x << 16);
                    else pk[w] = x;
                    x += c[w][r];
                }
                run[r] += x - x0;
            }
        }
        __syncthreads();
#pragma unroll
        for (u32 q = 0; q < SC_PER; q++) {
            if ((wid * SC_PER + q) * 64 + lane < m) {
                const u32 d = digit(kq[q]);
                const u32 x = pos[q] + (HALF ? (L.cnt[wid][d >> 1] >> (16 * (d & 1))) & 0xFFFFu : L.cnt[wid][d]);
                L.sk[x] = kq[q];
                L.sv[x] = vq[q];
            }
        }
        __syncthreads();
#pragma unroll
        for (u32 q = 0; q < SC_PER; q++) {
            const u32 x = q * NTB + threadIdx.x;
            if (x < m) {
                const u64 k = L.sk[x];
                const u32 dst = L.gofs[digit(k)] + x;
                kdst[dst] = k;
                vdst[dst] = L.sv[x];
            }
        }
        // (the next chunk's first barrier comes before anything here is rewritten,
        // but for the counts, which nothing above reads any more)
    }
}

template <bool LOOP, u32 W>
__global__ __launch_bounds__(NT) void k_scatter(const Seg *segs, const u32 *tstart, const u32 *nsegp, u32 tile,
                                                const u32 *hist, const u8 *scat, u64 *keyA, u32 *valA,
                                                u64 *keyB, u32 *valB, const u64 *dig, const u64 *split)
{
    constexpr u32 NB = Digits<W>::NB, DPT = Digits<W>::DPT;
    __shared__ ScatterLds<W> L;
    LevelDigit<LOOP && W == 8> digit;
    const u32 nseg = *nsegp;
    const u32 ntiles = LOOP ? tstart[nseg] : 0u;
    TILE_LOOP(t, ntiles) {
    const u32 s = seg_of_tile(tstart, nseg, t);
    if (!scat[s]) continue;  // (uniform over the workgroup)
    const Seg g = segs[s];
    const bool inb = g.aux & SEG_INB;
    const u64 *ksrc = inb ? keyB : keyA;
    const u32 *vsrc = inb ? valB : valA;
    u64 *kdst = inb ? keyA : keyB;
    u32 *vdst = inb ? valA : valB;
    const u32 ts = tstart[s];
    const u32 T = tstart[s + 1] - ts;
    const u32 lt = t - ts;
    digit.set(dig[s], split);
    const u32 b0 = g.begin + lt * tile;
    const u32 b1 = min(g.end, b0 + tile);
    const u32 base = hist[NB * ts];
    u32 run[DPT];  // next free position of the thread's digits, DPT neighbouring ones
#pragma unroll
    for (u32 r = 0; r < DPT; r++) run[r] = g.begin + hist[NB * ts + (threadIdx.x * DPT + r) * T + lt] - base;
    scatter_range<W>(L, digit, ksrc, vsrc, kdst, vdst, b0, b1, run);
    __syncthreads();  // (the next tile)
    }
}

// All radix levels of a segment by one workgroup, for the sorts that a captured
// graph repeats: their levels are enqueued whether or not there is work, and
// eight levels of six launches, most of them empty, were 240 of 410 us for 64
// sets of 100 to 10,000 strings.  Segments of up to WG_MAX strings come here
// at once (32 elements a thread and pass), and what one or two levels over the
// whole device leave: of segments above SPLIT_MIN about an eighth at most (see
// there), of smaller ones all if their keys are skewed (100,000 strings, 95 % of them
// sharing six bytes: 785 us, with all levels over the device 1125).  The segments of a level that need another wait
// in `stack`, which holds one entry per `slot` = small_max + 1 strings: each
// has more members than small_max, so those of one segment fit its own part.
//
// A workgroup of 1024: with 256 the sets of up to 10,000 strings took 46 us, now
// 40.
#define WG_NT 1024
#define WG_HEAVY 8192  // strings from which a segment's keys are sampled for one that an eighth of them share
#define WG_MAX 32768
// Levels over the whole device before it: none where no segment can be larger,
// one where its share of a sort of 16 such segments is left, else two.
static u32 wg_levels(u64 n) { return n <= WG_MAX ? 0 : (n <= 16 * WG_MAX ? 1 : 2); }
__global__ __launch_bounds__(WG_NT) void k_radix_wg(const Seg *wl, const u32 *nwl, const Seg *la, const u32 *nla,
                                                 Seg *stack, u32 slot, const u64 *rmask, u64 *keyA, u32 *valA,
                                                 u64 *keyB, u32 *valB, EmitOut o)
{
    __shared__ ScatterLds<8, WG_NT> L;
    __shared__ EmitLds E;
    __shared__ u32 h[256], wsum[4], s_push;
    __shared__ u8 kd[256];
    const u32 nw = *nwl, total = nw + *nla;
    const u32 t = threadIdx.x, lane = t & 63, wid = t >> 6;
    for (u32 s = blockIdx.x; s < total; s += gridDim.x) {  // (uniform over the workgroup)
        Seg g = s < nw ? wl[s] : la[s - nw];
        Seg *const st = stack + g.begin / slot;
        u32 sp = 0;
        for (;;) {
            const bool inb = g.aux & SEG_INB;
            const u64 *ksrc = inb ? keyB : keyA;
            const u32 *vsrc = inb ? valB : valA;
            const Digit D = digit_unpack(digit_spec(g, rmask, 8, false));
            // a key that many of a long segment's strings share is taken out
            // first, with the smaller and the larger ones beside it: as digits
            // it would keep them together for up to eight levels, one workgroup
            // over all of them each time
            bool heavy = false;
            u64 hk = 0;
            if (g.end - g.begin > WG_HEAVY) {
                hk = ksrc[g.begin + (u32)((u64)(g.end - g.begin) * lane / 64)];  // (the same in every wavefront)
                u32 c = 0;
                for (u32 l = 0; l < 64; l++) c += __shfl(hk, l, 64) == hk ? 1u : 0u;
                u32 best = (c << 6) | lane;
#pragma unroll
                for (int d = 1; d < 64; d <<= 1) {
                    const u32 y = __shfl_xor(best, d, 64);
                    best = y > best ? y : best;
                }
                hk = __shfl(hk, best & 63, 64);
                heavy = (best >> 6) >= 8;
            }
            auto digit = [&](u64 k) { return heavy ? (k < hk ? 0u : (k == hk ? 1u : 2u)) : digit_of(k, D); };
            if (t < 256) h[t] = 0;
            if (t == 0) s_push = 0;
            emit_zero(E);
            __syncthreads();
            u64 mn = ~0ull, mx = 0;
            for (u32 c0 = g.begin; c0 < g.end; c0 += RX_PF * WG_NT) {
                u64 kq[RX_PF];
#pragma unroll
                for (u32 q = 0; q < RX_PF; q++) {
                    const u32 i = c0 + q * WG_NT + t;
                    kq[q] = i < g.end ? ksrc[i] : 0;
                }
#pragma unroll
                for (u32 q = 0; q < RX_PF; q++) {
                    if (c0 + q * WG_NT >= g.end) break;  // (uniform)
                    const bool valid = c0 + q * WG_NT + t < g.end;
                    if (valid) {
                        mn = kq[q] < mn ? kq[q] : mn;
                        mx = kq[q] > mx ? kq[q] : mx;
                        atomicAdd(&h[digit(kq[q])], 1u);
                    }
                }
            }
            mn = block_min<u64, WG_NT>(mn);
            mx = ~block_min<u64, WG_NT>(~mx);  // (its barriers: h is complete)
            const u32 fd = mn == mx ? 64u : (u32)__clzll(mn ^ mx);
            EmitItem it[1] = {EmitItem{K_NONE, Seg{0, 0, 0, 0}, false, make_uint2(0, 0)}};
            if (!heavy && fd < 64 && fd > 63 - D.low) {  // the whole digit is common
                g.aux = fd | (g.aux & (SEG_INB | SEG_NOROOT));
                __syncthreads();
                continue;
            }
            if (fd == 64) {
                if (t == 0) it[0] = emit_whole(g, mn);
                emit_push(it, o, E);
                if (inb)
                    for (u32 i = g.begin + t; i < g.end; i += WG_NT) {
                        keyA[i] = keyB[i];
                        valA[i] = valB[i];
                    }
            } else {
                const u32 cnt = t < 256 ? h[t] : 0u;
                u32 x = cnt;
#pragma unroll
                for (u32 d = 1; d < 64; d <<= 1) {
                    const u32 y = __shfl_up(x, d, 64);
                    if (lane >= d) x += y;
                }
                if (lane == 63 && wid < 4) wsum[wid] = x;
                __syncthreads();
                x -= cnt;
#pragma unroll
                for (u32 w = 0; w < 4; w++)
                    if (w < wid) x += wsum[w];
                if (t < 256) {
                    // what a bucket's members share: the digit, all of the key, or nothing more
                    const u32 used = heavy ? (t == 1 ? 64u : (g.aux & 63)) : D.used;
                    it[0] = emit_bucket(g, used, (u32)(heavy ? hk : digit_put(mn, t, D)) & 0xFFu, x, cnt, o.small_max);
                    kd[t] = (u8)it[0].kind;
                }
                if (it[0].kind == K_LARGE) {
                    st[sp + atomicAdd(&s_push, 1u)] = it[0].ns;
                    it[0].kind = K_NONE;
                }
                emit_push(it, o, E);
                sp += s_push;
                u32 run[1] = {g.begin + x};
                scatter_range<8, WG_NT>(L, digit, ksrc, vsrc, inb ? keyA : keyB, inb ? valA : valB, g.begin, g.end, run);
                __syncthreads();
                if (!inb)  // what no later kernel rewrites back to A
                    for (u32 c0 = g.begin; c0 < g.end; c0 += RX_PF * WG_NT) {
                        u64 kq[RX_PF];
#pragma unroll
                        for (u32 q = 0; q < RX_PF; q++) {
                            const u32 i = c0 + q * WG_NT + t;
                            kq[q] = i < g.end ? keyB[i] : 0;
                        }
#pragma unroll
                        for (u32 q = 0; q < RX_PF; q++) {
                            const u32 i = c0 + q * WG_NT + t, c = kd[digit(kq[q])];
                            if (i < g.end && (c == K_NONE || c == K_NEXT || c == K_IDENT)) {
                                keyA[i] = kq[q];
                                valA[i] = valB[i];
                            }
                        }
                    }
            }
            __syncthreads();  // (s_push, h, kd and the stack's entry)
            if (sp == 0) break;
            g = st[--sp];
        }
    }
}

// After a level: buckets that no later kernel rewrites (singletons, runs for
// the next round, equal strings) are copied to A when the level left them in
// B.  Scattered segments read back their digits to find them; an unscattered
// segment that became such a run is copied whole.
template <bool LOOP, u32 W>
__global__ __launch_bounds__(NT) void k_settle(const Seg *segs, const u32 *tstart, const u32 *nsegp, u32 tile,
                                               const u8 *scat, const u8 *kinds, const u64 *keyB,
                                               const u32 *valB, u64 *keyA, u32 *valA, const u64 *dig,
                                               const u64 *split)
{
    LevelDigit<LOOP && W == 8> digit;
    const u32 nseg = *nsegp;
    const u32 ntiles = LOOP ? tstart[nseg] : 0u;
    TILE_LOOP(t, ntiles) {
    const u32 s = seg_of_tile(tstart, nseg, t);
    const Seg g = segs[s];
    const bool inb = g.aux & SEG_INB;
    const u32 lt = t - tstart[s];
    const u32 b0 = g.begin + lt * tile;
    const u32 b1 = min(g.end, b0 + tile);
    const u8 *kd = kinds + Digits<W>::NB * s;
    if (scat[s]) {
        if (inb) continue;  // scattered into A
        const u64 spec = dig[s];
        const bool by = LOOP && W == 8 && (spec & SPLIT_FLAG);  // (uniform)
        if (by) __syncthreads();  // (an earlier tile's splitters are in use no more)
        digit.set(spec, split);
        if (by) __syncthreads();
        for (u32 c0 = b0; c0 < b1; c0 += RX_PF * NT) {
            // RX_PF chunks' keys, then their buckets' kinds, loaded before any is used
            u64 kq[RX_PF];
            u32 cq[RX_PF];
#pragma unroll
            for (u32 q = 0; q < RX_PF; q++) {
                const u32 i = c0 + q * NT + threadIdx.x;
                kq[q] = i < b1 ? keyB[i] : 0ull;
            }
#pragma unroll
            for (u32 q = 0; q < RX_PF; q++) cq[q] = kd[digit(kq[q])];
#pragma unroll
            for (u32 q = 0; q < RX_PF; q++) {
                const u32 i = c0 + q * NT + threadIdx.x;
                const u32 c = cq[q];
                if (i < b1 && (c == K_NONE || c == K_NEXT || c == K_IDENT)) {
                    keyA[i] = kq[q];
                    valA[i] = valB[i];
                }
            }
        }
    } else if (inb && (kd[0] == K_NEXT || kd[0] == K_IDENT)) {
        for (u32 i = b0 + threadIdx.x; i < b1; i += NT) {
            keyA[i] = keyB[i];
            valA[i] = valB[i];
        }
    }
    }
}

__global__ void k_boundary(const uint2 *bnd, const u32 *nbp, const u64 *keys, u32 *lcp)
{
    const u32 nb = *nbp;
    GSTRIDE(j, nb) {
        const uint2 b = bnd[j];
        lcp[b.x] = key_lcp(keys[b.x - 1], keys[b.x], b.y);
    }
}

// Equal strings: LCP = their length for every member after the first.
template <bool LOOP>
__global__ __launch_bounds__(NT) void k_ident(const Seg *segs, const u32 *tstart, const u32 *nsegp, u32 et,
                                              u32 *lcp)
{
    const u32 nseg = *nsegp;
    const u32 ntiles = LOOP ? tstart[nseg] : 0u;
    TILE_LOOP(t, ntiles) {
        const u32 s = seg_of_tile(tstart, nseg, t);
        const Seg g = segs[s];
        const u32 lt = t - tstart[s];
        const u32 b0 = g.begin + lt * et;
        const u32 b1 = min(g.end, b0 + et);
        for (u32 i = b0 + threadIdx.x; i < b1; i += NT)
            if (i > g.begin) lcp[i] = g.depth;
    }
}

// ----------------------------------------------------------- block sort

// Segments of 129 .. 8 NTB strings, one workgroup of NTB threads each (NTB =
// 64 or 256): a merge sort of (key, payload) in LDS.  Every thread sorts eight
// consecutive elements in registers (odd-even transposition), then runs of 8,
// 16, ... are merged pairwise: a thread finds where its eight outputs start
// (the merge path, a binary search over two keys a step) and merges them
// serially.  Keys alone are compared and every step is stable, so equal keys
// keep the payload order the segment came in, which is index order.  The
// sorted elements then give the LCPs where keys differ, and runs of equal
// continuing keys become next-round segments.
//
// Bounded by vector instructions (about 25 per element and merge level) and
// LDS latency; keys and payloads move through HBM once.  It replaces a bitonic
// network over tiles of packed segments (up to 1024 strings, 66 exchanges per
// element for 2048) and, for segments of up to 2048, a radix level before it:
// 512 sets of 10^3..10^5 strings 349 -> 148 us; 16M D/N strings, whose segments
// of 1,479 strings took a radix level (about 250 us) and 366 us in the register
// sort, 266 us.

template <bool LOOP, int NTB>
__global__ __launch_bounds__(NTB) void k_block_sort(const Seg *list, const u32 *cntp, u64 *keys, u32 *vals,
                                                    const u64 *keyB, const u32 *valB, u32 *lcp, Seg *next, u32 *ctr,
                                                    u32 *elems)
{
    constexpr u32 CAP = NTB * BS_IPT;
    __shared__ u64 sk[CAP + NTB];
    __shared__ u32 sv[CAP + NTB];
    __shared__ u32 nq_count, nq_elems, nq_base;
    const u32 nlist = LOOP ? *cntp : 0u;
    TILE_LOOP(sg, nlist) {
    const Seg g = list[sg];
    const u32 cnt = g.end - g.begin;
    const u64 *ks = (g.aux & SEG_INB) ? keyB : keys;  // read where the segment is, write A
    const u32 *vs = (g.aux & SEG_INB) ? valB : vals;
    const u32 e0 = threadIdx.x * BS_IPT;  // this thread's elements (padding sorts last)
    u64 k[BS_IPT];
    u32 v[BS_IPT];
#pragma unroll
    for (u32 q = 0; q < BS_IPT; q++) {
        k[q] = ~0ull;
        v[q] = 0xFFFFFFFFu;
        if (e0 + q < cnt) {
            k[q] = ks[g.begin + e0 + q];
            v[q] = vs[g.begin + e0 + q];
        }
    }
    if (threadIdx.x == 0) nq_count = nq_elems = 0;
#pragma unroll
    for (u32 r = 0; r < BS_IPT; r++) {
#pragma unroll
        for (u32 q = r & 1; q + 1 < BS_IPT; q += 2) {
            const bool sw = k[q] > k[q + 1];
            const u64 a = sw ? k[q + 1] : k[q], b = sw ? k[q] : k[q + 1];
            const u32 x = sw ? v[q + 1] : v[q], y = sw ? v[q] : v[q + 1];
            k[q] = a;
            k[q + 1] = b;
            v[q] = x;
            v[q + 1] = y;
        }
    }
#pragma unroll
    for (u32 q = 0; q < BS_IPT; q++) {
        sk[bs_at(e0) + q] = k[q];
        sv[bs_at(e0) + q] = v[q];
    }
    __syncthreads();
    for (u32 w = BS_IPT; w < cnt; w *= 2) {  // (uniform)
        const u32 pb = e0 & ~(2 * w - 1);  // the pair of runs [pb, pb + w), [pb + w, pb + 2w)
        const u32 pa = pb + w;
        if (pa < cnt) {  // (else the second run is padding: nothing to merge)
            const u32 d = e0 - pb;
            u32 lo = d > w ? d - w : 0u, hi = d < w ? d : w;
            while (lo < hi) {
                const u32 mid = (lo + hi) >> 1;
                if (sk[bs_at(pb + mid)] <= sk[bs_at(pa + d - 1 - mid)]) lo = mid + 1;
                else hi = mid;
            }
            u32 i = pb + lo, j = pa + d - lo;
            const u32 ie = pa, je = pa + w;
            u64 ka = i < ie ? sk[bs_at(i)] : ~0ull, kb = j < je ? sk[bs_at(j)] : ~0ull;
#pragma unroll
            for (u32 q = 0; q < BS_IPT; q++) {
                const bool first = j >= je || (i < ie && ka <= kb);
                const u32 at = first ? i : j;
                k[q] = first ? ka : kb;
                v[q] = sv[bs_at(at)];
                i += first ? 1u : 0u;
                j += first ? 0u : 1u;
                const u32 nx = at + 1, ne = first ? ie : je;
                const u64 kn = nx < ne ? sk[bs_at(nx)] : ~0ull;
                ka = first ? kn : ka;
                kb = first ? kb : kn;
            }
        }
        __syncthreads();
        if (pa < cnt) {
#pragma unroll
            for (u32 q = 0; q < BS_IPT; q++) {
                sk[bs_at(e0) + q] = k[q];
                sv[bs_at(e0) + q] = v[q];
            }
        }
        __syncthreads();
    }
    // results, lanes on consecutive elements; only the segment's end keys are
    // read again (for the LCPs across bucket boundaries)
    u32 lasts = 0, it = 0;  // bit per element of this thread: the last of a run of tied keys
    for (u32 e = threadIdx.x; e < cnt; e += NTB, it++) {
        const u32 pos = g.begin + e;
        const u64 kb = sk[bs_at(e)];
        vals[pos] = sv[bs_at(e)];
        if (e == 0 || e == cnt - 1) keys[pos] = kb;
        if (e == 0) continue;
        const u64 ka = sk[bs_at(e - 1)];
        const u32 c8 = (u32)(kb & 0xFF);
        if (ka != kb) lcp[pos] = key_lcp(ka, kb, g.depth);
        else if (c8 < 8) lcp[pos] = g.depth + c8;
        else if (e + 1 == cnt || sk[bs_at(e + 1)] != kb) lasts |= 1u << it;
    }
    if (__syncthreads_or(lasts != 0)) {
        // tied runs: counted, then written.  (One update of a global counter, two
        // where the caller wants their members counted: such updates queue, and
        // with three of them 5,623 segments of text took 219 us, now 97.)
        for (int pass = 0; pass < 2; pass++) {
            for (u32 m = lasts; m; m &= m - 1) {
                const u32 e = threadIdx.x + NTB * (u32)(__ffs((int)m) - 1);
                const u64 kb = sk[bs_at(e)];
                u32 x = 0, y = e;  // first element with this key
                while (x < y) {
                    const u32 mid = (x + y) >> 1;
                    if (sk[bs_at(mid)] < kb) x = mid + 1;
                    else y = mid;
                }
                const u32 sz = e + 1 - x;
                const u32 slot = atomicAdd(&nq_count, 1u);
                if (pass == 0) {
                    atomicAdd(&nq_elems, sz);
                } else {
                    next[nq_base + slot] = Seg{g.begin + x, g.begin + e + 1, g.depth + 7, SEG_SKIP};
                }
            }
            __syncthreads();
            if (pass == 0 && threadIdx.x == 0) {
                nq_base = atomicAdd(&ctr[C_NEXT], nq_count);
                if (elems) atomicAdd(elems, nq_elems);
                nq_count = 0;
            }
            __syncthreads();
        }
    }
    __syncthreads();  // the tables are rewritten by the next segment
    }
}

#define WS_SPB 16  // tiny segments per workgroup (4 wavefronts, 4 segments each)

__device__ __forceinline__ bool kv_greater(u64 ka, u32 va, u64 kb, u32 vb)
{
    return ka != kb ? ka > kb : va > vb;
}

// Bitonic compare-exchange of element e with the element j lanes away
// (j < 64) in a merge of size k: the lower index of an ascending pair keeps
// the smaller (key, payload).
__device__ __forceinline__ void ws_step(u64 &key, u32 &val, u32 e, u32 j, u32 k)
{
    const u64 pk = __shfl_xor(key, (int)j, 64);
    const u32 pv = __shfl_xor(val, (int)j, 64);
    const bool want_small = ((e & j) == 0) == ((e & k) == 0);
    if (want_small == kv_greater(key, val, pk, pv)) {
        key = pk;
        val = pv;
    }
}

// LCP of sorted element e (e >= 1) from its predecessor's key, as in the LDS
// sort; returns whether e is the last of a run of >= 2 equal full keys (a
// next-round segment).
__device__ __forceinline__ bool ws_finish(u32 e, u32 cnt, u64 ka, u64 kb, u64 kn, u32 dep, u32 *lcp_out)
{
    if (e == 0 || e >= cnt) return false;
    if (ka != kb) {
        *lcp_out = key_lcp(ka, kb, dep);
        return false;
    }
    const u32 c8 = (u32)(kb & 0xFF);
    if (c8 < 8) {
        *lcp_out = dep + c8;
        return false;
    }
    return e + 1 == cnt || kn != kb;
}

__device__ __forceinline__ u32 hibit(u64 m) { return 63u - (u32)__clzll(m); }

#define WS_DEEP 3  // further 7-byte keys a wavefront reads for runs of equal continuing keys

__device__ __forceinline__ bool rkv_greater(u32 ra, u64 ka, u32 va, u32 rb, u64 kb, u32 vb)
{
    return ra != rb ? ra > rb : (ka != kb ? ka > kb : va > vb);
}

// ws_step on (run start, key, payload)
__device__ __forceinline__ void ws_step3(u32 &rs, u64 &key, u32 &val, u32 e, u32 j, u32 k)
{
    const u32 pr = __shfl_xor(rs, (int)j, 64);
    const u64 pk = __shfl_xor(key, (int)j, 64);
    const u32 pv = __shfl_xor(val, (int)j, 64);
    const bool want_small = ((e & j) == 0) == ((e & k) == 0);
    if (want_small == rkv_greater(rs, key, val, pr, pk, pv)) {
        rs = pr;
        key = pk;
        val = pv;
    }
}

__device__ __forceinline__ bool shfl_down_b(bool b, u32 lane, bool from_next)
{
    const int d = __shfl_down((int)b, 1, 64);
    return lane < 63 ? d != 0 : from_next;
}

// Segments of 2..128 strings, one wavefront each: bitonic sort of
// (key, payload) in registers (element e = lane + 64 r, r = 0, 1), then LCPs.
// Runs of equal continuing keys are not sent to the next round at once: the
// wavefront reads their strings' next 7-byte keys (up to WS_DEEP times) and
// sorts every run again by (run, key, payload), writing the LCPs of the
// pairs each key separates; runs still tied then become next-round segments,
// collected per workgroup and published with one atomic per counter.  (Equal
// strings, common in text, so end inside the wavefront instead of costing a
// workgroup per run in the next round's skip and key passes.)  Without DEEP
// (keys that are no string bytes) ties are published at once.
template <bool LOOP, bool DEEP = true>
__global__ __launch_bounds__(256) void k_wave_sort(const Seg *tiny, const u32 *ntinyp, u64 *keys, u32 *vals,
                                                   const u64 *keyB, const u32 *valB, u32 *lcp, Seg *next, u32 *ctr,
                                                   const u8 *bytes, u64 N, const u64 *off, u32 *elems)
{
    __shared__ Seg nq[WS_SPB * (WS_MAX / 2)];
    __shared__ u32 nq_count, nq_elems, nq_base;
    const u32 ntiny = *ntinyp;
    const u32 ngrp = LOOP ? (ntiny + WS_SPB - 1) / WS_SPB : 0u;
    TILE_LOOP(grp, ngrp) {
    if (threadIdx.x == 0) { nq_count = 0; nq_elems = 0; }
    __syncthreads();
    const u32 lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const u32 e0 = lane, e1 = lane + 64;
    // This wavefront's segments: all descriptors first, and each segment's
    // keys and payload loaded while the previous one is being sorted.
    Seg gq[WS_SPB / 4];
#pragma unroll
    for (u32 q = 0; q < WS_SPB / 4; q++) {
        const u32 sidx = grp * WS_SPB + q * 4 + wv;
        gq[q] = sidx < ntiny ? tiny[sidx] : Seg{0, 0, 0, 0};
    }
    u64 nk0 = ~0ull, nk1 = ~0ull;
    u32 nv0 = 0xFFFFFFFFu, nv1 = 0xFFFFFFFFu;
    auto fetch = [&](const Seg &g) {
        const u32 cnt = g.end - g.begin;
        const u64 *ks = (g.aux & SEG_INB) ? keyB : keys;  // read where the segment is, write A
        const u32 *vs = (g.aux & SEG_INB) ? valB : vals;
        nk0 = ~0ull; nk1 = ~0ull; nv0 = 0xFFFFFFFFu; nv1 = 0xFFFFFFFFu;
        if (e0 < cnt) { nk0 = ks[g.begin + e0]; nv0 = vs[g.begin + e0]; }
        if (e1 < cnt) { nk1 = ks[g.begin + e1]; nv1 = vs[g.begin + e1]; }
    };
    fetch(gq[0]);
#pragma unroll
    for (u32 q = 0; q < WS_SPB / 4; q++) {
        const u32 sidx = grp * WS_SPB + q * 4 + wv;
        if (sidx >= ntiny) break;  // uniform over the wavefront
        const Seg g = gq[q];
        const u32 cnt = g.end - g.begin;
        u64 k0 = nk0, k1 = nk1;
        // (keys of any payload are sorted with the element numbers, and the
        // payload follows: its own order need not be the segment's)
        u32 v0 = DEEP ? nv0 : e0, v1 = DEEP ? nv1 : e1;
        const u32 pv0 = nv0, pv1 = nv1;
        if (q + 1 < WS_SPB / 4) fetch(gq[q + 1]);
        u32 P = 2;
        while (P < cnt) P <<= 1;
        for (u32 k = 2; k <= P; k <<= 1) {
            for (u32 j = k >> 1; j > 0; j >>= 1) {
                if (j == 64) {
                    // partner of e0 is e1 in the same lane (k == 128: ascending)
                    if (kv_greater(k0, v0, k1, v1)) {
                        const u64 tk = k0; k0 = k1; k1 = tk;
                        const u32 tv = v0; v0 = v1; v1 = tv;
                    }
                } else {
                    ws_step(k0, v0, e0, j, k);
                    if (P == 128) ws_step(k1, v1, e1, j, k);
                }
            }
        }
        // (only the segment's end keys are read again, for the LCPs across bucket boundaries)
        if (e0 == 0 || e0 == cnt - 1) keys[g.begin + e0] = k0;
        if (e1 == cnt - 1) keys[g.begin + e1] = k1;
        // neighbours in sorted order
        const u64 k0_last = __shfl(k0, 63, 64), k1_first = __shfl(k1, 0, 64);
        const u64 up0 = __shfl_up(k0, 1, 64), up1 = __shfl_up(k1, 1, 64);
        const u64 dn0 = __shfl_down(k0, 1, 64), dn1 = __shfl_down(k1, 1, 64);
        const u64 pa0 = up0, pa1 = lane ? up1 : k0_last;
        const u64 nx0 = lane < 63 ? dn0 : k1_first, nx1 = dn1;
        u32 l0 = 0, l1 = 0;
        ws_finish(e0, cnt, pa0, k0, nx0, g.depth, &l0);
        ws_finish(e1, cnt, pa1, k1, nx1, g.depth, &l1);
        // LCP writes (skipped for the first element and for equal full keys)
        if (e0 >= 1 && e0 < cnt && !(pa0 == k0 && (k0 & 0xFF) == 8)) lcp[g.begin + e0] = l0;
        if (e1 < cnt && !(pa1 == k1 && (k1 & 0xFF) == 8)) lcp[g.begin + e1] = l1;
        const u64 le = lane == 63 ? ~0ull : ((2ull << lane) - 1ull);
        // tied with the predecessor: equal keys, both strings continue
        bool t0 = e0 >= 1 && e0 < cnt && pa0 == k0 && (k0 & 0xFF) == 8;
        bool t1 = e1 < cnt && pa1 == k1 && (k1 & 0xFF) == 8;
        u32 dep = g.depth;
        if (__ballot(t0 || t1)) {  // (uniform: most segments have no run of equal keys)
        for (u32 it = 0; it < (DEEP ? WS_DEEP : 0); it++) {
            // in a run: tied with the predecessor or the successor (e0's successor
            // is e0 + 1, lane 63's is e1 of lane 0); every lane shuffles first
            const bool f1 = __shfl((int)t1, 0, 64) != 0;
            const bool n0 = shfl_down_b(t0, lane, f1), n1 = shfl_down_b(t1, lane, false);
            const bool in0 = t0 || n0, in1 = t1 || n1;
            if (!__ballot(in0 || in1)) break;  // (uniform)
            dep += 7;
            // run of every element: its first position (padding sorts last)
            const u64 s0 = __ballot(!t0), s1 = __ballot(!t1);
            const u64 ms = s1 & le;
            u32 rs0 = e0 < cnt ? hibit(s0 & le) : 0xFFFFFFFFu;
            u32 rs1 = e1 < cnt ? (ms ? 64u + hibit(ms) : hibit(s0)) : 0xFFFFFFFFu;
            u64 q0 = e0 < cnt ? 0ull : ~0ull, q1 = e1 < cnt ? 0ull : ~0ull;
            if (in0) {
                const u64 o = off[v0];
                q0 = make_key(bytes, N, o, off[v0 + 1] - o, dep);
            }
            if (in1) {
                const u64 o = off[v1];
                q1 = make_key(bytes, N, o, off[v1 + 1] - o, dep);
            }
            for (u32 k = 2; k <= P; k <<= 1) {
                for (u32 j = k >> 1; j > 0; j >>= 1) {
                    if (j == 64) {
                        if (rkv_greater(rs0, q0, v0, rs1, q1, v1)) {
                            const u32 tr = rs0; rs0 = rs1; rs1 = tr;
                            const u64 tq = q0; q0 = q1; q1 = tq;
                            const u32 tv = v0; v0 = v1; v1 = tv;
                        }
                    } else {
                        ws_step3(rs0, q0, v0, e0, j, k);
                        if (P == 128) ws_step3(rs1, q1, v1, e1, j, k);
                    }
                }
            }
            const u32 rp0 = __shfl_up(rs0, 1, 64), rl0 = __shfl(rs0, 63, 64), ru1 = __shfl_up(rs1, 1, 64);
            const u32 rp1 = lane ? ru1 : rl0;
            const u64 qp0 = __shfl_up(q0, 1, 64), ql0 = __shfl(q0, 63, 64), qu1 = __shfl_up(q1, 1, 64);
            const u64 qp1 = lane ? qu1 : ql0;
            const bool same0 = e0 >= 1 && e0 < cnt && rp0 == rs0;  // same run as the predecessor
            const bool same1 = e1 < cnt && rp1 == rs1;
            t0 = same0 && qp0 == q0 && (q0 & 0xFF) == 8;
            t1 = same1 && qp1 == q1 && (q1 & 0xFF) == 8;
            if (same0 && !t0) lcp[g.begin + e0] = qp0 != q0 ? key_lcp(qp0, q0, dep) : dep + (u32)(q0 & 0xFF);
            if (same1 && !t1) lcp[g.begin + e1] = qp1 != q1 ? key_lcp(qp1, q1, dep) : dep + (u32)(q1 & 0xFF);
        }
        // still tied: the last element of each run publishes it for the next round
        const bool f1 = __shfl((int)t1, 0, 64) != 0;
        const bool n0 = shfl_down_b(t0, lane, f1), n1 = shfl_down_b(t1, lane, false);
        const bool end0 = t0 && !n0, end1 = t1 && !n1;
        const u64 s0 = __ballot(!t0), s1 = __ballot(!t1);
        if (end0) {
            const u32 f = hibit(s0 & le);
            const Seg ns{g.begin + f, g.begin + e0 + 1, dep + 7, SEG_SKIP};
            nq[atomicAdd(&nq_count, 1u)] = ns;
            atomicAdd(&nq_elems, ns.end - ns.begin);
        }
        if (end1) {
            const u64 mm = s1 & le;
            const u32 f = mm ? 64u + hibit(mm) : hibit(s0);
            const Seg ns{g.begin + f, g.begin + e1 + 1, dep + 7, SEG_SKIP};
            nq[atomicAdd(&nq_count, 1u)] = ns;
            atomicAdd(&nq_elems, ns.end - ns.begin);
        }
        }
        if (!DEEP) {
            const u32 a0 = __shfl(pv0, v0 & 63, 64), b0 = __shfl(pv1, v0 & 63, 64);
            const u32 a1 = __shfl(pv0, v1 & 63, 64), b1 = __shfl(pv1, v1 & 63, 64);
            v0 = v0 < 64 ? a0 : b0;
            v1 = v1 < 64 ? a1 : b1;
        }
        if (e0 < cnt) vals[g.begin + e0] = v0;
        if (e1 < cnt) vals[g.begin + e1] = v1;
    }
    __syncthreads();
    if (threadIdx.x == 0 && nq_count) {
        nq_base = atomicAdd(&ctr[C_NEXT], nq_count);
        if (elems) atomicAdd(elems, nq_elems);
    }
    __syncthreads();
    for (u32 k = threadIdx.x; k < nq_count; k += 256) next[nq_base + k] = nq[k];
    __syncthreads();  // nq and its counters are reset for the next group
    }
}

// ------------------------------------------------------------ host driver

void sort_ws_layout(u64 n, SortWs *w, WsArena *a, WsCounter *c)
{
    // Capacities: segments hold >= 2 strings (<= n/2 of them); radix segments
    // hold > 128 strings; radix tiles <= n/1024 + radix segments.
    const u64 nseg = n / 2 + 2;
    const u64 nlarge = n / 128 + 2;
    const u64 ntiles = n / 1024 + nlarge + 2;
    // histograms and bucket kinds: 256 buckets per radix tile / segment with
    // 8-bit digits; 2048 with 11-bit digits, which are used only with tiles
    // of >= 4096 and radix segments of > 512 strings
    const u64 nlarge11 = n / 512 + 2, ntiles11 = n / 4096 + nlarge11 + 2;
    const u64 nhist = 256 * ntiles > 2048 * ntiles11 ? 256 * ntiles : 2048 * ntiles11;
    const u64 nkinds = 256 * nlarge > 2048 * nlarge11 ? 256 * nlarge : 2048 * nlarge11;
    const u64 nscan = (nhist > nseg + 1 ? nhist : nseg + 1) + 1;
#define TAKE(field, T, cnt)                      \
    do {                                          \
        if (a) w->field = a->take<T>(cnt);        \
        else c->take<T>(cnt);                     \
    } while (0)
    TAKE(keyA, u64, n);
    TAKE(keyB, u64, n);
    TAKE(mword, u64, n);
    TAKE(mpr, uint2, n);
    TAKE(valB, u32, n);
    TAKE(lcp_scratch, u32, n);
    TAKE(act, Seg, nseg);
    TAKE(nxt, Seg, nseg);
    TAKE(tiny, Seg, nseg);
    TAKE(small, Seg, nlarge);
    TAKE(mid, Seg, nlarge);
    TAKE(ident, Seg, nseg);
    TAKE(largeA, Seg, nlarge);
    TAKE(largeB, Seg, nlarge);
    TAKE(wgl, Seg, nlarge);
    TAKE(bnd, uint2, n + 1);
    TAKE(skipv, u32, nseg);
    TAKE(smin, u64, nlarge);
    TAKE(smax, u64, nlarge);
    TAKE(rmask, u64, nlarge);
    TAKE(dig, u64, nlarge);
    TAKE(split, u64, (SPLITS + 1) * (n / SPLIT_MIN + 1 < SPLIT_LIST ? n / SPLIT_MIN + 1 : (u64)SPLIT_LIST));
    TAKE(scat, u8, nlarge);
    TAKE(kinds, u8, nkinds);
    TAKE(tstart, u32, nseg + 1);
    TAKE(hist, u32, nscan);
    TAKE(scan_scratch, u64, ss_scan_scratch_elems<u64>(nscan));
    TAKE(dscan, u64, SCAN_DEV_STATE);
    TAKE(hscan, u64, SCAN_DEV_STATE);
    TAKE(ctr, u32, C_NCTR);
    TAKE(hdr, u32, H_NHDR);
#undef TAKE
}

// Launch shapes.  A kernel over a list takes its items in a grid-stride loop;
// the host sizes its grid from the list's length when it knows it (read back),
// otherwise it launches a fixed grid bounded by the largest list possible.
static unsigned grid_of(u64 items, u64 per, u64 cap)
{
    const u64 g = ceil_div(items, per);
    return (unsigned)(g < 1 ? 1 : (g > cap ? cap : g));
}

// One round or level's lengths: known to the host (read back) or not.
struct Known {
    bool yes;
    u32 v;
};

struct RoundCtx {
    const SortJob &J;
    SortWs &w;
    u64 n;  // strings of the whole sort (bounds every list)
    u32 SM, TL;
    u32 W;   // radix digit bits (8, or 11 with tiles >= 4096 and a cutover >= 512)
    u32 ET;  // elements per workgroup of the element-wise kernels
    u32 BM;  // segments of up to this many strings are sorted in LDS
};

// Elements per workgroup of the element-wise round kernels in a sort of n
// strings: ETILE, but fewer below 2M strings so that there are about 1024
// workgroups (at 100,000 strings k_skip's 49 took 66 us, 391 take 15 us).  More
// of them in large sorts only repeat the set-up: 16M D/N strings take 4 % longer
// with 512.
static u32 elem_tile(u64 n)
{
    u32 t = ETILE;
    while (t > 256 && n < 1024ull * t) t /= 2;
    return t;
}

static u32 digit_bits_for(u32 SM, u32 TL) { return (g_digit_bits == 11 && TL >= 4096 && SM >= 512) ? 11u : 8u; }

// Strings per tile of the radix levels: g_tile, but in sorts of fewer than 256
// such tiles smaller ones (100,000 D/N strings: 199 us with 25 workgroups of 4096,
// 181 us with 98 of 1024; 64 sets of 100 to 10,000 strings 463 and 434 us).
static u32 radix_tile(u64 n)
{
    u32 t = (u32)g_tile;
    if (digit_bits_for((u32)g_small_max, t) == 8)
        while (t >= 2048 && n < 256ull * t) t /= 2;
    return t;
}

static RoundCtx round_ctx(const SortJob &J, SortWs &w)
{
    const u32 sm = (u32)g_small_max, tl = (u32)g_tile;
    const SortShape z = sort_shape(J.n_total);
    return RoundCtx{J, w, J.n_total, sm, z.tile, digit_bits_for(sm, tl), z.et, z.block_max};
}

// The scan of a list's tile counts (the kernel before it cleared the state).
static int scan_u32(RoundCtx &C, u32 *arr, const u32 *n_dev, u64 n_max)
{
    return ss_scan_exclusive_dev(arr, arr, n_dev, n_max, C.w.dscan, C.J.stream);
}

// The part of a round before the radix levels: skip, keys, routing.  The round's
// segments are w.act, their number in counter `from` (or, `begun`, the header,
// tiles and skip minima are set already).
static int round_head(RoundCtx &C, Known nact, Known atiles, u64 round_elems, bool first = false, u32 from = C_NEXT,
                      bool begun = false, u64 bound = 0)
{
    SortWs &w = C.w;
    const SortJob &J = C.J;
    hipStream_t st = J.stream;
    const u64 n = C.n;
    const u32 *nactp = w.hdr + H_ACT;
    const u64 most = nact.yes ? nact.v : (bound ? bound : n / 2);  // (bound: on a number not known)
    if (!begun && most <= LIST_ONE) {
        k_round_start<<<1, LIST_NT, 0, st>>>(w.act, w.ctr, w.hdr, from, C.ET, w.tstart, w.skipv, w.keyB,
                                            C.BM);
        SS_CHECK_LAUNCH();
    } else if (!begun) {
        k_round_begin<<<1, 64, 0, st>>>(w.ctr, w.hdr, from);
        SS_CHECK_LAUNCH();
        k_round_tiles<<<grid_of(most, 256, 1024), 256, 0, st>>>(w.act, nactp, C.ET, w.tstart, w.skipv, w.dscan, w.keyB,
                                                                C.BM);
        SS_CHECK_LAUNCH();
        SS_TRY(scan_u32(C, w.tstart, nactp, most));
    }
    const unsigned tg = atiles.yes ? grid_of(atiles.v, 1, 1u << 30) : 0u;  // (one tile per workgroup)
    {
        // algorithmic bytes: perm + offsets + one word per string, its mismatch
        // record out, plus the common prefix (added once the skips are known)
        // (seeded: the records in, the strings of members the seed left open)
        const bool sd = first && atiles.yes && J.seed_pos;
        SS_PROF("k_skip", st, (double)round_elems * (sd ? 8.0 : 44.0));
        if (sd) k_skip<false, true><<<tg, NT, 0, st>>>(w.act, w.tstart, nactp, C.ET, J.bytes, J.N, J.off, J.vals, w.skipv, J.seed_word, J.seed_pos, J.seed_ok);
        // (tiles of small segments, as later rounds leave them, hold few
        // members: one wavefront per tile then keeps four times as many in
        // flight)
        else if (atiles.yes && round_elems < 64ull * atiles.v)
            k_skip<false, false, 64><<<tg, 64, 0, st>>>(w.act, w.tstart, nactp, C.ET, J.bytes, J.N, J.off, J.vals, w.skipv, w.mword, w.mpr);
        else if (atiles.yes) k_skip<false><<<tg, NT, 0, st>>>(w.act, w.tstart, nactp, C.ET, J.bytes, J.N, J.off, J.vals, w.skipv, w.mword, w.mpr);
        else k_skip<true><<<grid_of(n, C.ET, resident(k_skip<true>, NT)), NT, 0, st>>>(w.act, w.tstart, nactp, C.ET, J.bytes, J.N, J.off, J.vals, w.skipv, w.mword, w.mpr);
    }
    SS_CHECK_LAUNCH();
    {
        // the first round of a seeded sort keeps its records in the seed
        const bool sd = first && atiles.yes && J.seed_pos;
        u64 *mw = sd ? J.seed_word : w.mword;
        uint2 *mp = sd ? J.seed_pos : w.mpr;
        SS_PROF("k_keys", st, (double)round_elems * 24.0);  // mismatch record in, key out
        if (atiles.yes && round_elems < 64ull * atiles.v)  // (small tiles: one wavefront each, as in the skip)
            k_keys<false, 64><<<tg, 64, 0, st>>>(w.act, w.tstart, nactp, C.ET, J.bytes, J.N, J.off, J.vals, w.skipv, mw, mp, w.keyA, w.keyB, C.BM);
        else if (atiles.yes) k_keys<false><<<tg, NT, 0, st>>>(w.act, w.tstart, nactp, C.ET, J.bytes, J.N, J.off, J.vals, w.skipv, mw, mp, w.keyA, w.keyB, C.BM);
        else k_keys<true><<<grid_of(n, C.ET, resident(k_keys<true>, NT)), NT, 0, st>>>(w.act, w.tstart, nactp, C.ET, J.bytes, J.N, J.off, J.vals, w.skipv, mw, mp, w.keyA, w.keyB, C.BM);
    }
    SS_CHECK_LAUNCH();
    k_classify<<<grid_of(nact.yes ? nact.v : n / 2, 256, 1024), 256, 0, st>>>(w.act, nactp, w.skipv, C.BM, C.TL,
                                                                             w.tiny, w.small, w.mid, w.largeA, w.ctr, w.keyB,
                                                                             w.rmask);
    SS_CHECK_LAUNCH();
    return SS_OK;
}

// One radix level over the list LA (its length in ctr[C_LARGE] when the level
// starts); its sub-lists go to LB and the round's lists.
template <u32 W>
static int radix_level_w(RoundCtx &C, Seg *LA, Seg *LB, Known nlarge, Known ltiles, u64 lelem, bool wg)
{
    constexpr u32 NB = Digits<W>::NB;
    SortWs &w = C.w;
    const SortJob &J = C.J;
    hipStream_t st = J.stream;
    const u64 n = C.n;
    const u32 *nlp = w.hdr + H_LARGE;
    // (enqueued levels are as many as full digits need)
    const bool narrow = ltiles.yes && lelem >= NARROW_MIN;
    const u64 most = nlarge.yes ? nlarge.v : n / C.BM;  // radix segments have more than BM strings
    if (most <= LIST_ONE) {
        auto *const start = wg ? k_level_start<true> : k_level_start<false>;
        start<<<1, LIST_NT, 0, st>>>(LA, w.ctr, w.hdr, NB, C.TL, w.tstart, w.smin, w.smax, w.hscan,
                                            w.rmask, w.dig, narrow, w.wgl, WG_MAX, w.keyA, w.keyB, w.split);
        SS_CHECK_LAUNCH();
    } else {
        k_level_begin<<<1, 256, 0, st>>>(w.ctr, w.hdr, NB, w.hscan);
        SS_CHECK_LAUNCH();
        k_level_tiles<<<grid_of(most, 256, 1024), 256, 0, st>>>(LA, nlp, C.TL, w.tstart, w.smin, w.smax, w.dscan,
                                                                w.rmask, w.dig, W, narrow);
        SS_CHECK_LAUNCH();
        SS_TRY(scan_u32(C, w.tstart, nlp, most));
    }
    const unsigned tg = ltiles.yes ? grid_of(ltiles.v, 1, 1u << 30) : 0u;  // (one tile per workgroup)
    {
        SS_PROF("k_hist", st, (double)lelem * 8.0);  // read the keys
        if (ltiles.yes) k_hist<false, W><<<tg, NT, 0, st>>>(LA, w.tstart, nlp, C.TL, w.keyA, w.keyB, w.hist, w.smin, w.smax, w.dig, w.split);
        else k_hist<true, W><<<grid_of(n, C.TL, resident(k_hist<true, W>, NT)), NT, 0, st>>>(LA, w.tstart, nlp, C.TL, w.keyA, w.keyB, w.hist, w.smin, w.smax, w.dig, w.split);
    }
    SS_CHECK_LAUNCH();
    // (three launches once there are more items than one range per workgroup holds)
    const u64 nh = (ltiles.yes ? ltiles.v : n / C.TL + n / C.BM) * (u64)NB;
    if (ltiles.yes && nh > SCAN_DEV_MAX) SS_TRY(ss_scan_exclusive<u32>(w.hist, w.hist, nh, (u32 *)w.scan_scratch, st));
    else SS_TRY(ss_scan_exclusive_dev(w.hist, w.hist, w.hdr + H_HIST, nh, w.hscan, st));
    EmitOut eo{w.tiny, w.small, w.mid, LB, w.nxt, w.ident, w.bnd, w.ctr, w.scat, w.kinds, C.BM, C.TL, C.ET};
    constexpr u32 SPG = EmitShape<W>::SPG;
    if (nlarge.yes) k_emit<false, W><<<grid_of(nlarge.v, SPG, 1u << 30), 256, 0, st>>>(LA, w.tstart, nlp, w.hist, w.smin, w.smax, w.dig, w.split, eo);
    else k_emit<true, W><<<grid_of(n / 128, SPG, resident(k_emit<true, W>, 256)), 256, 0, st>>>(LA, w.tstart, nlp, w.hist, w.smin, w.smax, w.dig, w.split, eo);
    SS_CHECK_LAUNCH();
    {
        SS_PROF("k_scatter", st, (double)lelem * 24.0);  // key+payload in and out
        if (ltiles.yes) k_scatter<false, W><<<tg, NT, 0, st>>>(LA, w.tstart, nlp, C.TL, w.hist, w.scat, w.keyA, J.vals, w.keyB, w.valB, w.dig, w.split);
        else k_scatter<true, W><<<grid_of(n, C.TL, resident(k_scatter<true, W>, NT)), NT, 0, st>>>(LA, w.tstart, nlp, C.TL, w.hist, w.scat, w.keyA, J.vals, w.keyB, w.valB, w.dig, w.split);
    }
    SS_CHECK_LAUNCH();
    {
        SS_PROF("k_settle", st, (double)lelem * 8.0);  // at most the scattered keys read back
        if (ltiles.yes) k_settle<false, W><<<tg, NT, 0, st>>>(LA, w.tstart, nlp, C.TL, w.scat, w.kinds, w.keyB, w.valB, w.keyA, J.vals, w.dig, w.split);
        else k_settle<true, W><<<grid_of(n, C.TL, resident(k_settle<true, W>, NT)), NT, 0, st>>>(LA, w.tstart, nlp, C.TL, w.scat, w.kinds, w.keyB, w.valB, w.keyA, J.vals, w.dig, w.split);
    }
    SS_CHECK_LAUNCH();
    return SS_OK;
}

static int radix_level(RoundCtx &C, Seg *LA, Seg *LB, Known nlarge, Known ltiles, u64 lelem, bool wg = false)
{
    return C.W == 11 ? radix_level_w<11>(C, LA, LB, nlarge, ltiles, lelem, wg)
                     : radix_level_w<8>(C, LA, LB, nlarge, ltiles, lelem, wg);
}

// The part of a round after the radix levels: small sorts, boundary LCPs,
// equal strings.  h (when known) holds the counters after the last level.
static int round_tail(RoundCtx &C, const u32 *h, bool keyed = false)
{
    SortWs &w = C.w;
    const SortJob &J = C.J;
    hipStream_t st = J.stream;
    const u64 n = C.n;
    u32 *lcp = J.lcp;
    const bool known = h != nullptr;
    u32 *const elems = keyed ? w.ctr + C_NELEM : nullptr;  // members of the tied runs, where the caller counts them
    if (!known || h[C_TINY] > 0) {
        SS_PROF("k_wave_sort", st, known ? (double)h[C_TINYN] * 28.0 : 0.0);  // key+payload in/out, LCP out
        if (known && keyed)
            k_wave_sort<false, false><<<grid_of(h[C_TINY], WS_SPB, 1u << 30), 256, 0, st>>>(
                w.tiny, w.ctr + C_TINY, w.keyA, J.vals, w.keyB, w.valB, lcp, w.nxt, w.ctr, J.bytes, J.N, J.off, elems);
        else if (known)
            k_wave_sort<false><<<grid_of(h[C_TINY], WS_SPB, 1u << 30), 256, 0, st>>>(
                w.tiny, w.ctr + C_TINY, w.keyA, J.vals, w.keyB, w.valB, lcp, w.nxt, w.ctr, J.bytes, J.N, J.off, elems);
        else
            k_wave_sort<true><<<grid_of(n / 2, WS_SPB, resident(k_wave_sort<true>, 256)), 256, 0, st>>>(
                w.tiny, w.ctr + C_TINY, w.keyA, J.vals, w.keyB, w.valB, lcp, w.nxt, w.ctr, J.bytes, J.N, J.off, elems);
        SS_CHECK_LAUNCH();
    }
    if (!known || h[C_SMALL] > 0 || h[C_MID] > 0) {
        SS_PROF("k_block_sort", st, known ? (double)h[C_SMALLN] * 28.0 : 0.0);  // key+payload in/out, LCP out
        if (known) {
            if (h[C_SMALL])
                k_block_sort<false, BS_SMALL / BS_IPT><<<h[C_SMALL], BS_SMALL / BS_IPT, 0, st>>>(
                    w.small, w.ctr + C_SMALL, w.keyA, J.vals, w.keyB, w.valB, lcp, w.nxt, w.ctr, elems);
            if (h[C_MID])
                k_block_sort<false, BS_MID / BS_IPT><<<h[C_MID], BS_MID / BS_IPT, 0, st>>>(
                    w.mid, w.ctr + C_MID, w.keyA, J.vals, w.keyB, w.valB, lcp, w.nxt, w.ctr, elems);
        } else {
            const auto ks = k_block_sort<true, BS_SMALL / BS_IPT>;
            const auto km = k_block_sort<true, BS_MID / BS_IPT>;
            ks<<<grid_of(n, WS_MAX, resident(ks, BS_SMALL / BS_IPT)), BS_SMALL / BS_IPT, 0, st>>>(
                w.small, w.ctr + C_SMALL, w.keyA, J.vals, w.keyB, w.valB, lcp, w.nxt, w.ctr, elems);
            km<<<grid_of(n, BS_SMALL, resident(km, BS_MID / BS_IPT)), BS_MID / BS_IPT, 0, st>>>(
                w.mid, w.ctr + C_MID, w.keyA, J.vals, w.keyB, w.valB, lcp, w.nxt, w.ctr, elems);
        }
        SS_CHECK_LAUNCH();
    }
    if (!known || h[C_BND] > 0) {
        k_boundary<<<grid_of(known ? h[C_BND] : n, 256, 1024), 256, 0, st>>>(w.bnd, w.ctr + C_BND, w.keyA, lcp);
        SS_CHECK_LAUNCH();
    }
    if (!known || h[C_IDENT] > 0) {
        const u64 most = known ? h[C_IDENT] : n / 2;
        if (most <= LIST_ONE) {
            k_list_tiles<<<1, LIST_NT, 0, st>>>(w.ident, w.ctr + C_IDENT, C.ET, w.tstart);
            SS_CHECK_LAUNCH();
        } else {
            k_tile_counts<<<grid_of(most, 256, 1024), 256, 0, st>>>(w.ident, w.ctr + C_IDENT, C.ET, w.tstart, w.dscan);
            SS_CHECK_LAUNCH();
            SS_TRY(scan_u32(C, w.tstart, w.ctr + C_IDENT, most));
        }
        if (known)
            k_ident<false><<<grid_of(h[C_ITILES], 1, 1u << 30), NT, 0, st>>>(w.ident, w.tstart, w.ctr + C_IDENT, C.ET, lcp);
        else
            k_ident<true><<<grid_of(n, C.ET, resident(k_ident<true>, NT)), NT, 0, st>>>(w.ident, w.tstart, w.ctr + C_IDENT, C.ET, lcp);
        SS_CHECK_LAUNCH();
    }
    return SS_OK;
}

// The radix levels of a round, from the counters after its routing (h), which
// are read back after every level.
static int radix_levels(RoundCtx &C, u32 *h)
{
    Seg *LA = C.w.largeA, *LB = C.w.largeB;
    while (h[C_LARGE] > 0) {
        SS_TRY(radix_level(C, LA, LB, Known{true, h[C_LARGE]}, Known{true, h[C_LTILES]}, h[C_LELEM]));
        SS_TRY(ss_read_u32(C.w.ctr, h, C_NCTR, C.J.stream));
        Seg *tmp = LA; LA = LB; LB = tmp;
    }
    return SS_OK;
}

// Host-driven rounds: the host reads the counters once after the routing,
// once per radix level and once at the end of a round, sizes every grid from
// them and stops when no segment is unresolved.  The caller has put the first
// round's segments in w.act and their count, tiles and strings in
// ctr[C_NEXT], ctr[C_NTILES], ctr[C_NELEM].
// `whole`: one segment, set up by k_init_whole; what it is routed to is known
// without a read-back (but for the profile's count of prefix bytes).
int sort_rounds(const SortJob &J, SortWs &w, u32 nact, u32 atiles, bool whole)
{
    RoundCtx C = round_ctx(J, w);
    u32 h[C_NCTR];
    u64 round_elems = J.n_first;
    bool first = true;
    while (nact > 0) {
        SS_TRY(round_head(C, Known{true, nact}, Known{true, atiles}, round_elems, first, first ? C_NEXT : C_RNEXT,
                          first && whole));
        if (first && whole && J.n_total > C.BM && !g_prof_on) {
            memset(h, 0, sizeof(h));
            h[C_LARGE] = 1;
            h[C_LTILES] = (u32)ceil_div(J.n_total, C.TL);
            h[C_LELEM] = (u32)J.n_total;
            SS_TRY(radix_levels(C, h));
        } else if (first && whole && J.n_total <= C.BM) {
            memset(h, 0, sizeof(h));
            h[J.n_total <= WS_MAX ? C_TINY : (J.n_total <= BS_SMALL ? C_SMALL : C_MID)] = 1;
            h[J.n_total <= WS_MAX ? C_TINYN : C_SMALLN] = (u32)J.n_total;
        } else {
            SS_TRY(ss_read_u32(w.ctr, h, C_NCTR, J.stream));
            // (a seeded first round's common prefix was read by the pass that made the seed)
            if (!(first && J.seed_pos)) ss_prof_add_bytes("k_skip", (double)(h[10] | ((u64)h[11] << 32)));
            SS_TRY(radix_levels(C, h));
        }
        first = false;
        SS_TRY(round_tail(C, h));
        {
            // the tied runs compared directly; what is left goes back to the
            // first list (its segments are all done) as the next round's
            SS_PROF("k_resolve", J.stream, 0.0);  // (the number of runs is not known)
            k_resolve<<<grid_of(J.n_total / 2, 32, 2048), 256, 0, J.stream>>>(w.nxt, J.bytes, J.N, J.off, J.vals, J.lcp,
                                                                              w.act, w.ctr, C.ET);
        }
        SS_CHECK_LAUNCH();
        SS_TRY(ss_read_u32(w.ctr, h, C_NCTR, J.stream));
        ss_prof_add_bytes("k_resolve", (double)h[C_NEXT] * 40.0);  // offsets, payload of two; not the bytes compared
        nact = h[C_RNEXT];
        atiles = h[C_RTILES];
        round_elems = h[C_RELEM];
    }
    return SS_OK;
}

SortShape sort_shape(u64 n)
{
    const u32 bm = 2 * (u32)g_small_max;
    return SortShape{elem_tile(n), radix_tile(n), bm < BS_MID ? bm : (u32)BS_MID};
}

int sort_keyed(const SortJob &J, SortWs &w, u32 *h)
{
    RoundCtx C = round_ctx(J, w);
    SS_TRY(ss_read_u32(w.ctr, h, C_NCTR, J.stream));
    if (!(h[C_TINY] | h[C_SMALL] | h[C_MID] | h[C_LARGE])) return SS_OK;
    SS_TRY(radix_levels(C, h));
    SS_TRY(round_tail(C, h, true));
    return ss_read_u32(w.ctr, h, C_NCTR, J.stream);
}

// Device-driven rounds: `rounds` rounds of as many levels as a key has digits
// are enqueued with fixed grids and nothing is read back (the launch sequence
// can be captured in a graph); rounds and levels without work find empty
// lists.  hdr[H_REMAIN] receives the number of segments still unresolved
// afterwards (0: the sort is complete).
// Their tiles and members go to ctr, for a continuation by the host.
__global__ __launch_bounds__(1024) void k_remaining(u32 *ctr, u32 *hdr, u32 *status, const Seg *left, u32 et)
{
    __shared__ u32 s_tiles, s_elems;
    if (threadIdx.x == 0) s_tiles = s_elems = 0;
    __syncthreads();
    const u32 cnt = ctr[C_NEXT];
    u32 tiles = 0, elems = 0;
    for (u32 j = threadIdx.x; j < cnt; j += 1024) {
        const u32 m = left[j].end - left[j].begin;
        tiles += (m + et - 1) / et;
        elems += m;
    }
    if (elems) {
        atomicAdd(&s_tiles, tiles);
        atomicAdd(&s_elems, elems);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        ctr[C_NTILES] = s_tiles;
        ctr[C_NELEM] = s_elems;
        hdr[H_REMAIN] = cnt;
        if (status) *status = cnt;
    }
}

// The next round's segments back into the first list (after an odd number of
// rounds they are in the second), so that a continuation finds them there.
__global__ void k_copy_segs(const Seg *src, const u32 *cnt, Seg *dst)
{
    const u32 c = *cnt;
    GSTRIDE(j, c) dst[j] = src[j];
}

// (cont: the first round's segments are not the sets)
static int sort_rounds_device(const SortJob &J, SortWs &w, u32 rounds, u32 *status, u32 num_sets, bool cont)
{
    Seg *const act0 = w.act;
    RoundCtx C = round_ctx(J, w);
    // One workgroup per radix segment: in small sorts, or where the sets are small
    // on average, so that a segment too long for one is the exception.  One set
    // among small ones of 50, with all levels over the device and so: 300,000 random
    // strings 865 and 256 us, half of them sharing seven bytes 1132 and 396; 2M among
    // 300 sets 1047 and 441, 1271 and 796; 7M among 1,000 sets 2125 and 859, 2661 and
    // 1258.  (Where keys tie in pairs by the hundred thousand the next round, without
    // their direct comparison, can cost more than it gains: 2M strings, half of
    // them sharing three bytes, 1169 and 1877.)  (The list of radix segments must fit
    // one workgroup's pass to be split by size.)
    const bool wg = C.W == 8 && J.n_total / C.BM <= LIST_ONE &&
                    (J.n_total <= 16 * WG_MAX || J.n_total / num_sets <= WG_MAX / 4);
    const Known unknown{false, 0};
    for (u32 r = 0; r < rounds; r++) {
        const u32 levels = wg ? wg_levels(J.n_total) : (C.W == 11 ? Digits<11>::LEVELS : Digits<8>::LEVELS);
        SS_TRY(round_head(C, unknown, unknown, 0, false, C_NEXT, false, r || cont ? 0 : num_sets));
        Seg *LA = w.largeA, *LB = w.largeB;
        for (u32 l = 0; l < levels; l++) {
            SS_TRY(radix_level(C, LA, LB, unknown, unknown, 0, wg));
            Seg *tmp = LA; LA = LB; LB = tmp;
        }
        if (wg) {
            const EmitOut eo{w.tiny, w.small, w.mid, LB, w.nxt, w.ident, w.bnd, w.ctr, w.scat, w.kinds, C.BM, C.TL, C.ET};
            k_radix_wg<<<grid_of(J.n_total, C.BM + 1, resident(k_radix_wg, WG_NT)), WG_NT, 0, J.stream>>>(
                w.wgl, w.ctr + C_WG, LA, w.ctr + C_LARGE, LB, C.BM + 1, w.rmask, w.keyA, J.vals, w.keyB, w.valB, eo);
            SS_CHECK_LAUNCH();
        }
        SS_TRY(round_tail(C, nullptr));
        Seg *tmp = w.act; w.act = w.nxt; w.nxt = tmp;
    }
    k_remaining<<<1, 1024, 0, J.stream>>>(w.ctr, w.hdr, status, w.act, C.ET);
    SS_CHECK_LAUNCH();
    if (w.act != act0) {
        k_copy_segs<<<grid_of(J.n_total / 2, 256, 1024), 256, 0, J.stream>>>(w.act, w.ctr + C_NEXT, act0);
        SS_CHECK_LAUNCH();
    }
    return SS_OK;
}

// ------------------------------------------------------------ entry points

__global__ void k_iota(u32 *p, u32 n)
{
    u32 i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = i;
}

__global__ void k_zero_u32(u32 *p, u32 count)
{
    const u32 i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = 0;
}

// The whole array as the first round's one segment (n >= 2), its payload (input
// indices) and the round begun: its header, its tiles, the segment's skip minimum
// and varying bits.
__global__ void k_init_whole(SortWs w, u32 n, u32 *vals, u32 *lcp, u32 et)
{
    const u32 i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) vals[i] = i;
    if (i < C_NCTR) w.ctr[i] = 0;
    if (i == 0) {
        w.act[0] = Seg{0, n, 0, SEG_SKIP};
        w.hdr[H_ACT] = 1;
        w.tstart[0] = 0;
        w.tstart[1] = (n + et - 1) / et;
        w.skipv[0] = 0xFFFFFFFFu;
        w.keyB[0] = 0;
        lcp[0] = 0;
    }
}

// One segment per set of two or more strings (the counters are zero before).
// A set whose bounds are not well placed (set_off non-decreasing from 0 to n)
// raises ctr[C_BADSET] and writes nothing, so a malformed set_off never leads
// outside the arrays.
__global__ void k_init_sets(const u64 *set_off, u32 nsets, u64 n, Seg *act, u32 *ctr, u32 *lcp, u32 et)
{
    u32 j = blockIdx.x * blockDim.x + threadIdx.x;
    bool valid = j < nsets;
    u32 b = 0, e = 0;
    if (valid) {
        const u64 b64 = set_off[j], e64 = set_off[j + 1];
        if (e64 < b64 || e64 > n || (j == 0 && b64 != 0) || (j + 1 == nsets && e64 != n)) {
            atomicOr(&ctr[C_BADSET], 1u);
            valid = false;
        } else {
            b = (u32)b64;
            e = (u32)e64;
            if (e > b) lcp[b] = 0;
        }
    }
    bool two = valid && e > b + 1;
    u32 a = wave_append(two, &ctr[C_NEXT]);
    if (two) act[a] = Seg{b, e, 0, SEG_SKIP};
    wave_add(two ? (e - b + et - 1) / et : 0u, &ctr[C_NTILES]);
    wave_add(two ? e - b : 0u, &ctr[C_NELEM]);
}

// A malformed set_off found by k_init_sets leaves no segment to sort: every
// set's work is dropped (nothing is written beyond the initial identity).
__global__ void k_drop_if_bad(u32 *ctr, u32 *status)
{
    if (ctr[C_BADSET]) {
        ctr[C_NEXT] = 0;
        ctr[C_NTILES] = 0;
        ctr[C_NELEM] = 0;
    }
    if (status) status[1] = ctr[C_BADSET] ? 1u : 0u;
}

// Input indices within each set instead of the whole array, once the sort is
// complete (*remaining == 0; a sort left incomplete keeps global indices, as
// its continuation needs them).
//
// Bounded by 8 B per element.  A workgroup searches the set of its first element
// and its threads step on from there (25M elements of 512 sets: 72 us with a
// search per element, 22 so).
#define LOC_PER 8
__global__ __launch_bounds__(256) void k_localize(const u64 *set_off, u32 nsets, u32 n, u32 *perm,
                                                  const u32 *remaining)
{
    const u64 i0 = (u64)blockIdx.x * (256 * LOC_PER);
    if (remaining && *remaining) return;
    // largest j with set_off[j] <= i0 (uniform over the workgroup)
    u32 lo = 0, hi = nsets;
    while (hi - lo > 1) {
        const u32 mid = (lo + hi) >> 1;
        if (set_off[mid] <= i0) lo = mid;
        else hi = mid;
    }
    u64 from = set_off[lo], to = lo + 1 < nsets ? set_off[lo + 1] : n;
    u32 v[LOC_PER];
#pragma unroll
    for (u32 q = 0; q < LOC_PER; q++) {
        const u64 i = i0 + q * 256 + threadIdx.x;
        v[q] = i < n ? perm[i] : 0u;
    }
#pragma unroll
    for (u32 q = 0; q < LOC_PER; q++) {
        const u64 i = i0 + q * 256 + threadIdx.x;
        if (i >= n) break;
        if (i >= to) {  // another set: the largest j with set_off[j] <= i
            u32 b = nsets;
            while (b - lo > 1) {
                const u32 mid = (lo + b) >> 1;
                if (set_off[mid] <= i) lo = mid;
                else b = mid;
            }
            from = set_off[lo];
            to = lo + 1 < nsets ? set_off[lo + 1] : n;
        }
        perm[i] = v[q] - (u32)from;
    }
}

extern "C" size_t ss_sort_workspace(uint64_t n)
{
    WsCounter c;
    SortWs w;
    sort_ws_layout(n, &w, nullptr, &c);
    return c.used;
}

static int sort_common_checks(const uint8_t *bytes, const uint64_t *offsets, uint64_t n, uint32_t *perm)
{
    if (n >= 0xFFFFFFFFull) {
        ss_set_error("n = %llu exceeds the 32-bit index limit", (unsigned long long)n);
        return SS_ERR_TOO_LARGE;
    }
    if (n > 0 && (!offsets || !perm)) {
        ss_set_error("null offsets or perm");
        return SS_ERR_INVALID_ARG;
    }
    (void)bytes;
    return SS_OK;
}

// Few strings (n <= RANK_MAX): one launch, no rounds.  Block i ranks string i
// among all others, (string, index) order: rank = #{ j : s_j < s_i, or s_j =
// s_i and j < i }.  The LCP with the predecessor in sorted order is the largest
// LCP of s_i with any string ranked before it (LCPs along a sorted sequence
// are range minima of the adjacent ones).
//
// Bounded by the launch and the latency of two dependent reads (offsets, bytes):
// a wavefront reads the offsets of all its strings at once, then the first 512
// bytes of RANK_Q strings side by side, 8 bytes a lane; strings that agree
// further are compared from there one by one.  48 strings: 8.4 us with 8
// wavefronts and one string after the other, 5.2 us so.
#define RANK_MAX 256
#define RANK_NT 1024
#define RANK_Q 4
__global__ __launch_bounds__(RANK_NT) void k_rank_sort(const u8 *bytes, u64 N, const u64 *off, u32 n, u32 *perm,
                                                       u32 *lcp)
{
    constexpr u32 NW = RANK_NT / 64;
    __shared__ u32 s_cnt[NW], s_max[NW];
    const u32 i = blockIdx.x;
    const u32 lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    // the wavefront's strings j = wv, wv + NW, ...: lane k holds the k-th's bounds
    const u32 jl = wv + lane * NW;
    const u64 ol = jl < n ? off[jl] : 0ull, ll = jl < n ? off[jl + 1] - ol : 0ull;
    const u64 oi = off[i], li = off[i + 1] - oi;
    const u32 at = 8 * lane;
    auto take = [&](u64 len) { return len > at ? (len - at < 8 ? (u32)(len - at) : 8u) : 0u; };
    const u64 wi = load_be(bytes, N, oi + at, take(li));
    u32 cnt = 0, mx = 0;
    for (u32 k0 = 0; wv + k0 * NW < n; k0 += RANK_Q) {  // (uniform over the wavefront)
        u64 oj[RANK_Q], lj[RANK_Q], wj[RANK_Q];
#pragma unroll
        for (u32 q = 0; q < RANK_Q; q++) {
            oj[q] = __shfl(ol, k0 + q, 64);
            lj[q] = __shfl(ll, k0 + q, 64);  // (0 past the last)
            wj[q] = load_be(bytes, N, oj[q] + at, take(lj[q]));
        }
#pragma unroll
        for (u32 q = 0; q < RANK_Q; q++) {
            const u32 j = wv + (k0 + q) * NW;
            if (j >= n || j == i) continue;  // (uniform)
            const u64 m = li < lj[q] ? li : lj[q];
            const u64 diff = __ballot(wi != wj[q]);
            u64 l = m;
            int c = lj[q] < li ? -1 : (lj[q] > li ? 1 : 0);
            u64 p = ~0ull;  // first differing byte of the first 512, zeros past an end
            u64 a = 0, b = 0;
            if (diff) {
                const u32 f = (u32)__ffsll((unsigned long long)diff) - 1;
                a = __shfl(wi, f, 64);
                b = __shfl(wj[q], f, 64);
                p = 8 * f + ((u32)__clzll(a ^ b) >> 3);
            }
            if (p < m) {
                l = p;
                c = b < a ? -1 : 1;
            } else if (m > 512) {
                c = wave_str_cmp(bytes, N, oj[q] + 512, lj[q] - 512, oi + 512, li - 512, &l);
                l += 512;
            }
            if (c < 0 || (c == 0 && j < i)) {
                cnt++;
                if (l > mx) mx = (u32)l;
            }
        }
    }
    if (lane == 0) { s_cnt[wv] = cnt; s_max[wv] = mx; }
    __syncthreads();
    if (wv == 0) {
        u32 r = lane < NW ? s_cnt[lane] : 0u, m = lane < NW ? s_max[lane] : 0u;
#pragma unroll
        for (u32 d = 1; d < NW; d <<= 1) {
            r += __shfl_xor(r, d, 64);
            const u32 y = __shfl_xor(m, d, 64);
            m = y > m ? y : m;
        }
        if (lane == 0) {
            perm[r] = i;
            if (lcp) lcp[r] = m;
        }
    }
}

// The first-round seed's arrays (layout: 256-byte header whose word 0 says
// whether the seed was written, the mismatch words (n), the records (n)).
static void attach_seed(SortJob &J, void *seed, u64 n)
{
    J.seed_ok = (const u32 *)seed;
    J.seed_word = (u64 *)((u8 *)seed + 256);
    J.seed_pos = (uint2 *)((u8 *)seed + 256 + 8 * n);
}

static int sort_single(const uint8_t *bytes, uint64_t N, const uint64_t *offsets, uint64_t n, void *seed,
                       uint32_t *perm, uint32_t *lcp, void *ws, size_t ws_bytes, void *stream)
{
    SS_TRY(sort_common_checks(bytes, offsets, n, perm));
    if (n == 0) return SS_OK;
    hipStream_t st = (hipStream_t)stream;
    WsArena a(ws, ws_bytes);
    SortWs w;
    sort_ws_layout(n, &w, &a, nullptr);
    if (a.overflow || !ws) {
        ss_set_error("workspace too small: need %zu bytes", ss_sort_workspace(n));
        return SS_ERR_WORKSPACE;
    }
    if (n <= RANK_MAX) {
        k_rank_sort<<<(unsigned)n, RANK_NT, 0, st>>>(bytes, N, offsets, (u32)n, perm, lcp);
        SS_CHECK_LAUNCH();
        return SS_OK;
    }
    SortJob J{bytes, N, offsets, perm, lcp ? lcp : w.lcp_scratch, st, n, n};
    if (seed) attach_seed(J, seed, n);
    // One segment: the first round begins in the launch that writes the indices,
    // and its one routing is known (1,000 text strings: 8 launches and one
    // read-back instead of 22 and four; 100,000 D/N strings 103 us instead of 111).
    const u32 et = elem_tile(n);
    k_init_whole<<<(unsigned)ceil_div(n, 256), 256, 0, st>>>(w, (u32)n, perm, J.lcp, et);
    SS_CHECK_LAUNCH();
    return sort_rounds(J, w, 1, (u32)ceil_div(n, et), true);
}

extern "C" int ss_sort(const uint8_t *bytes, uint64_t N, const uint64_t *offsets, uint64_t n,
                       uint32_t *perm, uint32_t *lcp, void *ws, size_t ws_bytes, void *stream)
{
    ss_clear_error();
    return sort_single(bytes, N, offsets, n, nullptr, perm, lcp, ws, ws_bytes, stream);
}

extern "C" int ss_sort_seeded(const uint8_t *bytes, uint64_t N, const uint64_t *offsets, uint64_t n,
                              void *sort_seed, uint32_t *perm, uint32_t *lcp, void *ws, size_t ws_bytes,
                              void *stream)
{
    ss_clear_error();
    if (!sort_seed) {
        ss_set_error("null sort_seed");
        return SS_ERR_INVALID_ARG;
    }
    return sort_single(bytes, N, offsets, n, sort_seed, perm, lcp, ws, ws_bytes, stream);
}

// The checks and first-round set-up shared by both batch forms.
static int batch_setup(const uint8_t *bytes, uint64_t N, const uint64_t *offsets, uint64_t n,
                       const uint64_t *set_off, uint32_t num_sets, uint32_t *perm, uint32_t *lcp, uint32_t flags,
                       void *ws, size_t ws_bytes, hipStream_t st, SortWs &w, SortJob &J)
{
    SS_TRY(sort_common_checks(bytes, offsets, n, perm));
    if (num_sets == 0 || !set_off) {
        ss_set_error("batch needs num_sets >= 1 and set_off");
        return SS_ERR_INVALID_ARG;
    }
    if (flags & ~(SS_BATCH_GLOBAL_IDS | SS_BATCH_CONTINUE)) {
        ss_set_error("unknown flags 0x%x", flags);
        return SS_ERR_INVALID_ARG;
    }
    if (n == 0) return SS_OK;
    WsArena a(ws, ws_bytes);
    sort_ws_layout(n, &w, &a, nullptr);
    if (a.overflow || !ws) {
        ss_set_error("workspace too small: need %zu bytes", ss_sort_workspace(n));
        return SS_ERR_WORKSPACE;
    }
    J = SortJob{bytes, N, offsets, perm, lcp ? lcp : w.lcp_scratch, st, 0, n};
    if (flags & SS_BATCH_CONTINUE) return SS_OK;  // the state of an incomplete device-driven sort
    k_iota<<<(unsigned)ceil_div(n, 256), 256, 0, st>>>(perm, (u32)n);
    SS_CHECK_LAUNCH();
    k_zero_u32<<<1, 64, 0, st>>>(w.ctr, C_NCTR);
    SS_CHECK_LAUNCH();
    k_init_sets<<<(unsigned)ceil_div(num_sets, 256), 256, 0, st>>>(set_off, num_sets, n, w.act, w.ctr, J.lcp,
                                                                     elem_tile(n));
    SS_CHECK_LAUNCH();
    return SS_OK;
}

static int sort_batch_impl(const uint8_t *bytes, uint64_t N, const uint64_t *offsets, uint64_t n,
                           const uint64_t *set_off, uint32_t num_sets, void *seed, uint32_t *perm_local,
                           uint32_t *lcp, uint32_t flags, void *ws, size_t ws_bytes, void *stream)
{
    hipStream_t st = (hipStream_t)stream;
    SortWs w;
    SortJob J{};
    SS_TRY(batch_setup(bytes, N, offsets, n, set_off, num_sets, perm_local, lcp, flags, ws, ws_bytes, st, w, J));
    if (n == 0) return SS_OK;
    if (seed) attach_seed(J, seed, n);
    u32 h[C_NCTR];
    SS_TRY(ss_read_u32(w.ctr, h, C_NCTR, st));
    if (h[C_BADSET]) {
        ss_set_error("set_off must be non-decreasing with set_off[0] = 0 and set_off[num_sets] = n");
        return SS_ERR_INVALID_ARG;
    }
    J.n_first = h[C_NELEM];
    SS_TRY(sort_rounds(J, w, h[C_NEXT], h[C_NTILES]));
    if (!(flags & SS_BATCH_GLOBAL_IDS)) {
        k_localize<<<(unsigned)ceil_div(n, 256 * LOC_PER), 256, 0, st>>>(set_off, num_sets, (u32)n, perm_local, nullptr);
        SS_CHECK_LAUNCH();
    }
    return SS_OK;
}

extern "C" int ss_sort_batch(const uint8_t *bytes, uint64_t N, const uint64_t *offsets, uint64_t n,
                             const uint64_t *set_off, uint32_t num_sets, uint32_t *perm_local,
                             uint32_t *lcp, uint32_t flags, void *ws, size_t ws_bytes, void *stream)
{
    ss_clear_error();
    return sort_batch_impl(bytes, N, offsets, n, set_off, num_sets, nullptr, perm_local, lcp, flags, ws, ws_bytes,
                           stream);
}

extern "C" int ss_sort_batch_seeded(const uint8_t *bytes, uint64_t N, const uint64_t *offsets, uint64_t n,
                                    const uint64_t *set_off, uint32_t num_sets, void *sort_seed,
                                    uint32_t *perm_local, uint32_t *lcp, uint32_t flags, void *ws,
                                    size_t ws_bytes, void *stream)
{
    ss_clear_error();
    if (!sort_seed || (flags & SS_BATCH_CONTINUE)) {
        ss_set_error(!sort_seed ? "null sort_seed" : "a seeded sort cannot continue a device-driven one");
        return SS_ERR_INVALID_ARG;
    }
    return sort_batch_impl(bytes, N, offsets, n, set_off, num_sets, sort_seed, perm_local, lcp, flags, ws,
                           ws_bytes, stream);
}

extern "C" uint32_t ss_sort_batch_device_rounds(uint32_t max_len)
{
    // a round consumes at least 7 bytes of every string it keeps
    return max_len / 7 + 2;
}

extern "C" int ss_sort_batch_device(const uint8_t *bytes, uint64_t N, const uint64_t *offsets, uint64_t n,
                                    const uint64_t *set_off, uint32_t num_sets, uint32_t *perm_local,
                                    uint32_t *lcp, uint32_t flags, uint32_t rounds, uint32_t *status, void *ws,
                                    size_t ws_bytes, void *stream)
{
    ss_clear_error();
    if (!status) {
        ss_set_error("status is required");
        return SS_ERR_INVALID_ARG;
    }
    if (rounds == 0 || rounds > 1024) {
        ss_set_error("rounds must be 1..1024");
        return SS_ERR_INVALID_ARG;
    }
    hipStream_t st = (hipStream_t)stream;
    SortWs w;
    SortJob J{};
    SS_TRY(batch_setup(bytes, N, offsets, n, set_off, num_sets, perm_local, lcp, flags, ws, ws_bytes, st, w, J));
    if (n == 0) {
        k_zero_u32<<<1, 64, 0, st>>>(status, 2);
        SS_CHECK_LAUNCH();
        return SS_OK;
    }
    if (!(flags & SS_BATCH_CONTINUE)) {
        k_drop_if_bad<<<1, 1, 0, st>>>(w.ctr, status);
        SS_CHECK_LAUNCH();
    }
    SS_TRY(sort_rounds_device(J, w, rounds, status, num_sets, flags & SS_BATCH_CONTINUE));
    if (!(flags & SS_BATCH_GLOBAL_IDS)) {
        k_localize<<<(unsigned)ceil_div(n, 256 * LOC_PER), 256, 0, st>>>(set_off, num_sets, (u32)n, perm_local,
                                                               w.ctr + C_NEXT);
        SS_CHECK_LAUNCH();
    }
    return SS_OK;
}

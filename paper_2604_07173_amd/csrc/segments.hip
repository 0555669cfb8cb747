// Segment builder: stable counting sort of the batch rows by key = adapter * E + expert,
// then segment boundaries and row tiles (App. A.2.2: rows of one adapter are aggregated so its
// weights are read once; Sec. 2.3: per (adapter, expert) in MoE layers).  One workgroup of
// 1024 threads does the whole job out of LDS (a batch has at most 16384 rows and the result
// feeds kernels that run right after it, so latency matters, not bandwidth; gfx950 has
// 160 KiB of LDS per workgroup).  Global memory is only read for the ids and only written for
// the results.  One CU issues one wave instruction per four cycles and SIMD, so the time of
// any path below is essentially its instruction count.
//
// Three paths with identical results (rows ordered by key, original order inside a key):
//
// * At most 4096 rows over at most 256 keys (segments_small_kernel): described at the kernel.
//
// * Radix path (segments_kernel; long segments, or key spaces too large for LDS counters).
//   LDS holds key[row] for the whole batch and two 16-bit row-index arrays that the radix
//   passes (8 key bits each, least significant first) ping-pong between; the keys never move.
//   Stability without order-defining atomics: in every pass wave w owns the contiguous
//   positions [w*CH, (w+1)*CH) of the current order; it walks them 64 at a time in order,
//   ranks equal digits inside a group of 64 by lane order (ballot match) and keeps a running
//   per-digit count of its own (LDS adds whose only effect is a sum, so their order does not
//   matter); an exclusive scan over (digit, wave) in digit-major order turns the counts into
//   start positions.  With a single pass (at most 256 keys) the scanned histogram already is
//   the segment table.  Otherwise thread t owns `items` consecutive sorted positions and keeps
//   the boundary flags of its positions as a bit mask; three block scans (count of
//   boundaries, last boundary before, first boundary after) give every position its segment
//   index, start and end without reading anything back from global memory.
//
// * Counting path (segments_bucket_kernel; many short segments): described at the kernel.
#include <cstdlib>

#include "segments_inline.h"

namespace lora {

namespace {

constexpr int kThreads = kSegThreads;
constexpr int kWaves = kSegWaves;
constexpr int kBins = kSegBins;
constexpr int kMaxItems = LORA_MAX_ROWS / kThreads;   // positions per thread, fits a 32-bit mask
static_assert(kMaxItems <= 32, "boundary flags are kept in a 32-bit mask");

struct ScanLds {
    int sum[kWaves];
    int mx[kWaves];
    int mn[kWaves];
    unsigned two[kWaves][2];
};

// three scans with one pair of barriers: exclusive sum of `cnt` (and total), exclusive
// running max of `last` over earlier threads, exclusive running min of `first` over later
// threads
__device__ inline void block_scan3(int cnt, int last, int first, ScanLds *s,
                                   int *cnt_before, int *cnt_total, int *last_before,
                                   int *first_after)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int isum = cnt, imax = last, imin = first;
#pragma unroll 1
    for (int o = 1; o < 64; o <<= 1) {
        const int a = __shfl_up(isum, o, 64), b = __shfl_up(imax, o, 64);
        const int c = __shfl_down(imin, o, 64);
        if (lane >= o) {
            isum += a;
            imax = max(imax, b);
        }
        if (lane + o < 64) imin = min(imin, c);
    }
    __syncthreads();
    if (lane == 63) {
        s->sum[w] = isum;
        s->mx[w] = imax;
    }
    if (lane == 0) s->mn[w] = imin;
    __syncthreads();
    // lane k < 16 fetches wave k's values; a 16-lane butterfly combines them
    const bool in = lane < kWaves;
    const int a = in ? s->sum[lane] : 0, b = in ? s->mx[lane] : -1, c = in ? s->mn[lane] : 0x7FFFFFFF;
    int tot = a, base = lane < w ? a : 0, mx = lane < w ? b : -1, mn = lane > w ? c : 0x7FFFFFFF;
#pragma unroll 1
    for (int o = 8; o > 0; o >>= 1) {
        tot += __shfl_xor(tot, o, 64);
        base += __shfl_xor(base, o, 64);
        mx = max(mx, __shfl_xor(mx, o, 64));
        mn = min(mn, __shfl_xor(mn, o, 64));
    }
    tot = __shfl(tot, 0, 64);
    base = __shfl(base, 0, 64);
    mx = __shfl(mx, 0, 64);
    mn = __shfl(mn, 0, 64);
    // exclusive within the wave: take the neighbour's inclusive value
    const int pmax = __shfl_up(imax, 1, 64), nmin = __shfl_down(imin, 1, 64);
    *cnt_before = base + isum - cnt;
    *cnt_total = tot;
    *last_before = lane > 0 ? max(mx, pmax) : mx;
    *first_after = lane < 63 ? min(mn, nmin) : mn;
}

// key_of[i] for the calling thread's rows; returns how many have a key.  The id loads of up to eight
// rows are issued before the first is used (the ids come from HBM; one round trip per row
// would otherwise dominate large batches).
__device__ inline int all_row_keys(const SegParams &p, unsigned *key_of, unsigned &bad)
{
    constexpr int U = 8;
    const int tid = threadIdx.x;
    int n_active = 0;
#pragma unroll 1
    for (int i0 = tid; i0 < p.P; i0 += U * kThreads) {
        int a[U], e[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * kThreads;
            a[u] = -1;
            e[u] = 0;
            if (i < p.P) {
                a[u] = p.adapter_id[i];
                if (p.expert_id) e[u] = p.expert_id[i];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * kThreads;
            if (i < p.P) {
                const unsigned k = row_key(p, a[u], e[u], bad);
                key_of[i] = k;
                n_active += k != kNoKey ? 1 : 0;
            }
        }
    }
    return n_active;
}

// The radix path, whole: passes, boundaries, tiles, counts.  put_keys(key_of, bad) writes the keys of the calling thread's
// rows and returns how many have one.
template <class PutKeys>
__device__ __forceinline__ void radix_body(const SegParams &p, PutKeys put_keys)
{
    __shared__ unsigned hist[kWaves][kBins];
    __shared__ ScanLds scan;
    __shared__ unsigned status_bits;
    __shared__ int n_active_total;
    extern __shared__ __attribute__((aligned(16))) unsigned char dyn_lds[];

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int P = p.P;
    const int P_pad = (P + 63) & ~63;
    unsigned *key_of = reinterpret_cast<unsigned *>(dyn_lds);                    // [P_pad]
    uint16_t *order[2] = {reinterpret_cast<uint16_t *>(key_of + P_pad),          // [P_pad] each
                          reinterpret_cast<uint16_t *>(key_of + P_pad) + P_pad};
    const unsigned n_keys = (unsigned)p.n_adapters * (unsigned)p.n_experts;
    const int items = (P + kThreads - 1) / kThreads;       // 64-row groups per wave
    const int wave_base = w * items * 64;
    const bool park = n_keys <= 0x10000u;                  // room for a 16-bit rank above the key
    const unsigned key_mask = park ? 0xFFFFu : 0xFFFFFFFFu;

    if (tid == 0) {
        status_bits = 0;
        n_active_total = 0;
    }
    for (int b = tid; b < kWaves * kBins; b += kThreads) (&hist[0][0])[b] = 0;
    __syncthreads();

    // ---- key of every row ------------------------------------------------------------------
    {
        unsigned bad = 0;
        int n_active = put_keys(key_of, bad);
        if (bad) atomicOr(&status_bits, bad);          // OR and + are order-independent
#pragma unroll 1
        for (int o = 32; o > 0; o >>= 1) n_active += __shfl_xor(n_active, o, 64);
        if (lane == 0 && n_active) atomicAdd(&n_active_total, n_active);
    }
    __syncthreads();
    const int P_act = n_active_total;

    // ---- radix passes over the row order ----------------------------------------------
    for (int pass = 0; pass < p.passes; ++pass) {
        const int shift = 8 * pass;
        const int nbits = min(8, p.key_bits - shift);      // digit bits that can be set
        const bool last = pass == p.passes - 1;
        const int n_in = pass == 0 ? P : P_act;            // pass 0 leaves the rows without adapter out
        const uint16_t *src = order[(pass + 1) & 1];   // unused in pass 0 (identity order)
        uint16_t *dst = order[pass & 1];
        unsigned *my_hist = hist[w];

        // count: rank of every element among the equal digits of its wave; when keys fit
        // 16 bits the rank is parked in the upper half of the key word for the scatter
#pragma unroll 1
        for (int g = 0; g < items; ++g) {
            const int i = wave_base + g * 64 + lane;
            const bool in = i < n_in;
            const unsigned row = in ? (pass == 0 ? (unsigned)i : (unsigned)src[i]) : 0u;
            const unsigned kfull = in ? key_of[row] : kNoKey;
            const bool val = in && (pass != 0 || kfull != kNoKey);
            const unsigned k = val ? kfull & key_mask : 0u;
            const unsigned dig = (k >> shift) & 255u;
            const Match m = match_digit(dig, val, nbits);
            const unsigned below = lanes_below(m);
            // every lane reads the digit's running count before the leader advances it; LDS
            // operations of one wave execute in program order
            const unsigned first = *(volatile unsigned *)&my_hist[dig];
            if (val && park) key_of[row] = k | ((first + below) << 16);
            __builtin_amdgcn_wave_barrier();
            if (val && below == 0) my_hist[dig] = first + __popc(m.lo) + __popc(m.hi);
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        // exclusive scan over (digit, wave), digit-major: thread t owns digit t/4 and waves
        // 4*(t%4) .. 4*(t%4)+3
        {
            const int bin = tid >> 2, w0 = (tid & 3) * 4;
            const unsigned c0 = hist[w0][bin], c1 = hist[w0 + 1][bin], c2 = hist[w0 + 2][bin],
                           c3 = hist[w0 + 3][bin];
            int tot;
            const unsigned base = (unsigned)block_excl_sum((int)(c0 + c1 + c2 + c3), &tot, scan.sum);
            hist[w0][bin] = base;
            hist[w0 + 1][bin] = base + c0;
            hist[w0 + 2][bin] = base + c0 + c1;
            hist[w0 + 3][bin] = base + c0 + c1 + c2;
        }
        __syncthreads();
        // scatter: position = start of (digit, wave) + rank within it
#pragma unroll 1
        for (int g = 0; g < items; ++g) {
            const int i = wave_base + g * 64 + lane;
            const bool in = i < n_in;
            const unsigned row = in ? (pass == 0 ? (unsigned)i : (unsigned)src[i]) : 0u;
            const unsigned kfull = in ? key_of[row] : kNoKey;
            const bool val = in && (pass != 0 || kfull != kNoKey);
            const unsigned kw = val ? kfull : 0u;
            const unsigned dig = ((kw & key_mask) >> shift) & 255u;
            unsigned pos;
            if (park) {
                pos = my_hist[dig] + (kw >> 16);
            } else {
                const Match m = match_digit(dig, val, nbits);
                const unsigned below = lanes_below(m);
                const unsigned first = *(volatile unsigned *)&my_hist[dig];
                pos = first + below;
                __builtin_amdgcn_wave_barrier();
                if (val && below == 0) my_hist[dig] = first + __popc(m.lo) + __popc(m.hi);
                __builtin_amdgcn_wave_barrier();
            }
            if (val) {
                if (p.passes > 1) dst[pos] = (uint16_t)row;       // one pass: nothing reads the order back
                if (last) p.perm[pos] = (int32_t)row;
            }
        }
        __syncthreads();
        if (!last) {
            for (int b = tid; b < kWaves * kBins; b += kThreads) (&hist[0][0])[b] = 0;
            __syncthreads();
        }
    }
    const int TR = p.tile_rows;       // a power of two

    // ---- one pass (at most 256 keys): the scanned histogram already is the segment table ----
    if (p.passes == 1) {
        __shared__ unsigned bin_tile0[kBins];     // first tile of the key (exclusive prefix)
        __shared__ unsigned bin_seg[kBins];       // segment index of the key
        const int tr_shift = 31 - __clz(TR);
        unsigned start = 0, n = 0;
        if (tid < kBins) {
            start = hist[0][tid];                                  // wave 0's start = the key's start
            n = (tid + 1 < kBins ? hist[0][tid + 1] : (unsigned)P_act) - start;
        }
        const unsigned my_tiles = (n + TR - 1) >> tr_shift;
        unsigned seg_before, tile_before, S, n_tiles;
        block_excl_sum2(n ? 1u : 0u, my_tiles, scan.two, &seg_before, &tile_before, &S, &n_tiles);
        if (tid < kBins) {
            bin_tile0[tid] = tile_before;
            bin_seg[tid] = seg_before;
            if (n) {
                p.seg_start[seg_before] = (int32_t)start;
                p.seg_key[seg_before] = tid;
            }
        }
        __syncthreads();
        // tiles, one per thread and turn: the key of tile ti is the last one whose first tile
        // is not beyond ti (an empty key shares its first tile with the next key, which wins)
#pragma unroll 1
        for (unsigned ti = tid; ti < n_tiles; ti += kThreads) {
            int key = 0;
#pragma unroll
            for (int step = kBins / 2; step > 0; step >>= 1)
                if (bin_tile0[key + step] <= ti) key += step;
            const unsigned kstart = hist[0][key];
            const unsigned kend = key + 1 < kBins ? hist[0][key + 1] : (unsigned)P_act;
            const unsigned r = (ti - bin_tile0[key]) << tr_shift;
            lora_tile t;
            t.key = key;
            t.row0 = (int32_t)(kstart + r);
            t.n_rows = (int32_t)min((unsigned)TR, kend - kstart - r);
            t.seg = (int32_t)bin_seg[key];
            p.tiles[ti] = t;
        }
        if (tid == 0) {
            p.seg_start[S] = P_act;
            p.counts[0] = (int32_t)S;
            p.counts[1] = P_act;
            p.counts[2] = (int32_t)n_tiles;
            p.counts[3] = 0;
            p.status[0] = status_bits;
        }
        return;
    }
    const uint16_t *sorted = order[(p.passes - 1) & 1];

    // ---- segment boundaries of my positions as a bit mask --------------------------------
    const int i0 = tid * items;
    unsigned F = 0;
    {
        unsigned prev = (i0 > 0 && i0 - 1 < P_act) ? (key_of[sorted[i0 - 1]] & key_mask) : 0xFFFFFFFFu;
        for (int q = 0; q < items; ++q) {
            const int i = i0 + q;
            if (i >= P_act) break;
            const unsigned k = key_of[sorted[i]] & key_mask;
            if (i == 0 || k != prev) F |= 1u << q;
            prev = k;
        }
    }
    const int my_last = F ? i0 + 31 - __clz(F) : -1;
    const int my_first = F ? i0 + __ffs(F) - 1 : 0x7FFFFFFF;
    int seg_before, S, start_before, next_after;
    block_scan3(__popc(F), my_last, my_first, &scan, &seg_before, &S, &start_before, &next_after);
    next_after = min(next_after, P_act);

    // ---- segment records and tile starts -------------------------------------------------
    unsigned T = 0;                   // tile starts among my positions
    {
        int sidx = seg_before;
        int seg_begin = start_before;
        for (int q = 0; q < items; ++q) {
            const int i = i0 + q;
            if (i >= P_act) break;
            if (F & (1u << q)) {
                seg_begin = i;
                p.seg_start[sidx] = i;
                p.seg_key[sidx] = (int32_t)(key_of[sorted[i]] & key_mask);
                ++sidx;
            }
            if (((i - seg_begin) & (TR - 1)) == 0) T |= 1u << q;
        }
    }
    if (tid == 0) p.seg_start[S] = P_act;
    int n_tiles;
    int tix = block_excl_sum(__popc(T), &n_tiles, scan.sum);
    for (unsigned rest = T; rest; rest &= rest - 1) {
        const int q = __ffs(rest) - 1;
        const int i = i0 + q;
        const unsigned above = q >= 31 ? 0u : F & (0xFFFFFFFEu << q);      // boundaries after i
        const int seg_end = above ? i0 + __ffs(above) - 1 : next_after;
        lora_tile t;
        t.key = (int32_t)(key_of[sorted[i]] & key_mask);
        t.row0 = i;
        t.n_rows = min(TR, seg_end - i);
        t.seg = seg_before + __popc(F & (0xFFFFFFFFu >> (31 - q))) - 1;
        p.tiles[tix++] = t;
    }
    if (tid == 0) {
        p.counts[0] = S;
        p.counts[1] = P_act;
        p.counts[2] = n_tiles;
        p.counts[3] = 0;
        p.status[0] = status_bits;
    }
}

__global__ __launch_bounds__(kThreads) void segments_kernel(SegParams p)
{
    radix_body(p, [&](unsigned *key_of, unsigned &bad) { return all_row_keys(p, key_of, bad); });
}

// ---- few keys, a few thousand rows -----------------------------------------------------------
// The sort that small batches do inside the first shrink (segments_inline.h), by one workgroup of sixteen waves: the
// groups of 64 rows of a wave are matched bit by bit together, where the radix path takes them one after the
// other and waits for the running count between them.  What is left is mostly that match (one workgroup's instructions).
// Back to back in a graph, before (radix or bucket path) / now: 64 rows 5.4 / 3.2 us, 1024 rows over 256 keys 6.4 /
// 3.5, 2048 8.0 / 4.3, 4096 10.6 / 5.8, 4096 rows of 8 requests 9.1 / 5.1; four threads per key for the sums over
// the groups: no change.
constexpr int kSmallMaxRows = 4096;
constexpr int kSmallGroups = kSmallMaxRows / 64;

template <int GROUPS, int TR>
__global__ __launch_bounds__(kThreads) void segments_small_kernel(SegParams p)
{
    __shared__ SortCounts<GROUPS> counts;
    __shared__ SortedSegments<64 * GROUPS, false> sorted;
    build_segments_inline_n<kWaves, GROUPS, TR>(p, counts, sorted, true);
}

template <int GROUPS, int TR>
void launch_small(const SegParams &p, hipStream_t s)
{
    hipLaunchKernelGGL((segments_small_kernel<GROUPS, TR>), dim3(1), dim3(kThreads), 0, s, p);
}

// ---- bucket path ---------------------------------------------------------------------------
// For batches of many short segments (decode): one LDS counter per key instead of radix
// passes over the key bits.
//   1. count the rows of every key with fetching LDS adds; what an add returns is the row's place among its key's
//      rows, which depends on the order the adds execute in (hence step 4);
//   2. thread t owns a contiguous range of keys: an exclusive scan over the counts gives every range its first row, segment
//      and tile; the keys that occur are the segments, so they are listed in LDS
//      and the segment records and tiles are then written one segment per thread;
//   3. every row goes to its place in its key's range;
//   4. every row is re-ranked inside its bucket by the number of rows of the bucket with a
//      smaller row index: the final order is by (key, row index), unique, hence bit-identical
//      run to run and identical to the stable sort of the radix path.
// Step 4 costs bucket length per row, and a counter has 8 bits: if one key holds more than 255 rows the
// workgroup drops this attempt and runs the radix path on the keys it has (a workgroup-uniform decision).  What a dropped attempt costs
// is seen only where the radix path was taken at once before the counters had 8 bits (65536 keys and 1025 to 11200 rows,
// 32768 keys from 8960, 16384 from 12800 on): a zipf batch of 4097 rows over 65536 keys 21.1 -> 23.1 us, 290 of 12288 rows
// on one of 32768 keys 49.0 -> 51.1, all of them 35.5 -> 45.9; against that 23.1 -> 11.1 and 49.5 -> 11.4 where the counts do.
//
// Longer batches are launched with several workgroups.  Step 1 and the sums of step 2 are repeated by every one of them
// (a workgroup cannot hand anything to another inside a launch, and repeating costs no time); the records and steps 3 and 4
// are shared out by threads of step 2: workgroup g of G takes those whose first row is in the g-th part of the sorted
// rows, a contiguous range of keys and of sorted positions.  If the radix path has to run, workgroup 0 runs it.
//
// Bound by the latency of one workgroup: ids from memory, then its instructions.  So a row's key and place stay in
// registers from step 1 to step 3, four 8-bit counters share a word, and a thread sums a word's four counts with one
// instruction, its segments and tiles with a few.  (With two 16-bit counters per word, a second round of adds for
// the places, fine-grained MoE shapes over 32768 keys, layer call before / now: 1024 tokens 133.3 / 130.4 us (this kernel 13.3 /
// 10.7), 256 tokens 60.4 / 59.1, 64 tokens 33.0 / 31.8.  Of its time at 1024 tokens, by clock stamps: ids 1.8, counts 1.8,
// sums 1.6, list 1.9, records 0.4, places 1.5, order 1.3; records written by the threads that own the keys took 5.)
//
// W: counter words per thread (up to 4096 W keys); R: rows per thread (up to 1024 R rows).  A row is some 60 instructions, so a thread
// has a form with about as many as it needs, and in the forms of 8 and 16 the last pairs are left out.  Within a pair there
// is no branch: a row without a key adds zero to a word that nobody reads and goes to a place behind the last.  Kernel alone in
// us, forms of 4, 8 and 16 with a branch per row / with a wave-uniform one, rows left out one by one / now: 4096 keys, 1024
// rows 6.7 / 6.5 / 6.1, 4096 rows 6.7 / 7.1 / 6.5, 8192 rows 8.1 / 8.8 / 7.9, 8193 rows 10.6 / 10.4 / 8.7, 16384 rows
// 12.3 / 13.2 / 11.7; 32768 keys, 8192 rows 9.5 / 10.1 / 9.3.
// Occupied keys of a thread up to which its wave lists them one after the other: at 1024 tokens of the fine-grained shapes
// dense and sparse key ranges are alike either way, at 64 and 256 tokens a wave has two or three (59.1 and 31.8 us; all
// keys without a branch 59.9 and 32.8; a branch per key 59.6 and 32.3).
constexpr unsigned kFewOccupied = 6;

template <int W, int R>
__global__ __launch_bounds__(kThreads) void segments_bucket_kernel(SegParams p)
{
    constexpr int KPT = 4 * W;                        // keys per thread
    constexpr int GRP = R <= 4 ? R : 2;               // rows that are left out together
    constexpr unsigned kNowhere = kThreads * W * 3 / 2;        // for rows without a key: the front of tmp, as a counter word
    __shared__ unsigned wave_sums[kWaves][2];
    __shared__ unsigned status_bits, overflow;
    __shared__ int own_lo, own_hi, pos_lo_s, pos_hi_s, seg_lo_s, seg_hi_s;
    extern __shared__ __attribute__((aligned(16))) unsigned char dyn_lds[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int G = gridDim.x, wg = blockIdx.x;         // workgroups that share the records and steps 3 and 4
    const int P = p.P;
    unsigned *cnt = reinterpret_cast<unsigned *>(dyn_lds);              // [kThreads * W] four counts per word
    uint16_t *start = reinterpret_cast<uint16_t *>(cnt + kThreads * W); // [kThreads * W] first position of a word's keys
    unsigned *tmp = reinterpret_cast<unsigned *>(start + kThreads * W); // [P, padded to 64, and 64] row | key << 16
    unsigned *seglist = tmp;               // key | first tile << 16 per segment, before tmp is used
    auto count_of = [&](unsigned key) { return (cnt[key >> 2] >> ((key & 3u) * 8u)) & 0xFFu; };
    auto start_of = [&](unsigned key) {
        return (unsigned)start[key >> 2] +
               __builtin_amdgcn_sad_u8(cnt[key >> 2] & ((1u << ((key & 3u) * 8u)) - 1u), 0u, 0u);
    };

    // ---- 1. keys, counts and places --------------------------------------------------------
    auto each_group = [&](auto body) {
#pragma unroll
        for (int u0 = 0; u0 < R; u0 += GRP)
            if (u0 <= R / 2 || kThreads * u0 < P) body(u0);
    };
    int a[R], e[R];
    each_group([&](int u0) {
#pragma unroll
        for (int u = u0; u < u0 + GRP; ++u) {
            const int i = tid + u * kThreads, r = min(i, P - 1);
            a[u] = p.adapter_id[r];
            e[u] = p.expert_id ? p.expert_id[r] : 0;
            if (i >= P) a[u] = -1;
        }
    });
    if (tid == 0) {
        status_bits = 0;
        overflow = 0;
        own_lo = kThreads;
        pos_lo_s = seg_lo_s = P;
        own_hi = pos_hi_s = seg_hi_s = 0;
    }
#pragma unroll
    for (int j = 0; j < W; ++j) cnt[tid + j * kThreads] = 0;
    __syncthreads();
    unsigned mine[R];                                 // key | place << 16, or kNoKey
    unsigned bad = 0;
    {
        unsigned old[R];
        bool over = false;
#pragma unroll
        for (int u = 0; u < R; ++u) mine[u] = kNoKey;
        each_group([&](int u0) {
#pragma unroll
            for (int u = u0; u < u0 + GRP; ++u) {
                mine[u] = row_key(p, a[u], e[u], bad);
                const bool yes = mine[u] != kNoKey;
                old[u] = atomicAdd(&cnt[yes ? mine[u] >> 2 : kNowhere + lane], yes ? 1u << ((mine[u] & 3u) * 8u) : 0u);
            }
        });
        each_group([&](int u0) {
#pragma unroll
            for (int u = u0; u < u0 + GRP; ++u) {
                const bool yes = mine[u] != kNoKey;
                const unsigned place = yes ? (old[u] >> ((mine[u] & 3u) * 8u)) & 0xFFu : 0u;
                over = over || place == 0xFFu;        // the counter has run into its neighbour
                mine[u] |= place << 16;
            }
        });
        if (bad) atomicOr(&status_bits, bad);
        if (over) overflow = 1;
    }
    __syncthreads();
    if (overflow) {                                   // every workgroup has seen the same counts
        __syncthreads();
        if (wg == 0)
            radix_body(p, [&](unsigned *key_of, unsigned &bad_rows) {
                int n_active = 0;
#pragma unroll
                for (int u = 0; u < R; ++u) {
                    const int i = tid + u * kThreads;
                    if (i < P) key_of[i] = mine[u] == kNoKey ? kNoKey : mine[u] & 0xFFFFu;
                    n_active += mine[u] != kNoKey ? 1 : 0;
                }
                bad_rows = bad;
                return n_active;
            });
        return;
    }

    // ---- 2. scan over the keys; segment records and tiles ----------------------------------
    const int TR = p.tile_rows;                       // a power of two, 16 or 32
    const int tr_shift = 31 - __clz(TR);
    unsigned cw[W];                                   // my words
    unsigned rows = 0, segs = 0, rs_before, rs_total, t_before, t_total;          // rows | segments << 16, and tiles
    {
        unsigned tiles = 0;
#pragma unroll
        for (int j = 0; j < W; ++j) cw[j] = cnt[tid * W + j];
        // bytes that are not zero: the sum with 0x7F carries into the top bit, of each byte on its own
        auto occupied = [](unsigned x) { return (unsigned)__popc((((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x) & 0x80808080u); };
        const unsigned whole = (0xFFu >> tr_shift) * 0x01010101u, rest = (unsigned)(TR - 1) * 0x01010101u;
#pragma unroll
        for (int j = 0; j < W; ++j) {
            rows = __builtin_amdgcn_sad_u8(cw[j], 0u, rows);
            segs += occupied(cw[j]);
            tiles = __builtin_amdgcn_sad_u8((cw[j] >> tr_shift) & whole, 0u, tiles) + occupied(cw[j] & rest);
        }
        // a batch has at most 16384 rows, so rows and segments share a word
        block_excl_sum2<kWaves>(rows | (segs << 16), tiles, wave_sums, &rs_before, &t_before, &rs_total, &t_total);
    }
    const int P_act = (int)(rs_total & 0xFFFFu), S = (int)(rs_total >> 16);
    const int first = (int)(rs_before & 0xFFFFu);
    const bool here = rows && first * G / P_act == wg;
    if (here) {
        // my keys' starts, and a list of those that occur with the first tile of each
        unsigned at = (unsigned)first, sidx = rs_before >> 16, tix = t_before;
        unsigned long long occ = 0;                   // which of my keys occur
#pragma unroll
        for (int j = 0; j < W; ++j) {
            start[tid * W + j] = (uint16_t)at;
            at = __builtin_amdgcn_sad_u8(cw[j], 0u, at);
            const unsigned top = ((((cw[j] & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | cw[j]) & 0x80808080u) >> 7;
            occ |= (unsigned long long)((top * 0x01020408u) >> 24 & 0xFu) << (4 * j);
        }
        if (!__any(segs > kFewOccupied)) {            // a wave with few of them takes one after the other,
            for (; occ; occ &= occ - 1) {
                const unsigned key = (unsigned)tid * KPT + (unsigned)__ffsll((long long)occ) - 1;
                seglist[sidx++] = key | (tix << 16);
                tix += (count_of(key) + TR - 1) >> tr_shift;
            }
        } else {                                      // one with many all keys without a branch
            const int nowhere = ((P + 63) & ~63) + lane;
#pragma unroll
            for (int j = 0; j < W; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const unsigned n = (cw[j] >> (8 * q)) & 0xFFu;
                    seglist[n ? sidx : (unsigned)nowhere] = (unsigned)((tid * W + j) * 4 + q) | (tix << 16);
                    sidx += n ? 1u : 0u;
                    tix += (n + TR - 1) >> tr_shift;
                }
        }
    }
    {
        const unsigned long long who = __ballot(here);
        if (who) {
            const int l0 = __ffsll((long long)who) - 1, l1 = 63 - __clzll((long long)who);
            if (lane == l0) {
                atomicMin(&own_lo, tid);
                atomicMin(&pos_lo_s, first);
                atomicMin(&seg_lo_s, (int)(rs_before >> 16));
            }
            if (lane == l1) {
                atomicMax(&own_hi, tid + 1);
                atomicMax(&pos_hi_s, first + (int)rows);
                atomicMax(&seg_hi_s, (int)(rs_before >> 16) + (int)segs);
            }
        }
    }
    __syncthreads();
    const unsigned lo = (unsigned)own_lo, hi = (unsigned)own_hi;        // this workgroup's threads of step 2
    const int pos_lo = pos_lo_s, pos_hi = pos_hi_s;
    // segment records and tiles, one segment per thread and turn
#pragma unroll 1
    for (int sidx = seg_lo_s + tid; sidx < seg_hi_s; sidx += kThreads) {
        const unsigned it = seglist[sidx], key = it & 0xFFFFu;
        const int at = (int)start_of(key), n = (int)count_of(key);
        int tix = (int)(it >> 16);
        p.seg_start[sidx] = at;
        p.seg_key[sidx] = (int32_t)key;
#pragma unroll 1
        for (int r = 0; r < n; r += TR) {
            lora_tile t;
            t.key = (int32_t)key;
            t.row0 = at + r;
            t.n_rows = min(TR, n - r);
            t.seg = sidx;
            p.tiles[tix++] = t;
        }
    }
    __syncthreads();

    // ---- 3. every row to its place in its key's range ---------------------------------------
    {
        unsigned to[R];
        each_group([&](int u0) {
#pragma unroll
            for (int u = u0; u < u0 + GRP; ++u) {       // all look-ups before the first store
                const unsigned k = mine[u] & 0xFFFFu, owner = k / KPT;
                const bool yes = mine[u] != kNoKey && owner >= lo && owner < hi;
                const unsigned at = start_of(yes ? k : 0u) + (mine[u] >> 16);
                to[u] = yes ? at : (unsigned)((P + 63) & ~63) + lane;
            }
        });
        each_group([&](int u0) {
#pragma unroll
            for (int u = u0; u < u0 + GRP; ++u) tmp[to[u]] = (unsigned)(tid + u * kThreads) | (mine[u] << 16);
        });
    }
    // filler around this workgroup's positions: step 4 reads aligned groups of four words
    if (pos_lo < pos_hi) {
        if (tid < 4 && (pos_lo & ~3) + tid < pos_lo) tmp[(pos_lo & ~3) + tid] = 0xFFFFFFFFu;
        if (tid >= 4 && tid < 8 && pos_hi + tid - 4 < ((pos_hi + 3) & ~3)) tmp[pos_hi + tid - 4] = 0xFFFFFFFFu;
    }
    __syncthreads();

    // ---- 4. order inside the bucket by row index -------------------------------------------
    // The bucket is read in aligned groups of four words; words of other keys (and the
    // filler around the workgroup's positions) fall outside [key << 16, mine) and count as not
    // smaller.
#pragma unroll 1
    for (int pos = pos_lo + tid; pos < pos_hi; pos += kThreads) {
        const unsigned me = tmp[pos];
        const unsigned k = me >> 16, row = me & 0xFFFFu, base = me & 0xFFFF0000u;
        const int b0 = (int)start_of(k), b1 = b0 + (int)count_of(k);
        int rank = 0;
#pragma unroll 1
        for (int j = b0 & ~3; j < b1; j += 4) {
            const u32x4 t = *reinterpret_cast<const u32x4 *>(tmp + j);
            rank += (t[0] - base < row ? 1 : 0) + (t[1] - base < row ? 1 : 0) +
                    (t[2] - base < row ? 1 : 0) + (t[3] - base < row ? 1 : 0);
        }
        p.perm[b0 + rank] = (int32_t)row;
    }
    if (tid == 0 && wg == 0) {
        p.seg_start[S] = P_act;
        p.counts[0] = S;
        p.counts[1] = P_act;
        p.counts[2] = (int32_t)t_total;
        p.counts[3] = 0;
        p.status[0] = status_bits;
    }
}
}  // namespace

size_t segments_lds_bytes(int P)
{
    const size_t P_pad = ((size_t)P + 63) & ~(size_t)63;
    return P_pad * 4 + 2 * P_pad * 2;
}

// counter words a thread of the bucket path owns, four keys each: a power of two
static int bucket_words_of(unsigned n_keys)
{
    int words = 1;
    while ((unsigned)(4 * kThreads * words) < n_keys) words *= 2;
    return words;
}

// dynamic LDS of the bucket path (it may fall back to the radix path inside the kernel)
static size_t bucket_lds_bytes(int P, unsigned n_keys)
{
    const size_t P_pad = ((size_t)P + 63) & ~(size_t)63;
    const size_t need = (size_t)kThreads * bucket_words_of(n_keys) * (4 + 2) + (P_pad + 64) * 4;
    return need > segments_lds_bytes(P) ? need : segments_lds_bytes(P);
}

constexpr size_t kBucketLdsMax = 140 * 1024;
constexpr int kBucketWorkgroups = 8;

template <int W, int R>
static hipError_t launch_bucket_wr(const SegParams &p, size_t dyn, hipStream_t s)
{
    static hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(segments_bucket_kernel<W, R>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)kBucketLdsMax);
    if (attr != hipSuccess) return attr;
    // the counting and the scan over the keys are done by every workgroup, the rest is shared out
    const int wgs = std::max(1, std::min(kBucketWorkgroups, p.P / 1024));
    hipLaunchKernelGGL((segments_bucket_kernel<W, R>), dim3(wgs), dim3(kThreads), dyn, s, p);
    return hipGetLastError();
}

template <int W>
static hipError_t launch_bucket(const SegParams &p, size_t dyn, hipStream_t s)
{
    static_assert(16 * kThreads == LORA_MAX_ROWS, "the last form takes the longest batch");
    if (p.P <= kThreads) return launch_bucket_wr<W, 1>(p, dyn, s);
    if (p.P <= 2 * kThreads) return launch_bucket_wr<W, 2>(p, dyn, s);
    if (p.P <= 4 * kThreads) return launch_bucket_wr<W, 4>(p, dyn, s);
    if (p.P <= 8 * kThreads) return launch_bucket_wr<W, 8>(p, dyn, s);
    return launch_bucket_wr<W, 16>(p, dyn, s);
}

hipError_t launch_segments(const SegParams &p_in, void *ws, hipStream_t s)
{
    SegParams p = p_in;
    // long batches of few keys: several workgroups (segments_large.hip)
    if (segments_large_handles(p)) return launch_segments_large(p, ws, s);
    const unsigned n_keys = (unsigned)p.n_adapters * (unsigned)p.n_experts;
    // LORA_SEGMENT_PATH=radix forces the radix path (all give the same result)
    static const bool force_radix = [] {
        const char *e = getenv("LORA_SEGMENT_PATH");
        return e && e[0] == 'r';
    }();
    // at most 256 keys and 4096 rows: a kernel of its own, ahead of both paths at every size it takes
    if (!force_radix && n_keys <= kInlineMaxKeys && p.P > 0 && p.P <= kSmallMaxRows) {
        if (p.tile_rows == kTileRows) launch_small<kSmallGroups, kTileRows>(p, s);
        else if (p.P <= 1024) launch_small<16, kDecodeTileRows>(p, s);
        else if (p.P <= 2048) launch_small<32, kDecodeTileRows>(p, s);
        else launch_small<kSmallGroups, kDecodeTileRows>(p, s);
        return hipGetLastError();
    }
    // Counting path: short segments on average and counters that fit LDS beside the radix path's static arrays.
    // Few keys with more rows than that (up to 5119, where several workgroups begin) have long buckets: one radix pass.
    // An empty batch takes the radix path.
    const bool few_keys = n_keys <= kInlineMaxKeys;
    if (!force_radix && p.P > 0 && p.P <= LORA_MAX_ROWS && !few_keys && (int64_t)p.P < 64 * (int64_t)n_keys && n_keys <= 0x10000u &&
        bucket_lds_bytes(p.P, n_keys) <= kBucketLdsMax) {
        const size_t dyn = bucket_lds_bytes(p.P, n_keys);
        switch (bucket_words_of(n_keys)) {
        case 1: return launch_bucket<1>(p, dyn, s);
        case 2: return launch_bucket<2>(p, dyn, s);
        case 4: return launch_bucket<4>(p, dyn, s);
        case 8: return launch_bucket<8>(p, dyn, s);
        default: return launch_bucket<16>(p, dyn, s);
        }
    }
    const size_t dyn = segments_lds_bytes(p.P);
    if (dyn > 48 * 1024) {
        // ask once for the largest dynamic LDS size this kernel is ever launched with
        static hipError_t attr = hipFuncSetAttribute(
            reinterpret_cast<const void *>(segments_kernel),
            hipFuncAttributeMaxDynamicSharedMemorySize, (int)segments_lds_bytes(LORA_MAX_ROWS));
        if (attr != hipSuccess) return attr;
    }
    hipLaunchKernelGGL(segments_kernel, dim3(1), dim3(kThreads), dyn, s, p);
    return hipGetLastError();
}

}  // namespace lora

// Segment build inside the first kernel that consumes the segments (App. A.2.2: rows that share
// an adapter are aggregated before shrink and expand; Sec. 5.2: few launches per layer call).
//
// For small decode batches the stand-alone builder is one short kernel whose time is mostly the
// latency of a launch, and the shrink that follows cannot start before it ends.  Here every
// workgroup of the shrink sorts the whole batch for itself in LDS before its first work item:
// the same stable counting sort (key = adapter * E + expert ascending, original order inside a
// key, rows without adapter left out), the same segment records and tiles, bit for bit.  The
// sort is repeated by every workgroup, which costs each about as much as the dependent loads
// of tile records and row indices it replaces; nobody waits for anybody.  Workgroup 0 also
// writes the result to the caller's lora_segments for the launches that follow.
//
// Limits: kInlineMaxRows rows, kInlineMaxKeys keys, tiles of kDecodeTileRows rows, workgroups
// of four waves and more (thread k < kInlineMaxKeys owns key k).
//
// The stand-alone builder of up to 4096 rows is the same sort with sixteen waves (segments.hip).
//
// Stability without order-defining atomics: the batch is cut into groups of 64 consecutive
// rows, one wave handles a group at a time and ranks equal keys inside it by lane order (ballot
// match); counts[group][key] is written by the group's first lane of that key.  Thread k then
// turns its key's counts into exclusive sums over the groups in order, a workgroup scan over
// the keys gives every key its start, and a row's position is
//   start of its key + rows of the key in earlier groups + lanes below it in its group.
#pragma once
#include "lora_device.h"
#include "segments_common.h"

namespace lora {

constexpr int kInlineMaxRows = 2048;
constexpr int kInlineMaxKeys = 256;
constexpr int kInlineGroups = kInlineMaxRows / 64;
constexpr int kInlineKeyWaves = kInlineMaxKeys / 64;             // waves whose threads own a key

// rows of every key per group of 64 rows; cleared with 16-byte stores
template <int GROUPS>
struct alignas(16) SortCounts {
    uint16_t n[GROUPS][kInlineMaxKeys];
};
typedef SortCounts<kInlineGroups> InlineCounts;                   // 16 KiB, free again after the build

// TILES: room for the tile records, which otherwise go straight to the caller's segments
template <int ROWS, bool TILES>
struct SortedSegments {
    static constexpr bool kKeepsTiles = TILES;
    uint16_t perm[ROWS];
    lora_tile tiles[TILES ? ROWS / kDecodeTileRows + kInlineMaxKeys : 1];
    unsigned key_tile[TILES ? 1 : kInlineMaxKeys];               // first tile of a key, its segment << 16
    unsigned key_start[kInlineMaxKeys];
    unsigned wave_sums[kInlineKeyWaves][3];
    unsigned status;
    int n_tiles;
};
typedef SortedSegments<kInlineMaxRows, true> InlineSegments;     // lives in LDS for the whole kernel

// G: groups of 64 rows that the code is unrolled for (batches of up to 64 * G rows); NW: waves of the
// workgroup; TR: rows per tile
template <int NW, int G, int TR = kDecodeTileRows, class Counts, class Segments>
__device__ inline void build_segments_inline_n(const SegParams &sp, Counts &counts, Segments &L, bool write_global)
{
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int P = sp.P;
    constexpr int GPW = (G + NW - 1) / NW;              // groups per wave; those beyond the batch are empty
    static_assert(NW >= kInlineKeyWaves, "a thread per key");
    static_assert(G % NW == 0 || G < NW, "the waves' groups are the first G");
    static_assert(alignof(Counts) >= sizeof(u32x4), "cleared with 16-byte stores");

    // ids of this wave's groups (wave w takes groups w, w + NW, ...): all loads first
    int a[GPW], e[GPW];
#pragma unroll
    for (int u = 0; u < GPW; ++u) {
        const int row = (w + NW * u) * 64 + lane;
        const int r = min(row, P - 1);                      // unconditional loads (P >= 1), then selects
        a[u] = sp.adapter_id[r];
        e[u] = sp.expert_id ? sp.expert_id[r] : 0;
        if (row >= P) a[u] = -1;
    }
    {
        const u32x4 zero = {0u, 0u, 0u, 0u};
        u32x4 *c4 = reinterpret_cast<u32x4 *>(&counts.n[0][0]);
        for (int i = tid; i < G * (kInlineMaxKeys * 2 / 16); i += 64 * NW) c4[i] = zero;
        if (tid == 0) L.status = 0;
    }
    __syncthreads();

    // equal keys inside each group, all of the wave's groups bit by bit together (the groups'
    // chains of ballots are independent, so they overlap)
    unsigned key[GPW], below[GPW];
    unsigned bad = 0;
    Match m[GPW];
#pragma unroll
    for (int u = 0; u < GPW; ++u) {
        key[u] = row_key(sp, a[u], e[u], bad);
        const unsigned long long v = __ballot(key[u] != kNoKey);
        m[u].lo = (unsigned)v;
        m[u].hi = (unsigned)(v >> 32);
    }
#pragma unroll 1
    for (int b = 0; b < sp.key_bits; ++b) {
#pragma unroll
        for (int u = 0; u < GPW; ++u) {
            // all ones if my bit is set; lanes without a key (all bits set) are in no mask
            const unsigned same = (unsigned)__builtin_amdgcn_sbfe((int)key[u], (unsigned)b, 1u);
            const unsigned long long bal = __ballot(same != 0);
            m[u].lo &= ~((unsigned)bal ^ same);
            m[u].hi &= ~((unsigned)(bal >> 32) ^ same);
        }
    }
#pragma unroll
    for (int u = 0; u < GPW; ++u) {
        const int g = w + NW * u;                           // wave-uniform
        below[u] = lanes_below(m[u]);
        if (key[u] != kNoKey && below[u] == 0) counts.n[g][key[u]] = (uint16_t)(__popc(m[u].lo) + __popc(m[u].hi));
    }
    if (bad) atomicOr(&L.status, bad);                      // OR is order-independent
    __syncthreads();

    // thread k: counts of key k per group -> rows of the key in earlier groups; its total
    const bool owner = w < kInlineKeyWaves;             // wave-uniform
    unsigned total = 0, my_tiles = 0, occ = 0, ir = 0, is = 0, it = 0;
    if (owner) {
        unsigned c[G];
#pragma unroll
        for (int g = 0; g < G; ++g) c[g] = counts.n[g][tid];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            counts.n[g][tid] = (uint16_t)total;
            total += c[g];
        }
        my_tiles = (total + TR - 1) / TR;
        occ = total ? 1u : 0u;
        ir = wave_incl_sum(total), is = wave_incl_sum(occ), it = wave_incl_sum(my_tiles);
        if (lane == 63) {
            L.wave_sums[w][0] = ir;
            L.wave_sums[w][1] = is;
            L.wave_sums[w][2] = it;
        }
    }
    __syncthreads();
    unsigned row0 = ir - total, seg = is - occ, tile0 = it - my_tiles, P_act = 0, S = 0, n_tiles = 0;
#pragma unroll
    for (int k = 0; k < kInlineKeyWaves; ++k) {
        const unsigned r = L.wave_sums[k][0], s = L.wave_sums[k][1], t = L.wave_sums[k][2];
        P_act += r;
        S += s;
        n_tiles += t;
        row0 += k < w ? r : 0u;
        seg += k < w ? s : 0u;
        tile0 += k < w ? t : 0u;
    }
    if (owner) L.key_start[tid] = row0;
    if (tid == 0) L.n_tiles = (int)n_tiles;
    // tiles and segment record of my key (a thread without a key has no rows)
    if constexpr (!Segments::kKeepsTiles) {
        if (owner) L.key_tile[tid] = tile0 | seg << 16;
    }
    auto put_tile = [&](int key, unsigned first, unsigned rows, unsigned s, unsigned tile_base, unsigned j) {
        lora_tile t;
        t.key = key;
        t.row0 = (int32_t)(first + j * TR);
        t.n_rows = (int32_t)min((unsigned)TR, rows - j * TR);
        t.seg = (int32_t)s;
        if constexpr (Segments::kKeepsTiles) L.tiles[tile_base + j] = t;
        else sp.tiles[tile_base + j] = t;
    };
    if constexpr (Segments::kKeepsTiles) {
        constexpr unsigned kOwnTiles = 3;
#pragma unroll
        for (unsigned j = 0; j < kOwnTiles; ++j)
            if (j < my_tiles) put_tile(tid, row0, total, seg, tile0, j);
        // the rest of a long segment by the whole wave (one thread writing the 112 tiles of a prompt of 1792 rows:
        // 150.2 us for the layer of llama shapes that it is part of, 148.4 so)
        for (unsigned long long more = __ballot(my_tiles > kOwnTiles); more; more &= more - 1) {
            const int l = __ffsll((long long)more) - 1;
            const unsigned r0 = __builtin_amdgcn_readlane(row0, l), n = __builtin_amdgcn_readlane(total, l);
            const unsigned s = __builtin_amdgcn_readlane(seg, l), t0 = __builtin_amdgcn_readlane(tile0, l);
            const unsigned nt = __builtin_amdgcn_readlane(my_tiles, l);
            for (unsigned j = kOwnTiles + lane; j < nt; j += 64) put_tile(w * 64 + l, r0, n, s, t0, j);
        }
    }
    if (write_global && total) {
        sp.seg_start[seg] = (int32_t)row0;
        sp.seg_key[seg] = tid;
    }
    __syncthreads();

    if constexpr (!Segments::kKeepsTiles) {
        // a tile per thread and turn: its key is the last one whose first tile is not beyond it (an empty key shares
        // its first tile with the next key, which wins)
        for (unsigned ti = tid; ti < n_tiles; ti += 64 * NW) {
            int key = 0;
#pragma unroll
            for (int step = kInlineMaxKeys / 2; step > 0; step >>= 1)
                if ((L.key_tile[key + step] & 0xFFFFu) <= ti) key += step;
            const unsigned first = L.key_start[key], end = key + 1 < kInlineMaxKeys ? L.key_start[key + 1] : P_act;
            const unsigned t0 = L.key_tile[key] & 0xFFFFu;
            put_tile(key, first, end - first, L.key_tile[key] >> 16, t0, ti - t0);
        }
    }
    // rows to their positions
#pragma unroll
    for (int u = 0; u < GPW; ++u) {
        const int g = w + NW * u;
        if (key[u] != kNoKey)
            L.perm[L.key_start[key[u]] + counts.n[g][key[u]] + below[u]] = (uint16_t)(g * 64 + lane);
    }
    __syncthreads();

    if (write_global) {
        for (unsigned i = tid; i < P_act; i += 64 * NW) sp.perm[i] = (int32_t)L.perm[i];
        if constexpr (Segments::kKeepsTiles)
            for (unsigned i = tid; i < n_tiles; i += 64 * NW) sp.tiles[i] = L.tiles[i];
        if (tid == 0) {
            sp.seg_start[S] = (int32_t)P_act;
            sp.counts[0] = (int32_t)S;
            sp.counts[1] = (int32_t)P_act;
            sp.counts[2] = (int32_t)n_tiles;
            sp.counts[3] = 0;
            sp.status[0] = L.status;
        }
    }
}

template <int NW>
__device__ inline void build_segments_inline(const SegParams &sp, InlineCounts &counts, InlineSegments &L,
                                             bool write_global)
{
    if (sp.P <= 256) build_segments_inline_n<NW, 4>(sp, counts, L, write_global);
    else if (sp.P <= 512) build_segments_inline_n<NW, 8>(sp, counts, L, write_global);
    else if (sp.P <= 1024) build_segments_inline_n<NW, 16>(sp, counts, L, write_global);
    else build_segments_inline_n<NW, kInlineGroups>(sp, counts, L, write_global);
}

}  // namespace lora

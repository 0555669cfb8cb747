// Internal declarations shared by the translation units of liblora (host side only;
// kernels live in the .hip files and are reached through the launch_* functions).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/lora.h"
#include "lora_layout.h"

namespace lora {

// One entry of the device pointer table: 32 bytes, ordered [layer][adapter][expert][proj].
struct Unit {
    const uint16_t *A;  // packed shrink operand of the unit
    const uint16_t *B;  // packed expand operand of the unit
    float scale;        // the adapter's scale
    int32_t rank;       // the adapter's own rank (<= pool rank; the rest is zero padding)
    // Rank of the adapter that A and B were last loaded with (0: not loaded yet): entries from there on are zeros in
    // memory and the decode kernels don't fetch them.  Not `rank`, which lora_pool_set_adapter changes ahead of a load.
    int32_t a_rank, b_rank;
};
static_assert(sizeof(Unit) == 32, "table entry is 32 bytes");

constexpr int kTileRows = 32;        // rows per tile of the long-segment kernels
constexpr int kLongRows = 128;       // rows of one segment per work item of the long-segment shrink
constexpr int kLongListedSegs = 64 * 64;    // segments that its waves hold in registers
constexpr int kDecodeTileRows = 16;  // rows per tile of the decode kernels
constexpr int kKBlock = 32;          // K elements per MFMA step (v_mfma_f32_16x16x32_bf16)
constexpr int kColChunk = 128;       // output columns one wave owns in expand
constexpr int kPartKBlocks = 32;     // long segments: K-blocks of a part that the workspace is sized by
constexpr int kMaxParts = 64;
// Shrink and expand in one launch (fused_decode.hip): limits and work split, measured on MI355X.
constexpr int kFusedWaves = 8;         // waves of a workgroup = 128-column chunks of a work item
constexpr int kFusedMaxK = 4096;       // longest input
constexpr int kFusedMaxChunks = 64;    // widest group, in 128-column chunks per tile
constexpr int kFusedMaxTiles = 64;     // largest batch, as the host's upper bound of the tile count
// Work items x rank x inputs, that is half the bytes of A that all items together read.  A workgroup
// fetches the whole A of its item at what one CU can pull, so one launch loses to two as that grows
// (whole call in us, one launch / two; 4096 -> 4096, rank 16: 1 row 6.7 / 7.7, 8 rows, 2.1 M: 7.4 /
// 8.4, 24 rows, 6.3 M: 8.8 / 8.6; rank 8, 24 rows, 3.1 M: 7.1 / 8.5; rank 64, 8 rows, 8.4 M: 16.2 /
// 10.7; query/key/value of the Llama shapes, 8 rows, 3.1 M: two launches win by 2 us).
constexpr int64_t kFusedMaxWork = 21ll << 17;      // twice that at rank 8, whose A is half the bytes of rank 16
// Cache hints of the activation streams of the decode kernels, measured on MI355X.  Input rows that
// are read once are streamed from kStreamXMiB on, fetched as whole lines (ranks 8 to 32).  A wave of rank 64
// takes 64 bytes of a row per step, and half a line that is fetched with the streaming hint costs where the
// line was in a cache, so rank 64 streams only from kStreamXRank64MiB on (two steps as one, which would
// fetch whole lines, cost the smaller batches 1-3 %: their order of sums has to be the same).
// Layer call in us, cacheable / streamed in one process, by where the activations are when it starts
// (in HBM only; just written by the kernels before; left in the memory-side cache by the previous call):
//   Mixtral shapes, 512 tokens (28 MiB), rank 8    85.4 / 80.3    81.9 / 82.7    77.2 / 78.2
//     rank 16  117.5 / 108.7  115.2 / 114.2  105.3 / 106.3;   rank 32  193.1 / 179.0  192.2 / 191.0  174.7 / 175.2
//   Mixtral shapes, 1024 tokens (56 MiB), rank 8   141.0 / 135.0  123.0 / 125.2  114.9 / 116.4
//     rank 16  176.8 / 168.2  158.0 / 160.3  141.1 / 142.1;   rank 32  270.9 / 259.0  258.5 / 257.8  227.5 / 224.9
//   llama shapes, 2048 rows (16 and 56 MiB), rank 8   157.1 / 152.0  147.2 / 144.9  140.0 / 133.2
//     rank 16  176.2 / 170.6  168.5 / 163.1  163.4 / 150.8;   rank 32  258.8 / 243.6  256.2 / 246.0  253.4 / 224.9
//   rank 64: Mixtral shapes, 512 tokens   337 / 321  340.4 / 343.9  313.7 / 314.7;   1024 tokens   440 / 430
//     441.6 / 448.6  408.9 / 401.2;   llama shapes, 1024 rows (28 MiB)   263.3 / 257.4  255.1 / 259.7  235.6 / 238.0
// 8 MiB as the limit of ranks 8 and 16 costs where rows were just written: llama shapes, 1024 rows (8 and
// 28 MiB), rank 8 95.1 against 94.2 us with 16 MiB, rank 16 108.8 against 108.2.
// The output rows of one call are streamed from kStreamYMiB on: just-written ones would lose what
// those in HBM gain (Mixtral shapes, 2048 tokens, 235 MiB: 246.8 / 259.1 against 258.9 / 247.4).
constexpr int kLongMinRowsTimesRank = 1 << 17;   // long-segment kernels from this many rows x rank on
constexpr int kLongMinRowsRank16 = 12288;        // rank 16: the long-segment kernels proper from here on, and
constexpr int kLongRowsPerKeyRank16 = 128;       // from this many rows per key
constexpr int kStreamXMiB = 16;
constexpr int kStreamXRank64MiB = 64;
constexpr int kStreamYMiB = 256;
constexpr int kMaxFused = 3;         // projections that share an input in one launch (q/k/v, gate/up)

// ---- packed layout sizes ---------------------------------------------------------------
inline int kunit_of(int rank) { return rank == 8 ? 64 : kKBlock; }   // K values per packed A block
inline int kblocks_of(int h_in, int rank) { return (h_in + kunit_of(rank) - 1) / kunit_of(rank); }
// K-blocks a wave of the decode shrink takes per step: 128 K values at ranks 8 and 16, 64 and 32 above
constexpr int shrink_wave_units(int rank) { return rank == 8 ? 2 : rank == 16 ? 4 : rank == 32 ? 2 : 1; }
// K parts of the long-segment shrink.  Two work items fit a CU at a time, and all of them run for about
// as long, so a second round that is nearly empty costs a whole one: as many K parts as one round of the
// chip takes.  Few items need less than a full round (more parts are more fp32 sums to write and read);
// many take several rounds, by how well those fill.  The tiles are counted, four to a full block: 16384 rows in 8 uneven requests (130
// fours and more), rank 64, 3 parts 270.5 us, 4 parts (two rounds) 278.7 (2 parts, with the kernels before these, 298 against
// 290 for 3); in 8 equal ones (128) 4 parts 284, 3 parts 288 (likewise); 4096 rows, 6 parts 93.5, 9 parts 96.6.  The tiles, and not a bound from the
// number of rows, because that cannot tell the equal requests from the uneven ones.  `most`: what the
// workspace has room for.  Whole numbers only: the shrink and the kernel that adds its parts both call it and
// have to come to the same result.
struct LongSplit {
    int n_parts, kb_per_part;
};

__host__ __device__ inline LongSplit long_split(int n_tiles, int kblocks, int most)
{
    constexpr int kPlaces = 512, kFew = 220;
    const int fours = n_tiles > 0 ? (n_tiles + 3) / 4 : 1;
    int n = 1;
    if (fours < 64) {
        n = kFew / fours;
    } else if (fours <= kPlaces) {
        n = kPlaces / fours;
    } else {
        // c parts take `rounds` rounds; the share of them that is filled, less 4 % for a part's sums
        long long best_filled = 0, best_rounds = 1;
        for (int c = 1; c <= 4; ++c) {
            const long long rounds = (fours * c + kPlaces - 1) / kPlaces;
            const long long filled = (long long)fours * c * (100 - 4 * c);
            if (filled * best_rounds > best_filled * rounds) {
                best_filled = filled;
                best_rounds = rounds;
                n = c;
            }
        }
    }
    n = n < most ? n : most;
    LongSplit s;
    s.kb_per_part = ((kblocks + n - 1) / n + 3) / 4 * 4;
    s.n_parts = (kblocks + s.kb_per_part - 1) / s.kb_per_part;
    return s;
}

inline int chunks_of(int h_out) { return (h_out + kColChunk - 1) / kColChunk; }
inline size_t packed_A_bytes(int h_in, int rank) { return (size_t)kblocks_of(h_in, rank) * kunit_of(rank) * rank * 2; }
inline size_t packed_B_bytes(int h_out, int rank) { return (size_t)chunks_of(h_out) * kColChunk * rank * 2; }
inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// ---- launch parameter blocks -----------------------------------------------------------
struct PackParams {
    const uint16_t *src;     // first unit's row-major matrix
    int64_t src_stride;      // elements between consecutive units' matrices
    uint16_t *dst;           // first unit's packed destination
    int64_t dst_stride;      // elements between consecutive units' packed matrices
    int n_units;
    int h;                   // h_in (A) or h_out (B)
    int rank;                // pool rank
    int src_rank;            // rank of the source matrices (<= rank)
    int32_t *rank_out;       // where the first unit's table entry notes src_rank (repacks into the pool only)
    int rank_stride;         // 32-bit words between consecutive units' entries
};

// all A and B repacks of one (adapter, layer) in one launch: job 2j = A, 2j+1 = B of projection j
struct PackLayerParams {
    PackParams job[2 * LORA_MAX_PROJ];
    int wg0[2 * LORA_MAX_PROJ + 1];      // first workgroup of a job; filled by launch_pack_layer
    int n_jobs;
    int aligned;             // every source is 16-byte aligned; filled by launch_pack_layer
};

struct SegParams {
    const int32_t *adapter_id;
    const int32_t *expert_id;
    int P;
    int n_adapters;
    int n_experts;
    int tile_rows;
    int passes;              // radix passes of 8 bits over the key
    int key_bits;            // bits of the largest key
    int32_t *perm;
    int32_t *seg_start;
    int32_t *seg_key;
    lora_tile *tiles;
    int32_t *counts;
    uint32_t *status;
};

// the multi-workgroup segment builder (segments_large.hip)
struct LargeSegParams {
    SegParams p;
    unsigned *header;        // [0] = active rows, written by the first pass for the next
    unsigned *wg_hist;       // [chunks][256] digit counts per chunk
    unsigned *wg_info;       // [chunks][2] active rows and status bits per chunk
    unsigned *key_g;         // [P] key of every row (kept for later passes), may be null
    const unsigned *order_in;    // rows in the order the previous pass left them
    unsigned *order_out;
    unsigned *chunk_info;    // [chunks][4] segment heads of every chunk of the sorted order
    int G;                   // chunks = workgroups
    int pass;                // 8-bit digit this pass sorts by
};

struct ShrinkParams {
    const Unit *units;       // table rows of the layer
    int n_proj;              // projections per unit (table stride)
    int proj0;               // first projection handled
    int n_fused;             // 1 .. kMaxFused consecutive projections sharing x (same h_in)
    const uint16_t *x;
    int64_t ldx;
    const int32_t *src_row;  // may be null
    const int32_t *perm;
    const lora_tile *tiles;
    const int32_t *seg_start;    // long-segment kernel
    const int32_t *seg_key;
    const int32_t *counts;
    float *v[kMaxFused];     // per fused projection: [n_parts][P][rank]
    int P;
    int h_in;
    int n_parts;             // long-segment kernel: the most parts there may be (long_split)
    FastDiv parts;           // decode kernel: division by n_parts
    int kb_per_part;         // decode kernel
    int rank;
    int grid;
    union {
        int tile_halves;     // decode kernel: the tiles have up to 32 rows and are taken in halves
        int by_tiles;        // long-segment kernel: work items are groups of four tiles, else blocks of one segment
    };
    union {
        int wave_per_tile;   // decode kernel: every wave takes a whole tile (no K split across waves)
        int blocks;          // long-segment kernel: blocks of one segment, at most kLongListedSegs segments
    };
    int build;               // decode kernel: the segments are built inside the launch, from `seg`
    int lower_ranks;         // decode kernel: the pool has adapters of a lower rank than its own
    int x_stream;            // decode kernel, K-split form: x rows loaded with the streaming hint (ranks 8, 16: as whole lines)
    SegParams seg;
};

// What the front of the expand looks like decides a small call: 1.4 us of a launch's 5 us went into scalar loads
// that waited for one another (arguments, tile count, a projection's arguments by a run-time index, tile record,
// table entry) and into two divisions.  So the arguments that every wave needs lie together, those of a projection
// in a structure that one load fetches beside the tile count and the record, and divisors come as FastDiv.
struct ExpandProj {          // one projection of an expand: a wave reads the one it works on, with one scalar load
    const float *v;
    void *y;
    int64_t ldy;
    void *img;               // long-segment kernel: operand images of the 16-row sub-tiles
    int h_out;
    int n_chunks;            // 128-column chunks
    int cps;                 // decode kernel: chunks per wave item (the last of a row may have fewer)
    int slice0;              // first wave item of the projection within a tile (long segments: chunk)
};

struct ExpandParams {
    const Unit *units;
    const lora_tile *tiles;
    const int32_t *counts;
    const int32_t *perm;
    int n_proj;
    int proj0;
    int n_fused;             // 1 .. kMaxFused consecutive projections; their widths may differ
    int P;
    int n_parts;             // long-segment kernels: the most parts there may be (long_split)
    int per_tile;            // wave items of a tile (one-launch kernel: workgroup items; long segments: chunks)
    int slice1, slice2;      // slice0 of the second and the third projection, per_tile where there is none
    FastDiv group_items;     // division by the wave items of a tile group (one-launch kernel: of a tile)
    int grid;
    ExpandProj proj[kMaxFused];
    int image_grid;          // long-segment kernel: workgroups of the image launch
    int waves;               // waves per workgroup
    int tile_halves;         // decode kernel: the tiles have up to 32 rows and are taken in halves
    union {
        int group_shift;     // decode kernel: consecutive wave items walk over 2^group_shift tiles
        int kblocks;         // long-segment kernels: K-blocks of the input
    };
    int item_shift;          // long-segment kernel: consecutive wave items take the tile groups of a run of 2^item_shift, then chunks
    int out_f32;
    int overwrite;           // decode kernel, bf16 output: write the update, do not read the rows
    int deep;                // decode kernel: two chunks in flight per wave, else one
    int lower_ranks;         // decode kernel: the pool has adapters of a lower rank than its own
    int share_b;             // decode kernel: B of full tiles loaded without the streaming hint
    int y_stream;            // decode kernel: output rows read and written with the streaming hint
    int rank;
};

// routing-weighted combine of per-pair update rows into token rows
struct CombineParams {
    const uint16_t *pair;    // bf16 [P][ld_pair] per-pair updates (rows of inactive pairs unspecified)
    int64_t ld_pair;
    const int32_t *adapter_id;
    const int32_t *expert_id;
    const float *route_w;    // [P]
    int T, top_k;
    int n_adapters, n_experts;
    int h_out;
    int waves;               // waves per token; these two are filled by launch_combine
    FastDiv waves_div;
    uint16_t *y;             // bf16 [T][ldy] token rows, updated in place
    int64_t ldy;
};

// shrink and expand of a decode batch in one launch
struct FusedParams {
    ShrinkParams s;          // n_parts = 1; v unused
    ExpandParams e;          // slices: workgroup items of a tile; v, cps unused
};

hipError_t launch_pack_layer(PackLayerParams &p, hipStream_t s);
hipError_t launch_unpack_A(const PackParams &p, hipStream_t s);   // src = packed, dst = row-major
hipError_t launch_unpack_B(const PackParams &p, hipStream_t s);
hipError_t launch_set_adapter(Unit *table, int n_layers, int n_adapters, int per_adapter, int adapter,
                              int rank, float scale, hipStream_t s);
hipError_t launch_segments(const SegParams &p, void *ws, hipStream_t s);
hipError_t launch_segments_large(const SegParams &p, void *ws, hipStream_t s);
size_t segments_large_ws_bytes(int P);
int inline_build_max_rows();      // limits of the segment build inside the decode shrink
int inline_build_max_keys();
bool segments_large_handles(const SegParams &p);    // does the multi-workgroup builder take this batch?
int segments_large_launches(const SegParams &p);    // kernels it enqueues for it
hipError_t launch_shrink(const ShrinkParams &p, hipStream_t s);
hipError_t launch_expand(const ExpandParams &p, hipStream_t s);
size_t expand_image_bytes(int rank, int64_t n_tiles);   // operand images of n_tiles 32-row tiles
// tiles per wave item of launch_expand: 16 KiB of output rows, all of which a wave has in registers
__host__ __device__ constexpr int expand_long_group(bool f32) { return f32 ? 1 : 2; }
hipError_t launch_shrink_decode(const ShrinkParams &p, hipStream_t s);   // tiles of <= 16 rows
hipError_t launch_expand_decode(const ExpandParams &p, hipStream_t s);
hipError_t launch_fused_decode(const FusedParams &p, hipStream_t s);
hipError_t launch_combine(const CombineParams &p, hipStream_t s);
int combine_max_top_k();
hipError_t launch_fill_zero(void *dst, size_t bytes, hipStream_t s);      // bytes a multiple of 16

}  // namespace lora

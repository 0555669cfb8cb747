// The wave-level work of the decode expand (tiles of at most 16 rows): one wave adds scale * v * B
// to the rows of one tile over a run of 128-column chunks.  (The kernel that runs shrink and expand
// in one launch uses ExpandWave on its own.)
//
// Prologue: the wave adds the K parts of the tile's v in a fixed order, applies the adapter's
// scale and splits the result into bf16 hi + lo planes held in MFMA operand registers (hi = v
// truncated to bf16, lo = the rounded remainder, so the product sees about 16 mantissa bits of
// v).  Main loop over the chunks, one or two of them in flight (the first ones' loads are issued before
// v is fetched): the packed B tile and the base-output rows of a chunk are fetched while others, of
// this wave or of the CU's other waves, are multiplied and written back (B with nontemporal loads: it is
// read once; y with ordinary accesses: read-modify-write runs faster through the L2).  All loads
// in the loop are unconditional and the loop is specialised on the number of row quads, so the
// code is straight-line and the hardware counters let the next chunk's loads stay outstanding
// across the current chunk's compute.
//
// A wave's start is a chain of dependent loads, and for a small batch that chain is the launch: arguments -> tile
// record, count, projection (together, expand_decode.hip) -> table entry, row indices, parts of v -> B, output
// rows.  With the loads of a link issued together and the row indices looked at only behind the loads of v and B:
// llama shapes, 256 rows 60.7 -> 56.2 us for the layer (four expands), 8 rows 34.6 -> 32.2, 333 ragged fp32 rows at
// rank 32 64.3 -> 60.0, Mixtral shapes, 64 tokens with the combine 46.5 -> 44.2, 512 tokens 104.3 -> 102.1.
//
// Row placement: tile row r sits in MFMA row slot (r % 4) * 4 + r / 4, so result register i of
// lane group g is row 4*i + g.  A tile of n rows then needs only ceil(n / 4) y loads and stores
// per chunk, each with all four lane groups busy (16 lanes cover 256 contiguous bytes of a row),
// instead of four quarter-empty ones.  B is streamed exactly once per (tile, chunk); after the
// eight MFMAs of a chunk a lane owns eight consecutive output columns of each of its rows.
#pragma once
#include <type_traits>

#include "expand_common.h"
#include "lora_internal.h"

namespace lora {

// OVW: the output rows are written, not updated: the base output counts as zero and is never
// read (used when the update goes to a buffer of its own rather than into base rows).
// YNT: the output rows are read and written with the streaming hint (for callers whose outputs
// are not in a cache when the call starts, or are too large to be).
// BNT: B is loaded with the streaming hint (it is read once), else left in the L2 for the other tiles
// of the segment.
// LOW: the pool has adapters of a lower rank than its own, whose zeros are not fetched: a buffer load beyond the
// buffer's records returns zeros without an access.  Layer call in us, everything fetched / not, half of the adapters with half
// the pool's rank: Mixtral shapes, 512 tokens, rank 16 102.4 / 88.4, rank 32 170 / 140, llama shapes, 256 rows,
// rank 64 137 / 122, ragged fp32 rows at rank 32 58.3 / 56.4, rank 8 (half lines of A) 49.0 / 48.6.  With adapters of the
// pool's rank only, plain loads are ahead (64 tokens with the combine 43.7 against 44.1, fine-grained MoE 133.3 / 134.3).
// D: chunks in flight per wave, one or two.  Two take the registers of a fifth wave per SIMD at rank 16
// (the third at rank 64); the host picks (three or four for the small rank-8 chunks measured no faster).
template <int R, bool F32, int NI, bool OVW, bool YNT, bool BNT, int D, bool LOW>
struct ExpandWave {
    using Tile = ExpandTile<R>;
    static constexpr int KS = Tile::KS;
    static constexpr int NY = F32 ? 2 : 1;
    static constexpr int ESZ = F32 ? 4 : 2;

    struct YBuf {
        u32x4 r[NI][NY];
    };

    int lane, g, i16, h_out;
    const uint16_t *Bp;
    typename Tile::Lanes at_b;
    char *yrow[NI];          // y rows of result registers 0..NI-1 (a valid row even if unused)
    bool rok[NI];            // whether result register i belongs to a row of the tile
    typename Tile::A a;

    __device__ inline void load(int c, typename Tile::B &b, YBuf &y) const
    {
        Tile::template load_b<BNT, LOW>(Bp, c, at_b, b);
        load_y(c, y);
    }

    __device__ inline void load_y(int c, YBuf &y) const
    {
        const int col = c * kColChunk + i16 * 8;
        const int colc = col < h_out ? col : 0;
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int q = 0; q < NY; ++q)
                y.r[i][q] = OVW ? u32x4{0u, 0u, 0u, 0u} : ld16<YNT>(yrow[i] + (int64_t)colc * ESZ + 16 * q);
    }

    __device__ inline void compute_store(int c, const typename Tile::B &b, const YBuf &y) const
    {
        f32x4 acc[8];
        Tile::mma(a, b, acc);
        const int col = c * kColChunk + i16 * 8;
        const bool col_ok = col < h_out;
        // the sums are formed for every lane; only the store itself is predicated
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            char *yp = yrow[i] + (int64_t)col * ESZ;
            const bool ok = col_ok && rok[i];
            if (F32) {
                u32x4 o0, o1;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    o0[q] = __float_as_uint(__uint_as_float(y.r[i][0][q]) + acc[q][i]);
                    o1[q] = __float_as_uint(__uint_as_float(y.r[i][NY - 1][q]) + acc[4 + q][i]);
                }
                if (ok) {
                    st16<YNT>(yp, o0);
                    st16<YNT>(yp + 16, o1);
                }
            } else {
                u32x4 o;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const unsigned u = y.r[i][0][q];
                    const float f0 = __uint_as_float(u << 16) + acc[2 * q][i];
                    const float f1 = __uint_as_float(u & 0xFFFF0000u) + acc[2 * q + 1][i];
                    o[q] = pack_bf16_rne(f0, f1);
                }
                if (ok) st16<YNT>(yp, o);
            }
        }
    }

    struct Stage {
        typename Tile::B b;
        YBuf y;
    };

    // issue the loads of the first D chunks of [c0, c1) (a slice shorter than D repeats its
    // last chunk; the repeats are never used)
    __device__ inline void prefetch_b(int c0, int c1, Stage (&st)[D]) const
    {
#pragma unroll
        for (int k = 0; k < D; ++k) Tile::template load_b<BNT, LOW>(Bp, min(c0 + k, c1 - 1), at_b, st[k].b);
    }

    __device__ inline void prefetch_y(int c0, int c1, Stage (&st)[D]) const
    {
#pragma unroll
        for (int k = 0; k < D; ++k) load_y(min(c0 + k, c1 - 1), st[k].y);
    }

    // chunks [c0, c1) after their first ones are in flight: D of them at a time; every load in the loop body is
    // unconditional
    __device__ inline void run(int c0, int c1, Stage (&st)[D]) const
    {
        int c = c0;
        for (; c + D < c1; c += D) {
#pragma unroll
            for (int k = 0; k < D; ++k) {
                compute_store(c + k, st[k].b, st[k].y);
                load(min(c + k + D, c1 - 1), st[k].b, st[k].y);
            }
        }
#pragma unroll
        for (int k = 0; k < D; ++k)
            if (c + k < c1) compute_store(c + k, st[k].b, st[k].y);      // wave-uniform
    }
};

template <int R, bool F32, int NI, bool OVW, bool YNT, bool BNT, int D, bool LOW>
__device__ inline void expand_item(const ExpandParams &p, const ExpandProj &pe, const lora_tile &t,
                                   const Unit &unit, int c0, int c1, int lane)
{
    using Tile = ExpandTile<R>;
    constexpr int KS = Tile::KS, KV = Tile::KV, ESZ = F32 ? 4 : 2;
    using Wave = ExpandWave<R, F32, NI, OVW, YNT, BNT, D, LOW>;
    Wave w;
    asm volatile("" : "+v"(lane));               // keeps what follows from the lane out of registers of the item loop
    w.lane = lane;
    w.g = lane >> 4;
    w.i16 = lane & 15;
    w.h_out = pe.h_out;
    w.Bp = unit.B;
    const float scale = unit.scale;
    int dst[NI];             // row indices: asked for first, looked at behind the loads of v and B
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int r = 4 * i + w.g;                       // row of result register i
        w.rok[i] = r < t.n_rows;
        dst[i] = p.perm[t.row0 + min(r, t.n_rows - 1)];
    }

    // v operand: this lane's row slot i16 holds tile row (i16 % 4) * 4 + i16 / 4.  The loads of
    // the K parts (PB rounds at a time) are issued before anything is added, and before the first
    // chunks' weights and base output, so that the wait for v leaves those in flight; a part
    // beyond the last re-reads the last one and counts as zero.
    //
    // Loads return in order, so parts that are fetched behind the first chunks wait for those as well:
    // one round trip more for every batch after the first.  Therefore a batch is PB * PQ parts: where a tile has at most
    // four (eight) rows, the four (two) lanes of a quad whose row slots share the lane's tile row or are empty
    // fetch a part each.  Batches that eight parts (a decode shrink has no more) come in: one for tiles of up to four rows;
    // for up to eight rows one at ranks 8 to 32, two at rank 64 (four with fp32 output); above two, at rank 64 four (eight).
    // Every lane of the quad adds all parts in ascending order through the cross-lane data path, so a row's sum is the
    // same in tiles of every height.
    constexpr int PQ = NI == 1 ? 4 : NI == 2 ? 2 : 1;            // parts per round, one per lane of a row
    constexpr int PB = R <= 32 ? (NI == 1 ? 2 : 4) : NI == 1 ? 2 : (F32 ? 1 : 2);      // registers permitting
    const int slot = w.i16;
    const int row = NI == 1 ? slot >> 2 : NI == 2 ? (slot & 1) * 4 + (slot >> 2) : (slot & 3) * 4 + (slot >> 2);
    const int sub = NI == 1 ? slot & 3 : NI == 2 ? (slot & 3) >> 1 : 0;
    const bool valid = row < t.n_rows && sub == 0;
    const unsigned vrow = (unsigned)(t.row0 + min(row, t.n_rows - 1)) * (R * 4);      // bytes; a part is at most 2^28 of them
    const int64_t part_stride = (int64_t)p.P * (R * 4);
    auto load_v = [&](int part0, f32x4 (&buf)[PB][KS][KV / 4]) {
#pragma unroll
        for (int u = 0; u < PB; ++u) {
            const char *src = reinterpret_cast<const char *>(pe.v) + min(part0 + u * PQ + sub, p.n_parts - 1) * part_stride;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int h = 0; h < KV / 4; ++h) 
                    buf[u][ks][h] = ld16f(reinterpret_cast<const float *>(src + (vrow + (Tile::jbase(w.g, ks) + 4 * h) * 4u)));
        }
    };
    float s[KS][KV];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int q = 0; q < KV; ++q) s[ks][q] = 0.f;
    auto add_v = [&](int part0, const f32x4 (&buf)[PB][KS][KV / 4]) {
#pragma unroll
        for (int u = 0; u < PB; ++u) {
            const bool in = part0 + u * PQ + sub < p.n_parts;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int h = 0; h < KV / 4; ++h)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float x = in ? buf[u][ks][h][q] : 0.f;
                        float &to = s[ks][4 * h + q];
                        if (PQ == 1) to += x;
                        if (PQ == 2) to = (to + quad_lane<0x44>(x)) + quad_lane<0xEE>(x);
                        if (PQ == 4) to = (((to + quad_lane<0x00>(x)) + quad_lane<0x55>(x)) + quad_lane<0xAA>(x)) + quad_lane<0xFF>(x);
                    }
        }
    };
    typename Wave::Stage st[D];
    // the first chunks' weights and base output, behind the loads of v: only the output rows wait for
    // the row indices
    auto prefetch = [&] {
        w.at_b = Tile::lanes_of(lane, LOW && unit.b_rank ? unit.b_rank : R);
        w.prefetch_b(c0, c1, st);
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            asm volatile("" : "+v"(dst[i]));      // here, and not where the two uses of this code part
            w.yrow[i] = static_cast<char *>(pe.y) + (int64_t)dst[i] * pe.ldy * ESZ;
        }
        w.prefetch_y(c0, c1, st);
    };
    if (p.n_parts == 1) {                                 // a single part: one load, no batch
        f32x4 one[KS][KV / 4];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int h = 0; h < KV / 4; ++h) 
                one[ks][h] = ld16f(reinterpret_cast<const float *>(reinterpret_cast<const char *>(pe.v) +
                                                                   (vrow + (Tile::jbase(w.g, ks) + 4 * h) * 4u)));
        __builtin_amdgcn_sched_barrier(0);                       // v first: everything waits for it
        prefetch();
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int h = 0; h < KV / 4; ++h)
#pragma unroll
                for (int q = 0; q < 4; ++q) s[ks][4 * h + q] = one[ks][h][q];
    } else {
        f32x4 vbuf[PB][KS][KV / 4];
        load_v(0, vbuf);
        __builtin_amdgcn_sched_barrier(0);                       // v first: everything waits for it
        prefetch();
        add_v(0, vbuf);
        for (int part0 = PB * PQ; part0 < p.n_parts; part0 += PB * PQ) {
            load_v(part0, vbuf);
            add_v(part0, vbuf);
        }
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        float sc[KV];
#pragma unroll
        for (int q = 0; q < KV; ++q) sc[q] = valid ? s[ks][q] * scale : 0.f;
        Tile::make_a(sc, w.g, ks, w.a);
    }
    w.run(c0, c1, st);
}

// one wave, one tile, chunks [c0, c1) of projection pj; the specialisation on the number of row
// quads is picked here (wave-uniform)
template <int R, bool F32, bool OVW, bool YNT, int D, bool LOW>
__device__ inline void expand_tile_chunks(const ExpandParams &p, const ExpandProj &pe, const lora_tile &t,
                                          const Unit &unit, int c0, int c1, int lane)
{
    switch ((t.n_rows + 3) >> 2) {
    case 1: expand_item<R, F32, 1, OVW, YNT, true, D, LOW>(p, pe, t, unit, c0, c1, lane); break;
    case 2: expand_item<R, F32, 2, OVW, YNT, true, D, LOW>(p, pe, t, unit, c0, c1, lane); break;
    case 3: expand_item<R, F32, 3, OVW, YNT, true, D, LOW>(p, pe, t, unit, c0, c1, lane); break;
    default:
        // a full tile is most likely one of several of its segment: its B is worth keeping in the L2
        if (p.share_b && t.n_rows == kDecodeTileRows)
            expand_item<R, F32, 4, OVW, YNT, false, D, LOW>(p, pe, t, unit, c0, c1, lane);
        else
            expand_item<R, F32, 4, OVW, YNT, true, D, LOW>(p, pe, t, unit, c0, c1, lane);
        break;
    }
}

}  // namespace lora

// Shrink and expand of a small decode batch in one launch (Sec. 5.2 discusses scheduling the
// LoRA computation with few, persistent launches; a decode layer call is short enough for
// every dependent launch to show).  For tiles of at most 16 rows and few tiles.
//
// Work item (per workgroup) = (row tile, projection, slice of as many 128-column chunks as the
// workgroup has waves).  The workgroup first computes the tile's whole v = gather(x) * A for its
// projection, the waves splitting the K range; their sums meet in LDS, behind the only barrier
// of an item every wave adds them in a fixed order straight into its MFMA operand, and then does
// what a wave of the expand kernel does (scale, hi/lo split, multiply with B, add into the tile's
// output rows) on its own chunk.
//
// The workgroups of one (tile, projection) all repeat the same shrink: A is fetched from HBM
// once and then served by the L2 to the other slices.  That trade is what makes one launch
// possible without any hand-off between workgroups: nobody waits for anybody, there is no
// intermediate in global memory, no counter, no fence, and the kernel cannot deadlock.
//
// What bounds it is the latency of that chain and the rate at which one CU fetches A (128 KiB at
// rank 16 and 4096 inputs), not the chip's bandwidth.  So the chain is kept short: the chunk's B and
// the output rows, which do not depend on v, are fetched behind the first loads of A and x, and the
// sums cross LDS once.  Measured, whole call of one 4096 -> 4096 projection at rank 16 and of 64
// rows of 1024 -> 1024 at rank 8: 7.6 -> 6.6 us and 6.9 -> 6.0 us (four waves, B and rows fetched
// behind the shrink, two barriers).  Sixteen waves (7.6 and 6.6) and four steps of A in flight
// instead of two (9.1 and 6.3) are slower: more loads at once do not come faster to one CU.
//
// Sums are formed in a fixed order, so results are bit-identical run to run.  The K range is
// split over the waves differently from the two-launch path (which also splits it over
// workgroups), so the two paths agree to fp32 rounding, not bit for bit.
#include <type_traits>

#include "expand_item.h"
#include "segments_inline.h"
#include "shrink_wave.h"

namespace lora {

namespace {

// BUILD: the segments are not there yet either; every workgroup sorts the batch for itself in LDS
// first (segments_inline.h), workgroup 0 writes the segments out, and the whole layer call of a
// small batch is this one launch.
// LOW: as in the two-launch kernels, for pools with adapters of a lower rank than their own.  Pools without, LOW form / plain
// loads, us per call of 4096 -> 4096: 1 row at rank 8 6.1 / 6.0, 8 rows at rank 16 7.2 / 7.1, 24 rows 9.1 / 8.9, 8 rows at
// rank 32 9.1 / 9.0, at rank 64 9.4 / 9.6; llama shapes with 8 rows 32.8 / 31.7.
template <int R, bool BUILD, bool LOW>
__global__ __launch_bounds__(64 * kFusedWaves) void fused16_kernel(FusedParams p,
                                                         const lora_tile *__restrict__ tiles,
                                                         const Unit *__restrict__ units,
                                                         const int32_t *__restrict__ counts)
{
    constexpr int NW = kFusedWaves;
    using Wave = ShrinkWave<R, 1, false, false, false, LOW>;
    using Out = ExpandWave<R, false, 4, false, false, true, 1, LOW>;
    using Tile = ExpandTile<R>;
    constexpr int NACC = Wave::NACC, KU = Wave::KU, KS = Tile::KS, KV = Tile::KV, ESZ = Out::ESZ;
    union Scratch {                   // the build's counts are dead before the first sums are added
        f32x4 red[NW][NACC][64];
        std::conditional_t<BUILD, InlineCounts, char> counts;
    };
    __shared__ Scratch scratch;
    __shared__ std::conditional_t<BUILD, InlineSegments, char> built;
    auto &red = scratch.red;

    const ShrinkParams &sp = p.s;
    const ExpandParams &ep = p.e;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    Wave w;
    w.lane = tid & 63;
    w.g = w.lane >> 4;
    w.i16 = w.lane & 15;
    w.h_in = sp.h_in;
    int n_tiles;
    if constexpr (BUILD) {
        build_segments_inline<NW>(sp.seg, scratch.counts, built, blockIdx.x == 0);   // `built` is complete behind its last barrier
        n_tiles = built.n_tiles;
    } else {
        n_tiles = counts[2];
    }
    const int per_tile = ep.per_tile;                            // workgroup items of one tile
    const int n_items = n_tiles * per_tile;
    const int kblocks = (sp.h_in + KU - 1) / KU;

    for (int item = blockIdx.x; item < n_items; item += gridDim.x) {
        const int tile_ix = item / ep.group_items;
        const int rem = item - tile_ix * per_tile;
        const int pj = (rem >= ep.slice1 ? 1 : 0) + (rem >= ep.slice2 ? 1 : 0);
        const ExpandProj &pe = ep.proj[pj];
        const int slice = rem - pe.slice0;
        lora_tile t;
        if constexpr (BUILD) {
            t = built.tiles[tile_ix];                            // the same for every lane: scalars from here on
            t.key = __builtin_amdgcn_readfirstlane(t.key);
            t.row0 = __builtin_amdgcn_readfirstlane(t.row0);
            t.n_rows = __builtin_amdgcn_readfirstlane(t.n_rows);
        } else {
            t = tiles[tile_ix];
        }
        const Unit unit = units[(int64_t)t.key * sp.n_proj + sp.proj0 + pj];
        auto row_of = [&](int at) -> int {
            if constexpr (BUILD) return built.perm[at];
            else return sp.perm[at];
        };

        // this wave's chunk, and the output rows of result registers 0..3
        const int c0 = slice * NW + wave;
        const bool has_chunk = c0 < pe.n_chunks;             // wave-uniform
        Out out;
        out.lane = w.lane;
        out.g = w.g;
        out.i16 = w.i16;
        out.h_out = pe.h_out;
        out.Bp = unit.B;
        out.at_b = Tile::lanes_of(w.lane, LOW && unit.b_rank ? unit.b_rank : R);
        w.set_rank(LOW && unit.a_rank ? unit.a_rank : R);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = 4 * i + w.g;
            out.rok[i] = r < t.n_rows;
            out.yrow[i] = static_cast<char *>(pe.y) + (int64_t)row_of(t.row0 + min(r, t.n_rows - 1)) * pe.ldy * ESZ;
        }
        typename Tile::B b;
        typename Out::YBuf y;

        // ---- shrink: this tile, this projection, the whole K range over the waves ----------------
        w.Ap[0] = unit.A;
        int at = row_of(t.row0 + min(w.i16, t.n_rows - 1));
        if (sp.src_row) at = sp.src_row[at];
        auto rows = [&] {
            asm volatile("" : "+v"(at));
            w.xp = sp.x + (int64_t)at * sp.ldx;
        };
        // a wave without a chunk re-reads the last one and does not use it: no branch around loads
        w.run(wave * Wave::KB, kblocks, NW * Wave::KB, rows,
              [&] { out.load(min(c0, pe.n_chunks - 1), b, y); });
#pragma unroll
        for (int a = 0; a < NACC; ++a) red[wave][a][w.lane] = w.acc[0][a];
        __syncthreads();

        // ---- expand: the waves' sums in a fixed order are v; row slot i16 holds tile row `row` ---
        if (has_chunk) {
            const int row = (w.i16 & 3) * 4 + (w.i16 >> 2);
            const bool valid = row < t.n_rows;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                float sc[KV];
#pragma unroll
                for (int h = 0; h < KV / 4; ++h) {
                    // entries j .. j + 3 of the row: accumulator j / 16, lane (j % 16) / 4 * 16 + row
                    const int j = Tile::jbase(w.g, ks) + 4 * h;
                    const int a = R >= 16 ? j >> 4 : 0, l = (R >= 16 ? (j & 15) >> 2 : j >> 2) * 16 + row;
                    f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int k = 0; k < NW; ++k) {
                        s += red[k][a][l];
                        if (R == 8) s += red[k][NACC - 1][l + 32];
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q) sc[4 * h + q] = valid ? s[q] * unit.scale : 0.f;
                }
                Tile::make_a(sc, w.g, ks, out.a);
            }
            out.compute_store(c0, b, y);
        }
        __syncthreads();              // red is reused by the next item
    }
}

template <int R, bool LOW>
hipError_t launch_r(const FusedParams &p, hipStream_t s)
{
    constexpr int kThreads = 64 * kFusedWaves;
    if (p.s.build) {
        if (p.s.seg.P > kInlineMaxRows || p.s.seg.n_adapters * (int64_t)p.s.seg.n_experts > kInlineMaxKeys)
            return hipErrorInvalidValue;
        hipLaunchKernelGGL((fused16_kernel<R, true, LOW>), dim3(p.s.grid), dim3(kThreads), 0, s, p, p.s.tiles,
                           p.s.units, p.s.counts);
    } else {
        hipLaunchKernelGGL((fused16_kernel<R, false, LOW>), dim3(p.s.grid), dim3(kThreads), 0, s, p, p.s.tiles,
                           p.s.units, p.s.counts);
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_fused_decode(const FusedParams &p, hipStream_t s)
{
    if (p.s.grid <= 0) return hipSuccess;
    switch (p.s.rank) {
    case 8: return p.s.lower_ranks ? launch_r<8, true>(p, s) : launch_r<8, false>(p, s);
    case 16: return p.s.lower_ranks ? launch_r<16, true>(p, s) : launch_r<16, false>(p, s);
    case 32: return p.s.lower_ranks ? launch_r<32, true>(p, s) : launch_r<32, false>(p, s);
    case 64: return p.s.lower_ranks ? launch_r<64, true>(p, s) : launch_r<64, false>(p, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace lora

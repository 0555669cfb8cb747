// Shrink for decode batches (tiles of at most 16 rows): v = gather(x) * A.
//
// Two ways of dealing out the work, chosen on the host:
//  * K split: work item = (row tile, K part); a workgroup of four waves takes one item, each
//    wave owns a quarter of the part's K range, and the four waves' sums are added through
//    LDS in a fixed order.  For batches with few tiles and long inputs.
//  * wave per tile: every wave takes a whole tile over the whole K range, no LDS, no barrier.
//    For batches with thousands of small tiles and short inputs (fine-grained MoE).
// In both a wave streams its slice of the packed A (and of the second fused projection's A)
// with 16-byte loads that are contiguous per wave, two steps in flight (shrink_wave.h), and multiplies it
// with the tile's gathered x rows.  The rank index sits on the M side of v_mfma_f32_16x16x32_bf16 and
// the rows on the N side, so a lane ends up with four consecutive rank entries of one row.
//
// Rank 8: a packed block holds 64 K values (two 32-deep halves side by side in the 16 M
// rows), is multiplied once with each half's x values, and rows 0..7 of the first product
// plus rows 8..15 of the second give the eight rank entries.
#include <type_traits>

#include "segments_inline.h"
#include "shrink_wave.h"

namespace lora {

namespace {

// tiles, units and counts are passed again as restrict-qualified kernel arguments: with a
// uniform index the compiler then reads them through the scalar cache, which shortens the
// dependent chain tile -> unit -> first data load.
//
// BUILD: the segments are not there yet; every workgroup sorts the batch for itself in LDS
// first (segments_inline.h) and takes tile records and row indices from there, and workgroup 0
// writes them out for the launches that follow.
//
// HALVES (rank 16): the tiles have up to 32 rows and are taken in halves.
// XNT: the x rows are loaded with the streaming hint (K-split form only).
// LINES: the x rows are fetched as whole cache lines and transposed through LDS (shrink_wave.h;
// K-split form, ranks 8 to 32).  Used together with XNT: a streamed line that is fetched in two
// halves by two instructions is fetched twice.  Measured on MI355X (rank 16, 14336 inputs): 4096
// rows of the Mixtral down projection 48.5 -> 41.7 us, of the Llama one 60.9 -> 51.0 us for the
// whole application; with inputs that stay cached (4096 wide, or few rows) it costs 5-10 %.  Rank 32,
// Mixtral shapes, 1024 tokens, streamed inputs that were just written: 266.0 -> 257.8 us (258.5 unstreamed).
template <int R, int NPROJ, bool NT, bool WPT, bool BUILD, bool XNT, bool LINES, bool HALVES, bool LOW>
__global__ __launch_bounds__(256, 2) void shrink16_kernel(ShrinkParams p,
                                                          const lora_tile *__restrict__ tiles,
                                                          const Unit *__restrict__ units,
                                                          const int32_t *__restrict__ counts)
{
    using Wave = ShrinkWave<R, NPROJ, NT, XNT, LINES, LOW>;
    constexpr int NACC = Wave::NACC, KU = Wave::KU;
    static_assert(!(BUILD && WPT), "the build needs the whole workgroup");
    static_assert(!(XNT && (BUILD || WPT)), "streamed x rows: K-split form without the build only");
    static_assert(!(LINES && WPT), "whole-line rows: K-split form only");
    union Scratch {                   // the build's counts are dead before the first sums are added
        f32x4 red[WPT ? 1 : 4][NPROJ][NACC][WPT ? 1 : 64];
        std::conditional_t<BUILD, InlineCounts, char> counts;
    };
    __shared__ Scratch scratch;
    __shared__ std::conditional_t<BUILD, InlineSegments, char> built;
    __shared__ u32x4 xt_all[LINES ? 4 * 64 * Wave::NQ : 1];      // LINES: NQ KiB per wave
    auto &red = scratch.red;

    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    Wave w;
    w.lane = tid & 63;
    w.g = w.lane >> 4;
    w.i16 = w.lane & 15;
    w.h_in = p.h_in;
    w.xt = xt_all + (LINES ? wave * 64 * Wave::NQ : 0);
    if constexpr (BUILD)
        build_segments_inline<4>(p.seg, scratch.counts, built, blockIdx.x == 0);   // `built` is complete behind its last barrier
    const int kblocks = (p.h_in + KU - 1) / KU;

    // item loop: a workgroup's item in the K-split form, a wave's item otherwise
    const int first = WPT ? (int)blockIdx.x * 4 + wave : blockIdx.x;
    const int stride = WPT ? p.grid * 4 : p.grid;
    for (int item = first;; item += stride) {
        const int tile_ix = item / p.parts;
        const int part = item - tile_ix * p.n_parts;
        lora_tile t;
        if constexpr (BUILD) {
            if (tile_ix >= built.n_tiles) break;
            t = built.tiles[tile_ix];                 // the same for every lane: scalars from here on
            t.key = __builtin_amdgcn_readfirstlane(t.key);
            t.row0 = __builtin_amdgcn_readfirstlane(t.row0);
            t.n_rows = __builtin_amdgcn_readfirstlane(t.n_rows);
        } else {
            // the number of tiles and the tile's record are fetched together; the record is looked at only
            // once the number says that there is one (the buffer has a record per row)
            const int count = counts[2];
            t = tiles[min(HALVES ? tile_ix >> 1 : tile_ix, p.P - 1)];
            asm volatile("" ::"s"(count), "s"(t.key), "s"(t.row0), "s"(t.n_rows));
            if (tile_ix >= (HALVES ? 2 * count : count)) break;
            if constexpr (HALVES) {                   // rows 0..15 or 16..31 of a 32-row tile
                const int off = (tile_ix & 1) * kDecodeTileRows;
                t.row0 += off;
                t.n_rows = min(t.n_rows - off, kDecodeTileRows);
                if (t.n_rows <= 0) continue;          // uniform over everyone who shares the item
            }
        }
        int rank = 0;
#pragma unroll
        for (int pj = 0; pj < NPROJ; ++pj) {
            const Unit &unit = units[(int64_t)t.key * p.n_proj + p.proj0 + pj];
            w.Ap[pj] = unit.A;
            rank = max(rank, LOW && unit.a_rank ? unit.a_rank : R);
        }
        w.set_rank(rank);
        const bool row_ok = w.i16 < t.n_rows;
        // Row indices: asked for here, looked at behind the first loads of A.  (Loads return in order, so the second
        // look-up has to be in front of those.)
        int at[LINES ? Wave::NQ : 1];
#pragma unroll
        for (int q = 0; q < (LINES ? Wave::NQ : 1); ++q) {
            const int row = t.row0 + min(LINES ? Wave::RPI * q + w.lane / Wave::PPR : w.i16, t.n_rows - 1);
            if constexpr (BUILD) at[q] = built.perm[row];
            else at[q] = p.perm[row];
        }
        if (p.src_row) {
#pragma unroll
            for (int q = 0; q < (LINES ? Wave::NQ : 1); ++q) at[q] = p.src_row[at[q]];
        }
        auto rows = [&] {
#pragma unroll
            for (int q = 0; q < (LINES ? Wave::NQ : 1); ++q) asm volatile("" : "+v"(at[q]));
            if constexpr (LINES) {
#pragma unroll
                for (int q = 0; q < Wave::NQ; ++q) w.xq[q] = p.x + (int64_t)at[q] * p.ldx;
            } else {
                w.xp = p.x + (int64_t)at[0] * p.ldx;
            }
        };
        const int part_begin = part * p.kb_per_part;
        const int part_end = min(part_begin + p.kb_per_part, kblocks);

        if constexpr (WPT) {
            w.run(part_begin, part_end, Wave::KB, rows, [] {});
            // lane (row i16, group g) holds rank entries 4g..4g+3 of its row; for rank 8 the
            // entries of groups 2,3 belong to the second half product and are added to the
            // first half's entries held 32 lanes below
#pragma unroll
            for (int pj = 0; pj < NPROJ; ++pj) {
                if (R == 8) {
                    f32x4 s = w.acc[pj][0];
#pragma unroll
                    for (int q = 0; q < 4; ++q) s[q] += __shfl_down(w.acc[pj][1][q], 32, 64);
                    if (row_ok && w.g < 2)
                        st16f(p.v[pj] + ((int64_t)part * p.P + t.row0 + w.i16) * R + w.g * 4, s);
                } else {
#pragma unroll
                    for (int nb = 0; nb < Wave::NB; ++nb)
                        if (row_ok)
                            st16f(p.v[pj] + ((int64_t)part * p.P + t.row0 + w.i16) * R + nb * 16 + w.g * 4,
                                  w.acc[pj][nb]);
                }
            }
        } else {
            // the four waves take the part's steps in turn, so that together they read a
            // contiguous kilobyte or more of every x row (and of A) at about the same time
            w.run(part_begin + wave * Wave::KB, part_end, 4 * Wave::KB, rows, [] {});

            // add the four waves' sums in a fixed order and store this part of v
#pragma unroll
            for (int pj = 0; pj < NPROJ; ++pj)
#pragma unroll
                for (int a = 0; a < NACC; ++a) red[wave][pj][a][w.lane] = w.acc[pj][a];
            __syncthreads();
            constexpr int NOUT = NPROJ * (R == 8 ? 1 : NACC) * 64;
            for (int o = tid; o < NOUT; o += 256) {
                const int l = o & 63;
                const int a = R == 8 ? 0 : (o >> 6) % NACC;
                const int pj = R == 8 ? (o >> 6) : (o >> 6) / NACC;
                const int row = l & 15;
                const int j = a * 16 + (l >> 4) * 4;
                if (row < t.n_rows && j < R) {
                    f32x4 s;
                    if (R == 8) {
                        s = red[0][pj][0][l] + red[0][pj][1][l + 32];
                        s += red[1][pj][0][l] + red[1][pj][1][l + 32];
                        s += red[2][pj][0][l] + red[2][pj][1][l + 32];
                        s += red[3][pj][0][l] + red[3][pj][1][l + 32];
                    } else {
                        s = red[0][pj][a][l];
                        s += red[1][pj][a][l];
                        s += red[2][pj][a][l];
                        s += red[3][pj][a][l];
                    }
                    st16f(p.v[pj] + ((int64_t)part * p.P + t.row0 + row) * R + j, s);
                }
            }
            __syncthreads();
        }
    }
}

template <int R, int NPROJ, bool HALVES, bool LOW>
void launch_form(const ShrinkParams &p, hipStream_t s)
{
    if (p.wave_per_tile)
        hipLaunchKernelGGL((shrink16_kernel<R, NPROJ, true, true, false, false, false, HALVES, LOW>), dim3(p.grid), dim3(256), 0,
                           s, p, p.tiles, p.units, p.counts);
    else if (p.x_stream)       // large inputs that are read once: streamed, as whole lines where a step is 256 bytes of a row
        hipLaunchKernelGGL((shrink16_kernel<R, NPROJ, true, false, false, true, (R <= 32), HALVES, LOW>), dim3(p.grid),
                           dim3(256), 0, s, p, p.tiles, p.units, p.counts);
    else
        hipLaunchKernelGGL((shrink16_kernel<R, NPROJ, true, false, false, false, false, HALVES, LOW>), dim3(p.grid), dim3(256),
                           0, s, p, p.tiles, p.units, p.counts);
}

template <int R, int NPROJ, bool LOW>
hipError_t launch_rn(const ShrinkParams &p, hipStream_t s)
{
    if (p.build) {
        if (p.wave_per_tile || p.seg.P > kInlineMaxRows || p.seg.n_adapters * (int64_t)p.seg.n_experts > kInlineMaxKeys)
            return hipErrorInvalidValue;
        hipLaunchKernelGGL((shrink16_kernel<R, NPROJ, true, false, true, false, false, false, LOW>), dim3(p.grid), dim3(256), 0, s, p,
                           p.tiles, p.units, p.counts);
    } else if (p.tile_halves) {
        if constexpr (R == 16) launch_form<R, NPROJ, true, LOW>(p, s);
        else return hipErrorInvalidValue;             // the other ranks' 32-row tiles have kernels of their own
    } else {
        launch_form<R, NPROJ, false, LOW>(p, s);
    }
    return hipGetLastError();
}

template <int R>
hipError_t launch_r(const ShrinkParams &p, hipStream_t s)
{
    switch (p.n_fused) {
    case 1: return p.lower_ranks ? launch_rn<R, 1, true>(p, s) : launch_rn<R, 1, false>(p, s);
    case 2: return p.lower_ranks ? launch_rn<R, 2, true>(p, s) : launch_rn<R, 2, false>(p, s);
    case 3: return p.lower_ranks ? launch_rn<R, 3, true>(p, s) : launch_rn<R, 3, false>(p, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

int inline_build_max_rows() { return kInlineMaxRows; }
int inline_build_max_keys() { return kInlineMaxKeys; }

hipError_t launch_shrink_decode(const ShrinkParams &p, hipStream_t s)
{
    if (p.grid <= 0) return hipSuccess;
    switch (p.rank) {
    case 8: return launch_r<8>(p, s);
    case 16: return launch_r<16>(p, s);
    case 32: return launch_r<32>(p, s);
    case 64: return launch_r<64>(p, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace lora

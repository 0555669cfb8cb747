// Expand for decode batches (tiles of at most 16 rows): y[row] += scale * v[row] * B, with
// every wave working on its own, no LDS and no barriers.
//
// Work item (per wave) = (row tile, projection, slice of 128-column chunks); what a wave does
// with an item is in expand_item.h.
#include "expand_item.h"

namespace lora {

namespace {

// tiles, units and counts are passed again as restrict-qualified kernel arguments: with a
// wave-uniform index the compiler then reads them through the scalar cache, which shortens
// the dependent chain tile -> unit -> first data load.
template <int R, bool F32, bool OVW, bool YNT, int D, bool HALVES, bool LOW>
__global__ __launch_bounds__(256, 2) void expand16_kernel(ExpandParams p,
                                                          const lora_tile *__restrict__ tiles,
                                                          const Unit *__restrict__ units,
                                                          const int32_t *__restrict__ counts)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int gw = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + wave), nw = p.grid * 4;
    const int per_tile = p.per_tile;
    // Item order: tile_group consecutive items take the same (projection, slice) of
    // tile_group consecutive tiles, so the waves of a workgroup that work on tiles of one
    // segment ask for the same B chunk at about the same time and all but one are served by
    // the L2.  tile_group 1: consecutive items are the slices of one tile.
    const int gs = p.group_shift;

    for (int item = gw;; item += nw) {
        const int grp = item / p.group_items;
        const int in_grp = item - grp * (per_tile << gs);
        const int rem = in_grp >> gs;
        const int tile_ix = (grp << gs) + (in_grp - (rem << gs));
        const int pj = (rem >= p.slice1 ? 1 : 0) + (rem >= p.slice2 ? 1 : 0);
        // What does not depend on one another is fetched together: the number of tiles, the tile's record
        // (looked at only once the number says that there is one; the buffer has a record per row) and the
        // projection's parameters.
        const int count = counts[2];
        lora_tile t = tiles[min(HALVES ? tile_ix >> 1 : tile_ix, p.P - 1)];
        const ExpandProj q = p.proj[pj];
        asm volatile("" ::"s"(count), "s"(t.key), "s"(t.row0), "s"(t.n_rows), "s"(q.v), "s"(q.y), "s"(q.ldy),
                     "s"(q.h_out), "s"(q.n_chunks), "s"(q.cps), "s"(q.slice0));
        const int n_tiles = HALVES ? 2 * count : count;
        if (grp << gs >= n_tiles) break;
        if (tile_ix >= n_tiles) continue;
        const int c0 = (rem - q.slice0) * q.cps, c1 = min(c0 + q.cps, q.n_chunks);
        if (c0 >= c1) continue;
        if constexpr (HALVES) {                                   // rows 0..15 or 16..31 of a 32-row tile
            const int off = (tile_ix & 1) * kDecodeTileRows;
            t.row0 += off;
            t.n_rows = min(t.n_rows - off, kDecodeTileRows);
            if (t.n_rows <= 0) continue;
        }
        const Unit unit = units[(int64_t)t.key * p.n_proj + p.proj0 + pj];
        expand_tile_chunks<R, F32, OVW, YNT, D, LOW>(p, q, t, unit, c0, c1, lane);
        // A wave's last item ends here: no decoding of a next one.  Before another item the loads that the last chunks
        // repeated come in (vmcnt(0)), so that the compiler does not wait for them in the middle of the next item's first loads.
        if (item + nw >= ((n_tiles + (1 << gs) - 1) >> gs) * (per_tile << gs)) break;
        __builtin_amdgcn_s_waitcnt(0x0f70);
    }
}

template <int R, bool F32, bool OVW, bool YNT, int D, bool HALVES>
void launch_d(const ExpandParams &p, hipStream_t s)
{
    if (p.lower_ranks)
        hipLaunchKernelGGL((expand16_kernel<R, F32, OVW, YNT, D, HALVES, true>), dim3(p.grid), dim3(p.waves * 64), 0, s, p,
                           p.tiles, p.units, p.counts);
    else
        hipLaunchKernelGGL((expand16_kernel<R, F32, OVW, YNT, D, HALVES, false>), dim3(p.grid), dim3(p.waves * 64), 0, s, p,
                           p.tiles, p.units, p.counts);
}

// HALVES (rank 16 only): a kernel of its own, because looking at the tile height at run time cost the
// others 1-2 % (256 rows of the llama shapes 61.9 -> 63.0 us, fine-grained MoE 138.2 -> 139.0)
template <int R, bool F32, bool OVW, bool YNT>
void launch_o(const ExpandParams &p, hipStream_t s)
{
    if constexpr (R == 16) {
        if (p.tile_halves) {
            if (p.deep) launch_d<R, F32, OVW, YNT, 2, true>(p, s);
            else launch_d<R, F32, OVW, YNT, 1, true>(p, s);
            return;
        }
    }
    if (p.deep) launch_d<R, F32, OVW, YNT, 2, false>(p, s);
    else launch_d<R, F32, OVW, YNT, 1, false>(p, s);
}

template <int R, bool YNT>
hipError_t launch_ry(const ExpandParams &p, hipStream_t s)
{
    if (p.out_f32) launch_o<R, true, false, YNT>(p, s);
    else if (p.overwrite) launch_o<R, false, true, YNT>(p, s);
    else launch_o<R, false, false, YNT>(p, s);
    return hipGetLastError();
}

template <int R>
hipError_t launch_r(const ExpandParams &p, hipStream_t s)
{
    return p.y_stream ? launch_ry<R, true>(p, s) : launch_ry<R, false>(p, s);
}

}  // namespace

hipError_t launch_expand_decode(const ExpandParams &p, hipStream_t s)
{
    if (p.grid <= 0) return hipSuccess;
    if (p.tile_halves && p.rank != 16) return hipErrorInvalidValue;
    switch (p.rank) {
    case 8: return launch_r<8>(p, s);
    case 16: return launch_r<16>(p, s);
    case 32: return launch_r<32>(p, s);
    case 64: return launch_r<64>(p, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace lora

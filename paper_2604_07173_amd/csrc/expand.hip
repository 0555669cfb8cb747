// Expand with fused scale-and-accumulate for batches with long segments (tiles of up to 32
// rows): y[row] += scale * v[row] * B
// (App. A.2.2 "expand phase"; Sec. 2.2: the update is added to the base output; Fig. 7b:
// final addition of the two outputs).
//
// With long segments the traffic is the read-modify-write of y; B is small and stays in the
// L2.  Two launches:
//
// 1. operand images: one wave per 16-row sub-tile adds the K parts of v in a fixed order,
//    applies the adapter's scale and writes the sub-tile's MFMA operand exactly as the lanes
//    of the second kernel want it: two bf16 planes hi + lo (hi = v truncated to bf16, lo =
//    the rounded remainder, so the product sees about 16 mantissa bits of v), 64 lanes x 8
//    or 16 bytes per plane and K step.  This is done once per sub-tile instead of once per
//    (sub-tile, column chunk).
//
// 2. the product: every wave works on its own, no LDS and no barriers.  Work item (per
//    wave) = (group of two consecutive tiles, one with fp32 output; projection; 128-column chunk).  The
//    wave asks for everything at once - the rows' indices, the chunk's packed B in MFMA operand registers,
//    all of the item's base output - and then multiplies sub-tile after sub-tile, the next one's operand image in
//    flight, and writes it back.  All loads are unconditional (rows beyond a
//    tile re-read a valid row and are not stored), so the code is straight-line.
//
// What bounds it is the read-modify-write of y in HBM, and that runs the faster the more of it a wave reads before it
// writes, and the less far down a strip of 256-byte pieces it goes.  Layer call in us, two projections of 4096
// inputs unless stated, by tiles per item and sub-tiles of y in flight, 4 and 1 / 2 and 1 / 2 and 2 / 2 and all 4 (now): 16384
// rows of 8 uneven requests, rank 64 286.5 / 282.8 / 278.4 / 270.9, 4096 rows of 8 requests 93.4 / 90.9 / 90.3 / 89.4,
// 16384 rows, rank 16 266.4 / 251.2 / 242.9 / 241.7, 12000 rows of 7 requests, rank 32 206.7 / 193.0 / 191.0 / 190.2;
// eight equal requests at rank 64, kernel
// alone in steady state, 212 to 214 us = 5.7 TB/s of y and B.  More tiles (3, all in flight: 312, registers spill) or fewer (1: 309, B is fetched
// for every 32 rows) are slower at rank 64; 8 tiles with one in flight 294.  Where four tiles were ahead of two: one narrow
// projection of segments that are whole multiples of 128 rows, of which they fetched B half as often and crossed into the
// next never (lora_expand, 64 segments of 256 rows, rank 64, 1024 columns 25.7 / 28.1, 4096 columns 64.7 / 62.2; of 128 rows, 1024 columns
// 25.8 / 28.6, at rank 32 20.3 / 21.3; but 64 uneven ones of 256 on average, whole call 1024 columns 8 % less, q, k and v together 5 % less).
//
// The base-output rows are read and written with nontemporal accesses: every byte of y is touched
// once, and keeping it out of the caches leaves them to the B tiles and operand images that many
// waves share (prefill workload: 250 -> 229 us; in the decode kernel, where a tile's rows are few
// and B is the larger stream, the same change costs 5 %).
//
// Row placement as in the decode kernel: tile row r of a sub-tile sits in MFMA row slot
// (r % 4) * 4 + r / 4, so result register i of lane group g is row 4*i + g and each y
// access of a wave covers four rows x 256 contiguous bytes.
#include <type_traits>

#include "expand_common.h"
#include "lora_internal.h"

namespace lora {

namespace {


// vec elements of one sub-tile's operand image
template <int R>
__host__ __device__ constexpr int image_vecs()
{
    return ExpandTile<R>::KS * 2 * 64;
}

template <int R>
__global__ __launch_bounds__(256) void operand_image_kernel(ExpandParams p,
                                                            const lora_tile *__restrict__ tiles,
                                                            const Unit *__restrict__ units,
                                                            const int32_t *__restrict__ counts)
{
    using Tile = ExpandTile<R>;
    typedef typename Tile::vec vec;
    constexpr int KS = Tile::KS, KV = Tile::KV;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int g = lane >> 4, i16 = lane & 15;
    const int gw = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + wave), nw = gridDim.x * 4;
    const int n_slots = counts[2] * 2;                 // 16-row sub-tiles, two per tile
    const int64_t part_stride = (int64_t)p.P * R;
    const int n_parts = long_split(counts[2], p.kblocks, p.n_parts).n_parts;        // as the shrink has it

    for (int s = gw; s < n_slots * p.n_fused; s += nw) {
        const int pj = s / n_slots;
        const int slot = s - pj * n_slots;
        const lora_tile t = tiles[slot >> 1];
        const float scale = units[(int64_t)t.key * p.n_proj + p.proj0 + pj].scale;
        const int row = (slot & 1) * 16 + (i16 & 3) * 4 + (i16 >> 2);
        const bool valid = row < t.n_rows;
        const float *vrow = p.proj[pj].v + (int64_t)(t.row0 + (valid ? row : 0)) * R;
        LORA_GLOBAL vec *img = (LORA_GLOBAL vec *)p.proj[pj].img + (int64_t)slot * image_vecs<R>();
        typename Tile::A a;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int jb = Tile::jbase(g, ks);
            float sum[KV];
#pragma unroll
            for (int q = 0; q < KV; ++q) sum[q] = 0.f;
            for (int part = 0; part < n_parts; ++part) {
#pragma unroll
                for (int h = 0; h < KV / 4; ++h) {
                    const f32x4 x = ld16f(vrow + part * part_stride + jb + 4 * h);
#pragma unroll
                    for (int q = 0; q < 4; ++q) sum[4 * h + q] += x[q];
                }
            }
#pragma unroll
            for (int q = 0; q < KV; ++q) sum[q] = valid ? sum[q] * scale : 0.f;
            Tile::make_a(sum, g, ks, a);
            img[(ks * 2 + 0) * 64 + lane] = a.hi[ks];
            img[(ks * 2 + 1) * 64 + lane] = a.lo[ks];
        }
    }
}

template <int R, bool F32>
struct LongWave {
    using Tile = ExpandTile<R>;
    typedef typename Tile::vec vec;
    static constexpr int KS = Tile::KS;
    static constexpr int NY = F32 ? 2 : 1;
    static constexpr int ESZ = F32 ? 4 : 2;
    static constexpr int GROUP = expand_long_group(F32);
    static constexpr int NSLOT = 2 * GROUP;

    struct Rows {                 // where a sub-tile's rows live, and its base output
        char *at[4];
        bool ok[4];
        u32x4 y[4][NY];
    };

    int lane, g, i16;
    const int32_t *perm;
    char *ybase;                  // y + this lane's first column
    int64_t ld_bytes;
    bool col_ok;
    const LORA_GLOBAL vec *img;
    lora_tile tl[GROUP];
    int tix[GROUP];
    bool live[GROUP];

    __device__ inline void rows_of(int q, Rows &r) const
    {
        const int k = q >> 1, sub = q & 1;
        const int n = live[k] ? tl[k].n_rows : 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = sub * 16 + 4 * i + g;
            r.ok[i] = col_ok && row < n;
            const int dst = perm[tl[k].row0 + min(row, tl[k].n_rows - 1)];
            r.at[i] = ybase + (int64_t)dst * ld_bytes;
        }
    }

    __device__ inline void load_y(Rows &r) const
    {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int h = 0; h < NY; ++h) r.y[i][h] = ld16<true>(r.at[i] + 16 * h);     // touched once: nontemporal
    }

    __device__ inline void load_image(int q, typename Tile::A &a) const
    {
        const LORA_GLOBAL vec *im = img + (int64_t)(tix[q >> 1] * 2 + (q & 1)) * image_vecs<R>();
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            a.hi[ks] = im[(ks * 2 + 0) * 64 + lane];
            a.lo[ks] = im[(ks * 2 + 1) * 64 + lane];
        }
    }

    // the base output becomes the output
    __device__ inline void compute(Rows &r, const typename Tile::A &a, const typename Tile::B &b) const
    {
        f32x4 acc[8];
        Tile::mma(a, b, acc);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (F32) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    r.y[i][0][q] = __float_as_uint(__uint_as_float(r.y[i][0][q]) + acc[q][i]);
                    r.y[i][NY - 1][q] = __float_as_uint(__uint_as_float(r.y[i][NY - 1][q]) + acc[4 + q][i]);
                }
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const unsigned u = r.y[i][0][q];
                    const float f0 = __uint_as_float(u << 16) + acc[2 * q][i];
                    const float f1 = __uint_as_float(u & 0xFFFF0000u) + acc[2 * q + 1][i];
                    r.y[i][0][q] = pack_bf16_rne(f0, f1);
                }
            }
        }
    }

    __device__ inline void store(const Rows &r) const
    {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (r.ok[i]) {
#pragma unroll
                for (int h = 0; h < NY; ++h) st16<true>(r.at[i] + 16 * h, r.y[i][h]);
            }
    }
};

template <int R, bool F32>
__global__ __launch_bounds__(256, 2) void expand_long_kernel(ExpandParams p,
                                                             const lora_tile *__restrict__ tiles,
                                                             const Unit *__restrict__ units,
                                                             const int32_t *__restrict__ counts)
{
    using Wave = LongWave<R, F32>;
    using Tile = ExpandTile<R>;
    constexpr int NSLOT = Wave::NSLOT, GROUP = Wave::GROUP;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int gw = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + wave), nw = gridDim.x * 4;
    const int n_tiles = counts[2];
    const int n_groups = (n_tiles + GROUP - 1) / GROUP;
    const int shift = p.item_shift;                                 // tile groups in runs of 2^shift
    const int per_run = p.per_tile << shift;                        // per_tile: chunks of all projections
    const int n_items = ((n_groups + (1 << shift) - 1) >> shift) * per_run;

    for (int item = gw; item < n_items; item += nw) {
        const int run = item / per_run, at = item - run * per_run;
        const int tg = (run << shift) + (at & ((1 << shift) - 1)), rem = at >> shift;
        if (tg >= n_groups) continue;
        const int pj = (rem >= p.slice1 ? 1 : 0) + (rem >= p.slice2 ? 1 : 0);
        const int chunk = rem - p.proj[pj].slice0;

        Wave w;
        w.lane = lane;
        w.g = lane >> 4;
        w.i16 = lane & 15;
        w.perm = p.perm;
        const int col = chunk * kColChunk + w.i16 * 8;
        w.col_ok = col < p.proj[pj].h_out;
        w.ybase = static_cast<char *>(p.proj[pj].y) + (int64_t)(w.col_ok ? col : 0) * Wave::ESZ;
        w.ld_bytes = p.proj[pj].ldy * Wave::ESZ;
        w.img = (const LORA_GLOBAL typename Wave::vec *)p.proj[pj].img;
#pragma unroll
        for (int k = 0; k < GROUP; ++k) {
            w.live[k] = tg * GROUP + k < n_tiles;
            w.tix[k] = min(tg * GROUP + k, n_tiles - 1);
            w.tl[k] = tiles[w.tix[k]];
        }

        typename Wave::Rows rows[NSLOT];
        typename Tile::A a[2];
        typename Tile::B b;
#pragma unroll
        for (int q = 0; q < NSLOT; ++q) w.rows_of(q, rows[q]);
        const typename Tile::Lanes lanes = Tile::lanes_of(lane, R);
        int b_key = w.tl[0].key;
        Tile::template load_b<false, false>(units[(int64_t)b_key * p.n_proj + p.proj0 + pj].B, chunk, lanes, b);
        w.load_image(0, a[0]);
#pragma unroll
        for (int q = 0; q < NSLOT; ++q) w.load_y(rows[q]);
#pragma unroll
        for (int q = 0; q < NSLOT; ++q) {
            if (q + 1 < NSLOT) w.load_image(q + 1, a[(q + 1) & 1]);
            const int key = w.tl[q >> 1].key;
            if (key != b_key) {                                   // wave-uniform, rare
                b_key = key;
                Tile::template load_b<false, false>(units[(int64_t)key * p.n_proj + p.proj0 + pj].B, chunk, lanes, b);
            }
            w.compute(rows[q], a[q & 1], b);
            if constexpr (R > 16) w.store(rows[q]);
            else __builtin_amdgcn_sched_barrier(0);               // one sub-tile's products at a time
        }
        // rank 16, whose B leaves the registers for it: 241.7 -> 238.7 us for the call named above
        if constexpr (R == 16) {
#pragma unroll
            for (int q = 0; q < NSLOT; ++q) w.store(rows[q]);
        }
    }
}

template <int R>
hipError_t launch_r(const ExpandParams &p, hipStream_t s)
{
    hipLaunchKernelGGL((operand_image_kernel<R>), dim3(p.image_grid), dim3(256), 0, s, p, p.tiles,
                       p.units, p.counts);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (p.out_f32)
        hipLaunchKernelGGL((expand_long_kernel<R, true>), dim3(p.grid), dim3(256), 0, s, p, p.tiles,
                           p.units, p.counts);
    else
        hipLaunchKernelGGL((expand_long_kernel<R, false>), dim3(p.grid), dim3(256), 0, s, p, p.tiles,
                           p.units, p.counts);
    return hipGetLastError();
}

}  // namespace

size_t expand_image_bytes(int rank, int64_t n_tiles)
{
    const int ks = rank >= 32 ? rank / 32 : 1;
    const size_t vec_bytes = rank <= 16 ? 8 : 16;
    return (size_t)n_tiles * 2 * ks * 2 * 64 * vec_bytes;
}

hipError_t launch_expand(const ExpandParams &p, hipStream_t s)
{
    if (p.grid <= 0) return hipSuccess;
    switch (p.rank) {
    case 16: return launch_r<16>(p, s);       // rank 8 always runs with 16-row tiles
    case 32: return launch_r<32>(p, s);
    case 64: return launch_r<64>(p, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace lora

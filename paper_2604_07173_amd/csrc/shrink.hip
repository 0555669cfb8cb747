// Shrink for batches with long segments (tiles of up to 32 rows): v = gather(x) * A
// (App. A.2.2 "shrink phase"; Sec. 2.2 x A).
//
// With long segments the traffic is the read of x; A is small, but a wave that multiplies it
// with only 32 rows re-reads it from the L2 four times as fast as x arrives from HBM.  So the
// four waves of a workgroup take up to 128 consecutive rows of one segment and share A through
// LDS: work item = (128 rows, K part).  Every wave owns its rows for the whole K part, so there is no
// cross-wave reduction; lora_expand adds the K parts in a fixed order, so results are bit-identical run to run.
//
// Two kernels (the host picks, do_shrink in api.hip):
//  * shrink_block_kernel: blocks of 128 rows of one segment, found in a list that every wave holds in
//    registers (BlockList).  For long segments, and for two projections.
//  * shrink_long_kernel: groups of four consecutive tiles, whatever their segments.  A group with a segment
//    boundary inside has no A to share: every wave fetches the A of its own tile.  For one projection of short
//    segments, which leave most of a block empty, and for key spaces larger than the list takes (with up to as many
//    segments as the list takes it runs blocks as well).
//
// shrink_block_kernel is bound by how many loads a CU has in flight.  x and A go straight from memory to LDS
// (global_load_lds, 16 bytes per lane), so nothing in flight costs registers: two stages of x and one or two of A are
// on their way while a third is multiplied, 80 KB of LDS and 183 registers at most, two workgroups per CU.  (Through
// registers, as shrink_long_kernel does it, one stage ahead takes 245 registers.)  A stage is two K blocks: 128 bytes
// of every row, one cache line.  Work items are dealt so that one XCD has the neighbouring blocks of one K part:
// their A comes into its L2 once.  Shrink alone, us, shrink_long_kernel / without that order / now: 16384 rows in 8
// uneven requests, 4096 inputs, rank 64, two projections 44.4 / 42.2 / 40.3 (as much x alone, without A, takes 32), 8 requests of
// exactly 2048 rows 42.7 / 34.4 / 34.1, 8192 rows in 8 requests 31.4 / 29.1 / 25.6, 4096 rows in 8 requests
// 25.1 / 18.7 / 18.2, 8192 rows in 64 segments at rank 32 31.6 / 30.2 / 28.0.  Three stages of A at rank 64 with two
// projections leave room for one workgroup per CU only: 45.4 for the first.  Over 10 layouts of 4096 to 32768 rows and 2048 to
// 28672 inputs the kernel takes 0.92 of shrink_long_kernel's time (geometric mean); where it is behind, it is by 2 to 5 %: 14336
// inputs and more, 16384 rows and more of few requests (rank 64, one projection, one request 79.7 / 83.4; with two stages of A
// 80.3, which costs 3 to 6 % at 8192 inputs).
//
// shrink_long_kernel: per stage of four K blocks the
// workgroup copies the packed A blocks of the segment's (adapter, expert) into one of two LDS
// buffers while the previous stage is being multiplied; every wave gathers the x rows of its
// own 32 rows (the next stage's rows are in flight during the current stage's MFMAs) and reads
// its MFMA operands from LDS with 16-byte reads that are contiguous per wave.  The x rows are
// fetched as whole cache lines, four rows x 256 bytes per instruction, and turned into the MFMA
// operand layout (16 rows x 64 bytes per operand) through 4 KiB of LDS per wave: fetching them
// in the operand layout directly costs the address path twice the line look-ups, which a
// load-only probe of the two streams puts at 32 against 27 us for the prefill workload.
//
// Whole call in us, groups whose waves fetch A without a step in flight / blocks in shrink_long_kernel, found by walking
// over the segment list for every item / by the list / now: 16384 rows in 8 uneven requests, rank 64, 308 / 291 / 290 / 286; 64
// adapters, 4096 rows, rank 64, 158 / 145 / 142; 4096 adapters with 32 rows each, 1024 inputs, rank 64 465 / 514 / 445,
// rank 32 347 / 411 / 334; 2048 adapters with 64 rows each, two projections, rank 64, 667 / 594 / 586.
//
// The rank index sits on the M side of v_mfma_f32_16x16x32_bf16 and the rows on the N side, so
// a lane ends up with four consecutive rank entries of one row.  With two fused projections
// (gate and up, or two projections of a group that read the same input) x is loaded once.
// Ranks 16, 32 and 64; rank-8 pools always use the 16-row-tile kernels.
#include "lora_device.h"
#include "segments_common.h"

namespace lora {

namespace {

constexpr int kLongTiles = 4;        // tiles (waves) per work item
static_assert(kLongRows == kLongTiles * kTileRows, "a wave takes a tile's rows");
constexpr int kStageKB = 4;          // K blocks per LDS stage

// The blocks of kLongRows rows of up to kLongListedSegs segments, in two levels: lane l of every wave keeps how
// many blocks segments q l .. q l + q - 1 have (q <= 64) and the number of the first one; which of the q
// segments a block belongs to is read again for each look-up, all of them at a time.  No LDS, no barrier.
struct BlockList {
    const int32_t *seg_start;
    int S, q;
    int first, n, total;               // the lane's first block and blocks, blocks of the batch

    __device__ inline void make(const int32_t *__restrict__ seg_start_, int S_)
    {
        const int lane = threadIdx.x & 63;
        seg_start = seg_start_;
        S = S_;
        q = (S + 63) / 64;
        n = 0;
        int at = seg_start[min(lane * q, S)];
        for (int k = 1; k <= q; ++k) {
            const int end = seg_start[min(lane * q + k, S)];
            n += (end - at + kLongRows - 1) / kLongRows;
            at = end;
        }
        const int incl = (int)wave_incl_sum((unsigned)n);
        first = incl - n;
        total = __builtin_amdgcn_readlane(incl, 63);
    }

    // segment, first row and end row of a block below `total`; the same for all lanes
    __device__ inline void find(int block, int &seg, int &row0, int &row_end) const
    {
        const int lane = threadIdx.x & 63;
        const int owner = __builtin_ctzll(__ballot(block >= first && block < first + n));
        const int left = block - __builtin_amdgcn_readlane(first, owner);
        const int s = min(owner * q + min(lane, q), S);              // lane q and up: no rows
        const int start = seg_start[s], end = seg_start[min(owner * q + min(lane + 1, q), S)];
        const int blocks = (end - start + kLongRows - 1) / kLongRows;
        const int before = (int)wave_incl_sum((unsigned)blocks) - blocks;
        const int which = __builtin_ctzll(__ballot(left >= before && left < before + blocks));
        seg = owner * q + which;
        row0 = __builtin_amdgcn_readlane(start, which) + (left - __builtin_amdgcn_readlane(before, which)) * kLongRows;
        row_end = __builtin_amdgcn_readlane(end, which);
    }
};

template <int R, int NPROJ>
__global__ __launch_bounds__(256, 2) void shrink_long_kernel(ShrinkParams p,
                                                             const lora_tile *__restrict__ tiles,
                                                             const int32_t *__restrict__ seg_start,
                                                             const int32_t *__restrict__ seg_key,
                                                             const Unit *__restrict__ units,
                                                             const int32_t *__restrict__ counts)
{
    constexpr int NB = R / 16;                         // 16-wide blocks of the rank index
    constexpr int BLK = NPROJ * NB;                    // 1 KiB operand blocks per K block
    constexpr int STAGE = kStageKB * BLK * 64;         // 16-byte vectors per stage
    constexpr int LOADS = STAGE / 256;                 // per thread and stage
    constexpr int SUB = kTileRows / 16;
    static_assert(STAGE % 256 == 0, "a stage is copied by whole workgroup passes");
    static_assert(kStageKB == 4, "a stage of x is 256 bytes per row: the transposition below is written for that");
    // dynamic LDS: two stages of A, then per wave 4 KiB in which a sub-tile's stage of x is
    // turned from the layout it is fetched in (whole lines per row) into the MFMA operand layout
    extern __shared__ __attribute__((aligned(16))) unsigned char dyn_lds[];
    u32x4 (*lds)[STAGE] = reinterpret_cast<u32x4 (*)[STAGE]>(dyn_lds);
    u32x4 *xt = reinterpret_cast<u32x4 *>(dyn_lds + 2 * STAGE * sizeof(u32x4)) + (threadIdx.x >> 6) * 256;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = lane >> 4, i16 = lane & 15;
    const int kblocks = (p.h_in + kKBlock - 1) / kKBlock;
    const int n_tiles = counts[2];
    const int S = counts[0];
    const bool listed = !p.by_tiles && S <= kLongListedSegs;   // blocks of one segment, else groups of four tiles
    const LongSplit split = long_split(n_tiles, kblocks, p.n_parts);
    BlockList list;
    if (listed) list.make(seg_start, S);
    const int n_items = split.n_parts * (listed ? list.total : (n_tiles + kLongTiles - 1) / kLongTiles);
    const u32x4 zero4 = {0u, 0u, 0u, 0u};

    for (int item = blockIdx.x; item < n_items; item += gridDim.x) {
        const int grp = item / split.n_parts;
        const int part = item - grp * split.n_parts;
        // this wave's rows (a wave without any re-reads valid ones and stores nothing), and whether the
        // workgroup's belong to one (adapter, expert); all but the rows is the same for all of it
        lora_tile t;
        bool live, same_key = true;
        const int w4 = __builtin_amdgcn_readfirstlane(wave);
        if (listed) {
            int block_row0, seg_end;
            list.find(grp, t.seg, block_row0, seg_end);
            t.key = seg_key[t.seg];
            t.row0 = block_row0 + w4 * kTileRows;
            live = t.row0 < seg_end;
            if (!live) t.row0 = block_row0;
            t.n_rows = live ? min(kTileRows, seg_end - t.row0) : 1;
        } else {
            const int tix = grp * kLongTiles + w4;
            live = tix < n_tiles;
            t = tiles[min(tix, n_tiles - 1)];
            const int key0 = tiles[grp * kLongTiles].key;
#pragma unroll
            for (int k = 1; k < kLongTiles; ++k)
                same_key = same_key && tiles[min(grp * kLongTiles + k, n_tiles - 1)].key == key0;
        }

        const uint16_t *Ag[NPROJ];                            // this wave's A; where it is shared, the group's
#pragma unroll
        for (int pj = 0; pj < NPROJ; ++pj) Ag[pj] = units[(int64_t)t.key * p.n_proj + p.proj0 + pj].A;

        // gathered input rows as they are fetched: one instruction reads four rows (lane group g) x
        // 256 contiguous bytes (16 lanes x 16 bytes), i.e. whole cache lines, which the address path
        // serves faster than 16 rows x 64 bytes; rows beyond the wave's re-read a valid one and are
        // replaced by zeros
        const uint16_t *xq[SUB][4];
        bool qv[SUB][4];
#pragma unroll
        for (int sub = 0; sub < SUB; ++sub)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int r = sub * 16 + j * 4 + g;
                qv[sub][j] = live && r < t.n_rows;
                int s = p.perm[t.row0 + min(r, t.n_rows - 1)];
                if (p.src_row) s = p.src_row[s];
                xq[sub][j] = p.x + (int64_t)s * p.ldx;            // start of the row
            }

        const int kb_begin = part * split.kb_per_part;
        const int kb_end = min(kb_begin + split.kb_per_part, kblocks);
        const int n_stages = (kb_end - kb_begin + kStageKB - 1) / kStageKB;

        f32x4 acc[NPROJ][SUB][NB];
#pragma unroll
        for (int pj = 0; pj < NPROJ; ++pj)
#pragma unroll
            for (int sub = 0; sub < SUB; ++sub)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) acc[pj][sub][nb] = f32x4{0.f, 0.f, 0.f, 0.f};

        // All loads are unconditional: a K block beyond the part re-reads the part's last
        // block and is replaced by zeros (x as well: the padding may hold anything).
        auto load_a = [&](int kb0, u32x4 (&a)[LOADS]) {
#pragma unroll
            for (int i = 0; i < LOADS; ++i) {
                const int b = 4 * i + wave;                   // operand block of the stage
                const int kbi = b / BLK, rem = b - kbi * BLK;
                const int pj = rem / NB, nb = rem - pj * NB;
                const bool k_ok = kb0 + kbi < kb_end;
                const int kb = k_ok ? kb0 + kbi : kb_end - 1;
                const uint16_t *Ap = NPROJ == 2 && pj == 1 ? Ag[NPROJ - 1] : Ag[0];
                const u32x4 v = ld16<false>(Ap + (((int64_t)kb * NB + nb) * 64 + lane) * 8);
                a[i] = k_ok ? v : zero4;
            }
        };
        auto store_a = [&](const u32x4 (&a)[LOADS], u32x4 *buf) {
#pragma unroll
            for (int i = 0; i < LOADS; ++i) buf[(4 * i + wave) * 64 + lane] = a[i];
        };
        // a stage of x as whole lines: lane (g, i16) of instruction j holds K values
        // kb0 * 32 + 8 * i16 .. + 7 of row 4 j + g of the sub-tile
        auto load_rows = [&](int kb0, u32x4 (&xr)[SUB][4]) {
            const int kb = kb0 + (i16 >> 2);                  // the K block this lane's 16 bytes belong to
            const bool k_ok = kb < kb_end;
            const bool c_ok = k_ok && kb0 * kKBlock + i16 * 8 < p.h_in;
            const int c = c_ok ? kb0 * kKBlock + i16 * 8 : 0;    // beyond the part: the row's first bytes, not used
#pragma unroll
            for (int sub = 0; sub < SUB; ++sub)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const u32x4 v = ld16<true>(xq[sub][j] + c);  // read once: nontemporal
                    xr[sub][j] = (c_ok && qv[sub][j]) ? v : zero4;
                }
        };
        // rows -> MFMA operands through this wave's 4 KiB of LDS.  The 16-byte column of a row
        // is stored at column (col ^ row): the writes of an instruction (one row per 16 lanes)
        // and the reads (16 rows, one column each per 16 lanes) both touch every bank once.
        // LDS operations of one wave execute in order, so no barrier is needed.
        auto to_operands = [&](const u32x4 (&xr)[SUB][4], u32x4 (&xv)[SUB][kStageKB]) {
#pragma unroll
            for (int sub = 0; sub < SUB; ++sub) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int row = j * 4 + g;
                    xt[row * 16 + (i16 ^ row)] = xr[sub][j];
                }
#pragma unroll
                for (int kbi = 0; kbi < kStageKB; ++kbi) xv[sub][kbi] = xt[i16 * 16 + ((kbi * 4 + g) ^ i16)];
            }
        };
        // one stage out of LDS: straight-line code, no global loads inside
        auto compute = [&](const u32x4 *buf, const u32x4 (&xv)[SUB][kStageKB]) {
#pragma unroll
            for (int kbi = 0; kbi < kStageKB; ++kbi)
#pragma unroll
                for (int pj = 0; pj < NPROJ; ++pj)
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        const u32x4 w = buf[((kbi * NPROJ + pj) * NB + nb) * 64 + lane];
#pragma unroll
                        for (int sub = 0; sub < SUB; ++sub)
                            acc[pj][sub][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                as_bf16x8(w), as_bf16x8(xv[sub][kbi]), acc[pj][sub][nb], 0, 0, 0);
                    }
        };

        u32x4 xr[SUB][4];                  // the next stage's x as fetched
        u32x4 xc[SUB][kStageKB];           // the current stage's x as MFMA operands
        if (same_key) {
            u32x4 areg[LOADS];
            load_a(kb_begin, areg);
            load_rows(kb_begin, xr);
            store_a(areg, lds[0]);
            to_operands(xr, xc);
            __syncthreads();
            if (live) {
#pragma unroll 1
                for (int s = 0; s < n_stages; ++s) {
                    const int kb0 = kb_begin + s * kStageKB;
                    const bool more = s + 1 < n_stages;
                    if (more) {
                        load_a(kb0 + kStageKB, areg);
                        load_rows(kb0 + kStageKB, xr);
                    }
                    __builtin_amdgcn_sched_barrier(0);        // all of the next stage's loads first
                    compute(lds[s & 1], xc);
                    if (more) {
                        store_a(areg, lds[(s + 1) & 1]);
                        to_operands(xr, xc);
                    }
                    __syncthreads();
                }
            } else {                                          // no rows: only this wave's share of A
                for (int s = 0; s < n_stages; ++s) {
                    if (s + 1 < n_stages) {
                        load_a(kb_begin + (s + 1) * kStageKB, areg);
                        store_a(areg, lds[(s + 1) & 1]);
                    }
                    __syncthreads();
                }
            }
        } else if (live) {
            // tiles of several segments: every wave reads the A of its own tile, a step of kOwn operand
            // blocks ahead, without LDS and without barriers
            constexpr int kOwn = NPROJ == 2 ? 4 : kStageKB * BLK < 8 ? kStageKB * BLK : 8;    // two projections: no registers for eight
            auto load_own = [&](int kb0, int b0, u32x4 (&a)[kOwn]) {
#pragma unroll
                for (int i = 0; i < kOwn; ++i) {
                    const int b = b0 + i, pj = b % BLK / NB, nb = b % NB;
                    const bool k_ok = kb0 + b / BLK < kb_end;
                    const int kb = k_ok ? kb0 + b / BLK : kb_end - 1;
                    const u32x4 v = ld16<false>(Ag[pj] + (((int64_t)kb * NB + nb) * 64 + lane) * 8);
                    a[i] = k_ok ? v : zero4;
                }
            };
            u32x4 a[kOwn], an[kOwn];
            load_rows(kb_begin, xr);
            load_own(kb_begin, 0, a);
            to_operands(xr, xc);
#pragma unroll 1
            for (int s = 0; s < n_stages; ++s) {
                const int kb0 = kb_begin + s * kStageKB;
                const bool more = s + 1 < n_stages;
#pragma unroll
                for (int b0 = 0; b0 < kStageKB * BLK; b0 += kOwn) {
                    load_own(kb0, b0 + kOwn, an);             // beyond the part: zeros, never multiplied
                    if (more && b0 == 0) load_rows(kb0 + kStageKB, xr);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int i = 0; i < kOwn; ++i)
#pragma unroll
                        for (int sub = 0; sub < SUB; ++sub) {
                            f32x4 &c = acc[(b0 + i) % BLK / NB][sub][(b0 + i) % NB];
                            c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a[i]), as_bf16x8(xc[sub][(b0 + i) / BLK]),
                                                                        c, 0, 0, 0);
                        }
#pragma unroll
                    for (int i = 0; i < kOwn; ++i) a[i] = an[i];
                }
                if (more) to_operands(xr, xc);
            }
        }

        // this wave's rows of this part of v: lane (row i16, group g) holds rank entries
        // nb*16 + 4g .. +3 of its row
#pragma unroll
        for (int pj = 0; pj < NPROJ; ++pj)
#pragma unroll
            for (int sub = 0; sub < SUB; ++sub)
                if (live && sub * 16 + i16 < t.n_rows) {
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
                        st16f(p.v[pj] + ((int64_t)part * p.P + t.row0 + sub * 16 + i16) * R + nb * 16 + g * 4,
                              acc[pj][sub][nb]);
                }
    }
}

// ---- blocks of one segment ---------------------------------------------------------------------------

// 16 bytes per lane from memory straight into LDS, lane l's at lds_at + 16 l (lds_at: a byte address, the same for every
// lane).  Counts as a vector-memory load that the compiler does not know of; it is in LDS once wait_loads says so.  m0, which
// holds the address, is named as clobbered, so that no value of the compiler's own lives in it across the statement; that
// nothing saves a reserved register, of which the compiler warns, is what is wanted here.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <bool NT>
__device__ inline void load_to_lds(const void *src, unsigned lds_at)
{
    const unsigned at = __builtin_amdgcn_readfirstlane(lds_at);
    if (NT) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off nt" ::"s"(at), "v"(src) : "memory", "m0");
    else asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(at), "v"(src) : "memory", "m0");
}
#pragma clang diagnostic pop

// until at most N of this wave's vector-memory operations are outstanding
template <int N>
__device__ inline void wait_loads()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

constexpr int kXcds = 8;              // consecutive workgroups go to the eight XCDs in turn
constexpr int kBlockKB = 2;          // K blocks per stage: a stage of x is one cache line per row
constexpr int kXStages = 3;          // stages of x in LDS
constexpr int kXStageBytes = kLongRows * kBlockKB * kKBlock * 2;
constexpr int kXWaveBytes = kXStageBytes / kLongTiles;

template <int R, int NPROJ>
__host__ __device__ constexpr int block_a_bytes()
{
    return kBlockKB * NPROJ * (R / 16) * 1024;
}

// stages of A in LDS: as many as two workgroups per CU have room for, up to three
template <int R, int NPROJ>
__host__ __device__ constexpr int block_a_stages()
{
    return kXStages * kXStageBytes + 3 * block_a_bytes<R, NPROJ>() <= 80 * 1024 ? 3 : 2;
}

template <int R, int NPROJ>
__host__ __device__ constexpr int block_lds_bytes()
{
    return kXStages * kXStageBytes + block_a_stages<R, NPROJ>() * block_a_bytes<R, NPROJ>();
}

template <int R, int NPROJ>
__global__ __launch_bounds__(256, 2) void shrink_block_kernel(ShrinkParams p,
                                                              const int32_t *__restrict__ seg_start,
                                                              const int32_t *__restrict__ seg_key,
                                                              const Unit *__restrict__ units,
                                                              const int32_t *__restrict__ counts)
{
    constexpr int NB = R / 16;                         // 16-wide blocks of the rank index
    constexpr int BLK = NPROJ * NB;                    // 1 KiB operand blocks per K block
    constexpr int A_BLOCKS = kBlockKB * BLK;           // per stage
    constexpr int SUB = kTileRows / 16;
    constexpr int A_STAGES = block_a_stages<R, NPROJ>();
    constexpr int LEAD = A_STAGES - 2;                 // stages of A in flight beyond the next one
    constexpr int NA = A_BLOCKS / 4;                   // loads of A per wave and stage (some waves of rank 16 have one more)
    constexpr int NX = kXWaveBytes / 1024;             // loads of x per wave and stage: 8 rows x 128 bytes each
    constexpr int A0 = kXStages * kXStageBytes;
    static_assert(NX * 8 == kTileRows, "a load is eight rows of one line");
    extern __shared__ __attribute__((aligned(16))) unsigned char dyn_lds[];
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)dyn_lds;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, i16 = lane & 15;
    const int kblocks = (p.h_in + kKBlock - 1) / kKBlock;
    const LongSplit split = long_split(counts[2], kblocks, p.n_parts);
    BlockList list;
    list.make(seg_start, counts[0]);
    const int n_items = split.n_parts * list.total;

    const int per_xcd = (n_items + kXcds - 1) / kXcds;

    for (int slot = blockIdx.x; slot < per_xcd * kXcds; slot += gridDim.x) {
        const int item = slot % kXcds * per_xcd + slot / kXcds;
        if (item >= n_items) continue;
        const int part = item / list.total;
        const int blk = item - part * list.total;
        // this wave's rows; a wave without any loads its share of A only
        int seg, row0, seg_end;
        list.find(blk, seg, row0, seg_end);
        const int key = seg_key[seg];
        row0 += wave * kTileRows;
        const bool live = row0 < seg_end;
        const int n_rows = min(kTileRows, seg_end - row0);

        const uint16_t *Ag[NPROJ];
#pragma unroll
        for (int pj = 0; pj < NPROJ; ++pj) Ag[pj] = units[(int64_t)key * p.n_proj + p.proj0 + pj].A;

        // load j of x: lane l fetches 16 bytes of row 8 j + l / 8, and they land at 16 l: a row's line is 128 bytes of
        // LDS.  Which 16 of the line: column c of row r is kept at place c ^ (r % 8), so that the operand reads (one
        // column of eight rows by eight lanes) touch every bank once.  Rows beyond the wave's re-read a valid one; their
        // results are columns that nobody reads.
        const int col = (lane & 7) ^ (lane >> 3);
        const char *xrow[NX];
        if (live) {
#pragma unroll
            for (int j = 0; j < NX; ++j) {
                int s = p.perm[row0 + min(8 * j + (lane >> 3), n_rows - 1)];
                if (p.src_row) s = p.src_row[s];
                xrow[j] = reinterpret_cast<const char *>(p.x + (int64_t)s * p.ldx);
            }
        }

        const int kb_begin = part * split.kb_per_part;
        const int kb_end = min(kb_begin + split.kb_per_part, kblocks);
        const int n_stages = (kb_end - kb_begin + kBlockKB - 1) / kBlockKB;
        const int last_col = min(kb_end * kKBlock, p.h_in) - 8;      // columns beyond the part or the row re-read these

        auto load_x = [&](int s) {
            const unsigned c = 2u * (unsigned)min((kb_begin + s * kBlockKB) * kKBlock + col * 8, last_col);
            const unsigned at = lds0 + (s % kXStages) * kXStageBytes + wave * kXWaveBytes;
#pragma unroll
            for (int j = 0; j < NX; ++j) load_to_lds<true>(xrow[j] + c, at + j * 1024);      // read once: nontemporal
        };
        auto load_a = [&](int s) {
#pragma unroll
            for (int i = 0; i < (A_BLOCKS + 3) / 4; ++i) {
                const int b = 4 * i + wave;                          // operand block of the stage
                if (A_BLOCKS % 4 == 0 || b < A_BLOCKS) {
                    const int kbi = b / BLK, rem = b - kbi * BLK;
                    const int pj = rem / NB, nb = rem - pj * NB;
                    const int kb = min(kb_begin + s * kBlockKB + kbi, kb_end - 1);
                    const uint16_t *Ap = NPROJ == 2 && pj == 1 ? Ag[NPROJ - 1] : Ag[0];
                    load_to_lds<false>(Ap + (((int64_t)kb * NB + nb) * 64 + lane) * 8,
                                       lds0 + A0 + (s % A_STAGES) * block_a_bytes<R, NPROJ>() + b * 1024);
                }
            }
        };

        f32x4 acc[NPROJ][SUB][NB];
#pragma unroll
        for (int pj = 0; pj < NPROJ; ++pj)
#pragma unroll
            for (int sub = 0; sub < SUB; ++sub)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) acc[pj][sub][nb] = f32x4{0.f, 0.f, 0.f, 0.f};

        auto compute = [&](int s) {
            const unsigned char *xs = dyn_lds + (s % kXStages) * kXStageBytes + wave * kXWaveBytes;
            const u32x4 *as = reinterpret_cast<const u32x4 *>(dyn_lds + A0 + (s % A_STAGES) * block_a_bytes<R, NPROJ>());
            u32x4 xv[kBlockKB][SUB], w[2][BLK];
            auto read_a = [&](int kbi) {
#pragma unroll
                for (int b = 0; b < BLK; ++b) w[kbi & 1][b] = as[(kbi * BLK + b) * 64 + lane];
            };
#pragma unroll
            for (int kbi = 0; kbi < kBlockKB; ++kbi)
#pragma unroll
                for (int sub = 0; sub < SUB; ++sub)
                    xv[kbi][sub] = *reinterpret_cast<const u32x4 *>(xs + (sub * 16 + i16) * 128 + (((kbi * 4 + g) ^ (i16 & 7)) * 16));
            read_a(0);
#pragma unroll
            for (int kbi = 0; kbi < kBlockKB; ++kbi) {
                const int kb = kb_begin + s * kBlockKB + kbi;
                if (kb >= kb_end) break;                             // uniform
                if (kbi + 1 < kBlockKB) read_a(kbi + 1);
                __builtin_amdgcn_sched_barrier(0);                   // the next block's operands before this one's products
                if ((kb + 1) * kKBlock > p.h_in && kb * kKBlock + g * 8 >= p.h_in)       // beyond the row: A is zero, x may be anything
#pragma unroll
                    for (int sub = 0; sub < SUB; ++sub) xv[kbi][sub] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
                for (int b = 0; b < BLK; ++b)
#pragma unroll
                    for (int sub = 0; sub < SUB; ++sub)
                        acc[b / NB][sub][b % NB] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            as_bf16x8(w[kbi & 1][b]), as_bf16x8(xv[kbi][sub]), acc[b / NB][sub][b % NB], 0, 0, 0);
            }
        };

        // Two stages of x and one or two of A in flight.  Loads complete in order, and they are asked for as x(s), A(s + LEAD),
        // x(s + 1), A(s + 1 + LEAD): at the top of a turn those of A(s + LEAD) on, if that is beyond s, and x(s + 1) may be
        // outstanding.  Behind the barrier every wave is done with stage s - 1, whose places the next loads take.
        if (live) load_x(0);
        load_a(0);
        if (n_stages > 1) {
            if (LEAD) load_a(1);
            if (live) load_x(1);
        }
#pragma unroll 1
        for (int s = 0; s < n_stages; ++s) {
            if (s + 1 >= n_stages) wait_loads<0>();
            else if (live) wait_loads<LEAD * NA + NX>();
            else wait_loads<LEAD * NA>();
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // this wave's reads of stage s - 1 as well
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if (s + 1 + LEAD < n_stages) load_a(s + 1 + LEAD);
            if (live) {
                if (s + 2 < n_stages) load_x(s + 2);
                compute(s);
            }
        }
        // before the next item's first loads: everyone is done with the last stages
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");

        // this wave's rows of this part of v: lane (row i16, group g) holds rank entries
        // nb*16 + 4g .. +3 of its row
#pragma unroll
        for (int pj = 0; pj < NPROJ; ++pj)
#pragma unroll
            for (int sub = 0; sub < SUB; ++sub)
                if (live && sub * 16 + i16 < n_rows) {
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
                        st16f(p.v[pj] + ((int64_t)part * p.P + row0 + sub * 16 + i16) * R + nb * 16 + g * 4,
                              acc[pj][sub][nb]);
                }
    }
}

template <int R, int NPROJ>
hipError_t launch_rn(const ShrinkParams &p, hipStream_t s)
{
    if (p.blocks) {
        constexpr int kLds = block_lds_bytes<R, NPROJ>();
        static hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(shrink_block_kernel<R, NPROJ>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
        if (attr != hipSuccess) return attr;
        hipLaunchKernelGGL((shrink_block_kernel<R, NPROJ>), dim3(p.grid), dim3(256), kLds, s, p, p.seg_start, p.seg_key,
                           p.units, p.counts);
        return hipGetLastError();
    }
    // two stages of A (kStageKB K blocks of NPROJ * R / 16 operand blocks of 1 KiB) + 4 KiB per wave
    constexpr int kLds = 2 * kStageKB * NPROJ * (R / 16) * 1024 + 4 * 4096;
    static hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(shrink_long_kernel<R, NPROJ>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL((shrink_long_kernel<R, NPROJ>), dim3(p.grid), dim3(256), kLds, s, p, p.tiles, p.seg_start,
                       p.seg_key, p.units, p.counts);
    return hipGetLastError();
}

template <int R>
hipError_t launch_r(const ShrinkParams &p, hipStream_t s)
{
    return p.n_fused == 2 ? launch_rn<R, 2>(p, s) : launch_rn<R, 1>(p, s);
}

}  // namespace

hipError_t launch_shrink(const ShrinkParams &p, hipStream_t s)
{
    if (p.grid <= 0) return hipSuccess;
    switch (p.rank) {
    case 16: return launch_r<16>(p, s);
    case 32: return launch_r<32>(p, s);
    case 64: return launch_r<64>(p, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace lora

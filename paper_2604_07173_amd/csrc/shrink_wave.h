// The wave-level work of the decode shrink (tiles of at most 16 rows), shared by the shrink
// kernel and the kernel that runs shrink and expand in one launch: one wave multiplies a run of
// K units of the packed A (of up to three projections that read the same input) with the
// gathered x rows of one tile.
//
// A wave streams its slice of the packed A with 16-byte loads that are contiguous per wave, two steps in
// flight: the loads of step s+1 are issued before the MFMAs of step s, all loads are unconditional so that the loop is
// branch-free, and nothing looks at loaded data but the MFMAs, so the hardware counters keep a whole step
// outstanding while the other is multiplied.  (With the rows and columns that do not count replaced by zeros where they
// are loaded, and the order left to the scheduler, a wave waited for everything it had asked for once
// per turn.)  Layer call, before / after: Mixtral shapes, 512 tokens, rank 64 331 -> 318 us; llama shapes, 256 rows,
// rank 64 145 -> 137, rank 32 89.3 -> 83.2, rank 8 53.0 -> 48.8; fine-grained MoE, 256 tokens 66.3 -> 61.3; rank 64 with
// one step in flight 322 and 137.
// The rank index sits on the M side of v_mfma_f32_16x16x32_bf16 and the rows on the N side, so a
// lane ends up with four consecutive rank entries of one row.
//
// Rank 8: a packed block holds 64 K values (two 32-deep halves side by side in the 16 M rows),
// is multiplied once with each half's x values, and rows 0..7 of the first product plus rows
// 8..15 of the second give the eight rank entries.
#pragma once
#include "lora_device.h"
#include "lora_internal.h"

namespace lora {

// NT: the packed A is loaded with the streaming hint (it is read once).  XNT: so are the x rows
// (for inputs too large to stay in a cache until anyone reads them again).
//
// LINES (ranks 8 to 32, where a step covers 128 or 64 K values = 256 or 128 bytes of a row): the x rows
// are fetched as whole cache lines - an instruction reads 4 rows x 256 or 8 rows x 128 contiguous bytes -
// and turned into the MFMA operand layout (16 rows on the lane index, 64 bytes of a row per operand)
// through 4 or 2 KiB of LDS owned by the wave, the 16-byte column of a row stored at another column so that
// the row-wise writes and the operand-wise reads both touch every bank once.  Fetched in the operand
// layout directly, an instruction reads 16 rows x 64 bytes: half a line per row, and the other half by
// the next instruction.
template <int R, int NPROJ, bool NT, bool XNT, bool LINES, bool LOW>
struct ShrinkWave {
    static constexpr int NB = R >= 16 ? R / 16 : 1;            // weight tiles per K unit
    static constexpr int XN = R == 8 ? 2 : 1;                  // x operands per K unit
    static constexpr int NACC = R == 8 ? 2 : NB;               // accumulators per projection
    static constexpr int KU = R == 8 ? 64 : 32;                // K values per unit
    static constexpr int KB = shrink_wave_units(R);            // units per step
    static constexpr int PPR = KB * KU / 8;                    // 16-byte pieces of a row in a step
    static constexpr int RPI = 64 / PPR;                       // LINES: rows per instruction
    static constexpr int NQ = 16 / RPI;                        // LINES: instructions per step
    static_assert(!LINES || PPR == 16 || PPR == 8, "whole-line rows: a step is 256 or 128 bytes of a row");

    int lane, g, i16, h_in;
    const uint16_t *Ap[NPROJ];
    const uint16_t *xp;      // this lane's x row (a valid row even if the lane's row is not)
    const uint16_t *xq[LINES ? NQ : 1];  // LINES: rows RPI * q + lane / PPR of the tile (valid rows likewise)
    u32x4 *xt;               // LINES: the wave's LDS, NQ KiB
    unsigned a_off;          // this lane's place in a block, or kOffNone: its rank entry is beyond the adapter's rank
    int a_rank;
    f32x4 acc[NPROJ][NACC];

    // LOW: rank entries from `rank` on are zeros in memory and are not fetched: lanes at ranks 8 and 16, blocks above.
    __device__ inline void set_rank(int rank)
    {
        a_rank = rank;
        a_off = R >= 32 || (R == 8 ? i16 & 7 : i16) < rank ? lane * 16u : kOffNone;
    }

    struct Step {
        u32x4 w[NPROJ][KB][NB];
        u32x4 x[KB][XN];
    };

    // All loads are unconditional: a K unit beyond the wave's range re-reads the last valid unit, columns
    // beyond the row re-read its last ones, and a row beyond the tile the tile's last row.  Only a wave's last step can have
    // such units and columns; its multiplications leave them out (mma<true>).  Rows beyond the tile are
    // columns of the result that nobody reads, so they need no zeros.
    __device__ inline void load(int kb0, int kb_end, Step &s) const
    {
        load_a(kb0, kb_end, s);
        load_x(kb0, kb_end, s);
    }

    __device__ inline void load_a(int kb0, int kb_end, Step &s) const
    {
        unsigned off = LOW ? 0u : (unsigned)lane * 16u;
        if (!LOW) asm volatile("" : "+v"(off));        // a 32-bit offset on a scalar base: not widened ahead of time
#pragma unroll
        for (int pj = 0; pj < NPROJ; ++pj) {
            const char *base = reinterpret_cast<const char *>(Ap[pj]) + (int64_t)kb0 * (NB * 1024);
#pragma unroll
            for (int u = 0; u < KB; ++u) {
                const int at = min(u, kb_end - 1 - kb0) * (NB * 1024);
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    if (LOW) s.w[pj][u][nb] = ld16_packed<NT>(base, a_off, at + nb * 1024, nb * 16 < a_rank);
                    else s.w[pj][u][nb] = ld16<NT>(base + at + off + nb * 1024);
            }
        }
    }

    __device__ inline void load_x(int kb0, int kb_end, Step &s) const
    {
        if constexpr (!LINES) {
#pragma unroll
            for (int u = 0; u < KB; ++u) {
                const int kb = min(kb0 + u, kb_end - 1);
#pragma unroll
                for (int h = 0; h < XN; ++h)
                    s.x[u][h] = ld16<XNT>(xp + (unsigned)min(kb * KU + h * 32 + g * 8, h_in - 8));
            }
        } else {
            // lane of instruction q: row RPI * q + lane / PPR, K values kb0 * KU + 8 * (lane % PPR) .. + 7
            const int piece = lane % PPR, c = kb0 * KU + piece * 8;
            const bool ok = kb0 + piece / (KU / 8) < kb_end && c < h_in;
#pragma unroll
            for (int q = 0; q < NQ; ++q) (&s.x[0][0])[q] = ld16<XNT>(xq[q] + (ok ? c : 0));
        }
    }

    // LINES: the step's rows through LDS into operand order
    __device__ inline void to_operands(Step &s) const
    {
        auto at = [](int row, int piece) { return row * PPR + (piece ^ (row / (16 / PPR))); };
#pragma unroll
        for (int q = 0; q < NQ; ++q) xt[at(RPI * q + lane / PPR, lane % PPR)] = (&s.x[0][0])[q];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int u = 0; u < KB; ++u)
#pragma unroll
            for (int h = 0; h < XN; ++h) s.x[u][h] = xt[at(i16, (u * KU + h * 32) / 8 + g)];
        __builtin_amdgcn_wave_barrier();
    }

    // LAST: the step may reach beyond the range (those units are left out; a uniform branch) and beyond the
    // row's end (zeros for x: the packed A holds zeros there, and zero times whatever was read may be a NaN)
    template <bool LAST>
    __device__ inline void mma(int kb0, int kb_end, Step &s)
    {
        if constexpr (LINES) to_operands(s);
#pragma unroll
        for (int u = 0; u < KB; ++u) {
            if (LAST && kb0 + u >= kb_end) break;
            if (LAST && (kb0 + u + 1) * KU > h_in) {
                const u32x4 zero4 = {0u, 0u, 0u, 0u};
#pragma unroll
                for (int h = 0; h < XN; ++h)
                    if ((kb0 + u) * KU + h * 32 + g * 8 >= h_in) s.x[u][h] = zero4;
            }
#pragma unroll
            for (int pj = 0; pj < NPROJ; ++pj) {
                if (R == 8) {
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        acc[pj][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            as_bf16x8(s.w[pj][u][0]), as_bf16x8(s.x[u][h]), acc[pj][h], 0, 0, 0);
                } else {
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
                        acc[pj][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            as_bf16x8(s.w[pj][u][nb]), as_bf16x8(s.x[u][0]), acc[pj][nb], 0, 0, 0);
                }
            }
        }
    }

    // K units kb_begin, kb_begin + stride, ... below kb_end in steps of KB units (stride = KB:
    // the contiguous range [kb_begin, kb_end)), two steps in flight.  `rows` sets the pointers of the x rows; it is
    // called behind the first loads of A, which do not wait for the row indices.  `between` issues loads of the
    // caller's behind those of the first step, so that they are in flight while the wave works through its range.
    template <typename G, typename F>
    __device__ inline void run(int kb_begin, int kb_end, int stride, G rows, F between)
    {
#pragma unroll
        for (int pj = 0; pj < NPROJ; ++pj)
#pragma unroll
            for (int a = 0; a < NACC; ++a) acc[pj][a] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (kb_begin >= kb_end) {
            rows();
            between();
            return;
        }
        // The barriers keep the loads of a step in front of the multiplications of the step before: without
        // them the scheduler puts both steps' loads behind, and a wave waits for everything it asked for.
        auto fence = [] { __builtin_amdgcn_sched_barrier(0); };
        int kb0 = kb_begin;
        Step s0, s1;
        load_a(kb0, kb_end, s0);
        rows();
        load_x(kb0, kb_end, s0);
        between();
        for (; kb0 + 2 * stride < kb_end; kb0 += 2 * stride) {
            load(kb0 + stride, kb_end, s1);
            fence();
            mma<false>(kb0, kb_end, s0);
            fence();
            load(kb0 + 2 * stride, kb_end, s0);
            fence();
            mma<false>(kb0 + stride, kb_end, s1);
            fence();
        }
        if (kb0 + stride < kb_end) {
            load(kb0 + stride, kb_end, s1);
            fence();
            mma<false>(kb0, kb_end, s0);
            mma<true>(kb0 + stride, kb_end, s1);
        } else {
            mma<true>(kb0, kb_end, s0);
        }
    }
};

}  // namespace lora

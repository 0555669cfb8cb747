// Repacking of row-major A[h_in][r] / B[r][h_out] into the pool's tiled storage and back.
//
// Loading an adapter is a pure copy, so it is bound by HBM if both sides move 16 bytes per lane in
// contiguous runs.  Sources that are 16-byte aligned (every matrix of a window is, if the window is)
// are packed that way: a wave carries 32 rows of A (64 at rank 8) through LDS, a thread carries an
// 8 x 8 piece of B through its registers.  One Mixtral-shaped layer of an adapter (14.2 MB in, 14.2
// MB out): 13.1 -> 7.7 us (3.7 TB/s; 5.6 us at the rate of a large copy, and an empty launch
// takes 1.6).  Sources at odd addresses, and the way back, move one value at a time: one thread per
// 16-byte group of the packed side (eight values that differ only in their K offset t).
#include <algorithm>

#include "lora_device.h"
#include "lora_internal.h"
#include "lora_layout.h"

namespace lora {

// direction: 0 = row-major -> packed, 1 = packed -> row-major (padding is dropped)
template <int DIR>
__device__ inline void pack_A_body(const PackParams &p, int64_t gid, int unit)
{
    const int kunit = packA_kunit(p.rank);
    const int k_pad = (p.h + kunit - 1) / kunit * kunit;
    const int64_t groups = (int64_t)(k_pad / 8) * p.rank;       // (c / 8, j)
    if (gid >= groups) return;
    const int j = (int)(gid % p.rank);
    const int c0 = (int)(gid / p.rank) * 8;
    uint16_t *packed = (DIR == 0 ? p.dst : const_cast<uint16_t *>(p.src)) +
                       (int64_t)unit * (DIR == 0 ? p.dst_stride : p.src_stride) +
                       packA_index(c0, j, p.rank);               // t = 0..7 are contiguous
    uint16_t *plain = (DIR == 0 ? const_cast<uint16_t *>(p.src) : p.dst) +
                      (int64_t)unit * (DIR == 0 ? p.src_stride : p.dst_stride);
    for (int t = 0; t < 8; ++t) {
        const int c = c0 + t;
        const bool in = c < p.h && j < p.src_rank;
        if (DIR == 0) packed[t] = in ? plain[(int64_t)c * p.src_rank + j] : (uint16_t)0;
        else if (in) plain[(int64_t)c * p.src_rank + j] = packed[t];
    }
}

template <int DIR>
__global__ __launch_bounds__(256) void pack_A_kernel(PackParams p)
{
    pack_A_body<DIR>(p, (int64_t)blockIdx.x * blockDim.x + threadIdx.x, blockIdx.y);
}

template <int DIR>
__device__ inline void pack_B_body(const PackParams &p, int64_t gid, int unit)
{
    const int chunks = (p.h + 127) / 128;
    const int jg = p.rank / 8;                                 // groups of 8 rank indices
    const int64_t groups = (int64_t)chunks * 128 * jg;         // (d, j/8)
    if (gid >= groups) return;
    const int d = (int)(gid % ((int64_t)chunks * 128));
    const int j0 = (int)(gid / ((int64_t)chunks * 128)) * 8;
    uint16_t *packed = (DIR == 0 ? p.dst : const_cast<uint16_t *>(p.src)) +
                       (int64_t)unit * (DIR == 0 ? p.dst_stride : p.src_stride);
    uint16_t *plain = (DIR == 0 ? const_cast<uint16_t *>(p.src) : p.dst) +
                      (int64_t)unit * (DIR == 0 ? p.src_stride : p.dst_stride);
    for (int t = 0; t < 8; ++t) {
        const int j = j0 + t;
        const bool in = d < p.h && j < p.src_rank;
        uint16_t *q = packed + packB_index(j, d, p.rank);
        if (DIR == 0) *q = in ? plain[(int64_t)j * p.h + d] : (uint16_t)0;
        else if (in) plain[(int64_t)j * p.h + d] = *q;
    }
}

template <int DIR>
__global__ __launch_bounds__(256) void pack_B_kernel(PackParams p)
{
    pack_B_body<DIR>(p, (int64_t)blockIdx.x * blockDim.x + threadIdx.x, blockIdx.y);
}

// ---- aligned sources -------------------------------------------------------------------------------

constexpr int kPackPad = 32;                 // bytes between the groups of eight rows in LDS, against bank conflicts
constexpr int kPackLdsBytes = 64 / 8 * (8 * 8 * 2 + kPackPad) > 4 * (8 * 64 * 2 + kPackPad)
                                  ? 64 / 8 * (8 * 8 * 2 + kPackPad)
                                  : 4 * (8 * 64 * 2 + kPackPad);      // of one wave: 32 rows at rank 64

// one K unit of A (32 rows, 64 at rank 8) by one wave.  The rows are contiguous in memory; eight of
// them are a group of 16 * src_rank bytes, so a 16-byte piece never spans two groups.  Lane 16 g + i
// of output block nb then collects its eight values.
__device__ inline void pack_A_wave(const PackParams &p, int kb, int unit, char *lds)
{
    const int lane = threadIdx.x & 63, g = lane >> 4, n = lane & 15;
    const int kunit = packA_kunit(p.rank);
    const int rows = min(kunit, p.h - kb * kunit);
    const int bytes = rows * p.src_rank * 2, group = 16 * p.src_rank;
    const char *src = reinterpret_cast<const char *>(p.src + (int64_t)unit * p.src_stride +
                                                     (int64_t)kb * kunit * p.src_rank);
    for (int at = lane * 16; at < bytes; at += 64 * 16)
        *reinterpret_cast<u32x4 *>(lds + at + at / group * kPackPad) = ld16<true>(src + at);
    __builtin_amdgcn_wave_barrier();         // LDS operations of one wave execute in order
    uint16_t *dst = p.dst + (int64_t)unit * p.dst_stride + (int64_t)kb * kunit * p.rank;
    const int blocks = p.rank == 8 ? 1 : p.rank / 16;
    for (int nb = 0; nb < blocks; ++nb) {
        const int j = p.rank == 8 ? n & 7 : nb * 16 + n;
        const int c0 = (p.rank == 8 ? (n >> 3) * 32 : 0) + 8 * g;      // the lane's eight rows: one group
        const char *col = lds + c0 / 8 * (group + kPackPad) + j * 2;
        u32x4 v = {0u, 0u, 0u, 0u};
        if (j < p.src_rank && c0 < rows) {                             // h is a multiple of 8: a group is whole or absent
            unsigned e[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) e[t] = *reinterpret_cast<const uint16_t *>(col + t * p.src_rank * 2);
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = e[2 * q] | e[2 * q + 1] << 16;
        }
        st16<false>(dst + ((int64_t)nb * 64 + lane) * 8, v);
    }
    __builtin_amdgcn_wave_barrier();
}

// eight columns (one MFMA column slot n of a chunk) of eight rank entries by one thread
__device__ inline void pack_B_thread(const PackParams &p, int64_t gid, int unit)
{
    const int octets = p.rank / 8;
    const int n = (int)(gid & 15), oct = (int)((gid >> 4) % octets);
    const int64_t chunk = (gid >> 4) / octets;
    if (chunk >= (p.h + 127) / 128) return;
    const int d0 = (int)chunk * 128 + n * 8, j0 = oct * 8;
    const uint16_t *src = p.src + (int64_t)unit * p.src_stride;
    u32x4 r[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const bool in = d0 < p.h && j0 + t < p.src_rank;               // h is a multiple of 8
        r[t] = in ? ld16<true>(src + (int64_t)(j0 + t) * p.h + d0) : u32x4{0u, 0u, 0u, 0u};
    }
    uint16_t *dst = p.dst + (int64_t)unit * p.dst_stride;
    auto lo = [](unsigned a, unsigned b) { return (a & 0xFFFFu) | b << 16; };
    auto hi = [](unsigned a, unsigned b) { return a >> 16 | (b & 0xFFFF0000u); };
#pragma unroll
    for (int q = 0; q < 4; ++q)                                        // columns 2q, 2q + 1 = sub-blocks 2q, 2q + 1
        if (p.rank <= 16) {
#pragma unroll
            for (int h = 0; h < 2; ++h)                                // four rank entries of both columns
                st16<false>(dst + packB_index(j0 + 4 * h, d0 + 2 * q, p.rank),
                            u32x4{lo(r[4 * h][q], r[4 * h + 1][q]), lo(r[4 * h + 2][q], r[4 * h + 3][q]),
                                  hi(r[4 * h][q], r[4 * h + 1][q]), hi(r[4 * h + 2][q], r[4 * h + 3][q])});
        } else {
            st16<false>(dst + packB_index(j0, d0 + 2 * q, p.rank),
                        u32x4{lo(r[0][q], r[1][q]), lo(r[2][q], r[3][q]), lo(r[4][q], r[5][q]), lo(r[6][q], r[7][q])});
            st16<false>(dst + packB_index(j0, d0 + 2 * q + 1, p.rank),
                        u32x4{hi(r[0][q], r[1][q]), hi(r[2][q], r[3][q]), hi(r[4][q], r[5][q]), hi(r[6][q], r[7][q])});
        }
}

// every repack of one (adapter, layer): workgroups wg0[job] .. wg0[job + 1] - 1 of a unit take job `job`
// (even: an A, a wave per K unit; odd: a B)
__global__ __launch_bounds__(256) void pack_layer_kernel(PackLayerParams ps)
{
    __shared__ __attribute__((aligned(16))) char lds[4][kPackLdsBytes];
    int job = 0;
    while (job + 1 < ps.n_jobs && (int)blockIdx.x >= ps.wg0[job + 1]) ++job;
    const PackParams &p = ps.job[job];
    const int wg = blockIdx.x - ps.wg0[job];
    const int64_t gid = (int64_t)wg * 256 + threadIdx.x;
    if (gid == 0) p.rank_out[(int64_t)blockIdx.y * p.rank_stride] = p.src_rank;
    if (!ps.aligned) {
        if (job & 1) pack_B_body<0>(p, gid, blockIdx.y);
        else pack_A_body<0>(p, gid, blockIdx.y);
    } else if (job & 1) {
        pack_B_thread(p, gid, blockIdx.y);
    } else {
        const int wave = threadIdx.x >> 6, kunit = packA_kunit(p.rank);
        const int kb = wg * 4 + wave;
        if (kb < (p.h + kunit - 1) / kunit) pack_A_wave(p, kb, blockIdx.y, lds[wave]);
    }
}

// scale and rank of one adapter's table entries, all layers: entry (layer, adapter, e, j) sits
// at ((layer * n_adapters + adapter) * per_adapter + (e * n_proj + j))
__global__ __launch_bounds__(256) void set_adapter_kernel(Unit *table, int n_layers, int n_adapters,
                                                          int per_adapter, int adapter, int rank,
                                                          float scale)
{
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= (int64_t)n_layers * per_adapter) return;
    const int layer = (int)(gid / per_adapter), k = (int)(gid % per_adapter);
    Unit *u = table + ((int64_t)layer * n_adapters + adapter) * per_adapter + k;
    u->scale = scale;
    u->rank = rank;
}

hipError_t launch_set_adapter(Unit *table, int n_layers, int n_adapters, int per_adapter, int adapter,
                              int rank, float scale, hipStream_t s)
{
    const int64_t n = (int64_t)n_layers * per_adapter;
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(set_adapter_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, table,
                       n_layers, n_adapters, per_adapter, adapter, rank, scale);
    return hipGetLastError();
}

template <typename K>
static hipError_t launch_pack(K kernel, const PackParams &p, int64_t groups, hipStream_t s)
{
    if (p.n_units <= 0 || groups <= 0) return hipSuccess;
    dim3 grid((unsigned)((groups + 255) / 256), (unsigned)p.n_units);
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, p);
    return hipGetLastError();
}

static int64_t groups_A(const PackParams &p)
{
    return (int64_t)kblocks_of(p.h, p.rank) * (kunit_of(p.rank) / 8) * p.rank;
}
static int64_t groups_B(const PackParams &p) { return (int64_t)chunks_of(p.h) * 128 * (p.rank / 8); }

hipError_t launch_pack_layer(PackLayerParams &ps, hipStream_t s)
{
    if (ps.n_jobs <= 0 || ps.job[0].n_units <= 0) return hipSuccess;
    ps.aligned = 1;
    for (int j = 0; j < ps.n_jobs; ++j)
        if (reinterpret_cast<uintptr_t>(ps.job[j].src) % 16 || ps.job[j].src_stride % 8) ps.aligned = 0;
    ps.wg0[0] = 0;
    for (int j = 0; j < ps.n_jobs; ++j) {
        const PackParams &p = ps.job[j];
        const int64_t wgs = !ps.aligned ? (((j & 1) ? groups_B(p) : groups_A(p)) + 255) / 256
                            : (j & 1)   ? ((int64_t)chunks_of(p.h) * 16 * (p.rank / 8) + 255) / 256
                                        : (kblocks_of(p.h, p.rank) + 3) / 4;
        ps.wg0[j + 1] = ps.wg0[j] + (int)wgs;
    }
    hipLaunchKernelGGL(pack_layer_kernel, dim3((unsigned)ps.wg0[ps.n_jobs], (unsigned)ps.job[0].n_units), dim3(256), 0,
                       s, ps);
    return hipGetLastError();
}

hipError_t launch_unpack_A(const PackParams &p, hipStream_t s)
{
    return launch_pack(pack_A_kernel<1>, p, groups_A(p), s);
}
hipError_t launch_unpack_B(const PackParams &p, hipStream_t s)
{
    return launch_pack(pack_B_kernel<1>, p, groups_B(p), s);
}

}  // namespace lora

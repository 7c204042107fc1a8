// The contraction kernels around the tile of peqa_tile.h, and their launches, for one number of row tiles (token rows / 16) of
// a tile: every peqa_gemm_r*.hip instantiates GemmRows for one of them (compiled side by side).  What the modes and forms are:
// peqa_gemm.hip.
#pragma once

#include <stddef.h>

#include "peqa_dw_tile.h"
#include "peqa_tile.h"

namespace peqa {

int gemm_pieces(const GemmArgs &a);                        // peqa_gemm.hip
int halves_per_workgroup(int tiles, bool paired);

namespace {

template <int BITS, int MODE, bool GROUPED, int KW, int RT>
__global__ __launch_bounds__(256 * KW, 3 - KW) void gemm_kernel(GemmArgs a)
{
    extern __shared__ __align__(16) uint8_t lds[];
    if constexpr (MODE == MODE_DX && GROUPED && KW == 1) {
        // Workgroups past the tiles: an independent, bandwidth-bound job of the same backward -- the transposed
        // copies of X and dY that the token contraction (the scale gradient, launched next) reads.  They are
        // dispatched last and take the places that the last tiles leave free on the compute units, so most of
        // their time is not added to the launch.
        const int spare = (int)blockIdx.x - ((int)gridDim.x - a.tp_blocks);
        if (spare >= 0) {                                  // a tile per wave, neighbouring columns
            const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), x = 4 * spare + wave;
            const int bts = a.tp_Tp >> 6, kb = a.K >> 6, nb = a.N >> 6;
            u32x4 *piece = reinterpret_cast<u32x4 *>(lds + wave * TRANSPOSE_LDS);
            if (x < bts * kb) transpose_pad_tile(a.tp_X, a.T, a.K, a.tp_Xt, x / kb, x % kb, piece);
            else if (x < bts * (kb + nb)) transpose_pad_tile(a.A, a.T, a.N, a.tp_dYt, (x - bts * kb) / nb, (x - bts * kb) % nb, piece);
            return;
        }
    }
    gemm_tile<BITS, MODE, GROUPED, KW, RT>(a, (int)blockIdx.x, lds);
}

// Row tiles of a split scale gradient's tiles, which take their row sums themselves: as many token rows, or more.
constexpr int piece_rows(int rt) { return rt == 4 ? 4 : 8; }

// Both contractions of a per-channel backward in one launch of four-wave workgroups: the first n_first
// workgroups are the tiles of one of them (the one with the longer contraction), the rest the tiles of the
// other.  Neither reads what the other writes.  Two launches of at most one tile per compute unit each -- which
// would run in the eight-wave form, ring fill and epilogue exposed, or leave most of the machine idle at small T --
// become one launch with up to two workgroups per compute unit, and the last round of the first contraction is
// filled with tiles of the second.
template <int BITS, int RT>
__global__ __launch_bounds__(256, 2) void gemm_bwd_pair_kernel(GemmArgs a_dds, GemmArgs a_dx, int n_first, int dx_first)
{
    extern __shared__ __align__(16) uint8_t lds[];
    const int b = (int)blockIdx.x;
    const bool first = b < n_first;
    const int wg = first ? b : b - n_first;
    if (first == (dx_first != 0)) gemm_tile<BITS, MODE_DX, false, 1, RT>(a_dx, wg, lds);
    else if (a_dds.split > 1) gemm_tile<BITS, MODE_DDS, false, 1, piece_rows(RT), true>(a_dds, wg, lds);
    else gemm_tile<BITS, MODE_DDS, false, 1, RT>(a_dds, wg, lds);
}

// Bandwidth-bound side work inside a multi-contraction launch: auxiliary workgroup `w` of `aux_wgs` walks units w, w + aux_wgs, ...
// Registers are a kernel's, not a workgroup's: what one of these takes, the tiles have taken too.  So a kernel has the side work of
// its own launches only, and that of 64-row tiles stays within what three workgroups per unit leave (see gemm_multi_kernel).
//
// Group-wise dX: the 64 x 64 tiles of the transpose jobs, one per wave.
__device__ __forceinline__ void multi_aux_copies(int n_tp, int aux_wgs, int w, uint8_t *lds)
{
    constexpr uint32_t TP0 = offsetof(MultiArgs, tp);
    auto end_of = [](int i) { return kernarg_load<int>(TP0 + (uint32_t)(i * sizeof(TransposeJob) + offsetof(TransposeJob, tile_end))); };
    const int n_tile = n_tp > 0 ? end_of(n_tp - 1) : 0;
    // a tile per wave; the wave's next tile is asked for before this one is turned
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    u32x4 *piece = reinterpret_cast<u32x4 *>(lds + wave * TRANSPOSE_LDS);
    struct Tile { TransposeJob J; int bt, bc; };
    auto tile_of = [&](int x) __attribute__((always_inline)) {
        int j = 0, x0 = 0;
        for (int i = 0; i + 1 < n_tp; ++i) {
            const int e = end_of(i);
            if (x >= e) { j = i + 1; x0 = e; }
        }
        Tile t;
        t.J = kernarg_load<TransposeJob>(TP0 + (uint32_t)(j * sizeof(TransposeJob)));
        const int bcs = t.J.C >> 6;
        t.bt = (x - x0) / bcs;
        t.bc = (x - x0) - t.bt * bcs;
        return t;
    };
    int x = 4 * w + wave;
    if (x >= n_tile) return;
    Tile t = tile_of(x);
    TransposeRows r;
    transpose_load(t.J.src, t.J.T, t.J.C, t.bt, t.bc, r);
    for (;;) {
        x += 4 * aux_wgs;
        Tile next = t;
        TransposeRows ahead;
        if (x < n_tile) {
            next = tile_of(x);
            transpose_load(next.J.src, next.J.T, next.J.C, next.bt, next.bc, ahead);
        }
        transpose_store(r, t.J.C, t.J.dst, t.bt, t.bc, piece);
        if (x >= n_tile) break;
        t = next;
        r = ahead;
    }
}

// Per channel: one index space, first the SDY_ROWS-row blocks of the scale_dy jobs, then the 256-element chunks of the reduce jobs.
template <int SDY_ROWS>
__device__ __forceinline__ void multi_aux(int n_sdy, int n_red, int aux_wgs, int w, uint8_t *lds)
{
    float *red = reinterpret_cast<float *>(lds);
    constexpr uint32_t SDY0 = offsetof(MultiArgs, sdy), RED0 = offsetof(MultiArgs, red);
    auto last = [](uint32_t table, int n, size_t size, size_t member) {   // a running total's value behind the last of n jobs
        return n > 0 ? kernarg_load<int>(table + (uint32_t)((n - 1) * size + member)) : 0;
    };
    const int n_blk = last(SDY0, n_sdy, sizeof(ScaleDyJob), offsetof(ScaleDyJob, blk_end));
    const int n_chunk = last(RED0, n_red, sizeof(ReduceJob), offsetof(ReduceJob, chunk_end));
    for (int u = w; u < n_blk + n_chunk; u += aux_wgs) {
        if (u < n_blk) {
            int j = 0, b0 = 0;
            for (int i = 0; i + 1 < n_sdy; ++i) {
                const int e = kernarg_load<int>(SDY0 + (uint32_t)(i * sizeof(ScaleDyJob) + offsetof(ScaleDyJob, blk_end)));
                if (u >= e) { j = i + 1; b0 = e; }
            }
            const ScaleDyJob J = kernarg_load<ScaleDyJob>(SDY0 + (uint32_t)(j * sizeof(ScaleDyJob)));
            scale_dy_rows<SDY_ROWS>(J.dY, J.s0, J.ds, J.z0, nullptr, J.T, J.N, J.dYs, J.crow, u - b0, red);
            __syncthreads();                                   // `red` is reused by the next block
        } else {
            const int c = u - n_blk;
            int j = 0, c0 = 0;
            for (int i = 0; i + 1 < n_red; ++i) {
                const int e = kernarg_load<int>(RED0 + (uint32_t)(i * sizeof(ReduceJob) + offsetof(ReduceJob, chunk_end)));
                if (c >= e) { j = i + 1; c0 = e; }
            }
            const ReduceJob J = kernarg_load<ReduceJob>(RED0 + (uint32_t)(j * sizeof(ReduceJob)));
            reduce_partials_at(J.partial, J.ntiles, (size_t)J.n, (size_t)(c - c0) * 256 + threadIdx.x, J.out);
        }
    }
}

// Several per-channel contractions as four-wave tiles of one launch (see MultiArgs): workgroup -> (job, tile) by the
// jobs' running totals; the job's arguments come out of the argument block with scalar loads.
// GMODE < 0: per-channel jobs of any mode; GMODE = MODE_Y or MODE_DX: group-wise jobs, all of that mode (their
// scale gradient is the token contraction of peqa_dw.hip).
//
// Per-channel tiles of 64 rows have 48 KB of LDS and 64 accumulators: three workgroups fit a unit as long as the kernel takes no
// more than 104 registers besides.  With the copies' two tiles in flight and the scaling of eight rows compiled in it took 127 (92
// without), and blocks of 513 to 768 workgroups a second round.  Blocks of d = 8192, f = 22016 (752 and 760 workgroups), us, two on a
// unit -> three: forward at T = 17 / 32 107.9 / 116.5 -> 104.2 / 111.9, training step 329 / 346 -> 302 / 322; d = 6656, f = 17920, T = 32
// 237 -> 230.
template <int BITS, int GMODE, int RT>
__global__ __launch_bounds__(256, 2) void gemm_multi_kernel(MultiArgs m)
{
    extern __shared__ __align__(16) uint8_t lds[];
    int b = (int)blockIdx.x;
    if constexpr (GMODE != MODE_Y) {                           // a group-wise forward has no side work
        if (b >= m.aux_begin) {
            if (b < m.aux_begin + m.aux_wgs) {
                if constexpr (GMODE < 0) multi_aux<aux_sdy_rows(RT)>(m.n_sdy, m.n_red, m.aux_wgs, b - m.aux_begin, lds);
                else multi_aux_copies(m.n_tp, m.aux_wgs, b - m.aux_begin, lds);
                return;
            }
            b -= m.aux_wgs;
        }
    }
    int j = 0, wg0 = 0;
#pragma unroll
    for (int i = 0; i < MULTI_MAX_JOBS - 1; ++i) {
        const int e = kernarg_load<int>((uint32_t)(i * sizeof(MultiJob) + offsetof(MultiJob, wg_end)));
        if (b >= e) { j = i + 1; wg0 = e; }
    }
    const GemmArgs a = kernarg_load<GemmArgs>((uint32_t)(j * sizeof(MultiJob) + offsetof(MultiJob, a)));
    if constexpr (GMODE >= 0) {
        gemm_tile<BITS, GMODE, true, 1, RT>(a, b - wg0, lds);
    } else {
        const int mode = kernarg_load<int>((uint32_t)(j * sizeof(MultiJob) + offsetof(MultiJob, mode)));
        if (mode == MODE_Y) gemm_tile<BITS, MODE_Y, false, 1, RT>(a, b - wg0, lds);
        else if (mode == MODE_DDS && a.split > 1) gemm_tile<BITS, MODE_DDS, false, 1, piece_rows(RT), true>(a, b - wg0, lds);
        else if (mode == MODE_DDS) gemm_tile<BITS, MODE_DDS, false, 1, RT>(a, b - wg0, lds);
        else gemm_tile<BITS, MODE_DX, false, 1, RT>(a, b - wg0, lds);
    }
}

// The dX tiles and the token contractions of a group-wise backward (GemmDwArgs), which read nothing of each other's: the
// workgroups that take longer first, so that the others fill the launch's end.  11008 x 4096 in groups of 64, T = 500, training
// step: 196 us in launches of their own, 184 in this one; 4864 x 512 in groups of 128, T = 39: 48 and 34.
template <int BITS, int RT>
__global__ __launch_bounds__(256, 2) void gemm_dw_kernel(GemmDwArgs m)
{
    extern __shared__ __align__(16) uint8_t lds[];
    int b = (int)blockIdx.x;
    int j = 0, wg0 = 0;
    if (b >= m.dw_begin && b < m.dw_begin + m.dw_total) {
        b -= m.dw_begin;
#pragma unroll
        for (int i = 0; i < DW_MAX_JOBS - 1; ++i) {
            const int e = kernarg_load<int>((uint32_t)(offsetof(GemmDwArgs, dw_end) + 4 * i));
            if (b >= e) { j = i + 1; wg0 = e; }
        }
        const DwArgs a = kernarg_load<DwArgs>((uint32_t)(offsetof(GemmDwArgs, dw) + j * sizeof(DwArgs)));
        dw_tile<BITS>(a, b - wg0, lds);
        return;
    }
    b -= m.gemm_begin;
#pragma unroll
    for (int i = 0; i < MULTI_MAX_JOBS - 1; ++i) {
        const int e = kernarg_load<int>((uint32_t)(i * sizeof(MultiJob) + offsetof(MultiJob, wg_end)));
        if (b >= e) { j = i + 1; wg0 = e; }
    }
    const GemmArgs a = kernarg_load<GemmArgs>((uint32_t)(j * sizeof(MultiJob) + offsetof(MultiJob, a)));
    gemm_tile<BITS, MODE_DX, true, 1, RT>(a, b - wg0, lds);
}

}  // namespace

template <int BITS, int MODE, bool GROUPED, int KW, int RT>
static hipError_t launch_one(const GemmArgs &a, hipStream_t stream)
{
    // dynamic LDS: the ring, plus the scale tables of the grouped forward / dX
    const int lds_bytes = ring_bytes(KW, RT) + (GROUPED && MODE != MODE_DDS ? tbl_bytes(KW) : 0);
    // the limit is a per-device attribute of every instantiation; raised to what a launch needs
    static int attr_bytes[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (attr_bytes[dev] < lds_bytes) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_kernel<BITS, MODE, GROUPED, KW, RT>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        if (e != hipSuccess) return e;
        attr_bytes[dev] = lds_bytes;
    }
    const int grid = gemm_multi_wgs(a);
    // grouped scale gradient: one pair of scale groups per workgroup along y
    const int gy = GROUPED && MODE == MODE_DDS ? (a.G + 1) / 2 : 1;
    // spare workgroups (see the kernel) exist in one instantiation only
    constexpr bool SPARE_TP = MODE == MODE_DX && GROUPED && KW == 1;
    if (!SPARE_TP && a.tp_blocks != 0) return hipErrorInvalidValue;
    const int spare_blocks = SPARE_TP ? a.tp_blocks : 0;
    hipLaunchKernelGGL((gemm_kernel<BITS, MODE, GROUPED, KW, RT>), dim3(grid + spare_blocks, gy), dim3(256 * KW), lds_bytes,
                       stream, a);
    return hipGetLastError();
}

template <int BITS, int MODE, bool GROUPED, int RT>
static hipError_t launch_halves(const GemmArgs &a, hipStream_t stream)
{
    constexpr bool PAIRED = GROUPED && MODE == MODE_DDS;
    if constexpr (!PAIRED) {
        if (halves_per_workgroup(a.tiles_t * a.tiles_c * gemm_pieces(a), false) == 1)
            return launch_one<BITS, MODE, GROUPED, 1, RT>(a, stream);
    }
    return launch_one<BITS, MODE, GROUPED, 2, RT>(a, stream);
}

template <int BITS, bool GROUPED, int RT>
static hipError_t dispatch_mode(int mode, const GemmArgs &a, hipStream_t stream)
{
    switch (mode) {
    case MODE_Y: return launch_halves<BITS, MODE_Y, GROUPED, RT>(a, stream);
    case MODE_DDS:
        if constexpr (GROUPED && RT != 8) return hipErrorInvalidValue;   // (the older route: whole tiles only)
        else return launch_halves<BITS, MODE_DDS, GROUPED, RT>(a, stream);
    default: return launch_halves<BITS, MODE_DX, GROUPED, RT>(a, stream);
    }
}

// Scale gradient and dX of one per-channel layer in one launch (see gemm_bwd_pair_kernel).
template <int BITS, int RT>
static hipError_t launch_pair(const GemmArgs &a_dds, const GemmArgs &a_dx, hipStream_t stream)
{
    const int lds_bytes = ring_bytes(1, RT);
    static int attr_bytes[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (attr_bytes[dev] < lds_bytes) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_bwd_pair_kernel<BITS, RT>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        if (e != hipSuccess) return e;
        attr_bytes[dev] = lds_bytes;
    }
    // the tiles that take longer go first: the short ones fill the last round better
    // (the numbers of workgroups are multiples of 8: both parts keep workgroup id % 8 = XCD)
    const int dx_first = a_dx.KC / gemm_pieces(a_dx) >= a_dds.KC / gemm_pieces(a_dds);
    const int n_first = gemm_multi_wgs(dx_first ? a_dx : a_dds), n_second = gemm_multi_wgs(dx_first ? a_dds : a_dx);
    hipLaunchKernelGGL((gemm_bwd_pair_kernel<BITS, RT>), dim3(n_first + n_second), dim3(256), lds_bytes, stream, a_dds, a_dx,
                       n_first, dx_first);
    return hipGetLastError();
}

template <int BITS, int GMODE, int RT>
static hipError_t launch_multi(dim3 grid, int lds_bytes, const MultiArgs &m, hipStream_t stream)
{
    static int attr_bytes[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (attr_bytes[dev] < lds_bytes) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_multi_kernel<BITS, GMODE, RT>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        if (e != hipSuccess) return e;
        attr_bytes[dev] = lds_bytes;
    }
    hipLaunchKernelGGL((gemm_multi_kernel<BITS, GMODE, RT>), grid, dim3(256), lds_bytes, stream, m);
    return hipGetLastError();
}

template <int RT>
hipError_t GemmRows<RT>::one(int bits, int mode, const GemmArgs &a, hipStream_t stream)
{
    const bool grouped = a.gsz > 0;
    if (bits == 4) return grouped ? dispatch_mode<4, true, RT>(mode, a, stream) : dispatch_mode<4, false, RT>(mode, a, stream);
    return grouped ? dispatch_mode<3, true, RT>(mode, a, stream) : dispatch_mode<3, false, RT>(mode, a, stream);
}

template <int RT>
hipError_t GemmRows<RT>::pair(int bits, const GemmArgs &a_dds, const GemmArgs &a_dx, hipStream_t stream)
{
    return bits == 4 ? launch_pair<4, RT>(a_dds, a_dx, stream) : launch_pair<3, RT>(a_dds, a_dx, stream);
}

template <int BITS, int RT>
static hipError_t launch_with_dw(int workgroups, const GemmDwArgs &m, hipStream_t stream)
{
    constexpr int gemm_lds = ring_bytes(1, RT) + tbl_bytes(1), lds_bytes = gemm_lds > DW_LDS ? gemm_lds : DW_LDS;
    static bool allowed[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (!allowed[dev]) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_dw_kernel<BITS, RT>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        if (e != hipSuccess) return e;
        allowed[dev] = true;
    }
    hipLaunchKernelGGL((gemm_dw_kernel<BITS, RT>), dim3(workgroups), dim3(256), lds_bytes, stream, m);
    return hipGetLastError();
}

template <int RT>
hipError_t GemmRows<RT>::with_dw(int bits, int workgroups, const GemmDwArgs &m, hipStream_t stream)
{
    return bits == 4 ? launch_with_dw<4, RT>(workgroups, m, stream) : launch_with_dw<3, RT>(workgroups, m, stream);
}

template <int RT>
hipError_t GemmRows<RT>::multi(int bits, int gmode, int workgroups, const MultiArgs &m, hipStream_t stream)
{
    // group-wise: the scale tables behind the ring
    const int lds_bytes = ring_bytes(1, RT) + (gmode >= 0 ? tbl_bytes(1) : 0);
    const dim3 grid(workgroups);
    if (gmode < 0)
        return bits == 4 ? launch_multi<4, -1, RT>(grid, lds_bytes, m, stream) : launch_multi<3, -1, RT>(grid, lds_bytes, m, stream);
    if (gmode == MODE_Y)
        return bits == 4 ? launch_multi<4, MODE_Y, RT>(grid, lds_bytes, m, stream)
                         : launch_multi<3, MODE_Y, RT>(grid, lds_bytes, m, stream);
    return bits == 4 ? launch_multi<4, MODE_DX, RT>(grid, lds_bytes, m, stream)
                     : launch_multi<3, MODE_DX, RT>(grid, lds_bytes, m, stream);
}

}  // namespace peqa

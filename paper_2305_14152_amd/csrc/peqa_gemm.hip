// Dense contractions of the PEQA linear layer on gfx950 MFMA (per-channel scales).
//
//   MODE_Y   : Y[t,i]    = s_i * sum_k X[t,k] (Q[i,k] - z_i)                (Eq. 2 forward)
//   MODE_DDS : part[i]   = sum_{t in tile} dY[t,i] * sum_k X[t,k] (Q[i,k] - z_i)
//                                                   (scale gradient, column-reduced epilogue)
//   MODE_DX  : dX[t,k]   = sum_i (dY[t,i] s_i) (Q[i,k] - z_i)                (chain rule on Eq. 2)
//
// A workgroup owns a 128 (tokens) x 256 (output columns) tile (peqa_tile.h) as four waves of 128 x 64 side by side
// along the columns: 8 x 4 MFMA 16x16x32 tiles, 128 fp32 AGPRs per wave.  Two forms:
//   KW = 1: four waves run the whole contraction range; two workgroups per compute unit, i.e. two waves per SIMD, so that
//           the LDS reads, the unpacking and the scalar bookkeeping of one hide behind the matrix instructions of the
//           other, and one workgroup's ring fill and epilogue behind the other's loop.
//   KW = 2: eight waves, four per half of the contraction range, one workgroup per compute unit with twice the ring; the
//           halves are summed through LDS in the epilogue (or, for MODE_DDS, after the column reduction, which is linear).
//           For launches with at most one tile per compute unit (see halves_per_workgroup below).
// The scale gradient and dX of one per-channel backward run as four-wave tiles of one launch (gemm_bwd_pair_kernel); in
// the group-wise dX launch, spare workgroups at the end of the grid write the transposed operands of the token contraction.
//
// Operand paths.  Both operands go global -> LDS by DMA (global_load_lds) into a ring of
// stages, one 32-deep contraction step per stage: the activation operand (X, or the pre-scaled
// dY) as 128 x 32 bf16 tiles (16-byte chunks XOR-swizzled by row), the weight operand as
// the packed 8x8 code blocks themselves, half a block per lane.  Each lane reads its words back and
// unpacks them in registers into bf16 (16 + Q) fragments (peqa_device.h): dequantised weights
// never exist in memory.  The contraction therefore runs on exact small integers; the offset 16,
// the zero-point and the scale are applied in the epilogue from row sums of the other
// operand:   sum_k X (Q - z) = sum_k X (16 + Q) - (16 + z) sum_k X.
//
// Group-wise scales (Sec. 4.2 and Table 5; group size a multiple of 64) use the GROUPED instantiations:
//   MODE_Y, MODE_DX : the scale cannot leave the contraction, so every weight enters the MFMA as
//                     bf16( s[i,g] (Q[i,k] - z[i,g]) ), formed in fp32 from a per-group table of
//                     (s, -s (16 + z)) that rides through LDS next to the operand ring; the
//                     epilogue is a plain store and the activation operand is X / dY itself.
//   MODE_DDS        : one workgroup contracts one pair of scale groups (blockIdx.y), each
//                     contraction half one group, and the column-reduced epilogue writes one
//                     partial per (token tile, channel, group).  This is the older of two routes to
//                     the grouped scale gradient (the default contracts over tokens, peqa_dw.hip)
//                     and runs only on request (option grouped_dds = 1).
#include <stddef.h>

#include "peqa_tile.h"

namespace peqa {

namespace {

template <int BITS, int MODE, bool GROUPED, int KW>
__global__ __launch_bounds__(256 * KW, 3 - KW) void gemm_kernel(GemmArgs a)
{
    extern __shared__ __align__(16) uint8_t lds[];
    if constexpr (MODE == MODE_DX && GROUPED && KW == 1) {
        // Workgroups past the tiles: an independent, bandwidth-bound job of the same backward -- the transposed
        // copies of X and dY that the token contraction (the scale gradient, launched next) reads.  They are
        // dispatched last and take the places that the last tiles leave free on the compute units, so most of
        // their time is not added to the launch.
        const int spare = (int)blockIdx.x - ((int)gridDim.x - a.tp_blocks);
        if (spare >= 0) {
            const int bts = a.tp_Tp >> 6, nx = bts * (a.K >> 6);
            uint16_t(*tile)[64 + 2] = reinterpret_cast<uint16_t(*)[64 + 2]>(lds);
            if (spare < nx) transpose_pad_tile(a.tp_X, a.T, a.K, a.tp_Xt, spare % bts, spare / bts, tile);
            else transpose_pad_tile(a.A, a.T, a.N, a.tp_dYt, (spare - nx) % bts, (spare - nx) / bts, tile);
            return;
        }
    }
    gemm_tile<BITS, MODE, GROUPED, KW>(a, (int)blockIdx.x, lds);
}

// Both contractions of a per-channel backward in one launch of four-wave workgroups: the first n_first
// workgroups are the tiles of one of them (the one with the longer contraction), the rest the tiles of the
// other.  Neither reads what the other writes.  Two launches of at most one tile per compute unit each -- which
// would run in the eight-wave form, ring fill and epilogue exposed, or leave most of the machine idle at small T --
// become one launch with up to two workgroups per compute unit, and the last round of the first contraction is
// filled with tiles of the second.
template <int BITS>
__global__ __launch_bounds__(256, 2) void gemm_bwd_pair_kernel(GemmArgs a_dds, GemmArgs a_dx, int n_first, int dx_first)
{
    extern __shared__ __align__(16) uint8_t lds[];
    const int b = (int)blockIdx.x;
    const bool first = b < n_first;
    const int wg = first ? b : b - n_first;
    if (first == (dx_first != 0)) gemm_tile<BITS, MODE_DX, false, 1>(a_dx, wg, lds);
    else if (a_dds.split > 1) gemm_tile<BITS, MODE_DDS, false, 1, true>(a_dds, wg, lds);
    else gemm_tile<BITS, MODE_DDS, false, 1>(a_dds, wg, lds);
}

// Bandwidth-bound side work inside a multi-contraction launch: auxiliary workgroup `w` of `m.aux_wgs` walks the
// units w, w + aux_wgs, ... of one index space: first the SDY_ROWS-row blocks of the scale_dy jobs, then the
// 256-element chunks of the reduce jobs.
static_assert(SDY_ROWS == SDY_ROWS_HOST, "row blocks of scale_dy_rows");
__device__ __forceinline__ void multi_aux(int n_sdy, int n_red, int n_tp, int aux_wgs, int w, uint8_t *lds)
{
    struct { int n_sdy, n_red, n_tp, aux_wgs; } m{n_sdy, n_red, n_tp, aux_wgs};
    float *red = reinterpret_cast<float *>(lds);
    constexpr uint32_t SDY0 = offsetof(MultiArgs, sdy), RED0 = offsetof(MultiArgs, red), TP0 = offsetof(MultiArgs, tp);
    auto last = [](uint32_t table, int n, size_t size, size_t member) {   // a running total's value behind the last of n jobs
        return n > 0 ? kernarg_load<int>(table + (uint32_t)((n - 1) * size + member)) : 0;
    };
    const int n_blk = last(SDY0, m.n_sdy, sizeof(ScaleDyJob), offsetof(ScaleDyJob, blk_end));
    const int n_chunk = last(RED0, m.n_red, sizeof(ReduceJob), offsetof(ReduceJob, chunk_end));
    const int n_tile = last(TP0, m.n_tp, sizeof(TransposeJob), offsetof(TransposeJob, tile_end));
    for (int u = w; u < n_blk + n_chunk + n_tile; u += m.aux_wgs) {
        if (u >= n_blk + n_chunk) {
            const int x = u - n_blk - n_chunk;
            int j = 0, x0 = 0;
            for (int i = 0; i + 1 < m.n_tp; ++i) {
                const int e = kernarg_load<int>(TP0 + (uint32_t)(i * sizeof(TransposeJob) + offsetof(TransposeJob, tile_end)));
                if (x >= e) { j = i + 1; x0 = e; }
            }
            const TransposeJob J = kernarg_load<TransposeJob>(TP0 + (uint32_t)(j * sizeof(TransposeJob)));
            const int bts = J.Tp >> 6;
            transpose_pad_tile(J.src, J.T, J.C, J.dst, (x - x0) % bts, (x - x0) / bts, reinterpret_cast<uint16_t(*)[64 + 2]>(lds));
            __syncthreads();                                   // the LDS tile is reused by the next one
            continue;
        }
        if (u < n_blk) {
            int j = 0, b0 = 0;
            for (int i = 0; i + 1 < m.n_sdy; ++i) {
                const int e = kernarg_load<int>(SDY0 + (uint32_t)(i * sizeof(ScaleDyJob) + offsetof(ScaleDyJob, blk_end)));
                if (u >= e) { j = i + 1; b0 = e; }
            }
            const ScaleDyJob J = kernarg_load<ScaleDyJob>(SDY0 + (uint32_t)(j * sizeof(ScaleDyJob)));
            scale_dy_rows(J.dY, J.s0, J.ds, J.z0, nullptr, J.T, J.N, J.dYs, J.crow, u - b0, red);
            __syncthreads();                                   // `red` is reused by the next block
        } else {
            const int c = u - n_blk;
            int j = 0, c0 = 0;
            for (int i = 0; i + 1 < m.n_red; ++i) {
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
template <int BITS, int GMODE>
__global__ __launch_bounds__(256, 2) void gemm_multi_kernel(MultiArgs m)
{
    extern __shared__ __align__(16) uint8_t lds[];
    int b = (int)blockIdx.x;
    if constexpr (GMODE != MODE_Y) {                           // a group-wise forward has no side work
        if (b >= m.aux_begin) {
            if (b < m.aux_begin + m.aux_wgs) {
                multi_aux(m.n_sdy, m.n_red, m.n_tp, m.aux_wgs, b - m.aux_begin, lds);
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
        gemm_tile<BITS, GMODE, true, 1>(a, b - wg0, lds);
    } else {
        const int mode = kernarg_load<int>((uint32_t)(j * sizeof(MultiJob) + offsetof(MultiJob, mode)));
        if (mode == MODE_Y) gemm_tile<BITS, MODE_Y, false, 1>(a, b - wg0, lds);
        else if (mode == MODE_DDS && a.split > 1) gemm_tile<BITS, MODE_DDS, false, 1, true>(a, b - wg0, lds);
        else if (mode == MODE_DDS) gemm_tile<BITS, MODE_DDS, false, 1>(a, b - wg0, lds);
        else gemm_tile<BITS, MODE_DX, false, 1>(a, b - wg0, lds);
    }
}

// One 256-thread workgroup per 1024 elements of a split contraction's result, four neighbouring columns per thread:
// HBM-bound, split x 4 + 2 bytes per element.
__global__ __launch_bounds__(256) void split_finish_kernel(FinishMulti f)
{
    const FinishJob J = kernarg_load<FinishJob>((uint32_t)(blockIdx.y * sizeof(FinishJob)));
    const GemmArgs &a = J.a;
    if (a.split < 2) return;
    const uint32_t c4 = (uint32_t)a.C >> 2;
    const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= (size_t)a.T * c4) return;
    const size_t t = e / c4;
    const int col = (int)(e - t * c4) * 4;
    const f32x4 *p = reinterpret_cast<const f32x4 *>(a.acc_part) + e;
    const size_t stride = (size_t)a.T * c4;
    f32x4 v = p[0];
    int i = 1;
    for (; i + 4 <= a.split; i += 4) {                         // four loads in flight, added in order
        f32x4 w[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) w[u] = p[(size_t)(i + u) * stride];
#pragma unroll
        for (int u = 0; u < 4; ++u) v += w[u];
    }
    for (; i < a.split; ++i) v += p[(size_t)i * stride];
    if (a.gsz == 0) {
        if (J.mode == MODE_Y) {
            const float r = a.rs[2 * t] + a.rs[2 * t + 1];
            const uint32_t zz = *reinterpret_cast<const uint32_t *>(a.z0 + col);
            f32x4 zoff;
#pragma unroll
            for (int u = 0; u < 4; ++u) zoff[u] = kCodeOffset + (float)((zz >> (8 * u)) & 0xFFu);
            if (a.dz) zoff += *reinterpret_cast<const f32x4 *>(a.dz + col);
            f32x4 sc = *reinterpret_cast<const f32x4 *>(a.s0 + col);
            if (a.ds) sc += *reinterpret_cast<const f32x4 *>(a.ds + col);
            v -= zoff * r;
            if (a.P) *reinterpret_cast<f32x4 *>(a.P + t * a.C + col) = v;
            v *= sc;
        } else {
            v -= a.crow[t];
        }
    }
    u32x2 o;
    o[0] = pack_bf16x2(v[0], v[1]);
    o[1] = pack_bf16x2(v[2], v[3]);
    *reinterpret_cast<u32x2 *>(a.out + t * a.C + col) = o;
}

}  // namespace

hipError_t launch_split_finish(const FinishMulti &f, hipStream_t stream)
{
    size_t most = 0;
    for (int j = 0; j < f.n; ++j) {
        const GemmArgs &a = f.job[j].a;
        if (a.split > 1 && (size_t)a.T * a.C > most) most = (size_t)a.T * a.C;
    }
    if (most == 0) return hipSuccess;
    trace_before(KID_GEMM_FINISH, stream);
    hipLaunchKernelGGL(split_finish_kernel, dim3((unsigned)((most + 1023) / 1024), f.n), dim3(256), 0, stream, f);
    trace_after(KID_GEMM_FINISH, stream);
    return hipGetLastError();
}

// Contraction halves per workgroup.  Eight waves with two halves, one workgroup per compute unit, when a launch
// has at most one tile per compute unit (a lone four-wave workgroup leaves every SIMD a single wave, which
// measures 7-10 % slower); otherwise four waves with the whole range and two workgroups per compute unit
// (72 KB of LDS each), which fill the same four SIMDs with two waves each, need no exchange of partial sums,
// and hide one workgroup's ring fill and epilogue behind the other's loop.  The option gemm_waves = 4 or 8
// (peqa_set_option) forces one of them, for tests and comparisons.
static int halves_per_workgroup(int tiles, bool paired)
{
    if (paired) return 2;
    if (options().gemm_waves == 4) return 1;
    if (options().gemm_waves == 8) return 2;
    const int cus = compute_units();
    return tiles > cus ? 1 : 2;
}

static int pieces(const GemmArgs &a) { return a.split > 1 ? a.split : 1; }

// Workgroups that the tiles of a contraction take in a launch: their number rounded up to a multiple of 8.
int gemm_multi_wgs(const GemmArgs &a) { return (a.tiles_t * a.tiles_c * pieces(a) + 7) / 8 * 8; }

// A launch lasts as long as its longest workgroup (a step of 32 takes 0.40 us with one workgroup on the compute unit, 0.66
// with two; 8 us to fill the ring, drain and store) or as the work that two workgroups per unit get through, plus about a
// third of a workgroup for the last round (per-channel figures; the vector instructions of group-wise scaling make a step
// 1.6 times as long).  Pieces of Y and dX cost a second launch and fp32 sums written and read again (3.5 TB/s).  Among
// splits into pieces of equal length over the launch the one with the least estimate is taken, if that is 13 % below the
// unsplit one: the estimate is no better than that, and splits with less to gain measured between 5 % faster and 7 %
// slower (4096 x 11008 backward at T = 800 and 1200).  Measured, whole -> split, us per call:
//                                     T = 17          T = 128         T = 500
//   7B block 4-bit, forward           124 ->  56      131 ->  71      whole
//                   backward          392 -> 108      397 -> 140      480 -> 367
//   13B block 3-bit g128, forward     239 ->  93      240 -> 113      whole
//                         backward    708 -> 310      749 -> 393      953 -> 853
//   4096 x 11008 4-bit alone, forward 103 ->  28      107 ->  37      112 ->  72
void gemm_plan_splits(int n, SplitJob *jobs, bool grouped, bool single, size_t max_bytes, int cus)
{
    int longest = 0;
    for (int j = 0; j < n; ++j) {
        jobs[j].split = 1;
        longest = jobs[j].KC > longest ? jobs[j].KC : longest;
    }
    if (options().gemm_waves != 0 || options().bwd_pair >= 0) return;   // forced forms are whole contractions
    constexpr int kMinPiece = 512;                             // shorter pieces are mostly fill and drain
    const double f = grouped ? 1.6 : 1.0;
    double best = 0.0;
    for (int d = 1; d <= 48; d += d < 6 ? 1 : (d < 12 ? 2 : 4)) {
        const int target = (longest + d - 1) / d;              // features (or channels) per piece
        if (d > 1 && target < kMinPiece) break;
        int s[FINISH_MAX], wgs = 0, piece = 0;
        double steps = 0.0;
        size_t bytes = 0;
        for (int j = 0; j < n; ++j) {
            s[j] = (jobs[j].KC + target - 1) / target;
            s[j] = s[j] < jobs[j].KC / kMinPiece ? s[j] : (jobs[j].KC < kMinPiece ? 1 : jobs[j].KC / kMinPiece);
            wgs += jobs[j].tiles * s[j];
            const int len = (jobs[j].KC / 128 + s[j] - 1) / s[j] * 4;
            piece = len > piece ? len : piece;
            steps += (double)jobs[j].tiles * jobs[j].KC / 32;
            if (s[j] > 1) bytes += s[j] * jobs[j].out_bytes;
        }
        if (d > 1 && bytes > max_bytes) continue;
        double us;
        if (single && wgs <= cus) {
            us = 0.33 * f * piece + 11.0;                      // the eight-wave form
        } else {
            const double chain = 0.40 * f * piece + 8.0, work = (0.66 * f * steps + 8.0 * wgs) / (2.0 * cus) + 0.3 * chain;
            us = chain > work ? chain : work;
        }
        if (bytes > 0) us += 4.0 + (double)bytes * 2.0 / 3.5e6;
        if (d == 1) {
            best = 0.87 * us;
        } else if (us < best) {
            best = us;
            for (int j = 0; j < n; ++j) jobs[j].split = s[j];
        }
    }
}

bool gemm_four_waves(int tiles) { return halves_per_workgroup(tiles, false) == 1; }

template <int BITS, int MODE, bool GROUPED, int KW>
static hipError_t launch_one(const GemmArgs &a, hipStream_t stream)
{
    // dynamic LDS: the ring, plus the scale tables of the grouped forward / dX
    const int lds_bytes = ring_bytes(KW) + (GROUPED && MODE != MODE_DDS ? tbl_bytes(KW) : 0);
    // the limit is a per-device attribute of every instantiation; raised to what a launch needs
    static int attr_bytes[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (attr_bytes[dev] < lds_bytes) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_kernel<BITS, MODE, GROUPED, KW>),
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
    hipLaunchKernelGGL((gemm_kernel<BITS, MODE, GROUPED, KW>), dim3(grid + spare_blocks, gy), dim3(256 * KW), lds_bytes,
                       stream, a);
    return hipGetLastError();
}

template <int BITS, int MODE, bool GROUPED>
static hipError_t launch_halves(const GemmArgs &a, hipStream_t stream)
{
    constexpr bool PAIRED = GROUPED && MODE == MODE_DDS;
    if constexpr (!PAIRED) {
        if (halves_per_workgroup(a.tiles_t * a.tiles_c * pieces(a), false) == 1)
            return launch_one<BITS, MODE, GROUPED, 1>(a, stream);
    }
    return launch_one<BITS, MODE, GROUPED, 2>(a, stream);
}

template <int BITS, bool GROUPED>
static hipError_t dispatch_mode(int mode, const GemmArgs &a, hipStream_t stream)
{
    switch (mode) {
    case MODE_Y: return launch_halves<BITS, MODE_Y, GROUPED>(a, stream);
    case MODE_DDS: return launch_halves<BITS, MODE_DDS, GROUPED>(a, stream);
    default: return launch_halves<BITS, MODE_DX, GROUPED>(a, stream);
    }
}

static hipError_t dispatch(int bits, int mode, const GemmArgs &a, hipStream_t stream)
{
    const bool grouped = a.gsz > 0;
    if (bits == 4) return grouped ? dispatch_mode<4, true>(mode, a, stream) : dispatch_mode<4, false>(mode, a, stream);
    return grouped ? dispatch_mode<3, true>(mode, a, stream) : dispatch_mode<3, false>(mode, a, stream);
}

hipError_t launch_gemm(int bits, int mode, const GemmArgs &a_in, hipStream_t stream)
{
    GemmArgs a = a_in;
    a.patch_t = a.tiles_t < 4 ? a.tiles_t : 4;
    const int kid = mode == MODE_Y ? KID_GEMM_Y : (mode == MODE_DDS ? KID_GEMM_DDS : KID_GEMM_DX);
    trace_before(kid, stream);
    const hipError_t e = dispatch(bits, mode, a, stream);
    trace_after(kid, stream);
    return e;
}

// Scale gradient and dX of one per-channel layer in one launch (see gemm_bwd_pair_kernel).
template <int BITS>
static hipError_t launch_pair(const GemmArgs &a_dds, const GemmArgs &a_dx, hipStream_t stream)
{
    const int lds_bytes = ring_bytes(1);
    static int attr_bytes[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (attr_bytes[dev] < lds_bytes) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_bwd_pair_kernel<BITS>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        if (e != hipSuccess) return e;
        attr_bytes[dev] = lds_bytes;
    }
    // the tiles that take longer go first: the short ones fill the last round better
    // (the numbers of workgroups are multiples of 8: both parts keep workgroup id % 8 = XCD)
    const int dx_first = a_dx.KC / pieces(a_dx) >= a_dds.KC / pieces(a_dds);
    const int n_first = gemm_multi_wgs(dx_first ? a_dx : a_dds), n_second = gemm_multi_wgs(dx_first ? a_dds : a_dx);
    hipLaunchKernelGGL((gemm_bwd_pair_kernel<BITS>), dim3(n_first + n_second), dim3(256), lds_bytes, stream, a_dds, a_dx,
                       n_first, dx_first);
    return hipGetLastError();
}

template <int BITS, int GMODE>
static hipError_t launch_multi(dim3 grid, int lds_bytes, const MultiArgs &m, hipStream_t stream)
{
    static int attr_bytes[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (attr_bytes[dev] < lds_bytes) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_multi_kernel<BITS, GMODE>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        if (e != hipSuccess) return e;
        attr_bytes[dev] = lds_bytes;
    }
    hipLaunchKernelGGL((gemm_multi_kernel<BITS, GMODE>), grid, dim3(256), lds_bytes, stream, m);
    return hipGetLastError();
}

hipError_t launch_gemm_multi(int bits, bool grouped, MultiArgs &m, hipStream_t stream)
{
    if (m.n_jobs < 0 || m.n_jobs > MULTI_MAX_JOBS || m.n_sdy < 0 || m.n_sdy > MULTI_MAX_JOBS || m.n_red < 0 ||
        m.n_red > MULTI_MAX_JOBS || m.n_tp < 0 || m.n_tp > 2 * MULTI_MAX_JOBS)
        return hipErrorInvalidValue;
    int total = 0;
    const int lds_bytes = ring_bytes(1) + (grouped ? tbl_bytes(1) : 0);   // group-wise: the scale tables behind the ring
    for (int j = 0; j < MULTI_MAX_JOBS; ++j) {
        if (j < m.n_jobs) {
            GemmArgs &a = m.job[j].a;
            if ((a.gsz > 0) != grouped || a.tp_blocks) return hipErrorInvalidValue;
            if (grouped && m.job[j].mode == MODE_DDS) return hipErrorInvalidValue;
            a.patch_t = a.tiles_t < 4 ? a.tiles_t : 4;
            total += gemm_multi_wgs(a);
        } else {
            m.job[j] = m.job[m.n_jobs > 0 ? m.n_jobs - 1 : 0];
        }
        m.job[j].wg_end = total;
    }
    if ((m.aux_begin & 7) || (m.aux_wgs & 7) || m.aux_begin < 0 || m.aux_begin > total) return hipErrorInvalidValue;
    if (total + m.aux_wgs == 0) return hipSuccess;
    const int mode0 = m.n_jobs > 0 ? m.job[0].mode : MODE_DX;
    if (grouped) {
        for (int j = 0; j < m.n_jobs; ++j)
            if (m.job[j].mode != mode0) return hipErrorInvalidValue;
        if (mode0 == MODE_Y && m.aux_wgs != 0) return hipErrorInvalidValue;
    }
    const int kid = mode0 == MODE_Y ? KID_GEMM_MULTI_Y : (mode0 == MODE_DDS ? KID_GEMM_MULTI_DDS : KID_GEMM_MULTI_DX);
    trace_before(kid, stream);
    const dim3 grid(total + m.aux_wgs);
    hipError_t e;
    if (!grouped)
        e = bits == 4 ? launch_multi<4, -1>(grid, lds_bytes, m, stream) : launch_multi<3, -1>(grid, lds_bytes, m, stream);
    else if (mode0 == MODE_Y)
        e = bits == 4 ? launch_multi<4, MODE_Y>(grid, lds_bytes, m, stream) : launch_multi<3, MODE_Y>(grid, lds_bytes, m, stream);
    else
        e = bits == 4 ? launch_multi<4, MODE_DX>(grid, lds_bytes, m, stream) : launch_multi<3, MODE_DX>(grid, lds_bytes, m, stream);
    trace_after(kid, stream);
    return e;
}

hipError_t launch_gemm_bwd_pair(int bits, const GemmArgs &dds_in, const GemmArgs &dx_in, hipStream_t stream)
{
    GemmArgs a_dds = dds_in, a_dx = dx_in;
    if (a_dds.gsz > 0 || a_dx.gsz > 0 || a_dds.tp_blocks || a_dx.tp_blocks || a_dds.tiles_t != a_dx.tiles_t)
        return hipErrorInvalidValue;
    a_dds.patch_t = a_dx.patch_t = a_dds.tiles_t < 4 ? a_dds.tiles_t : 4;
    trace_before(KID_GEMM_BWD, stream);
    const hipError_t e = bits == 4 ? launch_pair<4>(a_dds, a_dx, stream) : launch_pair<3>(a_dds, a_dx, stream);
    trace_after(KID_GEMM_BWD, stream);
    return e;
}

}  // namespace peqa

// Scale gradient of group-wise layers by the second route of the chain rule on Eq. 2:
//
//   dW[i,k]   = sum_t dY[t,i] X[t,k]                         (plain bf16 contraction over tokens)
//   d_ds[i,g] = sum_{k in g} dW[i,k] (Q[i,k] - z[i,g])       (codes applied once, in the epilogue)
//
// The first route (contract X with the codes group by group, then reduce over tokens) restarts its
// accumulators at every scale group: with 128 features per group a workgroup gets four steps of
// contraction between a ring fill and an epilogue.  Here the contraction runs over all tokens without a
// restart, no code is unpacked inside the loop, and the groups only appear in the epilogue.
//
// Both operands are needed with the token index contiguous, so X and dY are first copied (transpose_pad_kernel) into
// arrays of 32-token steps, Tp = T rounded up to 64, zero-filled, in which 16 rows (features or channels) of a step are
// one KB: exactly a matrix operand, lane by lane (transpose_pad_tile).  A tile's rows of a step are contiguous.
//
// dw_kernel: one workgroup = a 128 (features) x 256 (channels) tile of dW by 4 waves of 128 x 64 accumulators each
// (8 x 4 MFMA 16x16x32 tiles in 128 AGPRs), two workgroups per compute unit, of which one runs while the other waits at a
// barrier, fills its ring or is in its epilogue.  The features are shared by the four waves: global -> LDS by DMA into a
// ring of 6 stages of 8 KB, and from there into registers a step ahead.  The channels are the wave's own: straight from
// memory into registers, two steps ahead.  So LDS moves 80 KB per step of
// two workgroups (about 640 of 1024 cycles of matrix instructions), where one workgroup of 256 x 256 with both operands
// in LDS moved 128 KB and had nothing to run at its barrier: at T = 2048 the launch of a 13B block's
// layers (3 bits, groups of 128) took 1150-1230 us in that form and takes 1035, a 13824 x 5120 layer 316 and 253 us with
// the copies, 11008 x 4096 with groups of 64 at T = 500 72 and 61 us.  (Patches of 4 x 16 or 16 x 4 tiles, the DMAs in the
// middle of the step, feature reads spread over the whole step: within 1 %.)
// The epilogue takes each lane's codes from a copy of the tile's packed words that the first DMAs brought into LDS, at
// word positions and shifts worked out once per lane, forms sum dW Q - z sum dW over each chunk of 64 features (every
// group is a whole number of them) with two shuffles, and writes pc[i, chunk]; chunk_reduce_kernel adds the chunks of
// every group in order.  Groups of 64 and 128 lie within a tile and are complete there: they go to d_ds directly (without
// that launch: step of 11008 x 4096, groups of 64, T = 500 197.5 -> 195.6 us, of a 13B block 3484 -> 3467).
#include <stddef.h>

#include "peqa_dw_tile.h"

namespace peqa {

namespace {

template <int BITS>
__global__ __launch_bounds__(256, 2) void dw_kernel(DwArgs a)
{
    extern __shared__ __align__(16) uint8_t lds[];
    dw_tile<BITS>(a, (int)blockIdx.x, lds);
}

// The token contractions of several layers in one launch: the tiles of job 0 first, then job 1's, ...  One layer's
// tiles alone often fill the machine a fraction over a whole number of times (800 tiles in 512 places for a
// 5120 x 5120 layer); together only the last round of the launch is partly filled.
template <int BITS>
__global__ __launch_bounds__(256, 2) void dw_multi_kernel(DwMultiArgs m)
{
    extern __shared__ __align__(16) uint8_t lds[];
    const int b = (int)blockIdx.x;
    int j = 0, wg0 = 0;
#pragma unroll
    for (int i = 0; i < DW_MAX_JOBS - 1; ++i) {
        const int e = m.wg_end[i];
        if (b >= e) { j = i + 1; wg0 = e; }
    }
    const DwArgs a = kernarg_load<DwArgs>((uint32_t)(j * sizeof(DwArgs)));
    dw_tile<BITS>(a, b - wg0, lds);
}

// The step-major transposed copies (peqa_device.h) of both operands, X [T, K] and dY [T, N], in 64 x 64 tiles and one grid dimension (a
// second one ends at 65536).  One launch, 1.4 us less than two in a step of 193.  Bound by a wave's chain of instructions up to
// two tiles per unit, where four waves share one (transpose_pad_quarter); then workgroups of one wave up to 24 tiles per unit, of four
// past that (as group_prep_kernel); us, four / one: 1664 x 4096, T = 2352 (3330 tiles) 10.8 / 10.6, 11008 x 4096, T = 2048 (7552) 20.5 / 20.4,
// 8192 x 22016 (15104) 38.7 / 41.7.
__global__ __launch_bounds__(256) void transpose_pad_kernel(const uint16_t *__restrict__ X, int K, uint16_t *__restrict__ xt,
                                                             const uint16_t *__restrict__ dY, int N,
                                                             uint16_t *__restrict__ dyt, int T, int per_wg)
{
    extern __shared__ __align__(16) uint8_t lds[];
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int bts = (T + 63) >> 6, of_x = bts * (K >> 6);
    int b = per_wg == 4 ? 4 * (int)blockIdx.x + wave : (int)blockIdx.x;
    if (b >= of_x + bts * (N >> 6)) return;
    const bool x = b < of_x;
    b -= x ? 0 : of_x;
    const CopyTile c = copy_tile(b, bts, (x ? K : N) >> 6, per_wg);
    if (per_wg)
        transpose_pad_tile(x ? X : dY, T, x ? K : N, x ? xt : dyt, c.bt, c.bc, reinterpret_cast<u32x4 *>(lds + wave * TRANSPOSE_LDS));
    else
        transpose_pad_quarter(x ? X : dY, T, x ? K : N, x ? xt : dyt, c.bt, c.bc, wave);
}

// d_ds[i, g] = sum of pc[i, chunk] over the gsz / 64 chunks of group g, in order.
__global__ __launch_bounds__(256) void chunk_reduce_kernel(const float *__restrict__ pc, size_t n, int per,
                                                            float *__restrict__ d_ds)
{
    const size_t j = (size_t)blockIdx.x * 256 + threadIdx.x;   // = i * G + g; the chunks of j are contiguous
    if (j >= n) return;
    float s = 0.f;
    for (int e = 0; e < per; ++e) s += pc[j * per + e];
    d_ds[j] = s;
}

// chunk_reduce_kernel for the jobs of a dw_multi launch: blockIdx.y = job.
__global__ __launch_bounds__(256) void chunk_reduce_multi_kernel(DwMultiArgs m)
{
    const DwArgs a = kernarg_load<DwArgs>((uint32_t)(blockIdx.y * sizeof(DwArgs)));
    float *d_ds = m.d_ds[0];
#pragma unroll
    for (int i = 1; i < DW_MAX_JOBS; ++i)
        if ((int)blockIdx.y == i) d_ds = m.d_ds[i];
    if (dw_whole_groups(a.gsz)) return;                    // complete
    const size_t n = (size_t)a.N * a.G;
    const int per = a.gsz >> 6;
    const size_t j = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= n) return;
    float s = 0.f;
    for (int e = 0; e < per; ++e) s += global_load<float>(a.pc + j * per + e);
    global_store(d_ds + j, s);
}

constexpr int kMaxDev = 64;
bool g_attr_done[2][kMaxDev];
bool g_attr_done_multi[2][kMaxDev];

}  // namespace

int copies_per_wg(int tiles) { return tiles <= 2 * compute_units() ? 0 : tiles <= 24 * compute_units() ? 1 : 4; }

hipError_t launch_transpose_pad(const uint16_t *X, int K, uint16_t *xt, const uint16_t *dY, int N, uint16_t *dyt, int T,
                                hipStream_t stream)
{
    const int tiles = (T + 63) / 64 * ((K + N) / 64), per_wg = copies_per_wg(tiles);
    trace_before(KID_TRANSPOSE, stream);
    hipLaunchKernelGGL(transpose_pad_kernel, dim3(copies_wgs(tiles)), dim3(per_wg == 1 ? 64 : 256), per_wg * TRANSPOSE_LDS, stream, X, K, xt, dY, N,
                       dyt, T, per_wg);
    trace_after(KID_TRANSPOSE, stream);
    return hipGetLastError();
}

hipError_t launch_dw(int bits, const DwArgs &a_in, hipStream_t stream)
{
    if (!dw_args_ok(a_in)) return hipErrorInvalidValue;
    DwArgs a = a_in;
    a.strip_magic = 0xFFFFFFFFu / (8u * (uint32_t)a.tiles_c);
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDev) return hipErrorInvalidDevice;
    auto kern = bits == 4 ? dw_kernel<4> : dw_kernel<3>;
    bool &done = g_attr_done[bits == 4][dev];
    if (!done) {
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, DW_LDS);
        if (e != hipSuccess) return e;
        done = true;
    }
    trace_before(KID_GEMM_DW, stream);
    hipLaunchKernelGGL(kern, dim3(dw_wgs(a)), dim3(256), DW_LDS, stream, a);
    trace_after(KID_GEMM_DW, stream);
    return hipGetLastError();
}

bool dw_args_ok(const DwArgs &a)
{
    if (a.K % 128 != 0 || a.tiles_f != a.K / 128 || a.tiles_c != (a.N + 255) / 256 || a.N % 128 != 0 || a.Tp % 64 != 0 ||
        a.Tp < 64 || a.gsz % 64 != 0 || a.K % a.gsz != 0)
        return false;
    return (uint64_t)(a.K > a.N ? a.K : a.N) * 64u < ((uint64_t)1 << 32);   // 32-bit DMA offsets
}

hipError_t launch_dw_multi(int bits, DwMultiArgs &m, hipStream_t stream)
{
    if (m.n_jobs < 1 || m.n_jobs > DW_MAX_JOBS) return hipErrorInvalidValue;
    int total = 0;
    for (int j = 0; j < DW_MAX_JOBS; ++j) {
        if (j < m.n_jobs) {
            DwArgs &a = m.job[j];
            if (!dw_args_ok(a)) return hipErrorInvalidValue;
            a.strip_magic = 0xFFFFFFFFu / (8u * (uint32_t)a.tiles_c);
            total += dw_wgs(a);
        } else {
            m.job[j] = m.job[m.n_jobs - 1];
            m.d_ds[j] = m.d_ds[m.n_jobs - 1];
        }
        m.wg_end[j] = total;
    }
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDev) return hipErrorInvalidDevice;
    auto kern = bits == 4 ? dw_multi_kernel<4> : dw_multi_kernel<3>;
    bool &done = g_attr_done_multi[bits == 4][dev];
    if (!done) {
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, DW_LDS);
        if (e != hipSuccess) return e;
        done = true;
    }
    trace_before(KID_GEMM_DW, stream);
    hipLaunchKernelGGL(kern, dim3(total), dim3(256), DW_LDS, stream, m);
    trace_after(KID_GEMM_DW, stream);
    return hipGetLastError();
}

hipError_t launch_chunk_reduce_multi(const DwMultiArgs &m, hipStream_t stream)
{
    size_t nmax = 0;
    for (int j = 0; j < m.n_jobs; ++j) {
        const size_t n = dw_whole_groups(m.job[j].gsz) ? 0 : (size_t)m.job[j].N * m.job[j].G;
        nmax = n > nmax ? n : nmax;
    }
    if (nmax == 0) return hipSuccess;
    trace_before(KID_REDUCE, stream);
    hipLaunchKernelGGL(chunk_reduce_multi_kernel, dim3((unsigned)((nmax + 255) / 256), m.n_jobs), dim3(256), 0, stream, m);
    trace_after(KID_REDUCE, stream);
    return hipGetLastError();
}

hipError_t launch_chunk_reduce(const float *pc, size_t n, int per, float *d_ds, hipStream_t stream)
{
    trace_before(KID_REDUCE, stream);
    hipLaunchKernelGGL(chunk_reduce_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, pc, n, per, d_ds);
    trace_after(KID_REDUCE, stream);
    return hipGetLastError();
}

}  // namespace peqa

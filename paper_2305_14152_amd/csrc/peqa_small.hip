// Bandwidth-bound helper kernels around the MFMA contractions: row sums of X, the scaled
// copy of dY, the fixed-order reduction of scale-gradient partials, and the AdamW step.
#include <stddef.h>

#include "peqa_device.h"
#include "peqa_kernels.h"

namespace peqa {

namespace {

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// rs[t, h] = sum of X[t, k] over contraction half h (k < ksplit, k >= ksplit), fp32.
// One wave per token row; 16-byte loads.
__device__ __forceinline__ void rowsum_rows(const uint16_t *__restrict__ X, int T, int K, int ksplit, float *__restrict__ rs,
                                            int blk)
{
    const int lane = threadIdx.x & 63, t = blk * 4 + (threadIdx.x >> 6);
    if (t >= T) return;
    const u32x4 *row = reinterpret_cast<const u32x4 *>(X + (size_t)t * K);
    float s[2] = {0.f, 0.f};
    const int split8 = ksplit >> 3;
    const int n8 = K >> 3;
    // Bound by latency where there are few rows: eight 16-byte loads of a lane in flight while more than four are left, then four; chunks
    // past the row's end re-read its first chunk and add nothing.  The inputs of a 7B block, T = 333: 7.7 us with four throughout,
    // 6.5 so.
    auto add = [&](int k8, auto n_c) __attribute__((always_inline)) {
        constexpr int NL = decltype(n_c)::value;
        u32x4 v[NL];
#pragma unroll
        for (int u = 0; u < NL; ++u) v[u] = row[k8 + 64 * u < n8 ? k8 + 64 * u : 0];
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            float p = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) p += bf16_lo(v[u][i]) + bf16_hi(v[u][i]);
            const int kk = k8 + 64 * u;
            s[0] += kk < split8 ? p : 0.f;
            s[1] += kk >= split8 && kk < n8 ? p : 0.f;
        }
    };
    int at = 0;                                            // (uniform)
    for (; at + 256 < n8; at += 512) add(at + lane, std::integral_constant<int, 8>{});
    if (at < n8) add(at + lane, std::integral_constant<int, 4>{});
    s[0] = wave_sum(s[0]);
    s[1] = wave_sum(s[1]);
    if (lane == 0) { rs[2 * t] = s[0]; rs[2 * t + 1] = s[1]; }
}

__global__ __launch_bounds__(256) void rowsum_kernel(const uint16_t *__restrict__ X, int T, int K, int ksplit,
                                                      float *__restrict__ rs)
{
    rowsum_rows(X, T, K, ksplit, rs, (int)blockIdx.x);
}

// rowsum_kernel's work for several inputs of T rows each: blockIdx.y selects the input.
__global__ __launch_bounds__(256) void rowsum_multi_kernel(RowsumMulti a)
{
    const int y = blockIdx.y;
    const uint16_t *X = a.X[0];
    float *rs = a.rs[0];
    int K = a.K[0];
#pragma unroll
    for (int i = 1; i < ROWSUM_MAX; ++i)
        if (y == i) { X = a.X[i]; rs = a.rs[i]; K = a.K[i]; }
    rowsum_rows(X, a.T, K, K / 2, rs, (int)blockIdx.x);
}

// rsg[t, g] = sum of X[t, k] over scale group g (gsz features, a multiple of 64), fp32.
// One wave per token row: 8 lanes sum each run of 64 features, the run sums meet in LDS,
// and every group adds its gsz / 64 runs in order.
__global__ __launch_bounds__(256) void rowsum_groups_kernel(const uint16_t *__restrict__ X, int T, int K, int gsz,
                                                             float *__restrict__ rsg)
{
    extern __shared__ float runsum[];                      // [4 waves][K / 64]
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, t = blockIdx.x * 4 + w;
    const int nruns = K >> 6;
    float *mine = runsum + w * nruns;
    if (t < T) {
        const u32x4 *row = reinterpret_cast<const u32x4 *>(X + (size_t)t * K);
        for (int k8 = lane; k8 < (K >> 3); k8 += 64) {    // K % 128 == 0: whole 8-lane segments
            const u32x4 v = row[k8];
            float p = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) p += bf16_lo(v[i]) + bf16_hi(v[i]);
#pragma unroll
            for (int o = 4; o >= 1; o >>= 1) p += __shfl_xor(p, o);
            if ((lane & 7) == 0) mine[k8 >> 3] = p;
        }
    }
    __syncthreads();
    if (t < T) {
        const int per = gsz >> 6, G = K / gsz;
        for (int g = lane; g < G; g += 64) {
            float r = 0.f;
            for (int b = 0; b < per; ++b) r += mine[g * per + b];
            rsg[(size_t)t * G + g] = r;
        }
    }
}

// The per-group table from which the grouped contractions take their scales, with s = (s0 + ds)[n, g] and z = (z0 + dz)[n, g]:
//   sb[g][n] = (s, -s (16 + z)): the weights are scaled in the loop (forward, dX)
// by workgroups of GT_CH channels x all groups, through LDS: memory has a channel's groups next to each
// other and the table a group's channels, so entry by entry every 8-byte write is a transaction of its own (25 us for
// the four tables of a 13B block); here the reads run along the groups, four entries a thread, and the writes along the channels,
// 128 bytes per group.  `lds`: 2 x GT_CH x (G | 1) floats: with rows of an odd length a group's channels are in different banks.
// Bound by the latency of the one load and the one store of a workgroup, and by the workgroups that a launch hands out: with an
// entry at a time, and a grid as long as the largest layer for every layer (half of its workgroups had nothing to do), the four
// tables of a 13B block took 17 us.
constexpr int GT_CH = 16;
constexpr int gt_tile_bytes(int G) { return 2 * GT_CH * (G | 1) * (int)sizeof(float); }
__device__ __forceinline__ void group_table_tile(const float *__restrict__ s0, const float *__restrict__ ds,
                                                 const uint8_t *__restrict__ z0, const float *__restrict__ dz, int N, int G,
                                                 float *__restrict__ sb, int n0, float *lds)
{
    const int row = G | 1;
    float *s_l = lds, *z_l = lds + GT_CH * row;
    const size_t base = (size_t)n0 * G;                    // a multiple of GT_CH: the quads are aligned for any G
    for (int e = 4 * threadIdx.x; e < GT_CH * G; e += 4 * 256) {
        f32x4 s = *reinterpret_cast<const f32x4 *>(s0 + base + e);
        const uint32_t z = *reinterpret_cast<const uint32_t *>(z0 + base + e);
        if (ds) s += *reinterpret_cast<const f32x4 *>(ds + base + e);
        f32x4 d = {0.f, 0.f, 0.f, 0.f};
        if (dz) d = *reinterpret_cast<const f32x4 *>(dz + base + e);
        int nl = e / G, g = e - nl * G;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            s_l[nl * row + g] = s[u];
            z_l[nl * row + g] = kCodeOffset + (float)((z >> (8 * u)) & 0xFFu) + d[u];
            if (++g == G) { g = 0; ++nl; }
        }
    }
    __syncthreads();
    const int nl = threadIdx.x % GT_CH, n = n0 + nl;
    for (int g = threadIdx.x / GT_CH; g < G; g += 256 / GT_CH) {
        const float s = s_l[nl * row + g], zoff = z_l[nl * row + g];
        f32x2 o;
        o[0] = s;
        o[1] = -s * zoff;
        *reinterpret_cast<f32x2 *>(sb + ((size_t)g * N + n) * 2) = o;
    }
}

// The same by workgroups of GT_CH channels x GT_PART groups, numbered along the groups first: where all groups do not fit in LDS.  (Entry
// by entry, as before, 161 us for the seven tables of a block of d = 8064, f = 25600 in groups of 64, 57 so; forward at T = 52 332 -> 230.)
constexpr int GT_PART = 128;
__device__ __forceinline__ void group_table_part(const float *__restrict__ s0, const float *__restrict__ ds,
                                                 const uint8_t *__restrict__ z0, const float *__restrict__ dz, int N, int G,
                                                 float *__restrict__ sb, int wg, float *lds)
{
    const int parts = (G + GT_PART - 1) / GT_PART, n0 = wg / parts * GT_CH, g0 = wg % parts * GT_PART;
    const int gn = min(GT_PART, G - g0);
    constexpr int row = GT_PART | 1;
    float *s_l = lds, *z_l = lds + GT_CH * row;
#pragma unroll
    for (int e = threadIdx.x; e < GT_CH * GT_PART; e += 256) {
        const int nl = e / GT_PART, g = e % GT_PART;
        const size_t at = (size_t)(n0 + nl) * G + g0 + min(g, gn - 1);     // past the end: the last one again, not written
        s_l[nl * row + g] = ds ? s0[at] + ds[at] : s0[at];
        z_l[nl * row + g] = kCodeOffset + (float)z0[at] + (dz ? dz[at] : 0.f);
    }
    __syncthreads();
    const int nl = threadIdx.x % GT_CH, n = n0 + nl;
    for (int g = threadIdx.x / GT_CH; g < gn; g += 256 / GT_CH) {
        const float s = s_l[nl * row + g], zoff = z_l[nl * row + g];
        f32x2 o;
        o[0] = s;
        o[1] = -s * zoff;
        *reinterpret_cast<f32x2 *>(sb + ((size_t)(g0 + g) * N + n) * 2) = o;
    }
}

// A workgroup's share of a layer's table: whole rows of groups, or runs of GT_PART.
__device__ __forceinline__ void group_table_share(const float *__restrict__ s0, const float *__restrict__ ds,
                                                  const uint8_t *__restrict__ z0, const float *__restrict__ dz, int N, int G,
                                                  float *__restrict__ sb, int wg, bool whole_rows, float *lds)
{
    if (whole_rows) group_table_tile(s0, ds, z0, dz, N, G, sb, wg * GT_CH, lds);
    else group_table_part(s0, ds, z0, dz, N, G, sb, wg, lds);
}

// The table of one layer.  (As group_prep_kernel's only table it waits for the descriptors of eight: 512 x 256 in groups of 128 3.4 us,
// 2.7 so, of a training step of 27.)
__global__ __launch_bounds__(256) void group_table_kernel(const float *__restrict__ s0, const float *__restrict__ ds,
                                                           const uint8_t *__restrict__ z0, const float *__restrict__ dz, int N, int G,
                                                           float *__restrict__ sb, int whole_rows)
{
    extern __shared__ __align__(16) float gt_lds[];
    group_table_share(s0, ds, z0, dz, N, G, sb, (int)blockIdx.x, whole_rows != 0, gt_lds);
}

// Tables of group-wise layers and, for a backward, transposed copies (GroupPrep): the tables' workgroups first, then those of the copies, which
// take a 64 x 64 tile together, or one in each of one wave or four.  One launch where there were two, of 3 us and more each.
__global__ __launch_bounds__(256) void group_prep_kernel(GroupPrep a)
{
    extern __shared__ __align__(16) float gt_lds[];
    int b = (int)blockIdx.x;
    if (b < a.table_end[GT_MAX - 1]) {
        const float *s0 = a.table.s0[0], *ds = a.table.ds[0];
        const uint8_t *z0 = a.table.z0[0];
        float *sb = a.table.sb[0];
        int N = a.table.N[0], G = a.table.G[0], b0 = 0;
#pragma unroll
        for (int i = 1; i < GT_MAX; ++i)
            if (b >= a.table_end[i - 1]) {
                s0 = a.table.s0[i]; ds = a.table.ds[i]; z0 = a.table.z0[i]; sb = a.table.sb[i]; N = a.table.N[i]; G = a.table.G[i];
                b0 = a.table_end[i - 1];
            }
        group_table_share(s0, ds, z0, a.dz, N, G, sb, b - b0, a.whole_rows != 0, gt_lds);
        return;
    }
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    b -= a.table_end[GT_MAX - 1];
    if (a.copies_per_wg == 1 && wave > 0) return;
    if (a.copies_per_wg == 4) b = 4 * b + wave;
    if (b >= kernarg_load<int>((uint32_t)(offsetof(GroupPrep, tp) + (a.n_tp - 1) * sizeof(TransposeJob) + offsetof(TransposeJob, tile_end)))) return;
    int j = 0, b0 = 0;
    for (int i = 0; i + 1 < a.n_tp; ++i) {
        const int e = kernarg_load<int>((uint32_t)(offsetof(GroupPrep, tp) + i * sizeof(TransposeJob) + offsetof(TransposeJob, tile_end)));
        if (b >= e) { j = i + 1; b0 = e; }
    }
    const TransposeJob J = kernarg_load<TransposeJob>((uint32_t)(offsetof(GroupPrep, tp) + j * sizeof(TransposeJob)));
    const CopyTile c = copy_tile(b - b0, J.Tp >> 6, J.C >> 6, a.copies_per_wg);
    if (a.copies_per_wg) transpose_pad_tile(J.src, J.T, J.C, J.dst, c.bt, c.bc, reinterpret_cast<u32x4 *>(gt_lds) + wave * (TRANSPOSE_LDS / 16));
    else transpose_pad_quarter(J.src, J.T, J.C, J.dst, c.bt, c.bc, wave);
}

// scale_dy_rows (peqa_device.h) for every block of SDY_ROWS token rows.  Workgroups past the last row block do
// independent jobs of the same backward: the row sums of X for the scale gradient that follows (rs = NULL: none), or the
// fixed-order sum of the scale-gradient partials (n_red = 0: none).  A launch saved is 3 us of host time and 1 to 3 us
// of the GPU's: a 256 x 256 layer's step at T = 64, all of it launches, went from 36.2 to 31.6 us with the row sums here.
constexpr int SDY_ROWS = 4;
__global__ __launch_bounds__(256) void scale_dy_kernel(const uint16_t *__restrict__ dY, const float *__restrict__ s0,
                                                        const float *__restrict__ ds, const uint8_t *__restrict__ z0,
                                                        const float *__restrict__ dz, int T, int N,
                                                        uint16_t *__restrict__ dYs, float *__restrict__ crow,
                                                        const float *__restrict__ partial, int ntiles, size_t n_red,
                                                        float *__restrict__ red_out, const uint16_t *__restrict__ X, int K,
                                                        float *__restrict__ rs)
{
    __shared__ float red[SDY_ROWS * 4];
    const int row_blocks = (T + SDY_ROWS - 1) / SDY_ROWS;
    if ((int)blockIdx.x >= row_blocks) {
        const int past = (int)blockIdx.x - row_blocks, sum_blocks = rs ? (T + 3) / 4 : 0;
        if (past < sum_blocks) rowsum_rows(X, T, K, K / 2, rs, past);
        else reduce_partials_at(partial, ntiles, n_red, (size_t)(past - sum_blocks) * 256 + threadIdx.x, red_out);
        return;
    }
    scale_dy_rows<SDY_ROWS>(dY, s0, ds, z0, dz, T, N, dYs, crow, (int)blockIdx.x, red);
}

// Scale gradient from the product P[t,i] = sum_k X[t,k] (Q[i,k] - z0[i]) that the forward kept:
// partial[slice, i] = sum of dY[t,i] P[t,i] over the KEPT_ROWS token rows of the slice.  A workgroup
// takes 256 channels (4 per lane) of one slice; wave w adds rows w, w+4, ... in order and the four
// wave sums meet in LDS in a fixed order.
__global__ __launch_bounds__(256) void dds_kept_kernel(const uint16_t *__restrict__ dY, const float *__restrict__ P,
                                                        int T, int N, float *__restrict__ partial)
{
    __shared__ f32x4 part[4][64];
    const int q = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int col = blockIdx.y * 256 + 4 * q;
    const int tbeg = blockIdx.x * KEPT_ROWS;
    const int nrows = min(KEPT_ROWS, T - tbeg);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    if (col < N) {
        const size_t base = (size_t)tbeg * N + col;
#pragma unroll 4
        for (int r = w; r < nrows; r += 4) {
            const u32x2 d = *reinterpret_cast<const u32x2 *>(dY + base + (size_t)r * N);
            const f32x4 p = *reinterpret_cast<const f32x4 *>(P + base + (size_t)r * N);
            acc[0] += bf16_lo(d[0]) * p[0];
            acc[1] += bf16_hi(d[0]) * p[1];
            acc[2] += bf16_lo(d[1]) * p[2];
            acc[3] += bf16_hi(d[1]) * p[3];
        }
    }
    part[w][q] = acc;
    __syncthreads();
    if (w == 0 && col < N) {
        const f32x4 s = ((part[0][q] + part[1][q]) + part[2][q]) + part[3][q];
        *reinterpret_cast<f32x4 *>(partial + (size_t)blockIdx.x * N + col) = s;
    }
}

// Zero-point gradient of a per-channel layer, first stage: partial[slice, i] = sum over the slice's KEPT_ROWS token rows
// of dY[t,i] * (rs[t,0] + rs[t,1]).  Bound by the one pass over dY: a wave loads its 16 rows eight at a time, the row sums
// come by scalar loads.  (dz_partial_kernel, made for many groups, spent seven eighths of its sums on groups that are not
// there and 10 us on dY of 2048 x 4096.)
__global__ __launch_bounds__(256) void dz_rows_kernel(const uint16_t *__restrict__ dY, const float *__restrict__ rs, int T,
                                                       int N, float *__restrict__ partial)
{
    __shared__ f32x4 part[4][64];
    const int q = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = blockIdx.y * 256 + 4 * q;
    const int tbeg = blockIdx.x * KEPT_ROWS;
    const int nrows = min(KEPT_ROWS, T - tbeg);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    if (col < N) {
        const uint16_t *base = dY + (size_t)tbeg * N + col;
#pragma unroll 8
        for (int r = w; r < nrows; r += 4) {
            const u32x2 d = *reinterpret_cast<const u32x2 *>(base + (size_t)r * N);
            const float R = rs[2 * (tbeg + r)] + rs[2 * (tbeg + r) + 1];
            acc[0] += bf16_lo(d[0]) * R;
            acc[1] += bf16_hi(d[0]) * R;
            acc[2] += bf16_lo(d[1]) * R;
            acc[3] += bf16_hi(d[1]) * R;
        }
    }
    part[w][q] = acc;
    __syncthreads();
    if (w == 0 && col < N) {
        const f32x4 s = ((part[0][q] + part[1][q]) + part[2][q]) + part[3][q];
        *reinterpret_cast<f32x4 *>(partial + (size_t)blockIdx.x * N + col) = s;
    }
}

// Zero-point gradient, first stage (Appendix K trains zero-points too; z enters Eq. 2 only through -s z, so
// d_dz[i,g] = -s[i,g] * sum_t dY[t,i] R[t,g] with R[t,g] the sum of X[t,k] over scale group g):
// partial[slice, i, g] = sum over the slice's KEPT_ROWS token rows of dY[t,i] * R[t,g].
// A workgroup takes 256 channels (4 per lane) of one slice and walks the groups 8 at a time; wave w
// adds rows w, w+4, ... in order; the four wave sums meet in LDS in a fixed order.
__global__ __launch_bounds__(256) void dz_partial_kernel(const uint16_t *__restrict__ dY, const float *__restrict__ rsg,
                                                          int T, int N, int G, float *__restrict__ partial)
{
    __shared__ float part[4][32][64];                        // [wave][channel-in-lane * 8 + group][lane]
    const int q = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = blockIdx.y * 256 + 4 * q;
    const int tbeg = blockIdx.x * KEPT_ROWS;
    const int nrows = min(KEPT_ROWS, T - tbeg);
    const bool on = col < N;
    for (int gc = 0; gc < G; gc += 8) {
        float acc[4][8];
#pragma unroll
        for (int cc = 0; cc < 4; ++cc)
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[cc][j] = 0.f;
        if (on) {
            for (int r = w; r < nrows; r += 4) {
                const size_t t = (size_t)(tbeg + r);
                const u32x2 d = *reinterpret_cast<const u32x2 *>(dY + t * N + col);
                const float dv[4] = {bf16_lo(d[0]), bf16_hi(d[0]), bf16_lo(d[1]), bf16_hi(d[1])};
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const float R = rsg[t * G + min(gc + j, G - 1)];   // groups past G are dropped at the store
#pragma unroll
                    for (int cc = 0; cc < 4; ++cc) acc[cc][j] += dv[cc] * R;
                }
            }
        }
        __syncthreads();                                     // the previous chunk's sums have been read
#pragma unroll
        for (int cc = 0; cc < 4; ++cc)
#pragma unroll
            for (int j = 0; j < 8; ++j) part[w][cc * 8 + j][q] = acc[cc][j];
        __syncthreads();
        if (w == 0 && on) {
#pragma unroll
            for (int cc = 0; cc < 4; ++cc)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int e = cc * 8 + j;
                    const float s = ((part[0][e][q] + part[1][e][q]) + part[2][e][q]) + part[3][e][q];
                    if (gc + j < G) partial[((size_t)blockIdx.x * N + col + cc) * G + gc + j] = s;
                }
        }
    }
}

// d_dz[j] = -(s0 + ds)[j] * (partial[0][j] + partial[1][j] + ...) in that order.  Workgroups past those carry the
// independent sum of the same backward's scale-gradient partials (n_red = 0: none).
__global__ __launch_bounds__(256) void dz_finish_kernel(const float *__restrict__ partial, int slices, size_t n,
                                                         const float *__restrict__ s0, const float *__restrict__ ds,
                                                         float *__restrict__ d_dz, const float *__restrict__ red,
                                                         int red_rows, size_t n_red, float *__restrict__ red_out)
{
    const size_t j = (size_t)blockIdx.x * 256 + threadIdx.x, dz_end = (n + 255) / 256 * 256;
    if (j >= dz_end) {
        reduce_partials_at(red, red_rows, n_red, j - dz_end, red_out);
        return;
    }
    if (j >= n) return;
    const float sc = ds ? s0[j] + ds[j] : s0[j];
    d_dz[j] = -sc * partials_sum(partial, slices, n, j);
}

__global__ __launch_bounds__(256) void reduce_partials_kernel(const float *__restrict__ partial, int ntiles, size_t n,
                                                               float *__restrict__ out)
{
    reduce_partials_at(partial, ntiles, n, (size_t)blockIdx.x * 256 + threadIdx.x, out);
}

__global__ __launch_bounds__(256) void adamw_kernel(size_t n, float *__restrict__ ds, const float *__restrict__ g,
                                                     float *__restrict__ m, float *__restrict__ v,
                                                     const float *__restrict__ s0, float lr, float b1, float b2,
                                                     float eps, float wd, float inv_c1, float inv_c2)
{
    const size_t j = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= n) return;
    const float gj = g[j];
    const float mj = b1 * m[j] + (1.f - b1) * gj;
    const float vj = b2 * v[j] + (1.f - b2) * gj * gj;
    m[j] = mj;
    v[j] = vj;
    const float d = ds[j];
    ds[j] = d - lr * ((mj * inv_c1) / (sqrtf(vj * inv_c2) + eps) + wd * (s0[j] + d));
}

// The same update over several parameter vectors laid end to end in one index space.
__global__ __launch_bounds__(256) void adamw_multi_kernel(AdamwMulti a, float lr, float b1, float b2, float eps,
                                                           float wd, float inv_c1, float inv_c2)
{
    const unsigned long long idx = (unsigned long long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= a.end[ADAMW_MAX_TENSORS - 1]) return;
    int t = 0;
#pragma unroll
    for (int i = 0; i < ADAMW_MAX_TENSORS - 1; ++i) t += idx >= a.end[i];
    // selects instead of indexing: the argument block stays in scalar registers
    float *ds = a.ds[0]; const float *g = a.g[0]; float *m = a.m[0]; float *v = a.v[0]; const float *s0 = a.s0[0];
    unsigned long long beg = 0;
#pragma unroll
    for (int i = 1; i < ADAMW_MAX_TENSORS; ++i)
        if (t == i) { ds = a.ds[i]; g = a.g[i]; m = a.m[i]; v = a.v[i]; s0 = a.s0[i]; beg = a.end[i - 1]; }
    const size_t j = (size_t)(idx - beg);
    const float gj = g[j];
    const float mj = b1 * m[j] + (1.f - b1) * gj;
    const float vj = b2 * v[j] + (1.f - b2) * gj * gj;
    m[j] = mj;
    v[j] = vj;
    const float d = ds[j];
    ds[j] = d - lr * ((mj * inv_c1) / (sqrtf(vj * inv_c2) + eps) + wd * (s0[j] + d));
}

}  // namespace

hipError_t launch_adamw_multi(const AdamwMulti &a, float lr, float b1, float b2, float eps, float wd, float inv_c1,
                              float inv_c2, hipStream_t stream)
{
    const unsigned long long total = a.end[ADAMW_MAX_TENSORS - 1];
    trace_before(KID_ADAMW, stream);
    hipLaunchKernelGGL(adamw_multi_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream, a, lr, b1, b2, eps,
                       wd, inv_c1, inv_c2);
    trace_after(KID_ADAMW, stream);
    return hipGetLastError();
}

hipError_t launch_rowsum(const uint16_t *X, int T, int K, int ksplit, float *rs, hipStream_t stream)
{
    trace_before(KID_ROWSUM, stream);
    hipLaunchKernelGGL(rowsum_kernel, dim3((T + 3) / 4), dim3(256), 0, stream, X, T, K, ksplit, rs);
    trace_after(KID_ROWSUM, stream);
    return hipGetLastError();
}

hipError_t launch_rowsum_multi(const RowsumMulti &a, hipStream_t stream)
{
    trace_before(KID_ROWSUM, stream);
    hipLaunchKernelGGL(rowsum_multi_kernel, dim3((a.T + 3) / 4, a.n), dim3(256), 0, stream, a);
    trace_after(KID_ROWSUM, stream);
    return hipGetLastError();
}

hipError_t launch_rowsum_groups(const uint16_t *X, int T, int K, int gsz, float *rsg, hipStream_t stream)
{
    trace_before(KID_ROWSUM, stream);
    hipLaunchKernelGGL(rowsum_groups_kernel, dim3((T + 3) / 4), dim3(256), (size_t)4 * (K >> 6) * sizeof(float), stream,
                       X, T, K, gsz, rsg);
    trace_after(KID_ROWSUM, stream);
    return hipGetLastError();
}

// Groups of a layer up to which workgroups take whole rows of them (49 KB of LDS)
constexpr int GT_TILE_MAX_G = 391;
static_assert(gt_tile_bytes(GT_TILE_MAX_G) <= 49 * 1024, "what a launch may ask for without an attribute");

// workgroups of a layer's table, and their LDS
static int table_wgs(int N, int G, bool whole_rows) { return N / GT_CH * (whole_rows ? 1 : (G + GT_PART - 1) / GT_PART); }
static int table_lds(int G, bool whole_rows) { return gt_tile_bytes(whole_rows ? G : GT_PART); }

hipError_t launch_group_table(const float *s0, const float *ds, const uint8_t *z0, const float *dz, int N, int G,
                              float *sb, hipStream_t stream)
{
    const bool whole_rows = G <= GT_TILE_MAX_G;
    trace_before(KID_GROUP_TABLE, stream);
    hipLaunchKernelGGL(group_table_kernel, dim3(table_wgs(N, G, whole_rows)), dim3(256), table_lds(G, whole_rows), stream, s0, ds, z0, dz,
                       N, G, sb, whole_rows ? 1 : 0);
    trace_after(KID_GROUP_TABLE, stream);
    return hipGetLastError();
}

hipError_t launch_group_prep(GroupPrep &a, hipStream_t stream)
{
    const int n = a.table.n;
    if (n < 0 || n > GT_MAX || a.n_tp < 0 || a.n_tp > 2 * MULTI_MAX_JOBS || (a.dz && n != 1)) return hipErrorInvalidValue;
    int gmax = 0, blocks = 0;
    for (int i = 0; i < n; ++i) gmax = a.table.G[i] > gmax ? a.table.G[i] : gmax;
    a.whole_rows = gmax <= GT_TILE_MAX_G;
    for (int i = 0; i < GT_MAX; ++i) {
        if (i < n) blocks += table_wgs(a.table.N[i], a.table.G[i], a.whole_rows);
        a.table_end[i] = blocks;
    }
    const int tp = a.n_tp > 0 ? a.tp[a.n_tp - 1].tile_end : 0;
    if (blocks + tp == 0) return hipSuccess;
    // Every workgroup of the launch, the tables' among them, has the LDS of the copies' (copies_per_wg): with four tiles five fit a unit, with one as
    // many as there are waves for, which is what counts until the copies outlast the tables.  The launch, us, four tiles / one: blocks of
    // d = 2048 in groups of 256, T = 64 (520 tiles) 7.0 / 5.2, T = 128 (1040) 9.0 / 6.6, T = 333 (3120) 11.3 / 10.1, T = 700 (5720) 17.9 / 16.5,
    // T = 1400 (11440) 33.8 / 35.7; d = 4096 in groups of 128, T = 128 (2056) 13.8 / 12.5, T = 333 (6168) 24.9 / 24.8, T = 1400 (22616)
    // 63.1 / 65.3.
    a.copies_per_wg = copies_per_wg(tp);
    const int tables = n > 0 ? table_lds(gmax, a.whole_rows) : 0, copies = a.copies_per_wg * TRANSPOSE_LDS;
    trace_before(KID_GROUP_TABLE, stream);
    hipLaunchKernelGGL(group_prep_kernel, dim3(blocks + copies_wgs(tp)), dim3(256),
                       tables > copies ? tables : copies, stream, a);
    trace_after(KID_GROUP_TABLE, stream);
    return hipGetLastError();
}

hipError_t launch_group_table_multi(const GroupTableMulti &tables, hipStream_t stream)
{
    GroupPrep a{};
    a.table = tables;
    return launch_group_prep(a, stream);
}

hipError_t launch_scale_dy(const uint16_t *dY, const float *s0, const float *ds, const uint8_t *z0, const float *dz,
                           int T, int N, uint16_t *dYs, float *crow, const float *partial, int ntiles, size_t n_red,
                           float *red_out, const uint16_t *X, int K, float *rs, hipStream_t stream)
{
    trace_before(KID_SCALE_DY, stream);
    const unsigned row_blocks = (unsigned)((T + SDY_ROWS - 1) / SDY_ROWS), sum_blocks = rs ? (unsigned)((T + 3) / 4) : 0u;
    const unsigned blocks = row_blocks + sum_blocks + (unsigned)((n_red + 255) / 256);
    hipLaunchKernelGGL(scale_dy_kernel, dim3(blocks), dim3(256), 0, stream, dY, s0, ds, z0, dz, T, N, dYs, crow, partial,
                       ntiles, n_red, red_out, X, K, rs);
    trace_after(KID_SCALE_DY, stream);
    return hipGetLastError();
}

hipError_t launch_dds_kept(const uint16_t *dY, const float *P, int T, int N, float *partial, hipStream_t stream)
{
    trace_before(KID_DDS_KEPT, stream);
    hipLaunchKernelGGL(dds_kept_kernel, dim3((T + KEPT_ROWS - 1) / KEPT_ROWS, (N + 255) / 256), dim3(256), 0, stream,
                       dY, P, T, N, partial);
    trace_after(KID_DDS_KEPT, stream);
    return hipGetLastError();
}

hipError_t launch_dz_partial(const uint16_t *dY, const float *rsg, int T, int N, int G, float *partial,
                             hipStream_t stream)
{
    trace_before(KID_DZ_PARTIAL, stream);
    hipLaunchKernelGGL(dz_partial_kernel, dim3((T + KEPT_ROWS - 1) / KEPT_ROWS, (N + 255) / 256), dim3(256), 0, stream,
                       dY, rsg, T, N, G, partial);
    trace_after(KID_DZ_PARTIAL, stream);
    return hipGetLastError();
}

hipError_t launch_dz_rows(const uint16_t *dY, const float *rs, int T, int N, float *partial, hipStream_t stream)
{
    trace_before(KID_DZ_PARTIAL, stream);
    hipLaunchKernelGGL(dz_rows_kernel, dim3((T + KEPT_ROWS - 1) / KEPT_ROWS, (N + 255) / 256), dim3(256), 0, stream, dY,
                       rs, T, N, partial);
    trace_after(KID_DZ_PARTIAL, stream);
    return hipGetLastError();
}

hipError_t launch_dz_finish(const float *partial, int slices, size_t n, const float *s0, const float *ds, float *d_dz,
                            const float *red, int red_rows, size_t n_red, float *red_out, hipStream_t stream)
{
    trace_before(KID_DZ_FINISH, stream);
    hipLaunchKernelGGL(dz_finish_kernel, dim3((unsigned)((n + 255) / 256 + (n_red + 255) / 256)), dim3(256), 0, stream,
                       partial, slices, n, s0, ds, d_dz, red, red_rows, n_red, red_out);
    trace_after(KID_DZ_FINISH, stream);
    return hipGetLastError();
}

hipError_t launch_reduce_partials(const float *partial, int ntiles, size_t n, float *out, hipStream_t stream)
{
    trace_before(KID_REDUCE, stream);
    hipLaunchKernelGGL(reduce_partials_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, partial,
                       ntiles, n, out);
    trace_after(KID_REDUCE, stream);
    return hipGetLastError();
}

hipError_t launch_adamw(size_t n, float *ds, const float *g, float *m, float *v, const float *s0, float lr, float b1,
                        float b2, float eps, float wd, float inv_c1, float inv_c2, hipStream_t stream)
{
    trace_before(KID_ADAMW, stream);
    hipLaunchKernelGGL(adamw_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, n, ds, g, m, v, s0, lr,
                       b1, b2, eps, wd, inv_c1, inv_c2);
    trace_after(KID_ADAMW, stream);
    return hipGetLastError();
}

}  // namespace peqa

// Internal launch interface between the C-ABI layer (peqa_api.hip) and the kernel files.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace peqa {

enum { MODE_Y = 0, MODE_DDS = 1, MODE_DX = 2 };

// Test and comparison switches, set through peqa_set_option (peqa_api.hip); the defaults select by launch size.
struct Options {
    int gemm_waves = 0;     // 0 = by launch size, 4 or 8 = that form of the tiled contraction
    int bwd_pair = -1;      // -1 = pair the two contractions of a per-channel backward unless gemm_waves is 8; 0, 1 = never, always
    int grouped_dds = 0;    // 0 = group-wise scale gradient by the contraction over tokens, 1 = over features (older route)
};
Options &options();

// Arguments of the tiled MFMA contraction (peqa_gemm.hip).
struct GemmArgs {
    const uint32_t *packed;   // packed codes of the whole layer
    const uint16_t *A;        // activation operand [T, KC] bf16: X (MODE_Y, MODE_DDS) or scaled dY (MODE_DX)
    int T;                    // tokens
    int KC;                   // contraction length: K (MODE_Y/DDS) or N (MODE_DX)
    int C;                    // output columns:     N (MODE_Y/DDS) or K (MODE_DX)
    int K;                    // input features of the layer (fixes the block stride of `packed`)
    int tiles_c, tiles_t;     // ceil(C/256), ceil(T/(16 rt))
    int rt;                   // row tiles (of 16 tokens) per tile: 4, 6, 7 or 8, gemm_row_tiles(T) or what gemm_plan took instead
    // set by the launches: token tiles per L2 patch (at most 4), reciprocals (div_magic) of the numbers of tiles and of tiles
    // in patch_t rows, 128-deep units of a piece (one more in the first unit_rem pieces)
    int patch_t;
    uint32_t whole_magic, strip_magic;
    int piece_units, unit_rem;
    const float *s0;          // [N]            (MODE_Y)
    const float *ds;          // [N] or NULL    (MODE_Y)
    const uint8_t *z0;        // [N]            (MODE_Y, MODE_DDS)
    const float *dz;          // [N] or NULL: trained zero-point offset, z = z0 + dz (MODE_Y, MODE_DDS; [N, G] if grouped)
    const float *rs;          // [T, 2] sums of X[t, :] over each contraction half (MODE_Y, MODE_DDS)
    const float *crow;        // [T] sum_i A[t,i] (16 + z_i)                      (MODE_DX)
    const uint16_t *dY;       // [T, N] bf16    (MODE_DDS)
    float *partial;           // [tiles_t, N]   (MODE_DDS) per-token-tile column sums
    // MODE_DX, group-wise, four-wave form only: tp_blocks > 0 adds that many workgroups at the end of the grid, which
    // write the step-major transposed copies of X [T, K] and dY [T, N] (transpose_pad_tile) that the token contraction
    // of the same backward reads afterwards: Tp / 64 x K / 64 tiles of X first, then Tp / 64 x N / 64 of dY, four to a workgroup
    int tp_blocks, tp_Tp;
    const uint16_t *tp_X;
    uint16_t *tp_Xt, *tp_dYt;
    uint16_t *out;            // [T, C] bf16    (MODE_Y: Y, MODE_DX: dX)
    // pieces of the contraction per tile (0 or 1: whole).  MODE_Y, MODE_DX: piece p leaves its sums in acc_part [split, T, C]
    // fp32 for launch_split_finish; MODE_DDS (launches of several contractions only): its column sums in row
    // p tiles_t + tile_t of `partial`, and needs no rs.
    int split;
    float *acc_part;
    float *P;                 // [T, N] fp32 or NULL (MODE_Y, per-channel): sum_k X[t,k] (Q[i,k] - z0[i]), kept
    // group-wise layers (gsz > 0; a multiple of 64):
    int N;                    // output channels of the layer
    int gsz, G;               // group size and groups per channel
    const float *sb;          // [G, N, 2] (s0 + ds, -(s0 + ds)(16 + z0))  (MODE_Y, MODE_DX)
                              // rs is then [T, G]: sums of X over every scale group (MODE_DDS),
                              // partial is [tiles_t, N, G] and z0 is [N, G]
};

hipError_t launch_gemm(int bits, int mode, const GemmArgs &a, hipStream_t stream);
// Row tiles (of 16 tokens: 4, 6, 7 or 8) of the tiles that T tokens are dealt to; there are ceil(T / 128) of them in any case.
int gemm_row_tiles(int T);
inline int gemm_tiles_t(int T, int rt) { return (T + 16 * rt - 1) / (16 * rt); }

// Contractions of a launch whose tiles leave the machine idle (few tokens, or a few tiles of a long contraction) are split
// along the contraction: GemmArgs::split pieces per tile.  gemm_plan fills `split` of every job of one launch.
struct SplitJob {
    int tiles_c;              // column tiles
    int KC;                   // contraction length
    size_t out_bytes;         // fp32 bytes of one piece's partial result (T C 4); 0 for MODE_DDS, whose pieces add partial rows
    int split;                // out
};
// other_us: work of other tiles of the same launch, in us of one of two places per unit.
// Returns the row tiles per tile of the launch.  single: the jobs are one contraction that runs by itself (launch_gemm), which
// may take the eight-wave form.  dds: the launch has MODE_DDS jobs, whose partial rows go by gemm_row_tiles(T).
// max_bytes: the most the partial results may take.  cus: compute units.
int gemm_plan(int n, SplitJob *jobs, int T, bool grouped, bool single, bool dds, double other_us, size_t max_bytes, int cus);
// The estimate that it goes by: us of the launch of the jobs as split, in tiles of rt row tiles.
double gemm_form_us(int n, const SplitJob *jobs, int T, int rt, bool grouped, bool single, double other_us, int cus);
// Epilogue of the split MODE_Y / MODE_DX contractions of a launch: adds the pieces in order, then does what the tile's own
// epilogue would have done.  Jobs with split 1 are skipped.  The same launch adds up what else the call has left in parts:
// dst[j] = src[j step_j] + src[j step_j + step] + ... (count of them, in order) for j < n.
constexpr int FINISH_MAX = 8;
struct FinishJob {
    GemmArgs a;
    int mode;
};
struct SumJob {
    const float *src;
    float *dst;
    size_t n, step_j, step;
    int count;
};
struct FinishMulti {
    FinishJob job[FINISH_MAX];             // must stay the first member: indexed in the argument block
    SumJob sum[FINISH_MAX];
    int n, n_sums;
};
hipError_t launch_split_finish(const FinishMulti &f, hipStream_t stream);
// whether a launch of one contraction of that many tiles, or pieces of tiles, takes the four-wave form (two workgroups per compute unit);
// for a huge count: whether the four-wave form is allowed at all (the option gemm_waves = 8 forbids it)
bool gemm_four_waves(int tiles);
// Per-channel layers: the MODE_DDS and the MODE_DX contraction of one backward (arguments as for launch_gemm) as one
// launch of four-wave workgroups (measured faster than two launches at every T).  The dX arguments' input (the scaled dY)
// must be complete before the launch.
hipError_t launch_gemm_bwd_pair(int bits, const GemmArgs &a_dds, const GemmArgs &a_dx, hipStream_t stream);

// Several contractions in ONE launch of four-wave workgroups (gemm_multi_kernel): the tiles of job 0 first, then
// job 1's, ... (the caller orders them by contraction length, longest first, so that the last, partly filled round
// of the launch is made of short tiles).  Per-channel layers only.  Workgroups numbered [aux_begin, aux_begin +
// aux_wgs) do bandwidth-bound side work of the same backward instead of a tile: every one of them walks a share
// of the row blocks of the scale_dy jobs, of the 256-element chunks of the reduce jobs, or of the 64 x 64 tiles of
// the transpose jobs (the operands of the token contraction of group-wise layers).  They sit in the middle
// of the grid, where they start while most compute units still run tiles, so that their memory traffic hides
// behind matrix work.  All job sizes, aux_begin and aux_wgs are multiples of 8 (workgroup id % 8 = XCD throughout).
constexpr int MULTI_MAX_JOBS = 8;
struct MultiJob {
    GemmArgs a;
    int mode;                 // MODE_Y, MODE_DDS or MODE_DX
    int wg_end;               // tile workgroups of this job and all before it (unused entries: the total)
};
// Token rows per row block of the scaling in the auxiliary workgroups of a launch whose tiles have rt row tiles (see scale_dy_rows); without tiles
// launch_gemm_multi takes the kernel of the rows that it wants.
constexpr int aux_sdy_rows(int rt) { return rt == 4 ? 2 : 8; }
// Auxiliary workgroups for `blocks` row blocks of the scaling, `scaling_us` of work for one, beside `tiles` workgroups that take launch_us by
// themselves with so many places on the machine.
int scaling_wgs(int blocks, double scaling_us, int tiles, double launch_us, int places);
struct ScaleDyJob {           // dYs = bf16(dY (s0 + ds)), crow[t] = sum_i dYs[t,i] (16 + z0[i])   (scale_dy_rows)
    const uint16_t *dY;
    const float *s0, *ds;
    const uint8_t *z0;
    uint16_t *dYs;
    float *crow;
    int T, N;
    int blk_end;              // row blocks (of aux_sdy_rows rows) of this job and all before it (set by the launch)
};
struct ReduceJob {            // out[j] = sum over ntiles of partial[tile][j], fixed order
    const float *partial;
    float *out;
    int ntiles, n;
    int chunk_end;            // 256-element chunks of this job and all before it
};
// dst[t / 32][c / 16][(t % 32) / 8][c % 16][t % 8] = src[t, c], zeros from T to Tp   (transpose_pad_tile)
struct TransposeJob {
    const uint16_t *src;
    uint16_t *dst;
    int T, C, Tp;
    int tile_end;             // 64 x 64 tiles of this job and all before it
};
struct MultiArgs {
    MultiJob job[MULTI_MAX_JOBS];          // must stay the first member: indexed in the argument block
    ScaleDyJob sdy[MULTI_MAX_JOBS];
    ReduceJob red[MULTI_MAX_JOBS];
    TransposeJob tp[2 * MULTI_MAX_JOBS];
    int n_jobs, n_sdy, n_red, n_tp;
    int aux_begin, aux_wgs;
};
// Per-channel jobs (any mode), with scale_dy and reduce jobs beside them, or, with `grouped`, group-wise MODE_Y / MODE_DX jobs
// (their tables in a.sb), with transpose jobs beside dX.
static_assert(sizeof(MultiArgs) <= 4096, "kernel argument block");
hipError_t launch_gemm_multi(int bits, bool grouped, MultiArgs &m, hipStream_t stream);
// The launches themselves, of tiles of RT row tiles: a contraction, a backward pair, or `workgroups` of a multi-contraction
// launch (gmode: -1 per channel, else the mode of the group-wise jobs).
struct GemmDwArgs;
template <int RT>
struct GemmRows {
    static hipError_t one(int bits, int mode, const GemmArgs &a, hipStream_t stream);
    static hipError_t pair(int bits, const GemmArgs &a_dds, const GemmArgs &a_dx, hipStream_t stream);
    static hipError_t multi(int bits, int gmode, int workgroups, const MultiArgs &m, hipStream_t stream);
    static hipError_t with_dw(int bits, int workgroups, const GemmDwArgs &m, hipStream_t stream);
};
// workgroups a contraction's tiles (and pieces of tiles) take in a launch (a multiple of 8)
int gemm_multi_wgs(const GemmArgs &a);

// Arguments of the token contraction dW = dY^T X with the codes applied in its epilogue (peqa_dw.hip):
// the scale gradient of group-wise layers.
struct DwArgs {
    const uint16_t *Xt;       // [Tp / 32, K / 16, 4, 16, 8] bf16: X in 32-token steps (transpose_pad_tile), zeros from T to Tp
    const uint16_t *dYt;      // [Tp / 32, N / 16, 4, 16, 8] bf16, dY likewise
    const uint32_t *packed;   // packed codes of the layer
    const uint8_t *z0;        // [N, G]
    const float *dz;          // [N, G] or NULL
    float *pc;                // out: sums of dW[i,k] (Q[i,k] - z[i,g(k)]) over each 64-feature chunk [N, K / 64], or, if
                              // dw_whole_groups(gsz), over each group [N, G]: d_ds itself
    int N, K, Tp;             // Tp % 64 == 0
    int gsz, G;               // group size (multiple of 64) and groups per channel
    int tiles_f, tiles_c;     // K / 128, ceil(N / 256)
    uint32_t strip_magic;     // reciprocal (div_magic) of 8 tiles_c, set by the launches
};
// workgroups of a layer: its tiles, rounded up to a whole number per XCD
inline int dw_wgs(const DwArgs &a) { return (a.tiles_f * a.tiles_c + 7) / 8 * 8; }
bool dw_args_ok(const DwArgs &a);          // what the kernel's indexing assumes
// 64 x 64 tiles of the copies that a workgroup of a launch of so many takes: four or one, one per wave (transpose_pad_tile), or 0: one by
// all its waves (transpose_pad_quarter).
int copies_per_wg(int tiles);
inline int copies_wgs(int tiles) { return copies_per_wg(tiles) == 4 ? (tiles + 3) / 4 : tiles; }
// X [T, K] -> xt, dY [T, N] -> dyt
hipError_t launch_transpose_pad(const uint16_t *X, int K, uint16_t *xt, const uint16_t *dY, int N, uint16_t *dyt, int T,
                                hipStream_t stream);
// groups of 64 or 128 features lie within one tile of 128: no chunk sums to add up
constexpr bool dw_whole_groups(int gsz) { return gsz <= 128; }
// bytes of the chunk sums [N, K / 64] of other groups
constexpr size_t dw_chunk_bytes(int N, int K, int gsz)
{
    return dw_whole_groups(gsz) ? 0 : (size_t)N * (size_t)(K / 64) * sizeof(float);
}
hipError_t launch_dw(int bits, const DwArgs &a, hipStream_t stream);
hipError_t launch_chunk_reduce(const float *pc, size_t n, int per, float *d_ds, hipStream_t stream);
// The token contractions of up to DW_MAX_JOBS layers in one launch, and the sums of their chunks in another.
constexpr int DW_MAX_JOBS = 8;
struct DwMultiArgs {
    DwArgs job[DW_MAX_JOBS];               // must stay the first member: indexed in the argument block
    int wg_end[DW_MAX_JOBS];               // workgroups of job j and all before it (unused entries: the total)
    float *d_ds[DW_MAX_JOBS];              // [N, G] out of the chunk sums
    int n_jobs;
};
hipError_t launch_dw_multi(int bits, DwMultiArgs &m, hipStream_t stream);
hipError_t launch_chunk_reduce_multi(const DwMultiArgs &m, hipStream_t stream);
// Both contractions of a group-wise backward in ONE launch of four-wave workgroups: the dX tiles of the jobs and the tiles of
// the token contractions.  Everything that either reads (tables, transposed copies: launch_group_prep) is complete before.
struct GemmDwArgs {
    MultiJob job[MULTI_MAX_JOBS];          // must stay the first member: indexed in the argument block.  MODE_DX, group-wise
    DwArgs dw[DW_MAX_JOBS];
    int dw_end[DW_MAX_JOBS];               // workgroups of token contraction j and all before it (unused entries: the total)
    int n_jobs, n_dw;
    int gemm_begin, dw_begin, dw_total;    // set by the launch: one of the begins is 0
};
static_assert(sizeof(GemmDwArgs) <= 4096, "kernel argument block");
hipError_t launch_gemm_dw(int bits, GemmDwArgs &m, hipStream_t stream);
// us that a tile of the token contraction takes beside another or a dX tile, in launches that do not fill the machine for long
inline double dw_tile_us(int T) { return 0.55 * ((T + 63) / 64 * 2) + 8.0; }
// and with none
inline double dw_tile_alone_us(int T) { return 0.25 * ((T + 63) / 64 * 2) + 8.0; }
// its chunk sums pc [N, K / 64] -> d_ds [N, K / gsz]
inline SumJob chunk_sums(const float *pc, float *d_ds, int N, int K, int gsz)
{
    return SumJob{pc, d_ds, (size_t)N * (size_t)(K / gsz), (size_t)(gsz / 64), 1, gsz / 64};
}
// Whether a group-wise backward of both gradients goes that way: `tiles` of dX (of gemm_row_tiles rows) and of the token
// contractions together.  The others keep the copies in spare workgroups of the dX launch.
bool bwd_one_launch(long long tiles, int T, int cus);
inline bool bwd_few_tiles(long long tiles, int cus) { return tiles <= 8ll * cus; }
// Whether its dX, with the pieces planned beside the token contractions, is a few long chains that a launch of its own would cut up.
bool bwd_dx_chains(int n, const SplitJob *jobs, int T, int cus);
// The (s, b) tables of up to GT_MAX layers in one launch.
constexpr int GT_MAX = 8;
struct GroupTableMulti {
    const float *s0[GT_MAX], *ds[GT_MAX];
    const uint8_t *z0[GT_MAX];
    float *sb[GT_MAX];
    int N[GT_MAX], G[GT_MAX];
    int n;
};
hipError_t launch_group_table_multi(const GroupTableMulti &a, hipStream_t stream);
// Tables and transposed copies in one launch.
struct GroupPrep {
    GroupTableMulti table;
    TransposeJob tp[2 * MULTI_MAX_JOBS];   // tile_end: running totals
    const float *dz;                       // of the only table, or NULL
    int table_end[GT_MAX];                 // set by the launch, as are whole_rows and copies_per_wg
    int n_tp, whole_rows, copies_per_wg;
};
hipError_t launch_group_prep(GroupPrep &a, hipStream_t stream);

// Arguments of the T <= 16 forward (peqa_gemv.hip): up to GEMV_MAX_LAYERS layers in one launch, laid side by
// side along the workgroup index.  Every layer has its own shape, input and slicing, so that the linears of a
// whole decoder block (different K, different X) can share one launch; the bit width is the launch's.
constexpr int GEMV_MAX_LAYERS = 8;
// GemvLayer::form: mask of the ring's depth; tiles half as wide as the launch's (GemvForm::narrow); workgroups that go first
enum { GEMV_DEPTH = 7, GEMV_NARROW = 8, GEMV_URGENT = 16 };
struct GemvLayer {
    const uint32_t *packed;
    const float *s0, *ds;     // [N, G]; ds may be NULL
    const uint8_t *z0;        // [N, G]
    const float *dz;          // [N, G] or NULL: trained zero-point offset
    const uint16_t *X;        // [T, K] bf16
    uint16_t *Y;              // [T, N] bf16
    float *partial;           // [S, T, N] fp32 slice partials of this layer (S > 1)
    int N, K, G;
    int chunk;                // features per scale group (K for per-channel layers)
    int S;                    // feature slices: a channel tile is S workgroups
    // set by launch_gemv: rounds that a wave keeps in flight and flags (GEMV_*); rounds of 64 features per scale group; rounds of a slice, one more in the first slice_rem slices;
    // reciprocals (div_magic) of S and of chunk_rounds
    int form;
    int chunk_rounds, slice_rounds, slice_rem;
    uint32_t s_magic, chunk_magic;
};
struct GemvArgs {
    GemvLayer layer[GEMV_MAX_LAYERS];   // must stay the first member: the kernels index it in the argument block
    int wg_end[GEMV_MAX_LAYERS];        // workgroups of layer j and all before it (unused entries: the total)
    int n_layers;
    int T;
    int prio_step;                      // workgroups per step of priority, 0: none (set by launch_gemv)
};
// Form of such a launch: 64 h channels (h = 0: 32) per workgroup of that many waves; half as many in tiles of layer j where bit j
// of `narrow` is set.
struct GemvForm {
    int h, waves;
    uint32_t narrow = 0;
};
inline int gemv_channels(const GemvForm &f) { return f.h == 0 ? 32 : 64 * f.h; }
// The form, and the slices of every layer (S[0..n)).  zbyte: no layer has a trained zero-point offset, so zero-points are
// bytes in LDS.  most: the most bytes that the partial sums of the slices may take; 0 gives the fewest slices that LDS allows.
// cus: compute units.
GemvForm gemv_plan(int n, const int *N, const int *K, const int *chunk, int bits, int T, bool zbyte, size_t most, int cus, int *S);
// fp32 partial sums of the layers with S > 1
size_t gemv_partials(int n, const int *N, int T, const int *S);
hipError_t launch_gemv(int bits, const GemvForm &f, const GemvArgs &a, hipStream_t stream);

// peqa_small.hip
hipError_t launch_rowsum(const uint16_t *X, int T, int K, int ksplit, float *rs, hipStream_t stream);
// the same for up to ROWSUM_MAX inputs of T rows each in one launch
constexpr int ROWSUM_MAX = 8;
struct RowsumMulti {
    const uint16_t *X[ROWSUM_MAX];
    float *rs[ROWSUM_MAX];
    int K[ROWSUM_MAX];
    int n, T;
};
hipError_t launch_rowsum_multi(const RowsumMulti &a, hipStream_t stream);
// dYs = bf16(dY (s0 + ds)) and crow; with n_red > 0 the same launch also sums `ntiles` partial vectors of n_red
// floats into red_out (launch_reduce_partials' job), with rs != NULL it takes the row sums of X [T, K] into rs
// (launch_rowsum's): independent pieces of work of the same backward
hipError_t launch_scale_dy(const uint16_t *dY, const float *s0, const float *ds, const uint8_t *z0, const float *dz,
                           int T, int N, uint16_t *dYs, float *crow, const float *partial, int ntiles, size_t n_red,
                           float *red_out, const uint16_t *X, int K, float *rs, hipStream_t stream);
hipError_t launch_rowsum_groups(const uint16_t *X, int T, int K, int gsz, float *rsg, hipStream_t stream);
// sb [G, N, 2] = (s, -s (16 + z))
hipError_t launch_group_table(const float *s0, const float *ds, const uint8_t *z0, const float *dz, int N, int G,
                              float *sb, hipStream_t stream);
// zero-point gradient: partial [ceil(T / KEPT_ROWS), N, G] from dY and the group sums rsg [T, G] of X, then
// d_dz[j] = -(s0 + ds)[j] * (sum of the partials)
hipError_t launch_dz_partial(const uint16_t *dY, const float *rsg, int T, int N, int G, float *partial,
                             hipStream_t stream);
// the same partials of a per-channel layer from the row sums rs [T, 2] (launch_rowsum's)
hipError_t launch_dz_rows(const uint16_t *dY, const float *rs, int T, int N, float *partial, hipStream_t stream);
// with n_red > 0 also launch_reduce_partials' job over red [red_rows, n_red]
hipError_t launch_dz_finish(const float *partial, int slices, size_t n, const float *s0, const float *ds, float *d_dz,
                            const float *red, int red_rows, size_t n_red, float *red_out, hipStream_t stream);
constexpr int KEPT_ROWS = 64;   // token rows per partial of launch_dds_kept
hipError_t launch_dds_kept(const uint16_t *dY, const float *P, int T, int N, float *partial, hipStream_t stream);
hipError_t launch_reduce_partials(const float *partial, int ntiles, size_t n, float *out, hipStream_t stream);
hipError_t launch_adamw(size_t n, float *ds, const float *g, float *m, float *v, const float *s0,
                        float lr, float b1, float b2, float eps, float wd, float inv_c1, float inv_c2,
                        hipStream_t stream);

// AdamW on several parameter vectors in one launch: tensor j holds elements [end[j-1], end[j]) of the
// launch's index space
constexpr int ADAMW_MAX_TENSORS = 16;
struct AdamwMulti {
    float *ds[ADAMW_MAX_TENSORS];
    const float *g[ADAMW_MAX_TENSORS];
    float *m[ADAMW_MAX_TENSORS];
    float *v[ADAMW_MAX_TENSORS];
    const float *s0[ADAMW_MAX_TENSORS];
    unsigned long long end[ADAMW_MAX_TENSORS];   // running totals; unused entries repeat the last
    int n_tensors;
};
hipError_t launch_adamw_multi(const AdamwMulti &a, float lr, float b1, float b2, float eps, float wd, float inv_c1,
                              float inv_c2, hipStream_t stream);

// peqa_quantize.hip
hipError_t launch_quantize(const float *W0, int N, int K, int bits, int group, uint32_t *packed,
                           float *s0, uint8_t *z0, hipStream_t stream);

// error-minimising variant (clipped-range grid); only where the rows fit in registers and LDS
bool quantize_resident_fits(int K, int G, bool search);
hipError_t launch_quantize_search(const float *W0, int N, int K, int bits, int group, int n_ratios, float step,
                                  uint32_t *packed, float *s0, uint8_t *z0, hipStream_t stream);

// What the size queries, and the checks that a call makes before it touches the device, plan for: a whole MI355X.  A call on
// a device of fewer units (a partition of one) then plans for those, which needs no more at least.
constexpr int PLAN_UNITS = 256;
// Compute units of the current device (looked up once per device; PLAN_UNITS where there is none).
int compute_units();

// Tracing hook: every launch goes through these so that peqa_trace_* can time it.
void trace_before(int kernel_id, hipStream_t stream);
void trace_after(int kernel_id, hipStream_t stream);

enum {
    KID_QUANTIZE = 0, KID_ROWSUM, KID_GEMM_Y, KID_GEMM_DDS, KID_GEMM_DX, KID_SCALE_DY,
    KID_REDUCE, KID_ADAMW, KID_GEMV, KID_GEMV_FINISH, KID_GROUP_TABLE, KID_DDS_KEPT, KID_DZ_PARTIAL, KID_DZ_FINISH,
    KID_TRANSPOSE, KID_GEMM_DW, KID_GEMM_BWD, KID_GEMM_MULTI_Y, KID_GEMM_MULTI_DDS, KID_GEMM_MULTI_DX, KID_GEMM_FINISH,
    KID_COUNT
};

}  // namespace peqa

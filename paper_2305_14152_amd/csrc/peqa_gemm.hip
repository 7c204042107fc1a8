// Dense contractions of the PEQA linear layer on gfx950 MFMA (per-channel scales).
//
//   MODE_Y   : Y[t,i]    = s_i * sum_k X[t,k] (Q[i,k] - z_i)                (Eq. 2 forward)
//   MODE_DDS : part[i]   = sum_{t in tile} dY[t,i] * sum_k X[t,k] (Q[i,k] - z_i)
//                                                   (scale gradient, column-reduced epilogue)
//   MODE_DX  : dX[t,k]   = sum_i (dY[t,i] s_i) (Q[i,k] - z_i)                (chain rule on Eq. 2)
//
// A workgroup owns a tile of 64, 96, 112 or 128 tokens x 256 output columns (peqa_tile.h; gemm_plan takes the height) as four
// waves side by side along the columns: of 128 x 64 in the tallest, 8 x 4 MFMA 16x16x32 tiles, 128 fp32 AGPRs per wave.  Two forms:
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
// dY) as bf16 tiles of the tile's rows x 32 (16-byte chunks XOR-swizzled by row), the weight operand as
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
#include <math.h>
#include <stddef.h>

#include "peqa_device.h"
#include "peqa_kernels.h"

namespace peqa {

namespace {

// One 256-thread workgroup per 1024 elements of a split contraction's result, four neighbouring columns per thread:
// HBM-bound, split x 4 + 2 bytes per element, where there are many; else by its chain of latencies, so up to eight pieces are asked for
// together and a unit holds eight workgroups (64 registers; with 76, 11008 x 4096, T = 500, 6.5 us instead of 6.2).  us, four pieces at a time,
// those past the last re-read and left out / so: 31 pieces of 91 x 384 6.5 / 4.4, 27 of 22 x 1024 5.7 / 4.1, 11 of 23 x 896 4.0 / 3.6,
// a block of d = 1920, T = 37, 5.3 / 4.6.
__global__ __launch_bounds__(256, 8) void split_finish_kernel(FinishMulti f)
{
    if ((int)blockIdx.y >= f.n) {
        const SumJob S = kernarg_load<SumJob>((uint32_t)(offsetof(FinishMulti, sum) + (blockIdx.y - f.n) * sizeof(SumJob)));
        const size_t j = (size_t)blockIdx.x * 256 + threadIdx.x;
        if (j >= S.n) return;
        const float *src = S.src + j * S.step_j;
        float v = 0.f;
        int i = 0;
        for (; i + 8 <= S.count; i += 8) {                     // eight loads in flight, added in order
            float p[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) p[u] = global_load<float>(src + (size_t)(i + u) * S.step);
#pragma unroll
            for (int u = 0; u < 8; ++u) v += p[u];
        }
        for (; i < S.count; ++i) v += global_load<float>(src + (size_t)i * S.step);
        global_store(S.dst + j, v);
        return;
    }
    const FinishJob J = kernarg_load<FinishJob>((uint32_t)(blockIdx.y * sizeof(FinishJob)));
    const GemmArgs &a = J.a;
    if (a.split < 2) return;
    const uint32_t c4 = (uint32_t)a.C >> 2;
    const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= (size_t)a.T * c4) return;
    // (a 64-bit division is a hundred instructions)
    const size_t t = e >> 32 ? e / c4 : (size_t)((uint32_t)e / (uint32_t)c4);
    const int col = (int)(e - t * c4) * 4;
    // what the epilogue needs besides the pieces is asked for before them
    const bool scale = a.gsz == 0 && J.mode == MODE_Y, shift = a.gsz == 0 && J.mode != MODE_Y;
    f32x2 r = {0.f, 0.f};
    f32x4 sc = {0.f, 0.f, 0.f, 0.f}, dz = sc, ds = sc;
    uint32_t zz = 0;
    if (scale) {
        r = global_load<f32x2>(a.rs + 2 * t);
        zz = global_load<uint32_t>(a.z0 + col);
        sc = global_load<f32x4>(a.s0 + col);
        if (a.ds) ds = global_load<f32x4>(a.ds + col);
        if (a.dz) dz = global_load<f32x4>(a.dz + col);
    }
    if (shift) r[0] = global_load<float>(a.crow + t);
    const f32x4 *p = reinterpret_cast<const f32x4 *>(a.acc_part) + e;
    const size_t stride = (size_t)a.T * c4;
    // up to eight loads in flight, added in order
    f32x4 v = global_load<f32x4>(p);
    int left = a.split - 1;
    auto add = [&](auto n_c) __attribute__((always_inline)) {
        constexpr int NL = decltype(n_c)::value;
        f32x4 w[NL];
#pragma unroll
        for (int u = 0; u < NL; ++u) w[u] = global_load<f32x4>(p += stride);
#pragma unroll
        for (int u = 0; u < NL; ++u) v += w[u];
        left -= NL;
    };
    while (left >= 8) add(std::integral_constant<int, 8>{});
    if (left & 4) add(std::integral_constant<int, 4>{});
    if (left & 2) add(std::integral_constant<int, 2>{});
    if (left & 1) add(std::integral_constant<int, 1>{});
    if (scale) {
        f32x4 zoff;
#pragma unroll
        for (int u = 0; u < 4; ++u) zoff[u] = kCodeOffset + (float)((zz >> (8 * u)) & 0xFFu);
        if (a.dz) zoff += dz;
        if (a.ds) sc += ds;
        v -= zoff * (r[0] + r[1]);
        if (a.P) global_store(a.P + t * a.C + col, v);
        v *= sc;
    }
    if (shift) v -= r[0];
    u32x2 o;
    o[0] = pack_bf16x2(v[0], v[1]);
    o[1] = pack_bf16x2(v[2], v[3]);
    global_store(a.out + t * a.C + col, o);
}

}  // namespace

hipError_t launch_split_finish(const FinishMulti &f, hipStream_t stream)
{
    size_t most = 0;                                           // workgroups along x
    for (int j = 0; j < f.n; ++j) {
        const GemmArgs &a = f.job[j].a;
        const size_t wgs = a.split > 1 ? ((size_t)a.T * a.C + 1023) / 1024 : 0;
        most = wgs > most ? wgs : most;
    }
    for (int j = 0; j < f.n_sums; ++j) most = (f.sum[j].n + 255) / 256 > most ? (f.sum[j].n + 255) / 256 : most;
    if (most == 0) return hipSuccess;
    trace_before(KID_GEMM_FINISH, stream);
    hipLaunchKernelGGL(split_finish_kernel, dim3((unsigned)most, f.n + f.n_sums), dim3(256), 0, stream, f);
    trace_after(KID_GEMM_FINISH, stream);
    return hipGetLastError();
}

// Contraction halves per workgroup.  Eight waves with two halves, one workgroup per compute unit, when a launch
// has at most one tile per compute unit (a lone four-wave workgroup leaves every SIMD a single wave, which
// measures 7-10 % slower); otherwise four waves with the whole range and two workgroups per compute unit
// (72 KB of LDS each), which fill the same four SIMDs with two waves each, need no exchange of partial sums,
// and hide one workgroup's ring fill and epilogue behind the other's loop.  The option gemm_waves = 4 or 8
// (peqa_set_option) forces one of them, for tests and comparisons.
int halves_per_workgroup(int tiles, bool paired)
{
    if (paired) return 2;
    if (options().gemm_waves == 4) return 1;
    if (options().gemm_waves == 8) return 2;
    const int cus = compute_units();
    return tiles > cus ? 1 : 2;
}

// us per 32-deep step of a tile: alone on its compute unit, with a second one beside it, and as one of two halves of eight waves
// (per step of the whole).  Measured at K = 1024 to 4096, tiles of other columns on every unit; what is shared, a tenth less than
// with every unit full, as in the launches that are planned here (full ones: 0.66 of 128 rows per channel).
struct StepTimes {
    double alone, shared, halves;
};
static StepTimes step_times(int rt, bool grouped)
{
    if (grouped) return rt == 4 ? StepTimes{0.39, 0.59, 0.29} : rt == 6 ? StepTimes{0.46, 0.71, 0.36}
                      : rt == 7 ? StepTimes{0.48, 0.79, 0.39} : StepTimes{0.52, 0.83, 0.42};
    return rt == 4 ? StepTimes{0.28, 0.39, 0.19} : rt == 6 ? StepTimes{0.33, 0.50, 0.26}
         : rt == 7 ? StepTimes{0.36, 0.56, 0.29} : StepTimes{0.40, 0.61, 0.32};
}

int gemm_pieces(const GemmArgs &a) { return a.split > 1 ? a.split : 1; }

// Workgroups that the tiles of a contraction take in a launch: their number rounded up to a multiple of 8.
int gemm_multi_wgs(const GemmArgs &a) { return (a.tiles_t * a.tiles_c * gemm_pieces(a) + 7) / 8 * 8; }

// A launch lasts as long as its longest workgroup (StepTimes; 8 us to fill the ring, drain and store, 6 with tiles of 64 rows) or
// as the work that two workgroups per unit get through, plus about a
// third of the longest for the last round.  Pieces of Y and dX cost a second launch and fp32 sums written and read again (5 TB/s).
double gemm_form_us(int n, const SplitJob *jobs, int T, int rt, bool grouped, bool single, double other_us, int cus)
{
    const int tiles_t = gemm_tiles_t(T, rt);
    const StepTimes c = step_times(rt, grouped);
    const double fixed = rt == 4 ? 6.0 : 8.0;
    int wgs = 0, order[FINISH_MAX], len[FINISH_MAX];                   // jobs by falling length of a workgroup, as launched
    double steps = 0.0;
    size_t bytes = 0;
    for (int j = 0; j < n; ++j) {
        const int s = jobs[j].split;
        len[j] = (jobs[j].KC / 128 + s - 1) / s * 4;
        wgs += jobs[j].tiles_c * tiles_t * s;
        steps += (double)jobs[j].tiles_c * tiles_t * jobs[j].KC / 32;
        if (s > 1) bytes += s * jobs[j].out_bytes;
        int k = j;
        for (; k > 0 && len[order[k - 1]] < len[j]; --k) order[k] = order[k - 1];
        order[k] = j;
    }
    const int piece = len[order[0]];
    double us;
    if (single && wgs <= cus) {
        us = c.halves * piece + fixed + 3.0;                           // the eight-wave form
    } else {
        // Workgroups are dealt to the units in turn, the longest first: the longest shares its unit with number cus, 2 cus, ... of
        // them, for as long as those last.  The workgroups that fill a job up to a multiple of 8 count: they end at once, but the
        // dispatcher has dealt units to them (seven layers of a block of d = 896, T = 500: 250 pieces in 272 workgroups 35 us, 400
        // pieces of 64 rows 28; in groups of 128 35.5, 216 pieces in 224 workgroups 29.5).
        int slots = 0, shared = 0, next = cus, second = 0, third = 0;
        for (int k = 0; k < n; ++k) {
            const SplitJob &job = jobs[order[k]];
            slots += (job.tiles_c * tiles_t * job.split + 7) / 8 * 8;  // (as launched: gemm_multi_wgs)
            for (; next < slots && shared < piece; next += cus) shared += len[order[k]];
            if (second == 0 && slots >= 2 * cus) second = len[order[k]];
            if (third == 0 && slots > 2 * cus) third = len[order[k]];
        }
        shared = shared < piece ? shared : piece;
        const double chain = c.alone * (piece - shared) + c.shared * shared + fixed;
        const double tail = other_us > 0.0 ? 0.2 : 0.3;                // (token tiles are short and fill the end)
        const double work = (c.shared * steps + fixed * wgs + other_us) / (2.0 * cus) + tail * chain;
        us = chain > work ? chain : work;
        // Number 2 cus starts where the first pair ends, and most of it runs alone: forward of d = 3584, f = 10240 in groups of 64,
        // T = 65, 80 us in 342 workgroups, 85 in 520.
        const double late = third ? c.shared * second + fixed + c.alone * third + fixed : 0.0;
        us = late > us ? late : us;
        // a token tile by itself: 1664 x 384, T = 3147, backward 45 us with dX in 50 or 100 whole tiles, 48 in halves
        if (other_us > 0.0 && us < dw_tile_alone_us(T)) us = dw_tile_alone_us(T);
    }
    return bytes > 0 ? us + 4.0 + (double)bytes * 2.0 / 5e6 : us;
}

constexpr int kMinPiece = 512;                                 // shorter pieces are mostly fill and drain

// Cuts the longest contraction of a launch into d pieces and the others into as many of that length as they hold.  Returns the bytes
// of the partial results.
static size_t cut_jobs(int n, SplitJob *jobs, int longest, int d)
{
    const int target = (longest + d - 1) / d;
    size_t bytes = 0;
    for (int j = 0; j < n; ++j) {
        const int s = (jobs[j].KC + target - 1) / target, most = jobs[j].KC < kMinPiece ? 1 : jobs[j].KC / kMinPiece;
        jobs[j].split = s < most ? s : most;
        if (jobs[j].split > 1) bytes += jobs[j].split * jobs[j].out_bytes;
    }
    return bytes;
}

// What a launch is made of: tiles of gemm_row_tiles rows or of fewer, whole or cut into pieces of equal length over the launch.  Taken
// is the least estimate of those that lie below the plain launch (whole, gemm_row_tiles rows) by more than the estimate's own
// error: 5 %; for pieces, where the plain launch has more than one round of workgroups and little to gain, 17 % (six splits
// between 5 and 17 % of 580 to 1300 tiles of group-wise dX measured 3 to 9 % longer).
//
// Against all forms of 1600 launches (forwards, dX and scale gradients of blocks and layers, T = 20 to 1800), the time of the one
// taken is 1.017 times the best in the geometric mean.  With the longest sharing for its mean-length neighbour or not at all, shared
// steps as with every unit full, sums at 3.5 TB/s, 13 % throughout and no tiles of fewer rows past two per unit it was 1.032:
// forward of d = 3072, T = 458, 118 us in 536 workgroups, now 106 in 670 of 96 rows; d = 896, groups of 128, T = 607, 35.6 -> 33.5.
// Of 415 launches of dX beside token contractions 1.021 and 1.044.
// Whole -> split, us per call:
//                                     T = 17          T = 128         T = 500
//   7B block 4-bit, forward           124 ->  56      131 ->  71      whole
//                   backward          392 -> 108      397 -> 140      480 -> 367
//   13B block 3-bit g128, forward     239 ->  93      240 -> 113      whole
//                         backward    708 -> 310      749 -> 393      953 -> 853
//   4096 x 11008 4-bit alone, forward 103 ->  28      107 ->  37      112 ->  72
//
// Tiles of fewer rows where those of gemm_row_tiles leave the machine idle: a step of 64 rows is shorter by a third and more, and
// there are up to twice as many.  96 and 112 rows are weighed too: 11008 x 4096 in groups of 64, T = 500, has 172 tiles of 128 rows
// for 256 units and 215 of 112, training step 184 -> 180 us; and 16000 x 11264 3-bit, T = 131, forward 78 us in 189 whole tiles of
// 64 rows, 69 in 252 halves of 96.
int gemm_plan(int n, SplitJob *jobs, int T, bool grouped, bool single, bool dds, double other_us, size_t max_bytes, int cus)
{
    const int by_rows = gemm_row_tiles(T);
    int longest = 0;
    for (int j = 0; j < n; ++j) {
        jobs[j].split = 1;
        longest = jobs[j].KC > longest ? jobs[j].KC : longest;
    }
    if (options().gemm_waves != 0 || options().bwd_pair >= 0) return by_rows;   // forced forms are whole contractions
    struct Form {
        double us;
        int rt, d;
    };
    Form plain{0.0, by_rows, 1}, whole{HUGE_VAL, by_rows, 1}, cut{HUGE_VAL, by_rows, 1};
    int rounds = 1;                                            // of the plain launch
    const int forms[4] = {by_rows, 4, 6, 7};
    for (int form = 0; form < (by_rows > 4 && !dds ? 4 : 1); ++form) {
        const int rt = forms[form], tiles_t = gemm_tiles_t(T, rt);
        if (form && rt >= by_rows) continue;
        for (int d = 1; d <= 48; d += d < 6 ? 1 : (d < 12 ? 2 : 4)) {
            if (d > 1 && (longest + d - 1) / d < kMinPiece) break;     // features (or channels) per piece
            const size_t bytes = cut_jobs(n, jobs, longest, d);
            if (d > 1 && bytes > max_bytes) continue;
            int wgs = 0;
            for (int j = 0; j < n; ++j) wgs += jobs[j].tiles_c * tiles_t * jobs[j].split;
            if (form == 0 && d == 1) rounds = (wgs + 2 * cus - 1) / (2 * cus);
            if (form && wgs > 3 * cus) break;                          // not idle any more: fewer rows are the slower ones
            const double us = gemm_form_us(n, jobs, T, rt, grouped, single, other_us, cus);
            Form &least = d > 1 ? cut : form ? whole : plain;
            if (us < least.us || (d == 1 && form == 0)) least = Form{us, rt, d};
        }
    }
    Form best = plain;
    if (whole.us < 0.95 * plain.us) best = whole;
    if (cut.us < (rounds == 1 ? 0.95 : 0.83) * plain.us && cut.us < best.us) best = cut;
    (void)cut_jobs(n, jobs, longest, best.d);
    return best.rt;
}

bool gemm_four_waves(int tiles) { return halves_per_workgroup(tiles, false) == 1; }

// What a launch adds to a contraction's arguments.
static void prepare_args(GemmArgs &a)
{
    a.patch_t = a.tiles_t < 4 ? a.tiles_t : 4;
    a.whole_magic = 0xFFFFFFFFu / ((uint32_t)a.tiles_t * (uint32_t)a.tiles_c);
    a.strip_magic = 0xFFFFFFFFu / ((uint32_t)a.patch_t * (uint32_t)a.tiles_c);
    a.piece_units = a.KC / 128 / gemm_pieces(a);
    a.unit_rem = a.KC / 128 % gemm_pieces(a);
}

// Calls f with the instantiation for tiles of rt row tiles.
template <class F>
static hipError_t with_rows(int rt, F &&f)
{
    switch (rt) {
    case 4: return f(GemmRows<4>{});
    case 6: return f(GemmRows<6>{});
    case 7: return f(GemmRows<7>{});
    default: return f(GemmRows<8>{});
    }
}

// Row tiles (of 16 tokens) per tile: as few as cover T with no more tiles than 128 rows would take, so that the rows past T of
// the last tile, which cost as much as any other, are few.  Against tiles of 128 rows: 3-bit block of d = 3968, T = 49,
// training step 180 -> 127 us; 4-bit block of d = 4096, T = 149, 314 -> 290; 3-bit prefill of a 7B block, T = 333, 152.4 -> 147.7;
// 256 x 256 layer, T = 64, forward launch 9.1 -> 6.6.
int gemm_row_tiles(int T)
{
    const int tiles = (T + 127) / 128, rt = ((T + tiles - 1) / tiles + 15) / 16;
    return rt <= 4 ? 4 : (rt <= 6 ? 6 : rt);
}

hipError_t launch_gemm(int bits, int mode, const GemmArgs &a_in, hipStream_t stream)
{
    GemmArgs a = a_in;
    prepare_args(a);
    const int kid = mode == MODE_Y ? KID_GEMM_Y : (mode == MODE_DDS ? KID_GEMM_DDS : KID_GEMM_DX);
    trace_before(kid, stream);
    const hipError_t e = with_rows(a.rt, [&](auto rows) { return decltype(rows)::one(bits, mode, a, stream); });
    trace_after(kid, stream);
    return e;
}

// A workgroup of the scaling costs a place for as long as it lasts, so launches of many rounds get few; but no launch is over before the
// scaling is.  So it takes a quarter of the launch by the estimates, in no fewer than 192 workgroups where there are less than four
// rounds of tiles (those end early in a round that is not full), and in no more than 512.  Backward, us, with 64 / 128 / 192 / 256 / 512:
// blocks of d = 256, f = 640, T = 3727 130 / 80 / 63 / 60 / 51, d = 640, f = 1792, T = 1795 124 / 90 / 82 / 79 / 75, d = 1152, f = 3456, T = 2928
// 255 / 207 / 206 / 208 / 206, d = 3072, f = 8192, T = 1024 399 / 388 / 388 / 391 / 390, d = 4096, f = 11008, T = 512 369 / 354 / 348 / 349 / 350,
// and with five rounds, T = 2048, 1222 / 1227 / 1231 / 1230 / 1232.
int scaling_wgs(int blocks, double scaling_us, int tiles, double launch_us, int places)
{
    const double quarter = scaling_us / (0.25 * launch_us);
    int wgs = quarter < 512.0 ? 64 * (int)(quarter / 64 + 0.5) : 512;
    const int least = tiles < 4 * places ? 192 : 64;
    wgs = wgs < least ? least : wgs;
    return wgs < blocks ? wgs : (blocks + 7) / 8 * 8;
}

hipError_t launch_gemm_multi(int bits, bool grouped, MultiArgs &m, hipStream_t stream)
{
    if (m.n_jobs < 0 || m.n_jobs > MULTI_MAX_JOBS || m.n_sdy < 0 || m.n_sdy > MULTI_MAX_JOBS || m.n_red < 0 ||
        m.n_red > MULTI_MAX_JOBS || m.n_tp < 0 || m.n_tp > 2 * MULTI_MAX_JOBS)
        return hipErrorInvalidValue;
    int total = 0;
    int rt = 8;
    for (int j = 0; j < MULTI_MAX_JOBS; ++j) {
        if (j < m.n_jobs) {
            GemmArgs &a = m.job[j].a;
            if ((a.gsz > 0) != grouped || a.tp_blocks) return hipErrorInvalidValue;
            if (grouped && m.job[j].mode == MODE_DDS) return hipErrorInvalidValue;
            prepare_args(a);
            if (j > 0 && a.rt != rt) return hipErrorInvalidValue;
            rt = a.rt;
            total += gemm_multi_wgs(a);
        } else {
            m.job[j] = m.job[m.n_jobs > 0 ? m.n_jobs - 1 : 0];
        }
        m.job[j].wg_end = total;
    }
    if (grouped ? m.n_sdy + m.n_red > 0 : m.n_tp > 0) return hipErrorInvalidValue;   // (multi_aux)
    if (total == 0 && m.n_sdy > 0) {
        // The scaling alone: two rows at a time while blocks of eight are fewer than the units.  dX alone of per-channel blocks, us, eight / two:
        // d = 2048, f = 5632, T = 17 35.9 / 31.1, T = 400 72 / 69, T = 500 (252 blocks) 78 / 75; d = 4096, f = 11008, T = 60 62 / 56, T = 250 121 / 115.
        int blocks = 0;
        for (int j = 0; j < m.n_sdy; ++j) blocks += (m.sdy[j].T + aux_sdy_rows(8) - 1) / aux_sdy_rows(8);
        if (blocks < compute_units()) rt = 4;
    }
    for (int j = 0, blocks = 0; j < m.n_sdy; ++j) m.sdy[j].blk_end = blocks += (m.sdy[j].T + aux_sdy_rows(rt) - 1) / aux_sdy_rows(rt);
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
    const hipError_t e = with_rows(rt, [&](auto rows) {
        return decltype(rows)::multi(bits, grouped ? mode0 : -1, total + m.aux_wgs, m, stream);
    });
    trace_after(kid, stream);
    return e;
}

// One launch has one start and one end where two have two; it wants the copies made beforehand, where launches of their own hide part
// of them behind dX.  So up to eight tiles per unit, or 1536 tokens: what the copies take grows with the tokens, and an end
// is as long as a tile.  Training steps, us, one launch each -> one for both: block of d = 4096, 4 bits, g128, T = 300 497 -> 485,
// d = 5120, 3 bits, T = 1000 1772 -> 1749, d = 3072, g64, T = 1500 1011 -> 986, 22016 x 8192, T = 1024 1016 -> 997; at
// T = 2048 and more from 1.00 to 1.01, and 2048 x 12288, T = 3500 (2112 tiles) 525 -> 538.
constexpr int kOneLaunchTokens = 1536;
bool bwd_one_launch(long long tiles, int T, int cus)
{
    return options().gemm_waves == 0 && options().bwd_pair < 0 && options().grouped_dds == 0 &&
           (bwd_few_tiles(tiles, cus) || T <= kOneLaunchTokens);
}

// dX that gemm_plan leaves whole beside the token contractions, of tiles (counted as of gemm_row_tiles rows, whatever it takes) on no
// more than half of the units: workgroups that share with token tiles for as long as there are any and run on alone, where a launch
// of their own has pieces or many more of 64 rows.  Backward, us, one launch for both against one each: 9216 x 8192 in groups of
// 64, T = 400, 167 against 150; 8192 x 3072 in groups of 128, T = 1200, 149 / 132; even at 4096 x 4096, T = 900, 80 / 80.
// Short ones gain by the launches saved: 3072 x 4096, T = 900, 63 / 69; 2048 x 2048, T = 1800, 44 / 56.  More tiles, or pieces:
// 5120 x 5120, T = 1000, 113 / 126; 11008 x 4096, T = 922 (2 pieces), 169 / 180; 15872 x 3840, T = 922 (2), 226 / 236.
bool bwd_dx_chains(int n, const SplitJob *jobs, int T, int cus)
{
    const int tiles_t = gemm_tiles_t(T, gemm_row_tiles(T));
    int tiles = 0, longest = 0;
    for (int j = 0; j < n; ++j) {
        if (jobs[j].split > 1) return false;
        tiles += tiles_t * jobs[j].tiles_c;
        longest = jobs[j].KC > longest ? jobs[j].KC : longest;
    }
    return 2 * tiles <= cus && longest > 3072;
}

hipError_t launch_gemm_dw(int bits, GemmDwArgs &m, hipStream_t stream)
{
    if (m.n_jobs < 1 || m.n_jobs > MULTI_MAX_JOBS || m.n_dw < 1 || m.n_dw > DW_MAX_JOBS) return hipErrorInvalidValue;
    int total = 0, longest = 0, dw_steps = 0;
    for (int j = 0; j < MULTI_MAX_JOBS; ++j) {
        if (j < m.n_jobs) {
            GemmArgs &a = m.job[j].a;
            if (a.gsz <= 0 || a.tp_blocks || m.job[j].mode != MODE_DX || a.rt != m.job[0].a.rt) return hipErrorInvalidValue;
            prepare_args(a);
            total += gemm_multi_wgs(a);
            const int steps = a.KC / 32 / gemm_pieces(a);
            longest = steps > longest ? steps : longest;
        } else {
            m.job[j] = m.job[m.n_jobs - 1];
        }
        m.job[j].wg_end = total;
    }
    m.dw_total = 0;
    for (int j = 0; j < DW_MAX_JOBS; ++j) {
        if (j < m.n_dw) {
            if (!dw_args_ok(m.dw[j])) return hipErrorInvalidValue;
            m.dw[j].strip_magic = 0xFFFFFFFFu / (8u * (uint32_t)m.dw[j].tiles_c);
            m.dw_total += dw_wgs(m.dw[j]);
            dw_steps = m.dw[j].Tp / 32 > dw_steps ? m.dw[j].Tp / 32 : dw_steps;
        } else {
            m.dw[j] = m.dw[m.n_dw - 1];
        }
        m.dw_end[j] = m.dw_total;
    }
    // the longer workgroups first (a step of either takes about as long); both numbers of workgroups are multiples of 8
    m.gemm_begin = dw_steps > longest ? m.dw_total : 0;
    m.dw_begin = dw_steps > longest ? 0 : total;
    trace_before(KID_GEMM_BWD, stream);
    const hipError_t e = with_rows(m.job[0].a.rt, [&](auto rows) {
        return decltype(rows)::with_dw(bits, total + m.dw_total, m, stream);
    });
    trace_after(KID_GEMM_BWD, stream);
    return e;
}

hipError_t launch_gemm_bwd_pair(int bits, const GemmArgs &dds_in, const GemmArgs &dx_in, hipStream_t stream)
{
    GemmArgs a_dds = dds_in, a_dx = dx_in;
    if (a_dds.gsz > 0 || a_dx.gsz > 0 || a_dds.tp_blocks || a_dx.tp_blocks || a_dds.rt != a_dx.rt)
        return hipErrorInvalidValue;
    prepare_args(a_dds);
    prepare_args(a_dx);
    trace_before(KID_GEMM_BWD, stream);
    const hipError_t e = with_rows(a_dds.rt, [&](auto rows) {
        return decltype(rows)::pair(bits, a_dds, a_dx, stream);
    });
    trace_after(KID_GEMM_BWD, stream);
    return e;
}

}  // namespace peqa

// Block-level entry points of the C-ABI (include/peqa.h): the linears of a decoder block -- any list of up to
// PEQA_MAX_BLOCK independent PEQA layers, each with its own input -- behind one forward and one backward call.
#include "peqa_host.h"

using namespace peqa::host;

// every table of a launch holds an entry per item of a call
static_assert(peqa::MULTI_MAX_JOBS >= PEQA_MAX_BLOCK && peqa::DW_MAX_JOBS >= PEQA_MAX_BLOCK && peqa::GT_MAX >= PEQA_MAX_BLOCK &&
                  peqa::ROWSUM_MAX >= PEQA_MAX_BLOCK && peqa::FINISH_MAX >= PEQA_MAX_BLOCK && peqa::GEMV_MAX_LAYERS >= PEQA_MAX_BLOCK,
              "launch tables against PEQA_MAX_BLOCK");

namespace {

peqa_status check_items(int32_t n, const peqa_block_item *items, int32_t T)
{
    if (!items) return PEQA_ERR_NULL;
    if (n < 1 || n > PEQA_MAX_BLOCK) return PEQA_ERR_PARAM;
    if (T < 1 || T > (1 << 24)) return PEQA_ERR_SHAPE;
    for (int j = 0; j < n; ++j) {
        const peqa_status st = peqa_check_layout(&items[j].layout);
        if (st != PEQA_OK) return st;
        if (items[j].layout.bits != items[0].layout.bits) return PEQA_ERR_PARAM;
    }
    return PEQA_OK;
}

// Distinct inputs of the items, in order of first appearance: xi[j] = index of item j's input.
int distinct_inputs(int32_t n, const peqa_block_item *items, int *xi, const uint16_t **xs, int *ks)
{
    int nx = 0;
    for (int j = 0; j < n; ++j) {
        xi[j] = -1;
        for (int i = 0; i < nx; ++i)
            if (xs[i] == items[j].X && ks[i] == items[j].layout.k_in) xi[j] = i;
        if (xi[j] < 0) {
            xs[nx] = items[j].X;
            ks[nx] = items[j].layout.k_in;
            xi[j] = nx++;
        }
    }
    return nx;
}

// Regions of the workspace.  Sized per item, so that the size does not depend on which items share an input; a call
// uses the region of the first item that reads an input for all that share it.
struct BlockSpace {
    size_t rs[PEQA_MAX_BLOCK];       // per-channel item, T > 16: row sums of its input
    size_t dys[PEQA_MAX_BLOCK];      // backward, per-channel item j: bf16(dY (s0 + ds)) [T, N]
    size_t crow[PEQA_MAX_BLOCK];     //   its row factors [T]
    size_t partial[PEQA_MAX_BLOCK];  //   per-token-tile partials of its scale gradient [tiles_t, N]
    size_t table[PEQA_MAX_BLOCK];    // group-wise item j: its (s, b) table [G, N, 2]
    size_t xt[PEQA_MAX_BLOCK];       // backward, group-wise item j: step-major transposed copy of its input [K, T']
    size_t dyt[PEQA_MAX_BLOCK];      //   the same of its dY [N, T']
    size_t pc[PEQA_MAX_BLOCK];       //   scale gradient per 64-feature chunk [N, K / 64], groups past 128 only
    size_t total;
    // Pieces of the contractions (1 = whole) and the regions of their partial results, behind the others: `total` includes
    // them, and a workspace of at least `min_total` bytes is served too (plan_block).
    size_t min_total;
    int split_y[PEQA_MAX_BLOCK], split_dx[PEQA_MAX_BLOCK], split_dds[PEQA_MAX_BLOCK];
    int rt_y[2], rt_dx[2];           // row tiles per tile of the launches of per-channel and of group-wise items
    // Group-wise items: dX and token contractions in one launch (launch_gemm_dw), as split_dx and rt_dx[1] have it; the dX launch of
    // a call without that one (too many tiles and tokens, or no scale gradient asked for) has a plan of its own.
    bool one_launch, many_tiles;     // many_tiles: not by bwd_few_tiles
    int split_dx_alone[PEQA_MAX_BLOCK], rt_dx_alone;
    size_t acc[PEQA_MAX_BLOCK], acc_dds[PEQA_MAX_BLOCK];
};

// The regions of the pieces.
void lay_out_pieces(BlockSpace &w, int32_t n, const peqa_block_item *items, int32_t T)
{
    const size_t tiles_t = ((size_t)T + 127) / 128;
    w.total = w.min_total;
    for (int j = 0; j < n; ++j) {
        const size_t N = (size_t)items[j].layout.n_out, K = (size_t)items[j].layout.k_in;
        w.acc[j] = w.total;
        if (w.split_y[j] > 1) w.total += round256((size_t)w.split_y[j] * T * N * sizeof(float));
        const int dx = w.split_dx[j] > w.split_dx_alone[j] ? w.split_dx[j] : w.split_dx_alone[j];
        if (dx > 1) w.total += round256((size_t)dx * T * K * sizeof(float));
        w.acc_dds[j] = w.total;
        if (w.split_dds[j] > 1) w.total += round256((size_t)w.split_dds[j] * tiles_t * N * sizeof(float));
    }
}

BlockSpace carve_block(int32_t n, const peqa_block_item *items, int32_t T, int32_t op, int cus)
{
    BlockSpace w{};
    const size_t tiles_t = ((size_t)T + 127) / 128, Tp = ((size_t)T + 63) / 64 * 64;
    size_t off = 0;
    for (int j = 0; j < n; ++j) {
        const peqa_layout *L = &items[j].layout;
        const size_t N = (size_t)L->n_out, K = (size_t)L->k_in;
        if (grouped(L)) {
            w.table[j] = off; off += round256(N * (size_t)groups(L) * 2 * sizeof(float));
            if (op == PEQA_OP_BWD) {
                w.xt[j] = off;  off += round256(K * Tp * sizeof(uint16_t));
                w.dyt[j] = off; off += round256(N * Tp * sizeof(uint16_t));
                w.pc[j] = off;  off += round256(peqa::dw_chunk_bytes(L->n_out, L->k_in, L->group_size));
            }
            continue;
        }
        w.rs[j] = off; off += round256((size_t)T * 2 * sizeof(float));
        if (op == PEQA_OP_BWD) {
            w.dys[j] = off;     off += round256((size_t)T * N * sizeof(uint16_t));
            w.crow[j] = off;    off += round256((size_t)T * sizeof(float));
            w.partial[j] = off; off += round256(tiles_t * N * sizeof(float));
        }
    }
    w.total = w.min_total = off ? off : 256;
    // splits, planned per launch: the per-channel items' forward, scale-gradient and dX launches, the group-wise items'
    // forward and dX launches (as if every gradient of every item were asked for)
    for (int j = 0; j < n; ++j) w.split_y[j] = w.split_dx[j] = w.split_dds[j] = w.split_dx_alone[j] = 1;
    auto plan = [&](bool gw, int mode, int *split) {
        peqa::SplitJob job[PEQA_MAX_BLOCK];
        int of[PEQA_MAX_BLOCK], m = 0;
        for (int j = 0; j < n; ++j) {
            const peqa_layout *L = &items[j].layout;
            if (grouped(L) != gw) continue;
            const int C = mode == peqa::MODE_DX ? L->k_in : L->n_out, KC = mode == peqa::MODE_DX ? L->n_out : L->k_in;
            of[m] = j;
            const size_t out_bytes = mode == peqa::MODE_DDS ? 0 : (size_t)T * C * sizeof(float);
            job[m++] = peqa::SplitJob{(C + 255) / 256, KC, out_bytes, 1};
        }
        if (m == 0) return peqa::gemm_row_tiles(T);
        auto take = [&](double beside, int *to) {
            const int rt = peqa::gemm_plan(m, job, T, gw, false, mode == peqa::MODE_DDS, beside, ~(size_t)0, cus);
            for (int i = 0; i < m; ++i) to[of[i]] = job[i].split;
            return rt;
        };
        if (!gw || mode != peqa::MODE_DX) return take(0.0, split);
        long long dx_tiles = 0, dw_tiles = 0;                  // of dX, and of the token contractions beside it
        for (int i = 0; i < m; ++i) {
            const peqa_layout *L = &items[of[i]].layout;
            dx_tiles += (long long)tiles_t * job[i].tiles_c;
            dw_tiles += (long long)(L->k_in / 128) * ((L->n_out + 255) / 256);
        }
        w.rt_dx_alone = take(0.0, w.split_dx_alone);
        w.many_tiles = !peqa::bwd_few_tiles(dx_tiles + dw_tiles, cus);
        w.one_launch = peqa::bwd_one_launch(dx_tiles + dw_tiles, T, cus);
        int rt = w.rt_dx_alone;
        if (w.one_launch) {
            rt = take(dw_tiles * peqa::dw_tile_us(T), split);
            w.one_launch = !peqa::bwd_dx_chains(m, job, T, cus);
        }
        return rt;
    };
    if (op == PEQA_OP_FWD) {
        w.rt_y[0] = plan(false, peqa::MODE_Y, w.split_y);
        w.rt_y[1] = plan(true, peqa::MODE_Y, w.split_y);
    } else {
        plan(false, peqa::MODE_DDS, w.split_dds);
        w.rt_dx[0] = plan(false, peqa::MODE_DX, w.split_dx);
        w.rt_dx[1] = plan(true, peqa::MODE_DX, w.split_dx);
    }
    lay_out_pieces(w, n, items, T);
    return w;
}

// The regions of a call with a workspace of `bytes`, checked before the device is touched.  Where it is too small for the split
// contractions: whole ones, and group-wise items of many tiles as fit_workspace has it (block of d = 4736, f = 15744 in groups of 128, T = 138,
// shared and whole / launches of their own in pieces 455 / 325 us).
peqa_status plan_block(BlockSpace &w, int32_t n, const peqa_block_item *items, int32_t T, int32_t op, const void *workspace,
                       size_t bytes)
{
    w = carve_block(n, items, T, op, peqa::PLAN_UNITS);
    if (!workspace || bytes < w.min_total) return PEQA_ERR_WORKSPACE;
    if (!aligned16(workspace)) return PEQA_ERR_ALIGN;
    const int cus = peqa::compute_units();
    if (cus != peqa::PLAN_UNITS) w = carve_block(n, items, T, op, cus);      // (min_total does not hang on the units)
    if (bytes < w.total && w.one_launch && w.many_tiles) {
        w.one_launch = false;
        for (int j = 0; j < n; ++j)
            if (grouped(&items[j].layout)) w.split_dx[j] = w.split_dx_alone[j];
        lay_out_pieces(w, n, items, T);
    }
    if (bytes < w.total)
        for (int j = 0; j < n; ++j) w.split_y[j] = w.split_dx[j] = w.split_dds[j] = w.split_dx_alone[j] = 1;
    return PEQA_OK;
}

// A multi-contraction launch, and the sums of its split contractions.
peqa_status launch_multi(int bits, bool gw, peqa::MultiArgs &m, hipStream_t s)
{
    if (peqa::launch_gemm_multi(bits, gw, m, s) != hipSuccess) return PEQA_ERR_DEVICE;
    peqa::FinishMulti f{};
    for (int j = 0; j < m.n_jobs; ++j) {
        if (m.job[j].a.split < 2 || m.job[j].mode == peqa::MODE_DDS) continue;
        f.job[f.n].a = m.job[j].a;
        f.job[f.n++].mode = m.job[j].mode;
    }
    return f.n > 0 ? dev_status(peqa::launch_split_finish(f, s)) : PEQA_OK;
}

int piece_length(const peqa::MultiJob &j) { return j.a.KC / (j.a.split > 1 ? j.a.split : 1); }

// Jobs of a multi-contraction launch in order of falling contraction length (of a piece).
void sort_jobs(peqa::MultiArgs &m)
{
    for (int i = 1; i < m.n_jobs; ++i)
        for (int k = i; k > 0 && piece_length(m.job[k]) > piece_length(m.job[k - 1]); --k) {
            const peqa::MultiJob t = m.job[k];
            m.job[k] = m.job[k - 1];
            m.job[k - 1] = t;
        }
}

// Auxiliary workgroups of a multi-contraction launch: after the first round of tiles (two per compute unit), a
// multiple of 8.  A launch without tiles is made of auxiliary workgroups alone: four per compute unit.
void place_aux(peqa::MultiArgs &m, int aux_wgs)
{
    int total = 0;
    for (int j = 0; j < m.n_jobs; ++j) total += peqa::gemm_multi_wgs(m.job[j].a);
    const int cus = peqa::compute_units();
    const int first_round = 2 * cus / 8 * 8;
    m.aux_begin = total < first_round ? total : first_round;
    if (total == 0) aux_wgs = 4 * cus / 8 * 8;
    m.aux_wgs = (m.n_sdy > 0 || m.n_red > 0 || m.n_tp > 0) ? aux_wgs : 0;
}

// The auxiliary workgroups of a launch whose side work is the scaling of dY.
int launch_scaling_wgs(const peqa::MultiArgs &m)
{
    const int rows = peqa::aux_sdy_rows(m.n_jobs > 0 ? m.job[0].a.rt : 8), places = 2 * peqa::compute_units();
    int blocks = 0, tiles = 0;
    double scaling = 0.0, sum = 0.0, longest = 0.0;
    for (int j = 0; j < m.n_sdy; ++j) {
        const int b = (m.sdy[j].T + rows - 1) / rows;
        blocks += b;
        scaling += b * (2.0 + 1.4 * ((m.sdy[j].N + 2047) / 2048));
    }
    for (int j = 0; j < m.n_jobs; ++j) {
        const int n = peqa::gemm_multi_wgs(m.job[j].a);
        const double us = 8.0 + 0.55 * (piece_length(m.job[j]) / 32);
        tiles += n;
        sum += us * n;
        longest = us > longest ? us : longest;
    }
    return peqa::scaling_wgs(blocks, scaling, tiles, sum / places > longest ? sum / places : longest, places);
}

// Whether dX, in the pieces planned beside the token contractions of every group-wise item, is far from over when the work of those that a call
// asks for is, and a launch of its own has shorter pieces.  Of calls of many tiles that ask for some gradients only (backward, us, launches
// of their own / shared; the longest workgroup over the work by the estimates below): d = 3328, f = 9728 in groups of 64, T = 859, dX
// of the wide items and scale gradients of the others 303 / 343 (2.2), all dX and the scale gradient of q, k, v 353 / 376 (1.9), of q, k, v
// and o 370 / 388 (1.7); the first of d = 3584, f = 12544 in groups of 256, T = 1193 463 / 498 (1.6), of d = 3200, f = 9728 in groups of 128,
// T = 33 66 / 59 (1.4).  Where the pieces are the same, shared: d = 2176, f = 6272, T = 1532 263 / 246 (2.0), d = 5120, f = 13824, T = 700 539 / 505 (1.7).
bool dx_outlasts(int32_t n, const peqa_block_item *items, const BlockSpace &w, int32_t T)
{
    double sum = 0.0, longest = 0.0, alone = 0.0;
    auto us = [](int steps, int rt) { return 8.0 + 0.55 * rt / 8 * steps; };
    for (int j = 0; j < n; ++j) {
        const int N = items[j].layout.n_out, K = items[j].layout.k_in;
        if (!grouped(&items[j].layout)) continue;
        if (items[j].dX) {
            const double piece = us(N / 32 / w.split_dx[j], w.rt_dx[1]), own = us(N / 32 / w.split_dx_alone[j], w.rt_dx_alone);
            sum += piece * peqa::gemm_tiles_t(T, w.rt_dx[1]) * ((K + 255) / 256) * w.split_dx[j];
            longest = piece > longest ? piece : longest;
            alone = own > alone ? own : alone;
        }
        if (items[j].d_ds) sum += peqa::dw_tile_us(T) * (K / 128) * ((N + 255) / 256);
    }
    return longest > 1.6 * sum / (2 * peqa::compute_units()) && alone < 0.6 * longest;
}

// Tables of every group-wise item (of those whose dX is wanted, if only_dx): one launch.
peqa_status group_tables(int32_t n, const peqa_block_item *items, uint8_t *ws, const BlockSpace &w, bool only_dx,
                         hipStream_t s)
{
    peqa::GroupTableMulti gt{};
    for (int j = 0; j < n; ++j) {
        const peqa_block_item &it = items[j];
        if (!grouped(&it.layout) || (only_dx && !it.dX)) continue;
        const int i = gt.n++;
        gt.s0[i] = it.s0; gt.ds[i] = it.ds; gt.z0[i] = it.z0;
        gt.sb[i] = reinterpret_cast<float *>(ws + w.table[j]);
        gt.N[i] = it.layout.n_out; gt.G[i] = groups(&it.layout);
    }
    if (gt.n == 0) return PEQA_OK;
    for (int i = gt.n; i < peqa::GT_MAX; ++i) {
        gt.s0[i] = gt.s0[0]; gt.ds[i] = gt.ds[0]; gt.z0[i] = gt.z0[0]; gt.sb[i] = gt.sb[0]; gt.N[i] = gt.N[0]; gt.G[i] = gt.G[0];
    }
    return dev_status(peqa::launch_group_table_multi(gt, s));
}

}  // namespace

extern "C" {

size_t peqa_block_workspace_bytes(int32_t n, const peqa_block_item *items, int32_t T, int32_t op)
{
    if (check_items(n, items, T) != PEQA_OK) return 0;
    if (op != PEQA_OP_FWD && op != PEQA_OP_BWD) return 0;
    if (op == PEQA_OP_FWD && T <= GEMV_MAX_T) {
        GemvItem gi[PEQA_MAX_BLOCK]{};
        for (int j = 0; j < n; ++j) gi[j].L = &items[j].layout;
        const size_t b = round256(gemv_partial_bytes(n, gi, T, true, GEMV_ANY, peqa::PLAN_UNITS));
        return b ? b : 256;
    }
    return carve_block(n, items, T, op, peqa::PLAN_UNITS).total;
}

peqa_status peqa_block_fwd(int32_t n, const peqa_block_item *items, int32_t T, void *workspace,
                           size_t workspace_bytes, void *stream)
{
    peqa_status st = check_items(n, items, T);
    if (st != PEQA_OK) return st;
    for (int j = 0; j < n; ++j) {
        const peqa_block_item &it = items[j];
        if (!it.packed || !it.s0 || !it.z0 || !it.X || !it.Y) return PEQA_ERR_NULL;
        if (!aligned16(it.packed) || !aligned16(it.s0) || !aligned16(it.z0) || !aligned16(it.X) || !aligned16(it.Y) ||
            (it.ds && !aligned16(it.ds)) || (it.row_sums && !aligned16(it.row_sums)))
            return PEQA_ERR_ALIGN;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    uint8_t *ws = static_cast<uint8_t *>(workspace);

    if (T <= GEMV_MAX_T) {
        GemvItem gi[PEQA_MAX_BLOCK];
        for (int j = 0; j < n; ++j)
            gi[j] = GemvItem{&items[j].layout, items[j].packed, items[j].s0, items[j].ds, items[j].z0, nullptr,
                             items[j].X, items[j].Y};
        const size_t least = round256(gemv_partial_bytes(n, gi, T, true, 0, peqa::PLAN_UNITS));
        if (!workspace || workspace_bytes < (least ? least : 256)) return PEQA_ERR_WORKSPACE;
        if (!aligned16(workspace)) return PEQA_ERR_ALIGN;
        return gemv_forward(n, gi, T, GEMV_ANY, reinterpret_cast<float *>(ws), workspace_bytes, s);
    }

    BlockSpace w;
    st = plan_block(w, n, items, T, PEQA_OP_FWD, workspace, workspace_bytes);
    if (st != PEQA_OK) return st;
    int xi[PEQA_MAX_BLOCK], ks[PEQA_MAX_BLOCK];
    const uint16_t *xs[PEQA_MAX_BLOCK];
    const int nx = distinct_inputs(n, items, xi, xs, ks);
    const int bits = items[0].layout.bits;
    // row sums of every distinct input of the per-channel items, into each array that its items bring: one launch
    const float *rs[PEQA_MAX_BLOCK] = {nullptr};
    {
        peqa::RowsumMulti r{};
        int nr = 0;
        for (int i = 0; i < nx; ++i) {
            const int first = nr;                              // this input's entries (at most one per item in all)
            auto take = [&](float *dst) {
                for (int e = first; e < nr; ++e)
                    if (r.rs[e] == dst) return;
                r.X[nr] = xs[i]; r.K[nr] = ks[i]; r.rs[nr++] = dst;
            };
            float *own = nullptr;
            for (int j = 0; j < n; ++j) {
                if (xi[j] != i || grouped(&items[j].layout)) continue;
                if (!own) own = reinterpret_cast<float *>(ws + w.rs[j]);
                if (items[j].row_sums) take(items[j].row_sums);
            }
            if (!own) continue;
            if (nr == first) take(own);
            rs[i] = r.rs[first];
        }
        if (nr > 0) {
            for (int i = nr; i < peqa::ROWSUM_MAX; ++i) { r.X[i] = r.X[nr - 1]; r.K[i] = r.K[nr - 1]; r.rs[i] = r.rs[nr - 1]; }
            r.n = nr; r.T = T;
            if (peqa::launch_rowsum_multi(r, s) != hipSuccess) return PEQA_ERR_DEVICE;
        }
    }
    st = group_tables(n, items, ws, w, false, s);
    if (st != PEQA_OK) return st;
    // all per-channel contractions in one launch, all group-wise ones in another
    peqa::MultiArgs m{}, mg{};
    for (int j = 0; j < n; ++j) {
        const peqa_block_item &it = items[j];
        const int N = it.layout.n_out, K = it.layout.k_in;
        const bool gw = grouped(&it.layout);
        peqa::MultiArgs &dst = gw ? mg : m;
        peqa::MultiJob &job = dst.job[dst.n_jobs++];
        job.mode = peqa::MODE_Y;
        peqa::GemmArgs &a = job.a;
        a.packed = it.packed; a.A = it.X; a.T = T; a.KC = K; a.C = N; a.K = K;
        a.rt = w.rt_y[gw]; a.tiles_c = (N + 255) / 256; a.tiles_t = peqa::gemm_tiles_t(T, a.rt);
        a.out = it.Y;
        a.split = w.split_y[j]; a.acc_part = reinterpret_cast<float *>(ws + w.acc[j]);
        if (gw) {
            a.N = N; a.gsz = it.layout.group_size; a.G = groups(&it.layout);
            a.sb = reinterpret_cast<const float *>(ws + w.table[j]);
        } else {
            a.s0 = it.s0; a.ds = it.ds; a.z0 = it.z0; a.rs = rs[xi[j]];
        }
    }
    if (m.n_jobs > 0) {
        sort_jobs(m);
        place_aux(m, 0);
        st = launch_multi(bits, false, m, s);
        if (st != PEQA_OK) return st;
    }
    if (mg.n_jobs > 0) {
        sort_jobs(mg);
        place_aux(mg, 0);
        st = launch_multi(bits, true, mg, s);
        if (st != PEQA_OK) return st;
    }
    return PEQA_OK;
}

peqa_status peqa_block_bwd(int32_t n, const peqa_block_item *items, int32_t T, void *workspace,
                           size_t workspace_bytes, void *stream)
{
    peqa_status st = check_items(n, items, T);
    if (st != PEQA_OK) return st;
    for (int j = 0; j < n; ++j) {
        const peqa_block_item &it = items[j];
        if (!it.packed || !it.s0 || !it.z0 || !it.dY) return PEQA_ERR_NULL;
        if (it.d_ds && !it.X) return PEQA_ERR_NULL;
        if (!aligned16(it.packed) || !aligned16(it.s0) || !aligned16(it.z0) || !aligned16(it.dY) ||
            (it.X && !aligned16(it.X)) || (it.ds && !aligned16(it.ds)) || (it.dX && !aligned16(it.dX)) ||
            (it.d_ds && !aligned16(it.d_ds)) || (it.row_sums && !aligned16(it.row_sums)))
            return PEQA_ERR_ALIGN;
    }
    BlockSpace w;
    st = plan_block(w, n, items, T, PEQA_OP_BWD, workspace, workspace_bytes);
    if (st != PEQA_OK) return st;
    uint8_t *ws = static_cast<uint8_t *>(workspace);
    hipStream_t s = static_cast<hipStream_t>(stream);
    int xi[PEQA_MAX_BLOCK], ks[PEQA_MAX_BLOCK];
    const uint16_t *xs[PEQA_MAX_BLOCK];
    const int nx = distinct_inputs(n, items, xi, xs, ks);
    const int tiles_t = (T + 127) / 128, Tp = (T + 63) / 64 * 64;
    const int bits = items[0].layout.bits;

    // ---- per-channel items.  Row sums of the inputs whose scale gradient is wanted: the caller's (kept from the
    // forward, which stores none at T <= 16), else taken here, all in one launch.
    const float *rs[PEQA_MAX_BLOCK] = {nullptr};
    {
        peqa::RowsumMulti r{};
        int nr = 0;
        for (int i = 0; i < nx; ++i) {
            bool wanted = false;
            const float *have = nullptr;
            float *dst = nullptr;
            for (int j = 0; j < n; ++j)
                if (xi[j] == i && !grouped(&items[j].layout)) {
                    wanted = wanted || (items[j].d_ds != nullptr && w.split_dds[j] == 1);   // pieces take their own
                    if (items[j].row_sums && T > GEMV_MAX_T) have = items[j].row_sums;
                    if (!dst) dst = reinterpret_cast<float *>(ws + w.rs[j]);
                }
            if (have || !wanted) { rs[i] = have; continue; }
            r.X[nr] = xs[i]; r.K[nr] = ks[i]; r.rs[nr] = dst;
            ++nr;
            rs[i] = dst;
        }
        if (nr > 0) {
            for (int i = nr; i < peqa::ROWSUM_MAX; ++i) { r.X[i] = r.X[nr - 1]; r.K[i] = r.K[nr - 1]; r.rs[i] = r.rs[nr - 1]; }
            r.n = nr; r.T = T;
            if (peqa::launch_rowsum_multi(r, s) != hipSuccess) return PEQA_ERR_DEVICE;
        }
    }
    // First launch: every scale-gradient contraction, and in its auxiliary workgroups the scaling of dY for every
    // dX contraction.  Second launch: every dX contraction, and the fixed-order sums of the first launch's partials.
    peqa::MultiArgs ma{}, mb{};
    int red_chunks = 0;
    for (int j = 0; j < n; ++j) {
        const peqa_block_item &it = items[j];
        if (grouped(&it.layout)) continue;
        const int N = it.layout.n_out, K = it.layout.k_in;
        uint16_t *dys = reinterpret_cast<uint16_t *>(ws + w.dys[j]);
        float *crow = reinterpret_cast<float *>(ws + w.crow[j]);
        float *partial = reinterpret_cast<float *>(ws + (w.split_dds[j] > 1 ? w.acc_dds[j] : w.partial[j]));
        const int partial_rows = tiles_t * w.split_dds[j];
        if (it.d_ds && partial_rows == 1) partial = it.d_ds;   // one row of partials is the gradient
        if (it.d_ds) {
            peqa::MultiJob &job = ma.job[ma.n_jobs++];
            job.mode = peqa::MODE_DDS;
            peqa::GemmArgs &a = job.a;
            a.packed = it.packed; a.A = it.X; a.T = T; a.KC = K; a.C = N; a.K = K;
            a.rt = peqa::gemm_row_tiles(T); a.tiles_c = (N + 255) / 256; a.tiles_t = tiles_t;
            a.z0 = it.z0; a.rs = rs[xi[j]]; a.dY = it.dY; a.partial = partial;
            a.split = w.split_dds[j];
            if (partial_rows > 1) {
                peqa::ReduceJob &r = mb.red[mb.n_red++];
                r.partial = partial; r.out = it.d_ds; r.ntiles = partial_rows; r.n = N;
                red_chunks += (N + 255) / 256;
                r.chunk_end = red_chunks;
            }
        }
        if (it.dX) {
            peqa::ScaleDyJob &sd = ma.sdy[ma.n_sdy++];
            sd.dY = it.dY; sd.s0 = it.s0; sd.ds = it.ds; sd.z0 = it.z0; sd.dYs = dys; sd.crow = crow; sd.T = T; sd.N = N;
            peqa::MultiJob &job = mb.job[mb.n_jobs++];
            job.mode = peqa::MODE_DX;
            peqa::GemmArgs &a = job.a;
            a.packed = it.packed; a.A = dys; a.T = T; a.KC = N; a.C = K; a.K = K;
            a.rt = w.rt_dx[0]; a.tiles_c = (K + 255) / 256; a.tiles_t = peqa::gemm_tiles_t(T, a.rt);
            a.crow = crow; a.out = it.dX;
            a.split = w.split_dx[j]; a.acc_part = reinterpret_cast<float *>(ws + w.acc[j]);
        }
    }
    if (ma.n_jobs > 0 || ma.n_sdy > 0) {
        sort_jobs(ma);
        place_aux(ma, launch_scaling_wgs(ma));
        st = launch_multi(bits, false, ma, s);
        if (st != PEQA_OK) return st;
    }
    if (mb.n_jobs > 0 || mb.n_red > 0) {
        sort_jobs(mb);
        place_aux(mb, 64);
        st = launch_multi(bits, false, mb, s);
        if (st != PEQA_OK) return st;
    }

    // ---- group-wise items.  Few tiles or tokens (bwd_one_launch) and both gradients: the (s, b) tables and the transposed copies of X (once per distinct
    // input) and dY in one launch, dX and the token contractions of the scale gradients in the next, pieces and chunks added up in
    // the last.  Otherwise the tables in one launch; every dX contraction in one launch, whose auxiliary workgroups write the copies;
    // the token contractions in one launch; the sums of their chunks in one launch.
    bool want_dx = false, want_dds = false;
    for (int j = 0; j < n; ++j)
        if (grouped(&items[j].layout)) {
            want_dx = want_dx || items[j].dX;
            want_dds = want_dds || items[j].d_ds;
        }
    const bool one_launch = want_dx && want_dds && w.one_launch && !(w.many_tiles && dx_outlasts(n, items, w, T));
    peqa::MultiArgs mg{};
    peqa::DwMultiArgs dw{};
    const uint16_t *xt_of[PEQA_MAX_BLOCK] = {nullptr};
    int tp_tiles = 0;
    for (int j = 0; j < n; ++j) {
        const peqa_block_item &it = items[j];
        if (!grouped(&it.layout)) continue;
        const int N = it.layout.n_out, K = it.layout.k_in, G = groups(&it.layout);
        if (it.dX) {
            peqa::MultiJob &job = mg.job[mg.n_jobs++];
            job.mode = peqa::MODE_DX;
            peqa::GemmArgs &a = job.a;
            a.packed = it.packed; a.A = it.dY; a.T = T; a.KC = N; a.C = K; a.K = K;
            a.rt = one_launch ? w.rt_dx[1] : w.rt_dx_alone;
            a.tiles_c = (K + 255) / 256; a.tiles_t = peqa::gemm_tiles_t(T, a.rt);
            a.N = N; a.gsz = it.layout.group_size; a.G = G;
            a.sb = reinterpret_cast<const float *>(ws + w.table[j]); a.out = it.dX;
            a.split = one_launch ? w.split_dx[j] : w.split_dx_alone[j];
            a.acc_part = reinterpret_cast<float *>(ws + w.acc[j]);
        }
        if (it.d_ds) {
            if (!xt_of[xi[j]]) {
                uint16_t *xt = reinterpret_cast<uint16_t *>(ws + w.xt[j]);
                peqa::TransposeJob &t = mg.tp[mg.n_tp++];
                t.src = it.X; t.dst = xt; t.T = T; t.C = K; t.Tp = Tp;
                tp_tiles += (Tp / 64) * (K / 64);
                t.tile_end = tp_tiles;
                xt_of[xi[j]] = xt;
            }
            uint16_t *dyt = reinterpret_cast<uint16_t *>(ws + w.dyt[j]);
            peqa::TransposeJob &t = mg.tp[mg.n_tp++];
            t.src = it.dY; t.dst = dyt; t.T = T; t.C = N; t.Tp = Tp;
            tp_tiles += (Tp / 64) * (N / 64);
            t.tile_end = tp_tiles;
            peqa::DwArgs &a = dw.job[dw.n_jobs];
            a.Xt = xt_of[xi[j]]; a.dYt = dyt; a.packed = it.packed; a.z0 = it.z0;
            a.pc = peqa::dw_whole_groups(it.layout.group_size) ? it.d_ds : reinterpret_cast<float *>(ws + w.pc[j]);
            a.N = N; a.K = K; a.Tp = Tp; a.gsz = it.layout.group_size; a.G = G;
            a.tiles_f = K / 128; a.tiles_c = (N + 255) / 256;
            dw.d_ds[dw.n_jobs++] = it.d_ds;
        }
    }
    if (one_launch) {
        peqa::GroupPrep p{};
        for (int j = 0; j < n; ++j) {
            const peqa_block_item &it = items[j];
            if (!grouped(&it.layout) || !it.dX) continue;
            const int i = p.table.n++;
            p.table.s0[i] = it.s0; p.table.ds[i] = it.ds; p.table.z0[i] = it.z0;
            p.table.sb[i] = reinterpret_cast<float *>(ws + w.table[j]);
            p.table.N[i] = it.layout.n_out; p.table.G[i] = groups(&it.layout);
        }
        for (int i = 0; i < mg.n_tp; ++i) p.tp[i] = mg.tp[i];
        p.n_tp = mg.n_tp;
        if (peqa::launch_group_prep(p, s) != hipSuccess) return PEQA_ERR_DEVICE;
        sort_jobs(mg);
        peqa::GemmDwArgs m{};
        for (int i = 0; i < mg.n_jobs; ++i) m.job[i] = mg.job[i];
        for (int i = 0; i < dw.n_jobs; ++i) m.dw[i] = dw.job[i];
        m.n_jobs = mg.n_jobs; m.n_dw = dw.n_jobs;
        if (peqa::launch_gemm_dw(bits, m, s) != hipSuccess) return PEQA_ERR_DEVICE;
        peqa::FinishMulti f{};
        for (int i = 0; i < mg.n_jobs; ++i)
            if (mg.job[i].a.split > 1) f.job[f.n++] = peqa::FinishJob{m.job[i].a, peqa::MODE_DX};
        for (int i = 0; i < dw.n_jobs; ++i)
            if (!peqa::dw_whole_groups(dw.job[i].gsz))
                f.sum[f.n_sums++] = peqa::chunk_sums(dw.job[i].pc, dw.d_ds[i], dw.job[i].N, dw.job[i].K, dw.job[i].gsz);
        return dev_status(peqa::launch_split_finish(f, s));
    }
    st = group_tables(n, items, ws, w, true, s);
    if (st != PEQA_OK) return st;
    if (mg.n_jobs > 0 || mg.n_tp > 0) {
        sort_jobs(mg);
        place_aux(mg, 128);
        st = launch_multi(bits, true, mg, s);
        if (st != PEQA_OK) return st;
    }
    if (dw.n_jobs > 0) {
        if (peqa::launch_dw_multi(bits, dw, s) != hipSuccess) return PEQA_ERR_DEVICE;
        if (peqa::launch_chunk_reduce_multi(dw, s) != hipSuccess) return PEQA_ERR_DEVICE;
    }
    return PEQA_OK;
}

}  // extern "C"

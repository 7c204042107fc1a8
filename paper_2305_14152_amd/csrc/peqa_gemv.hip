// Deployment forward for T <= 16 tokens (Sec. 3.1 "Inference Latency": matrix-vector products bound
// by the weight bytes streamed from memory).  Y[t,i] = sum_g s[i,g] * sum_{k in g} X[t,k] (Q[i,k] - z[i,g]).
//
// Every packed word is read from HBM exactly once: a wave owns 64 output channels (lane (c, q):
// half of channel block c / 2, feature block q of each 32-feature step) -- or two such halves of 128 -- and walks a range of
// the input features; the up-to-16 token rows ride along as the 16-row operand of MFMA 16x16x32, so T = 1 and T = 16 cost
// the same weight traffic.  Codes enter the MFMAs as exact bf16 (16 + Q); one more MFMA per step against a fragment of ones
// yields the row sums of X over the same features, and at the end of every scale group   y += s * (acc - (16 + z) * rowsum)
// folds offset, zero-point and scale in fp32.  Per-channel layers are one group spanning the whole range.
//
// Grid: one workgroup per (layer, channel tile, feature slice); up to GEMV_MAX_LAYERS layers of different shapes and inputs
// share a launch (a decoder block's linears: a single LLaMA-size layer at such T is too short to fill the machine, and a
// launch costs as much as streaming several megabytes).  The K / 64 rounds of 64 features of a tile are dealt evenly to its
// S slices and, inside a slice, to the waves of the workgroup (a wave may start or stop in the middle of a scale group: the
// fold above is linear in the features, so it is applied to whatever part of a group the wave has seen); the waves are
// summed through LDS at the end.  S > 1 leaves fp32 partials [S, T, N] in the workspace for gemv_finish_kernel to add up in
// a fixed order, a second launch of 4 us.  Waves per workgroup, channels and slices: see gemv_plan.
//
// What bounds it.  HBM for a whole block (4.7 TB/s of the 4.8 to 5.2 that a copy or a read reaches), latency and the second
// launch for single layers, and below one workgroup per compute unit the unpacking (2 vector instructions per weight pair).
// Tiles of 64 channels instead of 128 need no slices where 128 needed two to six, i.e. no second launch, and put twice the
// workgroups behind a layer.  us per call at T = 5, 128 channels -> this form: 13B 3-bit g128 qkv 18.3 -> 11.9, o 13.7 -> 10.4,
// gate/up 22.7 -> 18.1, down 18.9 -> 14.5, whole block 36.1 -> 34.6; 7B 4-bit qkv 14.2 -> 9.3, o 11.4 -> 8.1, gate/up 18.4 -> 13.6,
// down 15.1 -> 11.8, whole block 29.5 -> 26.3.  What is read and written besides the DMAs goes by global instructions: with FLAT ones
// (the pointers come out of the argument block) every use of a part of the scale tile waited for all of memory (four 7B blocks, T = 1
// 91.4 -> 87.9 us, two 13B blocks, T = 16 72.0 -> 70.5).  Three rounds in flight instead of two cost 3 % (places on the unit).
//
// A wave moves its operands in rounds of 64 features (two MFMA steps): its packed words and the matching 128 bytes of each
// token row, by global -> LDS DMA into a private double buffer, from which each lane reads back its own words and
// activation fragments (token rows' 16-byte chunks XOR-swizzled by row, so that the reads of 16 rows spread over the
// banks).  No barrier is involved: a wave waits for its own DMA only.
#include <stddef.h>

#include <type_traits>

#include "peqa_device.h"
#include "peqa_kernels.h"

namespace peqa {

namespace {

// A workgroup owns 64 H channels (H = 1 or 2), or 32 (H = 0, T <= 8).
constexpr int gv_channels(int h) { return h == 0 ? 32 : 64 * h; }
constexpr int gv_srow(int h) { return gv_channels(h) + 4; }   // padded rows of the scale tile (floats) and of byte zero-points
constexpr int gv_zrow(int h) { return gv_channels(h) + 8; }
constexpr int GV_LDS_MAX = 160 * 1024;
constexpr int GV_SIMD_WAVES = 4;     // waves per SIMD that the registers of every form allow: the plan counts on them
// Rounds a wave keeps in flight (64 channels and more: three measured the same or slower).
constexpr int gv_nbuf(int h) { return h == 0 ? 4 : 2; }
// One round (64 features) of one wave in LDS: its packed words (2 KB per 64 channels; 1.5 KB of it at 3 bits), then NX KB of
// token rows (8 rows x 128 B per KB: one DMA when T <= 8, two otherwise).
constexpr int GV_B_BYTES = 2048;
constexpr int gv_round_bytes(int h, int nx) { return gv_channels(h) * (GV_B_BYTES / 64) + nx * 1024; }
// Bytes of LDS per scale group of a workgroup's tile: 64 scales, and 64 zero-points as bytes or, with a trained offset, fp32.
constexpr int gv_group_bytes(int h, bool zbyte) { return gv_srow(h) * 4 + (zbyte ? gv_zrow(h) : gv_srow(h) * 4); }

__device__ __forceinline__ void gv_dma16(uint32_t voff, const void *sbase, uint32_t lds_dst)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :: "v"(voff), "s"(sbase), "s"(lds_dst) : "memory");
}
template <int N>
__device__ __forceinline__ void gv_wait_vmcnt()
{
    __builtin_amdgcn_s_waitcnt((N & 0xF) | (0x7 << 4) | (0xF << 8) | ((N >> 4) << 14));
}

// H: 64-channel halves of a workgroup (0: half of one).  NX: KB of token rows per round (1: T <= 8, 2: T <= 16).
//
// H = 0: with at most 8 tokens, half of an MFMA's 16 rows would be padding.  Lanes c < 8 unpack the 8 half blocks of 32 channels for
// features 0..31 of a round, lanes c >= 8 those for features 32..63, and rows 8..15 of the other operand are the same tokens'
// features 32..63: of the product, rows 0..7 of columns c < 8 and rows 8..15 of columns c >= 8 are wanted (lanes (c, q) with
// q / 2 = c / 8) and added up at the end, the rest is ignored.  As much unpacking per weight in workgroups half as large: for layers
// of few channels, which the unpacking bounds on the compute units that they reach.
// ZBYTE: zero-points are the stored integers (no trained offset dz), kept as bytes in LDS.
template <int BITS, int H, int WAVES, int NX, bool ZBYTE>
__device__ __forceinline__ void gemv_tile(const GemvArgs &a, const GemvLayer &L, const int bx, const int wg0, uint8_t *stage)
{
    // [wave][ring slot][round]; then the scale tile: scale s0 + ds and zero-point (16 + z0 + dz as fp32, or z0 as stored) of
    // [group of the slice][channel] (rows padded: the transposing writes of consecutive groups of one channel then fall into
    // different banks); in the end all of it is [wave][column tile][row in lane][lane] fp32 (4 KB per wave) for the final sum
    // (not pinned: the compiler places the unpacking and the matrix instructions, and the wait states between them)
    typedef HalfBlockUnpacker<BITS, false, kFieldBf16, false> Unpacker;
    constexpr int WORDS = Unpacker::WORDS;
    constexpr bool SMALL = H == 0;
    constexpr int HH = SMALL ? 1 : H;                             // 16-column accumulators: 4 HH
    constexpr int NBUF = gv_nbuf(H), ROUND = gv_round_bytes(H, NX), NDMA = (SMALL ? 1 : 2 * H) + NX, THREADS = WAVES * 64;
    const int nbuf = SMALL ? L.form & GEMV_DEPTH : NBUF;                      // slots of the ring
    constexpr int X_AT = ROUND - NX * 1024;                       // token rows behind the packed words
    constexpr int GV_C = gv_channels(H), GV_SROW = gv_srow(H), GV_ZROW = gv_zrow(H);
    static_assert(NBUF == 2 || NBUF == 4, "the waits below");
    static_assert(!SMALL || NX == 1, "32 channels: T <= 8");
    typedef typename std::conditional<ZBYTE, uint8_t, float>::type zp_t;
    constexpr int ZROW = ZBYTE ? GV_ZROW : GV_SROW;
    float *sS = reinterpret_cast<float *>(stage + WAVES * nbuf * ROUND);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, q = lane >> 4;
    const int hb = SMALL ? c & 7 : c;                             // the lane's half block within 64 (32) channels
    const float *l_s0 = L.s0, *l_ds = L.ds, *l_dz = L.dz;
    const uint8_t *l_z0 = L.z0;
    const int l_N = L.N, l_S = L.S;
    const Quotient ts = div_magic((uint32_t)(bx - wg0), (uint32_t)l_S, L.s_magic);
    const int slice = (int)ts.r;
    const int n0 = (int)ts.q * GV_C;                             // first channel, within its layer
    const int K = L.K, G = L.G;
    const int chunk_rounds = L.chunk_rounds;                      // 64-feature rounds per scale group
    // this workgroup's rounds [rbeg, rend); wave w takes the w-th of WAVES equal parts of them
    const int rbeg = slice * L.slice_rounds + (slice < L.slice_rem ? slice : L.slice_rem);
    const int len = L.slice_rounds + (slice < L.slice_rem ? 1 : 0), rend = rbeg + len;
    const int wr0 = rbeg + (int)((uint32_t)(wave * len) / (uint32_t)WAVES);
    const int nrounds = rbeg + (int)((uint32_t)((wave + 1) * len) / (uint32_t)WAVES) - wr0;
    const int g_lo = (int)div_magic((uint32_t)rbeg, (uint32_t)chunk_rounds, L.chunk_magic).q;   // first scale group touched

    uint32_t magic = kMagic;
    asm("" : "+v"(magic));                                      // in a register: as a constant, and-or takes two instructions
    const u32x4 ones = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
    // A step of the wave (64 channels x 32 features) is half of a 128-channel tile of TILE bytes: contiguous; tiles follow
    // each other along the features.
    constexpr uint32_t BLK = 2 * BITS * 4, TILE = 64 * BLK, HALF = TILE / 2;
    const uint8_t *bsrc = reinterpret_cast<const uint8_t *>(L.packed) +
                          ((size_t)(n0 >> 7) * (K >> 5) + 2 * (size_t)wr0) * TILE +
                          (SMALL ? (size_t)((n0 >> 5) & 3) * (HALF / 2) : (size_t)((n0 >> 6) & 1) * HALF);
    const uint8_t *xsrc = reinterpret_cast<const uint8_t *>(L.X + ((size_t)wr0 << 6));
    const uint32_t ring = (uint32_t)(uintptr_t)stage + wave * nbuf * ROUND;
    uint32_t b_voff[2], x_voff[NX];
    if constexpr (SMALL) {
        // one DMA: 4 bits, lane (c, q) its own words, half hb % 2 of block (hb / 2, q) of the tile of its features; 3 bits, the 48
        // chunks of the two tiles in address order (the last 16 lanes repeat some into the buffer's unused tail)
        const int x = lane < 48 ? lane : lane - 16;
        b_voff[0] = BITS == 4 ? (uint32_t)(c >> 3) * TILE + (uint32_t)((hb >> 1) * 4 + q) * BLK + (uint32_t)(hb & 1) * 16u
                              : (uint32_t)(x / 24) * TILE + (uint32_t)(x % 24) * 16u;
        b_voff[1] = 0;
    } else if constexpr (BITS == 4) {
        // DMA of step s: lane (c, q) fetches its own words, half c % 2 of block (c / 2, q)
#pragma unroll
        for (int i = 0; i < 2; ++i) b_voff[i] = (uint32_t)i * TILE + (uint32_t)((c >> 1) * 4 + q) * BLK + (uint32_t)(c & 1) * 16u;
    } else {
        // the 96 16-byte chunks of the round's two steps in address order (the last 32 lanes repeat the second DMA's first 32
        // into the buffer's unused tail)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int x = 64 * i + (i == 0 ? lane : lane & 31);
            b_voff[i] = (uint32_t)(x / 48) * TILE + (uint32_t)(x % 48) * 16u;
        }
    }
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        const int x = 64 * i + lane, row = x >> 3;                // token row x / 8; its eight 16-byte chunks XOR-swizzled by row
        const int t = row < a.T ? row : a.T - 1;                  // rows beyond T repeat the last one (never stored)
        x_voff[i] = (uint32_t)t * (uint32_t)K * 2u + (uint32_t)((x & 7) ^ (row & 7)) * 16u;
    }
    // round r lives in ring slot r % nbuf; `slot` is the slot of the next round to be issued
    int issued = 0, slot = 0;
    auto issue_round = [&]() {
        const uint32_t dst = ring + slot * ROUND;
        if constexpr (SMALL) gv_dma16(b_voff[0], bsrc, dst);
#pragma unroll
        for (int h = 0; h < H; ++h) {
            gv_dma16(b_voff[0], bsrc + h * HALF, dst + h * GV_B_BYTES);
            gv_dma16(b_voff[1], bsrc + h * HALF, dst + h * GV_B_BYTES + 1024);
        }
#pragma unroll
        for (int i = 0; i < NX; ++i) gv_dma16(x_voff[i], xsrc, dst + X_AT + i * 1024);
        bsrc += 2 * TILE;
        xsrc += 128;
        ++issued;
        slot = slot + 1 == nbuf ? 0 : slot + 1;
    };
#pragma unroll
    for (int i = 0; i < NBUF; ++i)
        if (i < nrounds && (i < 2 || i < nbuf)) issue_round();

    // scale / zero-point tile of the slice: [groups touched][64 channels], transposed on the way into LDS (memory has a
    // channel's groups next to each other).  Channels are laid down so that a lane's four are neighbours.
    const int cols = rend > rbeg ? (int)div_magic((uint32_t)(rend - 1), (uint32_t)chunk_rounds, L.chunk_magic).q - g_lo + 1 : 1;
    zp_t *sZ = reinterpret_cast<zp_t *>(sS + cols * GV_SROW);
    auto store_entry = [&](int jj, int ch, float sv, uint32_t zv, float dzv) {
        const int pos = Unpacker::BY_PARITY ? (ch & ~7) + 4 * (ch & 1) + ((ch & 7) >> 1) : ch;
        sS[jj * GV_SROW + pos] = sv;
        if constexpr (ZBYTE) sZ[jj * ZROW + pos] = (uint8_t)zv;
        else sZ[jj * ZROW + pos] = kCodeOffset + (float)zv + dzv;
    };
    const float inv_cols = __builtin_amdgcn_rcpf((float)cols);    // (entry + 0.5) / cols in fp32: the entry's channel, exactly,
                                                                  // at one unit in the last place off: entries are below 2^16
    if (cols == G && (G & 3) == 0) {
        // whole rows of a multiple of four groups: one contiguous run of 64 G entries, four at a time (16 bytes of s0 and of
        // ds, 4 bytes of z0), the loads of a batch issued together (indices clamped instead of branching)
        const size_t base = (size_t)n0 * G;
        auto batch = [&](int e0, auto nb_c) {
            constexpr int NB = decltype(nb_c)::value;
            f32x4 ts[NB], td[NB], tdz[NB];
            uint32_t tz[NB];
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                int e = e0 + 4 * (tid + i * THREADS);
                e = e < GV_C * cols ? e : 0;
                ts[i] = global_load<f32x4>(l_s0 + base + e);
                tz[i] = global_load<uint32_t>(l_z0 + base + e);
                td[i] = l_ds ? global_load<f32x4>(l_ds + base + e) : f32x4{0.f, 0.f, 0.f, 0.f};
                if constexpr (!ZBYTE) tdz[i] = l_dz ? global_load<f32x4>(l_dz + base + e) : f32x4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const int e = e0 + 4 * (tid + i * THREADS);
                if (e < GV_C * cols) {
                    const int ch = (int)(((float)e + 0.5f) * inv_cols), j = e - ch * cols;   // (a quad stays within a channel)
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        store_entry(j + u, ch, ts[i][u] + td[i][u], (tz[i] >> (8 * u)) & 0xFFu, ZBYTE ? 0.f : tdz[i][u]);
                }
            }
        };
        if (GV_C * cols <= 4 * THREADS) batch(0, std::integral_constant<int, 1>{});
        else if (GV_C * cols <= 12 * THREADS) batch(0, std::integral_constant<int, 3>{});
        else
            for (int e0 = 0; e0 < GV_C * cols; e0 += 28 * THREADS) batch(e0, std::integral_constant<int, 7>{});
    } else {
        auto batch = [&](int e0, auto nb_c) {
            constexpr int NB = decltype(nb_c)::value;             // entries per thread
            float ts[NB], td[NB], tdz[NB];
            uint8_t tz[NB];
            int ch[NB], jj[NB];
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                int e = e0 + tid + i * THREADS;
                e = e < GV_C * cols ? e : 0;
                ch[i] = (int)(((float)e + 0.5f) * inv_cols);
                jj[i] = e - ch[i] * cols;
                const size_t si = (size_t)(n0 + ch[i]) * G + g_lo + jj[i];
                ts[i] = global_load<float>(l_s0 + si);
                tz[i] = global_load<uint8_t>(l_z0 + si);
                td[i] = l_ds ? global_load<float>(l_ds + si) : 0.f;
                if constexpr (!ZBYTE) tdz[i] = l_dz ? global_load<float>(l_dz + si) : 0.f;
            }
#pragma unroll
            for (int i = 0; i < NB; ++i)
                if (e0 + tid + i * THREADS < GV_C * cols) store_entry(jj[i], ch[i], ts[i] + td[i], tz[i], ZBYTE ? 0.f : tdz[i]);
        };
        if (GV_C * cols <= THREADS) batch(0, std::integral_constant<int, 1>{});
        else
            for (int e0 = 0; e0 < GV_C * cols; e0 += 8 * THREADS) batch(e0, std::integral_constant<int, 8>{});
    }
    __syncthreads();

    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 y[4 * HH], acc[4 * HH], accrs = zero;
#pragma unroll
    for (int ct = 0; ct < 4 * HH; ++ct) { y[ct] = zero; acc[ct] = zero; }

    // this lane's words and activation fragment of step 0 within a round (step 1: STEP_B bytes on; chunk 4 + q)
    constexpr int STEP_B = BITS == 4 ? 1024 : 768;
    const uint8_t *b_lane = stage + wave * nbuf * ROUND +
                            (BITS == 4 ? lane * 16 : (SMALL ? (c >> 3) * 384 : 0) + ((hb >> 1) * 4 + q) * 24 + 4 * (c & 1));
    // token row of this lane's activation fragment; with 8 rows staged, rows 8..15 (beyond T, never stored) read rows 0..7
    const uint8_t *x_lane = stage + wave * nbuf * ROUND + X_AT + (NX == 2 ? c : (c & 7)) * 128;
    const int x_pos[2] = {((SMALL ? 4 * (c >> 3) + q : q) ^ (c & 7)) * 16, ((4 + q) ^ (c & 7)) * 16};
    const Quotient wg = div_magic((uint32_t)wr0, (uint32_t)chunk_rounds, L.chunk_magic);
    int group_left = chunk_rounds - (int)wg.r;                    // rounds to the end of the scale group
    int gj = (int)wg.q - g_lo;                                    // its column of the tile
    uint32_t rd = 0;                                              // ring offset of the round being consumed
    // Workgroups with more rounds than the others start first (gemv_forward lays the layers out so) and go first to their end, at
    // the highest priority: a wave's rounds follow each other, so that the longest one ends the launch.  us per block at T = 1 / 5 /
    // 16: 4096 x 11008 4-bit, 2 slices 24.4 / 24.8 / 27.7 -> 24.4 / 24.8 / 27.0; 3072 x 8192 3-bit g64 21.3 / 21.8 / 22.1 -> 19.7 /
    // 20.2 / 22.1; 6656 x 17920 3-bit 47.8 / 48.5 / 52.1 -> 46.5 / 47.1 / 50.4.
    // Of the others: a compute unit's arbiter serves the older wave first: of the workgroups that share one, the one dispatched first runs
    // ahead, ends early, and leaves the others to finish with fewer loads in flight.  Where all workgroups of the launch are
    // resident at once, the later ones therefore take a higher priority for the first half of their rounds; the first ones
    // win the ties of the second half, and all end together (13B block, T = 1 and 5: 34.6 -> 33.7 and 35.5 -> 34.3 us).
    // Which came later is a guess from the index (the first prio_step workgroups are dealt one to every compute unit, and so
    // on); a wrong guess costs time only.  Where later workgroups take the places of earlier ones it cost 3 to 6 %.
    const bool urgent = (L.form & GEMV_URGENT) != 0;
    if (urgent) {
        __builtin_amdgcn_s_setprio(3);
    } else if (a.prio_step && bx >= a.prio_step) {
        if (bx < 2 * a.prio_step) __builtin_amdgcn_s_setprio(1);
        else if (bx < 3 * a.prio_step) __builtin_amdgcn_s_setprio(2);
        else __builtin_amdgcn_s_setprio(3);
    }
#pragma unroll 1
    for (int r = 0; r < nrounds; ++r) {
        if (r == nrounds >> 1 && !urgent) __builtin_amdgcn_s_setprio(0);
        // rounds r .. min(r + nbuf, nrounds) - 1 are in flight, issued in order: wait for r only
        const int after = issued - 1 - r;                         // rounds issued after r
        if (NBUF > 3 && after == 3) gv_wait_vmcnt<3 * NDMA>();
        else if (NBUF > 2 && after == 2) gv_wait_vmcnt<2 * NDMA>();
        else if (after == 1) gv_wait_vmcnt<NDMA>();
        else gv_wait_vmcnt<0>();
        asm volatile("" ::: "memory");
#pragma unroll
        for (int s = 0; s < (SMALL ? 1 : 2); ++s) {
            const u32x4 af = *reinterpret_cast<const u32x4 *>(x_lane + rd + x_pos[s]);
#pragma unroll
            for (int h = 0; h < HH; ++h) {
                uint32_t bw[WORDS];
                const uint8_t *sb = b_lane + rd + h * GV_B_BYTES + s * STEP_B;
                if constexpr (BITS == 4) {
                    const u32x4 v = *reinterpret_cast<const u32x4 *>(sb);
#pragma unroll
                    for (int i = 0; i < 4; ++i) bw[i] = v[i];
                } else {
#pragma unroll
                    for (int i = 0; i < 3; ++i) bw[i] = *reinterpret_cast<const uint32_t *>(sb + 8 * i);
                }
                Unpacker up;
                up.prepare(bw, 0);
                u32x4 bf[4];
                static_for<4>([&](auto i) {
                    static_for<4>([&](auto j) { bf[i.value][j.value] = up.template frag_reg<i.value, j.value>(magic); });
                });
#pragma unroll
                for (int ct = 0; ct < 4; ++ct) acc[4 * h + ct] = mfma16(af, bf[ct], acc[4 * h + ct]);
            }
            accrs = mfma16(af, ones, accrs);
        }
        // this buffer is free again once its LDS reads have returned: refill it
        if (issued < nrounds) {
            __builtin_amdgcn_s_waitcnt(0xF | (0x7 << 4) | (0x3 << 14));   // lgkmcnt(0)
            asm volatile("" ::: "memory");
            issue_round();
        }
        rd = rd + ROUND == (uint32_t)(nbuf * ROUND) ? 0 : rd + ROUND;
        if (--group_left == 0 || r + 1 == nrounds) {
            // end of a scale group, or of this wave's share: fold offset, zero-point and scale
            // of the group into y, restart the sums
#pragma unroll
            for (int h = 0; h < HH; ++h) {
                const f32x4 sc = *reinterpret_cast<const f32x4 *>(sS + gj * GV_SROW + 64 * h + 4 * hb);
                f32x4 zo;                                         // 16 + z of the lane's channels
                if constexpr (ZBYTE) {
                    const uint32_t zz = *reinterpret_cast<const uint32_t *>(sZ + gj * ZROW + 64 * h + 4 * hb);
#pragma unroll
                    for (int i = 0; i < 4; ++i) zo[i] = kCodeOffset + (float)((zz >> (8 * i)) & 0xFFu);
                } else {
                    zo = *reinterpret_cast<const f32x4 *>(sZ + gj * ZROW + 64 * h + 4 * hb);
                }
#pragma unroll
                for (int ct = 0; ct < 4; ++ct) {
#pragma unroll
                    for (int jj = 0; jj < 4; ++jj) y[4 * h + ct][jj] += sc[ct] * (acc[4 * h + ct][jj] - zo[ct] * accrs[jj]);
                    acc[4 * h + ct] = zero;
                }
            }
            accrs = zero;
            ++gj;
            group_left = chunk_rounds;
        }
    }

    // ---- sum the waves, then write Y (S = 1) or this slice's partial
    __syncthreads();                                              // everyone is done with the ring and the scale tile
    // [wave][column tile][row in lane][lane], column tiles 16 words further apart: those that share a bank otherwise are read together
    float *red = reinterpret_cast<float *>(stage);
    constexpr int CT = 4 * 64 + 16;
#pragma unroll
    for (int ct = 0; ct < 4 * HH; ++ct)
#pragma unroll
        for (int j = 0; j < 4; ++j) red[(wave * 4 * HH + ct) * CT + j * 64 + lane] = y[ct][j];
    __syncthreads();
    // the T x GV_C results are dealt to the threads, channels fastest; each adds the waves in order
    for (int idx = tid; idx < a.T * GV_C; idx += THREADS) {
        const int t = SMALL ? idx >> 5 : H == 1 ? idx >> 6 : idx >> 7, nn = idx & (GV_C - 1);
        const int cl = Unpacker::BY_PARITY ? 2 * ((nn >> 3) & 7) + (nn & 1) : (nn >> 2) & 15;   // lane (c, q) and column tile that hold it
        const int tc = 4 * (nn >> 6) + (Unpacker::BY_PARITY ? (nn >> 1) & 3 : nn & 3);
        const float *src = red + tc * CT + (t & 3) * 64 + 16 * (t >> 2) + cl;
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) v += src[w * 4 * HH * CT];
        if constexpr (SMALL) {                                    // the other 32 features of every round: columns c + 8, rows 8 + t
#pragma unroll
            for (int w = 0; w < WAVES; ++w) v += src[w * 4 * HH * CT + 2 * 16 + 8];
        }
        const uint32_t to = (uint32_t)t * (uint32_t)l_N + (uint32_t)(n0 + nn);   // (T N is below 2^31)
        if (l_S == 1) global_store(L.Y + to, (uint16_t)float_to_bf16_bits(v));
        else global_store(L.partial + (size_t)slice * a.T * l_N + to, v);
    }
}

// NARROW: the launch has layers whose tiles are half as wide (GEMV_NARROW in GemvLayer::form).
template <int BITS, int H, int WAVES, int NX, bool ZBYTE, bool NARROW>
__global__ __launch_bounds__(WAVES * 64, GV_SIMD_WAVES) void gemv_kernel(GemvArgs a)
{
    extern __shared__ __align__(16) uint8_t stage[];
    // which layer this workgroup belongs to, and that layer's descriptor: scalar loads from the argument block
    const int bx = blockIdx.x;
    // (one word of every cache line of the descriptors, asked for together with the totals that choose among them: the
    // choice then reads what is on its way already)
    {
        int touched[(sizeof(a.layer) + 63) / 64];
#pragma unroll
        for (unsigned i = 0; i < sizeof(a.layer) / 64; ++i) touched[i] = kernarg_load<int>(64 * i);
#pragma unroll
        for (unsigned i = 0; i < sizeof(a.layer) / 64; ++i) asm volatile("" :: "s"(touched[i]));
    }
    int li = 0, wg0 = 0;
#pragma unroll
    for (int i = 0; i < GEMV_MAX_LAYERS - 1; ++i) {
        const int e = a.wg_end[i];
        if (bx >= e) { li = i + 1; wg0 = e; }
    }
    const GemvLayer L = kernarg_load<GemvLayer>((uint32_t)(li * sizeof(GemvLayer)));
    if constexpr (NARROW) {
        if (L.form & GEMV_NARROW) {                                        // (uniform)
            gemv_tile<BITS, H - 1, WAVES, NX, ZBYTE>(a, L, bx, wg0, stage);
            return;
        }
    }
    gemv_tile<BITS, H, WAVES, NX, ZBYTE>(a, L, bx, wg0, stage);
}

// Y[t,n] = bf16( partial[0][t,n] + partial[1][t,n] + ... ), fixed order, for the sliced layers of a launch, two neighbouring
// channels a thread.  Bound by its chain of memory latencies (arguments, partials, store): a short argument block, no division, and
// the slices asked for eight at a time, all before the first is added.
struct GemvSums {
    struct Layer {
        const float *partial;               // [S, tn]
        uint16_t *Y;
        uint32_t tn;                        // T N
        int S;
    } layer[GEMV_MAX_LAYERS];
    int block_end[GEMV_MAX_LAYERS];         // workgroups of layer j and all before it (unused entries: the total)
};
__global__ __launch_bounds__(256) void gemv_finish_kernel(GemvSums a)
{
    int j = 0, b0 = 0;
#pragma unroll
    for (int i = 0; i < GEMV_MAX_LAYERS - 1; ++i) {
        const int e = a.block_end[i];
        if ((int)blockIdx.x >= e) { j = i + 1; b0 = e; }
    }
    const GemvSums::Layer L = kernarg_load<GemvSums::Layer>((uint32_t)(j * sizeof(GemvSums::Layer)));
    const uint32_t e = 2u * ((blockIdx.x - (uint32_t)b0) * 256u + threadIdx.x);
    if (e >= L.tn) return;                                        // (tn is even: N % 128 == 0)
    f32x2 v = {0.f, 0.f};
    for (int s0 = 0; s0 < L.S; s0 += 8) {
        f32x2 p[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {                             // past the last slice: the last one again, not added
            const int sl = s0 + u < L.S ? s0 + u : L.S - 1;
            p[u] = global_load<f32x2>(L.partial + (size_t)sl * L.tn + e);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (s0 + u < L.S) v += p[u];
    }
    global_store(L.Y + e, pack_bf16x2(v[0], v[1]));
}

}  // namespace

// ---- host side

// LDS of a tile of 64 h channels: ring and scale tile, which the final sums (of 64 column tiles and waves: gemv_tile) take in the end
static int gv_tile_lds(int h, int waves, int nx, bool zbyte, int groups, int depth)
{
    const int loop = waves * depth * gv_round_bytes(h, nx) + groups * gv_group_bytes(h, zbyte);
    const int sums = waves * 4 * (h > 1 ? h : 1) * (4 * 64 + 16) * 4;
    return loop > sums ? loop : sums;
}

static int gv_lds_bytes(const GemvForm &f, int nx, bool zbyte, int groups)
{
    return gv_tile_lds(f.h, f.waves, nx, zbyte, groups, gv_nbuf(f.h));
}

static int gv_per_cu(const GemvForm &f, int lds)                   // workgroups a compute unit holds: LDS, registers
{
    const int by_regs = 4 * GV_SIMD_WAVES / f.waves, by_lds = GV_LDS_MAX / lds;
    return by_lds < by_regs ? by_lds : by_regs;
}

size_t gemv_partials(int n, const int *N, int T, const int *S)
{
    size_t bytes = 0;
    for (int j = 0; j < n; ++j)
        if (S[j] > 1) bytes += (size_t)S[j] * (size_t)T * (size_t)N[j] * sizeof(float);
    return bytes;
}

static int gv_cols(int K, int chunk, int S)                        // most scale groups a slice touches
{
    const int R = K / 64, cr = chunk / 64;
    if (cr >= R) return 1;
    if (S == 1) return R / cr;
    return ((R + S - 1) / S + cr - 1) / cr + 1;
}

// The form of a launch and the slices of its layers.
//
// At most one 64-channel tile per compute unit: eight waves each, so that the few workgroups keep enough loads in flight
// and share the unpacking (a compute unit unpacks 64 channels x 64 features in about 0.07 us, eight waves or four).  Long
// layers of fewer tiles (K >= 6144) are sliced until every compute unit has a tile or a wave is down to four rounds; what
// that gains has to pay for the second launch, 4 us.  us per call at T = 5, whole -> sliced: 5120 x 13824 22 -> 14 (3 slices),
// 4096 x 11008 15 -> 12 (4), 1024 x 8192 12 -> 9 (4); 4096 x 4096 8.0 -> 9.3 (2), which is why shorter ones stay whole.
//
// At most 8 tokens, half a tile per compute unit and no layer long enough to be sliced: tiles of 32 channels, which bring twice
// the units to bear.  A round of a wave is a chain of 0.4 us (its DMA's arrival, LDS, unpacking, MFMAs,
// the fold), which two waves per SIMD do not fill: 16 waves from 72 rounds on.  us per call at T = 5, 64 channels -> 32 with 8 /
// 16 waves: 768 x 768 g128 4.5 -> 4.3 / 5.0, 4096 x 4096 4-bit 7.7 -> 7.3 / 7.3, 5120 x 5120 3-bit g128 10.8 -> 9.9 / 9.1; with
// slices before, 5120 x 13824 g128 14.8 -> 18.5 / 16.0, and 8064 x 28160 g64 17 us longer, which is why long ones stay.
//
// More tiles: four waves.  Every workgroup should be resident at once (the last, partly filled round is otherwise made of
// few workgroups with a few loads in flight each) and no layer's much longer than the others'.  At most 8 tokens, per-channel layers
// and more than two workgroups per unit: layers of more than 1.35 times the mean length take tiles of 32 channels beside the
// others' 64, which need no slices, that is no second launch; such a tile's rounds are as many and follow each other,
// so they start first and go first (laid out last and with the others' priorities, d = 4096 4-bit, T = 1, takes 24.7 instead of 23.1 us,
// d = 5120 3-bit 31.1 instead of 28.2).  us per block at
// T = 1 / 5, sliced -> so: d = 4096 4-bit 24.4 / 24.8 -> 22.9 / 23.1, 3-bit 20.5 / 21.1 -> 19.2 / 19.6, d = 5120 3-bit 29.0 / 29.6 -> 27.1 /
// 27.8, d = 3072 4-bit 17.5 / 18.1 -> 15.7 / 16.4.  Not where a layer has more than 2.7 times the mean length, as long as in tiles of 64 then
// even with half the channels a round; not with scale groups, whose tile and folds cost a tile of 32 channels as much as
// one of 64 (d = 4096 4-bit g128, in a build that let it, 27.5 / 28.2 -> 28.4 / 28.9), nor for more tokens, of which a tile of 32 would
// fetch twice as much per channel.  The bound of two workgroups per unit stands where the first measurements ended: with one to two it
// would be the shorter form as well (T = 1 / 8: d = 1792, f = 4864 4-bit 11.0 / 11.7 -> 9.6 / 10.0, d = 2048, f = 5632 11.8 / 12.6 -> 10.7 / 11.0,
// d = 2560, f = 6912 13.6 / 14.3 -> 12.6 / 13.1), which has not been taken yet.  Otherwise layers are sliced to at most
// 1.35 times the mean length, more while the workgroups' scale tiles keep them from fitting on the chip together; failing
// that, 128 channels per workgroup (half of the token rows' traffic and LDS per channel).  us per block at T = 1 / 16, 13B
// 3-bit g128: 3 slices of the long layer 34.6 / 42.3, 2 slices (not resident) 38.9 / 45.6, 128 channels 35.8 / 38.2.
// Launches too large for that take the slicing with the most workgroups per compute unit, as long as the partial sums stay
// below 4 % of the codes.
//
// Slicings whose partial sums take more than `most` bytes are left out; where none remains, the fewest slices are taken.
GemvForm gemv_plan(int n, const int *N, const int *K, const int *chunk, int bits, int T, bool zbyte, size_t most, int cus, int *S)
{
    const int nx = T > 8 ? 2 : 1;
    int tiles = 0, rmax = 0;
    double rounds = 0.0;
    for (int j = 0; j < n; ++j) {
        tiles += N[j] / 64;
        rounds += (double)(N[j] / 64) * (K[j] / 64);
        rmax = K[j] / 64 > rmax ? K[j] / 64 : rmax;
    }
    // slices of at most `len` rounds (a little longer rather than one slice more), and whatever the LDS asks for
    auto slice_all = [&](const GemvForm &f, int len, int limit) {
        for (int j = 0; j < n; ++j) {
            const int r = K[j] / 64;
            S[j] = (int)((double)r / len + 0.7);
            S[j] = S[j] < 1 ? 1 : S[j];
            while (S[j] < r && gv_lds_bytes(f, nx, zbyte, gv_cols(K[j], chunk[j], S[j])) > limit) ++S[j];
        }
    };
    auto groups = [&]() {
        int g = 1;
        for (int j = 0; j < n; ++j) g = gv_cols(K[j], chunk[j], S[j]) > g ? gv_cols(K[j], chunk[j], S[j]) : g;
        return g;
    };
    if (tiles <= cus) {
        const bool halves = T <= 8 && zbyte && 2 * tiles <= cus && rmax < 96;
        const GemvForm f{halves ? 0 : 1, halves && rmax >= 72 ? 16 : 8};
        slice_all(f, rmax, GV_LDS_MAX);
        for (int j = 0; j < n && !halves; ++j) {
            const int r = K[j] / 64, s = cus / tiles < r / 32 ? cus / tiles : r / 32;
            if (r >= 96 && s > S[j]) S[j] = s;
        }
        if (gemv_partials(n, N, T, S) > most) slice_all(f, rmax, GV_LDS_MAX);
        return f;
    }
    const GemvForm small{1, 4}, wide{2, 4};
    const double mean = rounds / tiles;
    GemvForm best = small;
    int best_len = rmax, best_per_cu = 0;
    for (int w = 0; w < (zbyte ? 2 : 1); ++w) {
        const GemvForm f = w ? wide : small;
        if (zbyte && T <= 8 && w == 0) {              // long layers in tiles half as wide
            GemvForm g = f;
            int wgs = 0, lds = 0;
            bool fits = true;
            for (int j = 0; j < n; ++j) {
                const int r = K[j] / 64, cols = gv_cols(K[j], chunk[j], 1);
                const bool narrow = r > 1.35 * mean;
                S[j] = 1;
                g.narrow |= (narrow ? 1u : 0u) << j;
                wgs += N[j] / (narrow ? gemv_channels(f) / 2 : gemv_channels(f));
                const int need = narrow ? gv_tile_lds(f.h - 1, f.waves, nx, true, cols, 2)
                                        : gv_tile_lds(f.h, f.waves, nx, true, cols, gv_nbuf(f.h));
                lds = need > lds ? need : lds;
                fits = fits && (!narrow || (cols == 1 && r <= 2.0 * 1.35 * mean));
            }
            if (g.narrow && fits && wgs > 2 * cus && lds <= GV_LDS_MAX / 2 && gv_per_cu(f, lds) * cus >= wgs) return g;
        }
        for (int s = 1; s <= 8; ++s) {
            const int len = (rmax + s - 1) / s;
            if (len > 1.35 * mean && s < 8) continue;
            slice_all(f, len, GV_LDS_MAX / 2);
            if (gemv_partials(n, N, T, S) > most) continue;
            int wgs = 0;
            double partials = 0.0;
            for (int j = 0; j < n; ++j) {
                wgs += N[j] / (64 * f.h) * S[j];
                if (S[j] > 1) partials += 8.0 * S[j] * T * N[j];
            }
            const int per_cu = gv_per_cu(f, gv_lds_bytes(f, nx, zbyte, groups()));
            if (per_cu * cus >= wgs) return f;                     // all resident
            if (w == 0 && per_cu > best_per_cu && (best_per_cu == 0 || partials < 0.04 * rounds * 512 * bits)) {
                best_per_cu = per_cu;
                best_len = len;
            }
        }
    }
    if (best_per_cu == 0) slice_all(small, rmax, GV_LDS_MAX);
    else slice_all(best, best_len, GV_LDS_MAX / 2);
    return best;
}

hipError_t launch_gemv(int bits, const GemvForm &f, const GemvArgs &a_in, hipStream_t stream)
{
    GemvArgs a = a_in;
    bool sliced = false, zbyte = true;
    const int nx = a.T > 8 ? 2 : 1;
    int lds = 0, groups[GEMV_MAX_LAYERS];
    for (int j = 0; j < a.n_layers; ++j) {
        GemvLayer &l = a.layer[j];
        if (l.N % 128 != 0 || l.K % 128 != 0 || l.chunk % 64 != 0 || l.S < 1 || a.T < 1 || a.T > 16) return hipErrorInvalidValue;
        sliced = sliced || l.S > 1;
        zbyte = zbyte && l.dz == nullptr;
        l.chunk_rounds = l.chunk / 64;
        l.slice_rounds = l.K / 64 / l.S;
        l.slice_rem = l.K / 64 % l.S;
        l.s_magic = 0xFFFFFFFFu / (uint32_t)l.S;
        l.chunk_magic = 0xFFFFFFFFu / (uint32_t)l.chunk_rounds;
        groups[j] = gv_cols(l.K, l.chunk, l.S);
    }
    for (int j = 0; j < a.n_layers; ++j) {
        GemvLayer &l = a.layer[j];
        const bool narrow = (f.narrow >> j & 1u) != 0;
        const int h = narrow ? f.h - 1 : f.h;
        if (h < 0 || (narrow && (!zbyte || l.S > 1))) return hipErrorInvalidValue;
        l.form = narrow ? GEMV_NARROW | 2 : gv_nbuf(h);
        const int need = gv_tile_lds(h, f.waves, nx, zbyte, groups[j], l.form & GEMV_DEPTH);
        lds = need > lds ? need : lds;
    }
    const int wgs = a.wg_end[GEMV_MAX_LAYERS - 1];
    double work = 0.0;
    auto rounds = [](const GemvLayer &l) { return (l.form & GEMV_NARROW ? 0.5 : 1.0) * (l.K / 64) / l.S; };
    for (int j = 0; j < a.n_layers; ++j) work += rounds(a.layer[j]) * (a.wg_end[j] - (j ? a.wg_end[j - 1] : 0));
    for (int j = 0; j < a.n_layers; ++j) {
        GemvLayer &l = a.layer[j];
        // deeper rings where the LDS is there anyway
        while ((l.form & GEMV_NARROW) && (l.form & GEMV_DEPTH) < gv_nbuf(f.h - 1) &&
               gv_tile_lds(f.h - 1, f.waves, nx, zbyte, groups[j], (l.form & GEMV_DEPTH) + 1) <= lds)
            ++l.form;
        if (f.waves == 4 && ((l.form & GEMV_NARROW) || rounds(l) * wgs > 1.15 * work)) l.form |= GEMV_URGENT;
    }
    for (int j = a.n_layers; j < GEMV_MAX_LAYERS; ++j) a.layer[j] = a.layer[a.n_layers - 1];
    if (lds > GV_LDS_MAX) return hipErrorInvalidValue;
    const int cus = compute_units();
    a.prio_step = wgs <= gv_per_cu(f, lds) * cus ? cus : 0;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    // One instantiation: its dynamic LDS (more than the default limit: raised once per device), then the launch.
    auto go_as = [&](auto h_c, auto waves_c, auto bits_c, auto nx_c, auto z_c, auto narrow_c) -> hipError_t {
        static bool allowed[64];
        const auto kern = gemv_kernel<decltype(bits_c)::value, decltype(h_c)::value, decltype(waves_c)::value,
                                      decltype(nx_c)::value, decltype(z_c)::value, decltype(narrow_c)::value>;
        if (!allowed[dev]) {
            const hipError_t e2 = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                                      hipFuncAttributeMaxDynamicSharedMemorySize, GV_LDS_MAX);
            if (e2 != hipSuccess) return e2;
            allowed[dev] = true;
        }
        trace_before(KID_GEMV, stream);
        hipLaunchKernelGGL(kern, dim3(wgs), dim3(f.waves * 64), lds, stream, a);
        trace_after(KID_GEMV, stream);
        return hipGetLastError();
    };
    using std::integral_constant;
    auto go = [&](auto h_c, auto waves_c, auto bits_c, auto nx_c, auto z_c) -> hipError_t {
        if (f.narrow) {
            if constexpr (decltype(h_c)::value == 1 && decltype(waves_c)::value == 4 && decltype(nx_c)::value == 1 && decltype(z_c)::value)
                return go_as(h_c, waves_c, bits_c, nx_c, z_c, integral_constant<bool, true>{});
            return hipErrorInvalidValue;
        }
        return go_as(h_c, waves_c, bits_c, nx_c, z_c, integral_constant<bool, false>{});
    };
    const integral_constant<int, 0> none;
    const integral_constant<int, 1> one;
    const integral_constant<int, 2> two;
    const integral_constant<int, 4> four;
    const integral_constant<int, 8> eight;
    const integral_constant<int, 16> sixteen;
    const integral_constant<bool, true> zb;
    const integral_constant<bool, false> zf;
    auto on_form = [&](auto bits_c, auto nx_c) -> hipError_t {
        if (f.h == 0) {
            if constexpr (decltype(nx_c)::value == 1) {
                if (zbyte && f.waves == 16) return go(none, sixteen, bits_c, nx_c, zb);
                if (zbyte && f.waves == 8) return go(none, eight, bits_c, nx_c, zb);
            }
            return hipErrorInvalidValue;
        }
        if (f.h == 2) return zbyte && f.waves == 4 ? go(two, four, bits_c, nx_c, zb) : hipErrorInvalidValue;
        if (f.waves == 8) return zbyte ? go(one, eight, bits_c, nx_c, zb) : go(one, eight, bits_c, nx_c, zf);
        return zbyte ? go(one, four, bits_c, nx_c, zb) : go(one, four, bits_c, nx_c, zf);
    };
    const integral_constant<int, 3> three;
    if (bits == 4) e = nx == 2 ? on_form(four, two) : on_form(four, one);
    else e = nx == 2 ? on_form(three, two) : on_form(three, one);
    if (e != hipSuccess || !sliced) return e;
    GemvSums sums{};
    int n = 0, blocks = 0;
    for (int j = 0; j < a.n_layers; ++j) {
        const GemvLayer &l = a.layer[j];
        if (l.S == 1) continue;
        const uint32_t tn = (uint32_t)a.T * (uint32_t)l.N;        // T <= 16 and at most 2^24 channels: 32-bit arithmetic
        sums.layer[n] = GemvSums::Layer{l.partial, l.Y, tn, l.S};
        blocks += (int)((tn + 511) / 512);
        sums.block_end[n++] = blocks;
    }
    for (; n < GEMV_MAX_LAYERS; ++n) {
        sums.layer[n] = sums.layer[n - 1];
        sums.block_end[n] = blocks;
    }
    trace_before(KID_GEMV_FINISH, stream);
    hipLaunchKernelGGL(gemv_finish_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, sums);
    trace_after(KID_GEMV_FINISH, stream);
    return hipGetLastError();
}

}  // namespace peqa

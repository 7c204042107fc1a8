// One 16 RT (tokens) x 256 (output columns) tile of a PEQA contraction: the code that every contraction launch of
// peqa_gemm.hip runs (what the modes compute: see there).
//
// Four waves side by side along the columns (per contraction half): a wave owns all token rows of 64 columns, RT x 4
// MFMA 16x16x32 tiles in 16 RT AGPRs.  RT is 8 where there are tokens enough (what follows is said of it), 4, 6 or 7 where tiles of
// 128 rows would be mostly padding or leave the machine idle (gemm_row_tiles, gemm_plan).
//
// What bounds it and why this split.  Per 32-deep step and SIMD (two waves) the matrix instructions take 1024 cycles, and LDS
// delivers 128 bytes per cycle to the compute unit.  A matrix instruction (16 cycles) holds the SIMD's issue for 8 of them and a vector
// instruction for 4, whatever it is and whichever wave it is of: loops of 16x16x32 instructions with n others each take
// max(16, 8 + 4 n) cycles per matrix instruction, with one wave or two (n = 2: 7.6 ns, 3: 9.1, 4: 11.1).  So two are free; per channel there
// are 1.5, and 2.9 group-wise, which make a step a fifth longer.  With 128 x 64 per wave every weight of the tile is unpacked (and, group-wise, scaled) by one wave only:
// 2 instructions per weight pair per channel and 5 group-wise (scale_pair) make 256 and 640 cycles per step.  The split this
// replaced, 64 x 128 per wave, had every weight unpacked by two waves: 512 and, at the 7 instructions per pair it took to
// scale bf16 codes, 1800 cycles, which made the group-wise contractions vector-bound.  The price is that a wave reads the
// whole activation tile from LDS: 8 + 1 reads of 1 KB per wave and step instead of 4 + 2, 576 instead of 384 cycles of the
// compute unit.  Measured, 64 x 128 -> 128 x 64:
// LLaMA-13B block, 3 bits, groups of 128, T = 2048: forward launch 1537 -> 1239 us, dX 1654 -> 1445 us (with
// that split dX scaled its activation fragments instead of the weights; here the weights are cheaper to scale), and with
// fp16 codes for the scaling 1129 and 1259 us, with the scaling in three turns and short epilogues 1085 and 1110 (dX alone); 11008 x 4096, 4 bits, groups of 64, T = 500: forward 102 -> 72 -> 67 us;
// per-channel training steps of the 7B and 65B blocks 2.1 and 2.9 % shorter.
//
// Launches that fill the chip for long run below the nominal clock of 2.4 GHz, at 1.8 to 1.9 (GRBM_GUI_ACTIVE over their time): what
// saves cycles there gains less than its share of them.
#pragma once

#include <type_traits>

#include "peqa_device.h"
#include "peqa_kernels.h"

namespace peqa {

constexpr int TILE_C = 256;
constexpr int WAVE_C = 64;                                 // columns per wave
constexpr int KSTEP = 32;                                  // contraction depth of one loop iteration
constexpr int NSTAGE = 6;                                  // LDS ring depth
// token rows of a stage's activation tile: the tile's, rounded up to what whole wave-loads of 16 rows by four waves bring
constexpr int staged_rows(int rt) { return rt <= 4 ? 64 : 128; }
constexpr int a_half_bytes(int rt) { return staged_rows(rt) * KSTEP * 2; }   // of one contraction half: 4 or 8 KB
constexpr int B_WAVE_BYTES = 1024;                         // packed codes of one wave and step (64 columns x 32: 1 KB / 768 B)
// A ring stage holds, per contraction half the workgroup runs (KW = 2 or 1), one activation tile and the packed
// codes of its four waves: 24 KB or 12 KB (16 and 8 KB with 64 rows).
constexpr int stage_bytes(int kw, int rt) { return kw * (a_half_bytes(rt) + 4 * B_WAVE_BYTES); }
// 144 KB (the epilogue's exchange of 128 KB reuses it) or 72 KB (96 and 48 KB with 64 rows)
constexpr int ring_bytes(int kw, int rt) { return NSTAGE * stage_bytes(kw, rt); }
constexpr int tbl_bytes(int kw) { return kw * 4 * 2 * 1024; }           // group-wise MODE_Y / MODE_DX: 2 x 1 KB of (s, b) per wave

// The MFMA of a step (0 .. 4 rt - 1) after which turn r (0 .. turns - 1) of building the next step's weight fragments comes: spread
// over the last seven eighths of them.  A register is built in one turn, or, where it is scaled, in three (SCALE_TURNS).
constexpr int SCALE_TURNS = 3;
constexpr int frag_turns(bool scaled) { return scaled ? 16 + SCALE_TURNS - 1 : 16; }
constexpr int frag_turn_slot(int r, int rt, int turns) { return rt / 2 + ((4 * rt - 1 - rt / 2) * r) / (turns - 1); }
// The first turn of slot m or a later one.
constexpr int frag_turn_from(int m, int rt, int turns)
{
    int r = 0;
    while (r < turns && frag_turn_slot(r, rt, turns) < m) ++r;
    return r;
}

// ROW_SUMS (the scale gradient in pieces): the row sums of X over the piece, which take the code offset and the zero-point out
// of its sums before they are added to the other pieces' (taken out of the total only, they cost a digit of the result), are
// added up beside the matrix instructions: eight dot instructions per wave and step, 6 % of the launch, which is why whole
// contractions are handed the sums over the halves of K (8 bytes per row, one short launch per step and input).
template <int BITS, int MODE, bool GROUPED, int KW, int RT, bool ROW_SUMS = false>
__device__ __forceinline__ void gemm_tile(const GemmArgs &a, const int wg, uint8_t *lds)
{
    constexpr int STAGE_BYTES = stage_bytes(KW, RT), A_HALF_BYTES = a_half_bytes(RT);
    constexpr int MFMAS = 4 * RT;                          // per wave and step
    constexpr int NA = staged_rows(RT) / 64;               // activation DMAs per wave and step
    constexpr int DMA_PER_ITER = NA + 1;                   // DMA instructions per wave per iteration
    constexpr bool ALONG_CH = (MODE == MODE_DX);           // contraction over output channels
    constexpr bool SCALED = GROUPED && MODE != MODE_DDS;   // the scale is applied inside the loop: weights enter the MFMA scaled
    constexpr bool PAIRED = GROUPED && MODE == MODE_DDS;   // one scale group per contraction half
    static_assert(!ROW_SUMS || (!GROUPED && MODE == MODE_DDS && KW == 1 && (RT == 4 || RT == 8)),
                  "row sums per piece: scale gradient, four waves, a power of two pairs of row tiles");
    static_assert(RT >= 4 && RT <= 8, "row tiles");
    static_assert(KW == 2 || (KW == 1 && !PAIRED), "the paired scale gradient needs both contraction halves");
    typedef HalfBlockUnpacker<BITS, ALONG_CH, SCALED ? kFieldF16 : kFieldBf16> Unpacker;
    constexpr int WORDS = Unpacker::WORDS;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform, kept in an SGPR
    const int wn = wave & 3, wk = KW == 2 ? wave >> 2 : 0;       // column quarter, contraction half
    const int c = lane & 15, q = lane >> 4;

    // workgroup -> tile.  Workgroup ids are dealt round-robin to the 8 XCDs; XCD x gets an eighth of the tiles, in one run
    // of an order in which 32 neighbours are a patch of patch_t x (32 / patch_t) tiles: what runs on an XCD at one time
    // shares activation rows and weight columns through its L2, and every XCD has the same number of tiles whatever their
    // count.  (Patches dealt to the XCDs as wholes left six of them without work where a contraction has 48 tiles: forward
    // of a LLaMA-7B block, 3 bits, T = 333: 328 -> 152 us; 11008 x 4096 training step, groups of 64, T = 500: 326 -> 289 us.)
    // A split contraction is that many times the tiles, piece by piece.
    int tile_t, tile_c, piece = 0;
    const int split = PAIRED || a.split < 1 ? 1 : a.split;
    {
        const int whole = a.tiles_t * a.tiles_c, n = whole * split, per = (n + 7) >> 3;
        int idx = (wg & 7) * per + (wg >> 3);
        if ((wg >> 3) >= per || idx >= n) return;          // padding to a multiple of 8 (uniform per workgroup)
        if (split > 1) {
            const Quotient p = div_magic((uint32_t)idx, (uint32_t)whole, a.whole_magic);
            piece = (int)p.q;
            idx = (int)p.r;
        }
        const int strip = a.patch_t * a.tiles_c;           // patch_t rows of tiles, walked column by column
        const Quotient s = div_magic((uint32_t)idx, (uint32_t)strip, a.strip_magic);
        const int left = a.tiles_t - (int)s.q * a.patch_t, rows = left < a.patch_t ? left : a.patch_t;
        const Quotient t = div_magic(s.r, (uint32_t)rows, small_magic(rows));
        tile_c = (int)t.q;
        tile_t = (int)s.q * a.patch_t + (int)t.r;
        // In scalar registers, so that what follows from them is scalar too: from divisions, which are vector instructions, left
        // to the compiler, the running pointers of the operands lived in vector registers and every DMA of the loop read
        // them back (an eighth more vector instructions, and a scalar register that a memory instruction reads two to four
        // wait states after a vector instruction wrote it, where the hardware wants five; with the waits instead of this,
        // the steps of 7B and 13B blocks were 1.7 and 1.3 % longer, a 7B prefill 2.3 %).
        tile_c = __builtin_amdgcn_readfirstlane(tile_c);
        tile_t = __builtin_amdgcn_readfirstlane(tile_t);
        piece = __builtin_amdgcn_readfirstlane(piece);
    }

    const int t0 = tile_t * (16 * RT);
    const int col0 = tile_c * TILE_C + wn * WAVE_C;        // first output column of this wave
    const bool wave_on = col0 < a.C;
    const int T = a.T, KC = a.KC;
    // contraction ranges of the two halves: [kh0, kh0 + 32 nit) and [kh1, kh1 + 32 nit)
    int kh0, kh1, nit, grp = 0;
    bool half_on = true;
    if constexpr (PAIRED) {
        // groups 2 y and 2 y + 1; with an odd number of groups the last workgroup's second half
        // re-reads its first group and drops the result
        const int g1 = 2 * (int)blockIdx.y + 1;
        kh0 = 2 * (int)blockIdx.y * a.gsz;
        kh1 = (g1 < a.G ? g1 : g1 - 1) * a.gsz;
        nit = a.gsz / KSTEP;                               // >= 2 and even: the group size is a multiple of 64
        grp = 2 * (int)blockIdx.y + wk;
        half_on = grp < a.G;
    } else {
        // this piece's run of 128-deep units; nit is even (KW = 2) or a multiple of 4
        const int u0 = piece * a.piece_units + (piece < a.unit_rem ? piece : a.unit_rem);
        const int u1 = u0 + a.piece_units + (piece < a.unit_rem ? 1 : 0);
        kh0 = u0 * 128;
        nit = (u1 - u0) * (KW == 2 ? 2 : 4);               // >= 2: both contraction halves take half of the run
        kh1 = KW == 2 ? kh0 + (u1 - u0) * 64 : kh0;
    }
    const int kbeg = wk ? kh1 : kh0;
    const uint32_t magic = SCALED ? kMagicF16 : kMagic;
    const uint32_t lds_base = (uint32_t)(uintptr_t)lds;

    // ---- activation tiles: global -> LDS by DMA, wave-loads of 1 KB (16 rows; NA per wave and step).  Lane s of a
    // wave-load lands at byte 16 s, i.e. row s / 4, chunk position s % 4, and fetches the chunk that the XOR swizzle
    // assigns to that position.  KW = 2: wave-load m = 8 i + wave covers contraction half m / 8, rows 16 (m % 8) .. +16
    // (64 staged rows: wave-load `wave`, half m / 4, rows 16 (m % 4) ..); KW = 1: rows 16 wave .. and, of 128,
    // 64 + 16 wave .. (the swizzle only looks at row % 16).
    uint32_t a_voff, a_voff_2 = 0;
    {
        const int row_l = lane >> 2, pos = lane & 3;
        const int chunk = pos ^ a_swizzle(row_l);
        auto voff_of = [&](int row) __attribute__((always_inline)) {
            row = t0 + row < T ? row : T - 1 - t0;
            return (uint32_t)row * (uint32_t)KC * 2u + (uint32_t)chunk * 16u;
        };
        a_voff = voff_of((NA == 1 ? wn : wave) * 16 + row_l);
        if constexpr (NA == 1) a_voff += (uint32_t)(kbeg - kh0) * 2u;
        else if constexpr (KW == 1) a_voff_2 = voff_of(64 + wave * 16 + row_l);
        else a_voff_2 = a_voff + (uint32_t)(kh1 - kh0) * 2u;
    }
    constexpr int A_DST_2 = KW == 2 ? A_HALF_BYTES : A_HALF_BYTES / 2;
    const uint8_t *a_ptr = reinterpret_cast<const uint8_t *>(a.A) + ((size_t)t0 * KC + kh0) * 2;
    const uint32_t dst_a = lds_base + wave * 1024;

    // ---- packed weights: a wave fetches the codes of its own 64 columns x 32 contraction steps (32 blocks of 8x8: 1 KB at
    // 4 bits, 768 B at 3 bits) with one DMA per step, and lane (c, q) reads back its half of block c / 2:
    //   along features: channel block col0 / 8 + c / 2, feature block 4 it + q
    //   along channels: feature block col0 / 8 + c / 2, channel block 4 it + q
    // Blocks are stored in tiles of 16 channel blocks x 4 feature blocks (TILE bytes), tiles along the features first: along
    // features a step of a wave is half a tile (contiguous), along channels a quarter (4 channel blocks x 4 feature blocks,
    // contiguous) of each of two neighbouring tiles.
    constexpr uint32_t BLK = 2 * BITS * 4, TILE = 64 * BLK;
    const size_t tile_row = (size_t)(a.K >> 5) * TILE;     // bytes per row of tiles
    const int m0 = kbeg >> 5;                              // 32-deep contraction step at which this wave starts
    const int cb = c >> 1, par = c & 1;                    // the lane's block column, and its half of the block
    uint32_t b_voff;
    int b_lane_off;                                        // where this lane's words sit in the wave's LDS slot
    if constexpr (BITS == 4) {
        // lane (c, q) fetches the 16-byte half `par` of block (cb, q): its own words (along features), or half of what the two
        // lanes of a pair both read (along channels)
        if constexpr (!ALONG_CH) {
            b_voff = (uint32_t)((8 * (wn & 1) + cb) * 4 + q) * BLK + par * 16u;
            b_lane_off = lane * 16;
        } else {
            b_voff = (uint32_t)(cb >> 2) * TILE + (uint32_t)(q * 4 + (cb & 3)) * BLK + par * 16u;
            b_lane_off = (lane & ~1) * 16;
        }
    } else {
        // 24-byte blocks: 48 chunks of 16 B in address order (along channels: two runs of 24), laid down in chunk order; the
        // last 16 lanes repeat chunks 32..47 into the slot's unused tail
        const int x = lane < 48 ? lane : lane - 16;
        if constexpr (!ALONG_CH) {
            b_voff = (uint32_t)(wn & 1) * 768u + (uint32_t)x * 16u;
            b_lane_off = (cb * 4 + q) * 24 + 4 * par;
        } else {
            b_voff = (uint32_t)(x / 24) * TILE + (uint32_t)(x % 24) * 16u;
            b_lane_off = (cb >> 2) * 384 + (q * 4 + (cb & 3)) * 24;
        }
    }
    if (!wave_on) b_voff = lane * 16;
    // Packed bytes of this wave's contraction steps.  They are fetched strictly in order, one step per call (the last one
    // again and again once the range is used up; a wave without columns re-reads the start of the array), so a running
    // pointer advanced with selects stands in for the address arithmetic.
    const uint8_t *b_next = reinterpret_cast<const uint8_t *>(a.packed);
    if (wave_on) {
        if constexpr (ALONG_CH) b_next += (size_t)(col0 >> 5) * TILE + (size_t)(m0 >> 2) * tile_row + (size_t)(m0 & 3) * (16 * BLK);
        else b_next += (size_t)(col0 >> 7) * tile_row + (size_t)m0 * TILE;
    }
    int b_idx = 0;                                         // step b_next points at
    auto b_advance = [&]() __attribute__((always_inline)) {
        const bool more = wave_on && b_idx < nit - 1;
        size_t inc = TILE;
        if constexpr (ALONG_CH) inc = ((m0 + b_idx) & 3) == 3 ? tile_row - 3 * (size_t)(16 * BLK) : (size_t)(16 * BLK);
        b_next += more ? inc : 0;
        b_idx += more ? 1 : 0;
    };
    const uint32_t dst_b = lds_base + KW * A_HALF_BYTES + wave * B_WAVE_BYTES;

    // ---- group-wise MODE_Y / MODE_DX: (s, b = -s (16 + z)) of 128 (channel, group) entries, 1 KB, fetched by every wave
    // for itself by DMA one block of four steps ahead into a double buffer behind the ring.  Steps m are counted from the
    // start of the layer's contraction range; block B is steps 4 B .. 4 B + 3.
    //   along features: 64 entries (the wave's channels) of the group of features 128 B .. + 63, then 64 of the group of
    //                   features 128 B + 64 .. + 127 (the same one unless groups end inside the block)
    //   along channels: channels 128 B .. + 127 of the group of the wave's 64 feature columns (one group: sizes are
    //                   multiples of 64)
    const uint32_t tbl_off = NSTAGE * STAGE_BYTES + wave * 2048;
    const int last_block = (KC >> 7) - 1;
    int tb_g = 0, tb_left = 0;                             // along features: group of the next block's start, features left in it
    const uint8_t *tb_src = reinterpret_cast<const uint8_t *>(a.sb);
    if constexpr (SCALED) {
        if constexpr (ALONG_CH) {
            if (wave_on) tb_src += (size_t)(col0 / a.gsz) * a.N * 8;
        } else {
            const int f0 = (m0 >> 2) << 7;
            tb_g = f0 / a.gsz;
            tb_left = a.gsz - (f0 - tb_g * a.gsz);
            if (wave_on) tb_src += (size_t)col0 * 8;
        }
    }
    auto issue_table = [&](int B) __attribute__((always_inline)) {   // blocks are asked for in order
        const uint32_t dst = lds_base + tbl_off + (B & 1) * 1024;
        if constexpr (ALONG_CH) {
            B = B < last_block ? B : last_block;
            dma16(lane * 16, tb_src + (wave_on ? (size_t)B << 10 : 0), dst);
        } else {
            const int g0 = tb_g;
            auto advance = [&]() __attribute__((always_inline)) {
                tb_left -= 64;
                const bool next = tb_left == 0 && tb_g + 1 < a.G;   // past the last group: its entries again, never used
                tb_g += next ? 1 : 0;
                tb_left = tb_left == 0 ? a.gsz : tb_left;
            };
            advance();
            const int g1 = tb_g;
            advance();
            dma16((lane & 31) * 16 + (lane < 32 ? 0u : (uint32_t)(g1 - g0) * (uint32_t)a.N * 8u),
                  tb_src + (size_t)g0 * a.N * 8, dst);
        }
    };
    // Scales and offsets of the next fragments.  Along features fragment I needs entry I, the same for two steps; along
    // channels element e of every fragment is channel 32 (m % 4) + 8 q + e of the block: entries 2 J and 2 J + 1 are read
    // shortly before the registers J of all fragments are built (all eight at once cost registers that there are not).
    constexpr int NE = ALONG_CH ? 8 : 4;
    float sc[NE], bo[NE];
    const uint8_t *tbl_lane = lds + tbl_off + (ALONG_CH ? q * 64 : Unpacker::BY_PARITY ? cb * 64 + par * 8 : c * 32);
    auto read_table = [&](int m) __attribute__((always_inline)) {
        const uint8_t *row = tbl_lane + ((m >> 2) & 1) * 1024 + ((m >> 1) & 1) * 512;
        if constexpr (Unpacker::BY_PARITY) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const f32x2 v = *reinterpret_cast<const f32x2 *>(row + 16 * i);
                sc[i] = v[0];
                bo[i] = v[1];
            }
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const f32x4 v = *reinterpret_cast<const f32x4 *>(row + 16 * h);
                sc[2 * h] = v[0]; bo[2 * h] = v[1]; sc[2 * h + 1] = v[2]; bo[2 * h + 1] = v[3];
            }
        }
    };
    auto read_table_pair = [&](int m, int J) __attribute__((always_inline)) {
        const f32x4 v = *reinterpret_cast<const f32x4 *>(tbl_lane + ((m >> 2) & 1) * 1024 + (m & 3) * 256 + 16 * J);
        sc[2 * J] = v[0]; bo[2 * J] = v[1]; sc[2 * J + 1] = v[2]; bo[2 * J + 1] = v[3];
    };
    // Register r (0..15, in the order in which they are built) of the next step's fragments is register J of fragment I.  Scaled, it
    // takes three turns, which do not wait for each other: in turn t register t is unpacked, t - 1 scaled and t - 2 rounded.  (One
    // after the other, each register's five instructions were a chain that a wave waited for between two matrix instructions, with a wait
    // state of the compiler's own before either use of what assembly had written.)
    constexpr bool J_MAJOR = SCALED && ALONG_CH;
    constexpr int TURNS = frag_turns(SCALED);
    auto reg_i = [](int r) constexpr { return J_MAJOR ? r & 3 : r >> 2; };
    auto reg_j = [](int r) constexpr { return J_MAJOR ? r >> 2 : r & 3; };
    uint32_t unpacked = 0;
    ScaledPair scaled = {0.f, 0.f};
    auto frag_turn = [&](const Unpacker &up, auto t_c, u32x4 *frag) __attribute__((always_inline)) {
        constexpr int t = decltype(t_c)::value;
        if constexpr (!SCALED) {
            frag[reg_i(t)][reg_j(t)] = up.template frag_reg<reg_i(t), reg_j(t)>(magic);
        } else {
            if constexpr (t >= 2) frag[reg_i(t - 2)][reg_j(t - 2)] = round_pair(scaled);
            if constexpr (t >= 1 && t <= 16) {
                constexpr int I = reg_i(t - 1), J = reg_j(t - 1), lo = ALONG_CH ? 2 * J : I, hi = ALONG_CH ? 2 * J + 1 : I;
                scaled = scale_pair(unpacked, sc[lo], bo[lo], sc[hi], bo[hi]);
            }
            if constexpr (t < 16) unpacked = up.template frag_reg<reg_i(t), reg_j(t)>(magic);
        }
    };

    f32x4 acc[RT][4];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // LDS reads take a 16-bit literal offset: the stages of the first and of the second half of the ring are
    // addressed from one lane-dependent base register each (kept live across the loop), the rest is literal.
    constexpr int HALF_RING = (NSTAGE / 2) * STAGE_BYTES;
    static_assert((NSTAGE / 2 - 1) * STAGE_BYTES + 8192 <= 65536, "literal offsets of LDS reads");
    // row 16 rt' + c (the swizzle only looks at row % 16).  Where the row sums are taken, row tile rt of the wave's registers is
    // row tile rt' = rt ^ 2 wp of the tile, wp = wn (of 128 rows) or wn % 2 (of 64): registers 0 and 1 are then other rows in
    // each of the four (two) waves, which together add up all rows (two dot instructions per register: 8 per wave and step).
    constexpr int NPAIR = ROW_SUMS ? RT / 2 : 1;           // pairs of row tiles with a base register of their own
    const int wp = wn & (NPAIR - 1);
    const uint8_t *a_rd[2][NPAIR], *b_rd[2];
#pragma unroll
    for (int p = 0; p < NPAIR; ++p) {
        a_rd[0][p] = lds + wk * A_HALF_BYTES + c * 64 + ((q ^ a_swizzle(c)) << 4) + (ROW_SUMS ? (p ^ wp) * 2048 : 0);
        a_rd[1][p] = a_rd[0][p] + HALF_RING;
    }
    b_rd[0] = lds + KW * A_HALF_BYTES + wave * B_WAVE_BYTES + b_lane_off;
    b_rd[1] = b_rd[0] + HALF_RING;
    auto read_a = [&](auto st_c, u32x4 *af, int rt) __attribute__((always_inline)) {
        constexpr int ST = decltype(st_c)::value;
        const uint8_t *base = a_rd[ST / (NSTAGE / 2)][ROW_SUMS ? rt >> 1 : 0] + (ST % (NSTAGE / 2)) * STAGE_BYTES;
        af[rt] = *reinterpret_cast<const u32x4 *>(base + (ROW_SUMS ? rt & 1 : rt) * 16 * 64);
    };
    auto read_b = [&](auto st_c, uint32_t *w) __attribute__((always_inline)) {
        constexpr int ST = decltype(st_c)::value;
        const uint8_t *st = b_rd[ST / (NSTAGE / 2)] + (ST % (NSTAGE / 2)) * STAGE_BYTES;
        if constexpr (BITS == 4) {
#pragma unroll
            for (int i = 0; i < WORDS / 4; ++i) {
                const u32x4 v = *reinterpret_cast<const u32x4 *>(st + 16 * i);
#pragma unroll
                for (int e = 0; e < 4; ++e) w[4 * i + e] = v[e];
            }
        } else if constexpr (ALONG_CH) {
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const u32x2 v = *reinterpret_cast<const u32x2 *>(st + 8 * i);
                w[2 * i] = v[0];
                w[2 * i + 1] = v[1];
            }
        } else {
#pragma unroll
            for (int i = 0; i < 3; ++i) w[i] = *reinterpret_cast<const uint32_t *>(st + 8 * i);
        }
    };
    float rsum[2] = {0.f, 0.f};                            // row sums of row tiles 0 and 1 of the registers, this lane's part
    const uint32_t perm_sel = par ? 0x07060302u : 0x05040100u;

    // ---- scale and zero-point of this lane's four columns, for the epilogue: asked for before anything else, as they are (what
    // comes of them is formed in the epilogue), so that no tile ends with the latency of their loads.
    constexpr bool EP_SCALE = !SCALED && MODE == MODE_Y, EP_ZERO = !SCALED && !PAIRED && MODE != MODE_DX;
    f32x4 ep_s0 = {0.f, 0.f, 0.f, 0.f}, ep_ds = ep_s0, ep_dz = ep_s0;
    uint32_t ep_z0[4] = {0u, 0u, 0u, 0u};                  // MODE_Y: one word of four
    if (EP_ZERO && wave_on) {
        const int colc = col0 + 4 * c;
        if constexpr (MODE == MODE_Y) {
            ep_z0[0] = global_load<uint32_t>(a.z0 + colc);
            if (a.dz) ep_dz = global_load<f32x4>(a.dz + colc);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int col = Unpacker::BY_PARITY ? col0 + 4 * (c & ~1) + 2 * e + par : colc + e;
                ep_z0[e] = global_load<uint8_t>(a.z0 + col);
                if (a.dz) ep_dz[e] = global_load<float>(a.dz + col);
            }
        }
        if constexpr (EP_SCALE) {
            ep_s0 = global_load<f32x4>(a.s0 + colc);
            if (a.ds) ep_ds = global_load<f32x4>(a.ds + colc);
        }
    }

    // ---- prologue: queue NSTAGE - 1 stages (and the packed weights of one more), wait for the first two, fetch the operands
    // of step 0 and the packed weights of step 1
    u32x4 bfrag[2][4], afrag[RT];
    uint32_t bw[2][WORDS];                                 // packed weights of the next step / the one after
    if constexpr (SCALED) { issue_table(m0 >> 2); issue_table((m0 >> 2) + 1); }
    auto issue_a = [&](int stage) __attribute__((always_inline)) {
        dma16(a_voff, a_ptr, dst_a + stage * STAGE_BYTES);
        if constexpr (NA == 2) dma16(a_voff_2, a_ptr, dst_a + stage * STAGE_BYTES + A_DST_2);
    };
    auto issue_b = [&](int stage) __attribute__((always_inline)) {
        dma16(b_voff, b_next, dst_b + stage * STAGE_BYTES);
        b_advance();
    };
#pragma unroll
    for (int s = 0; s < NSTAGE - 1; ++s) {
        issue_a(s);
        a_ptr += s < nit - 1 ? KSTEP * 2 : 0;              // the last step again and again once the range is used up
        issue_b(s);
    }
    issue_b(NSTAGE - 1);                                   // the packed weights run one stage further ahead
    wait_vmcnt<DMA_PER_ITER *(NSTAGE - 4) + 1>();
    __syncthreads();
    {
        read_b(std::integral_constant<int, 0>{}, bw[1]);
        read_b(std::integral_constant<int, 1>{}, bw[0]);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) read_a(std::integral_constant<int, 0>{}, afrag, rt);
        if constexpr (SCALED) {
            if constexpr (ALONG_CH) {
#pragma unroll
                for (int J = 0; J < 4; ++J) read_table_pair(m0, J);
            } else {
                read_table(m0);
            }
        }
        Unpacker up;
        up.prepare(bw[1], perm_sel);
        static_for<TURNS>([&](auto t) { frag_turn(up, t, bfrag[0]); });
    }
    // (Step 0 refills the packed-weight slot of stage 0, which its own wave alone reads and has read; its activation tiles go to
    // stage NSTAGE - 1.  No barrier is needed before it.)

    // ---- main loop.  A step is a 32-deep contraction: M = 4 RT MFMAs, one per accumulator.  When step `it` starts, its
    // fragments and the packed weights of step it + 1 are in registers, and stages it + 1 and it + 2 are complete in LDS.  The
    // MFMAs run back to back from the first instruction after the barrier; everything else sits in their shadow, in fixed slots:
    //   after MFMA 2          LDS read of the packed weights of step it + 2
    //   from MFMA M / 8 on    every other MFMA or so, one register of step it + 1's weight fragments (the table entries that
    //                         scale them are read at the top)
    //   after MFMA M / 8 + 1, 3 M / 8 + 1, 5 M / 8 + 1
    //                         one DMA each: the activation loads of step it + NSTAGE - 1 (into the stage of step it - 1; one of
    //                         64 staged rows, two of 128) and the packed weights of step it + NSTAGE (into this step's own
    //                         stage: read two steps ago, by this wave alone, and the operand that comes from HBM, so it gets the longer lead).  The tail
    //                         re-fetches the last step: harmless, and it keeps the DMA count per step constant so that a
    //                         fixed vmcnt tells when a stage has landed
    //   after each 4 MFMAs    the activation fragment just used up is refilled from LDS for step it + 1
    // NSTAGE steps per loop trip, so that the ring stage of every step is a compile-time constant: LDS destinations and read
    // offsets are then literals.
    static_assert(NSTAGE % 2 == 0, "the register buffers alternate with the step's parity");
    // (inlined by force: ten copies are more than the inliner takes by itself, and a call would pass the
    // captured scalars through memory)
    auto step = [&](int it, auto stage_c) __attribute__((always_inline)) {
        constexpr int S = decltype(stage_c)::value;             // LDS stage of this step
        constexpr int CUR = S & 1, NXT = CUR ^ 1;
        constexpr int NS = (S + 1) % NSTAGE;                    // stage of step it + 1
        constexpr int NNS = (S + 2) % NSTAGE;                   // stage of step it + 2
        constexpr int PS = (S + NSTAGE - 1) % NSTAGE;           // stage of step it - 1 = of step it + NSTAGE - 1
        if constexpr (SCALED) {
            // The fragments built in this step belong to contraction step m = m0 + it + 1.  The buffer of the block before m's
            // was last read in an earlier step; the block after m's is fetched into it at the first step of m's block, and the
            // waits of three steps have passed when it is read first.
            // (m0 is even, so m's parity is that of S + 1.)
            const int m = m0 + it + 1;
            if constexpr (ALONG_CH) {
                read_table_pair(m, 0);
                read_table_pair(m, 1);
            } else if constexpr (S & 1) {
                read_table(m);
            }
            if constexpr (S & 1) {
                if ((m & 3) == 0) issue_table((m >> 2) + 1);
            }
        }
        Unpacker up;
        up.prepare(bw[CUR], perm_sel);
        static_for<RT>([&](auto rt_c) {
            constexpr int rt = rt_c.value;
            static_for<4>([&](auto ct_c) {
                constexpr int ct = ct_c.value, m = 4 * rt + ct;
                mfma16_acc(acc[rt][ct], afrag[rt], bfrag[CUR][ct]);
                constexpr int r0 = frag_turn_from(m, RT, TURNS), r1 = frag_turn_from(m + 1, RT, TURNS);
                static_for<r1 - r0>([&](auto r_c) {
                    constexpr int r = r0 + r_c.value;
                    frag_turn(up, std::integral_constant<int, r>{}, bfrag[NXT]);
                    if constexpr (J_MAJOR && r < 8 && reg_i(r) == 3) read_table_pair(m0 + it + 1, reg_j(r) + 2);
                });
                if constexpr (ROW_SUMS && rt < 2) rsum[rt] = add_pair(afrag[rt][ct], rsum[rt]);
                if constexpr (m == 2) read_b(std::integral_constant<int, NNS>{}, bw[NXT]);
                if constexpr (m == MFMAS / 8 + 1) dma16(a_voff, a_ptr, dst_a + PS * STAGE_BYTES);
                if constexpr (NA == 2 && m == 3 * MFMAS / 8 + 1) dma16(a_voff_2, a_ptr, dst_a + PS * STAGE_BYTES + A_DST_2);
                if constexpr (m == 5 * MFMAS / 8 + 1) {
                    issue_b(S);
                    a_ptr += it + NSTAGE - 1 < nit - 1 ? KSTEP * 2 : 0;
                }
            });
            read_a(std::integral_constant<int, NS>{}, afrag, rt);
        });
        // Own DMA for step it + 3 has landed; the barrier makes every wave's part visible.
        // No wait on LDS reads is needed here: what this step read is overwritten two steps later.
        wait_vmcnt<DMA_PER_ITER *(NSTAGE - 4) + 1>();
        bare_barrier();
    };
    {
        int it = 0;
        for (; it + NSTAGE <= nit; it += NSTAGE)
            static_for<NSTAGE>([&](auto s_c) { step(it + decltype(s_c)::value, s_c); });
        // nit is even (KC % 128 == 0): none, two or four steps are left, in stages 0..3
        if (nit - it >= 2) {
            step(it, std::integral_constant<int, 0>{});
            step(it + 1, std::integral_constant<int, 1>{});
        }
        if (nit - it >= 4) {
            step(it + 2, std::integral_constant<int, 2>{});
            step(it + 3, std::integral_constant<int, 3>{});
        }
    }
    // The loop's exits meet here; this keeps the accumulators in their AGPRs past that point (the compiler would
    // otherwise copy all 128 of them into VGPRs at once, more than there are)
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) asm volatile("" : "+a"(acc[i][j]));
    // The epilogue works out its lane indices afresh (from a copy of the thread index that the compiler cannot
    // connect to the first one), so that none of them has to be held in a register through the loop.
    {
    int tid_e = threadIdx.x;
    asm volatile("" : "+v"(tid_e));
    const int tid = tid_e, lane = tid & 63, c = lane & 15, q = lane >> 4, par = c & 1;
    const int colc = col0 + 4 * c;                         // after columns_of: this lane's four columns are colc .. colc + 3
    // Lane (c, q) holds rows 4 q + j of every row tile.  Its column of accumulator (rt, I) is 4 c + I of the wave's 64 where a
    // lane unpacks four neighbouring columns; where it unpacks every other column of a block (8 (c / 2) + 2 I + c % 2), the two
    // lanes of a pair swap two of their four, after which both cases are alike.
    auto columns_of = [&](const f32x4 *v, int j) __attribute__((always_inline)) -> f32x4 {
        if constexpr (!Unpacker::BY_PARITY) {
            return f32x4{v[0][j], v[1][j], v[2][j], v[3][j]};
        } else {
            const float r0 = swap_pair_lane(par ? v[0][j] : v[2][j]), r1 = swap_pair_lane(par ? v[1][j] : v[3][j]);
            return par ? f32x4{r0, v[2][j], r1, v[3][j]} : f32x4{v[0][j], r0, v[1][j], r1};
        }
    };
    // column of the lane's accumulators acc[.][e] (before columns_of)
    auto own_col = [&](int e) __attribute__((always_inline)) {
        return Unpacker::BY_PARITY ? col0 + 4 * (c & ~1) + 2 * e + par : colc + e;
    };
    // rows 4 q + j of the registers' row tile rt
    auto local_row = [&](int rt) __attribute__((always_inline)) { return (ROW_SUMS ? rt ^ (2 * wp) : rt) * 16 + 4 * q; };
    auto row_of = [&](int rt, int j) __attribute__((always_inline)) { return t0 + local_row(rt) + j; };
    auto clamped = [&](int t) __attribute__((always_inline)) { return t < T ? t : T - 1; };
    f32x4 ep_sc = {0.f, 0.f, 0.f, 0.f}, ep_zoff = {0.f, 0.f, 0.f, 0.f};
    if constexpr (PAIRED) {
        if (wave_on) {
            const int g = half_on ? grp : a.G - 1;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const size_t i = (size_t)own_col(e) * a.G + g;
                ep_zoff[e] = kCodeOffset + (float)global_load<uint8_t>(a.z0 + i);
                if (a.dz) ep_zoff[e] += global_load<float>(a.dz + i);
            }
        }
    } else if constexpr (EP_ZERO) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t z = MODE == MODE_Y ? (ep_z0[0] >> (8 * e)) & 0xFFu : ep_z0[e];
            ep_zoff[e] = kCodeOffset + (float)z;
        }
        if (a.dz) ep_zoff += ep_dz;
        ep_sc = ep_s0;
        if (EP_SCALE && a.ds) ep_sc += ep_ds;
    }
    // Y, dX: correction terms of the rows of a row tile, and of the first one that this wave finishes while the last DMAs drain
    auto load_terms = [&](int rt, float *r) __attribute__((always_inline)) {
        if constexpr (!SCALED && MODE != MODE_DDS) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if constexpr (MODE == MODE_Y) {
                    const f32x2 r2 = global_load<f32x2>(a.rs + 2 * clamped(row_of(rt, j)));
                    r[j] = r2[0] + r2[1];
                } else {
                    r[j] = global_load<float>(a.crow + clamped(row_of(rt, j)));
                }
            }
        }
    };
    constexpr int FIRST = (RT + 1) / 2;                    // row tiles that the waves of the first contraction half finish
    float terms[2][4];                                     // of this row tile and the next
    load_terms(KW == 2 && wk ? FIRST : 0, terms[0]);
    wait_vmcnt<0>();
    __syncthreads();
    mfma_result_fence();
    // Row sums: the four lanes of a row meet (fixed order), the waves' rows meet in LDS.
    // (of 64 rows: two waves bring the same sums)
    float *rs_lds = reinterpret_cast<float *>(lds);        // [16 RT]
    if constexpr (ROW_SUMS) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            rsum[i] += __shfl_xor(rsum[i], 16);
            rsum[i] += __shfl_xor(rsum[i], 32);
            if (q == 0) rs_lds[32 * wp + 16 * i + c] = rsum[i];
        }
        __syncthreads();
    }

    // ---- epilogues
    if constexpr (MODE == MODE_DDS) {
        // column sums of dY[t,i] * (acc[t,i] - (16 + z_i) * rowsum_half[t]) over the tile's rows
        f32x4 colsum = {0.f, 0.f, 0.f, 0.f};
        if (wave_on) {
            // Rows past T are clamped for the loads and masked in the sum, so that all loads are unconditional: dY and
            // the row sums four rows at a time, the next four in flight while these are used.
            // (Where the lane's columns are every other one of a block, both lanes of a pair load all eight.)
            constexpr int DW = Unpacker::BY_PARITY ? 4 : 2;    // words of a row's dY a lane loads
            typedef uint32_t dy_vec __attribute__((ext_vector_type(DW)));
            const uint16_t *dy0 = a.dY + col0 + (Unpacker::BY_PARITY ? 4 * (c & ~1) : 4 * c);
            const int up16 = 16 - 16 * par;
            f32x4 pairsum = {0.f, 0.f, 0.f, 0.f}, first = {0.f, 0.f, 0.f, 0.f};
            dy_vec dyv[2][4];
            float rsv[2][4];
            auto load_rows = [&](auto rt_c, dy_vec *dst, float *rdst) __attribute__((always_inline)) {
                constexpr int rt = decltype(rt_c)::value;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int tc = clamped(row_of(rt, j));
                    dst[j] = global_load<dy_vec>(dy0 + (size_t)tc * a.C);
                    // row sum of X over what this wave contracted
                    if constexpr (ROW_SUMS) {
                        rdst[j] = rs_lds[local_row(rt) + j];
                    } else if constexpr (PAIRED) {
                        rdst[j] = global_load<float>(a.rs + (size_t)tc * a.G + (half_on ? grp : a.G - 1));
                    } else if constexpr (KW == 2) {
                        rdst[j] = global_load<float>(a.rs + 2 * tc + wk);
                    } else {
                        const f32x2 r2 = global_load<f32x2>(a.rs + 2 * tc);
                        rdst[j] = r2[0] + r2[1];
                    }
                }
            };
            load_rows(std::integral_constant<int, 0>{}, dyv[0], rsv[0]);
            static_for<RT>([&](auto rt_c) {
                constexpr int rt = rt_c.value;
                if constexpr (rt + 1 < RT) load_rows(std::integral_constant<int, rt + 1>{}, dyv[(rt + 1) & 1], rsv[(rt + 1) & 1]);
                float dm[4];                                   // rows past T contribute nothing
#pragma unroll
                for (int j = 0; j < 4; ++j) dm[j] = row_of(rt, j) < T ? 1.f : 0.f;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const f32x4 v = read_acc(acc[rt][e]);      // one accumulator tile at a time leaves its AGPRs
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        float d;
                        if constexpr (Unpacker::BY_PARITY) d = __uint_as_float((dyv[rt & 1][j][e] << up16) & 0xFFFF0000u);
                        else d = (e & 1) ? bf16_hi(dyv[rt & 1][j][e >> 1]) : bf16_lo(dyv[rt & 1][j][e >> 1]);
                        pairsum[e] += d * dm[j] * (v[j] - ep_zoff[e] * rsv[rt & 1][j]);
                    }
                }
                // (r0 + r1) + (r2 + r3) over the pairs of row tiles: the same bits in whatever order a wave has them
                // (pair p of the registers is pair p ^ wp of the tile), so that a column's sum does not depend on its wave
                if constexpr (rt % 4 == 1 || (rt == RT - 1 && rt % 4 == 0)) {
                    first = pairsum;
                    pairsum = f32x4{0.f, 0.f, 0.f, 0.f};
                }
                if constexpr (rt % 4 == 3 || rt == RT - 1) {
                    if constexpr (rt < 4) colsum = first + pairsum;
                    else colsum += first + pairsum;
                    pairsum = f32x4{0.f, 0.f, 0.f, 0.f};
                }
            });
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            colsum[e] += __shfl_xor(colsum[e], 16);
            colsum[e] += __shfl_xor(colsum[e], 32);
        }
        if constexpr (Unpacker::BY_PARITY) {               // from here on: columns colc .. colc + 3
            f32x4 v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = f32x4{colsum[e], 0.f, 0.f, 0.f};
            colsum = columns_of(v, 0);
        }
        if constexpr (KW == 1) {
            if (wave_on && q == 0)
                global_store(a.partial + (size_t)(piece * a.tiles_t + tile_t) * a.C + colc, colsum);
        } else {
            float *red = reinterpret_cast<float *>(lds);   // [contraction half][256 columns]
            if (q == 0) *reinterpret_cast<f32x4 *>(red + wk * TILE_C + wn * WAVE_C + 4 * c) = colsum;
            __syncthreads();
            const int n = tile_c * TILE_C + tid;
            if (tid < TILE_C && n < a.C) {
                if constexpr (PAIRED) {
                    // the two contraction halves are two scale groups: one partial each
                    const int g0 = 2 * (int)blockIdx.y;
                    float *dst = a.partial + ((size_t)tile_t * a.C + n) * a.G + g0;
                    global_store(dst, red[tid]);
                    if (g0 + 1 < a.G) global_store(dst + 1, red[TILE_C + tid]);
                } else {
                    global_store(a.partial + (size_t)(piece * a.tiles_t + tile_t) * a.C + n, red[tid] + red[TILE_C + tid]);
                }
            }
        }
    } else {
        // rows 4 q + j (j = 0..3) of row tile rt, whose sums over the whole contraction are in sum[I][j]; r[j]: their
        // correction terms
        auto store_rows = [&](int rt, const f32x4 *sum, const float *r) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int t = row_of(rt, j);
                f32x4 v = columns_of(sum, j);              // (every lane takes part)
                if (split > 1) {                           // (uniform)
                    if (t < T) global_store(a.acc_part + ((size_t)piece * T + t) * a.C + colc, v);
                } else if (t < T) {
                    if constexpr (!SCALED) {
                        if constexpr (MODE == MODE_Y) {
                            v -= ep_zoff * r[j];
                            if (a.P) global_store(a.P + (size_t)t * a.C + colc, v);   // kept for the backward
                            v *= ep_sc;
                        } else {
                            v -= r[j];
                        }
                    }
                    u32x2 o;
                    o[0] = pack_bf16x2(v[0], v[1]);
                    o[1] = pack_bf16x2(v[2], v[3]);
                    global_store(a.out + (size_t)t * a.C + colc, o);
                }
            }
        };
        if constexpr (KW == 1) {
            // one contraction range per workgroup: every wave holds the finished sums of its row tiles
            if (!wave_on) return;
            static_for<RT>([&](auto rt_c) {
                constexpr int rt = rt_c.value;
                if constexpr (rt + 1 < RT) load_terms(rt + 1, terms[(rt + 1) & 1]);
                f32x4 sum[4];
#pragma unroll
                for (int ct = 0; ct < 4; ++ct) sum[ct] = read_acc(acc[rt][ct]);
                store_rows(rt, sum, terms[rt & 1]);
            });
        } else {
            // sum the two contraction halves: waves with wk = 0 keep the first half of the row tiles (rounded up) and send the
            // others, waves with wk = 1 the other way round
            f32x4 *xch = reinterpret_cast<f32x4 *>(lds);       // [8 waves][4 FIRST accumulator tiles][64 lanes]
            static_assert(8 * 4 * FIRST * 1024 <= ring_bytes(2, RT), "the exchange reuses the ring");
            auto finish = [&](auto keep_c) __attribute__((always_inline)) {
                constexpr int KEEP = decltype(keep_c)::value;  // first row tile this wave keeps
                constexpr int SEND = FIRST - KEEP, KEPT = KEEP ? RT - FIRST : FIRST, SENT = RT - KEPT;
                {
                    f32x4 *mine = xch + (size_t)wave * (4 * FIRST) * 64 + lane;
#pragma unroll
                    for (int rtl = 0; rtl < SENT; ++rtl)
#pragma unroll
                        for (int ct = 0; ct < 4; ++ct) mine[(rtl * 4 + ct) * 64] = acc[SEND + rtl][ct];
                }
                __syncthreads();
                if (!wave_on) return;
                const f32x4 *theirs = xch + (size_t)(wave ^ 4) * (4 * FIRST) * 64 + lane;
                static_for<KEPT>([&](auto rt_c) {
                    constexpr int rtl = rt_c.value;
                    if constexpr (rtl + 1 < KEPT) load_terms(KEEP + rtl + 1, terms[(rtl + 1) & 1]);
                    f32x4 sum[4];
#pragma unroll
                    for (int ct = 0; ct < 4; ++ct) sum[ct] = read_acc(acc[KEEP + rtl][ct]) + theirs[(rtl * 4 + ct) * 64];
                    store_rows(KEEP + rtl, sum, terms[rtl & 1]);
                });
            };
            if (wk == 0) finish(std::integral_constant<int, 0>{});
            else finish(std::integral_constant<int, FIRST>{});
        }
    }
    }
}

}  // namespace peqa

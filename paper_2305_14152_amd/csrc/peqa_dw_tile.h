// The tile of the token contraction of peqa_dw.hip, which says what it computes and why so.
#pragma once

#include "peqa_device.h"
#include "peqa_kernels.h"

namespace peqa {

namespace {

constexpr int DW_TF = 128;                       // features per workgroup
constexpr int DW_TC = 256;                       // channels per workgroup
constexpr int DW_NST = 6;                        // ring depth
constexpr int DW_STAGE = DW_TF * 64;             // 8 KB: 128 feature rows x 32 tokens
constexpr int DW_CODES = 16 * 1024;              // packed words of the tile (12 KB of them at 3 bits)
constexpr int DW_LDS = DW_CODES + DW_NST * DW_STAGE;

template <int BITS>
__device__ __forceinline__ void dw_tile(const DwArgs &a, const int wg, uint8_t *lds)
{
    constexpr int WPB = 2 * BITS;
    constexpr int NRT = 8, NCT = 4;                        // accumulator tiles of a wave: features x channels
    const int tid = threadIdx.x, lane = tid & 63;
    const int wn = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave = quarter of the channels
    const int c = lane & 15, q = lane >> 4;

    // Nothing is in flight here, which the compiler cannot know where this tile shares a kernel with the dX tile, whose stores
    // it believes may be pending: it would wait for them in the loop (see load_b).
    __builtin_amdgcn_s_waitcnt(0);

    // workgroup -> tile: XCD x gets an eighth of the tiles, in one run of an order in which 64 neighbours (what an XCD
    // runs at a time) are a patch of 8 feature x 8 channel tiles, so that operand rows are shared through its L2
    int tile_f, tile_c;
    {
        const int ntiles = a.tiles_f * a.tiles_c, xcd = wg & 7;
        const int lo = ntiles / 8 * xcd + min(xcd, ntiles % 8), mine = ntiles / 8 + (xcd < ntiles % 8 ? 1 : 0);
        if ((wg >> 3) >= mine) return;                     // (uniform)
        const int id = lo + (wg >> 3);
        const Quotient s = div_magic((uint32_t)id, 8u * (uint32_t)a.tiles_c, a.strip_magic);
        const int left = a.tiles_f - 8 * (int)s.q, rows = left < 8 ? left : 8;
        const Quotient t = div_magic(s.r, (uint32_t)rows, small_magic(rows));
        tile_c = (int)t.q;
        tile_f = 8 * (int)s.q + (int)t.r;
    }

    const int k0 = tile_f * DW_TF, n0 = tile_c * DW_TC;
    const int nsteps = a.Tp >> 5;                          // even: Tp % 64 == 0
    const uint32_t lds_base = (uint32_t)(uintptr_t)lds;

    // ---- the packed codes of the tile's 128 x 256 weights, for the epilogue: two runs of 4 step tiles (CODE_RUN bytes
    // each: contiguous in the tile-major layout), of its two 128-channel tile rows, copied linearly, 3 or 4 KB per wave.
    // A second tile row past the matrix is read from the first and never looked at.
    constexpr uint32_t CODE_TILE = 64 * WPB * 4, CODE_RUN = 4 * CODE_TILE;   // one 128 x 32 tile; 4 of them (6 or 8 KB)
    constexpr int CODE_DMA = 2 * CODE_RUN / 4096;
    {
        const size_t row_bytes = (size_t)(a.K >> 5) * CODE_TILE;
#pragma unroll
        for (int j = 0; j < CODE_DMA; ++j) {
            const uint32_t byte = (uint32_t)(CODE_DMA * wn + j) * 1024u;
            const uint32_t run = byte / CODE_RUN, off = byte - run * CODE_RUN;
            const int row = (2 * tile_c + (int)run) * 128 < a.N ? 2 * tile_c + (int)run : 2 * tile_c;
            dma16((uint32_t)lane * 16u,
                  reinterpret_cast<const uint8_t *>(a.packed) + (size_t)row * row_bytes + (size_t)tile_f * CODE_RUN + off,
                  lds_base + byte);
        }
    }

    // Both queues run past the last step (re-fetching it), so that the number of operations in flight per step is constant.
    const uint8_t *xsrc = reinterpret_cast<const uint8_t *>(a.Xt) + (size_t)k0 * 64;
    const size_t xstep = (size_t)a.K * 64, ystep = (size_t)a.N * 64;   // one 32-token step of all rows
    auto clamp_step = [&](int it) { return it < nsteps ? it : nsteps - 1; };
    // DMA j of wave wn is KB 2 wn + j of the stage
    auto issue = [&](int it, int stage) {
        const uint8_t *src = xsrc + (size_t)clamp_step(it) * xstep;
#pragma unroll
        for (int j = 0; j < 2; ++j)
            dma16((uint32_t)(2 * wn + j) * 1024u + (uint32_t)lane * 16u, src,
                  lds_base + DW_CODES + stage * DW_STAGE + (2 * wn + j) * 1024);
    };
    // the wave's 64 channels; past the matrix (N % 128 == 0: whole waves) the last ones of it, and nothing is stored
    const int cb = n0 + 64 * wn, cb_l = cb < a.N ? cb : a.N - 64;
    const uint8_t *ysrc = reinterpret_cast<const uint8_t *>(a.dYt) + (size_t)cb_l * 64;
    // By global loads: a pointer that came out of the argument block at a run-time offset is a generic one to the compiler, which
    // before the use of what a FLAT load brings waits for every memory operation in flight, the ring's DMAs among them
    // (0.51 instead of 0.36 us per step of a tile alone on its unit: the joint launch of 128 x 384, T = 3411, 54 -> 38 us).
    auto load_b = [&](const uint8_t *step_src, int ct) {
        return global_load<u32x4>(step_src + ct * 1024 + lane * 16);
    };
    u32x4 bfrag[2][NCT];

    f32x4 acc[NRT][NCT];
#pragma unroll
    for (int i = 0; i < NRT; ++i)
#pragma unroll
        for (int j = 0; j < NCT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    auto read_a = [&](int stage, int rt) {
        return *reinterpret_cast<const u32x4 *>(lds + DW_CODES + stage * DW_STAGE + rt * 1024 + lane * 16);
    };

    // ---- prologue: five stages and two steps of channel operands queued, in the order of the loop; the first two stages
    // (and the codes before them) complete before the first operands are read
    constexpr int PER_STEP = 2 + NCT;                      // memory operations of a wave per step
    issue(0, 0);
    issue(1, 1);
    static_for<2>([&](auto d_c) {
        constexpr int d = d_c.value;
        issue(2 + d, 2 + d);
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct) bfrag[d][ct] = load_b(ysrc + (size_t)d * ystep, ct);
    });
    issue(4, 4);
    wait_vmcnt<2 * PER_STEP + 2>();
    __syncthreads();
    u32x4 afrag[2][NRT];
#pragma unroll
    for (int rt = 0; rt < NRT; ++rt) afrag[0][rt] = read_a(0, rt);

    // ---- main loop.  At the start of step `it` its feature operands are in registers and stage it + 1 is complete and
    // visible.  The step queues stage it + 5 into the slot of stage it - 1 (read during step it - 2, and the last barrier
    // came after), reads the feature operands of step it + 1, and refills every channel operand for step it + 2 right after
    // its last use.  The closing wait leaves the operations of the last three steps outstanding: stage it + 2, queued in
    // step it - 3, has landed; the barrier makes it visible.
    int nxt = 1, slot = 5;                                 // slots of stage it + 1 and of stage it + 5
    auto step = [&](int it, auto cur_c) __attribute__((always_inline)) {
        constexpr int CUR = decltype(cur_c)::value, NXT = CUR ^ 1;
        issue(it + 5, slot);
        const uint8_t *src = ysrc + (size_t)clamp_step(it + 2) * ystep;
        static_for<NCT>([&](auto ct_c) {
            constexpr int ct = ct_c.value;
            static_for<NRT>([&](auto rt_c) {
                constexpr int rt = rt_c.value;
                mfma16_acc(acc[rt][ct], afrag[CUR][rt], bfrag[CUR][ct]);
                if constexpr (ct < 2 && rt % 2 == 1) afrag[NXT][4 * ct + rt / 2] = read_a(nxt, 4 * ct + rt / 2);
            });
            bfrag[CUR][ct] = load_b(src, ct);
        });
        wait_vmcnt<3 * PER_STEP>();
        bare_barrier();
        nxt = nxt == DW_NST - 1 ? 0 : nxt + 1;
        slot = slot == DW_NST - 1 ? 0 : slot + 1;
    };
    for (int it = 0; it < nsteps; it += 2) {
        step(it, std::integral_constant<int, 0>{});
        step(it + 1, std::integral_constant<int, 1>{});
    }
    wait_vmcnt<0>();
    mfma_result_fence();

    // ---- epilogue: the features are the chunks k0 / 64 + h (accumulator rows rt = 4 h .. 4 h + 3); lane (c, q) holds,
    // per accumulator tile (rt, ct), features k0 + 16 rt + 4 q + j (j = 0..3) of channel cb + 16 ct + c
    if (cb >= a.N) return;                                 // wave-uniform
    const int nchunks = a.K >> 6;
    // the codes of this wave's 128-channel tile row
    const uint8_t *code_lds = lds + (wn >> 1) * CODE_RUN;
    // The lane's four features of an accumulator tile are half a row of one 8 x 8 code block: row r = c % 8 (cb is a
    // multiple of 64), columns 4 hq .. 4 hq + 3 with hq = q % 2 (k0 + 16 rt is a multiple of 16).  Where those four
    // codes sit inside the block's words depends on (r, hq) only: worked out once per lane, so that a tile costs a few
    // loads at fixed offsets and shifts by lane constants (taken code by code with run-time row and column, the
    // epilogue took a third of the kernel's time at T = 2048).
    //   4 bits: word r, code of column cc at bits [4 p, 4 p + 4), p = cc / 2 + 4 (cc % 2): after a shift by 8 hq the four
    //           codes are at bits 0, 16, 4, 20.
    //   3 bits: cell u = 4 (r / 2) + cc / 2 holds columns cc = 2 (u % 4), 2 (u % 4) + 1 in its low and high half-word:
    //           the lane has cells u0 = 4 (r / 2) + 2 hq and u0 + 1; cell u < 15 is field u % 5 of word 2 (u / 5) + r % 2,
    //           cell 15 is spread over the top bits of the half-words of words r % 2, 2 + r % 2, 4 + r % 2.
    const int r = c & 7, par = r & 1, hq = q & 1;
    const int u0 = 4 * (r >> 1) + 2 * hq, u1 = u0 + 1;
    const bool spare = u1 == 15;
    // word (within the block) and shift of the lane's two cells; the spare cell is put together in the same form
    // (low code at bit 0, high code at bit 16) from the top bits of the three words
    const int wi0 = 2 * (u0 / 5) + par, sh0 = 3 * (u0 % 5);
    const int wi1 = spare ? par : 2 * (u1 / 5) + par, sh1 = spare ? 0 : 3 * (u1 % 5);
    // one byte of a register to fp32 in one instruction (v_cvt_f32_ubyte0 / 2)
    auto byte0 = [](uint32_t v) { return (float)(v & 0xFFu); };
    auto byte2 = [](uint32_t v) { return (float)((v >> 16) & 0xFFu); };
    auto lane_codes = [&](const uint32_t *blk, float *code) {
        if constexpr (BITS == 4) {
            const uint32_t w = blk[r] >> (8 * hq);
            const uint32_t t0 = w & 0x000F000Fu, t1 = (w >> 4) & 0x000F000Fu;
            code[0] = byte0(t0);
            code[1] = byte2(t0);
            code[2] = byte0(t1);
            code[3] = byte2(t1);
        } else {
            const uint32_t A = blk[par], B = blk[2 + par], C = blk[4 + par];
            const uint32_t S = ((A >> 15) & 0x00010001u) | ((B >> 14) & 0x00020002u) | ((C >> 13) & 0x00040004u);
            const uint32_t t0 = (blk[wi0] >> sh0) & 0x00070007u;
            const uint32_t t1 = ((spare ? S : blk[wi1]) >> sh1) & 0x00070007u;
            code[0] = byte0(t0);
            code[1] = byte2(t0);
            code[2] = byte0(t1);
            code[3] = byte2(t1);
        }
    };
    float below[NCT];                                      // the lower chunk's sums
    static_for<NRT / 4>([&](auto h_c) {
        constexpr int h = h_c.value;
        const int fh = k0 + 64 * h;
        const int chunk = fh >> 6, grp = fh / a.gsz;
        // zero-points of the lane's channels, fetched together and by every lane: inside the q == 0 branch below
        // each would be a load of its own with a full memory latency in front of the store
        float zv[NCT];
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct) {
            const size_t sg = (size_t)(cb + 16 * ct + c) * a.G + grp;
            zv[ct] = (float)global_load<uint8_t>(a.z0 + sg) + (a.dz ? global_load<float>(a.dz + sg) : 0.f);
        }
        static_for<NCT>([&](auto ct_c) {
            constexpr int ct = ct_c.value;
            const int i = cb + 16 * ct + c;
            // blocks of channel block (i / 8) % 16 = 8 (wn % 2) + 2 ct + c / 8 within the tiles of the run
            const uint32_t *ch_tile = reinterpret_cast<const uint32_t *>(code_lds) + (8 * (wn & 1) + 2 * ct + (c >> 3)) * 4 * WPB;
            float s1 = 0.f, s0 = 0.f;
            static_for<4>([&](auto r_c) {
                constexpr int rt = 4 * h + r_c.value;
                const f32x4 v = read_acc(acc[rt][ct]);
                // the lane's features k0 + 16 rt + 4 q + j: step tile rt / 2 of the run, block column 2 (rt % 2) + q / 2
                const uint32_t *blk = ch_tile + (rt >> 1) * 64 * WPB + (2 * (rt & 1) + (q >> 1)) * WPB;
                float code[4];
                lane_codes(blk, code);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    s1 += v[j] * code[j];
                    s0 += v[j];
                }
            });
            s1 += __shfl_xor(s1, 16); s0 += __shfl_xor(s0, 16);
            s1 += __shfl_xor(s1, 32); s0 += __shfl_xor(s0, 32);
            const float sum = s1 - zv[ct] * s0;
            if (a.gsz == 128) {                            // (uniform) the tile's two chunks are the group
                if constexpr (h == 0) below[ct] = sum;
                else if (q == 0) global_store(a.pc + (size_t)i * a.G + grp, below[ct] + sum);
            } else if (q == 0) {
                global_store(a.pc + (size_t)i * nchunks + chunk, sum);
            }
        });
    });
}

}  // namespace

}  // namespace peqa

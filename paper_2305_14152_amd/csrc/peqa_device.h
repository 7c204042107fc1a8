// Device-side helpers shared by the gfx950 kernels of the PEQA library:
// vector types for MFMA operands, bf16 <-> fp32 bit tricks, and the in-register
// unpacking of packed 3/4-bit codes into bf16 MFMA operand fragments.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace peqa {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// Codes are turned into bf16 without any int->float conversion: a b-bit code q placed
// in mantissa bits 3.. of the bf16 pattern of 16.0 (0x4180) denotes exactly 16 + q.
// Kernels contract against 16 + Q and take the constant offset (and the zero-point)
// out afterwards through row sums of the other operand.
constexpr float kCodeOffset = 16.0f;
constexpr uint32_t kMagic = 0x41804180u;   // two bf16 16.0
// The same trick in fp16: bits 6.. of 16.0 (0x4C00), for weights that are scaled before they enter the contraction.
constexpr uint32_t kMagicF16 = 0x4C004C00u;
// lowest mantissa bit of the field: 3 (bf16) or 6 (fp16); a b-bit field there in each half-word
constexpr int kFieldBf16 = 3, kFieldF16 = 6;
constexpr uint32_t field_mask(int bits, int at) { return ((1u << bits) - 1u) * 0x00010001u << at; }

__device__ __forceinline__ float bf16_lo(uint32_t pair) { return __uint_as_float(pair << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t pair) { return __uint_as_float(pair & 0xFFFF0000u); }

// Two fp32 -> bf16 bits, round to nearest even: one instruction (from integer operations, as before, seven; the epilogue of a
// 128 x 256 tile rounds 128 numbers a lane).
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{lo, hi}), bf16x2));
}
__device__ __forceinline__ uint32_t float_to_bf16_bits(float f) { return pack_bf16x2(f, 0.f) & 0xFFFFu; }

// A pair of fp16 (16 + code), scaled and shifted in fp32 and rounded once (to nearest even) to a bf16 pair:
// lo -> s_lo * lo + b_lo,  hi -> s_hi * hi + b_hi: two mixed-precision fused multiply-adds that take a half of the register
// as it stands (as bf16 the halves have to be moved into place first: two instructions more), and a conversion.  All of it is
// volatile assembly, so that every instruction stays where the caller put it among its matrix instructions: those are
// assembly too, and the wait states that the hardware wants between a vector write and a matrix read of the same register
// are the distance the caller keeps (the compiler, free to move the conversion, put it right before its use, and the matrix
// instruction read the old value).  In two parts, for other instructions in between.
struct ScaledPair {
    float lo, hi;
};
__device__ __forceinline__ ScaledPair scale_pair(uint32_t pair, float s_lo, float b_lo, float s_hi, float b_hi)
{
    ScaledPair p;
    asm volatile("v_fma_mix_f32 %0, %1, %2, %3 op_sel_hi:[1,0,0]" : "=v"(p.lo) : "v"(pair), "v"(s_lo), "v"(b_lo));
    asm volatile("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(p.hi) : "v"(pair), "v"(s_hi), "v"(b_hi));
    return p;
}
__device__ __forceinline__ uint32_t round_pair(const ScaledPair &p)
{
    uint32_t d;
    asm volatile("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(d) : "v"(p.lo), "v"(p.hi));
    return d;
}

// c + a.lo + a.hi of a bf16 pair, in fp32 (one dot instruction against ones).
__device__ __forceinline__ float add_pair(uint32_t a, float c)
{
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a), __builtin_bit_cast(bf16x2, 0x3F803F80u), c, false);
}

// ((x >> SH) & mask) | magic (a left shift where SH < 0) in two VALU ops, one when no shift is needed.  mask rides the
// constant bus (SGPR), magic a VGPR.  PINNED: volatile assembly, shift included, so that the unpacking stays exactly where
// the caller interleaves it with matrix instructions.  The hardware wants two wait states between a vector write and a matrix
// instruction that reads the register, and the compiler, which keeps them for every write that it emits itself, does not
// know of writes in assembly: PINNED is for callers whose matrix instructions are assembly too and a step away.
template <int SH, bool PINNED>
__device__ __forceinline__ uint32_t and_or(uint32_t x, uint32_t mask, uint32_t magic)
{
    if constexpr (!PINNED) {
        return ((SH >= 0 ? x >> (SH & 31) : x << (-SH & 31)) & mask) | magic;
    } else {
        uint32_t d;
        if constexpr (SH == 0)
            asm volatile("v_and_or_b32 %0, %1, %2, %3" : "=v"(d) : "v"(x), "s"(mask), "v"(magic));
        else if constexpr (SH > 0)
            asm volatile("v_lshrrev_b32 %0, %1, %2\n\tv_and_or_b32 %0, %0, %3, %4"
                         : "=&v"(d) : "n"(SH), "v"(x), "s"(mask), "v"(magic));
        else
            asm volatile("v_lshlrev_b32 %0, %1, %2\n\tv_and_or_b32 %0, %0, %3, %4"
                         : "=&v"(d) : "n"(-SH), "v"(x), "s"(mask), "v"(magic));
        return d;
    }
}

// Field number F (of width b) of both half-words of v -> pair of (16 + code): bf16, or, with AT = kFieldF16 and the matching
// magic, fp16.
template <int BITS, int F, int AT, bool PINNED>
__device__ __forceinline__ uint32_t field_pair(uint32_t v, uint32_t magic)
{
    return and_or<BITS * F - AT, PINNED>(v, field_mask(BITS, AT), magic);
}

// The 3-bit cell that lives in the spare top bits (15 and 31) of three words.
template <int AT, bool PINNED>
__device__ __forceinline__ uint32_t spare_pair3(uint32_t v0, uint32_t v1, uint32_t v2, uint32_t magic)
{
    uint32_t t = and_or<15 - AT, PINNED>(v0, 0x00010001u << AT, magic);
    t = and_or<14 - AT, PINNED>(v1, 0x00020002u << AT, t);
    return and_or<13 - AT, PINNED>(v2, 0x00040004u << AT, t);
}

// ---------------------------------------------------------------------------------
// Half of an 8x8 block of codes (8 channels x 8 features; 2 BITS words; layout: peqa_bit_location() in peqa.h) -> four
// operand fragments of 8 bf16 (4 registers) each, produced register by register so that callers can spread the unpacking
// between matrix instructions.  The two lanes c = 2b, 2b + 1 of a wave of 64 columns share block b.
//   along features, 4 bits: the lane has channels 4h .. 4h + 3 (h = c % 2): words 4h .. 4h + 3 of the block
//   along features, 3 bits: channels p, 2 + p, 4 + p, 6 + p (p = c % 2), which are exactly words p, 2 + p, 4 + p
//   along channels:         features p, 2 + p, 4 + p, 6 + p: the low (p = 0) or high half-words of all words, partner
//                           channels merged by one byte permute per word pair
// so that every lane runs the same shifts and masks.  Fragment I belongs to column 4 c + I of the wave's 64, or, by parity,
// 8 (c / 2) + 2 I + c % 2.
// ---------------------------------------------------------------------------------
template <int BITS, bool ALONG_CH, int AT = kFieldBf16, bool PINNED = true>
struct HalfBlockUnpacker {
    static constexpr int WORDS = ALONG_CH ? 2 * BITS : BITS;      // words a lane reads
    static constexpr bool BY_PARITY = ALONG_CH || BITS == 3;
    uint32_t w[BITS];

    // sel: along channels, the byte permute of this lane's half-words (0x05040100 for p = 0, 0x07060302 for p = 1)
    __device__ __forceinline__ void prepare(const uint32_t *words, uint32_t sel)
    {
#pragma unroll
        for (int m = 0; m < BITS; ++m) {
            if constexpr (ALONG_CH) w[m] = __builtin_amdgcn_perm(words[2 * m + 1], words[2 * m], sel);
            else w[m] = words[m];
        }
    }

    // register J (elements 2J, 2J + 1 of the contraction) of fragment I (0..3)
    template <int I, int J>
    __device__ __forceinline__ uint32_t frag_reg(uint32_t magic) const
    {
        if constexpr (BITS == 4) {
            if constexpr (ALONG_CH) return field_pair<4, I, AT, PINNED>(w[J], magic);
            else return field_pair<4, J, AT, PINNED>(w[I], magic);
        } else {
            constexpr int u = ALONG_CH ? 4 * J + I : 4 * I + J;
            if constexpr (u < 15) return field_pair<3, u % 5, AT, PINNED>(w[u / 5], magic);
            else return spare_pair3<AT, PINNED>(w[0], w[1], w[2], magic);
        }
    }
};

// The neighbouring lane's value (lanes 2i and 2i + 1 swap).
__device__ __forceinline__ float swap_pair_lane(float v)
{
    return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), 0xB1, 0xF, 0xF, true));
}

// Loads and stores that are global ones whatever the compiler knows of the pointer.  What comes out of an argument block at a run-time
// offset is a generic pointer to it and would be used by FLAT instructions, which count as LDS operations too: between two of
// them, and before the use of what one brings, the compiler waits for every operation in flight, stores included.
template <class T>
__device__ __forceinline__ T global_load(const void *p)
{
    return *(const __attribute__((address_space(1))) T *)(uintptr_t)p;
}
template <class T>
__device__ __forceinline__ void global_store(void *p, const T &v)
{
    *(__attribute__((address_space(1))) T *)(uintptr_t)p = v;
}

// Per-channel backward, the part of dY the dX contraction reads:  dYs[t,i] = bf16(dY[t,i] (s0 + ds)[i])  and
// crow[t] = sum_i dYs[t,i] (16 + z0[i] + dz[i])  (from the rounded dYs, so that it cancels the code offset of the
// contraction exactly), for the ROWS token rows of row block `blk`, by one workgroup of 256 threads
// (the per-channel parameters are read once per ROWS rows).  `red` is 4 ROWS floats of LDS.  Rows do not mix.
//
// Bound by latency: what a workgroup has in flight is ROWS x 4 KB, and the next columns are asked for before these are scaled (a launch
// of its own: 104 registers instead of 70, 2048 x 11008 19.4 -> 18.4 us, 500 x 11008 11.2 -> 10.9, 4096 x 22016 and 1000 x 16384 the same).
// Four rows where there are workgroups enough to fill the machine (a launch of its own), eight beside matrix work, where every
// place that the scaling holds for longer is one less for tiles, and half as many workgroups: backward of a 7B block 1218 -> 1190 us;
// dX alone with the scaling before it 649 -> 636.  (Sixteen rows: the registers do not hold them.)  Two in launches without tiles and with few blocks (launch_gemm_multi), and beside tiles of 64 rows, where
// there are no more than 64 tokens, which four or eight rows deal to few workgroups, and where two sets of columns of eight rows take the
// registers of a third workgroup on the unit (gemm_multi_kernel).  Training steps, us, eight rows and one set / four / two: d = 2048,
// f = 7040, T = 47 67.0 / 62.4 / 62.8, d = 2432, f = 7552, T = 18 70.6 / 66.1 / 64.4, d = 6656, f = 17920, T = 64 288 / 282 / 276,
// d = 8192, f = 22016, T = 64 388 / 386 / 383.
template <int ROWS>
__device__ __forceinline__ void scale_dy_rows(const uint16_t *__restrict__ dY, const float *__restrict__ s0,
                                              const float *__restrict__ ds, const uint8_t *__restrict__ z0,
                                              const float *__restrict__ dz, int T, int N, uint16_t *__restrict__ dYs,
                                              float *__restrict__ crow, int blk, float *red)
{
    const int tid = threadIdx.x;
    const int t0 = blk * ROWS, rows = min(ROWS, T - t0);
    const int n8s = N >> 3;
    float acc[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) acc[r] = 0.f;
    struct Columns {
        u32x4 v[ROWS];                                 // rows past T re-read the last one and are dropped
        f32x4 sa, sb, da, db, za, zb;
        u32x2 zz;
    };
    auto load = [&](int n8, Columns &k) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
            k.v[r] = global_load<u32x4>(dY + (size_t)(t0 + min(r, rows - 1)) * N + 8 * n8);
        k.sa = global_load<f32x4>(s0 + 8 * n8);
        k.sb = global_load<f32x4>(s0 + 8 * n8 + 4);
        if (ds) {
            k.da = global_load<f32x4>(ds + 8 * n8);
            k.db = global_load<f32x4>(ds + 8 * n8 + 4);
        }
        k.zz = global_load<u32x2>(z0 + 8 * n8);
        if (dz) {
            k.za = global_load<f32x4>(dz + 8 * n8);
            k.zb = global_load<f32x4>(dz + 8 * n8 + 4);
        }
    };
    // the next columns (and their parameters: loads arrive in order) are on their way while these are scaled
    Columns ahead;
    if (tid < n8s) load(tid, ahead);
    for (int n8 = tid; n8 < n8s; n8 += 256) {
        const Columns k = ahead;
        if (n8 + 256 < n8s) load(n8 + 256, ahead);
        float s[8] = {k.sa[0], k.sa[1], k.sa[2], k.sa[3], k.sb[0], k.sb[1], k.sb[2], k.sb[3]};
        float zo[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) zo[i] = kCodeOffset + (float)((k.zz[i >> 2] >> (8 * (i & 3))) & 0xFFu);
        if (ds) {
#pragma unroll
            for (int i = 0; i < 4; ++i) { s[i] += k.da[i]; s[4 + i] += k.db[i]; }
        }
        if (dz) {
#pragma unroll
            for (int i = 0; i < 4; ++i) { zo[i] += k.za[i]; zo[4 + i] += k.zb[i]; }
        }
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            u32x4 o;
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                o[p] = pack_bf16x2(bf16_lo(k.v[r][p]) * s[2 * p], bf16_hi(k.v[r][p]) * s[2 * p + 1]);
                acc[r] += bf16_lo(o[p]) * zo[2 * p] + bf16_hi(o[p]) * zo[2 * p + 1];
            }
            if (r < rows) global_store(dYs + (size_t)(t0 + r) * N + 8 * n8, o);
        }
    }
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) acc[r] += __shfl_xor(acc[r], o);
        if ((tid & 63) == 0) red[r * 4 + (tid >> 6)] = acc[r];
    }
    __syncthreads();
    if (tid < rows) global_store(crow + t0 + tid, (red[tid * 4] + red[tid * 4 + 1]) + (red[tid * 4 + 2] + red[tid * 4 + 3]));
}

// partial[0][j] + partial[1][j] + ... in that order (deterministic).
__device__ __forceinline__ float partials_sum(const float *__restrict__ partial, int ntiles, size_t n, size_t j)
{
    // eight loads in flight, added in tile order
    float s = 0.f;
    int tt = 0;
    for (; tt + 8 <= ntiles; tt += 8) {
        float p[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) p[u] = global_load<float>(partial + (size_t)(tt + u) * n + j);
#pragma unroll
        for (int u = 0; u < 8; ++u) s += p[u];
    }
    for (; tt < ntiles; ++tt) s += global_load<float>(partial + (size_t)tt * n + j);
    return s;
}

// out[j] = that sum
__device__ __forceinline__ void reduce_partials_at(const float *__restrict__ partial, int ntiles, size_t n, size_t j,
                                                   float *__restrict__ out)
{
    if (j < n) global_store(out + j, partials_sum(partial, ntiles, n, j));
}

// The step-major transposed copy that the token contraction of group-wise layers reads:
// dst[t / 32][cc / 16][(t % 32) / 8][cc % 16][t % 8] = src[t, cc] for t < T, 0 for T <= t < Tp (the KB of 16 columns and a
// step is one matrix operand, lane by lane), C % 64 == 0, by one wave per 64 x 64 tile (bt, bc) of tokens x columns.
//
// Bound by memory where it has the machine to itself; beside matrix work by what it takes of LDS, of the vector units and of a
// place on a compute unit.  So a lane reads 8 columns of 8 tokens, 16 bytes each (transpose_load), turns them into 8 columns' pieces
// of 8 tokens in registers (32 byte permutes), and the pieces only change lanes in LDS, 16 bytes at a time, so that the stores are whole
// KB; nothing but the wave itself waits, and the next tile's loads are on their way meanwhile.
// By workgroups that moved 2 bytes at a time through LDS between two barriers, the copies of a 13B block (T = 2048, 675 MB read and
// written) lengthened the dX launch that they ride in by 140 us, and by 50 so (1283 -> 1196 -> 1159 us with the tiles' other changes).
struct TransposeRows {
    u32x4 row[8];                                          // tokens 8 (lane / 8) + j, columns 8 (lane % 8) .. + 7 of the tile
};
__device__ __forceinline__ void transpose_load(const uint16_t *__restrict__ src, int T, int C, int bt, int bc, TransposeRows &r)
{
    const int lane = threadIdx.x & 63, t0 = bt * 64 + 8 * (lane >> 3);
    const uint16_t *from = src + (size_t)bc * 64 + 8 * (lane & 7);
    if (bt * 64 + 64 <= T) {                               // (uniform)
#pragma unroll
        for (int j = 0; j < 8; ++j) r.row[j] = global_load<u32x4>(from + (size_t)(t0 + j) * C);
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            r.row[j] = u32x4{0u, 0u, 0u, 0u};
            if (t0 + j < T) r.row[j] = global_load<u32x4>(from + (size_t)(t0 + j) * C);
        }
    }
}
// `piece`: 8 KB of LDS of this wave's own.  Pieces lie there in the order of the copy, eight of them (128 bytes) permuted by the column
// block of the lane that wrote them: writes and reads of eight lanes then fall into different banks.
constexpr int TRANSPOSE_LDS = 8192;                        // per wave
__device__ __forceinline__ void transpose_store(const TransposeRows &r, int C, uint16_t *__restrict__ dst, int bt, int bc, u32x4 *piece)
{
    const int lane = threadIdx.x & 63, cb = lane & 7, tb = lane >> 3;
    const int at = (((tb >> 2) * 4 + (cb >> 1)) * 4 + (tb & 3)) * 16 + 8 * (cb & 1);   // step, 16 columns, 8 tokens, column
#pragma unroll
    for (int w = 0; w < 4; ++w)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            u32x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                o[e] = __builtin_amdgcn_perm(r.row[2 * e + 1][w], r.row[2 * e][w], h ? 0x07060302u : 0x05040100u);
            piece[at + ((2 * w + h) ^ cb)] = o;
        }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    uint16_t *to = dst + ((size_t)(2 * bt) * C + (size_t)bc * 64) * 32 + 8 * lane;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int p = 64 * i + lane, writer = ((p >> 3) & 1) | (((p >> 6) & 3) << 1);
        global_store(to + (i >> 2) * (size_t)C * 32 + (i & 3) * 512, piece[p ^ writer]);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();                       // the next tile's pieces overwrite these
}
__device__ __forceinline__ void transpose_pad_tile(const uint16_t *__restrict__ src, int T, int C, uint16_t *__restrict__ dst, int bt,
                                                   int bc, u32x4 *piece)
{
    TransposeRows r;
    transpose_load(src, T, C, bt, bc, r);
    transpose_store(r, C, dst, bt, bc, piece);
}

// 16 columns of such a tile by one wave, the quarter'th, without LDS: a lane has 2 columns of 8 tokens, which is two neighbouring pieces.
// For launches of few tiles, which the chain of a wave's own instructions bounds (a quarter of them here).  Scale gradient alone of one layer, us,
// a tile per wave / four waves per tile: 256 x 384, T = 125 (20 tiles) 9.06 / 8.83, 640 x 7552, T = 32 (128) 9.34 / 8.97, 2048 x 1536,
// T = 845 (784) 25.1 / 25.2, 1664 x 4096, T = 2352 (3330) 42.3 / 42.4.
__device__ __forceinline__ void transpose_pad_quarter(const uint16_t *__restrict__ src, int T, int C, uint16_t *__restrict__ dst, int bt,
                                                      int bc, int quarter)
{
    const int lane = threadIdx.x & 63, c2 = lane & 7, tb = lane >> 3, t0 = bt * 64 + 8 * tb, col = bc * 64 + quarter * 16;
    uint32_t row[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) row[j] = global_load<uint32_t>(src + (size_t)min(t0 + j, T - 1) * C + col + 2 * c2);
#pragma unroll
    for (int j = 0; j < 8; ++j) row[j] = t0 + j < T ? row[j] : 0u;
    uint16_t *to = dst + ((size_t)(2 * bt + (tb >> 2)) * C + col) * 32 + ((tb & 3) * 16 + 2 * c2) * 8;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        u32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = __builtin_amdgcn_perm(row[2 * e + 1], row[2 * e], h ? 0x07060302u : 0x05040100u);
        global_store(to + 8 * h, o);
    }
}

// Tile b of a launch of copies: along the columns first where workgroups take four (neighbours share rows of the source), else along the
// tokens (1664 x 4096, T = 2352, scale gradient alone 42.3 us along the columns, 41.4 so; 22016 x 8192, T = 700 214 and 216).
struct CopyTile {
    int bt, bc;
};
__device__ __forceinline__ CopyTile copy_tile(int b, int bts, int bcs, int per_wg)
{
    return per_wg == 4 ? CopyTile{b / bcs, b % bcs} : CopyTile{b % bts, b / bts};
}

// A piece of the kernel's argument block read at a run-time (wavefront-uniform) byte offset: scalar loads from the
// kernarg segment.  Indexing an array inside a by-value kernel argument with a run-time index would make the
// compiler keep a private copy of the whole argument in scratch memory; this reads the segment itself.
typedef uint32_t __attribute__((may_alias)) u32_alias;
template <class T>
__device__ __forceinline__ T kernarg_load(uint32_t byte_offset)
{
    static_assert(sizeof(T) % 4 == 0, "whole dwords");
    typedef const __attribute__((address_space(4))) u32_alias *cptr;
    const cptr p = (cptr)((const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr() + byte_offset);
    T out;
    u32_alias *o = reinterpret_cast<u32_alias *>(&out);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(T) / 4); ++i) o[i] = p[i];
    return out;
}

// n / d and n % d of wavefront-uniform numbers with the host's magic = (2^32 - 1) / d: the product's high half is the quotient or
// one less.  A few scalar instructions; the compiler's division is a chain of twenty vector instructions, 0.1 us each time
// in the start of a kernel that lasts 5.
struct Quotient {
    uint32_t q, r;
};
__device__ __forceinline__ Quotient div_magic(uint32_t n, uint32_t d, uint32_t magic)
{
    uint32_t q = (uint32_t)(((uint64_t)n * magic) >> 32), r = n - q * d;
    const bool up = r >= d;
    r -= up ? d : 0u;
    q = up ? q + 1u : q;
    return {q, r};
}

// div_magic's reciprocal of a number from 1 to 8
__device__ __forceinline__ uint32_t small_magic(int d)
{
    const uint32_t low = d == 1 ? 0xFFFFFFFFu : d == 2 ? 0x7FFFFFFFu : d == 3 ? 0x55555555u : 0x3FFFFFFFu;
    const uint32_t high = d == 5 ? 0x33333333u : d == 6 ? 0x2AAAAAAAu : d == 7 ? 0x24924924u : 0x1FFFFFFFu;
    return d < 5 ? low : high;
}

// s_barrier alone: no implied wait on outstanding LDS or memory operations.
__device__ __forceinline__ void bare_barrier() { asm volatile("s_barrier" ::: "memory"); }

// D = A * B + C on one 16x16 tile with a 32-deep contraction (compiler-scheduled form).
__device__ __forceinline__ f32x4 mfma16(const u32x4 &a, const u32x4 &b, const f32x4 &c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// D += A * B on one 16x16 tile with a 32-deep contraction.  Issued as inline assembly with the
// accumulator tied to an AGPR tuple: with the builtin, this compiler keeps rotating part of a
// 256-register accumulator set through VGPRs on every loop iteration.  The hardware does not
// interlock a read of the result by a non-matrix instruction: callers must put at least 18 wait
// states (mfma_result_fence) between the last of these and the first such read.
__device__ __forceinline__ void mfma16_acc(f32x4 &acc, const u32x4 &a, const u32x4 &b)
{
    // volatile: keeps the source order of the matrix instructions among themselves and relative
    // to the DMA queueing and the result fence (the scalar/vector work around them is still free)
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
// An accumulator tile copied from its AGPRs to VGPRs at this point of the program (volatile: the
// compiler would otherwise gather every such copy of a kernel at one place).
__device__ __forceinline__ f32x4 read_acc(const f32x4 &acc)
{
    f32x4 v;
    asm volatile("v_accvgpr_read_b32 %0, %4\n\tv_accvgpr_read_b32 %1, %5\n\tv_accvgpr_read_b32 %2, %6\n\tv_accvgpr_read_b32 %3, %7"
                 : "=v"(v[0]), "=v"(v[1]), "=v"(v[2]), "=v"(v[3])
                 : "a"(acc[0]), "a"(acc[1]), "a"(acc[2]), "a"(acc[3]));
    return v;
}
__device__ __forceinline__ void mfma_result_fence()
{
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
}

// Global -> LDS DMA of 16 bytes per lane: lane l's bytes land at lds_dst + 16 l.  The source
// is sbase (uniform) + voff (per lane).  Issued from inline assembly so that the compiler does not
// serialise the ring with a conservative vmcnt(0); completion is tracked by hand with wait_vmcnt().
__device__ __forceinline__ void dma16(uint32_t voff, const void *sbase, uint32_t lds_dst)
{
    // sbase is the same in every lane; saying so keeps it in scalar registers wherever the compiler cannot tell.  Where that
    // takes an instruction, a vector one, the hardware wants five wait states before the DMA and gets two here: callers keep
    // their pointers scalar, or form them well ahead (the build looks at the code that comes out, see build.py).
    const uint64_t u = (uint64_t)(uintptr_t)sbase;
    const uint64_t ub = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(u >> 32)) << 32) |
                        (uint32_t)__builtin_amdgcn_readfirstlane((int)u);
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :: "v"(voff), "s"(ub), "s"(lds_dst) : "memory");
}
// Activation tiles sit in LDS as rows of 64 B (four 16-byte chunks).  Chunk j of row r is stored at
// position j ^ a_swizzle(r): with it, the 16-byte reads of 8 (16) consecutive rows at one logical
// chunk fall into 8 (16) different 16-byte bank groups of a 128 (256) byte LDS line.
__device__ __forceinline__ int a_swizzle(int row) { return ((row >> 1) & 3) ^ ((row >> 3) & 1); }

template <int N, class F>
__device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (N > 0) {
        static_for<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}

template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    // gfx9 encoding: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt[5:4] << 14; other counters left open
    __builtin_amdgcn_s_waitcnt((N & 0xF) | (0x7 << 4) | (0xF << 8) | ((N >> 4) << 14));
}

}  // namespace peqa

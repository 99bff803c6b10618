// Device-side helpers shared by the bf16 MFMA kernels (gfx950).
//
// MFMA operand layouts, M x M results, K = 512 / M (lane l of a 64-wide wavefront, group = l / M: halves or quarters):
//   A (M x K): lane holds row  m = l % M, k = 8*group + 0..7        (bf16x8)
//   B (K x N): lane holds col  n = l % M, k = 8*group + 0..7        (bf16x8)
//   C/D (M x N, fp32): lane holds col n = l % M, register i <-> row (i/4)*8 + 4*group + i%4
//                      (M = 32: 16 registers; M = 16: 4 registers, i.e. row 4*group + i)
// head_dim 128 multiplies with M = 16 (the gradient accumulators of its dK/dV kernel apart, and small calls, wide_mfma()): launches
// that fill the chip are limited by the card's power, and on N(0,1) operands the 16x16x32 instruction does more per joule (a sum of
// 32 products per accumulator update instead of 16): a loop of nothing but MFMAs runs at 1990-2030 TFLOP/s with M = 16 and at 1800 with
// M = 32.  32768 queries of 64 / 8 heads over 131072 keys: forward 111.9 -> 105.5 ms, dQ 153.5 -> 141.0, dK/dV 207.4 -> 199.5.
// head_dim 64, which splits P and dS into three operands and is bound by vector instructions, keeps M = 32: half as many MFMAs to
// issue (16 x 16: 2.5 % slower).
//
// ds_read_tr16_b64 (transposing LDS read): inside each block of 16 lanes, lane r supplies the address
// of 4 consecutive 16-bit elements; the 16x4 elements are handed out so that lane i receives
// element (i % 4) of the rows supplied by lanes i/4, 4 + i/4, 8 + i/4, 12 + i/4.  With lane r
// pointing at mem[k0 + r/4][n0 + 4*(r%4)] (a 4 x 16 block of a row-major matrix), lane i therefore
// gets mem[k0 + 0..3][n0 + i]: four consecutive k for one n -- half of an MFMA operand whose
// contraction index runs along the matrix rows.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "chunkflow.h"

namespace cf {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

#define CF_LDS __attribute__((address_space(3)))
#define CF_GLOBAL __attribute__((address_space(1)))
#define CF_CONSTANT __attribute__((address_space(4)))

template <int SIZE>
struct Mfma {
    static constexpr int M = SIZE, K = 512 / M;
    static constexpr int R = M * M / 64;             // registers of a result
    static constexpr int N32 = 32 / M;               // blocks of M that make 32
    typedef float Acc __attribute__((ext_vector_type(R)));
    // The registers of results below each other, read as one array: element i is row place(i) + 4 * group, and elements 8 t .. 8 t + 7
    // are the operand of contraction group t (rows K t .. K t + K - 1), in the order in which LaneOffsets' transposing reads
    // fetch the other operand.
    __host__ __device__ static constexpr int place(int i) { return i / R * M + i % R / 4 * 8 + i % 4; }
    __device__ __forceinline__ static int group() { return (int)(threadIdx.x & 63) / M; }
    __device__ __forceinline__ static int column() { return (int)(threadIdx.x & 63) % M; }
    __device__ __forceinline__ static Acc zero()
    {
        Acc a;
#pragma unroll
        for (int i = 0; i < R; ++i) a[i] = 0.f;
        return a;
    }
    __device__ __forceinline__ static Acc mul(bf16x8 a, bf16x8 b, Acc c)
    {
        if constexpr (M == 32) return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
        else return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
};

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// acc += A B with the accumulator updated where it stands.  The builtin lets the compiler choose another register block
// for the result, and across branches it does: 128 accumulator registers then need up to 128 more, and spill.  (D = 64
// has registers to spare.)  Only for accumulators that nothing but this reads or writes inside the loop: what the
// compiler cannot see here is the latency before another instruction may read them (accumulators_done), and that
// operands just written by vector instructions need two wait states.
template <int D>
__device__ __forceinline__ void accumulate_in_place(f32x16 &acc, bf16x8 a, bf16x8 b)
{
    if (D == 64) acc = mfma32(a, b, acc);
    else asm("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
}
// Before the first other use of an accumulator: lets its last MFMA (8 passes) finish.
__device__ __forceinline__ void accumulator_done(f32x16 &acc) { asm volatile("s_nop 15" : "+v"(acc)); }

// Two transposing reads; result is one bf16x8 operand.
__device__ __forceinline__ bf16x8 lds_read_tr_pair(const char *lo_addr, const char *hi_addr)
{
    s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((CF_LDS s16x4 *)lo_addr);
    s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((CF_LDS s16x4 *)hi_addr);
    s16x8 r = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, r);
}

__device__ __forceinline__ bf16x8 lds_read_b128(const char *addr)
{
    return *(const bf16x8 *)addr;
}

// Packs 8 fp32 values into a bf16x8 (round to nearest even; v_cvt_pk_bf16_f32 on gfx950).
__device__ __forceinline__ bf16x8 pack8(const float (&f)[8])
{
    bf16x8 r;
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = (__bf16)f[e];
    return r;
}

// Eight fp32 values as three bf16 operands: x = w[0] + w[1] + w[2] exactly (8 of the 24 significant bits each, taken off by
// truncation), so that three MFMAs multiply the fp32 value and not its rounding.
__device__ __forceinline__ void split_exact(const float (&f)[8], bf16x8 (&w)[3])
{
    i32x4 u[3];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float x0 = f[2 * e], x1 = f[2 * e + 1];
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const unsigned b0 = __float_as_uint(x0), b1 = __float_as_uint(x1);
            u[t][e] = __builtin_amdgcn_perm(b1, b0, 0x07060302);      // the upper halves of both
            x0 -= __uint_as_float(b0 & 0xffff0000u);
            x1 -= __uint_as_float(b1 & 0xffff0000u);
        }
    }
#pragma unroll
    for (int t = 0; t < 3; ++t) w[t] = __builtin_bit_cast(bf16x8, u[t]);
}

// Swizzled LDS tile with rows of 2 D bytes (D bf16) and no padding: the 16-byte unit u of row r lives at unit
// u ^ swz(r).  LDS has 64 four-byte banks; a 16-byte row read (ds_read_b128) is served 16 lanes per clock and a
// transposing 8-byte read (ds_read_b64_tr_b16) 32 lanes per clock.  D = 128: a row covers the banks once.  Bits 2, 3 of
// swz() are the row's lowest two: the 4 consecutive rows of a transposing read lie in 4 different groups of 4 units.  The low
// two are a function f of a = row / 4 % 4, f = 0, 2, 3, 1:
//   M = 32  a row read takes one unit of 16 rows at a time (any f that is one to one), a transposing read four units of 4 rows;
//   M = 16  a row read is served in groups of lanes 0-3, 12-15, 20-23, 24-27 and 4-11, 16-19, 28-31: unit u of the rows with
//           a = 0, 3 beside unit u + 1 of those with a = 1, 2, and the other way round; f(0), f(3), f(1)^1, f(2)^1 all differ.
//           A transposing read takes two units of the rows a = 0 beside the same two of a = 1 (2 beside 3): f differs in bit 1.
// Both are free of conflicts (counted; with f = 0, 2, 1, 3 every row read of M = 16 took twice as long).  D = 64: two rows
// cover the banks, an even and an odd row never meet, and the row's bit 1 takes the place of its lowest two.
template <int D>
__device__ __forceinline__ int swz(int row)
{
    static_assert(D == 64 || D == 128, "row length");
    const int low = (((row >> 2) ^ (row >> 3)) & 1) << 1 | ((row >> 3) & 1);
    return D == 128 ? ((row & 3) << 2) | low : (((row >> 1) & 1) << 2) | low;
}
template <int D>
__device__ __forceinline__ int tile_off(int row, int unit) { return row * (2 * D) + ((unit ^ swz<D>(row)) << 4); }

// Lane-constant LDS byte offsets into a swizzled tile, computed once per kernel (the XOR of the swizzle
// cannot be folded into an instruction's immediate offset, so every distinct unit needs its own register;
// keeping them in registers beats recomputing them for each of the LDS reads of a tile).
//
//  row_unit[ks]  operand rows read with ds_read_b128 (MFMA row/col = tile row, contraction along the tile
//                row): offset of (row = lane % M, logical unit K / 8 * ks + group).  An M-row block further down
//                the tile adds M rows (swz() has period 16 rows).
//  tr_lo[db], tr_hi(db)
//                operands read with the transposing read (contraction along the tile's ROWS, MFMA
//                row/col = tile column M*db + lane % M): offsets of the two 4-row reads that make one
//                bf16x8 operand, for contraction rows 4*group + {0..3 by lane} and 8 (M = 32) or 16 rows further.
//                K rows further down the tile add K row lengths.
template <int D, int M>
struct LaneOffsets {
    static constexpr int UNITS = Mfma<M>::K / 8;
    int row_unit[D / 8 / UNITS];
    int tr_lo[D / M], tr_hi8[M == 32 ? D / M : 1];
    __device__ __forceinline__ int tr_hi(int db) const { return M == 32 ? tr_hi8[db] : tr_lo[db] + 16 * 2 * D; }
};
template <int D, int M>
__device__ __forceinline__ LaneOffsets<D, M> lane_offsets()
{
    constexpr int UNITS = LaneOffsets<D, M>::UNITS;
    const int lane = threadIdx.x & 63, group = lane / M, r16 = lane & 15, blk = M == 32 ? (lane >> 4) & 1 : 0;
    LaneOffsets<D, M> o;
#pragma unroll
    for (int ks = 0; ks < D / 8 / UNITS; ++ks) o.row_unit[ks] = tile_off<D>(lane % M, UNITS * ks + group);
    const int r_lo = 4 * group + (r16 >> 2), u0 = 2 * blk + ((r16 >> 1) & 1), sub = 8 * (r16 & 1);
#pragma unroll
    for (int db = 0; db < D / M; ++db) {
        o.tr_lo[db] = tile_off<D>(r_lo, M / 8 * db + u0) + sub;
        if (M == 32) o.tr_hi8[db] = tile_off<D>(r_lo + 8, M / 8 * db + u0) + sub;
    }
    return o;
}

// The offsets of the dK/dV kernel, which has no registers to spare: all follow from two bases by XOR (a row's units differ in
// bits above the group's; so do the halves of a transposed operand, of rows FIRST * half + 0..3 and STEP rows further, whose
// columns are those of M = 32), one instruction per read.
// forget(): from here on the compiler computes them anew instead of keeping the results of the last use.
template <int D, int M>
struct BlockAddress {
    static constexpr int STEP = M == 32 ? 8 : 4, FIRST = 12 - STEP;
    int row0, tr0;
    __device__ __forceinline__ BlockAddress()
    {
        const int lane = threadIdx.x & 63, r16 = lane & 15;
        row0 = lane_offsets<D, M>().row_unit[0];
        tr0 = tile_off<D>(FIRST * (lane >> 5) + (r16 >> 2), 2 * ((lane >> 4) & 1) + ((r16 >> 1) & 1)) + 8 * (r16 & 1);
    }
    // to the block `bytes` (a power of two beyond a block's size) further, and back
    __device__ __forceinline__ void flip(int bytes) { row0 ^= bytes, tr0 ^= bytes; }
    __device__ __forceinline__ void forget() { asm volatile("" : "+v"(row0), "+v"(tr0)); }
    __device__ __forceinline__ int row(int ks) const { return row0 ^ (ks * LaneOffsets<D, M>::UNITS * 16); }
    __device__ __forceinline__ int tr_lo(int db) const { return tr0 ^ (db << 6); }
    __device__ __forceinline__ int tr_hi(int db) const { return (tr_lo(db) ^ ((STEP == 8 ? 3 : 2) << 4)) + STEP * 2 * D; }
};

// Index of this wavefront inside its workgroup, as a value the compiler knows to be wave-uniform.
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }

// This lane's index, made anew where it is asked for: nothing that follows from it is kept in a register in between.
__device__ __forceinline__ int fresh_lane()
{
    int lane;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
    return lane;
}

// Direct global -> LDS copy of a swizzled tile of ROWS rows of D bf16 by a workgroup of WAVES wavefronts
// (buffer_load_dwordx4 ... lds: no staging registers; lane i of one instruction lands at LDS base + 16*i, so
// one instruction fills RPI = 512 / D tile rows and the swizzle is applied on the global side: the lane that fills
// physical unit u' of row r fetches logical unit u' ^ swz(r)).
// A tile takes ROWS / (RPI * WAVES) instructions per wavefront (PARTS); each costs the issuing wavefront some 30-45 clocks
// wherever it is placed (measured), so they are simply issued together at the start of a tile.
// Addressing is the buffer form on purpose: the tile's first row is a wave-uniform pointer that becomes the
// base of a buffer descriptor (scalar arithmetic), the lane's place inside a tile is ONE register (two where a part is half a
// swizzle period) computed at init, and a part adds a scalar offset, so a full tile costs no vector address arithmetic at all.  Only
// a ragged tile (rows beyond last_row, relative to src, re-read last_row; the caller masks them) computes
// clamped per-lane offsets.  The descriptor's size field is left at its maximum: nothing relies on the
// hardware's out-of-range behaviour.
// BLOCKS: the 32-row blocks that begin behind last_row are left as they are (for readers that pass over them: in the backward of
// 16 packed chunks of 512 tokens, 28 / 4 heads, most tiles are of sequences of up to 32 or 64 rows: 235 -> 228 us the step).
// Completion is tracked by vmcnt: wait_lds_dma() before the barrier that publishes the tile.
template <int ROWS, int D, int WAVES = 4, bool BLOCKS = false>
struct TileDma {
    static constexpr int RPI = 512 / D, UNITS = D / 8;      // rows per instruction, 16-byte units per row
    static constexpr int PARTS = ROWS / (RPI * WAVES);
    static constexpr int KINDS = (RPI * WAVES) % 16 == 0 ? 1 : 2;     // parts of half a swizzle period: even and odd ones
    static_assert(PARTS >= 1 && (RPI * WAVES) % 8 == 0, "a part must cover whole swizzle periods or halves");
    unsigned row_bytes;
    unsigned unit16[KINDS];       // byte offset of this lane's 16-byte unit inside its row
    int r0;                       // this lane's row in part 0; part c adds RPI * WAVES rows
    int wv;                       // index of this wavefront among the copying ones
    unsigned lane_off[KINDS];     // r0 * row_bytes + unit16: this lane's offset in a part of a full tile, from the part's first row

    // wave: index of the calling wavefront among the WAVES that copy (wave-uniform)
    __device__ __forceinline__ void init(int64_t row_bytes_, int wave, int lane)
    {
        row_bytes = (unsigned)row_bytes_;
        wv = wave;
        r0 = RPI * wave + lane / UNITS;
#pragma unroll
        for (int i = 0; i < KINDS; ++i) {            // swz() has period 16 rows
            unit16[i] = ((lane % UNITS) ^ swz<D>(r0 + RPI * WAVES * i)) * 16;
            lane_off[i] = (unsigned)r0 * row_bytes + unit16[i];
        }
    }
    __device__ __forceinline__ void init(int64_t row_bytes_) { init(row_bytes_, wave_id(), threadIdx.x & 63); }
    __device__ __forceinline__ CF_LDS void *part_dst(char *lds_tile, int c) const { return (CF_LDS void *)(lds_tile + (c * WAVES + wv) * 1024); }
    __device__ __forceinline__ static __amdgpu_buffer_rsrc_t descriptor(const char *src)
    {
        return __builtin_amdgcn_make_buffer_rsrc((void *)src, 0, -1, 0x00020000);
    }
    __device__ __forceinline__ void full_part(__amdgpu_buffer_rsrc_t rsrc, char *lds_tile, int c) const
    {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, part_dst(lds_tile, c), 16, (int)lane_off[c % KINDS], (int)(RPI * WAVES * c * row_bytes), 0, 0);
    }
    __device__ __forceinline__ void ragged_part(__amdgpu_buffer_rsrc_t rsrc, int last_row, char *lds_tile, int c) const
    {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, part_dst(lds_tile, c), 16,
                                                 (int)((unsigned)min(r0 + RPI * WAVES * c, last_row) * row_bytes + unit16[c % KINDS]), 0, 0, 0);
    }
    // last_row is wave-uniform, so the branch below is a scalar one.
    __device__ __forceinline__ void issue(const char *src, int last_row, char *lds_tile) const
    {
        const __amdgpu_buffer_rsrc_t rsrc = descriptor(src);
        if (last_row >= ROWS - 1) {
#pragma unroll
            for (int c = 0; c < PARTS; ++c) full_part(rsrc, lds_tile, c);
        } else {
#pragma unroll
            for (int c = 0; c < PARTS; ++c)
                if (!BLOCKS || RPI * WAVES * c / 32 * 32 <= last_row) ragged_part(rsrc, last_row, lds_tile, c);
        }
    }
};
// Makes a pointer / an int that is the same in every lane known as such to the compiler.
template <typename T>
__device__ __forceinline__ T *uniform(T *p)
{
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (T *)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
// A float that is the same in every lane, in a scalar register (what the vector unit computed would stay in a vector
// register: scalar float arithmetic does not exist here, and a readfirstlane of a uniform value is folded away, so the value passes
// through assembly of no instruction first).  The read itself is the compiler's: it needs a wait state behind the instruction that wrote
// its register, and what uses its result up to five behind it, which the compiler keeps for its own instructions only.
__device__ __forceinline__ float scalar(float x)
{
    asm("" : "+v"(x));
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x)));
}
__device__ __forceinline__ void wait_lds_dma() { __builtin_amdgcn_s_waitcnt(0x0F70); }   // vmcnt(0)

// What a workgroup needs of its chunk's arguments to find its rows and to ask for them, loaded together: the compiler fetches an argument
// where it is first used, each time with a wait of its own, eight or nine in a row before the first row was asked for, now three or four.
// Steps, with KeyArgs (dK/dV): 16 packed chunks of 512 tokens, 28 / 4 heads 213 -> 210 us; 16 / 4 heads, D = 64, five chunks of 4096 749 -> 742;
// packed chunks of 8192 as before, within the 0.5-1 % that runs of one side differ.
struct RowArgs {
    const char *q, *k, *v;
    int64_t q_tok, q_head, kv_tok, kv_head;          // strides, in elements
    const cf_q_tile *tiles;
    int n_tiles, n_q_heads, n_kv_heads;
    template <typename Params>
    __device__ __forceinline__ explicit RowArgs(const Params &p, bool together = true)
        : q_tok(p.q_stride_tok), q_head(p.q_stride_head), kv_tok(p.kv_stride_tok), kv_head(p.kv_stride_head), n_tiles(p.n_q_tiles),
          n_q_heads(p.n_q_heads), n_kv_heads(p.n_kv_heads)
    {
        // (one instruction that all of them go through; the pointers as ones to global and to constant memory, or flat loads would follow)
        auto q_ = (const CF_GLOBAL char *)p.q, k_ = (const CF_GLOBAL char *)p.k, v_ = (const CF_GLOBAL char *)p.v;
        auto tiles_ = (const CF_CONSTANT cf_q_tile *)p.q_tiles;
        if (together)
            asm("" : "+s"(q_), "+s"(k_), "+s"(v_), "+s"(q_tok), "+s"(q_head), "+s"(kv_tok), "+s"(kv_head), "+s"(tiles_), "+s"(n_tiles),
                 "+s"(n_q_heads), "+s"(n_kv_heads));
        q = (const char *)q_, k = (const char *)k_, v = (const char *)v_, tiles = (const cf_q_tile *)tiles_;
    }
};

// The 128-row query tile of workgroup rank `rank` from the caller's table (cf_attn_q_tiles: heaviest tile first,
// each record carries its segment's bounds): one uniform 32-byte read instead of the search of locate_tile.
struct QTile {
    int tile_in_seg, q_begin, q_len, k_begin, k_len;
};
__device__ __forceinline__ QTile read_q_tile(const cf_q_tile *table, int rank)
{
    const i32x4 *rec = (const i32x4 *)(table + rank);
    const i32x4 a = rec[0], b = rec[1];
    return QTile{uniform(b[0]), uniform(a[0]), uniform(a[1]), uniform(a[2]), uniform(a[3])};
}

// Stores a wavefront's 32 x D block of bf16 results (computed transposed: a lane owns row M n + lane % M of acc[..][n], four
// registers are 4 consecutive d) to global rows of 2 D bytes.
// A direct store would write 8-byte pieces of many different rows per instruction (a cache line touched per
// lane, 16 instructions); instead the block is turned around in `scratch` (this wavefront's own
// 32 padded rows of LDS, free at that point) and leaves as D / 16 instructions that each write 512 / D whole rows.
//   row_ptr(r): global address of row r of the block (r = 0..31), rows >= rows_valid are not written
template <int D>
struct RowScratch {
    static constexpr int stride = 2 * D + 16;       // keeps 16-byte alignment, spreads rows over banks
    static constexpr int bytes = 32 * stride;
};
template <int D, int M>
using RowBlock = typename Mfma<M>::Acc[D / M][Mfma<M>::N32];
template <int D, int M, typename RowPtr>
__device__ __forceinline__ void store_rows_bf16(const RowBlock<D, M> &acc, const float (&scale)[Mfma<M>::N32], char *scratch, int rows_valid,
                                                RowPtr row_ptr)
{
    constexpr int S = RowScratch<D>::stride, UNITS = D / 8, RPI = 512 / D;
    using F = Mfma<M>;
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int n = 0; n < F::N32; ++n)
#pragma unroll
        for (int i = 0; i < D * F::R / F::M; i += 4) {
            bf16x4 w;
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = (__bf16)(acc[i / F::R][n][i % F::R + e] * scale[n]);
            *(bf16x4 *)(scratch + (n * F::M + F::column()) * S + (F::place(i) + 4 * F::group()) * 2) = w;
        }
    __builtin_amdgcn_wave_barrier();
    bf16x8 v[D / 16];
#pragma unroll
    for (int i = 0; i < D / 16; ++i) v[i] = *(const bf16x8 *)(scratch + (RPI * i + lane / UNITS) * S + (lane % UNITS) * 16);
#pragma unroll
    for (int i = 0; i < D / 16; ++i) {
        const int r = RPI * i + lane / UNITS;
        if (r < rows_valid) *(bf16x8 *)(row_ptr(r) + (lane % UNITS) * 16) = v[i];
    }
}

// visit(r), by the whole wavefront, for every row r < rows_valid of a 32 x D block (as above, D = 64: a lane owns row lane % 32) whose
// results, scaled, are not finite.
template <int D, typename Visit>
__device__ __forceinline__ void for_rows_not_finite(const RowBlock<D, 32> &acc, float scale, int rows_valid, Visit visit)
{
    float zero = scale * 0.f;                        // stays 0 while everything is finite
#pragma unroll
    for (int j = 0; j < D / 32; ++j)
#pragma unroll
        for (int i = 0; i < 16; ++i) zero = __builtin_fmaf(acc[j][0][i], 0.f, zero);
    const unsigned long long lanes = __ballot(zero != 0.f);
    unsigned rows = (unsigned)lanes | (unsigned)(lanes >> 32);
    if (rows_valid < 32) rows &= (1u << rows_valid) - 1;
    for (; rows != 0; rows &= rows - 1) visit(__builtin_ctz(rows));
}

// Lane l and lane l ^ 32 combine a value without going through LDS: v_permlane32_swap with both operands = x
// returns (x of the lower half, x of the upper half) in every lane (checked on the device with a probe).
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float max_with_other_half(float x)
{
    const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_with_other_half(float x)
{
    const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Combines over the four lanes l, l ^ 16, l ^ 32, l ^ 48.
__device__ __forceinline__ float max_over_quarters(float x)
{
    const u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return max_with_other_half(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}
__device__ __forceinline__ float sum_over_quarters(float x)
{
    const u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return sum_with_other_half(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}
// Combines over the lanes of one column of an M x M result.
template <int M>
__device__ __forceinline__ float max_over_groups(float x) { return M == 32 ? max_with_other_half(x) : max_over_quarters(x); }
template <int M>
__device__ __forceinline__ float sum_over_groups(float x) { return M == 32 ? sum_with_other_half(x) : sum_over_quarters(x); }

// Finds the tile a workgroup owns.  Tiles of `tile` rows are counted per segment over cu[0..n_seg], from the LAST tile of the
// LAST segment backwards (the later tiles of a segment see more keys, so the heaviest tiles get the lowest ranks and start
// first).  Segment g has ranks for the tiles from cu[g] / tile + g on: at least as many as it needs, so that its place follows
// from cu[g] alone and is searched for instead of summed up.  Every lane of every wavefront computes the same answer.
// Returns false for a rank that is no tile; ranks go up to cu[n_seg] / tile + n_seg (n_rows: cu[n_seg]).
// The lanes that look at the last 64 candidates load their bounds in BOTH lists (cu: the list the tiles are counted
// over, cu_other: the other one), and the winner's values are handed out by lane reads: the caller gets
// the segment's four bounds without a second, dependent round of loads.
struct TileLocation {
    int seg, tile_in_seg;
    int begin, len;               // of the segment in cu
    int other_begin, other_len;   // of the segment in cu_other
};
// ANEW: nothing of the lane is kept for it (kernels with no register to spare).
template <bool ANEW = false>
__device__ __forceinline__ bool locate_tile(const int32_t *cu, const int32_t *cu_other, int n_seg, int n_rows, int tile, int rank,
                                            TileLocation &out)
{
    if (n_seg == 1) {                                // one slice of one sequence: nothing to search
        out.seg = 0;
        out.begin = cu[0], out.len = cu[1] - cu[0];
        out.other_begin = cu_other[0], out.other_len = cu_other[1] - cu_other[0];
        const int n = (out.len + tile - 1) / tile;
        out.tile_in_seg = n - 1 - rank;
        return rank < n;
    }
    const int lane = ANEW ? fresh_lane() : threadIdx.x & 63;
    const int place = n_rows / tile + n_seg - 1 - rank;
    if (place < 0) return false;
    int lo = 0, hi = n_seg;                          // the segment is one of [lo, hi): 64 probes at a time
    while (hi - lo > 64) {
        const int step = (hi - lo + 63) / 64, g = lo + lane * step;
        const unsigned long long before = __ballot(g < hi && cu[min(g, hi - 1)] / tile + g <= place);
        lo += (63 - __clzll((long long)before)) * step;      // (lane 0 always says yes)
        hi = min(hi, lo + step);
    }
    const int g = min(lo + lane, hi - 1);
    const int b0 = cu[g], b1 = cu[g + 1], o0 = cu_other[g], o1 = cu_other[g + 1];
    const int last = 63 - __clzll((long long)__ballot(lo + lane < hi && b0 / tile + g <= place));
    auto of_last = [&](int x) { return ANEW ? __builtin_amdgcn_readlane(x, last) : __builtin_amdgcn_readfirstlane(__shfl(x, last)); };
    out.seg = __builtin_amdgcn_readfirstlane(lo + last);
    out.begin = of_last(b0);
    out.len = of_last(b1 - b0);
    out.other_begin = of_last(o0);
    out.other_len = of_last(o1 - o0);
    out.tile_in_seg = __builtin_amdgcn_readfirstlane(place - out.begin / tile - out.seg);
    return out.tile_in_seg * tile < out.len;
}

}  // namespace cf

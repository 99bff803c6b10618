// Device-side helpers shared by the bf16 MFMA kernels (gfx950).
//
// MFMA 32x32x16 bf16 operand layout (lane l of a 64-wide wavefront, half = l / 32):
//   A (M x K): lane holds row  m = l % 32, k = 8*half + 0..7        (bf16x8)
//   B (K x N): lane holds col  n = l % 32, k = 8*half + 0..7        (bf16x8)
//   C/D (M x N, fp32x16): lane holds col n = l % 32, register i <-> row (i/4)*8 + 4*half + i%4
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

// Two transposing reads, 8 rows apart... the caller passes both addresses; result is one bf16x8 operand.
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
__device__ __forceinline__ bf16x8 pack8(float a0, float a1, float a2, float a3, float a4, float a5, float a6,
                                        float a7)
{
    bf16x8 r;
    r[0] = (__bf16)a0; r[1] = (__bf16)a1; r[2] = (__bf16)a2; r[3] = (__bf16)a3;
    r[4] = (__bf16)a4; r[5] = (__bf16)a5; r[6] = (__bf16)a6; r[7] = (__bf16)a7;
    return r;
}

// Eight fp32 values as three bf16 operands: x = w[0] + w[1] + w[2] exactly (8 of the 24 significant bits each, taken off by
// truncation), so that three MFMAs multiply the fp32 value and not its rounding.
__device__ __forceinline__ void split_exact(const f32x16 &f, int first, bf16x8 (&w)[3])
{
    i32x4 u[3];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float x0 = f[first + 2 * e], x1 = f[first + 2 * e + 1];
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
// transposing 8-byte read (ds_read_b64_tr_b16) 32 lanes per clock.  swz() maps 16 consecutive rows to 16 different
// bank groups (row reads of one column by 16 rows are conflict free) AND gives the 4 consecutive rows of a transposing
// read 4 different groups of 4 units (those are conflict free too).  D = 128: a row covers the banks once, so that
// takes four bits of the row number; D = 64: two rows cover the banks, an even and an odd row never meet, and three
// bits above the lowest remain, the lowest of them in the place that moves by four units.
template <int D>
__device__ __forceinline__ int swz(int row)
{
    static_assert(D == 64 || D == 128, "row length");
    return D == 128 ? ((row & 3) << 2) | ((row >> 2) & 3) : (((row >> 1) & 1) << 2) | ((row >> 2) & 3);
}
template <int D>
__device__ __forceinline__ int tile_off(int row, int unit) { return row * (2 * D) + ((unit ^ swz<D>(row)) << 4); }

// Lane-constant LDS byte offsets into a swizzled tile, computed once per kernel (the XOR of the swizzle
// cannot be folded into an instruction's immediate offset, so every distinct unit needs its own register;
// keeping them in D / 8 registers beats recomputing them for each of the ~100 LDS reads per tile).
//
//  row_unit[ks]  operand rows read with ds_read_b128 (MFMA row/col = tile row, contraction along the tile
//                row): offset of (row = lane % 32, logical unit 2*ks + half).  A 32-row block further down
//                the tile adds 32 rows (swz() has period 16 rows).
//  tr_lo[db], tr_hi[db]
//                operands read with the transposing read (contraction along the tile's ROWS, MFMA
//                row/col = tile column 32*db + lane % 32): offsets of the two 4-row reads that make one
//                bf16x8 operand, for contraction rows 4*half + {0..3 by lane group} and 8 rows further.
//                32 (16) rows further down the tile add 32 (16) row lengths.
template <int D>
struct LaneOffsets {
    int row_unit[D / 16];
    int tr_lo[D / 32], tr_hi[D / 32];
};
template <int D>
__device__ __forceinline__ LaneOffsets<D> lane_offsets()
{
    const int lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31, r16 = lane & 15, blk = (lane >> 4) & 1;
    LaneOffsets<D> o;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) o.row_unit[ks] = tile_off<D>(col, 2 * ks + half);
    const int r_lo = 4 * half + (r16 >> 2), u0 = 2 * blk + ((r16 >> 1) & 1), sub = 8 * (r16 & 1);
#pragma unroll
    for (int db = 0; db < D / 32; ++db) {
        o.tr_lo[db] = tile_off<D>(r_lo, 4 * db + u0) + sub;
        o.tr_hi[db] = tile_off<D>(r_lo + 8, 4 * db + u0) + sub;
    }
    return o;
}

// The same offsets for a kernel that has no registers to spare: all follow from two bases by XOR (unit 2 ks + half of a
// row is unit `half` with bits 1.. flipped; 8 rows further flips bit 1 of the swizzle), one instruction per read.
// forget(): from here on the compiler computes them anew instead of keeping the results of the last use.
template <int D>
struct BlockAddress {
    int row0, tr0;
    __device__ __forceinline__ BlockAddress()
    {
        const LaneOffsets<D> lo = lane_offsets<D>();
        row0 = lo.row_unit[0], tr0 = lo.tr_lo[0];
    }
    // to the block `bytes` (a power of two beyond a block's size) further, and back
    __device__ __forceinline__ void flip(int bytes) { row0 ^= bytes, tr0 ^= bytes; }
    __device__ __forceinline__ void forget() { asm volatile("" : "+v"(row0), "+v"(tr0)); }
    __device__ __forceinline__ int row(int ks) const { return row0 ^ (ks << 5); }
    __device__ __forceinline__ int tr_lo(int db) const { return tr0 ^ (db << 6); }
    __device__ __forceinline__ int tr_hi(int db) const { return (tr0 ^ (db << 6) ^ (2 << 4)) + 8 * 2 * D; }
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
// base of a buffer descriptor (scalar arithmetic), the lane's place inside a tile is ONE register computed
// at init, and a part adds a scalar offset, so a full tile costs no vector address arithmetic at all.  Only
// a ragged tile (rows beyond last_row, relative to src, re-read last_row; the caller masks them) computes
// clamped per-lane offsets.  The descriptor's size field is left at its maximum: nothing relies on the
// hardware's out-of-range behaviour.
// Completion is tracked by vmcnt: wait_lds_dma() before the barrier that publishes the tile.
template <int ROWS, int D, int WAVES = 4>
struct TileDma {
    static constexpr int RPI = 512 / D, UNITS = D / 8;      // rows per instruction, 16-byte units per row
    static constexpr int PARTS = ROWS / (RPI * WAVES);
    static_assert(PARTS >= 1 && (RPI * WAVES) % 16 == 0, "a part must cover whole swizzle periods");
    unsigned row_bytes, unit16;   // unit16: byte offset of this lane's 16-byte unit inside its row (same for all parts)
    int r0;                       // this lane's row in part 0; part c adds RPI * WAVES rows
    int wv;                       // index of this wavefront among the copying ones
    unsigned lane_off;            // r0 * row_bytes + unit16: this lane's offset in part 0 of a full tile

    // wave: index of the calling wavefront among the WAVES that copy (wave-uniform)
    __device__ __forceinline__ void init(int64_t row_bytes_, int wave, int lane)
    {
        row_bytes = (unsigned)row_bytes_;
        wv = wave;
        r0 = RPI * wave + lane / UNITS;
        unit16 = ((lane % UNITS) ^ swz<D>(r0)) * 16; // swz() has period 16 rows
        lane_off = (unsigned)r0 * row_bytes + unit16;
    }
    __device__ __forceinline__ void init(int64_t row_bytes_) { init(row_bytes_, wave_id(), threadIdx.x & 63); }
    __device__ __forceinline__ CF_LDS void *part_dst(char *lds_tile, int c) const { return (CF_LDS void *)(lds_tile + (c * WAVES + wv) * 1024); }
    __device__ __forceinline__ static __amdgpu_buffer_rsrc_t descriptor(const char *src)
    {
        return __builtin_amdgcn_make_buffer_rsrc((void *)src, 0, -1, 0x00020000);
    }
    __device__ __forceinline__ void full_part(__amdgpu_buffer_rsrc_t rsrc, char *lds_tile, int c) const
    {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, part_dst(lds_tile, c), 16, (int)lane_off, (int)(RPI * WAVES * c * row_bytes), 0, 0);
    }
    __device__ __forceinline__ void ragged_part(__amdgpu_buffer_rsrc_t rsrc, int last_row, char *lds_tile, int c) const
    {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, part_dst(lds_tile, c), 16,
                                                 (int)((unsigned)min(r0 + RPI * WAVES * c, last_row) * row_bytes + unit16), 0, 0, 0);
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
            for (int c = 0; c < PARTS; ++c) ragged_part(rsrc, last_row, lds_tile, c);
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
// register: scalar float arithmetic does not exist here, and a readfirstlane of a uniform value is folded away).
__device__ __forceinline__ float scalar(float x)
{
    float r;
    asm("v_readfirstlane_b32 %0, %1" : "=s"(r) : "v"(x));
    return r;
}
__device__ __forceinline__ void wait_lds_dma() { __builtin_amdgcn_s_waitcnt(0x0F70); }   // vmcnt(0)

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

// Stores a wavefront's 32 x D block of bf16 results (computed transposed: a lane owns one ROW, register group
// (j, g4) of acc holds its 4 consecutive d starting at 32*j + 8*g4 + 4*half) to global rows of 2 D bytes.
// A direct store would write 8-byte pieces of 32 different rows per instruction (64 cache lines touched per
// instruction, 16 instructions); instead the block is turned around in `scratch` (this wavefront's own
// 32 padded rows of LDS, free at that point) and leaves as D / 16 instructions that each write 512 / D whole rows.
//   row_ptr(r): global address of row r of the block (r = 0..31), rows >= rows_valid are not written
template <int D>
struct RowScratch {
    static constexpr int stride = 2 * D + 16;       // keeps 16-byte alignment, spreads rows over banks
    static constexpr int bytes = 32 * stride;
};
template <int D, typename RowPtr>
__device__ __forceinline__ void store_rows_bf16(const f32x16 (&acc)[D / 32], float scale, char *scratch, int rows_valid,
                                                RowPtr row_ptr)
{
    constexpr int S = RowScratch<D>::stride, UNITS = D / 8, RPI = 512 / D;
    const int lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
#pragma unroll
    for (int j = 0; j < D / 32; ++j)
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
            bf16x4 w;
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = (__bf16)(acc[j][g4 * 4 + e] * scale);
            *(bf16x4 *)(scratch + col * S + (j * 32 + g4 * 8 + half * 4) * 2) = w;
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

// visit(r), by the whole wavefront, for every row r < rows_valid of a 32 x D block (a lane owns row lane % 32, as above) whose
// results, scaled, are not finite.
template <int D, typename Visit>
__device__ __forceinline__ void for_rows_not_finite(const f32x16 (&acc)[D / 32], float scale, int rows_valid, Visit visit)
{
    float zero = scale * 0.f;                        // stays 0 while everything is finite
#pragma unroll
    for (int j = 0; j < D / 32; ++j)
#pragma unroll
        for (int i = 0; i < 16; ++i) zero = __builtin_fmaf(acc[j][i], 0.f, zero);
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
    const int lane = threadIdx.x & 63;
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
    out.seg = __builtin_amdgcn_readfirstlane(lo + last);
    out.begin = __builtin_amdgcn_readfirstlane(__shfl(b0, last));
    out.len = __builtin_amdgcn_readfirstlane(__shfl(b1 - b0, last));
    out.other_begin = __builtin_amdgcn_readfirstlane(__shfl(o0, last));
    out.other_len = __builtin_amdgcn_readfirstlane(__shfl(o1 - o0, last));
    out.tile_in_seg = __builtin_amdgcn_readfirstlane(place - out.begin / tile - out.seg);
    return out.tile_in_seg * tile < out.len;
}

}  // namespace cf

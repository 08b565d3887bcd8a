// gfx950 kernels and the compute half of the C ABI.
//
// One wavefront (64 lanes) owns one task of the plan's task table.
//
//   SpMM task    rows of B gathered into LDS 32 at a time (one per vector of a dense block, one
//                per residual nonzero) x the 16 x 32 piece of A that belongs to them, decoded
//                from block bitmaps in registers (Section 4.4 of the paper) or built from the
//                residual nonzeros, on v_mfma_f32_16x16x32; B comes back in operand layout with
//                ds_read_b64_tr_b16.  The sums stay in the accumulators until the window's rows
//                are written: plain coalesced stores for rows this task owns, fp32 atomics for
//                rows with other writers.  A segment of a decomposed long row is the same task
//                with no blocks and one atomic output row.  fp32 storage: dense blocks on
//                v_mfma_f32_16x16x4, residual nonzeros on the VALU.
//   SDDMM window task  X window x gathered Y rows on v_mfma_f32_16x16x32_f16 (both operands are
//                contiguous along K; the rows of Y pass through LDS), sampled through output
//                records made at plan time.
//   SDDMM segment task 16 residual nonzeros per tile on the same instruction; fp32 storage:
//                per-nonzero dot products on the VALU with a cross-lane reduction.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <type_traits>
#include <vector>

#include "plan_internal.h"

using namespace libra;

typedef _Float16 half_t;
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf8_t __attribute__((ext_vector_type(8)));
struct bf16_t { uint16_t bits; };     // bfloat16 storage: the upper half of a binary32

namespace {

constexpr int WAVE = 64;
constexpr int W = 16;    // window height the kernels are written for
constexpr int KB = 16;   // block width the kernels are written for

// SDDMM window tasks take their dense blocks in groups of SD_GROUP; the 16-bit output records of a group are stored in
// ascending CSR position with the LDS stage slot of their product (see sddmm_window_task).
constexpr int SD_GROUP = 4;
__host__ __device__ inline int sd_stage_slot(int block_in_group, int row, int slot) {
    return block_in_group * 256 + (row % 4) * 64 + (row / 4) * 16 + slot;
}

struct SpmmArgs {
    const DevTask *tasks;
    const int32_t *blk_cols;
    const uint64_t *blk_bitmap;
    const int32_t *blk_valptr;
    const void *dense_val;
    const void *res_ent;
    const void *B;
    float *C;
    int64_t ldb, ldc;
    int32_t tasks_per_die;  // the table holds die k's tasks (dispatch positions k, k + 8, ...) contiguously from k * tasks_per_die on
    int32_t pieces;         // the launch covers `pieces` adjacent column pieces of N features each: every task runs once per piece
    int32_t phase;          // 0: a task does all its work; 1: dense blocks only; 2: residual nonzeros only, added to what phase 1 wrote
    void *R;                // kernels with rounded output: where a row with one writer goes, in the storage type (phase 0 only)
    int64_t ldr;
};

// Per storage type: a residual entry's value as it is stored and as a number.
template <class T> struct Elem;
template <> struct Elem<half_t> {
    typedef uint16_t val_t;
    __device__ static float word_val(uint32_t bits) {
        const uint16_t lo = (uint16_t)bits;
        half_t h;
        __builtin_memcpy(&h, &lo, 2);
        return (float)h;
    }
};
template <> struct Elem<bf16_t> {
    typedef uint16_t val_t;
    __device__ static float word_val(uint32_t bits) { return __uint_as_float(bits << 16); }
};
template <> struct Elem<float> {
    typedef float val_t;
    __device__ static float word_val(uint32_t bits) { return __uint_as_float(bits); }
};
// fp32 storage, vector ALU paths: a lane's 16 bytes of row `row` of an operand, and what is done with them
__device__ inline float4_t load_row4(const void *base, int32_t row, uint32_t ld_bytes, int sub) {
    return *reinterpret_cast<const float4_t *>(reinterpret_cast<const char *>(base) + ((uint64_t)(uint32_t)row * ld_bytes + (uint32_t)sub * 16u));
}
__device__ inline float dot4(const float4_t &x, const float4_t &y) {
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) s = fmaf(x[e], y[e], s);
    return s;
}

// NW 32-bit words from a 16-byte aligned LDS address: 16-byte reads issued back to back; every word then goes through an
// opaque move, so that it is read once and whole however its fields are used.
template <int NW>
__device__ inline void lds_words(const void *lds, uint32_t (&w)[NW]) {
    static_assert(NW % 4 == 0, "whole 16-byte reads");
#pragma unroll
    for (int k = 0; k < NW / 4; ++k) {
        const uint4 v = reinterpret_cast<const uint4 *>(lds)[k];
        w[4 * k] = v.x; w[4 * k + 1] = v.y; w[4 * k + 2] = v.z; w[4 * k + 3] = v.w;
    }
#pragma unroll
    for (int k = 0; k < NW; ++k) asm volatile("" : "+v"(w[k]));
}
// entry i of the blocked layout: its word and its value
template <class V>
__device__ inline void load_blocked_entry(const void *base, int64_t i, uint32_t &word, V &val) {
    const uint32_t u = (uint32_t)i;                        // entries are counted in 31 bits
    const char *blk = reinterpret_cast<const char *>(base) + (uint64_t)(u / RES_BLOCK) * (RES_BLOCK * (4u + (uint32_t)sizeof(V)));
    const uint32_t slot = u % RES_BLOCK;
    word = reinterpret_cast<const uint32_t *>(blk)[slot];
    val = reinterpret_cast<const V *>(blk + RES_BLOCK * 4)[slot];
}

__device__ inline void global_add(float *p, float v) {
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One 16x16x32 tile step on the matrix cores for either 16-bit storage type; operands are passed as raw bits.
template <class T>
__device__ inline float4_t mfma_k32(const uint4 &a, const uint4 &b, float4_t c) {
    if constexpr (std::is_same<T, half_t>::value) {
        half8_t ha, hb;
        __builtin_memcpy(&ha, &a, 16);
        __builtin_memcpy(&hb, &b, 16);
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(ha, hb, c, 0, 0, 0);
    } else {
        bf8_t ba, bb;
        __builtin_memcpy(&ba, &a, 16);
        __builtin_memcpy(&bb, &b, 16);
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(ba, bb, c, 0, 0, 0);
    }
}
// fp32 -> storage type of the softmax output (round to nearest even)
template <class TO> __device__ inline TO to_storage(float x) { return (TO)x; }
template <> __device__ inline bf16_t to_storage<bf16_t>(float x) {
    uint32_t u = __float_as_uint(x);
    if ((u & 0x7fffffffu) > 0x7f800000u) return bf16_t{(uint16_t)((u >> 16) | 0x40u)};      // NaN stays NaN
    u += 0x7fffu + ((u >> 16) & 1u);
    return bf16_t{(uint16_t)(u >> 16)};
}

template <class T>
__device__ inline uint4 round8(const float4_t &lo, const float4_t &hi) {
    uint32_t w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const T a = to_storage<T>(k < 2 ? lo[2 * k] : hi[2 * k - 4]), b = to_storage<T>(k < 2 ? lo[2 * k + 1] : hi[2 * k - 3]);
        uint16_t x, y;
        __builtin_memcpy(&x, &a, 2);
        __builtin_memcpy(&y, &b, 2);
        w[k] = (uint32_t)x | (uint32_t)y << 16;
    }
    return uint4{w[0], w[1], w[2], w[3]};
}

// Workgroup b of a launch runs on die b mod 8, so the records of the tasks that one die runs are stored next to each
// other: a 128-byte line of the table then serves four consecutive workgroups of one die instead of four dies.
constexpr unsigned DIE_SHIFT = 3;
static_assert(LIBRA_XCDS == 1 << DIE_SHIFT, "workgroup b takes record (b mod dies) * tasks_per_die + b / dies");

// ---------------------------------------------------------------------------------------
// SpMM.  N = feature columns handled by this launch, T = storage type of values and B.
//
// A task is latency-bound unless few dependent memory round trips carry many row fetches, so
// the kernel is organised around round trips: (1) the task record; (2) all the metadata of the
// task at once - residual entries, block column ids, block bitmaps; (3..) the
// B-row fetches in large batches whose addresses are at hand, never from another global load.
// ---------------------------------------------------------------------------------------

// Orders the LDS accesses of one wavefront (the hardware runs a wave's LDS instructions in order;
// this only stops the compiler from moving them across the point).
__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// LDS addresses that are handed around keep their address space (a generic pointer costs a test and a select at every use).
typedef __attribute__((address_space(3))) unsigned char lds_byte;
typedef __attribute__((address_space(3))) float lds_float;
typedef uint32_t word4_t __attribute__((ext_vector_type(4)));
__device__ inline uint4 lds_read16(const lds_byte *p) {
    const word4_t v = *reinterpret_cast<const __attribute__((address_space(3))) word4_t *>(p);
    return uint4{v[0], v[1], v[2], v[3]};
}
// 16 bytes per lane from global memory to LDS, past the registers: lane l's piece lands at lds + 16 l.
__device__ inline void load_to_lds(const void *src, lds_byte *lds) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src, (__attribute__((address_space(3))) void *)lds, 16, 0, 0);
}
__device__ inline void wait_for_loads() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    wave_sync();
}

// The stage's readers are done: fetches into it may be issued.
__device__ inline void wait_for_lds() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    wave_sync();
}

// SpMM, 16-bit storage.  Every row of B that a task needs - one per vector of its dense blocks, one per residual nonzero -
// goes through the same LDS stage and the same instruction: 32 staged rows are the k dimension of v_mfma_f32_16x16x32, the
// other operand is the 16 x 32 piece of A that belongs to them, built in registers from the block bitmaps (Section 4.4) or,
// for residual nonzeros, with one value per column.  The sums stay in the accumulators until the task's rows are written.
// A row's 16-byte pieces are fetched by consecutive lanes straight into LDS (no registers, no address per piece to keep), in
// batches of ROWS rows; piece p of row r is kept at place p ^ 2 unit(r), so that the transposing reads of two lane groups
// (eight rows, 32 bytes of each) touch all banks once.
// Bound by the way from the L2s to the L1s (the data return units are busy 78 % of the kernel on the power-law graph at N = 128, 97
// % on the GAT graph): the power-law graph draws 6.5 M lines of 128 bytes, 39 us at the 21 TB/s of a bare gather that always hits;
// a quarter of them miss.  The irregular graph is bound behind the L2s, by 94 M lines at 54 G lines per second.  Against fetching
// residual rows into registers and adding their products on the vector ALUs (65 - 76 % busy with it, now 27 - 35 %; 24.7 -> 9.8 M
// wave instructions, power-law N = 128): power-law N = 32 / 64 / 128 44.7 / 43.7 / 65.5 -> 31.0 / 39.3 / 64.0 us, GAT graph
// N = 64 596 -> 555, irregular N = 32 1,888 -> 1,845, community N = 128 277 -> 268.
// Two half-size stages in turn, 64 rows at N = 64 and seven or eight waves per SIMD at N <= 64 are each slower somewhere.
template <int N>
struct GatherStage {
    static constexpr int ROW = 2 * N;                        // bytes of a staged row
    static constexpr int PIECES = N / 8;                     // 16-byte pieces of a row = lanes that fetch it
    static constexpr int RPL = WAVE / PIECES;                // rows per wave load
    static constexpr int ROWS = N >= 64 ? 32 : 64;           // rows staged together
    static constexpr int LOADS = ROWS / RPL;
    static constexpr int BYTES = ROWS * ROW;
    static_assert(N == 32 || N == 64 || N == 128, "piece widths");
    __device__ static int unit(int row) {
        return N == 128 ? (row & 3) | (row >> 1 & 4) : N == 64 ? (row >> 1 & 1) | (row >> 2 & 2) : row >> 3 & 1;
    }
    // rows ids[first .. first + count) of `base` (one id per lane of the wave) to the stage; whole loads, so up to RPL - 1 more
    __device__ static void fetch(const char *base, uint32_t ld_bytes, int ids, int first, int count, lds_byte *stage) {
        const int lane = threadIdx.x;
        int id[LOADS];
#pragma unroll
        for (int i = 0; i < LOADS; ++i) id[i] = __builtin_amdgcn_ds_bpermute((first + i * RPL + lane / PIECES) * 4, ids);
#pragma unroll
        for (int i = 0; i < LOADS; ++i) asm volatile("" : "+v"(id[i]));          // all ids before the first fetch
        auto load = [&](int i) {
            const int piece = (lane % PIECES) ^ unit(i * RPL + lane / PIECES) << 1;
            load_to_lds(base + ((uint64_t)(uint32_t)id[i] * ld_bytes + (uint32_t)piece * 16u), stage + i * RPL * ROW);
        };
        if (count > ROWS - RPL) {            // a whole batch, without a branch per load
#pragma unroll
            for (int i = 0; i < LOADS; ++i) load(i);
        } else {
#pragma unroll
            for (int i = 0; i < LOADS; ++i)
                if (i * RPL < count) load(i);
        }
    }
    // rows past the first `count` of an empty stage: the products take them times zero, so they have to be numbers
    __device__ static void clear_rest(int count, lds_byte *stage) {
        if (count > ROWS - RPL) return;
#pragma unroll
        for (int i = 0; i < LOADS; ++i)
            if (i * RPL >= count) *reinterpret_cast<__attribute__((address_space(3))) word4_t *>(stage + i * RPL * ROW + threadIdx.x * 16) = word4_t{0u, 0u, 0u, 0u};
    }
    // B operand of columns 16 n .. 16 n + 15 and staged rows at .. at + 31: lane (g, j) gets column j of rows at + 8 g .. + 7.
    // Lane i of a 16-lane group points at row i / 4, halves 4 (i % 4) .. + 3 of the 32-byte piece; the transposing read hands
    // lane j the four rows' element j.
    __device__ static uint4 operand(const lds_byte *stage, int at, int n, int g, int j) {
        const int row = 8 * g + (j >> 2);
        const lds_byte *p = stage + at * ROW + (row * ROW + ((n ^ unit(row)) * 32 + 8 * (j & 3)));
        typedef short4_t __attribute__((address_space(3))) *lds_t;
        const short4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t)p), hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t)(p + 4 * ROW));
        uint4 r;
        __builtin_memcpy(&r.x, &lo, 8);
        __builtin_memcpy(&r.z, &hi, 8);
        return r;
    }
};

// An Inf or NaN among staged rows must not meet the empty places of the A piece (0 * Inf = NaN).  What it gives where A does
// have a nonzero is counted on the matrix cores instead: per product +Inf counts 1, -Inf 64 and NaN at least 4160, which is
// the sum of two products of small numbers,
//   positive value: (1, 0), negative: (0, 1), stored zero: (64, 64), no value: (0, 0)
//   +Inf: (1, 64), -Inf: (64, 1), NaN: (8192, 8192), a number: (0, 0);
// 32 products without a NaN give at most 32 * 64, exact in binary32.  The sums themselves take +-1 in place of the Inf or NaN:
// nothing comes from empty places, and an infinite value of A keeps the sign of its product.
template <class T>
struct NonFinite {
    static constexpr bool F16 = std::is_same<T, half_t>::value;
    static constexpr uint32_t INF = F16 ? 0x7c00u : 0x7f80u;
    // 1, 64 and 8192 in both halves of a word; two 16-bit numbers are handled at once
    static constexpr uint32_t ONE = F16 ? 0x3c003c00u : 0x3f803f80u, P64 = F16 ? 0x54005400u : 0x42804280u, P8192 = F16 ? 0x70007000u : 0x46004600u;
    static constexpr float NANS = 64.f * 65.f;
    // per half: all ones if the sign bit is set; if the number without its sign is at least `least` (as bits)
    __device__ static uint32_t spread(uint32_t x) {
        typedef short short2_t __attribute__((ext_vector_type(2)));
        return __builtin_bit_cast(uint32_t, __builtin_bit_cast(short2_t, x) >> (short2_t)(short)15);
    }
    __device__ static uint32_t above(uint32_t w, uint32_t least) { return spread((w & 0x7fff7fffu) + (0x8000u - least) * 0x00010001u); }
    struct Pair {                                   // of B
        uint32_t w, infinite, nan, negative;
        __device__ explicit Pair(uint32_t x) : w(x), infinite(above(x, INF)), nan(above(x, INF + 1u)), negative(spread(x)) { infinite &= ~nan; }
        __device__ uint32_t finite() const { return (w & ~(infinite | nan)) | ((infinite | nan) & ((w & 0x80008000u) | ONE)); }
        // what it counts for values of a sign
        __device__ uint32_t for_positive() const { return (infinite & ((~negative & ONE) | (negative & P64))) | (nan & P8192); }
        __device__ uint32_t for_negative() const { return (infinite & ((negative & ONE) | (~negative & P64))) | (nan & P8192); }
    };
    // of A: what positive values count (`present`: the places that hold a value), and negative ones from that
    __device__ static uint32_t weight(uint32_t w, uint32_t present) {
        const uint32_t number = above(w, 1u);
        return present & ((number & ~spread(w) & ONE) | (~number & P64));
    }
    __device__ static uint32_t other_sign(uint32_t weight, uint32_t w) { return weight ^ (above(w, 1u) & ONE); }
    __device__ static float fold(float sum, float counts) {
        const int c = (int)fminf(counts, NANS);
        if (c & 63) sum += __builtin_huge_valf();
        if (c >> 6) sum -= __builtin_huge_valf();
        return counts >= NANS ? __builtin_nanf("") : sum;
    }
};

// The sums of a task that met an Inf or NaN, once more: 32 rows at a time as in the kernel, one batch after the other.  Bound by
// the chain of each 16 columns (LDS, some 100 vector instructions, three products), which go one after the other so that the
// kernel needs no more registers than without this.  All of B Inf, default options: power-law N = 128 310 us (finite 65), community
// N = 128 578 (263); one Inf, in the most referenced row: 135 and 267.  One nonzero at a time on the vector ALUs: 525, 2,060, 461
// and 322.
template <class T, int N>
__device__ inline void spmm_careful_sums(const SpmmArgs &a, const DevTask &t, int nblk, int L, const char *Bp, uint32_t ldb_bytes, lds_byte *stage,
                                         uint16_t *row_lds, uint16_t *val_lds, float4_t (&acc)[N / 16]) {
    using S = GatherStage<N>;
    typedef NonFinite<T> F;
    typedef typename F::Pair Pair;
    const int lane = threadIdx.x, g = lane >> 4, j = lane & 15;
#pragma unroll
    for (int n = 0; n < N / 16; ++n) acc[n] = float4_t{0.f, 0.f, 0.f, 0.f};
    const uint16_t *vals = reinterpret_cast<const uint16_t *>(a.dense_val);
    const int pairs = piece_count(nblk, 2), batches = pairs + piece_count(L, 32);          // dense blocks, then residual nonzeros
    for (int i = 0; i < batches; ++i) {
        uint32_t v[4], present[4];                          // this lane's A elements, and all ones where there is one
        if (i < pairs) {
            const int col = a.blk_cols[(int64_t)(t.blk_begin + min(2 * i + (g & 1), nblk - 1)) * KB + j];
            const int head = __builtin_amdgcn_ds_bpermute((lane & 48) * 4, col);
            S::fetch(Bp, ldb_bytes, col >= 0 ? col : head, 0, 2 * KB, stage);
            const int b = t.blk_begin + min(2 * i + (g >> 1), nblk - 1);
            int at = a.blk_valptr[b];
            const int q = j >> 2, shift = (j & 3) * 16 + 8 * (g & 1);
            for (int k = 0; k < q; ++k) at += __popcll(a.blk_bitmap[(int64_t)b * 4 + k]);
            const uint64_t w = a.blk_bitmap[(int64_t)b * 4 + q];
            at += __popcll(w & ((1ull << shift) - 1ull));
            const uint32_t set = 2 * i + (g >> 1) < nblk ? (uint32_t)(w >> shift) & 0xffu : 0u;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                v[k] = present[k] = 0;
#pragma unroll
                for (int e = 2 * k; e < 2 * k + 2; ++e)
                    if (set >> e & 1u) {
                        v[k] |= (uint32_t)vals[at++] << (e & 1) * 16;
                        present[k] |= 0xffffu << (e & 1) * 16;
                    }
            }
        } else {
            const int e0 = (i - pairs) * 32, n = min(32, L - e0);
            uint32_t word;
            uint16_t val;
            load_blocked_entry(a.res_ent, (int64_t)(t.res_begin + e0 + min(lane, n - 1)), word, val);
            S::fetch(Bp, ldb_bytes, (int)(word & RES_COL_MASK), 0, 32, stage);
            row_lds[lane] = lane < n ? (uint16_t)(word >> RES_ROW_SHIFT) : (uint16_t)W;
            val_lds[lane] = val;
            wave_sync();
            const uint4 rw = lds_read16((lds_byte *)row_lds + 16 * g), vw = lds_read16((lds_byte *)val_lds + 16 * g);
            const uint32_t r[4] = {rw.x, rw.y, rw.z, rw.w}, x[4] = {vw.x, vw.y, vw.z, vw.w};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                present[k] = ~F::above(r[k] ^ (uint32_t)j * 0x00010001u, 1u);
                v[k] = x[k] & present[k];
            }
        }
        uint32_t weight[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) weight[k] = F::weight(v[k], present[k]);
        wait_for_loads();
#pragma unroll
        for (int n = 0; n < N / 16; ++n) {
            __builtin_amdgcn_sched_barrier(0);              // one after the other, so that the kernel needs no more registers for this
            int l = lane;
            asm volatile("" : "+v"(l));                   // the addresses are formed again, not kept
            const uint4 op = S::operand(stage, 0, n, l >> 4, l & 15);
            uint32_t b[4] = {op.x, op.y, op.z, op.w}, x[4], any = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const Pair p(b[k]);
                x[k] = p.finite();
                any |= p.infinite | p.nan;
                asm volatile("" : "+v"(b[k]));              // nor are these
            }
            acc[n] = mfma_k32<T>(uint4{v[0], v[1], v[2], v[3]}, uint4{x[0], x[1], x[2], x[3]}, acc[n]);
            if (__any(any != 0)) {
                float4_t counts = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 0; k < 4; ++k) x[k] = Pair(b[k]).for_positive();
                counts = mfma_k32<T>(uint4{weight[0], weight[1], weight[2], weight[3]}, uint4{x[0], x[1], x[2], x[3]}, counts);
                uint32_t w[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    w[k] = F::other_sign(weight[k], v[k]);
                    x[k] = Pair(b[k]).for_negative();
                }
                counts = mfma_k32<T>(uint4{w[0], w[1], w[2], w[3]}, uint4{x[0], x[1], x[2], x[3]}, counts);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[n][e] = F::fold(acc[n][e], counts[e]);
            }
        }
        wait_for_lds();
    }
}

// ROUNDED: a row with one writer leaves in the storage type, rounded once from its fp32 sums, instead of as an fp32 row of C that
// another pass reads and rounds (a write of 4, a read of 4 and a write of 2 bytes per element become the last one).  A training
// step with attention on a power-law graph of 500,009 rows, bf16, N = K = 64, three such products: 1,697 -> 1,573 us; with fixed
// weights on an irregular graph of 300,007 rows, fp16, N = 128, one: 940 -> 897 us.
template <class T, int N, bool ROUNDED>
__global__ __launch_bounds__(WAVE) __attribute__((amdgpu_waves_per_eu(N >= 128 ? 5 : 6))) void spmm_gather_kernel(SpmmArgs a) {
    using S = GatherStage<N>;
    constexpr int NT = N / 16;
    constexpr int PAIRS = S::ROWS / (2 * KB);                // pairs of blocks per batch
    constexpr int TILE_BYTES = W * N * 4;
    constexpr int SMEM = TILE_BYTES > S::BYTES ? TILE_BYTES : S::BYTES;
    __shared__ __attribute__((aligned(16))) unsigned char smem[SMEM];        // the stage, afterwards the C tile
    __shared__ __attribute__((aligned(16))) uint16_t row_lds[WAVE], val_lds[WAVE];       // residual nonzeros: row in window, value bits
    lds_byte *stage = (lds_byte *)smem;

    // workgroup b: die b mod 8, then the pieces of one task next to each other (they read the same plan data through
    // the same L2), then the die's next task
    unsigned round = blockIdx.x >> DIE_SHIFT, piece = 0;
    if (a.pieces > 1) {
        piece = round % (unsigned)a.pieces;
        round /= (unsigned)a.pieces;
    }
    DevTask t = a.tasks[(int64_t)(blockIdx.x & (LIBRA_XCDS - 1)) * a.tasks_per_die + round];
    asm volatile("" : "+s"(t.id), "+s"(t.blk_begin), "+s"(t.blk_end), "+s"(t.res_begin), "+s"(t.res_end), "+s"(t.masks));      // one load
    const char *Bp = reinterpret_cast<const char *>(a.B) + (size_t)piece * S::ROW;
    float *Cp = a.C + (size_t)piece * N;
    const int lane = threadIdx.x, g = lane >> 4, j = lane & 15;
    const uint32_t atomic_mask = t.masks & 0xffffu, store_mask = t.masks >> 16;
    // The two-kernel mode (the paper's sequential schedule of Section 4.4.1: matrix-unit part, then scalar part) runs
    // the table twice.  Phase 1 takes the tasks that have blocks and writes all their rows; phase 2 takes the tasks that
    // have residual nonzeros or own rows that phase 1 did not write, and adds to rows that phase 1 wrote.
    const int nblk_all = t.blk_end - t.blk_begin;
    if (a.phase == 1 && nblk_all == 0) return;
    const int nblk = a.phase == 2 ? 0 : nblk_all;
    const int L = a.phase == 1 ? 0 : t.res_end - t.res_begin;
    if (a.phase == 2 && nblk_all > 0 && L == 0) return;
    const bool add_to_c = a.phase == 2 && nblk_all > 0;
    const uint32_t ldb_bytes = (uint32_t)a.ldb * 2u;

    // ---- the task's first metadata of each kind in one round trip, from clamped (always valid) addresses ----
    uint32_t word;
    uint16_t val;
    auto load_entries = [&](int e0) { load_blocked_entry(a.res_ent, (int64_t)(t.res_begin + max(min(e0 + lane, L - 1), 0)), word, val); };
    int col;                            // lane l: column of slot l of the batch
    uint64_t bits[PAIRS][4];            // bitmap of the block this lane's A elements come from, and its first packed value
    uint32_t vptr[PAIRS];
    auto load_blocks = [&](int b0) {
        const int last = max(nblk - 1, 0);
        col = a.blk_cols[(int64_t)(t.blk_begin + min(b0 + g, last)) * KB + j];
#pragma unroll
        for (int p = 0; p < PAIRS; ++p) {
            const int64_t b = t.blk_begin + min(b0 + 2 * p + (g >> 1), last);
            const uint64_t *bm = a.blk_bitmap + b * 4;
#pragma unroll
            for (int k = 0; k < 4; ++k) bits[p][k] = bm[k];
            vptr[p] = (uint32_t)a.blk_valptr[b];
        }
    };
    load_entries(0);
    if (nblk > 0) load_blocks(0);

    S::clear_rest(nblk > 0 ? nblk * KB : L, stage);
    float4_t acc[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[n] = float4_t{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](const uint4 &af, int at) {
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[n] = mfma_k32<T>(af, S::operand(stage, at, n, g, j), acc[n]);
    };

    // ---- dense blocks ----
    for (int b0 = 0; b0 < nblk; b0 += 2 * PAIRS) {
        // a padding slot fetches the row of its block's first slot (always a real one)
        const int head = __builtin_amdgcn_ds_bpermute((lane & 48) * 4, col);
        S::fetch(Bp, ldb_bytes, col >= 0 ? col : head, 0, (nblk - b0) * KB, stage);
        // this lane's A elements: row j, slots 8 (g & 1) .. + 7 of block g / 2 of each pair.  Their values are loaded
        // unconditionally (an unset slot reads a neighbouring value, at most 7 past the array's end, inside its 16 spare
        // bytes) and selected when they have arrived.
        uint32_t av[PAIRS][8], set[PAIRS];
#pragma unroll
        for (int p = 0; p < PAIRS; ++p) {
            const int q = j >> 2, shift = (j & 3) * 16 + 8 * (g & 1);
            const uint64_t w = q == 0 ? bits[p][0] : q == 1 ? bits[p][1] : q == 2 ? bits[p][2] : bits[p][3];
            const int c0 = __popcll(bits[p][0]), c1 = __popcll(bits[p][1]), c2 = __popcll(bits[p][2]);
            const int before = (q > 0 ? c0 : 0) + (q > 1 ? c1 : 0) + (q > 2 ? c2 : 0) + __popcll(w & ((1ull << shift) - 1ull));
            set[p] = b0 + 2 * p + (g >> 1) < nblk ? (uint32_t)(w >> shift) & 0xffu : 0u;
            uint32_t at = (vptr[p] + (uint32_t)before) * 2u;             // bytes: fewer than 2^32 for 31-bit counts
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                av[p][e] = *reinterpret_cast<const uint16_t *>(reinterpret_cast<const char *>(a.dense_val) + at);
                at += (set[p] >> e & 1u) * 2u;
            }
        }
        if (b0 + 2 * PAIRS < nblk) load_blocks(b0 + 2 * PAIRS);
        wait_for_loads();
#pragma unroll
        for (int p = 0; p < PAIRS; ++p) {
#pragma unroll
            for (int e = 0; e < 8; ++e) av[p][e] = set[p] >> e & 1u ? av[p][e] : 0u;
            const uint4 af{av[p][0] | av[p][1] << 16, av[p][2] | av[p][3] << 16, av[p][4] | av[p][5] << 16, av[p][6] | av[p][7] << 16};
            if (b0 + 2 * p < nblk) multiply(af, 2 * KB * p);
        }
        wait_for_lds();                  // the stage may be overwritten
    }

    // ---- residual nonzeros ----
    for (int e0 = 0; e0 < L; e0 += WAVE) {
        const int nE = min(WAVE, L - e0);
        row_lds[lane] = (uint16_t)(word >> RES_ROW_SHIFT);
        val_lds[lane] = lane < nE ? val : (uint16_t)0;
        const int ids = (int)(word & RES_COL_MASK);
#pragma unroll
        for (int h = 0; h < WAVE; h += S::ROWS) {
            if (h < nE) {
                S::fetch(Bp, ldb_bytes, ids, h, nE - h, stage);
                if (h == 0 && e0 + WAVE < L) load_entries(e0 + WAVE);        // they travel with the rows
                wait_for_loads();
#pragma unroll
                for (int k0 = 0; k0 < S::ROWS; k0 += 32) {
                    if (h + k0 < nE) {
                        // A elements: nonzero 8 g + e of these 32 in its own row, nothing in the others, two per word: the value
                        // times (1 - |row - j|, not below zero)
                        typedef unsigned short ushort8_t __attribute__((ext_vector_type(8)));
                        const uint4 rw = lds_read16((lds_byte *)row_lds + 2 * (h + k0 + 8 * g)), vw = lds_read16((lds_byte *)val_lds + 2 * (h + k0 + 8 * g));
                        ushort8_t r, v;
                        __builtin_memcpy(&r, &rw, 16);
                        __builtin_memcpy(&v, &vw, 16);
                        const ushort8_t one = (unsigned short)1;
                        r = __builtin_elementwise_sub_sat(one, r ^ (unsigned short)j) * v;
                        uint4 af;
                        __builtin_memcpy(&af, &r, 16);
                        multiply(af, k0);
                    }
                }
                wait_for_lds();
            }
        }
    }

    lds_float *tile = reinterpret_cast<lds_float *>(stage);
    float *cbase = Cp + (int64_t)t.id * W * a.ldc;
    // An Inf or NaN among the staged rows is in every row of the accumulators (0 * Inf = NaN): such a task (and one whose sums
    // overflow) forms its sums again.
    float probe = 0.f;
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int e = 0; e < 4; ++e) probe = fmaf(acc[n][e], 0.f, probe);
    if (__builtin_expect(__any(probe != probe), 0)) spmm_careful_sums<T, N>(a, t, nblk, L, Bp, ldb_bytes, stage, row_lds, val_lds, acc);

    // ---- the tile: accumulators to LDS (lane (g, j) holds rows 4g..4g+3, feature 16n + j), rows written once ----
    if (store_mask == 0 && (atomic_mask & (atomic_mask - 1u)) == 0) {
        // one row, other writers beside this task (a segment of a decomposed row)
        const int r = __builtin_ctz(atomic_mask | 1u << W);
        if (r < W) {
            if (g == r >> 2) {
#pragma unroll
                for (int n = 0; n < NT; ++n) {
                    const float lo = r & 1 ? acc[n][1] : acc[n][0], hi = r & 1 ? acc[n][3] : acc[n][2];
                    tile[16 * n + j] = r & 2 ? hi : lo;
                }
            }
            wave_sync();
            float *dst = cbase + (int64_t)r * a.ldc;
#pragma unroll
            for (int c = 0; c < N; c += WAVE)
                if (N >= WAVE || lane < N) global_add(dst + c + lane, tile[c + lane]);
        }
        return;
    }
    auto at = [](int row, int c) { return row * N + (c ^ (row >> 2 & (NT - 1)) * 16); };        // four rows' 64-byte pieces in different banks
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int n = 0; n < NT; ++n) tile[at(4 * g + e, 16 * n + j)] = acc[n][e];
    wave_sync();
    constexpr int LPF = N / 4;                                   // lanes per tile row at 4 floats each
    constexpr int RPP = WAVE / LPF;                              // tile rows per wave pass
    const int rr = lane / LPF, cl = lane % LPF;
    float *dst = cbase + (int64_t)rr * a.ldc + cl * 4;
    const int64_t step = RPP * a.ldc;
    if constexpr (ROUNDED) {
        // eight values of a row per lane; rows with other writers are added to C below and rounded when they are whole
        constexpr int LPR = N / 8, RPR = WAVE / LPR;
        const int r0 = lane / LPR, c = lane % LPR * 8;
        T *rdst = reinterpret_cast<T *>(a.R) + (int64_t)piece * N + ((int64_t)t.id * W + r0) * a.ldr + c;
#pragma unroll
        for (int k = 0; k < W / RPR; ++k, rdst += RPR * a.ldr) {
            if (!(store_mask >> (k * RPR + r0) & 1u)) continue;
            const lds_float *src = &tile[at(k * RPR + r0, c)];
            const float4_t lo = *reinterpret_cast<const __attribute__((address_space(3))) float4_t *>(src);
            const float4_t hi = *reinterpret_cast<const __attribute__((address_space(3))) float4_t *>(src + 4);
            *reinterpret_cast<uint4 *>(rdst) = round8<T>(lo, hi);
        }
        if (atomic_mask == 0) return;
    }
    if (!ROUNDED && atomic_mask == 0 && !add_to_c) {
        // streaming stores: C is written once and not read again by this call
        float4_t x[W / RPP];
#pragma unroll
        for (int k = 0; k < W / RPP; ++k) x[k] = *reinterpret_cast<const __attribute__((address_space(3))) float4_t *>(&tile[at(k * RPP + rr, cl * 4)]);
#pragma unroll
        for (int k = 0; k < W / RPP; ++k) {
            if (store_mask >> (k * RPP + rr) & 1u) __builtin_nontemporal_store(x[k], reinterpret_cast<float4_t *>(dst));
            dst += step;
        }
        return;
    }
#pragma unroll
    for (int k = 0; k < W / RPP; ++k, dst += step) {
        const int r = k * RPP + rr;
        if (!ROUNDED && (store_mask >> r & 1u)) {
            float4_t x = *reinterpret_cast<const __attribute__((address_space(3))) float4_t *>(&tile[at(r, cl * 4)]);
            if (add_to_c) {           // stream order: phase 1 has written the row
                const float4_t y = *reinterpret_cast<const float4_t *>(dst);
                x[0] += y[0]; x[1] += y[1]; x[2] += y[2]; x[3] += y[3];
            }
            __builtin_nontemporal_store(x, reinterpret_cast<float4_t *>(dst));
        } else if (atomic_mask >> r & 1u) {
            // each atomic instruction covers LPF consecutive floats of the row
#pragma unroll
            for (int e = 0; e < 4; ++e) global_add(dst - cl * 4 + e * LPF + cl, tile[at(r, e * LPF + cl)]);
        }
    }
}

// SpMM, fp32 storage: a product on the matrix cores costs a full-rate FMA there (v_mfma_f32_16x16x4), so only the dense
// blocks run on them and the residual nonzeros run on the vector ALUs.  The dense phase takes one block per round trip: the
// 16 rows of B go through an LDS stage that shares its bytes with the C tile, a lane's four A elements are the four k-steps
// of the product.  The accumulators are parked in the tile, and the residual nonzeros of the task, cut into equal contiguous
// runs per lane group, are added to it.
// Register budget: a 128-column task is held to four waves per SIMD by its LDS anyway; narrower ones gain from six, which
// four fetches in flight per group allow.
template <int N>
__global__ __launch_bounds__(WAVE) __attribute__((amdgpu_waves_per_eu(N >= 128 ? 4 : 6))) void spmm_task_kernel_f32(SpmmArgs a) {
    constexpr int PL = 4;                    // elements of a row per lane (16 bytes)
    constexpr int LPR = N / PL;              // lanes per row
    constexpr int RPW = WAVE / LPR;          // lane groups per wave
    static_assert(LPR >= 1 && LPR <= WAVE && WAVE % LPR == 0, "unsupported N");
    constexpr int LDC = N + 4;               // tile row stride (floats)
    constexpr int LDBS = N + 16;             // stage row stride: 2 consecutive rows cover all 32 banks
    constexpr int TILE_BYTES = W * LDC * 4;
    constexpr int STAGE_BYTES = KB * LDBS * 4;
    constexpr int SMEM = TILE_BYTES > STAGE_BYTES ? TILE_BYTES : STAGE_BYTES;
    constexpr int ECAP = 128;                // residual entries staged per round
    constexpr int BCAP = 8;                  // dense blocks whose metadata is staged per round
    constexpr int U = N >= 128 ? 8 : 4;      // B-row fetches in flight per lane group (narrow rows: fewer, for more waves)
    // the B stage (dense phase) and the C tile (afterwards) share the same LDS bytes
    __shared__ __attribute__((aligned(16))) unsigned char smem[SMEM];
    __shared__ __attribute__((aligned(16))) uint32_t ent_lds[ECAP];          // the staged entries' words (column | row in window) ...
    __shared__ __attribute__((aligned(16))) float val_lds[ECAP];             // ... and values
    __shared__ __attribute__((aligned(16))) int32_t cols_lds[BCAP * KB];
    __shared__ __attribute__((aligned(16))) uint64_t bm_lds[WAVE];           // BCAP * 4 words used
    float *tile = reinterpret_cast<float *>(smem);

    // workgroup b: die b mod 8, then the pieces of one task next to each other (they read the same plan data through
    // the same L2), then the die's next task
    const unsigned round = blockIdx.x >> DIE_SHIFT, piece = round % (unsigned)a.pieces;
    const DevTask t = a.tasks[(int64_t)(blockIdx.x & (LIBRA_XCDS - 1)) * a.tasks_per_die + round / (unsigned)a.pieces];
    const char *Bp = reinterpret_cast<const char *>(a.B) + (size_t)piece * N * 4;
    float *Cp = a.C + (size_t)piece * N;
    const int lane = threadIdx.x;
    const int sub = lane % LPR;              // which PL-wide piece of a row
    const int grp = lane / LPR;              // which lane group
    const uint32_t atomic_mask = t.masks & 0xffffu, store_mask = t.masks >> 16;
    const uint32_t out_mask = atomic_mask | store_mask;
    // two-kernel mode: see spmm_gather_kernel
    const int nblk_all = t.blk_end - t.blk_begin;
    if (a.phase == 1 && nblk_all == 0) return;
    const int nblk = a.phase == 2 ? 0 : nblk_all;
    const int L = a.phase == 1 ? 0 : t.res_end - t.res_begin;
    if (a.phase == 2 && nblk_all > 0 && L == 0) return;
    const bool add_to_c = a.phase == 2 && nblk_all > 0;
    const uint32_t ldb_bytes = (uint32_t)a.ldb * 4u;

    // ---- round trip 2: all metadata of the task (first round of each kind) ----
    // Loads are issued unconditionally from clamped (always valid) addresses and unused results are
    // masked afterwards: a load inside a branch makes the compiler wait for all earlier loads first.
    // First round of each kind of metadata, all loads in flight together, then the LDS writes.
    {
        const int nE = min(L, ECAP), nb = min(nblk, BCAP);
        uint32_t tmp[ECAP / WAVE];
        float tmp_val[ECAP / WAVE];
#pragma unroll
        for (int k = 0; k < ECAP / WAVE; ++k)
            load_blocked_entry(a.res_ent, (int64_t)t.res_begin + max(min(k * WAVE + lane, nE - 1), 0), tmp[k], tmp_val[k]);
        const int32_t *csrc = a.blk_cols + (int64_t)t.blk_begin * KB;
        int32_t c[BCAP * KB / WAVE];
#pragma unroll
        for (int k = 0; k < BCAP * KB / WAVE; ++k) c[k] = csrc[max(min(k * WAVE + lane, nb * KB - 1), 0)];
        const uint64_t w = a.blk_bitmap[(int64_t)t.blk_begin * 4 + max(min(lane, nb * 4 - 1), 0)];
#pragma unroll
        for (int k = 0; k < BCAP * KB / WAVE; ++k) cols_lds[k * WAVE + lane] = c[k];
        bm_lds[lane] = w;            // all 64 lanes write (the upper ones a copy of the last word): under a `lane < 32` branch
                                     // the compiler moves the load there too and issues it only after the loads before it returned
#pragma unroll
        for (int k = 0; k < ECAP / WAVE; ++k) {
            ent_lds[k * WAVE + lane] = tmp[k];
            val_lds[k * WAVE + lane] = tmp_val[k];
        }
    }
    // later rounds of a task with more than BCAP blocks are fetched in place
    auto fetch_blocks = [&](int b0, int nb) {
        const int32_t *csrc = a.blk_cols + (int64_t)(t.blk_begin + b0) * KB;
        int32_t c[BCAP * KB / WAVE];
#pragma unroll
        for (int k = 0; k < BCAP * KB / WAVE; ++k) c[k] = csrc[min(k * WAVE + lane, nb * KB - 1)];
        const uint64_t w = a.blk_bitmap[(int64_t)(t.blk_begin + b0) * 4 + min(lane, nb * 4 - 1)];
#pragma unroll
        for (int k = 0; k < BCAP * KB / WAVE; ++k) cols_lds[k * WAVE + lane] = c[k];
        bm_lds[lane] = w;
    };
    wave_sync();

    bool tile_ready = false;
    if (nblk > 0) {
        tile_ready = true;
        constexpr int NT = N / 16;
        constexpr int PASSES = KB / RPW > 0 ? KB / RPW : 1;  // wave loads per block
        static_assert(KB % RPW == 0, "stage shape");
        float *stage = reinterpret_cast<float *>(smem);
        const int g = lane >> 4, j = lane & 15;
        float4_t acc[NT];
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[n] = float4_t{0.f, 0.f, 0.f, 0.f};
        int vbase = t.val_begin;                             // first packed value of the current block
        for (int b0 = 0; b0 < nblk; b0 += BCAP) {
            const int nbr = min(BCAP, nblk - b0);
            if (b0 > 0) {
                wave_sync();
                fetch_blocks(b0, nbr);
                wave_sync();
            }
            for (int bb = 0; bb < nbr; ++bb) {
                // one round trip: the B rows of a block (padding slots become zero rows) ...
                float4_t raw[PASSES];
                int cc[PASSES];
#pragma unroll
                for (int ps = 0; ps < PASSES; ++ps) cc[ps] = cols_lds[bb * KB + ps * RPW + grp];
#pragma unroll
                for (int ps = 0; ps < PASSES; ++ps) {
                    // a padding slot fetches row 0 and is cleared by a mask the compiler cannot see through
                    // (so that it keeps the fetch outside any branch)
                    uint32_t keep = cc[ps] >= 0 ? 0xffffffffu : 0u;
                    asm volatile("" : "+v"(keep));
                    raw[ps] = load_row4(Bp, keep ? cc[ps] : 0, ldb_bytes, sub);
#pragma unroll
                    for (int e = 0; e < 4; ++e) raw[ps][e] = __uint_as_float(__float_as_uint(raw[ps][e]) & keep);
                }
                // ... and this lane's 4 A elements (row j, slots 4g..4g+3), decoded from the bitmap: unconditional loads (an
                // unset slot reads a neighbouring value, at most 3 values past the array's end, inside its 16 spare bytes),
                // and the selects afterwards
                float4_t af;
                {
                    const uint64_t *bm = &bm_lds[bb * 4];
                    const uint64_t w0 = bm[0], w1 = bm[1], w2 = bm[2], w3 = bm[3];
                    const int q = j >> 2;
                    const uint64_t word = q == 0 ? w0 : q == 1 ? w1 : q == 2 ? w2 : w3;
                    const int c0 = __popcll(w0), c1 = __popcll(w1), c2 = __popcll(w2), c3 = __popcll(w3);
                    int prefix = (q > 0 ? c0 : 0) + (q > 1 ? c1 : 0) + (q > 2 ? c2 : 0);
                    const int bitpos = (j & 3) * 16 + 4 * g;
                    prefix += __popcll(word & ((1ull << bitpos) - 1ull));
                    const unsigned nib = (unsigned)(word >> bitpos) & 0xFu;
                    const float *vals = reinterpret_cast<const float *>(a.dense_val) + vbase + prefix;
                    float av[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) av[e] = vals[__popc(nib & ((1u << e) - 1u))];
#pragma unroll
                    for (int e = 0; e < 4; ++e) af[e] = (nib >> e & 1u) ? av[e] : 0.f;
                    vbase += c0 + c1 + c2 + c3;
                }
                wave_sync();         // the previous operand reads are done
#pragma unroll
                for (int ps = 0; ps < PASSES; ++ps) *reinterpret_cast<float4_t *>(&stage[(ps * RPW + grp) * LDBS + sub * PL]) = raw[ps];
                wave_sync();
                // k-step e of the 16x16x4 product takes column slot 4g + e from lane group g (the same slots as this lane's
                // 4 A elements): B[4g+e][16n+j] is a plain 4-byte read
                const float *src = &stage[4 * g * LDBS + j];
#pragma unroll
                for (int n = 0; n < NT; ++n)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        acc[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(af[e], src[e * LDBS + 16 * n], acc[n], 0, 0, 0);
            }
        }
        wave_sync();
        // park the accumulators: lane (g, j) holds rows 4g..4g+3, feature 16n + j
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int e = 0; e < 4; ++e) tile[(4 * g + e) * LDC + 16 * n + j] = acc[n][e];
    }
    constexpr int LPF = N / 4;                                   // lanes per tile row at 4 floats each
    constexpr int RPP = WAVE / LPF >= 1 ? WAVE / LPF : 1;        // tile rows per wave pass
    static_assert(LPF <= WAVE, "N too wide for one wave pass");
    const int rr = lane / LPF, cl = lane % LPF;
    if (!tile_ready) {
        // clear the output rows of the tile
#pragma unroll
        for (int r0 = 0; r0 < W; r0 += RPP) {
            const int r = r0 + rr;
            if (out_mask >> r & 1u) *reinterpret_cast<float4_t *>(&tile[r * LDC + cl * 4]) = float4_t{0.f, 0.f, 0.f, 0.f};
        }
    }
    wave_sync();

    // ---- residual nonzeros, ECAP per round: equal contiguous runs per lane group, row sums flushed into the tile ----
    for (int e0 = 0; e0 < L; e0 += ECAP) {
        const int nE = min(ECAP, L - e0);
        // the next round's entries go in flight now and wait in registers until this round is done
        const int nE_next = min(ECAP, L - e0 - ECAP);
        uint32_t next_ent[ECAP / WAVE];
        float next_val[ECAP / WAVE];
        if (nE_next > 0) {
#pragma unroll
            for (int k = 0; k < ECAP / WAVE; ++k)
                load_blocked_entry(a.res_ent, (int64_t)t.res_begin + e0 + ECAP + min(k * WAVE + lane, nE_next - 1), next_ent[k], next_val[k]);
        }
        // runs are whole batches of U entries (the longest run, which sets the time of the round, needs no more batches
        // for it), so a batch is U consecutive entries from an aligned base address and never leaves the staged array
        static_assert(ECAP % U == 0, "a batch must not straddle the end of the staged entries");
        const int per = ((nE + RPW - 1) / RPW + U - 1) / U * U;
        const int q0 = min(grp * per, nE);
        const int q1 = min(nE, q0 + per);
        // A row is added into the tile by the group that holds its first entry (plain read-add-write:
        // one owner per row).  A group whose run starts inside a row keeps that row's partial sum in
        // registers instead and adds it after the others, in group order, so the order of additions is fixed.
        bool first_is_shared = q0 > 0 && q0 < q1 && ((ent_lds[q0 - 1] ^ ent_lds[q0]) >> RES_ROW_SHIFT) == 0;
        int kept_row = -1;
        float4_t kept = {0.f, 0.f, 0.f, 0.f};
        int cur = -1;
        float4_t acc = {0.f, 0.f, 0.f, 0.f};
        auto add_to_tile = [&](int r, const float4_t &v) {
            float4_t *p = reinterpret_cast<float4_t *>(&tile[r * LDC + sub * PL]);
            float4_t x = *p;
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] += v[e];
            *p = x;
        };
        auto add_product = [&](float v, const float4_t &row) {
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] = fmaf(v, row[e], acc[e]);
        };
        auto flush = [&]() {
            if (first_is_shared) {
                first_is_shared = false;
                kept_row = cur;
                kept = acc;
            } else {
                add_to_tile(cur, acc);
            }
        };
        for (int q = q0; q < q1; q += U) {
            // all entry reads, then all row fetches, back to back
            float4_t raw[U];
            const bool full = q + U <= q1;
            // U consecutive entries from one aligned base address; slots past the run hold valid entries whose fetch is
            // harmless and whose product is never formed
            int ecol[U], erow[U];
            float eval[U];
            {
                uint32_t cr[U], vw[U];
                lds_words<U>(ent_lds + q, cr);
                lds_words<U>(val_lds + q, vw);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    ecol[u] = (int)(cr[u] & RES_COL_MASK);
                    erow[u] = (int)(cr[u] >> RES_ROW_SHIFT);
                    eval[u] = __uint_as_float(vw[u]);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) raw[u] = load_row4(Bp, ecol[u], ldb_bytes, sub);
            bool one_row = full;
#pragma unroll
            for (int u = 1; u < U; ++u) one_row = one_row && erow[u] == erow[0];
            if (one_row) {
                // common case (long rows, segments of decomposed rows): the whole batch belongs to one row
                const int r = erow[0];
                if (r != cur) {
                    if (cur >= 0) flush();
                    acc = float4_t{0.f, 0.f, 0.f, 0.f};
                    cur = r;
                }
#pragma unroll
                for (int u = 0; u < U; ++u) add_product(eval[u], raw[u]);
            } else {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (q + u < q1) {
                        const int r = erow[u];
                        if (r != cur) {
                            if (cur >= 0) flush();
                            acc = float4_t{0.f, 0.f, 0.f, 0.f};
                            cur = r;
                        }
                        add_product(eval[u], raw[u]);
                    }
                }
            }
        }
        if (cur >= 0) flush();
        for (int gq = 1; gq < RPW; ++gq) {
            wave_sync();
            if (grp == gq && kept_row >= 0) add_to_tile(kept_row, kept);
        }
        if (nE_next > 0) {
            wave_sync();
#pragma unroll
            for (int k = 0; k < ECAP / WAVE; ++k) {
                ent_lds[k * WAVE + lane] = next_ent[k];
                val_lds[k * WAVE + lane] = next_val[k];
            }
            wave_sync();
        }
    }
    wave_sync();

    // ---- write the tile once: a wave pass covers RPP rows, LPF lanes per row ----
    {
        float *cbase = Cp + (int64_t)t.id * W * a.ldc;
#pragma unroll
        for (int r0 = 0; r0 < W; r0 += RPP) {
            const int r = r0 + rr;
            if (!(out_mask >> r & 1u)) continue;
            float *dst = cbase + (int64_t)r * a.ldc;
            if (store_mask >> r & 1u) {
                // streaming store: C is written once and not read again by this call
                float4_t x = *reinterpret_cast<const float4_t *>(&tile[r * LDC + cl * 4]);
                if (add_to_c) {           // stream order: phase 1 has written the row
                    const float4_t y = *reinterpret_cast<const float4_t *>(dst + cl * 4);
                    x[0] += y[0]; x[1] += y[1]; x[2] += y[2]; x[3] += y[3];
                }
                __builtin_nontemporal_store(x, reinterpret_cast<float4_t *>(dst + cl * 4));
            } else {
                // each atomic instruction covers LPF consecutive floats of the row
#pragma unroll
                for (int e = 0; e < 4; ++e) global_add(dst + e * LPF + cl, tile[r * LDC + e * LPF + cl]);
            }
        }
    }
}

// Clear the rows that several tasks accumulate into, n4 16-byte pieces each (at most 512 columns): CLEAR_ROWS rows per workgroup.
// Once per call and not per column piece: some 5 us each, most of it the launch (power-law graph of 200,003 rows, N = 256 200.8 ->
// 198.8 us; 4, 16 or 32 rows per workgroup are level).
constexpr int CLEAR_ROWS = 8;
__global__ __launch_bounds__(256) void zero_rows_kernel(const int32_t *rows, int64_t nrows, float *C, int64_t ldc, int n4) {
    for (int64_t r0 = (int64_t)blockIdx.x * CLEAR_ROWS; r0 < nrows; r0 += (int64_t)gridDim.x * CLEAR_ROWS) {
        const unsigned pieces = (unsigned)min((int64_t)CLEAR_ROWS, nrows - r0) * (unsigned)n4;
        for (unsigned i = threadIdx.x; i < pieces; i += 256) {
            const unsigned r = i / (unsigned)n4, c4 = i - r * (unsigned)n4;
            *reinterpret_cast<float4_t *>(C + (int64_t)rows[r0 + r] * ldc + c4 * 4) = float4_t{0.f, 0.f, 0.f, 0.f};
        }
    }
}

// fp32 rows of C to the storage type: the listed rows, or all of them (rows = nullptr); n8 groups of eight values each.
template <class T>
__global__ __launch_bounds__(256) void round_rows_kernel(const int32_t *rows, int64_t nrows, const float *C, int64_t ldc, T *R, int64_t ldr, int n8) {
    for (int64_t r0 = (int64_t)blockIdx.x * CLEAR_ROWS; r0 < nrows; r0 += (int64_t)gridDim.x * CLEAR_ROWS) {
        const unsigned groups = (unsigned)min((int64_t)CLEAR_ROWS, nrows - r0) * (unsigned)n8;
        for (unsigned i = threadIdx.x; i < groups; i += 256) {
            const unsigned k = i / (unsigned)n8, c = (i - k * (unsigned)n8) * 8u;
            const int64_t r = rows ? (int64_t)rows[r0 + k] : r0 + k;
            const float4_t *src = reinterpret_cast<const float4_t *>(C + r * ldc + c);
            *reinterpret_cast<uint4 *>(R + r * ldr + c) = round8<T>(src[0], src[1]);
        }
    }
}

// ---------------------------------------------------------------------------------------
// SDDMM
// ---------------------------------------------------------------------------------------
struct SddmmArgs {
    const DevTask *tasks;
    const int32_t *blk_cols;
    const uint64_t *blk_bitmap;
    const int32_t *blk_valptr;
    const uint2 *dense_pv;      // per packed dense nonzero: CSR position, value bits
    int32_t n_dense;
    const void *res_ent;        // blocked words and values
    const int32_t *res_base, *res_row;
    const int32_t *res_perm;    // nullptr: residual entry i is nonzero i
    const void *X;
    const void *Y;
    float *out;
    int64_t M;
    int32_t tasks_per_die;      // as in SpmmArgs
    int32_t tasks_left;         // of a die, from `tasks` on
    int32_t pattern_only;       // nonzero: out_p = <X_i, Y_j>, A's values are not applied
};
// ROUNDED: `out` holds values of the storage type (a template argument: as a flag it took 0.3 % off the fp32 calls)
template <class T, bool ROUNDED>
__device__ inline void put_output(const SddmmArgs &a, int32_t pos, float v) {
    if constexpr (ROUNDED) reinterpret_cast<T *>(a.out)[pos] = to_storage<T>(v);
    else a.out[pos] = v;
}

// Sum over the LPN consecutive lanes of a group; every lane of the group gets the total.
// Steps inside a 16-lane row are DPP moves (no LDS traffic); wider groups finish with wave shuffles.
template <int LPN>
__device__ inline float group_sum(float s) {
    auto dpp = [](float v, auto ctrl) {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), decltype(ctrl)::value, 0xf, 0xf, true));
    };
    if constexpr (LPN >= 2) s += dpp(s, std::integral_constant<int, 0xB1>{});      // quad_perm [1,0,3,2]
    if constexpr (LPN >= 4) s += dpp(s, std::integral_constant<int, 0x4E>{});      // quad_perm [2,3,0,1]
    if constexpr (LPN >= 8) s += dpp(s, std::integral_constant<int, 0x141>{});     // row_half_mirror
    if constexpr (LPN >= 16) s += dpp(s, std::integral_constant<int, 0x140>{});    // row_mirror
#pragma unroll
    for (int m = 16; m < LPN; m <<= 1) s += __shfl_xor(s, m, WAVE);
    return s;
}

// 16-bit rows of Y come through LDS: a row's consecutive pieces are fetched by consecutive lanes, so that the address unit
// handles 64 bytes per access, where operand-shaped loads touch four rows with every four lanes (window tasks of the community
// matrix K = 64 / 128 222 / 372 -> 201 / 328 us; K = 32, blocks only: 65.0 -> 34.5 M accesses of the L1s).  Piece c of row r is
// kept at place c ^ swizzle(r), which spreads the pieces that 16 lanes read together over all banks.
template <int K>
struct RowStage {
    static constexpr int ROW = 2 * K;                        // bytes of a row
    static constexpr int PIECES = K / 8;                     // 16-byte pieces of a row = lanes that fetch it
    static constexpr int RPL = WAVE / PIECES;                // rows per wave load
    static constexpr int ROWS = K >= 128 ? 32 : 64;          // rows staged together
    static constexpr int BYTES = ROWS * ROW;
    __device__ static int swizzle(int row) { return (row * PIECES / 16) & (PIECES - 1); }
    // rows ids[first], ids[first + 1], ... (one id per lane of the wave) of `base` to stage rows at, at + 1, ...
    template <int COUNT>
    __device__ static void fetch(const void *base, int ids, int first, lds_byte *stage, int at) {
        const int lane = threadIdx.x % WAVE;
        int id[COUNT / RPL];
#pragma unroll
        for (int i = 0; i < COUNT / RPL; ++i) id[i] = __builtin_amdgcn_ds_bpermute((first + i * RPL + lane / PIECES) * 4, ids);
#pragma unroll
        for (int i = 0; i < COUNT / RPL; ++i) asm volatile("" : "+v"(id[i]));        // all ids before the first fetch
#pragma unroll
        for (int i = 0; i < COUNT / RPL; ++i) {
            const int piece = (lane % PIECES) ^ swizzle(at + i * RPL + lane / PIECES);
            load_to_lds(reinterpret_cast<const char *>(base) + ((uint64_t)(uint32_t)id[i] * ROW + (uint32_t)piece * 16u), stage + (at + i * RPL) * ROW);
        }
    }
    // operand of 16 staged rows from `at` on: piece g + 4 s of row j
    __device__ static uint4 operand(const lds_byte *stage, int at, int g, int j, int s) {
        return lds_read16(stage + (at + j) * ROW + ((g + 4 * s) ^ swizzle(at + j)) * 16);
    }
};

// Dense blocks of one window: D = Xwin * Y[cols]^T on the MFMA.  The blocks of a task are taken in groups of SD_GROUP: the
// group's 64 rows of Y go through the row stage, and its 16 x 16 products come out of the matrix cores into the same LDS
// bytes (slot sd_stage_slot(block, row, column slot): lane l writes its e-th accumulator of block x to x * 256 + e * 64 + l,
// no bank conflicts, no bitmap needed).  The group's output records - {CSR position, value | stage slot << 16}, stored at
// plan time in ascending CSR position inside every group - are then read by consecutive lanes: coalesced record loads, and
// stores that fall into the row-contiguous runs of the output instead of one 4-byte store per matrix-core lane (the
// write-back of Section 4.4.2, with the popcount offsets resolved when the plan is built).
template <class T, int K, bool ROUNDED>
__device__ inline void sddmm_window_task(const SddmmArgs &a, const DevTask &t, lds_byte *stage) {
    using S = RowStage<K>;
    constexpr int KS = K / 32;               // MFMA k-steps
    constexpr int RU = 4;                    // record loads in flight per lane
    static_assert(SD_GROUP * KB == WAVE, "a lane holds the column of one slot of the group");
    const int lane = threadIdx.x % WAVE;
    const int g = lane >> 4, j = lane & 15;
    const uint16_t *X = reinterpret_cast<const uint16_t *>(a.X);
    lds_float *products = reinterpret_cast<lds_float *>(stage);
    // A operand: row j of the window, k = 32*s + 8g .. +7 (rows past M repeat the last row; no record points at them)
    const int64_t xr = min((int64_t)t.id * W + j, a.M - 1);
    uint4 xa[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) xa[s] = *reinterpret_cast<const uint4 *>(X + xr * K + 32 * s + 8 * g);
    for (int b0 = t.blk_begin; b0 < t.blk_end; b0 += SD_GROUP) {
        const int nb = min(SD_GROUP, t.blk_end - b0);
        // padding slots and blocks past the group fetch a row that no record points at
        const int col = max(a.blk_cols[(int64_t)(b0 + min(g, nb - 1)) * KB + j], 0);
        const unsigned v0 = (unsigned)a.blk_valptr[b0], v1 = (unsigned)a.blk_valptr[b0 + nb];         // unsigned: v1 + RU * WAVE may pass 2^31
        // the first records of the group travel with the Y rows
        uint2 rec[RU];
#pragma unroll
        for (int u = 0; u < RU; ++u) rec[u] = a.dense_pv[min(v0 + u * WAVE + lane, (unsigned)a.n_dense - 1u)];
        float4_t d[SD_GROUP];
#pragma unroll
        for (int h = 0; h < SD_GROUP; h += S::ROWS / KB) {
            if (h < nb) {
                if (S::ROWS > 2 * KB && nb <= 2) S::template fetch<2 * KB>(a.Y, col, h * KB, stage, 0);
                else S::template fetch<S::ROWS>(a.Y, col, h * KB, stage, 0);
                wait_for_loads();
#pragma unroll
                for (int x = 0; x < S::ROWS / KB; ++x) {
                    d[h + x] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int s = 0; s < KS; ++s) d[h + x] = mfma_k32<T>(xa[s], S::operand(stage, x * KB, g, j, s), d[h + x]);
                }
                wait_for_lds();
            }
        }
#pragma unroll
        for (int x = 0; x < SD_GROUP; ++x)
            if (x < nb) {
#pragma unroll
                for (int e = 0; e < 4; ++e) products[x * 256 + e * WAVE + lane] = d[x][e];
            }
        wave_sync();
        for (unsigned q = v0; q < v1; q += RU * WAVE) {
            if (q > v0) {
#pragma unroll
                for (int u = 0; u < RU; ++u) rec[u] = a.dense_pv[min(q + u * WAVE + lane, (unsigned)a.n_dense - 1u)];
            }
#pragma unroll
            for (int u = 0; u < RU; ++u)
                if (q + u * WAVE + lane < v1)
                    put_output<T, ROUNDED>(a, (int32_t)rec[u].x, (a.pattern_only ? 1.f : Elem<T>::word_val(rec[u].y)) * products[rec[u].y >> 16]);
        }
        wait_for_lds();                      // the next group overwrites the stage
    }
}

// fp32 storage: 16 rows of X in LDS, fetched by direct loads, consecutive lanes on one row.  Piece c (16 bytes) of row r is kept at place
// c ^ swizzle(r): 16 lanes that read one piece of 16 rows touch all banks.
template <int K>
struct XStage {
    static constexpr int ROW = 4 * K, PIECES = K / 4, RPL = WAVE / PIECES, BYTES = W * ROW;
    // Do segment tasks use it?  At K = 32 not beside window tasks: the registers of both tasks together would take a wave per SIMD (community
    // matrix of 300,017 rows, default options 67.5 -> 69 - 76 us with any budget; without window tasks 57 -> 49).
    template <bool DENSE> static constexpr bool SEGMENTS = !(DENSE && K == 32);
    __device__ static int swizzle(int row) { return K == 32 ? row >> 1 & 7 : row & 15; }
    // rows first .. first + count - 1; whole loads, whose further rows repeat the last one
    __device__ static void fetch(const void *X, int64_t first, int count, lds_byte *stage) {
        const int lane = threadIdx.x % WAVE;
#pragma unroll
        for (int i = 0; i < W / RPL; ++i) {
            const int r = i * RPL + lane / PIECES;
            if (i * RPL < count)
                load_to_lds(reinterpret_cast<const char *>(X) + ((uint64_t)(first + min(r, count - 1)) * ROW + (uint32_t)((lane % PIECES) ^ swizzle(r)) * 16u), stage + i * RPL * ROW);
        }
    }
    __device__ static float4_t piece(const lds_byte *stage, int row, int c) {
        return *reinterpret_cast<const __attribute__((address_space(3))) float4_t *>(stage + row * ROW + (c ^ swizzle(row)) * 16);
    }
};

// The same for fp32 storage: v_mfma_f32_16x16x4_f32.  A lane (g, j) fetches X[row j][16t + 4g .. +3] and Y[col j][16t + 4g .. +3] as
// 16-byte loads; k-step 4t + e of the product takes element e of both, i.e. lane group g contributes k = 16t + 4g + e to
// that step - any assignment of the k's to steps and lane groups gives the same sum as long as both operands use it.
// (fp32 records are 8 bytes of position and value with no room for a stage slot: they stay in bit order and this task keeps
// the per-lane popcount offsets and 4-byte stores.)
template <int K>
__device__ inline void sddmm_window_task_f32(const SddmmArgs &a, const DevTask &t) {
    static_assert(K <= 64, "wider rows: sddmm_wide_window_task_f32");
    constexpr int KT = K / 16;               // 16-byte pieces per lane and operand row
    constexpr int BB = K <= 32 ? 4 : 2;      // blocks per batch (register budget)
    const int lane = threadIdx.x % WAVE;
    const int g = lane >> 4, j = lane & 15;
    const float *X = reinterpret_cast<const float *>(a.X);
    const float *Y = reinterpret_cast<const float *>(a.Y);
    const int64_t xr = min((int64_t)t.id * W + j, a.M - 1);
    float4_t xa[KT];
#pragma unroll
    for (int s = 0; s < KT; ++s) xa[s] = *reinterpret_cast<const float4_t *>(X + xr * K + 16 * s + 4 * g);
    for (int b0 = t.blk_begin; b0 < t.blk_end; b0 += BB) {
        int col[BB], vptr[BB];
        uint64_t word[BB];
#pragma unroll
        for (int x = 0; x < BB; ++x) {
            const int b = min(b0 + x, t.blk_end - 1);
            col[x] = a.blk_cols[(int64_t)b * KB + j];
            word[x] = a.blk_bitmap[(int64_t)b * 4 + g];          // rows 4g..4g+3 of the block, bit e*16 + j
            vptr[x] = a.blk_valptr[b];
        }
        float4_t yb[BB][KT];
#pragma unroll
        for (int x = 0; x < BB; ++x) {
            const int c = max(col[x], 0);                        // padding slot: no bit is set in its column
#pragma unroll
            for (int s = 0; s < KT; ++s) yb[x][s] = *reinterpret_cast<const float4_t *>(Y + (int64_t)c * K + 16 * s + 4 * g);
        }
        int slot[BB][4];
#pragma unroll
        for (int x = 0; x < BB; ++x) {
            const int cnt = __popcll(word[x]);
            const int c0 = __builtin_amdgcn_readlane(cnt, 0), c1 = __builtin_amdgcn_readlane(cnt, 16), c2 = __builtin_amdgcn_readlane(cnt, 32);
            const int prefix = vptr[x] + (g > 0 ? c0 : 0) + (g > 1 ? c1 : 0) + (g > 2 ? c2 : 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) slot[x][e] = prefix + __popcll(word[x] & ((1ull << (e * 16 + j)) - 1ull));
        }
        uint2 pv[BB][4];
#pragma unroll
        for (int x = 0; x < BB; ++x)
#pragma unroll
            for (int e = 0; e < 4; ++e) pv[x][e] = a.dense_pv[min(slot[x][e], a.n_dense - 1)];
        float4_t d[BB];
#pragma unroll
        for (int x = 0; x < BB; ++x) {
            d[x] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < KT; ++s)
#pragma unroll
                for (int e = 0; e < 4; ++e) d[x] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[s][e], yb[x][s][e], d[x], 0, 0, 0);
        }
#pragma unroll
        for (int x = 0; x < BB; ++x)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (b0 + x < t.blk_end && (word[x] >> (e * 16 + j) & 1ull))
                    a.out[(int32_t)pv[x][e].x] = (a.pattern_only ? 1.f : __uint_as_float(pv[x][e].y)) * d[x][e];
    }
}

// The same for the widest rows, where one block of Y rows at a time left the task waiting: the metadata of four blocks comes in one round
// trip, X stays in LDS, and the registers that it leaves hold the rows of the next block, fetched before the products of this one.  Community
// matrix of 300,017 rows, K = 128, blocks of 32 nonzeros or more: 183.6 -> 173.9 us.  (At K = 64 97 -> 109 us, at K = 32 level.)
__device__ inline void sddmm_wide_window_task_f32(const SddmmArgs &a, const DevTask &t, lds_byte *stage) {
    constexpr int K = 128, GB = 4;           // blocks per group of metadata
    using S = XStage<K>;
    constexpr int KT = K / 16;               // 16-byte pieces per lane and operand row
    const int lane = threadIdx.x % WAVE;
    const int g = lane >> 4, j = lane & 15;
    const float *Y = reinterpret_cast<const float *>(a.Y);
    S::fetch(a.X, (int64_t)t.id * W, (int)min((int64_t)W, a.M - (int64_t)t.id * W), stage);
    for (int b0 = t.blk_begin; b0 < t.blk_end; b0 += GB) {
        const int nb = min(GB, t.blk_end - b0);
        int col[GB], vptr[GB];
        uint64_t word[GB];
#pragma unroll
        for (int x = 0; x < GB; ++x) {
            const int b = b0 + min(x, nb - 1);
            col[x] = a.blk_cols[(int64_t)b * KB + j];
            word[x] = a.blk_bitmap[(int64_t)b * 4 + g];          // rows 4g..4g+3 of the block, bit e*16 + j
            vptr[x] = a.blk_valptr[b];
        }
        float4_t yb[2][KT];
        uint2 pv[2][4];
        auto request = [&](int x) {                              // rows and records of block x
            const int c = max(col[x], 0);                        // padding slot: no bit is set in its column
#pragma unroll
            for (int s = 0; s < KT; ++s) yb[x & 1][s] = *reinterpret_cast<const float4_t *>(Y + (int64_t)c * K + 16 * s + 4 * g);
            const int cnt = __popcll(word[x]);
            const int c0 = __builtin_amdgcn_readlane(cnt, 0), c1 = __builtin_amdgcn_readlane(cnt, 16), c2 = __builtin_amdgcn_readlane(cnt, 32);
            const int prefix = vptr[x] + (g > 0 ? c0 : 0) + (g > 1 ? c1 : 0) + (g > 2 ? c2 : 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) pv[x & 1][e] = a.dense_pv[min(prefix + (int)__popcll(word[x] & ((1ull << (e * 16 + j)) - 1ull)), a.n_dense - 1)];
        };
        request(0);
        if (b0 == t.blk_begin) wait_for_loads();                 // the rows of X
#pragma unroll
        for (int x = 0; x < GB; ++x) {
            if (x < nb) {
                if (x + 1 < GB && x + 1 < nb) request(x + 1);
                float4_t d = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < KT; ++s) {
                    const float4_t xa = S::piece(stage, j, 4 * s + g);
#pragma unroll
                    for (int e = 0; e < 4; ++e) d = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[e], yb[x & 1][s][e], d, 0, 0, 0);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (word[x] >> (e * 16 + j) & 1ull) a.out[(int32_t)pv[x & 1][e].x] = (a.pattern_only ? 1.f : __uint_as_float(pv[x & 1][e].y)) * d[e];
            }
        }
    }
}

// A lane's residual entry: what is loaded, back to back, and what it says.
template <class T>
struct SegmentEntry {
    uint32_t word;
    typename Elem<T>::val_t v;
    int i, base, pos;
    __device__ void load(const SddmmArgs &a, int at) {
        i = at;
        load_blocked_entry(a.res_ent, (int64_t)i, word, v);
        base = a.res_base[i / RES_BLOCK];
        pos = i;
        if (a.res_perm) pos = a.res_perm[i];
    }
    __device__ int col() const { return (int)(word & RES_COL_MASK); }
    __device__ int row(const SddmmArgs &a) const {
        const uint32_t delta = word >> RES_ROW_SHIFT;
        int r = base + (int)delta;
        if (__any(delta == RES_FAR)) {           // rows far apart (nearly empty rows): one more load, whole waves only
            const int far = a.res_row[i];
            if (delta == RES_FAR) r = far;
        }
        return r;
    }
    __device__ float value() const {
        if constexpr (sizeof(v) == 2) return Elem<T>::word_val((uint32_t)v);
        else return v;
    }
};

// Residual nonzeros, 16-bit storage, on the matrix cores.  16 nonzeros are the 16 columns of a tile: lane (g, j) holds pieces
// g, g + 4, ... (16 bytes each) of Y[col of nonzero j] as B operand.  If the rows of 64 nonzeros in CSR order lie within 16
// consecutive rows (nearly always) the A operand is those rows of X, fetched once and not once per nonzero, and the products
// are the elements (row slot of j, j) of the tile; otherwise slot i of A is the row of nonzero i and the products are the
// diagonal.  Nothing is widened or summed across lanes.
// Bound by the data return units of the L1s (97 % busy on the GAT graph at K = 64, their address units 64 %).  When every nonzero
// fetched its two rows with K/8 lanes and the vector ALUs formed the dot product it was 97 and 86 %: X once per batch and 6
// instead of 16 bytes per entry halve the accesses (322 -> 172 M).  f16, against that version: GAT graph K = 64 772 -> 680 us
// (648 us with segments of 128), power-law K = 32 35.4 -> 27.3, community K = 32 177 -> 146, irregular 1,905 -> 1,770 us (98 M
// lines from behind the L2s, at the rate at which they come).  Fetching the next batch's entries early: no change.
template <class T, int K, bool ROUNDED>
__device__ inline void sddmm_segment_task(const SddmmArgs &a, const DevTask &t, lds_byte *stage) {
    using S = RowStage<K>;
    constexpr int KS = K / 32;                   // MFMA k-steps
    const int lane = threadIdx.x % WAVE;
    const int g = lane >> 4, j = lane & 15;
    lds_float *out_stage = reinterpret_cast<lds_float *>(stage);
    for (int q0 = t.res_begin; q0 < t.res_end; q0 += WAVE) {
        SegmentEntry<T> ent;
        ent.load(a, min(q0 + lane, t.res_end - 1));
        const int col = ent.col(), row = ent.row(a);
        const int r0 = __builtin_amdgcn_readfirstlane(row), r1 = __builtin_amdgcn_readlane(row, WAVE - 1);
        float v[4];
        bool mine[4];
        auto product = [&](int x, const uint4 (&xa)[KS], const uint4 (&yb)[KS], int slot) {
            float4_t d = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < KS; ++s) d = mfma_k32<T>(xa[s], yb[s], d);
#pragma unroll
            for (int e = 0; e < 4; ++e) asm volatile("" : "+v"(d[e]));           // selects, not branches
            const float lo = slot & 1 ? d[1] : d[0], hi = slot & 1 ? d[3] : d[2];
            v[x] = slot & 2 ? hi : lo;
            mine[x] = (slot >> 2) == g;          // the lane that holds row `slot` of column j
        };
        if (r1 - r0 < W) {
            uint4 xa[KS];
#pragma unroll
            for (int s = 0; s < KS; ++s)
                xa[s] = *reinterpret_cast<const uint4 *>(reinterpret_cast<const char *>(a.X) + ((uint64_t)(uint32_t)min(r0 + j, r1) * S::ROW + 64u * s + 16u * g));
#pragma unroll
            for (int h = 0; h < WAVE; h += S::ROWS) {
                S::template fetch<S::ROWS>(a.Y, col, h, stage, 0);
                wait_for_loads();
#pragma unroll
                for (int x = 0; x < S::ROWS / 16; ++x) {
                    uint4 yb[KS];
#pragma unroll
                    for (int s = 0; s < KS; ++s) yb[s] = S::operand(stage, x * 16, g, j, s);
                    product(h / 16 + x, xa, yb, __builtin_amdgcn_ds_bpermute((h + x * 16 + j) * 4, row - r0));
                }
                wait_for_lds();
            }
        } else {
            constexpr int HALF = S::ROWS / 2;    // rows of Y in one half of the stage, the same number of X in the other
#pragma unroll
            for (int h = 0; h < WAVE; h += HALF) {
                S::template fetch<HALF>(a.Y, col, h, stage, 0);
                S::template fetch<HALF>(a.X, row, h, stage, HALF);
                wait_for_loads();
#pragma unroll
                for (int x = 0; x < HALF / 16; ++x) {
                    uint4 xd[KS], yd[KS];
#pragma unroll
                    for (int s = 0; s < KS; ++s) { yd[s] = S::operand(stage, x * 16, g, j, s); xd[s] = S::operand(stage, HALF + x * 16, g, j, s); }
                    product(h / 16 + x, xd, yd, j);
                }
                wait_for_lds();
            }
        }
        // to entry order through the same LDS bytes: one store of 64 consecutive entries
#pragma unroll
        for (int x = 0; x < 4; ++x)
            if (mine[x]) out_stage[x * 16 + j] = v[x];
        wave_sync();
        if (q0 + lane < t.res_end) put_output<T, ROUNDED>(a, ent.pos, (a.pattern_only ? 1.f : ent.value()) * out_stage[lane]);
        wait_for_lds();                          // the next batch overwrites the stage
    }
}

// The same for fp32 storage, where the vector ALUs are the faster unit (v_mfma_f32_16x16x4 forms 16 products per column of
// the tile to use one): K/4 lanes per nonzero, NPW nonzeros per wave pass, U passes in one batch of loads.  If the rows of 64 nonzeros in
// CSR order lie within 16 consecutive rows (nearly always) those rows of X come through LDS, once and not once per nonzero: the data
// return units of the L1s then carry the rows of Y alone.  Residual nonzeros only, before -> with it: community matrix of 300,017 rows
// K = 32 / 64 / 128 57.4 / 96.3 / 254.9 -> 49.1 / 84.7 / 215.0 us, power-law graph of 2^17 rows 35.7 / 60.9 / 141.6 -> 30.5 / 55.1 / 121.7.
template <int K, bool STAGED>
__device__ inline void sddmm_segment_task_f32(const SddmmArgs &a, const DevTask &t, lds_byte *stage) {
    using S = XStage<K>;
    constexpr int LPN = K / 4;              // lanes per nonzero
    constexpr int NPW = WAVE / LPN;          // nonzeros per wave pass
    constexpr int U = 8;                     // passes in flight
    static_assert(LPN >= 4 && LPN % 4 == 0 && LPN <= WAVE && WAVE % (NPW * U) == 0, "unsupported K (whole quads per nonzero)");
    const int lane = threadIdx.x % WAVE;
    const int sub = lane % LPN, grp = lane / LPN;
    lds_float *sums = reinterpret_cast<lds_float *>(stage + (STAGED ? S::BYTES : 0));
    for (int q0 = t.res_begin; q0 < t.res_end; q0 += WAVE) {
        const int n = min(WAVE, t.res_end - q0);
        SegmentEntry<float> ent;
        ent.load(a, q0 + min(lane, n - 1));
        const int col = ent.col(), row = ent.row(a);
        const int r0 = __builtin_amdgcn_readfirstlane(row), rows = __builtin_amdgcn_readlane(row, WAVE - 1) - r0 + 1;
        const bool near = STAGED && rows <= W;
        if (near) S::fetch(a.X, r0, rows, stage);
        auto sum_up = [&](int e0, int u, const float4_t &x, const float4_t &y) {
            const float s = group_sum<LPN>(dot4(x, y));
            if (sub == 0) sums[e0 + u * NPW + grp] = s;
        };
        auto y_row = [&](int from) { return load_row4(a.Y, __builtin_amdgcn_ds_bpermute(from, col), K * 4, sub); };
        if (near) {
            for (int e0 = 0; e0 < n; e0 += NPW * U) {
                float4_t y[U];
#pragma unroll
                for (int u = 0; u < U; ++u) y[u] = y_row((e0 + u * NPW + grp) * 4);
                if (e0 == 0) wait_for_loads();
#pragma unroll
                for (int u = 0; u < U; ++u) sum_up(e0, u, S::piece(stage, __builtin_amdgcn_ds_bpermute((e0 + u * NPW + grp) * 4, row - r0), sub), y[u]);
            }
        } else {
            constexpr int V = STAGED ? U / 2 : U;  // both rows of a nonzero in registers
            for (int e0 = 0; e0 < n; e0 += NPW * V) {
                float4_t x[V], y[V];
#pragma unroll
                for (int u = 0; u < V; ++u) {
                    const int from = (e0 + u * NPW + grp) * 4;
                    x[u] = load_row4(a.X, __builtin_amdgcn_ds_bpermute(from, row), K * 4, sub);
                    y[u] = y_row(from);
                }
#pragma unroll
                for (int u = 0; u < V; ++u) sum_up(e0, u, x[u], y[u]);
            }
        }
        wave_sync();
        if (lane < n) a.out[ent.pos] = (a.pattern_only ? 1.f : ent.value()) * sums[lane];
        if constexpr (STAGED) wait_for_lds();                // the next batch overwrites the stage
        else wave_sync();
    }
}

// One launch for both kinds of SDDMM task: the window tasks, heaviest first, then the residual segments.  A workgroup is
// WPB waves, each with a task of its own; nothing is shared between them but the compute unit.  Workgroup b runs on die
// b mod 8 and takes WPB consecutive tasks of that die's part of the table.  WPB = 4 is used when the table is in the
// die-aware order: its consecutive tasks are then neighbouring windows (or runs of consecutive segments) that read the
// same rows of Y, and four of them on one compute unit find each other's rows in its L1 (community matrix, K = 64:
// matrix-unit-only 249 -> 208 us, hybrid 265 -> 247 us, same box).  Elsewhere one wave per workgroup is better (power-law
// graph 31.0 vs 32.3 us: a workgroup's slots are only free again when its slowest wave has finished).
// DENSE = false: the table has no window task (a plan without dense blocks).  At K = 64 the LDS allows five waves per SIMD
// and the registers are held to that (GAT 688 -> 674 us, power-law 41.9 -> 40.4); at K = 128 it would spill (327 -> 373).
// fp32: at K = 128 the window task would take registers for three waves per SIMD.
template <class T, int K> constexpr int SDDMM_WAVES = std::is_same<T, float>::value ? (K == 128 ? 4 : 1) : K == 64 ? 5 : 1;
template <class T, int K, int WPB, bool DENSE, bool ROUNDED>
__global__ __launch_bounds__(WAVE * WPB) __attribute__((amdgpu_waves_per_eu(SDDMM_WAVES<T, K>))) void sddmm_task_kernel(SddmmArgs a) {
    constexpr bool F32 = std::is_same<T, float>::value;
    constexpr int PRODUCTS = DENSE ? SD_GROUP * 256 * 4 : WAVE * 4, ROWS = RowStage<K>::BYTES;
    constexpr int STAGE = F32 ? (XStage<K>::template SEGMENTS<DENSE> ? XStage<K>::BYTES : 0) + WAVE * 4 : PRODUCTS > ROWS ? PRODUCTS : ROWS;           // bytes per wave
    __shared__ __attribute__((aligned(16))) unsigned char stage_all[WPB * STAGE];
    const unsigned wave = WPB == 1 ? 0u : (unsigned)__builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const unsigned seq = (blockIdx.x >> DIE_SHIFT) * WPB + wave;                // position in the die's part of the table
    if (seq >= (unsigned)a.tasks_left) return;
    const DevTask t = a.tasks[(int64_t)(blockIdx.x & (LIBRA_XCDS - 1)) * a.tasks_per_die + seq];
    lds_byte *stage = (lds_byte *)stage_all + wave * STAGE;
    if (DENSE && t.kind == LIBRA_TASK_WINDOW) {
        if constexpr (F32 && K == 128) sddmm_wide_window_task_f32(a, t, stage);
        else if constexpr (F32) sddmm_window_task_f32<K>(a, t);
        else sddmm_window_task<T, K, ROUNDED>(a, t, stage);
        return;
    }
    if constexpr (F32) sddmm_segment_task_f32<K, XStage<K>::template SEGMENTS<DENSE>>(a, t, stage);
    else sddmm_segment_task<T, K, ROUNDED>(a, t, stage);
}

// ---------------------------------------------------------------------------------------
// Edge softmax (one wave per row, rows dealt round-robin) and value scatter
// ---------------------------------------------------------------------------------------
// Maximum over a group of LPN (2, 4, 8 or 16) neighbouring lanes of a DPP row; every lane gets the result.
template <int LPN>
__device__ inline float group_max(float s) {
    static_assert(LPN == 2 || LPN == 4 || LPN == 8 || LPN == 16, "inside one DPP row");
    auto dpp = [](float v, auto ctrl) {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), decltype(ctrl)::value, 0xf, 0xf, true));
    };
    if constexpr (LPN >= 2) s = fmaxf(s, dpp(s, std::integral_constant<int, 0xB1>{}));      // quad_perm [1,0,3,2]
    if constexpr (LPN >= 4) s = fmaxf(s, dpp(s, std::integral_constant<int, 0x4E>{}));      // quad_perm [2,3,0,1]
    if constexpr (LPN >= 8) s = fmaxf(s, dpp(s, std::integral_constant<int, 0x141>{}));     // row_half_mirror
    if constexpr (LPN >= 16) s = fmaxf(s, dpp(s, std::integral_constant<int, 0x140>{}));    // row_mirror
    return s;
}
constexpr int SHORT_LANES = 8;                  // lanes per row of up to 64 nonzeros
constexpr int SHORT_LOADS = 64 / SHORT_LANES;   // scores per lane


// Rows of up to 64 nonzeros (the bulk of a graph): SHORT_LANES lanes per row, read once and kept in registers.
template <class TO>
__device__ inline void edge_softmax_short_rows(unsigned block, unsigned nblocks, const int32_t *rowptr, int64_t M, const float *score, float scale, TO *out) {
    constexpr int SL = SHORT_LANES, KPL = SHORT_LOADS;
    const int l = threadIdx.x % SL;
    const int64_t group = ((int64_t)block * blockDim.x + threadIdx.x) / SL;
    const int64_t ngroups = ((int64_t)nblocks * blockDim.x) / SL;
    for (int64_t i = group; i < M; i += ngroups) {
        const int s = rowptr[i], n = rowptr[i + 1] - s;
        if (n == 0 || n > 64) continue;         // longer rows are listed at plan time and run below
        {
            float v[KPL];
#pragma unroll
            for (int k = 0; k < KPL; ++k) v[k] = score[s + min(l + SL * k, n - 1)];
            float mx = -INFINITY;
#pragma unroll
            for (int k = 0; k < KPL; ++k) {
                v[k] = l + SL * k < n ? scale * v[k] : -INFINITY;
                mx = fmaxf(mx, v[k]);
            }
            mx = group_max<SL>(mx);
            float den = 0.f;
#pragma unroll
            for (int k = 0; k < KPL; ++k) { v[k] = __expf(v[k] - mx); den += v[k]; }      // exp(-inf) = 0 for the padding
            const float inv = 1.f / group_sum<SL>(den);
#pragma unroll
            for (int k = 0; k < KPL; ++k)
                if (l + SL * k < n) out[s + l + SL * k] = to_storage<TO>(v[k] * inv);
        }
    }
}

// Rows listed at plan time: 65 .. LIBRA_SOFTMAX_LONG_ROW nonzeros, THREADS = MEDIUM_LANES lanes per row (whole groups
// of lanes inside a wave), and longer ones, one 256-thread workgroup per row.  A thread takes UNR scores per round, all loads in flight
// together; the row's maximum and denominator come from one pass (running maximum, sum rescaled when it grows); the second
// pass writes, from the registers if the whole row fitted one round and from a second read (cache) otherwise.
template <int THREADS>
__device__ inline float list_sum(float x, float *red) {
#pragma unroll
    for (int m = 1; m < (THREADS < WAVE ? THREADS : WAVE); m <<= 1) x += __shfl_xor(x, m, WAVE);
    if constexpr (THREADS > WAVE) {
        __syncthreads();                // earlier readers of `red` are done
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
        __syncthreads();
        x = 0.f;
#pragma unroll
        for (int w = 0; w < THREADS / WAVE; ++w) x += red[w];
    }
    return x;
}
template <int THREADS>
__device__ inline float list_max(float x, float *red) {
#pragma unroll
    for (int m = 1; m < (THREADS < WAVE ? THREADS : WAVE); m <<= 1) x = fmaxf(x, __shfl_xor(x, m, WAVE));
    if constexpr (THREADS > WAVE) {
        __syncthreads();
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
        __syncthreads();
        x = red[0];
#pragma unroll
        for (int w = 1; w < THREADS / WAVE; ++w) x = fmaxf(x, red[w]);
    }
    return x;
}

template <class TO, int THREADS, int UNR>
__device__ inline void edge_softmax_listed_row(unsigned block, const int32_t *rowptr, const int32_t *rows, int nrows, const float *score, float scale, TO *out) {
    __shared__ float red[4];
    static_assert(THREADS == 256 || (THREADS <= WAVE && WAVE % THREADS == 0), "a workgroup per row, or whole groups of lanes inside a wave");
    const int tid = (int)threadIdx.x % THREADS;
    const int w = (int)((block * 256u + threadIdx.x) / THREADS);
    if (w >= nrows) return;             // whole lane groups or whole workgroups leave together
    const int64_t i = rows[w];
    const int s = rowptr[i], n = rowptr[i + 1] - s;
    const float *sc = score + s;
    float v[UNR];
    auto fetch = [&](int q0) {          // clamped addresses, padding becomes -inf afterwards
#pragma unroll
        for (int u = 0; u < UNR; ++u) v[u] = sc[min(q0 + u * THREADS + tid, n - 1)];
#pragma unroll
        for (int u = 0; u < UNR; ++u) v[u] = q0 + u * THREADS + tid < n ? scale * v[u] : -INFINITY;
    };
    float m = -INFINITY, d = 0.f;
    for (int q0 = 0; q0 < n; q0 += THREADS * UNR) {
        fetch(q0);
        float bm = v[0];
#pragma unroll
        for (int u = 1; u < UNR; ++u) bm = fmaxf(bm, v[u]);
        const float nm = fmaxf(m, bm);
        if (nm > -INFINITY) {           // this thread has seen a score
            float acc = 0.f;
#pragma unroll
            for (int u = 0; u < UNR; ++u) acc += __expf(v[u] - nm);
            d = d * __expf(m - nm) + acc;       // m = -inf: d is 0 and exp(-inf) = 0
            m = nm;
        }
    }
    const float mx = list_max<THREADS>(m, red);
    const float den = list_sum<THREADS>(m > -INFINITY ? d * __expf(m - mx) : 0.f, red);
    const float inv = 1.f / den;
    const bool in_registers = n <= THREADS * UNR;
    for (int q0 = 0; q0 < n; q0 += THREADS * UNR) {
        if (!in_registers) fetch(q0);
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const int q = q0 + u * THREADS + tid;
            if (q < n) out[s + q] = to_storage<TO>(__expf(v[u] - mx) * inv);
        }
    }
}

// The three row classes in one launch of 256-thread workgroups: first one workgroup per long row (the plan lists them
// longest first: the longest row sets the time of its class, so it starts first and the rest of the launch runs beside
// it), then 256 / MEDIUM_LANES medium rows per workgroup, then the workgroups that walk the rows of 64 nonzeros or fewer.
// GAT graph (2^20 rows, 60.7 M nonzeros): 196 us as three launches, 159 us as one, 150 us with 32 instead of 64 lanes per
// medium row (more rows in flight per wave; 16 lanes: 149 us).
constexpr int MEDIUM_LANES = 32;        // lanes per medium row
struct SoftmaxRows {
    const int32_t *rowptr, *long_rows, *medium_rows;
    int64_t M;
    int32_t nlong, nmedium;
    uint32_t medium_blocks, short_blocks;
};
__host__ inline SoftmaxRows softmax_rows(const libra_plan_t *P) {
    SoftmaxRows r{P->d_rowptr, P->d_long_rows, P->d_medium_rows, P->M, (int32_t)P->long_rows.size(), (int32_t)P->n_medium_rows, 0u, 0u};
    r.medium_blocks = ((uint32_t)r.nmedium + 256u / MEDIUM_LANES - 1u) / (256u / MEDIUM_LANES);
    r.short_blocks = (uint32_t)std::min<int64_t>((P->M * SHORT_LANES + 255) / 256, 1 << 18);
    return r;
}
template <class TO>
__global__ __launch_bounds__(256) void edge_softmax_kernel(SoftmaxRows r, const float *score, float scale, TO *out) {
    const unsigned b = blockIdx.x;
    if (b < (unsigned)r.nlong) edge_softmax_listed_row<TO, 256, 16>(b, r.rowptr, r.long_rows, r.nlong, score, scale, out);
    else if (b < (unsigned)r.nlong + r.medium_blocks) edge_softmax_listed_row<TO, MEDIUM_LANES, 8>(b - (unsigned)r.nlong, r.rowptr, r.medium_rows, r.nmedium, score, scale, out);
    else edge_softmax_short_rows<TO>(b - (unsigned)r.nlong - r.medium_blocks, r.short_blocks, r.rowptr, r.M, score, scale, out);
}

// TD: dalpha in alpha's 16-bit type or fp32.  Together with SDDMM results and value products that leave in 16 bits (no fp32 arrays and
// conversions between the steps) a training step with attention, 500,009 rows, bf16, K = 64 went from 1,573 to 1,487 us.
// Backward of the edge softmax: dscore_p = scale * alpha_p * (dalpha_p - sum_row alpha_q dalpha_q).  Same three row
// classes as the forward kernels.
template <class TA> __device__ inline float from_storage(TA x) { return (float)x; }
template <> __device__ inline float from_storage<bf16_t>(bf16_t x) { return __uint_as_float((uint32_t)x.bits << 16); }

template <class TA, class TD>
__device__ inline void edge_softmax_bwd_short_rows(unsigned block, unsigned nblocks, const int32_t *rowptr, int64_t M, const TA *alpha, const TD *dalpha, float scale, float *dscore) {
    constexpr int SL = SHORT_LANES, KPL = SHORT_LOADS;
    const int l = threadIdx.x % SL;
    const int64_t group = ((int64_t)block * blockDim.x + threadIdx.x) / SL;
    const int64_t ngroups = ((int64_t)nblocks * blockDim.x) / SL;
    for (int64_t i = group; i < M; i += ngroups) {
        const int s = rowptr[i], n = rowptr[i + 1] - s;
        if (n == 0 || n > 64) continue;
        // clamped addresses, all loads in flight together; the padding contributes zero
        TA ar[KPL];
        TD gr[KPL];
        float a[KPL], g[KPL], dot = 0.f;
#pragma unroll
        for (int k = 0; k < KPL; ++k) {
            const int q = s + min(l + SL * k, n - 1);
            ar[k] = alpha[q];
            gr[k] = dalpha[q];
        }
#pragma unroll
        for (int k = 0; k < KPL; ++k) {
            a[k] = l + SL * k < n ? from_storage<TA>(ar[k]) : 0.f;
            g[k] = from_storage<TD>(gr[k]);
            dot += a[k] * g[k];
        }
        dot = group_sum<SL>(dot);
#pragma unroll
        for (int k = 0; k < KPL; ++k)
            if (l + SL * k < n) dscore[s + l + SL * k] = scale * a[k] * (g[k] - dot);
    }
}

// MEDIUM_LANES lanes per listed row (65 .. LIBRA_SOFTMAX_LONG_ROW nonzeros), or one 256-thread workgroup per listed long row;
// UNR pairs per thread and round, as in the forward kernel
template <class TA, class TD, int THREADS, int UNR>
__device__ inline void edge_softmax_bwd_listed_row(unsigned block, const int32_t *rowptr, const int32_t *rows, int nrows, const TA *alpha, const TD *dalpha, float scale, float *dscore) {
    __shared__ float red[4];
    static_assert(THREADS == 256 || (THREADS <= WAVE && WAVE % THREADS == 0), "a workgroup per row, or whole groups of lanes inside a wave");
    const int tid = (int)threadIdx.x % THREADS;
    const int w = (int)((block * 256u + threadIdx.x) / THREADS);
    if (w >= nrows) return;             // whole lane groups or whole workgroups leave together
    const int64_t i = rows[w];
    const int s = rowptr[i], n = rowptr[i + 1] - s;
    float a[UNR], g[UNR];
    auto fetch = [&](int q0) {          // clamped addresses; padding contributes zero
        TA ar[UNR];
        TD gr[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const int q = min(q0 + u * THREADS + tid, n - 1);
            ar[u] = alpha[s + q];
            gr[u] = dalpha[s + q];
        }
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            a[u] = q0 + u * THREADS + tid < n ? from_storage<TA>(ar[u]) : 0.f;
            g[u] = from_storage<TD>(gr[u]);
        }
    };
    float dot = 0.f;
    for (int q0 = 0; q0 < n; q0 += THREADS * UNR) {
        fetch(q0);
#pragma unroll
        for (int u = 0; u < UNR; ++u) dot += a[u] * g[u];
    }
    dot = list_sum<THREADS>(dot, red);
    const bool in_registers = n <= THREADS * UNR;
    for (int q0 = 0; q0 < n; q0 += THREADS * UNR) {
        if (!in_registers) fetch(q0);
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const int q = q0 + u * THREADS + tid;
            if (q < n) dscore[s + q] = scale * a[u] * (g[u] - dot);
        }
    }
}

template <class TA, class TD>
__global__ __launch_bounds__(256) void edge_softmax_bwd_kernel(SoftmaxRows r, const TA *alpha, const TD *dalpha, float scale, float *dscore) {
    const unsigned b = blockIdx.x;
    if (b < (unsigned)r.nlong) edge_softmax_bwd_listed_row<TA, TD, 256, 8>(b, r.rowptr, r.long_rows, r.nlong, alpha, dalpha, scale, dscore);
    else if (b < (unsigned)r.nlong + r.medium_blocks) edge_softmax_bwd_listed_row<TA, TD, MEDIUM_LANES, 8>(b - (unsigned)r.nlong, r.rowptr, r.medium_rows, r.nmedium, alpha, dalpha, scale, dscore);
    else edge_softmax_bwd_short_rows<TA, TD>(b - (unsigned)r.nlong - r.medium_blocks, r.short_blocks, r.rowptr, r.M, alpha, dalpha, scale, dscore);
}

// out[p] = factor[p] * val[p], rounded once, in one pass (bound by memory: 8 bytes per nonzero; as conversion, product and
// rounding it was 26); eight per thread where the three arrays lie on 16-byte boundaries.
template <class T>
__global__ __launch_bounds__(256) void value_products_kernel(const T *val, const float *factor, int64_t n, T *out, bool whole) {
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, nthreads = (int64_t)gridDim.x * blockDim.x;
    const int64_t groups = whole ? n / 8 : 0;
    for (int64_t g = tid; g < groups; g += nthreads) {
        const uint4 raw = reinterpret_cast<const uint4 *>(val)[g];
        const float4_t f0 = reinterpret_cast<const float4_t *>(factor)[2 * g], f1 = reinterpret_cast<const float4_t *>(factor)[2 * g + 1];
        const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
        float4_t lo, hi;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            lo[2 * k] = f0[2 * k] * Elem<T>::word_val(w[k] & 0xffffu);
            lo[2 * k + 1] = f0[2 * k + 1] * Elem<T>::word_val(w[k] >> 16);
            hi[2 * k] = f1[2 * k] * Elem<T>::word_val(w[k + 2] & 0xffffu);
            hi[2 * k + 1] = f1[2 * k + 1] * Elem<T>::word_val(w[k + 2] >> 16);
        }
        reinterpret_cast<uint4 *>(out)[g] = round8<T>(lo, hi);
    }
    for (int64_t i = groups * 8 + tid; i < n; i += nthreads) out[i] = to_storage<T>(factor[i] * from_storage<T>(val[i]));
}

inline int hip_rc(hipError_t e) { return e == hipSuccess ? LIBRA_OK : LIBRA_ERR_HIP; }

// A launch has fewer than 2^32 threads (one of more is cut short without an error): a table with a wave per task takes several
// launches from LAUNCH_WAVES waves on.  In launches of whole rounds (a task of each die) the next one starts further into a.tasks.
constexpr int64_t LAUNCH_WAVES = 1 << 25;

template <class T, int N, bool ROUNDED = false>
int launch_spmm(const SpmmArgs &all, int64_t ntasks, hipStream_t s) {
    SpmmArgs a = all;
    const int64_t rounds = ntasks / LIBRA_XCDS, most = LAUNCH_WAVES / LIBRA_XCDS / a.pieces;
    for (int64_t r = 0; r < rounds; r += most, a.tasks += most) {
        const dim3 grid((unsigned)(std::min(most, rounds - r) * LIBRA_XCDS * a.pieces));
        if constexpr (std::is_same<T, float>::value) hipLaunchKernelGGL((spmm_task_kernel_f32<N>), grid, dim3(WAVE), 0, s, a);
        else hipLaunchKernelGGL((spmm_gather_kernel<T, N, ROUNDED>), grid, dim3(WAVE), 0, s, a);
        if (hipGetLastError() != hipSuccess) return LIBRA_ERR_HIP;
    }
    return LIBRA_OK;
}

int spmm_launch(const libra_plan_t *P, const SpmmArgs &a, int n, int64_t nt, hipStream_t s);

// `pieces` adjacent pieces of n columns each, one launch
int spmm_piece(const libra_plan_t *P, const void *B, int n, int pieces, int64_t ldb, float *C, int64_t ldc, void *R, int64_t ldr, hipStream_t s) {
    const SubPlan &sp = P->spmm;
    const int64_t per_die = (sp.n.tasks + LIBRA_XCDS - 1) / LIBRA_XCDS;
    SpmmArgs a{sp.dev.tasks, sp.dev.blk_cols, sp.dev.blk_bitmap, sp.dev.blk_valptr, sp.dev.dense_val,
               sp.dev.res_ent, B, C, ldb, ldc, (int32_t)per_die, pieces, 0, R, ldr};
    const int64_t nt = per_die * LIBRA_XCDS;         // every slot of the table (the last few may hold empty tasks)
    if (P->o.two_kernels && a.phase == 0) {
        // ablation / debugging schedule: the matrix-unit part and the scalar part as two launches on the stream
        for (int phase = 1; phase <= 2; ++phase) {
            SpmmArgs b = a;
            b.phase = phase;
            if (int rc = spmm_launch(P, b, n, nt, s)) return rc;
        }
        return LIBRA_OK;
    }
    return spmm_launch(P, a, n, nt, s);
}

int spmm_launch(const libra_plan_t *P, const SpmmArgs &a, int n, int64_t nt, hipStream_t s) {
    auto width16 = [&](auto tag, auto rounded) {
        typedef decltype(tag) T;
        constexpr bool ROUNDED = decltype(rounded)::value;
        switch (n) {
        case 32: return launch_spmm<T, 32, ROUNDED>(a, nt, s);
        case 64: return launch_spmm<T, 64, ROUNDED>(a, nt, s);
        case 128: return launch_spmm<T, 128, ROUNDED>(a, nt, s);
        }
        return (int)LIBRA_ERR_UNSUPPORTED;
    };
    if (P->vdt != LIBRA_F32) {
        if (P->vdt == LIBRA_F16) return a.R ? width16(half_t{}, std::true_type{}) : width16(half_t{}, std::false_type{});
        return a.R ? width16(bf16_t{}, std::true_type{}) : width16(bf16_t{}, std::false_type{});
    } else {
        switch (n) {
        case 16: return launch_spmm<float, 16>(a, nt, s);
        case 32: return launch_spmm<float, 32>(a, nt, s);
        case 64: return launch_spmm<float, 64>(a, nt, s);
        case 128: return launch_spmm<float, 128>(a, nt, s);
        }
    }
    return LIBRA_ERR_UNSUPPORTED;
}

}  // namespace

// =========================================================================================
// C ABI: upload and compute
// =========================================================================================
namespace {
size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// One row of workgroups per copy.
__global__ __launch_bounds__(256) void device_copies_kernel(DeviceCopies c) {
    const auto &p = c.part[blockIdx.y];
    const uint64_t tid = (uint64_t)blockIdx.x * 256 + threadIdx.x, nthreads = (uint64_t)gridDim.x * 256;
    const uintptr_t at = (uintptr_t)p.to | (uintptr_t)p.from;
    auto move = [&](auto tag, uint64_t begin) {
        typedef decltype(tag) V;
        const uint64_t n = p.bytes / sizeof(V);
        for (uint64_t i = begin / sizeof(V) + tid; i < n; i += nthreads) reinterpret_cast<V *>(p.to)[i] = reinterpret_cast<const V *>(p.from)[i];
        return n * sizeof(V);
    };
    uint64_t done = 0;
    if (!(at & 15)) done = move(uint4{}, 0);
    else if (!(at & 3)) done = move(uint32_t{}, 0);
    move(uint8_t{}, done);
}

// Lays arrays out back to back (256-byte aligned, 16 spare bytes each) and copies them from host memory, from
// device memory, or only reserves their place (arrays that a kernel packs afterwards).  `gathered`: copies inside device memory share
// launches, and arrays from host memory with nothing between them become one copy, which writes the spare bytes between them; they are
// queued by flush().
struct Uploader {
    char *base = nullptr;     // nullptr: size pass only
    size_t off = 0;
    hipStream_t s = nullptr;
    bool ok = true, gathered = false;
    DeviceCopies copies;
    struct FromHost { const void *from; size_t bytes, at; bool next; };      // next: only spare bytes and empty arrays lie between it and the one before
    std::vector<FromHost> from_host;
    bool host_before = false;                     // the last array that is not empty came from host memory
    std::vector<std::vector<char>> joined;        // alive until the copies have finished
    template <class P>
    void put(const void *host_src, const void *dev_src, size_t bytes, P *&dst) {
        if (base) {
            dst = reinterpret_cast<P *>(base + off);
            if (gathered) {
                if (bytes && host_src) from_host.push_back({host_src, bytes, off, host_before});
                if (bytes && !host_src && dev_src) {
                    if (copies.full()) ok = copies.flush(s) && ok;
                    copies.add(base + off, dev_src, bytes);
                }
                if (bytes) host_before = host_src != nullptr;
            } else {
                if (bytes && host_src && hipMemcpyAsync(base + off, host_src, bytes, hipMemcpyHostToDevice, s) != hipSuccess) ok = false;
                if (bytes && !host_src && dev_src && hipMemcpyAsync(base + off, dev_src, bytes, hipMemcpyDeviceToDevice, s) != hipSuccess) ok = false;
            }
        }
        off += align256(bytes + 16);
    }
    template <class V, class P>
    void putv(const V &v, P *&dst) { put(v.data(), nullptr, v.size() * sizeof(v[0]), dst); }
    void flush() {
        ok = copies.flush(s) && ok;
        for (size_t i = 0; i < from_host.size();) {
            size_t e = i + 1;
            while (e < from_host.size() && from_host[e].next) ++e;
            const size_t begin = from_host[i].at, end = from_host[e - 1].at + from_host[e - 1].bytes;
            joined.emplace_back(end - begin);
            for (; i < e; ++i) std::memcpy(joined.back().data() + (from_host[i].at - begin), from_host[i].from, from_host[i].bytes);
            if (hipMemcpyAsync(base + begin, joined.back().data(), end - begin, hipMemcpyHostToDevice, s) != hipSuccess) ok = false;
        }
        from_host.clear();
    }
};

// Slots of the device task table: the table's length rounded up to whole rounds of the dies.
size_t task_slots(int64_t ntasks) { return (size_t)((ntasks + LIBRA_XCDS - 1) / LIBRA_XCDS) * LIBRA_XCDS; }

// Device task records, die by die (see DIE_SHIFT); the slots past the last task hold empty tasks.
std::vector<DevTask> pack_tasks(const libra_plan_t *P, const SubPlan &sp, bool spmm) {
    const size_t per_die = task_slots((int64_t)sp.tasks.size()) / LIBRA_XCDS;
    const DevTask empty{0, 0, 0, 0, 0, 0u, (uint32_t)(spmm ? LIBRA_TASK_WINDOW : LIBRA_TASK_CHUNK), 0};
    std::vector<DevTask> out(per_die * LIBRA_XCDS, empty);
    for (size_t i = 0; i < sp.tasks.size(); ++i) {
        const libra_task_t &t = sp.tasks[i];
        DevTask d{t.id, t.blk_begin, t.blk_end, t.res_begin, t.res_end, (t.atomic_mask & 0xffffu) | (t.store_mask << 16),
                  (uint32_t)t.kind, t.kind == LIBRA_TASK_WINDOW ? sp.blk_valptr[t.blk_begin] : 0};
        if (spmm && t.kind == LIBRA_TASK_CHUNK) {
            // a segment of a decomposed row = a task of the row's window with one atomic output row
            d.id = t.id / P->o.W;
            d.blk_begin = d.blk_end = 0;
            d.masks = 1u << (t.id % P->o.W);
        }
        out[(i % LIBRA_XCDS) * per_die + i / LIBRA_XCDS] = d;
    }
    return out;
}

// Host staging of everything the kernels read in packed form; alive until the copies have finished.
struct Staging {
    std::vector<DevTask> tasks_a, tasks_d;
    std::vector<unsigned char> res_blocks;  // SpMM residual entries: blocked words and values
    std::vector<unsigned char> sd_res_blocks;
    std::vector<int32_t> sd_res_base;
    std::vector<SdPv> sdpv;
};

// Record layouts written on the device when the arrays come from the device planner.  `base`: nullptr for the SpMM entries
// (upper bits = row in the window); for the SDDMM ones, where the first rows of the blocks go (upper bits = row minus that).
template <class V>
__global__ __launch_bounds__(256) void pack_blocked_entries_kernel(const int32_t *col, const V *val, const int32_t *row, int64_t n, unsigned char *out, int32_t *base) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        unsigned char *blk = out + (i / RES_BLOCK) * (RES_BLOCK * (4 + (int)sizeof(V)));
        const int slot = (int)(i % RES_BLOCK);
        uint32_t upper;
        if (base) {
            const int32_t first = row[i - slot];
            upper = min((uint32_t)(row[i] - first), RES_FAR);
            if (slot == 0) base[i / RES_BLOCK] = first;
        } else {
            upper = (uint32_t)(row[i] % W);
        }
        reinterpret_cast<uint32_t *>(blk)[slot] = (uint32_t)col[i] | upper << RES_ROW_SHIFT;
        reinterpret_cast<V *>(blk + RES_BLOCK * 4)[slot] = val[i];
    }
}
void pack_entries(int value_bytes, const int32_t *col, const void *val, const int32_t *row, int64_t n, void *entries, int32_t *base, hipStream_t s) {
    const dim3 grid((unsigned)std::min<int64_t>((n + 255) / 256, 1 << 16)), block(256);
    if (value_bytes == 4) hipLaunchKernelGGL((pack_blocked_entries_kernel<uint32_t>), grid, block, 0, s, col, (const uint32_t *)val, row, n, (unsigned char *)entries, base);
    else hipLaunchKernelGGL((pack_blocked_entries_kernel<uint16_t>), grid, block, 0, s, col, (const uint16_t *)val, row, n, (unsigned char *)entries, base);
}
template <class V>
__global__ __launch_bounds__(256) void pack_sddmm_values_kernel(const int32_t *perm, const V *val, int64_t n, SdPv *out) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        out[i] = SdPv{perm[i], (uint32_t)val[i]};
}

// 16-bit SDDMM output records written on the device: one wave per window task.  Per group of SD_GROUP blocks the CSR
// positions of the group's packed values go to LDS; a lane then takes 4 bits of each block's bitmap, and for each set bit
// finds the packed value (popcount of the bits below), its rank among the group's positions (a count over the LDS array),
// and writes the record to that rank.
__global__ __launch_bounds__(WAVE) void pack_sddmm_sorted_records_kernel(const DevTask *tasks, const uint64_t *blk_bitmap, const int32_t *blk_valptr,
                                                                         const int32_t *dense_perm, const uint16_t *dense_val, SdPv *out) {
    __shared__ int32_t pos[SD_GROUP * 256];
    const DevTask t = tasks[blockIdx.x];                 // any order: every window task once
    if (t.kind != LIBRA_TASK_WINDOW) return;
    const int lane = threadIdx.x;
    for (int b0 = t.blk_begin; b0 < t.blk_end; b0 += SD_GROUP) {
        const int nb = min(SD_GROUP, t.blk_end - b0);
        const int v0 = blk_valptr[b0], n = blk_valptr[b0 + nb] - v0;
        for (int i = lane; i < n; i += WAVE) pos[i] = dense_perm[v0 + i];
        __syncthreads();
        for (int x = 0; x < nb; ++x) {
            const int b = b0 + x;
            const uint64_t word = blk_bitmap[(int64_t)b * 4 + lane / 16];       // bits 64 (lane / 16) .. + 63 of the block
            const int sh = (lane % 16) * 4;
            int before = 0;                                                     // set bits of the block below this lane's four
            for (int w = 0; w < lane / 16; ++w) before += __popcll(blk_bitmap[(int64_t)b * 4 + w]);
            before += __popcll(word & ((1ull << sh) - 1ull));
            int q = blk_valptr[b] + before;
            for (int e = 0; e < 4; ++e) {
                if (!(word >> (sh + e) & 1ull)) continue;
                const int bit = lane * 4 + e;
                const int32_t p = dense_perm[q];
                int rank = 0;
                for (int i = 0; i < n; ++i) rank += pos[i] < p;
                out[v0 + rank] = SdPv{p, (uint32_t)dense_val[q] | (uint32_t)sd_stage_slot(x, bit / KB, bit % KB) << 16};
                ++q;
            }
        }
        __syncthreads();
    }
}

// st == nullptr: size pass.  da/dd == nullptr: the arrays come from the plan's host vectors; otherwise from
// device memory, and the packed record arrays are only reserved here (adopt_device_arrays fills them).
void layout(libra_plan_t *P, Uploader &u, Staging *st, const DeviceSource *da, const DeviceSource *dd) {
    u.put(st && !da ? (const void *)P->rowptr.data() : nullptr, da ? da->rowptr : nullptr, (size_t)(P->M + 1) * 4, P->d_rowptr);
    u.putv(P->long_rows, P->d_long_rows);
    const bool listed = da && da->medium_rows;
    u.put(st && !listed ? (const void *)P->medium_rows.data() : nullptr, listed ? da->medium_rows : nullptr, (size_t)P->n_medium_rows * 4, P->d_medium_rows);
    SubPlan &sa = P->spmm, &sd = P->sddmm;
    const size_t vs = (size_t)P->vsize;
    const bool from_host = st && !da;
    auto H = [&](const void *p) { return from_host ? p : nullptr; };
    // ---- SpMM ----
    const bool pack_a = st && !(da && da->write_tasks);
    if (pack_a) st->tasks_a = pack_tasks(P, sa, true);
    u.put(pack_a ? (const void *)st->tasks_a.data() : nullptr, nullptr, task_slots(sa.n.tasks) * sizeof(DevTask), sa.dev.tasks);
    const bool pack_d = st && !(dd && dd->write_tasks);
    if (pack_d) st->tasks_d = pack_tasks(P, sd, false);
    u.put(pack_d ? (const void *)st->tasks_d.data() : nullptr, nullptr, task_slots(sd.n.tasks) * sizeof(DevTask), sd.dev.tasks);
    u.put(H(sa.blk_cols.data()), da ? da->blk_cols : nullptr, (size_t)sa.n.col_slots * 4, sa.dev.blk_cols);
    u.put(H(sa.blk_bitmap.data()), da ? da->blk_bitmap : nullptr, (size_t)sa.n.bitmap_words * 8, sa.dev.blk_bitmap);
    u.put(H(sa.blk_valptr.data()), da ? da->blk_valptr : nullptr, P->o.build_spmm ? (size_t)(sa.n.blocks + 1) * 4 : 0, sa.dev.blk_valptr);
    u.put(H(sa.dense_val.data()), da ? da->dense_val : nullptr, (size_t)sa.n.dense * vs, sa.dev.dense_val);
    u.put(H(sa.dense_perm.data()), da ? da->dense_perm : nullptr, (size_t)sa.n.dense * 4, sa.dev.dense_perm);
    const size_t nres = (size_t)sa.n.res;
    const size_t res_bytes = res_blocked_bytes(nres + 1, vs);      // + 1: a task without entries still reads the slot at its (clamped) first index
    // host-side packing of one sub-plan's entries into blocks; upper(i): what goes above the column
    auto pack_entries = [&](const SubPlan &sp, std::vector<unsigned char> &blocks, size_t bytes, auto upper) {
        blocks.assign(bytes, 0);
        for (size_t i = 0; i < (size_t)sp.n.res; ++i) {
            unsigned char *blk = blocks.data() + i / RES_BLOCK * res_block_bytes(vs);
            const uint32_t word = (uint32_t)sp.res_col[i] | upper(i) << RES_ROW_SHIFT;
            std::memcpy(blk + i % RES_BLOCK * 4, &word, 4);
            std::memcpy(blk + RES_BLOCK * 4 + i % RES_BLOCK * vs, sp.res_val.data() + i * vs, vs);
        }
    };
    if (from_host) pack_entries(sa, st->res_blocks, res_bytes, [&](size_t i) { return (uint32_t)(sa.res_row[i] % P->o.W); });
    u.put(from_host ? (const void *)st->res_blocks.data() : nullptr, nullptr, res_bytes, sa.dev.res_ent);
    u.put(H(sa.res_perm.data()), da ? da->res_perm : nullptr, nres * 4, sa.dev.res_perm);
    u.put(H(sa.zero_rows.data()), da ? da->zero_rows : nullptr, (size_t)sa.n.zero_rows * 4, sa.dev.zero_rows);
    // ---- SDDMM ----
    u.put(H(sd.blk_cols.data()), dd ? dd->blk_cols : nullptr, (size_t)sd.n.col_slots * 4, sd.dev.blk_cols);
    u.put(H(sd.blk_bitmap.data()), dd ? dd->blk_bitmap : nullptr, (size_t)sd.n.bitmap_words * 8, sd.dev.blk_bitmap);
    u.put(H(sd.blk_valptr.data()), dd ? dd->blk_valptr : nullptr, P->o.build_sddmm ? (size_t)(sd.n.blocks + 1) * 4 : 0, sd.dev.blk_valptr);
    const size_t ndd = (size_t)sd.n.dense;
    if (from_host) {
        st->sdpv.resize(ndd);
        for (size_t i = 0; i < ndd; ++i) {
            uint32_t bits = 0;
            std::memcpy(&bits, sd.dense_val.data() + i * vs, vs);
            st->sdpv[i] = {sd.dense_perm[i], bits};
        }
        if (sorted_records(P)) {
            // 16-bit records: inside every group of SD_GROUP blocks of a window task, ascending CSR position, each with the
            // stage slot of its product
            std::vector<SdPv> grp;
            for (const libra_task_t &t : sd.tasks) {
                if (t.kind != LIBRA_TASK_WINDOW) continue;
                for (int32_t b0 = t.blk_begin; b0 < t.blk_end; b0 += SD_GROUP) {
                    const int32_t b1 = std::min(t.blk_end, b0 + SD_GROUP);
                    grp.clear();
                    for (int32_t b = b0; b < b1; ++b) {
                        int32_t q = sd.blk_valptr[b];
                        for (int bit = 0; bit < W * KB; ++bit)
                            if (sd.blk_bitmap[(size_t)b * 4 + bit / 64] >> (bit % 64) & 1u) {
                                SdPv r = st->sdpv[q++];
                                r.val |= (uint32_t)sd_stage_slot(b - b0, bit / KB, bit % KB) << 16;
                                grp.push_back(r);
                            }
                    }
                    std::sort(grp.begin(), grp.end(), [](const SdPv &x, const SdPv &y) { return x.perm < y.perm; });
                    std::copy(grp.begin(), grp.end(), st->sdpv.begin() + sd.blk_valptr[b0]);
                }
            }
        }
    }
    u.put(from_host ? (const void *)st->sdpv.data() : nullptr, nullptr, ndd * sizeof(SdPv), sd.dev.dense_pv);
    u.put(H(sd.dense_perm.data()), dd ? dd->dense_perm : nullptr, ndd * 4, sd.dev.dense_perm);
    const size_t nrd = (size_t)sd.n.res, nblocks = (nrd + RES_BLOCK - 1) / RES_BLOCK;
    if (from_host) {
        auto first = [&](size_t i) { return sd.res_row[i / RES_BLOCK * RES_BLOCK]; };
        pack_entries(sd, st->sd_res_blocks, res_blocked_bytes(nrd, vs), [&](size_t i) { return std::min((uint32_t)(sd.res_row[i] - first(i)), RES_FAR); });
        st->sd_res_base.resize(nblocks);
        for (size_t b = 0; b < nblocks; ++b) st->sd_res_base[b] = first(b * RES_BLOCK);
    }
    u.put(from_host ? (const void *)st->sd_res_blocks.data() : nullptr, nullptr, res_blocked_bytes(nrd, vs), sd.dev.res_ent);
    u.put(from_host ? (const void *)st->sd_res_base.data() : nullptr, nullptr, nblocks * 4, sd.dev.res_base);
    u.put(H(sd.res_row.data()), dd ? dd->res_row : nullptr, nrd * 4, sd.dev.res_row);
    // the residual list is ascending in CSR position: if it is the whole matrix, entry i is nonzero i
    if ((int64_t)nrd == P->nnz) {
        if (st) sd.dev.res_perm = nullptr;      // the size pass writes nothing: another thread may be computing with the plan
    } else u.put(H(sd.res_perm.data()), dd ? dd->res_perm : nullptr, nrd * 4, sd.dev.res_perm);
}
}  // namespace

size_t libra::plan_buffer_bytes(const libra_plan_t *plan) {
    Uploader u;
    layout(const_cast<libra_plan_t *>(plan), u, nullptr, nullptr, nullptr);
    return u.off + 256;
}

void libra::pack_sddmm_entries(int value_bytes, const int32_t *col, const void *val, const int32_t *row, int64_t n, void *entries, int32_t *base, void *stream) {
    pack_entries(value_bytes, col, val, row, n, entries, base, (hipStream_t)stream);
}

bool libra::DeviceCopies::flush(void *stream) {
    if (n == 0) return true;
    uint64_t most = 0;
    for (int i = 0; i < n; ++i) most = std::max(most, part[i].bytes);
    const unsigned blocks = (unsigned)std::min<uint64_t>(most / (256 * 16) + 1, 2048);
    hipLaunchKernelGGL(device_copies_kernel, dim3(blocks, (unsigned)n), dim3(256), 0, (hipStream_t)stream, *this);
    n = 0;
    return hipGetLastError() == hipSuccess;
}

int libra::adopt_device_arrays(libra_plan_t *P, const DeviceSource &da, const DeviceSource &dd, void *dev_buf, size_t bytes, void *stream) {
    if (!dev_buf) return LIBRA_ERR_NULL;
    if (bytes < plan_buffer_bytes(P) || ((uintptr_t)dev_buf & 255)) return LIBRA_ERR_BUFFER;
    if (P->Kc > (int64_t)RES_COL_MASK + 1) return LIBRA_ERR_UNSUPPORTED;    // a residual entry keeps its column in RES_ROW_SHIFT bits
    hipStream_t s = (hipStream_t)stream;
    try {
        Staging st;
        Uploader u;
        u.base = (char *)dev_buf;
        u.s = s;
        u.gathered = true;
        layout(P, u, &st, &da, &dd);
        u.flush();
        auto grid = [](int64_t n) { return dim3((unsigned)std::min<int64_t>((n + 255) / 256, 1 << 16)); };
        const SubPlan &sa = P->spmm, &sd = P->sddmm;
        if (da.write_tasks && sa.n.tasks) da.write_tasks(const_cast<DevTask *>(sa.dev.tasks), sa.n.tasks);
        if (dd.write_tasks && sd.n.tasks) dd.write_tasks(const_cast<DevTask *>(sd.dev.tasks), sd.n.tasks);
        if (da.write_residuals) {
            da.write_residuals(sa.dev, sd.dev);
        } else {
            if (sa.n.res) pack_entries(P->vsize, da.res_col, da.res_val, da.res_row, sa.n.res, sa.dev.res_ent, nullptr, s);
            if (sd.n.res) pack_entries(P->vsize, dd.res_col, dd.res_val, dd.res_row, sd.n.res, sd.dev.res_ent, const_cast<int32_t *>(sd.dev.res_base), s);
        }
        if (sd.n.dense) {
            if (P->vdt == LIBRA_F32)
                hipLaunchKernelGGL((pack_sddmm_values_kernel<uint32_t>), grid(sd.n.dense), dim3(256), 0, s, dd.dense_perm,
                                   (const uint32_t *)dd.dense_val, sd.n.dense, (SdPv *)sd.dev.dense_pv);
            else if (sorted_records(P)) {     // reads the task table that has just been queued for writing on this stream
                const int64_t slots = (int64_t)task_slots(sd.n.tasks);
                for (int64_t k = 0; k < slots; k += LAUNCH_WAVES)
                    hipLaunchKernelGGL(pack_sddmm_sorted_records_kernel, dim3((unsigned)std::min(LAUNCH_WAVES, slots - k)), dim3(WAVE), 0, s, sd.dev.tasks + k,
                                       dd.blk_bitmap, dd.blk_valptr, dd.dense_perm, (const uint16_t *)dd.dense_val, (SdPv *)sd.dev.dense_pv);
            } else
                hipLaunchKernelGGL((pack_sddmm_values_kernel<uint16_t>), grid(sd.n.dense), dim3(256), 0, s, dd.dense_perm,
                                   (const uint16_t *)dd.dense_val, sd.n.dense, (SdPv *)sd.dev.dense_pv);
        }
        if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess || !u.ok) return LIBRA_ERR_HIP;
    } catch (...) {
        return LIBRA_ERR_NOMEM;
    }
    P->dev_base = dev_buf;
    P->dev_bytes = bytes;
    return LIBRA_OK;
}

extern "C" int libra_plan_device_bytes(const libra_plan_t *plan, size_t *bytes) {
    if (!plan || !bytes) return LIBRA_ERR_NULL;
    *bytes = plan_buffer_bytes(plan);
    return LIBRA_OK;
}

extern "C" int libra_plan_upload(libra_plan_t *plan, void *dev_buf, size_t bytes, void *stream) {
    if (!plan || !dev_buf) return LIBRA_ERR_NULL;
    if (!plan->host_arrays) return LIBRA_ERR_NOT_BUILT;      // built on the device without a host copy: nothing to upload
    size_t need = 0;
    libra_plan_device_bytes(plan, &need);
    if (bytes < need || ((uintptr_t)dev_buf & 255)) return LIBRA_ERR_BUFFER;
    if (plan->Kc > (int64_t)RES_COL_MASK + 1) return LIBRA_ERR_UNSUPPORTED;      // a residual entry keeps its column in RES_ROW_SHIFT bits
    try {
        Staging st;
        Uploader u;
        u.base = (char *)dev_buf;
        u.s = (hipStream_t)stream;
        layout(plan, u, &st, nullptr, nullptr);
        if (hipStreamSynchronize(u.s) != hipSuccess || !u.ok) return LIBRA_ERR_HIP;
    } catch (...) {
        return LIBRA_ERR_NOMEM;
    }
    plan->dev_base = dev_buf;
    plan->dev_bytes = bytes;
    return LIBRA_OK;
}

namespace {
// R: a second output of 16-bit rows (libra_spmm_rounded); nullptr: C is the output.
int spmm_call(const libra_plan_t *P, const void *B, int32_t N, int64_t ldb, float *C, int64_t ldc, void *R, int64_t ldr, void *stream) {
    if (!P->o.build_spmm) return LIBRA_ERR_NOT_BUILT;
    if (!P->dev_base) return LIBRA_ERR_NOT_UPLOADED;
    if (P->o.W != W || P->o.KB != KB) return LIBRA_ERR_UNSUPPORTED;
    const int unit = P->vdt != LIBRA_F32 ? 32 : 16;
    if (N < unit || N > 512) return LIBRA_ERR_SHAPE;
    if (N % unit) return LIBRA_ERR_UNSUPPORTED;
    // a kernel forms a row's byte offset as a 32 x 32 -> 64 bit product: the row stride in bytes has to fit in 32 bits
    if (ldb < N || ldc < N || ldb * (int64_t)P->vsize >= (1ll << 32)) return LIBRA_ERR_SHAPE;
    if (ldb % (P->vdt != LIBRA_F32 ? 8 : 4) || ldc % 4) return LIBRA_ERR_UNSUPPORTED;
    if (((uintptr_t)B & 15) || ((uintptr_t)C & 15)) return LIBRA_ERR_BUFFER;
    hipStream_t s = (hipStream_t)stream;
    const int esz = P->vsize;
    auto row_blocks = [](int64_t n) { return dim3((unsigned)std::min<int64_t>((n + CLEAR_ROWS - 1) / CLEAR_ROWS, 1 << 16)); };
    const int64_t nz = P->spmm.n.zero_rows;
    if (nz) {
        hipLaunchKernelGGL(zero_rows_kernel, row_blocks(nz), dim3(256), 0, s, P->spmm.dev.zero_rows, nz, C, ldc, N / 4);
        if (hipGetLastError() != hipSuccess) return LIBRA_ERR_HIP;
    }
    // the two-kernel mode adds its second launch to the rows of C: all of them are rounded afterwards
    const bool all_rows = R && P->o.two_kernels;
    // the feature dimension is cut into pieces the kernels are instantiated for; at most 128 columns, the widest
    // piece whose tile leaves four waves per SIMD (a 256-column piece ran at two and took 2.5x the time of a 128-column one)
    for (int n0 = 0; n0 < N;) {
        int n = 128;
        while (n > N - n0) n >>= 1;
        // The 128-column pieces of a wide operand go into one launch when the plan keeps neighbouring windows on one die
        // (matrices whose windows share columns: the pieces of a task then share the plan's data and the launch has one
        // tail; community N=256: 535 -> 508 us).  Elsewhere they run one after the other: together they would compete for
        // the L2 with twice the rows of B (power-law N=512: 267 us apart, 354 us together).
        const int pieces = (n == 128 && P->o.xcd_order == 1) ? (N - n0) / 128 : 1;
        int rc = spmm_piece(P, (const char *)B + (size_t)n0 * esz, n, pieces, ldb, C ? C + n0 : nullptr, ldc, R && !all_rows ? (char *)R + (size_t)n0 * esz : nullptr, ldr, s);
        if (rc != LIBRA_OK) return rc;
        n0 += n * pieces;
    }
    if (R && (nz || all_rows)) {
        auto run = [&](auto tag) {
            typedef decltype(tag) T;
            const int64_t rows = all_rows ? P->M : nz;
            hipLaunchKernelGGL((round_rows_kernel<T>), row_blocks(rows), dim3(256), 0, s, all_rows ? nullptr : P->spmm.dev.zero_rows, rows, C, ldc,
                               reinterpret_cast<T *>(R), ldr, N / 8);
        };
        if (P->vdt == LIBRA_F16) run(half_t{});
        else run(bf16_t{});
        if (hipGetLastError() != hipSuccess) return LIBRA_ERR_HIP;
    }
    return LIBRA_OK;
}
}  // namespace

extern "C" int libra_spmm(const libra_plan_t *P, const void *B, int32_t N, int64_t ldb, float *C, int64_t ldc, void *stream) {
    if (!P || !B || !C) return LIBRA_ERR_NULL;
    return spmm_call(P, B, N, ldb, C, ldc, nullptr, 0, stream);
}

extern "C" int libra_spmm_rounded(const libra_plan_t *P, const void *B, int32_t N, int64_t ldb, void *R, int64_t ldr, float *scratch, int64_t lds, void *stream) {
    if (!P || !B || !R) return LIBRA_ERR_NULL;
    if (!scratch && (P->spmm.n.zero_rows || P->o.two_kernels)) return LIBRA_ERR_NULL;
    if (P->vdt == LIBRA_F32) return LIBRA_ERR_DTYPE;
    if (ldr < N) return LIBRA_ERR_SHAPE;
    if (ldr % 8) return LIBRA_ERR_UNSUPPORTED;
    if ((uintptr_t)R & 15) return LIBRA_ERR_BUFFER;
    return spmm_call(P, B, N, ldb, scratch, scratch ? lds : N, R, ldr, stream);
}

namespace {
int sddmm_call(const libra_plan_t *P, const void *X, const void *Y, int32_t K, void *out, void *stream, int pattern_only, int rounded);
}
extern "C" int libra_sddmm(const libra_plan_t *P, const void *X, const void *Y, int32_t K, float *out, void *stream) {
    return sddmm_call(P, X, Y, K, out, stream, 0, 0);
}
extern "C" int libra_sddmm_pattern(const libra_plan_t *P, const void *X, const void *Y, int32_t K, float *out, void *stream) {
    return sddmm_call(P, X, Y, K, out, stream, 1, 0);
}
extern "C" int libra_sddmm_pattern_rounded(const libra_plan_t *P, const void *X, const void *Y, int32_t K, void *out, void *stream) {
    if (P && P->vdt == LIBRA_F32) return LIBRA_ERR_DTYPE;
    return sddmm_call(P, X, Y, K, out, stream, 1, 1);
}
namespace {
int sddmm_call(const libra_plan_t *P, const void *X, const void *Y, int32_t K, void *out, void *stream, int pattern_only, int rounded) {
    if (!P || !X || !Y) return LIBRA_ERR_NULL;
    if (!out && P->nnz > 0) return LIBRA_ERR_NULL;           // a matrix without nonzeros has no output
    if (!P->o.build_sddmm) return LIBRA_ERR_NOT_BUILT;
    if (!P->dev_base) return LIBRA_ERR_NOT_UPLOADED;
    if (P->o.W != W || P->o.KB != KB) return LIBRA_ERR_UNSUPPORTED;
    if (K <= 0) return LIBRA_ERR_SHAPE;
    if (K != 32 && K != 64 && K != 128) return LIBRA_ERR_UNSUPPORTED;
    if (((uintptr_t)X & 15) || ((uintptr_t)Y & 15) || ((uintptr_t)out & (rounded ? 1 : 3))) return LIBRA_ERR_BUFFER;
    hipStream_t s = (hipStream_t)stream;
    const SubPlan &sp = P->sddmm;
    SddmmArgs a{sp.dev.tasks, sp.dev.blk_cols, sp.dev.blk_bitmap, sp.dev.blk_valptr,
                reinterpret_cast<const uint2 *>(sp.dev.dense_pv), (int32_t)sp.n.dense,
                sp.dev.res_ent, sp.dev.res_base, sp.dev.res_row, sp.dev.res_perm, X, Y, (float *)out, P->M, 0, 0, pattern_only};
    if (sp.n.tasks == 0) return LIBRA_OK;
    a.tasks_per_die = a.tasks_left = (int32_t)((sp.n.tasks + LIBRA_XCDS - 1) / LIBRA_XCDS);
    constexpr int32_t most = LAUNCH_WAVES / LIBRA_XCDS;      // rounds of a launch: whole workgroups
    auto launch = [&](auto wpb, auto with_blocks) {
        constexpr int WPB = decltype(wpb)::value;
        constexpr bool DENSE = decltype(with_blocks)::value;
        const dim3 grid((unsigned)((std::min(a.tasks_left, most) + WPB - 1) / WPB * LIBRA_XCDS)), block(WAVE * WPB);
        auto width = [&](auto tag, auto round) {
            typedef decltype(tag) T;
            constexpr bool ROUNDED = decltype(round)::value;
            switch (K) {
            case 32: hipLaunchKernelGGL((sddmm_task_kernel<T, 32, WPB, DENSE, ROUNDED>), grid, block, 0, s, a); break;
            case 64: hipLaunchKernelGGL((sddmm_task_kernel<T, 64, WPB, DENSE, ROUNDED>), grid, block, 0, s, a); break;
            case 128: hipLaunchKernelGGL((sddmm_task_kernel<T, 128, WPB, DENSE, ROUNDED>), grid, block, 0, s, a); break;
            }
        };
        if (P->vdt == LIBRA_F32) width(float{}, std::false_type{});
        else if (P->vdt == LIBRA_F16) rounded ? width(half_t{}, std::true_type{}) : width(half_t{}, std::false_type{});
        else rounded ? width(bf16_t{}, std::true_type{}) : width(bf16_t{}, std::false_type{});
    };
    auto shape = [&](auto with_blocks) {
        if (P->o.xcd_order == 1) launch(std::integral_constant<int, 4>{}, with_blocks);
        else launch(std::integral_constant<int, 1>{}, with_blocks);
    };
    for (; a.tasks_left > 0; a.tasks += most, a.tasks_left -= most) {
        if (sp.n_window_tasks > 0) shape(std::true_type{});
        else shape(std::false_type{});
        if (hipGetLastError() != hipSuccess) return LIBRA_ERR_HIP;
    }
    return LIBRA_OK;
}
}  // namespace

extern "C" int libra_edge_softmax(const libra_plan_t *P, const float *scores, float scale, void *vals_out, int out_dtype, void *stream) {
    if (!P) return LIBRA_ERR_NULL;
    if ((!scores || !vals_out) && P->nnz > 0) return LIBRA_ERR_NULL;
    if (out_dtype != LIBRA_F16 && out_dtype != LIBRA_BF16 && out_dtype != LIBRA_F32) return LIBRA_ERR_DTYPE;
    if (!P->dev_base) return LIBRA_ERR_NOT_UPLOADED;
    hipStream_t s = (hipStream_t)stream;
    if (P->nnz == 0) return LIBRA_OK;
    const SoftmaxRows r = softmax_rows(P);
    const unsigned blocks = (unsigned)r.nlong + r.medium_blocks + r.short_blocks;
    auto run = [&](auto tag) {
        typedef decltype(tag) TO;
        hipLaunchKernelGGL((edge_softmax_kernel<TO>), dim3(blocks), dim3(256), 0, s, r, scores, scale, reinterpret_cast<TO *>(vals_out));
    };
    if (out_dtype == LIBRA_F16) run(half_t{});
    else if (out_dtype == LIBRA_BF16) run(bf16_t{});
    else run(float{});
    return hip_rc(hipGetLastError());
}

namespace {
// `same`: dalpha has alpha's type, otherwise fp32
int softmax_backward(const libra_plan_t *P, const void *alpha, int alpha_dtype, const void *dalpha, bool same, float scale, float *dscores, void *stream) {
    if (!P) return LIBRA_ERR_NULL;
    if ((!alpha || !dalpha || !dscores) && P->nnz > 0) return LIBRA_ERR_NULL;
    if (alpha_dtype != LIBRA_F16 && alpha_dtype != LIBRA_BF16 && alpha_dtype != LIBRA_F32) return LIBRA_ERR_DTYPE;
    if (!P->dev_base) return LIBRA_ERR_NOT_UPLOADED;
    hipStream_t s = (hipStream_t)stream;
    if (P->nnz == 0) return LIBRA_OK;
    const SoftmaxRows r = softmax_rows(P);
    const unsigned blocks = (unsigned)r.nlong + r.medium_blocks + r.short_blocks;
    auto run = [&](auto tag, auto dtag) {
        typedef decltype(tag) TA;
        typedef decltype(dtag) TD;
        hipLaunchKernelGGL((edge_softmax_bwd_kernel<TA, TD>), dim3(blocks), dim3(256), 0, s, r, reinterpret_cast<const TA *>(alpha),
                           reinterpret_cast<const TD *>(dalpha), scale, dscores);
    };
    if (alpha_dtype == LIBRA_F16) same ? run(half_t{}, half_t{}) : run(half_t{}, float{});
    else if (alpha_dtype == LIBRA_BF16) same ? run(bf16_t{}, bf16_t{}) : run(bf16_t{}, float{});
    else run(float{}, float{});
    return hip_rc(hipGetLastError());
}
}  // namespace
extern "C" int libra_edge_softmax_backward(const libra_plan_t *P, const void *alpha, int alpha_dtype, const float *dalpha, float scale,
                                           float *dscores, void *stream) {
    return softmax_backward(P, alpha, alpha_dtype, dalpha, false, scale, dscores, stream);
}
extern "C" int libra_edge_softmax_backward_rounded(const libra_plan_t *P, const void *alpha, const void *dalpha, int dtype, float scale,
                                                   float *dscores, void *stream) {
    return softmax_backward(P, alpha, dtype, dalpha, true, scale, dscores, stream);
}

extern "C" int libra_value_products(const void *vals, const float *factors, int64_t n, int dtype, void *out, void *stream) {
    if (n < 0) return LIBRA_ERR_SHAPE;
    if ((!vals || !factors || !out) && n > 0) return LIBRA_ERR_NULL;
    if (dtype != LIBRA_F16 && dtype != LIBRA_BF16) return LIBRA_ERR_DTYPE;
    if (((uintptr_t)vals & 1) || ((uintptr_t)factors & 3) || ((uintptr_t)out & 1)) return LIBRA_ERR_BUFFER;
    if (n == 0) return LIBRA_OK;
    const bool whole = !(((uintptr_t)vals | (uintptr_t)factors | (uintptr_t)out) & 15);
    const unsigned blocks = (unsigned)std::min<int64_t>(((whole ? n / 8 : n) + 255) / 256 + 1, 1 << 16);
    auto run = [&](auto tag) {
        typedef decltype(tag) T;
        hipLaunchKernelGGL((value_products_kernel<T>), dim3(blocks), dim3(256), 0, (hipStream_t)stream, reinterpret_cast<const T *>(vals), factors, n,
                           reinterpret_cast<T *>(out), whole);
    };
    if (dtype == LIBRA_F16) run(half_t{});
    else run(bf16_t{});
    return hip_rc(hipGetLastError());
}

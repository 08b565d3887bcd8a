// Device planner: the preprocessing of Section 4.5 (Algorithm 1) on the GPU.
//
// Builds the same plan as the host planner (plan.cpp), bit for bit, from a CSR matrix that is
// already in device memory.  The window-by-window loops of the host code become flat passes
// over arrays plus prefix sums:
//
//   1. the nonzeros of every window are sorted by (column, row), a tile of them at a time in LDS, which
//      puts the nonzeros of each column vector next to each other (the "census"); a vector is named by
//      the place of its first nonzero.  The vectors of each NNZ are counted per window;
//   2. per window, from those counts: how many vectors reach the SpMM threshold, how many fill padding,
//      how many SDDMM blocks reach the block threshold (their NNZ never increases along the order
//      (NNZ descending, column ascending), so a binary search finds the cut); prefix sums give block offsets;
//   3. the vectors in dense blocks go to their slots (the order is that of the SDDMM blocks and of the vectors
//      that fill the padding of the last SpMM block), blocks build bitmaps by ballots, packed values go
//      to the position given by the popcount of the bits below theirs;
//   4. nonzeros outside the dense vectors are numbered in CSR order by prefix sums; per window the
//      load-balancing rule of Section 4.3 emits the task records.
//
// Radix sorts and prefix sums are rocPRIM device primitives; everything else is written here.
// The arrays are produced in the host planner's format in the caller's workspace, copied to the
// plan's host vectors if a host copy is wanted; large task tables are ordered here, small ones
// by the host planner's tail.
#include <hip/hip_runtime.h>

#include <mutex>

#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>

#include <rocprim/rocprim.hpp>

#include "plan_internal.h"

using namespace libra;

namespace {

constexpr int W = 16, KB = 16;
typedef unsigned long long u64;

// Matrices of fewer rows have rowptr checked and the rows of the edge softmax listed on the host; here the launches and the extra
// wait cost some 80 us.  A plan of 8 nonzeros per row, host / here: 2^14 rows 585 / 665 us, 2^16 745 / 780, 98,304 813 / 820, 2^17
// level; 2^20 rows (plan and one step of the GAT graph) 13.15 / 12.05 ms.
constexpr int64_t DEVICE_ROWS_MIN = 1 << 17;

// Tables of fewer tasks are ordered on the host: there a task costs 40 - 70 ns (copies both ways, radix sorts of 40-byte records,
// merging), here the launches and waits cost 0.2 ms and a task 1 ns.  GAT graph (1.05 M tasks in both tables): 71 -> 1.5 ms,
// the whole plan 86.7 -> 24.1 ms; 8,000 tasks without segments: 0.32 ms on the host, 0.21 here.
constexpr int64_t DEVICE_ORDER_MIN = 8192;

enum Counter { C_NV = 0, C_NNZ1, C_SHORT, C_LONG, C_SPLIT, C_DV_A, C_PAD_A, C_DV_D, C_PAD_D, C_ERR, C_TOGETHER, C_APART, C_DNNZ_D, C_SEGMENTS, C_WIDE, C_COUNT };

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Bump allocator over the workspace (base == nullptr: size pass).
struct Arena {
    char *base;
    size_t off = 0;
    template <class T> T *take(size_t n) {
        off = align256(off);
        T *p = base ? reinterpret_cast<T *>(base + off) : nullptr;
        off += n * sizeof(T) + 64;
        return p;
    }
};

struct Sizes {
    int64_t M, n;
    int64_t nw, nbmax, tasks_a_max, tasks_d_max, segs_d_max;
};

Sizes make_sizes(int64_t M, int64_t n, const Resolved &o) {
    Sizes z;
    z.M = M; z.n = n;
    z.nw = (M + W - 1) / W;
    z.nbmax = n / KB + z.nw + 1;
    z.tasks_a_max = z.nbmax / o.Ts + 2 * z.nw + 2 * (n / o.Cs) + 8;
    z.tasks_d_max = z.nbmax / o.sddmm_Ts + z.nw + 8;
    z.segs_d_max = n / o.sddmm_Cs + 2;
    return z;
}

struct SubOut {      // one sub-plan in the host planner's format
    int32_t *slotvec, *blk_cols, *blknnz, *blk_valptr, *blkmask, *blkncols, *dense_perm;
    u64 *bitmap;
    uint8_t *dense_val, *res_val;
    int32_t *rescan, *res_perm, *res_row, *res_col;
    int32_t *nb, *ndv, *blkptr, *ntasks, *tbase;
    libra_task_t *tasks;
};

// Scratch of the task ordering: `items` entries per array (the longest region of either table).
struct OrderScratch {
    size_t items;
    uint32_t *key_in, *key_out;
    u64 *wide_in, *wide_out;
    int32_t *ord, *ord2, *flag, *scan, *first, *rank, *base, *queue;
    int32_t *meta;              // a few words that the host reads
    int32_t *pieces;            // MAX_PIECES x {queue, first slot, first queue item}
    int32_t *order_a, *order_d; // the ordered tables: task index, -1 for an empty task
};
constexpr int MAX_PIECES = 4096;

// Tiles of the census (see k_tile_sort).
constexpr int TILE_THREADS = 256, TILE_EACH = 7;             // an odd number of places per thread: their LDS accesses fall into different banks
constexpr int TILE_CAP = TILE_THREADS * TILE_EACH, TILE_STEP = TILE_CAP - W;
inline int tile_count(int64_t n) { return (int)((n + TILE_STEP - 1) / TILE_STEP); }
struct Tiles {
    int32_t *pos;       // per boundary: its place,
    int32_t *win;       // its window,
    int32_t *split;     // and per row of the window the first nonzero (CSR position) that lies behind it
    int32_t *tail;      // per tile: the vectors of each NNZ in the part of the next boundary's window that it holds
    int32_t *group;     // sums of `tail` over TAIL_GROUP tiles; nullptr: not formed
};
// A tile of a window that begins in an earlier one adds up the tails between.  Where a window has 4 groups of tiles (1.8 M nonzeros)
// it adds whole groups, or the time would be quadratic: plans of one window, tails / groups, 2^26 nonzeros 18.3 / 13.7 ms, 2^28 204 / 51, 2^29
// 822 / 102.  Below that the pass that forms the groups (9 us on the GAT graph) would be for nothing.
constexpr int TAIL_GROUP = 256, WIDE_WINDOW = 4 * TAIL_GROUP * TILE_STEP;

struct Layout {
    int32_t *win_ptr, *row_of, *rowbase, *scol, *spos;
    uint16_t *vmask;
    uint8_t *dense;
    u64 *ctr;
    Tiles tiles;
    int32_t *hist, *nzero, *zbase, *nres, *resptr, *zero_rows, *task_col, *seg_col;
    SubOut a, d;
    OrderScratch o;
    int32_t *sizes, *medium_rows, *long_rows;
    uint32_t *long_lens;
    void *tmp;
    char *stage;
    size_t tmp_bytes;
    size_t total;
};

struct RowsOfLength {                   // more than `above` and at most `most` nonzeros
    const int32_t *rowptr;
    int above, most;
    __device__ bool operator()(int32_t i) const { const int n = rowptr[i + 1] - rowptr[i]; return n > above && n <= most; }
};
struct NotDense {                       // of a nonzero's bits in `dense` (1: in a block of the SpMM sub-plan, 2: of the SDDMM one)
    unsigned bit;
    __host__ __device__ int32_t operator()(uint8_t f) const { return f & bit ? 0 : 1; }
};
size_t order_items(const Sizes &z) { return (size_t)std::max(z.tasks_a_max, std::max(z.tasks_d_max, z.segs_d_max)); }
int64_t order_slots(int64_t tasks) { return 2 * tasks + 64; }      // the die-aware orders add empty tasks

// Stable sorts of task keys.  By default rocPRIM merge-sorts up to 2^20 items, two launches for each doubling from 1,024 on; from
// SORT_BY_DIGITS items on the passes over 8-bit digits are fewer launches (GAT graph, three sorts of some 500,000 items: 0.75 ms, now 0.45).
constexpr size_t SORT_BY_DIGITS = 1 << 17;
template <bool DESC, class K, class In>
hipError_t sort_pairs(void *tmp, size_t &bytes, K *key_in, K *key_out, In in, int32_t *out, size_t n, unsigned bits, hipStream_t s) {
    typedef rocprim::radix_sort_config<rocprim::default_config, rocprim::default_config, rocprim::default_config, 0> ByDigits;
    auto run = [&](auto config) {
        typedef decltype(config) Config;
        if constexpr (DESC) return rocprim::radix_sort_pairs_desc<Config>(tmp, bytes, key_in, key_out, in, out, n, 0u, bits, s);
        else return rocprim::radix_sort_pairs<Config>(tmp, bytes, key_in, key_out, in, out, n, 0u, bits, s);
    };
    if (tmp) return n >= SORT_BY_DIGITS ? run(ByDigits{}) : run(rocprim::default_config{});
    size_t most = 0;                        // the size query: of either
    if (hipError_t e = run(ByDigits{})) return e;
    most = bytes;
    bytes = 0;
    if (hipError_t e = run(rocprim::default_config{})) return e;
    bytes = std::max(bytes, most);
    return hipSuccess;
}

size_t rocprim_temp_bytes(const Sizes &z) {
    size_t best = 0, sz = 0;
    (void)rocprim::exclusive_scan(nullptr, sz, (int32_t *)nullptr, (int32_t *)nullptr, (int32_t)0, (size_t)(z.n + z.nw + 2),
                            rocprim::plus<int32_t>());
    best = std::max(best, sz);
    const size_t m = std::max(order_items(z) + 16, (size_t)z.n / LIBRA_SOFTMAX_LONG_ROW + 1);
    sz = 0;
    (void)rocprim::exclusive_scan(nullptr, sz, rocprim::make_transform_iterator((const uint8_t *)nullptr, NotDense{1}), (int32_t *)nullptr, (int32_t)0, (size_t)(z.n + 1),
                            rocprim::plus<int32_t>());
    best = std::max(best, sz);
    sz = 0;
    (void)sort_pairs<false>(nullptr, sz, (uint32_t *)nullptr, (uint32_t *)nullptr, (const int32_t *)nullptr, (int32_t *)nullptr, m, 32, nullptr);
    best = std::max(best, sz);
    sz = 0;
    (void)sort_pairs<true>(nullptr, sz, (u64 *)nullptr, (u64 *)nullptr, rocprim::counting_iterator<int32_t>(0), (int32_t *)nullptr, m, 64, nullptr);
    best = std::max(best, sz);
    sz = 0;
    (void)sort_pairs<true>(nullptr, sz, (uint32_t *)nullptr, (uint32_t *)nullptr, rocprim::counting_iterator<int32_t>(0), (int32_t *)nullptr, m, 32, nullptr);
    best = std::max(best, sz);
    sz = 0;
    (void)rocprim::inclusive_scan(nullptr, sz, (u64 *)nullptr, (u64 *)nullptr, m, rocprim::maximum<u64>());
    best = std::max(best, sz);
    sz = 0;
    (void)rocprim::exclusive_scan(nullptr, sz, (int32_t *)nullptr, (int32_t *)nullptr, (int32_t)0, m, rocprim::plus<int32_t>());
    best = std::max(best, sz);
    sz = 0;
    (void)rocprim::exclusive_scan(nullptr, sz, (u64 *)nullptr, (u64 *)nullptr, (u64)0, m, rocprim::plus<u64>());
    best = std::max(best, sz);
    sz = 0;
    (void)rocprim::select(nullptr, sz, rocprim::counting_iterator<int32_t>(0), (int32_t *)nullptr, (int32_t *)nullptr, (size_t)z.M, RowsOfLength{nullptr, 0, 0});
    best = std::max(best, sz);
    return best + 4096;
}

// What goes to the host together: the counters, and tables that are ordered there with the first values of their blocks.
size_t stage_bytes(const Sizes &z) {
    return align256(C_COUNT * sizeof(u64)) + (size_t)DEVICE_ORDER_MIN * (sizeof(libra_task_t) + 2 * sizeof(int32_t)) + 2 * ((size_t)z.nbmax + 1) * sizeof(int32_t) + 8 * 256;
}

Layout make_layout(const Sizes &z, int vsize, void *base) {
    Layout L{};
    Arena A{(char *)base};
    const size_t n = (size_t)z.n, nw = (size_t)z.nw, nb = (size_t)z.nbmax;
    L.ctr = A.take<u64>(C_COUNT);
    L.hist = A.take<int32_t>(nw * W);       // right behind the counters: cleared together
    L.sizes = A.take<int32_t>(64);
    L.medium_rows = A.take<int32_t>((size_t)z.M);
    L.long_rows = A.take<int32_t>(n / LIBRA_SOFTMAX_LONG_ROW + 1);
    L.long_lens = A.take<uint32_t>(3 * (n / LIBRA_SOFTMAX_LONG_ROW + 1));        // lengths, sorted lengths, sorted rows
    L.win_ptr = A.take<int32_t>(nw + 1);
    const size_t boundaries = (size_t)tile_count(z.n) + 1;
    L.tiles.pos = A.take<int32_t>(boundaries);
    L.tiles.win = A.take<int32_t>(boundaries);
    L.tiles.split = A.take<int32_t>(boundaries * W);
    L.tiles.tail = A.take<int32_t>(boundaries * W);
    L.tiles.group = A.take<int32_t>((boundaries / TAIL_GROUP + 1) * W);
    L.scol = A.take<int32_t>(n);
    L.spos = A.take<int32_t>(n);
    L.vmask = A.take<uint16_t>(n);
    L.dense = A.take<uint8_t>(n + 1);
    L.row_of = A.take<int32_t>(n);
    L.rowbase = A.take<int32_t>((size_t)z.M + 1);
    L.nzero = A.take<int32_t>(nw + 1);
    L.zbase = A.take<int32_t>(nw + 1);
    L.nres = A.take<int32_t>(nw + 1);
    L.resptr = A.take<int32_t>(nw + 1);
    L.zero_rows = A.take<int32_t>((size_t)z.M);
    L.task_col = A.take<int32_t>((size_t)z.tasks_a_max);
    L.seg_col = A.take<int32_t>((size_t)z.segs_d_max);
    for (SubOut *s : {&L.a, &L.d}) {
        s->slotvec = A.take<int32_t>(nb * KB);
        s->blk_cols = A.take<int32_t>(nb * KB);
        s->bitmap = A.take<u64>(nb * 4);
        s->blknnz = A.take<int32_t>(nb + 1);
        s->blk_valptr = A.take<int32_t>(nb + 1);
        s->blkmask = A.take<int32_t>(nb);
        s->blkncols = A.take<int32_t>(nb);
        s->dense_perm = A.take<int32_t>(n);
        s->dense_val = A.take<uint8_t>(n * vsize);
        s->rescan = A.take<int32_t>(n + 1);
        s->res_perm = A.take<int32_t>(n);
        s->res_row = A.take<int32_t>(n);
        s->res_col = A.take<int32_t>(n);
        s->res_val = A.take<uint8_t>(n * vsize);
        s->nb = A.take<int32_t>(nw + 1);
        s->ndv = A.take<int32_t>(nw);
        s->blkptr = A.take<int32_t>(nw + 1);
        s->ntasks = A.take<int32_t>(nw + 1);
        s->tbase = A.take<int32_t>(nw + 1);
        s->tasks = A.take<libra_task_t>((size_t)(s == &L.a ? z.tasks_a_max : z.tasks_d_max));
    }
    {
        OrderScratch &o = L.o;
        o.items = order_items(z);
        const size_t m = o.items + 16;
        o.key_in = A.take<uint32_t>(m);
        o.key_out = A.take<uint32_t>(m);
        o.wide_in = A.take<u64>(m);
        o.wide_out = A.take<u64>(m);
        for (int32_t **q : {&o.ord, &o.ord2, &o.flag, &o.scan, &o.first, &o.rank, &o.base, &o.queue}) *q = A.take<int32_t>(m);
        o.meta = A.take<int32_t>(64);
        o.pieces = A.take<int32_t>(3 * MAX_PIECES);
        o.order_a = A.take<int32_t>((size_t)order_slots(z.tasks_a_max));
        o.order_d = A.take<int32_t>((size_t)order_slots(z.tasks_d_max + z.segs_d_max));
    }
    L.stage = A.take<char>(stage_bytes(z));
    L.tmp_bytes = rocprim_temp_bytes(z);
    L.tmp = A.take<uint8_t>(L.tmp_bytes);
    L.total = align256(A.off) + 256;
    return L;
}

// ------------------------------------------------------------------------------------------
// kernels
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_win_ptr(const int32_t *rowptr, int64_t M, int nw, int32_t *win_ptr, u64 *ctr) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t > nw) return;
    const int first = rowptr[min(M, t * W)];
    win_ptr[t] = first;
    if (rowptr[min(M, (t + 1) * W)] - first >= WIDE_WINDOW) ctr[C_WIDE] = 1;
}

__global__ __launch_bounds__(256) void k_check_rowptr(const int32_t *rowptr, int64_t M, int n, u64 *ctr) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool bad = i < M ? rowptr[i + 1] < rowptr[i] : i == M && (rowptr[0] != 0 || rowptr[M] != n);
    if (bad) atomicOr(&ctr[C_ERR], (u64)4);
}
__global__ __launch_bounds__(256) void k_row_lengths(const int32_t *rowptr, const int32_t *rows, int n, uint32_t *len) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) len[i] = rowptr[rows[i] + 1] - rowptr[rows[i]];
}

// The checks of the host planner on the columns, and every nonzero's row.  A workgroup takes ROWS_CHUNK nonzeros: the rows that
// begin among them mark their first nonzero in LDS (of rows that begin at one place the last one counts, the others are empty), and a
// nonzero's row is the largest mark up to it.  GAT graph: 217 us; a search through rowptr per wave of 64 nonzeros 601.
constexpr int ROWS_EACH = 8, ROWS_CHUNK = 256 * ROWS_EACH;
// Rows that a chunk's nonzeros may span for it: the workgroup walks them all, 0.2 us for each 256.  From here on, where nearly all are empty, a
// search per nonzero.  Whole plans of 2^26 rows, marks / searches: a row of one nonzero in every 16 (32,768 rows per chunk) 4.86 / 4.90 ms,
// in every 64 4.66 / 4.58, in every 1,024 7.8 / 4.3; 6,000 rows of 33 at both ends of 2^27 rows 232 / 5 ms.
constexpr int64_t ROWS_MARKED = 1 << 15;
__global__ __launch_bounds__(256) void k_rows(const int32_t *rowptr, const int32_t *col, int64_t M, int64_t Kc, int n, int32_t *row_of, u64 *ctr) {
    __shared__ __attribute__((aligned(16))) int32_t mark[ROWS_CHUNK];
    __shared__ int32_t wave_max[4];
    const int base = (int)(blockIdx.x * (unsigned)ROWS_CHUNK), end = (int)min((int64_t)base + ROWS_CHUNK, (int64_t)n), tid = threadIdx.x;
    for (int i = tid; i < ROWS_CHUNK; i += 256) mark[i] = -1;
    // first and last row, the same search in every lane: rowptr[lo] <= base < rowptr[lo + 1], and for end - 1
    int64_t lo = 0, hi = M;
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        if (rowptr[mid] <= base) lo = mid; else hi = mid;
    }
    int64_t step = 1;
    while (lo + step < M && rowptr[lo + step] <= end - 1) step <<= 1;
    int64_t last = lo;
    hi = min(M, lo + step);                 // rowptr[hi] > end - 1
    while (hi - last > 1) {
        const int64_t mid = (last + hi) >> 1;
        if (rowptr[mid] <= end - 1) last = mid; else hi = mid;
    }
    if (last - lo < ROWS_MARKED) {
        __syncthreads();
        if (tid == 0) mark[0] = (int32_t)lo;
        for (int64_t r = lo + 1 + tid; r <= last; r += 256) atomicMax(&mark[rowptr[r] - base], (int32_t)r);      // 0 < place < end - base
        __syncthreads();
        int row[ROWS_EACH], top = -1;
#pragma unroll
        for (int j = 0; j < ROWS_EACH; ++j) {
            top = max(top, mark[tid * ROWS_EACH + j]);
            row[j] = top;
        }
        int scan = top;
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) {
            const int x = __shfl_up(scan, m, 64);
            if (tid % 64 >= m) scan = max(scan, x);
        }
        if (tid % 64 == 63) wave_max[tid / 64] = scan;
        int before = __shfl_up(scan, 1, 64);
        if (tid % 64 == 0) before = -1;
        __syncthreads();
        for (int v = 0; v < tid / 64; ++v) before = max(before, wave_max[v]);
#pragma unroll
        for (int j = 0; j < ROWS_EACH; ++j) mark[tid * ROWS_EACH + j] = max(row[j], before);
        __syncthreads();
    } else {
        // between these nonzeros lie many empty rows: a search per nonzero, a thread's eight side by side
        int64_t from[ROWS_EACH];
#pragma unroll
        for (int j = 0; j < ROWS_EACH; ++j) from[j] = lo;
        for (int64_t half = (int64_t)1 << (63 - __clzll(last - lo)); half > 0; half >>= 1) {
#pragma unroll
            for (int j = 0; j < ROWS_EACH; ++j) {
                const int64_t r = from[j] + half;
                if (rowptr[min(r, last)] <= min(base + tid + j * 256, end - 1) && r <= last) from[j] = r;
            }
        }
#pragma unroll
        for (int j = 0; j < ROWS_EACH; ++j) mark[tid + j * 256] = (int32_t)from[j];
        __syncthreads();
    }
    unsigned bad = 0;
#pragma unroll
    for (int j = 0; j < ROWS_EACH; ++j) {
        const int i = tid + j * 256, p = base + i;
        if (p >= end) continue;
        const int r = mark[i], c = col[p];
        row_of[p] = r;
        if (c < 0 || c >= Kc) bad |= 1u;
        else if (p > 0 && col[p - 1] >= c && (i > 0 ? mark[i - 1] == r : rowptr[r] < p)) bad |= 2u;
    }
    if (bad) atomicOr(&ctr[C_ERR], (u64)bad);
}

// 16 lanes per boundary, one per row: the largest column with at most `target` of the window's nonzeros before it, by bisection;
// every lane keeps the part of its row between the columns that bound it.
__global__ __launch_bounds__(256) void k_tile_splits(const int32_t *rowptr, const int32_t *col, const int32_t *win_ptr, int64_t M, int64_t Kc, int n, int nw, int tiles, Tiles T) {
    const int k = (int)((blockIdx.x * blockDim.x + threadIdx.x) / W), r = threadIdx.x % W;
    if (k > tiles) return;
    if (k == tiles) {
        if (r == 0) { T.pos[k] = n; T.win[k] = nw; }
        T.split[(int64_t)k * W + r] = n;
        return;
    }
    const int at = k * TILE_STEP;           // < n
    int w = 0, end = nw;                    // win_ptr[w] <= at < win_ptr[end]
    while (end - w > 1) {
        const int mid = (w + end) >> 1;
        if (win_ptr[mid] <= at) w = mid; else end = mid;
    }
    const int64_t row = (int64_t)w * W + r;
    const int first = rowptr[min(row, M)], target = at - win_ptr[w];
    int a = first, b = rowptr[min(row + 1, M)];
    int64_t lo = 0, hi = Kc;                // nonzeros before column lo: at most target; before hi: more
    auto sum = [](int x) {
#pragma unroll
        for (int m = 1; m < W; m <<= 1) x += __shfl_xor(x, m, W);
        return x;
    };
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        int x = a, y = b;
        while (x < y) {
            const int z = x + ((y - x) >> 1);            // x + y may pass 2^31
            if ((int64_t)col[z] < mid) x = z + 1; else y = z;
        }
        const int before = sum(x - first);
        if (before <= target) { lo = mid; a = x; } else { hi = mid; b = x; }
        if (before == target) break;
    }
    const int before = sum(a - first);
    if (r == 0) { T.pos[k] = at - target + before; T.win[k] = w; }
    T.split[(int64_t)k * W + r] = a;
}

// The lanes of a wave that are `valid` and have the same 4-bit `cls` as `mine`.
struct ClassPlanes {
    u64 plane[4], valid;
    __device__ ClassPlanes(int cls, bool ok) {
        valid = __ballot(ok);
#pragma unroll
        for (int k = 0; k < 4; ++k) plane[k] = __ballot(cls >> k & 1);
    }
    __device__ u64 same(int cls) const {
        u64 m = valid;
#pragma unroll
        for (int k = 0; k < 4; ++k) m &= cls >> k & 1 ? plane[k] : ~plane[k];
        return m;
    }
};

// A workgroup per tile.  The nonzeros of equal row number in their windows form a list that is sorted by (window, column): the tile is 16
// such lists, merged in four rounds of pairs; in a round a thread finds where its places begin in the two lists by bisection and
// merges from there.  Bound by the vector ALUs and LDS.  GAT graph (59.7 M nonzeros), rows, boundaries and sort: 0.22 + 0.15 + 0.64 ms (0.76
// with the masks and counts); two merges of four lists with a search through the other lists per nonzero took 3.06 ms, one pass over all
// 16 rows 4.1, keys and a segmented radix sort 7.4.
__global__ __launch_bounds__(TILE_THREADS) void k_tile_sort(const int32_t *rowptr, const int32_t *col, const int32_t *win_ptr, const int32_t *row_of, int64_t M, Tiles T,
                                                            const u64 *ctr, int32_t *scol, int32_t *spos, uint16_t *vmask, int32_t *hist) {
    __shared__ u64 key[TILE_CAP];
    __shared__ int32_t pos[TILE_CAP];
    __shared__ int32_t run_first[2 * W + 1], run_at[2 * W + 2];
    __shared__ int32_t list[W + 1], wave_count[TILE_THREADS / 64][W], tail[W];
    if (ctr[C_ERR]) return;                 // unsorted rows: nothing below would hold (the host has the error before it reads on)
    const int k = blockIdx.x, tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
    const int w0 = T.win[k], w1 = T.win[k + 1], out = T.pos[k], count = min(T.pos[k + 1] - out, TILE_CAP);
    if (tid < 64) {
        // up to 33 stretches of CSR positions: rows of the first window, whole windows, rows of the last window
        int from = 0, to = 0;
        if (tid < W) {
            from = T.split[(int64_t)k * W + tid];
            to = w0 == w1 ? T.split[(int64_t)(k + 1) * W + tid] : rowptr[min((int64_t)w0 * W + tid + 1, M)];
        } else if (tid == W && w1 > w0) {
            from = win_ptr[w0 + 1];
            to = win_ptr[w1];
        } else if (tid > W && tid <= 2 * W && w1 > w0) {
            from = rowptr[min((int64_t)w1 * W + (tid - W - 1), M)];
            to = T.split[(int64_t)(k + 1) * W + (tid - W - 1)];
        }
        int sum = to - from;
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) {
            const int x = __shfl_up(sum, m, 64);
            if (lane >= m) sum += x;
        }
        if (tid <= 2 * W) {
            run_first[tid] = from;
            run_at[tid + 1] = sum;
        }
        if (tid == 0) run_at[0] = 0;
    }
    __syncthreads();
    // a wave takes 448 neighbouring nonzeros, and counts those of equal row number before each
    u64 kk[TILE_EACH];
    int pp[TILE_EACH], rank[TILE_EACH], seen = 0;            // seen: lane c < 16, of row number c
#pragma unroll
    for (int j = 0; j < TILE_EACH; ++j) {
        const int i = wave * (64 * TILE_EACH) + j * 64 + lane;
        const bool ok = i < count;
        int lo = 0, hi = 2 * W + 1;         // run_at[lo] <= i < run_at[hi]
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (run_at[mid] <= i) lo = mid; else hi = mid;
        }
        const int p = ok ? run_first[lo] + (i - run_at[lo]) : run_first[0];
        pp[j] = p;
    }
    {
        int rows[TILE_EACH], cols[TILE_EACH];
#pragma unroll
        for (int j = 0; j < TILE_EACH; ++j) {
            const bool ok = wave * (64 * TILE_EACH) + j * 64 + lane < count;
            rows[j] = ok ? row_of[pp[j]] : 0;
            cols[j] = ok ? col[pp[j]] : 0;
        }
#pragma unroll
        for (int j = 0; j < TILE_EACH; ++j) {
            const bool ok = wave * (64 * TILE_EACH) + j * 64 + lane < count;
            const int cls = rows[j] % W;
            kk[j] = (u64)(rows[j] / W - w0) << 36 | (u64)(uint32_t)cols[j] << 4 | (u64)cls;
            const ClassPlanes planes(cls, ok);
            rank[j] = __popcll(planes.same(cls) & ((1ull << lane) - 1ull)) + __shfl(seen, cls, 64);
            seen += lane < W ? __popcll(planes.same(lane)) : 0;
        }
    }
    if (lane < W) wave_count[wave][lane] = seen;
    __syncthreads();
    if (tid < 64) {
        int total = 0;
        if (tid < W)
            for (int v = 0; v < TILE_THREADS / 64; ++v) {
                const int x = wave_count[v][tid];
                wave_count[v][tid] = total;
                total += x;
            }
        int sum = total;
#pragma unroll
        for (int m = 1; m < W; m <<= 1) {
            const int x = __shfl_up(sum, m, 64);
            if (lane >= m) sum += x;
        }
        if (tid < W) list[tid + 1] = sum;
        if (tid == 0) list[0] = 0;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < TILE_EACH; ++j) {
        if (wave * (64 * TILE_EACH) + j * 64 + lane < count) {
            const int cls = (int)(kk[j] & 15), to = list[cls] + wave_count[wave][cls] + rank[j];
            key[to] = kk[j];
            pos[to] = pp[j];
        }
    }
    __syncthreads();
    const int o0 = tid * TILE_EACH;
#pragma unroll 1
    for (int width = 1; width < W; width <<= 1) {
        int g = 0;                          // the pair of lists that this thread's first place lies in
        while (g + 2 * width < W && list[g + 2 * width] <= o0) g += 2 * width;
        int s = list[g], m = list[g + width], e = list[g + 2 * width];
        int ia = s, ib = m;
        if (o0 < count) {
            const int d = o0 - s;
            int lo = max(0, d - (e - m)), hi = min(d, m - s);
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (key[s + mid] < key[m + d - 1 - mid]) lo = mid + 1; else hi = mid;
            }
            ia = s + lo;
            ib = m + d - lo;
        }
        constexpr u64 NONE = ~0ull;
        u64 ka = o0 < count && ia < m ? key[ia] : NONE, kb = o0 < count && ib < e ? key[ib] : NONE;
#pragma unroll
        for (int j = 0; j < TILE_EACH; ++j) {
            if (o0 + j < count) {
                if (o0 + j == e) {          // on to the next pair that holds something
                    do {
                        g += 2 * width;
                        s = list[g]; m = list[g + width]; e = list[g + 2 * width];
                    } while (e == o0 + j);
                    ia = s; ib = m;
                    ka = ia < m ? key[ia] : NONE;
                    kb = ib < e ? key[ib] : NONE;
                }
                const bool first = ka < kb;
                kk[j] = first ? ka : kb;
                pp[j] = pos[first ? ia : ib];
                if (first) {
                    ++ia;
                    ka = ia < m ? key[ia] : NONE;
                } else {
                    ++ib;
                    kb = ib < e ? key[ib] : NONE;
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < TILE_EACH; ++j)
            if (o0 + j < count) {
                key[o0 + j] = kk[j];
                pos[o0 + j] = pp[j];
            }
        __syncthreads();
    }
    // The places leave with what the rest of the planner asks of them: column, CSR position and, at the first place of a column vector,
    // the rows it holds.
    int cls[TILE_EACH], rel[TILE_EACH];     // of a vector's first place: NNZ - 1 and window; otherwise -1
#pragma unroll
    for (int j = 0; j < TILE_EACH; ++j) {
        const int i = tid + j * TILE_THREADS;
        cls[j] = -1;
        rel[j] = 0;
        if (i >= count) continue;
        const u64 mine = key[i], vec = mine >> 4;
        unsigned rows = 0;
        if (i == 0 || key[i - 1] >> 4 != vec) {
            rows = 1u << (unsigned)(mine & 15);
            for (int q = i + 1; q < count && key[q] >> 4 == vec; ++q) rows |= 1u << (unsigned)(key[q] & 15);
            cls[j] = __popc(rows) - 1;
            rel[j] = (int)(mine >> 36);
        }
        scol[out + i] = (int32_t)(uint32_t)vec;
        spos[out + i] = pos[i];
        vmask[out + i] = (uint16_t)rows;
    }
    __syncthreads();
    // vectors of each NNZ per window, in LDS (over `pos`) if the tile's windows are few enough, which they are unless most are nearly empty
    const int last = w1 - w0, windows = last + 1;
    const bool here = windows <= TILE_CAP / W;
    if (here)
        for (int i = tid; i < windows * W; i += TILE_THREADS) pos[i] = 0;
    if (tid < W) tail[tid] = 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < TILE_EACH; ++j) {
        // the vectors of one nonzero in the wave's first window, most of all, are added as one
        const int rel0 = __builtin_amdgcn_readfirstlane(rel[j]);
        const bool single = cls[j] == 0 && rel[j] == rel0;
        const u64 singles = __ballot(single);
        const int add = single ? (lane == __ffsll(singles) - 1 ? __popcll(singles) : 0) : 1;
        if (cls[j] < 0 || add == 0) continue;
        if (here) {
            atomicAdd(&pos[rel[j] * W + cls[j]], add);
        } else {
            atomicAdd(&hist[((int64_t)w0 + rel[j]) * W + cls[j]], add);
            if (rel[j] == last) atomicAdd(&tail[cls[j]], add);
        }
    }
    __syncthreads();
    if (here) {
        for (int i = tid; i < windows * W; i += TILE_THREADS) {
            const int v = pos[i], w = i / W;
            if (v == 0) continue;
            if (w > 0 && w < last) hist[(int64_t)w0 * W + i] = v;          // the whole window is in this tile
            else atomicAdd(&hist[(int64_t)w0 * W + i], v);
        }
        if (tid < W) tail[tid] = pos[last * W + tid];
        __syncthreads();
    }
    if (tid < W) T.tail[(int64_t)k * W + tid] = tail[tid];
}

// Sums of the tiles' tails over groups of tiles; a group per workgroup.
__global__ __launch_bounds__(256) void k_tail_groups(Tiles T, int tiles) {
    __shared__ int32_t sum[W];
    const int c = threadIdx.x % W, k0 = blockIdx.x * TAIL_GROUP, k1 = min(k0 + TAIL_GROUP, tiles);
    if (threadIdx.x < W) sum[c] = 0;
    __syncthreads();
    int x = 0;
    for (int k = k0 + threadIdx.x / W; k < k1; k += 256 / W) x += T.tail[(int64_t)k * W + c];
    if (x) atomicAdd(&sum[c], x);
    __syncthreads();
    if (threadIdx.x < W) T.group[(int64_t)blockIdx.x * W + c] = sum[c];
}

// The sampled column-sharing statistic: how many distinct columns the windows of each sampled group of LIBRA_LOCALITY_WINDOWS windows
// have together (a vector counts unless an earlier window of the group has its column) and one by one.  The places of all sampled
// groups are one list, dealt to the threads: a hub's group has more of them than all others together.  GAT graph: 223 us, with 64
// workgroups for each group 493.
constexpr int SHARE_SAMPLES = 256;
__global__ __launch_bounds__(SHARE_SAMPLES) void k_share(const int32_t *win_ptr, const int32_t *scol, const uint16_t *vmask, int nw, int64_t ngroups, int nsample, u64 *ctr) {
    __shared__ int64_t at[SHARE_SAMPLES + 1], wave_sum[SHARE_SAMPLES / 64];
    __shared__ int32_t first_window[SHARE_SAMPLES];
    __shared__ int together, apart;
    const int tid = threadIdx.x;
    {
        const int w0 = (int)(sampled_group(min(tid, nsample - 1), ngroups, nsample) * LIBRA_LOCALITY_WINDOWS);
        first_window[tid] = w0;
        int64_t sum = tid < nsample ? win_ptr[min(w0 + LIBRA_LOCALITY_WINDOWS, nw)] - win_ptr[w0] : 0;
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) {
            const int64_t x = __shfl_up(sum, m, 64);
            if (tid % 64 >= m) sum += x;
        }
        if (tid % 64 == 63) wave_sum[tid / 64] = sum;
        if (tid == 0) { together = apart = 0; at[0] = 0; }
        __syncthreads();
        for (int v = 0; v < tid / 64; ++v) sum += wave_sum[v];
        at[tid + 1] = sum;
        __syncthreads();
    }
    int mine = 0, all = 0;
    for (int64_t i = (int64_t)blockIdx.x * SHARE_SAMPLES + tid; i < at[SHARE_SAMPLES]; i += (int64_t)gridDim.x * SHARE_SAMPLES) {
        int lo = 0, hi = SHARE_SAMPLES;     // at[lo] <= i < at[hi]
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (at[mid] <= i) lo = mid; else hi = mid;
        }
        const int w0 = first_window[lo], w1 = min(w0 + LIBRA_LOCALITY_WINDOWS, nw), v = win_ptr[w0] + (int)(i - at[lo]);
        if (vmask[v] == 0) continue;
        ++all;
        const int c = scol[v];
        // first place with column >= c in each window before the vector's own, together: the searches are chains of loads
        constexpr int E = LIBRA_LOCALITY_WINDOWS - 1;
        int from[E], left[E], end[E];
        bool more = false;
#pragma unroll
        for (int u = 0; u < E; ++u) {
            const int w = min(w0 + u, w1 - 1);
            from[u] = win_ptr[w];
            end[u] = win_ptr[w + 1];
            left[u] = w0 + u < w1 && end[u] <= v ? end[u] - from[u] : 0;
            if (left[u] == 0) end[u] = from[u];
            more = more || left[u];
        }
        while (more) {
            int x[E];
#pragma unroll
            for (int u = 0; u < E; ++u) x[u] = scol[min(from[u] + (left[u] >> 1), v)];
            more = false;
#pragma unroll
            for (int u = 0; u < E; ++u) {
                const int half = left[u] >> 1;
                const bool before = left[u] > 0 && x[u] < c;
                from[u] = before ? from[u] + half + 1 : from[u];
                left[u] = before ? left[u] - half - 1 : half;
                more = more || left[u];
            }
        }
        bool seen = false;
#pragma unroll
        for (int u = 0; u < E; ++u) seen = seen || (from[u] < end[u] && scol[from[u]] == c);
        mine += seen ? 0 : 1;
    }
    if (mine) atomicAdd(&together, mine);
    if (all) atomicAdd(&apart, all);
    __syncthreads();
    if (tid == 0) {
        if (together) atomicAdd(&ctr[C_TOGETHER], (u64)together);
        if (apart) atomicAdd(&ctr[C_APART], (u64)apart);
    }
}

struct Rule {
    int mode, fill, tau_a, tau_d, Ts, Cs, short_len, build_a, build_d, Ts_d;
};

// Per window: dense vectors and blocks of both sub-plans (Section 4.2), from the numbers of its vectors of each NNZ.  hist then holds, for
// each NNZ, the vectors of more nonzeros: the place of the first one in sorted order.
__global__ __launch_bounds__(256) void k_window_counts(int32_t *hist, int nw, Rule R, int32_t *ndv_a, int32_t *nb_a, int32_t *ndv_d, int32_t *nb_d, u64 *ctr) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t == nw) { nb_a[nw] = 0; nb_d[nw] = 0; }
    if (t >= nw) return;
    int h[W], nvw = 0, ntau = 0;
#pragma unroll
    for (int q = 0; q < W; q += 4) {
        const int4 x = reinterpret_cast<const int4 *>(hist + (int64_t)t * W)[q / 4];
        h[q] = x.x; h[q + 1] = x.y; h[q + 2] = x.z; h[q + 3] = x.w;
    }
#pragma unroll
    for (int q = 0; q < W; ++q) {
        nvw += h[q];
        ntau += q + 1 >= R.tau_a ? h[q] : 0;
    }
    int ndv = 0, nb = 0;
    if (R.build_a) {
        int nprom = 0;
        if (R.fill && ntau > 0 && ntau % KB) nprom = min(KB - ntau % KB, nvw - ntau);
        ndv = ntau + nprom;
        nb = (ndv + KB - 1) / KB;
    }
    ndv_a[t] = ndv;
    nb_a[t] = nb;
    auto nonzeros = [&](int first) {        // of the first so many vectors of the order
        int sum = 0;
#pragma unroll
        for (int q = W - 1; q >= 0; --q) {
            const int take = min(first, h[q]);
            sum += take * (q + 1);
            first -= take;
        }
        return sum;
    };
    int nbd = 0;
    if (R.build_d && R.mode != LIBRA_MODE_SCALAR_ONLY) {
        const int nblk = (nvw + KB - 1) / KB;
        if (R.mode == LIBRA_MODE_DENSE_ONLY) {
            nbd = nblk;
        } else {
            // block NNZ never increases along the order: first block below the threshold by bisection
            int lo = 0, hi = nblk;          // blocks [0, lo) pass, blocks [hi, nblk) fail
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (nonzeros(min(nvw, mid * KB + KB)) - nonzeros(mid * KB) >= R.tau_d) lo = mid + 1; else hi = mid;
            }
            nbd = lo;
        }
    }
    const int ndvd = min(nvw, nbd * KB);
    ndv_d[t] = ndvd;
    nb_d[t] = nbd;
    int more = 0;
#pragma unroll
    for (int q = W - 4; q >= 0; q -= 4) {
        int4 x;
        x.w = more; more += h[q + 3];
        x.z = more; more += h[q + 2];
        x.y = more; more += h[q + 1];
        x.x = more; more += h[q];
        reinterpret_cast<int4 *>(hist + (int64_t)t * W)[q / 4] = x;
    }
    if (nvw) atomicAdd(&ctr[C_NV], (u64)nvw);
    if (h[0]) atomicAdd(&ctr[C_NNZ1], (u64)h[0]);
    if (ndv) { atomicAdd(&ctr[C_DV_A], (u64)ndv); }
    if (nb * KB - ndv) atomicAdd(&ctr[C_PAD_A], (u64)(nb * KB - ndv));
    if (ndvd) atomicAdd(&ctr[C_DV_D], (u64)ndvd);
    if (ndvd) atomicAdd(&ctr[C_DNNZ_D], (u64)nonzeros(ndvd));       // nonzeros in the window's dense SDDMM blocks
    if (nbd * KB - ndvd) atomicAdd(&ctr[C_PAD_D], (u64)(nbd * KB - ndvd));
}
// The whole-matrix utilisation rule: too small a dense share sends the whole SDDMM sub-plan to the scalar path.
__global__ __launch_bounds__(256) void k_share_rule(const u64 *ctr, int64_t nnz, int pct, int nw, int32_t *ndv_d, int32_t *nb_d) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nw || 100 * (int64_t)ctr[C_DNNZ_D] >= (int64_t)pct * nnz) return;
    ndv_d[t] = 0;
    nb_d[t] = 0;
}

// The vectors in dense blocks: their slots in the SpMM blocks (threshold vectors in column order, then the fillers in sorted order) and in
// the SDDMM blocks (sorted order), and which nonzeros they hold.  A workgroup per tile of the census, whose places are in column order:
// a vector's rank among the window's vectors of its NNZ is counted by ballots, over the part of the window in earlier tiles and waves
// from their totals.  (It replaces numbering the vectors, a stable sort of those with more than one nonzero, ranks, three scans and two
// scattering passes: 2.5 ms of the GAT graph's plan.  What the windows say is loaded for all seven chunks of a wave together: 610 -> 498 us.)
__global__ __launch_bounds__(TILE_THREADS) void k_dense_vectors(const int32_t *win_ptr, const int32_t *row_of, Tiles T, const int32_t *spos, const uint16_t *vmask, const int32_t *hist,
                                                                const int32_t *ndv_a, const int32_t *blkptr_a, const int32_t *ndv_d, const int32_t *blkptr_d, Rule R,
                                                                int32_t *slotvec_a, int32_t *slotvec_d, uint8_t *dense) {
    constexpr int WAVES = TILE_THREADS / 64;
    __shared__ int32_t carry[W], wave_tail[WAVES][W];
    __shared__ int wave_changed[WAVES];
    const int k = blockIdx.x, tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
    const int w0 = T.win[k], out = T.pos[k], count = T.pos[k + 1] - out;
    if (tid < W) carry[tid] = 0;
    __syncthreads();
    // the parts of the first window in earlier tiles: those before the boundaries inside it
    {
        const int c = tid % W, from = max(1, (int)(((int64_t)win_ptr[w0] + TILE_STEP - 1) / TILE_STEP)) - 1;           // tiles from .. k - 1
        int sum = 0, end = k;
        if (T.group) {
            const int g0 = (from + TAIL_GROUP - 1) / TAIL_GROUP, g1 = k / TAIL_GROUP;
            for (int g = g0 + tid / W; g < g1; g += TILE_THREADS / W) sum += T.group[(int64_t)g * W + c];
            if (g0 < g1) {
                for (int b = g1 * TAIL_GROUP + tid / W; b < k; b += TILE_THREADS / W) sum += T.tail[(int64_t)b * W + c];
                end = g0 * TAIL_GROUP;
            }
        }
        for (int b = from + tid / W; b < end; b += TILE_THREADS / W) sum += T.tail[(int64_t)b * W + c];
        if (sum) atomicAdd(&carry[c], sum);
    }
    int rows[TILE_EACH], win[TILE_EACH];
    u64 change[TILE_EACH];                  // the chunk's lanes that begin a window
    int run = 0;                            // lane c < 16: vectors of NNZ c + 1 since the last of them
    bool changed = false;
#pragma unroll
    for (int j = 0; j < TILE_EACH; ++j) {
        const int i = wave * (64 * TILE_EACH) + j * 64 + lane, e = out + min(i, count - 1);
        rows[j] = i < count ? vmask[e] : 0;
        win[j] = row_of[e] / W;             // a place's window is that of the nonzero there in CSR order
        change[j] = __ballot(i > 0 && i < count && row_of[e - (i > 0)] / W != win[j]);
    }
    // what the windows say, for all chunks together: nothing below waits for more than one load
    int da[TILE_EACH], dd[TILE_EACH], higher[TILE_EACH];     // vectors in dense blocks; vectors of more nonzeros than this one
#pragma unroll
    for (int j = 0; j < TILE_EACH; ++j) {
        da[j] = ndv_a[win[j]];
        dd[j] = ndv_d[win[j]];
        higher[j] = hist[(int64_t)win[j] * W + max((int)__popc(rows[j]) - 1, 0)];
    }
#pragma unroll
    for (int j = 0; j < TILE_EACH; ++j) {
        const ClassPlanes planes(__popc(rows[j]) - 1, rows[j] != 0);
        const u64 from = change[j] ? ~0ull << (63 - __clzll(change[j])) : ~0ull;
        run = (change[j] ? 0 : run) + __popcll(planes.same(lane) & from);
        changed = changed || change[j];
    }
    if (lane < W) wave_tail[wave][lane] = run;
    if (lane == 0) wave_changed[wave] = changed;
    __syncthreads();
    run = 0;
    {
        bool open = true;
        for (int v = wave - 1; v >= 0 && open; --v) {
            run += wave_tail[v][lane % W];
            open = !wave_changed[v];
        }
        if (open) run += carry[lane % W];
    }
    auto over_tau = [&](int x) {            // sum over the lanes c < 16 with c + 1 >= tau
        int sum = lane < W && lane + 1 >= R.tau_a ? x : 0;
#pragma unroll
        for (int m = 1; m < W; m <<= 1) sum += __shfl_xor(sum, m, 64);
        return __builtin_amdgcn_readfirstlane(sum);
    };
    int run_tau = over_tau(run), last_in = 0, slot_a[TILE_EACH], slot_d[TILE_EACH], bits[TILE_EACH];
#pragma unroll
    for (int j = 0; j < TILE_EACH; ++j) {
        const int nnz = __popc(rows[j]), cls = nnz - 1;
        const ClassPlanes planes(cls, nnz > 0);
        const u64 over = __ballot(nnz > 0 && nnz >= R.tau_a), below = (1ull << lane) - 1ull;
        const u64 begun = change[j] & (below << 1 | 1ull);                     // windows that begin at or before this lane
        const u64 from = begun ? ~0ull << (63 - __clzll(begun)) : ~0ull;
        const int carried = __shfl(run, cls & 15, 64);       // (by all lanes: a lane that has left the branch hands out nothing)
        const int rank = __popcll(planes.same(cls) & below & from) + (begun ? 0 : carried);
        const int rank_tau = __popcll(over & below & from) + (begun ? 0 : run_tau);
        const int place = higher[j] + rank;                          // in sorted order
        // of a vector's first place: 1, in a SpMM block; 2, in an SDDMM block
        const int in = nnz > 0 ? (place < da[j] ? 1 : 0) | (place < dd[j] ? 2 : 0) : 0;
        slot_a[j] = in & 1 ? (nnz >= R.tau_a ? rank_tau : place) : -1;
        slot_d[j] = in & 2 ? place : -1;
        // a place's bits are those of its vector's first place: in this chunk, or the last one of the chunk before
        const u64 heads = __ballot(nnz > 0), up_to = heads & (below << 1 | 1ull);
        const int mine = __shfl(in, up_to ? 63 - __clzll(up_to) : 0, 64);
        bits[j] = up_to ? mine : last_in;
        if (heads) last_in = __shfl(in, 63 - __clzll(heads), 64);
        const u64 all_from = change[j] ? ~0ull << (63 - __clzll(change[j])) : ~0ull;
        run = (change[j] ? 0 : run) + __popcll(planes.same(lane) & all_from);
        run_tau = (change[j] ? 0 : run_tau) + __popcll(over & all_from);
    }
    // (unsigned: near 2^31 nonzeros the places past the last tile's end are no int)
    const unsigned first = (unsigned)out + (unsigned)(wave * (64 * TILE_EACH) + lane), last = (unsigned)(out + count - 1), end = (unsigned)(out + min(count, (wave + 1) * 64 * TILE_EACH));
    int to_a[TILE_EACH], to_d[TILE_EACH], p[TILE_EACH];
#pragma unroll
    for (int j = 0; j < TILE_EACH; ++j) {
        const unsigned e = min(first + j * 64, last);
        to_a[j] = to_d[j] = p[j] = 0;
        if (slot_a[j] >= 0) to_a[j] = blkptr_a[win[j]];
        if (slot_d[j] >= 0) to_d[j] = blkptr_d[win[j]];
        if (bits[j]) p[j] = spos[e];
    }
#pragma unroll
    for (int j = 0; j < TILE_EACH; ++j) {
        const unsigned e = first + j * 64, in = (slot_a[j] >= 0 ? 1 : 0) | (slot_d[j] >= 0 ? 2 : 0);
        if (slot_a[j] >= 0) slotvec_a[(int64_t)to_a[j] * KB + slot_a[j]] = (int32_t)e;
        if (slot_d[j] >= 0) slotvec_d[(int64_t)to_d[j] * KB + slot_d[j]] = (int32_t)e;
        if (bits[j] && e < end) dense[p[j]] = (uint8_t)bits[j];
        // places of the next wave whose vector begins in this one
        if (in)
            for (unsigned q = end; q < e + __popc(rows[j]); ++q) dense[spos[q]] = (uint8_t)in;
    }
}

// 16 lanes per block: column ids, the bitmap (bit r*16+s) by ballots, NNZ, touched rows, real columns.
__global__ __launch_bounds__(256) void k_blocks(const int32_t *slotvec, const int32_t *scol, const uint16_t *vmask, int nb,
                                                int32_t *blk_cols, u64 *bitmap, int32_t *blknnz, int32_t *blkmask, int32_t *blkncols) {
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int b = (int)(gid >> 4), s = (int)(gid & 15);
    const int grp = (threadIdx.x & 63) >> 4;
    const bool live = b < nb;
    if (gid == 0) blknnz[nb] = 0;
    const int v = live ? slotvec[(int64_t)b * KB + s] : -1;
    const unsigned mask = v >= 0 ? vmask[v] : 0u;
    if (live) blk_cols[(int64_t)b * KB + s] = v >= 0 ? scol[v] : -1;
    u64 word = 0;           // lane s < 4 builds word s (rows 4s .. 4s+3)
    int nnz = 0;
    unsigned touched = 0;
    for (int r = 0; r < W; ++r) {
        const u64 bal = __ballot((mask >> r) & 1u);
        const u64 rb = (bal >> (16 * grp)) & 0xffffull;
        nnz += __popcll(rb);
        if (rb) touched |= 1u << r;
        if ((r >> 2) == s) word |= rb << (16 * (r & 3));
    }
    const u64 balc = __ballot(v >= 0);
    const int ncols = __popcll((balc >> (16 * grp)) & 0xffffull);
    if (live && s < 4) bitmap[(int64_t)b * 4 + s] = word;
    if (live && s == 0) {
        blknnz[b] = nnz;
        blkmask[b] = (int)touched;
        blkncols[b] = ncols;
    }
}

// 16 lanes per block: CSR position and value of every packed nonzero, at popcount(bits below its bit).
__global__ __launch_bounds__(256) void k_block_values(const int32_t *slotvec, const uint16_t *vmask, const u64 *bitmap,
                                                      const int32_t *blk_valptr, const int32_t *spos, const uint8_t *val, int vsize, int nb,
                                                      int32_t *dense_perm, uint8_t *dense_val) {
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int b = (int)(gid >> 4), s = (int)(gid & 15);
    if (b >= nb) return;
    const int v = slotvec[(int64_t)b * KB + s];
    if (v < 0) return;
    const unsigned mask = vmask[v];
    const u64 w0 = bitmap[(int64_t)b * 4], w1 = bitmap[(int64_t)b * 4 + 1], w2 = bitmap[(int64_t)b * 4 + 2], w3 = bitmap[(int64_t)b * 4 + 3];
    const int c0 = __popcll(w0), c1 = __popcll(w1), c2 = __popcll(w2);
    const int vbase = blk_valptr[b];
    int e = v;                              // a vector is named by its first place
    for (int r = 0; r < W; ++r) {
        if (!((mask >> r) & 1u)) continue;
        const int q = r >> 2;
        const u64 word = q == 0 ? w0 : q == 1 ? w1 : q == 2 ? w2 : w3;
        const int below = (q > 0 ? c0 : 0) + (q > 1 ? c1 : 0) + (q > 2 ? c2 : 0) + __popcll(word & ((1ull << ((r & 3) * 16 + s)) - 1ull));
        const int dst = vbase + below;
        const int p = spos[e];
        dense_perm[dst] = p;
        if (vsize == 2) reinterpret_cast<uint16_t *>(dense_val)[dst] = reinterpret_cast<const uint16_t *>(val)[p];
        else reinterpret_cast<uint32_t *>(dense_val)[dst] = reinterpret_cast<const uint32_t *>(val)[p];
        ++e;
    }
}

// The residual nonzeros of a sub-plan in CSR order.  scan = nullptr: all of the matrix.
struct Residual {
    const uint8_t *dense;
    const int32_t *scan;
    unsigned bit;
    __device__ int before(int p) const { return scan ? scan[p] : p; }
    __device__ bool has(int p) const { return !scan || !(dense[p] & bit); }
};

// The residual parts of a window's rows, a lane per row (16 neighbouring lanes per window).
struct RowPart {
    int before, len;            // residual nonzeros before the row, and in it
    unsigned valid, split, scalar;      // of the window: rows of the matrix, decomposed rows, others with residual nonzeros
};
__device__ inline int sum_over_rows(int x) {
#pragma unroll
    for (int m = 1; m < W; m <<= 1) x += __shfl_xor(x, m, W);
    return x;
}
__device__ inline unsigned rows_where(bool x) { return (unsigned)(__ballot(x) >> (threadIdx.x % 64 / W * W)) & 0xffffu; }
__device__ inline RowPart row_part(const int32_t *rowptr, const Residual &res, int64_t M, int t, const Rule &R) {
    const int64_t row = (int64_t)t * W + threadIdx.x % W;
    RowPart z;
    z.before = res.before(rowptr[min(row, M)]);
    z.len = res.before(rowptr[min(row + 1, M)]) - z.before;
    z.valid = rows_where(row < M);
    z.split = rows_where(z.len > 0 && z.len >= R.short_len && z.len > R.Cs);
    z.scalar = rows_where(z.len > 0) & ~z.split;
    return z;
}

__device__ inline void put_task(libra_task_t *t, int kind, int id, int b0, int b1, int q0, int q1, unsigned sc, unsigned at, unsigned st, unsigned cost) {
    t->kind = kind; t->id = id; t->blk_begin = b0; t->blk_end = b1; t->res_begin = q0; t->res_end = q1;
    t->scalar_mask = sc; t->atomic_mask = at; t->store_mask = st; t->cost = cost;
}

// Per window: the hybrid load-balancing rule (Section 4.3).  This pass counts tasks, rows to clear and residual nonzeros, 16 lanes per
// window.  The matrix's numbers go to their counters once per workgroup, of which there are few.
__global__ __launch_bounds__(256) void k_window_sizes(const int32_t *rowptr, Residual res_a, int64_t M, int nw, Rule R, const int32_t *blkptr_a, const int32_t *blkptr_d,
                                                      int32_t *ntasks_a, int32_t *nzero, int32_t *nres, int32_t *ntasks_d, u64 *ctr) {
    __shared__ unsigned counts[4];
    if (threadIdx.x < 4) counts[threadIdx.x] = 0;
    __syncthreads();
    const int r = threadIdx.x % W;
    if (blockIdx.x == 0 && threadIdx.x == 0) { ntasks_a[nw] = 0; nzero[nw] = 0; nres[nw] = 0; ntasks_d[nw] = 0; }
    unsigned n_short = 0, n_long = 0, n_split = 0, n_chunks = 0;
    for (int64_t t = (int64_t)blockIdx.x * (256 / W) + threadIdx.x / W; t < nw; t += (int64_t)gridDim.x * (256 / W)) {
        int ta = 0, zero = 0, residual = 0;
        if (R.build_a) {
            const RowPart z = row_part(rowptr, res_a, M, (int)t, R);
            const unsigned shorts = rows_where(z.len > 0 && z.len < R.short_len);
            const int chunks = sum_over_rows(z.split >> r & 1u ? piece_count(z.len, R.Cs) : 0), nb = blkptr_a[t + 1] - blkptr_a[t];
            const bool many = nb > R.Ts;
            ta = (many ? piece_count(nb, R.Ts) + (z.scalar ? 1 : 0) : 1) + chunks;
            zero = __popc(many ? z.valid : z.split);
            residual = sum_over_rows(z.len);
            n_short += __popc(shorts);
            n_long += __popc((z.scalar | z.split) & ~shorts);
            n_split += __popc(z.split);
            n_chunks += chunks;
        }
        if (r == 0) {
            ntasks_a[t] = ta;
            nzero[t] = zero;
            nres[t] = residual;
            ntasks_d[t] = R.build_d ? piece_count(blkptr_d[t + 1] - blkptr_d[t], R.Ts_d) : 0;
        }
    }
    if (r == 0) {
        const unsigned n[4] = {n_short, n_long, n_split, n_chunks};
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (n[k]) atomicAdd(&counts[k], n[k]);
    }
    __syncthreads();
    const int to[4] = {C_SHORT, C_LONG, C_SPLIT, C_SEGMENTS};
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if ((int)threadIdx.x == k && counts[k]) atomicAdd(&ctr[to[k]], (u64)counts[k]);
}

// The same rule: tasks and rows to clear at the offsets the prefix sums gave, a window per wave (a hub window has thousands of tasks);
// and where each row's residual nonzeros start in the SpMM residual array (rows that are not decomposed first, in row order, then
// the decomposed rows), minus the row's own prefix so that a nonzero only adds its scan value.  With a lane per row and per block:
// GAT graph 118 us in both passes; one thread or wave that walked the rows, and a third pass, 332.  A launch has fewer than 2^32 threads, so
// from 2^23 windows on a wave takes several.
__global__ __launch_bounds__(128) void k_window_tasks(const int32_t *rowptr, Residual res_a, int64_t M, int nw, Rule R,
                                                      const int32_t *blkptr_a, const int32_t *blkmask_a, const int32_t *blkncols_a,
                                                      const int32_t *blkptr_d, const int32_t *blkncols_d,
                                                      const int32_t *tbase_a, const int32_t *zbase, const int32_t *resptr, const int32_t *tbase_d,
                                                      libra_task_t *tasks_a, int32_t *zero_rows, int32_t *rowbase, libra_task_t *tasks_d) {
    const int lane = threadIdx.x % 64, r = lane % W;
    for (int t = (int)(blockIdx.x * 2 + threadIdx.x / 64); t < nw; t += (int)(gridDim.x * 2)) {
        const int64_t r0 = (int64_t)t * W;
        if (R.build_a) {
            const RowPart z = row_part(rowptr, res_a, M, t, R);
            const bool split = z.split >> r & 1u, mine = lane < W && (z.valid >> r & 1u);
            // places in the residual array: an inclusive sum over the rows of either kind
            int plain = split ? 0 : z.len, cut = split ? z.len : 0;
            const int plain_all = sum_over_rows(plain), own = z.len;
#pragma unroll
            for (int m = 1; m < W; m <<= 1) {
                const int x = __shfl_up(plain, m, W), y = __shfl_up(cut, m, W);
                if (r >= m) { plain += x; cut += y; }
            }
            const int q0 = resptr[t], q1 = q0 + plain_all, start = split ? q1 + cut - own : q0 + plain - own;
            if (mine) rowbase[r0 + r] = start - z.before;
            const int b0 = blkptr_a[t], b1 = blkptr_a[t + 1];
            libra_task_t *out = tasks_a + tbase_a[t];
            int32_t *zr = zero_rows + zbase[t];
            if (b1 - b0 > R.Ts) {
                const int groups = piece_count(b1 - b0, R.Ts);
                for (int g = lane; g < groups; g += 64) {
                    const int g0 = b0 + g * R.Ts, g1 = piece_end(g0, b1, R.Ts);
                    unsigned touched = 0, cols = 0;
                    for (int b = g0; b < g1; ++b) { touched |= (unsigned)blkmask_a[b]; cols += (unsigned)blkncols_a[b]; }
                    put_task(out + g, LIBRA_TASK_WINDOW, t, g0, g1, q0, q0, 0u, touched, 0u, cols);
                }
                out += groups;
                if (z.scalar) {
                    if (lane == 0) put_task(out, LIBRA_TASK_WINDOW, t, b1, b1, q0, q1, z.scalar, z.scalar, 0u, (unsigned)(q1 - q0));
                    ++out;
                }
                if (mine) zr[r] = (int32_t)(r0 + r);
            } else {
                unsigned touched = 0, cols = 0;
                for (int b = b0 + lane; b < b1; b += 64) { touched |= (unsigned)blkmask_a[b]; cols += (unsigned)blkncols_a[b]; }
#pragma unroll
                for (int m = 1; m < 64; m <<= 1) { touched |= __shfl_xor(touched, m, 64); cols += __shfl_xor(cols, m, 64); }
                if (lane == 0) put_task(out, LIBRA_TASK_WINDOW, t, b0, b1, q0, q1, z.scalar, z.split & touched, z.valid & ~z.split, cols + (unsigned)(q1 - q0));
                if (mine && split) zr[__popc(z.split & ((1u << r) - 1u))] = (int32_t)(r0 + r);
                ++out;
            }
            for (unsigned left = z.split; left; left &= left - 1u) {
                const int row = __ffs(left) - 1, q = __shfl(start, row, 64), len = __shfl(own, row, 64), n = piece_count(len, R.Cs);
                for (int k = lane; k < n; k += 64) {
                    const int qs = q + k * R.Cs, qe = piece_end(qs, q + len, R.Cs);
                    put_task(out + k, LIBRA_TASK_CHUNK, (int)(r0 + row), 0, 0, qs, qe, 0u, 0u, 0u, (unsigned)(qe - qs));
                }
                out += n;
            }
        }
        if (R.build_d) {
            const int b0 = blkptr_d[t], b1 = blkptr_d[t + 1];
            libra_task_t *out = tasks_d + tbase_d[t];
            for (int g = lane; g < piece_count(b1 - b0, R.Ts_d); g += 64) {
                const int g0 = b0 + g * R.Ts_d, g1 = piece_end(g0, b1, R.Ts_d);
                unsigned c = 0;
                for (int b = g0; b < g1; ++b) c += (unsigned)blkncols_d[b];
                put_task(out + g, LIBRA_TASK_WINDOW, t, g0, g1, 0, 0, 0u, 0u, 0u, c + (unsigned)W);
            }
        }
    }
}

// Where the residual nonzeros of a sub-plan go: arrays of the host planner's format, or the blocked entries of the plan's device copy
// (`entries`), with their CSR positions (perm; the SDDMM ones have none if they are the whole matrix) and the SDDMM ones' rows.
struct ResidualOut {
    int32_t *perm, *row, *col;
    uint8_t *val;
    unsigned char *entries;
    int32_t *base;              // SDDMM entries: first row per block
};
template <class V>
__device__ inline void put_entry(unsigned char *entries, int d, int col, unsigned upper, V v) {
    unsigned char *blk = entries + (int64_t)(d / RES_BLOCK) * (RES_BLOCK * (4 + (int)sizeof(V)));
    reinterpret_cast<uint32_t *>(blk)[d % RES_BLOCK] = (uint32_t)col | upper << RES_ROW_SHIFT;
    reinterpret_cast<V *>(blk + RES_BLOCK * 4)[d % RES_BLOCK] = v;
}
// Per nonzero (CSR order): residual nonzeros to their places.  SDDMM: CSR order.  Entries of SDDMM sub-plans that are not the whole matrix
// need the row of their block's first entry and are packed from the arrays by a pass of their own.  Bound by memory: GAT graph (59.7 M
// nonzeros, 35 bytes each) 521 us; to arrays that two passes packed and two copies moved, 1,250.
template <class V>
__global__ __launch_bounds__(256) void k_residual_fill(const int32_t *col, const V *val, int n, Rule R, const int32_t *row_of, Residual res_a, const int32_t *rowbase, ResidualOut a,
                                                      Residual res_d, ResidualOut d) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const bool ra = R.build_a && res_a.has(p), rd = R.build_d && res_d.has(p);
    if (!ra && !rd) return;
    const int i = row_of[p], c = col[p];
    const V v = val[p];
    if (ra) {
        const int q = rowbase[i] + res_a.before(p);
        a.perm[q] = p;
        if (a.entries) {
            put_entry(a.entries, q, c, (unsigned)(i % W), v);
        } else {
            a.row[q] = i; a.col[q] = c;
            reinterpret_cast<V *>(a.val)[q] = v;
        }
    }
    if (rd) {
        const int q = res_d.before(p);
        if (d.perm) d.perm[q] = p;
        d.row[q] = i;
        if (d.entries) {                    // the whole matrix: the block begins at nonzero p - p % RES_BLOCK
            const int first = row_of[p - p % RES_BLOCK];
            put_entry(d.entries, q, c, min((unsigned)(i - first), RES_FAR), v);
            if (p % RES_BLOCK == 0) d.base[p / RES_BLOCK] = first;
        } else {
            d.col[q] = c;
            reinterpret_cast<V *>(d.val)[q] = v;
        }
    }
}

// The nonzero (CSR position) that is residual nonzero x of those counted by `res`; it lies in [lo, hi).
__device__ inline int residual_at(const Residual &res, int x, int lo, int hi) {
    if (!res.scan) return x;
    while (lo < hi) {                       // the first with more than x of them before its successor
        const int mid = lo + ((hi - lo) >> 1);
        if (res.scan[mid + 1] <= x) lo = mid + 1; else hi = mid;
    }
    return lo;
}
// Per flat SDDMM residual segment (cs entries of the residual list): its first column if the segment lies in one row, else -1.
__global__ __launch_bounds__(256) void k_segment_cols(const int32_t *row_of, const int32_t *col, Residual res, int n, int nres, int cs, int nseg, int32_t *seg_col) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nseg) return;
    const int64_t q = (int64_t)i * cs, q1 = q + cs < nres ? q + cs : nres;
    const int p = residual_at(res, (int)q, 0, n), p1 = residual_at(res, (int)q1 - 1, p, n);
    seg_col[i] = row_of[p] == row_of[p1] ? col[p] : -1;
}
// Per SpMM task: first column of a row segment's entries (the tables order the segments by it), -1 for other tasks.
__global__ __launch_bounds__(256) void k_task_cols(const libra_task_t *tasks, int nt, const int32_t *rowptr, const int32_t *rowbase, const int32_t *col, Residual res, int32_t *task_col) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nt) return;
    const libra_task_t &t = tasks[i];
    int c = -1;
    if (t.kind == LIBRA_TASK_CHUNK) c = col[residual_at(res, t.res_begin - rowbase[t.id], rowptr[t.id], rowptr[t.id + 1])];
    task_col[i] = c;
}

// ------------------------------------------------------------------------------------------
// Order of the task tables: the rules of finish_plan (heaviest first, segments by column, die-aware groups) as stable sorts
// and prefix sums, with the same result.  A table is a list of task indices; SDDMM index nt + s is flat residual segment s.
// ------------------------------------------------------------------------------------------
constexpr int XC = LIBRA_XCDS;

struct TaskView {
    const libra_task_t *tasks;
    int nt, cs, nres;                   // SDDMM segments: cs entries each of nres
    __device__ u64 cost(int i) const {
        if (i < nt) return tasks[i].cost;
        return 2u * (unsigned)min(cs, nres - (i - nt) * cs);
    }
    __device__ bool empty(int i) const {          // writes nothing and reads nothing
        if (i >= nt) return false;
        const libra_task_t &t = tasks[i];
        return t.cost == 0 && t.blk_begin == t.blk_end && t.res_begin == t.res_end && t.store_mask == 0 && t.atomic_mask == 0;
    }
    __device__ int group(int i) const {
        if (i >= nt) return (i - nt) / LIBRA_LOCALITY_SEGMENTS;
        return (tasks[i].kind == LIBRA_TASK_WINDOW ? tasks[i].id : tasks[i].id / W) / LIBRA_LOCALITY_WINDOWS;
    }
};
// round r of the snake deal gives its p-th item to this queue
__device__ inline int snake(int r) { return r / XC & 1 ? XC - 1 - r % XC : r % XC; }
// how many of the first n items of the deal go to queue x
__host__ __device__ inline int snake_count(int n, int x) { return n / XC + ((n / XC & 1 ? XC - 1 - x : x) < n % XC ? 1 : 0); }

__global__ __launch_bounds__(256) void k_order_costs(TaskView v, int n, uint32_t *key) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) key[i] = (uint32_t)v.cost(i);
}
__global__ __launch_bounds__(256) void k_order_identity(int n, int first, int32_t *out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = first + i;
}
// flag = 1: the item goes by its column (SpMM: segments of decomposed rows; SDDMM: segments inside one row)
__global__ __launch_bounds__(256) void k_order_by_column_flag(TaskView v, const int32_t *list, const int32_t *col, int n, int32_t *flag) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i > n) return;
    flag[i] = i < n && (list[i] < v.nt ? v.tasks[list[i]].kind == LIBRA_TASK_CHUNK : col[list[i] - v.nt] >= 0) ? 1 : 0;
}
// the flagged items with their columns, the others with their costs, each in list order
__global__ __launch_bounds__(256) void k_order_split(TaskView v, const int32_t *list, const int32_t *col, const int32_t *flag, const int32_t *scan, int n,
                                                     uint32_t *key, int32_t *placed, int32_t *other, uint32_t *other_cost) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int item = list[i], k = scan[i];
    if (flag[i]) {
        key[k] = (uint32_t)col[item < v.nt ? item : item - v.nt];
        placed[k] = item;
    } else {
        other[i - k] = item;
        other_cost[i - k] = (uint32_t)v.cost(item);
    }
}
__global__ __launch_bounds__(256) void k_order_item_costs(TaskView v, const int32_t *list, int n, u64 *cost) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i <= n) cost[i] = i < n ? v.cost(list[i]) : 0;
}
// The die of segment k: LIBRA_XCDS runs of equal cost (run[k] = cost before it, run[n] = all).
__device__ inline int run_of(const u64 *run, int k, int n) {
    const u64 total = run[n] ? run[n] : 1;
    const u64 x = run[k] * XC / total;
    return x < XC - 1 ? (int)x : XC - 1;
}
__global__ void k_order_fill(int32_t *p, int n, int value) {
    if ((int)threadIdx.x < n) p[threadIdx.x] = value;
}
// first segment of every die's run (start was filled with n)
__global__ __launch_bounds__(256) void k_order_run_starts(const u64 *run, int n, int32_t *start) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const int x = run_of(run, k, n), before = k ? run_of(run, k - 1, n) : -1;
    for (int y = before + 1; y <= x; ++y) start[y] = k;
}
// A die's queue merges its share of the others (descending cost) with its run of segments (column order): segment k comes
// after the others of its die that cost no less than it or than a segment before it.  This counts the first kind; the maximum
// over the run (the die in the high word restarts it) adds the second.
__global__ __launch_bounds__(256) void k_order_others_before(TaskView v, const int32_t *seg, const u64 *run, int n, const uint32_t *other_cost, int no, u64 *before) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const uint32_t c = (uint32_t)v.cost(seg[k]);
    int lo = 0, hi = no;                // others [0, lo) cost at least c
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (other_cost[mid] >= c) lo = mid + 1; else hi = mid;
    }
    const int x = run_of(run, k, n);
    before[k] = (u64)x << 32 | (u64)snake_count(lo, x);
}
__global__ __launch_bounds__(256) void k_order_merge(const int32_t *seg, const u64 *before, const int32_t *start, int n, const int32_t *other, int no, int32_t *queue) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n + no) return;
    const bool is_seg = i < n;
    const int x = is_seg ? (int)(before[i] >> 32) : snake(i - n);
    int off = start[x];                 // the queues one after another: runs and shares of the dies before
    for (int y = 0; y < x; ++y) off += snake_count(no, y);
    if (is_seg) {
        queue[off + (i - start[x]) + (int)(before[i] & 0xffffffffull)] = seg[i];
    } else {
        const int r = (i - n) / XC, s0 = start[x], s1 = start[x + 1];
        int lo = s0, hi = s1;           // segments [s0, lo) come before the die's r-th other
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if ((int)(before[mid] & 0xffffffffull) <= r) lo = mid + 1; else hi = mid;
        }
        queue[off + r + (lo - s0)] = other[i - n];
    }
}
// SDDMM segments: those inside one row by column, cut into LIBRA_XCDS equal runs, then the others round-robin.
__global__ __launch_bounds__(256) void k_order_sddmm_queues(const int32_t *placed, int n, const int32_t *other, int no, int32_t *queue) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n + no) return;
    auto start = [&](int x) { return (int)(((int64_t)x * n + XC - 1) / XC); };
    const int x = i < n ? (int)((int64_t)i * XC / n) : (i - n) % XC;
    int off = start(x);
    for (int y = 0; y < x; ++y) off += (no - y + XC - 1) / XC;
    if (i < n) queue[off + i - start(x)] = placed[i];
    else queue[off + start(x + 1) - start(x) + (i - n) / XC] = other[i - n];
}
// ---- die-aware groups ----
__global__ __launch_bounds__(256) void k_order_groups(TaskView v, const int32_t *list, int n, uint32_t *key) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) key[i] = (uint32_t)v.group(list[i]);
}
__global__ __launch_bounds__(256) void k_order_heads(const uint32_t *key, int n, int32_t *flag) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i <= n) flag[i] = i < n && (i == 0 || key[i] != key[i - 1]) ? 1 : 0;
}
__global__ __launch_bounds__(256) void k_order_firsts(const int32_t *flag, const int32_t *scan, int n, int32_t *first) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i > n) return;
    if (i == n || flag[i]) first[scan[i]] = i;
}
__global__ __launch_bounds__(256) void k_order_group_costs(const u64 *run, const int32_t *first, int ng, u64 *cost) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g < ng) cost[g] = run[first[g + 1]] - run[first[g]];
}
// groups heaviest first -> sizes in queue order, the queues one after another (`rounds` places each)
__global__ __launch_bounds__(256) void k_order_deal(const int32_t *gord, const int32_t *first, int ng, int rounds, int32_t *size, int32_t *place) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r > rounds * XC) return;
    if (r == rounds * XC) { size[r] = 0; return; }
    const int at = snake(r) * rounds + r / XC;
    size[at] = r < ng ? first[gord[r] + 1] - first[gord[r]] : 0;
    if (r < ng) place[gord[r]] = at;
}
__global__ __launch_bounds__(256) void k_order_group_items(const int32_t *list, const int32_t *flag, const int32_t *scan, const int32_t *first, const int32_t *place,
                                                           const int32_t *base, int n, int32_t *queue) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int g = scan[i] + flag[i] - 1;
    queue[base[place[g]] + i - first[g]] = list[i];
}
__global__ void k_order_queue_starts(const int32_t *base, int rounds, int32_t *start) {
    if (threadIdx.x <= XC) start[threadIdx.x] = base[threadIdx.x * rounds];
}
// Slot 8 j + x of the region is the j-th item of queue x, or an empty task.
__global__ __launch_bounds__(256) void k_order_emit(const int32_t *queue, const int32_t *pieces, int4 p0, int4 p1, int np, int4 n0, int4 n1, int slots, int32_t *out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= slots) return;
    const int x = i % XC, j = i / XC;
    const int begin[XC + 1] = {p0.x, p0.y, p0.z, p0.w, p1.x, p1.y, p1.z, p1.w, np}, len[XC] = {n0.x, n0.y, n0.z, n0.w, n1.x, n1.y, n1.z, n1.w};
    int b = 0, e = 0, n = 0;
#pragma unroll
    for (int y = 0; y < XC; ++y)
        if (y == x) { b = begin[y]; e = begin[y + 1]; n = len[y]; }
    int item = -1;
    if (j < n) {
        while (e - b > 1) {             // the piece that holds the j-th item
            const int mid = (b + e) >> 1;
            if (pieces[3 * mid + 1] <= j) b = mid; else e = mid;
        }
        item = queue[pieces[3 * b + 2] + j - pieces[3 * b + 1]];
    }
    out[i] = item;
}
// The slots up to the last task that does something: one workgroup, from the end on (the queues are levelled, so it is near the end).  As
// a maximum that all waves of k_order_emit look at, two tables of 500,000 slots took 200 us and not 22.
__global__ __launch_bounds__(1024) void k_order_last(TaskView v, const int32_t *out, int slots, int32_t *last) {
    __shared__ int found;
    if (threadIdx.x == 0) found = 0;
    __syncthreads();
    for (int64_t end = slots; end > 0 && found == 0; end -= 1024) {
        const int64_t i = end - 1 - (int64_t)threadIdx.x;
        const int item = i >= 0 ? out[i] : -1;
        __syncthreads();                    // every thread has seen that nothing was found before
        if (item >= 0 && !v.empty(item)) atomicMax(&found, (int)i + 1);
        __syncthreads();
    }
    if (threadIdx.x == 0) *last = found;
}
// Device task records, die by die (as the host packs them); slots past the table's end and -1 hold empty tasks.
__global__ __launch_bounds__(256) void k_order_records(TaskView v, const int32_t *order, int n, int per_die, const int32_t *blk_valptr, int empty_kind, DevTask *out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= per_die * XC) return;
    DevTask d{0, 0, 0, 0, 0, 0u, (uint32_t)empty_kind, 0};
    const int item = i < n ? order[i] : -1;
    if (item >= v.nt) {
        const int q = (item - v.nt) * v.cs;
        d.res_begin = q;
        d.res_end = piece_end(q, v.nres, v.cs);
        d.kind = LIBRA_TASK_CHUNK;
    } else if (item >= 0) {
        const libra_task_t t = v.tasks[item];
        const bool window = t.kind == LIBRA_TASK_WINDOW;
        d = DevTask{t.id, t.blk_begin, t.blk_end, t.res_begin, t.res_end, (t.atomic_mask & 0xffffu) | (t.store_mask << 16), (uint32_t)t.kind,
                    window ? blk_valptr[t.blk_begin] : 0};
        if (!window) {                  // a segment of a decomposed row = a task of the row's window with one atomic output row
            d.id = t.id / W;
            d.blk_begin = d.blk_end = 0;
            d.masks = 1u << (t.id % W);
        }
    }
    out[(int64_t)(i % XC) * per_die + i / XC] = d;
}

// ------------------------------------------------------------------------------------------
// host driver
// ------------------------------------------------------------------------------------------
struct Fail { int code; };
inline void hip_ok(hipError_t e) { if (e != hipSuccess) throw Fail{LIBRA_ERR_HIP}; }
inline unsigned blocks_for(int64_t n, int per) { return (unsigned)std::max<int64_t>(1, (n + per - 1) / per); }

void scan(const Layout &L, const int32_t *in, int32_t *out, size_t n, hipStream_t s) {
    size_t sz = L.tmp_bytes;
    hip_ok(rocprim::exclusive_scan(L.tmp, sz, in, out, (int32_t)0, n, rocprim::plus<int32_t>(), s));
}

// Prefix sums of up to four short arrays in one launch, a workgroup each (two rounds of 8,192 items at most); longer ones are rocPRIM's.
constexpr int SHORT_SCAN = 16384;
struct ScanJobs { const int32_t *in[4]; int32_t *out[4]; int32_t n[4]; };
__global__ __launch_bounds__(1024) void k_scan_short(ScanJobs jobs) {
    __shared__ int32_t wave_sum[16];
    const int32_t *in = nullptr;
    int32_t *out = nullptr;
    int n = 0, carry = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if ((int)blockIdx.x == k) { in = jobs.in[k]; out = jobs.out[k]; n = jobs.n[k]; }
    const int tid = threadIdx.x;
    for (int base = 0; base < n; base += 8192) {
        int v[8], sum = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = base + tid * 8 + j < n ? in[base + tid * 8 + j] : 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) { const int x = v[j]; v[j] = sum; sum += x; }
        int scan = sum;
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) {
            const int x = __shfl_up(scan, m, 64);
            if (tid % 64 >= m) scan += x;
        }
        if (tid % 64 == 63) wave_sum[tid / 64] = scan;
        __syncthreads();
        int before = carry + scan - sum, all = 0;
        for (int w = 0; w < 16; ++w) {
            const int x = wave_sum[w];
            before += w < tid / 64 ? x : 0;
            all += x;
        }
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (base + tid * 8 + j < n) out[base + tid * 8 + j] = before + v[j];
        carry += all;
        __syncthreads();
    }
}
struct ScanJob { const int32_t *in; int32_t *out; int64_t n; };
void scan_all(const Layout &L, std::initializer_list<ScanJob> jobs, hipStream_t s) {
    ScanJobs small{};
    int count = 0;
    for (const ScanJob &j : jobs) {
        if (j.n > SHORT_SCAN) {
            scan(L, j.in, j.out, (size_t)j.n, s);
        } else {
            small.in[count] = j.in;
            small.out[count] = j.out;
            small.n[count++] = (int32_t)j.n;
        }
    }
    if (count) hipLaunchKernelGGL(k_scan_short, dim3((unsigned)count), dim3(1024), 0, s, small);
}

template <class T>
void fetch(std::vector<T> &dst, const void *src, size_t n, hipStream_t s) {
    dst.resize(n);
    if (n) hip_ok(hipMemcpyAsync(dst.data(), src, n * sizeof(T), hipMemcpyDeviceToHost, s));
}

void fill_bytes(void *p, int value, size_t bytes, hipStream_t s) {
    if (bytes) hip_ok(hipMemsetAsync(p, value, bytes, s));
}

int32_t peek(const int32_t *p, hipStream_t s) {
    int32_t v = 0;
    hip_ok(hipMemcpyAsync(&v, p, sizeof v, hipMemcpyDeviceToHost, s));
    hip_ok(hipStreamSynchronize(s));
    return v;
}

// ---- the order of one table region on the device ----
struct Orderer {
    const Layout &L;
    hipStream_t s;
    TaskView v;
    const int32_t *col;                 // first columns: per SpMM task, per SDDMM segment
    int colbits;

    static int bits_for(int64_t max_value) { int b = 1; while (b < 32 && (max_value >> b)) ++b; return b; }
    template <class F, class... A> void launch(F *k, unsigned blocks, unsigned threads, A... a) {
        hipLaunchKernelGGL(k, dim3(blocks), dim3(threads), 0, s, a...);
        hip_ok(hipGetLastError());
    }
    template <class F, class... A> void run(F *k, int64_t n, A... a) { launch(k, blocks_for(n, 256), 256, a...); }
    // numbers that come back from the device become launch sizes and indexes: they are not used out of their range
    static void check(bool ok) { if (!ok) throw Fail{LIBRA_ERR_HIP}; }
    static void check_queues(const int *start, int n) {
        check(start[0] == 0 && start[XC] == n);
        for (int x = 0; x < XC; ++x) check(start[x] <= start[x + 1]);
    }
    template <class T> void scan_sum(const T *in, T *out, size_t n) {
        size_t sz = L.tmp_bytes;
        hip_ok(rocprim::exclusive_scan(L.tmp, sz, in, out, (T)0, n, rocprim::plus<T>(), s));
    }
    void sort_by_key(const int32_t *in, int32_t *out, size_t n, int bits) {          // key_in -> key_out, stable
        size_t sz = L.tmp_bytes;
        hip_ok(sort_pairs<false>(L.tmp, sz, L.o.key_in, L.o.key_out, in, out, n, (unsigned)bits, s));
    }
    // items 0 .. n-1 by descending cost, stable
    void heaviest_first(int n, int32_t *out) {
        if (n == 0) return;
        run(k_order_costs, n, v, n, L.o.key_in);
        size_t sz = L.tmp_bytes;
        hip_ok(sort_pairs<true>(L.tmp, sz, L.o.key_in, L.o.key_out, rocprim::counting_iterator<int32_t>(0), out, (size_t)n, 32u, s));
    }
    void identity(int n, int first, int32_t *out) { if (n) run(k_order_identity, n, n, first, out); }
    int copy(const int32_t *list, int n, int32_t *out) {
        if (n) hip_ok(hipMemcpyAsync(out, list, (size_t)n * 4, hipMemcpyDeviceToDevice, s));
        return n;
    }
    // The queues lie one after another in L.o.queue, start[x] .. start[x + 1]: lengths levelled and interleaved as
    // interleave_queues does it; returns the region's length.
    int interleave(const int *start, int32_t *out) {
        struct Piece { int from, n; };
        std::vector<Piece> q[XC];
        int len[XC];
        for (int x = 0; x < XC; ++x) {
            len[x] = start[x + 1] - start[x];
            if (len[x]) q[x].push_back({start[x], len[x]});
        }
        for (;;) {
            int lo = 0, hi = 0;
            for (int x = 1; x < XC; ++x) {
                if (len[x] < len[lo]) lo = x;
                if (len[x] > len[hi]) hi = x;
            }
            if (len[hi] - len[lo] <= 1) break;
            const int move = (len[hi] - len[lo]) / 2;
            std::vector<Piece> tail;            // last pieces of the longest queue, in order
            for (int left = move; left > 0;) {
                Piece &b = q[hi].back();
                const int take = std::min(left, b.n);
                tail.push_back({b.from + b.n - take, take});
                b.n -= take;
                if (b.n == 0) q[hi].pop_back();
                left -= take;
            }
            q[lo].insert(q[lo].end(), tail.rbegin(), tail.rend());
            len[hi] -= move;
            len[lo] += move;
        }
        std::vector<int32_t> table;
        int begin[XC + 1], slots = 0;
        for (int x = 0; x < XC; ++x) {
            begin[x] = (int)table.size() / 3;
            int at = 0;
            for (const Piece &p : q[x]) {
                table.insert(table.end(), {x, at, p.from});
                at += p.n;
            }
            slots = std::max(slots, len[x] * XC);
        }
        begin[XC] = (int)table.size() / 3;
        if (begin[XC] > MAX_PIECES) throw Fail{LIBRA_ERR_HIP};
        hip_ok(hipMemcpyAsync(L.o.pieces, table.data(), table.size() * 4, hipMemcpyHostToDevice, s));
        run(k_order_emit, slots, (const int32_t *)L.o.queue, (const int32_t *)L.o.pieces, make_int4(begin[0], begin[1], begin[2], begin[3]),
            make_int4(begin[4], begin[5], begin[6], begin[7]), begin[XC], make_int4(len[0], len[1], len[2], len[3]),
            make_int4(len[4], len[5], len[6], len[7]), slots, out);
        launch(k_order_last, 1, 1024, v, (const int32_t *)out, slots, L.o.meta + 32);
        const int end = peek(L.o.meta + 32, s);         // also keeps `table` alive until it has been copied
        check(end >= 0 && end <= slots);
        return end;
    }
    // Die-aware groups of `list` (place in the list breaks ties); `max_group` bounds the group numbers.
    int grouped(const int32_t *list, int n, int64_t max_group, int32_t *out) {
        if (n < 2 * XC) return copy(list, n, out);
        const OrderScratch &o = L.o;
        run(k_order_groups, n, v, list, n, o.key_in);
        sort_by_key(list, o.ord2, (size_t)n, bits_for(max_group));
        run(k_order_heads, n + 1, (const uint32_t *)o.key_out, n, o.flag);
        scan_sum<int32_t>(o.flag, o.scan, (size_t)n + 1);
        run(k_order_item_costs, n + 1, v, (const int32_t *)o.ord2, n, o.wide_in);
        scan_sum<u64>(o.wide_in, o.wide_out, (size_t)n + 1);
        run(k_order_firsts, n + 1, (const int32_t *)o.flag, (const int32_t *)o.scan, n, o.first);
        const int ng = peek(o.scan + n, s), rounds = (ng + XC - 1) / XC;
        check(ng > 0 && ng <= n);
        run(k_order_group_costs, ng, (const u64 *)o.wide_out, (const int32_t *)o.first, ng, o.wide_in);
        int32_t *gord = reinterpret_cast<int32_t *>(o.key_in), *size = reinterpret_cast<int32_t *>(o.key_out);
        size_t sz = L.tmp_bytes;
        hip_ok(sort_pairs<true>(L.tmp, sz, o.wide_in, o.wide_out, rocprim::counting_iterator<int32_t>(0), gord, (size_t)ng, 40u, s));
        run(k_order_deal, rounds * XC + 1, (const int32_t *)gord, (const int32_t *)o.first, ng, rounds, size, o.rank);
        scan_sum<int32_t>(size, o.base, (size_t)rounds * XC + 1);
        run(k_order_group_items, n, (const int32_t *)o.ord2, (const int32_t *)o.flag, (const int32_t *)o.scan, (const int32_t *)o.first,
            (const int32_t *)o.rank, (const int32_t *)o.base, n, o.queue);
        launch(k_order_queue_starts, 1, 64, (const int32_t *)o.base, rounds, o.meta);
        int start[XC + 1];
        hip_ok(hipMemcpyAsync(start, o.meta, sizeof start, hipMemcpyDeviceToHost, s));
        hip_ok(hipStreamSynchronize(s));
        check_queues(start, n);
        return interleave(start, out);
    }
    // Segments by column; `list` is the whole SpMM table heaviest first, or the SDDMM segments in CSR order.
    int by_column(const int32_t *list, int n, bool spmm, int32_t *out) {
        const OrderScratch &o = L.o;
        if (n == 0) return 0;
        run(k_order_by_column_flag, n + 1, v, list, col, n, o.flag);
        scan_sum<int32_t>(o.flag, o.scan, (size_t)n + 1);
        const int ns = peek(o.scan + n, s), no = n - ns;
        check(ns >= 0 && ns <= n);
        if (ns < 8 * XC) return copy(list, n, out);
        int32_t *other = o.first, *placed = o.ord2, *sorted = o.base;
        uint32_t *other_cost = reinterpret_cast<uint32_t *>(o.rank);
        run(k_order_split, n, v, list, col, (const int32_t *)o.flag, (const int32_t *)o.scan, n, o.key_in, placed, other, other_cost);
        sort_by_key(placed, sorted, (size_t)ns, colbits);
        int start[XC + 1];
        if (spmm) {
            run(k_order_item_costs, ns + 1, v, (const int32_t *)sorted, ns, o.wide_in);
            scan_sum<u64>(o.wide_in, o.wide_out, (size_t)ns + 1);
            launch(k_order_fill, 1, 64, o.meta, XC + 1, ns);
            run(k_order_run_starts, ns, (const u64 *)o.wide_out, ns, o.meta);
            run(k_order_others_before, ns, v, (const int32_t *)sorted, (const u64 *)o.wide_out, ns, (const uint32_t *)other_cost, no, o.wide_in);
            size_t sz = L.tmp_bytes;
            hip_ok(rocprim::inclusive_scan(L.tmp, sz, o.wide_in, o.wide_out, (size_t)ns, rocprim::maximum<u64>(), s));
            run(k_order_merge, n, (const int32_t *)sorted, (const u64 *)o.wide_out, (const int32_t *)o.meta, ns, (const int32_t *)other, no, o.queue);
            hip_ok(hipMemcpyAsync(start, o.meta, sizeof start, hipMemcpyDeviceToHost, s));
            hip_ok(hipStreamSynchronize(s));
            for (int x = 0, before = 0; x <= XC; ++x) {
                start[x] += before;
                if (x < XC) before += snake_count(no, x);
            }
        } else {
            run(k_order_sddmm_queues, n, (const int32_t *)sorted, ns, (const int32_t *)other, no, o.queue);
            for (int x = 0, before = 0; x <= XC; ++x) {
                start[x] = (int)(((int64_t)x * ns + XC - 1) / XC) + before;
                if (x < XC) before += (no - x + XC - 1) / XC;
            }
        }
        check_queues(start, n);
        return interleave(start, out);
    }
};

// Noops of a table as the host planner writes them.
inline libra_task_t task_at(const std::vector<libra_task_t> &tasks, int item, int cs, int nres, int empty_kind) {
    if (item < 0) return libra_task_t{empty_kind, 0, 0, 0, 0, 0, 0u, 0u, 0u, 0u};
    if (item < (int)tasks.size()) return tasks[item];
    const int q = (item - (int)tasks.size()) * cs, q1 = piece_end(q, nres, cs);
    return libra_task_t{LIBRA_TASK_CHUNK, 0, 0, 0, q, q1, 0u, 0u, 0u, 2u * (uint32_t)(q1 - q)};
}

// Several single words in one copy and one wait (each peek is a round trip of some 10 us).
struct Words { const int32_t *at[7]; };
__global__ void k_gather_words(Words w, int n, int32_t *out) {
#pragma unroll
    for (int i = 0; i < 7; ++i)
        if (i < n && (int)threadIdx.x == i) out[i] = *w.at[i];
}
void peek_all(int32_t *scratch, std::initializer_list<const int32_t *> from, int32_t (&to)[7], hipStream_t s) {
    Words w{};
    std::copy(from.begin(), from.end(), w.at);
    hipLaunchKernelGGL(k_gather_words, dim3(1), dim3(64), 0, s, w, (int)from.size(), scratch);
    hip_ok(hipMemcpyAsync(to, scratch, from.size() * sizeof(int32_t), hipMemcpyDeviceToHost, s));
    hip_ok(hipStreamSynchronize(s));
}

}  // namespace

extern "C" int libra_plan_device_workspace(int64_t M, int64_t nnz, const libra_plan_opts_t *opts, size_t *bytes) {
    if (!bytes) return LIBRA_ERR_NULL;
    if (M < 1 || nnz < 0) return LIBRA_ERR_SHAPE;
    if (M >= (1ll << 31) - 64 || nnz >= (1ll << 31) - 64) return LIBRA_ERR_TOO_LARGE;
    Resolved o{};
    if (int rc = resolve_options(opts, LIBRA_F32, o)) return rc;       // the widest value type bounds the size
    if (o.W != W || o.KB != KB) return LIBRA_ERR_UNSUPPORTED;
    *bytes = make_layout(make_sizes(M, std::max<int64_t>(nnz, 1), o), 4, nullptr).total;
    return LIBRA_OK;
}

extern "C" int libra_plan_device_buffer_bound(int64_t M, int64_t nnz, int val_dtype, const libra_plan_opts_t *opts, size_t *bytes) {
    if (!bytes) return LIBRA_ERR_NULL;
    if (M < 1 || nnz < 0) return LIBRA_ERR_SHAPE;
    if (M >= (1ll << 31) - 64 || nnz >= (1ll << 31) - 64) return LIBRA_ERR_TOO_LARGE;
    if (val_dtype != LIBRA_F16 && val_dtype != LIBRA_BF16 && val_dtype != LIBRA_F32) return LIBRA_ERR_DTYPE;
    Resolved o{};
    if (int rc = resolve_options(opts, val_dtype, o)) return rc;
    if (o.W != W || o.KB != KB) return LIBRA_ERR_UNSUPPORTED;
    try {
        // a plan with the largest arrays this matrix size can produce (only the sizes matter)
        const Sizes z = make_sizes(M, std::max<int64_t>(nnz, 1), o);
        libra_plan_t fake;
        fake.M = M; fake.nnz = -1;      // no residual list is "the whole matrix": the SDDMM position array is counted
        fake.vdt = val_dtype; fake.vsize = val_dtype == LIBRA_F32 ? 4 : 2;
        fake.o = o;
        for (SubPlan *sp : {&fake.spmm, &fake.sddmm}) {
            sp->n.blocks = z.nbmax; sp->n.col_slots = z.nbmax * KB; sp->n.bitmap_words = z.nbmax * 4;
            sp->n.dense = nnz; sp->n.res = nnz;
        }
        fake.spmm.n.zero_rows = M;
        fake.spmm.n.tasks = 2 * z.tasks_a_max + 64;                                // the die-aware order may add empty tasks
        fake.sddmm.n.tasks = 2 * (z.tasks_d_max + nnz / o.sddmm_Cs + 1) + 64;
        *bytes = plan_buffer_bytes(&fake) + 2 * align256((size_t)M * 4 + 16);      // + the two row lists of the edge softmax
    } catch (...) {
        return LIBRA_ERR_NOMEM;
    }
    return LIBRA_OK;
}

extern "C" int libra_plan_device(int64_t M, int64_t Kc, int64_t nnz, const int32_t *d_rowptr, const int32_t *d_col, const void *d_val,
                                 int val_dtype, const libra_plan_opts_t *opts, void *workspace, size_t workspace_bytes,
                                 void *plan_buf, size_t plan_bytes, int keep_host_copy, void *stream, libra_plan_t **out) {
    if (!out) return LIBRA_ERR_NULL;
    *out = nullptr;
    if (!d_rowptr) return LIBRA_ERR_NULL;
    if (M < 1 || Kc < 1 || nnz < 0) return LIBRA_ERR_SHAPE;
    if (M >= (1ll << 31) - 64 || Kc >= (1ll << 31) || nnz >= (1ll << 31) - 64) return LIBRA_ERR_TOO_LARGE;
    if (val_dtype != LIBRA_F16 && val_dtype != LIBRA_BF16 && val_dtype != LIBRA_F32) return LIBRA_ERR_DTYPE;
    Resolved o{};
    if (int rc = resolve_options(opts, val_dtype, o)) return rc;
    if (o.W != W || o.KB != KB) return LIBRA_ERR_UNSUPPORTED;
    if (nnz > 0 && (!d_col || !d_val || !workspace)) return LIBRA_ERR_NULL;
    if (!plan_buf) keep_host_copy = 1;          // the plan has to live somewhere
    hipStream_t s = (hipStream_t)stream;
    const auto t0 = std::chrono::steady_clock::now();
    // LIBRA_TRACE=1 in the environment prints where the call's time goes (stderr)
    const bool trace = std::getenv("LIBRA_TRACE") != nullptr;
    auto mark = [&](const char *what) {
        if (trace) std::fprintf(stderr, "[libra_plan_device] %-28s %8.3f ms\n", what,
                                1e3 * std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count());
    };

    libra_plan_t *P = new (std::nothrow) libra_plan_t();
    if (!P) return LIBRA_ERR_NOMEM;
    try {
        P->M = M; P->Kc = Kc; P->nnz = nnz; P->vdt = val_dtype; P->vsize = val_dtype == LIBRA_F32 ? 4 : 2;
        P->o = o;
        const bool rows_here = M >= DEVICE_ROWS_MIN && !keep_host_copy && nnz > 0 && !((uintptr_t)workspace & 255) &&
                               workspace_bytes >= make_layout(make_sizes(M, nnz, o), P->vsize, workspace).total;
        if (rows_here) {
            const Layout L = make_layout(make_sizes(M, nnz, o), P->vsize, workspace);
            u64 bad = 0;
            fill_bytes(L.ctr, 0, C_COUNT * sizeof(u64), s);
            hipLaunchKernelGGL(k_check_rowptr, dim3(blocks_for(M + 1, 256)), dim3(256), 0, s, d_rowptr, M, (int)nnz, L.ctr);
            hip_ok(hipMemcpyAsync(&bad, L.ctr + C_ERR, sizeof bad, hipMemcpyDeviceToHost, s));
            hip_ok(hipStreamSynchronize(s));
            if (bad) throw Fail{LIBRA_ERR_ROWPTR};
            // longest first: one workgroup takes a long row, and the longest one sets the time of the whole class
            auto select = [&](int above, int most, int32_t *to, int32_t *count) {
                size_t sz = L.tmp_bytes;
                hip_ok(rocprim::select(L.tmp, sz, rocprim::counting_iterator<int32_t>(0), to, count, (size_t)M, RowsOfLength{d_rowptr, above, most}, s));
            };
            select(64, LIBRA_SOFTMAX_LONG_ROW, L.medium_rows, L.sizes);
            select(LIBRA_SOFTMAX_LONG_ROW, INT32_MAX, L.long_rows, L.sizes + 1);
            int32_t count[2];
            hip_ok(hipMemcpyAsync(count, L.sizes, sizeof count, hipMemcpyDeviceToHost, s));
            hip_ok(hipStreamSynchronize(s));
            P->n_medium_rows = count[0];
            if (count[1] > 0) {
                uint32_t *len = L.long_lens, *by_len = len + count[1];
                int32_t *sorted = reinterpret_cast<int32_t *>(by_len + count[1]);
                hipLaunchKernelGGL(k_row_lengths, dim3(blocks_for(count[1], 256)), dim3(256), 0, s, d_rowptr, L.long_rows, count[1], len);
                size_t sz = L.tmp_bytes;
                hip_ok(sort_pairs<true>(L.tmp, sz, len, by_len, (const int32_t *)L.long_rows, sorted, (size_t)count[1], 32u, s));
                fetch(P->long_rows, sorted, (size_t)count[1], s);
                hip_ok(hipStreamSynchronize(s));
            }
        } else {
            fetch(P->rowptr, d_rowptr, (size_t)M + 1, s);
            hip_ok(hipStreamSynchronize(s));
            if (P->rowptr[0] != 0 || P->rowptr[M] != nnz) throw Fail{LIBRA_ERR_ROWPTR};
            for (int64_t i = 0; i < M; ++i)
                if (P->rowptr[i + 1] < P->rowptr[i]) throw Fail{LIBRA_ERR_ROWPTR};
        }
        if (nnz == 0) {
            // nothing to sort or scan: the plan of a matrix without nonzeros (one empty task per window) needs no device work
            const std::vector<int32_t> rp = P->rowptr;
            delete P;
            int rc = libra_plan(M, Kc, rp.data(), nullptr, nullptr, val_dtype, opts, out);
            if (rc == LIBRA_OK && plan_buf && (rc = libra_plan_upload(*out, plan_buf, plan_bytes, stream)) != LIBRA_OK) {
                libra_plan_destroy(*out);
                *out = nullptr;
            }
            return rc;
        }
        mark("rowptr checked");
        const Sizes z = make_sizes(M, nnz, o);
        const Layout L = make_layout(z, P->vsize, workspace);
        if (((uintptr_t)workspace & 255) || workspace_bytes < L.total) throw Fail{LIBRA_ERR_BUFFER};
        const int n = (int)nnz, nw = (int)z.nw;
        const int vsize = P->vsize;
        const uint8_t *val = reinterpret_cast<const uint8_t *>(d_val);
        int colbits = 1;
        while ((1ll << colbits) < Kc) ++colbits;
        const int tau_a = o.mode == LIBRA_MODE_DENSE_ONLY ? 1 : o.mode == LIBRA_MODE_SCALAR_ONLY ? W + 1 : o.tau_spmm;
        Rule R{o.mode, o.fill && o.mode == LIBRA_MODE_HYBRID ? 1 : 0, tau_a, o.tau_sddmm, o.Ts, o.Cs, o.short_len, o.build_spmm ? 1 : 0, o.build_sddmm ? 1 : 0, o.sddmm_Ts};

        // ---- 1. census: the nonzeros of every window in (column, row) order ----
        fill_bytes(L.ctr, 0, (size_t)((char *)(L.hist + (size_t)nw * W) - (char *)L.ctr), s);
        hipLaunchKernelGGL(k_win_ptr, dim3(blocks_for(nw + 1, 256)), dim3(256), 0, s, d_rowptr, M, nw, L.win_ptr, L.ctr);
        const int tiles = tile_count(n);
        hipLaunchKernelGGL(k_rows, dim3(blocks_for(n, ROWS_CHUNK)), dim3(256), 0, s, d_rowptr, d_col, M, Kc, n, L.row_of, L.ctr);
        hipLaunchKernelGGL(k_tile_splits, dim3(blocks_for((int64_t)(tiles + 1) * W, 256)), dim3(256), 0, s, d_rowptr, d_col, L.win_ptr, M, Kc, n, nw, tiles, L.tiles);
        hipLaunchKernelGGL(k_tile_sort, dim3((unsigned)tiles), dim3(TILE_THREADS), 0, s, d_rowptr, d_col, L.win_ptr, L.row_of, M, L.tiles, L.ctr, L.scol, L.spos, L.vmask, L.hist);
        // ---- 2. per window: dense vectors and blocks ----
        hipLaunchKernelGGL(k_window_counts, dim3(blocks_for((int64_t)nw + 1, 256)), dim3(256), 0, s, L.hist, nw, R, L.a.ndv, L.a.nb, L.d.ndv, L.d.nb, L.ctr);
        const bool share_rule = o.build_sddmm && o.mode == LIBRA_MODE_HYBRID && o.sddmm_min_dense_pct > 0;
        if (share_rule)
            hipLaunchKernelGGL(k_share_rule, dim3(blocks_for(nw, 256)), dim3(256), 0, s, L.ctr, nnz, o.sddmm_min_dense_pct, nw, L.d.ndv, L.d.nb);
        scan_all(L, {{L.a.nb, L.a.blkptr, (int64_t)nw + 1}, {L.d.nb, L.d.blkptr, (int64_t)nw + 1}}, s);
        int32_t size[7];
        u64 ctr[C_COUNT];
        hip_ok(hipMemcpyAsync(ctr, L.ctr, sizeof ctr, hipMemcpyDeviceToHost, s));
        peek_all(L.sizes, {L.a.blkptr + nw, L.d.blkptr + nw}, size, s);
        if (hipGetLastError() != hipSuccess) throw Fail{LIBRA_ERR_HIP};
        if (ctr[C_ERR] & 1) throw Fail{LIBRA_ERR_COLUMN};
        if (ctr[C_ERR] & 2) throw Fail{LIBRA_ERR_UNSORTED};
        const int nv = (int)ctr[C_NV];
        if (nv < 1 || nv > n) throw Fail{LIBRA_ERR_HIP};
        const int nbA = size[0], nbD = size[1];
        if (nbA < 0 || nbD < 0 || nbA > z.nbmax || nbD > z.nbmax) throw Fail{LIBRA_ERR_HIP};
        if (share_rule && share_rule_fires(o, (int64_t)ctr[C_DNNZ_D], nnz)) {
            if (nbD != 0) throw Fail{LIBRA_ERR_HIP};
            fill_bytes(L.ctr + C_DV_D, 0, 2 * sizeof(u64), s);              // C_DV_D and C_PAD_D are neighbours
        }
        mark("census, window counts");
        // ---- 3. slots, blocks, packed values ----
        if (nbA + nbD > 0) {
            fill_bytes(L.a.slotvec, 0xff, (size_t)nbA * KB * sizeof(int32_t), s);
            fill_bytes(L.d.slotvec, 0xff, (size_t)nbD * KB * sizeof(int32_t), s);
            fill_bytes(L.dense, 0, (size_t)n + 1, s);
            Tiles parts = L.tiles;
            if (ctr[C_WIDE])
                hipLaunchKernelGGL(k_tail_groups, dim3(blocks_for(tiles, TAIL_GROUP)), dim3(256), 0, s, parts, tiles);
            else
                parts.group = nullptr;
            hipLaunchKernelGGL(k_dense_vectors, dim3((unsigned)tiles), dim3(TILE_THREADS), 0, s, L.win_ptr, L.row_of, parts, L.spos, L.vmask, L.hist,
                               L.a.ndv, L.a.blkptr, L.d.ndv, L.d.blkptr, R, L.a.slotvec, L.d.slotvec, L.dense);
        }
        const int nbs[2] = {nbA, nbD};
        const SubOut *subs[2] = {&L.a, &L.d};
        for (int k = 0; k < 2; ++k) {
            const SubOut &S = *subs[k];
            const int nb = nbs[k];
            if (nb == 0) {
                fill_bytes(S.blk_valptr, 0, sizeof(int32_t), s);
                continue;
            }
            hipLaunchKernelGGL(k_blocks, dim3(blocks_for((int64_t)nb * 16, 256)), dim3(256), 0, s, S.slotvec, L.scol, L.vmask, nb,
                               S.blk_cols, S.bitmap, S.blknnz, S.blkmask, S.blkncols);
            scan_all(L, {{S.blknnz, S.blk_valptr, (int64_t)nb + 1}}, s);
            hipLaunchKernelGGL(k_block_values, dim3(blocks_for((int64_t)nb * 16, 256)), dim3(256), 0, s, S.slotvec, L.vmask, S.bitmap,
                               S.blk_valptr, L.spos, val, vsize, nb, S.dense_perm, S.dense_val);
        }
        // ---- 4. residual nonzeros and tasks ----
        auto residual = [&](const SubOut &S, int nb, unsigned bit) {
            if (nb == 0) return Residual{L.dense, nullptr, bit};
            size_t sz = L.tmp_bytes;
            hip_ok(rocprim::exclusive_scan(L.tmp, sz, rocprim::make_transform_iterator((const uint8_t *)L.dense, NotDense{bit}), S.rescan, (int32_t)0, (size_t)n + 1,
                                           rocprim::plus<int32_t>(), s));
            return Residual{L.dense, S.rescan, bit};
        };
        const Residual resA = residual(L.a, nbA, 1u), resD = residual(L.d, nbD, 2u);
        hipLaunchKernelGGL(k_window_sizes, dim3(std::min(blocks_for(nw, 256 / W), 1024u)), dim3(256), 0, s, d_rowptr, resA, M, nw, R, L.a.blkptr, L.d.blkptr,
                           L.a.ntasks, L.nzero, L.nres, L.d.ntasks, L.ctr);
        scan_all(L, {{L.a.ntasks, L.a.tbase, (int64_t)nw + 1}, {L.nzero, L.zbase, (int64_t)nw + 1}, {L.nres, L.resptr, (int64_t)nw + 1}, {L.d.ntasks, L.d.tbase, (int64_t)nw + 1}}, s);
        peek_all(L.sizes, {L.a.tbase + nw, L.d.tbase + nw, L.zbase + nw, L.a.blk_valptr + nbA, L.d.blk_valptr + nbD}, size, s);
        const int ntA = size[0], ntD = size[1], nz = size[2], dnnzA = size[3], dnnzD = size[4];
        const int nresA = o.build_spmm ? n - dnnzA : 0, nresD = o.build_sddmm ? n - dnnzD : 0;
        if (ntA < 0 || ntA > z.tasks_a_max || ntD < 0 || ntD > z.tasks_d_max || nz < 0 || nz > M || nresA < 0 || nresA > n || nresD < 0 ||
            nresD > n || dnnzA < 0 || dnnzA > n || dnnzD < 0 || dnnzD > n)
            throw Fail{LIBRA_ERR_HIP};
        hipLaunchKernelGGL(k_window_tasks, dim3(std::min(blocks_for(nw, 2), 1u << 22)), dim3(128), 0, s, d_rowptr, resA, M, nw, R,
                           L.a.blkptr, L.a.blkmask, L.a.blkncols, L.d.blkptr, L.d.blkncols, L.a.tbase, L.zbase, L.resptr, L.d.tbase,
                           L.a.tasks, L.zero_rows, L.rowbase, L.d.tasks);
        const int64_t ngroups = (nw + LIBRA_LOCALITY_WINDOWS - 1) / LIBRA_LOCALITY_WINDOWS, nsample = share_samples(ngroups);
        hipLaunchKernelGGL(k_share, dim3(std::min(blocks_for(n, SHARE_SAMPLES), 1024u)), dim3(SHARE_SAMPLES), 0, s, L.win_ptr, L.scol, L.vmask, nw, ngroups, (int)nsample, L.ctr);
        auto fill_residuals = [&](const ResidualOut &a, const ResidualOut &d) {
            auto run = [&](auto tag) {
                typedef decltype(tag) V;
                hipLaunchKernelGGL((k_residual_fill<V>), dim3(blocks_for(n, 256)), dim3(256), 0, s, d_col, (const V *)d_val, n, R, L.row_of, resA, L.rowbase, a, resD, d);
            };
            if (vsize == 2) run(uint16_t{});
            else run(uint32_t{});
        };
        const ResidualOut arraysA{L.a.res_perm, L.a.res_row, L.a.res_col, L.a.res_val, nullptr, nullptr}, arraysD{L.d.res_perm, L.d.res_row, L.d.res_col, L.d.res_val, nullptr, nullptr};
        if (keep_host_copy) fill_residuals(arraysA, arraysD);                  // otherwise when the plan's device copy has its places
        if (o.build_spmm && ntA > 0)
            hipLaunchKernelGGL(k_task_cols, dim3(blocks_for(ntA, 256)), dim3(256), 0, s, L.a.tasks, ntA, d_rowptr, L.rowbase, d_col, resA, L.task_col);
        const int nsegD = o.build_sddmm ? piece_count(nresD, o.sddmm_Cs) : 0;
        if (nsegD > 0)
            hipLaunchKernelGGL(k_segment_cols, dim3(blocks_for(nsegD, 256)), dim3(256), 0, s, L.row_of, d_col, resD, n, nresD, o.sddmm_Cs, nsegD, L.seg_col);
        const bool order_here = (int64_t)ntA + ntD + nsegD >= DEVICE_ORDER_MIN;
        // small tables, which the host orders, come there with the counters: packed on the device, one copy, one wait
        struct Part { const void *from; size_t bytes, at; };
        std::vector<Part> parts;
        size_t packed = 0;
        auto part = [&](const void *from, size_t bytes) {
            parts.push_back({from, bytes, packed});
            packed += align256(bytes);
            return parts.size() - 1;
        };
        part(L.ctr, sizeof ctr);
        const bool staged = !order_here && !keep_host_copy;
        if (staged) {
            if (o.build_spmm) {
                part(L.a.tasks, (size_t)ntA * sizeof(libra_task_t));
                part(L.task_col, (size_t)ntA * 4);
                part(L.a.blk_valptr, ((size_t)nbA + 1) * 4);
            }
            if (o.build_sddmm) {
                part(L.d.tasks, (size_t)ntD * sizeof(libra_task_t));
                part(L.seg_col, (size_t)nsegD * 4);
                part(L.d.blk_valptr, ((size_t)nbD + 1) * 4);
            }
        }
        if (packed > stage_bytes(z)) throw Fail{LIBRA_ERR_HIP};
        std::vector<char> host(packed);
        {
            DeviceCopies copies;
            for (const Part &q : parts) copies.add(L.stage + q.at, q.from, q.bytes);
            if (!copies.flush(s)) throw Fail{LIBRA_ERR_HIP};
            hip_ok(hipMemcpyAsync(host.data(), L.stage, packed, hipMemcpyDeviceToHost, s));
        }
        hip_ok(hipStreamSynchronize(s));
        if (hipGetLastError() != hipSuccess) throw Fail{LIBRA_ERR_HIP};
        std::memcpy(ctr, host.data(), sizeof ctr);
        P->stats.device_seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
        mark("blocks, residual, tasks");

        // ---- sizes; small task tables come to the host, which orders them; large ones and the big arrays only on request ----
        SubPlan &sa = P->spmm, &sd = P->sddmm;
        const int nts[2] = {ntA, ntD}, nres2[2] = {nresA, nresD}, dn[2] = {dnnzA, dnnzD};
        SubPlan *hs[2] = {&sa, &sd};
        P->host_arrays = keep_host_copy != 0;
        size_t next = 1;
        auto unpack = [&](auto &to) {
            const Part &q = parts[next++];
            to.resize(q.bytes / sizeof(to[0]));
            if (q.bytes) std::memcpy(to.data(), host.data() + q.at, q.bytes);
        };
        for (int k = 0; k < 2; ++k) {
            if (!(k == 0 ? o.build_spmm : o.build_sddmm)) continue;
            const SubOut &S = *subs[k];
            SubPlan &H = *hs[k];
            H.n.blocks = nbs[k]; H.n.col_slots = (int64_t)nbs[k] * KB; H.n.bitmap_words = (int64_t)nbs[k] * 4;
            H.n.dense = dn[k]; H.n.res = nres2[k]; H.n.zero_rows = k == 0 ? nz : 0;
            if (staged) {
                unpack(H.tasks);
                if (k == 0) unpack(H.task_col);
                else unpack(H.seg_col);
                unpack(H.blk_valptr);
                continue;
            }
            if (!order_here || keep_host_copy) fetch(H.tasks, S.tasks, (size_t)nts[k], s);
            if (!order_here && k == 0) fetch(H.task_col, L.task_col, (size_t)nts[k], s);
            if (!order_here && k == 1) fetch(H.seg_col, L.seg_col, (size_t)nsegD, s);
            if (!order_here || keep_host_copy) fetch(H.blk_valptr, S.blk_valptr, (size_t)nbs[k] + 1, s);
            if (!keep_host_copy) continue;
            fetch(H.win_blkptr, S.blkptr, (size_t)nw + 1, s);
            fetch(H.blk_cols, S.blk_cols, (size_t)nbs[k] * KB, s);
            fetch(H.blk_bitmap, S.bitmap, (size_t)nbs[k] * 4, s);
            fetch(H.dense_perm, S.dense_perm, (size_t)dn[k], s);
            fetch(H.dense_val, S.dense_val, (size_t)dn[k] * vsize, s);
            fetch(H.res_perm, S.res_perm, (size_t)nres2[k], s);
            fetch(H.res_row, S.res_row, (size_t)nres2[k], s);
            fetch(H.res_col, S.res_col, (size_t)nres2[k], s);
            fetch(H.res_val, S.res_val, (size_t)nres2[k] * vsize, s);
        }
        if (o.build_spmm && keep_host_copy) {
            fetch(sa.win_resptr, L.resptr, (size_t)nw + 1, s);
            fetch(sa.zero_rows, L.zero_rows, (size_t)nz, s);
        }
        hip_ok(hipStreamSynchronize(s));
        sa.dense_vectors = (int64_t)ctr[C_DV_A]; sa.pad_slots = (int64_t)ctr[C_PAD_A];
        sd.dense_vectors = (int64_t)ctr[C_DV_D]; sd.pad_slots = (int64_t)ctr[C_PAD_D];
        sa.short_rows = (int64_t)ctr[C_SHORT]; sa.long_rows = (int64_t)ctr[C_LONG]; sa.split_rows = (int64_t)ctr[C_SPLIT];
        P->stats.n_vectors = nv;
        P->stats.n_vectors_nnz1 = (int64_t)ctr[C_NNZ1];
        mark("copies to the host");
        const int64_t share[2] = {(int64_t)ctr[C_TOGETHER], (int64_t)ctr[C_APART]};
        const TaskView va{L.a.tasks, ntA, 1, 0}, vd{L.d.tasks, ntD, o.sddmm_Cs, nresD};
        auto order = [&](bool heavy_first, bool xcd, bool segments_by_column) {
            int ends[2] = {0, 0};
            const int64_t max_group = (nw - 1) / LIBRA_LOCALITY_WINDOWS;
            if (o.build_spmm) {
                Orderer a{L, s, va, L.task_col, colbits};
                if (heavy_first) {
                    a.heaviest_first(ntA, L.o.ord);
                    ends[0] = xcd ? a.grouped(L.o.ord, ntA, max_group, L.o.order_a)
                              : segments_by_column ? a.by_column(L.o.ord, ntA, true, L.o.order_a) : a.copy(L.o.ord, ntA, L.o.order_a);
                } else {
                    a.identity(ends[0] = ntA, 0, L.o.order_a);
                }
            }
            if (o.build_sddmm) {
                Orderer d{L, s, vd, L.seg_col, colbits};
                if (heavy_first) {
                    d.heaviest_first(ntD, L.o.ord);
                    ends[1] = xcd ? d.grouped(L.o.ord, ntD, max_group, L.o.order_d) : d.copy(L.o.ord, ntD, L.o.order_d);
                    d.identity(nsegD, ntD, L.o.ord);
                    int32_t *segs = L.o.order_d + ends[1];
                    ends[1] += xcd ? d.grouped(L.o.ord, nsegD, nsegD / LIBRA_LOCALITY_SEGMENTS, segs)
                               : segments_by_column ? d.by_column(L.o.ord, nsegD, false, segs) : d.copy(L.o.ord, nsegD, segs);
                } else {
                    d.identity(ends[1] = ntD + nsegD, 0, L.o.order_d);
                }
            }
            sa.n.tasks = ends[0];
            sd.n.tasks = ends[1];
            sa.n_window_tasks = ends[0] - (int64_t)ctr[C_SEGMENTS];        // empty tasks count as windows there, as segments here
            sa.n_chunk_tasks = (int64_t)ctr[C_SEGMENTS];
            sd.n_window_tasks = ntD;
            sd.n_chunk_tasks = ends[1] - ntD;
            if (!keep_host_copy) return;
            for (int k = 0; k < 2; ++k) {
                if (!(k == 0 ? o.build_spmm : o.build_sddmm)) continue;
                SubPlan &H = *hs[k];
                std::vector<int32_t> at;
                fetch(at, k == 0 ? L.o.order_a : L.o.order_d, (size_t)ends[k], s);
                hip_ok(hipStreamSynchronize(s));
                std::vector<libra_task_t> out(at.size());
                for (size_t i = 0; i < at.size(); ++i) out[i] = task_at(H.tasks, at[i], o.sddmm_Cs, nresD, k == 0 ? LIBRA_TASK_WINDOW : LIBRA_TASK_CHUNK);
                H.tasks.swap(out);
            }
        };
        if (order_here) finish_plan(P, nullptr, share, order);
        else finish_plan(P, nullptr, share);
        mark("task order, statistics");
        if (plan_buf) {
            // the plan's device copy straight from the workspace: no round trip through host memory
            auto src = [&](const SubOut &S, const TaskView &v, const int32_t *list, int empty_kind, const int32_t *zero_rows) {
                DeviceSource d{S.blk_cols, S.blk_valptr, S.dense_perm, keep_host_copy ? S.res_perm : nullptr, keep_host_copy ? S.res_row : nullptr, S.res_col, zero_rows,
                               reinterpret_cast<const uint64_t *>(S.bitmap), S.dense_val, S.res_val, d_rowptr, rows_here ? L.medium_rows : nullptr, nullptr, nullptr};
                if (order_here)
                    d.write_tasks = [&S, v, list, empty_kind, s](DevTask *out, int64_t n) {
                        const int per_die = (int)((n + XC - 1) / XC);
                        hipLaunchKernelGGL(k_order_records, dim3(blocks_for((int64_t)per_die * XC, 256)), dim3(256), 0, s, v, list, (int)n, per_die,
                                           (const int32_t *)S.blk_valptr, empty_kind, out);
                    };
                return d;
            };
            DeviceSource source_a = src(L.a, va, L.o.order_a, LIBRA_TASK_WINDOW, L.zero_rows);
            if (!keep_host_copy)
                source_a.write_residuals = [&](const SubPlanDev &a, const SubPlanDev &d) {
                    ResidualOut to_a{const_cast<int32_t *>(a.res_perm), nullptr, nullptr, nullptr, (unsigned char *)a.res_ent, nullptr};
                    ResidualOut to_d{const_cast<int32_t *>(d.res_perm), const_cast<int32_t *>(d.res_row), L.d.res_col, L.d.res_val, nullptr, const_cast<int32_t *>(d.res_base)};
                    const bool whole = nresD == n;
                    if (whole) to_d.entries = (unsigned char *)d.res_ent;
                    fill_residuals(to_a, to_d);
                    if (nresD > 0 && !whole)
                        pack_sddmm_entries(vsize, L.d.res_col, L.d.res_val, d.res_row, nresD, d.res_ent, const_cast<int32_t *>(d.res_base), s);
                };
            if (int rc = adopt_device_arrays(P, source_a, src(L.d, vd, L.o.order_d, LIBRA_TASK_CHUNK, nullptr),
                                             plan_buf, plan_bytes, stream)) throw Fail{rc};
        }
        mark("plan buffer written");
        P->stats.plan_seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    } catch (const Fail &f) {
        (void)hipStreamSynchronize(s);       // queued passes may still use the workspace the caller is about to free
        delete P;
        return f.code;
    } catch (...) {
        (void)hipStreamSynchronize(s);
        delete P;
        return LIBRA_ERR_NOMEM;
    }
    *out = P;
    return LIBRA_OK;
}

// ------------------------------------------------------------------------------------------
// Transposition of a CSR pattern on the device (the backward pass of SpMM multiplies by the transposed matrix).
// ------------------------------------------------------------------------------------------
namespace {
// one wave per 16 rows: key = (column, CSR position); a stable sort by the column (the positions ascend already) lists the nonzeros column by column, rows ascending
__global__ __launch_bounds__(64) void k_transpose_keys(const int32_t *rowptr, const int32_t *col, int64_t M, u64 *key, int32_t *row_of) {
    const int lane = threadIdx.x;
    for (int64_t w = blockIdx.x; w * W < M; w += gridDim.x) {
        for (int r = 0; r < W; ++r) {
            const int64_t i = w * W + r;
            if (i >= M) break;
            const int s = rowptr[i], e = rowptr[i + 1];
            for (int p = s + lane; p < e; p += 64) {
                key[p] = ((u64)(uint32_t)col[p] << 32) | (u64)(uint32_t)p;
                row_of[p] = (int32_t)i;
            }
        }
    }
}
__global__ __launch_bounds__(256) void k_transpose_fill(const u64 *skey, const int32_t *row_of, int n, int32_t *col_t, int32_t *perm_t) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n) return;
    const int p = (int)(skey[q] & 0xffffffffull);
    perm_t[q] = p;
    col_t[q] = row_of[p];
}
// rowptr_t[c] = first sorted position whose column is >= c
__global__ __launch_bounds__(256) void k_transpose_rowptr(const u64 *skey, int n, int64_t Kc, int32_t *rowptr_t) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c > Kc) return;
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = lo + ((hi - lo) >> 1);       // lo + hi may pass 2^31
        if ((int64_t)(skey[mid] >> 32) < c) lo = mid + 1; else hi = mid;
    }
    rowptr_t[c] = lo;
}

struct TLayout { u64 *key_in, *key_out; int32_t *row_of; void *tmp; size_t tmp_bytes, total; };
TLayout transpose_layout(int64_t nnz, void *base) {
    TLayout L{};
    Arena A{(char *)base};
    const size_t n = (size_t)std::max<int64_t>(nnz, 1);
    L.key_in = A.take<u64>(n);
    L.key_out = A.take<u64>(n);
    L.row_of = A.take<int32_t>(n);
    size_t sz = 0;
    (void)rocprim::radix_sort_keys(nullptr, sz, (u64 *)nullptr, (u64 *)nullptr, n, 0, 64);
    L.tmp_bytes = sz + 4096;
    L.tmp = A.take<uint8_t>(L.tmp_bytes);
    L.total = align256(A.off) + 256;
    return L;
}
}  // namespace

extern "C" int libra_csr_transpose_workspace(int64_t nnz, size_t *bytes) {
    if (!bytes) return LIBRA_ERR_NULL;
    if (nnz < 0) return LIBRA_ERR_SHAPE;
    if (nnz >= (1ll << 31) - 64) return LIBRA_ERR_TOO_LARGE;
    *bytes = transpose_layout(nnz, nullptr).total;
    return LIBRA_OK;
}

namespace {
// The passes of the transposition on a workspace that is known to be large enough and aligned.  Only launches kernels
// and the sort on `s`; nothing is allocated and the stream is not synchronised.
int transpose_passes(int64_t M, int64_t Kc, int n, const int32_t *d_rowptr, const int32_t *d_col, int32_t *d_rowptr_t,
                     int32_t *d_col_t, int32_t *d_perm_t, const TLayout &L, hipStream_t s) {
    int colbits = 1;
    while ((1ll << colbits) < Kc) ++colbits;
    const int64_t nw = (M + W - 1) / W;
    // a launch has fewer than 2^32 threads: of large matrices a wave takes several groups of rows
    hipLaunchKernelGGL(k_transpose_keys, dim3((unsigned)std::min<int64_t>(nw, 1 << 24)), dim3(64), 0, s, d_rowptr, d_col, M, L.key_in, L.row_of);
    size_t sz = L.tmp_bytes;
    if (rocprim::radix_sort_keys(L.tmp, sz, L.key_in, L.key_out, (size_t)n, 32u, (unsigned)(32 + colbits), s) != hipSuccess) return LIBRA_ERR_HIP;
    hipLaunchKernelGGL(k_transpose_fill, dim3(blocks_for(n, 256)), dim3(256), 0, s, L.key_out, L.row_of, n, d_col_t, d_perm_t);
    hipLaunchKernelGGL(k_transpose_rowptr, dim3(blocks_for(Kc + 1, 256)), dim3(256), 0, s, L.key_out, n, Kc, d_rowptr_t);
    return hipGetLastError() == hipSuccess ? LIBRA_OK : LIBRA_ERR_HIP;
}

int transpose_args(int64_t M, int64_t Kc, int64_t nnz, const int32_t *d_rowptr, const int32_t *d_col, int32_t *d_rowptr_t,
                   int32_t *d_col_t, int32_t *d_perm_t) {
    if (!d_rowptr || !d_rowptr_t) return LIBRA_ERR_NULL;
    if (M < 1 || Kc < 1 || nnz < 0) return LIBRA_ERR_SHAPE;
    if (M >= (1ll << 31) - 64 || Kc >= (1ll << 31) - 64 || nnz >= (1ll << 31) - 64) return LIBRA_ERR_TOO_LARGE;
    if (nnz > 0 && (!d_col || !d_col_t || !d_perm_t)) return LIBRA_ERR_NULL;
    return LIBRA_OK;
}

// rowptr of a transposed matrix without nonzeros: Kc + 1 zeros, written by a kernel (a memset node in a captured graph
// is not reliable on replays)
__global__ __launch_bounds__(256) void k_zero_i32(int32_t *p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}
}  // namespace

extern "C" int libra_csr_transpose_device(int64_t M, int64_t Kc, int64_t nnz, const int32_t *d_rowptr, const int32_t *d_col,
                                          int32_t *d_rowptr_t, int32_t *d_col_t, int32_t *d_perm_t,
                                          void *workspace, size_t workspace_bytes, void *stream) {
    if (int rc = transpose_args(M, Kc, nnz, d_rowptr, d_col, d_rowptr_t, d_col_t, d_perm_t)) return rc;
    hipStream_t s = (hipStream_t)stream;
    if (nnz == 0) {
        hipLaunchKernelGGL(k_zero_i32, dim3(blocks_for(Kc + 1, 256)), dim3(256), 0, s, d_rowptr_t, Kc + 1);
        return hipGetLastError() == hipSuccess ? LIBRA_OK : LIBRA_ERR_HIP;
    }
    if (!workspace) return LIBRA_ERR_NULL;
    const TLayout L = transpose_layout(nnz, workspace);
    if (((uintptr_t)workspace & 255) || workspace_bytes < L.total) return LIBRA_ERR_BUFFER;
    if (int rc = transpose_passes(M, Kc, (int)nnz, d_rowptr, d_col, d_rowptr_t, d_col_t, d_perm_t, L, s)) return rc;
    if (hipStreamSynchronize(s) != hipSuccess) return LIBRA_ERR_HIP;     // the workspace may go now
    return LIBRA_OK;
}

// ------------------------------------------------------------------------------------------
// The same transposition for callers that cannot allocate: its workspace is a fixed array in device memory that every
// GPU the library runs on holds from the moment the code object is loaded until the process ends.
// ------------------------------------------------------------------------------------------
namespace {
constexpr size_t STATIC_SCRATCH_BYTES = (size_t)LIBRA_TRANSPOSE_STATIC_MAX_NNZ * 40;      // keys in, keys out, rows, sort storage
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

// In host code the array's name stands for the symbol, not for device memory: its address on the current device comes from
// hipGetSymbolAddress, once per device (every GPU has its own copy at its own address).
constexpr int MAX_DEVICES = 64;
std::mutex scratch_mutex;
void *scratch_ptr[MAX_DEVICES];

int static_scratch(void **out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return LIBRA_ERR_HIP;
    std::lock_guard<std::mutex> lock(scratch_mutex);
    if (!scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return LIBRA_ERR_HIP;
        scratch_ptr[dev] = p;
    }
    *out = scratch_ptr[dev];
    return LIBRA_OK;
}
}  // namespace

extern "C" int libra_csr_transpose_device_static(int64_t M, int64_t Kc, int64_t nnz, const int32_t *d_rowptr, const int32_t *d_col,
                                                 int32_t *d_rowptr_t, int32_t *d_col_t, int32_t *d_perm_t, void *stream) {
    if (int rc = transpose_args(M, Kc, nnz, d_rowptr, d_col, d_rowptr_t, d_col_t, d_perm_t)) return rc;
    if (nnz > LIBRA_TRANSPOSE_STATIC_MAX_NNZ) return LIBRA_ERR_TOO_LARGE;
    hipStream_t s = (hipStream_t)stream;
    if (nnz == 0) {
        hipLaunchKernelGGL(k_zero_i32, dim3(blocks_for(Kc + 1, 256)), dim3(256), 0, s, d_rowptr_t, Kc + 1);
        return hipGetLastError() == hipSuccess ? LIBRA_OK : LIBRA_ERR_HIP;
    }
    void *ws = nullptr;
    if (int rc = static_scratch(&ws)) return rc;
    const TLayout L = transpose_layout(nnz, ws);
    if (L.total > STATIC_SCRATCH_BYTES) return LIBRA_ERR_TOO_LARGE;      // the sort asked for more storage than the array was sized for
    // every array of the layout is written by a pass before a later pass reads it: nothing of the previous call's
    // contents is read, so nothing has to be cleared
    return transpose_passes(M, Kc, (int)nnz, d_rowptr, d_col, d_rowptr_t, d_col_t, d_perm_t, L, s);
}

// A's values in the plan: new CSR-ordered values into the packed arrays of both operators, and values that come in another
// order of the same nonzeros (the transposed matrix of a training step).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstring>

#include <rocprim/rocprim.hpp>

#include "plan_internal.h"

using namespace libra;

namespace {

// dst[i * stride + offset] (as T) = src[perm[i]]: new values into records
template <class T>
__global__ __launch_bounds__(256) void scatter_values_kernel(const T *src, const int32_t *perm, int64_t n, void *dst, int stride, int offset) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        *reinterpret_cast<T *>(reinterpret_cast<char *>(dst) + i * stride + offset) = src[perm[i]];
}

// new values into the 16-bit SDDMM output records, which carry their own CSR position (and keep their stage slot)
__global__ __launch_bounds__(256) void refresh_record_values_kernel(const uint16_t *src, int64_t n, SdPv *rec) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        rec[i].val = (rec[i].val & 0xffff0000u) | src[rec[i].perm];
}

// Where value i of the blocked residual entries lies; values i .. i + 7 of one block follow each other.
template <class V>
__device__ inline unsigned char *entry_value(unsigned char *res, int64_t i) {
    return res + (i / RES_BLOCK) * (RES_BLOCK * (4 + (int)sizeof(V))) + RES_BLOCK * 4 + (i % RES_BLOCK) * (int)sizeof(V);
}
template <class V> constexpr int GROUP = 16 / (int)sizeof(V);       // values that move together
static_assert(RES_BLOCK % GROUP<uint16_t> == 0 && RES_BLOCK % GROUP<uint32_t> == 0, "a group stays inside one block");

// The packed dense values and the values of the blocked entries of a sub-plan, one launch: a thread takes 16 bytes of consecutive
// destinations, so that the permutation arrives in 16-byte loads and the values leave in one store (GAT graph, 16 bits: 168 us with
// a value per thread, 103).  IDENTITY: entry i takes value i (a template argument: as a test of the pointer in the loop the copy of
// 25 M values took 26 us and not 16).
template <class V, bool IDENTITY>
__global__ __launch_bounds__(256) void place_values_kernel(const V *src, const int32_t *dense_perm, int64_t nd, V *dense, const int32_t *res_perm, int64_t nr, unsigned char *res) {
    constexpr int G = GROUP<V>;
    const int64_t gd = (nd + G - 1) / G, gr = (nr + G - 1) / G, nthreads = (int64_t)gridDim.x * blockDim.x;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < gd + gr; k += nthreads) {
        const bool to_dense = k < gd;
        const int64_t i = (to_dense ? k : k - gd) * G, n = to_dense ? nd : nr;
        const int32_t *perm = to_dense ? dense_perm : res_perm;
        unsigned char *dst = to_dense ? reinterpret_cast<unsigned char *>(dense + i) : entry_value<V>(res, i);
        if (i + G > n) {
            for (int64_t q = i; q < n; ++q, dst += sizeof(V)) *reinterpret_cast<V *>(dst) = src[IDENTITY ? q : (int64_t)perm[q]];
            continue;
        }
        V v[G];
        if constexpr (!IDENTITY) {
            int32_t p[G];
#pragma unroll
            for (int e = 0; e < G; e += 4) {
                const int4 x = *reinterpret_cast<const int4 *>(perm + i + e);
                p[e] = x.x; p[e + 1] = x.y; p[e + 2] = x.z; p[e + 3] = x.w;
            }
#pragma unroll
            for (int e = 0; e < G; ++e) v[e] = src[p[e]];
        } else if (((uintptr_t)src & 15) == 0) {
            *reinterpret_cast<uint4 *>(dst) = *reinterpret_cast<const uint4 *>(src + i);
            continue;
        } else {
#pragma unroll
            for (int e = 0; e < G; ++e) v[e] = src[i + e];
        }
        *reinterpret_cast<uint4 *>(dst) = *reinterpret_cast<const uint4 *>(v);
    }
}

inline unsigned grid_for(int64_t threads) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>((threads + 255) / 256, 1 << 16)); }

int place_values(int vdt, const void *src, const int32_t *dense_perm, int64_t nd, void *dense, const int32_t *res_perm, int64_t nr, void *res, hipStream_t s) {
    if (nd + nr == 0) return LIBRA_OK;
    auto run = [&](auto tag) {
        typedef decltype(tag) V;
        const dim3 grid(grid_for(nd / GROUP<V> + nr / GROUP<V> + 2)), block(256);
        if (nd == 0 && !res_perm)
            hipLaunchKernelGGL((place_values_kernel<V, true>), grid, block, 0, s, (const V *)src, dense_perm, nd, (V *)dense, res_perm, nr, (unsigned char *)res);
        else
            hipLaunchKernelGGL((place_values_kernel<V, false>), grid, block, 0, s, (const V *)src, dense_perm, nd, (V *)dense, res_perm, nr, (unsigned char *)res);
    };
    if (vdt == LIBRA_F32) run(uint32_t{});
    else run(uint16_t{});                      // 16-bit values are moved as raw bits
    return hipGetLastError() == hipSuccess ? LIBRA_OK : LIBRA_ERR_HIP;
}

// ---- values in another order of the nonzeros ----
// Destination slots: the packed dense values, padded to whole blocks of entries, then the entries.  Slot j takes value source(j).
// Small matrices gather: an array of sources and place_values_kernel.  Larger ones, whose values do not stay in an L2 (every gathered
// value then costs a line from behind it), are permuted in two passes that read and write runs: the values are cut into chunks and
// the slots into tiles of VALUES values (64 KiB, in LDS); the first pass sorts a chunk by tile and appends each tile's values to the
// tile's part of an intermediate array, the second puts a tile's values into slot order.  Bound by memory: 12 bytes per value of 16
// bits, 16.8 M values at 4.1 TB/s.  The first pass has the runs of its chunk, 8 bytes per tile, in LDS too: two workgroups per compute
// unit up to 2,047 tiles (67 M values of 16 bits, 33.5 M of 32), one from there on.
template <class V> constexpr int VALUES = 65536 / (int)sizeof(V);
// Random permutations, gather / two passes: fp16, 2^20 nonzeros 13 / 23 us, 2^21 20 / 26, 2^22 50 / 28, 2^24 291 / 49, 2^26 1,246 / 322;
// fp32, 2^20 15 / 22, 2^21 30 / 24, 2^22 67 / 31, 2^24 317 / 101: the lines cross where the values are some 5 MB.  (As an index pass of
// torch and set_values, fp16: 15, 25, 59, 309, 1,375.)  Upper bound: the runs of a chunk are listed in LDS beside it; at 2^27 nonzeros, the
// most, fp16 2,624 / 786, fp32 2,696 / 1,860.  The runs are chunks x tiles: the order takes 4.1 bytes per nonzero at 2^24, 5 (fp16) and
// 8 (fp32) at 2^27, where the gathered form takes 4.
constexpr int64_t ORDER_PASSES_MIN_BYTES = 5 << 20, ORDER_PASSES_MAX = 1 << 27;

struct OrderShape {
    int64_t nnz, nd, nd_pad, slots;
    int T;                      // values per chunk and per tile
    int chunks, tiles;
    bool passes;
};
OrderShape order_shape(const libra_plan_t *P) {
    OrderShape h;
    h.nnz = P->nnz;
    h.nd = P->spmm.n.dense;
    h.nd_pad = (h.nd + RES_BLOCK - 1) / RES_BLOCK * RES_BLOCK;
    h.slots = h.nd_pad + P->spmm.n.res;
    h.T = P->vsize == 4 ? VALUES<uint32_t> : VALUES<uint16_t>;
    h.passes = h.nnz * P->vsize >= ORDER_PASSES_MIN_BYTES && h.nnz <= ORDER_PASSES_MAX;
    h.chunks = (int)((h.nnz + h.T - 1) / h.T);
    h.tiles = (int)((h.slots + h.T - 1) / h.T);
    return h;
}
struct OrderArrays {
    int32_t *source;            // gather: per slot
    uint16_t *in_chunk;         // passes: per chunk, its values' places in the chunk, tile by tile
    uint16_t *in_tile;          //         per intermediate value, its slot's place in the tile
    int32_t *tile_first;        //         tiles + 1: intermediate values of a tile
    int32_t *run;               //         chunks x (tiles + 1): the run of each tile among a chunk's values ...
    int32_t *to;                //         chunks x tiles: ... and where it goes, minus where it starts
    size_t total;
};
struct Taker {
    char *base;
    size_t off = 0;
    template <class T> T *take(size_t n) {
        T *p = base ? reinterpret_cast<T *>(base + off) : nullptr;
        off = (off + n * sizeof(T) + 16 + 255) & ~(size_t)255;
        return p;
    }
};
OrderArrays order_arrays(const OrderShape &h, void *base) {
    OrderArrays a{};
    Taker t{(char *)base};
    if (!h.passes) {
        a.source = t.take<int32_t>((size_t)h.slots);
    } else {
        a.in_chunk = t.take<uint16_t>((size_t)h.nnz);
        a.in_tile = t.take<uint16_t>((size_t)h.nnz);
        a.tile_first = t.take<int32_t>((size_t)h.tiles + 1);
        a.run = t.take<int32_t>((size_t)h.chunks * (h.tiles + 1));
        a.to = t.take<int32_t>((size_t)h.chunks * h.tiles);
    }
    a.total = t.off;
    return a;
}
struct OrderWork {
    uint32_t *key_in, *key_out;
    int32_t *slot_in, *slot_out, *first, *bad;
    uint8_t *seen;              // gather: per value, does a slot take it?
    void *tmp;
    size_t tmp_bytes, total;
};
OrderWork order_work(const OrderShape &h, void *base) {
    OrderWork w{};
    Taker t{(char *)base};
    w.bad = t.take<int32_t>(1);
    if (h.passes) {
        const size_t n = (size_t)h.nnz;
        w.key_in = t.take<uint32_t>(n);
        w.key_out = t.take<uint32_t>(n);
        w.slot_in = t.take<int32_t>(n);
        w.slot_out = t.take<int32_t>(n);
        w.first = t.take<int32_t>((size_t)h.chunks * h.tiles + 1);
        (void)rocprim::radix_sort_pairs(nullptr, w.tmp_bytes, (uint32_t *)nullptr, (uint32_t *)nullptr, (int32_t *)nullptr, (int32_t *)nullptr, n, 0, 32);
        w.tmp_bytes += 4096;
        w.tmp = t.take<char>(w.tmp_bytes);
    } else {
        w.seen = t.take<uint8_t>((size_t)h.nnz);
    }
    w.total = t.off;
    return w;
}

__global__ __launch_bounds__(256) void k_order_clear(int32_t *bad, uint8_t *seen, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) *bad = 0;
    if (i < n) seen[i] = 0;
}
// the CSR position that slot j holds, and its value's place in the new order (a place out of range is reported and taken as 0)
__device__ inline int source_of(const int32_t *dense_perm, const int32_t *res_perm, int64_t nd, int64_t nd_pad, int64_t slot, const int32_t *order, int64_t nnz, int32_t *bad) {
    const int p = slot < nd_pad ? dense_perm[slot] : res_perm[slot - nd_pad];
    const int q = order[p];
    if (q >= 0 && q < nnz) return q;
    if (bad) *bad = 1;
    return 0;
}
// nonzero i of the slots, without the padding between the two kinds
__device__ inline int64_t slot_of(int64_t i, int64_t nd, int64_t nd_pad) { return i < nd ? i : i - nd + nd_pad; }

__global__ __launch_bounds__(256) void k_order_sources(const int32_t *dense_perm, const int32_t *res_perm, int64_t nd, int64_t nd_pad, int64_t nnz, const int32_t *order,
                                                       int32_t *source, uint8_t *seen, int32_t *bad) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nnz) return;
    const int64_t slot = slot_of(i, nd, nd_pad);
    const int q = source_of(dense_perm, res_perm, nd, nd_pad, slot, order, nnz, bad);
    source[slot] = q;
    seen[q] = 1;
}
// as many slots as values: an order that leaves no value out is a permutation
__global__ __launch_bounds__(256) void k_order_all_seen(const uint8_t *seen, int64_t nnz, int32_t *bad) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nnz && !seen[i]) *bad = 1;
}
__global__ __launch_bounds__(256) void k_order_keys(const int32_t *dense_perm, const int32_t *res_perm, int64_t nd, int64_t nd_pad, int64_t nnz, const int32_t *order,
                                                    int T, int chunks, uint32_t *key, int32_t *slots, int32_t *bad) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nnz) return;
    const int64_t slot = slot_of(i, nd, nd_pad);
    const int q = source_of(dense_perm, res_perm, nd, nd_pad, slot, order, nnz, bad);
    key[i] = (uint32_t)(slot / T) * (uint32_t)chunks + (uint32_t)(q / T);
    slots[i] = (int32_t)slot;
}
// first intermediate value of every (tile, chunk) pair
__global__ __launch_bounds__(256) void k_order_first(const uint32_t *key, int n, int64_t pairs, int32_t *first) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k > pairs) return;
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = lo + ((hi - lo) >> 1);
        if ((int64_t)key[mid] < k) lo = mid + 1; else hi = mid;
    }
    first[k] = lo;
}
// a thread per chunk: its runs.  Every chunk has to be whole: the places that follow from the runs would not be in the arrays otherwise
__global__ __launch_bounds__(64) void k_order_runs(const int32_t *first, int chunks, int tiles, int T, int64_t nnz, int32_t *run, int32_t *to, int32_t *tile_first, int32_t *bad) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= chunks) return;
    int at = 0;
    for (int t = 0; t < tiles; ++t) {
        const int64_t k = (int64_t)t * chunks + c;
        run[(int64_t)c * (tiles + 1) + t] = at;
        to[(int64_t)c * tiles + t] = first[k] - at;
        if (c == 0) tile_first[t] = first[k];
        at += first[k + 1] - first[k];
    }
    run[(int64_t)c * (tiles + 1) + tiles] = at;
    if (c == 0) tile_first[tiles] = (int32_t)nnz;
    if (at != min((int64_t)T, nnz - (int64_t)c * T)) *bad = 1;
}
__global__ __launch_bounds__(256) void k_order_places(const uint32_t *key, const int32_t *slots, const int32_t *dense_perm, const int32_t *res_perm, int64_t nd, int64_t nd_pad,
                                                      int64_t nnz, const int32_t *order, int T, int chunks, int tiles, const int32_t *to, uint16_t *in_chunk, uint16_t *in_tile) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= nnz) return;
    const int t = (int)(key[r] / (uint32_t)chunks), c = (int)(key[r] % (uint32_t)chunks);
    const int q = source_of(dense_perm, res_perm, nd, nd_pad, slots[r], order, nnz, nullptr);
    in_tile[r] = (uint16_t)(slots[r] - t * T);
    in_chunk[(int64_t)c * T + (r - to[(int64_t)c * tiles + t])] = (uint16_t)(q - c * T);
}

constexpr int PASS_THREADS = 1024;
// ... and no two of a chunk's values the same one: then the order is a permutation.  A workgroup per chunk, a bit per value.
__global__ __launch_bounds__(PASS_THREADS) void k_order_chunks_whole(const uint16_t *in_chunk, int64_t nnz, int T, int32_t *bad) {
    __shared__ uint32_t seen[VALUES<uint16_t> / 32];
    const int64_t c0 = (int64_t)blockIdx.x * T;
    const int n = (int)min((int64_t)T, nnz - c0);
    for (int i = threadIdx.x; i < T / 32; i += PASS_THREADS) seen[i] = 0;
    __syncthreads();
    bool twice = false;
    for (int i = threadIdx.x; i < n; i += PASS_THREADS) {
        const unsigned q = in_chunk[c0 + i], bit = 1u << (q % 32);
        twice = twice || (atomicOr(&seen[q / 32], bit) & bit);
    }
    if (twice) *bad = 1;
}

// First pass, a workgroup per chunk.  LDS: the chunk, then the runs' starts and destinations.
template <class V>
__global__ __launch_bounds__(PASS_THREADS) void order_chunks_kernel(const V *src, int64_t nnz, const uint16_t *in_chunk, const int32_t *run, const int32_t *to, int tiles, V *mid) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    constexpr int T = VALUES<V>, G = GROUP<V>;
    V *val = reinterpret_cast<V *>(lds);
    int32_t *start = reinterpret_cast<int32_t *>(lds + sizeof(V) * T), *shift = start + tiles + 1;
    const int64_t c0 = (int64_t)blockIdx.x * T;
    const int n = (int)min((int64_t)T, nnz - c0);
    const int tid = threadIdx.x, lane = tid % 64;
    if (((uintptr_t)src & 15) == 0) {
        for (int i = tid * G; i + G <= n; i += PASS_THREADS * G) *reinterpret_cast<uint4 *>(val + i) = *reinterpret_cast<const uint4 *>(src + c0 + i);
        for (int i = n / G * G + tid; i < n; i += PASS_THREADS) val[i] = src[c0 + i];
    } else {
        for (int i = tid; i < n; i += PASS_THREADS) val[i] = src[c0 + i];
    }
    for (int t = tid; t <= tiles; t += PASS_THREADS) start[t] = run[(int64_t)blockIdx.x * (tiles + 1) + t];
    for (int t = tid; t < tiles; t += PASS_THREADS) shift[t] = to[(int64_t)blockIdx.x * tiles + t];
    __syncthreads();
    // a wave takes a stretch of the chunk's values in tile order and walks along the runs with it
    constexpr int U = 8, STRETCH = T / (PASS_THREADS / 64);
    static_assert(STRETCH % (64 * U) == 0, "whole rounds");
    const int w0 = tid / 64 * STRETCH;
    if (w0 >= n) return;
    int lo = 0, hi = tiles;                              // start[lo] <= w0 < start[hi]
    while (hi - lo > 1) {
        const int mid_run = (lo + hi) >> 1;
        if (start[mid_run] <= w0) lo = mid_run; else hi = mid_run;
    }
    int t = lo;
    for (int i0 = w0; i0 < min(n, w0 + STRETCH); i0 += 64 * U) {
        int place[U];
#pragma unroll
        for (int u = 0; u < U; ++u) place[u] = in_chunk[c0 + min(i0 + 64 * u + lane, n - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + 64 * u + lane;
            if (i < n) {
                while (start[t + 1] <= i) ++t;           // start[tiles] = n ends it
                mid[shift[t] + i] = val[place[u]];
            }
        }
    }
}
// Second pass, a workgroup per tile.
template <class V>
__global__ __launch_bounds__(PASS_THREADS) void order_tiles_kernel(const V *mid, const uint16_t *in_tile, const int32_t *tile_first, int64_t nd, int64_t nd_pad, int64_t slots,
                                                                   V *dense, unsigned char *res) {
    constexpr int T = VALUES<V>, G = GROUP<V>;
    __shared__ __attribute__((aligned(16))) V val[T];
    const int tid = threadIdx.x;
    const int q0 = tile_first[blockIdx.x], q1 = tile_first[blockIdx.x + 1];
    constexpr int U = 8;
    for (int q = q0 + tid; q < q1; q += PASS_THREADS * U) {
        V v[U];
        int place[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = min(q + u * PASS_THREADS, q1 - 1);
            v[u] = mid[k];
            place[u] = in_tile[k];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) val[place[u]] = v[u];         // (the clamped ones write their own value again)
    }
    __syncthreads();
    // whole groups: past the last dense value a group ends inside the array's 16 spare bytes, past the last entry inside its block
    const int64_t s0 = (int64_t)blockIdx.x * T;
    const int n = (int)min((int64_t)T, slots - s0);
    for (int i = tid * G; i < n; i += PASS_THREADS * G) {
        const int64_t slot = s0 + i;
        if (slot < nd_pad && slot >= nd) continue;
        unsigned char *dst = slot < nd_pad ? reinterpret_cast<unsigned char *>(dense + slot) : entry_value<V>(res, slot - nd_pad);
        *reinterpret_cast<uint4 *>(dst) = *reinterpret_cast<const uint4 *>(val + i);
    }
}
template <class V> constexpr size_t chunks_lds(int tiles) { return VALUES<V> * sizeof(V) + ((size_t)2 * tiles + 1) * 4; }

// Lets order_chunks_kernel have the LDS of the most tiles, once per device.  (A size that follows the plan, set before each launch, would
// be another thread's limit.)
template <class V>
bool allow_chunks_lds() {
    static std::atomic<uint64_t> done{0};
    constexpr size_t most = chunks_lds<V>((int)((ORDER_PASSES_MAX + RES_BLOCK + VALUES<V> - 1) / VALUES<V>));
    static_assert(most <= 160 << 10, "the LDS of a compute unit");
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    const uint64_t bit = dev >= 0 && dev < 64 ? 1ull << dev : 0;
    if (done.load(std::memory_order_relaxed) & bit) return true;
    if (hipFuncSetAttribute((const void *)order_chunks_kernel<V>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)most) != hipSuccess) return false;
    done.fetch_or(bit, std::memory_order_relaxed);
    return true;
}
template <class V>
int run_passes(const libra_plan_t *P, const OrderShape &h, const OrderArrays &a, const void *src, void *scratch, hipStream_t s) {
    const SubPlan &sa = P->spmm;
    if (!allow_chunks_lds<V>()) return LIBRA_ERR_HIP;
    hipLaunchKernelGGL((order_chunks_kernel<V>), dim3((unsigned)h.chunks), dim3(PASS_THREADS), chunks_lds<V>(h.tiles), s, (const V *)src, h.nnz, a.in_chunk, a.run, a.to, h.tiles, (V *)scratch);
    hipLaunchKernelGGL((order_tiles_kernel<V>), dim3((unsigned)h.tiles), dim3(PASS_THREADS), 0, s, (const V *)scratch, a.in_tile, a.tile_first, h.nd, h.nd_pad, h.slots,
                       (V *)sa.dev.dense_val, (unsigned char *)sa.dev.res_ent);
    return hipGetLastError() == hipSuccess ? LIBRA_OK : LIBRA_ERR_HIP;
}

int order_args(const libra_plan_t *P) {
    if (!P) return LIBRA_ERR_NULL;
    if (!P->o.build_spmm) return LIBRA_ERR_NOT_BUILT;
    if (!P->dev_base) return LIBRA_ERR_NOT_UPLOADED;
    return LIBRA_OK;
}

}  // namespace

extern "C" int libra_plan_set_values(libra_plan_t *P, const void *vals, int dtype, void *stream) {
    return libra_plan_set_values_for(P, vals, dtype, LIBRA_OP_SPMM | LIBRA_OP_SDDMM, stream);
}

extern "C" int libra_plan_set_values_for(libra_plan_t *P, const void *vals, int dtype, int ops, void *stream) {
    if (!P) return LIBRA_ERR_NULL;
    if (!(ops & (LIBRA_OP_SPMM | LIBRA_OP_SDDMM)) || (ops & ~(LIBRA_OP_SPMM | LIBRA_OP_SDDMM))) return LIBRA_ERR_OPTION;
    if (!vals && P->nnz > 0) return LIBRA_ERR_NULL;
    if (dtype != P->vdt) return LIBRA_ERR_DTYPE;
    if (!P->dev_base) return LIBRA_ERR_NOT_UPLOADED;
    hipStream_t s = (hipStream_t)stream;
    const SubPlan &sa = P->spmm, &sd = P->sddmm;
    if (ops & LIBRA_OP_SPMM) {
        if (int rc = place_values(dtype, vals, sa.dev.dense_perm, sa.n.dense, sa.dev.dense_val, sa.dev.res_perm, sa.n.res, sa.dev.res_ent, s)) return rc;
    }
    if (ops & LIBRA_OP_SDDMM) {
        if (const int64_t n = sd.n.dense) {
            if (sorted_records(P))
                hipLaunchKernelGGL(refresh_record_values_kernel, dim3(grid_for(n)), dim3(256), 0, s, (const uint16_t *)vals, n, (SdPv *)sd.dev.dense_pv);
            else if (dtype != LIBRA_F32)
                hipLaunchKernelGGL((scatter_values_kernel<uint16_t>), dim3(grid_for(n)), dim3(256), 0, s, (const uint16_t *)vals, sd.dev.dense_perm, n, sd.dev.dense_pv, (int)sizeof(SdPv), 4);
            else
                hipLaunchKernelGGL((scatter_values_kernel<uint32_t>), dim3(grid_for(n)), dim3(256), 0, s, (const uint32_t *)vals, sd.dev.dense_perm, n, sd.dev.dense_pv, (int)sizeof(SdPv), 4);
            if (hipGetLastError() != hipSuccess) return LIBRA_ERR_HIP;
        }
        if (int rc = place_values(dtype, vals, nullptr, 0, nullptr, sd.dev.res_perm, sd.n.res, sd.dev.res_ent, s)) return rc;
    }
    return LIBRA_OK;
}

extern "C" int libra_value_order_bytes(const libra_plan_t *P, size_t *order_bytes, size_t *workspace_bytes, size_t *scratch_bytes) {
    if (int rc = order_args(P)) return rc;
    if (!order_bytes || !workspace_bytes || !scratch_bytes) return LIBRA_ERR_NULL;
    const OrderShape h = order_shape(P);
    *order_bytes = order_arrays(h, nullptr).total + 256;
    *workspace_bytes = order_work(h, nullptr).total + 256;
    *scratch_bytes = h.passes ? (size_t)h.nnz * P->vsize : 0;
    return LIBRA_OK;
}

extern "C" int libra_value_order(const libra_plan_t *P, const int32_t *order, void *out, size_t out_bytes, void *workspace, size_t workspace_bytes, void *stream) {
    if (int rc = order_args(P)) return rc;
    const OrderShape h = order_shape(P);
    if ((!order || !out || !workspace) && h.nnz > 0) return LIBRA_ERR_NULL;
    if (h.nnz == 0) return LIBRA_OK;
    const OrderArrays a = order_arrays(h, out);
    const OrderWork w = order_work(h, workspace);
    if (out_bytes < a.total || workspace_bytes < w.total || (((uintptr_t)out | (uintptr_t)workspace) & 255)) return LIBRA_ERR_BUFFER;
    hipStream_t s = (hipStream_t)stream;
    const SubPlanDev &d = P->spmm.dev;
    const dim3 each((unsigned)((h.nnz + 255) / 256)), block(256);
    hipLaunchKernelGGL(k_order_clear, h.passes ? dim3(1) : each, block, 0, s, w.bad, w.seen, h.passes ? 0 : h.nnz);
    if (!h.passes) {
        hipLaunchKernelGGL(k_order_sources, each, block, 0, s, d.dense_perm, d.res_perm, h.nd, h.nd_pad, h.nnz, order, a.source, w.seen, w.bad);
        hipLaunchKernelGGL(k_order_all_seen, each, block, 0, s, w.seen, h.nnz, w.bad);
    } else {
        hipLaunchKernelGGL(k_order_keys, each, block, 0, s, d.dense_perm, d.res_perm, h.nd, h.nd_pad, h.nnz, order, h.T, h.chunks, w.key_in, w.slot_in, w.bad);
        const int64_t pairs = (int64_t)h.chunks * h.tiles;
        unsigned bits = 1;
        while ((1ll << bits) < pairs) ++bits;
        size_t sz = w.tmp_bytes;
        if (rocprim::radix_sort_pairs(w.tmp, sz, w.key_in, w.key_out, w.slot_in, w.slot_out, (size_t)h.nnz, 0u, bits, s) != hipSuccess) return LIBRA_ERR_HIP;
        hipLaunchKernelGGL(k_order_first, dim3((unsigned)((pairs + 256) / 256)), block, 0, s, w.key_out, (int)h.nnz, pairs, w.first);
        hipLaunchKernelGGL(k_order_runs, dim3((unsigned)((h.chunks + 63) / 64)), dim3(64), 0, s, w.first, h.chunks, h.tiles, h.T, h.nnz, a.run, a.to, a.tile_first, w.bad);
    }
    // (both waits also keep the workspace until its last pass has ended)
    auto refused = [&](int &rc) {
        int32_t bad = 0;
        rc = hipMemcpyAsync(&bad, w.bad, sizeof bad, hipMemcpyDeviceToHost, s) != hipSuccess || hipStreamSynchronize(s) != hipSuccess ? LIBRA_ERR_HIP : bad ? LIBRA_ERR_SHAPE : LIBRA_OK;
        return rc != LIBRA_OK;
    };
    int rc = LIBRA_OK;
    if (refused(rc)) return rc;
    if (h.passes) {
        // (here too, so that a first call with the order, which may be captured, sets nothing)
        if (!(P->vsize == 4 ? allow_chunks_lds<uint32_t>() : allow_chunks_lds<uint16_t>())) return LIBRA_ERR_HIP;
        hipLaunchKernelGGL(k_order_places, each, block, 0, s, w.key_out, w.slot_out, d.dense_perm, d.res_perm, h.nd, h.nd_pad, h.nnz, order, h.T, h.chunks, h.tiles, a.to, a.in_chunk, a.in_tile);
        hipLaunchKernelGGL(k_order_chunks_whole, dim3((unsigned)h.chunks), dim3(PASS_THREADS), 0, s, a.in_chunk, h.nnz, h.T, w.bad);
        if (refused(rc)) return rc;
    }
    return hipGetLastError() == hipSuccess ? LIBRA_OK : LIBRA_ERR_HIP;
}

extern "C" int libra_plan_set_values_ordered(libra_plan_t *P, const void *vals, int dtype, const void *order, void *scratch, void *stream) {
    if (int rc = order_args(P)) return rc;
    const OrderShape h = order_shape(P);
    if (dtype != P->vdt) return LIBRA_ERR_DTYPE;
    if (h.nnz == 0) return LIBRA_OK;
    if (!vals || !order || (h.passes && !scratch)) return LIBRA_ERR_NULL;
    if (((uintptr_t)order & 255) || ((uintptr_t)vals & (P->vsize - 1)) || ((uintptr_t)scratch & (P->vsize - 1))) return LIBRA_ERR_BUFFER;
    hipStream_t s = (hipStream_t)stream;
    const OrderArrays a = order_arrays(h, const_cast<void *>(order));
    const SubPlan &sa = P->spmm;
    if (!h.passes) return place_values(dtype, vals, a.source, h.nd, sa.dev.dense_val, a.source + h.nd_pad, sa.n.res, sa.dev.res_ent, s);
    return P->vsize == 4 ? run_passes<uint32_t>(P, h, a, vals, scratch, s) : run_passes<uint16_t>(P, h, a, vals, scratch, s);
}

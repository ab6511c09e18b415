// Values of other aggregation matrices on the same structure (DualGCN Sec. 2.1: the
// aggregation phase of a message-passing layer multiplies by a matrix derived from the
// adjacency; the GCN normalisation is one choice).  The SpMM kernels take any values, so
// switching aggregator means filling `val` again: GCN 1/sqrt(d_r d_c), mean 1/d_r, sum 1
// with 1 + eps on self-loop entries (the GIN form).  d is the row length of the matrix as
// given.  Values are computed in float64 and rounded once to float32.
#include "internal.h"

#include <algorithm>

namespace dgc {
namespace {

constexpr int kThreads = 256;

// A workgroup fills kTile consecutive entries, so their rows are consecutive too.  A first
// kernel leaves every tile's first and last row where the tile's first and last value will be
// written (nothing else needs room for them); each row in between then counts itself at the
// entry it starts at, and a scan of the counts gives every entry its row -- or, where more rows
// than entries meet the tile (empty rows), a search between the tile's two rows.  With a
// search of all row pointers per entry the kernel took 466 us on 31.5M entries (n = 2^20, 20
// dependent reads each), with a search per tile 180 us, now 165 (GCN; the random row lengths
// are 31.5M requests to the L2s, which take 270 G/s at best: 117 us).  It checks the columns,
// which the validation then need not read.
constexpr int kTile = 2048;
constexpr int kPer = kTile / kThreads;
// A search per entry has every entry in flight at once and reads no row pointers but its own; the
// tiles have another launch, which reads all of them, and barriers.  Whole calls (us, search / tiles,
// GCN and mean):
//   0.45M entries     n = 135,000 40.1 / 42.2, 38.9 / 40.0
//   0.7M              n = 210,000 43.7 / 45.6, 41.6 / 41.8; n = 420,000 44.3 / 43.8, 42.1 / 40.6
//                     n = 700,000 (rows of random length, 30% empty) 45.5 / 55.4, 42.9 / 52.9
//   1M                n = 600,000 46.2 / 45.9, 43.8 / 41.4; n = 10^6 (random lengths) 60.8 / 67.9, 52.2 / 61.0
//   2.5M              n = 2.5M 88.6 / 74.1, 73.4 / 47.1; n = 5M 100 / 109, 81.8 / 78.8; n = 12.5M 115 / 143,
//                     89.3 / 107
//   10M               n = 20M 291 / 326, 229 / 185; n = 50M 338 / 434, 280 / 274
bool by_search(int kind, int64_t n, int64_t nnz) {
    if (nnz <= int64_t{5} << 17) return true;
    if (nnz < int64_t{5} << 18) return n >= nnz;
    return kind == DUALGCN_AGG_GCN ? 2 * n >= 3 * nnz : n >= 4 * nnz;
}

__global__ __launch_bounds__(kThreads) void aggregator_search_kernel(const int32_t *__restrict__ rowptr,
                                                                     const int32_t *__restrict__ col, int32_t n,
                                                                     int64_t nnz, int kind, double one_plus_eps,
                                                                     int32_t *__restrict__ bad,
                                                                     float *__restrict__ val) {
    const int64_t e = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
    if (e >= nnz) return;
    const int32_t flags = *bad;
    int32_t lo = 0, hi = n;                    // the last r in [lo, hi) with rowptr[r] <= e
    while (hi - lo > 1) {
        const int32_t mid = lo + (hi - lo) / 2;
        if (static_cast<int64_t>(rowptr[mid]) <= e) lo = mid;
        else hi = mid;
    }
    const int32_t c = col[e];
    const double dr = static_cast<double>(rowptr[lo + 1] - rowptr[lo]);
    if (flags & 1) return;                     // row pointers out of order (looked at this late, its
    double v = 0.0;                            // load adds no latency; the search stays in range)
    if (static_cast<uint32_t>(c) >= static_cast<uint32_t>(n)) atomicOr(bad, 2);
    else if (kind == DUALGCN_AGG_MEAN) v = 1.0 / dr;
    else if (kind == DUALGCN_AGG_SUM) v = c == lo ? one_plus_eps : 1.0;
    else v = 1.0 / sqrt(dr * static_cast<double>(rowptr[c + 1] - rowptr[c]));
    val[e] = static_cast<float>(v);
}

// One thread per row writes the tile ends inside it; those of a row that meets more than
// kOwnTiles tiles are shared by its wavefront (one thread alone writes an end in about 25 ns: with
// a row of 32.5M entries the call took 1,320 us, by the wavefront 266).
constexpr int64_t kOwnTiles = 16;

// The ends at entries [b, e) of row r: tiles first, first + step, ... of the tiles they meet.
__device__ __forceinline__ void write_tile_ends(int32_t *__restrict__ ends, int64_t b, int64_t e, int32_t r,
                                                int first, int step) {
    for (int64_t at = (b / kTile + first) * kTile; at < e; at += static_cast<int64_t>(step) * kTile) {
        if (at >= b) ends[at] = r;
        if (at + kTile - 1 < e && at + kTile - 1 >= b) ends[at + kTile - 1] = r;
    }
}

__global__ __launch_bounds__(kThreads) void tile_ends_kernel(const int32_t *__restrict__ rowptr, int32_t n,
                                                             int64_t nnz, const int32_t *__restrict__ bad,
                                                             int32_t *__restrict__ ends) {
    if (*bad & 1) return;                      // row pointers out of order
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
    const int lane = static_cast<int>(threadIdx.x) & 63;
    const int32_t b = i < n ? rowptr[i] : 0, e = i < n ? rowptr[i + 1] : 0;
    const bool many = static_cast<int64_t>(e) - b > kOwnTiles * kTile;
    if (b < e && !many) write_tile_ends(ends, b, e, static_cast<int32_t>(i), 0, 1);
    if (b < e && e == nnz) ends[nnz - 1] = static_cast<int32_t>(i);
    for (uint64_t m = __ballot(many); m != 0; m &= m - 1) {
        const int src = __ffsll(static_cast<unsigned long long>(m)) - 1;
        write_tile_ends(ends, __shfl(b, src, 64), __shfl(e, src, 64), static_cast<int32_t>(i - lane + src), lane, 64);
    }
}

__global__ __launch_bounds__(kThreads) void aggregator_kernel(const int32_t *__restrict__ rowptr,
                                                              const int32_t *__restrict__ col,
                                                              int32_t n, int64_t nnz, int kind,
                                                              double one_plus_eps, int32_t *__restrict__ bad,
                                                              float *val) {
    __shared__ __align__(16) uint32_t cnt[kTile];
    __shared__ uint32_t wsum[kThreads / 64];
    if (*bad & 1) return;                      // no tile ends
    const int t = static_cast<int>(threadIdx.x), lane = t & 63, wave = t >> 6;
    const int64_t e0 = static_cast<int64_t>(blockIdx.x) * kTile;
    const int64_t e1 = e0 + kTile < nnz ? e0 + kTile : nnz;
    const int32_t r0 = __float_as_int(val[e0]), r1 = __float_as_int(val[e1 - 1]);
    // columns and values stream past the L2, which the random row lengths live in
    int32_t c[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int64_t e = e0 + k * kThreads + t;
        c[k] = __builtin_nontemporal_load(col + (e < e1 ? e : e1 - 1));
        cnt[k * kThreads + t] = 0;
    }
    bool in = true;
#pragma unroll
    for (int k = 0; k < kPer; ++k) in &= static_cast<uint32_t>(c[k]) < static_cast<uint32_t>(n);
    if (!in) atomicOr(bad, 2);
    __syncthreads();
    const bool scanned = r1 - r0 <= kTile;
    if (scanned) {
        // row r0 covers the tile's start; each later row that starts inside counts itself there
        for (int32_t r = r0 + 1 + t; r <= r1; r += kThreads) atomicAdd(&cnt[rowptr[r] - e0], 1u);
        __syncthreads();
        uint32_t run[kPer], sum = 0;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            sum += cnt[t * kPer + k];
            run[k] = sum;
        }
        uint32_t inc = sum;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = __shfl_up(inc, off, 64);
            if (lane >= off) inc += y;
        }
        if (lane == 63) wsum[wave] = inc;
        __syncthreads();
        uint32_t base = inc - sum;
        for (int w = 0; w < wave; ++w) base += wsum[w];
#pragma unroll
        for (int k = 0; k < kPer; ++k) cnt[t * kPer + k] = base + run[k];
        __syncthreads();
    }
    int32_t r[kPer];
    double dr[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int32_t i = k * kThreads + t;
        if (scanned) {
            r[k] = r0 + static_cast<int32_t>(cnt[i]);     // past e1: the tile's last row
        } else {
            int32_t lo = r0, hi = r1;          // more rows than entries: search between the two
            while (lo < hi) {
                const int32_t mid = lo + (hi - lo + 1) / 2;
                if (static_cast<int64_t>(rowptr[mid]) <= e0 + i) lo = mid;
                else hi = mid - 1;
            }
            r[k] = lo;
        }
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) dr[k] = static_cast<double>(rowptr[r[k] + 1] - rowptr[r[k]]);
    float v[kPer];
    if (kind == DUALGCN_AGG_GCN) {
        // a column out of range (reported) reads row r's length instead
        double dc[kPer];
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int32_t q = static_cast<uint32_t>(c[k]) < static_cast<uint32_t>(n) ? c[k] : r[k];
            dc[k] = static_cast<double>(rowptr[q + 1] - rowptr[q]);
        }
#pragma unroll
        for (int k = 0; k < kPer; ++k) v[k] = static_cast<float>(1.0 / sqrt(dr[k] * dc[k]));
    } else {
#pragma unroll
        for (int k = 0; k < kPer; ++k)
            v[k] = static_cast<float>(kind == DUALGCN_AGG_MEAN ? 1.0 / dr[k] : c[k] == r[k] ? one_plus_eps : 1.0);
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int64_t e = e0 + k * kThreads + t;
        if (e < e1) __builtin_nontemporal_store(v[k], val + e);
    }
}

}  // namespace

int launch_aggregator_values(const dualgcn_csr *csr, int kind, float eps, int32_t *bad, float *val,
                             hipStream_t s) {
    if (csr->nnz == 0) return DUALGCN_OK;
    const int64_t blocks = (csr->nnz + kTile - 1) / kTile;      // below 2^20
    const double plus = 1.0 + static_cast<double>(eps);
    if (by_search(kind, csr->n, csr->nnz)) {
        hipLaunchKernelGGL(aggregator_search_kernel,
                           dim3(static_cast<unsigned>((csr->nnz + kThreads - 1) / kThreads)), dim3(kThreads), 0, s,
                           csr->rowptr, csr->col, csr->n, csr->nnz, kind, plus, bad, val);
        return hip_status(hipGetLastError());
    }
    const int64_t row_blocks = (static_cast<int64_t>(csr->n) + kThreads - 1) / kThreads;
    hipLaunchKernelGGL(tile_ends_kernel, dim3(static_cast<unsigned>(row_blocks)), dim3(kThreads), 0, s,
                       csr->rowptr, csr->n, csr->nnz, bad, reinterpret_cast<int32_t *>(val));
    hipLaunchKernelGGL(aggregator_kernel, dim3(static_cast<unsigned>(blocks)), dim3(kThreads), 0, s,
                       csr->rowptr, csr->col, csr->n, csr->nnz, kind, plus, bad, val);
    return hip_status(hipGetLastError());
}

}  // namespace dgc

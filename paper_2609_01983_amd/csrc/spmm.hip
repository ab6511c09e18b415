// Dual-path aggregation SpMM Y = A X on gfx950 (DualGCN Sec. 3.3), and the same
// aggregation fused with the next layer's update, T = bf16(act(A X)) W (further below).
//
// The kernels stream the plan's sorted copy of the matrix: row i of the copy is
// row order[i] of A, the sparse region is rows [0, n_sparse) and the dense region
// rows [n_sparse, n) (Eq. (1) was applied when the plan was built; inside a region
// rows go by row-length octave, then node id).  One launch
// covers both paths; every workgroup picks its path from its index:
//
//   parts      rows of the dense region longer than one chunk, split into parts
//              of the plan's dense chunk (512 to 4096 entries, by the matrix's size;
//              heaviest row first), one wavefront per part
//   long       the other dense rows of at least 256 entries (one or two octaves fewer
//              for groups narrower than 16 lanes), one wavefront per row, heaviest
//              first; where parts and rows of at least 512 entries are no more than the
//              CUs, a workgroup each
//   medium     the remaining dense rows, one lane group per row, heaviest first
//   sparse     tasks of up to kTaskRows short consecutive rows, one lane group per
//              task (the paper's "several rows per block")
//
// Feature layout.  A lane group of LPR lanes covers SW = LPR * VEC consecutive
// features of a row: with VEC = 4 every lane makes one 16-byte load, so one
// neighbour costs one coalesced load of the whole row (512 bytes = four 128-byte
// lines at F = 128, 32 lanes).  Features beyond 256 are processed in windows of
// 256; a window may be cut into S slices, workgroup b working on slice b % S (64 features
// each where rows are whole lines, so that each XCD reads its own slices: sliced_window;
// also the one-feature-per-lane path for F < 4).  Rows may start anywhere: a width that is no
// multiple of four lets its last lane overlap its neighbour (lane_feature).
//
// Gathers.  A group takes the entries of its row (or task) in rounds of 16:
// each lane loads 16 / LPR (column, value) pairs with coalesced loads, the
// pairs are broadcast inside the group with shuffles, and all 16 neighbour
// slices (a half or a quarter of them where the launch is bound by its gathers: pick_gathers)
// are requested before the first product, so every group
// keeps that many loads in flight (the ILP of the paper's dense path, Alg. 1, deepened).
// Nothing in a round branches (see gather), and the next round's pairs are requested with this
// round's slices.
// On large operands the rows of cold columns (marked by the plan) are read non-temporally
// (the cache classes below).  Before the rounds were free of branches a lone wavefront took
// 1.65 us a round (F = 128) and the launches on small and middling graphs were bound by that
// chain.  Measured before and after: R-MAT n = 30,007 (longest row 3,928), F = 128: 227 ->
// 112 us; R-MAT n = 4,096, F = 16: 15.8 -> 12.5 us; block model n = 2^18 (18.8M entries),
// F = 128: 496 -> 448 us (21.5 TB/s of gathers, out of the L2s).
//
// Dense path (paper: one row per block, 4-way ILP and a shared reduction): a long
// row gets a wavefront whose groups take rounds of the row in turn and are summed
// with a butterfly over the lanes; a dense row shorter than the long rows' bound
// gets one lane group, which fills its rounds better (measured: the SBM
// workload's dense rows of 100-250 entries run 9% faster than with a wavefront).
// A split row's parts each write a float64 partial, and a small second kernel
// sums them in part order and writes the row.  The kernel boundary makes the
// partials visible: a fence inside the SpMM would write back and invalidate the
// XCD's L2 once per part, which the gathers live on.  No floating-point atomics:
// Y is bit-reproducible.
//
// Sparse path (tasks): the group walks the task's entries as one stream, so even
// rows with one or two entries share a round of gathers; a row is written
// as soon as its last entry has been added.
//
// Summation: products and the sum of one round (<= 16 terms) are float32,
// rounds are added in float64, and each output is rounded once to float32.  The
// error of every element is below ~(16 + 2) * 2^-24 * sum |a||x|.
#include "internal.h"

#include <algorithm>
#include <type_traits>

namespace dgc {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kRound = 16;            // entries a lane group adds per round

typedef float f32x4 __attribute__((ext_vector_type(4)));
// rows of any width start at any multiple of 4 (or, in bfloat16, 2) bytes
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32_any __attribute__((aligned(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));

template <int VEC>
__device__ __forceinline__ void load_x(const float *__restrict__ p, float (&x)[VEC]) {
    if constexpr (VEC == 4) {
        const f32x4_any v = *reinterpret_cast<const f32x4_any *>(p);
        x[0] = v[0];
        x[1] = v[1];
        x[2] = v[2];
        x[3] = v[3];
    } else {
#pragma unroll
        for (int j = 0; j < VEC; ++j) x[j] = p[j];
    }
}

// Stores the rounded sums of one lane's VEC features at element offset `at` of Y
// (float32, or bfloat16 rounded from the float32 value when BF).
template <int VEC, bool BF>
__device__ __forceinline__ void store_y(void *__restrict__ Y, int64_t at, const double (&s)[VEC],
                                        bool relu) {
    float o[VEC];
#pragma unroll
    for (int j = 0; j < VEC; ++j) {
        o[j] = static_cast<float>(s[j]);
        if (relu) o[j] = o[j] > 0.f ? o[j] : 0.f;
    }
    if constexpr (BF) {
        unsigned short *p = static_cast<unsigned short *>(Y) + at;
        if constexpr (VEC == 4) {
            const uint2 v = make_uint2(static_cast<uint32_t>(to_bf16(o[0])) | (static_cast<uint32_t>(to_bf16(o[1])) << 16),
                                       static_cast<uint32_t>(to_bf16(o[2])) | (static_cast<uint32_t>(to_bf16(o[3])) << 16));
            __builtin_nontemporal_store(v.x, reinterpret_cast<u32_any *>(p));
            __builtin_nontemporal_store(v.y, reinterpret_cast<u32_any *>(p) + 1);
        } else {
#pragma unroll
            for (int j = 0; j < VEC; ++j) __builtin_nontemporal_store(to_bf16(o[j]), p + j);
        }
    } else {
        float *p = static_cast<float *>(Y) + at;
        if constexpr (VEC == 4) {
            const f32x4_any v = {o[0], o[1], o[2], o[3]};
            __builtin_nontemporal_store(v, reinterpret_cast<f32x4_any *>(p));
        } else {
#pragma unroll
            for (int j = 0; j < VEC; ++j) __builtin_nontemporal_store(o[j], p + j);
        }
    }
}

struct Args {
    const int32_t *pptr;        // sorted copy of the matrix
    const int32_t *pcol;
    const float *pval;
    const int32_t *perm;        // output row of each sorted row (the plan's order)
    const int32_t *tasks;
    const SplitPart *parts;
    double *partials;
    const float *X;
    void *Y;                    // float32, or bfloat16 when the kernel's BF is set (fused: H or null)
    uint32_t x_bytes;           // bytes of X that gathers may read (cache-class loads)
    int32_t n, n_sparse, n_tasks, n_parts, n_long;
    int32_t n_coop;             // rows of at least 2^kLongRowOctave entries that share workgroups, or 0
    int32_t coop;               // parts and those rows are a workgroup's each (see shares_rows)
    int32_t dense_chunk;        // entries per part of a split dense row (the plan's)
    int32_t ld;                 // leading dimension of X and Y (= F)
    int32_t f0;                 // first feature of this launch window
    int32_t fend;               // end of the valid features of the window
    int32_t fcap;               // last feature a lane's four may start at (see lane_feature)
    int32_t S;                  // feature slices in the window
    int32_t sw;                 // features per slice (at most those of a lane group)
    int32_t nb_parts;           // logical workgroups of hub-row parts
    int32_t nb_coop;            // logical workgroups of the longest dense rows (one each; 0: no sharing)
    int32_t nb_long;            // nb_coop + those of the other long dense rows (a wavefront each)
    int32_t nb_dense;           // nb_long + those of the other dense rows (a group each)
    int32_t relu;
};

// First of a lane's VEC features, for the lane at position `pos` of the window.  Rows whose width
// is no multiple of four end inside a lane's four: that lane takes the row's last four instead
// (F >= 4), the first of which its neighbour computes and stores as well, to the same bits.
template <int VEC>
__device__ __forceinline__ int32_t lane_feature(const Args &a, int32_t pos) {
    return VEC == 4 ? min(a.f0 + pos, a.fcap) : a.f0 + pos;
}

// Where a finished row goes.  Rows are emitted by whole lane groups (every lane of
// the group calls row() with the same arguments except its features): `slot` numbers
// the row inside the wavefront's current block of work (group gw, row j of its task:
// gw * kTaskRows + j; a wavefront's long row: 0).
//
// StoreRows writes the row to Y at output row `out`.
template <int VEC, bool BF>
struct StoreRows {
    void *Y;
    int32_t ld;
    bool relu;
    __device__ __forceinline__ void row(int64_t out, int slot, const double (&tot)[VEC], int f,
                                        bool fin) const {
        (void)slot;
        if (fin) store_y<VEC, BF>(Y, out * ld + f, tot, relu);
    }
};

// StageRows keeps the row for the fused update instead: act(row) rounded to bfloat16
// in the wavefront's LDS tile (row `slot`, ld elements apart), its output row in
// outs[slot]; when H is set, the same bfloat16 row is also stored to H (row `out`,
// ldH elements apart), as the plain kernel stores a bfloat16 Y.  VEC = 4; the window
// starts at feature 0.
struct StageRows {
    unsigned short *h;
    int32_t *outs;
    int32_t ld;
    bool relu;
    bool lead;          // the group's first lane records the output row
    unsigned short *H;
    int32_t ldH;
    __device__ __forceinline__ void row(int64_t out, int slot, const double (&tot)[4], int f,
                                        bool fin) const {
        if (fin) {
            float o[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                o[j] = static_cast<float>(tot[j]);
                if (relu) o[j] = o[j] > 0.f ? o[j] : 0.f;
            }
            const uint2 pk =
                make_uint2(static_cast<uint32_t>(to_bf16(o[0])) | (static_cast<uint32_t>(to_bf16(o[1])) << 16),
                           static_cast<uint32_t>(to_bf16(o[2])) | (static_cast<uint32_t>(to_bf16(o[3])) << 16));
            *reinterpret_cast<uint2 *>(h + static_cast<int64_t>(slot) * ld + f) = pk;
            if (H) {
                uint32_t *g = reinterpret_cast<uint32_t *>(H + out * ldH + f);
                __builtin_nontemporal_store(pk.x, g);
                __builtin_nontemporal_store(pk.y, g + 1);
            }
        }
        if (lead) outs[slot] = static_cast<int32_t>(out);
    }
};

// Cache classes of the gathers (kernels instantiated with kClasses): a gathered row is read
// with the default policy when its column is among the hottest (rows the L2s keep), and
// non-temporal otherwise, so that rows read a few times per launch do not push the hot
// rows out of the L2.  The plan marks the other columns with bit 31 of the sorted copy's
// column (columns are below 2^31); every kernel masks it off, and it never changes which
// row is read.
constexpr int kCpolNt = 2;                    // the nt field of a gfx950 buffer load
constexpr uint32_t kRowMask = 0x7FFFFFFFu;

// How a launch's gathers address X.
//   kBuffer   buffer loads at 32-bit byte offsets (X up to kMaxBufferBytes)
//   kClasses  the same with the cache classes above
//   kWide     64-bit addresses
enum GatherMode { kBuffer = 0, kClasses = 1, kWide = 2 };

// How many gathers a lane group requests at a time (kRound, a half or a quarter of it) and how
// many workgroups a CU holds (0: as many as fit); see pick_gathers.
struct Gathers {
    int mode, q, groups;
};

// Dynamic LDS that keeps a CU to `groups` workgroups whose kernel has `own` bytes of its own.
constexpr unsigned kCuLds = 160 * 1024;
constexpr unsigned groups_lds(int groups, unsigned own) {
    return groups == 0 ? 0 : kCuLds / static_cast<unsigned>(groups) - 2048 - own;
}
constexpr bool keeps(int groups) {
    const unsigned each = groups_lds(groups, 0);
    return groups * each <= kCuLds && (groups + 1) * each > kCuLds;
}
static_assert(keeps(4) && keeps(5), "the padding holds what it says");

// LDS for the sums of a long row's other wavefronts: launches that share rows (see share_rows).
template <int LPR, int VEC, int MODE>
constexpr int shared_sums() {
    return MODE == kBuffer ? (kWaves - 1) * LPR * VEC : 1;
}

// Offset of an entry that reads nothing: past the end of every buffer, also with a feature's
// offset (below 4 MiB) added, so that a buffer load of it returns zeros.
constexpr uint32_t kNoEntry = 0xFF800000u;
constexpr uint64_t kMaxBufferBytes = kNoEntry;
constexpr uint32_t kNoRow = 0x80000000u;        // marks an invalid entry's row in kWide

// Entries [e, min(e + kRound, e_end)) of the sorted copy (e_end > 0), as seen by lane li of
// a group: lane li loads entries e + li + k LPR; entry u is then held by lane u % LPR in
// register u / LPR.  The loads are unconditional (past the end they read the last entry).
// ready() turns the columns into what the gathers broadcast: byte offsets into X (one multiply
// per entry instead of one per lane and entry), or rows in kWide; an entry past the end gets
// weight zero and an offset that reads zeros.
template <int LPR, int MODE>
struct Round {
    static constexpr int EPL = (kRound + LPR - 1) / LPR;   // entries per lane
    int32_t c[EPL];
    float v[EPL];

    __device__ __forceinline__ void load(const Args &a, int32_t e, int32_t e_end, int li) {
#pragma unroll
        for (int k = 0; k < EPL; ++k) {
            const int32_t idx = min(e + li + k * LPR, e_end - 1);
            c[k] = a.pcol[idx];
            v[k] = a.pval[idx];
        }
    }

    __device__ __forceinline__ void ready(const Args &a, int32_t e, int32_t e_end, int li) {
#pragma unroll
        for (int k = 0; k < EPL; ++k) {
            const bool ok = li + k * LPR < kRound && e + li + k * LPR < e_end;
            v[k] = ok ? v[k] : 0.f;
            const uint32_t row = static_cast<uint32_t>(c[k]) & kRowMask;
            uint32_t at;
            if constexpr (MODE == kWide) {
                at = ok ? row : row | kNoRow;
            } else {
                at = row * (static_cast<uint32_t>(a.ld) * 4u);
                if constexpr (MODE == kClasses) at |= static_cast<uint32_t>(c[k]) >> 31;   // a marked (cold) column
                at = ok ? at : kNoEntry;
            }
            c[k] = static_cast<int32_t>(at);
        }
    }
};

template <int VEC, int POLICY>
__device__ __forceinline__ void load_x_buf(__amdgpu_buffer_rsrc_t rx, uint32_t off, float (&x)[VEC]) {
    if constexpr (VEC == 4) {
        const f32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rx, off, 0, POLICY);
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = v[j];
    } else {
        static_assert(VEC == 1, "one or four features per lane");
        x[0] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rx, off, 0, POLICY));
    }
}

// Requests the neighbour slices of entries U0 .. U0 + Q - 1 of a round (ready() done).
// The broadcasts read lane gbase + u % LPR with ds_bpermute: the group's base byte
// address is hidden from the optimiser, so that the constant u % LPR lanes go into the
// instruction's offset field instead of one precomputed address register per u
// (sixteen registers held through the whole kernel otherwise).
// No branches: with a branch per gather the compiler waited for the first gather inside its
// branch and for every broadcast before the next one, so a round took two memory latencies
// and sixteen LDS latencies (1.65 us on an idle chip, F = 128).
template <int LPR, int VEC, int MODE, int U0, int Q>
__device__ __forceinline__ void gather(const Args &a, const Round<LPR, MODE> &r, int gbase, int f, bool fin,
                                       float (&as)[Q], float (&xs)[Q][VEC]) {
    static_assert(MODE != kClasses || VEC == 4, "cache classes need 16-byte loads");
    int base4 = gbase * 4;
    asm volatile("" : "+v"(base4));
    if constexpr (MODE == kWide) {
        uint32_t row[Q];
#pragma unroll
        for (int u = 0; u < Q; ++u) {
            const int src = base4 + ((U0 + u) % LPR) * 4;
            row[u] = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(src, r.c[(U0 + u) / LPR]));
            as[u] = __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(r.v[(U0 + u) / LPR])));
        }
#pragma unroll
        for (int u = 0; u < Q; ++u)
#pragma unroll
            for (int j = 0; j < VEC; ++j) xs[u][j] = 0.f;
        // an invalid entry reads the row of the last one and drops it; with one feature a lane (F < 4)
        // most lanes have none and stay out (n = 358M, F = 3, one entry a row 30.7 ms, so 28.6)
        if (VEC != 1 || fin) {
#pragma unroll
            for (int u = 0; u < Q; ++u)
                load_x<VEC>(a.X + static_cast<int64_t>(row[u] & kRowMask) * a.ld + (fin ? f : a.f0), xs[u]);
        }
#pragma unroll
        for (int u = 0; u < Q; ++u)
#pragma unroll
            for (int j = 0; j < VEC; ++j) xs[u][j] = (row[u] & kNoRow) == 0 ? xs[u][j] : 0.f;
    } else {
        // a lane without features of its own reads the window's first ones, which nothing uses and
        // other lanes read (the row's first: another line per entry, F = 300 5-8% slower)
        const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float *>(a.X), 0, static_cast<int>(a.x_bytes), 0x00020000);
        const uint32_t lane_off = static_cast<uint32_t>(fin ? f : a.f0) * 4u;
#pragma unroll
        for (int u = 0; u < Q; ++u) {
            const int src = base4 + ((U0 + u) % LPR) * 4;
            const uint32_t at = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(src, r.c[(U0 + u) / LPR]));
            as[u] = __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(r.v[(U0 + u) / LPR])));
            if constexpr (MODE != kClasses) {
                load_x_buf<VEC, 0>(rx, at + lane_off, xs[u]);
            } else {
                const uint32_t off = (at & ~1u) + lane_off;
                if (at & 1u) load_x_buf<VEC, kCpolNt>(rx, off, xs[u]);
                else load_x_buf<VEC, 0>(rx, off, xs[u]);
            }
        }
    }
}

// Entries U0 .. kRound - 1 of a round that starts at e, Q gathers requested at a time; the next
// round's columns and values are requested behind the round's last gathers.
template <int LPR, int VEC, int MODE, int Q, int U0, bool PF, class Term>
__device__ __forceinline__ void round_terms(const Args &a, Round<LPR, MODE> &r, int32_t e, int32_t e1, int32_t step,
                                            int li, int gbase, int f, bool fin, const Term &term) {
    {
        float as[Q], xs[Q][VEC];
        gather<LPR, VEC, MODE, U0, Q>(a, r, gbase, f, fin, as, xs);
        if constexpr (PF && U0 + Q == kRound) r.load(a, e + step, e1, li);
#pragma unroll
        for (int u = 0; u < Q; ++u) term(e + U0 + u, as[u], xs[u]);
    }
    if constexpr (U0 + Q < kRound) {
        __builtin_amdgcn_sched_barrier(0);       // the next gathers stay behind
        if (e + U0 + Q < e1)
            round_terms<LPR, VEC, MODE, Q, U0 + Q, PF>(a, r, e, e1, step, li, gbase, f, fin, term);
    }
}

// A lane group's walk over the rounds of kRound entries at e0, e0 + step, ... below e1:
// term(e, weight, slice) for every entry in order (entries past e1 come with weight and
// slice zero), flush() after every round.  The next round's columns and values are requested
// behind the current round's gathers (not for groups of one or two lanes, which hold 16 or 8
// of them in registers: a wavefront less per SIMD).
template <int LPR, int VEC, int MODE, int Q, class Term, class Flush>
__device__ __forceinline__ void walk_rounds(const Args &a, int32_t e0, int32_t e1, int32_t step, int li,
                                            int gbase, int f, bool fin, const Term &term, const Flush &flush) {
    if (e0 >= e1) return;
    constexpr bool PF = LPR >= 4;
    Round<LPR, MODE> r;
    if constexpr (PF) r.load(a, e0, e1, li);
    for (int32_t e = e0; e < e1; e += step) {
        if constexpr (!PF) r.load(a, e, e1, li);
        r.ready(a, e, e1, li);
        round_terms<LPR, VEC, MODE, Q, 0, PF>(a, r, e, e1, step, li, gbase, f, fin, term);
        flush();
    }
}

// Dense path: a lane group's sums over its rounds of one row, in V = 1, 2 or 4 chains (round q
// of the group adds to chain q % V, by rotating them) that are then added pairwise: as (0 + 2)
// + (1 + 3) for four, whichever chain is first after the last rotation.
template <int LPR, int VEC, int MODE, int Q, int V>
__device__ __forceinline__ void dense_rounds(const Args &a, int32_t e0, int32_t e1, int32_t step, int li,
                                             int gbase, int f, bool fin, double (&tot)[VEC]) {
    float acc[VEC];
    double chain[V][VEC];
#pragma unroll
    for (int j = 0; j < VEC; ++j) {
        acc[j] = 0.f;
#pragma unroll
        for (int q = 0; q < V; ++q) chain[q][j] = 0.0;
    }
    walk_rounds<LPR, VEC, MODE, Q>(
        a, e0, e1, step, li, gbase, f, fin,
        [&](int32_t, float w, const float (&x)[VEC]) {
#pragma unroll
            for (int j = 0; j < VEC; ++j) acc[j] = fmaf(w, x[j], acc[j]);
        },
        [&]() {
#pragma unroll
            for (int j = 0; j < VEC; ++j) {
                const double first = chain[0][j] + static_cast<double>(acc[j]);
#pragma unroll
                for (int q = 0; q + 1 < V; ++q) chain[q][j] = chain[q + 1][j];
                chain[V - 1][j] = first;
                acc[j] = 0.f;
            }
        });
#pragma unroll
    for (int j = 0; j < VEC; ++j) {
        if constexpr (V == 1) tot[j] = chain[0][j];
        else if constexpr (V == 2) tot[j] = chain[0][j] + chain[1][j];
        else tot[j] = (chain[0][j] + chain[2][j]) + (chain[1][j] + chain[3][j]);
    }
}

// Entries [e0, e1) of one row by wavefront `wave` of `waves` that share it: their groups take
// rounds in turn and a butterfly adds a wavefront's; every lane then holds its sums of its
// features.  A wavefront's rounds form four chains, whatever the group's width: four 16-lane
// groups have one each, two 32-lane groups two each, a whole wavefront all four -- one after
// the other where a round's gathers leave no registers for four sets of sums.  So the SpMM's slices of 64 features and the
// fused kernel, which reads rows whole, add a long row in the same order and give the same bits.
template <int LPR, int VEC, int MODE, int Q>
__device__ __forceinline__ void long_row(const Args &a, int32_t e0, int32_t e1, int wave, int waves, int li,
                                         int gw, int gbase, int f, bool fin, double (&tot)[VEC]) {
    if constexpr (VEC == 4 && LPR == 64 && MODE == kBuffer && Q == kRound) {
        double even[VEC], t[VEC];
#pragma unroll 1
        for (int q = 0; q < 4; ++q) {                       // chains 0, 2, 1, 3
            const int chain = (q >> 1) | ((q & 1) << 1);
            dense_rounds<LPR, VEC, MODE, Q, 1>(a, e0 + (chain * waves + wave) * kRound, e1, 4 * waves * kRound, li,
                                            gbase, f, fin, t);
#pragma unroll
            for (int j = 0; j < VEC; ++j) {
                if (q % 2 == 0) even[j] = t[j];
                else tot[j] = q == 1 ? even[j] + t[j] : tot[j] + (even[j] + t[j]);
            }
        }
        return;
    }
    constexpr int GPW = 64 / LPR;
    dense_rounds<LPR, VEC, MODE, Q, VEC == 4 && LPR >= 32 ? LPR / 16 : 1>(
        a, e0 + (gw * waves + wave) * kRound, e1, GPW * waves * kRound, li, gbase, f, fin, tot);
#pragma unroll
    for (int m = 32; m >= LPR; m >>= 1)
#pragma unroll
        for (int j = 0; j < VEC; ++j) tot[j] += __shfl_xor(tot[j], m, 64);
}

// Selects register j / LPR of a per-lane array and reads it from lane j % LPR.
template <int LPR, int N>
__device__ __forceinline__ int32_t task_meta(const int32_t (&m)[N], int j, int gbase) {
    int32_t x = m[0];
#pragma unroll
    for (int k = 1; k < N; ++k)
        if (j / LPR == k) x = m[k];
    return __shfl(x, gbase + j % LPR, 64);
}

// The work of logical workgroup lb (feature slice `slice`) for wavefront `wave` of a
// workgroup of WAVES wavefronts; finished rows go to `emit`.  red: (WAVES - 1) x LPR x VEC
// float64 of LDS, used where wavefronts share a row.
template <int LPR, int VEC, int WAVES, int MODE, int Q, class Emit>
__device__ __forceinline__ void spmm_block(const Args &a, int lb, int slice, int wave,
                                           const Emit &emit, double *red) {
    constexpr int GPW = 64 / LPR;                 // lane groups per wavefront
    constexpr int RPL = (kTaskRows + LPR - 1) / LPR;

    const int lane = static_cast<int>(threadIdx.x) & 63;
    const int li = lane % LPR;
    const int gw = lane / LPR;
    const int gbase = lane - li;
    const int pos = slice * a.sw + li * VEC;      // the lane's features inside the window
    const bool fin = li * VEC < a.sw && a.f0 + pos < a.fend;
    const int f = lane_feature<VEC>(a, pos);

    if (lb >= a.nb_parts + a.nb_long && lb < a.nb_parts + a.nb_dense) {
        // ---------------- dense path, shorter rows: one lane group per row
        const int64_t gi = (static_cast<int64_t>(lb - a.nb_parts - a.nb_long) * WAVES + wave) * GPW + gw;
        const int64_t i = a.n - a.n_long - 1 - gi;
        if (i < a.n_sparse) return;           // the whole group leaves together
        double tot[VEC];
        dense_rounds<LPR, VEC, MODE, Q, 1>(a, a.pptr[i], a.pptr[i + 1], kRound, li, gbase, f, fin, tot);
        emit.row(a.perm[i], gw * kTaskRows, tot, f, fin);
        return;
    }
    if (lb < a.nb_parts + a.nb_long) {
        // ---------------- dense path, long rows and parts of split rows: a wavefront each, or
        // the workgroup's wavefronts together
        constexpr bool kMayShare = MODE == kBuffer;
        const bool share = kMayShare && a.coop && lb < a.nb_parts + a.nb_coop;
        int32_t i, e0, e1;
        int part = -1, first = 0;
        if (lb < a.nb_parts) {
            const int w = share ? lb : lb * WAVES + wave;
            if (w >= a.n_parts) return;
            const SplitPart sp = a.parts[a.n_parts - 1 - w];
            i = sp.row;
            part = sp.part;
            first = sp.first;
            e0 = a.pptr[i] + part * a.dense_chunk;
            e1 = min(e0 + a.dense_chunk, a.pptr[i + 1]);
        } else {
            const int q = lb - a.nb_parts;
            i = a.n - 1 - (share ? q : a.n_coop + (q - a.nb_coop) * WAVES + wave);
            if (i < a.n - a.n_long) return;
            e0 = a.pptr[i];
            e1 = a.pptr[i + 1];
            if (e1 - e0 > a.dense_chunk) return;   // covered by its parts
        }
        double tot[VEC];
        long_row<LPR, VEC, MODE, Q>(a, e0, e1, share ? wave : 0, share ? WAVES : 1, li, gw, gbase, f, fin, tot);
        if constexpr (kMayShare) {
            if (share) {
                // every wavefront of the workgroup is here with the same row: the first adds
                // the others' sums in order
                double *mine = red + li * VEC;
                if (wave != 0 && gw == 0)
#pragma unroll
                    for (int j = 0; j < VEC; ++j) mine[(wave - 1) * LPR * VEC + j] = tot[j];
                __syncthreads();
                if (wave == 0)
#pragma unroll
                    for (int q = 0; q < WAVES - 1; ++q)
#pragma unroll
                        for (int j = 0; j < VEC; ++j) tot[j] += mine[q * LPR * VEC + j];
                __syncthreads();                  // red is free for the next row
                if (wave != 0) return;
            }
        }
        if (part < 0) {
            if (gw == 0) emit.row(a.perm[i], 0, tot, f, fin);
            return;
        }
        // a part of a split row: its float64 partial, summed by combine_kernel after this launch
        if (gw == 0 && fin) {
            double *pp = a.partials + static_cast<int64_t>(first + part) * kMaxSlice + pos;
#pragma unroll
            for (int j = 0; j < VEC; ++j) pp[j] = tot[j];
        }
        return;
    }

    // ---------------- sparse path: one task (up to kTaskRows short rows) per lane group
    const int64_t t = (static_cast<int64_t>(lb - a.nb_parts - a.nb_dense) * WAVES + wave) * GPW + gw;
    if (t >= a.n_tasks) return;               // the whole group leaves together
    const int32_t r0 = a.tasks[t];
    const int m = a.tasks[t + 1] - r0;        // 1 .. kTaskRows rows
    int32_t rend[RPL], rout[RPL];             // row j: lane j % LPR, register j / LPR
#pragma unroll
    for (int k = 0; k < RPL; ++k) {
        const int j = li + k * LPR;
        rend[k] = j < m ? a.pptr[r0 + j + 1] : 0;
        rout[k] = j < m ? a.perm[r0 + j] : 0;
    }
    const int32_t e_begin = a.pptr[r0];
    const int32_t e_end = task_meta<LPR>(rend, m - 1, gbase);
    if (e_begin == e_end) {                   // a task of empty rows (a run of them is cut
        double z[VEC];                        // into tasks of at most kTaskRows)
#pragma unroll
        for (int j = 0; j < VEC; ++j) z[j] = 0.0;
        for (int j = 0; j < m; ++j) emit.row(task_meta<LPR>(rout, j, gbase), gw * kTaskRows + j, z, f, fin);
        return;
    }
    int cur = 0;                              // every row of a task with entries is non-empty
    int32_t cur_end = task_meta<LPR>(rend, 0, gbase);
    int32_t cur_out = task_meta<LPR>(rout, 0, gbase);
    double tot[VEC];
    float part[VEC];
#pragma unroll
    for (int j = 0; j < VEC; ++j) {
        tot[j] = 0.0;
        part[j] = 0.f;
    }
    walk_rounds<LPR, VEC, MODE, Q>(
        a, e_begin, e_end, kRound, li, gbase, f, fin,
        [&](int32_t e, float w, const float (&x)[VEC]) {
#pragma unroll
            for (int j = 0; j < VEC; ++j) part[j] = fmaf(w, x[j], part[j]);
            if (e + 1 == cur_end) {           // the current row ends with this entry
#pragma unroll
                for (int j = 0; j < VEC; ++j) {
                    tot[j] += static_cast<double>(part[j]);
                    part[j] = 0.f;
                }
                emit.row(cur_out, gw * kTaskRows + cur, tot, f, fin);
#pragma unroll
                for (int j = 0; j < VEC; ++j) tot[j] = 0.0;
                if (++cur < m) {
                    cur_end = task_meta<LPR>(rend, cur, gbase);
                    cur_out = task_meta<LPR>(rout, cur, gbase);
                }
            }
        },
        [&]() {
#pragma unroll
            for (int j = 0; j < VEC; ++j) {
                tot[j] += static_cast<double>(part[j]);
                part[j] = 0.f;
            }
        });
}

template <int LPR, int VEC, bool BF, int MODE, int Q>
__global__ __launch_bounds__(kThreads) void spmm_dual_kernel(const Args a) {
    const StoreRows<VEC, BF> emit{a.Y, a.ld, a.relu != 0};
    __shared__ double red[shared_sums<LPR, VEC, MODE>()];
    spmm_block<LPR, VEC, kWaves, MODE, Q>(
        a, static_cast<int>(blockIdx.x) / a.S, static_cast<int>(blockIdx.x) % a.S,
        static_cast<int>(threadIdx.x) >> 6, emit, red);
}

// The rows split into parts: row = the sum of its parts' float64 partials, in part order.
// One workgroup per part; only a row's first part does the work (a kernel boundary after
// the SpMM makes every partial visible, so no fence or counter is needed).
template <bool BF>
__global__ __launch_bounds__(kThreads) void combine_kernel(const Args a) {
    const SplitPart sp = a.parts[blockIdx.x];
    if (sp.part != 0) return;
    const int t = static_cast<int>(threadIdx.x);
    const int f = lane_feature<4>(a, t & ~3) + (t & 3);       // fcap keeps nothing back where VEC is 1
    if (a.f0 + (t & ~3) >= a.fend || f >= a.ld) return;
    const double *pp = a.partials + static_cast<int64_t>(sp.first) * kMaxSlice + t;
    double s[1] = {0.0};
    for (int q = 0; q < sp.nparts; ++q) s[0] += pp[static_cast<int64_t>(q) * kMaxSlice];
    store_y<1, BF>(a.Y, static_cast<int64_t>(a.perm[sp.row]) * a.ld + f, s, a.relu);
}

// ---------------- the aggregation fused with the next layer's update
//
// T = bf16(act(A X)) bf16(W), float32 accumulation: the product of a GCN layer's
// aggregated output with the next layer's weights without storing the aggregated
// features.  The aggregation is the plain kernel's (same schedule, same sums); a
// finished row is rounded to bfloat16 into its wavefront's LDS tile (and, if asked,
// also stored to H as the plain kernel's bfloat16 output) instead of Y.
// Every workgroup stages W^T in bfloat16 once and then takes logical workgroups
// blockIdx.x, blockIdx.x + gridDim.x, ... of the plain kernel's schedule (heaviest
// first as before); after each one, the wavefront multiplies its tile by W^T on the
// matrix cores (v_mfma_f32_16x16x32_bf16, 16-row tiles, k in the update kernel's
// order) and writes the finished rows of T.  Rows go through the same bfloat16
// values and the same MFMA sequence as dualgcn_spmm_act with a bfloat16 output
// followed by dualgcn_update, so both routes give identical T.
//
// MFMA 16x16x32 operands (l = lane): A row l % 16 and B column l % 16, eight
// consecutive k of group l / 16; D rows 4 (l / 16) + j, j < 4, column l % 16.
//
// Occupancy.  A wavefront loads its A fragments of a 16-row tile into registers before
// the tile's products, so the tile's LDS rows are free while its results are staged:
// when a 16-row tile of bfloat16 rows is at least as large as the output staging
// (K >= 128), the staging lives in the tile.  At K = 128, N = 64 that takes a workgroup
// from 51 to 35 KiB of LDS, and the kernel is compiled for 4 wavefronts per SIMD
// (at most 128 registers), so four workgroups share a CU instead of three.
constexpr int kXwPad = 8;                     // bfloat16 padding per LDS row
constexpr int kXwBlocksPerGroup = 8;          // logical workgroups per launched workgroup
constexpr int kXwStageLd = 68;                // floats per staged output row (64 + padding)
constexpr int kXwStageWords = 16 * kXwStageLd; // a wavefront's output staging

template <int LPR>
struct XwTile {
    static constexpr int kSlots = (64 / LPR) * kTaskRows;   // rows a wavefront finishes per block
    static constexpr int kRows = kSlots < 16 ? 16 : kSlots; // rows of its LDS tile
};

// Does a 16-row tile of bfloat16 rows K + kXwPad apart hold a wavefront's output staging?
__host__ __device__ constexpr bool xw_stage_in_tile(int K) {
    return (K + kXwPad) * 2 >= kXwStageLd * 4;
}

size_t xw_lds_bytes(int lpr, int K, int N) {
    const int slots = (64 / lpr) * kTaskRows;
    const size_t rows = slots < 16 ? 16 : slots;
    const size_t ld = static_cast<size_t>(K) + kXwPad;
    return (static_cast<size_t>(N) + kWaves * rows) * ld * sizeof(unsigned short) +
           kWaves * rows * sizeof(int32_t) +
           (xw_stage_in_tile(K) ? 0 : static_cast<size_t>(kWaves) * kXwStageWords * sizeof(float));
}

template <int LPR, int MODE, int Q>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4)))
void spmm_xw_kernel(const Args a, const float *__restrict__ W,
                                                           float *__restrict__ T, int32_t K,
                                                           int32_t N, int32_t nblocks) {
    constexpr int ROWS = XwTile<LPR>::kRows;
    extern __shared__ unsigned short xw_lds[];
    const int ld = K + kXwPad;
    const int ntiles = N / 16;
    const int lane = static_cast<int>(threadIdx.x) & 63;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
    unsigned short *wt = xw_lds;                                   // [N][ld]: W^T in bfloat16
    unsigned short *h = xw_lds + (N + wave * ROWS) * ld;           // this wavefront's rows
    int32_t *outs = reinterpret_cast<int32_t *>(xw_lds + (N + kWaves * ROWS) * ld) + wave * ROWS;
    const bool stage_in_tile = xw_stage_in_tile(K);
    float *stage_own = reinterpret_cast<float *>(reinterpret_cast<int32_t *>(xw_lds + (N + kWaves * ROWS) * ld) +
                                                 kWaves * ROWS) + wave * kXwStageWords;
    __shared__ double red[shared_sums<LPR, 4, MODE>()];
    stage_w<kThreads>(wt, ld, W, N, K, N);
    if (lane < ROWS) outs[lane] = -1;
    __syncthreads();

    const StageRows emit{h, outs, ld, a.relu != 0, lane % LPR == 0, static_cast<unsigned short *>(a.Y), a.ld};
    constexpr int KF = LPR / 8;               // A fragments of a row: K <= 4 LPR, 32 k each
    for (int lb = static_cast<int>(blockIdx.x); lb < nblocks; lb += static_cast<int>(gridDim.x)) {
        spmm_block<LPR, 4, kWaves, MODE, Q>(a, lb, 0, wave, emit, red);
        __syncwarp();
        // the lane's MFMA coordinates, recomputed here (hidden from the optimiser) rather
        // than held in registers through the aggregation
        int ln = static_cast<int>(threadIdx.x) & 63;
        asm volatile("" : "+v"(ln));
        const int lrow = ln & 15, kgrp = ln >> 4;
        const int sr = ln >> 4, sc = (ln & 15) * 4;        // first staged row and the columns a lane stores
#pragma unroll
        for (int rt = 0; rt < ROWS / 16; ++rt) {
            if (__ballot(outs[rt * 16 + lrow] >= 0) == 0) continue;   // no row in this tile
            int32_t orow[4];                                          // rows sr + 4 q of the tile
#pragma unroll
            for (int q = 0; q < 4; ++q) orow[q] = outs[rt * 16 + sr + 4 * q];
            const unsigned short *hrow = h + (rt * 16 + lrow) * ld + kgrp * 8;
            u16x8 afrag[KF];
#pragma unroll
            for (int q = 0; q < KF; ++q)
                afrag[q] = q * 32 < K ? *reinterpret_cast<const u16x8 *>(hrow + q * 32) : u16x8{};
            __syncwarp();
            float *stage = stage_in_tile ? reinterpret_cast<float *>(h + rt * 16 * ld) : stage_own;
            // one 16-column tile of T at a time (the k order of each tile is the update's),
            // staged in LDS and stored 64 columns at a time: each store instruction writes
            // four whole 256-byte row pieces (16 lanes x 16 bytes each)
            for (int t = 0; t < ntiles; ++t) {
                const unsigned short *wrow = wt + (t * 16 + lrow) * ld + kgrp * 8;
                f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int q = 0; q < KF; ++q) {
                    if (q * 32 >= K) break;
                    const u16x8 b16 = *reinterpret_cast<const u16x8 *>(wrow + q * 32);
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, afrag[q]),
                                                                  __builtin_bit_cast(bf16x8, b16), acc,
                                                                  0, 0, 0);
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) stage[(kgrp * 4 + j) * kXwStageLd + (t & 3) * 16 + lrow] = acc[j];
                if ((t & 3) == 3 || t == ntiles - 1) {
                    __syncwarp();
                    const int c0 = (t & ~3) * 16;                      // first column of this pass
                    if (c0 + sc < N) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            if (orow[q] >= 0) {
                                const f32x4 v = *reinterpret_cast<const f32x4 *>(stage + (sr + 4 * q) * kXwStageLd + sc);
                                __builtin_nontemporal_store(
                                    v, reinterpret_cast<f32x4 *>(T + static_cast<int64_t>(orow[q]) * N + c0 + sc));
                            }
                        }
                    }
                    __syncwarp();
                }
            }
        }
        __syncwarp();
        if (lane < ROWS) outs[lane] = -1;
        __syncwarp();
    }
}

// The split rows of the fused product: the row from its parts' partials (as in
// combine_kernel), rounded to bfloat16 as row 0 of a tile whose other rows are zero,
// then the same MFMA sequence on the first wavefront with W read from memory.
__global__ __launch_bounds__(kThreads) void combine_xw_kernel(const Args a, const float *__restrict__ W,
                                                              float *__restrict__ T, int32_t K,
                                                              int32_t N) {
    __shared__ unsigned short hrow[kMaxSlice];
    const SplitPart sp = a.parts[blockIdx.x];
    if (sp.part != 0) return;
    const int t = static_cast<int>(threadIdx.x);
    if (t < K) {
        const double *pp = a.partials + static_cast<int64_t>(sp.first) * kMaxSlice + t;
        double sum = 0.0;
        for (int q = 0; q < sp.nparts; ++q) sum += pp[static_cast<int64_t>(q) * kMaxSlice];
        float o = static_cast<float>(sum);
        if (a.relu) o = o > 0.f ? o : 0.f;
        hrow[t] = to_bf16(o);
        if (a.Y) static_cast<unsigned short *>(a.Y)[static_cast<int64_t>(a.perm[sp.row]) * K + t] = hrow[t];
    }
    __syncthreads();
    if (t >= 64) return;
    const int lrow = t & 15, kgrp = t >> 4;
    const int64_t out = static_cast<int64_t>(a.perm[sp.row]) * N;
    for (int u = 0; u < N / 16; ++u) {
        f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int kk = kgrp * 8; kk < K; kk += 32) {
            u16x8 a16, b16;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                a16[e] = lrow == 0 ? hrow[kk + e] : static_cast<unsigned short>(0);
                b16[e] = to_bf16(W[static_cast<int64_t>(kk + e) * N + u * 16 + lrow]);
            }
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a16),
                                                          __builtin_bit_cast(bf16x8, b16), acc, 0, 0, 0);
        }
        if (kgrp == 0) T[out + u * 16 + lrow] = acc[0];
    }
}

// Logical workgroups of the plain kernel's schedule (sets the nb_* fields).
template <int LPR>
int64_t schedule_blocks(Args &a) {
    constexpr int GPB = kThreads / LPR;       // sparse tasks per workgroup
    a.nb_parts = a.coop ? a.n_parts : (a.n_parts + kWaves - 1) / kWaves;
    a.nb_coop = a.n_coop;
    a.nb_long = a.nb_coop + (a.n_long - a.n_coop + kWaves - 1) / kWaves;
    a.nb_dense = a.nb_long + (a.n - a.n_sparse - a.n_long + GPB - 1) / GPB;
    const int64_t nb_sparse = (static_cast<int64_t>(a.n_tasks) + GPB - 1) / GPB;
    return static_cast<int64_t>(a.nb_parts) + a.nb_dense + nb_sparse;
}

template <int LPR, int MODE, int Q>
int launch_xw_window(Args a, const float *W, float *T, int32_t K, int32_t N, hipStream_t s) {
    const int64_t blocks = schedule_blocks<LPR>(a);
    if (blocks > 0x7FFFFFFF) return DUALGCN_ERR_UNSUPPORTED;
    if (blocks > 0) {
        const size_t lds = xw_lds_bytes(LPR, K, N);
        const void *kern = reinterpret_cast<const void *>(&spmm_xw_kernel<LPR, MODE, Q>);
        if (lds > 64 * 1024) {
            const int st = hip_status(hipFuncSetAttribute(
                kern, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)));
            if (st) return st;
        }
        // about kXwBlocksPerGroup logical workgroups each, and at least as many workgroups
        // as fit at once (LDS of one CU: 160 KiB; 2048 threads).  Measured on c5 (F 128 -> 64):
        // one pass of resident workgroups over all blocks is 12% slower than this (its static
        // share of blocks finishes unevenly); blocks of ~4 or fewer pay the W staging again.
        const int64_t per_cu = std::max<int64_t>(1, std::min<int64_t>(2048 / kThreads, (160 * 1024) / lds));
        const int64_t grid = std::min<int64_t>(
            blocks, std::max<int64_t>(per_cu * device_cus(), (blocks + kXwBlocksPerGroup - 1) / kXwBlocksPerGroup));
        hipLaunchKernelGGL((spmm_xw_kernel<LPR, MODE, Q>), dim3(static_cast<unsigned>(grid)), dim3(kThreads),
                           lds, s, a, W, T, K, N, static_cast<int32_t>(blocks));
    }
    if (a.n_parts > 0)
        hipLaunchKernelGGL(combine_xw_kernel, dim3(static_cast<unsigned>(a.n_parts)), dim3(kThreads),
                           0, s, a, W, T, K, N);
    return hip_status(hipGetLastError());
}

template <int LPR, int VEC, int MODE, int Q>
int launch_dual(Args a, int groups, bool bf, hipStream_t s) {
    const int64_t blocks = schedule_blocks<LPR>(a) * a.S;
    if (blocks == 0) return DUALGCN_OK;
    if (blocks > 0x7FFFFFFF) return DUALGCN_ERR_UNSUPPORTED;
    constexpr unsigned own = shared_sums<LPR, VEC, MODE>() * sizeof(double);
    static_assert(own < groups_lds(5, 0), "the padding goes on top of the kernel's own LDS");
    const unsigned lds = groups_lds(groups, own);
    if (bf)
        hipLaunchKernelGGL((spmm_dual_kernel<LPR, VEC, true, MODE, Q>), dim3(static_cast<unsigned>(blocks)),
                           dim3(kThreads), lds, s, a);
    else
        hipLaunchKernelGGL((spmm_dual_kernel<LPR, VEC, false, MODE, Q>), dim3(static_cast<unsigned>(blocks)),
                           dim3(kThreads), lds, s, a);
    return DUALGCN_OK;
}

template <int LPR, int VEC>
int launch_window(const Args &a, const Gathers &g, bool bf, hipStream_t s) {
    constexpr int kHalf = kRound / 2, kQuarter = kRound / 4;
    int st = DUALGCN_ERR_UNSUPPORTED;
    if (g.mode == kWide) {
        st = launch_dual<LPR, VEC, kWide, VEC == 1 ? kHalf : kRound>(a, g.groups, bf, s);
    } else if (g.mode == kClasses) {
        if constexpr (VEC == 4 && LPR >= 32)
            if (g.q == kQuarter) st = launch_dual<LPR, VEC, kClasses, kQuarter>(a, g.groups, bf, s);
        if constexpr (VEC == 4 && LPR >= 8)
            if (g.q == kHalf) st = launch_dual<LPR, VEC, kClasses, kHalf>(a, g.groups, bf, s);
    } else if (g.q == kRound) {
        st = launch_dual<LPR, VEC, kBuffer, kRound>(a, g.groups, bf, s);
    } else {
        if constexpr (VEC == 4 && LPR >= 16)
            st = g.q == kHalf ? launch_dual<LPR, VEC, kBuffer, kHalf>(a, g.groups, bf, s)
                              : launch_dual<LPR, VEC, kBuffer, kQuarter>(a, g.groups, bf, s);
    }
    if (st) return st;
    if (a.n_parts > 0) {
        if (bf)
            hipLaunchKernelGGL((combine_kernel<true>), dim3(static_cast<unsigned>(a.n_parts)),
                               dim3(kThreads), 0, s, a);
        else
            hipLaunchKernelGGL((combine_kernel<false>), dim3(static_cast<unsigned>(a.n_parts)),
                               dim3(kThreads), 0, s, a);
    }
    return hip_status(hipGetLastError());
}

Args plan_args(const Plan &p, const float *X, void *Y, int32_t F, bool relu) {
    Args a{};
    a.pptr = p.pptr;
    a.pcol = p.pcol;
    a.pval = p.pval;
    a.perm = p.order;
    a.tasks = p.tasks;
    a.parts = p.parts;
    a.partials = p.partials;
    a.X = X;
    a.Y = Y;
    a.n = p.n;
    a.n_sparse = p.n_sparse;
    a.n_tasks = p.n_tasks;
    a.n_parts = p.n_split_parts;
    a.dense_chunk = p.dense_chunk;
    a.n_long = p.n_long[0];
    a.ld = F;
    a.relu = relu ? 1 : 0;
    return a;
}

// Lane-group width for a window of w features with four features per lane, and the
// class of the long-row bound that goes with it.
int window_lpr(int32_t w) {
    return w <= 4 ? 1 : w <= 8 ? 2 : w <= 16 ? 4 : w <= 32 ? 8 : w <= 64 ? 16 : w <= 128 ? 32 : 64;
}

// Rows of at least 2^(kLongRowOctave - class) entries get a wavefront: class 1 (256 entries) for
// groups of 16 lanes and wider, an octave less per halving below; class 0 where the launch is
// bound by the memory fabric and rows are wider than 64 features (fused kernel 128 -> 64, n =
// 2^22: 3944 us against 4038, each long row being a 16-row matrix tile of its own there).
// The rule goes by the launch's shape and never by the group's width, so that the fused kernel
// and the SpMM split a row alike.
int long_row_class(int lpr, int mode, int32_t w) {
    int cls = (mode == kClasses || mode == kWide) && w > 64 ? 0 : 1;
    for (int g = lpr; g < 16 && cls < kLongRowClasses - 1; g *= 2) ++cls;
    return cls;
}

// Operands from which a launch of many long rows is bound by the lines it has in flight (see
// pick_gathers).
constexpr uint64_t kThrottleBytes = 88ull << 20;

// Are the rows of at least 2^kLongRowOctave entries and the parts of split rows no more than the
// CUs?  Then a workgroup each starts at once (share_rows), and the launch waits for them; with
// more of them it is bound by what its gathers request.
bool few_long_rows(const Plan &p) { return p.n_long[0] + p.n_split_parts <= device_cus(); }

// Do a workgroup's wavefronts share each long row?  On small graphs the longest row is the whole
// launch: a wavefront takes a row of 4,000 entries in 63 rounds (64 features), four
// together in 16.  Beyond as many such rows and parts as CUs the chip is full without (n = 2^19,
// 1,160 long rows, F = 128: 409 us alone, 430 shared; n = 2^17, 154 long rows and 420 parts, F = 64
// 37.6 / 38.4).  Measured (us) alone / shared: n = 30,007, 120 long rows, F = 64 57 / 22, F = 96
// 103 / 39; n = 20,001, 18 rows, F = 64 24 / 16.
// By the plan and the addressing alone, so the fused kernel and the SpMM add a row alike.
void share_rows(const Plan &p, int mode, Args &a) {
    const bool share = mode == kBuffer && few_long_rows(p);
    a.coop = share ? 1 : 0;
    a.n_coop = share ? p.n_long[0] : 0;
}

// A window of 128 or 256 features whose rows are whole 128-byte lines is cut into slices
// of 64 features, and workgroup b takes slice b % S: workgroups go to the 8 XCDs in turn, so
// an XCD reads every second (or fourth) 256-byte piece of the rows and its 4 MiB L2 keeps twice
// (four times) as many of the hottest rows.  Each slice reads the columns and values again
// (8 bytes an entry against 256 gathered).  Measured, whole rows and slices of 64 (us):
//   F = 128  block model n = 2^18 448 / 424, R-MAT n = 2^19 426 / 376, 1.5M 1031 / 967,
//            n = 2^21 3475 / 3331, n = 2^22 4201 / 4059
//   F = 256  n = 2^19 1036 / 860, 1.5M 2315 / 2048, n = 2^21 7891 / 7053
// Slices of 32 features, whose wavefronts walk eight rows side by side, lose it again (F = 128,
// n = 2^22: 4542).  Three slices (F = 192) do too, since eight XCDs taken in turn see all three
// (n = 2^20, 16.8M entries 1430 / 1570; n = 2^22 4,670 / 4,890), except on small launches that wait
// for a few long rows, where slices are more wavefronts (n = 20,001, 0.3M entries 49 / 29, n = 131,072,
// 0.8M 97 / 79; equal rows of 30 415 / 428).  So do slices
// that share lines or leave lanes idle (1.5M nodes, F = 96 788 / 929, F = 100 1048 / 1492, F = 160
// 1371 / 1592, F = 200 1949 / 2531).  Operands that only memory holds gain nothing without hot rows
// either: every row of 30 entries, n = 400,000, F = 256 2,215 / 2,424; of 20, n = 2^20, F = 128
// 2,056 / 2,115.
bool sliced_window(const Plan &p, int32_t ld, int32_t w) {
    if ((w != 128 && w != 192 && w != 256) || ld % 32 != 0) return false;
    const uint64_t operand = static_cast<uint64_t>(p.n) * w * sizeof(float);
    if (w == 192) return few_long_rows(p) && operand <= kGatherClassMinBytes / 2;
    return p.n_long[0] > 0 || operand <= kGatherClassMinBytes;
}

// Addressing.  Cache classes: the plan marks every column outside the hottest kHotRows; they
// apply from operands larger than the 256 MiB memory-side cache, below which non-temporal loads
// would only lose rows that cache holds, and where rows fill whole 128-byte lines (more than 16
// features).  Measured on R-MAT
// graphs with shuffled ids (c5: n = 2^22, 67M entries; c4: n = 2^21, 63M entries),
// F = 128: the layer-1 aggregation fused with the next update 4.27 -> 4.03 ms (c5) and
// 3.72 -> 3.45 ms (c4), the plain SpMM 4.46 -> 4.24 and 3.70 -> 3.47 ms; the L2 hit rate of
// the fused kernel rose from 22.5% to 26.8% and its fetched bytes fell from 28.6 to 27.0 GB.
// Hot sets of 16 MiB or less, or a third class loading warm rows with sc0, were slower.
//
// Gathers in flight.  16 gathers requested at once by 16 wavefronts a CU are up to 8 MiB of lines
// per XCD, twice its L2, and each request takes the place of a line: where many rows are long
// and the launch is bound by its gathers, fewer in flight are faster.  A short launch waits for
// a part of a split row instead (a chunk's round trips one after the other, four times as many
// in quarter rounds): `deep` says that the launch outlasts it.  Measured on R-MAT graphs of
// degree 5 to 60, n = 20,001 to 2^22, block models and rows of equal length; us, round / half with four
// workgroups a CU / quarter with four:
//   to kThrottleBytes     n = 90,000, 2.8M entries, F = 200 (68 MiB) 203 / 186 / 192; n = 131,072, 8.0M,
//                         F = 160 (80 MiB) 401 / 344 / 343
//   above                 n = 131,072, 8.0M, F = 200 (100 MiB) 616 / 536 / 489; n = 262,143, 16M, F = 100
//                         579 / 574 / 528; n = 2^19, 16.3M, F = 64 337 / 334 / 315
//   above, not deep       n = 2^19, 8.4M, F = 72 285 / 281 / 305 (and F = 200 875 / 884 / 991 under classes)
//   few long rows         n = 20,001, 0.2M, F = 100 22 / 22 / 29; block model n = 2^18, F = 200 798 / 771 /
//                         807, F = 64 208 / 205 / 220
//   classes, 65-96        (half with four / half with five / quarter with five) n = 2^20, 16.8M, F = 96 695
//                         / 681 / 674; n = 750,000, 12M 490 / 475 / 529
//   classes, 97-128       n = 2^20, 16.8M, F = 120 1,051 / 1,051 / 989; n = 2^22, F = 100 3,085 / 3,085 / 3,054
//   classes, 129-192      n = 2^20, F = 160 1,183 / 1,172 / 1,299
//   classes, 193-256      n = 2^21, 65M, F = 200 6,830 / 6,764 / 6,299
// 16-lane groups under classes, and 8-lane ones, keep half a round and every workgroup that fits;
// narrower groups a round (their lines are few).  64-bit addresses: a round (round / half with four:
// n = 8.4M, F = 132 7,183 / 7,311, n = 70M, F = 16 5,098 / 5,192), half of it with one feature a lane
// (n = 358M, F = 3 28.6 ms; four workgroups a CU 44.3), a quarter in the fused kernel (half / quarter:
// 256 -> 32, n = 2^22 8,870 / 8,557; 128 -> 64, n = 8.4M 10,126 / 9,970).  The sums are the same throughout.
Gathers pick_gathers(const Plan &p, int32_t ld, int32_t w, int lpr, Args &a) {
    constexpr int kHalf = kRound / 2, kQuarter = kRound / 4;
    const uint64_t bytes = static_cast<uint64_t>(p.n) * static_cast<uint64_t>(ld) * sizeof(float);
    if (bytes > kMaxBufferBytes) return {kWide, kRound, 0};
    a.x_bytes = static_cast<uint32_t>(bytes);
    const uint64_t operand = static_cast<uint64_t>(p.n) * static_cast<uint64_t>(w) * sizeof(float);
    const bool classes = w > 16 && p.cold_marked && operand > kGatherClassMinBytes;
    if (lpr < 16) return classes ? Gathers{kClasses, kHalf, 0} : Gathers{kBuffer, kRound, 0};
    const bool deep = p.nnz >= int64_t{2560} * p.dense_chunk;
    if (classes) {
        if (lpr == 16) return {kClasses, kHalf, 0};
        if (w <= 96) return {kClasses, kHalf, 5};
        return {kClasses, deep && (w <= 128 || w > 192) ? kQuarter : kHalf, 4};
    }
    if (!few_long_rows(p)) return {kBuffer, deep && operand > kThrottleBytes ? kQuarter : kHalf, 4};
    // few long rows: half a round only where the operand is larger than half the memory-side cache
    // (and, in 16-lane groups, the plan's columns are marked)
    const bool half = operand > kGatherClassMinBytes / 2 && (lpr == 64 || (lpr == 16 && p.cold_marked));
    return half ? Gathers{kBuffer, kHalf, 4} : Gathers{kBuffer, kRound, 0};
}

}  // namespace

size_t spmm_xw_lds_bytes(int32_t F_in, int32_t F_out) {
    return xw_lds_bytes(window_lpr(F_in), F_in, F_out);
}

// The fused junction pays where the aggregation is bound by the memory fabric: the
// operand is larger than the memory-side cache (then the n x F_in intermediate it never
// writes or reads back is traffic saved), and the kernel's LDS still lets at least
// kFusedMinGroups workgroups share a CU.  Measured (F_in -> F_out, fused / the two calls, us), R-MAT
// n = 2^20 (16.8M entries), n = 2^21 (65M), n = 2^22 (67M):
//   128 -> 64   900 / 941, 3,452 / 3,495, 3,937 / 4,334
//    64 -> 32   (256 MiB: two calls) 441 / 464, 1,761 / 1,786, 2,050 / 2,186
//   192 -> 32   1,352 / 1,478, 5,203 / 5,499, 5,895 / 6,660; 192 -> 64 1,511 / 1,513, 5,364 / 5,710, 6,356 / 6,836
//   256 -> 32   1,829 / 1,884, 7,041 / 7,109, 8,465 / 9,287
//   160 -> 32   1,159 / 1,260, 4,279 / 4,665, 4,975 / 5,600; 160 -> 64 1,398 / 1,292, 4,801 / 4,658, 5,837 / 5,796
//   256 -> 64   (two groups: two calls) 2,140 / 1,922, 7,451 / 7,202, 9,409 / 9,417
// and n = 2^18 (4.2M, below the cache) 128 -> 64 257 / 191, 256 -> 32 450 / 375.
constexpr int kFusedMinGroups = 3;

bool fused_junction_pays(const Plan &p, int32_t F_in, int32_t F_out) {
    const size_t lds = xw_lds_bytes(window_lpr(F_in), F_in, F_out);
    const uint64_t groups = (160 * 1024) / lds;
    return static_cast<uint64_t>(p.n) * F_in * sizeof(float) > kGatherClassMinBytes && groups >= kFusedMinGroups;
}

namespace {

// Orders work on stream s after the plan's sorted copy (written on the partition's stream);
// once the copy has been seen complete, launches need no wait (and no barrier packet).
int after_plan(const Plan &p, hipStream_t s) {
    if (!p.ready || p.ready_seen.load(std::memory_order_acquire)) return DUALGCN_OK;
    const hipError_t q = hipEventQuery(p.ready);
    if (q == hipSuccess) {
        p.ready_seen.store(true, std::memory_order_release);
        release_pending(p);
        return DUALGCN_OK;
    }
    if (q != hipErrorNotReady) return hip_status(q);
    return hip_status(hipStreamWaitEvent(s, p.ready, 0));
}

}  // namespace

int launch_spmm_xw(const Plan &p, const float *X, const float *W, float *T, void *H,
                   int32_t F_in, int32_t F_out, bool relu, hipStream_t s) {
    if (const int st = after_plan(p, s)) return st;
    Args a = plan_args(p, X, H, F_in, relu);
    a.f0 = 0;
    a.fend = F_in;
    a.fcap = F_in - 4;
    a.S = 1;
    a.sw = F_in;
    const int lpr = window_lpr(F_in);
    const Gathers g = pick_gathers(p, F_in, F_in, lpr, a);
    a.n_long = p.n_long[long_row_class(lpr, g.mode, F_in)];
    share_rows(p, g.mode, a);
    auto launch = [&](auto width) {
        constexpr int LPR = decltype(width)::value;
        if (g.mode == kWide) return launch_xw_window<LPR, kWide, kRound / 4>(a, W, T, F_in, F_out, s);
        // half a round whatever the width: rows are read whole here, and at most four workgroups
        // fit a CU
        if (g.mode == kClasses) return launch_xw_window<LPR, kClasses, kRound / 2>(a, W, T, F_in, F_out, s);
        if (g.q == kRound) return launch_xw_window<LPR, kBuffer, kRound>(a, W, T, F_in, F_out, s);
        return launch_xw_window<LPR, kBuffer, kRound / 2>(a, W, T, F_in, F_out, s);
    };
    int st = DUALGCN_ERR_UNSUPPORTED;
    if (lpr == 8) st = launch(std::integral_constant<int, 8>());
    else if (lpr == 16) st = launch(std::integral_constant<int, 16>());
    else if (lpr == 32) st = launch(std::integral_constant<int, 32>());
    else if (lpr == 64) st = launch(std::integral_constant<int, 64>());
    if (st) return st;
    return note_use(p, s);
}

int launch_spmm(const Plan &p, const float *X, void *Y, int32_t F, bool relu, bool bf,
                hipStream_t s) {
    if (const int st = after_plan(p, s)) return st;
    Args a = plan_args(p, X, Y, F, relu);

    // Four features per lane from F = 4 on, whatever the rows' alignment: loads and stores of 16
    // bytes need only that of a float (bfloat16 stores are split).  With one feature per lane and
    // groups of 64 an odd width ran at a quarter of it: n = 200,003 (3.4M entries), F = 47
    // 99 us, as 12 lanes of 16 83; block model n = 2^18 (18.8M entries), F = 47 424 -> 205, F = 7
    // 420 -> 152.
    const bool vec = F >= 4;
    a.fcap = vec ? F - 4 : 0x7FFFFFFF - 4;
    int st = DUALGCN_OK;
    for (int32_t f0 = 0, w = 0; f0 < F && !st; f0 += w) {
        // a window's last lane takes its last four features, so a window holds at least four: one
        // to three features past a multiple of kMaxSlice get four of the window before them
        w = std::min(F - f0, kMaxSlice);
        if (vec && F - f0 > w && F - f0 - w < 4) w -= 4;
        a.f0 = f0;
        a.fend = f0 + w;
        if (vec) {
            // the smallest power-of-two lane group with 4 features per lane that holds the
            // window, or slices of 64 features (see sliced_window)
            const int lpr = sliced_window(p, F, w) ? 16 : window_lpr(w);
            a.sw = 4 * lpr;
            a.S = (w + a.sw - 1) / a.sw;
            const Gathers g = pick_gathers(p, F, w, lpr, a);
            a.n_long = p.n_long[long_row_class(lpr, g.mode, w)];
            share_rows(p, g.mode, a);
            if (lpr == 1) st = launch_window<1, 4>(a, g, bf, s);
            else if (lpr == 2) st = launch_window<2, 4>(a, g, bf, s);
            else if (lpr == 4) st = launch_window<4, 4>(a, g, bf, s);
            else if (lpr == 8) st = launch_window<8, 4>(a, g, bf, s);
            else if (lpr == 16) st = launch_window<16, 4>(a, g, bf, s);
            else if (lpr == 32) st = launch_window<32, 4>(a, g, bf, s);
            else st = launch_window<64, 4>(a, g, bf, s);
        } else {
            // F < 4: one feature per lane
            a.sw = 64;
            a.S = (w + 63) / 64;
            const Gathers g = pick_gathers(p, F, w, 1, a);
            share_rows(p, g.mode, a);
            st = launch_window<64, 1>(a, g, bf, s);
        }
    }
    if (st) return st;
    return note_use(p, s);
}

}  // namespace dgc

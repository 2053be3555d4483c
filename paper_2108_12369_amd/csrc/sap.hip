// sap.hip -- string-averaging projections (SAP, Sec. II-D) on a CSR system A x = b
// (see include/pct.h for the method and the arithmetic).
//
//   pct_sap_prepare : k_sap_prepare   one wavefront per row: checks its bounds and
//                                     columns, coefficient lambda / ||a_i||^2 (FP64 sum),
//                                     negated for a row that holds a column twice (found
//                                     with a column bitmap in LDS, or a hash table when
//                                     n is large)
//                     k_sap_levels    which rows of a string can be projected side by side
//                     k_sap_prepare_levels  both, where y is in the workspace and the rows
//                                     are in their natural order
//   pct_sap_iterate : k_sap_levels    (only when the caller gives a row order)
//                     k_sap_string    one workgroup per string, y in LDS (when n floats
//                                     fit): y = x_k, then the relaxed projection of every
//                                     row of the string; y_t to the workspace
//                     k_sap_string_ws one workgroup per string, y in the workspace: eight
//                                     waves load the rows, eight project them
//                     k_sap_average   x_{k+1}[j] = sum_t w_t y_t[j] in FP64, t in order
//
// A string is a chain of row updates, but rows that share no column commute.  A workgroup
// takes the rows of its string in batches, one row per wave, and projects a batch level by
// level (k_sap_levels): the same updates of every component of y in the same order, so the
// result is the one of the rows taken one after another, bit for bit (but for rows that repeat
// a column, whose entries are added in no fixed order).  Measured per iteration, 100 strings:
// 640,000 rows of the paper's 200 x 160 system 3.20 -> 0.67 ms (one row at a time before),
// 368,640 curved rows on 400 x 400 5.85 -> 2.42 ms; with the rows in a random order (nearly
// every pair shares a column) 2.95 -> 1.54 and 5.93 -> 3.91 ms, since the loads and waits of the
// other rows leave the chain.
//
// LDS iterate: the metadata of 64 batches lies in the lanes of each wave, and the first 384
// entries of its next two rows are always in flight.  A row is projected with only as many
// chunks of 64 entries as it spans (a uniform branch on its length picks the body).
//
// Workspace iterate: each row update ends with a wait for its writes to y, and the
// vector-memory counter retires in issue order, so that wait would also drain any row
// loads in flight.  The loads therefore go to other wavefronts, which keep two rows each
// in flight and stage each row (768 entries, values as binary32) in one of two LDS
// slots; the waves meet at a workgroup barrier once per level.  A row whose columns
// are distinct (the prepare pass marks the others) is written back with plain stores,
// which stay in the XCD's L2 for the next row's gathers; global atomic adds would not.
// With several rows at a time the cache lines that a gather or a scattered store touches are
// the limit, not the waits, so y is kept in strips of the grid (YOrder): 4.42 -> 2.42 ms per
// iteration of the 400 x 400 system.
// The staged entries' gathers and stores go through a buffer resource over y: an entry
// past the row gets an offset outside it (the load returns 0, the store is dropped), so
// each chunk is one instruction with no branch around it.
#include "../../include/pct.h"
#include "pct_device.h"
#include "pct_wave.h"

#include <hip/hip_fp16.h>
#include <math.h>
#include <string.h>

namespace pct {
namespace {

constexpr int SAP_WAVES_PREP = 4;   // waves per block of k_sap_prepare
constexpr int SAP_HASH_BITS = 11;   // per-wave column table of k_sap_prepare: 2048 slots
constexpr int SAP_HASH = 1 << SAP_HASH_BITS;
// Ring of rows in flight per wave: D rows ahead, the first PF chunks of 64 entries of each.
// The LDS iterate takes short rows, the workspace iterate (large grids, long curved rows)
// longer ones.
template <bool LDS> struct Ring { static constexpr int D = 2, PF = 6; };
template <> struct Ring<false> { static constexpr int D = 2, PF = 12; };

// Rows of a string projected side by side (see k_sap_levels), one per wave: y in LDS, and
// y in the workspace (there each row has a loading and a projecting wave).
constexpr int SAP_W_LDS = 16, SAP_W_WS = 8;
constexpr int SAP_NAMES_BITS = 14;   // k_sap_prepare_levels' table: 2^14 words, two blocks per CU

struct SapLayout {
    size_t coef_off, lev_off, olev_off, w_off, y_off, total;
};

inline size_t a256(size_t v) { return (v + 255) & ~size_t(255); }

SapLayout sap_layout(int64_t m, int32_t n, int32_t M) {
    SapLayout L;
    L.coef_off = 256;   // [0, 256): status word (same header as the simulator workspace)
    // one byte per position (k_sap_levels): the natural order's, written by prepare only, and
    // those of a caller's order, written by each iterate that is given one
    L.lev_off = L.coef_off + (size_t)m * sizeof(float);
    L.olev_off = L.lev_off + (size_t)m;
    L.w_off = a256(L.olev_off + (size_t)m);
    L.y_off = a256(L.w_off + (size_t)M * sizeof(double));
    L.total = L.y_off + (size_t)M * (size_t)n * sizeof(float);
    return L;
}

// Order of a string's y in the workspace.  Columns of a grid of rows of s voxels go in strips
// of 8 grid rows, each stored by 8-voxel columns: a 128-byte line then holds a patch of 4 x 8
// voxels, which a path leaves after some 6 entries, where a line of 32 voxels of one grid row
// serves a steep path once.  The columns from `full` on (a multiple of 8 s) keep their place;
// full = 0: every column does.  Division by s: c / s = mulhi(c, magic) >> shift, exact for
// c < 2^29 (magic = ceil(2^(32 + shift) / s), 2^shift < s <= 2^(shift + 1)).
struct YOrder {
    uint32_t s, full, magic, shift;
};

__device__ __forceinline__ uint32_t by_s(const YOrder &o, uint32_t c) { return __umulhi(c, o.magic) >> o.shift; }
// place of column c
__device__ __forceinline__ uint32_t y_place(const YOrder &o, uint32_t c) {
    const uint32_t q = by_s(o, c), ix = c - q * o.s, r = q & 7u;
    return c < o.full ? c + 7u * ix + r - r * o.s : c;
}
// column at place i
__device__ __forceinline__ uint32_t y_column(const YOrder &o, uint32_t i) {
    const uint32_t strip = by_s(o, i >> 3), ix = (i >> 3) - strip * o.s;
    return i < o.full ? (8u * strip + (i & 7u)) * o.s + ix : i;
}

struct SapArgs {
    int64_t m, nnz;
    int32_t n, M;
    const int64_t *row_ptr;
    const int32_t *cols;
    const void *vals;
    const float *b;
    const int64_t *order;
    float *coef;
    uint8_t *lev;   // per position: its level in its batch | (levels of the batch - 1) << 4
    int32_t *status;
    uint32_t *row_len;   // in the workspace header (k_sap_row_length)
};

// The order of y for the row length that the prepare pass found (0: every column keeps its
// place).
__device__ __forceinline__ YOrder y_order(const SapArgs &a) {
    const uint32_t s = *a.row_len;
    if (s < 2 || s > (uint32_t)a.n / 8) return YOrder{1, 0, 0, 0};
    YOrder o{s, (uint32_t)a.n / (8 * s) * (8 * s), 0, 31u - (uint32_t)__builtin_clz(s - 1)};
    o.magic = (uint32_t)(((1ull << (32 + o.shift)) + s - 1) / s);
    return o;
}

template <typename VT> __device__ __forceinline__ float val_at(const void *v, int64_t e);
template <> __device__ __forceinline__ float val_at<float>(const void *v, int64_t e) {
    return ((const float *)v)[e];
}
template <> __device__ __forceinline__ float val_at<__half>(const void *v, int64_t e) {
    return __half2float(((const __half *)v)[e]);
}

// A stored value as loaded (binary32, or the 16 bits of a binary16 in a 32-bit register),
// widened only where it is used: converting, or packing two halves into one register,
// right after the load would make the wave wait for it there.
template <typename VT> struct RawOf { using T = float; };
template <> struct RawOf<__half> { using T = uint32_t; };
template <typename VT> __device__ __forceinline__ typename RawOf<VT>::T raw_at(const void *v, int64_t e);
template <> __device__ __forceinline__ float raw_at<float>(const void *v, int64_t e) { return ((const float *)v)[e]; }
template <> __device__ __forceinline__ uint32_t raw_at<__half>(const void *v, int64_t e) {
    return ((const unsigned short *)v)[e];
}
__device__ __forceinline__ float widen(float r) { return r; }
__device__ __forceinline__ float widen(uint32_t r) { return __half2float(__ushort_as_half((unsigned short)r)); }

// Row bounds clamped into [0, nnz]: a row whose stored bounds are outside is empty here
// (and was flagged by the prepare pass).
__device__ __forceinline__ void row_bounds(const SapArgs &a, int64_t i, int64_t &beg, int64_t &end) {
    beg = a.row_ptr[i];
    end = a.row_ptr[i + 1];
    if (beg < 0 || end < beg || end > a.nnz) {
        beg = 0;
        end = 0;
    }
}

// Enters column c of the row tagged `tag` in a wave's open-addressing table (slots hold
// tag << 32 | column; a slot with another tag is free).  True if the row already holds c,
// or if no free slot was found.
__device__ __forceinline__ bool seen_before(unsigned long long *tab, uint32_t tag, int32_t c) {
    const unsigned long long key = ((unsigned long long)tag << 32) | (uint32_t)c;
    uint32_t h = ((uint32_t)c * 2654435761u) >> (32 - SAP_HASH_BITS);
    for (int step = 0; step < SAP_HASH; ++step) {
        unsigned long long cur = tab[h];
        if ((uint32_t)(cur >> 32) != tag) {
            const unsigned long long prev = atomicCAS(&tab[h], cur, key);
            if (prev == cur) return false;   // claimed
            cur = prev;                      // another lane of this row took it
        }
        if (cur == key) return true;
        h = (h + 1) & (SAP_HASH - 1);
    }
    return true;
}

// The coefficient of row i = [beg, end) from each lane's share of the sum of squares, of the
// checks and of the repeats found (one wave; dup in any lane: some column repeats).
template <typename VT>
__device__ __forceinline__ void store_coef(const SapArgs &a, float relax, int64_t i, int64_t beg, int64_t end, double nrm,
                                           bool ok, bool dup, int lane) {
    const bool all_ok = __builtin_amdgcn_ballot_w64(!ok) == 0;
    const bool repeats = __builtin_amdgcn_ballot_w64(dup) != 0;
    if (repeats && all_ok) {
        // ||a_i||^2 of the row as a vector: entries that share a column add into one
        // component, so the sum over entries e of v_e * (sum of the values of e's
        // column), which counts each column's (sum of values)^2 once.  Every lane
        // compares its entries with all of the row's (loads of a uniform index),
        // quadratic in the row length; rows that repeat a column are few.
        nrm = 0.0;
        for (int64_t e0 = beg; e0 < end; e0 += 64) {
            const int64_t e = e0 + lane;
            const int32_t ce = e < end ? a.cols[e] : -1;
            const double ve = e < end ? (double)val_at<VT>(a.vals, e) : 0.0;
            double s = 0.0;
            for (int64_t f = beg; f < end; ++f) {
                const int32_t cf = a.cols[f];
                const double vf = (double)val_at<VT>(a.vals, f);
                s += cf == ce ? vf : 0.0;
            }
            nrm = fma(ve, s, nrm);
        }
    }
    nrm = wave_sum(nrm);
    if (lane == 0) {
        const float cf = (all_ok && nrm > 0.0) ? (float)((double)relax / nrm) : 0.0f;
        a.coef[i] = repeats ? -cf : cf;
        if (!all_ok) set_status_dev(a.status, PCT_EINVAL);
    }
}

// One wavefront per row: bounds and columns checked, coefficient lambda / ||a_i||^2 in
// binary64, the norm of the row as a vector of R^n (entries sharing a column summed into
// one component).  A row that holds some column more than once (a curved path can
// re-enter a voxel), or is too long for the column table, gets its coefficient negated:
// the workspace iterate then adds its updates atomically instead of storing them.
// BITS: the repeats are found with a bitmap of the n columns per wave in dynamic LDS
// (one atomic OR per entry, then the row's words cleared) instead of the hash table.
template <typename VT, bool BITS>
__global__ __launch_bounds__(64 * SAP_WAVES_PREP) void k_sap_prepare(SapArgs a, float relax) {
    extern __shared__ uint32_t bitmaps[];
    const int lane = threadIdx.x & 63;
    unsigned long long *tab = nullptr;
    uint32_t *bm = nullptr;
    if constexpr (BITS) {
        const uint32_t words = ((uint32_t)a.n + 31u) / 32u;
        bm = bitmaps + (size_t)(threadIdx.x >> 6) * words;
        for (uint32_t j = lane; j < words; j += 64) bm[j] = 0u;
    } else {
        __shared__ unsigned long long tabs[SAP_WAVES_PREP][SAP_HASH];
        tab = tabs[threadIdx.x >> 6];
        for (int j = lane; j < SAP_HASH; j += 64) tab[j] = ~0ull;   // tag 0xffffffff: never a row's
    }
    const int64_t wid = (int64_t)blockIdx.x * SAP_WAVES_PREP + (threadIdx.x >> 6);
    const int64_t nw = (int64_t)gridDim.x * SAP_WAVES_PREP;
    uint32_t tag = 0;
    for (int64_t i = wid; i < a.m; i += nw, ++tag) {
        const int64_t beg = a.row_ptr[i], end = a.row_ptr[i + 1];
        bool ok = beg >= 0 && end >= beg && end <= a.nnz;
        const bool hashable = BITS || (ok && end - beg <= SAP_HASH / 2);
        bool dup = false;
        double nrm = 0.0;
        if (ok) {
            // eight chunks of 64 entries loaded before any is used, so that a row's loads
            // overlap (the wave has little else to hide their latency); a row of at most
            // 512 entries is cleared from the columns still in registers
            constexpr int U = 8;
            const bool one_pass = end - beg <= 64 * U;   // uniform
            int32_t cu[U];
            float vu[U];
            for (int64_t e0 = beg + lane; e0 < end; e0 += 64 * U) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int64_t e = e0 + u * 64;
                    cu[u] = e < end ? a.cols[e] : 0;
                    vu[u] = e < end ? val_at<VT>(a.vals, e) : 0.0f;
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (e0 + u * 64 < end) {
                        const int32_t c = cu[u];
                        const bool okc = (uint32_t)c < (uint32_t)a.n;
                        ok = ok && okc;
                        const double v = (double)vu[u];
                        nrm = fma(v, v, nrm);
                        if constexpr (BITS) {
                            if (okc) {
                                const uint32_t bit = 1u << ((uint32_t)c & 31u);
                                if (atomicOr(bm + ((uint32_t)c >> 5), bit) & bit) dup = true;
                            }
                        } else {
                            if (hashable && seen_before(tab, tag, c)) dup = true;
                        }
                    }
                }
            }
            if constexpr (BITS) {
                // the row's words back to zero (the wave's LDS accesses are in order)
                __builtin_amdgcn_wave_barrier();
                if (one_pass) {
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        if (beg + lane + u * 64 < end && (uint32_t)cu[u] < (uint32_t)a.n) bm[(uint32_t)cu[u] >> 5] = 0u;
                } else {
                    for (int64_t e = beg + lane; e < end; e += 64) {
                        const int32_t c = a.cols[e];
                        if ((uint32_t)c < (uint32_t)a.n) bm[(uint32_t)c >> 5] = 0u;
                    }
                }
                __builtin_amdgcn_wave_barrier();
            }
        }
        store_coef<VT>(a, relax, i, beg, end, nrm, ok, !hashable || dup, lane);
        if (a.order && lane == 0) {
            const int64_t o = a.order[i];
            if (o < 0 || o >= a.m) set_status_dev(a.status, PCT_EINVAL);
        }
    }
}

// Metadata of one row of a string, fetched ahead.
struct RowMeta {
    int64_t beg, end;
    float b, coef;
};

__device__ __forceinline__ RowMeta fetch_meta(const SapArgs &a, int64_t s, int64_t s1) {
    RowMeta r{0, 0, 0.0f, 0.0f};
    if (s < s1) {
        const int64_t i = a.order ? a.order[s] : s;
        if (i >= 0 && i < a.m) {
            row_bounds(a, i, r.beg, r.end);
            r.b = a.b[i];
            r.coef = a.coef[i];
        }
    }
    return r;
}

// Batches of a string's rows that can be projected side by side.  A string's positions go
// in batches of W consecutive ones; two rows of a batch that share no column commute, bit
// for bit (neither reads or writes a component of y that the other writes).  A row's level
// is one more than the highest level among the batch's earlier rows that share a column
// with it (0 without one), so that projecting the rows level by level gives every
// component of y the same updates in the same order as row after row.  Consecutive rows of
// a beam lie at random offsets of one or two angles: a batch of 16 rows of the paper's
// 200 x 160 system has 1.7 levels on average, a batch of 8 curved rows on 400 x 400 1.4.
//
// A wave: lane r < W holds the rows of the batch that row r shares a column with, as bits;
// returns row r's byte of a.lev.
template <int W> __device__ __forceinline__ uint8_t level_byte(uint32_t mine, int lane) {
    int lv = 0;
#pragma unroll
    for (int v = 0; v < W; ++v) {   // lane v's level is final here
        const int l = __builtin_amdgcn_readlane(lv, v) + 1;
        if (lane > v && ((mine >> v) & 1u) && l > lv) lv = l;
    }
    int top = 0;
#pragma unroll
    for (int v = 0; v < W; ++v) {
        const int l = __builtin_amdgcn_readlane(lv, v);
        top = l > top ? l : top;
    }
    return (uint8_t)(lv | (top << 4));
}

// One block of W waves per batch, each wave a row.  In LDS a mask of W bits per column
// (of `span` columns at a time): every row sets its bit at its columns, then reads back
// the bits of the others there, then clears them.
template <int W>
__global__ __launch_bounds__(64 * W) void k_sap_levels(SapArgs a, uint32_t span) {
    static_assert(W == 8 || W == 16, "masks of 8 or 16 bits");
    constexpr uint32_t PER = 32 / W, SH = W == 8 ? 2 : 1, MASK = (1u << W) - 1u;
    constexpr int U = 8;   // chunks of 64 entries of the row kept in registers
    extern __shared__ uint32_t tabs[];
    __shared__ uint32_t conf[W];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t words = (span + PER - 1) / PER, n = (uint32_t)a.n;
    for (uint32_t j = threadIdx.x; j < words; j += 64 * W) tabs[j] = 0u;
    const int64_t longest = (a.m + a.M - 1) / a.M, per = (longest + W - 1) / W;
    for (int64_t q = blockIdx.x; q < per * a.M; q += gridDim.x) {
        const int64_t t = q / per, s0 = t * a.m / a.M, s1 = (t + 1) * a.m / a.M;
        const int64_t p0 = s0 + (q - t * per) * W;
        if (p0 >= s1) continue;   // the same for the whole block
        const RowMeta r = fetch_meta(a, p0 + wave, s1);
        int32_t c[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t e = r.beg + u * 64 + lane;
            c[u] = e < r.end ? a.cols[e] : -1;
        }
        const int64_t rest = r.beg + U * 64 + lane;
        uint32_t met = 0u;
        for (uint32_t lo = 0; lo < n; lo += span) {
            const uint32_t len = n - lo < span ? n - lo : span;
            __syncthreads();   // the table is clear
            auto mark = [&](int32_t col) {
                const uint32_t k = (uint32_t)col - lo;
                if (k < len) atomicOr(&tabs[k >> SH], 1u << ((k & (PER - 1)) * W + wave));
            };
            auto read = [&](int32_t col) {
                const uint32_t k = (uint32_t)col - lo;
                if (k < len) met |= tabs[k >> SH] >> ((k & (PER - 1)) * W);
            };
            auto clear = [&](int32_t col) {
                const uint32_t k = (uint32_t)col - lo;
                if (k < len) tabs[k >> SH] = 0u;
            };
#pragma unroll
            for (int u = 0; u < U; ++u) mark(c[u]);
            for (int64_t e = rest; e < r.end; e += 64) mark(a.cols[e]);
            __syncthreads();
#pragma unroll
            for (int u = 0; u < U; ++u) read(c[u]);
            for (int64_t e = rest; e < r.end; e += 64) read(a.cols[e]);
            __syncthreads();
#pragma unroll
            for (int u = 0; u < U; ++u) clear(c[u]);
            for (int64_t e = rest; e < r.end; e += 64) clear(a.cols[e]);
        }
        for (int off = 32; off > 0; off >>= 1) met |= __shfl_xor(met, off, 64);
        if (lane == 0) conf[wave] = met & MASK;
        __syncthreads();
        if (wave == 0) {
            const uint8_t byte = level_byte<W>(lane < W ? conf[lane] : 0u, lane);
            if (lane < W && p0 + lane < s1) a.lev[p0 + lane] = byte;
        }
        __syncthreads();   // conf is read before the next batch writes it
    }
}

// k_sap_prepare and k_sap_levels in one pass over A, for the natural order (whose batches hold
// every row once).  One block per batch, a wave per row.  The rows meet in an LDS table of T
// words: every entry writes its name (its column's high bits, its row, its place in the row) to
// its column's word, then reads the word back.  An entry that finds its own name is done; one
// that finds another of the same column has met that row, or its own: the row repeats a column,
// and the entry is done too, since that one stands for both.  Those that lost write again, and
// so on until all are done: of any two entries of one column in two rows, the later to be done
// met the other.  Nothing is cleared, since a word is only read by those that wrote it, and no
// column is out of the table's range.  The columns and values of the block's next batch are
// loaded meanwhile, those of its next but one are located.
//
// The word is the column modulo T, moved on by 35 at each turn of T columns, which is nearly the
// column modulo T - 35, a prime; it and the high bits give the column.  Modulo T a steep path on
// a grid of 512 voxels per row meets 32 words only, and each round finishes one entry of a word:
// 50,000 steep rows on 512 x 320 (where column bitmaps had taken 0.150 ms) 0.209 -> 0.143 ms,
// on 1024 x 1024 0.98 -> 0.40, on 2048 x 2048 4.9 -> 1.01; 100,000 curved rows on 400 x 400 0.288
// and 0.290.
//
// Bound by the barriers of a batch (three and two per further round; two blocks per CU).  100
// strings of 176M entries in 160,000 columns: k_sap_prepare, whose column bitmaps take an LDS
// atomic per entry, 1.53 ms, then k_sap_levels, which reads the columns again and sets, reads and
// clears its masks, 0.72; this 0.93.  With masks set and read here instead 1.20.  With 16 rows
// per batch (y in LDS) it is no faster than the two: 104M entries in 32,000 columns 0.97 and
// 0.96 ms.  Where the bitmaps do not fit LDS (above 163,840 columns) k_sap_prepare has a hash
// table, whose limit of 1,024 columns per row is not one here: 20,000 rows of 1,283 entries 28.9
// -> 0.31 ms (the longer rows had counted as repeating a column).
//
// A row of more than MAX_LEN entries is taken to meet every other row of its batch (each of its
// entries would have to be named), but whether it repeats a column is found: the block sets its
// columns in the table as a bitmap, 2^19 columns at a time.  Taken as repeating one, it would
// be projected with atomic adds, and its norm found by store_coef in quadratic time: 2,000 rows
// of 5,000 entries in 100,000 columns 53.7 ms, 0.105 so.
template <typename VT>
__global__ __launch_bounds__(64 * SAP_W_WS, 4) void k_sap_prepare_levels(SapArgs a, float relax) {
    constexpr int W = SAP_W_WS, U = 8;         // U: chunks of 64 entries of the row kept in registers
    constexpr uint32_t LOG_T = SAP_NAMES_BITS, T = 1u << LOG_T, ALL = (1u << W) - 1u;
    constexpr int MAX_LEN = 64 * 64;           // entries of a row that the lanes' 64-bit masks follow
    // a name: 16 high bits for the column (below 2^29), 4 for the row, 12 for the place
    static_assert(W <= 16 && MAX_LEN <= 1 << 12 && LOG_T >= 13, "a name fits a word");
    extern __shared__ uint32_t tab[];
    __shared__ uint32_t conf[W], longs;   // longs: rows of more than MAX_LEN entries, as bits
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t n = (uint32_t)a.n;
    if (threadIdx.x < W) conf[threadIdx.x] = 0u;
    if (threadIdx.x == 0) longs = 0u;
    const int64_t longest = (a.m + a.M - 1) / a.M, per = (longest + W - 1) / W, batches = per * a.M;

    struct Batch {
        int64_t p0, s1;      // first position, end of the string
        int64_t beg, end;    // the wave's row
        int32_t c[U];
        typename RawOf<VT>::T v[U];
    };
    auto locate = [&](Batch &b, int64_t q) {   // where batch q and the wave's row of it lie
        const int64_t t = q < batches ? q / per : 0;
        b.p0 = t * a.m / a.M + (q - t * per) * W;
        b.s1 = q < batches ? (t + 1) * a.m / a.M : 0;
        b.beg = b.end = 0;
        if (b.p0 + wave < b.s1) {
            b.beg = a.row_ptr[b.p0 + wave];
            b.end = a.row_ptr[b.p0 + wave + 1];
        }
    };
    auto sound = [&](const Batch &b) { return b.beg >= 0 && b.end >= b.beg && b.end <= a.nnz; };
    auto load = [&](Batch &b) {
        const bool ok = sound(b);
        const int64_t len = ok ? b.end - b.beg : 0;
        const int32_t *cb = a.cols + (ok ? b.beg : 0);
        const void *vb = (const char *)a.vals + (ok ? b.beg : 0) * (int64_t)sizeof(VT);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = u * 64 + lane;
            b.c[u] = e < len ? cb[e] : -1;
            b.v[u] = e < len ? raw_at<VT>(vb, e) : typename RawOf<VT>::T(0);
        }
    };
    auto process = [&](const Batch &b) {
        bool ok = sound(b);
        const int64_t len = ok ? b.end - b.beg : 0;
        const bool huge = len > MAX_LEN;                       // taken to meet every row
        const int chunks = huge ? 0 : (int)((len + 63) / 64);  // uniform in the wave
        const int32_t *cols = a.cols + (ok ? b.beg : 0);
        uint32_t met = 0u;
        bool dup = false;
        uint64_t todo = 0;   // bit u: chunk u's entry is still to be done (a column outside [0, n) is not)
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (!huge && (uint32_t)b.c[u] < n) todo |= 1ull << u;
        for (int u = U; u < chunks; ++u) {
            const int e = u * 64 + lane;
            if (e < len && (uint32_t)cols[e] < n) todo |= 1ull << u;
        }
        auto name = [&](int32_t c, int u) {
            return ((uint32_t)c >> LOG_T) << 16 | (uint32_t)wave << 12 | (uint32_t)(u * 64 + lane);
        };
        auto word = [&](int32_t c) { return ((uint32_t)c + ((uint32_t)c >> LOG_T) * 35u) & (T - 1); };
        auto check = [&](int32_t c, int u) {
            const uint32_t v = tab[word(c)], own = name(c, u);
            bool done = v == own;
            if (!done && (v ^ own) >> 16 == 0) {
                const uint32_t r = (v >> 12) & 15u;
                done = r == (uint32_t)wave;
                dup = dup || done;
                met |= 1u << r;
            }
            if (done) todo &= ~(1ull << u);
        };
        do {
#pragma unroll
            for (int u = 0; u < U; ++u)
                if ((todo >> u) & 1) tab[word(b.c[u])] = name(b.c[u], u);
            for (int u = U; u < chunks; ++u)
                if ((todo >> u) & 1) tab[word(cols[u * 64 + lane])] = name(cols[u * 64 + lane], u);
            __syncthreads();
            if (huge && lane == 0) atomicOr(&longs, 1u << wave);   // (reset before that barrier)
#pragma unroll
            for (int u = 0; u < U; ++u)
                if ((todo >> u) & 1) check(b.c[u], u);
            for (int u = U; u < chunks; ++u)
                if ((todo >> u) & 1) check(cols[u * 64 + lane], u);
        } while (__syncthreads_or(todo != 0));   // one entry of every contested word is done each time
        for (uint32_t rows = longs; rows != 0u; rows &= rows - 1u) {   // the same for the whole block
            const int w = __builtin_ctz(rows);
            const int64_t beg = a.row_ptr[b.p0 + w], end = a.row_ptr[b.p0 + w + 1];
            bool twice = false;
            for (uint32_t lo = 0; lo < n; lo += 32u * T) {
                const uint32_t span = n - lo < 32u * T ? n - lo : 32u * T;
                for (uint32_t j = threadIdx.x; j < (span + 31u) / 32u; j += 64u * W) tab[j] = 0u;
                __syncthreads();
                for (int64_t e = beg + threadIdx.x; e < end; e += 64 * W) {
                    const uint32_t k = (uint32_t)a.cols[e] - lo, bit = 1u << (k & 31u);
                    if (k < span && (atomicOr(&tab[k >> 5], bit) & bit)) twice = true;
                }
                __syncthreads();
            }
            twice = __syncthreads_or(twice);
            if (wave == w) dup = twice;
        }
        for (int off = 32; off > 0; off >>= 1) met |= __shfl_xor(met, off, 64);
        if (huge) met = ALL;
        // a conflict is the later row's: lane r tells row r of this one, lane `wave` keeps its own
        if (lane < W) {
            const uint32_t mine = lane == wave ? met & ((1u << wave) - 1u)
                                               : (lane > wave && ((met >> lane) & 1u) ? 1u << wave : 0u);
            if (mine != 0u) atomicOr(&conf[lane], mine);
        }
        if (b.p0 + wave < b.s1) {
            double nrm = 0.0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const double v = (double)widen(b.v[u]);
                nrm = fma(v, v, nrm);
                ok = ok && ((uint32_t)b.c[u] < n || u * 64 + lane >= b.end - b.beg);
            }
            for (int64_t e = U * 64 + lane; e < len; e += 64) {
                const double v = (double)val_at<VT>(a.vals, b.beg + e);
                nrm = fma(v, v, nrm);
                ok = ok && (uint32_t)cols[e] < n;
            }
            store_coef<VT>(a, relax, b.p0 + wave, b.beg, b.end, nrm, ok, dup, lane);
        }
        __syncthreads();
        if (wave == 0) {
            const uint32_t mine = lane < W ? conf[lane] : 0u;
            if (lane < W) conf[lane] = 0u;   // (the next batch writes it and longs after its barriers)
            if (lane == 0) longs = 0u;
            const uint8_t byte = level_byte<W>(mine, lane);
            if (lane < W && b.p0 + lane < b.s1) a.lev[b.p0 + lane] = byte;
        }
    };
    // batches q, q + g, ...: the one being processed, the next one's entries in flight, the
    // one after that located
    const int64_t g = gridDim.x;
    int64_t q = blockIdx.x;
    Batch A, B;
    locate(A, q);
    load(A);
    locate(B, q + g);
    while (q < batches) {   // the same for the whole block
        load(B);
        Batch C;
        locate(C, q + 2 * g);
        process(A);
        q += g;
        if (q >= batches) break;
        A.p0 = C.p0;
        A.s1 = C.s1;
        A.beg = C.beg;
        A.end = C.end;
        load(A);
        locate(C, q + 2 * g);
        process(B);
        q += g;
        B.p0 = C.p0;
        B.s1 = C.s1;
        B.beg = C.beg;
        B.end = C.end;
    }
}

// Workspace update of a row that holds some column twice.  (A row whose columns are distinct
// is written back with stores, which stay in this XCD's L2, where the next gathers find them;
// an atomic add makes them go further.  The same binary32 arithmetic.)
__device__ __forceinline__ void ws_add(float *y, int32_t c, float v) { unsafeAtomicAdd(y + c, v); }

// Workspace iterate: the wave's writes (performed in L2) are complete before its next
// loads (which read L2).  The fence keeps the compiler from moving memory accesses across.
__device__ __forceinline__ void ws_settle() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// First PF chunks of a row's entries.  The loads are unconditional (an index past the
// row reads a valid entry of the arrays, nnz > 0) so that nothing waits for them here;
// whether an entry belongs to the row is decided where it is used.
template <typename VT, int PF>
__device__ __forceinline__ void fetch_chunks(const SapArgs &a, const RowMeta &r, int lane, int32_t (&c)[PF],
                                             typename RawOf<VT>::T (&v)[PF]) {
    // a uniform base (the row's first entry, or the last entry of the arrays for an empty
    // row at their end) and 32-bit lane offsets clamped to the arrays' end
    const int64_t last = a.nnz - 1;
    const int64_t base = r.beg < last ? r.beg : last;
    const int64_t room = last - base;
    const uint32_t lim = room < 0x7fffffff ? (uint32_t)room : 0x7fffffffu;
    const int32_t *cb = a.cols + base;
    const void *vb = (const char *)a.vals + base * (int64_t)sizeof(VT);
#pragma unroll
    for (int k = 0; k < PF; ++k) {
        const uint32_t o = (uint32_t)(k * 64 + lane) < lim ? (uint32_t)(k * 64 + lane) : lim;
        c[k] = cb[o];
        v[k] = raw_at<VT>(vb, (int64_t)o);
    }
}

// One row of a string projected onto y in LDS with the first NC of the PF prefetched
// chunks in cc / cv (the row holds no entry past them unless NC = PF); the adds are LDS
// atomics, since the entries of a row may share a voxel.
template <typename VT, int PF, int NC>
__device__ __forceinline__ void project_chunks(const SapArgs &a, float *y, const RowMeta &r, uint32_t len,
                                               const int32_t (&cc)[PF], const typename RawOf<VT>::T (&cv)[PF],
                                               int lane) {
    const uint32_t n = (uint32_t)a.n;
    bool ok[NC];
    uint32_t at[NC];
    // an entry past the row or with a bad column takes its lane's spare slot past y, which
    // holds 0 (no branch)
#pragma unroll
    for (int k = 0; k < NC; ++k) {
        ok[k] = (uint32_t)(k * 64 + lane) < len && (uint32_t)cc[k] < n;
        at[k] = ok[k] ? (uint32_t)cc[k] : n + (uint32_t)lane;
    }
    // all gathers in flight before the first use
    float yv[NC];
#pragma unroll
    for (int k = 0; k < NC; ++k) yv[k] = y[at[k]];
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < NC; ++k) acc = fma((double)(ok[k] ? widen(cv[k]) : 0.0f), (double)yv[k], acc);
    const bool tail = NC == PF && len > (uint32_t)(PF * 64);   // uniform
    if (tail) {
        for (int64_t e = r.beg + PF * 64 + lane; e < r.end; e += 64) {
            const int32_t c = a.cols[e];
            const bool okc = (uint32_t)c < n;
            const float yc = y[okc ? c : 0];
            acc = fma((double)(okc ? val_at<VT>(a.vals, e) : 0.0f), (double)yc, acc);
        }
    }
    const double dot = wave_sum(acc);
    const float alpha = (float)(((double)r.b - dot) * (double)fabsf(r.coef));
    // distinct columns: y_c + alpha v stored, the arithmetic of the LDS atomic add, which
    // takes several times as long per lane (16 rows of the paper's system side by side:
    // 2.16 ms per iteration with atomic adds, 0.66 ms with stores)
    if (r.coef > 0.0f) {
#pragma unroll
        for (int k = 0; k < NC; ++k) y[at[k]] = ok[k] ? yv[k] + alpha * widen(cv[k]) : 0.0f;
    } else {
#pragma unroll
        for (int k = 0; k < NC; ++k) atomicAdd(y + at[k], ok[k] ? alpha * widen(cv[k]) : 0.0f);
    }
    if (tail) {
        for (int64_t e = r.beg + PF * 64 + lane; e < r.end; e += 64) {
            const int32_t c = a.cols[e];
            if ((uint32_t)c >= n) continue;
            const float av = alpha * val_at<VT>(a.vals, e);
            if (r.coef > 0.0f) y[c] += av;
            else atomicAdd(y + c, av);
        }
    }
}

template <typename VT, int PF>
__device__ __forceinline__ void project_row(const SapArgs &a, float *y, const RowMeta &r, const int32_t (&cc)[PF],
                                            const typename RawOf<VT>::T (&cv)[PF], int lane) {
    static_assert(PF == 6, "one body per chunk count");
    if (r.coef == 0.0f) return;
    const int64_t len64 = r.end - r.beg;   // a row is shorter than 2^31 entries
    const uint32_t len = len64 < 0x7fffffff ? (uint32_t)len64 : 0x7fffffffu;
    switch ((len + 63) / 64) {   // chunks the row spans (a row with coefficient != 0 has one)
    case 0: break;
    case 1: project_chunks<VT, PF, 1>(a, y, r, len, cc, cv, lane); break;
    case 2: project_chunks<VT, PF, 2>(a, y, r, len, cc, cv, lane); break;
    case 3: project_chunks<VT, PF, 3>(a, y, r, len, cc, cv, lane); break;
    case 4: project_chunks<VT, PF, 4>(a, y, r, len, cc, cv, lane); break;
    case 5: project_chunks<VT, PF, 5>(a, y, r, len, cc, cv, lane); break;
    default: project_chunks<VT, PF, PF>(a, y, r, len, cc, cv, lane); break;
    }
}

// Metadata of 64 positions of a string, one per lane, STEP positions apart, and the levels
// of their batches (`mine`: the position's own level, `top`: the highest of its batch).
struct LaneMeta {
    int64_t beg, end;
    float b, coef;
    int mine, top;
};

// Positions p0 + lane * STEP + w; the batch of lane l starts at p0 + l * STEP.
template <int STEP>
__device__ __forceinline__ LaneMeta lane_meta(const SapArgs &a, int64_t p0, int w, int64_t s1, int lane) {
    const int64_t first = p0 + (int64_t)lane * STEP, p = first + w;
    const RowMeta r = fetch_meta(a, p, s1);
    const int mine = p < s1 ? a.lev[p] & 15 : 0, top = first < s1 ? a.lev[first] >> 4 : 0;
    return LaneMeta{r.beg, r.end, r.b, r.coef, mine, top};
}

// Position `idx` (uniform, < 64) of the lane-held metadata, as scalars.
__device__ __forceinline__ RowMeta meta_at(const LaneMeta &m, int idx) {
    RowMeta r;
    const uint64_t bg = (uint64_t)m.beg, en = (uint64_t)m.end;
    r.beg = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(bg >> 32), idx) << 32) |
                      (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)bg, idx));
    r.end = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(en >> 32), idx) << 32) |
                      (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)en, idx));
    r.b = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, m.b), idx));
    r.coef = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, m.coef), idx));
    return r;
}

// Barrier between the waves of a string: their LDS accesses before it happen before those
// after it (lgkmcnt(0), s_barrier); global loads stay in flight.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <typename VT>
__global__ __launch_bounds__(64 * SAP_W_LDS) void k_sap_string(SapArgs a, const float *x, float *Y) {
    extern __shared__ float ys[];
    constexpr int D = Ring<true>::D, PF = Ring<true>::PF, W = SAP_W_LDS;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t = blockIdx.x;
    const int n = a.n;
    float *yg = Y + (size_t)t * (size_t)n;
    float *y = ys;
    for (int j = threadIdx.x; j < n; j += blockDim.x) y[j] = x[j];
    if (wave == 0) y[n + lane] = 0.0f;   // the spare slots
    __syncthreads();
    if (a.nnz > 0) {   // (else every row is empty: nothing to load, and no entry to clamp to)
        // Batch k of the string is positions s0 + k W + wave, one per wave; the metadata of
        // 64 batches lies in the lanes (this group in A, the next one in B).  Slot j of the
        // ring holds the first PF chunks of the wave's row of batch j (mod D), refilled as
        // soon as the batch is projected.
        const int64_t s0 = (int64_t)t * a.m / a.M, s1 = (int64_t)(t + 1) * a.m / a.M;
        const int64_t nb = (s1 - s0 + W - 1) / W;
        LaneMeta A = lane_meta<W>(a, s0, wave, s1, lane), B = lane_meta<W>(a, s0 + 64 * W, wave, s1, lane);
        int32_t cq[D][PF];
        typename RawOf<VT>::T vq[D][PF];
#pragma unroll
        for (int j = 0; j < D; ++j) {
            fetch_chunks<VT, PF>(a, meta_at(A, j), lane, cq[j], vq[j]);
            __builtin_amdgcn_sched_barrier(0);   // slots filled in order
        }
        static_assert(64 % D == 0, "whole ring turns per group");
        for (int64_t k0 = 0; k0 < nb; k0 += 64) {
            // whole ring turns: the batches past the string have no row and one level
            const int kn = nb - k0 < 64 ? (int)(nb - k0) : 64;
            for (int j0 = 0; j0 < kn; j0 += D) {
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    const RowMeta r = meta_at(A, j0 + j);
                    const int mine = __builtin_amdgcn_readlane(A.mine, j0 + j);
                    const int top = __builtin_amdgcn_readlane(A.top, j0 + j);
                    for (int l = 0; l <= top; ++l) {   // the same count in every wave
                        if (l == mine) project_row<VT, PF>(a, y, r, cq[j], vq[j], lane);
                        lds_barrier();
                    }
                    const int nx = j0 + j + D;
                    fetch_chunks<VT, PF>(a, nx < 64 ? meta_at(A, nx) : meta_at(B, nx - 64), lane, cq[j], vq[j]);
                }
            }
            A = B;
            B = lane_meta<W>(a, s0 + (k0 + 128) * W, wave, s1, lane);
        }
    }
    __syncthreads();
    for (int j = threadIdx.x; j < n; j += blockDim.x) yg[j] = ys[j];
}

// Buffer access to a string's y (n binary32): an offset at or past 4 n bytes is outside
// the resource (n < 2^29, checked on the host, so Y_OUT always is).  Cache policy as the
// workgroup-scope accesses above.
constexpr uint32_t Y_OUT = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t y_rsrc(float *y, int32_t n) {
    return __builtin_amdgcn_make_buffer_rsrc(y, (short)0, n * 4, 0x00020000);
}
__device__ __forceinline__ float yb_load(__amdgpu_buffer_rsrc_t r, uint32_t off) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 1));
}
__device__ __forceinline__ void yb_store(__amdgpu_buffer_rsrc_t r, uint32_t off, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, off, 0, 1);
}

// One staged row projected onto y in the workspace (cf: its signed coefficient).  Its
// updates are complete when it returns.
template <typename VT>
__device__ __forceinline__ void project_ws(const SapArgs &a, const YOrder &o, float *y, __amdgpu_buffer_rsrc_t yr,
                                           uint32_t nu, const int32_t *sc, const float *sv, int64_t beg, int64_t end, float b,
                                           float cf, int lane) {
    constexpr int PF = Ring<false>::PF, SLOT = PF * 64;
    if (cf == 0.0f) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");   // the other waves' updates before the barrier
    const bool repeats = cf < 0.0f;   // some column twice: atomic adds
    const float coef = fabsf(cf);
    int32_t cc[PF];
    float cv[PF], yv[PF];
    bool ok[PF];
#pragma unroll
    for (int q = 0; q < PF; ++q) {
        cc[q] = sc[q * 64 + lane];
        cv[q] = sv[q * 64 + lane];
        ok[q] = beg + q * 64 + lane < end && (uint32_t)cc[q] < nu;
    }
#pragma unroll
    for (int q = 0; q < PF; ++q) yv[q] = yb_load(yr, ok[q] ? (uint32_t)cc[q] * 4u : Y_OUT);
    double acc = 0.0;
#pragma unroll
    for (int q = 0; q < PF; ++q) acc = fma(ok[q] ? (double)cv[q] : 0.0, (double)yv[q], acc);
    // the entries past the slot, REST chunks of 64 with their loads in flight together (rows of
    // 1,283 entries, 1200 x 1200: 2.92 ms per iteration with one chunk at a time, 2.48 so)
    constexpr int REST = 4;
    uint32_t rc[REST];   // byte offset of y's component, or out of range
    float rv[REST], ry[REST];
    auto fetch_rest = [&](int64_t e0, bool gather) {
#pragma unroll
        for (int u = 0; u < REST; ++u) {
            const int64_t e = e0 + u * 64 + lane;
            const int32_t c = e < end ? a.cols[e] : -1;
            rv[u] = e < end ? val_at<VT>(a.vals, e) : 0.0f;
            rc[u] = (uint32_t)c < nu ? y_place(o, (uint32_t)c) * 4u : Y_OUT;
        }
        if (gather) {
#pragma unroll
            for (int u = 0; u < REST; ++u) ry[u] = yb_load(yr, rc[u]);
        }
    };
    for (int64_t e0 = beg + SLOT; e0 < end; e0 += 64 * REST) {
        fetch_rest(e0, true);
#pragma unroll
        for (int u = 0; u < REST; ++u) acc = fma(rc[u] != Y_OUT ? (double)rv[u] : 0.0, (double)ry[u], acc);
    }
    const double dot = wave_sum(acc);
    const float alpha = (float)(((double)b - dot) * (double)coef);
    if (repeats) {
#pragma unroll
        for (int q = 0; q < PF; ++q)
            if (ok[q]) ws_add(y, cc[q], alpha * cv[q]);
        for (int64_t e0 = beg + SLOT; e0 < end; e0 += 64 * REST) {
            fetch_rest(e0, false);
#pragma unroll
            for (int u = 0; u < REST; ++u)
                if (rc[u] != Y_OUT) ws_add(y, (int32_t)(rc[u] >> 2), alpha * rv[u]);
        }
    } else {
#pragma unroll
        for (int q = 0; q < PF; ++q) yb_store(yr, ok[q] ? (uint32_t)cc[q] * 4u : Y_OUT, yv[q] + alpha * cv[q]);
        for (int64_t e0 = beg + SLOT; e0 < end; e0 += 64 * REST) {
            fetch_rest(e0, true);
#pragma unroll
            for (int u = 0; u < REST; ++u) yb_store(yr, rc[u], ry[u] + alpha * rv[u]);
        }
    }
    ws_settle();
}

template <typename VT>
__global__ __launch_bounds__(128 * SAP_W_WS) void k_sap_string_ws(SapArgs a, const float *x, float *Y) {
    constexpr int D = Ring<false>::D, PF = Ring<false>::PF, SLOT = PF * 64, W = SAP_W_WS;
    __shared__ int32_t sc[2][W][SLOT];
    __shared__ float sv[2][W][SLOT];
    __shared__ int64_t sbeg[2][W], send[2][W];
    __shared__ float sb[2][W], scoef[2][W];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int w = wave % W;   // the row of each batch that the wave loads or projects
    const int t = blockIdx.x;
    const int n = a.n;
    float *y = Y + (size_t)t * (size_t)n;
    const YOrder o = y_order(a);
    for (int j = threadIdx.x; j < n; j += 128 * W) y[j] = x[y_column(o, j)];
    __syncthreads();   // (global and LDS) the copy is in L2 before the first gathers
    if (a.nnz == 0) return;   // every row empty (all waves leave here)

    const int64_t s0 = (int64_t)t * a.m / a.M, s1 = (int64_t)(t + 1) * a.m / a.M;
    const int64_t nb = (s1 - s0 + W - 1) / W;
    // Step k: the loaders stage batch k in slot k & 1 while the projectors project batch
    // k - 1 from slot (k - 1) & 1, level by level.  All waves take the same number of steps
    // (nb + 1 rounded up to a multiple of D) and the barriers of each (one per level of
    // batch k - 1); rows past the string are empty (coefficient 0, level 0).
    static_assert(D % 2 == 0 && 64 % D == 0, "ring depth");
    const int64_t steps = (nb + D) / D * D;
    LaneMeta A = lane_meta<W>(a, s0, w, s1, lane), B = lane_meta<W>(a, s0 + 64 * W, w, s1, lane);
    if (wave >= W) {
        // loader: ring of D rows whose first SLOT entries are in flight
        int32_t cq[D][PF];
        typename RawOf<VT>::T vq[D][PF];
        // the slots are filled in order (the scheduler may not interleave them), so a
        // slot's loads are always older than those of the slots after it
#pragma unroll
        for (int j = 0; j < D; ++j) {
            fetch_chunks<VT, PF>(a, meta_at(A, j), lane, cq[j], vq[j]);
            __builtin_amdgcn_sched_barrier(0);
        }
        int top = 0;   // of the batch being projected
        for (int64_t k0 = 0; k0 < steps; k0 += 64) {
            const int jn = steps - k0 < 64 ? (int)(steps - k0) : 64;
            for (int j0 = 0; j0 < jn; j0 += D) {
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    const int slot = j & 1;   // = k & 1, as k0 and j0 are even
                    const RowMeta r = meta_at(A, j0 + j);
#pragma unroll
                    for (int q = 0; q < PF; ++q) {
                        sc[slot][w][q * 64 + lane] = (int32_t)y_place(o, (uint32_t)cq[j][q]);
                        sv[slot][w][q * 64 + lane] = widen(vq[j][q]);
                    }
                    if (lane == 0) {
                        sbeg[slot][w] = r.beg;
                        send[slot][w] = r.end;
                        sb[slot][w] = r.b;
                        scoef[slot][w] = r.coef;
                    }
                    const int nx = j0 + j + D;
                    const RowMeta mn = nx < 64 ? meta_at(A, nx) : meta_at(B, nx - 64);
                    fetch_chunks<VT, PF>(a, mn, lane, cq[j], vq[j]);
                    for (int l = 0; l <= top; ++l) lds_barrier();
                    top = __builtin_amdgcn_readlane(A.top, j0 + j);
                }
            }
            A = B;
            B = lane_meta<W>(a, s0 + (k0 + 128) * W, w, s1, lane);
        }
    } else {
        // projector
        const uint32_t nu = (uint32_t)n;
        const __amdgpu_buffer_rsrc_t yr = y_rsrc(y, n);
        lds_barrier();   // step 0: nothing is staged yet
        for (int64_t k0 = 0; k0 < steps - 1; k0 += 64) {
            const int jn = steps - 1 - k0 < 64 ? (int)(steps - 1 - k0) : 64;
            for (int j = 0; j < jn; ++j) {
                const int slot = j & 1;   // batch k0 + j, k0 even
                const int mine = __builtin_amdgcn_readlane(A.mine, j), top = __builtin_amdgcn_readlane(A.top, j);
                for (int l = 0; l <= top; ++l) {
                    if (l == mine) project_ws<VT>(a, o, y, yr, nu, sc[slot][w], sv[slot][w], sbeg[slot][w], send[slot][w],
                                                  sb[slot][w], scoef[slot][w], lane);
                    // the next level's gathers, by any wave, see this level's updates
                    lds_barrier();
                }
            }
            A = B;
            B = lane_meta<W>(a, s0 + (k0 + 128) * W, w, s1, lane);
        }
    }
}

// STRIPS: y in the order of the workspace iterate.
template <bool STRIPS>
__global__ void k_sap_average(SapArgs a, const float *Y, const double *w, int32_t M, int32_t n, float *x) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    double s = 0.0;
#pragma unroll 8
    for (int32_t t = 0; t < M; ++t) s = fma(w[t], (double)Y[(size_t)t * (size_t)n + (size_t)j], s);
    x[STRIPS ? y_column(y_order(a), (uint32_t)j) : (uint32_t)j] = (float)s;
}

// The row length s of the grid the columns come from: consecutive entries of a path lie in
// neighbouring voxels, so their columns differ by 1 or s (or a plane).  The most frequent
// difference above 1 of 8,192 pairs spread over the entries, if an eighth of them show it and
// 8 rows of s fit n; else the columns keep their places.  Any s is correct.
constexpr int LEN_PAIRS = 8192, LEN_SLOTS = 2048, LEN_THREADS = 1024;
__global__ __launch_bounds__(LEN_THREADS) void k_sap_row_length(SapArgs a) {
    __shared__ uint32_t key[LEN_SLOTS], num[LEN_SLOTS];
    __shared__ unsigned long long best;
    for (int j = threadIdx.x; j < LEN_SLOTS; j += LEN_THREADS) key[j] = num[j] = 0u;
    if (threadIdx.x == 0) best = 0ull;
    __syncthreads();
    const int64_t pairs = a.nnz - 1 < LEN_PAIRS ? a.nnz - 1 : LEN_PAIRS;
    for (int64_t k = threadIdx.x; k < pairs; k += LEN_THREADS) {
        const int64_t e = (int64_t)((double)k * ((double)(a.nnz - 1) / (double)pairs));   // < nnz - 1
        int64_t d = (int64_t)a.cols[e + 1] - a.cols[e];
        d = d < 0 ? -d : d;
        if (d < 2 || d > a.n / 8) continue;
        uint32_t h = ((uint32_t)d * 2654435761u) >> 21;
        for (int step = 0; step < 16; ++step, h = (h + 1) & (LEN_SLOTS - 1)) {
            const uint32_t was = atomicCAS(&key[h], 0u, (uint32_t)d);
            if (was == 0u || was == (uint32_t)d) {
                atomicAdd(&num[h], 1u);
                break;
            }
        }
    }
    __syncthreads();
    for (int j = threadIdx.x; j < LEN_SLOTS; j += LEN_THREADS)
        atomicMax(&best, ((unsigned long long)num[j] << 32) | key[j]);
    __syncthreads();
    if (threadIdx.x == 0) *a.row_len = (best >> 32) * 8 >= (unsigned long long)pairs ? (uint32_t)best : 0u;
}

__global__ void k_sap_uniform(double *w, int32_t M) {
    const int32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < M) w[t] = 1.0 / (double)M;
}

// Levels of rows one after another, right for any order: strings of one row (level 0), and what
// a prepare with a caller's order leaves for an iterate without it.
__global__ void k_sap_one_by_one(SapArgs a, int W) {
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < a.m; p += step) {
        const int64_t t = ((p + 1) * a.M - 1) / a.m;   // the string of position p
        const int64_t s0 = t * a.m / a.M, s1 = (t + 1) * a.m / a.M;
        const int64_t lv = (p - s0) % W, rows = s1 - (p - lv);
        a.lev[p] = (uint8_t)(lv | ((rows < W ? rows : W) - 1) << 4);
    }
}

__global__ void k_sap_clear_status(int32_t *status) {
    if (threadIdx.x == 0) *status = PCT_OK;
}

pct_status check_sap(const pct_csr *A, const pct_sap *p) {
    if (!A || !p) return PCT_EINVAL;
    if (A->n_rows < 0 || A->n_cols < 1 || A->nnz < 0) return PCT_EINVAL;
    if (A->val_dtype != PCT_F32 && A->val_dtype != PCT_F16) return PCT_EINVAL;
    if (!A->row_ptr_dev) return PCT_EINVAL;
    if (A->n_rows > 0 && (!A->b_dev || (A->nnz > 0 && (!A->cols_dev || !A->vals_dev)))) return PCT_EINVAL;
    if (p->n_strings < 1) return PCT_EINVAL;
    if (!(p->relax > 0.0f && p->relax < 2.0f)) return PCT_EINVAL;
    if (p->weights) {
        double sum = 0.0;
        for (int32_t t = 0; t < p->n_strings; ++t) {
            const double w = p->weights[t];
            if (!(w >= 0.0) || !isfinite(w)) return PCT_EINVAL;
            sum += w;
        }
        if (!(fabs(sum - 1.0) <= 1e-9)) return PCT_EINVAL;
    }
    // (t + 1) * m must not overflow int64; the string iterates must be addressable
    if ((double)A->n_rows * (double)p->n_strings > 9.0e18) return PCT_ERANGE;
    if ((double)p->n_strings * (double)A->n_cols * 4.0 > 4.0e18) return PCT_ERANGE;
    if (A->n_cols >= (1 << 29)) return PCT_ERANGE;   // byte offsets into one string's y
    return PCT_OK;
}

SapArgs make_args(const pct_csr *A, const pct_sap *p, char *ws, const SapLayout &L) {
    SapArgs a;
    a.m = A->n_rows;
    a.nnz = A->nnz;
    a.n = A->n_cols;
    a.M = p->n_strings;
    a.row_ptr = A->row_ptr_dev;
    a.cols = A->cols_dev;
    a.vals = A->vals_dev;
    a.b = A->b_dev;
    a.order = p->order_dev;
    a.coef = (float *)(ws + L.coef_off);
    a.lev = (uint8_t *)(ws + L.lev_off);
    a.status = (int32_t *)ws;
    a.row_len = (uint32_t *)(ws + 64);
    return a;
}

// Largest dynamic LDS of one workgroup on the current device.
size_t lds_limit() {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) return 0;
    return v > 0 ? (size_t)v : 0;
}

// Whether a string's iterate (and one spare slot per lane, the target of the adds of
// entries past a row) fits a workgroup's LDS.
bool y_in_lds(int32_t n) { return ((size_t)n + 64) * sizeof(float) <= lds_limit(); }

// Positions of the longest string.
int64_t longest_string(const SapArgs &a) { return (a.m + a.M - 1) / a.M; }

// The levels of every batch of the strings (k_sap_levels), for the iterate that n takes.
template <int W>
pct_status launch_levels_w(const SapArgs &a, hipStream_t s) {
    const size_t room = lds_limit() > 1024 ? (lds_limit() - 1024) & ~size_t(15) : 0;
    const size_t cols = room * 8 / W;   // W bits per column
    const uint32_t span = (size_t)a.n < cols ? (uint32_t)a.n : (uint32_t)cols;
    if (span == 0) return PCT_EHIP;
    const size_t bytes = ((size_t)span * W / 8 + 3) / 4 * 4 + 4;
    const int64_t per = (longest_string(a) + W - 1) / W, batches = per * a.M;
    const unsigned blocks = (unsigned)(batches < 2048 ? batches : 2048);
    if (hipFuncSetAttribute((const void *)k_sap_levels<W>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) !=
        hipSuccess)
        return PCT_EHIP;
    hipLaunchKernelGGL((k_sap_levels<W>), dim3(blocks), dim3(64 * W), bytes, s, a, span);
    return hipGetLastError() == hipSuccess ? PCT_OK : PCT_EHIP;
}
pct_status launch_one_by_one(const SapArgs &a, hipStream_t s) {
    if (a.m == 0) return PCT_OK;
    const int64_t blocks = (a.m + 255) / 256;
    hipLaunchKernelGGL(k_sap_one_by_one, dim3((unsigned)(blocks < 65536 ? blocks : 65536)), dim3(256), 0, s, a,
                       y_in_lds(a.n) ? SAP_W_LDS : SAP_W_WS);
    return hipGetLastError() == hipSuccess ? PCT_OK : PCT_EHIP;
}

pct_status launch_levels(const SapArgs &a, hipStream_t s) {
    if (a.m == 0 || a.nnz == 0) return PCT_OK;   // no row to project
    if (longest_string(a) == 1) return launch_one_by_one(a, s);   // every batch is one row
    return y_in_lds(a.n) ? launch_levels_w<SAP_W_LDS>(a, s) : launch_levels_w<SAP_W_WS>(a, s);
}

template <typename VT>
pct_status launch_prepare_levels(const SapArgs &a, float relax, hipStream_t s) {
    constexpr int bytes = 4 << SAP_NAMES_BITS;
    const int64_t per = (longest_string(a) + SAP_W_WS - 1) / SAP_W_WS, batches = per * a.M;
    const unsigned blocks = (unsigned)(batches < 1024 ? batches : 1024);
    if (hipFuncSetAttribute((const void *)k_sap_prepare_levels<VT>, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) !=
        hipSuccess)
        return PCT_EHIP;
    hipLaunchKernelGGL((k_sap_prepare_levels<VT>), dim3(blocks), dim3(64 * SAP_W_WS), bytes, s, a, relax);
    return hipGetLastError() == hipSuccess ? PCT_OK : PCT_EHIP;
}

template <typename VT>
pct_status launch_strings(const SapArgs &a, const float *x, float *Y, hipStream_t s) {
    const size_t bytes = ((size_t)a.n + 64) * sizeof(float);
    if (y_in_lds(a.n)) {
        if (hipFuncSetAttribute((const void *)k_sap_string<VT>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)bytes) != hipSuccess)
            return PCT_EHIP;
        // strings shorter than a batch: only the waves that have a row
        const int64_t waves = longest_string(a) < SAP_W_LDS ? longest_string(a) : SAP_W_LDS;
        hipLaunchKernelGGL((k_sap_string<VT>), dim3((unsigned)a.M), dim3(64 * (unsigned)(waves > 1 ? waves : 1)), bytes,
                           s, a, x, Y);
    } else {
        hipLaunchKernelGGL((k_sap_string_ws<VT>), dim3((unsigned)a.M), dim3(128 * SAP_W_WS), 0, s, a, x, Y);
    }
    return hipGetLastError() == hipSuccess ? PCT_OK : PCT_EHIP;
}

}  // namespace
}  // namespace pct

using namespace pct;

extern "C" {

size_t pct_sap_workspace_bytes(const pct_csr *A, const pct_sap *p) {
    if (check_sap(A, p) != PCT_OK) return 0;
    return sap_layout(A->n_rows, A->n_cols, p->n_strings).total;
}

pct_status pct_sap_prepare(const pct_csr *A, const pct_sap *p, void *ws_dev, size_t ws_bytes, void *stream) {
    const pct_status st = check_sap(A, p);
    if (st != PCT_OK) return st;
    const SapLayout L = sap_layout(A->n_rows, A->n_cols, p->n_strings);
    if (!ws_dev || ws_bytes < L.total) return PCT_EWORKSPACE;
    if (p->n_strings > (1 << 30)) return PCT_ERANGE;
    hipStream_t s = (hipStream_t)stream;
    char *ws = (char *)ws_dev;
    const SapArgs a = make_args(A, p, ws, L);
    hipLaunchKernelGGL(k_sap_clear_status, dim3(1), dim3(64), 0, s, a.status);
    // weights in FP64 (uniform: 1/M)
    const int32_t M = p->n_strings;
    double *w = (double *)(ws + L.w_off);
    if (p->weights) {
        if (hipMemcpyAsync(w, p->weights, (size_t)M * sizeof(double), hipMemcpyHostToDevice, s) != hipSuccess)
            return PCT_EHIP;
    } else {
        hipLaunchKernelGGL(k_sap_uniform, dim3((unsigned)((M + 255) / 256)), dim3(256), 0, s, w, M);
    }
    // One pass for the coefficients and the levels (k_sap_prepare_levels) where y is in the
    // workspace; strings of fewer rows than two batches leave too many of its waves without one.
    const bool together = !p->order_dev && A->nnz > 0 && !y_in_lds(A->n_cols) && longest_string(a) >= 2 * SAP_W_WS;
    if (together) {
        const pct_status ls = A->val_dtype == PCT_F16 ? launch_prepare_levels<__half>(a, p->relax, s)
                                                      : launch_prepare_levels<float>(a, p->relax, s);
        if (ls != PCT_OK) return ls;
    } else if (A->n_rows > 0) {
        const int64_t blocks64 = (A->n_rows + SAP_WAVES_PREP - 1) / SAP_WAVES_PREP;
        const unsigned blocks = (unsigned)(blocks64 < 65536 ? blocks64 : 65536);
        // a column bitmap per wave when two blocks of them fit a CU's LDS, else the hash
        const size_t bm_bytes = (size_t)SAP_WAVES_PREP * (((size_t)A->n_cols + 31) / 32) * sizeof(uint32_t);
        const bool bits = 2 * bm_bytes <= lds_limit();
        if (bits) {
            const void *k = A->val_dtype == PCT_F16 ? (const void *)k_sap_prepare<__half, true>
                                                    : (const void *)k_sap_prepare<float, true>;
            if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bm_bytes) != hipSuccess)
                return PCT_EHIP;
            if (A->val_dtype == PCT_F16)
                hipLaunchKernelGGL((k_sap_prepare<__half, true>), dim3(blocks), dim3(64 * SAP_WAVES_PREP), bm_bytes, s,
                                   a, p->relax);
            else
                hipLaunchKernelGGL((k_sap_prepare<float, true>), dim3(blocks), dim3(64 * SAP_WAVES_PREP), bm_bytes, s,
                                   a, p->relax);
        } else if (A->val_dtype == PCT_F16) {
            hipLaunchKernelGGL((k_sap_prepare<__half, false>), dim3(blocks), dim3(64 * SAP_WAVES_PREP), 0, s, a,
                               p->relax);
        } else {
            hipLaunchKernelGGL((k_sap_prepare<float, false>), dim3(blocks), dim3(64 * SAP_WAVES_PREP), 0, s, a,
                               p->relax);
        }
    }
    if (!y_in_lds(A->n_cols) && A->nnz > 0) hipLaunchKernelGGL(k_sap_row_length, dim3(1), dim3(LEN_THREADS), 0, s, a);
    if (hipGetLastError() != hipSuccess) return PCT_EHIP;
    if (p->order_dev) return launch_one_by_one(a, s);
    return together ? PCT_OK : launch_levels(a, s);
}

pct_status pct_sap_iterate(const pct_csr *A, const pct_sap *p, float *x_dev, int32_t n_iter, void *ws_dev,
                           size_t ws_bytes, void *stream) {
    const pct_status st = check_sap(A, p);
    if (st != PCT_OK) return st;
    if (n_iter < 0 || !x_dev) return PCT_EINVAL;
    const SapLayout L = sap_layout(A->n_rows, A->n_cols, p->n_strings);
    if (!ws_dev || ws_bytes < L.total) return PCT_EWORKSPACE;
    if (p->n_strings > (1 << 30)) return PCT_ERANGE;
    hipStream_t s = (hipStream_t)stream;
    char *ws = (char *)ws_dev;
    SapArgs a = make_args(A, p, ws, L);
    if (p->order_dev) a.lev = (uint8_t *)(ws + L.olev_off);
    float *Y = (float *)(ws + L.y_off);
    const double *w = (const double *)(ws + L.w_off);
    const unsigned avg_blocks = (unsigned)((A->n_cols + 255) / 256);
    // the levels of the natural order are the prepare pass's; those of an order given by
    // the caller are taken from what its buffer holds now, and kept apart: calls with and
    // without an order may follow one another on one workspace
    if (p->order_dev && n_iter > 0) {
        const pct_status ls = launch_levels(a, s);
        if (ls != PCT_OK) return ls;
    }
    for (int32_t it = 0; it < n_iter; ++it) {
        const pct_status ls = A->val_dtype == PCT_F16 ? launch_strings<__half>(a, x_dev, Y, s)
                                                      : launch_strings<float>(a, x_dev, Y, s);
        if (ls != PCT_OK) return ls;
        if (y_in_lds(A->n_cols))
            hipLaunchKernelGGL((k_sap_average<false>), dim3(avg_blocks), dim3(256), 0, s, a, Y, w, p->n_strings, A->n_cols,
                               x_dev);
        else
            hipLaunchKernelGGL((k_sap_average<true>), dim3(avg_blocks), dim3(256), 0, s, a, Y, w, p->n_strings, A->n_cols,
                               x_dev);
        if (hipGetLastError() != hipSuccess) return PCT_EHIP;
    }
    return PCT_OK;
}

}  // extern "C"

// HIP kernels for gfx950 (MI355X): CSR products for one power, the p x SpMV
// baseline, the level-blocked kernels (one launch per diagonal, and three
// persistent dataflow forms: in ticket order, with skip-ahead parking, and
// with per-XCD queues), permutation, reset and a load-bandwidth probe.
//
// One launch per power, from the layout that suits the matrix: diagonal slices
// (dia_pass), few elements (few_sum), windowed rows (spmv_win_kernel), the sliced
// layout (run_sell) or CSR.  The level-blocked kernels use the last two.
// CSR rows go through one row routine.  For R < 4 right-hand sides
// (run_slices) the host cuts the rows into slices (consecutive rows whose
// products fit one LDS staging buffer, at most 256 rows; a longer row is a
// slice of its own) and a workgroup walks a range of slices:
//   1. it reads a slice's column indices and values with coalesced loads,
//      gathers the matching input entries and stores the products
//      a_e * x_{col(e), r} in LDS (one rounded multiply each);
//   2. each (row, right-hand side) pair is then summed by one thread,
//      sequentially in stored order starting from 0.0, with no fused
//      multiply-add.
// The loads of the next slice are issued before the current slice is summed
// (two LDS buffers), so one memory latency per slice is hidden behind the
// other's arithmetic.  For R >= 4 (run_rows) one thread per (row, right-hand
// side) sums its row directly, in the same order.  Either way the summation
// order is the plain CSR definition itself: results do not depend on
// slicing, chunking, schedule or right-hand-side count.  Values stored as
// float are promoted to double before the product; vectors and sums are
// double.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "mpk_internal.h"

namespace mpk {

// Dependency workspace of mpk_run_noalloc (done[] | tickets | err | fail),
// for callers that cannot allocate.  Every GPU holds its own copy until the
// process ends; host code uses the address from scratch_workspace, never
// this name.
static __device__ __align__(256) int32_t scratch[kScratchWords];

namespace {

constexpr int kBlock = 256;          // threads per workgroup (4 wavefronts of 64)
// Waves per SIMD the level-blocked kernels are built for: two 66 KB staging
// footprints fit a CU with 16 products per thread, four with 8.
constexpr int kTaskWaves = kTaskKP >= 16 ? 2 : 4;
constexpr int kWave = 64;
static_assert(kSliceRows == kBlock, "one thread per row of a slice");

__device__ __forceinline__ int ld_relaxed(const int32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A wait hit its limit: abandon the run and record the failure.
__device__ __forceinline__ void record_failure(const DevWorkspace &ws) {
    __hip_atomic_store(ws.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(ws.fail, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (ws.status) __hip_atomic_store(ws.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

struct PowerIO {
    const double *in;     // y_{k-1}
    const double *prev;   // y_{k-2} (recurrence; null at the very first power)
    double *out;          // y_k
    double alpha, beta, gamma;
    int recur;
    // weighted sums of the powers: weights of y_{k-2}, y_{k-1}, y_k and the
    // AccFlags of each sum (kernels with the sums only)
    double *acc_a, *acc_b;
    double wa2, wa1, wa0, wb2, wb1, wb0;
    int fa, fb;
};

// y = alpha*s + beta*y_{k-1} + gamma*y_{k-2} evaluated left to right, or s.
// A coefficient that is exactly zero omits its term (and its vector read):
// the Chebyshev recurrence has no beta term.
__device__ __forceinline__ double epilogue(const PowerIO &io, double s, size_t idx) {
    if (!io.recur) return s;
    double v = io.alpha * s;
    if (io.beta != 0.0) {
        const double b = io.beta * io.in[idx];
        v = v + b;
    }
    if (io.prev && io.gamma != 0.0) {
        const double g = io.gamma * io.prev[idx];
        v = v + g;
    }
    return v;
}

template <bool WT>
__device__ __forceinline__ void store_out(double *p, double v);

// One weighted sum at one element: the flush of this power (AccFlags f)
// adds w2*y_{k-2} (value y2), w1*y_{k-1} (the input row) and w0*y_k (v), as
// flagged and in that order, each product rounded and then added without
// contraction; the sum's first term starts it.
template <bool WT>
__device__ __forceinline__ void accumulate(double *acc, int f, double w2, double w1, double w0,
                                           double y2, const double *y1, double v, size_t idx) {
    if (!f) return;
    double r = 0.0;
    if (!(f & kAccZero)) {
        bool have = !(f & kAccStart);
        if (have) r = acc[idx];
        if (f & kAccT2) {
            const double t = w2 * y2;
            r = have ? r + t : t;
            have = true;
        }
        if (f & kAccT1) {
            const double t = w1 * *y1;
            r = have ? r + t : t;
            have = true;
        }
        if (f & kAccT0) {
            const double t = w0 * v;
            r = have ? r + t : t;
        }
    }
    store_out<WT>(acc + idx, r);
}

// Result of one (row, right-hand side): y_k from the row sum, stored, and
// the weighted sums updated.  The sums' loads and stores use the same
// element index as y_k, so each is touched by this thread only.
template <bool WT, bool ACC>
__device__ __forceinline__ void finish(const PowerIO &io, double s, size_t idx);

// Output store.  WT: an agent-scope atomic store, which writes through to
// memory (it must be coherent with agent-scope loads on every XCD), so a
// result is visible device-wide once the store has completed (vmcnt) and no
// L2 write-back is needed before publishing it; otherwise a plain store.
template <bool WT>
__device__ __forceinline__ void store_out(double *p, double v) {
    if (WT)
        __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
        *p = v;
}

template <bool WT, bool ACC>
__device__ __forceinline__ void finish(const PowerIO &io, double s, size_t idx) {
    if (!ACC) {
        store_out<WT>(io.out + idx, epilogue(io, s, idx));
        return;
    }
    // y_{k-2} is read once, for the recurrence and for the sums, and before
    // y_k is stored: in the two-vector ring both share this element
    const bool g = io.recur && io.prev && io.gamma != 0.0;
    const bool need2 = g || ((io.fa | io.fb) & kAccT2);
    const double y2 = need2 ? io.prev[idx] : 0.0;
    double v = s;
    if (io.recur) {
        v = io.alpha * s;
        if (io.beta != 0.0) {
            const double b = io.beta * io.in[idx];
            v = v + b;
        }
        if (g) {
            const double t = io.gamma * y2;
            v = v + t;
        }
    }
    store_out<WT>(io.out + idx, v);
    accumulate<WT>(io.acc_a, io.fa, io.wa2, io.wa1, io.wa0, y2, io.in + idx, v, idx);
    accumulate<WT>(io.acc_b, io.fb, io.wb2, io.wb1, io.wb0, y2, io.in + idx, v, idx);
}

// Loads of a slice with 1 <= nz nonzeros starting at nb, rows [rb, re):
// column and value of product q = tid + j*kBlock (nonzero q / R, right-hand
// side q % R) and the end of this thread's row.  Lanes past the end load a
// valid entry (clamped) whose product is never read, so all loads are
// unconditional.
template <typename V, int RC, int KP>
__device__ __forceinline__ void load_cols(const DevMatrix &m, int R, int32_t nb, int32_t nz,
                                          int32_t (&c)[KP]) {
    const int tid = threadIdx.x;
    const int last = nz - 1;
#pragma unroll
    for (int j = 0; j < KP; ++j) {
        const int q = tid + j * kBlock;
        c[j] = m.col[nb + min(RC ? q / RC : q / R, last)];
    }
}
template <typename V, int RC, int KP>
__device__ __forceinline__ void load_vals(const DevMatrix &m, int R, int32_t nb, int32_t nz,
                                          double (&a)[KP]) {
    const int tid = threadIdx.x;
    const V *val = static_cast<const V *>(m.val);
    const int last = nz - 1;
#pragma unroll
    for (int j = 0; j < KP; ++j) {
        const int q = tid + j * kBlock;
        a[j] = static_cast<double>(val[nb + min(RC ? q / RC : q / R, last)]);
    }
}
__device__ __forceinline__ int32_t load_row_end(const DevMatrix &m, int32_t nb, int32_t rb,
                                                int32_t re) {
    const int32_t i = rb + (int32_t)threadIdx.x + 1;
    return i <= re ? m.rowptr[i] : nb;
}

// Sum prod[e*R + rr] for e in [s0, s1) left to right from 0.0; the LDS
// reads are issued eight at a time ahead of the (ordered) additions.
__device__ __forceinline__ double ordered_sum(const double *prod, int R, int rr, int32_t s0,
                                              int32_t s1) {
    double s = 0.0;
    int32_t e = s0;
    for (; e + 8 <= s1; e += 8) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = prod[(e + u) * R + rr];
#pragma unroll
        for (int u = 0; u < 8; ++u) s = s + v[u];
    }
    for (; e < s1; ++e) s = s + prod[e * R + rr];
    return s;
}

// LDS of the row routine: two product buffers and two row-offset buffers.
template <int KP>
struct RowSmem {
    double prod[2][KP * kBlock];
    int32_t srp[2][kBlock + 1];
};

// One row longer than a slice buffer: summed buffer by buffer, one thread
// per right-hand side.  Starts and ends with a barrier.
template <typename V, int RC, int KP, bool WT, bool ACC>
__device__ void long_row(const DevMatrix &m, const PowerIO &io, int R, int32_t row, int32_t nb,
                         int32_t ne, RowSmem<KP> &sm) {
    const int tid = threadIdx.x;
    const int E = (KP * kBlock) / R;
    double s = 0.0;
    for (int32_t b = nb; b < ne; b += E) {
        const int32_t nz = min(E, ne - b);
        int32_t c[KP];
        double a[KP];
        load_cols<V, RC, KP>(m, R, b, nz, c);
        load_vals<V, RC, KP>(m, R, b, nz, a);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < KP; ++j) {
            const int q = tid + j * kBlock;
            const int rr = q - (RC ? q / RC : q / R) * R;
            sm.prod[0][q] = a[j] * io.in[(size_t)c[j] * R + rr];
        }
        __syncthreads();
        if (tid < R)
            for (int32_t e = 0; e < nz; ++e) s = s + sm.prod[0][e * R + tid];
    }
    if (tid < R) {
        const int32_t o = m.out_row ? m.out_row[row] : row;
        const size_t idx = (size_t)o * R + tid;
        finish<WT, ACC>(io, s, idx);
    }
    __syncthreads();
}

// Rows [r0, r1) of one power with one thread per (row, right-hand side): the
// thread sums its row in stored order from 0.0 (the same order as the
// slices), the R threads of a row share each column / value load and read
// the R entries of an input row together.  Used for R >= 4, where a row's
// R entries already fill a coalesced access; no LDS, no barrier.
template <typename V, int RC, bool WT, bool ACC>
__device__ void run_rows(const DevMatrix &m, const PowerIO &io, int R_rt, int32_t r0,
                         int32_t r1) {
    const int R = RC ? RC : R_rt;
    const int rows_per_step = kBlock / R;
    const int tid = threadIdx.x;
    const int rr = tid % R;
    const int li = tid / R;
    const V *val = static_cast<const V *>(m.val);
    if (li >= rows_per_step) return;  // idle lanes when R does not divide the block
    for (int32_t row = r0 + li; row < r1; row += rows_per_step) {
        const int32_t e0 = m.rowptr[row], e1 = m.rowptr[row + 1];
        double s = 0.0;
        // blocks of 8 nonzeros, the last one masked: all loads of a block are
        // issued before its products (lanes past the row end load its last
        // entry again and add nothing)
        for (int32_t e = e0; e < e1; e += 8) {
            int32_t c[8];
            double a[8], xv[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int32_t q = min(e + u, e1 - 1);
                c[u] = m.col[q];
                a[u] = static_cast<double>(val[q]);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) xv[u] = io.in[(size_t)c[u] * R + rr];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (e + u < e1) s = s + a[u] * xv[u];
        }
        const int32_t o = m.out_row ? m.out_row[row] : row;
        const size_t idx = (size_t)o * R + rr;
        finish<WT, ACC>(io, s, idx);
    }
}

// Rows [r0, r1) of one power in the sliced layout: one thread per (row,
// right-hand side) sums its row sequentially in stored order from 0.0, U
// slots at a time (the loads of a group are issued before its products; a
// slot past the row end reloads the row's last entry and adds nothing).  The
// 64 rows of a slice read each slot with one coalesced access, and the R
// threads of a row share it.  No LDS, no barrier: idle lanes (R not dividing
// the block) just skip.  U slots per group: fewer loads in flight per thread
// queue less in the memory system, more save round trips; the best width
// differs between the kernels (measured on 27-point rows and on 7-point rows
// with 8 right-hand sides; 6, 8 and 16 were slower everywhere):
// * the persistent level-blocked kernels, whose tasks wait on each other:
//   U = 4;
// * the one-launch-per-power baseline: U = 2 for one right-hand side (3.4%
//   faster than 4 on the 27-point stencil), U = 4 for more (2 and 3 were
//   13% and 6% slower with 8 right-hand sides).
template <int RC>
struct SellU {
    static constexpr int value = 4;
};
template <int RC>
struct SpmvSellU {
    static constexpr int value = RC == 1 ? 2 : 4;
};
constexpr int64_t kMallBytes = (int64_t)256 << 20;   // memory-side cache
constexpr int64_t kSpmvSellGrid = 4096;   // baseline workgroups per power (sliced layout)
// DEL: the columns come from the 16-bit offsets (col = row + offset, wrapped
// into [0, n)).  NT: the matrix is loaded non-temporally: by the one-launch-
// per-power baseline with one right-hand side, which reads each line once per
// launch (1.5% faster on the 27-point stencil; with 8 or 16 right-hand sides
// the rows of neighbouring waves share the lines, and the hint made it 5-28%
// slower), and by the level-blocked tasks of a segment's last power only
// (their reuse is the matrix kept in the caches between powers: the hint on
// every power made them 28% slower).
template <bool NT, typename T>
__device__ __forceinline__ T load_matrix(const T *p) {
    if constexpr (NT)
        return __builtin_nontemporal_load(p);
    else
        return *p;
}
template <typename V, int RC, bool WT, bool ACC, int U, bool DEL, bool NT>
__device__ __forceinline__ void run_sell_cols(const DevMatrix &m, const PowerIO &io, int R_rt,
                                              int32_t r0, int32_t r1) {
    const int R = RC ? RC : R_rt;
    const int rows_per_step = kBlock / R;
    const int tid = threadIdx.x;
    const int li = tid / R;
    const int rr = tid - li * R;
    if (li >= rows_per_step) return;
    const V *sval = static_cast<const V *>(m.sval);
    for (int32_t row = r0 + li; row < r1; row += rows_per_step) {
        const int32_t L = m.rlen[row];
        const int64_t base = m.soff[row / kSellRows] + row % kSellRows;
        double s = 0.0;
        for (int32_t j = 0; j < L; j += U) {
            int32_t c[U];
            double a[U], xv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t q = base + (int64_t)min(j + u, L - 1) * kSellRows;
                if constexpr (DEL) {  // row + offset, wrapped into [0, n)
                    int32_t cc = row + (int32_t)load_matrix<NT>(m.sdel + q);
                    cc += cc < 0 ? m.n : 0;
                    c[u] = cc >= m.n ? cc - m.n : cc;
                } else
                    c[u] = load_matrix<NT>(m.scol + q);
                a[u] = static_cast<double>(load_matrix<NT>(sval + q));
            }
#pragma unroll
            for (int u = 0; u < U; ++u) xv[u] = io.in[(size_t)c[u] * R + rr];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (j + u < L) s = s + a[u] * xv[u];
        }
        const int32_t o = m.out_row ? m.out_row[row] : row;
        finish<WT, ACC>(io, s, (size_t)o * R + rr);
    }
}
template <typename V, int RC, bool WT, bool ACC, int U, bool NT = false>
__device__ __forceinline__ void run_sell(const DevMatrix &m, const PowerIO &io, int R_rt,
                                         int32_t r0, int32_t r1) {
    if (m.sdel)  // uniform: the plan's layout
        run_sell_cols<V, RC, WT, ACC, U, true, NT>(m, io, R_rt, r0, r1);
    else
        run_sell_cols<V, RC, WT, ACC, U, false, NT>(m, io, R_rt, r0, r1);
}

// ------------------------------------------------------------------ diagonal slices

// Data written before the launch, read through the scalar cache where the
// address is the same for the whole wave.
template <typename T>
__device__ __forceinline__ T ld_const(const T *p) {
    return *(const __attribute__((address_space(4))) T *)(uintptr_t)p;
}

// Two consecutive doubles (8-byte aligned).
typedef double v2d __attribute__((ext_vector_type(2), aligned(8)));
typedef float v2f __attribute__((ext_vector_type(2), aligned(4)));
__device__ __forceinline__ void load_2(double (&v)[2], const double *p) {
    const v2d t = *reinterpret_cast<const v2d *>(p);
    v[0] = t.x;
    v[1] = t.y;
}
__device__ __forceinline__ void load_2(double (&v)[2], const float *p) {
    const v2f t = *reinterpret_cast<const v2f *>(p);
    v[0] = static_cast<double>(t.x);
    v[1] = static_cast<double>(t.y);
}
// NT: past the caches (a vector too large to be read from them again).
template <bool NT>
__device__ __forceinline__ void store_2(double *p, const double (&v)[2]) {
    typedef double v2n __attribute__((ext_vector_type(2)));
    if constexpr (NT) {
        typedef v2n v2u __attribute__((aligned(8)));
        __builtin_nontemporal_store(v2n{v[0], v[1]}, reinterpret_cast<v2u *>(p));
    } else
        *reinterpret_cast<v2d *>(p) = v2d{v[0], v[1]};
}

// accumulate and finish for two consecutive elements; y2: y_{k-2} there, where
// needs_prev says so (loaded ahead of the sum).
template <bool NT>
__device__ __forceinline__ void accumulate_2(double *acc, int f, double w2, double w1, double w0,
                                             const double (&y2)[2], const double (&y1)[2],
                                             const double (&v)[2], size_t idx) {
    if (!f) return;
    double r[2] = {0.0, 0.0};
    if (!(f & kAccZero)) {
        const bool start = f & kAccStart;
        if (!start) load_2(r, acc + idx);
        for (int i = 0; i < 2; ++i) {
            bool have = !start;
            if (f & kAccT2) {
                const double t = w2 * y2[i];
                r[i] = have ? r[i] + t : t;
                have = true;
            }
            if (f & kAccT1) {
                const double t = w1 * y1[i];
                r[i] = have ? r[i] + t : t;
                have = true;
            }
            if (f & kAccT0) {
                const double t = w0 * v[i];
                r[i] = have ? r[i] + t : t;
            }
        }
    }
    store_2<NT>(acc + idx, r);
}
template <bool ACC>
__device__ __forceinline__ bool needs_prev(const PowerIO &io) {
    return (io.recur && io.prev && io.gamma != 0.0) || (ACC && ((io.fa | io.fb) & kAccT2));
}
template <bool ACC, bool NT>
__device__ __forceinline__ void finish_2(const PowerIO &io, const double (&s)[2],
                                         const double (&y2)[2], size_t idx) {
    const bool b = io.recur && io.beta != 0.0;
    const bool g = io.recur && io.prev && io.gamma != 0.0;
    double y1[2] = {0.0, 0.0}, v[2];
    if (b || (ACC && ((io.fa | io.fb) & kAccT1))) load_2(y1, io.in + idx);
    for (int i = 0; i < 2; ++i) {
        v[i] = s[i];
        if (io.recur) {
            v[i] = io.alpha * s[i];
            if (b) {
                const double t = io.beta * y1[i];
                v[i] = v[i] + t;
            }
            if (g) {
                const double t = io.gamma * y2[i];
                v[i] = v[i] + t;
            }
        }
    }
    store_2<NT>(io.out + idx, v);
    if constexpr (ACC) {
        accumulate_2<NT>(io.acc_a, io.fa, io.wa2, io.wa1, io.wa0, y2, y1, v, idx);
        accumulate_2<NT>(io.acc_b, io.fb, io.wb2, io.wb1, io.wb0, y2, y1, v, idx);
    }
}

// How the lanes of a wave share a slice.  The kDiaRows * R elements of a
// vector's slice are consecutive; a pass takes 128 of them and a lane two
// neighbours (one 16-byte load per diagonal: the vector cache moves 64
// bytes a clock that way and 32 with 8-byte loads): two rows (kOneRhs), two
// right-hand sides of a row (kEven) or either (kOdd).  (Two passes at once per
// wave, to share the records, took 102 registers instead of 48 and was 5%
// slower on 27-point 64^3 with 16 right-hand sides.)
enum DiaMode { kOneRhs, kEven, kOdd };
struct DiaLane {
    int32_t row[2];   // of the slice
    int32_t sub0;     // first row of the pass (uniform)
    uint32_t at;      // byte offset of the first element in a vector
    bool live[2];     // the rows exist (slices with kDiaEdge)
};
// Rows sub0 .. sub0 + 63 of a mask (uniform).
__device__ __forceinline__ uint64_t mask_from(uint64_t lo, uint64_t hi, int32_t sub0) {
    if (sub0 >= 64) return hi >> (sub0 - 64);
    return sub0 ? lo >> sub0 | hi << (64 - sub0) : lo;
}

// The first U diagonals of group g, added to the lane's two sums.  All loads
// go out before the products; a row without a diagonal keeps its sum.
// vals: the group's first block of per-row values.  WHOLE: every row of the
// pass has every diagonal.  EDGE: every load address is a row's own or one of
// its columns; else any row plus any of the slice's offsets is inside the
// vector.  NT: the values are loaded past the caches.
template <typename V, int U, int MODE, int KIND, bool WHOLE, bool EDGE, bool NT>
__device__ __forceinline__ void dia_group(const DevMatrix &m, const double *in, int32_t g,
                                          const V *vals, const DiaLane &l, int32_t rbytes,
                                          double (&s)[2]) {
    typedef int v16i __attribute__((ext_vector_type(16), aligned(64)));
    typedef uint64_t v8u __attribute__((ext_vector_type(8), aligned(64)));
    const v16i h = ld_const(reinterpret_cast<const v16i *>(m.dgroup + g));
    v8u mk = {};
    if constexpr (MODE == kOneRhs)
        mk = ld_const(reinterpret_cast<const v8u *>(m.dgroup + g) + 1);
    else if constexpr (!WHOLE)
        mk = ld_const(reinterpret_cast<const v8u *>(m.dmask + g));
    double a[U][2], x[U][2];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint64_t ub = (uint64_t)(uint32_t)h[8 + 2 * u] | (uint64_t)(uint32_t)h[9 + 2 * u] << 32;
        a[u][0] = a[u][1] = __longlong_as_double((long long)ub);
        if (KIND == kDiaPerRow || (KIND == kDiaMixed && (h[5] >> u & 1))) {   // uniform
            if constexpr (MODE == kOneRhs) {
                typedef V v2v __attribute__((ext_vector_type(2)));   // aligned to both
                const v2v t = load_matrix<NT>(
                    reinterpret_cast<const v2v *>(vals + (uint32_t)l.row[0]));
                a[u][0] = static_cast<double>(t.x);
                a[u][1] = static_cast<double>(t.y);
            } else {
                a[u][0] = a[u][1] = static_cast<double>(load_matrix<NT>(vals + (uint32_t)l.row[0]));
                if (MODE == kOdd)
                    a[u][1] = static_cast<double>(load_matrix<NT>(vals + (uint32_t)l.row[1]));
            }
            vals += kDiaRows;
        }
    }
    const char *p = reinterpret_cast<const char *>(in);
    if constexpr (!EDGE) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            load_2(x[u], reinterpret_cast<const double *>(
                             p + (uint32_t)(l.at + (uint32_t)(h[u] * rbytes))));
        if (WHOLE || h[6] == 0) {   // uniform
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int i = 0; i < 2; ++i) s[i] = s[i] + a[u][i] * x[u][i];
            return;
        }
    }
    bool bit[U][2];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if constexpr (MODE == kOneRhs) {
            bit[u][0] = __builtin_amdgcn_inverse_ballot_w64(mk[u]);
            bit[u][1] = __builtin_amdgcn_inverse_ballot_w64(mk[4 + u]);
        } else {
            const uint64_t w = mask_from(mk[u], mk[4 + u], l.sub0);
            bit[u][0] = w >> (l.row[0] - l.sub0) & 1;
            bit[u][1] = MODE == kEven ? bit[u][0] : w >> (l.row[1] - l.sub0) & 1;
        }
        if constexpr (EDGE) {
            const uint32_t d = (uint32_t)(h[u] * rbytes);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                bit[u][i] = bit[u][i] && l.live[i];
                const uint32_t q = (l.live[i] ? l.at + 8u * i : 0u) + (bit[u][i] ? d : 0u);
                x[u][i] = *reinterpret_cast<const double *>(p + q);
            }
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const double t = s[i] + a[u][i] * x[u][i];
            s[i] = bit[u][i] ? t : s[i];
        }
}
// All `count` diagonals from group g on.
template <typename V, int MODE, int KIND, bool WHOLE, bool EDGE, bool NT>
__device__ __forceinline__ void dia_sum(const DevMatrix &m, const double *in, int32_t g,
                                        int32_t count, const V *vals, const DiaLane &l,
                                        int32_t rbytes, double (&s)[2]) {
    for (; count >= 4; count -= 4, ++g) {
        dia_group<V, 4, MODE, KIND, WHOLE, EDGE, NT>(m, in, g, vals, l, rbytes, s);
        if (KIND == kDiaPerRow) vals += 4 * kDiaRows;
        if (KIND == kDiaMixed)
            vals += (size_t)__popc((unsigned)ld_const(&m.dgroup[g].vary)) * kDiaRows;
    }
    switch (count) {   // uniform
    case 3: dia_group<V, 3, MODE, KIND, WHOLE, EDGE, NT>(m, in, g, vals, l, rbytes, s); break;
    case 2: dia_group<V, 2, MODE, KIND, WHOLE, EDGE, NT>(m, in, g, vals, l, rbytes, s); break;
    case 1: dia_group<V, 1, MODE, KIND, WHOLE, EDGE, NT>(m, in, g, vals, l, rbytes, s); break;
    }
}
template <typename V, int MODE, int KIND, bool NT>
__device__ __forceinline__ void dia_sum(const DevMatrix &m, const double *in, int32_t g,
                                        int32_t count, const V *vals, const DiaLane &l,
                                        int32_t rbytes, bool whole, double (&s)[2]) {
    if (MODE != kOneRhs && whole)   // uniform
        dia_sum<V, MODE, KIND, true, false, NT>(m, in, g, count, vals, l, rbytes, s);
    else
        dia_sum<V, MODE, KIND, false, false, NT>(m, in, g, count, vals, l, rbytes, s);
}

// The lane's place in pass q of slice s (both uniform; ds: the slice's record).
// inv = ceil(2^16 / R): f / R = f * inv >> 16 for f < 128 * 16.  Returns whether
// every row of the pass has every diagonal.
typedef int v8i __attribute__((ext_vector_type(8), aligned(16)));
template <int MODE>
__device__ __forceinline__ bool dia_place(const v8i &ds, int32_t R, int32_t inv, int32_t s,
                                          int32_t q, DiaLane &l, size_t &idx) {
    const int lane = (int)(threadIdx.x & (kWave - 1));
    const int32_t f0 = q * 128, f = f0 + 2 * lane;   // elements of the slice
    idx = (size_t)s * kDiaRows * R + f;
    l.at = (uint32_t)idx * (uint32_t)sizeof(double);
    bool whole = false;
    if constexpr (MODE == kOneRhs) {
        l.row[0] = f;
        l.row[1] = f + 1;
        l.sub0 = 0;
    } else {
        l.row[0] = f * inv >> 16;
        l.row[1] = MODE == kEven ? l.row[0] : (f + 1) * inv >> 16;
        l.sub0 = f0 * inv >> 16;
        const int32_t k = ((f0 + 127) * inv >> 16) + 1 - l.sub0;   // 8 .. 64 rows
        const uint64_t sub = ~0ull >> (64 - k);
        const uint64_t lo = (uint64_t)(uint32_t)ds[4] | (uint64_t)(uint32_t)ds[5] << 32;
        const uint64_t hi = (uint64_t)(uint32_t)ds[6] | (uint64_t)(uint32_t)ds[7] << 32;
        whole = (mask_from(lo, hi, l.sub0) & sub) == sub;
    }
    return whole;
}
// Whether every row of the slice exists and reads inside the vector wherever
// its diagonals point.
__device__ __forceinline__ bool dia_inner(const v8i &ds) { return ds[1] >= 0 && ds[3] < kDiaEdge; }

// The lane's two row sums in an inner slice.  STREAM: the per-row values of all
// but `keep` of every 16 slices are loaded past the caches.
template <typename V, int MODE, bool STREAM>
__device__ __forceinline__ void inner_sums(const DevMatrix &m, const double *in, int32_t R,
                                           const v8i &ds, int32_t s, const DiaLane &l, bool whole,
                                           int32_t keep, double (&sum)[2]) {
    const int32_t rbytes = R * (int32_t)sizeof(double);
    const V *vals = static_cast<const V *>(m.dvals) + (size_t)ds[2] * kDiaRows;
    if (ds[3] == kDiaShared)
        dia_sum<V, MODE, kDiaShared, false>(m, in, ds[0], ds[1], vals, l, rbytes, whole, sum);
    else if (ds[3] != kDiaPerRow)
        dia_sum<V, MODE, kDiaMixed, false>(m, in, ds[0], ds[1], vals, l, rbytes, whole, sum);
    else if (STREAM && (s & 15) >= keep)
        dia_sum<V, MODE, kDiaPerRow, true>(m, in, ds[0], ds[1], vals, l, rbytes, whole, sum);
    else
        dia_sum<V, MODE, kDiaPerRow, false>(m, in, ds[0], ds[1], vals, l, rbytes, whole, sum);
}
// The same from the sliced layout's rows.  Two right-hand sides of a row share its
// slots: a wave that read them once for each held up matrices with many such
// slices (16 entries a row, nearly every other 256 rows irregular, 250 k rows, us
// per power with 2 and 4 right-hand sides, before and now: 25 and 16; 30 and 19).  Two
// rows go one after the other: both at once do not fit 64 registers.
template <typename V, int MODE>
__device__ __forceinline__ void row_sums(const DevMatrix &m, const double *in, int32_t R,
                                         int32_t s, const DiaLane &l, double (&sum)[2]) {
    constexpr int N = MODE == kEven ? 2 : 1;   // elements of a row
    const V *sval = static_cast<const V *>(m.sval);
#pragma unroll
    for (int i = 0; i < 2; i += N) {
        if (!l.live[i]) continue;
        const int32_t row = s * kDiaRows + l.row[i], pr = m.drow ? m.drow[row] : row;
        const int32_t rr = (int32_t)(l.at / 8u + i - (uint32_t)row * (uint32_t)R);
        const int32_t L = m.rlen[pr];
        const int64_t b = m.soff[pr / kSellRows] + pr % kSellRows;
        double t[N] = {};
        for (int32_t j = 0; j < L; j += 4) {
            double a[4], x[4][N];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t c = b + (int64_t)min(j + u, L - 1) * kSellRows;
                a[u] = static_cast<double>(sval[c]);
                const double *at = in + (size_t)m.scol[c] * R + rr;
                if constexpr (N == 2) load_2(x[u], at);
                else x[u][0] = *at;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int k = 0; k < N; ++k)
                    if (j + u < L) t[k] = t[k] + a[u] * x[u][k];
        }
#pragma unroll
        for (int k = 0; k < N; ++k) sum[i + k] = t[k];
    }
}
// The same in any slice but an inner one; sets l.live.
template <typename V, int MODE>
__device__ __forceinline__ void outer_sums(const DevMatrix &m, const double *in, int32_t R,
                                           const v8i &ds, int32_t s, DiaLane &l,
                                           double (&sum)[2]) {
#pragma unroll
    for (int i = 0; i < 2; ++i) l.live[i] = s * kDiaRows + l.row[i] < m.n;
    if (ds[1] >= 0) {
        const V *vals = static_cast<const V *>(m.dvals) + (size_t)ds[2] * kDiaRows;
        dia_sum<V, MODE, kDiaMixed, false, true, false>(m, in, ds[0], ds[1], vals, l,
                                                        R * (int32_t)sizeof(double), sum);
    } else {
        row_sums<V, MODE>(m, in, R, s, l, sum);
    }
}

// Pass q of slice s by one wave.  STREAM: the power's data is larger than the
// memory-side cache: results are stored past it too.
template <typename V, int MODE, bool ACC, bool STREAM>
__device__ __forceinline__ void dia_pass(const DevMatrix &m, const PowerIO &io, int32_t R,
                                         int32_t inv, int32_t s, int32_t q, int32_t keep) {
    const v8i ds = ld_const(reinterpret_cast<const v8i *>(m.dsl + s));
    DiaLane l;
    size_t idx;
    const bool whole = dia_place<MODE>(ds, R, inv, s, q, l, idx);
    double sum[2] = {0.0, 0.0};
    if (__builtin_expect(dia_inner(ds), 1)) {
        double y2[2] = {0.0, 0.0};
        if (needs_prev<ACC>(io)) load_2(y2, io.prev + idx);
        inner_sums<V, MODE, STREAM>(m, io.in, R, ds, s, l, whole, keep, sum);
        finish_2<ACC, STREAM>(io, sum, y2, idx);
        return;
    }
    outer_sums<V, MODE>(m, io.in, R, ds, s, l, sum);
#pragma unroll
    for (int i = 0; i < 2; ++i)
        if (l.live[i]) finish<false, ACC>(io, sum[i], idx + i);
}

// Products staged per thread and buffer: the slice path for R < 4 (R = 0 is
// the generic instantiation, which takes either path at run time).
template <int RC, int KP>
struct Staging {
    static constexpr int value = (RC >= 4) ? 1 : KP;
};

// Slices [s0, s1) of one power.  Called by all threads of the workgroup;
// all control flow depends on uniform values only.  Ends with a barrier, so
// the caller may reuse the LDS right away.  Slices holding one row longer
// than a buffer are computed in a second pass.
template <typename V, int RC, int KP, bool WT, bool ACC>
__device__ void run_slices(const DevMatrix &m, const PowerIO &io, int R_rt, DevSlices sl,
                           int32_t s0, int32_t s1, RowSmem<KP> &sm) {
    const int R = RC ? RC : R_rt;
    if (R >= 4) {
        run_rows<V, RC, WT, ACC>(m, io, R, sl.srow[s0], sl.srow[s1]);
        __syncthreads();
        return;
    }
    const int E = (KP * kBlock) / R;  // nonzeros per slice buffer
    const int tid = threadIdx.x;
    int32_t c[KP];    // columns of the slice being processed (then of the next)
    double a[KP];     // its values
    int32_t rp = 0;   // its row end for this thread
    bool have = false;  // c / a / rp hold the loads of slice s
    int buf = 0;
    for (int32_t s = s0; s < s1; ++s) {
        const int32_t rb = sl.srow[s], re = sl.srow[s + 1];
        const int32_t nb = sl.snz[s], ne = sl.snz[s + 1];
        const int32_t nz = ne - nb;
        if (nz > E) {  // a single long row: done after this loop
            have = false;
            continue;
        }
        if (!have && nz > 0) {
            load_cols<V, RC, KP>(m, R, nb, nz, c);
            load_vals<V, RC, KP>(m, R, nb, nz, a);
            rp = load_row_end(m, nb, rb, re);
        }
        double xv[KP];
        if (nz > 0) {
#pragma unroll
            for (int j = 0; j < KP; ++j) {
                const int q = tid + j * kBlock;
                const int rr = q - (RC ? q / RC : q / R) * R;
                xv[j] = io.in[(size_t)c[j] * R + rr];
            }
        }
        const int32_t myrp = nz > 0 ? rp : nb;
        // issue the next slice's loads before this slice's products are formed
        double a2[KP];
        have = false;
        if (s + 1 < s1) {
            const int32_t rb2 = sl.srow[s + 1], re2 = sl.srow[s + 2];
            const int32_t nb2 = sl.snz[s + 1], nz2 = sl.snz[s + 2] - nb2;
            if (nz2 > 0 && nz2 <= E) {
                load_cols<V, RC, KP>(m, R, nb2, nz2, c);
                load_vals<V, RC, KP>(m, R, nb2, nz2, a2);
                rp = load_row_end(m, nb2, rb2, re2);
                have = true;
            }
        }
        double *prod = sm.prod[buf];
        int32_t *srp = sm.srp[buf];
        if (nz > 0) {
#pragma unroll
            for (int j = 0; j < KP; ++j) prod[tid + j * kBlock] = a[j] * xv[j];
        }
        if (have) {
#pragma unroll
            for (int j = 0; j < KP; ++j) a[j] = a2[j];
        }
        srp[tid + 1] = myrp - nb;
        if (tid == 0) srp[0] = 0;
        __syncthreads();
        const int32_t cnt = re - rb;
        const int npairs = cnt * R;
        for (int q = tid; q < npairs; q += kBlock) {
            const int li = RC ? q / RC : q / R;
            const int rr = q - li * R;
            const int32_t row = rb + li;
            const double sum = ordered_sum(prod, R, rr, srp[li], srp[li + 1]);
            const int32_t o = m.out_row ? m.out_row[row] : row;
            const size_t idx = (size_t)o * R + rr;
            finish<WT, ACC>(io, sum, idx);
        }
        buf ^= 1;
    }
    __syncthreads();
    // rows longer than a buffer, kept out of the pipelined loop (registers)
    for (int32_t s = s0; s < s1; ++s) {
        const int32_t nb = sl.snz[s], ne = sl.snz[s + 1];
        if (ne - nb > E) long_row<V, RC, KP, WT, ACC>(m, io, R, sl.srow[s], nb, ne, sm);
    }
}

// Inputs and outputs of the segment's power k.  ACC: the sequence is kept in
// a ring of two vectors (power g = k0 + k in slot (g-1) mod 2) and the
// weighted sums are updated.
template <bool ACC>
__device__ __forceinline__ PowerIO power_io(const SegArgs &a, const Coefs &cf,
                                            const AccCoefs *ac, int32_t k, int32_t n) {
    const size_t stride = (size_t)n * a.R;
    PowerIO io;
    if (ACC) {
        const int32_t g = a.k0 + k;
        io.in = (k == 1) ? a.in0 : a.Y + (size_t)((g - 2) & 1) * stride;
        io.prev = (k == 1) ? a.inm1 : (k == 2 ? a.in0 : a.Y + (size_t)((g - 3) & 1) * stride);
        io.out = a.Y + (size_t)((g - 1) & 1) * stride;
        io.acc_a = a.acc_a;
        io.acc_b = a.acc_b;
        io.wa2 = ac->wa[k - 1];  // weights of the sequence's powers g-2, g-1, g
        io.wa1 = ac->wa[k];
        io.wa0 = ac->wa[k + 1];
        io.wb2 = ac->wb[k - 1];
        io.wb1 = ac->wb[k];
        io.wb0 = ac->wb[k + 1];
        io.fa = ac->fa[k - 1];
        io.fb = ac->fb[k - 1];
    } else {
        io.in = (k == 1) ? a.in0 : a.Y + (size_t)(k - 2) * stride;
        io.prev = (k == 1) ? a.inm1 : (k == 2 ? a.in0 : a.Y + (size_t)(k - 3) * stride);
        io.out = a.Y + (size_t)(k - 1) * stride;
    }
    io.recur = a.recur;
    io.alpha = cf.alpha[k - 1];
    io.beta = cf.beta[k - 1];
    io.gamma = cf.gamma[k - 1];
    return io;
}

// ------------------------------------------------------------------ baseline

// One power of R >= 4 right-hand sides from CSR rows: workgroup b takes row
// blocks b, b + grid, ... of 256/R rows each.  A row is one thread's chain of
// loads for each right-hand side, so the chains of a power have to run side by
// side: a workgroup per block.  Random bands of 16 entries a row, us per power of
// 16 right-hand sides at 8192 and 200 k rows with 1, 4 and 16 blocks per
// workgroup: 5.9, 12, 39 and 79, 82, 99 (two slices of 4096 entries each, as
// fewer right-hand sides take them: 75 and 116).
template <typename V, int RC, bool ACC>
__device__ __forceinline__ void rows_power(const DevMatrix &m, const PowerIO &io, int32_t R) {
    const int32_t step = kBlock / (RC ? RC : R);
    for (int64_t r0 = (int64_t)blockIdx.x * step; r0 < m.n; r0 += (int64_t)gridDim.x * step)
        run_rows<V, RC, false, ACC>(m, io, R, (int32_t)r0, (int32_t)min((int64_t)m.n, r0 + step));
}
// Any count without an instantiation of its own (no LDS, which that of
// spmv_power_kernel holds for three).
template <typename V, bool ACC>
__global__ __launch_bounds__(kBlock) void spmv_rows_kernel(DevMatrix m, PowerIO io, int32_t R) {
    rows_power<V, 0, ACC>(m, io, R);
}

// One power from CSR rows: R < 4, workgroup b walks slices [b*per, min((b+1)*per,
// n_slices)); else row blocks.
template <typename V, int RC, bool ACC>
__global__ __launch_bounds__(kBlock, 2) void spmv_power_kernel(DevMatrix m, PowerIO io, int32_t R,
                                                           DevSlices sl, int32_t n_slices,
                                                           int32_t per) {
    if constexpr (RC >= 4) {
        rows_power<V, RC, ACC>(m, io, R);
    } else {
        __shared__ RowSmem<Staging<RC, kSpmvKP>::value> sm;
        const int32_t s0 = blockIdx.x * per;
        const int32_t s1 = min(n_slices, s0 + per);
        run_slices<V, RC, Staging<RC, kSpmvKP>::value, false, ACC>(m, io, R, sl, s0, s1, sm);
    }
}

// One power in the sliced layout: workgroup b walks row blocks b, b + grid,
// ... of 256/R rows each.
template <typename V, int RC, bool ACC>
__global__ __launch_bounds__(kBlock) void spmv_sell_kernel(DevMatrix m, PowerIO io, int32_t R) {
    const int32_t step = kBlock / (RC ? RC : R);
    for (int32_t r0 = blockIdx.x * step; r0 < m.n; r0 += gridDim.x * step)
        run_sell<V, RC, false, ACC, SpmvSellU<RC>::value, RC == 1>(m, io, R, r0,
                                                                   min(m.n, r0 + step));
}

// Few elements (few_elements): a wave per workgroup, a thread per (row,
// right-hand side).  A power then takes as long as one thread's chain of loads,
// so a batch holds a whole row of up to 8 slots, half a 27-point row otherwise,
// and the waves spread over the compute units.
template <typename V, int U>
__device__ __forceinline__ double few_sum(const DevMatrix &m, const double *in, int32_t row,
                                          int32_t L, uint32_t R, uint32_t rr) {
    const int64_t base = m.soff[row / kSellRows] + row % kSellRows;
    const V *sval = static_cast<const V *>(m.sval);
    double s = 0.0;
    for (int32_t j = 0; j < L; j += U) {
        int32_t c[U];
        double a[U], xv[U];
        if (m.sdel) {  // row + offset, wrapped into [0, n)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t q = base + (int64_t)min(j + u, L - 1) * kSellRows;
                int32_t cc = row + (int32_t)m.sdel[q];
                cc += cc < 0 ? m.n : 0;
                c[u] = cc >= m.n ? cc - m.n : cc;
                a[u] = static_cast<double>(sval[q]);
            }
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t q = base + (int64_t)min(j + u, L - 1) * kSellRows;
                c[u] = m.scol[q];
                a[u] = static_cast<double>(sval[q]);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) xv[u] = in[(size_t)c[u] * R + rr];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (j + u < L) s = s + a[u] * xv[u];
    }
    return s;
}
template <typename V, bool ACC>
__global__ __launch_bounds__(kWave) void spmv_few_kernel(DevMatrix m, PowerIO io, int32_t R) {
    const uint32_t e = blockIdx.x * kWave + threadIdx.x;
    const int32_t row = (int32_t)(e / (uint32_t)R);
    if (row >= m.n) return;
    const uint32_t rr = e - (uint32_t)row * (uint32_t)R;
    const int32_t L = m.rlen[row];
    const int32_t o = m.out_row ? m.out_row[row] : row;
    const double s = __any(L > 8) ? few_sum<V, 16>(m, io.in, row, L, R, rr)
                                  : few_sum<V, 8>(m, io.in, row, L, R, rr);
    finish<false, ACC>(io, s, (size_t)o * R + rr);
}

// One power from the windowed rows, one right-hand side: workgroup b takes the
// chunks [part[b], part[b + 1]), its ring of input rows moving on with them.  Each
// input row is gathered from memory about twice a power (a ring's first fill
// included) instead of once per entry, and the entries gather from LDS.  Random
// band, 2^22 rows, 67 M entries: 274 us per power against 400 from CSR rows
// staged in LDS, whose gathers take a cache line each.  670 MB of entries, but 1.68
// GB leave the L2, 6.1 TB/s: in the caller's numbering a ring's rows lie apart, and
// each of the two loads of a row takes a 128-byte line (in plan order 1.3 M rows
// take 49 us per power, here 98).
template <typename V, bool ACC>
__global__ __launch_bounds__(kWinRows) void spmv_win_kernel(DevMatrix m, PowerIO io, WinMatrix w,
                                                            int32_t keep) {
    constexpr int U = kWinPad;
    __shared__ double ring[kWinRing];
    const int t = (int)threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(t / kWave), lane = t & (kWave - 1);
    const int32_t c0 = ld_const(w.part + blockIdx.x), c1 = ld_const(w.part + blockIdx.x + 1);
    if (c0 >= c1) return;   // uniform
    const int32_t *map = m.out_row;
    // vector row of plan row r, -1 from `to` on
    auto place_of = [&](int32_t r, int32_t to) { return r < to ? (map ? map[r] : r) : -1; };
    // ring rows [from, to), eight loads of a thread in flight
    auto fill = [&](int32_t from, int32_t to) {
        for (int32_t r = from + t; r < to; r += 8 * kWinRows) {
            int32_t g[8];
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) g[u] = place_of(r + u * kWinRows, to);
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = g[u] >= 0 ? io.in[g[u]] : 0.0;
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (g[u] >= 0) ring[(r + u * kWinRows) % kWinRing] = v[u];
        }
    };
    int32_t h0 = ld_const(w.end + c0), h1 = c0 + 1 < c1 ? ld_const(w.end + c0 + 1) : h0;
    fill(max(0, h0 - kWinRing), h0);
    int32_t next_at = place_of(h0 + t, h1);
    uint32_t info = w.row[(size_t)c0 * kWinRows + t];
    __syncthreads();
    for (int32_t c = c0; c < c1; ++c) {
        // The first rows that the next window adds, whose places were loaded a
        // chunk ago, and the same a chunk on.
        const double next = next_at >= 0 ? io.in[next_at] : 0.0;
        const int32_t h2 = c + 2 < c1 ? ld_const(w.end + c + 2) : h1;
        next_at = place_of(h1 + t, h2);
        const int32_t L = (int32_t)(info >> 10);
        const int32_t prow = ld_const(w.start + c) + (int32_t)(info & 1023);
        const bool there = prow < ld_const(w.start + c + 1);
        const int32_t o = there ? (map ? map[prow] : prow) : 0;
        const int32_t off = ld_const(w.off + c * (kWinRows / kWave) + wave);
        const int32_t width = ld_const(w.off + c * (kWinRows / kWave) + wave + 1) - off;
        if (c + 1 < c1) info = w.row[(size_t)(c + 1) * kWinRows + t];
        const uint16_t *place = w.place + (size_t)off * kWave + lane;
        const V *val = static_cast<const V *>(w.val) + (size_t)off * kWave + lane;
        double s = 0.0;
        auto sum = [&](auto nt) {
            constexpr bool NT = decltype(nt)::value;
            for (int32_t j = 0; j < width; j += U) {   // uniform
                uint32_t q[U];
                double a[U], x[U];
                bool far = false;
#pragma unroll
                for (int u = 0; u < U; ++u) {   // padded: places 0 past a row's end
                    q[u] = load_matrix<NT>(place + (size_t)(j + u) * kWave);
                    a[u] = static_cast<double>(load_matrix<NT>(val + (size_t)(j + u) * kWave));
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (j + u >= L) q[u] = 0;   // the next slice's
                    far |= q[u] == kWinFar;
                    x[u] = ring[q[u] == kWinFar ? 0 : q[u]];
                }
                if (__any(far)) {   // the columns, then the inputs, all at once
                    const int32_t *col = m.col + m.rowptr[there ? prow : 0];
                    int32_t g[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) g[u] = q[u] == kWinFar ? col[j + u] : 0;
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const double y = io.in[g[u]];
                        x[u] = q[u] == kWinFar ? y : x[u];
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (j + u < L) s = s + a[u] * x[u];
            }
        };
        if ((c & 15) >= keep) sum(std::true_type());   // uniform
        else sum(std::false_type());
        if (there) finish<false, ACC>(io, s, (size_t)o);
        if (c + 1 == c1) break;   // uniform
        __syncthreads();          // the window's oldest rows are no longer read
        if (h0 + t < h1 && h0 + t >= h1 - kWinRing) ring[(h0 + t) % kWinRing] = next;
        fill(max(h0 + kWinRows, h1 - kWinRing), h1);
        __syncthreads();
        h0 = h1;
        h1 = h2;
    }
}

// u / d = u * inv >> 32 with inv = ceil(2^32 / d), exact while u * d < 2^32.
struct FastDiv {
    int32_t d;
    uint32_t inv;   // (d = 1: not used; 0: every quotient is 0)
    __device__ __forceinline__ int32_t operator()(int32_t u) const {
        return d == 1 ? u : (int32_t)__umulhi((uint32_t)u, inv);
    }
};
FastDiv fast_div(int32_t d) {
    return FastDiv{d, d == 1 ? 0u : (uint32_t)((((uint64_t)1 << 32) + d - 1) / d)};
}

// One power from the diagonal slices.  A wave takes one pass of one slice (per:
// passes per slice); workgroup b runs on XCD b mod 8, and the blocks are dealt
// in runs: XCD x takes run x, then run x + 8, ...
//
// Bound by: 27-point 128^3, one right-hand side: 18.5 us per power against
// 125 from the sliced layout; the vector caches (27 loads of 1 KB per 128 rows are
// 453 MB, and 615 MB of 64-byte accesses as they lie: 33 TB/s) and launches are
// the time, 37 MB leave the L2.  With general coefficients 71 against 125 us: 486
// MB leave it, 446 of them values, 6.8 TB/s.  Anderson 160^3 with 8 right-hand
// sides, recurrence: 189 against 364 us, 818 MB, 4.3 TB/s (a 4 GB copy: 4.8 TB/s).
template <typename V, int MODE, bool ACC, bool STREAM>
__global__ __launch_bounds__(kBlock, MODE == kOneRhs ? 8 : 1) void spmv_dia_kernel(
        DevMatrix m, PowerIO io, int32_t R, int32_t inv, int32_t units, FastDiv per, FastDiv run,
        int32_t keep) {
    const int32_t j = (int32_t)(blockIdx.x >> 3), c = run(j);
    const int32_t b = (c * 8 + (int32_t)(blockIdx.x & 7)) * run.d + (j - c * run.d);
    const int32_t u = b * (kBlock / kWave) +
                      __builtin_amdgcn_readfirstlane((int32_t)(threadIdx.x / kWave));
    if (u >= units) return;
    const int32_t s = MODE == kOneRhs ? u : per(u);
    dia_pass<V, MODE, ACC, STREAM>(m, io, MODE == kOneRhs ? 1 : R, inv, s,
                                   MODE == kOneRhs ? 0 : u - s * per.d, keep);
}

// All powers of a segment in one launch: right-hand sides do not depend on each
// other, so workgroup r computes column r alone, with the last two vectors in
// LDS and a barrier between the powers.  A launch per power takes 3.7 us
// however little it does; here a power of 5-point 32^2 takes 0.9 us and one of
// 64^2 2.5, by then the compute unit's instruction issue (some 250
// instructions per 128 rows; with the vectors in memory 3.1 us, by latency).
constexpr int kSmallBlock = 1024;
// Barrier of the workgroup that orders LDS only: stores to memory, which no
// other thread reads in this launch, stay in flight.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
template <typename V, bool ACC>
__device__ __forceinline__ void small_body(const DevMatrix &m, const SegArgs &a, const Coefs &cf,
                                           const AccCoefs *ac) {
    // y_{k-1} and y_{k-2}, whose place y_k takes (each element by its own lane)
    __shared__ double buf[2][kSmallRows];
    const int32_t R = a.R, r = (int32_t)blockIdx.x;
    for (int32_t i = threadIdx.x; i < m.n; i += kSmallBlock) {
        buf[0][i] = a.in0[(size_t)i * R + r];
        if (a.inm1) buf[1][i] = a.inm1[(size_t)i * R + r];
    }
    __syncthreads();
    const int32_t n_sl = (m.n + kDiaRows - 1) / kDiaRows;
    for (int32_t k = 1; k <= a.p; ++k) {
        PowerIO io = power_io<ACC>(a, cf, ac, k, m.n);
        const double *in = buf[(k - 1) & 1];
        double *out = buf[k & 1];
        const bool prev = io.prev != nullptr;
        for (int32_t s = __builtin_amdgcn_readfirstlane((int32_t)(threadIdx.x / kWave)); s < n_sl;
             s += kSmallBlock / kWave) {
            const v8i ds = ld_const(reinterpret_cast<const v8i *>(m.dsl + s));
            DiaLane l;
            size_t idx;
            dia_place<kOneRhs>(ds, 1, 0, s, 0, l, idx);
            double sum[2] = {0.0, 0.0};
            l.live[0] = l.live[1] = true;
            if (dia_inner(ds)) inner_sums<V, kOneRhs, false>(m, in, 1, ds, s, l, false, 0, sum);
            else outer_sums<V, kOneRhs>(m, in, 1, ds, s, l, sum);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                if (!l.live[i]) continue;
                const int32_t row = s * kDiaRows + l.row[i];
                const size_t e = (size_t)row * R + r;
                // as finish(), with the last two vectors from LDS
                const double y2 = prev ? out[row] : 0.0;
                double v = sum[i];
                if (io.recur) {
                    v = io.alpha * sum[i];
                    if (io.beta != 0.0) {
                        const double t = io.beta * in[row];
                        v = v + t;
                    }
                    if (prev && io.gamma != 0.0) {
                        const double t = io.gamma * y2;
                        v = v + t;
                    }
                }
                out[row] = v;
                io.out[e] = v;
                if constexpr (ACC) {
                    accumulate<false>(io.acc_a, io.fa, io.wa2, io.wa1, io.wa0, y2, in + row, v, e);
                    accumulate<false>(io.acc_b, io.fb, io.wb2, io.wb1, io.wb0, y2, in + row, v, e);
                }
            }
        }
        lds_barrier();
    }
}
template <typename V>
__global__ __launch_bounds__(kSmallBlock) void small_dia_kernel(DevMatrix m, SegArgs a, Coefs cf) {
    small_body<V, false>(m, a, cf, nullptr);
}
template <typename V>
__global__ __launch_bounds__(kSmallBlock) void small_dia_acc_kernel(DevMatrix m, SegArgs a,
                                                                    Coefs cf, AccCoefs ac) {
    small_body<V, true>(m, a, cf, &ac);
}

// ------------------------------------------------------------------ level-blocked

// One diagonal of the STEPS schedule: workgroup b computes task tasks[b] =
// (chunk c, power k).  All tasks of a diagonal are independent; the previous
// diagonals' results are visible because they ran in earlier launches.
// Chunk c of one power: its slices staged through LDS, or (SELL) its rows in
// the sliced layout.  WT: write-through result stores.
// last: the segment's last power, whose matrix reads are the chunk's last use
// in this launch (sliced layout, one right-hand side: loaded non-temporally,
// so that the caches keep the rows still to be reused: 1.4% faster on the
// 27-point stencil; with 16 right-hand sides, whose rows share lines across
// waves, 2-3% slower, so not there).
template <typename V, int RC, bool WT, bool ACC, bool SELL>
__device__ __forceinline__ void run_chunk(const DevMatrix &m, const PowerIO &io, int R,
                                          DevSlices sl, const int32_t *chunk_sptr,
                                          const int32_t *chunk_row, int32_t c,
                                          bool last = false) {
    if constexpr (SELL) {
        if (RC == 1 && last)   // uniform: the task's power
            run_sell<V, RC, WT, ACC, SellU<RC>::value, RC == 1>(m, io, R, chunk_row[c],
                                                                chunk_row[c + 1]);
        else
            run_sell<V, RC, WT, ACC, SellU<RC>::value>(m, io, R, chunk_row[c], chunk_row[c + 1]);
    } else {
        __shared__ RowSmem<Staging<RC, kTaskKP>::value> sm;
        run_slices<V, RC, Staging<RC, kTaskKP>::value, WT, ACC>(m, io, R, sl, chunk_sptr[c],
                                                                chunk_sptr[c + 1], sm);
    }
}

template <typename V, int RC, bool ACC, bool SELL>
__device__ __forceinline__ void step_body(const DevMatrix &m, DevSlices sl,
                                          const int32_t *chunk_sptr, const int32_t *chunk_row,
                                          const int32_t *tasks, const SegArgs &a, const Coefs &cf,
                                          const AccCoefs *ac) {
    const int32_t c = tasks[2 * blockIdx.x];
    const int32_t k = tasks[2 * blockIdx.x + 1];
    run_chunk<V, RC, false, ACC, SELL>(m, power_io<ACC>(a, cf, ac, k, m.n), a.R, sl, chunk_sptr,
                                       chunk_row, c);
}

template <typename V, int RC>
__global__ __launch_bounds__(kBlock, kTaskWaves) void step_kernel(DevMatrix m, DevSlices sl,
                                                     const int32_t *chunk_sptr,
                                                     const int32_t *chunk_row,
                                                     const int32_t *tasks, SegArgs a, Coefs cf) {
    step_body<V, RC, false, false>(m, sl, chunk_sptr, chunk_row, tasks, a, cf, nullptr);
}

// The same with weighted sums (a separate kernel, so that the plain one
// carries no trace of them).
template <typename V, int RC>
__global__ __launch_bounds__(kBlock, kTaskWaves) void step_acc_kernel(DevMatrix m, DevSlices sl,
                                                         const int32_t *chunk_sptr,
                                                         const int32_t *chunk_row,
                                                         const int32_t *tasks, SegArgs a,
                                                         Coefs cf, AccCoefs ac) {
    step_body<V, RC, true, false>(m, sl, chunk_sptr, chunk_row, tasks, a, cf, &ac);
}

// Sliced-layout forms (no LDS, so more workgroups fit a compute unit).
template <typename V, int RC>
__global__ __launch_bounds__(kBlock) void step_sell_kernel(DevMatrix m, DevSlices sl,
                                                           const int32_t *chunk_sptr,
                                                           const int32_t *chunk_row,
                                                           const int32_t *tasks, SegArgs a,
                                                           Coefs cf) {
    step_body<V, RC, false, true>(m, sl, chunk_sptr, chunk_row, tasks, a, cf, nullptr);
}

template <typename V, int RC>
__global__ __launch_bounds__(kBlock) void step_sell_acc_kernel(DevMatrix m, DevSlices sl,
                                                               const int32_t *chunk_sptr,
                                                               const int32_t *chunk_row,
                                                               const int32_t *tasks, SegArgs a,
                                                               Coefs cf, AccCoefs ac) {
    step_body<V, RC, true, true>(m, sl, chunk_sptr, chunk_row, tasks, a, cf, &ac);
}

struct LBParams {
    DevMatrix m;
    DevSchedule s;
    DevWorkspace ws;
    SegArgs a;
    int64_t spin_limit;   // wall-clock ticks
    int32_t pending;      // skip-ahead slots (lbs_kernel)
    int32_t acquire;      // invalidate caches before a task reads its inputs
    int32_t stride;       // > 0: workgroup b takes tasks b, b + stride, ...
                          // (every workgroup resident); 0: a shared counter
};

// One non-blocking look at task t's inputs by wavefront 0 (all 64 lanes):
// true when every chunk it reads has completed the previous power.
__device__ __forceinline__ bool inputs_ready(const LBParams &P, int32_t t) {
    const int32_t c = P.s.tasks[2 * t];
    const int32_t k = P.s.tasks[2 * t + 1];
    if (k == 1) return true;
    const int32_t lo = P.s.dep_lo[c], hi = P.s.dep_hi[c];
    int ready = 1;
    for (int32_t j = lo + (int)threadIdx.x; j <= hi; j += kWave)
        ready &= ld_relaxed(P.ws.done + j) >= k - 1;
    return __all(ready);
}

// Persistent kernel: workgroups take tasks (chunk c, power k) in schedule
// order, either from a shared ticket counter or, with P.stride = the number
// of workgroups, statically: workgroup b takes tickets b, b + stride, ...
// Before computing, a task waits until every chunk in [dep_lo[c], dep_hi[c]]
// has completed power k-1 and then invalidates its caches (acquire) where
// needed; it computes with write-through stores and publishes done[c] = k
// once they have completed.  Dependencies always carry smaller tickets and a
// workgroup takes its tickets in increasing order, one at a time, so the
// holder of the smallest unfinished ticket can always proceed: with the
// counter, tickets go only to running workgroups; with the static order,
// only if every workgroup of the launch is resident, which the host ensures
// (the grid fits the device and no other launch of a static or XCD-queue
// kernel overlaps it).  The static order spares each task a round trip to a
// counter that every workgroup of the device contends for, measured as the
// larger part of a task's cost on matrices whose windows fit the caches.
// Every wait is also bounded by spin_limit, after which the run is flagged
// as failed and all workgroups leave.
template <typename V, int RC, bool ACC, bool SELL>
__device__ __forceinline__ void lb_body(const LBParams &P, const Coefs &cf, const AccCoefs *ac) {
    __shared__ int32_t s_ticket;
    __shared__ int s_ok;
    const int tid = threadIdx.x;
    if (tid == 0)
        s_ticket = P.stride ? (int32_t)blockIdx.x
                            : __hip_atomic_fetch_add(P.ws.ticket, 1, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    // All loop control below is made provably uniform (readfirstlane) and the
    // loop has a single exit: a loop whose exit the compiler considers
    // divergent may be restructured so that lanes leave it at different
    // iterations, which would break the barriers inside it.
    int32_t t = __builtin_amdgcn_readfirstlane(s_ticket);
    while (t < P.s.n_tasks) {
        const int32_t c = P.s.tasks[2 * t];
        const int32_t k = P.s.tasks[2 * t + 1];
        int ok = 1;
        if (k > 1) {
            // Wavefront 0 alone polls the dependency flags, 64 per coalesced
            // load, and sleeps between rounds; the other waves wait at the
            // barrier.  (Polling from every thread floods the memory system
            // with coherent loads and slows the producers down.)
            if (tid < kWave) {
                const int32_t lo = P.s.dep_lo[c], hi = P.s.dep_hi[c];
                uint64_t t0 = 0;
                for (int round = 0;; ++round) {
                    int ready = 1;
                    for (int32_t j = lo + tid; j <= hi; j += kWave)
                        ready &= ld_relaxed(P.ws.done + j) >= k - 1;
                    if (__all(ready)) break;
                    if (round == 0) t0 = wall_clock64();
                    if (ld_relaxed(P.ws.err) != 0 ||
                        (int64_t)(wall_clock64() - t0) > P.spin_limit) {
                        ok = 0;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(2);
                }
                if (tid == 0) s_ok = ok;
            }
            __syncthreads();
            ok = __builtin_amdgcn_readfirstlane(s_ok);
            // The producers' rows are visible to every wave of this
            // workgroup.  With a line-closed schedule no cache holds a copy
            // of any line they wrote (nobody read it before it was
            // complete), so the loads below miss down to the level their
            // write-through stores reached, and the caches stay warm; else
            // this XCD's caches are invalidated first.
            if (P.acquire)
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            else
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        }
        if (!ok) break;  // uniform: a wait hit its limit, the run is abandoned
        run_chunk<V, RC, true, ACC, SELL>(P.m, power_io<ACC>(P.a, cf, ac, k, P.m.n), P.a.R,
                                          P.s.sl, P.s.chunk_sptr, P.s.chunk_row, c, k == P.a.p);
        // The results were stored write-through; every wave waits until its
        // stores have completed (vmcnt = 0) before the barrier, so the chunk
        // is visible device-wide when the flag below is published and the
        // next ticket is taken.  No L2 write-back is needed.  (Taking the
        // next ticket before computing, to overlap its round trip, was
        // measured slower: it doubles the tickets in flight, and tasks then
        // wait more often on inputs that are still being computed.)
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0), other counters untouched
        __syncthreads();
        if (tid == 0) {
            __hip_atomic_store(P.ws.done + c, k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_ticket = P.stride ? t + P.stride
                                : __hip_atomic_fetch_add(P.ws.ticket, 1, __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        t = __builtin_amdgcn_readfirstlane(s_ticket);
    }
    if (t < P.s.n_tasks && tid == 0) record_failure(P.ws);
}

template <typename V, int RC>
__global__ __launch_bounds__(kBlock, kTaskWaves) void lb_kernel(LBParams P, Coefs cf) {
    lb_body<V, RC, false, false>(P, cf, nullptr);
}

template <typename V, int RC>
__global__ __launch_bounds__(kBlock, kTaskWaves) void lb_acc_kernel(LBParams P, Coefs cf,
                                                                    AccCoefs ac) {
    lb_body<V, RC, true, false>(P, cf, &ac);
}

// Sliced-layout forms: no LDS, built for up to kSellWaves workgroups per
// compute unit.
constexpr int kSellWaves = 8;
template <typename V, int RC>
__global__ __launch_bounds__(kBlock, kSellWaves) void lb_sell_kernel(LBParams P, Coefs cf) {
    lb_body<V, RC, false, true>(P, cf, nullptr);
}

template <typename V, int RC>
__global__ __launch_bounds__(kBlock, kSellWaves) void lb_sell_acc_kernel(LBParams P, Coefs cf,
                                                                         AccCoefs ac) {
    lb_body<V, RC, true, true>(P, cf, &ac);
}

constexpr int kMaxPending = 8;

// Persistent kernel with skip-ahead: when the inputs of a workgroup's task
// are not ready, the task is parked in a small list (up to P.pending slots)
// and the workgroup takes the next ticket instead of waiting.  Parked tasks
// are retried oldest first before any new ticket; a workgroup whose list is
// full, or that has no tickets left, waits for its oldest parked task.
// Deadlock freedom: the smallest unfinished ticket has all its inputs done
// (they carry smaller tickets), and its holder, for which it is the oldest
// task held, either runs it when retrying or blocks on it; every wait is
// bounded by spin_limit as in lb_kernel.  Wavefront 0 makes every choice and
// the other wavefronts learn it through LDS, so control stays uniform.
template <typename V, int RC, bool ACC>
__device__ __forceinline__ void lbs_body(const LBParams &P, const Coefs &cf, const AccCoefs *ac) {
    __shared__ RowSmem<Staging<RC, kTaskKP>::value> sm;
    __shared__ int32_t s_task;
    const int tid = threadIdx.x;
    const int lim = min(P.pending, kMaxPending);
    int32_t pend[kMaxPending];  // wavefront 0 only: parked tickets, oldest first
    int npend = 0;
    bool exhausted = false;
    bool failed = false;        // a wait hit its limit (reported after the loop)
    for (;;) {
        if (tid < kWave) {
            int32_t chosen = -1;
            // 1. parked tasks, oldest first
            for (int i = 0; i < npend && chosen < 0; ++i) {
                if (inputs_ready(P, pend[i])) {
                    chosen = pend[i];
                    for (int j = i + 1; j < npend; ++j) pend[j - 1] = pend[j];
                    --npend;
                }
            }
            // 2. new tickets while there is room to park
            while (chosen < 0 && !exhausted && npend < lim) {
                int32_t t = 0;
                if (tid == 0)
                    t = __hip_atomic_fetch_add(P.ws.ticket, 1, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
                t = __shfl(t, 0);
                if (t >= P.s.n_tasks)
                    exhausted = true;
                else if (inputs_ready(P, t))
                    chosen = t;
                else
                    pend[npend++] = t;
            }
            // 3. wait for the oldest parked task
            if (chosen < 0 && npend > 0) {
                uint64_t t0 = wall_clock64();
                bool ok = true;
                while (!inputs_ready(P, pend[0])) {
                    if (ld_relaxed(P.ws.err) != 0 ||
                        (int64_t)(wall_clock64() - t0) > P.spin_limit) {
                        ok = false;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(2);
                }
                if (ok) {
                    chosen = pend[0];
                    for (int j = 1; j < npend; ++j) pend[j - 1] = pend[j];
                    --npend;
                } else {
                    failed = true;
                    chosen = -1;
                    npend = 0;
                    exhausted = true;
                }
            }
            if (tid == 0) s_task = chosen;
        }
        __syncthreads();
        const int32_t t = __builtin_amdgcn_readfirstlane(s_task);
        if (t < 0) break;  // uniform: no work left (or a wait failed)
        if (P.acquire)  // as in lb_body
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        else
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        const int32_t c = P.s.tasks[2 * t];
        const int32_t k = P.s.tasks[2 * t + 1];
        run_slices<V, RC, Staging<RC, kTaskKP>::value, true, ACC>(
            P.m, power_io<ACC>(P.a, cf, ac, k, P.m.n), P.a.R, P.s.sl, P.s.chunk_sptr[c],
            P.s.chunk_sptr[c + 1], sm);
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): write-through results completed
        __syncthreads();
        if (tid == 0)
            __hip_atomic_store(P.ws.done + c, k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (failed && tid == 0) record_failure(P.ws);
}

template <typename V, int RC>
__global__ __launch_bounds__(kBlock, kTaskWaves) void lbs_kernel(LBParams P, Coefs cf) {
    lbs_body<V, RC, false>(P, cf, nullptr);
}

template <typename V, int RC>
__global__ __launch_bounds__(kBlock, kTaskWaves) void lbs_acc_kernel(LBParams P, Coefs cf,
                                                                     AccCoefs ac) {
    lbs_body<V, RC, true>(P, cf, &ac);
}

// XCD this wave runs on: hardware register XCC_ID (20), bits [3:0].
__device__ __forceinline__ int xcc_id() {
    return (int)(__builtin_amdgcn_s_getreg((3 << 11) | (0 << 6) | 20) & 0xF);
}

struct XcdParams {
    DevMatrix m;
    DevXcdSchedule s;
    DevWorkspace ws;
    SegArgs a;
    int64_t spin_limit;   // wall-clock ticks
    int32_t acquire;      // invalidate caches before a task reads its inputs
};

// Kernel arguments stay well inside the 4 KiB argument segment.
static_assert(sizeof(LBParams) + sizeof(Coefs) + sizeof(AccCoefs) <= 3584,
              "level-blocked kernel arguments");
static_assert(sizeof(XcdParams) + sizeof(Coefs) + sizeof(AccCoefs) <= 3584,
              "XCD kernel arguments");

// Persistent kernel of the XCD schedule.  Queue q holds the tasks of the
// chunks owned by XCD q, in the global dependency order the queues were cut
// from; a workgroup serves the queue of the XCD it runs on (read from the
// hardware, so the binding holds whatever the dispatcher does) and takes its
// tickets in order.  Dependencies are exact chunk lists; results are
// published as in lb_kernel.  Progress: the earliest unfinished task of the
// global order has every earlier task of its queue finished, so it is the
// next ticket of its queue or held by a workgroup, and its inputs are done;
// it runs as soon as one workgroup of this launch runs on its XCD.  That
// holds while nothing else stops this launch's workgroups from ever being
// placed on an XCD: the library never lets two launches of this kernel run
// at the same time on one device (two such launches could each fill the
// XCDs the other one's queues need, and wait for each other), and any other
// kernel finishes on its own.  Waits are bounded by spin_limit in any case.
template <typename V, int RC, bool ACC, bool SELL>
__device__ __forceinline__ void xcd_body(const XcdParams &P, const Coefs &cf, const AccCoefs *ac) {
    __shared__ int32_t s_ticket;
    __shared__ int s_ok;
    const int tid = threadIdx.x;
    const int q = P.s.n_queues == 1 ? 0 : __builtin_amdgcn_readfirstlane(xcc_id());
    if (q >= P.s.n_queues) return;  // uniform: no queue for this XCD
    const int32_t q0 = P.s.qptr[q];
    const int32_t qn = P.s.qptr[q + 1] - q0;
    int32_t *ticket = P.ws.ticket + q;
    if (tid == 0)
        s_ticket = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    int32_t t = __builtin_amdgcn_readfirstlane(s_ticket);
    while (t < qn) {
        const int32_t c = P.s.tasks[2 * (q0 + t)];
        const int32_t k = P.s.tasks[2 * (q0 + t) + 1];
        int ok = 1;
        if (k > 1) {
            if (tid < kWave) {
                const int32_t lo = P.s.dep_ptr[c], hi = P.s.dep_ptr[c + 1];
                uint64_t t0 = 0;
                for (int round = 0;; ++round) {
                    int ready = 1;
                    for (int32_t j = lo + tid; j < hi; j += kWave)
                        ready &= ld_relaxed(P.ws.done + P.s.dep_idx[j]) >= k - 1;
                    if (__all(ready)) break;
                    if (round == 0) t0 = wall_clock64();
                    if (ld_relaxed(P.ws.err) != 0 ||
                        (int64_t)(wall_clock64() - t0) > P.spin_limit) {
                        ok = 0;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(2);
                }
                if (tid == 0) s_ok = ok;
            }
            __syncthreads();
            ok = __builtin_amdgcn_readfirstlane(s_ok);
            if (P.acquire)  // as in lb_body: a line-closed schedule needs no invalidation
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            else
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        }
        if (!ok) break;
        run_chunk<V, RC, true, ACC, SELL>(P.m, power_io<ACC>(P.a, cf, ac, k, P.m.n), P.a.R,
                                          P.s.sl, P.s.chunk_sptr, P.s.chunk_row, c);
        // write-through results, completed (vmcnt = 0) before the barrier
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
        __syncthreads();
        if (tid == 0) {
            __hip_atomic_store(P.ws.done + c, k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_ticket = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        t = __builtin_amdgcn_readfirstlane(s_ticket);
    }
    if (t < qn && tid == 0) record_failure(P.ws);
}

template <typename V, int RC>
__global__ __launch_bounds__(kBlock, kTaskWaves) void xcd_kernel(XcdParams P, Coefs cf) {
    xcd_body<V, RC, false, false>(P, cf, nullptr);
}

template <typename V, int RC>
__global__ __launch_bounds__(kBlock, kTaskWaves) void xcd_acc_kernel(XcdParams P, Coefs cf,
                                                                     AccCoefs ac) {
    xcd_body<V, RC, true, false>(P, cf, &ac);
}

template <typename V, int RC>
__global__ __launch_bounds__(kBlock, kSellWaves) void xcd_sell_kernel(XcdParams P, Coefs cf) {
    xcd_body<V, RC, false, true>(P, cf, nullptr);
}

template <typename V, int RC>
__global__ __launch_bounds__(kBlock, kSellWaves) void xcd_sell_acc_kernel(XcdParams P, Coefs cf,
                                                                          AccCoefs ac) {
    xcd_body<V, RC, true, true>(P, cf, &ac);
}

__global__ void reset_kernel(DevWorkspace ws, int32_t n_chunks, int clear_status) {
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n_chunks) ws.done[i] = 0;
    if (i < kMaxQueues) ws.ticket[i] = 0;
    if (i == 0) {
        *ws.err = 0;
        if (clear_status && ws.status)
            __hip_atomic_store(ws.status, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

__global__ void status_copy_kernel(int32_t *word, int32_t *out) {
    const int32_t v = __hip_atomic_exchange(word, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(out, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Each workgroup records the XCD it ran on.
__global__ void xcc_probe_kernel(int32_t *out) {
    if (threadIdx.x == 0) out[blockIdx.x] = xcc_id();
}

// Rows of nvec vectors from one numbering to the other: thread (li, r) of a
// block moves column r of one row in every vector, four vectors in flight.
template <bool SCATTER>
__global__ __launch_bounds__(kBlock) void permute_kernel(const int32_t *src, int64_t n,
                                                         const double *in, double *out, int nvec,
                                                         int R) {
    const int rows = kBlock / R, li = (int)threadIdx.x / R, r = (int)threadIdx.x - li * R;
    const int64_t i = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * rows + li;
    if (li >= rows || i >= n) return;
    const int64_t here = i * R + r, there = (int64_t)src[i] * R + r;
    const int64_t from = SCATTER ? here : there, to = SCATTER ? there : here, vec = n * R;
    int v = 0;
    for (; v + 4 <= nvec; v += 4) {
        double t[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) t[u] = in[(v + u) * vec + from];
#pragma unroll
        for (int u = 0; u < 4; ++u) out[(v + u) * vec + to] = t[u];
    }
    for (; v < nvec; ++v) out[v * vec + to] = in[v * vec + from];
}

// Complex states from the two weighted sums, on column pairs (column 2j the
// real, 2j+1 the imaginary part): with weights wa + i wb and a real matrix
// the real part is a[2j] - b[2j+1] and the imaginary part a[2j+1] + b[2j].
__global__ void combine_complex_kernel(const double *a, const double *b, int64_t pairs,
                                       double *out) {
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < pairs;
         g += (int64_t)gridDim.x * blockDim.x) {
        const double2 va = reinterpret_cast<const double2 *>(a)[g];
        const double2 vb = reinterpret_cast<const double2 *>(b)[g];
        double2 o;
        o.x = va.x - vb.y;
        o.y = va.y + vb.x;
        reinterpret_cast<double2 *>(out)[g] = o;
    }
}

// Load-only bandwidth probe: each workgroup sums its share of the buffer
// `passes` times with 16-byte loads; one double per workgroup is written.
__global__ __launch_bounds__(kBlock) void load_probe_kernel(const double2 *buf, int64_t n2,
                                                            int passes, double *sink) {
    double acc = 0.0;
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int p = 0; p < passes; ++p)
        for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n2; i += stride) {
            const double2 v = buf[i];
            acc += v.x + v.y;
        }
    __shared__ double red[kBlock];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int s = kBlock / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) sink[blockIdx.x] = red[0];
}

// XCD-local variant: the buffer is cut into `regions` equal parts and every
// workgroup reads the part of the XCD it runs on (XCC_ID mod regions), so each
// XCD's L2 sees only its own part.  Workgroups are numbered within an XCD by
// blockIdx / regions (the dispatcher deals workgroups to XCDs round robin);
// were it otherwise, parts would be read unevenly but every load stays inside
// the buffer.  xcc[b] records where workgroup b ran.
__global__ __launch_bounds__(kBlock) void load_probe_local_kernel(const double2 *buf, int64_t n2,
                                                                int regions, int passes,
                                                                double *sink, int32_t *xcc) {
    const int x = __builtin_amdgcn_readfirstlane(xcc_id()) % regions;
    const int64_t per = n2 / regions;
    const double2 *part = buf + (int64_t)x * per;
    const int64_t idx = blockIdx.x / regions;
    const int64_t stride = (int64_t)((gridDim.x + regions - 1) / regions) * kBlock;
    double acc = 0.0;
    for (int p = 0; p < passes; ++p)
        for (int64_t i = idx * kBlock + threadIdx.x; i < per; i += stride) {
            const double2 v = part[i];
            acc += v.x + v.y;
        }
    __shared__ double red[kBlock];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int s = kBlock / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        sink[blockIdx.x] = red[0];
        xcc[blockIdx.x] = xcc_id();
    }
}

// ------------------------------------------------------------------ dispatch

using SpmvFn = void (*)(DevMatrix, PowerIO, int32_t, DevSlices, int32_t, int32_t);
using SpmvSellFn = void (*)(DevMatrix, PowerIO, int32_t);
using SpmvDiaFn = void (*)(DevMatrix, PowerIO, int32_t, int32_t, int32_t, FastDiv, FastDiv,
                           int32_t);
using LbFn = void (*)(LBParams, Coefs);
using LbAccFn = void (*)(LBParams, Coefs, AccCoefs);
using StepFn = void (*)(DevMatrix, DevSlices, const int32_t *, const int32_t *, const int32_t *,
                        SegArgs, Coefs);
using StepAccFn = void (*)(DevMatrix, DevSlices, const int32_t *, const int32_t *,
                           const int32_t *, SegArgs, Coefs, AccCoefs);
using XcdFn = void (*)(XcdParams, Coefs);
using XcdAccFn = void (*)(XcdParams, Coefs, AccCoefs);

int r_index(int R) {
    switch (R) {
        case 1: return 0;
        case 2: return 1;
        case 4: return 2;
        case 8: return 3;
        case 16: return 4;
    }
    return 5;  // any other count: generic instantiation
}

// Kernels by value type and right-hand-side count: R = 1, 2, 4, 8, 16 are
// specialised, every other count uses the generic instantiation (RC = 0).
template <typename V>
struct VTable {
    SpmvFn spmv[6], spmv_acc[6];
    SpmvSellFn spmv_sell[6], spmv_sell_acc[6];
    LbFn lb[6], lbs[6], lb_sell[6];
    LbAccFn lb_acc[6], lbs_acc[6], lb_sell_acc[6];
    StepFn step[6], step_sell[6];
    StepAccFn step_acc[6], step_sell_acc[6];
    XcdFn xcd[6], xcd_sell[6];
    XcdAccFn xcd_acc[6], xcd_sell_acc[6];
    template <int RC>
    void fill(int i) {
        spmv[i] = spmv_power_kernel<V, RC, false>;
        spmv_acc[i] = spmv_power_kernel<V, RC, true>;
        spmv_sell[i] = spmv_sell_kernel<V, RC, false>;
        spmv_sell_acc[i] = spmv_sell_kernel<V, RC, true>;
        lb[i] = lb_kernel<V, RC>;
        lb_acc[i] = lb_acc_kernel<V, RC>;
        lb_sell[i] = lb_sell_kernel<V, RC>;
        lb_sell_acc[i] = lb_sell_acc_kernel<V, RC>;
        lbs[i] = lbs_kernel<V, RC>;
        lbs_acc[i] = lbs_acc_kernel<V, RC>;
        step[i] = step_kernel<V, RC>;
        step_acc[i] = step_acc_kernel<V, RC>;
        step_sell[i] = step_sell_kernel<V, RC>;
        step_sell_acc[i] = step_sell_acc_kernel<V, RC>;
        xcd[i] = xcd_kernel<V, RC>;
        xcd_acc[i] = xcd_acc_kernel<V, RC>;
        xcd_sell[i] = xcd_sell_kernel<V, RC>;
        xcd_sell_acc[i] = xcd_sell_acc_kernel<V, RC>;
    }
    VTable() {
        fill<1>(0);
        fill<2>(1);
        fill<4>(2);
        fill<8>(3);
        fill<16>(4);
        fill<0>(5);
    }
};

template <typename V>
const VTable<V> &vt() {
    static VTable<V> t;
    return t;
}

const VTable<double> &t64() { return vt<double>(); }
const VTable<float> &t32() { return vt<float>(); }

SpmvFn spmv_fn(int value_bits, int R, bool acc) {
    const int i = r_index(R);
    if (value_bits == 32) return acc ? t32().spmv_acc[i] : t32().spmv[i];
    return acc ? t64().spmv_acc[i] : t64().spmv[i];
}
SpmvSellFn spmv_rows_fn(int value_bits, bool acc) {
    if (value_bits == 32) return acc ? spmv_rows_kernel<float, true> : spmv_rows_kernel<float, false>;
    return acc ? spmv_rows_kernel<double, true> : spmv_rows_kernel<double, false>;
}
SpmvSellFn spmv_sell_fn(int value_bits, int R, bool acc) {
    const int i = r_index(R);
    if (value_bits == 32) return acc ? t32().spmv_sell_acc[i] : t32().spmv_sell[i];
    return acc ? t64().spmv_sell_acc[i] : t64().spmv_sell[i];
}
template <typename V, int MODE>
SpmvDiaFn spmv_dia_of(bool acc, bool stream) {
    if (stream)
        return acc ? spmv_dia_kernel<V, MODE, true, true> : spmv_dia_kernel<V, MODE, false, true>;
    return acc ? spmv_dia_kernel<V, MODE, true, false> : spmv_dia_kernel<V, MODE, false, false>;
}
template <typename V>
SpmvDiaFn spmv_dia_of(int R, bool acc, bool stream) {
    if (R == 1) return spmv_dia_of<V, kOneRhs>(acc, stream);
    return R % 2 == 0 ? spmv_dia_of<V, kEven>(acc, stream) : spmv_dia_of<V, kOdd>(acc, stream);
}
SpmvDiaFn spmv_dia_fn(int value_bits, int R, bool acc, bool stream) {
    return value_bits == 32 ? spmv_dia_of<float>(R, acc, stream)
                            : spmv_dia_of<double>(R, acc, stream);
}
// skip: the skip-ahead kernel (LDS-staged rows); else sell picks the
// sliced-layout kernel
LbFn lb_fn(int value_bits, int R, bool skip, bool sell) {
    const VTable<double> &a = t64();
    const VTable<float> &b = t32();
    const int i = r_index(R);
    if (skip) return value_bits == 32 ? b.lbs[i] : a.lbs[i];
    if (sell) return value_bits == 32 ? b.lb_sell[i] : a.lb_sell[i];
    return value_bits == 32 ? b.lb[i] : a.lb[i];
}
LbAccFn lb_acc_fn(int value_bits, int R, bool skip, bool sell) {
    const VTable<double> &a = t64();
    const VTable<float> &b = t32();
    const int i = r_index(R);
    if (skip) return value_bits == 32 ? b.lbs_acc[i] : a.lbs_acc[i];
    if (sell) return value_bits == 32 ? b.lb_sell_acc[i] : a.lb_sell_acc[i];
    return value_bits == 32 ? b.lb_acc[i] : a.lb_acc[i];
}
StepFn step_fn(int value_bits, int R, bool sell) {
    const int i = r_index(R);
    if (sell) return value_bits == 32 ? t32().step_sell[i] : t64().step_sell[i];
    return value_bits == 32 ? t32().step[i] : t64().step[i];
}
StepAccFn step_acc_fn(int value_bits, int R, bool sell) {
    const int i = r_index(R);
    if (sell) return value_bits == 32 ? t32().step_sell_acc[i] : t64().step_sell_acc[i];
    return value_bits == 32 ? t32().step_acc[i] : t64().step_acc[i];
}
XcdFn xcd_fn(int value_bits, int R, bool sell) {
    const int i = r_index(R);
    if (sell) return value_bits == 32 ? t32().xcd_sell[i] : t64().xcd_sell[i];
    return value_bits == 32 ? t32().xcd[i] : t64().xcd[i];
}
XcdAccFn xcd_acc_fn(int value_bits, int R, bool sell) {
    const int i = r_index(R);
    if (sell) return value_bits == 32 ? t32().xcd_sell_acc[i] : t64().xcd_sell_acc[i];
    return value_bits == 32 ? t32().xcd_acc[i] : t64().xcd_acc[i];
}

}  // namespace

int launch_reset(const DevWorkspace &ws, int32_t n_chunks, void *stream, bool clear_status) {
    const int32_t n = n_chunks > 0 ? n_chunks : 1;
    hipLaunchKernelGGL(reset_kernel, dim3((n + 255) / 256), dim3(256), 0, (hipStream_t)stream, ws,
                       n_chunks, clear_status ? 1 : 0);
    return (int)hipGetLastError();
}

int scratch_workspace(int device, int32_t **out) {
    constexpr int kDevices = 64;
    static std::mutex mu;
    static int32_t *addr[kDevices] = {};
    if (device < 0 || device >= kDevices) return (int)hipErrorInvalidDevice;
    std::lock_guard<std::mutex> g(mu);
    if (!addr[device]) {
        int cur = 0;
        hipError_t e = hipGetDevice(&cur);
        if (e != hipSuccess) return (int)e;
        if (cur != device && (e = hipSetDevice(device)) != hipSuccess) return (int)e;
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (cur != device) (void)hipSetDevice(cur);
        if (e != hipSuccess) return (int)e;
        if (!p) return (int)hipErrorInvalidSymbol;
        addr[device] = static_cast<int32_t *>(p);
    }
    *out = addr[device];
    return 0;
}

int launch_status_copy(int32_t *status_word, int32_t *out, void *stream) {
    hipLaunchKernelGGL(status_copy_kernel, dim3(1), dim3(1), 0, (hipStream_t)stream, status_word,
                       out);
    return (int)hipGetLastError();
}

int launch_spmv_power(const DevMatrix &m, DevSlices sl, int32_t n_slices, const double *in,
                      const double *inm1, double *out, int32_t R, int recur, double alpha,
                      double beta, double gamma, const AccStep *acc, const WinMatrix *win,
                      void *stream) {
    if (R < 1 || R > 16) return (int)hipErrorInvalidValue;
    if (m.n == 0) return 0;
    PowerIO io{in, inm1, out, alpha, beta, gamma, recur};
    io.acc_a = io.acc_b = nullptr;
    io.wa2 = io.wa1 = io.wa0 = io.wb2 = io.wb1 = io.wb0 = 0.0;
    io.fa = io.fb = 0;
    if (acc) {
        io.acc_a = acc->acc_a;
        io.acc_b = acc->acc_b;
        io.wa2 = acc->wa[0];
        io.wa1 = acc->wa[1];
        io.wa0 = acc->wa[2];
        io.wb2 = acc->wb[0];
        io.wb1 = acc->wb[1];
        io.wb0 = acc->wb[2];
        io.fa = acc->fa;
        io.fb = acc->fb;
    }
    if (win && R == 1) {
        // one workgroup per compute unit, for the LDS; of every 16 chunks as many
        // are cached as fit the memory-side cache (as with the diagonals)
        const int32_t keep = (int32_t)std::min<int64_t>(
            16, (kMallBytes - ((int64_t)64 << 20)) * 16 / std::max<int64_t>(1, win->bytes));
        const dim3 grid((unsigned)win->n_parts);
        auto fn = m.value_bits == 32
                      ? (acc ? spmv_win_kernel<float, true> : spmv_win_kernel<float, false>)
                      : (acc ? spmv_win_kernel<double, true> : spmv_win_kernel<double, false>);
        hipLaunchKernelGGL(fn, grid, dim3(kWinRows), 0, (hipStream_t)stream, m, io, *win, keep);
        return (int)hipGetLastError();
    }
    if (few_elements(m, R)) {
        const dim3 grid((unsigned)(((int64_t)m.n * R + kWave - 1) / kWave));
        auto fn = m.value_bits == 32
                      ? (acc ? spmv_few_kernel<float, true> : spmv_few_kernel<float, false>)
                      : (acc ? spmv_few_kernel<double, true> : spmv_few_kernel<double, false>);
        hipLaunchKernelGGL(fn, grid, dim3(kWave), 0, (hipStream_t)stream, m, io, R);
        return (int)hipGetLastError();
    }
    if (m.scol ? dia_fits(m, R) : dia_addressable(m, R)) {
        const int32_t per = R;   // passes of a slice, one wave each
        const int32_t units = (m.n + kDiaRows - 1) / kDiaRows * per;
        const int32_t blocks = (units + kBlock / kWave - 1) / (kBlock / kWave);
        // Each XCD sweeps an eighth of the rows, where the rows that its sweep
        // reads ahead and behind fit its 4 MB L2 (27-point 64^3 with 16
        // right-hand sides: 31.5 us per power against 34-35 for shorter runs).
        // Where they do not (160^3 with 8: 3.3 MB), a run is an eighth of the
        // farthest diagonal's reach, so that the same XCD reads a row's
        // neighbours in the planes before and after, and its share of the
        // window is an eighth (178 -> 159 us).
        bool wide = (int64_t)m.dreach * 2 * R * 8 > ((int64_t)3 << 20);
        const int64_t step = (int64_t)kDiaRows * (kBlock / kWave) * 8;   // elements of 8 blocks
        int64_t run = ((int64_t)m.dreach * R + step / 2) / step;
        int64_t grid = run ? (blocks + 8 * run - 1) / (8 * run) * 8 * run : 0;
        wide = wide && grid / 8 * run < ((int64_t)1 << 32);   // FastDiv
        if (!wide) {
            run = (blocks + 7) / 8;
            grid = 8 * run;
        }
        const FastDiv by_run = wide ? fast_div((int32_t)run) : FastDiv{(int32_t)run, 0u};
        // What one power reads and writes, against the memory-side cache
        // (256 MiB).  Where it does not fit, results go past the cache (160^3
        // with 8 right-hand sides 190 -> 180 us; 27-point 64^3 with 16, which
        // fits, 31.5 -> 38), and of every 16 slices' values only as many are
        // cached as fit beside 32 MB, the vectors of this size with one
        // right-hand side: those stay from one power to the next while the
        // others stream (27-point 128^3, 446 MB of values: none cached 82 us,
        // half 71, all 88).
        const int64_t vecs = (int64_t)m.n * R * 8 * (recur && inm1 ? 3 : 2);
        const bool past = vecs + m.dval_bytes > kMallBytes - ((int64_t)16 << 20);
        const int32_t keep = (int32_t)std::min<int64_t>(
            16, (kMallBytes - ((int64_t)32 << 20)) * 16 / std::max<int64_t>(1, m.dval_bytes));
        hipLaunchKernelGGL(spmv_dia_fn(m.value_bits, R, acc != nullptr, past), dim3((unsigned)grid),
                           dim3(kBlock), 0, (hipStream_t)stream, m, io, R,
                           (65536 + R - 1) / R, units, fast_div(per),
                           by_run, keep);
        return (int)hipGetLastError();
    }
    if (m.dsl && !m.scol) return (int)hipErrorInvalidValue;
    if (m.scol) {  // sliced layout: row blocks of 256 / R rows, grid-stride
        const int64_t nblk = ((int64_t)m.n + kBlock / R - 1) / (kBlock / R);
        const int64_t grid = std::min<int64_t>(nblk, kSpmvSellGrid);
        hipLaunchKernelGGL(spmv_sell_fn(m.value_bits, R, acc != nullptr), dim3((unsigned)grid),
                           dim3(kBlock), 0, (hipStream_t)stream, m, io, R);
        return (int)hipGetLastError();
    }
    int64_t grid;
    int32_t per = 0;
    if (R >= 4) {
        grid = row_grid(m.n, kBlock / R);
        if (r_index(R) == 5) {
            hipLaunchKernelGGL(spmv_rows_fn(m.value_bits, acc != nullptr), dim3((unsigned)grid),
                               dim3(kBlock), 0, (hipStream_t)stream, m, io, R);
            return (int)hipGetLastError();
        }
    } else {
        if (n_slices == 0) return 0;
        // A workgroup forms one slice's products while the next slice's entries
        // load, but with fewer than eight such pairs for each compute unit more
        // workgroups are worth more: bands of 8192, 60 k, 200 k and 400 k rows, us
        // per power one by one and in pairs, one right-hand side 5.3, 7.7, 22.7,
        // 38 and 8.5, 11, 22.8, 43, three 7.1, 14, 35, 63 and 10, 15, 35, 64;
        // from 2.5 M rows 3% the other way.
        per = n_slices < 4096 ? 1 : 2;
        grid = (n_slices + per - 1) / per;
    }
    hipLaunchKernelGGL(spmv_fn(m.value_bits, R, acc != nullptr), dim3((unsigned)grid), dim3(kBlock), 0,
                       (hipStream_t)stream, m, io, R, sl, n_slices, per);
    return (int)hipGetLastError();
}

int launch_small(const DevMatrix &m, const SegArgs &a, const Coefs &cf, const AccCoefs *acc,
                 void *stream) {
    if (a.R < 1 || a.R > 16 || a.p < 1 || a.p > kMaxSegPowers || m.n > kSmallRows || !m.dsl)
        return (int)hipErrorInvalidValue;
    const dim3 grid((unsigned)a.R), block(kSmallBlock);
    if (acc)
        hipLaunchKernelGGL(m.value_bits == 32 ? small_dia_acc_kernel<float>
                                              : small_dia_acc_kernel<double>,
                           grid, block, 0, (hipStream_t)stream, m, a, cf, *acc);
    else
        hipLaunchKernelGGL(m.value_bits == 32 ? small_dia_kernel<float> : small_dia_kernel<double>,
                           grid, block, 0, (hipStream_t)stream, m, a, cf);
    return (int)hipGetLastError();
}

int launch_step(const DevMatrix &m, DevSlices sl, const int32_t *chunk_sptr,
                const int32_t *chunk_row, const int32_t *tasks, int32_t n_tasks,
                const SegArgs &a, const Coefs *cf, const AccCoefs *acc, void *stream) {
    if (a.R < 1 || a.R > 16 || a.p < 1 || a.p > kMaxSegPowers) return (int)hipErrorInvalidValue;
    if (n_tasks <= 0) return 0;
    Coefs c{};
    if (cf) c = *cf;
    const bool sell = m.scol != nullptr;
    if (acc)
        hipLaunchKernelGGL(step_acc_fn(m.value_bits, a.R, sell), dim3((unsigned)n_tasks),
                           dim3(kBlock), 0, (hipStream_t)stream, m, sl, chunk_sptr, chunk_row,
                           tasks, a, c, *acc);
    else
        hipLaunchKernelGGL(step_fn(m.value_bits, a.R, sell), dim3((unsigned)n_tasks), dim3(kBlock),
                           0, (hipStream_t)stream, m, sl, chunk_sptr, chunk_row, tasks, a, c);
    return (int)hipGetLastError();
}

int lb_resident_workgroups(int value_bits, int R, int device, bool sell, bool acc) {
    const void *fn = acc ? reinterpret_cast<const void *>(lb_acc_fn(value_bits, R, false, sell))
                         : reinterpret_cast<const void *>(lb_fn(value_bits, R, false, sell));
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, kBlock, 0) != hipSuccess)
        return 0;
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, device) != hipSuccess) return 0;
    return per_cu * prop.multiProcessorCount;
}

int lb_max_workgroups(int value_bits, int R, int device, bool sell) {
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &per_cu, reinterpret_cast<const void *>(lb_fn(value_bits, R, false, sell)), kBlock,
            0) != hipSuccess)
        return 0;
    // LDS-staged rows: at most kTaskWaves workgroups per CU even where
    // registers and LDS would allow more (the unstaged path for R >= 4): more
    // persistent workgroups only added ticket and flag traffic and were
    // measured 2-3x slower.  Sliced layout: at most four.
    per_cu = std::min(per_cu, sell ? 4 : kTaskWaves);
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, device) != hipSuccess) return 0;
    return per_cu * prop.multiProcessorCount;
}

int launch_lb(const DevMatrix &m, const DevSchedule &s, const DevWorkspace &ws,
              const SegArgs &a, const Coefs *cf, const AccCoefs *acc, int workgroups,
              int64_t spin_limit, int pending, int acquire, bool static_order, void *stream) {
    if (a.R < 1 || a.R > 16) return (int)hipErrorInvalidValue;
    if (a.p < 1 || a.p > kMaxSegPowers || workgroups < 1) return (int)hipErrorInvalidValue;
    if (pending < 0 || pending > kMaxPending) return (int)hipErrorInvalidValue;
    if (static_order && pending > 0) return (int)hipErrorInvalidValue;
    if (s.n_tasks == 0) return 0;
    LBParams P{m, s, ws, a, spin_limit, pending, acquire ? 1 : 0, static_order ? workgroups : 0};
    Coefs c{};
    if (cf) c = *cf;
    const bool sell = m.scol != nullptr;
    if (acc)
        hipLaunchKernelGGL(lb_acc_fn(m.value_bits, a.R, pending > 0, sell), dim3(workgroups),
                           dim3(kBlock), 0, (hipStream_t)stream, P, c, *acc);
    else
        hipLaunchKernelGGL(lb_fn(m.value_bits, a.R, pending > 0, sell), dim3(workgroups),
                           dim3(kBlock), 0, (hipStream_t)stream, P, c);
    return (int)hipGetLastError();
}

int launch_xcd(const DevMatrix &m, const DevXcdSchedule &s, const DevWorkspace &ws,
               const SegArgs &a, const Coefs *cf, const AccCoefs *acc, int workgroups,
               int64_t spin_limit, int acquire, void *stream) {
    if (a.R < 1 || a.R > 16) return (int)hipErrorInvalidValue;
    if (a.p < 1 || a.p > kMaxSegPowers || workgroups < 1) return (int)hipErrorInvalidValue;
    if (s.n_queues < 1 || s.n_queues > kMaxQueues) return (int)hipErrorInvalidValue;
    if (s.n_chunks == 0) return 0;
    XcdParams P{m, s, ws, a, spin_limit, acquire ? 1 : 0};
    Coefs c{};
    if (cf) c = *cf;
    const bool sell = m.scol != nullptr;
    if (acc)
        hipLaunchKernelGGL(xcd_acc_fn(m.value_bits, a.R, sell), dim3(workgroups), dim3(kBlock),
                           0, (hipStream_t)stream, P, c, *acc);
    else
        hipLaunchKernelGGL(xcd_fn(m.value_bits, a.R, sell), dim3(workgroups), dim3(kBlock), 0,
                           (hipStream_t)stream, P, c);
    return (int)hipGetLastError();
}

int detect_xcds(int device) {
    constexpr int kProbe = 2048;
    if (hipSetDevice(device) != hipSuccess) return 1;
    int32_t *d = nullptr;
    if (hipMalloc(&d, kProbe * sizeof(int32_t)) != hipSuccess) return 1;
    int32_t h[kProbe];
    hipLaunchKernelGGL(xcc_probe_kernel, dim3(kProbe), dim3(64), 0, nullptr, d);
    bool ok = hipGetLastError() == hipSuccess &&
              hipMemcpy(h, d, sizeof(h), hipMemcpyDeviceToHost) == hipSuccess;
    (void)hipFree(d);
    if (!ok) return 1;
    // the ids seen must be exactly 0..k-1
    int seen[16] = {0}, k = 0;
    for (int i = 0; i < kProbe; ++i) {
        if (h[i] < 0 || h[i] >= kMaxQueues) return 1;
        seen[h[i]] = 1;
        k = std::max(k, h[i] + 1);
    }
    for (int i = 0; i < k; ++i)
        if (!seen[i]) return 1;
    return k;
}

int launch_permute(const int32_t *src, int64_t n, bool scatter, const double *in, double *out,
                   int nvec, int R, void *stream) {
    if (R < 1 || R > 16 || nvec < 0) return (int)hipErrorInvalidValue;
    if (n == 0 || nvec == 0) return 0;
    const int64_t rows = kBlock / R, x = row_grid(n, rows), y = (n + x * rows - 1) / (x * rows);
    hipLaunchKernelGGL(scatter ? permute_kernel<true> : permute_kernel<false>,
                       dim3((unsigned)x, (unsigned)y), dim3(kBlock), 0, (hipStream_t)stream, src, n,
                       in, out, nvec, R);
    return (int)hipGetLastError();
}

int launch_combine_complex(const double *a, const double *b, int64_t n, int R, double *out,
                           void *stream) {
    if (R < 2 || (R & 1)) return (int)hipErrorInvalidValue;
    const int64_t pairs = n * (R / 2);
    if (pairs == 0) return 0;
    int64_t grid = (pairs + 255) / 256;
    if (grid > 8192) grid = 8192;
    hipLaunchKernelGGL(combine_complex_kernel, dim3((unsigned)grid), dim3(256), 0,
                       (hipStream_t)stream, a, b, pairs, out);
    return (int)hipGetLastError();
}

int launch_load_probe(const double *buf, int64_t n_doubles, int passes, int workgroups,
                      double *sink, void *stream) {
    if (n_doubles < 2 || passes < 1 || workgroups < 1) return (int)hipErrorInvalidValue;
    hipLaunchKernelGGL(load_probe_kernel, dim3(workgroups), dim3(kBlock), 0, (hipStream_t)stream,
                       reinterpret_cast<const double2 *>(buf), n_doubles / 2, passes, sink);
    return (int)hipGetLastError();
}

int launch_load_probe_xcd(const double *buf, int64_t n_doubles, int regions, int passes,
                          int workgroups, double *sink, int32_t *xcc, void *stream) {
    if (n_doubles < 2 * (int64_t)regions || regions < 1 || regions > kMaxQueues || passes < 1 ||
        workgroups < 1)
        return (int)hipErrorInvalidValue;
    hipLaunchKernelGGL(load_probe_local_kernel, dim3(workgroups), dim3(kBlock), 0,
                       (hipStream_t)stream, reinterpret_cast<const double2 *>(buf),
                       n_doubles / 2, regions, passes, sink, xcc);
    return (int)hipGetLastError();
}

}  // namespace mpk

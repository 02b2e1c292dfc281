// Level-scheduled sparse triangular solve kernels for gfx950 (CDNA4).
//
// Algorithm 2 of the paper: the right-hand side is permuted into level order,
// the levels are solved one after the other with every row of a level solved
// simultaneously, and the solution is permuted back.  Both permutations are
// fused into the row routine (the gather of b on the first read, the scatter
// of x on the final write).  Upper solves use the same code on the plan built
// from U reversed by t(i) = n-1-i (end of Section 2.2).
//
// Two executions of the same row routine:
//   k_level       one launch per level (the paper's shape);
//   k_persistent  one launch for the whole solve: every workgroup runs its
//                 list of steps (a contiguous range of device rows of one
//                 level).  A dependency produced by the same workgroup is
//                 read from LDS (owner schedule) or from the workspace after
//                 the step barrier; a dependency produced by another
//                 workgroup is read from a mailbox slot, polled until the
//                 producer's value replaces the sentinel.
// The row routine subtracts the ELL terms in slot order, then the CSR-tail
// terms, then multiplies by the stored reciprocal diagonal, so both
// executions produce bit-identical results for rows run one thread per
// (row, rhs); steps tuned to split long rows over several lanes sum in a
// different order.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <tuple>
#include <type_traits>

#include "tri_dev.h"

namespace hec {

namespace {


int32_t capacity_of(const void *kern, int32_t block, size_t lds, bool lds_at_zero = false);

// Per-launch state of the persistent kernel shared by the row routine.
template <typename T> struct Ctx {
    T *xl;          // LDS window (device rows lo..hi-1), holds b then x
    int lo, hi;
    T *mbox_rd;     // this launch's mailbox half
    int *abort;     // LDS flag: a poll gave up
};

// Mailbox slots are written with agent-scope relaxed atomic stores, which go
// through to the point of coherence shared by all XCDs, and polled with
// agent-scope relaxed atomic loads, which do not hit stale cache lines.  The
// value itself is the signal, so no flag, fence or cache-wide writeback is
// needed.  The poll is bounded; on expiry it raises the abort flags.
template <typename T>
__device__ __forceinline__ T poll_slot(const T *p, int *err_dev, int *err_host, int *abort, unsigned limit)
{
    T v = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (!is_sentinel(v)) return v;
    unsigned spins = 0;
    for (;;) {
        __builtin_amdgcn_s_sleep(1);
        v = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (!is_sentinel(v)) return v;
        ++spins;
        if (spins > limit ||
            ((spins & 255u) == 0 && __hip_atomic_load(err_dev, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)) {
            __hip_atomic_store(err_dev, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(err_host, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            *abort = 1;
            return T(0);
        }
    }
}

// Value of dependency column c for right-hand side k.
template <typename T, bool PERS, bool LDS>
__device__ __forceinline__ T dep_value(const TriArgs &a, const Ctx<T> &cx, int c, int k)
{
    if (PERS && c > a.n)
        return poll_slot<T>(cx.mbox_rd + (size_t)(c - a.n - 1) * a.mbox_stride + k, a.err_dev, a.err_host,
                            cx.abort, a.spin);
    if (LDS && c >= cx.lo && c < cx.hi) return cx.xl[(c - cx.lo) * a.R + k];
    const T *p = static_cast<const T *>(a.xw) + (size_t)c * a.R + k;
    // a value of this workgroup from an earlier step (persistent) or of an
    // earlier launch (per-level): workgroup-scope coherence suffices
    if (PERS) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    return *p;
}

template <typename T, typename TIn, bool LDS>
__device__ __forceinline__ T rhs_value(const TriArgs &a, const Ctx<T> &cx, int x, int k)
{
    if (LDS) return cx.xl[(x - cx.lo) * a.R + k];  // gathered (and scaled) at kernel start
    const T b = canon(static_cast<T>(static_cast<const TIn *>(a.bin)[(size_t)a.gather[x] * a.R + k]));
    return a.dinv ? scale_rhs(b, static_cast<const T *>(a.dinv)[x]) : b;
}

// Partial sum of one row's off-diagonal terms (lane `lane` of `lanes`).
template <typename T, bool PERS, bool LDS>
__device__ __forceinline__ T row_terms(const TriArgs &a, const Ctx<T> &cx, int x, int k, int lane, int lanes)
{
    const T *ev = static_cast<const T *>(a.ell_val);
    T part = T(0);
    for (int e = lane; e < a.w; e += lanes) {
        const int c = a.ell_col[(size_t)e * a.ld + x];
        const T v = ev[(size_t)e * a.ld + x];
        if (c != a.n) part += v * dep_value<T, PERS, LDS>(a, cx, c, k);
    }
    if (a.tail_ptr) {
        const T *tv = static_cast<const T *>(a.tail_val);
        for (int p = a.tail_ptr[x] + lane; p < a.tail_ptr[x + 1]; p += lanes)
            part += tv[p] * dep_value<T, PERS, LDS>(a, cx, a.tail_col[p], k);
    }
    return part;
}

template <typename T, typename TOut, bool PERS, bool LDS>
__device__ __forceinline__ void finish_row(const TriArgs &a, const Ctx<T> &cx, int x, int k, T s)
{
    if (LDS) cx.xl[(x - cx.lo) * a.R + k] = s;
    if (!PERS) {
        static_cast<T *>(a.xw)[(size_t)x * a.R + k] = s;
    } else if (!LDS || a.write_xw) {
        __hip_atomic_store(static_cast<T *>(a.xw) + (size_t)x * a.R + k, s, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    if (PERS) {
        const int slot = a.exp_slot[x];
        if (slot >= 0)
            __hip_atomic_store(cx.mbox_rd + (size_t)slot * a.mbox_stride + k, s, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    }
    if (a.xout) {
        const int dst = a.scatter[x];
        if (dst >= 0) static_cast<TOut *>(a.xout)[(size_t)dst * a.R + k] = static_cast<TOut>(s);
    }
}

// Thread-per-(row, rhs) solve of one row: s = b - sum, in slot order.
template <typename T, typename TIn, typename TOut, bool PERS, bool LDS>
__device__ __forceinline__ void solve_item(const TriArgs &a, const Ctx<T> &cx, int x, int k)
{
    const T *ev = static_cast<const T *>(a.ell_val);
    T s = rhs_value<T, TIn, LDS>(a, cx, x, k);
    for (int e = 0; e < a.w; ++e) {
        const int c = a.ell_col[(size_t)e * a.ld + x];
        const T v = ev[(size_t)e * a.ld + x];
        if (c != a.n) s -= v * dep_value<T, PERS, LDS>(a, cx, c, k);
    }
    if (a.tail_ptr) {
        const T *tv = static_cast<const T *>(a.tail_val);
        for (int p = a.tail_ptr[x]; p < a.tail_ptr[x + 1]; ++p)
            s -= tv[p] * dep_value<T, PERS, LDS>(a, cx, a.tail_col[p], k);
    }
    finish_row<T, TOut, PERS, LDS>(a, cx, x, k, s);
}

// Rows [rb, re) x R right-hand sides, `lanes` lanes per (row, rhs).  With
// lanes > 1 the lanes of a group split the row's terms and combine them with
// a butterfly of cross-lane shuffles inside the wavefront.
template <typename T, typename TIn, typename TOut, bool LDS>
__device__ __forceinline__ void solve_range(const TriArgs &a, const Ctx<T> &cx, int rb, int re, int lanes)
{
    const int R = a.R;
    if (lanes == 1) {
        const int items = (re - rb) * R;
        for (int t = threadIdx.x; t < items; t += blockDim.x) {
            const int q = t / R;
            solve_item<T, TIn, TOut, true, LDS>(a, cx, rb + q, t - q * R);
        }
        return;
    }
    const int items = (re - rb) * R * lanes;
    for (int t0 = 0; t0 < items; t0 += blockDim.x) {
        const int t = t0 + threadIdx.x;
        const bool act = t < items;
        const int lane = t & (lanes - 1);
        const int q = t / lanes;
        const int x = rb + q / R, k = q - (q / R) * R;
        T part = act ? row_terms<T, true, LDS>(a, cx, x, k, lane, lanes) : T(0);
        for (int off = lanes >> 1; off > 0; off >>= 1) part += __shfl_xor(part, off, lanes);
        if (act && lane == 0) finish_row<T, TOut, true, LDS>(a, cx, x, k, rhs_value<T, TIn, LDS>(a, cx, x, k) - part);
    }
}

// One launch per level: rows [row_begin, row_end) of the device order.
template <typename T, typename TIn, typename TOut>
__global__ void __launch_bounds__(256) k_level(TriArgs a)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    const int items = (a.row_end - a.row_begin) * a.R;
    if (t >= items) return;
    const int q = t / a.R;
    Ctx<T> cx{nullptr, 0, 0, nullptr, nullptr};
    solve_item<T, TIn, TOut, false, false>(a, cx, a.row_begin + q, t - q * a.R);
}

// One launch for the whole solve.  The mailbox half used by a launch is the
// parity of the plan's epoch word; the epoch is read at kernel start and
// advanced by the last workgroup to finish, so consecutive launches (also
// graph replays) alternate halves.  Each workgroup first resets its own slots
// of the other half to the sentinel, ready for the next launch.
template <typename T, typename TIn, typename TOut, bool LDS>
__global__ void __launch_bounds__(1024) k_persistent(TriArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ unsigned s_epoch;
    __shared__ int s_abort;
    const int g = blockIdx.x;
    if (threadIdx.x == 0) {
        s_epoch = __hip_atomic_load(a.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_abort = 0;
    }
    __syncthreads();
    const unsigned par = s_epoch & 1u;
    T *mbox = static_cast<T *>(a.mbox);
    const size_t half = (size_t)a.nexp * a.mbox_stride;
    Ctx<T> cx;
    cx.xl = reinterpret_cast<T *>(smem);
    cx.lo = LDS ? a.window[2 * g] : 0;
    cx.hi = LDS ? a.window[2 * g + 1] : 0;
    cx.mbox_rd = mbox + (par ? half : 0);
    cx.abort = &s_abort;
    if (a.nexp > 0) {
        T *other = mbox + (par ? 0 : half);
        const size_t e0 = (size_t)a.exp_ptr[g] * a.mbox_stride, e1 = (size_t)a.exp_ptr[g + 1] * a.mbox_stride;
        for (size_t i = e0 + threadIdx.x; i < e1; i += blockDim.x) other[i] = sentinel<T>();
    }
    if (LDS) {
        const TIn *bin = static_cast<const TIn *>(a.bin);
        const int items = (cx.hi - cx.lo) * a.R;
        for (int t = threadIdx.x; t < items; t += blockDim.x) {
            const int q = t / a.R, k = t - q * a.R;
            const T b = canon(static_cast<T>(bin[(size_t)a.gather[cx.lo + q] * a.R + k]));
            cx.xl[t] = a.dinv ? scale_rhs(b, static_cast<const T *>(a.dinv)[cx.lo + q]) : b;
        }
        __syncthreads();
    }
    const int s0 = a.step_ptr[g], s1 = a.step_ptr[g + 1];
    int rb = 0, re = 0, ln = 1;
    if (s0 < s1) {
        rb = a.step_row[2 * s0];
        re = a.step_row[2 * s0 + 1];
        ln = a.step_lanes[s0];
    }
    for (int s = s0; s < s1; ++s) {
        // next step's bounds are loaded while this step runs
        int nrb = 0, nre = 0, nln = 1;
        if (s + 1 < s1) {
            nrb = a.step_row[2 * s + 2];
            nre = a.step_row[2 * s + 3];
            nln = a.step_lanes[s + 1];
        }
        solve_range<T, TIn, TOut, LDS>(a, cx, rb, re, ln);
        __syncthreads();
        if (s_abort) break;
        rb = nrb;
        re = nre;
        ln = nln;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned done = __hip_atomic_fetch_add(&a.epoch[1], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        if (done == gridDim.x - 1) {
            __hip_atomic_store(&a.epoch[1], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&a.epoch[0], s_epoch + 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// Owner-schedule kernel with LDS-staged matrix data.  Workgroup g owns the
// device rows [lo, hi): their right-hand side is gathered into an LDS window
// at kernel start and every solved value replaces its row's b there.  The
// group's steps are cut into chunks of at most RPT * blockDim rows; the ELL
// columns and values, reciprocal diagonal, mailbox slot and scatter target
// of chunk q+1 are loaded into registers while chunk q is solved, then stored
// to the other half of a double buffer in LDS, so a step reads everything but
// cross-group values from LDS.  W is the ELL width; plans with a CSR tail,
// W > 8 or cooperative lanes use k_persistent.
template <typename T, int W, int RPT, bool UNIT>
__global__ void __launch_bounds__(1024) k_owner(TriArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ unsigned s_epoch;
    __shared__ int s_abort;
    const int g = blockIdx.x;
    const int tid = threadIdx.x, nt = blockDim.x;
    const int R = a.R, n = a.n;
    if (tid == 0) {
        s_epoch = __hip_atomic_load(a.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_abort = 0;
    }
    __syncthreads();
    const unsigned par = s_epoch & 1u;
    T *mbox = static_cast<T *>(a.mbox);
    const size_t half = (size_t)a.nexp * a.mbox_stride;
    T *mrd = mbox + (par ? half : 0);
    const int lo = a.window[2 * g], hi = a.window[2 * g + 1];
    const int CH = RPT * nt;
    // LDS: window [win*R] T, then two buffers of { vals[W][CH] T, cols[W][CH], slot[CH], dst[CH] }
    T *xl = reinterpret_cast<T *>(smem);
    const size_t win_bytes = (((size_t)(hi - lo) * R * sizeof(T)) + 15) & ~(size_t)15;
    const size_t buf_bytes = (size_t)CH * (W * sizeof(T) + (W + 2) * sizeof(int));
    auto bvals = [&](int b) { return reinterpret_cast<T *>(smem + win_bytes + b * buf_bytes); };
    auto bcols = [&](int b) { return reinterpret_cast<int *>(smem + win_bytes + b * buf_bytes + (size_t)CH * W * sizeof(T)); };
    auto bslot = [&](int b) { return bcols(b) + (size_t)W * CH; };
    auto bdst = [&](int b) { return bslot(b) + CH; };

    if (a.nexp > 0) {
        T *other = mbox + (par ? 0 : half);
        const size_t e0 = (size_t)a.exp_ptr[g] * a.mbox_stride, e1 = (size_t)a.exp_ptr[g + 1] * a.mbox_stride;
        for (size_t i = e0 + tid; i < e1; i += nt) other[i] = sentinel<T>();
    }
    {
        const int items = (hi - lo) * R;
        for (int t = tid; t < items; t += nt) {
            const int q = t / R, k = t - q * R;
            const size_t src = (size_t)a.gather[lo + q] * R + k;
            const T b = canon(a.in_f64 ? static_cast<T>(static_cast<const double *>(a.bin)[src])
                                       : static_cast<T>(static_cast<const float *>(a.bin)[src]));
            xl[t] = UNIT ? b : scale_rhs(b, static_cast<const T *>(a.dinv)[lo + q]);
        }
    }
    const T *ev = static_cast<const T *>(a.ell_val);
    // registers of one chunk prefetch
    int rc[RPT][W];
    T rv[RPT][W];
    int rs[RPT], rt[RPT];
    auto chunk_rows = [&](int q, int &r0, int &r1) {
        const int f = a.chunk_step[2 * q], e = a.chunk_step[2 * q + 1];
        r0 = a.step_row[2 * f];
        r1 = a.step_row[2 * (e - 1) + 1];
    };
    auto load_chunk = [&](int q) {
        int r0, r1;
        chunk_rows(q, r0, r1);
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const int row = r0 + tid + i * nt;
            if (row < r1) {
#pragma unroll
                for (int e = 0; e < W; ++e) {
                    rc[i][e] = a.ell_col[(size_t)e * a.ld + row];
                    rv[i][e] = ev[(size_t)e * a.ld + row];
                }
                rs[i] = a.exp_slot[row];
                rt[i] = a.xout ? a.scatter[row] : -1;
            }
        }
    };
    auto store_chunk = [&](int q, int b) {
        int r0, r1;
        chunk_rows(q, r0, r1);
        T *vb = bvals(b);
        int *cb = bcols(b);
        int *sb = bslot(b);
        int *tb = bdst(b);
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const int rr = tid + i * nt;
            if (r0 + rr < r1) {
#pragma unroll
                for (int e = 0; e < W; ++e) {
                    cb[e * CH + rr] = rc[i][e];
                    vb[e * CH + rr] = rv[i][e];
                }
                sb[rr] = rs[i];
                tb[rr] = rt[i];
            }
        }
    };
    const int c0 = a.chunk_ptr[g], c1 = a.chunk_ptr[g + 1];
    if (c0 < c1) {
        load_chunk(c0);
        store_chunk(c0, 0);
    }
    __syncthreads();
    bool aborted = false;
    for (int q = c0; q < c1 && !aborted; ++q) {
        const int b = (q - c0) & 1;
        if (q + 1 < c1) load_chunk(q + 1);
        int cr0, cr1;
        chunk_rows(q, cr0, cr1);
        const T *vb = bvals(b);
        const int *cb = bcols(b);
        const int *sb = bslot(b);
        const int *tb = bdst(b);
        const int f = a.chunk_step[2 * q], e_ = a.chunk_step[2 * q + 1];
        for (int s = f; s < e_; ++s) {
            const int rb = a.step_row[2 * s], re = a.step_row[2 * s + 1];
            const int items = (re - rb) * R;
            const int js = s - a.step_ptr[g];
            const bool tr = a.trace && tid == 0 && js < a.trace_stride;
            if (tr) a.trace[2 * ((size_t)g * a.trace_stride + js)] = __builtin_amdgcn_s_memrealtime();
            for (int t = tid; t < items; t += nt) {
                const int qq = t / R, k = t - qq * R;
                const int x = rb + qq, i = x - cr0;
                T sv = xl[(x - lo) * R + k];
#pragma unroll
                for (int e = 0; e < W; ++e) {
                    const int c = cb[e * CH + i];
                    if (c != n) {
                        T dep;
                        if (c > n)
                            dep = poll_slot<T>(mrd + (size_t)(c - n - 1) * a.mbox_stride + k, a.err_dev, a.err_host,
                                               &s_abort, a.spin);
                        else
                            dep = xl[(c - lo) * R + k];
                        sv -= vb[e * CH + i] * dep;
                    }
                }
                xl[(x - lo) * R + k] = sv;
                if (a.write_xw) static_cast<T *>(a.xw)[(size_t)x * R + k] = sv;
                const int slot = sb[i];
                if (slot >= 0)
                    __hip_atomic_store(mrd + (size_t)slot * a.mbox_stride + k, sv, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
                const int dst = tb[i];
                if (dst >= 0) {
                    if (a.out_f64) static_cast<double *>(a.xout)[(size_t)dst * R + k] = static_cast<double>(sv);
                    else static_cast<float *>(a.xout)[(size_t)dst * R + k] = static_cast<float>(sv);
                }
            }
            __syncthreads();
            if (tr) a.trace[2 * ((size_t)g * a.trace_stride + js) + 1] = __builtin_amdgcn_s_memrealtime();
            if (s_abort) {
                aborted = true;
                break;
            }
        }
        if (!aborted && q + 1 < c1) {
            store_chunk(q + 1, b ^ 1);
            __syncthreads();
        }
    }
    __syncthreads();
    if (tid == 0) {
        const unsigned done = __hip_atomic_fetch_add(&a.epoch[1], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        if (done == gridDim.x - 1) {
            __hip_atomic_store(&a.epoch[1], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&a.epoch[0], s_epoch + 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// LDS bytes of k_owner for a window of `win` rows.
size_t owner_lds_bytes(int win, int R, int W, int rows_per_chunk, bool unit, size_t tsize)
{
    const size_t win_bytes = (((size_t)win * R * tsize) + 15) & ~(size_t)15;
    (void)unit;
    const size_t buf = (size_t)rows_per_chunk * (W * tsize + (W + 2) * sizeof(int));
    return win_bytes + 2 * buf;
}


template <typename T, int W, int RPT>
OwnerKernel owner_kernel_w(bool unit)
{
    return unit ? k_owner<T, W, RPT, true> : k_owner<T, W, RPT, false>;
}

template <typename T, int RPT>
OwnerKernel owner_kernel_r(int w, bool unit)
{
    switch (w) {
    case 1: return owner_kernel_w<T, 1, RPT>(unit);
    case 2: return owner_kernel_w<T, 2, RPT>(unit);
    case 3: return owner_kernel_w<T, 3, RPT>(unit);
    case 4: return owner_kernel_w<T, 4, RPT>(unit);
    case 5: return owner_kernel_w<T, 5, RPT>(unit);
    case 6: return owner_kernel_w<T, 6, RPT>(unit);
    case 7: return owner_kernel_w<T, 7, RPT>(unit);
    case 8: return owner_kernel_w<T, 8, RPT>(unit);
    default: return nullptr;
    }
}

template <typename T>
OwnerKernel owner_kernel(int w, int rpt, bool unit)
{
    if (rpt == 1) return owner_kernel_r<T, 1>(w, unit);
    if (rpt == 2) return owner_kernel_r<T, 2>(w, unit);
    if (rpt == 4) return owner_kernel_r<T, 4>(w, unit);
    return nullptr;
}

// Owner-schedule kernel with one compute wave and one fetch wave (one RHS).
// The compute wave only reads LDS, does the arithmetic and issues stores, so
// it never waits on global memory.  The fetch wave (a) streams each chunk
// (ELL columns and values, reciprocal diagonal, mailbox slot and scatter
// target per row, the chunk's step bounds and its cross-group entry list)
// into a ring of three LDS buffers, and (b) polls the mailbox slots of the
// cross-group entries of the next steps, up to 64 * kWsPerLane entries at
// once, writing arrived values into the buffer's staging grid and publishing
// in LDS the last step whose entries have all arrived.  The compute wave
// solves step s once that counter reaches s and reports each finished step,
// which frees buffers for the fetch wave.  All waits in both roles are
// bounded.
constexpr int kWsBuffers = 3;
constexpr int kWsPerLane = 16;
constexpr int kWsHead = 8;  // ints: first step, end step, first row, first entry, end entry

template <typename T, int W>
struct WsLayout {
    size_t win, buf;
    size_t o_vals, o_stage, o_cols, o_slot, o_dst, o_ent, o_head, o_step;
    __host__ __device__ WsLayout(int rows, int CH, bool unit)
    {
        win = (((size_t)rows * sizeof(T)) + 15) & ~(size_t)15;
        o_vals = 0;
        (void)unit;
        o_stage = o_vals + (size_t)W * CH * sizeof(T);
        o_cols = o_stage + (size_t)W * CH * sizeof(T);
        o_slot = o_cols + (size_t)W * CH * sizeof(int);
        o_dst = o_slot + (size_t)CH * sizeof(int);
        o_ent = o_dst + (size_t)CH * sizeof(int);
        o_head = o_ent + 2 * (size_t)W * CH * sizeof(int);
        o_step = o_head + kWsHead * sizeof(int);
        buf = (o_step + 3 * (size_t)CH * sizeof(int) + 15) & ~(size_t)15;
    }
    __host__ __device__ size_t total() const { return win + kWsBuffers * buf; }
};

template <typename T, int W, bool UNIT>
__global__ void __launch_bounds__(128) k_owner_split(TriArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ unsigned s_epoch;
    __shared__ int s_abort;
    __shared__ int s_fetched;  // last step whose cross-group values are staged
    __shared__ int s_done;     // last step the compute wave finished
    const int g = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = a.n, CH = a.chunk_rows;
    const int s0 = a.step_ptr[g], s1 = a.step_ptr[g + 1];
    const int c0 = a.chunk_ptr[g], c1 = a.chunk_ptr[g + 1];
    if (tid == 0) {
        s_epoch = __hip_atomic_load(a.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_abort = 0;
        s_fetched = s0 - 1;
        s_done = s0 - 1;
    }
    __syncthreads();
    const unsigned par = s_epoch & 1u;
    T *mbox = static_cast<T *>(a.mbox);
    const size_t half = (size_t)a.nexp * a.mbox_stride;
    T *mrd = mbox + (par ? half : 0);
    const int lo = a.window[2 * g], hi = a.window[2 * g + 1];
    const WsLayout<T, W> L(hi - lo, CH, UNIT);
    T *xl = reinterpret_cast<T *>(smem);
    auto buf = [&](int q) { return smem + L.win + (size_t)((q - c0) % kWsBuffers) * L.buf; };
    if (a.nexp > 0) {
        T *other = mbox + (par ? 0 : half);
        const size_t e0 = (size_t)a.exp_ptr[g] * a.mbox_stride, e1 = (size_t)a.exp_ptr[g + 1] * a.mbox_stride;
        for (size_t i = e0 + tid; i < e1; i += blockDim.x) other[i] = sentinel<T>();
    }
    for (int t = tid; t < hi - lo; t += blockDim.x) {
        const size_t src = (size_t)a.gather[lo + t];
        const T b = canon(a.in_f64 ? static_cast<T>(static_cast<const double *>(a.bin)[src])
                                   : static_cast<T>(static_cast<const float *>(a.bin)[src]));
        xl[t] = UNIT ? b : scale_rhs(b, static_cast<const T *>(a.dinv)[lo + t]);
    }
    __syncthreads();
    volatile int *v_fetched = &s_fetched;
    volatile int *v_done = &s_done;
    volatile int *v_abort = &s_abort;
    auto raise = [&]() {
        *v_abort = 1;
        __hip_atomic_store(a.err_dev, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(a.err_host, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    };
    if (wave == 1) {
        // ---------------- fetch wave ----------------
        const T *ev = static_cast<const T *>(a.ell_val);
        int q_next = c0;          // next chunk to load
        int loaded_end = s0;      // steps below this lie in loaded chunks
        int pub = s0 - 1;         // last published step
        int qa = c0;              // chunk holding step pub + 1
        int e_cur = a.rem_ptr[s0];
        unsigned idle = 0;
        while (pub < s1 - 1 && !*v_abort) {
            // keep chunk qa and the next one resident
            while (q_next < c1 && q_next <= qa + 1) {
                if (q_next - c0 >= kWsBuffers) {
                    const int need = a.chunk_step[2 * (q_next - kWsBuffers) + 1] - 1;
                    unsigned spins = 0;
                    while (*v_done < need && !*v_abort) {
                        if (++spins > a.spin) raise();
                        __builtin_amdgcn_s_sleep(1);
                    }
                    if (*v_abort) break;
                }
                unsigned char *B = buf(q_next);
                T *vb = reinterpret_cast<T *>(B + L.o_vals);
                int *cb = reinterpret_cast<int *>(B + L.o_cols);
                int *sb = reinterpret_cast<int *>(B + L.o_slot);
                int *tb = reinterpret_cast<int *>(B + L.o_dst);
                int *eb = reinterpret_cast<int *>(B + L.o_ent);
                int *hb = reinterpret_cast<int *>(B + L.o_head);
                int *pb = reinterpret_cast<int *>(B + L.o_step);
                const int f = a.chunk_step[2 * q_next], e = a.chunk_step[2 * q_next + 1];
                const int r0 = a.step_row[2 * f], r1 = a.step_row[2 * (e - 1) + 1];
                const int x0 = a.rem_ptr[f], x1 = a.rem_ptr[e];
                for (int i = lane; i < r1 - r0; i += 64) {
                    const int row = r0 + i;
#pragma unroll
                    for (int k = 0; k < W; ++k) {
                        cb[k * CH + i] = a.ell_col[(size_t)k * a.ld + row];
                        vb[k * CH + i] = ev[(size_t)k * a.ld + row];
                    }
                    sb[i] = a.exp_slot[row];
                    tb[i] = a.xout ? a.scatter[row] : -1;
                }
                for (int i = lane; i < 2 * (x1 - x0); i += 64) eb[i] = a.rem_ent[2 * x0 + i];
                for (int i = lane; i < e - f; i += 64) {
                    pb[3 * i] = a.step_row[2 * (f + i)];
                    pb[3 * i + 1] = a.step_row[2 * (f + i) + 1];
                    pb[3 * i + 2] = a.rem_ptr[f + i + 1];
                }
                if (lane == 0) {
                    hb[0] = f;
                    hb[1] = e;
                    hb[2] = r0;
                    hb[3] = x0;
                    hb[4] = x1;
                }
                loaded_end = e;
                ++q_next;
            }
            if (*v_abort) break;
            // resident chunks qa and (if loaded) qa + 1
            const int *ha = reinterpret_cast<const int *>(buf(qa) + L.o_head);
            const bool has_b = qa + 1 < q_next;
            const int *hbn = reinterpret_cast<const int *>(buf(qa + 1) + L.o_head);
            const int ent_split = has_b ? hbn[3] : ha[4];
            const int e_lim = has_b ? hbn[4] : ha[4];
            const int e_end = min(e_cur + 64 * kWsPerLane, e_lim);
            int first_pending = e_end;
#pragma unroll
            for (int j = 0; j < kWsPerLane; ++j) {
                const int idx = e_cur + lane + 64 * j;
                if (idx < e_end) {
                    const bool in_b = idx >= ent_split;
                    unsigned char *B = in_b ? buf(qa + 1) : buf(qa);
                    const int li = idx - (in_b ? hbn[3] : ha[3]);
                    const int *eb = reinterpret_cast<const int *>(B + L.o_ent);
                    const int pos = eb[2 * li], slot = eb[2 * li + 1];
                    const T v = __hip_atomic_load(mrd + (size_t)slot * a.mbox_stride, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT);
                    if (is_sentinel(v)) first_pending = min(first_pending, idx);
                    else reinterpret_cast<T *>(B + L.o_stage)[pos] = v;
                }
            }
            for (int off = 32; off > 0; off >>= 1) first_pending = min(first_pending, __shfl_xor(first_pending, off));
            // publish every step whose entries all lie before first_pending
            int np = pub;
            for (;;) {
                const int s = np + 1;
                if (s >= loaded_end) break;
                const int *hs = (s < ha[1]) ? ha : hbn;
                const int *ps = reinterpret_cast<const int *>(reinterpret_cast<const unsigned char *>(hs) - L.o_head +
                                                              L.o_step);
                if (ps[3 * (s - hs[0]) + 2] > first_pending) break;
                np = s;
            }
            e_cur = first_pending;
            if (np > pub) {
                pub = np;
                if (lane == 0) *v_fetched = pub;
                idle = 0;
                while (qa + 1 < q_next && a.chunk_step[2 * qa + 1] <= pub + 1) ++qa;
            } else {
                if (++idle > a.spin) {
                    raise();
                    break;
                }
                if ((idle & 255u) == 0 && __hip_atomic_load(a.err_dev, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                    *v_abort = 1;
                __builtin_amdgcn_s_sleep(1);
            }
        }
    } else {
        // ---------------- compute wave ----------------
        int q = c0;
        const unsigned char *B = buf(q);
        const int *hb = reinterpret_cast<const int *>(B + L.o_head);
        for (int s = s0; s < s1; ++s) {
            const bool tr = a.trace && lane == 0 && (s - s0) < a.trace_stride;
            if (tr) a.trace[2 * ((size_t)g * a.trace_stride + (s - s0))] = __builtin_amdgcn_s_memrealtime();
            unsigned spins = 0;
            while (*v_fetched < s) {
                if (*v_abort) break;
                if (++spins > (a.spin << 4)) {
                    raise();
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
            if (*v_abort) break;
            if (s >= hb[1]) {  // next chunk (its header is valid once step s is published)
                ++q;
                B = buf(q);
                hb = reinterpret_cast<const int *>(B + L.o_head);
            }
            const T *vb = reinterpret_cast<const T *>(B + L.o_vals);
            const T *st = reinterpret_cast<const T *>(B + L.o_stage);
            const int *cb = reinterpret_cast<const int *>(B + L.o_cols);
            const int *sb = reinterpret_cast<const int *>(B + L.o_slot);
            const int *tb = reinterpret_cast<const int *>(B + L.o_dst);
            const int *pb = reinterpret_cast<const int *>(B + L.o_step);
            const int cr0 = hb[2];
            const int js = s - hb[0];
            const int rb = pb[3 * js], re = pb[3 * js + 1];
            for (int x = rb + lane; x < re; x += 64) {
                const int i = x - cr0;
                T sv = xl[x - lo];
#pragma unroll
                for (int k = 0; k < W; ++k) {
                    const int c = cb[k * CH + i];
                    if (c != n) sv -= vb[k * CH + i] * (c > n ? st[i * W + k] : xl[c - lo]);
                }
                xl[x - lo] = sv;
                if (a.write_xw) static_cast<T *>(a.xw)[x] = sv;
                const int slot = sb[i];
                if (slot >= 0)
                    __hip_atomic_store(mrd + (size_t)slot * a.mbox_stride, sv, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
                const int dst = tb[i];
                if (dst >= 0) {
                    if (a.out_f64) static_cast<double *>(a.xout)[dst] = static_cast<double>(sv);
                    else static_cast<float *>(a.xout)[dst] = static_cast<float>(sv);
                }
            }
            if (tr) a.trace[2 * ((size_t)g * a.trace_stride + (s - s0)) + 1] = __builtin_amdgcn_s_memrealtime();
            if (lane == 0) *v_done = s;
        }
    }
    __syncthreads();
    if (tid == 0) {
        const unsigned done = __hip_atomic_fetch_add(&a.epoch[1], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        if (done == gridDim.x - 1) {
            __hip_atomic_store(&a.epoch[1], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&a.epoch[0], s_epoch + 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

template <typename T>
OwnerKernel split_kernel(int w, bool unit, size_t &lds, int rows, int CH)
{
    switch (w) {
#define HEC_SPLIT_CASE(WW)                                                                              \
    case WW:                                                                                            \
        lds = WsLayout<T, WW>(rows, CH, unit).total();                                                  \
        return unit ? k_owner_split<T, WW, true> : k_owner_split<T, WW, false>;
        HEC_SPLIT_CASE(1)
        HEC_SPLIT_CASE(2)
        HEC_SPLIT_CASE(3)
        HEC_SPLIT_CASE(4)
        HEC_SPLIT_CASE(5)
        HEC_SPLIT_CASE(6)
#undef HEC_SPLIT_CASE
    default: return nullptr;
    }
}

// Address of a dword of a packed row (RowRecord::first and stride).
__device__ __forceinline__ const unsigned char *rec_dword(const TriArgs &a, const unsigned char *p, int x, int dw)
{
    if (dw < 4 * a.rec_chunks) return p + ((size_t)(dw / 4) * a.ld + x) * 16 + 4 * (dw % 4);
    return p + (size_t)a.rec_chunks * a.ld * 16 + ((size_t)x * a.rec_rest + (dw - 4 * a.rec_chunks)) * 4;
}

// Barrier-free solve of a level-ordered plan through global memory, for
// solutions too large for LDS (the alternative to one launch per level).  The
// (row, rhs) items in level order are cut into chunks of 64, dealt
// round-robin to the wavefronts of the grid.  A chunk depends only on earlier
// chunks, and the earliest unfinished chunk belongs to a wavefront that has
// finished all its earlier ones, so the solve progresses when every
// wavefront is resident: the kernel is launched cooperatively, so that the
// runtime either makes the whole grid co-resident or refuses the launch.
// (Taking chunks from one shared counter instead needs no co-residency, but
// the counter serializes: with batches of 8 chunks per claim, 288K claims on
// one address made an application of the batched 256-system workload 3.7x
// slower.)  xw starts as the sentinel; an item reads its inputs with
// agent-scope loads and, once none holds the sentinel, computes exactly as
// solve_item does and publishes its value with an agent-scope store.  Lanes
// whose inputs are ready finish inside the wait loop, so a wavefront never
// waits on one of its own lanes.
// MAXW > 0: rows of at most MAXW ELL slots keep their columns and values in
// registers, loaded once, and every poll issues all input loads together (one
// memory round trip per poll); MAXW = 0: any width, columns re-read per poll.
// Packed rows (plans of the system queue that run here with few right-hand
// sides; at most 8 slots) are taken in level order through `order`.
template <typename T, typename TIn, typename TOut, int MAXW>
__global__ void __launch_bounds__(256) k_syncfree(TriArgs a, int waves)
{
    const int lane = threadIdx.x & 63;
    const int wave = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const long items = (long)a.n * a.R;
    const long nch = (items + 63) >> 6;
    const T *ev = static_cast<const T *>(a.ell_val);
    T *xw = static_cast<T *>(a.xw);
    constexpr int NW = MAXW > 0 ? MAXW : 1;
    for (long ch = wave; ch < nch; ch += waves) {
        const long t = (ch << 6) + lane;
        bool todo = t < items;
        const int row = todo ? (int)(t / a.R) : 0;
        const int k = todo ? (int)(t - (long)row * a.R) : 0;
        const int x = a.order ? a.order[row] : row;
        // a finished problem's rows are skipped: they feed only that problem
        if (todo && a.act && !a.act[(a.seg ? a.seg[x] : 0) * a.R + k]) todo = false;
        T b = T(0);
        if (todo) {
            b = canon(static_cast<T>(static_cast<const TIn *>(a.bin)[(size_t)a.gather[x] * a.R + k]));
            if (a.dinv) b = scale_rhs(b, static_cast<const T *>(a.dinv)[x]);
        }
        int cr[NW];
        T vr[NW];
        if (MAXW > 0) {
#pragma unroll
            for (int e = 0; e < NW; ++e) {
                cr[e] = e < a.w ? a.ell_col[(size_t)e * a.ld + x] : a.n;
                const T *v = ev + (size_t)e * a.ld + x;
                if (a.rec_chunks >= 0)
                    v = reinterpret_cast<const T *>(
                        rec_dword(a, static_cast<const unsigned char *>(a.ell_val), x, e * (int)(sizeof(T) / 4)));
                vr[e] = e < a.w ? *v : T(0);
            }
        }
        unsigned spins = 0;
        while (__ballot(todo)) {
            if (todo) {
                T s = b;
                bool ready = true;
                if (MAXW > 0) {
                    T dv[NW];
#pragma unroll
                    for (int e = 0; e < NW; ++e)
                        dv[e] = cr[e] != a.n ? __hip_atomic_load(xw + (size_t)cr[e] * a.R + k, __ATOMIC_RELAXED,
                                                                 __HIP_MEMORY_SCOPE_AGENT)
                                             : T(0);
                    __builtin_amdgcn_sched_barrier(0);  // all loads out before the first test
#pragma unroll
                    for (int e = 0; e < NW; ++e)
                        if (cr[e] != a.n && is_sentinel(dv[e])) ready = false;
                    if (ready) {
#pragma unroll
                        for (int e = 0; e < NW; ++e)
                            if (cr[e] != a.n) s -= vr[e] * dv[e];
                    }
                } else {
                    for (int e = 0; e < a.w && ready; ++e) {
                        const int c = a.ell_col[(size_t)e * a.ld + x];
                        if (c != a.n) {
                            const T v = __hip_atomic_load(xw + (size_t)c * a.R + k, __ATOMIC_RELAXED,
                                                          __HIP_MEMORY_SCOPE_AGENT);
                            if (is_sentinel(v)) ready = false;
                            else s -= ev[(size_t)e * a.ld + x] * v;
                        }
                    }
                }
                if (ready && a.tail_ptr) {
                    const T *tv = static_cast<const T *>(a.tail_val);
                    for (int p = a.tail_ptr[x]; p < a.tail_ptr[x + 1] && ready; ++p) {
                        const T v = __hip_atomic_load(xw + (size_t)a.tail_col[p] * a.R + k, __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_AGENT);
                        if (is_sentinel(v)) ready = false;
                        else s -= tv[p] * v;
                    }
                }
                if (ready) {
                    __hip_atomic_store(xw + (size_t)x * a.R + k, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (a.xout) {
                        const int d = a.scatter[x];
                        if (d >= 0) static_cast<TOut *>(a.xout)[(size_t)d * a.R + k] = static_cast<TOut>(s);
                    }
                    todo = false;
                }
            }
            if (__ballot(todo)) {
                __builtin_amdgcn_s_sleep(1);
                if ((++spins & 255u) == 0 &&
                    (spins > a.spin ||
                     __hip_atomic_load(a.err_dev, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)) {
                    __hip_atomic_store(a.err_dev, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(a.err_host, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                    return;
                }
            }
        }
    }
}

// System queue: every workgroup takes whole independent systems from a
// counter (largest first) and solves one system's levels in order, all of a
// level's (row, rhs) items spread over the workgroup, with a workgroup
// barrier between levels.  The values of the system's last levels stay in an
// LDS ring (slot = local level mod slots); a dependency further back is read
// from the workspace, which this workgroup wrote before an earlier barrier.
// A system is never shared between workgroups, so the solve needs no
// co-residency.  Rows are computed exactly as in k_level (ELL slots in order,
// then the CSR tail; ELL padding reads a zero row of the ring and subtracts
// 0 * 0), so results are bit-identical to it.
// With several right-hand sides an item of the queue is a system and a group
// of at most a.R of its columns (see k_sysq_pipe).
// PACKED: rows as records (vectors beyond the pipelined kernel's offsets); a
// test of it per entry instead took 2 to 4% more.
template <typename T, typename TIn, typename TOut, bool PACKED>
__global__ void __launch_bounds__(1024) k_sysq(TriArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int s_q;
    __shared__ unsigned s_epoch;
    T *ring = reinterpret_cast<T *>(smem);
    const int tid = threadIdx.x, nt = blockDim.x;
    const long ldr = a.ldr;
    const T *ev = static_cast<const T *>(a.ell_val);
    const T *tv = static_cast<const T *>(a.tail_val);
    T *xw = static_cast<T *>(a.xw);
    if (tid == 0) s_epoch = __hip_atomic_load(a.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (;;) {
        if (tid == 0)
            s_q = (int)__hip_atomic_fetch_add(&a.epoch[2], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        const int item = s_q;
        if (item >= a.nparts * a.cgroups) break;
        const int q = item / a.cgroups, g0 = (item - q * a.cgroups) * a.R, R = min(a.R, a.ldr - g0);
        const int slots = a.sq_ring[2 * q], W = a.sq_ring[2 * q + 1];
        const int zrow = slots * W;
        for (int t = tid; t < R; t += nt) ring[(size_t)zrow * R + t] = T(0);
        __syncthreads();
        const int l0 = a.sq_lvp[q], l1 = a.sq_lvp[q + 1];
        for (int l = l0; l < l1; ++l) {
            const int rb = a.sq_lvrow[l], re = a.sq_lvrow[l + 1];
            const int base = slots ? ((l - l0) % slots) * W : 0;
            const int items = (re - rb) * R;
            for (int t = tid; t < items; t += nt) {
                const int i = t / R, k = t - i * R;
                const int x = rb + i;
                T sv = canon(static_cast<T>(static_cast<const TIn *>(a.bin)[(size_t)a.gather[x] * ldr + g0 + k]));
                if (a.dinv) sv = scale_rhs(sv, static_cast<const T *>(a.dinv)[x]);
                for (int e = 0; e < a.w; ++e) {
                    int c;
                    T v;
                    if constexpr (PACKED) {
                        const unsigned char *p = static_cast<const unsigned char *>(a.ell_val);
                        v = *reinterpret_cast<const T *>(rec_dword(a, p, x, e * (int)(sizeof(T) / 4)));
                        c = reinterpret_cast<const uint16_t *>(rec_dword(a, p, x, a.w * (int)(sizeof(T) / 4) + e / 2))[e & 1];
                        if (c > (int)kSysqFar - a.sq_fars) c = -2 - a.sq_far[(size_t)a.sq_fars * x + ((int)kSysqFar - c)];
                    } else {
                        c = a.ell_col[(size_t)e * a.ld + x];
                        v = ev[(size_t)e * a.ld + x];
                    }
                    const T dep = c >= 0 ? ring[(size_t)min(c, zrow) * R + k]
                                         : __hip_atomic_load(xw + (size_t)(-2 - c) * ldr + g0 + k, __ATOMIC_RELAXED,
                                                             __HIP_MEMORY_SCOPE_WORKGROUP);
                    sv -= v * dep;
                }
                if (a.tail_ptr) {
                    for (int p = a.tail_ptr[x]; p < a.tail_ptr[x + 1]; ++p) {
                        const int c = a.tail_col[p];
                        const T dep = c >= 0 ? ring[(size_t)min(c, zrow) * R + k]
                                             : __hip_atomic_load(xw + (size_t)(-2 - c) * ldr + g0 + k, __ATOMIC_RELAXED,
                                                                 __HIP_MEMORY_SCOPE_WORKGROUP);
                        sv -= tv[p] * dep;
                    }
                }
                if (slots) ring[(size_t)(base + i) * R + k] = sv;
                if (a.write_xw)
                    __hip_atomic_store(xw + (size_t)x * ldr + g0 + k, sv, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                if (a.xout) {
                    const int d = a.scatter[x];
                    if (d >= 0) static_cast<TOut *>(a.xout)[(size_t)d * ldr + g0 + k] = static_cast<TOut>(sv);
                }
            }
            __syncthreads();
        }
    }
    if (tid == 0) {
        const unsigned done = __hip_atomic_fetch_add(&a.epoch[1], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        if (done == gridDim.x - 1) {
            // last workgroup out: every claim is over; reset the queue
            __hip_atomic_store(&a.epoch[2], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&a.epoch[1], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&a.epoch[0], s_epoch + 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

template <typename T>
__global__ void __launch_bounds__(256) k_fill_sentinel(T *p, size_t count, unsigned *counter)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = sentinel<T>();
    if (counter && i == 0) *counter = 0u;  // the next launch's chunk counter
}

// Columns of one item of the system queue without packed rows: those the rings
// were sized for, or fewer right-hand sides if the call has fewer.
int32_t sysq_columns(const DevTri &d, int32_t R)
{
    const size_t row = (size_t)std::max(1, d.sq_lds_rows) * (d.dt == HEC_F64 ? 8 : 4);
    int32_t c = std::min(R, std::max(d.sq_cols, kSysqColumns));
    while (c > 1 && row * c > (size_t)device_max_lds()) --c;
    return c;
}

bool capturing(hipStream_t st)
{
    hipStreamCaptureStatus s = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &s) != hipSuccess) {
        (void)hipGetLastError();  // another stream's capture forbids the question
        return true;
    }
    return s != hipStreamCaptureStatusNone;
}

// An item of the pipelined kernel: 1 << shift threads to a row, each with one
// or four columns (0: not for it, which needs packed rows and vectors within
// 32-bit buffer offsets).
struct SysqItem {
    int32_t columns = 0, shift = 0;
    bool few = false;  // the barrier-free kernel instead
    int32_t all() const { return columns << shift; }
};

// More columns to an item read a system's rows fewer times and share its chain
// of levels, fewer give more and shorter items.  A call takes about
// cost(item) * max(1, 1.35 * rounds): `rounds` are the items times the average
// system's work over the compute units and the largest system's (two
// workgroups of a compute unit slow each other down, hence 1.35), and the costs
// of items against one of one column are fitted to measurements: four columns
// of a thread, two and four threads to a row.  Both triangles, us, items of one
// column / four columns of a thread / two / four such threads:
//   512 subdomains of 4096 rows, FP32, 16 right-hand sides 1236 / 610 / 396 / 320
//   295 of 2280 rows, FP32, 16                              289 / 166 / 132 / 108
//   295 of 1576 rows, FP64, 16                              416 / 201 / 139 / 143
//   64 of 32768 rows, FP32, 4 and 8                239 / 303 / -, 501 / 353 / 390
//   64 uneven ones of a 128^3 grid, FP32, 4, 8, 16  723 / 1100, 1259 / 1114, 1887 / 1196
//   32 uneven ones of a 100^3 grid, FP64, 16       1116 / 1301
//   256 uneven ILU(1) systems, FP32, 4 and 8        847 / 1176, 1656 / 1222 / 1598
// and two threads of one column: 32 systems of 50000 to 150000 rows, FP32, 16
// right-hand sides 1738 -> 1107 (four columns of a thread 1272).
// One or four columns of one thread alone made many even systems slower than
// items of all their columns had been (512 subdomains, 4 / 8 / 16 right-hand
// sides 319 / 297 / 612 us, in one item each 173 / 225 / 359).
SysqItem sysq_pipe_item(const DevTri &d, int32_t R, hipStream_t st)
{
    SysqItem best;
    if (!d.sysq || !d.sq_packed || ((size_t)d.n + 1) * R * 8 >= kSysqDropped) return best;
    static constexpr double four[2] = {1.6, 1.95}, threads[2][kSysqShifts] = {{1.0, 1.47, 2.16}, {1.0, 1.75, 2.6}};
    const bool f64 = d.dt == HEC_F64;
    double least = 0.0;
    for (int32_t columns : {1, kSysqColumns})
        for (int32_t shift = 0; shift < (d.sq_global ? 1 : kSysqShifts); ++shift) {
            const int32_t all = columns << shift;
            if (columns > 1 && f64 && d.sq_fars == 4) continue;  // not built
            if (R % all != 0 || (size_t)std::max(1, d.sq_lds_rows) * all * (f64 ? 8 : 4) + 32 > (size_t)device_max_lds())
                continue;
            const double cost = (columns == 1 ? 1.0 : four[f64]) * threads[f64][shift];
            const double t = cost * std::max(1.0, 1.35 * d.sq_balance * (R / all) / device_cus());
            if (best.columns == 0 || t < least) {
                least = t;
                best.columns = columns;
                best.shift = shift;
            }
        }
    // A few uneven systems with few columns leave most compute units idle for
    // the largest one's time, which every unit shares on the barrier-free
    // kernel.  Both triangles, us, queue / barrier-free: 32 subdomains of a
    // 100^3 grid, FP64, 1 / 4 / 16 right-hand sides 609 / 522, 757 / 642, 1119 /
    // 1343; 64 of a 128^3 grid, FP32, 1 / 4 690 / 670, 725 / 942; 16 of a 64^3
    // grid, FP32, one 215 / 304.  (That kernel is launched cooperatively, so
    // not into a graph, where the queue stays.)
    best.few = d.sq_order.p && !d.trace && syncfree_us(d.nlev, d.n, R) < sysq_us(d.sq_most, d.sq_global) * least &&
               !capturing(st);
    if (best.few) best.columns = 0;
    return best;
}

SysqKernel sysq_pipe_kernel(const DevTri &d, const TriArgs &a, int32_t columns, int32_t shift)
{
    const bool in = a.in_f64 != 0, f64 = d.dt == HEC_F64;
    const int out = !a.xout ? 0 : (a.out_f64 ? 1 : 2);
    using Select = SysqKernel (*)(int, bool, int, int);
    static constexpr Select one[2][3] = {{sq_f32_x1, sq_f32_d1, sq_f32_f1}, {sq_f64_x1, sq_f64_d1, sq_f64_f1}};
    static constexpr Select four[2][3] = {{sq_f32_x4, sq_f32_d4, sq_f32_f4}, {sq_f64_x4, sq_f64_d4, sq_f64_f4}};
    return (columns == 1 ? one : four)[f64][out](d.w, in, d.sq_rows[shift], shift > 0 ? kSysqShared : d.sq_fars);
}

// Right-hand sides one launch of a dataflow plan holds.
int32_t dataflow_columns(const DevTri &d)
{
    return hec::dataflow_columns(d.df_rows, d.df_ints, d.df_step_rows, d.dt == HEC_F64 ? 8 : 4, (size_t)device_max_lds());
}

// A call's R right-hand sides as even groups of at most `most` columns, and the
// groups of one launch: no more than have a compute unit for each workgroup.
struct DataflowSplit {
    int32_t columns, groups;
    static int32_t even(int32_t R, int32_t most)
    {
        const int32_t all = (R + most - 1) / most;
        return (R + all - 1) / all;
    }
    DataflowSplit(int32_t R, int32_t most, int32_t parts, int32_t cap) : columns(even(R, most))
    {
        groups = std::max(1, std::min((R + columns - 1) / columns, std::min(cap, device_cus()) / std::max(1, parts)));
    }
    // groups of the launch that starts at column k0
    int32_t at(int32_t k0, int32_t R) const { return std::min(groups, (R - k0 + columns - 1) / columns); }
};

// Two import wavefronts, but one beside wide rows (see df_import) or where
// the workgroup has no room for another.
int32_t dataflow_import_waves(const DevTri &d)
{
    return d.w <= 8 && 64 * (d.df_waves + 3) <= dataflow_max_block(d.w) ? 2 : 1;
}

template <typename T> void launch_dataflow(DevTri &d, TriArgs a, hipStream_t st)
{
    // the plan's columns name group-local imports: only this kernel reads them.
    // One launch, or (a plan whose parts hold fewer right-hand sides than one
    // part per compute unit would) groups of columns
    a.ldr = a.R;
    const int32_t all = a.R, most = dataflow_columns(d);
    if (all > most && all > d.df_accept) {
        if ((int64_t)d.df_step_rows * all > 64)
            fail(HEC_ERR_INVALID_ARG, "dataflow plan: nrhs exceeds the plan's max_nrhs (steps are sized for it)");
        fail(HEC_ERR_CAPACITY, "dataflow kernel: LDS need exceeds the device limit at this nrhs");
    }
    a.R = DataflowSplit::even(all, most);
    const bool one = a.R == 1, f64 = sizeof(T) == 8;
    OwnerKernel k = nullptr;
    if (a.trace)
        k = f64 ? (one ? df_f64_one_tr : df_f64_many_tr)(d.w, d.unit, d.has_tail)
                : (one ? df_f32_one_tr : df_f32_many_tr)(d.w, d.unit, d.has_tail);
    else
        k = f64 ? (one ? df_f64_one : df_f64_many)(d.w, d.unit, d.has_tail)
                : (one ? df_f32_one : df_f32_many)(d.w, d.unit, d.has_tail);
    if (!k) fail(HEC_ERR_INVALID_ARG, "internal: dataflow plan with an unsupported ELL width");
    size_t lds = dataflow_lds_bytes(d.df_rows, d.df_ints, a.R, sizeof(T));
    if (a.trace) lds += 16 + 16 * (size_t)std::min(d.df_ints, a.trace_stride);  // per-step clocks
    a.lds_ctl = (int32_t)lds - kDataflowCtlBytes;
    a.imp_waves = dataflow_import_waves(d);
    const int block = 64 * (d.df_waves + 1 + a.imp_waves);
    if (block > dataflow_max_block(d.w)) fail(HEC_ERR_INVALID_ARG, "dataflow kernel: block too large");
    if (lds > (size_t)device_max_lds())
        fail(HEC_ERR_CAPACITY, "dataflow kernel: LDS need exceeds the device limit at this nrhs");
    const int32_t cap = capacity_of((const void *)k, block, lds, true);
    a.nparts = d.groups;
    a.queue = d.queue ? 1 : 0;
    int32_t grid = d.groups;
    if (d.queue) {
        // parts wait only on lower-numbered parts, which running
        // workgroups hold: any grid size makes progress
        grid = std::max(1, std::min(d.groups, cap));
    } else if (cap < d.groups) {
        fail(HEC_ERR_CAPACITY, "dataflow grid exceeds the co-resident capacity");
    }
    const DataflowSplit split(all, most, d.groups, cap);
    for (a.k0 = 0; a.k0 < all; a.k0 += split.groups * split.columns) {
        hipLaunchKernelGGL(k, dim3(grid, split.at(a.k0, all)), dim3(block), lds, st, a);
        hip_check(hipGetLastError(), "k_dataflow launch");
    }
}

template <typename T, typename TIn, typename TOut> void launch_syncfree(DevTri &d, const TriArgs &a, hipStream_t st)
{
    const size_t cnt = ((size_t)d.n + 1) * a.R;
    hipLaunchKernelGGL(k_fill_sentinel<T>, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, st,
                       static_cast<T *>(a.xw), cnt, (unsigned *)nullptr);
    // about one wavefront per chunk of an average level (at least two
    // workgroups per compute unit), within half the occupancy; the
    // cooperative launch guarantees co-residency (it costs tens of
    // microseconds, small beside this kernel's milliseconds)
    const long chunks = ((long)d.n * a.R + 63) / 64;
    // rows of at most 8 (or 16) ELL slots keep them in registers
    const void *kern = d.w <= 8 ? (const void *)k_syncfree<T, TIn, TOut, 8>
                     : (d.w <= 16 ? (const void *)k_syncfree<T, TIn, TOut, 16> : (const void *)k_syncfree<T, TIn, TOut, 0>);
    const int cap = capacity_of(kern, 256, 0);
    const long per_level = chunks / std::max(1, d.nlev);
    const long lim = std::min<long>(std::max(1, cap / 2), std::max<long>(2L * device_cus(), per_level / 4));
    const int grid = (int)std::max<long>(1, std::min<long>(lim, (chunks + 3) / 4));
    int waves = grid * 4;
    void *args[] = {(void *)&a, (void *)&waves};
    hip_check(hipLaunchCooperativeKernel(kern, dim3(grid), dim3(256), args, 0, st), "k_syncfree cooperative launch");
}

template <typename T, typename TIn, typename TOut>
void launch_typed(DevTri &d, TriArgs a, hipStream_t st)
{
    if (d.n == 0) return;
    if (d.kind == HEC_SCHED_LEVEL_LAUNCH && d.variant == 5) {
        launch_syncfree<T, TIn, TOut>(d, a, st);
        return;
    }
    if (d.sysq) {
        if ((size_t)d.sq_full_rows * a.R * sizeof(T) > (size_t)device_max_lds())
            fail(HEC_ERR_CAPACITY, "system queue: the LDS ring exceeds the device limit at this nrhs");
        a.nparts = d.groups;
        a.ldr = a.R;
        const SysqItem piped = sysq_pipe_item(d, a.ldr, st);
        if (piped.few) {
            a.order = d.sq_order.as<int32_t>();
            launch_syncfree<T, TIn, TOut>(d, a, st);
            return;
        }
        a.R = piped.columns ? piped.columns : sysq_columns(d, a.ldr);
        a.cshift = piped.shift;
        a.cgroups = piped.columns ? a.ldr / piped.all() : (a.ldr + a.R - 1) / a.R;
        const int items = d.groups * a.cgroups;
        const size_t lds = ((size_t)std::max(1, d.sq_lds_rows) * a.R << a.cshift) * sizeof(T);
        if (piped.columns) {
            const SysqKernel k = sysq_pipe_kernel(d, a, piped.columns, piped.shift);
            if (!k) fail(HEC_ERR_INVALID_ARG, "internal: system queue with an unsupported record width");
            const size_t all = ((lds + 15) & ~(size_t)15) + 16;
            a.lds_ctl = (int32_t)all - 16;
            const int32_t cap = capacity_of((const void *)k, kSysqThreads, all, true);
            const int grid = std::max(1, std::min(items, cap));
            hipLaunchKernelGGL(k, dim3(grid), dim3(kSysqThreads), all, st, a, d.sq_pcp[a.cshift].as<int32_t>(),
                               d.sq_pc[a.cshift].as<int4>(), a.sq_ring);
            hip_check(hipGetLastError(), "k_sysq_pipe launch");
            return;
        }
        const int block = std::max(64, std::min(1024, d.block));
        auto k = d.sq_packed ? k_sysq<T, TIn, TOut, true> : k_sysq<T, TIn, TOut, false>;
        const int32_t cap = capacity_of((const void *)k, block, lds);
        if (d.sq_global) a.write_xw = 1;  // dependencies beyond the ring are read back from xw
        const int grid = std::max(1, std::min(items, cap));
        hipLaunchKernelGGL(k, dim3(grid), dim3(block), lds, st, a);
        hip_check(hipGetLastError(), "k_sysq launch");
        return;
    }
    if (d.kind == HEC_SCHED_LEVEL_LAUNCH) {
        for (int32_t k = 0; k < d.nlev; ++k) {
            a.row_begin = d.levelptr[k];
            a.row_end = d.levelptr[k + 1];
            const int items = (a.row_end - a.row_begin) * a.R;
            const int grid = (items + 255) / 256;
            hipLaunchKernelGGL((k_level<T, TIn, TOut>), dim3(grid), dim3(256), 0, st, a);
        }
        hip_check(hipGetLastError(), "k_level launch");
        return;
    }
    if (d.dataflow) {
        launch_dataflow<T>(d, a, st);
        return;
    }
    if (d.kind == HEC_SCHED_OWNER_PERSISTENT && d.variant == 3 && a.R == 1 && !d.has_tail && d.max_lanes_one &&
        d.w >= 1 && d.w <= 6 && d.chunk_rows > 0) {
        size_t lds = 0;
        OwnerKernel k = split_kernel<T>(d.w, d.unit, lds, d.max_window, d.chunk_rows);
        if (k && lds <= (size_t)device_max_lds() && capacity_of((const void *)k, 128, lds) >= d.groups) {
            hipLaunchKernelGGL(k, dim3(d.groups), dim3(128), lds, st, a);
            hip_check(hipGetLastError(), "k_owner_split launch");
            return;
        }
    }
    if (d.kind == HEC_SCHED_OWNER_PERSISTENT && (d.variant == 0 || d.variant >= 2) && !d.has_tail &&
        d.max_lanes_one && d.w >= 1 && d.w <= 8 && d.chunk_rows > 0 && d.chunk_rows % d.block == 0) {
        const int rpt = d.chunk_rows / d.block;
        OwnerKernel k = owner_kernel<T>(d.w, rpt, d.unit);
        const size_t lds = owner_lds_bytes(d.max_window, a.R, d.w, d.chunk_rows, d.unit, sizeof(T));
        if (k && lds <= (size_t)device_max_lds() && capacity_of((const void *)k, d.block, lds) >= d.groups) {
            hipLaunchKernelGGL(k, dim3(d.groups), dim3(d.block), lds, st, a);
            hip_check(hipGetLastError(), "k_owner launch");
            return;
        }
    }
    size_t lds = 0;
    bool use_lds = false;
    auto k_lds = k_persistent<T, TIn, TOut, true>;
    auto k_glb = k_persistent<T, TIn, TOut, false>;
    if (d.kind == HEC_SCHED_OWNER_PERSISTENT && d.max_window > 0) {
        lds = (size_t)d.max_window * a.R * sizeof(T);
        use_lds = lds <= (size_t)device_max_lds() && capacity_of((const void *)k_lds, d.block, lds) >= d.groups;
        if (!use_lds) lds = 0;
    }
    if (!use_lds && capacity_of((const void *)k_glb, d.block, 0) < d.groups)
        fail(HEC_ERR_CAPACITY, "persistent grid exceeds the co-resident capacity");
    if (use_lds)
        hipLaunchKernelGGL(k_lds, dim3(d.groups), dim3(d.block), lds, st, a);
    else
        hipLaunchKernelGGL(k_glb, dim3(d.groups), dim3(d.block), 0, st, a);
    hip_check(hipGetLastError(), "k_persistent launch");
}

template <typename T>
void launch_in(DevTri &d, const TriArgs &a, hec_dtype_t in_dt, hec_dtype_t out_dt, hipStream_t st)
{
    if (in_dt == HEC_F64) {
        if (out_dt == HEC_F64) launch_typed<T, double, double>(d, a, st);
        else launch_typed<T, double, float>(d, a, st);
    } else {
        if (out_dt == HEC_F64) launch_typed<T, float, double>(d, a, st);
        else launch_typed<T, float, float>(d, a, st);
    }
}

// Co-resident workgroups of one kernel instance on the current device
// (cached: the occupancy query and the LDS attribute are set once per
// kernel, block size, LDS size and device).  lds_at_zero: the kernel takes its
// dynamic LDS to start at LDS address 0, so it must have no static LDS.
int32_t capacity_of(const void *kern, int32_t block, size_t lds, bool lds_at_zero)
{
    struct Key {
        const void *k;
        int32_t block;
        size_t lds;
        int dev;
        bool operator<(const Key &o) const
        {
            return std::tie(k, block, lds, dev) < std::tie(o.k, o.block, o.lds, o.dev);
        }
    };
    static std::mutex mu;
    static std::map<Key, int32_t> cache;
    int dev = 0;
    hip_check(hipGetDevice(&dev), "hipGetDevice");
    const Key key{kern, block, lds, dev};
    {
        std::lock_guard<std::mutex> g(mu);
        auto it = cache.find(key);
        if (it != cache.end()) return it->second;
    }
    if (lds_at_zero) {
        hipFuncAttributes fa{};
        hip_check(hipFuncGetAttributes(&fa, kern), "hipFuncGetAttributes");
        if (fa.sharedSizeBytes != 0) fail(HEC_ERR_HIP, "internal: a kernel addressing LDS from 0 has static LDS");
    }
    int cus = 0, per = 0;
    hip_check(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev), "attr CUs");
    if (lds > 0)
        hip_check(hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds),
                  "hipFuncSetAttribute");
    hip_check(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kern, block, lds), "occupancy");
    std::lock_guard<std::mutex> g(mu);
    cache[key] = per * cus;
    return per * cus;
}

template <typename T, bool LDS>
int32_t capacity_all(int32_t block, size_t lds)
{
    int32_t c = capacity_of((const void *)k_persistent<T, double, double, LDS>, block, lds);
    c = std::min(c, capacity_of((const void *)k_persistent<T, double, float, LDS>, block, lds));
    c = std::min(c, capacity_of((const void *)k_persistent<T, float, double, LDS>, block, lds));
    c = std::min(c, capacity_of((const void *)k_persistent<T, float, float, LDS>, block, lds));
    return c;
}

}  // namespace

int32_t persistent_capacity(hec_dtype_t dt, int32_t block, size_t lds)
{
    if (dt == HEC_F64) return lds ? capacity_all<double, true>(block, lds) : capacity_all<double, false>(block, 0);
    return lds ? capacity_all<float, true>(block, lds) : capacity_all<float, false>(block, 0);
}

namespace {
int32_t device_attr(hipDeviceAttribute_t attr)
{
    static std::mutex mu;
    static std::map<std::pair<int, int>, int32_t> cache;
    int dev = 0;
    hip_check(hipGetDevice(&dev), "hipGetDevice");
    std::lock_guard<std::mutex> g(mu);
    auto key = std::make_pair(dev, (int)attr);
    auto it = cache.find(key);
    if (it != cache.end()) return it->second;
    int v = 0;
    hip_check(hipDeviceGetAttribute(&v, attr, dev), "hipDeviceGetAttribute");
    cache[key] = v;
    return v;
}
}  // namespace

int32_t device_cus() { return device_attr(hipDeviceAttributeMultiprocessorCount); }

int32_t device_max_lds() { return device_attr(hipDeviceAttributeMaxSharedMemoryPerBlock); }

void fill_sentinel(void *p, size_t count, hec_dtype_t dt)
{
    if (count == 0) return;
    const unsigned grid = (unsigned)((count + 255) / 256);
    if (dt == HEC_F64)
        hipLaunchKernelGGL(k_fill_sentinel<double>, dim3(grid), dim3(256), 0, 0, static_cast<double *>(p), count,
                           nullptr);
    else
        hipLaunchKernelGGL(k_fill_sentinel<float>, dim3(grid), dim3(256), 0, 0, static_cast<float *>(p), count,
                           nullptr);
    hip_check(hipGetLastError(), "k_fill_sentinel launch");
    hip_check(hipDeviceSynchronize(), "hipDeviceSynchronize");
}

namespace {

TriArgs tri_args(const DevTri &d, const void *bin, hec_dtype_t in_dt, const int32_t *gather, void *xw, void *xout,
                 hec_dtype_t out_dt, const int32_t *scatter, int32_t R)
{
    if (R > d.ws_R) fail(HEC_ERR_INVALID_ARG, "internal: workspace narrower than nrhs");
    TriArgs a{};
    a.n = d.n;
    a.w = d.w;
    a.ld = d.ld;
    a.R = R;
    a.ell_col = d.ell_col.as<int32_t>();
    a.ell_val = d.ell_val.p;
    a.tail_ptr = d.has_tail ? d.tail_ptr.as<int32_t>() : nullptr;
    a.tail_col = d.tail_col.as<int32_t>();
    a.tail_val = d.tail_val.p;
    a.dinv = d.unit ? nullptr : d.dinv.p;
    a.step_ptr = d.step_ptr.as<int32_t>();
    a.step_row = d.step_row.as<int32_t>();
    a.step_lanes = d.step_lanes.as<int32_t>();
    a.window = d.window.as<int32_t>();
    a.exp_slot = d.exp_slot.as<int32_t>();
    a.exp_ptr = d.exp_ptr.as<int32_t>();
    a.mbox = d.mbox.p;
    a.nexp = d.nexp;
    a.mbox_stride = d.ws_R;
    a.epoch = d.epoch.as<unsigned int>();
    a.err_dev = d.err.as<int>();
    a.err_host = d.err_host;
    a.bin = bin;
    a.gather = gather;
    a.xw = xw;
    a.xout = xout;
    a.scatter = scatter;
    a.write_xw = xout ? 0 : 1;
    a.chunk_ptr = d.chunk_ptr.as<int32_t>();
    a.rem_ptr = d.rem_ptr.as<int32_t>();
    a.rem_ent = d.rem_ent.as<int32_t>();
    a.chunk_step = d.chunk_step.as<int32_t>();
    a.chunk_rows = d.chunk_rows;
    a.imp_ptr = d.imp_ptr.as<int32_t>();
    a.imp_slot = d.imp_slot.as<int32_t>();
    a.exp_row = d.exp_row.as<int32_t>();
    a.wave_ptr = d.wave_ptr.as<int32_t>();
    a.step_pack = d.step_pack.as<int32_t>();
    a.act = d.act;
    a.seg = d.seg.p ? d.seg.as<int32_t>() : nullptr;
    a.trace = d.trace;
    a.trace_stride = d.trace_stride;
    a.spin = d.spin;
    a.sq_lvp = d.sq_lvp.as<int32_t>();
    a.sq_lvrow = d.sq_lvrow.as<int32_t>();
    a.sq_ring = d.sq_ring.as<int32_t>();
    a.sq_keep = d.sq_keep.as<int8_t>();
    a.sq_far = d.sq_far.as<int32_t>();
    a.sq_fars = d.sq_fars;
    a.rec_chunks = -1;
    if (d.sysq && d.sq_packed) {
        const RowRecord rec(d.w, d.ld, d.dt == HEC_F64 ? 8 : 4);
        a.rec_chunks = rec.chunks;
        a.rec_rest = rec.rest;
    }
    a.in_f64 = in_dt == HEC_F64 ? 1 : 0;
    a.out_f64 = out_dt == HEC_F64 ? 1 : 0;
    return a;
}

void launch_any(DevTri &d, const TriArgs &a, hec_dtype_t in_dt, hec_dtype_t out_dt, hipStream_t st)
{
    if (d.dt == HEC_F64) launch_in<double>(d, a, in_dt, out_dt, st);
    else launch_in<float>(d, a, in_dt, out_dt, st);
}

}  // namespace

void launch_tri(DevTri &d, const void *bin, hec_dtype_t in_dt, const int32_t *gather, void *xw, void *xout,
                hec_dtype_t out_dt, const int32_t *scatter, int32_t R, hipStream_t st)
{
    launch_any(d, tri_args(d, bin, in_dt, gather, xw, xout, out_dt, scatter, R), in_dt, out_dt, st);
}

void launch_lu(DevTri &L, DevTri &U, bool lu_shared, const void *r, hec_dtype_t in_dt, const int32_t *gather_l, void *y,
               const int32_t *qmap, void *uw, void *z, hec_dtype_t out_dt, const int32_t *scatter_u, int32_t R,
               hipStream_t st)
{
    const int32_t most = lu_shared ? std::min(dataflow_columns(L), dataflow_columns(U)) : 0;
    if (lu_shared && L.n > 0 && !L.trace && !U.trace && (R <= most || (R <= L.df_accept && R <= U.df_accept))) {
        const bool f64 = L.dt == HEC_F64;
        TriArgs a = tri_args(L, r, in_dt, gather_l, nullptr, nullptr, in_dt, nullptr, R);
        TriArgs b = tri_args(U, nullptr, L.dt, qmap, nullptr, z, out_dt, scatter_u, R);
        a.ldr = b.ldr = R;
        a.R = b.R = DataflowSplit::even(R, most);
        LuKernel k = a.R == 1 ? (f64 ? lu_f64_one : lu_f32_one)(L.w) : (f64 ? lu_f64_many : lu_f32_many)(L.w);
        const size_t ts = f64 ? 8 : 4;
        const size_t lds = std::max(dataflow_lds_bytes(L.df_rows, L.df_ints, a.R, ts),
                                    dataflow_lds_bytes(U.df_rows, U.df_ints, a.R, ts));
        a.lds_ctl = b.lds_ctl = (int32_t)lds - kDataflowCtlBytes;
        a.imp_waves = b.imp_waves = dataflow_import_waves(L);
        const int block = 64 * (L.df_waves + 1 + a.imp_waves);
        const int32_t cap = capacity_of((const void *)k, block, lds, true);
        if (cap < L.groups) fail(HEC_ERR_CAPACITY, "dataflow grid exceeds the co-resident capacity");
        const DataflowSplit split(R, most, L.groups, cap);
        for (int32_t k0 = 0; k0 < R; k0 += split.groups * split.columns) {
            a.k0 = b.k0 = k0;
            hipLaunchKernelGGL(k, dim3(L.groups, split.at(k0, R)), dim3(block), lds, st, a, b);
            hip_check(hipGetLastError(), "k_dataflow_lu launch");
        }
        return;
    }
    // two system queues: y is stored group of columns by group of columns, so
    // that an item writes and reads whole cache lines of it
    const bool grouped = L.dt == U.dt && sysq_pipe_item(L, R, st).columns > 0 &&
                         sysq_pipe_item(L, R, st).columns == sysq_pipe_item(U, R, st).columns;
    TriArgs a = tri_args(L, r, in_dt, gather_l, y, nullptr, in_dt, nullptr, R);
    TriArgs b = tri_args(U, y, L.dt, qmap, uw, z, out_dt, scatter_u, R);
    a.xw_grouped = b.bin_grouped = grouped ? 1 : 0;
    launch_any(L, a, in_dt, in_dt, st);
    launch_any(U, b, L.dt, out_dt, st);
}

}  // namespace hec

// Dataflow owner kernel: one launch per triangle, no per-level barrier.
//
// A workgroup owns a part of the rows (a contiguous device-row window) and
// runs three kinds of wavefronts:
//   compute waves  walk their own contiguous pieces of the part in level
//                  order, a step (at most 64 (row, rhs) items of one level)
//                  at a time, one item per lane.  Each dependency is read
//                  from LDS and re-read until it no longer holds the
//                  sentinel, so a row starts as soon as its own inputs exist.
//                  Compute waves issue no global stores, so their waits cover
//                  loads only.
//   import waves   poll the mailbox slots this group reads, in order of first
//                  use, and copy each value into LDS when it arrives;
//   export wave    watches the group's exported rows in LDS and writes each
//                  one to its mailbox slot as soon as it is solved.
// Any row waits only on rows of lower levels, and every wave handles its
// items in level order, so the row of lowest level not yet solved can always
// proceed: the grid drains as long as all workgroups are co-resident.
// Right-hand sides beyond what a part's LDS and wavefronts hold are groups of
// columns, each solved by its own workgroups (grid y) beside the others: they
// share nothing but the mailbox, where every column has its place.  One launch
// per group instead: 32^3 ILU(0) with 16 right-hand sides, planned for one,
// 737 us; one part per compute unit in their place 209 us.
// The summation order (ELL slots, then the CSR tail, on a right-hand side
// scaled by the reciprocal diagonal) is the one of k_level, so results are
// bit-identical to it.
//
// What bounds it: the chain of levels.  A step is LDS write -> LDS read ->
// multiply-adds -> test (measured on one wavefront: 96 cycles for write, three
// reads and three FP64 multiply-adds, 20 more for the test), and a wavefront
// alone on its SIMD issues an instruction every 4-5 cycles, so every
// instruction of a step costs time although the unit it uses is idle.  Hence
// a row is one packed record (2 loads instead of 6 for three FP64 entries),
// LDS addresses start at 0 and are formed by one multiply-add from 16-bit
// columns before they are needed, a step's descriptor is a broadcast LDS read
// (decoding it with v_readlane and scalar instructions cost 40 cycles a step)
// and the polling code is out of line.  Against one 32-bit column and one
// value load per entry with the columns converted after the previous step:
// 64^2 ILU(0) 115.6 -> 106.2 us per L+U, 128^3 331.7 -> 309.8 us (FP64,
// three factors in turn), 100^3 ILUT(1e-3, 10) FP32 1910 -> 1395 us.
#pragma once

#include "row_record.h"

namespace hec {

template <typename T> __device__ __forceinline__ T lds_get(const T *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
template <typename T> __device__ __forceinline__ void lds_put(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Register sets in rotation: as many as the vector-memory counter (63
// outstanding loads) and about 144 registers hold, at most 8 (4 sets made
// 128^3 ILU(0) 6% slower, 6 to 16 were equal, and 16 made ILU(1) with four
// right-hand sides 12% slower than 8).
template <typename T, int W> constexpr int df_sets()
{
    using Rec = RowRec<T, W>;
    constexpr int byreg = 144 / Rec::ND < 3 ? 3 : 144 / Rec::ND, bycnt = 60 / Rec::LOADS + 1;
    constexpr int k = byreg < bycnt ? byreg : bycnt, sets = k < 8 ? k : 8;
    static_assert(sets <= kDataflowPad, "descriptors are read that many steps ahead");
    return sets;
}

// A workgroup's part of one triangle, its columns (R from k0) and its place in LDS: x [win][R], b
// [win][R], imports [nimp][R], one zero row (the target of ELL padding), then
// import slots, export rows (window offsets) and step descriptors (first
// window row | 16 (number of rows - 1) << 16) with kDataflowPad zeros behind.
template <typename T> struct DfPart {
    int g, lo, win, i0, nimp, e0, nex, s0, ns, k0;
    T *xl, *bl, *im;
    int *isl, *erl, *stl;
    unsigned long long *ltr;
};

template <typename T> __device__ __forceinline__ DfPart<T> df_part(const TriArgs &a, int g, int k0, int R, unsigned char *smem)
{
    // uniform values as scalars: behind a store the compiler reads them with
    // vector loads, and a buffer load whose offset it cannot prove uniform
    // becomes a loop over the lanes
    auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    DfPart<T> p;
    p.g = uni(g);
    p.k0 = k0;
    p.lo = uni(a.window[2 * g]);
    p.win = uni(a.window[2 * g + 1]) - p.lo;
    p.i0 = uni(a.imp_ptr[g]);
    p.nimp = uni(a.imp_ptr[g + 1]) - p.i0;
    p.e0 = uni(a.exp_ptr[g]);
    p.nex = uni(a.exp_ptr[g + 1]) - p.e0;
    p.s0 = uni(a.step_ptr[g]);
    p.ns = uni(a.step_ptr[g + 1]) - p.s0;
    p.xl = reinterpret_cast<T *>(smem);
    p.bl = p.xl + (size_t)p.win * R;
    p.im = p.bl + (size_t)p.win * R;
    const size_t ib = (((size_t)2 * p.win + p.nimp + 1) * R * sizeof(T) + 15) & ~(size_t)15;
    p.isl = reinterpret_cast<int *>(smem + ib);
    p.erl = p.isl + p.nimp;
    p.stl = p.erl + p.nex;
    // when tracing: 2*ns clocks after the ints, at an 8-byte boundary
    p.ltr = reinterpret_cast<unsigned long long *>(smem + ((ib + (size_t)(p.nimp + p.nex + p.ns + kDataflowPad) * 4 + 7) & ~(size_t)7));
    return p;
}

// LDS words all wavefronts share, behind everything else (the value area
// starts at LDS address 0, so that a value's address is its row times a
// constant).
struct DfCtl {
    unsigned epoch;
    int abort, part;
    unsigned epoch2;  // of the second triangle
};

constexpr int kDfFill = 8;  // independent loads a thread keeps in flight while LDS is filled

__device__ __forceinline__ void df_copy_ints(int *dst, const int32_t *src, int count, int add)
{
    const int nt = blockDim.x;
    for (int t0 = threadIdx.x; t0 < count; t0 += kDfFill * nt) {
        int v[kDfFill];
#pragma unroll
        for (int u = 0; u < kDfFill; ++u) v[u] = src[min(t0 + u * nt, count - 1)];
#pragma unroll
        for (int u = 0; u < kDfFill; ++u)
            if (t0 + u * nt < count) dst[t0 + u * nt] = v[u] + add;
    }
}

// Empty slots of the mailbox half the next launch reads: those of this
// workgroup's part (those that other workgroups had emptied took longer to
// arrive: 20011 irregular rows 228 -> 230 us), by the first group of columns
// for all of them.  Every launch does it before its first wait, for all its
// plans: one whose waits give up still advances the epochs, so a slot left out
// would offer the next launch the value of the one before.
template <typename T> __device__ __forceinline__ void df_clear(const TriArgs &a, int e0, int nex, T *other)
{
    if (blockIdx.y != 0) return;
    const size_t m0 = (size_t)e0 * a.mbox_stride, m1 = (size_t)(e0 + nex) * a.mbox_stride;
    for (size_t i = m0 + threadIdx.x; i < m1; i += blockDim.x) other[i] = sentinel<T>();
}
// The same for parts taken from a queue: every workgroup a share of all slots,
// also of the parts that no workgroup comes to when waits give up.
template <typename T> __device__ __forceinline__ void df_clear_share(const TriArgs &a, T *other)
{
    const size_t count = (size_t)a.nexp * a.mbox_stride, step = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += step) other[i] = sentinel<T>();
}

// Everything but the right-hand side: sentinels, the zero row and index lists.
template <typename T> __device__ __forceinline__ void df_fill_lists(const TriArgs &a, const DfPart<T> &p, int R)
{
    const int tid = threadIdx.x, nt = blockDim.x;
    for (int t = tid; t < p.win * R; t += nt) p.xl[t] = sentinel<T>();
    for (int t = tid; t < (p.nimp + 1) * R; t += nt) p.im[t] = t < p.nimp * R ? sentinel<T>() : T(0);
    df_copy_ints(p.isl, a.imp_slot + p.i0, p.nimp, 0);
    df_copy_ints(p.erl, a.exp_row + p.e0, p.nex, -p.lo);
    df_copy_ints(p.stl, a.step_pack + p.s0, p.ns, 0);
    if (tid < kDataflowPad) p.stl[p.ns + tid] = 0;
}

// The right-hand side, gathered and scaled.  The gather indices of a round
// are loaded while the values of the round before are in flight.
template <typename T, bool UNIT, bool R1, typename TIn>
__device__ __forceinline__ void df_fill_b(const TriArgs &a, const DfPart<T> &p, int R, const TIn *bin)
{
    const int tid = threadIdx.x, nt = blockDim.x, cnt = p.win * R;
    int gi[kDfFill];
    T dd[kDfFill];
    auto index = [&](int t0) {
#pragma unroll
        for (int u = 0; u < kDfFill; ++u) {
            const int t = min(t0 + u * nt, cnt - 1);
            gi[u] = a.gather[p.lo + (R1 ? t : t / R)];
        }
    };
    if (tid < cnt) index(tid);
    for (int t0 = tid; t0 < cnt; t0 += kDfFill * nt) {
        TIn bv[kDfFill];
#pragma unroll
        for (int u = 0; u < kDfFill; ++u) {
            const int t = min(t0 + u * nt, cnt - 1);
            bv[u] = bin[(size_t)gi[u] * a.ldr + (p.k0 + (R1 ? 0 : t % R))];
            if (!UNIT) dd[u] = static_cast<const T *>(a.dinv)[p.lo + (R1 ? t : t / R)];
        }
        if (t0 + kDfFill * nt < cnt) index(t0 + kDfFill * nt);
#pragma unroll
        for (int u = 0; u < kDfFill; ++u) {
            T v = canon(static_cast<T>(bv[u]));
            if (!UNIT) v = scale_rhs(v, dd[u]);
            if (t0 + u * nt < cnt) p.bl[t0 + u * nt] = v;
        }
    }
}

// Import wave `w` of `nw`: the part's imports in level order are dealt to
// LOOK * nw slots of 64 lanes; a slot polls its next item until it arrives,
// copies it into LDS and goes to its next one.  All of a wave's slots have a
// load in flight together.  What bounds a handoff (1.2-1.4 us) and the rate of
// a stream of them is the round: an uncached round trip plus the
// instructions between two, so addresses are kept in registers and computed
// only on arrival (against slots that searched the list for their next items
// every round: 128^3 ILU(0) 308 -> 264 us, 100^3 211 -> 183 us per L+U).  Two
// waves with one slot beat one wave with two (259 us, 181 us; ILU(1) of
// 47x41x37 with four right-hand sides 270 -> 239 us) but for wide rows, whose
// compute waves keep the LDS busy (100^3 ILUT, width 10: 1386 against 1455
// us; two waves of two slots 1631 us).  A slot past its last item polls that
// again.
template <typename T, int LOOK, bool R1>
__device__ __forceinline__ void df_import(const TriArgs &a, const DfPart<T> &pt, int R, T *mrd, int *s_abort, int w, int nw)
{
    const int items = pt.nimp * R, lane = threadIdx.x & 63;
    if (items <= 64 * w) return;
    T *im = pt.xl + 2 * pt.win * R;
    int idx[LOOK];
    unsigned at[LOOK];
    auto place = [&](int i) {
        i = min(i, items - 1);
        const int q = R1 ? i : i / R, k = R1 ? 0 : i - q * R;
        return (unsigned)pt.isl[q] * (unsigned)a.mbox_stride + (unsigned)k;
    };
#pragma unroll
    for (int u = 0; u < LOOK; ++u) {
        idx[u] = lane + 64 * (u * nw + w);
        at[u] = place(idx[u]);
    }
    unsigned quiet = 0;  // rounds since the last arrival
    for (;;) {
        T v[LOOK];
#pragma unroll
        for (int u = 0; u < LOOK; ++u) v[u] = __hip_atomic_load(mrd + at[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        bool fresh = false;
#pragma unroll
        for (int u = 0; u < LOOK; ++u) {
            if (!is_sentinel(v[u]) && idx[u] < items) {
                lds_put(im + idx[u], v[u]);
                idx[u] += 64 * LOOK * nw;
                at[u] = place(idx[u]);
                fresh = true;
            }
        }
        if (__ballot(fresh) != 0) {
            int left = idx[0];
#pragma unroll
            for (int u = 1; u < LOOK; ++u) left = min(left, idx[u]);
            if (__ballot(left < items) == 0) break;
            quiet = 0;
            continue;
        }
        if (++quiet > a.spin) {
            lds_put(s_abort, 2);
        } else if ((quiet & 255u) == 0 &&
                   __hip_atomic_load(a.err_dev, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
            lds_put(s_abort, 1);  // another workgroup gave up
        }
        if (((quiet & 15u) == 0 || quiet > a.spin) && lds_get(s_abort)) break;
    }
}

// One part of one triangle, from filled LDS to solved LDS.  `fill` puts the
// part's right-hand side and lists into LDS; the compute wavefronts issue
// their first matrix loads before it.
template <typename T, int W, bool TAIL, bool R1, bool TRACE, typename Fill>
__device__ __forceinline__ void df_sweep(const TriArgs &a, const DfPart<T> &pt, int R, T *mrd, int *s_abort,
                                         unsigned long long &t_fill, Fill fill)
{
    using Rec = RowRec<T, W>;
    constexpr int K = df_sets<T, W>();
    const int tid = threadIdx.x, nt = blockDim.x;
    const int lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nwc = (nt >> 6) - 1 - a.imp_waves;
    const int lo = pt.lo;
    T *xl = pt.xl;
    // the lane's row and right-hand side within any step (lanes past a
    // step's rows repeat its last row)
    const unsigned q0 = R1 ? lane : lane / R;
    const unsigned q16 = q0 * 16u;
    const unsigned rowb = (R1 ? 1u : (unsigned)R) * (unsigned)sizeof(T);
    const unsigned kb = R1 ? 0u : (lane - q0 * R) * (unsigned)sizeof(T);
    const unsigned bofs = (unsigned)(reinterpret_cast<unsigned char *>(pt.bl) - reinterpret_cast<unsigned char *>(xl));
    const unsigned long long nbytes = (unsigned long long)Rec::ND * 4u * (unsigned)a.ld;
    const BufRsrc rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<void *>(a.ell_val), 0, (int)(unsigned)(nbytes > 0xffffffffull ? 0xffffffffull : nbytes), 0x00020000);
    // the part's rows begin at lo: chunk c of its row r is 16 bytes at
    // (lo + c * ld + r) * 16, the remainder behind all chunks
    const unsigned ld = (unsigned)a.ld, base = (unsigned)lo * 16u, rbase = Rec::CH * ld * 16u + (unsigned)lo * (Rec::RE * 4u);
    uint32_t S[K][Rec::ND];
    unsigned xo[K];  // LDS byte offset of the item's value
    // Loads of the step with descriptor dsc into set i.  All of it is vector
    // work on a descriptor every lane holds: no scalar register is written by
    // a vector instruction, which would cost wait states before its use.
    auto load = [&](int i, unsigned dsc) {
        unsigned vo;
        asm("v_mad_u32_u16 %0, %1, 16, %2" : "=v"(vo) : "v"(dsc), "v"(min(q16, dsc >> 16)));
        row_load<T, W>(S[i], rsrc, ld, base, rbase, vo);
        xo[i] = R1 ? vo / (16u / (unsigned)sizeof(T)) : (vo / 16u) * rowb + kb;
        asm volatile("" : "+v"(xo[i]));  // here, not on the dependency chain
    };
    int j = 0, jend = 0;
    if (wv < nwc) {
        j = __builtin_amdgcn_readfirstlane(a.wave_ptr[pt.g * nwc + wv]) - pt.s0;
        jend = __builtin_amdgcn_readfirstlane(a.wave_ptr[pt.g * nwc + wv + 1]) - pt.s0;
        if (j < jend) {
            const int tab = a.step_pack[pt.s0 + min(j + lane, jend - 1)];
#pragma unroll
            for (int p = 0; p < K - 1; ++p) {
                load(p, (unsigned)__builtin_amdgcn_readlane(tab, p));
                // in order: the first wait of the loop then covers one set
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    fill();
    __syncthreads();
    t_fill = TRACE ? __builtin_amdgcn_s_memrealtime() : 0ull;

    if (wv < nwc) {
        const T *tv = static_cast<const T *>(a.tail_val);
        const int ntr = TRACE ? min(pt.ns, a.trace_stride - 1) : 0;
        bool aborted = false;
        T bv[K], dep[W];
        unsigned dsc = 0;  // descriptor of the step whose loads are issued next
        unsigned stp = 0;  // LDS address of descriptor j
        unsigned on[W];  // LDS byte offsets of the next step's inputs
        auto rhs = [&](int i) { bv[i] = *(LdsPtr<T>)(uintptr_t)(xo[i] + bofs); };
        auto offset = [&](const uint32_t (&u)[Rec::ND], int e) {
            if constexpr (R1) return row_off<T, W, (unsigned)sizeof(T)>(u, e);
            else return row_off<T, W>(u, e, rowb, kb);
        };
        auto offsets = [&](const uint32_t (&u)[Rec::ND]) {
#pragma unroll
            for (int e = 0; e < W; ++e) on[e] = offset(u, e);
        };
        auto read = [&](const unsigned *o) {
#pragma unroll
            for (int e = 0; e < W; ++e) dep[e] = lds_at<T>(o[e]);
        };
        auto step = [&](int p, bool more) {  // more: also issue the loads of step p + K - 1
            const uint32_t (&u)[Rec::ND] = S[p];
            if (TRACE && j + p < ntr && lane == 0) pt.ltr[2 * (j + p)] = __builtin_amdgcn_s_memrealtime();
            if (more) {
                load((p + K - 1) % K, dsc);
                dsc = *(LdsPtr<unsigned>)(uintptr_t)(stp + 4u * (unsigned)(p + K));
            }
            rhs((p + 2) % K);
            offsets(S[(p + 1) % K]);
            __builtin_amdgcn_sched_barrier(0);
            T acc = bv[p];
#pragma unroll
            for (int e = 0; e < W; ++e) acc -= row_val<T, W>(u, e) * dep[e];
            if (__builtin_expect(__ballot(acc != acc) != 0, 0)) {
                bool pend = false;
                unsigned oc[W];
#pragma unroll
                for (int e = 0; e < W; ++e) oc[e] = offset(u, e);
#pragma unroll
                for (int e = 0; e < W; ++e) pend |= is_sentinel(dep[e]);
                unsigned spins = 0;
                while (pend) {
                    read(oc);
                    pend = false;
#pragma unroll
                    for (int e = 0; e < W; ++e) pend |= is_sentinel(dep[e]);
                    if (pend && (++spins & 63u) == 0) {
                        if (lds_get(s_abort)) {
                            aborted = true;
                            break;
                        }
                        if (spins > (a.spin << 4)) {
                            lds_put(s_abort, 2);
                            aborted = true;
                            break;
                        }
                    }
                }
                acc = bv[p];
#pragma unroll
                for (int e = 0; e < W; ++e) acc -= row_val<T, W>(u, e) * dep[e];
            }
            if (TAIL) {
                const unsigned x = lo + (R1 ? xo[p] / (unsigned)sizeof(T) : (xo[p] - kb) / rowb);
                for (int t = a.tail_ptr[x]; t < a.tail_ptr[x + 1]; ++t) {
                    const unsigned o = (unsigned)a.tail_col[t] * rowb + kb;
                    T dd = lds_at<T>(o);
                    unsigned sp = 0;
                    while (is_sentinel(dd)) {
                        dd = lds_at<T>(o);
                        if ((++sp & 63u) == 0) {
                            if (lds_get(s_abort)) {
                                aborted = true;
                                break;
                            }
                            if (sp > (a.spin << 4)) {
                                lds_put(s_abort, 2);
                                aborted = true;
                                break;
                            }
                        }
                    }
                    acc -= tv[t] * dd;
                }
            }
            lds_set(xo[p], acc);
            read(on);
            __builtin_amdgcn_sched_barrier(0);
            if (TRACE && j + p < ntr && lane == 0) pt.ltr[2 * (j + p) + 1] = __builtin_amdgcn_s_memrealtime();
        };
        if (j < jend) {
            stp = (unsigned)(uintptr_t)(LdsPtr<int>)(pt.stl + j);
            asm volatile("" : "+v"(stp));
            dsc = *(LdsPtr<unsigned>)(uintptr_t)(stp + 4u * (unsigned)(K - 1));
            // the first sets have arrived (vmcnt 0, other counters as they
            // are): the loop's waits then count its own loads only
            __builtin_amdgcn_s_waitcnt(0x0f70);
            rhs(0);
            rhs(1);
            offsets(S[0]);
            read(on);
            const int rounds = (jend - j) / K, rest = (jend - j) - K * rounds;
            // the loop's place in the instruction stream, which a change of the
            // code before it moves: by four bytes the same steps of 20011
            // irregular rows, two right-hand sides, took 222 to 232 us (at 64
            // bytes plus 0, 4, 8 and 12: 224.7, 224.4, 229.4, 228.2)
            asm volatile(".p2align 6\n\ts_nop 0");
            for (int q = 0; q < rounds; ++q) {
#pragma unroll
                for (int p = 0; p < K; ++p) step(p, true);
                if (__ballot(aborted) != 0) break;
                j += K;
                stp += 4u * K;
            }
#pragma unroll
            for (int p = 0; p < K - 1; ++p)
                if (rest > p && __ballot(aborted) == 0) step(p, false);
        }
    } else if (wv < nwc + a.imp_waves) {
        if (a.imp_waves == 2) df_import<T, 1, R1>(a, pt, R, mrd, s_abort, wv - nwc, 2);
        else df_import<T, 2, R1>(a, pt, R, mrd, s_abort, 0, 1);
    } else {
        // export wave: each lane watches its next exported item; a round in
        // which no lane found a new value sleeps briefly, so the wave does
        // not take issue slots and LDS bandwidth from the compute waves
        const int items = pt.nex * R;
        int it = lane;
        unsigned off = 0, at = 0, rounds = 0;
        auto place = [&](int i) {
            const int q = R1 ? i : i / R, k = R1 ? 0 : i - q * R;
            off = (unsigned)pt.erl[q] * rowb + (unsigned)k * (unsigned)sizeof(T);
            at = (unsigned)(pt.e0 + q) * (unsigned)a.mbox_stride + (unsigned)k;
        };
        if (it < items) place(it);
        while (__ballot(it < items) != 0) {
            bool moved = false;
            if (it < items) {
                const T v = lds_at<T>(off);
                if (!is_sentinel(v)) {
                    __hip_atomic_store(mrd + at, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    it += 64;
                    moved = true;
                    if (it < items) place(it);
                }
            }
            if (__ballot(moved) != 0) {
                rounds = 0;
                continue;
            }
            __builtin_amdgcn_s_sleep(1);
            if ((++rounds & 15u) == 0) {
                if (rounds > (a.spin << 4)) lds_put(s_abort, 2);
                if (lds_get(s_abort)) break;
            }
        }
    }
    __syncthreads();
}

// The part's solution from LDS to the workspace and / or the caller's vector.
template <typename T> __device__ __forceinline__ void df_store(const TriArgs &a, const DfPart<T> &p, int R)
{
    const int nt = blockDim.x;
    for (int t = threadIdx.x; t < p.win * R; t += nt) {
        const int q = t / R, k = t - q * R;
        const int x = p.lo + q;
        const T v = p.xl[t];
        if (a.write_xw) static_cast<T *>(a.xw)[(size_t)x * a.ldr + p.k0 + k] = v;
        if (a.xout) {
            const int d = a.scatter[x];  // negative: the row is not written (RAS overlap rows)
            if (d >= 0) {
                const size_t dst = (size_t)d * a.ldr + p.k0 + k;
                if (a.out_f64) static_cast<double *>(a.xout)[dst] = static_cast<double>(v);
                else static_cast<float *>(a.xout)[dst] = static_cast<float>(v);
            }
        }
    }
}

// Report a wait that gave up (abort 2) to the other workgroups and the host.
__device__ __forceinline__ void df_report(const TriArgs &a, DfCtl *ctl)
{
    if (threadIdx.x == 0 && ctl->abort == 2) {
        __hip_atomic_store(a.err_dev, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(a.err_host, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        ctl->abort = 1;
    }
}

// The last workgroup out resets the plan's counters and advances its epoch.
__device__ __forceinline__ void df_leave(const TriArgs &a, unsigned epoch)
{
    const unsigned done = __hip_atomic_fetch_add(&a.epoch[1], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    if (done == gridDim.x * gridDim.y - 1) {
        __hip_atomic_store(&a.epoch[2], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&a.epoch[1], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&a.epoch[0], epoch + 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    }
}

template <typename T, int W, bool UNIT, bool TAIL, bool R1, bool TRACE>
__global__ void __launch_bounds__(512) k_dataflow(TriArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    DfCtl *ctl = reinterpret_cast<DfCtl *>(smem + a.lds_ctl);
    const int tid = threadIdx.x;
    const int k0 = a.k0 + (int)blockIdx.y * a.R, R = R1 ? 1 : min(a.R, a.ldr - k0);
    if (tid == 0) {
        ctl->epoch = __hip_atomic_load(a.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        ctl->abort = 0;
    }
    __syncthreads();
    const unsigned par = ctl->epoch & 1u;
    T *mbox = static_cast<T *>(a.mbox);
    const size_t half = (size_t)a.nexp * a.mbox_stride;
    T *mrd = mbox + (par ? half : 0) + k0, *other = mbox + (par ? 0 : half);
    for (int round = 0;; ++round) {
        if (a.queue) {
            if (tid == 0) ctl->part = (int)__hip_atomic_fetch_add(&a.epoch[2], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
        } else if (round > 0) {
            break;
        }
        const int g = a.queue ? ctl->part : (int)blockIdx.x;
        if (a.queue && round == 0) df_clear_share(a, other);
        if (g >= a.nparts) break;
        const DfPart<T> pt = df_part<T>(a, g, k0, R, smem);
        unsigned long long t_fill = 0;
        df_sweep<T, W, TAIL, R1, TRACE>(a, pt, R, mrd, &ctl->abort, t_fill, [&]() {
            if (a.in_f64) df_fill_b<T, UNIT, R1>(a, pt, R, static_cast<const double *>(a.bin));
            else df_fill_b<T, UNIT, R1>(a, pt, R, static_cast<const float *>(a.bin));
            df_fill_lists(a, pt, R);
            if (!a.queue) df_clear(a, pt.e0, pt.nex, other);
        });
        const unsigned long long t_done = TRACE ? __builtin_amdgcn_s_memrealtime() : 0ull;
        df_report(a, ctl);
        if (TRACE && blockIdx.y == 0) {
            const int ntr = min(pt.ns, a.trace_stride - 1);
            for (int t = tid; t < 2 * ntr; t += blockDim.x) a.trace[2 * (size_t)g * a.trace_stride + t] = pt.ltr[t];
            if (tid == 0) {
                a.trace[2 * ((size_t)g * a.trace_stride + a.trace_stride - 1)] = t_fill;
                a.trace[2 * ((size_t)g * a.trace_stride + a.trace_stride - 1) + 1] = t_done;
            }
        }
        if (!ctl->abort) df_store(a, pt, R);
        __syncthreads();  // LDS is refilled by the next part
        if (ctl->abort) break;
    }
    if (tid == 0) df_leave(a, ctl->epoch);
}

// U's right-hand side from L's solution, which is still in this workgroup's
// LDS: row t of U's part is row gather[t] - lo of L's (the parts hold the same
// rows).  Writes the b area, which L no longer needs, then the caller clears
// the x area the values came from.
template <typename T, bool R1>
__device__ __forceinline__ void df_fill_y(const TriArgs &u, const DfPart<T> &p, int R, int lo)
{
    const int tid = threadIdx.x, nt = blockDim.x, cnt = p.win * R;
    for (int t0 = tid; t0 < cnt; t0 += kDfFill * nt) {
        int gi[kDfFill];
        T dd[kDfFill];
#pragma unroll
        for (int v = 0; v < kDfFill; ++v) {
            const int t = min(t0 + v * nt, cnt - 1), x = p.lo + (R1 ? t : t / R);
            gi[v] = u.gather[x];
            dd[v] = static_cast<const T *>(u.dinv)[x];
        }
#pragma unroll
        for (int v = 0; v < kDfFill; ++v) {
            const int t = t0 + v * nt;
            if (t < cnt) p.bl[t] = scale_rhs(p.xl[(gi[v] - lo) * R + (R1 ? 0 : t % R)], dd[v]);
        }
    }
}

// Both triangles of an ILU application in one launch, for plans whose parts
// hold the same rows (same workgroup), with one ELL width and no CSR tail: L,
// then U on the same workgroup with L's solution taken from LDS.  Saves the
// second launch, the drain of the first (a workgroup starts U when its own
// part of L is done; U waits only on U), the round trip of y through memory
// and the two dependent gathers of it.  L's values never reach memory.
template <typename T, int W, bool R1>
__global__ void __launch_bounds__(512) k_dataflow_lu(TriArgs l, TriArgs u)
{
    extern __shared__ __align__(16) unsigned char smem[];
    DfCtl *ctl = reinterpret_cast<DfCtl *>(smem + l.lds_ctl);
    const int k0 = l.k0 + (int)blockIdx.y * l.R, R = R1 ? 1 : min(l.R, l.ldr - k0), g = blockIdx.x;
    const int ue0 = u.exp_ptr[g], ue1 = u.exp_ptr[g + 1];  // on their way with the epochs
    if (threadIdx.x == 0) {
        ctl->epoch = __hip_atomic_load(l.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        ctl->epoch2 = __hip_atomic_load(u.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        ctl->abort = 0;
    }
    __syncthreads();
    unsigned long long t_fill = 0;
    auto half = [&](const TriArgs &a, unsigned par) {
        return static_cast<T *>(a.mbox) + (par & 1u ? (size_t)a.nexp * a.mbox_stride : 0);
    };
    const DfPart<T> pl = df_part<T>(l, g, k0, R, smem);
    df_sweep<T, W, false, R1, false>(l, pl, R, half(l, ctl->epoch) + k0, &ctl->abort, t_fill, [&]() {
        if (l.in_f64) df_fill_b<T, true, R1>(l, pl, R, static_cast<const double *>(l.bin));
        else df_fill_b<T, true, R1>(l, pl, R, static_cast<const float *>(l.bin));
        df_fill_lists(l, pl, R);
        df_clear(l, pl.e0, pl.nex, half(l, ctl->epoch + 1u));
        df_clear(u, ue0, ue1 - ue0, half(u, ctl->epoch2 + 1u));
    });
    if (!ctl->abort) {
        const DfPart<T> pu = df_part<T>(u, g, k0, R, smem);
        df_sweep<T, W, false, R1, false>(u, pu, R, half(u, ctl->epoch2) + k0, &ctl->abort, t_fill, [&]() {
            df_fill_y<T, R1>(u, pu, R, pl.lo);
            __syncthreads();
            df_fill_lists(u, pu, R);
        });
        if (!ctl->abort) df_store(u, pu, R);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (ctl->abort == 2) {  // a wait gave up: tell the other workgroups, in either triangle
            for (int *e : {l.err_dev, u.err_dev}) __hip_atomic_store(e, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            for (int *e : {l.err_host, u.err_host}) __hip_atomic_store(e, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        df_leave(l, ctl->epoch);
        df_leave(u, ctl->epoch2);
    }
}

}  // namespace hec

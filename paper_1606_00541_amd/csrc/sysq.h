// Pipelined system queue: whole independent systems per workgroup, level by
// level, with the last levels' values in LDS.
#pragma once

#include "row_record.h"

namespace hec {

// What bounds it: a level is a chain of ring reads, multiply-adds, a ring
// write and a workgroup barrier, and a wavefront must find its row data and
// right-hand sides already loaded, or the level waits for memory.  The memory
// counter is in order and a count is only exact when every path issues the
// same operations, so nothing in a turn is conditional: loads are clamped to
// valid rows, results that must not be stored go to a buffer offset past the
// end (the hardware drops them), and a row is one packed record.  (With
// conditional stores each level also waited for the stores of the level
// before.)
//
// The workgroups take items, a system and a group of its columns, from a
// counter (largest system first).  A thread has C (one or four) columns of a
// row; 1 << cshift threads share a row of an item, neighbours in a wavefront, so
// that a row's record is fetched once for them.  Levels are cut into pieces
// of at most M rows per thread.  The wavefronts form
// k groups that take a system's pieces in turn (k as large as its widest
// piece allows); a turn's row data is loaded P turns ahead and its right-hand
// sides, whose address needs the row's gather index, H turns ahead.
// A row's values are computed as in k_level (right-hand side scaled by the
// reciprocal diagonal, then the ELL slots in order; padding reads the ring's
// zero row and subtracts 0 * 0), so results are bit-identical to it.
// FAR: some rows read values older than the ring (at most two or four each;
// uneven subdomain cuts give long level distances).  Those are loaded from the
// workspace together with the right-hand sides; the host sized the ring so
// that they were stored before an earlier barrier by then.
// Measured (both triangles, FP32 values, before: one item per system, rows
// gathered slot by slot): 64 overlapping subdomains of a 128^3 grid, 16
// right-hand sides 1985 -> 1140 us (they ran on the barrier-free kernel; on
// this queue without column groups 10.9 ms); 256 ILU(1) systems, 8 right-hand
// sides 2769 -> 1215 us; in FP64 with 1 / 4 / 5 right-hand sides 7850 -> 1035
// (items of one column), 2750 -> 1070 and 18240 -> 1310 us.  Column groups
// alone gave 1537 and 2375.  P / H of
// 5 / 2, 4 / 1 and 6 / 3 took 1203, 1193 and 1205 where 4 / 2 took 1189.
// Needs no CSR tail, columns in multiples of an item's and vectors below 4 GiB (checked by the host).

typedef uint32_t sq_u4 __attribute__((ext_vector_type(4)));
typedef uint32_t sq_u2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void sq_store(BufRsrc r, unsigned at, double x, double y)
{
    const unsigned long long p = __builtin_bit_cast(unsigned long long, x), q = __builtin_bit_cast(unsigned long long, y);
    __builtin_amdgcn_raw_buffer_store_b128(sq_u4{(uint32_t)p, (uint32_t)(p >> 32), (uint32_t)q, (uint32_t)(q >> 32)}, r,
                                           (int)at, 0, 0);
}
__device__ __forceinline__ void sq_store(BufRsrc r, unsigned at, float x, float y, float z, float w)
{
    __builtin_amdgcn_raw_buffer_store_b128(sq_u4{__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, y),
                                                 __builtin_bit_cast(uint32_t, z), __builtin_bit_cast(uint32_t, w)},
                                           r, (int)at, 0, 0);
}

// C values to / from byte offset `at`, C one or four; stored as FP64 or FP32.
template <bool F64, typename T, int C> __device__ __forceinline__ void sq_put(BufRsrc r, unsigned at, const T (&s)[C])
{
    if constexpr (C == 1 && F64) {
        const unsigned long long p = __builtin_bit_cast(unsigned long long, (double)s[0]);
        __builtin_amdgcn_raw_buffer_store_b64(sq_u2{(uint32_t)p, (uint32_t)(p >> 32)}, r, (int)at, 0, 0);
    } else if constexpr (C == 1) {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, (float)s[0]), r, (int)at, 0, 0);
    } else if constexpr (F64) {
        sq_store(r, at, (double)s[0], (double)s[1]);
        sq_store(r, at + 16u, (double)s[2], (double)s[3]);
    } else {
        sq_store(r, at, (float)s[0], (float)s[1], (float)s[2], (float)s[3]);
    }
}
template <typename T, int C> __device__ __forceinline__ void sq_load(T (&f)[C], BufRsrc r, unsigned at)
{
    if constexpr (C == 1 && sizeof(T) == 8) {
        auto v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)at, 0, 0);
        f[0] = __builtin_bit_cast(double, (unsigned long long)v[0] | ((unsigned long long)v[1] << 32));
    } else if constexpr (C == 1) {
        f[0] = __builtin_bit_cast(float, (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(r, (int)at, 0, 0));
    } else if constexpr (sizeof(T) == 8) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            auto v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)at, 16 * h, 0);
            f[2 * h] = __builtin_bit_cast(double, (unsigned long long)v[0] | ((unsigned long long)v[1] << 32));
            f[2 * h + 1] = __builtin_bit_cast(double, (unsigned long long)v[2] | ((unsigned long long)v[3] << 32));
        }
    } else {
        auto v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)at, 0, 0);
#pragma unroll
        for (int c = 0; c < 4; ++c) f[c] = __builtin_bit_cast(float, (uint32_t)v[c]);
    }
}

// FORM: 2 or 4: values beyond the ring a row may read (FAR), kSysqShared: several
// threads to a row, 0: neither.  (A kernel for both 0 and kSysqShared took a few
// registers more, which cost rows of six entries their second workgroup on a
// compute unit: 300 ILU(1) subdomains in FP32, one right-hand side 98 -> 119 us.)
// MODE 0: results to the workspace xw in device order, 1 / 2: to the caller's
// FP64 / FP32 vector through `scatter` (negative: not stored).
template <typename T, typename TIn, int W, int C, int M, int MODE, int FORM>
__global__ void __launch_bounds__(512) k_sysq_pipe(TriArgs a, const int32_t *__restrict__ pcp,
                                                   const int4 *__restrict__ pc,
                                                   const int32_t *__restrict__ rings)
{
    using Rec = RowRec<T, W>;
    constexpr int P = 4, H = kSysqAhead;
    constexpr unsigned RB = C * sizeof(T);  // a thread's bytes of a ring row
    constexpr bool SHARED = FORM == kSysqShared;
    constexpr int FAR = FORM == kSysqShared ? 0 : FORM;
    const int cs = SHARED ? a.cshift : 0;
    const unsigned rowb = RB << cs;
    extern __shared__ __align__(16) unsigned char smem[];
    int *s_q = reinterpret_cast<int *>(smem + a.lds_ctl);
    const int tid = threadIdx.x, nt = blockDim.x;
    // the wavefront index as a uniform value: level numbers derived from it
    // stay scalar, so the level table reads remain scalar loads
    const int nw = nt >> 6, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned epoch = tid == 0 ? __hip_atomic_load(a.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
    const bool scaled = a.dinv != nullptr;
    auto rsrc = [](const void *p, size_t bytes) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)(unsigned)(bytes > 0xffffffffull ? 0xffffffffull : bytes),
                                                 0x00020000);
    };
    const BufRsrc rrec = rsrc(a.ell_val, (size_t)Rec::ND * 4 * a.ld);
    const unsigned ld = (unsigned)a.ld;

    struct Row {                // a turn's rows of this thread
        RowRegs<T, W> d[M];     // records
        int gi[M], dst[M];      // gather and scatter indices
        T di[M];
        TIn b[M][C];
        int fi[M][FAR > 0 ? FAR : 1], keep[M];  // rows read beyond the ring; read back itself
        T f[M][FAR > 0 ? FAR : 1][C];
        int4 pc;                // the piece: first row, rows, first ring row
    };
    Row S[P];
    for (;;) {
        if (tid == 0)
            *s_q = (int)__hip_atomic_fetch_add(&a.epoch[2], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        const int item = __builtin_amdgcn_readfirstlane(*s_q);
        if (item >= a.nparts * a.cgroups) break;
        const int q = item / a.cgroups, cg = item - q * a.cgroups;
        const size_t k0 = (size_t)(cg * C) << cs;  // the item's first column
        const int slots = rings[2 * q], wide = rings[2 * q + 1];
        const unsigned zoff = (unsigned)(slots * wide) * rowb;
        if (a.trace && tid == 0 && cg == 0 && a.trace_stride > 0)
            a.trace[2 * (size_t)q * a.trace_stride] = __builtin_amdgcn_s_memrealtime();
        if (tid < C << cs) *reinterpret_cast<T *>(smem + zoff + tid * sizeof(T)) = T(0);
        const int l0 = pcp[q], l1 = pcp[q + 1];
        // a Krylov solve's mask of unfinished (system, rhs) problems: an item
        // whose right-hand sides have all finished is skipped (its rows feed
        // only its own problems)
        if (a.act && l1 > l0) {
            const int sys = a.seg ? a.seg[pc[l0].x] : 0;
            int live = 0;
            for (int c = 0; c < C << cs; ++c) live |= a.act[(size_t)sys * a.ldr + k0 + c];
            if (!live) {
                __syncthreads();  // every thread has read the item before it is replaced
                continue;
            }
        }
        // where the item's columns lie: in a vector of the caller (row after
        // row, all right-hand sides) or in a workspace that holds the column
        // groups one after the other
        const TIn *bin = static_cast<const TIn *>(a.bin) + (a.bin_grouped ? k0 * a.n : k0);
        const size_t ldin = a.bin_grouped ? C : a.ldr;
        const unsigned ldo = MODE == 0 && a.xw_grouped ? C : (unsigned)a.ldr;
        constexpr unsigned TO = MODE == 0 ? sizeof(T) : (MODE == 1 ? 8 : 4);
        const BufRsrc rout = MODE == 0 && a.xw_grouped
                                 ? rsrc(static_cast<T *>(a.xw) + k0 * a.n, ((size_t)a.n * C << cs) * TO)
                                 : rsrc(static_cast<unsigned char *>(MODE == 0 ? a.xw : a.xout) + k0 * TO,
                                        ((size_t)a.n * ldo - k0) * TO);
        // the workspace of a solve into the caller's vector is only read here
        const bool grouped = MODE != 0 || a.xw_grouped;
        const unsigned ldx = grouped ? C : (unsigned)a.ldr;
        const BufRsrc rxw = rsrc(static_cast<T *>(a.xw) + (grouped ? k0 * a.n : k0), ((size_t)a.n + 1) * ldx * sizeof(T));
        // wavefront groups: k groups take the pieces in turn (group g solves
        // pieces l0 + g, l0 + g + k, ...)
        const int need = (min(wide << cs, M * nt) + 64 * M - 1) / (64 * M);
        int wpg = 1;
        while (wpg < need && wpg < nw) wpg *= 2;
        const int k = nw / wpg, grp = wave / wpg;
        // rows a group takes at a time; the thread's row among them and its columns
        const int ng = wpg * 64 >> cs, tl = (tid - grp * wpg * 64) >> cs, sub = tid & ((1 << cs) - 1);
        const unsigned kb = (unsigned)sub * RB;
        const TIn *bsub = bin + (a.bin_grouped ? (size_t)sub * a.n * C : (size_t)(sub * C));
        const unsigned osub = (MODE == 0 && a.xw_grouped ? (unsigned)(sub * a.n * C) : (unsigned)(sub * C)) * TO;
        auto bounds = [&](int l) {
            int4 b = pc[min(l, l1 - 1)];
            if (l >= l1) b.y = 0;
            return b;
        };
        // row data of this thread's rows of a piece; a row past the piece
        // repeats its last one (pieces past the end: the last one's first)
        auto rows = [&](Row &u) {
#pragma unroll
            for (int m = 0; m < M; ++m) {
                const unsigned x = (unsigned)(u.pc.x + min(tl + m * ng, max(u.pc.y, 1) - 1));
                row_load<T, W>(u.d[m], rrec, ld, 0u, Rec::CH * ld * 16u, x * 16u);
                u.gi[m] = a.gather[x];
                if (MODE != 0) u.dst[m] = a.scatter[x];
                if constexpr (FAR == 2) {
                    const int2 f = reinterpret_cast<const int2 *>(a.sq_far)[x];
                    u.fi[m][0] = f.x;
                    u.fi[m][1] = f.y;
                }
                if constexpr (FAR == 4) {
                    const int4 f = reinterpret_cast<const int4 *>(a.sq_far)[x];
                    u.fi[m][0] = f.x;
                    u.fi[m][1] = f.y;
                    u.fi[m][2] = f.z;
                    u.fi[m][3] = f.w;
                }
                if (FAR && MODE != 0) u.keep[m] = a.sq_keep[x];
                u.di[m] = (scaled ? static_cast<const T *>(a.dinv) : static_cast<const T *>(a.ell_val))[x];
            }
        };
        auto rhs = [&](Row &u) {
#pragma unroll
            for (int m = 0; m < M; ++m) {
                const TIn *src = bsub + (size_t)(unsigned)u.gi[m] * ldin;
#pragma unroll
                for (int c = 0; c < C; ++c) u.b[m][c] = src[c];
                if constexpr (FAR) {
#pragma unroll
                    for (int j = 0; j < FAR; ++j)
                        sq_load(u.f[m][j], rxw, (unsigned)u.fi[m][j] * ldx * (unsigned)sizeof(T));
                }
            }
        };
        auto solve = [&](const Row &u, int m) {
            const int i = tl + m * ng;
            T s[C];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const T b = canon(static_cast<T>(u.b[m][c]));
                s[c] = scaled ? scale_rhs(b, u.di[m]) : b;
            }
#pragma unroll
            for (int e = 0; e < W; ++e) {
                unsigned o;
                if constexpr (SHARED) o = row_off<T, W>(u.d[m], e, rowb, kb);
                else o = row_off<T, W, RB>(u.d[m], e);
                const T v = row_val<T, W>(u.d[m], e);
                const unsigned code = o;
                if (FAR) o = min(o, zoff);
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    T dep = *(LdsPtr<T>)(uintptr_t)(o + c * (unsigned)sizeof(T));
#pragma unroll
                    for (int j = 0; j < FAR; ++j) dep = code == (kSysqFar - (unsigned)j) * RB ? u.f[m][j][c] : dep;
                    s[c] -= v * dep;
                }
            }
            const bool ok = i < u.pc.y;
            if (ok) {
                const unsigned o = (unsigned)(u.pc.z + i) * rowb + kb;
#pragma unroll
                for (int c = 0; c < C; ++c) *(LdsPtr<T>)(uintptr_t)(o + c * (unsigned)sizeof(T)) = s[c];
            }
            const int row = MODE == 0 ? u.pc.x + i : u.dst[m];
            sq_put<(TO == 8)>(rout, ok && row >= 0 ? (unsigned)row * ldo * TO + osub : kSysqDropped, s);
            if constexpr (FAR && MODE != 0)  // also read back by a later level
                sq_put<(sizeof(T) == 8)>(
                    rxw, ok && u.keep[m] ? (unsigned)(u.pc.x + i) * ldx * (unsigned)sizeof(T) : kSysqDropped, s);
        };
        if (l1 > l0) {
            // in order of their turns
#pragma unroll
            for (int p = 0; p < P; ++p) {
                S[p].pc = bounds(l0 + grp + p * k);
                rows(S[p]);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int p = 0; p < H; ++p) {
                rhs(S[p]);
                __builtin_amdgcn_sched_barrier(0);
            }
            __builtin_amdgcn_s_waitcnt(0x0f70);  // the loop's waits count its own operations only
        }
        __syncthreads();
        // one barrier per piece, for every wavefront: the pieces of the other
        // groups before and after this group's piece of the turn.  Whole
        // rotations: turns past the last piece have no rows, no barrier and
        // nothing to store (leaving early would cost the exact counts)
        const int nr = (l1 - l0 + k - 1) / k;
        for (int r0 = 0; r0 < nr; r0 += P) {
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const int r = r0 + p;
                const int nlr = min(k, l1 - l0 - r * k);  // pieces in this turn of the groups
                for (int g = 0; g < min(grp, nlr); ++g) __syncthreads();
                const int4 next = bounds(l0 + (r + P) * k + grp);
                rhs(S[(p + H) % P]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int m = 0; m < M; ++m) solve(S[p], m);
                __builtin_amdgcn_sched_barrier(0);
                S[p].pc = next;
                rows(S[p]);
                if (grp < nlr) __syncthreads();
                for (int g = grp + 1; g < nlr; ++g) __syncthreads();
            }
        }
        if (a.trace && tid == 0 && cg == 0 && a.trace_stride > 0)
            a.trace[2 * (size_t)q * a.trace_stride + 1] = __builtin_amdgcn_s_memrealtime();
    }
    if (tid == 0) {
        const unsigned done = __hip_atomic_fetch_add(&a.epoch[1], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        if (done == gridDim.x - 1) {
            // last workgroup out: every claim is over; reset the queue
            __hip_atomic_store(&a.epoch[2], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&a.epoch[1], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&a.epoch[0], epoch + 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

}  // namespace hec

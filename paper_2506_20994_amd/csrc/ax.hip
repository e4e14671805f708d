// The element-local stiffness operator w = A_e u (paper Sec. 4.2, Listing 2).
//
// Work decomposition (gfx950, wave64): a workgroup holds EPB elements; each
// element is owned by lx*lx threads (one whole wave at lx = 8), thread (i, j)
// owning the column
// u[e][0..lx)[j][i].  The column lives in registers, so the t-derivative is a
// register-only sum, and the t-flux of each slice is folded into the
// transposed t-sum as soon as it is formed.  The r- and s-derivatives need the
// rows of a k-slice, so the element is staged once in LDS; the r/s fluxes are
// staged in LDS for the transposed pass.
// The streamed arrays (u, w, h1, g11..g23) are read and written exactly once,
// with consecutive threads on consecutive addresses.  Where lx^2 columns fit waves
// and lines badly, or the registers of a column are what limits the waves, a second
// kernel takes whole elements as they lie in memory and forms the derivatives on the
// matrix cores (ax_flat_kernel; kFlat, flat_pays and kFlatSolver say where).
//
// Storage type TS (u, h1, G) and compute type TC:
//   double / double   (SEM_F64)
//   float  / float    (SEM_F32)
//   bf16   / float    (SEM_BF16, bf16 stored as uint16_t bit patterns)
#include <type_traits>
#include <vector>

#include "sem_internal.h"

namespace {

// Streamed arrays are touched once per application, so they are read and
// written with the nontemporal hint: on gfx950 this keeps them from displacing
// reusable lines and measurably raises the achieved HBM bandwidth.
template <typename T> struct Load;
template <> struct Load<double> {
    __device__ static double get(const double* p, int64_t o) { return __builtin_nontemporal_load(p + o); }
};
template <> struct Load<float> {
    __device__ static float get(const float* p, int64_t o) { return __builtin_nontemporal_load(p + o); }
};
template <> struct Load<uint16_t> {
    __device__ static float get(const uint16_t* p, int64_t o) {
        return __uint_as_float((uint32_t)__builtin_nontemporal_load(p + o) << 16);
    }
};

template <typename T>
__device__ __forceinline__ void store_nt(T* p, int64_t o, T v) { __builtin_nontemporal_store(v, p + o); }

// The same accesses through the caches, for element slices that are not whole
// 128-byte lines: a line shared by two slices (or two elements) is then read
// from HBM once, where the nontemporal form fetched it again for its second
// user.  In float64 the nontemporal form counted 1.43, 1.22 and 1.22 times the
// algorithmic bytes at lx = 5, 6, 7 and 1.08-1.11 at lx = 9, 10, 11; through the
// caches 1.00-1.10.  That made lx = 3, 5, 6, 7 faster (5: 67 -> 51 us at
// 32768 elements) but lx = 9, 10, 11 slower by 1-3 %: there the occupancy, not
// the bytes, bounds the kernel, so they keep the nontemporal form.
template <typename T> struct LoadC;
template <> struct LoadC<double> {
    __device__ static double get(const double* p, int64_t o) { return p[o]; }
};
template <> struct LoadC<float> {
    __device__ static float get(const float* p, int64_t o) { return p[o]; }
};
template <> struct LoadC<uint16_t> {
    __device__ static float get(const uint16_t* p, int64_t o) { return __uint_as_float((uint32_t)p[o] << 16); }
};
template <bool NT, typename T>
__device__ __forceinline__ auto ld(const T* p, int64_t o) {
    if constexpr (NT) return Load<T>::get(p, o);
    else return LoadC<T>::get(p, o);
}
template <bool NT, typename T>
__device__ __forceinline__ void st(T* p, int64_t o, T v) {
    if constexpr (NT) __builtin_nontemporal_store(v, p + o);
    else p[o] = v;
}
// nontemporal streaming when an lx^2 slice of TS is a whole number of lines, or lx >= 9
template <int LX, typename TS>
constexpr bool kStreamNT = (LX * LX * sizeof(TS)) % 128 == 0 || LX >= 9;

// Solver copies of the six factors (float64, float32), slice-blocked in
// pairs: for the slice (e, k) the pairs (g11, g22), (g33, g12), (g13, g23) of
// all lx*lx columns are stored as three consecutive runs of lx*lx two-element
// vectors, so each wave load is one contiguous block (1 KiB in float64 at
// lx = 8).  o is the node's local offset, ij its column.
typedef double dvec2 __attribute__((ext_vector_type(2)));
typedef float fvec2 __attribute__((ext_vector_type(2)));
template <typename TS> struct Packed;
template <> struct Packed<double> {
    __device__ static void get(const double* gp, int64_t o, int ij, int l2, double* g) {
        const dvec2* q = reinterpret_cast<const dvec2*>(gp) + (o - ij) * 3 + ij;
        const dvec2 a = __builtin_nontemporal_load(q), b = __builtin_nontemporal_load(q + l2),
                    c = __builtin_nontemporal_load(q + 2 * l2);
        g[0] = a.x; g[1] = a.y; g[2] = b.x; g[3] = b.y; g[4] = c.x; g[5] = c.y;
    }
};
template <> struct Packed<float> {
    __device__ static void get(const float* gp, int64_t o, int ij, int l2, float* g) {
        const fvec2* q = reinterpret_cast<const fvec2*>(gp) + (o - ij) * 3 + ij;
        const fvec2 a = __builtin_nontemporal_load(q), b = __builtin_nontemporal_load(q + l2),
                    c = __builtin_nontemporal_load(q + 2 * l2);
        g[0] = a.x; g[1] = a.y; g[2] = b.x; g[3] = b.y; g[4] = c.x; g[5] = c.y;
    }
};
// bfloat16 copies: one 12-byte record per node, (h1 g11, h1 g22, h1 g33,
// h1 g12, h1 g13, h1 g23), h1 folded in when the copy is made; a lane reads its
// node with one 12-byte load and a wave one contiguous block
template <> struct Packed<uint16_t> {
    __device__ static void get(const uint16_t* gp, int64_t o, int, int, float* g) {
        const uint32_t* q = reinterpret_cast<const uint32_t*>(gp) + 3 * o;
        const uint32_t a = __builtin_nontemporal_load(q), b = __builtin_nontemporal_load(q + 1),
                       c = __builtin_nontemporal_load(q + 2);
        g[0] = __uint_as_float(a << 16); g[1] = __uint_as_float(a & 0xffff0000u);
        g[2] = __uint_as_float(b << 16); g[3] = __uint_as_float(b & 0xffff0000u);
        g[4] = __uint_as_float(c << 16); g[5] = __uint_as_float(c & 0xffff0000u);
    }
};

#ifndef SEM_AX_PREFETCH
#define SEM_AX_PREFETCH(LX) ((LX) != 2 && (LX) != 8 && (LX) != 12)
#endif

template <int LX> struct Shape {
    static constexpr bool kWavePrivate = (64 % (LX * LX)) == 0;
    // occupancy floor (waves per SIMD) handed to the register allocator.  At
    // lx = 12 the kernel needs 169 VGPRs, two waves per SIMD; a floor of 3
    // brings it to 168 (two spilled, outside the slice loop) and, with the LDS
    // alias below, four workgroups per CU instead of two: 950 -> 774 us at
    // 32768 elements (without prefetch; with it 11 registers spill and it
    // slows down).  Floors elsewhere spilled inside the loop and lost (lx = 9,
    // 10: 4 waves per SIMD, 331 and 534 against 325 and 433 us).
    static constexpr int kWavesPerEU = LX == 12 ? 3 : 1;
    // fetch the next slice's h1 and G while the current slice is computed
    static constexpr bool kPrefetch = SEM_AX_PREFETCH(LX);
    // elements per workgroup: about four waves, LDS of float64 within ~64 KiB
    static constexpr int EPB = LX == 2 ? 64 : LX == 3 ? 28 : LX == 4 ? 16 : LX == 5 ? 10
                             : LX == 6 ? 7 : LX == 7 ? 5 : LX == 8 ? 4 : LX == 9 ? 3
                             : LX <= 11 ? 2 : 1;
};

// h1 and the six factors at offset o (node ij of a slice) of a live element;
// h = 1 and zero factors for a dead one
template <typename TS, typename TC, bool GATHER, bool NT = true>
__device__ __forceinline__ void load_factors(TC (&g)[6], TC& h, bool live, int64_t o, int ij, int l2,
                                             const TS* __restrict__ h1, const TS* __restrict__ g11,
                                             const TS* __restrict__ g22, const TS* __restrict__ g33,
                                             const TS* __restrict__ g12, const TS* __restrict__ g13,
                                             const TS* __restrict__ g23, const TS* __restrict__ gp) {
    h = 1;
    if (!live) {
#pragma unroll
        for (int a = 0; a < 6; ++a) g[a] = 0;
        return;
    }
    if constexpr (GATHER) {                    // the solver form reads the packed factors
        Packed<TS>::get(gp, o, ij, l2, g);
        if constexpr (std::is_same<TS, uint16_t>::value) return;   // h1 is folded into the record
    } else {
        g[0] = ld<NT>(g11, o); g[1] = ld<NT>(g22, o); g[2] = ld<NT>(g33, o);
        g[3] = ld<NT>(g12, o); g[4] = ld<NT>(g13, o); g[5] = ld<NT>(g23, o);
    }
    if (h1) h = ld<NT>(h1, o);
}

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// dot[blockIdx.x] = sum of v over the workgroup's NT threads, in a fixed order
template <int NT>
__device__ __forceinline__ void block_dot(double v, double* __restrict__ dot) {
    const int tid = threadIdx.x;
    if constexpr (NT % 64 == 0) {              // whole waves: shuffle, then one value per wave
        __shared__ double s_red[NT / 64];
        v = sem::wave_sum(v);
        if ((tid & 63) == 0) s_red[tid >> 6] = v;
        __syncthreads();
        if (tid == 0) {
            double t = 0.0;
            for (int q = 0; q < NT / 64; ++q) t += s_red[q];
            dot[blockIdx.x] = t;
        }
    } else {                                   // partial last wave: LDS tree
        __shared__ double s_red[NT];
        s_red[tid] = v;
        __syncthreads();
        constexpr int P2 = NT <= 128 ? 64 : NT <= 256 ? 128 : 256;
        for (int st = P2; st > 0; st >>= 1) {
            if (tid < st && tid + st < NT) s_red[tid] += s_red[tid + st];
            __syncthreads();
        }
        if (tid == 0) dot[blockIdx.x] = s_red[0];
    }
}

// Any form returns at once when skip is given and *skip is non-zero (a
// converged solve).  FUSE: the solver form's dot: each workgroup writes sum_L u_L w_L over its
// elements, accumulated in float64, to dot[blockIdx.x] (p^T A p before
// gather-scatter).
// GATHER: u is a unique-node vector, read as u[lid[L]] (lid streamed, u
// through the caches, since neighbouring elements share nodes; lid < 0 marks
// a Dirichlet node, read as 0).  The output stays in the local layout
// (coalesced nontemporal stores); the solver sums the copies of each unique
// node through the plan's links.
// TPE: threads per element (lx^2, or a power of two above it that divides 64,
// so that every element sits inside one wave; the extra lanes idle)
template <int LX, int EPB, typename TU, typename TS, typename TC, typename TW, bool FUSE, bool GATHER, bool HB,
          bool PF = Shape<LX>::kPrefetch, int TPE = LX * LX>
__global__ void __launch_bounds__(EPB * TPE) __attribute__((amdgpu_waves_per_eu(Shape<LX>::kWavesPerEU, 8)))
ax_kernel(TW* __restrict__ w, const TU* __restrict__ u,
          const TC* __restrict__ dx, const TC* __restrict__ dy, const TC* __restrict__ dz,
          const TC* __restrict__ dxt, const TC* __restrict__ dyt, const TC* __restrict__ dzt,
          const TS* __restrict__ h1, const TS* __restrict__ g11, const TS* __restrict__ g22,
          const TS* __restrict__ g33, const TS* __restrict__ g12, const TS* __restrict__ g13,
          const TS* __restrict__ g23, int64_t nel, const int* __restrict__ skip,
          double* __restrict__ dot, const int32_t* __restrict__ lid,
          const TS* __restrict__ gp, const TS* __restrict__ hb) {
    constexpr int L2 = LX * LX;
    constexpr int L3 = L2 * LX;
    constexpr bool WP = (64 % TPE) == 0;
    static_assert(TPE >= L2, "threads per element");
    constexpr bool NT = GATHER || kStreamNT<LX, TS>;
    if (skip && *skip) return;
    __shared__ TC s_u[EPB * L3];               // the element's u (wave-private: then the r-flux)
    __shared__ TC s_s[EPB * L3];               // s-flux
    // Elements spanning waves write the r-flux of slice k over slice k of u
    // after a workgroup barrier (every wave has read it) instead of into a third
    // array, where the LDS this frees admits one more workgroup per CU
    // (lx = 7: 3 -> 4, lx = 9 and 11: 2 -> 3, 4-5 % faster at lx 9 and 11;
    // lx = 12 with its register floor: 3 -> 4).  At the other lx the
    // registers, not the LDS, cap the workgroups, and the barrier per slice
    // would cost without a gain.
    constexpr bool ALIAS = !WP && (LX == 7 || LX == 9 || LX == 11 || LX == 12);
    __shared__ TC s_r0[(WP || ALIAS) ? 1 : EPB * L3];     // r-flux when elements span waves
    __shared__ TC s_d[6 * L2];                 // dx, dy, dz, dxt, dyt, dzt

    const int tid = threadIdx.x;
    const int el = tid / TPE;
    const int ijr = tid - el * TPE;
    const bool act = TPE == L2 || ijr < L2;    // a lane with a column
    const int ij = act ? ijr : 0;
    const int i = ij % LX;
    const int j = ij / LX;
    const int64_t e = (int64_t)blockIdx.x * EPB + el;
    const bool live = act && e < nel;
    const int64_t base = e * L3 + ij;
    TC* su = s_u + el * L3;
    TC* ss = s_s + el * L3;
    TC* sr = (WP || ALIAS) ? su : s_r0 + el * L3;
    const TC* sdz = s_d + 2 * L2;
    const TC* sdzt = s_d + 5 * L2;

    for (int q = tid; q < L2; q += EPB * TPE) {
        s_d[q] = dx[q];
        s_d[L2 + q] = dy[q];
        s_d[2 * L2 + q] = dz[q];
        s_d[3 * L2 + q] = dxt[q];
        s_d[4 * L2 + q] = dyt[q];
        s_d[5 * L2 + q] = dzt[q];
    }

    // the thread's column of u, kept in registers for the t-derivative
    TC uc[LX];
#pragma unroll
    for (int k = 0; k < LX; ++k) {
        if constexpr (GATHER) {
            const int32_t q = live ? __builtin_nontemporal_load(lid + base + k * L2) : -1;
            uc[k] = q >= 0 ? (TC)u[q] : TC(0);
        }
        else
            uc[k] = live ? (TC)ld<NT>(u, base + k * L2) : TC(0);
    }
    if (act) {
#pragma unroll
        for (int k = 0; k < LX; ++k) su[k * L2 + ij] = uc[k];
    }
    __syncthreads();   // s_d is shared by every wave of the workgroup

    // The float64 solver form at lx = 8 reads the j-direction rows of D from LDS
    // instead of keeping them in registers: 138 -> 122 VGPRs, four waves per
    // SIMD instead of three, and the float64 PCG iteration 436 -> 418 us at 32^3.
    // The public form measured the same either way (188.1 us) and the float32
    // and bfloat16 forms, already at 64-78 VGPRs, slower, so they keep them.
    constexpr bool DJL = LX == 8 && GATHER && std::is_same<TC, double>::value;
    TC di[LX], dj[DJL ? 1 : LX];
    const TC* sdj = s_d + L2;
#pragma unroll
    for (int l = 0; l < LX; ++l) {
        di[l] = s_d[l * LX + i];
        if constexpr (!DJL) dj[l] = s_d[L2 + l * LX + j];
    }

    // forward passes slice by slice; the t-flux of slice k is folded straight
    // into the transposed t-sum: wt[m] += dzt[k, m] * vt_k
    TC wt[LX];
#pragma unroll
    for (int m = 0; m < LX; ++m) wt[m] = 0;
    TC ng[6], nh;                              // the next slice's factors (prefetch)
    if constexpr (PF) load_factors<TS, TC, GATHER, NT>(ng, nh, live, base, ij, L2, h1, g11, g22, g33, g12, g13, g23, gp);
#pragma unroll 1
    for (int k = 0; k < LX; ++k) {
        const int64_t o = base + k * L2;
        TC g[6], H;
        if constexpr (PF) {
#pragma unroll
            for (int a = 0; a < 6; ++a) g[a] = ng[a];
            H = nh;
            if (k + 1 < LX)
                load_factors<TS, TC, GATHER, NT>(ng, nh, live, o + L2, ij, L2, h1, g11, g22, g33, g12, g13, g23, gp);
        } else {
            load_factors<TS, TC, GATHER, NT>(g, H, live, o, ij, L2, h1, g11, g22, g33, g12, g13, g23, gp);
        }
        TC r = 0, s = 0, t = 0;
#pragma unroll
        for (int l = 0; l < LX; ++l) {
            r += di[l] * su[k * L2 + j * LX + l];
            s += (DJL ? sdj[l * LX + j] : dj[DJL ? 0 : l]) * su[k * L2 + l * LX + i];
            t += sdz[l * LX + k] * uc[l];
        }
        const TC G11 = g[0], G22 = g[1], G33 = g[2], G12 = g[3], G13 = g[4], G23 = g[5];
        const TC vr = H * (G11 * r + G12 * s + G13 * t);
        const TC vs = H * (G12 * r + G22 * s + G23 * t);
        const TC vt = H * (G13 * r + G23 * s + G33 * t);
        if (WP) wave_sync();   // every lane has read slice k before it is overwritten
        else if (ALIAS) __syncthreads();
        if (act) {
            sr[k * L2 + ij] = vr;
            ss[k * L2 + ij] = vs;
        }
#pragma unroll
        for (int m = 0; m < LX; ++m) wt[m] += sdzt[k * LX + m] * vt;
    }
    if (WP) wave_sync(); else __syncthreads();

#pragma unroll
    for (int l = 0; l < LX; ++l) {
        di[l] = s_d[3 * L2 + l * LX + i];
        if constexpr (!DJL) dj[l] = s_d[4 * L2 + l * LX + j];
    }
    double pw = 0.0;
#pragma unroll
    for (int k = 0; k < LX; ++k) {
        TC acc = wt[k];
#pragma unroll
        for (int l = 0; l < LX; ++l) {
            acc += di[l] * sr[k * L2 + j * LX + l];
            acc += (DJL ? s_d[4 * L2 + l * LX + j] : dj[DJL ? 0 : l]) * ss[k * L2 + l * LX + i];
        }
        if (live) {
            if constexpr (HB) acc += ld<NT>(hb, base + k * L2) * uc[k];   // Helmholtz: + h2 B u
            st<NT>(w, base + k * L2, (TW)acc);
        }
        if (FUSE) pw += (double)uc[k] * (double)(TW)acc;
    }
    if constexpr (FUSE) block_dot<EPB * TPE>(pw, dot);
}

// ---- the operator on whole elements and matrix cores -------------------------
// Each derivative is a product of the lx x lx matrix with the element's lines:
// out[q][line] = sum_l D[l][q] in[l][line].  A wave takes 16 lines at a time as
// the columns of 16x16x4 MFMA blocks; lane (n, g), n = lane % 16, g = lane / 16,
// feeds in[4 s + g][line n] in step s and receives out[4 r + g][line n] in
// register r.  Every value passes LDS once per direction and product instead of
// being read 2 lx times by the column mapping, and no thread owns a node: the
// streamed arrays are read and written in memory order, V neighbouring nodes a lane
// from the workgroup's first node on, all of them issued at the start.
// What bounded the column mapping: at lx = 12 its 6 lx LDS reads per node (557 us
// of 775 at 32768 elements), elsewhere slices that are no whole lines (lx 5, 6, 7,
// 9, 10, 11) and loads of 2 and 4 bytes a lane.  Per 16.8M nodes with h1, column
// mapping against this kernel: float64 lx 5 231 / 205, lx 6 225 / 191, lx 12
// 232 / 203 us (6.0 TB/s); float32 lx 4 120 / 103, 5 134 / 105, 6 126 / 98,
// 7 124 / 106, 10 126 / 105, 12 130 / 104; bfloat16 lx 4 87 / 59, 5 96 / 77, 6 97 / 69,
// 7 109 / 74, 8 100 / 59, 9 123 / 86, 10 138 / 71, 11 147 / 83, 12 165 / 73.
typedef double mvec4d __attribute__((ext_vector_type(4)));
typedef float mvec4f __attribute__((ext_vector_type(4)));
template <typename TC> struct Mfma;
template <> struct Mfma<double> {
    typedef mvec4d acc;
    // logical row of A's lane n: the result's register r of group g is row 4 r + g
    __device__ static int row(int n) { return n; }
    __device__ static acc mul(double a, double b, acc c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
};
template <> struct Mfma<float> {
    typedef mvec4f acc;
    // the float32 block returns row 4 g + r there: A's rows are permuted to match
    __device__ static int row(int n) { return 4 * (n & 3) + (n >> 2); }
    __device__ static acc mul(float a, float b, acc c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
};

// Where it is the built-in kernel.  The column mapping stays where it measured no
// slower throughout: float64 lx 4 (194 against 195 us), 7 (224 / 242), 8 (187 / 188),
// 9 (224 / 242), 10 (223 / 211, but 21.9 / 22.5 us at 1500 elements), 11 (224 / 273);
// float32 lx 8 (100 / 101), 9 (131 / 123, but 11.0 / 12.9 at 1500 elements) and 11
// (127 / 126, 16.6 / 18.4).  The matrix blocks pad lx to a multiple of 4, which is what
// the odd orders pay for.
template <int LX, typename TS>
constexpr bool kFlat = std::is_same<TS, double>::value ? (LX == 5 || LX == 6 || LX == 12)
                     : std::is_same<TS, float>::value ? (LX >= 4 && LX != 8 && LX != 9 && LX != 11) : LX >= 4;

// Where it is that at every size; the others of kFlat take it for large arrays
// (flat_pays).  On the same arrays again and again, column / whole elements, us:
// float64 lx 12 at 64 elements 10.7 / 5.9, 512 17.1 / 12.5, 1000 25.1 / 24.8, 4000 106 / 89;
// float32 lx 10 at 64 7.0 / 6.3, 65 7.0 / 6.4, 1000 11.8 / 10.1, 3375 30.2 / 24.6; lx 12 at
// 64 8.5 / 5.9, 3375 47 / 39; bfloat16 lx 8 at 64 6.2 / 4.3, 67 6.2 / 4.7, 1001 7.0 / 4.6,
// 3375 10.7 / 9.0; lx 9 at 64 8.8 / 7.3, 67 8.8 / 8.4, 3375 20.6 / 19.1; lx 10 to 12 further
// apart.
template <int LX, typename TS>
constexpr bool kFlatAlways = kFlat<LX, TS> && LX > 7;

// Where the solver form takes it: not at lx = 4, 5 and float32 lx = 7, where the gather
// hides what the accesses gain (one conjugate-gradient iteration, column / whole
// elements, us: float64 lx 5 26.8 / 30.0 at 16^3 elements, float32 lx 5 47.1 / 49.5 at
// 26^3, lx 7 36.9 / 39.1 at 16^3, bfloat16 lx 5 42.1 / 46.8 at 26^3).  By the order alone,
// which the layout of its factors follows: at lx = 6 and bfloat16 lx = 7 it leads below
// and above a stretch of some 2000 to 9000 elements, in which its fewer and larger
// workgroups fill the chip in the coarser steps.  Float64 lx 6 17.6 / 15.6 at 6^3,
// 23.2 / 22.6 at 12^3, 32.3 / 33.9 at 15^3, 44.7 / 47.6 at 19^3 (the worst), 52.8 / 49.6
// at 20^3, 77.2 / 77.3 at 24^3, 160 / 154 at 32^3; float32 lx 6 21.3 / 19.6 at 12^3,
// 27.7 / 27.6 at 15^3, 42.5 / 43.9 at 22^3, 54.5 / 51.9 at 24^3, 98.1 / 93.1 at 32^3;
// bfloat16 lx 6 29.5 / 27.9 at 16^3, 37.9 / 39.2 at 21^3, 52.5 / 47.4 at 24^3, lx 7
// 29.5 / 26.3 at 12^3, 41.4 / 43.6 at 19^3, 56.0 / 51.2 at 21^3.  The orders above lead
// nearly everywhere: float64 lx 12 46.7 / 42.2 at 9^3, 120 / 102 at 13^3; float32 lx 10
// 32.6 / 28.3 at 9^3, 73.7 / 66.3 at 16^3; bfloat16 lx 8 24.2 / 18.3 at 9^3, 55.7 / 55.4 at
// 20^3, lx 9 48.0 / 47.4 at 15^3, 81.1 / 73.9 at 19^3, lx 12 78.2 / 59.5 at 13^3.
template <int LX, typename TS>
constexpr bool kFlatSolver = kFlat<LX, TS> && (LX > 7 || LX == 6 || (LX == 7 && std::is_same<TS, uint16_t>::value));

// EPB elements per workgroup of NW waves, V nodes per access (V divides the
// workgroup's nodes): two or three accesses per thread and array, and workgroups
// that fill the 16 waves that four per SIMD allow (six waves leave four idle:
// float32 lx = 9 measured 145 us with six and 123 with eight)
template <int LX, bool F64> struct ShapeF;
template <int LX> struct ShapeF<LX, true> {
    static constexpr int EPB = LX == 5 ? 8 : LX == 6 ? 4 : 1;
    static constexpr int NW = LX == 12 ? 8 : 4;
    static constexpr int V = 2;
};
template <int LX> struct ShapeF<LX, false> {
    static constexpr int EPB = LX == 4 ? 32 : LX == 5 ? 16 : LX == 6 ? 8 : LX <= 9 ? 4 : 2;
    static constexpr int NW = LX == 7 ? 3 : LX == 9 ? 8 : LX == 11 ? 7 : LX == 12 ? 8 : 4;
    static constexpr int V = LX == 11 ? 2 : 4;
};

// The waves per SIMD that its registers have to leave room for.  bfloat16 lx 9 and 12 run
// workgroups of eight waves, of which 81 registers leave room for two a CU and 80 for
// three: 139 and 243 us without this at 32768 elements, 120 and 234 with it.
template <int LX, typename TS, bool HB>
constexpr int min_waves = !std::is_same<TS, uint16_t>::value || LX == 4 ? 4 : (LX == 9 || LX == 12) && !HB ? 6 : 5;

template <bool WP>
__device__ __forceinline__ void element_sync() {
    if (WP) wave_sync();
    else __syncthreads();
}

template <int LX, int EPB, int NW, int V, typename TU, typename TS, typename TC, typename TW, bool FUSE, bool GATHER,
          bool HB>
__global__ void __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(min_waves<LX, TS, HB>, 8)))
ax_flat_kernel(TW* __restrict__ w, const TU* __restrict__ u,
               const TC* __restrict__ dx, const TC* __restrict__ dy, const TC* __restrict__ dz,
               const TC* __restrict__ dxt, const TC* __restrict__ dyt, const TC* __restrict__ dzt,
               const TS* __restrict__ h1, const TS* __restrict__ g11, const TS* __restrict__ g22,
               const TS* __restrict__ g33, const TS* __restrict__ g12, const TS* __restrict__ g13,
               const TS* __restrict__ g23, int64_t nel, const int* __restrict__ skip,
               double* __restrict__ dot, const int32_t* __restrict__ lid, const TS* __restrict__ hb) {
    typedef typename Mfma<TC>::acc acc_t;
    constexpr int L2 = LX * LX, L3 = L2 * LX, C = EPB * L2, N = EPB * L3;
    constexpr int KS = (LX + 3) / 4;
    constexpr int T = NW * 64, NQ = (N + V * T - 1) / (V * T);
    constexpr int TILES = (C + 15) / 16;
    // whole elements per wave, its nodes and its lines: no workgroup barriers
    constexpr bool WP = N == V * T * NQ && (V * 64 * NQ) % L3 == 0 && TILES * 16 == C && TILES % NW == 0;
    typedef TS vec_s __attribute__((ext_vector_type(V)));
    typedef TU vec_u __attribute__((ext_vector_type(V)));
    typedef TC vec_c __attribute__((ext_vector_type(V)));
    typedef TW vec_w __attribute__((ext_vector_type(V)));
    static_assert(N % V == 0, "vectors");
    if (skip && *skip) return;
    __shared__ __attribute__((aligned(16))) TC s_t[N], s_r[N], s_s[N];    // u and the t-direction; r; s
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int n = lane & 15, g = lane >> 4;
    const int64_t e0 = (int64_t)blockIdx.x * EPB, b0 = e0 * L3;           // first element and node of the workgroup
    const int nn = (nel - e0 < EPB ? (int)(nel - e0) : EPB) * L3;         // its nodes

    // A operand of out = D^T in: lane (n, g), step s holds D[4 s + g][row n]
    auto matrix = [&](TC (&a)[KS], const TC* __restrict__ m) {
        const int q = Mfma<TC>::row(n);
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int l = 4 * s + g;
            const bool in = l < LX && q < LX;
            const TC v = m[in ? l * LX + q : 0];
            a[s] = in ? v : TC(0);
        }
    };
    TC ar[KS], as[KS], at[KS];
    matrix(ar, dx);
    matrix(as, dy);
    matrix(at, dz);

    // this thread's vector q starts at node at_node(q)
    auto at_node = [&](int q) { return V * (WP ? (wv * NQ + q) * 64 + lane : q * T + tid); };
    const bool full = nn == N;                 // uniform: all but the mesh's last workgroup
    // Nodes o .. o + V - 1 of an array, without a branch: a vector past the last of the
    // workgroup's nn nodes reads that one, which in the mesh's last workgroup need not
    // start where the thread's does.  place() then moves value i + d to value i, `none`
    // past the end, once every load is under way.  (Loads there under a branch for each
    // value were a chain of waits that a ragged call ended with: bfloat16 lx 8 at 65
    // elements 8.6 us, this 4.6; 64 elements 4.3.)  The type promises the alignment of one
    // value only, which is also all that the solver's float64 h1 and h2 B, the caller's
    // arrays, have; the instruction is the same.
    auto load = [&](const auto* __restrict__ p, int o) {
        typedef std::remove_const_t<std::remove_reference_t<decltype(*p)>> T1;
        typedef T1 vec_1 __attribute__((ext_vector_type(V)));
        typedef T1 vec_any __attribute__((ext_vector_type(V), aligned(sizeof(T1))));
        const vec_1 x = __builtin_nontemporal_load(reinterpret_cast<const vec_any*>(p + b0 + min(o, nn - V)));
        return x;
    };
    auto place = [&](auto& v, int o, auto none) {
        const int d = o - min(o, nn - V);
        const auto x = v;
#pragma unroll
        for (int i = 0; i < V; ++i) {
            v[i] = none;
#pragma unroll
            for (int k = i; k < V; ++k)
                if (k == i + d) v[i] = x[k];
        }
    };
    auto to_c = [](const vec_s& v) {
        vec_c c;
#pragma unroll
        for (int i = 0; i < V; ++i) {
            if constexpr (std::is_same<TS, uint16_t>::value) c[i] = __uint_as_float((uint32_t)v[i] << 16);
            else c[i] = v[i];
        }
        return c;
    };
    vec_c uv[NQ];
    vec_s us[NQ], f11[NQ], f22[NQ], f33[NQ], f12[NQ], f13[NQ], f23[NQ], fh[NQ];
    typedef int32_t vec_i __attribute__((ext_vector_type(V)));
    vec_i id[NQ];
    if constexpr (GATHER)                      // the numbering ahead of the factors, its nodes of u after them
#pragma unroll
        for (int q = 0; q < NQ; ++q) id[q] = load(lid, at_node(q));
    else
#pragma unroll
        for (int q = 0; q < NQ; ++q) us[q] = load(u, at_node(q));
    if (h1)
#pragma unroll
        for (int q = 0; q < NQ; ++q) fh[q] = load(h1, at_node(q));
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int o = at_node(q);
        f11[q] = load(g11, o); f22[q] = load(g22, o); f33[q] = load(g33, o);
        f12[q] = load(g12, o); f13[q] = load(g13, o); f23[q] = load(g23, o);
    }
    if constexpr (GATHER) {
        if (!full)
#pragma unroll
            for (int q = 0; q < NQ; ++q) place(id[q], at_node(q), -1);
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int i = 0; i < V; ++i) uv[q][i] = id[q][i] >= 0 ? (TC)u[id[q][i]] : TC(0);
    }
    __builtin_amdgcn_sched_barrier(0);         // every load is in flight before anything waits
    if (!full) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int o = at_node(q);
            if constexpr (!GATHER) place(us[q], o, 0);
            if (h1) place(fh[q], o, 0);
            place(f11[q], o, 0); place(f22[q], o, 0); place(f33[q], o, 0);
            place(f12[q], o, 0); place(f13[q], o, 0); place(f23[q], o, 0);
        }
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        if constexpr (!GATHER) uv[q] = to_c(us[q]);
        if (at_node(q) < N) *reinterpret_cast<vec_c*>(s_t + at_node(q)) = uv[q];
    }
    element_sync<WP>();

    const bool last = LX % 4 == 0 || 4 * (KS - 1) + g < LX;   // row 4 (KS - 1) + g exists
    auto has = [&](int r) { return r + 1 < KS || last; };
    // one line: out[q] = sum_l D[l][q] in[l], nodes `step` apart
    auto product = [&](const TC (&a)[KS], const TC* in, int step) {
        acc_t c = {0, 0, 0, 0};
        TC b[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const TC v = in[has(s) ? (4 * s + g) * step : 0];
            b[s] = has(s) ? v : TC(0);         // rows past lx: zeros of the matrix times zero
        }
#pragma unroll
        for (int s = 0; s < KS; ++s) c = Mfma<TC>::mul(a[s], b[s], c);
        return c;
    };
    auto put = [&](TC* out, int step, const acc_t& c, bool ok) {
#pragma unroll
        for (int r = 0; r < KS; ++r)
            if (ok && has(r)) out[(4 * r + g) * step] = c[r];
    };
    // the wave's tiles; line c of the r-, s- and t-direction starts at
    auto first_tile = [&]() { return WP ? wv * (TILES / NW) : wv; };
    auto end_tile = [&]() { return WP ? (wv + 1) * (TILES / NW) : TILES; };
    constexpr int STEP = WP ? 1 : NW;
    auto r_at = [&](int c) { return c * LX; };
    auto s_at = [&](int c) { return c / LX * L2 + c % LX; };
    auto t_at = [&](int c) { return c / L2 * L3 + c % L2; };
    for (int t = first_tile(); t < end_tile(); t += STEP) {
        const bool ok = C % 16 == 0 || t * 16 + n < C;
        const int c = ok ? t * 16 + n : C - 1;
        const acc_t vr = product(ar, s_t + r_at(c), 1);
        const acc_t vs = product(as, s_t + s_at(c), LX);
        put(s_r + r_at(c), 1, vr, ok);
        put(s_s + s_at(c), LX, vs, ok);
    }
    matrix(ar, dxt);
    matrix(as, dyt);
    element_sync<WP>();                        // u has been read along r and s
    for (int t = first_tile(); t < end_tile(); t += STEP) {
        const bool ok = C % 16 == 0 || t * 16 + n < C;
        const int c = ok ? t * 16 + n : C - 1;
        put(s_t + t_at(c), L2, product(at, s_t + t_at(c), L2), ok);   // a line's lanes are one wave: in place
    }
    matrix(at, dzt);
    element_sync<WP>();
    double pw = 0.0;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int o = at_node(q);
        if (o >= N) continue;
        vec_c* pr = reinterpret_cast<vec_c*>(s_r + o);
        vec_c* ps = reinterpret_cast<vec_c*>(s_s + o);
        vec_c* pt = reinterpret_cast<vec_c*>(s_t + o);
        const vec_c r = *pr, s = *ps, t = *pt;
        const vec_c G11 = to_c(f11[q]), G22 = to_c(f22[q]), G33 = to_c(f33[q]), G12 = to_c(f12[q]), G13 = to_c(f13[q]),
                    G23 = to_c(f23[q]);
        vec_c H = 1;
        if (h1) H = to_c(fh[q]);
        const vec_c vr = H * (G11 * r + G12 * s + G13 * t);
        const vec_c vs = H * (G12 * r + G22 * s + G23 * t);
        const vec_c vt = H * (G13 * r + G23 * s + G33 * t);
        *pr = vr;
        *ps = vs;
        *pt = vt;
        // p^T A p = (D p)^T v (+ h2 B p^2)
        if constexpr (FUSE)
#pragma unroll
            for (int i = 0; i < V; ++i)
                pw += (double)r[i] * (double)vr[i] + (double)s[i] * (double)vs[i] + (double)t[i] * (double)vt[i];
    }
    element_sync<WP>();
    for (int t = first_tile(); t < end_tile(); t += STEP) {
        const bool ok = C % 16 == 0 || t * 16 + n < C;
        const int c = ok ? t * 16 + n : C - 1;
        const acc_t vr = product(ar, s_r + r_at(c), 1);
        const acc_t vs = product(as, s_s + s_at(c), LX);
        const acc_t vt = product(at, s_t + t_at(c), L2);
        put(s_r + r_at(c), 1, vr, ok);
        put(s_s + s_at(c), LX, vs, ok);
        put(s_t + t_at(c), L2, vt, ok);
    }
    element_sync<WP>();
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int o = at_node(q);
        if (o >= nn) continue;
        vec_c v = *reinterpret_cast<const vec_c*>(s_t + o) + *reinterpret_cast<const vec_c*>(s_r + o) +
                  *reinterpret_cast<const vec_c*>(s_s + o);
        if constexpr (HB) {                    // Helmholtz: + h2 B u
            vec_s b = load(hb, o);
            if (!full) place(b, o, 0);
            const vec_c m = to_c(b) * uv[q];
            if constexpr (FUSE)
#pragma unroll
                for (int i = 0; i < V; ++i) pw += (double)m[i] * (double)uv[q][i];
            v += m;
        }
        vec_w x;
#pragma unroll
        for (int i = 0; i < V; ++i) x[i] = (TW)v[i];
        if (full) {
            vec_w* d = reinterpret_cast<vec_w*>(w + b0 + o);
            __builtin_nontemporal_store(x, d);
        } else {
#pragma unroll
            for (int i = 0; i < V; ++i)
                if (o + i < nn) w[b0 + o + i] = x[i];
        }
    }
    if constexpr (FUSE) block_dot<T>(pw, dot);
}

// Slice-pipelined column mapping: one thread per (i, j) column as in
// ax_kernel, but the element passes through LDS one k-slice at a time.  Slice
// k of u and the r- and s-fluxes of slice k - 1 sit in double buffers, so each
// slice costs one workgroup barrier, and LDS holds 6 lx^2 values per element
// instead of ax_kernel's 2-3 lx^3: large elements keep several times more
// waves in flight.  Register arrays are indexed by the run-time slice only
// through selects, so they stay in registers.  Plain (public) form only.
template <int LX> struct ShapeSlice {
    static constexpr int EPB = (512 / (LX * LX)) < 1 ? 1 : 512 / (LX * LX);
};

template <int LX, int EPB, typename TS, typename TC, typename TW, bool HB>
__global__ void __launch_bounds__(EPB * LX * LX)
ax_slice_kernel(TW* __restrict__ w, const TS* __restrict__ u,
                const TC* __restrict__ dx, const TC* __restrict__ dy, const TC* __restrict__ dz,
                const TC* __restrict__ dxt, const TC* __restrict__ dyt, const TC* __restrict__ dzt,
                const TS* __restrict__ h1, const TS* __restrict__ g11, const TS* __restrict__ g22,
                const TS* __restrict__ g33, const TS* __restrict__ g12, const TS* __restrict__ g13,
                const TS* __restrict__ g23, int64_t nel, const TS* __restrict__ hb) {
    constexpr int L2 = LX * LX;
    constexpr int L3 = L2 * LX;
    constexpr int NS = EPB * L2;
    constexpr bool NT = kStreamNT<LX, TS>;
    __shared__ TC s_d[6 * L2];
    __shared__ TC s_u[2][NS];
    __shared__ TC s_r[2][NS];
    __shared__ TC s_s[2][NS];
    const int tid = threadIdx.x;
    const int el = tid / L2;
    const int ij = tid - el * L2;
    const int i = ij % LX;
    const int j = ij / LX;
    const int64_t e = (int64_t)blockIdx.x * EPB + el;
    const bool live = e < nel;
    const int64_t base = e * L3 + ij;
    const int off = el * L2;
    for (int q = tid; q < L2; q += NS) {
        s_d[q] = dx[q];
        s_d[L2 + q] = dy[q];
        s_d[2 * L2 + q] = dz[q];
        s_d[3 * L2 + q] = dxt[q];
        s_d[4 * L2 + q] = dyt[q];
        s_d[5 * L2 + q] = dzt[q];
    }
    TC uc[LX];
#pragma unroll
    for (int k = 0; k < LX; ++k) uc[k] = live ? (TC)ld<NT>(u, base + k * L2) : TC(0);
    s_u[0][off + ij] = uc[0];
    __syncthreads();
    TC di[LX], dj[LX], ti[LX], tj[LX];
#pragma unroll
    for (int l = 0; l < LX; ++l) {
        di[l] = s_d[l * LX + i];
        dj[l] = s_d[L2 + l * LX + j];
        ti[l] = s_d[3 * L2 + l * LX + i];
        tj[l] = s_d[4 * L2 + l * LX + j];
    }
    const TC* sdz = s_d + 2 * L2;
    const TC* sdzt = s_d + 5 * L2;
    TC wt[LX];
#pragma unroll
    for (int m = 0; m < LX; ++m) wt[m] = 0;
    // iteration k: the forward passes of slice k (k < LX) and the transposed
    // r- and s-sums of slice k - 1 (k > 0)
#pragma unroll 1
    for (int k = 0; k <= LX; ++k) {
        if (k > 0) __syncthreads();
        const int b = k & 1;
        TC vr = 0, vs = 0;
        if (k < LX) {
            TC g[6], H;
            load_factors<TS, TC, false, NT>(g, H, live, base + k * L2, ij, L2, h1, g11, g22, g33, g12, g13, g23,
                                            nullptr);
            TC r = 0, s = 0, t = 0;
#pragma unroll
            for (int l = 0; l < LX; ++l) {
                r += di[l] * s_u[b][off + j * LX + l];
                s += dj[l] * s_u[b][off + l * LX + i];
                t += sdz[l * LX + k] * uc[l];
            }
            vr = H * (g[0] * r + g[3] * s + g[4] * t);
            vs = H * (g[3] * r + g[1] * s + g[5] * t);
            const TC vt = H * (g[4] * r + g[5] * s + g[2] * t);
#pragma unroll
            for (int m = 0; m < LX; ++m) wt[m] += sdzt[k * LX + m] * vt;
        }
        if (k > 0) {
            const int pb = b ^ 1;
            TC acc = 0;
#pragma unroll
            for (int l = 0; l < LX; ++l) {
                acc += ti[l] * s_r[pb][off + j * LX + l];
                acc += tj[l] * s_s[pb][off + l * LX + i];
            }
#pragma unroll
            for (int m = 0; m < LX; ++m) wt[m] += (m == k - 1) ? acc : TC(0);
        }
        if (k < LX) {
            s_r[b][off + ij] = vr;
            s_s[b][off + ij] = vs;
            TC nx = 0;
#pragma unroll
            for (int m = 1; m < LX; ++m) nx = (m == k + 1) ? uc[m] : nx;
            if (k + 1 < LX) s_u[b ^ 1][off + ij] = nx;
        }
    }
    if (live) {
#pragma unroll
        for (int k = 0; k < LX; ++k) {
            TC acc = wt[k];
            if constexpr (HB) acc += ld<NT>(hb, base + k * L2) * uc[k];   // Helmholtz: + h2 B u
            st<NT>(w, base + k * L2, (TW)acc);
        }
    }
}

// One thread per node ("3D" mapping): every load and store of the streamed
// arrays is contiguous across the workgroup.  u and the three fluxes go
// through LDS; each thread keeps the derivative-matrix rows it needs (its i,
// j, k) in registers.  One of the variants the run-time tuning times; with
// the cached streaming of the column mapping it is the slower one at every lx
// measured (lx = 3: 18.1 against 13.9 us at 32768 elements).
template <int LX> struct Shape3D {
    // whole elements per workgroup of at most 1024 threads (none above lx = 10)
    static constexpr int EPB = LX == 3 ? 16 : (1024 / (LX * LX * LX));
};

template <int LX, int EPB, typename TS, typename TC, typename TW, bool HB>
__global__ void __launch_bounds__(EPB * LX * LX * LX)
ax3d_kernel(TW* __restrict__ w, const TS* __restrict__ u,
            const TC* __restrict__ dx, const TC* __restrict__ dy, const TC* __restrict__ dz,
            const TC* __restrict__ dxt, const TC* __restrict__ dyt, const TC* __restrict__ dzt,
            const TS* __restrict__ h1, const TS* __restrict__ g11, const TS* __restrict__ g22,
            const TS* __restrict__ g33, const TS* __restrict__ g12, const TS* __restrict__ g13,
            const TS* __restrict__ g23, int64_t nel, const TS* __restrict__ hb) {
    constexpr int L2 = LX * LX;
    constexpr int L3 = L2 * LX;
    __shared__ TC s_u[EPB * L3];
    __shared__ TC s_r[EPB * L3];
    __shared__ TC s_s[EPB * L3];
    __shared__ TC s_t[EPB * L3];
    const int tid = threadIdx.x;
    const int el = tid / L3;
    const int p = tid - el * L3;
    const int i = p % LX, j = (p / LX) % LX, k = p / L2;
    const int64_t e = (int64_t)blockIdx.x * EPB + el;
    const bool live = e < nel;
    const int64_t g = e * L3 + p;               // contiguous across the workgroup
    TC* su = s_u + el * L3;
    TC* sr = s_r + el * L3;
    TC* ss = s_s + el * L3;
    TC* st = s_t + el * L3;
    TC uv = 0, G11 = 0, G22 = 0, G33 = 0, G12 = 0, G13 = 0, G23 = 0, H = 1;
    if (live) {
        uv = Load<TS>::get(u, g);
        G11 = Load<TS>::get(g11, g); G22 = Load<TS>::get(g22, g); G33 = Load<TS>::get(g33, g);
        G12 = Load<TS>::get(g12, g); G13 = Load<TS>::get(g13, g); G23 = Load<TS>::get(g23, g);
        if (h1) H = Load<TS>::get(h1, g);
    }
    su[p] = uv;
    TC di[LX], dj[LX], dk[LX];
#pragma unroll
    for (int l = 0; l < LX; ++l) {
        di[l] = dx[l * LX + i];
        dj[l] = dy[l * LX + j];
        dk[l] = dz[l * LX + k];
    }
    __syncthreads();
    TC r = 0, s = 0, t = 0;
#pragma unroll
    for (int l = 0; l < LX; ++l) {
        r += di[l] * su[k * L2 + j * LX + l];
        s += dj[l] * su[k * L2 + l * LX + i];
        t += dk[l] * su[l * L2 + j * LX + i];
    }
    sr[p] = H * (G11 * r + G12 * s + G13 * t);
    ss[p] = H * (G12 * r + G22 * s + G23 * t);
    st[p] = H * (G13 * r + G23 * s + G33 * t);
#pragma unroll
    for (int l = 0; l < LX; ++l) {
        di[l] = dxt[l * LX + i];
        dj[l] = dyt[l * LX + j];
        dk[l] = dzt[l * LX + k];
    }
    __syncthreads();
    TC acc = 0;
#pragma unroll
    for (int l = 0; l < LX; ++l) {
        acc += di[l] * sr[k * L2 + j * LX + l];
        acc += dj[l] * ss[k * L2 + l * LX + i];
        acc += dk[l] * st[l * L2 + j * LX + i];
    }
    if constexpr (HB) if (live) acc += Load<TS>::get(hb, g) * uv;   // Helmholtz: + h2 B u
    if (live) store_nt(w, g, (TW)acc);
}

// values between the planes of a solver copy of n nodes: 16-byte steps in every type
constexpr int64_t plane_stride(int64_t n) { return (n + 7) / 8 * 8; }

// The Helmholtz term is a template flag (HB), so that the two forms are
// separate kernels (and separate rows of a kernel trace).
// the float64 public form's kernel variants (SEM_AX_* of sem.h)
constexpr bool variant_exists(int lx, int v) {
    return v == SEM_AX_COLUMN || v == SEM_AX_COLUMN_PF || v == SEM_AX_SLICE || (v == SEM_AX_3D && lx <= 10) ||
           (v == SEM_AX_WAVE && (lx == 3 || lx == 5 || lx == 6 || lx == 7));
}

template <int LX, typename TS, typename TC, typename TW, bool HB, bool PF>
void launch_column(sem_ctx_t ctx, void* w, const void* u, const void* const* D, const void* h1,
                   const void* const* G, int64_t nel, const void* hb) {
    constexpr int EPB = Shape<LX>::EPB;
    ax_kernel<LX, EPB, TS, TS, TC, TW, false, false, HB, PF><<<(unsigned)((nel + EPB - 1) / EPB), EPB * LX * LX, 0,
                                                               ctx->stream>>>(
        (TW*)w, (const TS*)u, (const TC*)D[0], (const TC*)D[1], (const TC*)D[2], (const TC*)D[3], (const TC*)D[4],
        (const TC*)D[5], (const TS*)h1, (const TS*)G[0], (const TS*)G[1], (const TS*)G[2], (const TS*)G[3],
        (const TS*)G[4], (const TS*)G[5], nel, nullptr, nullptr, nullptr, nullptr, (const TS*)hb);
}

template <int LX, typename TS, typename TC, typename TW, bool HB>
void launch_3d(sem_ctx_t ctx, void* w, const void* u, const void* const* D, const void* h1,
               const void* const* G, int64_t nel, const void* hb) {
    if constexpr (Shape3D<LX>::EPB >= 1) {
        constexpr int E3 = Shape3D<LX>::EPB;
        ax3d_kernel<LX, E3, TS, TC, TW, HB><<<(unsigned)((nel + E3 - 1) / E3), E3 * LX * LX * LX, 0, ctx->stream>>>(
            (TW*)w, (const TS*)u, (const TC*)D[0], (const TC*)D[1], (const TC*)D[2], (const TC*)D[3],
            (const TC*)D[4], (const TC*)D[5], (const TS*)h1, (const TS*)G[0], (const TS*)G[1],
            (const TS*)G[2], (const TS*)G[3], (const TS*)G[4], (const TS*)G[5], nel, (const TS*)hb);
    }
}

// The short orders take whole elements only for arrays well beyond the 256 MB
// last-level cache.  Within it a call on arrays just used finds them there, and the
// column mapping, whose smaller workgroups then set the pace and whose accesses go
// through the caches at these orders, is the faster.  Column / whole elements, us, on
// the same arrays again and again: float64 lx 5 at 16000 elements (144 MB) 25.2 / 28.2,
// at 32768 (295 MB) 52.9 / 54.2, at 40000 (360 MB) 70.3 / 65.2; lx 6 at 16000 (249 MB)
// 38.7 / 42.0, at 24000 (373 MB) 74.6 / 62.4; float32 lx 4 at 65536 (151 MB) 23.7 / 26.1;
// lx 5 at 32768 (147 MB) 26.6 / 29.2, at 65536 (295 MB) 61.4 / 53.8; lx 6 at 32768 (255 MB)
// 42.6 / 44.9, at 40000 (311 MB) 63.7 / 54.0; lx 7 at 16000 (198 MB) 33.9 / 37.5, at 24000
// (296 MB) 57.7 / 54.5; bfloat16 lx 5 at 65536 (147 MB) 37.8 / 40.3.  On arrays from
// memory whole elements lead from about 110 MB on (float64 lx 6 at 8000, 124 MB: 29.9 /
// 27.2), but by less.  bfloat16 lx 6 and 7 turn at about 40 MB (lx 6: 8000 elements,
// 31 MB, 10.8 / 11.3, 13000, 51 MB, 17.5 / 15.8; lx 7: 3000, 19 MB, 9.9 / 10.2, 8000,
// 49 MB, 20.1 / 16.6), lx 4 too (32768, 38 MB, 10.7 / 9.8), where the line is as for lx 5.
// With the mass term these two lead from 40 MB on for arrays from memory (lx 6 at 16000
// 27.3 / 21.2, lx 7 43.7 / 33.3, at 65536 88 / 68 and 138 / 114), but trail by 3 to 6 % on
// the same arrays up to 200 MB (lx 6 at 16000 19.7 / 20.4, at 40000 40.7 / 43.1, at 65536
// 85 / 67; lx 7 at 28000 49.1 / 51.9, at 32768 63.3 / 59.8): the larger gain sets the line.
template <int LX, typename TS, bool HB>
bool flat_pays(int64_t nel) {
    constexpr int64_t kLeast = (int64_t)(std::is_same<TS, uint16_t>::value && LX >= 6 ? 40 : 320) << 20;
    return kFlatAlways<LX, TS> || nel * (LX * LX * LX) * (9 + HB) * (int64_t)sizeof(TS) >= kLeast;
}

// Whole elements also ask for alignment: accesses are V values wide, so every array it
// streams has to lie on that (any array of torch or hipMalloc does; a view into one
// may not, and takes the column mapping).  The solver form has no such rule: its arrays
// are the library's own but for float64 h1 and h2 B, whose loads ask for one value's.
template <int LX, typename TS, typename TW>
bool flat_aligned(const void* w, const void* u, const void* h1, const void* const* G, const void* hb) {
    constexpr int V = ShapeF<LX, std::is_same<TS, double>::value>::V;
    uintptr_t bits = (uintptr_t)u | (uintptr_t)h1 | (uintptr_t)hb;
    for (int q = 0; q < 6; ++q) bits |= (uintptr_t)G[q];
    return bits % (V * sizeof(TS)) == 0 && (uintptr_t)w % (V * sizeof(TW)) == 0;
}

// whether the built-in kernel of the public form takes whole elements for this call
template <int LX, typename TS, typename TW, bool HB>
bool takes_flat(const void* w, const void* u, const void* h1, const void* const* G, int64_t nel, const void* hb) {
    if constexpr (!kFlat<LX, TS>) return false;
    else return nel <= 0x7fffffff && flat_pays<LX, TS, HB>(nel) && flat_aligned<LX, TS, TW>(w, u, h1, G, hb);
}

template <int LX, typename TU, typename TS, typename TC, typename TW, bool FUSE, bool GATHER, bool HB>
void launch_flat(sem_ctx_t ctx, void* w, const void* u, const void* const* D, const void* h1, const void* const* G,
                 int64_t nel, const int* skip, double* dot, const int32_t* lid, const void* hb) {
    typedef ShapeF<LX, std::is_same<TS, double>::value> F;
    ax_flat_kernel<LX, F::EPB, F::NW, F::V, TU, TS, TC, TW, FUSE, GATHER, HB>
        <<<(unsigned)((nel + F::EPB - 1) / F::EPB), F::NW * 64, 0, ctx->stream>>>(
            (TW*)w, (const TU*)u, (const TC*)D[0], (const TC*)D[1], (const TC*)D[2], (const TC*)D[3], (const TC*)D[4],
            (const TC*)D[5], (const TS*)h1, (const TS*)G[0], (const TS*)G[1], (const TS*)G[2], (const TS*)G[3],
            (const TS*)G[4], (const TS*)G[5], nel, skip, dot, lid, (const TS*)hb);
}

// a non-default variant of the float64 public form; false if it does not exist
template <int LX, typename TS, typename TC, typename TW, bool HB>
bool launch_variant(sem_ctx_t ctx, int variant, void* w, const void* u, const void* const* D, const void* h1,
                    const void* const* G, int64_t nel, const void* hb) {
    if constexpr (!std::is_same<TS, double>::value) {
        return false;
    } else {
        if (variant == SEM_AX_COLUMN_PF) {
            launch_column<LX, TS, TC, TW, HB, !Shape<LX>::kPrefetch>(ctx, w, u, D, h1, G, nel, hb);
            return true;
        }
        if (variant == SEM_AX_COLUMN) {
            launch_column<LX, TS, TC, TW, HB, Shape<LX>::kPrefetch>(ctx, w, u, D, h1, G, nel, hb);
            return true;
        }
        if (variant == SEM_AX_SLICE) {
            constexpr int ES = ShapeSlice<LX>::EPB;
            ax_slice_kernel<LX, ES, TS, TC, TW, HB><<<(unsigned)((nel + ES - 1) / ES), ES * LX * LX, 0, ctx->stream>>>(
                (TW*)w, (const TS*)u, (const TC*)D[0], (const TC*)D[1], (const TC*)D[2], (const TC*)D[3],
                (const TC*)D[4], (const TC*)D[5], (const TS*)h1, (const TS*)G[0], (const TS*)G[1],
                (const TS*)G[2], (const TS*)G[3], (const TS*)G[4], (const TS*)G[5], nel, (const TS*)hb);
            return true;
        }
        if constexpr (LX == 3 || LX == 5 || LX == 6 || LX == 7) {
            if (variant == SEM_AX_WAVE) {      // lx^2 columns padded to 16, 32 or 64 lanes
                constexpr int TPE = LX == 3 ? 16 : LX == 5 ? 32 : 64;
                constexpr int EW = 256 / TPE;
                ax_kernel<LX, EW, TS, TS, TC, TW, false, false, HB, Shape<LX>::kPrefetch, TPE>
                    <<<(unsigned)((nel + EW - 1) / EW), EW * TPE, 0, ctx->stream>>>(
                        (TW*)w, (const TS*)u, (const TC*)D[0], (const TC*)D[1], (const TC*)D[2], (const TC*)D[3],
                        (const TC*)D[4], (const TC*)D[5], (const TS*)h1, (const TS*)G[0], (const TS*)G[1],
                        (const TS*)G[2], (const TS*)G[3], (const TS*)G[4], (const TS*)G[5], nel, nullptr, nullptr,
                        nullptr, nullptr, (const TS*)hb);
                return true;
            }
        }
        if (variant == SEM_AX_3D && LX != 3 && LX <= 10) {
            launch_3d<LX, TS, TC, TW, HB>(ctx, w, u, D, h1, G, nel, hb);
            return true;
        }
        return false;
    }
}

template <int LX, typename TU, typename TS, typename TC, typename TW, bool HB>
int launch_form(sem_ctx_t ctx, void* w, const void* u, const void* const* D, const void* h1,
                const void* const* G, int64_t nel, const int* skip, double* dot, const int32_t* lid,
                const void* gp, const void* hb, int variant) {
    constexpr int EPB = Shape<LX>::EPB;
    const int64_t blocks = (nel + EPB - 1) / EPB;
    if (blocks > 0x7fffffff) return sem::fail(ctx, SEM_EINVAL, "sem_ax: nel too large");
    if (dot && !lid) return sem::fail(ctx, SEM_EINVAL, "launch_ax: the fused dot needs the solver form");
    if (lid && !gp) return sem::fail(ctx, SEM_EINVAL, "launch_ax: the solver form needs packed factors");
    if constexpr (kFlatSolver<LX, TS>) {
        if (lid) {                             // the solver's copy is planes (sem::factor_stride)
            const int64_t stride = plane_stride(nel * LX * LX * LX);
            const void* P[6];
            for (int q = 0; q < 6; ++q) P[q] = (const TS*)gp + q * stride;
            if (dot) launch_flat<LX, TU, TS, TC, TW, true, true, HB>(ctx, w, u, D, h1, P, nel, skip, dot, lid, hb);
            else launch_flat<LX, TU, TS, TC, TW, false, true, HB>(ctx, w, u, D, h1, P, nel, skip, dot, lid, hb);
            SEM_LAUNCH_CHECK(ctx);
            return SEM_OK;
        }
    }
    if constexpr (kFlat<LX, TS> && std::is_same<TU, TS>::value) {
        if (!lid && variant == SEM_AX_DEFAULT && takes_flat<LX, TS, TW, HB>(w, u, h1, G, nel, hb)) {
            launch_flat<LX, TU, TS, TC, TW, false, false, HB>(ctx, w, u, D, h1, G, nel, skip, nullptr, nullptr, hb);
            SEM_LAUNCH_CHECK(ctx);
            return SEM_OK;
        }
    }
    if (!lid && !dot && variant >= 0 &&
        launch_variant<LX, TS, TC, TW, HB>(ctx, variant, w, u, D, h1, G, nel, hb)) {
        SEM_LAUNCH_CHECK(ctx);
        return SEM_OK;
    }
#define SEM_AX_ARGS (TW*)w, (const TU*)u, (const TC*)D[0], (const TC*)D[1], (const TC*)D[2], \
        (const TC*)D[3], (const TC*)D[4], (const TC*)D[5], (const TS*)h1, (const TS*)G[0],  \
        (const TS*)G[1], (const TS*)G[2], (const TS*)G[3], (const TS*)G[4], (const TS*)G[5], \
        nel, skip, dot, lid, (const TS*)gp, (const TS*)hb
    const dim3 grid((unsigned)blocks), block(EPB * LX * LX);
    if constexpr (!kFlatSolver<LX, TS>) {
        if (dot)
            ax_kernel<LX, EPB, TU, TS, TC, TW, true, true, HB><<<grid, block, 0, ctx->stream>>>(SEM_AX_ARGS);
        else if (lid)
            ax_kernel<LX, EPB, TU, TS, TC, TW, false, true, HB><<<grid, block, 0, ctx->stream>>>(SEM_AX_ARGS);
    }
    if (!lid) ax_kernel<LX, EPB, TU, TS, TC, TW, false, false, HB><<<grid, block, 0, ctx->stream>>>(SEM_AX_ARGS);
#undef SEM_AX_ARGS
    SEM_LAUNCH_CHECK(ctx);
    return SEM_OK;
}

template <int LX, typename TU, typename TS, typename TC, typename TW>
int launch_lx(sem_ctx_t ctx, void* w, const void* u, const void* const* D, const void* h1,
              const void* const* G, int64_t nel, const int* skip, double* dot, const int32_t* lid,
              const void* gp, const void* hb, int variant) {
    if (hb) return launch_form<LX, TU, TS, TC, TW, true>(ctx, w, u, D, h1, G, nel, skip, dot, lid, gp, hb, variant);
    return launch_form<LX, TU, TS, TC, TW, false>(ctx, w, u, D, h1, G, nel, skip, dot, lid, gp, hb, variant);
}

template <typename TU, typename TS, typename TC, typename TW>
int dispatch(sem_ctx_t ctx, int lx, void* w, const void* u, const void* const* D,
             const void* h1, const void* const* G, int64_t nel, const int* skip, double* dot,
             const int32_t* lid = nullptr, const void* gp = nullptr,
             const void* hb = nullptr, int variant = SEM_AX_DEFAULT) {
    switch (lx) {
#define SEM_AX_CASE(L) case L: return launch_lx<L, TU, TS, TC, TW>(ctx, w, u, D, h1, G, nel, skip, dot, lid, gp, hb, variant);
        SEM_AX_CASE(2) SEM_AX_CASE(3) SEM_AX_CASE(4) SEM_AX_CASE(5) SEM_AX_CASE(6) SEM_AX_CASE(7)
        SEM_AX_CASE(8) SEM_AX_CASE(9) SEM_AX_CASE(10) SEM_AX_CASE(11) SEM_AX_CASE(12)
#undef SEM_AX_CASE
        default: return sem::fail(ctx, SEM_EUNSUPPORTED_LX, "sem_ax: lx=%d outside [2,12]", lx);
    }
}

// elements per workgroup of the solver form
template <int LX, typename TS>
constexpr int epb_of() {
    if constexpr (kFlatSolver<LX, TS>) return ShapeF<LX, std::is_same<TS, double>::value>::EPB;
    else return Shape<LX>::EPB;
}

size_t dsize(sem_dtype_t t) { return t == SEM_F64 ? 8 : t == SEM_F32 ? 4 : 2; }

bool overlaps(const void* a, size_t na, const void* b, size_t nb) {
    if (!a || !b) return false;
    const char* pa = (const char*)a;
    const char* pb = (const char*)b;
    return pa < pb + nb && pb < pa + na;
}

}  // namespace

namespace {

int ax_public(sem_ctx_t ctx, void* w, const void* u, const void* dx, const void* dy, const void* dz,
              const void* dxt, const void* dyt, const void* dzt, const void* h1, const void* g11,
              const void* g22, const void* g33, const void* g12, const void* g13, const void* g23,
              const void* hb, int64_t nel, int lx, sem_dtype_t field_dtype, sem_dtype_t out_dtype) {
    int rc = sem::enter(ctx);
    if (rc) return rc;
    if (!sem::lx_ok(lx)) return sem::fail(ctx, SEM_EUNSUPPORTED_LX, "sem_ax: lx=%d outside [2,12]", lx);
    if (nel < 0) return sem::fail(ctx, SEM_EINVAL, "sem_ax: nel=%lld < 0", (long long)nel);
    if (nel == 0) return SEM_OK;
    const void* D[6] = {dx, dy, dz, dxt, dyt, dzt};
    const void* G[6] = {g11, g22, g33, g12, g13, g23};
    if (!w || !u) return sem::fail(ctx, SEM_EINVAL, "sem_ax: null w or u");
    for (int q = 0; q < 6; ++q)
        if (!D[q] || !G[q]) return sem::fail(ctx, SEM_EINVAL, "sem_ax: null derivative or geometric-factor pointer");
    const bool f64 = field_dtype == SEM_F64;
    if (field_dtype != SEM_F64 && field_dtype != SEM_F32 && field_dtype != SEM_BF16)
        return sem::fail(ctx, SEM_EINVAL, "sem_ax: bad field dtype %d", (int)field_dtype);
    if (!(out_dtype == SEM_F32 || (out_dtype == SEM_F64 && f64)))
        return sem::fail(ctx, SEM_EINVAL, "sem_ax: unsupported out dtype %d for field dtype %d",
                         (int)out_dtype, (int)field_dtype);
    const int64_t n = nel * lx * lx * lx;
    const size_t nw = (size_t)n * dsize(out_dtype), nf = (size_t)n * dsize(field_dtype);
    const size_t nd = (size_t)lx * lx * (f64 ? 8 : 4);
    bool alias = overlaps(w, nw, u, nf) || overlaps(w, nw, h1, nf) || overlaps(w, nw, hb, nf);
    for (int q = 0; q < 6; ++q) alias = alias || overlaps(w, nw, G[q], nf) || overlaps(w, nw, D[q], nd);
    if (alias) return sem::fail(ctx, SEM_EINVAL, "sem_ax: output overlaps an input");
    if (f64)
        return dispatch<double, double, double, double>(ctx, lx, w, u, D, h1, G, nel, nullptr, nullptr, nullptr,
                                                        nullptr, hb,
                                                        ctx->ax_builtin[lx] ? SEM_AX_DEFAULT : ctx->ax_variant[lx]);
    if (field_dtype == SEM_F32)
        return dispatch<float, float, float, float>(ctx, lx, w, u, D, h1, G, nel, nullptr, nullptr, nullptr,
                                                    nullptr, hb);
    return dispatch<uint16_t, uint16_t, float, float>(ctx, lx, w, u, D, h1, G, nel, nullptr, nullptr, nullptr,
                                                      nullptr, hb);
}

}  // namespace

extern "C" int sem_ax(sem_ctx_t ctx, void* w, const void* u, const void* dx, const void* dy,
                      const void* dz, const void* dxt, const void* dyt, const void* dzt,
                      const void* h1, const void* g11, const void* g22, const void* g33,
                      const void* g12, const void* g13, const void* g23, int64_t nel, int lx,
                      sem_dtype_t field_dtype, sem_dtype_t out_dtype) {
    return ax_public(ctx, w, u, dx, dy, dz, dxt, dyt, dzt, h1, g11, g22, g33, g12, g13, g23, nullptr, nel, lx,
                     field_dtype, out_dtype);
}

extern "C" int sem_ax_helmholtz(sem_ctx_t ctx, void* w, const void* u, const void* dx, const void* dy,
                                const void* dz, const void* dxt, const void* dyt, const void* dzt,
                                const void* h1, const void* g11, const void* g22, const void* g33,
                                const void* g12, const void* g13, const void* g23, const void* h2b,
                                int64_t nel, int lx, sem_dtype_t field_dtype, sem_dtype_t out_dtype) {
    if (!h2b && nel > 0) return sem::fail(ctx, SEM_EINVAL, "sem_ax_helmholtz: null h2b");
    return ax_public(ctx, w, u, dx, dy, dz, dxt, dyt, dzt, h1, g11, g22, g33, g12, g13, g23, h2b, nel, lx,
                     field_dtype, out_dtype);
}

namespace sem {

// workgroups of the solver form
int ax_blocks(AxKind kind, int lx, int64_t nel) {
    int epb = 1;
    switch (lx) {
#define SEM_AX_EPB(L) case L: epb = kind == AxKind::F64 ? epb_of<L, double>() : kind == AxKind::F32 ? epb_of<L, float>() \
                                   : epb_of<L, uint16_t>(); break;
        SEM_AX_EPB(2) SEM_AX_EPB(3) SEM_AX_EPB(4) SEM_AX_EPB(5) SEM_AX_EPB(6) SEM_AX_EPB(7)
        SEM_AX_EPB(8) SEM_AX_EPB(9) SEM_AX_EPB(10) SEM_AX_EPB(11) SEM_AX_EPB(12)
#undef SEM_AX_EPB
        default: break;
    }
    return (int)((nel + epb - 1) / epb);
}

int64_t factor_stride(AxKind kind, int lx, int64_t n) {
    bool flat = false;
    switch (lx) {
#define SEM_AX_FLAT(L) case L: flat = kind == AxKind::F64 ? kFlatSolver<L, double> : kind == AxKind::F32 ? kFlatSolver<L, float> \
                                    : kFlatSolver<L, uint16_t>; break;
        SEM_AX_FLAT(2) SEM_AX_FLAT(3) SEM_AX_FLAT(4) SEM_AX_FLAT(5) SEM_AX_FLAT(6) SEM_AX_FLAT(7)
        SEM_AX_FLAT(8) SEM_AX_FLAT(9) SEM_AX_FLAT(10) SEM_AX_FLAT(11) SEM_AX_FLAT(12)
#undef SEM_AX_FLAT
        default: break;
    }
    return flat ? plane_stride(n) : 0;
}

int launch_ax(sem_ctx_t ctx, AxKind kind, const AxArgs& a, void* w, const void* u,
              const int* skip, double* dot, const int32_t* lid) {
    const void* D[6] = {a.D[0], a.D[1], a.D[2], a.D[3], a.D[4], a.D[5]};
    const void* G[6] = {a.G[0], a.G[1], a.G[2], a.G[3], a.G[4], a.G[5]};
    switch (kind) {
        case AxKind::F64:
            return dispatch<double, double, double, double>(ctx, a.lx, w, u, D, a.h1, G, a.nel, skip, dot, lid,
                                                            a.Gp, a.hb);
        case AxKind::F32:
            return dispatch<float, float, float, float>(ctx, a.lx, w, u, D, a.h1, G, a.nel, skip, dot, lid,
                                                        a.Gp, a.hb);
        case AxKind::F32_BF16:
            return dispatch<float, uint16_t, float, float>(ctx, a.lx, w, u, D, a.h1, G, a.nel, skip, dot, lid,
                                                           a.Gp, a.hb);
    }
    return fail(ctx, SEM_EINVAL, "launch_ax: bad kind");
}

}  // namespace sem

// ------------------------------------------------------------ variant choice
namespace {

// synthetic inputs for timing: a hash of the index mapped to [-1, 1) for u,
// positive-definite factors (diagonal 1 + |.|/2, off-diagonal ./10), h1 = 1
__global__ void tune_fill_kernel(double* __restrict__ u, double* __restrict__ g11, double* __restrict__ g22,
                                 double* __restrict__ g33, double* __restrict__ g12, double* __restrict__ g13,
                                 double* __restrict__ g23, double* __restrict__ h1, int64_t n) {
    for (int64_t L = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; L < n; L += (int64_t)gridDim.x * blockDim.x) {
        uint32_t h = (uint32_t)L * 2654435761u;
        h ^= h >> 16; h *= 0x7feb352du; h ^= h >> 15;
        const double v = (double)h * (2.0 / 4294967296.0) - 1.0;
        u[L] = v;
        g11[L] = 1.0 + 0.5 * fabs(v); g22[L] = 1.0 + 0.25 * fabs(v); g33[L] = 1.0 + 0.125 * fabs(v);
        g12[L] = 0.1 * v; g13[L] = -0.1 * v; g23[L] = 0.05 * v;
        h1[L] = 1.0;
    }
}

}  // namespace

extern "C" int sem_ax_set_variant(sem_ctx_t ctx, int lx, int variant) {
    int rc = sem::enter(ctx);
    if (rc) return rc;
    if (!sem::lx_ok(lx)) return sem::fail(ctx, SEM_EUNSUPPORTED_LX, "sem_ax_set_variant: lx=%d", lx);
    if (variant != SEM_AX_DEFAULT && !variant_exists(lx, variant))
        return sem::fail(ctx, SEM_EINVAL, "sem_ax_set_variant: variant %d does not exist at lx=%d", variant, lx);
    ctx->ax_variant[lx] = variant;
    ctx->ax_builtin[lx] = false;
    return SEM_OK;
}

extern "C" int sem_ax_get_variant(sem_ctx_t ctx, int lx, int* variant) {
    if (!ctx) return sem::fail(nullptr, SEM_EINVAL, "null context");
    if (!sem::lx_ok(lx)) return sem::fail(ctx, SEM_EUNSUPPORTED_LX, "sem_ax_get_variant: lx=%d", lx);
    if (!variant) return sem::fail(ctx, SEM_EINVAL, "sem_ax_get_variant: null output");
    *variant = ctx->ax_variant[lx];
    return SEM_OK;
}

namespace {

// every float64 variant that exists at lx timed on the given operands (`reps`
// launches after two warm-ups, HIP events on the context's stream) in two
// rounds, keeping each variant's faster round: the clocks of a GPU that was
// idle rise during the first launches, which would otherwise penalise the
// variant timed first.  The fastest is selected on the context.  Where the
// built-in kernel takes whole elements here it is timed after the variants; if it
// beats the column mapping it takes that one's place.
int time_variants(sem_ctx_t ctx, int lx, void* w, const void* u, const void* const* D, const void* h1,
                  const void* const* G, int64_t nel, int reps, double* us, int* best) {
    hipStream_t st = ctx->stream;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    SEM_HIP(ctx, hipEventCreate(&e0));
    hipError_t he = hipEventCreate(&e1);
    if (he != hipSuccess) { (void)hipEventDestroy(e0); return sem::check_hip(ctx, he, "hipEventCreate"); }
    constexpr int kBuiltin = SEM_AX_VARIANTS;  // its place behind the variants
    bool flat = false;
    switch (lx) {
#define SEM_AX_FLAT(L) case L: flat = takes_flat<L, double, double, false>(w, u, h1, G, nel, nullptr); break;
        SEM_AX_FLAT(5) SEM_AX_FLAT(6) SEM_AX_FLAT(12)
#undef SEM_AX_FLAT
        default: break;
    }
    double t_best[SEM_AX_VARIANTS + 1];
    for (int v = 0; v <= SEM_AX_VARIANTS; ++v) t_best[v] = -1.0;
    int rc = SEM_OK;
    for (int round = 0; round < 2 && rc == SEM_OK; ++round)
        for (int v = 0; v <= SEM_AX_VARIANTS && rc == SEM_OK; ++v) {
            if (v == kBuiltin ? !flat : !variant_exists(lx, v)) continue;
            for (int q = 0; q < 2 + reps && rc == SEM_OK; ++q) {
                if (q == 2) (void)hipEventRecord(e0, st);
                rc = dispatch<double, double, double, double>(ctx, lx, w, u, D, h1, G, nel, nullptr, nullptr,
                                                              nullptr, nullptr, nullptr,
                                                              v == kBuiltin ? SEM_AX_DEFAULT : v);
            }
            if (rc) break;
            (void)hipEventRecord(e1, st);
            (void)hipEventSynchronize(e1);
            float ms = 0.f;
            (void)hipEventElapsedTime(&ms, e0, e1);
            const double t = 1e3 * ms / reps;
            if (t_best[v] < 0.0 || t < t_best[v]) t_best[v] = t;
        }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc) return rc;
    const bool builtin = t_best[kBuiltin] >= 0.0 && t_best[kBuiltin] < t_best[SEM_AX_COLUMN];
    if (builtin) t_best[SEM_AX_COLUMN] = t_best[kBuiltin];
    int best_v = SEM_AX_COLUMN;
    for (int v = 0; v < SEM_AX_VARIANTS; ++v) {
        if (us) us[v] = t_best[v];
        if (t_best[v] >= 0.0 && (t_best[best_v] < 0.0 || t_best[v] < t_best[best_v])) best_v = v;
    }
    ctx->ax_variant[lx] = best_v;
    ctx->ax_builtin[lx] = builtin && best_v == SEM_AX_COLUMN;
    *best = best_v;
    return SEM_OK;
}

}  // namespace

extern "C" int sem_ax_tune(sem_ctx_t ctx, int lx, int64_t nel, int reps, double* us, int* best) {
    int rc = sem::enter(ctx);
    if (rc) return rc;
    if (!sem::lx_ok(lx)) return sem::fail(ctx, SEM_EUNSUPPORTED_LX, "sem_ax_tune: lx=%d", lx);
    if (nel < 1 || reps < 1 || !best) return sem::fail(ctx, SEM_EINVAL, "sem_ax_tune: bad argument");
    const int64_t n = nel * lx * lx * lx;
    const int l2 = lx * lx;
    hipStream_t st = ctx->stream;
    std::vector<void*> tmp;
    auto cleanup = [&]() {
        (void)hipStreamSynchronize(st);
        for (void* p : tmp) (void)hipFree(p);
    };
    double* a[10] = {};
    for (int q = 0; q < 9; ++q) {
        hipError_t e = hipMalloc((void**)&a[q], sizeof(double) * n);
        if (e != hipSuccess) { cleanup(); return sem::check_hip(ctx, e, "sem_ax_tune: hipMalloc"); }
        tmp.push_back(a[q]);
    }
    {
        hipError_t e = hipMalloc((void**)&a[9], sizeof(double) * 2 * l2);
        if (e != hipSuccess) { cleanup(); return sem::check_hip(ctx, e, "sem_ax_tune: hipMalloc"); }
        tmp.push_back(a[9]);
    }
    double *u = a[0], *w = a[1], *h1 = a[8], *Dd = a[9];
    std::vector<double> dx(l2), dxt(l2);
    sem_gll(lx, nullptr, nullptr, dx.data(), dxt.data());   // the argument layout of the operator
    {
        hipError_t e = hipMemcpy(Dd, dx.data(), sizeof(double) * l2, hipMemcpyHostToDevice);
        if (e == hipSuccess) e = hipMemcpy(Dd + l2, dxt.data(), sizeof(double) * l2, hipMemcpyHostToDevice);
        if (e != hipSuccess) { cleanup(); return sem::check_hip(ctx, e, "sem_ax_tune: hipMemcpy"); }
    }
    tune_fill_kernel<<<4096, 256, 0, st>>>(u, a[2], a[3], a[4], a[5], a[6], a[7], h1, n);
    const void* D[6] = {Dd, Dd, Dd, Dd + l2, Dd + l2, Dd + l2};
    const void* G[6] = {a[2], a[3], a[4], a[5], a[6], a[7]};
    rc = time_variants(ctx, lx, w, u, D, h1, G, nel, reps, us, best);
    cleanup();
    return rc;
}

extern "C" int sem_ax_tune_on(sem_ctx_t ctx, void* w, const void* u, const void* dx, const void* dy,
                              const void* dz, const void* dxt, const void* dyt, const void* dzt, const void* h1,
                              const void* g11, const void* g22, const void* g33, const void* g12,
                              const void* g13, const void* g23, int64_t nel, int lx, int reps, double* us,
                              int* best) {
    int rc = sem::enter(ctx);
    if (rc) return rc;
    if (!sem::lx_ok(lx)) return sem::fail(ctx, SEM_EUNSUPPORTED_LX, "sem_ax_tune_on: lx=%d", lx);
    if (nel < 1 || reps < 1 || !best || !w || !u) return sem::fail(ctx, SEM_EINVAL, "sem_ax_tune_on: bad argument");
    const void* D[6] = {dx, dy, dz, dxt, dyt, dzt};
    const void* G[6] = {g11, g22, g33, g12, g13, g23};
    for (int q = 0; q < 6; ++q)
        if (!D[q] || !G[q]) return sem::fail(ctx, SEM_EINVAL, "sem_ax_tune_on: null operator array");
    const size_t nb = (size_t)nel * lx * lx * lx * sizeof(double), nd = (size_t)lx * lx * sizeof(double);
    bool alias = overlaps(w, nb, u, nb) || overlaps(w, nb, h1, nb);
    for (int q = 0; q < 6; ++q) alias = alias || overlaps(w, nb, G[q], nb) || overlaps(w, nb, D[q], nd);
    if (alias) return sem::fail(ctx, SEM_EINVAL, "sem_ax_tune_on: output overlaps an input");
    return time_variants(ctx, lx, w, u, D, h1, G, nel, reps, us, best);
}

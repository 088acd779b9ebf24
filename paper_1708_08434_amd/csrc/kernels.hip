// HIP kernels (gfx950) for geometric multigrid on an octree of 8^3 boxes.
//
// Storage: every field is [box][colour][256] with colour = (i+j+k) & 1 and,
// inside a colour, index (k*8 + j)*4 + (i>>1).  A red (or black) half-sweep
// of red-black Gauss-Seidel (paper section 2.1.2) therefore streams this
// colour's right-hand side and the other colour's solution as contiguous
// 2 KB runs and writes one contiguous 2 KB run per box, which is the minimum
// traffic of a half-sweep.  Boxes of one level are consecutive (canonical
// order), so a launch over a level streams one contiguous range.
//
// Each stencil kernel stages one box and its one-cell ghost layer in LDS
// (section 2.1.3: a ghost layer lets every box be worked on independently).
// Ghosts are never stored in HBM; dedicated threads evaluate them from
// (a) the same-level neighbour box, (b) the physical boundary condition, or
// (c) at a refinement boundary, the tangentially interpolated coarse value
// (precomputed per level visit by the coarse-face pass) and the two interior
// fine cells along the normal.  All global loads of a thread are independent
// of each other, so a kernel costs one memory round trip plus one barrier.
#include <cmath>

#include "axis.h"
#include "kernels.h"

namespace mg {
namespace {

constexpr double kSixth = 1.0 / 6.0;
constexpr double kCfCoarse = 8.0 / 15.0;  // quadratic through the coarse value,
constexpr double kCfFine1 = 2.0 / 3.0;    // the first and the second interior
constexpr double kCfFine2 = 0.2;          // fine cell (ghost at the face + h/2)

__device__ __forceinline__ int cs_idx(int i, int j, int k) {
    return (((i + j + k) & 1) << 8) + ((k * 8 + j) << 2) + (i >> 1);
}
__device__ __forceinline__ int cs_idx3(const int c[3]) { return cs_idx(c[0], c[1], c[2]); }

// Workgroups are handed to the 8 XCDs in turn; give each XCD a contiguous run
// of boxes so that face neighbours of a box usually sit in the same L2.
__device__ __forceinline__ int64_t xcd_map(int64_t blk, int64_t n) {
    int64_t per = (n + 7) >> 3;
    return (blk & 7) * per + (blk >> 3);
}
__host__ __device__ inline int64_t xcd_grid(int64_t n) { return 8 * ((n + 7) >> 3); }

__device__ __forceinline__ void tangential(int a, int &t1, int &t2) {
    t1 = a == 0 ? 1 : 0;
    t2 = a == 2 ? 1 : 2;
}

// max that carries NaN through (a non-finite residual must reach the test)
// Loads of data that a launch reads exactly once (right-hand sides) carry
// the non-temporal hint, so that they do not displace from L2 the cells that
// neighbouring workgroups re-read as ghosts.
#ifndef MG_STREAM_RHS
#define MG_STREAM_RHS 1
#endif
template <typename T> struct StreamLd {
    static __device__ __forceinline__ T ld(const T *p) {
#if MG_STREAM_RHS
        return __builtin_nontemporal_load(p);
#else
        return *p;
#endif
    }
};
template <typename E, typename V, int N> struct StreamVec {
    typedef E native __attribute__((ext_vector_type(N)));
    static __device__ __forceinline__ V ld(const V *p) {
#if MG_STREAM_RHS
        native v = __builtin_nontemporal_load(reinterpret_cast<const native *>(p));
        V r;
#pragma unroll
        for (int i = 0; i < N; i++) reinterpret_cast<E *>(&r)[i] = v[i];
        return r;
#else
        return *p;
#endif
    }
};
template <> struct StreamLd<double2> : StreamVec<double, double2, 2> {};
template <> struct StreamLd<double4> : StreamVec<double, double4, 4> {};
template <> struct StreamLd<float2> : StreamVec<float, float2, 2> {};
template <> struct StreamLd<float4> : StreamVec<float, float4, 4> {};
template <typename T> __device__ __forceinline__ T ld_stream(const T *p) { return StreamLd<T>::ld(p); }

__device__ __forceinline__ double nanmax(double a, double b) { return (a > b || a != a) ? a : b; }

// Ghost values: Dirichlet face value gv reflected through the boundary cell,
// and the refinement-boundary quadratic through the coarse value ch and the
// first two interior fine cells.  Every kernel evaluates them through these
// two functions, so all paths round identically.
template <typename T> __device__ __forceinline__ T dirichlet_ghost(T gv, T own) {
    return (T)2 * gv - own;
}
// Fused multiply-adds written out, so that every kernel rounds the
// refinement-boundary ghost the same way whatever the compiler would contract.
__device__ __forceinline__ double fmadd(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fmadd(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
template <typename T> __device__ __forceinline__ T cf_ghost(T ch, T own, T inward) {
    return fmadd((T)kCfCoarse, ch, fmadd((T)kCfFine1, own, -((T)kCfFine2 * inward)));
}
// Residual b - (s - 6 own) / h^2 of a cell with neighbour sum s, with the
// multiply-adds written out so that every kernel that forms a residual
// (restriction, stopping test, bottom of the cycle) rounds it alike.
template <typename T> __device__ __forceinline__ T resid_of(T b, T s, T own, T inv_h2) {
    return fmadd(-fmadd((T)-6, own, s), inv_h2, b);
}
template <typename T>
__device__ __forceinline__ T bc_value(const Geo &g, int64_t b, int d, int u, int v) {
    return (T)(g.bcval ? g.bcval[(b * 6 + d) * 64 + v * 8 + u] : g.bcv[d]);
}

// Ghost of face cell (u, v) on face d of box b, read straight from global
// memory.  nb = nbr[b][d]; slot = cfslot[b][d].  T is the field type (double,
// or float for the correction cycles of the mixed-precision solve).
template <typename T>
__device__ __forceinline__ T ghost_at(const Geo &g, const T *__restrict__ phi,
                                      const T *__restrict__ chat, int64_t b, int d, int nb, int slot,
                                      int u, int v) {
    int a = d >> 1, side = d & 1, t1, t2;
    tangential(a, t1, t2);
    int c[3];
    c[t1] = u;
    c[t2] = v;
    if (nb >= 0) {
        c[a] = side ? 0 : 7;  // mirrored cell in the neighbour
        return phi[(int64_t)nb * 512 + cs_idx3(c)];
    }
    c[a] = side ? 7 : 0;
    T own = phi[b * 512 + cs_idx3(c)];
    if (nb == -2) {
        if (g.bct[d] == 1) return own;
        return dirichlet_ghost<T>(bc_value<T>(g, b, d, u, v), own);
    }
    c[a] = side ? 6 : 1;
    T inward = phi[b * 512 + cs_idx3(c)];
    return cf_ghost<T>(chat[(int64_t)slot * 64 + v * 8 + u], own, inward);
}

// The face tables of box b, read with block-uniform addresses (scalar loads
// issued at kernel start), so that a ghost's value load waits on no vector
// load of an index.
struct FaceTab {
    int nb[6], slot[6];
};
__device__ __forceinline__ FaceTab face_tab(const Geo &g, int64_t b) {
    FaceTab f;
#pragma unroll
    for (int d = 0; d < 6; d++) {
        f.nb[d] = g.nbr[b * 6 + d];
        f.slot[d] = g.cfslot[b * 6 + d];
    }
    return f;
}
__device__ __forceinline__ int pick6(const int v[6], int d) {
    return d == 0 ? v[0] : d == 1 ? v[1] : d == 2 ? v[2] : d == 3 ? v[3] : d == 4 ? v[4] : v[5];
}

// Stage the whole box (both colours, colour-split order) into P[512] and all
// 6 x 64 face ghosts into H[d*64 + v*8 + u]; 256 threads.  Caller syncs.
template <typename T>
__device__ __forceinline__ void stage_full(const Geo &g, const T *__restrict__ phi,
                                           const T *__restrict__ chat, int64_t b, T *P, T *H) {
    int t = threadIdx.x;
    const FaceTab ft = face_tab(g, b);
    P[t] = phi[b * 512 + t];
    P[256 + t] = phi[b * 512 + 256 + t];
#pragma unroll
    for (int r = 0; r < 2; r++) {
        int e = t + 256 * r;
        if (e < 384) {
            int d = e >> 6, w = e & 63;
            H[e] = ghost_at<T>(g, phi, chat, b, d, pick6(ft.nb, d), pick6(ft.slot, d), w & 7, w >> 3);
        }
    }
}

// Six-neighbour sum of cell (i, j, k) from a staged box, order -x, +x, -y,
// +y, -z, +z.
template <typename T>
__device__ __forceinline__ T sum_full(const T *P, const T *H, int i, int j, int k) {
    T xm = i > 0 ? P[cs_idx(i - 1, j, k)] : H[0 * 64 + k * 8 + j];
    T xp = i < 7 ? P[cs_idx(i + 1, j, k)] : H[1 * 64 + k * 8 + j];
    T ym = j > 0 ? P[cs_idx(i, j - 1, k)] : H[2 * 64 + k * 8 + i];
    T yp = j < 7 ? P[cs_idx(i, j + 1, k)] : H[3 * 64 + k * 8 + i];
    T zm = k > 0 ? P[cs_idx(i, j, k - 1)] : H[4 * 64 + j * 8 + i];
    T zp = k < 7 ? P[cs_idx(i, j, k + 1)] : H[5 * 64 + j * 8 + i];
    return xm + xp + ym + yp + zm + zp;
}

// ------------------------------------------------------------------ kernels

template <typename T>
__global__ void k_fill(T *p, int64_t count, T v) {
    int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q < count) p[q] = v;
}

template <typename T>
__global__ __launch_bounds__(256) void k_pack(const double *__restrict__ nat, T *__restrict__ cs,
                                              int64_t nbox) {
    int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (q >= nbox * 512) return;
    int64_t b = q >> 9;
    int c = (int)(q & 511), i = c & 7, j = (c >> 3) & 7, k = c >> 6;
    cs[b * 512 + cs_idx(i, j, k)] = (T)nat[q];
}

template <typename T>
__global__ __launch_bounds__(256) void k_unpack(const T *__restrict__ cs, double *__restrict__ nat,
                                                int64_t nbox) {
    int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (q >= nbox * 512) return;
    int64_t b = q >> 9;
    int c = (int)(q & 511), i = c & 7, j = (c >> 3) & 7, k = c >> 6;
    nat[q] = (double)cs[b * 512 + cs_idx(i, j, k)];
}

// One colour C of red-black Gauss-Seidel on boxes [b0, b0+nbx): 256/CPT
// threads per box, CPT neighbouring cells of colour C each (vector loads of
// CPT values, so a wave keeps CPT times the bytes in flight).  LDS holds the
// other colour S[256] and the 6 x 32 ghosts of this colour's face cells,
// H[d*32 + v*4 + (u>>1)].  XCD-aware box mapping when xcd != 0.  CPT and the
// mapping are the launch variants the autotuner chooses from; every variant
// performs the same arithmetic on every cell.
template <typename T>
__device__ __forceinline__ T gsrb_ghost_val(const Geo &g, const FaceTab &ft, const T *__restrict__ phi,
                                            const T *__restrict__ chat, int64_t b, int C, int e) {
    int d = e >> 5, q = e & 31, v = q >> 2;
    int layer = (d & 1) ? 7 : 0;
    int u = 2 * (q & 3) + ((layer + v + C) & 1);
    return ghost_at<T>(g, phi, chat, b, d, pick6(ft.nb, d), pick6(ft.slot, d), u, v);
}
template <typename T>
__device__ __forceinline__ void gsrb_ghost(const Geo &g, const FaceTab &ft, const T *__restrict__ phi,
                                           const T *__restrict__ chat, int64_t b, int C, int e, T *H) {
    H[e] = gsrb_ghost_val<T>(g, ft, phi, chat, b, C, e);
}

template <typename T, int N> struct VecN;
template <> struct VecN<double, 1> { using type = double; };
template <> struct VecN<double, 2> { using type = double2; };
template <> struct VecN<double, 4> { using type = double4; };
template <> struct VecN<float, 1> { using type = float; };
template <> struct VecN<float, 2> { using type = float2; };
template <> struct VecN<float, 4> { using type = float4; };

// Restriction of a box's 512 values (colour-split, in LDS) onto its parent's
// cells: the mean of the 8 children under each, k_restrict_leaves' order.
template <typename T>
__device__ __forceinline__ void restrict_box(const Geo &g, const T *U, int64_t b, T *__restrict__ dst, int e) {
    int pi = e & 3, pj = (e >> 2) & 3, pk = e >> 4;
    T sum = 0;
#pragma unroll
    for (int dk = 0; dk < 2; dk++)
#pragma unroll
        for (int dj = 0; dj < 2; dj++)
#pragma unroll
            for (int di = 0; di < 2; di++) sum += U[cs_idx(2 * pi + di, 2 * pj + dj, 2 * pk + dk)];
    int64_t p = g.parent[b];
    int ci = 4 * (g.ijk[b * 4] & 1) + pi, cj = 4 * (g.ijk[b * 4 + 1] & 1) + pj, ck = 4 * (g.ijk[b * 4 + 2] & 1) + pk;
    dst[p * 512 + cs_idx(ci, cj, ck)] = (T)0.125 * sum;
}

// phi64 += (double) e on N cells of each colour at colour-half position q0
// (k_ir_update's arithmetic); the updated values are also left in U
// (colour-split) when U is set.
template <typename T, int N>
__device__ __forceinline__ void ir_add(double *__restrict__ phi64, int64_t b, int C, int q0, const T *eC,
                                       const T *eO, double *U) {
    using D = typename VecN<double, N>::type;
    D *pc = reinterpret_cast<D *>(phi64 + b * 512 + C * 256 + q0);
    D *po = reinterpret_cast<D *>(phi64 + b * 512 + (1 - C) * 256 + q0);
    D vc = *pc, vo = *po;
    double *xc = reinterpret_cast<double *>(&vc), *xo = reinterpret_cast<double *>(&vo);
#pragma unroll
    for (int w = 0; w < N; w++) {
        xc[w] += (double)eC[w];
        xo[w] += (double)eO[w];
    }
    *pc = vc;
    *po = vo;
    if (U) {
#pragma unroll
        for (int w = 0; w < N; w++) {
            U[C * 256 + q0 + w] = xc[w];
            U[(1 - C) * 256 + q0 + w] = xo[w];
        }
    }
}

// Modes of the black half-sweep when it is a box's last sweep of the cycle
// before a stopping test:
//  kSweepRestrict: boxes with rmask[b] != 0 also set their parent cells to
//    the mean of the 8 children under each, from the swept values.
//  kSweepIrUpdate (FP32 correction cycle): phi64 += e on all 512 cells of
//    the box (the refinement update), and boxes with rmask set restrict the
//    updated phi64 onto their parents (rmask may be null).
constexpr int kSweepPlain = 0, kSweepRestrict = 1, kSweepIrUpdate = 2;
template <int C, typename T, int CPT, int MODE = kSweepPlain>
__global__ __launch_bounds__(256 / CPT) void k_gsrb(Geo g, T *__restrict__ phi,
                                                    const T *__restrict__ rhs,
                                                    const T *__restrict__ chat, int64_t b0,
                                                    int64_t nbx, T h2, int xcd,
                                                    const int32_t *__restrict__ rmask = nullptr,
                                                    double *__restrict__ phi64 = nullptr) {
    using V = typename VecN<T, CPT>::type;
    constexpr int NT = 256 / CPT;
    __shared__ T SB[MODE == kSweepRestrict ? 512 : 256], H[192];
    __shared__ double U[MODE == kSweepIrUpdate ? 512 : 1];
    T *S = SB;
    int64_t lb = xcd ? xcd_map(blockIdx.x, nbx) : (int64_t)blockIdx.x;
    if (lb >= nbx) return;
    int64_t b = b0 + lb;
    int t = threadIdx.x;
    const FaceTab ft = face_tab(g, b);
    V o = reinterpret_cast<const V *>(phi + b * 512 + (1 - C) * 256)[t];
    V bv = ld_stream(reinterpret_cast<const V *>(rhs + b * 512 + C * 256) + t);
#pragma unroll
    for (int e = t; e < 192; e += NT) gsrb_ghost<T>(g, ft, phi, chat, b, C, e, H);
    reinterpret_cast<V *>(S)[t] = o;
    __syncthreads();
    const T *bb = reinterpret_cast<const T *>(&bv);
    V res;
    T *out = reinterpret_cast<T *>(&res);
#pragma unroll
    for (int w = 0; w < CPT; w++) {
        int cq = CPT * t + w;
        int m = cq & 3, j = (cq >> 2) & 7, k = cq >> 5;
        int i = 2 * m + ((j + k + C) & 1);
        int row = (k * 8 + j) * 4;
        T xm = i > 0 ? S[row + ((i - 1) >> 1)] : H[0 * 32 + k * 4 + (j >> 1)];
        T xp = i < 7 ? S[row + ((i + 1) >> 1)] : H[1 * 32 + k * 4 + (j >> 1)];
        T ym = j > 0 ? S[row - 4 + m] : H[2 * 32 + k * 4 + m];
        T yp = j < 7 ? S[row + 4 + m] : H[3 * 32 + k * 4 + m];
        T zm = k > 0 ? S[row - 32 + m] : H[4 * 32 + j * 4 + m];
        T zp = k < 7 ? S[row + 32 + m] : H[5 * 32 + j * 4 + m];
        T s = xm + xp + ym + yp + zm + zp;
        out[w] = (s - h2 * bb[w]) * (T)kSixth;
    }
    reinterpret_cast<V *>(phi + b * 512 + C * 256)[t] = res;
    if (MODE == kSweepRestrict && rmask[b]) {  // block-uniform
        // SB: colour 0 (the staged other colour) then colour 1 (this sweep's)
        reinterpret_cast<V *>(SB + 256)[t] = res;
        __syncthreads();
        for (int e = t; e < 64; e += NT) restrict_box<T>(g, SB, b, phi, e);
    }
    if (MODE == kSweepIrUpdate) {
        const bool r = rmask && rmask[b];  // block-uniform
        ir_add<T, CPT>(phi64, b, C, CPT * t, out, reinterpret_cast<const T *>(&o), r ? U : nullptr);
        if (r) {
            __syncthreads();
            for (int e = t; e < 64; e += NT) restrict_box<double>(g, U, b, phi64, e);
        }
    }
}

// Workgroup barrier that orders LDS only: global loads issued before it stay
// in flight (the prefetch of the next box), unlike __syncthreads().
__device__ __forceinline__ void lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// One colour C of red-black Gauss-Seidel with persistent workgroups of 128
// threads (2 cells each): workgroup w takes boxes base, base + step, ...
// (with the XCD mapping: the boxes of its XCD's contiguous range, in turn
// with the XCD's other workgroups), and while it updates one box it has the
// next box's cells, right-hand side and ghosts in flight and the face table
// of the one after.  The ghosts of a box read only the other colour and the
// box's own cells, which no workgroup writes during this half-sweep before
// the box itself is updated, so loading them early changes nothing.  Same
// arithmetic per cell as k_gsrb.
template <int C, typename T>
__global__ __launch_bounds__(128) void k_gsrb_pipe(Geo g, T *__restrict__ phi, const T *__restrict__ rhs,
                                                   const T *__restrict__ chat, int64_t b0, int64_t nbx,
                                                   T h2, int xcd) {
    using V = typename VecN<T, 2>::type;
    __shared__ T S[256], H[192];
    const int t = threadIdx.x;
    int64_t base, step, end;
    if (xcd) {
        int64_t per = (nbx + 7) >> 3, x = blockIdx.x & 7;
        base = x * per + (blockIdx.x >> 3);
        step = gridDim.x >> 3;
        end = min((x + 1) * per, nbx);
    } else {
        base = blockIdx.x;
        step = gridDim.x;
        end = nbx;
    }
    if (base >= end) return;
    int64_t b = b0 + base;
    FaceTab ft = face_tab(g, b);
    V o = reinterpret_cast<const V *>(phi + b * 512 + (1 - C) * 256)[t];
    V bv = ld_stream(reinterpret_cast<const V *>(rhs + b * 512 + C * 256) + t);
    T g0 = gsrb_ghost_val<T>(g, ft, phi, chat, b, C, t);
    T g1 = t < 64 ? gsrb_ghost_val<T>(g, ft, phi, chat, b, C, t + 128) : (T)0;
    int64_t nxt = base + step;
    FaceTab ftn = ft;
    if (nxt < end) ftn = face_tab(g, b0 + nxt);
    for (;;) {
        const bool more = nxt < end;
        const int64_t bn = b0 + nxt;
        V on = o, bvn = bv;
        T g0n = 0, g1n = 0;
        FaceTab ftnn = ftn;
        if (more) {
            on = reinterpret_cast<const V *>(phi + bn * 512 + (1 - C) * 256)[t];
            bvn = ld_stream(reinterpret_cast<const V *>(rhs + bn * 512 + C * 256) + t);
            g0n = gsrb_ghost_val<T>(g, ftn, phi, chat, bn, C, t);
            if (t < 64) g1n = gsrb_ghost_val<T>(g, ftn, phi, chat, bn, C, t + 128);
            if (nxt + step < end) ftnn = face_tab(g, bn + step);
        }
        reinterpret_cast<V *>(S)[t] = o;
        H[t] = g0;
        if (t < 64) H[t + 128] = g1;
        lds_sync();
        const T *bb = reinterpret_cast<const T *>(&bv);
        V res;
        T *out = reinterpret_cast<T *>(&res);
#pragma unroll
        for (int w = 0; w < 2; w++) {
            int cq = 2 * t + w;
            int m = cq & 3, j = (cq >> 2) & 7, k = cq >> 5;
            int i = 2 * m + ((j + k + C) & 1);
            int row = (k * 8 + j) * 4;
            T xm = i > 0 ? S[row + ((i - 1) >> 1)] : H[0 * 32 + k * 4 + (j >> 1)];
            T xp = i < 7 ? S[row + ((i + 1) >> 1)] : H[1 * 32 + k * 4 + (j >> 1)];
            T ym = j > 0 ? S[row - 4 + m] : H[2 * 32 + k * 4 + m];
            T yp = j < 7 ? S[row + 4 + m] : H[3 * 32 + k * 4 + m];
            T zm = k > 0 ? S[row - 32 + m] : H[4 * 32 + j * 4 + m];
            T zp = k < 7 ? S[row + 32 + m] : H[5 * 32 + j * 4 + m];
            T s = xm + xp + ym + yp + zm + zp;
            out[w] = (s - h2 * bb[w]) * (T)kSixth;
        }
        reinterpret_cast<V *>(phi + b * 512 + C * 256)[t] = res;
        lds_sync();
        if (!more) break;
        b = bn;
        o = on;
        bv = bvn;
        g0 = g0n;
        g1 = g1n;
        ftn = ftnn;
        nxt += step;
    }
}

// One colour C of red-black Gauss-Seidel on the octets (complete sets of 8
// sibling boxes, consecutive in canonical order) of boxes [b0, b0+8*noct):
// one 512-thread workgroup per octet, which is a 16^3 grid.  Faces between
// siblings are read from LDS, so only the octet's outer surface (6 x 128
// cells of this colour) needs ghosts: half the ghost traffic per cell of the
// one-box launches.  S holds the other colour of the 16^3 grid (colour-split
// rows: (K*16 + J)*8 + I/2); thread t owns one box row (4 cells) of colour C,
// read and written as one vector.  Same arithmetic per cell as k_gsrb.  IR:
// k_gsrb's kSweepIrUpdate mode (each box's 64 threads restrict it).
template <int C, typename T, bool IR = false>
__global__ __launch_bounds__(512) void k_gsrb_oct(Geo g, T *__restrict__ phi, const T *__restrict__ rhs,
                                                  const T *__restrict__ chat, int64_t b0, int64_t noct,
                                                  T h2, int xcd, const int32_t *__restrict__ rmask = nullptr,
                                                  double *__restrict__ phi64 = nullptr) {
    using V4 = typename VecN<T, 4>::type;
    __shared__ T S[2048], H[6 * 128];
    __shared__ double U[IR ? 8 * 512 : 1];
    int64_t lo = xcd ? xcd_map(blockIdx.x, noct) : (int64_t)blockIdx.x;
    if (lo >= noct) return;
    int64_t ob = b0 + 8 * lo;
    int t = threadIdx.x;
    int o = t >> 6, rw = t & 63, j = rw & 7, k = rw >> 3;  // box of the octet, row (j, k) in it
    int64_t bx = ob + o;
    int ox = 8 * (o & 1), oy = 8 * ((o >> 1) & 1), oz = 8 * (o >> 2);
    // other colour of row (j, k) of box o: 4 values, I/2 = ox/2 + m
    V4 so = reinterpret_cast<const V4 *>(phi + bx * 512 + (1 - C) * 256)[rw];
    V4 bv = ld_stream(reinterpret_cast<const V4 *>(rhs + bx * 512 + C * 256) + rw);
    // ghosts of the outer surface: entry e = d*128 + v*8 + u/2 over the
    // 16 x 16 face (u along t1, v along t2), cells of colour C
    for (int e = t; e < 768; e += 512) {
        int d = e >> 7, q = e & 127, v = q >> 3;
        int a = d >> 1, side = d & 1;
        int L = side ? 15 : 0;
        int u = 2 * (q & 7) + ((L + v + C) & 1);
        int c[3];  // octant of the box holding face cell (u, v)
        c[a] = side;
        c[a == 0 ? 1 : 0] = u >> 3;
        c[a == 2 ? 1 : 2] = v >> 3;
        int64_t gb = ob + (c[0] | (c[1] << 1) | (c[2] << 2));
        H[e] = ghost_at<T>(g, phi, chat, gb, d, g.nbr[gb * 6 + d], g.cfslot[gb * 6 + d], u & 7, v & 7);
    }
    {
        const T *sv = reinterpret_cast<const T *>(&so);
        int row = ((oz + k) * 16 + oy + j) * 8 + (ox >> 1);
#pragma unroll
        for (int m = 0; m < 4; m++) S[row + m] = sv[m];
    }
    __syncthreads();
    const T *bb = reinterpret_cast<const T *>(&bv);
    V4 res;
    T *out = reinterpret_cast<T *>(&res);
    int J = oy + j, K = oz + k, row = (K * 16 + J) * 8;
#pragma unroll
    for (int m = 0; m < 4; m++) {
        int I = ox + 2 * m + ((j + k + C) & 1);
        T xm = I > 0 ? S[row + ((I - 1) >> 1)] : H[0 * 128 + K * 8 + (J >> 1)];
        T xp = I < 15 ? S[row + ((I + 1) >> 1)] : H[1 * 128 + K * 8 + (J >> 1)];
        T ym = J > 0 ? S[row - 8 + (I >> 1)] : H[2 * 128 + K * 8 + (I >> 1)];
        T yp = J < 15 ? S[row + 8 + (I >> 1)] : H[3 * 128 + K * 8 + (I >> 1)];
        T zm = K > 0 ? S[row - 128 + (I >> 1)] : H[4 * 128 + J * 8 + (I >> 1)];
        T zp = K < 15 ? S[row + 128 + (I >> 1)] : H[5 * 128 + J * 8 + (I >> 1)];
        T s = xm + xp + ym + yp + zm + zp;
        out[m] = (s - h2 * bb[m]) * (T)kSixth;
    }
    reinterpret_cast<V4 *>(phi + bx * 512 + C * 256)[rw] = res;
    if (IR) {
        ir_add<T, 4>(phi64, bx, C, 4 * rw, out, reinterpret_cast<const T *>(&so), rmask ? U + o * 512 : nullptr);
        if (rmask) {
            __syncthreads();
            if (rmask[bx]) restrict_box<double>(g, U + o * 512, bx, phi64, rw);
        }
    }
}

// One full red-black sweep (red half, then black half) of boxes [b0, b0+nbx)
// of one level, reading src and writing both colours to dst (src is left
// unchanged, dst must not alias it).  The values are those of the two
// half-sweeps of k_gsrb: the black half needs the new red values of the
// neighbours' face layers, so each box recomputes the 6 x 32 red cells of its
// same-level face neighbours that touch its black face cells, with the red
// update's own arithmetic on the old field (a red cell reads only black cells
// and ghosts).  One launch per sweep instead of two, with the same 24 B per
// cell plus the neighbours' face layers.  256 threads per box; thread t owns
// red cell t and black cell 256 + t (colour-split order), and in waves 0-2 one
// red and one black face cell of axis t / 64.
//
// What a thread does besides 7 FP64 operations a cell is finding addresses, so
// that is kept small: the box and its surroundings sit in LDS as one padded
// grid, cells -2..9 of each axis, colour-split like a box (rows of 6), where
// every ghost is stored in the cell that it stands for, so the six neighbours
// of a cell are at constant offsets from its own place; a wave holds the face
// entries of one axis, so that the axis is a scalar; a load reads one
// neighbour, from a scalar base; and all loads are issued before the first
// wait.  With the neighbours found by selects among the box and separate ghost
// arrays, and offsets per lane, a sweep of 64 boxes took 5.17 us, of 14224
// boxes 40.8 and of 187984 boxes 630 (FP64; FP32 4.92, 35.2 and 505); now 4.03,
// 34 and 540 (3.81, 25 and 400), against 6.2, 44.5 and 525 (5.9, 27.7 and 325)
// for two half-sweeps.
//
// The first sweep after a restriction can also complete the coarse
// right-hand side of the full approximation scheme (the values k_fas_rhs
// writes: L src + the restricted residual, on the boxes with children):
// fas = 1 computes it from src, which no workgroup writes, smooths with it
// and stores it in fasbuf; the right-hand side of a refined face neighbour
// under a recomputed red cell is formed the same way from the same inputs
// plus that cell's old value.  fas = 2 (the next sweep) reads those values
// from fasbuf and copies a box's own back into rhs; nothing reads rhs of a
// box with children meanwhile, so the copy races with no read.

// Places in the padded grid: red cells (i + j + k even) from 0, black from
// kSwC, the ghosts of the recomputed cells across the neighbour's tangential
// faces (6 faces x 4 edges x 4 cells: a place of the grid would have to hold
// two of them) from kSwE, and a FAS sweep's old red cells from kSwO.
constexpr int kSwC = 12 * 12 * 6, kSwE = 2 * kSwC, kSwO = kSwE + 96;
// Cell (layer, u, v) of a face of axis A (u, v along the tangential axes): its
// offset within a colour of a box, and its place in the grid within a colour.
template <int A> __device__ __forceinline__ int face_off(int layer, int u, int v) {
    return A == 0 ? v * 32 + u * 4 + (layer >> 1) : A == 1 ? v * 32 + layer * 4 + (u >> 1) : layer * 32 + v * 4 + (u >> 1);
}
template <int A> __device__ __forceinline__ int face_place(int layer, int u, int v) {
    return A == 0   ? (v + 2) * 72 + (u + 2) * 6 + ((layer + 2) >> 1)
           : A == 1 ? (v + 2) * 72 + (layer + 2) * 6 + ((u + 2) >> 1)
                    : (layer + 2) * 72 + (v + 2) * 6 + ((u + 2) >> 1);
}

template <typename T, bool FAS>
__global__ __launch_bounds__(256) void k_gsrb_sweep(Geo g, const T *__restrict__ src,
                                                    T *__restrict__ dst, T *__restrict__ rhs,
                                                    const T *__restrict__ chat, int64_t b0,
                                                    int64_t nbx, T h2, int xcd, int fas,
                                                    const int32_t *__restrict__ isleaf, T inv_h2,
                                                    T *__restrict__ fasbuf) {
    __shared__ T L[FAS ? kSwO + kSwC : kSwO];
    const int64_t lb = xcd ? xcd_map(blockIdx.x, nbx) : (int64_t)blockIdx.x;
    if (lb >= nbx) return;
    const int64_t b = b0 + lb;
    const int t = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);  // waves 0-2: the faces of axis w
    if (!FAS) fas = 0;
    const bool own_fas = fas != 0 && isleaf[b] == 0;
    const T *own = src + b * 512;
    T ob = own[256 + t];
    T br, bb;
    if (own_fas && fas == 2) {
        br = fasbuf[b * 512 + t];
        bb = fasbuf[b * 512 + 256 + t];
        rhs[b * 512 + t] = br;
        rhs[b * 512 + 256 + t] = bb;
    } else {
        br = rhs[b * 512 + t];
        bb = rhs[b * 512 + 256 + t];
    }
    T orr = (T)0;
    if (own_fas && fas == 1) orr = own[t];
    // this thread's cells: the same place in both colours' grids
    const int m = t & 3, j = (t >> 2) & 7, k = t >> 5;
    const int at = ((k + 2) * 12 + j + 2) * 6 + m + 1;
    const int odd = (j + k) & 1;  // the red cell is the row's second of the pair
    bool cf = false;
#pragma unroll
    for (int d = 0; d < 6; d++) cf = cf || g.nbr[b * 6 + d] == -1;
    // Face entries (waves 0-2, axis w): a lane holds one red face cell on side
    // hf and one black face cell on the other side (so a load from one
    // neighbour fills all lanes, from a scalar base), position (m, fv) of 4 x 8
    // in the layer.  lx, lo: the two sides' layers in the box; p_red: the place
    // of the red cell behind the black face cell.
    const int hf = (t >> 5) & 1, fv = (t >> 2) & 7, lx = 7 * hf, lo = 7 - lx;
    const int ur = 2 * m + ((lx + fv) & 1), ub = 2 * m + ((lo + fv + 1) & 1);
    int p_red = 0;
    bool same = false, slot = false, nb_fas = false;  // of the black face cell's face
    T bh = (T)0, nr = (T)0, ch = (T)0;
    auto load_faces = [&](auto A) __attribute__((always_inline)) {
        constexpr int a = decltype(A)::a, t1 = a == 0 ? 1 : 0, t2 = a == 2 ? 1 : 2;
        const int p_black = kSwC + face_place<a>(hf ? 8 : -1, ur, fv);
        p_red = face_place<a>(hf ? -1 : 8, ub, fv);
        // the black cell behind the red face cell and, on the other side, the
        // red cell to recompute (n_red) and the black cell behind that
        const int n_black = 256 + face_off<a>(lo, ur, fv), n_red = face_off<a>(lx, ub, fv);
        const int n_second = 256 + face_off<a>(hf ? 6 : 1, ub, fv);
        const int p_second = kSwC + face_place<a>(hf ? -2 : 9, ub, fv);
        // all loads are issued before the first value is stored in LDS
        const int nb0 = g.nbr[b * 6 + 2 * a], nb1 = g.nbr[b * 6 + 2 * a + 1];
        const bool f0 = fas != 0 && g.cfslot[b * 6 + 2 * a] == -2, f1 = fas != 0 && g.cfslot[b * 6 + 2 * a + 1] == -2;
        const int nbr_red = hf ? nb1 : nb0, nbr_black = hf ? nb0 : nb1;  // of the two face cells' faces
        const bool edge = (t & 31) < 16 && nbr_red >= 0;
        int2 x = make_int2(-2, -2);
        if (edge) x = reinterpret_cast<const int2 *>(g.xt)[(b * 6 + 2 * a + hf) * 4 + ((t >> 2) & 3)];
        T v0 = (T)0, v1 = (T)0, ev = (T)0;
        if (nb0 >= 0) {
            v0 = (src + (int64_t)nb0 * 512)[hf ? n_second : n_black];
            if (hf) bh = ((f0 && fas == 2 ? fasbuf : rhs) + (int64_t)nb0 * 512)[n_red];
            if (FAS && fas == 1 && hf) nr = (src + (int64_t)nb0 * 512)[n_red];
        }
        if (nb1 >= 0) {
            v1 = (src + (int64_t)nb1 * 512)[hf ? n_black : n_second];
            if (!hf) bh = ((f1 && fas == 2 ? fasbuf : rhs) + (int64_t)nb1 * 512)[n_red];
            if (FAS && fas == 1 && !hf) nr = (src + (int64_t)nb1 * 512)[n_red];
        }
        same = nbr_black >= 0;
        slot = nbr_black == -1;
        nb_fas = hf ? f0 : f1;
        if (edge) {
            // edge e4 (-t1, +t1, -t2, +t2) of the neighbour's layer, cell m
            // along it: the black cell across the neighbour's face there
            const int e4 = (t >> 2) & 3, end = (e4 & 1) ? 7 : 0, along = 2 * m + ((lx + 1 + (e4 & 1)) & 1);
            auto edge_off = [=](int across) { return face_off<a>(lo, e4 < 2 ? across : along, e4 < 2 ? along : across); };
            if (x.x >= 0) {
                ev = src[(int64_t)x.x * 512 + 256 + edge_off(7 - end)];
            } else {
                const T *N = src + (int64_t)nbr_red * 512;
                const int ef = (e4 < 2 ? 2 * t1 : 2 * t2) + (e4 & 1);
                // the cell on that face: u, v along the layer's axis and the
                // edge, in increasing order of axes
                const bool first = a < (e4 < 2 ? t2 : t1);
                const int eu = first ? lo : along, ew = first ? along : lo;
                ev = N[edge_off(end)];
                if (x.x == -1)
                    ev = cf_ghost<T>(chat[(int64_t)x.y * 64 + ew * 8 + eu], ev, N[256 + edge_off((e4 & 1) ? 6 : 1)]);
                else if (g.bct[ef] != 1)
                    ev = dirichlet_ghost<T>(bc_value<T>(g, nbr_red, ef, eu, ew), ev);
            }
        }
#pragma unroll
        for (int side = 0; side < 2; side++) {
            const int fd = 2 * a + side, nb = side ? nb1 : nb0;
            const bool red = hf == side;  // this side is the red face cell's
            if (nb >= 0) {
                L[red ? p_black : p_second] = side ? v1 : v0;
            } else if (nb == -2) {
                const T v = own[red ? face_off<a>(lx, ur, fv) : 256 + face_off<a>(lo, ub, fv)];
                const T gh = g.bct[fd] == 1 ? v : dirichlet_ghost<T>(bc_value<T>(g, b, fd, red ? ur : ub, fv), v);
                L[red ? p_black : p_red] = gh;
                if (FAS && !red) nr = gh;
            } else {
                const T c = chat[(int64_t)g.cfslot[b * 6 + fd] * 64 + fv * 8 + (red ? ur : ub)];
                if (red)
                    L[p_black] = cf_ghost<T>(c, own[face_off<a>(lx, ur, fv)], own[256 + face_off<a>(hf ? 6 : 1, ur, fv)]);
                else
                    ch = c;
            }
        }
        if (FAS) L[kSwO + p_red] = nr;
        if (edge) L[kSwE + 16 * (2 * a + hf) + (t & 15)] = ev;
    };
    if (w < 3) with_axis(w, load_faces);
    L[kSwC + at] = ob;
    if (own_fas && fas == 1) L[kSwO + at] = orr;
    __syncthreads();
    // neighbour sum of this thread's cell of the other colour than the grid R
    auto sum = [at](const T *R, int second) __attribute__((always_inline)) {
        const T *x = R + at - 1 + second, *y = R + at - 72;
        return x[0] + x[1] + y[66] + y[78] + y[0] + y[144];
    };
    if (own_fas && fas == 1) {  // black cell's right-hand side from the old field
        bb = (sum(L + kSwO, 1 - odd) - (T)6 * ob) * inv_h2 + bb;
        fasbuf[b * 512 + 256 + t] = bb;
    }
    {  // red cell (i + j + k even)
        const T sm = sum(L + kSwC, odd);
        if (own_fas && fas == 1) {
            br = (sm - (T)6 * orr) * inv_h2 + br;
            fasbuf[b * 512 + t] = br;
        }
        const T v = (sm - h2 * br) * (T)kSixth;
        L[at] = v;
        dst[b * 512 + t] = v;
    }
    // recomputed red cell of the same-level neighbour: its neighbours are at
    // constant offsets too, but for the edge ghosts at the ends of the layer
    auto recompute = [&](auto A) __attribute__((always_inline)) {
        constexpr int a = decltype(A)::a;
        const T *P = L + kSwC + p_red, *X = P - 1 + (a == 0 ? hf : ub & 1), *E = L + kSwE + 32 * a + 16 * (1 - hf);
        const T um = *(ub == 0 ? E + (fv >> 1) : a == 0 ? P - 6 : X);
        const T up = *(ub == 7 ? E + 4 + (fv >> 1) : a == 0 ? P + 6 : X + 1);
        const T vm = *(fv == 0 ? E + 8 + m : a == 2 ? P - 6 : P - 72);
        const T vp = *(fv == 7 ? E + 12 + m : a == 2 ? P + 6 : P + 72);
        const T nm = a == 0 ? X[0] : a == 1 ? P[-6] : P[-72], np = a == 0 ? X[1] : a == 1 ? P[6] : P[72];
        const T sm = a == 0 ? nm + np + um + up + vm + vp : a == 1 ? um + up + nm + np + vm + vp : um + up + vm + vp + nm + np;
        if (nb_fas && fas == 1) bh = (sm - (T)6 * nr) * inv_h2 + bh;
        L[p_red] = (sm - h2 * bh) * (T)kSixth;
    };
    if (same) with_axis(w, recompute);
    __syncthreads();
    if (cf) {  // block-uniform: the black ghosts at refinement boundaries read the new red cell behind
        auto ghosts = [&](auto A) __attribute__((always_inline)) {
            constexpr int a = decltype(A)::a;
            L[p_red] = cf_ghost<T>(ch, L[kSwC + face_place<a>(lo, ub, fv)], L[face_place<a>(hf ? 1 : 6, ub, fv)]);
        };
        if (slot) with_axis(w, ghosts);
        __syncthreads();
    }
    // black cell: its neighbours are new red values; domain ghosts as in the
    // black half-sweep (from the old black value)
    dst[b * 512 + 256 + t] = (sum(L, 1 - odd) - h2 * bb) * (T)kSixth;
}

// Coarse value of cell D = C + dir * e_ax (level l-1, relative to box Q),
// with the coarse physical ghost outside the domain; N is Q's neighbour
// across the face D leaves Q through.
template <typename T>
__device__ __forceinline__ T coarse_at(const Geo &g, const T *__restrict__ phi, int64_t Q,
                                       const int C[3], int ax, int dir, int N) {
    int D[3] = {C[0], C[1], C[2]};
    D[ax] += dir;
    if (D[ax] >= 0 && D[ax] < 8) return phi[Q * 512 + cs_idx3(D)];
    int face = 2 * ax + (dir > 0 ? 1 : 0);
    if (N >= 0) {
        D[ax] = dir > 0 ? 0 : 7;
        return phi[(int64_t)N * 512 + cs_idx3(D)];
    }
    T in = phi[Q * 512 + cs_idx3(C)];
    if (N != -2 || g.bct[face] == 1) return in;  // -1 cannot occur under 26-neighbour nesting
    int f1, f2;
    tangential(ax, f1, f2);
    T gv = (T)(g.bcval ? g.bcval[(Q * 6 + face) * 64 + C[f2] * 8 + C[f1]] : g.bcv[face]);
    return (T)2 * gv - in;
}

// Offset in a box of cell (layer, u, v) of a face of axis A.
template <int A> __device__ __forceinline__ int full_off(int layer, int u, int v) {
    return ((layer + u + v) & 1) * 256 +
           (A == 0 ? (v * 8 + u) * 4 + (layer >> 1) : A == 1 ? (v * 8 + layer) * 4 + (u >> 1) : (layer * 8 + v) * 4 + (u >> 1));
}

// Tangential quadratic interpolation of the coarse level at the 64 ghosts of
// one refinement-boundary face: c_hat = 7/8 c + sum_t [(1/32 + s_t/8) c_{+t}
// + (1/32 - s_t/8) c_{-t}], s_t = +-1 the side of the ghost in the coarse
// cell.  One 64-lane wavefront per face (slot s, wave-uniform).  The face's
// axis is a compile-time constant and the five loads go out together, a lane
// whose neighbour is across Q's face taking it from Q's neighbour N there, or,
// outside the domain, its own cell's place and the physical ghost afterwards.
// (Choosing axis, box and cell lane by lane, the c_hat of 104000 faces took 67.5
// us, now 43.7, of 18700 faces 12.0, now 8.2.)
template <int A, typename T>
__device__ __forceinline__ T cf_value(const Geo &g, const T *__restrict__ phi, const int4 x0, const int4 x1, int side,
                                      int lane) {
    constexpr int t1 = A == 0 ? 1 : 0, t2 = A == 2 ? 1 : 2;
    const int layer = side ? 0 : 7, u = lane & 7, v = lane >> 3;
    const int64_t Q = x0.x;
    const int c1 = x0.y + (u >> 1), c2 = x0.z + (v >> 1), nb[4] = {x0.w, x1.x, x1.y, x1.z};
    const T *q = phi + Q * 512;
    const int at = full_off<A>(layer, c1, c2);
    const T c = q[at];
    T n[4];  // -t1, +t1, -t2, +t2
    bool out[4];
#pragma unroll
    for (int e = 0; e < 4; e++) {
        const int N = nb[e], d = e & 1 ? 1 : -1, o1 = e < 2 ? c1 + d : c1, o2 = e < 2 ? c2 : c2 + d;
        out[e] = ((o1 | o2) & 8) != 0;
        const bool in = N >= 0 || !out[e];
        const T *p = out[e] && N >= 0 ? phi + (int64_t)N * 512 : q;
        n[e] = p[in ? full_off<A>(layer, o1 & 7, o2 & 7) : at];
    }
#pragma unroll
    for (int e = 0; e < 4; e++) {
        if (nb[e] != -2) continue;  // wave-uniform; -1 cannot occur under 26-neighbour nesting
        constexpr int f1[2] = {t1 == 0 ? 1 : 0, t2 == 0 ? 1 : 0}, f2[2] = {t1 == 2 ? 1 : 2, t2 == 2 ? 1 : 2};
        const int ax = e < 2 ? t1 : t2, face = 2 * ax + (e & 1);
        if (g.bct[face] == 1) continue;
        auto coord = [&](int f) { return f == A ? layer : f == t1 ? c1 : c2; };
        double gv = g.bcv[face];
        asm("" : "+s"(gv));  // (else one flat load through a selected address)
        if (g.bcval) gv = g.bcval[(Q * 6 + face) * 64 + coord(f2[e >> 1]) * 8 + coord(f1[e >> 1])];
        if (out[e]) n[e] = (T)2 * (T)gv - n[e];
    }
    T acc = (T)0.875 * c;
#pragma unroll
    for (int e = 0; e < 2; e++) {
        const T st = (((e ? v : u) & 1) ? (T)1 : (T)-1);
        acc += ((T)(1.0 / 32.0) + st / (T)8) * n[2 * e + 1] + ((T)(1.0 / 32.0) - st / (T)8) * n[2 * e];
    }
    return acc;
}
template <typename T>
__device__ __forceinline__ void cf_face(const Geo &g, const T *__restrict__ phi, T *__restrict__ chat,
                                        const int32_t *__restrict__ slots, int64_t s, int lane) {
    const int64_t sl = __builtin_amdgcn_readfirstlane((int)s);
    const int d = slots[2 * sl + 1];
    const int4 *x = reinterpret_cast<const int4 *>(g.slotx + 8 * sl);  // Q, base t1, base t2, Q's neighbours
    const int4 x0 = x[0], x1 = x[1];
    with_axis(d >> 1, [&](auto A) __attribute__((always_inline)) {
        chat[sl * 64 + lane] = cf_value<decltype(A)::a, T>(g, phi, x0, x1, d & 1, lane);
    });
}

// Four refinement-boundary faces per 256-thread block: slots [s0, s0+ns).
template <typename T>
__global__ __launch_bounds__(256) void k_cf_coarse(Geo g, const T *__restrict__ phi,
                                                   T *__restrict__ chat,
                                                   const int32_t *__restrict__ slots, int64_t s0,
                                                   int64_t ns) {
    int64_t s = 4 * (int64_t)blockIdx.x + (threadIdx.x >> 6);
    if (s >= ns) return;
    cf_face<T>(g, phi, chat, slots, s0 + s, threadIdx.x & 63);
}

// A whole box for a 7-point stencil on all of its cells, 128 threads: thread u
// holds the four cells i = 4 h .. 4 h + 3 (h = u & 1) of row j = (u >> 1) & 7,
// k = u >> 4, which are the colour positions 2u and 2u + 1 of both colours.
// The box and its y and z ghosts lie in a grid G[10][10][8] and the x ghosts in
// X[2][64], so that the rows on all sides are read in pairs at constant
// offsets; the ghosts of axis a are the a-th value of a thread (wave 0 the low
// side), so that the axis is a compile-time constant, and all loads go out
// before the first wait.  (With a colour-split copy and a table of ghosts, each
// of the 24 neighbour reads a thread picked its address; the stencil kernels
// then issued 900 to 1135 instructions a wavefront, now 500 to 690; on 206000
// boxes the stopping test went from 445 to 395 us.)
constexpr int kFullG = 800, kFullX = 128;
template <int A> __device__ __forceinline__ int full_place(int layer, int u, int v) {
    return A == 0 ? (v * 10 + u + 11) * 8 + layer : A == 1 ? ((v + 1) * 10 + layer + 1) * 8 + u : ((layer + 1) * 10 + v + 1) * 8 + u;
}
// The four cells of a thread from its two values of each colour, and back; odd
// = (j + k) & 1.
template <typename T, typename V>
__device__ __forceinline__ void to_cells(V c0, V c1, bool odd, T v[4]) {
    v[0] = odd ? c1.x : c0.x;
    v[1] = odd ? c0.x : c1.x;
    v[2] = odd ? c1.y : c0.y;
    v[3] = odd ? c0.y : c1.y;
}
// Stage box b (ZERO: of the zero field, which is not read) and leave the
// thread's cells in own.  Ends with a barrier.
template <typename T, bool ZERO>
__device__ __forceinline__ void full_stage(const Geo &g, const T *__restrict__ phi, const T *__restrict__ chat,
                                           int64_t b, T *G, T *X, T own[4]) {
    using V = typename VecN<T, 2>::type;
    const int u = threadIdx.x, side = __builtin_amdgcn_readfirstlane(u >> 6), fu = u & 7, fv = (u >> 3) & 7;
    const int edge = side ? 7 : 0, in = side ? 6 : 1;
    const FaceTab ft = face_tab(g, b);
    V p0, p1;
    p0.x = p0.y = p1.x = p1.y = (T)0;
    if (!ZERO) {
        p0 = reinterpret_cast<const V *>(phi + b * 512)[u];
        p1 = reinterpret_cast<const V *>(phi + b * 512 + 256)[u];
    }
    bool bnd = false;
#pragma unroll
    for (int d = 0; d < 6; d++) bnd = bnd || ft.nb[d] < 0;
    T raw[3];
    int nb[3];
    auto load = [&](auto A) __attribute__((always_inline)) {
        constexpr int a = decltype(A)::a;
        const int d = 2 * a + side, slot = side ? ft.slot[2 * a + 1] : ft.slot[2 * a];
        nb[a] = side ? ft.nb[2 * a + 1] : ft.nb[2 * a];
        raw[a] = (T)0;
        if (nb[a] >= 0) {
            if (!ZERO) raw[a] = (phi + (int64_t)nb[a] * 512)[full_off<a>(7 - edge, fu, fv)];
        } else if (nb[a] == -1) {
            raw[a] = (chat + (int64_t)slot * 64)[fv * 8 + fu];
        } else if (g.bcval) {
            raw[a] = (T)(g.bcval + (b * 6 + d) * 64)[fv * 8 + fu];
        }
    };
    load(Axis<0>());
    load(Axis<1>());
    load(Axis<2>());
    const int h = u & 1, j = (u >> 1) & 7, k = u >> 4, at = (k * 10 + j + 11) * 8 + 4 * h;
    to_cells<T, V>(p0, p1, (j + k) & 1, own);
    V w;
    w.x = own[0];
    w.y = own[1];
    *reinterpret_cast<V *>(G + at) = w;
    w.x = own[2];
    w.y = own[3];
    *reinterpret_cast<V *>(G + at + 2) = w;
    auto put = [&](auto A, T v) __attribute__((always_inline)) {
        constexpr int a = decltype(A)::a;
        if (a == 0)
            X[side * 64 + fv * 8 + fu] = v;
        else
            G[full_place<a>(side ? 8 : -1, fu, fv)] = v;
    };
    put(Axis<0>(), raw[0]);
    put(Axis<1>(), raw[1]);
    put(Axis<2>(), raw[2]);
    __syncthreads();
    if (bnd) {  // block-uniform: boundary ghosts read the box's cells
        auto ghost = [&](auto A) __attribute__((always_inline)) {
            constexpr int a = decltype(A)::a;
            if (nb[a] >= 0) return;
            const int d = 2 * a + side;
            T v = G[full_place<a>(edge, fu, fv)];
            if (nb[a] == -1)
                v = cf_ghost<T>(raw[a], v, G[full_place<a>(in, fu, fv)]);
            else if (g.bct[d] != 1)
                v = dirichlet_ghost<T>(g.bcval ? raw[a] : (T)g.bcv[d], v);
            put(A, v);
        };
        ghost(Axis<0>());
        ghost(Axis<1>());
        ghost(Axis<2>());
        __syncthreads();
    }
}
// The neighbour sums of the thread's four cells, in sum_full's order.
template <typename T> __device__ __forceinline__ void full_sums(const T *G, const T *X, const T own[4], T s[4]) {
    using V = typename VecN<T, 2>::type;
    const int u = threadIdx.x, h = u & 1, row = u >> 1, at = ((u >> 4) * 10 + (row & 7) + 11) * 8 + 4 * h;
    const T lo = *(h ? G + at - 1 : X + row), hi = *(h ? X + 64 + row : G + at + 4);
    s[0] = lo + own[1];
    s[1] = own[0] + own[2];
    s[2] = own[1] + own[3];
    s[3] = own[2] + hi;
#pragma unroll
    for (int q = 0; q < 4; q++) {
        const T *p = G + at + (q == 0 ? -8 : q == 1 ? 8 : q == 2 ? -80 : 80);
        const V a = *reinterpret_cast<const V *>(p), c = *reinterpret_cast<const V *>(p + 2);
        s[0] += a.x;
        s[1] += a.y;
        s[2] += c.x;
        s[3] += c.y;
    }
}
// Stages 16 .. 1 of a sum over 32 lanes (each half of a wavefront), every lane
// getting x[i] + x[i ^ w] in that order.  Below 16 the partner of a lane within
// its row of 16 is also w lanes on (the values repeat with period 2 w), which
// a row rotation reaches without LDS.
template <int W> __device__ __forceinline__ double row_ror(double x) {
    const uint64_t b = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, 0x120 + W, 0xf, 0xf, true);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x120 + W, 0xf, 0xf, true);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ double half_sum(double x) {
    x += __shfl_xor(x, 16);
    x += row_ror<8>(x);
    x += row_ror<4>(x);
    x += row_ror<2>(x);
    x += row_ror<1>(x);
    return x;
}
__device__ __forceinline__ double half_max(double x) {
    x = nanmax(__shfl_xor(x, 16), x);
    x = nanmax(row_ror<8>(x), x);
    x = nanmax(row_ror<4>(x), x);
    x = nanmax(row_ror<2>(x), x);
    x = nanmax(row_ror<1>(x), x);
    return x;
}
// Norms of a box from its thread's residuals: the sums follow k_leaf_norms' tree
// over the 256 positions (stages 32..2 over the threads, stage 1 the pair), so
// the partials are the same bits.
__device__ __forceinline__ void full_norms(const double r[4], bool odd, double *S, double *M) {
    const int u = threadIdx.x;
    // position 2u is cells 0 and 1, position 2u + 1 cells 2 and 3, red first
    const double s0 = half_sum(fmadd(odd ? r[0] : r[1], odd ? r[0] : r[1], (odd ? r[1] : r[0]) * (odd ? r[1] : r[0])));
    const double s1 = half_sum(fmadd(odd ? r[2] : r[3], odd ? r[2] : r[3], (odd ? r[3] : r[2]) * (odd ? r[3] : r[2])));
    const double m = half_max(nanmax(nanmax(fabs(r[0]), fabs(r[1])), nanmax(fabs(r[2]), fabs(r[3]))));
    if ((u & 31) == 0) {
        S[u >> 5] = s0 + s1;
        M[u >> 5] = m;
    }
}

// Residual on level l and restriction to level l-1 (full approximation
// scheme): the residual of all 512 cells goes to LDS, then each of 64 threads
// owns one parent cell and writes phi_c = mean(phi), old_c = phi_c and
// rhs_c = mean(residual) (the coarse right-hand side is completed by
// k_fas_rhs).  Extra blocks copy phi -> old on the listed leaf boxes of level
// l-1 (those with a refined face or edge neighbour: the only leaf boxes whose
// old values a prolongation reads).
//
// ZERO: phi is zero on every level (the top-down pass of an FMG solve from
// phi = 0), so it is not read: the box is zero and its ghosts are those of
// the zero field (the boundary data and the refinement-boundary values
// c_hat of the zero field), which are the values the general path reads and
// forms.  The residual of a leaf box is then the residual of phi = 0, and
// the box also writes its volume-weighted sum of r^2 and max |r| at its leaf
// position leafpos[b] of `partial`, with the arithmetic and the summation
// order of k_leaf_norms (the norm the stopping test divides by).
template <typename T, bool ZERO>
__global__ __launch_bounds__(128) void k_resid_restrict(Geo g, T *__restrict__ phi, T *__restrict__ rhs,
                                                        T *__restrict__ old, const T *__restrict__ chat,
                                                        int64_t b0, int64_t nbx,
                                                        const int32_t *__restrict__ leaf_prev,
                                                        int64_t nleaf_prev, T inv_h2,
                                                        const int32_t *__restrict__ leafpos,
                                                        double *__restrict__ partial, double vol) {
    using V = typename VecN<T, 2>::type;
    __shared__ __attribute__((aligned(16))) T G[kFullG], X[kFullX], R[512];
    __shared__ double S[4], M[4];
    int64_t blk = blockIdx.x;
    const int u = threadIdx.x;
    int64_t nmain = xcd_grid(nbx);
    if (blk >= nmain) {
        int64_t q = blk - nmain;
        if (q >= nleaf_prev) return;
        int64_t p = leaf_prev[q];
        V *dst = reinterpret_cast<V *>(old + p * 512);
        const V *src = reinterpret_cast<const V *>(phi + p * 512);
        V z;
        z.x = (T)0;
        z.y = (T)0;
        dst[u] = ZERO ? z : src[u];
        dst[128 + u] = ZERO ? z : src[128 + u];
        return;
    }
    int64_t lb = xcd_map(blk, nbx);
    if (lb >= nbx) return;
    int64_t b = b0 + lb;
    // indices of the parent cells, loaded with the data (not after the barriers)
    const int64_t p = g.parent[b];
    const int bi = g.ijk[b * 4] & 1, bj = g.ijk[b * 4 + 1] & 1, bk = g.ijk[b * 4 + 2] & 1;
    const V r0 = ld_stream(reinterpret_cast<const V *>(rhs + b * 512) + u);
    const V r1 = ld_stream(reinterpret_cast<const V *>(rhs + b * 512 + 256) + u);
    T own[4], sm[4], f[4];
    full_stage<T, ZERO>(g, phi, chat, b, G, X, own);
    const bool odd = ((u >> 1) + (u >> 4)) & 1;
    to_cells<T, V>(r0, r1, odd, f);
    full_sums<T>(G, X, own, sm);
#pragma unroll
    for (int q = 0; q < 4; q++) sm[q] = resid_of<T>(f[q], sm[q], own[q], inv_h2);
#pragma unroll
    for (int q = 0; q < 2; q++) {
        V w;
        w.x = sm[2 * q];
        w.y = sm[2 * q + 1];
        *reinterpret_cast<V *>(R + 4 * u + 2 * q) = w;  // natural order
    }
    if (ZERO && leafpos[b] >= 0) {  // block-uniform
        const double r[4] = {(double)sm[0], (double)sm[1], (double)sm[2], (double)sm[3]};
        full_norms(r, odd, S, M);
    }
    __syncthreads();
    if (ZERO && u == 0 && leafpos[b] >= 0) {
        int64_t q = leafpos[b];
        partial[2 * q] = ((S[0] + S[1]) + (S[2] + S[3])) * vol;
        partial[2 * q + 1] = nanmax(nanmax(M[0], M[1]), nanmax(M[2], M[3]));
    }
    // a parent cell a thread: wave 0 the mean of phi, wave 1 of the residual
    const int pi = u & 3, pj = (u >> 2) & 3, pk = (u >> 4) & 3;
    const bool res = __builtin_amdgcn_readfirstlane(u >> 6);
    const T *src = res ? R + (pk * 16 + pj * 2) * 8 + 2 * pi : G + (pk * 20 + pj * 2 + 11) * 8 + 2 * pi;
    const int zs = res ? 64 : 80;
    T mean = 0;
#pragma unroll
    for (int dk = 0; dk < 2; dk++)
#pragma unroll
        for (int dj = 0; dj < 2; dj++) {
            const V w = *reinterpret_cast<const V *>(src + dk * zs + dj * 8);
            mean += w.x;
            mean += w.y;
        }
    mean = (T)0.125 * mean;
    const int64_t pc = p * 512 + cs_idx(4 * bi + pi, 4 * bj + pj, 4 * bk + pk);
    if (res) {
        rhs[pc] = mean;
    } else {
        phi[pc] = mean;
        old[pc] = mean;
    }
}

// rhs <- L phi + rhs on the listed (refined) boxes: completes the coarse
// right-hand side L_c(R phi) + R r of the full approximation scheme.
template <typename T>
__global__ __launch_bounds__(128) void k_fas_rhs(Geo g, const T *__restrict__ phi, T *__restrict__ rhs,
                                                 const T *__restrict__ chat,
                                                 const int32_t *__restrict__ list, int64_t nlist,
                                                 T inv_h2) {
    using V = typename VecN<T, 2>::type;
    __shared__ __attribute__((aligned(16))) T G[kFullG], X[kFullX];
    int64_t q = xcd_map(blockIdx.x, nlist);
    if (q >= nlist) return;
    int64_t b = list[q];
    const int u = threadIdx.x;
    const V r0 = ld_stream(reinterpret_cast<const V *>(rhs + b * 512) + u);
    const V r1 = ld_stream(reinterpret_cast<const V *>(rhs + b * 512 + 256) + u);
    T own[4], s[4], f[4];
    full_stage<T, false>(g, phi, chat, b, G, X, own);
    const bool odd = ((u >> 1) + (u >> 4)) & 1;
    to_cells<T, V>(r0, r1, odd, f);
    full_sums<T>(G, X, own, s);
#pragma unroll
    for (int e = 0; e < 4; e++) s[e] = (s[e] - (T)6 * own[e]) * inv_h2 + f[e];
    V w;
    w.x = odd ? s[1] : s[0];
    w.y = odd ? s[3] : s[2];
    reinterpret_cast<V *>(rhs + b * 512)[u] = w;
    w.x = odd ? s[0] : s[1];
    w.y = odd ? s[2] : s[3];
    reinterpret_cast<V *>(rhs + b * 512 + 256)[u] = w;
}

// phi_f += 1/4 delta(C) + 1/4 (delta(C + s_x) + delta(C + s_y) + delta(C + s_z))
// with delta = phi - old on the parent level, C the parent cell and s the
// side of the fine cell inside it.  The parent's delta over the child's
// octant and its face-adjacent layer is staged in D[6][6][6] (outside the
// parent: the same-level neighbour or the homogeneous physical ghost): wave 0
// the octant, the others the two layers of one axis, and the two cells of a
// thread share their parent cell (with each of the 216 entries finding its box
// and cell, 64 boxes took 2.81 us, 14224 boxes 25.4; now 2.40 and 23.9).  Extra
// blocks compute c_hat for the refinement-boundary faces of level l (which
// read only level l-1, like the prolongation).
template <typename T>
__global__ __launch_bounds__(256) void k_prolong_cf(Geo g, T *__restrict__ phi, const T *__restrict__ old,
                                                    int64_t b0, int64_t nbx, T *__restrict__ chat,
                                                    const int32_t *__restrict__ slots, int64_t s0,
                                                    int64_t ns) {
    __shared__ T D[216];
    int64_t blk = blockIdx.x;
    int t = threadIdx.x;
    int64_t nmain = xcd_grid(nbx);
    if (blk >= nmain) {
        int64_t s = 4 * (blk - nmain) + (t >> 6);
        if (s < ns) cf_face<T>(g, phi, chat, slots, s0 + s, t & 63);
        return;
    }
    int64_t lb = xcd_map(blk, nbx);
    if (lb >= nbx) return;
    int64_t b = b0 + lb;
    const int64_t p = g.parent[b];
    const int o0 = g.ijk[b * 4] & 1, o1 = g.ijk[b * 4 + 1] & 1, o2 = g.ijk[b * 4 + 2] & 1;
    // this box's values, loaded with the correction (not after the barrier)
    const T f0 = phi[b * 512 + t], f1 = phi[b * 512 + 256 + t];
    const int w = __builtin_amdgcn_readfirstlane(t >> 6), x4 = t & 3, y4 = (t >> 2) & 3, z4 = (t >> 4) & 3;
    if (w == 0) {  // the octant's own 4^3 cells
        const int64_t q = p * 512 + cs_idx(4 * o0 + x4, 4 * o1 + y4, 4 * o2 + z4);
        D[((z4 + 1) * 6 + y4 + 1) * 6 + x4 + 1] = phi[q] - old[q];
    } else if ((t & 63) < 32) {
        // the layers on both sides of axis w - 1: inside the parent, or, on the
        // side of the parent's own face, in its neighbour N there
        with_axis(w - 1, [&](auto A) __attribute__((always_inline)) {
            constexpr int a = decltype(A)::a;
            const int o = a == 0 ? o0 : a == 1 ? o1 : o2, s = (t >> 4) & 1;
            const int N = g.nbr[p * 6 + 2 * a + o];
            const bool outer = s == o;
            const int layer = !outer ? (s ? 4 : 3) : (N >= 0) == (s != 0) ? 0 : 7;
            const int64_t q = (outer && N >= 0 ? (int64_t)N : p) * 512 +
                              full_off<a>(layer, 4 * (a == 0 ? o1 : o0) + x4, 4 * (a == 2 ? o1 : o2) + y4);
            const T d = phi[q] - old[q];
            const int at = 5 * s;
            // outside the domain (a refined box has no refinement-boundary
            // face): the homogeneous physical ghost
            D[a == 0 ? ((y4 + 1) * 6 + x4 + 1) * 6 + at : a == 1 ? ((y4 + 1) * 6 + at) * 6 + x4 + 1 : (at * 6 + y4 + 1) * 6 + x4 + 1] =
                outer && N < 0 && g.bct[2 * a + o] != 1 ? -d : d;
        });
    }
    __syncthreads();
    // the two cells of a thread, i = 2 m and 2 m + 1, have one parent cell
    const int m = t & 3, j = (t >> 2) & 7, k = t >> 5, odd = (j + k) & 1;
    const T *C = D + (((k >> 1) + 1) * 6 + (j >> 1) + 1) * 6 + m + 1;
    const T d0 = C[0], dy = C[(j & 1) ? 6 : -6], dz = C[(k & 1) ? 36 : -36], lo = C[-1], hi = C[1];
    phi[b * 512 + t] = f0 + ((T)0.25 * d0 + (T)0.25 * ((odd ? hi : lo) + dy + dz));
    phi[b * 512 + 256 + t] = f1 + ((T)0.25 * d0 + (T)0.25 * ((odd ? lo : hi) + dy + dz));
}

// ------------------------------------- prolongation fused into the up-sweep
// The first red-black sweep after the prolongation of a level reads the
// prolonged field only where the red and the black half-sweeps read it: the
// red half reads every black cell (its own, and the neighbours' face layers
// as ghosts) and, for the boundary ghosts of its face cells, the red face
// cells on domain and refinement-boundary faces; the black half reads the
// new red cells and, for the same boundary ghosts, its own black face cells
// on those faces.  Every other prolonged value is overwritten unread.  So the
// two half-sweeps below take the prolonged value f + p(delta) of each cell
// they read on the fly, from the unprolonged field and the parent's
// correction delta = phi - old, and nothing writes the prolongation itself:
// the level ends the sweep with the values of the prolongation followed by
// the two half-sweeps (same arithmetic in the same order, so the same bits).
//
// The correction is staged once per refined box P of level l-1 (k_delta_pad)
// as a padded block of 10^3 values, x fastest: delta over P's cells and one
// cell layer around them.  The layer comes from P's same-level face and edge
// neighbours (corners are never read: a fine cell's stencil steps at most
// one coarse cell along each of two axes from P's face layers), or outside
// the domain from P's own cell mirrored, with the sign of the homogeneous
// boundary condition (Dirichlet -, Neumann +), as k_prolong_cf takes it.  The
// children of the k-th refined box of level l-1 are the boxes 8k .. 8k+7 of
// level l (canonical order), octant = position & 7, and read the 6^3
// sub-block 4 o + 0..5 of block k.  Waves 0-2 hold the faces of one axis, wave 3
// the edges, and the block goes through LDS to be written in order (with each
// of the 1000 values finding its own box and cell, 680 vector instructions a
// wavefront, 23500 blocks with the c_hat of 75000 faces took 180 us, now 144).
template <typename T>
__global__ __launch_bounds__(256) void k_delta_pad(Geo g, const T *__restrict__ phi, const T *__restrict__ old,
                                                   const int32_t *__restrict__ refined, int64_t nref,
                                                   T *__restrict__ pad, T *__restrict__ chat,
                                                   const int32_t *__restrict__ slots, int64_t s0, int64_t ns) {
    __shared__ __attribute__((aligned(16))) T D[1000];
    int64_t blk = blockIdx.x;
    int t = threadIdx.x;
    int64_t nmain = xcd_grid(nref);
    if (blk >= nmain) {  // c_hat of the refinement-boundary faces of level l (reads level l-1 only)
        int64_t sl = 4 * (blk - nmain) + (t >> 6);
        if (sl < ns) cf_face<T>(g, phi, chat, slots, s0 + sl, t & 63);
        return;
    }
    int64_t k = xcd_map(blk, nref);
    if (k >= nref) return;
    const int64_t P = refined[k];
    const int32_t *NP = g.n27 + P * 27;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    T own[2], lay[2];
    int place[2] = {0, 0};
#pragma unroll
    for (int c = 0; c < 2; c++) own[c] = phi[P * 512 + 256 * c + t] - old[P * 512 + 256 * c + t];
    auto faces = [&](auto A) __attribute__((always_inline)) {
        constexpr int a = decltype(A)::a, step = a == 0 ? 1 : a == 1 ? 3 : 9;
        const int u = lane & 7, v = lane >> 3;
#pragma unroll
        for (int s = 0; s < 2; s++) {
            const int q = NP[s ? 13 + step : 13 - step];
            place[s] = a == 0 ? (v * 10 + u + 11) * 10 + 9 * s : a == 1 ? ((v + 1) * 10 + 9 * s) * 10 + u + 1 : (90 * s + v + 1) * 10 + u + 1;
            lay[s] = (T)0;
            if (q != -1) {  // always, for every value a prolongation reads (proper nesting)
                // P's face on this side is a domain face: its own cell, mirrored
                const int64_t at = (q >= 0 ? (int64_t)q : P) * 512 + full_off<a>((q >= 0) == (s != 0) ? 0 : 7, u, v);
                const T d = phi[at] - old[at];
                lay[s] = q < 0 && g.bct[2 * a + s] != 1 ? -d : d;
            }
        }
    };
    if (w < 3) {
        with_axis(w, faces);
    } else {  // the 12 edges: two rows of 8 values a half-wavefront, then one
        const int np = NP[min(lane, 26)];
        uint32_t odd_faces = 0;  // with a sign change
#pragma unroll
        for (int d = 0; d < 6; d++) odd_faces |= (uint32_t)(g.bct[d] != 1) << d;
#pragma unroll
        for (int r = 0; r < 2; r++) {
            const int e = lane + 64 * r, id = min(e, 95) >> 3, at0 = e & 7;
            const int al = id >> 2, b = al == 0 ? 1 : 0, c = al == 2 ? 1 : 2, sb = id & 1, sc = (id >> 1) & 1;
            const int wb = b == 0 ? 1 : 3, wc = c == 1 ? 3 : 9;
            int ob = sb ? wb : -wb, oc = sc ? wc : -wc;
            const bool mb = __shfl(np, 13 + ob) == -2, mc = __shfl(np, 13 + oc) == -2;
            const int xb = mb == (sb != 0) ? 7 : 0, xc = mc == (sc != 0) ? 7 : 0;
            const bool neg = ((mb ? odd_faces >> (2 * b + sb) : 0u) ^ (mc ? odd_faces >> (2 * c + sc) : 0u)) & 1u;
            const int q = __shfl(np, 13 + (mb ? 0 : ob) + (mc ? 0 : oc));
            lay[r] = (T)0;
            if (q >= 0) {
                const int i = al == 0 ? at0 : xb, j = al == 1 ? at0 : al == 0 ? xb : xc, kk = al == 2 ? at0 : xc;
                const int64_t at = (int64_t)q * 512 + cs_idx(i, j, kk);
                const T d = phi[at] - old[at];
                lay[r] = neg ? -d : d;
            }
            const int pb = 9 * sb, pc = 9 * sc, pa = at0 + 1;
            place[r] = (al == 2 ? pa : pc) * 100 + (al == 1 ? pa : al == 0 ? pb : pc) * 10 + (al == 0 ? pa : pb);
        }
    }
    {
        const int m = t & 3, j = (t >> 2) & 7, kk = t >> 5, i = 2 * m + ((j + kk) & 1);
        T *row = D + (kk * 10 + j + 11) * 10 + 1;
        row[i] = own[0];
        row[i ^ 1] = own[1];
    }
    D[place[0]] = lay[0];
    if (w < 3 || lane < 32) D[place[1]] = lay[1];
    if (t < 8) D[900 * (t >> 2) + 90 * ((t >> 1) & 1) + 9 * (t & 1)] = (T)0;
    __syncthreads();
    using V = typename VecN<T, 2>::type;
    V *out = reinterpret_cast<V *>(pad + k * 1000);
    out[t] = reinterpret_cast<const V *>(D)[t];
    if (t < 244) out[256 + t] = reinterpret_cast<const V *>(D)[256 + t];
}
// Offset of the 6^3 correction region of the box at position lb of its level
// (octant lb & 7) in its parent's padded block, and of region cell e
// (x fastest) from there.
__device__ __forceinline__ int pad_corner(int64_t lb) {
    int o = (int)(lb & 7);
    return 4 * ((o & 1) + 10 * ((o >> 1) & 1) + 100 * (o >> 2));
}
__device__ __forceinline__ int pad_off(int e) { return e % 6 + 10 * ((e / 6) % 6) + 100 * (e / 36); }
// Prolonged correction at fine cell (i, j, k) of the box, i, j, k in -1..8
// (at most one outside 0..7: a face ghost), as k_prolong_cf adds it.
template <typename T>
__device__ __forceinline__ T prolonged(const T *D, int i, int j, int k) {
    int x = (i + 2) >> 1, y = (j + 2) >> 1, z = (k + 2) >> 1;
    int sx = ((i + 2) & 1) ? 1 : -1, sy = ((j + 2) & 1) ? 6 : -6, sz = ((k + 2) & 1) ? 36 : -36;
    int at = (z * 6 + y) * 6 + x;
    T d0 = D[at], dx = D[at + sx], dy = D[at + sy], dz = D[at + sz];
    return (T)0.25 * d0 + (T)0.25 * (dx + dy + dz);
}
// The face cell of face d at tangential (u, v) and layer `layer` (0..7, or
// -1 / 8 outside the box), as (i, j, k)
__device__ __forceinline__ void face_cell(int d, int layer, int u, int v, int &i, int &j, int &k) {
    int a = d >> 1, t1, t2;
    tangential(a, t1, t2);
    int c[3];
    c[a] = layer;
    c[t1] = u;
    c[t2] = v;
    i = c[0];
    j = c[1];
    k = c[2];
}

// Red half of the first sweep after the prolongation into boxes [b0,
// b0+nbx) of level l >= 2 (128 threads, 2 cells each, XCD-aware mapping).
// LDS: S the prolonged black cells, H the ghosts of the red face cells, D
// the correction region.  Same-level ghost: the neighbour's black cell +
// its prolonged correction; domain and refinement-boundary ghosts from the
// prolonged red face cell (and, at a refinement boundary, the prolonged
// black cell behind it).  Writes the red cells only.
template <typename T>
__global__ __launch_bounds__(128) void k_gsrb_pro_red(Geo g, T *__restrict__ phi, const T *__restrict__ rhs,
                                                      const T *__restrict__ pad, const T *__restrict__ chat,
                                                      int64_t b0, int64_t nbx, T h2) {
    using V = typename VecN<T, 2>::type;
    __shared__ T S[256], H[192], D[216];
    int64_t lb = xcd_map(blockIdx.x, nbx);
    if (lb >= nbx) return;
    int64_t b = b0 + lb;
    const int t = threadIdx.x;
    const FaceTab ft = face_tab(g, b);
    V blk = reinterpret_cast<const V *>(phi + b * 512 + 256)[t];
    V bv = ld_stream(reinterpret_cast<const V *>(rhs + b * 512) + t);
    const T *pk = pad + (lb >> 3) * 1000 + pad_corner(lb);
    T dv0 = pk[pad_off(t)];
    T dv1 = t + 128 < 216 ? pk[pad_off(t + 128)] : (T)0;
    // ghost entries e = t, t + 128 (< 192): face d, red face cell (u, v) at layer L
    T raw[2], in_raw[2], ch[2];
#pragma unroll
    for (int r = 0; r < 2; r++) {
        int e = t + 128 * r;
        raw[r] = in_raw[r] = ch[r] = (T)0;
        if (e >= 192) continue;
        int d = e >> 5, q = e & 31, v = q >> 2, L = (d & 1) ? 7 : 0;
        int u = 2 * (q & 3) + ((L + v) & 1);
        int nb = pick6(ft.nb, d), i, j, k;
        if (nb >= 0) {
            face_cell(d, (d & 1) ? 0 : 7, u, v, i, j, k);  // mirrored cell in the neighbour
            raw[r] = phi[(int64_t)nb * 512 + cs_idx(i, j, k)];
        } else {
            face_cell(d, L, u, v, i, j, k);
            raw[r] = phi[b * 512 + cs_idx(i, j, k)];
            if (nb == -1) {
                face_cell(d, (d & 1) ? 6 : 1, u, v, i, j, k);
                in_raw[r] = phi[b * 512 + cs_idx(i, j, k)];
                ch[r] = chat[(int64_t)pick6(ft.slot, d) * 64 + v * 8 + u];
            }
        }
    }
    D[t] = dv0;
    if (t + 128 < 216) D[t + 128] = dv1;
    __syncthreads();
    {
        const T *bl = reinterpret_cast<const T *>(&blk);
        V sv;
        T *so = reinterpret_cast<T *>(&sv);
#pragma unroll
        for (int w = 0; w < 2; w++) {
            int cq = 2 * t + w;
            int m = cq & 3, j = (cq >> 2) & 7, k = cq >> 5;
            int i = 2 * m + ((j + k + 1) & 1);
            so[w] = bl[w] + prolonged<T>(D, i, j, k);
        }
        reinterpret_cast<V *>(S)[t] = sv;
    }
#pragma unroll
    for (int r = 0; r < 2; r++) {
        int e = t + 128 * r;
        if (e >= 192) continue;
        int d = e >> 5, q = e & 31, v = q >> 2, L = (d & 1) ? 7 : 0;
        int u = 2 * (q & 3) + ((L + v) & 1);
        int nb = pick6(ft.nb, d), i, j, k;
        T gv;
        if (nb >= 0) {
            face_cell(d, (d & 1) ? 8 : -1, u, v, i, j, k);
            gv = raw[r] + prolonged<T>(D, i, j, k);
        } else {
            face_cell(d, L, u, v, i, j, k);
            T own = raw[r] + prolonged<T>(D, i, j, k);
            if (nb == -2) {
                gv = g.bct[d] == 1 ? own : dirichlet_ghost<T>(bc_value<T>(g, b, d, u, v), own);
            } else {
                face_cell(d, (d & 1) ? 6 : 1, u, v, i, j, k);
                gv = cf_ghost<T>(ch[r], own, in_raw[r] + prolonged<T>(D, i, j, k));
            }
        }
        H[e] = gv;
    }
    __syncthreads();
    const T *bb = reinterpret_cast<const T *>(&bv);
    V res;
    T *out = reinterpret_cast<T *>(&res);
#pragma unroll
    for (int w = 0; w < 2; w++) {
        int cq = 2 * t + w;
        int m = cq & 3, j = (cq >> 2) & 7, k = cq >> 5;
        int i = 2 * m + ((j + k) & 1);
        int row = (k * 8 + j) * 4;
        T xm = i > 0 ? S[row + ((i - 1) >> 1)] : H[0 * 32 + k * 4 + (j >> 1)];
        T xp = i < 7 ? S[row + ((i + 1) >> 1)] : H[1 * 32 + k * 4 + (j >> 1)];
        T ym = j > 0 ? S[row - 4 + m] : H[2 * 32 + k * 4 + m];
        T yp = j < 7 ? S[row + 4 + m] : H[3 * 32 + k * 4 + m];
        T zm = k > 0 ? S[row - 32 + m] : H[4 * 32 + j * 4 + m];
        T zp = k < 7 ? S[row + 32 + m] : H[5 * 32 + j * 4 + m];
        T sm = xm + xp + ym + yp + zm + zp;
        out[w] = (sm - h2 * bb[w]) * (T)kSixth;
    }
    reinterpret_cast<V *>(phi + b * 512)[t] = res;
}

// Black half of the first sweep after the prolongation: as k_gsrb<1, T, 2>,
// except that the ghosts of black face cells on domain and
// refinement-boundary faces take the prolonged black face cell (its
// unprolonged value + the correction, from the correction region, staged
// only by boxes with such faces).
template <typename T>
__global__ __launch_bounds__(128) void k_gsrb_pro_black(Geo g, T *__restrict__ phi, const T *__restrict__ rhs,
                                                        const T *__restrict__ pad, const T *__restrict__ chat,
                                                        int64_t b0, int64_t nbx, T h2) {
    using V = typename VecN<T, 2>::type;
    __shared__ T S[256], H[192], D[216];
    int64_t lb = xcd_map(blockIdx.x, nbx);
    if (lb >= nbx) return;
    int64_t b = b0 + lb;
    const int t = threadIdx.x;
    const FaceTab ft = face_tab(g, b);
    bool bnd = false;
#pragma unroll
    for (int d = 0; d < 6; d++) bnd = bnd || ft.nb[d] < 0;
    V o = reinterpret_cast<const V *>(phi + b * 512)[t];
    V bv = ld_stream(reinterpret_cast<const V *>(rhs + b * 512 + 256) + t);
    T raw[2], in_new[2], ch[2];
#pragma unroll
    for (int r = 0; r < 2; r++) {
        int e = t + 128 * r;
        raw[r] = in_new[r] = ch[r] = (T)0;
        if (e >= 192) continue;
        int d = e >> 5, q = e & 31, v = q >> 2, L = (d & 1) ? 7 : 0;
        int u = 2 * (q & 3) + ((L + v + 1) & 1);
        int nb = pick6(ft.nb, d), i, j, k;
        if (nb >= 0) {
            face_cell(d, (d & 1) ? 0 : 7, u, v, i, j, k);
            raw[r] = phi[(int64_t)nb * 512 + cs_idx(i, j, k)];  // the neighbour's new red cell
        } else {
            face_cell(d, L, u, v, i, j, k);
            raw[r] = phi[b * 512 + cs_idx(i, j, k)];  // own black face cell, unprolonged
            if (nb == -1) {
                face_cell(d, (d & 1) ? 6 : 1, u, v, i, j, k);
                in_new[r] = phi[b * 512 + cs_idx(i, j, k)];  // new red cell behind it
                ch[r] = chat[(int64_t)pick6(ft.slot, d) * 64 + v * 8 + u];
            }
        }
    }
    if (bnd) {
        const T *pk = pad + (lb >> 3) * 1000 + pad_corner(lb);
        T dv0 = pk[pad_off(t)];
        T dv1 = t + 128 < 216 ? pk[pad_off(t + 128)] : (T)0;
        D[t] = dv0;
        if (t + 128 < 216) D[t + 128] = dv1;
    }
    reinterpret_cast<V *>(S)[t] = o;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 2; r++) {
        int e = t + 128 * r;
        if (e >= 192) continue;
        int d = e >> 5, q = e & 31, v = q >> 2, L = (d & 1) ? 7 : 0;
        int u = 2 * (q & 3) + ((L + v + 1) & 1);
        int nb = pick6(ft.nb, d), i, j, k;
        T gv = raw[r];
        if (nb < 0) {
            face_cell(d, L, u, v, i, j, k);
            T own = raw[r] + prolonged<T>(D, i, j, k);
            if (nb == -2)
                gv = g.bct[d] == 1 ? own : dirichlet_ghost<T>(bc_value<T>(g, b, d, u, v), own);
            else
                gv = cf_ghost<T>(ch[r], own, in_new[r]);
        }
        H[e] = gv;
    }
    __syncthreads();
    const T *bb = reinterpret_cast<const T *>(&bv);
    V res;
    T *out = reinterpret_cast<T *>(&res);
#pragma unroll
    for (int w = 0; w < 2; w++) {
        int cq = 2 * t + w;
        int m = cq & 3, j = (cq >> 2) & 7, k = cq >> 5;
        int i = 2 * m + ((j + k + 1) & 1);
        int row = (k * 8 + j) * 4;
        T xm = i > 0 ? S[row + ((i - 1) >> 1)] : H[0 * 32 + k * 4 + (j >> 1)];
        T xp = i < 7 ? S[row + ((i + 1) >> 1)] : H[1 * 32 + k * 4 + (j >> 1)];
        T ym = j > 0 ? S[row - 4 + m] : H[2 * 32 + k * 4 + m];
        T yp = j < 7 ? S[row + 4 + m] : H[3 * 32 + k * 4 + m];
        T zm = k > 0 ? S[row - 32 + m] : H[4 * 32 + j * 4 + m];
        T zp = k < 7 ? S[row + 32 + m] : H[5 * 32 + j * 4 + m];
        T sm = xm + xp + ym + yp + zm + zp;
        out[w] = (sm - h2 * bb[w]) * (T)kSixth;
    }
    reinterpret_cast<V *>(phi + b * 512 + 256)[t] = res;
}

// Exact solve on each root box by fast diagonalisation: with the 1-D
// eigenbases V_a, phi = (V_z x V_y x V_x) diag(h^2 / (l_x + l_y + l_z))
// (V_z x V_y x V_x)^T rhs, where rhs has the Dirichlet data folded in.
template <typename T>
__global__ __launch_bounds__(512) void k_coarse(Geo g, T *__restrict__ phi, const T *__restrict__ rhs,
                                                const double *__restrict__ eig, int64_t b0, double h) {
    __shared__ double X[512], Y[512], V[192], L[24];
    int64_t b = b0 + blockIdx.x;
    int t = threadIdx.x, i = t & 7, j = (t >> 3) & 7, k = t >> 6;
    if (t < 192) V[t] = eig[t];
    if (t < 24) L[t] = eig[192 + t];
    int c[3] = {i, j, k};
    double r = (double)rhs[b * 512 + cs_idx(i, j, k)];
#pragma unroll
    for (int d = 0; d < 6; d++) {
        int a = d >> 1, s = d & 1;
        bool edge = s ? (c[a] == 7) : (c[a] == 0);
        if (edge && g.bct[d] == 0) {
            int t1, t2;
            tangential(a, t1, t2);
            double gv = g.bcval ? g.bcval[(b * 6 + d) * 64 + c[t2] * 8 + c[t1]] : g.bcv[d];
            r -= 2.0 * gv / (h * h);
        }
    }
    X[t] = r;
    __syncthreads();
    // forward: contract each axis with V_a^T
    { double s = 0; for (int q = 0; q < 8; q++) s += V[0 * 64 + q * 8 + i] * X[(k * 8 + j) * 8 + q]; Y[t] = s; }
    __syncthreads();
    { double s = 0; for (int q = 0; q < 8; q++) s += V[1 * 64 + q * 8 + j] * Y[(k * 8 + q) * 8 + i]; X[t] = s; }
    __syncthreads();
    { double s = 0; for (int q = 0; q < 8; q++) s += V[2 * 64 + q * 8 + k] * X[(q * 8 + j) * 8 + i]; Y[t] = s; }
    __syncthreads();
    Y[t] = Y[t] * (h * h) / (L[i] + L[8 + j] + L[16 + k]);
    __syncthreads();
    // inverse: contract each axis with V_a
    { double s = 0; for (int q = 0; q < 8; q++) s += V[2 * 64 + k * 8 + q] * Y[(q * 8 + j) * 8 + i]; X[t] = s; }
    __syncthreads();
    { double s = 0; for (int q = 0; q < 8; q++) s += V[1 * 64 + j * 8 + q] * X[(k * 8 + q) * 8 + i]; Y[t] = s; }
    __syncthreads();
    { double s = 0; for (int q = 0; q < 8; q++) s += V[0 * 64 + i * 8 + q] * Y[(k * 8 + j) * 8 + q]; X[t] = s; }
    phi[b * 512 + cs_idx(i, j, k)] = (T)X[t];
}

// ------------------------------------------------- bottom of the V-cycle
// The two coarsest levels of every tree in one launch, one workgroup of 1024
// threads per tree: Gauss-Seidel on the tree's eight level-2 boxes,
// residual and restriction to the root, the root's FAS right-hand side, its
// exact solve, prolongation of the correction and the up-sweeps.  Level 2 of
// a tree is empty or all 8 children of the root (Morton = octant order from
// root2[tree]), i.e. one uniform 16^3 grid whose only ghosts are domain
// ghosts, so the ~20 dependent steps cost a workgroup barrier each instead of
// a launch each.  The arithmetic of every cell, and the order of every sum,
// are those of k_gsrb, k_resid_restrict, k_fas_rhs, k_coarse and k_prolong_cf.
// fmg != 0 first runs the FMG pass's own bottom (restriction, root solve,
// prolongation, without smoothing).
//
// One workgroup has one CU, so issuing instructions bounds it.  A thread owns
// the cells (I, J, K0 .. K0+3), two of each colour, with their values and
// right-hand sides in registers; the grid sits in LDS with a ghost layer,
// where each owner keeps its cells' domain ghosts up to date, so a cell's
// neighbours along x and y are at constant offsets, and along z three of four
// are the thread's own.  With both colours of the grid in LDS, ghosts formed
// by selects and all places computed anew, a V(2,2) bottom took 19.3 us (FP32
// 17.5); now 14.9 (12.7), of which 1.3 a sweep.
// Domain data of one axis of a cell: whether it lies at the axis' lower or
// upper face, and that face's ghost as sgn own + off (Dirichlet 2 g - own,
// Neumann own; 0 and 0 inside).  g is the face value at (u, v) of box b.
template <typename T> struct BotFace {
    int at;  // -1, +1 or 0: the side
    double g;
    T sgn, off;
};
template <typename T>
__device__ __forceinline__ BotFace<T> bot_face(const Geo &geo, int64_t b, int axis, bool lower, bool upper, int u,
                                               int v) {
    BotFace<T> f;
    // (values selected, not places: a selected place would put geo in scratch)
    const int c0 = geo.bct[2 * axis], c1 = geo.bct[2 * axis + 1];
    const double g0 = geo.bcv[2 * axis], g1 = geo.bcv[2 * axis + 1];
    const bool neumann = (upper ? c1 : c0) == 1;
    f.at = lower ? -1 : upper ? 1 : 0;
    f.g = upper ? g1 : g0;
    if (geo.bcval && f.at) f.g = geo.bcval[(b * 6 + 2 * axis + (upper ? 1 : 0)) * 64 + v * 8 + u];
    f.sgn = neumann ? (T)1 : (T)-1;
    f.off = neumann ? (T)0 : (T)2 * (T)f.g;
    if (neumann || !f.at) f.g = 0.0;
    return f;
}
// Place of cell (I, J, K), each -1..16, of the 16^3 grid with its ghost layer:
// rows of 18, planes padded to a multiple of 32 (the two planes that a wave
// of one colour reads then address the same LDS banks in turn)
constexpr int kBotRow = 18, kBotPlane = 352, kBotGrid = 18 * kBotPlane;
__device__ __forceinline__ int bot_at(int I, int J, int K) { return (K + 1) * kBotPlane + (J + 1) * kBotRow + I + 1; }
// colour-split index c of a box -> (i, j, k)
__device__ __forceinline__ void cs_cell(int c, int &i, int &j, int &k) {
    int q = c & 255;
    j = (q >> 2) & 7;
    k = q >> 5;
    i = 2 * (q & 3) + ((j + k + (c >> 8)) & 1);
}

template <typename T>
__global__ __launch_bounds__(1024) void k_bottom(Geo g, T *__restrict__ phi, T *__restrict__ rhs,
                                                 T *__restrict__ old, const double *__restrict__ eig,
                                                 int64_t r0, const int32_t *__restrict__ root2,
                                                 T h2_2, T inv_h2_2, T inv_h2_1, double h1, int nd,
                                                 int nu, int fmg, int fas2,
                                                 const int32_t *__restrict__ isleaf) {
    // F2: level-2 field with its ghost layer; F1, B1, O1: the root's phi, rhs,
    // old; W: the level-2 residual, then the root solve's X and Y, then the
    // root correction padded by its domain ghosts (10^3).
    __shared__ T F2[kBotGrid], F1[512], B1[512], O1[512];
    __shared__ double W[4096], V[192], L[24];
    T *R2 = reinterpret_cast<T *>(W);
    double *X = W, *Y = W + 512;
    T *D1 = reinterpret_cast<T *>(W + 1024);
    const int tid = threadIdx.x;
    const int64_t r = r0 + blockIdx.x;
    const int64_t first2 = root2[blockIdx.x];
    const bool has2 = first2 >= 0;
    // root cell of this thread (tid < 512), natural order
    const int ri = tid & 7, rj = (tid >> 3) & 7, rk = (tid >> 6) & 7;
    // this thread's run of cells (I, J, K0 + q), q = 0..3; its cells of colour
    // c are q = pc and pc + 2 with pc = (I + J + c) & 1, and f[c], b[c] hold
    // them.  at: place of q = 0.
    const int I = tid & 15, J = (tid >> 4) & 15, K0 = 4 * (tid >> 8), odd = (I + J) & 1;
    const int at = bot_at(I, J, K0);
    const int64_t box = first2 + ((I >> 3) | ((J >> 3) << 1) | ((K0 >> 3) << 2));
    T f[2][2], b[2][2];
    // offset in the level's fields of cell n of colour c
    auto cell = [&](int c, int n) __attribute__((always_inline)) {
        return box * 512 + c * 256 + (((K0 & 7) + (odd ^ c) + 2 * n) * 8 + (J & 7)) * 4 + ((I & 7) >> 1);
    };
    // the root cell's domain faces
    const BotFace<T> rx = bot_face<T>(g, r, 0, ri == 0, ri == 7, rj, rk), ry = bot_face<T>(g, r, 1, rj == 0, rj == 7, ri, rk),
                     rz = bot_face<T>(g, r, 2, rk == 0, rk == 7, ri, rj);
    const double tx = 2.0 * rx.g / (h1 * h1), ty = 2.0 * ry.g / (h1 * h1), tz = 2.0 * rz.g / (h1 * h1);
    // this thread's place in the padded root correction (tid < 1000): the
    // root cell it takes, 0 on edges and corners, and its sign in the domain
    // ghosts
    const int px = tid % 10 - 1, py = (tid / 10) % 10 - 1, pz = tid / 100 - 1;
    const int pout = (px < 0 || px > 7) + (py < 0 || py > 7) + (pz < 0 || pz > 7);
    const int pq = min(max(px, 0), 7) + 8 * min(max(py, 0), 7) + 64 * min(max(pz, 0), 7);
    const int c0 = g.bct[0], c1 = g.bct[1], c2 = g.bct[2], c3 = g.bct[3], c4 = g.bct[4], c5 = g.bct[5];
    const int pbc = px < 0 ? c0 : px > 7 ? c1 : py < 0 ? c2 : py > 7 ? c3 : pz < 0 ? c4 : pz > 7 ? c5 : 1;
    // the run's: along x and y per cell (they differ in g alone), along z of
    // the run's first or last cell
    T gx[2][2], gy[2][2];
    int dx = 0, dy = 0;
    T sx = (T)0, sy = (T)0;
    const BotFace<T> fz = bot_face<T>(g, has2 ? box : r, 2, K0 == 0, K0 == 12, I & 7, J & 7);
#pragma unroll
    for (int c = 0; c < 2; c++)
#pragma unroll
        for (int n = 0; n < 2; n++) {
            const int k = (K0 & 7) + (odd ^ c) + 2 * n;
            const BotFace<T> fx = bot_face<T>(g, has2 ? box : r, 0, I == 0, I == 15, J & 7, k);
            const BotFace<T> fy = bot_face<T>(g, has2 ? box : r, 1, J == 0, J == 15, I & 7, k);
            gx[c][n] = fx.off;
            gy[c][n] = fy.off;
            dx = fx.at;
            dy = fy.at * kBotRow;
            sx = fx.sgn;
            sy = fy.sgn;
        }
    if (tid < 192) V[tid] = eig[tid];
    if (tid < 24) L[tid] = eig[192 + tid];
    if (tid < 512) {
        int i, j, k;
        cs_cell(tid, i, j, k);
        F1[i + 8 * j + 64 * k] = phi[r * 512 + tid];
        B1[i + 8 * j + 64 * k] = rhs[r * 512 + tid];
    }
    // stores cell n of colour c and its domain ghosts
    auto put = [&](int c, int n) __attribute__((always_inline)) {
        const int q = (odd ^ c) + 2 * n, p = at + q * kBotPlane;
        const T v = f[c][n];
        F2[p] = v;
        if (dx) F2[p + dx] = sx * v + gx[c][n];
        if (dy) F2[p + dy] = sy * v + gy[c][n];
        if (K0 == 0 && q == 0) F2[p - kBotPlane] = fz.sgn * v + fz.off;
        if (K0 == 12 && q == 3) F2[p + kBotPlane] = fz.sgn * v + fz.off;
    };
    if (has2) {
        // in the order of the fields (read by runs, each load would touch four
        // times the cache lines), then handed to the owners through LDS
#pragma unroll
        for (int w = 0; w < 4; w++) {
            int e = tid + 1024 * w, o = e >> 9, i, j, k;
            cs_cell(e & 511, i, j, k);
            i += 8 * (o & 1);
            j += 8 * ((o >> 1) & 1);
            k += 8 * (o >> 2);
            F2[bot_at(i, j, k)] = phi[first2 * 512 + e];
            R2[k * 256 + j * 16 + i] = rhs[first2 * 512 + e];
        }
    }
    __syncthreads();
    if (has2) {
#pragma unroll
        for (int c = 0; c < 2; c++)
#pragma unroll
            for (int n = 0; n < 2; n++) {
                const int q = (odd ^ c) + 2 * n;
                f[c][n] = F2[at + q * kBotPlane];
                b[c][n] = R2[(K0 + q) * 256 + J * 16 + I];
                put(c, n);
            }
    }
    __syncthreads();
    // six-neighbour sums of the run's two cells of colour c, order -x, +x, -y,
    // +y, -z, +z
    auto sums = [&](int c, T s[2]) __attribute__((always_inline)) {
        const int pc = odd ^ c;
        const T *p = F2 + at + pc * kBotPlane;
        const T e = F2[at + (pc ? 4 : -1) * kBotPlane];  // the cell beyond the run, or its ghost
        const T o0 = f[1 - c][0], o1 = f[1 - c][1];
        const T zm0 = pc ? o0 : e, zp0 = pc ? o1 : o0, zm1 = pc ? o1 : o0, zp1 = pc ? e : o1;
        s[0] = p[-1] + p[1] + p[-kBotRow] + p[kBotRow] + zm0 + zp0;
        p += 2 * kBotPlane;
        s[1] = p[-1] + p[1] + p[-kBotRow] + p[kBotRow] + zm1 + zp1;
    };
    // FAS right-hand side of the level-2 boxes with children, L phi + rhs
    // (the level-3 restriction has just written both), as k_fas_rhs forms
    // it: same neighbour order, same domain ghosts; stored for the rest of
    // the cycle
    if (fas2 && has2 && !isleaf[box]) {
#pragma unroll
        for (int c = 0; c < 2; c++) {
            T s[2];
            sums(c, s);
#pragma unroll
            for (int n = 0; n < 2; n++) {
                b[c][n] = (s[n] - (T)6 * f[c][n]) * inv_h2_2 + b[c][n];
                rhs[cell(c, n)] = b[c][n];
            }
        }
    }
    __syncthreads();  // the sums above read cells that the first half-sweep writes

    auto smooth = [&](int n) __attribute__((always_inline)) {
        for (int it = 0; it < n; it++)
#pragma unroll
            for (int c = 0; c < 2; c++) {
                T s[2];
                sums(c, s);
#pragma unroll
                for (int m = 0; m < 2; m++) {
                    // (written as the fused multiply-add that the other kernels'
                    // s - h2 b becomes: h2 b is constant here, and taken out
                    // of the loop it would round on its own)
                    f[c][m] = fmadd(-h2_2, b[c][m], s[m]) * (T)kSixth;
                    put(c, m);
                }
                __syncthreads();
            }
    };
    // residual of level 2, restriction to the root, FAS right-hand side of
    // the root; a leaf root only copies phi -> old
    auto down = [&]() __attribute__((always_inline)) {
        if (!has2) {
            if (tid < 512) O1[tid] = F1[tid];
            __syncthreads();
            return;
        }
#pragma unroll
        for (int c = 0; c < 2; c++) {
            T s[2];
            sums(c, s);
#pragma unroll
            for (int n = 0; n < 2; n++)
                R2[(K0 + (odd ^ c) + 2 * n) * 256 + J * 16 + I] = resid_of<T>(b[c][n], s[n], f[c][n], inv_h2_2);
        }
        __syncthreads();
        if (tid < 512) {
            T sphi = 0, sres = 0;
            const T *pf = F2 + bot_at(2 * ri, 2 * rj, 2 * rk), *pr = R2 + 512 * rk + 32 * rj + 2 * ri;
#pragma unroll
            for (int dk = 0; dk < 2; dk++)
#pragma unroll
                for (int dj = 0; dj < 2; dj++)
#pragma unroll
                    for (int di = 0; di < 2; di++) {
                        sphi += pf[dk * kBotPlane + dj * kBotRow + di];
                        sres += pr[dk * 256 + dj * 16 + di];
                    }
            T mphi = (T)0.125 * sphi;
            F1[tid] = mphi;
            O1[tid] = mphi;
            B1[tid] = (T)0.125 * sres;
        }
        __syncthreads();
        if (tid < 512) {
            T own = F1[tid];
            const T hx = rx.sgn * own + rx.off, hy = ry.sgn * own + ry.off, hz = rz.sgn * own + rz.off;
            T xm = rx.at < 0 ? hx : F1[tid - 1], xp = rx.at > 0 ? hx : F1[tid + 1];
            T ym = ry.at < 0 ? hy : F1[tid - 8], yp = ry.at > 0 ? hy : F1[tid + 8];
            T zm = rz.at < 0 ? hz : F1[tid - 64], zp = rz.at > 0 ? hz : F1[tid + 64];
            T s = xm + xp + ym + yp + zm + zp;
            B1[tid] = (s - (T)6 * own) * inv_h2_1 + B1[tid];
        }
        __syncthreads();
    };
    // exact root solve, as k_coarse (threads < 512, root cell tid)
    auto coarse = [&]() __attribute__((always_inline)) {
        const int t = tid & 511, i = ri, j = rj, k = rk;
        if (tid < 512) {
            double rr = (double)B1[t];
            rr -= tx;
            rr -= ty;
            rr -= tz;
            X[t] = rr;
        }
        __syncthreads();
        if (tid < 512) { double s = 0; for (int q = 0; q < 8; q++) s += V[0 * 64 + q * 8 + i] * X[(k * 8 + j) * 8 + q]; Y[t] = s; }
        __syncthreads();
        if (tid < 512) { double s = 0; for (int q = 0; q < 8; q++) s += V[1 * 64 + q * 8 + j] * Y[(k * 8 + q) * 8 + i]; X[t] = s; }
        __syncthreads();
        if (tid < 512) {
            double s = 0;
            for (int q = 0; q < 8; q++) s += V[2 * 64 + q * 8 + k] * X[(q * 8 + j) * 8 + i];
            Y[t] = s * (h1 * h1) / (L[i] + L[8 + j] + L[16 + k]);
        }
        __syncthreads();
        if (tid < 512) { double s = 0; for (int q = 0; q < 8; q++) s += V[2 * 64 + k * 8 + q] * Y[(q * 8 + j) * 8 + i]; X[t] = s; }
        __syncthreads();
        if (tid < 512) { double s = 0; for (int q = 0; q < 8; q++) s += V[1 * 64 + j * 8 + q] * X[(k * 8 + q) * 8 + i]; Y[t] = s; }
        __syncthreads();
        if (tid < 512) {
            double s = 0;
            for (int q = 0; q < 8; q++) s += V[0 * 64 + i * 8 + q] * Y[(k * 8 + j) * 8 + q];
            F1[t] = (T)s;
        }
        __syncthreads();
    };
    // prolongation: the root correction delta = phi - old padded by its
    // homogeneous domain ghosts (faces only) into D1[10^3], then
    // phi_f += 1/4 d0 + 1/4 (dx + dy + dz) on every level-2 cell
    auto prolong = [&]() __attribute__((always_inline)) {
        if (!has2) return;
        if (tid < 1000) {
            T din = F1[pq] - O1[pq];
            D1[tid] = pout > 1 ? (T)0 : pbc == 1 ? din : -din;
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < 2; c++)
#pragma unroll
            for (int n = 0; n < 2; n++) {
                const int K = K0 + (odd ^ c) + 2 * n;
                const T *d = D1 + ((K >> 1) + 1) * 100 + ((J >> 1) + 1) * 10 + (I >> 1) + 1;
                T d0 = d[0], dx1 = d[(I & 1) ? 1 : -1], dy1 = d[(J & 1) ? 10 : -10], dz1 = d[(K & 1) ? 100 : -100];
                f[c][n] += (T)0.25 * d0 + (T)0.25 * (dx1 + dy1 + dz1);
                put(c, n);
            }
        __syncthreads();
    };

    if (fmg) {
        down();
        coarse();
        prolong();
    }
    if (has2) smooth(nd);
    down();
    coarse();
    prolong();
    if (has2) smooth(nu);

    if (tid < 512) {
        int i, j, k;
        cs_cell(tid, i, j, k);
        int n = i + 8 * j + 64 * k;
        phi[r * 512 + tid] = F1[n];
        rhs[r * 512 + tid] = B1[n];
        old[r * 512 + tid] = O1[n];
    }
    if (has2) {
#pragma unroll
        for (int w = 0; w < 4; w++) {
            int e = tid + 1024 * w, o = e >> 9, i, j, k;
            cs_cell(e & 511, i, j, k);
            phi[first2 * 512 + e] = F2[bot_at(8 * (o & 1) + i, 8 * ((o >> 1) & 1) + j, 8 * (o >> 2) + k)];
        }
    }
}

// Covered cells of level l-1 <- mean of their 8 children on level l.
template <typename T>
__global__ __launch_bounds__(64) void k_restrict_phi(Geo g, T *__restrict__ phi, int64_t b0,
                                                     int64_t nbx) {
    int64_t lb = xcd_map(blockIdx.x, nbx);
    if (lb >= nbx) return;
    int64_t b = b0 + lb;
    int t = threadIdx.x, pi = t & 3, pj = (t >> 2) & 3, pk = t >> 4;
    T s = 0;
#pragma unroll
    for (int dk = 0; dk < 2; dk++)
#pragma unroll
        for (int dj = 0; dj < 2; dj++)
#pragma unroll
            for (int di = 0; di < 2; di++) s += phi[b * 512 + cs_idx(2 * pi + di, 2 * pj + dj, 2 * pk + dk)];
    int64_t p = g.parent[b];
    int ci = 4 * (g.ijk[b * 4] & 1) + pi, cj = 4 * (g.ijk[b * 4 + 1] & 1) + pj,
        ck = 4 * (g.ijk[b * 4 + 2] & 1) + pk;
    phi[p * 512 + cs_idx(ci, cj, ck)] = (T)0.125 * s;
}

// The parent cells of every leaf box of level >= 2 <- the mean of the box's
// 8 cells under each (the arithmetic of k_restrict_phi), all levels in one
// launch.  Under 2:1 nesting every covered cell that a residual or a c_hat
// reads has only leaf children, so this is the restriction a stopping test
// needs; covered cells whose children have children are left as they are.
template <typename T>
__global__ __launch_bounds__(64) void k_restrict_leaves(Geo g, T *__restrict__ phi,
                                                        const int32_t *__restrict__ leaf, int64_t nleaf) {
    int64_t q = xcd_map(blockIdx.x, nleaf);
    if (q >= nleaf) return;
    int64_t b = leaf[q];
    if (g.ijk[b * 4 + 3] < 2) return;
    int t = threadIdx.x, pi = t & 3, pj = (t >> 2) & 3, pk = t >> 4;
    T s = 0;
#pragma unroll
    for (int dk = 0; dk < 2; dk++)
#pragma unroll
        for (int dj = 0; dj < 2; dj++)
#pragma unroll
            for (int di = 0; di < 2; di++) s += phi[b * 512 + cs_idx(2 * pi + di, 2 * pj + dj, 2 * pk + dk)];
    int64_t p = g.parent[b];
    int ci = 4 * (g.ijk[b * 4] & 1) + pi, cj = 4 * (g.ijk[b * 4 + 1] & 1) + pj,
        ck = 4 * (g.ijk[b * 4 + 2] & 1) + pk;
    phi[p * 512 + cs_idx(ci, cj, ck)] = (T)0.125 * s;
}


// Leaf residual norms: per listed box, sum of r^2 h^3 and max |r|.  When
// r_out is set the residual is also stored, rounded to FP32 (right-hand side
// of the mixed-precision correction solve).
__global__ __launch_bounds__(256) void k_leaf_norms(Geo g, const double *__restrict__ phi,
                                                    const double *__restrict__ rhs,
                                                    const double *__restrict__ chat,
                                                    const int32_t *__restrict__ leaf, int64_t nleaf,
                                                    double *__restrict__ partial,
                                                    float *__restrict__ r_out) {
    __shared__ double P[512], H[384], S[4], M[4];
    int64_t q = xcd_map(blockIdx.x, nleaf);
    if (q >= nleaf) return;
    int64_t b = leaf[q];
    int t = threadIdx.x;
    double r0 = rhs[b * 512 + t], r1 = rhs[b * 512 + 256 + t];
    int l = g.ijk[b * 4 + 3];
    stage_full<double>(g, phi, chat, b, P, H);
    __syncthreads();
    double h = g.len / (8.0 * (double)(1 << (l - 1)));
    double inv_h2 = 1.0 / (h * h), vol = h * h * h;
    int m = t & 3, j = (t >> 2) & 7, k = t >> 5;
    double ss = 0.0, mx = 0.0;
#pragma unroll
    for (int c = 0; c < 2; c++) {
        int i = 2 * m + ((j + k + c) & 1);
        double own = P[c * 256 + t];
        double s = sum_full<double>(P, H, i, j, k);
        double r = resid_of<double>(c ? r1 : r0, s, own, inv_h2);
        if (r_out) r_out[b * 512 + c * 256 + t] = (float)r;
        ss = fmadd(r, r, ss);
        mx = nanmax(fabs(r), mx);
    }
    for (int off = 32; off > 0; off >>= 1) {
        ss += __shfl_xor(ss, off);
        mx = nanmax(__shfl_xor(mx, off), mx);
    }
    if ((t & 63) == 0) {
        S[t >> 6] = ss;
        M[t >> 6] = mx;
    }
    __syncthreads();
    if (t == 0) {
        partial[2 * q] = ((S[0] + S[1]) + (S[2] + S[3])) * vol;
        partial[2 * q + 1] = nanmax(nanmax(M[0], M[1]), nanmax(M[2], M[3]));
    }
}

// The norms of k_leaf_norms on the leaf boxes leaf[q0 .. q0+nq), into
// partial at their leaf positions q.  Each XCD takes a contiguous share of
// the leaf list (XCD-aware mapping of q): over the box range instead, the
// refined boxes, which exit at once, crowd the first shares (on the
// two-streamer tree the busiest XCD had 14% more leaf boxes than the mean).
// With h = len 2^-(l+2), 1/h^2 and h^3 are the power-of-two
// scalings ilen2 2^(2(l+2)) and len3 2^(-3(l+2)) of ilen2 = 1/len^2 and
// len3 = len^3 (the same bits as dividing, in the normal range), so the
// kernel holds no divide.  OUT: the FP32 residual is also stored.
template <bool OUT>
__global__ __launch_bounds__(128) void k_box_norms(Geo g, const double *__restrict__ phi,
                                                   const double *__restrict__ rhs,
                                                   const double *__restrict__ chat,
                                                   const int32_t *__restrict__ leaf, int64_t q0, int64_t nq,
                                                   double *__restrict__ partial, float *__restrict__ r_out,
                                                   double ilen2, double len3) {
    __shared__ __attribute__((aligned(16))) double G[kFullG], X[kFullX];
    __shared__ double S[4], M[4];
    int64_t lq = xcd_map(blockIdx.x, nq);
    if (lq >= nq) return;
    const int64_t q = q0 + lq;
    const int64_t b = leaf[q];
    const int u = threadIdx.x;
    const double2 r0 = ld_stream(reinterpret_cast<const double2 *>(rhs + b * 512) + u);
    const double2 r1 = ld_stream(reinterpret_cast<const double2 *>(rhs + b * 512 + 256) + u);
    const int l = g.ijk[b * 4 + 3];
    double own[4], r[4], f[4];
    full_stage<double, false>(g, phi, chat, b, G, X, own);
    const bool odd = ((u >> 1) + (u >> 4)) & 1;
    to_cells<double, double2>(r0, r1, odd, f);
    full_sums<double>(G, X, own, r);
    const double inv_h2 = ldexp(ilen2, 2 * (l + 2)), vol = ldexp(len3, -3 * (l + 2));
#pragma unroll
    for (int e = 0; e < 4; e++) r[e] = resid_of<double>(f[e], r[e], own[e], inv_h2);
    if (OUT) {
        reinterpret_cast<float2 *>(r_out + b * 512)[u] = make_float2((float)(odd ? r[1] : r[0]), (float)(odd ? r[3] : r[2]));
        reinterpret_cast<float2 *>(r_out + b * 512 + 256)[u] = make_float2((float)(odd ? r[0] : r[1]), (float)(odd ? r[2] : r[3]));
    }
    full_norms(r, odd, S, M);
    __syncthreads();
    if (u == 0) {
        partial[2 * q] = ((S[0] + S[1]) + (S[2] + S[3])) * vol;
        partial[2 * q + 1] = nanmax(nanmax(M[0], M[1]), nanmax(M[2], M[3]));
    }
}

// out[q][e] = (L x)(cell e of leaf box leaf[q]) for the composite operator
// with the field's ghosts (same layout as the field, one 512-run per leaf
// position); the operator application of the per-level learned step.
template <typename T>
__global__ __launch_bounds__(256) void k_leaf_apply(Geo g, const T *__restrict__ x,
                                                    const T *__restrict__ chat,
                                                    const int32_t *__restrict__ leaf, int64_t nleaf,
                                                    T *__restrict__ out) {
    __shared__ T P[512], H[384];
    int64_t q = xcd_map(blockIdx.x, nleaf);
    if (q >= nleaf) return;
    int64_t b = leaf[q];
    int t = threadIdx.x;
    int l = g.ijk[b * 4 + 3];
    stage_full<T>(g, x, chat, b, P, H);
    __syncthreads();
    double h = g.len / (8.0 * (double)(1 << (l - 1)));
    T inv_h2 = (T)(1.0 / (h * h));
    int m = t & 3, j = (t >> 2) & 7, k = t >> 5;
#pragma unroll
    for (int c = 0; c < 2; c++) {
        int i = 2 * m + ((j + k + c) & 1);
        T own = P[c * 256 + t];
        out[q * 512 + c * 256 + t] = (sum_full<T>(P, H, i, j, k) - (T)6 * own) * inv_h2;
    }
}

// The sums of the learned step's least squares.  x holds the correction c of
// every leaf box (and its means on the covered cells that a leaf box reads),
// and q_m = A0 c_m is the operator on the corrections of level m alone.  A
// leaf cell of level j sees three of them: q_j through the box's own cells and
// those of its level, q_{j-1} through the leaf cells behind a
// refinement-boundary face, and q_{j+1} through the covered cells of refined
// neighbours.  So the three stencil sums of a box come from one set of
// ghosts, each filed under the level it belongs to (a refinement-boundary
// ghost under two: next to a box with children, the coarse values it is
// interpolated from are means of level j), and nothing is stored but the nine
// products <r, q>, <q, q'>.  (As three passes, one per level modulo 3, each
// with its restrictions and c_hat and writing its q, and a pass of dot
// products, the sums took 339 us on 16164 leaf boxes;
// this kernel takes 72, and 108 with two boxes a workgroup.)
//
// A workgroup sums over one chunk, at most `per` leaf positions of one (level,
// tree), into column blockIdx.x of part[9][nchunk].
__device__ __forceinline__ int learned_range(const LearnedRanges &R, const int32_t *__restrict__ tab, int c,
                                             int64_t &beg, int64_t &end) {
    int w = 0;
    if (!tab) {
        while (c >= R.chunk[w + 1]) w++;
        beg = R.leaf[w] + (int64_t)(c - R.chunk[w]) * R.per;
        end = min(beg + R.per, R.leaf[w + 1]);
    } else {
        const int32_t *ch = tab + R.nrange + 1;
        for (int lo = R.nrange; lo - w > 1;) {
            const int m = (w + lo) >> 1;
            if (c >= ch[m])
                w = m;
            else
                lo = m;
        }
        beg = tab[w] + (int64_t)(c - ch[w]) * R.per;
        end = min(beg + R.per, (int64_t)tab[w + 1]);
    }
    return w;
}
__global__ __launch_bounds__(512) void k_learned_sums(Geo g, const float *__restrict__ x,
                                                      const float *__restrict__ r32,
                                                      const int32_t *__restrict__ leaf,
                                                      const int32_t *__restrict__ tab, LearnedRanges R,
                                                      double *__restrict__ part) {
    __shared__ float P[512], H[384], X[384];
    __shared__ double S[8][9];
    const int t = threadIdx.x;
    int64_t q0, q1;
    const int l = learned_range(R, tab, blockIdx.x, q0, q1) / R.ntree + 1;
    const double h = g.len / (8.0 * (double)(1 << (l - 1)));
    const float inv_h2 = (float)(1.0 / (h * h));
    // the thread's cell and (below 384) its ghost of face d = wave, at (u, v)
    const int o = t >> 8, j = (t >> 2) & 7, k = (t >> 5) & 7, i = 2 * (t & 3) + ((j + k + o) & 1);
    const int d = __builtin_amdgcn_readfirstlane(t >> 6), u = t & 7, v = (t >> 3) & 7;
    const int a = d >> 1, side = d & 1;
    double s[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    for (int64_t q = q0; q < q1; q++) {
        const int64_t b = leaf[q];
        const FaceTab ft = face_tab(g, b);
        bool other = false;  // a face of another level (block-uniform)
#pragma unroll
        for (int f = 0; f < 6; f++) other = other || ft.nb[f] == -1 || ft.slot[f] == -2;
        const float own = x[b * 512 + t];
        const double r = r32[b * 512 + t];
        float hv = 0.0f, xv = 0.0f;
        if (d < 6) {
            const int nb = pick6(ft.nb, d), slot = pick6(ft.slot, d);
            if (nb == -1) {
                int t1, t2, c[3];
                tangential(a, t1, t2);
                c[t1] = u;
                c[t2] = v;
                c[a] = side ? 7 : 0;
                const float edge = x[b * 512 + cs_idx3(c)];
                c[a] = side ? 6 : 1;
                const float in = x[b * 512 + cs_idx3(c)];
                // c_hat as in cf_face, the covered cells apart
                const int32_t *y = g.slotx + 8 * (int64_t)slot;
                const int64_t Q = y[0];
                c[a] = side ? 0 : 7;
                c[t1] = y[1] + (u >> 1);
                c[t2] = y[2] + (v >> 1);
                float lf = 0.875f * x[Q * 512 + cs_idx3(c)], cov = 0.0f;
#pragma unroll
                for (int z = 0; z < 4; z++) {
                    const int ax = z < 2 ? t1 : t2, up = z & 1, N = y[3 + z];
                    const float st = ((z < 2 ? u : v) & 1) == up ? 1.0f / 32.0f + 0.125f : 1.0f / 32.0f - 0.125f;
                    const float val = st * coarse_at<float>(g, x, Q, c, ax, up ? 1 : -1, N);
                    if (c[ax] == (up ? 7 : 0) && N >= 0 && g.cfslot[Q * 6 + 2 * ax + up] == -2)
                        cov += val;
                    else
                        lf += val;
                }
                hv = cf_ghost<float>(cov, edge, in);
                xv = cf_ghost<float>(lf, 0.0f, 0.0f);
            } else {
                const float gv = ghost_at<float>(g, x, nullptr, b, d, nb, slot, u, v);
                hv = slot == -2 ? 0.0f : gv;
                xv = slot == -2 ? gv : 0.0f;
            }
        }
        __syncthreads();  // the previous box is done with the buffers
        P[t] = own;
        if (d < 6) {
            H[t] = hv;
            X[t] = xv;
        }
        __syncthreads();
        const double qc = (sum_full<float>(P, H, i, j, k) - 6.0f * own) * inv_h2;
        s[1] += r * qc;
        s[6] += qc * qc;
        if (!other) continue;
        // the faces of the coarser (A) and of the finer level (N)
        float A = 0.0f, N = 0.0f;
        auto face = [&](int f, bool at, int uv) __attribute__((always_inline)) {
            const float w = at ? X[64 * f + uv] : 0.0f;
            if (ft.nb[f] == -1)
                A += w;
            else
                N += w;
        };
        face(0, i == 0, k * 8 + j);
        face(1, i == 7, k * 8 + j);
        face(2, j == 0, k * 8 + i);
        face(3, j == 7, k * 8 + i);
        face(4, k == 0, j * 8 + i);
        face(5, k == 7, j * 8 + i);
        const double qa = A * inv_h2, qn = N * inv_h2;
        s[0] += r * qa;
        s[2] += r * qn;
        s[3] += qa * qa;
        s[4] += qa * qc;
        s[5] += qa * qn;
        s[7] += qc * qn;
        s[8] += qn * qn;
    }
    const double vol = h * h * h;
    // eight of the sums folded into one a lane (three exchanges halve the
    // sums a lane holds), then over the lanes; the ninth on its own
#pragma unroll
    for (int m = 4; m > 0; m >>= 1) {
        const bool hi = t & m;
#pragma unroll
        for (int e = 0; e < m; e++) {
            const double give = hi ? s[e] : s[e + m];
            s[e] = (hi ? s[e + m] : s[e]) + __shfl_xor(give, m);
        }
    }
#pragma unroll
    for (int m = 8; m < 64; m *= 2) s[0] += __shfl_xor(s[0], m);
#pragma unroll
    for (int m = 1; m < 64; m *= 2) s[8] += __shfl_xor(s[8], m);
    if ((t & 63) < 9) S[t >> 6][t & 63] = (t & 63) < 8 ? s[0] : s[8];
    __syncthreads();
    if (t < 9) {
        double w = 0.0;
#pragma unroll
        for (int m = 0; m < 8; m++) w += S[m][t];
        part[(int64_t)t * gridDim.x + blockIdx.x] = w * vol;
    }
}
// sums[range][9] (pinned host memory) <- the sums over the chunks of a range,
// one workgroup each.
__global__ __launch_bounds__(256) void k_learned_reduce(const double *__restrict__ part,
                                                        const int32_t *__restrict__ tab, LearnedRanges R, int nchunk,
                                                        double *__restrict__ sums) {
    __shared__ double S[4];
    const int w = blockIdx.x / 9, e = blockIdx.x % 9, t = threadIdx.x;
    const int c0 = tab ? tab[R.nrange + 1 + w] : R.chunk[w], c1 = tab ? tab[R.nrange + 2 + w] : R.chunk[w + 1];
    const double *__restrict__ p = part + (int64_t)e * nchunk;
    double v = 0.0;
    for (int c = c0 + t; c < c1; c += 2048) {
        double z[8];
#pragma unroll
        for (int k = 0; k < 8; k++) z[k] = c + 256 * k < c1 ? p[c + 256 * k] : 0.0;
#pragma unroll
        for (int k = 0; k < 8; k++) v += z[k];
    }
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if ((t & 63) == 0) S[t >> 6] = v;
    __syncthreads();
    if (t == 0) sums[blockIdx.x] = (S[0] + S[1]) + (S[2] + S[3]);
}

// Electric field of phi (section 2.3, E = -grad phi), one box per block:
// face components by central differences, (phi(f-1) - phi(f)) / h across face
// f = 0..8 of each axis (faces 0 and 8 with the box's ghosts), into
// e_face[((b*3 + a)*9 + f)*64 + v*8 + u]; and the strength at the cell
// centres, sqrt(Ex^2 + Ey^2 + Ez^2) with each component the mean of the
// cell's two faces, into e_norm[b*512 + natural index].  Either output may
// be null.  The 1728 face values are formed once (times 1/h) in LDS.
__global__ __launch_bounds__(256) void k_efield(Geo g, const double *__restrict__ phi,
                                                const double *__restrict__ chat, int64_t n,
                                                double *__restrict__ e_face, double *__restrict__ e_norm) {
    __shared__ double P[512], H[384], EF[1728];
    int64_t b = xcd_map(blockIdx.x, n);
    if (b >= n) return;
    int t = threadIdx.x;
    int l = g.ijk[b * 4 + 3];
    stage_full<double>(g, phi, chat, b, P, H);
    __syncthreads();
    const double inv_h = (8.0 * (double)(1 << (l - 1))) / g.len;
    // value of cell c along axis a (c = -1 or 8: the ghost on that face) at
    // tangential (u, v)
    auto val = [&](int a, int c, int u, int v) __attribute__((always_inline)) -> double {
        if (c < 0) return H[(2 * a) * 64 + v * 8 + u];
        if (c > 7) return H[(2 * a + 1) * 64 + v * 8 + u];
        int i = a == 0 ? c : u, j = a == 0 ? u : a == 1 ? c : v, k = a == 2 ? c : v;
        return P[cs_idx(i, j, k)];
    };
    for (int e = t; e < 3 * 9 * 64; e += 256) {
        int a = e / 576, r = e - 576 * a, f = r >> 6, v = (r >> 3) & 7, u = r & 7;
        double ef = (val(a, f - 1, u, v) - val(a, f, u, v)) * inv_h;
        EF[e] = ef;
        if (e_face) e_face[b * 1728 + e] = ef;
    }
    if (!e_norm) return;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < 2; w++) {
        int c = t + 256 * w, i = c & 7, j = (c >> 3) & 7, k = c >> 6;
        double ex = (EF[0 * 576 + i * 64 + k * 8 + j] + EF[0 * 576 + (i + 1) * 64 + k * 8 + j]) / 2.0;
        double ey = (EF[1 * 576 + j * 64 + k * 8 + i] + EF[1 * 576 + (j + 1) * 64 + k * 8 + i]) / 2.0;
        double ez = (EF[2 * 576 + k * 64 + j * 8 + i] + EF[2 * 576 + (k + 1) * 64 + j * 8 + i]) / 2.0;
        e_norm[b * 512 + c] = sqrt(ex * ex + ey * ey + ez * ez);
    }
}

// Faces of the face neighbours, formed from the uploaded face tables: for
// box b, face d with a same-level neighbour N, and the 4 faces of N across
// the two axes tangential to d (-t1, +t1, -t2, +t2), the pair (nbr[N][d'],
// cfslot[N][d']) (the fused Gauss-Seidel sweep recomputes N's face layer
// and needs N's ghosts); all -2 where face d has no same-level neighbour.
// One thread per (box, face).
__global__ __launch_bounds__(256) void k_face_xt(const int32_t *__restrict__ nbr, const int32_t *__restrict__ cfslot,
                                                 int64_t n, int32_t *__restrict__ xt) {
    int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= 6 * n) return;
    const int d = (int)(e % 6);
    const int32_t N = nbr[e];
    int32_t *out = xt + e * 8;
    if (N < 0) {
#pragma unroll
        for (int q = 0; q < 8; q++) out[q] = -2;
        return;
    }
    const int a = d >> 1, t1 = a == 0 ? 1 : 0, t2 = a == 2 ? 1 : 2;
    const int tf[4] = {2 * t1, 2 * t1 + 1, 2 * t2, 2 * t2 + 1};
#pragma unroll
    for (int q = 0; q < 4; q++) {
        out[2 * q] = nbr[6 * (int64_t)N + tf[q]];
        out[2 * q + 1] = cfslot[6 * (int64_t)N + tf[q]];
    }
}

// Refinement scores (section 2.5, the space-charge criterion |b| h^2 > c3):
// for box b, scores[b*27 + r] = the largest |b| h^2 over its cells in region
// r = (sx+1) + 3 (sy+1) + 9 (sz+1), where along each axis s = -1 takes cells
// 0..2, s = +1 cells 5..7 and s = 0 all cells (so r = 13 is the whole box
// and the 26 others the cells within 3 of each face, edge and corner).
//
// A region is a product of ranges, so the maxima are taken axis by axis: one
// wavefront per box, lane = x-row (its 8 cells are 4 consecutive values of
// each colour), then along y and z through LDS: 192, 72 and 27 maxima of at
// most 8 values instead of 27 of 512.  Bound by reading b (4 KB a box); the
// direct form, 27 running maxima a thread and 162 FP64 shuffles a wave, took
// 139 us on 9001 boxes, this one 10.8 (3.6 TB/s).  The maximum (fmax: a NaN cell is skipped) does not
// depend on the order.
__global__ __launch_bounds__(256) void k_refine_scores(Geo g, const double *__restrict__ rhs, int64_t n,
                                                       double *__restrict__ scores) {
    __shared__ double X[4][3 * 64], Y[4][9 * 8];
    const int w = threadIdx.x >> 6, t = threadIdx.x & 63;
    const int64_t nblk = (n + 3) >> 2, blk = xcd_map(blockIdx.x, nblk);
    if (blk >= nblk) return;
    const int64_t b = 4 * blk + w;
    const bool on = b < n;  // wave-uniform
    if (on) {
        const double h = g.len / (8.0 * (double)(1 << (g.ijk[b * 4 + 3] - 1))), h2 = h * h;
        const double4 c0 = ld_stream(reinterpret_cast<const double4 *>(rhs + b * 512) + t);
        const double4 c1 = ld_stream(reinterpret_cast<const double4 *>(rhs + b * 512 + 256) + t);
        const bool odd = ((t & 7) + (t >> 3)) & 1;  // the row's first cell is of colour 1
        auto v = [h2](double x) __attribute__((always_inline)) { return fabs(x) * h2; };
        const double e0 = v(odd ? c1.x : c0.x), o0 = v(odd ? c0.x : c1.x), e1 = v(odd ? c1.y : c0.y);
        const double o1 = v(odd ? c0.y : c1.y), e2 = v(odd ? c1.z : c0.z), o2 = v(odd ? c0.z : c1.z);
        const double e3 = v(odd ? c1.w : c0.w), o3 = v(odd ? c0.w : c1.w);
        const double lo = fmax(fmax(fmax(0.0, e0), o0), e1), hi = fmax(fmax(fmax(0.0, o2), e3), o3);
        X[w][t] = lo;
        X[w][64 + t] = fmax(fmax(lo, hi), fmax(o1, e2));
        X[w][128 + t] = hi;
    }
    __syncthreads();
    if (on)
        for (int e = t; e < 72; e += 64) {  // e = region of (x, y) * 8 + k
            const int k = e & 7, sx = (e >> 3) % 3, sy = (e >> 3) / 3;
            const double *r = X[w] + 64 * sx + 8 * k;
            double m = 0.0;
            for (int j = sy == 2 ? 5 : 0; j < (sy == 0 ? 3 : 8); j++) m = fmax(m, r[j]);
            Y[w][e] = m;
        }
    __syncthreads();
    if (on && t < 27) {
        const int sz = t / 9;
        const double *r = Y[w] + 8 * (t % 9);
        double m = 0.0;
        for (int k = sz == 2 ? 5 : 0; k < (sz == 0 ? 3 : 8); k++) m = fmax(m, r[k]);
        scores[b * 27 + t] = m;
    }
}

// The refinement criterion with its 3-cell buffer (section 2.5) reduced to
// one value per box: for a leaf box b, near[b] = the largest score over b's
// cells and the cells of its same-level leaf neighbours within 3 cells of
// it (region 26 - o of neighbour b + o; a missing or refined neighbour
// contributes b's own whole-box score r = 13); 0 for a refined box.  The
// maximum is taken as (m < x) ? x : m in the order o = 0..26 from m = the
// box's own score, the host planner's arithmetic, so the two give the same
// bits: the pairwise maximum below keeps the first of equal values, and a
// NaN x, which never replaces m, enters as m.
//
// 32 lanes a box, one neighbour each: three dependent loads instead of 27 x 3
// in turn (9001 boxes: 3.9 us; one thread a box: 18 us, the latency of 36
// blocks).
__global__ __launch_bounds__(256) void k_refine_near(const int32_t *__restrict__ n27,
                                                     const int32_t *__restrict__ isleaf,
                                                     const double *__restrict__ sc, int64_t n,
                                                     double *__restrict__ near) {
    const int64_t b = 8 * (int64_t)blockIdx.x + (threadIdx.x >> 5);
    const int o = threadIdx.x & 31;
    if (b >= n) return;  // whole groups of 32 lanes
    const bool leaf = isleaf[b] != 0;
    const double own = sc[27 * b + 13];
    double m = own;
    if (leaf && o < 27) {
        const int32_t N = n27[27 * b + o];
        if (N >= 0 && isleaf[N]) m = sc[27 * (int64_t)N + (26 - o)];
        if (m != m) m = own;
    }
    for (int off = 1; off < 32; off <<= 1) {
        const double p = __shfl_xor(m, off);
        const double first = (o & off) ? p : m, second = (o & off) ? m : p;
        m = (first < second) ? second : first;
    }
    if (o == 0) near[b] = !leaf ? 0.0 : (own < m) ? m : own;
}

// Transfer of phi to a new tree.  Copy: new box b takes the old box src[b]
// (same level and position) when src[b] >= 0.
__global__ __launch_bounds__(256) void k_transfer_copy(const double *__restrict__ from, double *__restrict__ to,
                                                       const int32_t *__restrict__ src, int64_t n) {
    int64_t b = xcd_map(blockIdx.x, n);
    if (b >= n) return;
    int64_t o = src[b];
    if (o < 0) return;
    int t = threadIdx.x;
    to[b * 512 + t] = from[o * 512 + t];
    to[b * 512 + 256 + t] = from[o * 512 + 256 + t];
}

// Interpolation: new box list[q] (level l, no counterpart in the old tree)
// from its parent in the new tree (already filled), with the stencil of the
// correction prolongation applied to phi itself, 1/4 p(C) + 1/4 (p(C + s_x) +
// p(C + s_y) + p(C + s_z)), C the parent cell and s the side of the fine cell
// in it; a neighbour outside the parent is the parent's ghost on that face
// (same-level neighbour, boundary condition or refinement-boundary value).
// Exact for linear functions.
__global__ __launch_bounds__(256) void k_transfer_interp(Geo g, double *__restrict__ phi,
                                                         const double *__restrict__ chat,
                                                         const int32_t *__restrict__ list, int64_t nlist) {
    __shared__ double P[512], H[384];
    int64_t q = xcd_map(blockIdx.x, nlist);
    if (q >= nlist) return;
    int64_t b = list[q];
    int64_t p = g.parent[b];
    int o[3] = {g.ijk[b * 4] & 1, g.ijk[b * 4 + 1] & 1, g.ijk[b * 4 + 2] & 1};
    int t = threadIdx.x;
    stage_full<double>(g, phi, chat, p, P, H);
    __syncthreads();
    // parent value at (x, y, z); at most one coordinate is -1 or 8 (a face ghost)
    auto pv = [&](int x, int y, int z) __attribute__((always_inline)) -> double {
        if (x < 0) return H[0 * 64 + z * 8 + y];
        if (x > 7) return H[1 * 64 + z * 8 + y];
        if (y < 0) return H[2 * 64 + z * 8 + x];
        if (y > 7) return H[3 * 64 + z * 8 + x];
        if (z < 0) return H[4 * 64 + y * 8 + x];
        if (z > 7) return H[5 * 64 + y * 8 + x];
        return P[cs_idx(x, y, z)];
    };
    int m = t & 3, j = (t >> 2) & 7, k = t >> 5;
#pragma unroll
    for (int c = 0; c < 2; c++) {
        int i = 2 * m + ((j + k + c) & 1);
        int cx = 4 * o[0] + (i >> 1), cy = 4 * o[1] + (j >> 1), cz = 4 * o[2] + (k >> 1);
        int sx = (i & 1) ? 1 : -1, sy = (j & 1) ? 1 : -1, sz = (k & 1) ? 1 : -1;
        double d0 = pv(cx, cy, cz), dx = pv(cx + sx, cy, cz), dy = pv(cx, cy + sy, cz),
               dz = pv(cx, cy, cz + sz);
        phi[b * 512 + c * 256 + t] = 0.25 * d0 + 0.25 * (dx + dy + dz);
    }
}

// phi (FP64) += e (FP32) on every cell: the update of the mixed-precision
// iterative refinement.
__global__ __launch_bounds__(256) void k_ir_update(double *__restrict__ phi, const float *__restrict__ e,
                                                   int64_t count) {
    int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (q < count) phi[q] += (double)e[q];
}

// Per-tree reduction of the per-box partials in a fixed order, in two
// stages.  Stage 1 sums the partials of chunk c, the leaf boxes at positions
// leaf_tree[chunk[c].begin .. chunk[c].end) (a range of one tree, at most
// kReduceChunk long).  Stage 2 sums the chunks choff[t] .. choff[t+1] of tree
// t into result[2t] (sum) and result[2t+1] (max).  result is pinned host
// memory: after a stream synchronisation the host reads it, with no copy.
//
// Where no tree has more than kReduceOneMax chunks, one launch does both
// stages (k_reduce_one, one workgroup per tree, four chunks at a time);
// larger trees spread their chunks over workgroups and sum them in a second
// launch.  Either way every sum is taken in the same order, so the results
// are the same bits.  A check on the uniform 32^3 grid spent 4.4 us on each
// of two reductions and 4.1 us on the copy, the price of three launches.

// Sum and max over the 256 threads t of a group (S, M: the group's 256), valid
// in its thread 0: pairs 128 and 64 apart through LDS, the rest in a wavefront.
__device__ __forceinline__ void block_sum_max(int t, double &s, double &m, double *S, double *M) {
    S[t] = s;
    M[t] = m;
    __syncthreads();
    if (t >= 64) return;
    s = (S[t] + S[t + 128]) + (S[t + 64] + S[t + 192]);
    m = nanmax(nanmax(M[t + 192], M[t + 64]), nanmax(M[t + 128], M[t]));
    for (int w = 32; w > 0; w >>= 1) {
        s += __shfl_down(s, w);
        m = nanmax(__shfl_down(m, w), m);
    }
}
// This thread's share of chunk c.  All loads go out before the first sum: as
// a loop of gather and sum, 8 chunks took a workgroup 17.6 us, now 10.2.
__device__ __forceinline__ void chunk_part(const double *__restrict__ partial, const int32_t *__restrict__ leaf_tree,
                                           const int32_t *__restrict__ chunk, int c, int t, double &s, double &m) {
    constexpr int n = kReduceChunk / 256;
    const int beg = chunk[3 * c + 1] + t, end = chunk[3 * c + 2];
    int p[n];
    double v[n], x[n];
#pragma unroll
    for (int k = 0; k < n; k++) p[k] = beg + 256 * k < end ? leaf_tree[beg + 256 * k] : -1;
#pragma unroll
    for (int k = 0; k < n; k++) {
        v[k] = x[k] = 0.0;
        if (p[k] >= 0) {
            v[k] = partial[2 * (int64_t)p[k]];
            x[k] = partial[2 * (int64_t)p[k] + 1];
        }
    }
#pragma unroll
    for (int k = 0; k < n; k++)
        if (p[k] >= 0) {
            s += v[k];
            m = nanmax(x[k], m);
        }
}

__global__ __launch_bounds__(256) void k_reduce_chunks(const double *__restrict__ partial,
                                                       const int32_t *__restrict__ leaf_tree,
                                                       const int32_t *__restrict__ chunk,
                                                       double *__restrict__ part2) {
    __shared__ double S[256], M[256];
    int c = blockIdx.x, t = threadIdx.x;
    double s = 0.0, m = 0.0;
    chunk_part(partial, leaf_tree, chunk, c, t, s, m);
    block_sum_max(t, s, m, S, M);
    if (t == 0) {
        part2[2 * c] = s;
        part2[2 * c + 1] = m;
    }
}

__global__ __launch_bounds__(256) void k_reduce_trees(const double *__restrict__ part2,
                                                      const int32_t *__restrict__ choff,
                                                      double *__restrict__ result) {
    __shared__ double S[256], M[256];
    int tr = blockIdx.x, t = threadIdx.x;
    double s = 0.0, m = 0.0;
    for (int c = choff[tr] + t; c < choff[tr + 1]; c += 256) {
        s += part2[2 * c];
        m = nanmax(part2[2 * c + 1], m);
    }
    block_sum_max(t, s, m, S, M);
    if (t == 0) {
        result[2 * tr] = s;
        result[2 * tr + 1] = m;
    }
}

__global__ __launch_bounds__(1024) void k_reduce_one(const double *__restrict__ partial,
                                                     const int32_t *__restrict__ leaf_tree,
                                                     const int32_t *__restrict__ chunk,
                                                     const int32_t *__restrict__ choff,
                                                     double *__restrict__ result) {
    __shared__ double S[1024], M[1024], CS[kReduceOneMax], CM[kReduceOneMax];
    const int tr = blockIdx.x, t = threadIdx.x & 255, g = threadIdx.x >> 8;
    const int c0 = choff[tr], nc = choff[tr + 1] - c0;
    for (int p = 0; p < nc; p += 4) {  // block-uniform
        double s = 0.0, m = 0.0;
        if (p + g < nc) chunk_part(partial, leaf_tree, chunk, c0 + p + g, t, s, m);
        block_sum_max(t, s, m, S + 256 * g, M + 256 * g);
        if (t == 0 && p + g < nc) {
            CS[p + g] = s;
            CM[p + g] = m;
        }
        __syncthreads();
    }
    double s = 0.0, m = 0.0;
    if (t < nc) {
        s += CS[t];
        m = nanmax(CM[t], m);
    }
    block_sum_max(t, s, m, S + 256 * g, M + 256 * g);
    if (threadIdx.x == 0) {
        result[2 * tr] = s;
        result[2 * tr + 1] = m;
    }
}

// Streaming copy with 16-byte vector accesses, grid-stride: the achievable
// device bandwidth reference of the roofline.
__global__ __launch_bounds__(256) void k_copy16(const uint4 *__restrict__ src, uint4 *__restrict__ dst,
                                                int64_t n16) {
    int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < n16; q += stride) dst[q] = src[q];
}

}  // namespace

// ------------------------------------------------------------- launchers

template <typename T>
void launch_fill(T *p, int64_t count, T v, hipStream_t s) {
    if (count <= 0) return;
    hipLaunchKernelGGL(k_fill<T>, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, p, count, v);
}
template <typename T>
void launch_pack(const double *nat, T *cs, int64_t nbox, hipStream_t s) {
    hipLaunchKernelGGL(k_pack<T>, dim3((unsigned)(nbox * 2)), dim3(256), 0, s, nat, cs, nbox);
}
template <typename T>
void launch_unpack(const T *cs, double *nat, int64_t nbox, hipStream_t s) {
    hipLaunchKernelGGL(k_unpack<T>, dim3((unsigned)(nbox * 2)), dim3(256), 0, s, cs, nat, nbox);
}
template <typename T, int CPT>
void launch_gsrb_cpt(const Geo &g, T *phi, const T *rhs, const T *chat, int64_t b0, int64_t nb,
                     T h2, int colour, int xcd, hipStream_t s, const int32_t *rmask, double *phi64) {
    dim3 grid((unsigned)(xcd ? xcd_grid(nb) : nb)), block(256 / CPT);
    if (colour == 0)
        hipLaunchKernelGGL((k_gsrb<0, T, CPT>), grid, block, 0, s, g, phi, rhs, chat, b0, nb, h2, xcd,
                           nullptr, nullptr);
    else if (phi64)
        hipLaunchKernelGGL((k_gsrb<1, T, CPT, kSweepIrUpdate>), grid, block, 0, s, g, phi, rhs, chat, b0, nb,
                           h2, xcd, rmask, phi64);
    else if (rmask)
        hipLaunchKernelGGL((k_gsrb<1, T, CPT, kSweepRestrict>), grid, block, 0, s, g, phi, rhs, chat, b0, nb,
                           h2, xcd, rmask, nullptr);
    else
        hipLaunchKernelGGL((k_gsrb<1, T, CPT>), grid, block, 0, s, g, phi, rhs, chat, b0, nb, h2, xcd,
                           nullptr, nullptr);
}

template <typename T>
void launch_gsrb_sweep(const Geo &g, const T *src, T *dst, T *rhs, const T *chat, int64_t b0,
                       int64_t nb, T h2, int xcd, hipStream_t s, int fas, const int32_t *isleaf,
                       T inv_h2, T *fasbuf) {
    if (nb <= 0) return;
    dim3 grid((unsigned)(xcd ? xcd_grid(nb) : nb));
    if (fas)
        hipLaunchKernelGGL((k_gsrb_sweep<T, true>), grid, dim3(256), 0, s, g, src, dst, rhs, chat, b0, nb, h2,
                           xcd, fas, isleaf, inv_h2, fasbuf);
    else
        hipLaunchKernelGGL((k_gsrb_sweep<T, false>), grid, dim3(256), 0, s, g, src, dst, rhs, chat, b0, nb,
                           h2, xcd, 0, isleaf, inv_h2, fasbuf);
}

template <typename T>
void launch_gsrb(const Geo &g, T *phi, const T *rhs, const T *chat, int64_t b0, int64_t nb, T h2,
                 int colour, int variant, hipStream_t s, const int32_t *rmask, double *phi64) {
    if (nb <= 0) return;
    if (colour != 1 || (phi64 ? !gsrb_updates(variant) : !gsrb_restricts(variant))) {
        rmask = nullptr;  // callers check gsrb_restricts / gsrb_updates first
        phi64 = nullptr;
    }
    if (sizeof(T) != 4) phi64 = nullptr;
    if (variant >= kGsrbPipeVariant) {
        // persistent workgroups: at most 2048 (c = 5) or 4096 (c = 6)
        int64_t cap = variant >= kGsrbPipeVariant + 2 ? 4096 : 2048;
        int xcd = variant & 1;
        int64_t nw = nb < cap ? nb : cap;
        dim3 grid((unsigned)(xcd ? xcd_grid(nw) : nw));
        if (colour == 0)
            hipLaunchKernelGGL((k_gsrb_pipe<0, T>), grid, dim3(128), 0, s, g, phi, rhs, chat, b0, nb, h2, xcd);
        else
            hipLaunchKernelGGL((k_gsrb_pipe<1, T>), grid, dim3(128), 0, s, g, phi, rhs, chat, b0, nb, h2, xcd);
        return;
    }
    if (variant >= kGsrbOctVariant && (nb & 7) == 0) {
        int64_t noct = nb >> 3;
        int xcd = variant & 1;
        dim3 grid((unsigned)(xcd ? xcd_grid(noct) : noct));
        if (colour == 0)
            hipLaunchKernelGGL((k_gsrb_oct<0, T>), grid, dim3(512), 0, s, g, phi, rhs, chat, b0, noct, h2, xcd,
                               nullptr, nullptr);
        else if (phi64)
            hipLaunchKernelGGL((k_gsrb_oct<1, T, true>), grid, dim3(512), 0, s, g, phi, rhs, chat, b0, noct, h2,
                               xcd, rmask, phi64);
        else
            hipLaunchKernelGGL((k_gsrb_oct<1, T>), grid, dim3(512), 0, s, g, phi, rhs, chat, b0, noct, h2, xcd,
                               nullptr, nullptr);
        return;
    }
    if (variant >= kGsrbHalfVariants) variant = kGsrbDefault;
    int xcd = variant & 1;
    switch (variant >> 1) {
    case 0: launch_gsrb_cpt<T, 1>(g, phi, rhs, chat, b0, nb, h2, colour, xcd, s, rmask, phi64); break;
    case 2: launch_gsrb_cpt<T, 4>(g, phi, rhs, chat, b0, nb, h2, colour, xcd, s, rmask, phi64); break;
    default: launch_gsrb_cpt<T, 2>(g, phi, rhs, chat, b0, nb, h2, colour, xcd, s, rmask, phi64); break;
    }
}
template <typename T>
void launch_cf_coarse(const Geo &g, const T *phi, T *chat, const int32_t *slots, int64_t s0,
                      int64_t ns, hipStream_t s) {
    if (ns <= 0) return;
    hipLaunchKernelGGL(k_cf_coarse<T>, dim3((unsigned)((ns + 3) / 4)), dim3(256), 0, s, g, phi, chat,
                       slots, s0, ns);
}
template <typename T>
void launch_resid_restrict(const Geo &g, T *phi, T *rhs, T *old, const T *chat, int64_t b0,
                           int64_t nb, const int32_t *leaf_prev, int64_t nleaf_prev, T inv_h2,
                           hipStream_t s, const int32_t *leafpos, double *partial, double vol) {
    if (nb + nleaf_prev <= 0) return;
    dim3 grid((unsigned)(xcd_grid(nb) + nleaf_prev));
    if (partial)
        hipLaunchKernelGGL((k_resid_restrict<T, true>), grid, dim3(128), 0, s, g, phi, rhs, old, chat, b0, nb,
                           leaf_prev, nleaf_prev, inv_h2, leafpos, partial, vol);
    else
        hipLaunchKernelGGL((k_resid_restrict<T, false>), grid, dim3(128), 0, s, g, phi, rhs, old, chat, b0, nb,
                           leaf_prev, nleaf_prev, inv_h2, leafpos, partial, vol);
}
template <typename T>
void launch_fas_rhs(const Geo &g, const T *phi, T *rhs, const T *chat, const int32_t *list,
                    int64_t nlist, T inv_h2, hipStream_t s) {
    if (nlist <= 0) return;
    hipLaunchKernelGGL(k_fas_rhs<T>, dim3((unsigned)xcd_grid(nlist)), dim3(128), 0, s, g, phi, rhs,
                       chat, list, nlist, inv_h2);
}
template <typename T>
void launch_prolong_cf(const Geo &g, T *phi, const T *old, int64_t b0, int64_t nb, T *chat,
                       const int32_t *slots, int64_t s0, int64_t ns, hipStream_t s) {
    if (nb <= 0 && ns <= 0) return;
    dim3 grid((unsigned)(xcd_grid(nb) + (ns + 3) / 4));
    hipLaunchKernelGGL(k_prolong_cf<T>, grid, dim3(256), 0, s, g, phi, old, b0, nb, chat, slots, s0, ns);
}
template <typename T>
void launch_delta_pad(const Geo &g, const T *phi, const T *old, const int32_t *refined, int64_t nref, T *pad,
                      T *chat, const int32_t *slots, int64_t s0, int64_t ns, hipStream_t s) {
    if (nref <= 0 && ns <= 0) return;
    dim3 grid((unsigned)(xcd_grid(nref) + (ns + 3) / 4));
    hipLaunchKernelGGL(k_delta_pad<T>, grid, dim3(256), 0, s, g, phi, old, refined, nref, pad, chat, slots, s0, ns);
}
template <typename T>
void launch_gsrb_pro(const Geo &g, T *phi, const T *rhs, const T *pad, const T *chat, int64_t b0, int64_t nb,
                     T h2, int colour, hipStream_t s) {
    if (nb <= 0) return;
    dim3 grid((unsigned)xcd_grid(nb));
    if (colour == 0)
        hipLaunchKernelGGL(k_gsrb_pro_red<T>, grid, dim3(128), 0, s, g, phi, rhs, pad, chat, b0, nb, h2);
    else
        hipLaunchKernelGGL(k_gsrb_pro_black<T>, grid, dim3(128), 0, s, g, phi, rhs, pad, chat, b0, nb, h2);
}
template <typename T>
void launch_coarse(const Geo &g, T *phi, const T *rhs, const double *eig, int64_t b0, int64_t nroot,
                   double h, hipStream_t s) {
    hipLaunchKernelGGL(k_coarse<T>, dim3((unsigned)nroot), dim3(512), 0, s, g, phi, rhs, eig, b0, h);
}
template <typename T>
void launch_bottom(const Geo &g, T *phi, T *rhs, T *old, const double *eig, int64_t r0, int ntree,
                   const int32_t *root2, double h2, double h1, int nd, int nu, int fmg, int fas2,
                   const int32_t *isleaf, hipStream_t s) {
    hipLaunchKernelGGL(k_bottom<T>, dim3((unsigned)ntree), dim3(1024), 0, s, g, phi, rhs, old, eig, r0, root2,
                       (T)(h2 * h2), (T)(1.0 / (h2 * h2)), (T)(1.0 / (h1 * h1)), h1, nd, nu, fmg, fas2,
                       isleaf);
}
template <typename T>
void launch_restrict_phi(const Geo &g, T *phi, int64_t b0, int64_t nb, hipStream_t s) {
    if (nb <= 0) return;
    hipLaunchKernelGGL(k_restrict_phi<T>, dim3((unsigned)xcd_grid(nb)), dim3(64), 0, s, g, phi, b0, nb);
}
template <typename T>
void launch_restrict_leaves(const Geo &g, T *phi, const int32_t *leaf, int64_t nleaf, hipStream_t s) {
    if (nleaf <= 0) return;
    hipLaunchKernelGGL(k_restrict_leaves<T>, dim3((unsigned)xcd_grid(nleaf)), dim3(64), 0, s, g, phi, leaf,
                       nleaf);
}
void launch_leaf_norms(const Geo &g, const double *phi, const double *rhs, const double *chat,
                       const int32_t *leaf, int64_t nleaf, double *partial, float *r_out,
                       hipStream_t s) {
    if (nleaf <= 0) return;
    hipLaunchKernelGGL(k_leaf_norms, dim3((unsigned)xcd_grid(nleaf)), dim3(256), 0, s, g, phi, rhs,
                       chat, leaf, nleaf, partial, r_out);
}
void launch_box_norms(const Geo &g, const double *phi, const double *rhs, const double *chat, const int32_t *leaf,
                      int64_t q0, int64_t nq, double *partial, float *r_out, hipStream_t s) {
    if (nq <= 0) return;
    const double ilen2 = 1.0 / (g.len * g.len), len3 = g.len * g.len * g.len;
    if (r_out)
        hipLaunchKernelGGL(k_box_norms<true>, dim3((unsigned)xcd_grid(nq)), dim3(128), 0, s, g, phi, rhs, chat,
                           leaf, q0, nq, partial, r_out, ilen2, len3);
    else
        hipLaunchKernelGGL(k_box_norms<false>, dim3((unsigned)xcd_grid(nq)), dim3(128), 0, s, g, phi, rhs, chat,
                           leaf, q0, nq, partial, r_out, ilen2, len3);
}
template <typename T>
void launch_leaf_apply(const Geo &g, const T *x, const T *chat, const int32_t *leaf, int64_t nleaf,
                       T *out, hipStream_t s) {
    if (nleaf <= 0) return;
    hipLaunchKernelGGL(k_leaf_apply<T>, dim3((unsigned)xcd_grid(nleaf)), dim3(256), 0, s, g, x, chat, leaf,
                       nleaf, out);
}
template void launch_leaf_apply<float>(const Geo &, const float *, const float *, const int32_t *,
                                       int64_t, float *, hipStream_t);
void launch_learned_sums(const Geo &g, const float *x, const float *r32, const int32_t *leaf, const int32_t *tab,
                         const LearnedRanges &R, int nchunk, double *part, double *sums, hipStream_t s) {
    hipLaunchKernelGGL(k_learned_sums, dim3((unsigned)nchunk), dim3(512), 0, s, g, x, r32, leaf, tab, R, part);
    hipLaunchKernelGGL(k_learned_reduce, dim3((unsigned)(9 * R.nrange)), dim3(256), 0, s, part, tab, R, nchunk,
                       sums);
}
void launch_efield(const Geo &g, const double *phi, const double *chat, int64_t n, double *e_face,
                   double *e_norm, hipStream_t s) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_efield, dim3((unsigned)xcd_grid(n)), dim3(256), 0, s, g, phi, chat, n, e_face, e_norm);
}
void launch_face_xt(const int32_t *nbr, const int32_t *cfslot, int64_t n, int32_t *xt, hipStream_t s) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_face_xt, dim3((unsigned)((6 * n + 255) / 256)), dim3(256), 0, s, nbr, cfslot, n, xt);
}
void launch_refine_near(const int32_t *n27, const int32_t *isleaf, const double *scores, int64_t n, double *near,
                        hipStream_t s) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_refine_near, dim3((unsigned)((n + 7) / 8)), dim3(256), 0, s, n27, isleaf, scores, n,
                       near);
}
void launch_refine_scores(const Geo &g, const double *rhs, int64_t n, double *scores, hipStream_t s) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_refine_scores, dim3((unsigned)xcd_grid((n + 3) / 4)), dim3(256), 0, s, g, rhs, n, scores);
}
void launch_transfer_copy(const double *from, double *to, const int32_t *src, int64_t n, hipStream_t s) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_transfer_copy, dim3((unsigned)xcd_grid(n)), dim3(256), 0, s, from, to, src, n);
}
void launch_transfer_interp(const Geo &g, double *phi, const double *chat, const int32_t *list, int64_t nlist,
                            hipStream_t s) {
    if (nlist <= 0) return;
    hipLaunchKernelGGL(k_transfer_interp, dim3((unsigned)xcd_grid(nlist)), dim3(256), 0, s, g, phi, chat, list,
                       nlist);
}
void launch_ir_update(double *phi, const float *e, int64_t count, hipStream_t s) {
    if (count <= 0) return;
    hipLaunchKernelGGL(k_ir_update, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, phi, e, count);
}
void launch_copy16(const void *src, void *dst, int64_t n16, int blocks, hipStream_t s) {
    if (n16 <= 0) return;
    hipLaunchKernelGGL(k_copy16, dim3((unsigned)blocks), dim3(256), 0, s, (const uint4 *)src, (uint4 *)dst,
                       n16);
}
void launch_reduce_trees(const double *partial, const int32_t *leaf_tree, const int32_t *chunk,
                         int64_t nchunk, int maxchunk, const int32_t *choff, int ntree, double *part2,
                         double *result, hipStream_t s) {
    if (maxchunk <= kReduceOneMax) {
        hipLaunchKernelGGL(k_reduce_one, dim3((unsigned)ntree), dim3(1024), 0, s, partial, leaf_tree, chunk, choff,
                           result);
        return;
    }
    hipLaunchKernelGGL(k_reduce_chunks, dim3((unsigned)nchunk), dim3(256), 0, s, partial, leaf_tree, chunk, part2);
    hipLaunchKernelGGL(k_reduce_trees, dim3((unsigned)ntree), dim3(256), 0, s, part2, choff, result);
}

#define MG_INSTANTIATE(T)                                                                        \
    template void launch_fill<T>(T *, int64_t, T, hipStream_t);                                  \
    template void launch_pack<T>(const double *, T *, int64_t, hipStream_t);                     \
    template void launch_unpack<T>(const T *, double *, int64_t, hipStream_t);                   \
    template void launch_gsrb<T>(const Geo &, T *, const T *, const T *, int64_t, int64_t, T, int, \
                                 int, hipStream_t, const int32_t *, double *);                   \
    template void launch_gsrb_sweep<T>(const Geo &, const T *, T *, T *, const T *, int64_t,       \
                                       int64_t, T, int, hipStream_t, int, const int32_t *, T, T *); \
    template void launch_restrict_leaves<T>(const Geo &, T *, const int32_t *, int64_t, hipStream_t); \
    template void launch_cf_coarse<T>(const Geo &, const T *, T *, const int32_t *, int64_t,     \
                                      int64_t, hipStream_t);                                     \
    template void launch_resid_restrict<T>(const Geo &, T *, T *, T *, const T *, int64_t,       \
                                           int64_t, const int32_t *, int64_t, T, hipStream_t,    \
                                           const int32_t *, double *, double);                   \
    template void launch_fas_rhs<T>(const Geo &, const T *, T *, const T *, const int32_t *,     \
                                    int64_t, T, hipStream_t);                                    \
    template void launch_prolong_cf<T>(const Geo &, T *, const T *, int64_t, int64_t, T *,       \
                                       const int32_t *, int64_t, int64_t, hipStream_t);          \
    template void launch_gsrb_pro<T>(const Geo &, T *, const T *, const T *, const T *, int64_t,   \
                                     int64_t, T, int, hipStream_t);                              \
    template void launch_delta_pad<T>(const Geo &, const T *, const T *, const int32_t *, int64_t, \
                                      T *, T *, const int32_t *, int64_t, int64_t, hipStream_t);   \
    template void launch_coarse<T>(const Geo &, T *, const T *, const double *, int64_t, int64_t, \
                                   double, hipStream_t);                                         \
    template void launch_restrict_phi<T>(const Geo &, T *, int64_t, int64_t, hipStream_t);        \
    template void launch_bottom<T>(const Geo &, T *, T *, T *, const double *, int64_t, int,     \
                                   const int32_t *, double, double, int, int, int, int,          \
                                   const int32_t *, hipStream_t);
MG_INSTANTIATE(double)
MG_INSTANTIATE(float)
#undef MG_INSTANTIATE

}  // namespace mg

// ax_kernels.hip -- element-local kernels of the SEM Helmholtz operator for gfx950.
//
// Operator (Jansson et al., arXiv 2107.01243, Section 2, Eq. 9):
//   w_e = h1 D^T G_e D u_e + h2 B_e u_e  on every hexahedral element,
// with D the 1-D GLL derivative matrix applied along r, s and t, and G_e the six
// geometric factors (G11, G22, G33, G12, G13, G23) per point.
//
// Work decomposition ("pencil" layout).  One element is handled by lx*lx lanes.
// A lane with in-element index t = a + lx*b owns, at different stages,
//   t-pencil: the lx points (i = a, j = b, k = 0..lx-1)   (its home layout)
//   r-pencil: the lx points (i = 0..lx-1, j = a, k = b)
//   s-pencil: the lx points (i = a, j = 0..lx-1, k = b)
// In the home layout the lanes of an element read and write HBM at offsets
// t + lx^2 k: for each k one wave instruction covers lx^2 consecutive values, so
// every global access is fully coalesced.  Each 1-D derivative is a
// register-only product with D in its even-odd form (half the FMAs of the dense
// lx x lx product); its entries are wave-uniform (they travel in the
// kernel-argument segment and are read through scalar loads).  LDS is used only
// to transpose pencils; every LDS row has stride lx+1 so that the three pencil
// access patterns are free of bank conflicts.
//
// This file is compiled once per lx (-DSEM_LX=<lx>) so that the per-lx
// instantiations build in parallel; it exports plain host launchers.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <type_traits>

#include "sem_kernels.h"
#include "sem_wave.h"
#include "sem_pencil.h"

#ifndef SEM_LX
#error "compile with -DSEM_LX=<lx>"
#endif
#define SEM_BOUNDS(NT) __launch_bounds__((NT))
#define SEM_BOUNDS2(NT, W) __launch_bounds__((NT)) __attribute__((amdgpu_waves_per_eu((W))))

namespace sem {

// ------------------------------------------------------------------ launch shape
// Elements per workgroup: fill whole wave64s where possible, keep the two LDS
// transpose buffers within 64 KB (up to 160 KB for a single large element), keep
// the register budget that the workgroup's size leaves each lane above what a lane
// needs, and aim at about 256 lanes per workgroup.
template <int LX, typename T>
struct Shape {
    static constexpr int NP = LX * LX;                       // lanes per element
    static constexpr int PAD = LX + 1;                       // LDS row stride
    static constexpr int ESZ = NP * PAD;                     // one LDS buffer, one element
    static constexpr int EBYTES = 2 * ESZ * (int)sizeof(T);  // LDS per element
    // 32-bit registers a lane needs, estimated: six geometric-factor rows and about
    // eight more pencil rows (u, its three derivatives, w, h1, h2 B, dinv), plus
    // scalars.  A SIMD gives 512 per lane to one wave, 512 / k to each of k waves, and
    // a workgroup of W waves puts ceil(W / 4) of them on one SIMD.
    static constexpr int REGS = 14 * LX * (int)sizeof(T) / 4 + 40;
    static constexpr int MAX_WAVES = 4 * (512 / REGS > 1 ? 512 / REGS : 1);
    static constexpr int pick()
    {
        int best = 1;
        double best_score = 1e9;
        for (int e = 1; e * NP <= 1024; ++e) {
            if (e > 1 && e * EBYTES > 64 * 1024) break;
            const int thr = e * NP;
            const int waves = (thr + 63) / 64;
            if (e > 1 && waves > MAX_WAVES) break;
            const double waste = double(waves * 64 - thr) / double(waves * 64);
            const double dist = (thr > 256 ? thr - 256 : 256 - thr) / 1024.0;
            const double score = waste + 0.25 * dist;
            if (score < best_score - 1e-12) { best_score = score; best = e; }
        }
        return best;
    }
#ifndef SEM_LEAN_LX
#define SEM_LEAN_LX 10
#endif
    // lx >= SEM_LEAN_LX: the register-lean kernels, one element per workgroup, with a
    // floor on the waves per SIMD the register allocation must leave room for (two
    // FP64 / four FP32 up to lx = 12, half that above)
    static constexpr bool LEAN = LX >= SEM_LEAN_LX;
    static constexpr int EPB = LEAN ? 1 : pick();
    static constexpr int NT = EPB * NP;
    static constexpr int MINW = !LEAN ? 1 : (sizeof(T) == 8 ? (LX <= 12 ? 2 : 1) : (LX <= 12 ? 4 : 2));
};

template <int LX, typename T>
struct Lds {
    T buf[2][Shape<LX, T>::EPB][Shape<LX, T>::ESZ];
};

// out = D in   (derivative along the pencil), even-odd form
template <int LX, typename T>
__device__ __forceinline__ void dmul(const DEo<LX, T> &D, const T (&in)[LX], T (&out)[LX])
{
    constexpr int H = LX / 2, N = LX - 1;
    T e[H > 0 ? H : 1], o[H > 0 ? H : 1];
#pragma unroll
    for (int l = 0; l < H; ++l) {
        e[l] = in[l] + in[N - l];
        o[l] = in[l] - in[N - l];
    }
#pragma unroll
    for (int m = 0; m < H; ++m) {
        T se = D.S[m * H] * e[0];
        T ao = D.A[m * H] * o[0];
#pragma unroll
        for (int l = 1; l < H; ++l) {
            se = fma(D.S[m * H + l], e[l], se);
            ao = fma(D.A[m * H + l], o[l], ao);
        }
        if constexpr (LX % 2 == 1) se = fma(D.cm[m], in[H], se);
        out[m] = ao + se;
        out[N - m] = ao - se;
    }
    if constexpr (LX % 2 == 1) {
        T c = T(0);
#pragma unroll
        for (int l = 0; l < H; ++l) c = fma(D.rm[l], o[l], c);
        out[H] = c;
    }
}

// out = D^T in   (transposed derivative along the pencil), even-odd form
template <int LX, typename T>
__device__ __forceinline__ void dtmul(const DEo<LX, T> &D, const T (&in)[LX], T (&out)[LX])
{
    constexpr int H = LX / 2, N = LX - 1;
    T e[H > 0 ? H : 1], o[H > 0 ? H : 1];
#pragma unroll
    for (int l = 0; l < H; ++l) {
        e[l] = in[l] + in[N - l];
        o[l] = in[l] - in[N - l];
    }
#pragma unroll
    for (int m = 0; m < H; ++m) {
        T se = D.A[m] * e[0];
        T ao = D.S[m] * o[0];
#pragma unroll
        for (int l = 1; l < H; ++l) {
            se = fma(D.A[l * H + m], e[l], se);
            ao = fma(D.S[l * H + m], o[l], ao);
        }
        if constexpr (LX % 2 == 1) se = fma(D.rm[m], in[H], se);
        out[m] = ao + se;
        out[N - m] = ao - se;
    }
    if constexpr (LX % 2 == 1) {
        T c = T(0);
#pragma unroll
        for (int l = 0; l < H; ++l) c = fma(D.cm[l], o[l], c);
        out[H] = c;
    }
}

// Where a kernel reads D from.  DArg: the kernel-argument copy (wave-uniform values
// the compiler keeps in scalar registers; right when they fit, as in FP32 and up to
// lx = 8 in FP64).  DMem: a copy in device memory read with scalar loads one row at a
// time where it is used; at lx = 12 in FP64 the 72 doubles of the even-odd D exceed the
// scalar register file, and holding them costs a spill to vector-register lanes plus
// two v_readlane per use (more VALU instructions than the FMAs themselves).
template <int LX, typename T>
struct DArg {
    const DEo<LX, T> &D;
    __device__ void mul(const T (&in)[LX], T (&out)[LX]) const { dmul<LX, T>(D, in, out); }
    __device__ void tmul(const T (&in)[LX], T (&out)[LX]) const { dtmul<LX, T>(D, in, out); }
};

// p + 0 with the 0 opaque to the optimiser: loads through the result are not merged
// with, or moved ahead of, loads through another such pointer; the address space of
// p is kept (an opaque pointer would turn global loads into flat ones).
template <typename T>
__device__ __forceinline__ const T *fresh(const T *p)
{
    int64_t z = 0;
    asm volatile("" : "+s"(z));
    return p + z;
}

template <int LX, typename T>
struct DMem {
    const DEo<LX, T> *Dg;
    __device__ void mul(const T (&in)[LX], T (&out)[LX]) const
    {
        constexpr int H = LX / 2, N = LX - 1;
        T e[H > 0 ? H : 1], o[H > 0 ? H : 1];
#pragma unroll
        for (int l = 0; l < H; ++l) {
            e[l] = in[l] + in[N - l];
            o[l] = in[l] - in[N - l];
        }
#pragma unroll
        for (int m = 0; m < H; ++m) {
            const DEo<LX, T> *R = fresh(Dg);  // this row's constants loaded here
            T se = R->S[m * H] * e[0];
            T ao = R->A[m * H] * o[0];
#pragma unroll
            for (int l = 1; l < H; ++l) {
                se = fma(R->S[m * H + l], e[l], se);
                ao = fma(R->A[m * H + l], o[l], ao);
            }
            if constexpr (LX % 2 == 1) se = fma(R->cm[m], in[H], se);
            out[m] = ao + se;
            out[N - m] = ao - se;
        }
        if constexpr (LX % 2 == 1) {
            const DEo<LX, T> *R = fresh(Dg);
            T c = T(0);
#pragma unroll
            for (int l = 0; l < H; ++l) c = fma(R->rm[l], o[l], c);
            out[H] = c;
        }
    }
    __device__ void tmul(const T (&in)[LX], T (&out)[LX]) const
    {
        constexpr int H = LX / 2, N = LX - 1;
        T e[H > 0 ? H : 1], o[H > 0 ? H : 1];
#pragma unroll
        for (int l = 0; l < H; ++l) {
            e[l] = in[l] + in[N - l];
            o[l] = in[l] - in[N - l];
        }
#pragma unroll
        for (int m = 0; m < H; ++m) {
            const DEo<LX, T> *R = fresh(Dg);
            T se = R->A[m] * e[0];
            T ao = R->S[m] * o[0];
#pragma unroll
            for (int l = 1; l < H; ++l) {
                se = fma(R->A[l * H + m], e[l], se);
                ao = fma(R->S[l * H + m], o[l], ao);
            }
            if constexpr (LX % 2 == 1) se = fma(R->rm[m], in[H], se);
            out[m] = ao + se;
            out[N - m] = ao - se;
        }
        if constexpr (LX % 2 == 1) {
            const DEo<LX, T> *R = fresh(Dg);
            T c = T(0);
#pragma unroll
            for (int l = 0; l < H; ++l) c = fma(R->cm[l], o[l], c);
            out[H] = c;
        }
    }
};

// Reference-space gradient of one field held as the lane's t-pencil `u`.
// Returns ur, us, ut as t-pencils.  Uses both LDS buffers; ends synchronised.
template <int LX, typename T>
__device__ __forceinline__ void grad(const DEo<LX, T> &D, const T (&u)[LX], T *s0, T *s1,
                                     int a, int b, T (&ur)[LX], T (&us)[LX], T (&ut)[LX])
{
    dmul<LX, T>(D, u, ut);
#pragma unroll
    for (int k = 0; k < LX; ++k) s0[lidx<LX>(a, b, k)] = u[k];
    esync<LX>();
    T v[LX], q[LX];
#pragma unroll
    for (int l = 0; l < LX; ++l) v[l] = s0[lidx<LX>(l, a, b)];   // r-pencil (j=a, k=b)
    dmul<LX, T>(D, v, q);
    T v2[LX], q2[LX];
#pragma unroll
    for (int l = 0; l < LX; ++l) v2[l] = s0[lidx<LX>(a, l, b)];  // s-pencil (i=a, k=b)
    dmul<LX, T>(D, v2, q2);
#pragma unroll
    for (int m = 0; m < LX; ++m) s1[lidx<LX>(m, a, b)] = q[m];
    esync<LX>();
#pragma unroll
    for (int m = 0; m < LX; ++m) s0[lidx<LX>(a, m, b)] = q2[m];
    esync<LX>();
#pragma unroll
    for (int k = 0; k < LX; ++k) {
        ur[k] = s1[lidx<LX>(a, b, k)];
        us[k] = s0[lidx<LX>(a, b, k)];
    }
    esync<LX>();
}

// acc = D_r^T wr + D_s^T ws + D_t^T wt for t-pencils wr, ws, wt.  Ends synchronised.
template <int LX, typename T>
__device__ __forceinline__ void div(const DEo<LX, T> &D, const T (&wr)[LX], const T (&ws)[LX],
                                    const T (&wt)[LX], T *s0, T *s1, int a, int b, T (&acc)[LX])
{
    dtmul<LX, T>(D, wt, acc);
#pragma unroll
    for (int k = 0; k < LX; ++k) {
        s0[lidx<LX>(a, b, k)] = wr[k];
        s1[lidx<LX>(a, b, k)] = ws[k];
    }
    esync<LX>();
    T v[LX], q[LX], v2[LX], q2[LX];
#pragma unroll
    for (int l = 0; l < LX; ++l) v[l] = s0[lidx<LX>(l, a, b)];
#pragma unroll
    for (int l = 0; l < LX; ++l) v2[l] = s1[lidx<LX>(a, l, b)];
    dtmul<LX, T>(D, v, q);
    dtmul<LX, T>(D, v2, q2);
    esync<LX>();
#pragma unroll
    for (int m = 0; m < LX; ++m) {
        s0[lidx<LX>(m, a, b)] = q[m];
        s1[lidx<LX>(a, m, b)] = q2[m];
    }
    esync<LX>();
#pragma unroll
    for (int k = 0; k < LX; ++k) acc[k] += s0[lidx<LX>(a, b, k)] + s1[lidx<LX>(a, b, k)];
    esync<LX>();
}

// A t-pencil in HBM: values p[k * lx^2], k = 0..lx-1 (p = element base + t).
template <int LX, typename T>
__device__ __forceinline__ void load_row(T (&r)[LX], const T *__restrict__ p, bool act)
{
    if (act) {
#pragma unroll
        for (int k = 0; k < LX; ++k) r[k] = p[k * LX * LX];
    } else {
#pragma unroll
        for (int k = 0; k < LX; ++k) r[k] = T(0);
    }
}

// Geometric-factor pencils are streamed once per application and the six planes
// (6 words per point) never fit the 256 MB last-level cache at production sizes, so
// they are read with non-temporal loads: this keeps the cache for the vectors
// (u, w, the Krylov vectors) that are reused between launches.  KEEP: plain loads, for a set
// that fits the cache and is found there by the next launch, and, where STREAM is unset, for
// rows of lx^2 values that are not whole lines: a line read non-temporally is dropped after
// its first use, and the part of it that another of the wave's loads wants is fetched again.
// reads_plainly has the rule by size.  (STREAM is not for the CG matvecs, which pass their
// vectors to the next kernels through the cache: FP32 of one field at lx = 9 gains, 135 -> 123 us
// an iteration, but at lx = 12 196 -> 217, of three at lx = 9 282 -> 304, FP64 at lx = 5 231 -> 247.)
template <int LX, typename T, int NF>
constexpr bool STREAM = sizeof(T) == 4 ? (LX & (LX - 1)) == 0 && !(LX == 16 && NF == 3)
                                       : LX != 5 && !(NF == 1 && (LX == 10 || LX == 11 || LX == 13));

// Whether w = A_L u (or with ADJ the h1-adjoint) of NF fields of n points reads G plainly;
// words: per point, all that the launch touches; mass: with a mass term; keep: AxArgs::keep.
// Up to 300 MB (340 where STREAM is unset) the set is found in the cache again.  Beyond, where
// STREAM is unset: as long as
// u and w stay in the cache between launches, G read plainly pushes them out, which most forms
// lose more by than the lines fetched twice cost them; when they no longer stay, all gain.
// Time with non-temporal loads over that with plain ones, Poisson (m: with a mass term), with
// the operands in the cache from the launch before / not there:
//  * up to 300 MB: FP64 at 4 million points lx = 5 1.16 / 1.32, 8 1.06 / 1.15, 10 1.20 / 1.29; FP32
//    at 6 million lx = 5 1.38 / 1.53, 8 1.07 / 1.16, 10 1.31 / 1.43, 12 1.14 / 1.23.
//  * one FP32 field at 12 million: lx = 5 1.11 / 1.22 (m 0.99 / 1.10), 6 1.09 / 1.24 (0.90 / 1.02), 7
//    1.05 / 1.21 (0.98 / 1.11), 9 1.06 / 1.23 (0.96 / 1.10), 10 1.00 / 1.14 (0.95 / 1.05), 11 0.99 / 1.12
//    (0.93 / 1.03), 12 0.92 / 1.02 (0.91 / 0.97), 13 0.98 / 1.11 (0.94 / 1.04), 14 0.95 / 1.01 (0.92 /
//    0.96), 15 1.01 / 1.04 (0.99 / 1.00); m at 25 million 0.93 to 1.16 / 1.02 to 1.19.
//  * three FP32 fields at 9 million: lx = 5 0.95 / 1.09, 6 0.86 / 1.04, 7 0.99 / 1.02, 9 0.91 / 1.06, 10
//    0.87 / 1.06, 12 0.92 / 0.99; at 16 million 1.00 to 1.20.
//  * FP64 at 9 million: lx = 5 0.90 / 1.05 (m 0.85 / 0.95), 10 0.94 / 1.05 (0.89 / 0.98), 11 0.91 /
//    1.01 (0.89 / 0.96), 13 0.94 / 1.03 (0.92 / 0.97); at 25 million 1.02 to 1.07 / 1.02 to 1.06.
//  * the adjoint at 12 million: FP32 lx = 5 1.12 / 1.10, 6 0.99 / 1.01, 10 1.06 / 1.07, 12 0.95 / 0.94
//    (34 million 0.89 / 0.96), 14 0.98 / 0.98 (25 million 0.93 / 1.02); FP64 lx = 5 0.93 / 1.02, 10
//    0.93 / 1.02, at 25 million 1.07 / 1.00, 1.08 / 1.04.
template <int LX, typename T, int NF, bool ADJ>
bool reads_plainly(int64_t n, int words, bool mass, bool keep)
{
    constexpr bool F32 = sizeof(T) == 4;
    const int64_t set = n * (int64_t)sizeof(T) * words, field = n * NF * (int64_t)sizeof(T);
    if (STREAM<LX, T, NF>) return keep && set <= 300000000;
    if (set <= 340000000) return true;
    constexpr bool EVEN12 = F32 && NF == 1 && (LX == 12 || LX == 14);
    if (ADJ && EVEN12) return false;
    if (field > (mass && NF == 1 && !EVEN12 ? (F32 ? 85000000 : 110000000) : 150000000)) return true;
    if (!F32) return LX == 10 && !ADJ && !mass;
    if (NF == 3) return LX == 3 || LX == 5 || LX == 7;
    return mass ? LX % 2 == 1 && LX != 11 && LX != 13 : !EVEN12;
}

template <int LX, typename T, bool KEEP>
__device__ __forceinline__ void load_g(T (&r)[LX], const T *__restrict__ p, bool act)
{
    if (!act) {
#pragma unroll
        for (int k = 0; k < LX; ++k) r[k] = T(0);
        return;
    }
#pragma unroll
    for (int k = 0; k < LX; ++k) r[k] = KEEP ? p[k * LX * LX] : __builtin_nontemporal_load(p + k * LX * LX);
}

template <int LX, typename T>
__device__ __forceinline__ void store_row(T *__restrict__ p, const T (&r)[LX], bool act)
{
    if (act) {
#pragma unroll
        for (int k = 0; k < LX; ++k) p[k * LX * LX] = r[k];
    }
}

// Helmholtz coefficients of one pencil.  GEN = false is the Poisson-type case
// (h1 a scalar, no mass term): nothing per point is held, which keeps the
// register footprint low; GEN = true handles h1 / h2 fields and the mass term.
template <int LX, typename T, bool GEN>
struct RowCoef {
    T h1[GEN ? LX : 1];
    T h2b[GEN ? LX : 1];  // h2 * B
    bool mass = false;
};

template <int LX, typename T, bool GEN, typename Args>
__device__ __forceinline__ void load_coef(RowCoef<LX, T, GEN> &c, const Args &A, int64_t row, bool act)
{
    if constexpr (GEN) {
        if (A.h1) load_row<LX, T>(c.h1, A.h1 + row, act);
        else {
#pragma unroll
            for (int i = 0; i < LX; ++i) c.h1[i] = A.h1s;
        }
        c.mass = A.h2 != nullptr || A.h2s != T(0);
        if (c.mass) {
            load_row<LX, T>(c.h2b, A.B + row, act);
            if (A.h2) {
                T h2[LX];
                load_row<LX, T>(h2, A.h2 + row, act);
#pragma unroll
                for (int i = 0; i < LX; ++i) c.h2b[i] *= h2[i];
            } else {
#pragma unroll
                for (int i = 0; i < LX; ++i) c.h2b[i] *= A.h2s;
            }
        }
    }
}

// Apply h1 * G at every point of the pencil (in place: ur,us,ut -> wr,ws,wt).
template <int LX, typename T, bool GEN>
__device__ __forceinline__ void apply_G(const T (&g)[6][LX], const RowCoef<LX, T, GEN> &c, T h1s,
                                        T (&ur)[LX], T (&us)[LX], T (&ut)[LX])
{
#pragma unroll
    for (int i = 0; i < LX; ++i) {
        const T h = GEN ? c.h1[i] : h1s;
        const T r = ur[i], s = us[i], t = ut[i];
        ur[i] = h * (g[0][i] * r + g[3][i] * s + g[4][i] * t);
        us[i] = h * (g[3][i] * r + g[1][i] * s + g[5][i] * t);
        ut[i] = h * (g[4][i] * r + g[5][i] * s + g[2][i] * t);
    }
}

// w += h2 B u (general case only).
template <int LX, typename T, bool GEN>
__device__ __forceinline__ void add_mass(const RowCoef<LX, T, GEN> &c, const T (&u)[LX], T (&w)[LX])
{
    if constexpr (GEN) {
        if (c.mass) {
#pragma unroll
            for (int i = 0; i < LX; ++i) w[i] = fma(c.h2b[i], u[i], w[i]);
        }
    }
}

// ------------------------------------------------------------------ w = A_L u
// NF fields share one read of G (and B, h1, h2).
template <int LX, typename T, int NF, bool GEN, bool KEEP>
__global__ SEM_BOUNDS2((Shape<LX, T>::NT), (Shape<LX, T>::MINW)) void k_ax_helm(AxArgs<T> A, DEo<LX, T> D)
{
    using S = Shape<LX, T>;
    __shared__ Lds<LX, T> lds;
    const int tid = threadIdx.x;
    const int slot = tid / S::NP;
    const int t = tid - slot * S::NP;
    const int a = t % LX, b = t / LX;
    const int64_t e = (int64_t)blockIdx.x * S::EPB + slot;
    const bool act = e < A.nelv;
    const int64_t row = e * (int64_t)(LX * LX * LX) + t;  // base of this lane's t-pencil
    T *s0 = lds.buf[0][slot], *s1 = lds.buf[1][slot];

    T g[6][LX];
#pragma unroll
    for (int f = 0; f < 6; ++f) load_g<LX, T, KEEP>(g[f], A.G + f * A.n + row, act);
    RowCoef<LX, T, GEN> c;
    load_coef<LX, T, GEN>(c, A, row, act);
    // the next field's row is loaded while the current one is processed
    T un[LX];
    load_row<LX, T>(un, A.u + row, act);
#pragma unroll 1
    for (int f = 0; f < NF; ++f) {
        T u[LX];
#pragma unroll
        for (int k = 0; k < LX; ++k) u[k] = un[k];
        if (f + 1 < NF) load_row<LX, T>(un, A.u + (f + 1) * A.n + row, act);
        T ur[LX], us[LX], ut[LX];
        grad<LX, T>(D, u, s0, s1, a, b, ur, us, ut);
        apply_G<LX, T, GEN>(g, c, A.h1s, ur, us, ut);
        T w[LX];
        div<LX, T>(D, ur, us, ut, s0, s1, a, b, w);
        add_mass<LX, T, GEN>(c, u, w);
        store_row<LX, T>(A.w + f * A.n + row, w, act);
    }
}

// ------------------------------------------------------------------ fused CG matvec
// Two-reduction CG (CG1 = false): p = dinv r + beta p (stored), w = A_L p.
// Single-reduction CG (CG1 = true, Chronopoulos-Gear): u = dinv r (not stored),
// w = A_L u.  Either way the workgroup's partial sum of v . w (v = p or u) is written:
// v^T A v by the unassembled identity of Eq. 10.
template <int LX, typename T, int NF, bool GEN, bool CG1, bool KEEP, bool FOLD>
__global__ SEM_BOUNDS2((Shape<LX, T>::NT), (Shape<LX, T>::MINW)) void k_cg_matvec(CgMatvecArgs<T> A, DEo<LX, T> D)
{
    using S = Shape<LX, T>;
    static_assert(S::NT >= 64, "the partial-sum reduction needs a full first wave");
    __shared__ Lds<LX, T> lds;
    __shared__ double red[NF][S::NT];
    const int tid = threadIdx.x;
    const int slot = tid / S::NP;
    const int t = tid - slot * S::NP;
    const int a = t % LX, b = t / LX;
    const int64_t e = (int64_t)blockIdx.x * S::EPB + slot;
    const bool act = e < A.nelv;
    const int64_t row = e * (int64_t)(LX * LX * LX) + t;  // base of this lane's t-pencil
    T *s0 = lds.buf[0][slot], *s1 = lds.buf[1][slot];
    // a launch queued after every field has stopped (between host polls) reads
    // nothing: the same flags for every lane, so the exit is uniform
    bool live = false;
#pragma unroll
    for (int f = 0; f < NF; ++f) live = live || !A.scal[f].stop;
    if (!live) {
        if (FOLD && blockIdx.x == 0 && tid == 0) *A.scal_out = *A.scal;
        return;
    }

    T g[6][LX];
#pragma unroll
    for (int f = 0; f < 6; ++f) load_g<LX, T, KEEP>(g[f], A.G + f * A.n + row, act);
    RowCoef<LX, T, GEN> c;
    load_coef<LX, T, GEN>(c, A, row, act);
    T dinv[LX];
    // the CG vectors too are streamed with non-temporal hints, unless KEEP: one iteration
    // moves several times the last-level cache, and keeping them out of it leaves room for
    // the gather-scatter's index lists and w, which the next kernel reads (measured:
    // 0.763 -> 0.687 s per FP64 solve at 32^3 x lx=8)
    load_g<LX, T, KEEP>(dinv, A.dinv + row, act);

    // FOLD: the end of the previous iteration, by every workgroup for itself, while G is on
    // its way (the sums of k_cg_finish, in its order); the first one hands the state on.  It
    // takes out a launch, 3.5 us of dependent accesses: 6^3 points in 64 elements 15.8 -> 13.7 us
    // per iteration, in 512 15.9 -> 15.0.  With three fields it is slower, 21.1 -> 22.0 and 25.4 ->
    // 26.8, where the three ends come one after the other.
    static_assert(!FOLD || NF == 1, "one field");
    __shared__ double fsum[FOLD ? 8 : 1], fbeta;
    __shared__ int fstop;
    if constexpr (FOLD) {
        const int lane = tid & 63, wave = tid >> 6;
        constexpr int NW = S::NT / 64;  // whole waves
        if (wave < NW) {
            for (int h = wave; h < 8; h += NW) {  // four chunks of 64 of each of the two sums
                const int q = (h & 3) * 64 + lane;
                const double v = wave_sum(q < A.nup ? A.upart[(h >> 2) * A.nup + q] : 0.0);
                if (lane == 0) fsum[h] = v;
            }
        }
        __syncthreads();
        if (tid == 0) {
            CgScalars sc = *A.scal;
            if (!sc.stop && sc.primed)
                cg_end_iteration(sc, ((fsum[0] + fsum[1]) + fsum[2]) + fsum[3], ((fsum[4] + fsum[5]) + fsum[6]) + fsum[7]);
            fbeta = sc.beta;
            fstop = sc.stop;
            if (blockIdx.x == 0) {
                sc.primed = 0;
                *A.scal_out = sc;
            }
        }
        __syncthreads();
        if (fstop) return;
    }

    double part[NF];
#pragma unroll 1
    for (int f = 0; f < NF; ++f) {
        part[f] = 0.0;
        const CgScalars *sc = A.scal + f;
        if (!FOLD && sc->stop) continue;  // uniform: every lane reads the same flag
        T r[LX], p[LX];
        load_g<LX, T, KEEP>(r, A.r + f * A.n + row, act);
        if constexpr (CG1) {
#pragma unroll
            for (int i = 0; i < LX; ++i) p[i] = dinv[i] * r[i];
        } else {
            const T beta = (T)(FOLD ? fbeta : sc->beta);
            load_g<LX, T, KEEP>(p, A.p + f * A.n + row, act);
            // (not with FOLD: see cg_iterate)
            if (!FOLD && cg_matvec_takes_x(LX, sizeof(T) == 8, NF) && A.x && sc->pend) {
                const T alpha = (T)sc->alpha;
                T *xp = A.x + f * A.n + row, x[LX];
                load_g<LX, T, KEEP>(x, xp, act);
                if (act) {
#pragma unroll
                    for (int k = 0; k < LX; ++k) {
                        const T v = fma(alpha, p[k], x[k]);
                        if constexpr (KEEP) xp[k * LX * LX] = v;
                        else __builtin_nontemporal_store(v, xp + k * LX * LX);
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < LX; ++i) p[i] = fma(beta, p[i], dinv[i] * r[i]);
            if (act) {
#pragma unroll
                for (int k = 0; k < LX; ++k) {
                    T *q = A.p + f * A.n + row + k * LX * LX;
                    if constexpr (KEEP) *q = p[k];
                    else __builtin_nontemporal_store(p[k], q);
                }
            }
        }
        T ur[LX], us[LX], ut[LX];
        grad<LX, T>(D, p, s0, s1, a, b, ur, us, ut);
        apply_G<LX, T, GEN>(g, c, A.h1s, ur, us, ut);
        T w[LX];
        div<LX, T>(D, ur, us, ut, s0, s1, a, b, w);
        add_mass<LX, T, GEN>(c, p, w);
        store_row<LX, T>(A.w + f * A.n + row, w, act);
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < LX; ++i) s += (double)p[i] * (double)w[i];
        part[f] = s;
    }
    // workgroup reduction in a fixed order (deterministic): the first wave (always
    // full, NT >= 64) sums strided slices, then that wave its lanes.
#pragma unroll
    for (int q = 0; q < NF; ++q) red[q][tid] = part[q];
    __syncthreads();
    if (tid < 64) {
#pragma unroll
        for (int q = 0; q < NF; ++q) {
            double v = 0.0;
            for (int k = tid; k < S::NT; k += 64) v += red[q][k];
            v = wave_sum(v);
            if (tid == 0) A.partial[(int64_t)q * gridDim.x + blockIdx.x] = v;
        }
    }
}

// ------------------------------------------------------------------ register-lean variants
// At large lx a lane's six G pencils (6 lx words) held next to a field's pencils
// exhaust the register file (one wave per SIMD at lx = 12 in FP64), which leaves a
// compute unit one workgroup that alternates between loading and computing.  The
// lean kernels (lx >= SEM_LEAN_LX) hold nothing across the phases of a field: G,
// h1, B and dinv are read in chunks of ceil(lx/2) points where they are used, the r
// and s derivatives run one after the other, and one element is one workgroup.  The
// registers saved let two (FP64) or four (FP32) waves share a SIMD, so the loads of
// one workgroup overlap the arithmetic of others.  With three fields the chunks are
// read again for every field, mostly from memory: those of the elements in flight on an
// XCD do not stay in its L2 (41.7 GB fetched for 15.3 GB needed, three FP64 Helmholtz fields of
// 191 million points at lx = 12).  Where G fits the registers it is held instead (LeanCfg::HOLD,
// and the matrix-core variants below).

template <bool NTL, typename T>
__device__ __forceinline__ T ldx(const T *p)
{
    if constexpr (NTL) return __builtin_nontemporal_load(p);
    else return *p;
}

// Reference-space gradient, the r and s derivatives sequenced to keep one pencil pair
// live at a time.  Same LDS protocol as grad (both buffers, ends synchronised).
template <int LX, typename T, typename DS>
__device__ __forceinline__ void grad_lean(const DS &D, const T (&u)[LX], T *s0, T *s1, int a, int b,
                                          T (&ur)[LX], T (&us)[LX], T (&ut)[LX])
{
#pragma unroll
    for (int k = 0; k < LX; ++k) s0[lidx<LX>(a, b, k)] = u[k];
    D.mul(u, ut);
    esync<LX>();
    {
        T v[LX], q[LX];
#pragma unroll
        for (int l = 0; l < LX; ++l) v[l] = s0[lidx<LX>(l, a, b)];   // r-pencil (j=a, k=b)
        D.mul(v, q);
#pragma unroll
        for (int m = 0; m < LX; ++m) s1[lidx<LX>(m, a, b)] = q[m];
    }
    __builtin_amdgcn_sched_barrier(0);
    {
        T v[LX], q[LX];
#pragma unroll
        for (int l = 0; l < LX; ++l) v[l] = s0[lidx<LX>(a, l, b)];   // s-pencil (i=a, k=b)
        D.mul(v, q);
        esync<LX>();
#pragma unroll
        for (int m = 0; m < LX; ++m) s0[lidx<LX>(a, m, b)] = q[m];
    }
    esync<LX>();
#pragma unroll
    for (int k = 0; k < LX; ++k) {
        ur[k] = s1[lidx<LX>(a, b, k)];
        us[k] = s0[lidx<LX>(a, b, k)];
    }
    esync<LX>();
}

// acc = D_r^T wr + D_s^T ws + D_t^T wt, sequenced as grad_lean.  Ends synchronised.
template <int LX, typename T, typename DS>
__device__ __forceinline__ void div_lean(const DS &D, const T (&wr)[LX], const T (&ws)[LX],
                                         const T (&wt)[LX], T *s0, T *s1, int a, int b, T (&acc)[LX])
{
#pragma unroll
    for (int k = 0; k < LX; ++k) {
        s0[lidx<LX>(a, b, k)] = wr[k];
        s1[lidx<LX>(a, b, k)] = ws[k];
    }
    D.tmul(wt, acc);
    esync<LX>();
    T q[LX], q2[LX];
    {
        T v[LX];
#pragma unroll
        for (int l = 0; l < LX; ++l) v[l] = s0[lidx<LX>(l, a, b)];
        D.tmul(v, q);
    }
    __builtin_amdgcn_sched_barrier(0);
    {
        T v[LX];
#pragma unroll
        for (int l = 0; l < LX; ++l) v[l] = s1[lidx<LX>(a, l, b)];
        D.tmul(v, q2);
    }
    esync<LX>();
#pragma unroll
    for (int m = 0; m < LX; ++m) {
        s0[lidx<LX>(m, a, b)] = q[m];
        s1[lidx<LX>(a, m, b)] = q2[m];
    }
    esync<LX>();
#pragma unroll
    for (int k = 0; k < LX; ++k) acc[k] += s0[lidx<LX>(a, b, k)] + s1[lidx<LX>(a, b, k)];
    esync<LX>();
}

// Four-buffer forms (A, B, C, E: one element each).  The transposes of a field pass
// go through buffers that no lane can still be reading, which takes four workgroup
// barriers per pass instead of eight: grad writes u to A, the r and s derivatives to B
// and C; div writes w_r to A and w_s to E, their transposed derivatives to B and C.
// Every buffer written after a barrier was last read before that barrier, including
// across consecutive passes (the next pass writes B and C only after its first
// barrier, which every lane reaches after its reads of B and C).
template <int LX, typename T, typename DS>
__device__ __forceinline__ void grad4(const DS &D, const T (&u)[LX], T *A, T *B, T *C, int a, int b,
                                      T (&ur)[LX], T (&us)[LX], T (&ut)[LX])
{
#pragma unroll
    for (int k = 0; k < LX; ++k) A[lidx<LX>(a, b, k)] = u[k];
    D.mul(u, ut);
    esync<LX>();
    {
        T v[LX], q[LX];
#pragma unroll
        for (int l = 0; l < LX; ++l) v[l] = A[lidx<LX>(l, a, b)];   // r-pencil (j=a, k=b)
        D.mul(v, q);
#pragma unroll
        for (int m = 0; m < LX; ++m) B[lidx<LX>(m, a, b)] = q[m];
    }
    __builtin_amdgcn_sched_barrier(0);
    {
        T v[LX], q[LX];
#pragma unroll
        for (int l = 0; l < LX; ++l) v[l] = A[lidx<LX>(a, l, b)];   // s-pencil (i=a, k=b)
        D.mul(v, q);
#pragma unroll
        for (int m = 0; m < LX; ++m) C[lidx<LX>(a, m, b)] = q[m];
    }
    esync<LX>();
#pragma unroll
    for (int k = 0; k < LX; ++k) {
        ur[k] = B[lidx<LX>(a, b, k)];
        us[k] = C[lidx<LX>(a, b, k)];
    }
}

template <int LX, typename T, typename DS>
__device__ __forceinline__ void div4(const DS &D, const T (&wr)[LX], const T (&ws)[LX], const T (&wt)[LX], T *A,
                                     T *B, T *C, T *E, int a, int b, T (&acc)[LX])
{
#pragma unroll
    for (int k = 0; k < LX; ++k) {
        A[lidx<LX>(a, b, k)] = wr[k];
        E[lidx<LX>(a, b, k)] = ws[k];
    }
    D.tmul(wt, acc);
    esync<LX>();
    {
        T v[LX], q[LX];
#pragma unroll
        for (int l = 0; l < LX; ++l) v[l] = A[lidx<LX>(l, a, b)];
        D.tmul(v, q);
#pragma unroll
        for (int m = 0; m < LX; ++m) B[lidx<LX>(m, a, b)] = q[m];
    }
    __builtin_amdgcn_sched_barrier(0);
    {
        T v[LX], q[LX];
#pragma unroll
        for (int l = 0; l < LX; ++l) v[l] = E[lidx<LX>(a, l, b)];
        D.tmul(v, q);
#pragma unroll
        for (int m = 0; m < LX; ++m) C[lidx<LX>(a, m, b)] = q[m];
    }
    esync<LX>();
#pragma unroll
    for (int k = 0; k < LX; ++k) acc[k] += B[lidx<LX>(a, b, k)] + C[lidx<LX>(a, b, k)];
}



// Pencil loads and stores of the lean kernels.  eb is the element's base in one plane
// (wave-uniform: one element per workgroup, every workgroup holds an element), t the
// lane's column; the address is a uniform base plus a small per-lane offset, which
// keeps per-lane 64-bit addresses out of the registers.
template <int LX, typename T, bool NTL>
__device__ __forceinline__ void lpencil(T (&r)[LX], const T *__restrict__ eb, unsigned t)
{
#pragma unroll
    for (int k = 0; k < LX; ++k) r[k] = ldx<NTL>(eb + k * LX * LX + t);
}

template <int LX, typename T>
__device__ __forceinline__ void spencil(T *__restrict__ eb, unsigned t, const T (&r)[LX])
{
#pragma unroll
    for (int k = 0; k < LX; ++k) eb[k * LX * LX + t] = r[k];
}

// Coefficient forms of the lean kernels, fixed at compile time so that no pointer test
// or branch sits between the loads and the arithmetic that uses them (a form tested at
// run time spilled up to 159 registers at lx = 12): bit 0, h1 is a field; bits 1-2, the
// mass term: none, h2 a scalar, h2 a field.
constexpr int KPOISSON = 0, KINDS = 6;
constexpr bool kind_h1f(int kind) { return kind & 1; }
constexpr int kind_mass(int kind) { return kind >> 1; }

// h (a x + b y + c z), the order of the products fixed so that every kernel that applies
// G (G in registers or in chunks, one field or three) rounds alike.
template <typename T>
__device__ __forceinline__ T row_G(T h, T a, T x, T b, T y, T c, T z)
{
    return h * fma(c, z, fma(b, y, a * x));
}

// (ur, us, ut) <- h1 G (ur, us, ut) with G (and the h1 field) read in chunks of C
// points, Ge = G + element base (plane stride n).  NTL: non-temporal loads (G used by
// one field only).  The chunks are not requested before the gradient is done.
template <int LX, typename T, int KIND, bool NTL>
__device__ __forceinline__ void apply_G_lean(const T *__restrict__ Ge, const T *__restrict__ h1e, T h1s, int64_t n,
                                             unsigned t, T (&ur)[LX], T (&us)[LX], T (&ut)[LX])
{
    constexpr int C = sizeof(T) == 8 ? (LX + 2) / 3 : (LX + 1) / 2;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k0 = 0; k0 < LX; k0 += C) {
        T g[6][C], h[C];
#pragma unroll
        for (int kk = 0; kk < C; ++kk) {
            if (k0 + kk < LX) {
                const unsigned o = (k0 + kk) * (LX * LX) + t;
#pragma unroll
                for (int f = 0; f < 6; ++f) g[f][kk] = ldx<NTL>(Ge + f * n + o);
                if constexpr (kind_h1f(KIND)) h[kk] = h1e[o];
                else h[kk] = h1s;
            }
        }
#pragma unroll
        for (int kk = 0; kk < C; ++kk) {
            const int k = k0 + kk;
            if (k < LX) {
                const T r = ur[k], s = us[k], q = ut[k];
                ur[k] = row_G(h[kk], g[0][kk], r, g[3][kk], s, g[4][kk], q);
                us[k] = row_G(h[kk], g[3][kk], r, g[1][kk], s, g[5][kk], q);
                ut[k] = row_G(h[kk], g[4][kk], r, g[5][kk], s, g[2][kk], q);
            }
        }
    }
}

// h2 B at the lane's points (forms with a mass term), B and the h2 field read here.
template <int LX, typename T, int KIND>
__device__ __forceinline__ T mass_coef(const T *__restrict__ Be, const T *__restrict__ h2e, T h2s, unsigned o)
{
    if constexpr (kind_mass(KIND) == 2) return h2e[o] * Be[o];
    else return h2s * Be[o];
}

// w += h2 B u for u held in registers.
template <int LX, typename T, int KIND>
__device__ __forceinline__ void add_mass_lean(const T *__restrict__ Be, const T *__restrict__ h2e, T h2s, unsigned t,
                                              const T (&u)[LX], T (&w)[LX])
{
    if constexpr (kind_mass(KIND) != 0) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < LX; ++k) w[k] = fma(mass_coef<LX, T, KIND>(Be, h2e, h2s, k * (LX * LX) + t), u[k], w[k]);
    }
}

// w += h2 B u with u reloaded from ue (read moments before, so served by the cache).
template <int LX, typename T, int KIND>
__device__ __forceinline__ void add_mass_reload(const T *__restrict__ Be, const T *__restrict__ h2e, T h2s, unsigned t,
                                                const T *__restrict__ ue, T (&w)[LX])
{
    if constexpr (kind_mass(KIND) != 0) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < LX; ++k) {
            const unsigned o = k * (LX * LX) + t;
            w[k] = fma(mass_coef<LX, T, KIND>(Be, h2e, h2s, o), ue[o], w[k]);
        }
    }
}

// (ur, us, ut) <- h1 G (ur, us, ut) from G pencils held in registers; an h1 field's values
// at hp[k * lx^2] (the lane's own column).
template <int LX, typename T, int KIND>
__device__ __forceinline__ void apply_G_regs(const T (&g)[6][LX], const T *hp, T h1s, T (&ur)[LX], T (&us)[LX],
                                             T (&ut)[LX])
{
#pragma unroll
    for (int k = 0; k < LX; ++k) {
        T h;
        if constexpr (kind_h1f(KIND)) h = hp[k * (LX * LX)];
        else h = h1s;
        const T r = ur[k], s = us[k], q = ut[k];
        ur[k] = row_G(h, g[0][k], r, g[3][k], s, g[4][k], q);
        us[k] = row_G(h, g[3][k], r, g[1][k], s, g[5][k], q);
        ut[k] = row_G(h, g[4][k], r, g[5][k], s, g[2][k], q);
    }
}

// The gradient and divergence halves of a field pass on NB LDS buffers.
template <int LX, typename T, int NB, typename DS>
__device__ __forceinline__ void grad_nb(const DS &D, const T (&u)[LX], T (*buf)[Shape<LX, T>::ESZ], int a, int b,
                                        T (&ur)[LX], T (&us)[LX], T (&ut)[LX])
{
    if constexpr (NB == 4) grad4<LX, T>(D, u, buf[0], buf[1], buf[2], a, b, ur, us, ut);
    else grad_lean<LX, T>(D, u, buf[0], buf[1], a, b, ur, us, ut);
}

template <int LX, typename T, int NB, typename DS>
__device__ __forceinline__ void div_nb(const DS &D, const T (&wr)[LX], const T (&ws)[LX], const T (&wt)[LX],
                                       T (*buf)[Shape<LX, T>::ESZ], int a, int b, T (&w)[LX])
{
    if constexpr (NB == 4) div4<LX, T>(D, wr, ws, wt, buf[0], buf[1], buf[2], buf[3], a, b, w);
    else div_lean<LX, T>(D, wr, ws, wt, buf[0], buf[1], a, b, w);
}

// Launch configuration of the lean kernels, per precision, field count and kernel
// (CG: the fused CG matvec, which also keeps p for its dot product).
//  * HOLD: with three fields sharing one G, hold G's six pencils in registers (loaded
//    once, non-temporal) instead of reading them in chunks for every field: the L2 does
//    not keep them, so they are read from memory three times otherwise.  It pays where
//    they fit: the FP32 operator up to lx = 12, the FP64 operator at lx = 10 and 11 at two
//    waves per SIMD (three Helmholtz fields, 20 million points: 635 -> 467 us and 676 ->
//    492 us; with h1 and h2 fields 1690 -> 508 and 2000 -> 649 us; FP32 at lx = 12 with
//    h1 and h2 fields 389 -> 294 us).  The FP32 CG matvec, which also holds p, is faster
//    reading chunks (48^3 elements, lx = 12: 4.6 ms held, 3.7 in chunks at the three waves per
//    SIMD that it gets; four are asked for, and 159 to 168 registers leave three).
//  * NB: LDS element buffers, 4 (grad4 / div4: four barriers per field pass) or 2
//    (grad_lean / div_lean: eight); in FP64 four would halve the workgroups a compute
//    unit holds.
//  * minw: waves per SIMD the register allocation is held to.  Three FP64 fields of lx = 13
//    without a mass term need 170 registers unless held to the 168 of three waves: 12.8 million
//    points, Poisson 432 -> 364 us, h1 field 472 -> 402.
template <int LX, typename T, int NF, bool CG>
struct LeanCfg {
    static constexpr bool F32 = sizeof(T) == 4;
    static constexpr bool HOLD = NF > 1 && !CG && LX <= (F32 ? 12 : 11);
    static constexpr int NB = F32 ? 4 : 2;
    static constexpr int minw(int kind)
    {
        if (!CG && NF == 3 && !F32 && LX == 13 && kind_mass(kind) == 0) return 3;
        return HOLD ? (F32 ? 3 : 2) : Shape<LX, T>::MINW;
    }
};

template <int LX, typename T, int NB>
struct LeanBufs {
    T buf[NB][Shape<LX, T>::ESZ];
};

// One element per workgroup; the grid holds exactly nelv workgroups.
template <int LX, typename T, int NF, int KIND, bool KEEP, typename DS>
__device__ __forceinline__ void ax_lean_body(const DS &D, const AxArgs<T> &A)
{
    using S = Shape<LX, T>;
    using C = LeanCfg<LX, T, NF, false>;
    constexpr bool HOLD = C::HOLD;
    constexpr int NB = C::NB;
    static_assert(S::EPB == 1, "one element per workgroup");
    __shared__ LeanBufs<LX, T, NB> lds;
    const unsigned t = threadIdx.x;
    const int a = t % LX, b = t / LX;
    const int64_t e0 = (int64_t)blockIdx.x * (LX * LX * LX);
    const T *Ge = A.G + e0, *Be = A.B + e0;
    const T *h1e = kind_h1f(KIND) ? A.h1 + e0 : nullptr, *h2e = kind_mass(KIND) == 2 ? A.h2 + e0 : nullptr;
    T g[HOLD ? 6 : 1][LX];
    // HOLD: with G in registers, h1 and h2 B of the lane's column wait in LDS (read back by
    // the same lane); read again for every field they would come from memory
    constexpr bool H1F = kind_h1f(KIND), MASS = kind_mass(KIND) != 0;
    __shared__ T park[HOLD && H1F + MASS ? (H1F + MASS) * LX * LX * LX : 1];
    T *hp = park + t, *mp = park + (H1F ? LX * LX * LX : 0) + t;
    if constexpr (HOLD) {
#pragma unroll
        for (int q = 0; q < 6; ++q) lpencil<LX, T, !KEEP>(g[q], Ge + q * A.n, t);
        T v[LX];
        if constexpr (H1F) {
            lpencil<LX, T, !KEEP>(v, h1e, t);
#pragma unroll
            for (int k = 0; k < LX; ++k) hp[k * (LX * LX)] = v[k];
        }
        if constexpr (MASS) {
            lpencil<LX, T, !KEEP>(v, Be, t);
            T v2[LX];
            if constexpr (kind_mass(KIND) == 2) lpencil<LX, T, !KEEP>(v2, h2e, t);
#pragma unroll
            for (int k = 0; k < LX; ++k) mp[k * (LX * LX)] = (kind_mass(KIND) == 2 ? v2[k] : A.h2s) * v[k];
        }
    }
#pragma unroll 1
    for (int f = 0; f < NF; ++f) {
        const int64_t fe = f * A.n + e0;
        T w[LX];
        {
            T ur[LX], us[LX], ut[LX];
            {
                T u[LX];
                lpencil<LX, T, false>(u, A.u + fe, t);
                grad_nb<LX, T, NB>(D, u, lds.buf, a, b, ur, us, ut);
            }
            if constexpr (HOLD) apply_G_regs<LX, T, KIND>(g, hp, A.h1s, ur, us, ut);
            else apply_G_lean<LX, T, KIND, NF == 1 && !KEEP>(fresh(Ge), H1F ? fresh(h1e) : h1e, A.h1s, A.n, t, ur, us, ut);
            div_nb<LX, T, NB>(D, ur, us, ut, lds.buf, a, b, w);
        }
        if constexpr (HOLD && MASS) {
            const T *ue = A.u + fe;
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < LX; ++k) w[k] = fma(mp[k * (LX * LX)], ue[k * (LX * LX) + t], w[k]);
        } else {
            // B and h2 are the same for every field: in FP64, held over the loop they would spill
            constexpr bool AGAIN = NF > 1 && sizeof(T) == 8;
            add_mass_reload<LX, T, KIND>(AGAIN ? fresh(Be) : Be, AGAIN && kind_mass(KIND) == 2 ? fresh(h2e) : h2e, A.h2s,
                                         t, A.u + fe, w);
        }
        spencil<LX, T>(A.w + fe, t, w);
    }
}

// DMem in FP64 (the even-odd D does not fit the scalar registers), DArg in FP32 but for three
// fields at lx = 15, where 112 values, kept over the loop, leave 127 scalars spilled: 11.4 million
// points, Poisson 304 -> 287 us, Helmholtz 394 -> 300, h1 and h2 fields 452 -> 315.
template <int LX, typename T, int NF, int KIND, bool KEEP>
__global__ SEM_BOUNDS2((Shape<LX, T>::NT), (LeanCfg<LX, T, NF, false>::minw(KIND))) void k_ax_helm_lean(
    AxArgs<T> A, DEo<LX, T> D, const DEo<LX, T> *__restrict__ Dg)
{
    if constexpr (sizeof(T) == 8 || (LX == 15 && NF == 3)) ax_lean_body<LX, T, NF, KIND, KEEP>(DMem<LX, T>{Dg}, A);
    else ax_lean_body<LX, T, NF, KIND, KEEP>(DArg<LX, T>{D}, A);
}

template <int LX, typename T, int NF, int KIND, bool CG1, typename DS>
__device__ __forceinline__ void cg_lean_body(const DS &D, const CgMatvecArgs<T> &A)
{
    using S = Shape<LX, T>;
    using C = LeanCfg<LX, T, NF, true>;
    static_assert(S::EPB == 1 && S::NT >= 64, "one element per workgroup of at least one wave");
    constexpr int NB = C::NB;
    __shared__ LeanBufs<LX, T, NB> lds;
    __shared__ double red[NF][S::NT];
    const unsigned t = threadIdx.x;
    const int a = t % LX, b = t / LX;
    const int64_t e0 = (int64_t)blockIdx.x * (LX * LX * LX);
    bool live = false;
#pragma unroll
    for (int f = 0; f < NF; ++f) live = live || !A.scal[f].stop;
    if (!live) return;
    const T *Ge = A.G + e0;
    const T *h1e = kind_h1f(KIND) ? A.h1 + e0 : nullptr;
    double part[NF];
#pragma unroll 1
    for (int f = 0; f < NF; ++f) {
        part[f] = 0.0;
        const CgScalars *sc = A.scal + f;
        if (sc->stop) continue;  // uniform
        const int64_t fe = f * A.n + e0;
        T p[LX];
        {
            T r[LX], dv[LX];
            lpencil<LX, T, true>(r, A.r + fe, t);
            lpencil<LX, T, NF == 1>(dv, A.dinv + e0, t);
            if constexpr (CG1) {
#pragma unroll
                for (int i = 0; i < LX; ++i) p[i] = dv[i] * r[i];
            } else {
                const T beta = (T)sc->beta;
                lpencil<LX, T, true>(p, A.p + fe, t);
                if (cg_matvec_takes_x(LX, sizeof(T) == 8, NF) && A.x && sc->pend) {
                    const T alpha = (T)sc->alpha;
                    T x[LX];
                    lpencil<LX, T, true>(x, A.x + fe, t);
#pragma unroll
                    for (int k = 0; k < LX; ++k)
                        __builtin_nontemporal_store(fma(alpha, p[k], x[k]), A.x + fe + k * LX * LX + t);
                }
#pragma unroll
                for (int i = 0; i < LX; ++i) p[i] = fma(beta, p[i], dv[i] * r[i]);
#pragma unroll
                for (int k = 0; k < LX; ++k) __builtin_nontemporal_store(p[k], A.p + fe + k * LX * LX + t);
            }
        }
        T w[LX];
        {
            T ur[LX], us[LX], ut[LX];
            grad_nb<LX, T, NB>(D, p, lds.buf, a, b, ur, us, ut);
            apply_G_lean<LX, T, KIND, NF == 1>(fresh(Ge), kind_h1f(KIND) ? fresh(h1e) : h1e, A.h1s, A.n, t, ur, us, ut);
            div_nb<LX, T, NB>(D, ur, us, ut, lds.buf, a, b, w);
        }
        const T *Be = A.B + e0, *h2e = kind_mass(KIND) == 2 ? A.h2 + e0 : nullptr;
        constexpr bool REUSE = NF > 1 && sizeof(T) == 8;  // as in ax_lean_body
        add_mass_lean<LX, T, KIND>(REUSE ? fresh(Be) : Be, REUSE && kind_mass(KIND) == 2 ? fresh(h2e) : h2e, A.h2s, t,
                                   p, w);
        spencil<LX, T>(A.w + fe, t, w);
        double sum = 0.0;
#pragma unroll
        for (int i = 0; i < LX; ++i) sum += (double)p[i] * (double)w[i];
        part[f] = sum;
    }
#pragma unroll
    for (int q = 0; q < NF; ++q) red[q][t] = part[q];
    __syncthreads();
    if (t < 64) {
#pragma unroll
        for (int q = 0; q < NF; ++q) {
            double v = 0.0;
            for (unsigned k = t; k < S::NT; k += 64) v += red[q][k];
            v = wave_sum(v);
            if (t == 0) A.partial[(int64_t)q * gridDim.x + blockIdx.x] = v;
        }
    }
}

template <int LX, typename T, int NF, int KIND, bool CG1>
__global__ SEM_BOUNDS2((Shape<LX, T>::NT), (LeanCfg<LX, T, NF, true>::minw(KIND))) void k_cg_matvec_lean(
    CgMatvecArgs<T> A, DEo<LX, T> D, const DEo<LX, T> *__restrict__ Dg)
{
    if constexpr (sizeof(T) == 8) cg_lean_body<LX, T, NF, KIND, CG1>(DMem<LX, T>{Dg}, A);
    else cg_lean_body<LX, T, NF, KIND, CG1>(DArg<LX, T>{D}, A);
}

// ------------------------------------------------------------------ matrix-core variants
// One element per workgroup, its points spread over W waves in tiles of 16 pencils: lane
// c + 16 g of a wave holds rows 4 t + g (t = 0 .. ceil(lx/4) - 1) of pencil c of each of
// its tiles, and a derivative along the pencils is a matrix product D x on the matrix
// cores whose result has the operand's layout (see Mat).  A lane holds lx^3 / (64 W)
// points instead of a whole pencil, so the six geometric factors of all of them fit
// its registers next to a field's derivatives, and with three fields G is read from
// memory once.
//
// Field pass (three LDS element buffers, four barriers): u in the t layout goes to A;
// A's r and s pencils are differentiated into B and C; every lane reads the r and s
// derivatives of its own points back from B and C, applies h1 G and writes w_r, w_s to the
// same places; B's r pencils and C's s pencils are multiplied with D^T in place (a tile's
// pencils belong to one wave), and every lane adds the two at its points to D^T w_t.  A
// buffer is written again only after a barrier that follows its last read.
//
// Matrix operand of D or D^T for the tile product.  FP64: 4x4x4 products of four
// blocks with the same matrix tile (A: row lane % 4, column g; B, C: row g, pencil c).
// FP32: 16x16x4 products (A: row lane % 16, column g; B: row g; C register r: row
// 4 g + r); with the matrix rows permuted so that A's row q holds row 4 (q % 4) + q / 4,
// C register r is row 4 r + g, the operand layout.
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <int LX, typename T>
struct Mat;

template <int LX>
struct Mat<LX, double> {
    static constexpr int N = (LX + 3) / 4;
    double m[N][N];
    // D row-major in memory; tr: the transpose
    __device__ __forceinline__ void load(const double *__restrict__ D, bool tr)
    {
        const int i = threadIdx.x & 3, k = (threadIdx.x >> 4) & 3;
#pragma unroll
        for (int a = 0; a < N; ++a)
#pragma unroll
            for (int b = 0; b < N; ++b) {
                const int row = 4 * a + i, col = 4 * b + k;
                const bool in = (4 * a + 3 < LX || row < LX) && (4 * b + 3 < LX || col < LX);
                m[a][b] = in ? D[tr ? col * LX + row : row * LX + col] : 0.0;
            }
    }
    __device__ __forceinline__ void mul(const double (&x)[N], double (&y)[N]) const
    {
#pragma unroll
        for (int b = 0; b < N; ++b)
#pragma unroll
            for (int a = 0; a < N; ++a)
                y[a] = __builtin_amdgcn_mfma_f64_4x4x4f64(m[a][b], x[b], b ? y[a] : 0.0, 0, 0, 0);
    }
};

template <int LX>
struct Mat<LX, float> {
    static constexpr int N = (LX + 3) / 4;
    float m[N];
    __device__ __forceinline__ void load(const float *__restrict__ D, bool tr)
    {
        const int q = threadIdx.x & 15, k = (threadIdx.x >> 4) & 3, row = 4 * (q & 3) + (q >> 2);
#pragma unroll
        for (int b = 0; b < N; ++b) {
            const int col = 4 * b + k;
            m[b] = row < LX && col < LX ? D[tr ? col * LX + row : row * LX + col] : 0.0f;
        }
    }
    __device__ __forceinline__ void mul(const float (&x)[N], float (&y)[N]) const
    {
        f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int b = 0; b < N; ++b) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(m[b], x[b], acc, 0, 0, 0);
#pragma unroll
        for (int a = 0; a < N; ++a) y[a] = acc[a];
    }
};

template <int LX, typename T, int W>
struct Tiles {
    static constexpr int L2 = LX * LX, NTILE = (L2 + 15) / 16;
    static constexpr int H = (NTILE + W - 1) / W;       // tiles per wave
    static constexpr int R = (LX + 3) / 4;              // rows per lane and tile
    static constexpr int P = (LX % 2) ? LX : LX + 1;    // LDS row stride
    static constexpr int ESZ = L2 * P;
    int wave, c, g;
    int p[H], pi[H], pj[H];  // pencil of tile h (clamped) and its two coordinates, p = pi + lx pj
    __device__ __forceinline__ Tiles()
    {
        wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        c = threadIdx.x & 15;
        g = (threadIdx.x >> 4) & 3;
#pragma unroll
        for (int h = 0; h < H; ++h) {
            const int q = 16 * (wave + W * h) + c;
            p[h] = 16 * W * (h + 1) <= L2 ? q : (q < L2 ? q : L2 - 1);
            pj[h] = p[h] / LX;
            pi[h] = p[h] - LX * pj[h];
        }
    }
    // tile h of this lane is a pencil of the element (a clamped lane is not)
    __device__ __forceinline__ bool own(int h) const
    {
        return 16 * W * (h + 1) <= L2 || 16 * (wave + W * h) + c < L2;
    }
    __device__ __forceinline__ bool row(int t) const { return 4 * t + 3 < LX || 4 * t + g < LX; }
    // LDS places of row 0 of the lane's t, r and s pencils and the strides of the rows
    __device__ __forceinline__ int at_t(int h) const { return pi[h] + P * pj[h]; }
    __device__ __forceinline__ int at_r(int h) const { return P * p[h]; }
    __device__ __forceinline__ int at_s(int h) const { return pi[h] + P * LX * pj[h]; }
    static constexpr int ST = P * LX, SR = 1, SS = P;
    template <int STRIDE>
    __device__ __forceinline__ void get(const T *b, T (&x)[R]) const
    {
#pragma unroll
        for (int t = 0; t < R; ++t) x[t] = row(t) ? b[(4 * t + g) * STRIDE] : T(0);
    }
    template <int STRIDE>
    __device__ __forceinline__ void put(T *b, int h, const T (&x)[R]) const
    {
        if (!own(h)) return;
#pragma unroll
        for (int t = 0; t < R; ++t)
            if (row(t)) b[(4 * t + g) * STRIDE] = x[t];
    }
    // the lane's points of one field or plane; eb: element base (wave-uniform)
    template <bool NTL>
    __device__ __forceinline__ void load(const T *__restrict__ eb, T (&x)[H][R]) const
    {
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int t = 0; t < R; ++t) x[h][t] = row(t) ? ldx<NTL>(eb + ((4 * t + g) * L2 + p[h])) : T(0);
    }
    template <bool NTS>
    __device__ __forceinline__ void store(T *__restrict__ eb, const T (&x)[H][R]) const
    {
#pragma unroll
        for (int h = 0; h < H; ++h)
            if (own(h)) {
#pragma unroll
                for (int t = 0; t < R; ++t)
                    if (row(t)) {
                        T *q = eb + ((4 * t + g) * L2 + p[h]);
                        if constexpr (NTS) __builtin_nontemporal_store(x[h][t], q);
                        else *q = x[h][t];
                    }
            }
    }
};

// The wave's pencils along r or s (at(h): row 0 of the lane's pencil of tile h) from buffer
// X through D into buffer Y; X may be Y.
template <int STRIDE, int LX, typename T, int W, typename TL, typename At>
__device__ __forceinline__ void tile_pass(const TL &L, const Mat<LX, T> &D, const T *X, T *Y, At at)
{
    T x[TL::H][TL::R];
#pragma unroll
    for (int h = 0; h < TL::H; ++h) L.template get<STRIDE>(X + at(h), x[h]);
#pragma unroll
    for (int h = 0; h < TL::H; ++h) {
        T v[TL::R];
        D.mul(x[h], v);
        L.template put<STRIDE>(Y + at(h), h, v);
    }
}

// (ur, us, ut) <- gradient of u at the lane's points; buffers A, B, C.
template <int LX, typename T, int W, typename TL>
__device__ __forceinline__ void tile_grad(const TL &L, const Mat<LX, T> &D, const T (&u)[TL::H][TL::R], T *A, T *B, T *C,
                                          T (&ur)[TL::H][TL::R], T (&us)[TL::H][TL::R], T (&ut)[TL::H][TL::R])
{
    constexpr int H = TL::H, R = TL::R;
#pragma unroll
    for (int h = 0; h < H; ++h) L.template put<TL::ST>(A + L.at_t(h), h, u[h]);
#pragma unroll
    for (int h = 0; h < H; ++h) D.mul(u[h], ut[h]);
    __syncthreads();
    tile_pass<TL::SR, LX, T, W>(L, D, A, B, [&](int h) { return L.at_r(h); });
    __builtin_amdgcn_sched_barrier(0);
    tile_pass<TL::SS, LX, T, W>(L, D, A, C, [&](int h) { return L.at_s(h); });
    __syncthreads();
#pragma unroll
    for (int h = 0; h < H; ++h) {
        L.template get<TL::ST>(B + L.at_t(h), ur[h]);
        L.template get<TL::ST>(C + L.at_t(h), us[h]);
    }
}

// w = D_r^T wr + D_s^T ws + D_t^T wt; wr and ws go through B and C in place.
template <int LX, typename T, int W, typename TL>
__device__ __forceinline__ void tile_div(const TL &L, const Mat<LX, T> &Dt, const T (&wr)[TL::H][TL::R],
                                         const T (&ws)[TL::H][TL::R], const T (&wt)[TL::H][TL::R], T *B, T *C,
                                         T (&w)[TL::H][TL::R])
{
    constexpr int H = TL::H, R = TL::R;
#pragma unroll
    for (int h = 0; h < H; ++h) {
        L.template put<TL::ST>(B + L.at_t(h), h, wr[h]);
        L.template put<TL::ST>(C + L.at_t(h), h, ws[h]);
    }
#pragma unroll
    for (int h = 0; h < H; ++h) Dt.mul(wt[h], w[h]);
    __syncthreads();
    tile_pass<TL::SR, LX, T, W>(L, Dt, B, B, [&](int h) { return L.at_r(h); });
    __builtin_amdgcn_sched_barrier(0);
    tile_pass<TL::SS, LX, T, W>(L, Dt, C, C, [&](int h) { return L.at_s(h); });
    __syncthreads();
#pragma unroll
    for (int h = 0; h < H; ++h) {
        T a[R], b[R];
        L.template get<TL::ST>(B + L.at_t(h), a);
        L.template get<TL::ST>(C + L.at_t(h), b);
#pragma unroll
        for (int t = 0; t < R; ++t) w[h][t] += a[t] + b[t];
    }
}

// Where the matrix-core kernels are used, waves per element W and waves per SIMD EU.
//  * FP64, lx = 12: 12^2 pencils are nine whole tiles of three whole rows, three tiles to a
//    wave, and a lane's 9 points of G are 108 of its 256 registers.  Curved elements, 21
//    million points, us with the pencil kernels -> with these: one field Poisson 260 -> 252,
//    Helmholtz 297 -> 272, h1 field 321 -> 299, h1 and h2 fields 544 -> 335; three fields
//    Helmholtz 714 -> 524 (G was read from memory three times, at 6.8 TB/s), h1 and h2
//    fields 2600 -> 553.
//  * FP32, lx = 16, three fields: sixteen whole tiles of four rows; 558 -> 262 us.
// Elsewhere the pencil kernels are faster: the padding of a tile (lx = 10: 16 pencils by 12
// rows for 14.3 by 10) costs up to half of the lanes (467 against 690 us for three fields
// at lx = 10, 330 against 250 us for one), FP64 G at lx = 16 does not fit (670 us either
// way), and in FP32 at lx = 12 the pencil kernels hold G too (243 against 266 us).
template <int LX, typename T, int NF, bool CG>
struct TileCfg {
    static constexpr bool F64 = sizeof(T) == 8;
    static constexpr bool USE = F64 ? LX == 12 : LX == 16 && NF == 3 && !CG;
    static constexpr int W = F64 ? 3 : 8;
    static constexpr int EU = 2;
};

// w = A_L u for NF fields (args AxArgs), or with CG the fused matvecs of k_cg_matvec
// (CgMatvecArgs): p = dinv r + beta p stored, w = A_L p, partial sums of p.w; CG1: the
// same of u = dinv r.
template <int LX, typename T, int NF, int KIND, bool CG, bool CG1, typename Args>
__device__ __forceinline__ void tile_body(const Args &A, const T *__restrict__ Dm)
{
    constexpr int W = TileCfg<LX, T, NF, CG>::W;
    using TL = Tiles<LX, T, W>;
    constexpr int H = TL::H, R = TL::R;
    __shared__ T buf[3][TL::ESZ];
    __shared__ double red[CG ? NF : 1][W];
    if constexpr (CG) {
        bool live = false;
#pragma unroll
        for (int f = 0; f < NF; ++f) live = live || !A.scal[f].stop;
        if (!live) return;
    }
    const TL L;
    const int64_t e0 = (int64_t)blockIdx.x * (LX * LX * LX);
    T u[H][R];
    if constexpr (!CG) L.template load<false>(A.u + e0, u);
    T G[6][H][R];
#pragma unroll
    for (int q = 0; q < 6; ++q) L.template load<CG || STREAM<LX, T, NF>>(A.G + q * A.n + e0, G[q]);
    // h1 and h2 B at the lane's points: with several fields in LDS (each lane reads back
    // its own values), since next to G they do not fit the registers
    constexpr bool H1F = kind_h1f(KIND), MASS = kind_mass(KIND) != 0, PARK = NF > 1;
    __shared__ T park[PARK && H1F + MASS ? H1F + MASS : 1][PARK ? H * R : 1][PARK && H1F + MASS ? 64 * W : 1];
    T h1[H1F && !PARK ? H : 1][R], mb[MASS && !PARK ? H : 1][R];
    if constexpr (H1F) {
        T v[H][R];
        L.template load<PARK && (CG || STREAM<LX, T, NF>)>(A.h1 + e0, v);
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int t = 0; t < R; ++t) {
                if constexpr (PARK) park[0][h * R + t][threadIdx.x] = v[h][t];
                else h1[h][t] = v[h][t];
            }
    }
    if constexpr (MASS) {
        T v[H][R], m2[H][R];
        L.template load<PARK && (CG || STREAM<LX, T, NF>)>(A.B + e0, v);
        if constexpr (kind_mass(KIND) == 2) L.template load<PARK && (CG || STREAM<LX, T, NF>)>(A.h2 + e0, m2);
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int t = 0; t < R; ++t) {
                const T m = v[h][t] * (kind_mass(KIND) == 2 ? m2[h][t] : A.h2s);
                if constexpr (PARK) park[H1F][h * R + t][threadIdx.x] = m;
                else mb[h][t] = m;
            }
    }
#pragma unroll 1
    for (int f = 0; f < NF; ++f) {
        const int64_t fe = f * A.n + e0;
        if constexpr (CG) {
            if (L.c + 16 * L.g == 0) red[f][L.wave] = 0.0;
            if (A.scal[f].stop) continue;  // uniform: every lane reads the same flag
            T r[H][R], dv[H][R];
            L.template load<true>(A.r + fe, r);
            L.template load<NF == 1>(A.dinv + e0, dv);
            if constexpr (CG1) {
#pragma unroll
                for (int h = 0; h < H; ++h)
#pragma unroll
                    for (int t = 0; t < R; ++t) u[h][t] = dv[h][t] * r[h][t];
            } else {
                const T beta = (T)A.scal[f].beta;
                L.template load<true>(A.p + fe, u);
                if constexpr (cg_matvec_takes_x(LX, sizeof(T) == 8, NF)) {
                    if (A.x && A.scal[f].pend) {
                        const T alpha = (T)A.scal[f].alpha;
                        T x[H][R];
                        L.template load<true>(A.x + fe, x);
#pragma unroll
                        for (int h = 0; h < H; ++h)
#pragma unroll
                            for (int t = 0; t < R; ++t) x[h][t] = fma(alpha, u[h][t], x[h][t]);
                        L.template store<true>(A.x + fe, x);
                    }
                }
#pragma unroll
                for (int h = 0; h < H; ++h)
#pragma unroll
                    for (int t = 0; t < R; ++t) u[h][t] = fma(beta, u[h][t], dv[h][t] * r[h][t]);
                L.template store<true>(A.p + fe, u);
            }
        }
        T ur[H][R], us[H][R], ut[H][R], w[H][R];
        Mat<LX, T> D;
        D.load(fresh(Dm), false);
        tile_grad<LX, T, W>(L, D, u, buf[0], buf[1], buf[2], ur, us, ut);
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int t = 0; t < R; ++t) {
                T hv;
                if constexpr (H1F && PARK) hv = park[0][h * R + t][threadIdx.x];
                else if constexpr (H1F) hv = h1[h][t];
                else hv = A.h1s;
                const T r = ur[h][t], s = us[h][t], q = ut[h][t];
                ur[h][t] = row_G(hv, G[0][h][t], r, G[3][h][t], s, G[4][h][t], q);
                us[h][t] = row_G(hv, G[3][h][t], r, G[1][h][t], s, G[5][h][t], q);
                ut[h][t] = row_G(hv, G[4][h][t], r, G[5][h][t], s, G[2][h][t], q);
            }
        Mat<LX, T> Dt;
        Dt.load(fresh(Dm), true);
        tile_div<LX, T, W>(L, Dt, ur, us, ut, buf[1], buf[2], w);
        double dot = 0.0;
        if constexpr (MASS || CG) {
#pragma unroll
            for (int h = 0; h < H; ++h) {
                // (u again from A, where it lies until the next field is written)
                T v[R];
                L.template get<TL::ST>(buf[0] + L.at_t(h), v);
#pragma unroll
                for (int t = 0; t < R; ++t) {
                    if constexpr (MASS && PARK) w[h][t] = fma(park[H1F][h * R + t][threadIdx.x], v[t], w[h][t]);
                    else if constexpr (MASS) w[h][t] = fma(mb[h][t], v[t], w[h][t]);
                    if constexpr (CG)
                        if (L.own(h) && L.row(t)) dot += (double)v[t] * (double)w[h][t];
                }
            }
        }
        if constexpr (!CG)
            if (f + 1 < NF) L.template load<false>(A.u + fe + A.n, u);
        L.template store<false>(A.w + fe, w);
        if constexpr (CG) {
            dot = wave_sum(dot);
            if (L.c + 16 * L.g == 0) red[f][L.wave] = dot;
        }
    }
    if constexpr (CG) {
        // workgroup sums, the waves in order (a stopped field's slots are zero)
        __syncthreads();
        if (threadIdx.x < NF) {
            double v = 0.0;
#pragma unroll
            for (int q = 0; q < W; ++q) v += red[threadIdx.x][q];
            A.partial[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = v;
        }
    }
}

template <int LX, typename T, int NF, int KIND>
__global__ __launch_bounds__((64 * TileCfg<LX, T, NF, false>::W)) __attribute__((amdgpu_waves_per_eu(
    TileCfg<LX, T, NF, false>::EU))) void k_ax_helm_tile(AxArgs<T> A, const T *__restrict__ Dm)
{
    tile_body<LX, T, NF, KIND, false, false>(A, Dm);
}

template <int LX, typename T, int NF, int KIND, bool CG1>
__global__ __launch_bounds__((64 * TileCfg<LX, T, NF, true>::W)) __attribute__((amdgpu_waves_per_eu(
    TileCfg<LX, T, NF, true>::EU))) void k_cg_matvec_tile(CgMatvecArgs<T> A, const T *__restrict__ Dm)
{
    tile_body<LX, T, NF, KIND, true, CG1>(A, Dm);
}

// g = (D v)^T G (D u) per point, lean form: G (D u) is formed first (G read in
// chunks), then the gradient of v is taken and contracted with it.
template <int LX, typename T, bool KEEP, typename DS>
__device__ __forceinline__ void adj_lean_body(const DS &D, const AdjArgs<T> &A)
{
    using S = Shape<LX, T>;
    static_assert(S::EPB == 1, "one element per workgroup");
    __shared__ Lds<LX, T> lds;
    const unsigned t = threadIdx.x;
    const int a = t % LX, b = t / LX;
    const int64_t e0 = (int64_t)blockIdx.x * (LX * LX * LX);
    T *s0 = lds.buf[0][0], *s1 = lds.buf[1][0];
    T wr[LX], ws[LX], wt[LX];
    {
        T u[LX];
        lpencil<LX, T, false>(u, A.u + e0, t);
        grad_lean<LX, T>(D, u, s0, s1, a, b, wr, ws, wt);
    }
    apply_G_lean<LX, T, KPOISSON, !KEEP>(fresh(A.G + e0), (const T *)nullptr, T(1), A.n, t, wr, ws, wt);
    T vr[LX], vs[LX], vt[LX];
    {
        T v[LX];
        lpencil<LX, T, false>(v, A.v + e0, t);
        grad_lean<LX, T>(D, v, s0, s1, a, b, vr, vs, vt);
    }
    T out[LX];
#pragma unroll
    for (int i = 0; i < LX; ++i) out[i] = vr[i] * wr[i] + vs[i] * ws[i] + vt[i] * wt[i];
    spencil<LX, T>(A.g + e0, t, out);
}

template <int LX, typename T, bool KEEP>
__global__ SEM_BOUNDS2((Shape<LX, T>::NT), (Shape<LX, T>::MINW)) void k_ax_adjoint_lean(
    AdjArgs<T> A, DEo<LX, T> D, const DEo<LX, T> *__restrict__ Dg)
{
    if constexpr (sizeof(T) == 8) adj_lean_body<LX, T, KEEP>(DMem<LX, T>{Dg}, A);
    else adj_lean_body<LX, T, KEEP>(DArg<LX, T>{D}, A);
}

// ------------------------------------------------------------------ h1-adjoint
// g = (D v)^T G (D u) per point.
template <int LX, typename T, bool KEEP>
__global__ SEM_BOUNDS2((Shape<LX, T>::NT), (Shape<LX, T>::MINW)) void k_ax_adjoint(AdjArgs<T> A, DEo<LX, T> D)
{
    using S = Shape<LX, T>;
    __shared__ Lds<LX, T> lds;
    const int tid = threadIdx.x;
    const int slot = tid / S::NP;
    const int t = tid - slot * S::NP;
    const int a = t % LX, b = t / LX;
    const int64_t e = (int64_t)blockIdx.x * S::EPB + slot;
    const bool act = e < A.nelv;
    const int64_t row = e * (int64_t)(LX * LX * LX) + t;  // base of this lane's t-pencil
    T *s0 = lds.buf[0][slot], *s1 = lds.buf[1][slot];

    T u[LX], v[LX];
    load_row<LX, T>(u, A.u + row, act);
    load_row<LX, T>(v, A.v + row, act);
    T g[6][LX];
#pragma unroll
    for (int f = 0; f < 6; ++f) load_g<LX, T, KEEP>(g[f], A.G + f * A.n + row, act);
    T ur[LX], us[LX], ut[LX], vr[LX], vs[LX], vt[LX];
    grad<LX, T>(D, u, s0, s1, a, b, ur, us, ut);
    grad<LX, T>(D, v, s0, s1, a, b, vr, vs, vt);
    T out[LX];
#pragma unroll
    for (int i = 0; i < LX; ++i) {
        const T r = ur[i], s = us[i], q = ut[i];
        out[i] = vr[i] * (g[0][i] * r + g[3][i] * s + g[4][i] * q)
               + vs[i] * (g[3][i] * r + g[1][i] * s + g[5][i] * q)
               + vt[i] * (g[4][i] * r + g[5][i] * s + g[2][i] * q);
    }
    store_row<LX, T>(A.g + row, out, act);
}

// ------------------------------------------------------------------ setup kernels
// Geometric factors from nodal coordinates (isoparametric metric, FP64).
// One thread per point; plain loops (setup only).
template <int LX>
__global__ __launch_bounds__(256) void k_geometry(GeomArgs A, DMat<LX, double> D, WVec<LX> W)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= A.n) return;
    constexpr int NPE = LX * LX * LX;
    const int64_t e = p / NPE;
    const int q = (int)(p - e * NPE);
    const int i = q % LX, j = (q / LX) % LX, k = q / (LX * LX);
    const int64_t b0 = e * NPE;
    double m[3][3];
    for (int c = 0; c < 3; ++c) {
        const double *X = A.xyz + c * A.n + b0;
        double dr = 0, ds = 0, dt = 0;
#pragma unroll
        for (int l = 0; l < LX; ++l) {
            dr = fma(D.d[i * LX + l], X[l + LX * (j + LX * k)], dr);
            ds = fma(D.d[j * LX + l], X[i + LX * (l + LX * k)], ds);
            dt = fma(D.d[k * LX + l], X[i + LX * (j + LX * l)], dt);
        }
        m[c][0] = dr;
        m[c][1] = ds;
        m[c][2] = dt;
    }
    // cofactors: C[c][d] = d(det)/d m[c][d];  inverse: dr_d/dx_c = C[c][d] / J
    double C[3][3];
    C[0][0] = m[1][1] * m[2][2] - m[1][2] * m[2][1];
    C[0][1] = m[1][2] * m[2][0] - m[1][0] * m[2][2];
    C[0][2] = m[1][0] * m[2][1] - m[1][1] * m[2][0];
    C[1][0] = m[0][2] * m[2][1] - m[0][1] * m[2][2];
    C[1][1] = m[0][0] * m[2][2] - m[0][2] * m[2][0];
    C[1][2] = m[0][1] * m[2][0] - m[0][0] * m[2][1];
    C[2][0] = m[0][1] * m[1][2] - m[0][2] * m[1][1];
    C[2][1] = m[0][2] * m[1][0] - m[0][0] * m[1][2];
    C[2][2] = m[0][0] * m[1][1] - m[0][1] * m[1][0];
    const double J = m[0][0] * C[0][0] + m[0][1] * C[0][1] + m[0][2] * C[0][2];
    const double rho = W.w[i] * W.w[j] * W.w[k];
    // G_ab = rho J sum_c (C[c][a]/J)(C[c][b]/J) = rho/J sum_c C[c][a] C[c][b]
    const double s = rho / J;
    const int ia[6] = {0, 1, 2, 0, 0, 1}, ib[6] = {0, 1, 2, 1, 2, 2};
    for (int f = 0; f < 6; ++f) {
        const double d = C[0][ia[f]] * C[0][ib[f]] + C[1][ia[f]] * C[1][ib[f]] + C[2][ia[f]] * C[2][ib[f]];
        A.G[f * A.n + p] = s * d;
    }
    A.B[p] = rho * J;
    if (!(J > 0.0)) atomicAdd(A.nbad, 1u);
}

// Diagonal of the unassembled operator (point Jacobi), FP64, one thread per point.
template <int LX>
__global__ __launch_bounds__(256) void k_diag(DiagArgs A, DMat<LX, double> D)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= A.n) return;
    constexpr int NPE = LX * LX * LX;
    const int64_t e = p / NPE;
    const int q = (int)(p - e * NPE);
    const int i = q % LX, j = (q / LX) % LX, k = q / (LX * LX);
    const int64_t b0 = e * NPE;
    const double *G = A.G;
    const int64_t n = A.n;
    double s = 0.0;
#pragma unroll
    for (int l = 0; l < LX; ++l) {
        const int64_t pr = b0 + l + LX * (j + LX * k);
        const int64_t ps = b0 + i + LX * (l + LX * k);
        const int64_t pt = b0 + i + LX * (j + LX * l);
        const double cr = A.h1 ? A.h1[pr] : A.h1s;
        const double cs = A.h1 ? A.h1[ps] : A.h1s;
        const double ct = A.h1 ? A.h1[pt] : A.h1s;
        const double dri = D.d[l * LX + i], dsj = D.d[l * LX + j], dtk = D.d[l * LX + k];
        s += dri * dri * cr * G[pr];
        s += dsj * dsj * cs * G[n + ps];
        s += dtk * dtk * ct * G[2 * n + pt];
    }
    const double c = A.h1 ? A.h1[p] : A.h1s;
    const double di = D.d[i * LX + i], dj = D.d[j * LX + j], dk = D.d[k * LX + k];
    s += 2.0 * di * dj * c * G[3 * n + p];
    s += 2.0 * di * dk * c * G[4 * n + p];
    s += 2.0 * dj * dk * c * G[5 * n + p];
    const double c2 = A.h2 ? A.h2[p] : A.h2s;
    if (c2 != 0.0) s += c2 * A.B[p];
    A.d[p] = s;
}

}  // namespace sem

// ------------------------------------------------------------------ host launchers
#define SEM_PASTE2(a, b) a##b
#define SEM_PASTE(a, b) SEM_PASTE2(a, b)

namespace {
template <int LX, typename T>
sem::DMat<LX, T> make_dmat(const double *D)
{
    sem::DMat<LX, T> m;
    for (int q = 0; q < LX * LX; ++q) m.d[q] = (T)D[q];
    return m;
}

template <int LX, typename T>
sem::DEo<LX, T> make_deo(const double *D)
{
    using E = sem::DEo<LX, T>;
    constexpr int H = E::H, N = LX - 1;
    E m{};
    for (int a = 0; a < H; ++a)
        for (int l = 0; l < H; ++l) {
            m.S[a * H + l] = (T)(0.5 * (D[a * LX + l] + D[a * LX + (N - l)]));
            m.A[a * H + l] = (T)(0.5 * (D[a * LX + l] - D[a * LX + (N - l)]));
        }
    if constexpr (LX % 2 == 1) {
        for (int a = 0; a < H; ++a) {
            m.cm[a] = (T)D[a * LX + H];
            m.rm[a] = (T)D[H * LX + a];
        }
    }
    return m;
}

// Coefficient form of a lean launch (see KINDS).
template <typename T>
int lean_kind(const T *h1, const T *h2, T h2s)
{
    return (h1 ? 1 : 0) + 2 * (h2 ? 2 : h2s != T(0) ? 1 : 0);
}

// f(integral_constant<int, kind>) for the coefficient form kind.
template <typename F>
void with_kind(int kind, F f)
{
    switch (kind) {
    case 0: f(std::integral_constant<int, 0>()); break;
    case 1: f(std::integral_constant<int, 1>()); break;
    case 2: f(std::integral_constant<int, 2>()); break;
    case 3: f(std::integral_constant<int, 3>()); break;
    case 4: f(std::integral_constant<int, 4>()); break;
    default: f(std::integral_constant<int, 5>()); break;
    }
}

// D row-major of this lx and precision, behind the even-odd form in the device copy.
template <typename T>
const T *dense_d(const void *deo)
{
    return (const T *)((const char *)deo + sizeof(sem::DEo<SEM_LX, T>));
}

// Forms with an instance that reads G plainly: the kernels of whole elements per wave or
// workgroup (lx < 10), and the others where STREAM is unset and the loads are the same for a
// field (with three fields read in chunks, G is read plainly in any case).
template <typename T, int NF>
struct PlainG {
    static constexpr bool LEAN = sem::Shape<SEM_LX, T>::LEAN;
    static constexpr bool CHUNKS3 = NF == 3 && !sem::LeanCfg<SEM_LX, T, NF, false>::HOLD;
    static constexpr bool POSSIBLE = !LEAN || (!sem::STREAM<SEM_LX, T, NF> && !CHUNKS3);
};

template <typename T, int NF>
void launch_ax_nf(const sem::AxArgs<T> &A, const sem::DEo<SEM_LX, T> &Dm, unsigned grid, hipStream_t st)
{
    using S = sem::Shape<SEM_LX, T>;
    using C = sem::TileCfg<SEM_LX, T, NF, false>;
    if constexpr (C::USE) {
        with_kind(lean_kind(A.h1, A.h2, A.h2s), [&](auto k) {
            hipLaunchKernelGGL((sem::k_ax_helm_tile<SEM_LX, T, NF, decltype(k)::value>), dim3(grid), dim3(64 * C::W), 0,
                               st, A, dense_d<T>(A.deo));
        });
    } else {
        const bool mass = A.h2 || A.h2s != T(0), gen = A.h1 || mass;
        auto go = [&](auto keep) {
            constexpr bool KEEP = decltype(keep)::value;
            if constexpr (S::LEAN) {
                with_kind(lean_kind(A.h1, A.h2, A.h2s), [&](auto k) {
                    hipLaunchKernelGGL((sem::k_ax_helm_lean<SEM_LX, T, NF, decltype(k)::value, KEEP>), dim3(grid),
                                       dim3(S::NT), 0, st, A, Dm, (const sem::DEo<SEM_LX, T> *)A.deo);
                });
            } else {
                if (gen) hipLaunchKernelGGL((sem::k_ax_helm<SEM_LX, T, NF, true, KEEP>), dim3(grid), dim3(S::NT), 0, st, A, Dm);
                else hipLaunchKernelGGL((sem::k_ax_helm<SEM_LX, T, NF, false, KEEP>), dim3(grid), dim3(S::NT), 0, st, A, Dm);
            }
        };
        if constexpr (PlainG<T, NF>::POSSIBLE) {
            const int words = 6 + (A.h1 != nullptr) + mass + (A.h2 != nullptr) + 2 * NF;
            if (sem::reads_plainly<SEM_LX, T, NF, false>(A.n, words, mass, A.keep)) return go(std::true_type{});
        }
        go(std::false_type{});
    }
}

template <typename T>
hipError_t launch_ax(const sem::AxArgs<T> &A, const double *D, int nfields, hipStream_t st)
{
    using S = sem::Shape<SEM_LX, T>;
    const unsigned grid = (unsigned)((A.nelv + S::EPB - 1) / S::EPB);
    if (grid == 0) return hipSuccess;
    if (S::LEAN && !A.deo) return hipErrorInvalidValue;
    const auto Dm = make_deo<SEM_LX, T>(D);
    if (nfields == 3) launch_ax_nf<T, 3>(A, Dm, grid, st);
    else launch_ax_nf<T, 1>(A, Dm, grid, st);
    return hipGetLastError();
}

template <typename T, int NF, bool CG1>
void launch_cg_nf(const sem::CgMatvecArgs<T> &A, const sem::DEo<SEM_LX, T> &Dm, unsigned grid, hipStream_t st)
{
    using S = sem::Shape<SEM_LX, T>;
    using C = sem::TileCfg<SEM_LX, T, NF, true>;
    if constexpr (C::USE) {
        with_kind(lean_kind(A.h1, A.h2, A.h2s), [&](auto k) {
            hipLaunchKernelGGL((sem::k_cg_matvec_tile<SEM_LX, T, NF, decltype(k)::value, CG1>), dim3(grid),
                               dim3(64 * C::W), 0, st, A, dense_d<T>(A.deo));
        });
    } else if constexpr (S::LEAN) {
        with_kind(lean_kind(A.h1, A.h2, A.h2s), [&](auto k) {
            hipLaunchKernelGGL((sem::k_cg_matvec_lean<SEM_LX, T, NF, decltype(k)::value, CG1>), dim3(grid), dim3(S::NT),
                               0, st, A, Dm, (const sem::DEo<SEM_LX, T> *)A.deo);
        });
    } else {
        const bool gen = A.h1 || A.h2 || A.h2s != T(0);
        auto go = [&](auto keep, auto fold) {
            constexpr bool KEEP = decltype(keep)::value, FOLD = decltype(fold)::value;
            if (gen)
                hipLaunchKernelGGL((sem::k_cg_matvec<SEM_LX, T, NF, true, CG1, KEEP, FOLD>), dim3(grid), dim3(S::NT), 0, st,
                                   A, Dm);
            else
                hipLaunchKernelGGL((sem::k_cg_matvec<SEM_LX, T, NF, false, CG1, KEEP, FOLD>), dim3(grid), dim3(S::NT), 0, st,
                                   A, Dm);
        };
        if constexpr (!CG1) {
            if constexpr (sizeof(T) == 8 && NF == 1) {
                if (A.nup > 0) return go(std::true_type{}, std::true_type{});
            }
            if (A.keep) return go(std::true_type{}, std::false_type{});
        }
        go(std::false_type{}, std::false_type{});
    }
}

template <typename T, bool CG1>
hipError_t launch_cg(const sem::CgMatvecArgs<T> &A, const double *D, int nfields, hipStream_t st)
{
    using S = sem::Shape<SEM_LX, T>;
    const unsigned grid = (unsigned)((A.nelv + S::EPB - 1) / S::EPB);
    if (grid == 0) return hipSuccess;
    if (S::LEAN && !A.deo) return hipErrorInvalidValue;
    const auto Dm = make_deo<SEM_LX, T>(D);
    if (nfields == 3) launch_cg_nf<T, 3, CG1>(A, Dm, grid, st);
    else launch_cg_nf<T, 1, CG1>(A, Dm, grid, st);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_adj(const sem::AdjArgs<T> &A, const double *D, hipStream_t st)
{
    using S = sem::Shape<SEM_LX, T>;
    const unsigned grid = (unsigned)((A.nelv + S::EPB - 1) / S::EPB);
    if (grid == 0) return hipSuccess;
    if (S::LEAN && sizeof(T) == 8 && !A.deo) return hipErrorInvalidValue;
    const auto Dm = make_deo<SEM_LX, T>(D);
    auto go = [&](auto keep) {
        constexpr bool KEEP = decltype(keep)::value;
        if constexpr (S::LEAN)
            hipLaunchKernelGGL((sem::k_ax_adjoint_lean<SEM_LX, T, KEEP>), dim3(grid), dim3(S::NT), 0, st, A, Dm,
                               (const sem::DEo<SEM_LX, T> *)A.deo);
        else
            hipLaunchKernelGGL((sem::k_ax_adjoint<SEM_LX, T, KEEP>), dim3(grid), dim3(S::NT), 0, st, A, Dm);
    };
    // FP32: plain or not at every size but for lx = 12 and 14 (reads_plainly), one instance: the
    // compiler schedules two of them apart, at lx = 10 and 2.7 million points 16.5 -> 18.3 us
    constexpr bool F32 = sizeof(T) == 4, ONE = sem::STREAM<SEM_LX, T, 1> || (F32 && SEM_LX != 12 && SEM_LX != 14);
    if constexpr (ONE) go(std::bool_constant<!sem::STREAM<SEM_LX, T, 1>>{});
    else if (sem::reads_plainly<SEM_LX, T, 1, true>(A.n, 9, false, true)) go(std::true_type{});
    else go(std::false_type{});
    return hipGetLastError();
}
}  // namespace

extern "C" {

hipError_t SEM_PASTE(sem_launch_ax_f64_lx, SEM_LX)(const sem::AxArgs<double> *A, const double *D,
                                                    int nfields, hipStream_t st)
{
    return launch_ax<double>(*A, D, nfields, st);
}
hipError_t SEM_PASTE(sem_launch_ax_f32_lx, SEM_LX)(const sem::AxArgs<float> *A, const double *D,
                                                    int nfields, hipStream_t st)
{
    return launch_ax<float>(*A, D, nfields, st);
}
hipError_t SEM_PASTE(sem_launch_cg_f64_lx, SEM_LX)(const sem::CgMatvecArgs<double> *A,
                                                    const double *D, int nfields, hipStream_t st)
{
    return launch_cg<double, false>(*A, D, nfields, st);
}
hipError_t SEM_PASTE(sem_launch_cg_f32_lx, SEM_LX)(const sem::CgMatvecArgs<float> *A,
                                                    const double *D, int nfields, hipStream_t st)
{
    return launch_cg<float, false>(*A, D, nfields, st);
}
hipError_t SEM_PASTE(sem_launch_cg1_f64_lx, SEM_LX)(const sem::CgMatvecArgs<double> *A,
                                                     const double *D, int nfields, hipStream_t st)
{
    return launch_cg<double, true>(*A, D, nfields, st);
}
hipError_t SEM_PASTE(sem_launch_adj_f64_lx, SEM_LX)(const sem::AdjArgs<double> *A, const double *D,
                                                     hipStream_t st)
{
    return launch_adj<double>(*A, D, st);
}
hipError_t SEM_PASTE(sem_launch_adj_f32_lx, SEM_LX)(const sem::AdjArgs<float> *A, const double *D,
                                                     hipStream_t st)
{
    return launch_adj<float>(*A, D, st);
}
hipError_t SEM_PASTE(sem_launch_geom_lx, SEM_LX)(const sem::GeomArgs *A, const double *D,
                                                  const double *w, hipStream_t st)
{
    if (A->n == 0) return hipSuccess;
    sem::WVec<SEM_LX> W;
    for (int i = 0; i < SEM_LX; ++i) W.w[i] = w[i];
    const unsigned grid = (unsigned)((A->n + 255) / 256);
    hipLaunchKernelGGL((sem::k_geometry<SEM_LX>), dim3(grid), dim3(256), 0, st, *A,
                       make_dmat<SEM_LX, double>(D), W);
    return hipGetLastError();
}
hipError_t SEM_PASTE(sem_launch_diag_lx, SEM_LX)(const sem::DiagArgs *A, const double *D,
                                                  hipStream_t st)
{
    if (A->n == 0) return hipSuccess;
    const unsigned grid = (unsigned)((A->n + 255) / 256);
    hipLaunchKernelGGL((sem::k_diag<SEM_LX>), dim3(grid), dim3(256), 0, st, *A,
                       make_dmat<SEM_LX, double>(D));
    return hipGetLastError();
}
// The even-odd D of this lx in FP64 and FP32 (the DEo layouts), for the device copy
// the lean FP64 kernels read (out64, out32: host buffers of the two struct sizes).
void SEM_PASTE(sem_deo_fill_lx, SEM_LX)(const double *D, void *out64, void *out32)
{
    const auto m64 = make_deo<SEM_LX, double>(D);
    const auto m32 = make_deo<SEM_LX, float>(D);
    memcpy(out64, &m64, sizeof(m64));
    memcpy(out32, &m32, sizeof(m32));
    const auto d64 = make_dmat<SEM_LX, double>(D);
    const auto d32 = make_dmat<SEM_LX, float>(D);
    memcpy((char *)out64 + sizeof(m64), &d64, sizeof(d64));
    memcpy((char *)out32 + sizeof(m32), &d32, sizeof(d32));
}
// number of per-workgroup partials the CG matvec writes per field
int64_t SEM_PASTE(sem_cg_nblocks_f64_lx, SEM_LX)(int64_t nelv)
{
    using S = sem::Shape<SEM_LX, double>;
    return (nelv + S::EPB - 1) / S::EPB;
}
int64_t SEM_PASTE(sem_cg_nblocks_f32_lx, SEM_LX)(int64_t nelv)
{
    using S = sem::Shape<SEM_LX, float>;
    return (nelv + S::EPB - 1) / S::EPB;
}
}

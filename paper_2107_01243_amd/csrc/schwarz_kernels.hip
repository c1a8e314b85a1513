// schwarz_kernels.hip -- local solves and coarse prolongation of the two-level
// additive Schwarz preconditioner of the pressure solve (Section 4 of arXiv
// 2107.01243), for gfx950.
//
// The local problem of an element is a separable box operator
//   A~ = h1 (Mt x Ms x Kr + Mt x Ks x Mr + Kt x Ms x Mr) + h2 Mt x Ms x Mr,
// solved by fast diagonalisation: with, per direction, the eigenvectors S (row-major
// [node][mode]) and eigenvalues of the 1-D generalised problem K S = M S Lambda,
//   z = (St x Ss x Sr) diag(1 / (h1 (lr_i + ls_j + lt_k) + h2)) (St x Ss x Sr)^T r.
// Two boxes: the element's own lx^3 points (k_fdm<LX, false>), and those points plus one
// layer of extension points beyond every face (k_fdm<LX, true>, (lx + 2)^3 points: the minimal
// overlap of one point, the extension layer's right-hand side gathered from the face
// neighbour; only the element's own points are written back).
//
// Compiled once per lx (-DSEM_LX=<lx>), like the operator kernels.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sem_kernels.h"
#include "sem_pencil.h"

#ifndef SEM_LX
#error "compile with -DSEM_LX=<lx>"
#endif

namespace sem {

// ------------------------------------------------------------------ local solves
// Each of the six 1-D transforms of a solve multiplies an X x X matrix with the X^2 pencils
// of the box.  The matrices differ from element to element, so on the vector units every
// multiply-add needs its matrix entry broadcast from LDS (8 cycles of the compute unit's
// LDS per 16 bytes, shared by four SIMDs), and that broadcast bounded the kernel.  On the
// matrix cores an entry is held by one lane and no broadcast is needed: FP64 4x4x4
// products of four independent blocks, the matrix tile the same in all four, so one
// instruction multiplies a 4x4 tile with 16 pencils at the vector units' FP64 rate.
//
// Operand layout (lane = c + 16 g): B holds row g of a 4-row tile of pencil c, the result
// holds row g of pencil c again, and A holds row c % 4, column g of the matrix tile.  A
// pencil's points are thus spread over the four lane groups (node or mode 4 tile + g), and
// the result of one transform is the operand of the next one along the same direction
// (forward and inverse along s are chained in registers); between directions the box goes
// through LDS (row stride odd: no bank conflicts).
//
// Nodes are ordered own points first (0 .. lx - 1), then with the overlap the extension
// points below and above (lx, lx + 1): the inverse transforms then form the tiles of the
// own points only.
//
// 32^3 elements, lx = 8, in a solve: element box 99 us with the multiply-adds on the vector
// units, 78 in this form; box with overlap 234 and 216.  Now
// neither a memory nor a matrix bound: the matrix cores are busy 38% of the time, the
// vector units (the FP64 divisions, addresses, the gathers of the overlap) 35%, LDS 43%.
template <int LX, bool OV>
struct FdmShape {
    static constexpr int X = OV ? LX + 2 : LX;
    static constexpr int P = (X % 2) ? X : X + 1;                  // LDS row stride
    static constexpr int T = (X + 3) / 4, TL = (LX + 3) / 4;       // tiles of all / own nodes
    // Waves per element W, tiles in flight per wave HG and waves per SIMD the registers
    // leave room for EU, measured per box size X at 9 to 17 million points (whole
    // application without the coarse steps, multiply-adds on the vector units -> here): X = 4 355 -> 300 us, 5 249 ->
    // 238, 6 262 -> 266 (EU 4: 276), 7 158 -> 160, 8 271 -> 249, 9 316 -> 306, 10 313 ->
    // 319 (W 2, HG 4: 330), 12 256 -> 230, 16 285 -> 260; with overlap X = 6 517 -> 483,
    // 7 380 -> 338, 8 347 -> 340, 9 298 -> 240, 10 416 -> 386 (W 1: 408, W 4: 397), 11
    // 424 -> 372, 12 447 -> 385, 14 350 -> 336, 18 506 -> 448.
    static constexpr int W = X <= 8 ? 1 : X <= 10 ? (OV ? 2 : 4) : X <= 14 ? 4 : 8;
    static constexpr int HG = X == 10 && !OV ? 2 : 4;
    static constexpr int EU = X == 6 ? 8 : X == 10 && !OV ? 6 : 4;
    static constexpr int NT = 64 * W;
};

// A operand of every tile of S^T (forward: rows are modes) or of S (inverse: rows are
// nodes); S in LDS, padded with zeros to whole tiles (row stride 4 TK').
template <int TS, int TM, int TK, bool FWD>
__device__ __forceinline__ void fdm_matrix(const double *Sd, double (&m)[TM][TK])
{
    const int i = threadIdx.x & 3, k = (threadIdx.x >> 4) & 3;
    const double *p = Sd + (FWD ? 4 * TS * k + i : 4 * TS * i + k);
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tk = 0; tk < TK; ++tk) m[tm][tk] = p[FWD ? 16 * TS * tk + 4 * tm : 16 * TS * tm + 4 * tk];
}

// One transform of the workgroup's COUNT pencils, 16 per tile, the tiles dealt to the W
// waves in turn: get(h, x) loads the operand rows of the wave's tile h, put(h, y) takes
// the result rows.  HG tiles are in flight together, so that consecutive matrix
// instructions are independent (a dependent one waits for its predecessor).
template <int COUNT, typename Sh, int TM, int TK, typename Get, typename Put>
__device__ __forceinline__ void fdm_stage(const double (&m)[TM][TK], Get get, Put put)
{
    constexpr int W = Sh::W, TPW = (COUNT + 16 * W - 1) / (16 * W), HG = TPW < Sh::HG ? TPW : Sh::HG;
#pragma unroll
    for (int h0 = 0; h0 < TPW; h0 += HG) {
        double x[HG][TK], y[HG][TM];
#pragma unroll
        for (int h = 0; h < HG; ++h)
            if (h0 + h < TPW) get(h0 + h, x[h]);
#pragma unroll
        for (int tk = 0; tk < TK; ++tk)
#pragma unroll
            for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                for (int h = 0; h < HG; ++h)
                    if (h0 + h < TPW)
                        y[h][tm] = __builtin_amdgcn_mfma_f64_4x4x4f64(m[tm][tk], x[h][tk], tk ? y[h][tm] : 0.0, 0, 0, 0);
#pragma unroll
        for (int h = 0; h < HG; ++h)
            if (h0 + h < TPW) put(h0 + h, y[h]);
    }
}

// Pencil of lane column c in the wave's tile h, clamped to the COUNT pencils there are
// (a clamped lane computes the last pencil again and stores nothing).
template <int COUNT, int W>
__device__ __forceinline__ int fdm_pencil(int wave, int c, int h)
{
    const int p = 16 * (wave + W * h) + c;
    return 16 * W * (h + 1) <= COUNT ? p : min(p, COUNT - 1);
}
template <int COUNT, int W>
__device__ __forceinline__ bool fdm_valid(int wave, int c, int h)
{
    return 16 * W * (h + 1) <= COUNT || 16 * (wave + W * h) + c < COUNT;
}

// Rows 4 t + g (of X in use) of the lane's pencil; p points at row 0, rows STRIDE apart.
template <int X, int T, int STRIDE>
__device__ __forceinline__ void fdm_get(const double *p, int g, double (&x)[T])
{
#pragma unroll
    for (int t = 0; t < T; ++t) x[t] = (4 * t + 3 < X || 4 * t + g < X) ? p[(4 * t + g) * STRIDE] : 0.0;
}
template <int X, int T, int STRIDE>
__device__ __forceinline__ void fdm_put(double *p, int g, const double (&y)[T])
{
#pragma unroll
    for (int t = 0; t < T; ++t)
        if (4 * t + 3 < X || 4 * t + g < X) p[(4 * t + g) * STRIDE] = y[t];
}

// Residual at the extension point of a face (face coordinates fa, fb; fc = the face's
// table entry {neighbour, base, sa, sb}); zero where the face has no neighbour.
template <int LX>
__device__ __forceinline__ double ext_value(const double *__restrict__ r, int4 fc, int fa, int fb)
{
    constexpr int L3 = LX * LX * LX;  // (a field has fewer than 2^31 points)
    return fc.x < 0 ? 0.0 : r[fc.x * L3 + fc.y + fa * fc.z + fb * fc.w];
}

// One element per workgroup of W waves; the waves share the 16-pencil tiles of every
// transform.  OV: the right-hand side of the extended box is
//  - own points: r of the element;
//  - one coordinate outside (a face layer): r at the neighbour's point one GLL index
//    inside it (face table A.face), zero without a neighbour;
//  - two or three coordinates outside (box edges and corners): zero.
// The 1-D operators of a face without a neighbour hold a decoupled extension node, so
// with its zero right-hand side the solve there equals the element-only one.
// With A.part the same pass restricts r to the coarse space: per element the eight sums
// over its owned points of r times the trilinear corner functions, contracted along t
// with the loads, then along s and along r between the transforms.
template <int LX, bool OV>
__global__ __launch_bounds__((FdmShape<LX, OV>::NT)) __attribute__((
    amdgpu_waves_per_eu(FdmShape<LX, OV>::EU))) void k_fdm(FdmArgs A)
{
    using Sh = FdmShape<LX, OV>;
    constexpr int X = Sh::X, P = Sh::P, T = Sh::T, TL = Sh::TL, W = Sh::W, NT = Sh::NT;
    constexpr int X2 = X * X, L2 = LX * LX, L3 = L2 * LX;
    __shared__ double cube[P * X2];
    __shared__ double red[2 * L2 + 4 * LX];
    __shared__ double lam[3 * X];
    constexpr int TS = T, S2 = 16 * T * T;  // padded matrix
    __shared__ double Ss[3 * S2];
    const int64_t e = blockIdx.x;
    const int tid = threadIdx.x, c = tid & 15, g = (tid >> 4) & 3;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const double *__restrict__ re = A.r + e * L3;
    const double *__restrict__ lin = A.lin;
    // everything the element reads from memory is requested at once
#pragma unroll
    for (int q0 = 0; q0 < 3 * S2; q0 += NT) {
        const int q = q0 + tid;
        if (3 * S2 % NT == 0 || q < 3 * S2) {
            const int col = q % (4 * T), row = q / (4 * T) % (4 * T), d = q / S2;
            Ss[q] = X % 4 == 0 || (col < X && row < X) ? A.S[(e * 3 + d) * X2 + row * X + col] : 0.0;
        }
    }
    for (int q = tid; q < 3 * X; q += NT) lam[q] = A.lam[e * 3 * X + q];
    constexpr int TPW = (X2 + 16 * W - 1) / (16 * W), PLANE = P * X;
    double xr[OV ? 1 : TPW][T];  // element box: the pencils along t
    unsigned ob[TPW];            // their owner flags, bit t for row 4 t + g
    int px[TPW], py[TPW];        // pencil p = px + X py
#pragma unroll
    for (int h = 0; h < TPW; ++h) {
        const int p = fdm_pencil<X2, W>(wave, c, h);
        py[h] = p / X;
        px[h] = p - X * py[h];
        if constexpr (!OV) fdm_get<X, T, L2>(re + p, g, xr[h]);
        ob[h] = 0;
        if (A.part && fdm_valid<X2, W>(wave, c, h) && (!OV || (px[h] < LX && py[h] < LX))) {
            const uint8_t *ow = A.owner + e * L3 + px[h] + LX * py[h];
#pragma unroll
            for (int t = 0; t < TL; ++t)
                if (4 * t + 3 < LX || 4 * t + g < LX) ob[h] |= ow[(4 * t + g) * L2] ? 1u << t : 0u;
        }
    }
    if constexpr (OV) {
        int4 fc[(6 * L2 + NT - 1) / NT];
        const int4 *__restrict__ face = (const int4 *)A.face + e * 6;
#pragma unroll
        for (int q0 = 0, u = 0; q0 < 6 * L2; q0 += NT, ++u) fc[u] = face[min((q0 + tid) / L2, 5)];
#pragma unroll
        for (int q0 = 0; q0 < L3; q0 += NT) {
            const int q = q0 + tid;
            if (L3 % NT == 0 || q < L3) cube[q % LX + P * (q / LX % LX + X * (q / L2))] = re[q];
        }
#pragma unroll
        for (int q0 = 0, u = 0; q0 < 6 * L2; q0 += NT, ++u) {
            const int q = q0 + tid;
            if (6 * L2 % NT == 0 || q < 6 * L2) {
                const int f = q / L2, fa = q % LX, fb = q / LX % LX, d = f >> 1, n = LX + (f & 1);
                // the face point's two coordinates, ascending direction order
                const int st = d == 0 ? P : 1, su = d == 2 ? P : PLANE, sn = d == 0 ? 1 : d == 1 ? P : PLANE;
                cube[st * fa + su * fb + sn * n] = ext_value<LX>(A.r, fc[u], fa, fb);
            }
        }
        for (int q = tid; q < 12 * X; q += NT) {
            const int o = q / (4 * X), n = q % X, u = LX + (q / X & 1), v = LX + (q / (2 * X) & 1);
            cube[o == 0 ? n + P * (u + X * v) : o == 1 ? u + P * (n + X * v) : u + P * (v + X * n)] = 0.0;
        }
    }
    bsync<NT>();
    // forward along t; the restriction's sums along t are one more (two-row) product
    {
        double mt[T][T], lt[1][TL];
        fdm_matrix<TS, T, T, true>(Ss + 2 * S2, mt);
#pragma unroll
        for (int t = 0; t < TL; ++t) {
            const int l = 4 * t + g, row = c & 3;
            lt[0][t] = row < 2 && (LX % 4 == 0 || l < LX) ? lin[row * LX + (LX % 4 == 0 || l < LX ? l : 0)] : 0.0;
        }
        fdm_stage<X2, Sh, T, T>(
            mt,
            [&](int h, double (&x)[T]) {
                if constexpr (OV) fdm_get<X, T, PLANE>(cube + px[h] + P * py[h], g, x);
                else {
#pragma unroll
                    for (int t = 0; t < T; ++t) x[t] = xr[h][t];
                }
                if (A.part) {
                    double s = 0.0;
#pragma unroll
                    for (int t = 0; t < TL; ++t)
                        s = __builtin_amdgcn_mfma_f64_4x4x4f64(lt[0][t], ob[h] >> t & 1 ? x[t] : 0.0, s, 0, 0, 0);
                    // row g < 2 of the result: the sum against linear function g
                    if (fdm_valid<X2, W>(wave, c, h) && g < 2 && (!OV || (px[h] < LX && py[h] < LX)))
                        red[g * L2 + px[h] + LX * py[h]] = s;
                }
            },
            [&](int h, const double (&y)[T]) {
                if (fdm_valid<X2, W>(wave, c, h)) fdm_put<X, T, PLANE>(cube + px[h] + P * py[h], g, y);
            });
    }
    bsync<NT>();
    if (A.part)
        for (int q = tid; q < 4 * LX; q += NT) {
            const int i = q % LX, cb = q / LX;  // cb = (j side) + 2 (k side)
            const double *rk = red + (cb >> 1) * L2 + i;
            const double *lj = lin + (cb & 1) * LX;
            double s = 0.0;
            for (int j = 0; j < LX; ++j) s = fma(lj[j], rk[LX * j], s);
            red[2 * L2 + q] = s;
        }
    // forward along r: pencil (j, k) is row p = j + X k
    {
        double mr[T][T];
        fdm_matrix<TS, T, T, true>(Ss, mr);
        fdm_stage<X2, Sh, T, T>(
            mr, [&](int h, double (&x)[T]) { fdm_get<X, T, 1>(cube + P * fdm_pencil<X2, W>(wave, c, h), g, x); },
            [&](int h, const double (&y)[T]) {
                if (fdm_valid<X2, W>(wave, c, h)) fdm_put<X, T, 1>(cube + P * fdm_pencil<X2, W>(wave, c, h), g, y);
            });
    }
    bsync<NT>();
    if (A.part && tid < 8) {
        const double *li = lin + (tid & 1) * LX;
        const double *u = red + 2 * L2 + (tid >> 1) * LX;
        double s = 0.0;
        for (int i = 0; i < LX; ++i) s = fma(li[i], u[i], s);
        A.part[e * 8 + tid] = s;
    }
    // forward along s, the division by the box operator's eigenvalues, inverse along s:
    // pencil (i, k), p = i + X k
    {
        double ms[T][T], is[TL][T], ls[T];
        fdm_matrix<TS, T, T, true>(Ss + S2, ms);
        fdm_matrix<TS, TL, T, false>(Ss + S2, is);
#pragma unroll
        for (int t = 0; t < T; ++t) ls[t] = lam[X + (4 * t + 3 < X ? 4 * t + g : min(4 * t + g, X - 1))];
        double v[TPW][T];
        fdm_stage<X2, Sh, T, T>(
            ms, [&](int h, double (&x)[T]) { fdm_get<X, T, P>(cube + px[h] + PLANE * py[h], g, x); },
            [&](int h, const double (&y)[T]) {
                // (a row past the last mode is zero here: its matrix rows are)
                const double lr = lam[px[h]], lt = lam[2 * X + py[h]];
#pragma unroll
                for (int t = 0; t < T; ++t) v[h][t] = y[t] / (A.h1 * (lr + ls[t] + lt) + A.h2);
            });
        fdm_stage<X2, Sh, TL, T>(
            is,
            [&](int h, double (&x)[T]) {
#pragma unroll
                for (int t = 0; t < T; ++t) x[t] = v[h][t];
            },
            [&](int h, const double (&z)[TL]) {
                if (fdm_valid<X2, W>(wave, c, h)) fdm_put<LX, TL, P>(cube + px[h] + PLANE * py[h], g, z);
            });
    }
    bsync<NT>();
    // inverse along r: pencils (j, k) with j an own point, p = j + lx k
    {
        constexpr int NR = LX * X;
        double ir[TL][T];
        fdm_matrix<TS, TL, T, false>(Ss, ir);
        auto row = [&](int h) {
            const int p = fdm_pencil<NR, W>(wave, c, h), k = p / LX;
            return cube + P * (p - LX * k + X * k);
        };
        fdm_stage<NR, Sh, TL, T>(
            ir, [&](int h, double (&x)[T]) { fdm_get<X, T, 1>(row(h), g, x); },
            [&](int h, const double (&y)[TL]) {
                if (fdm_valid<NR, W>(wave, c, h)) fdm_put<LX, TL, 1>(row(h), g, y);
            });
    }
    bsync<NT>();
    // inverse along t: own pencils (i, j), p = i + lx j; the own points go to z
    {
        double it[TL][T];
        fdm_matrix<TS, TL, T, false>(Ss + 2 * S2, it);
        fdm_stage<L2, Sh, TL, T>(
            it,
            [&](int h, double (&x)[T]) {
                const int p = fdm_pencil<L2, W>(wave, c, h), j = p / LX;
                fdm_get<X, T, PLANE>(cube + (p - LX * j) + P * j, g, x);
            },
            [&](int h, const double (&y)[TL]) {
                if (fdm_valid<L2, W>(wave, c, h))
                    fdm_put<LX, TL, L2>(A.z + e * L3 + fdm_pencil<L2, W>(wave, c, h), g, y);
            });
    }
}

// Coarse prolongation: the element's eight coarse values interpolated trilinearly
// (along r, then s on the two t faces, then t per point), added to the
// multiplicity-averaged local solution.  Lanes as in the t-pencil layout; whole
// elements per workgroup.
template <int LX>
struct ProlongShape {
    static constexpr int L2 = LX * LX;
    static constexpr int EPB = 256 / L2 > 0 ? 256 / L2 : 1;
    static constexpr int NT = EPB * L2;
};

template <int LX>
__global__ __launch_bounds__(ProlongShape<LX>::NT) void k_prolong(ProlongArgs A)
{
    constexpr int L2 = LX * LX, L3 = L2 * LX, EPB = ProlongShape<LX>::EPB;
    const int el = threadIdx.x / L2, t = threadIdx.x - el * L2;
    const int64_t e = (int64_t)blockIdx.x * EPB + el;
    if (e >= A.nelv) return;
    const int a = t % LX, b = t / LX;
    const double *__restrict__ lin = A.lin;
    // the element's values first (behind a store of z the compiler would hold back the next
    // point's loads), then the corner values, two round trips away
    double *z = A.z + e * L3;
    const uint8_t *mu = A.mult + e * L3;
    double zk[LX];
    int mk[LX];
#pragma unroll
    for (int k = 0; k < LX; ++k) {
        zk[k] = z[k * L2 + t];
        mk[k] = mu[k * L2 + t];
    }
    double c[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) c[q] = A.e0[A.cvert[e * 8 + q]];
    const double ra0 = lin[a], ra1 = lin[LX + a], sb0 = lin[b], sb1 = lin[LX + b];
    double f[2];
#pragma unroll
    for (int kc = 0; kc < 2; ++kc) {
        const double y0 = fma(ra1, c[4 * kc + 1], ra0 * c[4 * kc]);
        const double y1 = fma(ra1, c[4 * kc + 3], ra0 * c[4 * kc + 2]);
        f[kc] = fma(sb1, y1, sb0 * y0);
    }
#pragma unroll
    for (int k = 0; k < LX; ++k) {
        const double v = fma(lin[LX + k], f[1], lin[k] * f[0]);
        // 1, 2, 4 or 8 copies: an exact scaling, for which the division's ~30 operations are
        // not needed; 0 marks a Dirichlet point
        const int m = mk[k];
        double y = __builtin_ldexp(zk[k], 1 - __ffs(m));
        if (m & (m - 1)) y = zk[k] / (double)m;
        z[k * L2 + t] = m ? y + v : 0.0;
    }
}

}  // namespace sem

#define SEM_PASTE2(a, b) a##b
#define SEM_PASTE(a, b) SEM_PASTE2(a, b)

extern "C" {

// A->face set: the extended box (S, lam of size lx + 2 per direction); else the
// element's own box.
hipError_t SEM_PASTE(sem_launch_fdm_lx, SEM_LX)(const sem::FdmArgs *A, hipStream_t st)
{
    if (A->nelv == 0) return hipSuccess;
    if (A->nelv > 0x7fffffff) return hipErrorInvalidValue;
    if (A->part && (!A->owner || !A->lin)) return hipErrorInvalidValue;
    if (A->face)
        hipLaunchKernelGGL((sem::k_fdm<SEM_LX, true>), dim3((unsigned)A->nelv), dim3(sem::FdmShape<SEM_LX, true>::NT), 0,
                           st, *A);
    else
        hipLaunchKernelGGL((sem::k_fdm<SEM_LX, false>), dim3((unsigned)A->nelv), dim3(sem::FdmShape<SEM_LX, false>::NT),
                           0, st, *A);
    return hipGetLastError();
}
hipError_t SEM_PASTE(sem_launch_prolong_lx, SEM_LX)(const sem::ProlongArgs *A, hipStream_t st)
{
    using Sh = sem::ProlongShape<SEM_LX>;
    if (A->nelv == 0) return hipSuccess;
    const int64_t g = (A->nelv + Sh::EPB - 1) / Sh::EPB;
    if (g > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL((sem::k_prolong<SEM_LX>), dim3((unsigned)g), dim3(Sh::NT), 0, st, *A);
    return hipGetLastError();
}

}  // extern "C"

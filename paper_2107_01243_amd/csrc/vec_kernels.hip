// vec_kernels.hip -- gather-scatter, masking and Krylov-vector kernels of libsem (gfx950).
//
// Gather-scatter QQ^T (Jansson et al., arXiv 2107.01243, Eq. 10 and the local
// gather + scatter of Algorithm 1): ids with two copies are a pair list (the
// "injective" ids of Section 3.2), ids with more copies are CSR blocks.  One lane
// per pair / block sums the copies in ascending local order starting from +0 and
// writes the sum back, so the result is deterministic and bit-reproducible.
//
// CG / flexible-CG vector kernels: streaming, one point per lane per step with
// grid-stride loops, FP64 accumulation of every inner product, per-workgroup
// partial sums reduced afterwards in a fixed order by a single workgroup
// (deterministic; no floating-point atomics).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "sem_kernels.h"
#include "sem_wave.h"
#include "vec_kernels.h"

#ifndef SEM_GS_XCD
#define SEM_GS_XCD 1
#endif

namespace sem {

#ifndef SEM_VCH
#define SEM_VCH 2
#endif
#ifndef SEM_ARN_G
#define SEM_ARN_G 1024
#endif
#ifndef SEM_ARN_R
#define SEM_ARN_R 2
#endif

constexpr int VT = 256;   // lanes per workgroup of the streaming kernels
// Streaming kernels: workgroup b handles the contiguous chunk [b*CHUNK, (b+1)*CHUNK)
// (VCH points per lane); the grid is as wide as the vector, and the number of
// per-workgroup partial sums stays n / CHUNK.
constexpr int VCH = SEM_VCH;
constexpr int64_t CHUNK = (int64_t)VT * VCH;
constexpr int RT = 1024;  // lanes of the single-workgroup reduction kernels

#ifndef SEM_UPD64
#define SEM_UPD64 2
#endif
#ifndef SEM_GS_EPL
#define SEM_GS_EPL 2
#endif
constexpr int GEPL = SEM_GS_EPL;  // 64-entry segments per wave of the entry-parallel gs
#ifndef SEM_UPD32
#define SEM_UPD32 8
#endif
// Points per lane of one CG-update workgroup, per precision: an FP32 chunk moves half
// the bytes of an FP64 one, so it takes more points to amortise the workgroup's
// reduction epilogue (and it halves the partials the finish kernel sums).
template <typename T> struct UpdChunk;
// GV: the same for the update that gathers, which holds four more values per point.
template <> struct UpdChunk<double> { static constexpr int UV = SEM_UPD64, GV = 2; };
template <> struct UpdChunk<float> { static constexpr int UV = SEM_UPD32, GV = 4; };

// A value that is streamed, or (KEEP) one that stays in the last-level cache.
template <bool KEEP, typename T>
__device__ __forceinline__ T ld(const T *p)
{
    if constexpr (KEEP) return *p;
    else return __builtin_nontemporal_load(p);
}
template <bool KEEP, typename T>
__device__ __forceinline__ void stv(T v, T *p)
{
    if constexpr (KEEP) *p = v;
    else __builtin_nontemporal_store(v, p);
}

// Sum `nblk` partials in a fixed order inside one workgroup of NTH lanes: lane t
// accumulates entries t, t+NTH, ... into four interleaved accumulators (loads in
// flight), combines them, then a fixed binary tree, in LDS down to a wave's width.  Deterministic for a
// given (nblk, NTH).  Returns the sum to every lane.
template <int NTH>
__device__ double block_sum_fixed(const double *part, int64_t nblk, double *sh)
{
    const int tid = threadIdx.x;
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    int64_t q = tid;
    for (; q + 3 * NTH < nblk; q += 4 * NTH) {
        a0 += part[q];
        a1 += part[q + NTH];
        a2 += part[q + 2 * NTH];
        a3 += part[q + 3 * NTH];
    }
    for (; q < nblk; q += NTH) a0 += part[q];
    sh[tid] = (a0 + a1) + (a2 + a3);
    __syncthreads();
    for (int w = NTH / 2; w >= 64; w >>= 1) {
        if (tid < w) sh[tid] += sh[tid + w];
        __syncthreads();
    }
    const double r = wave_sum(sh[tid & 63]);
    __syncthreads();
    return r;
}

// Single-reduction CG (Chronopoulos-Gear) scalars once r_k and w_k = A u_k are known
// (u_k = dinv r_k): gamma = (r_k, u_k), delta = (u_k, A u_k), rr = (r_k, r_k).  On the
// first call (primed == 0) beta = 0 and alpha = gamma / delta; afterwards
// beta = gamma / gamma_old and alpha = gamma / (delta - beta gamma / alpha_old), which
// reproduce the two-reduction CG recurrences in exact arithmetic.
__device__ inline void cg1_fold(CgScalars &s, double gamma, double delta, double rr)
{
    if (s.stop) return;
    const bool first = s.primed == 0;
    if (!first) s.iter += 1;
    s.rr = rr;
    const double rel = s.bb > 0.0 ? sqrt(rr / s.bb) : 0.0;
    if (!isfinite(gamma) || !isfinite(delta) || !isfinite(rr)) {
        s.stop = 1;
        s.status = 2;
        return;
    }
    if ((s.rtol > 0.0 && rel <= s.rtol) || gamma == 0.0) {
        s.stop = 1;
        s.rz = gamma;
        return;
    }
    if (s.iter >= s.max_iter) {
        s.stop = 1;
        s.status = (s.rtol > 0.0) ? 1 : 0;
        return;
    }
    const double beta = first ? 0.0 : gamma / s.rz;
    const double den = first ? delta : delta - beta * gamma / s.alpha;
    if (!(den > 0.0) || !isfinite(den)) {
        s.stop = 1;
        s.status = 2;
        s.alpha = 0.0;
        return;
    }
    s.beta = beta;
    s.alpha = gamma / den;
    s.rz = gamma;
    s.primed = 1;
}

// Step length of one field, alpha = rz / (p, A p); stops it on a breakdown.
__device__ inline void cg_set_alpha(CgScalars &sc, double pw)
{
    if (sc.stop) return;
    if (!(pw > 0.0) || !isfinite(pw) || !isfinite(sc.rz)) {
        sc.stop = 1;
        sc.status = 2;
        sc.alpha = 0.0;
        sc.pend = 0;
    } else {
        sc.alpha = sc.rz / pw;
    }
}

// Fold of the CG scalars for every field by workgroup 0 of a gather-scatter launch
// (the matvec whose partials it reads ended before this launch began).
template <int NTH>
__device__ void fold_job(const AlphaJob &J, int nfields, double *sh)
{
    for (int f = 0; f < nfields; ++f) {
        if (J.mode == 0) {
            const double pw = block_sum_fixed<NTH>(J.partial + f * J.nblk, J.nblk, sh);
            if (threadIdx.x == 0) cg_set_alpha(J.scal[f], pw);
        } else {
            CgScalars &sc = J.scal[f];
            // read before the barriers of the first sum, and so by every wave before lane 0
            // writes the state: the branch below holds barriers too
            const bool primed = sc.primed != 0;
            const double d = block_sum_fixed<NTH>(J.partial + f * J.nblk, J.nblk, sh);
            double g = sc.rz, rr = sc.rr;  // before the first step: from the start kernels
            if (primed) {
                g = block_sum_fixed<NTH>(J.partial2 + (0 * nfields + f) * J.nblk2, J.nblk2, sh);
                rr = block_sum_fixed<NTH>(J.partial2 + (1 * nfields + f) * J.nblk2, J.nblk2, sh);
            }
            if (threadIdx.x == 0) cg1_fold(sc, g, d, rr);
            __syncthreads();  // the next field's reads follow lane 0's update
        }
    }
}

// ------------------------------------------------------------------ gather-scatter
template <typename T>
__global__ __launch_bounds__(VT) void k_gs(GsArgs<T> A)
{
    // Workgroups are dealt to the 8 XCDs round-robin by the hardware.  Map them so
    // that XCD x processes one contiguous slice of the group list (which is ordered
    // by element), so each XCD's L2 works on one contiguous range of elements.
#if SEM_GS_XCD
    const unsigned per = gridDim.x / 8;  // the launcher rounds the grid up to 8 * per
    const unsigned lb = (blockIdx.x % 8) * per + blockIdx.x / 8;
#else
    const unsigned lb = blockIdx.x;
#endif
    const int64_t tid = (int64_t)lb * VT + threadIdx.x;
    for (int f = 0; f < A.nfields; ++f) {
        if (A.skip && A.skip[f].stop) continue;
        T *u = A.u + f * A.n;
        if (tid < A.npairs) {
            const int32_t a = A.pairs[2 * tid], b = A.pairs[2 * tid + 1];
            const T s = (T(0) + u[a]) + u[b];
            u[a] = s;
            u[b] = s;
        } else if (tid < A.npairs + A.nblocks) {
            const int64_t g = tid - A.npairs;
            const int64_t lo = A.blk_ptr[g], hi = A.blk_ptr[g + 1];
            T s = T(0);
            for (int64_t c = lo; c < hi; ++c) s += u[A.blk_idx[c]];
            for (int64_t c = lo; c < hi; ++c) u[A.blk_idx[c]] = s;
        }
    }
    // Optional fold of the CG step length: alpha_f = rz_f / (p, A p)_f from the
    // matvec's partials (complete, since that kernel ended before this one began).
    if (A.alpha_job && blockIdx.x == 0) {
        __shared__ double sh[VT];
        fold_job<VT>(*A.alpha_job, A.nfields, sh);
    }
}

// Entry-parallel gather-scatter: a lane owns one shared entry in each of the
// wave's segments of 64 (ascending global id, groups never straddle a segment).  Every lane of a group reads the group's values
// from its neighbour lanes and sums them in ascending local order from +0, so all
// copies receive the identical, canonical sum; then each lane writes its own copy.
// The shuffle loop runs max_group times for the whole wave (all lanes active).
template <typename T>
__device__ __forceinline__ void gs_entries_wave(const GsArgs<T> &A, int64_t wave)
{
    // each wave owns GEPL consecutive 64-entry segments; lane l handles entry l of
    // each, so its GEPL index -> value loads are independent and in flight together
    const int lane = threadIdx.x & 63;
    const int64_t base = wave * (64 * GEPL) + lane;
    int32_t e[GEPL];
    int cnt[GEPL], lead[GEPL];
    // a group's extent from the start flags of the segment: its first lane is the
    // nearest flagged lane at or below this one, its end the next flagged lane (padding
    // counts as flagged, and every segment opens with a flagged lane)
    const uint64_t upto = lane == 63 ? ~0ull : ((2ull << lane) - 1);
#pragma unroll
    for (int k = 0; k < GEPL; ++k) {
        const int64_t t = base + 64 * k;
        const uint32_t wd = t < A.nent ? A.ent_word[t] : 0xffffffffu;
        const bool pad = wd == 0xffffffffu;
        e[k] = pad ? -1 : (int32_t)(wd & 0x7fffffffu);
        const uint64_t M = __ballot(pad || (wd >> 31) != 0);
        lead[k] = 63 - __clzll((long long)(M & upto));
        const uint64_t above = M & ~upto;
        cnt[k] = (above ? __ffsll((long long)above) - 1 : 64) - lead[k];
    }
    for (int f = 0; f < A.nfields; ++f) {
        if (A.skip && A.skip[f].stop) continue;
        T *u = A.u + f * A.n;
        T v[GEPL], s[GEPL];
#pragma unroll
        for (int k = 0; k < GEPL; ++k) {
            v[k] = (e[k] >= 0) ? u[e[k]] : T(0);
            s[k] = T(0);
        }
        for (int q = 0; q < A.max_group; ++q) {
#pragma unroll
            for (int k = 0; k < GEPL; ++k) {
                const int src = lead[k] + q;
                const T x = __shfl(v[k], src < 64 ? src : lane, 64);
                if (q < cnt[k]) s[k] += x;
            }
        }
#pragma unroll
        for (int k = 0; k < GEPL; ++k)
            if (e[k] >= 0) u[e[k]] = s[k];
    }
}

// Block b of nb (a multiple of 8) of the entry list: blocks are dealt to the XCDs in turn,
// and XCD x takes one contiguous range of the list.
__device__ __forceinline__ unsigned gs_block(unsigned b, unsigned nb)
{
#if SEM_GS_XCD
    return (b % 8) * (nb / 8) + b / 8;
#else
    return b;
#endif
}

template <typename T>
__global__ __launch_bounds__(VT) void k_gs_entries(GsArgs<T> A)
{
    if (A.skip) {
        // every field stopped: nothing to gather, and no step length left to set
        bool live = false;
        for (int f = 0; f < A.nfields; ++f) live = live || !A.skip[f].stop;
        if (!live) return;
    }
    gs_entries_wave(A, (int64_t)gs_block(blockIdx.x, gridDim.x) * (VT / 64) + (threadIdx.x >> 6));
    if (A.alpha_job && blockIdx.x == 0) {
        __shared__ double sh[VT];
        fold_job<VT>(*A.alpha_job, A.nfields, sh);
    }
}

// pmap of the updates that gather (see CgUpdateArgs) from the entry list, on a pmap of -1.
__global__ __launch_bounds__(VT) void k_gather_map(const uint32_t *ent_word, int64_t nent, const uint8_t *owner,
                                                   int32_t *pmap)
{
    const int64_t t = (int64_t)blockIdx.x * VT + threadIdx.x;  // (64 | VT: a wave is a segment)
    const int lane = threadIdx.x & 63;
    const uint32_t wd = t < nent ? ent_word[t] : 0xffffffffu;
    const bool pad = wd == 0xffffffffu;
    const uint64_t M = __ballot(pad || (wd >> 31) != 0), upto = lane == 63 ? ~0ull : ((2ull << lane) - 1);
    if (pad) return;
    const int lead = 63 - __clzll((long long)(M & upto));
    const uint64_t above = M & ~upto;
    const int cnt = (above ? __ffsll((long long)above) - 1 : 64) - lead;
    const int64_t first = t - lane + lead;
    const int32_t e = (int32_t)(wd & 0x7fffffffu);
    if (cnt == 2) pmap[e] = (int32_t)(ent_word[2 * first + 1 - t] & 0x7fffffffu);
    else pmap[e] = (int32_t)(-2 - (32 * first + 2 * (cnt - 1) + (owner[e] ? 1 : 0)));
}

// ------------------------------------------------------------------ basis combinations
// Linear combination of up to PB basis vectors (coefficients by value).
__global__ __launch_bounds__(VT) void k_comb(CombArgs A)
{
    // the starting vector is chosen once per launch (uniform): none, y itself, or src.
    // (Selecting it per point with a nested conditional was compiled, for src, into a
    // load through a scalar register that was never assigned on that path.)
    const double *s0 = (A.mode == 1) ? A.y : A.src;
    const bool start = A.mode != 0;
    const int64_t t_end = min(A.n, (int64_t)(blockIdx.x + 1) * CHUNK);
    for (int64_t t = (int64_t)blockIdx.x * CHUNK + threadIdx.x; t < t_end; t += VT) {
        double s = 0.0;
        if (start) s = s0[t];
#pragma unroll
        for (int i = 0; i < PB; ++i)
            if (i < A.l) s = fma(A.c[i], A.V[i * A.ld + t], s);
        A.y[t] = s;
    }
}

constexpr int log2up(int m) { return m <= 1 ? 0 : 1 + log2up((m + 1) / 2); }

// Sums over the wave of M rows held one value per lane and row (M a power of two, at
// most 64): on return lane l holds in v[0] the sum of row l >> (6 - log2 M).  Each stage
// (OFF = 32, 16, ...) exchanges half of the rows still held, so M rows cost
// M - 1 + 6 - log2 M exchanges (63 for 64 rows) instead of the 6 M of one butterfly per
// row, and the exchanges of a stage are independent of each other.
template <int M, int OFF = 32, int MT>
__device__ __forceinline__ void wave_sum_rows(double (&v)[MT])
{
    if constexpr (OFF > 0) {
        if constexpr (M > 1) {
            const bool up = threadIdx.x & OFF;
#pragma unroll
            for (int i = 0; i < M / 2; ++i) {
                const double give = up ? v[i] : v[i + M / 2], keep = up ? v[i + M / 2] : v[i];
                v[i] = keep + __shfl_xor(give, OFF, 64);
            }
            wave_sum_rows<M / 2, OFF / 2>(v);
        } else {
            v[0] += __shfl_xor(v[0], OFF, 64);
            wave_sum_rows<1, OFF / 2>(v);
        }
    }
}

// Sum of one row of per-workgroup partials over a wave, fixed order, four loads in
// flight per lane.
__device__ __forceinline__ double wave_row_sum(const double *row, int64_t nblk)
{
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    int64_t b = threadIdx.x & 63;
    for (; b + 192 < nblk; b += 256) {
#pragma unroll
        for (int u = 0; u < 4; ++u) a[u] += row[b + 64 * u];
    }
    for (int u = 0; b < nblk; b += 64, ++u) a[u & 3] += row[b];
    return wave_sum((a[0] + a[1]) + (a[2] + a[3]));
}

// Basis vector i of m at point t, streamed non-temporally; zero past the end.  The passes
// below hold MV >= m vectors in registers (MV a few sizes up to 32), the spare ones with
// zero coefficients or unused sums.
__device__ __forceinline__ double basis_load(const double *V, int64_t ld, int i, int m, int64_t t)
{
    return i < m ? __builtin_nontemporal_load(V + i * ld + t) : 0.0;
}

// Arnoldi pass (see ArnArgs).  Each workgroup streams one contiguous chunk of
// points; every lane keeps the m basis values of its point in registers, so the
// combination and the dots of the combined vector need one read of each vector.
// The basis (tens of vectors, far beyond the last-level cache) is read with
// non-temporal hints, as in the Gram-Schmidt passes below.
template <int MV, int MODE>
__global__ __launch_bounds__(VT) void k_arn(ArnArgs A, int64_t chunk)
{
    const int m = A.m;
    double c[MV];
    double sc = 1.0;
    if constexpr (MODE != 0) {
#pragma unroll
        for (int i = 0; i < MV; ++i) c[i] = (i < m) ? A.coef[i] : 0.0;
        if constexpr (MODE == 2) sc = A.scale[0];
    }
    constexpr int LG = log2up(MV), M2 = 1 << LG;
    double acc[M2], nn = 0.0;
#pragma unroll
    for (int i = 0; i < M2; ++i) acc[i] = 0.0;
    const int64_t t0 = (int64_t)blockIdx.x * chunk;
    const int64_t t1 = min(A.n, t0 + chunk);
    for (int64_t t = t0 + threadIdx.x; t < t1; t += VT) {
        double v[MV];
#pragma unroll
        for (int i = 0; i < MV; ++i) v[i] = basis_load(A.V, A.ld, i, m, t);
        double y = A.w[t];
        if constexpr (MODE != 0) {
#pragma unroll
            for (int i = 0; i < MV; ++i) y = fma(-c[i], v[i], y);
            if constexpr (MODE == 2) y *= sc;
            A.y[t] = y;
        }
        if constexpr (MODE != 2) {
            const double yo = A.owner[t] ? y : 0.0;
#pragma unroll
            for (int i = 0; i < MV; ++i) acc[i] = fma(v[i], yo, acc[i]);
            nn = fma(y, yo, nn);
        }
    }
    if constexpr (MODE != 2) {
        // rows: the m dots (transposed wave sums), then the squared norm
        __shared__ double sh[VT / 64][M2 + 1];
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        wave_sum_rows<M2>(acc);
        const double yy = wave_sum(nn);
        if ((lane & ((1 << (6 - LG)) - 1)) == 0) sh[wave][lane >> (6 - LG)] = acc[0];
        if (lane == 0) sh[wave][M2] = yy;
        __syncthreads();
        const int q = threadIdx.x;
        if (q <= m) {
            const int src = (q < m) ? q : M2;
            double x = 0.0;
#pragma unroll
            for (int w4 = 0; w4 < VT / 64; ++w4) x += sh[w4][src];
            A.partial[(int64_t)q * gridDim.x + blockIdx.x] = x;
        }
    }
}

// Sums of nq rows of per-workgroup partials, one wave per row, fixed order.  With
// pyth, the last row is a squared norm |y|^2 and the others the coefficients h of a
// second Gram-Schmidt pass: out[nq] = sqrt(|y|^2 - |h|^2) (the norm after that pass,
// by the Pythagorean identity) and out[nq + 1] = its reciprocal (0 if not positive).
__global__ __launch_bounds__(RT) void k_arn_finish(const double *partial, int64_t nblk, int nq, int pyth,
                                                   double *out)
{
    __shared__ double sh[ARN_MAXV + 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int q = wave; q < nq; q += RT / 64) {
        const double s = wave_row_sum(partial + (int64_t)q * nblk, nblk);
        if (lane == 0) {
            out[q] = s;
            sh[q] = s;
        }
    }
    if (pyth) {
        __syncthreads();
        if (threadIdx.x == 0) {
            const int m = nq - 1;
            double hh = sh[m];
            for (int i = 0; i < m; ++i) hh = fma(-sh[i], sh[i], hh);
            hh = hh > 0.0 ? hh : 0.0;
            out[nq] = sqrt(hh);
            out[nq + 1] = hh > 0.0 ? 1.0 / sqrt(hh) : 0.0;
        }
    }
}

// Dots pass of the delayed Gram-Schmidt step (see DcgsArgs).
template <int MV>
__global__ __launch_bounds__(VT) void k_dcgs_dots(DcgsArgs A, int64_t chunk)
{
    const int j = A.j;
    constexpr int LG = log2up(2 * MV), M2 = 1 << LG;
    double ab[M2], uu = 0.0, uw = 0.0, ww = 0.0;  // V^T u (from 0), V^T w (from MV)
#pragma unroll
    for (int i = 0; i < M2; ++i) ab[i] = 0.0;
    const int64_t t0 = (int64_t)blockIdx.x * chunk;
    const int64_t t1 = min(A.n, t0 + chunk);
    for (int64_t t = t0 + threadIdx.x; t < t1; t += VT) {
        double v[MV];
#pragma unroll
        for (int i = 0; i < MV; ++i) v[i] = basis_load(A.V, A.ld, i, j, t);
        const double u = A.u[t], w = A.w[t];
        const bool own = A.owner[t] != 0;
        const double uo = own ? u : 0.0, wo = own ? w : 0.0;
#pragma unroll
        for (int i = 0; i < MV; ++i) {
            ab[i] = fma(v[i], uo, ab[i]);
            ab[MV + i] = fma(v[i], wo, ab[MV + i]);
        }
        uu = fma(u, uo, uu);
        uw = fma(u, wo, uw);
        ww = fma(w, wo, ww);
    }
    // rows: a_0..a_{j-1}, (u,u), b_0..b_{j-1}, (u,w), (w,w).  The sums are formed
    // transposed (wave_sum_rows): with one butterfly per row this reduction took most of
    // the 41 us of a 30-vector pass over 2e5 points.
    __shared__ double sh[VT / 64][2 * MV + 3];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    wave_sum_rows<M2>(ab);
    uu = wave_sum(uu);
    uw = wave_sum(uw);
    ww = wave_sum(ww);
    if ((lane & ((1 << (6 - LG)) - 1)) == 0) {
        const int q = lane >> (6 - LG);
        if (q < j) sh[wave][q] = ab[0];
        else if (q >= MV && q - MV < j) sh[wave][j + 1 + q - MV] = ab[0];
    }
    if (lane == 0) {
        sh[wave][j] = uu;
        sh[wave][2 * j + 1] = uw;
        sh[wave][2 * j + 2] = ww;
    }
    __syncthreads();
    const int q = threadIdx.x;
    if (q < 2 * j + 3) {
        double x = 0.0;
#pragma unroll
        for (int w4 = 0; w4 < VT / 64; ++w4) x += sh[w4][q];
        A.partial[(int64_t)q * gridDim.x + blockIdx.x] = x;
    }
}

// Update pass of the delayed Gram-Schmidt step (see DcgsArgs).
template <int MV>
__global__ __launch_bounds__(VT) void k_dcgs_update(DcgsArgs A, int64_t chunk)
{
    const int j = A.j;
    const double *cf = A.coef;
    double ca[MV], cc[MV];
#pragma unroll
    for (int i = 0; i < MV; ++i) {
        ca[i] = (i < j) ? cf[i] : 0.0;
        cc[i] = (i < j) ? cf[j + i] : 0.0;
    }
    const double irho = cf[2 * j], del = cf[2 * j + 1], inu = cf[2 * j + 2];
    const int64_t t0 = (int64_t)blockIdx.x * chunk;
    const int64_t t1 = min(A.n, t0 + chunk);
    for (int64_t t = t0 + threadIdx.x; t < t1; t += VT) {
        double v[MV];
#pragma unroll
        for (int i = 0; i < MV; ++i) v[i] = basis_load(A.V, A.ld, i, j, t);
        const double u = A.u[t];
        double q = u, y = A.w[t];
#pragma unroll
        for (int i = 0; i < MV; ++i) {
            q = fma(-ca[i], v[i], q);
            y = fma(-cc[i], v[i], y);
        }
        y = fma(-del, u, y);
        A.u[t] = q * irho;
        A.w[t] = y * inu;
    }
}

// Reduction of the dots pass, one wave per row in a fixed order: out[0..2j+3) = the
// row sums; then at out + 2 j + 3 the update coefficients and the step's scalars:
//   rho^2 = (u,u) - |a|^2,  gamma = ((u,w) - a.b) / rho,  delta = gamma / rho,
//   nu^2 = (w,w) - |b|^2 - gamma^2  (Pythagorean identities),  c = b - delta a;
//   [a (j), c (j), 1/rho, delta, 1/nu, rho, gamma, nu]  (reciprocals 0 when not positive).
__global__ __launch_bounds__(RT) void k_dcgs_finish(const double *partial, int64_t nblk, int j, double *out)
{
    __shared__ double sh[2 * ARN_MAXV + 3];
    const int nq = 2 * j + 3;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int q = wave; q < nq; q += RT / 64) {
        const double s = wave_row_sum(partial + (int64_t)q * nblk, nblk);
        if (lane == 0) {
            out[q] = s;
            sh[q] = s;
        }
    }
    __syncthreads();
    if (threadIdx.x < 64) {  // lane i holds a_i and b_i (j < 32)
        const double a = lane < j ? sh[lane] : 0.0, b = lane < j ? sh[j + 1 + lane] : 0.0;
        const double aa = sh[j] - wave_sum(a * a), ab = sh[2 * j + 1] - wave_sum(a * b);
        const double bb = sh[2 * j + 2] - wave_sum(b * b);
        const double rho = aa > 0.0 ? sqrt(aa) : 0.0;
        const double gam = rho > 0.0 ? ab / rho : 0.0;
        const double del = rho > 0.0 ? gam / rho : 0.0;
        double nn = fma(-gam, gam, bb);
        nn = nn > 0.0 ? nn : 0.0;
        const double nu = sqrt(nn);
        double *cf = out + nq;
        if (lane < j) {
            cf[lane] = a;
            cf[j + lane] = fma(-del, a, b);
        }
        if (lane == 0) {
            cf[2 * j] = rho > 0.0 ? 1.0 / rho : 0.0;
            cf[2 * j + 1] = del;
            cf[2 * j + 2] = nu > 0.0 ? 1.0 / nu : 0.0;
            cf[2 * j + 3] = rho;
            cf[2 * j + 4] = gam;
            cf[2 * j + 5] = nu;
        }
    }
}

// y = a * b pointwise (point-Jacobi preconditioning of a Krylov vector).
__global__ __launch_bounds__(VT) void k_hadamard(double *y, const double *a, const double *b, int64_t n)
{
    const int64_t t_end = min(n, (int64_t)(blockIdx.x + 1) * CHUNK);
    for (int64_t t = (int64_t)blockIdx.x * CHUNK + threadIdx.x; t < t_end; t += VT) y[t] = a[t] * b[t];
}

// ------------------------------------------------------------------ two-level Schwarz
// Per element, the eight weighted sums against the trilinear corner functions (used at
// setup for the Galerkin products P_e^T A_e P_e from probe vectors; the restriction
// P^T r of an application is formed inside the local-solve kernel).
__global__ __launch_bounds__(VT) void k_corner(CornerArgs A)
{
    __shared__ double sh[8][VT / 64];
    const int64_t e = blockIdx.x;
    double acc[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[c] = 0.0;
    for (int p = threadIdx.x; p < A.lx3; p += VT) {
        const int64_t t = e * A.lx3 + p;
        const double x = (A.owner && !A.owner[t]) ? 0.0 : A.v[t];
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[c] = fma(A.phi[c * A.lx3 + p], x, acc[c]);
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        double x = acc[c];
        x = wave_sum(x);
        if (lane == 0) sh[c][wave] = x;
    }
    __syncthreads();
    if (threadIdx.x < 8) {
        double x = 0.0;
#pragma unroll
        for (int q = 0; q < VT / 64; ++q) x += sh[threadIdx.x][q];
        A.out[e * 8 + threadIdx.x] = x;
    }
}

// ---- coarse solve: a fixed number of Jacobi-CG steps on A0 x = b from x = 0.
//
// The system is small (one unknown per element vertex) and its time is launches and
// dependent memory round trips, not bytes.  Two forms, chosen by nv in
// sem_launch_coarse_cg:
//  * k_ccg_small: the whole solve in one workgroup, for systems that its registers and
//    LDS hold (nv <= 1536, rows of at most 28 entries).  Per step 0.95 us at nv <= 512,
//    1.3 us at 1000, 3.1 us at 1331, against 5.7 us of a launch per step.
//  * k_ccg_start + k_ccg_step: one launch per step in the single-reduction form; 5.7 us
//    per step at 2197 vertices, 6.1 us at 15,625 (10.6 and 11.1 us with the two
//    launches per step of the textbook form; the one-workgroup form needs the matrix
//    read again every step there, 27 x 12 bytes per row through one compute unit).

// Right-hand side of vertex v, gathered from the per-element restriction sums.
__device__ __forceinline__ double coarse_rhs(const CoarseArgs &A, int64_t v)
{
    double b = 0.0;
    if (!A.vdir[v])
        for (int64_t q = A.vptr[v]; q < A.vptr[v + 1]; ++q) b += A.part[A.vidx[q]];
    return b;
}

constexpr int CST = 512;              // lanes of k_ccg_small
constexpr int CCG_SMALL = 3 * CST;    // largest system it takes

constexpr int RESW = 28;    // most entries per row (a hexahedral box has 27)

// Sums of a and b over the workgroup in one fixed order, returned to every lane; one
// barrier.  Another must follow before the next call.
__device__ __forceinline__ void small_sum2(double &a, double &b, double (*sh)[CST / 64])
{
    a = wave_sum(a);
    b = wave_sum(b);
    if ((threadIdx.x & 63) == 0) {
        sh[0][threadIdx.x >> 6] = a;
        sh[1][threadIdx.x >> 6] = b;
    }
    __syncthreads();
    a = sh[0][0];
    b = sh[1][0];
#pragma unroll
    for (int q = 1; q < CST / 64; ++q) {
        a += sh[0][q];
        b += sh[1][q];
    }
}

// Whole coarse solve in one workgroup, in the single-reduction form of k_ccg_step (two
// barriers a step): lane t owns rows t, t + 512, ... (RPT of them) with the vectors in
// registers and u = D r shared through LDS for the matrix product.  The
// matrix stays on the compute unit for all steps: columns packed two to a register,
// values in registers, and with three rows per lane the last LW entries of each row in
// LDS (the 256 registers a lane has with two waves per SIMD do not hold them; spilled to
// memory, a step took 7 us).
template <int RPT>
__global__ __launch_bounds__(CST) void k_ccg_small(CoarseArgs A, int iters, GsArgs<double> G)
{
    if (blockIdx.x > 0) {  // the other workgroups: the gather-scatter
        gs_entries_wave(G, (int64_t)(blockIdx.x - 1) * (CST / 64) + (threadIdx.x >> 6));
        return;
    }
    constexpr int LW = RPT > 2 ? 12 : 0, RW = RESW - LW;
    __shared__ double ps[CST * RPT];
    __shared__ double sh[2][CST / 64];
    __shared__ double al[LW > 0 ? LW * RPT * CST : 1];
    double x[RPT], r[RPT], p[RPT], s[RPT], d[RPT], a[RPT][RW];
    unsigned c2[RPT][RESW / 2];
#pragma unroll
    for (int h = 0; h < RPT; ++h) {
        const int64_t v = threadIdx.x + h * CST;
        const bool in = v < A.nv;
#pragma unroll
        for (int w = 0; w < RESW; ++w) {
            const int64_t k = (w < A.width ? w : 0) * A.nv + (in ? v : 0);
            const double av = in && w < A.width ? A.val[k] : 0.0;
            if (w < RW) a[h][w] = av;
            else al[((w - RW) * RPT + h) * CST + threadIdx.x] = av;  // read back by this lane only
            const unsigned c = (unsigned)A.ci[k];
            c2[h][w / 2] = (w & 1) ? (c2[h][w / 2] | c << 16) : c;
        }
        r[h] = in ? coarse_rhs(A, v) : 0.0;
        d[h] = in ? A.dinv[v] : 0.0;
        x[h] = 0.0;
        p[h] = 0.0;
        s[h] = 0.0;
    }
    double gam = 0.0, alpha = 0.0;
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int h = 0; h < RPT; ++h) ps[threadIdx.x + h * CST] = d[h] * r[h];
        __syncthreads();
        double w[RPT], g = 0.0, del = 0.0;
#pragma unroll
        for (int h = 0; h < RPT; ++h) {
            double y = 0.0;
#pragma unroll
            for (int k = 0; k < RESW; ++k) {
                const double av = k < RW ? a[h][k] : al[((k - RW) * RPT + h) * CST + threadIdx.x];
                y = fma(av, ps[(k & 1) ? c2[h][k / 2] >> 16 : c2[h][k / 2] & 0xffffu], y);
                // bound the LDS reads in flight (their results would spill)
                if constexpr (RPT > 2) {
                    if (k % 7 == 6) __builtin_amdgcn_sched_barrier(0);
                }
            }
            w[h] = y;
            const double u = d[h] * r[h];
            g = fma(r[h], u, g);
            del = fma(u, y, del);
        }
        small_sum2(g, del, sh);
        const double beta = gam != 0.0 ? g / gam : 0.0;  // (0 at the first step)
        const double den = it > 0 ? del - beta * g / alpha : del;
        alpha = (den > 0.0 && isfinite(den)) ? g / den : 0.0;
        gam = g;
#pragma unroll
        for (int h = 0; h < RPT; ++h) {
            p[h] = fma(beta, p[h], d[h] * r[h]);
            s[h] = fma(beta, s[h], w[h]);
            x[h] = fma(alpha, p[h], x[h]);
            r[h] = fma(-alpha, s[h], r[h]);
        }
    }
#pragma unroll
    for (int h = 0; h < RPT; ++h) {
        const int64_t v = threadIdx.x + h * CST;
        if (v < A.nv) A.x[v] = x[h];
    }
}

// Blocks [lo, hi) of the nb of a gather-scatter of z that a launch of the coarse solve also
// runs: the coarse steps are a chain of short latency-bound launches that leaves the memory
// idle, and the sum of the local solves over shared points does not depend on them.  At
// 16.8M points and 35,937 vertices 11 launches of 14.7 us, against 8.8 us each and 75 us for
// the gather-scatter alone (all of it in the first launch 170 us together, in the first two
// 181); 960 elements, lx = 6: one launch of 52 us against 48 + 4.8.
struct GsSlice {
    GsArgs<double> G;
    unsigned lo, hi, nb;
};
__device__ __forceinline__ void gs_slice(const GsSlice &S, unsigned b)
{
    if (b < S.hi - S.lo)
        gs_entries_wave(S.G, (int64_t)gs_block(S.lo + b, S.nb) * (VT / 64) + (threadIdx.x >> 6));
}

// Start of the launch-per-step form: r = b, w = s = 0, p = x = 0.
__global__ __launch_bounds__(VT) void k_ccg_start(CoarseArgs A, unsigned nc, GsSlice S)
{
    if (blockIdx.x >= nc) {
        gs_slice(S, blockIdx.x - nc);
        return;
    }
    const int64_t v = (int64_t)blockIdx.x * VT + threadIdx.x;
    if (v >= A.nv) return;
    A.rec0[v] = CoarseRec{coarse_rhs(A, v), 0.0, 0.0, A.dinv[v]};
    A.x[v] = 0.0;
    A.p[v] = 0.0;
}

// One step of single-reduction Jacobi-CG (Chronopoulos-Gear) per launch.  With u = D r
// (D the Jacobi inverse), w = A u, gamma = (r, u), delta = (u, w) of the current iterate
// (reduced here from the previous launch's partials, by every workgroup in the same
// fixed order):
//   beta = gamma / gamma_old, alpha = gamma / (delta - beta gamma / alpha_old),
//   p = u + beta p, s = w + beta s, x += alpha p, r -= alpha s,
// then the new u, w, gamma, delta, with the new r of every column a row touches formed
// on the fly from that column's record (r, w, s, D: one 32-byte gather).  Launch 0 has
// alpha = beta = 0 and only forms w, gamma, delta; the last launch only updates x.
// Records alternate between rec0 (read by even launches) and rec1.  SPL lanes share a
// row (entries w = part, part + SPL, ...; summed across the lanes in a fixed order).
// The records are requested before the partial sums are reduced, so the two round trips
// overlap.
#ifndef SEM_CCG_SPL
#define SEM_CCG_SPL 4
#endif
constexpr int SPL = SEM_CCG_SPL;
constexpr int CCG_PRE = 28 / SPL;  // entries per lane requested ahead (27-point rows)
__global__ __launch_bounds__(VT) void k_ccg_step(CoarseArgs A, int it, int last, unsigned nc, GsSlice S)
{
    if (blockIdx.x >= nc) {
        gs_slice(S, blockIdx.x - nc);
        return;
    }
    __shared__ double sh[4][VT / 64];
    const CoarseRec *ro = (it & 1) ? A.rec1 : A.rec0;
    CoarseRec *rn = (it & 1) ? A.rec0 : A.rec1;
    const int64_t g = nc;
    const int part = threadIdx.x % SPL, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t v = ((int64_t)blockIdx.x * VT + threadIdx.x) / SPL;
    const bool in = v < A.nv;
    const int64_t vc = in ? v : 0;
    const CoarseRec own = ro[vc];
    const double pv = A.p[vc], xv = A.x[vc];
    CoarseRec c[CCG_PRE];
    double a[CCG_PRE];
    if (!last) {
#pragma unroll
        for (int q = 0; q < CCG_PRE; ++q) {
            const int w = part + q * SPL;
            const int64_t k = (int64_t)(w < A.width ? w : 0) * A.nv + vc;
            a[q] = w < A.width ? A.val[k] : 0.0;
            c[q] = ro[A.ci[k]];
        }
    }
    double alpha = 0.0, beta = 0.0;
    if (it > 0) {
        const double *pg = A.partial + (it & 1) * 2 * g;
        double s0 = 0.0, s1 = 0.0;
        for (int64_t q = threadIdx.x; q < g; q += VT) {
            s0 += pg[q];
            s1 += pg[g + q];
        }
        s0 = wave_sum(s0);
        s1 = wave_sum(s1);
        if (lane == 0) {
            sh[0][wave] = s0;
            sh[1][wave] = s1;
        }
        __syncthreads();
        double gam = sh[0][0], del = sh[1][0];
#pragma unroll
        for (int q = 1; q < VT / 64; ++q) {
            gam += sh[0][q];
            del += sh[1][q];
        }
        // scal: (gamma, alpha) of the previous step, two slots in turn
        const double *so = A.scal + 2 * ((it + 1) & 1);
        if (it > 1) beta = (so[0] != 0.0) ? gam / so[0] : 0.0;
        const double den = it > 1 ? del - beta * gam / so[1] : del;
        alpha = (den > 0.0 && isfinite(den)) ? gam / den : 0.0;
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            A.scal[2 * (it & 1)] = gam;
            A.scal[2 * (it & 1) + 1] = alpha;
        }
    }
    if (part == 0 && in && it > 0) {
        const double pn = fma(beta, pv, own.d * own.r);
        A.p[v] = pn;
        A.x[v] = fma(alpha, pn, xv);
    }
    if (last) return;
    const double so = fma(beta, own.s, own.w), rv = fma(-alpha, so, own.r), uv = own.d * rv;
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < CCG_PRE; ++q) {
        const double rc = fma(-alpha, fma(beta, c[q].s, c[q].w), c[q].r);
        s = fma(a[q], c[q].d * rc, s);
    }
    for (int w = part + CCG_PRE * SPL; w < A.width; w += SPL) {  // wider rows than a hexahedral box has
        const int64_t k = (int64_t)w * A.nv + vc;
        const CoarseRec e = ro[A.ci[k]];
        s = fma(A.val[k], e.d * fma(-alpha, fma(beta, e.s, e.w), e.r), s);
    }
#pragma unroll
    for (int off = 1; off < SPL; off <<= 1) s += __shfl_xor(s, off, 64);
    double gn = 0.0, dn = 0.0;
    if (part == 0 && in) {
        rn[v] = CoarseRec{rv, s, so, own.d};
        gn = rv * uv;
        dn = uv * s;
    }
    gn = wave_sum(gn);
    dn = wave_sum(dn);
    if (lane == 0) {
        sh[2][wave] = gn;
        sh[3][wave] = dn;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        double t = 0.0;
#pragma unroll
        for (int q = 0; q < VT / 64; ++q) t += sh[2 + threadIdx.x][q];
        A.partial[(((it + 1) & 1) * 2 + threadIdx.x) * g + blockIdx.x] = t;
    }
}

// Per element, the sums over its points of G_dd / B for d = r, s, t (the local
// solves' element lengths), in a fixed order: out[e][d].
__global__ __launch_bounds__(VT) void k_elem_gb(const double *G, const double *B, double *out, int64_t n, int lx3)
{
    __shared__ double sh[3][VT / 64];
    const int64_t e = blockIdx.x;
    double s[3] = {0.0, 0.0, 0.0};
    for (int p = threadIdx.x; p < lx3; p += VT) {
        const int64_t t = e * lx3 + p;
        const double b = B[t];
#pragma unroll
        for (int d = 0; d < 3; ++d) s[d] += G[d * n + t] / b;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        double x = s[d];
        x = wave_sum(x);
        if (lane == 0) sh[d][wave] = x;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        double x = 0.0;
#pragma unroll
        for (int q = 0; q < VT / 64; ++q) x += sh[threadIdx.x][q];
        out[e * 3 + threadIdx.x] = x;
    }
}

// Probe vector for the Galerkin coarse matrix: v[e][p] = phi[c][p] in every element.
__global__ __launch_bounds__(VT) void k_probe(double *v, const double *phi, int c, int64_t nelv, int lx3)
{
    const int64_t t = (int64_t)blockIdx.x * VT + threadIdx.x;
    if (t >= nelv * lx3) return;
    v[t] = phi[c * lx3 + (int)(t % lx3)];
}

// STREAM triad a = b + s c (bandwidth micro-benchmark).
__global__ __launch_bounds__(VT) void k_triad(double *__restrict__ a, const double *__restrict__ b,
                                              const double *__restrict__ c, double s, int64_t n)
{
    const int64_t t_end = min(n, (int64_t)(blockIdx.x + 1) * CHUNK);
#pragma unroll
    for (int64_t t = (int64_t)blockIdx.x * CHUNK + threadIdx.x; t < t_end; t += VT) a[t] = fma(s, c[t], b[t]);
}

// u[idx] = 0 for every listed index, each field.
template <typename T>
__global__ __launch_bounds__(VT) void k_mask(T *u, const int32_t *idx, int64_t m, int64_t n, int nfields)
{
    const int64_t t = (int64_t)blockIdx.x * VT + threadIdx.x;
    if (t >= m) return;
    for (int f = 0; f < nfields; ++f) u[f * n + idx[t]] = T(0);
}

template <typename T>
__global__ __launch_bounds__(VT) void k_fill(T *u, T v, int64_t m)
{
    for (int64_t t = (int64_t)blockIdx.x * CHUNK + threadIdx.x, t_end = min((int64_t)(m), (int64_t)(blockIdx.x + 1) * CHUNK); t < t_end; t += VT)
        u[t] = v;
}

// dst = (TD)(scale * src)
template <typename TD, typename TS>
__global__ __launch_bounds__(VT) void k_cast(TD *dst, const TS *src, double scale, int64_t m)
{
    for (int64_t t = (int64_t)blockIdx.x * CHUNK + threadIdx.x, t_end = min((int64_t)(m), (int64_t)(blockIdx.x + 1) * CHUNK); t < t_end; t += VT)
        dst[t] = (TD)(scale * (double)src[t]);
}

// ------------------------------------------------------------------ Jacobi inverse
// dinv = 1/d (d already summed over copies), 0 on Dirichlet points.
__global__ __launch_bounds__(VT) void k_invert(double *d, const uint8_t *dir, int64_t n)
{
    const int64_t t = (int64_t)blockIdx.x * VT + threadIdx.x;
    if (t >= n) return;
    d[t] = (dir && dir[t]) ? 0.0 : 1.0 / d[t];
}

// ------------------------------------------------------------------ CG kernels
// Initial residual: r = b - w (w = QQ^T A_L x0), zero where dinv == 0 (Dirichlet);
// p = 0; partials of (r, dinv r), (r, r), (b, b) over owned points.
template <typename T>
__global__ __launch_bounds__(VT) void k_cg_init(CgInitArgs<T> A)
{
    __shared__ double sh[3][VT];
    const int f = blockIdx.y;
    const T *b = A.b + f * A.n;
    const T *w = A.w ? A.w + f * A.n : nullptr;
    T *r = A.r + f * A.n;
    T *p = A.p + f * A.n;
    double rz = 0.0, rr = 0.0, bb = 0.0;
    for (int64_t t = (int64_t)blockIdx.x * CHUNK + threadIdx.x, t_end = min((int64_t)(A.n), (int64_t)(blockIdx.x + 1) * CHUNK); t < t_end; t += VT) {
        const T di = A.dinv[t];
        const T bi = b[t];
        const T ri = (di != T(0)) ? (w ? bi - w[t] : bi) : T(0);
        r[t] = ri;
        p[t] = T(0);
        if (A.owner[t]) {
            rz += (double)ri * (double)(di * ri);
            rr += (double)ri * (double)ri;
            bb += (double)bi * (double)bi;
        }
    }
    sh[0][threadIdx.x] = rz;
    sh[1][threadIdx.x] = rr;
    sh[2][threadIdx.x] = bb;
    __syncthreads();
    for (int s = VT / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s)
            for (int q = 0; q < 3; ++q) sh[q][threadIdx.x] += sh[q][threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        for (int q = 0; q < 3; ++q) A.partial[((int64_t)q * A.nfields + f) * gridDim.x + blockIdx.x] = sh[q][0];
}

// Finish the initial reductions: rz, rr, bb; beta = 0; stop at once when b = 0
// or the initial guess already meets the tolerance.
__global__ __launch_bounds__(RT) void k_cg_start(CgFinishArgs A)
{
    __shared__ double sh[RT];
    for (int f = 0; f < A.nfields; ++f) {
        const double rz = block_sum_fixed<RT>(A.partial + (0 * A.nfields + f) * A.nblk, A.nblk, sh);
        const double rr = block_sum_fixed<RT>(A.partial + (1 * A.nfields + f) * A.nblk, A.nblk, sh);
        const double bb = block_sum_fixed<RT>(A.partial + (2 * A.nfields + f) * A.nblk, A.nblk, sh);
        if (threadIdx.x == 0) {
            CgScalars &s = A.scal[f];
            s.rz = rz;
            s.rr = rr;
            s.bb = bb;
            s.beta = 0.0;
            s.alpha = 0.0;
            s.iter = 0;
            s.status = 0;
            s.stop = 0;
            const double rel = bb > 0.0 ? sqrt(rr / bb) : 0.0;
            if (A.hist) A.hist[(int64_t)f * A.hist_len] = rel;
            if (!isfinite(bb) || !isfinite(rr) || !isfinite(rz)) { s.stop = 1; s.status = 2; }
            else if (bb == 0.0 || (s.rtol > 0.0 && rel <= s.rtol)) s.stop = 1;
            else if (s.max_iter <= 0) { s.stop = 1; s.status = 1; }
        }
    }
}

// x += alpha p (where A.x is set: see CgMatvecArgs::x); r -= alpha w (not on Dirichlet
// points); partials of (r, dinv r), (r, r).
// Workgroup b streams the contiguous chunk of UV * VT points starting at b * UV * VT
// (UV per precision: see upd_chunk); its two partials are reduced per wave
// and then over the four waves in order (deterministic, one barrier).
template <typename T, bool KEEP>
__global__ __launch_bounds__(VT) void k_cg_update(CgUpdateArgs<T> A)
{
    constexpr int UV = UpdChunk<T>::UV;
    __shared__ double sh[2][VT / 64];
    const int f = blockIdx.y;
    double rz = 0.0, rr = 0.0;
    T *x = A.x + f * A.n;
    T *r = A.r + f * A.n;
    const T *p = A.p + f * A.n;
    const T *w = A.w + f * A.n;
    if constexpr (sizeof(T) == 4) {
        // FP32: the field's stop flag and step length (written by the previous
        // kernels, so not in the scalar cache) are requested together with the
        // chunk's operands, not before them (indices past the end are clamped to the
        // last point, so every load is in bounds and unconditional; those lanes store
        // and accumulate nothing).  Measured: 79 -> 67 us at 16.8M points.  (In FP64
        // the same form was slower.)
        // With several fields, launches queued after a field has stopped (its segment
        // ended between host polls) are frequent and each would still read every operand
        // of that field: there the flag is tested first (it costs one scalar-load latency
        // per workgroup, negligible against a multi-field chunk).
        if (A.nfields > 1 && A.scal[f].stop) return;
        const int stop = A.scal[f].stop;
        const T alpha = (T)A.scal[f].alpha;
        const int64_t t0 = (int64_t)blockIdx.x * UV * VT + threadIdx.x;
        T di[UV], xv[UV], pv[UV], rv[UV], wv[UV];
        uint8_t own[UV];
#pragma unroll
        for (int u = 0; u < UV; ++u) {
            const int64_t t = min(t0 + (int64_t)u * VT, A.n - 1);
            di[u] = ld<KEEP>(A.dinv + t);
            xv[u] = ld<KEEP>(x + t);
            pv[u] = ld<KEEP>(p + t);
            rv[u] = ld<KEEP>(r + t);
            wv[u] = w[t];
            own[u] = A.owner[t];
        }
        // keep the loads here (not sunk below the stop test): an empty use of each value
#pragma unroll
        for (int u = 0; u < UV; ++u)
            asm volatile("" ::"v"(di[u]), "v"(xv[u]), "v"(pv[u]), "v"(rv[u]), "v"(wv[u]), "v"((int)own[u]));
        asm volatile("" ::"s"(alpha), "s"(stop));
        if (!stop) {
#pragma unroll
            for (int u = 0; u < UV; ++u) {
                const int64_t t = t0 + (int64_t)u * VT;
                if (t >= A.n) break;
                stv<KEEP>(fma(alpha, pv[u], xv[u]), x + t);
                T ri = rv[u];
                if (di[u] != T(0)) {
                    ri = fma(-alpha, wv[u], ri);
                    stv<KEEP>(ri, r + t);
                }
                if (own[u]) {
                    rz += (double)ri * (double)(di[u] * ri);
                    rr += (double)ri * (double)ri;
                }
            }
        }
    } else {
        const CgScalars &sc = A.scal[f];
        if (!sc.stop) {
            const T alpha = (T)sc.alpha;
            const int64_t t0 = (int64_t)blockIdx.x * UV * VT;
            const int64_t t_end = min(A.n, t0 + (int64_t)UV * VT);
#pragma unroll
            for (int64_t t = t0 + threadIdx.x; t < t_end; t += VT) {
                const T di = ld<KEEP>(A.dinv + t);
                // unless KEEP, x, p, r and dinv are streamed (x is touched
                // only here; the others are next read a whole iteration later), so that
                // the last-level cache keeps w and the gather-scatter's index lists.
                if (A.x) stv<KEEP>(fma(alpha, ld<KEEP>(p + t), ld<KEEP>(x + t)), x + t);
                T ri = ld<KEEP>(r + t);
                if (di != T(0)) {
                    ri = fma(-alpha, w[t], ri);
                    stv<KEEP>(ri, r + t);
                }
                if (A.owner[t]) {
                    rz += (double)ri * (double)(di * ri);
                    rr += (double)ri * (double)ri;
                }
            }
        }
    }
    rz = wave_sum(rz);
    rr = wave_sum(rr);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) {
        sh[0][wave] = rz;
        sh[1][wave] = rr;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double a = 0.0, b = 0.0;
#pragma unroll
        for (int q = 0; q < VT / 64; ++q) {
            a += sh[0][q];
            b += sh[1][q];
        }
        A.partial[((int64_t)0 * A.nfields + f) * gridDim.x + blockIdx.x] = a;
        A.partial[((int64_t)1 * A.nfields + f) * gridDim.x + blockIdx.x] = b;
    }
}

// The same update with the gather-scatter of w inside it (A.pmap): every point sums the
// copies of its own value in the gather-scatter's order (the results are the same to the
// bit), so w is read once and never written back.  With NM > 0 every workgroup also sums the
// matvec's partials for the step length, NM a lane, while its operands are on their way: the
// iteration is then matvec, this, finish.  Small problems are bound by the latency of each
// launch's chain of loads, and this form takes out the gather-scatter's chain (6^3 points in
// 64 elements: 20.3 -> 16.8 us per iteration; 8^3 in 512: 25 -> 18.8).  On large ones it is
// bound by that chain too, scalars and index -> list -> copies -> stores, not by bandwidth
// (8^3 in 32768 elements: 5.1 TB/s in 207 us, against 145 + 66 us for update and
// gather-scatter).  All loads of one level are issued together for the GV points of a lane;
// lists are the gather-scatter's own entries, read four at a time: a fifth copy is rare.  Measured slower:
// one wave per chunk with the next index prefetched, GV = 1 and 4, index loads non-temporal,
// runs of 1, 64 and 256 chunks, one contiguous range per XCD.
// four consecutive entries of the gather-scatter's list, at any of them
struct __attribute__((packed, aligned(4))) List4 { uint32_t e[4]; };
constexpr int GATHER_NM = 1024;  // most partial sums of the matvec that it folds
template <typename T, int NM, bool KEEP>
__global__ __launch_bounds__(VT) void k_cg_update_gather(CgUpdateArgs<T> A, unsigned nblk, int run)
{
    constexpr int UV = UpdChunk<T>::GV;
    __shared__ double sh[2][VT / 64], sp[NM > 0 ? VT : 1];
    const int f = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // XCD x takes runs of 1 << run chunks, so that most copies of a point are in its own L2
    const unsigned i = blockIdx.x / 8, lb = (((i >> run) * 8 + blockIdx.x % 8) << run) + (i & ((1u << run) - 1));
    if (lb >= nblk) return;
    const int64_t off = f * A.n, t0 = (int64_t)lb * (UV * VT) + threadIdx.x;
    int32_t m[UV];
#pragma unroll
    for (int u = 0; u < UV; ++u) m[u] = A.pmap[min(t0 + (int64_t)u * VT, A.n - 1)];
    double pw = 0.0;
    if constexpr (NM > 0) {
        const double *mp = A.mpart + f * A.nm;
        double a[NM];
#pragma unroll
        for (int q = 0; q < NM; ++q) {
            const int64_t k = threadIdx.x + q * VT;
            a[q] = k < A.nm ? mp[k] : 0.0;
        }
        // (the order of block_sum_fixed<VT>, as in the gather-scatter's fold)
        const bool full = threadIdx.x + 3 * VT < A.nm;
        pw = full ? (a[0] + a[1]) + (a[2] + a[3]) : (a[0] + a[1]) + a[2];
        sp[threadIdx.x] = pw;
    }
    CgScalars &sc = A.scal[f];
    double rz = 0.0, rr = 0.0;
    if (NM > 0 && A.scal_out && sc.stop && lb == 0 && threadIdx.x == 0) A.scal_out[f] = sc;
    if (!sc.stop) {  // (no workgroup of this launch writes the flag: the barrier below is uniform)
        T *x = A.x + off, *r = A.r + off;
        const T *p = A.p + off, *w = A.w + off;
        T di[UV], xv[UV], pv[UV], rv[UV], v[UV][4];
        List4 g[UV];
#pragma unroll
        for (int u = 0; u < UV; ++u) {
            const int64_t t = min(t0 + (int64_t)u * VT, A.n - 1);
            v[u][0] = w[t];
            di[u] = ld<KEEP>(A.dinv + t);
            rv[u] = ld<KEEP>(r + t);
            xv[u] = pv[u] = T(0);
            if (A.x) {
                xv[u] = ld<KEEP>(x + t);
                pv[u] = ld<KEEP>(p + t);
            }
        }
#pragma unroll
        for (int u = 0; u < UV; ++u) {
            if (m[u] < -1) g[u] = *(const List4 *)(A.ent_word + ((-2 - m[u]) >> 5));
        }
#pragma unroll
        for (int u = 0; u < UV; ++u) {
            v[u][1] = T(0);
            if (m[u] >= 0) v[u][1] = w[m[u]];
        }
#pragma unroll
        for (int u = 0; u < UV; ++u) {
            v[u][2] = v[u][3] = T(0);
            if (m[u] < -1) {
                const int32_t o = -2 - m[u];
                v[u][0] = w[g[u].e[0] & 0x7fffffffu];
                v[u][1] = w[g[u].e[1] & 0x7fffffffu];
                v[u][2] = w[g[u].e[2] & 0x7fffffffu];
                if ((o & 31) >= 6) v[u][3] = w[g[u].e[3] & 0x7fffffffu];
            }
        }
        T alpha;
        bool ok = true;
        if constexpr (NM > 0) {
            __syncthreads();
            pw = (sp[lane] + sp[lane + 128]) + (sp[lane + 64] + sp[lane + 192]);
            pw = wave_sum(pw);
            const double rz0 = sc.rz;
            // every workgroup finds the same; on a breakdown none updates anything
            ok = pw > 0.0 && isfinite(pw) && isfinite(rz0);
            alpha = ok ? (T)(rz0 / pw) : T(0);
            if (lb == 0 && threadIdx.x == 0) {
                if (A.scal_out) {
                    CgScalars S = sc;
                    cg_set_alpha(S, pw);
                    S.primed = !S.stop;
                    A.scal_out[f] = S;
                } else if (ok) {
                    sc.alpha = rz0 / pw;
                } else {  // (cg_set_alpha but for the flag, which the finish sets)
                    sc.status = 2;
                    sc.alpha = 0.0;
                    sc.pend = 0;
                }
            }
        } else {
            alpha = (T)sc.alpha;
        }
        if (ok) {
#pragma unroll
            for (int u = 0; u < UV; ++u) {
                const int64_t t = t0 + (int64_t)u * VT;
                if (t >= A.n) break;
                T wi = v[u][0];
                bool own = true;
                if (m[u] >= 0) {
                    wi = (T(0) + wi) + v[u][1];  // (a sum of two is the same in either order)
                    own = t < m[u];
                } else if (m[u] < -1) {
                    const int32_t o = -2 - m[u], cnt = ((o >> 1) & 15) + 1;
                    own = o & 1;
                    wi = ((T(0) + wi) + v[u][1]) + v[u][2];
                    if (cnt > 3) wi += v[u][3];
                    for (int c = 4; c < cnt; c += 4) {
                        const List4 h = *(const List4 *)(A.ent_word + (o >> 5) + c);
                        T a[4];
#pragma unroll
                        for (int k = 0; k < 4; ++k) a[k] = w[c + k < cnt ? h.e[k] & 0x7fffffffu : (uint32_t)t];
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            if (c + k < cnt) wi += a[k];
                    }
                }
                if (A.x) stv<KEEP>(fma(alpha, pv[u], xv[u]), x + t);
                T ri = rv[u];
                if (di[u] != T(0)) {
                    ri = fma(-alpha, wi, ri);
                    stv<KEEP>(ri, r + t);
                }
                if (own) {
                    rz += (double)ri * (double)(di[u] * ri);
                    rr += (double)ri * (double)ri;
                }
            }
        }
    }
    rz = wave_sum(rz);
    rr = wave_sum(rr);
    if (lane == 0) {
        sh[0][wave] = rz;
        sh[1][wave] = rr;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        double a = 0.0;
#pragma unroll
        for (int q = 0; q < VT / 64; ++q) a += sh[threadIdx.x][q];
        A.partial[((int64_t)threadIdx.x * A.nfields + f) * nblk + lb] = a;
    }
}

// Assembly out of place: every point sums its copies from `in` (in the gather-scatter's
// order) and writes the masked sum, one pass where copy, gather-scatter and mask take three.
// A lane's points are VT apart and all fields share a point's index and flag; every load
// of one level is requested before the next.  4^3 to 8^3 elements: 18 us for the three calls,
// 8.6 for this one; 8^3 points in 32768 elements: 131 -> 121 us whether the operand is in the
// cache or not, 12^3 in 8000: 83 -> 82 from memory and 76 -> 79 from the cache, with three fields
// 303 -> 215.  The rate is that of the copies' separate cache requests (138
// points per ns at lx = 8, 177 at 12), not of memory: 1, 2 and 4 points a lane differ by 4%.
constexpr int ASM_V = 2;
template <typename T, int NF>
__global__ __launch_bounds__(VT) void k_assemble(AssembleArgs<T> A, unsigned nblk, int run)
{
    constexpr int AV = NF == 1 ? ASM_V : 1;
    const unsigned i = blockIdx.x / 8, lb = (((i >> run) * 8 + blockIdx.x % 8) << run) + (i & ((1u << run) - 1));
    if (lb >= nblk) return;
    const int64_t n = A.n, t0 = (int64_t)lb * (AV * VT) + threadIdx.x;
    int32_t m[AV];
    int dir[AV];
    T v[AV][NF][4];
    List4 g[AV];
#pragma unroll
    for (int u = 0; u < AV; ++u) m[u] = A.pmap[min(t0 + (int64_t)u * VT, n - 1)];
#pragma unroll
    for (int u = 0; u < AV; ++u) {
        const int64_t t = min(t0 + (int64_t)u * VT, n - 1);
        dir[u] = A.dir ? A.dir[t] : 0;
#pragma unroll
        for (int f = 0; f < NF; ++f) v[u][f][0] = A.in[f * n + t];
    }
#pragma unroll
    for (int u = 0; u < AV; ++u)
        if (m[u] < -1) g[u] = *(const List4 *)(A.ent_word + ((-2 - m[u]) >> 5));
#pragma unroll
    for (int u = 0; u < AV; ++u) {
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            v[u][f][1] = T(0);
            if (m[u] >= 0) v[u][f][1] = A.in[f * n + m[u]];
        }
    }
#pragma unroll
    for (int u = 0; u < AV; ++u) {
#pragma unroll
        for (int f = 0; f < NF; ++f) v[u][f][2] = v[u][f][3] = T(0);
        if (m[u] < -1) {
            const bool four = ((-2 - m[u]) & 31) >= 6;
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const T *in = A.in + f * n;
                v[u][f][0] = in[g[u].e[0] & 0x7fffffffu];
                v[u][f][1] = in[g[u].e[1] & 0x7fffffffu];
                v[u][f][2] = in[g[u].e[2] & 0x7fffffffu];
                if (four) v[u][f][3] = in[g[u].e[3] & 0x7fffffffu];
            }
        }
    }
#pragma unroll
    for (int u = 0; u < AV; ++u) {
        const int64_t t = t0 + (int64_t)u * VT;
        if (t >= n) break;
        T s[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f) s[f] = v[u][f][0];
        if (m[u] >= 0) {
#pragma unroll
            for (int f = 0; f < NF; ++f) s[f] = (T(0) + s[f]) + v[u][f][1];
        } else if (m[u] < -1) {
            const int32_t o = -2 - m[u], cnt = ((o >> 1) & 15) + 1;
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                s[f] = ((T(0) + s[f]) + v[u][f][1]) + v[u][f][2];
                if (cnt > 3) s[f] += v[u][f][3];
            }
            for (int c = 4; c < cnt; c += 4) {
                const List4 h = *(const List4 *)(A.ent_word + (o >> 5) + c);
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    T a[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        a[k] = A.in[f * n + (c + k < cnt ? (int64_t)(h.e[k] & 0x7fffffffu) : t)];
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        if (c + k < cnt) s[f] += a[k];
                }
            }
        }
#pragma unroll
        for (int f = 0; f < NF; ++f) A.out[f * n + t] = dir[u] ? T(0) : s[f];
    }
}

// x += alpha p of the last iteration for the fields that lack it (see CgMatvecArgs::x).
__global__ __launch_bounds__(VT) void k_cg_flush(double *x, const double *p, const CgScalars *scal, int64_t n)
{
    const int f = blockIdx.y;
    if (!scal[f].pend) return;
    const double alpha = scal[f].alpha;
    for (int64_t t = (int64_t)blockIdx.x * CHUNK + threadIdx.x, t_end = min(n, (int64_t)(blockIdx.x + 1) * CHUNK); t < t_end; t += VT)
        x[f * n + t] = fma(alpha, p[f * n + t], x[f * n + t]);
}

// Step lengths from the matvec's partial sums where they are too many for every workgroup
// of the update to add them up again, one workgroup per field: the additions of
// block_sum_fixed<VT> in the same order, with a lane for each of its four accumulators.
__global__ __launch_bounds__(RT) void k_cg_alpha(const double *part, int64_t nblk, CgScalars *scal)
{
    static_assert(RT == 4 * VT, "a lane per accumulator");
    __shared__ double sh[RT];
    const int tid = threadIdx.x, f = blockIdx.x, t = tid & (VT - 1);
    part += f * nblk;
    double a = 0.0;
    int64_t q = t;  // the first of this step's four entries
#pragma unroll 4
    for (; q + 3 * VT < nblk; q += RT) a += part[q + (tid - t)];
    if (tid < VT)
        for (; q < nblk; q += VT) a += part[q];
    sh[tid] = a;
    __syncthreads();
    if (tid < 64) {
        double s[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double *v = sh + tid + 64 * k;
            s[k] = (v[0] + v[VT]) + (v[2 * VT] + v[3 * VT]);
        }
        double pw = (s[0] + s[2]) + (s[1] + s[3]);
        pw = wave_sum(pw);
        if (tid == 0) cg_set_alpha(scal[f], pw);
    }
}

// Single-reduction CG update (Chronopoulos-Gear): with u = dinv r recomputed on the
// fly, p = u + beta p, s = w + beta s (s = A p carried as a vector), x += alpha p,
// r -= alpha s on non-Dirichlet points, and the partial sums of the new (r, dinv r)
// and (r, r) over owned points (per wave, then the waves in order).  They are
// reduced together with the next matvec's (u, A u): one reduction phase per iteration.
__global__ __launch_bounds__(VT) void k_cg1_update(Cg1UpdateArgs A)
{
    __shared__ double sh[2][VT / 64];
    const int f = blockIdx.y;
    const CgScalars &sc = A.scal[f];
    double rz = 0.0, rr = 0.0;
    if (!sc.stop) {
        const double alpha = sc.alpha, beta = sc.beta;
        double *x = A.x + f * A.n;
        double *r = A.r + f * A.n;
        double *p = A.p + f * A.n;
        double *s = A.s + f * A.n;
        const double *w = A.w + f * A.n;
        const int64_t t_end = min(A.n, (int64_t)(blockIdx.x + 1) * CHUNK);
#pragma unroll
        for (int64_t t = (int64_t)blockIdx.x * CHUNK + threadIdx.x; t < t_end; t += VT) {
            // every vector but w streamed non-temporally, as in the two-reduction update
            const double di = __builtin_nontemporal_load(A.dinv + t);
            double ri = __builtin_nontemporal_load(r + t);
            const double pn = fma(beta, __builtin_nontemporal_load(p + t), di * ri);
            const double sn = fma(beta, __builtin_nontemporal_load(s + t), w[t]);
            __builtin_nontemporal_store(pn, p + t);
            __builtin_nontemporal_store(sn, s + t);
            __builtin_nontemporal_store(fma(alpha, pn, __builtin_nontemporal_load(x + t)), x + t);
            if (di != 0.0) {
                ri = fma(-alpha, sn, ri);
                __builtin_nontemporal_store(ri, r + t);
            }
            if (A.owner[t]) {
                rz += ri * (di * ri);
                rr += ri * ri;
            }
        }
    }
    rz = wave_sum(rz);
    rr = wave_sum(rr);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) {
        sh[0][wave] = rz;
        sh[1][wave] = rr;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double a = 0.0, b = 0.0;
#pragma unroll
        for (int q = 0; q < VT / 64; ++q) {
            a += sh[0][q];
            b += sh[1][q];
        }
        A.partial[((int64_t)0 * A.nfields + f) * gridDim.x + blockIdx.x] = a;
        A.partial[((int64_t)1 * A.nfields + f) * gridDim.x + blockIdx.x] = b;
    }
}

// End of one CG iteration: beta = rz_new / rz_old, convergence and iteration cap.
// Two sums of nblk partials in one pass, fixed order: lane t accumulates entries
// t, t + NTH, ... of both arrays (four interleaved accumulators each, eight loads in
// flight), a sum per wave, then the NTH / 64 wave sums in order.  Every lane
// gets both results.
template <int NTH>
__device__ void block_sum2_fixed(const double *pa, const double *pb, int64_t nblk, double *sh, double &ra,
                                 double &rb)
{
    const int tid = threadIdx.x;
    double a[4] = {0.0, 0.0, 0.0, 0.0}, b[4] = {0.0, 0.0, 0.0, 0.0};
    int64_t q = tid;
    for (; q + 3 * NTH < nblk; q += 4 * NTH) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            a[u] += pa[q + u * NTH];
            b[u] += pb[q + u * NTH];
        }
    }
    for (; q < nblk; q += NTH) {
        a[0] += pa[q];
        b[0] += pb[q];
    }
    double x = (a[0] + a[1]) + (a[2] + a[3]), y = (b[0] + b[1]) + (b[2] + b[3]);
    x = wave_sum(x);
    y = wave_sum(y);
    if ((tid & 63) == 0) {
        sh[2 * (tid >> 6)] = x;
        sh[2 * (tid >> 6) + 1] = y;
    }
    __syncthreads();
    ra = 0.0;
    rb = 0.0;
#pragma unroll
    for (int w = 0; w < NTH / 64; ++w) {
        ra += sh[2 * w];
        rb += sh[2 * w + 1];
    }
    __syncthreads();
}

// One workgroup per field; a stopped field's sums are not read.
__global__ __launch_bounds__(RT) void k_cg_finish(CgFinishArgs A)
{
    __shared__ double sh[2 * (RT / 64)];
    const int f = blockIdx.x;
    CgScalars &s = A.scal[f];
    if (s.stop || (A.settle && !s.primed)) return;
    if (s.status == 2) {  // a breakdown that the update found (uniform: nothing wrote it here yet)
        __syncthreads();
        if (threadIdx.x == 0) s.stop = 1;
        return;
    }
    double rz, rr;
    block_sum2_fixed<RT>(A.partial + (0 * A.nfields + f) * A.nblk, A.partial + (1 * A.nfields + f) * A.nblk, A.nblk, sh,
                         rz, rr);
    if (threadIdx.x == 0) {
        cg_end_iteration(s, rz, rr);
        if (A.settle) s.primed = 0;
        if (A.hist && s.iter < A.hist_len) A.hist[(int64_t)f * A.hist_len + s.iter] = sqrt(rr / s.bb);
    }
}

// ------------------------------------------------------------------ reliable-update mixed CG
// Restart data for a new FP32 segment: the FP64 true residual b - w (0 on Dirichlet points;
// b itself for x = 0), rounded to FP32, the segment's zero iterate, and the partial sums of
// (r32, dinv r32), (r32, r32) and (r, r).  One pass: the FP64 residual is not stored, and w
// is gathered here (pmap) instead of by a gather-scatter before.  A workgroup takes REL_R
// rounds of VT points and all fields, which share the point's index, dinv and owner, so that
// few partial sums are left.  Three fields of 13.8M points at lx = 12: 281 us (4.1 TB/s of
// what it must move: the chain index -> entries -> copies bounds it, as in the gathering
// update), against 143 + 209 + 231 for the three passes that it stands for (gather-scatter;
// residual, stored in FP64; restart from it).  Chunks of 512 to 2048 points, runs of 4 or 16,
// the indices of all rounds loaded first: 275 to 306 us.
constexpr int REL_R = 8, REL_RUN = 4;
template <int NF, bool GA>
__global__ __launch_bounds__(VT) void k_rel_restart(RelRestartArgs A, unsigned nblk)
{
    __shared__ double sh[3 * NF][VT / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // XCD x takes runs of REL_RUN chunks, so that most copies of a point are in its own L2
    const unsigned i = blockIdx.x / 8, lb = (i / REL_RUN * 8 + blockIdx.x % 8) * REL_RUN + i % REL_RUN;
    if (lb >= nblk) return;
    const int64_t n = A.n, t0 = (int64_t)lb * (REL_R * VT) + threadIdx.x;
    bool live[NF];
    double acc[3 * NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        live[f] = !A.rel[f].done;
        acc[3 * f] = acc[3 * f + 1] = acc[3 * f + 2] = 0.0;
    }
#pragma unroll 1
    for (int q = 0; q < REL_R; ++q) {
        const int64_t t = t0 + q * VT;
        if (t >= n) break;
        const double di = __builtin_nontemporal_load(A.dinv + t);
        int32_t m = -1;
        if constexpr (GA) m = A.pmap[t];
        double rd[NF], wv[NF][4];
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            rd[f] = live[f] ? __builtin_nontemporal_load(A.b + f * n + t) : 0.0;
            wv[f][0] = live[f] && A.w ? A.w[f * n + t] : 0.0;
        }
        bool own = true;
        if constexpr (GA) {
            if (m >= 0) {
                own = t < m;
#pragma unroll
                for (int f = 0; f < NF; ++f)
                    if (live[f] && A.w) wv[f][0] = (0.0 + wv[f][0]) + A.w[f * n + m];
            } else if (m < -1) {
                const int32_t o = -2 - m, cnt = ((o >> 1) & 15) + 1;
                own = o & 1;
                double s[NF];
#pragma unroll
                for (int f = 0; f < NF; ++f) s[f] = 0.0;
                for (int c = 0; c < cnt && A.w; c += 4) {
                    const List4 h = *(const List4 *)(A.ent_word + (o >> 5) + c);
                    int64_t e[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) e[k] = c + k < cnt ? (int64_t)(h.e[k] & 0x7fffffffu) : t;
#pragma unroll
                    for (int f = 0; f < NF; ++f) {
                        if (!live[f]) continue;
#pragma unroll
                        for (int k = 0; k < 4; ++k) wv[f][k] = A.w[f * n + e[k]];
                    }
#pragma unroll
                    for (int f = 0; f < NF; ++f) {
                        if (!live[f]) continue;
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            if (c + k < cnt) s[f] += wv[f][k];
                    }
                }
#pragma unroll
                for (int f = 0; f < NF; ++f) wv[f][0] = s[f];
            }
        } else {
            own = A.owner[t] != 0;
        }
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            if (!live[f]) continue;
            const double r = A.w ? (di != 0.0 ? rd[f] - wv[f][0] : 0.0) : rd[f];
            const float ri = (float)r;
            __builtin_nontemporal_store(ri, A.r32 + f * n + t);
            __builtin_nontemporal_store(0.0f, A.x32 + f * n + t);
            if (A.p32) __builtin_nontemporal_store(0.0f, A.p32 + f * n + t);
            if (own) {
                acc[3 * f] += (double)ri * (double)((float)di * ri);
                acc[3 * f + 1] += (double)ri * (double)ri;
                acc[3 * f + 2] += r * r;
            }
        }
    }
#pragma unroll
    for (int k = 0; k < 3 * NF; ++k) {
        const double v = wave_sum(acc[k]);
        if (lane == 0) sh[k][wave] = v;
    }
    __syncthreads();
    if (threadIdx.x < 3 * NF) {
        double a = 0.0;
#pragma unroll
        for (int q = 0; q < VT / 64; ++q) a += sh[threadIdx.x][q];
        const int f = threadIdx.x / 3, k = threadIdx.x % 3;
        A.partial[((int64_t)k * NF + f) * nblk + lb] = a;
    }
}

// One workgroup per field: start (first = 1; with zero_x0 the residual is b) or resume an FP32 segment after a residual replacement.  The
// FP64 true residual decides convergence.  Resuming keeps the search direction p:
// beta is rescaled to the replaced residual, beta = (r_new, z_new) / (r_old, z_old).
// The segment stops once its residual has dropped by max(delta, half of the
// reduction still needed), at most 0.5.
__global__ __launch_bounds__(RT) void k_rel_resume(CgFinishArgs F, RelState *rel, int first, int zero_x0)
{
    __shared__ double sh[RT];
    const int f = blockIdx.x;
    const double rz = block_sum_fixed<RT>(F.partial + (0 * F.nfields + f) * F.nblk, F.nblk, sh);
    const double rr = block_sum_fixed<RT>(F.partial + (1 * F.nfields + f) * F.nblk, F.nblk, sh);
    const double r64 = block_sum_fixed<RT>(F.partial + (2 * F.nfields + f) * F.nblk, F.nblk, sh);
    if (threadIdx.x == 0) {
        RelState &R = rel[f];
        CgScalars &s = F.scal[f];
        if (R.done) return;
        if (zero_x0) R.bb64 = r64;
        R.rr64 = r64;
        R.outer += first ? 0 : 1;
        // the segment that just ended failed (breakdown) or used up the iterations
        if (!first && s.status != 0) {
            R.done = 1;
            s.stop = 1;
            return;
        }
        const double rel64 = R.bb64 > 0.0 ? sqrt(r64 / R.bb64) : 0.0;
        if (!isfinite(r64) || !isfinite(rz)) {
            R.done = 1;
            s.stop = 1;
            s.status = 2;
            return;
        }
        if (R.bb64 == 0.0 || rel64 <= R.tol) {
            R.done = 1;
            s.stop = 1;
            s.status = 0;
            return;
        }
        if (first) {
            s.beta = 0.0;
            s.iter = 0;
        } else {
            s.beta = (s.rz != 0.0) ? s.beta * (rz / s.rz) : 0.0;
            // a fast-converging system reaches delta within a few iterations:
            // ask for more reduction per segment so replacements stay rare
            if (s.iter - R.last_iter < 8) R.delta = fmax(R.delta * R.delta, 1e-3);
        }
        R.last_iter = s.iter;
        s.rz = rz;
        s.rr = rr;
        s.bb = rr;  // the segment's reference residual
        const double need = R.tol / rel64;
        s.rtol = fmin(0.5, fmax(R.delta, 0.5 * need));
        s.alpha = 0.0;
        s.status = 0;
        s.stop = 0;
        if (s.iter >= s.max_iter) {
            s.stop = 1;
            s.status = 1;
            R.done = 1;
        }
    }
}

// Residual replacement for a CG in precision T: partials of (r, dinv r) and (r, r)
// for a freshly recomputed residual r, on fields flagged in `redo`.
template <typename T>
__global__ __launch_bounds__(VT) void k_cg_replace(const T *r_all, const T *dinv, const uint8_t *owner,
                                                   const int *redo, double *partial, int64_t n, int nfields)
{
    __shared__ double sh[2][VT];
    const int f = blockIdx.y;
    double rz = 0.0, rr = 0.0;
    if (redo[f]) {
        const T *r = r_all + f * n;
        for (int64_t t = (int64_t)blockIdx.x * CHUNK + threadIdx.x, t_end = min(n, (int64_t)(blockIdx.x + 1) * CHUNK);
             t < t_end; t += VT) {
            if (owner[t]) {
                const T ri = r[t];
                rz += (double)ri * (double)(dinv[t] * ri);
                rr += (double)ri * (double)ri;
            }
        }
    }
    sh[0][threadIdx.x] = rz;
    sh[1][threadIdx.x] = rr;
    __syncthreads();
    for (int s = VT / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            sh[0][threadIdx.x] += sh[0][threadIdx.x + s];
            sh[1][threadIdx.x] += sh[1][threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0)
        for (int q = 0; q < 2; ++q) partial[((int64_t)q * nfields + f) * gridDim.x + blockIdx.x] = sh[q][0];
}

// Resume the CG of the fields flagged in `redo` after their residual was replaced:
// beta rescaled to the replaced residual, recursive norms reset, iteration continues
// (unless the iteration cap is reached).
__global__ __launch_bounds__(RT) void k_cg_resume(CgFinishArgs F, const int *redo)
{
    __shared__ double sh[RT];
    for (int f = 0; f < F.nfields; ++f) {
        const double rz = block_sum_fixed<RT>(F.partial + (0 * F.nfields + f) * F.nblk, F.nblk, sh);
        const double rr = block_sum_fixed<RT>(F.partial + (1 * F.nfields + f) * F.nblk, F.nblk, sh);
        if (threadIdx.x == 0) F.scal[f].pend = 0;  // x is complete at the end of a run
        if (threadIdx.x == 0 && redo[f]) {
            CgScalars &s = F.scal[f];
            s.beta = (s.rz != 0.0) ? s.beta * (rz / s.rz) : 0.0;
            s.rz = rz;
            s.rr = rr;
            if (!isfinite(rz) || !isfinite(rr)) {
                s.stop = 1;
                s.status = 2;
            } else if (s.iter >= s.max_iter) {
                s.stop = 1;
                s.status = 1;
            } else {
                s.stop = 0;
                s.status = 0;
            }
        }
    }
}

// x64 += (double) x32 on fields not done before this segment (done_before[f] == 0).
__global__ __launch_bounds__(VT) void k_add_f32(double *x64, const float *x32, const int *skip, int64_t n)
{
    const int f = blockIdx.y;
    if (skip[f]) return;
    for (int64_t t = (int64_t)blockIdx.x * CHUNK + threadIdx.x, t_end = min(n, (int64_t)(blockIdx.x + 1) * CHUNK);
         t < t_end; t += VT)
        x64[f * n + t] += (double)x32[f * n + t];
}

// ------------------------------------------------------------------ generic dots
// partial[q][f][block] for q in 0..nd-1: sum over owned points of a_q * b_q (FP64).
__global__ __launch_bounds__(VT) void k_dots(DotArgs A)
{
    __shared__ double sh[4][VT];
    const int f = blockIdx.y;
    double acc[4] = {0, 0, 0, 0};
    for (int64_t t = (int64_t)blockIdx.x * CHUNK + threadIdx.x, t_end = min((int64_t)(A.n), (int64_t)(blockIdx.x + 1) * CHUNK); t < t_end; t += VT) {
        if (!A.owner[t]) continue;
        for (int q = 0; q < A.nd; ++q) acc[q] += A.a[q][f * A.n + t] * A.b[q][f * A.n + t];
    }
    for (int q = 0; q < 4; ++q) sh[q][threadIdx.x] = acc[q];
    __syncthreads();
    for (int s = VT / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s)
            for (int q = 0; q < 4; ++q) sh[q][threadIdx.x] += sh[q][threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        for (int q = 0; q < A.nd; ++q)
            A.partial[((int64_t)q * A.nfields + f) * gridDim.x + blockIdx.x] = sh[q][0];
}

// out[q*nfields + f] = sum of partials, fixed order.
__global__ __launch_bounds__(RT) void k_dots_finish(const double *partial, int64_t nblk, int nq,
                                                     double *out)
{
    __shared__ double sh[RT];
    for (int q = 0; q < nq; ++q) {
        const double s = block_sum_fixed<RT>(partial + q * nblk, nblk, sh);
        if (threadIdx.x == 0) out[q] = s;
    }
}

// r = b - w masked (dinv == 0 marks Dirichlet points); used for true residuals.
__global__ __launch_bounds__(VT) void k_residual(double *r, const double *b, const double *w,
                                                 const double *dinv, int64_t n, int nfields)
{
    for (int64_t t = (int64_t)blockIdx.x * CHUNK + threadIdx.x, t_end = min((int64_t)(n), (int64_t)(blockIdx.x + 1) * CHUNK); t < t_end; t += VT) {
        const double di = dinv[t];
        for (int f = 0; f < nfields; ++f)
            r[f * n + t] = (di != 0.0) ? b[f * n + t] - w[f * n + t] : 0.0;
    }
}

// ------------------------------------------------------------------ flexible CG (outer, FP64)
// p = z - beta_f p   (beta_f from coef[f]);  fields with coef[f] flagged done are left alone.
__global__ __launch_bounds__(VT) void k_fcg_dir(double *p, const double *z, const double *beta,
                                                const int *done, int64_t n, int nfields)
{
    const int f = blockIdx.y;
    if (done[f]) return;
    const double bf = beta[f];
    for (int64_t t = (int64_t)blockIdx.x * CHUNK + threadIdx.x, t_end = min((int64_t)(n), (int64_t)(blockIdx.x + 1) * CHUNK); t < t_end; t += VT)
        p[f * n + t] = z[f * n + t] - bf * p[f * n + t];
}

// x += alpha p; r -= alpha q (not on Dirichlet points).
__global__ __launch_bounds__(VT) void k_fcg_update(double *x, double *r, const double *p,
                                                   const double *q, const double *dinv,
                                                   const double *alpha, const int *done, int64_t n,
                                                   int nfields)
{
    const int f = blockIdx.y;
    if (done[f]) return;
    const double a = alpha[f];
    for (int64_t t = (int64_t)blockIdx.x * CHUNK + threadIdx.x, t_end = min((int64_t)(n), (int64_t)(blockIdx.x + 1) * CHUNK); t < t_end; t += VT) {
        x[f * n + t] = fma(a, p[f * n + t], x[f * n + t]);
        if (dinv[t] != 0.0) r[f * n + t] = fma(-a, q[f * n + t], r[f * n + t]);
    }
}

// r32 = (float)(r / |r|_f)  per field (fields flagged done get 0).
__global__ __launch_bounds__(VT) void k_fcg_scale_down(float *r32, const double *r,
                                                       const double *inv_norm, const int *done,
                                                       int64_t n, int nfields)
{
    const int f = blockIdx.y;
    const double s = done[f] ? 0.0 : inv_norm[f];
    for (int64_t t = (int64_t)blockIdx.x * CHUNK + threadIdx.x, t_end = min((int64_t)(n), (int64_t)(blockIdx.x + 1) * CHUNK); t < t_end; t += VT)
        r32[f * n + t] = (float)(s * r[f * n + t]);
}

// z = |r|_f * (double) y32
__global__ __launch_bounds__(VT) void k_fcg_scale_up(double *z, const float *y32, const double *norm,
                                                     int64_t n, int nfields)
{
    const int f = blockIdx.y;
    const double s = norm[f];
    for (int64_t t = (int64_t)blockIdx.x * CHUNK + threadIdx.x, t_end = min((int64_t)(n), (int64_t)(blockIdx.x + 1) * CHUNK); t < t_end; t += VT)
        z[f * n + t] = s * (double)y32[f * n + t];
}

}  // namespace sem

// ------------------------------------------------------------------ host launchers
using namespace sem;

static unsigned stream_grid(int64_t n)
{
    const int64_t g = (n + CHUNK - 1) / CHUNK;
    return (unsigned)(g < 1 ? 1 : g);
}

static unsigned gs_grid(int64_t work)
{
    int64_t g = (work + VT - 1) / VT;
    if (g < 1) g = 1;
    return (unsigned)(8 * ((g + 7) / 8));  // multiple of 8: see the XCD mapping in k_gs
}

extern "C" {

unsigned sem_vec_grid(int64_t n) { return stream_grid(n); }
// workgroups of the CG update in precision f32 ? FP32 : FP64
unsigned sem_update_grid(int64_t n, int f32, int gather)
{
    const int64_t c = (int64_t)VT * (f32 ? (gather ? UpdChunk<float>::GV : UpdChunk<float>::UV)
                                         : (gather ? UpdChunk<double>::GV : UpdChunk<double>::UV));
    const int64_t g = (n + c - 1) / c;
    return (unsigned)(g < 1 ? 1 : g);
}
int64_t sem_gather_fold_max() { return GATHER_NM; }

}  // extern "C"

// Entry-parallel kernel for groups of up to 64 copies, then (rarely) the per-group
// kernel for larger groups.  The step-length fold runs in the first launch only.
template <typename T>
static hipError_t launch_gs_t(const GsArgs<T> *A, hipStream_t st)
{
    if (A->nent > 0) {
        hipLaunchKernelGGL(k_gs_entries<T>, dim3(gs_grid((A->nent + GEPL - 1) / GEPL)), dim3(VT), 0, st, *A);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess || A->npairs + A->nblocks == 0) return e;
        GsArgs<T> B = *A;
        B.alpha_job = nullptr;
        hipLaunchKernelGGL(k_gs<T>, dim3(gs_grid(B.npairs + B.nblocks)), dim3(VT), 0, st, B);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_gs<T>, dim3(gs_grid(A->npairs + A->nblocks)), dim3(VT), 0, st, *A);
    return hipGetLastError();
}
// Workgroups of the Arnoldi passes: contiguous chunks of whole 256-point rows, at
// most 1024 workgroups (four per CU), so the partial rows stay short.
static int64_t arn_chunk(int64_t n)
{
    const int64_t rows = (n + VT - 1) / VT;
    const int64_t per = (rows + SEM_ARN_G - 1) / SEM_ARN_G;
    const int64_t least = rows >= 256 * SEM_ARN_R ? SEM_ARN_R : 1;
    return (per < least ? least : per) * VT;
}
static unsigned arn_grid(int64_t n)
{
    const int64_t c = arn_chunk(n);
    const int64_t g = (n + c - 1) / c;
    return (unsigned)(g < 1 ? 1 : g);
}
template <typename T>
static hipError_t launch_gather(const CgUpdateArgs<T> *A, unsigned grid, hipStream_t st)
{
    if ((int64_t)grid * VT * UpdChunk<T>::GV < A->n) return hipErrorInvalidValue;
    if (A->nm > GATHER_NM || (A->nm > 0 && (!A->mpart || A->scal_out == A->scal))) return hipErrorInvalidValue;
    const int run = grid > 4096 ? 4 : 2;
    const unsigned per = 8u << run;
    const dim3 g((grid + per - 1) / per * per, A->nfields);
    constexpr int NM = GATHER_NM / VT;
    if (A->keep) {
        if (A->nm == 0) hipLaunchKernelGGL((k_cg_update_gather<T, 0, true>), g, dim3(VT), 0, st, *A, grid, run);
        else hipLaunchKernelGGL((k_cg_update_gather<T, NM, true>), g, dim3(VT), 0, st, *A, grid, run);
    } else {
        if (A->nm == 0) hipLaunchKernelGGL((k_cg_update_gather<T, 0, false>), g, dim3(VT), 0, st, *A, grid, run);
        else hipLaunchKernelGGL((k_cg_update_gather<T, NM, false>), g, dim3(VT), 0, st, *A, grid, run);
    }
    return hipGetLastError();
}
template <typename T>
static hipError_t launch_assemble(const AssembleArgs<T> *A, hipStream_t st)
{
    if (A->n == 0) return hipSuccess;
    if ((A->nfields != 1 && A->nfields != 3) || !A->pmap) return hipErrorInvalidValue;
    const int64_t c = (int64_t)VT * (A->nfields == 1 ? ASM_V : 1), nb = (A->n + c - 1) / c;
    const int run = nb > 4096 ? 4 : 2;
    const int64_t per = 8 << run;
    const dim3 g((unsigned)((nb + per - 1) / per * per));
    if (A->nfields == 1) hipLaunchKernelGGL((k_assemble<T, 1>), g, dim3(VT), 0, st, *A, (unsigned)nb, run);
    else hipLaunchKernelGGL((k_assemble<T, 3>), g, dim3(VT), 0, st, *A, (unsigned)nb, run);
    return hipGetLastError();
}
template <int MV>
static void launch_dcgs(const DcgsArgs &A, int pass, hipStream_t st)
{
    const unsigned g = arn_grid(A.n);
    const int64_t c = arn_chunk(A.n);
    if (pass == 0) hipLaunchKernelGGL((k_dcgs_dots<MV>), dim3(g), dim3(VT), 0, st, A, c);
    else hipLaunchKernelGGL((k_dcgs_update<MV>), dim3(g), dim3(VT), 0, st, A, c);
}
template <int MV>
static void launch_arn(const ArnArgs &A, int mode, hipStream_t st)
{
    const unsigned g = arn_grid(A.n);
    const int64_t c = arn_chunk(A.n);
    if (mode == 0) hipLaunchKernelGGL((k_arn<MV, 0>), dim3(g), dim3(VT), 0, st, A, c);
    else if (mode == 1) hipLaunchKernelGGL((k_arn<MV, 1>), dim3(g), dim3(VT), 0, st, A, c);
    else hipLaunchKernelGGL((k_arn<MV, 2>), dim3(g), dim3(VT), 0, st, A, c);
}
extern "C" {
hipError_t sem_launch_gs_f64(const GsArgs<double> *A, hipStream_t st) { return launch_gs_t<double>(A, st); }
hipError_t sem_launch_gs_f32(const GsArgs<float> *A, hipStream_t st) { return launch_gs_t<float>(A, st); }
hipError_t sem_launch_mask(void *u, int is_f32, const int32_t *idx, int64_t m, int64_t n, int nfields,
                           hipStream_t st)
{
    if (m == 0) return hipSuccess;
    const unsigned grid = (unsigned)((m + VT - 1) / VT);
    if (is_f32)
        hipLaunchKernelGGL(k_mask<float>, dim3(grid), dim3(VT), 0, st, (float *)u, idx, m, n, nfields);
    else
        hipLaunchKernelGGL(k_mask<double>, dim3(grid), dim3(VT), 0, st, (double *)u, idx, m, n, nfields);
    return hipGetLastError();
}
hipError_t sem_launch_fill_f64(double *u, double v, int64_t m, hipStream_t st)
{
    if (m == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill<double>, dim3(stream_grid(m)), dim3(VT), 0, st, u, v, m);
    return hipGetLastError();
}
hipError_t sem_launch_fill_f32(float *u, float v, int64_t m, hipStream_t st)
{
    if (m == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill<float>, dim3(stream_grid(m)), dim3(VT), 0, st, u, v, m);
    return hipGetLastError();
}
hipError_t sem_launch_cast_f32_f64(float *dst, const double *src, double scale, int64_t m, hipStream_t st)
{
    if (m == 0) return hipSuccess;
    hipLaunchKernelGGL((k_cast<float, double>), dim3(stream_grid(m)), dim3(VT), 0, st, dst, src, scale, m);
    return hipGetLastError();
}
hipError_t sem_launch_triad(double *a, const double *b, const double *c, double s, int64_t n, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_triad, dim3(stream_grid(n)), dim3(VT), 0, st, a, b, c, s, n);
    return hipGetLastError();
}
hipError_t sem_launch_invert(double *d, const uint8_t *dir, int64_t n, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_invert, dim3((unsigned)((n + VT - 1) / VT)), dim3(VT), 0, st, d, dir, n);
    return hipGetLastError();
}
hipError_t sem_launch_cg_init_f64(const CgInitArgs<double> *A, unsigned grid, hipStream_t st)
{
    hipLaunchKernelGGL(k_cg_init<double>, dim3(grid, A->nfields), dim3(VT), 0, st, *A);
    return hipGetLastError();
}
hipError_t sem_launch_cg_init_f32(const CgInitArgs<float> *A, unsigned grid, hipStream_t st)
{
    hipLaunchKernelGGL(k_cg_init<float>, dim3(grid, A->nfields), dim3(VT), 0, st, *A);
    return hipGetLastError();
}
hipError_t sem_launch_cg_start(const CgFinishArgs *A, hipStream_t st)
{
    hipLaunchKernelGGL(k_cg_start, dim3(1), dim3(RT), 0, st, *A);
    return hipGetLastError();
}
hipError_t sem_launch_cg_update_f64(const CgUpdateArgs<double> *A, unsigned grid, hipStream_t st)
{
    if (A->pmap) return launch_gather<double>(A, grid, st);
    if ((int64_t)grid * VT * UpdChunk<double>::UV < A->n) return hipErrorInvalidValue;
    if (A->keep) hipLaunchKernelGGL((k_cg_update<double, true>), dim3(grid, A->nfields), dim3(VT), 0, st, *A);
    else hipLaunchKernelGGL((k_cg_update<double, false>), dim3(grid, A->nfields), dim3(VT), 0, st, *A);
    return hipGetLastError();
}
hipError_t sem_launch_cg_update_f32(const CgUpdateArgs<float> *A, unsigned grid, hipStream_t st)
{
    if (A->pmap) return launch_gather<float>(A, grid, st);
    if ((int64_t)grid * VT * UpdChunk<float>::UV < A->n) return hipErrorInvalidValue;
    if (A->keep) hipLaunchKernelGGL((k_cg_update<float, true>), dim3(grid, A->nfields), dim3(VT), 0, st, *A);
    else hipLaunchKernelGGL((k_cg_update<float, false>), dim3(grid, A->nfields), dim3(VT), 0, st, *A);
    return hipGetLastError();
}
hipError_t sem_launch_assemble_f64(const AssembleArgs<double> *A, hipStream_t st) { return launch_assemble(A, st); }
hipError_t sem_launch_assemble_f32(const AssembleArgs<float> *A, hipStream_t st) { return launch_assemble(A, st); }
hipError_t sem_launch_gather_map(const uint32_t *ent_word, int64_t nent, const uint8_t *owner, int32_t *pmap, int64_t n,
                                 hipStream_t st)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill<int32_t>, dim3(stream_grid(n)), dim3(VT), 0, st, pmap, -1, n);
    if (nent > 0)
        hipLaunchKernelGGL(k_gather_map, dim3((unsigned)((nent + VT - 1) / VT)), dim3(VT), 0, st, ent_word, nent, owner,
                           pmap);
    return hipGetLastError();
}
hipError_t sem_launch_cg_alpha(const double *partial, int64_t nblk, CgScalars *scal, int nfields, hipStream_t st)
{
    hipLaunchKernelGGL(k_cg_alpha, dim3(nfields), dim3(RT), 0, st, partial, nblk, scal);
    return hipGetLastError();
}
hipError_t sem_launch_cg_flush(double *x, const double *p, const CgScalars *scal, int64_t n, int nf, hipStream_t st)
{
    hipLaunchKernelGGL(k_cg_flush, dim3(stream_grid(n), nf), dim3(VT), 0, st, x, p, scal, n);
    return hipGetLastError();
}
hipError_t sem_launch_cg1_update(const Cg1UpdateArgs *A, hipStream_t st)
{
    if (A->n == 0) return hipSuccess;
    if (!A->owner || !A->partial) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_cg1_update, dim3(stream_grid(A->n), A->nfields), dim3(VT), 0, st, *A);
    return hipGetLastError();
}
hipError_t sem_launch_cg_finish(const CgFinishArgs *A, hipStream_t st)
{
    hipLaunchKernelGGL(k_cg_finish, dim3(A->nfields), dim3(RT), 0, st, *A);
    return hipGetLastError();
}
unsigned sem_rel_grid(int64_t n)
{
    const int64_t c = (int64_t)VT * REL_R, g = (n + c - 1) / c;
    return (unsigned)(g < 1 ? 1 : g);
}
hipError_t sem_launch_rel_restart(const RelRestartArgs *A, hipStream_t st)
{
    const unsigned nb = sem_rel_grid(A->n), per = 8 * REL_RUN;
    const dim3 g((nb + per - 1) / per * per);
    if (A->nfields != 1 && A->nfields != 3) return hipErrorInvalidValue;
    if (A->nfields == 1) {
        if (A->pmap) hipLaunchKernelGGL((k_rel_restart<1, true>), g, dim3(VT), 0, st, *A, nb);
        else hipLaunchKernelGGL((k_rel_restart<1, false>), g, dim3(VT), 0, st, *A, nb);
    } else {
        if (A->pmap) hipLaunchKernelGGL((k_rel_restart<3, true>), g, dim3(VT), 0, st, *A, nb);
        else hipLaunchKernelGGL((k_rel_restart<3, false>), g, dim3(VT), 0, st, *A, nb);
    }
    return hipGetLastError();
}
hipError_t sem_launch_rel_resume(const CgFinishArgs *F, RelState *rel, int first, int zero_x0, hipStream_t st)
{
    hipLaunchKernelGGL(k_rel_resume, dim3(F->nfields), dim3(RT), 0, st, *F, rel, first, zero_x0);
    return hipGetLastError();
}
hipError_t sem_launch_add_f32(double *x64, const float *x32, const int *skip, int64_t n, int nfields,
                              hipStream_t st)
{
    hipLaunchKernelGGL(k_add_f32, dim3(stream_grid(n), nfields), dim3(VT), 0, st, x64, x32, skip, n);
    return hipGetLastError();
}
hipError_t sem_launch_cg_replace_f64(const double *r, const double *dinv, const uint8_t *owner, const int *redo,
                                     double *partial, int64_t n, int nfields, hipStream_t st)
{
    hipLaunchKernelGGL(k_cg_replace<double>, dim3(stream_grid(n), nfields), dim3(VT), 0, st, r, dinv, owner, redo,
                       partial, n, nfields);
    return hipGetLastError();
}
hipError_t sem_launch_cg_resume(const CgFinishArgs *F, const int *redo, hipStream_t st)
{
    hipLaunchKernelGGL(k_cg_resume, dim3(1), dim3(RT), 0, st, *F, redo);
    return hipGetLastError();
}
hipError_t sem_launch_comb(const CombArgs *A, hipStream_t st)
{
    if (A->l < 0 || A->l > PB || A->mode < 0 || A->mode > 2) return hipErrorInvalidValue;
    if (A->n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_comb, dim3(stream_grid(A->n)), dim3(VT), 0, st, *A);
    return hipGetLastError();
}
unsigned sem_arn_grid(int64_t n) { return arn_grid(n); }
hipError_t sem_launch_dcgs(const DcgsArgs *A, int pass, hipStream_t st)
{
    if (A->j < 0 || A->j >= ARN_MAXV || pass < 0 || pass > 1 || A->n < 1) return hipErrorInvalidValue;
    if (pass == 1 && !A->coef) return hipErrorInvalidValue;
    if (A->j <= 4) launch_dcgs<4>(*A, pass, st);
    else if (A->j <= 8) launch_dcgs<8>(*A, pass, st);
    else if (A->j <= 12) launch_dcgs<12>(*A, pass, st);
    else if (A->j <= 16) launch_dcgs<16>(*A, pass, st);
    else if (A->j <= 24) launch_dcgs<24>(*A, pass, st);
    else launch_dcgs<32>(*A, pass, st);
    return hipGetLastError();
}
hipError_t sem_launch_dcgs_finish(const double *partial, int64_t nblk, int j, double *out, hipStream_t st)
{
    if (j < 0 || j >= ARN_MAXV) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_dcgs_finish, dim3(1), dim3(RT), 0, st, partial, nblk, j, out);
    return hipGetLastError();
}
hipError_t sem_launch_arn(const ArnArgs *A, int mode, hipStream_t st)
{
    if (A->m < 1 || A->m > ARN_MAXV || mode < 0 || mode > 2 || A->n < 1) return hipErrorInvalidValue;
    if (mode != 0 && !A->coef) return hipErrorInvalidValue;
    if (mode == 2 && !A->scale) return hipErrorInvalidValue;
    if (A->m <= 4) launch_arn<4>(*A, mode, st);
    else if (A->m <= 8) launch_arn<8>(*A, mode, st);
    else if (A->m <= 12) launch_arn<12>(*A, mode, st);
    else if (A->m <= 16) launch_arn<16>(*A, mode, st);
    else if (A->m <= 24) launch_arn<24>(*A, mode, st);
    else launch_arn<32>(*A, mode, st);
    return hipGetLastError();
}
hipError_t sem_launch_arn_finish(const double *partial, int64_t nblk, int nq, int pyth, double *out, hipStream_t st)
{
    if (nq < 1 || nq > ARN_MAXV + 1 || (pyth && nq < 2)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_arn_finish, dim3(1), dim3(RT), 0, st, partial, nblk, nq, pyth, out);
    return hipGetLastError();
}
hipError_t sem_launch_hadamard(double *y, const double *a, const double *b, int64_t n, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_hadamard, dim3(stream_grid(n)), dim3(VT), 0, st, y, a, b, n);
    return hipGetLastError();
}
hipError_t sem_launch_corner(const CornerArgs *A, hipStream_t st)
{
    if (A->nelv == 0) return hipSuccess;
    if (A->nelv > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_corner, dim3((unsigned)A->nelv), dim3(VT), 0, st, *A);
    return hipGetLastError();
}
// workgroups of k_ccg_step
static int64_t ccg_grid(int64_t nv) { return (nv * SPL + VT - 1) / VT; }
// doubles of the coarse solve's vectors (x, p, two record arrays) and of its partial
// sums and scalars
int64_t sem_coarse_words(int64_t nv) { return 10 * nv; }
int64_t sem_coarse_partials(int64_t nv) { return 4 * ccg_grid(nv) + 4; }

// iters fixed-count Jacobi-CG steps on the coarse system from x = 0, no host sync, with the
// gather-scatter G of z (one field, no skip, no job) in the same launches where it can be.
hipError_t sem_launch_coarse_cg(const CoarseArgs *A, int iters, const GsArgs<double> *G, hipStream_t st)
{
    if (A->width < 1 || A->nv > 0x7fffffffLL || G->nfields != 1 || G->skip || G->alpha_job) return hipErrorInvalidValue;
    unsigned nb = G->nent > 0 ? gs_grid((G->nent + GEPL - 1) / GEPL) : 0;
    // points of more than 64 copies, or no coarse system: a launch of its own
    if (A->nv == 0 || G->npairs + G->nblocks > 0) {
        if (G->npairs + G->nblocks + G->nent > 0) {
            const hipError_t e = launch_gs_t<double>(G, st);
            if (e != hipSuccess || A->nv == 0) return e;
        }
        if (A->nv == 0) return hipSuccess;
        nb = 0;
    }
    if (iters > 0 && A->nv <= CCG_SMALL && A->width <= RESW) {
        const dim3 g(1 + (nb * VT + CST - 1) / CST);
        if (A->nv <= CST) hipLaunchKernelGGL(k_ccg_small<1>, g, dim3(CST), 0, st, *A, iters, *G);
        else if (A->nv <= 2 * CST) hipLaunchKernelGGL(k_ccg_small<2>, g, dim3(CST), 0, st, *A, iters, *G);
        else hipLaunchKernelGGL(k_ccg_small<3>, g, dim3(CST), 0, st, *A, iters, *G);
        return hipGetLastError();
    }
    const int launches = 2 + iters;  // start, iters steps, the last update
    auto slice = [&](int k) {
        auto at = [&](int q) { return (unsigned)((int64_t)(nb / 8) * q / launches) * 8; };
        return iters > 0 ? GsSlice{*G, at(k), at(k + 1), nb} : GsSlice{*G, 0, nb, nb};
    };
    {
        const GsSlice S = slice(0);
        const unsigned nc = (unsigned)((A->nv + VT - 1) / VT);
        hipLaunchKernelGGL(k_ccg_start, dim3(nc + (S.hi - S.lo)), dim3(VT), 0, st, *A, nc, S);
    }
    for (int it = 0; it <= iters && iters > 0; ++it) {
        const GsSlice S = slice(1 + it);
        const unsigned nc = (unsigned)ccg_grid(A->nv);
        hipLaunchKernelGGL(k_ccg_step, dim3(nc + (S.hi - S.lo)), dim3(VT), 0, st, *A, it, it == iters ? 1 : 0, nc, S);
    }
    return hipGetLastError();
}
hipError_t sem_launch_elem_gb(const double *G, const double *B, double *out, int64_t nelv, int lx3,
                              hipStream_t st)
{
    if (nelv == 0) return hipSuccess;
    if (nelv > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_elem_gb, dim3((unsigned)nelv), dim3(VT), 0, st, G, B, out, nelv * lx3, lx3);
    return hipGetLastError();
}
hipError_t sem_launch_probe(double *v, const double *phi, int c, int64_t nelv, int lx3, hipStream_t st)
{
    const int64_t n = nelv * lx3;
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_probe, dim3((unsigned)((n + VT - 1) / VT)), dim3(VT), 0, st, v, phi, c, nelv, lx3);
    return hipGetLastError();
}
hipError_t sem_launch_dots(const DotArgs *A, unsigned grid, hipStream_t st)
{
    hipLaunchKernelGGL(k_dots, dim3(grid, A->nfields), dim3(VT), 0, st, *A);
    return hipGetLastError();
}
hipError_t sem_launch_dots_finish(const double *partial, int64_t nblk, int nq, double *out, hipStream_t st)
{
    hipLaunchKernelGGL(k_dots_finish, dim3(1), dim3(RT), 0, st, partial, nblk, nq, out);
    return hipGetLastError();
}
hipError_t sem_launch_residual(double *r, const double *b, const double *w, const double *dinv,
                               int64_t n, int nfields, hipStream_t st)
{
    hipLaunchKernelGGL(k_residual, dim3(stream_grid(n)), dim3(VT), 0, st, r, b, w, dinv, n, nfields);
    return hipGetLastError();
}
hipError_t sem_launch_fcg_dir(double *p, const double *z, const double *beta, const int *done,
                              int64_t n, int nfields, hipStream_t st)
{
    hipLaunchKernelGGL(k_fcg_dir, dim3(stream_grid(n), nfields), dim3(VT), 0, st, p, z, beta, done, n, nfields);
    return hipGetLastError();
}
hipError_t sem_launch_fcg_update(double *x, double *r, const double *p, const double *q,
                                 const double *dinv, const double *alpha, const int *done,
                                 int64_t n, int nfields, hipStream_t st)
{
    hipLaunchKernelGGL(k_fcg_update, dim3(stream_grid(n), nfields), dim3(VT), 0, st, x, r, p, q, dinv,
                       alpha, done, n, nfields);
    return hipGetLastError();
}
hipError_t sem_launch_fcg_scale_down(float *r32, const double *r, const double *inv_norm,
                                     const int *done, int64_t n, int nfields, hipStream_t st)
{
    hipLaunchKernelGGL(k_fcg_scale_down, dim3(stream_grid(n), nfields), dim3(VT), 0, st, r32, r,
                       inv_norm, done, n, nfields);
    return hipGetLastError();
}
hipError_t sem_launch_fcg_scale_up(double *z, const float *y32, const double *norm, int64_t n,
                                   int nfields, hipStream_t st)
{
    hipLaunchKernelGGL(k_fcg_scale_up, dim3(stream_grid(n), nfields), dim3(VT), 0, st, z, y32, norm,
                       n, nfields);
    return hipGetLastError();
}

}  // extern "C"

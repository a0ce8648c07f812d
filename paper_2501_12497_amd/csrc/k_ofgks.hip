// Solve-OF (Alg. 2), p = q = 2 and p = q = 1: per frame pair, the flow s minimising
//   ||Y s + u_t||^2 + lambda ||L s||^2,  Y = [diag(I_x) diag(I_y)],  L = blockdiag(D, D)
// (eq. subproblem_motion_estimation_redefined) by the generalized Krylov subspace method
// (MMGKS with unit weights): ell Golub-Kahan steps on Y from b = -u_t, then n_iter projected
// solves, each with lambda chosen by generalized cross-validation (eq. gcv_functional) on the
// projected solution and the basis grown by the orthogonalised residual.
//
// One workgroup per pair runs the whole solve in FP64: the basis and the Golub-Kahan left
// vectors live in global memory (workspace of the caller), the Gram matrices (Y V)^T Y V and
// (L V)^T L V, (Y V)^T b and the per-wave factorizations of the GCV search in LDS.  The Gram
// matrices grow by one row per iteration; Y V and L V are never stored (Y is diagonal per
// pixel and L a two-point stencil, so their entries are formed from V on the fly).
//
// GCV: G(lambda) = ||Y V z - b||^2 / (m - trace(M^-1 G_Y))^2 with M = G_Y + lambda G_L and
// m the pixels of the pair; the numerator is ||b||^2 - 2 z.d + z^T G_Y z.  The search over
// x = log10 lambda: 32 points evenly over c + [-12, 12], c = log10(tr G_Y / tr G_L), then 5
// refinements of 8 points evenly over [x* - h, x* + h] around the best point so far (h the
// previous spacing); scanned in increasing x, a point wins only when it lowers G by more than
// a relative 1e-9 (closer values are ties, the earlier point stays, so that the choice does
// not depend on rounding where G is flat); a factorization that fails gives G = inf.  A wave
// evaluates four points at a time, one per 16 lanes, with the factor in registers (GcvFactor);
// where G_Y itself has no Cholesky factor, one point at a time in LDS (gcv_eval).
//
// The p = q = 1 variant (MMGKS on the smoothed l1 norms of the data rows and of the flow
// differences): before every projected solve the weights of the current iterate are formed
// per pixel (one data weight, four edge weights stored at an edge's left / upper pixel), the
// weighted Gram matrices, d and b^T W_d b are built from scratch, and GCV, z and the residual
// are those of the weighted problem.
#include <type_traits>

#include "dev.h"
#include "kernels.h"

namespace mmof {

namespace {

constexpr int GK_THREADS = 512;
constexpr int GK_WAVES = GK_THREADS / 64;
constexpr int GK_KC = 32;         // basis capacity (ell + n_iter - 1)
constexpr int GK_P = GK_KC + 1;   // padded LDS row stride of the factorization buffers
constexpr int GK_GRID0 = 32, GK_REFINE = 5, GK_GRIDR = 8;
constexpr double GK_SPAN = 12.0;
constexpr double GK_TIE = 1e-9;   // relative improvement of G a later grid point needs to win
constexpr int GK_RMAX = 2;        // largest workgroup sum

struct GksLds {
    double GA[GK_KC * GK_KC];     // (Y V)^T Y V
    double GL[GK_KC * GK_KC];     // (L V)^T L V
    double d[GK_KC];              // (Y V)^T b
    double z[GK_KC];
    double z0[GK_KC];             // the unregularised projected solution G_Y^-1 d
    double h[2 * GK_KC];          // Gram-Schmidt coefficients; inner products with one or two vectors
    double C[GK_KC * GK_P];       // the Cholesky factor of G_Y (lower, zeros above)
    double y0[GK_KC];             // C^-1 d
    int c_ok;                     // C and z0 exist
    double M[GK_WAVES][GK_KC * GK_P];
    double X[GK_WAVES][GK_KC * GK_P];
    double part[GK_WAVES * GK_RMAX];
    double tot[GK_RMAX];
    double gval[GK_GRID0], gxv[GK_GRID0];
};

// Orders a wave's LDS writes before its later LDS reads by other lanes of the same wave.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    return v;  // identical on every lane (each butterfly step adds the same two values)
}

// Workgroup sums of a[0..NV): fixed order (lanes by butterfly, then waves in order); the
// totals land in s.tot[0..NV) and in a.
template <int NV>
__device__ void wg_sum(double (&a)[NV], GksLds& s) {
    static_assert(NV <= GK_RMAX, "workgroup sum too wide");
    __syncthreads();  // earlier readers of s.tot are done
    const int w = threadIdx.x / 64, lane = threadIdx.x % 64;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const double v = wave_sum(a[j]);
        if (lane == 0) s.part[w * NV + j] = v;
    }
    __syncthreads();
    if (threadIdx.x < NV) {
        double t = s.part[threadIdx.x];
        for (int q = 1; q < GK_WAVES; ++q) t += s.part[q * NV + threadIdx.x];
        s.tot[threadIdx.x] = t;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NV; ++j) a[j] = s.tot[j];
}

// Inner products of columns 0..ncols-1 of Q (stride len) with x0 and, for NX = 2, with x1:
// s.h[c] = Q_c^T x0, s.h[GK_KC + c] = Q_c^T x1.  Each wave takes whole columns, up to four side by
// side: one butterfly per column and vector, where columns split over the workgroup would cost
// one per wave (the sums are latency: a 32 x 32 pair has 4 elements per thread and column).
// VEC = 2: 16-byte loads (the columns of V, whose length is even; the left vectors of odd
// frames take single loads).  The address is aligned to one element only: a pair's left vectors start
// (ell + 1) times the pixels of the pairs before it into their array, which may be an odd number.
template <int VEC>
struct GkVecOf {
    typedef double type __attribute__((ext_vector_type(VEC), aligned(sizeof(double))));
};
template <int VEC>
using GkVec = typename GkVecOf<VEC>::type;
static_assert(alignof(GkVec<2>) == alignof(double), "addresses of one element's alignment");

template <int NX, int NC, int VEC>
__device__ __forceinline__ void wave_dots(const double* __restrict__ Q, int64_t len, int c0,
                                          const double* __restrict__ x0, const double* __restrict__ x1, GksLds& s) {
    using VT = GkVec<VEC>;
    const int lane = threadIdx.x % 64;
    double a[NX][NC];
#pragma unroll
    for (int v = 0; v < NX; ++v)
#pragma unroll
        for (int c = 0; c < NC; ++c) a[v][c] = 0.0;
    const double* q = Q + (int64_t)c0 * len;
#pragma unroll 4
    for (int64_t p = VEC * lane; p < len; p += 64 * VEC) {
        const VT xa = *reinterpret_cast<const VT*>(x0 + p);
        VT xb = xa;
        if constexpr (NX == 2) xb = *reinterpret_cast<const VT*>(x1 + p);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const VT qv = *reinterpret_cast<const VT*>(q + (int64_t)c * len + p);
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                a[0][c] = fma(qv[e], xa[e], a[0][c]);
                if constexpr (NX == 2) a[1][c] = fma(qv[e], xb[e], a[1][c]);
            }
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1)
#pragma unroll
        for (int v = 0; v < NX; ++v)
#pragma unroll
            for (int c = 0; c < NC; ++c) a[v][c] += __shfl_xor(a[v][c], o);
    if (lane == 0) {
#pragma unroll
        for (int v = 0; v < NX; ++v)
#pragma unroll
            for (int c = 0; c < NC; ++c) s.h[v * GK_KC + c0 + c] = a[v][c];
    }
}

template <int NX, int VEC>
__device__ void wg_dots(const double* Q, int64_t len, int ncols, const double* x0, const double* x1, GksLds& s) {
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int per = (ncols + GK_WAVES - 1) / GK_WAVES;  // at most 4 (GK_KC = 4 GK_WAVES)
    const int c0 = w * per, nc = min(per, ncols - c0);
    if (nc == 4) wave_dots<NX, 4, VEC>(Q, len, c0, x0, x1, s);
    else if (nc == 3) wave_dots<NX, 3, VEC>(Q, len, c0, x0, x1, s);
    else if (nc == 2) wave_dots<NX, 2, VEC>(Q, len, c0, x0, x1, s);
    else if (nc == 1) wave_dots<NX, 1, VEC>(Q, len, c0, x0, x1, s);
    __syncthreads();
}

// Sum over the first ncols columns of Q (stride len), with the coefficients h, of the VEC
// elements at p: eight columns' loads in flight ahead of the ordered sum.
template <int VEC>
__device__ __forceinline__ GkVec<VEC> combine(const double* __restrict__ Q, int64_t len, int ncols, const double* h,
                                              int64_t p) {
    using VT = GkVec<VEC>;
    VT acc = VT(0.0);
    int c = 0;
    for (; c + 8 <= ncols; c += 8) {
        VT q[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) q[e] = *reinterpret_cast<const VT*>(Q + (int64_t)(c + e) * len + p);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc += h[c + e] * q[e];
    }
    if (c < ncols) {  // (a column past the last is read as the last and left out)
        VT q[8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            q[e] = *reinterpret_cast<const VT*>(Q + (int64_t)min(c + e, ncols - 1) * len + p);
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (c + e < ncols) acc += h[c + e] * q[e];
    }
    return acc;
}

// x <- x - Q (Q^T x), twice, against columns 0..ncols-1 of Q (column stride len, a multiple of
// VEC); returns ||x||.  x is written by the thread that owns the element and read by others:
// callers leave a barrier before.
template <int VEC>
__device__ double reorth(const double* Q, int64_t len, int ncols, double* x, GksLds& s) {
    using VT = GkVec<VEC>;
    double nrm[1] = {0.0};
    for (int pass = 0; pass < 2; ++pass) {
        wg_dots<1, VEC>(Q, len, ncols, x, nullptr, s);
#pragma unroll 2
        for (int64_t p = VEC * (int)threadIdx.x; p < len; p += VEC * GK_THREADS) {
            VT* xp = reinterpret_cast<VT*>(x + p);
            const VT v = *xp - combine<VEC>(Q, len, ncols, s.h, p);
            *xp = v;
            if (pass == 1)
#pragma unroll
                for (int e = 0; e < VEC; ++e) nrm[0] += v[e] * v[e];
        }
        __syncthreads();
    }
    wg_sum<1>(nrm, s);
    return sqrt(nrm[0]);
}

// Row j of the Gram matrices (against columns 0..j) and d[j]; with W (the p = q = 1 variant)
// every data row is weighted by W[p] and every difference by its edge weight W[n + 4p + e].
// The row is V^T (Y^T W_d Y v_j) and V^T (L^T W_r L v_j): the two vectors are formed once (ya, yl)
// and the K columns then only stream past them.
template <class T>
__device__ void gram_row(int j, const double* V, int n, int nx, int ny, const T* Ix, const T* Iy, const T* It,
                         double* ya, double* yl, GksLds& s, const double* W) {
    const int64_t N = 2 * (int64_t)n;
    const double* vx = V + (int64_t)j * N;
    const double* vy = vx + n;
    double dj[1] = {0.0};
    for (int p = threadIdx.x; p < n; p += GK_THREADS) {
        const int x = p % nx, y = p / nx;
        const double ix = (double)Ix[p], iy = (double)Iy[p];
        const double ax = vx[p], ay = vy[p];
        double e = ix * ax + iy * ay;
        if (W) e *= W[p];
        dj[0] += e * -(double)It[p];
        ya[p] = ix * e;
        ya[n + p] = iy * e;
        // an edge's weight is stored at its left / upper end
        const double* wp = W ? W + n + 4 * (int64_t)p : nullptr;
        double lx = 0.0, ly = 0.0;
        if (x > 0) {
            const double* wq = W ? wp - 4 : nullptr;
            lx += (W ? wq[0] : 1.0) * (ax - vx[p - 1]);
            ly += (W ? wq[1] : 1.0) * (ay - vy[p - 1]);
        }
        if (x + 1 < nx) {
            lx += (W ? wp[0] : 1.0) * (ax - vx[p + 1]);
            ly += (W ? wp[1] : 1.0) * (ay - vy[p + 1]);
        }
        if (y > 0) {
            const double* wq = W ? wp - 4 * (int64_t)nx : nullptr;
            lx += (W ? wq[2] : 1.0) * (ax - vx[p - nx]);
            ly += (W ? wq[3] : 1.0) * (ay - vy[p - nx]);
        }
        if (y + 1 < ny) {
            lx += (W ? wp[2] : 1.0) * (ax - vx[p + nx]);
            ly += (W ? wp[3] : 1.0) * (ay - vy[p + nx]);
        }
        yl[p] = lx;
        yl[n + p] = ly;
    }
    wg_sum<1>(dj, s);  // (its barriers also publish ya and yl)
    wg_dots<2, 2>(V, N, j + 1, ya, yl, s);
    if (threadIdx.x <= (unsigned)j) {
        const int i = threadIdx.x;
        s.GA[i * GK_KC + j] = s.GA[j * GK_KC + i] = s.h[i];
        s.GL[i * GK_KC + j] = s.GL[j * GK_KC + i] = s.h[GK_KC + i];
    }
    if (threadIdx.x == 0) s.d[j] = dj[0];
    __syncthreads();
}

// ---- four GCV points per wave
//
// 16 lanes hold one point's matrix M = G_Y + lambda G_L: lane i owns rows i and 16 + i, a row's
// entries in registers, and an entry of another row arrives by a DPP broadcast within the 16 lanes
// (no LDS: walking the matrix in LDS, one point per wave, its dependent round trips took half of
// the solve).  With G_Y = C C^T and the factor M = R R^T, X = R^-1 C is lower triangular and
//   trace(M^-1 G_Y) = ||X||_F^2,   C^T z = X^T y  (y = R^-1 d),   C^T z0 = C^-1 d = y0,
// so G needs one factorization and one triangular solve of K columns, no inverse and no backward
// solve: its numerator is rho0 + ||X^T y - y0||^2, a sum of non-negative terms.  A factorization of
// 25 columns takes 7.9k cycles and X 5.7k, for one point or four; a wave issues one FP64
// instruction every 7 to 10 cycles and two waves of a SIMD do not slow each other, so the chain of
// pivots bounds it.  With the column-per-wave inner products above, a solve of 15 pairs of 32 x 32
// (ell 10, 20 projected solves) takes 1.94 ms, 12.2 ms before; half of it is this search.
__device__ __forceinline__ double row16_sum(double v) {
#pragma unroll
    for (int o = 8; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// KB = 16, 24 or 32 >= K.
template <int KB>
struct GcvFactor {
    static constexpr bool TWO = KB > 16;
    static constexpr int K2 = KB - 16;   // columns held by second rows (K2 <= 0: none)
    double a1[16], a2[TWO ? KB : 1];     // rows i and 16 + i of R below the diagonal (zeros on and above it)
    double inv1, inv2;                   // 1 / diagonal of the lane's rows
    double y1, y2;                       // R^-1 d
    bool ok;                             // every pivot positive and finite (the same on the 16 lanes)

    // 1 / sqrt(piv): the hardware estimate (relative error e below 2^-22) times 1 + e/2 + 3 e^2/8
    // (the next term is below 2^-66), a shorter chain than two Newton steps.
    __device__ __forceinline__ double pivot(double piv) {
        ok = ok && piv > 0.0 && piv < INFINITY;
        const double r = __builtin_amdgcn_rsq(piv);
        const double e = fma(-piv * r, r, 1.0);
        return fma(r * e, fma(0.375, e, 0.5), r);
    }

    // Rows and columns from K on hold unused values that never reach the first K.
    __device__ __forceinline__ void factor(const GksLds& s, int K, double lam) {
        const int i = threadIdx.x % 16;
#pragma unroll
        for (int c = 0; c < 16; ++c) a1[c] = fma(lam, s.GL[c * GK_KC + i], s.GA[c * GK_KC + i]);
        y1 = s.d[i];
        y2 = 0.0;
        if constexpr (TWO) {
#pragma unroll
            for (int c = 0; c < KB; ++c) a2[c] = fma(lam, s.GL[c * GK_KC + 16 + i], s.GA[c * GK_KC + 16 + i]);
            y2 = s.d[16 + i];
        }
        inv1 = inv2 = 0.0;
        ok = true;
        static_for<0, 16>([&](auto J) {
            constexpr int j = decltype(J)::value;
            if (!TWO && j >= K) return;  // (KB > 16 has K > 16)
            const double r = pivot(row16_bcast<j>(a1[j]));
            const double l1 = i > j ? a1[j] * r : 0.0;
            a1[j] = l1;
            if constexpr (TWO) {
                const double l2 = a2[j] * r;
                a2[j] = l2;
                fmac_bcast<j + 1, 15 - j>(a1 + j + 1, l1, -l1);
                fmac_bcast<j + 1, 15 - j>(a2 + j + 1, l1, -l2);
                fmac_bcast<0, K2>(a2 + 16, l2, -l2);
            } else {
                fmac_bcast<j + 1, 15 - j>(a1 + j + 1, l1, -l1);
            }
            const double yj = row16_bcast<j>(y1) * r;
            inv1 = i == j ? r : inv1;
            y1 = i == j ? yj : fma(-l1, yj, y1);
            if constexpr (TWO) y2 = fma(-a2[j], yj, y2);
        });
        if constexpr (TWO) {
            static_for<16, KB>([&](auto J) {
                constexpr int j = decltype(J)::value;
                if (j >= K) return;
                const double r = pivot(row16_bcast<j - 16>(a2[j]));
                const double l2 = i > j - 16 ? a2[j] * r : 0.0;
                a2[j] = l2;
                fmac_bcast<j - 15, KB - 1 - j>(a2 + j + 1, l2, -l2);
                const double yj = row16_bcast<j - 16>(y2) * r;
                inv2 = i == j - 16 ? r : inv2;
                y2 = i == j - 16 ? yj : fma(-l2, yj, y2);
            });
        }
    }

    // G of the factored point (the same on its 16 lanes); lane i owns columns i and 16 + i of X.
    __device__ __forceinline__ double gcv(const GksLds& s, int K, double rho0, double m) const {
        const int i = threadIdx.x % 16;
        double x1[KB], x2[TWO ? K2 : 1];
#pragma unroll
        for (int r = 0; r < KB; ++r) x1[r] = s.C[r * GK_P + i];
        double v1 = -s.y0[i], v2 = 0.0, t1 = 0.0, t2 = 0.0;
        if constexpr (TWO) {
#pragma unroll
            for (int r = 0; r < K2; ++r) x2[r] = s.C[(16 + r) * GK_P + 16 + i];
            v2 = -s.y0[16 + i];
        }
        static_for<0, KB>([&](auto KK) {
            constexpr int k = decltype(KK)::value;
            if ((!TWO || k >= 16) && k >= K) return;
            const double ik = row16_bcast<k % 16>(k < 16 ? inv1 : inv2);
            const double yk = row16_bcast<k % 16>(k < 16 ? y1 : y2);
            x1[k] *= ik;
            const double nx1 = -x1[k];
            if constexpr (k < 16) {
                fmac_bcast<k + 1, 15 - k>(x1 + k + 1, a1[k], nx1);
                if constexpr (TWO) fmac_bcast<0, K2>(x1 + 16, a2[k], nx1);
            } else {
                x2[k - 16] *= ik;
                fmac_bcast<k - 15, KB - 1 - k>(x1 + k + 1, a2[k], nx1);
                fmac_bcast<k - 15, KB - 1 - k>(x2 + k - 15, a2[k], -x2[k - 16]);
                v2 = fma(x2[k - 16], yk, v2);
                t2 = fma(x2[k - 16], x2[k - 16], t2);
            }
            v1 = fma(x1[k], yk, v1);
            t1 = fma(x1[k], x1[k], t1);
        });
        double q = i < K ? v1 * v1 : 0.0, t = i < K ? t1 : 0.0;
        if (TWO && 16 + i < K) {
            q += v2 * v2;
            t += t2;
        }
        q = row16_sum(q);
        t = row16_sum(t);
        const double den = (m - t) * (m - t);
        const double g = den > 0.0 ? (rho0 + q) / den : INFINITY;
        return ok && isfinite(g) ? g : INFINITY;
    }

    // z = R^-T y (lanes 0..15 write) by the wave that holds the factor: R goes through Rl (LDS, KB
    // rows of GK_P, left there with its diagonal and zero rows from K on), y is left in yl.
    __device__ __forceinline__ void back(int K, double* Rl, double* yl, double* zl) const {
        const int lane = threadIdx.x % 64, i = lane % 16;
        double z1 = i < K ? y1 : 0.0, z2 = TWO && 16 + i < K ? y2 : 0.0;
        const double d1 = i < K ? inv1 : 0.0, d2 = TWO && 16 + i < K ? inv2 : 0.0;
        if (lane < 16) {
#pragma unroll
            for (int c = 0; c < KB; ++c) Rl[i * GK_P + c] = c < 16 && i < K ? a1[c < 16 ? c : 0] : 0.0;
            if (i < K) Rl[i * GK_P + i] = 1.0 / inv1;
            yl[i] = z1;
            if constexpr (TWO) {
                if (i < K2) {
#pragma unroll
                    for (int c = 0; c < KB; ++c) Rl[(16 + i) * GK_P + c] = 16 + i < K ? a2[c] : 0.0;
                    if (16 + i < K) Rl[(16 + i) * GK_P + 16 + i] = 1.0 / inv2;
                }
                yl[16 + i] = z2;
            }
        }
        wave_sync();
        if constexpr (TWO) {
            static_for<0, K2>([&](auto J) {
                constexpr int j = KB - 1 - decltype(J)::value;
                const double zj = row16_bcast<j - 16>(z2 * d2);
                z2 = i == j - 16 ? zj : (i < j - 16 ? fma(-Rl[j * GK_P + 16 + i], zj, z2) : z2);
                z1 = fma(-Rl[j * GK_P + i], zj, z1);
            });
        }
        static_for<0, 16>([&](auto J) {
            constexpr int j = 15 - decltype(J)::value;
            const double zj = row16_bcast<j>(z1 * d1);
            z1 = i == j ? zj : (i < j ? fma(-Rl[j * GK_P + i], zj, z1) : z1);
        });
        if (lane < 16) {
            zl[i] = z1;
            if (TWO) zl[16 + i] = z2;
        }
        wave_sync();
    }
};

// G(lambda) on the calling wave where G_Y has no Cholesky factor (its data rows are dependent, or
// K exceeds their rank).  One point per wave, Cholesky of M in LDS (lanes = rows), the K columns of G_Y
// and d solved together (lanes = columns); the numerator is ||b||^2 - 2 z.d + z^T G_Y z.
__device__ double gcv_eval(int K, double lam, double bb, double m, GksLds& s) {
    const int w = threadIdx.x / 64, lane = threadIdx.x % 64;
    double* M = s.M[w];
    double* X = s.X[w];
    for (int e = lane; e < K * K; e += 64) {
        const int i = e / K, k = e % K;
        M[i * GK_P + k] = fma(lam, s.GL[i * GK_KC + k], s.GA[i * GK_KC + k]);
    }
    wave_sync();
    // Cholesky M = R R^T in place (lower), lane i owns row i
    for (int j = 0; j < K; ++j) {
        const double mjj = M[j * GK_P + j];
        if (!(mjj > 0.0) || !isfinite(mjj)) return INFINITY;  // same value on every lane
        const double ljj = sqrt(mjj);
        double lij = 0.0;
        if (lane > j && lane < K) lij = M[lane * GK_P + j] / ljj;
        wave_sync();
        if (lane > j && lane < K) M[lane * GK_P + j] = lij;
        if (lane == j) M[j * GK_P + j] = ljj;
        wave_sync();
        if (lane > j && lane < K)
            for (int k = j + 1; k <= lane; ++k) M[lane * GK_P + k] -= lij * M[k * GK_P + j];
        wave_sync();
    }
    // columns c < K: M^-1 G_Y e_c; column K: z = M^-1 d (lane c owns column c of X)
    if (lane <= K) {
        for (int r = 0; r < K; ++r) {
            double y = lane < K ? s.GA[r * GK_KC + lane] : s.d[r];
            for (int k = 0; k < r; ++k) y -= M[r * GK_P + k] * X[k * GK_P + lane];
            X[r * GK_P + lane] = y / M[r * GK_P + r];
        }
        for (int r = K - 1; r >= 0; --r) {
            double x = X[r * GK_P + lane];
            for (int k = r + 1; k < K; ++k) x -= M[k * GK_P + r] * X[k * GK_P + lane];
            X[r * GK_P + lane] = x / M[r * GK_P + r];
        }
    }
    wave_sync();
    const double t = wave_sum(lane < K ? X[lane * GK_P + lane] : 0.0);
    double zd = 0.0, zgz = 0.0;
    if (lane < K) {
        const double zi = X[lane * GK_P + K];
        double gz = 0.0;
        for (int k = 0; k < K; ++k) gz += s.GA[lane * GK_KC + k] * X[k * GK_P + K];
        zd = zi * s.d[lane];
        zgz = zi * gz;
    }
    zd = wave_sum(zd);
    zgz = wave_sum(zgz);
    const double rho = fmax(bb - 2.0 * zd + zgz, 0.0);
    const double den = (m - t) * (m - t);
    const double g = den > 0.0 ? rho / den : INFINITY;
    return isfinite(g) ? g : INFINITY;
}

// lambda (every thread returns the same value) and, in s.z, the projected solution: the factor of
// G_Y with y0 and z0, rho0 = residual() of z0 (called by every thread; the sum of squares over the
// pixels), the grid search, and the solve at the lambda found (fixed_lambda > 0: only that).  One
// loop, so that its steps share the code of the factorization: the unrolled code is large, and
// separate copies of it would each run cold.  z is left alone when the last factorization fails.
template <int KB, class F>
__device__ __forceinline__ double gcv_lambda(int K, double bb, double m, double fixed_lambda, GksLds& s,
                                             F&& residual) {
    double tA = 0.0, tL = 0.0;
    for (int i = 0; i < K; ++i) {
        tA += s.GA[i * GK_KC + i];
        tL += s.GL[i * GK_KC + i];
    }
    const double c = log10(fmax(tA, 1e-300) / fmax(tL, 1e-300));
    const int w = threadIdx.x / 64, lane = threadIdx.x % 64;
    double best_g = INFINITY, best_x = c, rho0 = -1.0;
    double h = 2.0 * GK_SPAN / (GK_GRID0 - 1);
    double lam = 0.0;  // of the single points
    constexpr int BASE = -1, LAST = GK_REFINE + 1;
    int stage = BASE;
    if (fixed_lambda > 0.0) {
        stage = LAST;
        lam = fixed_lambda;
    }
    for (; stage <= LAST; ++stage) {
        const bool single = stage == BASE || stage == LAST;
        const int npt = single ? 1 : stage == 0 ? GK_GRID0 : GK_GRIDR;
        const double lo = stage == 0 ? c - GK_SPAN : best_x - h;
        const double step2 = stage == 0 ? 2.0 * GK_SPAN : 2.0 * h;
        const int den = npt - 1;
        if (single || rho0 >= 0.0) {
            // wave w: points 4 w .. 4 w + 3
            if (4 * w < npt) {
                const int p = 4 * w + lane / 16;
                const double x = single ? 0.0 : lo + step2 * p / den;
                GcvFactor<KB> f;
                f.factor(s, K, single ? lam : exp10(x));
                if (single) {
                    if (stage == BASE || f.ok)
                        f.back(K, stage == BASE ? s.C : s.M[0], stage == BASE ? s.y0 : s.X[0],
                               stage == BASE ? s.z0 : s.z);
                    if (threadIdx.x == 0) s.c_ok = f.ok;
                } else {
                    const double g = f.gcv(s, K, rho0, m);
                    if (lane % 16 == 0) {
                        s.gval[p] = g;
                        s.gxv[p] = x;
                    }
                }
            }
        } else {
            for (int p = w; p < npt; p += GK_WAVES) {
                const double x = lo + step2 * p / den;
                const double g = gcv_eval(K, exp10(x), bb, m, s);
                if (lane == 0) {
                    s.gval[p] = g;
                    s.gxv[p] = x;
                }
            }
        }
        __syncthreads();
        if (stage == BASE) {
            if (s.c_ok) {
                rho0 = residual();
                if (!(rho0 >= 0.0)) rho0 = -1.0;
            }
            continue;
        }
        if (stage == LAST) break;
#pragma unroll 8
        for (int p = 0; p < npt; ++p) {
            const double g = s.gval[p], x = s.gxv[p];
            if (g < best_g * (1.0 - GK_TIE)) {
                best_g = g;
                best_x = x;
            }
        }
        __syncthreads();
        if (stage > 0) h = 2.0 * h / (GK_GRIDR - 1);
        lam = exp10(best_x);
    }
    return lam;
}

template <class T>
__global__ __launch_bounds__(GK_THREADS) void k_of_gks(const Tile* __restrict__ pairs,
                                                       const FrameInfo* __restrict__ frames,
                                                       const T* __restrict__ I, T* __restrict__ vout,
                                                       double* __restrict__ Vw, double* __restrict__ Uw,
                                                       double* __restrict__ Sw, double* __restrict__ Rw,
                                                       double* __restrict__ lam_out, int ell, int n_iter, int kc,
                                                       double fixed_lambda, double* __restrict__ Ww, double eps) {
    __shared__ GksLds s;
    const FrameInfo f = frames[pairs[blockIdx.x].frame];
    const int nx = f.nx, ny = f.ny, n = nx * ny;
    const int64_t N = 2 * (int64_t)n;
    const T* Ix = I + 3 * f.pair_off;
    const T* Iy = Ix + n;
    const T* It = Iy + n;
    double* V = Vw + (int64_t)kc * 2 * f.pair_off;   // column j: V + j N
    double* U = Uw + (int64_t)(ell + 1) * f.pair_off;  // column j: U + j n
    double* sv = Sw + 2 * f.pair_off;
    double* r = Rw + 2 * f.pair_off;
    double* lam = lam_out + (int64_t)blockIdx.x * n_iter;
    // p = q = 1: weights of the current iterate, W[p] for the data row and W[n + 4p + e] for
    // the differences (e: x of s_x, x of s_y, y of s_x, y of s_y) (null: p = q = 2)
    double* W = Ww ? Ww + 5 * f.pair_off : nullptr;
    T* vo = vout + 2 * f.pair_off;
    const int tid = threadIdx.x;
    for (int k = tid; k < n_iter; k += GK_THREADS) lam[k] = 0.0;

    // ||b||^2 and ||Y^T b||^2, b = -I_t
    double a2[2] = {0.0, 0.0};
    for (int p = tid; p < n; p += GK_THREADS) {
        const double bt = -(double)It[p];
        const double gx = (double)Ix[p] * bt, gy = (double)Iy[p] * bt;
        a2[0] += bt * bt;
        a2[1] += gx * gx + gy * gy;
    }
    wg_sum<2>(a2, s);
    const double bb = a2[0], atb = sqrt(a2[1]);
    if (atb == 0.0) {
        for (int64_t p = tid; p < N; p += GK_THREADS) vo[p] = T(0);
        return;
    }

    // ell Golub-Kahan steps, both bases re-orthogonalised
    double beta = sqrt(bb);
    for (int p = tid; p < n; p += GK_THREADS) U[p] = -(double)It[p] / beta;
    double a1[1] = {0.0};
    for (int p = tid; p < n; p += GK_THREADS) {
        const double gx = (double)Ix[p] * U[p], gy = (double)Iy[p] * U[p];
        a1[0] += gx * gx + gy * gy;
    }
    wg_sum<1>(a1, s);
    double alpha = sqrt(a1[0]);
    for (int p = tid; p < n; p += GK_THREADS) {
        V[p] = (double)Ix[p] * U[p] / alpha;
        V[n + p] = (double)Iy[p] * U[p] / alpha;
    }
    for (int i = 1; i <= ell; ++i) {
        double* ui = U + (int64_t)i * n;
        const double* up = U + (int64_t)(i - 1) * n;
        const double* vp = V + (int64_t)(i - 1) * N;
        for (int p = tid; p < n; p += GK_THREADS)
            ui[p] = ((double)Ix[p] * vp[p] + (double)Iy[p] * vp[n + p]) - alpha * up[p];
        __syncthreads();
        beta = n % 2 == 0 ? reorth<2>(U, n, i, ui, s) : reorth<1>(U, n, i, ui, s);
        for (int p = tid; p < n; p += GK_THREADS) ui[p] = ui[p] / beta;
        if (i == ell) break;
        double* vi = V + (int64_t)i * N;
        for (int p = tid; p < n; p += GK_THREADS) {
            vi[p] = (double)Ix[p] * ui[p] - beta * vp[p];
            vi[n + p] = (double)Iy[p] * ui[p] - beta * vp[n + p];
        }
        __syncthreads();
        alpha = reorth<2>(V, N, i, vi, s);
        for (int64_t p = tid; p < N; p += GK_THREADS) vi[p] = vi[p] / alpha;
        __syncthreads();  // element n + p of vi is read next by the thread of pixel p
    }
    __syncthreads();

    // generalized Krylov iterations
    int K = ell;
    // the Gram rows' two vectors: r is free between the residuals, the left vectors' workspace
    // ((ell + 1) n >= 2 n values) after the start
    double *ya = r, *yl = U;
    for (int e = tid; e < GK_KC * GK_KC; e += GK_THREADS) s.GA[e] = s.GL[e] = 0.0;
    if (tid < GK_KC) s.d[tid] = 0.0;
    __syncthreads();
    if (!W)
        for (int j = 0; j < K; ++j) gram_row(j, V, n, nx, ny, Ix, Iy, It, ya, yl, s, (const double*)nullptr);
    else
        for (int64_t p = tid; p < N; p += GK_THREADS) sv[p] = 0.0;  // s^(0)
    const double m = (double)n;
    double bbw = bb;  // b^T W_d b
    for (int k = 0; k < n_iter; ++k) {
        if (W) {
            // weights of the iterate s^(k), then the weighted Gram matrices from scratch
            __syncthreads();
            double a1w[1] = {0.0};
            for (int p = tid; p < n; p += GK_THREADS) {
                const int x = p % nx, y = p / nx;
                const double sx = sv[p], sy = sv[n + p];
                const double e = (double)Ix[p] * sx + (double)Iy[p] * sy + (double)It[p];
                const double wd = 1.0 / sqrt(e * e + eps * eps);
                W[p] = wd;
                const double bt = (double)It[p];
                a1w[0] += wd * bt * bt;
                double* we = W + n + 4 * (int64_t)p;
                const double gxx = x + 1 < nx ? sv[p + 1] - sx : 0.0, gxy = x + 1 < nx ? sv[n + p + 1] - sy : 0.0;
                const double gyx = y + 1 < ny ? sv[p + nx] - sx : 0.0, gyy = y + 1 < ny ? sv[n + p + nx] - sy : 0.0;
                we[0] = x + 1 < nx ? 1.0 / sqrt(gxx * gxx + eps * eps) : 0.0;
                we[1] = x + 1 < nx ? 1.0 / sqrt(gxy * gxy + eps * eps) : 0.0;
                we[2] = y + 1 < ny ? 1.0 / sqrt(gyx * gyx + eps * eps) : 0.0;
                we[3] = y + 1 < ny ? 1.0 / sqrt(gyy * gyy + eps * eps) : 0.0;
            }
            wg_sum<1>(a1w, s);
            bbw = a1w[0];
            __syncthreads();
            for (int j = 0; j < K; ++j) gram_row(j, V, n, nx, ny, Ix, Iy, It, ya, yl, s, (const double*)W);
        }
        // ||Y V z0 - b||^2 (weighted for p = q = 1) from a pass over the pixels
        auto residual = [&]() {
            double e2[1] = {0.0};
            auto pass = [&](auto vec) {
                constexpr int VEC = decltype(vec)::value;
                for (int p = VEC * tid; p < n; p += VEC * GK_THREADS) {
                    const GkVec<VEC> sx = combine<VEC>(V, N, K, s.z0, p), sy = combine<VEC>(V, N, K, s.z0, n + p);
#pragma unroll
                    for (int q = 0; q < VEC; ++q) {
                        const double e = (double)Ix[p + q] * sx[q] + (double)Iy[p + q] * sy[q] + (double)It[p + q];
                        e2[0] += (W ? W[p + q] : 1.0) * e * e;
                    }
                }
            };
            if (n % 2 == 0) pass(std::integral_constant<int, 2>{});
            else pass(std::integral_constant<int, 1>{});
            wg_sum<1>(e2, s);
            return e2[0];
        };
        const double lk = K <= 16   ? gcv_lambda<16>(K, bbw, m, fixed_lambda, s, residual)
                          : K <= 24 ? gcv_lambda<24>(K, bbw, m, fixed_lambda, s, residual)
                                    : gcv_lambda<32>(K, bbw, m, fixed_lambda, s, residual);
        if (tid == 0) lam[k] = lk;
#pragma unroll 2
        for (int64_t p = 2 * tid; p < N; p += 2 * GK_THREADS)
            *reinterpret_cast<GkVec<2>*>(sv + p) = combine<2>(V, N, K, s.z, p);
        if (k == n_iter - 1) break;
        __syncthreads();
        // r = Y^T W_d (Y s - b) + lambda L^T W_r L s (W = I for p = q = 2)
        for (int p = tid; p < n; p += GK_THREADS) {
            const int x = p % nx, y = p / nx;
            const double sx = sv[p], sy = sv[n + p];
            double e = (double)Ix[p] * sx + (double)Iy[p] * sy + (double)It[p];
            double lx = 0.0, ly = 0.0;
            // L^T W_r L s: every edge (p, q) adds w_pq (s(p) - s(q)), its weight stored at the
            // edge's left / upper end (all ones for p = q = 2)
            const double* wp = W ? W + n + 4 * (int64_t)p : nullptr;
            if (x > 0) {
                const double* wq = W ? W + n + 4 * (int64_t)(p - 1) : nullptr;
                lx += (W ? wq[0] : 1.0) * (sx - sv[p - 1]);
                ly += (W ? wq[1] : 1.0) * (sy - sv[n + p - 1]);
            }
            if (x + 1 < nx) {
                lx += (W ? wp[0] : 1.0) * (sx - sv[p + 1]);
                ly += (W ? wp[1] : 1.0) * (sy - sv[n + p + 1]);
            }
            if (y > 0) {
                const double* wq = W ? W + n + 4 * (int64_t)(p - nx) : nullptr;
                lx += (W ? wq[2] : 1.0) * (sx - sv[p - nx]);
                ly += (W ? wq[3] : 1.0) * (sy - sv[n + p - nx]);
            }
            if (y + 1 < ny) {
                lx += (W ? wp[2] : 1.0) * (sx - sv[p + nx]);
                ly += (W ? wp[3] : 1.0) * (sy - sv[n + p + nx]);
            }
            if (W) e *= W[p];
            r[p] = (double)Ix[p] * e + lk * lx;
            r[n + p] = (double)Iy[p] * e + lk * ly;
        }
        __syncthreads();
        const double nr = reorth<2>(V, N, K, r, s);
        if (nr <= 1e-14 * atb) break;  // breakdown: keep the last s
        double* vk = V + (int64_t)K * N;
        for (int64_t p = tid; p < N; p += GK_THREADS) vk[p] = r[p] / nr;
        __syncthreads();
        ++K;
        if (!W) gram_row(K - 1, V, n, nx, ny, Ix, Iy, It, ya, yl, s, (const double*)nullptr);
    }
    __syncthreads();
    for (int64_t p = tid; p < N; p += GK_THREADS) vo[p] = (T)sv[p];
}

}  // namespace

int of_gks_capacity() { return GK_KC; }

void check_gks_frames(const Geom& g, int f, int ell, int n_iter) {
    MMOF_CHECK(ell >= 1 && n_iter >= 1 && ell + n_iter - 1 <= GK_KC, MMOF_ERR_INVALID,
               "need ell >= 1, n_iter >= 1, ell + n_iter - 1 <= " + std::to_string(GK_KC));
    for (int s = 0; s < g.n_seq; ++s) {
        if (g.n_t[s] < 2) continue;
        const int64_t n = (int64_t)((g.ny[s] + f - 1) / f) * ((g.nx[s] + f - 1) / f);
        MMOF_CHECK(n > ell && n < ((int64_t)1 << 30), MMOF_ERR_INVALID,
                   "Solve-OF needs frames of more than ell and fewer than 2^30 pixels");
    }
}

GksWork gks_work(Ctx& c, const Geom& g, const FlowMethod& fm, const std::string& prefix) {
    const int64_t P = std::max<int64_t>(g.pair_px, 1);
    GksWork w;
    w.V = static_cast<double*>(c.work(prefix + "V", sizeof(double) * (size_t)(fm.ell + fm.n_iter - 1) * 2 * P));
    w.U = static_cast<double*>(c.work(prefix + "U", sizeof(double) * (size_t)(fm.ell + 1) * P));
    w.S = static_cast<double*>(c.work(prefix + "S", sizeof(double) * 2 * (size_t)P));
    w.R = static_cast<double*>(c.work(prefix + "R", sizeof(double) * 2 * (size_t)P));
    w.lam = static_cast<double*>(
        c.work(prefix + "lam", sizeof(double) * (size_t)std::max<int64_t>(g.n_pairs, 1) * fm.n_iter));
    if (fm.of_p == 1) w.W = static_cast<double*>(c.work(prefix + "W", sizeof(double) * 5 * (size_t)P));
    return w;
}

void launch_of_gks(Ctx& c, Geom& g, int dt, const void* I, void* v, int ell, int n_iter, double fixed_lambda,
                   const GksWork& w, bool l1, double eps) {
    MMOF_CHECK(!l1 || (w.W && eps > 0 && std::isfinite(eps)), MMOF_ERR_INVALID, "p = q = 1 needs eps > 0");
    if (g.n_pairs == 0) return;
    const int kc = ell + n_iter - 1;
    MMOF_CHECK(ell >= 1 && n_iter >= 1 && kc <= GK_KC, MMOF_ERR_INVALID,
               "need ell >= 1, n_iter >= 1, ell + n_iter - 1 <= " + std::to_string(GK_KC));
    // one tile per pair: the list of pairs
    const TileList& tl = g.tile_list(c.stream, 65535, 65535, true);
    MMOF_CHECK(tl.count == g.n_pairs, MMOF_ERR_SHAPE, "pair list");
    dispatch(dt, [&](auto z) {
        using T = decltype(z);
        ScopedTime st(&c, "of_gks", sizeof(T) * 5.0 * g.pair_px, 0.0);
        hipLaunchKernelGGL(k_of_gks<T>, dim3((unsigned)tl.count), dim3(GK_THREADS), 0, c.stream, tl.buf.as<Tile>(),
                           g.dframes(), (const T*)I, (T*)v, w.V, w.U, w.S, w.R, w.lam, ell, n_iter, kc, fixed_lambda,
                           l1 ? w.W : nullptr, eps);
        MMOF_LAUNCH_CHECK();
    });
}

}  // namespace mmof

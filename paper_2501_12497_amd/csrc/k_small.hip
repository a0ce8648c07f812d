// Small projected problem of MMGKS (eq. minKryov2) and the discrepancy principle
// (Sec. 4.1.3), in FP64 on one wavefront.
//
// With G_H = (HV)^T(HV), G_T = (P Theta V)^T (P Theta V) and d = (HV)^T b, the projected
// normal equations read (G_H + lambda G_T) z = d and the discrepancy of u = V z is
//   D(lambda)^2 = ||H V z - b||^2 = ||b||^2 - d^T z - lambda z^T G_T z.
// lambda solves D(lambda) = eta*delta.  D^2 increases with lambda; its derivative is
//   dD^2/dlambda = 2 lambda w^T (G_H + lambda G_T)^{-1} w,   w = G_T z.
// The root is bracketed in mu = log10(lambda) on [-12, 12] + log10(tr G_H / tr G_T)
// (an end is taken when the root lies beyond it) and found by Newton steps in mu,
// safeguarded by bisection of the bracket, starting from the previous lambda.
//
// K <= 64: one wavefront, lane i owning row i; 16-column blocks in registers, matrix cores for the
// blocks of the factored columns, the factor in LDS.  Broadcasts within 16 lanes are DPP operands of
// the FMAs.  D^2 and its derivative only need forward solves (d^T z = ||L^{-1} d||^2,
// w^T M^{-1} w = ||L^{-1} w||^2) plus one backward solve for z.
// 64 < K <= 256: eight wavefronts by the same steps, the matrix in their accumulators, the factor in the
// LDS up to 128 columns and in an L2-resident global workspace beyond.  The root search is the same for both.
#include "dev.h"
#include "krylov.h"

// Optional per-iteration trace (a probe build can define it; no-op in the library).
#ifndef MMOF_SMALL_TRACE
#define MMOF_SMALL_TRACE(it, mu, e, f, lo, hi)
#endif

namespace mmof {

static constexpr int KP = KMAX_SMALL + 1;  // padded row length (odd: no LDS bank aliasing)

struct SmallLds {
    double A[KMAX_SMALL][KP];
    double T[KMAX_SMALL][KP];
    double L[KMAX_SMALL][KP];
    double piv[KMAX_SMALL], inv[KMAX_SMALL];  // the pivots and their reciprocals
};

__device__ __forceinline__ double bcast(double v, int lane) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), lane);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Wave sum whose result is bitwise identical in every lane: the root finder branches on
// it, and a butterfly alone is not lane-symmetric once the compiler fuses the first add
// with the product that feeds it.  Lane 0's sum is broadcast.
__device__ __forceinline__ double wave_sum64(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return bcast(v, 0);
}

typedef double dbl4 __attribute__((ext_vector_type(4)));

// 1/x for x > 0: hardware estimate refined by two Newton steps (each squares the relative error), a
// short dependency chain on the pivot path.
__device__ __forceinline__ double rcp_nr(double x) {
    double r = __builtin_amdgcn_rcp(x);
#pragma unroll
    for (int it = 0; it < 2; ++it) r = fma(r, fma(-x, r, 1.0), r);
    return r;
}

// Sums of two values over the wave, bitwise identical in every lane (the sums of the four rows of
// 16 lanes are taken from one lane each).
__device__ __forceinline__ void wave_sum2(double& a, double& b) {
    auto row = [](double v) {
        v += __builtin_amdgcn_update_dpp(0.0, v, 0x128, 0xf, 0xf, true);  // row_ror:8
        v += __builtin_amdgcn_update_dpp(0.0, v, 0x124, 0xf, 0xf, true);
        v += __builtin_amdgcn_update_dpp(0.0, v, 0x122, 0xf, 0xf, true);
        v += __builtin_amdgcn_update_dpp(0.0, v, 0x121, 0xf, 0xf, true);
        return v;
    };
    a = row(a);
    b = row(b);
    a = (bcast(a, 0) + bcast(a, 16)) + (bcast(a, 32) + bcast(a, 48));
    b = (bcast(b, 0) + bcast(b, 16)) + (bcast(b, 32) + bcast(b, 48));
}

// M = A + lam T = U diag(p) U^T with U unit lower triangular, in 16-column blocks (rows and columns
// K..16*ceil(K/16)-1 are padded with the identity).  -U goes below the diagonal of s.L, the pivots p
// to s.piv.  A block column starts as M less the products of the factored columns, on the FP64 matrix
// cores: M_{I,J} - U_{I,J'} (p U_{J,J'})^T with v_mfma_f64_16x16x4f64 (lane l supplies A[l%16][l/16]
// and B[l/16][l%16]; the 16x16 result is D[l/16 + 4v][l%16] in four doubles per lane).  Then each
// lane holds its row's 16 entries and, in every row of 16 lanes, a copy of the diagonal block's row
// l % 16, so that a pivot and the entries of its column reach all lanes as DPP operands (one FMA per
// entry; two readlanes and an FMA before).  The last block column has no rows below its diagonal
// block.  Bound by the instructions one wave issues, 11 cycles apart; the factorization and its solves take 4 us at
// K = 16, 12 at 39 and 17 at 64 (9, 22 and 32 with readlane broadcasts and masked steps; a cold start at K = 39, eight
// of them, 180 -> 95 us).
// Returns false on a pivot that is not positive (uniform across the wave); on success *inv holds
// 1 / p[lane].
__device__ bool factor(SmallLds& s, int K, double lam, double* inv) {
    const int i = threadIdx.x, r = i & 15, lk = i >> 4;
    const int nbk = (K + 15) >> 4;
    bool ok = true;
    for (int J = 0; J < nbk; ++J) {
        const int c0 = J << 4;
        const bool last = J == nbk - 1;
        if (J > 0) {
            for (int I = J; I < nbk; ++I) {
                dbl4 acc;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int row = (I << 4) + lk + 4 * v, col = c0 + r;
                    acc[v] = fma(lam, s.T[row][col], s.A[row][col]) + (row == col && row >= K ? 1.0 : 0.0);
                }
                for (int b0 = 0; b0 < c0; b0 += 16) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int col = b0 + 4 * q + lk;
                        // (both factors negated in s.L: the product of the pivot takes the sign)
                        const double av = s.L[(I << 4) + r][col];
                        const double bv = -s.piv[col] * s.L[c0 + r][col];
                        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc, 0, 0, 0);
                    }
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) s.L[(I << 4) + lk + 4 * v][c0 + r] = acc[v];
            }
            __syncthreads();
        }
        auto columns = [&](auto below) {
            constexpr bool BELOW = decltype(below)::value;
            double P[16], D[16];
            if (J == 0) {
#pragma unroll
                for (int c = 0; c < 16; ++c) {
                    D[c] = fma(lam, s.T[r][c], s.A[r][c]);
                    if (!BELOW) D[c] += r == c && r >= K ? 1.0 : 0.0;  // (K <= 16)
                    P[c] = BELOW ? fma(lam, s.T[i][c], s.A[i][c]) : 0.0;
                }
            } else {
#pragma unroll
                for (int c = 0; c < 16; ++c) {
                    D[c] = s.L[c0 + r][c0 + c];
                    P[c] = BELOW ? s.L[i][c0 + c] : 0.0;  // (rows above the block: nothing reads what they become)
                }
            }
            int at = c0;  // (in a vector register: the stores then take their offset)
            asm volatile("" : "+v"(at));
            static_for<0, 16>([&](auto C) {
                constexpr int c = decltype(C)::value;
                const double p = row16_bcast<c>(D[c]);
                ok = ok && p > 0.0;
                const double q = rcp_nr(p);
                s.piv[at + c] = p;  // (the same value from every lane)
                s.inv[at + c] = q;
                const double nu = D[c] * -q;
                fmac_bcast<c + 1, 15 - c>(D + c + 1, D[c], nu);
                if constexpr (BELOW) {
                    const double nl = P[c] * -q;
                    fmac_bcast<c + 1, 15 - c>(P + c + 1, D[c], nl);
                    P[c] = nl;
                } else {
                    P[c] = nu;
                }
            });
            if (BELOW || lk == J) {
                // zeros on and above the diagonal, which the solves multiply by
                const int rr = i - c0;
#pragma unroll
                for (int c = 0; c < 16; ++c) s.L[i][c0 + c] = rr > c ? P[c] : 0.0;
            }
        };
        if (last)
            columns(std::false_type{});
        else
            columns(std::true_type{});
        if (!ok) return false;
        __syncthreads();
    }
    *inv = s.inv[i];
    return true;
}

// Steps of a block's triangular solve on the copies of its entries x in every row of 16 lanes, four columns N, N + S,
// N + 2 S, N + 3 S, and what each finished entry adds to the lane's own row (a) and product (w):
//   x += x(lane c) d[c],   a += x(lane c) l[c],   w += x(lane c) t[c].
// (A DPP source may not have been written within two wait states.)
#define SS_FMAC(dst, m, q) \
    "v_fmac_f64_dpp %[" #dst "], %[x], %[" #m #q "] row_newbcast:%[n" #q "] row_mask:0xf bank_mask:0xf\n\t"
template <int N, int S>
__device__ __forceinline__ void solve_steps(double& x, double& a, const double* d, const double* l) {
#define SS_STEP(q) "s_nop 1\n\t" SS_FMAC(x, d, q) "s_nop 1\n\t" SS_FMAC(a, l, q)
    asm volatile(SS_STEP(0) SS_STEP(1) SS_STEP(2) SS_STEP(3)
                 : [x] "+&v"(x), [a] "+&v"(a)
                 : [d0] "v"(d[0]), [d1] "v"(d[S]), [d2] "v"(d[2 * S]), [d3] "v"(d[3 * S]), [l0] "v"(l[0]),
                   [l1] "v"(l[S]), [l2] "v"(l[2 * S]), [l3] "v"(l[3 * S]), [n0] "n"(N), [n1] "n"(N + S),
                   [n2] "n"(N + 2 * S), [n3] "n"(N + 3 * S));
#undef SS_STEP
}
template <int N, int S>
__device__ __forceinline__ void solve_steps(double& x, double& a, double& w, const double* d, const double* l,
                                            const double* t) {
#define SS_STEP(q) "s_nop 1\n\t" SS_FMAC(x, d, q) "s_nop 1\n\t" SS_FMAC(a, l, q) SS_FMAC(w, t, q)
    asm volatile(SS_STEP(0) SS_STEP(1) SS_STEP(2) SS_STEP(3)
                 : [x] "+&v"(x), [a] "+&v"(a), [w] "+&v"(w)
                 : [d0] "v"(d[0]), [d1] "v"(d[S]), [d2] "v"(d[2 * S]), [d3] "v"(d[3 * S]), [l0] "v"(l[0]),
                   [l1] "v"(l[S]), [l2] "v"(l[2 * S]), [l3] "v"(l[3 * S]), [t0] "v"(t[0]), [t1] "v"(t[S]),
                   [t2] "v"(t[2 * S]), [t3] "v"(t[3 * S]), [n0] "n"(N), [n1] "n"(N + S), [n2] "n"(N + 2 * S),
                   [n3] "n"(N + 3 * S));
#undef SS_STEP
}
#undef SS_FMAC

// y = U^{-1} b (one entry per lane): each row of 16 lanes solves a copy of a diagonal block, and the
// rows below take its entries as they are finished.
__device__ double fwd_solve(const SmallLds& s, int K, double b) {
    const int i = threadIdx.x, r = i & 15, g = i >> 4;
    double y = i < K ? b : 0.0;
    for (int c0 = 0; c0 < K; c0 += 16) {
        double l[16], d[16];
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            d[c] = s.L[c0 + r][c0 + c];
            l[c] = s.L[i][c0 + c];
        }
        double x = __shfl(y, c0 + r), below = y;
        static_for<0, 4>([&](auto Q) {
            constexpr int c = 4 * decltype(Q)::value;
            solve_steps<c, 1>(x, below, d + c, l + c);
        });
        y = g == (c0 >> 4) ? x : (i > c0 ? below : y);
    }
    return i < K ? y : 0.0;
}

// z = U^{-T} y, blocks from the last one up, and w = T z with it.
__device__ double bwd_solve(const SmallLds& s, int K, double y, double& w) {
    const int i = threadIdx.x, r = i & 15, g = i >> 4;
    double z = i < K ? y : 0.0;
    w = 0.0;
    for (int c0 = ((K - 1) >> 4) << 4; c0 >= 0; c0 -= 16) {
        double l[16], d[16], t[16];
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            d[c] = s.L[c0 + c][c0 + r];
            l[c] = s.L[c0 + c][i];
            t[c] = s.T[i][c0 + c];
        }
        double x = __shfl(z, c0 + r), above = z;
        static_for<0, 4>([&](auto Q) {
            constexpr int c = 15 - 4 * decltype(Q)::value;
            solve_steps<c, -1>(x, above, w, d + c, l + c, t + c);
        });
        z = g == (c0 >> 4) ? x : (i < c0 ? above : z);
    }
    w = i < K ? w : 0.0;
    return i < K ? z : 0.0;
}

struct Eval {
    bool ok;
    double D2, dD2, z;  // z: this lane's entry
};

__device__ Eval evaluate(SmallLds& s, int K, double lam, double bb, double d, bool deriv, int& nfac) {
    Eval e{false, 0.0, 0.0, 0.0};
    ++nfac;
    double inv;
    if (!factor(s, K, lam, &inv)) return e;
    e.ok = true;
    const double y = fwd_solve(s, K, d);
    const double yp = (int)threadIdx.x < K ? y * inv : 0.0;
    double w;
    e.z = bwd_solve(s, K, yp, w);
    double dz = y * yp, zw = e.z * w;  // d^T z = y^T diag(1/p) y
    wave_sum2(dz, zw);
    e.D2 = bb - dz - lam * zw;
    if (deriv) {
        const double q = fwd_solve(s, K, w);
        double qq = (int)threadIdx.x < K ? q * q * inv : 0.0, none = 0.0;
        wave_sum2(qq, none);
        e.dD2 = 2.302585092994046 * 2.0 * lam * lam * qq;
    }
    return e;
}

// The discrepancy-principle root in mu = log10(lambda) (or the fixed lambda), given
// ev(lambda, with_derivative) -> Eval and the traces of G_H and G_T (all three uniform across
// the threads of the solve).  Leaves the last accepted evaluation in e, lambda in lam and
// 0 (root) / 2 (clamped to an end of the bracket) in status.
template <class EV>
__device__ void dp_root(EV&& ev, double trA, double trT, double target, double bb, double prev, double fixed_lambda,
                        Eval& e, double& lam, int& status) {
    if (fixed_lambda > 0.0) {
        e = ev(lam, false);
        return;
    }
    const double shift = log10(trA / fmax(trT, 1e-300));
    const double LO = -12.0 + shift, HI = 12.0 + shift;
    double lo = LO, hi = HI;
    bool lo_checked = false, hi_checked = false;
    double mu = 0.5 * (lo + hi);
    if (prev > 0.0) {
        const double m = log10(prev);
        if (m > lo && m < hi) mu = m;
    }
    // Newton in mu inside the bracket [lo, hi].  An end of the search interval is only
    // evaluated when a step would leave through it: an interior root proves, by
    // monotonicity of D^2, that neither end needs clamping.
    for (int it = 0; it < 200; ++it) {
        e = ev(exp10(mu), true);
        const double f = e.ok ? e.D2 - target : -target;
        MMOF_SMALL_TRACE(it, mu, e, f, lo, hi);
        if (f < 0.0)
            lo = mu;
        else
            hi = mu;
        if (e.ok && fabs(f) <= 1e-13 * bb) break;  // rounding level of D^2
        double nmu = (e.ok && e.dD2 > 0.0) ? mu - f / e.dD2 : 0.5 * (lo + hi);
        if (!(nmu > lo && nmu < hi)) {
            if (f < 0.0 && !hi_checked && hi == HI) {
                hi_checked = true;
                const Eval eh = ev(exp10(HI), false);
                if (eh.ok && eh.D2 < target) {
                    e = eh;
                    mu = HI;
                    status = 2;
                    break;
                }
            }
            if (f > 0.0 && !lo_checked && lo == LO) {
                lo_checked = true;
                const Eval el = ev(exp10(LO), false);
                if (el.ok && el.D2 > target) {
                    e = el;
                    mu = LO;
                    status = 2;
                    break;
                }
            }
            nmu = 0.5 * (lo + hi);
        }
        if (fabs(nmu - mu) <= 1e-11 * fmax(1.0, fabs(mu)) || hi - lo <= 1e-14 * fmax(1.0, fabs(mu))) {
            // converged to ~1e-11 in log10(lambda): keep the evaluation at mu (its z and
            // D^2 differ from those at the root by the same relative amount) unless it failed
            if (!e.ok) {
                mu = nmu;
                e = ev(exp10(mu), false);
            }
            break;
        }
        mu = nmu;
    }
    lam = exp10(mu);
}

__global__ __launch_bounds__(64) void k_small_solve(int K, const double* __restrict__ GA, const double* __restrict__ GT,
                                                    const double* __restrict__ dvec, const double* __restrict__ sc,
                                                    double fixed_lambda, double* __restrict__ zout,
                                                    double* __restrict__ res, double* __restrict__ lam_out,
                                                    const double* __restrict__ Tb, double* __restrict__ zt) {
    __shared__ SmallLds s;
    const int i = threadIdx.x;
    // coalesced loads: each instruction moves one contiguous row of the matrices, eight rows of both
    // in flight; entries outside K x K are zero up to the padded size
    const int KP16 = (K + 15) & ~15;
    for (int r0 = 0; r0 < KP16; r0 += 8) {
        double ga[8], gt[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const bool in = r0 + q < K && i < K;
            ga[q] = in ? GA[(int64_t)(r0 + q) * KLD + i] : 0.0;
            gt[q] = in ? GT[(int64_t)(r0 + q) * KLD + i] : 0.0;
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            s.A[r0 + q][i] = ga[q];
            s.T[r0 + q][i] = gt[q];
        }
    }
    const double d = i < K ? dvec[i] : 0.0;
    __syncthreads();
    const double bb = sc[0], target = sc[1];
    double lam = fixed_lambda;
    int status = 0;
    int nfac = 0;
    Eval e{false, 0.0, 0.0, 0.0};
    const double trA = fixed_lambda > 0.0 ? 0.0 : wave_sum64(i < K ? s.A[i][i] : 0.0);
    const double trT = fixed_lambda > 0.0 ? 0.0 : wave_sum64(i < K ? s.T[i][i] : 0.0);
    dp_root([&](double l, bool deriv) { return evaluate(s, K, l, bb, d, deriv, nfac); }, trA, trT, target, bb, sc[2],
            fixed_lambda, e, lam, status);
    if (!e.ok) status = 4;
    const double z = e.ok && i < K ? e.z : 0.0;
    if (i < K) zout[i] = z;
    if (i == 0) {
        res[0] = lam;
        res[1] = e.D2;
        res[2] = (double)status;
        res[3] = (double)nfac;
        if (lam_out) lam_out[0] = lam;
    }
    if (!zt) return;
    // T z (T(k, j) = Tb[j * KLD + k], unit diagonal): the columns' entries eight at a time
    double a = z;
    for (int j0 = 1; Tb && j0 < K; j0 += 8) {
        double t[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) t[q] = j0 + q < K && i < j0 + q ? Tb[(int64_t)(j0 + q) * KLD + i] : 0.0;
#pragma unroll
        for (int q = 0; q < 8; ++q) a = fma(t[q], bcast(z, min(j0 + q, KMAX_SMALL - 1)), a);
    }
    if (i < K) zt[i] = a;
}

// ----------------------------------------------------------------------------- 64 < K <= 256
//
// Eight waves.  The lower 16 x 16 blocks of M stay in the accumulators of the waves (block b of the column-major list on
// wave b % 8: 17 blocks each at K = 256), a block column passes through the LDS to be factored by the waves that own its
// rows, with the steps of factor(), and updates the blocks right of it on the matrix cores from there.  The factor stays
// in the LDS up to 128 columns (the largest square that fits beside the rest) and goes to an L2-resident workspace
// beyond, by columns and by rows, for the triangular solves: thread i < 256 owns row i, and every row of 16 lanes solves
// a copy of the diagonal block (one barrier per block of a solve, three of the factorization).  An evaluation takes 25 us
// at K = 80, 41 at 120, 67 at 130 and 111 at 200 (34 and 57 at 80 and 120 with the factor in L2; 126, 261 and 514 at 80,
// 130 and 200 with the trailing matrix there too, updated entry by entry).

static constexpr int BIG_T = 512, BIG_W = BIG_T / 64;  // threads, waves

// NB block columns at most: 8 (K <= 128), the factor in the LDS, or 16, in L2.
template <int NB>
struct BigLds {
    static constexpr bool IN_LDS = NB <= 8;
    static constexpr int SLOTS = (NB * (NB + 1) / 2 + BIG_W - 1) / BIG_W;  // blocks per wave
    static constexpr int RW = NB / 4;                                      // waves that own rows
    static constexpr int LD = IN_LDS ? 16 * NB + 1 : 17;
    // IN_LDS: the factor, block column by block column; otherwise the current block column, two in turn (padded rows)
    double F[IN_LDS ? 1 : 2][16 * NB][LD];
    __device__ __forceinline__ double* row(int J, int i) { return IN_LDS ? &F[0][i][16 * J] : &F[J & 1][i][0]; }
    double piv[KMAX], inv[KMAX];
    double vec[KMAX];       // the vector of a product
    double x[2][16];        // a block's right-hand side, two in turn
    double red[BIG_W], red2[BIG_W];
    int fail;
};

// Sums of two values over the workgroup, bitwise identical in every thread (the wave totals added in a fixed order).
template <int NB>
__device__ __forceinline__ void block_sum2(BigLds<NB>& s, double& a, double& b) {
    wave_sum2(a, b);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
        s.red[threadIdx.x >> 6] = a;
        s.red2[threadIdx.x >> 6] = b;
    }
    __syncthreads();
    a = b = 0.0;
#pragma unroll
    for (int w = 0; w < BIG_W; ++w) {
        a += s.red[w];
        b += s.red2[w];
    }
}

// M = A + lam T = U diag(p) U^T as in factor() (A, T row-major with leading dimension KLD): -U to the LDS, or by columns
// to L[c * KLD + r] and by rows to L[(KMAX + r) * KLD + c], zeros on and above the diagonal of its diagonal blocks; p and
// 1/p to the LDS.  Returns false, uniformly, on a pivot that is not positive.
template <int NB>
__device__ bool factor_big(BigLds<NB>& s, double* L, const double* __restrict__ A, const double* __restrict__ T, int K,
                           double lam) {
    const int lane = threadIdx.x & 63, r = lane & 15, lk = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nbk = (K + 15) >> 4, nblk = nbk * (nbk + 1) / 2;
    if (threadIdx.x == 0) s.fail = 0;
    constexpr int SLOTS = BigLds<NB>::SLOTS;
    dbl4 acc[SLOTS];
    int bi[SLOTS], bj[SLOTS];  // block row and column of a slot (uniform)
#pragma unroll
    for (int q = 0; q < SLOTS; ++q) {
        int b = q * BIG_W + wave, J = 0;
        const bool used = b < nblk;
        while (used && b >= nbk - J) b -= nbk - J++;
        bi[q] = used ? J + b : -1;
        bj[q] = used ? J : -1;
        if (!used) continue;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = (bi[q] << 4) + lk + 4 * v, col = (bj[q] << 4) + r;
            const bool in = row < K && col < K;
            const int64_t o = (int64_t)min(row, K - 1) * KLD + min(col, K - 1);
            const double m = fma(lam, T[o], A[o]);
            acc[q][v] = in ? m : (row == col ? 1.0 : 0.0);
        }
    }
    for (int J = 0; J < nbk; ++J) {
        const int c0 = J << 4;
#pragma unroll
        for (int q = 0; q < SLOTS; ++q) {
            if (bj[q] != J) continue;
#pragma unroll
            for (int v = 0; v < 4; ++v) s.row(J, (bi[q] << 4) + lk + 4 * v)[r] = acc[q][v];
        }
        __syncthreads();
        const int i = (wave << 6) + lane;
        double D[16];
#pragma unroll
        for (int c = 0; c < 16; ++c) D[c] = s.row(J, c0 + r)[c];
        // every wave has read the diagonal block: the one that owns its rows writes their factor over it
        __syncthreads();
        if (wave < BigLds<NB>::RW && (wave << 6) + 63 >= c0 && (wave << 6) < (nbk << 4)) {
            double Pr[16];
#pragma unroll
            for (int c = 0; c < 16; ++c) Pr[c] = s.row(J, i)[c];  // (rows above the block: nothing reads what they become)
            bool ok = true;
            double pv = 1.0, iv = 1.0;
            static_for<0, 16>([&](auto C) {
                constexpr int c = decltype(C)::value;
                const double p = row16_bcast<c>(D[c]);
                ok = ok && p > 0.0;
                const double q = rcp_nr(p);
                pv = r == c ? p : pv;
                iv = r == c ? q : iv;
                const double nu = D[c] * -q, nl = Pr[c] * -q;
                fmac_bcast<c + 1, 15 - c>(D + c + 1, D[c], nu);
                fmac_bcast<c + 1, 15 - c>(Pr + c + 1, D[c], nl);
                Pr[c] = nl;
            });
            if (!ok) s.fail = 1;  // (the same on every wave that factors the block)
            const int rr = i - c0;
            if (rr >= 0 && rr < 16) {
                s.piv[i] = pv;
                s.inv[i] = iv;
            }
            if (rr >= 0 && i < (nbk << 4)) {
#pragma unroll
                for (int c = 0; c < 16; ++c) {
                    const double v = rr > c ? Pr[c] : 0.0;
                    s.row(J, i)[c] = v;
                    if (!BigLds<NB>::IN_LDS) {
                        L[(int64_t)(c0 + c) * KLD + i] = v;
                        L[(int64_t)(KMAX + i) * KLD + c0 + c] = v;
                    }
                }
            }
        }
        __syncthreads();
        if (s.fail) return false;
#pragma unroll
        for (int q = 0; q < SLOTS; ++q) {
            if (bj[q] <= J) continue;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const double av = s.row(J, (bi[q] << 4) + r)[4 * k + lk];
                const double bv = -s.piv[c0 + 4 * k + lk] * s.row(J, (bj[q] << 4) + r)[4 * k + lk];
                acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc[q], 0, 0, 0);
            }
        }
    }
    return true;
}

// y = U^{-1} b, one entry per thread i < KMAX.
template <int NB>
__device__ double fwd_big(BigLds<NB>& s, const double* L, int K, double b) {
    const int i = threadIdx.x, r = i & 15, nbk = (K + 15) >> 4;
    double y = i < K ? b : 0.0;
    for (int J = 0; J < nbk; ++J) {
        const int c0 = J << 4;
        const bool work = (i | 63) >= c0 && (i & ~63) < (nbk << 4);  // (whole waves)
        double l[16], d[16];
        if (work) {
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                d[c] = BigLds<NB>::IN_LDS ? s.row(J, c0 + r)[c] : L[(int64_t)(c0 + c) * KLD + c0 + r];
                l[c] = BigLds<NB>::IN_LDS ? s.row(J, i)[c] : L[(int64_t)(c0 + c) * KLD + i];
            }
        }
        if ((i >> 4) == J) s.x[J & 1][r] = y;
        __syncthreads();
        if (work) {
            double x = s.x[J & 1][r], below = y;
            static_for<0, 4>([&](auto Q) {
                constexpr int c = 4 * decltype(Q)::value;
                solve_steps<c, 1>(x, below, d + c, l + c);
            });
            y = (i >> 4) == J ? x : (i > c0 ? below : y);
        }
    }
    return i < K ? y : 0.0;
}

// z = U^{-T} y, blocks from the last one up.
template <int NB>
__device__ double bwd_big(BigLds<NB>& s, const double* L, int K, double y) {
    const int i = threadIdx.x, r = i & 15, nbk = (K + 15) >> 4;
    const double* R = L + (int64_t)KMAX * KLD;  // by rows
    double z = i < K ? y : 0.0;
    __syncthreads();  // (the last block of a forward solve is still read from s.x)
    for (int J = nbk - 1; J >= 0; --J) {
        const int c0 = J << 4;
        const bool work = (i & ~63) <= c0 + 15;  // (whole waves)
        double l[16], d[16];
        if (work) {
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                d[c] = BigLds<NB>::IN_LDS ? s.row(J, c0 + c)[r] : R[(int64_t)(c0 + c) * KLD + c0 + r];
                l[c] = BigLds<NB>::IN_LDS ? s.F[0][c0 + c][i] : R[(int64_t)(c0 + c) * KLD + i];
            }
        }
        if ((i >> 4) == J) s.x[J & 1][r] = z;
        __syncthreads();
        if (work) {
            double x = s.x[J & 1][r], above = z;
            static_for<0, 4>([&](auto Q) {
                constexpr int c = 15 - 4 * decltype(Q)::value;
                solve_steps<c, -1>(x, above, d + c, l + c);
            });
            z = (i >> 4) == J ? x : (i < c0 ? above : z);
        }
    }
    __syncthreads();
    return i < K ? z : 0.0;
}

template <int NB>
__device__ Eval evaluate_big(BigLds<NB>& s, double* L, const double* __restrict__ GA, const double* __restrict__ GT, int K,
                             double lam, double bb, double d, bool deriv, int& nfac) {
    const int i = threadIdx.x;
    Eval e{false, 0.0, 0.0, 0.0};
    ++nfac;
    __syncthreads();  // (every thread is past the previous evaluation's reads)
    if (!factor_big(s, L, GA, GT, K, lam)) return e;
    e.ok = true;
    const double inv = i < K ? s.inv[i] : 0.0;
    const double y = fwd_big(s, L, K, d), yp = y * inv;
    e.z = bwd_big(s, L, K, yp);
    // w = T z (T symmetric: row i read along column i, coalesced), the odd columns by the upper threads
    if (i < KMAX) s.vec[i] = e.z;
    __syncthreads();
    const int row = i & (KMAX - 1);
    double w = 0.0;
    if (row < K) {
#pragma unroll 8
        for (int j = i >> 8; j < K; j += 2) w = fma(GT[(int64_t)j * KLD + row], s.vec[j], w);
    }
    __syncthreads();
    if (i >= KMAX) s.vec[row] = w;
    __syncthreads();
    w = i < K ? w + s.vec[i] : 0.0;
    double dz = y * yp, zw = e.z * w;  // d^T z = y^T diag(1/p) y
    block_sum2(s, dz, zw);
    e.D2 = bb - dz - lam * zw;
    if (deriv) {
        const double q = fwd_big(s, L, K, w);
        double qq = q * q * inv, none = 0.0;
        block_sum2(s, qq, none);
        e.dD2 = 2.302585092994046 * 2.0 * lam * lam * qq;
    }
    return e;
}

template <int NB>
__global__ __launch_bounds__(BIG_T) void k_small_solve_big(int K, const double* __restrict__ GA,
                                                           const double* __restrict__ GT,
                                                           const double* __restrict__ dvec,
                                                           const double* __restrict__ sc, double fixed_lambda,
                                                           double* L, double* __restrict__ zout,
                                                           double* __restrict__ res, double* __restrict__ lam_out) {
    __shared__ BigLds<NB> s;
    const int i = threadIdx.x;
    const double d = i < K ? dvec[i] : 0.0;
    const double bb = sc[0], target = sc[1];
    double lam = fixed_lambda;
    int status = 0;
    int nfac = 0;
    Eval e{false, 0.0, 0.0, 0.0};
    double trA = 0.0, trT = 0.0;
    if (!(fixed_lambda > 0.0)) {
        trA = i < K ? GA[(int64_t)i * KLD + i] : 0.0;
        trT = i < K ? GT[(int64_t)i * KLD + i] : 0.0;
        block_sum2(s, trA, trT);
    }
    dp_root([&](double l, bool deriv) { return evaluate_big(s, L, GA, GT, K, l, bb, d, deriv, nfac); }, trA, trT,
            target, bb, sc[2], fixed_lambda, e, lam, status);
    if (!e.ok) status = 4;
    if (i < K) zout[i] = e.ok ? e.z : 0.0;
    if (i == 0) {
        res[0] = lam;
        res[1] = e.D2;
        res[2] = (double)status;
        res[3] = (double)nfac;
        if (lam_out) lam_out[0] = lam;
    }
}

void small_solve(Ctx& c, int K, const double* GA, const double* GT, const double* d, const double* sc,
                 double fixed_lambda, double* z, double* res, double* lam_out, const double* T, double* zt) {
    MMOF_CHECK(K >= 1 && K <= KMAX, MMOF_ERR_SHAPE, "Krylov basis size out of range");
    ScopedTime st(&c, "small_solve");
    if (K <= KMAX_SMALL) {
        hipLaunchKernelGGL(k_small_solve, dim3(1), dim3(64), 0, c.stream, K, GA, GT, d, sc, fixed_lambda, z, res,
                           lam_out, T, zt);
    } else {
        const bool lds = K <= 128;
        double* Lg = lds ? nullptr
                         : static_cast<double*>(c.work("small_L", sizeof(double) * 2 * (size_t)KLD * KLD));
        hipLaunchKernelGGL(lds ? k_small_solve_big<8> : k_small_solve_big<16>, dim3(1), dim3(BIG_T), 0, c.stream, K, GA,
                           GT, d, sc, fixed_lambda, Lg, z, res, lam_out);
        if (zt && T)
            basis_coef(c, K, T, z, zt);
        else if (zt)
            MMOF_HIP(hipMemcpyAsync(zt, z, sizeof(double) * (size_t)K, hipMemcpyDeviceToDevice, c.stream));
    }
    MMOF_LAUNCH_CHECK();
}

}  // namespace mmof

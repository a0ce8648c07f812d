// Parallel-beam projector H^t (hat model, unit pixels and bins) and its transpose.
//
//   (H u)_{theta,j} = sum_p max(0, 1 - |X_p cos(theta) + Y_p sin(theta) - d_j|) u_p
//
// Forward (ray-driven gather, one lane per detector bin): for |cos| >= |sin| the ray
// crosses every row y once; inside row y the pixels with non-zero weight sit within
// 1/|cos| of xs(y) = cx + (d_j - Y sin)/cos, and their weight is 1 - |cos| |x - xs|.
// Steep angles use the same loop over the columns of a transposed copy of the frame,
// so every lane of a wavefront walks contiguous memory.  Transpose (pixel-driven
// gather, one lane per pixel): each angle contributes (1-f) b[j0] + f b[j0+1] with
// j0 + f = tau_p + (n_d-1)/2.  Sample positions are formed in double (the FP32 forward steps
// through a group of rows in 64-bit fixed point, the FP32 transpose from a tile's centre in FP32);
// the weights are evaluated in the operator's precision.
#include "dev.h"
#include "kernels.h"

namespace mmof {

struct RadonFrame {
    int64_t u_off;     // pixel offset of the frame
    int64_t sino_off;  // offset of its sinogram [n_ang][n_bins]
    int64_t trig_off;  // index of its first angle in the trig table
    int32_t n_ang, n_bins, ny, nx;
};

struct RayTile {
    int32_t frame, angle, bin0, pad;
};

// 64 bins of one angle with what the forward needs of the frame and the angle, in one load.
struct alignas(16) RayRec {
    double c, s;       // the angle
    int64_t u_off;     // pixel offset of the frame
    int64_t out_off;   // offset of the angle's row of the sinogram
    int32_t nx, ny, n_bins, bin0;
};

// Per-frame transpose uT[f][x][y] = u[f][y][x] through a 32x33 LDS tile.
template <class T>
__global__ __launch_bounds__(256) void k_transpose_frames(const Tile* __restrict__ tiles,
                                                          const RadonFrame* __restrict__ rf, const T* __restrict__ u,
                                                          T* __restrict__ ut) {
    __shared__ T s[32][33];
    const Tile tl = tiles[xcd_remap(blockIdx.x, gridDim.x)];
    const RadonFrame f = rf[tl.frame];
    const int lx = threadIdx.x % 32, ly = threadIdx.x / 32;  // 32 x 8
    for (int r = ly; r < 32; r += 8) {
        const int y = tl.y0 + r, x = tl.x0 + lx;
        if (y < f.ny && x < f.nx) s[r][lx] = u[f.u_off + (int64_t)y * f.nx + x];
    }
    __syncthreads();
    for (int r = ly; r < 32; r += 8) {
        const int x = tl.x0 + r, y = tl.y0 + lx;
        if (y < f.ny && x < f.nx) ut[f.u_off + (int64_t)x * f.ny + y] = s[lx][r];
    }
}

// The same transpose with 16-byte accesses, for stacks whose frame sides and offsets are all
// multiples of 4 (Plan::tr_vec): a tile row is 32 / VEC vectors of VEC = 16 / sizeof(T) pixels,
// and each thread reads one (FP32) or two (FP64) of them and writes as many of the transposed
// tile.
template <class T>
__global__ __launch_bounds__(256) void k_transpose_frames4(const Tile* __restrict__ tiles,
                                                           const RadonFrame* __restrict__ rf,
                                                           const T* __restrict__ u, T* __restrict__ ut) {
    constexpr int VEC = 16 / (int)sizeof(T);      // 4 FP32 or 2 FP64 pixels per access
    constexpr int VPR = 32 / VEC;                  // vectors per tile row
    typedef T VT __attribute__((ext_vector_type(VEC)));
    __shared__ T s[32][33];
    const Tile tl = tiles[xcd_remap(blockIdx.x, gridDim.x)];
    const RadonFrame f = rf[tl.frame];
    for (int i = threadIdx.x; i < 32 * VPR; i += 256) {
        const int r = i / VPR, c = VEC * (i % VPR);
        const int y = tl.y0 + r, x = tl.x0 + c;
        if (y < f.ny && x < f.nx) {   // (x < nx implies x + VEC - 1 < nx: nx is a multiple of 4)
            const VT q = *reinterpret_cast<const VT*>(u + f.u_off + (int64_t)y * f.nx + x);
#pragma unroll
            for (int e = 0; e < VEC; ++e) s[r][c + e] = q[e];
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 32 * VPR; i += 256) {
        const int xr = i / VPR, c = VEC * (i % VPR);   // output row (x) and its first y
        const int x = tl.x0 + xr, y = tl.y0 + c;
        if (x < f.nx && y < f.ny) {
            VT q;
#pragma unroll
            for (int e = 0; e < VEC; ++e) q[e] = s[c + e][xr];
            *reinterpret_cast<VT*>(ut + f.u_off + (int64_t)x * f.ny + y) = q;
        }
    }
}

// G rows of a ray whose centre crosses row q (`line`: its first pixel) at xb and moves by step per row:
// with n = round(xs) and d = xs - n in [-1/2, 1/2], the pixels n - 1, n, n + 1 have the weights
// max(0, 1 - |a| (1 + d)), 1 - |a| |d| and max(0, 1 - |a| (1 - d)), and no other pixel is within
// 1/|a| <= sqrt(2) of xs.
// INNER: all three are inside the line on every row.  Otherwise the three are read at the nearest
// place inside (lines of at least 3 pixels), weigh by their own distance and are left out at weight 0.
// FP32: xb - 1/2 (FP64) and step are taken as fixed-point numbers of 32 fraction bits, so that row k is at the sum of
// the first and k steps within 2^-29 px, n - 1 is its upper word and f = d + 1/2 its lower one, rounded to FP32 as a
// fraction formed in FP64 would be.  That is three instructions a row, as many as positions held in FP32 take, which
// are off by up to 1e-6 px: 16 frames of 128 x 128 of either sign, 30 angles: error of H u 1.5e-7 with those, 0.9e-7 so,
// at the same time.  The three pixels come in one 12-byte load at a 32-bit offset from a base
// that is the same for the whole wave, and the outer weights (1 - |a|/2) - |a| f and (1 - 3|a|/2) +
// |a| f are single FMAs clamped to [0, 1] by the FMA's output clamp.
static constexpr double INTERIOR_MARGIN = 1e-3;
static constexpr float FIX_ONE = 4294967296.f;  // 2^32: a whole pixel in units of the last fraction bit

// A number in 32.32 fixed point.
struct Fixed {
    int32_t whole;
    uint32_t frac;
    __device__ __forceinline__ void add(Fixed o) {
        unsigned c;
        frac = __builtin_addc(frac, o.frac, 0u, &c);
        whole = (int32_t)((uint32_t)whole + (uint32_t)o.whole + c);
    }
};

// v in fixed point, its floor clamped to lo .. hi.
__device__ __forceinline__ Fixed fixed32(double v, double lo, double hi) {
    const double fl = floor(v);
    return Fixed{(int32_t)fmin(fmax(fl, lo), hi), (uint32_t)fmin((v - fl) * (double)FIX_ONE, 4294967295.0)};
}

// A position's step per row as hat_rows and fan_rows take it (|step| <= 1).
template <class T>
__device__ __forceinline__ auto row_step(double step) {
    if constexpr (sizeof(T) == 4) return fixed32(step, -1.0, 1.0);
    else return step;
}

template <bool INNER, int G>
__device__ __forceinline__ float hat_rows(const float* __restrict__ line, int ncol, double xb, Fixed step, float aa) {
    // pixel n - 1 and f (positions beyond the line are only known to be beyond it)
    Fixed at = fixed32(xb - 0.5, -16.0, (double)ncol + 16.0);
    const float am = aa / FIX_ONE, cm = 1.f - 0.5f * aa, cp = 1.f - 1.5f * aa;
    const char* __restrict__ base = reinterpret_cast<const char*>(line);
    const uint32_t ncolb = (uint32_t)ncol * 4u;
    typedef float F3 __attribute__((ext_vector_type(3), aligned(4)));
    float s0 = 0.f, s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int k = 0; k < G; ++k) {
        const int i = at.whole;
        const float f = (float)at.frac;  // (times 2^32)
        at.add(step);
        const char* __restrict__ row = base + (size_t)k * ncolb;
        if constexpr (INNER) {
            const F3 q = *reinterpret_cast<const F3*>(row + (uint32_t)(i << 2));
            s0 = fmaf(__builtin_amdgcn_fmed3f(fmaf(-am, f, cm), 0.f, 1.f), q.x, s0);
            s1 = fmaf(fmaf(-am, fabsf(f - 0.5f * FIX_ONE), 1.f), q.y, s1);
            s2 = fmaf(__builtin_amdgcn_fmed3f(fmaf(am, f, cp), 0.f, 1.f), q.z, s2);
        } else {
            const int c = min(max(i, 0), ncol - 3);
            const F3 q = *reinterpret_cast<const F3*>(row + (uint32_t)(c << 2));
            // the centre's distances from the pixels, each rounded once
            const float m = (float)(i - c);
            auto from = [&](float whole) { return fabsf(fmaf(f, 1.f / FIX_ONE, m + whole)); };
            const float w0 = fmaf(-aa, from(0.5f), 1.f), w1 = fmaf(-aa, from(-0.5f), 1.f), w2 = fmaf(-aa, from(-1.5f), 1.f);
            s0 = w0 > 0.f ? fmaf(w0, q.x, s0) : s0;
            s1 = w1 > 0.f ? fmaf(w1, q.y, s1) : s1;
            s2 = w2 > 0.f ? fmaf(w2, q.z, s2) : s2;
        }
    }
    return (s0 + s2) + s1;
}
template <bool INNER, int G>
__device__ __forceinline__ double hat_rows(const double* __restrict__ line, int ncol, double xb, double step,
                                           double aa) {
    typedef double D2 __attribute__((ext_vector_type(2), aligned(8)));
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    const double c0 = 1.0 - aa;
#pragma unroll
    for (int k = 0; k < G; ++k) {
        const double xs = fma((double)k, step, xb);
        const double n = rint(xs);
        const double* __restrict__ row = line + (size_t)k * ncol;
        if constexpr (INNER) {
            const double d = xs - n;
            const double* __restrict__ p = row + ((int)n - 1);
            const D2 q = *reinterpret_cast<const D2*>(p);
            const double q2 = p[2];
            s0 = fma(fmax(fma(-aa, d, c0), 0.0), q.x, s0);
            s1 = fma(fma(-aa, fabs(d), 1.0), q.y, s1);
            s2 = fma(fmax(fma(aa, d, c0), 0.0), q2, s2);
        } else {
            const int i = (int)fmin(fmax(n, -3.0), (double)ncol + 3.0) - 1, c = min(max(i, 0), ncol - 3);
            const double x = xs - (double)c;
            const D2 q = *reinterpret_cast<const D2*>(row + c);
            const double q2 = row[c + 2];
            const double w0 = fma(-aa, fabs(x), 1.0), w1 = fma(-aa, fabs(x - 1.0), 1.0),
                         w2 = fma(-aa, fabs(x - 2.0), 1.0);
            s0 = w0 > 0.0 ? fma(w0, q.x, s0) : s0;
            s1 = w1 > 0.0 ? fma(w1, q.y, s1) : s1;
            s2 = w2 > 0.0 ? fma(w2, q2, s2) : s2;
        }
    }
    return (s0 + s2) + s1;
}
// One row of two pixels (frames too narrow for the three-pixel form).
template <class T>
__device__ __forceinline__ T hat_row2(const T* __restrict__ line, double xs, T aa) {
    T acc = T(0);
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        const T w = T(1) - aa * (T)fabs((double)x - xs);
        if (w > T(0)) acc += w * line[x];
    }
    return acc;
}

// One workgroup of 8 waves per (frame, ANG consecutive angles, 64 bins): lane = bin, wave w takes
// angle w / (8/ANG) and the (w % (8/ANG))-th block of rows, partial sums added in a fixed order.  The
// wave walks its rows together in groups of G, so that a gather's lanes read one row; lanes whose ray
// misses the frame on the whole group sit it out, and the others take the unchecked form when all of
// them stay inside.  Bound by the cache's accesses (16 to 18 per gather: four lanes a cycle) and vector
// issue (12.5 instructions per ray and row).  Measured against waves whose lanes started at rows of
// their own and, on blocks of less than 48 rows, checked every pixel: FP32 128 x 128 x 16, 30 angles
// 23 -> 12 us, 256 x 256 x 16 61 -> 27 us, 1024 x 1024 x 64, 90 angles 2.99 -> 2.71 ms; FP64 251 x 310 x
// 16, 45 angles 126 -> 70 us, 1024 x 1024 x 16, 90 angles 1.59 -> 1.46 ms.
// ANG = 1 finds frame and angle in its record, where they were three loads one after the other (0.7 us of the first).
template <class T, int ANG>
__global__ __launch_bounds__(512) void k_radon_fwd(const RayTile* __restrict__ rays, const RadonFrame* __restrict__ rf,
                                                   const double2* __restrict__ trig, const RayRec* __restrict__ recs,
                                                   const T* __restrict__ u,
                                                   const T* __restrict__ ut, T* __restrict__ b) {
    constexpr int RSL = 8 / ANG;
    constexpr int G = sizeof(T) == 4 ? 8 : 4;
    __shared__ T part[8][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // (uniform: angle, image in SGPRs)
    const int sl = wave % RSL;
    RayRec f;
    bool have = true;  // the wave's angle exists
    if constexpr (ANG == 1) {
        f = recs[xcd_remap(blockIdx.x, gridDim.x)];
    } else {
        const RayTile rt = rays[xcd_remap(blockIdx.x, gridDim.x)];
        const RadonFrame fr = rf[rt.frame];
        const int ang = rt.angle + wave / RSL;
        have = ang < fr.n_ang;
        const double2 cs = trig[fr.trig_off + min(ang, fr.n_ang - 1)];
        f = RayRec{cs.x, cs.y, fr.u_off, fr.sino_off + (int64_t)ang * fr.n_bins, fr.nx, fr.ny, fr.n_bins, rt.bin0};
    }
    const int j = f.bin0 + lane;
    T acc = T(0);
    if (have && j < f.n_bins) {
        const double c = f.c, s = f.s;
        const double cx = 0.5 * (f.nx - 1), cy = 0.5 * (f.ny - 1);
        const double dj = (double)j - 0.5 * (f.n_bins - 1);
        // row walk over (rows, cols) = (ny, nx) of u, or over (nx, ny) of the transpose
        const bool steep = fabs(s) > fabs(c);
        const double a = steep ? s : c;   // coefficient of the in-row coordinate
        const double bb = steep ? c : s;  // coefficient of the row coordinate
        const int nrow = steep ? f.nx : f.ny, ncol = steep ? f.ny : f.nx;
        const double crow = steep ? cx : cy, ccol = steep ? cy : cx;
        const T* img = (steep ? ut : u) + f.u_off;
        // ray centre in row r: xs(r) = ccol + (dj - (r - crow) bb) / a
        const double xs0 = ccol + (dj + crow * bb) / a;
        const double step = -bb / a;
        const auto row_st = row_step<T>(step);
        const T aa = (T)fabs(a);
        const double x_in_lo = 0.5 + INTERIOR_MARGIN, x_in_hi = (double)ncol - 1.5 - INTERIOR_MARGIN;
        const int q_n = ((nrow + RSL - 1) / RSL + G - 1) / G * G;
        const int q_hi = min(nrow, (sl + 1) * q_n);
        int q = sl * q_n;
        for (; ncol < 3 && q < q_hi; q += G) {
            const double xb = fma((double)q, step, xs0), xe = fma((double)(G - 1), step, xb);
            if (!__any(fmax(xb, xe) > -1.5 && fmin(xb, xe) < (double)ncol + 0.5)) continue;
            for (int r = q; r < min(q + G, q_hi); ++r)
                acc += hat_row2(img + (int64_t)r * ncol, fma((double)r, step, xs0), aa);
        }
        for (; q < q_hi; q += G) {
            const T* line = img + (int64_t)q * ncol;
            const double xb = fma((double)q, step, xs0), xe = fma((double)(G - 1), step, xb);
            const double lo = fmin(xb, xe), hi = fmax(xb, xe);
            // (a ray weighs on pixels within sqrt(2) of its centre)
            const bool near = hi > -1.5 && lo < (double)ncol + 0.5;
            if (!__any(near)) continue;
            if (q + G <= q_hi) {
                const bool inner = __all(!near || (lo >= x_in_lo && hi < x_in_hi));
                if (near) {
                    // (the unchecked form also multiplies pixels of weight 0, which must not count when they are not
                    // finite: a group whose sum is not is taken again; 0.5% at 1024 x 1024)
                    T v = T(0);
                    if (inner) v = hat_rows<true, G>(line, ncol, xb, row_st, aa);
                    if (!inner || !isfinite(v)) v = hat_rows<false, G>(line, ncol, xb, row_st, aa);
                    acc += v;
                }
            } else {
                for (int r = q; r < q_hi; ++r, line += ncol)
                    acc += hat_rows<false, 1>(line, ncol, fma((double)r, step, xs0), row_st, aa);
            }
        }
    }
    part[wave][lane] = acc;
    __syncthreads();
    if (sl == 0 && have && j < f.n_bins) {
        T sum[RSL];
#pragma unroll
        for (int k = 0; k < RSL; ++k) sum[k] = part[wave + k][lane];
#pragma unroll
        for (int h = RSL / 2; h >= 1; h /= 2)  // (pairwise: fewer roundings than one after the other)
#pragma unroll
            for (int k = 0; k < h; ++k) sum[k] += sum[k + h];
        b[f.out_off + j] = sum[0];
    }
}

// Transpose: one workgroup per 32 x 16 PY pixel tile, each lane 2 PY pixels 16 apart in its rows
// and columns.  For each angle the tile projects onto fewer than AW - 2 consecutive bins (its
// extent sqrt(31^2 + 31^2) < 44 bins for PY = 2); those sinogram windows are staged in LDS, AC
// angles at a time, as pairs (b_j, b_{j+1} - b_j) with zeros outside the detector, and a pixel
// then gathers b_j0 + f (b_j0+1 - b_j0) per angle with one LDS load.  FP32: per 16 rows of
// the tile and angle the detector coordinate of their centre in FP64, split into its floor J and an
// FP32 fraction; the lane's first pixel at (dx, dy) from that centre (|dx| <= 15.5, |dy| <= 7.5) is
// at J + t, t = frac + dx cos + dy sin in FP32, the second at t + 16 cos (error below 5e-6 bins,
// whatever PY), and the weights come from floor(t) and fract(t); the window has one bin of margin on
// each side, so a floor one off at an integer stays inside it (and gives the same value).  FP64: each lane's first position in FP64 from its own coordinates, the others 16 cos and 16 sin further,
// counted from the window's first bin: at least 1, so that the bin is one conversion and the weight
// one fract.
// The windows cover the whole tile, also where it overhangs the frame, so every lane's
// gathers stay inside them; pixels outside the frame are not written.
// Bound by the reads of the LDS (per angle and lane the record of the angle, 16 or 24 bytes, and a
// pair per pixel) and by vector issue: four pixels share a record and a window where two did.
// 1024 x 1024 x 16, 90 angles: FP32 280 -> 265 us, FP64 565 -> 367 (470 from the cheaper positions
// alone); 16 x 128 x 128, 30 angles, FP64 (PY = 1) 6.4 -> 5.8; 251 x 310 x 16, 45 angles, FP64 32 -> 23.
static constexpr int ATW = 32, ATH = 16;  // pixel tiles of the transposes (parallel with PY = 1, and fan beam)
static constexpr int AW = 48, AC = 32;

struct AdjAngle {
    float frac;
    uint32_t base;   // LDS byte offset of bin J in the angle's window (from the window array)
    float c, s;
};

struct AdjAngle64 {
    double c, s, at;   // at: the detector coordinate of the frame's centre, counted from the window's first bin
};

template <class T, int PY>
__global__ __launch_bounds__(256, PY == 1 && sizeof(T) == 4 ? 6 : 4) void k_radon_adj(
    const Tile* __restrict__ tiles, const RadonFrame* __restrict__ rf, const double2* __restrict__ trig,
    const T* __restrict__ b, T* __restrict__ u) {
    constexpr int TH = ATH * PY;
    typedef T P2 __attribute__((ext_vector_type(2)));  // {b_j, b_{j+1} - b_j}
    __shared__ P2 win[AC][AW];
    __shared__ int jlo[AC];
    __shared__ AdjAngle64 scs[AC];
    __shared__ AdjAngle aa[PY][AC];
    const Tile tl = tiles[xcd_remap(blockIdx.x, gridDim.x)];
    const RadonFrame f = rf[tl.frame];
    const int lx = (int)(threadIdx.x % 16), ly = (int)(threadIdx.x / 16);
    const int x = tl.x0 + lx, y = tl.y0 + ly;  // the lane's first pixel
    const double hx = 0.5 * (f.nx - 1), hy = 0.5 * (f.ny - 1);
    const double X = x - hx, Y = y - hy;
    const double cd = 0.5 * (f.n_bins - 1);
    // corners of the whole tile for the window bounds
    const double X0 = tl.x0 - hx, X1 = tl.x0 + ATW - 1 - hx;
    const double Y0 = tl.y0 - hy, Y1 = tl.y0 + TH - 1 - hy;
    const T* sino = b + f.sino_off;
    T acc[PY][2] = {};
    const double XC = tl.x0 + 0.5 * (ATW - 1) - hx, YC = tl.y0 + 0.5 * (ATH - 1) - hy;
    const float dxc = (float)lx - 0.5f * (ATW - 1);
    const float dyc = (float)ly - 0.5f * (ATH - 1);
    for (int k0 = 0; k0 < f.n_ang; k0 += AC) {
        const int nk = min(AC, f.n_ang - k0);
        __syncthreads();  // the previous chunk's windows are no longer read
        if (threadIdx.x < nk) {
            const double2 cs = trig[f.trig_off + k0 + threadIdx.x];
            const double pmin = cd + fmin(X0 * cs.x, X1 * cs.x) + fmin(Y0 * cs.y, Y1 * cs.y);
            const int lo = (int)floor(pmin) - 1;
            jlo[threadIdx.x] = lo;
            if constexpr (sizeof(T) == 8) {
                scs[threadIdx.x] = AdjAngle64{cs.x, cs.y, cd - lo};
            } else {
#pragma unroll
                for (int r = 0; r < PY; ++r) {
                    const double pc = fma(XC, cs.x, fma(YC + ATH * r, cs.y, cd));
                    const double J = floor(pc);
                    aa[r][threadIdx.x] =
                        AdjAngle{(float)(pc - J), (uint32_t)((int)threadIdx.x * AW + (int)J - lo) * (uint32_t)sizeof(P2),
                                 (float)cs.x, (float)cs.y};
                }
            }
        }
        __syncthreads();
        // (a chunk's loads all in flight together: 16 x 128 x 128, FP32, 30 angles 5.9 -> 5.7 us)
        constexpr int NW = AC * AW / 256;
        T v0[NW], v1[NW];
#pragma unroll
        for (int m = 0; m < NW; ++m) {
            const int i = (int)threadIdx.x + 256 * m, kk = i / AW;
            v0[m] = v1[m] = T(0);
            if (kk < nk) {
                const int j = jlo[kk] + i % AW;
                const T* row = sino + (int64_t)(k0 + kk) * f.n_bins;
                if (j >= 0 && j < f.n_bins) v0[m] = row[j];
                if (j + 1 >= 0 && j + 1 < f.n_bins) v1[m] = row[j + 1];
            }
        }
#pragma unroll
        for (int m = 0; m < NW; ++m) {
            const int i = (int)threadIdx.x + 256 * m;
            if (i / AW < nk) win[i / AW][i % AW] = P2{v0[m], v1[m] - v0[m]};
        }
        __syncthreads();
        if (x >= f.nx || y >= f.ny) continue;
        if constexpr (sizeof(T) == 4) {
            const char* wb = reinterpret_cast<const char*>(&win[0][0]);
            float a[PY][2] = {}, d[PY][2] = {};
            auto one = [&](int kk) {
                const float gc = aa[0][kk].c, gs = aa[0][kk].s;
#pragma unroll
                for (int r = 0; r < PY; ++r) {
                    const float tr = fmaf(dxc, gc, fmaf(dyc, gs, aa[r][kk].frac));
                    const uint32_t base = aa[r][kk].base;
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const float t = e ? fmaf(16.f, gc, tr) : tr;
                        int w;
                        asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(w) : "v"(t));
                        const P2 v = *reinterpret_cast<const P2*>(wb + (base + ((uint32_t)w << 3)));
                        a[r][e] += v.x;
                        d[r][e] = fmaf(__builtin_amdgcn_fractf(t), v.y, d[r][e]);
                    }
                }
            };
            int kk = 0;
            for (; kk + 4 <= nk; kk += 4) {
                one(kk);
                one(kk + 1);
                one(kk + 2);
                one(kk + 3);
            }
            for (; kk < nk; ++kk) one(kk);
#pragma unroll
            for (int q = 0; q < 2 * PY; ++q) acc[q / 2][q % 2] += a[q / 2][q % 2] + d[q / 2][q % 2];
        } else {
#pragma unroll 4
            for (int kk = 0; kk < nk; ++kk) {
                const AdjAngle64 g = scs[kk];
                const double pf = fma(X, g.c, fma(Y, g.s, g.at));
#pragma unroll
                for (int q = 0; q < 2 * PY; ++q) {
                    const int r = q / 2, e = q % 2;
                    const double pr = r ? fma(16.0, g.s, pf) : pf;
                    const double t = e ? fma(16.0, g.c, pr) : pr;
                    const P2 v = win[kk][(int)t];  // (t >= 1, so truncation is the floor)
                    acc[r][e] += v.x + (T)__builtin_amdgcn_fract(t) * v.y;
                }
            }
        }
    }
#pragma unroll
    for (int q = 0; q < 2 * PY; ++q) {
        const int px = x + 16 * (q % 2), py = y + 16 * (q / 2);
        if (px < f.nx && py < f.ny) u[f.u_off + (int64_t)py * f.nx + px] = acc[q / 2][q % 2];
    }
}

// ----------------------------------------------------------------------------- host side

void radon_plan_init(Ctx& c, Plan& p, const double* cs) {
    Geom& g = *p.geom;
    std::vector<RadonFrame> rfs;
    std::vector<RayTile> rays[4];  // angle groups of 1, 2, 4, 8
    std::vector<RayRec> recs;      // those of 1 (parallel beam)
    std::vector<Tile> px, tr;
    int64_t sino = 0, trig = 0;
    p.tr_vec = true;
    size_t n_recs = 0;
    for (int64_t fi = 0; fi < g.n_frames; ++fi)
        n_recs += (size_t)p.n_ang[g.frames[fi].seq] * (size_t)cdiv(p.n_bins[g.frames[fi].seq], 64);
    rays[0].reserve(n_recs);
    if (p.kind == 0) recs.reserve(n_recs);
    for (int64_t fi = 0; fi < g.n_frames; ++fi) {
        const FrameInfo& fr = g.frames[fi];
        // the projectors address pixels by 32-bit offsets within a frame
        MMOF_CHECK((int64_t)fr.ny * fr.nx < ((int64_t)1 << 31), MMOF_ERR_SHAPE, "frames must have fewer than 2^31 pixels");
        if (fr.nx % 4 != 0 || fr.ny % 4 != 0 || fr.off % 4 != 0) p.tr_vec = false;
        RadonFrame r{};
        r.u_off = fr.off;
        r.sino_off = sino;
        r.trig_off = trig;
        r.n_ang = p.n_ang[fr.seq];
        r.n_bins = p.n_bins[fr.seq];
        r.ny = fr.ny;
        r.nx = fr.nx;
        rfs.push_back(r);
        p.sino_off.push_back(sino);
        // a frame's angle groups that walk the rows of u, then those that walk the rows of its
        // transpose (a group is placed by its first angle): consecutive tiles, which run together
        // on one XCD (xcd_remap), then read one image, not both
        for (int gi = 0; gi < 4; ++gi) {
            const int ag = 1 << gi;
            for (int pass = 0; pass < 2; ++pass)
                for (int k = 0; k < r.n_ang; k += ag) {
                    const double c0 = cs[2 * (trig + k)], s0 = cs[2 * (trig + k) + 1];
                    if ((std::fabs(s0) > std::fabs(c0)) != (pass == 1)) continue;
                    for (int j0 = 0; j0 < r.n_bins; j0 += 64) {
                        rays[gi].push_back(RayTile{(int32_t)fi, k, j0, 0});
                        if (gi == 0 && p.kind == 0)
                            recs.push_back(RayRec{c0, s0, fr.off, sino + (int64_t)k * r.n_bins, fr.nx, fr.ny, r.n_bins,
                                                  j0});
                    }
                }
        }
        // pixel tiles of the transposes
        for (int y0 = 0; y0 < fr.ny; y0 += ATH)
            for (int x0 = 0; x0 < fr.nx; x0 += ATW) px.push_back(Tile{(int32_t)fi, y0, x0, 0});
        for (int y0 = 0; y0 < fr.ny; y0 += 32)
            for (int x0 = 0; x0 < fr.nx; x0 += 32) tr.push_back(Tile{(int32_t)fi, y0, x0, 0});
        sino += (int64_t)r.n_ang * r.n_bins;
        trig += r.n_ang;
        p.radon_flops += 4.0 * (double)fr.ny * fr.nx * r.n_ang;
    }
    p.m = sino;
    p.d_rinfo.ensure(sizeof(RadonFrame) * rfs.size());
    MMOF_HIP(hipMemcpyAsync(p.d_rinfo.ptr, rfs.data(), sizeof(RadonFrame) * rfs.size(), hipMemcpyHostToDevice, c.stream));
    for (int gi = 0; gi < 4; ++gi) {
        p.n_rays[gi] = (int64_t)rays[gi].size();
        p.d_rays[gi].ensure(sizeof(RayTile) * std::max<size_t>(rays[gi].size(), 1));
        if (!rays[gi].empty())
            MMOF_HIP(hipMemcpyAsync(p.d_rays[gi].ptr, rays[gi].data(), sizeof(RayTile) * rays[gi].size(),
                                    hipMemcpyHostToDevice, c.stream));
    }
    if (!recs.empty()) {
        p.d_ray_recs.ensure(sizeof(RayRec) * recs.size());
        MMOF_HIP(hipMemcpyAsync(p.d_ray_recs.ptr, recs.data(), sizeof(RayRec) * recs.size(), hipMemcpyHostToDevice,
                                c.stream));
    }
    p.n_tiles_a = (int64_t)px.size();
    p.d_tiles_a.ensure(sizeof(Tile) * px.size());
    MMOF_HIP(hipMemcpyAsync(p.d_tiles_a.ptr, px.data(), sizeof(Tile) * px.size(), hipMemcpyHostToDevice, c.stream));
    p.n_tiles_b = (int64_t)tr.size();
    p.d_tiles_b.ensure(sizeof(Tile) * tr.size());
    MMOF_HIP(hipMemcpyAsync(p.d_tiles_b.ptr, tr.data(), sizeof(Tile) * tr.size(), hipMemcpyHostToDevice, c.stream));
    MMOF_HIP(hipStreamSynchronize(c.stream));
}

// ---------------------------------------------------------------- fan beam
//
// Flat-detector fan beam by Joseph's method.  Angle theta: detector axis a = (cos, sin),
// central ray e = (-sin, cos), source S = -dso e, ray j along d_j = dsd e + u_j a with
// u_j = (j - (n_d-1)/2) du.  A ray with |d_y| >= |d_x| is sampled on every pixel row at
// X_c(Y) = S_x + (Y - S_y) d_x / d_y by linear interpolation between the two pixels around
// it (out-of-frame pixels are 0), each sample weighted by the path length per row
// |d| / |d_y|; other rays on the columns.  Forward: one lane per ray, column-stepping rays read
// the transposed frame so that the lanes stay on neighbouring addresses.  Transpose: a lane per
// pixel or two; per angle, the rays that can sample the pixel are those whose detector
// coordinate lies between the projections of its row neighbours (X -+ 1, Y) or of its column
// neighbours (X, Y -+ 1); each candidate ray's weight on the pixel is formed from the same
// crossing as in the forward.

struct FanGeo {
    double dso, dsd, du;
};

// Source and direction of ray j (no contraction: the row / column choice is taken on values
// rounded exactly like plain double arithmetic).
__device__ __forceinline__ void fan_ray(double c, double s, int j, int nb, const FanGeo& g, double& sx, double& sy,
                                        double& dx, double& dy) {
#pragma clang fp contract(off)
    const double uj = ((double)j - (nb - 1) / 2.0) * g.du;
    dx = -g.dsd * s + uj * c;
    dy = g.dsd * c + uj * s;
    sx = g.dso * s;
    sy = -g.dso * c;
}

// Per-ray table, built once per plan in the sinogram layout: {A, B, step, dir} with the
// sample position of the ray on row y (dir > 0: |d_y| >= |d_x|) x_c = A + B y, or on column
// x (dir < 0) y_c = A + B x, in pixel-index coordinates, and the path length per step.  Both
// the forward and the transpose evaluate positions as fma(B, index, A) from this table, so
// their weights are the same numbers.
__global__ __launch_bounds__(256) void k_fan_rays(const RayTile* __restrict__ rays, const RadonFrame* __restrict__ rf,
                                                  const double2* __restrict__ trig, FanGeo geo,
                                                  double4* __restrict__ table) {
    const RayTile rt = rays[xcd_remap(blockIdx.x, gridDim.x)];
    const RadonFrame f = rf[rt.frame];
    const int k = rt.angle + (int)threadIdx.x / 64, j = rt.bin0 + (int)threadIdx.x % 64;
    if (k >= f.n_ang || j >= f.n_bins) return;
    const double2 cs = trig[f.trig_off + k];
    double sx, sy, dx, dy;
    fan_ray(cs.x, cs.y, j, f.n_bins, geo, sx, sy, dx, dy);
    const double cx = (f.nx - 1) / 2.0, cy = (f.ny - 1) / 2.0;
    double4 e;
    if (fabs(dy) >= fabs(dx)) {
        e.y = dx / dy;
        e.x = sx + (-cy - sy) * e.y + cx;
        e.z = sqrt(dx * dx + dy * dy) / fabs(dy);
        e.w = 1.0;
    } else {
        e.y = dy / dx;
        e.x = sy + (-cx - sx) * e.y + cy;
        e.z = sqrt(dx * dx + dy * dy) / fabs(dx);
        e.w = -1.0;
    }
    table[f.sino_off + (int64_t)k * f.n_bins + j] = e;
}

// G samples of a lane's ray on lines q .. q + G - 1 (q the same for the wave; `line` points to line q
// of the image): the sample's two neighbours are weighted 1 - f and f.
// INNER: every lane's samples have both neighbours inside the line.  Otherwise the pair is read at
// the nearest place inside, and a pixel of it counts where it is within one of the position.
// FP32: positions in fixed point with 32 fraction bits, as in hat_rows; the pair is one 8-byte load at a 32-bit offset
// within its line.
template <bool INNER, int G>
__device__ __forceinline__ float fan_rows(const float* __restrict__ line, int nline, double xb, Fixed step) {
    Fixed at = fixed32(xb, -16.0, (double)nline + 16.0);
    const char* __restrict__ base = reinterpret_cast<const char*>(line);
    const uint32_t nlineb = (uint32_t)nline * 4u;
    typedef float F2 __attribute__((ext_vector_type(2), aligned(4)));
    float s0 = 0.f, s1 = 0.f;
#pragma unroll
    for (int k = 0; k < G; ++k) {
        const int i = at.whole;
        const float f = (float)at.frac;  // (times 2^32)
        at.add(step);
        const char* __restrict__ row = base + (size_t)k * nlineb;
        if constexpr (INNER) {
            const F2 v = *reinterpret_cast<const F2*>(row + (uint32_t)(i << 2));
            s0 = fmaf(fmaf(f, -1.f / FIX_ONE, 1.f), v.x, s0);
            s1 = fmaf(f * (1.f / FIX_ONE), v.y, s1);
        } else {
            const int c = min(max(i, 0), nline - 2);
            const F2 v = *reinterpret_cast<const F2*>(row + (uint32_t)(c << 2));
            // the position, from each pixel of the pair
            const float m = (float)(i - c);
            const float w0 = 1.f - fabsf(fmaf(f, 1.f / FIX_ONE, m)), w1 = 1.f - fabsf(fmaf(f, 1.f / FIX_ONE, m - 1.f));
            s0 = w0 > 0.f ? fmaf(w0, v.x, s0) : s0;
            s1 = w1 > 0.f ? fmaf(w1, v.y, s1) : s1;
        }
    }
    return s0 + s1;
}
template <bool INNER, int G>
__device__ __forceinline__ double fan_rows(const double* __restrict__ line, int nline, double A, double Bs, int q) {
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < G; ++k) {
        const double pc = fma(Bs, (double)(q + k), A);
        const double fl = floor(pc), f = pc - fl;
        const double* __restrict__ row = line + (size_t)k * nline;
        if constexpr (INNER) {
            const Pair<double> v = ld2(row + (int)fl);
            acc += (1.0 - f) * v.a;
            acc += f * v.b;
        } else {
            const int i = (int)fmin(fmax(fl, -2.0), (double)nline + 2.0), c = min(max(i, 0), nline - 2);
            const Pair<double> v = ld2(row + c);
            // (one pixel off the pair at most counts: i = c, or i = -1, or i = nline - 1)
            const double w0 = i == c ? 1.0 - f : (i == c - 1 ? f : 0.0);
            const double w1 = i == c ? f : (i == c + 1 ? 1.0 - f : 0.0);
            if (w0 != 0.0) acc += w0 * v.a;
            if (w1 != 0.0) acc += w1 * v.b;
        }
    }
    return acc;
}

// A workgroup of 4 waves takes 4 / RSL angles x 64 bins, a ray's lines split over RSL waves (their
// partial sums added in a fixed order): one lane per ray.  The wave walks the lines together, so that
// a gather's lanes read one line (with a start of its own per lane a gather touched 24 cache lines,
// measured 162e6 accesses for 6.7e6 loads); a group of lines takes the unchecked form when the
// positions of all its rays stay inside, and is skipped when none comes near.  Bound by the cache's
// accesses (17 per gather: four lanes a cycle) and vector issue.  FP32, 512 x 512 x 16, 90 angles,
// 725 bins: 455 -> 241 us; 128 x 128 x 16, 30 angles: 43 -> 12 us (the ray split over four waves).
template <class T, int RSL>
__global__ __launch_bounds__(256) void k_fan_fwd(const RayTile* __restrict__ rays, const RadonFrame* __restrict__ rf,
                                                 const double4* __restrict__ table, const T* __restrict__ u,
                                                 const T* __restrict__ ut, T* __restrict__ b) {
    constexpr int G = sizeof(T) == 4 ? 8 : 4;
    __shared__ T part[4][64];
    const RayTile rt = rays[xcd_remap(blockIdx.x, gridDim.x)];
    const RadonFrame f = rf[rt.frame];
    const int lane = (int)threadIdx.x % 64;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int k = rt.angle + wave / RSL, sl = wave % RSL, j = rt.bin0 + lane;
    const bool ray = k < f.n_ang && j < f.n_bins;
    const int64_t ri = f.sino_off + (int64_t)k * f.n_bins + j;
    const double4 e = ray ? table[ri] : make_double4(0.0, 0.0, 0.0, 0.0);
    T acc = T(0);
    const auto row_st = row_step<T>(e.y);
    // rows: samples along x of row y; columns: along y of column x (transposed frame).  A wave
    // whose rays are of both kinds walks both.
    for (int kind = 0; kind < 2; ++kind) {
        const bool mine = ray && (e.w > 0.0) == (kind == 0);
        if (!__any(mine)) continue;
        const int nsteps = kind == 0 ? f.ny : f.nx, nline = kind == 0 ? f.nx : f.ny;
        const T* img = (kind == 0 ? u : ut) + f.u_off;
        const int q_n = ((nsteps + RSL - 1) / RSL + G - 1) / G * G;
        const int q_hi = min(nsteps, (sl + 1) * q_n);
        if (mine) {
            for (int q = sl * q_n; q < q_hi; q += G) {
                const T* line = img + (int64_t)q * nline;
                const double xb = fma(e.y, (double)q, e.x);
                // |B| <= 1: the group's positions stay within G of the first
                if (!__any(xb > -1.0 - G && xb < (double)(nline + G))) continue;
                const double xe = fma((double)(G - 1), e.y, xb);
                const bool inner = fmin(xb, xe) >= INTERIOR_MARGIN && fmax(xb, xe) < (double)(nline - 1) - INTERIOR_MARGIN;
                if constexpr (sizeof(T) == 4) {
                    if (q + G <= q_hi) {
                        if (__all(inner)) acc += fan_rows<true, G>(line, nline, xb, row_st);
                        else acc += fan_rows<false, G>(line, nline, xb, row_st);
                    } else {
                        for (int r = q; r < q_hi; ++r, line += nline)
                            acc += fan_rows<false, 1>(line, nline, fma(e.y, (double)r, e.x), row_st);
                    }
                } else {
                    if (q + G <= q_hi) {
                        if (__all(inner)) acc += fan_rows<true, G>(line, nline, e.x, e.y, q);
                        else acc += fan_rows<false, G>(line, nline, e.x, e.y, q);
                    } else {
                        for (int r = q; r < q_hi; ++r, line += nline)
                            acc += fan_rows<false, 1>(line, nline, e.x, e.y, r);
                    }
                }
            }
        }
    }
    if constexpr (RSL == 1) {
        if (ray) b[ri] = acc * (T)e.z;
    } else {
        part[wave][lane] = acc;
        __syncthreads();
        if (sl == 0 && ray) {
            T sum = T(0);
#pragma unroll
            for (int w = 0; w < RSL; ++w) sum += part[wave + w][lane];
            b[ri] = sum * (T)e.z;
        }
    }
}

// Detector position (in bin units) of the ray from the source through the point (X, Y); the
// reciprocal of the depth from the hardware FP32 reciprocal and two Newton steps (relative
// error near FP64 rounding, no FP64 division): it only bounds candidate rays (margin 0.05 bins).
__device__ __forceinline__ double fan_pos_bound(double X, double Y, double c, double s, double dso, double g,
                                                double off) {
    const double t = X * c + Y * s, den = dso - X * s + Y * c;
    double inv = (double)__builtin_amdgcn_rcpf((float)den);
    inv = inv * (2.0 - den * inv);
    inv = inv * (2.0 - den * inv);
    return g * t * inv + off;
}

__device__ __forceinline__ float uniform(float v) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

constexpr int FAC = 16;  // angles per staged chunk of the transpose
constexpr int FAW = 96;  // staged bins per angle (wider tile windows read the table directly)

// What the pixels of a tile share at one angle: the position of a pixel (X, Y) in the staged window
// is g t / den + off (t = X c + Y s, den = dso - X s + Y c; gc = g c, gs = g s), and the n bins from
// floor(position - h) + 1 on hold every ray that weighs on it.  The window: cnt bins from j0 on, nray
// of them on the detector (cnt 0: nothing to add, < 0: not staged).
struct FanAngle {
    float c, s, gc, gs, off, h;  // off includes 1 - h
    int n, j0, cnt, nray;
};

// Transpose: a 32 x 16 pixel tile per workgroup (TH = 8: half a tile, for small frames), a lane PX = 2 pixels 16 apart in a
// row (PX = 1: one pixel, twice the lanes, for stacks of too few tiles to fill the chip).  Per chunk of FAC angles, the
// bins whose rays can touch the tile are staged in LDS as the line {A, B} and the product of path
// length and sinogram value.  A ray j weighs on a pixel by 1 - |d| with d the distance from the pixel
// to the ray's crossing of its row (column), where that is positive; it sits at detector position j,
// and moving the pixel by one along the row (column) moves its own position by at most h (the
// largest derivative of the position over the tile grown by one pixel), so the rays within h of the
// pixel's position are the candidates: their number is the same for the whole tile, the loop over
// them does not diverge, and a candidate that misses the pixel falls out by its weight.  The
// position only selects candidates: FP32, with the caller's margin in h.  The crossings are the
// forward's fma(B, index, A) in FP64.  Windows wider than FAW bins, geometries whose FP32 margin
// would exceed half a bin (fp32 = 0) and angles where the source comes near the tile take the
// candidates between the FP64 projections of the pixel's four neighbours, from the table.
// Bound by vector issue: 46 instructions per pixel and angle, about 8 of them per candidate (four
// projections per pixel and 20 per candidate before).  FP32, 512 x 512 x 16, 90 angles, 725 bins:
// 1008 -> 534 us; 128 x 128 x 16, 30 angles: 33 -> 26 us.
template <class T, int PX, int TH>
__global__ __launch_bounds__(ATW * TH / PX) void k_fan_adj(const Tile* __restrict__ tiles,
                                                      const RadonFrame* __restrict__ rf,
                                                      const double2* __restrict__ trig,
                                                      const double4* __restrict__ table, const T* __restrict__ b,
                                                      T* __restrict__ u, FanGeo geo, float margin, int fp32) {
    constexpr int NT = ATW * TH / PX, TX = ATW / PX, PARTS = ATH / TH;  // threads, lanes per tile row, workgroups per tile
    constexpr bool OWN = TH < ATH;  // candidates by the lane's own half-width (one pixel a lane)
    static_assert(!OWN || PX == 1, "one pixel a lane");
    __shared__ double2 s_ab[FAC][FAW];
    __shared__ T s_v[FAC][FAW];
    __shared__ FanAngle s_ang[FAC];
    __shared__ int s_ncol[FAC];                  // column rays of the window
    __shared__ unsigned s_cols[FAC][FAW / 32];   // which they are
    const int64_t item = xcd_remap(blockIdx.x, gridDim.x);
    Tile tl = tiles[item / PARTS];
    tl.y0 += TH * (int)(item % PARTS);
    const RadonFrame f = rf[tl.frame];
    if (tl.y0 >= f.ny) return;
    const int lx = (int)threadIdx.x % TX, y0 = tl.y0 + (int)threadIdx.x / TX;
    bool in[PX];
    int xs[PX];
    double xd[PX];
    float Xf[PX];
    T acc[PX];
    const double hx = (f.nx - 1) / 2.0, hy = (f.ny - 1) / 2.0;
    // pixels beyond the frame compute the nearest one's value and do not store it
    const int y = min(y0, f.ny - 1);
    const double yd = (double)y;
    const float Yf = (float)(y - hy);
#pragma unroll
    for (int p = 0; p < PX; ++p) {
        const int x = tl.x0 + lx + TX * p;
        in[p] = x < f.nx && y0 < f.ny;
        xs[p] = min(x, f.nx - 1);
        xd[p] = (double)xs[p];
        Xf[p] = (float)(xs[p] - hx);
        acc[p] = T(0);
    }
    const int nb = f.n_bins;
    const double gsc = geo.dsd / geo.du, off = (nb - 1) / 2.0;
    const float dsof = (float)geo.dso, gscf = (float)gsc;
    // the tile's pixels, clipped to the frame
    const double Xa = tl.x0 - hx, Xb = min(tl.x0 + ATW, f.nx) - 1 - hx, Ya = tl.y0 - hy,
                 Yb = min(tl.y0 + TH, f.ny) - 1 - hy;
    for (int k0 = 0; k0 < f.n_ang; k0 += FAC) {
        const int nk = min(FAC, f.n_ang - k0);
        __syncthreads();  // the previous chunk is no longer read
        if (threadIdx.x < 4 * FAC) {
            // four lanes per angle: one corner each, the extremes over the four
            const int kk = min((int)threadIdx.x / 4, nk - 1), corner = (int)threadIdx.x % 4;
            const double2 cs = trig[f.trig_off + k0 + kk];
            const double X = corner & 1 ? Xb : Xa, Y = corner & 2 ? Yb : Ya;
            // the corner grown by one pixel
            const double Xg = corner & 1 ? Xb + 1.0 : Xa - 1.0, Yg = corner & 2 ? Yb + 1.0 : Ya - 1.0;
            double lo = fan_pos_bound(X, Y, cs.x, cs.y, geo.dso, gsc, off), hi = lo;
            // derivatives of the position: g (c dso + Y) / den^2 along X, g (s dso - X) / den^2 along Y
            double den = geo.dso - Xg * cs.y + Yg * cs.x;
            double mv = fmax(fabs(cs.x * geo.dso + Yg), fabs(cs.y * geo.dso - Xg));
#pragma unroll
            for (int o = 1; o < 4; o *= 2) {
                lo = fmin(lo, __shfl_xor(lo, o));
                hi = fmax(hi, __shfl_xor(hi, o));
                den = fmin(den, __shfl_xor(den, o));
                mv = fmax(mv, __shfl_xor(mv, o));
            }
            const double h = gsc * mv / (den * den) + (double)margin;
            FanAngle a{(float)cs.x, (float)cs.y, (float)(gsc * cs.x), (float)(gsc * cs.y), 0.f, (float)h, 0, 0, -1, 0};
            if (fp32 && den > 0.0 && h < FAW) {
                // (FP32 positions reach from lo - margin to hi + margin)
                a.j0 = (int)fmin(fmax(floor(lo - h - 1.0), -1048576.0), 1048576.0);
                const double top = fmin(fmax(ceil(hi + h + 1.0), -1048576.0), 1048576.0);
                a.n = (int)floor(2.0 * h) + 1;
                a.off = (float)(off - (double)a.j0 - h + 1.0);
                const double need = top - a.j0 + 1.0 + a.n;
                if (need <= FAW) {
                    a.cnt = (int)need;
                    a.nray = min(a.j0 + a.cnt, nb) - max(a.j0, 0);
                    if (a.nray <= 0) a.cnt = 0;  // the whole window off the detector
                }
            }
            if (corner == 0 && (int)threadIdx.x / 4 < nk) s_ang[kk] = a;
        }
        __syncthreads();
        // 32 threads per angle
        for (int kk = (int)threadIdx.x / 32; kk < nk; kk += NT / 32) {
            const int cnt = s_ang[kk].cnt, j0 = s_ang[kk].j0;
            int ncol = 0;
            for (int w0 = 0; w0 < cnt; w0 += 32) {
                const int w = w0 + (int)threadIdx.x % 32, j = j0 + w;
                double2 ab = make_double2(0.0, 0.0);
                T v = T(0);
                bool col = false;
                if (w < cnt && j >= 0 && j < nb) {
                    const int64_t ri = f.sino_off + (int64_t)(k0 + kk) * nb + j;
                    const double4 e = table[ri];
                    ab = make_double2(e.x, e.y);
                    v = (T)e.z * b[ri];
                    col = e.w < 0.0;
                }
                if (w < cnt) {
                    s_ab[kk][w] = ab;
                    s_v[kk][w] = v;
                }
                // (the 32 lanes' column rays, from the wave's mask)
                const unsigned cols = (unsigned)(__ballot(col) >> (threadIdx.x & 32));
                ncol += __popc(cols);
                if (threadIdx.x % 32 == 0) s_cols[kk][w0 / 32] = cols;
            }
            if (threadIdx.x % 32 == 0) s_ncol[kk] = ncol;
        }
        __syncthreads();
        for (int kk = 0; kk < nk; ++kk) {
            // (uniform: in scalar registers)
            const FanAngle a = s_ang[kk];
            const int cnt = __builtin_amdgcn_readfirstlane(a.cnt);
            if (cnt == 0) continue;
            if (cnt > 0) {
                const int n = __builtin_amdgcn_readfirstlane(a.n), ncol = __builtin_amdgcn_readfirstlane(s_ncol[kk]);
                const int nray = __builtin_amdgcn_readfirstlane(a.nray);
                const float ac = uniform(a.c), as = uniform(a.s), agc = uniform(a.gc), ags = uniform(a.gs);
                const float aoff = uniform(a.off);
                const double2* l[PX];
                const T* v[PX];
                const float ys = Yf * ags, yc = fmaf(Yf, ac, dsof);
#pragma unroll
                for (int p = 0; p < PX; ++p) {
                    const float gt = fmaf(Xf[p], agc, ys), den = fmaf(-Xf[p], as, yc);
                    const float pos = fmaf(gt, __builtin_amdgcn_rcpf(den), aoff);
                    int i;
                    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(i) : "v"(pos));
                    // (inside the window by construction; the clamp keeps every access there)
                    i = min(max(i, 0), cnt - n);
                    l[p] = s_ab[kk] + i;
                    v[p] = s_v[kk] + i;
                }
                int nl = n;
                if (OWN && n > 2) {
                    // the lane's own half-width: its derivatives at the least depth one pixel away
                    const float den = fmaf(-Xf[0], as, yc), in1 = __builtin_amdgcn_rcpf(den - 1.f);
                    const float mv = fmaxf(fabsf(fmaf(agc, dsof, Yf * gscf)), fabsf(fmaf(ags, dsof, -Xf[0] * gscf)));
                    const float hh = uniform(a.h), hl = fminf(fmaf(mv * 1.00001f, in1 * in1, margin), hh);
                    nl = max((int)(2.f * hl) + 1, 2);
                    int i = (int)fmaf(fmaf(Xf[0], agc, ys), __builtin_amdgcn_rcpf(den), aoff + (hh - hl));
                    i = min(max(i, 0), cnt - nl);
                    l[0] = s_ab[kk] + i;
                    v[0] = s_v[kk] + i;
                }
                const int last = OWN ? nl : n;
                // candidate q of every pixel: its distance from the crossing of its row (column)
                auto cand = [&](int q, bool rows) {
#pragma unroll
                    for (int p = 0; p < PX; ++p) {
                        const double2 e = l[p][q];
                        const double own = rows ? xd[p] : yd, oth = rows ? yd : xd[p];
                        const T w = T(1) - fabs((T)(own - fma(e.y, oth, e.x)));
                        const T next = fma(w, v[p][q], acc[p]);
                        acc[p] = w > T(0) ? next : acc[p];
                    }
                };
                if (ncol == 0) {
                    cand(0, true);
                    if (n > 1) cand(1, true);
                    for (int q = 2; q < last; ++q) cand(q, true);
                } else if (ncol == nray) {
                    cand(0, false);
                    if (n > 1) cand(1, false);
                    for (int q = 2; q < last; ++q) cand(q, false);
                } else {
#pragma unroll
                    for (int p = 0; p < PX; ++p) {
                        const int i0 = (int)(v[p] - s_v[kk]);
                        for (int q = 0; q < last; ++q) {
                            const double2 e = l[p][q];
                            const bool col = (s_cols[kk][(i0 + q) >> 5] >> ((i0 + q) & 31)) & 1u;
                            const double own = col ? yd : xd[p], oth = col ? xd[p] : yd;
                            const T w = T(1) - fabs((T)(own - fma(e.y, oth, e.x)));
                            const T next = fma(w, v[p][q], acc[p]);
                            acc[p] = w > T(0) ? next : acc[p];
                        }
                    }
                }
            } else {
                const int k = k0 + kk;
                const double2 cs = trig[f.trig_off + k];
                const int64_t row = f.sino_off + (int64_t)k * nb;
                for (int p = 0; p < PX; ++p) {
                    const double X = xs[p] - hx, Y = y - hy;
                    const double p0 = fan_pos_bound(X - 1.0, Y, cs.x, cs.y, geo.dso, gsc, off);
                    const double p1 = fan_pos_bound(X + 1.0, Y, cs.x, cs.y, geo.dso, gsc, off);
                    const double p2 = fan_pos_bound(X, Y - 1.0, cs.x, cs.y, geo.dso, gsc, off);
                    const double p3 = fan_pos_bound(X, Y + 1.0, cs.x, cs.y, geo.dso, gsc, off);
                    const double lo = fmin(fmin(p0, p1), fmin(p2, p3)) - 0.05;
                    const double hi = fmax(fmax(p0, p1), fmax(p2, p3)) + 0.05;
                    const int jlo = (int)fmin(fmax(ceil(lo), 0.0), (double)nb);
                    const int jhi = (int)fmax(fmin(floor(hi), (double)(nb - 1)), -1.0);
                    for (int j = jlo; j <= jhi; ++j) {
                        const double4 e = table[row + j];
                        const bool rows = e.w > 0.0;
                        const double own = rows ? xd[p] : yd, oth = rows ? yd : xd[p];
                        const T w = T(1) - fabs((T)(own - fma(e.y, oth, e.x)));
                        if (w > T(0)) acc[p] = fma(w, (T)e.z * b[row + j], acc[p]);
                    }
                }
            }
        }
    }
#pragma unroll
    for (int p = 0; p < PX; ++p)
        if (in[p]) u[f.u_off + (int64_t)y * f.nx + xs[p]] = acc[p];
}

void fan_plan_init(Ctx& c, Plan& p) {
    p.d_fanrays.ensure(sizeof(double4) * (size_t)std::max<int64_t>(p.m, 1));
    if (p.n_rays[2] == 0) return;
    const FanGeo geo{p.fan_dso, p.fan_dsd, p.fan_du};
    hipLaunchKernelGGL(k_fan_rays, dim3((unsigned)p.n_rays[2]), dim3(256), 0, c.stream, p.d_rays[2].as<RayTile>(),
                       p.d_rinfo.as<RadonFrame>(), p.d_trig.as<double2>(), geo, p.d_fanrays.as<double4>());
    MMOF_LAUNCH_CHECK();
    MMOF_HIP(hipStreamSynchronize(c.stream));
}

// ut = the per-frame transpose of u (16-byte accesses when the stack allows them)
template <class T>
static void launch_transpose(Ctx& c, Plan& p, const T* u, T* ut) {
    if (p.tr_vec && aligned_to(16, {u, ut}))
        hipLaunchKernelGGL(k_transpose_frames4<T>, dim3((unsigned)p.n_tiles_b), dim3(256), 0, c.stream,
                           p.d_tiles_b.as<Tile>(), p.d_rinfo.as<RadonFrame>(), u, ut);
    else
        hipLaunchKernelGGL(k_transpose_frames<T>, dim3((unsigned)p.n_tiles_b), dim3(256), 0, c.stream,
                           p.d_tiles_b.as<Tile>(), p.d_rinfo.as<RadonFrame>(), u, ut);
    MMOF_LAUNCH_CHECK();
}

void launch_fan_fwd(Ctx& c, Plan& p, int dt, const void* u, void* b) {
    if (p.n_rays[2] == 0) return;
    dispatch(dt, [&](auto z) {
        using T = decltype(z);
        T* ut = static_cast<T*>(c.work("radon_transpose", sizeof(T) * p.n));
        launch_transpose<T>(c, p, (const T*)u, ut);
        ScopedTime st(&c, "fan_fwd", (double)sizeof(T) * (p.n + p.m), 0.0);
        // the fewest waves per ray that fill the chip twice (2 x 32 waves a CU), at most 4:
        // 10 frames of 28 x 36, 46 angles, 17 us with one and 4.4 with four
        const int64_t waves = 4 * p.n_rays[2], full = (int64_t)2 * c.cu_count * 32;
        const int gi = waves >= full ? 2 : 2 * waves >= full ? 1 : 0;  // angles per workgroup: 4, 2, 1
        auto k = gi == 2 ? k_fan_fwd<T, 1> : gi == 1 ? k_fan_fwd<T, 2> : k_fan_fwd<T, 4>;
        hipLaunchKernelGGL(k, dim3((unsigned)p.n_rays[gi]), dim3(256), 0, c.stream, p.d_rays[gi].as<RayTile>(),
                           p.d_rinfo.as<RadonFrame>(), p.d_fanrays.as<double4>(), (const T*)u, (const T*)ut, (T*)b);
        MMOF_LAUNCH_CHECK();
    });
}

// Margin (bins) that covers the rounding of the FP32 candidate bounds: with every point at
// most R from the centre, |t| <= R and den >= dso - R; each of t and den is off by at most a few
// FP32 ulps of dso + R, and the position g t / den + off by the propagated relative errors; a
// factor 4 on top, plus the FP64 path's 0.05.  Geometries where this exceeds 0.5 bins take the
// FP64 bounds.
static float fan_bound_margin(const Plan& p, bool& fp32) {
    const Geom& g = *p.geom;
    double R = 0.0;
    int nbmax = 1;
    for (int s = 0; s < g.n_seq; ++s) {
        R = std::max(R, 0.5 * std::hypot((double)g.nx[s], (double)g.ny[s]) + 1.5);
        nbmax = std::max(nbmax, p.n_bins[s]);
    }
    const double dmin = p.fan_dso - R, gsc = p.fan_dsd / p.fan_du, u = std::ldexp(1.0, -24);
    const double ea = 16.0 * u * (p.fan_dso + R + 2.0);  // absolute error of t and den
    const double pos = gsc * R / dmin;                   // |g t / den|
    const double err = gsc * ea / dmin + pos * (ea / dmin + 8.0 * u) + 4.0 * u * (pos + 0.5 * nbmax);
    const double m = 0.05 + 4.0 * err;
    fp32 = dmin > 0.0 && m <= 0.5;
    return (float)m;
}

void launch_fan_adj(Ctx& c, Plan& p, int dt, const void* b, void* u) {
    const FanGeo geo{p.fan_dso, p.fan_dsd, p.fan_du};
    bool fp32 = false;
    const float margin = fan_bound_margin(p, fp32);
    dispatch(dt, [&](auto z) {
        using T = decltype(z);
        ScopedTime st(&c, "fan_adj", (double)sizeof(T) * (p.n + p.m), 0.0);
        // with less than two tiles per CU a lane takes one pixel: a wave then has half the chain
        // (10 frames of 28 x 36, 46 angles: 39 us, 66 with two pixels).  On frames of up to 48 pixels (FP64: 36) the
        // half-width changes much across a tile: half a tile per workgroup and each lane's own half-width (FP32 / FP64:
        // 10 x 32 x 32, 46 angles 41 / 43 -> 32 / 32 us, 1000 x 32 x 32, 30 angles 115 / 123 -> 98 / 112, 400 x 48 x 48
        // 100 / 107 -> 100 / 118, 400 x 40 x 40 107 / 114 -> 103 / 120; 300 x 64 x 64 88 / 94 against 97 / 113)
        const bool one = p.n_tiles_a < 2 * c.cu_count;
        const bool half = std::max(p.geom->max_nx, p.geom->max_ny) <= (sizeof(T) == 4 ? 48 : 36);
        auto k = half ? k_fan_adj<T, 1, ATH / 2> : one ? k_fan_adj<T, 1, ATH> : k_fan_adj<T, 2, ATH>;
        hipLaunchKernelGGL(k, dim3((unsigned)(half ? 2 * p.n_tiles_a : p.n_tiles_a)), dim3(one && !half ? 512 : 256), 0,
                           c.stream, p.d_tiles_a.as<Tile>(),
                           p.d_rinfo.as<RadonFrame>(), p.d_trig.as<double2>(), p.d_fanrays.as<double4>(),
                           (const T*)b, (T*)u, geo, margin, (int)fp32);
        MMOF_LAUNCH_CHECK();
    });
}

const int kRadonCandidates = 4;  // angle groups of 1, 2, 4, 8 per workgroup

int radon_fwd_choice(Plan& p, int dt) {
    auto it = p.geom->tuned.find(std::string("radon_fwd") + (dt == MMOF_F32 ? "/f32" : "/f64"));
    if (it != p.geom->tuned.end()) return it->second;
    // untuned: one angle per workgroup, the best or within 2% of it from 32 x 32 to 768 x 768 (16 frames of 256 x 256,
    // 90 angles: 63 us, with 2, 4, 8 angles 66, 69, 75).  On 64 frames of 1024 x 1024 four angles depend on the
    // plan's: in order 2.64 ms against 2.70 in FP32 and 5.63 against 5.91 in FP64, in no order 2.84 against 2.70
    // and 6.05 against 5.86 (a group is placed by its first angle); the autotuner times the plan's own.
    return 0;
}

void launch_radon_fwd(Ctx& c, Plan& p, int dt, const void* u, void* b, int choice) {
    if (choice < 0) choice = radon_fwd_choice(p, dt);
    MMOF_CHECK(choice >= 0 && choice < kRadonCandidates, MMOF_ERR_INVALID, "radon_fwd candidate out of range");
    if (p.n_rays[choice] == 0) return;
    dispatch(dt, [&](auto z) {
        using T = decltype(z);
        T* ut = static_cast<T*>(c.work("radon_transpose", sizeof(T) * p.n));
        launch_transpose<T>(c, p, (const T*)u, ut);
        ScopedTime st(&c, "radon_fwd", (double)sizeof(T) * (p.n + p.m), p.radon_flops);
        auto k = choice == 0 ? k_radon_fwd<T, 1> : choice == 1 ? k_radon_fwd<T, 2> : choice == 2 ? k_radon_fwd<T, 4>
                                                                                                 : k_radon_fwd<T, 8>;
        hipLaunchKernelGGL(k, dim3((unsigned)p.n_rays[choice]), dim3(512), 0, c.stream, p.d_rays[choice].as<RayTile>(),
                           p.d_rinfo.as<RadonFrame>(), p.d_trig.as<double2>(), p.d_ray_recs.as<RayRec>(), (const T*)u,
                           (const T*)ut, (T*)b);
        MMOF_LAUNCH_CHECK();
    });
}

void launch_radon_adj(Ctx& c, Plan& p, int dt, const void* b, void* u) {
    dispatch(dt, [&](auto z) {
        using T = decltype(z);
        ScopedTime st(&c, "radon_adj", (double)sizeof(T) * (p.n + p.m), p.radon_flops);
        // Tiles of 32 rows where enough of them keep each CU busy to its end: in FP64 from 4 per CU on (16 frames of
        // 256 x 256, 45 angles 17.2 us against 20.2 with 16 rows, 12 frames the same, 8 frames 12.5 against 11.1), in
        // FP32, which gains less, from 16 (16 frames of 256 x 256, 4 per CU, 12.9 against 13.9, but 20 of 250 x 250, 5 per CU, 12.1
        // against 11.5; 32 of 512 x 512, 32 per CU, 94 against 100); and where the rows that they overhang the frames by
        // cost less than they gain (0.95 of the time per pixel in FP32, 0.81 in FP64).
        const int64_t per_cu = sizeof(T) == 4 ? 16 : 4;
        const double cost = sizeof(T) == 4 ? 0.95 : 0.81;
        const bool two = p.n_tiles_b >= per_cu * c.cu_count && 2.0 * cost * (double)p.n_tiles_b < (double)p.n_tiles_a;
        auto k = two ? k_radon_adj<T, 2> : k_radon_adj<T, 1>;
        hipLaunchKernelGGL(k, dim3((unsigned)(two ? p.n_tiles_b : p.n_tiles_a)), dim3(256), 0, c.stream,
                           (two ? p.d_tiles_b : p.d_tiles_a).as<Tile>(), p.d_rinfo.as<RadonFrame>(),
                           p.d_trig.as<double2>(), (const T*)b, (T*)u);
        MMOF_LAUNCH_CHECK();
    });
}

}  // namespace mmof

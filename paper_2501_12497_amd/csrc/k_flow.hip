// The optical-flow temporal operator L(v) of the image subproblem, in warp form:
//   direction +1:  r_t = W(v_t) u_{t+1} - u_t      (-M-bar(s), Sec. 3)
//   direction -1:  r_t = W(v_t) u_t - u_{t+1}      (-M-bar'(s'))
// W(v) pulls a bilinear (or nearest, ties to even) sample at p + v(p) with clipped
// coordinates.  The adjoint scatters through the bilinear weights; here it is a
// deterministic gather: every output pixel sums, in a fixed order (per corner of the sample
// cell, sources in raster order), the sources whose sample cell has it as a corner.
// Sources are staged in LDS per output tile and bucketed by cell, so a pixel only visits
// the sources that reach it.
#include <climits>
#include <type_traits>

#include "dev.h"
#include "kernels.h"

namespace mmof {

static constexpr int FTW = 64, FTH = 4;          // dv tiles
static constexpr int RMAX = 8;                   // LDS path of the adjoint handles radius <= RMAX

// Bilinear (INTERP 0) or nearest (INTERP 1) sample of src at (x + vx, y + vy), computed in T
// (source values of type S are rounded to T first).
template <class T, int INTERP, class S = T>
__device__ __forceinline__ T warp_sample(const S* __restrict__ src, int nx, int ny, int x, int y, T vx, T vy) {
    if (INTERP == 1) {
        const int xr = round_clip(x, vx, nx), yr = round_clip(y, vy, ny);
        return (T)src[(int64_t)yr * nx + xr];
    }
    int x0, y0;
    T fx, fy;
    bool cx, cy;
    clip_cell(x, vx, nx, x0, fx, cx);
    clip_cell(y, vy, ny, y0, fy, cy);
    const int y1 = min(y0 + 1, ny - 1);
    const S* r0 = src + (int64_t)y0 * nx;
    const S* r1 = src + (int64_t)y1 * nx;
    // the two pixels of a row as one 2-element load at xa = min(x0, nx - 2) (nx >= 2); a cell
    // clipped to the last column (x0 = nx - 1, fx = 0) takes its value from the second one
    const int xa = min(x0, nx - 2);
    const Pair<S> p0 = ld2(r0 + xa), p1 = ld2(r1 + xa);
    const bool edge = xa != x0;
    const T a0 = (T)(edge ? p0.b : p0.a), a1 = (T)p0.b, b0 = (T)(edge ? p1.b : p1.a), b1 = (T)p1.b;
    return (T(1) - fx) * (T(1) - fy) * a0 + fx * (T(1) - fy) * a1 + (T(1) - fx) * fy * b0 + fx * fy * b1;
}

// A sample position prepared once and used for many source images of the same frame
// geometry: the offsets of the two pixel pairs read (or of the nearest pixel for INTERP 1),
// the edge flag and the fractions, as warp_sample forms them.
template <class T>
struct SampleCell {
    int o0, o1;    // row * nx + xa of the rows y0 and y1 (INTERP 1: the pixel's offset in o0)
    T fx, fy;
    bool edge;
};

template <class T, int INTERP>
__device__ __forceinline__ SampleCell<T> sample_cell(int nx, int ny, int x, int y, T vx, T vy) {
    SampleCell<T> c;
    if (INTERP == 1) {
        c.o0 = round_clip(y, vy, ny) * nx + round_clip(x, vx, nx);
        c.o1 = c.o0;
        c.fx = c.fy = T(0);
        c.edge = false;
        return c;
    }
    int x0, y0;
    bool cx, cy;
    clip_cell(x, vx, nx, x0, c.fx, cx);
    clip_cell(y, vy, ny, y0, c.fy, cy);
    const int y1 = min(y0 + 1, ny - 1);
    const int xa = min(x0, nx - 2);
    c.o0 = y0 * nx + xa;
    c.o1 = y1 * nx + xa;
    c.edge = xa != x0;
    return c;
}

// warp_sample(src, ...) for a prepared cell (the same arithmetic, so the same value).
template <class T, int INTERP, class S>
__device__ __forceinline__ T sample_at(const S* __restrict__ src, const SampleCell<T>& c) {
    if (INTERP == 1) return (T)src[c.o0];
    const Pair<S> p0 = ld2(src + c.o0), p1 = ld2(src + c.o1);
    const T a0 = (T)(c.edge ? p0.b : p0.a), a1 = (T)p0.b, b0 = (T)(c.edge ? p1.b : p1.a), b1 = (T)p1.b;
    const T fx = c.fx, fy = c.fy;
    return (T(1) - fx) * (T(1) - fy) * a0 + fx * (T(1) - fy) * a1 + (T(1) - fx) * fy * b0 + fx * fy * b1;
}

template <class T, int INTERP, int FTW, int FTH>
__global__ __launch_bounds__(256) void k_flow_fwd(const Tile* __restrict__ tiles, const FrameInfo* __restrict__ fr,
                                                  const T* __restrict__ u, const T* __restrict__ v,
                                                  T* __restrict__ r, int direction) {
    const Tile tl = tiles[xcd_remap(blockIdx.x, gridDim.x)];
    const FrameInfo f = fr[tl.frame];
    const int x = tl.x0 + (int)(threadIdx.x % FTW);
    const int y = tl.y0 + (int)(threadIdx.x / FTW);
    if (x >= f.nx || y >= f.ny) return;
    const int64_t np = (int64_t)f.nx * f.ny;
    const int64_t p = (int64_t)y * f.nx + x;
    const T* ut = u + f.off;
    const T* ut1 = ut + np;
    const T* vx = v + 2 * f.pair_off;
    const T vxx = vx[p], vyy = vx[np + p];
    const T* src = direction > 0 ? ut1 : ut;
    const T* sub = direction > 0 ? ut : ut1;
    r[f.pair_off + p] = warp_sample<T, INTERP>(src, f.nx, f.ny, x, y, vxx, vyy) - sub[p];
}

// Forward and (when vr is not null) reverse flow rows of Theta for K columns at once:
// column j of U (S: FP64, or already T; leading dimension ldu) is rounded to T and mapped to
// out[j*ldo + oF + pair pixel] (forward) and out[j*ldo + oR + pair pixel] (reverse).  The
// values equal those of k_flow_fwd applied to the rounded column.
template <class T, class S, int INTERP, int FTW, int FTH>
__global__ __launch_bounds__(256) void k_flow_fwd_cols(const Tile* __restrict__ tiles,
                                                       const FrameInfo* __restrict__ fr,
                                                       const S* __restrict__ U, int64_t ldu,
                                                       const T* __restrict__ v, const T* __restrict__ vr,
                                                       T* __restrict__ out, int64_t ldo, int64_t oF, int64_t oR) {
    const Tile tl = tiles[xcd_remap(blockIdx.x, gridDim.x)];
    const FrameInfo f = fr[tl.frame];
    const int x = tl.x0 + (int)(threadIdx.x % FTW);
    const int y = tl.y0 + (int)(threadIdx.x / FTW);
    if (x >= f.nx || y >= f.ny) return;
    const int64_t np = (int64_t)f.nx * f.ny;
    const int64_t p = (int64_t)y * f.nx + x;
    const S* ut = U + (int64_t)blockIdx.y * ldu + f.off;
    const S* ut1 = ut + np;
    T* o = out + (int64_t)blockIdx.y * ldo;
    const T* vf = v + 2 * f.pair_off;
    o[oF + f.pair_off + p] = warp_sample<T, INTERP, S>(ut1, f.nx, f.ny, x, y, vf[p], vf[np + p]) - (T)ut[p];
    if (vr) {
        const T* vb = vr + 2 * f.pair_off;
        o[oR + f.pair_off + p] = warp_sample<T, INTERP, S>(ut, f.nx, f.ny, x, y, vb[p], vb[np + p]) - (T)ut1[p];
    }
}

// Vector forms of the two kernels above: each thread owns 4 consecutive pixels of one row of
// a (4*LW)-pixel-wide tile, so flows, the subtracted frame and the output move as 4-element
// vectors (16 bytes per FP32 access, from element-aligned addresses: frames of any width and
// offset); a row whose width is not a multiple of 4 ends with a thread of 1..3 pixels, whose
// accesses go element by element.  The bilinear samples stay single loads.  Values equal those
// of the scalar kernels.
template <class T, int INTERP, int LW>
__global__ __launch_bounds__(256) void k_flow_fwd4(const Tile* __restrict__ tiles, const FrameInfo* __restrict__ fr,
                                                   const T* __restrict__ u, const T* __restrict__ v,
                                                   T* __restrict__ r, int direction) {
    const Tile tl = tiles[xcd_remap(blockIdx.x, gridDim.x)];
    const FrameInfo f = fr[tl.frame];
    const int x = tl.x0 + 4 * (int)(threadIdx.x % LW);
    const int y = tl.y0 + (int)(threadIdx.x / LW);
    if (x >= f.nx || y >= f.ny) return;
    const int64_t np = (int64_t)f.nx * f.ny;
    const int64_t p = (int64_t)y * f.nx + x;
    const T* ut = u + f.off;
    const T* ut1 = ut + np;
    const int nv = min(4, f.nx - x);   // (fewer than 4 at the end of a row whose width is not a multiple of 4)
    const T* vf = v + 2 * f.pair_off;
    const Quad<T> vx = ld4n(vf + p, nv), vy = ld4n(vf + np + p, nv);
    const T* src = direction > 0 ? ut1 : ut;
    const Quad<T> sub = ld4n((direction > 0 ? ut : ut1) + p, nv);
    Quad<T> o;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        o.v[j] = warp_sample<T, INTERP>(src, f.nx, f.ny, x + j, y, vx.v[j], vy.v[j]) - sub.v[j];
    st4n(r + f.pair_off + p, o, nv);
}

// All rows of Theta u from one read of u: a thread takes a quad (4 pixels of a row, any frame width; QuadPos) of a frame
// and forms its horizontal and vertical differences and, where the frame begins a pair, the pair's forward, reverse and
// temporal-difference rows, whichever are wanted, each with its MM-weighted copy when its m is not null.  Values equal
// those of the separate kernels.  Bound by memory.  Measured against a launch per kind of row: 8 x 32 x 32, FP64,
// with both flows 5.2 us (4.0 and 5.2 us in two launches, 12.2 in three); 64 x 1024 x 1024, FP32, with temporal
// differences 333 us over the calls of a solve, 29 of 69 weighted (226 and 153, and once a weighting pass of 490).
template <class T>
struct ThetaRowsT {
    const T* __restrict__ v;
    T* __restrict__ r;
    const T* __restrict__ nu;
    T* __restrict__ m;
};

template <class T, int INTERP>
__global__ __launch_bounds__(256) void k_theta(const Tile* __restrict__ tiles, const FrameInfo* __restrict__ fr,
                                               const T* __restrict__ u, ThetaRowsT<T> gx, ThetaRowsT<T> gy,
                                               ThetaRowsT<T> fwd, ThetaRowsT<T> rev, ThetaRowsT<T> diff, double eps2) {
    const Tile tl = tiles[xcd_remap(blockIdx.x, gridDim.x)];
    const FrameInfo f = fr[tl.frame];
    const int nx = f.nx, ny = f.ny;
    const QuadPos q = quad_pos(tl, nx, ny);
    if (!q.in) return;  // (the frame's last quads: no lane reads from one past them)
    const int64_t np = (int64_t)nx * ny;
    const int64_t p = (int64_t)q.y * nx + q.x;
    const T* ut = u + f.off;
    const bool pair = f.t + 1 < f.n_t, has_y = q.y < ny - 1;
    const Quad<T> c = ld4n(ut + p, q.nv);
    Quad<T> below = zero4<T>(), next = zero4<T>();
    if (has_y) below = ld4n(ut + p + nx, q.nv);
    if (pair && (rev.r || diff.r)) next = ld4n(ut + np + p, q.nv);
    T right = __shfl_down(c.v[0], 1);
    if (q.edge_r && q.x + 4 < nx) right = ut[p + 4];
    auto put = [&](const ThetaRowsT<T>& w, int64_t o, const Quad<T>& d, int n) {
        st4n(w.r + o, d, n);
        if (w.m) {
            const Quad<T> nq = ld4n(w.nu + o, n);
            Quad<T> m;
#pragma unroll
            for (int j = 0; j < 4; ++j) m.v[j] = mm_weighted(d.v[j], nq.v[j], eps2);
            st4n(w.m + o, m, n);
        }
    };
    Quad<T> d;
    const int ngx = min(4, nx - 1 - q.x);
    if (ngx > 0) {
#pragma unroll
        for (int j = 0; j < 4; ++j) d.v[j] = (j < 3 ? c.v[j + 1] : right) - c.v[j];
        put(gx, f.gx_off + (int64_t)q.y * (nx - 1) + q.x, d, ngx);
    }
    if (has_y) {
#pragma unroll
        for (int j = 0; j < 4; ++j) d.v[j] = below.v[j] - c.v[j];
        put(gy, f.gy_off + p, d, q.nv);
    }
    if (!pair) return;
    auto warp = [&](const ThetaRowsT<T>& w, const T* src, const Quad<T>& sub) {
        const T* vf = w.v + 2 * f.pair_off;
        const Quad<T> vx = ld4n(vf + p, q.nv), vy = ld4n(vf + np + p, q.nv);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            d.v[j] = warp_sample<T, INTERP>(src, nx, ny, q.x + j, q.y, vx.v[j], vy.v[j]) - sub.v[j];
        put(w, f.pair_off + p, d, q.nv);
    };
    if (fwd.r) warp(fwd, ut + np, c);
    if (rev.r) warp(rev, ut, next);
    if (diff.r) {
#pragma unroll
        for (int j = 0; j < 4; ++j) d.v[j] = next.v[j] - c.v[j];
        put(diff, f.pair_off + p, d, q.nv);
    }
}

template <class T, class S, int INTERP, int LW>
__global__ __launch_bounds__(256) void k_flow_fwd_cols4(const Tile* __restrict__ tiles,
                                                        const FrameInfo* __restrict__ fr,
                                                        const S* __restrict__ U, int64_t ldu,
                                                        const T* __restrict__ v, const T* __restrict__ vr,
                                                        T* __restrict__ out, int64_t ldo, int64_t oF, int64_t oR) {
    const Tile tl = tiles[xcd_remap(blockIdx.x, gridDim.x)];
    const FrameInfo f = fr[tl.frame];
    const int x = tl.x0 + 4 * (int)(threadIdx.x % LW);
    const int y = tl.y0 + (int)(threadIdx.x / LW);
    if (x >= f.nx || y >= f.ny) return;
    const int64_t np = (int64_t)f.nx * f.ny;
    const int64_t p = (int64_t)y * f.nx + x;
    const S* ut = U + (int64_t)blockIdx.y * ldu + f.off;
    const S* ut1 = ut + np;
    T* o = out + (int64_t)blockIdx.y * ldo;
    const int nv = min(4, f.nx - x);
    const Quad<S> a = ld4n(ut + p, nv), b = ld4n(ut1 + p, nv);
    {
        const T* vf = v + 2 * f.pair_off;
        const Quad<T> vx = ld4n(vf + p, nv), vy = ld4n(vf + np + p, nv);
        Quad<T> q;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            q.v[j] = warp_sample<T, INTERP, S>(ut1, f.nx, f.ny, x + j, y, vx.v[j], vy.v[j]) - (T)a.v[j];
        st4n(o + oF + f.pair_off + p, q, nv);
    }
    if (vr) {
        const T* vb = vr + 2 * f.pair_off;
        const Quad<T> vx = ld4n(vb + p, nv), vy = ld4n(vb + np + p, nv);
        Quad<T> q;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            q.v[j] = warp_sample<T, INTERP, S>(ut, f.nx, f.ny, x + j, y, vx.v[j], vy.v[j]) - (T)b.v[j];
        st4n(o + oR + f.pair_off + p, q, nv);
    }
}

// k_flow_fwd_cols4 with the sample cells of a lane's four pixels (both directions) formed
// once from the flows and reused for JC consecutive columns (grid.y = column groups): the
// flows are read once per JC columns instead of once per column.
template <class T, class S, int INTERP, int LW, int JC>
__global__ __launch_bounds__(256) void k_flow_fwd_colsJ(const Tile* __restrict__ tiles,
                                                        const FrameInfo* __restrict__ fr,
                                                        const S* __restrict__ U, int64_t ldu, int K,
                                                        const T* __restrict__ v, const T* __restrict__ vr,
                                                        T* __restrict__ out, int64_t ldo, int64_t oF, int64_t oR) {
    const Tile tl = tiles[xcd_remap(blockIdx.x, gridDim.x)];
    const FrameInfo f = fr[tl.frame];
    const int x = tl.x0 + 4 * (int)(threadIdx.x % LW);
    const int y = tl.y0 + (int)(threadIdx.x / LW);
    if (x >= f.nx || y >= f.ny) return;
    const int64_t np = (int64_t)f.nx * f.ny;
    const int64_t p = (int64_t)y * f.nx + x;
    const int nv = min(4, f.nx - x);
    SampleCell<T> cf[4], cr[4];
    {
        const T* vf = v + 2 * f.pair_off;
        const Quad<T> vx = ld4n(vf + p, nv), vy = ld4n(vf + np + p, nv);
#pragma unroll
        for (int j = 0; j < 4; ++j) cf[j] = sample_cell<T, INTERP>(f.nx, f.ny, x + j, y, vx.v[j], vy.v[j]);
    }
    if (vr) {
        const T* vb = vr + 2 * f.pair_off;
        const Quad<T> vx = ld4n(vb + p, nv), vy = ld4n(vb + np + p, nv);
#pragma unroll
        for (int j = 0; j < 4; ++j) cr[j] = sample_cell<T, INTERP>(f.nx, f.ny, x + j, y, vx.v[j], vy.v[j]);
    }
    const int c0 = blockIdx.y * JC;
    for (int jj = 0; jj < JC; ++jj) {
        const int col = c0 + jj;
        if (col >= K) break;
        const S* ut = U + (int64_t)col * ldu + f.off;
        const S* ut1 = ut + np;
        T* o = out + (int64_t)col * ldo;
        const Quad<S> a = ld4n(ut + p, nv), b = ld4n(ut1 + p, nv);
        Quad<T> q;
#pragma unroll
        for (int j = 0; j < 4; ++j) q.v[j] = sample_at<T, INTERP, S>(ut1, cf[j]) - (T)a.v[j];
        st4n(o + oF + f.pair_off + p, q, nv);
        if (vr) {
#pragma unroll
            for (int j = 0; j < 4; ++j) q.v[j] = sample_at<T, INTERP, S>(ut, cr[j]) - (T)b.v[j];
            st4n(o + oR + f.pair_off + p, q, nv);
        }
    }
}

// Cell of a source pixel: clipped floor coordinates and fractions (0 for INTERP 1).
template <class T, int INTERP>
__device__ __forceinline__ void source_cell(int sx, int sy, T vx, T vy, int nx, int ny, int& x0, int& y0, T& fx,
                                            T& fy) {
    if (INTERP == 1) {
        x0 = round_clip(sx, vx, nx);
        y0 = round_clip(sy, vy, ny);
        fx = T(0);
        fy = T(0);
    } else {
        bool c;
        clip_cell(sx, vx, nx, x0, fx, c);
        clip_cell(sy, vy, ny, y0, fy, c);
    }
}

// Cell of a source pixel that no clip can reach (an interior tile: |v| < radius).
template <class T, int INTERP>
__device__ __forceinline__ void source_cell_inner(int sx, int sy, T vx, T vy, int& x0, int& y0, T& fx, T& fy) {
    if (INTERP == 1) {
        x0 = rint_shift(sx, vx);
        y0 = rint_shift(sy, vy);
        fx = T(0);
        fy = T(0);
    } else {
        const T gx = floor(vx), gy = floor(vy);
        x0 = sx + (int)gx;
        y0 = sy + (int)gy;
        fx = vx - gx;
        fy = vy - gy;
    }
}

// The weighted values a source hands to the four corners of its cell, in the order (1,1), (0,1), (1,0), (0,0) of the
// corner's offset from the cell's origin.
template <class T>
__device__ __forceinline__ void corner_terms(T fx, T fy, T val, T t[4]) {
    const T gx = T(1) - fx, gy = T(1) - fy;
    t[0] = fx * fy * val;
    t[1] = gx * fy * val;
    t[2] = fx * gy * val;
    t[3] = gx * gy * val;
}

// Adjoint over an ATX x ATY output tile per workgroup of 256 threads.  The sources within the radius of the tile are
// loaded together; each adds its four weighted values into the four corner sums of its cell in LDS, and an output adds
// the sums of the four cells it is a corner of in a fixed order.  A cell sum of one or two sources does not depend on
// their order.  A cell with more (a converging flow) takes its sources again from a list in LDS and sums them in raster
// order, so no value depends on the tile shape or on the order of arrival (each source finds its place in its cell's
// run by counting the ranks below its own: 16 x 128 x 128, FP32, a flow that leaves the frame by up to 7.5 px and clips
// 64 sources into a corner cell 14 us, 121 when one thread per cell picked them in order); a tile whose crowded cells
// hold more than ADJ_LIST sources forms the same sums by the wide-window path.
// Bound by the vector instructions of the sources (184 per output and lane, VALU 90% busy; 269 when every output formed
// the weights of its four cells' sources itself): 576 sources at radius 4 for the 256 outputs of a 16 x 16 tile.
// Interior tiles skip the clip.  Measured over 31 pairs of 512 x 512 with the radius, before and now: smooth flow 105 ->
// 68 us (FP32), 145 -> 99 (FP64); a flow of unit noise, whose cells are often crowded, 699 -> 135 and 991 -> 198.
constexpr int ADJ_LIST = 384;

template <class T, int INTERP, int ATX, int ATY>
__global__ __launch_bounds__(256) void k_flow_adj(const AdjTile* __restrict__ tiles, const T* __restrict__ r,
                                                  const T* __restrict__ v, T* __restrict__ u, int direction,
                                                  int accumulate, const int32_t* __restrict__ d_radius,
                                                  const T* __restrict__ cx, const double* __restrict__ clam,
                                                  double* __restrict__ cout) {
    constexpr int RPT = ATX * ATY / 256;
    constexpr int SMAX = (ATX + 2 * RMAX) * (ATY + 2 * RMAX);  // source window (raster rank < 2^16)
    constexpr int NI = (SMAX + 255) / 256;
    constexpr int CW = ATX + 1, NC = (ATX + 1) * (ATY + 1);     // cells touching the tile
    constexpr int CROWDED = 1 << 30;  // s_cnt of a cell with a list: this flag, below it the next free entry
    static_assert(SMAX <= 65536, "source ranks are kept in 16 bits");
    // FP64 adds into the corner sums of a cell by LDS atomics; FP32, whose LDS add is several times slower than its
    // store (32 x 512 x 512: 200 us against 51), stores a cell's first and second source apart
    constexpr int NS = sizeof(T) == 4 ? 2 : 1;
    __shared__ T s_sum[NS][4][NC];
    __shared__ int s_cnt[NC];
    __shared__ T s_term[4][ADJ_LIST];
    __shared__ unsigned short s_rank[ADJ_LIST];
    __shared__ int s_over, s_top;

    const AdjTile tl = tiles[xcd_remap(blockIdx.x, gridDim.x)];
    const int R = *d_radius;  // (independent of the tile: both loads are in flight together)
    const int nx = tl.nx, ny = tl.ny;
    const int64_t np = (int64_t)nx * ny;
    const int lx = (int)(threadIdx.x % ATX), ly0 = (int)(threadIdx.x / ATX) * RPT;
    const int qx = tl.x0 + lx;
    const int qy0 = tl.y0 + ly0;
    const bool col_in = qx < nx;

    // direct terms and the pair whose warp gathers into this frame
    const int64_t dp = direction > 0 ? tl.po : tl.pp;  // pair offset of the direct term (-1: none)
    const int64_t gp = direction > 0 ? tl.pp : tl.po;  // pair offset of the gathering pair (-1: none)
    T acc[RPT], direct[RPT], old[RPT];
    // the direct terms and old outputs are loaded first, with the sources (their latency
    // then overlaps the staging instead of following it)
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        acc[k] = direct[k] = old[k] = T(0);
        const int qy = qy0 + k;
        if (col_in && qy < ny) {
            const int64_t q = (int64_t)qy * nx + qx;
            if (dp >= 0) direct[k] = -r[dp + q];
            if (accumulate) old[k] = u[tl.off + q];
        }
    }

    if (gp >= 0) {
        const T* rg = r + gp;
        const T* vxg = v + 2 * gp;
        const T* vyg = vxg + np;
        // (the window is addressed by 32-bit byte offsets: its rows have at most 2^23 pixels)
        bool wide = R > RMAX || nx > (1 << 23);
        if (!wide) {
            const int sx0 = max(tl.x0 - R, 0), sx1 = min(tl.x0 + ATX - 1 + R, nx - 1);
            const int sy0 = max(tl.y0 - R, 0), sy1 = min(tl.y0 + ATY - 1 + R, ny - 1);
            const int sw = sx1 - sx0 + 1, sh = sy1 - sy0 + 1;
            const bool inner = tl.x0 - 2 * R >= 0 && tl.x0 + ATX + 2 * R < nx && tl.y0 - 2 * R >= 0 &&
                               tl.y0 + ATY + 2 * R < ny;
            for (int i = threadIdx.x; i < NC; i += 256) {
                s_cnt[i] = 0;
#pragma unroll
                for (int q = 0; q < 4 * NS; ++q) s_sum[q >> 2][q & 3][i] = T(0);
            }
            if (threadIdx.x == 0) s_over = s_top = 0;
            // A thread first loads all of its sources (independent loads, in flight together), then forms their cells.
            // Source i of the window (its raster index, pitch sw, which is also its rank) is taken by thread i mod 256;
            // the row is i / sw from an FP32 product (exact: i < 2^16 and the quotient's fraction is at least 1/(2 sw)
            // away from an integer).
            const int nsrc = sw * sh;
            const float inv_sw = 1.0f / (float)sw;
            const int64_t pw = (int64_t)sy0 * nx + sx0;
            const char* bx = reinterpret_cast<const char*>(vxg + pw);
            const char* by = reinterpret_cast<const char*>(vyg + pw);
            const char* br = reinterpret_cast<const char*>(rg + pw);
            T lvx[NI], lvy[NI], lr[NI];
#pragma unroll
            for (int k = 0; k < NI; ++k) {
                const int i = (int)threadIdx.x + 256 * k;
                lvx[k] = lvy[k] = lr[k] = T(0);
                if (i < nsrc) {
                    const int ly = (int)(((float)i + 0.5f) * inv_sw);
                    const unsigned o = (unsigned)(ly * (nx - sw) + i) * (unsigned)sizeof(T);
                    lvx[k] = *reinterpret_cast<const T*>(bx + o);
                    lvy[k] = *reinterpret_cast<const T*>(by + o);
                    lr[k] = *reinterpret_cast<const T*>(br + o);
                }
            }
            __syncthreads();  // slots cleared
            // the cell of every source (-1: it touches no output), its fractions in place of the flow, and its turn there
            int cell[NI], slot[NI];
            auto cells = [&](auto in_tag) {
#pragma unroll
                for (int k = 0; k < NI; ++k) {
                    const int i = (int)threadIdx.x + 256 * k;
                    cell[k] = -1;
                    slot[k] = 0;
                    if (i < nsrc) {
                        const int ly = (int)(((float)i + 0.5f) * inv_sw), wx = i - ly * sw;
                        int x0, y0;
                        T fx, fy;
                        if (decltype(in_tag)::value)
                            source_cell_inner<T, INTERP>(sx0 + wx, sy0 + ly, lvx[k], lvy[k], x0, y0, fx, fy);
                        else
                            source_cell<T, INTERP>(sx0 + wx, sy0 + ly, lvx[k], lvy[k], nx, ny, x0, y0, fx, fy);
                        lvx[k] = fx;
                        lvy[k] = fy;
                        const int cx = x0 - tl.x0 + 1, cy = y0 - tl.y0 + 1;
                        if ((unsigned)cx <= (unsigned)ATX && (unsigned)cy <= (unsigned)ATY) {
                            cell[k] = cy * CW + cx;
                            slot[k] = atomicAdd(&s_cnt[cell[k]], 1);
                        }
                    }
                }
            };
            if (inner)
                cells(std::true_type{});
            else
                cells(std::false_type{});
            int most = 0;
#pragma unroll
            for (int k = 0; k < NI; ++k)
                if (cell[k] >= 0) {
                    T t[4];
                    corner_terms(lvx[k], lvy[k], lr[k], t);
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        if (NS == 2)
                            s_sum[slot[k] & (NS - 1)][q][cell[k]] = t[q];
                        else
                            unsafeAtomicAdd(&s_sum[0][q][cell[k]], t[q]);
                    }
                    most = max(most, slot[k]);
                }
            if (most > 1) s_over = 1;
            __syncthreads();
            if (s_over) {
                // crowded cells: a run of list entries per cell (its count is kept in its first sum meanwhile)
                for (int i = threadIdx.x; i < NC; i += 256) {
                    const int n = s_cnt[i];
                    if (n > 2) {
                        s_cnt[i] = CROWDED | atomicAdd(&s_top, n);
                        s_sum[0][0][i] = (T)n;
                    }
                }
                __syncthreads();
                wide = s_top > ADJ_LIST;  // (the same value on every thread)
                if (!wide) {
#pragma unroll
                    for (int k = 0; k < NI; ++k)
                        if (cell[k] >= 0 && (s_cnt[cell[k]] & CROWDED)) {
                            const int e = atomicAdd(&s_cnt[cell[k]], 1) & (CROWDED - 1);
                            s_rank[e] = (unsigned short)(threadIdx.x + 256 * k);
                        }
                    __syncthreads();
                    // each source goes to its place by rank in its cell's run, found by the ranks below its own
#pragma unroll
                    for (int k = 0; k < NI; ++k)
                        if (cell[k] >= 0 && (s_cnt[cell[k]] & CROWDED)) {
                            const int e1 = s_cnt[cell[k]] & (CROWDED - 1), e0 = e1 - (int)s_sum[0][0][cell[k]];
                            int at = e0;
#pragma unroll 8
                            for (int e = e0; e < e1; ++e) at += s_rank[e] < threadIdx.x + 256 * k ? 1 : 0;
                            T t[4];
                            corner_terms(lvx[k], lvy[k], lr[k], t);
#pragma unroll
                            for (int q = 0; q < 4; ++q) s_term[q][at] = t[q];
                        }
                    __syncthreads();
                    for (int i = threadIdx.x; i < NC; i += 256) {
                        if (!(s_cnt[i] & CROWDED)) continue;
                        const int e1 = s_cnt[i] & (CROWDED - 1), e0 = e1 - (int)s_sum[0][0][i];
                        T a[4] = {T(0), T(0), T(0), T(0)};
#pragma unroll 4
                        for (int e = e0; e < e1; ++e)
#pragma unroll
                            for (int q = 0; q < 4; ++q) a[q] += s_term[q][e];
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            s_sum[0][q][i] = a[q];
                            if (NS == 2) s_sum[NS - 1][q][i] = T(0);
                        }
                    }
                    __syncthreads();
                }
            }
            if (!wide) {
                // the output is corner (1,1), (0,1), (1,0), (0,0) of the cells at (qx-1, qy-1), (qx, qy-1), (qx-1, qy),
                // (qx, qy)
#pragma unroll
                for (int k = 0; k < RPT; ++k) {
                    const int c00 = (ly0 + k) * CW + lx;
                    auto part = [&](int q, int cell) { return NS == 2 ? s_sum[0][q][cell] + s_sum[NS - 1][q][cell] : s_sum[0][q][cell]; };
                    acc[k] = ((part(0, c00) + part(1, c00 + 1)) + part(2, c00 + CW)) + part(3, c00 + CW + 1);
                }
            }
        }
        if (wide && col_in) {
            // Large displacements or crowded cells: scan the full window in global memory,
            // with the per-corner partial sums and their combination of the LDS path (same
            // values).
            const int Rw = max(R, 1);
#pragma unroll
            for (int k = 0; k < RPT; ++k) {
                const int qy = qy0 + k;
                if (qy >= ny) break;
                const int py_lo = max(qy - Rw, 0), py_hi = min(qy + Rw, ny - 1);
                const int px_lo = max(qx - Rw, 0), px_hi = min(qx + Rw, nx - 1);
                T part[4] = {T(0), T(0), T(0), T(0)};
                for (int py = py_lo; py <= py_hi; ++py)
                    for (int px = px_lo; px <= px_hi; ++px) {
                        const int64_t p = (int64_t)py * nx + px;
                        int x0, y0;
                        T fx, fy;
                        source_cell<T, INTERP>(px, py, vxg[p], vyg[p], nx, ny, x0, y0, fx, fy);
                        const int ex = qx - x0, ey = qy - y0;  // 1: the output is the cell's far corner
                        if ((unsigned)ex > 1u || (unsigned)ey > 1u) continue;
                        T t[4];
                        corner_terms(fx, fy, rg[p], t);
                        const int cr = (1 - ex) + 2 * (1 - ey);
                        {
#pragma clang fp contract(off)  // (the product is rounded before the sum, as in the LDS path)
                            if (cr == 0) part[0] += t[0];
                            else if (cr == 1) part[1] += t[1];
                            else if (cr == 2) part[2] += t[2];
                            else part[3] += t[3];
                        }
                    }
                acc[k] = ((part[0] + part[1]) + part[2]) + part[3];
            }
        }
    }
    if (!col_in) return;
    // cout (may be null): instead of u, the residual cout = cx + lambda u (ResidualOut)
    const double lam = cout ? clam[0] : 0.0;
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        const int qy = qy0 + k;
        if (qy >= ny) break;
        const T val = acc[k] + direct[k];
        const T out = accumulate ? old[k] + val : val;
        const int64_t o = tl.off + (int64_t)qy * nx + qx;
        if (cout)
            cout[o] = (double)cx[o] + lam * (double)out;
        else
            u[o] = out;
    }
}

template <class T>
__global__ __launch_bounds__(256) void k_flow_dv(const Tile* __restrict__ tiles, const FrameInfo* __restrict__ fr,
                                                 const T* __restrict__ u, const T* __restrict__ v,
                                                 const T* __restrict__ w, T* __restrict__ gv, int direction) {
    const Tile tl = tiles[xcd_remap(blockIdx.x, gridDim.x)];
    const FrameInfo f = fr[tl.frame];
    const int x = tl.x0 + (int)(threadIdx.x % FTW);
    const int y = tl.y0 + (int)(threadIdx.x / FTW);
    if (x >= f.nx || y >= f.ny) return;
    const int nx = f.nx, ny = f.ny;
    const int64_t np = (int64_t)nx * ny;
    const int64_t p = (int64_t)y * nx + x;
    const T* src = u + f.off + (direction > 0 ? np : 0);
    const T* vv = v + 2 * f.pair_off;
    int x0, y0;
    T fx, fy;
    bool cx, cy;
    clip_cell(x, vv[p], nx, x0, fx, cx);
    clip_cell(y, vv[np + p], ny, y0, fy, cy);
    const int y1 = min(y0 + 1, ny - 1);
    // row pairs as in warp_sample (a cell clipped to the last column reads the second element)
    const int xa = min(x0, nx - 2);
    const Pair<T> p0 = ld2(src + (int64_t)y0 * nx + xa), p1 = ld2(src + (int64_t)y1 * nx + xa);
    const bool edge = xa != x0;
    const T s00 = edge ? p0.b : p0.a, s01 = p0.b, s10 = edge ? p1.b : p1.a, s11 = p1.b;
    const T ww = w[f.pair_off + p];
    T dx = (T(1) - fy) * (s01 - s00) + fy * (s11 - s10);
    T dy = (T(1) - fx) * (s10 - s00) + fx * (s11 - s01);
    if (cx) dx = T(0);
    if (cy) dy = T(0);
    gv[2 * f.pair_off + p] = ww * dx;
    gv[2 * f.pair_off + np + p] = ww * dy;
}

// out[blockIdx] = floor(max |v|) + 1 over the workgroup's share of the n values of the flows (a NaN counts as 1e30): the
// radius of the adjoint's source windows, whole for one workgroup (then also into out2, when not null).
template <class T, int VEC>
__global__ __launch_bounds__(1024) void k_flow_radius(const T* __restrict__ v, int64_t n, int32_t* __restrict__ out,
                                                      int32_t* __restrict__ out2) {
    // VEC values per load (16 bytes when the flow is 16-byte aligned), four loads in flight per
    // step; the last n % VEC values singly
    typedef T VT __attribute__((ext_vector_type(VEC), aligned(sizeof(T) * VEC)));
    __shared__ T s_m[16];
    T m = T(0);
    auto take = [&](T x) {
        x = fabs(x);
        m = (x != x) ? T(1e30) : fmax(m, x);
    };
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t nv = n / VEC;
    const VT* vv = reinterpret_cast<const VT*>(v);
    for (int64_t i0 = tid; i0 < nv; i0 += 4 * stride) {
        VT a[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) a[u] = i0 + u * stride < nv ? vv[i0 + u * stride] : VT{};
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int e = 0; e < VEC; ++e) take(a[u][e]);
    }
    for (int64_t i = nv * VEC + tid; i < n; i += stride) take(v[i]);
    for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o));
    if ((threadIdx.x & 63) == 0) s_m[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < (int)blockDim.x / 64; ++w) m = fmax(m, s_m[w]);
        const int32_t r = (int32_t)fmin(floor(m), T(1 << 20)) + 1;
        out[blockIdx.x] = r;
        if (out2) *out2 = r;
    }
}

// out (and out2, when not null) = the largest of the n values (one wave)
__global__ __launch_bounds__(64) void k_max_int(const int32_t* __restrict__ p, int n, int32_t* __restrict__ out,
                                                int32_t* __restrict__ out2) {
    int m = 1;
    for (int i = (int)threadIdx.x; i < n; i += 64) m = max(m, p[i]);
    for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o));
    if (threadIdx.x == 0) {
        *out = m;
        if (out2) *out2 = m;
    }
}

void launch_flow_radius(Ctx& c, Geom& g, int dt, const void* v, int32_t* d_out, int32_t* d_out2) {
    const int64_t n = 2 * g.pair_px;
    if (n == 0) {
        hipLaunchKernelGGL(k_max_int, dim3(1), dim3(64), 0, c.stream, (const int32_t*)nullptr, 0, d_out, d_out2);
        MMOF_LAUNCH_CHECK();
        return;
    }
    dispatch(dt, [&](auto z) {
        using T = decltype(z);
        // Up to 32768 values: one workgroup, one launch.  More: a workgroup per 32768 values, two per CU at most, whose
        // maxima a second launch joins.  One integer atomic per workgroup took 15 ns each, one after the other:
        // 30 us over the flows of 31 pairs of 512 x 512 (2048 workgroups).
        constexpr int VEC = 16 / (int)sizeof(T);
        const int nb = (int)std::min<int64_t>(cdiv(n, 32768), 2 * c.cu_count);
        int32_t* part = nb > 1 ? static_cast<int32_t*>(c.work("radius_part", sizeof(int32_t) * 2 * c.cu_count)) : d_out;
        auto k = reinterpret_cast<uintptr_t>(v) % 16 == 0 ? k_flow_radius<T, VEC> : k_flow_radius<T, 1>;
        hipLaunchKernelGGL(k, dim3(nb), dim3(1024), 0, c.stream, (const T*)v, n, part,
                           nb > 1 ? nullptr : d_out2);
        MMOF_LAUNCH_CHECK();
        if (nb > 1) {
            hipLaunchKernelGGL(k_max_int, dim3(1), dim3(64), 0, c.stream, part, nb, d_out, d_out2);
            MMOF_LAUNCH_CHECK();
        }
    });
}

const TileShape kFlowShapes[] = {{64, 4, 0}, {32, 8, 0}, {128, 2, 0}, {16, 16, 0}};
const int kFlowCandidates = sizeof(kFlowShapes) / sizeof(kFlowShapes[0]);
const TileShape kFlowAdjShapes[] = {{16, 16, 0}, {32, 16, 0}, {64, 16, 0}, {32, 32, 0}};
const int kFlowAdjCandidates = sizeof(kFlowAdjShapes) / sizeof(kFlowAdjShapes[0]);
// vector-form candidates of the forward operator: lanes per tile row (4 pixels each) and
// waves per workgroup
struct Flow4Shape {
    int lw, nw;
    int tw() const { return 4 * lw; }
    int th() const { return 64 * nw / lw; }
};
static const Flow4Shape kFlow4Shapes[] = {{64, 4}, {32, 4}, {64, 2}, {32, 2}};
static_assert(sizeof(kFlow4Shapes) / sizeof(kFlow4Shapes[0]) == sizeof(kFlowShapes) / sizeof(kFlowShapes[0]),
              "both forms offer the same number of tile candidates");

TileShape flow_tile(const Geom& g, int choice) {
    (void)g;   // (the forward runs in its 4-pixel form for every frame width)
    return TileShape{kFlow4Shapes[choice].tw(), kFlow4Shapes[choice].th(), 0};
}

template <class T, int INTERP>
static auto flow_fwd_kernel(int choice) {
    return choice == 0 ? k_flow_fwd<T, INTERP, 64, 4>
           : choice == 1 ? k_flow_fwd<T, INTERP, 32, 8>
           : choice == 2 ? k_flow_fwd<T, INTERP, 128, 2>
                         : k_flow_fwd<T, INTERP, 16, 16>;
}
template <class T, int INTERP>
static auto flow_fwd4_kernel(int choice) {
    return kFlow4Shapes[choice].lw == 64 ? k_flow_fwd4<T, INTERP, 64> : k_flow_fwd4<T, INTERP, 32>;
}
template <class T, int INTERP>
static auto flow_adj_kernel(int choice) {
    return choice == 0 ? k_flow_adj<T, INTERP, 16, 16>
           : choice == 1 ? k_flow_adj<T, INTERP, 32, 16>
           : choice == 2 ? k_flow_adj<T, INTERP, 64, 16>
                         : k_flow_adj<T, INTERP, 32, 32>;
}

void launch_theta(Ctx& c, Geom& g, int dt, int interp, const void* u, const ThetaRows& gx, const ThetaRows& gy,
                  const ThetaRows& fwd, const ThetaRows& rev, const ThetaRows& diff, double eps2) {
    dispatch(dt, [&](auto z) {
        using T = decltype(z);
        // u read, the rows written, a flow read per flow row; nu read and the weighted rows written.  The launch is
        // timed under the name of each kind of row, with that kind's work, and under its own with all of it.
        const double per = gx.m ? 3.0 : 1.0, flows = (fwd.r ? 1.0 : 0.0) + (rev.r ? 1.0 : 0.0);
        const double ng = (double)(g.gx_len + g.gy_len), np = (double)g.pair_px, td = diff.r ? 1.0 : 0.0, es = sizeof(T);
        ScopedTime t0(&c, "theta", es * ((double)g.n + per * ng + (flows * (per + 2.0) + td * per) * np),
                      ng + (12.0 * flows + td) * np);
        ScopedTime t1(&c, "grad_fwd", es * ((double)g.n + per * ng), ng);
        ScopedTime t2(flows > 0.0 ? &c : nullptr, "flow_fwd", es * flows * (per + 4.0) * np, 12.0 * flows * np);
        ScopedTime t3(diff.r ? &c : nullptr, "tdiff_fwd", es * (per + 2.0) * np, np);
        auto typed = [](const ThetaRows& w) {
            return ThetaRowsT<T>{(const T*)w.v, (T*)w.r, (const T*)w.nu, (T*)w.m};
        };
        // a wave per workgroup while that leaves CUs free (8 x 32 x 32: 32 workgroups, where 256 threads make 8)
        const int per_wg = g.n / 4 < (int64_t)256 * 4 * c.cu_count ? 64 : 256;
        const TileList& tl = g.quad_list(c.stream, per_wg);
        auto k = interp == MMOF_INTERP_ROUND ? k_theta<T, 1> : k_theta<T, 0>;
        hipLaunchKernelGGL(k, dim3((unsigned)tl.count), dim3(per_wg), 0, c.stream, tl.buf.as<Tile>(), g.dframes(),
                           (const T*)u, typed(gx), typed(gy), typed(fwd), typed(rev), typed(diff), eps2);
        MMOF_LAUNCH_CHECK();
    });
}

void launch_flow_fwd(Ctx& c, Geom& g, int dt, int direction, int interp, const void* u, const void* v, void* r,
                     int choice) {
    if (g.n_pairs == 0) return;
    if (choice < 0) choice = g.choice("flow_fwd", dt, 1);
    MMOF_CHECK(choice >= 0 && choice < kFlowCandidates, MMOF_ERR_INVALID, "flow tile candidate out of range");
    dispatch(dt, [&](auto z) {
        using T = decltype(z);
        ScopedTime st(&c, "flow_fwd", 5.0 * sizeof(T) * g.pair_px, 12.0 * g.pair_px);
        if (aligned_to(sizeof(T), {u, v, r})) {
            const Flow4Shape sh = kFlow4Shapes[choice];
            const TileList& tl = g.tile_list(c.stream, sh.tw(), sh.th(), true);
            auto k = interp == MMOF_INTERP_ROUND ? flow_fwd4_kernel<T, 1>(choice) : flow_fwd4_kernel<T, 0>(choice);
            hipLaunchKernelGGL(k, dim3((unsigned)tl.count), dim3(64 * sh.nw), 0, c.stream, tl.buf.as<Tile>(),
                               g.dframes(), (const T*)u, (const T*)v, (T*)r, direction);
        } else {
            const TileShape sh = kFlowShapes[choice];
            const TileList& tl = g.tile_list(c.stream, sh.tw, sh.th, true);
            auto k = interp == MMOF_INTERP_ROUND ? flow_fwd_kernel<T, 1>(choice) : flow_fwd_kernel<T, 0>(choice);
            hipLaunchKernelGGL(k, dim3((unsigned)tl.count), dim3(256), 0, c.stream, tl.buf.as<Tile>(), g.dframes(),
                               (const T*)u, (const T*)v, (T*)r, direction);
        }
        MMOF_LAUNCH_CHECK();
    });
}

void launch_flow_fwd_cols(Ctx& c, Geom& g, int dt, int interp, const void* Uv, bool u_op, int64_t ldu, int K,
                          const void* v, const void* vr, void* out, int64_t ldo, int64_t oF, int64_t oR) {
    if (g.n_pairs == 0 || K <= 0) return;
    const int choice = g.choice("flow_fwd", dt, 1);
    dispatch(dt, [&](auto z) {
        using T = decltype(z);
        auto run = [&](auto s_tag) {
            using S = decltype(s_tag);
            const S* U = static_cast<const S*>(Uv);
            ScopedTime st(&c, "flow_fwd_cols", (vr ? 2.0 : 1.0) * K * (4.0 * sizeof(T) + 2.0 * sizeof(S)) * g.pair_px,
                          (vr ? 2.0 : 1.0) * K * 12.0 * g.pair_px);
            const bool v4 = aligned_to(sizeof(S), {U}) && aligned_to(sizeof(T), {v, vr, out});
            if (v4) {
                const Flow4Shape sh = kFlow4Shapes[choice];
                const TileList& tl = g.tile_list(c.stream, sh.tw(), sh.th(), true);
                if ((int64_t)g.max_ny * g.max_nx < ((int64_t)1 << 31)) {
                    // (prepared cells hold 32-bit offsets within a frame)
                    // columns per thread: 8, or 2 while that leaves fewer than two workgroups per CU (a thread
                    // walks its columns one after the other: 7 pairs of 32 x 32, 30 FP64 columns 15 us with 8,
                    // 6.9 with 2)
                    const int JC = (int64_t)tl.count * cdiv(K, 8) < 2 * c.cu_count ? 2 : 8;
                    auto pick = [&](auto interp_tag) {
                        constexpr int I = decltype(interp_tag)::value;
                        return JC == 2 ? (sh.lw == 64 ? k_flow_fwd_colsJ<T, S, I, 64, 2> : k_flow_fwd_colsJ<T, S, I, 32, 2>)
                                       : (sh.lw == 64 ? k_flow_fwd_colsJ<T, S, I, 64, 8> : k_flow_fwd_colsJ<T, S, I, 32, 8>);
                    };
                    auto k = interp == MMOF_INTERP_ROUND ? pick(std::integral_constant<int, 1>{})
                                                         : pick(std::integral_constant<int, 0>{});
                    hipLaunchKernelGGL(k, dim3((unsigned)tl.count, (unsigned)cdiv(K, JC)), dim3(64 * sh.nw), 0,
                                       c.stream, tl.buf.as<Tile>(), g.dframes(), U, ldu, K, (const T*)v, (const T*)vr,
                                       (T*)out, ldo, oF, oR);
                } else {
                    auto pick = [&](auto interp_tag) {
                        constexpr int I = decltype(interp_tag)::value;
                        return sh.lw == 64 ? k_flow_fwd_cols4<T, S, I, 64> : k_flow_fwd_cols4<T, S, I, 32>;
                    };
                    auto k = interp == MMOF_INTERP_ROUND ? pick(std::integral_constant<int, 1>{})
                                                         : pick(std::integral_constant<int, 0>{});
                    hipLaunchKernelGGL(k, dim3((unsigned)tl.count, (unsigned)K), dim3(64 * sh.nw), 0, c.stream,
                                       tl.buf.as<Tile>(), g.dframes(), U, ldu, (const T*)v, (const T*)vr, (T*)out,
                                       ldo, oF, oR);
                }
            } else {
                const TileShape sh = kFlowShapes[choice];
                const TileList& tl = g.tile_list(c.stream, sh.tw, sh.th, true);
                auto pick = [&](auto interp_tag) {
                    constexpr int I = decltype(interp_tag)::value;
                    return choice == 0 ? k_flow_fwd_cols<T, S, I, 64, 4>
                           : choice == 1 ? k_flow_fwd_cols<T, S, I, 32, 8>
                           : choice == 2 ? k_flow_fwd_cols<T, S, I, 128, 2>
                                         : k_flow_fwd_cols<T, S, I, 16, 16>;
                };
                auto k = interp == MMOF_INTERP_ROUND ? pick(std::integral_constant<int, 1>{})
                                                     : pick(std::integral_constant<int, 0>{});
                hipLaunchKernelGGL(k, dim3((unsigned)tl.count, (unsigned)K), dim3(256), 0, c.stream,
                                   tl.buf.as<Tile>(), g.dframes(), U, ldu, (const T*)v, (const T*)vr, (T*)out, ldo,
                                   oF, oR);
            }
            MMOF_LAUNCH_CHECK();
        };
        if (u_op)
            run(T{});
        else
            run(double{});
    });
}

void launch_flow_adj(Ctx& c, Geom& g, int dt, int direction, int interp, const void* r, const void* v, void* u,
                     bool accumulate, const int32_t* d_radius, int choice, const ResidualOut* res) {
    int32_t* rad = const_cast<int32_t*>(d_radius);
    if (!rad) {
        rad = static_cast<int32_t*>(c.work("flow_radius", 256));
        launch_flow_radius(c, g, dt, v, rad);
    }
    // untuned: 16 x 16 for every frame, the fastest or within 3% of it (8 x 32 x 32: 13 us against 15 to 19 for the larger
    // tiles, 12 x 1024 x 1024: 93 against 93 to 113)
    if (choice < 0) choice = g.choice("flow_adj", dt, 0);
    MMOF_CHECK(choice >= 0 && choice < kFlowAdjCandidates, MMOF_ERR_INVALID, "flow adjoint tile candidate out of range");
    const TileShape sh = kFlowAdjShapes[choice];
    const TileList& tl = g.adj_tile_list(c.stream, sh.tw, sh.th);
    dispatch(dt, [&](auto z) {
        using T = decltype(z);
        ScopedTime st(&c, "flow_adj", 5.0 * sizeof(T) * g.pair_px, 12.0 * g.pair_px);
        auto k = interp == MMOF_INTERP_ROUND ? flow_adj_kernel<T, 1>(choice) : flow_adj_kernel<T, 0>(choice);
        hipLaunchKernelGGL(k, dim3((unsigned)tl.count), dim3(256), 0, c.stream, tl.buf.as<AdjTile>(), (const T*)r,
                           (const T*)v, (T*)u, direction, accumulate ? 1 : 0, rad,
                           res ? (const T*)res->x : (const T*)nullptr, res ? res->lam : nullptr,
                           res ? res->out : nullptr);
        MMOF_LAUNCH_CHECK();
    });
}

template <class T>
__global__ void k_zero(T* p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = T(0);
}

void launch_flow_dv(Ctx& c, Geom& g, int dt, int direction, int interp, const void* u, const void* v,
                    const void* w, void* gv) {
    if (g.n_pairs == 0) return;
    dispatch(dt, [&](auto z) {
        using T = decltype(z);
        if (interp == MMOF_INTERP_ROUND) {  // piecewise-constant warp: zero derivative
            hipLaunchKernelGGL(k_zero<T>, grid_for(2 * g.pair_px, 256), dim3(256), 0, c.stream, (T*)gv,
                               2 * g.pair_px);
            MMOF_LAUNCH_CHECK();
            return;
        }
        const TileList& tl = g.tile_list(c.stream, FTW, FTH, true);
        ScopedTime st(&c, "flow_dv");
        hipLaunchKernelGGL(k_flow_dv<T>, dim3((unsigned)tl.count), dim3(256), 0, c.stream, tl.buf.as<Tile>(),
                           g.dframes(), (const T*)u, (const T*)v, (const T*)w, (T*)gv, direction);
        MMOF_LAUNCH_CHECK();
    });
}

}  // namespace mmof

// Per-frame Gaussian blur with zero boundary, K = k1 k1^T (k1 normalised to unit sum, so
// sum K = 1).  Because K(i,j) = K(-i,-j) the transpose applies the same sum, so one
// kernel serves H and H^T.  Separable: a horizontal then a vertical pass over an LDS
// tile of outputs plus a halo of ksize/2 on every side (tile shape chosen per geometry).
#include "dev.h"
#include "kernels.h"

namespace mmof {

static constexpr int BRMAX = 7;

// TW x TH output tile per workgroup of 256 threads.  PERS: a grid of a few workgroups per
// CU loops over the tile list (persistent launch); otherwise one workgroup per tile.
template <class T, int TW, int TH, bool PERS>
__global__ __launch_bounds__(256) void k_blur(const Tile* __restrict__ tiles, int64_t n_tiles,
                                              const FrameInfo* __restrict__ fr, const double* __restrict__ k1d,
                                              int r, const T* __restrict__ in, T* __restrict__ out) {
    __shared__ T s_in[TH + 2 * BRMAX][TW + 2 * BRMAX];
    __shared__ T s_h[TH + 2 * BRMAX][TW];
    __shared__ T s_k[2 * BRMAX + 1];
    if (threadIdx.x < 2 * r + 1) s_k[threadIdx.x] = (T)k1d[threadIdx.x];
    const int64_t step = PERS ? gridDim.x : n_tiles;
    for (int64_t ti = PERS ? blockIdx.x : xcd_remap(blockIdx.x, gridDim.x); ti < n_tiles; ti += step) {
        const Tile tl = tiles[ti];
        const FrameInfo f = fr[tl.frame];
        const int nx = f.nx, ny = f.ny;
        const T* src = in + f.off;
        const int hw = TW + 2 * r, hh = TH + 2 * r;
        __syncthreads();  // LDS of the previous tile is free
        for (int i = threadIdx.x; i < hw * hh; i += 256) {
            const int ly = i / hw, lx = i % hw;
            const int y = tl.y0 - r + ly, x = tl.x0 - r + lx;
            s_in[ly][lx] = (y >= 0 && y < ny && x >= 0 && x < nx) ? src[(int64_t)y * nx + x] : T(0);
        }
        __syncthreads();
        for (int i = threadIdx.x; i < TW * hh; i += 256) {
            const int ly = i / TW, lx = i % TW;
            T acc = T(0);
            for (int j = 0; j <= 2 * r; ++j) acc += s_k[j] * s_in[ly][lx + j];
            s_h[ly][lx] = acc;
        }
        __syncthreads();
        for (int i = threadIdx.x; i < TW * TH; i += 256) {
            const int ly = i / TW, lx = i % TW;
            const int y = tl.y0 + ly, x = tl.x0 + lx;
            if (y >= ny || x >= nx) continue;
            T acc = T(0);
            for (int k = 0; k <= 2 * r; ++k) acc += s_k[k] * s_h[ly + k][lx];
            out[f.off + (int64_t)y * nx + x] = acc;
        }
    }
}

// The same sums with the radius R <= 4 compiled in (the 9-tap case).  Horizontal pass: a lane reads the
// quads left, at and right of its 4 pixels from global memory (any alignment; the neighbours' quads
// hit the cache) and forms its 4 outputs in registers, so that only the horizontal sums pass through
// LDS (staging the input there first cost a second pass and a barrier).  Vertical pass: a lane forms a
// 4 x 4 block from 4 + 2R quads of LDS.  Per output the taps are added in the order of k_blur, so the
// values are identical.  Bound by memory: 40 sequences of 64^2 to 256^2 pixels (2.1e7, FP32) take
// 31.5 us (5.3 TB/s), 80 with the input staged in LDS, and 38 to 36 with 64 x 64 and 128 x 32 tiles.
template <class T, int TW, int TH, bool PERS, int R>
__global__ __launch_bounds__(256) void k_blur_r(const Tile* __restrict__ tiles, int64_t n_tiles,
                                                const FrameInfo* __restrict__ fr, const double* __restrict__ k1d,
                                                const T* __restrict__ in, T* __restrict__ out) {
    constexpr int HH = TH + 2 * R, QW = TW / 4;   // rows of horizontal sums, quads per row
    static_assert(TW % 4 == 0 && TH % 4 == 0 && R <= 4 && 256 % QW == 0, "tiles split into 4-output segments");
    __shared__ Quad<T> s_h[HH][QW];
    T kk[2 * R + 1];
#pragma unroll
    for (int j = 0; j <= 2 * R; ++j) kk[j] = (T)k1d[j];
    const int64_t step = PERS ? gridDim.x : n_tiles;
    const int qx = (int)threadIdx.x % QW, ty = (int)threadIdx.x / QW;
    for (int64_t ti = PERS ? blockIdx.x : xcd_remap(blockIdx.x, gridDim.x); ti < n_tiles; ti += step) {
        const Tile tl = tiles[ti];
        const FrameInfo f = fr[tl.frame];
        const int nx = f.nx, ny = f.ny;
        const T* src = in + f.off;
        const int x = tl.x0 + 4 * qx, nv = min(4, nx - x);
        if constexpr (PERS) __syncthreads();  // LDS of the previous tile is free
        if (nv > 0) {
#pragma unroll 2
            for (int ly = ty; ly < HH; ly += 256 / QW) {
                const int y = tl.y0 - R + ly;
                Quad<T> o = zero4<T>();
                if (y >= 0 && y < ny) {
                    const T* row = src + (int64_t)y * nx + x;
                    // pixels x - 4 .. x + 7 (zeros outside the frame)
                    T v[12];
                    const Quad<T> l = x > 0 ? ld4u(row - 4) : zero4<T>(), m = ld4n(row, nv),
                                  r = nx - x > 4 ? ld4n(row + 4, nx - x - 4) : zero4<T>();
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        v[e] = l.v[e];
                        v[4 + e] = m.v[e];
                        v[8 + e] = r.v[e];
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        T acc = T(0);
#pragma unroll
                        for (int j = 0; j <= 2 * R; ++j) acc += kk[j] * v[4 - R + q + j];
                        o.v[q] = acc;
                    }
                }
                s_h[ly][qx] = o;
            }
        }
        __syncthreads();
        if (nv > 0) {
            for (int ly0 = 4 * ty; ly0 < TH; ly0 += 4 * (256 / QW)) {
                if (tl.y0 + ly0 >= ny) break;
                T acc[4][4];
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[q][e] = T(0);
#pragma unroll
                for (int c = 0; c < 4 + 2 * R; ++c) {
                    const Quad<T> h = s_h[ly0 + c][qx];
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (c - q >= 0 && c - q <= 2 * R)
#pragma unroll
                            for (int e = 0; e < 4; ++e) acc[q][e] += kk[c - q] * h.v[e];
                }
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (tl.y0 + ly0 + q < ny)
                        st4n(out + f.off + (int64_t)(tl.y0 + ly0 + q) * nx + x,
                             Quad<T>{{acc[q][0], acc[q][1], acc[q][2], acc[q][3]}}, nv);
            }
        }
    }
}

// tiles of the 9-tap kernel and of the general one
static const TileShape kBlur9Shapes[] = {{64, 32, 0}, {64, 64, 0}, {128, 32, 0}, {32, 32, 0}, {64, 32, 1}};
static const TileShape kBlurShapes[] = {{64, 16, 0}, {32, 32, 0}, {128, 8, 0}, {32, 16, 0}, {64, 16, 1}};
const int kBlurCandidates = sizeof(kBlurShapes) / sizeof(kBlurShapes[0]);
static_assert(sizeof(kBlur9Shapes) == sizeof(kBlurShapes), "both forms offer the same number of tile candidates");

TileShape blur_tile(const Plan& p, int choice) { return p.ksize == 9 ? kBlur9Shapes[choice] : kBlurShapes[choice]; }

void launch_blur(Ctx& c, Plan& p, int dt, const void* in, void* out, int choice) {
    Geom& g = *p.geom;
    if (choice < 0) choice = g.choice("blur", dt);
    MMOF_CHECK(choice >= 0 && choice < kBlurCandidates, MMOF_ERR_INVALID, "blur tile candidate out of range");
    const TileShape sh = blur_tile(p, choice);
    const TileList& tl = g.tile_list(c.stream, sh.tw, sh.th, false);
    if (tl.count == 0) return;
    dispatch(dt, [&](auto z) {
        using T = decltype(z);
        ScopedTime st(&c, "blur", 2.0 * sizeof(T) * g.n, 4.0 * p.ksize * g.n);
        const int64_t grid = sh.persistent ? std::min<int64_t>(tl.count, (int64_t)c.cu_count * 4) : tl.count;
        if (p.ksize == 9) {
            auto k = choice == 0 ? k_blur_r<T, 64, 32, false, 4>
                     : choice == 1 ? k_blur_r<T, 64, 64, false, 4>
                     : choice == 2 ? k_blur_r<T, 128, 32, false, 4>
                     : choice == 3 ? k_blur_r<T, 32, 32, false, 4>
                                   : k_blur_r<T, 64, 32, true, 4>;
            hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(256), 0, c.stream, tl.buf.as<Tile>(), tl.count,
                               g.dframes(), p.d_k1.as<double>(), (const T*)in, (T*)out);
        } else {
            auto k = choice == 0 ? k_blur<T, 64, 16, false>
                     : choice == 1 ? k_blur<T, 32, 32, false>
                     : choice == 2 ? k_blur<T, 128, 8, false>
                     : choice == 3 ? k_blur<T, 32, 16, false>
                                   : k_blur<T, 64, 16, true>;
            hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(256), 0, c.stream, tl.buf.as<Tile>(), tl.count,
                               g.dframes(), p.d_k1.as<double>(), p.ksize / 2, (const T*)in, (T*)out);
        }
        MMOF_LAUNCH_CHECK();
    });
}

}  // namespace mmof

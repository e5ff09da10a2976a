// vs_var.hip -- the variational alternative of the section 3.2 flow (flow = 2):
// coarse-to-fine warping with brightness and gradient constancy, a
// Charbonnier smoothness term and lagged Jacobi steps, on the same pyramids
// and flow domain as the plain estimator.  Every kernel is one pixel per
// thread over every field (pair x direction, or pair x camera for the
// derivatives) of every context in the group; FP32 in one prescribed order,
// correctly rounded division and square root.
#include "vs_device.h"

namespace vs {
namespace {

constexpr float VAR_EPS2 = 0.01f;   // Charbonnier epsilon^2 (epsilon = 0.1 luma)

// field f of level l for block b (fields of 256-pixel blocks, var_off)
__device__ __forceinline__ bool var_pixel(const DevPlan* __restrict__ P, int l, int b, int& f, int& x, int& y,
                                          int& w, int& h)
{
    f = find_field(P->var_off[l], 2 * P->n_pairs, b);
    const int p = f >> 1;
    w = P->lw[p][l];
    h = P->lh[p][l];
    const int i = (b - P->var_off[l][f]) * 256 + (int)threadIdx.x;
    if (i >= w * h) return false;
    x = i % w;
    y = i / w;
    return true;
}

__device__ __forceinline__ float at_clamped(const float* __restrict__ a, int w, int h, int x, int y)
{
    return a[(size_t)clampi(y, 0, h - 1) * w + clampi(x, 0, w - 1)];
}

__device__ __forceinline__ float cdx(const float* __restrict__ a, int w, int h, int x, int y)
{
    return 0.5f * (at_clamped(a, w, h, x + 1, y) - at_clamped(a, w, h, x - 1, y));
}

__device__ __forceinline__ float cdy(const float* __restrict__ a, int w, int h, int x, int y)
{
    return 0.5f * (at_clamped(a, w, h, x, y + 1) - at_clamped(a, w, h, x, y - 1));
}

// Bilinear samples of level planes at (X, Y), the position clamped into the
// level: the clamped corners and weights computed once for several planes.
struct BilAt {
    int i00, i10, i01, i11;
    float fx, fy;
};

__device__ __forceinline__ BilAt bil_at(int w, int h, float X, float Y)
{
    const float cx = clampf(X, 0.0f, (float)(w - 1)), cy = clampf(Y, 0.0f, (float)(h - 1));
    const float flx = floorf(cx), fly = floorf(cy);
    const int x0 = (int)flx, y0 = (int)fly;
    const int x1 = x0 + 1 < w ? x0 + 1 : w - 1, y1 = y0 + 1 < h ? y0 + 1 : h - 1;
    return BilAt{y0 * w + x0, y0 * w + x1, y1 * w + x0, y1 * w + x1, cx - flx, cy - fly};
}

__device__ __forceinline__ float bil_of(const float* __restrict__ a, const BilAt& B)
{
    const float p00 = a[B.i00], p10 = a[B.i10], p01 = a[B.i01], p11 = a[B.i11];
    const float t = __builtin_fmaf(B.fx, p10 - p00, p00);
    const float b = __builtin_fmaf(B.fx, p11 - p01, p01);
    return __builtin_fmaf(B.fy, b - t, t);
}

// Derivative planes of each camera's level image (field f = 2 p + camera):
// Dx, Dy central differences with clamped indices; Dxx, Dxy the central
// differences of Dx, Dyy of Dy (the first differences taken at the clamped
// neighbours, as the planes they are differences of).
__global__ __launch_bounds__(256) void k_var_deriv(const Batch B, int l)
{
    int c;
    const int b = batch_block(B, blockIdx.x, c);
    const DevPlan* __restrict__ P = B.plan[c];
    int f, x, y, w, h;
    if (!var_pixel(P, l, b, f, x, y, w, h)) return;
    const int p = f >> 1, cam = f & 1;
    if (kept_by_surrogate(P, p)) return;
    const float* __restrict__ I = P->pyr[p][cam][l];
    float* __restrict__ D = P->var_D[p][cam][l];
    const size_t n = (size_t)w * h, q = (size_t)y * w + x;
    const int xm = clampi(x - 1, 0, w - 1), xp = clampi(x + 1, 0, w - 1);
    const int ym = clampi(y - 1, 0, h - 1), yp = clampi(y + 1, 0, h - 1);
    D[q] = cdx(I, w, h, x, y);
    D[n + q] = cdy(I, w, h, x, y);
    D[2 * n + q] = 0.5f * (cdx(I, w, h, xp, y) - cdx(I, w, h, xm, y));
    D[3 * n + q] = 0.5f * (cdx(I, w, h, x, yp) - cdx(I, w, h, x, ym));
    D[4 * n + q] = 0.5f * (cdy(I, w, h, x, yp) - cdy(I, w, h, x, ym));
}

// Level start: the flow is 0 at the coarsest level, else 2 x the bilinear
// sample of the coarser level's flow at (x / 2 - 1/4, y / 2 - 1/4).  `added`: the
// coarser level's last increments have not been folded into its flow; each sampled
// flow takes them.
__device__ __forceinline__ float2 var_start(const DevPlan* __restrict__ P, int p, int dir, int l, int x, int y, bool added)
{
    if (l + 1 >= P->levels) return make_float2(0.0f, 0.0f);
    const int wc = P->lw[p][l + 1], hc = P->lh[p][l + 1];
    const float2* __restrict__ uc = P->flow[p][dir][l + 1];
    const float2* __restrict__ dc = P->var_dd[p][dir][l + 1][0];
    const float cx = clampf(__builtin_fmaf((float)x, 0.5f, -0.25f), 0.0f, (float)(wc - 1));
    const float cy = clampf(__builtin_fmaf((float)y, 0.5f, -0.25f), 0.0f, (float)(hc - 1));
    const float flx = floorf(cx), fly = floorf(cy);
    const int xa = (int)flx, ya = (int)fly;
    const float fx = cx - flx, fy = cy - fly;
    const int xb = xa + 1 < wc ? xa + 1 : wc - 1, yb = ya + 1 < hc ? ya + 1 : hc - 1;
    const size_t q[4] = {(size_t)ya * wc + xa, (size_t)ya * wc + xb, (size_t)yb * wc + xa, (size_t)yb * wc + xb};
    float2 v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[i] = uc[q[i]];
        if (added) {
            const float2 d = dc[q[i]];
            v[i] = make_float2(v[i].x + d.x, v[i].y + d.y);
        }
    }
    float a = __builtin_fmaf(fx, v[1].x - v[0].x, v[0].x);
    float b = __builtin_fmaf(fx, v[3].x - v[2].x, v[2].x);
    const float ux = 2.0f * __builtin_fmaf(fy, b - a, a);
    a = __builtin_fmaf(fx, v[1].y - v[0].y, v[0].y);
    b = __builtin_fmaf(fx, v[3].y - v[2].y, v[2].y);
    return make_float2(ux, 2.0f * __builtin_fmaf(fy, b - a, a));
}

// The level start by itself (without warps the level ends there).
__global__ __launch_bounds__(256) void k_var_init(const Batch B, int l)
{
    int c;
    const int b = batch_block(B, blockIdx.x, c);
    const DevPlan* __restrict__ P = B.plan[c];
    int f, x, y, w, h;
    if (!var_pixel(P, l, b, f, x, y, w, h)) return;
    const int p = f >> 1, dir = f & 1;
    if (kept_by_surrogate(P, p)) return;
    P->flow[p][dir][l][(size_t)y * w + x] = var_start(P, p, dir, l, x, y, false);
}

// One warp: the moving image and its derivatives sampled at x + (u, v), the
// data and gradient terms' coefficients (Iz Ix Iy Ixz Iyz Ixx Ixy Iyy).  The flow is
// the level's start at the first warp (a pass of its own before it took 20 us at
// level 0 of the 4 x 1080p ring), later the previous warp's with its increments
// added.  `reset`: the increments are set to 0 (no Jacobi steps follow: the first of
// those takes 0 by itself).
__global__ __launch_bounds__(256) void k_var_warp(const Batch B, int l, int first, int reset)
{
    int c;
    const int b = batch_block(B, blockIdx.x, c);
    const DevPlan* __restrict__ P = B.plan[c];
    int f, x, y, w, h;
    if (!var_pixel(P, l, b, f, x, y, w, h)) return;
    const int p = f >> 1, dir = f & 1;
    if (kept_by_surrogate(P, p)) return;
    const int tc = dir == 0 ? 0 : 1, mc = 1 - tc;
    const size_t n = (size_t)w * h, q = (size_t)y * w + x;
    float2* __restrict__ U = P->flow[p][dir][l];
    float2* __restrict__ dd = P->var_dd[p][dir][l][0];
    float2 u;
    if (first) {
        u = var_start(P, p, dir, l, x, y, true);
    } else {
        u = U[q];
        const float2 d = dd[q];
        u = make_float2(u.x + d.x, u.y + d.y);
    }
    U[q] = u;
    const float X = (float)x + u.x, Y = (float)y + u.y;
    const float* __restrict__ Mv = P->pyr[p][mc][l];
    const float* __restrict__ MD = P->var_D[p][mc][l];
    const float* __restrict__ TD = P->var_D[p][tc][l];
    const BilAt at = bil_at(w, h, X, Y);
    const float mw = bil_of(Mv, at), mx = bil_of(MD, at), my = bil_of(MD + n, at);
    const float mxx = bil_of(MD + 2 * n, at), mxy = bil_of(MD + 3 * n, at), myy = bil_of(MD + 4 * n, at);
    float* __restrict__ co = P->var_co[p][dir][l];
    co[q] = mw - P->pyr[p][tc][l][q];
    co[n + q] = mx;
    co[2 * n + q] = my;
    co[3 * n + q] = mx - TD[q];
    co[4 * n + q] = my - TD[n + q];
    co[5 * n + q] = mxx;
    co[6 * n + q] = mxy;
    co[7 * n + q] = myy;
    if (reset) dd[q] = make_float2(0.0f, 0.0f);
}

// VAR_T Jacobi steps of the linearised equations in one launch, increments src ->
// src ^ 1 (first: the increments before them are 0 and not read).  A block of 8
// wavefronts holds a region of 64 columns x 8 NP rows of one field, NP pixels per
// thread; a pixel's step reads one pixel to the left and up and two to the right and
// down, so each step makes good one column and row less at the start and two less at
// the end, and the block writes the pixels that are right after the last.  Per step
// the sums V = U + dU of the region and its ring (the ring as loaded: what it makes
// wrong is not written) lie in LDS; from them the smoothness Psi' of the region and
// a one-pixel ring (forward differences of V, 0 beyond the last column / row of the
// level), then each pixel's update from its 4 neighbours in the level.  Same
// operations as the per-pixel form: every V is the same sum, every Psi' the same
// expression.  The coefficients and the flow stay in registers over the steps.
// Bound by memory at the large levels (49 B read and 8 B written per pixel and
// launch; one step per launch moved them at the rate of a copy) and by the steps'
// latency at the small ones.  4 x 1080p ring, per step, levels 0 to 3: one step per
// launch 50.5, 20.4, 8.9, 7.2 us; this form 29, 12, 5.5, 3.7 us (with 32-row regions, 4 pixels
// per thread, 40 us at level 0: fewer wavefronts; with 1024 threads 30 us).

// 0.5 / sqrt(x) of the Charbonnier terms: x >= VAR_EPS2, or not a number
__device__ __forceinline__ float var_weight(float x)
{
    return __any(x > 0x1p100f) ? 0.5f / sqrtf(x) : half_rsqrt(x);
}

// Psi' of smoothness at a position with the sums v0, r to its right and d below
__device__ __forceinline__ float var_psi(float2 v0, float2 r, float2 d, bool right, bool down)
{
    const float ux = right ? r.x - v0.x : 0.0f, vx = right ? r.y - v0.y : 0.0f;
    const float uy = down ? d.x - v0.x : 0.0f, vy = down ? d.y - v0.y : 0.0f;
    return var_weight(__builtin_fmaf(ux, ux, __builtin_fmaf(uy, uy, __builtin_fmaf(vx, vx, __builtin_fmaf(vy, vy, VAR_EPS2)))));
}

// EDGE: the region or its ring leaves the level
template <int NP, bool EDGE>
__device__ __forceinline__ void var_steps(const int w, const int h, const int x0, const int y0, const float alpha,
                                          const float gamma, const float (&cf)[NP][8], const float2 (&u)[NP],
                                          float2 (&dq)[NP], uint32_t nd, float2* sV, float* sS)
{
    constexpr int ROWS = VAR_WV * NP, RW = VAR_TX + 3, SW = VAR_TX + 2;
    const int tid = threadIdx.x, lx = tid & 63, wv = tid >> 6;
    // this thread's position of Psi's ring: rows -1 and ROWS, columns -1 and 64
    constexpr int NRING = 2 * SW + 2 * ROWS;
    static_assert(NRING <= 64 * VAR_WV, "a ring position per thread");
    const int rr = tid < 2 * SW ? (tid < SW ? -1 : ROWS) : (tid - 2 * SW) >> 1;
    const int rc = tid < 2 * SW ? (tid < SW ? tid : tid - SW) - 1 : ((tid - 2 * SW) & 1 ? VAR_TX : -1);
    for (int t = 0; t < VAR_T; ++t) {
        if (t > 0) __syncthreads();   // every pixel has read its neighbours
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const int ty = wv + VAR_WV * k;
            float2 v = make_float2(u[k].x + dq[k].x, u[k].y + dq[k].y);
            if (EDGE && !(x0 + lx >= 0 && x0 + lx < w && y0 + ty >= 0 && y0 + ty < h)) v = make_float2(0.0f, 0.0f);
            sV[(1 + ty) * RW + 1 + lx] = v;
        }
        __syncthreads();
        auto psi = [&](int r, int c) {   // at region row r, column c
            const int vi = (r + 1) * RW + c + 1, xx = x0 + c, yy = y0 + r;
            const float s = var_psi(sV[vi], sV[vi + 1], sV[vi + RW], !EDGE || xx + 1 < w, !EDGE || yy + 1 < h);
            sS[(r + 1) * SW + c + 1] = EDGE && (xx < 0 || xx >= w || yy < 0 || yy >= h) ? 0.0f : s;
        };
#pragma unroll 1
        for (int k = 0; k < NP; ++k) psi(wv + VAR_WV * k, lx);
        if (tid < NRING) psi(rr, rc);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const int ty = wv + VAR_WV * k, x = x0 + lx, y = y0 + ty;
            float A11 = 0.0f, A12 = 0.0f, A22 = 0.0f, b1 = 0.0f, b2 = 0.0f;
            if (nd >> k & 1u) {
                const float c0 = cf[k][0], c1 = cf[k][1], c2 = cf[k][2], c3 = cf[k][3];
                const float c4 = cf[k][4], c5 = cf[k][5], c6 = cf[k][6], c7 = cf[k][7];
                const float e = __builtin_fmaf(c2, dq[k].y, __builtin_fmaf(c1, dq[k].x, c0));
                const float pd = var_weight(__builtin_fmaf(e, e, VAR_EPS2));
                const float gx = __builtin_fmaf(c6, dq[k].y, __builtin_fmaf(c5, dq[k].x, c3));
                const float gy = __builtin_fmaf(c7, dq[k].y, __builtin_fmaf(c6, dq[k].x, c4));
                const float pg = gamma * var_weight(__builtin_fmaf(gx, gx, __builtin_fmaf(gy, gy, VAR_EPS2)));
                A11 = __builtin_fmaf(pd, c1 * c1, pg * __builtin_fmaf(c5, c5, c6 * c6));
                A12 = __builtin_fmaf(pd, c1 * c2, pg * __builtin_fmaf(c5, c6, c6 * c7));
                A22 = __builtin_fmaf(pd, c2 * c2, pg * __builtin_fmaf(c6, c6, c7 * c7));
                b1 = -__builtin_fmaf(pd, c1 * c0, pg * __builtin_fmaf(c5, c3, c6 * c4));
                b2 = -__builtin_fmaf(pd, c2 * c0, pg * __builtin_fmaf(c6, c3, c7 * c4));
            }
            const int si = (ty + 1) * SW + lx + 1, vi = (ty + 1) * RW + lx + 1;
            const float s0 = sS[si];
            float S = 0.0f, Su = 0.0f, Sv = 0.0f;
            const bool has[4] = {x >= 1, x + 1 < w, y >= 1, y + 1 < h};
            const int so[4] = {-1, 1, -SW, SW}, vo[4] = {-1, 1, -RW, RW};
#pragma unroll
            for (int n = 0; n < 4; ++n) {
                const float wn = 0.5f * (s0 + sS[si + so[n]]);
                const float2 vn = sV[vi + vo[n]];
                if (!EDGE || has[n]) {
                    S += wn;
                    Su = __builtin_fmaf(wn, vn.x - u[k].x, Su);
                    Sv = __builtin_fmaf(wn, vn.y - u[k].y, Sv);
                }
            }
            const float nx = __builtin_fmaf(alpha, Su, __builtin_fmaf(-A12, dq[k].y, b1)), dx = __builtin_fmaf(alpha, S, A11);
            const float ny = __builtin_fmaf(alpha, Sv, __builtin_fmaf(-A12, dq[k].x, b2)), dy = __builtin_fmaf(alpha, S, A22);
            const bool ok = fminf(dx, dy) >= DIV_LO && fmaxf(dx, dy) <= DIV_HI && div_ok(nx, ny);
            if (__any(!ok))
                dq[k] = make_float2(nx / dx, ny / dy);
            else
                dq[k] = make_float2(div_by(nx, dx, div_rcp(dx)), div_by(ny, dy, div_rcp(dy)));
        }
    }
}

template <int NP>
__global__ __launch_bounds__(64 * VAR_WV) void k_var_jacobi(const Batch B, int l, int src, int first)
{
    constexpr int ROWS = VAR_WV * NP, RW = VAR_TX + 3, RH = ROWS + 3, SW = VAR_TX + 2;
    __shared__ float2 sV[RH * RW];
    __shared__ float sS[(ROWS + 2) * SW];
    int c;
    const int b = batch_block(B, blockIdx.x, c);
    const DevPlan* __restrict__ P = B.plan[c];
    const int f = find_field(P->var_toff[l], 2 * P->n_pairs, b);
    const int p = f >> 1, dir = f & 1;
    if (kept_by_surrogate(P, p)) return;
    const int w = P->lw[p][l], h = P->lh[p][l];
    constexpr int lost = VAR_T - 1, OX = VAR_OX, OY = var_oy(ROWS);   // pixels written
    const int t = b - P->var_toff[l][f], ntx = (w + OX - 1) / OX;
    const int x0 = (t % ntx) * OX - lost, y0 = (t / ntx) * OY - lost;
    const float2* __restrict__ U = P->flow[p][dir][l];
    const float2* __restrict__ d = P->var_dd[p][dir][l][src];
    const uint8_t* __restrict__ need = P->need[p][l];
    const int tid = threadIdx.x, lx = tid & 63, wv = tid >> 6;
    const size_t n = (size_t)w * h;
    const float* __restrict__ co = P->var_co[p][dir][l];
    // this thread's pixels' values (outside the level: the nearest one's, unused)
    float cf[NP][8];
    float2 u[NP], dq[NP];
    uint32_t nd = 0;
    const int xc = clampi(x0 + lx, 0, w - 1);
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        const size_t q = (size_t)clampi(y0 + wv + VAR_WV * k, 0, h - 1) * w + xc;
        u[k] = U[q];
        dq[k] = first ? make_float2(0.0f, 0.0f) : d[q];
        nd |= (uint32_t)(need[q] != 0) << k;
#pragma unroll
        for (int j = 0; j < 8; ++j) cf[k][j] = co[j * n + q];
    }
    // the ring of V: row -1, rows ROWS and ROWS + 1, columns -1, 64 and 65
    constexpr int NRING = 3 * RW + 3 * ROWS;
    static_assert(NRING <= 64 * VAR_WV, "a ring position per thread");
    if (tid < NRING) {
        const int e = tid - 3 * RW;
        const int r = tid < 3 * RW ? (tid < RW ? -1 : tid < 2 * RW ? ROWS : ROWS + 1) : e / 3;
        const int cc = tid < 3 * RW ? tid % RW - 1 : (e % 3 == 0 ? -1 : VAR_TX - 1 + e % 3);
        const int xx = x0 + cc, yy = y0 + r;
        float2 v = make_float2(0.0f, 0.0f);
        if (xx >= 0 && xx < w && yy >= 0 && yy < h) {
            const size_t q = (size_t)yy * w + xx;
            const float2 a = U[q], da = first ? make_float2(0.0f, 0.0f) : d[q];
            v = make_float2(a.x + da.x, a.y + da.y);
        }
        sV[(r + 1) * RW + cc + 1] = v;
    }
    const float alpha = P->var_alpha, gamma = P->var_gamma;
    if (x0 >= 1 && y0 >= 1 && x0 + VAR_TX + 2 <= w && y0 + ROWS + 2 <= h)
        var_steps<NP, false>(w, h, x0, y0, alpha, gamma, cf, u, dq, nd, sV, sS);
    else
        var_steps<NP, true>(w, h, x0, y0, alpha, gamma, cf, u, dq, nd, sV, sS);
    float2* __restrict__ out = P->var_dd[p][dir][l][src ^ 1];
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        const int ty = wv + VAR_WV * k, x = x0 + lx, y = y0 + ty;
        if (lx >= lost && lx < lost + OX && ty >= lost && ty < lost + OY && x < w && y < h)
            out[(size_t)y * w + x] = dq[k];
    }
}

// the last warp's increments added to the flow
__global__ __launch_bounds__(256) void k_var_fold(const Batch B, int l)
{
    int c;
    const int b = batch_block(B, blockIdx.x, c);
    const DevPlan* __restrict__ P = B.plan[c];
    int f, x, y, w, h;
    if (!var_pixel(P, l, b, f, x, y, w, h)) return;
    const int p = f >> 1, dir = f & 1;
    if (kept_by_surrogate(P, p)) return;
    const size_t q = (size_t)y * w + x;
    float2* __restrict__ U = P->flow[p][dir][l];
    const float2 u = U[q], d = P->var_dd[p][dir][l][0][q];
    U[q] = make_float2(u.x + d.x, u.y + d.y);
}

}  // namespace

// The variational flow of one level for every context of the group (their
// flow = 2): derivatives, initialisation, `var_outer` warps of `var_inner`
// Jacobi steps each (even steps end in increment buffer 0), the last
// increments folded in.
hipError_t launch_var(const Group& g, int l, hipStream_t s)
{
    Batch B;
    auto blocks = [&](const DevPlan& h) {
        return h.use_flow == 2 && h.flow_mode != VS_FLOW_SURROGATE && l < h.levels ? h.var_off[l][2 * h.n_pairs] : 0;
    };
    if (!make_batch(g, B, blocks)) return hipSuccess;
    const dim3 grid(B.off[B.n]), blk(256);
    int outer = g.hp[0]->var_outer, inner = g.hp[0]->var_inner;
    for (int c = 1; c < g.n; ++c)
        if (g.hp[c]->var_outer != outer || g.hp[c]->var_inner != inner) return hipErrorInvalidValue;
    if (inner % VAR_T) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_var_deriv, grid, blk, 0, s, B, l);
    if (outer == 0) hipLaunchKernelGGL(k_var_init, grid, blk, 0, s, B, l);
    auto jacobi = [&](int src, int first) {
        for (int rows = 8; rows <= 16; rows *= 2) {
            Batch BT;
            if (!make_batch(g, BT, [&](const DevPlan& h) {
                    return h.use_flow == 2 && h.flow_mode != VS_FLOW_SURROGATE && l < h.levels && h.var_rows[l] == rows
                               ? h.var_toff[l][2 * h.n_pairs] : 0; }))
                continue;
            const dim3 tg(BT.off[BT.n]);
            if (rows == 8) hipLaunchKernelGGL(k_var_jacobi<1>, tg, dim3(512), 0, s, BT, l, src, first);
            else hipLaunchKernelGGL(k_var_jacobi<2>, tg, dim3(512), 0, s, BT, l, src, first);
        }
    };
    const int launches = inner / VAR_T;
    for (int o = 0; o < outer; ++o) {
        hipLaunchKernelGGL(k_var_warp, grid, blk, 0, s, B, l, o == 0 ? 1 : 0, launches == 0 ? 1 : 0);
        // the last launch writes increment buffer 0
        for (int it = 0; it < launches; ++it) jacobi((launches - it) & 1, it == 0 ? 1 : 0);
    }
    // (a coarser level's last increments are added where the finer one starts)
    if (outer > 0 && l == 0) hipLaunchKernelGGL(k_var_fold, grid, blk, 0, s, B, l);
    return hipGetLastError();
}

}  // namespace vs

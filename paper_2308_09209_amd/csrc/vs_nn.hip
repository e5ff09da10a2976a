// vs_nn.hip -- the learned flow surrogate: a small 3x3 convolution network in
// BF16 with FP32 accumulation, forward and backward on the matrix cores
// (v_mfma_f32_16x16x32_bf16 forward, v_mfma_f32_16x16x16_bf16 weight
// gradient; wave64), plus the pointwise, loss and optimiser
// kernels its training needs.  Activations are NHWC with 16 or 32 channels;
// weights are [Cout][tap][Cin] (tap = 3 ky + kx).
#include <algorithm>
#include <atomic>

#include "vs_nn.h"

namespace vs {
namespace nn {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t f2bf(float f)
{
    // round to nearest even (finite inputs)
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// The image of block (tile, unit) b: lane i holds where image i ends, so one
// ballot counts the images that end at or before b.  (A walk over the table in the
// kernel arguments is a dependent scalar load per image and tile: 8 images of
// 256 x 1080, 32 -> 32, 63.9 us with it and 62.2 us without; a training step on 16
// images of 64 x 270 355 and 320 us.)
static_assert(MAXI <= 64, "an image per lane");

__device__ __forceinline__ int img_end(const ImgTable& T)
{
    const int lane = threadIdx.x & 63;
    return lane < T.n ? T.tile_off[lane + 1] : 0x7fffffff;
}

__device__ __forceinline__ int find_img(int end, int b) { return __popcll(__ballot(b >= end)); }

// ---------------------------------------------------------------------------
// 3x3 convolution, zero padding, as an implicit GEMM on the matrix cores with
// the weights as the A operand:
//   D[cout][pixel] = sum_k W[cout][k] X[pixel + off(tap)][cin],  k = tap CIN + cin,
// in 32-long k chunks (v_mfma_f32_16x16x32_bf16).  The grid is persistent: a
// block walks the CONV_T x CONV_T pixel tiles t = blockIdx.x, + gridDim.x, ...
// Each wavefront loads its A fragments (the weights, at most 72 VGPRs) once;
// per tile the block stages the tile and its one-pixel halo in LDS (16-byte
// vectors, pixel stride padded by one vector so that the 16 pixels a
// fragment read touches fall in distinct banks) and, while it multiplies,
// already holds the next tile's loads in flight.  A wavefront computes 4 rows
// of 16 pixels for every output channel (independent accumulator chains);
// every accumulator sums its chunks in k order.
// MFMA 16x16x32 BF16 fragments: lane l holds A[m = l % 16][k = 8 (l / 16) + i],
// B[k = 8 (l / 16) + i][n = l % 16] (i < 8) and D[m = 4 (l / 16) + i][n = l % 16]
// (i < 4): here m is the output channel and n the pixel, so a lane ends with
// 4 consecutive channels of one pixel.
// ---------------------------------------------------------------------------
constexpr int CONV_T = 16;                  // tile side (pixels)
constexpr int CONV_H = CONV_T + 2;          // tile with halo

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

struct ConvTile {
    int x0, y0, W, H;
    long base;
};

__device__ __forceinline__ ConvTile conv_tile(const ImgTable& T, int end, int t)
{
    const int img = find_img(end, t);
    ConvTile c;
    c.W = T.w[img];
    c.H = T.h[img];
    c.base = T.pix_off[img];
    const int ntx = (c.W + CONV_T - 1) / CONV_T;
    const int r = t - T.tile_off[img];
    c.x0 = (r % ntx) * CONV_T;
    c.y0 = (r / ntx) * CONV_T;
    return c;
}

template <int CIN, int COUT, int MODE>
__global__ __launch_bounds__(256) void k_conv3x3(const uint16_t* __restrict__ X, const uint16_t* __restrict__ Wt,
                                                 const float* __restrict__ bias, void* __restrict__ Y,
                                                 const ImgTable T, float alpha, void* __restrict__ aux)
{
    static_assert(CIN % 16 == 0 && COUT % 16 == 0, "channels in multiples of 16");
    constexpr int NT = COUT / 16;                  // 16-channel output groups
    constexpr int KT = 9 * CIN;                    // reduction length
    constexpr int NK = (KT + 31) / 32;             // 32-long chunks (the last one padded with zeros)
    constexpr int PV = CIN / 8;                    // 16-byte vectors per pixel
    constexpr int PSV = PV + 1;                    // LDS pixel stride in vectors
    constexpr int NV = CONV_H * CONV_H * PV;       // vectors per tile with halo
    constexpr int NL = (NV + 255) / 256;           // of them per thread
    __shared__ uint4 sX[CONV_H * CONV_H * PSV];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int m = lane & 15, kg = lane >> 4;
    const int ntiles = T.tile_off[T.n], iend = img_end(T);
    const uint4* __restrict__ Xv = reinterpret_cast<const uint4*>(X);

    bf16x8 wa[NT][NK];
#pragma unroll
    for (int tt = 0; tt < NT; ++tt)
#pragma unroll
        for (int kc = 0; kc < NK; ++kc) {
            const int k0 = kc * 32 + 8 * kg;
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (k0 < KT) v = *reinterpret_cast<const uint4*>(Wt + (long)(tt * 16 + m) * KT + k0);
            wa[tt][kc] = __builtin_bit_cast(bf16x8, v);
        }
    float bb[NT][4];
#pragma unroll
    for (int tt = 0; tt < NT; ++tt)
#pragma unroll
        for (int i = 0; i < 4; ++i) bb[tt][i] = bias ? bias[tt * 16 + 4 * kg + i] : 0.0f;

    // this thread's staging vectors, the same for every tile: halo row and
    // column and 16-byte vector of the pixel (packed r << 16 | c << 8 | v)
    int st[NL];
#pragma unroll
    for (int j = 0; j < NL; ++j) {
        const int e = tid + j * 256, px = e / PV;
        st[j] = e < NV ? (px / CONV_H) << 16 | (px % CONV_H) << 8 | (e % PV) : -1;
    }
    uint4 pf[NL];
    auto fetch = [&](const ConvTile& c) {
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (st[j] >= 0) {
                const int yy = c.y0 - 1 + (st[j] >> 16), xx = c.x0 - 1 + ((st[j] >> 8) & 255);
                if (yy >= 0 && yy < c.H && xx >= 0 && xx < c.W)
                    v = Xv[(c.base + (long)yy * c.W + xx) * PV + (st[j] & 255)];
            }
            pf[j] = v;
        }
    };

    ConvTile cur;
    if ((int)blockIdx.x < ntiles) {
        cur = conv_tile(T, iend, blockIdx.x);
        fetch(cur);
    }
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
        __syncthreads();                           // every wavefront is done with the previous tile
#pragma unroll
        for (int j = 0; j < NL; ++j)
            if (st[j] >= 0) sX[((st[j] >> 16) * CONV_H + ((st[j] >> 8) & 255)) * PSV + (st[j] & 255)] = pf[j];
        __syncthreads();
        const ConvTile c = cur;
        if (t + (int)gridDim.x < ntiles) {
            cur = conv_tile(T, iend, t + gridDim.x);
            fetch(cur);                            // the next tile's loads overlap this tile's products
        }

        // CONV_DGRAD: the layer's outputs, read before the products (clamped into the
        // image; used inside it; read after them: 15.7 us instead of 15.1 at
        // 16 images of 64 x 270)
        uint2 hv[4][NT];
        if (MODE == CONV_DGRAD) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const long q = c.base + (long)min(c.y0 + wv * 4 + g, c.H - 1) * c.W + min(c.x0 + m, c.W - 1);
#pragma unroll
                for (int tt = 0; tt < NT; ++tt)
                    hv[g][tt] = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(aux) + q * COUT + tt * 16 + 4 * kg);
            }
        }

        f32x4 acc[4][NT];
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int tt = 0; tt < NT; ++tt) acc[g][tt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int kc = 0; kc < NK; ++kc) {
            const int k0 = kc * 32 + 8 * kg;
            const bool kin = k0 < KT;
            const int tap = kin ? k0 / CIN : 8, cv = (k0 % CIN) / 8;
            const int dy = tap / 3, dx = tap % 3;          // halo offsets 0..2
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int r = wv * 4 + g;
                uint4 v = sX[((r + dy) * CONV_H + m + dx) * PSV + cv];
                if (!kin) v = make_uint4(0u, 0u, 0u, 0u);
                const bf16x8 b = __builtin_bit_cast(bf16x8, v);
#pragma unroll
                for (int tt = 0; tt < NT; ++tt)
                    acc[g][tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[tt][kc], b, acc[g][tt], 0, 0, 0);
            }
        }

        const int x = c.x0 + m;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int y = c.y0 + wv * 4 + g;
            if (y >= c.H || x >= c.W) continue;
            const long q = c.base + (long)y * c.W + x;
#pragma unroll
            for (int tt = 0; tt < NT; ++tt) {
                float v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    v[i] = acc[g][tt][i] + bb[tt][i];
                    if (MODE == CONV_LRELU) v[i] = v[i] > 0.0f ? v[i] : alpha * v[i];
                }
                const int co = tt * 16 + 4 * kg;
                if (MODE == CONV_DGRAD) {
                    // the gradient through the leaky ReLU that made aux = lrelu(z):
                    // rounded to BF16 before and after the slope
                    const uint2 hq = hv[g][tt];
                    const uint32_t hw[4] = {hq.x & 0xffffu, hq.x >> 16, hq.y & 0xffffu, hq.y >> 16};
                    uint32_t o[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float g = bf2f(__builtin_bit_cast(uint16_t, (__bf16)v[i]));
                        o[i] = f2bf(bf2f((uint16_t)hw[i]) > 0.0f ? g : alpha * g);
                    }
                    reinterpret_cast<uint2*>(static_cast<uint16_t*>(Y) + q * COUT + co)[0] =
                        make_uint2(o[0] | o[1] << 16, o[2] | o[3] << 16);
                } else if (MODE == CONV_FLOW2) {
                    if (co == 0) reinterpret_cast<float2*>(Y)[q] = make_float2(v[0], v[1]);
                } else if (MODE == CONV_F32) {
                    reinterpret_cast<float4*>(static_cast<float*>(Y) + q * COUT + co)[0] =
                        make_float4(v[0], v[1], v[2], v[3]);
                    if (aux)
                        reinterpret_cast<float4*>(static_cast<float*>(aux) + q * COUT + co)[0] =
                            make_float4(v[0], v[1], v[2], v[3]);
                } else {
                    // round to nearest even (v_cvt_pk_bf16_f32)
                    const bf16x2 lo = {(__bf16)v[0], (__bf16)v[1]}, hi = {(__bf16)v[2], (__bf16)v[3]};
                    reinterpret_cast<uint2*>(static_cast<uint16_t*>(Y) + q * COUT + co)[0] =
                        make_uint2(__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi));
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Weight gradient: dW[cout][tap][cin] = sum_pixels dZ[p][cout] X[p + tap][cin],
// db[cout] = sum_pixels dZ[p][cout].  A block reduces units of 256 consecutive
// pixels of one image, each on the matrix cores (M = cout, N = cin, K = pixels, 16 at a time in
// pixel order) into partial sums of its own; k_reduce_partials adds the partials
// in unit order, so the result does not depend on scheduling.  Wavefront w
// takes tap w, the tenth one the bias.
// The unit's dZ and, for each row of taps, its pixels shifted by that row (and
// one more at each end) sit in LDS pixel by pixel as in memory.  A fragment needs
// 4 pixels of one channel per lane, which ds_read_b64_tr_b16 gives: of 16 lanes,
// lane j names channels 4 (j % 4) .. + 3 of pixel j / 4 and receives channel j
// of the 4 pixels.  At 32 channels the two 32-byte halves of a pixel change
// places with every second pair of pixels, so that the 4 pixels a group reads
// lie in distinct banks.  Taps across a row's end are cleared by masks (4 pixels
// each) laid down with the unit.
// Bound by memory and its latency: 16 images of 64 x 270, 32 -> 32, 85 MB (40 of them
// the partial sums, 37 KB per unit) in 25 us, 3.4 TB/s; a wavefront waits for loads and
// barriers half of its time, the LDS is busy 5 %, the matrix cores 19 %.  11 us to
// add the sums (2-byte global loads per fragment and one thread per sum: 118 and 252 us).
// A block that walks units with the next one's loads in flight: 25 us, one block per
// unit: 27 us.
// ---------------------------------------------------------------------------
constexpr int WG_PIX = 256;
constexpr int WG_THREADS = 10 * 64;
constexpr int WG_SEG = WG_PIX + 2;          // pixels of one row of taps
constexpr int WG_BLOCKS = 512;              // two blocks per compute unit (LDS), each walking units of 256 pixels

typedef short short4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) short4v lds_short4;

// LDS position (2-byte values) of channel c (a multiple of 4) of pixel s
template <int CH>
__device__ __forceinline__ int wg_at(int s, int c)
{
    return s * CH + (CH == 32 ? c ^ ((s & 2) << 3) : c);
}

// vectors at the callers' own alignment: activations are 2-byte aligned here,
// partial sums 4-byte
typedef uint32_t u32x4_a2 __attribute__((ext_vector_type(4), aligned(2)));
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));

// a block's partial sums as its lanes hold them, [tap][a][c][lane][4], then the
// bias; wg_param: the parameter w[cout][9][cin], b[cout] that value k is of
template <int CIN, int COUT>
__device__ __forceinline__ int wg_param(int k)
{
    constexpr int MT = COUT / 16, NC = CIN / 16;
    if (k >= COUT * 9 * CIN) return k;
    const int i = k & 3, lane = (k >> 2) & 63, t = k >> 8;
    const int c = t % NC, a = (t / NC) % MT, tap = t / (NC * MT);
    return ((a * 16 + (lane >> 4) * 4 + i) * 9 + tap) * CIN + c * 16 + (lane & 15);
}

// 4 pixels of this lane's channel
__device__ __forceinline__ uint2 lds_tr4(const uint16_t* p)
{
    return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)p));
}

template <int CIN, int COUT>
__global__ __launch_bounds__(WG_THREADS) void k_conv3x3_wgrad(const uint16_t* __restrict__ X,
                                                              const uint16_t* __restrict__ dZ,
                                                              float* __restrict__ part, const ImgTable T)
{
    constexpr int MT = COUT / 16, NC = CIN / 16, NPAR = COUT * 9 * CIN + COUT;
    constexpr int VX = CIN / 8, VZ = COUT / 8;                       // 16-byte vectors per pixel
    constexpr int NX = 3 * WG_SEG * VX, NZ = WG_PIX * VZ;
    constexpr int LX = (NX + WG_THREADS - 1) / WG_THREADS, LZ = (NZ + WG_THREADS - 1) / WG_THREADS;
    __shared__ __align__(16) uint16_t sX[3 * WG_SEG * CIN];
    __shared__ __align__(16) uint16_t sZ[WG_PIX * COUT];
    __shared__ uint2 sMask[3][WG_PIX / 4];                           // per column of taps: the pixels that have it
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int j = lane & 15, kg = lane >> 4;
    const int nunits = T.tile_off[T.n], iend = img_end(T);
    const u32x4_a2* __restrict__ Xv = reinterpret_cast<const u32x4_a2*>(X);
    const u32x4_a2* __restrict__ Zv = reinterpret_cast<const u32x4_a2*>(dZ);

    // outside the image 0 (the rows above the first and below the last lie outside
    // its pixel range)
    u32x4_a2 px[LX], pz[LZ];
    auto fetch = [&](int u) {
        const int img = find_img(iend, u), W = T.w[img], npix = W * T.h[img], p0 = (u - T.tile_off[img]) * WG_PIX;
        const long base = T.pix_off[img];
#pragma unroll
        for (int i = 0; i < LX; ++i) {
            const int e = tid + i * WG_THREADS, sg = e / VX;
            const long q = (long)p0 + sg % WG_SEG - 1 + (long)(sg / WG_SEG - 1) * W;
            px[i] = u32x4_a2{0u, 0u, 0u, 0u};
            if (e < NX && q >= 0 && q < npix) px[i] = Xv[(base + q) * VX + e % VX];
        }
#pragma unroll
        for (int i = 0; i < LZ; ++i) {
            const int e = tid + i * WG_THREADS, q = p0 + e / VZ;
            pz[i] = u32x4_a2{0u, 0u, 0u, 0u};
            if (e < NZ && q < npix) pz[i] = Zv[(base + q) * VZ + e % VZ];
        }
    };
    const int tap = wv, dy = tap / 3, dx = tap % 3;                  // offsets 0..2 (wavefront 9: the bias)
    // the pixel and channels this lane names: k = 4 kg + i of each 16 pixels
    const int lp = 4 * kg + (j >> 2), lc = 4 * (j & 3);
    const uint16_t* sXd = sX + dy * (WG_SEG * CIN);

    if ((int)blockIdx.x < nunits) fetch(blockIdx.x);
    for (int u = blockIdx.x; u < nunits; u += gridDim.x) {
        const int img = find_img(iend, u), W = T.w[img], npix = W * T.h[img], p0 = (u - T.tile_off[img]) * WG_PIX;
        __syncthreads();                           // every wavefront is done with the previous pixels
        if (tid < 3 * (WG_PIX / 4)) {
            const int mx = tid / (WG_PIX / 4), g = tid % (WG_PIX / 4);
            uint32_t mk[4];
            int x = (p0 + 4 * g) % W;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bool ok = p0 + 4 * g + i < npix && !(mx == 0 && x == 0) && !(mx == 2 && x == W - 1);
                mk[i] = ok ? 0xffffu : 0u;
                x = x + 1 == W ? 0 : x + 1;
            }
            sMask[mx][g] = make_uint2(mk[0] | mk[1] << 16, mk[2] | mk[3] << 16);
        }
#pragma unroll
        for (int i = 0; i < LX; ++i) {
            const int e = tid + i * WG_THREADS, sg = e / VX;
            if (e < NX)
                *reinterpret_cast<uint4*>(sX + sg / WG_SEG * (WG_SEG * CIN) + wg_at<CIN>(sg % WG_SEG, 8 * (e % VX))) =
                    __builtin_bit_cast(uint4, px[i]);
        }
#pragma unroll
        for (int i = 0; i < LZ; ++i) {
            const int e = tid + i * WG_THREADS;
            if (e < NZ)
                *reinterpret_cast<uint4*>(sZ + wg_at<COUT>(e / VZ, 8 * (e % VZ))) = __builtin_bit_cast(uint4, pz[i]);
        }
        __syncthreads();
        if (u + (int)gridDim.x < nunits) fetch(u + gridDim.x);   // in flight during this unit's products
        float* out = part + (long)u * NPAR;
        if (wv == 9) {
            // bias gradient: lane co sums its channel over the pixels in order
            if (lane < COUT) {
                // (those past the image are 0)
                float s = 0.0f;
#pragma unroll 32
                for (int k = 0; k < WG_PIX; ++k) s += bf2f(sZ[wg_at<COUT>(k, lane & ~3) + (lane & 3)]);
                out[COUT * 9 * CIN + lane] = s;
            }
            continue;
        }
        f32x4 acc[MT][NC];
#pragma unroll
        for (int a = 0; a < MT; ++a)
#pragma unroll
            for (int c = 0; c < NC; ++c) acc[a][c] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 4
        for (int kb = 0; kb < WG_PIX; kb += 16) {
            const uint2 mk = sMask[dx][(kb >> 2) + kg];
            bf16x4 af[MT], bfr[NC];
#pragma unroll
            for (int a = 0; a < MT; ++a)
                af[a] = __builtin_bit_cast(bf16x4, lds_tr4(sZ + wg_at<COUT>(kb + lp, a * 16 + lc)));
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                uint2 v = lds_tr4(sXd + wg_at<CIN>(kb + lp + dx, c * 16 + lc));
                v.x &= mk.x;
                v.y &= mk.y;
                bfr[c] = __builtin_bit_cast(bf16x4, v);
            }
#pragma unroll
            for (int a = 0; a < MT; ++a)
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    acc[a][c] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(af[a], bfr[c], acc[a][c], 0, 0, 0);
        }
#pragma unroll
        for (int a = 0; a < MT; ++a)
#pragma unroll
            for (int c = 0; c < NC; ++c)
                *reinterpret_cast<f32x4_a4*>(out + (((tap * MT + a) * NC + c) * 64 + lane) * 4) = acc[a][c];
    }
}

// The gradients: sums of part[b][j] over the units b in order.  The sums are chains
// of nblocks additions each, so few threads can add; the block's other wavefronts
// bring the values in: 16 x RED_R rows of 64 sums at a time go through LDS, the
// next ones' loads in flight while the first wavefront adds.
// 1088 units of 37 KB: 11 us (32 sums per block 16 us, the LDS reads unrolled past
// 16 rows 15 to 22 us).
constexpr int RED_J = 64, RED_W = 16, RED_R = 16;
template <int CIN, int COUT>
__global__ __launch_bounds__(RED_J * RED_W) void k_reduce_partials(const float* __restrict__ part, int nblocks, int n,
                                                                   float* __restrict__ out)
{
    __shared__ float s_row[RED_W * RED_R][RED_J];
    const int lane = threadIdx.x % RED_J, wv = threadIdx.x / RED_J;
    const int j = blockIdx.x * RED_J + lane, jc = min(j, n - 1);
    float v[RED_R];
    auto fetch = [&](int b0) {
#pragma unroll
        for (int r = 0; r < RED_R; ++r) v[r] = part[(long)min(b0 + wv * RED_R + r, nblocks - 1) * n + jc];
    };
    fetch(0);
    float s = 0.0f;
    for (int b0 = 0; b0 < nblocks; b0 += RED_W * RED_R) {
        __syncthreads();
#pragma unroll
        for (int r = 0; r < RED_R; ++r) s_row[wv * RED_R + r][lane] = v[r];
        __syncthreads();
        if (b0 + RED_W * RED_R < nblocks) fetch(b0 + RED_W * RED_R);
        if (wv == 0) {
            const int m = min(RED_W * RED_R, nblocks - b0);
#pragma unroll 16
            for (int r = 0; r < m; ++r) s += s_row[r][lane];
        }
    }
    if (wv == 0 && j < n) out[wg_param<CIN, COUT>(j)] = s;
}

// W'[cin][tap][cout] = W[cout][8 - tap][cin]: the data-gradient convolution
// is the forward convolution with these weights.
__global__ __launch_bounds__(256) void k_flip_weights(const uint16_t* __restrict__ W, uint16_t* __restrict__ Wf,
                                                      int cin, int cout)
{
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= cin * 9 * cout) return;
    const int co = j % cout, tap = (j / cout) % 9, ci = j / (cout * 9);
    Wf[j] = W[((long)co * 9 + (8 - tap)) * cin + ci];
}

// dZ = dH * lrelu'(Z), with the sign of Z read from H = lrelu(Z) (alpha > 0)
__global__ __launch_bounds__(256) void k_lrelu_bwd(const uint16_t* __restrict__ dH, const uint16_t* __restrict__ Hh,
                                                   uint16_t* __restrict__ dZ, long n, float alpha)
{
    const long j = (long)blockIdx.x * 256 + threadIdx.x;
    if (j >= n) return;
    const float g = bf2f(dH[j]);
    dZ[j] = f2bf(bf2f(Hh[j]) > 0.0f ? g : alpha * g);
}

// ---------------------------------------------------------------------------
// Input packing: level luma images of a template / moving pair -> 16-channel
// BF16 (channel 0 template, 1 moving, rest 0), normalised (Y - 128) / 64.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_pack_pair(const float* __restrict__ Yt, const float* __restrict__ Ym,
                                                   uint16_t* __restrict__ X, long npix)
{
    const long p = (long)blockIdx.x * 256 + threadIdx.x;
    if (p >= npix) return;
    uint16_t v[16];
    v[0] = f2bf((Yt[p] - 128.0f) * (1.0f / 64.0f));
    v[1] = f2bf((Ym[p] - 128.0f) * (1.0f / 64.0f));
#pragma unroll
    for (int c = 2; c < 16; ++c) v[c] = 0;
    uint4* d = reinterpret_cast<uint4*>(X + p * 16);
    d[0] = make_uint4(v[0] | (uint32_t)v[1] << 16, 0u, 0u, 0u);
    d[1] = make_uint4(0u, 0u, 0u, 0u);
}

// ---------------------------------------------------------------------------
// Loss: mean end-point error of channels 0-1 of the FP32 prediction against
// the label flow, with its gradient (BF16, 16 channels, 2..15 zero) and one
// partial sum per block.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_epe_loss(const float* __restrict__ pred, const float* __restrict__ label,
                                                  uint16_t* __restrict__ dZ, float* __restrict__ block_loss, long npix,
                                                  float inv_n)
{
    __shared__ float s_red[4];
    const long p = (long)blockIdx.x * 256 + threadIdx.x;
    float e = 0.0f;
    uint16_t g0 = 0, g1 = 0;
    if (p < npix) {
        const float dx = pred[p * 16] - label[p * 2], dy = pred[p * 16 + 1] - label[p * 2 + 1];
        e = sqrtf(dx * dx + dy * dy + 1e-6f);
        g0 = f2bf(dx / e * inv_n);
        g1 = f2bf(dy / e * inv_n);
        uint4* d = reinterpret_cast<uint4*>(dZ + p * 16);
        d[0] = make_uint4(g0 | (uint32_t)g1 << 16, 0u, 0u, 0u);
        d[1] = make_uint4(0u, 0u, 0u, 0u);
    }
    for (int o = 32; o > 0; o >>= 1) e += __shfl_xor(e, o, 64);
    if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = e;
    __syncthreads();
    if (threadIdx.x == 0) block_loss[blockIdx.x] = ((s_red[0] + s_red[1]) + s_red[2]) + s_red[3];
}

// Adam on FP32 master parameters, with a BF16 copy of the weights
__global__ __launch_bounds__(256) void k_adam(float* __restrict__ w, float* __restrict__ m, float* __restrict__ v,
                                              const float* __restrict__ g, uint16_t* __restrict__ w_bf16, long n,
                                              float lr, float b1, float b2, float eps, float c1, float c2)
{
    const long j = (long)blockIdx.x * 256 + threadIdx.x;
    if (j >= n) return;
    const float gj = g[j];
    const float mj = b1 * m[j] + (1.0f - b1) * gj;
    const float vj = b2 * v[j] + (1.0f - b2) * gj * gj;
    m[j] = mj;
    v[j] = vj;
    const float wj = w[j] - lr * (mj / c1) / (sqrtf(vj / c2) + eps);
    w[j] = wj;
    if (w_bf16) w_bf16[j] = f2bf(wj);
}

// The Adam step of a whole network in one launch (4.9 us for 5 layers; 11 launches
// took 49 us): every parameter as k_adam does it, a weight's BF16 rounding stored as it is and in its flipped
// transpose's place (k_to_bf16, k_flip_weights).
__global__ __launch_bounds__(256) void k_adam_net(const NetTable N, float* __restrict__ w, float* __restrict__ m,
                                                  float* __restrict__ v, const float* __restrict__ g, float lr,
                                                  float b1, float b2, float eps, float c1, float c2)
{
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= N.off[N.n]) return;
    int l = 0;
    while (l + 1 < N.n && j >= N.off[l + 1]) ++l;
    const float gj = g[j];
    const float mj = b1 * m[j] + (1.0f - b1) * gj;
    const float vj = b2 * v[j] + (1.0f - b2) * gj * gj;
    m[j] = mj;
    v[j] = vj;
    const float wj = w[j] - lr * (mj / c1) / (sqrtf(vj / c2) + eps);
    w[j] = wj;
    const int i = j - N.off[l], ci = N.cin[l], co = N.cout[l];
    if (i >= co * 9 * ci) return;   // a bias
    const uint16_t b = f2bf(wj);
    N.w16[l][i] = b;
    const int c = i % ci, tap = (i / ci) % 9, o = i / (ci * 9);
    N.wf16[l][((long)c * 9 + (8 - tap)) * co + o] = b;
}

__global__ __launch_bounds__(256) void k_to_bf16(const float* __restrict__ a, uint16_t* __restrict__ b, long n)
{
    const long j = (long)blockIdx.x * 256 + threadIdx.x;
    if (j < n) b[j] = f2bf(a[j]);
}

// Sum of n per-block partial sums into one value (one block, fixed order:
// each thread adds a strided subset in index order, then a fixed tree).
__global__ __launch_bounds__(256) void k_sum_blocks(const float* __restrict__ part, int n, float* __restrict__ out)
{
    __shared__ float s_red[256];
    float acc = 0.0f;
    for (int i = threadIdx.x; i < n; i += 256) acc += part[i];
    s_red[threadIdx.x] = acc;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) s_red[threadIdx.x] += s_red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = s_red[0];
}

// Average pooling of a flow field by f x f blocks (the last row and column of
// blocks may be partial: the mean over the pixels they hold), divided by f
// so the result is in pooled-grid pixels: training labels of a coarser level.
__global__ __launch_bounds__(256) void k_pool_flow(const float* __restrict__ flow, int w, int h, int f,
                                                   float* __restrict__ out, int wo, int ho)
{
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= wo * ho) return;
    const int X = j % wo, Y = j / wo;
    const int x1 = min(w, (X + 1) * f), y1 = min(h, (Y + 1) * f);
    float sx = 0.0f, sy = 0.0f;
    for (int y = Y * f; y < y1; ++y)
        for (int x = X * f; x < x1; ++x) {
            sx += flow[((long)y * w + x) * 2];
            sy += flow[((long)y * w + x) * 2 + 1];
        }
    const float n = (float)((x1 - X * f) * (y1 - Y * f));
    out[(long)j * 2] = sx / n / (float)f;
    out[(long)j * 2 + 1] = sy / n / (float)f;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

template <int CIN, int COUT>
static hipError_t conv_mode(const uint16_t* X, const uint16_t* W, const float* b, void* Y, const ImgTable& T0,
                            int mode, float alpha, void* aux, hipStream_t s)
{
    // 16-byte vector loads and stores
    const bool vec_ok = ((uintptr_t)X | (uintptr_t)W | (uintptr_t)Y | (uintptr_t)aux) % 16 == 0;
    if (!vec_ok) return hipErrorInvalidValue;
    ImgTable T = T0;   // tiles of CONV_T x CONV_T pixels
    T.tile_off[0] = 0;
    for (int i = 0; i < T.n; ++i)
        T.tile_off[i + 1] = T.tile_off[i] + ((T.w[i] + CONV_T - 1) / CONV_T) * ((T.h[i] + CONV_T - 1) / CONV_T);
    for (int i = T.n + 1; i <= MAXI; ++i) T.tile_off[i] = T.tile_off[T.n];
    // persistent grid: as many blocks as the device holds at once
    static std::atomic<int> resident_blocks{0};
    int resident = resident_blocks.load(std::memory_order_relaxed);
    if (resident == 0) {
        int dev = 0, ncu = 0, per_cu = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e == hipSuccess) e = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
        if (e == hipSuccess)
            e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_conv3x3<CIN, COUT, CONV_LRELU>, 256, 0);
        if (e != hipSuccess) return e;
        resident = std::max(1, ncu * std::max(1, per_cu));
        resident_blocks.store(resident, std::memory_order_relaxed);
    }
    const dim3 g(std::min(T.tile_off[T.n], resident)), blk(256);
    switch (mode) {
    case CONV_LRELU: hipLaunchKernelGGL((k_conv3x3<CIN, COUT, CONV_LRELU>), g, blk, 0, s, X, W, b, Y, T, alpha, aux); break;
    case CONV_LINEAR: hipLaunchKernelGGL((k_conv3x3<CIN, COUT, CONV_LINEAR>), g, blk, 0, s, X, W, b, Y, T, alpha, aux); break;
    case CONV_F32: hipLaunchKernelGGL((k_conv3x3<CIN, COUT, CONV_F32>), g, blk, 0, s, X, W, b, Y, T, alpha, aux); break;
    case CONV_FLOW2: hipLaunchKernelGGL((k_conv3x3<CIN, COUT, CONV_FLOW2>), g, blk, 0, s, X, W, b, Y, T, alpha, aux); break;
    case CONV_DGRAD: hipLaunchKernelGGL((k_conv3x3<CIN, COUT, CONV_DGRAD>), g, blk, 0, s, X, W, b, Y, T, alpha, aux); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t conv3x3(const uint16_t* X, int cin, const uint16_t* W, const float* b, void* Y, int cout,
                   const ImgTable& T, int mode, float alpha, hipStream_t s, void* aux)
{
    if (T.tile_off[T.n] <= 0) return hipSuccess;
    if (cin == 16 && cout == 32) return conv_mode<16, 32>(X, W, b, Y, T, mode, alpha, aux, s);
    if (cin == 32 && cout == 32) return conv_mode<32, 32>(X, W, b, Y, T, mode, alpha, aux, s);
    if (cin == 32 && cout == 16) return conv_mode<32, 16>(X, W, b, Y, T, mode, alpha, aux, s);
    if (cin == 16 && cout == 16) return conv_mode<16, 16>(X, W, b, Y, T, mode, alpha, aux, s);
    return hipErrorInvalidValue;
}

int wgrad_blocks(const ImgTable& T)
{
    int n = 0;
    for (int i = 0; i < T.n; ++i) n += (T.w[i] * T.h[i] + WG_PIX - 1) / WG_PIX;
    return n;
}

template <int CIN, int COUT>
static void wgrad_launch(const uint16_t* X, const uint16_t* dZ, float* part, float* dWb, const ImgTable& G, hipStream_t s)
{
    const int nb = G.tile_off[G.n], n = COUT * 9 * CIN + COUT;
    hipLaunchKernelGGL((k_conv3x3_wgrad<CIN, COUT>), dim3(std::min(nb, WG_BLOCKS)), dim3(WG_THREADS), 0, s, X, dZ, part, G);
    hipLaunchKernelGGL((k_reduce_partials<CIN, COUT>), dim3((n + RED_J - 1) / RED_J), dim3(RED_J * RED_W), 0, s, part, nb,
                       n, dWb);
}

hipError_t conv3x3_wgrad(const uint16_t* X, int cin, const uint16_t* dZ, int cout, const ImgTable& T, float* part,
                         float* dWb, hipStream_t s)
{
    ImgTable G = T;   // tiles of WG_PIX pixels
    G.tile_off[0] = 0;
    for (int i = 0; i < T.n; ++i) G.tile_off[i + 1] = G.tile_off[i] + (T.w[i] * T.h[i] + WG_PIX - 1) / WG_PIX;
    const int nb = G.tile_off[G.n];
    if (nb <= 0) return hipSuccess;
    if (cin == 16 && cout == 32) wgrad_launch<16, 32>(X, dZ, part, dWb, G, s);
    else if (cin == 32 && cout == 32) wgrad_launch<32, 32>(X, dZ, part, dWb, G, s);
    else if (cin == 32 && cout == 16) wgrad_launch<32, 16>(X, dZ, part, dWb, G, s);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t flip_weights(const uint16_t* W, uint16_t* Wf, int cin, int cout, hipStream_t s)
{
    const int n = cin * 9 * cout;
    hipLaunchKernelGGL(k_flip_weights, dim3((n + 255) / 256), dim3(256), 0, s, W, Wf, cin, cout);
    return hipGetLastError();
}

hipError_t lrelu_bwd(const uint16_t* dH, const uint16_t* H, uint16_t* dZ, long n, float alpha, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_lrelu_bwd, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, dH, H, dZ, n, alpha);
    return hipGetLastError();
}

hipError_t pack_pair(const float* Yt, const float* Ym, uint16_t* X, long npix, hipStream_t s)
{
    if (npix <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_pack_pair, dim3((unsigned)((npix + 255) / 256)), dim3(256), 0, s, Yt, Ym, X, npix);
    return hipGetLastError();
}

hipError_t epe_loss(const float* pred, const float* label, uint16_t* dZ, float* block_loss, long npix, hipStream_t s)
{
    if (npix <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_epe_loss, dim3((unsigned)((npix + 255) / 256)), dim3(256), 0, s, pred, label, dZ, block_loss,
                       npix, 1.0f / (float)npix);
    return hipGetLastError();
}

hipError_t adam(float* w, float* m, float* v, const float* g, uint16_t* w_bf16, long n, float lr, float b1, float b2,
                float eps, int step, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
    hipLaunchKernelGGL(k_adam, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, w, m, v, g, w_bf16, n, lr, b1, b2,
                       eps, c1, c2);
    return hipGetLastError();
}

hipError_t adam_net(const NetTable& N, float* w, float* m, float* v, const float* g, float lr, float b1, float b2,
                    float eps, int step, hipStream_t s)
{
    const float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
    hipLaunchKernelGGL(k_adam_net, dim3((N.off[N.n] + 255) / 256), dim3(256), 0, s, N, w, m, v, g, lr, b1, b2, eps, c1,
                       c2);
    return hipGetLastError();
}

hipError_t to_bf16(const float* a, uint16_t* b, long n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_to_bf16, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a, b, n);
    return hipGetLastError();
}

hipError_t sum_blocks(const float* part, int n, float* out, hipStream_t s)
{
    hipLaunchKernelGGL(k_sum_blocks, dim3(1), dim3(256), 0, s, part, n, out);
    return hipGetLastError();
}

hipError_t pool_flow(const float* flow, int w, int h, int f, float* out, hipStream_t s)
{
    const int wo = (w + f - 1) / f, ho = (h + f - 1) / f;
    hipLaunchKernelGGL(k_pool_flow, dim3((unsigned)((wo * ho + 255) / 256)), dim3(256), 0, s, flow, w, h, f, out, wo, ho);
    return hipGetLastError();
}

size_t wgrad_scratch_bound(long npix, int nimg, int cin, int cout)
{
    return ((size_t)(npix + WG_PIX - 1) / WG_PIX + (size_t)nimg) * (size_t)(cout * 9 * cin + cout) * sizeof(float);
}

}  // namespace nn
}  // namespace vs

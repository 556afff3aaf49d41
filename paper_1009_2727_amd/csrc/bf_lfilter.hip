// bf_lfilter.hip -- learned current filter on the gfx950 matrix cores.
//
// The filter is three 5x5 convolutions with channels 1 -> 16 -> 16 -> 1, identity activations
// and no bias, shared by J_x, J_y and J_z.  It is linear and shift-invariant, so like the
// bilinear filter of Sec. 4.1 it commutes with the discrete divergence and keeps Gauss's law;
// its 13x13 footprint contains the 11x11 separable kernel of 4 bilinear passes + compensation,
// which it represents exactly (factors (1,4,6,4,1)/16, (1,4,6,4,1)/16 and (-1,3,-1) per axis).
//
// Precision: weights are BF16; every layer input x is split into hi = bf16(x) and
// lo = bf16(x - hi), both multiplied by the BF16 weights, accumulated in FP32, so the products
// keep ~16 significant bits of the input (BF16 rounding of the input alone would not be
// linear).  Each layer is an implicit GEMM on v_mfma_f32_16x16x32_bf16:
//   M = 16 consecutive output pixels of a row, N = 16 output channels (1-channel outputs pad N),
//   K = 25 taps x C_in x {hi, lo}, ordered k = t (2 C_in) + part C_in + ci.
// Operand layouts of the 16x16x32 BF16 MFMA (64 lanes, l = 16 g + i):
//   A (16x32): lane holds row i, k = 8g .. 8g+7;  B (32x16): lane holds column i, k = 8g .. 8g+7;
//   D (16x16 FP32): lane holds column i, rows 4g .. 4g+3.
//
// Training: backward-data is the same convolution with the adjoint weights
// W'(t, a, b) = W(24 - t, b, a); the weight gradient dW(t, ci, co) = sum_p in(p + o_t, ci)
// g(p, co) is an MFMA GEMM over pixels (hi/lo products hi*hi + hi*lo + lo*hi), each workgroup's
// share summed in registers and written once; the last kernel adds the shares in a fixed order
// and Adam (Kingma & Ba 2015) updates the FP32 master weights.
#include "bf_lfilter.h"
#include <algorithm>
#include <type_traits>

namespace bf {
namespace lf {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short us8 __attribute__((ext_vector_type(8)));

// output tile of a convolution: 256 pixels, 64 x 4 or 32 x 8 (a wave takes 64 of them: one row, or
// two); the 32-wide tile wastes less on images such as 32 x 32 patches
template <int TX> struct ConvTile {
    static constexpr int Y = 256 / TX, HX = TX + 4, HY = Y + 4;   // rows; extents with the 2-pixel halo
};

__device__ __forceinline__ unsigned short bf16_rne(float x)
{
    unsigned u = __float_as_uint(x);
    u += 0x7fffu + ((u >> 16) & 1u);   // round to nearest even (finite inputs)
    return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float bf16_val(unsigned short h) { return __uint_as_float((unsigned)h << 16); }

__device__ __forceinline__ f32x4 mfma(us8 a, us8 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

__device__ __forceinline__ long vaddr(const View& v, int img, int y, int x)
{
    int r = y + v.zoff;
    if (r >= v.rows) r -= v.rows;
    return (long)img * v.istride + (long)r * v.rstride + (long)x * v.ch;
}

// domain coordinate after the boundary rule: wrap on periodic axes, -1 outside otherwise
__device__ __forceinline__ int dwrap(int i, int n, int per)
{
    if (per) { i %= n; return i < 0 ? i + n : i; }
    return (i < 0 || i >= n) ? -1 : i;
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// two BF16 values (round to nearest even, in hardware) in one word
__device__ __forceinline__ unsigned pk_bf16(float a, float b)
{
    const bf16x2 p = {(__bf16)a, (__bf16)b};
    return __builtin_bit_cast(unsigned, p);
}

// hi and lo BF16 parts of four values
__device__ __forceinline__ void split4(const float4& v, uint2& hi, uint2& lo)
{
    hi.x = pk_bf16(v.x, v.y);
    hi.y = pk_bf16(v.z, v.w);
    lo.x = pk_bf16(v.x - __uint_as_float(hi.x << 16), v.y - __uint_as_float(hi.x & 0xffff0000u));
    lo.y = pk_bf16(v.z - __uint_as_float(hi.y << 16), v.w - __uint_as_float(hi.y & 0xffff0000u));
}

// A 16-channel tile of ROWS x COLS pixels from (y0, x0), four channels of a pixel per item: every
// item's load is issued before the first is used (one load at a time made staging the longest
// part of the training kernels), then put(pixel, first channel, hi, lo) stores it.  Beyond the
// domain: 0, or wrapped when WRAP asks for the boundary rule.
template <int ROWS, int COLS, bool WRAP, typename Put>
__device__ __forceinline__ void stage16(const View& v, const Domain& d, int img, int x0, int y0, Put put)
{
    constexpr int N = ROWS * COLS * 4, NI = (N + 255) / 256;
    float4 r[NI];
#pragma unroll
    for (int m = 0; m < NI; m++) {
        const int q = (int)threadIdx.x + 256 * m, c = 4 * (q & 3), p = q >> 2;
        int x = x0 + p % COLS, y = y0 + p / COLS;
        if constexpr (WRAP) {
            x = dwrap(x, d.nx, d.perx);
            y = dwrap(y, d.ny, d.pery);
        }
        const bool in = q < N && x >= 0 && y >= 0 && x < d.nx && y < d.ny;
        r[m] = in ? *reinterpret_cast<const float4*>(v.p + vaddr(v, img, y, x) + c) : float4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int m = 0; m < NI; m++) {
        const int q = (int)threadIdx.x + 256 * m;
        if (q < N) {
            uint2 hi, lo;
            split4(r[m], hi, lo);
            put(q >> 2, 4 * (q & 3), hi, lo);
        }
    }
}

// stage the input tile (halo 2) as [pixel][hi c0..c(C-1)][lo c0..c(C-1)]
template <int CIN, int TX>
__device__ __forceinline__ void stage_input(const View& in, const Domain& d, int img, int x0, int y0,
                                            unsigned short* tile)
{
    constexpr int HX = ConvTile<TX>::HX, HY = ConvTile<TX>::HY;
    if constexpr (CIN == 16) {
        stage16<HY, HX, true>(in, d, img, x0 - 2, y0 - 2, [&](int pix, int c, uint2 hi, uint2 lo) {
            *reinterpret_cast<uint2*>(tile + pix * 32 + c) = hi;
            *reinterpret_cast<uint2*>(tile + pix * 32 + 16 + c) = lo;
        });
    } else {
        for (int pix = threadIdx.x; pix < HY * HX; pix += 256) {
            const int x = dwrap(x0 - 2 + pix % HX, d.nx, d.perx);
            const int y = dwrap(y0 - 2 + pix / HX, d.ny, d.pery);
            const float v = (x >= 0 && y >= 0) ? in.p[vaddr(in, img, y, x)] : 0.f;
            const unsigned short hi = bf16_rne(v);
            tile[pix * 2] = hi;
            tile[pix * 2 + 1] = bf16_rne(v - bf16_val(hi));
        }
    }
}

// one convolution layer: out(p, co) = sum_{t, ci} W(t, ci, co) in(p + o_t, ci) on the
// domain, zero padding (or wrap) outside.  wpk holds the packed B fragments (nq x 64 lanes).
template <int CIN, int COUT, int TX>
__global__ void __launch_bounds__(256) k_lf_conv(View in, View out, Domain d, const us8* __restrict__ wpk)
{
    constexpr int NQ = (TAPS * CIN * 2 + 31) / 32, HX = ConvTile<TX>::HX, HY = ConvTile<TX>::HY;
    __shared__ __attribute__((aligned(16))) unsigned short tile[HY * HX * 2 * CIN];
    const int img = blockIdx.z, x0 = blockIdx.x * TX, y0 = blockIdx.y * ConvTile<TX>::Y;
    stage_input<CIN, TX>(in, d, img, x0, y0, tile);
    __syncthreads();
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
    f32x4 acc[4];
#pragma unroll
    for (int m = 0; m < 4; m++) acc[m] = f32x4{0.f, 0.f, 0.f, 0.f};
    // the wave's m-th group of 16 pixels: row and first column in the tile
    auto row_of = [&](int m) { return (wave * 64 + m * 16) / TX; };
    auto col_of = [&](int m) { return (m * 16) % TX; };
#pragma unroll 5
    for (int q = 0; q < NQ; q++) {
        const us8 b = wpk[q * 64 + lane];
#pragma unroll
        for (int m = 0; m < 4; m++) {
            const int px = col_of(m) + i, ty = row_of(m);
            us8 a;
            if constexpr (CIN == 16) {
                const int pix = (ty + q / 5) * HX + px + q % 5;   // tap q: offset (q/5-2, q%5-2)
                a = *reinterpret_cast<const us8*>(&tile[pix * 32 + g * 8]);
            } else {
#pragma unroll
                for (int j = 0; j < 8; j += 2) {
                    const int t = 16 * q + 4 * g + j / 2;
                    unsigned short h = 0, l = 0;
                    if (t < TAPS) {
                        const int pix = (ty + t / 5) * HX + px + t % 5;
                        h = tile[pix * 2];
                        l = tile[pix * 2 + 1];
                    }
                    a[j] = h;
                    a[j + 1] = l;
                }
            }
            acc[m] = mfma(a, b, acc[m]);
        }
    }
    if (i < COUT) {
#pragma unroll
        for (int m = 0; m < 4; m++) {
            const int y = y0 + row_of(m);
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const int x = x0 + col_of(m) + 4 * g + r;
                if (x < d.nx && y < d.ny) out.p[vaddr(out, img, y, x) + i] = acc[m][r];
            }
        }
    }
}

// packed B fragment q of a layer (or of its adjoint) by 64 threads
__device__ __forceinline__ void pack_chunk(const float* __restrict__ w, int cin, int cout, int adjoint, us8* wpk, int q)
{
    const int lane = threadIdx.x, n = lane & 15, g = lane >> 4;
    const int ci_n = adjoint ? cout : cin, co_n = adjoint ? cin : cout;
    us8 v;
#pragma unroll
    for (int j = 0; j < 8; j++) {
        const int k = 32 * q + 8 * g + j;
        const int t = k / (2 * ci_n), c = (k % (2 * ci_n)) % ci_n;
        float x = 0.f;
        if (t < TAPS && n < co_n)
            x = adjoint ? w[((TAPS - 1 - t) * cin + n) * cout + c] : w[(t * cin + c) * cout + n];
        v[j] = bf16_rne(x);
    }
    wpk[q * 64 + lane] = v;
}

// the packings a call needs, one block per fragment over all of them, and a double to clear
struct PackJob {
    const float* w;
    int cin, cout, adjoint, nq;
    us8* out;
};
struct PackJobs {
    PackJob j[5];
    int n;
    double* clear;
};
__global__ void k_lf_pack(PackJobs J)
{
    int q = blockIdx.x;
    if (q == 0 && threadIdx.x == 0 && J.clear) *J.clear = 0.0;
    for (int k = 0; k < J.n; k++) {
        if (q < J.j[k].nq) {
            pack_chunk(J.j[k].w, J.j[k].cin, J.j[k].cout, J.j[k].adjoint, J.j[k].out, q);
            return;
        }
        q -= J.j[k].nq;
    }
}

// ---- weight gradients ----------------------------------------------------------------------
// A workgroup goes over tiles of 32 x 8 pixels (blockIdx.x + k gridDim.x) and keeps its sums in
// registers, so that each writes its share once (share blockIdx.x of part): with a tile per
// workgroup and an atomic per weight and tile, 1024 workgroups added to the same few hundred
// addresses, 112, 57 and 30 us for the three layers of 128 patches of 32 x 32, against 8, 17 and
// 8 us; the whole training step 316 -> 89 us.
// K is 32 pixels of a row; channels are planes in LDS (hi and lo), so that a lane's eight pixels
// are one 16-byte read.
constexpr int WTX = 32, WTY = 8;
struct WTiles {
    int nx, ny, total;                  // tiles along x and y of an image, tiles in all
};
// plane strides in 16-bit words: 4 (mod 8) dwords, so the 16 lanes of a fragment's rows (one plane
// each) read 16-byte words that fall in different banks
constexpr int WG_P = WTY * WTX + 8;            // a channel of the gradient tile
constexpr int WI_W = 40;                       // row of the 16-channel input tile (36 used)
constexpr int WI_P = (WTY + 4) * WI_W + 8;     // a channel of it

// 16 channels of a tile into planes hi and lo of COLS-wide rows W words apart, channels P words apart
template <int ROWS, int COLS, int W, int P, bool WRAP>
__device__ __forceinline__ void stage_planes(const View& v, const Domain& d, int img, int x0, int y0,
                                             unsigned short* hi, unsigned short* lo)
{
    stage16<ROWS, COLS, WRAP>(v, d, img, x0, y0, [&](int pix, int c, uint2 h, uint2 l) {
        const int o = c * P + pix / COLS * W + pix % COLS;
        hi[o] = (unsigned short)h.x;
        hi[o + P] = (unsigned short)(h.x >> 16);
        hi[o + 2 * P] = (unsigned short)h.y;
        hi[o + 3 * P] = (unsigned short)(h.y >> 16);
        lo[o] = (unsigned short)l.x;
        lo[o + P] = (unsigned short)(l.x >> 16);
        lo[o + 2 * P] = (unsigned short)l.y;
        lo[o + 3 * P] = (unsigned short)(l.y >> 16);
    });
}

// eight consecutive 16-bit words of a row from the six dwords that start at word 0, shifted by s words
template <int S>
__device__ __forceinline__ us8 window8(const unsigned* w)
{
    unsigned r[4];
#pragma unroll
    for (int j = 0; j < 4; j++)
        r[j] = S % 2 == 0 ? w[S / 2 + j] : __builtin_amdgcn_alignbit(w[S / 2 + j + 1], w[S / 2 + j], 16);
    return __builtin_bit_cast(us8, uint4{r[0], r[1], r[2], r[3]});
}

// 16 -> 16 channels: rows of the product are (tap, ci), so a wave's 25 accumulators are the 25
// taps; the taps of one row dy share the lane's window of twelve pixels
__global__ void __launch_bounds__(256) k_lf_wgrad_wide(View in, View gout, Domain d, WTiles wt, float* part)
{
    __shared__ __attribute__((aligned(16))) unsigned short sm[2 * 16 * WI_P + 2 * 16 * WG_P];
    unsigned short *ih = sm, *il = ih + 16 * WI_P, *gh = il + 16 * WI_P, *gl = gh + 16 * WG_P;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
    f32x4 acc[TAPS];
#pragma unroll
    for (int t = 0; t < TAPS; t++) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int tile = blockIdx.x; tile < wt.total; tile += gridDim.x) {
        const int img = tile / (wt.nx * wt.ny), r = tile % (wt.nx * wt.ny), x0 = r % wt.nx * WTX, y0 = r / wt.nx * WTY;
        __syncthreads();                // the previous tile is done with the LDS
        stage_planes<WTY + 4, WTX + 4, WI_W, WI_P, true>(in, d, img, x0 - 2, y0 - 2, ih, il);
        stage_planes<WTY, WTX, WTX, WG_P, false>(gout, d, img, x0, y0, gh, gl);   // pixels beyond the image: 0
        __syncthreads();
#pragma unroll 1
        for (int yy = 0; yy < 2; yy++) {
            const int y = 2 * wave + yy;
            const us8 bh = *reinterpret_cast<const us8*>(gh + i * WG_P + y * WTX + 8 * g);
            const us8 bl = *reinterpret_cast<const us8*>(gl + i * WG_P + y * WTX + 8 * g);
#pragma unroll
            for (int dy = 0; dy < 5; dy++) {
                unsigned wh[6], wl[6];
                const int o = i * WI_P + (y + dy) * WI_W + 8 * g;
                *reinterpret_cast<uint4*>(wh) = *reinterpret_cast<const uint4*>(ih + o);
                *reinterpret_cast<uint2*>(wh + 4) = *reinterpret_cast<const uint2*>(ih + o + 8);
                *reinterpret_cast<uint4*>(wl) = *reinterpret_cast<const uint4*>(il + o);
                *reinterpret_cast<uint2*>(wl + 4) = *reinterpret_cast<const uint2*>(il + o + 8);
                auto tap = [&](auto dx) {
                    constexpr int DX = decltype(dx)::value;
                    const us8 ah = window8<DX>(wh), al = window8<DX>(wl);
                    f32x4& c = acc[5 * dy + DX];
                    c = mfma(ah, bh, c);
                    c = mfma(ah, bl, c);
                    c = mfma(al, bh, c);
                };
                tap(std::integral_constant<int, 0>{});
                tap(std::integral_constant<int, 1>{});
                tap(std::integral_constant<int, 2>{});
                tap(std::integral_constant<int, 3>{});
                tap(std::integral_constant<int, 4>{});
            }
        }
    }
    // the four waves' sums, then the share: element (t, ci = 4 g + r, co = i)
    float* red = reinterpret_cast<float*>(sm);
    static_assert(sizeof(sm) >= TAPS * 256 * 4, "the share fits the tiles' LDS");
    for (int w = 0; w < 4; w++) {
        __syncthreads();
        if (wave == w) {
#pragma unroll
            for (int t = 0; t < TAPS; t++)
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    float* p = red + t * 256 + (4 * g + r) * 16 + i;
                    *p = w == 0 ? acc[t][r] : *p + acc[t][r];
                }
        }
    }
    __syncthreads();
    float* out = part + (long)blockIdx.x * TAPS * 256;
    for (int q = threadIdx.x; q < TAPS * 256; q += 256) out[q] = red[q];
}

// 1 -> 16 channels: rows of the product are the taps (two groups of 16, 25 used).  A tap's shift
// along x would leave its eight pixels unaligned: the one-channel tile is kept twice, the second
// copy one word on, so that every window starts on a dword.  With flip, the transposed problem of
// a 16 -> 1 layer: dW(t, ci) = sum_q h(q, ci) g(q - o_t), in = g, gout = h and the taps reversed.
constexpr int WN_W = 40;
__global__ void __launch_bounds__(256) k_lf_wgrad_narrow(View in, View gout, Domain d, WTiles wt, int flip, float* part)
{
    __shared__ __attribute__((aligned(16))) unsigned short sn[2][2][(WTY + 4) * WN_W];   // [hi, lo][copy]
    __shared__ __attribute__((aligned(16))) unsigned short sg[2 * 16 * WG_P];
    __shared__ float red[TAPS * 16];
    unsigned short *gh = sg, *gl = sg + 16 * WG_P;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
    // this lane's row of each group: its tap's offset in the tile and which copy holds it
    int off[2], copy[2];
#pragma unroll
    for (int m = 0; m < 2; m++) {
        const int t = min(16 * m + i, TAPS - 1), dx = t % 5;
        copy[m] = dx & 1;
        off[m] = (t / 5) * WN_W + (dx & ~1) + 8 * g;
    }
    f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
    for (int tile = blockIdx.x; tile < wt.total; tile += gridDim.x) {
        const int img = tile / (wt.nx * wt.ny), r = tile % (wt.nx * wt.ny), x0 = r % wt.nx * WTX, y0 = r / wt.nx * WTY;
        __syncthreads();
        for (int q = threadIdx.x; q < (WTY + 4) * (WTX + 4); q += 256) {
            const int cx = q % (WTX + 4), cy = q / (WTX + 4);
            const int x = dwrap(x0 - 2 + cx, d.nx, d.perx), y = dwrap(y0 - 2 + cy, d.ny, d.pery);
            const float f = (x >= 0 && y >= 0) ? in.p[vaddr(in, img, y, x)] : 0.f;
            const unsigned short h = bf16_rne(f), l = bf16_rne(f - bf16_val(h));
            sn[0][0][cy * WN_W + cx] = h;
            sn[1][0][cy * WN_W + cx] = l;
            if (cx > 0) {
                sn[0][1][cy * WN_W + cx - 1] = h;
                sn[1][1][cy * WN_W + cx - 1] = l;
            }
        }
        stage_planes<WTY, WTX, WTX, WG_P, false>(gout, d, img, x0, y0, gh, gl);   // pixels beyond the image: 0
        __syncthreads();
#pragma unroll
        for (int yy = 0; yy < 2; yy++) {
            const int y = 2 * wave + yy;
            const us8 bh = *reinterpret_cast<const us8*>(gh + i * WG_P + y * WTX + 8 * g);
            const us8 bl = *reinterpret_cast<const us8*>(gl + i * WG_P + y * WTX + 8 * g);
#pragma unroll
            for (int m = 0; m < 2; m++) {
                const unsigned* ph = reinterpret_cast<const unsigned*>(sn[0][copy[m]] + y * WN_W + off[m]);
                const unsigned* pl = reinterpret_cast<const unsigned*>(sn[1][copy[m]] + y * WN_W + off[m]);
                const us8 ah = __builtin_bit_cast(us8, uint4{ph[0], ph[1], ph[2], ph[3]});
                const us8 al = __builtin_bit_cast(us8, uint4{pl[0], pl[1], pl[2], pl[3]});
                acc[m] = mfma(ah, bh, acc[m]);
                acc[m] = mfma(ah, bl, acc[m]);
                acc[m] = mfma(al, bh, acc[m]);
            }
        }
    }
    for (int w = 0; w < 4; w++) {
        __syncthreads();
        if (wave == w) {
#pragma unroll
            for (int m = 0; m < 2; m++)
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    const int t = 16 * m + 4 * g + r;
                    if (t >= TAPS) continue;
                    float* p = red + (flip ? TAPS - 1 - t : t) * 16 + i;
                    *p = w == 0 ? acc[m][r] : *p + acc[m][r];
                }
        }
    }
    __syncthreads();
    float* out = part + (long)blockIdx.x * TAPS * 16;
    for (int q = threadIdx.x; q < TAPS * 16; q += 256) out[q] = red[q];
}

// mean squared error over the pixels at least `margin` from the image edges:
// loss += sum (out - target)^2 / count, g = 2 (out - target) / count there, 0 elsewhere
__global__ void __launch_bounds__(256) k_lf_loss(const float* __restrict__ out,
                                                 const float* __restrict__ target, float* g, Domain d,
                                                 int margin, double inv_count, double* loss)
{
    __shared__ double red[4];
    const long n = (long)d.nimg * d.ny * d.nx;
    double s = 0.0;
    for (long q = (long)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (long)gridDim.x * blockDim.x) {
        const int x = (int)(q % d.nx), y = (int)((q / d.nx) % d.ny);
        const bool in = x >= margin && x < d.nx - margin && y >= margin && y < d.ny - margin;
        const double e = in ? (double)out[q] - (double)target[q] : 0.0;
        s += e * e;
        g[q] = (float)(2.0 * e * inv_count);
    }
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(loss, (red[0] + red[1] + red[2] + red[3]) * inv_count);
}

// The end of a training step: the gradient as the sum of the workgroups' shares (32 parameters and
// 8 slices of the shares per workgroup), the caller's copies of gradient and loss, and Adam on the
// FP32 master weights when step is set; c1 = 1/(1 - beta1^t), c2 = 1/(1 - beta2^t)
struct Shares {
    const float* p[3];                  // of the layers' weights
    int n[3];
};
struct AdamArgs {
    float *w, *m, *v;
    float lr, b1, b2, eps, c1, c2;
    int step;
};
__global__ void __launch_bounds__(256) k_lf_finish(Shares S, AdamArgs A, const double* loss, double* loss_out,
                                                   float* grad_out)
{
    __shared__ float red[8][32];
    const int q = blockIdx.x * 32 + (threadIdx.x & 31), slice = threadIdx.x >> 5;
    static_assert(NPARAM % 32 == 0, "whole workgroups");
    const int l = q < OFF_W2 ? 0 : q < OFF_W3 ? 1 : 2, first = l == 0 ? OFF_W1 : l == 1 ? OFF_W2 : OFF_W3;
    const int size = l == 1 ? TAPS * C * C : TAPS * C;
    float sum = 0.f;
#pragma unroll 8
    for (int k = slice; k < S.n[l]; k += 8) sum += S.p[l][(long)k * size + q - first];
    red[slice][threadIdx.x & 31] = sum;
    __syncthreads();
    if (blockIdx.x == 0 && threadIdx.x == 0 && loss_out) *loss_out = *loss;
    if (slice) return;
    float g = red[0][threadIdx.x];
#pragma unroll
    for (int k = 1; k < 8; k++) g += red[k][threadIdx.x];
    if (grad_out) grad_out[q] = g;
    if (!A.step) return;
    const float m = A.b1 * A.m[q] + (1.f - A.b1) * g;
    const float v = A.b2 * A.v[q] + (1.f - A.b2) * g * g;
    A.m[q] = m;
    A.v[q] = v;
    A.w[q] -= A.lr * (m * A.c1) / (sqrtf(v * A.c2) + A.eps);
}

// ---- streamed forward pass (inference) ---------------------------------------------------
// A workgroup walks down a strip of SOW output columns, one row per step, with all three
// layers in flight: at step s layer 1 produces h1 row s+1, layer 2 consumes h1 row s and
// completes h2 row s-2, layer 3 consumes h2 row s-3 and completes output row s-5.  Each layer
// reads its source one row at a time from small LDS rings (the input 8 rows, h1 and h2 two):
//  * layer 2 (16 -> 16) keeps five accumulator tiles for the h2 rows s-2 .. s+2, so one A
//    fragment of h1 row s (16 pixels x 16 channels, tap dx) feeds five MFMAs (taps dy = 0..4);
//    its 25 B fragments stay in registers;
//  * layer 3 (16 -> 1) puts the tap row dy in the MFMA's N dimension: column dy of the
//    accumulator holds the partial sum of output row r + 2 - dy after h2 row r; shifting the
//    columns by one lane (DPP row_shr) before each row moves every partial to its next dy, and
//    column 4 leaves complete;
//  * layer 1 (1 -> 16) gathers its 25 taps x {hi, lo} from the input ring (two MFMAs).
// Layers 1 and 2 take the weights as the MFMA's A operand and the pixels as B, so that a lane
// ends with four consecutive channels of one pixel: their hi and lo BF16 parts are converted in
// hardware and stored as two 8-byte words.  The input ring keeps every row twice (rows r and
// r + SIR of a 2 SIR-row buffer), so the five rows a layer-1 tap set reads are contiguous.
// Out-of-domain h1 and h2 pixels on non-periodic axes are written as zeros, as the separate
// layers read them.  Four waves: wave w computes h1 strip w, h2 strip w and output strip w,
// strips of 16 columns; the last four columns of h1 and h2 are zero padding that only feeds
// columns beyond the workgroup's outputs.
constexpr int SOW = 56;              // output columns per workgroup: [x0, x0 + 56)
constexpr int SH1W = 68;             // h1 columns [x0 - 4, x0 + 64): 64 computed, 4 of padding
constexpr int SH2W = 68;             // h2 columns [x0 - 2, x0 + 66): 64 computed, 4 of padding
constexpr int SIW = 68;              // input columns: [x0 - 6, x0 + 62)
constexpr int SIR = 8;               // input ring rows

// one image plane per blockIdx.z % n (up to 3: the current components), images blockIdx.z / n
struct Planes {
    View in[3], out[3];
    Domain d[3];
    int n, oh;                      // planes, output rows per workgroup
};

// A row of h1 or h2 in LDS is four planes of W pixels x 8 BF16 words: the 32 words of a pixel
// (hi parts of channels 0-7, 8-15, then lo parts of 0-7, 8-15) split into 16-byte chunks by k, so
// the 16 lanes that read one k chunk of a fragment (consecutive pixels) touch 256 consecutive
// bytes.  Channels 4g .. 4g + 3 of pixel c go to chunk g / 2 (hi) and 2 + g / 2 (lo), half g % 2.
__device__ __forceinline__ void store_ch4(unsigned short* row, int W, int c, int g, f32x4 v)
{
    const unsigned h01 = pk_bf16(v[0], v[1]), h23 = pk_bf16(v[2], v[3]);
    const unsigned l01 = pk_bf16(v[0] - __uint_as_float(h01 << 16), v[1] - __uint_as_float(h01 & 0xffff0000u));
    const unsigned l23 = pk_bf16(v[2] - __uint_as_float(h23 << 16), v[3] - __uint_as_float(h23 & 0xffff0000u));
    unsigned short* p = row + ((g >> 1) * W + c) * 8 + 4 * (g & 1);
    *reinterpret_cast<uint2*>(p) = make_uint2(h01, h23);
    *reinterpret_cast<uint2*>(p + 2 * W * 8) = make_uint2(l01, l23);
}

// hi | lo << 16 of one value
__device__ __forceinline__ unsigned hilo(float v)
{
    const unsigned h = pk_bf16(v, 0.f) & 0xffffu;
    return h | (pk_bf16(v - __uint_as_float(h << 16), 0.f) << 16);
}

__device__ __forceinline__ f32x4 shift_columns(f32x4 t)
{
    // lane i of each 16-lane row takes lane i - 1; lane 0 takes 0 (row_shr:1, bound_ctrl)
    f32x4 r;
#pragma unroll
    for (int k = 0; k < 4; k++)
        r[k] = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(t[k]), 0x111, 0xf, 0xf, true));
    return r;
}

__global__ void __launch_bounds__(256) k_lf_stream(Planes P, const us8* __restrict__ w1, const us8* __restrict__ w2,
                                                   const us8* __restrict__ w3)
{
    __shared__ unsigned sin[2 * SIR * SIW];                               // hi | lo << 16
    __shared__ __attribute__((aligned(16))) unsigned short sh1[2 * SH1W * 32];   // [row][k chunk][col][8]
    __shared__ __attribute__((aligned(16))) unsigned short sh2[2 * SH2W * 32];
    const int pl = blockIdx.z % P.n, img = blockIdx.z / P.n;
    const View in = P.in[pl], out = P.out[pl];
    const Domain d = P.d[pl];
    const int x0 = blockIdx.x * SOW, y0 = blockIdx.y * P.oh;
    if (x0 >= d.nx || y0 >= d.ny || img >= d.nimg) return;
    const int yend = min(y0 + P.oh, d.ny);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;

    for (int q = threadIdx.x; q < SH1W * 32; q += 256) reinterpret_cast<unsigned*>(sh1)[q] = 0u;
    for (int q = threadIdx.x; q < SH2W * 32; q += 256) reinterpret_cast<unsigned*>(sh2)[q] = 0u;
    us8 b1[2], b2[TAPS], b3[5];
#pragma unroll
    for (int q = 0; q < 2; q++) b1[q] = w1[q * 64 + lane];
#pragma unroll
    for (int t = 0; t < TAPS; t++) b2[t] = w2[t * 64 + lane];
#pragma unroll
    for (int dx = 0; dx < 5; dx++) b3[dx] = i < 5 ? w3[(5 * i + dx) * 64 + 16 * g] : us8{0, 0, 0, 0, 0, 0, 0, 0};

    // this thread's column of input row r (wrapped or zero outside the domain)
    const int xin = threadIdx.x < SIW ? dwrap(x0 - 6 + (int)threadIdx.x, d.nx, d.perx) : -1;
    auto load_in = [&](int r) -> float {
        const int y = dwrap(r, d.ny, d.pery);
        return (xin >= 0 && y >= 0) ? in.p[vaddr(in, img, y, xin)] : 0.f;
    };
    auto put_in = [&](int r, float v) {
        if (threadIdx.x < SIW) {
            const unsigned h = hilo(v);
            sin[(r & (SIR - 1)) * SIW + threadIdx.x] = h;
            sin[((r & (SIR - 1)) + SIR) * SIW + threadIdx.x] = h;
        }
    };
    // layer 1's taps t = 16 q + 4 g + jj of this lane: offset from the first of its five input
    // rows, and whether the tap exists (t < 25; the weights of the padding are zero)
    int toff[2][4];
    bool tok[2][4];
#pragma unroll
    for (int q = 0; q < 2; q++)
#pragma unroll
        for (int jj = 0; jj < 4; jj++) {
            const int t = 16 * q + 4 * g + jj;
            tok[q][jj] = t < TAPS;
            toff[q][jj] = t < TAPS ? (t / 5) * SIW + t % 5 + i : 0;
        }
    // this lane's h1 and h2 columns lie in the domain (or x is periodic)
    const int xh1 = x0 - 4 + 16 * wave + i, xh2 = x0 - 2 + 16 * wave + i;
    const bool ok1 = d.perx || (xh1 >= 0 && xh1 < d.nx), ok2 = d.perx || (xh2 >= 0 && xh2 < d.nx);
    const int s0 = y0 - 5;
    for (int r = s0 - 1; r <= s0 + 3; r++) put_in(r, load_in(r));
    // input rows in flight ten rows ahead: at row s = s5 + u, q0[u] holds row s + 4 (staged at
    // the end of the row) and q1[u] row s + 9
    float q0[5], q1[5];
#pragma unroll
    for (int u = 0; u < 5; u++) {
        q0[u] = load_in(s0 + 4 + u);
        q1[u] = load_in(s0 + 9 + u);
    }
    __syncthreads();

    f32x4 acc[5], T = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < 5; k++) acc[k] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int nsteps = (yend - y0 + 10 + 4) / 5 * 5;
    for (int s5 = s0; s5 < s0 + nsteps; s5 += 5) {
#pragma unroll
        for (int u = 0; u < 5; u++) {
            const int s = s5 + u;
            // every LDS read of the row first: all of it was written before the last barrier,
            // and the row's writes go to ring slots the row does not read (h1 row s + 1, h2 row
            // s - 2, input row s + 4)
            const unsigned* rows = sin + ((s - 1) & (SIR - 1)) * SIW + 16 * wave;
            unsigned A1[2][4];
#pragma unroll
            for (int q = 0; q < 2; q++)
#pragma unroll
                for (int jj = 0; jj < 4; jj++) A1[q][jj] = rows[toff[q][jj]];
            const unsigned short* src2 = sh1 + (s & 1) * SH1W * 32 + (g * SH1W + 16 * wave + i) * 8;
            const unsigned short* src3 = sh2 + ((s - 3) & 1) * SH2W * 32 + (g * SH2W + 16 * wave + i) * 8;
            us8 A2[5], A3[5];
#pragma unroll
            for (int dx = 0; dx < 5; dx++) {
                A2[dx] = *reinterpret_cast<const us8*>(src2 + dx * 8);
                A3[dx] = *reinterpret_cast<const us8*>(src3 + dx * 8);
            }
            // layer 1: h1 row s + 1 from input rows s - 1 .. s + 3
            f32x4 a = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int q = 0; q < 2; q++) {
#pragma unroll
                for (int jj = 0; jj < 4; jj++) A1[q][jj] = q == 0 || tok[q][jj] ? A1[q][jj] : 0u;   // taps 0 .. 15 exist
                a = mfma(b1[q], __builtin_bit_cast(us8, A1[q]), a);
            }
            // layer 2: h1 row s into the h2 rows s - 2 .. s + 2; row s - 2 (tap row dy = 4)
            // first, so that its conversion and store overlap the other 20 MFMAs
#pragma unroll
            for (int dx = 0; dx < 5; dx++) acc[(u + 3) % 5] = mfma(b2[20 + dx], A2[dx], acc[(u + 3) % 5]);
            {
                unsigned short* h1 = sh1 + ((s + 1) & 1) * SH1W * 32;
                const int yr = s + 1;
                const bool ok = (d.pery || (yr >= 0 && yr < d.ny)) && ok1;
#pragma unroll
                for (int r = 0; r < 4; r++) a[r] = ok ? a[r] : 0.f;
                store_ch4(h1, SH1W, 16 * wave + i, g, a);
            }
#pragma unroll
            for (int dx = 0; dx < 5; dx++)
#pragma unroll
                for (int dy = 0; dy < 4; dy++) {
                    const int k = (u + 7 - dy) % 5;
                    acc[k] = mfma(b2[5 * dy + dx], A2[dx], acc[k]);
                }
            // layer 3: h2 row s - 3; output row s - 5 completes in column 4
            T = shift_columns(T);
#pragma unroll
            for (int dx = 0; dx < 5; dx++) T = mfma(A3[dx], b3[dx], T);
            {
                f32x4& c2 = acc[(u + 3) % 5];
                unsigned short* h2 = sh2 + ((s - 2) & 1) * SH2W * 32;
                const int yr = s - 2;
                const bool ok = (d.pery || (yr >= 0 && yr < d.ny)) && ok2;
#pragma unroll
                for (int r = 0; r < 4; r++) c2[r] = ok ? c2[r] : 0.f;
                store_ch4(h2, SH2W, 16 * wave + i, g, c2);
                c2 = f32x4{0.f, 0.f, 0.f, 0.f};
            }
            {
                const int y = s - 5;
                if (i == 4 && y >= y0 && y < yend) {
#pragma unroll
                    for (int r = 0; r < 4; r++) {
                        const int c = 16 * wave + 4 * g + r, x = x0 + c;
                        if (c < SOW && x < d.nx) out.p[vaddr(out, img, y, x)] = T[r];
                    }
                }
            }
            put_in(s + 4, q0[u]);
            q0[u] = q1[u];
            q1[u] = load_in(s + 14);
            __syncthreads();
        }
    }
}

// ---- host launchers ---------------------------------------------------------------------

int chunks(int cin) { return (TAPS * cin * 2 + 31) / 32; }

static void launch_packs(const PackJobs& J, hipStream_t s)
{
    int n = 0;
    for (int k = 0; k < J.n; k++) n += J.j[k].nq;
    hipLaunchKernelGGL(k_lf_pack, dim3(n), dim3(64), 0, s, J);
}

static PackJob pack_job(const float* w, int cin, int cout, bool adjoint, void* wpk)
{
    return PackJob{w, cin, cout, adjoint ? 1 : 0, chunks(adjoint ? cout : cin), reinterpret_cast<us8*>(wpk)};
}

template <int CIN, int COUT, int TX>
static void conv_tiles(const View& in, const View& out, const Domain& d, const void* wpk, hipStream_t s)
{
    const dim3 grid((d.nx + TX - 1) / TX, (d.ny + ConvTile<TX>::Y - 1) / ConvTile<TX>::Y, d.nimg);
    hipLaunchKernelGGL((k_lf_conv<CIN, COUT, TX>), grid, dim3(256), 0, s, in, out, d,
                       reinterpret_cast<const us8*>(wpk));
}

template <int CIN, int COUT>
void launch_conv(const View& in, const View& out, const Domain& d, const void* wpk, hipStream_t s)
{
    // the tile shape that covers the image with fewer tiles (all of 256 pixels)
    auto tiles = [&](int tx) { return (long)((d.nx + tx - 1) / tx) * ((d.ny + 256 / tx - 1) / (256 / tx)); };
    if (tiles(32) < tiles(64)) conv_tiles<CIN, COUT, 32>(in, out, d, wpk, s);
    else conv_tiles<CIN, COUT, 64>(in, out, d, wpk, s);
}

template void launch_conv<1, 16>(const View&, const View&, const Domain&, const void*, hipStream_t);
template void launch_conv<16, 16>(const View&, const View&, const Domain&, const void*, hipStream_t);
template void launch_conv<16, 1>(const View&, const View&, const Domain&, const void*, hipStream_t);

void launch_loss(const float* out, const float* target, float* g, const Domain& d, int margin,
                 double inv_count, double* loss, hipStream_t s)
{
    hipLaunchKernelGGL(k_lf_loss, dim3(256), dim3(256), 0, s, out, target, g, d, margin, inv_count, loss);
}

// the three-layer forward pass: in (1 channel) -> h1 (16) -> h2 (16) -> out (1 channel), kept
// in separate layers when the intermediates are needed (training)
void forward(const View& in, const View& h1, const View& h2, const View& out, const Domain& d,
             const Packed& pk, hipStream_t s)
{
    launch_conv<1, 16>(in, h1, d, pk.fwd[0], s);
    launch_conv<16, 16>(h1, h2, d, pk.fwd[1], s);
    launch_conv<16, 1>(h2, out, d, pk.fwd[2], s);
}

// the forward pass streamed in one kernel (inference), on up to three image planes at once
void forward_fused(const View* in, const View* out, const Domain* d, int nplanes, const Packed& pk, hipStream_t s)
{
    Planes P{};
    P.n = nplanes;
    int nx = 0, ny = 0, nimg = 0;
    for (int k = 0; k < nplanes; k++) {
        P.in[k] = in[k];
        P.out[k] = out[k];
        P.d[k] = d[k];
        nx = std::max(nx, d[k].nx);
        ny = std::max(ny, d[k].ny);
        nimg = std::max(nimg, d[k].nimg);
    }
    // rows per workgroup: each workgroup also walks 10 rows of reach (rounded up to 5), so take
    // the height for which (rounds of resident workgroups) x (rows walked) is least
    static int slots = 0;
    if (!slots) {
        int dev = 0, cus = 0, occ = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
            cus = 256;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, (const void*)k_lf_stream, 256, 0) != hipSuccess ||
            occ < 1)
            occ = 1;
        slots = occ * cus;
    }
    const long cols = (long)((nx + SOW - 1) / SOW) * nimg * nplanes;
    int oh = 16;
    double best = 1e300;
    for (int c = 16; c <= 512; c += 8) {
        const long wg = cols * ((ny + c - 1) / c);
        const double t = (double)((wg + slots - 1) / slots) * ((c + 14) / 5 * 5);
        if (t < best * (1.0 - 1e-9)) {
            best = t;
            oh = c;
        }
        if (c >= ny) break;
    }
    P.oh = oh;
    const dim3 grid((nx + SOW - 1) / SOW, (ny + oh - 1) / oh, nimg * nplanes);
    hipLaunchKernelGGL(k_lf_stream, grid, dim3(256), 0, s, P, reinterpret_cast<const us8*>(pk.fwd[0]),
                       reinterpret_cast<const us8*>(pk.fwd[1]), reinterpret_cast<const us8*>(pk.fwd[2]));
}

void pack_forward(const float* params, const Packed& pk, hipStream_t s)
{
    PackJobs J{};
    J.n = 3;
    J.j[0] = pack_job(params + OFF_W1, 1, C, false, pk.fwd[0]);
    J.j[1] = pack_job(params + OFF_W2, C, C, false, pk.fwd[1]);
    J.j[2] = pack_job(params + OFF_W3, C, 1, false, pk.fwd[2]);
    launch_packs(J, s);
}

void pack_training(const float* params, const Packed& pk, double* clear, hipStream_t s)
{
    PackJobs J{};
    J.n = 5;
    J.j[0] = pack_job(params + OFF_W1, 1, C, false, pk.fwd[0]);
    J.j[1] = pack_job(params + OFF_W2, C, C, false, pk.fwd[1]);
    J.j[2] = pack_job(params + OFF_W3, C, 1, false, pk.fwd[2]);
    J.j[3] = pack_job(params + OFF_W2, C, C, true, pk.adj[1]);
    J.j[4] = pack_job(params + OFF_W3, C, 1, true, pk.adj[2]);
    J.clear = clear;
    launch_packs(J, s);
}

// one training pass's backward part (data and weights) and the parameter update.  The layers'
// gradient shares go where nothing is read any more: W3's over out, W2's over h2, W1's over h1;
// a layer whose room is less than one share (a few hundred pixels in all) has one workgroup,
// which writes to dw.
void backward(const View& in, const View& h1, const View& h2, const View& out, const View& gout,
              const View& gh1, const View& gh2, const Domain& d, const Packed& pk, float* dw,
              const double* loss, double* loss_out, float* grad_out, const AdamStep& st, hipStream_t s)
{
    WTiles wt;
    wt.nx = (d.nx + WTX - 1) / WTX;
    wt.ny = (d.ny + WTY - 1) / WTY;
    wt.total = wt.nx * wt.ny * d.nimg;
    const long px = (long)d.nimg * d.ny * d.nx;
    Shares S;
    auto shares = [&](int l, float* room, long room_floats, int size, int first) {
        // a workgroup per CU: more only makes more shares to write and add
        const long n = std::min<long>(std::min<long>(256, wt.total), room_floats / size);
        S.n[l] = (int)std::max<long>(n, 1);
        S.p[l] = n >= 1 ? room : dw + first;
        return const_cast<float*>(S.p[l]);
    };
    float* p3 = shares(2, out.p, px, TAPS * C, OFF_W3);
    hipLaunchKernelGGL(k_lf_wgrad_narrow, dim3(S.n[2]), dim3(256), 0, s, gout, h2, d, wt, 1, p3);
    launch_conv<1, 16>(gout, gh2, d, pk.adj[2], s);
    float* p2 = shares(1, h2.p, px * C, TAPS * C * C, OFF_W2);
    hipLaunchKernelGGL(k_lf_wgrad_wide, dim3(S.n[1]), dim3(256), 0, s, h1, gh2, d, wt, p2);
    launch_conv<16, 16>(gh2, gh1, d, pk.adj[1], s);
    float* p1 = shares(0, h1.p, px * C, TAPS * C, OFF_W1);
    hipLaunchKernelGGL(k_lf_wgrad_narrow, dim3(S.n[0]), dim3(256), 0, s, in, gh1, d, wt, 0, p1);
    const AdamArgs A{st.w, st.m, st.v, st.lr, st.b1, st.b2, st.eps, st.c1, st.c2, st.w ? 1 : 0};
    hipLaunchKernelGGL(k_lf_finish, dim3(NPARAM / 32), dim3(256), 0, s, S, A, loss, loss_out, grad_out);
}

}  // namespace lf
}  // namespace bf

// ======================================================================================
// C ABI: standalone learned filter (batched inference and training on device images)
// ======================================================================================

#include <algorithm>
#include <cmath>
#include <vector>
#include "../../include/bfpic.h"

namespace {

using namespace bf::lf;

size_t up256(size_t v) { return (v + 255) / 256 * 256; }

// sub-allocation of the caller's work buffer for nimg images of ny x nx
struct LfWork {
    size_t packed[5], h1, h2, gh1, gh2, out, gout, dw, loss, bytes;
};

LfWork lf_work(int nimg, int ny, int nx)
{
    LfWork w;
    size_t o = 0;
    auto take = [&](size_t b) { size_t r = o; o = up256(o + b); return r; };
    const int nq[5] = {chunks(1), chunks(C), chunks(C), chunks(C), chunks(1)};
    for (int k = 0; k < 5; k++) w.packed[k] = take((size_t)nq[k] * CHUNK_BYTES);
    const size_t px = (size_t)nimg * ny * nx;
    w.h1 = take(px * C * 4);
    w.h2 = take(px * C * 4);
    w.gh1 = take(px * C * 4);
    w.gh2 = take(px * C * 4);
    w.out = take(px * 4);
    w.gout = take(px * 4);
    w.dw = take((size_t)NPARAM * 4);
    w.loss = take(2 * sizeof(double));
    w.bytes = o;
    return w;
}

Packed packed_of(unsigned char* base, const LfWork& w)
{
    Packed p;
    p.fwd[0] = base + w.packed[0];
    p.fwd[1] = base + w.packed[1];
    p.fwd[2] = base + w.packed[2];
    p.adj[0] = nullptr;
    p.adj[1] = base + w.packed[3];
    p.adj[2] = base + w.packed[4];
    return p;
}

View image_view(const float* p, int ny, int nx, int ch)
{
    View v;
    v.p = const_cast<float*>(p);
    v.rstride = (long)nx * ch;
    v.istride = (long)ny * nx * ch;
    v.ch = ch;
    v.zoff = 0;
    v.rows = ny;
    return v;
}

bool dims_ok(int nimg, int ny, int nx)
{
    return nimg > 0 && ny > 0 && nx > 0 && nimg <= 65535 && (long)nimg * ny * nx <= (1L << 31) / C;
}

// exact learned-filter form of the n-pass bilinear filter + compensation (Sec. 4.1): per axis
// the composed 1D stencil ((1 + z) / 2)^(2n) (times the compensation pass) is cut into three
// factors of at most five taps; each layer carries the outer product of its factor with itself
// in channel 0
bool bilinear_params(int npass, int comp, float* out)
{
    const int room[3] = {4, 4, comp ? 2 : 4};
    int left = 2 * npass;
    std::vector<double> st[3];
    for (int l = 0; l < 3; l++) {
        const int k = std::min(room[l], left);
        left -= k;
        std::vector<double> f{1.0};
        for (int r = 0; r < k; r++) {                   // convolve with (1/2, 1/2)
            std::vector<double> g(f.size() + 1, 0.0);
            for (size_t i = 0; i < f.size(); i++) {
                g[i] += 0.5 * f[i];
                g[i + 1] += 0.5 * f[i];
            }
            f.swap(g);
        }
        st[l] = f;
    }
    if (left > 0) return false;
    if (comp) {                                         // (1 - a)/2, a, (1 - a)/2 with a = n/2 + 1
        const double a = 0.5 * npass + 1.0;
        const double c3[3] = {0.5 * (1.0 - a), a, 0.5 * (1.0 - a)};
        std::vector<double> g(st[2].size() + 2, 0.0);
        for (size_t i = 0; i < st[2].size(); i++)
            for (int j = 0; j < 3; j++) g[i + j] += st[2][i] * c3[j];
        st[2].swap(g);
    }
    for (int i = 0; i < NPARAM; i++) out[i] = 0.f;
    const int off[3] = {OFF_W1, OFF_W2, OFF_W3}, cc[3] = {C, C * C, C};   // (t, ci, co) strides
    for (int l = 0; l < 3; l++) {
        double s5[5] = {0, 0, 0, 0, 0};
        const int n = (int)st[l].size(), o = (5 - n) / 2;
        for (int i = 0; i < n; i++) s5[o + i] = st[l][i];
        for (int a = 0; a < 5; a++)
            for (int b = 0; b < 5; b++) out[off[l] + (5 * a + b) * cc[l]] = (float)(s5[a] * s5[b]);
    }
    return true;
}

}  // namespace

extern "C" {

bf_status bf_lf_bilinear_params(int npass, int compensate, float* host_params, int64_t n)
{
    if (!host_params || n != NPARAM || npass < 0) return BF_EINVAL;
    return bilinear_params(npass, compensate ? 1 : 0, host_params) ? BF_OK : BF_EINVAL;
}

int64_t bf_lf_work_bytes(int nimg, int ny, int nx)
{
    if (!dims_ok(nimg, ny, nx)) return -1;
    return (int64_t)lf_work(nimg, ny, nx).bytes;
}

bf_status bf_lf_apply(void* work, int64_t work_bytes, const float* params, const float* in, float* out,
                      int nimg, int ny, int nx, int periodic_x, int periodic_y, void* hip_stream)
{
    if (!work || !params || !in || !out || !dims_ok(nimg, ny, nx)) return BF_EINVAL;
    const LfWork w = lf_work(nimg, ny, nx);
    if (work_bytes < (int64_t)w.bytes) return BF_EINVAL;
    hipStream_t s = reinterpret_cast<hipStream_t>(hip_stream);
    unsigned char* b = static_cast<unsigned char*>(work);
    const Packed pk = packed_of(b, w);
    const Domain d{nimg, ny, nx, periodic_x ? 1 : 0, periodic_y ? 1 : 0};
    (void)hipGetLastError();
    pack_forward(params, pk, s);
    const View vin = image_view(in, ny, nx, 1), vout = image_view(out, ny, nx, 1);
    forward_fused(&vin, &vout, &d, 1, pk, s);
    return hipGetLastError() == hipSuccess ? BF_OK : BF_EDEVICE;
}

bf_status bf_lf_train_step(void* work, int64_t work_bytes, float* params, float* adam_m, float* adam_v,
                           const float* in, const float* target, int nimg, int ny, int nx, int margin,
                           int periodic_x, int periodic_y, float lr, float beta1, float beta2, float eps,
                           int64_t step, float* grad_out, double* loss_out, void* hip_stream)
{
    if (!work || !params || !in || !target || !dims_ok(nimg, ny, nx)) return BF_EINVAL;
    if (margin < 0 || 2 * margin >= ny || 2 * margin >= nx) return BF_EINVAL;
    if (lr != 0.f && (!adam_m || !adam_v || step < 1)) return BF_EINVAL;
    const LfWork w = lf_work(nimg, ny, nx);
    if (work_bytes < (int64_t)w.bytes) return BF_EINVAL;
    hipStream_t s = reinterpret_cast<hipStream_t>(hip_stream);
    unsigned char* b = static_cast<unsigned char*>(work);
    const Packed pk = packed_of(b, w);
    const Domain d{nimg, ny, nx, periodic_x ? 1 : 0, periodic_y ? 1 : 0};
    float* dw = reinterpret_cast<float*>(b + w.dw);
    double* loss = reinterpret_cast<double*>(b + w.loss);
    const View vin = image_view(in, ny, nx, 1);
    const View h1 = image_view(reinterpret_cast<float*>(b + w.h1), ny, nx, C);
    const View h2 = image_view(reinterpret_cast<float*>(b + w.h2), ny, nx, C);
    const View gh1 = image_view(reinterpret_cast<float*>(b + w.gh1), ny, nx, C);
    const View gh2 = image_view(reinterpret_cast<float*>(b + w.gh2), ny, nx, C);
    const View vout = image_view(reinterpret_cast<float*>(b + w.out), ny, nx, 1);
    const View gout = image_view(reinterpret_cast<float*>(b + w.gout), ny, nx, 1);
    (void)hipGetLastError();
    pack_training(params, pk, loss, s);
    forward(vin, h1, h2, vout, d, pk, s);
    const double count = (double)nimg * (ny - 2 * margin) * (nx - 2 * margin);
    launch_loss(vout.p, target, gout.p, d, margin, 1.0 / count, loss, s);
    AdamStep st{};
    if (lr != 0.f) {
        st.w = params;
        st.m = adam_m;
        st.v = adam_v;
        st.lr = lr;
        st.b1 = beta1;
        st.b2 = beta2;
        st.eps = eps;
        st.c1 = (float)(1.0 / (1.0 - std::pow((double)beta1, (double)step)));
        st.c2 = (float)(1.0 / (1.0 - std::pow((double)beta2, (double)step)));
    }
    backward(vin, h1, h2, vout, gout, gh1, gh2, d, pk, dw, loss, loss_out, grad_out, st, s);
    return hipGetLastError() == hipSuccess ? BF_OK : BF_EDEVICE;
}

}  // extern "C"

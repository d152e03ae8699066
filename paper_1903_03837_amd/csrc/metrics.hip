// metrics.hip -- image similarity of light-field views against ground-truth
// views: mean SSIM (Wang, Bovik, Sheikh, Simoncelli 2004, the index the
// paper reports) with the 11 x 11 Gaussian window of sigma 1.5, over the
// positions where the window lies inside the image, per colour channel, then
// averaged over the channels.
//
// One workgroup computes 16 x 16 window positions of one channel: the 26 x 26
// input tiles of both images go to LDS, a horizontal pass forms the five
// windowed moments (means, second moments, cross moment) for 26 rows, a
// vertical pass finishes them, and each thread evaluates its SSIM term.  The
// workgroup sum (FP64) goes to its own slot; a second kernel adds the slots
// of each image in a fixed order, so the result is the same on every run.
#include <algorithm>

#include "internal.hpp"

namespace lp {

constexpr int kWin = 11, kHalo = kWin - 1, kTile = 16, kIn = kTile + kHalo;

__global__ __launch_bounds__(256) void ssim_tile_kernel(SsimParams P) {
    __shared__ float A[kIn][kIn + 1], B[kIn][kIn + 1];
    __shared__ float Hm[5][kIn][kTile + 1];
    __shared__ double red[256];
    const int Wv = P.W - kHalo, Hv = P.H - kHalo;
    const int x0 = blockIdx.x * kTile, y0 = blockIdx.y * kTile;
    const int img = blockIdx.z / 3, ch = blockIdx.z % 3;
    const float* a = P.a + (size_t)img * P.H * P.W * 3;
    const float* b = P.b + (size_t)img * P.H * P.W * 3;
    for (int e = threadIdx.x; e < kIn * kIn; e += 256) {
        const int ty = e / kIn, tx = e - ty * kIn;
        const int x = x0 + tx, y = y0 + ty;
        float va = 0.0f, vb = 0.0f;
        if (x < P.W && y < P.H) {
            const size_t o = ((size_t)y * P.W + x) * 3 + ch;
            va = a[o];
            vb = b[o];
        }
        A[ty][tx] = va;
        B[ty][tx] = vb;
    }
    __syncthreads();
    // horizontal pass: 26 rows x 16 columns of the five moments
    for (int e = threadIdx.x; e < kIn * kTile; e += 256) {
        const int ty = e / kTile, tx = e - ty * kTile;
        float ma = 0.0f, mb = 0.0f, aa = 0.0f, bb = 0.0f, ab = 0.0f;
#pragma unroll
        for (int t = 0; t < kWin; ++t) {
            const float w = P.w[t], va = A[ty][tx + t], vb = B[ty][tx + t];
            ma = fmaf(w, va, ma);
            mb = fmaf(w, vb, mb);
            aa = fmaf(w, va * va, aa);
            bb = fmaf(w, vb * vb, bb);
            ab = fmaf(w, va * vb, ab);
        }
        Hm[0][ty][tx] = ma;
        Hm[1][ty][tx] = mb;
        Hm[2][ty][tx] = aa;
        Hm[3][ty][tx] = bb;
        Hm[4][ty][tx] = ab;
    }
    __syncthreads();
    // vertical pass and the SSIM term of this thread's window position
    const int tx = threadIdx.x & (kTile - 1), ty = threadIdx.x / kTile;
    double term = 0.0;
    if (x0 + tx < Wv && y0 + ty < Hv) {
        float m[5] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int t = 0; t < kWin; ++t) {
            const float w = P.w[t];
#pragma unroll
            for (int q = 0; q < 5; ++q) m[q] = fmaf(w, Hm[q][ty + t][tx], m[q]);
        }
        const float va = m[2] - m[0] * m[0], vb = m[3] - m[1] * m[1], cab = m[4] - m[0] * m[1];
        const float num = (2.0f * m[0] * m[1] + P.c1) * (2.0f * cab + P.c2);
        const float den = (m[0] * m[0] + m[1] * m[1] + P.c1) * (va + vb + P.c2);
        term = (double)(num / den);
    }
    red[threadIdx.x] = term;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const size_t slot = ((size_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
        P.partial[slot] = red[0];
    }
}

// Mean SSIM of each image: its 3 * tiles slots in order, over 3 Wv Hv terms.
__global__ void ssim_reduce_kernel(SsimParams P, int slots_per_image) {
    const int img = blockIdx.x;
    __shared__ double red[256];
    double s = 0.0;
    for (int e = threadIdx.x; e < slots_per_image; e += 256) s += P.partial[(size_t)img * slots_per_image + e];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) P.out[img] = red[0] / (3.0 * (double)(P.W - kHalo) * (double)(P.H - kHalo));
}

hipError_t launch_ssim(const SsimParams& P, int n_images, hipStream_t s) {
    const int Wv = P.W - kHalo, Hv = P.H - kHalo;
    dim3 grid((Wv + kTile - 1) / kTile, (Hv + kTile - 1) / kTile, 3 * n_images);
    ssim_tile_kernel<<<grid, 256, 0, s>>>(P);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    ssim_reduce_kernel<<<n_images, 256, 0, s>>>(P, (int)(3 * grid.x * grid.y));
    return hipGetLastError();
}

size_t ssim_partial_count(int n_images, int W, int H) {
    const size_t gx = (size_t)(W - kHalo + kTile - 1) / kTile, gy = (size_t)(H - kHalo + kTile - 1) / kTile;
    return gx * gy * 3 * (size_t)n_images;
}

// ---------------------------------------------------------------------------
// CW-SSIM (Wang & Simoncelli 2005, Sampat et al. 2009; the second index the
// paper reports): complex subbands of a steerable filter bank defined in the
// DFT domain, 2 scales x 4 orientations (the eight levels the paper names),
// and the local index
//     S = (2 |sum c_x conj(c_y)| + K) / (sum |c_x|^2 + sum |c_y|^2 + K)
// over 7 x 7 windows inside the image, averaged over positions, subbands and
// channels.  Filter of scale s, orientation k at DFT index (u, v): signed
// frequencies f = u (2u < n) or u - n, w = 2 pi f / n, r = |w|, theta =
// atan2(w_y, w_x); R_s = cos(pi/2 log2(r / r_s)) for |log2(r / r_s)| < 1,
// r_s = pi / 2^(s+1); A_k = cos(d)^3 for |d| < pi/2, d = theta - pi k / 4
// wrapped to (-pi, pi].
//
// Per image, the six planes (two images x three channels) go through a
// direct separable DFT (rows, then columns; twiddle index (u x) mod n, so no
// phase rounding grows with the index), then per subband: the filter (with
// the 1 / (W H) of the inverse), inverse columns with the filter applied as
// they load, inverse rows, and the windowed index of 16 x 16 positions per
// workgroup from LDS tiles.  Workgroup sums (FP64) go to slots that are added
// in a fixed order.

constexpr int kCwScales = 2, kCwOrients = 4, kCwBands = kCwScales * kCwOrients;
constexpr int kCwWin = 7, kCwHalo = kCwWin - 1, kCwTile = 16, kCwIn = kCwTile + kCwHalo;

__global__ void cw_twiddle_kernel(int n, float2* tw) {
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= n) return;
    double sn, cs;
    sincospi(2.0 * (double)m / (double)n, &sn, &cs);
    tw[m] = make_float2((float)cs, (float)sn);
}

// ---------------------------------------------------------------------------
// The DFT passes as matrix products on MFMA.  A pass multiplies lines of n
// complex inputs by the n x n twiddle matrix; in real terms each input is the
// pair of rows (im, re) and each output the pair of columns (re, im) of
//     [ -ws  wx ]
//     [  wx  ws ],   ws = +- sin, wx = cos of 2 pi (u x mod n) / n,
// and v_mfma_f32_32x32x2_f32 adds one input's two products to 32 x 32 sums.
// The instruction forms each sum as a chain of fused multiply-adds in the
// order of k (checked bit for bit against fmaf chains, denormals included), so
// an output is the same chain over x, im term first, that one lane per output
// would run, with the same bits.
//
// What bounds it: the FP32 matrix rate (156 TFLOP/s measured), of which a pass
// reaches 50-70 %, where one lane per output was bound by two reads per four
// multiply-adds.  Terms that are zero are left out, since adding them changes
// nothing: imaginary parts of the image (forward rows take two inputs per
// instruction), columns on which a subband's filter vanishes (inverse rows
// skip them, inverse columns do not form them) and runs of rows of a column
// where it does.  A 1920 x 1080 pair 120.5 -> 14.1 ms (inverse rows 6.97 ->
// 0.43-1.82 ms per subband, inverse columns 6.42 -> 0.18-0.67 ms), four 480 x
// 270 pairs 9.6 -> 2.8 ms, 1279 x 719 35.6 -> 5.0 ms.  (A mixed-radix
// transform takes 1.9 ms per 1920 x 1080 pair, but its smaller rounding errors
// move the index by 1e-8.)
//
// A wave holds (32 T) lines x (16 T) outputs, a workgroup 2 x 2 waves; 16
// steps of inputs at a time go to LDS as [step][im, re][line], the next ones
// in flight meanwhile, and the twiddles are read from an LDS copy of the table
// at an index that each lane advances by u per step.
// ---------------------------------------------------------------------------
typedef float v16f __attribute__((ext_vector_type(16)));
constexpr int kDftStep = 16;  // steps (complex inputs, or pairs of real ones) per LDS chunk

// The columns on which a subband's filter can be nonzero: u < pos or u >= neg.
struct CwColumns {
    int pos, neg;
};

// False only if F_sk is zero on all columns [u0, u1) x rows [v0, v1) of the
// DFT grid: by the extremes of |w| and of w along the orientation over the
// block, with a margin far above rounding.  Blocks that hold the jump of the
// signed frequency count as nonzero.
__device__ __forceinline__ bool cw_band_reaches(int W, int H, int sc, int k, int u0, int u1, int v0, int v1) {
    if ((2 * u0 < W && 2 * (u1 - 1) >= W) || (2 * v0 < H && 2 * (v1 - 1) >= H)) return true;
    const float tau = 6.2831853f;
    const float xa = tau * (float)(2 * u0 < W ? u0 : u0 - W) / (float)W, xb = xa + tau * (float)(u1 - 1 - u0) / (float)W;
    const float ya = tau * (float)(2 * v0 < H ? v0 : v0 - H) / (float)H, yb = ya + tau * (float)(v1 - 1 - v0) / (float)H;
    const float ax = fmaxf(fabsf(xa), fabsf(xb)), ay = fmaxf(fabsf(ya), fabsf(yb));
    const float ix = fmaxf(0.0f, fmaxf(xa, -xb)), iy = fmaxf(0.0f, fmaxf(ya, -yb));
    const float rs = 3.14159265f / (float)(2 << sc), eps = 1e-3f;
    const float far2 = ax * ax + ay * ay, near2 = ix * ix + iy * iy;
    const float along = k == 0 ? xb : k == 1 ? xb + yb : k == 2 ? yb : yb - xa;
    return far2 > (0.5f * rs - eps) * (0.5f * rs - eps) && near2 < (2.0f * rs + eps) * (2.0f * rs + eps) && along > -eps;
}

// One pass.  COLS false: rows, lines (p, y) in flattened order, out[line][u] =
// sum_x in[line][x] w(u x).  COLS true: columns of plane blockIdx.z, out[v][x]
// = sum_y in[y][x] w(v y).  IMAGE: the inputs are the real channels of images
// a (planes 0..2) and b (rows only).  FILTER: inputs are multiplied by g
// (columns only).  cols: the columns u that hold inputs (rows) or are formed
// (columns).  band: scale * 4 + orientation, for FILTER.
template <bool COLS, bool INV, bool IMAGE, bool FILTER, int T>
__global__ __launch_bounds__(256, 2) void cw_dft_kernel(const float* a, const float* b, const float2* in,
                                                        const float* g, float2* out, const float2* tw_g, int W, int H,
                                                        CwColumns cols, int band) {
    constexpr int LINES = 64 * T, OUTS = 32 * T;  // of the workgroup
    constexpr int PER = LINES * kDftStep / 256;   // complex inputs (pairs, IMAGE) a thread loads per chunk
    extern __shared__ float cw_lds[];
    float* data = cw_lds;                                     // [2][kDftStep][2][LINES]
    float* tw = cw_lds + 2 * kDftStep * 2 * LINES;            // [n][2]
    const int n = COLS ? H : W;
    for (int i = threadIdx.x; i < 2 * n; i += 256) tw[i] = ((const float*)tw_g)[i];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, j = lane & 31, q = lane >> 5;
    const int wl = wave & 1, wo = wave >> 1;

    // lines of this workgroup: columns u0 .. u_end (COLS) or flattened rows
    const int pos_tiles = (cols.pos + LINES - 1) / LINES;
    const int tile = blockIdx.y;
    const int u0 = COLS ? (tile < pos_tiles ? tile * LINES : cols.neg + (tile - pos_tiles) * LINES) : 0;
    const int u_end = COLS ? min(u0 + LINES, tile < pos_tiles ? cols.pos : W) : 0;
    const int line0 = tile * LINES, line_end = 6 * H;
    const float2* src = COLS ? in + (size_t)blockIdx.z * H * W : in;

    // input chunks: step kDftStep (IMAGE: twice as many real inputs)
    constexpr int SPAN = IMAGE ? 2 * kDftStep : kDftStep;
    const int chunks1 = COLS ? (H + SPAN - 1) / SPAN : (cols.pos + SPAN - 1) / SPAN;
    const int chunks = COLS ? chunks1 : chunks1 + (W - cols.neg + SPAN - 1) / SPAN;
    auto start = [&](int c) { return c < chunks1 ? c * SPAN : cols.neg + (c - chunks1) * SPAN; };
    auto limit = [&](int c) { return COLS ? H : (c < chunks1 ? cols.pos : W); };
    auto next = [&](int c) {  // the next chunk that can hold a nonzero input
        if constexpr (FILTER)
            while (c < chunks && !cw_band_reaches(W, H, band / kCwOrients, band % kCwOrients, u0, u_end, c * SPAN,
                                                  min(H, (c + 1) * SPAN)))
                ++c;
        return c;
    };

    // Addresses are 32-bit byte offsets from a uniform base (a plane set is at
    // most 6 x 2^24 x 8 bytes); chunks that lie whole inside the inputs load
    // without bounds tests (these and the address arithmetic took a seventh of
    // the pass).
    float2 reg[PER];
    const int fl = COLS ? (int)threadIdx.x % LINES : (int)threadIdx.x / (kDftStep / PER);      // line of this thread
    const int fk = COLS ? (int)threadIdx.x / LINES : (int)threadIdx.x % (kDftStep / PER) * PER;  // its first step
    const bool whole_lines = COLS ? u0 + LINES <= u_end : line0 + LINES <= line_end;
    const float* image = a;
    uint32_t at0;  // byte offset of this thread's line
    if constexpr (COLS) {
        at0 = 8u * (uint32_t)min(u0 + fl, W - 1);
    } else {
        const int line = min(line0 + fl, line_end - 1);
        if constexpr (IMAGE) {
            const int p = line / H, y = line - p * H;
            image = p < 3 ? a : b;
            at0 = 4u * ((uint32_t)y * (uint32_t)W * 3u + (uint32_t)(p % 3));
        } else {
            at0 = 8u * (uint32_t)line * (uint32_t)W;
        }
    }
    auto fetch = [&](int c) {
        const int x0 = start(c), xe = limit(c);
        auto load = [&](bool whole) {
            const bool in_line = whole || (COLS ? u0 + fl < u_end : line0 + fl < line_end);
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                float2 z = make_float2(0.0f, 0.0f);
                if constexpr (COLS) {
                    const int y = x0 + fk + i * (256 / LINES);
                    if (whole || (in_line && y < xe)) {
                        const uint32_t at = at0 + 8u * (uint32_t)y * (uint32_t)W;
                        z = *(const float2*)((const char*)src + at);
                        if constexpr (FILTER) {
                            const float f = *(const float*)((const char*)g + at / 2);
                            z = make_float2(z.x * f, z.y * f);
                        }
                    }
                } else if constexpr (IMAGE) {
                    const int x = x0 + 2 * (fk + i);
                    const float* r = (const float*)((const char*)image + at0) + 3 * x;
                    if (whole || (in_line && x < xe)) z.y = r[0];  // the pair's first term
                    if (whole || (in_line && x + 1 < xe)) z.x = r[3];
                } else {
                    const int x = x0 + fk + i;
                    if (whole || (in_line && x < xe)) z = *(const float2*)((const char*)src + (at0 + 8u * (uint32_t)x));
                }
                reg[i] = z;
            }
        };
        if (whole_lines && x0 + SPAN <= xe) load(true);  // (uniform)
        else load(false);
    };
    auto stage = [&](int buf) {
        float* d = data + buf * (kDftStep * 2 * LINES) + fl;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int k = COLS ? fk + i * (256 / LINES) : fk + i;
            d[(2 * k) * LINES] = reg[i].y;
            d[(2 * k + 1) * LINES] = reg[i].x;
        }
    };

    // twiddle operand of this lane: output o[t], part j & 1, row q of the 2 x 2 block
    const int part = j & 1;
    const bool sine = IMAGE ? part == 1 : q == part;
    const uint32_t flip = sine && ((IMAGE || q == 1) ? !INV : INV) ? 0x80000000u : 0u;
    int o[T], o2[T], idx[T];  // o2: the index's advance per step, below n
    const int o_base = blockIdx.x * OUTS + wo * 16 * T;
#pragma unroll
    for (int t = 0; t < T; ++t) {
        o[t] = o_base + t * 16 + (j >> 1);
        if (o[t] >= n) o[t] = 0;  // (not stored)
        if constexpr (IMAGE) o2[t] = 2 * o[t] >= n ? 2 * o[t] - n : 2 * o[t];
        else o2[t] = o[t];
    }
    v16f acc[T][T] = {};
    int c = next(0), at = -1, buf = 0;
    if (c < chunks) {
        fetch(c);
        stage(0);
    }
    __syncthreads();
    while (c < chunks) {
        const int after = next(c + 1);
        if (after < chunks) fetch(after);
        const int x0 = start(c);
        if (x0 != at) {  // (otherwise the indices stand at this chunk's first input)
#pragma unroll
            for (int t = 0; t < T; ++t) idx[t] = (int)(((uint32_t)o[t] * (uint32_t)(x0 + (IMAGE ? q : 0))) % (uint32_t)n);
        }
        at = x0 + SPAN;
        const float* d = data + buf * (kDftStep * 2 * LINES) + q * LINES + wl * 32 * T + j;
        // operands of a step are read while the step before it runs
        float w[2][T], z[2][T];
        auto operands = [&](int k) {
#pragma unroll
            for (int t = 0; t < T; ++t) {
                w[k & 1][t] = tw[2 * idx[t] + (sine ? 1 : 0)];
                z[k & 1][t] = d[2 * k * LINES + 32 * t];
                // the next input's (IMAGE: the one after next) index, below n
                idx[t] += o2[t];
                idx[t] = (int)min((uint32_t)idx[t], (uint32_t)(idx[t] - n));
            }
        };
        operands(0);
#pragma unroll
        for (int k = 0; k < kDftStep; ++k) {
            if (k + 1 < kDftStep) operands(k + 1);
            __builtin_amdgcn_sched_barrier(0);
            float wk[T];
#pragma unroll
            for (int t = 0; t < T; ++t) wk[t] = __uint_as_float(__float_as_uint(w[k & 1][t]) ^ flip);
#pragma unroll
            for (int l = 0; l < T; ++l)
#pragma unroll
                for (int t = 0; t < T; ++t)
                    acc[l][t] = COLS ? __builtin_amdgcn_mfma_f32_32x32x2f32(wk[t], z[k & 1][l], acc[l][t], 0, 0, 0)
                                     : __builtin_amdgcn_mfma_f32_32x32x2f32(z[k & 1][l], wk[t], acc[l][t], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (after < chunks) stage(buf ^ 1);
        __syncthreads();
        buf ^= 1;
        c = after;
    }

    // D[i][j] in lane j + 32 ((i / 4) % 2), register 4 (i / 8) + i % 4
#pragma unroll
    for (int l = 0; l < T; ++l)
#pragma unroll
        for (int t = 0; t < T; ++t) {
            if constexpr (COLS) {  // rows: outputs (re, im); columns: lines
                const int u = u0 + wl * 32 * T + 32 * l + j;
                float2* dst = out + (size_t)blockIdx.z * H * W + u;
#pragma unroll
                for (int r = 0; r < 16; r += 2) {
                    const int v = o_base + t * 16 + (8 * (r >> 2) + 4 * q + (r & 3)) / 2;
                    if (u < u_end && v < H) dst[(size_t)v * W] = make_float2(acc[l][t][r], acc[l][t][r + 1]);
                }
            } else {  // rows: lines; columns: outputs (re, im)
                const int u = o_base + t * 16 + (j >> 1);
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int line = line0 + wl * 32 * T + 32 * l + 8 * (r >> 2) + 4 * q + (r & 3);
                    if (line < line_end && u < W) ((float*)out)[((size_t)line * W + u) * 2 + part] = acc[l][t][r];
                }
            }
        }
}

// g[v][u] = F_sk / (W H), evaluated in FP64 and rounded once.  The angular
// window needs no angle: cos(theta - pi k / 4) = (w_x cos + w_y sin)(pi k / 4) / r,
// and it is positive exactly where the wrapped difference is below pi / 2.
__global__ void cw_filter_kernel(float* g, int W, int H, int s, int k) {
    const int u = blockIdx.x * blockDim.x + threadIdx.x, v = blockIdx.y;
    if (u >= W) return;
    const double pi = 3.141592653589793, h = 0.70710678118654752;
    const double fu = 2 * u < W ? u : u - W, fv = 2 * v < H ? v : v - H;
    const double wx = 2.0 * pi * fu / W, wy = 2.0 * pi * fv / H;
    const double r2 = wx * wx + wy * wy;
    const double along = k == 0 ? wx : k == 1 ? h * (wx + wy) : k == 2 ? wy : h * (wy - wx);
    float f = 0.0f;
    if (r2 > 0.0 && along > 0.0) {
        const double r = sqrt(r2), lr = log2(r / (pi / (double)(2 << s)));
        if (fabs(lr) < 1.0) {
            const double c = along / r;
            f = (float)(cospi(0.5 * lr) * c * c * c / ((double)W * (double)H));
        }
    }
    g[(size_t)v * W + u] = f;
}

// windowed index of 16 x 16 positions of channel blockIdx.z of one subband;
// the workgroup's FP64 sum goes to slots[(ch * gy + by) * gx + bx]
__global__ __launch_bounds__(256) void cw_map_kernel(const float2* coef, int W, int H, float K, double* slots) {
    __shared__ float Q[4][kCwIn][kCwIn + 1];     // re, im of c_x conj(c_y), |c_x|^2, |c_y|^2
    __shared__ float Hs[4][kCwIn][kCwTile + 1];  // horizontal 7-sums
    __shared__ double red[256];
    const int Wv = W - kCwHalo, Hv = H - kCwHalo;
    const int x0 = blockIdx.x * kCwTile, y0 = blockIdx.y * kCwTile, ch = blockIdx.z;
    const size_t n = (size_t)W * H;
    const float2* cx = coef + ch * n;
    const float2* cy = coef + (3 + ch) * n;
    for (int e = threadIdx.x; e < kCwIn * kCwIn; e += 256) {
        const int ty = e / kCwIn, tx = e - ty * kCwIn;
        const int x = x0 + tx, y = y0 + ty;
        float2 a = make_float2(0.0f, 0.0f), b = a;
        if (x < W && y < H) {
            a = cx[(size_t)y * W + x];
            b = cy[(size_t)y * W + x];
        }
        Q[0][ty][tx] = a.x * b.x + a.y * b.y;
        Q[1][ty][tx] = a.y * b.x - a.x * b.y;
        Q[2][ty][tx] = a.x * a.x + a.y * a.y;
        Q[3][ty][tx] = b.x * b.x + b.y * b.y;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < kCwIn * kCwTile; e += 256) {
        const int ty = e / kCwTile, tx = e - ty * kCwTile;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float sum = 0.0f;
#pragma unroll
            for (int d = 0; d < kCwWin; ++d) sum += Q[q][ty][tx + d];
            Hs[q][ty][tx] = sum;
        }
    }
    __syncthreads();
    const int tx = threadIdx.x % kCwTile, ty = threadIdx.x / kCwTile;
    double term = 0.0;
    if (x0 + tx < Wv && y0 + ty < Hv) {
        float q[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            float sum = 0.0f;
#pragma unroll
            for (int d = 0; d < kCwWin; ++d) sum += Hs[c][ty + d][tx];
            q[c] = sum;
        }
        const float num = 2.0f * sqrtf(q[0] * q[0] + q[1] * q[1]) + K;
        const float den = q[2] + q[3] + K;
        term = den > 0.0f ? (double)(num / den) : 1.0;
    }
    red[threadIdx.x] = term;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) slots[((size_t)ch * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x] = red[0];
}

// out[b] = scale * sum of block b's run of the slots, in a fixed order (a
// first launch over kCwRuns runs, then one workgroup over their sums: one
// workgroup over all slots of a 1920 x 1080 pair waited 280 us on its loads).
constexpr int kCwRuns = 256;
__global__ __launch_bounds__(256) void cw_reduce_kernel(const double* slots, int nslots, double scale, double* out) {
    __shared__ double red[256];
    const int run = (nslots + (int)gridDim.x - 1) / (int)gridDim.x, lo = blockIdx.x * run, hi = min(nslots, lo + run);
    double s = 0.0;
    for (int e = lo + (int)threadIdx.x; e < hi; e += 256) s += slots[e];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[blockIdx.x] = red[0] * scale;
}

size_t cw_ssim_slots(int W, int H) {
    const size_t gx = (size_t)(W - kCwHalo + kCwTile - 1) / kCwTile, gy = (size_t)(H - kCwHalo + kCwTile - 1) / kCwTile;
    return gx * gy * 3 * kCwBands;
}

// One DFT pass (cw_dft_kernel).  The large tile reuses each operand twice; the
// small one gives four times the workgroups, for passes that would leave CUs
// idle (fewer than two large workgroups per CU).
template <bool COLS, bool INV, bool IMAGE, bool FILTER, int T>
static hipError_t launch_cw_dft_t(const float* a, const float* b, const float2* in, const float* g, float2* out,
                                  const float2* tw, int W, int H, CwColumns cols, int band, dim3 grid, hipStream_t s) {
    const size_t lds = sizeof(float) * (size_t)(2 * kDftStep * 2 * 64 * T + 2 * (COLS ? H : W));
    cw_dft_kernel<COLS, INV, IMAGE, FILTER, T><<<grid, 256, lds, s>>>(a, b, in, g, out, tw, W, H, cols, band);
    return hipGetLastError();
}
template <bool COLS, bool INV, bool IMAGE, bool FILTER>
static hipError_t launch_cw_dft(const float* a, const float* b, const float2* in, const float* g, float2* out,
                                const float2* tw, int W, int H, CwColumns cols, int band, hipStream_t s) {
    auto grid = [&](int T) {
        const unsigned L = 64 * T, O = 32 * T;
        // outputs fastest: the column tiles' work differs by what the filter
        // leaves, and workgroups go round-robin over the XCDs
        if (COLS) return dim3((H + O - 1) / O, (cols.pos + L - 1) / L + (W - cols.neg + L - 1) / L, 6);
        return dim3((W + O - 1) / O, (6 * H + L - 1) / L, 1);
    };
    const dim3 g2 = grid(2);
    if ((size_t)g2.x * g2.y * g2.z >= 512)
        return launch_cw_dft_t<COLS, INV, IMAGE, FILTER, 2>(a, b, in, g, out, tw, W, H, cols, band, g2, s);
    return launch_cw_dft_t<COLS, INV, IMAGE, FILTER, 1>(a, b, in, g, out, tw, W, H, cols, band, grid(1), s);
}

hipError_t launch_cw_ssim(const CwParams& P, int n_images, hipStream_t s) {
    const int W = P.W, H = P.H;
    const long long n = (long long)W * H;
    const int gx = (W - kCwHalo + kCwTile - 1) / kCwTile, gy = (H - kCwHalo + kCwTile - 1) / kCwTile;
    const size_t band_slots = (size_t)gx * gy * 3;
    const double scale = 1.0 / (3.0 * kCwBands * (double)(W - kCwHalo) * (double)(H - kCwHalo));
    const CwColumns all = {W, W};
    float* filter = (float*)P.t1;  // (free until the subband's coefficients are written)
    cw_twiddle_kernel<<<(W + 255) / 256, 256, 0, s>>>(W, P.tw_w);
    cw_twiddle_kernel<<<(H + 255) / 256, 256, 0, s>>>(H, P.tw_h);
    for (int img = 0; img < n_images; ++img) {
        const float* a = P.a + (size_t)img * n * 3;
        const float* b = P.b + (size_t)img * n * 3;
        hipError_t e = launch_cw_dft<false, false, true, false>(a, b, nullptr, nullptr, P.t2, P.tw_w, W, H, all, 0, s);
        if (e == hipSuccess)
            e = launch_cw_dft<true, false, false, false>(a, b, P.t2, nullptr, P.spec, P.tw_h, W, H, all, 0, s);
        for (int band = 0; band < kCwBands && e == hipSuccess; ++band) {
            const int sc = band / kCwOrients, k = band % kCwOrients;
            // column frequencies f that the filter can reach: |f| < W / 2
            // (scale 0; r reaches pi at f = -W / 2, where the window ends) or
            // |f| <= W / 4 (scale 1), f >= 0 for orientation 0
            const int reach = sc == 0 ? W : W / 4 + 1;
            const CwColumns cols = {std::min((W + 1) / 2, reach), k == 0 ? W : std::max(W / 2 + 1, W - reach)};
            cw_filter_kernel<<<dim3((W + 255) / 256, H), 256, 0, s>>>(filter, W, H, sc, k);
            e = launch_cw_dft<true, true, false, true>(a, b, P.spec, filter, P.t2, P.tw_h, W, H, cols, band, s);
            if (e == hipSuccess)
                e = launch_cw_dft<false, true, false, false>(a, b, P.t2, nullptr, P.t1, P.tw_w, W, H, cols, band, s);
            cw_map_kernel<<<dim3(gx, gy, 3), 256, 0, s>>>(P.t1, W, H, P.K, P.slots + band * band_slots);
        }
        if (e != hipSuccess) return e;
        double* runs = (double*)P.t2;
        cw_reduce_kernel<<<kCwRuns, 256, 0, s>>>(P.slots, (int)(band_slots * kCwBands), 1.0, runs);
        cw_reduce_kernel<<<1, 256, 0, s>>>(runs, kCwRuns, scale, P.out + img);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace lp

// nn_kernels.hpp -- BF16 MFMA kernels of the warm-start network (gfx950).
//
// Activations and gradients are BF16 tensors in NHWC order with a channel
// count that is a multiple of 16; products accumulate in FP32 on the matrix
// cores with gfx950's double-depth instruction v_mfma_f32_16x16x32_bf16.  A
// 3x3 convolution is an implicit GEMM: M = output pixels, N = output
// channels, K = 9 taps x input channels (tap-major), taken 32 at a time.
// Operand layout of the 16x16x32 instruction (lane l of a wavefront):
//   A (16 x 32, rows = M): lane l holds A[l % 16][8 (l / 16) + j], j < 8
//   B (32 x 16, rows = K): lane l holds B[8 (l / 16) + j][l % 16]
//   D (16 x 16 FP32):      lane l holds D[4 (l / 16) + j][l % 16]
// Eight consecutive K values of one lane lie in one tap (channel counts
// are multiples of 8), so each A and B fragment is one 16-byte load; K
// values past 9 x cin (cin = 16: 144 = 4.5 x 32) are zero.  Weights are
// kept as [tap][Cout][Cin].
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace lbm {
namespace nn {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef double v4d __attribute__((ext_vector_type(4)));
typedef short v4s __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));  // 16 bytes = 8 BF16 values

__device__ __forceinline__ v4f mfma32(v4u a, v4u b, v4f c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
}

__device__ __forceinline__ float bf2f(uint16_t v) { return __uint_as_float((uint32_t)v << 16); }
__device__ __forceinline__ uint16_t f2bf(float f) {
    const uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
    return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);  // nearest even
}

// 16 bytes at a buffer's byte offset (a lane's part plus a uniform one); zeros past its end
__device__ __forceinline__ __amdgpu_buffer_rsrc_t nn_rsrc(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ v4u nn_load16(__amdgpu_buffer_rsrc_t r, uint32_t lane_offset, uint32_t offset) {
    return __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(r, (int)lane_offset, (int)offset, 0));
}

struct ConvArgs {
    const uint16_t* x;   // [P][cin], P = n h w
    const uint16_t* wt;  // [9][cout][cin]
    const float* bias;   // [cout] or null
    const uint16_t* mask;  // [P][cout] or null: the output is 0 where the mask is not positive
    uint16_t* y;         // [P][cout]
    int32_t n, h, w, cin, cout, relu;
    uint32_t P, ptiles;  // pixels, 16-pixel tiles
    uint32_t tap_group;  // conv3x3_lds_kernel: taps whose weights are staged together (1 or 3)
};

// One wavefront computes 16 MT pixels x (16 NT) output channels: each K
// step loads MT activation fragments and NT weight fragments and issues
// MT x NT MFMAs (the weight fragments are shared by the MT pixel tiles).
template <int NT, int MT = 1>
__global__ __launch_bounds__(256) void conv3x3_kernel(ConvArgs a) {
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t gw = blockIdx.x * 4 + (threadIdx.x >> 6);
    const uint32_t groups = (uint32_t)a.cout / (16 * NT);
    const uint32_t pgroups = (a.ptiles + MT - 1) / MT;
    if (gw >= pgroups * groups) return;
    const uint32_t pg = gw % pgroups, cg = gw / pgroups;
    const uint32_t m = lane & 15, kg = lane >> 4;
    bool pin[MT];
    int32_t pj[MT], pi[MT], pn[MT];
#pragma unroll
    for (int u = 0; u < MT; ++u) {
        const uint32_t p = (pg * MT + u) * 16 + m;
        pin[u] = p < a.P;
        pj[u] = pin[u] ? (int32_t)(p % a.w) : 0;
        pi[u] = pin[u] ? (int32_t)((p / a.w) % a.h) : 0;
        pn[u] = pin[u] ? (int32_t)(p / ((uint32_t)a.w * a.h)) : 0;
    }
    v4f acc[MT][NT];
#pragma unroll
    for (int u = 0; u < MT; ++u)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[u][t] = v4f{0.f, 0.f, 0.f, 0.f};
    const uint32_t K = 9u * (uint32_t)a.cin;
    for (uint32_t k0 = 0; k0 < K; k0 += 32) {
        // this lane's eight K values: tap, first input channel
        const uint32_t k = k0 + 8 * kg;
        const bool kin = k < K;
        const uint32_t tap = kin ? k / (uint32_t)a.cin : 0, ci0 = kin ? k % (uint32_t)a.cin : 0;
        const int32_t dy = (int32_t)tap / 3 - 1, dx = (int32_t)tap % 3 - 1;
        v4u av[MT];
#pragma unroll
        for (int u = 0; u < MT; ++u) {
            const int32_t si = pi[u] + dy, sj = pj[u] + dx;
            const bool ok = kin && pin[u] && si >= 0 && si < a.h && sj >= 0 && sj < a.w;
            av[u] = v4u{0u, 0u, 0u, 0u};
            if (ok) av[u] = *(const v4u*)(a.x + ((size_t)((size_t)pn[u] * a.h + si) * a.w + sj) * a.cin + ci0);
        }
        const uint16_t* wtap = a.wt + (size_t)tap * a.cout * a.cin + ci0;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const uint32_t co = (cg * NT + t) * 16 + m;
            v4u bv = v4u{0u, 0u, 0u, 0u};
            if (kin) bv = *(const v4u*)(wtap + (size_t)co * a.cin);
#pragma unroll
            for (int u = 0; u < MT; ++u) acc[u][t] = mfma32(av[u], bv, acc[u][t]);
        }
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const uint32_t co = (cg * NT + t) * 16 + m;
        const float bb = a.bias ? a.bias[co] : 0.0f;
#pragma unroll
        for (int u = 0; u < MT; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t q = (pg * MT + u) * 16 + 4 * kg + j;
                if (q < a.P) {
                    float v = acc[u][t][j] + bb;
                    if (a.relu) v = fmaxf(v, 0.0f);
                    const size_t e = (size_t)q * a.cout + co;
                    a.y[e] = !a.mask || bf2f(a.mask[e]) > 0.0f ? f2bf(v) : (uint16_t)0;
                }
            }
    }
}

// The same convolution with both operands staged in LDS, for cin a multiple
// of 32.  A block of WM x WN wavefronts computes 16 MT WM consecutive pixels
// x 16 NT WN output channels.  Per tap row dy it stages the source pixels
// p + dy w - 1 .. p + dy w + 1 of its pixels p (all channels; pixel order, so
// the left and right neighbours are the rows before and after, whatever the
// image width), and for one tap or for the row's three (tap_group) the
// weights of its output channels; a tap that leaves the image reads a row of
// zeros.  Both are loaded into registers a stage early.  The K order (tap,
// then channel, 32 at a time, one accumulator) is that of conv3x3_kernel, so
// the results are the same bit for bit.  The operands are swapped (rows of D
// = output channels), so a lane holds four consecutive channels of one pixel
// and stores 8 bytes.
//
// conv3x3_kernel re-reads each activation nine times and each weight once per
// wavefront from L1, 16 rows per 16 lanes, in front of the MFMA that needs
// it.  Measured, us, that kernel / this one: 96 -> 32 channels at 16 x 136 x
// 136 120 / 44; 64 -> 64 at 68 x 68 55 / 15; 192 -> 64 150 / 42; 128 -> 384 at
// 34 x 34 141 / 32; 256 -> 256 at 17 x 17 83 / 20 (270 to 500 TFLOP/s of the
// 2500 of the matrix cores): bound by the stages' barriers and the LDS reads,
// of which an MFMA takes 1 (2 x 2 tiles) to 0.75 (4 x 2).
// LDS rows carry 16 bytes of padding: 16 lanes that read consecutive rows
// then cover all banks for every cin that is a multiple of 32.
__host__ __device__ constexpr uint32_t conv_row_bytes(uint32_t cin) { return 2 * cin + 16; }
// bm + 2 source pixels, a row of zeros, bn weight rows per tap, a scratch piece
__host__ __device__ constexpr size_t conv_lds_bytes(uint32_t bm, uint32_t bn, uint32_t taps, uint32_t cin) {
    return (size_t)(bm + 3 + bn * taps) * conv_row_bytes(cin) + 16;
}

template <int WM, int WN, int MT, int NT>
__global__ __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(MT * NT >= 8 ? 3 : 4)))
void conv3x3_lds_kernel(ConvArgs a) {
    extern __shared__ __align__(16) unsigned char conv_lds[];
    constexpr uint32_t BM = 16 * MT * WM, BN = 16 * NT * WN, T = 64 * WM * WN;
    const uint32_t lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const uint32_t wm = wv % WM, wn = wv / WM;
    const uint32_t m = lane & 15, kg = lane >> 4;
    const uint32_t cin = (uint32_t)a.cin, cout = (uint32_t)a.cout, w = (uint32_t)a.w, h = (uint32_t)a.h;
    // an XCD's blocks are neighbours: they share source rows in its L2
    const uint32_t cgs = cout / BN, per_xcd = gridDim.x / 8;
    const uint32_t blk = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    const uint32_t p0 = blk / cgs * BM;
    if (p0 >= a.P) return;  // whole block
    const uint32_t cb = blk % cgs * BN, co0 = cb + wn * (16 * NT);
    const uint32_t row = conv_row_bytes(cin), zero_row = (BM + 2) * row, w_row = zero_row + row;
    const uint32_t tg = a.tap_group, scratch = w_row + BN * tg * row;

    // this lane's pixels: LDS offset of the centre tap, and which of the nine
    // taps lie inside the image (bit = tap)
    uint32_t at[MT], inside[MT];
#pragma unroll
    for (int u = 0; u < MT; ++u) {
        const uint32_t q = (wm * MT + u) * 16 + m, p = p0 + q;
        const uint32_t r = p / w, j = p - r * w, i = r % h;
        at[u] = (q + 1) * row + kg * 16;
        uint32_t bits = 0x1ffu;
        if (i == 0) bits &= ~0x007u;
        if (i + 1 == h) bits &= ~0x1c0u;
        if (j == 0) bits &= ~0x049u;
        if (j + 1 == w) bits &= ~0x124u;
        inside[u] = p < a.P ? bits : 0u;
    }
    const uint32_t zero_at = zero_row + kg * 16;
    for (uint32_t k = threadIdx.x; k < row / 16; k += T) *(v4u*)(conv_lds + zero_row + k * 16) = v4u{0u, 0u, 0u, 0u};

    v4f acc[MT][NT];
#pragma unroll
    for (int u = 0; u < MT; ++u)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[u][t] = v4f{0.f, 0.f, 0.f, 0.f};

    // Staging: thread t copies 16-byte piece t, t + T, ... of the rows.  Rows
    // outside the tensor read zeros (buffer loads), pieces past the last row
    // go to a scratch piece, so nothing branches around a load.
    const uint32_t c8 = cin / 8;
    const uint32_t r0 = threadIdx.x / c8, k0 = threadIdx.x % c8, dr = T / c8, dk = T % c8;
    auto advance = [&](uint32_t& r, uint32_t& k) __attribute__((always_inline)) {
        k += dk;
        r += dr + (k >= c8 ? 1u : 0u);
        k -= k >= c8 ? c8 : 0u;
    };
    // activations of tap row dy: pieces 0 .. kHeld T - 1 a row early, the rest in place
    constexpr int kHeld = 5;
    v4u held[kHeld];
    const uint32_t pieces = (BM + 2) * c8;
    auto row_source = [&](int dy, uint32_t& shift) __attribute__((always_inline)) {
        const int64_t s0 = (int64_t)p0 + ((int64_t)dy - 1) * w - 1;  // source pixel of LDS row 0
        const int64_t lo = s0 > 0 ? s0 : 0, hi = s0 + BM + 2 < (int64_t)a.P ? s0 + BM + 2 : (int64_t)a.P;
        shift = (uint32_t)(lo - s0) * 2 * cin;  // rows before the tensor: their offsets wrap and read zeros
        return nn_rsrc(a.x + (size_t)lo * cin, hi > lo ? (uint32_t)(hi - lo) * 2 * cin : 0u);
    };
    auto load_x = [&](int dy, uint32_t& r, uint32_t& k) __attribute__((always_inline)) {
        uint32_t shift;
        const __amdgpu_buffer_rsrc_t rx = row_source(dy, shift);
#pragma unroll
        for (int x = 0; x < kHeld; ++x) {
            held[x] = nn_load16(rx, r * 2 * cin + k * 16 - shift, 0);
            advance(r, k);
        }
    };
    auto store_x = [&](uint32_t& r, uint32_t& k) __attribute__((always_inline)) {
#pragma unroll
        for (int x = 0; x < kHeld; ++x) {
            *(v4u*)(conv_lds + (r < BM + 2 ? r * row + k * 16 : scratch)) = held[x];
            advance(r, k);
        }
    };
    // weights of tg taps: rows (tap, channel), the same way
    constexpr int kHeldW = 4;
    v4u held_w[kHeldW];
    const uint32_t w_rows = tg * BN, w_pieces = w_rows * c8;
    const __amdgpu_buffer_rsrc_t rw = nn_rsrc(a.wt, 18u * cin * cout);
    auto load_w = [&](int tap, uint32_t& r, uint32_t& k) __attribute__((always_inline)) {
#pragma unroll
        for (int x = 0; x < kHeldW; ++x) {
            const uint32_t t = r / BN;
            held_w[x] = nn_load16(rw, (((uint32_t)tap + t) * cout + cb + (r - t * BN)) * 2 * cin + k * 16, 0);
            advance(r, k);
        }
    };
    auto store_w = [&](uint32_t& r, uint32_t& k) __attribute__((always_inline)) {
#pragma unroll
        for (int x = 0; x < kHeldW; ++x) {
            *(v4u*)(conv_lds + (r < w_rows ? w_row + r * row + k * 16 : scratch)) = held_w[x];
            advance(r, k);
        }
    };
    {
        uint32_t r = r0, k = k0;
        load_x(0, r, k);
        r = r0, k = k0;
        load_w(0, r, k);
    }
    const uint32_t w_at = w_row + (wn * (16 * NT) + m) * row + kg * 16;
    for (int tap0 = 0; tap0 < 9; tap0 += (int)tg) {
        const int dy = tap0 / 3;
        if (tap0 > 0) __syncthreads();  // the previous stage has been read
        if (tap0 % 3 == 0) {
            uint32_t r = r0, k = k0, r2, k2;
            store_x(r, k);
            r2 = r, k2 = k;
            for (uint32_t e = kHeld * T; e < pieces; e += kHeld * T) {
                load_x(dy, r, k);
                store_x(r2, k2);
            }
        }
        {
            uint32_t r = r0, k = k0, r2, k2;
            store_w(r, k);
            r2 = r, k2 = k;
            for (uint32_t e = kHeldW * T; e < w_pieces; e += kHeldW * T) {
                load_w(tap0, r, k);
                store_w(r2, k2);
            }
        }
        __syncthreads();
        if (tap0 + (int)tg < 9) {
            uint32_t r = r0, k = k0;
            load_w(tap0 + (int)tg, r, k);
            if ((tap0 + (int)tg) % 3 == 0) {
                r = r0, k = k0;
                load_x(dy + 1, r, k);
            }
        }
        for (uint32_t g = 0; g < tg; ++g) {
            const int tap = tap0 + (int)g;
            uint32_t from[MT];
#pragma unroll
            for (int u = 0; u < MT; ++u)
                from[u] = (inside[u] >> tap) & 1u ? at[u] + (uint32_t)(tap - 3 * dy) * row - row : zero_at;
            const uint32_t wf = w_at + g * BN * row;
            for (uint32_t c = 0; c < 2 * cin; c += 64) {
                v4u av[MT], bv[NT];
#pragma unroll
                for (int t = 0; t < NT; ++t) bv[t] = *(const v4u*)(conv_lds + wf + (uint32_t)t * 16 * row + c);
#pragma unroll
                for (int u = 0; u < MT; ++u) av[u] = *(const v4u*)(conv_lds + from[u] + c);
#pragma unroll
                for (int u = 0; u < MT; ++u)
#pragma unroll
                    for (int t = 0; t < NT; ++t) acc[u][t] = mfma32(bv[t], av[u], acc[u][t]);
            }
        }
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const uint32_t co = co0 + t * 16 + 4 * kg;
        v4f bb = v4f{0.f, 0.f, 0.f, 0.f};
        if (a.bias) {
#pragma unroll
            for (int j = 0; j < 4; ++j) bb[j] = a.bias[co + j];
        }
#pragma unroll
        for (int u = 0; u < MT; ++u) {
            const uint32_t p = p0 + (wm * MT + u) * 16 + m;
            if (p >= a.P) continue;
            v4s out;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float v = acc[u][t][j] + bb[j];
                if (a.relu) v = fmaxf(v, 0.0f);
                out[j] = __builtin_bit_cast(short, (__bf16)v);  // nearest even
            }
            if (a.mask) {
                const v4s mk = *(const v4s*)(a.mask + (size_t)p * cout + co);
#pragma unroll
                for (int j = 0; j < 4; ++j) out[j] = bf2f((uint16_t)mk[j]) > 0.0f ? out[j] : (short)0;
            }
            *(v4s*)(a.y + (size_t)p * cout + co) = out;
        }
    }
}

// flipped, transposed weights for the data gradient:
// wf[tap'][ci][co] = wt[8 - tap'][co][ci], of up to kFlipMost layers in one
// launch: a block transposes 32 x 32 values of one tap through LDS
constexpr int kFlipMost = 32;
struct FlipArgs {
    const uint16_t* wt[kFlipMost];
    uint16_t* wf[kFlipMost];
    int32_t cin[kFlipMost], cout[kFlipMost];
    uint32_t first[kFlipMost + 1];  // first block of each layer
    int32_t count;
};
__global__ __launch_bounds__(256) void wflip_kernel(FlipArgs a) {
    __shared__ uint16_t t[32][33];
    const uint32_t x = threadIdx.x & 31, y = threadIdx.x >> 5;
    int l = 0;
    for (uint32_t b = blockIdx.x; b < a.first[a.count]; b += gridDim.x) {
        while (l + 1 < a.count && b >= a.first[l + 1]) ++l;
        const uint32_t ci = (uint32_t)a.cin[l], co = (uint32_t)a.cout[l];
        const uint32_t ti = (ci + 31) / 32, to = (co + 31) / 32, r = b - a.first[l];
        const uint32_t tap = r / (ti * to), i0 = r % ti * 32, o0 = r / ti % to * 32;
        const uint16_t* src = a.wt[l] + (size_t)(8 - tap) * co * ci;
        uint16_t* dst = a.wf[l] + (size_t)tap * co * ci;
        if (b > blockIdx.x) __syncthreads();  // the previous square has been read
#pragma unroll
        for (uint32_t k = 0; k < 32; k += 8)
            if (o0 + y + k < co && i0 + x < ci) t[y + k][x] = src[(size_t)(o0 + y + k) * ci + i0 + x];
        __syncthreads();
#pragma unroll
        for (uint32_t k = 0; k < 32; k += 8)
            if (i0 + y + k < ci && o0 + x < co) dst[(size_t)(i0 + y + k) * co + o0 + x] = t[x][y + k];
    }
}

// division of e < 2^31 by d (Granlund and Montgomery, 1994): with s = ceil(log2
// d) and m = ceil(2^(31 + s) / d) < 2^32, m d exceeds 2^(31 + s) by less than
// 2^s, so e m / 2^(31 + s) exceeds e / d by less than 1 / d
struct Div31 {
    uint32_t m, s;
    __device__ uint32_t of(uint32_t e) const { return (uint32_t)((uint64_t)e * m >> s); }
};

struct WGradArgs {
    const uint16_t* x;   // [n][h][w][cin]
    const uint16_t* dz;  // [n][h][w][cout]
    float* partial;      // [chunks][9][cout][cin]
    float* bias;         // [chunks][cout], or null
    int32_t n, h, w, cin, cout;
    uint32_t tiles_x, tiles_y, tiles;  // pixel tiles per row and per image column (not stacked), and in all
    uint32_t per, chunks;              // tiles per chunk, chunks
    // stacked: images beside each other, columns and rows of the stack, columns
    // from image to image (2^31 - 1 with one across), and division by that and by h + 1
    uint32_t across, cols, rows, col_pitch;
    Div31 by_col_pitch, by_pitch;
};

// dW[tap][co][ci] = sum_p dz[p][co] x[p shifted by tap][ci] and db[co] =
// sum_p dz[p][co], on the matrix cores with K = pixels: 8 x 4 of them per
// instruction.  A wavefront holds 32 x 32 channels of all nine taps (144
// accumulators), so a pixel tile staged once in LDS, x with its halo, serves
// 36 MFMAs per K step.  Both tensors are pixel-major; the operand fragments
// (eight pixels of one channel per lane) come from LDS through the
// transposing read: of the 16 lanes of a group, lanes 4r .. 4r + 3 point at
// the 16 channels of pixel r, and lane i receives channel i of the four
// pixels.  A tap is then an offset of whole pixels.  Pixels outside the image
// are zeros in both tiles.  Images of a few rows are stacked, and narrow ones
// set beside each other too, with a row and a column of zeros between them, so
// that they fill tiles (Stacked; 4096 images of 1 x 1, 256 -> 256 channels:
// 60 us, 320 with tiles of each image's own; 16 of 2 x 2 19 and 37).  The block's WCO x WCI wavefronts tile the
// channels, WK of them split the K steps and add their sums at the end; the
// chunks (runs of tiles) are summed by sum_chunks_kernel.  The bias gradient
// is one more MFMA against ones.
//
// The kernel this replaced ran one tap per wavefront: it loaded both operands
// nine times and transposed them through 16-bit LDS writes.  us before /
// after, sums included: 32 -> 32 channels at 16 x 136 x 136 156 / 28, 96 -> 32
// 202 / 45, 64 -> 64 at 68 x 68 96 / 26, 256 -> 256 at 17 x 17 103 / 33.  Bound
// by the latency of a tile's loads and the partial sums' traffic: two
// wavefronts per SIMD (the accumulators) hold few tiles in flight.
// LDS pixels carry 32 bytes of padding, so four consecutive pixels of a
// transposing read fall into different banks.
using lds_v4s = __attribute__((address_space(3))) v4s;
__device__ __forceinline__ v4u lds_transposed(const unsigned char* p, const unsigned char* p4) {
    const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)p);
    const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)p4);
    struct P { v4s lo, hi; } r{lo, hi};
    return __builtin_bit_cast(v4u, r);
}

constexpr int kWgTileH = 16;  // rows of a pixel tile (four K steps)
template <int WCO, int WCI, int WK, int KX, bool Stacked>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void wgrad_kernel(WGradArgs a) {
    static_assert(WCO * WCI * WK == 4, "four wavefronts");
    constexpr int TW = 8 * KX, TH = kWgTileH, COB = 32 * WCO, CIB = 32 * WCI;
    constexpr uint32_t SD = COB * 2 + 32, SX = CIB * 2 + 32;  // bytes per LDS pixel
    constexpr int ND = TW * TH * (COB / 8), NX = (TW + 2) * (TH + 2) * (CIB / 8);  // 16-byte pieces
    constexpr int PD = (ND + 255) / 256, PX = (NX + 255) / 256;
    constexpr uint32_t kXAt = TW * TH * SD, kZeroAt = kXAt + (TW + 2) * (TH + 2) * SX;
    constexpr uint32_t kZeroBytes = (2 * (TW + 2) + 2) * SX + 48;  // as far as a lane's reads of the nine taps go
    constexpr uint32_t kTileBytes = kZeroAt + kZeroBytes;
    constexpr uint32_t kSumBytes = WCO * WCI * 64 * 48 * 4;  // three taps of one wavefront per channel tile
    __shared__ __align__(16) unsigned char lds[kTileBytes > kSumBytes || WK == 1 ? kTileBytes : kSumBytes];
    const uint32_t lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const uint32_t wco = wv % WCO, wci = wv / WCO % WCI, wk = wv / (WCO * WCI);
    const uint32_t i = lane & 15, kg = lane >> 4;
    const uint32_t cot = ((uint32_t)a.cout + COB - 1) / COB, cit = ((uint32_t)a.cin + CIB - 1) / CIB;
    // an XCD's blocks are neighbours: the channel tiles of one chunk share its pixels in the L2
    const uint32_t per_xcd = gridDim.x / 8, blk = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    const uint32_t chunk = blk / (cot * cit), cb = blk % cot, ib = blk / cot % cit;
    if (chunk >= a.chunks) return;  // whole block
    const uint32_t t_begin = chunk * a.per, t_end = min(t_begin + a.per, a.tiles);

    v4f acc[9][2][2], accb[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        accb[u] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int tap = 0; tap < 9; ++tap) acc[tap][u][t] = v4f{0.f, 0.f, 0.f, 0.f};
    }
    v4u ones;
#pragma unroll
    for (int k = 0; k < 4; ++k) ones[k] = 0x3f803f80u;
    const bool with_bias = a.bias && ib == 0 && wci == 0;

    for (uint32_t k = threadIdx.x; k < kZeroBytes / 16; k += 256) *(v4u*)(lds + kZeroAt + k * 16) = v4u{0u, 0u, 0u, 0u};

    // a tile: its first column, the image row of its first pixel row (not
    // stacked: the image) and the row in it, and that row's place in the stack
    struct Tile {
        uint32_t x0, img, y0, v0;
    };
    const uint32_t h = (uint32_t)a.h, w = (uint32_t)a.w, n = (uint32_t)a.n, pitch = h + 1, cpitch = a.col_pitch;
    // Stacked: the image, row and column of place (u, c) from image row r0 on
    struct Pixel {
        uint32_t img, y, x;
        bool in;
    };
    auto pixel = [&](uint32_t r0, uint32_t u, uint32_t c) __attribute__((always_inline)) {
        const uint32_t d = a.by_pitch.of(u), g = a.by_col_pitch.of(c);
        Pixel q{(r0 + d) * a.across + g, u - d * pitch, c - g * cpitch, false};
        q.in = q.y < h && q.x < w && g < a.across && q.img < n;
        return q;
    };
    v4u dv[PD], xv[PX];
    auto load = [&](uint32_t t) __attribute__((always_inline)) {
        Tile at;
        at.v0 = t / a.tiles_x * TH;
        at.x0 = t % a.tiles_x * TW;
        at.img = Stacked ? at.v0 / pitch : t / (a.tiles_x * a.tiles_y);
        at.y0 = at.v0 - at.img * (Stacked ? pitch : a.tiles_y * TH);
        const size_t base = Stacked ? 0 : (size_t)at.img * h * w;
#pragma unroll
        for (int p = 0; p < PD; ++p) {
            const int e = p * 256 + (int)threadIdx.x, px = e / (COB / 8), k = e % (COB / 8);
            const uint32_t ch = cb * COB + k * 8, y = at.y0 + px / TW, x = at.x0 + px % TW;
            size_t from = base + (size_t)y * w + x;
            bool in = y < h && x < w;
            if constexpr (Stacked) {
                const Pixel q = pixel(at.img, y, x);
                from = ((size_t)q.img * h + q.y) * w + q.x;
                in = q.in;
            }
            dv[p] = v4u{0u, 0u, 0u, 0u};
            if (e < ND && in && ch < (uint32_t)a.cout) dv[p] = *(const v4u*)(a.dz + from * a.cout + ch);
        }
#pragma unroll
        for (int p = 0; p < PX; ++p) {
            const int e = p * 256 + (int)threadIdx.x, px = e / (CIB / 8), k = e % (CIB / 8);
            // row and column -1 wrap and lie outside too
            const uint32_t ch = ib * CIB + k * 8, y = at.y0 + px / (TW + 2) - 1, x = at.x0 + px % (TW + 2) - 1;
            size_t from = base + (size_t)y * w + x;
            bool in = y < h && x < w;
            if constexpr (Stacked) {
                const Pixel q = pixel(at.img - 1, y + pitch, x);  // from the zeros above image row at.img on
                from = ((size_t)q.img * h + q.y) * w + q.x;
                in = x + 1 > 0 && q.in;
            }
            xv[p] = v4u{0u, 0u, 0u, 0u};
            if (e < NX && in && ch < (uint32_t)a.cin) xv[p] = *(const v4u*)(a.x + from * a.cin + ch);
        }
        return at;
    };
    Tile next = load(t_begin);
    for (uint32_t t = t_begin; t < t_end; ++t) {
        if (t > t_begin) __syncthreads();  // the previous tile has been read
#pragma unroll
        for (int p = 0; p < PD; ++p) {
            const uint32_t e = p * 256 + threadIdx.x;
            if (ND % 256 == 0 || e < ND) *(v4u*)(lds + e / (COB / 8) * SD + e % (COB / 8) * 16) = dv[p];
        }
#pragma unroll
        for (int p = 0; p < PX; ++p) {
            const uint32_t e = p * 256 + threadIdx.x;
            if (NX % 256 == 0 || e < NX) *(v4u*)(lds + kXAt + e / (CIB / 8) * SX + e % (CIB / 8) * 16) = xv[p];
        }
        __syncthreads();
        const Tile at = next;
        if (t + 1 < t_end) next = load(t + 1);
        for (uint32_t ks = wk; ks < KX * (TH / 4); ks += WK) {
            const uint32_t kx = ks % KX * 8, ky = ks / KX * 4;
            const bool rows_in = Stacked ? at.v0 + ky < a.rows : at.y0 + ky < h;
            if (!rows_in || at.x0 + kx >= (Stacked ? a.cols : w)) continue;  // all outside
            const unsigned char* pd = lds + ((ky + kg) * TW + kx + (i >> 2)) * SD + wco * 64 + (i & 3) * 8;
            // this lane's pixels of the K step, four apart.  Outside the image
            // dz is 0, but the x beside it may lie inside, and 0 times an
            // infinity must not reach a tap that does not use it: there a
            // lane points at zeros.
            const unsigned char* px = lds + kXAt + ((ky + kg) * (TW + 2) + kx + (i >> 2)) * SX + wci * 64 + (i & 3) * 8;
            const uint32_t y = at.y0 + ky + kg, x = at.x0 + kx + (i >> 2);
            const bool in = Stacked ? pixel(at.img, y, x).in : y < h && x < w;
            const bool in4 = Stacked ? pixel(at.img, y, x + 4).in : y < h && x + 4 < w;
            const unsigned char* px4 = in4 ? px + 4 * SX : lds + kZeroAt;
            px = in ? px : lds + kZeroAt;
            v4u av[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) av[u] = lds_transposed(pd + u * 32, pd + u * 32 + 4 * SD);
            if (with_bias) {
#pragma unroll
                for (int u = 0; u < 2; ++u) accb[u] = mfma32(av[u], ones, accb[u]);
            }
#pragma unroll
            for (int tap = 0; tap < 9; ++tap) {
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    const uint32_t at = (tap / 3 * (TW + 2) + tap % 3) * SX + s * 32;
                    const v4u bv = lds_transposed(px + at, px4 + at);
#pragma unroll
                    for (int u = 0; u < 2; ++u) acc[tap][u][s] = mfma32(av[u], bv, acc[tap][u][s]);
                }
            }
            // x fragments are read three ahead of the MFMAs that use them; the
            // compiler's own order has one, for want of registers (64 -> 64
            // channels at 16 x 136 x 136: 46 us, 56 in that order)
            __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
#pragma unroll
            for (int k = 0; k < 15; ++k) {
                __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            }
            __builtin_amdgcn_sched_group_barrier(0x008, 6, 0);
        }
    }
    // the sums of the wavefronts that split the K steps, three taps at a time, in order
    if constexpr (WK > 1) {
        v4f* sum = (v4f*)lds + (size_t)(wv % (WCO * WCI)) * 64 * 12;
#pragma unroll
        for (int g = 0; g < 3; ++g) {
            for (uint32_t k = 1; k < WK; ++k) {
                __syncthreads();
                if (wk == k) {
#pragma unroll
                    for (int e = 0; e < 12; ++e) sum[e * 64 + lane] = acc[g * 3 + e / 4][e / 2 % 2][e % 2];
                }
                __syncthreads();
                if (wk == 0) {
#pragma unroll
                    for (int e = 0; e < 12; ++e) acc[g * 3 + e / 4][e / 2 % 2][e % 2] += sum[e * 64 + lane];
                }
            }
        }
        for (uint32_t k = 1; k < WK; ++k) {
            __syncthreads();
            if (wk == k) {
#pragma unroll
                for (int e = 0; e < 2; ++e) sum[e * 64 + lane] = accb[e];
            }
            __syncthreads();
            if (wk == 0) {
#pragma unroll
                for (int e = 0; e < 2; ++e) accb[e] += sum[e * 64 + lane];
            }
        }
        if (wk != 0) return;
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const uint32_t co = cb * COB + wco * 32 + u * 16 + 4 * kg;
        if (co >= (uint32_t)a.cout) continue;
        if (with_bias && i == 0) {
#pragma unroll
            for (int j = 0; j < 4; ++j) a.bias[(size_t)chunk * a.cout + co + j] = accb[u][j];
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const uint32_t ci = ib * CIB + wci * 32 + s * 16 + i;
            if (ci >= (uint32_t)a.cin) continue;
#pragma unroll
            for (int tap = 0; tap < 9; ++tap)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    a.partial[(((size_t)chunk * 9 + tap) * a.cout + co + j) * a.cin + ci] = acc[tap][u][s][j];
        }
    }
}

// dw[e] = sum over the chunks of partial[c][e], and db likewise: a block takes
// 64 values, its 16 rows of threads every 16th chunk, and the row sums are added
// in a fixed tree; with four chunks or fewer a block takes 1024 values, a
// thread's in order (512 -> 512 channels at 1 x 16 x 16, weight gradient and
// sums: 38 us with rows of which two held chunks, 20).  The bias gradient's sums
// are FP64, as the matrix cores' sums of a chunk lose by themselves what its
// former kernels lost in all (relative error at 16 x 136 x 136, 32 channels:
// 7.8e-8 before, 9.4e-8 with FP32 sums here, 3.6e-8 so; the weights' is below the
// former one either way, 3.7e-7 and 1.2e-7).
struct SumChunksArgs {
    const float* partial;
    float* dw;
    size_t count;
    uint32_t chunks;
    const float* bias;
    float* db;
    uint32_t bias_count;
};
template <uint32_t ROWS>  // of threads: 16, or 1
__global__ __launch_bounds__(256) void sum_chunks_kernel(SumChunksArgs a) {
    __shared__ v4d lds[256];
    constexpr uint32_t cols = 256 / ROWS, each = cols * 4;
    const uint32_t col = threadIdx.x % cols, part = threadIdx.x / cols;
    const size_t blocks_w = (a.count + each - 1) / each;
    const size_t blocks = blocks_w + (a.bias_count + each - 1) / each;
    // block b of the sums, in the precision of vector v
    auto sum = [&](auto v, const float* src, float* dst, size_t count, size_t b) __attribute__((always_inline)) {
        using V = decltype(v);
        V* mine = (V*)lds;
        const size_t e = b * each + col * 4;  // counts are multiples of 16
        if (e < count)
            for (uint32_t c = part; c < a.chunks; c += ROWS) {
                const float* p = src + c * count + e;
#pragma unroll
                for (int j = 0; j < 4; ++j) v[j] += p[j];
            }
        mine[threadIdx.x] = v;
        for (uint32_t o = 128; o >= cols; o >>= 1) {
            __syncthreads();
            if (threadIdx.x < o) mine[threadIdx.x] += mine[threadIdx.x + o];
        }
        if (part == 0 && e < count) {
#pragma unroll
            for (int j = 0; j < 4; ++j) dst[e + j] = (float)mine[threadIdx.x][j];
        }
    };
    for (size_t b = blockIdx.x; b < blocks; b += gridDim.x) {
        if (b > blockIdx.x) __syncthreads();  // the previous sums have been read
        if (b < blocks_w) sum(v4f{0.f, 0.f, 0.f, 0.f}, a.partial, a.dw, a.count, b);
        else sum(v4d{0.0, 0.0, 0.0, 0.0}, a.bias, a.db, a.bias_count, b - blocks_w);
    }
}

// ------------------------------------------------- layers without products
// Memory-bound passes over NHWC tensors.  A thread takes eight channels (16
// bytes) of one pixel of the output, in its order in memory, so blocks are
// full whatever the image's width (a block per run of an image row left most
// threads idle on narrow ones: pooling 4 images of 200000 x 2, 8 channels, 147
// us, 9 now); row and column come from two multiplications.  The
// element-per-thread kernels (below) spend their time on four 64-bit
// divisions per value.  In one gradient of the 257^2
// network (batch 16) the upsampling, concatenation, pooling and ReLU passes,
// forward and backward, took 670 us in 41 launches; joined they take 104 us in
// 12, and the ReLU masks of the others ride in the convolutions' stores.
struct Vec8 {
    v4u v;
    __device__ float get(int j) const { return bf2f((uint16_t)(v[j / 2] >> (16 * (j % 2)))); }
    __device__ void set(int j, float f) {
        const uint32_t b = (uint32_t)f2bf(f) << (16 * (j % 2));
        v[j / 2] = j % 2 ? (v[j / 2] & 0xffffu) | b : (v[j / 2] & 0xffff0000u) | b;
    }
};
__device__ __forceinline__ Vec8 load8(const uint16_t* p) { return Vec8{*(const v4u*)p}; }
__device__ __forceinline__ void store8(uint16_t* p, Vec8 x) { *(v4u*)p = x.v; }
// x where the ReLU output m is positive, else 0
__device__ __forceinline__ Vec8 relu_mask(Vec8 x, Vec8 m) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t lo = m.get(2 * j) > 0.0f ? 0x0000ffffu : 0u, hi = m.get(2 * j + 1) > 0.0f ? 0xffff0000u : 0u;
        x.v[j] &= lo | hi;
    }
    return x;
}
// the output of a pass: `items` groups of eight channels, c8 per pixel, w pixels per row
struct RowShape {
    uint32_t items, c8, w;
    Div31 by_c8, by_w;
};
// this thread's item e: channel group k of pixel j in row r = image * height + i
struct RowPlace {
    uint32_t e, k, j, r;
    bool in;
    __device__ explicit RowPlace(const RowShape& a) {
        e = blockIdx.x * 256 + threadIdx.x;
        in = e < a.items;
        const uint32_t q = a.by_c8.of(e);
        k = e - q * a.c8;
        r = a.by_w.of(q);
        j = q - r * a.w;
    }
};

// x [n][h/2][w/2][cx] nearest-upsampled beside skip [n][h][w][cs] -> y [n][h][w][cx + cs]
__global__ __launch_bounds__(256) void up_concat_kernel(const uint16_t* x, const uint16_t* skip, uint16_t* y,
                                                        RowShape a, uint32_t cx, uint32_t cs) {
    const RowPlace p(a);
    if (!p.in) return;
    const size_t k = (size_t)p.k * 8, low = (size_t)(p.r / 2) * (a.w / 2) + p.j / 2, q = (size_t)p.r * a.w + p.j;
    store8(y + (size_t)p.e * 8, k < cx ? load8(x + low * cx + k) : load8(skip + q * cs + (k - cx)));
}

// gradient of the upsampled part: dx [n][h][w][c] = sums of the 2x2 blocks of
// channels 0 .. c - 1 of dy [n][2h][2w][cd], where mask (null: everywhere) is positive
__global__ __launch_bounds__(256) void up_backward_kernel(const uint16_t* dy, const uint16_t* mask, uint16_t* dx,
                                                          RowShape a, uint32_t cd) {
    const RowPlace p(a);
    if (!p.in) return;
    const size_t row = (size_t)2 * a.w * cd;
    const uint16_t* s = dy + 2 * p.r * row + (size_t)2 * p.j * cd + (size_t)p.k * 8;
    const Vec8 s0 = load8(s), s1 = load8(s + cd), s2 = load8(s + row), s3 = load8(s + row + cd);
    Vec8 o{v4u{0u, 0u, 0u, 0u}};
#pragma unroll
    for (int j = 0; j < 8; ++j) o.set(j, s0.get(j) + s1.get(j) + s2.get(j) + s3.get(j));
    if (mask) o = relu_mask(o, load8(mask + (size_t)p.e * 8));
    store8(dx + (size_t)p.e * 8, o);
}

// x [n][2h][2w][c] -> y [n][h][w][c], 2x2 means
__global__ __launch_bounds__(256) void pool_kernel(const uint16_t* x, uint16_t* y, RowShape a) {
    const RowPlace p(a);
    if (!p.in) return;
    const size_t c = (size_t)a.c8 * 8, row = 2 * a.w * c;
    const uint16_t* s = x + 2 * p.r * row + 2 * p.j * c + (size_t)p.k * 8;
    const Vec8 s0 = load8(s), s1 = load8(s + c), s2 = load8(s + row), s3 = load8(s + row + c);
    Vec8 o{v4u{0u, 0u, 0u, 0u}};
#pragma unroll
    for (int j = 0; j < 8; ++j) o.set(j, 0.25f * (s0.get(j) + s1.get(j) + s2.get(j) + s3.get(j)));
    store8(y + (size_t)p.e * 8, o);
}

// gradient of the pooling: dx [n][h][w][c] = dy [n][h/2][w/2][c] / 4, plus
// channels ao .. ao + c - 1 of add [n][h][w][ca] (null: nothing), where mask
// (null: everywhere) is positive; each sum rounded to BF16 as it is formed
__global__ __launch_bounds__(256) void pool_backward_kernel(const uint16_t* dy, const uint16_t* add, const uint16_t* mask,
                                                            uint16_t* dx, RowShape a, uint32_t ca, uint32_t ao) {
    const RowPlace p(a);
    if (!p.in) return;
    const size_t k = (size_t)p.k * 8, low = (size_t)(p.r / 2) * (a.w / 2) + p.j / 2;
    const Vec8 s = load8(dy + low * a.c8 * 8 + k);
    Vec8 o{v4u{0u, 0u, 0u, 0u}};
#pragma unroll
    for (int j = 0; j < 8; ++j) o.set(j, 0.25f * s.get(j));
    if (add) {
        const Vec8 d = load8(add + ((size_t)p.r * a.w + p.j) * ca + ao + k);
#pragma unroll
        for (int j = 0; j < 8; ++j) o.set(j, o.get(j) + d.get(j));
    }
    if (mask) o = relu_mask(o, load8(mask + (size_t)p.e * 8));
    store8(dx + (size_t)p.e * 8, o);
}

// dst[p][doff + k] (+)= src[p][soff + k] for k < cc; c8 = cc / 8
__global__ __launch_bounds__(256) void copy_channels8_kernel(const uint16_t* src, uint32_t cs, uint32_t soff, uint16_t* dst,
                                                             uint32_t cd, uint32_t doff, uint32_t c8, uint32_t items,
                                                             int32_t accumulate) {
    for (uint32_t e = blockIdx.x * 256 + threadIdx.x; e < items; e += gridDim.x * 256) {
        const uint32_t p = e / c8, k = (e - p * c8) * 8;
        const Vec8 v = load8(src + (size_t)p * cs + soff + k);
        uint16_t* d = dst + (size_t)p * cd + doff + k;
        if (!accumulate) {
            store8(d, v);
            continue;
        }
        Vec8 o = load8(d);
#pragma unroll
        for (int j = 0; j < 8; ++j) o.set(j, o.get(j) + v.get(j));
        store8(d, o);
    }
}

// eight values per thread, then the rest one by one
__global__ __launch_bounds__(256) void relu_backward_kernel(const uint16_t* y, const uint16_t* dy, uint16_t* dz,
                                                            size_t groups, size_t count) {
    for (size_t e = blockIdx.x * (size_t)256 + threadIdx.x; e < groups; e += (size_t)gridDim.x * 256)
        store8(dz + e * 8, relu_mask(load8(dy + e * 8), load8(y + e * 8)));
    for (size_t e = groups * 8 + blockIdx.x * (size_t)256 + threadIdx.x; e < count; e += (size_t)gridDim.x * 256)
        dz[e] = bf2f(y[e]) > 0.0f ? dy[e] : (uint16_t)0;
}

// the same one value per thread, for channel counts or pointers that rule
// out 16-byte accesses
// x [n][h][w][c] -> y [n][h/2][w/2][c], 2x2 means
__global__ void avgpool2_kernel(const uint16_t* x, uint16_t* y, int32_t n, int32_t h, int32_t w, int32_t c) {
    const size_t total = (size_t)n * (h / 2) * (w / 2) * c;
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
        const int32_t ch = (int32_t)(e % c);
        const size_t q = e / c;
        const int32_t j = (int32_t)(q % (w / 2)), i = (int32_t)((q / (w / 2)) % (h / 2));
        const int32_t b = (int32_t)(q / ((size_t)(w / 2) * (h / 2)));
        const size_t base = (((size_t)b * h + 2 * i) * w + 2 * j) * c + ch;
        const float s = bf2f(x[base]) + bf2f(x[base + c]) + bf2f(x[base + (size_t)w * c]) +
                        bf2f(x[base + (size_t)w * c + c]);
        y[e] = f2bf(0.25f * s);
    }
}

// gradient of avgpool2: dx[n][h][w][c] = dy[n][h/2][w/2][c] / 4
__global__ void avgpool2_backward_kernel(const uint16_t* dy, uint16_t* dx, int32_t n, int32_t h, int32_t w, int32_t c) {
    const size_t total = (size_t)n * h * w * c;
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
        const int32_t ch = (int32_t)(e % c);
        const size_t q = e / c;
        const int32_t j = (int32_t)(q % w), i = (int32_t)((q / w) % h), b = (int32_t)(q / ((size_t)w * h));
        dx[e] = f2bf(0.25f * bf2f(dy[(((size_t)b * (h / 2) + i / 2) * (w / 2) + j / 2) * c + ch]));
    }
}

// nearest upsampling x [n][h][w][c] -> y [n][2h][2w][c]
__global__ void upsample2_kernel(const uint16_t* x, uint16_t* y, int32_t n, int32_t h, int32_t w, int32_t c) {
    const size_t total = (size_t)n * 4 * h * w * c;
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
        const int32_t ch = (int32_t)(e % c);
        const size_t q = e / c;
        const int32_t j = (int32_t)(q % (2 * w)), i = (int32_t)((q / (2 * w)) % (2 * h));
        const int32_t b = (int32_t)(q / ((size_t)4 * w * h));
        y[e] = x[(((size_t)b * h + i / 2) * w + j / 2) * c + ch];
    }
}

// gradient of upsample2: dx[n][h][w][c] = sum of the 2x2 block of dy
__global__ void upsample2_backward_kernel(const uint16_t* dy, uint16_t* dx, int32_t n, int32_t h, int32_t w, int32_t c) {
    const size_t total = (size_t)n * h * w * c;
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
        const int32_t ch = (int32_t)(e % c);
        const size_t q = e / c;
        const int32_t j = (int32_t)(q % w), i = (int32_t)((q / w) % h), b = (int32_t)(q / ((size_t)w * h));
        const size_t base = (((size_t)b * 2 * h + 2 * i) * 2 * w + 2 * j) * c + ch;
        const float s = bf2f(dy[base]) + bf2f(dy[base + c]) + bf2f(dy[base + (size_t)2 * w * c]) +
                        bf2f(dy[base + (size_t)2 * w * c + c]);
        dx[e] = f2bf(s);
    }
}

// dst[p][doff + k] (+)= src[p][soff + k] for k < cc
__global__ void copy_channels_kernel(const uint16_t* src, int32_t cs, int32_t soff, uint16_t* dst, int32_t cd,
                                     int32_t doff, int32_t cc, size_t pixels, int32_t accumulate) {
    const size_t total = pixels * cc;
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
        const size_t p = e / cc;
        const int32_t k = (int32_t)(e % cc);
        const uint16_t v = src[p * cs + soff + k];
        uint16_t& d = dst[p * cd + doff + k];
        d = accumulate ? f2bf(bf2f(d) + bf2f(v)) : v;
    }
}

// masked MSE over the first `used` channels: per-block partial sums of
// mask (y - t)^2, and dy = 2 mask (y - t) / count (BF16)
__global__ __launch_bounds__(256) void mse_kernel(const uint16_t* y, int32_t cy, const float* target,
                                                  const float* mask, size_t pixels, int32_t used, float inv_count,
                                                  uint16_t* dy, float* partial) {
    __shared__ float lds[256];
    float s = 0.0f;
    const size_t total = pixels * cy;
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
        const size_t p = e / cy;
        const int32_t k = (int32_t)(e % cy);
        float g = 0.0f;
        if (k < used) {
            const float mk = mask[p * used + k];
            const float d = (bf2f(y[e]) - target[p * used + k]) * mk;
            s += d * d;
            g = 2.0f * d * inv_count;
        }
        if (dy) dy[e] = f2bf(g);
    }
    lds[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) lds[threadIdx.x] += lds[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = lds[0];
}

// out[0] = scale * (sum of the partials), one block, a fixed tree
__global__ __launch_bounds__(256) void sum_partials_kernel(const float* partial, int32_t n, float scale, float* out) {
    __shared__ float lds[256];
    float s = 0.0f;
    for (int32_t i = threadIdx.x; i < n; i += 256) s += partial[i];
    lds[threadIdx.x] = s;
    for (uint32_t o = 128; o > 0; o >>= 1) {
        __syncthreads();
        if (threadIdx.x < o) lds[threadIdx.x] += lds[threadIdx.x + o];
    }
    if (threadIdx.x == 0) out[0] = lds[0] * scale;
}

// Adam (Kingma & Ba, 2015) on FP32 master weights; also refreshes the
// BF16 copy used by the kernels
__global__ void adam_kernel(float* w, const float* g, float* m, float* v, size_t count, float lr, float b1, float b2,
                            float eps, float c1, float c2, uint16_t* wbf) {
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < count; e += (size_t)gridDim.x * blockDim.x) {
        const float gi = g[e];
        const float mi = b1 * m[e] + (1.0f - b1) * gi;
        const float vi = b2 * v[e] + (1.0f - b2) * gi * gi;
        m[e] = mi;
        v[e] = vi;
        const float wi = w[e] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
        w[e] = wi;
        if (wbf) wbf[e] = f2bf(wi);
    }
}

__global__ void f32_to_bf16_kernel(const float* src, uint16_t* dst, size_t count) {
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < count; e += (size_t)gridDim.x * blockDim.x)
        dst[e] = f2bf(src[e]);
}

__global__ void bf16_to_f32_kernel(const uint16_t* src, float* dst, size_t count) {
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < count; e += (size_t)gridDim.x * blockDim.x)
        dst[e] = bf2f(src[e]);
}

}  // namespace nn
}  // namespace lbm

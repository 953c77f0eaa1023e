// nn_api.hip -- host side of include/lbm_nn.h: shape checks and launches of
// the BF16 MFMA network kernels on the caller's stream.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include <cmath>
#include <cstdarg>
#include <cstdio>

#include "../../include/lbm_nn.h"
#include "nn_kernels.hpp"

using namespace lbm::nn;

namespace {

thread_local char g_nn_err[512] = "";

lbm_status nn_fail(lbm_status st, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_nn_err, sizeof(g_nn_err), fmt, ap);
    va_end(ap);
    return st;
}

lbm_status launched(const char* what) {
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return nn_fail(LBM_E_DEVICE, "%s: %s", what, hipGetErrorString(e));
    return LBM_OK;
}

unsigned grid1(size_t n, unsigned bs = 256, unsigned cap = 65536) {
    const size_t g = (n + bs - 1) / bs;
    return (unsigned)(g < 1 ? 1 : (g > cap ? cap : g));
}

bool pos(int32_t v) { return v > 0; }

bool aligned16(const void* p) { return (uintptr_t)p % 16 == 0; }

Div31 div31(uint32_t d) {
    uint32_t s = 0;
    while (s < 31 && (1u << s) < d) ++s;
    return {(uint32_t)((((uint64_t)1 << (31 + s)) + d - 1) / d), 31 + s};
}

// the passes over an output of n x h x w pixels and c channels, a thread per
// eight channels.  false: channels not a multiple of 8, or 2^31 groups of them
// and more (the element kernels take those).
bool row_grid(int64_t n, int64_t h, int64_t w, int64_t c, RowShape* a, dim3* grid) {
    if (c % 8 || (double)n * h * w * (c / 8) >= 2147483648.0) return false;
    a->items = (uint32_t)(n * h * w * (c / 8));
    a->c8 = (uint32_t)(c / 8);
    a->w = (uint32_t)w;
    a->by_c8 = div31(a->c8);
    a->by_w = div31(a->w);
    *grid = dim3((a->items + 255) / 256);
    return true;
}

constexpr size_t kMaxLds = 160 * 1024;
constexpr uint32_t kMostBlocks = 65536;  // of kernels whose blocks loop over any number of pieces

template <int WM, int WN, int MT, int NT> bool conv3x3_lds_go(ConvArgs a, uint32_t taps, hipStream_t s) {
    constexpr uint32_t BM = 16 * MT * WM, BN = 16 * NT * WN;
    a.tap_group = taps;
    const size_t lds = conv_lds_bytes(BM, BN, taps, (uint32_t)a.cin);
    const uint64_t blocks = ((uint64_t)a.P + BM - 1) / BM * ((uint32_t)a.cout / BN);
    if (lds > kMaxLds || blocks > 0x7ffffff0ull) return false;
    hipLaunchKernelGGL((conv3x3_lds_kernel<WM, WN, MT, NT>), dim3((unsigned)((blocks + 7) / 8 * 8)),
                       dim3(64 * WM * WN), lds, s, a);
    return true;
}

// The LDS convolution where it applies: whole K steps inside a tap (cin a
// multiple of 32), operands that fit the LDS, and addresses that allow its
// 16-byte loads and the 8-byte accesses to mask and output (conv3x3_kernel
// goes through those one value at a time).  The block follows the
// shape; us for pixels x channels (wavefronts, tiles per wavefront):
//   32 input channels: the stages are short, so each takes 256 pixels: 32 ->
//     96 at 16 x 136 x 136 41 with 256 x 32, 52 with 128 x 32;
//   up to 96: 128 x 32, the weights of three taps per stage: 64 -> 64 at 68 x
//     68 15.4 against 16.9 (256 x 32) and 17.7 (one tap per stage);
//   more: 64 x 64, one tap per stage: 128 -> 128 at 34 x 34 16.5 against 18.8
//     (128 x 32); 192 -> 64 at 68 x 68 42 / 45;
//   fewer than two such blocks per compute unit: 64 x 32: 256 -> 256 at 17 x
//     17 19.7 against 22.3;
//   cout not a multiple of 32: 256 x 16 (32 -> 16 at 136 x 136: 14.3, and
//     23.0 with conv3x3_kernel).
bool conv3x3_lds(const ConvArgs& a, hipStream_t s) {
    if (a.cin % 32 || 18.0 * a.cin * a.cout > 4.0e9) return false;
    if (!aligned16(a.x) || !aligned16(a.wt) || (uintptr_t)a.mask % 8 || (uintptr_t)a.y % 8) return false;
    const uint32_t taps = a.cin <= 96 ? 3 : 1;
    if (a.cout % 32) return conv3x3_lds_go<4, 1, 4, 1>(a, taps, s) || conv3x3_lds_go<4, 1, 1, 1>(a, 1, s);
    const uint64_t few = 512, wide = ((uint64_t)a.P + 255) / 256 * ((uint32_t)a.cout / 32);
    if (a.cin == 32 && wide >= few && conv3x3_lds_go<4, 1, 4, 2>(a, taps, s)) return true;
    if (a.cin <= 96 && 2 * wide >= few && conv3x3_lds_go<4, 1, 2, 2>(a, taps, s)) return true;
    if (a.cout % 64 == 0 && 2 * wide >= few && conv3x3_lds_go<2, 2, 2, 2>(a, taps, s)) return true;
    return conv3x3_lds_go<2, 2, 2, 1>(a, taps, s);
}

}  // namespace

extern "C" {

const char* lbm_nn_last_error(void) { return g_nn_err; }

// y = act(conv(x, wt) + bias), 0 where mask is not positive
static lbm_status conv3x3(const uint16_t* x, int32_t n, int32_t h, int32_t w, int32_t cin, const uint16_t* wt,
                          const float* bias, const uint16_t* mask, int32_t cout, int32_t relu, uint16_t* y,
                          void* stream) {
    if (!x || !wt || !y) return nn_fail(LBM_E_INVALID, "conv3x3: null tensor");
    if (!pos(n) || !pos(h) || !pos(w) || !pos(cin) || !pos(cout) || cin % 16 || cout % 16)
        return nn_fail(LBM_E_INVALID, "conv3x3: bad shape n=%d h=%d w=%d cin=%d cout=%d", n, h, w, cin, cout);
    const double P = (double)n * h * w;
    if (P * (cin > cout ? cin : cout) > 4.0e9) return nn_fail(LBM_E_INVALID, "conv3x3: tensor too large");
    ConvArgs a{x, wt, bias, mask, y, n, h, w, cin, cout, relu, (uint32_t)P, (uint32_t)((P + 15) / 16), 0};
    if (conv3x3_lds(a, (hipStream_t)stream)) return launched("conv3x3");
    const int NT = cout % 64 == 0 ? 4 : cout % 32 == 0 ? 2 : 1;
    // pixel tiles per wavefront: as many as keep at least 4096 wavefronts
    // (16 per compute unit) in the launch
    const size_t waves1 = (size_t)a.ptiles * (cout / (16 * NT));
    const int MT = waves1 >= 4 * 4096 ? 4 : waves1 >= 2 * 4096 ? 2 : 1;
    const size_t waves = ((size_t)a.ptiles + MT - 1) / MT * (cout / (16 * NT));
    const dim3 grid((unsigned)((waves + 3) / 4)), block(256);
    hipStream_t s = (hipStream_t)stream;
    auto go = [&](auto ntc, auto mtc) {
        hipLaunchKernelGGL((conv3x3_kernel<decltype(ntc)::value, decltype(mtc)::value>), grid, block, 0, s, a);
    };
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I4 = std::integral_constant<int, 4>;
    auto by_mt = [&](auto ntc) {
        if (MT == 4) go(ntc, I4{});
        else if (MT == 2) go(ntc, I2{});
        else go(ntc, I1{});
    };
    if (NT == 4) by_mt(I4{});
    else if (NT == 2) by_mt(I2{});
    else by_mt(I1{});
    return launched("conv3x3");
}

lbm_status lbm_nn_conv3x3(const uint16_t* x, int32_t n, int32_t h, int32_t w, int32_t cin, const uint16_t* wt,
                          const float* bias, int32_t cout, int32_t relu, uint16_t* y, void* stream) {
    return conv3x3(x, n, h, w, cin, wt, bias, nullptr, cout, relu, y, stream);
}

lbm_status lbm_nn_conv3x3_masked(const uint16_t* x, int32_t n, int32_t h, int32_t w, int32_t cin, const uint16_t* wt,
                                 const uint16_t* mask, int32_t cout, uint16_t* y, void* stream) {
    if (!mask) return nn_fail(LBM_E_INVALID, "conv3x3_masked: null mask");
    return conv3x3(x, n, h, w, cin, wt, nullptr, mask, cout, 0, y, stream);
}

lbm_status lbm_nn_conv3x3_flip_many(int32_t count, const uint16_t* const* wt, const int32_t* cin, const int32_t* cout,
                                    uint16_t* const* wf, void* stream) {
    if (count < 0 || (count && (!wt || !cin || !cout || !wf)))
        return nn_fail(LBM_E_INVALID, "conv3x3_flip: bad arguments");
    for (int32_t k = 0; k < count; ++k)
        if (!wt[k] || !wf[k] || !pos(cin[k]) || !pos(cout[k]))
            return nn_fail(LBM_E_INVALID, "conv3x3_flip: bad arguments");
    for (int32_t k0 = 0; k0 < count; k0 += kFlipMost) {
        FlipArgs a{};
        a.count = std::min(count - k0, kFlipMost);
        for (int32_t k = 0; k < a.count; ++k) {
            a.wt[k] = wt[k0 + k];
            a.wf[k] = wf[k0 + k];
            a.cin[k] = cin[k0 + k];
            a.cout[k] = cout[k0 + k];
            const uint64_t blocks = 9ull * (((uint64_t)a.cin[k] + 31) / 32) * (((uint64_t)a.cout[k] + 31) / 32);
            if (a.first[k] + blocks > 0x7fffffffull) return nn_fail(LBM_E_INVALID, "conv3x3_flip: layer too large");
            a.first[k + 1] = a.first[k] + (uint32_t)blocks;
        }
        hipLaunchKernelGGL(wflip_kernel, dim3(std::min(a.first[a.count], kMostBlocks)), dim3(256), 0, (hipStream_t)stream, a);
        const lbm_status st = launched("conv3x3_flip");
        if (st) return st;
    }
    return LBM_OK;
}

lbm_status lbm_nn_conv3x3_flip(const uint16_t* wt, int32_t cin, int32_t cout, uint16_t* wf, void* stream) {
    return lbm_nn_conv3x3_flip_many(1, &wt, &cin, &cout, &wf, stream);
}

lbm_status lbm_nn_conv3x3_wgrad(const uint16_t* x, const uint16_t* dz, int32_t n, int32_t h, int32_t w,
                                int32_t cin, int32_t cout, float* partial, int32_t chunks, float* dw, float* db,
                                void* stream) {
    if (!x || !dz || !partial || !dw) return nn_fail(LBM_E_INVALID, "conv3x3_wgrad: null tensor");
    if (!pos(n) || !pos(h) || !pos(w) || !pos(cin) || !pos(cout) || cin % 16 || cout % 16 || chunks < 1 ||
        chunks > 4096)
        return nn_fail(LBM_E_INVALID, "conv3x3_wgrad: bad shape");
    if (db && cout > 256) return nn_fail(LBM_E_INVALID, "conv3x3_wgrad: bias gradient needs cout <= 256");
    if (((uint64_t)h + 1) * (uint64_t)n > 0xfffffff0ull || h > 0x3fffff00)
        return nn_fail(LBM_E_INVALID, "conv3x3_wgrad: tensor too large");
    WGradArgs a{};
    a.x = x;
    a.dz = dz;
    a.partial = partial;
    a.n = n;
    a.h = h;
    a.w = w;
    a.cin = cin;
    a.cout = cout;
    hipStream_t s = (hipStream_t)stream;
    const size_t count = (size_t)9 * cout * cin;
    auto go = [&](auto wco, auto wci, auto wk, auto kx) {
        constexpr int WCO = decltype(wco)::value, WCI = decltype(wci)::value, WK = decltype(wk)::value,
                      KX = decltype(kx)::value;
        a.tiles_x = ((uint32_t)w + 8 * KX - 1) / (8 * KX);
        a.tiles_y = ((uint32_t)h + kWgTileH - 1) / kWgTileH;
        a.across = a.tiles_x == 1 ? (8 * KX + 1) / ((uint32_t)w + 1) : 1;
        a.cols = a.across > 1 ? a.across * ((uint32_t)w + 1) - 1 : (uint32_t)w;
        a.col_pitch = a.across > 1 ? (uint32_t)w + 1 : 0x7fffffffu;
        a.rows = ((uint32_t)n + a.across - 1) / a.across * ((uint32_t)h + 1) - 1;
        a.by_col_pitch = div31(a.col_pitch);
        a.by_pitch = div31((uint32_t)h + 1);
        // stacked where that saves three tiles in five: the place of a pixel
        // in it costs two divisions (us with tiles of each image's own /
        // stacked: 256 -> 256 channels at 16 x 34 x 34 58 / 71 in 27 % fewer, at
        // 512 x 8 x 8 82 / 94 in 44 % fewer; 32 -> 32 at 16 x 4 x 4 20 / 15 in 69 %)
        const uint64_t own = (uint64_t)n * a.tiles_y, stacked = ((uint64_t)a.rows + kWgTileH - 1) / kWgTileH;
        const bool stack = 5 * stacked <= 2 * own;
        a.tiles = a.tiles_x * (uint32_t)(stack ? stacked : own);
        // with a bias gradient the last chunk's place holds its partial sums
        // (9 cin >= 144 per channel), unless one chunk writes db itself
        uint32_t want = std::min<uint32_t>((uint32_t)chunks, a.tiles);
        if (db && chunks > 1) want = std::min<uint32_t>({want, (uint32_t)chunks - 1, 9u * (uint32_t)cin});
        a.per = (a.tiles + want - 1) / want;
        a.chunks = (a.tiles + a.per - 1) / a.per;
        a.bias = !db ? nullptr : a.chunks == 1 ? db : partial + (size_t)(chunks - 1) * count;
        a.partial = a.chunks == 1 ? dw : partial;  // one chunk: its sums are the result
        const uint32_t blocks = a.chunks * (uint32_t)((cout + 32 * WCO - 1) / (32 * WCO)) *
                                (uint32_t)((cin + 32 * WCI - 1) / (32 * WCI));
        const dim3 grid((blocks + 7) / 8 * 8);
        if (stack) hipLaunchKernelGGL((wgrad_kernel<WCO, WCI, WK, KX, true>), grid, dim3(256), 0, s, a);
        else hipLaunchKernelGGL((wgrad_kernel<WCO, WCI, WK, KX, false>), grid, dim3(256), 0, s, a);
    };
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I4 = std::integral_constant<int, 4>;
    // 64 channels share a staged tile where there are as many
    if (cout >= 64 && cin >= 64) go(I2{}, I2{}, I1{}, I1{});
    else if (cout >= 64) go(I2{}, I1{}, I2{}, I1{});
    else if (cin >= 64) go(I1{}, I2{}, I2{}, I1{});
    else go(I1{}, I1{}, I4{}, I2{});
    lbm_status st = launched("conv3x3_wgrad");
    if (st) return st;
    if (a.chunks == 1) return LBM_OK;
    const SumChunksArgs sa{partial, dw, count, a.chunks, a.bias, db, db ? (uint32_t)cout : 0u};
    const bool few = a.chunks <= 4;
    const size_t each = few ? 1024 : 64, blocks = (count + each - 1) / each + (sa.bias_count + each - 1) / each;
    const dim3 grid((unsigned)std::min<size_t>(blocks, kMostBlocks));
    if (few) hipLaunchKernelGGL(sum_chunks_kernel<1>, grid, dim3(256), 0, s, sa);
    else hipLaunchKernelGGL(sum_chunks_kernel<16>, grid, dim3(256), 0, s, sa);
    return launched("conv3x3_wgrad sum");
}

lbm_status lbm_nn_relu_backward(const uint16_t* y, const uint16_t* dy, uint16_t* dz, int64_t count, void* stream) {
    if (!y || !dy || !dz || count < 0) return nn_fail(LBM_E_INVALID, "relu_backward: bad arguments");
    const size_t groups = aligned16(y) && aligned16(dy) && aligned16(dz) ? (size_t)count / 8 : 0;
    const size_t threads = std::max<size_t>(groups, (size_t)count - groups * 8);
    hipLaunchKernelGGL(relu_backward_kernel, dim3(grid1(threads)), dim3(256), 0, (hipStream_t)stream, y, dy, dz,
                       groups, (size_t)count);
    return launched("relu_backward");
}

lbm_status lbm_nn_avgpool2(const uint16_t* x, int32_t n, int32_t h, int32_t w, int32_t c, uint16_t* y,
                           void* stream) {
    if (!x || !y || !pos(n) || !pos(h) || !pos(w) || !pos(c) || h % 2 || w % 2)
        return nn_fail(LBM_E_INVALID, "avgpool2: bad arguments");
    RowShape rows;
    dim3 grid;
    if (aligned16(x) && aligned16(y) && row_grid(n, h / 2, w / 2, c, &rows, &grid))
        hipLaunchKernelGGL(pool_kernel, grid, dim3(256), 0, (hipStream_t)stream, x, y, rows);
    else
        hipLaunchKernelGGL(avgpool2_kernel, dim3(grid1((size_t)n * h * w * c / 4)), dim3(256), 0, (hipStream_t)stream,
                           x, y, n, h, w, c);
    return launched("avgpool2");
}

lbm_status lbm_nn_avgpool2_backward(const uint16_t* dy, int32_t n, int32_t h, int32_t w, int32_t c, uint16_t* dx,
                                    void* stream) {
    if (!dy || !dx || !pos(n) || !pos(h) || !pos(w) || !pos(c) || h % 2 || w % 2)
        return nn_fail(LBM_E_INVALID, "avgpool2_backward: bad arguments");
    RowShape rows;
    dim3 grid;
    if (aligned16(dy) && aligned16(dx) && row_grid(n, h, w, c, &rows, &grid))
        hipLaunchKernelGGL(pool_backward_kernel, grid, dim3(256), 0, (hipStream_t)stream, dy, (const uint16_t*)nullptr,
                           (const uint16_t*)nullptr, dx, rows, 0u, 0u);
    else
        hipLaunchKernelGGL(avgpool2_backward_kernel, dim3(grid1((size_t)n * h * w * c)), dim3(256), 0,
                           (hipStream_t)stream, dy, dx, n, h, w, c);
    return launched("avgpool2_backward");
}

lbm_status lbm_nn_avgpool2_backward_add(const uint16_t* dy, int32_t n, int32_t h, int32_t w, int32_t c,
                                        const uint16_t* add, int32_t ca, int32_t aoff, const uint16_t* mask,
                                        uint16_t* dx, void* stream) {
    RowShape rows;
    dim3 grid;
    if (!dy || !dx || !pos(n) || !pos(h) || !pos(w) || !pos(c) || h % 2 || w % 2 ||
        (add && (!pos(ca) || ca % 8 || aoff < 0 || aoff % 8 || (int64_t)aoff + c > ca)) || !aligned16(dy) ||
        !aligned16(dx) || !aligned16(add) || !aligned16(mask) || !row_grid(n, h, w, c, &rows, &grid))
        return nn_fail(LBM_E_INVALID, "avgpool2_backward_add: bad arguments");
    hipLaunchKernelGGL(pool_backward_kernel, grid, dim3(256), 0, (hipStream_t)stream, dy, add, mask, dx, rows,
                       (uint32_t)ca, (uint32_t)aoff);
    return launched("avgpool2_backward_add");
}

lbm_status lbm_nn_upsample2(const uint16_t* x, int32_t n, int32_t h, int32_t w, int32_t c, uint16_t* y,
                            void* stream) {
    if (!x || !y || !pos(n) || !pos(h) || !pos(w) || !pos(c)) return nn_fail(LBM_E_INVALID, "upsample2: bad arguments");
    RowShape rows;
    dim3 grid;
    if (aligned16(x) && aligned16(y) && row_grid(n, 2 * (int64_t)h, 2 * (int64_t)w, c, &rows, &grid))
        hipLaunchKernelGGL(up_concat_kernel, grid, dim3(256), 0, (hipStream_t)stream, x, (const uint16_t*)nullptr, y,
                           rows, (uint32_t)c, 0u);
    else
        hipLaunchKernelGGL(upsample2_kernel, dim3(grid1((size_t)n * 4 * h * w * c)), dim3(256), 0, (hipStream_t)stream,
                           x, y, n, h, w, c);
    return launched("upsample2");
}

lbm_status lbm_nn_upsample2_concat(const uint16_t* x, int32_t n, int32_t h, int32_t w, int32_t cx, const uint16_t* skip,
                                   int32_t cs, uint16_t* y, void* stream) {
    RowShape rows;
    dim3 grid;
    if (!x || !skip || !y || !pos(n) || !pos(h) || !pos(w) || !pos(cx) || !pos(cs) || cx % 8 || cs % 8 ||
        !aligned16(x) || !aligned16(skip) || !aligned16(y) ||
        !row_grid(n, 2 * (int64_t)h, 2 * (int64_t)w, (int64_t)cx + cs, &rows, &grid))
        return nn_fail(LBM_E_INVALID, "upsample2_concat: bad arguments");
    hipLaunchKernelGGL(up_concat_kernel, grid, dim3(256), 0, (hipStream_t)stream, x, skip, y, rows,
                       (uint32_t)cx, (uint32_t)cs);
    return launched("upsample2_concat");
}

lbm_status lbm_nn_upsample2_backward(const uint16_t* dy, int32_t n, int32_t h, int32_t w, int32_t c, uint16_t* dx,
                                     void* stream) {
    if (!dy || !dx || !pos(n) || !pos(h) || !pos(w) || !pos(c))
        return nn_fail(LBM_E_INVALID, "upsample2_backward: bad arguments");
    RowShape rows;
    dim3 grid;
    if (aligned16(dy) && aligned16(dx) && row_grid(n, h, w, c, &rows, &grid))
        hipLaunchKernelGGL(up_backward_kernel, grid, dim3(256), 0, (hipStream_t)stream, dy, (const uint16_t*)nullptr,
                           dx, rows, (uint32_t)c);
    else
        hipLaunchKernelGGL(upsample2_backward_kernel, dim3(grid1((size_t)n * h * w * c)), dim3(256), 0,
                           (hipStream_t)stream, dy, dx, n, h, w, c);
    return launched("upsample2_backward");
}

lbm_status lbm_nn_upsample2_concat_backward(const uint16_t* dy, int32_t n, int32_t h, int32_t w, int32_t c, int32_t cd,
                                            const uint16_t* mask, uint16_t* dx, void* stream) {
    RowShape rows;
    dim3 grid;
    if (!dy || !dx || !pos(n) || !pos(h) || !pos(w) || !pos(c) || cd < c || cd % 8 || !aligned16(dy) ||
        !aligned16(dx) || !aligned16(mask) || !row_grid(n, h, w, c, &rows, &grid))
        return nn_fail(LBM_E_INVALID, "upsample2_concat_backward: bad arguments");
    hipLaunchKernelGGL(up_backward_kernel, grid, dim3(256), 0, (hipStream_t)stream, dy, mask, dx, rows, (uint32_t)cd);
    return launched("upsample2_concat_backward");
}

lbm_status lbm_nn_unet_forward(int32_t levels, const uint16_t* x, int32_t n, int32_t h, int32_t w, int32_t cin,
                               const int32_t* cout, const uint16_t* const* wt, const float* const* bias,
                               uint16_t* const* out, void* stream) {
    constexpr int32_t kMost = 32;
    if (!cout || !wt || !bias || !out || levels < 1 || levels > kMost)
        return nn_fail(LBM_E_INVALID, "unet_forward: bad arguments");
    const uint16_t* skip[kMost];
    int32_t skip_c[kMost], k = 0;
    const uint16_t* t = x;
    auto conv = [&](int32_t relu) {
        const lbm_status st = conv3x3(t, n, h, w, cin, wt[k], bias[k], nullptr, cout[k], relu, *out, stream);
        t = *out++;
        cin = cout[k++];
        return st;
    };
    lbm_status st = LBM_OK;
    for (int32_t l = 0; l < levels && !st; ++l) {
        if (l) {
            st = lbm_nn_avgpool2(t, n, h, w, cin, *out, stream);
            t = *out++;
            h /= 2, w /= 2;
        }
        if (!st) st = conv(1);
        if (!st) st = conv(1);
        skip[l] = t, skip_c[l] = cin;
    }
    for (int32_t l = levels - 2; l >= 0 && !st; --l) {
        st = lbm_nn_upsample2_concat(t, n, h, w, cin, skip[l], skip_c[l], *out, stream);
        t = *out++;
        h *= 2, w *= 2, cin += skip_c[l];
        if (!st) st = conv(1);
        if (!st) st = conv(1);
    }
    return st ? st : conv(0);
}

lbm_status lbm_nn_copy_channels(const uint16_t* src, int32_t cs, int32_t soff, uint16_t* dst, int32_t cd,
                                int32_t doff, int32_t cc, int64_t pixels, int32_t accumulate, void* stream) {
    if (!src || !dst || !pos(cs) || !pos(cd) || !pos(cc) || soff < 0 || doff < 0 || soff + cc > cs ||
        doff + cc > cd || pixels < 0)
        return nn_fail(LBM_E_INVALID, "copy_channels: bad arguments");
    const uint64_t items = (uint64_t)pixels * (uint32_t)(cc / 8);
    if (!((cs | soff | cd | doff | cc) % 8) && aligned16(src) && aligned16(dst) && items < 0x80000000ull)
        hipLaunchKernelGGL(copy_channels8_kernel, dim3(grid1((size_t)items)), dim3(256), 0, (hipStream_t)stream, src,
                           (uint32_t)cs, (uint32_t)soff, dst, (uint32_t)cd, (uint32_t)doff, (uint32_t)cc / 8,
                           (uint32_t)items, accumulate);
    else
        hipLaunchKernelGGL(copy_channels_kernel, dim3(grid1((size_t)pixels * cc)), dim3(256), 0, (hipStream_t)stream,
                           src, cs, soff, dst, cd, doff, cc, (size_t)pixels, accumulate);
    return launched("copy_channels");
}

lbm_status lbm_nn_mse(const uint16_t* y, int32_t cy, const float* target, const float* mask, int64_t pixels,
                      int32_t used, double count, uint16_t* dy, float* loss, float* scratch, void* stream) {
    if (!y || !target || !mask || !loss || !scratch || !pos(cy) || !pos(used) || used > cy || pixels < 0 ||
        !(count > 0))
        return nn_fail(LBM_E_INVALID, "mse: bad arguments");
    const unsigned grid = grid1((size_t)pixels * cy, 256, 1024);
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(mse_kernel, dim3(grid), dim3(256), 0, s, y, cy, target, mask, (size_t)pixels, used,
                       (float)(1.0 / count), dy, scratch);
    lbm_status st = launched("mse");
    if (st) return st;
    hipLaunchKernelGGL(sum_partials_kernel, dim3(1), dim3(256), 0, s, (const float*)scratch, (int32_t)grid,
                       (float)(1.0 / count), loss);
    return launched("mse sum");
}

lbm_status lbm_nn_adam(float* w, const float* g, float* m, float* v, int64_t count, float lr, float beta1,
                       float beta2, float eps, int32_t step, uint16_t* w_bf16, void* stream) {
    if (!w || !g || !m || !v || count < 0 || step < 1) return nn_fail(LBM_E_INVALID, "adam: bad arguments");
    const float c1 = 1.0f - powf(beta1, (float)step), c2 = 1.0f - powf(beta2, (float)step);
    hipLaunchKernelGGL(adam_kernel, dim3(grid1((size_t)count)), dim3(256), 0, (hipStream_t)stream, w, g, m, v,
                       (size_t)count, lr, beta1, beta2, eps, c1, c2, w_bf16);
    return launched("adam");
}

lbm_status lbm_nn_to_bf16(const float* src, uint16_t* dst, int64_t count, void* stream) {
    if (!src || !dst || count < 0) return nn_fail(LBM_E_INVALID, "to_bf16: bad arguments");
    hipLaunchKernelGGL(f32_to_bf16_kernel, dim3(grid1((size_t)count)), dim3(256), 0, (hipStream_t)stream, src, dst,
                       (size_t)count);
    return launched("to_bf16");
}

lbm_status lbm_nn_to_f32(const uint16_t* src, float* dst, int64_t count, void* stream) {
    if (!src || !dst || count < 0) return nn_fail(LBM_E_INVALID, "to_f32: bad arguments");
    hipLaunchKernelGGL(bf16_to_f32_kernel, dim3(grid1((size_t)count)), dim3(256), 0, (hipStream_t)stream, src, dst,
                       (size_t)count);
    return launched("to_f32");
}

}  // extern "C"

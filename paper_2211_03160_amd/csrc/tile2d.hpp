// tile2d.hpp -- several time steps per launch through LDS tiles (2D).
//
// A block of RX x RY threads holds a region of RX x RY nodes, one node per
// thread, and advances it K steps.  Step 1 gathers from global memory (the
// one-step kernel's pull and wall rules), so it is valid on the whole region;
// every further step pulls the 12 moving populations of its neighbours from
// one LDS buffer (the node's own ones stay in registers) and is valid one
// node further inside; step K stores the inner (RX - 2 (K - 1)) x (RY - 2 (K
// - 1)) nodes.  Every node update is step_node on the same (storage-rounded)
// values as a one-step launch, so results are bitwise those of single steps.
//
// The register-row kernel (stream_kernel) walks a wavefront down the rows of a
// segment plus 3 NS rows of pipeline fill, a serial chain of 60 to 100 us, and
// leaves most of the chip idle below about 2000 units.  Here a launch is K
// collisions deep whatever the grid, and a wavefront holds no rings: 56
// registers in FP32, so 8 wavefronts per SIMD cover the barriers.
#pragma once

namespace lbm {

template <class St> struct Tile2Args {
    const typename St::TF* fsrc;
    const typename St::TG* gsrc;
    typename St::TF* fdst;
    typename St::TG* gdst;
    double* flux;       // wall heat flux area: two slots, faces back to back
    uint32_t slot[2];   // first element of flux slot 0 and slot 1
    int32_t t_parity;   // (t of the input state) mod 2: step j writes slot (t + j) mod 2
    int32_t steps;      // K, 2 .. 5
    uint32_t tiles_x, tiles;
    uint32_t blocks_per_xcd;
    Geometry geo;
    Coef<typename St::R> c;
};

// pull source of steps 2 .. K: moving population i of the region in LDS plane
// i - 1 (f) or 7 + i (g) of N nodes, `lds` at the thread's own node; the
// node's own populations (at rest, and across a wall) in registers
template <class St, int N, int RX> struct TileSrc {
    using R = typename St::R;
    const R* lds;
    const R (&f)[9];
    const R (&g)[5];
    template <int i, int ex, int ey, int ez, int o> __device__ R pull_f(bool out) const {
        if constexpr (i == 0) return f[0];
        else return out ? f[o] : lds[(i - 1) * N - ex - ey * RX];
    }
    template <int i, int ex, int ey, int ez, int o> __device__ R pull_g(bool out) const {
        if constexpr (i == 0) return g[0];
        else return out ? g[o] : lds[(7 + i) * N - ex - ey * RX];
    }
};

// a step's result into registers and LDS, decoded after rounding through the
// storage type (what a single step would store and reload)
template <class St, int N> struct TileDst {
    using R = typename St::R;
    R* lds;
    R (&f)[9];
    R (&g)[5];
    __device__ void sf(int i, typename St::TF v) const {
        f[i] = St::EF::dec(v);
        if (i > 0) lds[(i - 1) * N] = f[i];
    }
    __device__ void sg(int i, typename St::TG v) const {
        g[i] = St::EG::dec(v);
        if (i > 0) lds[(7 + i) * N] = g[i];
    }
};

// wall heat flux of an owned node (2D: four faces back to back in one slot)
struct TileFlux {
    double* slot;
    bool on;
    template <int face> __device__ void put(const Geometry& g, uint32_t local, double v, bool wall) const {
        constexpr bool in2d = face < 4;
        if (in2d && on && wall)
            slot[(face == 0 ? 0u : face == 1 ? g.ny : face == 2 ? 2u * g.ny : 2u * g.ny + g.nx) + local] = v;
    }
};

// One block's K steps, with (Walls) or without wall rules, from the state of
// parity tp.  With Report, returns false on a thread that computed, at any
// step, a node of the domain from valid sources whose new rho or T is not
// finite or whose speed exceeds the lattice sound speed.
template <class St, int RX, int RY, int KT, bool Walls, bool Report>
__device__ __forceinline__ bool tile2_steps(const Tile2Args<St>& a, typename St::R* lds, int32_t x0, int32_t y0,
                                            int32_t tp) {
    using R = typename St::R;
    using L = Flow<2>;
    using H = Heat<2>;
    constexpr int QF = L::Q, QG = H::Q, N = RX * RY;
    const Geometry& g = a.geo;
    const int K = KT > 0 ? KT : a.steps;
    const int tx = (int)(threadIdx.x % RX), ty = (int)(threadIdx.x / RX);
    // this thread's node, unwrapped, and its domain coordinates (a stand-in
    // inside the domain beyond a wall: never read by a node of the domain)
    const int32_t cx = x0 + tx, cy = y0 + ty;
    const int32_t rx = region_coord(cx, g.nx, g.periodic[0]), ry = region_coord(cy, g.ny, g.periodic[1]);
    const uint32_t x = (uint32_t)(rx >= 0 ? rx : min(max(cx, 0), (int32_t)g.nx - 1));
    const uint32_t y = (uint32_t)(ry >= 0 ? ry : min(max(cy, 0), (int32_t)g.ny - 1));
    const bool own = tx >= K - 1 && tx <= RX - K && ty >= K - 1 && ty <= RY - K && cx < (int32_t)g.nx &&
                     cy < (int32_t)g.ny;
    // the rows of this wavefront: it skips a step none of whose valid rows
    // (j - 1 .. RY - j) it holds
    const int wy0 = (int)__builtin_amdgcn_readfirstlane(ty), wy1 = wy0 + 64 / RX - 1;
    const uint32_t idx = x + g.nx * y;
    const Neighbours nb = neighbours(g, x, y, 0);
    R* mine = lds + (RX + 1) + threadIdx.x;  // a margin takes the edge threads' reads
    R f[QF], h[QG];
    // a slot keeps the last step of its parity: only steps K - 1 and K write
    auto flux = [&](int j) { return TileFlux{a.flux + a.slot[(tp + j) & 1], own && j >= K - 1}; };
    // the last step at which this thread's node is valid (0: none)
    const int edge = min(min(tx, RX - 1 - tx), min(ty, RY - 1 - ty));
    const int valid = Report && rx >= 0 && ry >= 0 ? edge + 1 : 0;
    bool bad = false;
    {
        const bool ok = step_node<2, St, Walls>(g, a.c, nb, x, y, 0u,
                                                global_src<St, QF, QG>(g, nb, a.fsrc, a.gsrc, idx),
                                                TileDst<St, N>{mine, f, h}, flux(1));
        if constexpr (Report) bad = !ok && valid >= 1;
    }
    auto middle = [&](const int j) __attribute__((always_inline)) {
        const bool need = wy1 >= j - 1 && wy0 <= RY - j;
        R pf[QF], pg[QG];  // the pull of step j, read before any thread overwrites step j - 1
        __syncthreads();
        if (need) {
            const TileSrc<St, N, RX> src{mine, f, h};
            auto out = [&](int ex, int ey) {
                return Walls && ((ex > 0 && !nb.okxm) || (ex < 0 && !nb.okxp) || (ey > 0 && !nb.okym) ||
                                 (ey < 0 && !nb.okyp));
            };
            static_for<0, QF>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                pf[i] = src.template pull_f<i, L::ex[i], L::ey[i], 0, L::opp[i]>(out(L::ex[i], L::ey[i]));
            });
            static_for<0, QG>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                pg[i] = src.template pull_g<i, H::ex[i], H::ey[i], 0, H::opp[i]>(out(H::ex[i], H::ey[i]));
            });
        }
        __syncthreads();
        if (need) {
            const bool ok = step_node<2, St, Walls>(g, a.c, nb, x, y, 0u, PreSrc<St, QF, QG>{pf, pg},
                                                    TileDst<St, N>{mine, f, h}, flux(j));
            if constexpr (Report) bad = bad || (!ok && valid >= j);
        }
    };
    if constexpr (KT > 0) {
        static_for<2, KT>([&](auto jc) { middle(decltype(jc)::value); });
    } else {
        for (int j = 2; j < K; ++j) middle(j);
    }
    __syncthreads();
    if (own) {
        const bool ok = step_node<2, St, Walls>(g, a.c, nb, x, y, 0u, TileSrc<St, N, RX>{mine, f, h},
                                                GlobalDst<St, QF, QG, false, false>(a.fdst, a.gdst, idx), flux(K));
        if constexpr (Report) bad = bad || !ok;
    }
    return !bad;
}

// tile `tile` of a
template <class St, int RX, int RY, int KT, bool Report>
__device__ __forceinline__ bool tile2_tile(const Tile2Args<St>& a, typename St::R* lds, uint32_t tile, int32_t tp) {
    const Geometry& g = a.geo;
    const int32_t halo = (KT > 0 ? KT : a.steps) - 1;
    const int32_t x0 = (int32_t)(tile % a.tiles_x) * (RX - 2 * halo) - halo;
    const int32_t y0 = (int32_t)(tile / a.tiles_x) * (RY - 2 * halo) - halo;
    // a region that stays one node clear of every wall runs without wall rules
    const bool inner_x = g.periodic[0] || (x0 >= 1 && x0 + RX - 1 <= (int32_t)g.nx - 2);
    const bool inner_y = g.periodic[1] || (y0 >= 1 && y0 + RY - 1 <= (int32_t)g.ny - 2);
    if (inner_x && inner_y) return tile2_steps<St, RX, RY, KT, false, Report>(a, lds, x0, y0, tp);
    return tile2_steps<St, RX, RY, KT, true, Report>(a, lds, x0, y0, tp);
}

template <int RX, int RY> constexpr int tile2_lds() { return 12 * RX * RY + 2 * (RX + 1); }

template <class St, int RX, int RY, int KT> __global__ __launch_bounds__(RX* RY) void tile2_kernel(Tile2Args<St> a) {
    __shared__ typename St::R lds[tile2_lds<RX, RY>()];
    const uint32_t blk = logical_block(a.blocks_per_xcd);
    if (blk >= a.tiles) return;  // whole block
    tile2_tile<St, RX, RY, KT, false>(a, lds, blk, a.t_parity);
}

// Many 2D cavities: block b takes tile b of the concatenated tiles of all
// cavities, which tile_cavity maps to its cavity.
template <class St> struct BatchTile2Args {
    const Tile2Args<St>* desc;    // [2][count]: the cavities' arguments with buffer A, B as source
    const uint16_t* tile_cavity;  // [tiles]
    const uint32_t* tile0;        // [count] first tile of each cavity
    uint32_t tiles, count, blocks_per_xcd;
    int32_t src;                  // source buffer of this launch
    int32_t t_parity;             // (t of the input state) mod 2
    int32_t* unstable;            // per-cavity flag, set on a non-finite node
};

template <class St, int RX, int RY, int KT>
__global__ __launch_bounds__(RX* RY) void batch_tile2_kernel(BatchTile2Args<St> b) {
    __shared__ typename St::R lds[tile2_lds<RX, RY>()];
    const uint32_t blk = logical_block(b.blocks_per_xcd);
    if (blk >= b.tiles) return;  // whole block
    const uint32_t k = b.tile_cavity[blk];
    // through the constant address space, like the streaming kernel's
    using CArgs = const __attribute__((address_space(4))) Tile2Args<St>;
    const Tile2Args<St>& a = *(const Tile2Args<St>*)((CArgs*)b.desc + ((uint32_t)b.src * b.count + k));
    if (!tile2_tile<St, RX, RY, KT, true>(a, lds, blk - b.tile0[k], b.t_parity)) b.unstable[k] = 1;
}

}  // namespace lbm

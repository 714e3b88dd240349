// D2Q9 passes of T steps (T >= 2) over tiles kept in LDS.
//
// A workgroup owns a core of cols x rows nodes and works on the region that
// reaches T - 1 nodes further on every side (at most W x H nodes).  The
// first step of the region pulls from HBM, the last stores the core; the
// steps between pass through LDS in the storage type, exactly as they would
// through HBM, and each is done on a region one node smaller on every side,
// so a pass equals T launches of k_step bit for bit.
//
// One copy of the region's nine populations is enough: a step writes each
// value where it read one, so that no node's write meets another node's
// read and one barrier per step orders them.  After an odd step slot i of a
// node holds its own post-collision h*_i.  An even step pulls h_i from slot i
// of node x - e_i and leaves h*_ibar there; the next odd step finds its h_i
// in its own slot ibar and leaves h*_i in slot i.  With a solid source (or
// the inlet wall) the even step uses its own slot ibar in place of the
// source's slot i: the value that bounces back, and the place where the
// following odd step looks for it.  Lanes and rows past a
// step's region compute values that no later step of the core reads, in
// slots of their own (the slot map is one to one on the linear node index),
// so no lane is masked before the last store.
//
// What bounds it and why this shape: instruction issue.  A wave updates a
// row of 64 nodes with about 105 VALU instructions, 9 LDS reads and 9 LDS
// writes with compile-time offsets from one address register.  At 2048^2 the
// SIMDs spend as many quads of clocks on VALU instructions as a pass takes in
// FP32 (107 % of the busy clocks), 77 % of them in FP64, whose registers
// leave four waves per SIMD; HBM moves 1.05 times the state in and out per
// pass (FP64 1.18: halos of narrower regions).  Two workgroups per CU, one computing while the other waits for its first
// step's loads.  Measured against the passes of two steps along rows
// (k_step2_2d; us a step, before -> after): 2048^2 FP32 36.7 -> 17.7,
// FP64 64.8 -> 36.5; 4096^2 FP32 156 -> 71, FP16 (one step a pass before)
// 94 -> 78; 509 x 381 FP32 3.69 -> 1.70; 64^2 FP64 2.32 -> 0.93; 512
// lattices of 32 to 512 nodes a side FP32 407 -> 178.
#pragma once

#include "step2.hpp"

namespace ptrt {

// Region of W x H nodes, NW waves.  A: lattices with more tiles than CUs
// (16-wave workgroups, two per CU in FP32); B: the same for FP64, whose
// registers allow 16 waves per CU; C, D: small lattices, where a pass is a
// chain of T dependent steps and short chains of more, smaller tiles win.
template <int W_, int H_, int NW_>
struct TileShape {
    static constexpr int W = W_, H = H_, NW = NW_;
    // an even step's slots reach W + 1 elements before and after the region
    static constexpr int PAD = W + 8;
    static constexpr int PLANE = W * H + PAD;
    static constexpr int elems = 9 * PLANE + PAD;
};
using TileA = TileShape<64, 32, 16>;
using TileB = TileShape<32, 32, 8>;
using TileC = TileShape<32, 24, 12>;
using TileD = TileShape<32, 16, 8>;

// One tile, run by the workgroup.  FLAGS: the tile reads the mask (null:
// no solids) and, with OPEN, may meet an open x boundary (x not periodic, as
// pull<..., OPEN>); fl then holds per node of the region bit 0 for a node
// that is solid or outside an open lattice, and bit i where population i
// bounces back.
template <class S, class SH, int FORCING, bool FLAGS, bool OPEN>
__device__ __forceinline__ void
tile_2d_task(const S *__restrict__ src, S *__restrict__ dst, const uint8_t *__restrict__ mask,
             const uint8_t *__restrict__ near, const Geom &g,
             const Coef<D2Q9, typename Codec<S>::compute> &r, S *lds, uint16_t *fl, int x0, int y0,
             int cols, int core_rows, int T)
{
    using L = D2Q9;
    using C = typename Codec<S>::compute;
    static_assert(FLAGS || !OPEN, "open boundaries need the flags");
    constexpr int W = SH::W, NW = SH::NW, PLANE = SH::PLANE, B = SH::PAD;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = (int)(threadIdx.x & 63);
    const int col = lane & (W - 1);
    const int halo = T - 1, rows = core_rows + 2 * halo;
    auto mod = [](int v, int n) {
        v %= n;
        return v < 0 ? v + n : v;
    };
    const int xr = x0 - halo + col; // not wrapped
    const int x = mod(xr, g.nx);
    const bool out_x = OPEN && (xr < 0 || xr >= g.nx);
    auto row_of = [&](int n0) { return W == 64 ? n0 >> 6 : (n0 + lane) / W; };
    auto open_fix = [&](C(&h)[L::Q]) {
        if constexpr (OPEN) {
            if (xr == 0)
                static_for<L::Q>([&](auto ic) {
                    constexpr int i = decltype(ic)::value;
                    if constexpr (L::ex(i) == 1) h[i] = h[i] + C(6.0 * L::w(i)) * C(g.uin);
                });
            if (xr == g.nx - 1) zou_he_east(h, C(g.drhoout));
        }
    };
    // v: the result in the storage type, rounded right behind the collision
    // (in FP16 the compiler fuses that rounding with the last multiply-add,
    // here as in the one-step kernel; behind a branch it would not)
    auto update = [&](C(&h)[L::Q], S(&v)[L::Q]) {
        open_fix(h);
        C rho, ux, uy, uz;
        collide<L, C, true, FORCING, Codec<S>::fast_recip>(h, r, rho, ux, uy, uz);
        static_for<L::Q>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            Codec<S>::template store<false>(&v[i], h[i]);
        });
    };

    // first step, from HBM; f: the row's flags
    auto load_row = [&](int n0, S (&raw)[L::Q], unsigned &f) __attribute__((always_inline)) {
        const int y = mod(y0 - halo + row_of(n0), g.ny);
        if constexpr (FLAGS) {
            const Nbr nb(g, x, y, 0);
            f = out_x ? 1u : 0u;
            // the mask is read in rows that hold or pull from a solid only
            const bool near_row = mask && (W == 64 ? near[y] != 0 : __any(near[y] != 0));
            auto pull_row = [&](auto mc) __attribute__((always_inline)) {
                constexpr bool M = decltype(mc)::value;
                if (M && mask[(size_t)y * (unsigned)g.nx + (unsigned)x]) f |= 1u;
                static_for<L::Q>([&](auto ic) {
                    constexpr int i = decltype(ic)::value;
                    if constexpr (i == 0) {
                        raw[0] = *at(src, g, 0, (unsigned)y, x);
                    } else {
                        int sx;
                        unsigned srow;
                        source_of<L, i>(g, nb, x, y, 0, sx, srow);
                        bool back = M && mask[(size_t)srow * (unsigned)g.nx + (unsigned)sx] != 0;
                        if constexpr (OPEN && L::ex(i) == 1) back = back || xr == 0;
                        if (back) f |= 1u << i;
                        raw[i] = *(back ? at(src, g, L::opp(i), (unsigned)y, x) : at(src, g, i, srow, sx));
                    }
                });
            };
            if (near_row)
                pull_row(std::true_type{});
            else
                pull_row(std::false_type{});
        } else {
            pull<L, S, false>(src, mask, g, x, y, 0, raw, [](const S *p) { return *p; });
        }
    };
    auto first = [&](int n0, const S (&raw)[L::Q], unsigned f) __attribute__((always_inline)) {
        if constexpr (FLAGS) fl[n0 + lane] = (uint16_t)f;
        C h[L::Q];
        S v[L::Q];
        static_for<L::Q>([&](auto ic) { h[decltype(ic)::value] = Codec<S>::load(&raw[decltype(ic)::value]); });
        update(h, v);
        static_for<L::Q>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            lds[i * PLANE + B + n0 + lane] = v[i];
        });
    };
    const int end = rows * W;
    S ra[L::Q];
    unsigned fa = 0;
    int n0 = w * 64;
    if constexpr (FLAGS) {
        for (; n0 < end; n0 += NW * 64) {
            load_row(n0, ra, fa);
            first(n0, ra, fa);
        }
    } else {
        // the loads of a wave's next row are in flight while a row collides:
        // 2048^2 FP64 40.2 -> 38.9 us a step, FP32 18.3 -> 17.6 (in the tiles
        // with flags their registers spill)
        S rb[L::Q];
        unsigned fb = 0;
        if (n0 < end) load_row(n0, ra, fa);
        for (; n0 < end; n0 += 2 * NW * 64) {
            const int n1 = n0 + NW * 64, n2 = n1 + NW * 64;
            if (n1 < end) load_row(n1, rb, fb);
            first(n0, ra, fa);
            if (n2 < end) load_row(n2, ra, fa);
            if (n1 < end) first(n1, rb, fb);
        }
    }
    // step s on rows s - 1 ... rows - s of the region; EVEN: s is even
    auto step = [&](auto ec, int s) __attribute__((always_inline)) {
        constexpr bool EVEN = decltype(ec)::value;
        const int end = rows - s + 1;
        for (int n0 = (s - 1) * W + w * 64; n0 < end * W; n0 += NW * 64) {
            const int n = n0 + lane;
            unsigned f = 0;
            if constexpr (FLAGS) f = fl[n];
            auto row = [&](auto bc) __attribute__((always_inline)) {
                constexpr bool BACK = decltype(bc)::value;
                // slot of h_i (and, after an even step, of h*_ibar)
                auto slot = [&](auto ic) {
                    constexpr int i = decltype(ic)::value;
                    constexpr int own = L::opp(i) * PLANE;
                    if constexpr (!EVEN) return own + B + n;
                    constexpr int from = i * PLANE - (L::ey(i) * W + L::ex(i));
                    if constexpr (BACK && i != 0) return ((f >> i) & 1u ? own : from) + B + n;
                    return from + B + n;
                };
                C h[L::Q];
                static_for<L::Q>([&](auto ic) { h[decltype(ic)::value] = Codec<S>::load(&lds[slot(ic)]); });
                S v[L::Q];
                update(h, v);
                if (s == T) {
                    const int rr = row_of(n0);
                    if (col >= halo && col < halo + cols && rr < end && !(BACK && (f & 1u)))
                        static_for<L::Q>([&](auto ic) {
                            constexpr int i = decltype(ic)::value;
                            *at(dst, g, i, (unsigned)(y0 + rr - halo), x) = v[i];
                        });
                } else if (!(BACK && (f & 1u))) {
                    static_for<L::Q>([&](auto ic) {
                        constexpr int i = decltype(ic)::value;
                        if constexpr (EVEN)
                            lds[slot(std::integral_constant<int, L::opp(i)>{})] = v[i];
                        else
                            lds[i * PLANE + B + n] = v[i];
                    });
                }
            };
            if constexpr (FLAGS) {
                if (__any(f != 0)) {
                    row(std::true_type{});
                    continue;
                }
            }
            row(std::false_type{});
        }
    };
    for (int s = 2; s <= T; ++s) {
        lds_barrier();
        if (s & 1)
            step(std::false_type{}, s);
        else
            step(std::true_type{}, s);
    }
}

// Waves per SIMD: 64 VGPRs suffice for FP32 arithmetic; FP64 and the
// stochastic rounding of nine stores take up to 128.
template <class S>
constexpr int tile_waves_per_simd =
    sizeof(S) == 8 || std::is_same<S, f16sr_t>::value || std::is_same<S, bf16sr_t>::value ? 4 : 8;

// A lattice of a batch: its blocks of the shared state, mask and near-row
// arrays, its layout and its constants.
template <class C>
struct BInst {
    long long off, moff, noff; // populations, mask and near-solid row flags
    Geom g;
    Coef<D2Q9, C> r;
};

// One lattice: tile t of tiles_x columns of cw x ch cores.  special[t] != 0
// (null: none): the tile's region holds or pulls from a solid, or meets an
// open x boundary.  Compiling both kinds of tile into one kernel costs the
// plain ones nothing (FP32 64 VGPRs instead of 42, FP64 96 instead of 88:
// the same waves per SIMD).
template <class S, class SH, int FORCING, bool OPEN>
__global__ void __launch_bounds__(64 * SH::NW)
__attribute__((amdgpu_waves_per_eu(tile_waves_per_simd<S>, tile_waves_per_simd<S>)))
k_tile_2d(const S *__restrict__ src, S *__restrict__ dst, const uint8_t *__restrict__ mask,
          const uint8_t *__restrict__ near, const uint8_t *__restrict__ special, Geom g,
          Coef<D2Q9, typename Codec<S>::compute> r, int T, int cw, int ch, int tiles_x)
{
    __shared__ S lds[SH::elems];
    __shared__ uint16_t fl[SH::W * SH::H];
    int t, unused_y, unused_z;
    xcd_block(t, unused_y, unused_z);
    const int ty = t / tiles_x, tx = t - ty * tiles_x;
    const int x0 = tx * cw, y0 = ty * ch;
    const int cols = min(cw, g.nx - x0), rows = min(ch, g.ny - y0);
    if (special && special[t])
        tile_2d_task<S, SH, FORCING, true, OPEN>(src, dst, mask, near, g, r, lds, fl, x0, y0, cols, rows,
                                                T);
    else
        tile_2d_task<S, SH, FORCING, false, false>(src, dst, mask, near, g, r, lds, fl, x0, y0, cols,
                                                   rows, T);
}

// Many lattices: workgroup t runs tasks[t] = {instance, x0, y0, cols | rows
// << 15 | special << 30} on its instance's block of the state and mask.
template <class S, class SH>
__global__ void __launch_bounds__(64 * SH::NW)
__attribute__((amdgpu_waves_per_eu(tile_waves_per_simd<S>, tile_waves_per_simd<S>)))
k_batch_tile(const S *__restrict__ src, S *__restrict__ dst, const uint8_t *__restrict__ mask,
             const uint8_t *__restrict__ near, const BInst<typename Codec<S>::compute> *__restrict__ inst,
             const int4 *__restrict__ tasks, int T)
{
    __shared__ S lds[SH::elems];
    __shared__ uint16_t fl[SH::W * SH::H];
    int t, unused_y, unused_z;
    xcd_block(t, unused_y, unused_z);
    const int4 tk = tasks[t];
    const BInst<typename Codec<S>::compute> p = inst[tk.x];
    const int cols = tk.w & 0x7fff, rows = (tk.w >> 15) & 0x7fff;
    if (tk.w >> 30)
        tile_2d_task<S, SH, FORCE_II, true, false>(src + p.off, dst + p.off, mask + p.moff,
                                                   near + p.noff, p.g, p.r, lds, fl, tk.y, tk.z, cols, rows, T);
    else
        tile_2d_task<S, SH, FORCE_II, false, false>(src + p.off, dst + p.off, mask + p.moff,
                                                    near + p.noff, p.g, p.r, lds, fl, tk.y, tk.z, cols, rows, T);
}

} // namespace ptrt

// Two fused steps per pass for D3Q19 without solids on lattices of any
// width, and on small ones (the counterpart of k_step2, which needs nx a
// multiple of 64 and many columns).
//
// A workgroup owns a column of cols (at most 62) x BY nodes and marches up a
// chunk of planes like k_step2, but a wave's row holds the halo columns too
// (lanes 0 ... cols + 1 are columns x0 - 1 ... x0 + cols): each of its BY + 2
// waves computes one row of first steps a plane, and BY of them the second
// step of their own row, with no separate halo task and one set of pulls
// per wave in flight.  FP32 100 registers, two workgroups per CU; FP64 190,
// one.  Bound by instruction issue (14 collisions for six rows of two steps,
// idle lanes past cols) and, on small lattices, by the chain of a chunk's
// planes, about 4 us each with two workgroups on a CU.  The strips start
// anywhere in a 128-byte line: plain stores, whose parts meet in L2 (the
// non-temporal ones of k_step2 measured up to 13 % slower here).
#pragma once

#include "step2.hpp"

namespace ptrt {

// Columns of a strip: near-equal strips of at most 62.
inline int march_cols(int nx)
{
    const int strips = (nx + 61) / 62;
    return (nx + strips - 1) / strips;
}

template <class S, int BY_>
struct MarchShape {
    static constexpr int W = 64, BY = BY_, AY = BY + 2, AP = AY * W;
    using K = Step2Classes<D3Q19, 2>;
    static constexpr int PAD = W; // sources of the garbage lanes 0 and 63
    static constexpr int elems = K::planes * AP + 2 * PAD;
};

template <class S, class SH>
__global__ void __launch_bounds__((64 * SH::AY))
__attribute__((amdgpu_waves_per_eu(sizeof(S) == 4 ? 4 : 2, sizeof(S) == 4 ? 4 : 2)))
k_march3d(const S *__restrict__ src, S *__restrict__ dst, Geom g,
          Coef<D3Q19, typename Codec<S>::compute> r, int zc, int cols)
{
    using L = D3Q19;
    using C = typename Codec<S>::compute;
    using K = typename SH::K;
    constexpr int W = SH::W, BY = SH::BY, AP = SH::AP;
    __shared__ S lds_all[SH::elems];
    S *const lds = lds_all + SH::PAD;
    int bx, by, bz;
    xcd_block(bx, by, bz);
    const int x0 = bx * cols, y0 = by * BY, zs = bz * zc, ze = min(zs + zc, g.nz);
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = (int)(threadIdx.x & 63);
    auto mod = [](int v, int n) {
        v %= n;
        return v < 0 ? v + n : v;
    };
    auto wrapz = [&](int k) { return k < 0 ? k + g.nz : (k >= g.nz ? k - g.nz : k); };
    // this lane's node in every plane (lanes past the halo repeat its last
    // column: their values are not used)
    const int x = mod(x0 - 1 + min(lane, cols + 1), g.nx), y = mod(y0 - 1 + w, g.ny);
    const bool b_lane = lane >= 1 && lane <= cols && x0 - 1 + lane < g.nx;
    const bool b_wave = w >= 1 && w <= BY;
    // byte offsets of the lane's sources inside a plane of the layout
    const long long zstride = (long long)(g.ny >> g.lr) * g.tile * (long long)sizeof(S);
    unsigned off[L::Q];
    const unsigned m = (1u << g.lr) - 1u;
    static_for<L::Q>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        const int sx = mod(x - L::ex(i), g.nx), sy = mod(y - L::ey(i), g.ny);
        off[i] = ((unsigned)(sy >> g.lr) * (unsigned)g.tile + (unsigned)i * (unsigned)g.plane +
                  ((unsigned)sy & m) * (unsigned)g.pitch + (unsigned)sx) *
                 (unsigned)sizeof(S);
    });
    const unsigned dir = (unsigned)g.plane * (unsigned)sizeof(S);
    auto load = [&](int k, S (&raw)[L::Q]) __attribute__((always_inline)) {
        const int gz = wrapz(k);
        const int zm = gz == 0 ? g.nz - 1 : gz - 1, zp = gz == g.nz - 1 ? 0 : gz + 1;
        const char *sb = reinterpret_cast<const char *>(src);
        const char *base[3] = {sb + (long long)zm * zstride, sb + (long long)gz * zstride,
                               sb + (long long)zp * zstride};
        static_for<L::Q>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            raw[i] = *reinterpret_cast<const S *>(base[1 - L::ez(i)] + off[i]);
        });
    };
    auto slot_of = [&](int i_cls, int i_idx, int slot, int a) {
        return (K::region(i_cls) + slot * K::count(i_cls) + i_idx) * AP + a;
    };
    const int own = w * W + lane;
    auto first = [&](int it, const S (&raw)[L::Q]) __attribute__((always_inline)) {
        C h[L::Q];
        static_for<L::Q>([&](auto ic) { h[decltype(ic)::value] = Codec<S>::load(&raw[decltype(ic)::value]); });
        C rho, ux, uy, uz;
        collide_pass<L, S>(h, r, rho, ux, uy, uz);
        static_for<L::Q>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            constexpr int c = K::cls(i);
            Codec<S>::template store<false>(&lds[slot_of(c, K::index(i), it % K::slots(c), own)], h[i]);
        });
    };
    // second step of plane k - 1, iteration it (first steps up to plane k)
    auto second = [&](int k, int it) __attribute__((always_inline)) {
        C h[L::Q];
        static_for<L::Q>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            constexpr int c = K::cls(i);
            h[i] = Codec<S>::load(
                &lds[slot_of(c, K::index(i), (it - c) % K::slots(c), own - (L::ey(i) * W + L::ex(i)))]);
        });
        C rho, ux, uy, uz;
        collide_pass<L, S>(h, r, rho, ux, uy, uz);
        if (!b_lane) return;
        char *db = reinterpret_cast<char *>(dst) + (long long)wrapz(k - 1) * zstride;
        static_for<L::Q>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            Codec<S>::store(reinterpret_cast<S *>(db + (size_t)i * dir + off[0]), h[i]);
        });
    };

    // first steps of planes zs - 1, zs and zs + 1; then for k = zs + 1 ... ze
    // the second step of plane k - 1 and the first step of plane k + 1,
    // whose pulls were issued an iteration before (past the chunk the last
    // plane is loaded again)
    S raw[L::Q];
    load(zs - 1, raw);
    first(0, raw);
    load(zs, raw);
    first(1, raw);
    load(zs + 1, raw);
    first(2, raw);
    load(min(zs + 2, ze), raw);
    for (int k = zs + 1, it = 2;; ++k, ++it) {
        lds_barrier();
        if (b_wave) second(k, it);
        lds_barrier();
        if (k == ze) break;
        first(it + 1, raw);
        load(min(k + 2, ze), raw);
    }
}

} // namespace ptrt

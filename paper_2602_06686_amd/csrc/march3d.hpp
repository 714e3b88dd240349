// Two fused steps per pass for D3Q19 on lattices of any width, on small
// ones, and with solids (the counterpart of k_step2, which needs nx a
// multiple of 64, many columns and no solid near them).
//
// A workgroup owns a column of cols (at most 62) x BY nodes and marches up a
// chunk of planes like k_step2, but a wave's row holds the halo columns too
// (lanes 0 ... cols + 1 are columns x0 - 1 ... x0 + cols): each of its BY + 2
// waves computes one row of first steps a plane, and BY of them the second
// step of their own row, with no separate halo task and one set of pulls
// per wave in flight.  FP32 100 registers (with solids 128, 5 of them
// spilled), two workgroups per CU; FP64 190, one.  Bound by instruction issue
// (14 collisions for six rows of two steps, idle lanes past cols) and, on
// small lattices, by the chain of a chunk's planes, about 4 us each with two
// workgroups on a CU.  The strips start
// anywhere in a 128-byte line: plain stores, whose parts meet in L2 (the
// non-temporal ones of k_step2 measured up to 13 % slower here).
//
// SOLID: link flags per node, formed once per lattice, are loaded one plane
// before the pulls that depend on them; a row of 64 lanes without any takes
// the plain code, so walls and blocks cost the rows at them only.  For the
// second step a node puts what bounces back to it into the LDS slot of the
// solid that it would be read from (a solid writes no slots, and each slot
// has one reader): for e_z >= 0 in its own first step, for e_z = -1, whose
// source's plane comes next, an iteration later from its own slot.  The
// second step then reads as without solids.  Registers of the nodes'
// e_z = -1 values over three planes instead, and a second step with a branch
// on the flags, took 214 registers in FP64 and spilled 21 in FP32 (us a
// step, one step per pass / that / this, with walls: FP32 160 x 100 x 102
// 38.6 / 42.4 / 34.5, FP64 128 x 100 x 102 69.4 / 54.6 / 53.0).
#pragma once

#include "step2.hpp"

namespace ptrt {

// Columns of a strip: near-equal strips of at most W - 2 (rows of W lanes).
inline int march_cols(int nx, int W = 64)
{
    const int strips = (nx + W - 3) / (W - 2);
    return (nx + strips - 1) / strips;
}

// Link flags of every node, once per lattice: bit i: the source of
// population i is solid, bit 0: the node is.
template <class L>
__global__ void __launch_bounds__(256)
k_link_flags(const uint8_t *__restrict__ mask, Geom g, NodeRange r, unsigned *__restrict__ flags)
{
    if (!r.place(g)) return;
    const Nbr n(g, r.x, r.y, r.z);
    unsigned f = mask[r.node] ? 1u : 0u;
    static_for<L::Q>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        if constexpr (i != 0) {
            int sx;
            unsigned srow;
            source_of<L, i>(g, n, r.x, r.y, r.z, sx, srow);
            if (mask[srow * (unsigned)g.nx + (unsigned)sx]) f |= 1u << i;
        }
    });
    flags[r.node] = f;
}

// Rows of W lanes: a wave's whole row, or two rows of 32 lanes a wave for
// lattices that fill so few of 64 (24 to 40 columns, and 63 to 80, whose
// strips of 64 lanes would be half empty).
template <class S, int BY_, int W_ = 64>
struct MarchShape {
    static constexpr int W = W_, BY = BY_, AY = BY + 2, AP = AY * W;
    static_assert(W == 64 || W == 32, "rows of a wave or half a wave");
    using K = Step2Classes<D3Q19, 2>;
    static constexpr int PAD = W; // sources of the garbage lanes 0 and 63
    static constexpr int elems = K::planes * AP + 2 * PAD;
    template <class T>
    static constexpr int waves_per_simd = sizeof(T) == 8 ? 2 : (BY == 4 ? 3 : 4);
};

template <class S, class SH, bool SOLID>
__global__ void __launch_bounds__(SH::AP)
__attribute__((amdgpu_waves_per_eu(SH::template waves_per_simd<S>, SH::template waves_per_simd<S>)))
k_march3d(const S *__restrict__ src, S *__restrict__ dst, const unsigned *__restrict__ flags, Geom g,
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
    // row of the workgroup and lane of the row
    int w = (int)threadIdx.x / W;
    if constexpr (W == 64) w = __builtin_amdgcn_readfirstlane(w);
    const int lane = (int)threadIdx.x & (W - 1);
    auto mod = [](int v, int n) {
        v %= n;
        return v < 0 ? v + n : v;
    };
    auto wrapz = [&](int k) { return k < 0 ? k + g.nz : (k >= g.nz ? k - g.nz : k); };
    // this lane's node in every plane (lanes past the halo repeat its last
    // column: their values are not used)
    const int x = mod(x0 - 1 + min(lane, cols + 1), g.nx), y = mod(y0 - 1 + w, g.ny);
    const bool b_lane = lane >= 1 && lane <= cols && x0 - 1 + lane < g.nx;
    const bool b_row = w >= 1 && w <= BY;
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
    // pull plane k; f: its link flags
    auto load = [&](int k, unsigned f, S (&raw)[L::Q]) __attribute__((always_inline)) {
        const int gz = wrapz(k);
        const int zm = gz == 0 ? g.nz - 1 : gz - 1, zp = gz == g.nz - 1 ? 0 : gz + 1;
        const char *sb = reinterpret_cast<const char *>(src);
        const char *base[3] = {sb + (long long)zm * zstride, sb + (long long)gz * zstride,
                               sb + (long long)zp * zstride};
        auto row = [&](auto bc) __attribute__((always_inline)) {
            static_for<L::Q>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                const char *p = base[1 - L::ez(i)] + off[i];
                if constexpr (decltype(bc)::value && i != 0)
                    if ((f >> i) & 1u) p = base[1] + (off[0] + (unsigned)L::opp(i) * dir);
                raw[i] = *reinterpret_cast<const S *>(p);
            });
        };
        if (SOLID && __any(f != 0)) row(std::bool_constant<SOLID>{});
        else row(std::false_type{});
    };
    const unsigned node = (unsigned)y * (unsigned)g.nx + (unsigned)x;
    auto load_flags = [&](int k) -> unsigned {
        if constexpr (SOLID) return flags[(size_t)wrapz(k) * ((size_t)g.ny * (size_t)g.nx) + node];
        return 0u;
    };
    auto slot_of = [&](int i_cls, int i_idx, int slot, int a) {
        return (K::region(i_cls) + slot * K::count(i_cls) + i_idx) * AP + a;
    };
    const int own = w * W + lane;
    // first step of plane `it`; f, fp: link flags of this plane and of the one
    // below
    auto first = [&](int it, const S (&raw)[L::Q], unsigned f, unsigned fp) __attribute__((always_inline)) {
        C h[L::Q];
        static_for<L::Q>([&](auto ic) { h[decltype(ic)::value] = Codec<S>::load(&raw[decltype(ic)::value]); });
        C rho, ux, uy, uz;
        collide_pass<L, S>(h, r, rho, ux, uy, uz);
        if (!(SOLID && (f & 1u)))
            static_for<L::Q>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                constexpr int c = K::cls(i);
                Codec<S>::template store<false>(&lds[slot_of(c, K::index(i), it % K::slots(c), own)], h[i]);
            });
        if constexpr (SOLID) {
            const bool core = b_row && b_lane && it > 0;
            if (__any(core && (f | fp) > 1u)) {
                if (!core) return;
                static_for<L::Q>([&](auto ic) {
                    constexpr int i = decltype(ic)::value;
                    constexpr int c = K::cls(i), o = L::opp(i), co = K::cls(o);
                    const int to = own - (L::ey(i) * W + L::ex(i));
                    if constexpr (i != 0 && c != 0) {
                        // from the source's plane, this one or the one below
                        if ((f >> i) & 1u && !(f & 1u))
                            Codec<S>::template store<false>(
                                &lds[slot_of(c, K::index(i), (it + 1 - c) % K::slots(c), to)], h[o]);
                    } else if constexpr (c == 0) {
                        // of the node below this one, whose source is in this plane
                        if ((fp >> i) & 1u && !(fp & 1u))
                            lds[slot_of(c, K::index(i), it % K::slots(c), to)] =
                                lds[slot_of(co, K::index(o), (it - 1) % K::slots(co), own)];
                    }
                });
            }
        }
    };
    // second step of plane k - 1, iteration it (first steps up to plane k); f:
    // link flags of plane k - 1
    auto second = [&](int k, int it, unsigned f) __attribute__((always_inline)) {
        C h[L::Q];
        static_for<L::Q>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            constexpr int c = K::cls(i);
            h[i] = Codec<S>::load(&lds[slot_of(c, K::index(i), (it - c) % K::slots(c),
                                               own - (L::ey(i) * W + L::ex(i)))]);
        });
        C rho, ux, uy, uz;
        collide_pass<L, S>(h, r, rho, ux, uy, uz);
        if (!b_lane || (SOLID && (f & 1u))) return;
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
    unsigned f0 = load_flags(zs - 1), f1 = load_flags(zs), f2 = load_flags(zs + 1),
             f3 = load_flags(min(zs + 2, ze));
    load(zs - 1, f0, raw);
    first(0, raw, f0, 0);
    load(zs, f1, raw);
    first(1, raw, f1, f0);
    load(zs + 1, f2, raw);
    // a value that bounces back from plane zs + 1 must not be met by one of
    // plane zs - 1 or zs in the same slot
    if constexpr (SOLID) lds_barrier();
    first(2, raw, f2, f1);
    // f0 ... f3: flags of planes k - 1 ... k + 2
    f0 = f1;
    f1 = f2;
    f2 = f3;
    load(min(zs + 2, ze), f2, raw);
    f3 = load_flags(min(zs + 3, ze));
    for (int k = zs + 1, it = 2;; ++k, ++it) {
        lds_barrier();
        if (b_row) second(k, it, f0);
        lds_barrier();
        if (k == ze) break;
        first(it + 1, raw, f2, f1);
        f0 = f1;
        f1 = f2;
        f2 = f3;
        load(min(k + 2, ze), f2, raw);
        f3 = load_flags(min(k + 3, ze));
    }
}

} // namespace ptrt

// pair_kernel.hpp -- two steps of a 3D grid in one launch (temporal blocking).
//
// A step of a 3D grid reads and writes every population once, so it is bound
// by memory; two steps in one pass over memory halve that.  A workgroup owns
// a column of W x H x chunk cells and marches through it along z.  At plane p
// it
//   1. computes step k of plane p on the W + 2 by H + 2 columns around its
//      own (one cell per thread, pulled from global memory, prefetched one
//      plane ahead), leaving the post-collision populations in LDS;
//   2. computes step k + 1 of plane p - 1 on its own W x H columns, pulling
//      from the neighbouring columns' LDS slots, and stores it.
// Step k of the halo columns and of the planes below and above the chunk is
// computed by neighbouring workgroups too: (W + 2)(H + 2)/(W H) (chunk + 2)/
// chunk of the cells, which the tile's shape (chosen on the host) keeps small.
//
// LDS holds only what a later plane still pulls: populations moving up
// (xi_z = 1) of planes p - 2 .. p, level ones of p - 1 and p, downward ones of
// p - 1 and p (that of p - 1 for links bounced at a wall).  Populations that
// stay in their column (rest, straight up, straight down) stay in registers.
//
// A link's source is a constant of the thread except for the plane's uniform
// offset: periodic wrap, and at x and y walls the bounce to the cell's own
// opposite population, are folded into one 32-bit offset per link direction
// before the march, so that a wall costs no instruction per plane.  Planes
// next to the z faces, where wrap and bounce depend on z, take per-link tests.
// The collision is collide's and LDS holds stored values, so the result
// equals two launches of step_cells bit for bit.
#pragma once

#include "step_kernel.hpp"

namespace lbm {

struct PairArgs {
    int W, H, EW;             // own columns of a workgroup, and W + 2
    int cols;                 // (W + 2) (H + 2)
    int ntx, nty, chunk;      // tiles along x and y, planes of a workgroup
    int ntiles;               // workgroups
    uint32_t bytes;           // bytes of a population buffer
    uint32_t moving;          // bit f set: face f is a moving wall
    int sensor;               // bit 0: the first step evaluates the sensor, bit 1: the second
    void *max1, *max2;        // max bits of the two steps' sensors per block ...
    int max_stride;           // ... this many values apart
};

// LDS values per column: lateral populations of the three z directions times
// the planes they are kept for.
template <int Q>
constexpr int pair_lateral(int cz) {
    int n = 0;
    for (int i = 1; i < Q; ++i) n += Lattice<Q>::c[i][2] == cz && (Lattice<Q>::c[i][0] || Lattice<Q>::c[i][1]);
    return n;
}
constexpr int kRingU = 3, kRingM = 2, kRingD = 2;   // planes kept of upward, level and downward populations
template <int Q>
constexpr int pair_slots() {
    return kRingU * pair_lateral<Q>(1) + kRingM * pair_lateral<Q>(0) + kRingD * pair_lateral<Q>(-1);
}
// Index of lateral population I among those of its z direction.
template <int Q>
constexpr int pair_index(int I) {
    int n = 0;
    for (int i = 1; i < I; ++i)
        n += Lattice<Q>::c[i][2] == Lattice<Q>::c[I][2] && (Lattice<Q>::c[i][0] || Lattice<Q>::c[i][1]);
    return n;
}

// First population with the weight of population I.
template <int Q>
constexpr int weight_representative(int I) {
    auto len2 = [](int i) {
        return Lattice<Q>::c[i][0] * Lattice<Q>::c[i][0] + Lattice<Q>::c[i][1] * Lattice<Q>::c[i][1] +
               Lattice<Q>::c[i][2] * Lattice<Q>::c[i][2];
    };
    for (int i = 0; i < I; ++i)
        if (len2(i) == len2(I)) return i;
    return I;
}

constexpr int kPairBlocks = 64;   // most sensor blocks (columns of blocks) a tile touches
constexpr int kPairLds = 160 * 1024 - 4 * kPairBlocks * 8 - 256;

// Most columns of a workgroup (one thread each): what LDS holds, at most 1024.
template <int Q, typename R>
constexpr int pair_columns() {
    const int fit = kPairLds / (pair_slots<Q>() * (int)sizeof(R));
    const int most = Q == 19 && sizeof(R) == 4 ? 768 : 512;   // 3 or 2 waves per SIMD: what their registers allow
    return fit < most ? fit / 8 * 8 : most;
}
template <int Q, typename R>
constexpr int pair_threads() {
    return (pair_columns<Q, R>() + 63) / 64 * 64;
}

// Where step_pair exists.  Without force and Smagorinsky together, and in
// float64 without force, whose registers spill; without D3Q27 in float64
// (the spills made it 2.4 times slower than two steps) and without the
// 16-bit storages, whose steps are bound by vector arithmetic, which a pair
// does not save.
template <int Q, typename T, int MODEL>
constexpr bool pair_supported() {
    if constexpr (std::is_same_v<T, double>) return Q == 19 && (MODEL & kModelForce) == 0;
    else if constexpr (std::is_same_v<T, float>) return (Q == 19 || Q == 27) && MODEL != (kModelForce | kModelSmag);
    else return false;
}

// A barrier that orders LDS only: global loads and stores stay in flight.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// v, opaque to the compiler: what is computed from it is computed where it is
// used, in scalar instructions beside the vector ones, instead of being kept
// in scalar registers across the march (which would spill).
__device__ __forceinline__ uint32_t opaque(uint32_t v) {
    asm volatile("" : "+s"(v));
    return v;
}

__device__ __forceinline__ uint32_t opaque_lane(uint32_t v) {
    asm volatile("" : "+v"(v));
    return v;
}

template <typename R>
__device__ __forceinline__ R buffer_load(__amdgpu_buffer_rsrc_t b, uint32_t voff, uint32_t soff) {
    if constexpr (sizeof(R) == 8)
        return __builtin_bit_cast(R, __builtin_amdgcn_raw_buffer_load_b64(b, (int)voff, (int)soff, 0));
    else
        return __builtin_bit_cast(R, __builtin_amdgcn_raw_buffer_load_b32(b, (int)voff, (int)soff, 0));
}

// Stores go through L2 like the loads: a tile's rows start and end inside
// lines that its neighbours complete (non-temporal stores wrote those lines
// in parts: 230^3 float32 380 us per step against 243, 256^3 330 / 316).
template <typename R>
__device__ __forceinline__ void buffer_store(__amdgpu_buffer_rsrc_t b, R v, uint32_t voff, uint32_t soff) {
    if constexpr (sizeof(R) == 8) {
        typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), b, (int)voff, (int)soff, 0);
    } else {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), b, (int)voff, (int)soff, 0);
    }
}

// SWAPPED: population i of the buffers sits in plane opp(i) (the in-place
// scheme's order after a local step).
template <int Q, typename T, typename C, bool SHIFTED, bool SENSOR, int SKIND, int MODEL, bool SWAPPED>
__global__ __launch_bounds__((pair_threads<Q, T>())) void step_pair(const StepArgs<C> arg, const PairArgs p) {
    static_assert(pair_supported<Q, T, MODEL>());
    using R = T;
    using U = std::conditional_t<sizeof(C) == 8, unsigned long long, unsigned>;
    constexpr int NC = pair_columns<Q, R>();
    constexpr int NU = pair_lateral<Q>(1), NM = pair_lateral<Q>(0), ND = pair_lateral<Q>(-1);
    __shared__ R lds[pair_slots<Q>() * NC];
    __shared__ U red[SENSOR ? 4 * kPairBlocks : 1];   // [step][plane parity][block column]
    constexpr int M0 = kRingU * NU * NC, D0 = M0 + kRingM * NM * NC;   // first values of the level and down rings

    // w_i rho0 takes one value per weight: 3 or 4 scalar registers
    StepArgs<C> a = arg;
    static_for<0, Q>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        a.shift[i] = arg.shift[weight_representative<Q>(i)];
    });
    const int t = threadIdx.x;
    const int tile = xcd_tile(blockIdx.x, p.ntiles);
    const int tix = tile % p.ntx, tiy = (tile / p.ntx) % p.nty;
    const int x0 = tix * p.W, y0 = tiy * p.H, z0 = tile / (p.ntx * p.nty) * p.chunk;
    const int nx = a.nx, ny = a.ny, nz = a.nz, slab = nx * ny;
    const int z1 = min(z0 + p.chunk, nz);
    const int ey = t / p.EW, ex = t - ey * p.EW;
    const int ux = x0 - 1 + ex, uy = y0 - 1 + ey;
    const bool perx = !(a.wall & 3u), pery = !(a.wall & 12u), perz = !(a.wall & 48u);
    const int x = perx ? (ux < 0 ? ux + nx : (ux >= nx ? ux - nx : ux)) : ux;
    const int y = pery ? (uy < 0 ? uy + ny : (uy >= ny ? uy - ny : uy)) : uy;
    const bool active = t < p.cols && (perx ? ux <= nx : ux >= 0 && ux < nx) && (pery ? uy <= ny : uy >= 0 && uy < ny);
    const bool own = active && ex >= 1 && ex <= p.W && ux < nx && ey >= 1 && ey <= p.H && uy < ny;
    const bool wxm = !perx && x == 0, wxp = !perx && x == nx - 1;
    const bool wym = !pery && y == 0, wyp = !pery && y == ny - 1;
    const bool lane_moving = active && ((wxm && (p.moving & 1u)) || (wxp && (p.moving & 2u)) ||
                                        (wym && (p.moving & 4u)) || (wyp && (p.moving & 8u)));
    const bool wave_moving = __any(lane_moving);
    // faces beyond which a link of the thread's column bounces
    const uint32_t wall_bits = (wxm ? 1u : 0u) | (wxp ? 2u : 0u) | (wym ? 4u : 0u) | (wyp ? 8u : 0u);
    const bool wave_walls = __any(active && wall_bits != 0);

    const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.src), 0, p.bytes, 0x27000);
    const __amdgpu_buffer_rsrc_t dst = __builtin_amdgcn_make_buffer_rsrc(a.dst, 0, p.bytes, 0x27000);
    constexpr uint32_t S = sizeof(R);
    const uint32_t cell = (uint32_t)(y * nx + x), own_off = cell * S;
    const int dxm = x == 0 ? nx - 1 : -1, dxp = x == nx - 1 ? 1 - nx : 1;
    const int dym = y == 0 ? (ny - 1) * nx : -nx, dyp = y == ny - 1 ? (1 - ny) * nx : nx;
    auto bounced = [&](auto ic) {   // at an x or y wall of the thread's column
        using V = Vel<Q, decltype(ic)::value>;
        return (V::x > 0 && wxm) || (V::x < 0 && wxp) || (V::y > 0 && wym) || (V::y < 0 && wyp);
    };
    // Plane of population I in the buffers, and of the two planes {I, opp(I)}
    // the lower one (the uniform part of an address starts there).
    auto plane_of = [](int i, int o) { return SWAPPED ? o : i; };
    // byte offset of link I of the thread's column beyond the uniform offset
    // (lower plane of the pair, slab min(z - xi_z, z))
    auto link_off = [&](auto ic) {
        constexpr int i = decltype(ic)::value;
        using V = Vel<Q, i>;
        constexpr int o = V::opp, lo = o < i ? o : i;
        int d = 0;
        if constexpr (V::x > 0) d += dxm;
        if constexpr (V::x < 0) d += dxp;
        if constexpr (V::y > 0) d += dym;
        if constexpr (V::y < 0) d += dyp;
        const bool b = bounced(ic);
        const uint32_t pull = cell + (uint32_t)d + (uint32_t)(plane_of(i, o) - lo) * a.pitch + (V::z < 0 ? slab : 0);
        const uint32_t back = cell + (uint32_t)(plane_of(o, i) - lo) * a.pitch + (V::z > 0 ? slab : 0);
        return (b ? back : pull) * S;
    };
    uint32_t voff[Q];
    static_for<1, Q>([&](auto ic) { voff[decltype(ic)::value] = link_off(ic); });
    voff[0] = own_off;

    // the thread's populations of plane z (in the grid), as stored
    R next[Q];
    auto fetch = [&](int z) {
        if (!active) return;
        const uint32_t pitch = opaque(a.pitch);
        if (z > 0 && z < nz - 1) {
            static_for<0, Q>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                using V = Vel<Q, i>;
                constexpr int lo = (V::opp < i) ? V::opp : i;
                const uint32_t soff = ((uint32_t)lo * pitch + (uint32_t)(V::z > 0 ? z - 1 : z) * (uint32_t)slab) * S;
                next[i] = buffer_load<R>(src, voff[i], soff);
            });
        } else {
            const int zm = z == 0 ? nz - 1 : z - 1, zp = z == nz - 1 ? 0 : z + 1;
            static_for<0, Q>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                using V = Vel<Q, i>;
                constexpr int o = V::opp, lo = o < i ? o : i;
                int d = 0, zs = z;
                if constexpr (V::x > 0) d += dxm;
                if constexpr (V::x < 0) d += dxp;
                if constexpr (V::y > 0) d += dym;
                if constexpr (V::y < 0) d += dyp;
                if constexpr (V::z > 0) zs = zm;
                if constexpr (V::z < 0) zs = zp;
                const bool b = bounced(ic) || (!perz && ((V::z > 0 && z == 0) || (V::z < 0 && z == nz - 1)));
                const uint32_t off = b ? cell + (uint32_t)(z * slab) + (uint32_t)(plane_of(o, i) - lo) * pitch
                                       : cell + (uint32_t)(d + zs * slab) + (uint32_t)(plane_of(i, o) - lo) * pitch;
                next[i] = buffer_load<R>(src, off * S, (uint32_t)lo * pitch * S);
            });
        }
    };
    // moving-wall terms of the links of cell (x, y, z), 0 off moving walls
    auto add_walls = [&](int z, C (&d)[Q]) {
        const Geo<C> g = make_geo<3>(arg, x, y, z);
        // the table through an opaque offset, which keeps its loads inside this
        // branch and in one run (they are waited for together)
        const C *tab = reinterpret_cast<const C *>(reinterpret_cast<const char *>(&arg.wcorr[0][0]) + opaque(0u));
        static_for<1, Q>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            using V = Vel<Q, i>;
            const C *w = tab + 6 * i;
            C corr = C(0);   // as link()
            if constexpr (V::x > 0) corr += w[0] * g.fw[0];
            if constexpr (V::x < 0) corr += w[1] * g.fw[1];
            if constexpr (V::y > 0) corr += w[2] * g.fw[2];
            if constexpr (V::y < 0) corr += w[3] * g.fw[3];
            if constexpr (V::z > 0) corr += w[4] * g.fw[4];
            if constexpr (V::z < 0) corr += w[5] * g.fw[5];
            d[i] += corr;
        });
    };

    U m1 = 0, m2 = 0;   // bits of the running sensor maxima (>= 0, +inf or NaN: unsigned order)
    const int bx0 = x0 / kBlockEdge, by0 = y0 / kBlockEdge;
    const int tbx = min(x0 + p.W - 1, nx - 1) / kBlockEdge - bx0 + 1;
    const int tby = min(y0 + p.H - 1, ny - 1) / kBlockEdge - by0 + 1;
    const int rslot = (uy / kBlockEdge - by0) * tbx + (ux / kBlockEdge - bx0);
    // A flush of plane z's running maxima into the tile's block columns, and
    // after a barrier a drain of those into the blocks' words.  Flushes of
    // neighbouring planes use different arrays: a wave may flush the next
    // plane while another still drains this one.
    auto red_of = [&](int step, int z) { return red + (2 * step + (z & 1)) * kPairBlocks; };
    auto flush_at = [&](int z) { return (z & (kBlockEdge - 1)) == kBlockEdge - 1 || z == z1 - 1; };
    auto drain = [&](U *r, void *words, int z) {
        if (t >= tbx * tby) return;
        const U v = r[t];
        r[t] = 0;
        const int b = ((z / kBlockEdge) * a.nby + by0 + t / tbx) * a.nbx + bx0 + t % tbx;
        if (v) __hip_atomic_fetch_max(static_cast<U *>(words) + (int64_t)b * p.max_stride, v, __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
    };
    if constexpr (SENSOR) {
        for (int k = t; k < 4 * kPairBlocks; k += blockDim.x) red[k] = 0;
    }

    Geo<C> g{};   // collide reads only the cell index, the key of stochastic rounding, which is not paired
    R rest_s{}, up_s{}, up_s1{}, down_s{};   // of plane s = p - 1 (up_s1: of s - 1)
    int u0 = 0, e0 = 0;                      // ring slots of plane pl: up; level and down
    const int first = z0 - 1, last = z1;     // planes of step k
    auto in_grid = [&](int z) { return perz ? (z < 0 ? z + nz : (z >= nz ? z - nz : z)) : z; };
#pragma unroll 1
    for (int pl = first - 1; pl <= last; ++pl) {   // the first pass only fetches
        const int z = in_grid(pl);
        const bool have = pl >= first && z >= 0 && z < nz;
        const int u1 = u0 == 0 ? kRingU - 1 : u0 - 1;   // of plane pl - 1
        const int u2 = u1 == 0 ? kRingU - 1 : u1 - 1;   // of plane pl - 2
        const int e1 = e0 == 0 ? kRingM - 1 : e0 - 1;   // of plane pl - 1
        R rest_p{}, up_p{}, down_p{};
        C d[Q];
        if (have && active)
            static_for<0, Q>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                C v = static_cast<C>(next[i]);
                if constexpr (!SHIFTED) v -= a.shift[i];
                d[i] = v;
            });
        if (pl < last) {
            const int zn = in_grid(pl + 1);
            if (zn >= 0 && zn < nz) fetch(zn);
        }
        if (have) {
            if (active) {
                if (wave_moving || (z == 0 && (p.moving & 16u)) || (z == nz - 1 && (p.moving & 32u))) add_walls(z, d);
                const C s = collide<Q, T, C, SHIFTED, SENSOR, SKIND, MODEL>(a, g, d, [&](auto ic, C out, uint32_t) {
                    constexpr int i = decltype(ic)::value;
                    using V = Vel<Q, i>;
                    const R v = to_storage<T>(out, 0u);
                    if constexpr (V::x != 0 || V::y != 0) {
                        if constexpr (V::z > 0) lds[(u0 * NU + pair_index<Q>(i)) * NC + t] = v;
                        else if constexpr (V::z < 0) lds[D0 + (e0 * ND + pair_index<Q>(i)) * NC + t] = v;
                        else lds[M0 + (e0 * NM + pair_index<Q>(i)) * NC + t] = v;
                    } else if constexpr (V::z > 0) up_p = v;
                    else if constexpr (V::z < 0) down_p = v;
                    else rest_p = v;
                });
                if constexpr (SENSOR) {
                    if (own && pl >= z0 && pl < z1) {
                        m1 = max(m1, __builtin_bit_cast(U, s));
                        if ((p.sensor & 1) && flush_at(pl)) {
                            atomicMax(&red_of(0, pl)[rslot], m1);
                            m1 = 0;
                        }
                    }
                }
            }
        }
        lds_barrier();
        if constexpr (SENSOR) {
            if ((p.sensor & 1) && pl >= z0 && pl < z1 && flush_at(pl)) drain(red_of(0, pl), p.max1, pl);
            if ((p.sensor & 2) && pl - 2 >= z0 && flush_at(pl - 2)) drain(red_of(1, pl - 2), p.max2, pl - 2);
        }
        const int s = pl - 1;
        if (s >= z0 && own) {
            C d2[Q];
            const bool zb = !perz && s == 0, zt = !perz && s == nz - 1;
            // first LDS value of population j (I, or opp(I) for a bounced link) of
            // the plane that link I of plane s reads it from
            auto slot = [&](auto ic, int j) {
                constexpr int i = decltype(ic)::value;
                using V = Vel<Q, i>;
                const int plane = j == i ? s - V::z : s;   // relative to pl: s = pl - 1
                const int vz = j == i ? V::z : -V::z, k = pair_index<Q>(j);
                if (vz > 0) return ((plane == s ? u1 : u2) * NU + k) * NC;
                if (vz < 0) return D0 + ((plane == s ? e1 : e0) * ND + k) * NC;
                return M0 + (e1 * NM + k) * NC;
            };
            R v2[Q];
            v2[0] = rest_s;
            v2[5] = zb ? down_s : up_s1;   // straight up and down stay in the column
            v2[6] = zt ? up_s : down_p;
            if (wave_walls || zb || zt) {
                const uint32_t bits = opaque_lane(wall_bits);
                static_for<1, Q>([&](auto ic) {
                    constexpr int i = decltype(ic)::value;
                    using V = Vel<Q, i>;
                    constexpr int o = V::opp;
                    if constexpr (V::x != 0 || V::y != 0) {
                        constexpr uint32_t crosses = (V::x > 0 ? 1u : (V::x < 0 ? 2u : 0u)) | (V::y > 0 ? 4u : (V::y < 0 ? 8u : 0u));
                        const bool back = (bits & crosses) || (V::z > 0 && zb) || (V::z < 0 && zt);
                        v2[i] = lds[back ? slot(ic, o) + t : slot(ic, i) + t - V::x - V::y * p.EW];
                    }
                });
            } else {
                static_for<1, Q>([&](auto ic) {
                    constexpr int i = decltype(ic)::value;
                    using V = Vel<Q, i>;
                    if constexpr (V::x != 0 || V::y != 0) v2[i] = lds[slot(ic, i) + t - V::x - V::y * p.EW];
                });
            }
            static_for<0, Q>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                C f = static_cast<C>(v2[i]);
                if constexpr (!SHIFTED && !SWAPPED) f -= a.shift[i];
                d2[i] = f;
            });
            if (wave_moving || (s == 0 && (p.moving & 16u)) || (s == nz - 1 && (p.moving & 32u))) add_walls(s, d2);
            // in place, the first of two steps stores a bounced value with its
            // moving-wall term, the second takes the shift off
            if constexpr (!SHIFTED && SWAPPED)
                static_for<0, Q>([&](auto ic) { d2[decltype(ic)::value] -= a.shift[decltype(ic)::value]; });
            const uint32_t pitch = opaque(a.pitch), zoff = (uint32_t)s * (uint32_t)slab;
            const C sv = collide<Q, T, C, SHIFTED, SENSOR, SKIND, MODEL>(a, g, d2, [&](auto ic, C out, uint32_t) {
                constexpr int i = decltype(ic)::value;
                const uint32_t plane = (uint32_t)plane_of(i, Vel<Q, i>::opp);
                buffer_store(dst, to_storage<T>(out, 0u), own_off, (plane * pitch + zoff) * S);
            });
            if constexpr (SENSOR) {
                m2 = max(m2, __builtin_bit_cast(U, sv));
                if ((p.sensor & 2) && flush_at(s)) {
                    atomicMax(&red_of(1, s)[rslot], m2);
                    m2 = 0;
                }
            }
        }
        lds_barrier();   // the next plane overwrites slots read above
        rest_s = rest_p;
        up_s1 = up_s;
        up_s = up_p;
        down_s = down_p;
        u0 = u0 == kRingU - 1 ? 0 : u0 + 1;
        e0 = e0 == kRingM - 1 ? 0 : e0 + 1;
    }
    if constexpr (SENSOR) {   // the last plane's flush
        lds_barrier();
        if (p.sensor & 2) drain(red_of(1, z1 - 1), p.max2, z1 - 1);
    }
}

}  // namespace lbm

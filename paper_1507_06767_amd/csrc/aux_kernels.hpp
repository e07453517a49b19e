// aux_kernels.hpp -- kernels outside the time loop: state initialisation,
// host-transfer conversion, macroscopic fields and the conservation totals.
// None of them runs per step; all of them read or write the same SoA planes
// as the step kernel.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lattice.hpp"
#include "step_kernel.hpp"

namespace lbm {

// Conversions between the storage type and float64 (16-bit types go
// through float32).
template <typename T>
__device__ __forceinline__ T to_store(double v) {
    if constexpr (sizeof(T) == 2) return static_cast<T>(static_cast<float>(v));
    else return static_cast<T>(v);
}

template <typename T>
__device__ __forceinline__ double from_store(T v) {
    if constexpr (sizeof(T) == 2) return static_cast<double>(static_cast<float>(v));
    else return static_cast<double>(v);
}

template <typename T>
struct Planes {
    T *f;              // plane i at f + i*pitch
    int64_t pitch;
    int cells;
    double shift[kMaxQ];  // storage shift per population (0 for plain storage)
    // population I of cell c; EX: plane i at f + opp(i)*pitch, the slot order of
    // the in-place scheme before a gather step
    template <int Q, int I, bool EX>
    __device__ __forceinline__ double load(int64_t c) const {
        return from_store<T>(f[(int64_t)(EX ? Vel<Q, I>::opp : I) * pitch + c]);
    }
};

// Rest state: f_i = w_i rho0 (stored as f_i - shift_i).
template <int Q, typename T>
__global__ void init_rest_kernel(Planes<T> p, double rho0) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= p.cells) return;
    static_for<0, Q>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        p.f[(int64_t)i * p.pitch + c] = to_store<T>(Vel<Q, i>::w * rho0 - p.shift[i]);
    });
}

// Clears n 64-bit words (the per-block accumulators of the step kernel).
__global__ void zero_words_kernel(unsigned long long *p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

// out[opp(i)][c] = in[i][c]: between natural order and the exchanged-slot
// order of the in-place scheme (an involution).
template <int Q, typename T>
__global__ void swap_planes_kernel(const T *in, T *out, int64_t pitch, int cells) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= cells) return;
    static_for<0, Q>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        out[(int64_t)Vel<Q, i>::opp * pitch + c] = in[(int64_t)i * pitch + c];
    });
}

// One plane from float64 staging: out = (T)(in - shift).
template <typename T>
__global__ void import_plane_kernel(const double *in, T *out, int cells, double shift) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c < cells) out[c] = to_store<T>(in[c] - shift);
}

// One plane to float64 staging: out = (double)in + shift.
template <typename T>
__global__ void export_plane_kernel(const T *in, double *out, int cells, double shift) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c < cells) out[c] = from_store<T>(in[c]) + shift;
}

// f^eq(rho, u) of Eq. feq_i in float64, stored as f^eq_i - shift_i.
// rho == nullptr: rho0 everywhere; u == nullptr: at rest.  u has 3 planes.
template <int Q, typename T>
__global__ void equilibrium_kernel(Planes<T> p, const double *rho, const double *u, double rho0) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= p.cells) return;
    const double r = rho ? rho[c] : rho0;
    double uu[3] = {0.0, 0.0, 0.0};
    if (u) {
        uu[0] = u[c];
        uu[1] = u[(int64_t)p.cells + c];
        uu[2] = (Lattice<Q>::D == 3) ? u[2 * (int64_t)p.cells + c] : 0.0;
    }
    const double usq = uu[0] * uu[0] + uu[1] * uu[1] + uu[2] * uu[2];
    static_for<0, Q>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        using V = Vel<Q, i>;
        const double cu = V::x * uu[0] + V::y * uu[1] + V::z * uu[2];
        const double feq = V::w * r * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * usq);
        p.f[(int64_t)i * p.pitch + c] = to_store<T>(feq - p.shift[i]);
    });
}

// rho = sum_i S_i and u = (sum_i xi_i S_i - F/2) / rho of a cell, in float64:
// r = (rho, u).
template <int Q, bool EX, typename T>
__device__ __forceinline__ void cell_macros(const Planes<T> &p, int64_t c, double Fx, double Fy, double Fz,
                                            double (&r)[4]) {
    double rho = 0.0, m[3] = {0.0, 0.0, 0.0};
    static_for<0, Q>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        using V = Vel<Q, i>;
        const double v = p.template load<Q, i, EX>(c);
        rho += v + p.shift[i];
        if constexpr (V::x != 0) m[0] += V::x * v;   // the shifts cancel in pairs
        if constexpr (V::y != 0) m[1] += V::y * v;
        if constexpr (V::z != 0) m[2] += V::z * v;
    });
    r[0] = rho;
    r[1] = (m[0] - 0.5 * Fx) / rho;
    r[2] = (m[1] - 0.5 * Fy) / rho;
    r[3] = (m[2] - 0.5 * Fz) / rho;
}

template <int Q, typename T, bool EX>
__global__ void macros_kernel(Planes<T> p, double *rho_out, double *u_out, double Fx, double Fy,
                              double Fz) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= p.cells) return;
    double r[4];
    cell_macros<Q, EX>(p, c, Fx, Fy, Fz, r);
    if (rho_out) rho_out[c] = r[0];
    if (u_out) {
        u_out[c] = r[1];
        u_out[(int64_t)p.cells + c] = r[2];
        u_out[2 * (int64_t)p.cells + c] = r[3];
    }
}

// Per-block means of (rho - rho0, u_x, u_y, u_z), cells summed in z, y, x
// order; edge blocks average the cells they hold.  Output [block][4].  A
// workgroup takes kMeansBlocks blocks in a row: its threads form the cells'
// values from the populations, rows of 32 cells, a wavefront two rows at a
// time, into LDS, and one lane per block and quantity adds them up there (a
// chain of 512 additions, about 4 us, behind the loads of the other
// workgroups).  The populations are read once and nothing is written but the
// means.  (128^3 float32: 46 us, 3.5 TB/s; the per-cell fields written
// out, 43, and then summed by one thread per block, 182.)
constexpr int kMeansBlocks = 4, kMeansThreads = 512;
constexpr int kMeansLds = kMeansBlocks * 512 * 4 * 8;
template <int Q, typename T, bool EX>
__global__ __launch_bounds__(kMeansThreads) void block_means_kernel(Planes<T> p, int nx, int ny, int nz, int nbx,
                                                                    int bz, double rho0, double Fx, double Fy,
                                                                    double Fz, double *out) {
    extern __shared__ double vals[];   // [block][cell z, y, x ^ block: the blocks' lanes in different banks][quantity]
    const int groups = (nbx + kMeansBlocks - 1) / kMeansBlocks, row0 = blockIdx.x / groups, nby = (ny + 7) / 8;
    const int t = threadIdx.x, bx0 = (blockIdx.x - row0 * groups) * kMeansBlocks, z0 = row0 / nby * bz, y0 = row0 % nby * 8;
    const int tx = t & 31, x = 8 * bx0 + tx, ty = t >> 5 & 7, y = y0 + ty;
    if (x < nx && y < ny)
        for (int z = z0 + (t >> 8); z < min(nz, z0 + bz); z += kMeansThreads / 256) {
            double r[4];
            cell_macros<Q, EX>(p, ((int64_t)z * ny + y) * nx + x, Fx, Fy, Fz, r);
            double *v = vals + ((((tx >> 3) * 8 + z - z0) * 8 + ty) * 8 + ((tx & 7) ^ (tx >> 3))) * 4;
            v[0] = r[0] - rho0;
            v[1] = r[1];
            v[2] = r[2];
            v[3] = r[3];
        }
    __syncthreads();
    const int b = t >> 2, k = t & 3;
    if (b >= min(kMeansBlocks, nbx - bx0)) return;
    const int ex = min(8, nx - 8 * (bx0 + b)), ey = min(8, ny - y0), ez = min(bz, nz - z0);
    double s = 0.0;
    for (int z = 0; z < ez; ++z)
        for (int yy = 0; yy < ey; ++yy) {
            const double *row = vals + ((b * 8 + z) * 8 + yy) * 32 + k;
            if (ex == 8) {
#pragma unroll
                for (int xx = 0; xx < 8; ++xx) s += row[4 * (xx ^ b)];
            } else {
                for (int xx = 0; xx < ex; ++xx) s += row[4 * (xx ^ b)];
            }
        }
    out[4 * ((int64_t)row0 * nbx + bx0 + b) + k] = s / (double)(ex * ey * ez);
}

// Refinement level of every block from its sensor maximum (Sec. 3.4):
// l = clamp(floor(a log2 M + b), lmin, lmax); non-finite M -> lmax, M <= 0 -> lmin.
template <typename C>
__global__ void levels_kernel(const C *bmax, int8_t *lev, int nblocks, double a, double b, int lmin,
                              int lmax) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nblocks) return;
    const double K = static_cast<double>(bmax[i]);
    int l;
    if (!(K == K) || K == HUGE_VAL) l = lmax;
    else if (K <= 0.0) l = lmin;
    else {
        const double x = floor(a * log2(K) + b);
        l = (x < lmin) ? lmin : (x > lmax) ? lmax : (int)x;
    }
    lev[i] = (int8_t)l;
}

// Buffer layer (Sec. 5.2): every block takes the largest level within `r`
// blocks of it (Chebyshev distance).
__global__ void dilate_kernel(const int8_t *in, int8_t *out, int nbx, int nby, int nbz, int r) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nbx * nby * nbz) return;
    const int x = i % nbx, y = (i / nbx) % nby, z = i / (nbx * nby);
    int best = -128;
    for (int dz = -r; dz <= r; ++dz)
        for (int dy = -r; dy <= r; ++dy)
            for (int dx = -r; dx <= r; ++dx) {
                const int xx = x + dx, yy = y + dy, zz = z + dz;
                if (xx < 0 || yy < 0 || zz < 0 || xx >= nbx || yy >= nby || zz >= nbz) continue;
                const int v = in[(zz * nby + yy) * nbx + xx];
                best = v > best ? v : best;
            }
    out[i] = (int8_t)best;
}

// Block maxima and flags of a sensor step whose workgroups folded max bits
// into per-block words (words[b * stride], as values of type C), which are
// cleared for the next sensor step, as are those of the other step of a pair
// (other; nullptr: none); the L2 sensor's square root is taken here, once per
// block.
template <typename C>
__global__ void finish_blocks_kernel(C *words, C *other, int stride, int nblocks, bool l2, C *block_max, int8_t *flags,
                                     double theta_r, double theta_c) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= nblocks) return;
    C M = words[(int64_t)b * stride];
    words[(int64_t)b * stride] = C(0);
    if (other) other[(int64_t)b * stride] = C(0);
    if (l2) M = sqrt(M);
    block_max[b] = M;
    flags[b] = block_flag(static_cast<double>(M), theta_r, theta_c);
}

// Per block: the largest time-averaged cell sensor, sum / samples, NaN-propagating
// (the per-cell sums are float64).
__global__ void average_block_max_kernel(const double *sum, double *out, int nx, int ny, int nz, int bx, int by,
                                         int bz, int nbx, int nby, int nbz, double inv_samples) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nbx * nby * nbz) return;
    const int x0 = (i % nbx) * bx, y0 = ((i / nbx) % nby) * by, z0 = (i / (nbx * nby)) * bz;
    double m = 0.0;
    bool nan = false;
    for (int z = z0; z < min(z0 + bz, nz); ++z)
        for (int y = y0; y < min(y0 + by, ny); ++y)
            for (int x = x0; x < min(x0 + bx, nx); ++x) {
                const double v = sum[((int64_t)z * ny + y) * nx + x] * inv_samples;
                if (!(v == v)) nan = true;
                else if (v > m) m = v;
            }
    out[i] = nan ? __longlong_as_double(0x7ff8000000000000ll) : m;
}

constexpr int kReduceThreads = 256;

// Fixed-order tree over the workgroup's 256 slots of 4 doubles.
__device__ __forceinline__ void tree_reduce4(double (*sh)[4], double acc[4]) {
    const int t = threadIdx.x;
#pragma unroll
    for (int k = 0; k < 4; ++k) sh[t][k] = acc[k];
    __syncthreads();
    for (int s = kReduceThreads / 2; s > 0; s >>= 1) {
        if (t < s) {
#pragma unroll
            for (int k = 0; k < 4; ++k) sh[t][k] += sh[t + s][k];
        }
        __syncthreads();
    }
}

// Pass 1: workgroup g sums cells g*256 + t, stepping by the grid size, into
// partial[g][4] = (mass, momentum x, y, z).
// (The slot order is a template parameter: with a select at each load 128^3
// float64 took 98 us, 20 more.)
template <int Q, typename T, bool EX>
__global__ __launch_bounds__(kReduceThreads) void conservation_pass1(Planes<T> p, double *partial) {
    __shared__ double sh[kReduceThreads][4];
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    const int stride = gridDim.x * kReduceThreads;
    for (int c = blockIdx.x * kReduceThreads + threadIdx.x; c < p.cells; c += stride) {
        static_for<0, Q>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            using V = Vel<Q, i>;
            const double v = p.template load<Q, i, EX>(c);
            acc[0] += v + p.shift[i];
            if constexpr (V::x != 0) acc[1] += V::x * v;
            if constexpr (V::y != 0) acc[2] += V::y * v;
            if constexpr (V::z != 0) acc[3] += V::z * v;
        });
    }
    tree_reduce4(sh, acc);
    if (threadIdx.x == 0)
        for (int k = 0; k < 4; ++k) partial[4 * blockIdx.x + k] = sh[0][k];
}

// Pass 2: one workgroup folds the partials in a fixed order.
__global__ __launch_bounds__(kReduceThreads) void conservation_pass2(const double *partial, int n,
                                                                     double *out) {
    __shared__ double sh[kReduceThreads][4];
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int j = threadIdx.x; j < n; j += kReduceThreads)
        for (int k = 0; k < 4; ++k) acc[k] += partial[4 * j + k];
    tree_reduce4(sh, acc);
    if (threadIdx.x == 0)
        for (int k = 0; k < 4; ++k) out[k] = sh[0][k];
}

}  // namespace lbm

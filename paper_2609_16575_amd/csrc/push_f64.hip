// push_f64.hip -- plain FP64 particle step for gfx950: global FP64 positions,
// kept in the caller's order.  Same operations as the paper's cycle (Sec.
// 2.4-2.5): staggered CIC gather of E^n and of the centred B^n, relativistic
// Boris push, x += dt u/gamma, ZigZag deposit.  Periodic grids only
// (empic_create refuses walls on this path).
//
// Bytes per particle: 48 read + 48 written (+ 8 with a per-particle weight).
//
// k_push_f64: one thread per particle in storage order, fields gathered
// straight from global memory, the current scattered with global FP64
// atomics.
// k_bin_* and k_push_f64_tiles: the particles' slots are first binned by 8 x 8
// x 4 tiles of cells into an index list (two passes over the positions; the
// particles themselves stay where they are), then a workgroup per tile, or per
// slice of a dense one, pushes its particles from LDS windows of E, B and J.  Global FP64 atomics
// are what bounds the direct kernel: 24 G/s on scattered addresses, against
// 1600-2200 G/s for FP64 atomics in LDS.  64^3 cells, 2 x 2.1 M particles: see
// F64_TILED_MIN below.
#include "internal.hpp"

namespace empic {

namespace {

// index i of axis a wrapped into the grid
__device__ __forceinline__ int wrap64(const GridP &g, int a, long long i) {
    const long long n = g.n[a];
    if ((unsigned long long)i < (unsigned long long)n) return (int)i;
    if (i == -1) return (int)n - 1;
    if (i == n) return 0;
    const long long m = i % n;
    return (int)(m < 0 ? m + n : m);
}

// Interpolation points of one axis: offsets (index times the axis' stride) of
// the two node points and of the two half-cell points, and the fractions
struct Axis64 {
    int n[2], h[2];
    double fn, fh;
};

// staggered CIC interpolation of one component; sx, sy, sz: half-cell
__device__ __forceinline__ double gather_one(const double *F, bool sx, bool sy, bool sz,
                                             const Axis64 ax[3]) {
    const double fx = sx ? ax[0].fh : ax[0].fn, fy = sy ? ax[1].fh : ax[1].fn,
                 fz = sz ? ax[2].fh : ax[2].fn;
    double s = 0.0;
#pragma unroll
    for (int oz = 0; oz < 2; ++oz)
#pragma unroll
        for (int oy = 0; oy < 2; ++oy)
#pragma unroll
            for (int ox = 0; ox < 2; ++ox) {
                const int p = (sx ? ax[0].h[ox] : ax[0].n[ox]) + (sy ? ax[1].h[oy] : ax[1].n[oy]) +
                              (sz ? ax[2].h[oz] : ax[2].n[oz]);
                const double w = (ox ? fx : 1.0 - fx) * (oy ? fy : 1.0 - fy) * (oz ? fz : 1.0 - fz);
                s += w * F[p];
            }
    return s;
}

// E and centred B at a particle; F[q]: the six component arrays
__device__ __forceinline__ void gather_all(const double *const F[6], const Axis64 ax[3],
                                           double Ep[3], double Bp[3]) {
    Ep[0] = gather_one(F[0], true, false, false, ax);
    Ep[1] = gather_one(F[1], false, true, false, ax);
    Ep[2] = gather_one(F[2], false, false, true, ax);
    Bp[0] = gather_one(F[3], false, true, true, ax);
    Bp[1] = gather_one(F[4], true, false, true, ax);
    Bp[2] = gather_one(F[5], true, true, false, ax);
}

// relativistic Boris (standard t/s rotation), r = q dt / (2 m)
__device__ __forceinline__ void boris(double u[3], const double E[3], const double B[3], double r) {
    double um[3], t[3], s[3], up[3], upl[3];
    for (int a = 0; a < 3; ++a) um[a] = u[a] + r * E[a];
    const double gm = sqrt(1.0 + um[0] * um[0] + um[1] * um[1] + um[2] * um[2]);
    for (int a = 0; a < 3; ++a) t[a] = r * B[a] / gm;
    const double tt = t[0] * t[0] + t[1] * t[1] + t[2] * t[2];
    for (int a = 0; a < 3; ++a) s[a] = 2.0 * t[a] / (1.0 + tt);
    up[0] = um[0] + (um[1] * t[2] - um[2] * t[1]);
    up[1] = um[1] + (um[2] * t[0] - um[0] * t[2]);
    up[2] = um[2] + (um[0] * t[1] - um[1] * t[0]);
    upl[0] = um[0] + (up[1] * s[2] - up[2] * s[1]);
    upl[1] = um[1] + (up[2] * s[0] - up[0] * s[2]);
    upl[2] = um[2] + (up[0] * s[1] - up[1] * s[0]);
    for (int a = 0; a < 3; ++a) u[a] = upl[a] + r * E[a];
}

// one straight segment inside one cell: line integral of the bilinear weights,
// v[4 c + o1 + 2 o2] for the edge of component c at (o1, o2) along its two
// other axes c + 1, c + 2; amp[c] = q w d_c / (dt dV)
__device__ __forceinline__ void segment64(const double cell[3], const double s[3],
                                          const double e[3], const double amp[3], double v[12]) {
    double dxi[3], W[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        dxi[a] = e[a] - s[a];
        W[a] = 0.5 * (s[a] + e[a]) - cell[a];
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const int b1 = (c + 1) % 3, b2 = (c + 2) % 3;
        const double A = amp[c] * dxi[c];
        const double cross = dxi[b1] * dxi[b2] / 12.0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const double w1 = (q & 1) ? W[b1] : 1.0 - W[b1];
            const double w2 = (q >> 1) ? W[b2] : 1.0 - W[b2];
            const double sg = ((q & 1) == (q >> 1)) ? 1.0 : -1.0;
            v[4 * c + q] = A * (w1 * w2 + sg * cross);
        }
    }
}

struct F64Args {
    const double *F[6];  // E, centred B
    double *J[3];
    double kc[3];        // q d_c / (dt dV) (times the weight per particle)
    double r;            // q dt / (2 m)
};

// the 12 edge values of a segment in cell (i, j, k) (any index) to global J
__device__ __forceinline__ void add_global(const GridP &g, const F64Args &A, const double cell[3],
                                           const double v[12]) {
    int o[3][2];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const long long i = (long long)cell[a];
        const int st = a == 0 ? 1 : (a == 1 ? g.ext[0] : g.ext[0] * g.ext[1]);
        o[a][0] = wrap64(g, a, i) * st;
        o[a][1] = wrap64(g, a, i + 1) * st;
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const int b1 = (c + 1) % 3, b2 = (c + 2) % 3;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            atomicAdd(A.J[c] + o[c][0] + o[b1][q & 1] + o[b2][q >> 1], v[4 * c + q]);
    }
}

// ZigZag: relay point per axis, two segments each inside one cell.  add(cell,
// v) takes the 12 values of a cell; both segments of a move inside one cell
// are added at once.
template <class Add>
__device__ __forceinline__ void zigzag(const double xi1[3], const double xi2[3],
                                       const double f1[3], const double f2[3],
                                       const double amp[3], Add add) {
    double xr[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double lo = fmin(f1[a], f2[a]) + 1.0, hi = fmax(f1[a], f2[a]);
        const double mid = 0.5 * (xi1[a] + xi2[a]);
        xr[a] = fmin(lo, fmax(hi, mid));
    }
    double vA[12], vB[12];
    segment64(f1, xi1, xr, amp, vA);
    segment64(f2, xr, xi2, amp, vB);
    if (f1[0] == f2[0] && f1[1] == f2[1] && f1[2] == f2[2]) {
#pragma unroll
        for (int q = 0; q < 12; ++q) vA[q] += vB[q];
        add(f1, vA);
    } else {
        add(f1, vA);
        add(f2, vB);
    }
}

// the move after the Boris push: fault bits, xi2, and x += dt u / gamma
// (periodic wrap)
__device__ __forceinline__ void move64(const GridP &g, const double un[3], double gm,
                                       const double xi1[3], double xi2[3], double pos[3],
                                       uint32_t &bits) {
    if (!isfinite(gm)) bits |= EMPIC_FAULT_NONFINITE;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        xi2[a] = xi1[a] + g.dt * un[a] / (gm * g.d[a]);
        if (fabs(xi2[a] - xi1[a]) >= 1.0) bits |= EMPIC_FAULT_FAST;
        const double L = g.n[a] * g.d[a];
        double x = pos[a] + g.dt * un[a] / gm;
        if (x >= L) x -= L;
        if (x < 0.0) {
            x += L;
            if (x >= L) x = 0.0;
        }
        pos[a] = x;
    }
}

template <bool DRY>
__global__ __launch_bounds__(256) void k_push_f64(GridP g, F64Args A, SpeciesP sp,
                                                  long long count, uint32_t *fault,
                                                  double *partial) {
    __shared__ double sm[16];
    double *X = (double *)sp.pos[0], *Y = (double *)sp.pos[1], *Z = (double *)sp.pos[2];
    double *UX = (double *)sp.u[0], *UY = (double *)sp.u[1], *UZ = (double *)sp.u[2];
    const double *W = (const double *)sp.w;
    double ksum = 0.0;
    uint32_t bits = 0;
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x; p < count; p += stride) {
        double pos[3] = {X[p], Y[p], Z[p]};
        if (isnan(pos[0])) continue;
        const double wp = (sp.per_particle_w && W) ? W[p] : sp.w_species;
        double xi1[3], f1[3], Ep[3], Bp[3];
        Axis64 ax[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int st = a == 0 ? 1 : (a == 1 ? g.ext[0] : g.ext[0] * g.ext[1]);
            xi1[a] = pos[a] / g.d[a];
            f1[a] = floor(xi1[a]);
            const double t = xi1[a] - 0.5, fh = floor(t);
            const long long in = (long long)f1[a], ih = (long long)fh;
            ax[a].n[0] = wrap64(g, a, in) * st;
            ax[a].n[1] = wrap64(g, a, in + 1) * st;
            ax[a].h[0] = wrap64(g, a, ih) * st;
            ax[a].h[1] = wrap64(g, a, ih + 1) * st;
            ax[a].fn = xi1[a] - f1[a];
            ax[a].fh = t - fh;
        }
        gather_all(A.F, ax, Ep, Bp);
        double un[3] = {UX[p], UY[p], UZ[p]};
        boris(un, Ep, Bp, A.r);
        const double uu = un[0] * un[0] + un[1] * un[1] + un[2] * un[2];
        const double gm = sqrt(1.0 + uu);
        if (DRY) {
            ksum += wp * sp.m * uu / (gm + 1.0);
            continue;
        }
        double xi2[3], f2[3];
        move64(g, un, gm, xi1, xi2, pos, bits);
#pragma unroll
        for (int a = 0; a < 3; ++a) f2[a] = floor(xi2[a]);
        const double amp[3] = {wp * A.kc[0], wp * A.kc[1], wp * A.kc[2]};
        zigzag(xi1, xi2, f1, f2, amp,
               [&](const double cell[3], const double v[12]) { add_global(g, A, cell, v); });
        X[p] = pos[0];
        Y[p] = pos[1];
        Z[p] = pos[2];
        UX[p] = un[0];
        UY[p] = un[1];
        UZ[p] = un[2];
    }
    if (DRY) {
        const double s = block_reduce<false>(ksum, sm);
        if (threadIdx.x == 0) partial[blockIdx.x] = s;
    } else if (bits) {
        atomicOr(fault, bits);
    }
}

// ---------------------------------------------------------------------------
// Binned path
// ---------------------------------------------------------------------------
// 8 x 8 x 4 tiles; the field window holds cells -1 .. 8 (the half-cell points
// reach one cell down, the node points one up), the current window -1 .. 9
// (a move of less than a cell, and the far edges)
constexpr int T64X = 8, T64Y = 8, T64Z = 4;
constexpr int F64X = T64X + 2, F64Y = T64Y + 2, F64Z = T64Z + 2, F64V = F64X * F64Y * F64Z;
constexpr int J64X = T64X + 3, J64Y = T64Y + 3, J64Z = T64Z + 3, J64V = J64X * J64Y * J64Z;
constexpr int BIN_T = 1024, BIN_PER = 8;      // particles of one workgroup of the binning passes
constexpr int BIN_LDS = 16384;                // tiles whose counters fit in LDS (64 KB)

struct Tiles64 {
    int nt[3];
    int ntiles;
    int32_t *counts, *offs, *cursor;  // ntiles, ntiles + 1, ntiles
    int32_t *more;                    // slices beyond the first of the tiles before, ntiles + 1
    int32_t *perm;                    // slots grouped by tile
    int slice;                        // particles of one workgroup of the push
};

// tile of slot p, -1: skipped (NaN)
__device__ __forceinline__ int tile64(const GridP &g, const Tiles64 &t, const SpeciesP &sp,
                                      long long p) {
    const double x = ((const double *)sp.pos[0])[p];
    if (isnan(x)) return -1;
    const double y = ((const double *)sp.pos[1])[p], z = ((const double *)sp.pos[2])[p];
    const int i = wrap64(g, 0, (long long)floor(x / g.d[0])),
              j = wrap64(g, 1, (long long)floor(y / g.d[1])),
              k = wrap64(g, 2, (long long)floor(z / g.d[2]));
    return i / T64X + t.nt[0] * (j / T64Y + t.nt[1] * (k / T64Z));
}

// FILL = false: tile populations into counts.  FILL = true: slots into perm,
// from the tiles' cursors.  With the counters in LDS (dyn), a workgroup makes
// one global atomic per tile that it meets.
template <bool FILL, bool LDS>
__global__ __launch_bounds__(BIN_T) void k_bin(GridP g, Tiles64 t, SpeciesP sp, long long count) {
    extern __shared__ int hist[];
    const long long p0 = blockIdx.x * (long long)(BIN_T * BIN_PER) + threadIdx.x;
    int tl[BIN_PER], rk[BIN_PER];
#pragma unroll
    for (int k = 0; k < BIN_PER; ++k) {
        const long long p = p0 + (long long)k * BIN_T;
        tl[k] = p < count ? tile64(g, t, sp, p) : -1;
    }
    if constexpr (LDS) {
        for (int e = threadIdx.x; e < t.ntiles; e += BIN_T) hist[e] = 0;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < BIN_PER; ++k)
            if (tl[k] >= 0) rk[k] = atomicAdd(hist + tl[k], 1);
        __syncthreads();
        for (int e = threadIdx.x; e < t.ntiles; e += BIN_T) {
            const int h = hist[e];
            if (h) hist[e] = atomicAdd((FILL ? t.cursor : t.counts) + e, h);
        }
        if constexpr (FILL) {
            __syncthreads();
#pragma unroll
            for (int k = 0; k < BIN_PER; ++k)
                if (tl[k] >= 0) t.perm[hist[tl[k]] + rk[k]] = (int32_t)(p0 + (long long)k * BIN_T);
        }
    } else {
#pragma unroll
        for (int k = 0; k < BIN_PER; ++k)
            if (tl[k] >= 0) {
                const int d = atomicAdd((FILL ? t.cursor : t.counts) + tl[k], 1);
                if (FILL) t.perm[d] = (int32_t)(p0 + (long long)k * BIN_T);
            }
    }
}

// exclusive scans of the populations into offs and cursor, and of the slices
// beyond a tile's first into more (one workgroup, both in one 64-bit scan); the
// populations are cleared for the next species or step
__global__ __launch_bounds__(1024) void k_bin_scan(Tiles64 t) {
    __shared__ unsigned long long sm[16];
    unsigned long long carry = 0;
    for (int base = 0; base < t.ntiles; base += 1024) {
        const int e = base + threadIdx.x;
        const unsigned n = e < t.ntiles ? (unsigned)t.counts[e] : 0u;
        const unsigned long long v =
            n ? n | (unsigned long long)((n - 1u) / (unsigned)t.slice) << 32 : 0ull;
        const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
        unsigned long long x = v;
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned long long y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63) sm[wid] = x;
        __syncthreads();
        unsigned long long off = carry, tot = 0;
        for (int w = 0; w < 16; ++w) {
            if (w < wid) off += sm[w];
            tot += sm[w];
        }
        __syncthreads();
        if (e < t.ntiles) {
            const unsigned long long b = off + x - v;
            t.offs[e] = t.cursor[e] = (int32_t)b;
            t.more[e] = (int32_t)(b >> 32);
            t.counts[e] = 0;
        }
        carry += tot;
    }
    if (threadIdx.x == 0) {
        t.offs[t.ntiles] = (int32_t)carry;
        t.more[t.ntiles] = (int32_t)(carry >> 32);
    }
}

__global__ __launch_bounds__(256, 2) void k_push_f64_tiles(GridP g, F64Args A, Tiles64 t,
                                                           SpeciesP sp, uint32_t *fault) {
    __shared__ double sF[6 * F64V];
    __shared__ double sJ[3 * J64V];
    // first the tiles' first slices, XCD-contiguous, then the others in turn
    const int nb8 = (t.ntiles + 7) / 8;
    int tile = ((int)blockIdx.x & 7) * nb8 + ((int)blockIdx.x >> 3), part = 0;
    if ((int)blockIdx.x >= 8 * nb8) {
        const int q = (int)blockIdx.x - 8 * nb8;
        if (q >= t.more[t.ntiles]) return;
        tile = 0;  // the last tile with more[tile] <= q
        for (int hi = t.ntiles; hi - tile > 1;) {
            const int mid = (tile + hi) >> 1;
            if (t.more[mid] <= q) tile = mid;
            else hi = mid;
        }
        part = q - t.more[tile] + 1;
    }
    if (tile >= t.ntiles) return;
    // (beg + slice, and the loop's last q, can pass 2^31 - 1)
    const int beg = t.offs[tile] + part * t.slice, end = beg + min(t.offs[tile + 1] - beg, t.slice);
    if (beg >= end) return;
    const int tx = tile % t.nt[0], tyz = tile / t.nt[0];
    const int org[3] = {tx * T64X, (tyz % t.nt[1]) * T64Y, (tyz / t.nt[1]) * T64Z};
    const int tid = threadIdx.x;
    for (int e = tid; e < F64V; e += 256) {
        const int lz = e / (F64X * F64Y), r = e - lz * (F64X * F64Y), ly = r / F64X, lx = r - ly * F64X;
        const int o = wrap64(g, 0, org[0] - 1 + lx) +
                      g.ext[0] * (wrap64(g, 1, org[1] - 1 + ly) + g.ext[1] * wrap64(g, 2, org[2] - 1 + lz));
#pragma unroll
        for (int q = 0; q < 6; ++q) sF[q * F64V + e] = A.F[q][o];
    }
    for (int e = tid; e < 3 * J64V; e += 256) sJ[e] = 0.0;
    __syncthreads();
    const double *const F[6] = {sF, sF + F64V, sF + 2 * F64V, sF + 3 * F64V, sF + 4 * F64V, sF + 5 * F64V};
    double *X[3] = {(double *)sp.pos[0], (double *)sp.pos[1], (double *)sp.pos[2]};
    double *U[3] = {(double *)sp.u[0], (double *)sp.u[1], (double *)sp.u[2]};
    const double *W = sp.per_particle_w ? (const double *)sp.w : nullptr;
    uint32_t bits = 0;
    for (unsigned q = (unsigned)(beg + tid); q < (unsigned)end; q += 256u) {
        const int p = t.perm[q];
        double pos[3], un[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            pos[a] = X[a][p];
            un[a] = U[a][p];
        }
        const double wp = W ? W[p] : sp.w_species;
        double xi1[3], f1[3], Ep[3], Bp[3];
        int l[3];
        Axis64 ax[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int st = a == 0 ? 1 : (a == 1 ? F64X : F64X * F64Y);
            xi1[a] = pos[a] / g.d[a];
            f1[a] = floor(xi1[a]);
            const double th = xi1[a] - 0.5, fh = floor(th);
            l[a] = wrap64(g, a, (long long)f1[a]) - org[a];  // 0 .. tile side - 1
            const int h = l[a] + 1 - (fh < f1[a] ? 1 : 0);   // window index of the half-cell point
            ax[a].n[0] = (l[a] + 1) * st;
            ax[a].n[1] = (l[a] + 2) * st;
            ax[a].h[0] = h * st;
            ax[a].h[1] = (h + 1) * st;
            ax[a].fn = xi1[a] - f1[a];
            ax[a].fh = th - fh;
        }
        gather_all(F, ax, Ep, Bp);
        boris(un, Ep, Bp, A.r);
        const double gm = sqrt(1.0 + (un[0] * un[0] + un[1] * un[1] + un[2] * un[2]));
        double xi2[3], f2[3];
        move64(g, un, gm, xi1, xi2, pos, bits);
        bool near = true;  // the move ends in this cell or one next to it
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            f2[a] = floor(xi2[a]);
            near = near && fabs(f2[a] - f1[a]) <= 1.0;
        }
        const double amp[3] = {wp * A.kc[0], wp * A.kc[1], wp * A.kc[2]};
        zigzag(xi1, xi2, f1, f2, amp, [&](const double cell[3], const double v[12]) {
            if (!near) {
                add_global(g, A, cell, v);
                return;
            }
            const int b = (l[0] + 1 + (int)(cell[0] - f1[0])) +
                          J64X * ((l[1] + 1 + (int)(cell[1] - f1[1])) +
                                  J64Y * (l[2] + 1 + (int)(cell[2] - f1[2])));
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const int s1 = c == 0 ? J64X : (c == 1 ? J64X * J64Y : 1);
                const int s2 = c == 0 ? J64X * J64Y : (c == 1 ? 1 : J64X);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    atomicAdd(sJ + c * J64V + b + (e & 1) * s1 + (e >> 1) * s2, v[4 * c + e]);
            }
        });
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            X[a][p] = pos[a];
            U[a][p] = un[a];
        }
    }
    if (bits) atomicOr(fault, bits);
    __syncthreads();
    for (int e = tid; e < J64V; e += 256) {
        const int lz = e / (J64X * J64Y), r = e - lz * (J64X * J64Y), ly = r / J64X, lx = r - ly * J64X;
        const int o = wrap64(g, 0, org[0] - 1 + lx) +
                      g.ext[0] * (wrap64(g, 1, org[1] - 1 + ly) + g.ext[1] * wrap64(g, 2, org[2] - 1 + lz));
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double v = sJ[c * J64V + e];
            if (v != 0.0) atomicAdd(A.J[c] + o, v);
        }
    }
}

__global__ void k_kinetic_f64(SpeciesP sp, long long count, double *partial) {
    __shared__ double sm[16];
    const double *UX = (const double *)sp.u[0], *UY = (const double *)sp.u[1],
                 *UZ = (const double *)sp.u[2], *X = (const double *)sp.pos[0];
    const double *W = (const double *)sp.w;
    double ksum = 0.0;
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x; p < count; p += stride) {
        if (isnan(X[p])) continue;
        const double uu = UX[p] * UX[p] + UY[p] * UY[p] + UZ[p] * UZ[p];
        const double wp = (sp.per_particle_w && W) ? W[p] : sp.w_species;
        ksum += wp * sp.m * uu / (sqrt(1.0 + uu) + 1.0);
    }
    const double s = block_reduce<false>(ksum, sm);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// CIC charge density at nodes, rho += (q w / dV) prod_a w_a
__global__ void k_rho_f64(GridP g, SpeciesP sp, long long count, double *rho) {
    const long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (p >= count) return;
    const double *X = (const double *)sp.pos[0], *Y = (const double *)sp.pos[1],
                 *Z = (const double *)sp.pos[2];
    const double *W = (const double *)sp.w;
    if (isnan(X[p])) return;
    const double dV = g.d[0] * g.d[1] * g.d[2];
    const double qsp = sp.q * ((sp.per_particle_w && W) ? W[p] : sp.w_species);
    const double pos[3] = {X[p], Y[p], Z[p]};
    long long i0[3];
    double f[3];
    for (int a = 0; a < 3; ++a) {
        const double t = pos[a] / g.d[a];
        const double fl = floor(t);
        i0[a] = (long long)fl;
        f[a] = t - fl;
    }
    for (int oz = 0; oz < 2; ++oz)
        for (int oy = 0; oy < 2; ++oy)
            for (int ox = 0; ox < 2; ++ox) {
                const long long ip =
                    wrap64(g, 0, i0[0] + ox) +
                    (long long)g.ext[0] * (wrap64(g, 1, i0[1] + oy) +
                                           (long long)g.ext[1] * wrap64(g, 2, i0[2] + oz));
                const double wt = (ox ? f[0] : 1.0 - f[0]) * (oy ? f[1] : 1.0 - f[1]) *
                                  (oz ? f[2] : 1.0 - f[2]);
                atomicAdd(rho + ip, qsp / dV * wt);
            }
}

__global__ void k_load_f64(GridP g, SpeciesP sp, long long count, const double *pos,
                           const double *u, const double *w, const int32_t *ids, uint32_t *fault) {
    const long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (p >= count) return;
    for (int a = 0; a < 3; ++a) {
        const double x = pos[3 * p + a];
        if (!(x >= 0.0 && x < g.n[a] * g.d[a])) atomicOr(fault, (uint32_t)EMPIC_FAULT_CELL);
        ((double *)sp.pos[a])[p] = x;
        ((double *)sp.u[a])[p] = u[3 * p + a];
    }
    if (sp.id) sp.id[p] = ids ? ids[p] : (int32_t)p;
    if (sp.w && w) ((double *)sp.w)[p] = w[p];
}

__global__ void k_store_f64(SpeciesP sp, long long count, double *pos, double *u, int32_t *ids) {
    const long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (p >= count) return;
    const bool dead = isnan(((const double *)sp.pos[0])[p]);
    for (int a = 0; a < 3; ++a) {
        pos[3 * p + a] = ((const double *)sp.pos[a])[p];
        u[3 * p + a] = ((const double *)sp.u[a])[p];
    }
    if (ids) ids[p] = dead ? -1 : (sp.id ? sp.id[p] : (int32_t)p);
}

inline unsigned nblk(long long n, int t) { return (unsigned)((n + t - 1) / t); }

}  // namespace

namespace {
F64Args args64(const GridP &g, double *const E[3], double *const Bbar[3], double *const J[3],
               const SpeciesP &sp) {
    F64Args A{};
    const double dV = g.d[0] * g.d[1] * g.d[2];
    for (int a = 0; a < 3; ++a) {
        A.F[a] = E[a];
        A.F[3 + a] = Bbar[a];
        A.J[a] = J ? J[a] : nullptr;
        A.kc[a] = sp.q * g.d[a] / (g.dt * dV);
    }
    A.r = sp.q * g.dt / (2.0 * sp.m);
    return A;
}
}  // namespace

// From this many particles on, and this many per tile, the binned path is taken.
// One step of 8 particles per cell, fresh and after 600 steps of mixing (direct |
// binned): 55 k particles (4 per cell): 49, 43 | 62, 60 us (its four launches cost
// more than it saves); 131 k: 94, 77 | 64, 63; 2.1 M: 1133, 868 | 156, 183; 7.1 M:
// 3914, 2854 | 486, 667.  (2.1 M took 2912 us for the push alone with 64-bit modulo
// index arithmetic and 24 global atomics per particle.)  On sparse grids the
// windows cost more than they save, 256^3: 12 per tile 1684 | 1826 us, 24: 2463 |
// 2082; 128^3: 12 per tile 158 | 195, 24: 269 | 210; 512 x 2 x 512: 103 | 148, 198 | 153.
// The binned push is bound by its scattered 8-byte particle accesses once the
// plasma has mixed: the storage order is the caller's.
constexpr long long F64_TILED_MIN = 98304, F64_TILE_MIN = 20;
// A tile's particles are pushed in slices of 1 / F64_SLICES of all of them, by a
// workgroup each: a plasma that fills a few tiles has them share the chip, an even
// one of as many tiles is left whole (every slice loads and flushes the windows).
// Whole tiles | slices for 128, 256, 512 workgroups: 1 M on 8 x 8 x 4 11500 | 166, 143,
// 136 us; 3.2 M on 16^3 2634 | 473, 550, 516; 2 M in 8^3 cells of 128^3 11076 | 572, 418,
// 341; 3.2 M on 32^3 542 | 546, 655, 644.
constexpr long long F64_SLICES = 128, F64_SLICE_MIN = 1024;

void launch_push_f64(const GridP &g, double *const E[3], double *const Bbar[3],
                     double *const J[3], const SpeciesP &sp, long long count, int32_t *counts,
                     int32_t *slots, uint32_t *fault, hipStream_t s) {
    if (count <= 0) return;
    const F64Args A = args64(g, E, Bbar, J, sp);
    Tiles64 t;
    t.nt[0] = (g.n[0] + T64X - 1) / T64X;
    t.nt[1] = (g.n[1] + T64Y - 1) / T64Y;
    t.nt[2] = (g.n[2] + T64Z - 1) / T64Z;
    t.ntiles = t.nt[0] * t.nt[1] * t.nt[2];
    if (count < F64_TILED_MIN || count < F64_TILE_MIN * t.ntiles) {
        hipLaunchKernelGGL(k_push_f64<false>, dim3(nblk(count, 256)), dim3(256), 0, s, g, A, sp,
                           count, fault, nullptr);
        return;
    }
    t.counts = counts;
    t.offs = counts + t.ntiles;
    t.cursor = t.offs + t.ntiles + 1;
    t.more = t.cursor + t.ntiles;
    t.perm = slots;
    t.slice = (int)(count / F64_SLICES > F64_SLICE_MIN ? count / F64_SLICES : F64_SLICE_MIN);
    const dim3 nb(nblk(count, BIN_T * BIN_PER));
    const bool lds = t.ntiles <= BIN_LDS;
    const unsigned shm = lds ? (unsigned)t.ntiles * 4u : 0u;
    hipLaunchKernelGGL(lds ? (k_bin<false, true>) : (k_bin<false, false>), nb, dim3(BIN_T), shm, s,
                       g, t, sp, count);
    hipLaunchKernelGGL(k_bin_scan, dim3(1), dim3(1024), 0, s, t);
    hipLaunchKernelGGL(lds ? (k_bin<true, true>) : (k_bin<true, false>), nb, dim3(BIN_T), shm, s, g,
                       t, sp, count);
    // (the tiles' slices beyond their first are at most count / slice)
    hipLaunchKernelGGL(k_push_f64_tiles,
                       dim3((unsigned)(8 * ((t.ntiles + 7) / 8) + count / t.slice)), dim3(256), 0,
                       s, g, A, t, sp, fault);
}

void launch_dry_push_f64(const GridP &g, double *const E[3], double *const Bbar[3],
                         const SpeciesP &sp, long long count, double *partial_slot,
                         uint32_t *fault, hipStream_t s) {
    const F64Args A = args64(g, E, Bbar, nullptr, sp);
    hipLaunchKernelGGL(k_push_f64<true>, dim3(RED_BLOCKS), dim3(256), 0, s, g, A, sp, count,
                       fault, partial_slot);
}

void launch_kinetic_f64(const SpeciesP &sp, long long count, double *partial_slot,
                        hipStream_t s) {
    hipLaunchKernelGGL(k_kinetic_f64, dim3(RED_BLOCKS), dim3(256), 0, s, sp, count, partial_slot);
}

void launch_rho_f64(const GridP &g, const SpeciesP &sp, long long count, double *rho,
                    hipStream_t s) {
    if (count <= 0) return;
    hipLaunchKernelGGL(k_rho_f64, dim3(nblk(count, 256)), dim3(256), 0, s, g, sp, count, rho);
}

void launch_load_f64(const GridP &g, const SpeciesP &sp, long long count, const double *pos,
                     const double *u, const double *w, const int32_t *ids, uint32_t *fault,
                     hipStream_t s) {
    if (count <= 0) return;
    hipLaunchKernelGGL(k_load_f64, dim3(nblk(count, 256)), dim3(256), 0, s, g, sp, count, pos, u,
                       w, ids, fault);
}

void launch_store_f64(const SpeciesP &sp, long long count, double *pos, double *u, int32_t *ids,
                      hipStream_t s) {
    if (count <= 0) return;
    hipLaunchKernelGGL(k_store_f64, dim3(nblk(count, 256)), dim3(256), 0, s, sp, count, pos, u,
                       ids);
}

}  // namespace empic

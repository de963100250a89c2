// fields.hip -- Yee FDTD kernels for gfx950 (Sec. 2.3 of KEMPIC-3D).
//
// One thread per grid point on the flat index (x fastest), so that every
// component load and store of a wave is 256 contiguous bytes whatever the
// grid's width; a thread updates all three components at its point.
// Workgroups of one XCD take a contiguous run of the grid, so that the y and
// z neighbours of a stencil come from that XCD's own L2.  Periodic neighbours
// wrap; on a walled (absorbing or PEC) axis the validity rules below keep
// every neighbour inside the stored array.
//
// Bytes per cell (FP32): Faraday reads E, B (24) and writes B, Bbar (24) and
// zeroes the int64 sums of J (24); Ampere reads those, E and B (48) and
// writes E (12), and J (12) in the last step of a call.  Without particles there
// is no Bbar and there are no sums: 36 and 36 (+12), or 48 in one pass where
// k_vacuum takes the step (vacuum_fits).
// Bound by HBM and the memory-side cache.  The vacuum waveguide on 91 x 46 x 3001
// nodes: 0.645 ms per step with one 64 x 4 workgroup per patch of rows (the second
// of two per row 42 % full), the sums zeroed and read, J written every step and the
// Mur and PEC planes in kernels of their own; 0.224 with the two point kernels on
// the flat index, 0.202 in one pass (3.0 TB/s; a large copy: 4.7).
#include <cmath>
#include <utility>

#include "internal.hpp"

namespace empic {

namespace {

struct Pt {
    int idx[3];
    long long p;
    long long st[3];  // strides
};

constexpr int PT_THREADS = 256;

__device__ __forceinline__ bool make_point(const GridP &g, Pt &q) {
    const uint32_t nb8 = gridDim.x >> 3;
    const uint32_t b = (blockIdx.x & 7u) * nb8 + (blockIdx.x >> 3);  // XCD-contiguous
    const uint32_t p = b * PT_THREADS + threadIdx.x;
    if (p >= (uint32_t)g.V) return false;
    const uint32_t r = fastdiv(p, g.div[0]), k = fastdiv(r, g.div[1]);
    q.idx[0] = (int)(p - r * g.div[0].d);
    q.idx[1] = (int)(r - k * g.div[1].d);
    q.idx[2] = (int)k;
    q.st[0] = 1;
    q.st[1] = g.ext[0];
    q.st[2] = (long long)g.ext[0] * g.ext[1];
    q.p = p;
    return true;
}

// offset of the +1 / -1 neighbour along axis a (periodic wrap)
__device__ inline long long up(const GridP &g, const Pt &q, int a) {
    return (g.bc[a] == EMPIC_BC_PERIODIC && q.idx[a] == g.n[a] - 1) ? -(long long)(g.n[a] - 1) * q.st[a]
                                                                   : q.st[a];
}
__device__ inline long long dn(const GridP &g, const Pt &q, int a) {
    return (g.bc[a] == EMPIC_BC_PERIODIC && q.idx[a] == 0) ? (long long)(g.n[a] - 1) * q.st[a]
                                                           : -q.st[a];
}

// A component half-staggered along walled axis a has n values: entry n is padding.
__device__ inline bool valid_B(const GridP &g, const Pt &q, int c) {
    for (int a = 0; a < 3; ++a)
        if (g.bc[a] != EMPIC_BC_PERIODIC && a != c && q.idx[a] == g.n[a]) return false;
    return true;
}
// E_c updated by Ampere: valid and not tangential on a walled face (those
// belong to the Mur or PEC condition).
__device__ inline bool ampere_E(const GridP &g, const Pt &q, int c) {
    for (int a = 0; a < 3; ++a) {
        if (g.bc[a] == EMPIC_BC_PERIODIC) continue;
        if (a == c && q.idx[a] == g.n[a]) return false;
        if (a != c && (q.idx[a] == 0 || q.idx[a] == g.n[a])) return false;
    }
    return true;
}

// on a PEC face with E_c tangential to it: stays zero
__device__ inline bool pec_zero(const GridP &g, const int idx[3], int c) {
    bool z = false;
#pragma unroll
    for (int a = 0; a < 3; ++a)
        z = z || (g.bc[a] == EMPIC_BC_PEC && a != c && (idx[a] == 0 || idx[a] == g.n[a]));
    return z;
}

// First-order Mur faces (READING of the boundary module: tangential E on the
// faces of an absorbing axis) need E^n on the node planes 0, 1, n - 1, n of
// the axis after Ampere has updated E in place.  Faraday reads E^n everywhere
// and saves them: planes[a][c'][q][point], q = the plane, point = i_b1 +
// ext[b1] * i_b2 over the other two axes.
template <typename T>
__device__ __forceinline__ void mur_save(const GridP &g, const Pt &q, const T *const E[3],
                                         T *planes, long long pstride) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (g.bc[a] != EMPIC_BC_ABSORBING) continue;
        const int i = q.idx[a], n = g.n[a];
        if (i > 1 && i < n - 1) continue;
        const int b1 = a == 0 ? 1 : 0, b2 = a == 2 ? 1 : 2;
        const long long t = q.idx[b1] + (long long)g.ext[b1] * q.idx[b2];
        const int at[4] = {0, 1, n - 1, n};  // with n = 2 plane 1 is saved as both
#pragma unroll
        for (int ci = 0; ci < 2; ++ci) {
            const T v = E[ci == 0 ? b1 : b2][q.p];
#pragma unroll
            for (int qq = 0; qq < 4; ++qq)
                if (i == at[qq]) planes[(((long long)a * 2 + ci) * 4 + qq) * pstride + t] = v;
        }
    }
}

template <typename T>
__global__ __launch_bounds__(PT_THREADS) void k_faraday(
    GridP g, const T *__restrict__ Ex, const T *__restrict__ Ey, const T *__restrict__ Ez,
    T *__restrict__ Bx, T *__restrict__ By, T *__restrict__ Bz, T *__restrict__ Bbx,
    T *__restrict__ Bby, T *__restrict__ Bbz, T *__restrict__ Jx, T *__restrict__ Jy,
    T *__restrict__ Jz, unsigned long long *__restrict__ Jfx,
    unsigned long long *__restrict__ Jfy, unsigned long long *__restrict__ Jfz,
    unsigned *__restrict__ fb_reset, int write_B, T *__restrict__ planes, long long pstride) {
    Pt q;
    if (!make_point(g, q)) return;
    const long long p = q.p;
    if (fb_reset && p == 0) {  // the out-of-window counts of the coming push
        fb_reset[0] = 0u;
        fb_reset[1] = 0u;
        fb_reset[2] = 0u;
    }
    if (Jx) {
        Jx[p] = T(0);
        Jy[p] = T(0);
        Jz[p] = T(0);
    }
    if (Jfx) {  // the fixed-point current of the FP32 path
        Jfx[p] = 0ull;
        Jfy[p] = 0ull;
        Jfz[p] = 0ull;
    }
    if (planes) {
        const T *const E[3] = {Ex, Ey, Ez};
        mur_save(g, q, E, planes, pstride);
    }
    // evaluated in FP64 and rounded once per stored value (see k_ampere)
    const double dt = g.dt;
    const double ix = g.inv_d[0], iy = g.inv_d[1], iz = g.inv_d[2];
    // B^{n+1/2} = B^{n-1/2} - dt curl E^n (forward differences); Bbar = average
    if (valid_B(g, q, 0)) {
        const double curl = ((double)Ez[p + up(g, q, 1)] - (double)Ez[p]) * iy -
                            ((double)Ey[p + up(g, q, 2)] - (double)Ey[p]) * iz;
        const double old = (double)Bx[p], nw = old - dt * curl;
        if (write_B) Bx[p] = (T)nw;
        if (Bbx) Bbx[p] = (T)(0.5 * (old + nw));
    } else if (Bbx) {
        Bbx[p] = T(0);
    }
    if (valid_B(g, q, 1)) {
        const double curl = ((double)Ex[p + up(g, q, 2)] - (double)Ex[p]) * iz -
                            ((double)Ez[p + up(g, q, 0)] - (double)Ez[p]) * ix;
        const double old = (double)By[p], nw = old - dt * curl;
        if (write_B) By[p] = (T)nw;
        if (Bbx) Bby[p] = (T)(0.5 * (old + nw));
    } else if (Bbx) {
        Bby[p] = T(0);
    }
    if (valid_B(g, q, 2)) {
        const double curl = ((double)Ey[p + up(g, q, 0)] - (double)Ey[p]) * ix -
                            ((double)Ex[p + up(g, q, 1)] - (double)Ex[p]) * iy;
        const double old = (double)Bz[p], nw = old - dt * curl;
        if (write_B) Bz[p] = (T)nw;
        if (Bbx) Bbz[p] = (T)(0.5 * (old + nw));
    } else if (Bbx) {
        Bbz[p] = T(0);
    }
}

// J in units of 1/jscale (int64, exact sums of the deposit) -> T, one rounding
template <typename T>
__device__ __forceinline__ T j_from_fixed(long long x, double jinv) {
    return (T)((double)x * jinv);
}

// MODE J_FIXED (the FP32 path): J is formed from the fixed-point sums at every
// point; J_NONE: J is zero.  WJ writes that J out: only the last step of a call
// needs to, the push neither reads nor adds to it.  Bound by memory: with the
// Faraday kernel 84 bytes per point and step of a grid without particles where
// every step writes J, 72 where it does not (91 x 46 x 3001, 50 steps: 12.74
// and 11.19 ms).  Tangential E on PEC faces is set to zero here
// (launch_mur_apply leaves it so).
template <typename T, int MODE, bool WJ>
__global__ __launch_bounds__(PT_THREADS) void k_ampere(
    GridP g, T *__restrict__ Ex, T *__restrict__ Ey, T *__restrict__ Ez, const T *__restrict__ Bx,
    const T *__restrict__ By, const T *__restrict__ Bz, T *__restrict__ Jx, T *__restrict__ Jy,
    T *__restrict__ Jz, const long long *__restrict__ Jfx, const long long *__restrict__ Jfy,
    const long long *__restrict__ Jfz, double jinv) {
    Pt q;
    if (!make_point(g, q)) return;
    const long long p = q.p;
    // Evaluated in FP64 and rounded once per stored value: in FP32 the
    // rounding of J, of curl - J and of the two-part update add up coherently
    // on a quiet plasma (every cell of a wave front rounds alike).  The kernel
    // is bound by memory, and gfx950 issues FP64 at the FP32 (unpacked) rate.
    double jx = 0.0, jy = 0.0, jz = 0.0;
    if constexpr (MODE == J_FIXED) {
        jx = (double)Jfx[p] * jinv;
        jy = (double)Jfy[p] * jinv;
        jz = (double)Jfz[p] * jinv;
    }
    if constexpr (MODE == J_READ) {
        jx = (double)Jx[p];
        jy = (double)Jy[p];
        jz = (double)Jz[p];
    } else if constexpr (WJ) {
        Jx[p] = (T)jx;
        Jy[p] = (T)jy;
        Jz[p] = (T)jz;
    }
    const double dt = g.dt;
    const double ix = g.inv_d[0], iy = g.inv_d[1], iz = g.inv_d[2];
    // E^{n+1} = E^n + dt curl B^{n+1/2} - dt J^{n+1/2} (backward differences)
    if (ampere_E(g, q, 0)) {
        const double curl = ((double)Bz[p] - (double)Bz[p + dn(g, q, 1)]) * iy -
                            ((double)By[p] - (double)By[p + dn(g, q, 2)]) * iz;
        Ex[p] = (T)((double)Ex[p] + dt * (curl - jx));
    } else if (pec_zero(g, q.idx, 0)) {
        Ex[p] = T(0);
    }
    if (ampere_E(g, q, 1)) {
        const double curl = ((double)Bx[p] - (double)Bx[p + dn(g, q, 2)]) * iz -
                            ((double)Bz[p] - (double)Bz[p + dn(g, q, 0)]) * ix;
        Ey[p] = (T)((double)Ey[p] + dt * (curl - jy));
    } else if (pec_zero(g, q.idx, 1)) {
        Ey[p] = T(0);
    }
    if (ampere_E(g, q, 2)) {
        const double curl = ((double)By[p] - (double)By[p + dn(g, q, 0)]) * ix -
                            ((double)Bx[p] - (double)Bx[p + dn(g, q, 1)]) * iy;
        Ez[p] = (T)((double)Ez[p] + dt * (curl - jz));
    } else if (pec_zero(g, q.idx, 2)) {
        Ez[p] = T(0);
    }
}

// Faraday and Ampere of a step without particles in one pass, from E, B to
// Eo, Bo (neighbouring workgroups still read the old values).  A workgroup
// marches along z over zc planes of a 31 x 15 patch: its 32 x 16 threads form
// B' at the patch and at the row and column below it, hand it to their +x and
// +y neighbours through LDS and to the plane above in registers, and E' follows
// without a trip to memory.  Loads run one plane ahead of the arithmetic.
// Bound by memory: 48 bytes per point and step, where the two point kernels
// move 72 (the halos come from the XCD's L2, whose workgroups share a range of
// z).  Out of place the arrays take twice the room in the memory-side cache,
// which the point kernels live on (vacuum_fits): 91 x 46 x 3001, 224 -> 202 us per
// step, and not by the ratio of the bytes; nontemporal accesses lose what is left
// of it (249).  The same expressions as k_faraday and k_ampere and the same bits,
// so that a run does not depend on how its steps are grouped into calls.
constexpr int VX = 32, VY = 16, VT = VX * VY;

template <typename T>
struct VacIO {
    const T *E[3], *B[3];
    T *Eo[3], *Bo[3];
    T *J[3];  // zeroed when given (the last step of a call)
    T *planes;
    long long pstride;
};

// what a thread reads of one plane: E beside its point and old B
template <typename T>
struct VacPlane {
    T ez, eyx, ezx, exy, ezy, exz, eyz, b[3];
};

template <typename T>
__global__ __launch_bounds__(VT, 4) void k_vacuum(GridP g, VacIO<T> F, int nbx, int nby, int nbz,
                                                  int zc) {
    __shared__ T sB[2][3][VT];
    const int nb8 = gridDim.x >> 3;
    const int id = (blockIdx.x & 7) * nb8 + (blockIdx.x >> 3);  // XCD-contiguous
    if (id >= nbx * nby * nbz) return;
    const int bz = id / (nbx * nby), bxy = id - bz * (nbx * nby);
    const int by = bxy / nbx, bx = bxy - by * nbx;
    const int tid = threadIdx.x, tx = tid & (VX - 1), ty = tid / VX;

    Pt q;
    q.st[0] = 1;
    q.st[1] = g.ext[0];
    q.st[2] = (long long)g.ext[0] * g.ext[1];
    q.idx[0] = bx * (VX - 1) + tx - 1;
    q.idx[1] = by * (VY - 1) + ty - 1;
    bool in = true;  // the thread's column lies on the grid
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        if (q.idx[a] >= g.ext[a]) in = false;
        if (q.idx[a] < 0) {
            q.idx[a] = g.n[a] - 1;  // below a periodic axis' first point
            in = in && g.bc[a] == EMPIC_BC_PERIODIC;
        }
    }
    const bool own = in && tx > 0 && ty > 0;
    const int zs = bz * zc, ze = min(zs + zc, g.ext[2]);
    // the plane below: of a walled axis' first point nothing reads it
    const bool below = zs > 0 || g.bc[2] == EMPIC_BC_PERIODIC;
    int z = below ? (zs > 0 ? zs - 1 : g.n[2] - 1) : zs;

    // +1 neighbours; past a wall the component is padding and nothing reads them
    const auto upc = [&](int a) {
        return g.bc[a] != EMPIC_BC_PERIODIC && q.idx[a] == g.n[a] ? 0ll : up(g, q, a);
    };
    const long long ux = in ? upc(0) : 0, uy = in ? upc(1) : 0;
    const long long col = q.idx[0] + (long long)g.ext[0] * q.idx[1];
    const auto load = [&](int zz, VacPlane<T> &v) {
        q.idx[2] = zz;
        const long long p = col + zz * q.st[2], uz = upc(2);
        v.ez = F.E[2][p];
        v.eyx = F.E[1][p + ux];
        v.ezx = F.E[2][p + ux];
        v.exy = F.E[0][p + uy];
        v.ezy = F.E[2][p + uy];
        v.exz = F.E[0][p + uz];
        v.eyz = F.E[1][p + uz];
#pragma unroll
        for (int c = 0; c < 3; ++c) v.b[c] = F.B[c][p];
    };
    VacPlane<T> v{}, w{};
    T ex = T(0), ey = T(0);  // E_x, E_y at the thread's point
    if (in) {
        ex = F.E[0][col + z * q.st[2]];
        ey = F.E[1][col + z * q.st[2]];
        load(z, v);
    }
    const double dt = g.dt;
    const double ix = g.inv_d[0], iy = g.inv_d[1], iz = g.inv_d[2];
    T bxd = T(0), byd = T(0);  // B'_x, B'_y one plane below
    int buf = 0;
    for (int k = below ? -1 : 0; zs + k < ze; ++k) {
        const int zn = zs + k + 1;  // the next plane
        if (in && zn < ze) load(zn, w);
        q.idx[2] = z;
        q.p = col + z * q.st[2];
        T b[3] = {v.b[0], v.b[1], v.b[2]};
        if (in) {
            if (valid_B(g, q, 0)) {
                const double curl = ((double)v.ezy - (double)v.ez) * iy -
                                    ((double)v.eyz - (double)ey) * iz;
                b[0] = (T)((double)b[0] - dt * curl);
            }
            if (valid_B(g, q, 1)) {
                const double curl = ((double)v.exz - (double)ex) * iz -
                                    ((double)v.ezx - (double)v.ez) * ix;
                b[1] = (T)((double)b[1] - dt * curl);
            }
            if (valid_B(g, q, 2)) {
                const double curl = ((double)v.eyx - (double)ey) * ix -
                                    ((double)v.exy - (double)ex) * iy;
                b[2] = (T)((double)b[2] - dt * curl);
            }
        }
        if (k >= 0) {
#pragma unroll
            for (int c = 0; c < 3; ++c) sB[buf][c][tid] = b[c];
            __syncthreads();  // (the other buffer is read before this barrier only)
            if (own) {
                const long long p = q.p;
                if (F.planes) mur_save(g, q, F.E, F.planes, F.pstride);
                T e[3] = {ex, ey, v.ez};
                if (ampere_E(g, q, 0)) {
                    const double curl = ((double)b[2] - (double)sB[buf][2][tid - VX]) * iy -
                                        ((double)b[1] - (double)byd) * iz;
                    e[0] = (T)((double)e[0] + dt * (curl - 0.0));
                } else if (pec_zero(g, q.idx, 0)) {
                    e[0] = T(0);
                }
                if (ampere_E(g, q, 1)) {
                    const double curl = ((double)b[0] - (double)bxd) * iz -
                                        ((double)b[2] - (double)sB[buf][2][tid - 1]) * ix;
                    e[1] = (T)((double)e[1] + dt * (curl - 0.0));
                } else if (pec_zero(g, q.idx, 1)) {
                    e[1] = T(0);
                }
                if (ampere_E(g, q, 2)) {
                    const double curl = ((double)b[1] - (double)sB[buf][1][tid - 1]) * ix -
                                        ((double)b[0] - (double)sB[buf][0][tid - VX]) * iy;
                    e[2] = (T)((double)e[2] + dt * (curl - 0.0));
                } else if (pec_zero(g, q.idx, 2)) {
                    e[2] = T(0);
                }
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    F.Eo[c][p] = e[c];
                    F.Bo[c][p] = b[c];
                    if (F.J[0]) F.J[c][p] = T(0);
                }
            }
            buf ^= 1;
        }
        bxd = b[0];
        byd = b[1];
        ex = v.exz;
        ey = v.eyz;
        v = w;
        z = zn;
    }
}

// Six arrays of n floats copied in one launch (the fields of a state)
struct Copy6 {
    const float *src[6];
    float *dst[6];
};

__global__ void k_copy6(Copy6 c, long long n) {
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
#pragma unroll
        for (int a = 0; a < 6; ++a) c.dst[a][i] = c.src[a][i];
    }
}

// J = the fixed-point sums converted (before the current filter)
__global__ void k_j_from_fixed(GridP g, float *__restrict__ Jx, float *__restrict__ Jy,
                               float *__restrict__ Jz, const long long *__restrict__ Jfx,
                               const long long *__restrict__ Jfy,
                               const long long *__restrict__ Jfz, double jinv) {
    Pt q;
    if (!make_point(g, q)) return;
    const long long p = q.p;
    Jx[p] = j_from_fixed<float>(Jfx[p], jinv);
    Jy[p] = j_from_fixed<float>(Jfy[p], jinv);
    Jz[p] = j_from_fixed<float>(Jfz[p], jinv);
}

// The Mur faces of one axis from the saved planes of E^n (mur_save); points
// that a PEC face holds at zero stay zero.  One thread per point, component
// (blockIdx.y) and face (blockIdx.z): a few thousand points with one chain of
// loads each, those of an x face a cache line apart, so latency is what it
// costs (box 1024 x 128 x 128: 5.4 us per launch, 15.7 with a
// point's four updates in one thread).
constexpr int MUR_T = 64;
template <typename T>
__global__ __launch_bounds__(MUR_T) void k_mur_apply(GridP g, int a, T *Ex, T *Ey, T *Ez,
                                                     const T *planes, long long pstride) {
    const int b1 = a == 0 ? 1 : 0, b2 = a == 2 ? 1 : 2;
    const long long npt = (long long)g.ext[b1] * g.ext[b2];
    const long long t = blockIdx.x * (long long)MUR_T + threadIdx.x;
    if (t >= npt) return;
    const int i1 = (int)(t % g.ext[b1]), i2 = (int)(t / g.ext[b1]);
    const int ci = blockIdx.y, c = ci == 0 ? b1 : b2;
    T *const E = c == 0 ? Ex : (c == 1 ? Ey : Ez);
    const long long st[3] = {1, g.ext[0], (long long)g.ext[0] * g.ext[1]};
    const T coef = (T)((g.dt - g.d[a]) / (g.dt + g.d[a]));
    int idx[3];
    idx[a] = 0;
    idx[b1] = i1;
    idx[b2] = i2;
    if (pec_zero(g, idx, c)) return;
    const T *pl = planes + ((long long)a * 2 + ci) * 4 * pstride;
    const long long base = st[b1] * i1 + st[b2] * i2;
    if (blockIdx.z == 0) {
        // face at index 0: E_0^{n+1} = E_1^n + coef (E_1^{n+1} - E_0^n)
        E[base] = pl[1 * pstride + t] + coef * (E[base + st[a]] - pl[0 * pstride + t]);
    } else {
        // face at index n: E_n^{n+1} = E_{n-1}^n + coef (E_{n-1}^{n+1} - E_n^n)
        const long long pn = base + st[a] * g.n[a];
        E[pn] = pl[2 * pstride + t] + coef * (E[pn - st[a]] - pl[3 * pstride + t]);
    }
}

// Soft current sheet J_y on x-node plane i_s (READING of the external-source
// module), applied to E after Ampere: E_y -= dt J_sheet(t^{n+1/2}).
template <typename T>
__global__ void k_laser(GridP g, T *Ey, empic_laser_desc L, double t_half) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    const int k = blockIdx.y;
    const int cy = g.n[1];                                              // E_y half along y
    const int cz = g.bc[2] != EMPIC_BC_PERIODIC ? g.n[2] + 1 : g.n[2];  // node along z
    if (j >= cy || k >= cz) return;
    if (g.bc[0] != EMPIC_BC_PERIODIC && (L.i_s == 0 || L.i_s == g.n[0])) return;
    if (g.bc[2] != EMPIC_BC_PERIODIC && (k == 0 || k == g.n[2])) return;
    const double y = ((double)j + 0.5) * g.d[1];
    const double z = (double)k * g.d[2];
    const double ry2 = L.slab ? 0.0 : (y - L.yc) * (y - L.yc);
    const double r2 = ry2 + (z - L.zc) * (z - L.zc);
    const double tt = t_half - L.t0;
    const double einc = L.a0 * exp(-r2 / (L.w0 * L.w0)) *
                        exp(-2.0 * log(2.0) * tt * tt / (L.tau * L.tau)) * sin(L.omega0 * tt);
    const double Jy = -2.0 * einc / g.d[0];
    const long long p = L.i_s + (long long)g.ext[0] * (j + (long long)g.ext[1] * k);
    Ey[p] -= (T)(g.dt * Jy);
}

// Waveguide port (hard source): E_comp = e0 sin(pi s/L) g(t) sin(omega t) on
// the node plane of axis P.axis, s the component's position along
// P.prof_axis, with the amplitude factor computed on the host in FP64.
template <typename T>
__global__ void k_port(GridP g, T *Ec, empic_port_desc P, double amp) {
    const int a = P.axis, c = P.comp, pa = P.prof_axis;
    const int b1 = a == 0 ? 1 : 0, b2 = a == 2 ? 1 : 2;
    // E_c holds ext values along a transverse axis, n where it is
    // half-staggered on a walled axis (entry n is padding)
    const int n1 = (g.bc[b1] == EMPIC_BC_PERIODIC || c != b1) ? g.ext[b1] : g.n[b1];
    const int n2 = (g.bc[b2] == EMPIC_BC_PERIODIC || c != b2) ? g.ext[b2] : g.n[b2];
    const long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (t >= (long long)n1 * n2) return;
    int idx[3];
    idx[a] = P.plane;
    idx[b1] = (int)(t % n1);
    idx[b2] = (int)(t / n1);
    const double s = ((double)idx[pa] + (c == pa ? 0.5 : 0.0)) * g.d[pa];
    const double L = g.n[pa] * g.d[pa];
    const long long p = idx[0] + (long long)g.ext[0] * (idx[1] + (long long)g.ext[1] * idx[2]);
    const double sw = fmin(s, L - s);  // sin(pi s/L) from the nearer wall: exactly 0 on both
    Ec[p] = (T)(amp * sin(3.14159265358979323846 * sw / L));
}

// The current filter: per axis x, y, z, `passes` binomial passes dst = (src[-1]
// + 2 src + src[+1])/4, then the compensator; every pass rounds to T.  Each
// component on its own sub-grid: periodic axes wrap, on a walled axis values
// beyond the stored ones (entry n of a half-cell component is padding) count
// as zero in every pass.
template <typename T>
__device__ __forceinline__ T filter_point(T lo, T mid, T hi, bool comp) {
    const T a = comp ? T(-0.25) : T(0.25), b = comp ? T(1.5) : T(0.5);
    return a * lo + b * mid + a * hi;
}

// One pass along axis AX (where filter_by_patches says no)
template <typename T, int AX>
__global__ __launch_bounds__(PT_THREADS) void k_filter_pass(
    GridP g, const T *__restrict__ s0, const T *__restrict__ s1, const T *__restrict__ s2,
    T *__restrict__ d0, T *__restrict__ d1, T *__restrict__ d2, bool comp) {
    Pt q;
    if (!make_point(g, q)) return;
    const T *src[3] = {s0, s1, s2};
    T *dst[3] = {d0, d1, d2};
    const long long p = q.p;
    const bool per = g.bc[AX] == EMPIC_BC_PERIODIC;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        // stored values of component c along every axis
        if (g.bc[c] != EMPIC_BC_PERIODIC && q.idx[c] == g.n[c]) {
            dst[c][p] = T(0);
            continue;
        }
        const int L = (!per && AX == c) ? g.n[AX] : g.ext[AX];
        const int i = q.idx[AX];
        T lo = T(0), hi = T(0);
        if (i > 0) lo = src[c][p - q.st[AX]];
        else if (per) lo = src[c][p + (long long)(L - 1) * q.st[AX]];
        if (i < L - 1) hi = src[c][p + q.st[AX]];
        else if (per) hi = src[c][p - (long long)(L - 1) * q.st[AX]];
        dst[c][p] = filter_point(lo, src[c][p], hi, comp);
    }
}

// The whole filter of M passes per axis in one launch: a workgroup takes one
// component of a 32 x 8 x 4 patch with M points around it through LDS, the
// passes ping-ponging between two buffers.  Bound by LDS and latency, not by
// HBM (the patch's halo comes from L2).  FIXED: the source is the int64
// current sums (J = sum x jinv rounded once, as k_j_from_fixed).  One binomial
// pass and the compensator on 75 x 49 x 53 took the conversion and six passes
// of 27.6 us, whose arrays a run-time axis index kept in scratch: 171 us.  In
// one launch with each pass over the shrinking window, its coordinates worked
// out by divisions: 25.4 us; with fixed points per thread as below: 15.9 us.
constexpr int FTX = 32, FTY = 8, FTZ = 4;
template <typename T>
struct FilterPtr {
    const T *src[3];
    const long long *fix[3];
    T *dst[3];
};
template <typename T, int M, bool FIXED>
__global__ __launch_bounds__(256) void k_filter_tile(GridP g, FilterPtr<T> P, int passes,
                                                     double jinv) {
    constexpr int WX = FTX + 2 * M, WY = FTY + 2 * M, WZ = FTZ + 2 * M, V = WX * WY * WZ;
    __shared__ T buf[2][V];
    __shared__ int sX[WX], sY[WY], sZ[WZ];  // offsets of the window's rows, -1: counts as zero
    const int c = blockIdx.y, tid = threadIdx.x;
    const int ntx = (g.ext[0] + FTX - 1) / FTX, nty = (g.ext[1] + FTY - 1) / FTY;
    const int bx = blockIdx.x % ntx, byz = blockIdx.x / ntx;
    const int org[3] = {bx * FTX, (byz % nty) * FTY, (byz / nty) * FTZ};
    if (tid < WX + WY + WZ) {
        const int a = tid < WX ? 0 : (tid < WX + WY ? 1 : 2);
        const int l = tid - (a == 0 ? 0 : (a == 1 ? WX : WX + WY));
        const int n = a == 0 ? g.n[0] : (a == 1 ? g.n[1] : g.n[2]);
        const int ext = a == 0 ? g.ext[0] : (a == 1 ? g.ext[1] : g.ext[2]);
        const int bc = a == 0 ? g.bc[0] : (a == 1 ? g.bc[1] : g.bc[2]);
        const int o = a == 0 ? org[0] : (a == 1 ? org[1] : org[2]);
        int i = o - M + l;
        if (bc == EMPIC_BC_PERIODIC) {
            i %= n;
            i = i < 0 ? i + n : i;
        } else if (i < 0 || i >= (a == c ? n : ext)) {
            i = -1;
        }
        if (a == 0) sX[l] = i;
        else if (a == 1) sY[l] = i < 0 ? -1 : i * g.ext[0];
        else sZ[l] = i < 0 ? -1 : i * (g.ext[0] * g.ext[1]);
    }
    __syncthreads();
    const T *src = c == 0 ? P.src[0] : (c == 1 ? P.src[1] : P.src[2]);
    const long long *fix = c == 0 ? P.fix[0] : (c == 1 ? P.fix[1] : P.fix[2]);
    T *dst = c == 0 ? P.dst[0] : (c == 1 ? P.dst[1] : P.dst[2]);
    // A thread keeps the same points e = tid + 256 i through every pass, and a
    // pass covers the whole window: no index arithmetic but e +- stride (the
    // outermost points go stale by one a pass and are not used), with the
    // points that count as zero in a bit mask
    constexpr int NE = (V + 255) / 256;
    static_assert(NE <= 32, "one mask bit per point of a thread");
    uint32_t zero = 0u;
#pragma unroll
    for (int i = 0; i < NE; ++i) {
        const int e = tid + 256 * i;
        if (e >= V) break;
        const int lx = e % WX, r = e / WX, ly = r % WY, lz = r / WY;
        const int ox = sX[lx], oy = sY[ly], oz = sZ[lz];
        T v = T(0);
        if ((ox | oy | oz) >= 0) {
            if constexpr (FIXED) v = j_from_fixed<T>(fix[ox + oy + oz], jinv);
            else v = src[ox + oy + oz];
        } else {
            zero |= 1u << i;
        }
        buf[0][e] = v;
    }
    T *A = buf[0], *B = buf[1];
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        constexpr int ST[3] = {1, WX, WX * WY};
        const int st = ST[ax];
#pragma unroll 1
        for (int k = 0; k < M; ++k) {
            __syncthreads();
#pragma unroll
            for (int i = 0; i < NE; ++i) {
                const int e = tid + 256 * i;
                if (e >= V) break;
                const T lo = A[max(e - st, 0)], hi = A[min(e + st, V - 1)];
                const T v = filter_point(lo, A[e], hi, k == passes);
                B[e] = (zero >> i) & 1u ? T(0) : v;
            }
            T *t = A;
            A = B;
            B = t;
        }
    }
    __syncthreads();
    for (int i = tid; i < FTX * FTY * FTZ; i += 256) {
        const int lx = i % FTX, ly = (i / FTX) % FTY, lz = i / (FTX * FTY);
        const int x = org[0] + lx, y = org[1] + ly, z = org[2] + lz;
        if (x < g.ext[0] && y < g.ext[1] && z < g.ext[2])
            dst[x + (long long)g.ext[0] * (y + (long long)g.ext[1] * z)] =
                A[lx + M + WX * (ly + M + WY * (lz + M))];
    }
}

// Moving window: every value moves `cells` planes toward index 0 along axis
// ax; values that would come from beyond the stored ones are zero (the new
// front planes); padding entries stay zero.  isB selects the B staggering.
template <typename T>
__global__ void k_window_shift(GridP g, int ax, int cells, int isB, const T *__restrict__ s0,
                               const T *__restrict__ s1, const T *__restrict__ s2,
                               T *__restrict__ d0, T *__restrict__ d1, T *__restrict__ d2) {
    Pt q;
    if (!make_point(g, q)) return;
    const T *src[3] = {s0, s1, s2};
    T *dst[3] = {d0, d1, d2};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        bool pad = false;
        for (int b = 0; b < 3; ++b) {
            const bool half = isB ? (b != c) : (b == c);
            if (g.bc[b] != EMPIC_BC_PERIODIC && half && q.idx[b] == g.n[b]) pad = true;
        }
        const bool half_ax = isB ? (ax != c) : (ax == c);
        const int L = (g.bc[ax] != EMPIC_BC_PERIODIC && half_ax) ? g.n[ax] : g.ext[ax];
        const int m = q.idx[ax];
        dst[c][q.p] = (!pad && m + cells < L) ? src[c][q.p + (long long)cells * q.st[ax]] : T(0);
    }
}

// FP64 partial sums of |E|^2 and B^{n-1/2}.B^{n+1/2} (B^{n+1/2} formed on the fly)
template <typename T>
__global__ void k_field_energy(GridP g, const T *__restrict__ Ex, const T *__restrict__ Ey,
                               const T *__restrict__ Ez, const T *__restrict__ Bx,
                               const T *__restrict__ By, const T *__restrict__ Bz,
                               double *partials) {
    __shared__ double sm[16];
    double ee = 0.0, bb = 0.0;
    const int bid = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
    const T dt = (T)g.dt;
    const T ix = (T)g.inv_d[0], iy = (T)g.inv_d[1], iz = (T)g.inv_d[2];
    for (int k = blockIdx.z; k < g.ext[2]; k += gridDim.z)
        for (int j = blockIdx.y * blockDim.y + threadIdx.y; j < g.ext[1]; j += gridDim.y * blockDim.y)
            for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < g.ext[0];
                 i += gridDim.x * blockDim.x) {
                Pt q;
                q.idx[0] = i;
                q.idx[1] = j;
                q.idx[2] = k;
                q.st[0] = 1;
                q.st[1] = g.ext[0];
                q.st[2] = (long long)g.ext[0] * g.ext[1];
                const long long p = i + q.st[1] * j + q.st[2] * k;
                ee += (double)Ex[p] * Ex[p] + (double)Ey[p] * Ey[p] + (double)Ez[p] * Ez[p];
                if (valid_B(g, q, 0)) {
                    const T c = (Ez[p + up(g, q, 1)] - Ez[p]) * iy - (Ey[p + up(g, q, 2)] - Ey[p]) * iz;
                    bb += (double)Bx[p] * (double)(Bx[p] - dt * c);
                }
                if (valid_B(g, q, 1)) {
                    const T c = (Ex[p + up(g, q, 2)] - Ex[p]) * iz - (Ez[p + up(g, q, 0)] - Ez[p]) * ix;
                    bb += (double)By[p] * (double)(By[p] - dt * c);
                }
                if (valid_B(g, q, 2)) {
                    const T c = (Ey[p + up(g, q, 0)] - Ey[p]) * ix - (Ex[p + up(g, q, 1)] - Ex[p]) * iy;
                    bb += (double)Bz[p] * (double)(Bz[p] - dt * c);
                }
            }
    const double se = block_reduce<false>(ee, sm);
    const double sb = block_reduce<false>(bb, sm);
    if (threadIdx.x == 0 && threadIdx.y == 0) {
        partials[Q_EE * PSTRIDE + bid] = se;
        partials[Q_BB * PSTRIDE + bid] = sb;
    }
}

// workgroups of the point kernels: a multiple of 8 for the XCD-contiguous map
dim3 point_grid(const GridP &g) {
    const long long nb = (g.V + PT_THREADS - 1) / PT_THREADS;
    return dim3((unsigned)((nb + 7) / 8 * 8));
}

}  // namespace

// Grid of the (64, 4) point reductions: every kernel strides over all three
// axes, and gx * gy * gz <= PSTRIDE keeps one partial slot per workgroup.
dim3 reduction_grid(const GridP &g) {
    int gx = (g.ext[0] + 63) / 64;
    if (gx > 64) gx = 64;
    int gy = (g.ext[1] + 3) / 4;
    if (gy > PSTRIDE / gx) gy = PSTRIDE / gx;
    int gz = PSTRIDE / (gx * gy);
    if (gz > g.ext[2]) gz = g.ext[2];
    if (gz < 1) gz = 1;
    return dim3(gx, gy, gz);
}

template <typename T>
void launch_faraday(const GridP &g, T *const E[3], T *const B[3], T *const Bbar[3],
                    T *const J[3], unsigned long long *const Jf[3], bool write_B, hipStream_t s,
                    unsigned *fb_reset, T *mur_planes, long long plane_stride) {
    hipLaunchKernelGGL(k_faraday<T>, point_grid(g), dim3(PT_THREADS), 0, s, g, E[0], E[1], E[2],
                       B[0], B[1], B[2], Bbar ? Bbar[0] : nullptr, Bbar ? Bbar[1] : nullptr,
                       Bbar ? Bbar[2] : nullptr, J ? J[0] : nullptr, J ? J[1] : nullptr,
                       J ? J[2] : nullptr, Jf ? Jf[0] : nullptr, Jf ? Jf[1] : nullptr,
                       Jf ? Jf[2] : nullptr, fb_reset, write_B ? 1 : 0, mur_planes, plane_stride);
}

template <typename T>
void launch_ampere(const GridP &g, T *const E[3], T *const B[3], T *const J[3], JMode mode,
                   bool write_J, const long long *const Jf[3], double jinv, hipStream_t s) {
    const auto fixed = write_J ? k_ampere<T, J_FIXED, true> : k_ampere<T, J_FIXED, false>;
    const auto none = write_J ? k_ampere<T, J_NONE, true> : k_ampere<T, J_NONE, false>;
    const auto k = mode == J_FIXED ? fixed : (mode == J_NONE ? none : k_ampere<T, J_READ, false>);
    hipLaunchKernelGGL(k, point_grid(g), dim3(PT_THREADS), 0, s, g, E[0], E[1], E[2], B[0], B[1],
                       B[2], J[0], J[1], J[2], Jf ? Jf[0] : nullptr, Jf ? Jf[1] : nullptr,
                       Jf ? Jf[2] : nullptr, jinv);
}

// Patches and chunks of planes of k_vacuum, and the fraction of their points that
// lies on the grid
struct VacGrid {
    int nbx, nby, nbz, zc;
    double used;
};
static VacGrid vacuum_grid(const GridP &g) {
    VacGrid v;
    v.nbx = (g.ext[0] + VX - 2) / (VX - 1);
    v.nby = (g.ext[1] + VY - 2) / (VY - 1);
    // 16 planes per workgroup where that leaves two workgroups per CU, else 8: 61 x
    // 31 x 2001 (756 of 16) 47 us per step with 16 and 54 with 8, 46 x 23 x 1501
    // (376 of 16) 41 and 31, 91 x 46 x 3001 (2256) 202 and 197; with 4 and with
    // 32 slower than the better of these everywhere.
    v.zc = (long long)v.nbx * v.nby * ((g.ext[2] + 15) / 16) >= 512 ? 16 : 8;
    v.nbz = (g.ext[2] + v.zc - 1) / v.zc;
    v.used = (double)g.V / ((double)v.nbx * (VX - 1) * v.nby * (VY - 1) * v.nbz * v.zc);
    return v;
}

// What decides is the memory-side cache (256 MiB): the point kernels work in place
// on E and B, k_vacuum on two sets of them.  One pass pays where both sets stay in
// the cache and the grid is large enough for the march along z, and where not
// even one does; between, it leaves the cache and they do not.  It also has to fill
// its patches, the less so the further E and B exceed the cache.  Point kernels |
// one pass, us per step, FP32: 1.0 M points 17 | 21, 2.1 M 30 | 27, 4.1 M 50 | 46, 5.2 M
// 62 | 74, 8.0 M 91 | 110, 10.5 M 121 | 132, 11.5 M 182 | 164, 12.5 M 209 | 164, 17 M
// 276 | 200; with 70 % of the patches used 4.1 M 50 | 58, 12.5 M 201 | 205, 17 M 266 | 252;
// with 57 % 12.5 M 209 | 199, 17 M 273 | 246; 6 x 512 x 1024 (19 %) 41 | 111.  FP64: 2.1 M
// 44 | 44, 4.0 M 78 | 118, 6.0 M 186 | 152, 12.5 M 368 | 303; with 70 % 6.0 M 184 | 188, 12.5 M
// 348 | 326; with 57 % 8.0 M 232 | 240, 17 M 518 | 492.
template <typename T>
bool vacuum_fits(const GridP &g) {
    if (g.ext[2] < 16) return false;
    constexpr double CACHE = 256.0 * (1 << 20);
    const double one = 6.0 * sizeof(T) * (double)g.V;  // bytes of E and B
    const bool both_fit = sizeof(T) == 4 && g.V >= (1ll << 21) && 2.0 * one <= 0.75 * CACHE;
    if (!both_fit && one <= CACHE) return false;
    return vacuum_grid(g).used >= (one > 1.5 * CACHE ? 0.55 : 0.72);
}

// A step without particles of E, B into Eo, Bo (J zeroed when given).
template <typename T>
void launch_vacuum(const GridP &g, T *const E[3], T *const B[3], T *const Eo[3], T *const Bo[3],
                   T *const J[3], T *mur_planes, long long plane_stride, hipStream_t s) {
    VacIO<T> F;
    for (int c = 0; c < 3; ++c) {
        F.E[c] = E[c];
        F.B[c] = B[c];
        F.Eo[c] = Eo[c];
        F.Bo[c] = Bo[c];
        F.J[c] = J ? J[c] : nullptr;
    }
    F.planes = mur_planes;
    F.pstride = plane_stride;
    const VacGrid v = vacuum_grid(g);
    const long long nb = (long long)v.nbx * v.nby * v.nbz;
    hipLaunchKernelGGL(k_vacuum<T>, dim3((unsigned)((nb + 7) / 8 * 8)), dim3(VT), 0, s, g, F,
                       v.nbx, v.nby, v.nbz, v.zc);
}

void launch_copy6(const float *const src[6], float *const dst[6], long long n, hipStream_t s) {
    Copy6 c;
    for (int a = 0; a < 6; ++a) {
        c.src[a] = src[a];
        c.dst[a] = dst[a];
    }
    long long nb = (n + 255) / 256;
    if (nb > 4096) nb = 4096;
    if (nb < 1) nb = 1;
    hipLaunchKernelGGL(k_copy6, dim3((unsigned)nb), dim3(256), 0, s, c, n);
}

void launch_j_from_fixed(const GridP &g, float *const J[3], const long long *const Jf[3],
                         double jinv, hipStream_t s) {
    hipLaunchKernelGGL(k_j_from_fixed, point_grid(g), dim3(PT_THREADS), 0, s, g, J[0], J[1], J[2],
                       Jf[0], Jf[1], Jf[2], jinv);
}

template <typename T>
void launch_mur_apply(const GridP &g, T *const E[3], const T *planes, long long pstride,
                      hipStream_t s) {
    for (int a = 0; a < 3; ++a) {
        if (g.bc[a] != EMPIC_BC_ABSORBING) continue;
        const int b1 = a == 0 ? 1 : 0, b2 = a == 2 ? 1 : 2;
        const long long npt = (long long)g.ext[b1] * g.ext[b2];
        hipLaunchKernelGGL(k_mur_apply<T>, dim3((unsigned)((npt + MUR_T - 1) / MUR_T), 2, 2),
                           dim3(MUR_T), 0, s, g, a, E[0], E[1], E[2], planes, pstride);
    }
}

namespace {
// Filters of up to FTILE_M passes per axis can go through the patch kernel: both its
// buffers fit the 64 KB of static LDS (M = 4 in FP32: 60 KB; M = 2 in FP64: 54 KB).
// It does M passes on every window point, so it pays where all workgroups are
// resident at once, and else where the windows, with their halos and what hangs
// over the grid's edge, hold few times the grid's points.  Pass by pass | patches, us
// per step, FP32: 1 pass, 128^3 (2.0 times) 119 | 107, 512 x 4 x 256 (4.0) 56 | 54, 512 x 2 x
// 512 (8.0) 50 | 58; 2 passes, 128^3 (3.4) 151 | 142, 40 x 128 x 128 (5.4) 79 | 78, 512 x 4 x
// 256 (6.8) 68 | 74, 2 x 512 x 512 (54) 73 | 254; 3, 64^3 (5.2, resident) 62 | 53, 128^3 185 |
// 228; 4, 48^3 (7.5, resident) 77 | 71, 64^3 (not) 72 | 83, 128^3 218 | 412.  FP64: 1
// pass, 512 x 6 x 256 (2.7) 89 | 89, 40 x 128 x 128 (3.2) 85 | 86, 512 x 4 x 256 (4.0) 76 | 82; 2, 32^3
// (3.4, resident) 54 | 53, 128^3 191 | 244.
template <typename T>
bool filter_by_patches(const GridP &g, int M) {
    constexpr int FTILE_M = sizeof(T) == 4 ? 4 : 2;
    constexpr long long LDS = 160 * 1024, CUS = 256;
    if (M > FTILE_M) return false;
    const long long nt = (long long)((g.ext[0] + FTX - 1) / FTX) * ((g.ext[1] + FTY - 1) / FTY) *
                         ((g.ext[2] + FTZ - 1) / FTZ);
    const long long window = (FTX + 2 * M) * (FTY + 2 * M) * (long long)(FTZ + 2 * M);
    if (3 * nt <= CUS * (LDS / (2 * window * (long long)sizeof(T)))) return true;
    return (double)(nt * window) <= (sizeof(T) == 4 ? 5.0 : 2.7) * (double)g.V;
}

template <typename T, int M>
void filter_tile(const GridP &g, const FilterPtr<T> &P, int passes, double jinv, hipStream_t s) {
    const int nt = ((g.ext[0] + FTX - 1) / FTX) * ((g.ext[1] + FTY - 1) / FTY) *
                   ((g.ext[2] + FTZ - 1) / FTZ);
    if (P.fix[0])
        hipLaunchKernelGGL((k_filter_tile<T, M, true>), dim3(nt, 3), dim3(256), 0, s, g, P, passes,
                           jinv);
    else
        hipLaunchKernelGGL((k_filter_tile<T, M, false>), dim3(nt, 3), dim3(256), 0, s, g, P, passes,
                           jinv);
}
}  // namespace

// The whole filter by patches (filter_by_patches), or pass by pass
template <typename T>
void launch_filter(const GridP &g, T *const S[3], const long long *const Jf[3], double jinv,
                   T *const F[3], T *const tmp[3], int passes, int compensate, hipStream_t s) {
    const int M = passes + (compensate ? 1 : 0);
    if (filter_by_patches<T>(g, M)) {
        FilterPtr<T> P{};
        const bool inplace = !Jf && S[0] == F[0];
        for (int c = 0; c < 3; ++c) {
            P.src[c] = S[c];
            P.fix[c] = Jf ? Jf[c] : nullptr;
            P.dst[c] = inplace ? tmp[c] : F[c];
        }
        if (M == 1) filter_tile<T, 1>(g, P, passes, jinv, s);
        if (M == 2) filter_tile<T, 2>(g, P, passes, jinv, s);
        if constexpr (sizeof(T) == 4) {
            if (M == 3) filter_tile<T, 3>(g, P, passes, jinv, s);
            if (M == 4) filter_tile<T, 4>(g, P, passes, jinv, s);
        }
        if (inplace)
            for (int c = 0; c < 3; ++c)
                (void)hipMemcpyAsync(F[c], tmp[c], (size_t)g.V * sizeof(T),
                                     hipMemcpyDeviceToDevice, s);
        return;
    }
    // pass by pass, alternating so that the last one writes F; an odd number of
    // passes in place starts from a copy
    const int N = 3 * M;
    T *cur[3], *oth[3];
    for (int c = 0; c < 3; ++c) {
        cur[c] = N % 2 ? tmp[c] : F[c];
        oth[c] = N % 2 ? F[c] : tmp[c];
    }
    if (Jf) {
        if constexpr (sizeof(T) == 4) launch_j_from_fixed(g, cur, Jf, jinv, s);
    } else if (cur[0] != S[0]) {
        for (int c = 0; c < 3; ++c)
            (void)hipMemcpyAsync(cur[c], S[c], (size_t)g.V * sizeof(T), hipMemcpyDeviceToDevice, s);
    }
    for (int ax = 0; ax < 3; ++ax)
        for (int k = 0; k < M; ++k) {
            const auto kern = ax == 0 ? k_filter_pass<T, 0>
                                      : (ax == 1 ? k_filter_pass<T, 1> : k_filter_pass<T, 2>);
            hipLaunchKernelGGL(kern, point_grid(g), dim3(PT_THREADS), 0, s, g, cur[0], cur[1],
                               cur[2], oth[0], oth[1], oth[2], k == passes);
            for (int c = 0; c < 3; ++c) std::swap(cur[c], oth[c]);
        }
}

template <typename T>
void launch_window_shift(const GridP &g, T *const F[3], T *const tmp[3], int ax, int cells,
                         bool isB, hipStream_t s) {
    hipLaunchKernelGGL(k_window_shift<T>, point_grid(g), dim3(PT_THREADS), 0, s, g, ax, cells,
                       isB ? 1 : 0, F[0], F[1], F[2], tmp[0], tmp[1], tmp[2]);
    for (int c = 0; c < 3; ++c)
        (void)hipMemcpyAsync(F[c], tmp[c], (size_t)g.V * sizeof(T), hipMemcpyDeviceToDevice, s);
}

template <typename T>
void launch_port(const GridP &g, T *const E[3], const empic_port_desc &P, double t,
                 hipStream_t s) {
    const double amp = P.e0 * (1.0 - std::exp(-t / P.tau)) * std::sin(P.omega * t);
    const int a = P.axis;
    const int b1 = a == 0 ? 1 : 0, b2 = a == 2 ? 1 : 2;
    const long long npt = (long long)g.ext[b1] * g.ext[b2];
    hipLaunchKernelGGL(k_port<T>, dim3((unsigned)((npt + 255) / 256)), dim3(256), 0, s, g,
                       E[P.comp], P, amp);
}

template <typename T>
void launch_laser(const GridP &g, T *const E[3], const empic_laser_desc &L, double t_half,
                  hipStream_t s) {
    const int cz = g.bc[2] != EMPIC_BC_PERIODIC ? g.n[2] + 1 : g.n[2];
    empic_laser_desc P = L;
    if (g.bc[0] == EMPIC_BC_PERIODIC && P.i_s == g.n[0]) P.i_s = 0;  // the same node plane
    hipLaunchKernelGGL(k_laser<T>, dim3((g.n[1] + 63) / 64, cz), dim3(64), 0, s, g, E[1], P,
                       t_half);
}

template <typename T>
void launch_field_energy(const GridP &g, T *const E[3], T *const B[3], double *partials,
                         hipStream_t s) {
    hipLaunchKernelGGL(k_field_energy<T>, reduction_grid(g), dim3(64, 4), 0, s, g, E[0], E[1],
                       E[2], B[0], B[1], B[2], partials);
}

#define EMPIC_INST(T)                                                                          \
    template void launch_faraday<T>(const GridP &, T *const[3], T *const[3], T *const[3],      \
                                    T *const[3], unsigned long long *const[3], bool,           \
                                    hipStream_t, unsigned *, T *, long long);                  \
    template void launch_ampere<T>(const GridP &, T *const[3], T *const[3], T *const[3],       \
                                   JMode, bool, const long long *const[3], double,             \
                                   hipStream_t);                                               \
    template bool vacuum_fits<T>(const GridP &);                                               \
    template void launch_vacuum<T>(const GridP &, T *const[3], T *const[3], T *const[3],       \
                                   T *const[3], T *const[3], T *, long long, hipStream_t);     \
    template void launch_mur_apply<T>(const GridP &, T *const[3], const T *, long long,        \
                                      hipStream_t);                                            \
    template void launch_laser<T>(const GridP &, T *const[3], const empic_laser_desc &, double, \
                                  hipStream_t);                                                \
    template void launch_window_shift<T>(const GridP &, T *const[3], T *const[3], int, int,    \
                                         bool, hipStream_t);                                   \
    template void launch_filter<T>(const GridP &, T *const[3], const long long *const[3],      \
                                   double, T *const[3], T *const[3], int, int, hipStream_t);   \
    template void launch_port<T>(const GridP &, T *const[3], const empic_port_desc &, double,  \
                                 hipStream_t);                                                 \
    template void launch_field_energy<T>(const GridP &, T *const[3], T *const[3], double *,    \
                                         hipStream_t);
EMPIC_INST(float)
EMPIC_INST(double)
#undef EMPIC_INST

}  // namespace empic

// Setup of the demagnetizing tensor of Eq. (2) in double precision: Newell's
// closed forms (ref. [24]) near the origin, Gauss quadrature far away, and
// the fold of its FFT into the real k-space kernel of the z pass.
#include <hip/hip_runtime.h>

#include <cmath>

#include "kernels.hpp"

namespace llgx {

constexpr int NT = 256;

// ------------------------------------------------------------------------
// Newell tensor (ref. [24]) in double precision.
// f and g are evaluated on |x|,|y|,|z|; g carries sign(x) sign(y).
__device__ double newell_f(double x, double y, double z) {
    x = fabs(x);
    y = fabs(y);
    z = fabs(z);
    const double x2 = x * x, y2 = y * y, z2 = z * z;
    const double R = sqrt(x2 + y2 + z2);
    double t = (2.0 * x2 - y2 - z2) * R / 6.0;
    const double rxz = sqrt(x2 + z2), rxy = sqrt(x2 + y2);
    if (y > 0.0 && rxz > 0.0) t += 0.5 * y * (z2 - x2) * asinh(y / rxz);
    if (z > 0.0 && rxy > 0.0) t += 0.5 * z * (y2 - x2) * asinh(z / rxy);
    if (x > 0.0 && y > 0.0 && z > 0.0) t -= x * y * z * atan(y * z / (x * R));
    return t;
}

__device__ double newell_g(double x, double y, double z) {
    if (x == 0.0 || y == 0.0) return 0.0;
    const double sgn = ((x < 0.0) != (y < 0.0)) ? -1.0 : 1.0;
    x = fabs(x);
    y = fabs(y);
    z = fabs(z);
    const double x2 = x * x, y2 = y * y, z2 = z * z;
    const double R = sqrt(x2 + y2 + z2);
    double t = -x * y * R / 3.0;
    if (z > 0.0) {
        t += x * y * z * asinh(z / sqrt(x2 + y2));
        t -= z2 * z / 6.0 * atan(x * y / (z * R));
        t -= 0.5 * z * y2 * atan(x * z / (y * R));
        t -= 0.5 * z * x2 * atan(y * z / (x * R));
    }
    t += y / 6.0 * (3.0 * z2 - y2) * asinh(x / sqrt(y2 + z2));
    t += x / 6.0 * (3.0 * z2 - x2) * asinh(y / sqrt(x2 + z2));
    return sgn * t;
}

// Near offsets (R < Rs, see below): 27-point second difference (weights 2, -1,
// -1 per axis) of the six component functions, /(4 pi dx dy dz).  32 lanes
// take one offset: lane l < 27 evaluates the six functions at stencil point
// l, then lane i < 6 adds the 27 values of component i in the order of the
// points, so the sum rounds as a serial loop's does.  The work is a few
// hundred offsets (those of the box nbx x nby x nbz around the origin) of 162
// evaluations with an arctangent or two inverse hyperbolic sines each, a long
// serial chain for one thread: with one thread per offset and the far field
// in the same kernel the setup of a 32x32x2 mesh spent 1.45 ms here.
constexpr int NEAR_GROUPS = NT / 32;
__global__ __launch_bounds__(NT) void k_newell_near(int nx, int ny, int nz, int nbx, int nby, int nbz, double ux,
                                                    double uy, double uz, double Rs, double* __restrict__ oct) {
    __shared__ double val[NEAR_GROUPS][27][6];
    const long n = (long)nx * ny * nz;
    const int grp = threadIdx.x >> 5, l = threadIdx.x & 31;
    const int id = (int)blockIdx.x * NEAR_GROUPS + grp;
    const bool in = id < nbx * nby * nbz;
    const int ix = id % nbx, iy = (id / nbx) % nby, iz = id / (nbx * nby);
    const double X = ix * ux, Y = iy * uy, Z = iz * uz;
    const bool on = in && sqrt(X * X + Y * Y + Z * Z) < Rs;
    if (on && l < 27) {
        const double x = X + (l / 9 - 1) * ux, y = Y + (l / 3 % 3 - 1) * uy, z = Z + (l % 3 - 1) * uz;
        val[grp][l][0] = newell_f(x, y, z);
        val[grp][l][1] = newell_f(y, x, z);
        val[grp][l][2] = newell_f(z, y, x);
        val[grp][l][3] = newell_g(x, y, z);
        val[grp][l][4] = newell_g(x, z, y);
        val[grp][l][5] = newell_g(y, z, x);
    }
    __syncthreads();
    if (on && l < 6) {
        double acc = 0.0;
        for (int q = 0; q < 27; ++q) {
            const double w = (q / 9 == 1 ? 2.0 : -1.0) * (q / 3 % 3 == 1 ? 2.0 : -1.0) * (q % 3 == 1 ? 2.0 : -1.0);
            acc += w * val[grp][q][l];
        }
        double N = acc * (1.0 / (4.0 * M_PI * ux * uy * uz));
        // components odd along an axis vanish at zero offset along it
        if ((ix == 0 && (l == 3 || l == 4)) || (iy == 0 && (l == 3 || l == 5)) || (iz == 0 && (l == 4 || l == 5)))
            N = 0.0;
        oct[l * n + ((long)iz * ny + iy) * nx + ix] = N;
    }
}

// Far field (R >= Rs): the cell-pair average of the dipole kernel,
//   N_ij(R) = V/(4 pi) E_u[(r^2 delta_ij - 3 r_i r_j) / r^5], r = R + u,
// with u the difference of two points drawn uniformly from a cell (per axis
// the triangular distribution on [-d, d]), by the Gauss rule of that weight
// per axis: n nodes integrate every moment of u through order 2n - 1 per
// axis.  Nodes and weights: eigenvalues and first eigenvector components of
// the Jacobi matrix of the moments 2/((k+1)(k+2)) (Golub and Welsch, Math.
// Comp. 23 (1969) 221), computed with 60 digits.
// The rule's error falls like (R + sqrt(R^2 - 1))^-2n (R in units of the
// longest side).  Each rule is used from the R where its error reached
// rounding (below 5e-15 of V/(4 pi R^3), against a 60-node rule, cells 1:1:1
// to 1:1:0.05), the 8-node rule below R = 12 (2e-15 there at R = 6; at most
// the truncation error of a moment expansion through order 14 everywhere).
// Rs = min(6 max(dx,dy,dz), 7 (dx dy dz)^(1/3)): the float64 cancellation of
// the exact form grows with R in units of the cube root of the cell volume,
// the quadrature's error falls with R in units of the longest side.
//
// 4 lanes take one offset and split the x nodes.  Bound by FP64 arithmetic
// (about 40 operations a node, 64 nodes for most offsets of a large mesh).
// The moment expansion it replaces kept its three coefficient layers (459
// doubles) in scratch memory: 256x256x16 14.7 ms, 160x80x8 2.48 ms.
constexpr double FAR_SWITCH_SIDE = 6.0;
constexpr double FAR_SWITCH_VOL = 7.0;
constexpr int FAR_RULES = 5, FAR_MAXN = 8;
struct FarRule {
    int n;
    double from;  // used from this R on
    double u[FAR_MAXN], w[FAR_MAXN];
};
__constant__ const FarRule far_rules[FAR_RULES] = {
    {3, 300.0,
     {-0.6324555320336758664, 0.0, 0.6324555320336758664},
     {0.20833333333333333333, 0.58333333333333333333, 0.20833333333333333333}},
    {4, 60.0,
     {-0.75092514330444738455, -0.26222984265274796383, 0.26222984265274796383, 0.75092514330444738455},
     {0.098866304579875626786, 0.40113369542012437321, 0.40113369542012437321, 0.098866304579875626786}},
    {5, 24.0,
     {-0.82144059973838152787, -0.44992035245984196335, 0.0, 0.44992035245984196335, 0.82144059973838152787},
     {0.051658257765490621791, 0.23947324070545739044, 0.41773700305810397554, 0.23947324070545739044,
      0.051658257765490621791}},
    {6, 12.0,
     {-0.86573829497881909617, -0.5766148082484873353, -0.19426367677503889161, 0.19426367677503889161,
      0.5766148082484873353, 0.86573829497881909617},
     {0.029496561655309346531, 0.14748123370527284826, 0.32302220463941780521, 0.32302220463941780521,
      0.14748123370527284826, 0.029496561655309346531}},
    {8, 0.0,
     {-0.91649860178182341063, -0.7301261104488862007, -0.46470084488963896783, -0.15462908084026113352,
      0.15462908084026113352, 0.46470084488963896783, 0.7301261104488862007, 0.91649860178182341063},
     {0.011529448606035851691, 0.062272586069543357121, 0.15758423371338039155, 0.26861373161104039964,
      0.26861373161104039964, 0.15758423371338039155, 0.062272586069543357121, 0.011529448606035851691}}};

__global__ __launch_bounds__(NT) void k_newell_far(int nx, int ny, int nz, double ux, double uy, double uz, double Rs,
                                                   double* __restrict__ oct) {
    const long n = (long)nx * ny * nz;
    const long at = ((long)blockIdx.x * NT + threadIdx.x) >> 2;
    const int part = threadIdx.x & 3;
    const long idx = at < n ? at : n - 1;
    const int ix = (int)(idx % nx);
    const int iy = (int)((idx / nx) % ny);
    const int iz = (int)(idx / ((long)nx * ny));
    const double X = ix * ux, Y = iy * uy, Z = iz * uz;
    const double R = sqrt(X * X + Y * Y + Z * Z);
    const bool on = R >= Rs;
    if (!__any(on)) return;  // a whole wave of near offsets
    // one rule for the wave: the one its nearest far offset needs
    int rule = 0;
    for (int q = 0; q + 1 < FAR_RULES; ++q)
        if (__any(on && R < far_rules[q].from)) rule = q + 1;
    const FarRule& fr = far_rules[rule];
    double acc[6] = {0, 0, 0, 0, 0, 0};
    for (int a = part; a < fr.n; a += 4) {
        const double x = X + fr.u[a] * ux, wa = on ? fr.w[a] : 0.0, x2 = x * x;
        for (int b = 0; b < fr.n; ++b) {
            const double y = Y + fr.u[b] * uy, wb = wa * fr.w[b], s2 = x2 + y * y;
            double e = 0.0, f = 0.0, fz = 0.0, fzz = 0.0;  // sums over z of w/r^3, 3 w/r^5, 3 w z/r^5, 3 w z^2/r^5
            for (int c = 0; c < fr.n; ++c) {
                const double z = on ? Z + fr.u[c] * uz : 1.0;
                const double q = rsqrt(s2 + z * z), q2 = q * q;
                const double i3 = fr.w[c] * q * q2, i5 = 3.0 * i3 * q2;
                e += i3;
                f += i5;
                fz += i5 * z;
                fzz += i5 * z * z;
            }
            acc[0] += wb * (e - x2 * f);
            acc[1] += wb * (e - y * y * f);
            acc[2] += wb * (e - fzz);
            acc[3] -= wb * (x * y * f);
            acc[4] -= wb * (x * fz);
            acc[5] -= wb * (y * fz);
        }
    }
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        acc[i] += __shfl_xor(acc[i], 1, 64);
        acc[i] += __shfl_xor(acc[i], 2, 64);
    }
    if (!on || at >= n || part != 0) return;
    const double s = ux * uy * uz / (4.0 * M_PI);
    if (ix == 0) acc[3] = acc[4] = 0.0;
    if (iy == 0) acc[3] = acc[5] = 0.0;
    if (iz == 0) acc[4] = acc[5] = 0.0;
#pragma unroll
    for (int i = 0; i < 6; ++i) oct[i * n + idx] = s * acc[i];
}

// place component comp of the octant at wrap-around indices of the padded
// real grid [Pz][Py][Px] (zero elsewhere), with its parity signs
__global__ void k_scatter_tensor(const double* __restrict__ oct, int comp, int nx, int ny, int nz, int Px, int Py,
                                 int Pz, double* __restrict__ real) {
    const long n = (long)nx * ny * nz;
    const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= n) return;
    const int ix = (int)(idx % nx);
    const int iy = (int)((idx / nx) % ny);
    const int iz = (int)(idx / ((long)nx * ny));
    const bool ox = comp == 3 || comp == 4, oy = comp == 3 || comp == 5, oz = comp == 4 || comp == 5;
    const double v = oct[comp * n + idx];
    for (int sz = 0; sz < (iz > 0 ? 2 : 1); ++sz)
        for (int sy = 0; sy < (iy > 0 ? 2 : 1); ++sy)
            for (int sx = 0; sx < (ix > 0 ? 2 : 1); ++sx) {
                const int pz = sz ? Pz - iz : iz, py = sy ? Py - iy : iy, px = sx ? Px - ix : ix;
                double sg = 1.0;
                if (ox && sx) sg = -sg;
                if (oy && sy) sg = -sg;
                if (oz && sz) sg = -sg;
                real[((long)pz * Py + py) * Px + px] = sg * v;
            }
}

// real part of one component's spectrum [Pz][Py][SX] -> folded kernel
// (kernel_index) and, for the fused pass of thin meshes (kcol given), its
// [kx][kz][comp][KYS] form, times scale; per-block max |Im| for the realness check
template <typename T>
__global__ __launch_bounds__(NT) void k_fold(const cx<double>* __restrict__ spec, int SX, int Kx, int Py, int Kyf,
                                             int Kzf, double scale, int comp, T* __restrict__ kfold,
                                             T* __restrict__ kcol, int KYS, double* __restrict__ parts) {
    __shared__ double red[NT];
    const long n = (long)Kzf * Kyf * Kx;
    double mx = 0.0;
    for (long e = (long)blockIdx.x * NT + threadIdx.x; e < n; e += (long)gridDim.x * NT) {
        const int kx = (int)(e % Kx);
        const long r = e / Kx;
        const int kyf = (int)(r % Kyf), kzf = (int)(r / Kyf);
        const cx<double> v = spec[((long)kzf * Py + kyf) * SX + kx];
        kfold[kernel_index<T>(kyf, kx, kzf, comp, SX, Kzf)] = (T)(v.x * scale);
        if (kcol) kcol[(((long)kx * Kzf + kzf) * 6 + comp) * KYS + kyf] = (T)(v.x * scale);
        mx = fmax(mx, fabs(v.y * scale));
    }
    red[threadIdx.x] = mx;
    __syncthreads();
    for (int s = NT / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + s]);
        __syncthreads();
    }
    if (threadIdx.x == 0) parts[blockIdx.x] = red[0];
}

hipError_t launch_newell_octant(hipStream_t s, int nx, int ny, int nz, double dx, double dy, double dz,
                                double* octant) {
    const long n = (long)nx * ny * nz;
    // N is invariant under a common scaling of offsets and cell: use units of the largest side
    const double m = std::fmax(dx, std::fmax(dy, dz));
    const double ux = dx / m, uy = dy / m, uz = dz / m;
    const double Rs = std::fmin(FAR_SWITCH_SIDE, FAR_SWITCH_VOL * std::cbrt(ux * uy * uz));  // longest side = 1
    // the box that holds every offset with R < Rs (one more per axis than
    // rounding of the products could leave out)
    auto box = [&](int nn, double u) { return (int)std::fmin((double)nn, std::floor(Rs / u) + 2.0); };
    const int bx = box(nx, ux), by = box(ny, uy), bz = box(nz, uz);
    const long nbox = (long)bx * by * bz;
    if (nbox > (1L << 30) || (4 * n + NT - 1) / NT > 0x7fffffffL) return hipErrorInvalidValue;
    k_newell_near<<<(unsigned)((nbox + NEAR_GROUPS - 1) / NEAR_GROUPS), NT, 0, s>>>(nx, ny, nz, bx, by, bz, ux, uy, uz,
                                                                                     Rs, octant);
    k_newell_far<<<(unsigned)((4 * n + NT - 1) / NT), NT, 0, s>>>(nx, ny, nz, ux, uy, uz, Rs, octant);
    return hipGetLastError();
}

hipError_t launch_scatter_tensor(hipStream_t s, const double* octant, int comp, int nx, int ny, int nz, int Px,
                                 int Py, int Pz, double* real) {
    const long n = (long)nx * ny * nz;
    k_scatter_tensor<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(octant, comp, nx, ny, nz, Px, Py, Pz, real);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_fold(hipStream_t s, const cx<double>* spec, int SX, int Kx, int Py, int Pz, int Kyf, int Kzf,
                       double scale, int comp, T* kfold, T* kcol, int KYS, double* parts, int nparts) {
    (void)Pz;
    k_fold<T><<<(unsigned)nparts, NT, 0, s>>>(spec, SX, Kx, Py, Kyf, Kzf, scale, comp, kfold, kcol, KYS, parts);
    return hipGetLastError();
}

template hipError_t launch_fold<float>(hipStream_t, const cx<double>*, int, int, int, int, int, int, double, int,
                                       float*, float*, int, double*, int);
template hipError_t launch_fold<double>(hipStream_t, const cx<double>*, int, int, int, int, int, int, double, int,
                                        double*, double*, int, double*, int);

}  // namespace llgx

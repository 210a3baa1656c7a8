// kernels_demag.hip -- the demagnetising kernel, built in FP64 on the GPU.
//
// Section "Magnetostatic field", paragraph "Magnetostatic kernel": the field of
// a uniformly magnetised cell, averaged over the destination cell.  For every
// displacement d = (i dx, j dy, k dz) of the non-negative octant:
//   near (|d| < 2.5 cell diagonals): the closed form of Newell, Williams and
//     Dunlop (1993), a weighted second difference (weights 2, -1, -1 per
//     axis) of f (diagonal) and g (off-diagonal) over the corner lattice;
//   far: N_ij = -(V/4 pi) <(3 w_i w_j - |w|^2 delta_ij)/|w|^5>, the dipole
//     tensor averaged over the triangular density of destination-minus-source
//     offsets with the Gauss rule of that density along each axis; the number of
//     points per axis falls from 11 to 3 with distance (the paper's "number of
//     integration points chosen by distance"), keeping the relative error near
//     1e-12 where Newell's cancellation would not.
// The octant is mirrored into the padded grid with the parities of each
// component (xx, yy, zz even; xy odd in x, y; xz odd in x, z; yz odd in y, z;
// every displacement with |i| >= nx is zero), scaled by -mu0/(px py pz),
// Fourier transformed in FP64, and the real spectrum's octant kept in FP32.
// The mirrored array is never formed: along each axis it is even or odd, so its
// transform is a cosine or sine sum over the octant alone, a product with a
// small table that the FP64 matrix cores take.
#include <math.h>

#include "mm_internal.h"

namespace mm {

// Gauss rules of the triangular density 1 - |t| on [-1, 1] with n = 1..11 points,
// table offset n(n-1)/2.  Far from the source the dipole tensor is smooth across
// the density's kink, so n points integrate what took n Gauss-Legendre points on
// each half axis.  Largest relative error of the tensor, and points per cell, over
// cells of aspect 1 to 40 at the nearest distance (cell diagonals) of each band:
//   from 2.5: 11 points 9e-14, 1331 (8 per half axis: 2e-12, 4096)
//   from 4:    8 points 3e-13,  512 (6: 7e-12, 1728)
//   from 6:    6 points 5e-12,  216 (5: 1e-11, 1000)
//   from 12:   5 points 5e-13,  125 (4: 2e-11,  512)
//   from 24:   4 points 8e-13,   64 (4 until 50, then 3: 3e-12, 216)
//   from 80:   3 points 9e-13,   27 (3, and 2 from 400: 9e-12, 64)
constexpr int GT_MAXN = 11;
constexpr int GT_TABLE = GT_MAXN * (GT_MAXN + 1) / 2;
struct TriangleGauss {
    double x[GT_TABLE], w[GT_TABLE];
    TriangleGauss() {
        // the density's moments by Gauss-Legendre points on [0, 1] (exact to
        // degree 2 NL - 1; degree 2 GT_MAXN + 1 is needed), even part only: the
        // orthonormal polynomials p_k alternate in parity
        constexpr int NL = 12;
        double s[NL], m[NL], beta[GT_MAXN + 1], pa[NL], pb[NL];
        for (int i = 0; i < NL; ++i) {
            double t = cos(M_PI * (i + 0.75) / (NL + 0.5)), dp = 1.0;
            for (int it = 0; it < 100; ++it) {
                const double pn = legendre(NL, t, dp), dt = pn / dp;
                t -= dt;
                if (fabs(dt) < 1e-16) break;
            }
            (void)legendre(NL, t, dp);
            s[i] = 0.5 * (1.0 + t);
            m[i] = 2.0 * (1.0 - s[i]) / ((1.0 - t * t) * dp * dp);  // both halves
            pa[i] = 0.0;
            pb[i] = 1.0;  // p_0: the density's integral is 1
        }
        // recurrence t p_k = beta_{k+1} p_{k+1} + beta_k p_{k-1}, orthogonalised on the points
        beta[0] = 0.0;
        for (int k = 0; k < GT_MAXN; ++k) {
            double q[NL], n2 = 0.0;
            for (int i = 0; i < NL; ++i) {
                q[i] = s[i] * pb[i] - beta[k] * pa[i];
                n2 += m[i] * q[i] * q[i];
            }
            beta[k + 1] = sqrt(n2);
            for (int i = 0; i < NL; ++i) {
                pa[i] = pb[i];
                pb[i] = q[i] / beta[k + 1];
            }
        }
        // nodes: the zeros of p_n, symmetric about 0; weights 1 / sum_{k<n} p_k^2
        for (int n = 1; n <= GT_MAXN; ++n) {
            double* xn = x + n * (n - 1) / 2;
            double* wn = w + n * (n - 1) / 2;
            int found = 0;
            if (n & 1) xn[found++] = 0.0;
            constexpr int SCAN = 512;
            for (int c = 0; c < SCAN && found < n; ++c) {
                double lo = (c + 0.5) / SCAN, hi = (c + 1.5) / SCAN, sum;
                if (c == 0) lo = 0.25 / SCAN;
                const double flo = value(beta, n, lo, sum);
                if (flo * value(beta, n, hi, sum) > 0.0) continue;
                for (int it = 0; it < 60; ++it) {
                    const double mid = 0.5 * (lo + hi);
                    if (flo * value(beta, n, mid, sum) > 0.0)
                        lo = mid;
                    else
                        hi = mid;
                }
                xn[found++] = 0.5 * (lo + hi);
                xn[found++] = -0.5 * (lo + hi);
            }
            for (int i = 0; i < n; ++i) {
                double sum;
                (void)value(beta, n, xn[i], sum);
                wn[i] = 1.0 / sum;
            }
        }
    }
    // P_n(t) by the recurrence, P_n'(t) in dp
    static double legendre(int n, double t, double& dp) {
        double p0 = 1.0, p1 = t;
        for (int k = 2; k <= n; ++k) {
            const double p2 = ((2 * k - 1) * t * p1 - (k - 1) * p0) / k;
            p0 = p1;
            p1 = p2;
        }
        dp = n * (t * p1 - p0) / (t * t - 1.0);
        return p1;
    }
    // p_n(t); sum: sum_{k<n} p_k(t)^2
    static double value(const double* beta, int n, double t, double& sum) {
        double p0 = 0.0, p1 = 1.0;
        sum = 0.0;
        for (int k = 0; k < n; ++k) {
            sum += p1 * p1;
            const double p2 = (t * p1 - beta[k] * p0) / beta[k + 1];
            p0 = p1;
            p1 = p2;
        }
        return p1;
    }
};

__device__ inline double newell_f(double x, double y, double z) {
    const double x2 = x * x, y2 = y * y, z2 = z * z;
    const double r = sqrt(x2 + y2 + z2);
    double o = (2.0 * x2 - y2 - z2) * r / 6.0;
    const double rxz = sqrt(x2 + z2), rxy = sqrt(x2 + y2);
    if (rxz > 0.0) o += 0.5 * y * (z2 - x2) * asinh(y / rxz);
    if (rxy > 0.0) o += 0.5 * z * (y2 - x2) * asinh(z / rxy);
    if (x * r != 0.0) o -= x * y * z * atan(y * z / (x * r));
    return o;
}

__device__ inline double newell_g(double x, double y, double z) {
    const double x2 = x * x, y2 = y * y, z2 = z * z;
    const double r = sqrt(x2 + y2 + z2);
    double o = -x * y * r / 3.0;
    const double rxy = sqrt(x2 + y2), ryz = sqrt(y2 + z2), rxz = sqrt(x2 + z2);
    if (rxy > 0.0) o += x * y * z * asinh(z / rxy);
    if (ryz > 0.0) o += y / 6.0 * (3.0 * z2 - y2) * asinh(x / ryz);
    if (rxz > 0.0) o += x / 6.0 * (3.0 * z2 - x2) * asinh(y / rxz);
    if (z * r != 0.0) o -= z2 * z / 6.0 * atan(x * y / (z * r));
    if (y * r != 0.0) o -= z * y2 / 2.0 * atan(x * z / (y * r));
    if (x * r != 0.0) o -= z * x2 / 2.0 * atan(y * z / (x * r));
    return o;
}

// weight of corner offset o (0, 1, 2 for -1, 0, 1) along one axis
__device__ inline double corner_weight(int o) { return o == 1 ? 2.0 : -1.0; }

// Distance from the source in cell diagonals.  Nothing fuses here, so the near and
// the far kernel get the same bits for a cell and exactly one of them writes it,
// also where the distance is RHO_WAVE itself ((20, 4, 4) of cubic cells).
__device__ inline double cell_distance(double X, double Y, double Z, const double (&cell)[3]) {
#pragma clang fp contract(off)
    return sqrt(X * X + Y * Y + Z * Z) / sqrt(cell[0] * cell[0] + cell[1] * cell[1] + cell[2] * cell[2]);
}

// Quadrature points per axis (TriangleGauss).
constexpr double RHO_NEAR = 2.5, RHO_WAVE = 12.0;
__device__ inline int far_order(double rho) {
    if (rho < 4.0) return 11;
    if (rho < 6.0) return 8;
    if (rho < RHO_WAVE) return 6;
    if (rho < 24.0) return 5;
    if (rho < 80.0) return 4;
    return 3;
}

// Nodes and weights of every order along each axis, scaled to [-h, h].
struct AxisTable {
    double s[3][GT_TABLE], w[3][GT_TABLE];
};
__device__ inline void axis_table(AxisTable& t, const TriangleGauss& gt, const double (&cell)[3], int tid, int nth) {
    for (int e = tid; e < 3 * GT_TABLE; e += nth) {
        const int ax = e / GT_TABLE, r = e - ax * GT_TABLE;
        t.s[ax][r] = cell[ax] * gt.x[r];
        t.w[ax][r] = gt.w[r];
    }
}

// Sums over the quadrature points of one (x, y) node pair: w |u|^-5 times xx,
// yy, zz, xy, xz, yz of u.  Along z only three sums are needed per point; the
// trace part of the dipole tensor follows from the same sums.
__device__ inline void dipole_line(double ux, double uy, double wab, double Z, const double* sz, const double* wz,
                                   int np, double (&acc)[6]) {
    const double q = ux * ux + uy * uy;
    double a0 = 0.0, a1 = 0.0, a2 = 0.0;
    for (int c = 0; c < np; ++c) {
        const double uz = Z + sz[c];
        const double ir = rsqrt(q + uz * uz), ir2 = ir * ir;
        const double w = wz[c] * (ir2 * ir2 * ir), wu = w * uz;
        a0 += w;
        a1 += wu;
        a2 += wu * uz;
    }
    a0 *= wab;
    a1 *= wab;
    acc[0] += ux * ux * a0;
    acc[1] += uy * uy * a0;
    acc[2] += wab * a2;
    acc[3] += ux * uy * a0;
    acc[4] += ux * a1;
    acc[5] += uy * a1;
}
// N from the sums: -(V/4 pi) (3 <u u> - tr <u u>)
__device__ inline void dipole_finish(const double (&acc)[6], double vol, double (&t)[6]) {
    const double pre = -vol / (4.0 * M_PI);
    t[0] = pre * (2.0 * acc[0] - acc[1] - acc[2]);
    t[1] = pre * (2.0 * acc[1] - acc[0] - acc[2]);
    t[2] = pre * (2.0 * acc[2] - acc[0] - acc[1]);
    t[3] = pre * 3.0 * acc[3];
    t[4] = pre * 3.0 * acc[4];
    t[5] = pre * 3.0 * acc[5];
}

// Cells from RHO_WAVE cell diagonals on: a thread per cell, bound by FP64
// arithmetic (27 to 125 points, about 25 operations each): 1 M cells (256 x 256
// x 16) 298 us with 216 or 512 points of the half-axis rules, 67 us.
__global__ void __launch_bounds__(256) k_tensor_far(int nx, int ny, int nz, double dx, double dy, double dz,
                                                    const TriangleGauss gt, double* __restrict__ out) {
    __shared__ AxisTable tab;
    const double cell[3] = {dx, dy, dz};
    axis_table(tab, gt, cell, threadIdx.x, 256);
    __syncthreads();
    const long long n = (long long)nx * ny * nz;
    const long long id = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= n) return;
    const int i = (int)(id % nx);
    const long long rest = id / nx;
    const int j = (int)(rest % ny), k = (int)(rest / ny);
    const double X = i * dx, Y = j * dy, Z = k * dz;
    const double rho = cell_distance(X, Y, Z, cell);
    if (rho < RHO_WAVE) return;
    const int np = far_order(rho), off = np * (np - 1) / 2;
    double acc[6] = {0, 0, 0, 0, 0, 0}, t[6];
    for (int a = 0; a < np; ++a)
        for (int b = 0; b < np; ++b)
            dipole_line(X + tab.s[0][off + a], Y + tab.s[1][off + b], tab.w[0][off + a] * tab.w[1][off + b], Z,
                        tab.s[2] + off, tab.w[2] + off, np, acc);
    dipole_finish(acc, dx * dy * dz, t);
    for (int c = 0; c < 6; ++c) out[c * n + id] = t[c];
}

// Cells nearer than RHO_WAVE, a wave each (grid: the box bx x by x bz that
// holds them): their 216 to 1331 quadrature points or 162 evaluations of
// Newell's functions, spread over the lanes.  (In a thread they took 1.3 ms
// whatever the grid, a chain the rest of the launch waited for.)
__global__ void __launch_bounds__(256) k_tensor_near(int nx, int ny, int nz, int bx, int by, int bz, double dx,
                                                     double dy, double dz, const TriangleGauss gt,
                                                     double* __restrict__ out) {
    __shared__ AxisTable tab;
    __shared__ double val[4][162];
    const double cell[3] = {dx, dy, dz};
    axis_table(tab, gt, cell, threadIdx.x, 256);
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long long cid = (long long)blockIdx.x * 4 + wave;
    if (cid >= (long long)bx * by * bz) return;
    const int i = (int)(cid % bx);
    const long long rest = cid / bx;
    const int j = (int)(rest % by), k = (int)(rest / by);
    const double X = i * dx, Y = j * dy, Z = k * dz;
    const double rho = cell_distance(X, Y, Z, cell);
    if (rho >= RHO_WAVE) return;
    double t[6];
    if (rho < RHO_NEAR) {
        // component c at corner p (x offset slowest), the axes permuted so
        // that f takes xx and g takes xy
        for (int e = lane; e < 162; e += 64) {
            const int c = e / 27, p = e - 27 * c;
            const int o0 = p / 9, o1 = p / 3 % 3, o2 = p % 3;
            const int a0 = c == 1 || c == 5 ? 1 : (c == 2 ? 2 : 0);
            const int a1 = c == 0 || c == 2 || c == 3 ? 1 : (c == 1 ? 0 : 2);
            const int a2 = 3 - a0 - a1;
            const double P[3] = {X, Y, Z};
            const double u = P[a0] + (o0 - 1) * cell[a0], v = P[a1] + (o1 - 1) * cell[a1],
                         w = P[a2] + (o2 - 1) * cell[a2];
            val[wave][e] = corner_weight(o0) * corner_weight(o1) * corner_weight(o2) *
                           (c < 3 ? newell_f(u, v, w) : newell_g(u, v, w));
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int c = 0; c < 6; ++c) {
            double s = 0.0;
            for (int p = 0; p < 27; ++p) s += val[wave][27 * c + p];
            t[c] = s / (4.0 * M_PI * dx * dy * dz);
        }
    } else {
        const int np = far_order(rho), off = np * (np - 1) / 2;
        double acc[6] = {0, 0, 0, 0, 0, 0};
        for (int p = lane; p < np * np; p += 64) {
            const int a = p / np, b = p - a * np;
            dipole_line(X + tab.s[0][off + a], Y + tab.s[1][off + b], tab.w[0][off + a] * tab.w[1][off + b], Z,
                        tab.s[2] + off, tab.w[2] + off, np, acc);
        }
#pragma unroll
        for (int c = 0; c < 6; ++c)
            for (int o = 32; o > 0; o >>= 1) acc[c] += __shfl_xor(acc[c], o, 64);
        dipole_finish(acc, dx * dy * dz, t);
    }
    if (lane == 0) {
        const long long n = (long long)nx * ny * nz, id = ((long long)k * ny + j) * nx + i;
#pragma unroll
        for (int c = 0; c < 6; ++c) out[c * n + id] = t[c];
    }
}

hipError_t demag_tensor_octant(int nx, int ny, int nz, double dx, double dy, double dz, double* out,
                               hipStream_t s) {
    static const TriangleGauss gt;
    const long long n = (long long)nx * ny * nz;
    const double reach = RHO_WAVE * sqrt(dx * dx + dy * dy + dz * dz);
    // a cell of slack: both kernels test rho themselves
    auto box = [&](int m, double d) { return reach / d + 2.0 < m ? (int)(reach / d) + 2 : m; };
    const int bx = box(nx, dx), by = box(ny, dy), bz = box(nz, dz);
    const long long nb = (long long)bx * by * bz;
    const double cx = (nx - 1) * dx, cy = (ny - 1) * dy, cz = (nz - 1) * dz;
    hipLaunchKernelGGL(k_tensor_near, dim3((unsigned)((nb + 3) / 4)), dim3(256), 0, s, nx, ny, nz, bx, by, bz, dx, dy,
                       dz, gt, out);
    if (sqrt(cx * cx + cy * cy + cz * cz) > 0.999 * reach)
        hipLaunchKernelGGL(k_tensor_far, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, nx, ny, nz, dx, dy, dz,
                           gt, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Periodic images (paragraph "Periodic boundary conditions"): the kernel entry
// of box displacement (i, j, k) is the sum of N over the displacements
// i + s nx (and likewise along y, z) that stay inside the window |d| <= n P - 1
// of a periodic axis; a non-periodic axis keeps d = i.  The window tensor is
// stored for d >= 0 (lengths wx, wy, wz); a negative d takes the parity of the
// component along that axis.  With these sums in place of the octant, the
// mirrored entries (next section) give the displacement -d the entry of the box
// displacement n - d (the sums satisfy S(n - d) = parity S(d)), so the padded
// linear convolution becomes the cyclic one along the periodic axes.
__global__ void __launch_bounds__(256) k_fold_images(int nx, int ny, int nz, int wx, int wy, int wz, int qx,
                                                     int qy, int qz, const double* __restrict__ win,
                                                     double* __restrict__ oct) {
    const long long n = (long long)nx * ny * nz;
    const long long id = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= n) return;
    const int i = (int)(id % nx);
    const long long rest = id / nx;
    const int j = (int)(rest % ny), k = (int)(rest / ny);
    const long long wn = (long long)wx * wy * wz;
    double acc[6] = {0, 0, 0, 0, 0, 0};
    for (int sz = -qz; sz <= qz; ++sz) {
        const int dk = k + sz * nz;
        if (dk <= -wz || dk >= wz) continue;
        const int ak = dk < 0 ? -dk : dk;
        const bool nzg = dk < 0;
        for (int sy = -qy; sy <= qy; ++sy) {
            const int dj = j + sy * ny;
            if (dj <= -wy || dj >= wy) continue;
            const int aj = dj < 0 ? -dj : dj;
            const bool nyg = dj < 0;
            for (int sx = -qx; sx <= qx; ++sx) {
                const int di = i + sx * nx;
                if (di <= -wx || di >= wx) continue;
                const int ai = di < 0 ? -di : di;
                const bool nxg = di < 0;
                const long long e = ((long long)ak * wy + aj) * wx + ai;
                acc[0] += win[e];
                acc[1] += win[wn + e];
                acc[2] += win[2 * wn + e];
                acc[3] += (nxg != nyg ? -1.0 : 1.0) * win[3 * wn + e];  // xy: odd in x, y
                acc[4] += (nxg != nzg ? -1.0 : 1.0) * win[4 * wn + e];  // xz: odd in x, z
                acc[5] += (nyg != nzg ? -1.0 : 1.0) * win[5 * wn + e];  // yz: odd in y, z
            }
        }
    }
    for (int c = 0; c < 6; ++c) oct[c * n + id] = acc[c];
}

hipError_t demag_fold_images(int nx, int ny, int nz, const int* w, const int* pbc, const double* win,
                             double* oct, hipStream_t s) {
    const long long n = (long long)nx * ny * nz;
    hipLaunchKernelGGL(k_fold_images, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, nx, ny, nz, w[0], w[1],
                       w[2], pbc[0], pbc[1], pbc[2], win, oct);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The spectrum of the mirrored octant, axis by axis.  Along an axis of n cells
// and padded length p the mirrored entries are a(d), 0 <= d < n, and +-a(d) at
// p - d, so output k is the real sum over d of f(d) cos(2 pi k d / p) a(d) for
// an even component and -i times that of f(d) sin(2 pi k d / p) a(d) for an odd
// one (f(0) = 1, else 2; an unpadded periodic axis, p = n, holds every entry
// itself: f = 1).  Each component is odd in two axes or none: the two factors
// -i give the sign -1.
//
// Why products instead of transforms: the octant has an eighth of the padded
// points, and n x (p/2 + 1) tables on the FP64 matrix cores need no exchange,
// no twiddles and no second pass over memory per axis.  One 256 x 256 x 16
// kernel: mirror fill, 18 complex transforms and extraction 4.8 ms -> 0.34 ms.  The
// work per point grows with the axis, so long axes gain least: the whole
// construction, tensor included, of 2048 x 2048 cells 7.95 -> 4.61 ms, of
// 2048 x 1 x 1 1.45 -> 0.56 ms, of 128 x 128 x 128 11.5 -> 0.56 ms.

typedef double f64x4 __attribute__((ext_vector_type(4)));

// A[m = lane % 16][k = lane / 16], B[k = lane / 16][n = lane % 16],
// result register i = D[m = 4 i + lane / 16][n = lane % 16]
__device__ inline f64x4 mfma64(double a, double b, f64x4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Tables of one axis: cosines then sines, [d][k], d padded with zero rows to a
// multiple of 4 and k with zero columns to a multiple of 32.
struct AxisDim {
    int n, p, kh;   // cells, padded length, outputs p/2 + 1
    __host__ __device__ int rows() const { return (n + 3) & ~3; }
    __host__ __device__ int cols() const { return (kh + 31) & ~31; }
    __host__ __device__ long long table() const { return (long long)rows() * cols(); }
};
static AxisDim axis_dim(int n, int p) { return AxisDim{n, p, p / 2 + 1}; }

__global__ void __launch_bounds__(256) k_axis_table(AxisDim a, double* __restrict__ tab) {
    const long long e = (long long)blockIdx.x * 256 + threadIdx.x;
    if (e >= a.table()) return;
    const int d = (int)(e / a.cols()), k = (int)(e - (long long)d * a.cols());
    double c = 0.0, s = 0.0;
    if (d < a.n && k < a.kh) {
        const int m = (int)((long long)k * d & (a.p - 1));
        sincospi(2.0 * (double)m / (double)a.p, &s, &c);
        const double f = (a.p > a.n && d > 0) ? 2.0 : 1.0;
        c *= f;
        s *= f;
    }
    tab[e] = c;
    tab[a.table() + e] = s;
}

// dst[c][o][k][i] = sum_d T[d][k] src[c][o][d][i], i < inner: a wave takes 32
// outputs k of 64 columns i (eight accumulator tiles for six operand loads).
// odd: bit c set when component c takes the sine table.
__global__ void __launch_bounds__(256) k_axis(AxisDim a, const double* __restrict__ tab, int odd, int outer,
                                              int inner, const double* __restrict__ src,
                                              double* __restrict__ dst) {
    const int lane = threadIdx.x & 63, l = lane & 15, q = lane >> 4;
    const int i0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * 64, k0 = blockIdx.y * 32;
    if (i0 >= inner) return;
    for (int co = blockIdx.z; co < outer; co += gridDim.z) {
        const int c = co / (outer / (odd >> 8)), cols = a.cols();
        const double* T = tab + ((odd >> c) & 1 ? a.table() : 0) + k0 + l;
        const double* x = src + (long long)co * a.n * inner;
        int col[4];
        bool in[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            in[t] = i0 + 16 * t + l < inner;
            col[t] = in[t] ? i0 + 16 * t + l : 0;
        }
        f64x4 acc[2][4] = {};
#pragma unroll 2
        for (int d0 = 0; d0 < a.n; d0 += 4) {
            const int d = d0 + q;
            const double ta = T[d * cols], tb = T[d * cols + 16];  // zero rows past n
            const double* row = x + (long long)(d < a.n ? d : 0) * inner;
            double v[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) v[t] = row[col[t]];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                acc[0][t] = mfma64(ta, v[t], acc[0][t]);
                acc[1][t] = mfma64(tb, v[t], acc[1][t]);
            }
        }
        double* y = dst + (long long)co * a.kh * inner;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int k = k0 + 16 * u + 4 * r + q;
                    if (k < a.kh && in[t]) y[(long long)k * inner + col[t]] = acc[u][t][r];
                }
    }
}

// The x axis, scaled and rounded to FP32 in the layout the convolution reads,
// [kx][ky_h][kz_h][ncomp]: a workgroup takes 32 kx of 32 (ky, kz) rows, a wave
// per component; the tile goes through LDS so that it is written in runs.
__global__ void __launch_bounds__(384) k_axis_x(AxisDim a, const double* __restrict__ tab, int odd, int kyh, int kzh,
                                                int ncomp, const double* __restrict__ src, double scale,
                                                float* __restrict__ khat) {
    __shared__ float tile[32 * 32 * 6];
    const int lane = threadIdx.x & 63, l = lane & 15, q = lane >> 4, c = threadIdx.x >> 6;
    const long long rows = (long long)kyh * kzh, r0 = (long long)blockIdx.x * 32;
    const int k0 = blockIdx.y * 32, cols = a.cols();
    const double* T = tab + ((odd >> c) & 1 ? a.table() : 0) + k0 + l;
    const double* x[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        long long r = r0 + 16 * t + l;
        if (r >= rows) r = 0;
        const long long ky = r / kzh, kz = r - ky * kzh;
        x[t] = src + (((long long)c * kzh + kz) * kyh + ky) * a.n;
    }
    f64x4 acc[2][2] = {};
#pragma unroll 4
    for (int d0 = 0; d0 < a.n; d0 += 4) {
        const int d = d0 + q, dc = d < a.n ? d : 0;
        const double ta = T[d * cols], tb = T[d * cols + 16];
        const double v0 = x[0][dc], v1 = x[1][dc];
        acc[0][0] = mfma64(ta, v0, acc[0][0]);
        acc[1][0] = mfma64(tb, v0, acc[1][0]);
        acc[0][1] = mfma64(ta, v1, acc[0][1]);
        acc[1][1] = mfma64(tb, v1, acc[1][1]);
    }
    const double sc = c < 3 ? scale : -scale;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                tile[((16 * u + 4 * r + q) * 32 + 16 * t + l) * ncomp + c] = (float)(sc * acc[u][t][r]);
    __syncthreads();
    const int run = 32 * ncomp;
    const long long left = (rows - r0) * ncomp;  // floats of this tile's rows that exist
    for (int e = threadIdx.x; e < 32 * run; e += blockDim.x) {
        const int k = e / run, f = e - k * run;
        if (k0 + k < a.kh && f < left) khat[((long long)(k0 + k) * rows + r0) * ncomp + f] = tile[e];
    }
}

// Doubles of the octant's buffer (the y results of a 3D grid overwrite the
// octant) and of the scratch (the tables, then the z or 2D y results).
size_t demag_octant_doubles(int nx, int ny, int nz, int py, int pz) {
    const size_t oct = (size_t)6 * nx * ny * nz, by = pz > 1 ? (size_t)6 * (pz / 2 + 1) * (py / 2 + 1) * nx : 0;
    return oct > by ? oct : by;
}
size_t demag_spectrum_work(int nx, int ny, int nz, int px, int py, int pz) {
    const AxisDim x = axis_dim(nx, px), y = axis_dim(ny, py), z = axis_dim(nz, pz);
    return (size_t)(2 * (x.table() + y.table() + z.table())) +
           (pz > 1 ? (size_t)6 * z.kh * ny * nx : (size_t)4 * y.kh * nx);
}

hipError_t demag_kernel_spectrum(int nx, int ny, int nz, int px, int py, int pz, double* octant, double* work,
                                 float* khat, int ncomp, hipStream_t s) {
    const AxisDim x = axis_dim(nx, px), y = axis_dim(ny, py), z = axis_dim(nz, pz);
    double* tx = work;
    double* ty = tx + 2 * x.table();
    double* tz = ty + 2 * y.table();
    double* rest = tz + 2 * z.table();
    const int kz = pz > 1 ? z.kh : 1;
    double* by = pz > 1 ? octant : rest;
    auto table = [&](const AxisDim& a, double* t) {
        hipLaunchKernelGGL(k_axis_table, dim3((unsigned)((a.table() + 255) / 256)), dim3(256), 0, s, a, t);
    };
    // components odd along x: xy, xz; y: xy, yz; z: xz, yz (the count of components above bit 8)
    const int odd_x = 8 | 16, odd_y = 8 | 32, odd_z = 16 | 32, count = ncomp << 8;
    auto axis = [&](const AxisDim& a, const double* t, int odd, int outer, int inner, const double* in, double* out) {
        const int gz = outer < 32768 ? outer : 32768;
        hipLaunchKernelGGL(k_axis, dim3((unsigned)((inner + 255) / 256), (unsigned)((a.kh + 31) / 32), (unsigned)gz),
                           dim3(256), 0, s, a, t, odd | count, outer, inner, in, out);
    };
    table(x, tx);
    table(y, ty);
    const double* in = octant;
    if (pz > 1) {
        table(z, tz);
        axis(z, tz, odd_z, ncomp, ny * nx, in, rest);
        in = rest;
    }
    axis(y, ty, odd_y, ncomp * kz, nx, in, by);
    const long long rows = (long long)y.kh * kz;
    hipLaunchKernelGGL(k_axis_x, dim3((unsigned)((rows + 31) / 32), (unsigned)((x.kh + 31) / 32)), dim3(64 * ncomp), 0,
                       s, x, tx, odd_x, y.kh, kz, ncomp, by, -MU0 / ((double)px * py * pz), khat);
    return hipGetLastError();
}

}  // namespace mm

// Adjoint of the periodic 2D field solve in three launches: lam_rho = A^T lam_E,
// lam_rho_hat = (i kappa_x lam_Ex_hat + i kappa_y lam_Ey_hat) / K^2 (0 at k = 0),
// through the line transforms of the forward solve.
//
//   1. k_adj_rows: one workgroup per row, the transform along x of lam_Ex + i lam_Ey
//      (cleared behind it).
//   2. k_adj_cols: one workgroup per column pair kx, nx - kx. The x-spectra X and Y of
//      the two real fields follow from the pair; V = i kappa_x X + (the centred
//      difference of Y along y), whose symbol is i kappa_y; one transform along y, the
//      division by K^2, one back: the half spectra of the rows of lam_rho.
//   3. k_adj_rows_inv: one workgroup per pair of rows, W = H_0 + i H_1 back along x.
//
// Bound by launch and memory latency. The gradient of 40 steps, 256 x 256, 1.0M
// particles mixed: 8.56 ms with seven launches through the library, 7.69 here.
#include "apic_dftlds.h"

namespace apic {
namespace {

// A line's transform, and its LDS in lines of n complex: power-of-two sides.
struct Pow2Side {
    static constexpr int kLines = 2;
    int n, lg, lgmax;
    const double2 *tw;
    __device__ __forceinline__ void prepare(double2 *) const {}
    template <int SIGN>
    __device__ __forceinline__ double2 *run(double2 *a, double2 *b, const double2 *) const {
        return fft_lds_one<SIGN>(a, b, lg, tw, lgmax, fft_twiddles(lg, tw, lgmax));
    }
};

// Sides of any length: the table of roots in a third line.
struct DftSide {
    static constexpr int kLines = 3;
    DftLine f;
    const double2 *tw;
    __device__ __forceinline__ void prepare(double2 *T) const { load_roots(T, tw, f.n); }
    template <int SIGN>
    __device__ __forceinline__ double2 *run(double2 *a, double2 *b, const double2 *T) const {
        return dft_line<SIGN>(a, b, T, f);
    }
};

template <typename Side>
__global__ void __launch_bounds__(kDftBlock) k_adj_rows(Geo g, double *lE, double2 *Z, Side sx) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int nx = g.nx;
    const int64_t row = (int64_t)blockIdx.x * nx, G = (int64_t)nx * g.ny;
    double2 *a = (double2 *)smem, *b = a + nx, *T = b + nx;
    sx.prepare(T);
    for (int i = threadIdx.x; i < nx; i += blockDim.x) {
        a[i] = make_double2(lE[row + i], lE[G + row + i]);
        lE[row + i] = 0.0;
        lE[G + row + i] = 0.0;
    }
    __syncthreads();
    const double2 *R = sx.template run<-1>(a, b, T);
    for (int i = threadIdx.x; i < nx; i += blockDim.x) Z[row + i] = R[i];
}

// Columns of one XCD adjacent: per = ceil(hx / 8).
template <typename Side>
__global__ void __launch_bounds__(kDftBlock) k_adj_cols(Geo g, const double2 *Z, double2 *H, Side sy, int per,
                                                        CtxDev c) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int nx = g.nx, ny = g.ny, hx = nx / 2 + 1;
    const int kx = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
    if (kx >= hx) return;
    const int km = kx == 0 ? 0 : nx - kx;
    double2 *A = (double2 *)smem, *B = A + ny, *T = B + ny;
    sy.prepare(T);
    const double kx2 = c.kx2[kx], kax = c.kapx[kx], hy = 0.5 * g.inv_dy;
    for (int y = threadIdx.x; y < ny; y += blockDim.x) {
        const double2 p = Z[(int64_t)y * nx + kx], m = Z[(int64_t)y * nx + km];
        A[y] = make_double2(0.5 * (p.x + m.x), 0.5 * (p.y - m.y));    // X
        B[y] = make_double2(0.5 * (p.y + m.y), -0.5 * (p.x - m.x));   // Y
    }
    __syncthreads();
    for (int y = threadIdx.x; y < ny; y += blockDim.x) {
        const double2 q = B[y == ny - 1 ? 0 : y + 1], r = B[y == 0 ? ny - 1 : y - 1], x = A[y];
        A[y] = make_double2((q.x - r.x) * hy - kax * x.y, (q.y - r.y) * hy + kax * x.x);
    }
    __syncthreads();
    double2 *R = sy.template run<-1>(A, B, T);
    double2 *S = (R == A) ? B : A;
    const double norm = 1.0 / ((double)nx * (double)ny);
    for (int ky = threadIdx.x; ky < ny; ky += blockDim.x) {
        const double inv = (kx == 0 && ky == 0) ? 0.0 : norm / (kx2 + c.ky2[ky]);
        S[ky] = make_double2(R[ky].x * inv, R[ky].y * inv);
    }
    __syncthreads();
    const double2 *P = sy.template run<+1>(S, R, T);
    const bool self = kx == 0 || 2 * kx == nx;   // the spectrum of a real row is real there
    for (int y = threadIdx.x; y < ny; y += blockDim.x) {
        const double2 p = P[y];
        H[(int64_t)y * hx + kx] = make_double2(p.x, self ? 0.0 : p.y);
    }
}

template <typename Side>
__global__ void __launch_bounds__(kDftBlock) k_adj_rows_inv(Geo g, const double2 *H, double *lrho, Side sx) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int nx = g.nx, hx = nx / 2 + 1;
    const bool two = 2 * (int)blockIdx.x + 1 < g.ny;
    const int64_t h0 = (int64_t)(2 * blockIdx.x) * hx, h1 = two ? h0 + hx : h0;
    double2 *a = (double2 *)smem, *b = a + nx, *T = b + nx;
    sx.prepare(T);
    for (int k = threadIdx.x; k < hx; k += blockDim.x) {
        const double2 p = H[h0 + k], q = H[h1 + k];
        a[k] = make_double2(p.x - q.y, p.y + q.x);
        // the negative wavenumbers: conj H_0 + i conj H_1
        if (k > 0 && 2 * k != nx) a[nx - k] = make_double2(p.x + q.y, q.x - p.y);
    }
    __syncthreads();
    const double2 *R = sx.template run<+1>(a, b, T);
    const int64_t r0 = (int64_t)(2 * blockIdx.x) * nx;
    for (int i = threadIdx.x; i < nx; i += blockDim.x) {
        lrho[r0 + i] = R[i].x;
        if (two) lrho[r0 + nx + i] = R[i].y;
    }
}

template <typename Side>
hipError_t launch(const Geo &g, double *lE, double2 *Z, double2 *H, double *lrho, const Side &sx, const Side &sy,
                  int bx, int by, const CtxDev &c, hipStream_t s) {
    const size_t shx = Side::kLines * (size_t)g.nx * sizeof(double2), shy = Side::kLines * (size_t)g.ny * sizeof(double2);
    const int per = (g.nx / 2 + 1 + 7) / 8;
    hipLaunchKernelGGL(k_adj_rows<Side>, dim3(g.ny), dim3(bx), shx, s, g, lE, Z, sx);
    hipLaunchKernelGGL(k_adj_cols<Side>, dim3(8 * per), dim3(by), shy, s, g, Z, H, sy, per, c);
    hipLaunchKernelGGL(k_adj_rows_inv<Side>, dim3((g.ny + 1) / 2), dim3(bx), shx, s, g, H, lrho, sx);
    return hipGetLastError();
}

int log2_of(int v) {
    int l = 0;
    while ((1 << l) < v) ++l;
    return l;
}

}  // namespace

hipError_t launch_adj_field(const Geo &g, bool pow2, double *lE, void *Z, void *H, double *lrho, const double *tw,
                            const DftPlan &p, const CtxDev &c, hipStream_t s) {
    const double2 *t = (const double2 *)tw;
    if (pow2) {
        const int lx = log2_of(g.nx), ly = log2_of(g.ny), lm = std::max(lx, ly);
        return launch(g, lE, (double2 *)Z, (double2 *)H, lrho, Pow2Side{g.nx, lx, lm, t}, Pow2Side{g.ny, ly, lm, t},
                      kBlock, kBlock, c, s);
    }
    return launch(g, lE, (double2 *)Z, (double2 *)H, lrho, DftSide{p.x, t}, DftSide{p.y, t + g.nx},
                  dft_threads(g.nx), dft_threads(g.ny), c, s);
}

}  // namespace apic

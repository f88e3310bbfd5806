// Periodic 2D Poisson solve in three launches on grids whose sides are not both
// powers of two: the launches of the power-of-two solve (charge -> half spectra
// of the rows; per column the transform along y, phi_hat, its inverse and the
// field's x-spectrum; rows back), with lines of any length up to kDftMax in LDS
// (apic_dftlds.h).
//
// Bound by launch and memory latency on the sides this is for. 300 x 182, FP64, per
// solve: 38.8 us through the library's transforms (seven launches), 19.4 here; the
// step with 1.0M particles 69.7 and 47.0.
#include "apic_dftlds.h"

namespace apic {
namespace {

// One workgroup per pair of rows (the last row of an odd number alone). LDS: two
// buffers and the table, nx complex each. qacc as in the power-of-two solve.
template <bool MIX, bool WALLS>
__global__ void __launch_bounds__(kDftBlock) k_dft_rows(Geo g, typename AccOf<MIX>::T *acc, double scale, double add,
                                                        int clear, double2 *H, const double2 *tw, DftLine fx,
                                                        unsigned long long *qacc) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int nx = g.nx;
    double2 *b0 = (double2 *)smem, *b1 = b0 + nx, *T = b1 + nx;
    const bool two = 2 * (int)blockIdx.x + 1 < g.ny;
    const int64_t r0 = (int64_t)(2 * blockIdx.x) * nx, r1 = two ? r0 + nx : r0;
    const int sd = g.S * g.dim;
    QSum q{0, 0};
    load_roots(T, tw, nx);
    for (int i = threadIdx.x; i < nx; i += blockDim.x) {
        double v0, v1;
        if constexpr (WALLS) {
            // odd extension of the physical rows [0, nxp]: zero on the walls
            const int nxp = g.nxp;
            if (i == 0 || i == nxp) {
                v0 = v1 = 0.0;
            } else {
                const int src = i < nxp ? i : nx - i;
                const double sg = i < nxp ? 1.0 : -1.0;
                v0 = sg * acc_value<MIX>(acc, r0 + src, scale, add);
                v1 = sg * acc_value<MIX>(acc, r1 + src, scale, add);
            }
        } else {
            const typename AccOf<MIX>::T a0 = acc[r0 + i], a1 = acc[r1 + i];
            if constexpr (MIX) {
                if (qacc) {
                    qsum_add(q, (int64_t)a0, sd);
                    if (two) qsum_add(q, (int64_t)a1, sd);
                }
            }
            v0 = acc_to_rho<MIX>(a0, scale, add);
            v1 = acc_to_rho<MIX>(a1, scale, add);
        }
        b0[i] = make_double2(v0, two ? v1 : 0.0);
    }
    if constexpr (MIX) {
        if (qacc) {
            // between walls: the physical nodes 0..nxp, walls included
            if constexpr (WALLS) {
                for (int i = threadIdx.x; i <= g.nxp; i += blockDim.x) {
                    qsum_add(q, (int64_t)acc[r0 + i], sd);
                    if (two) qsum_add(q, (int64_t)acc[r1 + i], sd);
                }
            }
            qsum_flush(q, sd, qacc);
        }
    }
    __syncthreads();
    if (clear) {
        // after every read of the two rows (the walls read mirrored entries)
        for (int i = threadIdx.x; i < nx; i += blockDim.x) {
            acc[r0 + i] = (typename AccOf<MIX>::T)0;
            if (two) acc[r1 + i] = (typename AccOf<MIX>::T)0;
        }
    }
    const double2 *R = dft_line<-1>(b0, b1, T, fx);
    // split: rho_j0_hat(k) = (Z(k) + conj Z(-k)) / 2, rho_j1_hat(k) = (Z(k) - conj Z(-k)) / (2i)
    const int hx = nx / 2 + 1;
    const int64_t h0 = (int64_t)(2 * blockIdx.x) * hx, h1 = h0 + hx;
    for (int k = threadIdx.x; k < hx; k += blockDim.x) {
        const double2 zk = R[k], zm = R[k == 0 ? 0 : nx - k];
        H[h0 + k] = make_double2(0.5 * (zk.x + zm.x), 0.5 * (zk.y - zm.y));
        if (two) H[h1 + k] = make_double2(0.5 * (zk.y + zm.y), -0.5 * (zk.x - zm.x));
    }
}

// One workgroup per column kx of the half spectra, columns of one XCD adjacent
// (per = ceil(hx / 8)); those past the last only write their zero partial. LDS:
// two buffers and the table, ny complex each.
__global__ void __launch_bounds__(kDftBlock) k_dft_cols(Geo g, const double2 *H, double2 *Z, const double2 *tw,
                                                        DftLine fy, int per, CtxDev c) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double sRed[kDftBlock / 64];
    const int nx = g.nx, ny = g.ny, hx = nx / 2 + 1;
    double2 *A = (double2 *)smem, *B = A + ny, *T = B + ny;
    const int kx = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
    double part = 0.0;
    if (kx < hx) {
        load_roots(T, tw, ny);
        for (int y = threadIdx.x; y < ny; y += blockDim.x) A[y] = H[(int64_t)y * hx + kx];
        __syncthreads();
        double2 *R = dft_line<-1>(A, B, T, fy);
        double2 *S = (R == A) ? B : A;
        const double norm = 1.0 / ((double)nx * (double)ny);
        const double kx2 = c.kx2[kx], kax = c.kapx[kx];
        const bool self = kx == 0 || 2 * kx == nx;
        const double wgt = self ? 1.0 : 2.0;
        // phi_hat (scaled by 1/G for the unnormalised inverse) into S
        for (int ky = threadIdx.x; ky < ny; ky += blockDim.x) {
            const double2 r = R[ky];
            if (kx == 0 && ky == 0) *c.rho0 = r.x;
            const double inv = (kx == 0 && ky == 0) ? 0.0 : 1.0 / (kx2 + c.ky2[ky]);
            const double pr = r.x * inv, pi = r.y * inv;
            const double kay = c.kapy[ky];
            part += wgt * (kax * kax + kay * kay) * (pr * pr + pi * pi);
            S[ky] = make_double2(pr * norm, pi * norm);
        }
        __syncthreads();
        // P = inverse_y(phi_hat), the x-spectrum of phi at this kx: Ex~ = -i kappa_x P,
        // Ey~ its centred difference along y; Z of Ex + i Ey at kx and nx - kx
        const double2 *P = dft_line<+1>(S, R, T, fy);
        const double hy = 0.5 * g.inv_dy;
        const int64_t c0 = (int64_t)kx * ny, c1 = (int64_t)(nx - kx) * ny;   // column-major Z
        for (int y = threadIdx.x; y < ny; y += blockDim.x) {
            const double2 p = P[y], pm = P[y == 0 ? ny - 1 : y - 1], pp = P[y == ny - 1 ? 0 : y + 1];
            const double dx_ = (pp.x - pm.x) * hy, dy_ = (pp.y - pm.y) * hy;   // centred difference of P
            if (self) {
                // a self-conjugate column of two real fields: their real parts
                Z[c0 + y] = make_double2(kax * p.y, -dx_);
            } else {
                Z[c0 + y] = make_double2(kax * p.y + dy_, -kax * p.x - dx_);
                Z[c1 + y] = make_double2(kax * p.y - dy_, kax * p.x - dx_);
            }
        }
    }
    const double bs = block_sum(part, sRed);
    if (threadIdx.x == 0) c.part_spec[blockIdx.x] = bs;
}

// One workgroup per row, rows of one XCD adjacent (per = ceil(ny / 8)); the last
// workgroup reduces the diagnostics. LDS as in k_dft_rows.
__global__ void __launch_bounds__(kDftBlock) k_dft_rows_inv(Geo g, const double2 *Z, double *E, float *E32,
                                                            const double2 *tw, DftLine fx, int per, FinArgs f,
                                                            CtxDev c) {
    if (blockIdx.x == gridDim.x - 1) {
        finalize_block(f, c);
        return;
    }
    extern __shared__ __align__(16) unsigned char smem[];
    const int nx = g.nx, ny = g.ny;
    const int64_t G = (int64_t)nx * ny;
    double2 *b0 = (double2 *)smem, *b1 = b0 + nx, *T = b1 + nx;
    const int y = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
    if (y >= ny) return;
    const int64_t row = (int64_t)y * nx;
    load_roots(T, tw, nx);
    for (int i = threadIdx.x; i < nx; i += blockDim.x) b0[i] = Z[(int64_t)i * ny + y];
    __syncthreads();
    const double2 *U = dft_line<+1>(b0, b1, T, fx);
    for (int i = threadIdx.x; i < nx; i += blockDim.x) {
        const double2 e = U[i];
        if (E) {
            E[row + i] = e.x;
            E[G + row + i] = e.y;
        }
        if (E32) {
            E32[row + i] = (float)e.x;
            E32[G + row + i] = (float)e.y;
        }
    }
}

// The factors of n with the least sum of (factor + kPassCost), found by trying
// every divisor as the next factor.
constexpr int kPassCost = 8;   // a pass's barrier and index arithmetic, in terms of a sum

inline int dft_plan(int n, int left, DftLine &f) {
    if (n == 1) {
        f.passes = 0;
        return 0;
    }
    int best = 1 << 30;
    if (left == 0) return best;
    DftLine t{};
    for (int p = 2; p <= n; ++p) {
        if (n % p) continue;
        const int rest = dft_plan(n / p, left - 1, t);
        if (rest + p + kPassCost < best) {
            best = rest + p + kPassCost;
            f.passes = t.passes + 1;
            f.p[0] = p;
            for (int i = 0; i < t.passes; ++i) f.p[i + 1] = t.p[i];
        }
    }
    return best;
}

inline DftLine dft_line_of(int n) {
    DftLine f{};
    dft_plan(n, kDftPasses, f);
    f.n = n;
    return f;
}

}  // namespace

// Where the sums of a line, n times the plan's cost, stay below kLineTerms; beyond,
// the library is faster. Per solve here and through the library, us: 67 x 63 17 and
// 51, 251 x 241 (65000) 48 and 77, 720 x 720 51 and 63, 1000 x 1000 (79000) 77 and
// 81; 633 x 669 (162000) 166 and 174, 662 x 694 (248000) 271 and 126, 509 x 503
// (263000) 161 and 112, 1021 x 1019 (1.05M) 1090 and 225.
constexpr int kLineTerms = 90000;
// With rows of kDftMax points, the library's best length, it is also faster from here on. 1024 x
// 600 72 and 72, 720 75 and 77, 750 78 and 78, 768 80 and 78, 840 89 and 84, 960 91 and
// 84, 1000 89 and 86 (1020 93 and 95); rows of 1000 x 1024 82 and 84.
constexpr int kLongRows = 750;

bool dft_field_supported(int dim, int nx, int ny) {
    if (dim != 2 || nx < 2 || ny < 2 || nx > kDftMax || ny > kDftMax) return false;
    if (nx == kDftMax && ny >= kLongRows) return false;
    DftLine f{};
    return nx * dft_plan(nx, kDftPasses, f) <= kLineTerms && ny * dft_plan(ny, kDftPasses, f) <= kLineTerms;
}

DftPlan dft_plan_of(int nx, int ny, const double *tw) { return DftPlan{dft_line_of(nx), dft_line_of(ny), tw}; }

hipError_t launch_dft_field(const Geo &g, bool mixed_acc, void *acc, double scale, double add, int clear, void *H,
                            void *Z, double *E, float *E32, const DftPlan &p, const FinArgs &f0, const CtxDev &c,
                            hipStream_t s) {
    const DftLine &fx = p.x, &fy = p.y;
    const double2 *twx = (const double2 *)p.tw, *twy = twx + g.nx;
    const size_t sh_rows = 3 * (size_t)g.nx * sizeof(double2), sh_cols = 3 * (size_t)g.ny * sizeof(double2);
    const dim3 rows((g.ny + 1) / 2), bx(dft_threads(g.nx)), by(dft_threads(g.ny));
    auto first = [&](auto kern, auto *a, unsigned long long *qacc) {
        hipLaunchKernelGGL(kern, rows, bx, sh_rows, s, g, a, scale, add, clear, (double2 *)H, twx, fx, qacc);
    };
    if (mixed_acc) {
        auto *a = (unsigned long long *)acc;
        if (g.walls) first(k_dft_rows<true, true>, a, f0.sd ? c.qacc : nullptr);
        else first(k_dft_rows<true, false>, a, f0.sd ? c.qacc : nullptr);
    } else {
        auto *a = (double *)acc;
        if (g.walls) first(k_dft_rows<false, true>, a, nullptr);
        else first(k_dft_rows<false, false>, a, nullptr);
    }
    const int perx = (g.nx / 2 + 1 + 7) / 8, pery = (g.ny + 7) / 8;
    hipLaunchKernelGGL(k_dft_cols, dim3(8 * perx), by, sh_cols, s, g, (const double2 *)H, (double2 *)Z, twy, fy, perx,
                       c);
    FinArgs f = f0;
    f.nspec = 8 * perx;
    hipLaunchKernelGGL(k_dft_rows_inv, dim3(8 * pery + 1), bx, sh_rows, s, g, (const double2 *)Z, E, E32, twx, fx,
                       pery, f, c);
    return hipGetLastError();
}

}  // namespace apic

// Complex transforms of lines of any length in LDS and the choice of their
// passes, shared by the 2D field solve and its adjoint.
//
// A line of n = p1 p2 .. points is transformed in one Stockham pass per factor,
// each output of a pass the plain sum of its p terms: threads take outputs, the
// terms' twiddles come from a table of the n roots of unity in LDS (every one a
// single rounding of the exact value). No factor needs code of its own, a prime
// side is one pass; the factors are the ones with the shortest sums, e.g.
// 300 = 15 * 20. The lines are short, and what the passes spend on longer sums
// they save in barriers.
#pragma once

#include <algorithm>

#include "apic_fftlds.h"

namespace apic {
namespace {

// The length-n transform of a (kernel exp(SIGN 2 pi i j k / n)), through the other
// buffer; T[j] = exp(-2 pi i j / n). Returns the buffer that holds the result.
// Y[k][q], k < L, q < n / L = M, at k M + q: the length-L transforms of the
// subsequences a[q + M t]. A pass of radix p takes p of them to one of L p:
// Y'[k][q] = sum_r exp(SIGN 2 pi i r k / (L p)) Y[k mod L][q + M' r], M' = M / p.
// All threads call; ends with a barrier.
template <int SIGN>
__device__ double2 *dft_line(double2 *a, double2 *b, const double2 *T, const DftLine &f) {
    const int n = f.n;
    int L = 1;
    for (int s = 0; s < f.passes; ++s) {
        const int p = f.p[s], M = n / L, M1 = M / p;
        for (int o = threadIdx.x; o < n; o += blockDim.x) {
            const int k = o / M1, q = o - k * M1;
            const double2 *in = a + (k % L) * M + q;
            const int step = o - q;   // k M': the exponent's step, in n-ths of a turn
            int e = 0;
            double re = 0.0, im = 0.0;
#pragma unroll 4
            for (int r = 0; r < p; ++r) {
                const double2 v = in[r * M1], w = T[e];
                const double wy = SIGN < 0 ? w.y : -w.y;
                re = __builtin_fma(v.x, w.x, re);
                re = __builtin_fma(-v.y, wy, re);
                im = __builtin_fma(v.x, wy, im);
                im = __builtin_fma(v.y, w.x, im);
                e += step;
                e = e >= n ? e - n : e;
            }
            b[o] = make_double2(re, im);
        }
        __syncthreads();
        double2 *t = a;
        a = b;
        b = t;
        L *= p;
    }
    return a;
}

__device__ __forceinline__ void load_roots(double2 *T, const double2 *tw, int n) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) T[i] = tw[i];
}

inline int dft_threads(int n) { return std::min(kDftBlock, (n + 63) / 64 * 64); }

}  // namespace
}  // namespace apic

// Counting sort of particles in any order by bucket: stable LSD radix passes
// that move the particles themselves.
//
// A pass orders by the next digit of the bucket index. Every workgroup takes a
// chunk of 512 to 4096 particles (per_of below), ranks them by digit (wave by
// wave, so equal digits keep their order), and writes the chunk through LDS in
// digit order: each digit's particles of a chunk form one run of consecutive places, so that every
// array is read and written in whole lines. Digits are as short as the passes
// allow (two passes of half the bits up to 65536 buckets, else four): shorter
// digits are longer runs (1024 buckets: 32 digits, 64 particles a run of 2048). The
// number of passes is even, so the state returns to the caller's arrays without
// a copy; the input index travels as one more array where the caller wants the
// permutation.
//
// Thermal 2D2V, 512 x 512 cells, 16.8M mixed particles in no order: sorting (key,
// index) pairs and gathering the arrays through the indices took 2350 us, 1455 of
// them the gather (a line read for every word); the passes here move 20 bytes per
// particle twice.
#include <algorithm>
#include <type_traits>

#include "apic_device.h"

namespace apic {
namespace {

constexpr int kScan = 2048;              // tallies per workgroup of the scan
constexpr int kMaxDigits = 256;

// Bucket of particle i; one outside the domain (or the box between the walls)
// counts as one of cell 0. ok: whether it is a valid particle (CHECK: offsets
// and all).
template <bool MIX, int DIM, int VDIM, bool CHECK = false>
__device__ __forceinline__ int key_of(const Geo &g, const Parts &p, int64_t i, bool &ok) {
    Pt<MIX> q;
    if constexpr (MIX) {
        unpack_cell<DIM>(p.cell[i], q.ix, q.iy, q.iz);
        ok = (unsigned)q.ix < (unsigned)g.nx;
        if constexpr (DIM >= 2) ok = ok && (unsigned)q.iy < (unsigned)g.ny;
        if constexpr (DIM == 3) ok = ok && (unsigned)q.iz < (unsigned)g.nz;
        if (!ok) q.ix = q.iy = q.iz = 0;
        if constexpr (CHECK) {
            const float fx = p.ox[i], fy = (DIM >= 2) ? p.oy[i] : 0.0f, fz = (DIM == 3) ? p.oz[i] : 0.0f;
            ok = ok && fx >= 0.0f && fx < 1.0f && fy >= 0.0f && fy < 1.0f && fz >= 0.0f && fz < 1.0f;
        }
    } else {
        double f;
        q.iy = q.iz = 0;
        ok = cell_f64(p.x[i], g.inv_dx, g.nx, q.ix, f);
        if constexpr (DIM >= 2) ok = cell_f64(p.y[i], g.inv_dy, g.ny, q.iy, f) && ok;
        if constexpr (DIM == 3) ok = cell_f64(p.z[i], g.inv_dz, g.nz, q.iz, f) && ok;
        if (!ok) q.ix = q.iy = q.iz = 0;
    }
    if (g.walls && q.ix >= g.nxp) {
        ok = false;
        q.ix = 0;
    }
    return bucket_of<MIX, DIM>(g, q.ix, q.iy, q.iz);
}

// Digit tallies of every chunk, digit-major: cnt[d * chunks + chunk]. CHECK (the
// first pass): invalid particles are reported.
// PER particles per thread: a chunk is kBlock * PER.
template <bool MIX, int DIM, int VDIM, int PER, bool CHECK>
__global__ void __launch_bounds__(kBlock) k_sort_count(Geo g, Parts p, int64_t n, int shift, int bits, int32_t *cnt,
                                                       CtxDev c) {
    __shared__ int32_t s[kMaxDigits];
    const int nd = 1 << bits;
    for (int d = threadIdx.x; d < nd; d += kBlock) s[d] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * (kBlock * PER) + threadIdx.x;
    bool good = true;
    for (int j = 0; j < PER; ++j) {
        const int64_t i = base + j * kBlock;
        if (i < n) {
            bool ok;
            const int key = key_of<MIX, DIM, VDIM, CHECK>(g, p, i, ok);
            good = good && ok;
            atomicAdd(&s[(key >> shift) & (nd - 1)], 1);
        }
    }
    if (CHECK && !good) raise_err(c.err, ERR_DOMAIN);
    __syncthreads();
    for (int d = threadIdx.x; d < nd; d += kBlock) cnt[(int64_t)d * gridDim.x + blockIdx.x] = s[d];
}

// Exclusive prefix of one value per thread over the workgroup, and the total.
__device__ __forceinline__ int block_prefix(int v, int &total, int32_t *sh /* [kWaves] */) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int inc = v;
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(inc, o);
        if (lane >= o) inc += y;
    }
    __syncthreads();
    if (lane == 63) sh[w] = inc;
    __syncthreads();
    int pre = 0;
    total = 0;
    for (int i = 0; i < kWaves; ++i) {
        pre += i < w ? sh[i] : 0;
        total += sh[i];
    }
    return pre + inc - v;
}

// The tallies become exclusive sums inside each group of kScan, and the groups'
// totals go to part (a single group: zero, the sum of those before it).
__global__ void __launch_bounds__(kBlock) k_sort_scan(int32_t *cnt, int64_t m, int32_t *part) {
    __shared__ int32_t sh[kWaves];
    constexpr int P = kScan / kBlock;
    const int64_t base = (int64_t)blockIdx.x * kScan + threadIdx.x * P;
    int v[P], s = 0;
#pragma unroll
    for (int j = 0; j < P; ++j) {
        v[j] = base + j < m ? cnt[base + j] : 0;
        s += v[j];
    }
    int total;
    int run = block_prefix(s, total, sh);
#pragma unroll
    for (int j = 0; j < P; ++j) {
        if (base + j < m) cnt[base + j] = run;
        run += v[j];
    }
    if (threadIdx.x == 0) part[blockIdx.x] = gridDim.x == 1 ? 0 : total;
}

// Exclusive sums of the groups' totals (one workgroup).
__global__ void __launch_bounds__(kBlock) k_sort_base(int32_t *part, int groups) {
    __shared__ int32_t sh[kWaves];
    int carry = 0;
    for (int b = 0; b < groups; b += kBlock) {
        const int i = b + (int)threadIdx.x;
        const int v = i < groups ? part[i] : 0;
        int total;
        const int pre = block_prefix(v, total, sh);
        if (i < groups) part[i] = carry + pre;
        carry += total;
    }
}

// One array of the chunk to its places: through LDS into digit order, then in
// runs. pos: this thread's places inside the chunk, dst: the global place of
// chunk position j * kBlock + thread.
template <int PER, typename T>
__device__ __forceinline__ void move_array(const T *in, T *out, T *s, int64_t i0, int64_t n, int m, const int *pos,
                                           const int32_t *dst) {
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    T v[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int k = w * 64 * PER + j * 64 + lane;
        v[j] = in[min(i0 + k, n - 1)];
    }
    __syncthreads();   // the previous array has left LDS
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if (pos[j] >= 0) s[pos[j]] = v[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int k = j * kBlock + threadIdx.x;
        if (k < m) out[dst[j]] = s[k];
    }
}

// idx_in NULL with idx_out set: the input index starts here.
template <bool MIX, int DIM, int VDIM, int PER>
__global__ void __launch_bounds__(kBlock) k_sort_move(Geo g, Parts in, Parts out, int64_t n, int shift, int bits,
                                                      const int32_t *cnt, const int32_t *part, const int32_t *idx_in,
                                                      int32_t *idx_out, CtxDev c) {
    using R = typename Pt<MIX>::R;
    extern __shared__ __align__(16) unsigned char smem[];   // one array of the chunk
    __shared__ int32_t sRun[kWaves][kMaxDigits];            // next place of each (wave, digit)
    __shared__ int32_t sGlob[kMaxDigits];                   // global place of a digit's run less its place in the chunk
    __shared__ uint8_t sDig[kBlock * PER];                  // digit of each chunk position
    __shared__ int32_t sh[kWaves];
    const int nd = 1 << bits, w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t i0 = (int64_t)blockIdx.x * (kBlock * PER);
    const int m = (int)min((int64_t)(kBlock * PER), n - i0);
    for (int d = threadIdx.x; d < kWaves * kMaxDigits; d += kBlock) (&sRun[0][0])[d] = 0;
    __syncthreads();
    // wave w owns the consecutive particles [w, w + 1) * 64 * PER of the chunk; ranks inside (wave, digit)
    const uint64_t lt = lanemask_lt();
    int pos[PER], dig[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int k = w * 64 * PER + j * 64 + lane;
        const bool act = k < m;
        bool ok;
        const int key = key_of<MIX, DIM, VDIM>(g, in, min(i0 + k, n - 1), ok);
        dig[j] = (key >> shift) & (nd - 1);
        uint64_t peers = __ballot(act);
        for (int bit = 0; bit < bits; ++bit) {
            const uint64_t bb = __ballot(act && ((dig[j] >> bit) & 1));
            peers &= ((dig[j] >> bit) & 1) ? bb : ~bb;
        }
        pos[j] = -1;
        if (act) {
            const int before = sRun[w][dig[j]];
            pos[j] = before + (int)__popcll(peers & lt);
            // the group's lowest lane moves the count on (the other lanes have read it: one wave)
            __builtin_amdgcn_wave_barrier();
            if ((peers & lt) == 0) sRun[w][dig[j]] = before + (int)__popcll(peers);
        }
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // places inside the chunk: digit by digit, wave by wave
    {
        const int d = threadIdx.x;
        int t[kWaves], own = 0;
#pragma unroll
        for (int i = 0; i < kWaves; ++i) {
            t[i] = d < nd ? sRun[i][d] : 0;
            own += t[i];
        }
        int total;
        int run = block_prefix(own, total, sh);
        if (d < nd) {
            const int64_t e = (int64_t)d * gridDim.x + blockIdx.x;
            sGlob[d] = cnt[e] + part[e / kScan] - run;
#pragma unroll
            for (int i = 0; i < kWaves; ++i) {
                sRun[i][d] = run;
                run += t[i];
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        if (pos[j] >= 0) {
            pos[j] += sRun[w][dig[j]];
            sDig[pos[j]] = (uint8_t)dig[j];
        }
    }
    __syncthreads();
    int32_t dst[PER];
    bool bad = false;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int k = j * kBlock + (int)threadIdx.x;
        const int64_t to = k < m ? (int64_t)sGlob[sDig[k]] + k : 0;
        bad = bad || to < 0 || to >= n;
        dst[j] = (int32_t)min(max(to, (int64_t)0), n - 1);
    }
    if (bad) raise_err(c.err, ERR_ORDER);
    auto mv = [&](auto *a, auto *b) {
        move_array<PER>(a, b, (std::remove_reference_t<decltype(*b)> *)smem, i0, n, m, pos, dst);
    };
    if constexpr (MIX) {
        mv(in.cell, out.cell);
        mv(in.ox, out.ox);
        if constexpr (DIM >= 2) mv(in.oy, out.oy);
        if constexpr (DIM == 3) mv(in.oz, out.oz);
    } else {
        mv(in.x, out.x);
        if constexpr (DIM >= 2) mv(in.y, out.y);
        if constexpr (DIM == 3) mv(in.z, out.z);
    }
    mv((R *)in.vx, (R *)out.vx);
    if constexpr (VDIM >= 2) mv((R *)in.vy, (R *)out.vy);
    if constexpr (VDIM >= 3) mv((R *)in.vz, (R *)out.vz);
    if (idx_out) {
        if (idx_in) {
            mv(idx_in, idx_out);
        } else {
            int32_t *s = (int32_t *)smem;
            __syncthreads();
#pragma unroll
            for (int j = 0; j < PER; ++j)
                if (pos[j] >= 0) s[pos[j]] = (int32_t)(i0 + w * 64 * PER + j * 64 + lane);
            __syncthreads();
#pragma unroll
            for (int j = 0; j < PER; ++j) {
                const int k = j * kBlock + (int)threadIdx.x;
                if (k < m) idx_out[dst[j]] = s[k];
            }
        }
    }
}

// Bucket table of the sorted particles: start[b] is the first place whose key
// is at least b (start[nb] = n). Place i (0 <= i <= n) writes the entries of
// the buckets in (key[i-1], key[i]], with key[-1] = -1 and key[n] = nb, so each
// entry has exactly one writer.
template <bool MIX, int DIM, int VDIM>
__global__ void __launch_bounds__(kBlock) k_sort_table(Geo g, Parts p, int64_t n, int32_t *start) {
    const int nb = g.nbuckets;
    constexpr int U = 4;   // places per thread, their keys loaded before the first is used
    const int64_t step = (int64_t)gridDim.x * kBlock * U;
    for (int64_t base = (int64_t)blockIdx.x * kBlock * U + threadIdx.x; base <= n + (int)threadIdx.x; base += step) {
        int key[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            bool ok;
            key[u] = n > 0 ? key_of<MIX, DIM, VDIM>(g, p, min(base + u * kBlock, n - 1), ok) : 0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = base + u * kBlock;
            // the key before: the lower lane's, the wave's first lane reads it
            int prev = __shfl_up(key[u], 1);
            if ((threadIdx.x & 63) == 0 && i > 0 && i <= n) {
                bool ok;
                prev = key_of<MIX, DIM, VDIM>(g, p, i - 1, ok);
            }
            if (i > n) continue;
            const int lo = i == 0 ? 0 : prev + 1, hi = i == n ? nb : key[u];
            for (int b = lo; b <= hi; ++b) start[b] = (int32_t)i;
        }
    }
}

// Buckets holding more particles than the fixed-point node sums allow.
__global__ void k_bucket_check(const int32_t *start, int nb, int64_t max_per, CtxDev c) {
    for (int b = blockIdx.x * blockDim.x + threadIdx.x; b < nb; b += gridDim.x * blockDim.x)
        if ((int64_t)start[b + 1] - start[b] > max_per) raise_err(c.err, ERR_OVERFLOW);
}

// Passes, and the bits of each, for nb buckets.
void plan(int nb, int &passes, int &bits) {
    int all = 1;
    while ((int64_t(1) << all) < nb) ++all;
    passes = all <= 16 ? 2 : 4;
    bits = (all + passes - 1) / passes;
}

// Particles per thread of a chunk: few where the sort is short, so that there
// are chunks for the chip, more where the runs of a digit count, and twice as
// many with more than 64 digits. Input in no order / sorted, with 2, 4, 8 and 16
// particles, us: 512 x 512 cells mixed, n = 0.1M (8-bit keys) 33, 36, 49, 79 / 39, 43,
// 57, 87; 1.0M 53, 54, 65, 91 / 60, 63, 72, 99; 4.0M 153, 136, 146, 139 / 140, 137, 158,
// 148; 16.8M 749, 658, 594, 613 / 687, 592, 589, 649; 16-bit keys (2048 x 2048 cells in
// 8 x 8 tiles): 1.0M 109, 83, 75, 97 / 72, 71, 78, 104; 16.8M 1823, 1147, 860, 770 /
// 881, 668, 602, 638.
int per_of(int64_t n, int bits) {
    const int per = n < (int64_t(1) << 19) ? 2 : n < (int64_t(1) << 23) ? 4 : 8;
    return bits > 6 ? 2 * per : per;
}

int64_t chunks_of(int64_t n, int bits) {
    const int64_t chunk = (int64_t)kBlock * per_of(n, bits);
    return std::max<int64_t>((n + chunk - 1) / chunk, 1);
}

}  // namespace

#define APIC_SORT_DISPATCH(g, mixed, ...)                                        \
    do {                                                                        \
        if ((g).dim == 3) APIC_DISPATCH_MIX(mixed, false, 3, 3, __VA_ARGS__);   \
        else APIC_DISPATCH_2D(g, mixed, __VA_ARGS__);                           \
    } while (0)

int64_t sort_tallies(int64_t n, int nb) {
    int passes, bits;
    plan(nb, passes, bits);
    return chunks_of(n, bits) << bits;
}

int64_t sort_groups(int64_t n, int nb) { return (sort_tallies(n, nb) + kScan - 1) / kScan; }

hipError_t launch_sort(const Geo &g, bool mixed, const Parts &p, const Parts &tmp, int64_t n, int32_t *perm,
                       int32_t *idx, int32_t *cnt, int32_t *part, int32_t *start, int64_t max_per_bucket,
                       const CtxDev &c, hipStream_t s) {
    int passes, bits;
    plan(g.nbuckets, passes, bits);
    const int chunks = (int)chunks_of(n, bits);
    const int64_t m = (int64_t)chunks << bits;
    const int groups = (int)((m + kScan - 1) / kScan);
    auto pass = [&](auto per, int k) {
        constexpr int PER = decltype(per)::value;
        const size_t sh = (size_t)kBlock * PER * (mixed ? 4 : 8);
        const Parts &in = k & 1 ? tmp : p, &out = k & 1 ? p : tmp;
        const int32_t *iin = k == 0 ? nullptr : k & 1 ? idx : perm;
        int32_t *iout = !perm ? nullptr : k & 1 ? perm : idx;
        APIC_SORT_DISPATCH(g, mixed, {
            if (k == 0)
                hipLaunchKernelGGL((k_sort_count<MIX, DIM, VDIM, PER, true>), dim3(chunks), dim3(kBlock), 0, s, g, in,
                                   n, 0, bits, cnt, c);
            else
                hipLaunchKernelGGL((k_sort_count<MIX, DIM, VDIM, PER, false>), dim3(chunks), dim3(kBlock), 0, s, g, in,
                                   n, k * bits, bits, cnt, c);
            hipLaunchKernelGGL(k_sort_scan, dim3(groups), dim3(kBlock), 0, s, cnt, m, part);
            if (groups > 1) hipLaunchKernelGGL(k_sort_base, dim3(1), dim3(kBlock), 0, s, part, groups);
            hipLaunchKernelGGL((k_sort_move<MIX, DIM, VDIM, PER>), dim3(chunks), dim3(kBlock), sh, s, g, in, out, n,
                               k * bits, bits, cnt, part, iin, iout, c);
        });
    };
    for (int k = 0; k < passes && n > 0; ++k) {
        switch (per_of(n, bits)) {
        case 2: pass(std::integral_constant<int, 2>{}, k); break;
        case 4: pass(std::integral_constant<int, 4>{}, k); break;
        case 8: pass(std::integral_constant<int, 8>{}, k); break;
        default: pass(std::integral_constant<int, 16>{}, k);
        }
    }
    APIC_SORT_DISPATCH(g, mixed,
                       hipLaunchKernelGGL((k_sort_table<MIX, DIM, VDIM>),
                                          dim3((int)std::min<int64_t>(n / (4 * kBlock) + 1, 4096)), dim3(kBlock), 0, s,
                                          g, p, n, start));
    hipLaunchKernelGGL(k_bucket_check, dim3(std::min((g.nbuckets + kBlock - 1) / kBlock, 4096)), dim3(kBlock), 0, s,
                       start, g.nbuckets, max_per_bucket, c);
    return hipGetLastError();
}

}  // namespace apic

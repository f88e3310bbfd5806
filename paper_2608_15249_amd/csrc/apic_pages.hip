// The step with the particles kept in place: calls of several steps.
//
// A step that writes every particle to its slot of the next bucket order
// (apic_kernels.hip) streams the state through write runs that start mid-line,
// ranks every particle against its workgroup, and reads part of the state
// twice (the tallies must be known before the slots). Between two steps of a
// call nobody sees the order, and only the particles that leave their tile
// (0.3 to 3% per step at the tiles in use) have to move. Here a bucket's particles
// live in pages of kPage slots of a pool; the push reads a page, advances it
// and writes it back to the same addresses, and only the leavers are copied
// out and dealt to their new buckets:
//
//   k_page_push  per bucket: first the exchange of the step before (arrivals
//                from the neighbours' outboxes fill the bucket's holes, further
//                ones are appended with pages from a queue of free ones, holes
//                left over are filled from the bucket's end and pages given
//                back); then gather, advance, move, deposit, the whole state
//                written back in place, the leavers copied to the bucket's part
//                of an outbox and listed by direction, their slots as holes
//
// A call starts with k_page_scan and k_page_fill (bucket counts, page table),
// its first push reads the caller's arrays and writes the pages, and it ends
// with k_page_end, which copies the pages back to the caller's arrays in
// bucket order. The order inside a bucket is a function of the order at the
// call's start alone: leavers are listed in wave, chunk, lane order, arrivals
// are dealt in direction order; only far arrivals take slots in the order in which
// they joined their chains, and which page a bucket gets from the queue decides no
// result.
//
// Magnetized 2D3V, 1024 x 1024 cells, 33.5M mixed particles, 32 x 16 tiles: the
// reordering step's count, scan and push took 16 + 6 + 418 us, the push with its
// exchange 364 us (1.61 GB of state read and written: 4.4 TB/s, where a copy of
// 1 GB on the same card runs at 5.07 TB/s; the same push with the arithmetic left out,
// in a copy of this file that is not kept, took 331 us).
#include <algorithm>
#include <type_traits>

#include "apic_index.h"
#include "apic_pages.h"
#include "apic_step.h"

namespace apic {

namespace {

constexpr int kPageScanMax = 4096;   // buckets up to which the exchange scans the counts itself

// ---- page table of a call ------------------------------------------------------
// Exclusive scans of the bucket counts (ds: first outbox entry and dense slot
// of a bucket, ds[nb] the total) and of their pages (ps). BEGIN: the counts are
// those of the caller's bucket table; a table that is not one (overlapping or
// falling ranges) is reported, and with more entries than particles the call
// runs on empty buckets, in bounds.
template <bool BEGIN>
__global__ void __launch_bounds__(1024) k_page_scan(int nb, int64_t n, int walls, int64_t max_per,
                                                    const int32_t *bstart, int32_t *cnt, int32_t *ds, int32_t *ps,
                                                    CtxDev c) {
    __shared__ int64_t sD[17], sP[17];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    int64_t d0 = 0, p0 = 0;
    bool over = false;
    for (int base = 0; base < nb; base += blockDim.x) {
        const int b = base + (int)threadIdx.x;
        int v = 0;
        if (b < nb) {
            if constexpr (BEGIN) {
                const int64_t lo = min(max((int64_t)bstart[b], (int64_t)0), n);
                const int64_t hi = min(max((int64_t)bstart[b + 1], lo), n);
                v = (int)(hi - lo);
                cnt[b] = v;
            } else {
                v = cnt[b];
            }
        }
        over = over || v > max_per;
        int64_t di = v, pi = (v + kPage - 1) / kPage;
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t y = __shfl_up(di, o), z = __shfl_up(pi, o);
            if (lane >= o) {
                di += y;
                pi += z;
            }
        }
        if (lane == 63) {
            sD[w] = di;
            sP[w] = pi;
        }
        __syncthreads();
        int64_t dw = 0, pw = 0, dt = 0, pt = 0;
        for (int i = 0; i < nw; ++i) {
            if (i < w) {
                dw += sD[i];
                pw += sP[i];
            }
            dt += sD[i];
            pt += sP[i];
        }
        if (b < nb) {
            ds[b] = (int32_t)(d0 + dw + di - v);
            ps[b] = (int32_t)(p0 + pw + pi - (v + kPage - 1) / kPage);
        }
        d0 += dt;
        p0 += pt;
        __syncthreads();
    }
    if (over) raise_err(c.err, ERR_OVERFLOW);
    const bool bad = d0 > n;
    if (bad) {
        for (int b = threadIdx.x; b < nb; b += blockDim.x) {
            cnt[b] = 0;
            ds[b] = 0;
            ps[b] = 0;
        }
    }
    if (threadIdx.x == 0) {
        ds[nb] = bad ? 0 : (int32_t)d0;
        ps[nb] = bad ? 0 : (int32_t)p0;
        if (walls ? d0 > n : d0 != n) raise_err(c.err, ERR_COUNT);
        if (BEGIN) *c.step = -1;
    }
}

// The pages in use are the first ps[nb] of the pool, in table order; the
// others wait in the queue. Clears what the first push adds to.
__global__ void __launch_bounds__(kBlock) k_page_fill(int nb, PageStep t, int32_t *cnt3, int32_t *head2,
                                                      uint64_t *acc, int64_t nacc) {
    const int64_t i0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, st = (int64_t)gridDim.x * blockDim.x;
    const int used = t.ps[nb];
    for (int64_t i = i0; i < t.npages; i += st) {
        if (i < used) t.tab[i] = (int32_t)i;
        if (i < t.npages - used) t.queue[i] = used + (int32_t)i;
    }
    for (int64_t i = i0; i < nacc; i += st) acc[i] = 0;
    for (int64_t i = i0; i < 2 * (int64_t)nb; i += st) cnt3[nb + i] = 0;   // the counts of the call's start come first
    for (int64_t i = i0; i < 2 * (int64_t)nb * kFarChains; i += st) head2[i] = 0;
    if (i0 == 0) {
        t.head[0] = 0;
        t.head[1] = (unsigned long long)(t.npages - used);
        *t.live = t.ds[nb];
        *t.done = 0;
    }
}

// ---- pages ------------------------------------------------------------------------
// A particle's record: the words of its state in a fixed order (cell, offsets,
// velocities; FP64: position, velocities), kept in pieces of 16, 8 or 4 bytes
// (FP64: 16 or 8), each piece an array of its own over the page's slots. A wave
// reads and writes whole lines of every piece, a leaver or an arrival touches
// two or three places and not one per component (thermal 3D, 128^3, 16.8M mixed:
// the exchange took 85 us with one array per component).
template <typename T, int U> using Vec = T __attribute__((ext_vector_type(U)));

template <bool MIX, int DIM, int VDIM> struct Rec {
    using T = std::conditional_t<MIX, int32_t, double>;
    static constexpr int K = (MIX ? 1 : 0) + DIM + VDIM;   // words
    static constexpr int64_t kPageBytes = (int64_t)K * kPage * sizeof(T);
};

// Words OFF .. of the piece that starts there.
template <typename T, int K, int OFF>
constexpr int piece() { return (sizeof(T) == 4 && K - OFF >= 4) ? 4 : (K - OFF >= 2) ? 2 : 1; }

// NT: the nontemporal hint, for whole pages, each read and written once per step.
template <bool NT, typename T, int K, int OFF = 0>
__device__ __forceinline__ void load_words(const char *base, int64_t slots, unsigned i, T *w) {
    constexpr int N = piece<T, K, OFF>();
    const Vec<T, N> *p = (const Vec<T, N> *)(base + OFF * (int64_t)sizeof(T) * slots) + i;
    Vec<T, N> v;
    if constexpr (NT) v = __builtin_nontemporal_load(p);
    else v = *p;
#pragma unroll
    for (int j = 0; j < N; ++j) w[OFF + j] = v[j];
    if constexpr (OFF + N < K) load_words<NT, T, K, OFF + N>(base, slots, i, w);
}
template <bool NT, typename T, int K, int OFF = 0>
__device__ __forceinline__ void store_words(char *base, int64_t slots, unsigned i, const T *w) {
    constexpr int N = piece<T, K, OFF>();
    Vec<T, N> *p = (Vec<T, N> *)(base + OFF * (int64_t)sizeof(T) * slots) + i;
    Vec<T, N> v;
#pragma unroll
    for (int j = 0; j < N; ++j) v[j] = w[OFF + j];
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
    if constexpr (OFF + N < K) store_words<NT, T, K, OFF + N>(base, slots, i, w);
}

template <bool MIX, int DIM, int VDIM>
__device__ __forceinline__ void to_words(const Raw<MIX> &r, typename Rec<MIX, DIM, VDIM>::T *w) {
    int k = 0;
    if constexpr (MIX) {
        w[k++] = r.c;
        w[k++] = __float_as_int(r.ox);
        if constexpr (DIM >= 2) w[k++] = __float_as_int(r.oy);
        if constexpr (DIM == 3) w[k++] = __float_as_int(r.oz);
        w[k++] = __float_as_int(r.vx);
        if constexpr (VDIM >= 2) w[k++] = __float_as_int(r.vy);
        if constexpr (VDIM >= 3) w[k++] = __float_as_int(r.vz);
    } else {
        w[k++] = r.x;
        if constexpr (DIM >= 2) w[k++] = r.y;
        if constexpr (DIM == 3) w[k++] = r.z;
        w[k++] = r.vx;
        if constexpr (VDIM >= 2) w[k++] = r.vy;
        if constexpr (VDIM >= 3) w[k++] = r.vz;
    }
}
template <bool MIX, int DIM, int VDIM>
__device__ __forceinline__ void from_words(const typename Rec<MIX, DIM, VDIM>::T *w, Raw<MIX> &r) {
    int k = 0;
    r = Raw<MIX>{};
    if constexpr (MIX) {
        r.c = w[k++];
        r.ox = __int_as_float(w[k++]);
        if constexpr (DIM >= 2) r.oy = __int_as_float(w[k++]);
        if constexpr (DIM == 3) r.oz = __int_as_float(w[k++]);
        r.vx = __int_as_float(w[k++]);
        if constexpr (VDIM >= 2) r.vy = __int_as_float(w[k++]);
        if constexpr (VDIM >= 3) r.vz = __int_as_float(w[k++]);
    } else {
        r.x = w[k++];
        if constexpr (DIM >= 2) r.y = w[k++];
        if constexpr (DIM == 3) r.z = w[k++];
        r.vx = w[k++];
        if constexpr (VDIM >= 2) r.vy = w[k++];
        if constexpr (VDIM >= 3) r.vz = w[k++];
    }
}

template <bool MIX, int DIM, int VDIM>
__device__ __forceinline__ char *page_at(const PageStep &t, int page) {
    return t.pool + page * Rec<MIX, DIM, VDIM>::kPageBytes;
}

// Slot i of a page.
template <bool MIX, int DIM, int VDIM, bool NT = true>
__device__ __forceinline__ void load_slot(const char *page, unsigned i, Raw<MIX> &r) {
    using T = typename Rec<MIX, DIM, VDIM>::T;
    T w[Rec<MIX, DIM, VDIM>::K];
    load_words<NT, T, Rec<MIX, DIM, VDIM>::K>(page, kPage, i, w);
    from_words<MIX, DIM, VDIM>(w, r);
}
template <bool MIX, int DIM, int VDIM, bool NT = true>
__device__ __forceinline__ void store_slot(char *page, unsigned i, const Raw<MIX> &r) {
    using T = typename Rec<MIX, DIM, VDIM>::T;
    T w[Rec<MIX, DIM, VDIM>::K];
    to_words<MIX, DIM, VDIM>(r, w);
    store_words<NT, T, Rec<MIX, DIM, VDIM>::K>(page, kPage, i, w);
}

// Slot s of a bucket whose page ids are tab.
template <bool MIX, int DIM, int VDIM>
__device__ __forceinline__ Raw<MIX> read_raw(const PageStep &t, const int32_t *tab, int s) {
    Raw<MIX> r;
    load_slot<MIX, DIM, VDIM, false>(page_at<MIX, DIM, VDIM>(t, tab[s / kPage]), s % kPage, r);
    return r;
}
template <bool MIX, int DIM, int VDIM>
__device__ __forceinline__ void write_raw(const PageStep &t, const int32_t *tab, int s, const Raw<MIX> &r) {
    store_slot<MIX, DIM, VDIM, false>(page_at<MIX, DIM, VDIM>(t, tab[s / kPage]), s % kPage, r);
}

// Entry e of the outbox, in the same pieces.
template <bool MIX, int DIM, int VDIM>
__device__ __forceinline__ void out_put(const PageStep &t, int e, const Raw<MIX> &r) {
    using T = typename Rec<MIX, DIM, VDIM>::T;
    T w[Rec<MIX, DIM, VDIM>::K];
    to_words<MIX, DIM, VDIM>(r, w);
    store_words<false, T, Rec<MIX, DIM, VDIM>::K>(t.to.out, t.out_slots, e, w);
}
template <bool MIX, int DIM, int VDIM>
__device__ __forceinline__ Raw<MIX> out_get(const PageStep &t, int e) {
    using T = typename Rec<MIX, DIM, VDIM>::T;
    T w[Rec<MIX, DIM, VDIM>::K];
    load_words<false, T, Rec<MIX, DIM, VDIM>::K>(t.in.out, t.out_slots, e, w);
    Raw<MIX> r;
    from_words<MIX, DIM, VDIM>(w, r);
    return r;
}

// One particle from the caller's arrays (through the caches: a bucket starts
// mid-line, and neighbouring waves share lines).
template <bool MIX, int DIM, int VDIM>
__device__ __forceinline__ void read_array(const Parts &s, int i, Raw<MIX> &r) {
    r = Raw<MIX>{};
    if constexpr (MIX) {
        r.c = s.cell[i];
        r.ox = s.ox[i];
        if constexpr (DIM >= 2) r.oy = s.oy[i];
        if constexpr (DIM == 3) r.oz = s.oz[i];
        r.vx = ((const float *)s.vx)[i];
        if constexpr (VDIM >= 2) r.vy = ((const float *)s.vy)[i];
        if constexpr (VDIM >= 3) r.vz = ((const float *)s.vz)[i];
    } else {
        r.x = s.x[i];
        if constexpr (DIM >= 2) r.y = s.y[i];
        if constexpr (DIM == 3) r.z = s.z[i];
        r.vx = ((const double *)s.vx)[i];
        if constexpr (VDIM >= 2) r.vy = ((const double *)s.vy)[i];
        if constexpr (VDIM >= 3) r.vz = ((const double *)s.vz)[i];
    }
}

// One particle to the caller's arrays.
template <bool MIX, int DIM, int VDIM>
__device__ __forceinline__ void store_raw(const Parts &s, int i, const Raw<MIX> &r) {
    if constexpr (MIX) {
        s.cell[i] = r.c;
        s.ox[i] = r.ox;
        if constexpr (DIM >= 2) s.oy[i] = r.oy;
        if constexpr (DIM == 3) s.oz[i] = r.oz;
        ((float *)s.vx)[i] = r.vx;
        if constexpr (VDIM >= 2) ((float *)s.vy)[i] = r.vy;
        if constexpr (VDIM >= 3) ((float *)s.vz)[i] = r.vz;
    } else {
        s.x[i] = r.x;
        if constexpr (DIM >= 2) s.y[i] = r.y;
        if constexpr (DIM == 3) s.z[i] = r.z;
        ((double *)s.vx)[i] = r.vx;
        if constexpr (VDIM >= 2) ((double *)s.vy)[i] = r.vy;
        if constexpr (VDIM >= 3) ((double *)s.vz)[i] = r.vz;
    }
}

template <bool MIX, int DIM>
__device__ __forceinline__ void encode(const Pt<MIX> &q, Raw<MIX> &r) {
    if constexpr (MIX) {
        r.c = pack_cell<DIM>(q.ix, q.iy, q.iz);
        r.ox = q.fx;
        if constexpr (DIM >= 2) r.oy = q.fy;
        if constexpr (DIM == 3) r.oz = q.fz;
    } else {
        r.x = q.x;
        if constexpr (DIM >= 2) r.y = q.y;
        if constexpr (DIM == 3) r.z = q.z;
    }
    r.vx = q.vx;
    r.vy = q.vy;
    r.vz = q.vz;
}

__device__ __forceinline__ int pages_of(int count) { return (count + kPage - 1) / kPage; }

// Exclusive rank of the threads with `on` in thread order over the workgroup,
// and their number; sh: one word per wave.
__device__ __forceinline__ int block_rank(bool on, int &total, int32_t *sh) {
    const uint64_t m = __ballot(on);
    const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    __syncthreads();   // the words of the previous call have been read
    if ((threadIdx.x & 63) == 0) sh[w] = (int)__popcll(m);
    __syncthreads();
    int pre = 0;
    total = 0;
    for (int i = 0; i < nw; ++i) {
        pre += i < w ? sh[i] : 0;
        total += sh[i];
    }
    return pre + (int)__popcll(m & lanemask_lt());
}

// ---- a group of particles without branches ----------------------------------------
// Particles in the pages are this library's own output: inside their bucket's
// tile, offsets in range. The loop below therefore checks nothing on the way
// in, computes a group of particles in straight-line code (so that their LDS
// reads and dependent chains overlap) and leaves what is rare (a non-finite
// move, a particle that leaves the tile) to one branch per group. Same
// arithmetic and bits as decode(), advance() and move_pt().
template <typename R>
__device__ __forceinline__ void boris_rot(R &vx, R &vy, R ex, R ey, R a, R t, R s) {
    const R mx = vx + a * ex, my = vy + a * ey;
    const R px = mx + my * t, py = my - mx * t;
    const R qx = mx + py * s, qy = my - px * s;
    vx = qx + a * ex;
    vy = qy + a * ey;
}

// One axis of the move, the cell left unwrapped: shift in cells, false when
// the general form is needed (non-finite or runaway; FP64: more than a box).
__device__ __forceinline__ bool move_axis_fast(float &f, float v, float dtd, int &shift) {
    float o = f + v * dtd;
    const float fl = floorf(o);
    o = o - fl;
    const bool up = o >= 1.0f;
    f = up ? o - 1.0f : o;
    shift = (int)fl + (up ? 1 : 0);
    return fabsf(fl) < 1.0e8f;
}
__device__ __forceinline__ bool move_axis_fast(double &xc, int ic, double &f, double v, double dt, double L,
                                               double inv_d, int n, int &shift) {
    double x = xc + v * dt;
    x = x < 0.0 ? x + L : x;
    x = x >= L ? x - L : x;
    xc = x;
    const double gx = x * inv_d, fl = floor(gx);
    f = gx - fl;
    int i = (int)fl;
    i = i >= n ? i - n : i;
    int d = i - ic;
    d = d > n / 2 ? d - n : d;
    d = d < -(n / 2) ? d + n : d;
    shift = d;
    return x >= 0.0 && x < L;
}

template <bool MIX> struct Moved {
    using R = typename Pt<MIX>::R;
    Pt<MIX> q;               // after the move, its cell aside
    int lx, ly, lz;          // tile-local cell after the move, unwrapped
    R v2;                    // |v|^2 (or its relativistic form) before the advance
    bool ok;
};

// Gather, advance and move of particle j = 0 .. N-1 of a full unit.
template <bool MIX, int DIM, int VDIM, bool HC, bool ROT, int N>
__device__ __forceinline__ void advance_group(const Raw<MIX> *r, const Geo &g, const PushC &pc,
                                              const typename Pt<MIX>::R *sE, int ex_w, int ey_w, int ez_w, int x0,
                                              int y0, int z0, Moved<MIX> *m) {
    using R = typename Pt<MIX>::R;
    const int wxy = ex_w * ey_w;
    R ex[N], ey[N], ez[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
        Pt<MIX> &q = m[j].q;
        if constexpr (MIX) {
            unpack_cell<DIM>(r[j].c, q.ix, q.iy, q.iz);
            q.fx = r[j].ox;
            q.fy = (DIM >= 2) ? r[j].oy : 0.0f;
            q.fz = (DIM == 3) ? r[j].oz : 0.0f;
        } else {
            auto cell = [](double x, double inv_d, int n, int &i, double &f) {
                const double gx = x * inv_d, fl = floor(gx);
                f = gx - fl;
                i = (int)fl;
                i = i >= n ? i - n : i;
            };
            q.x = r[j].x;
            cell(q.x, g.inv_dx, g.nx, q.ix, q.fx);
            q.y = q.z = 0.0;
            q.iy = q.iz = 0;
            q.fy = q.fz = 0.0;
            if constexpr (DIM >= 2) {
                q.y = r[j].y;
                cell(q.y, g.inv_dy, g.ny, q.iy, q.fy);
            }
            if constexpr (DIM == 3) {
                q.z = r[j].z;
                cell(q.z, g.inv_dz, g.nz, q.iz, q.fz);
            }
        }
        q.vx = r[j].vx;
        q.vy = r[j].vy;
        q.vz = r[j].vz;
        m[j].lx = q.ix - x0;
        m[j].ly = (DIM >= 2) ? q.iy - y0 : 0;
        m[j].lz = (DIM == 3) ? q.iz - z0 : 0;
        ez[j] = R(0);
        if constexpr (DIM == 3)
            gather_lds3<R>(sE, ex_w, wxy, wxy * ez_w, m[j].lx, m[j].ly, m[j].lz, q.fx, q.fy, q.fz, ex[j], ey[j],
                           ez[j]);
        else
            gather_lds<R, DIM>(sE, ex_w, wxy, m[j].lx, m[j].ly, q.fx, q.fy, ex[j], ey[j]);
    }
    const R a = MIX ? (R)pc.af : (R)pc.a, tt = MIX ? (R)pc.tf : (R)pc.t, ss = MIX ? (R)pc.sf : (R)pc.s;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        Pt<MIX> &q = m[j].q;
        m[j].v2 = (R)vsq<MIX, VDIM, HC>(q, pc);
        R ux, uy, uz;
        if constexpr (HC) {
            const R ic2 = MIX ? (R)pc.ic2f : (R)pc.ic2;
            higuera_cary<R>(q.vx, q.vy, q.vz, ex[j], ey[j], ez[j], a, tt, ic2);
            const R gm = lorentz<R>(q.vx, q.vy, q.vz, ic2);
            if constexpr (MIX) {
                const R ig = R(1) / gm;
                ux = q.vx * ig;
                uy = q.vy * ig;
                uz = q.vz * ig;
            } else {
                ux = q.vx / gm;
                uy = q.vy / gm;
                uz = q.vz / gm;
            }
        } else {
            if constexpr (DIM == 3) boris_z<R>(q.vz, ez[j], a);
            if constexpr (ROT)
                boris_rot<R>(q.vx, q.vy, ex[j], ey[j], a, tt, ss);
            else
                boris<R, VDIM>(q.vx, q.vy, ex[j], ey[j], a, R(0), R(0));
            ux = q.vx;
            uy = q.vy;
            uz = q.vz;
        }
        int sx, sy = 0, sz = 0;
        bool ok;
        if constexpr (MIX) {
            ok = move_axis_fast(q.fx, ux, pc.dtdx, sx);
            if constexpr (DIM >= 2) ok = move_axis_fast(q.fy, uy, pc.dtdy, sy) && ok;
            if constexpr (DIM == 3) ok = move_axis_fast(q.fz, uz, pc.dtdz, sz) && ok;
        } else {
            ok = move_axis_fast(q.x, q.ix, q.fx, ux, pc.dt, g.lx, g.inv_dx, g.nx, sx);
            if constexpr (DIM >= 2) ok = move_axis_fast(q.y, q.iy, q.fy, uy, pc.dt, g.ly, g.inv_dy, g.ny, sy) && ok;
            if constexpr (DIM == 3) ok = move_axis_fast(q.z, q.iz, q.fz, uz, pc.dt, g.lz, g.inv_dz, g.nz, sz) && ok;
        }
        m[j].lx += sx;
        m[j].ly += sy;
        m[j].lz += sz;
        m[j].ok = ok;
    }
}

// ---- exchange --------------------------------------------------------------------
// What a bucket's workgroup does before it touches the bucket's pages: the
// leavers of the step before come in from the neighbours' lists. The new counts
// are complete (the push added every stay and every leaver to its bucket), so
// each workgroup sums those of the buckets before its own (a few KiB, cache
// resident) for the bucket's list and page-table entries; with more than
// kPageScanMax buckets k_page_scan has done it (t.scanned). Arrival i takes hole i while
// there are holes, then slot old + i - holes; a bucket that shrinks closes its
// remaining holes with the particles beyond its new end.
struct ExchangeLds {
    static constexpr int kBits = 8192;   // slots per bitmap round of a shrinking bucket
    int64_t d[kPagePushMax / 64];
    unsigned long long q;
    int32_t p[kPagePushMax / 64], rank[kPagePushMax / 64];
    int32_t in[kStepTab + 1], src[kStepTab];   // arrivals before direction d, its first list entry
    int32_t left;
    uint32_t map[kBits / 32];
};

template <bool MIX, int DIM, int VDIM>
__device__ void exchange_bucket(const Geo &g, const PageStep &t, int b, int64_t n, int64_t max_per, const CtxDev &c,
                                ExchangeLds &sh) {
    constexpr int kFar = Dir<DIM>::kFar, kStay = Dir<DIM>::kStay, kTab = Dir<DIM>::kTab;
    const int nb = g.nbuckets;
    const int lane = (int)(threadIdx.x & 63), w = (int)(threadIdx.x >> 6), nw = (int)(blockDim.x >> 6);
    const int old = t.cnt_old[b], dsb = t.ds_old[b], psb = t.ps_old[b];
    const int now = t.cnt[b];
    // arrivals by direction (one lane each) and the bucket's own leavers
    if (w == 0) {
        int v = 0, o = 0, own = 0;
        if (lane < kTab) {
            own = t.in.cnt[b * kTab + lane];
            if (lane < kFar && lane != kStay) {
                const int from = dir_source<DIM>(g, b, lane);
                v = t.in.cnt[from * kTab + lane];
                o = t.ds_old[from] + t.in.off[from * kTab + lane];
            }
        }
        int inc = v;
        for (int off = 1; off < 64; off <<= 1) {
            const int y = __shfl_up(inc, off);
            if (lane >= off) inc += y;
        }
        for (int off = 32; off > 0; off >>= 1) own += __shfl_xor(own, off);
        if (lane < kTab) {
            sh.in[lane] = inc - v;
            sh.src[lane] = o;
        }
        if (lane == kTab - 1) sh.in[kTab] = inc;
        if (lane == 0) sh.left = own;
    }
    // page table: the bucket's pages, more from the queue or the last ones back to it
    const int np_old = pages_of(old), np_new = pages_of(now);
    if (threadIdx.x == 0) {
        if (np_new > np_old) sh.q = atomicAdd(&t.head[0], (unsigned long long)(np_new - np_old));
        if (np_new < np_old) sh.q = atomicAdd(&t.head[1], (unsigned long long)(np_old - np_new));
    }
    int pn, dn;   // the bucket's first entries now
    if (t.scanned) {
        pn = t.ps[b];
        dn = t.ds[b];
        __syncthreads();
    } else {
        int64_t d = 0;
        int p = 0;
        for (int i = threadIdx.x; i < b; i += blockDim.x) {
            const int v = t.cnt[i];
            d += v;
            p += pages_of(v);
        }
        for (int off = 32; off > 0; off >>= 1) {
            d += __shfl_xor(d, off);
            p += __shfl_xor(p, off);
        }
        if (lane == 0) {
            sh.d[w] = d;
            sh.p[w] = p;
        }
        __syncthreads();
        d = 0;
        pn = 0;
        for (int i = 0; i < nw; ++i) {
            d += sh.d[i];
            pn += sh.p[i];
        }
        dn = (int)d;
        if (threadIdx.x == 0) {
            t.ds[b] = dn;
            t.ps[b] = pn;
            if (now > max_per) raise_err(c.err, ERR_OVERFLOW);
            if (b == nb - 1) {
                const int64_t total = d + now;
                t.ds[nb] = (int32_t)total;
                t.ps[nb] = pn + np_new;
                if (g.walls ? total > n : total != n) raise_err(c.err, ERR_COUNT);
            }
        }
    }
    for (int i = threadIdx.x; i < max(np_old, np_new); i += blockDim.x) {
        if (i < np_old) {
            const int page = t.tab_old[psb + i];
            if (i < np_new)
                t.tab[pn + i] = page;
            else
                t.queue[(sh.q + (i - np_new)) % t.npages] = page;
        } else {
            t.tab[pn + i] = t.queue[(sh.q + (i - np_old)) % t.npages];
        }
    }
    const int near = sh.in[kTab], nout = sh.left;
    const int total_in = now - (old - nout);      // near and far arrivals
    const int32_t *low = t.in.hole + dsb;         // holes that stay inside the bucket
    if (now < old) {
        // a shrinking bucket: the holes below its new end, then the particles
        // beyond it into those that no arrival takes
        int32_t *keep = t.raw_slot + dn;   // (fewer than the bucket will hold)
        int nlow = 0;
        for (int e0 = 0; e0 < nout; e0 += blockDim.x) {
            const int e = e0 + (int)threadIdx.x;
            const int s = e < nout ? t.in.hole[dsb + e] : now;
            int tot;
            const int r = block_rank(s < now, tot, sh.rank);
            if (s < now) keep[nlow + r] = s;
            nlow += tot;
        }
        low = keep;
        int moved = total_in;
        for (int s0 = now; s0 < old; s0 += ExchangeLds::kBits) {
            const int len = min(ExchangeLds::kBits, old - s0);
            __syncthreads();
            for (int i = threadIdx.x; i < (len + 31) / 32; i += blockDim.x) sh.map[i] = 0;
            __syncthreads();
            for (int e = threadIdx.x; e < nout; e += blockDim.x) {
                const int s = t.in.hole[dsb + e] - s0;
                if (s >= 0 && s < len) atomicOr(&sh.map[s >> 5], 1u << (s & 31));
            }
            __syncthreads();
            for (int j0 = 0; j0 < len; j0 += blockDim.x) {
                const int j = j0 + (int)threadIdx.x;
                const bool live = j < len && !((sh.map[j >> 5] >> (j & 31)) & 1u);
                int tot;
                const int r = block_rank(live, tot, sh.rank);
                if (live && moved + r < nlow)
                    write_raw<MIX, DIM, VDIM>(t, t.tab_old + psb, keep[moved + r],
                                              read_raw<MIX, DIM, VDIM>(t, t.tab_old + psb, s0 + j));
                moved += tot;
            }
        }
    }
    __syncthreads();   // the new page table and the kept holes are written
    // arrival i, from an outbox entry
    auto place = [&](int i, int from) {
        const int to = (now < old || i < nout) ? low[i] : old + (i - nout);
        write_raw<MIX, DIM, VDIM>(t, t.tab + pn, to, out_get<MIX, DIM, VDIM>(t, from));
    };
    for (int i = threadIdx.x; i < near; i += blockDim.x) {
        int d = 0;
        for (int e = 1; e < kTab; ++e) d = sh.in[e] <= i ? e : d;
        place(i, t.in.order[sh.src[d] + (i - sh.in[d])]);
    }
    // arrivals from beyond the neighbours (normally none), a chain per lane: the next
    // entries of all chains are on their way while the states of these are moved. The
    // cost is the bucket's own arrivals (every bucket going through one list of all far
    // leavers, behind one counter, took buckets x leavers): 256 x 256 cells in 1024
    // buckets, 4.0M mixed particles, a share of 0, 1 and 10% beyond the neighbours per
    // step: 68.5, 317 and 1404 us per step with the one list, 67.0, 77.9 and 231 with
    // chains (75, 127 and 711 where every step reorders)
    if (total_in > near && w == 0) {
        int32_t *head = t.in.far_head + (int64_t)b * kFarChains + lane;
        int e = *head;
        if (e) *head = 0;
        int done = near;
        for (uint64_t m = __ballot(e != 0); m; m = __ballot(e != 0)) {
            const int at = e - 1, i = done + (int)__popcll(m & lanemask_lt());
            if (e) {
                e = t.in.far_next[at];
                if (i < total_in) place(i, at);
            }
            done += (int)__popcll(m);
        }
    }
    if (threadIdx.x == 0) t.cnt_old[b] = 0;
    __syncthreads();   // the bucket's pages and tables are written
}

// ---- push -----------------------------------------------------------------------
// Waves per SIMD the push is compiled for: in 3D the FP64 state and gather want
// more registers than four leave (its LDS tile allows three anyway; thermal 128^3,
// 16.8M: 584 us per step with spills at four, 556 at three).
template <bool MIX, int DIM> constexpr int push_waves_per_simd() { return (!MIX && DIM == 3) ? 3 : 4; }

// The end of a 1D push: the workgroup that ends last solves the field of the
// charge that all have added and leaves the sums at zero for the next step.
// (What the others wrote and this one reads, the sums, the partials and the step,
// passes through device-scope atomics; each thread waits for its own, the barrier
// for everyone's, before the workgroup is counted. No workgroup waits for
// another.) The solve and its diagnostics were launches
// of their own: 64 nodes, 16384 particles in 4 buckets 27.0 us per step in calls
// of 20, 23.5 with the solve here (FP64 27.0 and 22.9).
template <bool MIX>
__device__ void field_by_last(const Geo &g, const PageStep &t, const PageField &f, typename AccOf<MIX>::T *acc,
                              const double *part, unsigned char *smem, const CtxDev &c) {
    using A = typename AccOf<MIX>::T;
    __shared__ double sRed[kPagePushMax / 64];
    __shared__ int sLast;
    double *sr = (double *)smem, *sScan = sr + g.nx;
    __builtin_amdgcn_s_waitcnt(kWaitVmem);
    __syncthreads();
    if (threadIdx.x == 0) sLast = atomicAdd(t.done, 1) == g.nbuckets - 1;
    __syncthreads();
    if (!sLast) return;
    const int sd = g.S * g.dim;
    double tot = 0.0;
    QSum q{0, 0};
    for (int i = threadIdx.x < kBlock ? threadIdx.x : g.nx; i < g.nx; i += kBlock) {
        double w;
        if constexpr (MIX) {
            const int64_t v = (int64_t)atomicExch(&acc[i], (A)0);
            w = (double)v;
            qsum_add(q, v, sd);
        } else {
            w = __longlong_as_double((long long)atomicExch((unsigned long long *)&acc[i], 0ull));
        }
        const double r = f.ion + f.scale * w;
        sr[i] = r;
        tot += r - f.ion;
    }
    double charge = block_sum(tot, sRed) * f.dx;
    if constexpr (MIX) {
        const QSum qt = qsum_block(q, sd);
        if (threadIdx.x == 0) {
            c.qexact[0] = qt.whole;
            c.qexact[1] = (int64_t)qt.rem;
            charge = qsum_charge(qt, sd, f.q_macro);
        }
    }
    const double wsum = field1d_block(sr, g.nx, f.dx, f.E, f.E32, sRed, sScan);
    if (f.diag) {
        double k = 0.0, p = 0.0;
        for (int i = threadIdx.x; i < g.nbuckets; i += blockDim.x) {
            k += __hip_atomic_load(&part[2 * i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            p += __hip_atomic_load(&part[2 * i + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        k = block_sum(k, sRed);
        p = block_sum(p, sRed);
        if (threadIdx.x == 0) {
            double *d = f.diag + 4 * __hip_atomic_load(c.step, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            d[0] = charge;
            d[1] = 0.5 * wsum * f.dx;
            d[2] = 0.5 * f.mass * k;
            d[3] = f.mass * p;
        }
    }
    if (threadIdx.x == 0) *t.done = 0;
}

// One workgroup per bucket. A unit is one page: wave w takes the pages w, w + nw,
// ... of the bucket, each lane kPage / 64 of a page's slots, and reads and writes
// them in pieces of the record (16, 8 or 4 bytes a lane, whole lines both ways).
// No slot is computed and no barrier stands in the loop; a wave appends the slots
// of its leavers to its own part of the bucket's list. FIRST: the particles come
// from the caller's arrays (bucket b from bstart[b]), one by one, and go to the
// same slots of the pages. NT: the pages are read and written past the caches.
template <bool MIX, int DIM, int VDIM, bool HC, bool EM, bool ROT, bool FIRST, bool NT>
__global__ void __launch_bounds__(kPagePushMax, (push_waves_per_simd<MIX, DIM>())) k_page_push(Geo g, PageStep t, Parts src, const int32_t *bstart,
                                                            int64_t n, int64_t max_per, const double *E, const float *E32, PushC pc,
                                                            typename AccOf<MIX>::T *acc, double *part, PageField f, CtxDev c) {
    static_assert(!EM || (DIM == 2 && VDIM == 3), "the electromagnetic step is 2D3V");
    using R = typename Pt<MIX>::R;
    using A = typename AccOf<MIX>::T;
    constexpr int kFar = Dir<DIM>::kFar, kStay = Dir<DIM>::kStay, kTab = Dir<DIM>::kTab;
    constexpr int U = kPage / 64;   // particles of one lane per page
    constexpr int kMaxW = kPagePushMax / 64;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int sErr;
    __shared__ int32_t sCnt[kTab], sOff[kTab];   // leavers by direction (kStay: absorbed), their first outbox entry
    __shared__ int32_t sList[kMaxW];             // leavers of each wave
    __shared__ int32_t sMv[kMaxW][kTab];
    __shared__ double sKe[kMaxW], sPx[kMaxW];
    const int ex_w = (1 << g.tsx) + 1, ey_w = (DIM >= 2) ? (1 << g.tsy) + 1 : 1;
    const int ez_w = (DIM == 3) ? (1 << g.tsz) + 1 : 1;
    const int wx = (1 << g.tsx) + 1 + 2 * g.halo;
    const int wy = (DIM >= 2) ? (1 << g.tsy) + 1 + 2 * g.halo : 1;
    const int wz = (DIM == 3) ? (1 << g.tsz) + 1 + 2 * g.halo : 1;
    const int wxy = wx * wy;
    const int jw = EM ? (1 << g.tsx) + 3 : 0, jh = EM ? (1 << g.tsy) + 3 : 0;
    const int fw = EM ? (1 << g.tsx) + 2 : 0, fh = EM ? (1 << g.tsy) + 2 : 0;
    const size_t acc_bytes = EM ? (size_t)3 * jw * jh * sizeof(double) : (size_t)wxy * wz * sizeof(A);
    A *sA = (A *)smem;
    R *sE = (R *)(smem + ((acc_bytes + 15) & ~(size_t)15));
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
    const int lane = (int)(threadIdx.x & 63);
    const uint64_t lt = lanemask_lt();
    if (threadIdx.x == 0) sErr = 0;
    const int b = bucket_of_block(g.nbuckets);
    if (b >= g.nbuckets) return;
    if (b == 0 && threadIdx.x == 0) {
        // (the workgroup that solves the 1D field reads the step in this launch)
        __hip_atomic_store(c.step, *c.step + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if constexpr (!FIRST) {
        __shared__ ExchangeLds sEx;
        exchange_bucket<MIX, DIM, VDIM>(g, t, b, n, max_per, c, sEx);
    }
    {
        int bx, by, bz;
        tile_coords<DIM>(g, b, bx, by, bz);
        const int x0 = bx << g.tsx, y0 = (DIM >= 2) ? (by << g.tsy) : 0, z0 = (DIM == 3) ? (bz << g.tsz) : 0;
        const TileNb tn = tile_nb<DIM>(g, bx, by, bz);
        const int count = t.cnt[b], dsb = t.ds[b], psb = t.ps[b];
        const int i0 = FIRST ? min(max(bstart[b], 0), g.np) : 0;
        const int npages = (count + kPage - 1) / kPage;
        const int mine = npages > w ? (npages - w + nw - 1) / nw : 0;   // units of this wave
        // this wave's part of the bucket's list: as long as its particles
        int seg = dsb;
        {
            int before = 0;
            for (int w2 = 0; w2 < w; ++w2) before += npages > w2 ? (npages - w2 + nw - 1) / nw : 0;
            // the last unit, which may be partly filled, belongs to wave (npages - 1) % nw
            const bool last_before = npages > 0 && (npages - 1) % nw < w;
            seg += before * kPage - (last_before ? npages * kPage - count : 0);
        }
        // page ids of this wave's units, 64 at a time, one per lane
        int pids = 0;
        auto ids = [&](int i) {
            pids = t.tab[psb + w + min(i + lane, mine - 1) * nw];
        };
        auto page_of = [&](int i) { return page_at<MIX, DIM, VDIM>(t, __builtin_amdgcn_readlane(pids, i & 63)); };
        Raw<MIX> ra[U], rb[U];
        char *sa = nullptr, *sb = nullptr;   // where the loaded units lie
        auto fetch = [&](Raw<MIX> *r, char *&s, int i) {
            i = min(i, mine - 1);
            s = page_of(i);
            if constexpr (FIRST) {
#pragma unroll
                for (int j = 0; j < U; ++j)
                    read_array<MIX, DIM, VDIM>(src, i0 + min((w + i * nw) * kPage + j * 64 + lane, count - 1), r[j]);
            } else {
#pragma unroll
                for (int j = 0; j < U; ++j) load_slot<MIX, DIM, VDIM, NT>(s, j * 64 + lane, r[j]);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        if (mine > 0) {
            ids(0);
            fetch(ra, sa, 0);
        }
        {
            const int na = EM ? 3 * jw * jh : wxy * wz;
            for (int t2 = threadIdx.x; t2 < na; t2 += blockDim.x) sA[t2] = (A)0;
        }
        if (threadIdx.x < kTab) sCnt[threadIdx.x] = 0;
        if constexpr (EM)
            load_f_tile<R>(sE, E, g, x0, y0, fw, fh);
        else if (MIX && E32)
            load_tile_any<R, float, DIM>(sE, E32, g, x0, y0, z0, ex_w, ey_w, ez_w);
        else
            load_tile_any<R, double, DIM>(sE, E, g, x0, y0, z0, ex_w, ey_w, ez_w);
        __syncthreads();
        double ke = 0.0, px = 0.0;
        int nlist = 0;   // leavers of this wave
        // a leaver for a bucket beyond the neighbours: its outbox entry joins one of the bucket's chains
        auto far_leaver = [&](int at, int nbk) {
            t.to.far_next[at] = atomicExch(&t.to.far_head[(int64_t)nbk * kFarChains + lane], at + 1);
            atomicAdd(&t.cnt_next[nbk], 1);
        };
        auto process = [&](Raw<MIX> *r, char *s, int i) {
#pragma unroll
            for (int j = 0; j < U; ++j) {
                // slot inside the bucket
                const int k = (w + i * nw) * kPage + j * 64 + lane;
                bool leaves = false;
                int code = 0, nbk = 0;
                if (k < count) {
                    Pt<MIX> q;
                    bool good = decode<MIX, DIM, VDIM>(r[j], g, q);
                    const double v2o = vsq<MIX, VDIM, HC>(q, pc);
                    int lx, ly, lz = 0, sx, sy, sz = 0;
                    R f0x = R(0), f0y = R(0), ig = R(1);
                    if constexpr (EM) {
                        good = advance_em<MIX, HC>(q, g, pc, sE, fw, x0, y0, lx, ly, sx, sy, f0x, f0y, ig) && good;
                    } else {
                        good = advance<MIX, DIM, VDIM, HC>(q, g, pc, sE, ex_w, ey_w, ez_w, x0, y0, z0, lx, ly, lz, sx,
                                                           sy, sz) && good;
                    }
                    if (!good) atomicOr(&sErr, ERR_DOMAIN);
                    const double v2n = vsq<MIX, VDIM, HC>(q, pc);
                    ke += v2o + v2n;   // halved once per bucket (exact: a power of two)
                    px += (double)q.vx;
                    code = dir_local<DIM>(tn, lx + sx, ly + sy, lz + sz);
                    leaves = code != kStay;
                    // absorbed by a wall: no deposit, no destination (listed as kStay)
                    const bool dead = g.walls && q.ix >= g.nxp;
                    if (dead) {
                        code = kStay;
                        leaves = true;
                    } else if constexpr (EM) {
                        const R wvx = q.vx * ig, wvy = q.vy * ig, wvz = q.vz * ig;
                        R ddx, ddy;
                        if constexpr (MIX) {
                            ddx = wvx * pc.dtdx;
                            ddy = wvy * pc.dtdy;
                        } else {
                            ddx = (wvx * pc.dt) * g.inv_dx;
                            ddy = (wvy * pc.dt) * g.inv_dy;
                        }
                        if (!esirkepov_lds<R>((double *)sA, jw, jw * jh, lx, ly, f0x, f0y, ddx, ddy,
                                              (R)(pc.jz * (double)wvz)))
                            atomicOr(&sErr, ERR_DOMAIN);
                    } else {
                        A wgt[8];
                        dep_weights<MIX, DIM>(q, g, wgt);
                        const int dlx = lx + sx + g.halo;
                        const int dly = (DIM >= 2) ? ly + sy + g.halo : 0;
                        const int dlz = (DIM == 3) ? lz + sz + g.halo : 0;
                        bool inl = (unsigned)dlx <= (unsigned)(wx - 2);
                        if constexpr (DIM >= 2) inl = inl && (unsigned)dly <= (unsigned)(wy - 2);
                        if constexpr (DIM == 3) inl = inl && (unsigned)dlz <= (unsigned)(wz - 2);
                        if (inl) {
                            const int a0 = (dlz * wy + dly) * wx + dlx;
                            acc_add_lds<MIX>(&sA[a0], wgt[0]);
                            acc_add_lds<MIX>(&sA[a0 + 1], wgt[1]);
                            if constexpr (DIM >= 2) {
                                acc_add_lds<MIX>(&sA[a0 + wx], wgt[2]);
                                acc_add_lds<MIX>(&sA[a0 + wx + 1], wgt[3]);
                            }
                            if constexpr (DIM == 3) {
                                acc_add_lds<MIX>(&sA[a0 + wxy], wgt[4]);
                                acc_add_lds<MIX>(&sA[a0 + wxy + 1], wgt[5]);
                                acc_add_lds<MIX>(&sA[a0 + wxy + wx], wgt[6]);
                                acc_add_lds<MIX>(&sA[a0 + wxy + wx + 1], wgt[7]);
                            }
                        } else if constexpr (DIM == 3) {
                            deposit_global3<MIX>(acc, g, q.ix, q.iy, q.iz, wgt);
                        } else {
                            deposit_global<MIX, DIM>(acc, g, q.ix, q.iy, wgt);
                        }
                    }
                    if (code == kFar) nbk = bucket_of<MIX, DIM>(g, q.ix, q.iy, q.iz);
                    encode<MIX, DIM>(q, r[j]);
                }
                const uint64_t m = __ballot(leaves);
                if (m) {
                    if (leaves) {
                        const int at = seg + nlist + (int)__popcll(m & lt);
                        t.raw_slot[at] = k;
                        t.raw_code[at] = (uint8_t)code;
                        out_put<MIX, DIM, VDIM>(t, at, r[j]);
                        atomicAdd(&sCnt[code], 1);
                        if (code == kFar) far_leaver(at, nbk);
                    }
                    nlist += (int)__popcll(m);
                }
            }
#pragma unroll
            for (int j = 0; j < U; ++j) store_slot<MIX, DIM, VDIM, NT>(s, j * 64 + lane, r[j]);
        };
        // a unit of a later step: groups of kGroup particles in straight-line code
        constexpr int kGroup = (MIX && DIM < 3) ? U : 1;
        auto process_group = [&](Raw<MIX> *r, char *s, int i) {
            const int rem = count - (w + i * nw) * kPage;   // particles from this unit's first slot on
            if (rem < kPage) {
                // the bucket's last unit: slots past its end hold anything; a resting particle in their place
#pragma unroll
                for (int j = 0; j < U; ++j) {
                    if (j * 64 + lane >= rem) {
                        Pt<MIX> q{};
                        q.ix = x0;
                        q.iy = y0;
                        q.iz = z0;
                        if constexpr (MIX) {
                            q.fx = q.fy = q.fz = 0.5f;
                        } else {
                            q.x = (x0 + 0.5) / g.inv_dx;
                            q.y = (y0 + 0.5) / g.inv_dy;
                            q.z = (z0 + 0.5) / g.inv_dz;
                        }
                        encode<MIX, DIM>(q, r[j]);
                    }
                }
            }
#pragma unroll
            for (int h = 0; h < U; h += kGroup) {
                Moved<MIX> m[kGroup];
                advance_group<MIX, DIM, VDIM, HC, ROT, kGroup>(r + h, g, pc, sE, ex_w, ey_w, ez_w, x0, y0, z0, m);
                bool ok = true;
#pragma unroll
                for (int j = 0; j < kGroup; ++j) ok = ok && m[j].ok;
                if (__ballot(!ok)) {
#pragma unroll
                    for (int j = 0; j < kGroup; ++j) {
                        if (m[j].ok) continue;
                        // the general move from the old position
                        Pt<MIX> q;
                        decode<MIX, DIM, VDIM>(r[h + j], g, q);
                        const int lx = q.ix - x0, ly = q.iy - y0, lz = q.iz - z0;
                        q.vx = m[j].q.vx;
                        q.vy = m[j].q.vy;
                        q.vz = m[j].q.vz;
                        R ux = q.vx, uy = q.vy, uz = q.vz;
                        if constexpr (HC) {
                            const R gm = lorentz<R>(q.vx, q.vy, q.vz, MIX ? (R)pc.ic2f : (R)pc.ic2);
                            const R ig = R(1) / gm;
                            ux = MIX ? q.vx * ig : q.vx / gm;
                            uy = MIX ? q.vy * ig : q.vy / gm;
                            uz = MIX ? q.vz * ig : q.vz / gm;
                        }
                        int sx, sy, sz;
                        if (!move_pt_v<MIX, DIM>(q, g, pc, ux, uy, uz, sx, sy, sz) && (h + j) * 64 + lane < rem)
                            atomicOr(&sErr, ERR_DOMAIN);
                        m[j].q = q;
                        m[j].lx = lx + sx;
                        m[j].ly = (DIM >= 2) ? ly + sy : 0;
                        m[j].lz = (DIM == 3) ? lz + sz : 0;
                    }
                }
                bool leaves[kGroup], some = false;
#pragma unroll
                for (int j = 0; j < kGroup; ++j) {
                    const Pt<MIX> &q = m[j].q;
                    const int lx = m[j].lx, ly = m[j].ly, lz = m[j].lz;
                    const bool act = (h + j) * 64 + lane < rem;
                    bool stay = (unsigned)lx < (unsigned)tn.txe;
                    bool inl = act && (unsigned)(lx + g.halo) <= (unsigned)(wx - 2);
                    if constexpr (DIM >= 2) {
                        stay = stay && (unsigned)ly < (unsigned)tn.tye;
                        inl = inl && (unsigned)(ly + g.halo) <= (unsigned)(wy - 2);
                    }
                    if constexpr (DIM == 3) {
                        stay = stay && (unsigned)lz < (unsigned)tn.tze;
                        inl = inl && (unsigned)(lz + g.halo) <= (unsigned)(wz - 2);
                    }
                    if constexpr (DIM == 2) inl = inl && !(g.walls && (unsigned)(x0 + lx) >= (unsigned)g.nxp);
                    leaves[j] = act && !stay;
                    some = some || leaves[j];
                    A wgt[8];
                    dep_weights<MIX, DIM>(q, g, wgt);
                    const int a0 = ((lz + (DIM == 3 ? g.halo : 0)) * wy + (ly + (DIM >= 2 ? g.halo : 0))) * wx + lx +
                                   g.halo;
                    if (inl) {
                        ke += (double)m[j].v2 + vsq<MIX, VDIM, HC>(q, pc);   // halved once per bucket
                        px += (double)q.vx;
                        acc_add_lds<MIX>(&sA[a0], wgt[0]);
                        acc_add_lds<MIX>(&sA[a0 + 1], wgt[1]);
                        if constexpr (DIM >= 2) {
                            acc_add_lds<MIX>(&sA[a0 + wx], wgt[2]);
                            acc_add_lds<MIX>(&sA[a0 + wx + 1], wgt[3]);
                        }
                        if constexpr (DIM == 3) {
                            acc_add_lds<MIX>(&sA[a0 + wxy], wgt[4]);
                            acc_add_lds<MIX>(&sA[a0 + wxy + 1], wgt[5]);
                            acc_add_lds<MIX>(&sA[a0 + wxy + wx], wgt[6]);
                            acc_add_lds<MIX>(&sA[a0 + wxy + wx + 1], wgt[7]);
                        }
                    }
                    // the state of a particle that stays (its cell needs no wrap)
                    Pt<MIX> qs = q;
                    qs.ix = x0 + lx;
                    qs.iy = y0 + ly;
                    qs.iz = z0 + lz;
                    encode<MIX, DIM>(qs, r[h + j]);
                }
                if (__ballot(some)) {
#pragma unroll
                    for (int j = 0; j < kGroup; ++j) {
                        const uint64_t mk = __ballot(leaves[j]);
                        if (!mk) continue;
                        if (leaves[j]) {
                            Pt<MIX> q = m[j].q;
                            const int lx = m[j].lx, ly = m[j].ly, lz = m[j].lz;
                            auto wrap = [](int v, int n) {
                                if (v >= n || v < 0) {
                                    v %= n;
                                    if (v < 0) v += n;
                                }
                                return v;
                            };
                            q.ix = wrap(x0 + lx, g.nx);
                            q.iy = (DIM >= 2) ? wrap(y0 + ly, g.ny) : 0;
                            q.iz = (DIM == 3) ? wrap(z0 + lz, g.nz) : 0;
                            encode<MIX, DIM>(q, r[h + j]);
                            int code = dir_local<DIM>(tn, lx, ly, lz);
                            bool inl = (unsigned)(lx + g.halo) <= (unsigned)(wx - 2);
                            if constexpr (DIM >= 2) inl = inl && (unsigned)(ly + g.halo) <= (unsigned)(wy - 2);
                            if constexpr (DIM == 3) inl = inl && (unsigned)(lz + g.halo) <= (unsigned)(wz - 2);
                            if constexpr (DIM == 2) inl = inl && !(g.walls && (unsigned)(x0 + lx) >= (unsigned)g.nxp);
                            const bool dead = g.walls && q.ix >= g.nxp;
                            if (!inl) {
                                ke += (double)m[j].v2 + vsq<MIX, VDIM, HC>(q, pc);
                                px += (double)q.vx;
                            }
                            // absorbed by a wall: no deposit, no destination (listed as kStay)
                            if (dead) {
                                code = kStay;
                            } else if (!inl) {
                                A wgt[8];
                                dep_weights<MIX, DIM>(q, g, wgt);
                                if constexpr (DIM == 3)
                                    deposit_global3<MIX>(acc, g, q.ix, q.iy, q.iz, wgt);
                                else
                                    deposit_global<MIX, DIM>(acc, g, q.ix, q.iy, wgt);
                            }
                            const int at = seg + nlist + (int)__popcll(mk & lt);
                            t.raw_slot[at] = (w + i * nw) * kPage + (h + j) * 64 + lane;
                            t.raw_code[at] = (uint8_t)code;
                            out_put<MIX, DIM, VDIM>(t, at, r[h + j]);
                            atomicAdd(&sCnt[code], 1);
                            if (code == kFar) far_leaver(at, bucket_of<MIX, DIM>(g, q.ix, q.iy, q.iz));
                        }
                        nlist += (int)__popcll(mk);
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < U; ++j) store_slot<MIX, DIM, VDIM, NT>(s, j * 64 + lane, r[j]);
        };
        // (the caller's arrays take the form that checks its input, and the
        // electromagnetic step its own)
        auto unit = [&](Raw<MIX> *r, char *s, int i) {
            if constexpr (FIRST || EM)
                process(r, s, i);
            else
                process_group(r, s, i);
        };
        // two register sets, each unit's loads issued one unit ahead of its
        // use; the fetches are unconditional (clamped to the wave's units)
        for (int i = 0; i < mine; i += 2) {
            fetch(rb, sb, i + 1);
            unit(ra, sa, i);
            if ((i & 63) == 62) ids(i + 2);
            fetch(ra, sa, i + 2);
            if (i + 1 < mine) unit(rb, sb, i + 1);
        }
        for (int off = 32; off > 0; off >>= 1) {
            ke += __shfl_xor(ke, off);
            px += __shfl_xor(px, off);
        }
        if (lane == 0) {
            sList[w] = nlist;
            sKe[w] = ke;
            sPx[w] = px;
        }
        __syncthreads();   // the deposit tile, the pages and the lists are complete
        if constexpr (EM)
            flush_j((double *)acc, (const double *)sA, g, x0, y0, jw, jh, pc.jx, pc.jy);
        else if constexpr (DIM == 3)
            flush_region3<MIX>(acc, sA, g, x0, y0, z0, wx, wy, wz, g.halo);
        else
            flush_region<MIX, DIM>(acc, sA, g, x0, y0, wx, wy, g.halo);
        int nout = 0;
        for (int w2 = 0; w2 < nw; ++w2) nout += sList[w2];
        if (threadIdx.x == 0) {
            if (part) {
                double kt = 0.0, pt = 0.0;
                for (int w2 = 0; w2 < nw; ++w2) {
                    kt += sKe[w2];
                    pt += sPx[w2];
                }
                __hip_atomic_store(&part[2 * b], 0.5 * kt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(&part[2 * b + 1], pt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            if (count > nout) atomicAdd(&t.cnt_next[b], count - nout);
        }
        if (threadIdx.x < kTab) {
            const int d = threadIdx.x, v = sCnt[d];
            int off = 0;
            for (int e = 0; e < d; ++e) off += sCnt[e];
            sOff[d] = off;
            t.to.off[b * kTab + d] = off;
            t.to.cnt[b * kTab + d] = v;
            if (v && d == kStay) atomicSub(t.live, v);   // absorbed by a wall
            if (v && d < kFar && d != kStay) atomicAdd(&t.cnt_next[dir_target<DIM>(g, bx, by, bz, d)], v);
        }
        // the leavers in direction order, ranked in list order: their slots (the
        // bucket's holes) and their outbox entries
        for (int e0 = 0; e0 < nout; e0 += blockDim.x) {
            const int e = e0 + (int)threadIdx.x;
            int code = -1, slot = 0, at = dsb;
            if (e < nout) {
                // entry e of the waves' parts, one after the other
                int r = e, before = 0;
                for (int w2 = 0; w2 < nw; ++w2) {
                    const int units = npages > w2 ? (npages - w2 + nw - 1) / nw : 0;
                    const bool last_before = npages > 0 && (npages - 1) % nw < w2;
                    const int sg = dsb + before * kPage - (last_before ? npages * kPage - count : 0);
                    if (r >= 0 && r < sList[w2]) at = sg + r;
                    r -= sList[w2];
                    before += units;
                }
                slot = t.raw_slot[at];
                code = t.raw_code[at];
            }
            uint64_t peers = __ballot(code >= 0);
#pragma unroll
            for (int bit = 0; bit < 5; ++bit) {
                const uint64_t bb = __ballot(code >= 0 && ((code >> bit) & 1));
                peers &= ((code >> bit) & 1) ? bb : ~bb;
            }
            __syncthreads();   // sOff is complete, the previous round's counts are read
            if (lane < kTab) sMv[w][lane] = 0;
            if (code >= 0 && (peers & lt) == 0) sMv[w][code] = (int)__popcll(peers);
            __syncthreads();
            if (code >= 0) {
                int off = sOff[code] + (int)__popcll(peers & lt);
                for (int w2 = 0; w2 < w; ++w2) off += sMv[w2][code];
                t.to.hole[dsb + off] = slot;
                t.to.order[dsb + off] = at;
            }
            __syncthreads();
            if (threadIdx.x < kTab) {
                int v = 0;
                for (int w2 = 0; w2 < nw; ++w2) v += sMv[w2][threadIdx.x];
                sOff[threadIdx.x] += v;
            }
        }
        __syncthreads();
    }
    __syncthreads();
    if (threadIdx.x == 0 && sErr) raise_err(c.err, sErr);
    if constexpr (DIM == 1) {
        if (f.E) field_by_last<MIX>(g, t, f, acc, part, smem, c);
    }
}

// ---- back to the caller's arrays --------------------------------------------------
template <bool MIX, int DIM, int VDIM>
__global__ void __launch_bounds__(kBlock) k_page_end(Geo g, PageStep t, int64_t n, int64_t max_per, Parts dst,
                                                     int32_t *bstart, CtxDev c) {
    __shared__ ExchangeLds sEx;
    const int nb = g.nbuckets;
    const int b = bucket_of_block(nb);
    if (b >= nb) return;
    exchange_bucket<MIX, DIM, VDIM>(g, t, b, n, max_per, c, sEx);
    {
        const int count = t.cnt[b], dsb = t.ds[b], psb = t.ps[b];
        if (threadIdx.x == 0) {
            bstart[b] = dsb;
            if (b == nb - 1) bstart[nb] = dsb + count;
        }
        // four particles per thread and round, their loads issued before the first
        // store; the rounds start at the line boundary at or below the bucket's
        // first place, so that the waves store whole lines
        constexpr int P = 4;
        const int ahead = dsb & (MIX ? 31 : 15);
        const int rounds = copy_rounds(count, ahead, P * kBlock);
        for (int q = 0; q < rounds; ++q) {
            const int k0 = q * P * kBlock - ahead;
            Raw<MIX> r[P];
#pragma unroll
            for (int j = 0; j < P; ++j) {
                const int k = copy_slot(k0 + j * kBlock + (int)threadIdx.x, count);
                load_slot<MIX, DIM, VDIM>(page_at<MIX, DIM, VDIM>(t, t.tab[psb + k / kPage]), k % kPage, r[j]);
            }
#pragma unroll
            for (int j = 0; j < P; ++j) {
                const int k = k0 + j * kBlock + (int)threadIdx.x;
                if (k >= 0 && k < count) store_raw<MIX, DIM, VDIM>(dst, dsb + k, r[j]);
            }
        }
    }
}

}  // namespace

// ================================================================ launchers

hipError_t load_page_kernels() {
    hipFuncAttributes a;
    return hipFuncGetAttributes(&a, (const void *)k_page_fill);
}

hipError_t launch_page_begin(const Geo &g, const PageStep &t, int32_t *cnt3, int32_t *head2, int64_t n,
                             int64_t max_per_bucket, const int32_t *bstart, uint64_t *acc, int64_t nacc,
                             const CtxDev &c, hipStream_t s) {
    hipLaunchKernelGGL(k_page_scan<true>, dim3(1), dim3(1024), 0, s, g.nbuckets, n, g.walls, max_per_bucket, bstart,
                       cnt3, t.ds, t.ps, c);
    const int64_t most = std::max<int64_t>(std::max<int64_t>(t.npages, nacc), 2 * (int64_t)g.nbuckets * kFarChains);
    const int blocks = (int)std::min<int64_t>((most + kBlock - 1) / kBlock, 2048);
    hipLaunchKernelGGL(k_page_fill, dim3(blocks), dim3(kBlock), 0, s, g.nbuckets, t, cnt3, head2, acc, nacc);
    return hipGetLastError();
}

// The step with the sums over the buckets before a push or a call's end taken
// apart, where the workgroups do not take them themselves.
static PageStep scan_apart(const Geo &g, const PageStep &step, int64_t n, int64_t max_per_bucket, const CtxDev &c,
                           hipStream_t s) {
    PageStep t = step;
    t.scanned = g.nbuckets > kPageScanMax;
    if (t.scanned)
        hipLaunchKernelGGL(k_page_scan<false>, dim3(1), dim3(1024), 0, s, g.nbuckets, n, g.walls, max_per_bucket,
                           nullptr, (int32_t *)t.cnt, t.ds, t.ps, c);
    return t;
}

// Threads per bucket: 256, or twice that with at most two buckets per CU, which
// leave its SIMDs short of waves. Per step in calls of 20: electromagnetic 8.4M
// mixed in 512 buckets 175 us with 256 threads, 157 with 512; two-stream 64 x 64,
// 0.52M mixed in 128 buckets 43.9 us with 256, 38.6 with 512, 40.7 with 1024; but
// 4.2M mixed between walls in 1024 buckets 73.7 us with 256, 82.8 with 512.
int push_block(const Geo &g) { return g.nbuckets <= 2 * cu_count() ? kPagePushMax : kBlock; }

hipError_t launch_page_push(const Geo &g, bool mixed, const PageStep &step, const Parts *src, const int32_t *bstart,
                            int64_t n, int64_t max_per_bucket, const double *E, const float *E32, const PushC &pc,
                            void *acc, double *part, const PageField &f, const CtxDev &c, hipStream_t s) {
    const dim3 grid(grid_for_buckets(g.nbuckets));
    const Parts from = src ? *src : Parts{};
    const PageStep t = src ? step : scan_apart(g, step, n, max_per_bucket, c, s);
    if (g.em) {
        const size_t sh = em_j_tile_bytes(g) + em_f_tile_bytes(g, mixed);
        auto go = [&](auto kern, auto *accp) {
            hipLaunchKernelGGL(kern, grid, dim3(push_block(g)), sh, s, g, t, from, bstart, n, max_per_bucket,
                               E, nullptr, pc, accp, part, f, c);
        };
        unsigned long long *am = (unsigned long long *)acc;
        double *ad = (double *)acc;
        auto pick = [&](auto first) {
            constexpr bool F = decltype(first)::value;
            if (mixed && g.hc) go(k_page_push<true, 2, 3, true, true, false, F, true>, am);
            else if (mixed) go(k_page_push<true, 2, 3, false, true, false, F, true>, am);
            else if (g.hc) go(k_page_push<false, 2, 3, true, true, false, F, true>, ad);
            else go(k_page_push<false, 2, 3, false, true, false, F, true>, ad);
        };
        if (src) pick(std::true_type{});
        else pick(std::false_type{});
        return hipGetLastError();
    }
    // Below 3D, pages that the memory-side cache (256 MB) can hold from step to step
    // go through the caches, others past them with the nontemporal hint. Per step in
    // calls of 20 with the hint and without: 2D2V FP64 128 MB 94.9 and 86.0 us, 208 MB
    // 141 and 135, 288 MB 202 and 214, 537 MB 288 and 339; 2D3V mixed 144 MB 111 and
    // 100, 216 MB 163 and 157, 288 MB 186 and 197; walls 160 MB 126 and 122, 240 MB
    // 184 and 189. 3D mixed 56 MB 173 and 170, 168 MB 225 and 230, 470 MB 384 and 431.
    // (The electromagnetic push is not bound by its pages: 201 MB 156 and 158.)
    const bool cached = particle_state_bytes(g, mixed, n) <= kCachedBytes;
    const size_t tile = tile_acc_bytes(g, g.halo) + tile_e_bytes(g, mixed);
    const size_t sh = f.E ? std::max(tile, (size_t)(g.nx + 2 * kBlock) * sizeof(double)) : tile;
    APIC_DISPATCH(g, mixed, {
        auto go = [&](auto kern) {
            hipLaunchKernelGGL(kern, grid, dim3(push_block(g)), sh, s, g, t, from, bstart, n,
                               max_per_bucket, E, MIX ? E32 : nullptr, pc, (typename AccOf<MIX>::T *)acc, part, f, c);
        };
        // the rotation about z in its own build (in a zero field it is left out)
        auto pick = [&](auto rot) {
            constexpr bool ROT = decltype(rot)::value;
            if constexpr (DIM < 3) {
                if (cached) {
                    go(k_page_push<MIX, DIM, VDIM, HC, false, ROT, false, false>);
                    return;
                }
            }
            go(k_page_push<MIX, DIM, VDIM, HC, false, ROT, false, true>);
        };
        if (src) {
            go(k_page_push<MIX, DIM, VDIM, HC, false, false, true, true>);
        } else if constexpr (VDIM >= 2 && !HC) {
            if (pc.t != 0.0) pick(std::true_type{});
            else pick(std::false_type{});
        } else {
            pick(std::false_type{});
        }
    });
    return hipGetLastError();
}

#define APIC_PAGE_DISPATCH(g, mixed, ...)                                                                   \
    do {                                                                                                    \
        if ((g).dim == 3) APIC_DISPATCH_MIX(mixed, false, 3, 3, __VA_ARGS__);                               \
        else APIC_DISPATCH_2D(g, mixed, __VA_ARGS__);                                                       \
    } while (0)

hipError_t launch_page_end(const Geo &g, bool mixed, const PageStep &step, int64_t n, int64_t max_per_bucket,
                           const Parts &dst, int32_t *bstart, const CtxDev &c, hipStream_t s) {
    const dim3 grid(grid_for_buckets(g.nbuckets));
    const PageStep t = scan_apart(g, step, n, max_per_bucket, c, s);
    APIC_PAGE_DISPATCH(g, mixed,
                       hipLaunchKernelGGL((k_page_end<MIX, DIM, VDIM>), grid, dim3(kBlock), 0, s, g, t, n,
                                          max_per_bucket, dst, bstart, c));
    return hipGetLastError();
}

}  // namespace apic

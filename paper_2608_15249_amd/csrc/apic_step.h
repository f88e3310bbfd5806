// Device helpers of the fused step shared by the passes that reorder the
// particles (apic_kernels.hip) and the passes that keep them in place
// (apic_pages.hip): direction codes of a move, the advance of one particle of
// a bucket's tile, raw loads and their decoding, LDS sizes of the tiles.
#pragma once

#include "apic_device.h"
#include "apic_em.h"

namespace apic {
namespace {

// ------------------------------------------------- step: bucket directions
//
// A particle of bucket (bx, by[, bz]) lands after the move in bucket
// (bx+dbx, by+dby[, bz+dbz]) (periodic). Moves with every |db| <= 1 get the
// direction code d = (dby+1)*3 + (dbx+1) in 0..8 (1D, 2D), or
// d = ((dbz+1)*3 + (dby+1))*3 + (dbx+1) in 0..26 (3D); larger jumps get the
// far code. The count pass tallies particles per (source bucket, wave, d);
// the scan turns the tallies into start offsets inside the destination
// buckets (ordered by d, then wave); the push pass hands out consecutive
// slots per (wave, d) in the order the wave meets its particles. The order is
// therefore fixed by the previous order alone: no atomics decide where a near
// particle goes. Far movers (rare) take slots from an atomic cursor at the
// end of their bucket.
template <int DIM> struct Dir {
    static constexpr int kN = (DIM == 3) ? 28 : 10;      // direction codes (near + far)
    static constexpr int kFar = kN - 1;
    static constexpr int kStay = (DIM == 3) ? 13 : 4;    // the code of a particle that stays
    static constexpr int kTab = kN;                      // per-bucket table entries (one per direction)
    static constexpr int kCodeBits = (DIM == 3) ? 5 : 4; // bits of a near code
};
static_assert(Dir<3>::kTab <= kStepTab && Dir<2>::kTab <= kStepTab, "direction table size");
static_assert(kDeepTab == 2, "deep table size");

// Tile coordinates of bucket b (tiles numbered x fastest, then y, then z).
template <int DIM>
__device__ __forceinline__ void tile_coords(const Geo &g, int b, int &bx, int &by, int &bz) {
    if constexpr (DIM == 1) {
        bx = b; by = 0; bz = 0;
    } else if constexpr (DIM == 2) {
        bx = b % g.nbx; by = b / g.nbx; bz = 0;
    } else {
        bx = b % g.nbx; const int r = b / g.nbx; by = r % g.nby; bz = r / g.nby;
    }
}

template <int DIM>
__device__ __forceinline__ int bucket_index(const Geo &g, int bx, int by, int bz) {
    if constexpr (DIM == 1) return bx;
    if constexpr (DIM == 2) return by * g.nbx + bx;
    return (bz * g.nby + by) * g.nbx + bx;
}

__device__ __forceinline__ int wrap_tile(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }

// Bucket reached from (bx, by, bz) with near direction d.
template <int DIM>
__device__ __forceinline__ int dir_target(const Geo &g, int bx, int by, int bz, int d) {
    const int tx = wrap_tile(bx + d % 3 - 1, g.nbx);
    const int ty = (DIM >= 2) ? wrap_tile(by + (d / 3) % 3 - 1, g.nby) : 0;
    const int tz = (DIM == 3) ? wrap_tile(bz + d / 9 - 1, g.nbz) : 0;
    return bucket_index<DIM>(g, tx, ty, tz);
}

// Source bucket that reaches bucket nbk with direction d.
template <int DIM>
__device__ __forceinline__ int dir_source(const Geo &g, int nbk, int d) {
    int bx, by, bz;
    tile_coords<DIM>(g, nbk, bx, by, bz);
    const int sx = wrap_tile(bx - (d % 3 - 1), g.nbx);
    const int sy = (DIM >= 2) ? wrap_tile(by - ((d / 3) % 3 - 1), g.nby) : 0;
    const int sz = (DIM == 3) ? wrap_tile(bz - (d / 9 - 1), g.nbz) : 0;
    return bucket_index<DIM>(g, sx, sy, sz);
}

// Direction code from a particle's tile-local cell after the move, (lxn,
// lyn, lzn) = old tile-local cell + unwrapped cell shift: the widths of the
// tile and of its neighbours (the last tile of an axis may be cut by the grid
// edge; neighbours wrap periodically) decide whether it stayed, crossed into
// a neighbour, or jumped farther (the far code), without per-particle wrap
// arithmetic.
struct TileNb {
    int txe, lw, rw;   // widths (cells) of this tile and its left / right neighbour
    int tye, dw, uw;   // same along y
    int tze, bw, fw;   // same along z
};

__device__ __forceinline__ int tile_width(int i, int t, int n) { return min(t, n - i * t); }

// A wave-uniform 32-bit value moved into a vector register (when ON):
// per-lane arithmetic reads it from there, leaving the scalar registers to
// the state the chunk loop itself carries.
template <bool ON, typename T>
__device__ __forceinline__ T vreg(T x) {
    static_assert(sizeof(T) == 4, "a 32-bit value");
    if constexpr (ON) asm("" : "+v"(x));
    return x;
}

template <int DIM>
__device__ __forceinline__ TileNb tile_nb(const Geo &g, int bx, int by, int bz = 0) {
    TileNb t;
    const int T = 1 << g.tsx;
    t.txe = tile_width(bx, T, g.nx);
    t.lw = tile_width(bx == 0 ? g.nbx - 1 : bx - 1, T, g.nx);
    t.rw = tile_width(bx == g.nbx - 1 ? 0 : bx + 1, T, g.nx);
    t.tye = t.dw = t.uw = 1;
    t.tze = t.bw = t.fw = 1;
    if constexpr (DIM >= 2) {
        const int V = 1 << g.tsy;
        t.tye = tile_width(by, V, g.ny);
        t.dw = tile_width(by == 0 ? g.nby - 1 : by - 1, V, g.ny);
        t.uw = tile_width(by == g.nby - 1 ? 0 : by + 1, V, g.ny);
    }
    if constexpr (DIM == 3) {
        const int Z = 1 << g.tsz;
        t.tze = tile_width(bz, Z, g.nz);
        t.bw = tile_width(bz == 0 ? g.nbz - 1 : bz - 1, Z, g.nz);
        t.fw = tile_width(bz == g.nbz - 1 ? 0 : bz + 1, Z, g.nz);
    }
    return t;
}

template <int DIM>
__device__ __forceinline__ int dir_local(const TileNb &t, int lxn, int lyn, int lzn = 0) {
    const int dbx = (lxn < 0) ? -1 : (lxn >= t.txe) ? 1 : 0;
    bool far = lxn < -t.lw || lxn >= t.txe + t.rw;
    int dby = 0, dbz = 0;
    if constexpr (DIM >= 2) {
        dby = (lyn < 0) ? -1 : (lyn >= t.tye) ? 1 : 0;
        far = far || lyn < -t.dw || lyn >= t.tye + t.uw;
    }
    if constexpr (DIM == 3) {
        dbz = (lzn < 0) ? -1 : (lzn >= t.tze) ? 1 : 0;
        far = far || lzn < -t.bw || lzn >= t.tze + t.fw;
        return far ? Dir<3>::kFar : ((dbz + 1) * 3 + (dby + 1)) * 3 + (dbx + 1);
    }
    return far ? Dir<DIM>::kFar : (dby + 1) * 3 + (dbx + 1);
}

// Twice the kinetic energy per unit mass of a particle for the diagnostic:
// |v|^2 (binary32 squares on the mixed path, FP64 on the FP64 path), or for
// the Higuera-Cary state 2 (gamma - 1) c^2 = 2 |u|^2 / (gamma + 1): in FP64
// on the FP64 path, on the mixed path in binary32 with the hardware square
// root and reciprocal (each within 1 ulp; a diagnostic, summed in FP64).
template <bool MIX, int VDIM, bool HC>
__device__ __forceinline__ double vsq(const Pt<MIX> &q, const PushC &pc) {
    if constexpr (HC && MIX) {
        const float u2 = (q.vx * q.vx + q.vy * q.vy) + q.vz * q.vz;
        const float gp1 = __builtin_amdgcn_sqrtf(1.0f + u2 * pc.ic2f) + 1.0f;
        return (double)(2.0f * u2 * __builtin_amdgcn_rcpf(gp1));
    } else if constexpr (HC) {
        const double ux = q.vx, uy = q.vy, uz = q.vz;
        const double u2 = (ux * ux + uy * uy) + uz * uz;
        return 2.0 * u2 / (sqrt(1.0 + u2 * pc.ic2) + 1.0);
    }
    auto v2 = q.vx * q.vx;
    if constexpr (VDIM >= 2) v2 = v2 + q.vy * q.vy;
    if constexpr (VDIM >= 3) v2 = v2 + q.vz * q.vz;
    return (double)v2;
}

// Gather + Boris + move of one loaded particle of the block's tile; shared by
// the count and the push pass so that both compute identical bits. A particle
// outside the tile (the bucket table does not match the order) is flagged
// and clamped into the tile so that every access stays in bounds. The E tile
// spans ex_w x ey_w x ez_w nodes from (x0, y0, z0).
template <bool MIX, int DIM, int VDIM, bool HC>
__device__ __forceinline__ bool advance(Pt<MIX> &q, const Geo &g, const PushC &pc,
                                        const typename Pt<MIX>::R *sE, int ex_w, int ey_w, int ez_w, int x0, int y0,
                                        int z0, int &lx, int &ly, int &lz, int &sx, int &sy, int &sz) {
    using R = typename Pt<MIX>::R;
    lx = q.ix - x0;
    ly = (DIM >= 2) ? q.iy - y0 : 0;
    lz = (DIM == 3) ? q.iz - z0 : 0;
    bool in = (unsigned)lx < (unsigned)(ex_w - 1);
    if constexpr (DIM >= 2) in = in && (unsigned)ly < (unsigned)(ey_w - 1);
    if constexpr (DIM == 3) in = in && (unsigned)lz < (unsigned)(ez_w - 1);
    if (!in) {
        lx = min(max(lx, 0), ex_w - 2);
        ly = (DIM >= 2) ? min(max(ly, 0), ey_w - 2) : 0;
        lz = (DIM == 3) ? min(max(lz, 0), ez_w - 2) : 0;
        q.ix = x0 + lx;
        q.iy = y0 + ly;
        q.iz = z0 + lz;
    }
    R ex, ey, ez = R(0);
    if constexpr (DIM == 3) {
        const int wxy = ex_w * ey_w;
        gather_lds3<R>(sE, ex_w, wxy, wxy * ez_w, lx, ly, lz, q.fx, q.fy, q.fz, ex, ey, ez);
    } else {
        gather_lds<R, DIM>(sE, ex_w, ex_w * ey_w, lx, ly, q.fx, q.fy, ex, ey);
    }
    return push_move<MIX, DIM, VDIM, HC>(q, g, pc, ex, ey, ez, true, sx, sy, sz) && in;
}

// Electromagnetic form (2D3V): E and B gathered from the Yee field tile
// (nodes from (x0-1, y0-1), width fw), Boris (or Higuera-Cary with the state
// u = gamma v) in B, move. (lx, ly) and (fx0, fy0) return the old local cell
// and fractions for the current deposit, ig the factor 1 / gamma the move
// multiplied u by (1 for Boris).
template <bool MIX, bool HC>
__device__ __forceinline__ bool advance_em(Pt<MIX> &q, const Geo &g, const PushC &pc,
                                           const typename Pt<MIX>::R *sF, int fw, int x0, int y0, int &lx, int &ly,
                                           int &sx, int &sy, typename Pt<MIX>::R &fx0, typename Pt<MIX>::R &fy0,
                                           typename Pt<MIX>::R &ig) {
    using R = typename Pt<MIX>::R;
    const int tx = 1 << g.tsx, ty = 1 << g.tsy;
    lx = q.ix - x0;
    ly = q.iy - y0;
    const bool in = (unsigned)lx < (unsigned)tx && (unsigned)ly < (unsigned)ty;
    if (!in) {
        lx = min(max(lx, 0), tx - 1);
        ly = min(max(ly, 0), ty - 1);
        q.ix = x0 + lx;
        q.iy = y0 + ly;
    }
    fx0 = q.fx;
    fy0 = q.fy;
    R e[3], b[3];
    gather_em<R>(sF, fw, fw * (ty + 2), lx, ly, q.fx, q.fy, e, b);
    int sz;
    if constexpr (HC) {
        const R ic2 = MIX ? (R)pc.ic2f : (R)pc.ic2;
        hc3<R>(q.vx, q.vy, q.vz, e, b, MIX ? (R)pc.af : (R)pc.a, ic2);
        ig = recip<R>(lorentz<R>(q.vx, q.vy, q.vz, ic2));
        return move_pt_v<MIX, 2>(q, g, pc, q.vx * ig, q.vy * ig, q.vz * ig, sx, sy, sz) && in;
    } else {
        boris3<R>(q.vx, q.vy, q.vz, e, b, MIX ? (R)pc.af : (R)pc.a);
        ig = R(1);
        return move_pt<MIX, 2>(q, g, pc, sx, sy, sz) && in;
    }
}

// Raw stored words of one particle: loaded unconditionally (the caller clamps
// the index) so that a wave issues all its loads before it needs any data.
template <bool MIX> struct Raw {
    int32_t c;
    float ox, oy, oz, vx, vy, vz;
};
template <> struct Raw<false> {
    double x, y, z, vx, vy, vz;
};

template <bool MIX, int DIM, int VDIM, bool NT = MIX>
__device__ __forceinline__ void load_raw(const Parts &s, int i, Raw<MIX> &r) {
    // each particle is read once per pass, in whole 128-byte lines per wave
    // (the passes align their chunks). The mixed state of the step's passes loads
    // with the nontemporal hint (NT): measured at 512^2 (2D2V), 1024^2 (2D3V) and
    // 128^3, it was faster or equal; the FP64 state loads through the caches (the
    // hint made its push 5% slower). Nontemporal stores of the scattered
    // destination slots made the mixed push 1.6x slower.
    static_assert(MIX || !NT, "the FP64 state loads through the caches");
    if constexpr (MIX && !NT) {
        r.c = s.cell[i];
        r.ox = s.ox[i];
        r.oy = (DIM >= 2) ? s.oy[i] : 0.0f;
        r.oz = (DIM == 3) ? s.oz[i] : 0.0f;
        r.vx = (VDIM >= 1) ? ((const float *)s.vx)[i] : 0.0f;
        r.vy = (VDIM >= 2) ? ((const float *)s.vy)[i] : 0.0f;
        r.vz = (VDIM >= 3) ? ((const float *)s.vz)[i] : 0.0f;
    } else if constexpr (MIX) {
        r.c = __builtin_nontemporal_load(&s.cell[i]);
        r.ox = __builtin_nontemporal_load(&s.ox[i]);
        r.oy = (DIM >= 2) ? __builtin_nontemporal_load(&s.oy[i]) : 0.0f;
        r.oz = (DIM == 3) ? __builtin_nontemporal_load(&s.oz[i]) : 0.0f;
        r.vx = (VDIM >= 1) ? __builtin_nontemporal_load(&((const float *)s.vx)[i]) : 0.0f;
        r.vy = (VDIM >= 2) ? __builtin_nontemporal_load(&((const float *)s.vy)[i]) : 0.0f;
        r.vz = (VDIM >= 3) ? __builtin_nontemporal_load(&((const float *)s.vz)[i]) : 0.0f;
    } else {
        r.x = s.x[i];
        r.y = (DIM >= 2) ? s.y[i] : 0.0;
        r.z = (DIM == 3) ? s.z[i] : 0.0;
        r.vx = (VDIM >= 1) ? ((const double *)s.vx)[i] : 0.0;
        r.vy = (VDIM >= 2) ? ((const double *)s.vy)[i] : 0.0;
        r.vz = (VDIM >= 3) ? ((const double *)s.vz)[i] : 0.0;
    }
}

// Decode raw words into the working form (same checks as load_pt).
template <bool MIX, int DIM, int VDIM>
__device__ __forceinline__ bool decode(const Raw<MIX> &r, const Geo &g, Pt<MIX> &p) {
    bool ok;
    if constexpr (MIX) {
        unpack_cell<DIM>(r.c, p.ix, p.iy, p.iz);
        p.fx = r.ox;
        p.fy = (DIM >= 2) ? r.oy : 0.0f;
        p.fz = (DIM == 3) ? r.oz : 0.0f;
        ok = (unsigned)p.ix < (unsigned)g.nx && (p.fx >= 0.0f) && (p.fx < 1.0f);
        if constexpr (DIM >= 2) ok = ok && (unsigned)p.iy < (unsigned)g.ny && (p.fy >= 0.0f) && (p.fy < 1.0f);
        if constexpr (DIM == 3) ok = ok && (unsigned)p.iz < (unsigned)g.nz && (p.fz >= 0.0f) && (p.fz < 1.0f);
        if (!ok) { p.ix = 0; p.iy = 0; p.iz = 0; p.fx = 0.0f; p.fy = 0.0f; p.fz = 0.0f; }
    } else {
        p.x = r.x;
        double f;
        ok = cell_f64(p.x, g.inv_dx, g.nx, p.ix, f);
        p.fx = f;
        p.y = 0.0; p.iy = 0; p.fy = 0.0;
        p.z = 0.0; p.iz = 0; p.fz = 0.0;
        if constexpr (DIM >= 2) {
            p.y = r.y;
            ok = cell_f64(p.y, g.inv_dy, g.ny, p.iy, f) && ok;
            p.fy = f;
        }
        if constexpr (DIM == 3) {
            p.z = r.z;
            ok = cell_f64(p.z, g.inv_dz, g.nz, p.iz, f) && ok;
            p.fz = f;
        }
    }
    p.vx = r.vx;
    p.vy = r.vy;
    p.vz = r.vz;
    return ok;
}

inline size_t tile_e_bytes(const Geo &g, bool mixed) {
    const int ex_w = (1 << g.tsx) + 1, ey_w = (g.dim >= 2) ? (1 << g.tsy) + 1 : 1;
    const int ez_w = (g.dim == 3) ? (1 << g.tsz) + 1 : 1;
    return (size_t)ex_w * ey_w * ez_w * g.dim * (mixed ? 4 : 8);
}

// electromagnetic step: six-component field tile ((T+2)^2 each) and the
// three-component current tile ((T+3)^2 each), rounded to 16 bytes
inline size_t em_f_tile_bytes(const Geo &g, bool mixed) {
    return ((size_t)6 * ((1 << g.tsx) + 2) * ((1 << g.tsy) + 2) * (mixed ? 4 : 8) + 15) & ~(size_t)15;
}
inline size_t em_j_tile_bytes(const Geo &g) {
    return ((size_t)3 * ((1 << g.tsx) + 3) * ((1 << g.tsy) + 3) * sizeof(double) + 15) & ~(size_t)15;
}

inline size_t tile_acc_bytes(const Geo &g, int halo) {
    const int wx = (1 << g.tsx) + 1 + 2 * halo;
    const int wy = (g.dim >= 2) ? (1 << g.tsy) + 1 + 2 * halo : 1;
    const int wz = (g.dim == 3) ? (1 << g.tsz) + 1 + 2 * halo : 1;
    return (((size_t)wx * wy * wz * 8) + 15) & ~(size_t)15;
}

inline int cu_count() {
    static int cus = 0;
    if (!cus) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
            cus = 256;
    }
    return cus;
}

// Workgroups of a bucket kernel resident on one CU during a launch over
// nbuckets buckets: what its registers and LDS allow, at most the buckets'
// share of a CU.
template <typename K>
int resident_per_cu(K kernel, size_t shmem, int nbuckets, int block) {
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, block, shmem) != hipSuccess || per_cu <= 0)
        per_cu = 1;
    const int cus = cu_count();
    const int share = (nbuckets + cus - 1) / cus;
    return per_cu < share ? per_cu : share;
}

// Persistent grid: as many blocks as fit on the device at once (a multiple of
// 8 for the XCD walk), never more than the bucket count needs.
template <typename K>
int persistent_grid(K kernel, size_t shmem, int nbuckets, int block = kBlock) {
    const int cus = cu_count();
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, block, shmem) != hipSuccess || per_cu <= 0)
        per_cu = 4;
    int g = cus * per_cu;
    const int need = grid_for_buckets(nbuckets);
    if (g > need) g = need;
    return ((g + 7) >> 3) << 3;
}

}  // namespace
}  // namespace apic

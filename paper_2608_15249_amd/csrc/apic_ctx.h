// Host-side context of libapic shared by the host translation units (the
// C-ABI entry points, the adjoint): the context object, its workspace layout
// and the helpers that launch the kernels for it. Not part of the public ABI.
#pragma once

#include "apic.h"
#include "apic_index.h"
#include "apic_internal.h"
#include "apic_pages.h"

#include <hipfft/hipfft.h>

#include <string>
#include <vector>

struct apic_ctx {
    apic_grid_desc d;
    int64_t n;
    apic::Geo g;
    bool mixed;
    apic::CtxDev dev;
    void *dev_block = nullptr;
    hipfftHandle fwd = 0, inv = 0;
    bool have_fft = false;
    bool fused_fft = false;   // 2D periodic field solve by the fused three-launch path
    bool dft_field = false;   // the same on other 2D grids, lines of any length
    apic::DftPlan dft{};
    bool fused_fft3 = false;  // 3D periodic field solve by the fused transforms in LDS
    std::string err;
    // workspace layout (byte offsets)
    size_t o_x, o_y, o_z, o_cell, o_ox, o_oy, o_oz, o_vx, o_vy, o_vz;
    size_t o_bstart, o_acc, o_rho, o_rhat, o_ehat;
    size_t o_jacc;    // electromagnetic step: J [2][3][G] (two buffers)
    size_t o_f2;      // electromagnetic step: the second field buffer [6][G]
    size_t o_e32;     // mixed electrostatic step in 2D and 3D: E between steps, binary32 [dim][G]
    size_t o_cnt, o_offs, o_farcnt, o_farcur, o_tot, o_deep;
    size_t o_idx, o_rcnt, o_rpart;
    // paged storage of calls of several steps (npages = 0: not used by this context);
    // it shares the front of the workspace with the arrays that only the sort
    // and the reordering step use
    int64_t npages = 0;
    size_t o_pool, o_out, o_ptab, o_pqueue, o_phead, o_praw, o_phole, o_pcode, o_porder, o_pfar, o_pfarhead, o_plcnt, o_ploff,
        o_pcnt, o_pds, o_pps;
    size_t ws_bytes;
    size_t ws_step_bytes;     // the workspace without the paged storage's part beyond the shared front
    double dV, mass;
    // per-phase timing (apic_profile_enable)
    std::vector<hipEvent_t> ev;   // 5 events per profiled step
    int prof_max = 0, prof_used = 0;
    bool prof_all = true;          // events around every phase, or only around the push pass
    std::vector<char> ev_paged;    // whether a profiled step kept the particles in place (no count pass)
    int prof_every = 1;            // events on one step in prof_every
    int64_t prof_step = 0;         // steps seen since profiling was armed
};

namespace apic_host {

using apic::Parts;
using apic::PushC;

apic_status fail(apic_ctx *c, apic_status st, const char *msg);
apic_status hip_fail(apic_ctx *c, hipError_t e, const char *where);

#define HIPCHK(ctx, expr)                                   \
    do {                                                    \
        hipError_t e_ = (expr);                             \
        if (e_ != hipSuccess) return hip_fail(ctx, e_, #expr); \
    } while (0)

#define FFTCHK(ctx, expr)                                                    \
    do {                                                                     \
        hipfftResult r_ = (expr);                                            \
        if (r_ != HIPFFT_SUCCESS) {                                          \
            (ctx)->err = std::string(#expr) + " failed (" + std::to_string((int)r_) + ")"; \
            return APIC_EHIP;                                                \
        }                                                                    \
    } while (0)

inline size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// Pointer at a byte offset of the workspace (NULL for an absent array).
template <typename T>
T *wsp(void *ws, size_t off) {
    return off == (size_t)-1 ? nullptr : (T *)((char *)ws + off);
}

Parts parts_of(const apic_particles *p);
Parts parts_ws(const apic_ctx *c, void *ws);
apic_status check_parts(apic_ctx *c, const apic_particles *p, bool need_bstart);
PushC push_coeffs(const apic_ctx *c, double dt_scale, int move);
double acc_scale(const apic_ctx *c);
int64_t max_per_bucket(const apic_ctx *c);
apic_status field_from_acc(apic_ctx *c, void *acc, bool acc_is_rho, double *E, float *E32, double *diag,
                           double *we, double *charge, int npush, int clear, void *ws, hipStream_t s,
                           const int32_t *nlive = nullptr);
// Paged storage of a call's step k in the workspace ws, and the launches that start a call: acc (nacc 64-bit words) is
// what the first push adds to.
apic::PageStep page_step(const apic_ctx *c, void *ws, int k);
apic_status page_begin(apic_ctx *c, const int32_t *bstart, void *acc, int64_t nacc, void *ws, hipStream_t s);
// Events of the step about to run (NULL: not profiled); paged: it keeps the particles in place.
hipEvent_t *profile_events(apic_ctx *c, bool paged);
// Particles, bucket table and field of one time level, in arrays of the caller's choice.
struct Level {
    Parts parts;
    int32_t *bstart;
    double *E;
};
// Steps from lv[0] to lv[m], each level left where lv says; perm[k]: the
// reordering of step k (as apic_particles::perm).
apic_status run_levels(apic_ctx *c, const Level *lv, int m, int32_t *const *perm, void *ws, hipStream_t s);
apic_status copy_parts(apic_ctx *c, const Parts &dst, const Parts &src, hipStream_t s);

}  // namespace apic_host

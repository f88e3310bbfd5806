// Paged particle storage of a call of several steps (apic_pages.hip): the
// tables of one step and the launchers. Not part of the public ABI.
#pragma once

#include "apic_internal.h"

namespace apic {

// Particle slots of a page: what a wave reads and writes at a time, 1.5 KiB (mixed
// 1D1V) to 6 KiB (FP64 3D3V).
// Pages of 256 were slower where they are a power of two of bytes (FP64 2D2V,
// 8 KiB: the push at 512 x 512, 16.8M particles 276 us against 235) and a
// little slower elsewhere (mixed 2D3V, 6 KiB: 350 against 345 us at 1024 x 1024,
// 33.5M).
constexpr int kPage = 128;
constexpr int kPagePushMax = 512;  // threads of a push workgroup, at most
// Chains of a bucket's far arrivals, one per lane of the wave that walks them: a
// bucket reads its own arrivals alone, and the chain a leaver joins (its lane's)
// keeps the heads' atomics apart.
constexpr int kFarChains = 64;

// The leavers of one step, bucket by bucket (a bucket's entries start at its ds).
struct PageList {
    int32_t *cnt, *off;       // [nb][directions] leavers, the first one's place in the bucket's list
    int32_t *hole, *order;    // [n] their slots and outbox entries in direction order
    // those bound beyond the neighbours, chained by destination: chain c of bucket
    // b starts at far_head[b * kFarChains + c] and goes on at far_next[entry]; both
    // hold an outbox entry + 1, 0 at the end
    int32_t *far_head;        // [nb][kFarChains], zero once read
    int32_t *far_next;        // [n], by outbox entry
    char *out;                // [out_slots] outbox, in pieces as the pages
};

// What the push of one step sees. The buckets as the step before found them
// (_old) and as its leavers leave them (cnt is complete when the push starts,
// ds, ps and tab are its own work), and the counts it adds to for the next
// step. The host rotates the buffers.
struct PageStep {
    int32_t *cnt_old;                // [nb] particles, cleared once read
    const int32_t *cnt;
    int32_t *cnt_next;               // zero at the start
    const int32_t *ds_old;           // [nb + 1] sums of the counts before: the bucket's first list and dense entry
    int32_t *ds;
    const int32_t *ps_old;           // [nb + 1] sums of the pages before: the bucket's first page-table entry
    int32_t *ps;
    const int32_t *tab_old;          // [npages] page table: pool page of each page-table entry
    int32_t *tab;
    int32_t *queue;                  // [npages] ring of free pages
    unsigned long long *head;        // [2] pages taken from and given to the ring so far
    int64_t npages;
    int scanned;                     // ds and ps are k_page_scan's work already
    int32_t *live;                   // [1] particles not absorbed by a wall
    int32_t *done;                   // [1] buckets whose 1D push has ended, zero between the steps
    char *pool;                      // [npages] pages
    int64_t out_slots;               // n rounded up
    // this launch's own scratch, a bucket's part where its entries of ds start
    int32_t *raw_slot;               // [n] the leavers' slots, as listed (their state: the same entries of
                                     // to.out); during the exchange the holes that a shrinking bucket keeps
    uint8_t *raw_code;               // [n] their directions, as listed
    PageList in, to;                 // leavers of the step before, of this one
};

// The 1D field solve inside the push (E set): the workgroup that ends last solves
// it, with the step's diagnostics, from the charge that all have added.
struct PageField {
    double *E;
    float *E32;                       // or NULL
    double *diag;                     // or NULL
    double scale, ion, dx, q_macro, mass;
};

// Whether the push can take the field solve along: 1D, the nodes held in LDS
// beside the workgroups of a whole chip.
inline bool page_field_folds(const Geo &g) { return g.dim == 1 && g.nx <= 2048; }

// Brings the kernels of this file onto the device, which their first launch would
// do otherwise.
hipError_t load_page_kernels();
// t: the call's first step, head2 [2][nb][kFarChains]: the chain heads of both sides
hipError_t launch_page_begin(const Geo &g, const PageStep &t, int32_t *cnt3, int32_t *head2, int64_t n,
                             int64_t max_per_bucket, const int32_t *bstart, uint64_t *acc, int64_t nacc,
                             const CtxDev &c, hipStream_t s);
// src: the caller's arrays (with bstart) in a call's first step, else NULL
hipError_t launch_page_push(const Geo &g, bool mixed, const PageStep &t, const Parts *src, const int32_t *bstart,
                            int64_t n, int64_t max_per_bucket, const double *E, const float *E32, const PushC &pc,
                            void *acc, double *part, const PageField &f, const CtxDev &c, hipStream_t s);
hipError_t launch_page_end(const Geo &g, bool mixed, const PageStep &t, int64_t n, int64_t max_per_bucket,
                           const Parts &dst, int32_t *bstart, const CtxDev &c, hipStream_t s);

}  // namespace apic

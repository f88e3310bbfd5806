// Rules that are plain functions of counts, without any HIP type, so that the
// CPU tests can go through them: which calls keep the particles in pages, the
// indices of kernels whose rounds start before a bucket's first particle or end
// behind its last, and the work split of the 3D field solve.
#pragma once

namespace apic {

// Calls of at least this many steps keep the particles in pages between the
// steps: what a step saves then pays for the first push, which reads the
// caller's arrays, and for the copy at the call's end. us per step of calls of 7
// steps, which reorder, of 8 and of 20: 16384 mixed particles in 1D 31.1, 24.1 and
// 23.1, 0.52M in 2D 53.2, 41.1, 40.1, 2.1M in 3D 114, 88.9, 85.5, electromagnetic
// 2.1M 201, 100, 96.6; the largest gain least: 16.8M in 2D mixed 243, 213, 197, FP64 346, 309,
// 290 (at tiles of 32 x 16 they lose 3% at 8 steps and gain 4% at 20).
constexpr int kPagedSteps = 8;

// Copy of a paged bucket back to the caller's arrays (k_page_end): rounds of
// `width` places, the first from the line boundary `ahead` places before the
// bucket's own first one. An empty bucket has no round: it has no page either.
constexpr int copy_rounds(int count, int ahead, int width) {
    return count > 0 ? (int)(((unsigned)count + (unsigned)ahead + (unsigned)width - 1) / (unsigned)width) : 0;
}

// The particle read for place k of such a round (count > 0): the nearest one
// of the bucket where k lies outside it.
constexpr int copy_slot(int k, int count) { return k < 0 ? 0 : k < count ? k : count - 1; }


// The particle loaded for place k of the bucket of `count` particles from
// `first` on (tiled deposit and gather + push, several places ahead of their
// use). k is unsigned and counts from the bucket's start: there are up to
// 2^31 - 2 particles, and the places run past a bucket by a round.
constexpr int ahead_index(int first, unsigned k, unsigned count) { return first + (int)(k < count ? k : count - 1); }

// Work split of the 3D field solve's launches (powers of two): rows per x
// workgroup, planes per y workgroup, ky values per z workgroup.
struct Split3 {
    int Y, ZB, KY;
};

// Small workgroups, several to a CU, so that the loads of some overlap the passes
// of others: about 512 points each (two per thread), in at least 8 rows or 4 lines
// (64-byte runs in the y launches) and at most 16, or 8 on grids so small that the
// chip is short of workgroups. Lines shorter than 128 points take more than the
// least: with 8 rows, 4 planes and 4 ky for every grid, threads were left without a
// point. Solve and gradient, mixed, us, with (16 rows, or 8 from 256 points per row
// on; 8 planes; 8 ky, or 4 above 128 planes) / (8; 4, or 8 above 128 planes; 4) /
// this rule: 128^3 92.7, 90.6, 90.0; 32^3 25.8, 25.7, 25.7 (26.4 with 16); 256 x 64 x
// 32 46.6, 52.3, 44.5; 64 x 256 x 32 51.0, 56.9, 50.1; 32 x 64 x 256 55.7, 58.5, 54.4;
// 128 x 128 x 32 48.0, 52.7, 47.0; 256 x 256 x 64 153, 164, 151; 16 x 256 x 256 103,
// 108, 91; 256^3 (8 planes for its longer runs along z) 580, 583, 583.
constexpr int split_lines(int wanted, int least, int cap, int most) {
    const int n = wanted < least ? least : wanted > cap ? cap : wanted;
    return n < most ? n : most;
}
constexpr Split3 split3_of(int nx, int ny, int nz) {
    const int cap = nx * ny * nz <= 32768 ? 8 : 16;
    return Split3{split_lines(1024 / nx, 8, cap, ny),   // (two rows to a line)
                  split_lines(512 / ny, nz <= 128 ? 4 : 8, cap, nz), split_lines(512 / nz, 4, cap, ny)};
}

}  // namespace apic

// Rules that are plain functions of counts, without any HIP type, so that the
// CPU tests can go through them: which calls keep the particles in pages, and
// the indices of kernels whose rounds start before a bucket's first particle or
// end behind its last.
#pragma once

namespace apic {

// Calls of at least this many steps keep the particles in pages between the
// steps: what a step saves then pays for the copy at the call's end.
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

}  // namespace apic

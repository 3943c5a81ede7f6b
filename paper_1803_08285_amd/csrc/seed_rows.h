// Which segments the matrix-core dirty map's operand slots hold: host arithmetic
// shared with the kernels.
//
// A chunk has 16 slots, eight per half-wave (half 0 and 1, slot e = 0 .. 7), and a
// day of nt segments ceil(nt / 16) chunks.  Every slot reads a row of the seeds, so
// every row has to lie inside them: the last chunk's window is the day's last 16
// segments, and for days shorter than that the halves overlap.  A segment that an
// earlier slot holds already has zero data-side operands (slot_is_new), which a
// finite seed turns into exactly nothing; a seed that is not finite spoils its
// pixel in its own slot already.
#pragma once

#include <stdint.h>

namespace sgwb {

constexpr int kXmT = 16;        // segments per chunk (MFMA K)
constexpr int kXmHalf = kXmT / 2;

// First row of the chunk's window.
constexpr int64_t chunk_row(int32_t nt, int64_t chunk)
{
    const int64_t last = nt > kXmT ? nt - kXmT : 0, first = chunk * kXmT;
    return first < last ? first : last;
}

// Rows from the lower half's first to the upper half's first.
constexpr int32_t half_row(int32_t nt) { return nt >= kXmT ? kXmHalf : nt > kXmHalf ? nt - kXmHalf : 0; }

// Rows from a half's first to its slot e: e itself, or where the day has fewer than
// eight segments (XmArgs::ext) the last one again.
constexpr int32_t slot_row(int32_t nt, int32_t e) { return e < nt ? e : nt - 1; }

// Whether slot (half, e) of a chunk is the one that holds its segment.
constexpr bool slot_is_new(int32_t nt, int64_t chunk, int32_t half, int32_t e)
{
    const int64_t first = chunk_row(nt, chunk), t = first + half * half_row(nt) + e;
    return e < nt && t >= chunk * kXmT && (half == 0 || t >= first + kXmHalf);
}

}  // namespace sgwb

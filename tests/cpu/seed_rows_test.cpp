// The segments of the matrix-core dirty map's operand slots: every row read lies in
// the day, every segment has exactly one slot, and a row a slot repeats is one
// that an earlier slot holds.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "seed_rows.h"

using namespace sgwb;

int main()
{
    for (int32_t nt = 1; nt <= 1200; ++nt) {
        std::vector<int> held(nt, 0);
        const int64_t chunks = (nt + kXmT - 1) / kXmT;
        for (int64_t ch = 0; ch < chunks; ++ch)
            for (int32_t half = 0; half < 2; ++half)
                for (int32_t e = 0; e < kXmHalf; ++e) {
                    const int64_t row = chunk_row(nt, ch) + half * half_row(nt) + slot_row(nt, e);
                    const bool fresh = slot_is_new(nt, ch, half, e);
                    if (row < 0 || row >= nt || (!fresh && !held[row])) {
                        std::printf("nt %d chunk %lld half %d slot %d: row %lld\n", nt, (long long)ch, half, e,
                                    (long long)row);
                        return 1;
                    }
                    if (fresh) {
                        // the data side takes the unclamped row
                        if (slot_row(nt, e) != e || held[row]++) return 1;
                    }
                }
        for (int h : held)
            if (h != 1) {
                std::printf("nt %d: a segment is held %d times\n", nt, h);
                return 1;
            }
    }
    // the window of a chunk spans at most 16 rows (32-bit offsets)
    for (int32_t nt = 1; nt <= 64; ++nt)
        if (half_row(nt) + slot_row(nt, kXmHalf - 1) >= kXmT) return 1;
    std::printf("all checks passed\n");
    return 0;
}

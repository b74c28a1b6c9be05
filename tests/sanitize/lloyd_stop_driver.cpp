// The stop of the device codebook training as its launches see it: a wave of a launch may read the state before or after the
// launch's one writer has written, and has to go the same way.  The exit status is what the test reads.
#include <cstdio>

#include "qamw_lloyd_stop.hpp"

using namespace qamw;

static int fails = 0;
#define EXPECT(c) do { if (!(c)) { std::printf("FAILED: %s (line %d, iterations %d, stop after %d, launch %d)\n", #c, __LINE__, launched, last, t); ++fails; } } while (0)

int main() {
    // `launched` iterations are queued; the error settles in iteration `last` (beyond the queue: not yet)
    for (int launched = 1; launched <= 40; ++launched)
        for (int last = 0; last <= launched; ++last) {
            LloydState s = lloyd_begin();
            for (int t = 0; t < launched; ++t) {
                const bool before = lloyd_seen_by_table(s, t) == LC_RUNNING;
                lloyd_table_decides(s, t, t - 1 == last);
                const bool after = lloyd_seen_by_table(s, t) == LC_RUNNING;
                EXPECT(before == after);                        // an early and a late wave of the table launch
                EXPECT(before == (t - 1 <= last));              // the launch that decides still runs, later ones return
                EXPECT((lloyd_seen_by_assignment(s, t) == LC_RUNNING) == (t <= last));
                EXPECT(lloyd_seen_by_assignment(s, t) == (t <= last ? LC_RUNNING : last));
            }
        }
    if (fails == 0) std::printf("lloyd stop driver ok\n");
    return fails != 0;
}

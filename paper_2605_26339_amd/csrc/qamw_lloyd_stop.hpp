// What the launches of the device codebook training know of the stop, and when.  Plain C++, so that it runs on the CPU too.
//   Iteration t is a table launch and an assignment.  The table launch decides whether iteration t - 1 was the last, while its
// other waves ask whether to run at all: so a launch never writes the word that it reads.  Table launch t reads the word of the
// other parity, which launch t - 1 left, and writes its own; assignment t reads that.  All waves of a launch go the same way.
#pragma once

namespace qamw {

constexpr int LC_RUNNING = 0x7fffffff;
struct LloydState {
    double D[2];                          // mean squared error of iteration t in D[t mod 2]
    int stopped_at[2];                    // the last iteration, LC_RUNNING before it is known; table launch t writes [t mod 2]
    int last;                             // the same for the host, written after the launches that it has queued
};

constexpr LloydState lloyd_begin() { return {{0.0, 0.0}, {LC_RUNNING, LC_RUNNING}, LC_RUNNING}; }
// the last iteration, as far as table launch t and assignment t know it: they return unless it is LC_RUNNING
constexpr int lloyd_seen_by_table(const LloydState &s, int t) { return s.stopped_at[(t + 1) & 1]; }
constexpr int lloyd_seen_by_assignment(const LloydState &s, int t) { return s.stopped_at[t & 1]; }
// by one thread of table launch t, whatever the launch has seen.  stops: iteration t - 1 was the last
constexpr void lloyd_table_decides(LloydState &s, int t, bool stops) {
    const int seen = lloyd_seen_by_table(s, t);
    s.stopped_at[t & 1] = seen != LC_RUNNING ? seen : stops ? t - 1 : LC_RUNNING;
}

}  // namespace qamw

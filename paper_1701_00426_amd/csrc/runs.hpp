// runs.hpp -- how many iterations of a solve are queued between two looks at its flags, and
// whether such a run ends with the true-residual update.  Host arithmetic only.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace stg {

// Shortest run that ends with the update.
constexpr int kQueuedRun = 8;

// Whether every run of iterations ends with the true-residual update, queued without a
// look at the flags (its kernels leave at once when no system is parked): mixed solves on
// small lattices, whose systems park every few dozen iterations.  Left to the host, each
// update waited for up to two runs of iterations that had nothing to do, 7 us each: 311
// iterations of 4^4 with 11 updates took 14.3 ms with runs of 64 iterations and 5.4 with
// the update in runs of 12; 16^4 with BF16-12 links 23.5 and 10.1; 8^4 with 4 RHS 28.5 and
// 11.3 (7.9 with the per-field vector kernels since).
// On larger lattices the five idle launches cost more than the wait, and so they do when the
// caller asks for runs of a few iterations, after which the host sees a parked system soon
// enough.  poll_every = 1 / 2 / 4 / 6 / 8 / 16, ms with the host's update | with the update
// in every run: 4^4 12.5 10.8 10.0 10.1 10.2 10.8 | 22.5 15.1 11.6 10.8 10.3 9.8; 8^4, 4 RHS,
// 20.6 18.3 17.8 17.6 18.6 19.2 | 29.8 22.3 19.2 18.3 17.2 16.2; 16^4 20.7 19.1 18.8 19.1
// 19.0 19.9 | 29.7 22.3 19.3 18.7 18.1 17.7.
// site_fields: half sites times the systems that have not finished.
inline bool queued_update(int poll_every, bool mixed, uint64_t site_fields) {
    if (poll_every > 0 && poll_every < kQueuedRun) return false;
    return mixed && site_fields <= (1u << 17);
}

// Iterations queued between two looks at the flags.  A look costs a copy of a few bytes
// (4 us on the stream); a system that has parked or converged waits for one to two runs.
// Small lattices: 12 with the update in the run, else 8 (mixed) or 16 (FP64, where only
// the end of a system waits); a large one about 4 million site updates, at least 8.
// Several systems share launches that go on with their fields while they wait, so there a
// run is 2 million site-field updates, at least 2 iterations (16 shifts x 2 RHS at 24^3 x
// 48: 328 ms with at least 4 and twice the work, 324 so; 16^4, 12 x 3: 52.0 and 49.1).
inline int run_iterations(int poll_every, bool with_update, bool mixed, uint32_t Vh, int live) {
    if (poll_every > 0) return poll_every;
    if (with_update) return 12;
    const uint32_t most = mixed ? 8 : 16;
    if (live > 1) {
        const uint32_t work = (1u << 21) / Vh / (uint32_t)live;
        return (int)std::min<uint32_t>(most, std::max<uint32_t>(2, work));
    }
    return (int)std::min<uint32_t>(most, std::max<uint32_t>(8, (1u << 22) / Vh));
}

// Batches.  Small ones (all tiles' hop passes in one merged launch) end every replay of at
// least kQueuedRun iterations with the true-residual update of the systems parked by then.
// Its kernels leave the tiles without a parked system alone, so a replay that parks none
// pays for five launches, and a parked system waits for the end of its replay; with the
// update launched by the host it waits for the next replay too, and the update drains the
// stream (16 solves of 8^4 to 16^4: 816 iterations of the batch instead of about 660).
// Large batches keep the host's update: there the five launches over every tile cost 1 %
// (1.250 s against 1.238 for 12 solves up to 32^4) and the wait is hidden by the other
// solves.  So do shorter replays that the caller asks for: poll_every = 1 / 2 / 4 / 6 / 8 /
// 16, ms with the host's update | with it in the replay, the 16 solves: 33.4 28.3 25.9 27.7
// 25.9 27.1 | 37.2 30.4 27.3 26.9 25.0 24.4.
inline bool batch_queued_update(int run, bool small_batch) {
    return run >= kQueuedRun && small_batch;
}

// Iterations per replay of the batch's graph.
inline int batch_run(int poll_every, bool small_batch) {
    if (poll_every > 0) return poll_every;
    return small_batch ? kQueuedRun : 16;
}

}  // namespace stg

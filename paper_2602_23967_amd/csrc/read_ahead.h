// read_ahead.h -- results of a batch on their way to the caller: instances
// fetched in their order come from the device in blocks.  No HIP types (a
// test drives it on the CPU).
#pragma once

#include <stdint.h>

#include <algorithm>
#include <mutex>
#include <new>
#include <vector>

namespace pdhcg {

// A copy to the host takes 25 us however short it is, and two for each of
// 4096 MPC problems were 213 ms after a solve of 23; in blocks of READ_AHEAD
// doubles fetching them all is 44 ms, most of it the caller's.  Any other
// order copies what is asked for alone.
constexpr int64_t READ_AHEAD = 1 << 18;   // doubles in a block at most (2 MiB)

struct ReadAhead {
    std::mutex lock;
    int64_t i0 = 0, i1 = 0, next = 1;   // instances held; the one after the last one asked for
    std::vector<double> x, y;

    void drop()
    {
        std::lock_guard<std::mutex> hold(lock);
        i0 = i1 = 0;
        next = 1;
    }

    // x and y (either may be NULL) of instance i of `count`, whose values are
    // [voff[i], voff[i + 1]) and [roff[i], roff[i + 1]).  fetch(a, b, x, y)
    // brings those of the instances [a, b) and returns 0 or an error code; it
    // may throw std::bad_alloc for more than one instance.
    template <class Fetch>
    int get(int64_t i, int64_t count, const int64_t* voff, const int64_t* roff, double* xi, double* yi, Fetch fetch)
    {
        std::lock_guard<std::mutex> hold(lock);
        bool held = i >= i0 && i < i1;
        int64_t e = i + 1;
        if (!held && i == next)
            while (e < count && voff[e + 1] - voff[i] + roff[e + 1] - roff[i] <= READ_AHEAD) ++e;
        if (e > i + 1) {
            i0 = i1 = 0;
            try {
                x.resize((size_t)(voff[e] - voff[i]));
                y.resize((size_t)(roff[e] - roff[i]));
                if (int rc = fetch(i, e, x.data(), y.data())) return rc;
                i0 = i;
                i1 = e;
                held = true;
            } catch (const std::bad_alloc&) {
                // no room on the host: this instance alone
            }
        }
        if (held) {
            if (xi) std::copy_n(x.data() + (voff[i] - voff[i0]), voff[i + 1] - voff[i], xi);
            if (yi) std::copy_n(y.data() + (roff[i] - roff[i0]), roff[i + 1] - roff[i], yi);
        } else if (int rc = fetch(i, i + 1, xi, yi)) {
            return rc;
        }
        next = i + 1;
        return 0;
    }
};

}  // namespace pdhcg

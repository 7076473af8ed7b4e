// Whether the tasks of a map call may run in any order: the condition under
// which sparkcl_map runs them all in one launch.  Host logic without HIP.
#pragma once

#include <algorithm>
#include <cstdint>
#include <vector>

#include "sparkcl.h"

namespace sparkcl {

// True when no task's output shares memory with another task's arrays.
inline bool tasks_independent(const sparkcl_task *tasks, uint32_t ntasks)
{
    // The arrays as byte ranges, by start.  Sweeping them, a range conflicts
    // with an earlier one of another task that ends past its start when
    // either is an output; of the earlier ranges only the furthest end and
    // the furthest end of a second task matter, for outputs and for all.
    struct Range {
        uintptr_t lo, hi;
        uint32_t task;
        bool out;
    };
    std::vector<Range> r;
    r.reserve(3 * (size_t)ntasks);
    for (uint32_t i = 0; i < ntasks; ++i) {
        const sparkcl_task &t = tasks[i];
        if (t.n == 0)
            continue;
        const uintptr_t bytes = (uintptr_t)t.n * 4;
        const float *arr[3] = {t.in0, t.kernel_id == SPARKCL_FMUL ? t.in1 : nullptr, t.out};
        for (int a = 0; a < 3; ++a)
            if (arr[a])
                r.push_back({(uintptr_t)arr[a], (uintptr_t)arr[a] + bytes, i, a == 2});
    }
    std::sort(r.begin(), r.end(), [](const Range &a, const Range &b) { return a.lo < b.lo; });
    struct Ends {
        uintptr_t hi[2] = {0, 0}; // the furthest end, and another task's furthest
        uint32_t task = 0;        // of the furthest
        uintptr_t beyond(uint32_t t) const { return hi[task == t ? 1 : 0]; }
        void add(const Range &x)
        {
            if (x.task == task || hi[0] == 0) {
                task = x.task;
                hi[0] = std::max(hi[0], x.hi);
            } else if (x.hi > hi[0]) {
                hi[1] = hi[0];
                hi[0] = x.hi;
                task = x.task;
            } else {
                hi[1] = std::max(hi[1], x.hi);
            }
        }
    } outs, all;
    for (const Range &x : r) {
        if ((x.out ? all : outs).beyond(x.task) > x.lo)
            return false;
        all.add(x);
        if (x.out)
            outs.add(x);
    }
    return true;
}

} // namespace sparkcl

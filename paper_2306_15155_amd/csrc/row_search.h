// One wavefront's search for the first place of an ascending array of n + 1 numbers whose value reaches a target: the range is narrowed
// 65-fold a round by one look of every lane.  Host and device, so that its places can be checked where nothing faults.
#pragma once

namespace sensei {

struct RowSearch {
    int lo, hi;   // row_ptr[lo - 1] < target (or lo = 0), row_ptr[hi] >= target (or hi = n); found where they meet
    __host__ __device__ bool open() const { return lo < hi; }
    __host__ __device__ int step() const { return (hi - lo + 64) / 65; }
    // Where a lane looks, always in [0, n]; at `hi` there is nothing to look at (past the range, or the search is over: the other end of a
    // chunk may take a round longer, and a closed range has no place before it to look at).
    __host__ __device__ int place(int lane) const {
        const int p = lo + step() * (lane + 1) - 1;
        return open() && p < hi ? p : hi;
    }
    // `smaller` lanes, the first ones, found values below the target
    __host__ __device__ void narrow(int smaller) {
        if (!open()) return;
        const int s = step();
        lo += s * smaller;
        if (smaller < 64 && lo + s - 1 < hi) hi = lo + s - 1;   // the look after the last smaller one bounds the place from above, if there is one
        if (lo > hi) lo = hi;
    }
};

}  // namespace sensei

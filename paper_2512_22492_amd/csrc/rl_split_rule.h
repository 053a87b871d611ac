// rl_split_rule.h -- how a decode handle divides a sequence into splits.  Plain
// integer functions of the handle and of a sequence's length, for the host and
// the device.

#pragma once

#include <stdint.h>

#if defined(__HIP__)
#define RL_HD __host__ __device__
#else
#define RL_HD
#endif

namespace rl_da {

// How a sequence's pages are divided.  Every split takes `pages` and the last one
// what is left; of a handle that splits by length, sequences of more than
// `whole` pages are cut evenly instead, into splits of about min_pages, `most` of
// them at most, or as few as hold the sequence where those are more.  A
// function of the sequence's own length and of the handle, never of the batch.
struct SplitRule {
    int32_t pages;      // the handle's split size
    int32_t min_pages;  // == pages: no even cut; else pages / 2 at most
    int32_t whole;      // a sequence of one page more has two splits at least
    int32_t most;       // no more than a sequence that fills the handle's table has
    RL_HD bool by_length() const { return min_pages != pages; }
    // a sequence's splits: also the most of any sequence that is no longer
    RL_HD int splits_of(int npages) const
    {
        const int n = (npages + pages - 1) / pages;
        if (!by_length() || npages <= whole)
            return n;
        const int fine = (npages + min_pages / 2) / min_pages;
        const int m = fine < most ? fine : most;
        return m > n ? m : n;
    }
    // pages of each split but the last
    RL_HD int pages_of(int npages) const
    {
        if (!by_length() || npages <= whole)
            return pages;
        const int n = splits_of(npages);
        return (npages + n - 1) / n;
    }
};

}  // namespace rl_da

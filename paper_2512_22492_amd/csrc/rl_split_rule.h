// rl_split_rule.h -- how a decode handle divides a sequence into splits, and in
// which order a launch takes them.  Plain integer functions of the handle and
// of a sequence's length, for the host and the device.

#pragma once

#include <stdint.h>

#if defined(__HIP__)
#define RL_HD __host__ __device__
#else
#define RL_HD
#endif

namespace rl_da {

// Classes of split sizes, longest first; a launch takes its units by class.
constexpr int kLengthClasses = 8;

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

// Class of a split of `n` pages: 0 for one of the handle's split size, rising as
// it gets shorter; an empty sequence's is the last.
RL_HD inline int length_class(int pages, int n)
{
    return (pages - n) * kLengthClasses / (pages + 1);
}

// What the plan of a launch holds of a sequence of npages pages, on a handle that
// splits by length: its full splits (none of a sequence of one split) and its
// last one, each with the class it is taken in.  An empty sequence counts one
// split, whose unit writes its zeros.
struct PlanShape {
    int pages;     // of each split but the last
    int full;      // splits before the last one
    int full_cls;
    int last_cls;
    RL_HD PlanShape(const SplitRule& r, int npages) : pages(r.pages_of(npages))
    {
        const int n = (npages + pages - 1) / pages;
        full = n > 1 ? n - 1 : 0;
        full_cls = length_class(r.pages, pages);
        last_cls = length_class(r.pages, npages - full * pages);
    }
};

// An entry of that plan in 32 bits: the sequence, the pages of its splits and the
// number of the entry's first split.
constexpr int kPlanBatchByLength = 128;  // sequences a plan by length can hold
constexpr int kPlanSplitsByLength = 1 << 11;  // splits of a sequence
RL_HD inline int pack_entry(int b, int pages, int split)
{
    return (int)((uint32_t)split << 19 | (uint32_t)pages << 10 | (uint32_t)b);
}
RL_HD inline void unpack_entry(int entry, int& b, int& pages, int& split)
{
    b = entry & 1023;
    pages = entry >> 10 & 511;
    split = (int)((uint32_t)entry >> 19);
}

}  // namespace rl_da

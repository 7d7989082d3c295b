// What the host layer checks of a call's buffers, for every entry point. Host code only.
#ifndef LASP_CHECKS_H
#define LASP_CHECKS_H

#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <initializer_list>
#include <new>
#include <vector>

#include "../../include/lasp.h"
#include "lasp_internal.h"

namespace lasp {

inline size_t elem_bytes(int dtype) { return dtype == LASP_F32 ? 4 : 2; }

struct Span {
    const void *p;
    size_t n;
};
inline bool overlap(Span a, Span b) {
    const char *x = (const char *)a.p, *y = (const char *)b.p;
    return x && y && x < y + b.n && y < x + a.n;
}

inline bool overlap_any(Span a, std::initializer_list<Span> others) {
    for (const Span &x : others)
        if (overlap(a, x)) return true;
    return false;
}

// Outputs must not overlap inputs or each other, and the kernels move data in 16-byte pieces.
// NULL (an absent optional buffer) passes both checks.
inline int check_buffers(std::initializer_list<Span> ins, std::initializer_list<Span> outs) {
    for (const Span &x : ins)
        if ((uintptr_t)x.p % 16 != 0) return LASP_ERR_ALIGN;
    for (const Span &x : outs)
        if ((uintptr_t)x.p % 16 != 0) return LASP_ERR_ALIGN;
    for (const Span &o : outs) {
        for (const Span &i : ins)
            if (overlap(o, i)) return LASP_ERR_ALIAS;
        for (const Span &o2 : outs)
            if (&o != &o2 && overlap(o, o2)) return LASP_ERR_ALIAS;
    }
    return LASP_OK;
}

// Whether sub-sequences can share a launch: no output of one may touch another's buffers (in a loop over them that is the
// caller's affair: the later call reads what the earlier one wrote, or writes over it).
class Together {
    struct Item {
        const char *begin, *end;
        bool out;
    };
    std::vector<Item> items;
    bool full = false;   // no memory to note them all: not together, then
    void note(const void *p, size_t n, bool out) {
        if (!p || full) return;
        try {
            items.push_back({(const char *)p, (const char *)p + n, out});
        } catch (const std::bad_alloc &) {
            full = true;
        }
    }

public:
    void in(const void *p, size_t n) { note(p, n, false); }
    void out(const void *p, size_t n) { note(p, n, true); }
    bool disjoint() {
        if (full) return false;
        std::sort(items.begin(), items.end(), [](const Item &a, const Item &b) { return a.begin < b.begin; });
        const char *any_end = nullptr, *out_end = nullptr;   // ends of what has begun so far
        for (const Item &x : items) {
            if (x.begin < out_end || (x.out && x.begin < any_end)) return false;
            any_end = std::max(any_end, x.end);
            if (x.out) out_end = std::max(out_end, x.end);
        }
        return true;
    }
};

// The bidirectional calls' plan (lasp_api.cpp), and the next record of the diagnostic profiler, if it is on (kind: 0 forward,
// 1 backward).
int make_bidir_plan(const lasp_shape *s, BidirPlan *p);
size_t bidir_scratch(const BidirPlan &p);
const KernelEvents *next_slot(int kind);

}  // namespace lasp
#endif

// The destination checks of a load that need only the addresses: kept apart
// from the HIP queries that complete them so that the two ways to make them
// can be compared on the host.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <vector>

#include "ii_internal.h"

namespace ii {

// Whether dst is the plan's own layout at one address: dst[i] = *base +
// dst_offset[i] for every non-empty tensor, what a caller that carves one
// arena passes. Such destinations need no further look one by one: the
// layout is disjoint and in order, every offset is a multiple of its
// tensor's alignment, so all are aligned when the base is a multiple of the
// largest one, and all lie in [*base, *end). False for anything else --
// other destinations, NULL, a base that leaves a tensor misaligned, a range
// past 2^64 -- which dst_ranges then accepts or reports. One pass over two
// arrays, against a sort and a range per tensor there.
inline bool arena_base(const ii_plan_s* p, const uint64_t* dst, uint64_t* base, uint64_t* end) {
    const size_t n = p->nbytes.size();
    if (p->first_live >= n) return false;
    const uint64_t b = dst[p->first_live] - p->dst_offset[p->first_live];
    if (!b || (b & (p->live_align - 1))) return false;
    if (__builtin_add_overflow(b, p->layout_end, end)) return false;
    uint64_t off = 0;
    if (p->has_empty) {  // an empty tensor's pointer is not read
        for (size_t i = 0; i < n; ++i)
            off |= p->nbytes[i] ? dst[i] - p->dst_offset[i] - b : 0;
    } else {
        for (size_t i = 0; i < n; ++i) off |= dst[i] - p->dst_offset[i] - b;
    }
    *base = b;
    return off == 0;
}

// Destination ranges of the non-empty tensors, sorted by address, after
// checking that each is present, aligned and disjoint from the others.
inline int dst_ranges(const ii_plan_s* p, const uint64_t* dst, std::vector<DstRange>* out) {
    const size_t n = p->nbytes.size();
    std::vector<DstRange>& v = *out;
    v.clear();
    v.reserve(n);
    for (size_t i = 0; i < n; ++i) {
        if (!p->nbytes[i]) continue;
        if (!dst[i]) return fail(II_EINVAL, "dst_ptrs[%zu] is NULL for a non-empty tensor", i);
        if (dst[i] & (p->dst_align[i] - 1))
            return fail(II_EALIGN, "dst_ptrs[%zu]=%#llx is not aligned to %llu", i,
                        (unsigned long long)dst[i], (unsigned long long)p->dst_align[i]);
        uint64_t e;
        if (__builtin_add_overflow(dst[i], p->nbytes[i], &e))
            return fail(II_EOVERFLOW, "dst_ptrs[%zu] + nbytes overflows", i);
        v.push_back({dst[i], e, i});
    }
    auto by_address = [](const DstRange& a, const DstRange& b) { return a.b < b.b; };
    if (!std::is_sorted(v.begin(), v.end(), by_address)) std::sort(v.begin(), v.end(), by_address);
    for (size_t j = 1; j < v.size(); ++j)
        if (v[j].b < v[j - 1].e)
            return fail(II_EOVERLAP, "destinations of tensors %zu and %zu overlap", v[j - 1].i,
                        v[j].i);
    return II_OK;
}

}  // namespace ii

// The two ways a load checks its destinations (dst_check.h) against each
// other: whatever arena_base takes for the plan's layout in one arena,
// dst_ranges accepts with the same first and last byte, and whatever
// dst_ranges refuses, arena_base does not take. Random tables (empty
// tensors, every alignment, one to a few rows) at random bases, with one
// destination moved, made NULL or misaligned in many of them. Built with
// AddressSanitizer and UndefinedBehaviorSanitizer; prints OK and the number
// of arenas taken, or the first failed case.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "dst_check.h"
#include "ii.h"

namespace ii {
void runtime_destroy(ii_plan_t*) {}  // no device state in a host-only build
}

static uint64_t state = 88172645463325252ull;
static uint64_t pick(uint64_t n) {  // xorshift64
    state ^= state << 13;
    state ^= state >> 7;
    state ^= state << 17;
    return state % n;
}

#define CHECK(c)                                                                  \
    do {                                                                          \
        if (!(c)) {                                                               \
            printf("check failed: %s (case %d, line %d)\n", #c, it, __LINE__); \
            exit(1);                                                              \
        }                                                                         \
    } while (0)

int main(int argc, char** argv) {
    const int iters = argc > 1 ? atoi(argv[1]) : 20000;
    int arenas = 0, refused = 0, plain = 0;
    for (int it = 0; it < iters; ++it) {
        const size_t n = pick(9);
        std::vector<int64_t> shape(n);
        std::vector<ii_tensor_desc> t(n, ii_tensor_desc{});
        uint64_t pos = 0;
        for (size_t i = 0; i < n; ++i) {
            shape[i] = pick(4) == 0 ? 0 : (int64_t)(1 + pick(70));
            t[i].dtype = II_U8;
            t[i].ndim = 1;
            t[i].shape = &shape[i];
            t[i].src_offset = pos;
            t[i].dst_align = 1ull << pick(8);
            pos += (uint64_t)shape[i];
        }
        ii_plan_t* p = nullptr;
        CHECK(ii_plan(t.data(), n, 64, &p) == II_OK);
        uint64_t base = pick(10) == 0 ? ~0ull - pick(512) : pick(10) == 0 ? pick(2) : 4096 + pick(4096);
        if (pick(2)) base &= ~(p->max_align - 1);
        std::vector<uint64_t> dst(n);
        for (size_t i = 0; i < n; ++i)
            dst[i] = p->nbytes[i] || pick(2) ? base + p->dst_offset[i] : pick(3);
        if (n && pick(2)) {
            uint64_t& d = dst[pick(n)];
            switch (pick(4)) {
            case 0: d = 0; break;
            case 1: d += 1 + pick(3); break;
            case 2: d += 128 * (1 + pick(4)); break;
            default: d -= 1 + pick(256); break;
            }
        }
        uint64_t b = 0, e = 0;
        std::vector<ii::DstRange> v;
        const bool arena = ii::arena_base(p, dst.data(), &b, &e);
        const int rc = ii::dst_ranges(p, dst.data(), &v);
        if (arena) {
            CHECK(rc == II_OK && !v.empty());
            CHECK(v.front().b == b && v.back().e == e);
            for (const ii::DstRange& r : v) CHECK(r.b == b + p->dst_offset[r.i]);
            ++arenas;
        } else {
            rc == II_OK ? ++plain : ++refused;
            // the layout itself, at an address it may stand at, is always taken
            bool layout = !v.empty() && rc == II_OK;
            for (const ii::DstRange& r : v)
                layout &= r.b == v.front().b + p->dst_offset[r.i];
            CHECK(!layout);
        }
        ii_plan_free(p);
    }
    const int it = iters;
    CHECK(iters < 100 || (arenas && plain && refused));
    printf("OK arenas=%d other=%d refused=%d\n", arenas, plain, refused);
    return 0;
}

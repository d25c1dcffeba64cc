// Searches a synthetic non-increasing sequence of lengths of up to 2^31 - 3 positions with the
// search of the group chain.  Positions are checked against the sequence's bounds before they
// are used; prints one line per mistake and returns 1 if there was any.
#include <cstdio>

#include "odb_search.h"

namespace {

constexpr int kSamples = 1024;

int check(int64_t last, int64_t fall) {
    // lengths 9 on [0, fall), 5 on [fall, last)
    int bad = 0;
    auto len = [&](int64_t p) -> int64_t {
        if (p < 0 || p >= last) {
            if (!bad) std::printf("last %lld fall %lld: position %lld read\n", (long long)last, (long long)fall, (long long)p);
            bad = 1;
            return 0;   // ends the search
        }
        return p < fall ? 9 : 5;
    };
    const int64_t stride = odb::search_stride(last, kSamples);
    if (stride < 1 || stride * kSamples < last) {
        std::printf("last %lld: stride %lld\n", (long long)last, (long long)stride);
        return 1;
    }
    auto sample = [&](int64_t i) -> int64_t { return i * stride < last ? len(i * stride) : 0; };
    const int64_t ats[] = {4, 5, 8, 9}, want[] = {last, fall, fall, 0};
    for (int k = 0; k < 4; ++k) {
        const int64_t got = odb::first_at_most(sample, len, last, stride, kSamples, ats[k]);
        if (got != want[k]) {
            std::printf("last %lld fall %lld threshold %lld: %lld, not %lld\n", (long long)last, (long long)fall,
                        (long long)ats[k], (long long)got, (long long)want[k]);
            bad = 1;
        }
    }
    return bad;
}

}  // namespace

int main() {
    int bad = 0;
    const int64_t lasts[] = {1, 2, 1023, 1024, 1025, 4097, (1ll << 30) - 1, (1ll << 30) + 1, (1ll << 30) + (1ll << 29),
                             (1ll << 31) - 1025, (1ll << 31) - 1023, (1ll << 31) - 3};
    for (const int64_t last : lasts) {
        const int64_t falls[] = {0, 1, last / 3, last / 2, last / 2 + last / 4, last - 1, last};
        for (const int64_t fall : falls) bad |= check(last, fall);
    }
    return bad;
}

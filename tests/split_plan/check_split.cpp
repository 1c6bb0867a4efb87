// Checks of csrc/wkv6_split_plan.h over shapes on both sides of its rules: every token in exactly one segment, and for the
// split that an entry point makes by itself every segment long enough for its hand-over, one workgroup per compute unit at
// most, and no split of a shape that the rule leaves whole; arguments "B T H segments length" (any number of them) pin plans.  Prints "ok <shapes>" or the first shape that fails.
#include "../../paper_2407_12077_amd/csrc/wkv6_split_plan.h"

#include <cstdio>
#include <cstdlib>

static int fail(const char* what, int B, int T, int H, const wkv6::SplitPlan& p) {
    std::printf("%s: B=%d T=%d H=%d segs=%d seg_len=%d\n", what, B, T, H, p.segs, p.seg_len);
    return 1;
}

int main(int argc, char** argv) {
    long long shapes = 0;
    for (int i = 1; i + 4 < argc; i += 5) {
        const int B = std::atoi(argv[i]), T = std::atoi(argv[i + 1]), H = std::atoi(argv[i + 2]);
        const wkv6::SplitPlan p = wkv6::plan_own_split(B, T, H);
        ++shapes;
        if (p.segs != std::atoi(argv[i + 3]) || p.seg_len != std::atoi(argv[i + 4])) return fail("another plan", B, T, H, p);
    }
    const int heads[] = {1, 3, 12, 16, 32, 40, 64, 85, 86, 128, 256, 257, 262144};
    for (int B = 1; B <= 90; B += B < 12 ? 1 : 13)
        for (int H : heads)
            for (long long t = 1; t <= 2147483647LL; t += t < 6000 ? 1 : t < 200000 ? 4099 : 400000009LL) {
                const int T = static_cast<int>(t);
                const wkv6::SplitPlan p = wkv6::plan_own_split(B, T, H);
                const long long units = static_cast<long long>(B) * H;
                ++shapes;
                if (p.segs < 1) return fail("no segment", B, T, H, p);
                if (p.segs == 1) {
                    if (p.seg_len != T) return fail("whole, but another length", B, T, H, p);
                    continue;
                }
                const long long before = static_cast<long long>(p.segs - 1) * p.seg_len, last = T - before;
                if (p.segs < 3 || units * p.segs > 256) return fail("too few or too many workgroups", B, T, H, p);
                if (p.seg_len % 32 != 0 || last < 1 || last > p.seg_len) return fail("tokens left out or twice", B, T, H, p);
                if (p.seg_len < wkv6::kSegPlaceTokens || last < wkv6::kSegPlaceTokens) return fail("no room for the hand-over", B, T, H, p);
                if (T - p.seg_len < (units > 80 ? 800 : 640)) return fail("too little saved", B, T, H, p);
            }
    for (int T = 1; T < 3000; ++T)
        for (int segments = 1; segments < 70; ++segments) {
            const wkv6::SplitPlan p = wkv6::plan_split(T, segments);
            const long long before = static_cast<long long>(p.segs - 1) * p.seg_len;
            ++shapes;
            if (p.segs < 1 || p.segs > segments || p.seg_len % 32 != 0 || before >= T || T - before > p.seg_len)
                return fail("explicit split", segments, T, 0, p);
        }
    std::printf("ok %lld\n", shapes);
    return 0;
}

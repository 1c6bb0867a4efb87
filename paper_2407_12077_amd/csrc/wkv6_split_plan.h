// How the token axis is cut into segments.  Plain host arithmetic without HIP, so that it can be checked on any machine.
#pragma once

namespace wkv6 {

// Tokens of `out` that a segment's hand-over covers when it lies there: 65 rows of two 128-byte halves.
constexpr int kSegPlaceTokens = 130;

struct SplitPlan {
    int segs;        // segments actually used
    int seg_len;     // tokens per segment (multiple of 32), last one shorter
};

inline SplitPlan plan_split(int T, int segments) {
    SplitPlan p;
    if (segments < 1) segments = 1;
    long long len = (static_cast<long long>(T) + segments - 1) / segments;
    len = (len + 31) / 32 * 32;
    if (len < 32) len = 32;
    p.seg_len = static_cast<int>(len);
    p.segs = static_cast<int>((T + len - 1) / len);
    if (p.segs < 1) p.segs = 1;
    return p;
}

// The split that an entry point without a workspace makes by itself when its (batch, head) units leave compute units
// idle: as many segments as fill the 256 of an MI355X once.  The hand-over between the passes lies in
// the first rows of every segment of `out`, which the last pass overwrites, so every segment needs that many
// tokens.  A function of the shape alone, the same for every form and output type, so that forms that agree bit for
// bit still do.
// The two passes in front cost about 12 us and, in the last pass, every chunk that a workgroup no longer walks saves 0.75
// us: the split pays from about 20 chunks on.  Measured, microseconds, whole -> split (Finch, H = 32): 700 tokens 21.9 -> 22.4,
// 1024 29.0 -> 22.7, 4096 97 -> 38, 32 768 727 -> 221; Finch-C2 with two sequences 700 tokens 27.1 -> 28.3, 1024
// 35.7 -> 29.9, 4096 121 -> 70.  Two segments never pay: what they save the state pass takes (Finch-C2, four sequences of 4096:
// 128 -> 124; of 2048 67 -> 68).
inline SplitPlan plan_own_split(int B, int T, int H) {
    const SplitPlan whole{1, T};
    const long long units = static_cast<long long>(B) * H;
    long long segs = 256 / units;
    if (segs > T / kSegPlaceTokens) segs = T / kSegPlaceTokens;
    for (; segs > 2; --segs) {
        const SplitPlan p = plan_split(T, static_cast<int>(segs));
        if (p.segs < 3 || T - p.seg_len < 20 * 32) return whole;
        if (p.seg_len >= kSegPlaceTokens && T - static_cast<long long>(p.segs - 1) * p.seg_len >= kSegPlaceTokens)
            return p;
    }
    return whole;
}

}  // namespace wkv6

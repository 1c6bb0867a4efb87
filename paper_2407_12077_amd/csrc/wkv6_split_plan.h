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
// The two passes in front cost 11 to 17 us and, in the last pass, every chunk that a workgroup no longer walks saves 0.65 us
// (Finch-C2 0.75): the split pays from about 20 chunks on, with more than 80 units, whose three segments
// leave the state pass the most to read again for the least gain, from 25 on.  Measured, microseconds, whole -> split: Finch 1 x 32 heads 700 tokens 21.9 -> 22.4,
// 800 22.2 -> 19.3, 1100 29.6 -> 20.5, 4096 92 -> 37, 32 768 727 -> 221; 64 heads (four segments) 870 tokens 25.4 -> 23.3; 5 x 16
// (three segments) 1050 28.7 -> 28.4, 1100 30.0 -> 30.4, 1200 32.2 -> 31.4; 7 x 12 1100 30.0 -> 31.1, 1150 30.8 -> 31.6, 1200 32.1 -> 32.0,
// 1300 34.2 -> 32.9, 4096 93 -> 70; 85 x 1 1050 28.3 -> 29.3, 1100 29.5 -> 31.6, 1200 31.7 -> 32.2; Finch-C2 2 x 32 heads 870 29.7 -> 25.5,
// 4096 113 -> 69, 5 x 16 1050 33.6 -> 31.2, 1200 37.9 -> 34.6, 7 x 12 1100 34.4 -> 34.1, 1300 39.5 -> 37.2.  Two segments never
// pay: what they save the state pass takes (Finch-C2, four sequences of 4096: 128 -> 124; of 2048 67 -> 68).
inline SplitPlan plan_own_split(int B, int T, int H) {
    const SplitPlan whole{1, T};
    const long long units = static_cast<long long>(B) * H;
    long long segs = 256 / units;
    if (segs > T / kSegPlaceTokens) segs = T / kSegPlaceTokens;
    for (; segs > 2; --segs) {
        const SplitPlan p = plan_split(T, static_cast<int>(segs));
        if (p.segs < 3 || T - p.seg_len < 32 * (units > 80 ? 25 : 20)) return whole;
        if (p.seg_len >= kSegPlaceTokens && T - static_cast<long long>(p.segs - 1) * p.seg_len >= kSegPlaceTokens)
            return p;
    }
    return whole;
}

}  // namespace wkv6

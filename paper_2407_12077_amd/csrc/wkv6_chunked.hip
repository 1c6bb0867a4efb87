// Chunked WKV6 prefill kernel for gfx950 (MI355X): one workgroup per (batch, head) -- or, with
// more units than compute units, several units back to back per workgroup -- fp32 state
// carried in MFMA accumulators, every dense contraction on the matrix cores
// (v_mfma_f32_16x16x32_f16, fp32 accumulation).
//
// The recurrence (Finch-C2 Time Mixing: decay map w = exp(-exp(x)), wkv_t, read-out; Finch
// bonus u) is evaluated in chunks of 32 tokens.  With tokens 0..31 of a chunk, S0 the state
// entering it, and W(t,i) = prod_{s=i+1}^{t-1} w_s (a per-key-channel vector, empty product = 1):
//
//   o_t = (r_t * W(t,-1)) . S0                                   inter-chunk read
//       + sum_{i<t} ( sum_n r_t[n] k_i[n] W(t,i)[n] ) v_i        intra-chunk, strictly causal
//       + ( sum_n r_t[n] u[n] k_t[n] ) v_t                       bonus on the diagonal
//   S32 = diag(W(32,-1)) S0 + sum_i (k_i * W(32,i))^T v_i        state update
//
// Only PRODUCTS of decays are ever formed (never a reciprocal or a positive exponent), so
// every scale factor is <= 1 and any decay logit, +-inf included, is handled exactly.  To
// write W(t,i) as (factor of t) x (factor of i) the causal triangle is cut by binary
// levels m = 16,8,4,2,1: the pair (t,i) belongs to the level of the highest bit in which
// t and i differ; there i lies in the first half and t in the second half of the same
// 2m-aligned block, and with `mid` that block's midpoint
//       W(t,i) = (prod_{s=mid}^{t-1} w_s) * (prod_{s=i+1}^{mid-1} w_s),
// a prefix product inside t's m-block times a suffix product inside i's m-block.  Tile Z_m
// holds, row by row, the scaled key (rows in a first half) or the scaled receptance (rows in
// a second half); one MFMA per level and 16x16 block followed by a select assembles the
// score matrix.
//
// Work split inside the workgroup (16 wavefronts, 4 per SIMD), one barrier per window:
//   waves 0..11  three PRODUCER groups of four waves; group g owns the chunks c = g (mod 3) and
//               spends three windows on each: D (decays, products inside 4-token groups, HBM
//               loads six chunks ahead), T (multipliers from all groups' totals, every fp16
//               operand tile), S (score MFMAs, finished output rows of chunk c-2 to HBM).  The
//               groups run one window apart, so every window has one group in each phase and
//               vector-ALU, LDS and matrix-core work of different chunks overlap.
//   waves 12..15 CONSUMERS: each owns 16 value columns of the state and runs the three
//               state-dependent contractions, the only sequential chain of the method.
// In window n: D(chunk n), T(n-1), S(n-2), consumers' state chain on chunk n-2 and A.V on n-3.
// LDS buffers (tiles, scores, decay totals, output staging) are indexed by chunk parity.
//
// Finch-C2 form (template flag): the key is multiplied by (1 - w) in phase D, u does not enter
// the level-1 tiles, the diagonal of the scores is zero, and the second value u' is added to the
// fp32-staged rows before the store.
//
// Modes (template parameter kMode): 0 bf16 output, 1 fp32 output, 3 bf16 output plus
// the per-head partial sums of the LayerNorm over all heads (Finch-C2 output equation) taken in
// the store phase, 4 bf16 output with the decay logits formed in the kernel from the low-rank
// decay path (d = lambda + y B, consumers' MFMAs, handed to phase D through LDS) instead of
// read as x, 5 both.
//
// A workgroup may also own one token segment of a sequence (the token split): its entering state then
// comes from where the segment passes left it (wkv6_segments.hip).
//
// LDS tiles whose contraction index is the channel (scores, inter-chunk read) are [token][channel]
// fp16 with a 160-byte row stride; the two tiles whose contraction index is the token (k^T V, A V:
// scaled keys and values) are stored transposed, [channel][token] with a 96-byte row stride and
// the 16-byte granules of a row XOR-swizzled by two row bits.  With these layouts every MFMA
// operand is one 16-byte row read at the full rate of the gfx950 LDS (measured 254 B/clk), and a
// producer thread, which owns four consecutive tokens of a channel pair, writes a transposed
// tile with two 8-byte stores instead of four 4-byte ones (LDS stores cost about 4 clk per
// instruction up to 4 bytes per lane and 6-8 clk for 8 bytes: the kernel is bound by the LDS
// pipeline, and stores are its slow half).  The output tile is produced transposed by swapping
// the operands of the consumers' MFMAs, so that a lane holds four consecutive value channels of
// one token and stages them with one store.
#include "wkv6_launch.h"
#include "wkv6_tiles.h"
#include "wkv6_windows.h"

#include <type_traits>

namespace wkv6 {
namespace {

constexpr int kProducerGroups = kWindowGroups;   // 4 waves each
constexpr int kThreads = 64 * (4 * kProducerGroups + 4);
constexpr int kRow = 160;                  // fp16 tile row stride in bytes (64 halfs + 16 pad)
constexpr int kTile = kChunk * kRow;       // one [32 tokens][64 channels] tile
constexpr int kRowT = 96;                  // transposed tile [channel][32 tokens]: 64 B + 32 pad
constexpr int kTileT = 64 * kRowT;

// LDS map (bytes).  Everything up to kBuf exists twice, once per chunk parity.
enum : int {
    kZ16 = 0 * kTile,
    kZ8 = 1 * kTile,
    kZ4 = 2 * kTile,
    kZ2 = 3 * kTile,
    kQ1 = 4 * kTile,       // level 1 and bonus, query side: r (odd tokens), r*u (even tokens)
    kK1 = 5 * kTile,       // level 1 and bonus, key side:   k (even tokens), k*u (odd tokens)
    kRT = 6 * kTile,       // r * W(t,-1), channel order permuted to match the state registers
    kKT = 7 * kTile,       // k * W(32,i), transposed: [key channel][token]
    kVT = kKT + kTileT,    // v as fp16, transposed: [value channel][token]
    kA0 = kVT + kTileT,    // scores A[t][i], contraction over channels 0..31
    kA1 = kA0 + kTile,     // scores A[t][i], contraction over channels 32..63
    kG = kA1 + kTile,                      // per 4-token group decay products [8][64] fp32
    kD = kG + 8 * 64 * 4,                  // whole-chunk decay product [64] fp32
    kO = kD + 64 * 4,                      // output staging [32 tokens][64]
    kBuf = (kO + kChunk * kORowF32 * 4 + 1023) / 1024 * 1024,
    kLdsBytes = 2 * kBuf
};
static_assert(kBuf % 16 == 0 && kLdsBytes <= 160 * 1024, "LDS budget");

// Fused decay path only: the chunk's decay logits d[channel pair][parity][token] in fp32, written
// by the consumers and read by the producers' phase D, one buffer per chunk parity after the
// two main buffers.  272 bytes per channel pair (2 x 32 tokens x 4 + 16 pad): the 16-byte
// accesses of 16 neighbouring lanes, a channel pair apart, cover all banks once.
constexpr int kDxPair = 2 * kChunk * 4 + 16;
constexpr int kDxBuf = 32 * kDxPair;
constexpr int kDx = kLdsBytes;
constexpr int kLdsBytesLora = kLdsBytes + 2 * kDxBuf;
static_assert(kLdsBytesLora <= 160 * 1024, "LDS budget");

// Units of several heads in a workgroup, Finch form: the bonus of all heads as fp16 pairs, behind the two main buffers.
constexpr int kTurnHeads = (160 * 1024 - kLdsBytes) / (kHeadSize * 2);

// Byte offset, inside a transposed tile, of the 16-byte granule `granule` (tokens 8*granule .. +7)
// of row `row` (a channel).  The XOR with two row bits makes the producers' 8-byte stores (32
// lanes on 32 different rows, two lanes per granule) and the consumers' 16-byte reads (16
// consecutive rows) both run without bank conflicts beyond the store pipeline's own rate.
__device__ __forceinline__ int tile_t_off(int row, int granule) {
    return row * kRowT + ((granule ^ ((row >> 2) & 3)) << 4);
}
// Score tiles A[t][i] (rows of 64 bytes, stride kRow): granule `granule` (keys 8*granule .. +7) of
// token row t, swizzled by one row bit for the 8-byte score stores.
__device__ __forceinline__ int score_off(int t, int granule) {
    return t * kRow + ((granule ^ ((t >> 2) & 1)) << 4);
}
// Cache policies of a launch, by the bytes that it touches (once, all of them).
//   kCached    While two or three such calls fit the 256 MB memory-side cache: rows that lie there from the kernel that wrote
//              them are loaded temporally, and final states are streamed past.
//   kLarge     Rows streamed, states left to the L2s.
//   kStreamed  The same with the output rows, which the other two write through into the memory-side cache, streamed as well: from
//              where that cannot hold them anyway.  (Below, streaming them gains as much in a loop of such calls as it loses in a
//              first call, whose writes the cache would have taken in, and it takes them from the kernel that reads them next.)
// Microseconds, kLarge (the only policy once) -> the one taken: 8 x 60 tokens x 32 heads (17 MB) 7.05 -> 6.2, 16 x 64 (36 MB) 11.4 ->
// 10.1, Finch-C2 32 x 64 (80 MB) 18.4 -> 16.2; Finch-C2 256 x 512 (3.3 GB) 742 -> 677, first calls 757 -> 728; 64 x 1000 (1.3 GB) 274 -> 252, first
// 291 -> 284.  Not taken: temporal rows at 110 MB 25.8 -> 26.9, at 164 MB 36.7 -> 42.7; streamed output at 680 MB 191 -> 180 but first calls
// 188 -> 206; streamed states at 144 MB 28.9 -> 32.0.  The modes with LayerNorm partials or fused logits stand in a chain with kernels that read
// and write as much again: temporal rows at 90 MB make the prefill 27 -> 24 but the chain 67.9 -> 68.6, streamed output the chain of
// 20 x 900 216 -> 219.  (As run-time branches in the stores the choice costs 2 to 7 %.)
// The line between kCached and kLarge is drawn for rows that the caches hold, as those that a kernel has just written; rows that none holds
// lose by kCached.  kLarge -> kCached, one set of tensors over and over / three sets in turn / sets that no cache holds: Finch 8 x 200 x 32
// (39 MiB) 13.1 -> 11.8 / 14.8 -> 14.0 / 15.0 -> 15.3, 8 x 400 (70) 18.8 -> 19.3 / 20.5 -> 19.5 / 21.2 -> 22.3, 16 x 300 (110) 27.7 -> 27.2 /
// 27.7 -> 28.4 / 27.9 -> 29.9.  Behind copies that have just written the rows from elsewhere, the prefill's share: Finch 8 x 100 10.1 -> 9.6,
// 8 x 300 15.9 -> 15.8, 8 x 400 18.4 -> 18.3, 12 x 250 21.7 -> 21.2, fp32 out 8 x 300 16.2 -> 16.6, fused Finch-C2 with moments 8 x 300
// 20.0 -> 19.0.  The last pass of a split call, whose first pass has read k, v and x, has the same line: Finch-C2 1 x 2000
// (48 MiB) 27.6 -> 26.5 / 27.5 -> 26.1 / 28.6 -> 28.6, 1 x 4096 (97) 43.3 -> 41.5 / 42.5 -> 42.2 / 41.8 -> 43.7, 1 x 5000 (118) 48.5 -> 46.9 /
// 47.7 -> 48.4 / 48.0 -> 49.5.
enum class Traffic { kCached, kLarge, kStreamed };

// The four input streams of one (batch, head) are read through raw buffer descriptors whose
// base is the chunk's first token row (uniform, rebuilt per chunk with scalar adds) and whose
// extent ends with the unit's last token, so rows past the end of the sequence read as zero
// without predicates.  Row offsets of a thread's 4 tokens are kernel-lifetime constants.
struct Streams {
    const char* r;
    const char* k;
    const char* v;
    const char* x;
    long long row_bytes;       // bytes between consecutive tokens
    long long span_bytes;      // bytes from the unit's first token row to the end of its last one
};

// A chunk's loads are issued in two halves (x and r; k and v) so that two different phases can
// share the cost of issuing them.
// kPolicy: the cache policy of the loads, kStreamOnce or 0 (temporal).
template <bool kSkipX, int kPolicy>
__device__ __forceinline__ void load_rows_xr(Raw& d, const Streams& st, long long unit_bytes, int t0,
                                             const int (&voff)[4]) {
    const long long off = static_cast<long long>(t0) * st.row_bytes;       // uniform
    if constexpr (!kSkipX) {
        const __amdgpu_buffer_rsrc_t rx = chunk_rsrc(st.x + unit_bytes, off, st.span_bytes);
#pragma unroll
        for (int s = 0; s < 4; ++s) d.x[s] = __builtin_amdgcn_raw_buffer_load_b32(rx, voff[s], 0, kPolicy);
    } else {
#pragma unroll
        for (int s = 0; s < 4; ++s) d.x[s] = 0u;
    }
    const __amdgpu_buffer_rsrc_t rr = chunk_rsrc(st.r + unit_bytes, off, st.span_bytes);
#pragma unroll
    for (int s = 0; s < 4; ++s) d.r[s] = __builtin_amdgcn_raw_buffer_load_b32(rr, voff[s], 0, kPolicy);
}

template <int kPolicy>
__device__ __forceinline__ void load_rows_kv(Raw& d, const Streams& st, long long unit_bytes, int t0,
                                             const int (&voff)[4]) {
    const long long off = static_cast<long long>(t0) * st.row_bytes;       // uniform
    const __amdgpu_buffer_rsrc_t rk = chunk_rsrc(st.k + unit_bytes, off, st.span_bytes);
    const __amdgpu_buffer_rsrc_t rv = chunk_rsrc(st.v + unit_bytes, off, st.span_bytes);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        d.k[s] = __builtin_amdgcn_raw_buffer_load_b32(rk, voff[s], 0, kPolicy);
        d.v[s] = __builtin_amdgcn_raw_buffer_load_b32(rv, voff[s], 0, kPolicy);
    }
}

// The units (batch, head) of one workgroup.  A workgroup keeps its pipeline running across unit
// boundaries: its chunks form one sequence, unit after unit, and only the state (consumers) and
// the base addresses change at a boundary, so short sequences do not pay the fill and drain of
// the pipeline once per unit.  The stride between the units of a workgroup is a multiple of H, so they share the head
// unless they take the heads in turn (kTurn: the head moves on by one from each unit to the next); they have the same length T, and
// their token rows lie `step` elements apart.
struct Units {
    int first;            // index (batch * H + head) of the first one: selects state_in / state_out / moments
    int stride;           // unit index stride
    int count;            // how many
    int nchunks;          // chunks per unit
    long long base0;      // element offset of the first unit's token 0 in r,k,v,x,out
    long long step;       // element offset between consecutive units of this workgroup
    float* state_out;     // where final states go, indexed like state_in (nullptr: not written)
    int t0;               // the sequence's token that is token 0 here (a token segment's start, else 0)
    int tokens;           // tokens of a unit
    const char* entering; // segment's entering state ([64][64] fp32 with the pitches below), or nullptr: state_in
    int pitch_row, pitch_half;
    int heads, head0;     // heads of a token row; the first unit's
    __device__ __forceinline__ int next_head(int hd) const { return hd + 1 == heads ? 0 : hd + 1; }
    __device__ __forceinline__ long long index(int ui, int hd) const { return first + static_cast<long long>(ui) * stride + (hd - head0); }
};

// Position in the workgroup's chunk sequence: unit ui, chunk c of it.  Advanced without
// divisions; c < 0 (before the start) and ui >= count (past the end) mean "no chunk".
// With a single unit per workgroup ui stays 0 and "past the end" is c >= nchunks.
template <bool kTurn, bool kMulti>
struct Cursor {
    int ui, c, hd;        // hd: the head of unit ui
    __device__ __forceinline__ void advance(int by, const Units& un) {
        c += by;
        if constexpr (kMulti) {
            while (c >= un.nchunks) {
                c -= un.nchunks;
                ++ui;
                if constexpr (kTurn) hd = un.next_head(hd);
            }
        }
    }
    __device__ __forceinline__ bool live(const Units& un) const {
        if constexpr (kMulti) return ui < un.count;
        return c < un.nchunks;
    }
    __device__ __forceinline__ long long unit_elems(const Units& un) const {
        if constexpr (kTurn) return ui * un.step + (hd - un.head0) * kHeadSize;
        if constexpr (kMulti) return ui * un.step;
        return 0;
    }
};

// ------------------------------------------------------------------------------------------
// Producer waves: group pg (0..2) = chunk index mod 3, wq = wave inside the group
// ------------------------------------------------------------------------------------------
template <int kMode, bool kC2, bool kTurn, bool kMulti, Traffic kTraffic>
__device__ __forceinline__ void producer(const Args& a, char* lds_all, int tid, int pg, int wq, int h,
                                         const Units& un, long long tok_stride, int T) {
    constexpr int kRows = kTraffic == Traffic::kCached ? 0 : kStreamOnce;
    constexpr int kOutRows = kTraffic == Traffic::kStreamed ? kStoreThrough | kStreamOnce : kStoreThrough;
    constexpr bool kOutF32 = kMode == 1;
    constexpr bool kMoments = kMode == 3 || kMode == 5;   // bf16 out plus the per-head LayerNorm partials
    constexpr bool kLora = kMode >= 4;           // decay logits from the consumers (LDS), not from x
    constexpr bool kStageF32 = kOutF32 || kC2;   // staging precision of the finished rows
    const int lane = tid & 63;
    const int gtid = tid & 255;              // thread inside the group
    const int cp = lane & 31;                // channel pair: channels 2cp, 2cp+1
    const int hl = lane >> 5;
    const int g8 = 2 * wq + hl;              // 4-token group 0..7 inside the chunk
    const bool q4 = hl != 0;                 // query side at level 4 (per lane half)
    const int l16 = lane & 15;
    const int g4 = lane >> 4;

    // the bonus u of this channel pair as an fp16 pair (Finch form only)
    [[maybe_unused]] unsigned hu = kC2 ? 0u : pack_h2(a.u[h * kHeadSize + 2 * cp], a.u[h * kHeadSize + 2 * cp + 1]);
    constexpr bool kTurnU = kTurn && !kC2;  // all heads' u wait in LDS
    if constexpr (kTurnU) {
        for (int i = tid; i < a.H * (kHeadSize / 2); i += 4 * 64 * kProducerGroups)
            lds_write_u32(lds_all, kLdsBytes + 4 * i, pack_h2(a.u[2 * i], a.u[2 * i + 1]));
    }

    Streams st;
    st.r = static_cast<const char*>(a.r) + un.base0 * 2;
    st.k = static_cast<const char*>(a.k) + un.base0 * 2;
    st.v = static_cast<const char*>(a.v) + un.base0 * 2;
    st.x = static_cast<const char*>(a.x) + un.base0 * 2;
    st.row_bytes = tok_stride * 2;
    st.span_bytes = static_cast<long long>(T - 1) * st.row_bytes + kHeadSize * 2;
    int voff[4];                                   // byte offsets of this thread's 4 token rows
#pragma unroll
    for (int s = 0; s < 4; ++s)
        voff[s] = static_cast<int>((4 * g8 + s) * st.row_bytes + 4 * cp);

    // the score block above the diagonal that the A.V product still touches, (t-block 0,
    // i-block 1), stays zero for good in both partial score tiles: 2 x 16x16 halfs = 256 dwords
    if (pg < 2) {
        char* lds = lds_all + pg * kBuf;
        const int which = gtid >> 7;                 // A0 / A1
        const int e = gtid & 127;                    // row = e>>3, column pair = e&7
        lds_write_u32(lds, (which ? kA1 : kA0) + (e >> 3) * kRow + (16 + 2 * (e & 7)) * 2, 0u);
    }

    // column (in halfs) of this channel pair in the permuted r*W(t,-1) tile: slot order matches
    // the state accumulator registers that serve as the B operand of the inter-chunk read
    const int n0 = 2 * cp;
    const int m5 = n0 & 31;
    const int rt_col = (n0 & 32) + 8 * ((m5 >> 2) & 3) + 4 * (m5 >> 4) + (m5 & 3);

    Raw raw_a, raw_b;      // raw inputs of this group's next two chunks (in flight or landed)
    Prep pr;

    // Phase D.  Digest the raw inputs in `cur` (chunk c): decays, their products inside
    // the thread's 4-token group (published in G), and every operand that needs nothing else.
    auto digest = [&](int g, int c, int hd, Raw& cur) {     // g: position in the sequence, c: chunk of its unit, hd: head
        char* lds = lds_all + (g & 1) * kBuf;
        const int t0 = c * kChunk;
        if constexpr (kTurnU) {                              // this group's first chunk of a unit is one of its first three
            if (c < kProducerGroups) hu = *reinterpret_cast<const unsigned*>(lds_all + kLdsBytes + (hd * (kHeadSize / 2) + cp) * 4);
        }
        if (t0 + kChunk > T) {
            // last, partial chunk: tokens past the end were read as zeros; give them w = 1
#pragma unroll
            for (int s = 0; s < 4; ++s)
                if (t0 + 4 * g8 + s >= T) cur.x[s] = 0xff80ff80u;      // bf16 -inf, twice
        }
        float w[2][4];
        [[maybe_unused]] float omw[2][4];       // Finch-C2: 1 - w
        if constexpr (kLora) {
            // the chunk's logits were left in LDS by the consumers one window ago: this thread's
            // 4 tokens of its two channels
            const char* dx = lds_all + kDx + (g & 1) * kDxBuf + cp * kDxPair + g8 * 16;
            const float4 de = *reinterpret_cast<const float4*>(dx);
            const float4 dq = *reinterpret_cast<const float4*>(dx + kChunk * 4);
            const float d0[4] = {de.x, de.y, de.z, de.w}, d1[4] = {dq.x, dq.y, dq.z, dq.w};
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const bool past = t0 + 4 * g8 + s >= T;          // tokens past the end: w = 1
                float e0 = 0.f, e1 = 0.f;
                const float w0 = decay_of(d0[s], e0), w1 = decay_of(d1[s], e1);
                w[0][s] = past ? 1.f : w0;
                w[1][s] = past ? 1.f : w1;
                if constexpr (kC2) {
                    omw[0][s] = one_minus_decay(e0, w0);               // past the end the key is zero
                    omw[1][s] = one_minus_decay(e1, w1);
                }
            }
        } else {
            decays_of<kC2>(cur.x, w, omw);
        }
        *reinterpret_cast<float2*>(lds + kG + (g8 * 64 + 2 * cp) * 4) = form_operands<kC2>(pr, cur, w, omw, hu);
    };

    // Phase T: multipliers from the other groups' decay totals, then every operand tile.  (Writing
    // the four tiles that need no totals -- Z4, Z2, Q1, K1 -- a window earlier, in phase D, into a
    // slot per producer group was measured and dropped: the digest phase grew by what the tile
    // phase should have lost and the window did not get shorter; the compute unit's LDS queue, not
    // one phase's share of it, is what the window waits for.  Also measured and dropped: neighbouring
    // lanes trading two values so that each token-row tile takes two 8-byte stores instead of four
    // 4-byte ones -- 9 % slower in the kernel although 8-byte stores run at 85 against 62 B/clk in
    // isolation.)  The
    // body is instantiated per wave position kWq so that the level-8 and level-16 roles (key or
    // query side) and the neighbouring group products are compile-time choices.
    auto write_tiles_at = [&](auto wq_const, int c) {
        constexpr int kWq = decltype(wq_const)::value;
        constexpr bool kQ8 = (kWq & 1) != 0;     // query side at level 8
        constexpr bool kQ16 = (kWq & 2) != 0;    // query side at level 16
        char* lds = lds_all + (c & 1) * kBuf;
        float m_rt[2], m_kt[2], m16[2], m8[2];
        float2 own[8];
#pragma unroll
        for (int g = 0; g < 8; ++g)
            own[g] = *reinterpret_cast<const float2*>(lds + kG + (g * 64 + 2 * cp) * 4);
        // Writes are grouped by tile, the four tokens of a tile back to back, so that neighbouring
        // writes pair up into two-address LDS instructions.  The tiles that need no multiplier go
        // out first, right behind the reads of the group totals: at the start of a window every
        // wave of the workgroup queues LDS work, and the totals take hundreds of cycles to return.
        const int nat0 = 4 * g8 * kRow + 4 * cp;             // token 0 of the group, natural channel order
        auto put4 = [&](int tile, unsigned v0, unsigned v1, unsigned v2, unsigned v3) {
            lds_write_u32(lds, tile + nat0, v0);
            lds_write_u32(lds, tile + nat0 + kRow, v1);
            lds_write_u32(lds, tile + nat0 + 2 * kRow, v2);
            lds_write_u32(lds, tile + nat0 + 3 * kRow, v3);
        };
        // transposed tiles: this thread's 4 tokens of channel 2cp (and 2cp+1) are 8 contiguous bytes
        const int tr0 = tile_t_off(2 * cp, wq) + 8 * hl;          // tokens 4*g8 .. +3 = half hl of granule wq
        const int tr1 = tile_t_off(2 * cp + 1, wq) + 8 * hl;
        lds_write_u64(lds, kVT + tr0, pr.vt[0], pr.vt[1]);
        lds_write_u64(lds, kVT + tr1, pr.vt[2], pr.vt[3]);
        // level 4: the even group of an 8-block holds keys, the odd one queries
        put4(kZ4, q4 ? pr.rp[0] : pr.ks[0], q4 ? pr.rp[1] : pr.ks[1], q4 ? pr.rp[2] : pr.ks[2],
             q4 ? pr.rp[3] : pr.ks[3]);
        put4(kZ2, pr.z2[0], pr.z2[1], pr.z2[2], pr.z2[3]);
        put4(kQ1, pr.q1[0], pr.q1[1], pr.q1[2], pr.q1[3]);
        if constexpr (!kC2) put4(kK1, pr.k1[0], pr.k1[1], pr.k1[2], pr.k1[3]);
        __builtin_amdgcn_sched_barrier(0);       // keep these writes ahead of the wait for the totals
#pragma unroll
        for (int ch = 0; ch < 2; ++ch) {
            float o[8];
#pragma unroll
            for (int g = 0; g < 8; ++g) o[g] = ch ? own[g].y : own[g].x;
            // pl / ph: decays of the group pairs before / after this wave's pair;
            // f16: this wave's share of the level-16 multiplier
            float pl, ph, f16;
            if constexpr (kWq == 0) { pl = 1.f; ph = (o[2] * o[3]) * ((o[4] * o[5]) * (o[6] * o[7])); f16 = o[2] * o[3]; }
            else if constexpr (kWq == 1) { pl = o[0] * o[1]; ph = (o[4] * o[5]) * (o[6] * o[7]); f16 = 1.f; }
            else if constexpr (kWq == 2) { pl = (o[0] * o[1]) * (o[2] * o[3]); ph = o[6] * o[7]; f16 = 1.f; }
            else { pl = ((o[0] * o[1]) * (o[2] * o[3])) * (o[4] * o[5]); ph = 1.f; f16 = o[4] * o[5]; }
            // the other group of this wave's pair lies before the odd group (hl=1) and after
            // the even one (hl=0)
            const float before = hl ? o[2 * kWq] : 1.f;
            const float after = hl ? 1.f : o[2 * kWq + 1];
            m_rt[ch] = pl * before;            // decays of the chunk's tokens before this group
            m_kt[ch] = after * ph;             // decays of the chunk's tokens after this group
            m16[ch] = kQ16 ? f16 * before : after * f16;   // level 16: inside the 16-token half
            m8[ch] = kQ8 ? before : after;                 // level 8: inside the 8-token block
            if constexpr (kWq == 0)
                if (hl == 0) *reinterpret_cast<float*>(lds + kD + (2 * cp + ch) * 4) = o[0] * m_kt[ch];
        }
        // the multipliers as fp16 channel pairs: one packed multiply per tile entry
        const unsigned h_rt = pack_h2(m_rt[0], m_rt[1]);
        const unsigned h_kt = pack_h2(m_kt[0], m_kt[1]);
        const unsigned h16 = pack_h2(m16[0], m16[1]);
        const unsigned h8 = pack_h2(m8[0], m8[1]);
        {
            const unsigned k0 = mul_h2(pr.ks[0], h_kt), k1 = mul_h2(pr.ks[1], h_kt);
            const unsigned k2 = mul_h2(pr.ks[2], h_kt), k3 = mul_h2(pr.ks[3], h_kt);
            lds_write_u64(lds, kKT + tr0, lo_halves(k0, k1), lo_halves(k2, k3));
            lds_write_u64(lds, kKT + tr1, hi_halves(k0, k1), hi_halves(k2, k3));
        }
        const unsigned* z16 = kQ16 ? pr.rp : pr.ks;
        const unsigned* z8 = kQ8 ? pr.rp : pr.ks;
        put4(kZ16, mul_h2(z16[0], h16), mul_h2(z16[1], h16), mul_h2(z16[2], h16), mul_h2(z16[3], h16));
        put4(kZ8, mul_h2(z8[0], h8), mul_h2(z8[1], h8), mul_h2(z8[2], h8), mul_h2(z8[3], h8));
        put4(kRT + (rt_col - 2 * cp) * 2, mul_h2(pr.rp[0], h_rt), mul_h2(pr.rp[1], h_rt),
             mul_h2(pr.rp[2], h_rt), mul_h2(pr.rp[3], h_rt));
    };
    auto write_tiles = [&](int c) {
        switch (wq) {                             // wave-uniform
            case 0: write_tiles_at(std::integral_constant<int, 0>{}, c); break;
            case 1: write_tiles_at(std::integral_constant<int, 1>{}, c); break;
            case 2: write_tiles_at(std::integral_constant<int, 2>{}, c); break;
            default: write_tiles_at(std::integral_constant<int, 3>{}, c); break;
        }
    };

    // Phase S, part 1.  Scores of chunk c; the contraction over the 64 channels is
    // split in two halves (kk), each wave writes its partial scores to tile A0 or A1 and the
    // consumers add the two products.  Wave wq: diagonal block wq&1, channel half wq>>1; the
    // waves with an even wq also take the level-16 block (t-block 1, i-block 0).
    auto scores = [&](int c) {
        char* lds = lds_all + (c & 1) * kBuf;
        const int q = wq & 1;
        const int kk = wq >> 1;
        const int at = kk ? kA1 : kA0;
        const int rowq = (16 * q + l16) * kRow + 16 * g4 + 64 * kk;
        const half8 z8 = lds_read_h8(lds, kZ8 + rowq);
        const half8 z4 = lds_read_h8(lds, kZ4 + rowq);
        const half8 z2 = lds_read_h8(lds, kZ2 + rowq);
        const half8 q1 = lds_read_h8(lds, kQ1 + rowq);
        const half8 k1 = kC2 ? q1 : lds_read_h8(lds, kK1 + rowq);
        const float4v zero{0.f, 0.f, 0.f, 0.f};
        const float4v acc8 = mfma(z8, z8, zero);
        const float4v acc4 = mfma(z4, z4, zero);
        const float4v acc2 = mfma(z2, z2, zero);
        const float4v acc1 = mfma(k1, q1, zero);     // pairs (odd t, t-1) and, on the diagonal, the bonus
        // keys 16q + 4*g4 .. +3 of token row 16q + l16: half (g4 & 1) of granule 2q + (g4 >> 1)
        *reinterpret_cast<uint2*>(lds + at + score_off(16 * q + l16, 2 * q + (g4 >> 1)) + 8 * (g4 & 1)) =
            choose_levels<kC2>(acc8, acc4, acc2, acc1, l16, g4);
        if (q == 0) {
            const int rq = (16 + l16) * kRow + 16 * g4 + 64 * kk;
            const half8 zq = lds_read_h8(lds, kZ16 + rq);
            const half8 zk = lds_read_h8(lds, kZ16 + rq - 16 * kRow);
            const float4v acc = mfma(zk, zq, zero);
            *reinterpret_cast<uint2*>(lds + at + score_off(16 + l16, g4 >> 1) + 8 * (g4 & 1)) =
                make_uint2(pack_h2(acc[0], acc[1]), pack_h2(acc[2], acc[3]));
        }
    };

    // Phase S, part 2.  Finished output rows of chunk c (staged by the consumers): full
    // 128-byte (bf16) rows to HBM, 8 threads per row.  Finch-C2: the rows are staged in fp32 and
    // the second value u' of the same 8 channels (16 bytes, loaded two windows earlier) is added
    // before the single rounding of the output.  (Letting the consumer waves load u' in their
    // accumulator layout and start the chunk's accumulator from it -- bf16 staging, nothing to add
    // here -- gives the same bits and was 25 % slower: a load issued by any wave of the workgroup
    // returns behind the chunk loads the producers already have in flight, four to six windows
    // of them, and the consumers cannot wait that long.)
    const int srow = gtid >> 3;                  // token row inside the chunk this thread stores
    const int scol = 8 * (gtid & 7);             // first of its 8 channels
    [[maybe_unused]] uint4v up_raw = {0u, 0u, 0u, 0u};
    // fp32 rows (256 bytes): the row's 8 threads store its first 128 bytes, then its second (whole cache lines per
    // instruction), so thread j holds channels 4j .. and 32 + 4j ..; a bf16 row's threads hold channels 8j ..
    [[maybe_unused]] const int up_voff = static_cast<int>(srow * st.row_bytes + (kOutF32 ? scol : scol * 2));
    [[maybe_unused]] const char* up_base = kC2 ? static_cast<const char*>(a.uprime) + un.base0 * 2 : nullptr;
    auto load_uprime = [&](const Cursor<kTurn, kMulti>& at) {
        if constexpr (kC2) {
            // unconditional (exact wait counts): before the start it re-reads chunk 0, past the
            // end the descriptor is empty
            const int cc = at.c < 0 ? 0 : at.c;
            const bool live = at.c < 0 || at.live(un);
            const long long off = static_cast<long long>(cc) * kChunk * st.row_bytes;
            const __amdgpu_buffer_rsrc_t ru = chunk_rsrc(up_base + (live ? at.unit_elems(un) * 2 : 0), off, live ? st.span_bytes : 0);
            if constexpr (kOutF32) {
                const uint2v lo = __builtin_bit_cast(uint2v, __builtin_amdgcn_raw_buffer_load_b64(ru, up_voff, 0, kRows));
                const uint2v hi = __builtin_bit_cast(uint2v, __builtin_amdgcn_raw_buffer_load_b64(ru, up_voff + 64, 0, kRows));
                up_raw = uint4v{lo[0], lo[1], hi[0], hi[1]};
            } else {
                up_raw = __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(ru, up_voff, 0, kRows));
            }
        }
    };
    // Output rows leave through a raw buffer descriptor that starts at the chunk's first row and ends
    // with the unit's last token: rows past the end of the sequence are dropped by the bounds check.
    constexpr int kOutElem = kOutF32 ? 4 : 2;
    [[maybe_unused]] const long long out_row_bytes = tok_stride * kOutElem;
    [[maybe_unused]] const long long out_span = static_cast<long long>(T - 1) * out_row_bytes + kHeadSize * kOutElem;
    [[maybe_unused]] const int out_voff = static_cast<int>(srow * out_row_bytes + scol * kOutElem);
    [[maybe_unused]] const char* out_base = static_cast<const char*>(a.out) + un.base0 * kOutElem;
    auto store_rows = [&](int g, const Cursor<kTurn, kMulti>& at) {   // g: position in the sequence (LDS parity)
        const char* lds = lds_all + (g & 1) * kBuf;
        const int t = at.c * kChunk + srow;
        const __amdgpu_buffer_rsrc_t ro = chunk_rsrc(out_base + at.unit_elems(un) * kOutElem,
                                                     static_cast<long long>(at.c) * kChunk * out_row_bytes, out_span);
        auto put = [&](uint4v q, int byte) {
            __builtin_amdgcn_raw_buffer_store_b128(q, ro, out_voff + byte, 0, kOutRows);
        };
        if (t < T) {
            if constexpr (kStageF32) {
                const float4* src = reinterpret_cast<const float4*>(
                    lds + kO + (srow * kORowF32 + (kOutF32 ? scol / 2 : scol)) * 4);
                float4 q0 = src[0], q1 = src[kOutF32 ? 8 : 1];
                if constexpr (kC2) add_uprime(q0, q1, up_raw);
                if constexpr (kMoments) {
                    const float2v pair = row_moments(q0, q1);        // the row's first thread writes it
                    if (scol == 0) {
                        const long long unit_index = kMulti ? un.index(at.ui, at.hd) : un.first;
                        // streamed like the output rows (measured: 7 % of the kernel's time on many
                        // short units against a plain store)
                        __builtin_nontemporal_store(pair, reinterpret_cast<float2v*>(a.moments + (unit_index * a.T + un.t0 + t) * 2));
                    }
                }
                if constexpr (kOutF32) {
                    put(__builtin_bit_cast(uint4v, q0), -scol * 2);               // byte 16 j of the row
                    put(__builtin_bit_cast(uint4v, q1), 128 - scol * 2);          // byte 128 + 16 j
                } else {
                    put(pack_row(q0, q1), 0);
                }
            } else {
                put(*reinterpret_cast<const uint4v*>(lds + kO + (srow * kORowBf16 + scol) * 2), 0);
            }
        }
    };

    // A group spends three consecutive windows on each of its chunks g = pg, pg+3, ... of the
    // workgroup's chunk sequence:
    //   window g    phase D: decays and group products of chunk g from one of two raw register
    //               sets, then the HBM loads of x and r of the group's chunk after next (g+6) into
    //               the same set (k and v follow in phase T); they stay in flight for four to six
    //               windows.  Issued unconditionally: past the end the descriptor is empty and the
    //               loads return zeros without touching memory.
    //   window g+1  phase T: multipliers from all groups' decay totals, every operand tile.
    //   window g+2  phase S: score MFMAs, and the finished output rows of chunk g-2.
    // The three groups are one window apart, so every window sees one group in each phase
    // next to the consumers: vector-ALU, LDS and matrix-core work of different chunks overlap.
    // Wave priorities (s_setprio, an issue-arbitration hint inside the compute unit): the score
    // phase and the consumers (3) sit on MFMA and LDS-read latency chains and the consumers carry
    // the only dependency from window to window; the digest (2) starts with the exponentials
    // everything else waits for; the tile phase (0) is throughput work, mostly LDS writes nobody
    // reads before the barrier, and fills the gaps.  Measured against equal priorities: config 2
    // -3 %, config 5 -4 to -12 % depending on the box, fp32 output -8 %, nothing slower.
    const int total = un.count * un.nchunks;
    const int nwin = window_count(total);
    Cursor<kTurn, kMulti> cur{0, 0, un.head0}, ld{0, 0, un.head0}, stc{0, pg - 2, un.head0};      // chunk g, chunk g+6 (loads), chunk g-2 (stores)
    cur.advance(pg, un);
    ld.advance(pg, un);
    stc.advance(0, un);
    auto fetch_xr = [&](Raw& buf, const Cursor<kTurn, kMulti>& at) {
        const bool live = at.live(un);                // uniform; dead: offset past the span = empty descriptor
        load_rows_xr<kLora, kRows>(buf, st, live ? at.unit_elems(un) * 2 : 0, live ? at.c * kChunk : T + kChunk, voff);
    };
    auto fetch_kv = [&](Raw& buf, const Cursor<kTurn, kMulti>& at) {
        const bool live = at.live(un);
        load_rows_kv<kRows>(buf, st, live ? at.unit_elems(un) * 2 : 0, live ? at.c * kChunk : T + kChunk, voff);
    };
    // one chunk of this group through its three windows; `buf` holds its raw inputs and is
    // refilled with the group's chunk after next (six chunks ahead) right after the digest
    auto cycle = [&](int g, Raw& buf) {
        const bool live = cur.live(un);
        __builtin_amdgcn_s_setprio(2);            // see the note on wave priorities above
        if (live) digest(g, cur.c, cur.hd, buf);
        load_uprime(stc);                         // older than the chunk loads: waited for first
        fetch_xr(buf, ld);
        __syncthreads();                                                        // window barrier
        __builtin_amdgcn_s_setprio(0);
        if (live) write_tiles(g);
        fetch_kv(buf, ld);                        // the other half: issued a window later, measured best here
        __syncthreads();                                                        // window barrier
        __builtin_amdgcn_s_setprio(3);
        if (live) scores(g);
        if (stc.c >= 0 && stc.live(un)) store_rows(g - 2, stc);
        __syncthreads();                                                        // window barrier
        cur.advance(3, un);
        ld.advance(3, un);
        stc.advance(3, un);
    };
    fetch_xr(raw_a, ld);
    fetch_kv(raw_a, ld);
    ld.advance(3, un);
    fetch_xr(raw_b, ld);
    fetch_kv(raw_b, ld);
    ld.advance(3, un);                    // now six chunks ahead of `cur`
    __syncthreads();                                                            // start barrier
    int done = 0;                                                               // windows passed
    for (; done < pg; ++done) {
        __syncthreads();                                                        // window barrier
    }
    int g = pg;
#pragma clang loop unroll(disable)
    for (; has_cycle_pair(g, nwin); g += 6) {       // same walk as producer_walk() in wkv6_windows.h
        cycle(g, raw_a);
        cycle(g + 3, raw_b);
        done += 6;
    }
    if (has_cycle(g, nwin)) {
        cycle(g, raw_a);
        done += 3;
    }
    for (; done < nwin; ++done) {
        __syncthreads();                                                        // window barrier
    }
}

// ------------------------------------------------------------------------------------------
// Consumer waves
// ------------------------------------------------------------------------------------------
template <int kMode, bool kC2, bool kTurn, bool kMulti, Traffic kTraffic>
__device__ __forceinline__ void consumer(const Args& a, char* lds_all, int lane, int cw, const Units& un) {
    constexpr int kState = kTraffic == Traffic::kCached ? kStoreThrough | kStreamOnce : 0;
    constexpr bool kOutF32 = kMode == 1;
    constexpr bool kLora = kMode >= 4;
    const int l16 = lane & 15;
    const int g4 = lane >> 4;
    const int j = 16 * cw + l16;            // value column of this lane
    // the consumers carry the only sequential chain: let the SIMD arbiter prefer them
    __builtin_amdgcn_s_setprio(3);

    // S[nb][e] = state[n = 16nb + 4g4 + e][j]; Snext: the state entering the workgroup's next
    // unit, fetched while the current unit is still being processed
    // State traffic goes through a raw buffer descriptor of the unit's 16 KiB with the
    // (nb, e) part of the offset as a scalar: one vector register of addressing for all 16
    // accesses instead of a 64-bit address each.
    float4v S[4];
    [[maybe_unused]] float4v Snext[4];
    const int state_voff = (4 * g4 * 64 + j) * 4;
    auto state_rsrc = [&](const float* base, int ui, int hd) {
        const long long unit = un.index(ui, hd);
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base + unit * 4096), 0, 4096 * 4, 0x00020000);
    };
    auto fetch_state = [&](float4v (&dst)[4], int ui, int hd) {
        if (a.state_in && ui < un.count) {
            const __amdgpu_buffer_rsrc_t rs = state_rsrc(a.state_in, ui, hd);
#pragma unroll
            for (int nb = 0; nb < 4; ++nb)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    dst[nb][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, state_voff, (16 * nb + e) * 256, 0));
        } else {
#pragma unroll
            for (int nb = 0; nb < 4; ++nb) dst[nb] = float4v{0.f, 0.f, 0.f, 0.f};
        }
    };
    if constexpr (kMulti) {
        fetch_state(Snext, 0, un.head0);
    } else if (un.entering) {
        // A token segment: its entering state, rows and half rows at the pitches of where it was left.  When
        // that is the segment's own rows of `out`, this load has returned before the first of them is
        // overwritten: chunk 0's read-out takes S, and its rows leave after a barrier behind that.
        const int voff = 4 * g4 * un.pitch_row + (j >> 5) * un.pitch_half + (j & 31) * 4;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(un.entering), 0, 64 * un.pitch_row, 0x00020000);
#pragma unroll
        for (int nb = 0; nb < 4; ++nb)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                S[nb][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, voff, (16 * nb + e) * un.pitch_row, 0));
    } else {
        fetch_state(S, 0, un.head0);
    }

    // Output of the chunk whose state chain ran last, transposed: o[tq][e] belongs to token
    // 16*tq + l16 and value channel 16*cw + 4*g4 + e (the state is the A operand and the token rows
    // the B operand of the MFMAs below), so a lane's four values are contiguous in the output row.
    float4v o[2];
    half8 vt;           // V^T operand of that chunk: this lane's value channel, tokens 8*g4 .. +7

    const int total = un.count * un.nchunks;
    const int nwin = window_count(total);

    // Fused decay path.  This wave forms the decay logits of its 16 channels (16cw .. 16cw+15, as
    // key channels) for all 32 tokens of the chunk the producers digest in the next window:
    // d = lambda + y B_h, two 16-token row blocks x two 32-wide steps over the rank, bf16 operands
    // (exact products) with fp32 accumulation started at lambda.  The head's 64x16 slice of B
    // stays in registers for the whole kernel; y rows (128 bytes per token, shared by all heads, so served by L2) are
    // requested right behind the use of the chunk before: a load returns behind the chunk loads that the producers have
    // in flight, and one requested at the start of the window that uses it lengthens the window (8 sequences of 2048 tokens and
    // 32 heads 86.7 -> 80.3 us, with no request at all 78.3; 4 x 3000 x 64 121 -> 115).  In the Finch form, whose windows are shorter, the
    // request costs where everything lies in the caches (1 x 600 tokens x 32 heads 20.6 -> 21.6 us, 2 x 800 25.2 -> 26.6): there it goes out
    // without a branch, past the end with an empty descriptor, while the products are formed (21.1, 25.7; 8 x 2048 74.4 -> 73.8; 1 x 100
    // 9.3 -> 9.4, 9.5 with the request at the start).  In the Finch-C2 form the two are level, but for short sequences (1 x 100 10.8 -> 11.0).
    [[maybe_unused]] bf16x8 bw[2];
    [[maybe_unused]] bf16x8 ya[2][2];
    [[maybe_unused]] float lam = 0.f;
    [[maybe_unused]] int y_b0 = 0, y_bstep = 0;
    [[maybe_unused]] const int y_voff = l16 * (kLoraRank * 2) + 16 * g4;
    if constexpr (kLora) {
        const int width = a.H * kHeadSize;
        const int col = (un.first % a.H) * kHeadSize + 16 * cw + l16;
        const unsigned short* bwp = static_cast<const unsigned short*>(a.bw);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int e = 0; e < 8; ++e)
                bw[ks][e] = __builtin_bit_cast(__bf16, bwp[static_cast<long long>(32 * ks + 8 * g4 + e) * width + col]);
        lam = a.lambda[col];
        y_b0 = un.first / a.H;
        y_bstep = un.stride / a.H;
    }
    auto y_fetch = [&](const Cursor<kTurn, kMulti>& dn) {
        const long long batch = y_b0 + (kMulti ? static_cast<long long>(dn.ui) * y_bstep : 0);
        const __amdgpu_buffer_rsrc_t ry = chunk_rsrc(static_cast<const char*>(a.y) + (batch * a.T + un.t0) * (kLoraRank * 2),
                                                     static_cast<long long>(dn.c) * kChunk * (kLoraRank * 2),
                                                     kC2 || dn.live(un) ? static_cast<long long>(un.tokens) * (kLoraRank * 2) : 0);
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
                ya[rt][ks] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(
                                                            ry, y_voff + 16 * rt * (kLoraRank * 2) + 64 * ks, 0, 0));
    };
    auto d_finish = [&](int pos, auto request) {     // pos: the chunk's position in the sequence (LDS parity)
        char* dx = lds_all + kDx + (pos & 1) * kDxBuf + (8 * cw + (l16 >> 1)) * kDxPair + (l16 & 1) * (kChunk * 4) + 16 * g4;
        float4v acc[2];
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) {
            acc[rt] = float4v{lam, lam, lam, lam};
            acc[rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ya[rt][0], bw[0], acc[rt], 0, 0, 0);
            acc[rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ya[rt][1], bw[1], acc[rt], 0, 0, 0);
        }
        if constexpr (!kC2) request();
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) *reinterpret_cast<float4v*>(dx + 64 * rt) = acc[rt];     // tokens 16rt + 4g4 .. +3 of this lane's channel
        if constexpr (kC2) request();
    };
    Cursor<kTurn, kMulti> dn{0, 0, un.head0};                         // the chunk whose logits are formed next
    if constexpr (kLora) {
        if (total > 0) {
            y_fetch(dn);
            d_finish(0, [&] {
                dn.advance(1, un);
                if (!kC2 || total > 1) y_fetch(dn);
            });
        }
    }

    __syncthreads();                                                            // start barrier
    Cursor<kTurn, kMulti> at{0, 0, un.head0};                         // chunk n-2 of the sequence: the state chain's
#pragma clang loop unroll(disable)
    for (int n = 0; n < nwin; ++n) {
        [[maybe_unused]] const bool dlive = kLora && n + 1 < total;
        // (The two parts below in one straight line for the steady state -- every LDS read of the window
        // first, then the matrix-core work of both chunks -- shortens the consumers' own chain from
        // 1430 to 1260 clocks and lengthens the window from 1850 to 1960: their reads then arrive at
        // the LDS queue in one burst at the highest priority and the producers wait behind them.)
        if (n >= 3 && n - 3 < total) {
            // chunk n-3: o += A V (two partial score tiles), then stage for the producers' stores
            char* lds = lds_all + ((n - 3) & 1) * kBuf;
#pragma unroll
            for (int tq = 0; tq < 2; ++tq) {
                const int off = score_off(16 * tq + l16, g4);
                const half8 a0 = lds_read_h8(lds, kA0 + off);
                const half8 a1 = lds_read_h8(lds, kA1 + off);
                o[tq] = mfma(vt, a0, o[tq]);
                o[tq] = mfma(vt, a1, o[tq]);
                const int row = 16 * tq + l16, col = 16 * cw + 4 * g4;
                if constexpr (kOutF32 || kC2)
                    *reinterpret_cast<float4v*>(lds + kO + (row * kORowF32 + col) * 4) = o[tq];
                else
                    *reinterpret_cast<uint2*>(lds + kO + (row * kORowBf16 + col) * 2) =
                        make_uint2(pack_bf2(o[tq][0], o[tq][1]), pack_bf2(o[tq][2], o[tq][3]));
            }
        }
        if (n >= 2 && n - 2 < total) {
            // chunk n-2: the state chain
            const char* lds = lds_all + (n & 1) * kBuf;
            if (at.c == 0) {
                // a unit begins: take its entering state, start fetching the next unit's
                if constexpr (kMulti) {
#pragma unroll
                    for (int nb = 0; nb < 4; ++nb) S[nb] = Snext[nb];
                    fetch_state(Snext, at.ui + 1, kTurn ? un.next_head(at.hd) : at.hd);
                }
            }
            // inter-chunk read: o[t][j] = sum_n (r_t W(t,-1))[n] S[n][j]; the state registers,
            // rounded to fp16, are the A operand (k-slot order = the r tile's column permutation)
            half8 sh[2];
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    sh[kk][e] = static_cast<_Float16>(S[2 * kk + (e >> 2)][e & 3]);
#pragma unroll
            for (int tq = 0; tq < 2; ++tq) {
                o[tq] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kk = 0; kk < 2; ++kk) {
                    const half8 rt = lds_read_h8(lds, kRT + (16 * tq + l16) * kRow + (32 * kk + 8 * g4) * 2);
                    o[tq] = mfma(sh[kk], rt, o[tq]);
                }
            }
            // The scheduler must not mix the two halves: with the LDS reads and products of the state update pulled up
            // between those of the read-out, the Finch form's window is 2 to 3 % longer (12 sequences of 10 218 tokens and 12
            // heads: 234.5 -> 226.3 us; one sequence of 4096 tokens and 32 heads, split, 36.0 -> 35.0).  Vector and scalar ALU
            // instructions may cross (mask 6: 100 sequences of 60 tokens and 64 heads, fp32 out, 81.9 -> 79.9 against a full
            // barrier), but for fp32 rows with one unit per workgroup (28.9 -> 28.5 us at 5 x 961 tokens x 16 heads with a full one).
            __builtin_amdgcn_sched_barrier(kOutF32 && !kMulti ? 0 : 6);
            // state update: S = diag(W(32,-1)) S + (k W(32,i))^T V over the chunk's 32 tokens
            vt = lds_read_h8(lds, kVT + tile_t_off(16 * cw + l16, g4));
#pragma unroll
            for (int nb = 0; nb < 4; ++nb) {
                const float4 d = *reinterpret_cast<const float4*>(lds + kD + (16 * nb + 4 * g4) * 4);
                S[nb][0] *= d.x;
                S[nb][1] *= d.y;
                S[nb][2] *= d.z;
                S[nb][3] *= d.w;
                const half8 kt = lds_read_h8(lds, kKT + tile_t_off(16 * nb + l16, g4));
                S[nb] = mfma(kt, vt, S[nb]);
            }
            if (at.c == un.nchunks - 1) {
                // the unit ends: its final state
                if (un.state_out) {
                    const __amdgpu_buffer_rsrc_t rs = state_rsrc(un.state_out, at.ui, at.hd);
#pragma unroll
                    for (int nb = 0; nb < 4; ++nb)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float value = S[nb][e];        // (a bit cast straight from the vector element reads element 0)
                            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(value), rs, state_voff,
                                                                  (16 * nb + e) * 256, kState);
                        }
                }
            }
            at.advance(1, un);
        }
        if constexpr (kLora) {
            if (dlive) {
                d_finish(n + 1, [&] {
                    dn.advance(1, un);
                    if (!kC2 || n + 2 < total) y_fetch(dn);
                });
            }
        }
        __syncthreads();                                                        // window barrier
    }
}

template <int kMode, bool kC2, bool kTurn, bool kMulti, Traffic kTraffic>
__global__ __launch_bounds__(kThreads) void chunked_kernel(Args a) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    clamp_fp16_overflow();
    const int tid = threadIdx.x;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    int unit = blockIdx.x;                       // (batch * segs + segment) * H + head
    if constexpr (kMode >= 4) {
        // Fused decay path: the heads of a batch share its y rows.  Workgroups go to the 8 XCDs
        // (each with its own L2) round-robin by index, so give XCD i the i-th eighth of the
        // units: neighbouring heads of a batch then read y through the same L2.
        const int per_xcd = gridDim.x >> 3;
        if ((gridDim.x & 7) == 0) unit = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    }
    const int bs = unit / a.H;
    const int h = unit - bs * a.H;
    const int b = bs / a.segs;
    const int seg = bs - b * a.segs;
    const long long tok_stride = static_cast<long long>(a.H) * kHeadSize;
    // The workgroup's units: this one and, when the launch gave a stride (a multiple of H, whole
    // sequences only), every stride-th unit after it, batch index advancing: same head, or the next one each time.
    Units un;
    un.t0 = seg * a.seg_len;
    const int T = a.T - un.t0 < a.seg_len ? a.T - un.t0 : a.seg_len;
    un.tokens = T;
    un.first = b * a.H + h;
    un.stride = a.unit_stride;
    un.state_out = seg == a.segs - 1 ? a.state_out : nullptr;      // only the last segment leaves the sequence's state
    un.entering = nullptr;
    if (a.segs > 1) un.entering = a.place.base + b * a.place.batch + seg * a.place.seg + h * a.place.head;
    un.pitch_row = a.place.row;
    un.pitch_half = a.place.half;
    un.heads = a.H;
    un.head0 = h;
    un.count = 1;
    un.nchunks = (T + kChunk - 1) / kChunk;
    un.base0 = static_cast<long long>(b) * a.batch_stride + un.t0 * tok_stride + static_cast<long long>(h) * kHeadSize;
    un.step = 0;
    if constexpr (kMulti) {
        const long long total = static_cast<long long>(a.B) * a.H;
        un.count = static_cast<int>((total - unit + a.unit_stride - 1) / a.unit_stride);
        un.step = static_cast<long long>(a.unit_stride / a.H) * a.batch_stride;
    }
    if (wid < 4 * kProducerGroups)
        producer<kMode, kC2, kTurn, kMulti, kTraffic>(a, lds, tid, wid >> 2, wid & 3, h, un, tok_stride, T);
    else
        consumer<kMode, kC2, kTurn, kMulti, kTraffic>(a, lds, tid & 63, wid - 4 * kProducerGroups, un);
}

template <int kMode, bool kC2>
constexpr int lds_bytes_of(bool turn, int heads) {
    return (kMode >= 4 ? kLdsBytesLora : kLdsBytes) + (turn && !kC2 ? heads * kHeadSize * 2 : 0);
}

// Which kernels take the heads in turn (heads_in_turn below): not those of a layer's modes, and in the Finch form with bf16 rows not
// beyond a GiB.
template <int kMode, bool kC2, Traffic kTraffic>
constexpr bool kHasTurn = kMode < 3 && (kTraffic == Traffic::kLarge || (kTraffic == Traffic::kStreamed && (kMode == 1 || kC2)));

template <int kMode, bool kC2>
hipError_t raise_mode_limits() {
    struct Tag {};
    return once_per_device<Tag>([] {
        constexpr int bytes = lds_bytes_of<kMode, kC2>(false, 0);
        [[maybe_unused]] constexpr int turn = lds_bytes_of<kMode, kC2>(true, kTurnHeads);
        hipError_t e = set_lds_limit(&chunked_kernel<kMode, kC2, false, false, Traffic::kCached>, bytes);
        if (e == hipSuccess) e = set_lds_limit(&chunked_kernel<kMode, kC2, false, true, Traffic::kCached>, bytes);
        if (e == hipSuccess) e = set_lds_limit(&chunked_kernel<kMode, kC2, false, false, Traffic::kLarge>, bytes);
        if (e == hipSuccess) e = set_lds_limit(&chunked_kernel<kMode, kC2, false, true, Traffic::kLarge>, bytes);
        if constexpr (kMode < 3)
            if (e == hipSuccess) e = set_lds_limit(&chunked_kernel<kMode, kC2, false, true, Traffic::kStreamed>, bytes);
        if constexpr (kHasTurn<kMode, kC2, Traffic::kLarge>)
            if (e == hipSuccess) e = set_lds_limit(&chunked_kernel<kMode, kC2, true, true, Traffic::kLarge>, turn);
        if constexpr (kHasTurn<kMode, kC2, Traffic::kStreamed>)
            if (e == hipSuccess) e = set_lds_limit(&chunked_kernel<kMode, kC2, true, true, Traffic::kStreamed>, turn);
        return e;
    });
}

// Whether the units of a workgroup take the heads in turn.  Where a token row is a multiple of 1 KiB, all rows of a head share
// address bits 7 to 9, and so do all streams of a unit where the tensors start equally aligned, as an allocator has them.  The memory serves one of
// the eight classes more slowly (a unit of it takes 7 % longer in the Finch form, 22 % in Finch-C2), so a workgroup that kept its
// head would end last, or early; in turn, each takes its share of every class.  Same head -> in turn, us, tensors of one allocation each:
// Finch-C2 256 x 512 tokens x 32 heads 688 -> 628, 16 x 4096 x 32 364 -> 351, 10 x 4000 x 40 317 -> 296, 32 x 300 x 32 54.1 -> 53.0; Finch
// 16 x 4096 x 32 323 -> 311, 10 x 5000 x 64 459 -> 436, 32 x 1000 x 32 140 -> 134, fp32 out 64 x 2500 x 32 804 -> 753.  Not taken: bf16 rows whose
// streams start 128 bytes apart, which lie in every class by themselves (Finch-C2 64 x 1000 x 32 298 -> 306; fp32 rows, of 256
// bytes, gain there too: 341 -> 323, Finch 64 x 2500 755 -> 727); Finch, bf16 out, from 1 GiB on, which the kernel's own cycles bound (64 x 1000 x
// 32 255 -> 257, 12 x 12 000 x 32 698 -> 700); calls that the memory-side cache holds for the most part, to 300 MiB in the Finch form with bf16
// rows (10 x 412 x 64 40.4 -> 41.0, 20 x 700 x 16 44.7 -> 45.1; at 306 MiB 24 x 600 x 32 65.5 -> 62.9), to 150 MiB in the others (20 x 60 x
// 32 13.6 -> 13.8, 9 x 500 x 32 39.4 -> 39.9; at 213 10 x 412 x 64 49.8 -> 49.2, fp32 out 20 x 300 x 32 36.8 -> 35.3); fewer units than one and
// three quarters rounds, most of whose workgroups have one (bf16 rows, 256 a round: Finch-C2 384 units x 900 tokens 70.9 -> 72.3, x 6000
// 425 -> 431, 416 x 2000 140.2 -> 141.2, 448 x 900 75.0 -> 73.5; Finch 384 x 1500 86.0 -> 86.5, 416 x 2000 113.5 -> 114.2, 448 x 2000 126 ->
// 123; fp32 rows gain or tie from one and a half rounds on: Finch-C2 384 x 600 53.4 -> 49.7, Finch 384 x 900 60.4 -> 59.8); and fused
// logits, whose consumers hold their head's slice of B in registers.
template <int kMode, bool kC2>
bool heads_in_turn(const Args& a, long long units, long long mib) {
    if (a.H % 8 != 0 || (!kC2 && a.H > kTurnHeads) || 4 * units < (kMode == 1 ? 6ll : 7ll) * a.unit_stride) return false;
    if (mib < (kMode == 1 || kC2 ? 150 : 300)) return false;
    if (kMode == 1) return true;
    const auto address_class = [](const void* p) { return reinterpret_cast<unsigned long long>(p) >> 7 & 7; };
    const auto c = address_class(a.r);
    return address_class(a.k) == c && address_class(a.v) == c && address_class(a.x) == c && address_class(a.out) == c &&
           (!kC2 || address_class(a.uprime) == c);
}

template <int kMode, bool kC2>
hipError_t launch_mode(const Args& args, hipStream_t stream) {
    const hipError_t err = raise_mode_limits<kMode, kC2>();
    if (err != hipSuccess) return err;
    Args a = args;
    long long units = static_cast<long long>(a.B) * a.segs * a.H;
    a.unit_stride = 0;
    // With more (batch, head) units than compute units each workgroup takes several of them back to back.
    const int cus = compute_units();
    if (a.segs == 1 && a.H <= cus) {
        const int per_round = a.H * (cus / a.H);                 // a multiple of H: every round begins with head 0
        if (units > per_round) {
            a.unit_stride = per_round;
            units = per_round;
        }
    }
    const dim3 grid(static_cast<unsigned>(units));
    const long long row_bytes = kHeadSize * 2 * (kMode >= 4 ? 3 : 4) + kHeadSize * (kMode == 1 ? 4 : 2) + (kC2 ? kHeadSize * 2 : 0);
    const long long mib = static_cast<long long>(a.B) * a.H * (a.T * row_bytes + 2 * 4096 * 4) >> 20;     // the call's rows and states
    auto go = [&](auto kernel, bool turn = false) {
        hipLaunchKernelGGL(kernel, grid, dim3(kThreads), (lds_bytes_of<kMode, kC2>(turn, a.H)), stream, a);
        return hipGetLastError();
    };
    const bool cached = mib < (kMode >= 3 ? 64 : 90);
    if (a.unit_stride == 0)
        return cached ? go(&chunked_kernel<kMode, kC2, false, false, Traffic::kCached>) : go(&chunked_kernel<kMode, kC2, false, false, Traffic::kLarge>);
    if (cached) return go(&chunked_kernel<kMode, kC2, false, true, Traffic::kCached>);
    auto several = [&](auto traffic) {
        constexpr Traffic kTraffic = decltype(traffic)::value;
        if constexpr (kHasTurn<kMode, kC2, kTraffic>)
            if (heads_in_turn<kMode, kC2>(a, static_cast<long long>(a.B) * a.H, mib)) return go(&chunked_kernel<kMode, kC2, true, true, kTraffic>, true);
        return go(&chunked_kernel<kMode, kC2, false, true, kTraffic>);
    };
    if constexpr (kMode < 3)
        if (mib >= 1024) return several(std::integral_constant<Traffic, Traffic::kStreamed>{});
    return several(std::integral_constant<Traffic, Traffic::kLarge>{});
}

}  // namespace

namespace {

// f(mode, form) with the two as compile-time constants
template <typename F>
hipError_t with_mode(const Args& a, ChunkedMode mode, F f) {
    constexpr std::true_type c2;
    constexpr std::false_type finch;
    switch (mode) {
        case ChunkedMode::kBf16Out: return a.finch_c2 ? f(std::integral_constant<int, 0>{}, c2) : f(std::integral_constant<int, 0>{}, finch);
        case ChunkedMode::kF32Out: return a.finch_c2 ? f(std::integral_constant<int, 1>{}, c2) : f(std::integral_constant<int, 1>{}, finch);
        case ChunkedMode::kBf16OutMoments:
            if (!a.finch_c2 || !a.moments) return hipErrorInvalidValue;
            return f(std::integral_constant<int, 3>{}, c2);
        default:
            if (!a.y || !a.lambda || !a.bw) return hipErrorInvalidValue;
            if (mode == ChunkedMode::kBf16OutLora)
                return a.finch_c2 ? f(std::integral_constant<int, 4>{}, c2) : f(std::integral_constant<int, 4>{}, finch);
            if (!a.finch_c2 || !a.moments) return hipErrorInvalidValue;
            return f(std::integral_constant<int, 5>{}, c2);
    }
}

}  // namespace

hipError_t raise_chunked_limits(const Args& a, ChunkedMode mode) {
    return with_mode(a, mode, [](auto m, auto c2) { return raise_mode_limits<decltype(m)::value, decltype(c2)::value>(); });
}

hipError_t launch_chunked(const Args& a, ChunkedMode mode, hipStream_t stream) {
    return with_mode(a, mode, [&](auto m, auto c2) { return launch_mode<decltype(m)::value, decltype(c2)::value>(a, stream); });
}

}  // namespace wkv6

// Chunked WKV6 prefill of fp32 tensors for gfx950 (MI355X), Finch form: everything in fp32, the contractions on the
// matrix cores (v_mfma_f32_16x16x4_f32, fp32 products and sums).  The recurrence (Finch-C2 Time Mixing: decay map
// w = exp(-exp(x)), wkv_t, read-out; Finch bonus u) in chunks of 16 tokens, S0 the state entering the chunk:
//
//     o_t = (r_t * W(t,-1)) . S0 + sum_{i<t} ( sum_n r_t[n] k_i[n] W(t,i)[n] ) v_i + ( sum_n r_t[n] u[n] k_t[n] ) v_t
//     S16 = diag(W(16,-1)) S0 + sum_i (k_i * W(16,i))^T v_i,         W(t,i) = prod_{s=i+1}^{t-1} w_s
//
// As in the bf16 chunked kernel only products of decays are formed, never a quotient or a positive exponent, and the
// causal triangle is cut by binary levels m = 8, 4, 2, 1: a pair (t, i) belongs to the highest bit in which the two differ, and
// with `mid` the middle of its 2m-aligned block W(t,i) = (prod_{mid <= s < t} w_s) (prod_{i < s < mid} w_s).  A level has
// eight queries and eight keys, so two levels share one 16 x 16 product (8 with 4, 2 with 1).
//
// A workgroup owns 16 kCB of a unit's 64 value columns (a state's columns do not depend on one another).  PRODUCER
// waves take whole chunks: lane n holds channel n of all 16 tokens, so every decay product is lane-local, the level tiles
// and the scores stay inside the wave, and only r W, k W, the scores and the total decay go to the consumers.  CONSUMERS (four waves)
// carry the state in MFMA accumulators: wave (cb, kh) columns 16 cb .. +15 and key part kh of 4 / kCB.  They walk the chunks
// of a round (one per producer) while the producers make the next round's: one barrier per round, two slots per producer.
// With kCB < 4 the partial read-outs of the key parts are added, and stored, by the producers one round later.
//
// Few units and many tokens (the rule is at the launch): a kernel of its own makes the scores first, a wave a chunk over the whole
// chip, and leaves them in the rows of `out` that the column groups write later, a copy for each: 16 scores a token are
// the 16 columns of a group.  The producers then only read them.  The same bits: 32 units x 512 tokens 31.7 -> 25.2 us, x 2048 112 -> 76; what is
// left per chunk is the producers' decays and the consumers' state products, 1100 clocks of a SIMD, vector and matrix
// instructions in turn.  (Rows fetched two rounds ahead instead of one: no gain, 25.9.)
//
// Bound by the vector ALUs: the fp32 matrix instructions run at twice their rate but do not overlap with them.  Per chunk a
// workgroup issues about 2900 clocks of vector work, 1024 of scores and 1152 kCB / 4 of state work per wave, over four
// SIMDs; a unit's column groups repeat the producers' part, so columns are spread only while compute units are idle.  The token-by-token
// kernels it replaces need 196 clocks a token at few units and 4 instructions per state element and 64 lanes at many.  Microseconds,
// token by token -> here: 32 units x 512 tokens 42.5 -> 31.7 (25.2 with the scores in a kernel of their own), x 128 14.4 -> 11.1; 128 x 512 75 -> 37.6; 256 x 512
// 130 -> 52.6, x 1000 247 -> 95; 512 x 512 197 -> 101.  Error against 64 bits no larger: `out` 9.4e-8 (9.4e-8), state 5.8e-8 (6.0e-8);
// that takes sums in pairs, tokens in their order, and decays from sums of exponents where the comments say so.
// Also tried: six or eight producers (more registers than three waves a SIMD have: up to 1.6 times slower), one register set
// with few columns (short sequences 10 to 20 % slower).
#include "wkv6_launch.h"
#include "wkv6_math.h"

namespace wkv6 {
namespace {

typedef float float4v __attribute__((ext_vector_type(4)));
typedef unsigned uint4v __attribute__((ext_vector_type(4)));

constexpr int kChunk = 16;
constexpr int kConsumers = 4;

// One chunk's hand-over (bytes).  A producer's level tiles, 16 query rows and 16 key rows of 64 channels, lie where its r W
// and k W go afterwards.
constexpr int kRow = 256 + 16;                       // row of 64 channels: 16-byte reads of 16 rows cover every bank once
constexpr int kOffRT = 0;                            // r W(t,-1)   [16 tokens][64 channels]
constexpr int kOffKT = kOffRT + kChunk * kRow;       // k W(16,i)   [64 channels][16 tokens]
constexpr int kOffA = kOffRT + 2 * kChunk * kRow;    // scores      [16 t][16 i], zero above the diagonal
constexpr int kOffD = kOffA + kChunk * 64;           // W(16,-1)    [64]
constexpr int kSlotBytes = kOffD + 256;
static_assert(kOffKT + 64 * 64 <= kOffA, "k W beside r W");

template <int kCB, int kProducers>
struct Shape {
    static constexpr int kKeyParts = 4 / kCB;
    // partial read-outs of the key parts and, behind them, scores times values: [part][column block][16 t][16 j]
    static constexpr int kSlot = kSlotBytes + (kKeyParts > 1 ? (kKeyParts + 1) * kCB * 1024 : 0);
    static constexpr int kLds = 2 * kProducers * kSlot;
    static constexpr int kThreads = 64 * (kProducers + kConsumers);
    static_assert(kLds <= 160 * 1024, "LDS budget");
    static_assert(kThreads == kChunkedF32Threads, "what the callers count with");
};

// Rows of 16 tokens are four granules of 16 bytes: granule g holds tokens g, 4 + g, 8 + g, 12 + g, so that a lane's read is its
// operand for four instructions which take the tokens in their order (the older ones, the smaller summands, first: the
// sums round less).  Rows four apart start at the same bank, hence the swizzle.
__device__ __forceinline__ int token_off(int row, int granule) { return row * 64 + ((granule ^ ((row >> 2) & 3)) << 4); }

__device__ __forceinline__ float4v mfma(float a, float b, float4v c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// Products over 16 channels, four instructions' sums added in pairs.  (In one chain over a head's 64 channels the
// rounding of the sums is what the result's error consists of: 1.6e-7 of `out` against 0.9e-7.)
__device__ __forceinline__ float4v four(float4v a, float4v b) {
    const float4v zero = {0.f, 0.f, 0.f, 0.f};
    return (mfma(a[0], b[0], zero) + mfma(a[1], b[1], zero)) + (mfma(a[2], b[2], zero) + mfma(a[3], b[3], zero));
}

__device__ __forceinline__ void wave_lds_order() {       // a wave's own LDS writes before its own reads, and back
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// log2(e) exp(x): the factor rides in the argument, as log2(log2(e)) rounded down; the second step adds what that loses
// (2e-8 of the value: without it the decays have a bias of 1e-8, which a long memory adds up)
__device__ __forceinline__ float exponent_of(float x) {
    constexpr float kLog2Log2e = 0.5287663340568542f, kRest = 2.695514e-08f;
    const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(x, kLog2e, kLog2Log2e));
    return __builtin_fmaf(e, kRest, e);
}
__device__ __forceinline__ float decay_over(float exponents) { return __builtin_amdgcn_exp2f(-exponents); }

template <int kCtrl>
__device__ __forceinline__ float dpp_lanes(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), kCtrl, 0xf, 0xf, false));
}
// v[0..15] of 64 lanes -> in every lane the sum over all lanes of v[lane >> 2]
__device__ __forceinline__ float sum_scatter16(float (&v)[16], int lane) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {                    // halves of the wave: v[i] and v[i + 8]
        const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i]), __float_as_uint(v[i + 8]), false, false);
        v[i] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {                    // rows of 16 lanes: v[i] and v[i + 4]
        const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[i]), __float_as_uint(v[i + 4]), false, false);
        v[i] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {                    // row_ror:8, lane ^ 8
        const float keep = lane & 8 ? v[i + 2] : v[i], give = lane & 8 ? v[i] : v[i + 2];
        v[i] = keep + dpp_lanes<0x128>(give);
    }
    const float keep = lane & 4 ? v[1] : v[0], give = lane & 4 ? v[0] : v[1];
    float s = keep + dpp_lanes<0x141>(give);         // row_half_mirror, 7 - lane of each 8
    s += dpp_lanes<0x4E>(s);                         // quad_perm [2,3,0,1]
    s += dpp_lanes<0xB1>(s);                         // quad_perm [1,0,3,2]
    return s;
}

// `v` again, unknown to the compiler: what is derived from it is formed here and not kept in registers from before the loop
__device__ __forceinline__ int here(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// The scores of a chunk, bonus on the diagonal, into the slot (which has zeros above the diagonal); the level tiles pass through
// the r W and k W of the slot.  kStaged: the compiler keeps the stages apart.  Without it registers are short where the
// next chunk's rows have their own, and the addresses are formed here (kept from outside, 16 registers spill: 32 -> 39 us).
template <bool kStaged>
__device__ __forceinline__ void chunk_scores(const float (&r)[kChunk], const float (&k)[kChunk], const float (&ex)[kChunk],
                                             const float (&w)[kChunk], float u, char* slot, int lane) {
    const int ln = kStaged ? lane : here(lane);
    const int l16 = ln & 15, g4 = ln >> 4;
    auto put = [&](int row, float v) { *reinterpret_cast<float*>(slot + row * kRow + 4 * ln) = v; };     // this lane's channel of a row
    auto stage_end = [] {
        if constexpr (kStaged) __builtin_amdgcn_sched_barrier(0);
    };
    // decays between a token and the middle of its 8-token half's block: behind a key, in front of a query
    float behind[8], before[8];
    behind[7] = before[0] = 1.f;
    float after = 0.f, until = 0.f;
#pragma unroll
    for (int i = 6; i >= 0; --i) behind[i] = decay_over(after += ex[i + 1]);
#pragma unroll
    for (int i = 1; i < 8; ++i) before[i] = decay_over(until += ex[7 + i]);
    // levels 8 and 4: query rows 0..7 are tokens 8.., rows 8..15 tokens 4..7 and 12..15; key rows (16 on) 0..7 and 0..3, 8..11
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        put(j, r[8 + j] * before[j]);
        put(16 + j, k[j] * behind[j]);
    }
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        const int b = 8 * half;
        const float s2 = w[b + 3], s1 = w[b + 2] * s2, s0 = w[b + 1] * s1;
        const float q1 = w[b + 4], q2 = q1 * w[b + 5], q3 = q2 * w[b + 6];
        put(24 + 4 * half, k[b] * s0);
        put(25 + 4 * half, k[b + 1] * s1);
        put(26 + 4 * half, k[b + 2] * s2);
        put(27 + 4 * half, k[b + 3]);
        put(8 + 4 * half, r[b + 4]);
        put(9 + 4 * half, r[b + 5] * q1);
        put(10 + 4 * half, r[b + 6] * q2);
        put(11 + 4 * half, r[b + 7] * q3);
    }
    wave_lds_order();
    // product of the tile: rows (registers) are keys, columns (lanes) queries
    auto scores = [&] {
        float4v sum[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4v qv = *reinterpret_cast<const float4v*>(slot + l16 * kRow + 64 * q + 16 * g4);
            const float4v kv = *reinterpret_cast<const float4v*>(slot + (16 + l16) * kRow + 64 * q + 16 * g4);
            sum[q] = four(kv, qv);
        }
        return (sum[0] + sum[1]) + (sum[2] + sum[3]);
    };
    const float4v s84 = scores();
    wave_lds_order();
    stage_end();
    // levels 2 and 1: query rows 0..7 are tokens 2, 3, 6, 7, .., rows 8..15 the odd ones; keys 0, 1, 4, 5, .. and the even ones
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        put(2 * b, r[4 * b + 2]);
        put(2 * b + 1, r[4 * b + 3] * w[4 * b + 2]);
        put(16 + 2 * b, k[4 * b] * w[4 * b + 1]);
        put(16 + 2 * b + 1, k[4 * b + 1]);
    }
#pragma unroll
    for (int m = 0; m < 8; ++m) {
        put(8 + m, r[2 * m + 1]);
        put(24 + m, k[2 * m]);
    }
    wave_lds_order();
    const float4v s21 = scores();
    wave_lds_order();
    stage_end();
    // bonus on the diagonal
    float diag[kChunk];
#pragma unroll
    for (int t = 0; t < kChunk; ++t) diag[t] = r[t] * u * k[t];
    const float dg = sum_scatter16(diag, lane);
    // the scores where the two of a pair meet: a lane has four keys of its query
    auto put_score = [&](int t, int i, float v) { *reinterpret_cast<float*>(slot + kOffA + token_off(t, i & 3) + 4 * (i >> 2)) = v; };
    if (l16 < 8 && g4 < 2) {                         // level 8
#pragma unroll
        for (int e = 0; e < 4; ++e) put_score(8 + l16, 4 * g4 + e, s84[e]);
    }
    if (l16 >= 8 && g4 == 2 + ((l16 >> 2) & 1)) {    // level 4
#pragma unroll
        for (int e = 0; e < 4; ++e) put_score(l16 < 12 ? l16 - 4 : l16, (l16 < 12 ? 0 : 8) + e, s84[e]);
    }
    if (l16 < 8 && g4 == (l16 >> 2)) {               // level 2
        const int blk = l16 >> 1;
        put_score(4 * blk + 2 + (l16 & 1), 4 * blk, blk & 1 ? s21[2] : s21[0]);
        put_score(4 * blk + 2 + (l16 & 1), 4 * blk + 1, blk & 1 ? s21[3] : s21[1]);
    }
    if (l16 >= 8 && g4 == (l16 >> 2)) {              // level 1
        const int m = l16 - 8, e = l16 & 3;
        put_score(2 * m + 1, 2 * m, e == 0 ? s21[0] : e == 1 ? s21[1] : e == 2 ? s21[2] : s21[3]);
    }
    if ((lane & 3) == 0) put_score(lane >> 2, lane >> 2, dg);
}

template <int kCB, int kProducers, bool kScored>
__device__ __forceinline__ void producer(const Args& a, char* lds, int lane, int p, int h, long long base, int col0, int nrounds) {
    using SH = Shape<kCB, kProducers>;
    const long long row_bytes = static_cast<long long>(a.H) * (kHeadSize * 4);
    const long long span = static_cast<long long>(a.T - 1) * row_bytes + kHeadSize * 4;
    const int nchunks = (a.T + kChunk - 1) / kChunk;
    const float u = a.u[h * kHeadSize + lane];
    // rows past the end read as zero (w is set to 1 there); past the last chunk the descriptor is empty
    auto fetch = [&](float (&d)[kChunk], const void* src, int c) {
        const __amdgpu_buffer_rsrc_t rs = chunk_rsrc(static_cast<const char*>(src) + base * 4, c < nchunks ? c * (kChunk * row_bytes) : span, span);
        const int at = 4 * here(lane);
#pragma unroll
        for (int t = 0; t < kChunk; ++t) d[t] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, static_cast<int>(t * row_bytes) + at, 0, 0));
    };
    // Columns spread over several workgroups leave each with little matrix work: the next chunk's rows have registers of
    // their own and the compiler may mix the stages.  A workgroup with all columns is better off with one set and a stage at a time.
    constexpr bool kTwoSets = kCB < 4;
    auto stage_end = [] {
        if constexpr (!kTwoSets) __builtin_amdgcn_sched_barrier(0);
    };
    struct Raw {
        float r[kChunk], k[kChunk], x[kChunk];
        float4v score;                                       // token lane >> 2, granule lane & 3
    };
    auto fetch_score = [&](float4v& d, int c) {
        if constexpr (kScored) {
            const __amdgpu_buffer_rsrc_t rs = chunk_rsrc(static_cast<const char*>(a.out) + base * 4, c < nchunks ? c * (kChunk * row_bytes) : span, span);
            d = __builtin_bit_cast(float4v, __builtin_amdgcn_raw_buffer_load_b128(
                                                rs, static_cast<int>((lane >> 2) * row_bytes) + (col0 + 4 * (lane & 3)) * 4, 0, 0));
        }
    };
    auto round = [&](int rd, Raw& raw, Raw& next) {
        float(&r)[kChunk] = raw.r, (&k)[kChunk] = raw.k, (&x)[kChunk] = raw.x;
        char* slot = lds + ((rd & 1) * kProducers + p) * SH::kSlot;
        const int c = rd * kProducers + p;
        if constexpr (SH::kKeyParts > 1) {
            // the finished chunk of two rounds ago: its key parts' partial read-outs, added and stored
            const int done = c - 2 * kProducers;
            if (done >= 0 && done < nchunks) {
                const int t = lane >> 2, quad = lane & 3;
                const __amdgpu_buffer_rsrc_t ro = chunk_rsrc(static_cast<const char*>(a.out) + base * 4, done * (kChunk * row_bytes), span);
#pragma unroll
                for (int cb = 0; cb < kCB; ++cb) {
                    auto part = [&](int kh) { return *reinterpret_cast<const float4v*>(slot + kSlotBytes + (kh * kCB + cb) * 1024 + token_off(t, quad)); };
                    float4v sum = part(0) + part(1);
                    if constexpr (SH::kKeyParts == 4) sum += part(2) + part(3);
                    sum += part(SH::kKeyParts);
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uint4v, sum), ro,
                                                           static_cast<int>(t * row_bytes) + (col0 + 16 * cb + 4 * quad) * 4, 0, 0);
                }
            }
        }
        if (c < nchunks) {
            if constexpr (kTwoSets) {
                fetch(next.x, a.x, c + kProducers);
                fetch(next.r, a.r, c + kProducers);
                fetch(next.k, a.k, c + kProducers);
                fetch_score(next.score, c + kProducers);
            }
            float ex[kChunk], w[kChunk];                     // w = 2^-ex
#pragma unroll
            for (int t = 0; t < kChunk; ++t) {
                ex[t] = exponent_of(x[t]);
                if (c * kChunk + t >= a.T) ex[t] = 0.f;      // uniform
                w[t] = decay_over(ex[t]);
            }
            if constexpr (!kTwoSets) fetch(x, a.x, c + kProducers);
            stage_end();
            if constexpr (kScored) *reinterpret_cast<float4v*>(slot + kOffA + token_off(lane >> 2, lane & 3)) = raw.score;
            else chunk_scores<!kTwoSets>(r, k, ex, w, u, slot, lane);
            auto put = [&](int row, float v) { *reinterpret_cast<float*>(slot + row * kRow + 4 * lane) = v; };     // this lane's channel of a row
            // r W(t,-1), k W(16,i) and the chunk's decay
            stage_end();
            // each decay from the sum of its exponents: one rounding that matters where a product of 15 has 14
            float sum = 0.f;
#pragma unroll
            for (int t = 0; t < kChunk; ++t) {
                put(t, t ? r[t] * decay_over(sum) : r[t]);
                sum += ex[t];
            }
            *reinterpret_cast<float*>(slot + kOffD + 4 * lane) = decay_over(sum);
            sum = 0.f;
#pragma unroll
            for (int i = kChunk - 1; i >= 0; --i) {
                if (i < kChunk - 1) k[i] *= decay_over(sum);
                sum += ex[i];
            }
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *reinterpret_cast<float4v*>(slot + kOffKT + token_off(lane, g)) = float4v{k[g], k[4 + g], k[8 + g], k[12 + g]};
            if constexpr (!kTwoSets) {
                stage_end();
                fetch(r, a.r, c + kProducers);
                fetch(k, a.k, c + kProducers);
                fetch_score(raw.score, c + kProducers);
            }
        }
        __syncthreads();                                     // round barrier
    };
    Raw raw0;
    fetch(raw0.x, a.x, p);
    fetch(raw0.r, a.r, p);
    fetch(raw0.k, a.k, p);
    fetch_score(raw0.score, p);
    int rd = 0;
    if constexpr (kTwoSets) {
        Raw raw1;
#pragma clang loop unroll(disable)
        for (; rd + 1 < nrounds; rd += 2) {
            round(rd, raw0, raw1);
            round(rd + 1, raw1, raw0);
        }
        if (rd < nrounds) round(rd, raw0, raw1);
    } else {
#pragma clang loop unroll(disable)
        for (; rd < nrounds; ++rd) round(rd, raw0, raw0);
    }
}

template <int kCB, int kProducers>
__device__ __forceinline__ void consumer(const Args& a, char* lds, int lane, int cw, int unit, long long base, int col0, int nrounds) {
    using SH = Shape<kCB, kProducers>;
    const int l16 = lane & 15, g4 = lane >> 4;
    const int cb = cw % kCB, kh = cw / kCB;                  // column block; key part: blocks kh kCB .. of 16 keys
    const int j = col0 + 16 * cb + l16;
    const long long row_bytes = static_cast<long long>(a.H) * (kHeadSize * 4);
    const long long span = static_cast<long long>(a.T - 1) * row_bytes + kHeadSize * 4;
    const int nchunks = (a.T + kChunk - 1) / kChunk;

    // S[nb][e] = state[16 (kh kCB + nb) + 4 g4 + e][j]
    float4v S[kCB];
    const long long s_at = static_cast<long long>(unit) * (kHeadSize * kHeadSize) + (16 * kh * kCB + 4 * g4) * kHeadSize + j;
#pragma unroll
    for (int nb = 0; nb < kCB; ++nb)
#pragma unroll
        for (int e = 0; e < 4; ++e) S[nb][e] = a.state_in ? a.state_in[s_at + (16 * nb + e) * kHeadSize] : 0.f;

    // v of a chunk as operand: tokens 4 e + g4 of column j, fetched a round ahead
    int voff[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) voff[e] = static_cast<int>((4 * e + g4) * row_bytes) + 4 * j;
    auto fetch = [&](float4v& d, int c) {
        const __amdgpu_buffer_rsrc_t rs = chunk_rsrc(static_cast<const char*>(a.v) + base * 4, c < nchunks ? c * (kChunk * row_bytes) : span, span);
#pragma unroll
        for (int e = 0; e < 4; ++e) d[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, voff[e], 0, 0));
    };
    float4v v[kProducers];
#pragma unroll
    for (int i = 0; i < kProducers; ++i) fetch(v[i], i);
    const int o_voff = static_cast<int>(l16 * row_bytes) + (col0 + 16 * cb + 4 * g4) * 4;

    // the scores are zero above the diagonal for good
    for (int i = cw * 64 + lane; i < 2 * kProducers * 256; i += 64 * kConsumers)
        *reinterpret_cast<float*>(lds + (i >> 8) * SH::kSlot + kOffA + 4 * (i & 255)) = 0.f;
    __syncthreads();                                         // start barrier

    __syncthreads();                                         // round 0: nothing to do yet
#pragma clang loop unroll(disable)
    for (int rd = 1; rd < nrounds; ++rd) {
        char* slots = lds + ((rd - 1) & 1) * kProducers * SH::kSlot;
        const int c0 = (rd - 1) * kProducers;
        struct Ops {
            float4v rt[kCB], kt[kCB], d[kCB], am;
        };
        auto read = [&](Ops& q, const char* slot) {
#pragma unroll
            for (int nb = 0; nb < kCB; ++nb) {
                const int blk = kh * kCB + nb;
                q.rt[nb] = *reinterpret_cast<const float4v*>(slot + kOffRT + l16 * kRow + 64 * blk + 16 * g4);
                q.kt[nb] = *reinterpret_cast<const float4v*>(slot + kOffKT + token_off(16 * blk + l16, g4));
                q.d[nb] = *reinterpret_cast<const float4v*>(slot + kOffD + (16 * blk + 4 * g4) * 4);
            }
            q.am = *reinterpret_cast<const float4v*>(slot + kOffA + token_off(l16, g4));
        };
        // an infinite or undefined value must not meet the zeros above the diagonal; its product with zero is not a number
        float zero = 0.f;
#pragma unroll
        for (int i = 0; i < kProducers; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) zero = __builtin_fmaf(v[i][e], 0.f, zero);
        const bool finite = __all(zero == 0.f);
        constexpr int kAhead = kCB < 4 ? 1 : 0;              // a chunk's operands are read while the one before is worked on, registers allowing
        Ops ops[1 + kAhead];
        if constexpr (kAhead) read(ops[0], slots);
#pragma unroll
        for (int i = 0; i < kProducers; ++i) {
            if (i + kAhead < kProducers) read(ops[(i + kAhead) % (1 + kAhead)], slots + (i + kAhead) * SH::kSlot);      // (a slot without a chunk is not used)
            if (c0 + i < nchunks) {                          // uniform
                char* slot = slots + i * SH::kSlot;
                const float4v(&rt)[kCB] = ops[i % (1 + kAhead)].rt, (&kt)[kCB] = ops[i % (1 + kAhead)].kt, (&d)[kCB] = ops[i % (1 + kAhead)].d;
                const float4v am = ops[i % (1 + kAhead)].am;
                // read-out, transposed: lane (t = l16) gets columns 4 g4 + e of the block
                float4v part[kCB];
#pragma unroll
                for (int nb = 0; nb < kCB; ++nb) part[nb] = four(S[nb], rt[nb]);
                float4v o;
                if constexpr (kCB == 4) o = (part[0] + part[1]) + (part[2] + part[3]);
                else if constexpr (kCB == 2) o = part[0] + part[1];
                else o = part[0];
                // scores times values: one key part, in turn
                float4v av = {0.f, 0.f, 0.f, 0.f};
                const bool mine = i % SH::kKeyParts == kh;   // uniform
                if (mine) {
                    if (__builtin_expect(finite, 1)) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) av = mfma(v[i][e], am[e], av);
                    } else {
#pragma unroll
                        for (int s = 0; s < kChunk; ++s) {
                            const float score = *reinterpret_cast<const float*>(slot + kOffA + token_off(l16, s & 3) + 4 * (s >> 2));
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const float val = __shfl(v[i][s >> 2], (s & 3) * 16 + 4 * g4 + e, 64);
                                if (s <= l16) av[e] = __builtin_fmaf(score, val, av[e]);
                            }
                        }
                    }
                }
                // state
#pragma unroll
                for (int nb = 0; nb < kCB; ++nb) {
                    S[nb] *= d[nb];
#pragma unroll
                    for (int e = 0; e < 4; ++e) S[nb] = mfma(kt[nb][e], v[i][e], S[nb]);
                }
                if constexpr (SH::kKeyParts > 1) {
                    *reinterpret_cast<float4v*>(slot + kSlotBytes + (kh * kCB + cb) * 1024 + token_off(l16, g4)) = o;
                    if (mine) *reinterpret_cast<float4v*>(slot + kSlotBytes + (SH::kKeyParts * kCB + cb) * 1024 + token_off(l16, g4)) = av;
                } else {
                    o += av;
                    const __amdgpu_buffer_rsrc_t ro = chunk_rsrc(static_cast<const char*>(a.out) + base * 4, (c0 + i) * (kChunk * row_bytes), span);
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uint4v, o), ro, o_voff, 0, 0);
                }
                fetch(v[i], c0 + i + kProducers);
            }
        }
        __syncthreads();                                     // round barrier
    }
    if (a.state_out) {
#pragma unroll
        for (int nb = 0; nb < kCB; ++nb)
#pragma unroll
            for (int e = 0; e < 4; ++e) a.state_out[s_at + (16 * nb + e) * kHeadSize] = S[nb][e];
    }
}

template <int kCB, int kProducers, bool kScored>
__device__ __forceinline__ void chunks_of_a_unit(const Args& a, char* lds) {
    using SH = Shape<kCB, kProducers>;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Workgroups go round the 8 XCDs by index: a unit's column groups take consecutive turns of one XCD, so that r, k and x
    // reach its L2 once.
    const int turn = blockIdx.x >> 3;
    const int unit = turn / SH::kKeyParts * 8 + (blockIdx.x & 7);
    const int col0 = turn % SH::kKeyParts * (16 * kCB);
    if (unit >= a.B * a.H) return;                           // padding of the units to a multiple of 8
    const int b = unit / a.H, h = unit - b * a.H;
    const long long base = static_cast<long long>(b) * a.batch_stride + static_cast<long long>(h) * kHeadSize;
    const int nchunks = (a.T + kChunk - 1) / kChunk;
    // rounds of production, one more for the consumers, one more for the sums
    const int nrounds = (nchunks + kProducers - 1) / kProducers + (SH::kKeyParts > 1 ? 2 : 1);
    if (wave < kProducers) {
        __syncthreads();                                     // start barrier
        producer<kCB, kProducers, kScored>(a, lds, lane, wave, h, base, col0, nrounds);
    } else {
        consumer<kCB, kProducers>(a, lds, lane, wave - kProducers, unit, base, col0, nrounds);
    }
}

template <int kCB, int kProducers>
__global__ __launch_bounds__((Shape<kCB, kProducers>::kThreads)) void chunked_f32_kernel(Args a) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    chunks_of_a_unit<kCB, kProducers, false>(a, lds);
}

// Few units and many tokens: the scores come from a kernel of their own, below, that all compute units share in
template <int kCB, int kProducers>
__global__ __launch_bounds__((Shape<kCB, kProducers>::kThreads)) void chunked_f32_scored_kernel(Args a) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    chunks_of_a_unit<kCB, kProducers, true>(a, lds);
}

// The scores of every chunk of every unit, a wave a chunk, into `out`: row t of a chunk holds its 16 scores in the granules of
// token_off, once for each column group that will read them (and then write its outputs over them).
constexpr int kScoreWaves = 4;
constexpr long long kMaxScoreGroups = 1 << 20;       // workgroups; their waves go on to further chunks
__global__ __launch_bounds__(64 * kScoreWaves) void chunked_f32_scores_kernel(Args a, int group_columns) {
    __shared__ __attribute__((aligned(16))) char lds[kScoreWaves * kSlotBytes];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    char* slot = lds + wave * kSlotBytes;
    const int t = lane >> 2, quad = lane & 3;
    *reinterpret_cast<float4v*>(slot + kOffA + token_off(t, quad)) = float4v{0.f, 0.f, 0.f, 0.f};
    const int nchunks = (a.T + kChunk - 1) / kChunk;
    const long long row_bytes = static_cast<long long>(a.H) * (kHeadSize * 4);
    const long long span = static_cast<long long>(a.T - 1) * row_bytes + kHeadSize * 4;
    const long long jobs = static_cast<long long>(a.B) * a.H * nchunks, step = static_cast<long long>(gridDim.x) * kScoreWaves;
#pragma clang loop unroll(disable)
    for (long long job = static_cast<long long>(blockIdx.x) * kScoreWaves + wave; job < jobs; job += step) {
        const int unit = static_cast<int>(job / nchunks), c = static_cast<int>(job - static_cast<long long>(unit) * nchunks);
        const int b = unit / a.H, h = unit - b * a.H;
        const long long base = static_cast<long long>(b) * a.batch_stride + static_cast<long long>(h) * kHeadSize;
        float r[kChunk], k[kChunk], x[kChunk], ex[kChunk], w[kChunk];
        auto fetch = [&](float (&d)[kChunk], const void* src) {
            const __amdgpu_buffer_rsrc_t rs = chunk_rsrc(static_cast<const char*>(src) + base * 4, c * (kChunk * row_bytes), span);
#pragma unroll
            for (int i = 0; i < kChunk; ++i) d[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, static_cast<int>(i * row_bytes) + 4 * lane, 0, 0));
        };
        fetch(x, a.x);
        fetch(r, a.r);
        fetch(k, a.k);
        const float u = a.u[h * kHeadSize + lane];
#pragma unroll
        for (int i = 0; i < kChunk; ++i) {
            ex[i] = exponent_of(x[i]);
            if (c * kChunk + i >= a.T) ex[i] = 0.f;
            w[i] = decay_over(ex[i]);
        }
        chunk_scores<false>(r, k, ex, w, u, slot, lane);
        wave_lds_order();
        const uint4v row = *reinterpret_cast<const uint4v*>(slot + kOffA + token_off(t, quad));
        const __amdgpu_buffer_rsrc_t ro = chunk_rsrc(static_cast<const char*>(a.out) + base * 4, c * (kChunk * row_bytes), span);
        for (int col = 0; col < kHeadSize; col += group_columns)
            __builtin_amdgcn_raw_buffer_store_b128(row, ro, static_cast<int>(t * row_bytes) + (col + 4 * quad) * 4, 0, 0);
        wave_lds_order();
    }
}

}  // namespace

template <int kCB, int kProducers>
hipError_t launch_cb(const Args& a, bool scored, hipStream_t stream) {
    using SH = Shape<kCB, kProducers>;
    const unsigned units = (static_cast<unsigned>(a.B) * static_cast<unsigned>(a.H) + 7) / 8 * 8;
    const dim3 grid(units * SH::kKeyParts), block(SH::kThreads);
    if constexpr (kCB == 1) {
        if (scored) {
            const long long groups = (static_cast<long long>(a.B) * a.H * ((a.T + kChunk - 1) / kChunk) + kScoreWaves - 1) / kScoreWaves;
            hipLaunchKernelGGL(chunked_f32_scores_kernel, dim3(static_cast<unsigned>(groups < kMaxScoreGroups ? groups : kMaxScoreGroups)),
                               dim3(64 * kScoreWaves), 0, stream, a, 16 * kCB);
            const hipError_t err = hipGetLastError();
            if (err != hipSuccess) return err;
            hipLaunchKernelGGL((chunked_f32_scored_kernel<kCB, kProducers>), grid, block, SH::kLds, stream, a);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((chunked_f32_kernel<kCB, kProducers>), grid, block, SH::kLds, stream, a);
    return hipGetLastError();
}

hipError_t raise_chunked_f32_limits() {
    struct Tag {};
    return once_per_device<Tag>([] {
        hipError_t e = set_lds_limit(&chunked_f32_kernel<1, 4>, Shape<1, 4>::kLds);
        if (e == hipSuccess) e = set_lds_limit(&chunked_f32_scored_kernel<1, 4>, Shape<1, 4>::kLds);
        if (e == hipSuccess) e = set_lds_limit(&chunked_f32_kernel<2, 4>, Shape<2, 4>::kLds);
        if (e == hipSuccess) e = set_lds_limit(&chunked_f32_kernel<4, 4>, Shape<4, 4>::kLds);
        return e;
    });
}

hipError_t launch_chunked_f32(const Args& a, hipStream_t stream) {
    const hipError_t err = raise_chunked_f32_limits();
    if (err != hipSuccess) return err;
    // Column groups while the workgroups fit the chip once
    const long long cus = compute_units(), units = static_cast<long long>(a.B) * a.H;
    // Scores in a kernel of their own: a launch more (2 to 3 us) against 0.4 us a chunk, and the more units the longer that
    // kernel takes itself.  Microseconds, one kernel : two: 4 units 192 tokens 14.1 : 14.4, 224 16.9 : 15.7; 16 units 192
    // 14.4 : 14.7, 224 17.3 : 15.9; 32 units 224 17.4 : 16.5, 256 18.0 : 17.1, 512 31.7 : 25.3, 2048 112 : 76; 48 units 256 18.1 : 17.9,
    // 320 21.5 : 20.1; 64 units 256 18.4 : 18.5, 320 21.7 : 22.1, 512 32.1 : 28.8, 2048 122 : 102.  With two or four column blocks a workgroup
    // the producers' part is hardly repeated and one kernel is the better one: 128 units x 512 37.8 : 42.2, 256 x 512 52.5 : 75.
    if (4 * units <= cus) return launch_cb<1, 4>(a, a.T >= 200 + 2 * units, stream);
    if (2 * units <= cus) return launch_cb<2, 4>(a, false, stream);
    return launch_cb<4, 4>(a, false, stream);
}

}  // namespace wkv6

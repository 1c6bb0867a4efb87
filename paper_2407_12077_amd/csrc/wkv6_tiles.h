// What the kernels that evaluate 32-token chunks share (wkv6_chunked.hip, which also explains the method, and wkv6_short.hip):
// the operands that a thread forms from its four tokens of a channel pair, the choice of a score's level, and the
// finished rows.
#pragma once
#include "wkv6_launch.h"
#include "wkv6_math.h"

namespace wkv6 {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef unsigned uint2v __attribute__((ext_vector_type(2)));
typedef unsigned uint4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kChunk = kChunkTokens;       // tokens per chunk
constexpr int kORowF32 = 68;               // output staging row stride, fp32 mode (floats)
constexpr int kORowBf16 = 72;              // output staging row stride, bf16 mode (halfs)

// Cache policy of the streams that are touched exactly once (r, k, v, x, u', out): the
// non-temporal bit, so they do not displace each other in the caches on their way through.
constexpr int kStreamOnce = 2;
// Cache policy of the output rows: scope bit sc1 without the non-temporal bit, i.e. written
// through the XCD's L2 as they are produced instead of lingering there as dirty lines.  Measured
// with a streaming probe of this layout (four non-temporal input streams, one output stream of
// 128-byte rows 4 KiB apart): 130.7 us against 135.8 us with non-temporal stores.
constexpr int kStoreThrough = 16;

// two floats to a bf16 pair (round to nearest even), one packed conversion
__device__ __forceinline__ unsigned pack_bf2(float a, float b) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float float2v __attribute__((ext_vector_type(2)));
    const float2v f = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(f, bf16x2));
}

__device__ __forceinline__ half8 lds_read_h8(const char* lds, int byte_off) {
    return *reinterpret_cast<const half8*>(lds + byte_off);
}
__device__ __forceinline__ void lds_write_u32(char* lds, int byte_off, unsigned val) {
    *reinterpret_cast<unsigned*>(lds + byte_off) = val;
}
__device__ __forceinline__ void lds_write_u64(char* lds, int byte_off, unsigned lo, unsigned hi) {
    *reinterpret_cast<uint2*>(lds + byte_off) = make_uint2(lo, hi);
}
// low halves / high halves of two packed fp16 pairs as one pair
__device__ __forceinline__ unsigned lo_halves(unsigned a, unsigned b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }
__device__ __forceinline__ unsigned hi_halves(unsigned a, unsigned b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }

__device__ __forceinline__ float4v mfma(half8 a, half8 b, float4v c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// Sum over the 8 lanes of an aligned group of 8 (every lane gets the total): neighbours, pairs,
// then the mirrored half-row, all as data-parallel-primitive moves inside the vector ALU.
template <int kCtrl>
__device__ __forceinline__ float dpp_move(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), kCtrl, 0xf, 0xf, false));
}
__device__ __forceinline__ float row8_sum(float v) {
    v += dpp_move<0xB1>(v);       // quad_perm [1,0,3,2]
    v += dpp_move<0x4E>(v);       // quad_perm [2,3,0,1]
    v += dpp_move<0x141>(v);      // row_half_mirror: lane i <-> 7 - i of each 8
    return v;
}

struct Raw {           // one chunk's inputs of a producer thread: 4 tokens x one channel pair
    unsigned r[4], k[4], v[4], x[4];
};

// The decays of the four tokens and, Finch-C2, the key factors 1 - w, of a channel pair from its logits.
template <bool kC2>
__device__ __forceinline__ void decays_of(const unsigned (&x)[4], float (&w)[2][4], float (&omw)[2][4]) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        float e0 = 0.f, e1 = 0.f;
        w[0][s] = decay_of(bf16_lo(x[s]), e0);
        w[1][s] = decay_of(bf16_hi(x[s]), e1);
        if constexpr (kC2) {
            omw[0][s] = one_minus_decay(e0, w[0][s]);
            omw[1][s] = one_minus_decay(e1, w[1][s]);
        }
    }
}

// What a producer thread carries from phase D (where it digests the raw inputs of its chunk)
// to phase T (where the other groups' decay totals are known and the tiles are written).
struct Prep {
    unsigned z2[4], q1[4], k1[4];                         // finished fp16 pairs (two channels), one per token
    unsigned vt[4];            // v as fp16 pairs of consecutive tokens: [2*channel + token pair]
    unsigned rp[4];            // r * prefix product inside the group, fp16 pair (2 channels)
    unsigned ks[4];            // k * suffix product inside the group, fp16 pair
};

// Forms them from the rows and the decays; returns the group's decays, whole.  hu: the bonus u of the channel
// pair as an fp16 pair (Finch form only).
template <bool kC2>
__device__ __forceinline__ float2 form_operands(Prep& pr, const Raw& cur, const float (&w)[2][4], const float (&omw)[2][4], unsigned hu) {
    // products of decays inside the group, fp32: prefix of token 2 and 3, suffix of token 1
    // and 0, and the group total
    float p2[2], p3[2], s1[2], s0[2];
#pragma unroll
    for (int ch = 0; ch < 2; ++ch) {
        p2[ch] = w[ch][0] * w[ch][1];
        p3[ch] = p2[ch] * w[ch][2];
        s1[ch] = w[ch][2] * w[ch][3];
        s0[ch] = w[ch][1] * s1[ch];
    }
    // r, k, v as fp16 channel pairs (exact: bf16 has fewer significant bits); every scaled
    // operand is one packed fp16 multiply with a multiplier rounded to fp16
    unsigned rh[4], kh[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        rh[s] = pack_h2(bf16_lo(cur.r[s]), bf16_hi(cur.r[s]));
        if constexpr (kC2)      // Finch-C2: k = kbar (1 - w), the factor applied in fp32
            kh[s] = pack_h2(bf16_lo(cur.k[s]) * omw[0][s], bf16_hi(cur.k[s]) * omw[1][s]);
        else
            kh[s] = pack_h2(bf16_lo(cur.k[s]), bf16_hi(cur.k[s]));
    }
    // v goes to a transposed tile: pairs of consecutive tokens of one channel
    pr.vt[0] = pack_h2(bf16_lo(cur.v[0]), bf16_lo(cur.v[1]));
    pr.vt[1] = pack_h2(bf16_lo(cur.v[2]), bf16_lo(cur.v[3]));
    pr.vt[2] = pack_h2(bf16_hi(cur.v[0]), bf16_hi(cur.v[1]));
    pr.vt[3] = pack_h2(bf16_hi(cur.v[2]), bf16_hi(cur.v[3]));
    pr.rp[0] = rh[0];
    pr.rp[1] = mul_h2(rh[1], pack_h2(w[0][0], w[1][0]));
    pr.rp[2] = mul_h2(rh[2], pack_h2(p2[0], p2[1]));
    pr.rp[3] = mul_h2(rh[3], pack_h2(p3[0], p3[1]));
    const unsigned hw3 = pack_h2(w[0][3], w[1][3]);
    pr.ks[0] = mul_h2(kh[0], pack_h2(s0[0], s0[1]));
    pr.ks[1] = mul_h2(kh[1], pack_h2(s1[0], s1[1]));
    pr.ks[2] = mul_h2(kh[2], hw3);
    pr.ks[3] = kh[3];
    // level 2: tokens 0,1 of the group are keys, 2,3 queries
    pr.z2[0] = mul_h2(kh[0], pack_h2(w[0][1], w[1][1]));
    pr.z2[1] = kh[1];
    pr.z2[2] = rh[2];
    pr.z2[3] = mul_h2(rh[3], pack_h2(w[0][2], w[1][2]));
    // level 1 (odd token t reads even token t-1, no decay between them) and the bonus on the
    // diagonal share one query tile and one key tile: u rides on the query for even tokens
    // and on the key for odd tokens, so the diagonal gets r.u.k and the pair gets plain r.k
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        if constexpr (kC2) {
            // no diagonal term: one tile, keys in the even token rows, receptances in the odd ones
            pr.q1[s] = (s & 1) ? rh[s] : kh[s];
        } else {
            pr.q1[s] = (s & 1) ? rh[s] : mul_h2(rh[s], hu);
            pr.k1[s] = !(s & 1) ? kh[s] : mul_h2(kh[s], hu);
        }
    }
    return make_float2(p3[0] * w[0][3], p3[1] * w[1][3]);
}

// Scores of a 16 x 16 diagonal block, keys 4 g4 .. +3 of query l16, from the levels' products: the pair's level is the highest bit in
// which the two differ.
template <bool kC2>
__device__ __forceinline__ uint2 choose_levels(const float4v& acc8, const float4v& acc4, const float4v& acc2, const float4v& acc1, int l16, int g4) {
    float sel[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int i = 4 * g4 + e, t = l16;
        const int d = i ^ t;
        const float val = d >= 8 ? acc8[e] : d >= 4 ? acc4[e] : d >= 2 ? acc2[e] : acc1[e];
        sel[e] = (kC2 ? i >= t : i > t) ? 0.f : val;    // Finch-C2 has no diagonal term
    }
    return make_uint2(pack_h2(sel[0], sel[1]), pack_h2(sel[2], sel[3]));
}

// Eight finished values of a row: u' added (Finch-C2)
__device__ __forceinline__ void add_uprime(float4& q0, float4& q1, const uint4v& up_raw) {
    q0.x += bf16_lo(up_raw[0]); q0.y += bf16_hi(up_raw[0]);
    q0.z += bf16_lo(up_raw[1]); q0.w += bf16_hi(up_raw[1]);
    q1.x += bf16_lo(up_raw[2]); q1.y += bf16_hi(up_raw[2]);
    q1.z += bf16_lo(up_raw[3]); q1.w += bf16_hi(up_raw[3]);
}
// The 8 threads of a row hold the head's 64 finished values of this token: their
// sum, then the squared deviations from the head's own mean, each folded over
// the 8 lanes.
typedef float float2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float2v row_moments(const float4& q0, const float4& q1) {
    const float s = row8_sum(((q0.x + q0.y) + (q0.z + q0.w)) + ((q1.x + q1.y) + (q1.z + q1.w)));
    const float m = s * (1.f / kHeadSize);
    float m2 = (q0.x - m) * (q0.x - m);
    m2 = fmaf(q0.y - m, q0.y - m, m2);
    m2 = fmaf(q0.z - m, q0.z - m, m2);
    m2 = fmaf(q0.w - m, q0.w - m, m2);
    m2 = fmaf(q1.x - m, q1.x - m, m2);
    m2 = fmaf(q1.y - m, q1.y - m, m2);
    m2 = fmaf(q1.z - m, q1.z - m, m2);
    m2 = fmaf(q1.w - m, q1.w - m, m2);
    m2 = row8_sum(m2);
    return float2v{s, m2};
}
__device__ __forceinline__ uint4v pack_row(const float4& q0, const float4& q1) {
    uint4v q;
    q.x = pack_bf2(q0.x, q0.y);
    q.y = pack_bf2(q0.z, q0.w);
    q.z = pack_bf2(q1.x, q1.y);
    q.w = pack_bf2(q1.z, q1.w);
    return q;
}

}  // namespace
}  // namespace wkv6

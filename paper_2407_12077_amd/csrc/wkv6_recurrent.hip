// Token-by-token WKV6 kernel for gfx950: one wavefront per (batch, head), or four that share its key rows; lane j owns
// column j of the state (64 or 16 fp32 registers), r/k/w of the current token are exchanged
// through LDS and read back as broadcasts.  Follows the recurrence one step at a time
// (Finch-C2 Time Mixing: decay map, wkv_t, read-out; plus the Finch bonus u):
//     o_t[j] = sum_i r_t[i] S[i][j]  +  (sum_i r_t[i] u[i] k_t[i]) v_t[j]
//     S[i][j] = w_t[i] S[i][j] + k_t[i] v_t[j],   w_t = exp(-exp(x_t))
// It is bound by the fp32 vector ALUs (about 3*N*N operations per token and head), which
// is why the chunked kernel exists; this one serves the decode / short-append shapes (one or a
// few tokens per sequence, many sequences), where the work is streaming the fp32 state through
// once: 64 (16) row loads of 256 contiguous bytes per wave, all in flight together.  Long sequences
// of the fp32 and cross-check entry points take the four-wave form or, with few units, the form that spreads a
// unit's columns over the chip, both further down.
// Finch-C2 form (template flag): k = kbar (1 - w), no bonus, second value u' added to o.
#include "wkv6_launch.h"
#include "wkv6_math.h"

#include <type_traits>

#include <hip/hip_bf16.h>

namespace wkv6 {
namespace {

template <bool kInBf16>
__device__ __forceinline__ float load_in(const void* p, long long idx) {
    if constexpr (kInBf16) {
        unsigned short bits = static_cast<const unsigned short*>(p)[idx];
        return __uint_as_float(static_cast<unsigned>(bits) << 16);
    } else {
        return static_cast<const float*>(p)[idx];
    }
}

__device__ __forceinline__ float wave_sum(float a) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) a += __shfl_xor(a, m, 64);
    return a;
}

// kLora: the decay logit is formed here, lambda + y B, from the token's 64 low-rank activations and this channel's column of
// B (32 registers of bf16 pairs; products exact and sums in fp32, as on the matrix cores).  With a.moments
// (Finch-C2) the wave also leaves the head's LayerNorm partials of every token.
// kWaves: 1 or 4 (the rule is at the launch).  Wave q of four holds the key rows 16 q .. 16 q + 15 of the state and sums its sixteen
// terms of a read-out, and with kLora of a logit; they meet in LDS, one barrier each, and wave 0 writes the row.  Everything else of a token
// each wave does by itself.  So states have the same bits in both forms, except with kLora, where the logits' sums differ in their last
// bits; errors against 64 bits, one : four waves, 2-norm: fp32 read-outs 1.5e-7 : 9.6e-8, with kLora states 3.6e-8 : 3.4e-8 (1 token), 6.7e-8 :
// 6.6e-8 (4), head sums 2.0e-7 : 1.2e-7.
template <bool kInBf16, bool kOutBf16, bool kC2, bool kLora, int kWaves>
__global__ __launch_bounds__(64 * kWaves) void recurrent_kernel(Args a) {
    constexpr int N = kHeadSize, kRows = N / kWaves;
    const int unit = blockIdx.x;           // b * H + h
    const int b = unit / a.H;
    const int h = unit - b * a.H;
    const int j = threadIdx.x & 63;
    const int q = kWaves == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    __shared__ __attribute__((aligned(16))) float s_in[kWaves][3][N];      // r, k, w of the token, a copy for each wave
    __shared__ __attribute__((aligned(16))) float s_y[kLora ? kWaves : 1][kLora ? N : 4];
    // partial logits and read-outs by token parity: a wave writes a slot again two barriers after the last read of it
    __shared__ float s_logit[2][kWaves > 1 && kLora ? kWaves : 1][N], s_out[2][kWaves][N];
    float(&s_r)[N] = s_in[q][0];
    float(&s_k)[N] = s_in[q][1];
    float(&s_w)[N] = s_in[q][2];
    static_assert(!kLora || kLoraRank == kHeadSize, "a lane brings in one activation");
    auto order = [] {                      // this wave's LDS accesses before and behind it
        if constexpr (kWaves == 1) {
            __syncthreads();
        } else {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
    };

    [[maybe_unused]] unsigned bw[kLora ? kRows / 2 : 1];
    [[maybe_unused]] float lam = 0.f;
    if constexpr (kLora) {
        const long long width = static_cast<long long>(a.H) * N;
        const unsigned short* col = static_cast<const unsigned short*>(a.bw) + q * kRows * width + h * N + j;
#pragma unroll
        for (int i = 0; i < kRows / 2; ++i)
            bw[i] = static_cast<unsigned>(col[2 * i * width]) | (static_cast<unsigned>(col[(2 * i + 1) * width]) << 16);
        lam = a.lambda[h * N + j];
    }

    float S[kRows];
    if (a.state_in) {
        const float* s0 = a.state_in + static_cast<long long>(unit) * N * N + q * kRows * N;
#pragma unroll
        for (int i = 0; i < kRows; ++i) S[i] = __builtin_nontemporal_load(&s0[i * N + j]);   // streamed once
    } else {
#pragma unroll
        for (int i = 0; i < kRows; ++i) S[i] = 0.f;
    }

    const float uj = kC2 ? 0.f : a.u[h * N + j];
    const long long tok_stride = static_cast<long long>(a.H) * N;
    long long idx = static_cast<long long>(b) * a.batch_stride + static_cast<long long>(h) * N + j;

    // x (or, with kLora, the token's activation y_j) of a token
    auto load_x = [&](int t, long long e) {
        if constexpr (kLora) return load_in<true>(a.y, (static_cast<long long>(b) * a.T + t) * kLoraRank + j);
        else return load_in<kInBf16>(a.x, e);
    };
    float rj = 0.f, kj = 0.f, vj = 0.f, xj = 0.f, pj = 0.f;
    if (a.T > 0) {
        rj = load_in<kInBf16>(a.r, idx);
        kj = load_in<kInBf16>(a.k, idx);
        vj = load_in<kInBf16>(a.v, idx);
        xj = load_x(0, idx);
        if constexpr (kC2) pj = load_in<kInBf16>(a.uprime, idx);
    }
    for (int t = 0; t < a.T; ++t) {
        const float r_cur = rj, v_cur = vj, p_cur = pj, x_cur = xj, kraw = kj;
        const long long idx_cur = idx;
        idx += tok_stride;
        if (t + 1 < a.T) {                     // next token's loads overlap this token's math
            rj = load_in<kInBf16>(a.r, idx);
            kj = load_in<kInBf16>(a.k, idx);
            vj = load_in<kInBf16>(a.v, idx);
            xj = load_x(t + 1, idx);
            if constexpr (kC2) pj = load_in<kInBf16>(a.uprime, idx);
        }
        float logit = x_cur;
        if constexpr (kLora) {
            s_y[q][j] = x_cur;                 // (the last token's reads are behind its second barrier)
            order();
            logit = q == 0 ? lam : 0.f;
#pragma unroll
            for (int i = 0; i < kRows; i += 4) {
                const float4 y4 = *reinterpret_cast<const float4*>(&s_y[q][q * kRows + i]);
                logit = fmaf(y4.x, __uint_as_float(bw[i / 2] << 16), logit);
                logit = fmaf(y4.y, __uint_as_float(bw[i / 2] & 0xffff0000u), logit);
                logit = fmaf(y4.z, __uint_as_float(bw[i / 2 + 1] << 16), logit);
                logit = fmaf(y4.w, __uint_as_float(bw[i / 2 + 1] & 0xffff0000u), logit);
            }
            if constexpr (kWaves > 1) {
                s_logit[t & 1][q][j] = logit;
                __syncthreads();
                logit = (s_logit[t & 1][0][j] + s_logit[t & 1][1][j]) + (s_logit[t & 1][2][j] + s_logit[t & 1][3][j]);
            }
        }
        const float w_cur = expf(-expf(logit));
        // Finch-C2 key factor 1 - w = -expm1(-exp(x)): no cancellation for decays close to 1
        const float k_cur = kC2 ? kraw * -expm1f(-expf(logit)) : kraw;
        order();                               // previous token's LDS reads are done
        s_r[j] = r_cur;
        s_k[j] = k_cur;
        s_w[j] = w_cur;
        float o = 0.f;                         // Finch-C2: the second value; Finch: the bonus term
        if (q == 0) {
            o = p_cur;
            if constexpr (!kC2) o = wave_sum(r_cur * uj * k_cur) * v_cur;
        }
        order();

#pragma unroll
        for (int i4 = 0; i4 < kRows; i4 += 4) {
            const float4 r4 = *reinterpret_cast<const float4*>(&s_r[q * kRows + i4]);
            const float4 k4 = *reinterpret_cast<const float4*>(&s_k[q * kRows + i4]);
            const float4 w4 = *reinterpret_cast<const float4*>(&s_w[q * kRows + i4]);
            o = fmaf(r4.x, S[i4 + 0], o);
            S[i4 + 0] = fmaf(w4.x, S[i4 + 0], k4.x * v_cur);
            o = fmaf(r4.y, S[i4 + 1], o);
            S[i4 + 1] = fmaf(w4.y, S[i4 + 1], k4.y * v_cur);
            o = fmaf(r4.z, S[i4 + 2], o);
            S[i4 + 2] = fmaf(w4.z, S[i4 + 2], k4.z * v_cur);
            o = fmaf(r4.w, S[i4 + 3], o);
            S[i4 + 3] = fmaf(w4.w, S[i4 + 3], k4.w * v_cur);
        }
        if constexpr (kWaves > 1) {
            s_out[t & 1][q][j] = o;
            __syncthreads();
            if (q != 0) continue;
            o = (o + s_out[t & 1][1][j]) + (s_out[t & 1][2][j] + s_out[t & 1][3][j]);
        }
        if constexpr (kOutBf16)
            static_cast<unsigned short*>(a.out)[idx_cur] =
                __builtin_bit_cast(unsigned short, static_cast<__bf16>(o));
        else
            static_cast<float*>(a.out)[idx_cur] = o;
        if constexpr (kLora && kC2) {
            if (a.moments) {                   // uniform
                const float sum = wave_sum(o), dev = o - sum * (1.f / N);
                const float m2 = wave_sum(dev * dev);
                if (j == 0) *reinterpret_cast<float2*>(a.moments + (static_cast<long long>(unit) * a.T + t) * 2) = make_float2(sum, m2);
            }
        }
    }

    if (a.state_out) {
        float* so = a.state_out + static_cast<long long>(unit) * N * N + q * kRows * N;
#pragma unroll
        for (int i = 0; i < kRows; ++i) __builtin_nontemporal_store(S[i], &so[i * N + j]);
    }
}

// The same recurrence for long sequences, four wavefronts per (batch, head): wave w owns value
// columns 16w .. 16w+15, and its lane (q, c) = (lane / 16, lane % 16) owns key rows 16q .. 16q+15
// of column 16w + c (16 fp32 state registers).  Tokens are taken in blocks of 8.  The workgroup's
// 256 threads fetch a block together, two neighbouring channels of one token each (r, k, x, v),
// form w once per element and leave the fp32 vectors in LDS one block
// ahead of their use, two slots by block parity, one workgroup barrier per block; the loads of
// the block after that are in flight meanwhile, which is what hides the memory latency a
// token-by-token prefetch cannot.  A lane then reads its quarter of r, k, w as broadcasts, runs
// its 16 rows, and the four quarters of a column meet through two cross-lane moves per token,
// issued together at the end of the block.  The Finch bonus enters inside the row loop
// (o += r_i (S_ij + u_i k_i v_j)), so no sum over the whole wave is needed.  Finch form only: the
// Finch-C2 entry points that take this file's kernels are single steps and short appends.
constexpr int kWideBlock = 8;

template <bool kInBf16>
struct WidePair {                          // two neighbouring channels of one token
    float lo, hi;
    __device__ __forceinline__ void load(const void* p, long long elem) {
        if constexpr (kInBf16) {
            const unsigned w = *reinterpret_cast<const unsigned*>(static_cast<const unsigned short*>(p) + elem);
            lo = __uint_as_float(w << 16);
            hi = __uint_as_float(w & 0xffff0000u);
        } else {
            const float2 f = *reinterpret_cast<const float2*>(static_cast<const float*>(p) + elem);
            lo = f.x;
            hi = f.y;
        }
    }
};

template <bool kInBf16, bool kOutBf16>
__global__ __launch_bounds__(256) void recurrent_wide_kernel(Args a) {
    constexpr int N = kHeadSize;
    using Pair = WidePair<kInBf16>;
    const int unit = blockIdx.x;           // b * H + h
    const int b = unit / a.H;
    const int h = unit - b * a.H;
    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int q = lane >> 4, c = lane & 15;
    const int j = 16 * wave + c;

    // [block parity][r, k, w, v][token][channel]
    __shared__ __attribute__((aligned(16))) float s_in[2][4][kWideBlock][N];

    float S[16], uq[16];
    if (a.state_in) {
        const float* s0 = a.state_in + static_cast<long long>(unit) * N * N + (16 * q) * N + j;
#pragma unroll
        for (int i = 0; i < 16; ++i) S[i] = __builtin_nontemporal_load(&s0[i * N]);
    } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) S[i] = 0.f;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) uq[i] = a.u[h * N + 16 * q + i];

    const long long tok_stride = static_cast<long long>(a.H) * N;
    const long long base = static_cast<long long>(b) * a.batch_stride + static_cast<long long>(h) * N;
    const int st = tid >> 5;               // token of this thread inside a block when staging
    const int sc = 2 * (tid & 31);         // its two channels

    Pair raw_r, raw_k, raw_x, raw_v;
    auto fetch = [&](int t0) {             // rows past the end are not touched
        raw_r.lo = raw_r.hi = raw_k.lo = raw_k.hi = raw_x.lo = raw_x.hi = 0.f;
        raw_v.lo = raw_v.hi = 0.f;
        if (t0 + st < a.T) {
            const long long e = base + static_cast<long long>(t0 + st) * tok_stride + sc;
            raw_r.load(a.r, e);
            raw_k.load(a.k, e);
            raw_x.load(a.x, e);
            raw_v.load(a.v, e);
        }
    };
    auto stage = [&](int parity) {
        const float e0 = expf(raw_x.lo), e1 = expf(raw_x.hi);
        *reinterpret_cast<float2*>(&s_in[parity][0][st][sc]) = make_float2(raw_r.lo, raw_r.hi);
        *reinterpret_cast<float2*>(&s_in[parity][1][st][sc]) = make_float2(raw_k.lo, raw_k.hi);
        *reinterpret_cast<float2*>(&s_in[parity][2][st][sc]) = make_float2(expf(-e0), expf(-e1));
        *reinterpret_cast<float2*>(&s_in[parity][3][st][sc]) = make_float2(raw_v.lo, raw_v.hi);
    };
    // one token of this lane's 16 rows
    auto token = [&](int parity, int tt) {
        const float* rkw = &s_in[parity][0][tt][16 * q];
        const float v_cur = s_in[parity][3][tt][j];
        float o = 0.f;
#pragma unroll
        for (int i4 = 0; i4 < 16; i4 += 4) {
            const float4 r4 = *reinterpret_cast<const float4*>(rkw + i4);
            const float4 k4 = *reinterpret_cast<const float4*>(rkw + kWideBlock * N + i4);
            const float4 w4 = *reinterpret_cast<const float4*>(rkw + 2 * kWideBlock * N + i4);
            const float rr[4] = {r4.x, r4.y, r4.z, r4.w};
            const float kk[4] = {k4.x, k4.y, k4.z, k4.w};
            const float ww[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float kv = kk[e] * v_cur;
                o = fmaf(rr[e], fmaf(uq[i4 + e], kv, S[i4 + e]), o);
                S[i4 + e] = fmaf(ww[e], S[i4 + e], kv);
            }
        }
        return o;
    };

    if (a.T > 0) {
        fetch(0);
        stage(0);
        fetch(kWideBlock);
    }
    int parity = 0;
    for (int t0 = 0; t0 < a.T; t0 += kWideBlock, parity ^= 1) {
        __syncthreads();                       // this block is staged; the other slot has been read
        if (t0 + kWideBlock < a.T) {           // the next block into the other slot, the one after on its way
            stage(parity ^ 1);
            fetch(t0 + 2 * kWideBlock);
        }
        const int nb = a.T - t0 < kWideBlock ? a.T - t0 : kWideBlock;
        float part[kWideBlock];
        if (nb == kWideBlock) {                // straight line: the reads of one token overlap the rows of another
#pragma unroll
            for (int tt = 0; tt < kWideBlock; ++tt) part[tt] = token(parity, tt);
        } else {
#pragma unroll
            for (int tt = 0; tt < kWideBlock; ++tt) {
                part[tt] = 0.f;
                if (tt < nb) part[tt] = token(parity, tt);
            }
        }
        // the four key quarters of every column meet; quarter q then stores tokens 2q and 2q+1
#pragma unroll
        for (int tt = 0; tt < kWideBlock; ++tt) part[tt] += __shfl_xor(part[tt], 16, 64);
#pragma unroll
        for (int tt = 0; tt < kWideBlock; ++tt) part[tt] += __shfl_xor(part[tt], 32, 64);
#pragma unroll
        for (int tt = 0; tt < kWideBlock; ++tt) {
            if ((tt >> 1) == q && tt < nb) {
                const float o = part[tt];
                const long long e = base + static_cast<long long>(t0 + tt) * tok_stride + j;
                if constexpr (kOutBf16)
                    static_cast<unsigned short*>(a.out)[e] = __builtin_bit_cast(unsigned short, static_cast<__bf16>(o));
                else
                    static_cast<float*>(a.out)[e] = o;
            }
        }
    }

    if (a.state_out) {
        float* so = a.state_out + static_cast<long long>(unit) * N * N + (16 * q) * N + j;
#pragma unroll
        for (int i = 0; i < 16; ++i) __builtin_nontemporal_store(S[i], &so[i * N]);
    }
}

// The same for few (batch, head) units: the columns of a state do not depend on one another, so a unit's 64 are
// dealt to 64 / kCols waves, four to a workgroup, and every SIMD of the chip gets work.  Lane i owns key row i of the
// wave's kCols columns: r, k, w and u k of its row are one 16-byte LDS read per token, the wave's v values one
// broadcast, and a token costs 4 kCols multiply-adds with no exchange between lanes.  The sums over the
// rows wait until 64 of them are due (64 / kCols tokens): a reduce-scatter over the 64 lanes then leaves each lane one finished
// value, in 141 instructions where folding each by itself would take 12 x 64.  Tokens are staged as in the
// kernel above, one block of 64 / kCols tokens ahead with the loads of the next in flight, each unit's w formed once per workgroup.
// Bound by the instruction issue of one or two waves per SIMD (two columns: 196 clocks a token at 32 units of 512 tokens).
template <int kCtrl>
__device__ __forceinline__ float dpp_lanes(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), kCtrl, 0xf, 0xf, false));
}
// One step inside rows of 16 lanes: kCount pairs (v[i], v[i + kCount]); lanes with `high` unset keep the first of
// a pair and give the second to their partner, the others the reverse.
template <int kCount, int kCtrl>
__device__ __forceinline__ void fold_pairs(float (&v)[64], bool high) {
#pragma unroll
    for (int i = 0; i < kCount; ++i) {
        const float keep = high ? v[i + kCount] : v[i], give = high ? v[i] : v[i + kCount];
        v[i] = keep + dpp_lanes<kCtrl>(give);
    }
}
// v[0 .. 63] of 64 lanes -> in v[0] of lane l, the sum over all lanes of v[l] (every step keeps, of a pair 2^n apart, the one
// that bit n of the lane's number selects)
__device__ __forceinline__ float reduce_scatter(float (&v)[64], int lane) {
#pragma unroll
    for (int i = 0; i < 32; ++i) {                 // halves: lanes 0..31 take v[i], 32..63 v[i + 32]
        const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i]), __float_as_uint(v[i + 32]), false, false);
        v[i] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {                 // rows of 16: even rows take v[i], odd ones v[i + 16]
        const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[i]), __float_as_uint(v[i + 16]), false, false);
        v[i] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
    }
    fold_pairs<8, 0x128>(v, lane & 8);             // row_ror:8: lane ^ 8
    fold_pairs<4, 0x141>(v, lane & 4);             // row_half_mirror: 7 - lane of each 8
    fold_pairs<2, 0x1B>(v, lane & 2);              // quad_perm [3,2,1,0]
    fold_pairs<1, 0xB1>(v, lane & 1);              // quad_perm [1,0,3,2]
    return v[0];
}

// 4 to 32 bytes of a row: what a thread loads at once
template <int kBytes>
struct Piece;
template <>
struct Piece<4> {
    typedef unsigned type __attribute__((ext_vector_type(1)));
    static __device__ __forceinline__ type load(__amdgpu_buffer_rsrc_t r, int voff) { return type{__builtin_amdgcn_raw_buffer_load_b32(r, voff, 0, 0)}; }
};
template <>
struct Piece<8> {
    typedef unsigned type __attribute__((ext_vector_type(2)));
    static __device__ __forceinline__ type load(__amdgpu_buffer_rsrc_t r, int voff) { return __builtin_bit_cast(type, __builtin_amdgcn_raw_buffer_load_b64(r, voff, 0, 0)); }
};
template <>
struct Piece<16> {
    typedef unsigned type __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ type load(__amdgpu_buffer_rsrc_t r, int voff) { return __builtin_bit_cast(type, __builtin_amdgcn_raw_buffer_load_b128(r, voff, 0, 0)); }
};
template <>
struct Piece<32> {
    typedef unsigned type __attribute__((ext_vector_type(8)));
    static __device__ __forceinline__ type load(__amdgpu_buffer_rsrc_t r, int voff) {
        const auto lo = Piece<16>::load(r, voff), hi = Piece<16>::load(r, voff + 16);
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    }
};
template <bool kInBf16, typename T>
__device__ __forceinline__ float piece_value(const T& q, int i) {
    if constexpr (!kInBf16) return __uint_as_float(q[i]);
    else return __uint_as_float(i & 1 ? q[i >> 1] & 0xffff0000u : q[i >> 1] << 16);
}

template <int kCols, bool kInBf16>
__global__ __launch_bounds__(256) void recurrent_columns_kernel(Args a) {
    constexpr int N = kHeadSize;
    constexpr int kTokens = 64 / kCols;            // tokens of a block
    constexpr int kPer = kTokens / 4;              // channels a thread stages
    constexpr int kGroups = N / (4 * kCols);       // workgroups of a unit
    const int unit = blockIdx.x / kGroups;         // b * H + h
    const int b = unit / a.H, h = unit - b * a.H;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int j0 = (blockIdx.x - unit * kGroups) * (4 * kCols);      // the workgroup's first column
    const int jw = j0 + kCols * wave;                                // the wave's

    __shared__ __attribute__((aligned(16))) float4 s_rows[2][kTokens][N];        // r, k, w, u k of a key row
    __shared__ __attribute__((aligned(16))) float s_v[2][kTokens][4 * kCols];

    float S[kCols];
#pragma unroll
    for (int c = 0; c < kCols; ++c) S[c] = 0.f;
    if (a.state_in) {
        const float* s0 = a.state_in + static_cast<long long>(unit) * N * N + lane * N + jw;
#pragma unroll
        for (int c = 0; c < kCols; ++c) S[c] = s0[c];
    }
    const long long tok_stride = static_cast<long long>(a.H) * N;
    const long long base = static_cast<long long>(b) * a.batch_stride + static_cast<long long>(h) * N;
    const int st = tid / (N / kPer), sc = kPer * (tid % (N / kPer));             // staged token and first channel
    const int vt = tid / (4 * kCols), vc = tid % (4 * kCols);                    // 256 = kTokens * 4 kCols values of v
    float u[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) u[i] = a.u[h * N + sc + i];

    // Loads through raw buffer descriptors that end with the sequence: rows past the end read as zero with no
    // branch (r = k = v = 0; w is set to 1 when staged), so a block is one straight line.
    constexpr int kElem = kInBf16 ? 2 : 4;
    const long long row_bytes = tok_stride * kElem, span = static_cast<long long>(a.T - 1) * row_bytes + N * kElem;
    const int voff = static_cast<int>(st * row_bytes) + sc * kElem, v_voff = static_cast<int>(vt * row_bytes) + (j0 + vc) * kElem;
    typedef typename Piece<kPer * kElem>::type Raw;
    Raw raw_r, raw_k, raw_x;
    float raw_v = 0.f;
    auto fetch = [&](int t0) {
        const long long off = t0 * row_bytes;
        raw_r = Piece<kPer * kElem>::load(chunk_rsrc(static_cast<const char*>(a.r) + base * kElem, off, span), voff);
        raw_k = Piece<kPer * kElem>::load(chunk_rsrc(static_cast<const char*>(a.k) + base * kElem, off, span), voff);
        raw_x = Piece<kPer * kElem>::load(chunk_rsrc(static_cast<const char*>(a.x) + base * kElem, off, span), voff);
        const __amdgpu_buffer_rsrc_t rv = chunk_rsrc(static_cast<const char*>(a.v) + base * kElem, off, span);
        if constexpr (kInBf16)
            raw_v = __uint_as_float(static_cast<unsigned>(__builtin_amdgcn_raw_buffer_load_b16(rv, v_voff, 0, 0)) << 16);
        else
            raw_v = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rv, v_voff, 0, 0));
    };
    auto stage = [&](int t0, int parity) {
        const bool past = t0 + st >= a.T;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const float rr = piece_value<kInBf16>(raw_r, i), kk = piece_value<kInBf16>(raw_k, i), xx = piece_value<kInBf16>(raw_x, i);
            const float w = expf(-expf(xx));
            s_rows[parity][st][sc + i] = make_float4(rr, kk, past ? 1.f : w, u[i] * kk);
        }
        s_v[parity][vt][vc] = raw_v;
    };

    if (a.T > 0) {
        fetch(0);
        stage(0, 0);
        fetch(kTokens);
    }
    const int ot = lane / kCols, oc = lane % kCols;              // token and column of the value this lane ends up with
    int parity = 0;
    for (int t0 = 0; t0 < a.T; t0 += kTokens, parity ^= 1) {
        __syncthreads();                           // this block is staged; the other slot has been read
        stage(t0 + kTokens, parity ^ 1);
        fetch(t0 + 2 * kTokens);
        float part[64];
#pragma unroll
        for (int t = 0; t < kTokens; ++t) {
            const float4 q = s_rows[parity][t][lane];
            const float* v = &s_v[parity][t][kCols * wave];
#pragma unroll
            for (int c = 0; c < kCols; ++c) {
                part[t * kCols + c] = q.x * fmaf(q.w, v[c], S[c]);
                S[c] = fmaf(q.z, S[c], q.y * v[c]);
            }
        }
        const float o = reduce_scatter(part, lane);
        if (t0 + ot < a.T) static_cast<float*>(a.out)[base + static_cast<long long>(t0 + ot) * tok_stride + jw + oc] = o;
    }

    if (a.state_out) {
        float* so = a.state_out + static_cast<long long>(unit) * N * N + lane * N + jw;
#pragma unroll
        for (int c = 0; c < kCols; ++c) so[c] = S[c];
    }
}

__global__ __launch_bounds__(256) void state_passthrough_kernel(const float* in, float* out,
                                                                long long n4) {
    const long long i = static_cast<long long>(blockIdx.x) * 256 + threadIdx.x;
    if (i < n4) {
        float4 val = make_float4(0.f, 0.f, 0.f, 0.f);
        if (in) val = reinterpret_cast<const float4*>(in)[i];
        reinterpret_cast<float4*>(out)[i] = val;
    }
}

}  // namespace

// Sequences of at least this many tokens take the four-wave form; shorter ones (decode, short
// appends: the work is streaming the state once) the one-wave form with its 256-byte state rows.
constexpr int kWideMinTokens = 16;

hipError_t launch_recurrent(const Args& a, bool in_bf16, bool out_bf16, hipStream_t stream) {
    const dim3 grid(static_cast<unsigned>(a.B) * static_cast<unsigned>(a.H));
    const bool c2 = a.finch_c2;
    // Four waves a unit or one.  Four hold a quarter of the state and of a token's work each, so that few units keep more of
    // the chip busy; one needs no exchange.  One -> four, us, the same tensors again and again:
    // decode: 1024 units 5.7 -> 5.4.  With 1025 to 2500 units eight workgroups of four waves do not fit a compute unit beside
    // one another: 1536 7.0 -> 8.4, 2048 8.9 -> 11.4.  From there on a step streams the states at the memory's rate, and the
    // shorter waves keep it busier: with states that no cache holds 2560 15.9 -> 15.6, 3200 19.7 -> 19.1, 8192 46.7 -> 44.2,
    // 32 768 177 -> 170 (2560 units whose 42 MB stay in the memory-side cache lose, 13.5 -> 13.8).
    // Appends: 256 units x 6 tokens 8.6 -> 7.2, 1024 x 6 11.5 -> 9.7, 1056 x 4 9.4 -> 8.9, 1280 x 3 9.0 -> 8.6, 1536 x 2 9.1 -> 8.1,
    // x 6 13.4 -> 11.9; fp32 32 units x 12 tokens 14.6 -> 10.2, 1536 x 15 26.1 -> 24.2.  With more units than six a compute
    // unit the waves wait for one another at every token in a second round: 1600 x 2 9.3 -> 11.1, x 6 13.8 -> 16.7; 2560 x 3
    // 13.8 -> 16.1; fp32 1568 x 12 21.9 -> 26.2.
    // Fused logits, Finch-C2 (with one wave its registers leave four units a compute unit): 1024 units x 1 token 7.8 -> 6.6,
    // 1056 x 2 14.2 -> 10.7, 2048 x 1 14.7 -> 13.4, x 2 18.5 -> 14.0.  Finch (eight units of one wave, five of four): 1024 x 1
    // 7.2 -> 6.2, x 4 11.4 -> 9.2, 1280 x 2 9.5 -> 8.1, x 4 12.3 -> 10.6; but 1056 x 1 7.3 -> 7.6, 1408 x 2 10.2 -> 11.4, 1536 x 4
    // 13.4 -> 15.8, 2048 x 1 10.4 -> 13.2, x 4 15.6 -> 17.8.
    const long long units = grid.x;
    auto shared_work = [&] {
        const long long cus = compute_units();
        if (units <= 4 * cus) return true;
        if (a.y) return units <= (c2 ? 8 : a.T > 1 ? 5 : 4) * cus;
        return a.T > 1 ? units <= 6 * cus : units >= 10 * cus;
    };
    const bool four = units <= 64 || (fits_a_launch(units, 256) && shared_work());
    auto step = [&](auto one_wave, auto four_waves) {
        hipLaunchKernelGGL(four ? four_waves : one_wave, grid, dim3(four ? 256 : 64), 0, stream, a);
    };
    if (a.y) {                                 // fused decay path: bf16 in and out
        if (c2)
            step(&recurrent_kernel<true, true, true, true, 1>, &recurrent_kernel<true, true, true, true, 4>);
        else
            step(&recurrent_kernel<true, true, false, true, 1>, &recurrent_kernel<true, true, false, true, 4>);
        return hipGetLastError();
    }
    if (a.T >= kWideMinTokens && !c2 && !out_bf16) {
        // A unit's columns over as many workgroups as the chip has room for: one round of 256 with two columns a wave,
        // two with four or eight.  Measured, fp32, microseconds, four waves a unit -> here (2, 4, 8 columns): 4 units x 256 tokens 77
        // -> 22, 31, 45; 32 x 512 154 -> 44, 60, 90; 96 x 300 100 -> 75, 46, 56; 256 x 300 101 -> 151, 82, 74; 512 x 1024 382
        // -> 855, 492, 426: from there the four-wave form, whose waves hold all rows of a column, issues fewer instructions.
        // Short sequences, four waves -> here: 32 units x 16 tokens 6.7 -> 5.6, 128 x 17 8.5 -> 7.5; eight columns (blocks of 8
        // tokens) 256 units x 16 7.8 -> 7.2, x 17 9.0 -> 9.4, x 18 9.2 -> 9.4, x 20 9.7 -> 9.5 to 10.0, x 22 10.1 -> 9.7, x 33 13.9 -> 13.7,
        // 192 x 17 8.8 -> 9.0, x 18 9.0 -> 9.0: a third block for a few tokens is what loses.
        auto columns = [&](auto bf16) {
            constexpr bool kIn = decltype(bf16)::value;
            if (units <= 32)
                hipLaunchKernelGGL((recurrent_columns_kernel<2, kIn>), dim3(grid.x * 8), dim3(256), 0, stream, a);
            else if (units <= 128)
                hipLaunchKernelGGL((recurrent_columns_kernel<4, kIn>), dim3(grid.x * 4), dim3(256), 0, stream, a);
            else
                hipLaunchKernelGGL((recurrent_columns_kernel<8, kIn>), dim3(grid.x * 2), dim3(256), 0, stream, a);
            return hipGetLastError();
        };
        const bool third_block = a.T > kWideMinTokens && a.T <= kWideMinTokens + 4;
        if (units <= 128 || (units <= 256 && !third_block)) return in_bf16 ? columns(std::true_type{}) : columns(std::false_type{});
    }
    if (a.T >= kWideMinTokens && !c2) {
        if (!in_bf16)
            hipLaunchKernelGGL((recurrent_wide_kernel<false, false>), grid, dim3(256), 0, stream, a);
        else if (!out_bf16)
            hipLaunchKernelGGL((recurrent_wide_kernel<true, false>), grid, dim3(256), 0, stream, a);
        else
            hipLaunchKernelGGL((recurrent_wide_kernel<true, true>), grid, dim3(256), 0, stream, a);
        return hipGetLastError();
    }
    if (!in_bf16)
        step(&recurrent_kernel<false, false, false, false, 1>, &recurrent_kernel<false, false, false, false, 4>);
    else if (!out_bf16 && !c2)
        step(&recurrent_kernel<true, false, false, false, 1>, &recurrent_kernel<true, false, false, false, 4>);
    else if (!out_bf16 && c2)
        step(&recurrent_kernel<true, false, true, false, 1>, &recurrent_kernel<true, false, true, false, 4>);
    else if (!c2)
        step(&recurrent_kernel<true, true, false, false, 1>, &recurrent_kernel<true, true, false, false, 4>);
    else
        step(&recurrent_kernel<true, true, true, false, 1>, &recurrent_kernel<true, true, true, false, 4>);
    return hipGetLastError();
}

hipError_t launch_state_passthrough(const Args& a, hipStream_t stream) {
    if (!a.state_out || a.state_out == a.state_in) return hipSuccess;
    const long long n4 = static_cast<long long>(a.B) * a.H * kHeadSize * kHeadSize / 4;
    const unsigned blocks = static_cast<unsigned>((n4 + 255) / 256);
    hipLaunchKernelGGL(state_passthrough_kernel, dim3(blocks), dim3(256), 0, stream,
                       a.state_in, a.state_out, n4);
    return hipGetLastError();
}

}  // namespace wkv6

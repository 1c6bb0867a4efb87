// Token statistics of the LayerNorm over all heads (Finch-C2 Time Mixing, output equation) from
// the per-head partial moments the prefill kernel emits next to its output.
//
// Each (batch, head, token) contributes the sum s of its N values and the squared deviations m2 from its own mean.  With the mean
// mu of the token known from the sums, the heads' deviations d_h = s_h / N - mu about it add up without cancellation: M2 = sum of m2_h +
// N d_h^2 (Chan, Golub, LeVeque).  What mu lacks for rounding is the mean of the d_h, which then corrects both (the corrected two-pass
// form): heads of equal sums s have the mean s / N and no deviation, whatever their number, and a common offset of 1e5 standard
// deviations leaves rstd its 5e-8 (without the correction 1e-5, pair after pair 3e-4).
//
// A workgroup takes 64 consecutive tokens of one batch; each of its four waves has every fourth head (a lane per token, so every read
// is a contiguous run of 8-byte pairs); sums and then deviations meet in LDS.  Bound by latency: up to 256 heads stay in
// registers, all requested at once, and nothing but the result is divided.  Folding the pairs one after the other, with two divisions each,
// took longer (figures at the launch); the calls of a layer 156.4 us where they take 153.9 (8 x 2048 tokens x 32 heads), 27.8 and 26.9 (24 x 1).
#include "wkv6_launch.h"

namespace wkv6 {
namespace {

constexpr float kInvN = 1.f / kHeadSize;

// deviations of the heads about the token's mean as it was first rounded
struct Deviations {
    float m2 = 0.f, left = 0.f;
    __device__ __forceinline__ void add(const float2 p, float mean) {
        const float d = fmaf(p.x, kInvN, -mean);
        m2 += fmaf(d * kHeadSize, d, p.y);
        left += d;
    }
    __device__ __forceinline__ float2 mean_rstd(float mean, float heads, float per_head, float eps) const {
        const float by = left * per_head;
        float m = fmaf(by * -kHeadSize, left, m2);
        if (m < 0.f) m = 0.f;              // (NaN stays)
        return make_float2(mean + by, 1.f / sqrtf(m / (heads * kHeadSize) + eps));
    }
};

// kKept: heads of a wave in registers, all requested before the first is used.  As few as hold all heads (the rule is at the launch),
// since a place without a head costs its instructions all the same: 8 x 2048 tokens x 8 heads 2.00 us with 4, 2.49 with 16; x 32 heads 2.14
// with 8, 2.49 with 16; x 130 heads 3.6 with 40, 4.9 with 64.  (Branches around absent heads took longer where all are there: x 64
// 2.72 against 2.51.)  kRest: there are more heads, which are read twice.
template <int kKept, bool kRest>
__global__ __launch_bounds__(256) void layernorm_finalize_kernel(int T, int H, const float2* moments, float eps,
                                                                 float2* mean_rstd) {
    __shared__ float part[4][64];
    __shared__ float2 devs[4][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t0 = blockIdx.x * 64, t = t0 + lane;
    const int b = blockIdx.y;
    // A head's pairs of the 64 tokens, from a descriptor of their own, which is empty for a head that is not there: zeros, without a branch.
    float2* src = const_cast<float2*>(moments) + static_cast<long long>(b) * H * T + t0;
    const int bytes = (T - t0 < 64 ? T - t0 : 64) * 8;
    auto pair_of = [&](int h) {
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc(src + (h < H ? static_cast<long long>(h) * T : 0), 0, h < H ? bytes : 0, 0x00020000);
        return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rs, lane * 8, 0, 0));
    };
    float2 kept[kKept];
    float sums[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < kKept; ++i) kept[i] = pair_of(wave + 4 * i);
#pragma unroll
    for (int i = 0; i < kKept; ++i) sums[i % 4] = fmaf(kept[i].x, kInvN, sums[i % 4]);
    constexpr int kAtOnce = 8;             // of the heads that are not kept
    if constexpr (kRest) {
        for (int h = wave + 4 * kKept; h < H; h += 4 * kAtOnce) {
            float2 p[kAtOnce];
#pragma unroll
            for (int i = 0; i < kAtOnce; ++i) p[i] = pair_of(h + 4 * i);
#pragma unroll
            for (int i = 0; i < kAtOnce; ++i) sums[i % 4] = fmaf(p[i].x, kInvN, sums[i % 4]);
        }
    }
    part[wave][lane] = (sums[0] + sums[1]) + (sums[2] + sums[3]);
    const float heads = static_cast<float>(H), per_head = __builtin_amdgcn_rcpf(heads);
    __syncthreads();
    const float mean = ((part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane])) * per_head;
    Deviations dev;
#pragma unroll
    for (int i = 0; i < kKept; ++i) dev.add(kept[i], wave + 4 * i < H ? mean : 0.f);
    if constexpr (kRest) {
        for (int h = wave + 4 * kKept; h < H; h += 4 * kAtOnce) {
            float2 p[kAtOnce];
#pragma unroll
            for (int i = 0; i < kAtOnce; ++i) p[i] = pair_of(h + 4 * i);
#pragma unroll
            for (int i = 0; i < kAtOnce; ++i) dev.add(p[i], h + 4 * i < H ? mean : 0.f);
        }
    }
    devs[wave][lane] = make_float2(dev.m2, dev.left);
    __syncthreads();
    if (wave == 0 && t < T) {
        dev.m2 = (devs[0][lane].x + devs[1][lane].x) + (devs[2][lane].x + devs[3][lane].x);
        dev.left = (devs[0][lane].y + devs[1][lane].y) + (devs[2][lane].y + devs[3][lane].y);
        mean_rstd[static_cast<long long>(b) * T + t] = dev.mean_rstd(mean, heads, per_head, eps);
    }
}

// The two halves of a wave added: the sum of a's in the lower half of the lanes, of b's in the upper one.
__device__ __forceinline__ float add_halves(float a, float b) {
    const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}

template <int kBy>
__device__ __forceinline__ float rotated(float v) {        // within a row of sixteen lanes
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x120 + kBy, 0xf, 0xf, false));
}

// Sum over the 32 lanes of a half, in every lane of it, in pairs of lanes 16, 8, 4, 2 and 1 apart (a rotation by as much as the period
// to which the sums are equal already).  No step passes LDS; through shuffles 65 535 x 1 token x 12 heads took 13.1 us where this takes 11.0.
__device__ __forceinline__ float half_sum(float v) {
    const auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(q[0]) + __uint_as_float(q[1]);
    v += rotated<8>(v);
    v += rotated<4>(v);
    v += rotated<2>(v);
    return v + rotated<1>(v);
}

// Sequences of a few tokens: a wave per token with the heads on its lanes, since a lane per token would leave
// most lanes without one.  Partial results meet in pairs over the lanes.
__global__ __launch_bounds__(256) void layernorm_finalize_few_kernel(long long tokens, int T, int H, const float2* moments,
                                                                     float eps, float2* mean_rstd) {
    const int lane = threadIdx.x & 63;
    const long long token = static_cast<long long>(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (token >= tokens) return;
    // (fewer than 2^32 tokens: at most 65 535 sequences, of fewer than 16)
    const unsigned b = static_cast<unsigned>(token) / static_cast<unsigned>(T);
    const float2* src = moments + static_cast<long long>(b) * H * T + (token - static_cast<long long>(b) * T);
    const float2 mine = lane < H ? src[static_cast<long long>(lane) * T] : make_float2(0.f, 0.f);
    float sum = mine.x * kInvN;
    for (int h = lane + 64; h < H; h += 64) sum = fmaf(src[static_cast<long long>(h) * T].x, kInvN, sum);
    sum = half_sum(add_halves(sum, sum));
    const float heads = static_cast<float>(H), per_head = __builtin_amdgcn_rcpf(heads), mean = sum * per_head;
    Deviations dev;
    if (lane < H) dev.add(mine, mean);
    for (int h = lane + 64; h < H; h += 64) dev.add(src[static_cast<long long>(h) * T], mean);
    const float both = half_sum(add_halves(dev.m2, dev.left));
    dev.m2 = both;
    dev.left = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(both), 32));
    if (lane == 0) mean_rstd[token] = dev.mean_rstd(mean, heads, per_head, eps);
}

// The normalisation itself, for callers whose projection GEMM has no row-scaling epilogue:
// y = (o - mean) * rstd * gamma + beta over the D = H*N values of each token; 8 channels (16 bytes
// of bf16) per item, every tensor touched once, fp32 arithmetic, one rounding of the result.  A thread
// keeps four items in flight (four loads, then four stores; a thread reads an item before it writes
// it, so y may be o).  Two forms: when a token's D/8 items are a multiple of 256 a workgroup owns a
// strip of 256 item columns over a run of tokens, so a thread's gain and offset stay in registers
// and the token's (mean, rstd) is a scalar load; otherwise items are dealt out in runs of 1024 and
// the gain and offset are fetched per item (they stay in L1).
typedef unsigned uint4v __attribute__((ext_vector_type(4)));
constexpr int kInFlight = 4;

// Cache policy of the stores.  Written through the L2 (sc1), as those of the prefill, but not non-temporal, bf16 rows are in the
// memory-side cache when the product that reads them next does, as long as that holds them beside what else the layer touches.
// Five calls of a layer in a row, streamed -> through, microseconds, repeated on one set of tensors / on sets that no cache holds:
// D = 2048 4 x 500 tokens (8 MiB of rows) 54.5 -> 53.4 / 56.0 -> 56.1, 8 x 2048 (64 MiB) 164 -> 158 / 165 -> 161, 9 x 2048 (72) 246 -> 242 /
// 247 -> 244, 10 x 2048 (80) 249 -> 248 / 251 -> 253, 12 x 2048 (96) 262 -> 255 / 258 -> 265; D = 4096 4 x 1024 (32) 126 -> 123 / 125 -> 124,
// 8 x 1024 (64) 186 -> 182 / 190 -> 190, 9 x 1024 (72) 233 -> 234 / 240 -> 243.  The kernel for other widths, whose workgroups write runs
// across rows: D = 1024 8 x 2048 (32) 118 -> 114 / 117 -> 117, 12 x 2048 (48) 135 -> 134 / 135 -> 136, 16 x 2048 (64) 154 -> 156 / 157 -> 158;
// few rows leave it later: D = 768 500 tokens (0.7 MiB) 40.7 -> 41.2 (alone 4.0 -> 4.3), 1000 (1.5) 42.0 -> 42.2, 1500 (2.2) 43.6 -> 43.1.
// fp32 rows, which leave half a line at a time, stay non-temporal (92 -> 206 written through).
constexpr int kStoreThrough = 16, kStoreStreamed = 2;

// item `item` of the `items` from `first` on
template <bool kOutF32, int kStore>
__device__ __forceinline__ void normalise_item(const uint4v raw, const float2 ms, const float4 g0, const float4 g1,
                                               const float4 b0, const float4 b1, void* y, long long first, long long items, int item) {
    const float gm[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
    const float bt[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
    float v[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[2 * i] = __uint_as_float(raw[i] << 16);
        v[2 * i + 1] = __uint_as_float(raw[i] & 0xffff0000u);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = fmaf((v[i] - ms.x) * ms.y, gm[i], bt[i]);
    if constexpr (kOutF32) {
        typedef float float4v __attribute__((ext_vector_type(4)));
        float4v* dst = static_cast<float4v*>(y) + 2 * (first + item);
        __builtin_nontemporal_store(float4v{v[0], v[1], v[2], v[3]}, dst);
        __builtin_nontemporal_store(float4v{v[4], v[5], v[6], v[7]}, dst + 1);
    } else {
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        typedef float float2v __attribute__((ext_vector_type(2)));
        uint4v q;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            q[i] = __builtin_bit_cast(unsigned, __builtin_convertvector(float2v{v[2 * i], v[2 * i + 1]}, bf16x2));
        const __amdgpu_buffer_rsrc_t rows =
            __builtin_amdgcn_make_buffer_rsrc(static_cast<uint4v*>(y) + first, 0, static_cast<int>(items * 16), 0x00020000);
        __builtin_amdgcn_raw_buffer_store_b128(q, rows, 16 * item, 0, kStore);
    }
}

// grid (token runs, strips of 256 item columns); items_per_token is a multiple of 256
template <bool kOutF32, int kStore>
__global__ __launch_bounds__(256) void layernorm_apply_strip_kernel(long long tokens, int tokens_per_block,
                                                                    int items_per_token, const uint4v* o,
                                                                    const float2* mean_rstd, const float4* gamma,
                                                                    const float4* beta, void* y) {
    const int column = blockIdx.y * 256 + threadIdx.x;
    const float4 g0 = gamma[2 * column], g1 = gamma[2 * column + 1], b0 = beta[2 * column], b1 = beta[2 * column + 1];
    const long long t0 = static_cast<long long>(blockIdx.x) * tokens_per_block;
    const long long t1 = t0 + tokens_per_block < tokens ? t0 + tokens_per_block : tokens;
    for (long long t = t0; t < t1; t += kInFlight) {
        uint4v raw[kInFlight];
        float2 ms[kInFlight];
#pragma unroll
        for (int j = 0; j < kInFlight; ++j)
            if (t + j < t1) {
                raw[j] = __builtin_nontemporal_load(o + (t + j) * items_per_token + column);
                ms[j] = mean_rstd[t + j];
            }
#pragma unroll
        for (int j = 0; j < kInFlight; ++j)
            if (t + j < t1) normalise_item<kOutF32, kStore>(raw[j], ms[j], g0, g1, b0, b1, y, (t + j) * items_per_token, items_per_token, column);
    }
}

// any items_per_token: block b owns items [b * items_per_block, (b + 1) * items_per_block), a multiple of 1024
template <bool kOutF32, int kStore>
__global__ __launch_bounds__(256) void layernorm_apply_kernel(long long items, long long items_per_block,
                                                              int items_per_token, const uint4v* o,
                                                              const float2* mean_rstd, const float4* gamma,
                                                              const float4* beta, void* y) {
    const long long i0 = blockIdx.x * items_per_block;
    const long long i1 = i0 + items_per_block < items ? i0 + items_per_block : items;
    for (long long base = i0 + threadIdx.x; base < i1; base += kInFlight * 256) {
        uint4v raw[kInFlight];
#pragma unroll
        for (int j = 0; j < kInFlight; ++j)
            if (base + j * 256 < i1) raw[j] = __builtin_nontemporal_load(o + base + j * 256);
#pragma unroll
        for (int j = 0; j < kInFlight; ++j) {
            const long long item = base + j * 256;
            if (item < i1) {
                const long long token = item / items_per_token;
                const int c8 = static_cast<int>(item - token * items_per_token);
                normalise_item<kOutF32, kStore>(raw[j], mean_rstd[token], gamma[2 * c8], gamma[2 * c8 + 1], beta[2 * c8],
                                        beta[2 * c8 + 1], y, i0, i1 - i0, static_cast<int>(item - i0));
            }
        }
    }
}

}  // namespace

hipError_t launch_layernorm_apply(long long tokens, int D, const void* o, const float* mean_rstd, const float* gamma,
                                  const float* beta, void* y, bool out_f32, hipStream_t stream) {
    const int items_per_token = D / 8;
    const long long items = tokens * items_per_token;
    const long long bytes = items * 16;                       // of bf16 rows
    const int cus = compute_units();
    const uint4v* src = static_cast<const uint4v*>(o);
    const float2* ms = reinterpret_cast<const float2*>(mean_rstd);
    const float4* gm = reinterpret_cast<const float4*>(gamma);
    const float4* bt = reinterpret_cast<const float4*>(beta);
    if (items_per_token % 256 == 0) {
        // about eight workgroups per compute unit, each a run of at least kInFlight tokens
        const int strips = items_per_token / 256;
        long long runs = (8ll * cus + strips - 1) / strips;
        const long long most = (tokens + kInFlight - 1) / kInFlight;
        if (runs > most) runs = most;
        const int tokens_per_block = static_cast<int>((tokens + runs - 1) / runs);
        const dim3 grid(static_cast<unsigned>((tokens + tokens_per_block - 1) / tokens_per_block),
                        static_cast<unsigned>(strips));
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, tokens, tokens_per_block, items_per_token, src, ms, gm, bt, y);
        };
        out_f32 ? go(&layernorm_apply_strip_kernel<true, kStoreStreamed>)
                : bytes <= 68ll << 20 ? go(&layernorm_apply_strip_kernel<false, kStoreThrough>) : go(&layernorm_apply_strip_kernel<false, kStoreStreamed>);
        return hipGetLastError();
    }
    const long long step = kInFlight * 256;
    long long blocks = 8ll * cus;
    long long items_per_block = ((items + blocks - 1) / blocks + step - 1) / step * step;
    blocks = (items + items_per_block - 1) / items_per_block;
    const dim3 grid(static_cast<unsigned>(blocks));
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, items, items_per_block, items_per_token, src, ms, gm, bt, y);
    };
    const bool through = bytes >= 2ll << 20 && bytes <= 36ll << 20;
    out_f32 ? go(&layernorm_apply_kernel<true, kStoreStreamed>)
            : through ? go(&layernorm_apply_kernel<false, kStoreThrough>) : go(&layernorm_apply_kernel<false, kStoreStreamed>);
    return hipGetLastError();
}

hipError_t launch_layernorm_finalize(int B, int T, int H, const float* moments, float eps, float* mean_rstd,
                                     hipStream_t stream) {
    // Below 16 tokens a sequence the lane-per-token form uses fewer than a quarter of its lanes and one workgroup per
    // sequence, but it reads a line of a head's pairs once where a wave per token reads it for every token again.  So
    // the wave per token takes launches of up to 2048 tokens (one round of waves) and, with more, the lengths where the
    // heads make the other form's chain the longer one.  Lane per token : wave per token, us inside a graph: 24 sequences of one token
    // 2.15 : 1.91 (12 heads), 2.26 : 1.90 (32), 2.60 : 1.90 (64); 136 x 15 x 12 2.07 : 2.04, 1024 x 2 x 12 2.57 : 2.03, 2048 x 1 x 32 4.1 : 2.0; 1024 x
    // 8 x 12 2.5 : 2.9, x 15 2.5 : 4.0; 4096 x 2 x 32 6.0 : 2.9, x 15 6.0 : 14.0; 65 535 x 1 x 12 38 : 11; 1024 x 4 x 64 3.8 : 2.3; 1024 x 8 x 128
    // 5.8 : 3.8, x 11 5.8 : 8.2; 4096 x 8 x 256 32 : 27, x 9 32 : 43.  The lines were drawn when both folded pair after pair and err towards
    // the lanes where sequences of 2 to 6 tokens are many: 4096 x 3 x 32 6.0 : 3.5, x 4 5.9 : 4.1, 1024 x 6 x 64 3.8 : 2.7, 65 535 x 2 x 12 38 : 21.
    const long long tokens = static_cast<long long>(B) * T;
    const int longest = H / 16 < 8 ? H / 16 : 8;
    if (T < 16 && (tokens <= 2048 || T == 1 || T <= longest)) {
        hipLaunchKernelGGL(layernorm_finalize_few_kernel, dim3(static_cast<unsigned>((tokens + 3) / 4)), dim3(256), 0, stream, tokens, T, H,
                           reinterpret_cast<const float2*>(moments), eps, reinterpret_cast<float2*>(mean_rstd));
        return hipGetLastError();
    }
    const dim3 grid(static_cast<unsigned>((T + 63) / 64), static_cast<unsigned>(B));
    // Pairs folded one after the other : here, us inside a graph: 8 x 2048 tokens x 8 heads 2.24 : 2.00, x 16 2.33 : 2.00, x 32 2.62 : 2.14,
    // x 64 3.21 : 2.51, x 128 4.43 : 3.30, x 256 7.32 : 5.15, x 300 10.5 : 9.4; 1024 x 11 x 32 4.02 : 2.93, 32 x 4096 x 2 2.50 : 2.43, and of
    // one head, with nothing to fold, 2.29 : 2.41.
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, T, H, reinterpret_cast<const float2*>(moments), eps, reinterpret_cast<float2*>(mean_rstd));
    };
    if (H <= 4) go(&layernorm_finalize_kernel<1, false>);
    else if (H <= 16) go(&layernorm_finalize_kernel<4, false>);
    else if (H <= 32) go(&layernorm_finalize_kernel<8, false>);
    else if (H <= 48) go(&layernorm_finalize_kernel<12, false>);
    else if (H <= 64) go(&layernorm_finalize_kernel<16, false>);
    else if (H <= 96) go(&layernorm_finalize_kernel<24, false>);
    else if (H <= 128) go(&layernorm_finalize_kernel<32, false>);
    else if (H <= 160) go(&layernorm_finalize_kernel<40, false>);
    else if (H <= 192) go(&layernorm_finalize_kernel<48, false>);
    else if (H <= 256) go(&layernorm_finalize_kernel<64, false>);
    else go(&layernorm_finalize_kernel<64, true>);
    return hipGetLastError();
}

}  // namespace wkv6

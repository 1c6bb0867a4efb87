// The two passes of the token split in front of the chunked kernel, for gfx950 (MI355X).  The recurrence
// (Finch-C2 Time Mixing: decay map w = exp(-exp(x)), state wkv_t) is linear in the state, so over a segment of tokens
//
//     S_out = diag(D) S_in + S_local,   S_local = sum_i diag(prod_{s>i} w_s) k_i^T v_i,   D = prod w
//
// First pass: S_local and D of every segment but the last.  Each of a workgroup's eight waves takes an eighth of the
// segment's 32-token chunks, carries its own 64 x 64 state over them in MFMA registers (v_mfma_f32_16x16x32_f16, fp32
// accumulation), and the eight results are scaled by the later waves' total decays and added through LDS at the
// end.  There is no barrier in the loop: the contraction index (the token) and the rows and columns (value and key channels) of
// the product may be dealt to lanes in any order that all operands share, so lane (l16, g4) takes tokens 8 g4 .. +7 and
// channels 4 l16 .. +3 of k, v and x alike: each is eight 8-byte loads of whole 128-byte rows, already in operand layout.
//
// The fp16 operands are the chunked kernel's, bit for bit: the same products of decays in the same order, the same two
// roundings of a scaled key.  The states that the segments hand on therefore differ from those of an unsplit walk by the
// rounding of fp32 sums alone (a few 1e-7), not by the rounding of operands, whatever the segments are.
//
// Bound by HBM when the segments fill the chip (7 segments of 16 384 tokens, 32 heads: 1.41 GB) and by the latency of a few
// chunks when they are short (7 segments of 512 tokens, 32 heads: 11 us).  The chunked kernel's own pipeline, which made this
// pass before, needs five windows of 0.5 us to fill and drain.  Whole calls of the explicit split, microseconds, before ->
// now, with the tensors spread over address bits 7..9 and, in brackets, equally aligned: Finch 131 072 tokens x 32 heads
// 748 -> 701 (814 -> 817), 131 072 x 16 382 -> 356 (419 -> 413), 8192 x 24 86 -> 81 (87 -> 84); Finch-C2 131 072 x 32
// 907 -> 858 (983 -> 952), 131 072 x 16 466 -> 426 (500 -> 478).  Equally aligned Finch inputs are where it loses: up to 1.3 %
// at 32 heads, and more where a token's rows lie a multiple of 5 KiB apart (40 heads: 8192 tokens 97 -> 100, 131 072
// 1082 -> 1129).  The earlier pass, brought back for comparison, has the better figure there and loses 2 to 6 % with tensors
// that are spread out; the two add up in another order, and the bits of a result must not depend on where its tensors lie,
// so the choice cannot follow the alignment.
#include "wkv6_launch.h"
#include "wkv6_math.h"

#include <type_traits>

namespace wkv6 {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef unsigned uint4v __attribute__((ext_vector_type(4)));
typedef unsigned uint2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kChunk = 32;
constexpr int kWaves = 8;
constexpr int kStateLds = kWaves * 64 * 64 * 4;       // the waves' scaled states (during the walk the decay path's outer factor)
constexpr int kDecayOff = kStateLds;                  // their total decays [wave][64]
constexpr int kSegLds = kStateLds + kWaves * 64 * 4;
static_assert(kSegLds <= 160 * 1024, "LDS budget");

// The value of `v` in the wave's four rows of 16 lanes, each in every lane of a column: v(l16, 0), (l16, 1), ..
__device__ __forceinline__ void rows_of(float v, float& r0, float& r1, float& r2, float& r3) {
    const unsigned u = __float_as_uint(v);
    const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);         // rows 0 0 2 2 and 1 1 3 3
    const auto b = __builtin_amdgcn_permlane32_swap(a[0], a[0], false, false);
    const auto c = __builtin_amdgcn_permlane32_swap(a[1], a[1], false, false);
    r0 = __uint_as_float(b[0]);
    r2 = __uint_as_float(b[1]);
    r1 = __uint_as_float(c[0]);
    r3 = __uint_as_float(c[1]);
}

struct SegRegs {                                      // one chunk: this lane's 8 tokens x 4 channels
    uint2v k[8], v[8], x[8];
    bf16x8 y[2][2];                                   // fused decay path: y rows instead of x
};

// kPolicy: cache policy of the k, v, x loads, 0 (temporal) or 2 (non-temporal).  The last pass reads the same rows again
// soon: when they fit the 256 MB memory-side cache, temporal loads leave them there (B = 1, T = 4096, H = 32, the whole call:
// 40.5 -> 38.3 us; B = 2, T = 8192, Finch-C2: 129.6 -> 124.0); beyond that they only displace one another (T =
// 65 536: 396 -> 405).
constexpr long long kMemorySideCache = 256ll << 20;

template <bool kC2, bool kLora, int kPolicy>
__global__ __launch_bounds__(64 * kWaves) void segment_state_kernel(Args a) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    clamp_fp16_overflow();
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int bs = blockIdx.x / a.H;                  // batch * (segs - 1) + segment
    const int h = blockIdx.x - bs * a.H;
    const int b = bs / (a.segs - 1);
    const int seg = bs - b * (a.segs - 1);
    const long long row_bytes = static_cast<long long>(a.H) * kHeadSize * 2;
    const long long first = static_cast<long long>(seg) * a.seg_len;             // the segment's first token
    const long long base = b * a.batch_stride * 2 + first * row_bytes + h * (kHeadSize * 2);
    const int nchunks = a.seg_len / kChunk;           // whole chunks only: the last segment has no workgroup here
    const int c_lo = nchunks * wave / kWaves, c_hi = nchunks * (wave + 1) / kWaves;
    int voff[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) voff[j] = static_cast<int>((8 * g4 + j) * row_bytes) + 8 * l16;

    // fused decay path: the head's 64 x 64 slice of B as eight MFMA operands (columns 4 l16 + c, half ks of the rank)
    // in LDS, one brought in by each wave; rows of y come per chunk
    [[maybe_unused]] float4v lam = {0.f, 0.f, 0.f, 0.f};
    if constexpr (kLora) {
        const int width = a.H * kHeadSize, c = wave >> 1, ks = wave & 1;
        const __bf16* bwp = static_cast<const __bf16*>(a.bw) + h * kHeadSize;
        bf16x8 q;
#pragma unroll
        for (int e = 0; e < 8; ++e) q[e] = bwp[static_cast<long long>(32 * ks + 8 * g4 + e) * width + 4 * l16 + c];
        *reinterpret_cast<bf16x8*>(lds + wave * 1024 + lane * 16) = q;
        lam = *reinterpret_cast<const float4v*>(a.lambda + h * kHeadSize + 4 * l16);
        __syncthreads();
    }
    [[maybe_unused]] auto b_operand = [&](int c, int ks) { return *reinterpret_cast<const bf16x8*>(lds + (2 * c + ks) * 1024 + lane * 16); };
    // rows of the product y B: row m of half `hf` is token 8 (m >> 2) + 4 hf + (m & 3), so that a lane's results
    // are its own tokens
    [[maybe_unused]] const int y_voff = (8 * (l16 >> 2) + (l16 & 3)) * (kLoraRank * 2) + 16 * g4;

    auto rows_rsrc = [&](const void* p, int c) {      // chunk c of a [B][T][H][N] stream; past the wave's last one an empty descriptor
        const bool live = c < c_hi;                   // uniform
        const long long off = static_cast<long long>(live ? c : 0) * kChunk * row_bytes;
        return chunk_rsrc(static_cast<const char*>(p) + base, off, live ? off + kChunk * row_bytes : 0);
    };
    auto fetch_keys = [&](SegRegs& s, int c) {
        const __amdgpu_buffer_rsrc_t rk = rows_rsrc(a.k, c);
        if constexpr (kLora) {
            const bool live = c < c_hi;
            const long long y0 = static_cast<long long>(live ? c : 0) * kChunk * (kLoraRank * 2);
            const __amdgpu_buffer_rsrc_t ry = chunk_rsrc(static_cast<const char*>(a.y) + (b * static_cast<long long>(a.T) + first) * (kLoraRank * 2),
                                                         y0, live ? y0 + kChunk * (kLoraRank * 2) : 0);
#pragma unroll
            for (int hf = 0; hf < 2; ++hf)
#pragma unroll
                for (int ks = 0; ks < 2; ++ks)
                    s.y[hf][ks] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(
                                                                 ry, y_voff + 4 * hf * (kLoraRank * 2) + 64 * ks, 0, 0));
        } else {
            const __amdgpu_buffer_rsrc_t rx = rows_rsrc(a.x, c);
#pragma unroll
            for (int j = 0; j < 8; ++j) s.x[j] = __builtin_bit_cast(uint2v, __builtin_amdgcn_raw_buffer_load_b64(rx, voff[j], 0, kPolicy));
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) s.k[j] = __builtin_bit_cast(uint2v, __builtin_amdgcn_raw_buffer_load_b64(rk, voff[j], 0, kPolicy));
    };
    auto fetch_values = [&](SegRegs& s, int c) {
        const __amdgpu_buffer_rsrc_t rv = rows_rsrc(a.v, c);
#pragma unroll
        for (int j = 0; j < 8; ++j) s.v[j] = __builtin_bit_cast(uint2v, __builtin_amdgcn_raw_buffer_load_b64(rv, voff[j], 0, kPolicy));
    };

    // S[jb][nb][e] = state[key channel 4 l16 + nb][value channel 16 g4 + 4 e + jb]: a lane's key channels are those it
    // forms the decays of
    float4v S[4][4];
#pragma unroll
    for (int jb = 0; jb < 4; ++jb)
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) S[jb][nb] = float4v{0.f, 0.f, 0.f, 0.f};
    float4v total = {1.f, 1.f, 1.f, 1.f};             // decays of the wave's tokens so far, channels 4 l16 ..

    auto value = [](const uint2v& q, int c) { return c & 1 ? bf16_hi(q[c >> 1]) : bf16_lo(q[c >> 1]); };
    uint4v kt[4];                                     // the chunk's scaled keys, channel by channel: the product's B operand
    auto scale_keys = [&](const SegRegs& s) {         // and the state's decay over the chunk
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            [[maybe_unused]] float4v d[2];            // fused decay path: the channel's logits
            if constexpr (kLora) {
#pragma unroll
                for (int hf = 0; hf < 2; ++hf) {
                    d[hf] = float4v{lam[c], lam[c], lam[c], lam[c]};
                    d[hf] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(s.y[hf][0], b_operand(c, 0), d[hf], 0, 0, 0);
                    d[hf] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(s.y[hf][1], b_operand(c, 1), d[hf], 0, 0, 0);
                }
            }
            float o[2];                               // products over the lane's two 4-token groups
#pragma unroll
            for (int gr = 0; gr < 2; ++gr) {
                float w[4], kk[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    float e = 0.f;
                    w[j] = decay_of(kLora ? d[gr][j] : value(s.x[4 * gr + j], c), e);
                    kk[j] = value(s.k[4 * gr + j], c);
                    if constexpr (kC2) kk[j] *= one_minus_decay(e, w[j]);
                }
                // decays behind each token inside the group, rounded to fp16 as the key's first factor
                const float s1 = w[2] * w[3], s0 = w[1] * s1;
                o[gr] = w[0] * w[1] * w[2] * w[3];
                kt[c][2 * gr] = mul_h2(pack_h2(kk[0], kk[1]), pack_h2(s0, s1));
                kt[c][2 * gr + 1] = mul_h2(pack_h2(kk[2], kk[3]), pack_h2(w[3], 1.f));
            }
            // decays of the groups behind it in the chunk, the second factor; p[i]: groups 2 i, 2 i + 1
            float p0, p1, p2, p3, first0, unused1, unused2, unused3;
            rows_of(o[0] * o[1], p0, p1, p2, p3);
            const float q3 = g4 < 3 ? p3 : 1.f, q2 = g4 < 2 ? p2 : 1.f, q1 = g4 < 1 ? p1 : 1.f;
            const float behind = q1 * (q2 * q3);
            const float first = o[1] * behind;        // behind the first of the two groups
            const unsigned f0 = pack_h2(first, first), f1 = pack_h2(behind, behind);
            kt[c][0] = mul_h2(kt[c][0], f0);
            kt[c][1] = mul_h2(kt[c][1], f0);
            kt[c][2] = mul_h2(kt[c][2], f1);
            kt[c][3] = mul_h2(kt[c][3], f1);
            rows_of(o[0] * first, first0, unused1, unused2, unused3);    // row 0: the whole chunk's decay
            total[c] *= first0;
#pragma unroll
            for (int jb = 0; jb < 4; ++jb) S[jb][c] *= first0;
            __builtin_amdgcn_sched_barrier(0);        // one channel's temporaries at a time: the registers are full
        }
    };
    auto accumulate = [&](const SegRegs& s) {
#pragma unroll
        for (int jb = 0; jb < 4; ++jb) {
            uint4v q;
#pragma unroll
            for (int p = 0; p < 4; ++p) q[p] = pack_h2(value(s.v[2 * p], jb), value(s.v[2 * p + 1], jb));
#pragma unroll
            for (int nb = 0; nb < 4; ++nb)
                S[jb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, q), __builtin_bit_cast(half8, kt[nb]), S[jb][nb], 0, 0, 0);
        }
    };
    if constexpr (kLora) {
        // one register set (two spill): the next chunk's keys and y rows are requested behind this one's scaling
        SegRegs s;
        fetch_keys(s, c_lo);
        fetch_values(s, c_lo);
#pragma clang loop unroll(disable)
        for (int c = c_lo; c < c_hi; ++c) {
            scale_keys(s);
            fetch_keys(s, c + 1);
            accumulate(s);
            fetch_values(s, c + 1);
        }
    } else {
        // The next chunk's keys and logits are requested in front of this one's scaling, its values behind it: all 24 loads
        // at once reach the memory as one burst, which is worst where k, v and x start at equally aligned addresses
        // (whole calls, Finch: one sequence of 131 072 tokens and 32 heads, spread out 707.7 -> 700.9 us, equally
        // aligned 818.6 -> 817.3, 8192 tokens and 40 heads 102.8 -> 99.8).
        SegRegs s0, s1;
        fetch_keys(s0, c_lo);
        fetch_values(s0, c_lo);
        int c = c_lo;
#pragma clang loop unroll(disable)
        for (; c + 1 < c_hi; c += 2) {
            fetch_keys(s1, c + 1);
            scale_keys(s0);
            fetch_values(s1, c + 1);
            accumulate(s0);
            fetch_keys(s0, c + 2);
            scale_keys(s1);
            fetch_values(s0, c + 2);
            accumulate(s1);
        }
        if (c < c_hi) {
            scale_keys(s0);
            accumulate(s0);
        }
    }

    // the waves' total decays (behind the barrier B is not read any more); each wave's state scaled by the later waves'
    float* decay = reinterpret_cast<float*>(lds + kDecayOff);
    if (g4 == 0) *reinterpret_cast<float4v*>(decay + wave * 64 + 4 * l16) = total;
    __syncthreads();
    float4v later = {1.f, 1.f, 1.f, 1.f};
#pragma unroll
    for (int w = kWaves - 1; w > 0; --w)
        if (w > wave) later *= *reinterpret_cast<const float4v*>(decay + w * 64 + 4 * l16);
    char* place = a.place.base + b * a.place.batch + seg * a.place.seg + h * a.place.head;
    if (wave == 0 && g4 == 0)                         // the segment's total decay: the row behind the state
        *reinterpret_cast<float4v*>(place + 64ll * a.place.row + (l16 >> 3) * a.place.half + (l16 & 7) * 16) = later * total;
    // 16-byte granules of a state row are swizzled by its channel quad, so that the sixteen lanes of a write, four rows
    // apart, spread over all banks
    char* part = lds + wave * (64 * 64 * 4);
#pragma unroll
    for (int nb = 0; nb < 4; ++nb)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            *reinterpret_cast<float4v*>(part + (4 * l16 + nb) * 256 + 16 * ((4 * g4 + e) ^ l16)) =
                float4v{S[0][nb][e], S[1][nb][e], S[2][nb][e], S[3][nb][e]} * later[nb];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int at = tid + 64 * kWaves * i, row = at >> 4, granule = at & 15;
        const int off = row * 256 + 16 * (granule ^ (row >> 2));
        float4v sum = *reinterpret_cast<const float4v*>(lds + off);
#pragma unroll
        for (int w = 1; w < kWaves; ++w) sum += *reinterpret_cast<const float4v*>(lds + w * (64 * 64 * 4) + off);
        *reinterpret_cast<float4v*>(place + static_cast<long long>(row) * a.place.row + (granule >> 3) * a.place.half + (granule & 7) * 16) = sum;
    }
}

// Second pass: the state entering every segment, in place.  One workgroup per 16 rows of a (batch, head)'s state, 4
// values per thread; the segments' states do not depend on one another, so eight of them are fetched together and
// only the multiply-adds are a chain.
__global__ __launch_bounds__(256) void segment_fold_kernel(Args a) {
    constexpr int kAhead = 8;
    const int unit = blockIdx.x >> 2;                 // batch * H + head
    const int b = unit / a.H, h = unit - b * a.H;
    const int row = 16 * (blockIdx.x & 3) + (threadIdx.x >> 4), col = 4 * (threadIdx.x & 15);
    char* place = a.place.base + b * a.place.batch + h * a.place.head;
    const long long at = static_cast<long long>(row) * a.place.row + (col >> 5) * a.place.half + (col & 31) * 4;
    const long long at_d = 64ll * a.place.row + (row >> 5) * a.place.half + (row & 31) * 4;
    float4v S = {0.f, 0.f, 0.f, 0.f};
    if (a.state_in) S = *reinterpret_cast<const float4v*>(a.state_in + static_cast<long long>(unit) * 4096 + row * 64 + col);
    for (int p0 = 0; p0 < a.segs - 1; p0 += kAhead) {
        float4v local[kAhead];
        float d[kAhead];
#pragma unroll
        for (int i = 0; i < kAhead; ++i)
            if (p0 + i < a.segs - 1) {
                local[i] = *reinterpret_cast<const float4v*>(place + (p0 + i) * a.place.seg + at);
                d[i] = *reinterpret_cast<const float*>(place + (p0 + i) * a.place.seg + at_d);
            }
#pragma unroll
        for (int i = 0; i < kAhead; ++i)
            if (p0 + i < a.segs - 1) {
                *reinterpret_cast<float4v*>(place + (p0 + i) * a.place.seg + at) = S;      // entering segment p0 + i
#pragma unroll
                for (int e = 0; e < 4; ++e) S[e] = fmaf(d[i], S[e], local[i][e]);
            }
    }
    *reinterpret_cast<float4v*>(place + (a.segs - 1) * a.place.seg + at) = S;              // entering the last one
}

}  // namespace

hipError_t raise_segment_limits() {
    struct Tag {};
    return once_per_device<Tag>([] {
        hipError_t e = set_lds_limit(&segment_state_kernel<false, false, 0>, kSegLds);
        if (e == hipSuccess) e = set_lds_limit(&segment_state_kernel<true, false, 0>, kSegLds);
        if (e == hipSuccess) e = set_lds_limit(&segment_state_kernel<false, true, 0>, kSegLds);
        if (e == hipSuccess) e = set_lds_limit(&segment_state_kernel<true, true, 0>, kSegLds);
        if (e == hipSuccess) e = set_lds_limit(&segment_state_kernel<false, false, 2>, kSegLds);
        if (e == hipSuccess) e = set_lds_limit(&segment_state_kernel<true, false, 2>, kSegLds);
        if (e == hipSuccess) e = set_lds_limit(&segment_state_kernel<false, true, 2>, kSegLds);
        if (e == hipSuccess) e = set_lds_limit(&segment_state_kernel<true, true, 2>, kSegLds);
        return e;
    });
}

hipError_t launch_segment_states(const Args& a, bool lora, hipStream_t stream) {
    const hipError_t err = raise_segment_limits();
    if (err != hipSuccess || a.segs < 2) return err;      // (a call with one segment only raises the limits)
    const dim3 grid(static_cast<unsigned>(a.B) * static_cast<unsigned>(a.segs - 1) * static_cast<unsigned>(a.H));
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(64 * kWaves), kSegLds, stream, a); };
    auto pass = [&](auto policy) {
        constexpr int kPolicy = decltype(policy)::value;
        if (lora)
            a.finch_c2 ? go(&segment_state_kernel<true, true, kPolicy>) : go(&segment_state_kernel<false, true, kPolicy>);
        else
            a.finch_c2 ? go(&segment_state_kernel<true, false, kPolicy>) : go(&segment_state_kernel<false, false, kPolicy>);
    };
    const long long read_again = static_cast<long long>(a.B) * a.T * a.H * kHeadSize * 2 * (lora ? 2 : 3);
    if (read_again <= kMemorySideCache)
        pass(std::integral_constant<int, 0>{});
    else
        pass(std::integral_constant<int, 2>{});
    const hipError_t launched = hipGetLastError();
    if (launched != hipSuccess) return launched;
    hipLaunchKernelGGL(segment_fold_kernel, dim3(4u * static_cast<unsigned>(a.B) * static_cast<unsigned>(a.H)), dim3(256), 0, stream, a);
    return hipGetLastError();
}

}  // namespace wkv6

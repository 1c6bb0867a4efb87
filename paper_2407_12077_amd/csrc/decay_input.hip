// The operators in front of the fused decay path, for gfx950 (Finch-C2 Time Mixing: lerp, lora and
// ddlerp operator equations and d_t = lora_omega(ddlerp_d(x_t, x_{t-1}))): from the layer input x to
//
//     z_t = x_t + (x_{t-1} - x_t) * (lambda_d + tanh((x_t + (x_{t-1} - x_t) * mu_x) A_d) B_d)
//     y_t = tanh(z_t A_omega)                                         64 values per token
//
// which wkv6_finch_c2_prefill_lora_bf16 turns into decay logits per head.  Per token this is a chain
// of three skinny matrix products (D -> 32, 32 -> D, D -> 64) bound by the one HBM read of x.
//
// Two kernels; the rule is at the launch.  With enough tokens to fill the chip:
// One workgroup owns 128 consecutive tokens of one sequence and walks the D axis twice in steps of 128
// channels (the second walk needs tanh(q A_d) of the whole first one; its reads of x are served by
// L2 / the last-level cache).  Sixteen waves in two roles, one barrier per step; the steps are this
// heavy (and the workgroup this large) because a step has to last long enough for loads issued two
// steps ahead to arrive: with 64 tokens and 64 channels per step the same pipeline ran at the memory
// latency, not the memory rate (102 us against 180 us for a version without a pipeline at all).
//   waves 8..15 LOADERS: fetch, two steps ahead, the step's x rows (128 tokens and the row before the
//               first one: 256-byte pieces, 16 lanes each) and its weight slices with 16-byte loads,
//               convert the weights to fp16 and park everything in one of two LDS stages.  Rows past
//               the end of the sequence go through shrunk raw buffer descriptors and read as zero.
//   waves 0..7  WORKERS: wave w owns tokens 16w .. 16w+15 through the whole chain, in registers:
//     walk 1    q = x_t + (x_{t-1} - x_t) mu_x in fp32, rounded to fp16 (11 significant bits: bf16
//               operands would put the result outside the 2e-3 bar), times A_d
//               (v_mfma_f32_16x16x32_f16, weights as the A operand so that a lane ends up with its
//               own token's 8 inner-rank sums); tanh; that is already the B operand p of walk 2.
//     walk 2    per block of 16 channels: (lambda_d + B_d^T p) by one MFMA whose result layout (a
//               lane holds four consecutive channels of its token) is the operand layout of the
//               16x16x16 MFMA, so z = x_t + (x_{t-1} - x_t) * mix is formed in registers and fed
//               straight into the product with A_omega; mix and z never touch LDS or HBM.
//               The y accumulators (a lane: four consecutive outputs of its token per 16-column
//               block) get their tanh and leave through the wave's own piece of LDS as whole rows
//               (1 % faster than 8-byte stores straight from the accumulator layout).
// One workgroup per compute unit (134 KB of LDS, 128 registers per thread).
//
// Weight layouts are the ones an MFMA operand can be read from with the contraction index
// contiguous: A_d and A_omega column by column ([r][D]), B_d column by column ([D][r]).
#include "wkv6_launch.h"
#include "wkv6_lds_loads.h"

namespace wkv6 {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef unsigned uint4v __attribute__((ext_vector_type(4)));
typedef unsigned uint2v __attribute__((ext_vector_type(2)));

constexpr int kTokens = 128;         // tokens per workgroup
constexpr int kStepCh = 128;         // channels per step
constexpr int kInnerRank = 32;       // columns of A_d
constexpr int kOuterRank = 64;       // columns of A_omega
constexpr int kWorkerWaves = kTokens / 16;
constexpr int kLoaderThreads = 512;
constexpr int kDiThreads = 64 * kWorkerWaves + kLoaderThreads;      // 8 worker waves + 8 loader waves
constexpr int kXRowB = 288;          // LDS row stride of 128-channel rows (256 B + 32 pad: full-rate 16-byte reads)
constexpr int kBdRow = 96;           // LDS row stride of the B_d slice (32 ranks = 64 B + 32 pad)
// one LDS stage (bytes): x rows 0..127 = tokens, row 128 = the row before the first token
constexpr int kOffX = 0;
constexpr int kOffVec = kOffX + (kTokens + 1) * kXRowB; // mu_x (walk 1) or lambda_d (walk 2) slice: 128 fp32
constexpr int kOffW1 = kOffVec + kStepCh * 4;           // walk 1: A_d slice [32 columns][128 channels] fp16
constexpr int kOffBd = kOffVec + kStepCh * 4;           // walk 2: B_d slice [128 channels][32 ranks] fp16
constexpr int kOffWo = kOffBd + kStepCh * kBdRow;       // walk 2: A_omega slice [64 columns][128 channels] fp16
constexpr int kStageBytes = (kOffWo + kOuterRank * kXRowB + 255) / 256 * 256;
constexpr int kDiLds = 2 * kStageBytes;
static_assert(kOffW1 + kInnerRank * kXRowB <= kStageBytes && kDiLds <= 160 * 1024, "stage layout");

struct DiArgs {
    int B, T, D;
    int tiles_per_seq;
    const char* x;          // [B][T][D] bf16
    const char* x_prev;     // [B][D] bf16 or nullptr
    const char* mu_x;       // [D] fp32
    const char* lambda_d;   // [D] fp32
    const char* a_d;        // [32][D] bf16
    const char* b_d;        // [D][32] bf16
    const char* a_omega;    // [64][D] bf16
    void* y;                // [B][T][64] bf16 or fp32
};

__device__ __forceinline__ float lo_f(unsigned bits) { return __uint_as_float(bits << 16); }
__device__ __forceinline__ float hi_f(unsigned bits) { return __uint_as_float(bits & 0xffff0000u); }

__device__ __forceinline__ unsigned pack_h2f(float a, float b) {
    typedef _Float16 half2v __attribute__((ext_vector_type(2)));
    half2v p;
    p.x = static_cast<_Float16>(a);
    p.y = static_cast<_Float16>(b);
    return __builtin_bit_cast(unsigned, p);
}
// eight bf16 (four dwords) as four fp16 pairs (exact for magnitudes inside the fp16 range)
__device__ __forceinline__ uint4v bf16x8_to_f16x8(uint4v q) {
    uint4v h;
#pragma unroll
    for (int i = 0; i < 4; ++i) h[i] = pack_h2f(lo_f(q[i]), hi_f(q[i]));
    return h;
}

// tanh through one exponential and one reciprocal: 1 - 2 / (exp(2a) + 1); exact limits at +-inf
__device__ __forceinline__ float fast_tanh(float a) {
    const float e = __builtin_amdgcn_exp2f(a * 2.8853900817779268f);     // exp(2a)
    return 1.f - 2.f * __builtin_amdgcn_rcpf(e + 1.f);
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_of(const char* base, long long bytes) {
    if (bytes < 0) bytes = 0;
    if (bytes > 0x7fffffffLL) bytes = 0x7fffffffLL;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), 0, static_cast<int>(bytes), 0x00020000);
}

struct StepRegs {          // a loader thread's share of one step
    uint4v x0, x1, x2, x3, xp;   // x rows xr + 32 i; the row before the first token (threads 0..15)
    uint4v w0, w1, w2;     // walk 1: A_d piece (w0); walk 2: B_d piece (w0), two A_omega pieces (w1, w2)
    uint4v vec;            // mu_x / lambda_d piece (threads 0..31)
};

// ------------------------------------------------------------------------------------------
// loader waves (512 threads)
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ void di_loader(const DiArgs& a, char* lds, int lt, int b, int t0, int ntok, int nsteps,
                                          int first) {
    const long long row_bytes = static_cast<long long>(a.D) * 2;
    const char* tile = a.x + (static_cast<long long>(b) * a.T + t0) * row_bytes;
    const char* pred = t0 > 0 ? tile - row_bytes : (a.x_prev ? a.x_prev + static_cast<long long>(b) * row_bytes : nullptr);
    const long long tile_bytes = static_cast<long long>(ntok) * row_bytes;
    const int nchunks = a.D / kStepCh;
    const int xr = lt >> 4, xg = lt & 15;                   // 16 lanes per 256-byte row piece, 32 rows per pass
    const int x_voff0 = static_cast<int>(xr * row_bytes + 16 * xg);
    const int x_vstep = static_cast<int>(32 * row_bytes);
    const long long wcol_bytes = row_bytes;                 // a_d / a_omega: one column = D bf16

    auto fetch = [&](StepRegs& s, int step) {
        const bool live = step < nsteps;                                   // uniform
        // Both walks are sums over the channel blocks, so their order is free: walk 1 goes up from a
        // block that differs between workgroups (workgroups marching through the channels in step
        // would all ask the same memory channels for their row pieces, which are D*2 bytes apart),
        // walk 2 comes back down, so that it starts with the blocks most recently brought into L2.
        const bool walk2 = step >= nchunks;
        int chunk = walk2 ? first + 2 * nchunks - 1 - step : first + step;
        if (chunk >= nchunks) chunk -= nchunks;
        if (!live) chunk = 0;                                              // nothing is fetched: keep the bases in range
        const long long coff = static_cast<long long>(chunk) * (kStepCh * 2);   // byte offset of the chunk in a row
        const __amdgpu_buffer_rsrc_t rx = rsrc_of(tile + coff, live ? tile_bytes - coff : 0);
        s.x0 = __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(rx, x_voff0, 0, 0));
        s.x1 = __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(rx, x_voff0 + x_vstep, 0, 0));
        s.x2 = __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(rx, x_voff0 + 2 * x_vstep, 0, 0));
        s.x3 = __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(rx, x_voff0 + 3 * x_vstep, 0, 0));
        const __amdgpu_buffer_rsrc_t rp = rsrc_of(pred ? pred + coff : a.x, (live && pred) ? kStepCh * 2 : 0);
        s.xp = __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(rp, lt < 16 ? 16 * lt : 0x7ffffff0, 0, 0));
        const char* vec = walk2 ? a.lambda_d : a.mu_x;
        const __amdgpu_buffer_rsrc_t rv = rsrc_of(vec + chunk * (kStepCh * 4), live ? kStepCh * 4 : 0);
        s.vec = __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(rv, lt < 32 ? 16 * lt : 0x7ffffff0, 0, 0));
        // walk 1: A_d slice (column lt>>4, 16-byte piece lt&15 of its 128 channels); walk 2: B_d slice (channel
        // lt>>2 of the chunk, 16-byte piece lt&3 of its 32 ranks) and A_omega slice (columns lt>>4 and
        // 32 + (lt>>4)).  Every load is issued in both walks, through an empty descriptor where it has
        // nothing to fetch, so that the step's registers are plain values on every path.
        const __amdgpu_buffer_rsrc_t rw0 =
            walk2 ? rsrc_of(a.b_d + static_cast<long long>(chunk) * (kStepCh * kInnerRank * 2), live ? kStepCh * kInnerRank * 2 : 0)
                  : rsrc_of(a.a_d + coff, live ? kInnerRank * wcol_bytes - coff : 0);
        const int w0_voff = walk2 ? (lt >> 2) * (kInnerRank * 2) + 16 * (lt & 3) : static_cast<int>(xr * wcol_bytes + 16 * xg);
        s.w0 = __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(rw0, w0_voff, 0, 0));
        const __amdgpu_buffer_rsrc_t ro = rsrc_of(a.a_omega + coff, (live && walk2) ? kOuterRank * wcol_bytes - coff : 0);
        s.w1 = __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(ro, static_cast<int>(xr * wcol_bytes + 16 * xg), 0, 0));
        s.w2 = __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(ro, static_cast<int>((xr + 32) * wcol_bytes + 16 * xg), 0, 0));
    };
    auto park = [&](const StepRegs& s, int step) {
        char* st = lds + (step & 1) * kStageBytes;
        const bool walk2 = step >= nchunks;
        char* xdst = st + kOffX + xr * kXRowB + 16 * xg;
        *reinterpret_cast<uint4v*>(xdst) = s.x0;
        *reinterpret_cast<uint4v*>(xdst + 32 * kXRowB) = s.x1;
        *reinterpret_cast<uint4v*>(xdst + 64 * kXRowB) = s.x2;
        *reinterpret_cast<uint4v*>(xdst + 96 * kXRowB) = s.x3;
        if (lt < 16) *reinterpret_cast<uint4v*>(st + kOffX + kTokens * kXRowB + 16 * lt) = s.xp;
        if (lt < 32) *reinterpret_cast<uint4v*>(st + kOffVec + 16 * lt) = s.vec;
        if (!walk2) {
            *reinterpret_cast<uint4v*>(st + kOffW1 + xr * kXRowB + 16 * xg) = bf16x8_to_f16x8(s.w0);
        } else {
            // The inner ranks of a B_d row are stored in the order in which walk 1 leaves them in a
            // worker lane: 16-byte granule g4 holds ranks 4*g4 .. 4*g4+3 and 16 + 4*g4 .. 16 + 4*g4+3.
            // This thread has ranks 8g .. 8g+7 (g = lt & 3): two 8-byte halves of two granules.
            const uint4v h = bf16x8_to_f16x8(s.w0);
            const int g = lt & 3;
            char* rowp = st + kOffBd + (lt >> 2) * kBdRow + 8 * (g >> 1);
            *reinterpret_cast<uint2v*>(rowp + 16 * (2 * (g & 1))) = uint2v{h[0], h[1]};
            *reinterpret_cast<uint2v*>(rowp + 16 * (2 * (g & 1) + 1)) = uint2v{h[2], h[3]};
            *reinterpret_cast<uint4v*>(st + kOffWo + xr * kXRowB + 16 * xg) = bf16x8_to_f16x8(s.w1);
            *reinterpret_cast<uint4v*>(st + kOffWo + (xr + 32) * kXRowB + 16 * xg) = bf16x8_to_f16x8(s.w2);
        }
    };

    // nsteps is even (two walks of D / 128 steps); same barrier sequence as the workers: one before the
    // first step and one after every step
    StepRegs s0, s1;
    fetch(s0, 0);
    fetch(s1, 1);
    park(s0, 0);
    fetch(s0, 2);
    __syncthreads();                                   // stage of step 0 is in LDS
#pragma clang loop unroll(disable)
    for (int step = 0; step < nsteps; step += 2) {
        park(s1, step + 1);                            // while the workers are on `step`
        fetch(s1, step + 3);
        __syncthreads();
        if (step + 2 < nsteps) park(s0, step + 2);
        fetch(s0, step + 4);
        __syncthreads();
    }
}

// ------------------------------------------------------------------------------------------
// worker waves (512 threads): wave w owns tokens 16w .. 16w + 15
// ------------------------------------------------------------------------------------------
template <bool kOutF32>
__device__ __forceinline__ void di_worker(const DiArgs& a, char* lds, int lane, int w, int b, int t0, int ntok,
                                          int nsteps) {
    const int l16 = lane & 15;
    const int g4 = lane >> 4;
    const int nchunks = a.D / kStepCh;
    const int trow = 16 * w + l16;                               // this lane's token row in the stage
    const int prow = trow == 0 ? kTokens : trow - 1;             // and its previous token's
    const int xt_off = kOffX + trow * kXRowB, xp_off = kOffX + prow * kXRowB;

    float4v pacc[2] = {float4v{0.f, 0.f, 0.f, 0.f}, float4v{0.f, 0.f, 0.f, 0.f}};
    float4v yacc[4];
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) yacc[nb] = float4v{0.f, 0.f, 0.f, 0.f};
    half8 pt;                                                    // tanh(q A_d) of this lane's token, walk 1's rank order

    auto walk1 = [&](const char* st) {
#pragma unroll
        for (int kb = 0; kb < kStepCh / 32; ++kb) {
            const int col = 64 * kb + 16 * g4;                   // byte column of this lane's 8 channels
            const uint4v xt = *reinterpret_cast<const uint4v*>(st + xt_off + col);
            const uint4v xp = *reinterpret_cast<const uint4v*>(st + xp_off + col);
            const float4 m0 = *reinterpret_cast<const float4*>(st + kOffVec + 2 * col);
            const float4 m1 = *reinterpret_cast<const float4*>(st + kOffVec + 2 * col + 16);
            const float mu[8] = {m0.x, m0.y, m0.z, m0.w, m1.x, m1.y, m1.z, m1.w};
            uint4v q;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float c0 = lo_f(xt[i]), c1 = hi_f(xt[i]);
                q[i] = pack_h2f(__builtin_fmaf(lo_f(xp[i]) - c0, mu[2 * i], c0),
                                __builtin_fmaf(hi_f(xp[i]) - c1, mu[2 * i + 1], c1));
            }
            const half8 qh = __builtin_bit_cast(half8, q);
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) {
                // A operand: A_d columns 16nb + l16 (rows of the slice), B operand: q of token l16
                const half8 wgt = *reinterpret_cast<const half8*>(st + kOffW1 + (16 * nb + l16) * kXRowB + col);
                pacc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(wgt, qh, pacc[nb], 0, 0, 0);
            }
        }
    };
    auto walk2 = [&](const char* st) {
        // Two 16-channel blocks at a time, over 32 consecutive channels.  Which channel sits in which row
        // of the B_d^T operand is free as long as z and A_omega agree, so block `half` of a pair takes the
        // channels 8*(m>>2) + 4*half + (m&3), m = 0..15: lane group g4 then owns the eight consecutive
        // channels 8*g4 .. 8*g4+7 of the pair, and x_t, x_{t-1} and A_omega are one 16-byte read each
        // (the worker's LDS reads, not its arithmetic, bound this walk).
#pragma unroll
        for (int pair = 0; pair < kStepCh / 32; ++pair) {
            const int ch = 32 * pair + 8 * g4;                   // this lane's eight channels of the step
            const int row0 = 32 * pair + 8 * (l16 >> 2) + (l16 & 3);     // B_d^T operand row of this lane, first block
            const uint4v xt = *reinterpret_cast<const uint4v*>(st + xt_off + ch * 2);
            const uint4v xp = *reinterpret_cast<const uint4v*>(st + xp_off + ch * 2);
            half8 wo[4];
#pragma unroll
            for (int nb = 0; nb < 4; ++nb)
                wo[nb] = *reinterpret_cast<const half8*>(st + kOffWo + (16 * nb + l16) * kXRowB + ch * 2);
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const half8 bd = *reinterpret_cast<const half8*>(st + kOffBd + (row0 + 4 * half) * kBdRow + 16 * g4);
                const float4 lam = *reinterpret_cast<const float4*>(st + kOffVec + (ch + 4 * half) * 4);
                // mix[e] = lambda_d + sum_k B_d[k][channel ch + 4*half + e] p[token][k], for this lane's token
                const float4v mix = __builtin_amdgcn_mfma_f32_16x16x32_f16(bd, pt, float4v{lam.x, lam.y, lam.z, lam.w}, 0, 0, 0);
                uint2v z;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const unsigned t = xt[2 * half + i], q = xp[2 * half + i];
                    const float c0 = lo_f(t), c1 = hi_f(t);
                    z[i] = pack_h2f(__builtin_fmaf(lo_f(q) - c0, mix[2 * i], c0), __builtin_fmaf(hi_f(q) - c1, mix[2 * i + 1], c1));
                }
                const half4 zh = __builtin_bit_cast(half4, z);
#pragma unroll
                for (int nb = 0; nb < 4; ++nb) {
                    // A operand: A_omega columns 16nb + l16, this block's four channels; B operand: z of token l16
                    const half4 w4 = half ? __builtin_shufflevector(wo[nb], wo[nb], 4, 5, 6, 7)
                                          : __builtin_shufflevector(wo[nb], wo[nb], 0, 1, 2, 3);
                    yacc[nb] = __builtin_amdgcn_mfma_f32_16x16x16f16(w4, zh, yacc[nb], 0, 0, 0);
                }
            }
        }
    };
    auto step_of = [&](int step) {
        const char* st = lds + (step & 1) * kStageBytes;
        if (step < nchunks) {
            walk1(st);
            if (step == nchunks - 1) {
                // pacc[nb][e] = sum for rank 16nb + 4g4 + e of this lane's token: the order B_d was parked in
                uint4v p;
                p[0] = pack_h2f(fast_tanh(pacc[0][0]), fast_tanh(pacc[0][1]));
                p[1] = pack_h2f(fast_tanh(pacc[0][2]), fast_tanh(pacc[0][3]));
                p[2] = pack_h2f(fast_tanh(pacc[1][0]), fast_tanh(pacc[1][1]));
                p[3] = pack_h2f(fast_tanh(pacc[1][2]), fast_tanh(pacc[1][3]));
                pt = __builtin_bit_cast(half8, p);
            }
        } else {
            walk2(st);
        }
    };

    __syncthreads();                                   // stage of step 0 is in LDS
#pragma clang loop unroll(disable)
    for (int step = 0; step < nsteps; step += 2) {
        step_of(step);
        __syncthreads();
        step_of(step + 1);
        __syncthreads();
    }

    // yacc[nb][e] = pre-activation of output 16nb + 4g4 + e of token trow.  The wave's 16 rows go
    // through its own piece of LDS (free after the last barrier; this wave alone touches it), so that
    // every store instruction writes whole rows: 8 (bf16) or 16 (fp32) lanes of 16 bytes per row.
    constexpr int kYRow = kOuterRank * 4 + 16;                   // fp32 row + pad
    char* mine = lds + w * 16 * kYRow;
#pragma unroll
    for (int nb = 0; nb < 4; ++nb)
        *reinterpret_cast<float4*>(mine + l16 * kYRow + (16 * nb + 4 * g4) * 4) =
            make_float4(fast_tanh(yacc[nb][0]), fast_tanh(yacc[nb][1]), fast_tanh(yacc[nb][2]), fast_tanh(yacc[nb][3]));
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const long long m0 = static_cast<long long>(b) * a.T + t0 + 16 * w;   // the wave's first token
    if constexpr (kOutF32) {
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int row = 4 * p + (lane >> 4), c4 = 4 * (lane & 15);
            if (16 * w + row < ntok)
                *reinterpret_cast<float4*>(static_cast<float*>(a.y) + (m0 + row) * kOuterRank + c4) =
                    *reinterpret_cast<const float4*>(mine + row * kYRow + c4 * 4);
        }
    } else {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int row = 8 * p + (lane >> 3), c8 = 8 * (lane & 7);
            if (16 * w + row < ntok) {
                typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
                typedef float float2v __attribute__((ext_vector_type(2)));
                const float4 lo = *reinterpret_cast<const float4*>(mine + row * kYRow + c8 * 4);
                const float4 hi = *reinterpret_cast<const float4*>(mine + row * kYRow + c8 * 4 + 16);
                const uint4v q = {__builtin_bit_cast(unsigned, __builtin_convertvector(float2v{lo.x, lo.y}, bf16x2)),
                                  __builtin_bit_cast(unsigned, __builtin_convertvector(float2v{lo.z, lo.w}, bf16x2)),
                                  __builtin_bit_cast(unsigned, __builtin_convertvector(float2v{hi.x, hi.y}, bf16x2)),
                                  __builtin_bit_cast(unsigned, __builtin_convertvector(float2v{hi.z, hi.w}, bf16x2))};
                *reinterpret_cast<uint4v*>(static_cast<unsigned short*>(a.y) + (m0 + row) * kOuterRank + c8) = q;
            }
        }
    }
}

template <bool kOutF32>
__global__ __launch_bounds__(kDiThreads) void decay_input_kernel(DiArgs a) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = blockIdx.x / a.tiles_per_seq;
    const int t0 = (blockIdx.x - b * a.tiles_per_seq) * kTokens;
    const int left = a.T - t0;
    const int ntok = left < kTokens ? left : kTokens;
    const int nsteps = 2 * (a.D / kStepCh);
    // both roles pass 1 + nsteps barriers
    if (wave >= kWorkerWaves) {
        __builtin_amdgcn_s_setprio(2);
        di_loader(a, lds, tid - 64 * kWorkerWaves, b, t0, ntok, nsteps, static_cast<int>((blockIdx.x * 3u) % (a.D / kStepCh)));
    } else {
        __builtin_amdgcn_s_setprio(1);
        di_worker<kOutF32>(a, lds, tid & 63, wave, b, t0, ntok, nsteps);
    }
}

// ------------------------------------------------------------------------------------------
// The contraction split over the waves, for fewer tokens than fill the chip with the tiles above
// ------------------------------------------------------------------------------------------
// A workgroup owns 16 kTB consecutive rows of the flattened [B * T] tokens (so sequences of a token or two share a
// tile) and its waves take the 32-channel blocks of D in turn; the partial sums of q A_d and of z A_omega meet
// through LDS, once each.  No barrier and no shared stage inside the walks: a wave brings its block's x rows and weight
// slices in whole 64-byte pieces straight into a piece of LDS of its own (loads that bypass the registers), reads them from there as
// operands, and asks for what comes next in the places that these have left: the weights one block ahead, x two.  A token's
// predecessor is an LDS row as well: the row above it, or the carried row where a sequence starts.
// What bounds it.  64 rows: walk 1 streams x at 5.1 TB/s, the rate of a large copy; walk 2 reads it again from the last-level cache, as
// long as its conversions and interpolations keep the vector ALUs; together 24 of 34 us at 16 384 tokens and D = 2048.  16 rows: what
// one compute unit takes in of the weights (18 bytes a clock), and both exchanges, 1.5 us each.  Through registers and LDS stores, with
// one block ahead of both, a kernel of more code: 16 384 tokens x 2048 35.3 -> 33.6 us, 33 792 x 4096 169 -> 157, 24 x 2048 12.2 -> 11.0, 24 x
// 768 7.05 -> 6.3, 1000 x 128 4.7 -> 4.1, 6000 x 1024 11.8 -> 10.7.  One place more for weights and x: 24 x 2048 12.0, 6000 x 1024 11.4, 16 384 x
// 768 15.1 -> 15.5: short calls pay for every line of code that they pass once.  Straight operand loads from global memory
// (sixteen lines per quarter wave) took 26.4 us where the register form took 16.6, bf16 weights with the other operand as two bf16
// values the same time, six waves instead of twelve 17.0, 64 rows with four waves, two workgroups per compute unit, 36 instead of 31
// (24 sequences of one token; 16 384 tokens; D = 2048).
//
// With few tiles kGroups workgroups share a tile: each forms z from all of A_d and B_d, and 64 / kGroups of its outputs,
// so that what a compute unit takes in and passes through its LDS is A_omega's part less (D = 2048: 512 -> 320 KB of weights at four
// groups; 24 tokens 16.7 -> 14.0 us when this was added).  An output's sums are the same ones in the same order.
template <int kTB, int kSplitWaves, int kGroups>
struct SplitTile {
    static constexpr int kCols = kOuterRank / kGroups;   // columns of A_omega, outputs of a token, of this workgroup
    static constexpr int kRows = 16 * kTB;
    static constexpr int kWaves = kSplitWaves;
    static constexpr int kThreads = 64 * kWaves;
    static constexpr int kCarry = kTB == 1 ? 16 : 1;     // rows of a tile that can start a sequence (kTB > 1: T >= kRows)
    // A block's x in LDS: the tile's rows (32 channels, 64 bytes each), the row before the tile, mu_x or lambda_d
    // (128 bytes), one carried row; kTB == 1: sixteen carried rows behind them.
    static constexpr int kOffP = 1024 * kTB, kOffV = kOffP + 64, kOffC1 = kOffV + 128, kOffC = kOffP + 256;
    static constexpr int kXBytes = kOffC + (kCarry > 1 ? 1024 : 0);
    static constexpr int kXLoads = kTB + 1;              // (and one for the carried rows of kTB == 1)
    // its weights: A_d (32 columns of 64 bytes), or B_d (32 channels of 64 bytes) and A_omega (kCols columns)
    static constexpr int kWBytes1 = 2048, kWBytes2 = 2048 + 64 * kCols;
    // a wave's piece: two places for x, one for weights
    static constexpr int kPiece1 = 2 * kXBytes + kWBytes1;
    // values of the exchanged sums that a thread adds up: few, where the rows are, so that most waves take part (16 rows 0.25 us faster
    // with two than with four; 64 rows 0.1 slower)
    static constexpr int kSum = kTB == 4 ? 4 : 2;
    static constexpr int kPRow = kInnerRank + 4;         // row strides (floats) of the waves' partial sums
    static constexpr int kYRow = kCols + 4;
    static constexpr int kPtRow = kInnerRank * 2 + 16;   // row stride (bytes) of tanh(q A_d)
    // Walk 2's first block is on its way while the waves' partial sums of walk 1 meet, so it lies behind these; the other place
    // for x lies where they were.
    static constexpr int kPPart = kWaves * kRows * kPRow * 4;
    static constexpr int kYPart = kWaves * kRows * kYRow * 4;
    static constexpr int kFirst2 = kXBytes + kWBytes2;                       // a wave's first block of walk 2
    static constexpr int kMeet = kPPart > kWaves * kXBytes ? kPPart : kWaves * kXBytes;
    static constexpr int kWalk1 = kWaves * kPiece1, kWalk2 = kMeet + kWaves * kFirst2;
    static constexpr int kMost = kWalk1 > kWalk2 ? kWalk1 : kWalk2;
    static constexpr int kZero = kMost > kYPart ? kMost : kYPart;            // 64 bytes of zeros a wave
    static constexpr int kPtOff = kZero + 64 * kWaves;
    static constexpr int kLds = kPtOff + kRows * kPtRow;
    static_assert(kLds <= 160 * 1024, "LDS budget");
};

__device__ __forceinline__ void wait_lds() {             // the wave's own LDS reads and writes
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(15 | 3 << 14 | 7 << 4);
    __builtin_amdgcn_sched_barrier(0);
}
__device__ __forceinline__ void lds_barrier() {          // all waves; loads into LDS stay on their way
    wait_lds();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
}

template <int kTB, int kSplitWaves, bool kOutF32, int kGroups>
__global__ __launch_bounds__(64 * kSplitWaves) void decay_input_split_kernel(DiArgs a) {
    using TL = SplitTile<kTB, kSplitWaves, kGroups>;
    constexpr int kNB = TL::kCols / 16, kW = TL::kWaves;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const long long M = static_cast<long long>(a.B) * a.T;
    const unsigned tile = kGroups == 1 ? blockIdx.x : blockIdx.x / kGroups, group = kGroups == 1 ? 0 : blockIdx.x % kGroups;
    const long long m0 = static_cast<long long>(tile) * TL::kRows;
    const int rows = M - m0 < TL::kRows ? static_cast<int>(M - m0) : TL::kRows;
    const int row_bytes = a.D * 2;
    const int nkb = a.D / 32;
    const int mine = wave < nkb ? (nkb - 1 - wave) / kW + 1 : 0;      // this wave's blocks: wave, wave + kW, ...
    // sequence of the tile's first row (fewer than 2^32 tokens: a row has at least 256 bytes)
    const unsigned T = static_cast<unsigned>(a.T);
    const int b0 = __builtin_amdgcn_readfirstlane(static_cast<int>(static_cast<unsigned>(m0) / T));
    const unsigned t0 = static_cast<unsigned>(m0) - static_cast<unsigned>(b0) * T;
    const int first_start = t0 == 0 ? 0 : 1;                   // first sequence, counted from b0, whose start can lie in the tile
    const bool has_start = t0 == 0 || t0 + rows > T;           // some row starts a sequence

    // Global loads go by rows, four lanes to the 64 bytes of a row's 32 channels (sixteen different lines per
    // quarter wave, as the operand layout would have it, cost four times as much in the L1's tag lookups), straight into LDS, where lane
    // i's 16 bytes lie 16 i behind the wave's address.  Rows lie 64 bytes apart there, their 16-byte granules XOR-ed by
    // bits 2 and 3 of the row (B_d: 3 and 4), so that both the lanes' reads of sixteen rows, at one granule each, and the loads take every
    // bank once: lane i asks for the granule that belongs in its place.
    const int lr = lane >> 2, lp = 16 * ((lane & 3) ^ ((lane >> 4) & 3));
    typedef __attribute__((address_space(3))) char* lds_ptr;
    auto load = [&](const char* base, int bytes, int voff, int soff, int to) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), 0, bytes, 0x00020000),
                                                 (lds_ptr)(lds + to), 16, voff, soff, 0, 0);
    };
    const char* x_base = a.x + m0 * row_bytes;
    const int x_bytes = rows * row_bytes;
    int x_voff[kTB];                                           // rows past the tile's end: the last one again, whose result is not stored
#pragma unroll
    for (int tb = 0; tb < kTB; ++tb) x_voff[tb] = (16 * tb + lr < rows ? 16 * tb + lr : rows - 1) * row_bytes + lp;
    const int w_voff = lr * row_bytes + lp, w_pass = 16 * row_bytes;   // columns of A_d, A_omega
    const int b_voff = lr * 64 + 16 * ((lane & 3) ^ (lane >> 5));      // channels of B_d; the second pass: granule ^ 2

    // The row before the tile, the vector and the carried row come with one load of sixteen lanes with addresses of their own (a
    // row that is not there is not asked for below: its reads go to the zeros).
    const bool has_before = t0 > 0;
    const int c0 = b0 + first_start;                           // carried rows of the sequences that start in the tile
    const bool has_carry = a.x_prev && has_start && c0 < a.B;
    const char* misc = lane < 4 ? x_base - (has_before ? row_bytes : 0) + 16 * lane
                                : a.x_prev && lane >= 12 ? a.x_prev + static_cast<long long>(has_carry ? c0 : 0) * row_bytes + 16 * (lane - 12) : a.x;
    const bool misc_x = lane < 4 || lane >= 12;
    const int c_rows = a.B - c0 < TL::kCarry ? a.B - c0 : TL::kCarry;
    const int c_voff = (lr < c_rows ? lr : c_rows - 1) * row_bytes + lp;

    auto fetch_x = [&](int kb, const char* vec, int to) {
        const int soff = kb * 64;
#pragma unroll
        for (int tb = 0; tb < kTB; ++tb) load(x_base, x_bytes, x_voff[tb], soff, to + 1024 * tb);
        if (lane < 16) {
            const char* from = misc_x ? misc + soff : vec + 2 * soff + 16 * (lane - 4);
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)from, (lds_ptr)(lds + to + TL::kOffP), 16, 0, 0);
        }
        if constexpr (TL::kCarry > 1)
            if (has_carry) load(a.x_prev + static_cast<long long>(c0) * row_bytes, c_rows * row_bytes, c_voff, soff, to + TL::kOffC);
    };
    auto fetch1 = [&](int kb, int to) {
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) load(a.a_d, kInnerRank * row_bytes, w_voff + nb * w_pass, kb * 64, to + 1024 * nb);
    };
    const char* omega = a.a_omega + static_cast<long long>(group) * TL::kCols * row_bytes;
    auto fetch2 = [&](int kb, int to) {
#pragma unroll
        for (int i = 0; i < 2; ++i) load(a.b_d, a.D * kInnerRank * 2, (b_voff ^ 32 * i) + 1024 * i, kb * 2048, to + 1024 * i);
#pragma unroll
        for (int nb = 0; nb < kNB; ++nb) load(omega, TL::kCols * row_bytes, w_voff + nb * w_pass, kb * 64, to + 2048 + 1024 * nb);
    };
    // A walk: trip i reads the operands of this wave's i-th block from LDS, asks for the weights of block i + 1 and the x of block i + 2 in
    // the places that these have left, and computes.
    const int piece = wave * TL::kPiece1;
    auto ask_w1 = [&](int i) { if (i < mine) fetch1(wave + i * kW, piece + 2 * TL::kXBytes); };
    auto ask_x1 = [&](int i) { if (i < mine) fetch_x(wave + i * kW, a.mu_x, piece + (i & 1) * TL::kXBytes); };
    ask_x1(0);
    ask_w1(0);
    ask_x1(1);

    auto row_off = [](int row, int granule) { return 64 * row + 16 * (granule ^ ((row >> 2) & 3)); };

    const int zeros = TL::kZero + 64 * wave;
    if (lane < 4) *reinterpret_cast<uint4v*>(lds + zeros + 16 * lane) = uint4v{0u, 0u, 0u, 0u};
    // LDS places of this lane's tokens, within a block's x, and of their predecessors (kInZeros: none)
    constexpr int kInZeros = -1;
    int prev_off[kTB];
#pragma unroll
    for (int tb = 0; tb < kTB; ++tb) {
        // (kTB > 1: T >= kRows, so that at most one sequence starts in the tile)
        const unsigned row = 16 * tb + l16, db = kTB == 1 ? (t0 + row) / T : t0 + row >= T ? 1 : 0;
        const bool start = t0 + row == db * T;
        prev_off[tb] = row > 0 ? row_off(row - 1, g4) : TL::kOffP + 16 * g4;
        if (start) {
            // (a row past the end of the tile may find a sequence past the carried rows: its result is not stored)
            const int slot = static_cast<int>(db) - first_start;
            prev_off[tb] = !has_carry || slot >= c_rows ? kInZeros : TL::kCarry > 1 ? TL::kOffC + row_off(slot, g4) : TL::kOffC1 + 16 * g4;
        }
    }
    const int cur0 = row_off(l16, g4);                         // a block's rows 16 tb + l16, and columns 16 nb + l16 of its weights
    auto read_u4 = [&](int off) { return *reinterpret_cast<const uint4v*>(lds + off); };
    auto read_f4 = [&](int off) { return *reinterpret_cast<const float4v*>(lds + off); };
    auto interpolate = [](unsigned cur, unsigned prev, float w0, float w1) {   // two channels, fp32, rounded to fp16
        const float c0 = lo_f(cur), c1 = hi_f(cur);
        return pack_h2f(__builtin_fmaf(lo_f(prev) - c0, w0, c0), __builtin_fmaf(hi_f(prev) - c1, w1, c1));
    };
    struct X {
        uint4v cur[kTB], prev[kTB];
        float4v vec[2];
    };
    auto read_x = [&](X& s, int at) {
#pragma unroll
        for (int tb = 0; tb < kTB; ++tb) {
            s.cur[tb] = read_u4(at + cur0 + 1024 * tb);
            s.prev[tb] = read_u4(prev_off[tb] == kInZeros ? zeros : at + prev_off[tb]);
        }
        s.vec[0] = read_f4(at + TL::kOffV + 32 * g4);
        s.vec[1] = read_f4(at + TL::kOffV + 32 * g4 + 16);
    };
    // walk 1: this wave's share of q A_d
    float4v pacc[kTB][2];
#pragma unroll
    for (int tb = 0; tb < kTB; ++tb) pacc[tb][0] = pacc[tb][1] = float4v{0.f, 0.f, 0.f, 0.f};
    auto wait_block = [&](int i) {                             // only the x of block i + 1 is behind block i's weights
        if (i + 1 >= mine) wait_loads<0>();
        else if (TL::kCarry > 1 && has_carry) wait_loads<TL::kXLoads + 1>();
        else wait_loads<TL::kXLoads>();
    };
#pragma clang loop unroll(disable)
    for (int i = 0; i < mine; ++i) {
        wait_block(i);
        X x;
        uint4v wgt[2];
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) wgt[nb] = read_u4(piece + 2 * TL::kXBytes + cur0 + 1024 * nb);
        read_x(x, piece + (i & 1) * TL::kXBytes);
        wait_lds();                                            // the operands are in registers: their places may be written again
        ask_w1(i + 1);
        ask_x1(i + 2);
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) wgt[nb] = bf16x8_to_f16x8(wgt[nb]);
#pragma unroll
        for (int tb = 0; tb < kTB; ++tb) {
            uint4v q;
#pragma unroll
            for (int e = 0; e < 4; ++e) q[e] = interpolate(x.cur[tb][e], x.prev[tb][e], x.vec[e >> 1][2 * (e & 1)], x.vec[e >> 1][2 * (e & 1) + 1]);
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)
                pacc[tb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, wgt[nb]), __builtin_bit_cast(half8, q), pacc[tb][nb], 0, 0, 0);
        }
    }

    // walk 2, from the blocks most recently brought into the caches down; its first block does not wait for the exchange
    const int first2 = TL::kMeet + wave * TL::kFirst2;
    auto x_place = [&](int i) { return i & 1 ? wave * TL::kXBytes : first2; };
    auto ask_w2 = [&](int i) { if (i < mine) fetch2(wave + (mine - 1 - i) * kW, first2 + TL::kXBytes); };
    auto ask_x2 = [&](int i) { if (i < mine) fetch_x(wave + (mine - 1 - i) * kW, a.lambda_d, x_place(i)); };

    // the waves' shares of q A_d meet; p = tanh of the sum, as fp16
    float* part = reinterpret_cast<float*>(lds);
    lds_barrier();                                             // every wave is done with its piece
    ask_x2(0);
    ask_w2(0);
#pragma unroll
    for (int tb = 0; tb < kTB; ++tb)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
            *reinterpret_cast<float4v*>(part + (wave * TL::kRows + 16 * tb + l16) * TL::kPRow + 16 * nb + 4 * g4) = pacc[tb][nb];
    lds_barrier();
    constexpr int kSum = TL::kSum;
    typedef float floats __attribute__((ext_vector_type(kSum)));
    for (int i = tid; i < TL::kRows * (kInnerRank / kSum); i += TL::kThreads) {
        const int row = i / (kInnerRank / kSum), c = kSum * (i % (kInnerRank / kSum));
        floats sum = 0.f;
#pragma unroll
        for (int w = 0; w < TL::kWaves; ++w)
            sum += *reinterpret_cast<const floats*>(part + (w * TL::kRows + row) * TL::kPRow + c);
#pragma unroll
        for (int e = 0; e < kSum; e += 2)
            *reinterpret_cast<unsigned*>(lds + TL::kPtOff + row * TL::kPtRow + 2 * (c + e)) = pack_h2f(fast_tanh(sum[e]), fast_tanh(sum[e + 1]));
    }
    lds_barrier();
    ask_x2(1);
    half8 pt[kTB];                                             // ranks 8*g4 .. +7 of this lane's tokens
#pragma unroll
    for (int tb = 0; tb < kTB; ++tb)
        pt[tb] = *reinterpret_cast<const half8*>(lds + TL::kPtOff + (16 * tb + l16) * TL::kPtRow + 16 * g4);

    // this wave's share of z A_omega
    float4v yacc[kTB][kNB];
#pragma unroll
    for (int tb = 0; tb < kTB; ++tb)
#pragma unroll
        for (int nb = 0; nb < kNB; ++nb) yacc[tb][nb] = float4v{0.f, 0.f, 0.f, 0.f};
    // Which channel sits in which row of the B_d^T operand is free as long as z and A_omega agree: with row m of
    // block `half` holding channel 8*(m>>2) + 4*half + (m&3) a lane's results are its own channels 8*g4 .. +7
    int bd_off[2];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        const int ch = 8 * (l16 >> 2) + 4 * half + (l16 & 3);
        bd_off[half] = 64 * ch + 16 * (g4 ^ ((ch >> 3) & 3));
    }
#pragma clang loop unroll(disable)
    for (int i = 0; i < mine; ++i) {
        wait_block(i);
        const int wat = first2 + TL::kXBytes;
        X x;
        uint4v bd[2], wo[kNB];
#pragma unroll
        for (int half = 0; half < 2; ++half) bd[half] = read_u4(wat + bd_off[half]);
#pragma unroll
        for (int nb = 0; nb < kNB; ++nb) wo[nb] = read_u4(wat + 2048 + cur0 + 1024 * nb);
        read_x(x, x_place(i));
        wait_lds();                                            // the operands are in registers: their places may be written again
        ask_w2(i + 1);
        ask_x2(i + 2);
#pragma unroll
        for (int half = 0; half < 2; ++half) bd[half] = bf16x8_to_f16x8(bd[half]);
#pragma unroll
        for (int nb = 0; nb < kNB; ++nb) wo[nb] = bf16x8_to_f16x8(wo[nb]);
#pragma unroll
        for (int tb = 0; tb < kTB; ++tb) {
            uint4v z;
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                // mix[e] = lambda_d + sum_k B_d[k][channel 8*g4 + 4*half + e] p[token][k]
                const float4v mix = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, bd[half]), pt[tb], x.vec[half], 0, 0, 0);
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    z[2 * half + e] = interpolate(x.cur[tb][2 * half + e], x.prev[tb][2 * half + e], mix[2 * e], mix[2 * e + 1]);
            }
#pragma unroll
            for (int nb = 0; nb < kNB; ++nb)
                yacc[tb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, wo[nb]), __builtin_bit_cast(half8, z), yacc[tb][nb], 0, 0, 0);
        }
    }

    lds_barrier();                                             // every wave is done with its piece
#pragma unroll
    for (int tb = 0; tb < kTB; ++tb)
#pragma unroll
        for (int nb = 0; nb < kNB; ++nb)
            *reinterpret_cast<float4v*>(part + (wave * TL::kRows + 16 * tb + l16) * TL::kYRow + 16 * nb + 4 * g4) = yacc[tb][nb];
    __syncthreads();
    for (int i = tid; i < TL::kRows * (TL::kCols / kSum); i += TL::kThreads) {
        const int row = i / (TL::kCols / kSum), c = kSum * (i % (TL::kCols / kSum));
        floats sum = 0.f;
#pragma unroll
        for (int w = 0; w < TL::kWaves; ++w)
            sum += *reinterpret_cast<const floats*>(part + (w * TL::kRows + row) * TL::kYRow + c);
        if (row < rows) {
            const long long e = (m0 + row) * kOuterRank + group * TL::kCols + c;
#pragma unroll
            for (int i2 = 0; i2 < kSum; ++i2) sum[i2] = fast_tanh(sum[i2]);
            if constexpr (kOutF32) {
                *reinterpret_cast<floats*>(static_cast<float*>(a.y) + e) = sum;
            } else {
                typedef __bf16 bf16s __attribute__((ext_vector_type(kSum)));
                *reinterpret_cast<bf16s*>(static_cast<unsigned short*>(a.y) + e) = __builtin_convertvector(sum, bf16s);
            }
        }
    }
}

}  // namespace

namespace {

template <int kTB, int kSplitWaves, bool kOutF32, int kGroups = 1>
hipError_t launch_split(const DiArgs& a, hipStream_t stream) {
    using TL = SplitTile<kTB, kSplitWaves, kGroups>;
    const long long M = static_cast<long long>(a.B) * a.T;
    hipLaunchKernelGGL((decay_input_split_kernel<kTB, kSplitWaves, kOutF32, kGroups>), dim3(static_cast<unsigned>((M + TL::kRows - 1) / TL::kRows * kGroups)),
                       dim3(TL::kThreads), TL::kLds, stream, a);
    return hipGetLastError();
}

template <bool kOutF32>
hipError_t raise_lds_limits() {
    hipError_t err = set_lds_limit(&decay_input_split_kernel<1, 12, kOutF32, 1>, SplitTile<1, 12, 1>::kLds);
    if (err == hipSuccess) err = set_lds_limit(&decay_input_split_kernel<1, 12, kOutF32, 2>, SplitTile<1, 12, 2>::kLds);
    if (err == hipSuccess) err = set_lds_limit(&decay_input_split_kernel<1, 12, kOutF32, 4>, SplitTile<1, 12, 4>::kLds);
    if (err == hipSuccess) err = set_lds_limit(&decay_input_split_kernel<2, 8, kOutF32, 1>, SplitTile<2, 8, 1>::kLds);
    if (err == hipSuccess) err = set_lds_limit(&decay_input_split_kernel<4, 8, kOutF32, 1>, SplitTile<4, 8, 1>::kLds);
    if (err == hipSuccess) err = set_lds_limit(&decay_input_kernel<kOutF32>, kDiLds);
    return err;
}

}  // namespace

hipError_t launch_decay_input(int B, int T, int D, const void* x, const void* x_prev, const float* mu_x,
                              const float* lambda_d, const void* a_d, const void* b_d, const void* a_omega, void* y,
                              bool out_f32, hipStream_t stream) {
    DiArgs a;
    a.B = B;
    a.T = T;
    a.D = D;
    a.tiles_per_seq = (T + kTokens - 1) / kTokens;
    a.x = static_cast<const char*>(x);
    a.x_prev = static_cast<const char*>(x_prev);
    a.mu_x = reinterpret_cast<const char*>(mu_x);
    a.lambda_d = reinterpret_cast<const char*>(lambda_d);
    a.a_d = static_cast<const char*>(a_d);
    a.b_d = static_cast<const char*>(b_d);
    a.a_omega = static_cast<const char*>(a_omega);
    a.y = y;
    struct Tag {};
    const hipError_t err = once_per_device<Tag>([] {
        const hipError_t e = raise_lds_limits<false>();
        return e == hipSuccess ? raise_lds_limits<true>() : e;
    });
    if (err != hipSuccess) return err;
    // Which kernel: rounds of one workgroup per compute unit, times what a round takes.  A 128-token workgroup
    // takes as long with one token as with 128 and serves one sequence, so it is the better one only when it fills the
    // chip; the split tiles take rows of any sequences, but every tile takes all weights and the launch, the two exchanges
    // and the last reduction weigh more the narrower the model is.  Nanoseconds a round, a fixed part and one per 128
    // channels, fitted to a full round at D = 128, 256, 768, 1024, 2048, 4096: 128 tokens 7.0, 9.6, 20.2, 25.4, 46.4, 88 us; split 64 rows
    // 7.1, 8.3, 13.5, 16.1, 27.2, 52, 32 rows 5.1, 6.0, 9.2, 10.7, 17.4, 29 to 37, 16 rows 4.5, 5.2, 7.5, 8.3, 13.4, 22.7.  Where a line lies,
    // measured on both sides: 128 tokens : 16 rows: D = 128 24 x 1 token 6.7 : 4.0, 1000 x 20 24.4 : 18.0, D = 256 1000 x 20 34.7 : 21.3, D =
    // 2048 24 x 1 46 : 10.1; 16 : 32 rows: 4000 tokens 4.6 : 5.0, 8.9 : 10.4, 13.9 : 16.3 and 4200 7.4 : 5.0, 15.3 : 10.4, 24.5 : 16.3 (D = 128,
    // 1024, 2048); 32 : 64 rows: 8192 tokens 10.7 : 15.5, 17.5 : 25.1 and 8320 19.2 : 15.6, 30.7 : 25.1 (1024, 2048); 128 tokens : 32 rows:
    // 1000 x 40 24.9 : 20.2 (128), 35.2 : 24.5 (256), 500 x 50 13.3 : 16.3 (128), 28.9 : 26.1 (512, the rule errs), 39.1 : 32.7 (768), 49.6 : 38.9
    // (1024); 128 tokens : 64 rows: 16 384 tokens 7.4 : 7.1 (128, the rule errs), 10.0 : 8.3 (256), 46.7 : 27.2 (2048); 20 000 26.0 : 30.1 (1024),
    // 47 : 50 (2048), 33 792 13.9 : 18.4 (128), 19.4 : 21.7 (256), 40.1 : 39.1 (768, the rule errs), 50.4 : 46.8 (1024), 92.6 : 76.5 (2048).
    const long long cus = compute_units(), rows = static_cast<long long>(B) * T, blocks = D / 128;
    auto rounds = [&](long long groups) { return (groups + cus - 1) / cus; };
    const long long whole = (4300 + 2640 * blocks) * rounds(static_cast<long long>(B) * a.tiles_per_seq);
    const long long r64 = T >= 64 ? (5600 + 1360 * blocks) * rounds((rows + 63) / 64) : whole;
    const long long r32 = T >= 32 ? (4400 + 810 * blocks) * rounds((rows + 31) / 32) : whole;
    const long long r16 = (3900 + 585 * blocks) * rounds((rows + 15) / 16);
    if (r16 < whole && r16 <= r32 && r16 <= r64) {
        // A tile's outputs over four or two workgroups while these still fit the chip once.  One, two, four of them, us: D = 128, 256
        // x 1 token 4.4, 4.2, 4.1; D = 768, 24 x 1 7.1, 6.5, 6.3; D = 2048, 24 x 1 12.1, 10.7, 10.1; 1000 tokens 12.0, 10.7, 10.8; 2000 12.2,
        // 11.2; 4000 13.4, 20.6 (a second round); D = 4096, 24 x 1 19.2, 16.9, 15.8.
        const long long tiles = (rows + 15) / 16;
        if (4 * tiles <= cus) return out_f32 ? launch_split<1, 12, true, 4>(a, stream) : launch_split<1, 12, false, 4>(a, stream);
        if (2 * tiles <= cus) return out_f32 ? launch_split<1, 12, true, 2>(a, stream) : launch_split<1, 12, false, 2>(a, stream);
        return out_f32 ? launch_split<1, 12, true>(a, stream) : launch_split<1, 12, false>(a, stream);
    }
    if (r32 < whole && r32 <= r64) return out_f32 ? launch_split<2, 8, true>(a, stream) : launch_split<2, 8, false>(a, stream);
    if (r64 < whole) return out_f32 ? launch_split<4, 8, true>(a, stream) : launch_split<4, 8, false>(a, stream);
    const dim3 grid(static_cast<unsigned>(static_cast<long long>(B) * a.tiles_per_seq));
    if (out_f32)
        hipLaunchKernelGGL(decay_input_kernel<true>, grid, dim3(kDiThreads), kDiLds, stream, a);
    else
        hipLaunchKernelGGL(decay_input_kernel<false>, grid, dim3(kDiThreads), kDiLds, stream, a);
    return hipGetLastError();
}

}  // namespace wkv6

// Internal launch interface between the C ABI (wkv6_api.hip) and the kernels.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>

namespace wkv6 {

constexpr int kHeadSize = 64;   // N: the only head size the kernels are built for

// Where the token split keeps what a segment hands over: the [64][64] fp32 state and, in the row behind
// it, the 64 total decays.  A row is two halves of 32 values.  Byte strides; either a workspace (rows of
// 256 bytes) or the first rows of the segment in `out` itself (which the last pass overwrites): a bf16 token
// row of a head holds half a state row, an fp32 one a whole.
struct SegPlace {
    char* base = nullptr;
    long long batch = 0, seg = 0, head = 0;
    int row = 0, half = 0;
};

struct Args {
    int B, T, H;              // T: tokens of a sequence
    const void* r;
    const void* k;
    const void* v;
    const void* x;
    const float* u;           // Finch bonus [H][N]; unused in the Finch-C2 form
    bool finch_c2;            // false: Finch form (bonus u).  true: Finch-C2 form: k is the key before its
                              // (1 - w) factor, no bonus, and the second value uprime is added to the read-out
    const void* uprime;       // Finch-C2 only: [B][T][H][N] bf16, laid out like out; not read by the
                              // segments' first pass
    const float* state_in;    // may be nullptr (zero state)
    void* out;
    float* state_out;         // may be nullptr (not written)
    long long batch_stride;   // elements between consecutive batches of r,k,v,x,out
    // Token-axis segments (chunked kernel only).  Each sequence is cut into `segs` segments of seg_len
    // tokens (a multiple of 32; the last one may be shorter); a workgroup handles one (batch, segment,
    // head), takes its entering state from `place`, and the last segment's writes state_out.  segs == 1:
    // seg_len == T and the plain layout.
    int segs;
    int seg_len;
    SegPlace place;
    float* moments;           // with the LayerNorm partials only: [B][H][T][2] per (batch, head, token): the sum of
                              // the head's N output values and their squared deviations from the
                              // head's own mean (taken before the rounding to bf16)
    // kBf16OutLora / kBf16OutLoraMoments only (x unused): the decay logit is formed in the kernel as
    // d[b][t][h][n] = lambda[h*N+n] + sum_k y[b][t][k] * bw[k][h*N+n], k < 64
    const void* y;            // [B][T][64] bf16
    const float* lambda;      // [H*N] fp32
    const void* bw;           // [64][H*N] bf16
    int unit_stride;          // set by launch_chunked: 0 = one unit per workgroup; otherwise workgroup w
                              // handles units w, w + unit_stride, ... (a multiple of H, segs == 1 only)
};

enum class ChunkedMode { kBf16Out, kF32Out, kBf16OutMoments, kBf16OutLora, kBf16OutLoraMoments };

constexpr int kLoraRank = 64;   // R: the only rank of the decay path the fused kernel is built for

// Token-by-token fp32 kernel; inputs bf16 or fp32 (fp32 inputs: fp32 out, Finch form only);
// with bf16 inputs the output is fp32 or bf16 and a.finch_c2 selects the form.  With a.y the decay logits are formed
// from a.y, a.lambda, a.bw (bf16 in and out) and a.moments, if set, is written (Finch-C2 form).
hipError_t launch_recurrent(const Args& a, bool in_bf16, bool out_bf16, hipStream_t stream);

// Chunked kernel of fp32 tensors (Finch form, fp32 throughout).  Units, to a multiple of eight, in workgroups of kChunkedF32Threads.
constexpr int kChunkedF32Threads = 512;
hipError_t launch_chunked_f32(const Args& a, hipStream_t stream);

// Raises the dynamic LDS limits that launch_chunked_f32 needs, without launching.
hipError_t raise_chunked_f32_limits();

// Chunked matrix-core kernel; inputs bf16, out bf16 or fp32.  kBf16OutMoments: bf16 out
// plus a.moments, Finch-C2 form only.  kBf16OutLora: bf16 out with the decay
// logits formed in the kernel from a.y, a.lambda, a.bw instead of read from a.x (either form);
// kBf16OutLoraMoments: that plus a.moments (Finch-C2 form).
hipError_t launch_chunked(const Args& a, ChunkedMode mode, hipStream_t stream);

// The same, bit for bit, for sequences of at most kChunkTokens tokens; a workgroup of kOneChunkThreads per (batch, head) unit.
constexpr int kChunkTokens = 32, kOneChunkThreads = 256;
hipError_t launch_one_chunk(const Args& a, ChunkedMode mode, hipStream_t stream);

// Raises the dynamic LDS limits that launch_chunked needs for this form and mode, without launching.
hipError_t raise_chunked_limits(const Args& a, ChunkedMode mode);

// The two passes in front of it when a.segs > 1: the local state and total decay of every segment but the
// last, from a zero state (k, v and x, or y, lambda and bw when `lora`), left in a.place; then, in place, the state
// entering every segment (from a.state_in on).
hipError_t launch_segment_states(const Args& a, bool lora, hipStream_t stream);

// Raises the dynamic LDS limits that launch_segment_states needs for any form, without launching.
hipError_t raise_segment_limits();

// GOLD key compression c = x W: x [M][D] bf16, w [D][D/16] bf16, c [M][D/16] bf16 or fp32.
// D must be a multiple of 256 (16 output columns per MFMA block, an even number of 64-channel steps).
hipError_t launch_key_compress(long long M, int D, const void* x, const void* w, void* c, bool out_f32,
                               hipStream_t stream);

// Folds the H per-head (sum, squared deviations) pairs of every token into the token's mean and
// 1/sqrt(variance + eps) over all H*N channels: moments [B][H][T][2] -> mean_rstd [B][T][2].
hipError_t launch_layernorm_finalize(int B, int T, int H, const float* moments, float eps, float* mean_rstd,
                                     hipStream_t stream);

// Applies the token statistics: y = (o - mean) * rstd * gamma + beta; o [tokens][D] bf16, mean_rstd
// [tokens][2], gamma and beta [D] fp32, y [tokens][D] bf16 or fp32.  D must be a multiple of 8.
hipError_t launch_layernorm_apply(long long tokens, int D, const void* o, const float* mean_rstd, const float* gamma,
                                  const float* beta, void* y, bool out_f32, hipStream_t stream);

// Front of the decay path: y = tanh(ddlerp_d(x_t, x_{t-1}) A_omega), x [B][T][D] bf16, x_prev [B][D] bf16 or
// nullptr, mu_x and lambda_d [D] fp32, a_d [32][D], b_d [D][32], a_omega [64][D] bf16, y [B][T][64] bf16
// or fp32.  D must be a multiple of 128.
hipError_t launch_decay_input(int B, int T, int D, const void* x, const void* x_prev, const float* mu_x,
                              const float* lambda_d, const void* a_d, const void* b_d, const void* a_omega, void* y,
                              bool out_f32, hipStream_t stream);

// Whether one launch holds `workgroups` of `threads` each: HIP takes fewer than 2^32 work items in a dimension.
constexpr bool fits_a_launch(long long workgroups, int threads) { return workgroups * threads < 1ll << 32; }

// The current device as an index below 64.  With one visible device there is nothing to ask (a short append of one user, where the
// host bounds the call, checks two flags: 5.12 -> 5.00 us).
inline int device_index() {
    static const bool one = [] {
        int n = 0;
        return hipGetDeviceCount(&n) == hipSuccess && n == 1;
    }();
    int dev = 0;
    if (!one && (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64)) dev = 0;
    return dev;
}

// Runs `f` (returning hipError_t) once per device; a call that fails is tried again by the next one.
// `Tag` makes one flag set per use.
template <typename Tag, typename F>
inline hipError_t once_per_device(F f) {
    static std::atomic<unsigned long long> done{0};
    const unsigned long long bit = 1ull << device_index();
    if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
    const hipError_t err = f();
    if (err == hipSuccess) done.fetch_or(bit, std::memory_order_release);
    return err;
}

// A kernel's dynamic LDS limit.  The attribute belongs to the loaded function on a device, so it is set once per
// device and not at every launch, and it is no stream operation: a process that captures should make its first call to an
// entry point outside the capture.  An entry point whose sizes choose between kernels sets the limits of all of
// them on its first call, so that the size of that call does not matter.
template <typename Kernel>
inline hipError_t set_lds_limit(Kernel kernel, int bytes) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}


// Compute units of the current device (256 on an MI355X), read once per device; 256 if the
// query fails.
inline int compute_units() {
    static std::atomic<int> cached[64];
    const int dev = device_index();
    int n = cached[dev].load(std::memory_order_relaxed);
    if (n <= 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        cached[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

// T == 0: state_out = state_in (or zero).
hipError_t launch_state_passthrough(const Args& a, hipStream_t stream);

}  // namespace wkv6

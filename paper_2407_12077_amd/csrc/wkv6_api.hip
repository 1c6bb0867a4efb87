// C ABI of the WKV6 prefill library: argument validation and dispatch only.
// Every step of the computation runs in the kernels this file launches.
#include "../../include/wkv6.h"
#include "wkv6_launch.h"
#include "wkv6_split_plan.h"

#include <cstdint>
#include <mutex>

namespace {

inline bool misaligned(const void* p) { return (reinterpret_cast<std::uintptr_t>(p) & 15u) != 0; }

enum class Path { kChunked, kRecurrent, kBySize, kF32 };

// Sequences at most this long go to the token-by-token kernel when the caller leaves the
// choice to the library (append / decode shapes): with thousands of (batch, head) units and
// a few tokens each the work is streaming the state once, and the token-by-token kernel does it with fp32
// operands.  (The line was drawn against the chunked kernel, which was level at about 8 tokens with 8192
// units; the one-chunk kernel would be the faster one from 4 tokens on, with fp16 operands.)
constexpr int kRecurrentMaxTokens = 6;

// fp32 tensors: whether the chunked kernel takes the sequences.  It takes whole chunks of 16 tokens, four at a time, and a round to
// fill, the token-by-token kernels blocks of 8 to 32, so the line follows the form that those take at this number of units.  Measured,
// microseconds, token by token : chunked: 24 units 64 tokens 8.9 : 8.6, 80 11.3 : 10.8, 96 11.2 : 11.2, 97 13.5 : 11.5; 32 units 32
// tokens 6.8 : 8.1, 33 9.1 : 8.4; 96 units 32 8.6 : 8.9, 33 11.0 : 9.6; 128 units 24 8.8 : 9.1 with the inputs in the caches, 9.3 : 8.5 without;
// 256 units 24 11.0 : 10.0; 320 units (two rounds of workgroups) 40 17.5 : 18.9, 48 20.1 : 19.2; 512 units 40 20.7 : 21.0, 48 23.8 : 21.8.
// Beyond that both are in rounds, three units to a compute unit token by token, one here.  The fourth round of one is the second of the
// other: 769 units 48 39.6 : 36.5, 65 53.4 : 49.6, 1024 units 48 44.2 : 39.4.  Elsewhere only long sequences and those that just
// fill the four chunks: 513 units 48 26.6 : 27.5, 63 33.6 : 31.7, 72 37.1 : 37.9, 80 40.6 : 38.0; 2048 units 48 75 : 76, 64 95 : 92, 65
// 99 : 106, 80 119 : 116; 4096 units 48 143 : 159, 56 169 : 174, 64 198 : 179, 72 219 : 220, 80 247 : 223.
bool f32_in_chunks(long long units, int T) {
    if (units <= 24) return T >= 97;
    if (units <= 96) return T >= 33;
    if (units <= 256) return T >= 24;
    if (units <= 512 || (units > 768 && units <= 1024)) return T >= 48;
    return T >= 80 || (T > 56 && T <= 64);
}

// Fills in the segments of `p` with their hand-over in the segments' own rows of out.
void split_into_out(wkv6::Args& a, const wkv6::SplitPlan& p, bool out_f32) {
    a.segs = p.segs;
    a.seg_len = p.seg_len;
    const long long elem = out_f32 ? 4 : 2;
    const long long row = static_cast<long long>(a.H) * wkv6::kHeadSize * elem;      // H < 256 here: fits an int
    a.place.base = static_cast<char*>(a.out);
    a.place.batch = a.batch_stride * elem;
    a.place.seg = p.seg_len * row;
    a.place.head = wkv6::kHeadSize * elem;
    a.place.row = static_cast<int>(out_f32 ? row : 2 * row);
    a.place.half = static_cast<int>(out_f32 ? 128 : row);
}

// The passes of a prefill whose Args are complete but for the segments.  Sequences of one chunk go to the kernel that runs several
// units per compute unit and not several chunks of one: at no number of units is it the slower one (figures there), and the bits
// are the same.  More units than a launch has workgroups for (2^24; one token of them without states is 11 GB) stay with the
// other kernel, whose workgroups take several.  The limits of the other kernels behind the entry point are raised all the same.
hipError_t launch_prefill(wkv6::Args& a, wkv6::ChunkedMode mode, bool own_split, hipStream_t s) {
    const bool lora = mode == wkv6::ChunkedMode::kBf16OutLora || mode == wkv6::ChunkedMode::kBf16OutLoraMoments;
    if (own_split) {
        const wkv6::SplitPlan p = wkv6::plan_own_split(a.B, a.T, a.H);
        if (p.segs > 1) split_into_out(a, p, mode == wkv6::ChunkedMode::kF32Out);
    }
    hipError_t err = wkv6::launch_segment_states(a, lora, s);
    if (a.segs == 1 && a.T <= wkv6::kChunkTokens && wkv6::fits_a_launch(static_cast<long long>(a.B) * a.H, wkv6::kOneChunkThreads)) {
        if (err == hipSuccess) err = wkv6::raise_chunked_limits(a, mode);
        return err == hipSuccess ? wkv6::launch_one_chunk(a, mode, s) : err;
    }
    return err == hipSuccess ? wkv6::launch_chunked(a, mode, s) : err;
}

// A call that the token-by-token kernel takes because it is short: its entry point launches the kernels of
// launch_prefill at other sizes, so their limits are raised here as well.
hipError_t launch_short(const wkv6::Args& a, wkv6::ChunkedMode mode, hipStream_t s) {
    hipError_t err = wkv6::raise_segment_limits();
    if (err == hipSuccess) err = wkv6::raise_chunked_limits(a, mode);
    return err == hipSuccess ? wkv6::launch_recurrent(a, true, true, s) : err;
}

// All-fp32 tensors; the limits as in launch_short.
hipError_t launch_f32(const wkv6::Args& a, hipStream_t s) {
    const hipError_t err = wkv6::raise_chunked_f32_limits();
    if (err != hipSuccess) return err;
    const long long units = static_cast<long long>(a.B) * a.H;
    const bool chunked = f32_in_chunks(units, a.T) && wkv6::fits_a_launch(units + 7, wkv6::kChunkedF32Threads);
    return chunked ? wkv6::launch_chunked_f32(a, s) : wkv6::launch_recurrent(a, false, false, s);
}

// `uprime` selects the form: nullptr = Finch (bonus u), otherwise Finch-C2 (u unused, may be null).
int run(int B, int T, int H, int N, const void* r, const void* k, const void* v, const void* x,
        const float* u, const float* state_in, void* out, float* state_out,
        long long batch_stride, bool in_bf16, bool out_f32, Path path, void* stream,
        const void* uprime = nullptr, bool finch_c2 = false, float* moments = nullptr,
        bool want_moments = false, bool own_split = true) {
    if (N != wkv6::kHeadSize) return WKV6_ERR_UNSUPPORTED;
    if (B < 0 || T < 0 || H < 1 || H > 262144) return WKV6_ERR_SHAPE;   // 32-bit row offsets in the kernels
    if (!finch_c2 && !u) return WKV6_ERR_NULL;
    if (B == 0) return WKV6_OK;
    const long long need = static_cast<long long>(T) * H * N;
    if (T > 0) {
        if (!r || !k || !v || !x || !out || (finch_c2 && !uprime)) return WKV6_ERR_NULL;
        if (batch_stride < need) return WKV6_ERR_SHAPE;
        if (misaligned(r) || misaligned(k) || misaligned(v) || misaligned(x) || misaligned(out) ||
            misaligned(uprime))
            return WKV6_ERR_ALIGN;
        if (batch_stride % 8 != 0) return WKV6_ERR_ALIGN;
    }
    if (misaligned(u) || misaligned(state_in) || misaligned(state_out)) return WKV6_ERR_ALIGN;
    if (static_cast<long long>(B) * H > 0x7fffffffLL) return WKV6_ERR_SHAPE;
    if (want_moments && T > 0) {
        if (!moments) return WKV6_ERR_NULL;
        if (misaligned(moments)) return WKV6_ERR_ALIGN;
    }

    wkv6::Args a;
    a.B = B; a.T = T; a.H = H;
    a.r = r; a.k = k; a.v = v; a.x = x; a.u = u;
    a.finch_c2 = finch_c2;
    a.uprime = finch_c2 ? uprime : nullptr;
    a.state_in = state_in; a.out = out; a.state_out = state_out;
    a.batch_stride = batch_stride;
    a.segs = 1; a.seg_len = T; a.unit_stride = 0;
    a.moments = moments;
    a.y = nullptr; a.lambda = nullptr; a.bw = nullptr;

    hipStream_t s = static_cast<hipStream_t>(stream);
    hipError_t err;
    if (T == 0)
        err = wkv6::launch_state_passthrough(a, s);
    else if (path == Path::kF32)
        err = launch_f32(a, s);
    else if (path == Path::kRecurrent)
        err = wkv6::launch_recurrent(a, in_bf16, in_bf16 && !out_f32, s);
    else if (path == Path::kBySize && T <= kRecurrentMaxTokens)          // bf16 in and out
        err = launch_short(a, wkv6::ChunkedMode::kBf16Out, s);
    else if (want_moments)
        err = launch_prefill(a, wkv6::ChunkedMode::kBf16OutMoments, own_split, s);
    else
        err = launch_prefill(a, out_f32 ? wkv6::ChunkedMode::kF32Out : wkv6::ChunkedMode::kBf16Out, own_split, s);
    return err == hipSuccess ? WKV6_OK : WKV6_ERR_LAUNCH;
}

}  // namespace

extern "C" {

int wkv6_prefill_bf16(int B, int T, int H, int N, const void* r, const void* k, const void* v,
                      const void* x, const float* u, const float* state_in, void* out,
                      float* state_out, void* stream) {
    return run(B, T, H, N, r, k, v, x, u, state_in, out, state_out,
               static_cast<long long>(T) * H * N, true, false, Path::kChunked, stream);
}

int wkv6_prefill_bf16_f32out(int B, int T, int H, int N, const void* r, const void* k,
                             const void* v, const void* x, const float* u, const float* state_in,
                             float* out, float* state_out, void* stream) {
    return run(B, T, H, N, r, k, v, x, u, state_in, out, state_out,
               static_cast<long long>(T) * H * N, true, true, Path::kChunked, stream);
}

int wkv6_prefill_bf16_strided(int B, int T, int H, int N, const void* r, const void* k,
                              const void* v, const void* x, const float* u, const float* state_in,
                              void* out, float* state_out, long long batch_stride, int out_dtype,
                              void* stream) {
    if (out_dtype != WKV6_DTYPE_BF16 && out_dtype != WKV6_DTYPE_F32) return WKV6_ERR_UNSUPPORTED;
    return run(B, T, H, N, r, k, v, x, u, state_in, out, state_out, batch_stride, true,
               out_dtype == WKV6_DTYPE_F32, Path::kChunked, stream);
}

int wkv6_finch_c2_prefill_bf16(int B, int T, int H, int N, const void* r, const void* kbar,
                               const void* v, const void* x, const void* uprime,
                               const float* state_in, void* out, float* state_out, void* stream) {
    return run(B, T, H, N, r, kbar, v, x, nullptr, state_in, out, state_out,
               static_cast<long long>(T) * H * N, true, false, Path::kChunked, stream, uprime, true);
}

int wkv6_finch_c2_prefill_bf16_f32out(int B, int T, int H, int N, const void* r, const void* kbar,
                                      const void* v, const void* x, const void* uprime,
                                      const float* state_in, float* out, float* state_out,
                                      void* stream) {
    return run(B, T, H, N, r, kbar, v, x, nullptr, state_in, out, state_out,
               static_cast<long long>(T) * H * N, true, true, Path::kChunked, stream, uprime, true);
}

int wkv6_finch_c2_prefill_bf16_strided(int B, int T, int H, int N, const void* r, const void* kbar,
                                       const void* v, const void* x, const void* uprime,
                                       const float* state_in, void* out, float* state_out,
                                       long long batch_stride, int out_dtype, void* stream) {
    if (out_dtype != WKV6_DTYPE_BF16 && out_dtype != WKV6_DTYPE_F32) return WKV6_ERR_UNSUPPORTED;
    return run(B, T, H, N, r, kbar, v, x, nullptr, state_in, out, state_out, batch_stride, true,
               out_dtype == WKV6_DTYPE_F32, Path::kChunked, stream, uprime, true);
}

int wkv6_finch_c2_prefill_bf16_moments(int B, int T, int H, int N, const void* r, const void* kbar,
                                       const void* v, const void* x, const void* uprime,
                                       const float* state_in, void* out, float* moments, float* state_out,
                                       void* stream) {
    return run(B, T, H, N, r, kbar, v, x, nullptr, state_in, out, state_out,
               static_cast<long long>(T) * H * N, true, false, Path::kChunked, stream, uprime, true, moments,
               true);
}

}  // extern "C"

namespace {

// Fused decay path: sequences at most this long go to the token-by-token kernel, which works on fp32 operands; the one-chunk kernel, which
// takes the next longer ones, rounds its operands to fp16.  The lines were drawn as lines of speed against the chunked kernel, one
// window per round of workgroups at any of these lengths.  Against the one-chunk kernel, which takes any of them in one pass over the states,
// the token-by-token kernel is the faster one for a single token only, and the lines stay for the precision: a call of 2 to 4 tokens is not moved to
// fewer bits.  Microseconds, token by token : one chunk, Finch-C2 with moments: 256 units 1 token 6.0 : 6.6, 2 tokens 7.6 : 6.5; 512 units 1 token
// 6.6 : 7.5, 3 tokens 10.0 : 7.6; 1024 units 1 token 8.7 : 10.0, 4 tokens 14.7 : 10.2; 2048 units 1 token 15.9 : 17.5, 2 tokens 19.7 : 17.5;
// 8192 units 1 token 54.6 : 63.3, 2 tokens 71.1 : 63.4.  Finch: 256 units 2 tokens 6.8 : 5.9; 1024 units 4 tokens 12.9 : 9.4; 2048 units 1
// token 12.1 : 17.0, 3 tokens 15.9 : 16.1, 4 tokens 17.5 : 16.3; 8192 units 1 token 49.7 : 55.3, 2 tokens 55.6 : 55.1, 4 tokens 68.7 : 57.8.
int fused_short_tokens(int B, int H, bool finch_c2) {
    const long long units = static_cast<long long>(B) * H;
    if (units <= 256) return 2;
    if (units <= 512) return 3;
    return units <= 1024 || !finch_c2 ? 4 : 2;
}

// Both forms of the prefill with the decay logits formed in the kernel; `uprime` non-null selects
// the Finch-C2 form (then `u` is unused), otherwise `u` is the Finch bonus.
int run_lora(int B, int T, int H, int N, int R, const void* r, const void* k, const void* v, const void* y,
             const float* lambda, const void* b_omega, const float* u, const void* uprime, bool finch_c2,
             const float* state_in, void* out, float* moments, float* state_out, void* stream) {
    if (N != wkv6::kHeadSize || R != wkv6::kLoraRank) return WKV6_ERR_UNSUPPORTED;
    if (B < 0 || T < 0 || H < 1 || H > 262144) return WKV6_ERR_SHAPE;
    if (!finch_c2 && !u) return WKV6_ERR_NULL;
    if (B == 0) return WKV6_OK;
    if (T > 0) {
        if (!r || !k || !v || !y || !lambda || !b_omega || (finch_c2 && !uprime) || !out) return WKV6_ERR_NULL;
        if (misaligned(r) || misaligned(k) || misaligned(v) || misaligned(y) || misaligned(lambda) ||
            misaligned(b_omega) || misaligned(uprime) || misaligned(out) || misaligned(moments))
            return WKV6_ERR_ALIGN;
    }
    if (misaligned(u) || misaligned(state_in) || misaligned(state_out)) return WKV6_ERR_ALIGN;
    if (static_cast<long long>(B) * H > 0x7fffffffLL) return WKV6_ERR_SHAPE;

    wkv6::Args a;
    a.B = B; a.T = T; a.H = H;
    a.r = r; a.k = k; a.v = v; a.x = nullptr; a.u = u;
    a.finch_c2 = finch_c2;
    a.uprime = finch_c2 ? uprime : nullptr;
    a.state_in = state_in; a.out = out; a.state_out = state_out;
    a.batch_stride = static_cast<long long>(T) * H * N;
    a.segs = 1; a.seg_len = T; a.unit_stride = 0;
    a.moments = moments;
    a.y = y; a.lambda = lambda; a.bw = b_omega;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const wkv6::ChunkedMode mode = moments ? wkv6::ChunkedMode::kBf16OutLoraMoments : wkv6::ChunkedMode::kBf16OutLora;
    hipError_t err;
    if (T == 0)
        err = wkv6::launch_state_passthrough(a, s);
    else if (T <= fused_short_tokens(B, H, finch_c2))
        err = launch_short(a, mode, s);
    else
        err = launch_prefill(a, mode, true, s);
    return err == hipSuccess ? WKV6_OK : WKV6_ERR_LAUNCH;
}

}  // namespace

extern "C" {

int wkv6_finch_c2_prefill_lora_bf16(int B, int T, int H, int N, int R, const void* r, const void* kbar,
                                    const void* v, const void* y, const float* lambda, const void* b_omega,
                                    const void* uprime, const float* state_in, void* out, float* moments,
                                    float* state_out, void* stream) {
    return run_lora(B, T, H, N, R, r, kbar, v, y, lambda, b_omega, nullptr, uprime, true, state_in, out, moments,
                    state_out, stream);
}

int wkv6_prefill_lora_bf16(int B, int T, int H, int N, int R, const void* r, const void* k, const void* v,
                           const void* y, const float* lambda, const void* b_omega, const float* u,
                           const float* state_in, void* out, float* state_out, void* stream) {
    return run_lora(B, T, H, N, R, r, k, v, y, lambda, b_omega, u, nullptr, false, state_in, out, nullptr, state_out,
                    stream);
}

int wkv6_layernorm_finalize(int B, int T, int H, int N, const float* moments, float eps, float* mean_rstd,
                            void* stream) {
    if (N != wkv6::kHeadSize) return WKV6_ERR_UNSUPPORTED;
    if (B < 0 || T < 0 || H < 1 || H > 262144 || B > 65535 || !(eps >= 0.f)) return WKV6_ERR_SHAPE;
    if (B == 0 || T == 0) return WKV6_OK;
    if (!moments || !mean_rstd) return WKV6_ERR_NULL;
    if (misaligned(moments) || misaligned(mean_rstd)) return WKV6_ERR_ALIGN;
    const hipError_t err = wkv6::launch_layernorm_finalize(B, T, H, moments, eps, mean_rstd,
                                                           static_cast<hipStream_t>(stream));
    return err == hipSuccess ? WKV6_OK : WKV6_ERR_LAUNCH;
}

int wkv6_layernorm_apply_bf16(int B, int T, int H, int N, const void* o, const float* mean_rstd, const float* gamma,
                              const float* beta, void* y, int out_dtype, void* stream) {
    if (out_dtype != WKV6_DTYPE_BF16 && out_dtype != WKV6_DTYPE_F32) return WKV6_ERR_UNSUPPORTED;
    if (N != wkv6::kHeadSize) return WKV6_ERR_UNSUPPORTED;
    if (B < 0 || T < 0 || H < 1 || H > 262144) return WKV6_ERR_SHAPE;
    if (B == 0 || T == 0) return WKV6_OK;
    const long long tokens = static_cast<long long>(B) * T;
    if (!o || !mean_rstd || !gamma || !beta || !y) return WKV6_ERR_NULL;
    if (misaligned(o) || misaligned(mean_rstd) || misaligned(gamma) || misaligned(beta) || misaligned(y))
        return WKV6_ERR_ALIGN;
    const hipError_t err = wkv6::launch_layernorm_apply(tokens, H * N, o, mean_rstd, gamma, beta, y,
                                                        out_dtype == WKV6_DTYPE_F32, static_cast<hipStream_t>(stream));
    return err == hipSuccess ? WKV6_OK : WKV6_ERR_LAUNCH;
}

int wkv6_append_bf16(int B, int T, int H, int N, const void* r, const void* k, const void* v,
                     const void* x, const float* u, const float* state_in, void* out,
                     float* state_out, void* stream) {
    return run(B, T, H, N, r, k, v, x, u, state_in, out, state_out,
               static_cast<long long>(T) * H * N, true, false, Path::kBySize, stream);
}

int wkv6_finch_c2_append_bf16(int B, int T, int H, int N, const void* r, const void* kbar,
                              const void* v, const void* x, const void* uprime,
                              const float* state_in, void* out, float* state_out, void* stream) {
    return run(B, T, H, N, r, kbar, v, x, nullptr, state_in, out, state_out,
               static_cast<long long>(T) * H * N, true, false, Path::kBySize, stream, uprime, true);
}

int wkv6_decode_bf16(int B, int H, int N, const void* r, const void* k, const void* v,
                     const void* x, const float* u, float* state, void* out, void* stream) {
    if (!state) return WKV6_ERR_NULL;
    return run(B, 1, H, N, r, k, v, x, u, state, out, state,
               static_cast<long long>(H) * N, true, false, Path::kRecurrent, stream);
}

int wkv6_finch_c2_decode_bf16(int B, int H, int N, const void* r, const void* kbar, const void* v,
                              const void* x, const void* uprime, float* state, void* out,
                              void* stream) {
    if (!state) return WKV6_ERR_NULL;
    return run(B, 1, H, N, r, kbar, v, x, nullptr, state, out, state,
               static_cast<long long>(H) * N, true, false, Path::kRecurrent, stream, uprime, true);
}

int wkv6_prefill_f32(int B, int T, int H, int N, const float* r, const float* k, const float* v,
                     const float* x, const float* u, const float* state_in, float* out,
                     float* state_out, void* stream) {
    return run(B, T, H, N, r, k, v, x, u, state_in, out, state_out,
               static_cast<long long>(T) * H * N, false, true, Path::kF32, stream);
}

int wkv6_prefill_bf16_recurrent(int B, int T, int H, int N, const void* r, const void* k,
                                const void* v, const void* x, const float* u,
                                const float* state_in, float* out, float* state_out,
                                void* stream) {
    return run(B, T, H, N, r, k, v, x, u, state_in, out, state_out,
               static_cast<long long>(T) * H * N, true, true, Path::kRecurrent, stream);
}

int wkv6_key_compress_bf16(long long M, int D, const void* x, const void* w_kd, void* c, int out_dtype,
                           void* stream) {
    if (out_dtype != WKV6_DTYPE_BF16 && out_dtype != WKV6_DTYPE_F32) return WKV6_ERR_UNSUPPORTED;
    if (D < 256 || D % 256 != 0 || D > 65536) return WKV6_ERR_UNSUPPORTED;
    if (M < 0 || ((M + 127) / 128 + 8) * ((D / 16 + 127) / 128) > 0x7fffffffLL) return WKV6_ERR_SHAPE;   // grid size
    if (M == 0) return WKV6_OK;
    if (!x || !w_kd || !c) return WKV6_ERR_NULL;
    if (misaligned(x) || misaligned(w_kd) || misaligned(c)) return WKV6_ERR_ALIGN;
    const hipError_t err = wkv6::launch_key_compress(M, D, x, w_kd, c, out_dtype == WKV6_DTYPE_F32,
                                                     static_cast<hipStream_t>(stream));
    return err == hipSuccess ? WKV6_OK : WKV6_ERR_LAUNCH;
}

int wkv6_decay_lora_input_bf16(int B, int T, int D, int R_d, int R, const void* x, const void* x_prev,
                               const float* mu_x, const float* lambda_d, const void* a_d, const void* b_d,
                               const void* a_omega, void* y, int out_dtype, void* stream) {
    if (out_dtype != WKV6_DTYPE_BF16 && out_dtype != WKV6_DTYPE_F32) return WKV6_ERR_UNSUPPORTED;
    if (R_d != 32 || R != wkv6::kLoraRank) return WKV6_ERR_UNSUPPORTED;
    if (D < 128 || D % 128 != 0 || D > 65536) return WKV6_ERR_UNSUPPORTED;
    if (B < 0 || T < 0) return WKV6_ERR_SHAPE;
    if (B == 0 || T == 0) return WKV6_OK;
    if (static_cast<long long>(B) * ((T + 127) / 128) > 0x7fffffffLL) return WKV6_ERR_SHAPE;  // grid size
    if (!x || !mu_x || !lambda_d || !a_d || !b_d || !a_omega || !y) return WKV6_ERR_NULL;
    if (misaligned(x) || misaligned(x_prev) || misaligned(mu_x) || misaligned(lambda_d) || misaligned(a_d) ||
        misaligned(b_d) || misaligned(a_omega) || misaligned(y))
        return WKV6_ERR_ALIGN;
    const hipError_t err = wkv6::launch_decay_input(B, T, D, x, x_prev, mu_x, lambda_d, a_d, b_d, a_omega, y,
                                                    out_dtype == WKV6_DTYPE_F32, static_cast<hipStream_t>(stream));
    return err == hipSuccess ? WKV6_OK : WKV6_ERR_LAUNCH;
}

long long wkv6_arena_layout(int count, const long long* bytes, long long* offsets) {
    if (count < 0 || count > 64) return -1;
    if (count > 0 && (!bytes || !offsets)) return -1;
    long long cursor = 0;
    for (int i = 0; i < count; ++i) {
        if (bytes[i] < 0 || bytes[i] > (1ll << 46)) return -1;
        cursor = (cursor + WKV6_PLACEMENT_ALIGN - 1) / WKV6_PLACEMENT_ALIGN * WKV6_PLACEMENT_ALIGN;
        offsets[i] = cursor + WKV6_PLACEMENT_STEP * (i % 8);
        cursor = offsets[i] + bytes[i];
    }
    return (cursor + WKV6_PLACEMENT_ALIGN - 1) / WKV6_PLACEMENT_ALIGN * WKV6_PLACEMENT_ALIGN;
}

const char* wkv6_status_string(int status) {
    switch (status) {
        case WKV6_OK: return "ok";
        case WKV6_ERR_NULL: return "a required pointer is NULL";
        case WKV6_ERR_SHAPE: return "invalid shape or stride";
        case WKV6_ERR_UNSUPPORTED: return "unsupported head size or dtype";
        case WKV6_ERR_LAUNCH: return "kernel launch failed";
        case WKV6_ERR_ALIGN: return "pointer or stride not 16-byte aligned";
        case WKV6_ERR_WORKSPACE: return "shape needs more scratch than the library holds";
        default: return "unknown status";
    }
}

int wkv6_version(void) { return 500; }

}  // extern "C"

// ---- token-split variant: three enqueued passes over caller-provided workspace

extern "C" {

// The recommendation for the explicit split entries; the entry points that split by themselves follow plan_own_split.
int wkv6_split_segments(int B, int T, int H, int N) {
    if (N != wkv6::kHeadSize || B < 1 || T < 1 || H < 1) return 1;
    const long long units = static_cast<long long>(B) * H;
    const int cus = 256;                         // workgroups resident at once on an MI355X (one per CU); a
                                                 // pure function of the shape so that it needs no device
    if (units * 4 > cus * 3) return 1;           // already fills three quarters of the chip
    long long segs = cus / units;
    const long long by_len = T / 2048;           // keep segments long enough to amortise pass 1
    if (segs > by_len) segs = by_len;
    return segs < 2 ? 1 : static_cast<int>(segs);
}

long long wkv6_split_workspace_bytes(int B, int T, int H, int N, int segments) {
    if (N != wkv6::kHeadSize || B < 0 || T < 0 || H < 1 || segments < 1) return -1;
    const wkv6::SplitPlan p = wkv6::plan_split(T > 0 ? T : 1, segments);
    return static_cast<long long>(B) * p.segs * H * (wkv6::kHeadSize * wkv6::kHeadSize + wkv6::kHeadSize) * 4;
}

}  // extern "C"

// ---- library-owned scratch for the entry point that may not allocate

namespace {

// Per-segment local states and decay totals of wkv6_prefill_bf16_split_noalloc.  Every GPU the
// library runs on holds its own copy of this array, at its own address, until the process ends.
// In host code the array's name is only a handle for hipGetSymbolAddress; the device address it
// returns is what kernels, copies and fills must be given.
constexpr long long kScratchBytes = 8ll << 20;
static __device__ __align__(256) __attribute__((used)) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_lock;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device, looked up once per device.
int scratch_of_current_device(void** ptr) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return WKV6_ERR_LAUNCH;
    std::lock_guard<std::mutex> hold(g_scratch_lock);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return WKV6_ERR_LAUNCH;
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return WKV6_OK;
}

int run_split(int B, int T, int H, int N, const void* r, const void* k, const void* v, const void* x,
              const float* u, const void* uprime, bool finch_c2, const float* state_in, void* out,
              float* state_out, int out_dtype, int segments, void* workspace,
              long long workspace_bytes, void* stream) {
    if (out_dtype != WKV6_DTYPE_BF16 && out_dtype != WKV6_DTYPE_F32) return WKV6_ERR_UNSUPPORTED;
    if (N != wkv6::kHeadSize) return WKV6_ERR_UNSUPPORTED;
    if (B < 0 || T < 0 || H < 1 || H > 262144 || segments < 1) return WKV6_ERR_SHAPE;
    const wkv6::SplitPlan p = wkv6::plan_split(T > 0 ? T : 1, segments);
    if (T == 0 || B == 0 || p.segs == 1)
        return run(B, T, H, N, r, k, v, x, u, state_in, out, state_out,
                   static_cast<long long>(T) * H * N, true, out_dtype == WKV6_DTYPE_F32,
                   Path::kChunked, stream, uprime, finch_c2, nullptr, false, false);
    if ((!finch_c2 && !u) || (finch_c2 && !uprime) || !r || !k || !v || !x || !out || !workspace)
        return WKV6_ERR_NULL;
    if (misaligned(r) || misaligned(k) || misaligned(v) || misaligned(x) || misaligned(out) ||
        misaligned(u) || misaligned(uprime) || misaligned(state_in) || misaligned(state_out) ||
        misaligned(workspace))
        return WKV6_ERR_ALIGN;
    if (workspace_bytes < wkv6_split_workspace_bytes(B, T, H, N, segments)) return WKV6_ERR_SHAPE;
    if (static_cast<long long>(B) * p.segs * H > 0x7fffffffLL) return WKV6_ERR_SHAPE;

    wkv6::Args a;
    a.B = B; a.T = T; a.H = H;
    a.r = r; a.k = k; a.v = v; a.x = x; a.u = u;
    a.finch_c2 = finch_c2;
    a.uprime = finch_c2 ? uprime : nullptr;
    a.state_in = state_in; a.out = out; a.state_out = state_out;
    a.batch_stride = static_cast<long long>(T) * H * N;
    a.segs = p.segs; a.seg_len = p.seg_len; a.unit_stride = 0; a.moments = nullptr;
    a.y = nullptr; a.lambda = nullptr; a.bw = nullptr;
    // pass 1: every segment but the last (nothing follows it) from a zero state, no output: its local state and
    // total decay; pass 2: the state entering every segment (in place); pass 3: the full computation of every
    // segment from its true entering state; the last segment's workgroups leave the sequence's final state
    constexpr long long kPlaceBytes = (wkv6::kHeadSize * wkv6::kHeadSize + wkv6::kHeadSize) * 4;
    a.place.base = static_cast<char*>(workspace);
    a.place.head = kPlaceBytes;
    a.place.seg = H * kPlaceBytes;
    a.place.batch = p.segs * a.place.seg;
    a.place.row = 256;
    a.place.half = 128;
    const wkv6::ChunkedMode mode = out_dtype == WKV6_DTYPE_F32 ? wkv6::ChunkedMode::kF32Out
                                                               : wkv6::ChunkedMode::kBf16Out;
    if (launch_prefill(a, mode, false, static_cast<hipStream_t>(stream)) != hipSuccess) return WKV6_ERR_LAUNCH;
    return WKV6_OK;
}

}  // namespace

extern "C" {

int wkv6_prefill_bf16_split(int B, int T, int H, int N, const void* r, const void* k, const void* v,
                            const void* x, const float* u, const float* state_in, void* out,
                            float* state_out, int out_dtype, int segments, void* workspace,
                            long long workspace_bytes, void* stream) {
    return run_split(B, T, H, N, r, k, v, x, u, nullptr, false, state_in, out, state_out, out_dtype,
                     segments, workspace, workspace_bytes, stream);
}

int wkv6_prefill_bf16_split_noalloc(int B, int T, int H, int N, const void* r, const void* k, const void* v,
                                    const void* x, const float* u, const float* state_in, void* out,
                                    float* state_out, int out_dtype, int segments, void* stream) {
    const long long need = wkv6_split_workspace_bytes(B, T, H, N, segments);
    if (need < 0) return N != wkv6::kHeadSize ? WKV6_ERR_UNSUPPORTED : WKV6_ERR_SHAPE;
    if (need > kScratchBytes) return WKV6_ERR_WORKSPACE;
    void* ws = nullptr;
    const int status = scratch_of_current_device(&ws);
    if (status != WKV6_OK) return status;
    return run_split(B, T, H, N, r, k, v, x, u, nullptr, false, state_in, out, state_out, out_dtype,
                     segments, ws, kScratchBytes, stream);
}

int wkv6_finch_c2_prefill_bf16_split(int B, int T, int H, int N, const void* r, const void* kbar,
                                     const void* v, const void* x, const void* uprime,
                                     const float* state_in, void* out, float* state_out,
                                     int out_dtype, int segments, void* workspace,
                                     long long workspace_bytes, void* stream) {
    return run_split(B, T, H, N, r, kbar, v, x, nullptr, uprime, true, state_in, out, state_out,
                     out_dtype, segments, workspace, workspace_bytes, stream);
}

}  // extern "C"

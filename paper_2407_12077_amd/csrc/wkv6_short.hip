// Sequences of one chunk (the next turn of a conversation, short prompts), for gfx950 (MI355X): what wkv6_chunked.hip computes
// for a chunk of 32 tokens, operand for operand and sum for sum (the bits are the same), by four waves per (batch, head) that do
// all of its roles in turn.
//
// A unit's work is one pass over its state (16 KiB in, 16 KiB out) and its rows, between which lies a chain of four
// barriers; what counts is how many units a compute unit has in flight.  The chunked kernel's workgroup holds one in each of
// its stages, in 140 KB of LDS, and fills and drains them: nine windows for four units.  Here a unit takes 36 KB (Finch form 40),
// four of them share a compute unit, and each requests its state and rows at once.  Microseconds, chunked kernel -> here,
// Finch-C2, 32 heads: 8 x 24 tokens 6.1 -> 5.5, 9 x 24 8.1 -> 5.8, 20 x 24 11.5 -> 8.0, 32 x 24 14.1 -> 10.1 (52 MB: 5.2 TB/s), 64 x 24 20.9 ->
// 17.9, 256 x 7 63 -> 56, 256 x 32 90 -> 84; Finch 32 x 24 12.4 -> 9.0, 128 x 16 36 -> 30; fused decay path with moments 32 x 24 15.8 -> 11.1.
// (Two chunks and more by the same waves, one after the other, lose: 8 x 64 tokens 7.5 -> 8.2, 64 x 80 38 -> 41.)
//
// LDS: the tiles as there, with unpadded rows of 128 bytes (tile rows) and 64 (transposed ones, scores) whose granules are swizzled so that
// 16-byte reads meet no bank conflicts; the group products share their place with the scores, the staged rows and the final state with the tiles, the logits of
// the fused decay path with the transposed tiles, its outer factor with the level tiles.
#include "wkv6_launch.h"
#include "wkv6_tiles.h"

namespace wkv6 {
namespace {

constexpr int kRow = 128;                  // fp16 row of 64 channels
constexpr int kTile = kChunk * kRow;
// Cache policies.  The state leaves in whole lines, through the L2 and non-temporal: written back from there at the kernel's
// end it costs 512 units x 24 tokens 1.5 us.
constexpr int kStatePolicy = kStoreThrough | kStreamOnce;
constexpr int kBwRow = 160;                // row of the outer factor's 64 x 64 slice: 128 B + 32 pad (transposing reads)

template <bool kC2>
struct Lds {
    static constexpr int kZ16 = 0, kZ8 = kTile, kZ4 = 2 * kTile, kZ2 = 3 * kTile, kQ1 = 4 * kTile, kRT = 5 * kTile;
    static constexpr int kK1 = 6 * kTile;                        // Finch form only
    static constexpr int kKT = (kC2 ? 6 : 7) * kTile;            // [64 channels][32 tokens]
    static constexpr int kVT = kKT + 64 * 64;
    static constexpr int kA0 = kVT + 64 * 64, kA1 = kA0 + kChunk * 64;      // [32 t][32 i]
    static constexpr int kBytes = kA1 + kChunk * 64;
    static constexpr int kG = kA0;                               // group products [8][64] fp32: read before the scores are written
    static constexpr int kO = 0;                                 // staged rows: the level tiles have been read
    static constexpr int kState = kChunk * kORowF32 * 4;         // behind them the final state [64][64] fp32: every tile has been read
    static constexpr int kBw = 0;                                // outer factor: before there are tiles
    static constexpr int kDx = kKT;                              // logits [channel pair][parity][token] fp32: likewise
    static_assert(kA1 - kG >= 8 * 64 * 4 && kA0 >= kState + 64 * 256 && kKT >= 64 * kBwRow && kA0 - kDx >= 64 * kChunk * 4, "overlays");
    static_assert(kBytes <= 40 * 1024, "four units to a compute unit");
};

// byte of a row of 64 channels: rows two apart start at the same bank, so the 16-byte granules turn with the row pair
__device__ __forceinline__ int row_off(int row, int byte) { return row * kRow + (byte ^ (((row >> 1) & 7) << 4)); }

// 16-byte granule (8 tokens) of a 64-byte row; rows four apart start at the same bank
__device__ __forceinline__ int token_off(int row, int granule) { return row * 64 + ((granule ^ ((row >> 2) & 3)) << 4); }
// byte of a state row: the four rows that a write's lane groups hold go to different quarters
__device__ __forceinline__ int state_off(int row, int byte) { return row * 256 + (byte ^ (((row >> 2) & 3) << 6)); }
// The chunk's decays, four channels each, lie where the scores of tokens 0 .. 15 with keys 16 .. 23 would: none is written.
__device__ __forceinline__ int decay_off(int quad) { return token_off(quad, 2); }
// granule (4 tokens) of a channel's logits; pairs all start at the same bank
__device__ __forceinline__ int logit_off(int pair, int parity, int quad) { return pair * 256 + (((8 * parity + quad) ^ (pair & 15)) << 4); }

// 8 consecutive rows of one column of a row-major 16-bit tile as an MFMA operand: two transposing reads of 4 rows.  Within a
// group of 16 lanes, lane i passes the address of the entries [i >> 2][4 (i & 3) ..] of a 4 x 16 block and receives its column i.
__device__ __forceinline__ bf16x8 lds_read_column8(const char* lds, int off) {
    typedef short short4v __attribute__((ext_vector_type(4)));
    typedef short short8v __attribute__((ext_vector_type(8)));
    typedef short4v __attribute__((address_space(3))) * lds_s4_ptr;
    const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_ptr)(lds + off));
    const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_ptr)(lds + off + 4 * kBwRow));
    const short8v both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, both);
}

// kRows: cache policy of the rows' loads, kStreamOnce or 0 (temporal)
template <bool kC2, bool kLora, bool kOutF32, bool kMoments, int kRows>
__global__ __launch_bounds__(kOneChunkThreads, 4) void one_chunk_kernel(Args a) {
    using L = Lds<kC2>;
    constexpr bool kStageF32 = kOutF32 || kC2;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    clamp_fp16_overflow();
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g4 = lane >> 4;
    const int wq = __builtin_amdgcn_readfirstlane(tid >> 6);
    int unit = blockIdx.x;                         // batch * H + head
    if constexpr (kLora) {                         // as in the chunked kernel: neighbouring heads of a batch read y through one L2
        const int per_xcd = gridDim.x >> 3;
        if ((gridDim.x & 7) == 0) unit = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    }
    const int b = unit / a.H, h = unit - b * a.H;
    const int cp = lane & 31, hl = lane >> 5;      // this thread forms the operands of channels 2 cp, 2 cp + 1 and
    const int g8 = 2 * wq + hl;                    // tokens 4 g8 .. + 3
    const int T = a.T;                             // at most kChunk
    const long long row_bytes = static_cast<long long>(a.H) * (kHeadSize * 2);
    const long long base = static_cast<long long>(b) * a.batch_stride + h * kHeadSize;
    const long long span = static_cast<long long>(T - 1) * row_bytes + kHeadSize * 2;      // rows past the end read as zero

    // ---- everything the unit needs, requested in the order of its use
    [[maybe_unused]] bf16x8 ya[2][2];
    [[maybe_unused]] uint4v bw_rows[2];
    [[maybe_unused]] float lam = 0.f;
    if constexpr (kLora) {
        const __amdgpu_buffer_rsrc_t ry = chunk_rsrc(static_cast<const char*>(a.y) + static_cast<long long>(b) * T * (kLoraRank * 2), 0, T * (kLoraRank * 2));
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
                ya[rt][ks] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(ry, (16 * rt + l16) * (kLoraRank * 2) + 16 * g4 + 64 * ks, 0, 0));
        const char* bw = static_cast<const char*>(a.bw) + h * (kHeadSize * 2) + 16 * (tid & 7);
#pragma unroll
        for (int i = 0; i < 2; ++i) bw_rows[i] = *reinterpret_cast<const uint4v*>(bw + static_cast<long long>((tid >> 3) + 32 * i) * row_bytes);
        lam = a.lambda[h * kHeadSize + 16 * wq + l16];
    }
    Raw raw;
    auto rows = [&](unsigned (&d)[4], const void* p) {
        const __amdgpu_buffer_rsrc_t rs = chunk_rsrc(static_cast<const char*>(p) + base * 2, 0, span);
#pragma unroll
        for (int s = 0; s < 4; ++s) d[s] = __builtin_amdgcn_raw_buffer_load_b32(rs, static_cast<int>((4 * g8 + s) * row_bytes) + 4 * cp, 0, kRows);
    };
    if constexpr (!kLora) rows(raw.x, a.x);
    rows(raw.k, a.k);
    rows(raw.r, a.r);
    rows(raw.v, a.v);
    const unsigned hu = kC2 ? 0u : pack_h2(a.u[h * kHeadSize + 2 * cp], a.u[h * kHeadSize + 2 * cp + 1]);
    // S[nb][e] = state[16 nb + 4 g4 + e][16 wq + l16]
    float4v S[4];
    const int state_voff = (4 * g4 * kHeadSize + 16 * wq + l16) * 4;
    auto state_rsrc = [&](const float* p) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p + static_cast<long long>(unit) * 4096), 0, 4096 * 4, 0x00020000);
    };
    if (a.state_in) {
        const __amdgpu_buffer_rsrc_t rs = state_rsrc(a.state_in);
#pragma unroll
        for (int nb = 0; nb < 4; ++nb)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                S[nb][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, state_voff, (16 * nb + e) * 256, 0));
    } else {
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) S[nb] = float4v{0.f, 0.f, 0.f, 0.f};
    }
    const int srow = tid >> 3, scol = 8 * (tid & 7);         // row and first channel that this thread stores
    [[maybe_unused]] uint4v up_raw = {0u, 0u, 0u, 0u};
    if constexpr (kC2) {
        const __amdgpu_buffer_rsrc_t ru = chunk_rsrc(static_cast<const char*>(a.uprime) + base * 2, 0, span);
        const int up_voff = static_cast<int>(srow * row_bytes) + (kOutF32 ? scol : scol * 2);
        if constexpr (kOutF32) {                             // thread j of an fp32 row: channels 4 j .. and 32 + 4 j ..
            const uint2v lo = __builtin_bit_cast(uint2v, __builtin_amdgcn_raw_buffer_load_b64(ru, up_voff, 0, kRows));
            const uint2v hi = __builtin_bit_cast(uint2v, __builtin_amdgcn_raw_buffer_load_b64(ru, up_voff + 64, 0, kRows));
            up_raw = uint4v{lo[0], lo[1], hi[0], hi[1]};
        } else {
            up_raw = __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(ru, up_voff, 0, kRows));
        }
    }

    // ---- decays
    float w[2][4];
    [[maybe_unused]] float omw[2][4];
    if constexpr (kLora) {
        // logits of this wave's 16 channels, d = lambda + y B
#pragma unroll
        for (int i = 0; i < 2; ++i) *reinterpret_cast<uint4v*>(lds + L::kBw + ((tid >> 3) + 32 * i) * kBwRow + 16 * (tid & 7)) = bw_rows[i];
        __syncthreads();
        bf16x8 bw[2];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) bw[ks] = lds_read_column8(lds, L::kBw + (32 * ks + 8 * g4 + (l16 >> 2)) * kBwRow + 8 * (l16 & 3) + 32 * wq);
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) {
            float4v acc = {lam, lam, lam, lam};
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ya[rt][0], bw[0], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ya[rt][1], bw[1], acc, 0, 0, 0);
            *reinterpret_cast<float4v*>(lds + L::kDx + logit_off(8 * wq + (l16 >> 1), l16 & 1, 4 * rt + g4)) = acc;
        }
        __syncthreads();
#pragma unroll
        for (int ch = 0; ch < 2; ++ch) {
            const float4v d = *reinterpret_cast<const float4v*>(lds + L::kDx + logit_off(cp, ch, g8));
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                float e = 0.f;
                const float ws = decay_of(d[s], e);
                w[ch][s] = 4 * g8 + s >= T ? 1.f : ws;       // past the end: w = 1 (and the key is zero)
                if constexpr (kC2) omw[ch][s] = one_minus_decay(e, ws);
            }
        }
    } else {
#pragma unroll
        for (int s = 0; s < 4; ++s)
            if (4 * g8 + s >= T) raw.x[s] = 0xff80ff80u;     // bf16 -inf, twice: w = 1
        decays_of<kC2>(raw.x, w, omw);
    }
    Prep pr;
    *reinterpret_cast<float2*>(lds + L::kG + (g8 * 64 + 2 * cp) * 4) = form_operands<kC2>(pr, raw, w, omw, hu);
    __syncthreads();                                         // group products

    // ---- tiles
    {
        float2 own[8];
#pragma unroll
        for (int g = 0; g < 8; ++g) own[g] = *reinterpret_cast<const float2*>(lds + L::kG + (g * 64 + 2 * cp) * 4);
        auto put4_at = [&](int tile, int byte, unsigned v0, unsigned v1, unsigned v2, unsigned v3) {      // the group's four rows
            const int lo = tile + row_off(4 * g8, byte), hi = tile + row_off(4 * g8 + 2, byte);
            lds_write_u32(lds, lo, v0);
            lds_write_u32(lds, lo + kRow, v1);
            lds_write_u32(lds, hi, v2);
            lds_write_u32(lds, hi + kRow, v3);
        };
        auto put4 = [&](int tile, unsigned v0, unsigned v1, unsigned v2, unsigned v3) { put4_at(tile, 4 * cp, v0, v1, v2, v3); };
        const int tr0 = token_off(2 * cp, wq) + 8 * hl, tr1 = token_off(2 * cp + 1, wq) + 8 * hl;
        lds_write_u64(lds, L::kVT + tr0, pr.vt[0], pr.vt[1]);
        lds_write_u64(lds, L::kVT + tr1, pr.vt[2], pr.vt[3]);
        const bool q4 = hl != 0;                             // query side at level 4
        put4(L::kZ4, q4 ? pr.rp[0] : pr.ks[0], q4 ? pr.rp[1] : pr.ks[1], q4 ? pr.rp[2] : pr.ks[2], q4 ? pr.rp[3] : pr.ks[3]);
        put4(L::kZ2, pr.z2[0], pr.z2[1], pr.z2[2], pr.z2[3]);
        put4(L::kQ1, pr.q1[0], pr.q1[1], pr.q1[2], pr.q1[3]);
        if constexpr (!kC2) put4(L::kK1, pr.k1[0], pr.k1[1], pr.k1[2], pr.k1[3]);
        const bool q8 = wq & 1, q16 = wq & 2;                // query side at levels 8 and 16 (uniform)
        float m_rt[2], m_kt[2], m16[2], m8[2];
#pragma unroll
        for (int ch = 0; ch < 2; ++ch) {
            float o[8];
#pragma unroll
            for (int g = 0; g < 8; ++g) o[g] = ch ? own[g].y : own[g].x;
            // pl / ph: decays of the group pairs before / after this wave's; f16: its share of the level-16 multiplier
            const float o01 = o[0] * o[1], o23 = o[2] * o[3], o45 = o[4] * o[5], o67 = o[6] * o[7];
            const float pl = wq == 0 ? 1.f : wq == 1 ? o01 : wq == 2 ? o01 * o23 : (o01 * o23) * o45;
            const float ph = wq == 0 ? o23 * (o45 * o67) : wq == 1 ? o45 * o67 : wq == 2 ? o67 : 1.f;
            const float f16 = wq == 0 ? o23 : wq == 3 ? o45 : 1.f;
            const float even = wq == 0 ? o[0] : wq == 1 ? o[2] : wq == 2 ? o[4] : o[6];
            const float odd = wq == 0 ? o[1] : wq == 1 ? o[3] : wq == 2 ? o[5] : o[7];
            const float before = hl ? even : 1.f, after = hl ? 1.f : odd;      // the pair's other group
            m_rt[ch] = pl * before;                          // decays of the tokens before this group
            m_kt[ch] = after * ph;                           // and behind it
            m16[ch] = q16 ? f16 * before : after * f16;
            m8[ch] = q8 ? before : after;
            if (wq == 0 && hl == 0) *reinterpret_cast<float*>(lds + L::kA1 + decay_off(cp >> 1) + 8 * (cp & 1) + 4 * ch) = o[0] * m_kt[ch];
        }
        const unsigned h_rt = pack_h2(m_rt[0], m_rt[1]), h_kt = pack_h2(m_kt[0], m_kt[1]);
        const unsigned h16 = pack_h2(m16[0], m16[1]), h8 = pack_h2(m8[0], m8[1]);
        const unsigned k0 = mul_h2(pr.ks[0], h_kt), k1 = mul_h2(pr.ks[1], h_kt), k2 = mul_h2(pr.ks[2], h_kt), k3 = mul_h2(pr.ks[3], h_kt);
        lds_write_u64(lds, L::kKT + tr0, lo_halves(k0, k1), lo_halves(k2, k3));
        lds_write_u64(lds, L::kKT + tr1, hi_halves(k0, k1), hi_halves(k2, k3));
        unsigned z16[4], z8[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            z16[s] = mul_h2(q16 ? pr.rp[s] : pr.ks[s], h16);
            z8[s] = mul_h2(q8 ? pr.rp[s] : pr.ks[s], h8);
        }
        put4(L::kZ16, z16[0], z16[1], z16[2], z16[3]);
        put4(L::kZ8, z8[0], z8[1], z8[2], z8[3]);
        // column of this channel pair in the r W(t,-1) tile: slot order of the state registers
        const int n0 = 2 * cp, m5 = n0 & 31;
        const int rt_col = (n0 & 32) + 8 * ((m5 >> 2) & 3) + 4 * (m5 >> 4) + (m5 & 3);
        put4_at(L::kRT, rt_col * 2, mul_h2(pr.rp[0], h_rt), mul_h2(pr.rp[1], h_rt), mul_h2(pr.rp[2], h_rt), mul_h2(pr.rp[3], h_rt));
    }
    __syncthreads();                                         // tiles

    // ---- scores: diagonal block q, channel half kk; waves with q == 0 also the level-16 block
    {
        const int q = wq & 1, kk = wq >> 1, at = kk ? L::kA1 : L::kA0;
        const int rowq = row_off(16 * q + l16, 16 * g4 + 64 * kk);
        const half8 z8 = lds_read_h8(lds, L::kZ8 + rowq);
        const half8 z4 = lds_read_h8(lds, L::kZ4 + rowq);
        const half8 z2 = lds_read_h8(lds, L::kZ2 + rowq);
        const half8 q1 = lds_read_h8(lds, L::kQ1 + rowq);
        const half8 k1 = kC2 ? q1 : lds_read_h8(lds, L::kK1 + rowq);
        const float4v zero{0.f, 0.f, 0.f, 0.f};
        const float4v acc8 = mfma(z8, z8, zero), acc4 = mfma(z4, z4, zero), acc2 = mfma(z2, z2, zero), acc1 = mfma(k1, q1, zero);
        *reinterpret_cast<uint2*>(lds + at + token_off(16 * q + l16, 2 * q + (g4 >> 1)) + 8 * (g4 & 1)) = choose_levels<kC2>(acc8, acc4, acc2, acc1, l16, g4);
        if (q == 0) {
            const half8 zq = lds_read_h8(lds, L::kZ16 + row_off(16 + l16, 16 * g4 + 64 * kk));
            const half8 zk = lds_read_h8(lds, L::kZ16 + row_off(l16, 16 * g4 + 64 * kk));
            const float4v acc = mfma(zk, zq, zero);
            lds_write_u64(lds, at + token_off(16 + l16, g4 >> 1) + 8 * (g4 & 1), pack_h2(acc[0], acc[1]), pack_h2(acc[2], acc[3]));
        }
    }
    // ---- read-out of the entering state, then the state: value columns 16 wq ..
    half8 sh[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int e = 0; e < 8; ++e) sh[kk][e] = static_cast<_Float16>(S[2 * kk + (e >> 2)][e & 3]);
    float4v o[2];
#pragma unroll
    for (int tq = 0; tq < 2; ++tq) {
        o[tq] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) o[tq] = mfma(sh[kk], lds_read_h8(lds, L::kRT + row_off(16 * tq + l16, 64 * kk + 16 * g4)), o[tq]);
    }
    const half8 vt = lds_read_h8(lds, L::kVT + token_off(16 * wq + l16, g4));
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
        S[nb] *= *reinterpret_cast<const float4v*>(lds + L::kA1 + decay_off(4 * nb + g4));
        S[nb] = mfma(lds_read_h8(lds, L::kKT + token_off(16 * nb + l16, g4)), vt, S[nb]);
    }
    __syncthreads();                                         // scores; every level tile has been read

    // ---- scores times values, staging (transposed: a lane holds four channels of one token)
#pragma unroll
    for (int tq = 0; tq < 2; ++tq) {
        const int off = token_off(16 * tq + l16, g4);
        half8 a0 = lds_read_h8(lds, L::kA0 + off), a1 = lds_read_h8(lds, L::kA1 + off);
        if (tq == 0 && g4 >= 2) a0 = a1 = half8{};           // keys 16 .. 31 of tokens 0 .. 15 have no score
        o[tq] = mfma(vt, a0, o[tq]);
        o[tq] = mfma(vt, a1, o[tq]);
        const int row = 16 * tq + l16, col = 16 * wq + 4 * g4;
        if constexpr (kStageF32)
            *reinterpret_cast<float4v*>(lds + L::kO + (row * kORowF32 + col) * 4) = o[tq];
        else
            lds_write_u64(lds, L::kO + (row * kORowBf16 + col) * 2, pack_bf2(o[tq][0], o[tq][1]), pack_bf2(o[tq][2], o[tq][3]));
    }
    // the state through LDS as well: whole lines leave, 16 bytes a thread
    if (a.state_out) {
#pragma unroll
        for (int nb = 0; nb < 4; ++nb)
#pragma unroll
            for (int e = 0; e < 4; ++e) *reinterpret_cast<float*>(lds + L::kState + state_off(16 * nb + 4 * g4 + e, 64 * wq + 4 * l16)) = S[nb][e];
    }
    __syncthreads();                                         // rows, state

    if (a.state_out) {
        const __amdgpu_buffer_rsrc_t rs = state_rsrc(a.state_out);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = (tid >> 4) + 16 * i, byte = 16 * (tid & 15);
            __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const uint4v*>(lds + L::kState + state_off(row, byte)), rs, row * 256 + byte, 0, kStatePolicy);
        }
    }
    // ---- rows, 8 threads each
    if (srow >= T) return;
    constexpr int kOutElem = kOutF32 ? 4 : 2;
    const long long out_row = static_cast<long long>(a.H) * (kHeadSize * kOutElem);
    const __amdgpu_buffer_rsrc_t ro = chunk_rsrc(static_cast<const char*>(a.out) + base * kOutElem, 0, (T - 1) * out_row + kHeadSize * kOutElem);
    const int out_voff = static_cast<int>(srow * out_row) + scol * kOutElem;
    auto put = [&](uint4v q, int byte) { __builtin_amdgcn_raw_buffer_store_b128(q, ro, out_voff + byte, 0, kStoreThrough); };
    if constexpr (kStageF32) {
        // fp32 rows: thread j holds floats 4 j .. and 32 + 4 j .., whole lines per instruction
        const float4* src = reinterpret_cast<const float4*>(lds + L::kO + (srow * kORowF32 + (kOutF32 ? scol / 2 : scol)) * 4);
        float4 q0 = src[0], q1 = src[kOutF32 ? 8 : 1];
        if constexpr (kC2) add_uprime(q0, q1, up_raw);
        if constexpr (kMoments) {
            const float2v pair = row_moments(q0, q1);
            if (scol == 0) __builtin_nontemporal_store(pair, reinterpret_cast<float2v*>(a.moments + (static_cast<long long>(unit) * T + srow) * 2));
        }
        if constexpr (!kOutF32) {
            put(pack_row(q0, q1), 0);
        } else {
            put(__builtin_bit_cast(uint4v, q0), -scol * 2);
            put(__builtin_bit_cast(uint4v, q1), 128 - scol * 2);
        }
    } else {
        put(*reinterpret_cast<const uint4v*>(lds + L::kO + (srow * kORowBf16 + scol) * 2), 0);
    }
}

template <bool kC2, bool kLora, bool kOutF32, bool kMoments>
hipError_t go(const Args& a, hipStream_t stream) {
    const dim3 grid(static_cast<unsigned>(a.B) * static_cast<unsigned>(a.H));
    // Temporal loads let rows that a kernel has just written, or that the memory-side cache still holds, come from there, as long
    // as the call's bytes are a part of what it holds; smaller calls lose by it the L2 that their states lie in.  Temporal against
    // streamed, microseconds, Finch-C2: 512 units x 24 tokens (26 MB) 7.0 : 6.5, 1024 x 24 (52 MB) 10.0 : 12.5, 1536 x 8 (59 MB) 12.0 :
    // 13.8, 2048 x 24 (104 MB) 17.9 : 21.2, 4096 x 8 (159 MB) 28.7 : 29.3, 4096 x 24 (209 MB) 41.0 : 36.1.
    const long long bytes = static_cast<long long>(grid.x) * (2 * 4096 * 4 + a.T * (kHeadSize * 2) * (kC2 ? 6 : 5));
    if (bytes >= 32ll << 20 && bytes <= 160ll << 20)
        hipLaunchKernelGGL((one_chunk_kernel<kC2, kLora, kOutF32, kMoments, 0>), grid, dim3(kOneChunkThreads), Lds<kC2>::kBytes, stream, a);
    else
        hipLaunchKernelGGL((one_chunk_kernel<kC2, kLora, kOutF32, kMoments, kStreamOnce>), grid, dim3(kOneChunkThreads), Lds<kC2>::kBytes, stream, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_one_chunk(const Args& a, ChunkedMode mode, hipStream_t stream) {
    switch (mode) {
        case ChunkedMode::kBf16Out: return a.finch_c2 ? go<true, false, false, false>(a, stream) : go<false, false, false, false>(a, stream);
        case ChunkedMode::kF32Out: return a.finch_c2 ? go<true, false, true, false>(a, stream) : go<false, false, true, false>(a, stream);
        case ChunkedMode::kBf16OutMoments:
            if (!a.finch_c2 || !a.moments) return hipErrorInvalidValue;
            return go<true, false, false, true>(a, stream);
        default:
            if (!a.y || !a.lambda || !a.bw) return hipErrorInvalidValue;
            if (mode == ChunkedMode::kBf16OutLora) return a.finch_c2 ? go<true, true, false, false>(a, stream) : go<false, true, false, false>(a, stream);
            if (!a.finch_c2 || !a.moments) return hipErrorInvalidValue;
            return go<true, true, false, true>(a, stream);
    }
}

}  // namespace wkv6

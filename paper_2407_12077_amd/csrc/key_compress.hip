// GOLD key compression for gfx950 (MI355X): c = x W^KD, a skinny bf16 GEMM (GOLD Key
// Compression: every token's hidden state of D channels times the D x D/16 matrix W^KD gives its
// compressed key-cache entry).  M tokens x D channels are streamed from HBM exactly once; W^KD
// (D x C, C = D/16, at most a few hundred KB) stays in the L2 of every XCD.  The kernel is bound
// by the HBM read of x; all arithmetic is on the matrix cores (v_mfma_f32_16x16x32_bf16, fp32
// accumulation, bf16 products are exact in fp32).
//
// Three kernels; the rules are at the launch.  With more large tiles than compute units: one workgroup
// owns 128 tokens x kBN output columns (kBN = 128 up to D = 2048, 256 above that if there are more tiles than
// compute units, so that up to D = 4096 a workgroup has all columns and x passes through a compute unit's vector
// memory path once; fewer columns in the last tile when D/16 is not a multiple of kBN) and walks the D
// axis in steps of 64 channels (cyclically, from a start that differs between workgroups).  Its
// waves split into two roles that meet at one barrier per step:
//   kBN/32 LOADER waves (the last ones): fetch the x tile (128 x 64: full 128-byte row pieces, 8
//               lanes each) and the W tile (64 x kBN, an L2 hit) of a step two (kBN = 128) or four
//               (kBN = 256) steps ahead into registers with
//               16-byte loads, and park the tiles of the next step in one of two LDS buffers.
//               Rows past M and steps past D go through shrunk raw buffer descriptors and read
//               as zero without touching memory, so no load is predicated and the wait counters
//               stay exact.
//   kBN/32 MFMA waves: each owns a 64 x 64 block of the result in accumulator
//               registers; per step 8 row reads of x (row stride 160 B: full-rate 16-byte LDS reads), 16
//               transposing reads of W (its contraction index is the tile's row) and 32 MFMAs.
//               They issue no global loads, so nothing but LDS latency sits between their MFMAs.
// With kBN = 128 registers and LDS are sized so that two workgroups share a compute unit: the
// waits, prologue and epilogue of one overlap the steady state of the other.  With kBN = 256 a
// compute unit holds one workgroup of sixteen waves, and its loaders keep four steps in flight
// instead (in-flight bytes, not arithmetic, limit this shape).
#include "wkv6_launch.h"
#include "wkv6_lds_loads.h"

namespace wkv6 {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef unsigned uint4v __attribute__((ext_vector_type(4)));

constexpr int kBM = 128;            // tokens per workgroup
constexpr int kBK = 64;             // channels per step
constexpr int kXRow = 160;          // LDS row stride of the x tile (64 bf16 + 32 B pad)
constexpr int kXTile = kBM * kXRow; // 20480
constexpr int kCRow = 128 * 4 + 16; // staging row of 128 columns of the fp32 result tile

// per width of the workgroup's column tile (kBN = 128 or 256)
constexpr int kWNB = 4;             // 16-column blocks of an MFMA wave
template <int kBN>
struct Tile {
    static constexpr int kWRow = kBN * 2 + 32;          // LDS row stride of the W tile (kBN bf16 + 32 B pad)
    static constexpr int kWTile = kBK * kWRow;
    static constexpr int kStage = kXTile + kWTile;
    static constexpr int kLds = 2 * kStage;
    static constexpr int kMfmaWaves = 2 * kBN / (16 * kWNB);     // blocks of 64 rows x 16 kWNB columns
    static constexpr int kLoaders = 2 * kBN;            // loader threads
    static constexpr int kThreads = 64 * kMfmaWaves + kLoaders;
    static constexpr int kXLoads = kBM * 8 / kLoaders;  // 16-byte loads per loader thread and step: x,
    static constexpr int kWLoads = kBK * kBN / 8 / kLoaders;   // W
    // steps a loader has in flight: two when two workgroups share a compute unit (they overlap each
    // other's waits), four when one workgroup has it alone
    static constexpr int kDepth = kBN == 128 ? 2 : 4;
    static constexpr int kPerCu = kBN == 128 ? 2 : 1;
    static constexpr int kHalves = kBN / 128;           // the result leaves through LDS 128 columns at a time
    static_assert(kLds >= kBM * kCRow, "result staging reuses the operand buffers");
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_of(const void* base, long long bytes) {
    if (bytes < 0) bytes = 0;
    if (bytes > 0x7fffffffLL) bytes = 0x7fffffffLL;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, static_cast<int>(bytes), 0x00020000);
}

__device__ __forceinline__ bf16x8 lds_read_b8(const char* lds, int off) {
    return *reinterpret_cast<const bf16x8*>(lds + off);
}

// 8 consecutive rows (contraction index) of one column of a row-major 16-bit tile, as an MFMA
// operand: two transposing reads of 4 rows each.  Within a group of 16 lanes, lane i passes the
// address of the 4 entries M[i>>2][4(i&3)..+3] of a 4 x 16 block and receives M[0..3][i].
template <int kWRow>
__device__ __forceinline__ bf16x8 lds_read_tr8(const char* lds, int off) {
    typedef short4v __attribute__((address_space(3))) * lds_s4_ptr;
    const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_ptr)(lds + off));
    const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_ptr)(lds + off + 4 * kWRow));
    typedef short short8v __attribute__((ext_vector_type(8)));
    const short8v both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, both);
}

struct KcArgs {
    long long M;
    int D, C;
    const void* x;
    const void* w;
    void* c;
};

template <typename TL>
struct StepRegs {          // a loader thread's share of one step, 16 bytes each
    uint4v x[TL::kXLoads], w[TL::kWLoads];
};

// ------------------------------------------------------------------------------------------
// loader waves (256 threads): tiles of step s+2 into registers, tiles of step s+1 into LDS
// ------------------------------------------------------------------------------------------
template <int kBN>
__device__ __forceinline__ void kc_loader(const KcArgs& a, char* lds, int lt, long long m0, int n0, int rows,
                                          int nsteps, int first) {
    using TL = Tile<kBN>;
    constexpr int kWRow = TL::kWRow, kStage = TL::kStage, kXLoads = TL::kXLoads, kWLoads = TL::kWLoads;
    constexpr int kXRowsPerPass = TL::kLoaders / 8;
    constexpr int kLanesPerWRow = kBN / 8, kWRowsPerPass = TL::kLoaders / kLanesPerWRow;
    const long long x_row_bytes = static_cast<long long>(a.D) * 2;
    const char* x_base = static_cast<const char*>(a.x) + m0 * x_row_bytes;
    const long long x_bytes = rows * x_row_bytes;
    const long long w_row_bytes = static_cast<long long>(a.C) * 2;
    const char* w_base = static_cast<const char*>(a.w);
    const long long w_bytes = static_cast<long long>(a.D) * w_row_bytes;

    // x tile: 8 lanes per 128-byte row piece; W tile: kBN/8 lanes per row piece of kBN columns
    const int xr = lt >> 3, xg = lt & 7;
    const int wr = lt / kLanesPerWRow, wg = lt % kLanesPerWRow;
    int x_voff[kXLoads], w_voff[kWLoads];
#pragma unroll
    for (int p = 0; p < kXLoads; ++p) x_voff[p] = static_cast<int>((xr + kXRowsPerPass * p) * x_row_bytes + 16 * xg);
#pragma unroll
    for (int p = 0; p < kWLoads; ++p)
        // columns past C (the last column tile may be partial): an offset no descriptor covers
        w_voff[p] = n0 + 8 * wg < a.C ? static_cast<int>((wr + kWRowsPerPass * p) * w_row_bytes + n0 * 2 + 16 * wg)
                                      : 0x7ffffff0;
    const int x_lds = xr * kXRow + 16 * xg;
    const int w_lds = kXTile + wr * kWRow + 16 * wg;

    auto fetch = [&](StepRegs<TL>& s, int step) {
        const bool live = step < nsteps;                                          // uniform
        int ks = step + first;                                                    // this step's channel block
        if (ks >= nsteps) ks -= nsteps;
        const long long xs = static_cast<long long>(ks) * kBK * 2;                // byte offset along a row of x
        const long long ws = static_cast<long long>(ks) * kBK * w_row_bytes;     // first W row of the step
        const __amdgpu_buffer_rsrc_t rx = rsrc_of(x_base + (live ? xs : 0), live ? x_bytes - xs : 0);
        const __amdgpu_buffer_rsrc_t rw = rsrc_of(w_base + (live ? ws : 0), live ? w_bytes - ws : 0);
#pragma unroll
        for (int p = 0; p < kWLoads; ++p)
            s.w[p] = __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(rw, w_voff[p], 0, 0));
#pragma unroll
        for (int p = 0; p < kXLoads; ++p)
            s.x[p] = __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(rx, x_voff[p], 0, 0));
    };
    auto park = [&](const StepRegs<TL>& s, int buf) {
        char* b = lds + buf * kStage;
#pragma unroll
        for (int p = 0; p < kXLoads; ++p) *reinterpret_cast<uint4v*>(b + x_lds + kXRowsPerPass * p * kXRow) = s.x[p];
#pragma unroll
        for (int p = 0; p < kWLoads; ++p) *reinterpret_cast<uint4v*>(b + w_lds + kWRowsPerPass * p * kWRow) = s.w[p];
    };

    // D / 64 steps, a multiple of four; one barrier per step, as many as the MFMA waves pass
    if constexpr (TL::kDepth == 2) {
        // the tiles of two steps in flight per workgroup, and two workgroups share a compute unit
        StepRegs<TL> s0, s1;
        fetch(s0, 0);
        fetch(s1, 1);
        park(s0, 0);
        fetch(s0, 2);
        __syncthreads();                               // tiles of step 0 are in LDS
#pragma clang loop unroll(disable)
        for (int step = 0; step < nsteps; step += 2) {
            park(s1, 1);                               // step+1, while the MFMA waves work on step
            fetch(s1, step + 3);
            __syncthreads();
            park(s0, 0);
            fetch(s0, step + 4);
            __syncthreads();
        }
    } else {
        // four steps in flight: with one workgroup per compute unit nothing else covers the latency
        StepRegs<TL> s0, s1, s2, s3;
        fetch(s0, 0);
        fetch(s1, 1);
        fetch(s2, 2);
        fetch(s3, 3);
        park(s0, 0);
        fetch(s0, 4);
        __syncthreads();                               // tiles of step 0 are in LDS
#pragma clang loop unroll(disable)
        for (int step = 0; step < nsteps; step += 4) {
            park(s1, 1);                               // step+1, while the MFMA waves work on step
            fetch(s1, step + 5);
            __syncthreads();
            park(s2, 0);
            fetch(s2, step + 6);
            __syncthreads();
            park(s3, 1);
            fetch(s3, step + 7);
            __syncthreads();
            park(s0, 0);
            fetch(s0, step + 8);
            __syncthreads();
        }
    }
    // the result tile leaves through LDS, 128 columns at a time: one barrier after each staging and
    // one before the next
#pragma unroll
    for (int i = 0; i < 2 * TL::kHalves - 1; ++i) __syncthreads();
}

// ------------------------------------------------------------------------------------------
// MFMA waves (256 threads)
// ------------------------------------------------------------------------------------------
template <int kBN, bool kOutF32>
__device__ __forceinline__ void kc_worker(const KcArgs& a, char* lds, int tid, int wave, long long m0, int n0,
                                          int rows, int nsteps) {
    using TL = Tile<kBN>;
    constexpr int kWRow = TL::kWRow, kStage = TL::kStage, kColBlocks = kBN / (16 * kWNB);
    const int lane = tid & 63;
    const int l16 = lane & 15;
    const int g4 = lane >> 4;
    // wave (wr, wc) owns rows 64 wr .. +63 and columns 16 kWNB wc ..: 4 x kWNB blocks of 16 x 16
    const int wr2 = wave / kColBlocks, wc2 = wave % kColBlocks;
    float4v acc[4][kWNB];
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
        for (int nb = 0; nb < kWNB; ++nb) acc[rb][nb] = float4v{0.f, 0.f, 0.f, 0.f};

    const int a_lane = (64 * wr2 + l16) * kXRow + 16 * g4;                                      // + 16*kXRow*rb + 64*kb
    const int b_lane = kXTile + (8 * g4 + (l16 >> 2)) * kWRow + 8 * (l16 & 3) + 32 * kWNB * wc2;     // + 32*kWRow*kb + 32*nb
    auto compute = [&](int buf) {
        const char* b = lds + buf * kStage;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            bf16x8 av[4], wt[kWNB];
#pragma unroll
            for (int rb = 0; rb < 4; ++rb) av[rb] = lds_read_b8(b, a_lane + 16 * kXRow * rb + 64 * kb);
#pragma unroll
            for (int nb = 0; nb < kWNB; ++nb) wt[nb] = lds_read_tr8<kWRow>(b, b_lane + 32 * kWRow * kb + 32 * nb);
#pragma unroll
            for (int rb = 0; rb < 4; ++rb)
#pragma unroll
                for (int nb = 0; nb < kWNB; ++nb)
                    acc[rb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[rb], wt[nb], acc[rb][nb], 0, 0, 0);
        }
    };

    __syncthreads();                                   // tiles of step 0 are in LDS
#pragma clang loop unroll(disable)
    for (int step = 0; step < nsteps; step += 2) {
        compute(0);
        __syncthreads();
        compute(1);
        __syncthreads();
    }

    // result tile through LDS (fp32, row stride kCRow, 128 columns at a time), then full rows to HBM
    constexpr int kRowsPerPass = 64 * TL::kMfmaWaves / 8;          // 8 lanes per row, 16 columns each
    const int cr = tid >> 3, cg = tid & 7;
#pragma unroll
    for (int hf = 0; hf < TL::kHalves; ++hf) {
        if (hf > 0) __syncthreads();                               // the previous half has been read
        if (16 * kWNB * wc2 / 128 == hf) {
#pragma unroll
            for (int rb = 0; rb < 4; ++rb)
#pragma unroll
                for (int nb = 0; nb < kWNB; ++nb)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        *reinterpret_cast<float*>(lds + (64 * wr2 + 16 * rb + 4 * g4 + e) * kCRow +
                                                  (16 * kWNB * wc2 % 128 + 16 * nb + l16) * 4) = acc[rb][nb][e];
        }
        __syncthreads();
        // A row's eight threads store one whole 128-byte line per instruction: thread cg takes the
        // cg-th 16 bytes of every line of the row's 128-column piece (2 lines in bf16, 4 in fp32).
        constexpr int kColsPerStore = kOutF32 ? 4 : 8, kLines = 128 / (8 * kColsPerStore);
#pragma unroll
        for (int p = 0; p < kBM / kRowsPerPass; ++p) {
            const int row = cr + kRowsPerPass * p;
            if (row >= rows) continue;
#pragma unroll
            for (int ln = 0; ln < kLines; ++ln) {
                const int lc = 8 * kColsPerStore * ln + kColsPerStore * cg;      // column within the piece
                const int col = n0 + 128 * hf + lc;
                if (col >= a.C) continue;
                const float4* src = reinterpret_cast<const float4*>(lds + row * kCRow + lc * 4);
                const long long e = (m0 + row) * a.C + col;
                if constexpr (kOutF32) {
                    *reinterpret_cast<float4*>(static_cast<float*>(a.c) + e) = src[0];
                } else {
                    auto pk = [](float lo, float hi) {
                        return static_cast<unsigned>(__builtin_bit_cast(unsigned short, static_cast<__bf16>(lo))) |
                               (static_cast<unsigned>(__builtin_bit_cast(unsigned short, static_cast<__bf16>(hi))) << 16);
                    };
                    const float4 q0 = src[0], q1 = src[1];
                    *reinterpret_cast<uint4*>(static_cast<unsigned short*>(a.c) + e) =
                        make_uint4(pk(q0.x, q0.y), pk(q0.z, q0.w), pk(q1.x, q1.y), pk(q1.z, q1.w));
                }
            }
        }
    }
}

template <bool kOutF32, int kBN>
__device__ __forceinline__ void kc_roles(const KcArgs& a, char* lds) {
    using TL = Tile<kBN>;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Block -> tile map.  With more than one column tile (D > 16 kBN: 2048 or 4096) the column tiles of one row tile
    // must meet in the same L2 so that x comes from HBM once: consecutive block ids go round the
    // 8 XCDs, so the id is read as (slot, xcd) and the column tiles of a row tile take consecutive
    // slots of one XCD.
    const int nct = (a.C + kBN - 1) / kBN;
    const int xcd = blockIdx.x & 7;
    const int slot = blockIdx.x >> 3;
    const long long row_tile = static_cast<long long>(slot / nct) * 8 + xcd;
    const long long m0 = row_tile * kBM;
    const int n0 = (slot % nct) * kBN;
    if (m0 >= a.M) return;                     // padding of the row tiles to a multiple of 8
    const long long rows_left = a.M - m0;
    const int rows = rows_left < kBM ? static_cast<int>(rows_left) : kBM;
    const int nsteps = a.D / kBK;
    // Every workgroup walks all channel blocks, but starts at a different one (the column tiles of
    // a row tile at the same one): the rows of x are D*2 bytes apart, so workgroups that march
    // through the channels in step would all ask the same few memory channels for their 128-byte
    // row pieces, and the same L2 channel for the same rows of W (config 2's width: 127 -> 113 us).
    const int first = static_cast<int>((slot / nct + 4 * xcd) % nsteps);
    // both roles pass 1 + nsteps + 2 kHalves - 1 barriers
    // the loaders' few instructions per step go ahead of the MFMA waves' long streams (wave
    // priority is an issue-arbitration hint): measured 2-3 % on the benchmark shapes
    if (wave >= TL::kMfmaWaves) {
        __builtin_amdgcn_s_setprio(2);
        kc_loader<kBN>(a, lds, tid - 64 * TL::kMfmaWaves, m0, n0, rows, nsteps, first);
    } else {
        __builtin_amdgcn_s_setprio(1);
        kc_worker<kBN, kOutF32>(a, lds, tid, wave, m0, n0, rows, nsteps);
    }
}

// ------------------------------------------------------------------------------------------
// At most one large tile per compute unit: loads straight into LDS, all waves load and multiply
// ------------------------------------------------------------------------------------------
// A workgroup owns kRowTile tokens x 128 columns and walks D in steps of 64 channels, cyclically from a start of its own.  Its eight waves each
// bring an eighth of a step's x and W tiles straight into LDS, two steps ahead, and multiply: four waves the first 32 channels of a step,
// four the second, 32 columns each, so that a step's x is read from LDS four times and its W once.  One barrier a step.  No registers hold loads
// on their way and no LDS stores stand in the way of the operand reads.  What bounds it at 16 384 tokens and D = 2048 (15.0 us; the 67 MB of x
// alone take 13 at the copy rate): what a compute unit takes in, 768 KB of x and W.
template <int kRowTile>
struct DmaTile {
    static constexpr int kX = kRowTile * 128, kStage = kX + 64 * 256;
    // steps in LDS: with as many as fit the first one begins later (5 to 10 % slower)
    static constexpr int kStages = 3;
    static constexpr int kXLoads = kRowTile / 64, kLoads = kXLoads + 2;      // of a wave and step
    static constexpr int kRB = kRowTile / 16;                               // 16-row blocks
    static constexpr int kPRow = 128 + 4;                                   // row stride (floats) of the two partial results
    static constexpr int kLds = kStages * kStage > 2 * kRowTile * kPRow * 4 ? kStages * kStage : 2 * kRowTile * kPRow * 4;
    static_assert(kLds <= 160 * 1024 && kLoads * (kStages - 2) < 64, "LDS budget, vmcnt");
};

// kCount operands as lds_read_tr8 reads them, from the byte offsets of their first four rows behind `base`, the next four kHi bytes further; waits for all
// LDS accesses of the wave.  (Before the builtin the compiler waits for every load into LDS.)
template <int kCount, int kHi = 4 * 32 * kCount>
__device__ __forceinline__ void lds_read_tr8_all(__attribute__((address_space(3))) const char* base, const int (&off)[kCount], bf16x8 (&q)[kCount]) {
#if defined(__HIP_DEVICE_COMPILE__)
    typedef short short8v __attribute__((ext_vector_type(8)));
    unsigned p[kCount];
    short4v lo[kCount], hi[kCount];
#pragma unroll
    for (int i = 0; i < kCount; ++i) p[i] = static_cast<unsigned>(reinterpret_cast<unsigned long long>(base)) + off[i];
    if constexpr (kCount == 1) {
        asm volatile("ds_read_b64_tr_b16 %0, %2\n\tds_read_b64_tr_b16 %1, %2 offset:%3\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(lo[0]), "=&v"(hi[0]) : "v"(p[0]), "n"(kHi) : "memory");
    } else if constexpr (kCount == 2) {
        asm volatile("ds_read_b64_tr_b16 %0, %4\n\tds_read_b64_tr_b16 %1, %4 offset:%6\n\t"
                     "ds_read_b64_tr_b16 %2, %5\n\tds_read_b64_tr_b16 %3, %5 offset:%6\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(lo[0]), "=&v"(hi[0]), "=&v"(lo[1]), "=&v"(hi[1]) : "v"(p[0]), "v"(p[1]), "n"(kHi) : "memory");
    } else {
        static_assert(kCount == 4, "1, 2 or 4 operands");
        asm volatile("ds_read_b64_tr_b16 %0, %8\n\tds_read_b64_tr_b16 %1, %8 offset:%12\n\t"
                     "ds_read_b64_tr_b16 %2, %9\n\tds_read_b64_tr_b16 %3, %9 offset:%12\n\t"
                     "ds_read_b64_tr_b16 %4, %10\n\tds_read_b64_tr_b16 %5, %10 offset:%12\n\t"
                     "ds_read_b64_tr_b16 %6, %11\n\tds_read_b64_tr_b16 %7, %11 offset:%12\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(lo[0]), "=&v"(hi[0]), "=&v"(lo[1]), "=&v"(hi[1]), "=&v"(lo[2]), "=&v"(hi[2]), "=&v"(lo[3]), "=&v"(hi[3])
                     : "v"(p[0]), "v"(p[1]), "v"(p[2]), "v"(p[3]), "n"(kHi) : "memory");
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < kCount; ++i) {
        const short8v both = __builtin_shufflevector(lo[i], hi[i], 0, 1, 2, 3, 4, 5, 6, 7);
        q[i] = __builtin_bit_cast(bf16x8, both);
    }
#endif
}

template <bool kOutF32, int kRowTile>
__device__ __forceinline__ void kc_direct(const KcArgs& a, char* lds) {
    using TL = DmaTile<kRowTile>;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // the column tiles of a row tile in consecutive slots of one XCD, as above
    const int nct = (a.C + 127) / 128;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const long long m0 = (static_cast<long long>(slot / nct) * 8 + xcd) * kRowTile;
    const int n0 = slot % nct * 128;
    if (m0 >= a.M) return;                     // padding of the row tiles to a multiple of 8
    const int rows = a.M - m0 < kRowTile ? static_cast<int>(a.M - m0) : kRowTile;
    const int nsteps = a.D / kBK;
    int at = (slot / nct + 4 * xcd) % nsteps;  // the channel block asked for next

    // A load brings 1 KiB: lane i's 16 bytes lie 16 i behind the wave's LDS address.  x: eight rows of 128 bytes, the granule of a row r at
    // place (granule ^ (r >> 1 & 7)); W: four rows k of 256 bytes, the 32-byte pair p of a row at place p ^ (k & 3 | k >> 1 & 4).  With these the
    // reads of an operand, sixteen rows at one granule or pair, take every bank equally often.  Rows past the end of x are the last one again, columns
    // past C lie at an offset that no descriptor covers: their results are not stored.
    const int x_row_bytes = a.D * 2, w_row_bytes = a.C * 2;
    const char* x_base = static_cast<const char*>(a.x) + m0 * x_row_bytes;
    int x_voff[TL::kXLoads], w_voff[2];
#pragma unroll
    for (int p = 0; p < TL::kXLoads; ++p) {
        const int r = 8 * (wave + 8 * p) + (lane >> 3);
        x_voff[p] = (r < rows ? r : rows - 1) * x_row_bytes + 16 * ((lane & 7) ^ (r >> 1 & 7));
    }
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int k = 4 * (wave + 8 * p) + (lane >> 4);
        const int col = n0 + 16 * ((lane & 15) >> 1 ^ ((k & 3) | (k >> 1 & 4))) + 8 * (lane & 1);
        w_voff[p] = col < a.C ? k * w_row_bytes + col * 2 : 0x7ffffff0;
    }
    typedef __attribute__((address_space(3))) char* lds_ptr;
    const __amdgpu_buffer_rsrc_t rx = rsrc_of(x_base, static_cast<long long>(rows) * x_row_bytes);
    const __amdgpu_buffer_rsrc_t rw = rsrc_of(a.w, static_cast<long long>(a.D) * w_row_bytes);
    auto ask = [&](int place) {
        const int to = place * TL::kStage + 1024 * wave;
#pragma unroll
        for (int p = 0; p < 2; ++p)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_ptr)(lds + to + TL::kX + 8192 * p), 16, w_voff[p], at * (kBK * w_row_bytes), 0, 0);
#pragma unroll
        for (int p = 0; p < TL::kXLoads; ++p)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_ptr)(lds + to + 8192 * p), 16, x_voff[p], at * (kBK * 2), 0, 0);
        at = at + 1 == nsteps ? 0 : at + 1;
    };

    const int kb = wave >> 2, wc = wave & 3;   // this wave's half of a step's channels, and its 32 columns
    // rows l16 and 16 + l16 (the others 32 rows further); columns 16 nb, channels 8 g4 .. +3 (the next four 1024 further)
    int a_off[2], b_off[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int r = 16 * i + l16;
        a_off[i] = r * 128 + 16 * ((4 * kb + g4) ^ (r >> 1 & 7));
    }
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
        const int k = 32 * kb + 8 * g4 + (l16 >> 2);
        b_off[nb] = TL::kX + k * 256 + 32 * ((2 * wc + nb) ^ ((k & 3) | (k >> 1 & 4))) + 8 * (l16 & 3);
    }
    float4v acc[TL::kRB][2];
#pragma unroll
    for (int rb = 0; rb < TL::kRB; ++rb) acc[rb][0] = acc[rb][1] = float4v{0.f, 0.f, 0.f, 0.f};

    int asked = 0;
    // (D >= 256: there are more steps than places.  With a constant count here the loop below is compiled to a slower one: 6900 x 2048 12.8 ->
    // 13.0 us, 6900 x 4096 22.8 -> 23.3.)
    for (; asked < TL::kStages - 1 && asked < nsteps; ++asked) ask(asked);
    int place = 0, free_place = TL::kStages - 1;
#pragma clang loop unroll(disable)
    for (int step = 0; step < nsteps; ++step) {
        if (asked - step == TL::kStages - 1) wait_loads<TL::kLoads * (TL::kStages - 2)>();     // the younger steps are on their way
        else wait_loads<0>();
        __builtin_amdgcn_s_barrier();          // the step's tiles are there, and all waves are done with the place of the one before
        __builtin_amdgcn_sched_barrier(0);
        if (asked < nsteps) {
            ask(free_place);
            ++asked;
        }
        free_place = place;
        const char* b = lds + place * TL::kStage;
        place = place + 1 == TL::kStages ? 0 : place + 1;
        if (n0 + 32 * wc >= a.C) continue;     // no columns: the wave only loads
        bf16x8 av[TL::kRB];
#pragma unroll
        for (int rb = 0; rb < TL::kRB; ++rb) av[rb] = lds_read_b8(b, a_off[rb & 1] + 4096 * (rb >> 1));
        bf16x8 wt[2];
        lds_read_tr8_all<2, 1024>((lds_ptr)b, b_off, wt);      // with a wait for all of the step's LDS reads: after the next barrier its place is free
#pragma unroll
        for (int rb = 0; rb < TL::kRB; ++rb)
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)     // columns as the rows of the product: a lane ends with four neighbouring columns of its token
                acc[rb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wt[nb], av[rb], acc[rb][nb], 0, 0, 0);
    }

    // the two halves meet in LDS; whole rows leave
    __syncthreads();
    float* part = reinterpret_cast<float*>(lds);
#pragma unroll
    for (int rb = 0; rb < TL::kRB; ++rb)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
            *reinterpret_cast<float4v*>(part + (kb * kRowTile + 16 * rb + l16) * TL::kPRow + 32 * wc + 16 * nb + 4 * g4) = acc[rb][nb];
    __syncthreads();
    constexpr int kPer = kOutF32 ? 4 : 8, kLanes = 128 / kPer;   // columns of a thread's 16 bytes, threads of a row
    const int cr = tid / kLanes, col = tid % kLanes * kPer;
    if (n0 + col >= a.C) return;
#pragma unroll
    for (int p = 0; p < kRowTile * kLanes / 512; ++p) {
        const int row = cr + 512 / kLanes * p;
        if (row >= rows) break;
        float4v q[kPer / 4];
#pragma unroll
        for (int i = 0; i < kPer / 4; ++i)
            q[i] = *reinterpret_cast<const float4v*>(part + row * TL::kPRow + col + 4 * i) +
                   *reinterpret_cast<const float4v*>(part + (kRowTile + row) * TL::kPRow + col + 4 * i);
        const long long e = (m0 + row) * a.C + n0 + col;
        if constexpr (kOutF32) {
            *reinterpret_cast<float4v*>(static_cast<float*>(a.c) + e) = q[0];
        } else {
            typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
            typedef unsigned uint2v __attribute__((ext_vector_type(2)));
            const uint2v lo = __builtin_bit_cast(uint2v, __builtin_convertvector(q[0], bf16x4));
            const uint2v hi = __builtin_bit_cast(uint2v, __builtin_convertvector(q[1], bf16x4));
            *reinterpret_cast<uint4v*>(static_cast<unsigned short*>(a.c) + e) = uint4v{lo[0], lo[1], hi[0], hi[1]};
        }
    }
}

// The two kernels behind one name: kForm 4 with loader waves and 128 tokens (Tile), kForm 2 with all waves alike, 64 or 128 tokens (DmaTile).
constexpr int kLoaderWaves = 4, kWavesAlike = 2;
template <int kBN, int kForm, bool kOutF32, int kRowTile>
__global__ __launch_bounds__(kForm == kWavesAlike ? 512 : Tile<kBN>::kThreads, kForm == kWavesAlike ? 128 / kRowTile : Tile<kBN>::kPerCu)
void key_compress_kernel(KcArgs a) {
    static_assert(kForm == kWavesAlike ? kBN == 128 : kForm == kLoaderWaves && kRowTile == kBM, "forms");
    extern __shared__ __attribute__((aligned(16))) char lds[];
    if constexpr (kForm == kWavesAlike) kc_direct<kOutF32, kRowTile>(a, lds);
    else kc_roles<kOutF32, kBN>(a, lds);
}

// ------------------------------------------------------------------------------------------
// Few tokens (a decode batch, short prompts): the contraction split over the waves.  Bound by latency up to a
// few hundred tokens (launch, two rounds of loads, the reduction: 3.7 to 5.6 us), then by W through L2.
// ------------------------------------------------------------------------------------------
// The tiles above need 64 tokens per workgroup to be worth their loads: with a few row tiles most
// compute units have nothing to do and the others walk D / 64 dependent steps.  Here a workgroup owns a
// small tile, 16 kTB tokens x 16 kNB columns, and its sixteen waves take the 32-channel blocks of D in
// turn (wave w: blocks w, w + 16, ...), so that a walk is D / 512 steps long and needs no barrier: a wave brings its x and W blocks straight into a
// piece of LDS of its own, W kAhead blocks ahead and x one more (x loaded into operand layout from global memory touches sixteen lines per quarter
// wave, which the L1's tag lookups charge four times), and reads them from there as operands.  The sixteen partial results are added in
// wave order, in fp32, at the end.  Through registers and LDS stores, two blocks ahead of both, the same sums took longer: D = 2048, 24
// tokens 4.55 us against 3.85 now, 2048 tokens 7.4 against 6.3, 4096 11.7 against 10.5, 6500 19.0 against 16.7; D = 768 3000 tokens
// 4.8 against 3.7; D = 4096 16 tokens 6.0 against 5.1.
constexpr int kFewWaves = 16;

template <int kTB, int kNB>
struct FewTile {
    static constexpr int kX = 1024 * kTB, kW = 1024 * kNB;                  // bytes of a block: rows of 64 bytes; 32 rows of 32 kNB bytes
    static constexpr int kAhead = kNB == 4 ? 1 : 2;                         // places for W blocks; one more for x
    static constexpr int kPiece = (kAhead + 1) * kX + kAhead * kW;
    static constexpr int kPRow = 16 * kNB + 4;          // row stride (floats) of a wave's partial result
    static constexpr int kPart = 16 * kTB * kPRow;      // floats per wave
    static constexpr int kWBytes = kFewWaves * kPiece, kPBytes = kFewWaves * kPart * 4;
    static constexpr int kLds = kWBytes > kPBytes ? kWBytes : kPBytes;
    static_assert(kLds <= 160 * 1024, "LDS budget");
};

template <int kTB, int kNB, bool kOutF32>
__device__ __forceinline__ void kc_few(const KcArgs& a, char* lds) {
    using TL = FewTile<kTB, kNB>;
    constexpr int kA = TL::kAhead;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nct = (a.C + 16 * kNB - 1) / (16 * kNB);
    const long long m0 = static_cast<long long>(blockIdx.x / nct) * (16 * kTB);
    const int n0 = static_cast<int>(blockIdx.x % nct) * (16 * kNB);
    const int rows = a.M - m0 < 16 * kTB ? static_cast<int>(a.M - m0) : 16 * kTB;
    const int x_row_bytes = a.D * 2, w_row_bytes = a.C * 2;
    const int nkb = a.D / 32, mine = wave < nkb ? (nkb - 1 - wave) / kFewWaves + 1 : 0;     // this wave's blocks

    // A load brings 1 KiB, lane i's 16 bytes 16 i behind the wave's LDS address.  x: sixteen rows, granules XOR-ed by two row bits; W: rows of kNB
    // 32-byte pairs, the pairs XOR-ed by row bits, so that the reads of an operand take every bank equally often.  Rows past the end are
    // the last one again, columns past C lie at an offset that no descriptor covers: their results are not stored.
    typedef __attribute__((address_space(3))) char* lds_ptr;
    auto pair_of = [](int k) { return kNB == 4 ? (k >> 1 & 1) | (k >> 2 & 2) : kNB == 2 ? k >> 3 & 1 : 0; };
    int x_voff[kTB], w_voff[kNB];
#pragma unroll
    for (int tb = 0; tb < kTB; ++tb) {
        const int r = 16 * tb + (lane >> 2);
        x_voff[tb] = (r < rows ? r : rows - 1) * x_row_bytes + 16 * ((lane & 3) ^ (r >> 2 & 3));
    }
#pragma unroll
    for (int nb = 0; nb < kNB; ++nb) {
        const int k = (64 * nb + lane) / (2 * kNB), at = lane % (2 * kNB);
        const int col = n0 + 16 * (at >> 1 ^ pair_of(k)) + 8 * (at & 1);
        w_voff[nb] = col < a.C ? k * w_row_bytes + col * 2 : 0x7ffffff0;
    }
    const char* x_base = static_cast<const char*>(a.x) + m0 * x_row_bytes;
    const __amdgpu_buffer_rsrc_t rx = rsrc_of(x_base, static_cast<long long>(rows) * x_row_bytes);
    const int piece = wave * TL::kPiece;
    auto x_place = [&](int i) { return piece + i % (kA + 1) * TL::kX; };
    auto w_place = [&](int i) { return piece + (kA + 1) * TL::kX + i % kA * TL::kW; };
    auto ask_x = [&](int i) {
        if (i >= mine) return;
#pragma unroll
        for (int tb = 0; tb < kTB; ++tb)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_ptr)(lds + x_place(i) + 1024 * tb), 16, x_voff[tb], (wave + i * kFewWaves) * 64, 0, 0);
    };
    auto ask_w = [&](int i) {
        if (i >= mine) return;
        const long long ws = static_cast<long long>(wave + i * kFewWaves) * 32 * w_row_bytes;
        const __amdgpu_buffer_rsrc_t rw = rsrc_of(static_cast<const char*>(a.w) + ws, 32 * w_row_bytes);
#pragma unroll
        for (int nb = 0; nb < kNB; ++nb)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_ptr)(lds + w_place(i) + 1024 * nb), 16, w_voff[nb], 0, 0, 0);
    };
    ask_x(0);
#pragma clang loop unroll(disable)
    for (int i = 0; i < kA; ++i) {
        ask_w(i);
        ask_x(i + 1);
    }

    float4v acc[kTB][kNB];
#pragma unroll
    for (int tb = 0; tb < kTB; ++tb)
#pragma unroll
        for (int nb = 0; nb < kNB; ++nb) acc[tb][nb] = float4v{0.f, 0.f, 0.f, 0.f};
    const int a_off = 64 * l16 + 16 * (g4 ^ (l16 >> 2 & 3));
    const int k0 = 8 * g4 + (l16 >> 2);                  // this lane's row of W, and the one four further (the same pair_of)
    int b_off[kNB];
#pragma unroll
    for (int nb = 0; nb < kNB; ++nb) b_off[nb] = k0 * 32 * kNB + 32 * (nb ^ pair_of(k0)) + 8 * (l16 & 3);
#pragma clang loop unroll(disable)
    for (int i = 0; i < mine; ++i) {
        // behind block i's W: the x of the next block and what follows
        if (i + kA < mine) wait_loads<(kA - 1) * kNB + kA * kTB>();
        else wait_loads<0>();
        bf16x8 xv[kTB], wt[kNB];
#pragma unroll
        for (int tb = 0; tb < kTB; ++tb) xv[tb] = lds_read_b8(lds + x_place(i), a_off + 1024 * tb);
        lds_read_tr8_all<kNB>((lds_ptr)(lds + w_place(i)), b_off, wt);      // (and a wait for all LDS reads: the places are free)
        ask_w(i + kA);
        ask_x(i + kA + 1);
#pragma unroll
        for (int nb = 0; nb < kNB; ++nb)
#pragma unroll
            for (int tb = 0; tb < kTB; ++tb)   // columns as the rows of the product: a lane ends with four neighbouring columns of its token
                acc[tb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wt[nb], xv[tb], acc[tb][nb], 0, 0, 0);
    }

    // the partial results meet in LDS
    float* part = reinterpret_cast<float*>(lds);
    __syncthreads();                                   // every wave is done with its W blocks
#pragma unroll
    for (int tb = 0; tb < kTB; ++tb)
#pragma unroll
        for (int nb = 0; nb < kNB; ++nb)
            *reinterpret_cast<float4v*>(part + wave * TL::kPart + (16 * tb + l16) * TL::kPRow + 16 * nb + 4 * g4) = acc[tb][nb];
    __syncthreads();
    constexpr int kPairs = 16 * kTB * 8 * kNB;         // two neighbouring columns per thread
    for (int i = tid; i < kPairs; i += 64 * kFewWaves) {
        const int row = i / (8 * kNB), col = 2 * (i % (8 * kNB));
        const float* src = part + row * TL::kPRow + col;
        float lo = 0.f, hi = 0.f;
#pragma unroll
        for (int w = 0; w < kFewWaves; ++w) {
            const float2 p = *reinterpret_cast<const float2*>(src + w * TL::kPart);
            lo += p.x;
            hi += p.y;
        }
        if (row < rows && n0 + col < a.C) {            // C is a multiple of 16
            const long long e = (m0 + row) * a.C + n0 + col;
            if constexpr (kOutF32)
                *reinterpret_cast<float2*>(static_cast<float*>(a.c) + e) = make_float2(lo, hi);
            else
                *reinterpret_cast<unsigned*>(static_cast<unsigned short*>(a.c) + e) =
                    static_cast<unsigned>(__builtin_bit_cast(unsigned short, static_cast<__bf16>(lo))) |
                    (static_cast<unsigned>(__builtin_bit_cast(unsigned short, static_cast<__bf16>(hi))) << 16);
        }
    }
}

template <int kTB, int kNB, bool kOutF32>
__global__ __launch_bounds__(64 * kFewWaves) void key_compress_few_kernel(KcArgs a) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    kc_few<kTB, kNB, kOutF32>(a, lds);
}

}  // namespace

namespace {

template <int kTB, int kNB, bool kOutF32>
hipError_t launch_few(const KcArgs& a, hipStream_t stream) {
    using TL = FewTile<kTB, kNB>;
    const long long row_tiles = (a.M + 16 * kTB - 1) / (16 * kTB);
    const dim3 grid(static_cast<unsigned>(row_tiles * ((a.C + 16 * kNB - 1) / (16 * kNB))));
    hipLaunchKernelGGL((key_compress_few_kernel<kTB, kNB, kOutF32>), grid, dim3(64 * kFewWaves), TL::kLds, stream, a);
    return hipGetLastError();
}

template <int kBN, int kForm, int kRowTile = kBM>
hipError_t launch_tile(const KcArgs& a, bool out_f32, hipStream_t stream) {
    constexpr bool kAlike = kForm == kWavesAlike;
    const long long row_tiles = (a.M + kRowTile - 1) / kRowTile;
    const dim3 grid(static_cast<unsigned>((row_tiles + 7) / 8 * 8 * ((a.C + kBN - 1) / kBN)));
    const auto kernel = out_f32 ? &key_compress_kernel<kBN, kForm, true, kRowTile> : &key_compress_kernel<kBN, kForm, false, kRowTile>;
    hipLaunchKernelGGL(kernel, grid, dim3(kAlike ? 512 : Tile<kBN>::kThreads), kAlike ? DmaTile<kRowTile>::kLds : Tile<kBN>::kLds, stream, a);
    return hipGetLastError();
}

}  // namespace

namespace {

template <bool kOutF32>
hipError_t raise_lds_limits() {
    hipError_t err = set_lds_limit(&key_compress_few_kernel<1, 1, kOutF32>, FewTile<1, 1>::kLds);
    if (err == hipSuccess) err = set_lds_limit(&key_compress_few_kernel<1, 2, kOutF32>, FewTile<1, 2>::kLds);
    if (err == hipSuccess) err = set_lds_limit(&key_compress_few_kernel<1, 4, kOutF32>, FewTile<1, 4>::kLds);
    if (err == hipSuccess) err = set_lds_limit(&key_compress_few_kernel<2, 4, kOutF32>, FewTile<2, 4>::kLds);
    if (err == hipSuccess) err = set_lds_limit(&key_compress_kernel<128, kLoaderWaves, kOutF32, kBM>, Tile<128>::kLds);
    if (err == hipSuccess) err = set_lds_limit(&key_compress_kernel<256, kLoaderWaves, kOutF32, kBM>, Tile<256>::kLds);
    if (err == hipSuccess) err = set_lds_limit(&key_compress_kernel<128, kWavesAlike, kOutF32, 64>, DmaTile<64>::kLds);
    if (err == hipSuccess) err = set_lds_limit(&key_compress_kernel<128, kWavesAlike, kOutF32, 128>, DmaTile<128>::kLds);
    return err;
}

}  // namespace

hipError_t launch_key_compress(long long M, int D, const void* x, const void* w, void* c, bool out_f32,
                               hipStream_t stream) {
    KcArgs a;
    a.M = M; a.D = D; a.C = D / 16;
    a.x = x; a.w = w; a.c = c;
    struct Tag {};
    const hipError_t err = once_per_device<Tag>([] {
        const hipError_t e = raise_lds_limits<false>();
        return e == hipSuccess ? raise_lds_limits<true>() : e;
    });
    if (err != hipSuccess) return err;
    // The contraction-split form while it fits the chip once: then a call takes as long as one workgroup, and
    // its walk of D / 512 steps is shorter than the D / 64 of the large tiles.  The smallest tile that still
    // gives at most one workgroup per compute unit, since a workgroup's time grows with its tile.  Measured, D
    // = 2048, microseconds, large tiles -> this form: 19.7 -> 4.4 at 1 token, 20.9 -> 5.2 at 512, 21.0 -> 5.5 at
    // 1024, 21.0 -> 6.3 at 2048, 21.0 -> 10.6 at 4096 (256 workgroups of the largest tile); D = 1024: 11.5 -> 3.8 at 16 tokens, 12.3
    // -> 5.7 at 8192.  From D = 2048 on a large tile's walk is so long that further rounds of these won, or tied, against the tiles with
    // loader waves, which took these calls when the lines were drawn: up to five thirds of a round at D = 2048 (6700 tokens 19.8 against
    // 20.1, 7200 20.4 against 20.1), wider models the whole second round (4096 x 4096 33.6 against 36.4).
    // Beyond the first round the 64-token tiles below, with all waves alike, are the faster ones now.  These : those, with x in the
    // caches and from HBM: D = 2048, 4097 tokens 14.4 : 12.8 and 16.4 : 16.7, 5000 15.1 : 12.9 and 19.9 : 17.0, 6816 17.1 : 13.1 and 20.7 : 17.6;
    // D = 2304, 3000 17.3 : 14.1 and 21.0 : 16.9; D = 3072, 5000 22.1 : 18.1 and 26.6 : 22.3; D = 4096, 2049 24.1 : 22.5 and 26.8 : 27.9,
    // 4096 31.8 : 23.0 and 35.5 : 29.2.  But sixteen short sums are closer to 64 bits than two long ones, 0.98e-7 : 1.87e-7 at D =
    // 2048, 1.02e-7 : 1.99e-7 at 2304, 1.15e-7 : 2.72e-7 at 4096 (2-norm), so the lines stay for the precision: no call is moved to less.
    const int cus = compute_units();
    auto groups = [&](int tb, int nb) {
        return (M + 16 * tb - 1) / (16 * tb) * ((a.C + 16 * nb - 1) / (16 * nb));
    };
    if (groups(1, 1) <= cus) return out_f32 ? launch_few<1, 1, true>(a, stream) : launch_few<1, 1, false>(a, stream);
    if (groups(1, 2) <= cus) return out_f32 ? launch_few<1, 2, true>(a, stream) : launch_few<1, 2, false>(a, stream);
    if (groups(1, 4) <= cus) return out_f32 ? launch_few<1, 4, true>(a, stream) : launch_few<1, 4, false>(a, stream);
    if (3 * groups(2, 4) <= (a.C > 128 ? 6 : a.C == 128 ? 5 : 3) * cus)
        return out_f32 ? launch_few<2, 4, true>(a, stream) : launch_few<2, 4, false>(a, stream);
    // At most one large tile per compute unit: 128 columns a tile, also above D = 2048 (x then comes from L2 the second time), loads
    // straight into LDS by all waves, 64 tokens a tile while these fit the chip once (twice with at most 64 columns, whose tiles share a compute
    // unit), which doubles the compute units of the shorter calls.  Microseconds, loader waves and 128 tokens -> here: D = 2048, 7000 tokens
    // 20.3 -> 13.3, 16 384 20.8 -> 15.0, with 128 tokens a tile 17 000 20.9 -> 19.0, 20 000 22.7 -> 21.8, 32 768 30.1 -> 29.4; D = 4096 5000 36.7 -> 24.0,
    // 8192 37.1 -> 24.7, 16 000 47.5 -> 45.4; D = 1024 12 000 11.8 -> 8.4, 20 000 12.2 -> 10.6, D = 768 30 000 10.9 -> 10.1.  64 tokens a tile in two rounds
    // take all of W again: D = 2048 20 000 27.2, 32 768 36.9.  Beyond, two workgroups of loader waves share a compute unit and overlap: 131 072
    // tokens 114 against 119 (128 tokens a tile), D = 1024 57 against 58 (64), D = 4096 65 536 160 against 226, D = 256 500 000 60 against 70.
    // (The direct form addresses W with 32 bits.)
    if (D <= 32768) {
        const long long col_tiles = (a.C + 127) / 128;
        if ((M + 63) / 64 * col_tiles <= (a.C <= 64 ? 2 : 1) * cus) return launch_tile<128, kWavesAlike, 64>(a, out_f32, stream);
        if ((M + 127) / 128 * col_tiles <= cus) return launch_tile<128, kWavesAlike, 128>(a, out_f32, stream);
    }
    return a.C > 128 ? launch_tile<256, kLoaderWaves>(a, out_f32, stream) : launch_tile<128, kLoaderWaves>(a, out_f32, stream);
}

}  // namespace wkv6

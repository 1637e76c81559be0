// W4A4 MXFP4 GEMM (the Q(X^) . Q(W^) product of the paper's Eq. 5) for operands in the tiled layout, on gfx950's
// block-scaled matrix cores (v_mfma_scale_f32_32x32x64_f8f6f4, FP4 x FP4): one kernel, a family of tile shapes.
//
// Shape of the kernel (MT, NT, W, D are template parameters)
//   workgroup  W waves side by side along the output channels; the tile is 32 MT tokens x 32 NT W channels, and wave w
//              owns all of its tokens against its own 32 NT channels: MT x NT MFMA tiles of 32 x 32.
//   weights    go straight from global memory into the registers of the one wave that multiplies them (no LDS): the
//              16 code bytes of (row r, group 4 g + q) of a row tile are the operand of lane (r, g) for MFMA q of a K step
//              of 256, so a request is two runs of 512 contiguous bytes.  D register sets: D steps are in flight.
//   tokens     are shared by the waves: their codes and scale words go by LDS-DMA into one of D + 1 stages, and every
//              wave reads its fragments from there, one quarter step ahead of the MFMAs.
//   K loop     one workgroup barrier per step.  A step's requests are spread between its MFMAs, and the registers of a
//              weight fragment are requested anew right behind their last use.  The last D steps, which have nothing left
//              to request, are a copy of the loop's body of their own.
// K is a summation index, so feeding groups to the instruction in this permuted order changes nothing but the order of
// the fp32 additions; that order is the same for every tile shape, and so is the result, bit for bit.
//
// What bounds it.  With every CU busy on real codes the chip runs at its power limit: at 2048 x 14336 x 4096 the K loop
// takes the same 1307 cycles per step of 128 x 256 outputs (1024 of them MFMA) on zero and on random codes, but the clock
// is 2.24 GHz on the former and 1.52 GHz on the latter; with half of the CUs it stays at 2.39 GHz.  What costs energy
// beside the MFMAs is the transfer from L2 (taken out: 48 -> 38 us of loop) and the LDS reads (-> 43 us), so the family
// keeps the weights out of LDS (per step of 128 x 256 outputs 17 KiB written to and 64 KiB read from LDS; with both
// operands staged and the waves as 2 x 2 it was 52 and 96) and takes the tile that covers the output with the fewest
// tiles per CU.  A tile of few MFMAs is bound by the path from L2 into the CU (about 44 bytes per cycle).
// Measured against the kernels it replaced (both operands through LDS, 64 x 128, 128 x 256 and persistent 256 x 256 tiles),
// both in turn on one MI355X, us per launch, T x N x K, weights in HBM (sets of 640 MB in turn) and in brackets cached:
//   160 x 4096 x 4096 11.7 -> 8.1 (10.4 -> 5.1), 512 x 4096 x 4096 12.4 -> 9.7 (11.2 -> 7.3), 333 x 14336 x 4096 21.0 -> 17.4 (18.8 -> 14.4),
//   777 x 4096 x 14336 49.8 -> 38.0 (43.8 -> 29.9), 2048 x 4096 x 14336 61.1 -> 56.8 (60.4 -> 55.8), 3001 x 14336 x 4096 102.6 -> 93.9
//   (100.0 -> 89.2), 8192 x 4096 x 4096 69.4 -> 68.6 (69.1 -> 65.8), 8192 x 14336 x 4096 239.9 -> 229.4 (231.8 -> 227.2),
//   4096 x 8192 x 28672 413.7 -> 390.4 (400.6 -> 387.6).  Of 176 products (33 to 8192 tokens, eleven linears) one is slower by more
//   than 2 %, 1024 x 14336 x 4096 with its weights in HBM, 34.4 -> 36.0 (33.2 -> 32.0): constants that pick 256 x 256 tiles there (33.6
//   and 32.8) lose as much at five others.
//
// Requests and LDS-DMA transfers are builtins, so that the compiler knows which registers are still being written and counts
// every transfer in its waits for them.  Its waits for the transfers themselves would drain the whole queue before every LDS
// read, so gemm_tile is given the LDS twice, as the destination of the transfers and as what is read, each restrict: the
// compiler leaves that order to arrive(), which counts on the order of the requests (hence the sched_barriers).
#include <type_traits>
#include <utility>

#include "duqpp_internal.h"
#include "mxfp4_device.h"

namespace duqpp {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));   // fp32 pairs convert to it in one instruction, round to nearest even

namespace {

constexpr int kTileStepBytes = 8 * 512;                 // codes of one row tile for one K step (8 groups)

#define DUQPP_MFMA(ACC, A, B, SA, SB, SEL) \
    ACC = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fp4_operand(A), fp4_operand(B), ACC, 4, 4, SEL, (int)(SA), SEL, (int)(SB))

template <int N, typename F, int... I>
__device__ __forceinline__ void unroll_impl(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void unroll(F&& f) {
    unroll_impl<N>(f, std::make_integer_sequence<int, N>{});
}

// 16 (4) bytes per lane from base + voff + OFF.  Ordinary loads: the compiler knows which registers are still being written
// and waits for them itself ahead of their use.
typedef const __attribute__((address_space(1))) uint8_t* GlobalBytes;
template <int OFF>
__device__ __forceinline__ u32x4 request_b128(uint32_t voff, const uint8_t* base) {
    asm("" : "+v"(voff));   // keeps the lane's offset a 32-bit register: widened ahead of the loop it would cost an addition per request
    return *(const __attribute__((address_space(1))) u32x4*)((GlobalBytes)base + voff + OFF);
}
__device__ __forceinline__ uint32_t request_b32(uint32_t voff, const uint8_t* base) {
    asm("" : "+v"(voff));
    return *(const __attribute__((address_space(1))) uint32_t*)((GlobalBytes)base + voff);
}
// 16 (4) bytes per lane from base + soff + voff + OFF to dst + OFF + 16 (4) * lane in LDS.  The form with a buffer descriptor: the
// compiler takes the one with a plain address for an access to LDS as well and drains the whole queue at the next wait.
typedef __attribute__((address_space(3))) uint8_t* LdsBytes;
typedef __attribute__((address_space(3))) uint16_t* LdsU16;
typedef const __attribute__((address_space(3))) uint32_t* LdsU32;
typedef const __attribute__((address_space(3))) u32x4* LdsU32x4;
template <int BYTES, int OFF>
__device__ __forceinline__ void dma(const uint8_t* base, uint32_t soff, uint32_t voff, LdsBytes dst) {
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, 0xFFFFFFFF, 0x00020000);
    const auto to = (__attribute__((address_space(3))) void*)dst;
    if constexpr (BYTES == 16) __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, to, 16, voff, soff, OFF, 0);
    else __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, to, 4, voff, soff, OFF, 0);
}

// At most N requests outstanding, every LDS access of this wave completed, and all waves of the workgroup come this far.
template <int N>
__device__ __forceinline__ void arrive() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(N) : "memory");
}

// Every LDS access this wave has issued has completed, then workgroup barrier.
__device__ __forceinline__ void workgroup_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int MT, int NT, int D, int W, bool B_ROWS = false>
struct Tile {
    static constexpr int kBM = 32 * MT, kBN = 32 * NT * W;
    static constexpr int kScalesOff = MT * kTileStepBytes;    // scale words follow the codes in a stage
    static constexpr int kBOff = kScalesOff + MT * 256;       // B_ROWS: behind them the weights' codes, 4 KiB of each wave and row tile
    static constexpr int kStageBytes = kBOff + (B_ROWS ? W * NT * 4096 : 0);
    static constexpr int kStages = D + 1;
    static constexpr int kPieces = 4 / W;                     // KiB of a token row tile's step that one wave transfers
    static constexpr int kCOps = MT * kPieces;
    static constexpr int kSOps = (MT + W - 1) / W;            // scale transfers per wave and step
    static constexpr int kBOps = B_ROWS ? 4 * NT : 0;
    static constexpr int kDma = kCOps + kSOps + kBOps;        // LDS-DMA transfers per wave and step
    static constexpr int kOps = kDma + (B_ROWS ? 1 : 5) * NT; // all requests per wave and step, in the order they complete
    static constexpr int kLate = (B_ROWS ? 1 : 2) * NT;       // of them behind the step's wait
    static constexpr int kPitch = 64 * NT + 16;               // a row of the bf16 transpose
    static constexpr int kEpBytes = 32 * kPitch;
    static constexpr int kLdsBytes = kStages * kStageBytes > W * kEpBytes ? kStages * kStageBytes : W * kEpBytes;
    static_assert(kOps * (D - 1) <= 63, "the wait counter holds 63");
    static_assert(D % 2 == 0, "scale registers alternate by step parity");
};

constexpr int kGroupM = 8;

// the weight codes of the steps that pad a run of K steps to a multiple of D: their products are exact zeros
static __device__ __align__(1024) const uint8_t zero_codes[kTileStepBytes] = {};

// The tile of this workgroup, among tiles_m x tiles_n.
template <int OCC>
__device__ __forceinline__ void tile_of_workgroup(int tiles_m, int tiles_n, int& tile_m, int& tile_n) {
    // Workgroups are dealt to the XCDs in turn.  Within each round of as many as the chip holds at once they are renumbered
    // so that an XCD owns a contiguous range, and tile numbers run through groups of kGroupM M-tiles swept along N: the
    // workgroups sharing an L2 cover a compact block of the output, and the blocks of one round lie side by side (with
    // one contiguous range per XCD over the whole launch instead, 8192 x 14336 x 4096 takes 270 us, by rounds 234).
    int pid;
    {
        constexpr int kRound = kNumCU * OCC;
        const int first = (int)blockIdx.x / kRound * kRound;
        const int id = (int)blockIdx.x - first, left_wgs = (int)gridDim.x - first, n = left_wgs < kRound ? left_wgs : kRound;
        const int per = n / kNumXCD, rem = n % kNumXCD;
        const int xcd = id % kNumXCD, slot = id / kNumXCD;
        pid = first + xcd * per + (xcd < rem ? xcd : rem) + slot;
    }
    // No division by a runtime number where there is one group, and within a group a multiplication: floor(rem / gm) is the upper
    // word of rem * ceil(2^32 / gm) while rem * (gm - 1) < 2^32.  Three divisions ahead of the first request took 0.1 us of every launch
    // (512 x 4096 x 4096 6.88 -> 6.82, 130 x 14336 x 4096 9.11 -> 9.00; 80 products 0.5 % faster on average).
    int first_m = 0, rem = pid;
    if (tiles_m > kGroupM) {
        const int group_sz = kGroupM * tiles_n, group = pid / group_sz;
        first_m = group * kGroupM;
        rem = pid - group * group_sz;
    }
    static_assert(kGroupM == 8, "reciprocals of 2 to 8");
    const int gm = (tiles_m - first_m) < kGroupM ? (tiles_m - first_m) : kGroupM;
    const uint32_t reciprocal = gm == 8   ? 0x20000000u
                                : gm == 7 ? 0x24924925u
                                : gm == 6 ? 0x2AAAAAABu
                                : gm == 5 ? 0x33333334u
                                : gm == 4 ? 0x40000000u
                                : gm == 3 ? 0x55555556u
                                          : 0x80000000u;
    tile_n = gm == 1 ? rem : (int)__umulhi((uint32_t)rem, reciprocal);
    tile_m = first_m + rem - tile_n * gm;
}

// The tile of MT token row tiles from row_tile and of channels tile_n.
// B_ROWS: the codes of the weights are in the row-major layout (rows_form; their scales are tiled: 8 bytes of each row and step would fetch
// as much from L2 as the codes).  They go to LDS as the tokens' do, to a part of the stage that is the wave's own: a transfer takes
// whole lines of 8 rows, lane l the 16 bytes (l % 8) ^ (l / 8) of row l / 8, so that the 8 lanes that read the same group of
// 8 rows meet in no bank.  (Requests into registers gathered from 16 rows: 512 x 4096 x 4096 12 us for the product, 8 on tiled weights.)
template <bool OUT_BF16, int MT, int NT, int D, int W, int OCC, bool B_ROWS = false>
__device__ __forceinline__ void gemm_tile(const TiledGemmParams& p, int row_tile, int tile_n, LdsBytes __restrict__ staged,
                                          LdsBytes __restrict__ lds) {
    using TL = Tile<MT, NT, D, W, B_ROWS>;
    constexpr int kStepB = B_ROWS ? 128 : kTileStepBytes;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 31, g = lane >> 5;

    const int RTa = (p.T + 31) / 32, RTb = (p.N + 31) / 32;
    const int NI = p.GP / 8;                               // K steps
    const int64_t tile_bytes = (int64_t)p.GP * 512;        // codes of one row tile
    const int64_t tile_sbytes = (int64_t)NI * 256;         // scale words of one row tile

    // sources of the step to request next; tiles past the ragged edge are replaced by the last valid one (their outputs
    // are never stored)
    const uint8_t* b_src[NT];
    const uint8_t* bs_src[NT];
    // tokens: the tile's first row tile, and the others' distance from it (below 4 GiB: best_shape)
    const uint8_t* a_src = p.a_codes + (int64_t)row_tile * tile_bytes;
    const uint8_t* as_src = p.a_scales + (int64_t)row_tile * tile_sbytes;
    auto valid = [&](int m) { return (uint32_t)(row_tile + m < RTa ? m : RTa - 1 - row_tile); };
    uint32_t a_off[MT], as_off[TL::kSOps];
#pragma unroll
    for (int m = 0; m < MT; ++m) a_off[m] = valid(m) * (uint32_t)tile_bytes;
    LdsBytes as_dst[TL::kSOps];
#pragma unroll
    for (int x = 0; x < TL::kSOps; ++x) {
        const int m = wave + W * x < MT ? wave + W * x : MT - 1;   // a wave without a tile of its own repeats the last one
        as_off[x] = valid(m) * (uint32_t)tile_sbytes;
        as_dst[x] = staged + TL::kScalesOff + m * 256;
    }
#pragma unroll
    for (int n = 0; n < NT; ++n) {
        int rt = (tile_n * W + wave) * NT + n;
        if (rt >= RTb) rt = RTb - 1;
        b_src[n] = p.b_codes + rt * tile_bytes;
        bs_src[n] = p.b_scales + rt * tile_sbytes;
    }
    const uint32_t voff_dma = wave * (TL::kPieces * 1024) + lane * 16, voff_word = lane * 4;
    const uint32_t row_bytes = (uint32_t)p.GP * 16;        // of row-major codes
    uint32_t voff_b = B_ROWS ? (lane >> 3) * row_bytes + ((lane & 7) ^ (lane >> 3)) * 16 : g * 2048 + r * 16;
    uint32_t eight_rows = 8 * row_bytes;
    const LdsBytes b_dst = staged + TL::kBOff + wave * NT * 4096;
    const LdsBytes a_dst = staged + wave * (TL::kPieces * 1024);

    // No branch: the K loop has to stay one straight piece of code, or the compiler moves products out from between the
    // requests and copies registers whose contents are still on their way (waiting for them first).
    int left = NI - 1;                                     // steps after the one the sources point at
    uint64_t zero_addr = (uint64_t)zero_codes;
    asm volatile("" : "+s"(zero_addr));                    // one register pair: or it is computed again in every step
    auto advance = [&]() {
        const uint32_t more = left > 0 ? 1u : 0u;
        const uint64_t keep = 0ull - more, zeros = zero_addr & ~keep;
        --left;
        a_src += more * kTileStepBytes;
        as_src += more * 256;
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            b_src[n] = (const uint8_t*)((((uint64_t)b_src[n] + kStepB) & keep) | zeros);
            bs_src[n] += more * 256;
        }
        if constexpr (B_ROWS) {                            // within the zero codes
            voff_b = more ? voff_b : 0u;
            eight_rows = more ? eight_rows : 0u;
        }
    };

    u32x4 b[D][NT][4];                                     // (B_ROWS: fb instead)
    u32x4 fb[2][NT];
    uint32_t sb[D][NT];
    u32x4 fa[2][MT];
    uint32_t sa[2][MT];

    auto dma_op = [&](auto kc, uint32_t so) {
        constexpr int k = decltype(kc)::value;
        if constexpr (k < TL::kCOps) {
            constexpr int m = k / TL::kPieces, piece = k % TL::kPieces;
            dma<16, piece * 1024>(a_src, a_off[m], voff_dma, a_dst + m * kTileStepBytes + so);
        } else if constexpr (k < TL::kDma) {
            if constexpr (k < TL::kCOps + TL::kSOps) {
                dma<4, 0>(as_src, as_off[k - TL::kCOps], voff_word, as_dst[k - TL::kCOps] + so);
            } else {
                constexpr int n = (k - TL::kCOps - TL::kSOps) / 4, piece = (k - TL::kCOps - TL::kSOps) % 4;
                dma<16, 0>(b_src[n], piece * eight_rows, voff_b, b_dst + n * 4096 + piece * 1024 + so);
            }
        }
    };

    // ---- prologue: D steps in flight
    unroll<D>([&](auto dc) {
        constexpr int d = decltype(dc)::value;
        unroll<TL::kDma>([&](auto kc) { dma_op(kc, d * TL::kStageBytes); });
        unroll<NT>([&](auto nc) {
            constexpr int n = decltype(nc)::value;
            if constexpr (!B_ROWS) {
                b[d][n][0] = request_b128<0>(voff_b, b_src[n]);
                b[d][n][1] = request_b128<512>(voff_b, b_src[n]);
                b[d][n][2] = request_b128<1024>(voff_b, b_src[n]);
                b[d][n][3] = request_b128<1536>(voff_b, b_src[n]);
            }
            sb[d][n] = request_b32(voff_word, bs_src[n]);
        });
        advance();
        __builtin_amdgcn_sched_barrier(0);                 // the waits count on the steps' order
    });
    f32x16 acc[MT][NT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[m][n][e] = 0.f;

    const LdsBytes pa0 = lds + g * 2048 + r * 16;
    const LdsBytes ps0 = lds + TL::kScalesOff + lane * 4;
    arrive<(D - 1) * TL::kOps>();
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        fa[0][m] = *(LdsU32x4)(pa0 + m * kTileStepBytes);
        sa[0][m] = *(LdsU32)(ps0 + m * 256);
    }
    // B_ROWS: group 4 g + Q of row r
    LdsBytes pb0[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) pb0[q] = lds + TL::kBOff + wave * NT * 4096 + r * 128 + (((4 * g + q) ^ (r & 7)) * 16);
    if constexpr (B_ROWS) {
#pragma unroll
        for (int n = 0; n < NT; ++n) fb[0][n] = *(LdsU32x4)(pb0[0] + n * 4096);
    }

    uint32_t stage = 0, spare = (TL::kStages - 1) * TL::kStageBytes;   // offsets of the stage in use and of the one before it
    // One K step; P: its register set.  MORE: it requests the step D ahead; the last D steps (MORE = false) request nothing,
    // and the wait of step P of them leaves the D - 2 - P steps behind the next one outstanding.
    auto step = [&](auto pc, auto more_c) {
        constexpr bool MORE = decltype(more_c)::value;
        constexpr int P = decltype(pc)::value, P1 = (P + 1) % D;
        const uint32_t stage1 = stage == (TL::kStages - 1) * TL::kStageBytes ? 0 : stage + TL::kStageBytes;
        const uint32_t so = spare;                                 // consumed in the previous step
        const LdsBytes pa = pa0 + stage;
#define DUQPP_PIN __builtin_amdgcn_sched_barrier(0)
        constexpr int kSlots = 3 * MT * NT;   // transfers spread over the first three quarters
        unroll<3>([&](auto qc) {
            constexpr int Q = decltype(qc)::value;
            unroll<NT>([&](auto nc) {
                constexpr int n = decltype(nc)::value;
                unroll<MT>([&](auto mc) {
                    constexpr int m0 = decltype(mc)::value, m = (n & 1) ? MT - 1 - m0 : m0;
                    constexpr int slot = (Q * NT + n) * MT + m0;
                    if constexpr (MORE) {
                        constexpr int k0 = (slot * TL::kDma + kSlots - 1) / kSlots, k1 = ((slot + 1) * TL::kDma + kSlots - 1) / kSlots;
                        unroll<k1 - k0>([&](auto kc) { dma_op(std::integral_constant<int, k0 + decltype(kc)::value>{}, so); });
                    }
                    if constexpr (n == 0) fa[(Q + 1) & 1][m] = *(LdsU32x4)(pa + m * kTileStepBytes + (Q + 1) * 512);
                    if constexpr (B_ROWS && m0 == 0) fb[(Q + 1) & 1][n] = *(LdsU32x4)(pb0[Q + 1] + n * 4096 + stage);
                    DUQPP_PIN;
                    if constexpr (B_ROWS) DUQPP_MFMA(acc[m][n], fa[Q & 1][m], fb[Q & 1][n], sa[P & 1][m], sb[P][n], Q);
                    else DUQPP_MFMA(acc[m][n], fa[Q & 1][m], b[P][n][Q], sa[P & 1][m], sb[P][n], Q);
                    DUQPP_PIN;
                });
                if constexpr (MORE && !B_ROWS) b[P][n][Q] = request_b128<Q * 512>(voff_b, b_src[n]);
                DUQPP_PIN;
            });
        });
        // the next step's operands have arrived, for this wave and then for all
        if constexpr (MORE) arrive<(D - 2) * TL::kOps + TL::kOps - TL::kLate>();
        else if constexpr (P < D - 1) arrive<(D - 2 - P) * TL::kOps>();
        DUQPP_PIN;
        const LdsBytes na = pa0 + stage1;
        const LdsBytes ns = ps0 + stage1;
        unroll<NT>([&](auto nc) {
            constexpr int n = decltype(nc)::value;
            unroll<MT>([&](auto mc) {
                constexpr int m0 = decltype(mc)::value, m = (n & 1) ? MT - 1 - m0 : m0;
                if constexpr (n == 0 && (MORE || P < D - 1)) {
                    fa[0][m] = *(LdsU32x4)(na + m * kTileStepBytes);
                    sa[(P + 1) & 1][m] = *(LdsU32)(ns + m * 256);
                }
                if constexpr (B_ROWS && m0 == 0 && (MORE || P < D - 1)) fb[0][n] = *(LdsU32x4)(pb0[0] + n * 4096 + stage1);
                DUQPP_PIN;
                if constexpr (B_ROWS) DUQPP_MFMA(acc[m][n], fa[1][m], fb[1][n], sa[P & 1][m], sb[P][n], 3);
                else DUQPP_MFMA(acc[m][n], fa[1][m], b[P][n][3], sa[P & 1][m], sb[P][n], 3);
                DUQPP_PIN;
            });
            if constexpr (MORE) {
                if constexpr (!B_ROWS) b[P][n][3] = request_b128<1536>(voff_b, b_src[n]);
                sb[P][n] = request_b32(voff_word, bs_src[n]);
                DUQPP_PIN;
            }
        });
#undef DUQPP_PIN
        if constexpr (MORE) advance();
        spare = stage;
        stage = stage1;
    };
    for (int it = (NI + D - 1) / D; it > 1; --it) unroll<D>([&](auto dc) { step(dc, std::true_type{}); });
    unroll<D>([&](auto dc) { step(dc, std::false_type{}); });
    // the last products happen here, whatever is stored below (or the compiler moves them into the branches of the stores)
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            if constexpr (OCC == 1) asm volatile("" : "+a"(acc[m][n]));
            else asm volatile("" : "+v"(acc[m][n]));
        }
    workgroup_barrier();                                   // the stages become the scratch of the transpose below

    // ---- epilogue: acc[m][n][e] of lane (r, g) is row 32 m + 8 (e / 4) + 4 g + e % 4, column 32 n + r of the wave's tile
    const int m0 = row_tile * 32, n0 = tile_n * TL::kBN + wave * 32 * NT;
    if constexpr (OUT_BF16) {
        if ((reinterpret_cast<uintptr_t>(p.y) & 15) == 0 && (p.ldy % 8) == 0) {
            constexpr int kChunks = 4 * NT, kRows = 64 / kChunks;      // 16-byte pieces of a row; rows per store instruction
            const LdsBytes ep = lds + wave * TL::kEpBytes;
            const int ch = lane % kChunks, row0 = lane / kChunks;
            const int gcol = n0 + ch * 8;
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                __builtin_amdgcn_sched_barrier(0);         // one row tile's values in registers at a time
#pragma unroll
                for (int n = 0; n < NT; ++n)
#pragma unroll
                    for (int e = 0; e < 16; e += 2) {
                        const bf16x2 v = __builtin_convertvector((f32x2){acc[m][n][e], acc[m][n][e + 1]}, bf16x2);
                        const uint32_t u = __builtin_bit_cast(uint32_t, v);
                        const LdsBytes q = ep + (8 * (e / 4) + 4 * g + (e % 4)) * TL::kPitch + (32 * n + r) * 2;
                        *(LdsU16)q = (uint16_t)u;
                        *(LdsU16)(q + TL::kPitch) = (uint16_t)(u >> 16);
                    }
#pragma unroll
                for (int k = 0; k < 32 / kRows; ++k) {
                    const int row = k * kRows + row0, grow = m0 + 32 * m + row;
                    const u32x4 v = *(LdsU32x4)(ep + row * TL::kPitch + ch * 16);
                    if (grow < p.T && gcol < p.N) {
                        uint16_t* dst = (uint16_t*)p.y + (int64_t)grow * p.ldy + gcol;
                        if (gcol + 8 <= p.N) {
                            __builtin_nontemporal_store(v, (u32x4*)dst);
                        } else {                           // ragged right edge
                            for (int c = 0; c < 8 && gcol + c < p.N; ++c) dst[c] = (uint16_t)(v[c / 2] >> (16 * (c & 1)));
                        }
                    }
                }
            }
            return;
        }
    }
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            const int col = n0 + 32 * n + r;
            if (col >= p.N) continue;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int row = m0 + 32 * m + 8 * (e / 4) + 4 * g + (e % 4);
                if (row < p.T) {
                    if (OUT_BF16) ((uint16_t*)p.y)[(int64_t)row * p.ldy + col] = f32_to_bf16_rne(acc[m][n][e]);
                    else ((float*)p.y)[(int64_t)row * p.ldy + col] = acc[m][n][e];
                }
            }
        }
}

template <bool OUT_BF16, int MT, int NT, int D, int W, int OCC>
__global__ __launch_bounds__(64 * W, OCC) void gemm_tiled_kernel(TiledGemmParams p) {
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    using TL = Tile<MT, NT, D, W>;
    int tile_m, tile_n;
    tile_of_workgroup<OCC>((p.T + TL::kBM - 1) / TL::kBM, (p.N + TL::kBN - 1) / TL::kBN, tile_m, tile_n);
    gemm_tile<OUT_BF16, MT, NT, D, W, OCC>(p, tile_m * MT, tile_n, (LdsBytes)lds, (LdsBytes)lds);
}

// The same with row-major weights.  (Renumbered in rounds of OCC workgroups per CU, too, although of four waves one fits: in rounds of one per CU
// it comes out level, 0.999 of the time over 4400 pairs of tile and product.)
template <bool OUT_BF16, int MT, int NT, int D, int W, int OCC>
__global__ __launch_bounds__(64 * W, OCC) void gemm_rows_kernel(TiledGemmParams p) {
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    using TL = Tile<MT, NT, D, W, true>;
    int tile_m, tile_n;
    tile_of_workgroup<OCC>((p.T + TL::kBM - 1) / TL::kBM, p.N / TL::kBN, tile_m, tile_n);
    gemm_tile<OUT_BF16, MT, NT, D, W, OCC, true>(p, tile_m * MT, tile_n, (LdsBytes)lds, (LdsBytes)lds);
}

// The same tiles where the token row tiles do not fill them: spread evenly, so that some hold MT of them and the others MT - 1 and
// do a row tile less, instead of all but the last holding MT and the last doing the work of MT for what is left.  At the power
// limit the products saved let the others run faster.
template <bool OUT_BF16, int MT, int NT, int D, int W, int OCC>
__global__ __launch_bounds__(64 * W, OCC) void gemm_spread_kernel(TiledGemmParams p) {
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    using TL = Tile<MT, NT, D, W>;
    const int row_tiles = (p.T + 31) / 32, tiles_m = (row_tiles + MT - 1) / MT;
    int tile_m, tile_n;
    tile_of_workgroup<OCC>(tiles_m, (p.N + TL::kBN - 1) / TL::kBN, tile_m, tile_n);
    const int more = row_tiles - (MT - 1) * tiles_m;         // so many tiles hold MT, the others MT - 1
    const int row_tile = tile_m * (MT - 1) + (tile_m < more ? tile_m : more);
    if (tile_m >= more) gemm_tile<OUT_BF16, MT - 1, NT, D, W, OCC>(p, row_tile, tile_n, (LdsBytes)lds, (LdsBytes)lds);
    else gemm_tile<OUT_BF16, MT, NT, D, W, OCC>(p, row_tile, tile_n, (LdsBytes)lds, (LdsBytes)lds);
}

// Whether a call's row tiles are spread: every tile can hold MT or MT - 1 of them, and not all MT.  Long reductions only: with few
// K steps what both bodies' code costs to fetch outweighs the products (T x N x K in us on one MI355X, weights cached: 1200 x 4096 x 4096
// 12.7 -> 13.1, in HBM 390 x 14336 x 4096 19.3 -> 20.0).  From K = 8192 on, over 60 ragged products of the tiles below, 1.1 % faster
// on average (cached 777 x 4096 x 14336 29.7 -> 28.5, 390 x 14336 x 8192 29.6 -> 28.2; in HBM 1800 x 8192 x 8192 61.2 -> 58.9, at worst
// 390 x 8192 x 8192 23.9 -> 24.2, cached 19.0 -> 18.1).  96 x 128 tiles lost there (in HBM 700 x 4096 x 14336 28.9 -> 30.1, 300 x 8192 x 8192
// 18.7 -> 19.5) what they gained cached, those of fewer tokens or two waves gain and lose alike.
constexpr int spread_from(int mt, int nt, int w) { return w == 4 && (mt >= 4 || nt == 2) ? 256 : 0; }   // groups of K; 0: never
template <int MT, int NT, int W>
bool spreads(const TiledGemmParams& p) {
    const int64_t row_tiles = ((int64_t)p.T + 31) / 32, tiles_m = (row_tiles + MT - 1) / MT;
    return row_tiles % MT != 0 && (MT - 1) * tiles_m <= row_tiles && p.GP >= spread_from(MT, NT, W);
}

template <int MT, int NT, int D, int W, int OCC>
hipError_t allow() {
    hipError_t e = allow_dynamic_lds((const void*)gemm_tiled_kernel<true, MT, NT, D, W, OCC>, Tile<MT, NT, D, W>::kLdsBytes);
    if (e != hipSuccess) return e;
    e = allow_dynamic_lds((const void*)gemm_tiled_kernel<false, MT, NT, D, W, OCC>, Tile<MT, NT, D, W>::kLdsBytes);
    if constexpr (NT == 1) {
        if (e != hipSuccess) return e;
        e = allow_dynamic_lds((const void*)gemm_rows_kernel<true, MT, NT, D, W, OCC>, Tile<MT, NT, D, W, true>::kLdsBytes);
        if (e != hipSuccess) return e;
        e = allow_dynamic_lds((const void*)gemm_rows_kernel<false, MT, NT, D, W, OCC>, Tile<MT, NT, D, W, true>::kLdsBytes);
    }
    if constexpr (spread_from(MT, NT, W) > 0) {
        if (e != hipSuccess) return e;
        e = allow_dynamic_lds((const void*)gemm_spread_kernel<true, MT, NT, D, W, OCC>, Tile<MT, NT, D, W>::kLdsBytes);
        if (e != hipSuccess) return e;
        e = allow_dynamic_lds((const void*)gemm_spread_kernel<false, MT, NT, D, W, OCC>, Tile<MT, NT, D, W>::kLdsBytes);
    }
    return e;
}
template <int MT, int NT, int D, int W, int OCC>
hipError_t run(const TiledGemmParams& p, hipStream_t stream) {
    using TL = Tile<MT, NT, D, W>;
    const int64_t tiles = (int64_t)((p.T + TL::kBM - 1) / TL::kBM) * ((p.N + TL::kBN - 1) / TL::kBN);
    const dim3 grid((unsigned)tiles), block(64 * W);
    if constexpr (NT == 1) {
        if (p.b_rows)
            return p.out_bf16 ? launch(gemm_rows_kernel<true, MT, NT, D, W, OCC>, grid, block, Tile<MT, NT, D, W, true>::kLdsBytes, stream, p)
                              : launch(gemm_rows_kernel<false, MT, NT, D, W, OCC>, grid, block, Tile<MT, NT, D, W, true>::kLdsBytes, stream, p);
    }
    if constexpr (spread_from(MT, NT, W) > 0) {
        if (spreads<MT, NT, W>(p))
            return p.out_bf16 ? launch(gemm_spread_kernel<true, MT, NT, D, W, OCC>, grid, block, TL::kLdsBytes, stream, p)
                              : launch(gemm_spread_kernel<false, MT, NT, D, W, OCC>, grid, block, TL::kLdsBytes, stream, p);
    }
    return p.out_bf16 ? launch(gemm_tiled_kernel<true, MT, NT, D, W, OCC>, grid, block, TL::kLdsBytes, stream, p)
                      : launch(gemm_tiled_kernel<false, MT, NT, D, W, OCC>, grid, block, TL::kLdsBytes, stream, p);
}

// The tile shapes.  Two workgroups of the four-wave tiles fit a CU, but for the two largest (one; and one of those on row-major codes, for
// which these figures are not made, see rows_pay): while one of them waits for its first operands or stores its tile, the other has the
// matrix cores.  one / two: microseconds per K step of
// 256 while a CU holds one or two tiles; fixed: per round of tiles, what the pipeline's start and the store take.  Fitted
// to the time of every shape at 400 products (33 to 8192 tokens, seven linears of the 8B and 70B models and four generic
// ones, weights in the last-level cache and in HBM).  Over 170 products the shape chosen takes on average 1.3 % longer than
// the fastest of the eleven with the weights in HBM (18 % at worst) and 1.2 % with them cached (21 %).
struct Shape {
    int mt, nt, w, per_cu;
    double one, two, fixed;
    hipError_t (*allow)();
    hipError_t (*run)(const TiledGemmParams&, hipStream_t);
};
#define DUQPP_SHAPE(MT, NT, D, W, OCC, PER_CU, ONE, TWO, FIXED) \
    {MT, NT, W, PER_CU, ONE, TWO, FIXED, allow<MT, NT, D, W, OCC>, run<MT, NT, D, W, OCC>}
const Shape kShapes[] = {
    // 64 channels wide, for outputs that these cut into no more tiles than there are CUs: per output a 64 x 64 tile fetches
    // four fifths of the bytes of a 32 x 128 one (256 x 4096 x 14336 from HBM: 19.4 us, 32 x 128 tiles 23.2 us)
    DUQPP_SHAPE(1, 1, 4, 2, 2, 1, 0.194, 0.0, 2.16),
    DUQPP_SHAPE(2, 1, 4, 2, 2, 1, 0.232, 0.0, 2.68),
    DUQPP_SHAPE(3, 1, 4, 2, 2, 1, 0.296, 0.0, 3.80),
    // 128 channels wide
    DUQPP_SHAPE(1, 1, 4, 4, 2, 2, 0.237, 0.540, 2.60),
    DUQPP_SHAPE(2, 1, 4, 4, 2, 2, 0.372, 0.655, 2.97),
    DUQPP_SHAPE(3, 1, 4, 4, 2, 2, 0.414, 0.730, 3.43),
    DUQPP_SHAPE(4, 1, 2, 4, 2, 2, 0.526, 0.930, 3.60),
    // 256 channels wide
    DUQPP_SHAPE(3, 2, 2, 4, 2, 2, 0.616, 1.386, 3.58),
    DUQPP_SHAPE(4, 2, 2, 4, 2, 2, 0.695, 1.601, 6.37),
    DUQPP_SHAPE(6, 2, 2, 4, 1, 1, 1.151, 0.0, 8.42),
    DUQPP_SHAPE(8, 2, 2, 4, 1, 1, 1.414, 0.0, 10.11),
};
#undef DUQPP_SHAPE

int64_t tiles_of(const Shape& s, const TiledGemmParams& p) {
    return (int64_t)((p.T + 32 * s.mt - 1) / (32 * s.mt)) * ((p.N + 32 * s.nt * s.w - 1) / (32 * s.nt * s.w));
}

// Rounds of tiles over the CUs, the last one with one tile per CU where that is all there is.
double cost_of(const Shape& s, const TiledGemmParams& p) {
    const int64_t n = tiles_of(s, p), cap = (int64_t)kNumCU * s.per_cu;
    const int64_t full = n / cap, rest = n % cap;
    const double steps = p.GP / 8;
    if (s.per_cu == 1) return (double)(full + (rest != 0)) * (steps * s.one + s.fixed);
    return (double)full * (steps * s.two + s.fixed) +
           (rest == 0 ? 0.0 : steps * (rest > kNumCU ? s.two : s.one) + s.fixed);
}

// distances within a tile's tokens are 32-bit
bool distances_fit(const Shape& s, const TiledGemmParams& p) { return (int64_t)(s.mt - 1) * p.GP * 512 < (int64_t)0xFFFFE000; }

template <typename Pred>
const Shape* best_shape(const TiledGemmParams& p, Pred&& allowed) {
    const Shape* best = nullptr;
    double best_cost = 0.0;
    for (const Shape& s : kShapes) {
        if (!allowed(s) || (s.w < 4 && tiles_of(s, p) > kNumCU) || !distances_fit(s, p)) continue;
        const double c = cost_of(s, p);
        if (!best || c < best_cost) { best = &s; best_cost = c; }
    }
    return best;
}

bool any_shape(const Shape&) { return true; }
bool streaming_shape(const Shape& s) { return s.mt == 1 || s.w < 4; }
bool small_shape(const Shape& s) { return s.nt == 1; }
bool mid_shape(const Shape& s) { return s.nt == 2 && s.mt <= 4; }
bool large_shape(const Shape& s) { return s.nt == 2 && s.mt > 4; }
bool unaligned_shape(const Shape& s) { return s.mt <= 4; }

// N a multiple of 8 for either output type: the fp32 and the bf16 result of a shape come from the same tile
bool large_ok(const TiledGemmParams& p) { return (p.N % 8) == 0 && gemm_tiled_large_accepts(p); }

const Shape* choose_shape(const TiledGemmParams& p) { return large_ok(p) ? best_shape(p, any_shape) : best_shape(p, unaligned_shape); }

}  // namespace

// what the name DUQPP_GEMM_KERNEL_LARGE promises: bf16 results leave in whole 16-byte pieces
bool gemm_tiled_large_accepts(const TiledGemmParams& p) {
    if (!p.out_bf16) return true;
    return (reinterpret_cast<uintptr_t>(p.y) & 15) == 0 && (p.ldy % 8) == 0 && (p.N % 8) == 0;
}

hipError_t setup_gemm_tiled() {
    static PerDeviceOnce once;
    return once.run([] {
        for (const Shape& s : kShapes) {
            const hipError_t e = s.allow();
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    });
}

int gemm_tiles() { return (int)(sizeof(kShapes) / sizeof(kShapes[0])); }

// The tile that `kernel` runs a call with, null where K is split over the waves instead or the kernel cannot run the call.
static const Shape* tile_of(const TiledGemmParams& p, int kernel) {
    switch (kernel) {
        case DUQPP_GEMM_KERNEL_AUTO:
            if (decode_splits_k(p)) return nullptr;
            return p.T <= 32 ? best_shape(p, streaming_shape) : choose_shape(p);
        case DUQPP_GEMM_KERNEL_DECODE: return decode_splits_k(p) || p.T > kDecodeMaxT ? nullptr : best_shape(p, streaming_shape);
        case DUQPP_GEMM_KERNEL_SMALL: return best_shape(p, small_shape);
        case DUQPP_GEMM_KERNEL_MID: return best_shape(p, mid_shape);
        case DUQPP_GEMM_KERNEL_LARGE: return gemm_tiled_large_accepts(p) ? best_shape(p, large_shape) : nullptr;
    }
    const int i = kernel - DUQPP_GEMM_KERNEL_TILE;
    return i >= 0 && i < gemm_tiles() && distances_fit(kShapes[i], p) ? &kShapes[i] : nullptr;
}

int gemm_tile_for(const TiledGemmParams& p, int kernel, int* tokens, int* channels) {
    const Shape* s = tile_of(p, kernel);
    if (!s) return kernel <= DUQPP_GEMM_KERNEL_DECODE && decode_splits_k(p) ? DUQPP_GEMM_SPLIT_K : -1;
    if (tokens) *tokens = 32 * s->mt;
    if (channels) *channels = 32 * s->nt * s->w;
    return (int)(s - kShapes);
}

// Which kernel runs a shape, by the names of the ABI.
int choose_gemm_kernel(const TiledGemmParams& p) {
    const Shape* s = tile_of(p, DUQPP_GEMM_KERNEL_AUTO);
    if (!s || p.T <= 32 || (p.T <= 64 && streaming_shape(*s))) return DUQPP_GEMM_KERNEL_DECODE;
    return small_shape(*s) ? DUQPP_GEMM_KERNEL_SMALL : mid_shape(*s) ? DUQPP_GEMM_KERNEL_MID : DUQPP_GEMM_KERNEL_LARGE;
}

hipError_t launch_gemm_tiled_as(const TiledGemmParams& p, int kernel, hipStream_t stream) {
    if (const Shape* s = tile_of(p, kernel)) {
        const hipError_t e = setup_gemm_tiled();
        return e == hipSuccess ? s->run(p, stream) : e;
    }
    return kernel <= DUQPP_GEMM_KERNEL_DECODE ? launch_gemm_decode(p, stream) : hipErrorInvalidValue;
}

hipError_t launch_gemm_tiled(const TiledGemmParams& p, hipStream_t stream) {
    return launch_gemm_tiled_as(p, DUQPP_GEMM_KERNEL_AUTO, stream);
}

// The tile of a call with row-major weights whose K is not split over the waves.  All of them are 32 channels per wave.
static const Shape* rows_shape(const TiledGemmParams& p) { return p.T <= 32 ? best_shape(p, streaming_shape) : best_shape(p, small_shape); }

// Row-major weights are multiplied as they are, instead of being read and written tiled first, where re-tiling is a large part of the call:
// whole K steps and tiles only, rows of scales on 8 bytes, and a row tile's rows within 32 bits of each other.  The kernels that split K
// over their waves take codes and scales, the tiles only the codes (the launch that rotates tiles the scales, a sixteenth of the bytes).
// That loses with few row tiles, i.e. few CUs fetching, where all CUs re-tile, and with many tokens, when the weights' way through LDS
// costs more than re-tiling them once.  The whole call, weights in HBM, re-tiled first / as they are, us, K x N:
//   T = 1    4096 x 1024 5.7 / 6.3, 14336 x 1024 9.7 / 11.2, 4096 x 2048 6.4 / 6.2, 4096 x 4096 9.0 / 6.4, 4096 x 14336 21.8 / 11.9,
//            14336 x 4096 22.0 / 13.4, 8192 x 28672 63 / 33, 28672 x 8192 67 / 35
//   T = 64   4096 x 2048 7.2 / 7.4, 4096 x 4096 10.1 / 7.8, 4096 x 14336 22.5 / 14.6, 14336 x 4096 26.8 / 20.4, 28672 x 8192 78 / 47
//   T = 128  4096 x 1024 6.6 / 7.6, 4096 x 4096 10.5 / 8.8, 14336 x 4096 27.9 / 21.2, 1024 x 16384 10.0 / 7.6, 8192 x 8192 27.6 / 19.0
//   T = 256  4096 x 1024 8.0 / 8.4, 4096 x 4096 12.2 / 9.9, 14336 x 4096 32.4 / 27.5, 4096 x 14336 27.5 / 19.0, 8192 x 28672 92 / 61
//   T = 512  4096 x 4096 15.2 / 13.5, 8192 x 8192 37.5 / 32.6, 4096 x 14336 34.8 / 32.0, 2048 x 2048 9.0 / 9.0
// The lines at 4096 channels and 16 M weights are where single calls came out even (4096 x 2048 and 4096 x 1024 above).  In graphs of calls with
// other weights each it gains below them as well, up to 256 tokens of 2048 channels and more or 4 M weights by 10 to 35 %: 4096 x 2048 T = 1 7.9 / 6.5,
// T = 256 10.4 / 9.1, T = 512 14.6 / 10.8; 2048 x 4096 T = 256 9.9 / 7.9; 4096 x 3072 T = 64 9.9 / 7.8; 8192 x 2048 T = 512 20.3 / 18.5; but 14336 x 2048 T = 256
// 23.4 / 23.7, T = 512 27.0 / 29.7, 28672 x 2048 T = 512 47.2 / 49.4, 8192 x 3072 T = 512 22.9 / 24.6.  They stand as they are.
// The codes take so much LDS that one of the 128-channel tiles fits a CU, where two of those on tiled weights do.  While the tiles are one
// round over the CUs the calls take 0.85 of the time on average (4500 of 65 to 1024 tokens); below 5248 channels with K of 8192 and more
// they come out level from 300 tokens on, 0.8 to 1.1 (12288 x 4224, T = 320 31.2 / 34.8, T = 512 36.0 / 34.8).  Further rounds
// lose against the tiles of 256 channels, which need half as many: T = 480 2560 x 10240 20.0 / 22.4, 12288 x 10240 62.1 / 70.4, 6144 x 8320 1.24
// of the time; T = 384 12288 x 11008 1.15; T = 288 4096 x 14336 29.1 / 28.3, 12288 x 14336 66.5 / 71.0.  They pay
//   where K is short     T = 416 2048 x 10240 19.0 / 15.7, T = 448 2048 x 8320 0.80 of the time (2560 x 8320, T = 480 1.10); of three rounds and more
//                        with few steps the starts and stores are the call (256 x 65536, T = 288 19.9 / 24.9; 1536 x 28672 0.88 of the time)
//   where they are nearly full and there is much to re-tile or K is not long     T = 448 4096 x 14336 35.1 / 30.7, T = 416 12288 x 12288 0.93 of
//                        the time, 12288 x 11008 1.0, T = 448 1.06, 4096 x 11520 0.90; 8192 x 28672 T = 288 86.0 / 72.5, T = 512 101.5 / 102.7;
//                        13 / 16 leaves 384 tiles out (12288 x 12288, T = 384 65.5 / 70.2)
// Of 1440 calls of two rounds and more these lines leave 17 that lose more than 3 % (2560 x 11520, T = 480 1.08) and 88 that would have gained as much
// (2560 x 12288, T = 512 0.85).
static bool rows_pay(const TiledGemmParams& p) {
    const int64_t K = (int64_t)p.GP * 32, tiles = tiles_of(*rows_shape(p), p), rounds = (tiles + kNumCU - 1) / kNumCU;
    if (p.T <= 128 || rounds == 1) return true;
    if (p.T > 512) return false;
    return (rounds == 2 && K <= 2304) || (K >= 1536 && 16 * tiles >= 13 * rounds * kNumCU && (p.N >= 12032 || K <= 4096));
}
RowsForm rows_form(const TiledGemmParams& p, const uint8_t* scales) {
    const int64_t K = (int64_t)p.GP * 32, N = p.N;
    if (N % 128 != 0 || K > (int64_t)1 << 24 || (reinterpret_cast<uintptr_t>(scales) & 7) != 0) return kRowsTiled;
    if (N < 4096 || N * K < (int64_t)1 << 24) return kRowsTiled;
    return decode_splits_k(p) ? kRowsAsTheyAre : rows_pay(p) ? kRowsScalesTiled : kRowsTiled;
}
hipError_t launch_gemm_rows(const TiledGemmParams& call, hipStream_t stream) {
    TiledGemmParams p = call;
    p.b_rows = 1;
    if (decode_splits_k(p)) return launch_gemm_decode(p, stream);
    const Shape* s = rows_shape(p);
    const hipError_t e = setup_gemm_tiled();
    return e == hipSuccess ? s->run(p, stream) : e;
}

}  // namespace duqpp

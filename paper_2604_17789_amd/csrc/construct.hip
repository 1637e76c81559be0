// Offline: greedy outlier-aware construction of the shared 32x32 rotation block (paper Sec. 4.2, paragraph
// "Fine-grained Block-diagonal Rotation", steps (1)-(3); all blocks share the matrix built from the block that
// holds the largest outlier).  The paper gives the construction as a sketch; the reading implemented here:
//   b*  = block of 32 channels with the largest |x| (smallest index among equals);  Z_0 = X[:, b*],  R^(0) = I
//   for t = 1 .. steps:  d = channel of Z_{t-1} with the largest magnitude (smallest index among equals)
//                        R_t = E_d . H . diag(1, Q'_t) . E_d      E_d exchanges coordinates 0 and d, H is the
//                              normalised Sylvester-Hadamard matrix (uniform first row: what sits in coordinate 0
//                              is spread evenly), Q'_t a caller-drawn orthogonal 31 x 31 matrix
//                        Z_t = Z_{t-1} . R_t,   R^(t) = R^(t-1) . R_t,   peak_t = max |Z_t|
//   result R^(t*), t* = the step count with the smallest peak (smallest t among equals; t = 0 keeps the identity)
// Arithmetic: fp64, every dot product accumulated in index order from zero with one rounding per multiply and per
// add (contraction into fused multiply-adds is switched off for this file), so that the argmax / argmin decisions
// and the result do not depend on how the work is spread over the chip.  Maxima are taken with integer atomics on
// the bit patterns of |z| (order-independent).
//
// Every step needs the largest magnitude of the whole state before it, so the steps are a chain of exchanges between all
// workgroups.  Two forms:
//   search kernel   (construct_search_kernel) one launch for all steps: a workgroup keeps its 16 or 32 rows of the state in LDS and
//                   registers, publishes the largest magnitude among them after every step, waits for everybody's, and goes on.
//                   For as many rows as workgroups that run at once hold: 16 rows each and one workgroup per CU, or 32 rows
//                   and two per CU (T <= 16352 on 256 CUs).  Should they not come to run together, because other work holds the CUs for
//                   longer than they wait (1 to 2 ms), they give up, and up to 64 workgroups with the state in memory do the
//                   search (construct_again_kernel); should not even these come to run together (within 20 ms and more), one
//                   does it, which waits for nobody: nothing ever waits without a limit.  128 steps, with what is waited ahead
//                   of it left out: 64 workgroups 2.7 ms at T = 512, 2.8 at 4064, 3.1 at 16000; one 5.2, 24, 82 ms.  Two calls of
//                   16000 rows on two streams at once: 4.0 to 5.1 ms each (with one workgroup behind 20 ms of waiting 140 to 160;
//                   a launch per step, alone, 1.5); three of 8160: one 0.4, the others 4.2.
//   launch per step (construct_step_kernel) for more rows, and for a single one: the state in memory, the maxima by atomics, all
//                   CUs waiting for each other at the launch.
// What a step's result does not depend on is done ahead of the steps, for all of them at once: the matrices H . diag(1, Q'_t).
// What a step of the search kernel takes (2048 rows, 130 workgroups, 2.0 us = 4900 cycles): 560 the workgroup's own maximum, 2100
// the exchange, 500 the maximum of what came, 800 to 1250 the products (768 of them fp64 and its operands' moves, two waves
// taking turns on a SIMD), 300 their maxima, the rest barriers.  128 steps on one MI355X, us, a launch per step / 16 rows / 32 rows
// per workgroup (K = 4096): T = 64 554 / 244 / 337, 512 559 / 235 / 329, 1024 565 / 266 / -, 2048 601 / 262 / 325, 4096 705 / - / 333,
// 8192 1048 / - / 457, 16000 1550 / - / 562.  The call is offline.
#include <type_traits>
#include <utility>

#include "duqpp_internal.h"

#pragma clang fp contract(off)

namespace duqpp {

namespace {

constexpr double kHadamardEntry = 0.17677669529663687;   // 1 / sqrt(32)
constexpr int kTileRows = 32;                            // rows of the state per workgroup of a step
constexpr int kStepWaves = 8;                            // waves of that workgroup; 4 columns each
constexpr int kMaxPartials = 1024;                       // workgroups of the block search (their keys fill one slot of 8 KiB)
constexpr int kExchangeCopies = 8;                       // copies of what the workgroups of the search kernel publish
constexpr int kExchangeWords = 2;                        // 64-bit words between one workgroup's and the next one's (two are used)
constexpr uint32_t kPatience = 2000;                     // looks for what the others publish, half a microsecond or more each: about what
                                                         // doing it in a few workgroups takes
constexpr int kFewWorkgroups = 64;                       // these (a wave looks at all of them at once)
constexpr uint32_t kPatienceAgain = 40000;               // and what doing it in one takes

typedef double f64x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ double hadamard_entry(int i, int k) { return (__popc(i & k) & 1) ? -kHadamardEntry : kHadamardEntry; }

// workspace: [header 64 B: u64 block key, u64 search given up, u64 given up again][colmax (S + 1) x 32 u64][slots (S + 1) x 1024 f64][Z T x 32 f64]
// Slot 0 holds the block search's partial keys, then the maxima below; slot t >= 1 holds M_t = H . diag(1, Q'_t), then R^(t).
// The search kernel keeps the state on the chip; the place of Z holds what its workgroups publish, that of colmax what those of the
// kernel behind it do.
struct Workspace {
    unsigned long long* key;
    unsigned long long* given_up;        // two words
    unsigned long long* colmax;
    double* slots;
    double* z;
};
__host__ __device__ inline Workspace carve(void* ws, int steps) {
    Workspace w;
    uint8_t* p = static_cast<uint8_t*>(ws);
    w.key = reinterpret_cast<unsigned long long*>(p);
    w.given_up = w.key + 1;
    w.colmax = reinterpret_cast<unsigned long long*>(p + 64);
    w.slots = reinterpret_cast<double*>(p + 64 + (size_t)(steps + 1) * 256);
    w.z = reinterpret_cast<double*>(p + 64 + (size_t)(steps + 1) * 256 + (size_t)(steps + 1) * 8192);
    return w;
}

__device__ __forceinline__ unsigned long long abs_bits(double v) { return (unsigned long long)__double_as_longlong(v) & 0x7FFFFFFFFFFFFFFFull; }
__device__ __forceinline__ unsigned long long max_u64(unsigned long long a, unsigned long long b) { return a > b ? a : b; }

// Column maxima while the steps run.  Atomics on one address are done one after the other, and with 64 workgroups merging
// their 32 maxima into 32 addresses they took 3.2 of a step's 7.3 us: kCopies copies of the 32 take an eighth of the workgroups each.
// Three sets take turns: step t merges into set t % 3, reads set (t - 1) % 3 and clears set (t + 1) % 3.
constexpr int kCopies = 8;
__device__ __forceinline__ unsigned long long* maxima(const Workspace& w, int t) {
    return reinterpret_cast<unsigned long long*>(w.slots) + (size_t)(t % 3) * kCopies * 32;
}
// maximum of column lane % 32 of the state after step t
__device__ __forceinline__ unsigned long long column_max(const Workspace& w, int t, int lane) {
    if (t == 0) return w.colmax[lane & 31];
    const unsigned long long* m = maxima(w, t) + (lane >> 5) * (kCopies / 2) * 32 + (lane & 31);
    unsigned long long v = m[0];
#pragma unroll
    for (int k = 1; k < kCopies / 2; ++k) v = max_u64(v, m[k * 32]);
    return max_u64(v, __shfl_xor(v, 32));
}

// The state: tile k holds rows 32 k ... of it, n = 32 of them or what is left, as [column pair][n rows][2].
__device__ __forceinline__ double* state_tile(const Workspace& w, int64_t tile) { return w.z + tile * (kTileRows * 32); }
__device__ __forceinline__ int tile_rows(int64_t tile, int64_t T) {
    const int64_t left = T - tile * kTileRows;
    return (int)(left < kTileRows ? left : kTileRows);
}

// Maxima over lanes, moved by the ALU.  A step takes the maximum with the value of another lane: quad permutation 0xB1 = lane ^ 1,
// 0x4E = lane ^ 2, 0x141 and 0x140 = mirrored within 8 and 16 lanes (lanes that hold the same maximum may stand in for each other,
// so the mirrors do what lane ^ 4 and lane ^ 8 would), 0x142 and 0x143 = lane 15 of a row of 16 into the next row, lane 31 into the
// upper half.  Of 64-bit values the upper words first, then the lower words of the lanes that have the largest upper one: a step
// is one instruction then, a comparison and selection of pairs would be five.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_max(uint32_t v) {
    const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
    return v > o ? v : o;
}
template <typename Steps>
__device__ __forceinline__ unsigned long long words_max(unsigned long long v, Steps&& steps) {
    const uint32_t hi = steps((uint32_t)(v >> 32));
    const uint32_t lo = steps((uint32_t)(v >> 32) == hi ? (uint32_t)v : 0u);
    return ((unsigned long long)hi << 32) | lo;
}
// maximum over each 16 lanes, in every one of them
__device__ __forceinline__ unsigned long long row16_max(unsigned long long v) {
    return words_max(v, [](uint32_t m) { return dpp_max<0x140>(dpp_max<0x141>(dpp_max<0x4E>(dpp_max<0xB1>(m)))); });
}
// maximum over each half of the wave, in every lane of the half
__device__ __forceinline__ unsigned long long half_max(unsigned long long v) {
    v = row16_max(v);
    return max_u64(v, __shfl_xor(v, 16));
}
// maximum over the 64 lanes, uniform
__device__ __forceinline__ unsigned long long wave_max(unsigned long long v) {
    return words_max(v, [](uint32_t m) {
        m = dpp_max<0x143>(dpp_max<0x142>(dpp_max<0x140>(dpp_max<0x141>(dpp_max<0x4E>(dpp_max<0xB1>(m))))));
        return (uint32_t)__builtin_amdgcn_readlane((int)m, 63);
    });
}

// The largest |x| per block of 32 channels -> one 64-bit key per workgroup of 256 threads: magnitude bits above, inverted block
// index below, so that the integer maximum is the largest magnitude in the smallest block.
__device__ __forceinline__ void block_key(const ConstructParams& p, const Workspace& w, int workgroups, unsigned long long* red) {
    const int64_t stride = (int64_t)workgroups * 256, at = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t chunks = p.K / 8;                          // 16-byte pieces of 8 bf16 in a row; 4 per block
    const int64_t dr = stride / chunks, dc = stride % chunks;
    int64_t row = at / chunks, ch = at % chunks;
    unsigned long long best = 0ull;
    auto take = [&](const uint4& v, int64_t c) {
        uint32_t m = 0;
        const uint32_t words[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t lo = words[k] & 0x7FFFu, hi = (words[k] >> 16) & 0x7FFFu;
            m = m > lo ? m : lo;
            m = m > hi ? m : hi;
        }
        best = max_u64(best, ((unsigned long long)m << 32) | (0xFFFFFFFFu - (uint32_t)(c / 4)));
    };
    auto next = [&]() {
        row += dr;
        ch += dc;
        if (ch >= chunks) { ch -= chunks; ++row; }
    };
    while (row < p.T) {
        uint4 v[4];
        int64_t c[4];
        int n = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {                        // four loads in flight
            c[k] = ch;
            v[k] = make_uint4(0, 0, 0, 0);
            if (row < p.T) { v[k] = *reinterpret_cast<const uint4*>(p.x + row * p.ldx + ch * 8); n = k + 1; }
            next();
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (k < n) take(v[k], c[k]);
    }
    best = wave_max(best);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = best;
    __syncthreads();
    if (threadIdx.x == 0)
        reinterpret_cast<unsigned long long*>(w.slots)[blockIdx.x] = max_u64(max_u64(red[0], red[1]), max_u64(red[2], red[3]));
}

// Clears the first column maxima, and the keys.
__global__ __launch_bounds__(256) void construct_blockmax_kernel(ConstructParams p) {
    __shared__ unsigned long long red[4];
    Workspace w = carve(p.workspace, p.steps);
    if (blockIdx.x == 0 && threadIdx.x < 32) w.colmax[threadIdx.x] = 0ull;
    block_key(p, w, gridDim.x, red);
}

// The chosen block from the partial keys, in every thread of a workgroup of kStepWaves waves.
__device__ __forceinline__ unsigned long long chosen_key(const Workspace& w, int partials, unsigned long long* red) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned long long key = 0ull;
    for (int i = threadIdx.x; i < partials; i += 64 * kStepWaves) key = max_u64(key, reinterpret_cast<const unsigned long long*>(w.slots)[i]);
    key = wave_max(key);
    if (lane == 0) red[wave] = key;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kStepWaves; ++k) key = max_u64(key, red[k]);
    return key;
}
__device__ __forceinline__ int64_t block_of(unsigned long long key) { return 0xFFFFFFFFu - (uint32_t)(key & 0xFFFFFFFFull); }

// Z_0 = the chosen block's columns as doubles, and their column maxima.  Every workgroup finds the block again from the
// partial keys.
__global__ __launch_bounds__(64 * kStepWaves) void construct_extract_kernel(ConstructParams p, int partials) {
    __shared__ unsigned long long red[kStepWaves];
    Workspace w = carve(p.workspace, p.steps);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const unsigned long long key = chosen_key(w, partials, red);
    if (blockIdx.x == 0 && threadIdx.x == 0) *w.key = key;
    const int64_t b = block_of(key);

    const int n = tile_rows(blockIdx.x, p.T);
    double* z = state_tile(w, blockIdx.x);
    const int row = lane & 31, h = lane >> 5;                // columns 4 wave + 2 h and the next one
    const bool ok = row < n;
    uint32_t v = 0;
    if (ok) v = *reinterpret_cast<const uint32_t*>(p.x + ((int64_t)blockIdx.x * kTileRows + row) * p.ldx + 32 * b + 4 * wave + 2 * h);
    const f64x2 d = {(double)__uint_as_float(v << 16), (double)__uint_as_float(v & 0xFFFF0000u)};
    if (ok) *reinterpret_cast<f64x2*>(z + ((2 * wave + h) * n + row) * 2) = d;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const unsigned long long m = half_max(abs_bits(d[k]));
        if (row == 0 && m) atomicMax(w.colmax + 4 * wave + 2 * h + k, m);
    }
}

// Slot 0: no maxima yet; slot t = M_t = H . diag(1, Q'_t): column 0 passes through, the others sum terms k = 1 .. 31 in order.
__device__ __forceinline__ void step_matrix(const ConstructParams& p, const Workspace& w, int t, double* q /* 31 * 31 */) {
    double* out = w.slots + (size_t)t * 1024;
    if (t > 0)
        for (int e = threadIdx.x; e < 31 * 31; e += 256) q[e] = p.q_steps[(size_t)(t - 1) * 31 * 31 + e];
    __syncthreads();
    for (int e = threadIdx.x; e < 1024; e += 256) {
        const int i = e >> 5, j = e & 31;
        double acc;
        if (t == 0) {
            acc = 0.0;
        } else if (j == 0) {
            acc = hadamard_entry(i, 0);
        } else {
            acc = 0.0;
            for (int k = 1; k < 32; ++k) acc = acc + hadamard_entry(i, k) * q[(k - 1) * 31 + (j - 1)];
        }
        out[e] = acc;
    }
}
__global__ __launch_bounds__(256) void construct_matrices_kernel(ConstructParams p) {
    __shared__ double q[31 * 31];
    step_matrix(p, carve(p.workspace, p.steps), blockIdx.x, q);
}

// The largest of the lanes' values, uniform, and the lanes that hold it.
__device__ __forceinline__ unsigned long long lanes_of_max(unsigned long long v, unsigned long long& top) {
    auto most = [](uint32_t m) {
        m = dpp_max<0x143>(dpp_max<0x142>(dpp_max<0x140>(dpp_max<0x141>(dpp_max<0x4E>(dpp_max<0xB1>(m))))));
        return (uint32_t)__builtin_amdgcn_readlane((int)m, 63);
    };
    const uint32_t hi = (uint32_t)(v >> 32), lo = (uint32_t)v, most_hi = most(hi);
    unsigned long long lanes = __ballot(hi == most_hi);
    uint32_t most_lo;
    if (lanes & (lanes - 1)) {                               // the lower words decide
        most_lo = most(hi == most_hi ? lo : 0u);
        lanes = __ballot(hi == most_hi && lo == most_lo);
    } else {
        most_lo = (uint32_t)__builtin_amdgcn_readlane((int)lo, __ffsll(lanes) - 1);
    }
    top = ((unsigned long long)most_hi << 32) | most_lo;
    return lanes;
}

// The channel that step t exchanges with channel 0: largest magnitude in the state before it, smallest index among equals.
// The same in every lane of every wave (lanes 32 .. 63 repeat lanes 0 .. 31).
__device__ __forceinline__ int exchanged_channel(unsigned long long colmax_of_lane) {
    const unsigned long long best = wave_max(colmax_of_lane);
    return __builtin_amdgcn_readfirstlane(__ffsll(__ballot(colmax_of_lane == best)) - 1);
}

// Slot t = R^(t) = R^(t-1) . R_t, R_t[r][c] = M_t[sigma(r)][sigma(c)], sigma exchanging 0 and d (one workgroup).
__device__ __forceinline__ void extend_product(const Workspace& w, int t, double* lds /* 2048 */) {
    double* m = lds;
    double* prev = lds + 1024;
    const unsigned long long cm = w.colmax[(size_t)(t - 1) * 32 + (threadIdx.x & 31)];
    for (int e = threadIdx.x; e < 1024; e += 64 * kStepWaves) {
        m[e] = w.slots[(size_t)t * 1024 + e];
        prev[e] = t > 1 ? w.slots[(size_t)(t - 1) * 1024 + e] : (e / 32 == e % 32 ? 1.0 : 0.0);   // R^(0) = I
    }
    const int d = exchanged_channel(cm);
    __syncthreads();
    for (int e = threadIdx.x; e < 1024; e += 64 * kStepWaves) {
        const int i = e >> 5, j = e & 31;
        const int sj = j == 0 ? d : (j == d ? 0 : j);
        double acc = 0.0;
#pragma unroll
        for (int r = 0; r < 32; ++r) acc = acc + prev[i * 32 + r] * m[(r == 0 ? d : (r == d ? 0 : r)) * 32 + sj];
        w.slots[(size_t)t * 1024 + e] = acc;
    }
}

// Greedy step t >= 1: Z <- Z . R_t and the new column maxima.  The last workgroup clears the next set of maxima, keeps the
// last step's and extends the product by that step (nobody else reads its slots).
__global__ __launch_bounds__(64 * kStepWaves) void construct_step_kernel(ConstructParams p, int t) {
    __shared__ double lds[2048];
    Workspace w = carve(p.workspace, p.steps);
    if (blockIdx.x == gridDim.x - 1) {
        if (threadIdx.x < kCopies * 32) maxima(w, t + 1)[threadIdx.x] = 0ull;
        if (t > 1) {
            const unsigned long long last = column_max(w, t - 1, threadIdx.x & 63);
            if (threadIdx.x < 32) w.colmax[(size_t)(t - 1) * 32 + threadIdx.x] = last;
            extend_product(w, t - 1, lds);
        }
        return;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int row = lane & 31, h = lane >> 5;
    const int n = tile_rows(blockIdx.x, p.T);
    double* z = state_tile(w, blockIdx.x);
    const int rl = row < n ? row : n - 1;                    // lanes past the end repeat the last row and store nothing

    // everything the step reads is asked for before anything is waited for
    const unsigned long long cm = column_max(w, t - 1, lane);
    const f64x2 entries = reinterpret_cast<const f64x2*>(w.slots + (size_t)t * 1024)[threadIdx.x];   // of M_t, row threadIdx.x / 16
    f64x2 x[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) x[k] = *reinterpret_cast<const f64x2*>(z + (k * n + rl) * 2);
    unsigned long long* const mine = maxima(w, t) + (blockIdx.x % kCopies) * 32;
    const int d = exchanged_channel(cm);
    // M_t with its rows in the order sigma(0), sigma(1), ...
    const int mr = threadIdx.x >> 4;
    *reinterpret_cast<f64x2*>(lds + (mr == 0 ? d : (mr == d ? 0 : mr)) * 32 + 2 * (threadIdx.x & 15)) = entries;
    __syncthreads();                                         // also: every wave has read the tile
    // columns 4 wave + 2 h and the next one of Z . M_t; column m of it is column sigma(m) of the new state
    const double* m = lds + 4 * wave + 2 * h;
    double acc[2] = {0.0, 0.0};
#pragma unroll
    for (int r = 0; r < 32; ++r) {
        const f64x2 e = *reinterpret_cast<const f64x2*>(m + 32 * r);
        acc[0] = acc[0] + x[r >> 1][r & 1] * e[0];
        acc[1] = acc[1] + x[r >> 1][r & 1] * e[1];
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int mc = 4 * wave + 2 * h + k, c = mc == 0 ? d : (mc == d ? 0 : mc);
        if (row < n) z[((c >> 1) * n + row) * 2 + (c & 1)] = acc[k];
        const unsigned long long top = half_max(abs_bits(acc[k]));
        if (row == 0 && top) atomicMax(mine + c, top);
    }
}

// The last product, the peaks, the first minimum, the kept product rounded to fp32.
__global__ __launch_bounds__(64 * kStepWaves) void construct_final_kernel(ConstructParams p) {
    __shared__ double lds[2048];
    __shared__ unsigned long long wbest[kStepWaves];
    __shared__ int wstep[kStepWaves];
    Workspace w = carve(p.workspace, p.steps);
    if (p.steps > 0) {
        const unsigned long long last = column_max(w, p.steps, threadIdx.x & 63);
        if (threadIdx.x < 32) w.colmax[(size_t)p.steps * 32 + threadIdx.x] = last;
        extend_product(w, p.steps, lds);
        __syncthreads();
    }
    unsigned long long best = ~0ull;
    int bt = 0;
    for (int t = threadIdx.x; t <= p.steps; t += 64 * kStepWaves) {
        unsigned long long peak = 0ull;
#pragma unroll
        for (int c = 0; c < 32; ++c) peak = max_u64(peak, w.colmax[(size_t)t * 32 + c]);
        if (p.peaks) p.peaks[t] = __longlong_as_double((long long)peak);
        if (peak < best) { best = peak; bt = t; }
    }
    auto better = [&](unsigned long long b, int s) {
        if (b < best || (b == best && s < bt)) { best = b; bt = s; }
    };
    for (int off = 32; off > 0; off >>= 1) {
        const unsigned long long b = __shfl_xor(best, off);
        const int s = __shfl_xor(bt, off);
        better(b, s);
    }
    if ((threadIdx.x & 63) == 0) { wbest[threadIdx.x >> 6] = best; wstep[threadIdx.x >> 6] = bt; }
    __syncthreads();                                         // also: the last product is in its slot
    for (int k = 0; k < kStepWaves; ++k) better(wbest[k], wstep[k]);
    if (threadIdx.x == 0) {
        p.info[0] = (int)(0xFFFFFFFFu - (uint32_t)(*w.key & 0xFFFFFFFFull));
        p.info[1] = bt;
    }
    const double* r = w.slots + (size_t)bt * 1024;
    for (int e = threadIdx.x; e < 1024; e += 64 * kStepWaves) p.R_out[e] = bt > 0 ? (float)r[e] : (e / 32 == e % 32 ? 1.0f : 0.0f);
}

// ---- All steps in one launch ---------------------------------------------------------------------------------------
struct SearchPlan {
    int partials;                        // keys of the block search
    int tiles;                           // workgroups that hold rows of the state; those behind them hold the product R^(t)
    int participants;                    // all of them
    uint32_t patience;                   // looks at what the others have published before one gives up; 0: gives up in any case
    int cus;                             // CUs they have
    int few;                             // workgroups of the search behind it
    int asked;                           // for those: the word of given_up that asks for them; the next one is theirs
};

// What the workgroups tell each other after step t: two words each, the largest magnitude among their rows and the smallest
// channel it stands in, into set t % 2.  Bit 63 of a word (a magnitude's sign, so free) changes with every use of a set and says
// that the word is there: (t / 2) % 2, opposite to what was there before.  Nobody writes set t % 2 again before everybody has read
// it: a workgroup publishes step t + 2 after it has seen all of step t + 1, which they publish after reading step t.  The words
// are relaxed atomics of device scope, which the eight L2s do not keep to themselves; nothing else passes between workgroups, so no
// cache has to be written back or invalidated (with an acquire per exchange instead the exchange alone takes longer than a step).
// Requests to one line are served one after the other: eight copies of everyone's words.  (Side by side: with 64 bytes for each and
// two copies an exchange alone is faster, but the steps slower, 2048 rows 375 against 338 us for 128: more requests per look.)
__device__ __forceinline__ uint32_t exchange_at(int participants, int copy, int who) {
    return (uint32_t)(copy * participants + who) * kExchangeWords;
}
inline size_t exchange_bytes(int participants) { return (size_t)2 * kExchangeCopies * participants * kExchangeWords * 8; }

// Keys of the block search, the matrices of all steps, and nothing published yet.
__global__ __launch_bounds__(256) void construct_prepare_kernel(ConstructParams p, SearchPlan s) {
    __shared__ double q[31 * 31];
    Workspace w = carve(p.workspace, p.steps);
    const int words = 2 * kExchangeCopies * kExchangeWords * s.participants;
    const int at = blockIdx.x * 256 + threadIdx.x;
    if (at < 2) w.given_up[at] = 0ull;
    if (at < 4 * s.few) w.colmax[at] = ~0ull;
    for (int i = at; i < words; i += gridDim.x * 256) reinterpret_cast<unsigned long long*>(w.z)[i] = ~0ull;
    if ((int)blockIdx.x < s.partials) block_key(p, w, s.partials, reinterpret_cast<unsigned long long*>(q));
    else step_matrix(p, w, (int)blockIdx.x - s.partials + 1, q);
}

// value of lane N of each 16 lanes, in all 16
template <int N>
__device__ __forceinline__ double row16_broadcast(double v) {
    return __longlong_as_double(__builtin_amdgcn_update_dpp(0ll, __double_as_longlong(v), 0x150 + N, 0xF, 0xF, true));
}

template <typename F, int... I>
__device__ __forceinline__ void each_row(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}

// Every LDS access this wave has issued has completed, then workgroup barrier (loads from memory stay in flight).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// A workgroup holds 16 RH rows.  Lane (i, q) = (lane % 16, lane / 16) of wave (rh, cs) computes RH columns of row 16 rh + i: the
// row is in its registers, read from LDS while the exchange is under way, and the entries of M_t are in the registers of the 16
// lanes that need the same ones, from where an ALU move hands them round: read from LDS by every lane they cost more than the
// products (32 rows: 2048 cycles of LDS against 1024 of fp64).
template <int RH, int LOOKS, int PER_CU>
__global__ __launch_bounds__(64 * kStepWaves, 2 * PER_CU) void construct_search_kernel(ConstructParams p, SearchPlan s) {
    constexpr int kRows = 16 * RH, kPitch = 34, kMPitch = 33;
    __shared__ __attribute__((aligned(16))) double z[2][kRows * kPitch];   // the state after even and odd steps
    __shared__ double mt[2][32 * kMPitch];                   // M_t by columns, likewise
    __shared__ unsigned long long colmax[32], seen[64], red[kStepWaves];
    __shared__ int seen_channel[64];
    const Workspace w = carve(p.workspace, p.steps);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i = lane & 15, q = lane >> 4;
    const int row = (wave % RH) * 16 + i, col0 = ((wave / RH) * 4 + q) * RH;
    const bool product = (int)blockIdx.x >= s.tiles;         // the rows of R^(t), updated like rows of the state
    const int64_t grow = ((int64_t)blockIdx.x - (product ? s.tiles : 0)) * kRows + row;
    const bool counts = !product && grow < p.T;
    const int mr = threadIdx.x >> 4, mc = 2 * (threadIdx.x & 15);   // this thread's two entries of a matrix on its way to LDS
    auto matrix = [&](int t) {                               // (a uniform address and a 32-bit offset, here and below: registers)
        return reinterpret_cast<const f64x2*>(w.slots + (size_t)(t < p.steps ? t : p.steps) * 1024)[threadIdx.x];
    };
    auto stage = [&](int t, const f64x2& e) {
        mt[t & 1][mc * kMPitch + mr] = e[0];
        mt[t & 1][(mc + 1) * kMPitch + mr] = e[1];
    };
    double acc[RH], kept[RH];
    int at[RH], kept_at[RH];                                 // channels of acc and kept
    auto take = [&](int t) {                                 // the new values of this lane's row
#pragma unroll
        for (int k = 0; k < RH; ++k) {
            z[t & 1][row * kPitch + at[k]] = acc[k];
            const unsigned long long top = row16_max(counts ? abs_bits(acc[k]) : 0ull);
            if (i == 0 && top) atomicMax(&colmax[at[k]], top);
        }
    };

    if (threadIdx.x < 32) colmax[threadIdx.x] = 0ull;
    const unsigned long long key = chosen_key(w, s.partials, red);   // (holds a barrier: colmax is cleared)
    const int64_t block = block_of(key);
    f64x2 next = {0.0, 0.0};
    if (p.steps > 0) {
        stage(1, matrix(1));
        next = matrix(2);
    }
#pragma unroll
    for (int k = 0; k < RH; ++k) {
        at[k] = col0 + k;
        kept_at[k] = at[k];
        acc[k] = 0.0;
        if (product) acc[k] = grow == at[k] ? 1.0 : 0.0;
        else if (counts) acc[k] = (double)__uint_as_float((uint32_t)p.x[grow * p.ldx + 32 * block + at[k]] << 16);
        kept[k] = acc[k];
    }
    take(0);
    lds_barrier();

    unsigned long long* const words = reinterpret_cast<unsigned long long*>(w.z);
    const uint32_t set_words = exchange_at(s.participants, kExchangeCopies, 0);
    unsigned long long lowest = ~0ull;
    int steps_kept = 0;
    for (int t = 0;; ++t) {
        const unsigned long long there = (unsigned long long)((t >> 1) & 1) << 63;
        unsigned long long* const set = words + ((t & 1) ? set_words : 0u);
        if (wave == 0) {
            const unsigned long long cm = lane < 32 ? colmax[lane] : 0ull;
            unsigned long long top;
            const int d = __ffsll(lanes_of_max(cm, top)) - 1;
            if (lane < kExchangeCopies) {
                unsigned long long* const mine = set + exchange_at(s.participants, lane, blockIdx.x);
                __hip_atomic_store(mine, top | there, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(mine + 1, (unsigned long long)d | there, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            if (lane < 32) colmax[lane] = 0ull;
        }
        const double* zr = &z[t & 1][row * kPitch];
        double x[32];
#pragma unroll
        for (int k = 0; k < 32; ++k) x[k] = zr[k];           // while the exchange is under way
        if (wave == 0) {                                     // this wave waits, lane l for l, l + 64, ...
            const unsigned long long* const copy = set + exchange_at(s.participants, blockIdx.x % kExchangeCopies, 0);
            // Whoever looks too early is in the way of those still publishing (128 steps, 2048 rows, 130 workgroups, in an earlier
            // form of this loop: 374 us without the pause, 323 with 8 here, 293 with 12, 282 with 16, 313 with 24; 6 workgroups: 241
            // without, 243 with 12, 256 with 16)
            __builtin_amdgcn_s_sleep(LOOKS > 1 ? 12 : 10);
            unsigned long long best = 0ull;
            int channel = 32;
            bool here = s.patience > 0;
            uint32_t looks = 0;
            for (int first = 0; first < s.participants; first += 64 * LOOKS) {
                unsigned long long v[LOOKS], d[LOOKS], all;  // bit 63 of all: not everyone's words are there
                do {
                    all = 0ull;
#pragma unroll
                    for (int k = 0; k < LOOKS; ++k) {
                        const int l = first + 64 * k + lane, who = l < s.participants ? l : s.participants - 1;   // lanes without one: the last
                        const unsigned long long* const theirs = copy + (uint32_t)who * kExchangeWords;
                        v[k] = __hip_atomic_load(theirs, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ^ there;
                        d[k] = __hip_atomic_load(theirs + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ^ there;
                    }
#pragma unroll
                    for (int k = 0; k < LOOKS; ++k) all |= v[k] | d[k];
                } while (__any((all >> 63) != 0) && ++looks < s.patience);
                here = here & ((all >> 63) == 0);
#pragma unroll
                for (int k = 0; k < LOOKS; ++k) {            // no branch: & and | of the comparisons
                    const bool more = (v[k] > best) | ((v[k] == best) & ((int)d[k] < channel));
                    best = more ? v[k] : best;
                    channel = more ? (int)d[k] : channel;
                }
            }
            seen[lane] = best;
            seen_channel[lane] = here ? channel : -1;
        }
        lds_barrier();
        // largest magnitude of all, in the smallest channel
        const unsigned long long v = seen[lane];
        const int c = seen_channel[lane];
        const bool missing = c < 0;
        const bool given_up = __any(missing);
        unsigned long long peak, tops = lanes_of_max(v, peak);
        int d = __builtin_amdgcn_readlane(c, __ffsll(tops) - 1);
        while (tops &= tops - 1) {                           // almost always one
            const int other = __builtin_amdgcn_readlane(c, __ffsll(tops) - 1);
            d = other < d ? other : d;
        }
        if (given_up) {                                      // the same for every thread of the workgroup
            if (threadIdx.x == 0) __hip_atomic_store(w.given_up, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return;
        }
        if (product) {
            if (peak < lowest) {
                lowest = peak;
                steps_kept = t;
#pragma unroll
                for (int k = 0; k < RH; ++k) { kept[k] = acc[k]; kept_at[k] = at[k]; }
            }
            if (p.peaks && (int)blockIdx.x == s.tiles && threadIdx.x == 0) p.peaks[t] = __longlong_as_double((long long)peak);
        }
        if (t == p.steps) break;

        // step t + 1: row . M with the rows of M in the order sigma(0), sigma(1), ..., sigma exchanging 0 and d
        auto sigma = [&](int r) { return r == 0 ? d : (r == d ? 0 : r); };
        double lo[RH], hi[RH];
        const int r0 = sigma(i), r1 = sigma(16 + i);
#pragma unroll
        for (int k = 0; k < RH; ++k) {
            const double* m = &mt[(t + 1) & 1][(col0 + k) * kMPitch];
            lo[k] = m[r0];
            hi[k] = m[r1];
            acc[k] = 0.0;
            at[k] = sigma(col0 + k);
        }
        if (t + 2 <= p.steps) {
            stage(t + 2, next);                              // its last reader was step t
            next = matrix(t + 3);
        }
        auto term = [&](auto rc) {
            constexpr int R = decltype(rc)::value;
#pragma unroll
            for (int k = 0; k < RH; ++k) acc[k] = acc[k] + x[R] * row16_broadcast<R % 16>(R < 16 ? lo[k] : hi[k]);
            if constexpr (R % 4 == 3) {                      // the compiler gathers the moves of all rows ahead of the products otherwise
#pragma unroll
                for (int k = 0; k < RH; ++k) asm volatile("" : "+v"(acc[k]), "+v"(lo[k]), "+v"(hi[k]));
            }
        };
        each_row(term, std::make_integer_sequence<int, 32>{});
        take(t + 1);
        lds_barrier();
    }
    if (product) {
        if (grow < 32) {
#pragma unroll
            for (int k = 0; k < RH; ++k) p.R_out[grow * 32 + kept_at[k]] = (float)kept[k];
        }
        if ((int)blockIdx.x == s.tiles && threadIdx.x == 0) {
            p.info[0] = (int)block;
            p.info[1] = steps_kept;
        }
    }
}

// The search again where the search kernel's workgroups did not come to run together: in a few workgroups, which find room where
// hundreds do not, and if not even these did, in one, which waits for nobody.  The rows are in memory, a lane has a row at a time,
// 64 rows going to the first wave of each workgroup in turn, then to the second.  The same result; bound by the reads of M_t from LDS.
__global__ __launch_bounds__(64 * kStepWaves, 4) void construct_again_kernel(ConstructParams p, SearchPlan s) {
    __shared__ __attribute__((aligned(16))) double m[1024];
    __shared__ double product[1024], best[1024];
    __shared__ unsigned long long red[kStepWaves], peak_of_all;
    __shared__ int red_channel[kStepWaves], channel_of_all;
    const Workspace w = carve(p.workspace, p.steps);
    if (w.given_up[s.asked] == 0ull) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t first = ((int64_t)wave * gridDim.x + blockIdx.x) * 64, stride = (int64_t)64 * kStepWaves * gridDim.x;
    const int64_t block = block_of(chosen_key(w, s.partials, red));
    const bool writes = blockIdx.x == 0;                     // this workgroup has the product R^(t) and the results
    unsigned long long top = 0ull;                           // the largest magnitude this lane has seen, and its smallest channel
    int channel = 32;
    auto seen = [&](double v, int c) {
        const unsigned long long a = abs_bits(v);
        const bool more = (a > top) | ((a == top) & (c < channel));
        top = more ? a : top;
        channel = more ? c : channel;
    };
    for (int e = threadIdx.x; e < 1024; e += 64 * kStepWaves) product[e] = best[e] = e / 32 == e % 32 ? 1.0 : 0.0;
    for (int64_t r = first + lane; r < p.T; r += stride)
        for (int c = 0; c < 32; ++c) {
            const double v = (double)__uint_as_float((uint32_t)p.x[r * p.ldx + 32 * block + c] << 16);
            w.z[r * 32 + c] = v;
            seen(v, c);
        }
    unsigned long long lowest = ~0ull;
    int steps_kept = 0;
    for (int t = 0;; ++t) {
        // the workgroup's largest magnitude and the smallest channel it stands in
        auto smallest_channel = [&](unsigned long long v, int c, unsigned long long of) { return 32 - (int)wave_max(v == of ? 32 - c : 0); };
        const unsigned long long wave_top = wave_max(top);
        const int wave_channel = smallest_channel(top, channel, wave_top);
        __syncthreads();                                     // the last reader of red was the exchange before, or chosen_key
        if (lane == 0) { red[wave] = wave_top; red_channel[wave] = wave_channel; }
        __syncthreads();
        if (wave == 0) {
            unsigned long long v = lane < kStepWaves ? red[lane] : 0ull;
            int c = lane < kStepWaves ? red_channel[lane] : 32;
            unsigned long long peak = wave_max(v);
            int d = smallest_channel(v, c, peak);
            if (gridDim.x > 1) {                             // among all, by the rules of the search kernel's exchange
                const unsigned long long there = (unsigned long long)((t >> 1) & 1) << 63;
                unsigned long long* const set = w.colmax + (t & 1) * 2 * gridDim.x;
                if (lane == 0) {
                    __hip_atomic_store(set + 2 * blockIdx.x, peak | there, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(set + 2 * blockIdx.x + 1, (unsigned long long)d | there, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                const unsigned long long* const theirs = set + 2 * (lane < (int)gridDim.x ? lane : (int)gridDim.x - 1);
                unsigned long long dd;
                uint32_t looks = 0;
                bool missing;
                do {
                    __builtin_amdgcn_s_sleep(8);
                    v = __hip_atomic_load(theirs, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ^ there;
                    dd = __hip_atomic_load(theirs + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ^ there;
                    missing = __any(((v | dd) >> 63) != 0);
                } while (missing && ++looks < s.patience);
                peak = wave_max(v);
                d = missing || s.patience == 0 ? -1 : smallest_channel(v, (int)dd, peak);
            }
            if (lane == 0) { peak_of_all = peak; channel_of_all = d; }
        }
        __syncthreads();
        const unsigned long long peak = peak_of_all;
        const int d = channel_of_all;
        if (d < 0) {                                         // the same for every thread of the workgroup
            if (threadIdx.x == 0) __hip_atomic_store(w.given_up + s.asked + 1, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return;
        }
        if (writes && p.peaks && threadIdx.x == 0) p.peaks[t] = __longlong_as_double((long long)peak);
        if (peak < lowest) {
            lowest = peak;
            steps_kept = t;
            for (int e = threadIdx.x; e < 1024; e += 64 * kStepWaves) best[e] = product[e];
        }
        if (t == p.steps) break;
        auto sigma = [&](int r) { return r == 0 ? d : (r == d ? 0 : r); };
        for (int e = threadIdx.x; e < 1024; e += 64 * kStepWaves) m[sigma(e >> 5) * 32 + (e & 31)] = w.slots[(size_t)(t + 1) * 1024 + e];
        __syncthreads();
        top = 0ull;
        channel = 32;
        auto multiply = [&](double* z, bool counts) {
            double x[32];
#pragma unroll
            for (int k = 0; k < 32; ++k) x[k] = z[k];
#pragma unroll 1
            for (int c = 0; c < 32; c += 2) {
                double v0 = 0.0, v1 = 0.0;
#pragma unroll
                for (int k = 0; k < 32; ++k) {
                    const f64x2 e = *reinterpret_cast<const f64x2*>(m + k * 32 + c);
                    v0 = v0 + x[k] * e[0];
                    v1 = v1 + x[k] * e[1];
                }
                z[sigma(c)] = v0;
                z[sigma(c + 1)] = v1;
                if (counts) { seen(v0, sigma(c)); seen(v1, sigma(c + 1)); }
            }
        };
        for (int64_t r = first + lane; r < p.T; r += stride) multiply(w.z + r * 32, true);
        if (writes && wave == kStepWaves - 1 && lane < 32) multiply(product + lane * 32, false);
    }
    __syncthreads();
    if (!writes) return;
    for (int e = threadIdx.x; e < 1024; e += 64 * kStepWaves) p.R_out[e] = (float)best[e];
    if (threadIdx.x == 0) {
        p.info[0] = (int)block;
        p.info[1] = steps_kept;
    }
}

}  // namespace

size_t construct_workspace_bytes(int64_t T, int steps) {
    return 64 + (size_t)(steps + 1) * 256 + (size_t)(steps + 1) * 8192 + (size_t)T * 256;
}

namespace {

// CUs that a kernel on the stream can be given: the device's (fewer than a whole chip's where it is partitioned), or those of the
// stream's mask.
int cus_of(hipStream_t stream) {
    int dev = 0, n = 0;
    uint32_t mask[32] = {};
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (hipExtStreamGetCUMask(stream, 32, mask) != hipSuccess) {
        (void)hipGetLastError();                             // not the caller's to find
        return n;
    }
    int masked = 0;
    for (uint32_t word : mask) masked += __builtin_popcount(word);
    return masked > 0 && masked < n ? masked : n;
}

// One launch for all steps (form: DUQPP_CONSTRUCT_ONE_*); false: the workspace has no room for what they publish, or there
// would be more workgroups than run at once on so many CUs.
bool plan_search(int64_t T, int steps, int form, int cus, SearchPlan& s) {
    const int64_t rows = 16 << (form - DUQPP_CONSTRUCT_ONE_16), tiles = (T + rows - 1) / rows, all = tiles + (rows < 32 ? 2 : 1);
    if (all > (form == DUQPP_CONSTRUCT_ONE_16 ? cus : 2 * (int64_t)cus) || (int64_t)exchange_bytes((int)all) > T * 256) return false;
    // of the search behind it: not more than have rows, nor than the place of their words holds
    const int64_t waves = (T + 63) / 64, room = 8 * ((int64_t)steps + 1);
    int64_t few = waves < kFewWorkgroups ? waves : kFewWorkgroups;
    few = few < room ? few : room;
    s = SearchPlan{0, (int)tiles, (int)all, kPatience, cus, (int)few, 0};
    return true;
}

hipError_t launch_search(const ConstructParams& p, const SearchPlan& s, int form, uint32_t patience_again, hipStream_t stream) {
    hipError_t e = launch(construct_prepare_kernel, dim3((unsigned)(s.partials + p.steps)), dim3(256), 0, stream, p, s);
    if (e != hipSuccess) return e;
    const dim3 grid((unsigned)s.participants), block(64 * kStepWaves);
    if (form == DUQPP_CONSTRUCT_ONE_16)
        e = s.participants <= 64 ? launch(construct_search_kernel<1, 1, 1>, grid, block, 0, stream, p, s)
                                 : launch(construct_search_kernel<1, 4, 1>, grid, block, 0, stream, p, s);
    else
        e = s.participants <= s.cus ? launch(construct_search_kernel<2, 4, 1>, grid, block, 0, stream, p, s)
                                     : launch(construct_search_kernel<2, 2, 2>, grid, block, 0, stream, p, s);
    if (e != hipSuccess) return e;
    SearchPlan again = s;
    again.patience = patience_again;
    if (s.few > 1) {
        e = launch(construct_again_kernel, dim3((unsigned)s.few), block, 0, stream, p, again);
        if (e != hipSuccess) return e;
        again.asked = 1;
    }
    return launch(construct_again_kernel, dim3(1), block, 0, stream, p, again);
}

hipError_t launch_steps(const ConstructParams& p, int partials, hipStream_t stream) {
    hipError_t e = launch(construct_blockmax_kernel, dim3(partials), dim3(256), 0, stream, p);
    if (e != hipSuccess) return e;
    const unsigned tiles = (unsigned)((p.T + kTileRows - 1) / kTileRows);
    e = launch(construct_extract_kernel, dim3(tiles), dim3(64 * kStepWaves), 0, stream, p, partials);
    if (e != hipSuccess) return e;
    e = launch(construct_matrices_kernel, dim3(p.steps + 1), dim3(256), 0, stream, p);
    if (e != hipSuccess) return e;
    for (int t = 1; t <= p.steps; ++t) {
        e = launch(construct_step_kernel, dim3(tiles + 1), dim3(64 * kStepWaves), 0, stream, p, t);
        if (e != hipSuccess) return e;
    }
    return launch(construct_final_kernel, dim3(1), dim3(64 * kStepWaves), 0, stream, p);
}

}  // namespace

int construct_form(int64_t T, int steps, int form, int cus) {
    SearchPlan s{};
    if (form == DUQPP_CONSTRUCT_AUTO) {
        form = DUQPP_CONSTRUCT_ONE_16;
        while (form < DUQPP_CONSTRUCT_STEPS && !plan_search(T, steps, form, cus, s)) ++form;
    }
    return form == DUQPP_CONSTRUCT_STEPS || plan_search(T, steps, form, cus, s) ? form : -1;
}

hipError_t launch_construct_rotation(const ConstructParams& p, int how, hipStream_t stream, bool& runs) {
    const int64_t chunks = (int64_t)p.T * (p.K / 8);
    const int partials = (int)((chunks + 1023) / 1024 < kMaxPartials ? (chunks + 1023) / 1024 : kMaxPartials);
    const int cus = cus_of(stream), form = construct_form(p.T, p.steps, how & ~DUQPP_CONSTRUCT_ALONE, cus);
    runs = form >= 0;
    if (!runs) return hipSuccess;
    if (form == DUQPP_CONSTRUCT_STEPS) return launch_steps(p, partials, stream);
    SearchPlan s{};
    plan_search(p.T, p.steps, form, cus, s);
    s.partials = partials;
    if (how & DUQPP_CONSTRUCT_IMPATIENT) s.patience = 0;
    return launch_search(p, s, form, (how & DUQPP_CONSTRUCT_ALONE) == DUQPP_CONSTRUCT_ALONE ? 0 : kPatienceAgain, stream);
}

}  // namespace duqpp

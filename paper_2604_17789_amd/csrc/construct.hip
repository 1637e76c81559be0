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
// workgroups, unless only a few rows can hold it.  Three forms:
//   rows that count (construct_rows_kernel) where massive values leave at most 22 rows, beyond 992 rows 28, that can ever hold the largest magnitude, every one
//                   of sixteen workgroups follows just those, without an exchange.  Tried first by calls of up to 16352 rows.
//   search kernel   (construct_search_kernel) one launch for all steps: a workgroup keeps its 16 or 32 rows of the state in LDS and
//                   registers, publishes the largest magnitude among them after every step, waits for everybody's, and goes on.
//                   For as many rows as workgroups that run at once hold: 16 rows each and one workgroup per CU, or 32 rows
//                   and two per CU (T <= 16352 on 256 CUs).  Should they not come to run together, because other work holds the CUs for
//                   longer than they wait (1 to 2 ms), they give up, and up to 64 workgroups with the state in memory do the
//                   search (construct_again_kernel); should not even these come to run together (within 20 ms and more), the first
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
// per workgroup (K = 4096; the kernels of the form alone, none ahead of them): T = 64 554 / 244 / 337, 512 559 / 235 / 329,
// 1024 565 / 266 / -, 2048 601 / 262 / 325, 4096 705 / - / 333, 8192 1048 / - / 457, 16000 1550 / - / 562.  The call is offline.
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

// workspace: [header 64 B: u64 block key, u64 search given up, u64 given up again, u64 done by the rows that count][colmax (S + 1) x 32 u64][slots (S + 1) x 1024 f64][Z T x 32 f64]
// Slot 0 holds the block search's partial keys, then the maxima below; slot t >= 1 holds M_t = H . diag(1, Q'_t), then R^(t).
// The search kernel keeps the state on the chip; the place of Z holds what its workgroups publish, that of colmax what those of the
// kernel behind it do, and at its end, a word per step, how far the step's draw is from orthogonal.
struct Workspace {
    unsigned long long* key;
    unsigned long long* given_up;        // two words
    unsigned long long* done;
    unsigned long long* colmax;
    double* slots;
    double* z;
};
__host__ __device__ inline Workspace carve(void* ws, int steps) {
    Workspace w;
    uint8_t* p = static_cast<uint8_t*>(ws);
    w.key = reinterpret_cast<unsigned long long*>(p);
    w.given_up = w.key + 1;
    w.done = w.key + 3;
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
__device__ __forceinline__ void block_key(const ConstructParams& p, const Workspace& w, int index, int workgroups, unsigned long long* red) {
    const int64_t stride = (int64_t)workgroups * 256, at = (int64_t)index * 256 + threadIdx.x;
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
        reinterpret_cast<unsigned long long*>(w.slots)[index] = max_u64(max_u64(red[0], red[1]), max_u64(red[2], red[3]));
}

// Clears the first column maxima, and the keys.
__global__ __launch_bounds__(256) void construct_blockmax_kernel(ConstructParams p) {
    __shared__ unsigned long long red[4];
    Workspace w = carve(p.workspace, p.steps);
    if (blockIdx.x == 0 && threadIdx.x < 32) w.colmax[threadIdx.x] = 0ull;
    block_key(p, w, blockIdx.x, gridDim.x, red);
}

// The chosen block from the partial keys, in every thread of a workgroup.
template <int WAVES = kStepWaves>
__device__ __forceinline__ unsigned long long chosen_key(const Workspace& w, int partials, unsigned long long* red) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned long long key = 0ull;
    for (int i = threadIdx.x; i < partials; i += 64 * WAVES) key = max_u64(key, reinterpret_cast<const unsigned long long*>(w.slots)[i]);
    key = wave_max(key);
    if (lane == 0) red[wave] = key;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < WAVES; ++k) key = max_u64(key, red[k]);
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
    // a thread's four entries stand in one column, rows 8 apart
    const int i = threadIdx.x >> 5, j = threadIdx.x & 31;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    if (t > 0 && j > 0)
        for (int k = 1; k < 32; ++k) {
            const double v = q[(k - 1) * 31 + (j - 1)];
#pragma unroll
            for (int n = 0; n < 4; ++n) acc[n] = acc[n] + hadamard_entry(i + 8 * n, k) * v;
        }
#pragma unroll
    for (int n = 0; n < 4; ++n) out[threadIdx.x + 256 * n] = t > 0 && j == 0 ? hadamard_entry(i + 8 * n, 0) : acc[n];
}
__global__ __launch_bounds__(256) void construct_matrices_kernel(ConstructParams p) {
    __shared__ double q[31 * 31];
    step_matrix(p, carve(p.workspace, p.steps), blockIdx.x, q);
}

// The largest of the first LANES lanes' values (the others hold 0), uniform, and the lanes that hold it.
template <int LANES = 64>
__device__ __forceinline__ unsigned long long lanes_of_max(unsigned long long v, unsigned long long& top) {
    auto most = [](uint32_t m) {
        m = dpp_max<0x140>(dpp_max<0x141>(dpp_max<0x4E>(dpp_max<0xB1>(m))));
        if constexpr (LANES > 16) m = dpp_max<0x143>(dpp_max<0x142>(m));
        return (uint32_t)__builtin_amdgcn_readlane((int)m, LANES - 1);
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
    int leaves;                          // the exchange after which the first of those gives up, whatever it finds there; -1: none
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

// How far step t's draw is from orthogonal: the largest entry of |Q'.Q'^T - 1|, as the bits of a double (a NaN is larger than all).
__device__ __forceinline__ unsigned long long* deviation(const Workspace& w, int steps, int t) { return w.colmax + (size_t)(steps + 1) * 32 - t; }
__device__ __forceinline__ void step_deviation(const ConstructParams& p, const Workspace& w, int t, const double* q, unsigned long long* red) {
    unsigned long long most = 0ull;
    // the upper triangle: rows a and 30 - a of it have 32 entries together (row 15 comes twice)
    const int b = threadIdx.x & 31;
    int i[2], j[2];
    double acc[2] = {0.0, 0.0};
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        const int a = (threadIdx.x >> 5) + 8 * n;
        i[n] = b < 31 - a ? a : 30 - a;
        j[n] = b < 31 - a ? a + b : b - 1;
    }
    for (int k = 0; k < 31; ++k) {
#pragma unroll
        for (int n = 0; n < 2; ++n) acc[n] = acc[n] + q[31 * i[n] + k] * q[31 * j[n] + k];
    }
#pragma unroll
    for (int n = 0; n < 2; ++n) most = max_u64(most, abs_bits(i[n] == j[n] ? acc[n] - 1.0 : acc[n]));
    most = wave_max(most);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = most;
    __syncthreads();
    if (threadIdx.x == 0) *deviation(w, p.steps, t) = max_u64(max_u64(red[0], red[1]), max_u64(red[2], red[3]));
}

// The matrices of all steps, keys of the block search, and nothing published yet.
__global__ __launch_bounds__(256) void construct_prepare_kernel(ConstructParams p, SearchPlan s) {
    __shared__ double q[31 * 31];
    __shared__ unsigned long long red[4];
    Workspace w = carve(p.workspace, p.steps);
    const int words = 2 * kExchangeCopies * kExchangeWords * s.participants;
    const int at = blockIdx.x * 256 + threadIdx.x;
    if (at < 2) w.given_up[at] = 0ull;
    if (at == 2) *w.done = 0ull;
    if (at < 5 * s.few) w.colmax[at] = at < 4 * s.few ? ~0ull : 0ull;
    for (int i = at; i < words; i += gridDim.x * 256) reinterpret_cast<unsigned long long*>(w.z)[i] = ~0ull;
    if ((int)blockIdx.x < p.steps) {
        step_matrix(p, w, (int)blockIdx.x + 1, q);
        step_deviation(p, w, (int)blockIdx.x + 1, q, red);
    } else {
        block_key(p, w, (int)blockIdx.x - p.steps, s.partials, red);
    }
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
    const unsigned long long done = *w.done;
    const unsigned long long key = chosen_key(w, s.partials, red);   // (holds a barrier: colmax is cleared)
    if (done != 0ull) return;
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

// The search on the rows that count.  A step keeps a row's 2-norm, so that no entry of a row ever exceeds the norm the row begins
// with, while the row of the largest norm N always has an entry of N / sqrt(32) or more: rows with less than that never hold the
// largest magnitude, and the search need not follow them.  Activations with massive values leave few: of 2048 or 8192 tokens with a
// value of 900 and a channel at 50 times the others in the block 4 to 15, without such a channel one.  Up to kRowsKept of them, every
// workgroup does the whole search by itself, waits for nobody, and carries two rows of the product R^(t) along.
// Norms are kept as far as the draws are orthogonal, which the kernel ahead has measured: a singular value of Q' lies within
// sqrt(1 -+ 31 d), d the largest entry of |Q'.Q'^T - 1|.  With 31 d times the steps up to 0.02 norms stay within a factor of 0.9898
// to 1.0101, which the 0.95 below leaves room for (0.960 would do).  Otherwise, with more rows than that or with infinities or NaN
// the kernel leaves the search to the one behind it.
// A step is a chain of latencies of one workgroup, about 1700 cycles: 350 until the row is back from LDS, from where every lane needs all
// of it, 400 for the products that do not depend on the exchanged channel d, 230 for the largest magnitude, 250 for the two that do,
// 400 for the 32 additions in order and the next matrix column's way to registers.  128 steps on one MI355X, K = 4096, us, search kernel by itself /
// behind this: with massive values T = 64 250 / 102, 2048 266 / 106, 8160 347 / 124, 16000 563 / 151; without, where it only finds that out,
// 64 250 / 255, 2048 264 / 270, 8160 347 / 350, 16000 563 / 571.  (Calls from Python, which allocate: 2048 289 / 131 and 289 / 295.)
constexpr int kRowsWaves = 8;
constexpr int kRowsOnce = 2 * (kRowsWaves - 1);          // the first wave has two rows of the product, the others two rows each,
constexpr int kRowsKept = 2 * kRowsOnce;                 // and two more each where there are more
// So many pay: 1 to 6 rows take 102 to 119 us for 128 steps of 2048 rows, 7 to 14 162 to 185, 15 217, 20 228, 24 261, 28 272, the search kernel 267
// (8160 rows: 28 289, search 347); up to 992 rows, which the search kernel looks at in one go, 20 take 225, 24 257, 28 269, that 241 to 252.
constexpr int kRowsFew = 22;
constexpr int64_t kRowsFewTo = 992;
constexpr int kRowsBring = 4;                            // the last waves bring the matrices, whether they have rows or not
constexpr int kRowsWorkgroups = kBlock / 2;              // two rows of the product each
constexpr int64_t kRowsScanned = 16384;                  // rows whose norms fit beside each other
typedef double f64x16 __attribute__((ext_vector_type(16)));

// max(top, |v|) of finite values (the compiler's own first makes quiet NaN of signalling ones, an instruction more per operand)
__device__ __forceinline__ double larger(double top, double v) {
    asm("v_max_f64 %0, %0, |%1|" : "+v"(top) : "v"(v));
    return top;
}

__global__ __launch_bounds__(64 * kRowsWaves) void construct_rows_kernel(ConstructParams p, SearchPlan s) {
    constexpr int kPitch = 34, kThreads = 64 * kRowsWaves;
    constexpr int kRowsLds = 4 * kRowsWaves * kPitch;
    __shared__ __attribute__((aligned(16))) double lds[3 * 1024 + 2 * kRowsLds];
    __shared__ unsigned long long red[2][kRowsWaves];
    __shared__ int kept_rows[kRowsKept], count, many;
    double* const mt = lds;                                  // M_t in place t % 3
    double* const z = lds + 3 * 1024;                        // four rows of the state per wave, after even and odd steps
    uint16_t* const norms = reinterpret_cast<uint16_t*>(lds);    // before that: upper words of the squared norms
    static_assert(kRowsScanned * 2 <= (int64_t)sizeof(lds), "norms");
    const Workspace w = carve(p.workspace, p.steps);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    if (threadIdx.x == 0) count = many = 0;
    unsigned long long most = 0ull;
    for (int t = 1 + threadIdx.x; t <= p.steps; t += kThreads) most = max_u64(most, *deviation(w, p.steps, t));
    const unsigned long long key = chosen_key<kRowsWaves>(w, s.partials, red[0]);
    const int64_t block = block_of(key);
    most = wave_max(most);
    if (lane == 0) red[1][wave] = most;

    // squared norms: four lanes to a row, 16 rows of every wave in flight eight times
    const uint16_t* const xb = p.x + 32 * block + 8 * (threadIdx.x & 3);
    unsigned long long top = 0ull;
    const double largest = (double)__uint_as_float((uint32_t)(key >> 32) << 16);
    for (int64_t first = 0; first < p.T; first += 8 * (kThreads / 4)) {
        const int64_t r0 = first + (threadIdx.x >> 2);
        bool large = false;
        uint4 v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {                        // (no branch around the loads: past the end the last row)
            const int64_t r = r0 + k * (kThreads / 4);
            v[k] = *reinterpret_cast<const uint4*>(xb + (r < p.T ? r : p.T - 1) * p.ldx);
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const uint32_t words[4] = {v[k].x, v[k].y, v[k].z, v[k].w};
            double n = 0.0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const double lo = (double)__uint_as_float(words[j] << 16), hi = (double)__uint_as_float(words[j] & 0xFFFF0000u);
                n = n + lo * lo;
                n = n + hi * hi;
            }
            n = n + __shfl_xor(n, 1);
            n = n + __shfl_xor(n, 2);
            const unsigned long long bits = abs_bits(n);
            top = max_u64(top, bits);
            const int64_t r = r0 + k * (kThreads / 4);
            if ((threadIdx.x & 3) == 0 && r < p.T) {
                norms[r] = (uint16_t)(bits >> 48);
                large |= n >= 0.125 * largest * largest;
            }
        }
        // Where many of the first 1024 rows are not far below the largest magnitude there is no point in looking at the others: a row of
        // an eighth of its square counts unless N^2 is more than four times that.  (A quarter let activations pass that have channels at 50
        // times the others but no massive values, to find out from all rows: 128 steps, us, the search kernel by itself / behind this one with a
        // quarter / with an eighth: T = 4064 273 / 289 / 280, 16000 564 / 608 / 571.  Asked behind every 1024 rows it costs those that go on 20 us
        // at 16000.)
        if (first == 0 && p.T > kRowsKept) {
            const int here = __popcll(__ballot(large));
            if (lane == 0 && here) atomicAdd(&many, here);
            __syncthreads();
            if (many > kRowsKept) return;                    // here and below the same for every thread of the launch
        }
    }
    __syncthreads();                                         // red[0] has been read
    top = wave_max(top);
    if (lane == 0) red[0][wave] = top;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kRowsWaves; ++k) {
        top = max_u64(top, red[0][k]);
        most = max_u64(most, red[1][k]);
    }
    if ((top >> 52) == 0x7FF) return;                        // infinities or NaN
    const bool orthogonal = __longlong_as_double((long long)most) * 31.0 * p.steps <= 0.02;   // (false for a NaN)
    if (!orthogonal) return;                                 // (also with few rows: nothing becomes infinite below)
    const unsigned long long least = (unsigned long long)__double_as_longlong(__longlong_as_double((long long)top) * (0.95 / 32.0)) >> 48;
    for (int64_t r = threadIdx.x; r < p.T; r += kThreads)
        if (norms[r] >= least) {                             // (upper words: less is less of the whole, equal stays)
            const int i = atomicAdd(&count, 1);
            if (i < kRowsKept) kept_rows[i] = (int)r;
        }
    __syncthreads();
    const int kept = __builtin_amdgcn_readfirstlane(count);
    if (kept > (p.T <= kRowsFewTo ? kRowsFew : kRowsKept)) return;
    for (int e = threadIdx.x; e < 2 * kRowsLds; e += kThreads) z[e] = 0.0;   // rows that nobody has
    __syncthreads();
    if (blockIdx.x == 0 && threadIdx.x == 0) *w.done = 1ull;
    const bool product = wave == 0, works = product || 2 * (wave - 1) < kept, brings = wave >= kRowsWaves - kRowsBring;
    const bool twice = !product && kRowsOnce + 2 * (wave - 1) < kept;
    if (!works && !brings) return;                           // (a wave that has ended no longer counts for the barriers)

    // Lane (h, c) has a row, and column c of the matrices: of the first wave row h of the workgroup's two of the product, of the others
    // row h of two of those that count, and perhaps of two more
    const int h = lane >> 5, c = lane & 31;
    const int prow = 2 * (int)blockIdx.x + h;
    double* const mine = z + (4 * wave + h) * kPitch;
    auto state = [&](int i) {
        return i < kept ? (double)__uint_as_float((uint32_t)p.x[kept_rows[i] * p.ldx + 32 * block + c] << 16) : 0.0;
    };
    double acc = product ? (prow == c ? 1.0 : 0.0) : state(2 * (wave - 1) + h), more = twice ? state(kRowsOnce + 2 * (wave - 1) + h) : 0.0;
    double best = acc;
    int at = c, best_at = c;                                 // the channels of acc and more, and of best
    unsigned long long lowest = ~0ull;
    int steps_kept = 0;
    // A matrix comes from memory a step ahead of its way to LDS, four entries a thread
    const int bringer = threadIdx.x - 64 * (kRowsWaves - kRowsBring);
    auto matrix = [&](int t, int k) {
        return reinterpret_cast<const f64x2*>(w.slots + (size_t)(t < p.steps ? t : p.steps) * 1024)[bringer + 64 * kRowsBring * k];
    };
    auto stage = [&](int place, const f64x2* e) {
#pragma unroll
        for (int k = 0; k < 2; ++k) reinterpret_cast<f64x2*>(mt + place)[bringer + 64 * kRowsBring * k] = e[k];
    };
    f64x2 next[2] = {};
    if (brings && p.steps > 0) {
        const f64x2 first[2] = {matrix(1, 0), matrix(1, 1)};
        stage(0, first);
        next[0] = matrix(2, 0);
        next[1] = matrix(2, 1);
    }
    lds_barrier();
    // places of M_{t+1}, M_{t+2} and M_{t+3}; the last was read in step t - 1, a barrier before M_{t+3} comes
    int m1 = 0, m2 = 1024, m3 = 2048;
    auto bring = [&](int t) {
        if (brings && t + 2 <= p.steps) {
            stage(m2, next);
            next[0] = matrix(t + 3, 0);
            next[1] = matrix(t + 3, 1);
        }
    };
    auto turn = [&] {
        const int m0 = m1;
        m1 = m2;
        m2 = m3;
        m3 = m0;
    };
    if (!works) {
        for (int t = 0; t <= p.steps; ++t) {
            bring(t);
            turn();
            lds_barrier();
        }
        return;
    }
    double m[32];                                            // column c of M_{t+1}
    auto column = [&](int place) {
#pragma unroll
        for (int r = 0; r < 32; ++r) m[r] = mt[place + r * 32 + c];
    };
    column(m1);
    // Where the loop's code lies among the 32 bytes fetched at once is 1 to 5 % of the call, whatever ends ahead of it: of the eight places
    // (1 / 7 / 14 rows that count, 64 rows, us: 103 / 160 / 179 here, 103 / 159 / 182, 104 / 164 / 181, 105 / 157 / 181, 105 / 161 / 183,
    // 105 / 164 / 182, 107 / 160 / 181, 108 / 167 / 184)
    asm volatile(".p2align 5\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0");
    for (int t = 0;; ++t) {
        double* const z0 = mine + (t & 1) * kRowsLds;
        double* const z1 = z0 + 2 * kPitch;
        z0[at] = acc;
        if (twice) z1[at] = more;
        bring(t);
        __builtin_amdgcn_sched_barrier(0);
        f64x2 x[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) x[k] = *reinterpret_cast<const f64x2*>(z0 + 2 * k);
        __builtin_amdgcn_sched_barrier(0);
        // What has been written is there (accesses complete in order, at most 12 are left and 16 reads stand behind the writes), the rest
        // of the reads is on its way
        asm volatile("s_waitcnt lgkmcnt(12)\n\ts_barrier" ::: "memory");
        // the largest magnitude of each channel, lane (h, c) among rows h and 2 + h of all waves
        const double* const column_c = z + (t & 1) * kRowsLds + h * kPitch + c;
        double top = 0.0, of[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) of[k] = column_c[4 * (k + 1) * kPitch];
        __builtin_amdgcn_sched_barrier(0);
        f64x16 lo, hi;                                       // x_r . M[r][c], right for all r but 0 and d
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            lo[r] = x[r / 2][r % 2] * m[r];
            hi[r] = x[8 + r / 2][r % 2] * m[16 + r];
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) asm volatile("" ::"v"(lo[r]), "v"(hi[r]));   // made here, not behind d
#pragma unroll
        for (int k = 0; k < 3; ++k) top = larger(top, of[k]);
        if (kept > 6) {
#pragma unroll
            for (int k = 4; k < kRowsWaves; ++k) top = larger(top, column_c[4 * k * kPitch]);
        }
        if (kept > kRowsOnce) {
#pragma unroll
            for (int k = 1; k < kRowsWaves; ++k) top = larger(top, column_c[(4 * k + 2) * kPitch]);
        }
        unsigned long long peak;
        const unsigned long long lanes = lanes_of_max(abs_bits(top), peak);
        const int d = __builtin_amdgcn_readfirstlane(__ffs((uint32_t)lanes | (uint32_t)(lanes >> 32)) - 1);
        if (product) {
            if (peak < lowest) {
                lowest = peak;
                steps_kept = t;
                best = acc;
                best_at = at;
            }
            if (p.peaks && blockIdx.x == 0 && threadIdx.x == 0) p.peaks[t] = __longlong_as_double((long long)peak);
        }
        if (t == p.steps) break;
        // row . M with the rows of M in the order sigma(0), sigma(1), ..., sigma exchanging 0 and d
        const double md = mt[m1 + d * 32 + c], first = z0[0] * md, other = z0[d] * m[0];
        if (twice) {
            const double other1 = z1[d] * m[0];
            more = 0.0 + z1[0] * md;
#pragma unroll
            for (int r = 1; r < 32; ++r) {
                const double term = z1[r] * m[r];
                more = more + (r == d ? other1 : term);
            }
        }
        lo[d < 16 ? d : 0] = other;                          // (term 0 is `first`)
        hi[d < 16 ? 0 : d - 16] = d < 16 ? hi[0] : other;    // (no branch: the compiler copies the whole vector around one)
        __builtin_amdgcn_sched_barrier(0);
        column(m2);                                          // while the additions run (past the last step whatever stands there)
        __builtin_amdgcn_sched_barrier(0);
        acc = 0.0 + first;
#pragma unroll
        for (int r = 1; r < 16; ++r) acc = acc + lo[r];
#pragma unroll
        for (int r = 0; r < 16; ++r) acc = acc + hi[r];
        at = c == 0 ? d : (c == d ? 0 : c);
        turn();
    }
    if (product) {
        p.R_out[prow * 32 + best_at] = (float)best;
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            p.info[0] = (int)block;
            p.info[1] = steps_kept;
        }
    }
}

// The search again where the search kernel's workgroups did not come to run together: in a few workgroups, which find room where
// hundreds do not, and if not even these did, in the first of them, which waits for nobody then.  The rows are in memory, a lane has a row at a time,
// 64 rows going to the first wave of each workgroup in turn, then to the second.  The same result; bound by the reads of M_t from LDS.
constexpr unsigned long long kNotBegun = 0, kBegun = 1, kLeft = 2;

__global__ __launch_bounds__(64 * kStepWaves, 4) void construct_again_kernel(ConstructParams p, SearchPlan s) {
    __shared__ __attribute__((aligned(16))) double m[1024];
    __shared__ double product[1024], best[1024];
    __shared__ unsigned long long red[kStepWaves], peak_of_all;
    __shared__ int red_channel[kStepWaves], channel_of_all;
    const Workspace w = carve(p.workspace, p.steps);
    __shared__ int goes;
    if (w.given_up[0] == 0ull) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // A workgroup that begins says so, unless the first has given up by then, and when it leaves, whether it has given up or done all
    // steps (it may have seen everybody's words of the last one where the first looked too early).  The first goes on alone when those that
    // began have left: they wait for nobody for longer than it did, and what they wrote must not come after what it writes.
    unsigned long long* const state = w.colmax + 4 * s.few;
    if (blockIdx.x > 0) {
        if (threadIdx.x == 0) goes = atomicCAS(state + blockIdx.x, kNotBegun, kBegun) == kNotBegun;
        __syncthreads();
        if (!goes) return;
    }
    int workgroups = gridDim.x;
    int64_t first = ((int64_t)wave * workgroups + blockIdx.x) * 64, stride = (int64_t)64 * kStepWaves * workgroups;
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
    unsigned long long lowest = ~0ull;
    int steps_kept = 0;
    auto begin = [&]() {
        top = 0ull;
        channel = 32;
        lowest = ~0ull;
        steps_kept = 0;
        for (int e = threadIdx.x; e < 1024; e += 64 * kStepWaves) product[e] = best[e] = e / 32 == e % 32 ? 1.0 : 0.0;
#pragma unroll 1
        for (int64_t r = first + lane; r < p.T; r += stride)
#pragma unroll 1
            for (int c = 0; c < 32; ++c) {
                const double v = (double)__uint_as_float((uint32_t)p.x[r * p.ldx + 32 * block + c] << 16);
                w.z[r * 32 + c] = v;
                seen(v, c);
            }
    };
    begin();
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
            if (workgroups > 1) {                            // among all, by the rules of the search kernel's exchange
                const unsigned long long there = (unsigned long long)((t >> 1) & 1) << 63;
                unsigned long long* const set = w.colmax + (t & 1) * 2 * workgroups;
                if (lane == 0) {
                    __hip_atomic_store(set + 2 * blockIdx.x, peak | there, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(set + 2 * blockIdx.x + 1, (unsigned long long)d | there, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                const unsigned long long* const theirs = set + 2 * (lane < workgroups ? lane : workgroups - 1);
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
                d = missing || s.patience == 0 || (writes && t == s.leaves) ? -1 : smallest_channel(v, (int)dd, peak);
            }
            if (lane == 0) { peak_of_all = peak; channel_of_all = d; }
        }
        __syncthreads();
        const unsigned long long peak = peak_of_all;
        const int d = channel_of_all;
        if (d < 0) {                                         // the same for every thread of the workgroup
            if (!writes) break;
            if (threadIdx.x == 0) w.given_up[1] = 1ull;
            if (threadIdx.x > 0 && (int)threadIdx.x < workgroups && atomicCAS(state + threadIdx.x, kNotBegun, kLeft) == kBegun)
                while (__hip_atomic_load(state + threadIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != kLeft) __builtin_amdgcn_s_sleep(64);
            __syncthreads();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            workgroups = 1;
            first = wave * 64;
            stride = 64 * kStepWaves;
            begin();
            t = -1;
            continue;
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
    if (!writes) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __syncthreads();
    if (!writes) {                                           // the only way out once it has begun
        if (threadIdx.x == 0) __hip_atomic_store(state + blockIdx.x, kLeft, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
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
    const int64_t waves = (T + 63) / 64, room = 31 * ((int64_t)steps + 1) / 5;
    int64_t few = waves < kFewWorkgroups ? waves : kFewWorkgroups;
    few = few < room ? few : room;
    s = SearchPlan{0, (int)tiles, (int)all, kPatience, cus, (int)few, -1};
    return true;
}

hipError_t launch_search(const ConstructParams& p, const SearchPlan& s, int form, bool rows, uint32_t patience_again, hipStream_t stream) {
    hipError_t e = launch(construct_prepare_kernel, dim3((unsigned)(s.partials + p.steps)), dim3(256), 0, stream, p, s);
    if (e == hipSuccess && rows) e = launch(construct_rows_kernel, dim3(kRowsWorkgroups), dim3(64 * kRowsWaves), 0, stream, p, s);
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
    return launch(construct_again_kernel, dim3((unsigned)s.few), block, 0, stream, p, again);
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
    const int cus = cus_of(stream), form = construct_form(p.T, p.steps, how % DUQPP_CONSTRUCT_IMPATIENT, cus);
    runs = form >= 0;
    if (!runs) return hipSuccess;
    if (form == DUQPP_CONSTRUCT_STEPS) return launch_steps(p, partials, stream);
    SearchPlan s{};
    plan_search(p.T, p.steps, form, cus, s);
    s.partials = partials;
    if (how & DUQPP_CONSTRUCT_IMPATIENT) s.patience = 0;
    s.leaves = how / DUQPP_CONSTRUCT_LEAVES - 1;
    const bool rows = how == DUQPP_CONSTRUCT_AUTO && p.T <= kRowsScanned;
    return launch_search(p, s, form, rows, (how & DUQPP_CONSTRUCT_ALONE) == DUQPP_CONSTRUCT_ALONE ? 0 : kPatienceAgain, stream);
}

}  // namespace duqpp

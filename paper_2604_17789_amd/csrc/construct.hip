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
// One kernel launch per step: the step needs the column maxima of the whole previous state, and all CUs wait for each other at
// a launch (1.3 us of a step's 4.7).  What a step's result does not depend on is done ahead of the steps, for all
// of them at once: the matrices H . diag(1, Q'_t) by construct_matrices_kernel, one workgroup per step.  A step is bound by
// its chain of latencies (launch, column maxima, state, sums, atomics), so everything in it is spread wide: a workgroup
// takes 32 rows, each of its eight waves 4 of the 32 columns, a lane two of them for one row.  The state is kept in tiles
// of 32 rows with the rows adjacent, so that a wave reads and writes whole lines.
// The call is offline.  2048 x 4096 activations, 128 steps on one MI355X: 2310 -> 667 us against a step kernel that
// rebuilt M_t in every workgroup (a step 15.7 -> 4.7 us, of which an empty launch takes 1.3; the search for the block
// 97 -> 5.6 us with one key per workgroup instead of one atomic per wave; the last kernel 142 -> 7 us).
#include "duqpp_internal.h"

#pragma clang fp contract(off)

namespace duqpp {

namespace {

constexpr double kHadamardEntry = 0.17677669529663687;   // 1 / sqrt(32)
constexpr int kTileRows = 32;                            // rows of the state per workgroup of a step
constexpr int kStepWaves = 8;                            // waves of that workgroup; 4 columns each
constexpr int kMaxPartials = 1024;                       // workgroups of the block search (their keys fill one slot of 8 KiB)

typedef double f64x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ double hadamard_entry(int i, int k) { return (__popc(i & k) & 1) ? -kHadamardEntry : kHadamardEntry; }

// workspace: [header 64 B: u64 block key][colmax (S + 1) x 32 u64][slots (S + 1) x 1024 f64][Z T x 32 f64]
// Slot 0 holds the block search's partial keys, then the maxima below; slot t >= 1 holds M_t = H . diag(1, Q'_t), then R^(t).
struct Workspace {
    unsigned long long* key;
    unsigned long long* colmax;
    double* slots;
    double* z;
};
__host__ __device__ inline Workspace carve(void* ws, int steps) {
    Workspace w;
    uint8_t* p = static_cast<uint8_t*>(ws);
    w.key = reinterpret_cast<unsigned long long*>(p);
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

// One step of a maximum over the wave: with the value of another lane, moved by the ALU (quad permutation 0xB1 = lane ^ 1,
// 0x4E = lane ^ 2, 0x141 and 0x140 = mirrored within 8 and 16 lanes; lanes that hold the same maximum may stand in for
// each other, so the mirrors do what lane ^ 4 and lane ^ 8 would).
template <int CTRL>
__device__ __forceinline__ unsigned long long dpp_max(unsigned long long v) {
    const int lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)v, CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(v >> 32), CTRL, 0xF, 0xF, true);
    return max_u64(v, ((unsigned long long)(uint32_t)hi << 32) | (uint32_t)lo);
}
// maximum over each half of the wave, in every lane of the half
__device__ __forceinline__ unsigned long long half_max(unsigned long long v) {
    v = dpp_max<0xB1>(v);
    v = dpp_max<0x4E>(v);
    v = dpp_max<0x141>(v);
    v = dpp_max<0x140>(v);
    return max_u64(v, __shfl_xor(v, 16));
}
// maximum over the 64 lanes, in every lane
__device__ __forceinline__ unsigned long long wave_max(unsigned long long v) {
    v = half_max(v);
    return max_u64(v, __shfl_xor(v, 32));
}

// Clears the first column maxima, and the largest |x| per block of 32 channels -> one 64-bit key per workgroup: magnitude bits
// above, inverted block index below, so that the integer maximum is the largest magnitude in the smallest block.
__global__ __launch_bounds__(256) void construct_blockmax_kernel(ConstructParams p) {
    __shared__ unsigned long long red[4];
    Workspace w = carve(p.workspace, p.steps);
    const int64_t stride = (int64_t)gridDim.x * 256, at = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (at < 32) w.colmax[at] = 0ull;
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

// Z_0 = the chosen block's columns as doubles, and their column maxima.  Every workgroup finds the block again from the
// partial keys.
__global__ __launch_bounds__(64 * kStepWaves) void construct_extract_kernel(ConstructParams p, int partials) {
    __shared__ unsigned long long red[kStepWaves];
    Workspace w = carve(p.workspace, p.steps);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned long long key = 0ull;
    for (int i = threadIdx.x; i < partials; i += 64 * kStepWaves) key = max_u64(key, reinterpret_cast<const unsigned long long*>(w.slots)[i]);
    key = wave_max(key);
    if (lane == 0) red[wave] = key;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kStepWaves; ++k) key = max_u64(key, red[k]);
    if (blockIdx.x == 0 && threadIdx.x == 0) *w.key = key;
    const int64_t b = 0xFFFFFFFFu - (uint32_t)(key & 0xFFFFFFFFull);

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
__global__ __launch_bounds__(256) void construct_matrices_kernel(ConstructParams p) {
    __shared__ double q[31 * 31];
    Workspace w = carve(p.workspace, p.steps);
    const int t = blockIdx.x;
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

// The channel that step t exchanges with channel 0: largest magnitude in the state before it, smallest index among equals.
// The same in every lane of every wave (lanes 32 .. 63 repeat lanes 0 .. 31).
__device__ __forceinline__ int exchanged_channel(unsigned long long colmax_of_lane) {
    const unsigned long long best = half_max(colmax_of_lane);
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

}  // namespace

size_t construct_workspace_bytes(int64_t T, int steps) {
    return 64 + (size_t)(steps + 1) * 256 + (size_t)(steps + 1) * 8192 + (size_t)T * 256;
}

hipError_t launch_construct_rotation(const ConstructParams& p, hipStream_t stream) {
    const int64_t chunks = (int64_t)p.T * (p.K / 8);
    const int partials = (int)((chunks + 1023) / 1024 < kMaxPartials ? (chunks + 1023) / 1024 : kMaxPartials);
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

}  // namespace duqpp

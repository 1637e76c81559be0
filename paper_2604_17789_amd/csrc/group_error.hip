// Per-group normalised quantisation error -- the statistic of Fig. 1 (Sec. 4.1): for every token and every group of
// 32 channels ||Q(y) - y||_2 / ||y||_2, where y is the group after the block rotation of Eq. 4 (or the group itself:
// the figure's "Original" setting) and Q the MXFP4 quantiser of Eq. 2.  An analysis tool beside the hot path: it
// rotates and quantises with the hot path's own device functions (rotq_device.h), so the error it reports is the
// error of the codes the hot path produces.
#include "duqpp_internal.h"
#include "rotq_device.h"

namespace duqpp {

namespace {

constexpr int kErrWaves = 4;            // waves per workgroup, two groups each
// Up to this many (token tile, group) pairs a wave of its own for each: no more than a wave per SIMD, and half the arithmetic in
// the one chain that such a call is (ratios alone, one against two groups per wave: 64 x 512 2.6 / 3.2 us, 256 x 4096, 1024 pairs,
// 3.0 / 3.3, 288 x 4096 3.3 / 3.5, 511 x 4096, 2048 pairs, 3.7 / 3.6).  Four times as many without rotation, where a wave has
// nothing to keep from tile to tile, as long as the mean needs no partial sums (511 x 4096 3.5 / 3.4, 1500 x 2048, 3008 pairs, 4.1 / 5.4,
// 1024 x 4096, 4096 pairs, 4.8 / 5.5).
constexpr int64_t kOneGroupTo = 1024;
constexpr int kErrWorkgroups = 512;     // aimed at: two per CU (1024: 11.1 us at 2048 x 4096, 512: 9.3, 256: 10.0)
// From this many ratios on the mean is formed from the partial sums of the workgroups that compute them.
constexpr int64_t kPartialsFrom = 65536;

struct ErrPlan {
    int chunks, runs;                   // workgroups: column chunks x token runs
    int ntiles;                         // token tiles of 32 in play
    int64_t keep_from, keep_to;         // ratios stored: their place in err, in floats
    int partials;                       // each workgroup's partial sum and count are kept: as four words, or (kPairs) as two doubles
};
constexpr int kWords = 1, kPairs = 2;

// value of an E2M1 code (sign, two exponent bits, one mantissa bit): 0, 0.5, 1, 1.5, 2, 3, 4, 6
__device__ __forceinline__ double e2m1_value(uint32_t nib) {
    const uint32_t e = (nib >> 1) & 3u, m = nib & 1u;
    const double mag = e == 0u ? 0.5 * m : (1.0 + 0.5 * m) * (double)(1u << (e - 1u));
    return (nib & 8u) ? -mag : mag;
}

typedef float f32x2 __attribute__((ext_vector_type(2)));

// This lane's 16 of a token's 32 values: sums of (Q(y) - y)^2 and of y^2.
__device__ __forceinline__ void error_sums(const f32x16& acc, double& num, double& den) {
    uint32_t p0, p1;
    const uint32_t byte = quantize_lane(acc, p0, p1);
    num = 0.0;
    den = 0.0;
    if (__any(byte < 32u)) {
        // a group near the bottom of fp32's range: in fp64 throughout (2^(byte - 127) as a double: the fp32 form of 2^-127
        // would be subnormal)
        const double scale = __longlong_as_double((long long)(byte + 896u) << 52);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const double y = (double)acc[i];
            const double d = e2m1_value(((i < 8 ? p0 : p1) >> (4 * (i & 7))) & 15u) * scale - y;
            num += d * d;
            den += y * y;
        }
        return;
    }
    // Q(y) - y is exact in fp32: Q(y) and y are multiples of the last place of y, and their difference is no larger than y.
    const float sc = __uint_as_float(byte << 23);
    auto two = [&](float y0, float y1, const f32x2& q) {
        const double d0 = (double)(q[0] - y0), d1 = (double)(q[1] - y1);
        num += d0 * d0;
        den += (double)y0 * (double)y0;
        num += d1 * d1;
        den += (double)y1 * (double)y1;
    };
    two(acc[0], acc[1], __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(p0, sc, 0));
    two(acc[2], acc[3], __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(p0, sc, 1));
    two(acc[4], acc[5], __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(p0, sc, 2));
    two(acc[6], acc[7], __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(p0, sc, 3));
    two(acc[8], acc[9], __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(p1, sc, 0));
    two(acc[10], acc[11], __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(p1, sc, 1));
    two(acc[12], acc[13], __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(p1, sc, 2));
    two(acc[14], acc[15], __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(p1, sc, 3));
}

// v0 summed over the lane pair (c, c + 32) in the lower half of the wave, v1 in the upper half.
__device__ __forceinline__ double pair_sums(double v0, double v1) {
    const unsigned long long a = (unsigned long long)__double_as_longlong(v0), b = (unsigned long long)__double_as_longlong(v1);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)a, (uint32_t)b, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
    return __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0])) +
           __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1]));
}

// A wave takes GROUPS = 2 adjacent groups (one 128-byte line per token row) and walks its run of 32-token tiles with their
// rotation blocks in registers and the next tile's line requested ahead, or one group and one tile.  Lane (c, h) computes half
// of token c's values of each group, then of two groups the ratio of group h: one division and square root per lane.
// Bound by the fp64 sums and the start (rotation blocks, first tiles), a third of it by reading x.  2048 x 4096 on one
// MI355X: 13.2 -> 9.3 us against a wave per (tile, group) that formed the codes' values in fp64; the mean 86 -> 6.3 us (2.4 from
// the partial sums, 3.9 to compute the first ratios again) against one workgroup with one load in flight per thread, and 2.4
// where the caller has a place for the partial sums.  (Both in one launch of one workgroup: 15.3 us.)
template <bool ROTATED, int GROUPS>
__global__ __launch_bounds__(64 * (GROUPS == 2 ? kErrWaves : 1)) void group_error_kernel(GroupErrorParams p, ErrPlan e) {
    constexpr int kWaves = GROUPS == 2 ? kErrWaves : 1;
    __shared__ double sums[kWaves][2];
    const int lane = threadIdx.x & 63, c = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int chunk = blockIdx.x, run = blockIdx.y;          // (a division ahead of the first load: 2048 x 4096 7.60 -> 7.48 us without)
    const int j0 = (chunk * kWaves + wave) * GROUPS;
    double sum = 0.0, count = 0.0;
    if (j0 < p.G) {
        const int j1 = GROUPS == 2 && j0 + 1 < p.G ? j0 + 1 : j0;   // an odd last group: computed twice, stored once
        RotOperand op0, op1;
        const int step1 = 32 * (j1 - j0);
        auto load = [&](u32x4 (&v)[4], int tile) {
            const int token = tile * 32 + c;
            const uint16_t* xr = p.x + (int64_t)(token < p.rows ? token : p.rows - 1) * p.ldx + 32 * j0;   // past the end: a valid row
            if constexpr (ROTATED) {
                v[0] = *(const u32x4*)(xr + 8 * h);
                v[1] = *(const u32x4*)(xr + 8 * h + 16);
                if constexpr (GROUPS == 2) {
                    v[2] = *(const u32x4*)(xr + step1 + 8 * h);
                    v[3] = *(const u32x4*)(xr + step1 + 8 * h + 16);
                }
            } else {
                // channels 8 q + 4 h .. + 3 of each group, the layout rotate_tile would give
#pragma unroll
                for (int q = 0; q < 4; ++q) {
#pragma unroll
                    for (int k = 0; k < GROUPS; ++k) {
                        const uint2 a = *(const uint2*)(xr + k * step1 + 8 * q + 4 * h);
                        v[2 * k + q / 2][2 * (q & 1)] = a.x;
                        v[2 * k + q / 2][2 * (q & 1) + 1] = a.y;
                    }
                }
            }
        };
        auto values = [&](const u32x4* v, const RotOperand& op) {
            if constexpr (ROTATED) {
                const u32x4 xv[2] = {v[0], v[1]};
                return rotate_tile(op, xv);
            } else {
                f32x16 acc;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const uint32_t w = v[i / 4][i % 4];
                    acc[2 * i] = __uint_as_float(w << 16);
                    acc[2 * i + 1] = __uint_as_float(w & 0xFFFF0000u);
                }
                return acc;
            }
        };
        u32x4 x[4], nx[4];
        if constexpr (ROTATED) {
            load_rot_operand(p.R + (int64_t)j0 * p.r_stride, c, h, op0);
            if constexpr (GROUPS == 2) load_rot_operand(p.R + (int64_t)j1 * p.r_stride, c, h, op1);
        }
        if (run < e.ntiles) load(x, run);
        for (int tile = run; tile < e.ntiles; tile += e.runs) {
            if constexpr (GROUPS == 2) load(nx, tile + e.runs < e.ntiles ? tile + e.runs : tile);
            double n0, d0;
            error_sums(values(x, op0), n0, d0);
            double n1 = n0, d1 = d0;
            if constexpr (GROUPS == 2) error_sums(values(x + 2, op1), n1, d1);
            const double num = pair_sums(n0, n1), den = pair_sums(d0, d1);
            const int token = tile * 32 + c;
            if (token < p.rows && (GROUPS == 2 ? j0 + h < p.G : h == 0)) {
                const float r = den > 0.0 ? (float)sqrt(num / den) : -1.0f;
                const int64_t at = (int64_t)token * p.G + j0 + h;
                if (at >= e.keep_from && at < e.keep_to) p.err[at] = r;
                if (r >= 0.f) { sum += (double)r; count += 1.0; }
            }
            if constexpr (GROUPS == 2) {
#pragma unroll
                for (int k = 0; k < 4; ++k) x[k] = nx[k];
            }
        }
    }
    if (!e.partials) return;
    for (int off = 32; off > 0; off >>= 1) {
        sum += __shfl_xor(sum, off);
        count += __shfl_xor(count, off);
    }
    if (lane == 0) { sums[wave][0] = sum; sums[wave][1] = count; }
    __syncthreads();
    if (threadIdx.x < 2) {
        double t = 0.0;
        for (int k = 0; k < kWaves; ++k) t += sums[k][threadIdx.x];
        const unsigned long long bits = (unsigned long long)__double_as_longlong(t);
        if (e.partials == kPairs) {                          // may be host memory: one store each
            ((double*)p.partials)[((int64_t)run * e.chunks + chunk) * 2 + threadIdx.x] = t;
            return;
        }
        uint32_t* out = (uint32_t*)p.partials + ((int64_t)run * e.chunks + chunk) * 4 + 2 * threadIdx.x; // may be err, aligned to a float only
        out[0] = (uint32_t)bits;
        out[1] = (uint32_t)(bits >> 32);
    }
}

// Mean of the ratios over the groups that have one (err >= 0), summed in a fixed order: each thread its elements or partial
// sums in order, then a tree over the 1024 threads.
template <bool PARTIALS, int AHEAD>
__global__ __launch_bounds__(1024) void group_error_mean_kernel(GroupErrorMeanParams p) {
    __shared__ double ssum[1024];
    __shared__ double scnt[1024];
    double s = 0.0, cnt = 0.0;
    if constexpr (PARTIALS) {
        const uint32_t* w = (const uint32_t*)p.err;
        for (int64_t i = threadIdx.x; i < p.n; i += 1024) {
            const uint32_t* q = w + 4 * i;
            s += __longlong_as_double((long long)(((unsigned long long)q[1] << 32) | q[0]));
            cnt += __longlong_as_double((long long)(((unsigned long long)q[3] << 32) | q[2]));
        }
    } else {
        // AHEAD elements in flight per thread: one workgroup reads at what a CU takes in
        for (int64_t i = threadIdx.x; i < p.n; i += AHEAD * 1024) {
            float e[AHEAD];
#pragma unroll
            for (int k = 0; k < AHEAD; ++k) {                // no branch around a load: they would be waited for one by one
                const int64_t at = i + k * 1024;
                const float v = p.err[at < p.n ? at : p.n - 1];
                e[k] = at < p.n ? v : -1.f;
            }
#pragma unroll
            for (int k = 0; k < AHEAD; ++k)
                if (e[k] >= 0.f) { s += (double)e[k]; cnt += 1.0; }
        }
    }
    ssum[threadIdx.x] = s;
    scnt[threadIdx.x] = cnt;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            ssum[threadIdx.x] += ssum[threadIdx.x + w];
            scnt[threadIdx.x] += scnt[threadIdx.x + w];
        }
        __syncthreads();
    }
    // the caller may have it in pinned host memory: stored once, read nowhere
    if (threadIdx.x == 0) *p.mean = scnt[0] > 0.0 ? ssum[0] / scnt[0] : 0.0;
}

}  // namespace

// column chunks x token runs
static int64_t error_workgroups(int64_t tiles, int64_t G, int64_t& chunks, int64_t& runs) {
    chunks = (G + 2 * kErrWaves - 1) / (2 * kErrWaves);
    runs = kErrWorkgroups / chunks;
    runs = runs < 1 ? 1 : (runs > tiles ? tiles : runs);
    return chunks * runs;
}

// of the partial sums of a call with a mean; 0: it takes none
size_t group_error_workspace_bytes(int64_t rows, int64_t G) {
    int64_t chunks, runs;
    return rows * G < kPartialsFrom ? 0 : (size_t)error_workgroups((rows + 31) / 32, G, chunks, runs) * 16;
}

static bool one_group_each(int64_t tiles, int64_t G) { return tiles * G <= kOneGroupTo; }

size_t group_error_partials_bytes(int64_t rows, int64_t G) {
    int64_t chunks, runs;
    const int64_t tiles = (rows + 31) / 32;
    return (size_t)(one_group_each(tiles, G) ? tiles * G : error_workgroups(tiles, G, chunks, runs)) * 16;
}

double group_error_mean(const double* partials, size_t bytes) {
    const int64_t n = (int64_t)(bytes / 16);
    double sum[1024] = {}, count[1024] = {};                 // in the order of group_error_mean_kernel
    for (int64_t i = 0; i < n; ++i) {
        sum[i & 1023] += partials[2 * i];
        count[i & 1023] += partials[2 * i + 1];
    }
    for (int w = 512; w > 0; w >>= 1)
        for (int i = 0; i < w; ++i) {
            sum[i] += sum[i + w];
            count[i] += count[i + w];
        }
    return count[0] > 0.0 ? sum[0] / count[0] : 0.0;
}

hipError_t launch_group_error(const GroupErrorParams& call, bool mean_by_caller, hipStream_t stream) {
    GroupErrorParams p = call;
    const int64_t tiles = ((int64_t)p.rows + 31) / 32;
    if (p.G < 1 || p.rows < 1 || tiles > kGroupErrorMaxTiles) return hipErrorInvalidValue;
    const int64_t n = (int64_t)p.rows * p.G;
    auto plan = [&](int ntiles) {
        ErrPlan e{};
        int64_t chunks, runs;
        error_workgroups(ntiles, p.G, chunks, runs);
        e.chunks = (int)chunks;
        e.runs = (int)runs;
        e.ntiles = ntiles;
        e.keep_to = n;
        return e;
    };
    auto run = [&](const ErrPlan& e) {
        const dim3 grid((unsigned)e.chunks, (unsigned)e.runs), block(64 * kErrWaves);
        return p.R ? launch(group_error_kernel<true, 2>, grid, block, 0, stream, p, e)
                   : launch(group_error_kernel<false, 2>, grid, block, 0, stream, p, e);
    };
    auto run_one_group = [&](const ErrPlan& e) {
        const dim3 grid((unsigned)e.chunks, (unsigned)e.runs), block(64);
        return p.R ? launch(group_error_kernel<true, 1>, grid, block, 0, stream, p, e)
                   : launch(group_error_kernel<false, 1>, grid, block, 0, stream, p, e);
    };
    auto mean_of_ratios = [&] {
        const GroupErrorMeanParams m{p.err, n, p.mean};
        // few ratios: seven loads too many cost more than a second round trip (2048 ratios, the whole call 6.9 and 6.5 us)
        return n <= 2048 ? launch(group_error_mean_kernel<false, 1>, dim3(1), dim3(1024), 0, stream, m)
                         : launch(group_error_mean_kernel<false, 8>, dim3(1), dim3(1024), 0, stream, m);
    };
    if (mean_by_caller) {                                    // a launch less; the sums of 512 workgroups take the host a microsecond
        ErrPlan e = plan((int)tiles);
        e.partials = kPairs;
        if (!one_group_each(tiles, p.G)) return run(e);
        e.chunks = p.G;
        e.runs = (int)tiles;
        return run_one_group(e);
    }
    if (tiles * p.G <= (p.R ? kOneGroupTo : 4 * kOneGroupTo) && (!p.mean || n < kPartialsFrom)) {
        ErrPlan one = plan((int)tiles);
        one.chunks = p.G;
        one.runs = (int)tiles;
        const hipError_t st = run_one_group(one);
        return st != hipSuccess || !p.mean ? st : mean_of_ratios();
    }
    ErrPlan e = plan((int)tiles);
    const int64_t workgroups = (int64_t)e.chunks * e.runs, held = 4 * workgroups;   // floats the partial sums take
    if (!p.mean || n < kPartialsFrom || held > n) {
        const hipError_t st = run(e);
        return st != hipSuccess || !p.mean ? st : mean_of_ratios();
    }
    // The partial sums need a place until the mean is formed.  Where the call brings none they take the first floats of err,
    // whose ratios (at most 64 token tiles, with one group per token) are computed once more afterwards.
    const bool scratch = p.partials != nullptr;
    if (!scratch) p.partials = p.err;
    e.partials = kWords;
    e.keep_from = scratch ? 0 : held;
    hipError_t st = run(e);
    if (st != hipSuccess) return st;
    st = launch(group_error_mean_kernel<true, 1>, dim3(1), dim3(1024), 0, stream, GroupErrorMeanParams{p.partials, workgroups, p.mean});
    if (st != hipSuccess || scratch) return st;
    ErrPlan again = plan((int)(((held + p.G - 1) / p.G + 31) / 32));
    again.keep_to = held;
    return run(again);
}

}  // namespace duqpp

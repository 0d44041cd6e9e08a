// Statistics of the softmax inputs (Section 3, the distribution of x_i from which the
// unified scaling factor and its bounds are chosen): a fixed-width histogram of every
// valid scaled logit x = s <q, k_j>, plus their minimum and maximum.  Reads K (256 B
// per key and KV head, once per block of query heads that share it), nothing else of size.
//
// A wavefront's unit of work is a run of keys of one KV head; one workgroup of 16 wavefronts (4 where there are few
// runs) per compute unit strides over the runs.  Query heads that share a KV head go through the matrix cores, 16 heads at a time, so that every key
// is read once per 16 of them; ungrouped heads take the vector ALU with the lane layout and the dot product of
// the chunk kernels (fd_chunk.h).  Counts go to an
// LDS histogram first and reach the device histogram as 64-bit integer atomic adds
// when the workgroup is done: integer sums, so the result does not depend on order.
#include "fd_chunk.h"

namespace fd {
namespace {

constexpr int kStatsWaves = 16, kStatsFew = 4;    // wavefronts per workgroup: many runs, few runs

// float minimum / maximum through integer atomics (the IEEE order of same-sign floats is
// the order of their bit patterns, reversed for negatives).  NaN never reaches here.
__device__ __forceinline__ void atomic_max_float(float *addr, float v)
{
    if (v >= 0.f) atomicMax(reinterpret_cast<int *>(addr), __builtin_bit_cast(int, v));
    else atomicMin(reinterpret_cast<unsigned *>(addr), __builtin_bit_cast(unsigned, v));
}
__device__ __forceinline__ void atomic_min_float(float *addr, float v)
{
    if (v >= 0.f) atomicMin(reinterpret_cast<int *>(addr), __builtin_bit_cast(int, v));
    else atomicMax(reinterpret_cast<unsigned *>(addr), __builtin_bit_cast(unsigned, v));
}

// The slot of a logit in the histogram, NaN with the logits above the window.
__device__ __forceinline__ int slot_of(float x, float x_min, float inv_width, int n_bins)
{
    if (x != x) return n_bins + 1;
    const float t = floorf((x - x_min) * inv_width);
    return t < 0.f ? 0 : (t >= (float)n_bins ? n_bins + 1 : (int)t + 1);
}

// GROUPED: score tile, K staging in LDS and lane layout of the grouped decode kernel (16 keys x 16 heads by four
// 16x16x32 MFMAs; lane (n, g) ends up with the logits of head n, keys 4r + g).
// Bound: HBM reads of K, and at the end the adds of all workgroups to the same n_bins + 2 addresses, which serialize
// (with 1024 smaller workgroups for grouped heads, four dot products per key on the vector ALU and K fetched once per four
// heads, the 203 MB of 32 ragged sequences x 64/8 heads x 4096 keys took 89.2 us, now 43.3 with the calls around it; with 512 for
// ungrouped heads, 1 x 32 heads x 8192 keys 22.9, now 17.3).
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
template <bool GROUPED, bool LIVE>
__global__ __launch_bounds__(kStatsWaves * 64) void logit_histogram_kernel(
    const Problem p, const float x_min, const float inv_width, const int n_bins, const int run,
    unsigned long long *__restrict__ hist, float *__restrict__ min_max)
{
    // (GROUPED: 4 KiB of K staging per wavefront), counters, 2 floats per wavefront
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    const int waves = blockDim.x >> 6;
    unsigned *lds_hist = reinterpret_cast<unsigned *>(lds_raw + (GROUPED ? waves * 4096 : 0));
    float *lds_mm = reinterpret_cast<float *>(lds_hist + n_bins + 2);
    const int tid = threadIdx.x, lane = tid & 63, wave = LIVE ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid >> 6;
    const int n = lane & 15, g = lane >> 4;
    u32x4 *kst = reinterpret_cast<u32x4 *>(lds_raw) + wave * 256;
    for (int i = tid; i < n_bins + 2; i += blockDim.x) lds_hist[i] = 0u;
    __syncthreads();

    const int runs = (p.Smax + run - 1) / run;
    const int hblocks = (p.G + 15) / 16;
    unsigned items = (unsigned)(p.B * p.Hkv * hblocks) * (unsigned)runs;         // < 2^31: at most rows * ceil(Smax / 64)
    const unsigned stride = (unsigned)waves * gridDim.x;
    float lo = INFINITY, hi = -INFINITY;
    // Consecutive items to consecutive workgroups: the runs of a KV head spread over the chip.  Where they are many (runs of more than 64
    // keys: two per wavefront or more) ragged lengths would load the compute units unevenly, all runs of a workgroup lying at the same place of
    // their sequences where the number of runs divides that of the workgroups.  LIVE (the lengths of the batch fit a wavefront): the items are the runs
    // that hold keys; every wavefront has all lengths, one a lane, and finds its runs by their prefix sums, (sequence, KV head) after (sequence, KV head).
    // Otherwise each (sequence, KV head) starts at a place of its own, the next for every round of the workgroups: `turned`.  Whole call, one after
    // the other / turned / LIVE: 32 x 64/8 heads x 2048 .. 4096 keys 47.5 / 45.0 / 43.3 us; turned / LIVE 5 x 64/8 x 5000 .. 40000 52.0 / 48.1, 24 x 32/8 x 700 ..
    // 5600 40.2 / 37.7, full lengths 32 x 64/8 x 4096 51.1 / 51.0.  With hardly a run per wavefront there is little to even out, and it helps that the
    // workgroups at the sequences' ends have nothing to add to memory: one after the other / turned 32 x 64/8 x 100 .. 1000 12.7 / 14.2, 32 x 64/8 x 200 .. 1500
    // 17.1 / 18.0, 6 x 40 x 200 .. 1500 17.0 / 17.8, 16 x 16 x 1500 20.7 / 21.1; one after the other / LIVE 32 x 64/8 x 100 .. 1000 19.7 / 22.9, 12 x 32/8 x 670 .. 5367 26.4 / 27.6.
    const bool turned = run > 64;
    int len = 0, own = 0, upto = 0;                      // lane b: keys of sequence b, its runs, those of the sequences up to it for all KV heads
    if constexpr (LIVE) {
        if (lane < p.B) len = valid_len(p, lane);
        own = (len + run - 1) / run;
        upto = lanes_scan(own * p.Hkv * hblocks);
        items = (unsigned)__builtin_amdgcn_readlane(upto, 63);
    }
    for (unsigned it = (unsigned)wave * gridDim.x + blockIdx.x; it < items; it += stride) {
        int b, t, hb, hkv, gi, nvalid;                   // gi: (sequence, KV head)
        if constexpr (LIVE) {
            b = __popcll(__ballot(upto <= (int)it));
            const unsigned of_b = (unsigned)__builtin_amdgcn_readlane(own, b);
            const unsigned at = it - (unsigned)__builtin_amdgcn_readlane(upto, b) + of_b * (unsigned)(p.Hkv * hblocks);
            const unsigned r = at / of_b;
            t = (int)(at - r * of_b);
            hkv = (int)(r / (unsigned)hblocks);
            hb = (int)r - hkv * hblocks;
            gi = b * p.Hkv + hkv;
            nvalid = min(run, __builtin_amdgcn_readlane(len, b) - t * run);
        } else {
            const unsigned r = it / (unsigned)runs;
            t = (int)((turned ? it + r * (unsigned)runs / gridDim.x : it) % (unsigned)runs);
            hb = (int)(r % (unsigned)hblocks);
            gi = (int)(r / (unsigned)hblocks);
            b = gi / p.Hkv;
            hkv = gi - b * p.Hkv;
            nvalid = min(run, valid_len(p, b) - t * run);
            if (nvalid <= 0) continue;
        }
        const int last = nvalid - 1;
        const int nh = min(16, p.G - 16 * hb);           // heads of this block
        const int row0 = b * p.Hq + hkv * p.G + 16 * hb;
        // GROUPED: Q as the B operand, heads past the last are zero rows; else this lane's 16-byte segment of q
        u32x4 qv[GROUPED ? 4 : 1];
        if constexpr (GROUPED) {
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) {
                qv[kb] = u32x4{0u, 0u, 0u, 0u};
                if (n < nh) qv[kb] = *reinterpret_cast<const u32x4 *>(p.q + (size_t)(row0 + n) * kHeadDim + 32 * kb + 8 * g);
            }
        } else {
            qv[0] = reinterpret_cast<const u32x4 *>(p.q + (size_t)row0 * kHeadDim)[n];
        }
        const u32x4 *kp = reinterpret_cast<const u32x4 *>(p.k + ((size_t)gi * p.Smax + (size_t)t * run) * kHeadDim) + n;
        auto issue = [&](int blk, u32x4 (&kk)[4]) {
#pragma unroll
            for (int i = 0; i < 4; ++i) kk[i] = load_stream(kp + (size_t)min(16 * blk + 4 * i + g, last) * 16);
        };
        auto add = [&](float x) {
            lo = fminf(lo, x);                           // (the minimum with a NaN is the other operand)
            hi = fmaxf(hi, x);
            atomicAdd(&lds_hist[slot_of(x, x_min, inv_width, n_bins)], 1u);
        };
        auto count = [&](int blk, const u32x4 (&kk)[4]) {
            if constexpr (GROUPED) {
#pragma unroll
                for (int i = 0; i < 4; ++i) kst[(4 * i + g) * 16 + (n ^ (i | (g << 2)))] = kk[i];
                const int pk = 4 * (n & 3) + (n >> 2);
                f32x4 sc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kb = 0; kb < 4; ++kb)
                    sc = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, kst[pk * 16 + ((4 * kb + g) ^ n)]),
                                                                __builtin_bit_cast(f16x8, qv[kb]), sc, 0, 0, 0);
                if (n < nh) {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (16 * blk + 4 * i + g <= last) add(sc[i] * p.scale);
                }
            } else {
                // every lane of a key's 16 ends up with its logit; lane i of them bins key 4i + g
                float x = 0.f;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float xi = row16_sum(dot8(qv[0], kk[i])) * p.scale;
                    x = n == i ? xi : x;
                }
                if (n < 4 && 16 * blk + 4 * n + g <= last) add(x);
            }
        };
        // two blocks in flight; loads past the last valid key re-read it and are not counted
        const int nblk = (nvalid + 15) / 16;
        u32x4 kA[4], kB[4];
        issue(0, kA);
        int blk = 0;
#pragma unroll 1
        for (; blk + 2 < nblk; blk += 2) {
            issue(blk + 1, kB);
            count(blk, kA);
            issue(blk + 2, kA);
            count(blk + 1, kB);
        }
        if (blk + 2 == nblk) {
            issue(blk + 1, kB);
            count(blk, kA);
            count(blk + 1, kB);
        } else {
            count(blk, kA);
        }
    }
    // the workgroup's counts and extremes to memory
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        lo = fminf(lo, __shfl_xor(lo, o));
        hi = fmaxf(hi, __shfl_xor(hi, o));
    }
    if (lane == 0) { lds_mm[2 * wave] = lo; lds_mm[2 * wave + 1] = hi; }
    __syncthreads();
    for (int i = tid; i < n_bins + 2; i += blockDim.x) {
        const unsigned c = lds_hist[i];
        if (c) atomicAdd(&hist[i], (unsigned long long)c);
    }
    if (tid == 0 && min_max) {
        for (int w = 0; w < waves; ++w) { lo = fminf(lo, lds_mm[2 * w]); hi = fmaxf(hi, lds_mm[2 * w + 1]); }
        if (lo <= hi) {                                  // at least one logit that is not NaN was seen
            atomic_min_float(&min_max[0], lo);
            atomic_max_float(&min_max[1], hi);
        }
    }
}

}  // namespace

hipError_t launch_logit_histogram(const Problem &p, float x_min, float bin_width, int n_bins,
                                  unsigned long long *hist, float *min_max, hipStream_t s)
{
    if (p.rows == 0) return hipSuccess;
    // Runs of 64 .. 256 keys: the longest that give every wavefront two.
    const long long units = (long long)p.B * p.Hkv * ((p.G + 15) / 16);
    int run = 256;
    while (run > 64 && units * ((p.Smax + run - 1) / run) < 2ll * kStatsWaves * kComputeUnits) run /= 2;
    const long long items = units * ((p.Smax + run - 1) / run);
    // Up to four runs per compute unit: small workgroups, and no more of them than have work (512 runs, 1 x 32 heads x 1024
    // keys: 10.3 us on 256 workgroups of 16 wavefronts, 7.5 on 128 of 4; 1304 runs, 1 x 28/4 x 20816: 12.4 / 14.7).
    const int waves = items <= (long long)kStatsFew * kComputeUnits ? kStatsFew : kStatsWaves;
    const long long wanted = (items + waves - 1) / waves;
    const unsigned grid = (unsigned)(wanted < kComputeUnits ? wanted : kComputeUnits);
    const float inv_width = 1.0f / bin_width;
    const size_t lds = (p.G > 1 ? waves * 4096 : 0) + (size_t)(n_bins + 2) * sizeof(unsigned) + waves * 2 * sizeof(float);
    void *args[] = {(void *)&p, (void *)&x_min, (void *)&inv_width, (void *)&n_bins, (void *)&run, (void *)&hist, (void *)&min_max};
    const bool live = run > 64 && p.B <= 64;
    const void *fn = p.G > 1 ? (live ? reinterpret_cast<const void *>(&logit_histogram_kernel<true, true>)
                                     : reinterpret_cast<const void *>(&logit_histogram_kernel<true, false>))
                             : (live ? reinterpret_cast<const void *>(&logit_histogram_kernel<false, true>)
                                     : reinterpret_cast<const void *>(&logit_histogram_kernel<false, false>));
    return hipLaunchKernel(fn, dim3(grid), dim3(waves * 64), args, lds, s);
}

}  // namespace fd

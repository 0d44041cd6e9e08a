// Small kernels: the flag reduction of fd_list_flagged_rows, the synchronized merge of
// Eq. 2 (fd_decode_attn_sync; third launch of the literal chain), the row epilogue as a
// launch of its own, and the counter clear of fd_workspace_init.
#include "fd_chunk.h"

namespace fd {
namespace {

__global__ __launch_bounds__(256) void clear_tickets_kernel(int32_t *ticket, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) ticket[i] = 0;
}

// The row epilogue as a launch of its own (one workgroup per row), used when the
// chunk kernels run without electing a finisher.
__global__ __launch_bounds__(256) void row_epilogue_kernel(const Problem p)
{
    __shared__ __attribute__((aligned(16))) float scratch[8 * kHeadDim + 16];
    const int row = blockIdx.x;
    // one batch of argument loads at the top instead of one per first use
    asm volatile("" ::"s"(p.ws.num), "s"(p.ws.meta), "s"(p.ws.row_flags), "s"(p.seq_lens), "s"(p.out), "s"(p.nc),
                 "s"(p.Hq), "s"(p.C), "s"(p.Smax));
    // every slot of the row holds defined values, so the loads need not wait for the length
    row_epilogue(p, row, p.nc, [&] { return (valid_len(p, row / p.Hq) + p.C - 1) / p.C; }, scratch);
}

// The same for rows of at most 32 chunks: a workgroup of one wavefront per row, no LDS, no barrier; with FLAGS = false also the
// merge of the synchronized scheme (Eq. 2).  Whole call, 32 threads per row and eight or two rows to a workgroup / this: 12 x 32/8 heads x
// 300 .. 6000 keys in 5 chunks 38.8 / 38.4 us, 16 x 64/8 x 4096 in 4 46.1 / 45.7, 1 x 64/8 x 32768 in 32 (eight slices through LDS)
// 26.8 / 25.9; fd_decode_attn_sync 1 x 32 x 1024 in 8 8.76 / 8.60, 4 x 32 x 4096 in 4 43.7 / 43.4.  Four rows to a workgroup draw
// their sums through one compute unit: 0.2 us more at 8 chunks per row, 1 us at 64.  At 64 chunks per row the forms with more
// threads per row win (27.5 / 27.75) or tie.
template <bool FLAGS>
__global__ __launch_bounds__(64) void finish_rows_kernel(const Problem p)
{
    const int row = blockIdx.x;
    asm volatile("" ::"s"(p.ws.num), "s"(p.ws.meta), "s"(p.ws.row_flags), "s"(p.seq_lens), "s"(p.out), "s"(p.nc),
                 "s"(p.Hq), "s"(p.C), "s"(p.Smax));
    // every slot of a row holds defined values, so the loads need not wait for the length
    finish_row<false, FLAGS>(p, row, p.nc, [&] { return (valid_len(p, row / p.Hq) + p.C - 1) / p.C; });
}

// Chunk flags -> row flags, ascending list of flagged rows, their count.
// A single workgroup: the compaction is a block-wide prefix sum, no atomics.
__global__ __launch_bounds__(1024) void flag_reduce_kernel(const Problem p)
{
    __shared__ int wave_cnt[16];
    __shared__ int base_s;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid == 0) base_s = 0;
    __syncthreads();
    for (int r0 = 0; r0 < p.rows; r0 += 1024) {
        const int row = r0 + tid;
        int f = 0;
        if (row < p.rows) {
            const int S = valid_len(p, row / p.Hq);
            const int nb = (S + p.C - 1) / p.C;
            const uint8_t *cf = p.ws.chunk_flags + (size_t)row * p.nc;
            for (int c = 0; c < nb; ++c) f |= cf[c];
            f = f ? 1 : 0;
            p.ws.row_flags[row] = (uint8_t)f;
        }
        const unsigned long long mask = __ballot(f);
        const int before = __popcll(mask & ((1ull << lane) - 1ull));
        if (lane == 0) wave_cnt[wave] = __popcll(mask);
        __syncthreads();
        int off = base_s, total = 0;
        for (int w = 0; w < 16; ++w) {
            if (w < wave) off += wave_cnt[w];
            total += wave_cnt[w];
        }
        if (f) p.ws.list[off + before] = row;
        __syncthreads();
        if (tid == 0) base_s += total;
        __syncthreads();
    }
    if (tid == 0) *p.ws.count = base_s;
}

// The merge of the synchronized scheme (Eq. 2) over rows of more than 32 chunks: two rows per workgroup, 32 threads each that own four
// elements; 16 chunks to a memory round trip, lane j of the row's two groups of 16 holding the record of chunk c0 + j, no further than the
// row's last chunk (1 x 32 rows of 2000 keys in a cache of 512 chunks 26.2 us, 45.1 if every chunk is walked).  Every slot holds defined
// values, so the first loads need not wait for the length.
__global__ __launch_bounds__(64) void combine_sync_kernel(const Problem p)
{
    const int t4 = threadIdx.x & 31;
    const int row = blockIdx.x * 2 + (threadIdx.x >> 5);
    if (row >= p.rows) return;
    const size_t r0 = (size_t)row * p.nc;
    const u32x4 *num = reinterpret_cast<const u32x4 *>(p.ws.num + r0 * kHeadDim) + t4;
    const u32x4 *meta = reinterpret_cast<const u32x4 *>(p.ws.meta + r0);
    float m = -INFINITY, l = 0.f;
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    int nb = 0;
    for (int c0 = 0; c0 == 0 || c0 < nb; c0 += 16) {
        const u32x4 mv = meta[min(c0 + (t4 & 15), p.nc - 1)];
        u32x4 nv[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) nv[i] = num[(size_t)min(c0 + i, p.nc - 1) * (kHeadDim / 4)];
        if (c0 == 0) nb = (valid_len(p, row / p.Hq) + p.C - 1) / p.C;        // a load of its own, in flight with the others
        const bool in_row = (t4 & 15) < min(16, nb - c0);
        const float ref = in_row ? as_f32(mv[1]) : -INFINITY;
        const float bm = row16_max(ref);
        if (bm > m) {                                        // rescale what was summed so far
            const float a = __builtin_amdgcn_exp2f((m - bm) * kLog2e);       // 0 on the first block
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] *= a;
            l *= a;
            m = bm;
        }
        // exactly 1 when ref == m; 0 for slots outside the row (their sums are finite)
        const float a = ref == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((ref - m) * kLog2e);
        const float ad = a * (in_row ? as_f32(mv[0]) : 0.f);
        each16(std::make_integer_sequence<int, 16>{}, [&](auto lane_of) {
            constexpr int i = decltype(lane_of)::value;
            const float ac = row16_lane<i>(a);
            l += row16_lane<i>(ad);
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] = __builtin_fmaf(ac, as_f32(nv[i][e]), s[e]);
        });
    }
    uint2 o = make_uint2(0u, 0u);                            // an empty sequence: zeros
    if (nb > 0) {
        o.x = (unsigned)to_half_bits(s[0] / l) | ((unsigned)to_half_bits(s[1] / l) << 16);
        o.y = (unsigned)to_half_bits(s[2] / l) | ((unsigned)to_half_bits(s[3] / l) << 16);
    }
    *reinterpret_cast<uint2 *>(p.out + (size_t)row * kHeadDim + 4 * t4) = o;
}

// Third launch of the literal chain.  Blocks 0 .. gridDim.x - 2 stride over the rows and finish the
// flagged ones: Eq. 2 over the row's recomputed partial vectors, m = max_c m_c, result =
// sum_c e^{m_c - m} (f.V)_c / sum_c e^{m_c - m} l_c.  The last block turns the row flags into the
// ascending list of flagged rows and their count (prefix sums over ballots, no atomics).
__global__ __launch_bounds__(kHeadDim) void chain_finish_kernel(const Problem p)
{
    const int t = threadIdx.x;
    const int workers = (int)gridDim.x - 1;
    if ((int)blockIdx.x == workers) {
        __shared__ int cnt[2];
        const int lane = t & 63, wave = t >> 6;
        int base = 0;
        for (int r0 = 0; r0 < p.rows; r0 += kHeadDim) {
            const int row = r0 + t;
            const int f = row < p.rows ? (int)p.ws.row_flags[row] : 0;
            const unsigned long long mask = __ballot(f);
            if (lane == 0) cnt[wave] = __popcll(mask);
            __syncthreads();
            const int before = (wave ? cnt[0] : 0) + __popcll(mask & ((1ull << lane) - 1ull));
            if (f) p.ws.list[base + before] = row;
            base += cnt[0] + cnt[1];
            __syncthreads();
        }
        if (t == 0) *p.ws.count = base;
        return;
    }
    for (int row = blockIdx.x; row < p.rows; row += workers) {
        if (!p.ws.row_flags[row]) continue;
        const int S = valid_len(p, row / p.Hq);
        const int nb = (S + p.C - 1) / p.C;
        const float *num = p.ws.num + (size_t)row * p.nc * kHeadDim + t;
        const float *den = p.ws.den + (size_t)row * p.nc;
        const float *mloc = p.ws.mloc + (size_t)row * p.nc;
        float m = -INFINITY;
        for (int c = 0; c < nb; ++c) m = fmaxf(m, mloc[c]);
        float s = 0.f, l = 0.f;
#pragma unroll 4
        for (int c = 0; c < nb; ++c) {
            const float a = __builtin_amdgcn_exp2f((mloc[c] - m) * kLog2e);
            s = __builtin_fmaf(a, num[(size_t)c * kHeadDim], s);
            l = __builtin_fmaf(a, den[c], l);
        }
        p.out[(size_t)row * kHeadDim + t] = nb > 0 ? to_half_bits(s / l) : (uint16_t)0;
    }
}

}  // namespace

hipError_t launch_clear_tickets(int32_t *ticket, size_t n, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    const size_t blocks = (n + 255) / 256;
    return launch(clear_tickets_kernel, dim3((unsigned)(blocks < 4096 ? blocks : 4096)), dim3(256), s, ticket, n);
}

hipError_t launch_row_epilogue(const Problem &p, hipStream_t s)
{
    if (p.rows == 0) return hipSuccess;
    if (p.nc <= 32) return launch(finish_rows_kernel<true>, dim3(p.rows), dim3(64), s, p);
    return launch(row_epilogue_kernel, dim3(p.rows), dim3(256), s, p);
}

hipError_t launch_flag_reduce(const Problem &p, hipStream_t s)
{
    return launch(flag_reduce_kernel, dim3(1), dim3(1024), s, p);
}

hipError_t launch_chain_finish(const Problem &p, hipStream_t s)
{
    if (p.rows == 0) return hipSuccess;
    return launch(chain_finish_kernel, dim3((p.rows < 1024 ? p.rows : 1024) + 1), dim3(kHeadDim), s, p);
}

hipError_t launch_combine_sync(const Problem &p, hipStream_t s)
{
    if (p.rows == 0) return hipSuccess;
    if (p.nc <= 32) return launch(finish_rows_kernel<false>, dim3(p.rows), dim3(64), s, p);
    return launch(combine_sync_kernel, dim3((p.rows + 1) / 2), dim3(64), s, p);
}

}  // namespace fd

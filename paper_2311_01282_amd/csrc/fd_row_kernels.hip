// Chunk kernels that treat every query head as an independent row (VALU path).
// One workgroup of NW wavefronts handles one (row, chunk); see fd_chunk.h for the
// lane layout.
//
//   decode_fused_kernel    : the whole method in one launch.  Every workgroup
//       computes its chunk's Eq. 4 inner sums under the range guard; a chunk whose
//       guard fires goes on with references of its own, or is redone (Eq. 2); the
//       workgroup that finishes a row last (elected by a small tree of arrival
//       counters) runs the row epilogue.
//   partial_unified_kernel : Eq. 4 inner sums + guard, which only flags (first launch of the chain).
//   chain_combine_kernel   : row flags; Eq. 4 outer sums for clean rows, per-chunk
//       synchronized recomputation for flagged rows (second launch of the chain).
//   partial_sync_kernel    : every (row, chunk) by Eq. 2, in two passes, where that is
//       better than the SYNC form of decode_fused_kernel (SyncLauncher).
#include "fd_chunk.h"

namespace fd {
namespace {

// Wavefronts per workgroup and pipeline depth per chunk size, from a sweep on
// MI355X at the 8K-context shape: 8 wavefronts pay off once a chunk holds at
// least 512 keys; 4 groups (4 KiB of K and of V per wavefront) per pipeline stage.
template <int C> struct Tune {
    static constexpr int NW = C >= 512 ? 8 : 4;
    static constexpr int NG = C / (4 * NW);
    static constexpr int UP = NG < 4 ? NG : 4;
};

// Launches that hand nothing over: whether the workgroups simply take one chunk after the other, row by row, instead of the same chunk
// of eight rows on the eight XCDs (row_slot), then the next.  Where the rows do not divide among the XCDs that order leaves some of them
// idle; and where the chunks of a row do not divide by 4, one after the other they go round all XCDs, too, and a compute unit's
// neighbours stream neighbouring chunks: whole call, by eight rows / this, 3 x 32 x 4000 .. 30000 keys in 30 chunks 213 / 200 us, 30 x 16 x 1718 .. 3436 in 14
// 110.6 / 107.5, 12 x 40 x 187 .. 1500 in 6 41.6 / 41.0, 4 x 16 x 30000 in 30 156.7 / 155.8, 2 x 40 x 12564 .. 25128 in 25 a tie.  Where they do divide by 4, an XCD gets the
// same few chunks of every row, which in a ragged batch are the full or the empty ones (16 x 32 x 512 .. 4096 in 8 110 / 136, 24 x 16 x 500 .. 4000
// in 16 84.7 / 93.4, 23 x 16 x 379 .. 3037 in 12 59.0 / 61.8); rows of more than 32 chunks are turned (2 x 16 x 6740 .. 53923 in 53 130.2 / 133.6).
// Two chunks, and six, leave an XCD one of the two, or every other of the six, which is no better in a ragged batch (110 x 16 x 465 .. 930 in 2 101.5 /
// 110.7, 25 x 32 x 209 .. 1678 in 2 72.2 / 77.2, 25 x 16 x 759 .. 6073 in 6 109.5 / 113.4, 20 x 16 x 800 .. 2900 in 6 55.6 / 56.7; equal lengths would gain 2 %: 110 x
// 16 x 1941 in 2 259 / 254); from ten on there are enough of them (2 x 40 x 3306 .. 13224 in 26 84.7 / 82.7).  The synchronized scheme keeps the
// order there: 10 x 40 x 1339 .. 5356 in 6 127.8 / 122.9, 3 x 32 x 1525 .. 6103 in 6 44.4 / 36.2, 29 x 16 x 1700 in 2 66.6 / 65.0 (but 38 x 32 x 224 .. 1799 in 2 117.4 / 124.8).
template <bool SYNC> __device__ __forceinline__ bool plain_order(const Problem &p)
{
    return (p.rows & 7) != 0 || ((p.nc & 3) != 0 && p.nc <= 32 && (SYNC || (p.nc & 1) != 0 || p.nc > 8));
}

// The synchronized scheme's order where heads share KV heads: the heads of a group take a chunk one after the other on the same XCD, so that its L2
// fetches the keys once, whatever the number of chunks.  Whole call, one chunk after the other / this: 2 x 32/4 x 1536 keys in 512 14.1 / 9.8 us, 1 x 28/4 x 1573 in 64 10.1 / 8.5, 1 x
// 16/2 x 5580 in 512 14.3 / 10.1; of more heads than the tile takes 2 x 32/1 x 2000 .. 5000 in 512 21.2 / 15.9, 4 x 64/2 x 3000 .. 9000 in 1024 110.5 / 60.8 (bound by the L2s then).
// False: a workgroup that only fills up the last eight.
__device__ __forceinline__ bool shared_order(const Problem &p, int &row, int &c)
{
    const int j = (int)blockIdx.x >> 3, item = j / p.G * 8 + ((int)blockIdx.x & 7);      // (sequence, KV head, chunk)
    const int group = item / p.nc;
    c = item - group * p.nc;
    row = group * p.G + j % p.G;
    return group < p.B * p.Hkv;
}
inline unsigned shared_grid(const Problem &p) { return (unsigned)(((long long)p.B * p.Hkv * p.nc + 7) / 8 * 8 * p.G); }

// ELECT: rows are finished in the launch (elect_per_row in fd_api.hip says which launches do).
// PAGED: K and V are page pools addressed through the sequence's block table.
// EARLY: the first loads go out before the sequence length has arrived -- for launches of at
//        most one workgroup per compute unit, where every workgroup starts with the launch and
//        the length load is on its critical path.  In a larger launch the later workgroups
//        start behind somebody else's stream anyway, and where the launch covers more than the
//        sequences hold (max_seq beyond the lengths) many of them are chunks without keys,
//        which then leave without reading any.
// ONE: one block of keys in flight per wavefront, not two (LoadAhead).
// SYNC: the synchronized partial softmax of every (row, chunk) instead (fd_decode_attn_sync); no election.
template <int C, bool ELECT, bool PAGED = false, bool EARLY = false, bool ONE = false, bool SYNC = false>
__global__ __launch_bounds__(Tune<C>::NW * 64) void decode_fused_kernel(const Problem p)
{
    static_assert(!EARLY || ((ELECT || SYNC) && !PAGED), "early loads: in-kernel hand-over, contiguous cache");
    static_assert(!(SYNC && ELECT), "the synchronized scheme has no counters to elect by");
    constexpr int NW = Tune<C>::NW, UP = SYNC && C == 128 ? 8 : Tune<C>::UP;
    __shared__ ChunkLds<NW> lds;
    const int tid = threadIdx.x;
    if constexpr (ELECT || SYNC) fetch_arguments_now(p);
    // Workgroups are dealt to the 8 XCDs round-robin by index.  In a short launch that hands its rows
    // over inside the kernel all chunks of a row go to the same XCD (row % 8), so the row's counters
    // and partial results stay in one L2 instead of bouncing between eight; long ones and those that leave the
    // epilogue to a second launch spread them, as do long rows of which there are fewer than eight (FusedLauncher, row_slot).  Placement only affects speed: every
    // hand-over below is device-coherent wherever the workgroups land.
    // Order within that: row-major -- all chunks of rows 0..7, then of rows 8..15, ... -- except in
    // the launches of at most one workgroup per compute unit (EARLY), which go chunk-major and whose
    // order hardly matters (every workgroup is resident at once).  Chunk-major order -- chunk 0 of
    // every row, then chunk 1, ... -- used to serve every launch of up to 1024 workgroups, because it
    // dispatches the chunks past the end of the sequences last (8192 keys in a cache of 16384: 33.5 ->
    // 29 us); but it confines a round of the chip to one slice of every row, and for rows of a
    // power-of-two stride that costs up to 20 % on some boxes (2 x 32 rows of 8192 keys, 1024-key
    // chunks: 54.3 us against 44.7 row-major on the same box; 1 x 32 rows of 16384 keys, 512-key chunks:
    // 51.1 against 46.3; other boxes: 45.8 either way), where row-major with the in-kernel hand-over
    // loses 4 % on the half-empty cache (24.2 -> 25.2 us, 25.9 -> 26.8 us at a quarter).
    const int groups8 = (p.rows + 7) >> 3;
    const int j = blockIdx.x >> 3;
    constexpr bool CM = EARLY;                 // chunk-major in the one-round launches only (see below)
    const bool plain = !ELECT && plain_order<SYNC>(p);
    int c = plain ? (int)blockIdx.x % p.nc : CM ? j / groups8 : j % p.nc;
    int row = plain ? (int)blockIdx.x / p.nc : row_slot(p, blockIdx.x & 7, c) + 8 * (CM ? j - c * groups8 : j / p.nc);
    if (SYNC && p.G > 1 && !shared_order(p, row, c)) return;
    if (row >= p.rows) return;
    FD_PHASE(0);
    if constexpr (SYNC) {
        chunk_body<C, NW, UP, true, EARLY, PAGED, ONE>(p, row, c, lds);
        return;
    }
    int S;
    const bool redo = chunk_body<C, NW, UP, false, EARLY, PAGED, ONE>(p, row, c, lds, &S);
    FD_PHASE(3);
    const int nb = (S + p.C - 1) / p.C;        // chunks of this row that hold a valid key
    if (c >= nb) {                             // padding chunk: zero partials were written
        if (nb == 0 && c == 0 && ELECT) {    // empty sequence: nobody else owns the row
            if (tid < kHeadDim) p.out[(size_t)row * kHeadDim + tid] = 0;
            if (tid == 0) p.ws.row_flags[row] = 0;
        }
        return;
    }
    if (redo) {                                // Section 3 "Recomputation", for this partial vector (not done in place)
        __syncthreads();
        chunk_body<C, NW, UP < 2 ? UP : 2, true, false, PAGED>(p, row, c, lds);
    }

    if (!ELECT) return;                        // a row-epilogue launch follows
    // Publish this chunk's results (written through by wavefront 0), then arrive; the last arrival owns the row and reads
    // the others' results past the caches.
    if (tid >= 64) return;
    wait_stores_performed();
    FD_PHASE(4);
    const bool last = arrive_and_elect(p, row, c, nb);
    FD_PHASE(5);
    if (!last) return;
    finish_row<true, true>(p, row, nb, [nb] { return nb; });
#ifdef FD_PHASE_PROBE
    wait_stores_performed();
    FD_PHASE(7);
#endif
}

// First launch of the literal chain: Eq. 4 inner sums and the range guard, nothing else (no
// recomputation, no hand-over; a flagged chunk's sums are whatever they come to until the second launch replaces
// them.  Going on in place as the fused kernel does took 1 x 32 heads x 1024 keys 10.95 us, now 10.75, 16 x 32 x 125 .. 1000 42.65, now
// 42.3; 2 x 16 x 30000 79.0, now 79.9).  Same workgroup shape, workgroup order and early loads as the
// fused kernel: SMALL = a launch of at most 1024 workgroups (kernel arguments fetched in one batch),
// EARLY = of at most 256 (chunk-major order, first loads before the sequence length has arrived).  ONE: see
// LoadAhead.
template <int C, bool SMALL, bool EARLY, bool ONE = false>
__global__ __launch_bounds__(Tune<C>::NW * 64) void partial_unified_kernel(const Problem p)
{
    static_assert(!EARLY || SMALL, "early loads belong to the small launches");
    constexpr int NW = Tune<C>::NW, UP = Tune<C>::UP;
    __shared__ ChunkLds<NW> lds;
    if constexpr (SMALL) fetch_arguments_now(p);
    const int groups8 = (p.rows + 7) >> 3;
    const int j = blockIdx.x >> 3;
    const int c = EARLY ? j / groups8 : j % p.nc;              // the fused kernel's orders
    const int row = row_slot(p, blockIdx.x & 7, c) + 8 * (EARLY ? j - c * groups8 : j / p.nc);
    if (row >= p.rows) return;
    chunk_body<C, NW, UP, false, EARLY, false, ONE, true>(p, row, c, lds);
}

// Second launch of the literal chain, over (row, chunk) items: every item first forms its row's
// flag, the OR of the row's chunk flags (Section 3 "Recomputation": one logit out of range
// condemns the whole vector).
//   row clean   : the item of chunk 0 adds the row's partial sums and divides -- Eq. 4 outer
//                 sums, fixed order, no atomics; the other items have nothing to do;
//   row flagged : every item recomputes its chunk by the synchronized partial softmax -- chunk
//                 maximum m, l = sum e^{x-m}, f.V -- into the chunk's slot (Eq. 2, per partial
//                 vector); the third launch merges them.
// The grid is bounded; workgroups stride over the items.
template <int C> struct ChainTune {
    static constexpr int NW = 8;
    static constexpr int NG = C / (4 * NW);
    // (chunks from 256 keys: with 4 the kernel takes up to 161 registers, a compute unit holds one workgroup instead of two, and the launch of 512 runs in
    // two rounds: 4 x 32 heads x 32768 keys 30.9 us, with 2 21)
    static constexpr int UP = C >= 256 ? 2 : NG < 4 ? NG : 4;
};
template <int C>
__global__ __launch_bounds__(ChainTune<C>::NW * 64) void chain_combine_kernel(const Problem p)
{
    constexpr int NW = ChainTune<C>::NW, UP = ChainTune<C>::UP;
    constexpr int KB = NW * 2;                  // items per batch: one per half wavefront
    __shared__ ChunkLds<NW> lds;
    __shared__ int item_flag[KB];
    const int tid = threadIdx.x, half = tid >> 5, j = tid & 31;
    const long long items = (long long)p.rows * p.nc;
    // Workgroups stride over the items (the chunks of a flagged row go to different workgroups) and
    // take them in batches of KB: the row flags of a whole batch are fetched at once -- 32 threads
    // per item OR the row's chunk flags -- so a batch of clean rows costs one memory round trip.
    // All nc slots are read: chunks without a valid key carry flag 0 and zero sums, so neither the
    // decision nor the outer sums need the sequence length.
    for (long long w0 = blockIdx.x; w0 < items; w0 += (long long)KB * gridDim.x) {
        const long long mine = w0 + (long long)half * gridDim.x;
        int f = 0;
        if (mine < items) {
            const uint8_t *cf = p.ws.chunk_flags + (size_t)(mine / p.nc) * p.nc;
            for (int i = j; i < p.nc; i += 32) f |= cf[i];
        }
        const unsigned long long any = __ballot(f != 0);
        if (j == 0) item_flag[half] = ((any >> (32 * (half & 1))) & 0xffffffffull) != 0ull;
        __syncthreads();
        for (int k = 0; k < KB; ++k) {
            const long long w = w0 + (long long)k * gridDim.x;
            if (w >= items) break;
            const int row = (int)(w / p.nc), c = (int)(w % p.nc);
            const int flagged = item_flag[k];
            if (c == 0 && tid == 0) p.ws.row_flags[row] = flagged ? 1 : 0;
            if (flagged) {
                chunk_body<C, NW, UP, true>(p, row, c, lds);                // (a chunk without keys leaves at once)
                __syncthreads();                                             // lds is reused by the next item
            } else if (c == 0) {
                // 4 slices of 128 threads; slice s adds chunks s, s+4, ...; the slices are added in order
                const int slice = tid >> 7, t = tid & 127;
                const float *num = p.ws.num + (size_t)row * p.nc * kHeadDim + t;
                const float *den = p.ws.den + (size_t)row * p.nc;
                float s = 0.f, l = 0.f;
#pragma unroll 4
                for (int i = slice; i < p.nc; i += 4) {
                    s += num[(size_t)i * kHeadDim];
                    l += den[i];
                }
                lds.acc[slice][t] = s;
                if (t == 0) lds.den[slice] = l;
                __syncthreads();
                if (tid < kHeadDim) {
                    const float st = ((lds.acc[0][t] + lds.acc[1][t]) + lds.acc[2][t]) + lds.acc[3][t];
                    const float lt = ((lds.den[0] + lds.den[1]) + lds.den[2]) + lds.den[3];
                    // an empty sequence has no term at all: zeros
                    p.out[(size_t)row * kHeadDim + t] = lt > 0.f ? to_half_bits(st / lt) : (uint16_t)0;
                }
                __syncthreads();
            }
        }
        __syncthreads();                        // item_flag is rewritten by the next batch
    }
}

template <template <int> class Launcher, typename... Args>
hipError_t dispatch_chunk(int C, Args... args)
{
    switch (C) {
        case 64:   return Launcher<64>::run(args...);
        case 128:  return Launcher<128>::run(args...);
        case 256:  return Launcher<256>::run(args...);
        case 512:  return Launcher<512>::run(args...);
        case 1024: return Launcher<1024>::run(args...);
        case 2048: return Launcher<2048>::run(args...);
        case 4096: return Launcher<4096>::run(args...);
        default:   return hipErrorInvalidValue;
    }
}

// Whether a wavefront asks for a block of keys only when the one before has arrived (chunk_body's ONE), instead of keeping two in
// flight.  Whole call, two blocks / one.
//   Where the chunks are turned (more than 32 per row, see `rot` there) what bounds rows of a power-of-two stride is the memory
// channels that the workgroups in flight share, and more requests at a time make it worse; rows of other strides do not mind.  Chunks of
// 1024 keys: 16 rows x 65536 keys 98.1 / 92.1 us, 2 x 8 x 20000 .. 65536 91.2 / 84.6, 8 x 131072 102.6 / 94.6, 32 x 131072 396 / 362, 16 x
// 66560 107.3 / 101.4, 16 x 60000 80.4 / 80.2; of 512 16 x 65536 94.3 / 93.8; of 256 1 x 32 x 16384 49.1 / 49.0.
//   A launch of more than three workgroups per compute unit that hands nothing over has other workgroups to cover the wait, and
// wins or ties: 2 x 32 x 29393 in 29 157.6 / 153.5 us (14696 .. 29393 144.1 / 140.0), 4 x 16 x 30000 in 30 163.1 / 160.2, 3 x 32 x 14602
// 116.0 / 114.3, 4 x 32 x 16000 .. 32768 279.1 / 276.2, 8 x 32 x 8192 162.9 / 163.3, 16 x 32 x 4096 164.0 / 163.8.
//   Smaller launches of up to 32 chunks per row lose (3 x 32 x 1500 in 5 15.0 / 15.35, 3 x 32 x 4096 33.15 / 33.8), and so do chunks of
// 2048 keys (1 x 40 x 60000 in 30 198.0 / 202.1, 32 x 131072 314.7 / 316.4).  Shorter chunks than 256 keys have no third block.
//   Paged caches in launches without a hand-over the same: 3 x 32 x 2470 .. 19765 (page 256) 95.7 / 93.6, 8 x 16 x 4000 .. 16000 (64) 108.75 / 108.3,
// 11 x 16 x 1275 .. 10200 (16) 101.4 / 101.8.  With a hand-over chunks of more than 512 keys do: 1 x 32 x 46680 (256) in 2048 122.8 / 119.1, 2 x 16 x 30000 (256) in
// 2048 81.95 / 79.5, 1 x 16 x 18074 (256) in 1216 26.95 / 26.06, 1 x 32 x 8192 (64) in 1024 31.55 / 31.0; of 512 2 x 32 x 3000 (64) 19.8 / 19.9, 1 x 40 x 4000 (16)
// 18.4 / 18.5.
template <int C> struct LoadAhead {
    static constexpr bool kOneBuilt = C >= 256 && C <= 1024;
    static bool one(const Problem &p)
    {
        return kOneBuilt && (p.nc > 32 || (!p.elect && (long long)p.rows * p.nc > 3 * kComputeUnits));
    }
};

template <int C> struct FusedLauncher {
    static hipError_t run(const Problem &p0, hipStream_t s)
    {
        const unsigned grid = (unsigned)(8ll * ((p0.rows + 7) / 8) * p0.nc);
        if (grid == 0) return hipSuccess;
        Problem p = p0;
        // Every XCD reads from every row where the launch is long: more than 1024 workgroups, or more than one round of the
        // chip over 320 MiB of cache (see row_slot); the results cross between XCDs as well as within one.  So they do in rows of more
        // than 32 chunks where there are fewer than eight, which would else use as many XCDs as there are rows: whole call, rows on fixed
        // XCDs / this, 2 rows x 131072 keys 59.4 / 38.1 us, 1 x 131072 32.5 / 21.4, 4 x 131072 73.0 / 50.8, 4 x 16384 14.6 / 12.3, 2 x 2 x 8192 10.1 / 9.0,
        // 2 x 4096 7.8 / 7.5; not up to 32: 1 x 1000 in 16 5.1 / 5.4, 4 x 700 in 11 5.5 / 5.8, 4 x 2048 in 32 5.95 / 5.98.
        const bool few = p.rows < 8 && grid > (unsigned)kComputeUnits;
        p.scatter |= !p.elect || few || grid > 1024u || (grid > (unsigned)kComputeUnits && cache_bytes(p) >= kLongLaunchBytes);
        if constexpr (LoadAhead<C>::kOneBuilt) {
            if (p.block_table && !p.elect && LoadAhead<C>::one(p))
                return launch(decode_fused_kernel<C, false, true, false, true>, dim3(grid), dim3(Tune<C>::NW * 64), s, p);
        }
        if (p.block_table)
            return p.elect ? launch(decode_fused_kernel<C, true, true, false, (C >= 1024)>, dim3(grid), dim3(Tune<C>::NW * 64), s, p)
                           : launch(decode_fused_kernel<C, false, true>, dim3(grid), dim3(Tune<C>::NW * 64), s, p);
        if (p.elect && grid <= (unsigned)kComputeUnits)
            return launch(decode_fused_kernel<C, true, false, true>, dim3(grid), dim3(Tune<C>::NW * 64), s, p);
        if constexpr (LoadAhead<C>::kOneBuilt) {
            if (LoadAhead<C>::one(p))
                return p.elect ? launch(decode_fused_kernel<C, true, false, false, true>, dim3(grid), dim3(Tune<C>::NW * 64), s, p)
                               : launch(decode_fused_kernel<C, false, false, false, true>, dim3(grid), dim3(Tune<C>::NW * 64), s, p);
        }
        return p.elect ? launch(decode_fused_kernel<C, true>, dim3(grid), dim3(Tune<C>::NW * 64), s, p)
                       : launch(decode_fused_kernel<C, false>, dim3(grid), dim3(Tune<C>::NW * 64), s, p);
    }
};

template <int C> struct UnifiedLauncher {
    static hipError_t run(const Problem &p0, hipStream_t s)
    {
        const unsigned grid = (unsigned)(8ll * ((p0.rows + 7) / 8) * p0.nc);
        if (grid == 0) return hipSuccess;
        Problem p = p0;
        p.scatter |= grid > 1024u;                 // no hand-over in this launch; measured on large grids only
        const dim3 block(Tune<C>::NW * 64);
        if (grid <= (unsigned)kComputeUnits) return launch(partial_unified_kernel<C, true, true>, dim3(grid), block, s, p);
        if constexpr (LoadAhead<C>::kOneBuilt) {
            if (LoadAhead<C>::one(p))
                return grid <= 1024u ? launch(partial_unified_kernel<C, true, false, true>, dim3(grid), block, s, p)
                                     : launch(partial_unified_kernel<C, false, false, true>, dim3(grid), block, s, p);
        }
        if (grid <= 1024u) return launch(partial_unified_kernel<C, true, false>, dim3(grid), block, s, p);
        return launch(partial_unified_kernel<C, false, false>, dim3(grid), block, s, p);
    }
};

template <int C> struct ChainCombineLauncher {
    static hipError_t run(const Problem &p, hipStream_t s)
    {
        const long long items = (long long)p.rows * p.nc;
        if (items == 0) return hipSuccess;
        // two workgroups of 8 wavefronts fit a compute unit: one round of the chip, striding over the items
        const unsigned grid = (unsigned)(items < 512 ? items : 512);
        return launch(chain_combine_kernel<C>, dim3(grid), dim3(ChainTune<C>::NW * 64), s, p);
    }
};

// The synchronized scheme of a (row, chunk) in two passes: the logits into LDS and their maximum; weights and V.  See SyncLauncher.
template <int C>
__global__ __launch_bounds__(256) void partial_sync_kernel(const Problem p)
{
    constexpr int NW = 4, UP = 8, NBLK = C / (4 * NW * UP);
    __shared__ ChunkLds<NW> lds;
    __shared__ float logit[C];
    fetch_arguments_now(p);
    const bool plain = plain_order<true>(p) || p.nc > 32;
    const int j = blockIdx.x >> 3;
    int c = plain ? (int)blockIdx.x % p.nc : j % p.nc;
    int row = plain ? (int)blockIdx.x / p.nc : row_slot(p, blockIdx.x & 7, c) + 8 * (j / p.nc);
    if (p.G > 1 && !shared_order(p, row, c)) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, seg = lane & 15, sub = lane >> 4;
    const int b = row / p.Hq, hkv = (row - b * p.Hq) / p.G, start = c * p.C;
    const size_t slot = (size_t)row * p.nc + c;
    const int last = min(p.C, clamp_len(p, p.seq_lens[b]) - start) - 1;
    if (last < 0) {                            // empty chunk: zero partials
        if (tid < kHeadDim) p.ws.num[slot * kHeadDim + tid] = 0.f;
        if (tid == 0) {
            p.ws.den[slot] = 0.f;
            p.ws.mloc[slot] = -INFINITY;
            store_meta(p, slot, 0.f, p.phi, 0);
        }
        return;
    }
    const u32x4 qv = reinterpret_cast<const u32x4 *>(p.q + (size_t)row * kHeadDim)[seg];
    const size_t base = (((size_t)b * p.Hkv + hkv) * p.Smax + start) * 16 + seg;
    const u32x4 *kp = reinterpret_cast<const u32x4 *>(p.k) + base, *vp = reinterpret_cast<const u32x4 *>(p.v) + base;
    auto key_of = [&](int g) { return (g * NW + wave) * 4 + sub; };
    const int nblk = min(NBLK, last / (UP * NW * 4) + 1);
    float m = -INFINITY;
#pragma unroll 1
    for (int blk = 0; blk < nblk; ++blk) {
        u32x4 kk[UP];
#pragma unroll
        for (int u = 0; u < UP; ++u) kk[u] = load_stream(kp + (size_t)min(key_of(blk * UP + u), last) * 16);
#pragma unroll
        for (int u = 0; u < UP; ++u) {
            const int key = key_of(blk * UP + u);
            float x = row16_sum(dot8(qv, kk[u])) * p.scale;
            x = key <= last ? x : -INFINITY;
            if (seg == 0) logit[key] = x;
            m = fmaxf(m, x);
        }
    }
    m = columns_max(m);
    if (lane == 0) lds.top[wave] = m;
    __syncthreads();
    m = lds.top[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) m = fmaxf(m, lds.top[w]);
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float den = 0.f;
#pragma unroll 1
    for (int blk = 0; blk < nblk; ++blk) {
        u32x4 vv[UP];
#pragma unroll
        for (int u = 0; u < UP; ++u) vv[u] = load_stream(vp + (size_t)min(key_of(blk * UP + u), last) * 16);
#pragma unroll
        for (int u = 0; u < UP; ++u) {
            const float e = __builtin_amdgcn_exp2f((logit[key_of(blk * UP + u)] - m) * kLog2e);   // 0 for padding
            den += e;
            axpy8(acc, e, vv[u]);
        }
    }
    float u[2];
    wave_sums(acc, den, u);
    *sums_place(lds.acc[wave], lane) = make_float2(u[0], u[1]);
    if (lane == 0) lds.den[wave] = den;
    __syncthreads();
    if (wave != 0) return;
    u[0] = u[1] = den = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {             // wavefront order
        const float2 o = *sums_read(lds.acc[w], lane);
        u[0] += o.x;
        u[1] += o.y;
        den += lds.den[w];
    }
    *reinterpret_cast<float2 *>(&p.ws.num[slot * kHeadDim + 2 * lane]) = make_float2(u[0], u[1]);
    if (lane == 0) {
        p.ws.den[slot] = den;
        p.ws.mloc[slot] = m;
        store_meta(p, slot, den, m, 1);
    }
}

// Chunks beyond 512 keys in launches of more than one workgroup per compute unit, and beyond 1024 always, take two passes: with K and V streamed one after
// the other the chip reads from half as many places at a time.  Shorter chunks, and launches whose workgroups are alone on their compute units,
// take the loop of the other kernels in one.  Whole call, one pass / two: 4 x 32 x 4096 keys in 1024 43.6 / 42.7 us, 2 x 16 x 65536 166.8 / 160.4,
// 2 x 32 x 11851 .. 23703 117.4 / 114.5, 1 x 16 x 60000 in 2048 78.0 / 75.6, 1 x 40 x 52622 173 / 176; 3 x 16 x 2252 .. 4504 in 912 18.6 / 22.0, 16 x 32 x
// 512 .. 4096 in 512 110.8 / 119.1, 23 x 16 x 379 .. 3037 in 256 58.8 / 61.0, 3 x 5 x 3000 in 192 9.4 / 10.8, 8 x 16 x 2000 in 256 25.3 / 24.8.  Both go by
// plain_order; the two passes took one chunk after the other in every launch before, which cost 16 x 32 x 512 .. 4096 138 us, 32 x 32 x
// 127 .. 1022 70.8 (now 60).
template <int C> struct SyncLauncher {
    static hipError_t run(const Problem &p0, hipStream_t s)
    {
        const unsigned grid = (unsigned)((long long)p0.rows * p0.nc);       // (rows that 8 does not divide: plain_order)
        if (grid == 0) return hipSuccess;
        Problem p = p0;
        p.scatter = 1;
        const dim3 blocks(p.G > 1 ? shared_grid(p) : grid);
        const dim3 block(Tune<C>::NW * 64);
        if constexpr (C <= 1024) {
            if (grid <= (unsigned)kComputeUnits) return launch(decode_fused_kernel<C, false, false, true, false, true>, blocks, block, s, p);
        }
        if constexpr (C >= 1024) return launch(partial_sync_kernel<C>, blocks, dim3(256), s, p);
        else {
            if constexpr (LoadAhead<C>::kOneBuilt) {
                if (LoadAhead<C>::one(p)) return launch(decode_fused_kernel<C, false, false, false, true, true>, blocks, block, s, p);
            }
            return launch(decode_fused_kernel<C, false, false, false, false, true>, blocks, block, s, p);
        }
    }
};

}  // namespace

#ifdef FD_PHASE_PROBE
// Probe build only: copies the phase log of the last fused per-row launch to the host
// (synchronizes the device).  `n` = number of 64-bit stamps wanted, <= 4096 * 8.
extern "C" int fd_phase_probe_read(unsigned long long *host_dst, size_t n)
{
    if (!host_dst || n > (size_t)kPhaseMaxGrid * kPhaseSlots) return 1;
    if (hipDeviceSynchronize() != hipSuccess) return 6;
    return hipMemcpyFromSymbol(host_dst, HIP_SYMBOL(fd_phase_log), n * sizeof(unsigned long long), 0,
                               hipMemcpyDeviceToHost) == hipSuccess ? 0 : 6;
}
#endif

hipError_t launch_decode_fused(const Problem &p, hipStream_t s)
{
    return dispatch_chunk<FusedLauncher>(chunk_capacity(p.C), p, s);
}

hipError_t launch_partial_unified(const Problem &p, hipStream_t s)
{
    return dispatch_chunk<UnifiedLauncher>(chunk_capacity(p.C), p, s);
}

hipError_t launch_chain_combine(const Problem &p, hipStream_t s)
{
    return dispatch_chunk<ChainCombineLauncher>(chunk_capacity(p.C), p, s);
}

hipError_t launch_partial_sync(const Problem &p, hipStream_t s)
{
    return dispatch_chunk<SyncLauncher>(chunk_capacity(p.C), p, s);
}

}  // namespace fd

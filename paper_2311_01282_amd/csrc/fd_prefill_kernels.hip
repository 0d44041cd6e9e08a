// Prompt (prefill) phase with the asynchronized softmax of Section 3: every token of a
// prompt attends to itself and the tokens before it (Eq. 1 under the causal mask), all
// weights taken against the unified scaling factor phi.  Partial sums over successive key
// tiles then simply add (Eq. 4): no running maximum, and the output accumulators are never
// rescaled while the keys stream by.  A tile of queries whose guard fires is redone on the
// spot with the synchronized scheme (running maximum per query, Eq. 2).
//
// Matrix-core mapping (16x16x32 MFMA; lane = (n, g) = (lane % 16, lane / 16)):
//   scores   S^T[key][query] = K . Q^T      A = 16 keys of the K tile in LDS, B = Q^T held in
//            registers for the whole kernel.  Row 4g + r of key block t is key
//            k0 + 8g + 4t + r: with that permutation the two score tiles of a 32-key
//            step leave lane (n, g) holding keys k0 + 8g .. 8g + 7 of query n -- exactly
//            the B operand of the second product, no data movement.
//   weights  P = e^{s S^T - phi}, fp32, guard, causal mask.  They go to the matrix cores as fp16
//            hi + lo pairs (22 significant bits).  fp16 has the precision but not the range of
//            e^{x - phi} over the admissible x - phi, so every query carries a scale of its own,
//            2^{k_q}, fixed after its first key step so that the largest weight seen there becomes
//            2^4: numerator and denominator of a query are both scaled by it and it cancels in the
//            division; being constant over the keys of a query it leaves the sums of Eq. 4 as
//            they are -- partial sums still just add, nothing is ever rescaled.  A query whose later
//            logits exceed its first step's maximum by more than 2^11.9 would overflow fp16: its
//            tile is redone with the synchronized scheme, like a tile whose guard fired (but
//            without raising the guard's flag).
//   output   O^T[d][query] = V^T . P^T       A = V^T, taken out of the V tile in LDS by the
//            transposing LDS read (ds_read_b64_tr_b16: four keys of one d per lane); V is
//            fp16 as it is.  Two MFMAs per tile (V Ph + V Pl).
// K and V tiles are loaded from global memory straight into LDS, once per workgroup, and
// shared by its four wavefronts (rings of four tiles; layouts free of bank conflicts for the
// 16-byte operand reads).
#include <type_traits>
#include <utility>

#include "fd_chunk.h"

namespace fd {

namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

constexpr float kFirstStepLog2 = 4.f;     // a query's largest weight of its first key step becomes 2^4 ...
constexpr float kOverflowLog2 = 15.9f;    // ... and no later weight may reach 2^16 (fp16 ends at 65504)

// 16-query blocks per wavefront.  Before the loop was woven, 8192 tokens: 401 TFLOP/s with 1, 471-500 with 2, 426 with 4 (one
// wavefront per SIMD); the woven loop exists for 2 only.
constexpr int kQB = 2;
constexpr int kWaveQ = 16 * kQB;  // queries per wavefront
constexpr int kQTile = 4 * kWaveQ; // query rows per workgroup
constexpr int kStep = 32;        // keys per wavefront step

// ---- the attention kernel ----
// A workgroup owns 128 queries of one head (64 in small launches, see tile_unified): wavefront w the 32 queries i0 + 32w .. +31 (two
// blocks of 16).  The K and V tiles of a 32-key step are loaded once per workgroup into LDS
// and read from there by all four wavefronts as MFMA A operands; Q^T stays in registers as the B
// operand.  Every output row belongs to one wavefront: nothing is reduced across wavefronts, and
// with the unified phi nothing is ever rescaled.
// A 16-byte LDS access of a wavefront is served 16 lanes per cycle, and the 16 are not
// consecutive lanes: lanes 0-3, 12-15, 20-27 share a cycle, lanes 4-11, 16-19, 28-31 the next
// (measured with a two-lane probe; likewise for the upper half).  In terms of lane = 16g + n a
// cycle holds every n once, taken from two different g.  A layout is conflict-free when the
// 16-byte unit (address / 16 mod 16) of lane (n, g) is a permutation of n, as n ^ g (the K layout).
constexpr int kTileBytes = kStep * kHeadDim * 2;                // 8 KiB: one 32-key tile of K or V
constexpr int kVTileBytes = kTileBytes + 384;                   // ... of V as it lies in LDS (see v_block)
constexpr int kRing = 4;                                        // tiles of each in LDS (see tile_unified)
struct PrefillLds {
    alignas(16) unsigned char k[kRing][kTileBytes];             // [key][16 chunks of 16 bytes, XOR-swizzled]
    alignas(16) unsigned char v[kRing][kVTileBytes];            // [key][8 chunks of 32 bytes], swizzled and shifted
    int bad[4], redo[4];
};

// V keeps its own layout (a key's 256 bytes in a row); ds_read_b64_tr_b16 turns it round: of 16 lanes, lane 4j + i reads
// 8 bytes, piece i of the 32 bytes (16 d) of key j, and lane n receives d = n of the four keys.  Lane (n, g) of the A
// operand of tile dt needs keys 8g .. 8g + 7 of d = 16 dt + n: two such reads, keys 8g + (0..3) and 8g + (4..7).  Eight
// keys are read at a time, 8g + 4h + (0..3) of two neighbouring g, 32 bytes of each: they have to lie in different
// 32-byte units modulo 8.  So the unit of a row is XORed with key % 4 within its half of the row, and the
// blocks of four keys of each g are shifted by half a row (128 bytes) against those of g - 1: blocks stay 1 KiB in a row,
// as the tile fetch writes them, and the unit of tile dt is an XOR with dt % 4 plus an immediate 128 (dt / 4).
// (Before, a launch of its own wrote a transposed copy of V: 8 - 26 us and 4 bytes of traffic per element.  Whole call, that form /
// this: 4 ragged prompts of up to 1024 tokens 68.6 / 56.3 us, 1 x 32 heads x 8192 695.7 / 690.6, 2 x 64/8 heads x 4001, where
// eight heads share the copy, 578.9 / 588.0: a tile of V takes 16 of these reads where it took 8 of 16 bytes.)
__device__ __forceinline__ int v_block(int blk) { return blk * 1024 + (blk >> 1) * 128; }   // keys 4 blk .. 4 blk + 3

// K row r, 16-byte chunk c sits in chunk c ^ k_key(r) of the row.  Lane (n, g) reads row r(n) in {0..3, 8..11,
// 16..19, 24..27} (+4 for the second key block), chunk 4 kb + g: k_key(r) = n for those rows, which puts it in unit
// (4 kb + g) ^ n; a row's 16 chunks stay a permutation of themselves, so the row-wise writes are conflict-free too.
__device__ __forceinline__ int k_key(int r) { return (r & 3) | (((r >> 3) & 3) << 2); }

// What both schemes share: a wavefront's place in the tile, its operands in registers, the tile fetch.
struct TileWave {
    int lane, wave, n, g;
    int w0;                      // first query of this wavefront
    int nsteps, mine;            // key steps of the workgroup, of this wavefront (0: it has no query)
    const unsigned char *kbase, *vbase;
    int keys;                    // the prompt's length: K rows that hold a key
    int k_voff0, k_voff1;        // this thread's two chunks of a K tile, from the tile's start
    int v_voff0;                 // ... and its first of a V tile (the second is 4 KiB further)
    int k_rd[4], v_rd[4];        // this lane's operand reads, from the start of the LDS tile
    bool masked;                 // its last step holds its own 32 keys (SPLIT: of the two wavefronts of a query group, of one)
    f16x8 qB[kQB][4];            // Q^T as the B operand: lane (n, g) holds d = 32 kb + 8g .. +7 of query w0 + 16 qb + n

    // SPLIT: see tile_unified
    __device__ __forceinline__ TileWave(const PrefillProblem &p, int b, int hq, int i0, int S, bool split = false)
    {
        const int tid = threadIdx.x;
        lane = tid & 63;
        wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        n = lane & 15;
        g = lane >> 4;
        w0 = i0 + kWaveQ * (split ? wave >> 1 : wave);
        nsteps = (min(i0 + (split ? kQTile / 2 : kQTile), S) - 1) / kStep + 1;
        const int last_q = min(w0 + kWaveQ, S) - 1;                  // < w0 when the wavefront has no query (as in front of the prompt)
        mine = last_q >= w0 && w0 >= 0 ? last_q / kStep + 1 : 0;
        masked = true;
        const int part = split ? wave & 1 : 0;
        if (split) {
            nsteps = (nsteps + 1) / 2;
            masked = ((mine - 1) & 1) == part;
            mine = (mine - part + 1) / 2;                            // steps of this parity
        }
        const size_t kv_head = (size_t)b * p.Hkv + hq / p.G;
        kbase = reinterpret_cast<const unsigned char *>(p.k + kv_head * p.Smax * kHeadDim);
        vbase = reinterpret_cast<const unsigned char *>(p.v + kv_head * p.Smax * kHeadDim);
        keys = S;
        const int r = tid >> 4, c = (tid & 15) ^ k_key(r);
        k_voff0 = r * 256 + c * 16;
        k_voff1 = (r + 16) * 256 + (c ^ 8) * 16;                     // k_key(r + 16) = k_key(r) ^ 8
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) k_rd[kb] = part * kTileBytes + (8 * (n >> 2) + (n & 3)) * 256 + (((4 * kb + g) ^ n) << 4);
        v_voff0 = r * 256 + (((tid & 15) ^ ((r & 3) << 1)) << 4);    // 32-byte unit ^ key % 4, in 16-byte chunks
#pragma unroll
        for (int x = 0; x < 4; ++x) v_rd[x] = part * kVTileBytes + v_block(2 * g) + (n >> 2) * 256 + ((x ^ (n >> 2)) << 5) + (n & 3) * 8;
        // rows past the prompt may hold anything: zeros in their place
        const uint16_t *qbase = p.q + (((size_t)b * p.Hq + hq) * p.Smax) * kHeadDim;
#pragma unroll
        for (int qb = 0; qb < kQB; ++qb) {
            const int row = w0 + 16 * qb + n;
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) {
                u32x4 t = {0u, 0u, 0u, 0u};
                if ((unsigned)row < (unsigned)S) t = *reinterpret_cast<const u32x4 *>(qbase + (size_t)row * kHeadDim + 32 * kb + 8 * g);
                qB[qb][kb] = __builtin_bit_cast(f16x8, t);
            }
        }
    }
    // Tile fetch, global memory straight into LDS (no staging registers): a wavefront's load instruction fills 1 KiB
    // of LDS, lane l the 16 bytes at 16 l from the wavefront's base.  Thread t moves chunks t and t + 256 of a tile.
    // Buffer loads through a window of kRing tiles: what lies past the last key of the prompt (or past the last tile)
    // arrives as zeros and touches no memory, so the loop can run its fetches ahead without a condition, and
    // inside a window a fetch costs three scalar instructions.
    __device__ __forceinline__ u32x4 window(const unsigned char *base, int t0) const
    {
        const unsigned left = __builtin_amdgcn_readfirstlane(max(min(keys - t0 * kStep, kRing * kStep), 0));      // (uniform: keep it scalar)
        const unsigned long long at = reinterpret_cast<unsigned long long>(base) + (unsigned long long)t0 * kTileBytes;
        return u32x4{(unsigned)at, (unsigned)(at >> 32) & 0xffffu, left * (kHeadDim * 2), 0x00027000u};          // raw buffer, stride 0
    }
    __device__ __forceinline__ u32x4 k_window(int t0) const { return window(kbase, t0); }
    __device__ __forceinline__ u32x4 v_window(int t0) const { return window(vbase, t0); }
    // In assembly, because the compiler waits for the loads it knows to write LDS before every transposing LDS read
    // (a step then takes 1120 cycles instead of 920); no register is written -- the LDS address goes into m0 as an operand, so that
    // the compiler knows what m0 holds -- and the waits are wait_fetches.  KNOWN: the builtin, for the prologue, whose loads the
    // compiler has to tell from those of Q^T; all_landed tells it that they are there.
    template <bool KNOWN> static __device__ __forceinline__ void load(u32x4 rs, int voff, int soff, unsigned char *lds_1k)
    {
        auto *to = (__attribute__((address_space(3))) unsigned char *)lds_1k;
        if constexpr (KNOWN) {
            const unsigned long long base = rs.x | ((unsigned long long)rs.y << 32);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>(base), 0, (int)rs.z, (int)rs.w),
                                                     (__attribute__((address_space(3))) void *)to, 16, voff, soff, 0, 0);
        } else {
            const unsigned at = (unsigned)reinterpret_cast<uintptr_t>(to);
            asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"{m0}"(at), "v"(voff), "s"(rs), "s"(soff) : "memory");
        }
    }
    // tile u of a window, into place `slot` of the ring
    template <bool KNOWN = false> __device__ __forceinline__ void fetch_k(PrefillLds &lds, u32x4 rs, int u, int slot) const
    {
        load<KNOWN>(rs, k_voff0, u * kTileBytes, lds.k[slot] + wave * 1024);
        load<KNOWN>(rs, k_voff1, u * kTileBytes, lds.k[slot] + wave * 1024 + 4096);
    }
    template <bool KNOWN = false> __device__ __forceinline__ void fetch_v(PrefillLds &lds, u32x4 rs, int u, int slot) const
    {
        load<KNOWN>(rs, v_voff0, u * kTileBytes, lds.v[slot] + v_block(wave));
        load<KNOWN>(rs, v_voff0, u * kTileBytes + 4096, lds.v[slot] + v_block(wave + 4));
    }
    // one of the four loads of a thread: K tile u of window rk into place k_slot, V tile u of window rv into place v_slot
    __device__ __forceinline__ void fetch_piece(PrefillLds &lds, int piece, u32x4 rk, u32x4 rv, int u, int k_slot, int v_slot) const
    {
        if (piece == 0) load<false>(rk, k_voff0, u * kTileBytes, lds.k[k_slot] + wave * 1024);
        if (piece == 1) load<false>(rk, k_voff1, u * kTileBytes, lds.k[k_slot] + wave * 1024 + 4096);
        if (piece == 2) load<false>(rv, v_voff0, u * kTileBytes, lds.v[v_slot] + v_block(wave));
        if (piece == 3) load<false>(rv, v_voff0, u * kTileBytes + 4096, lds.v[v_slot] + v_block(wave + 4));
    }
    __device__ __forceinline__ void fetch_k(PrefillLds &lds, int t) const { fetch_k(lds, k_window(t), 0, t & (kRing - 1)); }
    __device__ __forceinline__ void fetch_v(PrefillLds &lds, int t) const { fetch_v(lds, v_window(t), 0, t & (kRing - 1)); }
    __device__ __forceinline__ u32x4 read_k(const PrefillLds &lds, int slot, int kb, int t) const
    {
        // row m = n of key block t is key 8 (n >> 2) + 4t + (n & 3) of the step, so that the two score
        // tiles leave lane (n, g) holding keys 8g .. 8g + 7 of query n
        return *reinterpret_cast<const u32x4 *>(&lds.k[0][0] + slot * kTileBytes + k_rd[kb] + 1024 * t);
    }
    // V^T operand of tile dt: keys 8g .. 8g + 7 of d = 16 dt + n
    __device__ __forceinline__ f16x8 read_v(PrefillLds &lds, int slot, int dt) const
    {
        typedef __attribute__((address_space(3))) s16x4 *lds_s16x4;
        unsigned char *at = &lds.v[0][0] + slot * kVTileBytes + v_rd[dt & 3] + 128 * (dt >> 2);
        const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)at);
        const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(at + 1024));
        return __builtin_bit_cast(f16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
    }
    // scores of one step
    __device__ __forceinline__ void scores(const PrefillLds &lds, int slot, f32x4 (&sc)[kQB][2]) const
    {
#pragma unroll
        for (int qb = 0; qb < kQB; ++qb)
#pragma unroll
            for (int t = 0; t < 2; ++t) sc[qb][t] = f32x4{0.f, 0.f, 0.f, 0.f};
        u32x4 ka[2][4];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) ka[t][kb] = read_k(lds, slot, kb, t);
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int qb = 0; qb < kQB; ++qb)
                    sc[qb][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, ka[t][kb]), qB[qb][kb], sc[qb][t], 0, 0, 0);
    }
};

// The weights of a step as B operands of the second product: fp16 hi and lo parts of keys 8g .. 8g + 7.
struct Weights {
    u32x4 hi[kQB], lo[kQB];
};

// O^T += V^T P^T with P = Ph + Pl, one step
__device__ __forceinline__ void add_pv(const TileWave &tw, PrefillLds &lds, int slot, const Weights &w, f32x4 (&acc)[8][kQB])
{
    f16x8 av[8];
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) av[dt] = tw.read_v(lds, slot, dt);
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) {
#pragma unroll
        for (int qb = 0; qb < kQB; ++qb)
            acc[dt][qb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av[dt], __builtin_bit_cast(f16x8, w.hi[qb]), acc[dt][qb], 0, 0, 0);
#pragma unroll
        for (int qb = 0; qb < kQB; ++qb)
            acc[dt][qb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av[dt], __builtin_bit_cast(f16x8, w.lo[qb]), acc[dt][qb], 0, 0, 0);
    }
}
// hi = the weights cut to fp16 (11 bits), lo = what that leaves (exact in fp32), rounded to fp16.  neg1 is -1.0 in a
// register the compiler cannot see through: it keeps e - (float)hi a single mixed-precision fused multiply-add.
__device__ __forceinline__ void split_pair(float e0, float e1, float neg1, unsigned &hi, unsigned &lo)
{
    const f16x2 h = __builtin_bit_cast(f16x2, __builtin_amdgcn_cvt_pkrtz(e0, e1));
    const _Float16 h0 = h.x, h1 = h.y;
    f16x2 l;
    l.x = (_Float16)__builtin_fmaf((float)h0, neg1, e0);
    l.y = (_Float16)__builtin_fmaf((float)h1, neg1, e1);
    hi = __builtin_bit_cast(unsigned, h);
    lo = __builtin_bit_cast(unsigned, l);
}

// Over the four lane groups of a query (lanes n, n + 16, n + 32, n + 48): its sum and its maximum, in every lane.
__device__ __forceinline__ float query_sum(float a)
{
    a = rows_sum(a, a);
    return halves_sum(a, a);
}
__device__ __forceinline__ float query_max(float a) { return columns_max(a); }

// Output rows of a wavefront: acc / den, zeros for rows past the prompt.  The accumulators hold 8 bytes of each of 16 rows
// per instruction; they go through 8 KiB of LDS of the wavefront's own (16-byte chunk c of row r in chunk c ^ (r % 16)), so that a
// store instruction writes four whole rows (up to row `end`); all of it is under way at once, without a branch.  What bounds a short prompt is
// what a workgroup does outside its loop: straight from the accumulators, 16 stores of 16 half lines each took a wavefront 3500
// cycles, this 2000.  The rings have to be out of use.
__device__ __forceinline__ void store_rows(const PrefillProblem &p, const TileWave &tw, PrefillLds &lds, int b, int hq, int S, const f32x4 (&acc)[8][kQB], const float (&den)[kQB], int end)
{
    static_assert(4 * kWaveQ * kHeadDim * 2 <= sizeof(lds.k));
    unsigned char *rows = &lds.k[0][0] + tw.wave * (kWaveQ * kHeadDim * 2);
    const int n = tw.n, g = tw.g;
#pragma unroll
    for (int qb = 0; qb < kQB; ++qb) {
        const float inv = 1.f / den[qb];
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) {
            f16x2 a, c;
            a.x = (_Float16)(acc[dt][qb][0] * inv);
            a.y = (_Float16)(acc[dt][qb][1] * inv);
            c.x = (_Float16)(acc[dt][qb][2] * inv);
            c.y = (_Float16)(acc[dt][qb][3] * inv);
            *reinterpret_cast<u32x2 *>(rows + (16 * qb + n) * 256 + (((2 * dt + (g >> 1)) ^ n) << 4) + (g & 1) * 8) =
                u32x2{__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, c)};
        }
    }
    u32x4 t[kWaveQ / 4];                                       // lane (n, g): chunk n of rows 4 i + g
#pragma unroll
    for (int i = 0; i < kWaveQ / 4; ++i) {
        const int r = 4 * i + g;
        t[i] = *reinterpret_cast<const u32x4 *>(rows + r * 256 + ((n ^ (r & 15)) << 4));
    }
    // through a window that ends at the buffer's last row: what lies past it is not written
    const int row0 = max(tw.w0, 0);
    uint16_t *o = p.out + (((size_t)b * p.Hq + hq) * p.Smax + row0) * kHeadDim;
    const int left = __builtin_amdgcn_readfirstlane(tw.w0 < 0 ? 0 : max(min(end - row0, kWaveQ), 0)) * (kHeadDim * 2);
    const auto window = __builtin_amdgcn_make_buffer_rsrc(o, 0, left, 0x00027000);
#pragma unroll
    for (int i = 0; i < kWaveQ / 4; ++i) {
        const int r = 4 * i + g;
        const bool live = tw.w0 + r < S;
        const u32x4 x = {live ? t[i][0] : 0u, live ? t[i][1] : 0u, live ? t[i][2] : 0u, live ? t[i][3] : 0u};
        __builtin_amdgcn_raw_buffer_store_b128(x, window, r * 256 + n * 16, 0, 0);
    }
}

__device__ __forceinline__ void wait_reads() { __builtin_amdgcn_s_waitcnt(0xc07f); }   // lgkmcnt(0): LDS reads have arrived
template <int N> __device__ __forceinline__ void wait_fetches()        // at most N of this wavefront's loads outstanding
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// No load outstanding, and the compiler takes note of it: it does not see the wait above, and what it still counts as pending it
// would wait for again before the first use -- in order, so with it for every tile fetched in between.  (So it did in the last two
// steps of every wavefront: 4 ragged prompts of up to 1024 tokens 54.8 us, 53.9 without.)
__device__ __forceinline__ void all_landed()
{
    wait_fetches<0>();
    __builtin_amdgcn_s_waitcnt(0x0f70);                                // vmcnt(0)
    asm volatile("" ::: "memory");
}
// Of the LDS tiles: past it a place that this wavefront has read may be filled again, so its LDS reads have to have returned (the
// compiler would let the last ones, and the matrix instructions that use them, drift past a bare barrier); loads in flight are not waited for.
__device__ __forceinline__ void workgroup_barrier()
{
    asm volatile("" ::: "memory");
    wait_reads();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// One 128-query tile, unified scaling factor (Eq. 4).  Returns true when the tile has to be redone with the
// synchronized scheme -- its guard fired (recorded in tile_flags) or a weight left the range of the fp16 operands (not
// recorded: the result is the same either way).
//
// What bounds it: the matrix pipe and the issue port of a SIMD, and at that rate power (a run of 8192 tokens holds
// 1.65 GHz; one wavefront per SIMD 2.1).  A step of a wavefront is 48 matrix instructions of 16 pipe cycles (768) and 88
// vector instructions; the vector instructions of one wavefront do not run under the matrix instructions of the other
// wavefront of its SIMD, but within a wavefront up to two independent ones do per matrix instruction (a probe of 48 + 96 takes
// 810 cycles, with 16 exponentials 955).  So the three parts of a step are taken from three different steps, which do not
// depend on each other, and woven together by hand: iteration s runs
//     P.V of step s  |  weights of step s + 1  |  scores of step s + 2
// The two wavefronts of a SIMD then take a step per 864 cycles between them, against 1560 for scores, weights and P.V
// of one step after the other.  1 x 32 heads x 8192 tokens: 853 TFLOP/s of useful work (710 before the weaving and
// what followed it), 1.28 PFLOP/s issued.  32x32x16 matrix instructions in the same loop: 839 cycles where this one then took
// 947, but the clock fell from 1.77 to 1.48 GHz (726 us against 685).
template <class F, int... I> __device__ __forceinline__ void unrolled(std::integer_sequence<int, I...>, F f)
{
    (f(std::integral_constant<int, I>{}), ...);
}
// SPLIT: a tile of 64 queries, two wavefronts to 32 of them: one takes the even key steps, the other the odd ones, each under scales of its own;
// at the end the sums of the odd ones are brought to the common scale and added (Eq. 4).  A step is two tiles of K and of V for the workgroup, the rings hold
// two, what iteration s fetches (K of s + 3, V of s + 1) it also waits for, and V is not read ahead.  Where a launch has few tiles its length is that of the
// longest walk, and a step takes 0.65 us whether a SIMD holds one wavefront or two: here a walk is half the steps,
// of two tiles each (1 x 32 heads x 1024 tokens, heaviest tile: 32 steps before, 16 now; whole call 24.9 / 21.2 us).
template <bool SPLIT>
__device__ __forceinline__ bool tile_unified(const PrefillProblem &p, PrefillLds &lds, int b, int hq, int i0, int S)
{
    const TileWave tw(p, b, hq, i0, S, SPLIT);
    const int tid = threadIdx.x, lane = tw.lane, wave = tw.wave, n = tw.n, g = tw.g, mine = tw.mine;
    const float c1 = p.scale * kLog2e, c0 = -p.phi * kLog2e;      // log2 of e^{s x - phi} = c1 x + c0
    const float lo2 = p.lo * kLog2e, hi2 = p.hi * kLog2e;
    float neg1;
    asm("v_mov_b32 %0, -1.0" : "=v"(neg1));

    f32x4 acc[8][kQB];
#pragma unroll
    for (int dt = 0; dt < 8; ++dt)
#pragma unroll
        for (int qb = 0; qb < kQB; ++qb) acc[dt][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
    // running extremes of log2 of the SCALED weights (guard, fp16 range), and the queries' scale exponents
    // k_q, folded into the additive constant of the logit
    float den[kQB], zlo[kQB], zhi[kQB], kq[kQB], c0q[kQB];
#pragma unroll
    for (int qb = 0; qb < kQB; ++qb) { den[qb] = 0.f; zlo[qb] = INFINITY; zhi[qb] = -INFINITY; kq[qb] = 0.f; c0q[qb] = c0; }

    // Tiles in LDS: rings of four.  Entering iteration s, K tile s + 2 and V tiles s and s + 1 have landed for
    // every wavefront; iteration s fetches K tile s + 4 and V tile s + 3, whose places were last read in iteration
    // s - 1 at the latest (those reads have returned: workgroup_barrier), and waits at its end for what iteration s - 1 fetched: a
    // load has two iterations to land.
    const u32x4 k0 = tw.k_window(0), v0 = tw.v_window(0);
    if constexpr (SPLIT) {
#pragma unroll
        for (int u = 0; u < 4; ++u) tw.fetch_k<true>(lds, k0, u, u);
        tw.fetch_v<true>(lds, v0, 0, 0); tw.fetch_v<true>(lds, v0, 1, 1);
    } else {
        tw.fetch_k<true>(lds, k0, 0, 0); tw.fetch_k<true>(lds, k0, 1, 1);
        tw.fetch_v<true>(lds, v0, 0, 0); tw.fetch_k<true>(lds, k0, 2, 2);
        tw.fetch_v<true>(lds, v0, 1, 1);
        tw.fetch_k<true>(lds, k0, 3, 3); tw.fetch_v<true>(lds, v0, 2, 2);
    }
    // one of the eight loads of a thread for step s (SPLIT), odd: s is odd
    auto split_piece = [&](int piece, u32x4 rk, u32x4 rv, int odd) {
        const int half = (piece >> 1) & 1, u = piece & 1;              // piece 0 .. 3: K tiles, 4 .. 7: V tiles
        const int k_slot = odd ? u : 2 + u, v_slot = odd ? u : 2 + u;  // places of steps s + 3 and s + 1
        if (piece < 4) tw.load<false>(rk, half ? tw.k_voff1 : tw.k_voff0, u * kTileBytes, lds.k[k_slot] + wave * 1024 + 4096 * half);
        else tw.load<false>(rv, tw.v_voff0, u * kTileBytes + 4096 * half, lds.v[v_slot] + v_block(wave + 4 * half));
    };
    auto fetch_ahead = [&](int s) {
        if constexpr (SPLIT) {
            const u32x4 rk = tw.k_window(2 * (s + 3)), rv = tw.v_window(2 * (s + 1));
#pragma unroll
            for (int i = 0; i < 8; ++i) split_piece(i, rk, rv, s & 1);
        } else {
            tw.fetch_k(lds, s + 4);
            tw.fetch_v(lds, s + 3);
        }
    };
    const auto place = [](int s) { return SPLIT ? 2 * (s & 1) : s & (kRing - 1); };       // of step s in the rings
    auto next_iteration = [&]() { wait_fetches<SPLIT ? 0 : 4>(); workgroup_barrier(); };

    // The last step of a wavefront holds its own 32 keys (causal mask): key 8g + j of the step, j = 4t + r, is visible to query
    // 16 qb + n of the wavefront where j - 16 qb <= own.
    const int own = tw.masked ? n - 8 * g : 64;
    // weights of a wavefront's first step from its scores, not woven into anything; last: it is its last one, too
    auto first_weights = [&](bool last, const f32x4 (&sc)[kQB][2], Weights &w) {
#pragma unroll
        for (int qb = 0; qb < kQB; ++qb) {
            float z[8];
            bool ok[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                ok[j] = !last | (j - 16 * qb <= own);
                z[j] = ok[j] ? __builtin_fmaf(sc[qb][j >> 2][j & 3], c1, c0q[qb]) : -INFINITY;
            }
            // The query's scale: its largest weight of this first step becomes 2^kFirstStepLog2.
            // The four lane groups of a query hold different keys: they agree on the maximum first.
            float m = fmaxf(fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3])), fmaxf(fmaxf(z[4], z[5]), fmaxf(z[6], z[7])));
            m = query_max(m);
            const float k = (m == -INFINITY || m != m) ? 0.f : kFirstStepLog2 - m;      // no visible key, or NaN: leave as is
            kq[qb] = k;
            c0q[qb] = c0 + k;
#pragma unroll
            for (int j = 0; j < 8; ++j) z[j] += k;
#pragma unroll
            for (int j = 0; j < 8; j += 2) {
                zhi[qb] = fmaxf(fmaxf(z[j], z[j + 1]), zhi[qb]);
                zlo[qb] = fminf(fminf(ok[j] ? z[j] : INFINITY, ok[j + 1] ? z[j + 1] : INFINITY), zlo[qb]);
                const float e0 = __builtin_amdgcn_exp2f(z[j]), e1 = __builtin_amdgcn_exp2f(z[j + 1]);
                den[qb] += e0;
                den[qb] += e1;
                unsigned h, l;
                split_pair(e0, e1, neg1, h, l);
                w.hi[qb][j >> 1] = h;
                w.lo[qb][j >> 1] = l;
            }
        }
    };

    // Iteration s in full.  av: the V operands of step s, the first four read ahead (and left holding those of s + 1).
    // The 48 matrix instructions in order, P.V (32) before scores (16); behind each up to two or three vector
    // instructions of the weights -- pair i of 8 in slots 6i .. 6i + 5, its last two in the next pair's -- and
    // at most one of the 24 LDS reads or four tile fetches.  The reads of 16 slots are waited for at once, before the 16 that use
    // them (a wait per operand, 17 an iteration, cost 90 of 1560 cycles, the wavefront that leads its SIMD counted), and the fetches
    // are spread because the four wavefronts are in step: 16 loads at a time queue for the address unit (another 80).
    // 1 x 32 heads x 8192 tokens: 673 us with neither, 653 with the first, 648 with both.
    // slot: s modulo the ring; rk, rv: windows that hold K tile s + 4 and V tile s + 3 as their tile u.
    // last: step s + 1 is the wavefront's last (its weights are masked, there are no scores of step s + 2).
    auto iteration = [&](auto last, int slot, u32x4 rk, u32x4 rv, int u, const f32x4 (&sc)[kQB][2], f32x4 (&scn)[kQB][2],
                         const Weights &w, Weights &wn, f16x8 (&av)[8]) {
        constexpr bool kLast = decltype(last)::value;
        float y0 = 0.f, y1 = 0.f;                                                // z0, z1 as the minimum takes them
        u32x4 ka[8];
        float z0 = 0.f, z1 = 0.f, e0 = 0.f, e1 = 0.f, f0 = 0.f, f1 = 0.f;      // the pair in work; f: its predecessor's weights
        _Float16 h0 = 0, h1 = 0;                                                 // ... and their hi parts
        unsigned hp = 0;
        f16x2 lp = {0, 0};
        if constexpr (kLast) {
#pragma unroll
            for (int dt = 0; dt < 8; ++dt) av[dt] = tw.read_v(lds, slot, dt);
        } else if constexpr (SPLIT) {
#pragma unroll
            for (int dt = 0; dt < 4; ++dt) av[dt] = tw.read_v(lds, slot, dt);
        }
        __builtin_amdgcn_sched_barrier(0);
        unrolled(std::make_integer_sequence<int, 48>{}, [&](auto slot_index) {
            constexpr int m = decltype(slot_index)::value;
            // matrix instruction m
            if constexpr (m < 32) {
                constexpr int dt = m >> 2, qb = m & 1;
                const u32x4 pw = (m & 2) ? w.lo[qb] : w.hi[qb];
                acc[dt][qb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av[dt], __builtin_bit_cast(f16x8, pw), acc[dt][qb], 0, 0, 0);
            } else if constexpr (!kLast) {
                constexpr int op = (m - 32) >> 1, kb = op >> 1, t = op & 1, qb = m & 1;
                const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
                scn[qb][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, ka[op]), tw.qB[qb][kb], kb == 0 ? zero : scn[qb][t], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            // operand reads and tile fetches
            if constexpr (!kLast && m < 8 && m % 2 == 1) av[4 + m / 2] = tw.read_v(lds, slot, 4 + m / 2);
            if constexpr (!kLast && m >= 17 && m < 25) ka[m - 17] = tw.read_k(lds, SPLIT ? slot : (slot + 2) & (kRing - 1), (m - 17) >> 1, (m - 17) & 1);
            if constexpr (!SPLIT && !kLast && m >= 33 && m < 41 && m % 2 == 1) av[(m - 33) / 2] = tw.read_v(lds, (slot + 1) & (kRing - 1), (m - 33) / 2);
            if constexpr (SPLIT && m >= 9 && m < 33 && (m - 9) % 3 == 0) split_piece((m - 9) / 3, rk, rv, u);
            if constexpr (!SPLIT && m >= 6 && (m - 6) % 11 == 0) tw.fetch_piece(lds, (m - 6) / 11, rk, rv, u, slot, (slot + 3) & (kRing - 1));
            if constexpr (!kLast && m % 16 == 15 && m < 47) wait_reads();                // (the last 16 slots' reads: at the barrier)
            // weights: pair pr = (query block, keys 2j, 2j + 1)
            constexpr int pr = m / 6, qb = pr >> 2, j = pr & 3;
            constexpr int pp = pr - 1, pqb = pp >> 2, pj = pp & 3;               // the pair before
            switch (m % 6) {
                case 0:
                    z0 = __builtin_fmaf(sc[qb][j >> 1][2 * (j & 1)], c1, c0q[qb]);
                    z1 = __builtin_fmaf(sc[qb][j >> 1][2 * (j & 1) + 1], c1, c0q[qb]);
                    y0 = z0; y1 = z1;
                    if constexpr (kLast) {
                        const bool ok0 = 2 * j - 16 * qb <= own, ok1 = 2 * j + 1 - 16 * qb <= own;
                        y0 = ok0 ? z0 : INFINITY; z0 = ok0 ? z0 : -INFINITY;
                        y1 = ok1 ? z1 : INFINITY; z1 = ok1 ? z1 : -INFINITY;
                    }
                    break;
                case 1:
                    e0 = __builtin_amdgcn_exp2f(z0);
                    zhi[qb] = fmaxf(fmaxf(z0, z1), zhi[qb]);
                    break;
                case 2:
                    e1 = __builtin_amdgcn_exp2f(z1);
                    zlo[qb] = fminf(fminf(y0, y1), zlo[qb]);
                    break;
                case 3:
                    den[qb] += e0;
                    if constexpr (pp >= 0) lp.x = (_Float16)__builtin_fmaf((float)h0, neg1, f0);
                    break;
                case 4:
                    den[qb] += e1;
                    if constexpr (pp >= 0) {
                        lp.y = (_Float16)__builtin_fmaf((float)h1, neg1, f1);
                        wn.lo[pqb][pj] = __builtin_bit_cast(unsigned, lp);
                    }
                    break;
                default: {
                    const f16x2 h = __builtin_bit_cast(f16x2, __builtin_amdgcn_cvt_pkrtz(e0, e1));
                    h0 = h.x; h1 = h.y;
                    hp = __builtin_bit_cast(unsigned, h);
                    wn.hi[qb][j] = hp;
                    f0 = e0; f1 = e1;
                    if constexpr (pr == 7) {
                        lp.x = (_Float16)__builtin_fmaf((float)h0, neg1, f0);
                        lp.y = (_Float16)__builtin_fmaf((float)h1, neg1, f1);
                        wn.lo[qb][j] = __builtin_bit_cast(unsigned, lp);
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        next_iteration();
    };

    f32x4 scA[kQB][2], scB[kQB][2];
    Weights wA, wB;
    f16x8 av[8];
    wait_fetches<SPLIT ? 4 : 10>();                           // K tiles 0 and 1 (SPLIT: 0 to 3)
    workgroup_barrier();
    if (mine > 0) {
        // (step 1's scores also where there is no such step: they run under the weights of step 0)
        tw.scores(lds, 0, scB);
        tw.scores(lds, place(1), scA);
    }
    if constexpr (SPLIT) {                                    // step 2's K tiles where step 0's were
        workgroup_barrier();
        const u32x4 k2 = tw.k_window(4);
        tw.fetch_k<true>(lds, k2, 0, 0); tw.fetch_k<true>(lds, k2, 1, 1);
    }
    if (mine > 0) first_weights(mine == 1, scB, wA);
    all_landed();                                             // V tiles 0 to 2, K tiles 2 and 3; Q^T on every path
    workgroup_barrier();
    int s = 0;
    if (mine > 2) {
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) av[dt] = tw.read_v(lds, 0, dt);
        wait_reads();                                         // (SPLIT: every iteration reads them itself)
        // four at a time, left after any of them: places in the ring and registers are then fixed (nothing is computed, nothing is
        // moved; up to three iterations of a loop of their own took 1740 cycles each, these 1300.  Whole call, with those / this:
        // 2 x 28/4 heads x 700 tokens 21.6 / 21.1 us, 8 ragged prompts of up to 900 32.4 / 31.6, 1 x 32 x 512 15.2 / 14.9)
        constexpr std::false_type inner;
        const int end = mine - 2;
#pragma unroll 1
        for (; SPLIT;) {
            iteration(inner, 0, tw.k_window(2 * (s + 3)), tw.v_window(2 * (s + 1)), 0, scA, scB, wA, wB, av);
            if (s + 1 == end) break;
            iteration(inner, 2, tw.k_window(2 * (s + 4)), tw.v_window(2 * (s + 2)), 1, scB, scA, wB, wA, av);
            s += 2;
            if (s == end) break;
        }
#pragma unroll 1
        for (; !SPLIT;) {
            const u32x4 rk = tw.k_window(s + 4), rv = tw.v_window(s + 3);
            iteration(inner, 0, rk, rv, 0, scA, scB, wA, wB, av);
            if (s + 1 == end) break;
            iteration(inner, 1, rk, rv, 1, scB, scA, wB, wA, av);
            if (s + 2 == end) break;
            iteration(inner, 2, rk, rv, 2, scA, scB, wA, wB, av);
            if (s + 3 == end) break;
            iteration(inner, 3, rk, rv, 3, scB, scA, wB, wA, av);
            s += kRing;
            if (s == end) break;
        }
        s = end;
        if (s & 1) {
#pragma unroll
            for (int qb = 0; qb < kQB; ++qb) {
#pragma unroll
                for (int t = 0; t < 2; ++t) scA[qb][t] = scB[qb][t];
                wA.hi[qb] = wB.hi[qb];
                wA.lo[qb] = wB.lo[qb];
            }
        }
    }
    // The last two steps of the wavefront, then the fetches and barriers of the steps that only later wavefronts have.
    // (The first of the two is woven like the loop's, with its V operands read at the start.  P.V and masked weights one after the other,
    // V one operand ahead, took 2000 to 2500 cycles, this 1450.  With the stores through LDS and the first two steps' scores
    // together before the first weights (2400 cycles, now 1660), whole call before / now: 4 ragged prompts of up to 1024 tokens 55.5 /
    // 52.0 us, 1 x 32 heads x 100 8.9 / 7.6, 1 x 32 x 1024 27.2 / 25.7, 2 x 64/8 x 4001 560 / 550, 1 x 32 x 8192 663 / 658.)
    if (mine > 1) {                                           // s == mine - 2
        if constexpr (SPLIT) iteration(std::true_type{}, place(s), tw.k_window(2 * (s + 3)), tw.v_window(2 * (s + 1)), s & 1, scA, scB, wA, wB, av);
        else iteration(std::true_type{}, s & (kRing - 1), tw.k_window(s + 4), tw.v_window(s + 3), 0, scA, scB, wA, wB, av);
#pragma unroll
        for (int qb = 0; qb < kQB; ++qb) { wA.hi[qb] = wB.hi[qb]; wA.lo[qb] = wB.lo[qb]; }
        ++s;
    }
    if (mine > 0) {                                           // s == mine - 1
        fetch_ahead(s);
        add_pv(tw, lds, place(s), wA, acc);
        next_iteration();
        ++s;
    }
    for (; s < tw.nsteps; ++s) {
        fetch_ahead(s);
        next_iteration();
    }
    wait_fetches<0>();                                        // nothing may land in LDS after this tile

    // the four lane groups of a query hold disjoint keys: total per query
#pragma unroll
    for (int qb = 0; qb < kQB; ++qb) {
        den[qb] = query_sum(den[qb]);
    }
    // strict guard on x - phi (the extremes carry the query's scale exponent); a NaN logit, which
    // minimum and maximum skip, shows as a NaN denominator.  Apart from the guard: a weight at or
    // beyond 2^kOverflowLog2 does not fit the fp16 operands.
    bool bad = false, range = false;
#pragma unroll
    for (int qb = 0; qb < kQB; ++qb) {
        const bool live = tw.w0 + 16 * qb + n < S;
        bad |= live & ((zhi[qb] >= hi2 + kq[qb]) | (zlo[qb] <= lo2 + kq[qb]) | (den[qb] != den[qb]));
        range |= live & (zhi[qb] >= kOverflowLog2);
    }
    const unsigned long long any_bad = __ballot(bad), any_range = __ballot(range);
    if (lane == 0) { lds.bad[wave] = any_bad != 0ull; lds.redo[wave] = (any_bad | any_range) != 0ull; }
    // SPLIT: the odd wavefront's sums, through 16 KiB of the rings (out of use since the last barrier, which all fetches were waited for at)
    f32x4 *half_acc = reinterpret_cast<f32x4 *>(&lds.k[0][0] + (wave >> 1) * 16384) + lane;
    float *half_den = reinterpret_cast<float *>(&lds.v[0][0]) + (wave >> 1) * 256 + lane;
    if constexpr (SPLIT) {
        static_assert(2 * 16384 <= sizeof(lds.k));
        if (wave & 1) {
#pragma unroll
            for (int dt = 0; dt < 8; ++dt)
#pragma unroll
                for (int qb = 0; qb < kQB; ++qb) half_acc[64 * (kQB * dt + qb)] = acc[dt][qb];
#pragma unroll
            for (int qb = 0; qb < kQB; ++qb) { half_den[64 * qb] = den[qb]; half_den[64 * (kQB + qb)] = kq[qb]; }
        }
    }
    __syncthreads();
    // one flag byte per 64 queries
    constexpr int kFlagTiles = SPLIT ? 1 : kQTile / 64, kWavesPerFlag = 4 / kFlagTiles;
    if (tid < kFlagTiles) {
        const int t64 = i0 / 64 + tid;
        int f = 0;
#pragma unroll
        for (int w = 0; w < kWavesPerFlag; ++w) f |= lds.bad[tid * kWavesPerFlag + w];
        if ((unsigned)t64 < (unsigned)p.tiles) p.tile_flags[((size_t)b * p.Hq + hq) * p.tiles + t64] = f != 0;
    }
    if ((lds.redo[0] | lds.redo[1] | lds.redo[2] | lds.redo[3]) != 0) return true;   // uniform: the tile is redone, nothing stored
    if constexpr (SPLIT) {
        if (wave & 1) return false;
#pragma unroll
        for (int qb = 0; qb < kQB; ++qb) {
            // both to the smaller of the two scales (that of the larger logit); an odd wavefront without a key the query sees has none
            const float d1 = half_den[64 * qb], k1 = half_den[64 * (kQB + qb)];
            const float k = d1 == 0.f ? kq[qb] : fminf(kq[qb], k1);
            const float f0 = __builtin_amdgcn_exp2f(k - kq[qb]), f1 = d1 == 0.f ? 0.f : __builtin_amdgcn_exp2f(k - k1);
            den[qb] = __builtin_fmaf(d1, f1, den[qb] * f0);
#pragma unroll
            for (int dt = 0; dt < 8; ++dt) {
                const f32x4 o = half_acc[64 * (kQB * dt + qb)];
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[dt][qb][e] = __builtin_fmaf(o[e], f1, acc[dt][qb][e] * f0);
            }
        }
        wait_reads();
    }
    store_rows(p, tw, lds, b, hq, S, acc, den, p.Smax);
    return false;
}

// The same tile by the synchronized scheme (running maximum per query, Eq. 2); rare, so plain: one step after the
// other, one barrier per step, the next step's tiles in flight meanwhile.
__device__ __forceinline__ void tile_sync(const PrefillProblem &p, PrefillLds &lds, int b, int hq, int i0, int S, int end)
{
    const TileWave tw(p, b, hq, i0, S);
    const float c1 = p.scale * kLog2e, c0 = -p.phi * kLog2e;
    float neg1;
    asm("v_mov_b32 %0, -1.0" : "=v"(neg1));
    f32x4 acc[8][kQB];
#pragma unroll
    for (int dt = 0; dt < 8; ++dt)
#pragma unroll
        for (int qb = 0; qb < kQB; ++qb) acc[dt][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
    float den[kQB], mrun[kQB];
#pragma unroll
    for (int qb = 0; qb < kQB; ++qb) { den[qb] = 0.f; mrun[qb] = -INFINITY; }
    tw.fetch_k(lds, 0);
    tw.fetch_v(lds, 0);
    all_landed();                                             // (Q^T too: no wait for it under the loop's fetches)
    __syncthreads();
#pragma unroll 1
    for (int s = 0; s < tw.nsteps; ++s) {
        tw.fetch_k(lds, s + 1);                                // their places were last read in step s - 3
        tw.fetch_v(lds, s + 1);
        if (s < tw.mine) {                                    // uniform over the wavefront
            f32x4 sc[kQB][2];
            tw.scores(lds, s & (kRing - 1), sc);
            Weights w;
#pragma unroll
            for (int qb = 0; qb < kQB; ++qb) {
                const int qrow = tw.w0 + 16 * qb + tw.n;
                float z[8];
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    z[j] = s * kStep + 8 * tw.g + j <= qrow ? __builtin_fmaf(sc[qb][j >> 2][j & 3], c1, c0) : -INFINITY;
                float m = fmaxf(fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3])), fmaxf(fmaxf(z[4], z[5]), fmaxf(z[6], z[7])));
                m = query_max(m);
                const float mnew = fmaxf(mrun[qb], m);
                if (mnew > mrun[qb]) {                        // rescale what was summed so far
                    const float alpha = mrun[qb] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mrun[qb] - mnew);
#pragma unroll
                    for (int dt = 0; dt < 8; ++dt) acc[dt][qb] *= alpha;
                    den[qb] *= alpha;
                    mrun[qb] = mnew;
                }
                const float shift = mnew == -INFINITY ? 0.f : mnew;
#pragma unroll
                for (int j = 0; j < 8; j += 2) {
                    const float e0 = __builtin_amdgcn_exp2f(z[j] - shift), e1 = __builtin_amdgcn_exp2f(z[j + 1] - shift);
                    den[qb] += e0 + e1;
                    unsigned h, l;
                    split_pair(e0, e1, neg1, h, l);
                    w.hi[qb][j >> 1] = h;
                    w.lo[qb][j >> 1] = l;
                }
            }
            add_pv(tw, lds, s & (kRing - 1), w, acc);
        }
        wait_fetches<0>();
        __syncthreads();
    }
#pragma unroll
    for (int qb = 0; qb < kQB; ++qb) {
        den[qb] = query_sum(den[qb]);
    }
    store_rows(p, tw, lds, b, hq, S, acc, den, end);
}

// Which tile of the order below workgroup i of `grid` runs: a permutation that keeps i % 8.
__device__ __forceinline__ int tile_order(int i, int grid)
{
    if (i < kComputeUnits || grid > 2 * kComputeUnits || grid % 8 != 0) return i;
    return kComputeUnits + grid - 8 - (i & ~7) + (i & 7);
}

template <bool SPLIT>
__global__ __launch_bounds__(256, 2) void prefill_kernel(const PrefillProblem p)
{
    constexpr int kTile = SPLIT ? kQTile / 2 : kQTile;             // queries per workgroup
    __shared__ PrefillLds lds;
    // Order: heavy tiles (late queries see more keys) of all heads first, so that what runs last is short.
    // Workgroups are dealt to the 8 XCDs round-robin by index; each XCD has its own L2.  Where the KV heads divide by 8,
    // the query heads that share one go to the same XCD (kv head % 8), so that an XCD streams an eighth of K and V;
    // otherwise that would leave XCDs with less work or none, and the tiles go round-robin as they come.
    // (One head after the other, heavy first within a head, the last head's heavy tiles ran alone at the end.  Whole call,
    // that order / this: 4 ragged prompts of up to 1024 tokens 79.2 / 68.6 us, 2 x 64/8 heads x 4001 623.1 / 578.9, 1 x 32 x
    // 8192 753.5 / 695.7.)
    const int heads = p.B * p.Hq, kv_heads = p.B * p.Hkv;
    const int qtiles = (p.Smax + kTile - 1) / kTile;
    // A launch of one to two tiles per compute unit: a compute unit holds workgroups i and i + 256 from the start, so the second
    // half runs light tiles first and the heaviest shares its compute unit with the lightest (the XCD stays the same).  Whole call,
    // without / with: 1 x 32 heads x 2048 tokens 60.7 / 55.5 us, 1 x 16 x 4096 107.0 / 96.8, 2 x 32 x 1024 37.7 / 35.4,
    // 1 x 32 x 1100 28.8 / 28.7.
    const int item = tile_order(blockIdx.x, gridDim.x);
    int first = 0, left = item, size = heads;                    // the heads whose tiles are dealt out together (see head_group)
    if (p.group < heads) {
        const int part = min(item / (p.group * qtiles), p.parts - 1);
        first = part * p.group;
        left = item - first * qtiles;
        size = part == p.parts - 1 ? heads - first : p.group;
    }
    const int rank = left / size;                                // 0: the last tile of every head
    const int u = first + left - rank * size;
    int head = u;
    if (kv_heads % 8 == 0) {                                      // u % 8 == item % 8 == blockIdx.x % 8
        const int m = u >> 3;
        head = ((u & 7) + 8 * (m / p.G)) * p.G + m % p.G;
    }
    const int qt = qtiles - 1 - rank;
    const int b = head / p.Hq, hq = head - b * p.Hq;
    const int i0 = qt * kTile - p.shift;
    int S = p.seq_lens[b];
    // (uniform, as the compiler has to see: else the loop's counters end up in vector registers, 0.4 % of 8192 tokens)
    S = __builtin_amdgcn_readfirstlane(S < 0 ? 0 : (S > p.Smax ? p.Smax : S));
    if (i0 >= S) {                                       // no prompt token in this tile: zeros, no flag
        const int at = max(i0, 0);
        uint16_t *o = p.out + (((size_t)b * p.Hq + hq) * p.Smax + at) * kHeadDim;
        const int rows = min(i0 + kTile, p.Smax) - at;
        for (int i = threadIdx.x; i < rows * (kHeadDim / 8); i += 256)
            reinterpret_cast<u32x4 *>(o)[i] = u32x4{0u, 0u, 0u, 0u};
        const int t64 = i0 / 64 + (int)threadIdx.x;
        if (threadIdx.x < kTile / 64 && (unsigned)t64 < (unsigned)p.tiles) p.tile_flags[((size_t)b * p.Hq + hq) * p.tiles + t64] = 0;
        return;
    }
    if (tile_unified<SPLIT>(p, lds, b, hq, i0, S)) {            // Section 3 "Recomputation", for this tile
        __syncthreads();
        tile_sync(p, lds, b, hq, i0, S, min(p.Smax, i0 + kTile));
    }
}

}  // namespace

// Heads whose tiles are dealt out together, heaviest first, before those of the next: all of them, except in launches of many heads that share
// nothing.  There the tiles in flight at a time are one or two of every head, each streams K and V past the L2s for itself, and the
// launch draws 5 TB/s from the memory behind them.  In groups of half a round of the chip the tiles of a head run together and find its keys in
// their XCD's L2; the last group, of two rounds and more, evens out what is left.  Whole call, all heads / groups: 8 x 40 heads x 1280 tokens 226.5 /
// 208.0 us, 7 x 40 x 667 .. 2003 261 / 251, 7 x 32 x 328 .. 984 67.6 / 65.8; groups of a round, without the large last one 216, 269, 73.  Fewer heads lose what the
// group ends cost: 4 x 32 x 1024 61.0 / 61.2, 8 x 16 x 2808 347.7 / 350.1, 2 x 40 x 4000 426 / 430, 1 x 32 x 8192 648 / 662, 8 x 32/8 x 498 .. 1496 133 / 136, 2 x 64/8 x
// 4001 583 / 602.
static void head_group(PrefillProblem &p, int qtiles)
{
    const int heads = p.B * p.Hq;
    const long long tiles = (long long)heads * qtiles;
    p.group = heads;
    p.parts = 1;
    if ((long long)p.B * p.Hkv < 192 || tiles < 5 * kComputeUnits) return;
    p.group = (kComputeUnits / qtiles + 7) / 8 * 8;              // (a multiple of 8: a head's tiles stay on one XCD)
    if (p.group == 0) p.group = 8;
    p.parts = (int)((tiles - 4 * kComputeUnits) / ((long long)p.group * qtiles)) + 1;
    if (p.parts == 1) p.group = heads;
}

hipError_t launch_prefill(const PrefillProblem &p0, hipStream_t s)
{
    if (p0.B == 0) return hipSuccess;
    PrefillProblem p = p0;
    const int qtiles = (p.Smax + kQTile - 1) / kQTile;
    const long long tiles = (long long)p.B * p.Hq * qtiles;
    // Launches that would leave compute units with one workgroup or none: tiles of 64 queries, walked by twice the wavefronts (see
    // tile_unified).  Whole call, without / with: 1 x 32 heads x 256 tokens 10.0 / 8.7 us, 512 14.6 / 11.7, 1024 24.0 / 20.4, 1 x 16 x 2000 38.9 /
    // 31.8, 2 x 28/4 x 500 15.8 / 14.0.  What bounds short prompts is a tile's beginning and end, of which there are more then.  Up to 96 tokens a tile
    // as it comes has at most three wavefronts at work and 64 queries gain nothing (1 x 32 x 64 5.8 / 6.6, 16 x 12/2 x 64 6.4 / 7.1, 1 x 32 x 88 6.74 /
    // 6.74, 100 7.4 / 6.9); heads of one or two tiles of 128 need a compute unit for each of 64 (64 heads x 217 tokens, 256 of them, 9.3 / 8.5, 128 x 100, 256,
    // 7.7 / 7.3; 160 x 100, 320, 7.9 / 9.1, 96 x 217, 384, 9.7 / 10.7), and heads of three 192 tiles or a last one with all four wavefronts
    // at work (64 x 280, 192, 10.7 / 10.4, 80 x 384, 240, 13.5 / 12.6; 80 x 290, 240, 11.3 / 11.6).  A few tiles more than compute units where a head has
    // more than four, of unequal length
    // (1 x 32 x 1152, 288 tiles, 27.6 / 24.0, 1 x 28/4 x 1260, 280, 29.2 / 25.1).  With more the keys' second
    // reading costs more than the shorter walk gives: 2 x 28/4 x 650, 336 tiles, 19.1 / 22.8, 1 x 32 x 1536, 384, 37.2 / 40.1, 2 x 32 x 1024, 512, 31.7 / 37.9.
    const int halves = (p.Smax + kQTile / 2 - 1) / (kQTile / 2);               // tiles of 64 queries of a head
    const int over = p.Smax % kQTile;                                          // queries of the last tile as they come (0: all)
    const bool last_busy = over == 0 || over > 3 * kWaveQ;
    const bool split = qtiles > 4    ? tiles <= kComputeUnits + kComputeUnits / 8
                       : qtiles == 4 ? tiles <= kComputeUnits
                       : qtiles == 3 ? tiles <= (last_busy ? kComputeUnits : 3 * kComputeUnits / 4)
                                     : p.Smax > 3 * kWaveQ && (long long)p.B * p.Hq * halves <= kComputeUnits;
    if (split) {
        p.group = p.B * p.Hq;
        p.parts = 1;
        p.shift = 0;
        return launch(prefill_kernel<true>, dim3((unsigned)(p.group * halves)), dim3(256), s, p);
    }
    head_group(p, qtiles);
    // Tiles end at a multiple of 128 queries, or of 64 where that leaves the last one of a prompt as long as the buffer at least half
    // full: it sees all keys, and with its queries as they come one or two wavefronts would walk them by themselves.  The first tile then starts 64 in
    // front of the prompt and its first two wavefronts have nothing to do; there are as many tiles as without.  Whole call, without / with: 8 x 40
    // heads x 1284 tokens 233.9 / 218.7 us, 4 x 32 x 1030 67.2 / 64.8, 8 x 64/8 x 400 57.0 / 55.5, 1 x 32 x 4100 175.2 / 173.2.  A launch of up to two
    // tiles per compute unit ends with its longest tile, and one of short prompts has little else: both take longer over a last tile with four wavefronts
    // at work than with two, and shift for one only (2 x 28/4 x 650, 336 tiles, one wavefront, 20.5 / 19.6; 8 x 32 x 300, two, 25.1 / 27.2).
    const int most = tiles > 2 * kComputeUnits && qtiles > 4 ? 2 * kWaveQ : kWaveQ;
    p.shift = over > 0 && over <= most ? 64 : 0;
    return launch(prefill_kernel<false>, dim3((unsigned)tiles), dim3(256), s, p);
}

}  // namespace fd

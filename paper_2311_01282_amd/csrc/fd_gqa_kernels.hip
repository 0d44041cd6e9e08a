// Grouped-query chunk kernel (MFMA path): the G <= 16 query heads that share one
// KV head are processed together, so every K and V element is read from HBM once
// per group instead of once per query head.  With G = 8 the work is 8 flop per KV
// byte, more than the vector ALUs sustain at HBM rate once fp16->fp32 conversions
// are counted, hence the matrix cores:
//
//   scores   S^T[key][head] = sum_d K[key][d] Q[head][d]
//            v_mfma_f32_16x16x32_f16: A = a 16-key block of K, B = Q padded to 16
//            heads (zero rows), 4 instructions per block (d = 4 x 32).
//   weights  P = e^{s S^T - phi} in fp32, in place in the accumulator layout
//            (lane (head, g) holds keys g, 4+g, 8+g, 12+g of the block) -- Eq. 4, no maximum.
//            fp16 has neither the range of e^{x-phi} over the admissible x - phi nor, with 11
//            bits, the precision, so P goes to the matrix cores as fp16 hi + lo pairs (22 bits)
//            under a scale 2^k of the (wavefront, head)'s own: k, an integer, is fixed after the
//            wavefront's first 16-key block so that the head's largest weight there lies in
//            [2^3, 2^4]; it is constant over the keys the wavefront sums, so the sums of Eq. 4 stay
//            plain sums, and it is taken out again (exactly: a power of two) before the
//            wavefronts' tiles are added.  V is fp16 and is used as it is:
//   P.V      out[head][d] += sum_key P[head][key] V[key][d]
//            v_mfma_f32_16x16x16_f16, two per tile (P_hi V + P_lo V): A = P, whose four weights
//            per lane are exactly contraction indices 4g..4g+3 when index 4g + r stands for key
//            4r + g; B = V, where lane (n, g) loads the 16 bytes d = 8n..8n+7 of the same keys
//            4r + g (r = 0..3) and feeds element e of the four rows to accumulator tile e (d = 8n
//            + e), so V needs no transpose, only a byte permute per pair of rows: 16 matrix
//            instructions per 16-key block.  (Earlier forms: fp32 16x16x4, 32 instructions of 16
//            passes; then bf16 with P in three and V in two pieces, 40 instructions and about 4
//            vector-ALU operations per V element for the split.)
//            A weight at or beyond 2^15.9 -- a logit more than 8 above the largest of the
//            wavefront's first block -- does not fit: that (head, chunk) is redone on the per-row
//            path like a flagged one, but without the flag.
//
// K reaches the A layout through a per-wavefront LDS tile (coalesced 1 KiB global
// loads in, 16-byte reads out, XOR-swizzled so both directions are bank-conflict
// free).  One workgroup = 4 wavefronts = one (sequence, KV head, chunk); the
// wavefronts interleave 16-key blocks.  The rest of the method -- guard, on-the-spot
// recomputation of a flagged (head, chunk) with the synchronized scheme, election of
// the workgroup that completes the group, row epilogue -- is shared with the per-row
// kernels (fd_chunk.h).
#include "fd_chunk.h"

namespace fd {
namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// NW wavefronts per workgroup (4 or 8; the launcher uses 4).
template <int NW>
struct GqaLds {
    // K staging (NW wavefronts x 4 KiB) during the main loop, then the reduction tile
    // [wave][head][d] (NW x 8 KiB), then (rarely) the per-row recomputation's workspace:
    // never live together.
    alignas(16) float tile[NW * 16 * kHeadDim];
    alignas(16) float den[16][NW];   // per head: the wavefronts' denominators ...
    alignas(16) float inv[16][NW];   // ... and what takes their scales out of their tiles again (SYNC: the references ...
    alignas(16) float top[16][NW];   // ... and the wavefronts' largest logits)
    alignas(16) unsigned mask[NW];   // heads out of bounds, and << 16 heads with a weight beyond the fp16 operand
    float e_new[16];                 // weight of an appended key per head (written where there is one)
    int last;
};

typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr float kFirstBlockLog2 = 4.f;    // a head's largest weight of the wavefront's first block lies in [2^3, 2^4] ...
constexpr float kOverflowLog2 = 15.9f;    // ... and no later weight may reach 2^16 (fp16 ends at 65504)
// SYNC: the weight of a logit that equals the reference, and how far above it a logit raises the reference (2^10 e^4 is under 2^15.9).  High, so
// that the smallest fp16 numbers lie 2^-34 below it: sums lose nothing there that fp32 would keep.  A factor of its own, not an
// addition in the exponent, whose rounding error would grow with it.
constexpr float kSyncScale = 1024.f, kHeadroom = 4.f;

// Order by length (launches of more than one workgroup per compute unit, at most 64 sequences; see GqaLauncher): the chunks
// that are full first, then the sequences' last, partial chunks from the longest to the shortest, then the chunks without keys; each for
// all KV heads.  Every workgroup of up to three rounds of the chip starts with the launch and a compute unit holds workgroups i, i + 256, ...,
// so what it has to stream is decided here.
//   Up to 256 full chunks: the first 256 go in reverse, and the shortest of them share their compute units with the longest of
// the rest.
//   More: some compute units take a full chunk more than others in any order, and as a compute unit draws 38 bytes a nanosecond at most they
// end late while the rest has nothing left to do (first in reverse, 48 with two chunks beside 160 with one).  But fewer than all saturate
// the memory: the live chunks are dealt to as many compute units as take the same number each, the others get what has no keys.  General
// order / first in reverse / this: 8 x 64/8 heads x 2725 .. 21800 keys (352 live chunks, 288 full) 80.0 / 88.1 / 77.1 us, 16 x 12/2 x 6427 .. 51420
// (334, 302) 101 / 105.7 / 91.6, 19 x 12/2 x 26865 .. 53731 (566, 528) 139.3 / 143.6 / 126.8, 12 x 32/8 x 300 .. 6000 39.4 / 40.1 / 37.3, 7 x 64/8 x
// 1041 .. 8335 33.8 / 34.2 / 31.1.  Beyond three rounds workgroups wait for others to end, wherever that is, and nothing is dealt (28 x 16/8 x 87 ..
// 696, 920 full chunks, in reverse / dealt 15.6 / 16.0); nor are chunks of less than 256 keys, too short to be bound by what a compute unit
// draws (of 160 22 x 32/8 x 79 .. 632 10.85 / 11.0, of 224 18 x 32/8 x 138 .. 1104 13.3 / 13.5, of 288 9 x 64/8 x 990 .. 1980 15.7 / 15.6); nor where the partial chunks make a round of their own (22 x 28/4 x 12577 .. 25155, 512 full and 88:
// 155.1 / 157.8).
// `res`: resident keys of sequence `lane` (p.B <= 64).
// Returns false for a workgroup beyond the last chunk; else sequence, chunk and KV head.
__device__ __forceinline__ bool chunk_by_length(const Problem &p, int res, int &b, int &c, int &hkv)
{
    const int lane = threadIdx.x & 63;
    int full = 0, rest = 0, empty = 0;
    if (lane < p.B) {
        const int len = effective_len(p, res);
        full = (int)((float)len * __builtin_amdgcn_rcpf((float)p.C));      // the quotient, or one off
        full -= full * p.C > len;
        full += len - full * p.C >= p.C;
        rest = len - full * p.C;
        empty = p.nc - full - (rest > 0);
    }
    const int scan = lanes_scan(full);
    const unsigned long long parts = __ballot(rest > 0);
    const int n_full = __builtin_amdgcn_readlane(scan, 63), n_part = __popcll(parts);
    const int live = (n_full + n_part) * p.Hkv;
    int i = blockIdx.x;
    const int fulls = n_full * p.Hkv;
    bool dealt = false;
    if (fulls > kComputeUnits && fulls <= 3 * kComputeUnits && p.C >= 256) {
        const int rounds = (fulls + kComputeUnits - 1) / kComputeUnits;
        // live / rounds rounded up (exact, as below), to the same number of compute units of each XCD
        const int used = ((int)(((float)(live + rounds - 1) + 0.5f) * __builtin_amdgcn_rcpf((float)rounds)) + 7) & ~7;
        const int last = kComputeUnits * (rounds - 1);                     // first workgroup of the last round
        dealt = used < kComputeUnits && last + used <= 8 * ((p.B * p.Hkv + 7) >> 3) * p.nc;
        if (dealt && i < last + kComputeUnits) {                           // (a permutation: the rest of each round takes what is left)
            const int k = i / kComputeUnits, j = i % kComputeUnits;
            i = j < used ? k * used + j : used * rounds + k * (kComputeUnits - used) + (j - used);
        }
    }
    if (!dealt && live > kComputeUnits && i < kComputeUnits) i = kComputeUnits - 1 - i;
    int q = (int)(((float)i + 0.5f) * __builtin_amdgcn_rcpf((float)p.Hkv));   // i / Hkv: exact, i < 2^20
    const int h = i - q * p.Hkv;
    if (q < n_full) {
        b = __popcll(__ballot(scan <= q));
        c = q - (__builtin_amdgcn_readlane(scan, b) - __builtin_amdgcn_readlane(full, b));
    } else if (q < n_full + n_part) {
        // the q-th longest, lengths taken in 64 steps of a chunk: the step it is in, six halvings; in that step by sequence
        q -= n_full;
        const int step = rest > 0 ? (int)((float)rest * (64.f * __builtin_amdgcn_rcpf((float)p.C))) : -1;
        int at = 0;
#pragma unroll
        for (int bit = 32; bit > 0; bit >>= 1) at += __popcll(__ballot(step >= at + bit)) > q ? bit : 0;
        q -= __popcll(__ballot(step > at));
        const unsigned long long same = __ballot(step == at);
        const int before = __builtin_amdgcn_mbcnt_hi((unsigned)(same >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)same, 0u));
        b = __ffsll((unsigned long long)__ballot((step == at) & (before == q))) - 1;
        c = __builtin_amdgcn_readlane(full, b);
    } else {
        q -= n_full + n_part;
        const int escan = lanes_scan(empty);
        b = __popcll(__ballot(escan <= q));
        if (b >= p.B) return false;
        c = p.nc - (__builtin_amdgcn_readlane(escan, b) - q);
    }
    hkv = h + min(c & 7, p.Hkv - 1);           // turned by the chunk: an XCD does not stay with one head
    hkv -= hkv >= p.Hkv ? p.Hkv : 0;
    return true;
}

// kEarly: the first loads go out before the sequence length has arrived (launches of at most one workgroup per compute unit,
// contiguous cache; see decode_fused_kernel); kByLength: chunk_by_length.
enum Start { kPlain, kEarly, kByLength };

// SYNC: the chunk's part of the synchronized partial softmax (Eq. 2; fd_decode_attn_sync) by the same tile: m = max x, l = sum
// e^{x-m}, f.V = sum e^{x-m} v, no guard, no flag.  A (wavefront, head) has a reference in place of the running maximum: the largest logit of the
// first block, and where a later one lies more than kHeadroom above it the reference becomes that and the sums are brought to it; m itself enters
// at the workgroup reduction.  It is taken off the rounded logit before anything is multiplied: in a difference of products rounded one by
// one, logits from 1e8 on would lose the scale.  Bound by HBM reads like the rest; the check is a compare and a branch per 16 keys.  The per-row form
// read K and V once per query head, out of the caches where they held them: whole call, that / this, 5 x 28/4 heads x 14729 keys 107.0 / 28.8
// us, 12 x 12/2 x 7924 79.4 / 20.0, 2 x 64/8 x 1000 10.5 / 8.35.
template <int C, bool PAGED, Start START, bool SYNC = false, int NW = 4>
__global__ __launch_bounds__(NW * 64, NW == 4 ? 3 : 1) void decode_fused_gqa_kernel(const Problem p)
{
    static_assert(NW == 4 || NW == 8, "the appended key's lane assignment covers 16 heads with 4 wavefronts");
    static_assert(sizeof(ChunkLds<NW>) <= sizeof(GqaLds<NW>::tile), "recompute workspace must fit the tile");
    constexpr int kGqaThreads = NW * 64;
    constexpr int UP = SYNC ? (C < 256 ? 1 : 2) : C / (4 * NW) < 4 ? C / (4 * NW) : 4;    // stage depth of the per-row recomputation (no register spilled)
    __shared__ GqaLds<NW> lds;
    constexpr int NBLK = C / 16;               // 16-key blocks in the chunk
    static_assert(!(PAGED && START == kEarly), "the page table has to arrive before the first load");
    static_assert(!(PAGED && SYNC), "the synchronized entry point takes contiguous caches");
    constexpr bool EARLY = START == kEarly, BY_LENGTH = START == kByLength;
    fetch_arguments_now(p);
    asm volatile("" ::"s"(p.B), "s"(p.C), "s"(p.scatter), "s"(p.chunk_major));
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = lane & 15, g = lane >> 4;    // n: head (scores) / 16-byte segment (loads); g: lane group
    const int G = p.G;

    int b, c, gi;                              // sequence, chunk, (sequence, KV head)
    const int groups = p.B * p.Hkv, groups8 = (groups + 7) >> 3;
    int res = 0;
    bool by_length = BY_LENGTH;
    if constexpr (BY_LENGTH) {
        if (lane < p.B) res = clamp_len(p, p.seq_lens[lane]);
        // equal lengths have nothing to sort, unless the rows do not divide among the XCDs
        by_length = __ballot((lane < p.B) & (res != __builtin_amdgcn_readfirstlane(res))) != 0ull || groups8 * 8 != groups;
    }
    if (by_length) {
        int hkv;
        if (!chunk_by_length(p, res, b, c, hkv)) return;
        gi = b * p.Hkv + hkv;
    } else {
        // All chunks of a KV-head group go to the same XCD, or in turn to all (row_slot); chunk-major in a launch of up
        // to 1024 workgroups, so that chunks past the end of the sequences come last; row-major beyond.
        const int j = blockIdx.x >> 3;
        const bool cm = p.chunk_major != 0;
        c = cm ? j / groups8 : j % p.nc;
        gi = row_slot(p, blockIdx.x & 7, c) + 8 * (cm ? j - c * groups8 : j / p.nc);
        if (gi >= groups) return;
        b = gi / p.Hkv;
    }
    const int row0 = b * p.Hq + (gi - b * p.Hkv) * G;       // first query row of the group
    int raw = 0;
    if constexpr (EARLY) raw = seq_len_issue(p, b);
    const int len = p.C;                                    // keys per chunk (<= C, the kernel's capacity)
    const int start = c * len;

    // Q as the B operand: lane (n, g) holds d = 32kb + 8g .. +7 of head n; heads >= G are zero rows.
    u32x4 qr[4];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
        qr[kb] = *reinterpret_cast<const u32x4 *>(p.q + (size_t)(row0 + min(n, G - 1)) * kHeadDim + 32 * kb + 8 * g);

    const KvRows<PAGED> at(p, b, gi - b * p.Hkv, start, lane);   // rows of the chunk's keys (contiguous or paged)
    const u32x4 *kp = reinterpret_cast<const u32x4 *>(p.k) + at.base + n;
    const u32x4 *vp = reinterpret_cast<const u32x4 *>(p.v) + at.base + n;
    u32x4 kA[4], vA[4];
    if constexpr (EARLY) {                     // this wavefront's first block, clamped to the chunk's extent in the buffer
        const int cap = min(len, p.Smax - start) - 1;
#pragma unroll
        for (int r = 0; r < 4; ++r) kA[r] = load_stream(kp + at(min(16 * wave + 4 * r + g, cap)));
#pragma unroll
        for (int r = 0; r < 4; ++r) vA[r] = load_stream(vp + at(min(16 * wave + 4 * r + g, cap)));
        asm volatile("" ::: "memory");         // the loads go out before the length is awaited, whatever it decides
        __builtin_amdgcn_sched_barrier(0);
    }

    // keys resident in the cache
    const int S_res = EARLY ? seq_len_finish(p, raw) : BY_LENGTH ? __builtin_amdgcn_readlane(res, b) : clamp_len(p, p.seq_lens[b]);
    const int S = effective_len(p, S_res);                  // plus the appended one, if any
    const int nb = (S + len - 1) / len;
    const int nvalid = min(len, S - start);
    const int nres = min(len, S_res - start);
    const bool owner = !SYNC & (S != S_res) & (S_res >= start) & (S_res < start + len);   // this chunk takes the appended key

    if (!EARLY && nvalid <= 0) {               // padding chunk: zero partials, no flag (EARLY: by the ordinary path)
        for (int i = tid; i < G * kHeadDim; i += kGqaThreads)
            p.ws.num[((size_t)(row0 + i / kHeadDim) * p.nc + c) * kHeadDim + (i & (kHeadDim - 1))] = 0.f;
        if (tid < G) {
            const size_t slot = (size_t)(row0 + tid) * p.nc + c;
            p.ws.den[slot] = 0.f; p.ws.mloc[slot] = SYNC ? -INFINITY : p.phi;
            if (!SYNC) p.ws.chunk_flags[slot] = 0;
            store_meta(p, slot, 0.f, p.phi, 0);
            if (nb == 0 && c == 0 && p.elect) p.ws.row_flags[row0 + tid] = 0;
        }
        if (nb == 0 && c == 0 && p.elect)      // empty sequence: nobody else owns these rows
            for (int i = tid; i < G * kHeadDim; i += kGqaThreads) p.out[(size_t)row0 * kHeadDim + i] = 0;
        return;
    }

    f16x8 qb[4];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) qb[kb] = __builtin_bit_cast(f16x8, n < G ? qr[kb] : u32x4{0u, 0u, 0u, 0u});
    const int last = nres - 1;                 // last resident key; the appended one joins at the reduction
    const float nphi = -p.phi, lo = p.lo, hi = p.hi, scale = p.scale;
    u32x4 *kst = reinterpret_cast<u32x4 *>(lds.tile) + wave * 256;     // this wavefront's 16 x 16 slots

    f32x4 acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = f32x4{0.f, 0.f, 0.f, 0.f};
    float den = 0.f;
    bool bad = false;
    const bool head_on = n < G;
    float kq = 0.f;                            // scale exponent of (this wavefront, head n), set by the first block
    float ref = kNoRef;                        // SYNC: what the logits of (this wavefront, head n) are taken against
    float zmax = -INFINITY;                    // largest log2 of a scaled weight of head n so far
    float xmax = -INFINITY;                    // SYNC: largest logit of this lane's keys so far
    float neg1;                                // -1.0 the compiler cannot fold: keeps e - (float)hi one mixed-precision FMA
    asm("v_mov_b32 %0, -1.0" : "=v"(neg1));

    // Keys past the valid length re-read the last valid key and get weight zero.
    auto issue = [&](int blk, u32x4 (&kk)[4], u32x4 (&vv)[4]) {
        const int k0 = blk * 16;
        if constexpr (PAGED) {
            // the block holds a resident key (k0 <= last), so a clamped key stays inside it: one page per block
            const size_t blk0 = at.block16(k0);
#pragma unroll
            for (int r = 0; r < 4; ++r) kk[r] = load_stream(kp + blk0 + (size_t)(min(k0 + 4 * r + g, last) - k0) * 16);
#pragma unroll
            for (int r = 0; r < 4; ++r) vv[r] = load_stream(vp + blk0 + (size_t)(min(k0 + 4 * r + g, last) - k0) * 16);
            return;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) kk[r] = load_stream(kp + at(min(k0 + 4 * r + g, last)));
#pragma unroll
        for (int r = 0; r < 4; ++r) vv[r] = load_stream(vp + at(min(k0 + 4 * r + g, last)));
    };
    auto reduce = [&](int blk, bool first, const u32x4 (&kk)[4], const u32x4 (&vv)[4]) {
        const int k0 = blk * 16;
        // K block -> LDS row (4i + g), 16-byte slot n ^ row; then out in the A layout.
        // Row i of the A operand is key pk = 4(i%4) + i/4 of the block, so that score
        // register r of lane group g belongs to key 4r + g -- the key whose V row the
        // same lane group fetched with load r (1 KiB contiguous per load).
        // Swizzle key swz(r) = the two 2-bit halves of r swapped: the read of lane (n, g) then
        // lands in 16-byte unit (4 kb + g) ^ n, which is conflict-free on this chip (a 16-byte
        // LDS access serves 16 lanes a cycle, every n once, from two lane groups g; measured:
        // no conflict cycles).
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = 4 * i + g;
            kst[r * 16 + (n ^ (i | (g << 2)))] = kk[i];
        }
        const int pk = 4 * (n & 3) + (n >> 2);
        const int pswz = n;                            // swz(pk) = (pk >> 2) | ((pk & 3) << 2) = n
        f32x4 sc = {0.f, 0.f, 0.f, 0.f};
        if constexpr (SYNC) {
            // added as a tree: in a chain of four, large logits are less exact than by the per-row kernel's tree (error of logits beyond twice their
            // spread against 64 bits, relative to the spread: per-row 1.17e-7, chain 1.53e-7, this 1.07e-7)
            f32x4 part[4];
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) {
                const f16x8 ka = __builtin_bit_cast(f16x8, kst[pk * 16 + ((4 * kb + g) ^ pswz)]);
                part[kb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ka, qb[kb], sc, 0, 0, 0);
            }
            sc = (part[0] + part[1]) + (part[2] + part[3]);
        } else {
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) {
                const f16x8 ka = __builtin_bit_cast(f16x8, kst[pk * 16 + ((4 * kb + g) ^ pswz)]);
                sc = __builtin_amdgcn_mfma_f32_16x16x32_f16(ka, qb[kb], sc, 0, 0, 0);
            }
        }
        // sc[r] = <q_head n, k_key>, key = k0 + 4r + g.  Guard on x - phi, then the scaled weight.
        float dd[4];
        bool valid[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            valid[r] = k0 + 4 * r + g <= last;
            dd[r] = SYNC ? rounded_product(sc[r], scale) : sc[r] * scale + nphi;
            if constexpr (!SYNC) bad |= valid[r] & head_on & !((dd[r] > lo) & (dd[r] < hi));
        }
        if constexpr (SYNC) {
            float top = -INFINITY;
#pragma unroll
            for (int r = 0; r < 4; ++r) top = fmaxf(top, valid[r] ? dd[r] : -INFINITY);
            xmax = fmaxf(xmax, top);
            if (__ballot(top - ref > kHeadroom) != 0ull) {       // the first block; rarely another
                // the four lane groups of a head hold different keys: they agree on the new reference
                float m = fmaxf(top, __shfl_xor(top, 16));
                m = fmaxf(m, __shfl_xor(m, 32));
                const bool moves = m - ref > kHeadroom;
                const float by = moves ? __builtin_amdgcn_exp2f((ref - m) * kLog2e) : 1.f;     // 0 where there was none (the sums are zeros then)
                ref = moves ? m : ref;
                den *= by;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float f = __shfl(by, 4 * g + r);             // acc[e][r] is of head 4g + r
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[e][r] *= f;
                }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) dd[r] -= ref;
        } else if (first) {
            // the head's scale: the four lane groups of a head hold different keys and agree on the maximum first
            float m = -INFINITY;
#pragma unroll
            for (int r = 0; r < 4; ++r) m = fmaxf(m, valid[r] ? dd[r] * kLog2e : -INFINITY);
            m = fmaxf(m, __shfl_xor(m, 16));
            m = fmaxf(m, __shfl_xor(m, 32));
            kq = m > -INFINITY ? kFirstBlockLog2 - ceilf(m) : 0.f;      // (no finite logit: the guard has fired anyway)
        }
        float pw[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float z = SYNC ? dd[r] * kLog2e : __builtin_fmaf(dd[r], kLog2e, kq);
            if constexpr (!SYNC) zmax = fmaxf(zmax, valid[r] ? z : -INFINITY);
            const float e = SYNC ? __builtin_amdgcn_exp2f(z) * kSyncScale : __builtin_amdgcn_exp2f(z);
            pw[r] = valid[r] ? e : 0.f;
            den += pw[r];
        }
        // P as the A operand of the 16x16x16 product: lane (head n, g) holds contraction indices
        // 4g .. 4g+3, which stand for keys g, 4+g, 8+g, 12+g -- its own four weights.
        // hi = the weight cut to fp16, lo = what that leaves (exact in fp32) cut to fp16: 22 bits.  SYNC: both rounded to nearest, which
        // leaves an error of 2^-24 of the weight at most, as rounding to fp32 does (error of f.V against 64 bits with weights in fp32 / cut / rounded,
        // chunks of 256 keys whose weights are alike 1.20e-7 / 1.88e-7 / 1.18e-7, the cut ones all too small; spread as usual 1.68e-7 / 2.42e-7 / 1.59e-7).
        const auto halves = [](float a, float b) {
            if constexpr (SYNC) return __builtin_convertvector(f32x2{a, b}, f16x2);
            else return __builtin_bit_cast(f16x2, __builtin_amdgcn_cvt_pkrtz(a, b));
        };
        const f16x2 h01 = halves(pw[0], pw[1]), h23 = halves(pw[2], pw[3]);
        const _Float16 h0 = h01.x, h1 = h01.y, h2 = h23.x, h3 = h23.y;
        const float l0 = __builtin_fmaf((float)h0, neg1, pw[0]), l1 = __builtin_fmaf((float)h1, neg1, pw[1]);
        const float l2 = __builtin_fmaf((float)h2, neg1, pw[2]), l3 = __builtin_fmaf((float)h3, neg1, pw[3]);
        const f16x4 p_hi = __builtin_bit_cast(f16x4, make_uint2(__builtin_bit_cast(unsigned, h01), __builtin_bit_cast(unsigned, h23)));
        const f16x4 p_lo = __builtin_bit_cast(f16x4, make_uint2(__builtin_bit_cast(unsigned, halves(l0, l1)), __builtin_bit_cast(unsigned, halves(l2, l3))));
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            // dword w of the four V rows holds elements d = 8n + 2w (low halves) and 8n + 2w + 1 (high
            // halves): the B operands of accumulator tiles 2w and 2w + 1 are the low, resp. high, halves
            // of rows 0..3 (v_perm_b32: two halves of two registers into one)
            const uint32_t v0 = vv[0][w], v1 = vv[1][w], v2 = vv[2][w], v3 = vv[3][w];
            const f16x4 b_even = __builtin_bit_cast(f16x4, make_uint2(__builtin_amdgcn_perm(v1, v0, 0x05040100u), __builtin_amdgcn_perm(v3, v2, 0x05040100u)));
            const f16x4 b_odd = __builtin_bit_cast(f16x4, make_uint2(__builtin_amdgcn_perm(v1, v0, 0x07060302u), __builtin_amdgcn_perm(v3, v2, 0x07060302u)));
            // the small product first
            acc[2 * w] = __builtin_amdgcn_mfma_f32_16x16x16f16(p_lo, b_even, acc[2 * w], 0, 0, 0);
            acc[2 * w + 1] = __builtin_amdgcn_mfma_f32_16x16x16f16(p_lo, b_odd, acc[2 * w + 1], 0, 0, 0);
            acc[2 * w] = __builtin_amdgcn_mfma_f32_16x16x16f16(p_hi, b_even, acc[2 * w], 0, 0, 0);
            acc[2 * w + 1] = __builtin_amdgcn_mfma_f32_16x16x16f16(p_hi, b_odd, acc[2 * w + 1], 0, 0, 0);
        }
    };
    // This wavefront's blocks are wave, wave + NW, ...; nmine of them hold a valid key.
    // Two-stage software pipeline, steady state free of branches around loads.
    const int nblk_valid = min(NBLK, (nres + 15) / 16);
    const int nmine = nblk_valid > wave ? (nblk_valid - wave + NW - 1) / NW : 0;
    if (nmine > 0) {
        // Rows of more than 32 chunks: the wavefront starts at a different one of its blocks in every
        // workgroup and wraps around (as in the per-row kernel: workgroups that start a power of two
        // apart and advance in step are served badly by the memory system for some shapes; 1 x 64/8
        // heads x 262144 keys: 188 us against 161 for the same bytes as 4 x 65536).  Whichever block
        // comes first fixes the scale of the fp16 weights.
        const int rot = (!EARLY && p.nc > 32 && nmine > 1) ? (int)((unsigned)(c * 3 + gi) % (unsigned)nmine) : 0;
        auto blk_of = [&](int i) { const int t = i + rot; return wave + NW * (t >= nmine ? t - nmine : t); };
        constexpr bool kMoreBlocks = !SYNC || NBLK > NW;      // than one per wavefront (a matter of registers: five were spilled)
        u32x4 kB[4], vB[4];
        if constexpr (EARLY) {                 // (no launch of this kind has 32 chunks per row: rot = 0)
            if (16 * wave + 15 > last)         // what lies past the last key may be anything: no NaN into the products
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (16 * wave + 4 * r + g > last) vA[r] = u32x4{0u, 0u, 0u, 0u};
        } else {
            issue(blk_of(0), kA, vA);
        }
        int i = 0;
#pragma unroll 1
        for (; kMoreBlocks && i + 2 < nmine; i += 2) {
            issue(blk_of(i + 1), kB, vB);
            __builtin_amdgcn_sched_barrier(0);     // keep the prefetch ahead of the arithmetic
            reduce(blk_of(i), i == 0, kA, vA);
            issue(blk_of(i + 2), kA, vA);
            __builtin_amdgcn_sched_barrier(0);
            reduce(blk_of(i + 1), false, kB, vB);
        }
        if (kMoreBlocks && i + 2 == nmine) {
            issue(blk_of(i + 1), kB, vB);
            __builtin_amdgcn_sched_barrier(0);
            reduce(blk_of(i), i == 0, kA, vA);
            reduce(blk_of(i + 1), false, kB, vB);
        } else {
            reduce(blk_of(i), i == 0, kA, vA);
        }
    }

    // ---- the appended key, if this chunk takes it: one more term of Eq. 4 per head ----
    // Lane group (wave, g) of the first four wavefronts handles head 4 wave + g on the vector ALU: weight e^{x - phi}
    // and guard from the step's own K row.  The weights go to LDS and enter the sums at
    // the reduction below, multiplied with the step's V row.
    unsigned new_mask = 0;                     // heads whose appended key left the bounds
    const size_t row_new = at.absolute(owner ? S_res - start : 0);   // where the appended row goes (all lanes look the page up)
    if (owner) {
        const int hh = 4 * wave + g;
        const size_t at_new = (size_t)gi * kHeadDim;
        const u32x4 kn = reinterpret_cast<const u32x4 *>(p.k_new + at_new)[n];
        const u32x4 qh = reinterpret_cast<const u32x4 *>(p.q + (size_t)(row0 + min(hh, G - 1)) * kHeadDim)[n];
        const float d = row16_sum(dot8(qh, kn)) * scale + nphi;
        // (hh < G never holds for a wavefront past the fourth: hh >= 16)
        if (n == 0 && hh < 16) lds.e_new[hh] = hh < G ? __builtin_amdgcn_exp2f(d * kLog2e) : 0.f;
        const unsigned long long out = __ballot((n == 0) & (hh < G) & !((d > lo) & (d < hi)));
        new_mask = (unsigned)((out | (out >> 15) | (out >> 30) | (out >> 45)) & 0xfull) << (4 * wave);
        if (wave == 0 && g == 0) {             // 16 lanes put the rows into the cache
            reinterpret_cast<u32x4 *>(p.k_store)[row_new + n] = kn;
            reinterpret_cast<u32x4 *>(p.v_store)[row_new + n] = reinterpret_cast<const u32x4 *>(p.v_new + at_new)[n];
        }
    }

    // ---- workgroup reduction and publication of the G rows' partial results ----
    // What a wavefront knows about its heads is brought together before it goes to LDS, so that little is left to do
    // behind the barrier: this part is a chain of instructions of lone wavefronts, 1.1 us when every thread read 16
    // denominators, 16 flags and four scales for itself, 0.85 now (2 x 64/8 heads x 9001 keys: whole call with the finish's loads
    // below 17.9 / 17.5 us; 1 x 12/2 x 700: 7.6 / 7.1).
    const auto heads_of = [](unsigned long long lanes) {       // lane (n, g) -> head n
        return (unsigned)((lanes | (lanes >> 16) | (lanes >> 32) | (lanes >> 48)) & 0xffffull);
    };
    const unsigned mask = heads_of(__ballot(bad)) | new_mask | heads_of(__ballot(head_on & (zmax >= kOverflowLog2))) << 16;
    // the scales are taken out where the tiles are added (exact: integer powers of two)
    const float inv = SYNC ? ref : __builtin_amdgcn_exp2f(-kq);
    den = halves_sum(den, den);
    den = rows_sum(den, den);
    if constexpr (SYNC) {
        xmax = fmaxf(xmax, __shfl_xor(xmax, 16));
        xmax = fmaxf(xmax, __shfl_xor(xmax, 32));
    } else {
        den *= inv;
    }
    __syncthreads();                           // every wavefront is done with its K staging
    // acc[e][r] is (head 4g + r, d = 8n + e) of this wavefront's partial tile.
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int h = 4 * g + r;
        if (h < G) {
            // Row layout in LDS: elements 8n..8n+3 at 4n, elements 8n+4..8n+7 at 64 + 4n, so that
            // consecutive lanes write consecutive 16-byte slots (no bank conflicts).
            float4 *dst = reinterpret_cast<float4 *>(&lds.tile[(wave * 16 + h) * kHeadDim + 4 * n]);
            dst[0] = make_float4(acc[0][r], acc[1][r], acc[2][r], acc[3][r]);
            dst[16] = make_float4(acc[4][r], acc[5][r], acc[6][r], acc[7][r]);
        }
    }
    if (g == 0) {
        lds.den[n][wave] = den;
        lds.inv[n][wave] = inv;
        if constexpr (SYNC) lds.top[n][wave] = xmax;
    }
    if (lane == 0) lds.mask[wave] = mask;
    __syncthreads();
    unsigned any = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) any |= lds.mask[w];
    any = __builtin_amdgcn_readfirstlane(any);
    const unsigned flagged_heads = any & 0xffffu;
    // heads whose sums have to be redone: the flagged ones, and those with a weight that did not fit
    const unsigned redo_heads = flagged_heads | any >> 16;
    auto den_of = [&](int h) {                 // Eq. 4's denominator of head h over this chunk
        float s = owner ? lds.e_new[h] : 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) s += lds.den[h][w];
        return s;
    };
    // SYNC: head h's maximum over the chunk, and what brings each wavefront's sums from its reference and the scale to it (0 for a
    // wavefront without a finite logit)
    auto sync_scales = [&](int h, float (&by)[NW]) {
        float m = lds.top[h][0];
#pragma unroll
        for (int w = 1; w < NW; ++w) m = fmaxf(m, lds.top[h][w]);
#pragma unroll
        for (int w = 0; w < NW; ++w)
            by[w] = lds.top[h][w] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((lds.inv[h][w] - m) * kLog2e) * (1.f / kSyncScale);
        return m;
    };
    bool unsound = false;                      // SYNC: this thread met a sum that is not a finite number, or an impossible l
    // A sequence of one chunk whose guard stayed quiet is complete here: its rows' results are
    // this workgroup's own sums, so they go out directly instead of through the workspace and
    // the epilogue (same arithmetic: the epilogue's factors are exactly 1 for such a row).
    const bool solo = p.elect && nb == 1 && nvalid > 0 && !redo_heads;
    // 4 consecutive elements per thread: one 16-byte LDS read per wavefront tile, 16 bytes out (a whole row per wavefront, 8
    // bytes per thread, took 0.4 us more where the results are written through)
    for (int i = 4 * tid; i < G * kHeadDim; i += 4 * kGqaThreads) {
        float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
        float by[NW];
        if constexpr (SYNC) sync_scales(i / kHeadDim, by);
#pragma unroll
        for (int w = 0; w < NW; ++w) {         // wavefront order
            const float4 t = *reinterpret_cast<const float4 *>(&lds.tile[w * 16 * kHeadDim + i]);
            const float k = SYNC ? by[w] : lds.inv[i / kHeadDim][w];
            o.x = __builtin_fmaf(k, t.x, o.x); o.y = __builtin_fmaf(k, t.y, o.y);
            o.z = __builtin_fmaf(k, t.z, o.z); o.w = __builtin_fmaf(k, t.w, o.w);
        }
        if constexpr (SYNC)
            unsound |= !(fabsf(o.x) + fabsf(o.y) + fabsf(o.z) + fabsf(o.w) < INFINITY);
        const int q = i & (kHeadDim - 1);      // LDS position -> element index (see the layout above)
        const int d0 = 2 * (q & 63) + 4 * (q >> 6);
        if (owner) {                           // + e_new[head] * v_new[d0 .. d0 + 3]
            const float en = lds.e_new[i / kHeadDim];
            const uint2 vn = *reinterpret_cast<const uint2 *>(p.v_new + (size_t)gi * kHeadDim + d0);
            const half2_t v01 = as_h2(vn.x), v23 = as_h2(vn.y);
            o.x = __builtin_fmaf(en, (float)v01.x, o.x); o.y = __builtin_fmaf(en, (float)v01.y, o.y);
            o.z = __builtin_fmaf(en, (float)v23.x, o.z); o.w = __builtin_fmaf(en, (float)v23.y, o.w);
        }
        if (solo) {
            const float l = den_of(i / kHeadDim);
            uint2 h;
            h.x = (unsigned)to_half_bits(o.x / l) | ((unsigned)to_half_bits(o.y / l) << 16);
            h.y = (unsigned)to_half_bits(o.z / l) | ((unsigned)to_half_bits(o.w / l) << 16);
            *reinterpret_cast<uint2 *>(p.out + (size_t)(row0 + i / kHeadDim) * kHeadDim + d0) = h;
        }
        float *dst = &p.ws.num[((size_t)(row0 + i / kHeadDim) * p.nc + c) * kHeadDim + d0];
        if (p.elect && !solo) {      // read by another workgroup of this launch: write through
            store_coherent2(dst, o.x, o.y);
            store_coherent2(dst + 2, o.z, o.w);
        } else {
            *reinterpret_cast<float4 *>(dst) = o;
        }
    }
    if constexpr (SYNC) {
        if (wave == NW - 1 && lane < G) {
            float by[NW], s = 0.f;
            const float m = sync_scales(lane, by);
#pragma unroll
            for (int w = 0; w < NW; ++w) s = __builtin_fmaf(by[w], lds.den[lane][w], s);
            unsound |= !(s >= 0.5f);                               // the largest logit alone makes it 1
            const size_t slot = (size_t)(row0 + lane) * p.nc + c;
            store_coherent(&p.ws.den[slot], s);
            store_coherent(&p.ws.mloc[slot], m);
            store_meta(p, slot, s, m, 1);
        }
        // Where a logit or a V element is not a finite number the result is what the per-row path makes of it (hi and lo parts of a
        // weight would turn an infinite V element into NaN).
        if (__syncthreads_or(unsound) && nvalid > 0) {
            wait_stores_performed();           // the stores above must not overtake the rewrite
            for (int h = 0; h < G; ++h) {
                __syncthreads();
                chunk_body<C, NW, UP, true>(p, row0 + h, c, *reinterpret_cast<ChunkLds<NW> *>(lds.tile));
            }
        }
        return;
    }
    if (wave == NW - 1 && lane < G) {
        const float s = den_of(lane);
        const size_t slot = (size_t)(row0 + lane) * p.nc + c;
        const int f = (flagged_heads >> lane) & 1;
        store_coherent(&p.ws.den[slot], s);
        store_coherent(&p.ws.mloc[slot], p.phi);
        store_meta(p, slot, s, p.phi, f);
        p.ws.chunk_flags[slot] = (uint8_t)f;
        if (solo) p.ws.row_flags[row0 + lane] = 0;
    }
    if (solo) return;
    if (EARLY && nvalid <= 0) {                // padding chunk; of an empty sequence, nobody else owns the rows
        if (nb == 0 && c == 0 && p.elect) {
            for (int i = tid; i < G * kHeadDim; i += kGqaThreads) p.out[(size_t)row0 * kHeadDim + i] = 0;
            if (tid < G) p.ws.row_flags[row0 + tid] = 0;
        }
        return;
    }

    // Section 3 "Recomputation": a (head, chunk) whose guard fired is redone with the
    // synchronized scheme on the per-row path (rare; re-reads this chunk only).  So is one whose
    // weights did not fit the fp16 operands; its slot record then says "not flagged".
    if (redo_heads) {
        wait_stores_performed();               // the stores above must not overtake the rewrite
        for (int h = 0; h < G; ++h) {
            if (!((redo_heads >> h) & 1)) continue;
            __syncthreads();
            chunk_body<C, NW, UP, true, false, PAGED>(p, row0 + h, c, *reinterpret_cast<ChunkLds<NW> *>(lds.tile), nullptr,
                                                      (int)((flagged_heads >> h) & 1));
        }
    }

    if (!p.elect) return;                      // a row-epilogue launch follows
    // Publish, arrive, and let the last arrival of the group finish its G rows.
    wait_stores_performed();
    __syncthreads();
    if (wave == 0) {
        const bool last = arrive_and_elect(p, row0, c, nb);
        if (lane == 0) lds.last = last;
    }
    __syncthreads();
    if (!lds.last) return;
    group_epilogue(p, row0, G, nb);
}

template <int C, bool SYNC> struct GqaLauncher {
    static hipError_t run(const Problem &p0, hipStream_t s)
    {
        const long long groups = (long long)p0.B * p0.Hkv;
        const unsigned grid = (unsigned)(8ll * ((groups + 7) / 8) * p0.nc);
        if (grid == 0) return hipSuccess;
        Problem p = p0;
        p.chunk_major = grid <= 1024u;
        // every XCD reads from every head group, unless the launch is short and hands over inside (see row_slot)
        p.scatter |= !p.elect || grid > (unsigned)kComputeUnits;
        // 4 wavefronts per workgroup.  (8 were measured for launches of at most one workgroup per
        // compute unit: within 2 % either way at 256 workgroups, 12 % faster only for a lone
        // 4096-key chunk, which fd_pick_chunk never chooses.)
        // By length where a compute unit holds more than one workgroup and the lengths of the batch fit a wavefront: what has to be
        // streamed is spread evenly, and over all XCDs also where the head groups do not divide by 8.  Whole call, general order / this:
        // 12 x 32/8 heads x 300 .. 6000 keys 37.6 / 34.2 us, 32 x 64/8 x 512 .. 4096 in 1024-key chunks 64.4 / 59.8, 64 x 64/8 x 300 ..
        // 8192 203 / 182, 5 x 28/4 x 3000 .. 20000 40.4 / 26.4, 1 x 28/4 x 20000 16.4 / 14.8, 1 x 12/2 x 30000 18.4 / 15.0; equal lengths
        // pay for looking at them: 12 x 64/8 x 4096 36.5 / 36.7, 32 x 64/8 x 16384 320.7 / 321.2.  Beyond 4096 workgroups a
        // workgroup is short beside the 0.3 us that finding its chunk takes (32 x 64/8 x 1500 .. 3000 in 128-key chunks, 6144
        // workgroups, 63.0 / 64.2), and they even out by themselves.
        // Early loads in the launches of one workgroup per compute unit: 2 x 64/8 x 9001 17.1 / 16.8 us, 4 x 32/8 x 4096 14.85 /
        // 14.6, 1 x 28/4 x 700 7.4 / 7.15.
        const dim3 g(grid), t(256);
        const bool by_length = grid > (unsigned)kComputeUnits && grid <= 4096u && p.B <= 64;
        if constexpr (!SYNC) {
            if (p.block_table)
                return by_length ? launch(decode_fused_gqa_kernel<C, true, kByLength>, g, t, s, p)
                                 : launch(decode_fused_gqa_kernel<C, true, kPlain>, g, t, s, p);
        }
        return by_length                          ? launch(decode_fused_gqa_kernel<C, false, kByLength, SYNC>, g, t, s, p)
               : grid <= (unsigned)kComputeUnits ? launch(decode_fused_gqa_kernel<C, false, kEarly, SYNC>, g, t, s, p)
                                                 : launch(decode_fused_gqa_kernel<C, false, kPlain, SYNC>, g, t, s, p);
    }
};

}  // namespace

template <bool SYNC> static hipError_t dispatch_gqa(const Problem &p, hipStream_t s)
{
    switch (chunk_capacity(p.C)) {
        case 64:   return GqaLauncher<64, SYNC>::run(p, s);
        case 128:  return GqaLauncher<128, SYNC>::run(p, s);
        case 256:  return GqaLauncher<256, SYNC>::run(p, s);
        case 512:  return GqaLauncher<512, SYNC>::run(p, s);
        case 1024: return GqaLauncher<1024, SYNC>::run(p, s);
        case 2048: return GqaLauncher<2048, SYNC>::run(p, s);
        case 4096: return GqaLauncher<4096, SYNC>::run(p, s);
        default:   return hipErrorInvalidValue;
    }
}

hipError_t launch_decode_fused_gqa(const Problem &p, hipStream_t s) { return dispatch_gqa<false>(p, s); }
hipError_t launch_partial_sync_gqa(const Problem &p, hipStream_t s) { return dispatch_gqa<true>(p, s); }

}  // namespace fd

// Device code shared by the chunk kernels: the per-(row, chunk) body of the VALU
// path and the row epilogue (outer sums / synchronized merge).
//
// Lane layout of the VALU path.  A K or V row is 256 bytes = 16 segments of 16
// bytes; lane l of a wavefront owns segment l%16 of key (l/16) within a group of
// 4 consecutive keys, so one wavefront load instruction reads 1 KiB of contiguous
// cache memory with 128-bit loads.  The four wavefronts of a workgroup interleave
// groups, i.e. the workgroup walks the chunk front to back 4 KiB at a time.  The
// 16 lanes of a key reduce their 8-element partial dot products with DPP row
// operations (a DPP row is exactly 16 lanes), after which every one of the 16
// lanes holds the key's logit and scales its own 8 elements of the V row.
// K and V are read exactly once and never reused, so they are loaded with
// non-temporal loads straight into registers; LDS only carries the final
// cross-wavefront reduction.
#pragma once

#include <type_traits>
#include <utility>

#include "fd_internal.h"

namespace fd {

// Phase probe (a build of its own, -DFD_PHASE_PROBE, never the product library): thread 0 of
// every workgroup of the per-row fused kernel stamps the device's constant-rate clock (100 MHz)
// at fixed points into a log that fd_phase_probe_read copies out.  Slots: 0 kernel entered,
// 1 first block's data used, 2 chunk loop done, 3 workgroup's sums reduced and stores issued,
// 4 stores performed, 5 arrival counted, 6 (finisher) partial results loaded and merged, 7
// (finisher) output stored and performed.
#ifdef FD_PHASE_PROBE
constexpr int kPhaseSlots = 8, kPhaseMaxGrid = 4096;
static __device__ unsigned long long fd_phase_log[kPhaseMaxGrid * kPhaseSlots];
#define FD_PHASE(i)                                                                                         \
    do {                                                                                                    \
        __builtin_amdgcn_sched_barrier(0);                                                                  \
        if (threadIdx.x == 0 && blockIdx.x < (unsigned)kPhaseMaxGrid)                                       \
            fd_phase_log[(size_t)blockIdx.x * kPhaseSlots + (i)] = wall_clock64();                          \
        __builtin_amdgcn_sched_barrier(0);                                                                  \
    } while (0)
#else
#define FD_PHASE(i) do { } while (0)
#endif

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// (bit-casting a vector ELEMENT in place is unreliable: take the element by value first)
__device__ __forceinline__ half2_t as_h2(uint32_t u) { return __builtin_bit_cast(half2_t, u); }
__device__ __forceinline__ float as_f32(uint32_t u) { return __builtin_bit_cast(float, u); }

// 128-bit streaming load: the data is used once, keep it from displacing other lines.
__device__ __forceinline__ u32x4 load_stream(const u32x4 *p) { return __builtin_nontemporal_load(p); }

// fp32 dot product of 8 fp16 pairs, two products to an instruction: asked for by name, so that every place that forms a logit rounds it alike (left to
// itself the compiler made this of some chains of multiply-adds and not of others, and equal keys got logits an ulp apart, which is whole units
// for large ones).  As exact as the chain: 128 elements of N(0, 1) by 16 lanes, rms error 7.8e-7, chain 8.3e-7.
__device__ __forceinline__ float dot8(const u32x4 &a, const u32x4 &b)
{
    float acc = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_fdot2(as_h2(a[i]), as_h2(b[i]), acc, false);
    return acc;
}

// a * b as an fp32 number, whatever it is used in next: fused into an addition the product would not be rounded, and where logits are so large
// that neighbouring fp32 numbers are whole units apart, equal ones have to come out equal.
__device__ __forceinline__ float rounded_product(float a, float b)
{
#pragma clang fp contract(off)
    return a * b;
}

// acc[0..7] += p * v[0..7]
__device__ __forceinline__ void axpy8(float (&acc)[8], float p, const u32x4 &v)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const half2_t x = as_h2(v[i]);
        acc[2 * i]     = __builtin_fmaf(p, (float)x.x, acc[2 * i]);
        acc[2 * i + 1] = __builtin_fmaf(p, (float)x.y, acc[2 * i + 1]);
    }
}

template <int CTRL>
__device__ __forceinline__ float dpp_swap(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}

// Sum over the 16 lanes of a DPP row; every lane ends with the total.
__device__ __forceinline__ float row16_sum(float x)
{
    x += dpp_swap<0xB1>(x);   // quad_perm [1,0,3,2]  : lane ^ 1
    x += dpp_swap<0x4E>(x);   // quad_perm [2,3,0,1]  : lane ^ 2
    x += dpp_swap<0x141>(x);  // row_half_mirror      : other quad of the 8
    x += dpp_swap<0x140>(x);  // row_mirror           : other half of the 16
    return x;
}

// Maximum over the 16 lanes of a DPP row; every lane ends with it.
__device__ __forceinline__ float row16_max(float x)
{
    x = fmaxf(x, dpp_swap<0xB1>(x));
    x = fmaxf(x, dpp_swap<0x4E>(x));
    x = fmaxf(x, dpp_swap<0x141>(x));
    return fmaxf(x, dpp_swap<0x140>(x));
}
// The value of lane I of the DPP row in all its lanes (row_newbcast).
template <int I> __device__ __forceinline__ float row16_lane(float x) { return dpp_swap<0x150 + I>(x); }
template <class F, int... I> __device__ __forceinline__ void each16(std::integer_sequence<int, I...>, F f)
{
    (f(std::integral_constant<int, I>{}), ...);
}

// Device-coherent accesses for results that another workgroup of the SAME launch
// reads (the per-chunk partial results and the per-row ticket).  Each XCD has its
// own L2, so such data is written through and read past the L2 ("agent scope"
// relaxed atomics); ordinary cached accesses would need an L2 write-back fence per
// workgroup, which costs about a microsecond each and serializes per XCD.
template <typename T>
__device__ __forceinline__ void store_coherent(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T load_coherent(const T *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The (den, reference, flag) record of a slot, written through as two 8-byte words.
__device__ __forceinline__ void store_meta(const Problem &p, size_t slot, float den, float ref, int flagged)
{
    unsigned long long *w = reinterpret_cast<unsigned long long *>(&p.ws.meta[slot]);
    store_coherent(&w[0], (unsigned long long)__builtin_bit_cast(unsigned, den) |
                              ((unsigned long long)__builtin_bit_cast(unsigned, ref) << 32));
    store_coherent(&w[1], (unsigned long long)(unsigned)flagged);
}

// Two consecutive floats written through as one 8-byte word (8-byte aligned).
__device__ __forceinline__ void store_coherent2(float *ptr, float a, float b)
{
    store_coherent(reinterpret_cast<unsigned long long *>(ptr),
                   (unsigned long long)__builtin_bit_cast(unsigned, a) | ((unsigned long long)__builtin_bit_cast(unsigned, b) << 32));
}

// Wait until this thread's earlier stores are performed (vector memory counter at
// zero); with write-through stores this is the release half of the hand-over.
__device__ __forceinline__ void wait_stores_performed()
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// Wait until this wavefront's earlier vector loads have arrived (and nothing else: vmcnt(0) alone).
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0f70); }

__device__ __forceinline__ uint16_t to_half_bits(float x)
{
    return __builtin_bit_cast(uint16_t, (_Float16)x);   // round to nearest even
}

// The value of the other half of the wavefront / of the neighbouring row of 16 added in, two registers at a time:
// halves_sum(a, b): lanes 0-31 get a summed over the halves, lanes 32-63 b; rows_sum(a, b): the even rows of 16 get a
// summed over the pair of rows, the odd ones b.  (Vector elements are taken by value first, see as_h2.)
__device__ __forceinline__ float halves_sum(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b), false, false);
    const unsigned x = r[0], y = r[1];
    return as_f32(x) + as_f32(y);
}
__device__ __forceinline__ float rows_sum(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b), false, false);
    const unsigned x = r[0], y = r[1];
    return as_f32(x) + as_f32(y);
}

// Inclusive sum over the lanes of a wavefront.
__device__ __forceinline__ int lanes_scan(int x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr 1, 2, 4, 8: within rows of 16
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // lane 15 to row 1, lane 47 to row 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // lane 31 to rows 2 and 3
    return x;
}

// The maximum over the four rows of 16 of a wavefront, in every lane.
__device__ __forceinline__ float columns_max(float a)
{
    const unsigned u = __builtin_bit_cast(unsigned, a);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const unsigned r0 = r[0], r1 = r[1];
    const unsigned v = __builtin_bit_cast(unsigned, fmaxf(as_f32(r0), as_f32(r1)));
    const auto h = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    const unsigned h0 = h[0], h1 = h[1];
    return fmaxf(as_f32(h0), as_f32(h1));
}

// LDS of one workgroup of NW wavefronts.
template <int NW>
struct ChunkLds {
    alignas(16) float acc[NW][kHeadDim];   // [wave][pairs of elements, see chunk_body]
    alignas(16) float den[NW];
    alignas(16) int   flag[NW];
    alignas(16) float ref[NW];             // what the wavefronts' sums are scaled by ...
    alignas(16) float top[NW];             // ... and their largest logits (unified scheme: largest weights)
};

// References that move (chunk_body).
constexpr float kNoRef = -3e38f;           // the largest logit of no logit
constexpr float kRaise = 40.f;             // a logit this far above the wavefront's reference raises it
// The bounds within which the weights of in-range logits leave sums that can be brought to another reference: e^-64 and 4096 e^60 max|v|
// are ordinary fp32 numbers.
constexpr float kInPlaceLo = -64.f, kInPlaceHi = 60.f;
// And how far from 0 and from the old reference a new one may lie: the difference of two such numbers, rounded, is within 2^-7 of the exact one, so
// the largest weight is 1 to within that.
constexpr float kInPlaceReach = 65536.f;

// A wavefront's four columns of sums added in registers, exchanging halves and rows of
// two registers at a time, so that lane (sub, seg) ends up with elements 8 seg + 2 sub and the next: 12 instructions.
__device__ __forceinline__ void wave_sums(const float (&acc)[8], float &den, float (&u)[2])
{
    float t[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i] = halves_sum(acc[i], acc[i + 4]);
#pragma unroll
    for (int i = 0; i < 2; ++i) u[i] = rows_sum(t[i], t[i + 2]);
    den = halves_sum(den, den);
    den = rows_sum(den, den);
}
// The pair of lane (sub, seg), number 4 seg + sub of its vector, sits in place 4 seg + (sub ^ 2 (seg / 8)) of a wavefront's vector in LDS: few bank
// conflicts there (4 cycles per wavefront), and none where lane l reads pair l back, so that the slot is written in whole lines (pairs stored as the
// lanes hold them, 32 bytes apart, cost launches of full caches 1 %).
__device__ __forceinline__ float2 *sums_place(float *acc, int lane)
{
    const int seg = lane & 15, sub = lane >> 4;
    return reinterpret_cast<float2 *>(acc + 8 * seg + 2 * (sub ^ ((seg >> 2) & 2)));
}
__device__ __forceinline__ const float2 *sums_read(const float *acc, int lane)
{
    return reinterpret_cast<const float2 *>(acc + 2 * (lane ^ ((lane >> 4) & 2)));
}

// One (row, chunk) on the VALU path, by a workgroup of NW wavefronts.
//   SYNC == false : unified scaling factor phi -- Eq. 4 inner sums and the range
//                   guard of Section 3 "Recomputation".  Writes num, den,
//                   chunk_flags and mloc = phi (the reference the sums are scaled by).  Where the guard fires the wavefront goes on by the
//                   synchronized scheme from that block of keys on (see `adapt` below), and the slot's reference is the chunk's largest
//                   logit, as after SYNC (formed from the largest weight: to within fp32 rounding); with bounds beyond kInPlaceLo, kInPlaceHi,
//                   and for logits beyond kInPlaceReach, the caller has to redo the chunk instead.
//   SYNC == true  : the chunk's part of the synchronized partial softmax, Eq. 2, in one pass: a wavefront keeps a reference that
//                   a logit more than kRaise above it raises, and its sums are brought to m = max x at the end: l = sum e^{x-m}, f.V = sum
//                   e^{x-m} v.  Writes num, den, mloc = m and leaves chunk_flags alone; `sync_flag` is what the
//                   slot's record tells the row epilogue about the guard.
// UP = groups of 4 keys per wavefront per pipeline stage.
// Returns (uniformly over the workgroup) whether the chunk has to be redone with SYNC.
// Pins the kernel arguments the chunk loop needs into scalar registers at this point,
// so that their loads leave in one batch at the top of the kernel.  Left alone the
// compiler fetches each cache line of the argument block where it is first used --
// behind the early-exit test, behind the index arithmetic -- and a fresh wavefront
// then pays three dependent memory latencies instead of one.
__device__ __forceinline__ void fetch_arguments_now(const Problem &p)
{
    asm volatile("" ::"s"(p.q), "s"(p.k), "s"(p.v), "s"(p.seq_lens), "s"(p.Hq), "s"(p.G), "s"(p.Hkv), "s"(p.Smax),
                 "s"(p.nc), "s"(p.rows));
}

// The sequence length through a vector load, in two halves.  Scalar loads return out
// of order, so waiting for any of them waits for all: a scalar length load would be
// waited for together with the kernel arguments, before the first K/V load can go
// out.  Vector loads return in order; this one stays in flight behind the loads
// issued between the two halves.  (The opaque zero keeps the compiler from proving
// the address uniform and turning the load back into a scalar one.)
__device__ __forceinline__ int seq_len_issue(const Problem &p, int b)
{
    int zero;
    asm("v_mov_b32 %0, 0" : "=v"(zero));
    return p.seq_lens[b + zero];
}
__device__ __forceinline__ int seq_len_finish(const Problem &p, int raw)
{
    return clamp_len(p, __builtin_amdgcn_readfirstlane(raw));     // resident keys
}

// Where the rows of a chunk's keys are, in 16-byte units from the start of K (or V; both are
// laid out alike): consecutive rows of the caller's buffer, or -- paged cache -- row t % page of
// the page the sequence's table names for t / page.  A chunk spans at most 64 pages (the
// entry points see to it); each lane fetches one table entry when the chunk starts and a lane
// exchange hands every lane the page of the key it is about to load.  Entries of pages that
// hold no valid key may be anything: they are clamped into the pool and what they bring in is
// never used.
template <bool PAGED> struct KvRows {
    size_t base;             // first row of the chunk (contiguous), 0 (paged)
    int pages, first, start, shift, hkv, Hkv;
    __device__ __forceinline__ KvRows(const Problem &p, int b, int hkv_, int start_, int lane)
        : base(PAGED ? 0 : (((size_t)b * p.Hkv + hkv_) * p.Smax + start_) * 16), pages(0), first(0), start(start_),
          shift(p.page_shift), hkv(hkv_), Hkv(p.Hkv)
    {
        if constexpr (PAGED) {
            first = start_ >> shift;
            const int entry = p.block_table[(size_t)b * p.pages_per_seq + min(first + lane, p.pages_per_seq - 1)];
            pages = min(max(entry, 0), p.n_pages - 1);
        }
    }
    // First row, relative to `base`, of the 16 keys key0 .. key0 + 15 (key0 a multiple of 16, the same
    // for the whole wavefront): they share a page, which one lane-to-scalar read finds.
    __device__ __forceinline__ size_t block16(int key0) const
    {
        if constexpr (PAGED) {
            const int t = start + key0;
            const int page = __builtin_amdgcn_readlane(pages, (t >> shift) - first);
            return ((((size_t)page * Hkv + hkv) << shift) + (size_t)(t & ((1 << shift) - 1))) * 16;
        } else {
            return (size_t)key0 * 16;
        }
    }
    // row of chunk-relative key `key` from the start of the buffer or pool (for the store of an appended row)
    __device__ __forceinline__ size_t absolute(int key) const { return base + (*this)(key); }
    // row of chunk-relative key `key`, relative to `base`
    __device__ __forceinline__ size_t operator()(int key) const
    {
        if constexpr (PAGED) {
            const int t = start + key;
            const int page = __builtin_amdgcn_ds_bpermute(((t >> shift) - first) << 2, pages);
            return ((((size_t)page * Hkv + hkv) << shift) + (size_t)(t & ((1 << shift) - 1))) * 16;
        } else {
            return (size_t)key * 16;
        }
    }
};

// EARLY: the first block's loads are issued before the
// sequence length has arrived, clamped to the chunk's extent in the padded buffer
// instead of to the last valid key; what they bring in from beyond the valid
// length is replaced by zeros before use.  Takes the length load off the critical
// path of a short launch; a padding chunk then reads one block for nothing, so
// large ragged launches leave it off.
// ONE: a wavefront asks for a block of keys only when the one before has arrived, instead of
// keeping two in flight (LoadAhead in fd_row_kernels.hip says where).
// REDONE: another launch sums every chunk of a flagged row anew, so nothing is done about a guard that fires.
template <int C, int NW, int UP, bool SYNC, bool EARLY = false, bool PAGED = false, bool ONE = false, bool REDONE = false>
__device__ __forceinline__ bool chunk_body(const Problem &p, int row, int c, ChunkLds<NW> &lds, int *len_out = nullptr,
                                           int sync_flag = 1)
{
    static_assert(!(EARLY && PAGED), "the page table has to arrive before the first load");
    constexpr int NG = C / (4 * NW);           // groups of 4 keys each wavefront handles
    static_assert(NG >= 1 && NG % UP == 0, "chunk, wavefront count and stage depth must divide");
    constexpr int NBLK = NG / UP;
    // Keys whose logits are checked together, before any of them is added: a stage, but half of one where its registers would take a
    // wavefront per SIMD (133 in the long paged kernels).  One or two at a time made no difference elsewhere (23 shapes within 1 %).
    constexpr int UG = PAGED && C >= 1024 ? 2 : UP;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int seg = lane & 15, sub = lane >> 4;

    const int b = row / p.Hq;
    const int hq = row - b * p.Hq;
    const int hkv = hq / p.G;
    int S_raw = 0;
    if constexpr (EARLY) S_raw = seq_len_issue(p, b);
    const int len = p.C;                       // keys per chunk (<= C, the kernel's capacity)
    const int start = c * len;
    const size_t slot = (size_t)row * p.nc + c;

    const u32x4 qv = reinterpret_cast<const u32x4 *>(p.q + (size_t)row * kHeadDim)[seg];
    const KvRows<PAGED> at(p, b, hkv, start, lane);
    const u32x4 *kp = reinterpret_cast<const u32x4 *>(p.k) + at.base + seg;
    const u32x4 *vp = reinterpret_cast<const u32x4 *>(p.v) + at.base + seg;
    // key handled by this lane in group g of the chunk: the NW wavefronts interleave
    auto key_of = [&](int g) { return (g * NW + wave) * 4 + sub; };
    u32x4 kA[UP], vA[UP];
    if constexpr (EARLY) {
        const int cap = min(len, p.Smax - start) - 1;   // the chunk's last key inside the buffer (start < Smax)
#pragma unroll
        for (int u = 0; u < UP; ++u) kA[u] = load_stream(kp + at(min(key_of(u), cap)));
#pragma unroll
        for (int u = 0; u < UP; ++u) vA[u] = load_stream(vp + at(min(key_of(u), cap)));
    }

    if constexpr (EARLY) __builtin_amdgcn_sched_barrier(0);   // the loads above go out before the length is awaited
    const int S_res = EARLY ? seq_len_finish(p, S_raw) : clamp_len(p, p.seq_lens[b]);
    const int S = effective_len(p, S_res);
    if (len_out) *len_out = S;
    const int nvalid = min(len, S - start);    // <= 0: no valid key in this chunk
    const int nres = min(len, S_res - start);  // of them resident in the cache
    // A fused append puts the new key at offset jn of exactly one chunk of the row.
    const int jn = S_res - start;
    const bool owner = (S != S_res) & (jn >= 0) & (jn < len);
    // where the appended row goes (all lanes take part in the page lookup of a paged cache)
    const size_t row_new = at.absolute(owner ? jn : 0);
    // With early loads an empty chunk takes the ordinary path below (no block beyond the
    // first is touched, every key is masked): a branch here would pull the loads behind it.
    if (!EARLY && nvalid <= 0) {               // empty chunk: zero partials, no flag
        if (tid < kHeadDim) p.ws.num[slot * kHeadDim + tid] = 0.f;
        if (tid == 0) {
            p.ws.den[slot] = 0.f;
            p.ws.mloc[slot] = SYNC ? -INFINITY : p.phi;
            store_meta(p, slot, 0.f, p.phi, 0);
            if (!SYNC) p.ws.chunk_flags[slot] = 0;
        }
        return false;
    }

    const int last = nres - 1;                 // last resident key; the appended one is handled apart
    // blocks (of UP groups per wavefront) that hold at least one resident key
    const int nblk = min(NBLK, (nres + UP * NW * 4 - 1) / (UP * NW * 4));
    // the appended rows of this row's KV head
    const u32x4 *knp = reinterpret_cast<const u32x4 *>(p.k_new + ((size_t)b * p.Hkv + hkv) * kHeadDim) + seg;
    const u32x4 *vnp = reinterpret_cast<const u32x4 *>(p.v_new + ((size_t)b * p.Hkv + hkv) * kHeadDim) + seg;

    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float den = 0.f;

    // Software pipeline over blocks of UP groups: the loads of block i+1 are in
    // flight while block i is reduced.  Keys past the valid length re-read the
    // last valid key (always in bounds, never padding) and get weight zero.
    const float scale = p.scale;
    float nref = SYNC ? 0.f : -p.phi;          // minus this wavefront's reference
    float lo = p.lo, hi = SYNC ? -INFINITY : p.hi;                                // (SYNC: the logit that raises it; the first block in any case)
    const bool in_place = SYNC || (!REDONE && p.lo >= kInPlaceLo && p.hi <= kInPlaceHi);      // uniform
    int out_of_range = 0;                      // 1: a logit of this wavefront was outside (lo, hi); | 2: and the chunk has to be redone for it
    float top = SYNC ? kNoRef : 0.f;           // largest logit of this lane's keys (SYNC), their largest weight
    // A logit is out of range: the wavefront's reference becomes the largest of the block, or stays if it is larger, and the sums
    // are brought to it (Eq. 2); from here on only a logit far above moves it again.  Without sums it takes that largest in any case.
    // d: this lane's largest, less the reference.  SYNC: d is the logit itself, and the reference a logit: taken
    // off the others, rounded like it, it leaves 0 for every equal one, however far apart fp32 numbers of that size are.  (Re-reading the chunk by a second,
    // synchronized pass cost a short launch the time in which one workgroup streams a chunk by itself: whole call with one flagged row, that / this,
    // 1 x 32 x 8192 34.1 / 22.4 us, 4 x 16 x 6400 53.2 / 35.5, 1 x 32 x 1024 9.0 / 6.1, 1 x 16 x 9000 .. 60000 96 / 79.7.)
    auto adapt = [&](float d) {
        d = columns_max(d);
        if constexpr (SYNC) {
            if (d == -INFINITY) return;
        } else if (!(fmaxf(fabsf(d), fabsf(nref - d)) < kInPlaceReach)) {        // (also where no logit of the block is a finite number)
            out_of_range = 3;
            return;
        }
        const bool fresh = __ballot(den != 0.f) == 0ull;
        const float ref = fresh ? d : fmaxf(d, SYNC ? -nref : 0.f);
        if (!fresh) {
            const float f = __builtin_amdgcn_exp2f((SYNC ? -nref - ref : -ref) * kLog2e);
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[i] *= f;
            den *= f;
            if constexpr (!SYNC) top *= f;
        }
        nref = SYNC ? -ref : nref - ref;
        lo = -INFINITY;
        hi = SYNC ? ref + kRaise : kRaise;
    };
    {
        // Rows of more than 32 chunks: every workgroup starts its chunk at a different block and wraps
        // around (the sums do not care about the order).  The workgroups of such a launch start at
        // addresses a power of two apart and walk them in step, and for some shapes the memory system
        // serves that badly: 1 x 32 rows x 131072 keys in 1024-key chunks 462 -> 338 us, 2 x 131072
        // 718 -> 652, 1 x 131072 in 2048-key chunks 333 -> 317; the shapes that were fine lose up to
        // 1.4 % (4 x 65536), and with 32 chunks per row or fewer (4 x 32768: 321 -> 330 us) it only costs.
        const int rot = (!EARLY && p.nc > 32 && nblk > 1) ? (int)((unsigned)(c * 3 + row) % (unsigned)nblk) : 0;
        auto phys = [&](int blk) { const int b = blk + rot; return b >= nblk ? b - nblk : b; };
        auto issue = [&](int blk0, u32x4 (&kk)[UP], u32x4 (&vv)[UP]) {
            const int blk = phys(blk0);
#pragma unroll
            for (int u = 0; u < UP; ++u) kk[u] = load_stream(kp + at(min(key_of(blk * UP + u), last)));
#pragma unroll
            for (int u = 0; u < UP; ++u) vv[u] = load_stream(vp + at(min(key_of(blk * UP + u), last)));
        };
        auto reduce = [&](int blk0, const u32x4 (&kk)[UP], const u32x4 (&vv)[UP]) {
            const int blk = phys(blk0);
#pragma unroll
            for (int u0 = 0; u0 < UP; u0 += UG) {
                bool valid[UG], bad = false;
                float d[UG];                                        // x - phi (SYNC: x)
#pragma unroll
                for (int u = 0; u < UG; ++u) {
                    valid[u] = key_of(blk * UP + u0 + u) <= last;
                    const float x = row16_sum(dot8(qv, kk[u0 + u]));
                    if constexpr (SYNC) {
                        d[u] = rounded_product(x, scale);
                        top = fmaxf(top, valid[u] ? d[u] : kNoRef);
                        bad |= valid[u] & !(d[u] < hi);
                    } else {
                        d[u] = __builtin_fmaf(x, scale, nref);
                        bad |= valid[u] & !((d[u] > lo) & (d[u] < hi));          // equality and NaN flag
                    }
                }
                if (__builtin_expect(__ballot(bad) != 0ull, 0)) {
                    out_of_range |= 1;
                    if (in_place) {
                        float most = -INFINITY;
#pragma unroll
                        for (int u = 0; u < UG; ++u) most = fmaxf(most, valid[u] ? d[u] : -INFINITY);
                        adapt(most);
                        // formed anew from the key, the difference is the same for equal keys of any block
                        if constexpr (!SYNC) {
#pragma unroll
                            for (int u = 0; u < UG; ++u) d[u] = __builtin_fmaf(row16_sum(dot8(qv, kk[u0 + u])), scale, nref);
                        }
                    }
                }
#pragma unroll
                for (int u = 0; u < UG; ++u) {
                    float e = __builtin_amdgcn_exp2f((SYNC ? d[u] + nref : d[u]) * kLog2e);      // e^{x - phi}
                    e = valid[u] ? e : 0.f;
                    den += e;
                    if constexpr (!SYNC) top = fmaxf(top, e);
                    axpy8(acc, e, vv[u0 + u]);
                }
            }
        };
        u32x4 kB[UP], vB[UP];
        int blk = 0;
        if constexpr (EARLY) {
            // Block 0 is already in flight.  Block 1 goes out before block 0 is touched
            // (clamped into the chunk even when no key is valid), then the loop keeps two
            // blocks in flight; loads past the last block re-read the last valid key.
            if constexpr (NBLK > 1) {
#pragma unroll
                for (int u = 0; u < UP; ++u) kB[u] = load_stream(kp + at(max(min(key_of(UP + u), last), 0)));
#pragma unroll
                for (int u = 0; u < UP; ++u) vB[u] = load_stream(vp + at(max(min(key_of(UP + u), last), 0)));
            }
#pragma unroll
            for (int u = 0; u < UP; ++u)
                if (key_of(u) > last) vA[u] = u32x4{0u, 0u, 0u, 0u};   // padding may hold anything
#ifdef FD_PHASE_PROBE
            // (probe build only: the first block peeled so that its arrival can be stamped)
            if (blk + 2 < nblk) {
                reduce(blk, kA, vA);
                FD_PHASE(1);
                issue(blk + 2, kA, vA);
                reduce(blk + 1, kB, vB);
                issue(blk + 3, kB, vB);
                blk += 2;
            }
#endif
#pragma unroll 1
            for (; blk + 2 < nblk; blk += 2) {
                reduce(blk, kA, vA);
                issue(blk + 2, kA, vA);
                reduce(blk + 1, kB, vB);
                issue(blk + 3, kB, vB);
            }
            reduce(blk, kA, vA);
            if constexpr (NBLK > 1) {
                if (blk + 1 < nblk) reduce(blk + 1, kB, vB);
            }
        } else if (nres > 0) {                     // (a chunk may hold the appended key only)
            // The steady-state loop issues unconditionally (a load inside a branch
            // would force a full wait at the join); the last one or two blocks are peeled.
            issue(0, kA, vA);
#pragma unroll 1
            for (; blk + 2 < nblk; blk += 2) {
                if constexpr (ONE) wait_loads();
                issue(blk + 1, kB, vB);
                reduce(blk, kA, vA);
                if constexpr (ONE) wait_loads();
                issue(blk + 2, kA, vA);
                reduce(blk + 1, kB, vB);
            }
            if (blk + 2 == nblk) {
                issue(blk + 1, kB, vB);
                reduce(blk, kA, vA);
                reduce(blk + 1, kB, vB);
            } else {
                reduce(blk, kA, vA);
            }
        }
        if (owner && wave == 0) {
            // The appended key: one more term of Eq. 4, taken from the step's own K/V rows by
            // the 16 lanes of the first key column, which also put the rows into the cache (a chunk that is redone has
            // stored them already).
            const u32x4 kn = *knp, vn = *vnp;
            float x = row16_sum(dot8(qv, kn));
            if constexpr (SYNC) {
                x = rounded_product(x, scale);
                top = fmaxf(top, x);
            }
            auto less_ref = [&] { return SYNC ? x + nref : __builtin_fmaf(x, scale, nref); };
            const float d = less_ref();
            if (SYNC ? !(x < hi) : !((d > lo) & (d < hi))) {
                out_of_range |= 1;
                if (in_place) adapt(SYNC ? x : d);
            }
            if (sub == 0) {
                const float e = __builtin_amdgcn_exp2f(less_ref() * kLog2e);
                if constexpr (!SYNC) top = fmaxf(top, e);
                den += e;
                axpy8(acc, e, vn);
                if (!SYNC && hq == hkv * p.G) {     // one writer per KV head
                    reinterpret_cast<u32x4 *>(p.k_store)[row_new + seg] = kn;
                    reinterpret_cast<u32x4 *>(p.v_store)[row_new + seg] = vn;
                }
            }
        }
    }
    auto hand_over_reference = [&] {
        top = columns_max(top);
        if (lane == 0) { lds.ref[wave] = -nref; lds.top[wave] = top; }
    };
    if constexpr (SYNC) hand_over_reference();
    else if (lane == 0) lds.flag[wave] = out_of_range;

    if constexpr (!SYNC) FD_PHASE(2);
    // Workgroup reduction.  Within a wavefront in registers; then wavefront 0 adds the others' sums and writes the slot by itself, and
    // what follows (the arrival, the row's finish) needs no barrier; the other wavefronts are done and make room.  (Before, all NW * 4 vectors
    // went through LDS and two wavefronts added them, with a barrier before and after the arrival.)
    float u[2];
    wave_sums(acc, den, u);
    *sums_place(lds.acc[wave], lane) = make_float2(u[0], u[1]);
    if (lane == 0) lds.den[wave] = den;
    __syncthreads();
    int flagged = 0;
    if constexpr (!SYNC) {
#pragma unroll
        for (int w = 0; w < NW; ++w) flagged |= lds.flag[w];
    }
    const bool redo = flagged != 0 && (!in_place || flagged != 1);
    const bool in_place_sums = !SYNC && __builtin_expect(flagged != 0 && !redo, 0);
    if (in_place_sums) {                       // (uniform; only now are the references needed, so that other chunks do without them)
        hand_over_reference();
        __syncthreads();
    }
    if (wave == 0) {
        u[0] = u[1] = den = 0.f;
        float mc = p.phi;
        if (SYNC || in_place_sums) {
            // from each wavefront's reference to the largest logit
            mc = kNoRef;
#pragma unroll
            for (int w = 0; w < NW; ++w)
                mc = fmaxf(mc, SYNC ? lds.top[w] : lds.top[w] > 0.f ? __builtin_fmaf(__builtin_amdgcn_logf(lds.top[w]), 1.f / kLog2e, lds.ref[w]) : kNoRef);
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const float2 o = *sums_read(lds.acc[w], lane);
                const float l = lds.den[w], f = l == 0.f ? 0.f : __builtin_amdgcn_exp2f((lds.ref[w] - mc) * kLog2e);
                u[0] = __builtin_fmaf(f, o.x, u[0]);
                u[1] = __builtin_fmaf(f, o.y, u[1]);
                den = __builtin_fmaf(f, l, den);
            }
            if (mc == kNoRef) mc = -INFINITY;      // no key, or no logit above -infinity
        } else {
#pragma unroll
            for (int w = 0; w < NW; ++w) {         // wavefront order
                const float2 o = *sums_read(lds.acc[w], lane);
                u[0] += o.x;
                u[1] += o.y;
                den += lds.den[w];
            }
        }
        store_coherent2(&p.ws.num[slot * kHeadDim + 2 * lane], u[0], u[1]);
        if (lane == 0) {
            store_coherent(&p.ws.den[slot], den);
            store_coherent(&p.ws.mloc[slot], mc);
            // the flag the row epilogue ORs into the row flag: the guard's; a recomputed chunk carries what its caller
            // says (1 when the guard sent it here, 0 when it is redone for another reason)
            store_meta(p, slot, den, mc, SYNC ? sync_flag : (int)(flagged != 0));
            if (!SYNC) p.ws.chunk_flags[slot] = flagged != 0;
        }
    }
    return redo;
}

// Row epilogue of a workgroup of 256 threads, in a launch of its own: the synchronized update of Eq. 2 over the row's
// partial results, each scaled by its own reference r_c -- phi for chunks summed
// with the unified factor, the chunk's largest logit for those whose guard fired or that were recomputed:
//     m = max_c r_c,   out = sum_c e^{r_c-m} num_c / sum_c e^{r_c-m} den_c,
// evaluated in one pass with a running maximum (partial sums are merged by the same
// rule).  For a row without flags every r_c is phi, every factor is exactly 1 and
// the expression IS the plain outer sum of Eq. 4, so one code path serves both.
// Work split: 8 slices of 32 threads; slice k takes chunks k, k+8, ...; a thread
// owns 4 consecutive output elements, so a chunk costs it one 16-byte load of the
// numerator and one of the slot record.  Fixed summation order: no atomics on data,
// same bits on every run.
// Slots [0, n_load) are loaded (all of them hold defined values: chunks without a
// valid key carry zeros), slots [0, nb) enter the result; passing n_load = nc lets
// the loads start before the sequence length is known.
// `scratch` is >= 8 * 128 + 16 floats of LDS.
template <typename NbFn>
__device__ __forceinline__ void row_epilogue(const Problem &p, int row, int n_load, NbFn nb_fn, float *scratch)
{
    const int tid = threadIdx.x;
    const int slice = tid >> 5, t4 = tid & 31;
    const size_t r0 = (size_t)row * p.nc;
    const float *num = p.ws.num + r0 * kHeadDim + 4 * t4;
    const SlotMeta *meta = p.ws.meta + r0;

    // Within a batch of 32 chunks the loads are unconditional and clamped to the last loaded slot (a load
    // inside a divergent branch would force a full wait where the branch rejoins); slots
    // outside the row are masked in the arithmetic.  Two batches are in flight.
    float m = -INFINITY, l = 0.f;
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    int f = 0;
    int nb = 0;
    {
        const int cap = max(n_load - 1, 0);
        auto issue = [&](int c0, auto &nv, auto &mv, auto n) {
#pragma unroll
            for (int i = 0; i < decltype(n)::value; ++i) {
                const int c = min(c0 + 8 * i + slice, cap);
                nv[i] = *reinterpret_cast<const u32x4 *>(num + (size_t)c * kHeadDim);
                mv[i] = *reinterpret_cast<const u32x4 *>(meta + c);
            }
        };
        auto process = [&](int c0, const auto &nv, const auto &mv, auto n) {
            constexpr int N = decltype(n)::value;
            float r[N], bm = -INFINITY;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const bool in_row = c0 + 8 * i + slice < nb;
                r[i] = in_row ? as_f32(mv[i][1]) : -INFINITY;
                bm = fmaxf(bm, r[i]);
                f |= in_row ? (int)mv[i][2] : 0;
            }
            if (bm > m) {                       // rescale what was summed so far (never for unflagged rows)
                const float a = __builtin_amdgcn_exp2f((m - bm) * kLog2e);   // 0 on the first batch
#pragma unroll
                for (int e = 0; e < 4; ++e) s[e] *= a;
                l *= a;
                m = bm;
            }
#pragma unroll
            for (int i = 0; i < N; ++i) {
                // exactly 1 when r_c == m; 0 for slots outside the row (their sums are finite)
                const float a = r[i] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((r[i] - m) * kLog2e);
#pragma unroll
                for (int e = 0; e < 4; ++e) s[e] = __builtin_fmaf(a, as_f32(nv[i][e]), s[e]);
                l = __builtin_fmaf(a, as_f32(mv[i][0]), l);
            }
        };
        constexpr std::integral_constant<int, 4> n{};
        u32x4 nA[4], mA[4], nB[4], mB[4];
        issue(0, nA, mA, n);
        nb = nb_fn();                           // may be a load of its own, in flight with the batch
        for (int c0 = 0; c0 == 0 || c0 < nb; c0 += 64) {      // (no further than the row's last chunk)
            issue(c0 + 32, nB, mB, n);
            process(c0, nA, mA, n);
            issue(c0 + 64, nA, mA, n);
            if (c0 + 32 < nb) process(c0 + 32, nB, mB, n);
        }
    }
    // merge the 8 slices (slice order), divide, round to fp16
    float *S = scratch, *L = scratch + 8 * kHeadDim, *M = L + 8;
    *reinterpret_cast<float4 *>(&S[slice * kHeadDim + 4 * t4]) = make_float4(s[0], s[1], s[2], s[3]);
    if (t4 == 0) { L[slice] = l; M[slice] = m; }
    const int rf = __syncthreads_or(f);
    if (tid < 32) {
        float mm = M[0];
#pragma unroll
        for (int k = 1; k < 8; ++k) mm = fmaxf(mm, M[k]);
        float o[4] = {0.f, 0.f, 0.f, 0.f}, lt = 0.f;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const float a = M[k] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((M[k] - mm) * kLog2e);   // 1 for unflagged rows
            const float4 v = *reinterpret_cast<const float4 *>(&S[k * kHeadDim + 4 * tid]);
            o[0] = __builtin_fmaf(a, v.x, o[0]); o[1] = __builtin_fmaf(a, v.y, o[1]);
            o[2] = __builtin_fmaf(a, v.z, o[2]); o[3] = __builtin_fmaf(a, v.w, o[3]);
            lt = __builtin_fmaf(a, L[k], lt);
        }
        uint2 h = make_uint2(0u, 0u);
        if (nb > 0) {
            h.x = (unsigned)to_half_bits(o[0] / lt) | ((unsigned)to_half_bits(o[1] / lt) << 16);
            h.y = (unsigned)to_half_bits(o[2] / lt) | ((unsigned)to_half_bits(o[3] / lt) << 16);
        }
        *reinterpret_cast<uint2 *>(p.out + (size_t)row * kHeadDim + 4 * tid) = h;
    }
    if (tid == 0) p.ws.row_flags[row] = rf ? 1 : 0;
}

// The row epilogue for the G <= 16 rows of one head group at once, nb <= 16 chunks each (elect_grouped sees to it), by 256
// threads: thread (h, t) = (tid / 32, tid % 32) owns elements 2t, 2t + 1, 64 + 2t and 65 + 2t of row row0 + h (so that a load takes
// whole lines: with 4t .. 4t + 3, two loads of half of every line, the 64 KB of eight rows of 16 chunks took 1.8 us, now 1.6; what one
// compute unit draws past the caches is the bound) and adds
// that row's nb partial results in chunk order, each scaled from its own reference to the maximum of the
// references (Eq. 2; every factor is exactly 1 for an unflagged row, which makes it
// the plain sum of Eq. 4).  No LDS and no barrier, one memory round trip: threads t and 16 + t
// fetch the slot record of chunk t, and all numerators are on their way before the first record is looked at; maximum
// and factors then go round each group of 16 lanes by DPP row operations (through LDS exchanges, five dependent ones for the maximum,
// 0.3 us more).  (Walking records and numerators together, four
// chunks at a time, was one round trip per eight chunks and two loads per chunk and thread: whole call, that form / this,
// 4 x 32/8 heads x 4096 keys 16.2 / 15.4 us, 1 x 32 heads x 1024 keys 7.5 / 7.0.)  Loads pass the caches
// (the partial results come from other workgroups of the same launch).
__device__ __forceinline__ void group_epilogue(const Problem &p, int row0, int G, int nb)
{
    const int tid = threadIdx.x, t4 = tid & 31;
    auto two = [](unsigned long long a, unsigned long long b) {
        return u32x4{(unsigned)a, (unsigned)(a >> 32), (unsigned)b, (unsigned)(b >> 32)};
    };
    for (int h = tid >> 5; h < G; h += (int)(blockDim.x >> 5)) {
        const int row = row0 + h;
        const size_t r0 = (size_t)row * p.nc;
        const float *num = p.ws.num + r0 * kHeadDim + 2 * t4;
        const SlotMeta *meta = p.ws.meta + r0;
        float l = 0.f;
        float s[4] = {0.f, 0.f, 0.f, 0.f};
        int f = 0;
        // a row of up to N <= 16 chunks: its numerators in flight together, lane j of the row's two groups of 16 holds the
        // record of chunk j
        auto block = [&](auto n) {
            constexpr int N = decltype(n)::value;
            const unsigned long long *w = reinterpret_cast<const unsigned long long *>(meta + min(t4 & 15, nb - 1));
            const u32x4 mv = two(load_coherent(&w[0]), load_coherent(&w[1]));
            u32x4 nv[N];
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const unsigned long long *at = reinterpret_cast<const unsigned long long *>(num + (size_t)min(i, nb - 1) * kHeadDim);
                nv[i] = two(load_coherent(at), load_coherent(at + 32));
            }
            const bool in_row = (t4 & 15) < nb;
            const float ref = in_row ? as_f32(mv[1]) : -INFINITY;
            f = in_row ? (int)mv[2] : 0;
            // Where all references agree, in both rows of the wavefront -- no recomputed chunk -- every factor is 1.  (This is in
            // line, as the larger blocks are: a launch runs this part once, and jumps to code not fetched before cost 0.2 us at 8 chunks.)
            const float ref0 = row16_lane<0>(ref);
            if (__builtin_expect(__ballot(in_row & (ref != ref0)) == 0ull, 1)) {
                l = row16_sum(in_row ? as_f32(mv[0]) : 0.f);
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    const unsigned keep = i < nb ? ~0u : 0u;
#pragma unroll
                    for (int e = 0; e < 4; ++e) s[e] += as_f32(nv[i][e] & keep);
                }
                return;
            }
            // exactly 1 where the reference is the maximum; 0 for slots outside the row (their sums are finite)
            const float m = row16_max(ref);
            const float a = ref == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((ref - m) * kLog2e);
            const float ad = a * (in_row ? as_f32(mv[0]) : 0.f);
            each16(std::make_integer_sequence<int, N>{}, [&](auto lane_of) {
                constexpr int i = decltype(lane_of)::value;
                const float ac = row16_lane<i>(a);
                l += row16_lane<i>(ad);
#pragma unroll
                for (int e = 0; e < 4; ++e) s[e] = __builtin_fmaf(ac, as_f32(nv[i][e]), s[e]);
            });
        };
        if (nb > 8) block(std::integral_constant<int, 16>{});
        else if (nb > 4) block(std::integral_constant<int, 8>{});
        else block(std::integral_constant<int, 4>{});
        FD_PHASE(6);
        const unsigned any = (unsigned)(__ballot(f != 0) >> (tid & 32));   // of this row's 32 lanes
        unsigned *out = reinterpret_cast<unsigned *>(p.out + (size_t)row * kHeadDim + 2 * t4);
        out[0] = (unsigned)to_half_bits(s[0] / l) | ((unsigned)to_half_bits(s[1] / l) << 16);
        out[32] = (unsigned)to_half_bits(s[2] / l) | ((unsigned)to_half_bits(s[3] / l) << 16);
        if (t4 == 0) p.ws.row_flags[row] = any ? 1 : 0;
    }
}

// Elects the workgroup that completes a row: a radix-8 tree of arrival counters
// over the row's nb chunks.  Same-address device-scope atomics complete one after
// another (about 0.13 us each on MI355X), so a flat counter costs nb of them on the
// critical path when the workgroups of a row finish together; the tree costs at
// most 8 per level plus one memory round trip per level.  Called by one whole wavefront after the workgroup's results are
// performed; lane 0 counts.  Returns true, uniformly, to exactly one caller per row, after every other chunk arrived.
// Counters are zero before and after (the last arrival at a node resets it).
__device__ __forceinline__ bool arrive_and_elect(const Problem &p, int row, int c, int nb)
{
    constexpr int LR = 3, R = 1 << LR;
    const bool one = (threadIdx.x & 63) == 0;
    int32_t *node = p.ws.ticket + (size_t)row * p.nc;
    int idx = c, n = nb;
    while (n > 1) {
        const int parent = idx >> LR;
        const int children = min(R, n - (parent << LR));
        int t = 0;
        if (one) t = __hip_atomic_fetch_add(&node[parent], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (__builtin_amdgcn_readfirstlane(t) != children - 1) return false;
        if (one) store_coherent(&node[parent], 0);
        n = (n + R - 1) >> LR;
        node += n;
        idx = parent;
    }
    return true;
}

// The row's finish by one wavefront: the rule of row_epilogue, lane l owning elements 2l and 2l + 1.  Up to 32 chunks
// take one memory round trip: lane j fetches the slot record of chunk j, and the numerators of all chunks are on their way before the
// first record is looked at.  Where all references agree -- every row without a recomputed chunk -- every factor is 1 and the chunks
// are simply added (Eq. 4); otherwise each lane has its chunk's factor, which goes round as a scalar.  Fixed order, same
// bits on every run.  Bound by latency: a round trip past the caches and some eighty instructions in a chain.
// COHERENT: the partial results come from other workgroups of the same launch and are read past the caches; false is for a
// launch of its own.
// n_load: slots that hold defined values whatever the row's length (a launch of its own: all nc of them), so that the first
// loads need not wait for the length; nb_of gives the row's chunks and may be a load of its own, in flight with them.
// FLAGS: whether the row flags are written (the synchronized scheme has none).
template <bool COHERENT, bool FLAGS, typename NbFn>
__device__ __forceinline__ void finish_row(const Problem &p, int row, int n_load, NbFn nb_of)
{
    auto ld8 = [](const void *ptr) {
        if constexpr (COHERENT) return load_coherent(static_cast<const unsigned long long *>(ptr));
        else return *static_cast<const unsigned long long *>(ptr);
    };
    const int lane = threadIdx.x & 63;
    const size_t r0 = (size_t)row * p.nc;
    const float *num = p.ws.num + r0 * kHeadDim + 2 * lane;
    const SlotMeta *meta = p.ws.meta + r0;
    float m = -INFINITY, l = 0.f, s[2] = {0.f, 0.f};
    bool any = false;
    int nb = 0;
    auto block = [&](int c0, auto count) {
        constexpr int N = decltype(count)::value;
        const unsigned long long *w = reinterpret_cast<const unsigned long long *>(meta + min(c0 + (lane & (N - 1)), n_load - 1));
        const unsigned long long w0 = ld8(&w[0]), w1 = ld8(&w[1]);
        unsigned long long nv[N];
#pragma unroll
        for (int i = 0; i < N; ++i) nv[i] = ld8(num + (size_t)min(c0 + i, n_load - 1) * kHeadDim);
        if (c0 == 0) nb = nb_of();
        const int left = nb - c0;                            // uniform
        const bool mine = lane < min(N, left);
        const float den = mine ? as_f32((unsigned)w0) : 0.f;
        const float ref = as_f32((unsigned)(w0 >> 32));
        any |= __ballot(mine & ((int)w1 != 0)) != 0ull;
        const float ref0 = as_f32(__builtin_amdgcn_readfirstlane((unsigned)(w0 >> 32)));
        if ((c0 == 0 || m == ref0) && __ballot(mine & (ref != ref0)) == 0ull) {
            m = ref0;
            float d = row16_sum(den);                        // lanes past the row's chunks carry zeros
            if constexpr (N > 16) d = rows_sum(d, d);
            l += as_f32(__builtin_amdgcn_readfirstlane(__builtin_bit_cast(unsigned, d)));
            float t[2][2] = {{s[0], s[1]}, {0.f, 0.f}};      // even and odd chunks: two chains
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const unsigned keep = i < left ? ~0u : 0u;   // (no branch per chunk)
                t[i & 1][0] += as_f32((unsigned)nv[i] & keep);
                t[i & 1][1] += as_f32((unsigned)(nv[i] >> 32) & keep);
            }
            s[0] = t[0][0] + t[1][0];
            s[1] = t[0][1] + t[1][1];
            return;
        }
        // (By DPP.  With six dependent exchanges through LDS, whole call with one recomputed row, those / this: 1 x 32 heads x 2500 keys
        // 16.7 / 16.5 us, 2 x 16 x 3000 18.8 / 18.6, 1 x 40 x 4000 24.9 / 24.8.)
        const float rm = row16_max(mine ? ref : -INFINITY);
        float bm = as_f32(__builtin_amdgcn_readlane(__builtin_bit_cast(unsigned, rm), 0));
        if constexpr (N > 16) bm = fmaxf(bm, as_f32(__builtin_amdgcn_readlane(__builtin_bit_cast(unsigned, rm), 16)));
        if (bm > m) {                                        // rescale what was summed so far
            const float a = __builtin_amdgcn_exp2f((m - bm) * kLog2e);   // 0 on the first block
            s[0] *= a;
            s[1] *= a;
            l *= a;
            m = bm;
        }
        // exactly 1 when ref == m
        const float a = ref == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((ref - m) * kLog2e);
        const float ad = a * den;
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (i < left) {
                const float ac = as_f32(__builtin_amdgcn_readlane(__builtin_bit_cast(unsigned, a), i));
                l += as_f32(__builtin_amdgcn_readlane(__builtin_bit_cast(unsigned, ad), i));
                s[0] = __builtin_fmaf(ac, as_f32((unsigned)nv[i]), s[0]);
                s[1] = __builtin_fmaf(ac, as_f32((unsigned)(nv[i] >> 32)), s[1]);
            }
    };
    if (n_load <= 4) block(0, std::integral_constant<int, 4>{});
    else if (n_load <= 8) block(0, std::integral_constant<int, 8>{});
    else if (n_load <= 16) block(0, std::integral_constant<int, 16>{});
    else
        for (int c0 = 0; c0 == 0 || c0 < nb; c0 += 32) block(c0, std::integral_constant<int, 32>{});
    FD_PHASE(6);
    unsigned o = 0u;                                         // an empty sequence: zeros, no flag
    if (nb > 0) o = (unsigned)to_half_bits(s[0] / l) | ((unsigned)to_half_bits(s[1] / l) << 16);
    *reinterpret_cast<unsigned *>(p.out + (size_t)row * kHeadDim + 2 * lane) = o;
    if (FLAGS && lane == 0) p.ws.row_flags[row] = any ? 1 : 0;
}

}  // namespace fd
